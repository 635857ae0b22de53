// A context's captured chunks of iterations, by the key of everything their kernels receive.
//
// One solve replays up to four graphs: the mixed solver's FP64 and FP32 chunks, each without
// and, once an iteration has paused for the explicit Gram, with the fallback launches. With
// room for all of them the next equal solve captures none; a single slot would capture every
// one of them in every solve. Host code only.
#pragma once

#include <string>

template <typename Graph>
class GraphCache {
 public:
  static constexpr int kSlots = 4;
  struct Slot {
    std::string key;
    Graph graph = nullptr;
    long used = 0;
  };

  // the graph of this key, or NULL
  Graph find(const std::string& key) {
    for (Slot& s : slots_)
      if (s.graph && s.key == key) {
        s.used = ++tick_;
        return s.graph;
      }
    return nullptr;
  }
  // The slot of a new graph: an empty one, else the one used longest ago, whose graph the
  // caller destroys. Marked as just used.
  Slot& place() {
    Slot* v = &slots_[0];
    for (Slot& s : slots_) {
      if (!s.graph) {
        v = &s;
        break;
      }
      if (s.used < v->used) v = &s;
    }
    v->used = ++tick_;
    return *v;
  }
  template <typename Destroy>
  void clear(Destroy destroy) {
    for (Slot& s : slots_) {
      if (s.graph) destroy(s.graph);
      s = Slot();
    }
  }

 private:
  Slot slots_[kSlots];
  long tick_ = 0;
};
