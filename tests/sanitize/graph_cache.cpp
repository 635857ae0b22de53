// GraphCache on the host: which chunks a sequence of solves captures, and that every graph
// that loses its place is destroyed once. Graphs are numbers here.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <set>

#include "../../paper_1808_01829_amd/csrc/graph_cache.h"

#define CHECK(x)                                      \
  do {                                                \
    if (!(x)) {                                       \
      printf("line %d: %s\n", __LINE__, #x);          \
      exit(1);                                        \
    }                                                 \
  } while (0)

static GraphCache<int*> cache;
static std::set<int*> alive;
static int captured = 0;

static void destroy(int* g) {
  CHECK(alive.erase(g) == 1);
  delete g;
}

// what a solve does for each of its chunks
static int run(std::initializer_list<const char*> keys) {
  captured = 0;
  for (const char* k : keys) {
    int* g = cache.find(k);
    if (!g) {
      auto& s = cache.place();
      if (s.graph) {
        destroy(s.graph);
        s.graph = nullptr;
      }
      g = new int(0);
      alive.insert(g);
      s.graph = g;
      s.key = k;
      ++captured;
    }
    CHECK(alive.count(g) == 1 && cache.find(k) == g);
  }
  return captured;
}

int main() {
  // an FP64 solve that pauses, twice; then a mixed one, twice
  CHECK(run({"f64", "f64+", "f64+"}) == 2);
  CHECK(run({"f64", "f64+", "f64+"}) == 0);
  CHECK(run({"f64", "f64+", "f32", "f32", "f32+"}) == 2);
  CHECK(run({"f64", "f64+", "f32", "f32", "f32+"}) == 0);
  // full: the one used longest ago goes
  CHECK(alive.size() == 4);
  CHECK(run({"f64", "f32", "other"}) == 1);
  CHECK(run({"f64", "f32", "f32+", "other"}) == 0);
  CHECK(run({"f64+"}) == 1 && run({"f64"}) == 1);
  CHECK(alive.size() == 4);
  // an emptied slot (a capture that failed) is the next one taken
  auto& s = cache.place();
  if (s.graph) destroy(s.graph);
  s.graph = nullptr;
  CHECK(alive.size() == 3 && run({"again"}) == 1 && alive.size() == 4);
  cache.clear(destroy);
  CHECK(alive.empty() && !cache.find("f64") && run({"f64"}) == 1);
  cache.clear(destroy);
  CHECK(alive.empty());
  printf("ok\n");
  return 0;
}
