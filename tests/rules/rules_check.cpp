// Walks the scheduler's rules (csrc/dfx_rules.h, the functions that the kernel compiles) through small models of what the kernel does
// with them.  Prints a line per violation; `rules_check NAME` runs one model.
#include <stdio.h>
#include <string.h>

#include <vector>

#include "../../paper_2303_06324_amd/csrc/dfx_rules.h"

static int bad = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { printf("line %d: ", __LINE__); printf(__VA_ARGS__); printf("\n"); ++bad; } } while (0)

// A workgroup's fetches, the step that goes to the movers straight from a lone entry, and later visits of queued ones.  An entry's
// buffers stand for the invocation that they belong to.
struct Entry { uint32_t coll, seq, buffers; bool table; };
struct Workgroup {
  uint32_t held_of = 0, held_seq = 0, held = 0;
  std::vector<Entry> queue;
  std::vector<uint32_t> moved;                       // buffers of the jobs posted, in turn
  void head(const Entry& e, bool lone, bool at_once, uint32_t jobs) {      // the first 64 entries of a fetch, one of them this workgroup's
    held_of = 0;
    if (lone && e.table) {
      held_of = e.coll + 1u; held_seq = e.seq; held = e.buffers;
      if (at_once) { moved.push_back(e.buffers); if (jobs == 1) return; }      // (through: no place in the queue)
    }
    queue.push_back(e);
  }
  void behind(const Entry& e) { queue.push_back(e); }      // ... and the entries behind them
  void visit() {
    for (const Entry& e : queue)                     // without the table: what the ranks have published for the invocation
      moved.push_back(table_serves(held_of, held_seq, e.coll, e.seq) ? held : e.buffers);
    queue.clear();
  }
};

static void tables() {
  for (uint32_t seq : {0u, 7u, 0x7fffffffu, 0xffffffffu})
    for (uint32_t coll : {0u, 5u, 4095u})
      for (bool at_once : {false, true})
        for (uint32_t jobs : {1u, 3u}) {
          Workgroup w;
          const Entry first{coll, seq, 100, true}, other{coll ^ 1u, seq, 200, false}, again{coll, seq + 1u, 300, false};
          w.head(first, true, at_once, jobs);
          w.behind(other);
          const bool through = at_once && jobs == 1;
          if (through) w.behind(again);              // completed by the others meanwhile, and submitted anew with other buffers
          w.visit();
          std::vector<uint32_t> want;
          if (at_once) want.push_back(100);
          if (!through) want.push_back(100);
          want.push_back(200);
          if (through) want.push_back(300);
          EXPECT(w.moved == want, "collective %u, invocation %u, at once %d, %u jobs: a job moves another invocation's buffers", coll, seq, at_once, jobs);
        }
}

int main(int argc, char** argv) {
  const struct { const char* name; void (*run)(); } models[] = {{"tables", tables}};
  bool any = false;
  for (const auto& m : models)
    if (argc < 2 || !strcmp(argv[1], m.name)) { m.run(); any = true; }
  if (!any) { printf("no such model\n"); return 2; }
  return bad ? 1 : 0;
}
