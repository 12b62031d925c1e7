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

// Passes over a queue of runnable short collectives: each hands the movers gangs of up to `most` of them until its bytes are spent.
static void gangs() {
  for (uint32_t focus : {1u, 4096u, 20000u, 32u << 10, 128u << 10, 0x80000000u, 0xffffffffu})
   for (bool priority : {false, true}) {
    const uint32_t budget = gang_budget(focus, priority);
    EXPECT(budget >= focus && budget / 2u <= focus && (!priority || budget == focus), "focus %u: %u", focus, budget);
    for (uint32_t most : {1u, 2u, 8u, 16u})
      for (uint32_t step = 0; step < 40; ++step) {
        std::vector<uint32_t> share;
        for (uint32_t i = 0; i < 64; ++i) share.push_back(16u + (i * 7919u * (step + 1u)) % (16u << 10) / 16u * 16u);
        uint32_t passes = 0;
        for (size_t at = 0; at < share.size(); ++passes) {
          uint32_t spent = 0, went = 0;
          for (bool full = false; at < share.size() && spent < focus && !full; ) {
            const uint32_t first = spent;                  // (the gang: one job)
            for (uint32_t n = 0; n < most && at < share.size(); ++n) {
              if (!gang_takes(spent, share[at], budget)) { full = true; break; }
              spent += share[at++]; ++went;
            }
            EXPECT(spent <= budget || (first == 0 && went == 1), "budget %u, gangs of %u: %u bytes handed to the movers", budget, most, spent);
          }
          EXPECT(went > 0, "budget %u: a pass without a job", budget);
          if (!went) return;
        }
      }
   }
}

// A workgroup's queue under steady traffic: as many short collectives as there are outstanding come back to its tail as soon as they have gone, and a
// long one, or one that only has its completion left, waits among them.
static void turns() {
  for (uint32_t nshort : {9u, 20u, 40u})
    for (uint32_t share : {2048u, 16384u})
      for (uint64_t done : {0ull, 1ull, 5ull, 1ull << 40})
        for (uint32_t stuck : {0u, 1u, 5u}) {      // others that look runnable, are further along, and are given up at every visit
          struct Q { bool is_short; uint64_t done; bool stuck; };
          std::vector<Q> q(nshort, Q{true, 0, false});
          for (uint32_t i = 0; i < stuck; ++i) q.push_back(Q{false, done + 1u, true});
          q.push_back(Q{false, done, false});
          bool went = false;
          uint32_t passes = 0, behind = 0, turns_had = 0;
          for (; passes < 1000 && !went; ++passes) {
            const uint32_t n = (uint32_t)q.size(), others = stuck + 1u;
            std::vector<uint32_t> order(n, 0);
            for (uint32_t i = 0; i < n; ++i) {
              uint32_t at = 0;
              for (uint32_t k = 0; k < n; ++k) at += pass_key(q[k].is_short, q[k].done, k) > pass_key(q[i].is_short, q[i].done, i);
              order[at] = i;
            }
            uint32_t bytes = 0, rk = 0;
            std::vector<bool> gone(n, false);
            auto visit = [&](uint32_t i) {
              if (q[i].stuck) return;
              gone[i] = true;
              bytes += share;
              went = went || !q[i].is_short;
            };
            for (; rk < n && bytes < (128u << 10); ++rk) visit(order[rk]);
            if (turn_due(behind)) {
              const uint32_t at = nshort + turn_of(turns_had++, others);
              EXPECT(at < n && !q[order[at]].is_short, "the turn is none of the others'");
              if (rk <= at && at < n) visit(order[at]);
            }
            behind = passes_over(behind, others, n - rk);
            EXPECT(behind <= PASSES_OVER, "%u passes in a row", behind);
            std::vector<Q> next;
            uint32_t came = 0;
            for (uint32_t i = 0; i < n; ++i) if (gone[i]) ++came; else next.push_back(q[i]);
            for (uint32_t i = 0; i < came; ++i) next.push_back(Q{true, 0, false});
            q = next;
          }
          const uint32_t bound = (PASSES_OVER + 1u) * (stuck + 1u);
          EXPECT(went && passes <= bound, "%u short ones of %u bytes, %llu steps done, %u that are given up: not visited in %u passes", nshort, share, (unsigned long long)done, stuck, bound);
        }
}

// A fetch that goes on reads slots through a resource of sq_depth slots: its size and the offset of every 16-byte part, in 32 bits.
static void rings() {
  const uint32_t slot = 128;
  for (uint32_t sh = 1; sh < 32; ++sh) {
    const uint32_t depth = 1u << sh;
    if (!run_goes_on(depth, slot)) { EXPECT(sh > 24, "a ring of 2^%u slots: refused", sh); continue; }
    const uint32_t size = depth * slot;
    for (uint64_t idx : {0ull, (1ull << sh) - 1u, (1ull << sh), 3ull * (1ull << sh) - 1u, 1ull << 40}) {
      const uint32_t at = ((uint32_t)idx & (depth - 1u)) * slot + 80u;
      EXPECT((uint64_t)at == (idx & ((1ull << sh) - 1u)) * slot + 80u && at + 16u <= size, "a ring of 2^%u slots, entry %llu: at %u of %u", sh, (unsigned long long)idx, at, size);
    }
  }
}

int main(int argc, char** argv) {
  const struct { const char* name; void (*run)(); } models[] = {{"tables", tables}, {"gangs", gangs}, {"turns", turns}, {"rings", rings}};
  bool any = false;
  for (const auto& m : models)
    if (argc < 2 || !strcmp(argv[1], m.name)) { m.run(); any = true; }
  if (!any) { printf("no such model\n"); return 2; }
  return bad ? 1 : 0;
}
