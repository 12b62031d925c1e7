// Rules of the scheduler that stand on their own: pure functions of their arguments, compiled for the device (the kernel) and for the
// host (tests/rules/rules_check.cpp walks them without a GPU).
#ifndef DFX_RULES_H
#define DFX_RULES_H

#include <stdint.h>

#if defined(__HIPCC__)
#define DFX_RULE __host__ __device__ __forceinline__
#else
#define DFX_RULE inline
#endif

// The table of buffers that came with a lone entry (DfxPeer) stays in LDS for the further jobs of that invocation: held_of is its
// collective + 1 (0 = no table), held_seq the invocation.  The id alone does not say whose buffers they are: a fetch that goes on behind its
// first 64 entries may take the next invocation of the same collective, with buffers of its own, while the table of the one before,
// whose only job went to the movers at the head of the fetch, still lies there.
DFX_RULE bool table_serves(uint32_t held_of, uint32_t held_seq, uint32_t coll, uint32_t seq) { return held_of == coll + 1u && held_seq == seq; }

// Whether a fetch may go on behind its first 64 entries, which it reads through a buffer resource: sizes and offsets of that are 32 bits, so
// the ring (a power of two of slots) must be shorter.  (From 2^25 slots on its size read as 0 and every entry as nobody's.)
DFX_RULE bool run_goes_on(uint32_t sq_depth, uint32_t slot_bytes) { return (uint64_t)sq_depth * slot_bytes <= 0x80000000u; }

// Whether another short collective goes with the gang in hand: spent, the bytes that the pass has handed to the movers, those of the gang's
// members so far among them; share, its own; budget, gang_budget.  A gang is one job that nothing overtakes, so a budget holds inside it as
// well; the first member of a pass always goes.
DFX_RULE bool gang_takes(uint32_t spent, uint32_t share, uint32_t budget) { return spent == 0 || (uint64_t)spent + share <= budget; }
// A pass hands the movers focus bytes before the SQ and the queue are looked at again (under priority ordering 32 KiB at most, and that is a
// promise to urgent collectives).  Under FIFO ordering a gang may take twice as much, which is a whole one of sixteen shares of 16 KiB by
// default: sixty all-reduces of 2 MiB on four ranks 397 us, with once as much 443, of 1 MiB on two ranks 272 and 300 (eight ranks, whose gangs
// are of eight, level).
DFX_RULE uint32_t gang_budget(uint32_t focus, bool priority) { return priority || focus > 0x7fffffffu ? focus : 2u * focus; }

// Order of a focused pass under FIFO ordering, largest key first: the short ones that may go in gangs, then the others, of each furthest along
// first, then queue order.
DFX_RULE uint32_t pass_key(bool short_one, uint64_t done, uint32_t lane) {
  return ((short_one ? 1u << 28 : 0u) | ((uint32_t)(done > 0xfffffu ? 0xfffffu : done) << 8) | (63u - lane)) + 1u;
}
// A pass ends when its bytes are spent, and as long as short ones keep coming they alone may spend them.  Behind seven passes in a row that
// left others unvisited comes one in which one of these has its turn whatever the short ones have spent.  (Without turns an all-reduce of
// 25 MiB was not complete when 5000 of 128 KiB that came behind it were, forty of them outstanding on its channel; 48 without gangs.)  A turn
// is one visit: with every eighth pass in plain order instead, where long ones part the gangs, 64 mixed collectives took 944 us, without turns 939.
constexpr uint32_t PASSES_OVER = 7u;
DFX_RULE bool turn_due(uint32_t over) { return over >= PASSES_OVER; }
// Which of the others, by the turns there have been: each in its turn, since the first may be a last wait that looks over on this workgroup's
// channel and is not on another one, whose job waits for its own turn behind a wait like it.
DFX_RULE uint32_t turn_of(uint32_t turns, uint32_t others) { return others ? turns % others : 0u; }
// The passes in a row, behind one more: others, its runnable entries behind short ones; left, its entries that were not visited.
DFX_RULE uint32_t passes_over(uint32_t over, uint32_t others, uint32_t left) { return !turn_due(over) && others != 0 && left != 0 ? over + 1u : 0u; }

#endif
