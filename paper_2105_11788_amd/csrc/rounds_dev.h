// The refinement loop of Algorithm 3 (section 4) by one workgroup, with the
// iterations that split nothing decided ahead of their turn.
//
// An iteration picks the smallest unstable label C, and most of them split
// nothing (about 85-95 % on the generated LTSs).  That verdict keeps: if no
// block holds two states with different marks under C, then no refinement of
// those blocks does either, so it stands until C itself loses a member.  A
// round therefore takes the next labels that are unstable and have no verdict
// (up to kCand, in label order), marks all of them side by side in one hash
// table keyed by (candidate, source), and checks every touched block against
// its leader.  Labels found stable lose their bit in Q (unstable, no verdict)
// and keep their bit in U (unstable).  When the smallest label left in Q
// splits something, every label of U before it is an iteration without a
// split (counted, bit cleared), and its own iteration is carried out from the
// marks the table already holds.  The splitter sequence, the partitions and
// the iteration count are those of the lock-step loop.
//
// Why a workgroup and not the grid: an iteration is a chain of dependent
// steps over a few hundred transitions.  A barrier costs well under 0.1 us in
// a workgroup and 2.5-3 us as a kernel boundary, and with the verdicts taken
// side by side one CU has enough lanes for a round's transitions.
//
// A large block is marked again and again because single states leave it.
// Such a label is tracked: the partition is known to be stable under a set B
// of states that was the block (when it was last found stable, or after an
// iteration of its own that left no block with two different marks), and the
// states that have left since are listed.  Under the block as it is now, a
// state's marks can differ from its marks under B only if it has a transition
// to a listed state, so only those sources are visited; their outgoing
// transitions tell which marks they lost, and two states of a block have equal
// marks iff they lost the same ones.  The table then holds the lost marks in
// place of the marks, and the rest of the round is the same.  (Uniform LTS of
// 300k states 1,290 -> 929 ms, chain of 100k 2,640 -> 816, 48 instances of up
// to 200k states in a batch 1,014 -> 500; with the shorter rounds 840, 660 and
// 430.)
//
// Bound: the chain of a round's dependent steps, about 7.5 us when something
// splits (uniform LTS of 20k states, 3,464 rounds for 27,089 iterations):
// members 1.0, transitions 1.3, comparison 1.0, verdicts 0.3, split list 0.9,
// split 0.5 + 1.0, and the next round's candidates beside the moves 1.7.  A
// trip to the L2 is about 0.2 of these, to LDS 0.06, and waves that have
// nothing to do still take issue slots, so a step's loads are issued together,
// searches are bit counts of start bitmaps, values that all lanes agree on go
// through scalar registers, and sums over the workgroup are skipped while one
// wave holds the members.  Against two grid-wide kernels per iteration: uniform
// LTS of 20k states 232 -> 25 ms, Kripke structure of 1000 states 14.6 -> 2.2 ms,
// 25k states with as many actions as transitions 134 -> 5.5 ms, planted quotient
// of 1.03M states 746 -> 283 ms (load and read-back included).
//
// The partition is a refinable partition: perm lists the states block by
// block, block b (a label, its smallest member) owns perm[bs[b] .. be[b]),
// and pin[p] is the in-transition range of perm[p].  A split moves the
// split-off states to the tail of the range.  Up to 256 split states go
// through tables in LDS; more of them through lists in global memory, whose
// counters per block are added to once per wave (one atomic per state queued
// at 10 ns each); and a block whose leader was touched and that has 256
// untouched members or more is relabelled as a whole (backward chain of 3,000
// states 210 -> 25 ms, of 40,000 19.5 -> 0.49 s).
#pragma once

#include <stdint.h>

#include "internal.h"

namespace bisim {

constexpr uint32_t kCand = 32;       // candidates per round (at most a wave's lanes)
constexpr uint32_t kKeyBits = 27;    // state bits of a table key
constexpr uint32_t kRoundsMaxN = (1u << kKeyBits) - 1;  // so that no key is kNone
constexpr uint32_t kTracked = 64;    // labels tracked at a time
constexpr uint32_t kLost = 64;       // states a tracked block can have lost
// In-transitions from which a label is tracked: below, marking the whole block
// costs a round no more than the visits of its lost states' sources (2.5 us).
// While the mark words of all states fit LDS, marking a whole block is cheaper
// (3 us and a table to clear for 5000 transitions) and the line lies higher
// (chains of 1000 / 5000 / 15000 states: never tracked 7.9 / 41.5 / 189 ms,
// from 1536 on 7.9 / 34.3 / 102).  It starts there once kTrackAfter whole
// blocks were marked and stops when no block is as large: a round with tracking
// costs 5-15 % more, which a large block that is hardly ever a splitter does
// not repay.  For the same reason the loop is compiled with and without
// tracking (product of 20,736 states 48.0 / 51.9 ms, 25k states with as many
// actions as transitions 4.8 / 5.7), and a run changes from one to the other.
constexpr uint32_t kTrackEdges = 384, kTrackEdgesDense = 1536;
constexpr uint32_t kTrackAfter = 8;
constexpr uint32_t kTrackLook = 256;  // rounds between two looks at the largest block
// outgoing transitions in flight per thread (the batched kernel: as its
// registers allow)
template <class MaskT, int kMode, bool kBm>
constexpr uint32_t out_u() { return kMode != 2 ? 8 : sizeof(MaskT) == 4 && kBm ? 6 : 2; }
constexpr uint32_t kListCap = 64;    // listed blocks kept in LDS
constexpr uint32_t kWideCap = 8;     // blocks split by what stays, at a time
// members of such blocks from which the iteration is the grid's
constexpr uint32_t kGridMembers = 1u << 18;
constexpr uint32_t kOwnBlock = 128;  // members up to which a wave takes a listed block alone
constexpr uint32_t kScanU = 2;       // states or transitions in flight per thread
// members of a wide block in flight per thread
template <int kMode, bool kBm>
constexpr uint32_t wide_u() { return kMode == 2 && !kBm ? 2 : 4; }
// transitions per thread and round
template <int WG>
constexpr uint32_t edges_per_thread() { return WG >= 512 ? 2 : 4; }
// split states that are moved by the tables in LDS (one per thread)
template <int WG>
constexpr uint32_t small_split() { return WG < 256 ? WG : 256; }

// results of rounds_loop
constexpr uint32_t kRoundsDone = 0, kRoundsGrid = 1, kRoundsBad = 2, kRoundsCap = 3;
constexpr uint32_t kRoundsTrack = 4;  // go on in the loop with (or again without) tracking
constexpr uint32_t kRoundsGo = 5;  // (inside: the next round)

// One instance; per-state arrays start at its first state, state ids in
// in_src are shifted by s0.
template <class MaskT>
struct RoundsArgs {
  uint32_t n, s0;
  uint32_t iter_cap;
  uint32_t rcpp;        // Algorithm 2: one mark per state, C not re-marked
  uint32_t grid_edges;  // estimated in-transitions from which a splitter is left to the grid (0: never)
  uint32_t grid_dense;  // the same while the mark words of all states fit LDS
  uint32_t mean_deg;    // mean in-degree, rounded up
  const uint32_t* in_ptr;
  const int32_t *in_src, *in_ord;
  int32_t *blk, *perm, *pos, *bs, *be;
  uint64_t* pin;
  // used by splitters beyond the table, and by splits of more than WG states
  MaskT* mw;                              // zero between iterations
  int32_t *cnt, *fc, *gc;                 // zero between iterations
  uint64_t *nlb, *tmp64;
  int32_t *ts, *tb;                       // touched states and their blocks
  int32_t *lb, *llo, *lsz;                // listed blocks and their ranges
  int32_t *ss, *sbk, *sr, *sfi, *sps;
  // transitions by source, and per label its entry among the tracked ones plus
  // one (0: not tracked); null: no tracking
  uint32_t* out_ptr;
  int32_t *out_dst, *out_ord;
  uint32_t* out_cur;   // [n], 0 when not in use: the workgroup lays them out, if it
                       // tracks (null: they are there)
  uint8_t* trk;
  uint32_t* trk_save;  // [kTrackSave] between launches of one run (nullable)
  // bitmaps over labels and their summaries (bit w set iff word w is not 0)
  uint64_t *ub, *qb, *us, *qs;
};

// Work totals of a run, in LDS (kEither only: the others' callers read none):
// members and transitions of the labels marked, (label, source) pairs, blocks
// with untouched members and their members, split states, new blocks.
constexpr int kWMembers = 0, kWEdges = 1, kWTouched = 2, kWListed = 3, kWVisits = 4, kWSplit = 5,
              kWBlocks = 6, kWorkTotals = 7;

// What the grid did between two launches of one run: the iteration of `label`
// (kNone: none), the split states it listed, and whether the split part of
// some block holds different marks.
struct RoundsResume {
  uint32_t label = kNone, nS = 0, mixed = 0;
  uint32_t nbig = 0;       // whole blocks marked since the last look at the largest
  bool may_track = false;  // the loop without tracking may end for it
  bool lay_out = false;    // the transitions by source are to be laid out
};

template <int WG>
struct RoundsShared {
  uint32_t cand[kCand], cb[kCand], cpre[kCand], cend[kCand], unst[kCand];
  uint32_t ctrk[kCand];  // tracked entry of the candidate plus one
  uint32_t cbeg[kCand];  // its first transition of the round's (cend: past its last)
  uint32_t wl[kWave];    // words of Q
  // the candidates with members, in order: first member (and, after the last,
  // their number), first position, candidate, tracked entry to visit plus one
  uint32_t rfirst[kCand + 1], rb[kCand], rc[kCand], rtrk[kCand];
  uint64_t cstarts[WG / kWave];  // bit i: member i is the first of a candidate
  uint32_t tn[kTracked], tlabel[kTracked];  // tracked labels: lost states, label
  uint32_t wsum[WG / kWave], wnz[WG / kWave];
  // the members with in-transitions (mbeg, mpre, mc), and bit e: transition e
  // of the round is the first of one
  uint64_t starts[edges_per_thread<WG>() * WG / kWave];
  unsigned long long work[kWorkTotals];
  uint32_t mbeg[WG], mpre[WG];
  uint8_t mc[WG];
  int32_t ss[small_split<WG>()], sb[small_split<WG>()];  // the first split states and their blocks
  uint32_t lb[kListCap], llo[kListCap], lsz[kListCap];   // the first listed blocks
  // blocks whose touched leader has kSmall untouched members or more:
  // candidate, block, first position, members
  uint32_t wc[kWideCap], wb[kWideCap], wlo[kWideCap], wsz[kWideCap];
  uint32_t nW;                      // such blocks found
  uint32_t wmin, wstay, wfront, wback;  // of the one at hand
  uint32_t nc, np, mtot, etot, csz0, nT, tctr, bad;
  union {
    unsigned long long nSL;
    struct {
      uint32_t nS, nL;  // split states, listed blocks
    };
  };
  uint32_t inc;              // candidates visited through their lost states
  uint32_t tnext;            // next tracked entry to take
  uint32_t fent, ffresh;     // the splitter's entry plus one; taken in this round
  uint32_t fold;             // lost states its entry already had
  uint32_t most;             // members of the largest block
  uint32_t nbig;             // whole blocks marked, for the next launch
  uint32_t mixed, nself;     // a split part with different marks; split states of C itself
  uint32_t it;  // iterations so far
};

// a value that is the same on every lane, as a scalar
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// lane l's value (l the same on every lane), without a trip through the LDS unit
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, uint32_t l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, uint32_t l) {
  return (uint64_t)lane_u32((uint32_t)(v >> 32), l) << 32 | lane_u32((uint32_t)v, l);
}
// set bits of v below this lane's position
__device__ __forceinline__ uint32_t bits_below(uint64_t v) {
  return (uint32_t)__builtin_amdgcn_mbcnt_hi(
      (uint32_t)(v >> 32), (uint32_t)__builtin_amdgcn_mbcnt_lo((uint32_t)v, 0u));
}
// LDS writes of the wave's lanes before are seen by its lanes after
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <class MaskT>
__device__ __forceinline__ MaskT mask_or(MaskT* p, MaskT v);
template <>
__device__ __forceinline__ uint32_t mask_or<uint32_t>(uint32_t* p, uint32_t v) {
  return atomicOr(p, v);
}
template <>
__device__ __forceinline__ uint64_t mask_or<uint64_t>(uint64_t* p, uint64_t v) {
  return atomicOr((unsigned long long*)p, (unsigned long long)v);
}

template <class MaskT>
__device__ __forceinline__ void mask_and(MaskT* p, MaskT v) {
  if (sizeof(MaskT) == 4) atomicAnd((unsigned int*)p, (unsigned int)v);
  else atomicAnd((unsigned long long*)p, (unsigned long long)v);
}

__device__ __forceinline__ uint32_t table_hash(uint32_t key, uint32_t shift) {
  return (key * 2654435761u) >> shift;
}
// slot of key, inserted if absent (first: by this call).  The table is never
// more than half full, so the probe ends.
__device__ __forceinline__ uint32_t table_insert(uint32_t* tab, uint32_t mask, uint32_t shift,
                                                 uint32_t key, bool& first) {
  uint32_t h = table_hash(key, shift);
  for (;;) {
    const uint32_t old = atomicCAS(&tab[h], kNone, key);
    first = old == kNone;
    if (first || old == key) return h;
    h = (h + 1) & mask;
  }
}
// slot of key, kNone if absent
__device__ __forceinline__ uint32_t table_find(const uint32_t* tab, uint32_t mask, uint32_t shift,
                                               uint32_t key) {
  uint32_t h = table_hash(key, shift);
  for (;;) {
    const uint32_t v = tab[h];
    if (v == key) return h;
    if (v == kNone) return kNone;
    h = (h + 1) & mask;
  }
}

// Append one entry per lane with pred (one atomic per wave); the entry's
// index, kNone without pred.  Wave-uniform call.
__device__ __forceinline__ uint32_t list_push(uint32_t* counter, bool pred) {
  const uint64_t bal = __ballot(pred);
  if (!bal) return kNone;
  const int leader = __ffsll((unsigned long long)bal) - 1;
  uint32_t base = 0;
  if ((int)lane() == leader) base = atomicAdd(counter, (uint32_t)__popcll(bal));
  base = lane_u32(base, (uint32_t)leader);
  return pred ? base + bits_below(bal) : kNone;
}

// Lanes with equal keys: for the first few keys of the wave, the lane that
// speaks for this one, how many it speaks for, and how many of them are below
// (every other lane speaks for itself).  Wave-uniform call.
struct Group {
  uint32_t lead, count, below;
};
template <int kKeys = 4>
__device__ __forceinline__ Group group_of(uint32_t key, bool on) {
  Group g{lane(), on ? 1u : 0u, 0u};
  uint64_t todo = __ballot(on);
  for (int k = 0; k < kKeys && todo; ++k) {
    const uint32_t l = (uint32_t)(__ffsll((unsigned long long)todo) - 1);
    const uint32_t first = lane_u32(key, l);
    const bool mine = on && key == first;
    const uint64_t same = __ballot(mine);
    todo &= ~same;
    if (__popcll(same) == 1) break;  // (keys that differ mostly differ all)
    if (mine) g = {l, (uint32_t)__popcll(same), bits_below(same)};
  }
  return g;
}
// counter[key] += 1 per lane with `on`, by one atomic per group (the counter of
// a large block otherwise takes 10 ns per state): the value before, on the
// lanes that lead.  rank_in: the value before each lane's (wave-uniform call).
__device__ __forceinline__ int32_t add_group(int32_t* counter, uint32_t key, bool on,
                                             const Group& g) {
  int32_t base = 0;
  if (on && lane() == g.lead) base = atomicAdd(&counter[key], (int32_t)g.count);
  return base;
}
__device__ __forceinline__ int32_t rank_in(int32_t base, const Group& g) {
  return (int32_t)__shfl(base, (int)g.lead, kWave) + (int32_t)g.below;
}
__device__ __forceinline__ int32_t add_one(int32_t* counter, uint32_t key, bool on,
                                           const Group& g) {
  return rank_in(add_group(counter, key, on, g), g);
}
// word[key] = max(word[key], epoch | kNone - s) per lane with `on`, by one
// atomic per group.  Wave-uniform call.
__device__ __forceinline__ void bid_min(uint64_t* word, uint32_t key, uint64_t epoch, uint32_t s,
                                        bool on, const Group& g) {
  uint64_t leads = __ballot(on && lane() == g.lead && g.count > 1);
  while (leads) {
    const uint32_t l = (uint32_t)(__ffsll((unsigned long long)leads) - 1);
    leads &= leads - 1;
    const bool mine = on && g.lead == l;
    const uint32_t least = wave_min_u32(mine ? s : kNone);
    if (mine) s = least;
  }
  if (on && lane() == g.lead)
    atomicMax((unsigned long long*)&word[key],
              (unsigned long long)(epoch | (uint64_t)(kNone - s)));
}

// entry i of the split list and of the list of blocks: in LDS, beyond its
// capacity in global memory
template <class A, class S, class M>
__device__ __forceinline__ void put_split(const A& a, S& sh, M* marks, uint32_t cap, uint32_t i,
                                          int32_t s, int32_t b, M mv) {
  if (i < cap) {
    sh.ss[i] = s;
    sh.sb[i] = b;
    if (marks) marks[i] = mv;
  } else {
    a.ss[i] = s;
    a.sbk[i] = b;
  }
}
template <class A, class S>
__device__ __forceinline__ void put_block(const A& a, S& sh, uint32_t i, uint32_t b, uint32_t lo,
                                          uint32_t sz) {
  if (i < kListCap) {
    sh.lb[i] = b;
    sh.llo[i] = lo;
    sh.lsz[i] = sz;
  } else {
    a.lb[i] = (int32_t)b;
    a.llo[i] = (int32_t)lo;
    a.lsz[i] = (int32_t)sz;
  }
}

// Lane l holds the set v of items 64 id .. 64 id + 63: the items of all lanes
// in lane order to out[0 .. lim), one wave; their number (not capped).  A lane
// writes its own items where it has few; of a lane with many, every lane of
// the wave takes one (both are a few steps: of the latter there are at most
// lim / 5).
__device__ __forceinline__ uint32_t expand_bits(uint64_t v, uint32_t id, uint32_t* out,
                                                uint32_t lim) {
  constexpr uint32_t kFew = 4;
  const uint32_t pc = (uint32_t)__popcll(v);
  const uint32_t incl = wave_incl_scan_u32(pc);
  const uint32_t total = lane_u32(incl, kWave - 1);
  const uint32_t at = incl - pc;
  uint64_t many = __ballot(pc > kFew && at < lim);
  if (pc <= kFew) {
    uint64_t x = v;
    for (uint32_t k = at; x && k < lim; ++k, x &= x - 1)
      out[k] = (id << 6) + (uint32_t)(__ffsll((unsigned long long)x) - 1);
  }
  while (many) {
    const uint32_t o = (uint32_t)(__ffsll((unsigned long long)many) - 1);
    many &= many - 1;
    const uint64_t w = lane_u64(v, o);
    const uint32_t k = lane_u32(at, o) + bits_below(w), i = lane_u32(id, o);
    if (((w >> lane()) & 1ull) && k < lim) out[k] = (i << 6) + lane();
  }
  return total;
}

__device__ __forceinline__ void label_set(uint64_t* words, uint64_t* sum, uint32_t b) {
  const uint32_t w = b >> 6;
  const uint64_t old = atomicOr((unsigned long long*)&words[w], 1ull << (b & 63));
  if (old == 0) atomicOr((unsigned long long*)&sum[w >> 6], 1ull << (w & 63));
}
// labels a and b join U and Q; the four words are updated side by side
__device__ __forceinline__ void label_set2(uint64_t* U, uint64_t* US, uint64_t* Q, uint64_t* QS,
                                           uint32_t a, uint32_t b) {
  const uint32_t wa = a >> 6, wb = b >> 6;
  const unsigned long long ba = 1ull << (a & 63), bb = 1ull << (b & 63);
  const uint64_t ua = atomicOr((unsigned long long*)&U[wa], ba);
  const uint64_t ub = atomicOr((unsigned long long*)&U[wb], bb);
  const uint64_t qa = atomicOr((unsigned long long*)&Q[wa], ba);
  const uint64_t qb = atomicOr((unsigned long long*)&Q[wb], bb);
  if (ua == 0) atomicOr((unsigned long long*)&US[wa >> 6], 1ull << (wa & 63));
  if (ub == 0) atomicOr((unsigned long long*)&US[wb >> 6], 1ull << (wb & 63));
  if (qa == 0) atomicOr((unsigned long long*)&QS[wa >> 6], 1ull << (wa & 63));
  if (qb == 0) atomicOr((unsigned long long*)&QS[wb >> 6], 1ull << (wb & 63));
}
__device__ __forceinline__ void label_clear(uint64_t* words, uint64_t* sum, uint32_t b) {
  const uint32_t w = b >> 6;
  const uint64_t bit = 1ull << (b & 63);
  const uint64_t old = atomicAnd((unsigned long long*)&words[w], ~bit);
  if ((old & ~bit) == 0)
    atomicAnd((unsigned long long*)&sum[w >> 6], ~(1ull << (w & 63)));
}

// Lane l of the wave owns a run of v items (incl: inclusive scan over the
// wave): the lane owning item e < total.
__device__ __forceinline__ uint32_t wave_owner(uint32_t incl, uint32_t e) {
  uint32_t j = 0;
#pragma unroll
  for (uint32_t step = 32; step >= 1; step >>= 1) {
    const uint32_t probe = (uint32_t)__shfl((int)incl, (int)(j + step - 1), kWave);
    if (probe <= e) j += step;
  }
  return j;
}

// bytes of the LDS region that the table takes for `slots` slots
template <class MaskT>
__host__ __device__ constexpr uint32_t table_bytes(uint32_t slots) {
  return slots * (uint32_t)(4 + 4 + sizeof(MaskT));
}
// bytes of the tables of a split of up to small_split states: block table
// (key, new label, split count, two counters, base of its staying states),
// set of split states, staying states of the tails (state, position, range),
// marks of the split states and, per block, their union and intersection
template <int WG>
__host__ __device__ constexpr uint32_t split_bytes() {
  return small_split<WG>() * (2u * 24u + 2u * 4u + 16u + 5u * 8u);
}
// bytes of the tracked labels' lists
constexpr uint32_t kTrackBytes = 4u * kTracked * kLost;
constexpr uint32_t kTrackSave = kTracked * (2 + kLost) + 1;
constexpr uint32_t log2_u32(uint32_t v) { return v <= 1 ? 0 : 1 + log2_u32(v >> 1); }

// Bit words of n labels plus summaries, twice (U and Q).
__host__ __device__ inline uint32_t rounds_bitmap_bytes(uint32_t n) {
  const uint32_t nw = (n + 63u) >> 6, nsw = (nw + 63u) >> 6;
  return 16u * (nw + nsw);
}

// The set-up of a run by one workgroup: blk from start, member lists, ranges,
// all labels unstable without verdict (global bitmaps), scratch zeroed.
// Returns false if the partition is inconsistent (never expected).
template <class MaskT, int WG>
__device__ __forceinline__ bool rounds_setup(const RoundsArgs<MaskT>& a, RoundsShared<WG>& sh,
                                             const int32_t* start, bool zero_mw) {
  const uint32_t tid = threadIdx.x, wid = tid / kWave, n = a.n;
  const uint32_t nw = (n + 63u) >> 6, nsw = (nw + 63u) >> 6;
  for (uint32_t s = tid; s < n; s += WG) {
    a.blk[s] = start[s] - (int32_t)a.s0;
    a.cnt[s] = 0;
    a.fc[s] = 0;
    a.gc[s] = 0;
    a.nlb[s] = 0;
    if (a.trk) a.trk[s] = 0;
    if (zero_mw) a.mw[s] = 0;
  }
  for (uint32_t q = wid; q < nw; q += WG / kWave) {
    const uint32_t s = (q << 6) + lane();
    const uint64_t bits = __ballot(s < n && (uint32_t)(start[s < n ? s : 0] - (int32_t)a.s0) == s);
    if (lane() == 0) {
      a.ub[q] = bits;
      a.qb[q] = bits;
    }
  }
  if (tid == 0) sh.bad = 0;
  __syncthreads();
  for (uint32_t q = wid; q < nsw; q += WG / kWave) {
    const uint32_t w = (q << 6) + lane();
    const uint64_t bits = __ballot(w < nw && a.ub[w < nw ? w : 0] != 0);
    if (lane() == 0) {
      a.us[q] = bits;
      a.qs[q] = bits;
    }
  }
  for (uint32_t i0 = wid * kWave; i0 < n; i0 += WG) {
    const uint32_t s = i0 + lane();
    const uint32_t b = s < n ? (uint32_t)a.blk[s] : 0u;
    (void)add_group(a.cnt, b, s < n, group_of(b, s < n));
  }
  __syncthreads();
  {  // block ranges: exclusive prefix sums of the sizes in label order
    const uint32_t per = (n + WG - 1) / WG;
    const uint32_t lo = min(n, tid * per), hi = min(n, lo + per);
    uint32_t sum = 0;
    for (uint32_t b = lo; b < hi; ++b) sum += (uint32_t)a.cnt[b];
    const uint32_t incl = wave_incl_scan_u32(sum);
    if (lane() == kWave - 1) sh.wsum[wid] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (uint32_t q = 0; q < wid; ++q) run += sh.wsum[q];
    for (uint32_t b = lo; b < hi; ++b) {
      const uint32_t c = (uint32_t)a.cnt[b];
      a.bs[b] = (int32_t)run;
      a.be[b] = (int32_t)run;  // fill cursor, ends at the block's end
      run += c;
    }
  }
  __syncthreads();
  for (uint32_t i0 = wid * kWave; i0 < n; i0 += WG) {
    const uint32_t s = i0 + lane();
    const uint32_t b = s < n ? (uint32_t)a.blk[s] : 0u;
    const uint32_t p = (uint32_t)add_one(a.be, b, s < n, group_of(b, s < n));
    if (s >= n) continue;
    if (p >= n) {  // cannot happen with consistent counts; report, never write
      sh.bad = 1;
      continue;
    }
    a.perm[p] = (int32_t)s;
    a.pos[s] = (int32_t)p;
    const uint32_t e0 = a.in_ptr[s];
    a.pin[p] = ((uint64_t)e0 << 32) | (a.in_ptr[s + 1] - e0);
  }
  __syncthreads();
  const bool ok = sh.bad == 0;
  for (uint32_t s = tid; s < n; s += WG) a.cnt[s] = 0;
  __syncthreads();
  return ok;
}

// The transitions by source, from those by target.
template <class MaskT, int WG>
__device__ __forceinline__ void rounds_by_source(const RoundsArgs<MaskT>& a, RoundsShared<WG>& sh) {
  const uint32_t tid = threadIdx.x, wid = tid / kWave, n = a.n;
  for (uint32_t s = tid; s < n; s += WG) a.out_cur[s] = 0;
  __syncthreads();
  for (uint32_t pass = 0; pass < 2; ++pass) {  // count, then place
    // every in-transition of the states, a wave's 64 states at a time
    for (uint32_t t0 = wid * kWave; t0 < n; t0 += WG) {
      const uint32_t t = t0 + lane();
      const uint32_t beg = t < n ? a.in_ptr[t] : 0u, deg = t < n ? a.in_ptr[t + 1] - beg : 0u;
      const uint32_t incl = wave_incl_scan_u32(deg), total = lane_u32(incl, kWave - 1);
      for (uint32_t e0 = 0; e0 < total; e0 += kWave) {
        const uint32_t x = min(e0 + lane(), total - 1);
        const uint32_t o = wave_owner(incl, x);
        const uint32_t b = (uint32_t)__shfl((int)beg, (int)o, kWave);
        const uint32_t y = (uint32_t)__shfl((int)(incl - deg), (int)o, kWave);
        if (e0 + lane() >= total) continue;
        const uint32_t e = b + (x - y);
        const uint32_t q = atomicAdd(&a.out_cur[(uint32_t)a.in_src[e] - a.s0], 1u);
        if (pass) {
          a.out_dst[q] = (int32_t)(t0 + o + a.s0);
          a.out_ord[q] = a.in_ord[e];
        }
      }
    }
    __syncthreads();
    if (pass) break;
    const uint32_t per = (n + WG - 1) / WG;
    const uint32_t lo = min(n, tid * per), hi = min(n, lo + per);
    uint32_t sum = 0;
    for (uint32_t s = lo; s < hi; ++s) sum += a.out_cur[s];
    const uint32_t incl = wave_incl_scan_u32(sum);
    if (lane() == kWave - 1) sh.wsum[wid] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (uint32_t q = 0; q < wid; ++q) run += sh.wsum[q];
    for (uint32_t s = lo; s < hi; ++s) {
      const uint32_t c = a.out_cur[s];
      a.out_ptr[s] = run;
      a.out_cur[s] = run;
      run += c;
    }
    if (tid == WG - 1) a.out_ptr[n] = run;
    __syncthreads();
  }
  for (uint32_t s = tid; s < n; s += WG) a.out_cur[s] = 0;
  __syncthreads();
}

// kBm: the bitmaps live in LDS during the loop (loaded from and stored back
// to the global ones); else they stay in global memory.
// kMode: kPlain without tracked labels, kTracking with them, kEither the two in
// one (the batched kernel, whose registers do not hold two loops).
constexpr int kPlain = 0, kTracking = 1, kEither = 2;
template <class MaskT, int WG, bool kBm, int kMode>
__device__ __forceinline__ uint32_t rounds_loop(const RoundsArgs<MaskT>& a, RoundsShared<WG>& sh,
                                                char* lds, uint32_t lds_bytes, uint32_t it0,
                                                const RoundsResume& resume, uint32_t& grid_C) {
  constexpr uint32_t kWaves = WG / kWave;
  const uint32_t tid = threadIdx.x, wid = uniform_u32(tid / kWave);
  const uint32_t n = a.n, s0 = a.s0;
  const uint32_t nw = (n + 63u) >> 6, nsw = (nw + 63u) >> 6;
  // one lane adds v to a total
  const auto count = [&](bool lead, int total, uint32_t v) {
    if (kMode == kEither && lead) atomicAdd(&sh.work[total], (unsigned long long)v);
  };

  // ---- LDS: bitmaps, then the region of the table (and of the splits)
  uint64_t *U = a.ub, *Q = a.qb, *US = a.us, *QS = a.qs;
  char* region = lds;
  uint32_t rbytes = lds_bytes;
  if (kBm) {
    U = reinterpret_cast<uint64_t*>(lds);
    Q = U + nw;
    US = Q + nw;
    QS = US + nsw;
    region = lds + 16u * (nw + nsw);
    rbytes = lds_bytes - 16u * (nw + nsw);
    for (uint32_t q = tid; q < nw; q += WG) {
      U[q] = a.ub[q];
      Q[q] = a.qb[q];
    }
    for (uint32_t q = tid; q < nsw; q += WG) {
      US[q] = a.us[q];
      QS[q] = a.qs[q];
    }
  }
  // labels x and y join U and Q (one after the other where the registers for
  // eight addresses are not there)
  const auto set2 = [&](uint32_t x, uint32_t y) {
    if (kBm || kMode != kEither) {
      label_set2(U, US, Q, QS, x, y);
    } else {
      label_set(U, US, x);
      label_set(U, US, y);
      label_set(Q, QS, x);
      label_set(Q, QS, y);
    }
  };
  // split tables (LDS that does not hold them: the global path), then the table
  constexpr uint32_t kSmall = small_split<WG>(), kB = 2u * kSmall, kBShift = 32 - log2_u32(kB);
  constexpr uint32_t kOutU = out_u<MaskT, kMode, kBm>(), kWideU = wide_u<kMode, kBm>();
  constexpr uint32_t EU = edges_per_thread<WG>(), kChunks = EU * WG / kWave;
  static_assert(kChunks <= kWave && kWaves >= 2, "one chunk of transitions per lane");
  const bool small_ok = split_bytes<WG>() + table_bytes<MaskT>(256) <= rbytes;
  MaskT* b_or = reinterpret_cast<MaskT*>(region);  // 8 bytes each are set aside
  MaskT* b_and = b_or + kB;
  MaskT* s_mv = small_ok ? b_and + kB : nullptr;
  uint64_t* x_pin = reinterpret_cast<uint64_t*>(region + 5u * 8u * kSmall);
  uint32_t* x_u = reinterpret_cast<uint32_t*>(x_pin + kSmall);
  uint32_t* x_q = x_u + kSmall;
  uint32_t* b_key = x_q + kSmall;
  uint32_t* b_nl = b_key + kB;
  uint32_t* b_cnt = b_nl + kB;
  uint32_t* b_fc = b_cnt + kB;
  uint32_t* b_gc = b_fc + kB;
  uint32_t* b_base = b_gc + kB;
  uint32_t* s_set = b_base + kB;
  if (small_ok) {
    region += split_bytes<WG>();
    rbytes -= split_bytes<WG>();
    for (uint32_t q = tid; q < kB; q += WG) {  // empty between splits
      b_key[q] = kNone;
      b_nl[q] = kNone;
      b_cnt[q] = 0;
      b_fc[q] = 0;
      b_gc[q] = 0;
      s_set[q] = kNone;
      b_or[q] = 0;
      b_and[q] = ~(MaskT)0;
    }
  }
  const bool can_track = a.out_ptr && small_ok && kTrackBytes + table_bytes<MaskT>(1024) <= rbytes;
  const bool track_dense = can_track && (uint64_t)n * sizeof(MaskT) <= rbytes - kTrackBytes;
  const uint32_t track_edges = track_dense ? kTrackEdgesDense : kTrackEdges;
  // is some block large enough to be tracked?  (Blocks only shrink.)
  const auto any_large = [&]() {
    uint32_t most = 0;
    for (uint32_t b = tid; b < n; b += WG)
      if ((uint32_t)a.blk[b] == b) most = max(most, (uint32_t)(a.be[b] - a.bs[b]));
    if (tid == 0) sh.most = 0;
    __syncthreads();
    atomicMax(&sh.most, most);
    __syncthreads();
    return (uint64_t)uniform_u32(sh.most) * a.mean_deg >= track_edges;
  };
  bool track = kMode == kEither ? can_track && !track_dense : kMode == kTracking;
  // mark words beyond LDS: a whole block costs tens of us, so tracking starts
  // at once, unless the transitions by source would have to be laid out for it
  if (kMode == kPlain && can_track && !track_dense && !a.out_cur && resume.may_track) {
    if (tid == 0) sh.it = it0;
    return kRoundsTrack;
  }
  if (kMode == kTracking && resume.lay_out) rounds_by_source(a, sh);
  uint32_t* lost = reinterpret_cast<uint32_t*>(region);  // [kTracked][kLost]
  if (kMode == kEither ? can_track : track) {
    region += kTrackBytes;
    rbytes -= kTrackBytes;
    const bool load = a.trk_save && resume.label != kNone;
    for (uint32_t q = tid; q < kTracked; q += WG) {
      sh.tlabel[q] = load ? a.trk_save[q] : kNone;
      sh.tn[q] = load ? a.trk_save[kTracked + q] : 0u;
    }
    if (load)
      for (uint32_t q = tid; q < kTracked * kLost; q += WG) lost[q] = a.trk_save[2 * kTracked + q];
  }
  uint32_t lg = 0;  // log2 of the table's slots; none below 32
  while ((2u << lg) <= 2 * EU * WG && table_bytes<MaskT>(2u << lg) <= rbytes) ++lg;
  // more states than a key has bits for (in a batch): no table, so every
  // splitter with in-transitions is marked by words per state
  const uint32_t slots = lg >= 5 && n <= kRoundsMaxN ? 1u << lg : 0u;
  const uint32_t tmask = slots - 1, tshift = 32 - lg;
  const uint32_t ecap = slots / 2;
  MaskT* t_mv = reinterpret_cast<MaskT*>(region);
  uint32_t* t_key = reinterpret_cast<uint32_t*>(t_mv + slots);
  uint32_t* t_cnt = t_key + slots;
  const bool dense = (uint64_t)n * sizeof(MaskT) <= rbytes;  // mark words of a big splitter in LDS

  // entry for label C, its lost states none (one lane per label)
  const auto track_new = [&](uint32_t C) {
    const uint32_t e = atomicAdd(&sh.tnext, 1u) % kTracked;
    const uint32_t old = sh.tlabel[e];
    if (old != kNone) a.trk[old] = 0;
    sh.tlabel[e] = C;
    sh.tn[e] = 0;
    a.trk[C] = (uint8_t)(e + 1);
    return e + 1;
  };
  // block b, tracked by entry e, loses state s
  const auto track_lost = [&](uint32_t e, uint32_t b, uint32_t s) {
    const uint32_t i = atomicAdd(&sh.tn[e], 1u);
    if (i < kLost) lost[e * kLost + i] = s;
    else a.trk[b] = 0;  // too many: no longer tracked
  };
  if (tid == 0) {
    sh.it = it0;
    sh.bad = 0;
    sh.tnext = track && a.trk_save && resume.label != kNone ? a.trk_save[kTracked * (2 + kLost)] : 0u;
  }
  if (track && resume.label != kNone && !resume.mixed) {  // workgroup-uniform
    __syncthreads();
    if (tid == 0) sh.fent = track_new(resume.label);
    __syncthreads();
    for (uint32_t i = tid; i < resume.nS; i += WG)
      if ((uint32_t)a.sbk[i] == resume.label)
        track_lost(sh.fent - 1, resume.label, (uint32_t)a.ss[i]);
  }
  bool dirty = true;  // the region does not hold an empty table (workgroup-uniform)
  bool start = true;  // before the first round
  uint32_t rc = kRoundsDone;
  // candidates of the next round: after a split the next one is a few labels
  // away (the mean gap is 4-12 iterations), so the rest would be marked for
  // nothing; a round without a split is followed by a full one
  uint32_t want = kCand;

  // ---- the next candidates, by the last wave (the first ones are busy with
  // the split that may still be under way): the smallest labels of Q ...
  const auto collect_labels = [&]() {
    uint32_t nword = 0;
    for (uint32_t q0 = 0; q0 < nsw && nword < want; q0 += kWave) {
      const uint32_t q = q0 + lane();
      const uint64_t sv = q < nsw ? QS[q] : 0ull;
      if (__ballot(sv != 0) == 0) continue;
      nword += expand_bits(sv, q, sh.wl + nword, want - nword);
    }
    nword = min(nword, want);
    wave_sync();
    const uint32_t word = lane() < nword ? sh.wl[lane()] : 0u;
    const uint64_t v = lane() < nword ? Q[word] : 0ull;
    return min(expand_bits(v, word, sh.cand, want), want);
  };
  // ... and their ranges
  const auto collect_ranges = [&](uint32_t nc) {
    if (lane() < kWaves) sh.cstarts[lane()] = 0;
    wave_sync();
    uint32_t lo = 0, sz = 0, te = 0;
    if (lane() < nc) {
      const uint32_t C = sh.cand[lane()];
      if (track) te = a.trk[C];
      lo = (uint32_t)a.bs[C];
      sz = (uint32_t)a.be[C] - lo;
      if (lo > n || sz > n - lo) {  // never expected: report, visit nothing
        sh.bad = 1;
        lo = 0;
        sz = 0;
      }
    }
    const uint32_t whole = sz;
    // (a longer list ends the tracking; never read past it all the same)
    const bool inc = te != 0 && sh.tn[te - 1] < min(sz, kLost + 1);
    if (inc) sz = sh.tn[te - 1];
    const uint32_t incs = (uint32_t)__ballot(inc);
    const uint32_t mi = wave_incl_scan_u32(sz);
    const uint64_t fit = __ballot(lane() < nc && mi <= (uint32_t)WG);
    const uint32_t np = (uint32_t)__popcll(fit);  // sizes add up: a prefix of the lanes
    // the candidates with members, and bit i: member i is the first of one
    const bool any = lane() < np && sz != 0;
    const uint64_t some = __ballot(any);
    const uint32_t r = bits_below(some), m0 = mi - sz;
    if (any) {
      sh.rfirst[r] = m0;
      sh.rb[r] = lo;
      sh.rc[r] = lane();
      sh.rtrk[r] = inc ? te : 0u;
      atomicOr((unsigned long long*)&sh.cstarts[m0 >> 6], 1ull << (m0 & 63));
    }
    if (np && lane() == np - 1) sh.rfirst[__popcll(some)] = mi;
    if (lane() < kCand) {
      sh.cb[lane()] = lo;
      sh.cpre[lane()] = mi - sz;
      sh.unst[lane()] = 0;
      sh.ctrk[lane()] = te;
      sh.cbeg[lane()] = 0;
      sh.cend[lane()] = 0;
    }
    if (lane() == 0) {
      sh.nc = nc;
      sh.np = np;
      sh.csz0 = whole;
      sh.inc = incs;
    }
    if (np && lane() == np - 1) sh.mtot = mi;
  };
  const auto reset = [&]() {  // the first wave
    if (tid == 0) {
      sh.nS = sh.nL = sh.nT = 0;
      sh.nW = 0;
      sh.tctr = 0;
      sh.fent = sh.ffresh = sh.mixed = sh.nself = 0;
    }
    if (tid < kChunks) sh.starts[tid] = 0;
  };
  uint32_t look = 0, nbig = resume.nbig;

  // a split by the tables in LDS: this thread's split state
  bool on = false, ok = false;  // there is one; its entries are consistent
  uint32_t C = 0;               // the splitter
  uint32_t s = 0, ps = 0, q = 0, at = 0, fi = kNone, other = 0, self = kNone;
  uint64_t px = 0, pq = 0;
  bool small = false;  // such a split is under way (workgroup-uniform)

  // One round, up to the moves of a split by the tables in LDS.
  const auto round = [&]() -> uint32_t {
    __syncthreads();
    small = on = ok = false;
    s = ps = q = at = other = 0;  // (so that no registers hold them meanwhile)
    px = pq = 0;
    fi = self = kNone;
    if (can_track && __builtin_expect(track ? track_dense && ++look == kTrackLook
                                            : nbig >= kTrackAfter && resume.may_track, 0)) {
      look = 0;
      nbig = 0;
      if (any_large() != track) {
        if (kMode != kEither) return kRoundsTrack;
        track = !track;  // (entries that candidates already refer to stay valid)
      }
    }
    // (loads that do not wait for one another: each is a trip of 0.06 us)
    const uint32_t v_nc = sh.nc, v_np = sh.np, v_mtot = sh.mtot, v_inc = sh.inc, v_bad = sh.bad,
                   v_it = sh.it;
    const uint64_t v_cs = sh.cstarts[lane() & (kWaves - 1)];
    const uint32_t nc = uniform_u32(v_nc);
    uint32_t np = uniform_u32(v_np);
    const uint32_t mtot = np ? uniform_u32(v_mtot) : 0u;
    if (uniform_u32(v_bad)) return kRoundsBad;
    if (v_it > a.iter_cap || (v_it == a.iter_cap && nc)) return kRoundsCap;
    uint32_t E = 0;
    if (np) {
      // ---- members: one per thread, with its in-transition range; up to a
      // wave of them need no sums over the workgroup
      const bool one = mtot <= (uint32_t)kWave;
      uint32_t beg = 0, deg = 0, c = 0, first = 0, next = 0, incl = 0;
      uint64_t some = 0;
      if (wid * kWave < mtot) {  // wave-uniform
        // the last candidate whose members start at tid or before
        const uint64_t own = lane_u64(v_cs, wid);
        uint32_t k = bits_below(own) + (uint32_t)((own >> lane()) & 1ull) - 1u;
        if (wid) {  // wave-uniform
          const uint32_t pc = lane() < wid ? (uint32_t)__popcll(v_cs) : 0u;
          k += lane_u32(wave_incl_scan_u32(pc), kWave - 1);
        }
        if (tid < mtot) {
          first = sh.rfirst[k];
          next = sh.rfirst[k + 1];
          c = sh.rc[k];
          const uint32_t base = sh.rb[k], te = sh.rtrk[k];
          const uint32_t i = tid - first;
          if (te) {
            const uint32_t s = lost[(te - 1) * kLost + i];
            beg = a.in_ptr[s];
            deg = a.in_ptr[s + 1] - beg;
          } else {
            const uint64_t x = a.pin[base + i];
            beg = (uint32_t)(x >> 32);
            deg = (uint32_t)x;
          }
        }
        incl = wave_incl_scan_u32(deg);
        some = __ballot(deg != 0);
      }
      uint32_t before = 0, sbefore = 0;
      if (!one) {
        if (lane() == kWave - 1) {
          sh.wsum[wid] = incl;
          sh.wnz[wid] = (uint32_t)__popcll(some);
        }
        __syncthreads();
        const bool lower = lane() < wid;
        const uint32_t ws = lower ? sh.wsum[lane()] : 0u, wz = lower ? sh.wnz[lane()] : 0u;
        before = lane_u32(wave_incl_scan_u32(ws), kWave - 1);
        sbefore = lane_u32(wave_incl_scan_u32(wz), kWave - 1);
      }
      if (tid < mtot) {
        const uint32_t e0 = before + incl - deg;
        if (deg) {
          const uint32_t j = sbefore + bits_below(some);
          sh.mbeg[j] = beg;
          sh.mpre[j] = e0;
          sh.mc[j] = (uint8_t)c;
          if (e0 < EU * WG)
            atomicOr((unsigned long long*)&sh.starts[e0 >> 6], 1ull << (e0 & 63));
        }
        if (tid == first) sh.cbeg[c] = e0;
        if (tid + 1 == next) sh.cend[c] = before + incl;
      }
      if (tid == (one ? kWave : WG) - 1) sh.etot = before + incl;
      __syncthreads();
      // as many candidates as the table holds (one without members ends at 0)
      const uint32_t ce = sh.cend[lane() & (kCand - 1)], etot = sh.etot;
      const uint64_t over = __ballot(lane() < np && ce > ecap);
      if (__builtin_expect(over != 0, 0)) {
        np = (uint32_t)(__ffsll((unsigned long long)over) - 1);
        const uint64_t part = __ballot(lane() < np && ce != 0);
        E = part ? lane_u32(ce, 63u - (uint32_t)__builtin_clzll(part)) : 0u;
      } else {
        E = uniform_u32(etot);
      }
      if (tid == 0 && np) {
        count(true, kWMembers, np < v_np ? sh.cpre[np] : mtot);
        count(true, kWEdges, E);
      }
    }
    const bool big = np == 0 && nc != 0;
    uint32_t es[EU], eb[EU], ek[EU], sl[EU], lo[EU], sz[EU];
    MaskT mv[EU], lmv[EU];  // a touched state's marks, its leader's
    bool part[EU];          // it leads a block with untouched members
    uint64_t split = 0;  // candidates that split something
    uint32_t nwide = 0;  // wide blocks of all candidates
    if (np) {
      // ---- transitions: insert (candidate, source), collect its marks
      uint32_t eo[EU];
      uint64_t st = 0;
      uint32_t sbefore = 0;
      if (wid * kWave < E) {  // wave-uniform
        if (lane() < kChunks) st = sh.starts[lane()];
        const uint32_t stn = (uint32_t)__popcll(st);
        sbefore = wave_incl_scan_u32(stn) - stn;
      }
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u) {
        const uint32_t e = tid + u * WG, chunk = wid + u * kWaves;
        sl[u] = kNone;
        es[u] = kNone;
        if (chunk * kWave < E) {  // wave-uniform
          // the last member that starts at e or before
          const uint64_t own = lane_u64(st, chunk);
          const uint32_t j = lane_u32(sbefore, chunk) + bits_below(own) +
                             (uint32_t)((own >> lane()) & 1ull) - 1u;
          if (e < E) {
            const uint32_t edge = sh.mbeg[j] + (e - sh.mpre[j]);
            es[u] = (uint32_t)a.in_src[edge] - s0;
            eo[u] = a.rcpp ? 0u : (uint32_t)a.in_ord[edge];
            ek[u] = (uint32_t)sh.mc[j] << kKeyBits;
          }
        }
      }
      // the range of the block that a source leads, beside its block while the
      // round is latency-bound (should it lead none, the range is not used)
      const bool wide = E > (uint32_t)WG;
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u)
        if (es[u] != kNone) {
          eb[u] = (uint32_t)a.blk[es[u]];
          if (!wide) {
            lo[u] = (uint32_t)a.bs[es[u]];
            sz[u] = (uint32_t)a.be[es[u]];
          }
        }
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u) {
        if (es[u] == kNone) continue;
        bool first;
        const uint32_t slot = table_insert(t_key, tmask, tshift, ek[u] | es[u], first);
        mask_or<MaskT>(&t_mv[slot], (MaskT)1 << (eo[u] & (sizeof(MaskT) * 8 - 1)));
        if (!first) continue;
        sl[u] = slot;
        if (eb[u] == es[u]) {
          if (wide) {
            lo[u] = (uint32_t)a.bs[es[u]];
            sz[u] = (uint32_t)a.be[es[u]];
          }
          sz[u] -= lo[u];
        }
      }
      if (kMode == kEither && wid * kWave < E) {  // wave-uniform
        uint32_t t = 0;
#pragma unroll
        for (uint32_t u = 0; u < EU; ++u) t += (uint32_t)__popcll(__ballot(sl[u] != kNone));
        count(lane() == 0, kWTouched, t);
      }
      __syncthreads();
      const uint32_t incs = uniform_u32(v_inc) & (np < 32 ? (1u << np) - 1u : ~0u);
      if (__builtin_expect(incs != 0, 0)) {  // workgroup-uniform
        // sources of lost states: the marks that no other transition into the
        // block still gives.  Long lists of outgoing transitions are searched
        // by the whole wave, and only until every mark is found again.
#pragma unroll
        for (uint32_t u = 0; u < EU; ++u) {
          const uint32_t c = es[u] != kNone ? ek[u] >> kKeyBits : 0u;
          const bool need = sl[u] != kNone && ((incs >> c) & 1u);
          if (__ballot(need) == 0) continue;
          const MaskT had = need ? t_mv[sl[u]] : (MaskT)0;
          const uint32_t label = sh.cand[c];
          MaskT left = had;
          uint32_t e = 0, end = 0;
          if (need) {
            e = a.out_ptr[es[u]];
            end = a.out_ptr[es[u] + 1];
          }
          const uint32_t own = min(end, e + 4 * kOutU);
          for (; e < own && left; e += kOutU) {
            uint32_t vd[kOutU], vo[kOutU];
#pragma unroll
            for (uint32_t v = 0; v < kOutU; ++v) {
              vd[v] = kNone;
              if (e + v < own) {
                vd[v] = (uint32_t)a.out_dst[e + v] - s0;
                vo[v] = a.rcpp ? 0u : (uint32_t)a.out_ord[e + v];
              }
            }
#pragma unroll
            for (uint32_t v = 0; v < kOutU; ++v)
              if (vd[v] != kNone) vd[v] = (uint32_t)a.blk[vd[v]];
#pragma unroll
            for (uint32_t v = 0; v < kOutU; ++v)
              if (vd[v] == label) left &= ~((MaskT)1 << (vo[v] & (sizeof(MaskT) * 8 - 1)));
          }
          uint64_t more = __ballot(need && left != 0 && own < end);
          while (more) {
            const int o = __ffsll((unsigned long long)more) - 1;
            more &= more - 1;
            const uint32_t oe = (uint32_t)__shfl((int)end, o, kWave);
            const uint32_t ol = (uint32_t)__shfl((int)label, o, kWave);
            MaskT rest = (MaskT)__shfl((unsigned long long)left, o, kWave);
            for (uint32_t x = (uint32_t)__shfl((int)own, o, kWave); x < oe && rest; x += kWave) {
              MaskT got = 0;
              if (x + lane() < oe) {
                const uint32_t d = (uint32_t)a.out_dst[x + lane()] - s0;
                const uint32_t r = a.rcpp ? 0u : (uint32_t)a.out_ord[x + lane()];
                if ((uint32_t)a.blk[d] == ol) got = (MaskT)1 << (r & (sizeof(MaskT) * 8 - 1));
              }
#pragma unroll
              for (int d = 32; d >= 1; d >>= 1)
                got |= (MaskT)__shfl_xor((unsigned long long)got, d, kWave);
              rest &= ~got;
            }
            if ((int)lane() == o) left = rest;
          }
          if (need) t_mv[sl[u]] = left;
        }
        __syncthreads();
      }
      // ---- every touched state against its leader (the leader of b is the
      // state b); the touched members of a block counted at its leader
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u) {
        mv[u] = 0;
        if (sl[u] == kNone) continue;
        mv[u] = t_mv[sl[u]];
        const uint32_t lead = eb[u] == es[u] ? sl[u]
                                             : table_find(t_key, tmask, tshift, ek[u] | eb[u]);
        if (mv[u] == 0) continue;  // no mark lost
        lmv[u] = lead != kNone ? t_mv[lead] : (MaskT)0;
        if (lead != kNone) atomicAdd(&t_cnt[lead], 1u);
        if (lmv[u] != mv[u]) sh.unst[ek[u] >> kKeyBits] = 1;
      }
      __syncthreads();
      // a touched leader with untouched members
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u) {
        part[u] = false;
        if (mv[u] == 0 || eb[u] != es[u]) continue;
        const uint32_t untouched = sz[u] - t_cnt[sl[u]];
        part[u] = untouched != 0;
        if (!part[u]) continue;
        const uint32_t c = ek[u] >> kKeyBits;
        sh.unst[c] = 1;
        if (__builtin_expect(untouched >= kSmall, 0)) {
          const uint32_t i = atomicAdd(&sh.nW, 1u);
          if (i < kWideCap) {
            sh.wc[i] = c;
            sh.wb[i] = es[u];
            sh.wlo[i] = lo[u];
            sh.wsz[i] = sz[u];
          }
        }
      }
      __syncthreads();
      const uint32_t unst = sh.unst[lane() & (kCand - 1)], v_nw = sh.nW;
      split = __ballot(lane() < np && unst != 0);
      nwide = min(uniform_u32(v_nw), kWideCap);
    }
    const uint32_t f = split ? (uint32_t)(__ffsll((unsigned long long)split) - 1) : np;
    // ---- verdicts, and the iterations that split nothing: every unstable
    // label before the next one without a verdict
    const bool turn = f < np || big;  // the iteration of C is carried out now
    C = uniform_u32(turn ? sh.cand[f < np ? f : 0] : 0u);
    if (wid == kWaves - 1 && ((lane() < np && !((split >> lane()) & 1ull)) || (turn && lane() == (f < np ? f : 0))))
      label_clear(Q, QS, sh.cand[lane()]);
    if (track && wid == kWaves - 1) {
      // a stable label is tracked from now on (its entry, if it has one,
      // starts over); so is the splitter, should its split parts be uniform
      const uint32_t l = lane() & (kCand - 1);
      const bool mine = turn && lane() == (f < np ? f : 0);
      const bool stable = lane() < np && !((split >> lane()) & 1ull);
      uint32_t te = sh.ctrk[l];
      bool fresh = false;
      if (stable || mine) {
        const bool inc = (v_inc >> l) & 1u;
        if (stable && te) sh.tn[te - 1] = 0;
        if (!te && (big || (!inc && sh.cend[l] - sh.cbeg[l] >= track_edges))) {
          te = track_new(sh.cand[l]);
          fresh = true;
        }
      }
      // A lane above may have been given the splitter's own entry: it is that
      // label's now, and the splitter has none.
      wave_sync();
      if (mine) {
        if (te && sh.tlabel[te - 1] != C) te = 0;
        sh.fent = te;
        sh.ffresh = fresh;
        sh.fold = te && !fresh ? sh.tn[te - 1] : 0u;
      }
    }
    uint32_t limit = n;  // labels before it are taken, C's own iteration included
    if (turn) limit = C + 1;
    else if (np < nc) limit = sh.cand[np];
    else if (nc == want) limit = sh.cand[want - 1] + 1;
    {
      uint32_t taken = 0;
      const uint32_t wend = (limit + 63u) >> 6;
      // (the last wave is at the verdicts: it takes the last words)
      const uint32_t first = tid < WG - kWave ? WG - kWave - 1 - tid : tid;
      for (uint32_t w = first; w < wend; w += WG) {
        if (!kBm && !((US[w >> 6] >> (w & 63)) & 1ull)) continue;
        uint64_t v = U[w];
        if (!v) continue;
        uint64_t keep = 0;
        if (w == (limit >> 6)) keep = v & (~0ull << (limit & 63));
        v &= ~keep;
        if (!v) continue;
        taken += (uint32_t)__popcll(v);
        U[w] = keep;
        if (!keep) atomicAnd((unsigned long long*)&US[w >> 6], ~(1ull << (w & 63)));
      }
      if (taken) atomicAdd(&sh.it, taken);
    }
    if (nc == 0) return kRoundsDone;  // every unstable label had its verdict: the final pass follows
    const auto clear_own = [&]() {  // this thread's slots of the table
      if (np == 0) return;
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u)
        if (sl[u] != kNone) {
          t_mv[sl[u]] = 0;
          t_key[sl[u]] = kNone;
          t_cnt[sl[u]] = 0;
        }
    };
    if (!turn) {
      clear_own();
      want = kCand;
      return kRoundsGo;
    }
    want = kCand / 2;
    // C's iteration (counted already) is carried out by the grid
    const auto to_grid = [&]() -> uint32_t {
      grid_C = C;
      if (track && wid == kWaves - 1) {  // the wave that took the entry
        wave_sync();
        if (lane() == 0 && sh.ffresh) a.trk[C] = 0;
      }
      if (tid == 0) sh.nbig = nbig;
      return kRoundsGrid;
    };
    uint32_t wides = 0;  // wide blocks that C splits
    // the members of the listed blocks that `is_split` says are split off
    const auto members = [&](const auto& is_split) {
      const uint32_t nL = uniform_u32(sh.nL);
      count(tid == 0, kWListed, nL);
      if (nL <= kWaves) {  // a block per wave, if all are small
        const uint32_t z = lane() < nL ? sh.lsz[lane()] : 0u;
        if (__ballot(z > kOwnBlock) == 0) {  // workgroup-uniform
          if (wid < nL) {
            const uint32_t b = uniform_u32(sh.lb[wid]), l = uniform_u32(sh.llo[wid]);
            const uint32_t size = lane_u32(z, wid);
            count(lane() == 0, kWVisits, size);
            for (uint32_t e0 = 0; e0 < size; e0 += kWave) {
              const uint32_t e = e0 + lane();
              uint32_t s = 0;
              bool sp = false;
              if (e < size) {
                s = (uint32_t)a.perm[l + e];
                sp = is_split(s);
              }
              const uint32_t si = list_push(&sh.nS, sp);
              if (sp) put_split(a, sh, s_mv, kSmall, si, (int32_t)s, (int32_t)b, (MaskT)0);
            }
          }
          return;
        }
      }
      for (uint32_t j0 = 0; j0 < nL; j0 += kWave) {
        const uint32_t j = j0 + lane();
        uint32_t b = 0, l = 0, z = 0;
        if (j < nL) {
          b = j < kListCap ? sh.lb[j] : (uint32_t)a.lb[j];
          l = j < kListCap ? sh.llo[j] : (uint32_t)a.llo[j];
          z = j < kListCap ? sh.lsz[j] : (uint32_t)a.lsz[j];
        }
        const uint32_t incl = wave_incl_scan_u32(z);
        const uint32_t total = lane_u32(incl, kWave - 1);
        count(tid == 0, kWVisits, total);
        for (uint32_t e0 = wid * kWave; e0 < total; e0 += WG) {
          const uint32_t e = e0 + lane();
          const uint32_t ee = min(e, total - 1);
          const uint32_t o = wave_owner(incl, ee);
          const uint32_t ob = (uint32_t)__shfl((int)b, (int)o, kWave);
          const uint32_t ol = (uint32_t)__shfl((int)l, (int)o, kWave);
          const uint32_t oi = (uint32_t)__shfl((int)(incl - z), (int)o, kWave);
          uint32_t s = 0;
          bool sp = false;
          if (e < total) {
            s = (uint32_t)a.perm[ol + (ee - oi)];
            sp = is_split(s);
          }
          const uint32_t si = list_push(&sh.nS, sp);
          if (sp) put_split(a, sh, s_mv, kSmall, si, (int32_t)s, (int32_t)ob, (MaskT)0);
        }
      }
    };
    if (__builtin_expect(big, 0)) {
      // ---- a splitter beyond the table: mark words per state
      ++nbig;
      const uint32_t cb = uniform_u32(sh.cb[0]), csz = uniform_u32(sh.csz0);
      bool grid = false;
      if (dense) {
        grid = a.grid_dense && (uint64_t)csz * a.mean_deg >= a.grid_dense;
      } else if (a.grid_edges) {
        grid = (uint64_t)csz * a.mean_deg >= a.grid_edges;
        if (!grid) {  // few members, but they may be hubs: count
          uint32_t edges = 0;
          for (uint32_t i = tid; i < csz; i += WG)
            edges += min((uint32_t)a.pin[cb + i], a.grid_edges);
          if (tid == 0) sh.most = 0;
          __syncthreads();
          if (edges) atomicAdd(&sh.most, min(edges, a.grid_edges));
          __syncthreads();
          grid = uniform_u32(sh.most) >= a.grid_edges;
        }
      }
      if (grid) return to_grid();
      count(tid == 0, kWMembers, csz);
      if (dense) {
        // mark words of all states in LDS.  Four members per thread are in
        // flight; a member of many in-transitions is the whole wave's.
        MaskT* mw = reinterpret_cast<MaskT*>(region);
        for (uint32_t s = tid; s < n; s += WG) mw[s] = 0;
        dirty = true;
        __syncthreads();
        const auto mark = [&](uint32_t s, uint32_t o) {
          // a hub's transitions find its bit set: plain reads of one word do
          // not serialise, atomics on it do
          const MaskT bit = (MaskT)1 << (o & (sizeof(MaskT) * 8 - 1));
          if (!(mw[s] & bit)) mask_or<MaskT>(&mw[s], bit);
        };
        for (uint32_t i0 = wid * kWave; i0 < csz; i0 += kScanU * WG) {
          uint32_t beg[kScanU], deg[kScanU];
          uint32_t most = 0;
#pragma unroll
          for (uint32_t u = 0; u < kScanU; ++u) {
            const uint32_t i = i0 + u * WG + lane();
            const uint64_t x = i < csz ? a.pin[cb + i] : 0ull;
            beg[u] = (uint32_t)(x >> 32);
            deg[u] = (uint32_t)x;
          }
#pragma unroll
          for (uint32_t u = 0; u < kScanU; ++u) {
            uint64_t hb = __ballot(deg[u] > 2 * kWave);
            while (hb) {
              const int o = __ffsll((unsigned long long)hb) - 1;
              hb &= hb - 1;
              const uint32_t ob = (uint32_t)__shfl((int)beg[u], o, kWave);
              const uint32_t od = (uint32_t)__shfl((int)deg[u], o, kWave);
              for (uint32_t e = lane(); e < od; e += kWave)
                mark((uint32_t)a.in_src[ob + e] - s0, a.rcpp ? 0u : (uint32_t)a.in_ord[ob + e]);
            }
            count(deg[u] != 0, kWEdges, deg[u]);
            if (deg[u] > 2 * kWave) deg[u] = 0;
            most = max(most, deg[u]);
          }
          for (uint32_t e = 0; e < most; e += 2) {
            uint32_t vs[2 * kScanU], vo[2 * kScanU];
#pragma unroll
            for (uint32_t u = 0; u < kScanU; ++u)
#pragma unroll
              for (uint32_t v = 0; v < 2; ++v) {
                vs[2 * u + v] = kNone;
                if (e + v < deg[u]) {
                  vs[2 * u + v] = (uint32_t)a.in_src[beg[u] + e + v] - s0;
                  vo[2 * u + v] = a.rcpp ? 0u : (uint32_t)a.in_ord[beg[u] + e + v];
                }
              }
#pragma unroll
            for (uint32_t v = 0; v < 2 * kScanU; ++v)
              if (vs[v] != kNone) mark(vs[v], vo[v]);
          }
        }
        __syncthreads();
        // every state against its leader
        for (uint32_t i0 = wid * kWave; i0 < n; i0 += kScanU * WG) {
          uint32_t vb[kScanU];
#pragma unroll
          for (uint32_t u = 0; u < kScanU; ++u) {
            const uint32_t s = i0 + u * WG + lane();
            vb[u] = s < n ? (uint32_t)a.blk[s] : 0u;
          }
#pragma unroll
          for (uint32_t u = 0; u < kScanU; ++u) {
            const uint32_t s = i0 + u * WG + lane();
            const bool sp = s < n && mw[s] != mw[vb[u]];
            const uint32_t si = list_push(&sh.nS, sp);
            if (sp) put_split(a, sh, s_mv, kSmall, si, (int32_t)s, (int32_t)vb[u], mw[s]);
          }
        }
        __syncthreads();
      } else {
        // mark words in global memory, with a list of the touched states
        MaskT* mw = a.mw;
        __syncthreads();
        for (uint32_t i0 = wid * kWave; i0 < csz; i0 += WG) {
          const uint32_t i = i0 + lane();
          uint32_t beg = 0, deg = 0;
          if (i < csz) {
            const uint64_t x = a.pin[cb + i];
            beg = (uint32_t)(x >> 32);
            deg = (uint32_t)x;
          }
          const uint32_t incl = wave_incl_scan_u32(deg);
          const uint32_t total = lane_u32(incl, kWave - 1);
          count(lane() == 0, kWEdges, total);
          for (uint32_t e0 = 0; e0 < total; e0 += kWave * kScanU) {
            uint32_t vs[kScanU], vo[kScanU], vb[kScanU], vl[kScanU], vh[kScanU];
            bool first[kScanU];
#pragma unroll
            for (uint32_t u = 0; u < kScanU; ++u) {
              const uint32_t e = e0 + u * kWave + lane();
              const uint32_t ee = min(e, total - 1);
              const uint32_t j = wave_owner(incl, ee);
              const uint32_t jb = (uint32_t)__shfl((int)beg, (int)j, kWave);
              const uint32_t ji = (uint32_t)__shfl((int)(incl - deg), (int)j, kWave);
              vs[u] = kNone;
              if (e < total) {
                const uint32_t edge = jb + (ee - ji);
                vs[u] = (uint32_t)a.in_src[edge] - s0;
                vo[u] = a.rcpp ? 0u : (uint32_t)a.in_ord[edge];
              }
            }
#pragma unroll
            for (uint32_t u = 0; u < kScanU; ++u) {
              first[u] = false;
              vb[u] = vl[u] = vh[u] = 0;
              if (vs[u] == kNone) continue;
              const MaskT bit = (MaskT)1 << (vo[u] & (sizeof(MaskT) * 8 - 1));
              first[u] = mask_or<MaskT>(&mw[vs[u]], bit) == 0;
              vb[u] = (uint32_t)a.blk[vs[u]];
              vl[u] = (uint32_t)a.bs[vs[u]];
              vh[u] = (uint32_t)a.be[vs[u]];
            }
#pragma unroll
            for (uint32_t u = 0; u < kScanU; ++u) {
              const uint32_t ti = list_push(&sh.nT, first[u]);
              if (first[u]) {
                a.ts[ti] = (int32_t)vs[u];
                a.tb[ti] = (int32_t)vb[u];
              }
              // a touched leader of a one-state block has no untouched member
              const bool lead = first[u] && vb[u] == vs[u] && vh[u] - vl[u] > 1;
              const uint32_t li = list_push(&sh.nL, lead);
              if (lead) put_block(a, sh, li, vs[u], vl[u], vh[u] - vl[u]);
            }
          }
        }
        __syncthreads();
        const uint32_t nT = uniform_u32(sh.nT);
        count(tid == 0, kWTouched, nT);
        for (uint32_t i0 = wid * kWave; i0 < nT; i0 += WG) {
          const uint32_t i = i0 + lane();
          int32_t s = 0, b = 0;
          bool sp = false;
          if (i < nT) {
            s = a.ts[i];
            b = a.tb[i];
            sp = s != b && mw[s] != mw[b];
          }
          const uint32_t si = list_push(&sh.nS, sp);
          if (sp) put_split(a, sh, s_mv, kSmall, si, s, b, mw[s]);
        }
        __syncthreads();
      }
    } else {
      // ---- the split states of C from the table: touched states that differ
      // from their leader, and the untouched members of blocks whose leader
      // was touched
      // (those of wide blocks are not listed)
      if (__builtin_expect(nwide != 0, 0)) {  // workgroup-uniform
        const uint32_t w = lane() & (kWideCap - 1);
        const bool its = lane() < nwide && sh.wc[w] == f;
        wides = (uint32_t)__ballot(its);
        const uint32_t z = wave_incl_scan_u32(its ? sh.wsz[w] : 0u);
        if (a.grid_edges && lane_u32(z, kWave - 1) >= kGridMembers) {
          clear_own();
          return to_grid();
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < EU; ++u) {
        if ((wid + u * kWaves) * kWave >= E) continue;  // wave-uniform
        bool mine = sl[u] != kNone && (ek[u] >> kKeyBits) == f && mv[u] != 0;
        if (__builtin_expect(wides != 0, 0)) {
          bool wide = false;
          for (uint32_t w = wides; w; w &= w - 1) wide |= eb[u] == sh.wb[__ffs((int)w) - 1];
          wide = wide && mine;
          const uint32_t i = list_push(&sh.nT, wide && lmv[u] == mv[u]);  // it stays
          if (i != kNone) {
            a.ts[i] = (int32_t)es[u];
            a.tb[i] = (int32_t)eb[u];
          }
          mine = mine && !wide;
        }
        const bool sp = mine && es[u] != eb[u] && lmv[u] != mv[u];
        const bool pt = mine && part[u];
        const uint64_t sbal = __ballot(sp), pbal = __ballot(pt);
        if ((sbal | pbal) == 0) continue;
        unsigned long long base = 0;  // both lists by one atomic
        if (lane() == 0)
          base = atomicAdd(&sh.nSL, (unsigned long long)__popcll(pbal) << 32 |
                                        (unsigned long long)__popcll(sbal));
        base = lane_u64(base, 0);
        if (sp)
          put_split(a, sh, s_mv, kSmall, (uint32_t)base + bits_below(sbal), (int32_t)es[u],
                    (int32_t)eb[u], mv[u]);
        if (pt) put_block(a, sh, (uint32_t)(base >> 32) + bits_below(pbal), eb[u], lo[u], sz[u]);
      }
      __syncthreads();
    }
    if (sh.nL) {  // workgroup-uniform (none where all states were compared)
      members([&](uint32_t t) {
        if (big) return a.mw[t] == 0;
        const uint32_t x = table_find(t_key, tmask, tshift, (f << kKeyBits) | t);
        return x == kNone || t_mv[x] == 0;
      });
      __syncthreads();
    }
    // ---- wide blocks: the members that stay are touched states, and listed;
    // by far the most members are untouched.  So the block is gone through
    // twice, for its smallest split state and to relabel, and the few that stay
    // get their label back and go to the front.
    for (uint32_t w = wides; __builtin_expect(w != 0, 0); w &= w - 1) {
      const uint32_t j = (uint32_t)__ffs((int)w) - 1;
      const uint32_t b = uniform_u32(sh.wb[j]), l = uniform_u32(sh.wlo[j]), z = uniform_u32(sh.wsz[j]);
      const uint32_t lx = table_find(t_key, tmask, tshift, (f << kKeyBits) | b);
      const MaskT lm = lx != kNone ? t_mv[lx] : (MaskT)0;
      const auto stays = [&](uint32_t s) {
        const uint32_t x = table_find(t_key, tmask, tshift, (f << kKeyBits) | s);
        return x != kNone && t_mv[x] == lm;
      };
      if (tid == 0) {
        sh.wmin = kNone;
        sh.wstay = sh.wfront = sh.wback = 0;
      }
      __syncthreads();
      const uint32_t nT = uniform_u32(sh.nT);
      uint32_t kept = 0;
      for (uint32_t i0 = wid * kWave; i0 < nT; i0 += WG)
        kept += (uint32_t)__popcll(
            __ballot(i0 + lane() < nT && (uint32_t)a.tb[min(i0 + lane(), nT - 1)] == b));
      if (lane() == 0 && kept) atomicAdd(&sh.wstay, kept);
      // (only a member below the least one so far is looked up)
      for (uint32_t i0 = wid * kWave; i0 < z; i0 += kWideU * WG) {
        uint32_t v[kWideU];
#pragma unroll
        for (uint32_t u = 0; u < kWideU; ++u) {
          const uint32_t i = i0 + u * WG + lane();
          v[u] = i < z ? (uint32_t)a.perm[l + i] : kNone;
        }
        const uint32_t before = sh.wmin;
        uint32_t least = before;
#pragma unroll
        for (uint32_t u = 0; u < kWideU; ++u)
          if (v[u] < least && !stays(v[u])) least = v[u];
        if (__ballot(least != before) == 0) continue;
        least = wave_min_u32(least);
        if (lane() == 0) atomicMin(&sh.wmin, least);
      }
      __syncthreads();
      const uint32_t nl = uniform_u32(sh.wmin), t = uniform_u32(sh.wstay);
      if (nl >= n || t == 0 || t >= z) {  // never expected: the leader stays, some are untouched
        if (tid == 0) sh.bad = 1;
        __syncthreads();
        continue;
      }
      for (uint32_t i0 = tid; i0 < z; i0 += kWideU * WG) {
        uint32_t v[kWideU];
#pragma unroll
        for (uint32_t u = 0; u < kWideU; ++u) {
          const uint32_t i = i0 + u * WG;
          v[u] = i < z ? (uint32_t)a.perm[l + i] : kNone;
        }
#pragma unroll
        for (uint32_t u = 0; u < kWideU; ++u)
          if (v[u] != kNone) a.blk[v[u]] = (int32_t)nl;
      }
      __syncthreads();
      for (uint32_t i0 = wid * kWave; i0 < nT; i0 += WG) {
        const uint32_t i = min(i0 + lane(), nT - 1);
        const bool on = i0 + lane() < nT && (uint32_t)a.tb[i] == b;
        uint32_t p = 0;
        if (on) {
          const uint32_t s = (uint32_t)a.ts[i];
          a.blk[s] = (int32_t)b;
          p = (uint32_t)a.pos[s];
        }
        const uint32_t y = list_push(&sh.wback, on && p >= l + t);
        if (y != kNone) a.sfi[y] = (int32_t)p;
      }
      for (uint32_t i0 = wid * kWave; i0 < t; i0 += WG) {
        const uint32_t i = i0 + lane();
        const bool on = i < t && !stays((uint32_t)a.perm[l + i]);
        const uint32_t x = list_push(&sh.wfront, on);
        if (x != kNone) a.sps[x] = (int32_t)(l + i);
      }
      __syncthreads();
      for (uint32_t i = tid; i < min(sh.wfront, sh.wback); i += WG) {
        const uint32_t p = (uint32_t)a.sps[i], q = (uint32_t)a.sfi[i];
        const uint32_t u = (uint32_t)a.perm[p], v = (uint32_t)a.perm[q];
        const uint64_t xp = a.pin[p], xq = a.pin[q];
        a.perm[p] = (int32_t)v;
        a.pos[v] = (int32_t)p;
        a.pin[p] = xq;
        a.perm[q] = (int32_t)u;
        a.pos[u] = (int32_t)q;
        a.pin[q] = xp;
      }
      if (tid == 0) {
        a.bs[nl] = (int32_t)(l + t);
        a.be[nl] = (int32_t)(l + z);
        a.be[b] = (int32_t)(l + t);
        set2(b, nl);
        count(true, kWBlocks, 1);
        count(true, kWSplit, z - t);
        count(true, kWVisits, z);
        // neither the block nor C is tracked any longer, and C needs a verdict
        // (its split parts may hold different marks)
        if (track) {
          a.trk[b] = 0;
          a.trk[C] = 0;
          sh.fent = 0;
          if (!a.rcpp) label_set(Q, QS, C);
        }
      }
      __syncthreads();
    }
    if (__builtin_expect(big, 0)) {
      if (!dense) {
        const uint32_t nT = uniform_u32(sh.nT);
        for (uint32_t i = tid; i < nT; i += WG) a.mw[a.ts[i]] = 0;
      }
      if (sh.nS == 0) {  // stable: its entry starts over
        if (tid == 0 && track) sh.tn[sh.fent - 1] = 0;
        return kRoundsGo;
      }
    } else {
      clear_own();
    }
    // ---- split: the split part of each block goes to the tail of its range
    // and takes its smallest member as label; front split states trade places
    // with the staying states of the tail
    const uint32_t nS = uniform_u32(sh.nS);
    count(tid == 0, kWSplit, nS);
    if (__builtin_expect(nS <= kSmall && small_ok, 1)) {
      uint32_t b = 0, blo = 0, bhi = 0, r = 0, te = 0, slot = 0;
      on = tid < nS;
      small = true;
      if (on) {
        s = (uint32_t)sh.ss[tid];
        b = (uint32_t)sh.sb[tid];
        ps = (uint32_t)a.pos[s];
        blo = (uint32_t)a.bs[b];
        bhi = (uint32_t)a.be[b];
        if (track) te = a.trk[b];
        bool first;
        slot = table_insert(b_key, kB - 1, kBShift, b, first);
        r = atomicAdd(&b_cnt[slot], 1u);
        atomicMin(&b_nl[slot], s);
        at = slot | table_insert(s_set, kB - 1, kBShift, s, first) << 16;
        if (track) {
          const MaskT mv = s_mv[tid];
          mask_or<MaskT>(&b_or[slot], mv);
          mask_and<MaskT>(&b_and[slot], mv);
        }
      }
      __syncthreads();
      if (on) {
        const uint32_t c = b_cnt[slot], nl = b_nl[slot], ne = bhi - c;
        q = ne + r;
        ok = bhi <= n && blo < ne && ne < bhi && ps >= blo && ps < bhi;  // else never expected
        if (!ok) {
          sh.bad = 1;
        } else {
          other = (uint32_t)a.perm[q];  // every tail position is examined once
          pq = a.pin[q];
          if (ps < ne) {
            px = a.pin[ps];
            fi = atomicAdd(&b_fc[slot], 1u);
          }
          if (r == 0) b_base[slot] = atomicAdd(&sh.tctr, c);
          // Algorithm 3 re-marks C (below); it needs a verdict if it changed
          // (it joins Q as a part then) or a split part is not uniform
          if (track && s == nl && b_or[slot] != b_and[slot]) {
            sh.mixed = 1;
            if (!a.rcpp) label_set(Q, QS, C);
          }
          if (track && b == C) self = atomicAdd(&sh.nself, 1u);
          else if (track && te) track_lost(te - 1, b, s);
          a.blk[s] = (int32_t)nl;
          if (s == nl) {  // the new leader: one thread per split block
            a.bs[s] = (int32_t)ne;
            a.be[s] = (int32_t)bhi;
            a.be[b] = (int32_t)ne;
            set2(b, s);
            count(true, kWBlocks, 1);
          }
        }
      }
      if (tid == WG - 1 && !a.rcpp) {
        label_set(U, US, C);
        if (!track) label_set(Q, QS, C);
      }
    } else {
      // more split states: the same through global arrays, and the blocks that
      // split are no longer tracked
      if (tid == WG - 1) {
        if (!a.rcpp) set2(C, C);
        if (track) a.trk[C] = 0;
      }
      const uint64_t epoch = (uint64_t)sh.it << 32;  // this iteration's number
      const auto entry = [&](uint32_t i, uint32_t& s, uint32_t& b) {
        const bool on = i < nS;
        s = b = 0;
        if (on) {
          s = (uint32_t)(i < kSmall ? sh.ss[i] : a.ss[i]);
          b = (uint32_t)(i < kSmall ? sh.sb[i] : a.sbk[i]);
        }
        return on;
      };
      // the smallest split state of each block, and a rank for every one
      for (uint32_t i0 = wid * kWave; i0 < nS; i0 += WG) {
        uint32_t s, b;
        const bool on = entry(i0 + lane(), s, b);
        const Group g = group_of(b, on);
        bid_min(a.nlb, b, epoch, s, on, g);
        const int32_t r = add_one(a.cnt, b, on, g);
        if (on) a.sr[i0 + lane()] = r;
      }
      __syncthreads();
      // the new label; states in front of the tail are numbered
      for (uint32_t i0 = wid * kWave; i0 < nS; i0 += WG) {
        uint32_t s, b;
        const bool on = entry(i0 + lane(), s, b);
        int32_t e = 0, l = 0, ps = 0, c = 0;
        if (on) {
          e = a.be[b];
          l = a.bs[b];
          ps = a.pos[s];
          c = a.cnt[b];
          a.blk[s] = (int32_t)(kNone - (uint32_t)a.nlb[b]);
        }
        const int32_t ne = e - c;
        const bool ok = on && l >= 0 && l < ne && ne < e && e <= (int32_t)n && ps >= l && ps < e;
        if (on && !ok) sh.bad = 1;  // never expected: the entry does nothing
        const bool front = ok && ps < ne;
        const int32_t f = add_one(a.fc, b, front, group_of(b, front));
        if (on) {
          a.sfi[i0 + lane()] = front ? ne + f : -1;
          a.sps[i0 + lane()] = ok ? ps : -1;
        }
      }
      __syncthreads();
      // the staying states of each tail
      for (uint32_t i0 = wid * kWave; i0 < nS; i0 += WG) {
        uint32_t s, b;
        bool on = entry(i0 + lane(), s, b);
        int32_t ne = 0, q = 0, e = 0;
        uint32_t u = 0;
        on = on && a.sps[i0 + lane()] >= 0;
        if (on) {
          e = a.be[b];
          ne = e - a.cnt[b];
          q = ne + a.sr[i0 + lane()];
          on = q < e;
          if (!on) sh.bad = 1;  // never expected
        }
        if (on) {
          u = (uint32_t)a.perm[q];  // every tail position is examined once
          on = (uint32_t)a.blk[u] == b;
        }
        const int32_t j = add_one(a.gc, b, on, group_of(b, on));
        if (!on) continue;
        if (ne + j < e) a.tmp64[ne + j] = ((uint64_t)u << 32) | (uint32_t)q;
        else sh.bad = 1;  // never expected
      }
      __syncthreads();
      for (uint32_t i = tid; i < nS; i += WG) {
        uint32_t s, b;
        (void)entry(i, s, b);
        const int32_t x = a.sfi[i], ps = a.sps[i];
        if (x >= 0) {
          const uint64_t uq = a.tmp64[x];
          const uint32_t q = (uint32_t)uq, u = (uint32_t)(uq >> 32);
          if (q < n && u < n) {
            const uint64_t xq = a.pin[q], xp = a.pin[ps];
            a.perm[ps] = (int32_t)u;
            a.pos[u] = ps;
            a.pin[ps] = xq;
            a.perm[q] = (int32_t)s;
            a.pos[s] = (int32_t)q;
            a.pin[q] = xp;
          } else {
            sh.bad = 1;  // never expected
          }
        }
        if (ps >= 0 && (uint32_t)a.blk[s] == s) {  // the new leader: one thread per split block
          const int32_t e = a.be[b], ne = e - a.cnt[b];
          a.bs[s] = ne;
          a.be[s] = e;
          a.be[b] = ne;
          a.cnt[b] = 0;
          a.fc[b] = 0;
          a.gc[b] = 0;
          if (track) a.trk[b] = 0;
          set2(b, s);
          count(true, kWBlocks, 1);
        }
      }
    }
    return kRoundsGo;
  };

  for (;;) {
    if (!start) {
      rc = round();
      if (rc != kRoundsGo) break;
    }
    start = false;
    // The candidates of the next round, by the last wave; after a split by the
    // tables in LDS, whose labels, ranges and tracked entries are final behind
    // this barrier, beside the moves.
    __syncthreads();
    const uint32_t slot = at & 0xFFFFu;  // of the block, and of the state in the set
    if (small) {
      if (ok && table_find(s_set, kB - 1, kBShift, other) == kNone) {
        const uint32_t x = b_base[slot] + atomicAdd(&b_gc[slot], 1u);
        if (x < kSmall) {
          x_u[x] = other;
          x_q[x] = q;
          x_pin[x] = pq;
        } else {
          sh.bad = 1;  // never expected
        }
      }
      // C's own entry: with uniform split parts the partition is stable under
      // what C was, so its lost states are those of this iteration; else they
      // join the earlier ones, and an entry taken in this round ends
      if (track) {
        const uint32_t fent = sh.fent, mixed = sh.mixed, nself = sh.nself;
        const bool ends = mixed && sh.ffresh;
        const uint32_t had = mixed ? sh.fold : 0u;
        if (self != kNone && fent && !ends && had + self < kLost)
          lost[(fent - 1) * kLost + had + self] = s;
        if (tid == WG - 1 && fent) {
          sh.tn[fent - 1] = had + nself;
          if (ends || had + nself > kLost) a.trk[C] = 0;
        }
      }
    }
    uint32_t next_nc = 0;
    if (wid == kWaves - 1) next_nc = collect_labels();
    if (small) {
      __syncthreads();
      if (on) {  // the tables are empty again
        b_key[slot] = kNone;
        b_nl[slot] = kNone;
        b_cnt[slot] = 0;
        b_fc[slot] = 0;
        b_gc[slot] = 0;
        s_set[at >> 16] = kNone;
        if (track) {
          b_or[slot] = 0;
          b_and[slot] = ~(MaskT)0;
        }
      }
      if (ok && fi != kNone) {
        const uint32_t x = b_base[slot] + fi;
        const uint32_t v = x_u[x], vq = x_q[x];
        if (v < n && vq < n) {
          a.perm[ps] = (int32_t)v;
          a.pos[v] = (int32_t)ps;
          a.pin[ps] = x_pin[x];
          a.perm[vq] = (int32_t)s;
          a.pos[s] = (int32_t)vq;
          a.pin[vq] = px;
        } else {
          sh.bad = 1;  // never expected
        }
      }
    }
    if (wid == kWaves - 1) collect_ranges(next_nc);
    else if (wid == 0) reset();
    if (__builtin_expect(dirty, 0)) {
      for (uint32_t i = tid; i < slots; i += WG) {
        t_mv[i] = 0;
        t_key[i] = kNone;
        t_cnt[i] = 0;
      }
      dirty = false;
    }
  }
  __syncthreads();
  if (kBm) {
    for (uint32_t q = tid; q < nw; q += WG) {
      a.ub[q] = U[q];
      a.qb[q] = Q[q];
    }
    for (uint32_t q = tid; q < nsw; q += WG) {
      a.us[q] = US[q];
      a.qs[q] = QS[q];
    }
    __syncthreads();
  }
  if (track && a.trk_save && rc == kRoundsGrid) {
    for (uint32_t q = tid; q < kTracked; q += WG) {
      a.trk_save[q] = sh.tlabel[q];
      a.trk_save[kTracked + q] = sh.tn[q];
    }
    for (uint32_t q = tid; q < kTracked * kLost; q += WG) a.trk_save[2 * kTracked + q] = lost[q];
    if (tid == 0) a.trk_save[kTracked * (2 + kLost)] = sh.tnext;
  }
  return rc;
}

}  // namespace bisim
