// The rounds of one workgroup (rounds_dev.h) on host lanes: the run of one
// LTS, as k_rounds goes (the loops without and with tracked labels in turn)
// or as k_batch goes (both in one).  Arrays that the set-up has to initialise
// start with arbitrary values, and every array is of its exact size.
#include "internal.h"
#include "rounds_dev.h"

using namespace bisim;

namespace {
struct Run {
  int32_t n, m, K;
  const int32_t* start;
  const uint32_t* in_ptr;
  const int32_t *in_src, *in_ord;
  const uint32_t* out_ptr;  // transitions by source (null: not tracked)
  const int32_t *out_dst, *out_ord;
  int32_t rcpp, lds_bytes, bitmaps_in_lds, either;
  uint32_t seed;
  int32_t* block;
  int64_t* iterations;
};

template <class MaskT, int WG, bool kBm>
uint32_t go(const Run& r) {
  const size_t n = (size_t)r.n, m = (size_t)r.m, nw = (n + 63) / 64, nsw = (nw + 63) / 64;
  std::vector<std::vector<uint64_t>> kept;
  const auto words = [&](size_t count, size_t size, uint64_t value) {
    kept.emplace_back((count * size + 7) / 8, value);
    return kept.back().data();
  };
  constexpr uint64_t kAny = 0x5a5a5a5a5a5a5a5aull;
  RoundsArgs<MaskT> a{};
  a.n = (uint32_t)r.n;
  a.iter_cap = 3 * a.n + 1;
  a.rcpp = (uint32_t)r.rcpp;
  a.mean_deg = n ? (uint32_t)((m + n - 1) / n) : 1u;
  a.in_ptr = r.in_ptr;
  a.in_src = r.in_src;
  a.in_ord = r.in_ord;
  int32_t** state[] = {&a.blk, &a.perm, &a.pos, &a.bs, &a.be, &a.cnt, &a.fc, &a.gc, &a.ts, &a.tb,
                       &a.lb, &a.llo, &a.lsz, &a.ss, &a.sbk, &a.sr, &a.sfi, &a.sps};
  for (int32_t** p : state) *p = (int32_t*)words(n, 4, kAny);
  a.pin = words(n, 8, kAny);
  a.nlb = words(n, 8, kAny);
  a.tmp64 = words(n, 8, kAny);
  a.mw = (MaskT*)words(n, sizeof(MaskT), kAny);
  for (uint64_t** p : {&a.ub, &a.qb}) *p = words(nw, 8, kAny);
  for (uint64_t** p : {&a.us, &a.qs}) *p = words(nsw, 8, kAny);
  if (r.out_ptr) {
    a.trk = (uint8_t*)words(n, 1, kAny);
    if (r.either) {
      a.out_ptr = (uint32_t*)r.out_ptr;
      a.out_dst = (int32_t*)r.out_dst;
      a.out_ord = (int32_t*)r.out_ord;
    } else {  // laid out by the workgroup
      a.out_ptr = (uint32_t*)words(n + 1, 4, kAny);
      a.out_dst = (int32_t*)words(m, 4, kAny);
      a.out_ord = (int32_t*)words(m, 4, kAny);
      a.out_cur = (uint32_t*)words(n, 4, 0);
    }
  }
  std::vector<RoundsShared<WG>> shared(1);
  memset((void*)shared.data(), 0x3c, sizeof shared[0]);
  RoundsShared<WG>& sh = shared[0];
  uint64_t* lds = words((size_t)r.lds_bytes, 1, kAny);
  uint32_t rc = kRoundsBad;
  lanes::run(WG, r.seed, [&]() {
    if (!rounds_setup<MaskT, WG>(a, sh, r.start, true)) return;
    uint32_t none = 0, it = 0, got = kRoundsBad;
    RoundsResume resume;
    resume.may_track = true;
    resume.lay_out = a.out_cur != nullptr;
    for (bool track = false;; track = !track) {
      if (r.either)
        got = rounds_loop<MaskT, WG, kBm, kEither>(a, sh, (char*)lds, r.lds_bytes, it, resume, none);
      else if (track)
        got = rounds_loop<MaskT, WG, kBm, kTracking>(a, sh, (char*)lds, r.lds_bytes, it, resume, none);
      else
        got = rounds_loop<MaskT, WG, kBm, kPlain>(a, sh, (char*)lds, r.lds_bytes, it, resume, none);
      if (got != kRoundsTrack) break;
      resume.may_track = false;  // a run changes to tracking once, and back once
      __syncthreads();
      it = sh.it;
      __syncthreads();
    }
    if (threadIdx.x == 0) rc = got;
  });
  memcpy(r.block, a.blk, 4 * n);
  *r.iterations = (int64_t)sh.it + 1;  // with the final pass
  return rc;
}

template <class MaskT>
uint32_t go_any(const Run& r) {
  return r.bitmaps_in_lds ? go<MaskT, 128, true>(r) : go<MaskT, 128, false>(r);
}
}  // namespace

extern "C" int32_t model_run(const Run* r) {
  return (int32_t)(r->K > 32 ? go_any<uint64_t>(*r) : go_any<uint32_t>(*r));
}
