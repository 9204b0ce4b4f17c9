// Annealing chains under static admission for at most 16 requests that stay hot: four
// proposals per round, one per 16-lane row of the chain's wave (gfx950).
//
// At the paper's scale (4 to 16 requests) the register kernel leaves three quarters of the
// wave empty and its time is one wave's latency per proposal; and at the paper's temperatures
// (500 down to 20) nearly every proposal is kept. So a round scores proposals k .. k + 3 at
// once, each on top of the ones before it as if those were kept, and takes the decisions in
// order up to the first rejection, after which the rest is scored again on the right order: the
// trajectory, accept count, digest and best order are those of one proposal at a time. An order
// is one 64-bit scalar of 4-bit request ids: a move is a few scalar shifts and masks, and
// accepting one a register copy. Lane r of every row's table holds request r; a lane's request
// comes by one lane permute per field. Batches lie inside a row, so every reduction and scan
// stops at the row; the acceptance rule runs once for all four rows, each against the key of
// the row before.
//
// Bound by one wave's latency (1024 chains are one wave per SIMD): about 3100 cycles per round of
// up to four. 10 requests in batches of 4, 1024 chains x 6300 proposals under the paper's
// schedule and ratio objective: 2.08 ms, the register kernel 3.24 ms. (With trees for cooler
// chains, as in anneal_cont_spec.h, the decisions' scalar code outweighs the 2.3 proposals a
// round then completes: 1.2 ms against 1.0 ms at 59 % kept.)
#pragma once
#include "anneal_reg.h"

namespace sa {

__device__ __forceinline__ uint64_t nib_from(int i) { return ~uint64_t(0) << (4 * i); }               // nibbles i ..
__device__ __forceinline__ uint64_t nib_after(int i) { return (~uint64_t(0) << (4 * i)) << 4; }        // nibbles i + 1 ..

// The order after a move packed as ProposalStream packs it: a swap, or an insert whose
// positions between move by one towards i.
__device__ __forceinline__ uint64_t nib_move(uint64_t v, uint32_t pk) {
  const int i = (int)(pk & 1023u), j = (int)((pk >> 10) & 1023u);
  const bool swap = ((pk >> 20) & 1u) == 0u;
  const uint64_t x = (v >> (4 * i)) & 15u, y = (v >> (4 * j)) & 15u;
  const int lo = min(i, j), hi = max(i, j);
  const uint64_t in = nib_from(lo) & ~nib_after(hi);  // positions lo .. hi
  const uint64_t ends = (uint64_t(15) << (4 * i)) | (uint64_t(15) << (4 * j));
  const uint64_t moved = i < j ? v >> 4 : v << 4;
  const uint64_t mid = swap ? (v & in & ~ends) | (y << (4 * i)) : moved & in & ~(uint64_t(15) << (4 * j));
  return (v & ~in) | mid | (x << (4 * j));
}

// inclusive add-scan within each 16-lane row
__device__ __forceinline__ uint32_t row_scan32(uint32_t v) {
  v += dpp_old<kDppRowShr1, 0xF>(0u, v);
  v += dpp_old<kDppRowShr2, 0xF>(0u, v);
  v += dpp_old<kDppRowShr4, 0xF>(0u, v);
  v += dpp_old<kDppRowShr8, 0xF>(0u, v);
  return v;
}

// Replay of four orders, one per row, with a 32-bit timeline: the ballot of the requests that
// meet their SLO, and the row's latency sum as two 16-bit-half sums on every lane. b0, b1: the
// lane's batch bounds (lanes at or above n in the row: themselves), for kRegAny.
template <int LG>
__device__ __forceinline__ uint64_t row_replay(const RegState &s, bool valid, int b0, int b1, int maxb, uint32_t d0,
                                               uint32_t d2, int lane, uint32_t &lo, uint32_t &hi) {
  const uint32_t L = s.A & 0xFFFFu, e = s.E & 0x3FFFFFFFu, kind = s.E >> 30;
  uint32_t ttft, dec;  // time to first token, decode time
  if constexpr (LG >= 0) {
    const uint32_t acc = mad24_v(L, mad24_v(d2, L, e), pair_sum_others<LG>(L, e, d2, lane));
    const uint32_t P = Seg<LG>::template all<OpAdd>(s.PF, lane);
    dec = valid ? __umul24(L, d0) + (acc >> 1) : 0u;
    const uint32_t D = Seg<LG>::template all<OpMax>(valid ? P + dec : 0u, lane);
    // the batch durations up to the lane's batch (the same on every lane of a batch)
    uint32_t v = D;
    if constexpr (LG <= 0) v += dpp_old<kDppRowShr1, 0xF>(0u, v);
    if constexpr (LG <= 1) v += dpp_old<kDppRowShr2, 0xF>(0u, v);
    if constexpr (LG <= 2) v += dpp_old<kDppRowShr4, 0xF>(0u, v);
    if constexpr (LG <= 3) v += dpp_old<kDppRowShr8, 0xF>(0u, v);
    ttft = v - D + P;
  } else {
    const uint32_t pend = bperm(row_scan32(s.PF), b1);
    const int bl = b1 - b0 + 1;
    const uint32_t acc = maxb <= 8 ? pair_round<8>(L, e, d2, b0, bl, 0, 0u) : pair_round<16>(L, e, d2, b0, bl, 0, 0u);
    dec = valid ? __umul24(L, d0) + (acc >> 1) : 0u;
    uint32_t v = dec;  // the batch's longest decode at its last lane
    v = max(v, dpp_old<kDppRowShr1, 0xF>(0u, b1 >= lane + 1 ? v : 0u));
    v = max(v, dpp_old<kDppRowShr2, 0xF>(0u, b1 >= lane + 2 ? v : 0u));
    v = max(v, dpp_old<kDppRowShr4, 0xF>(0u, b1 >= lane + 4 ? v : 0u));
    v = max(v, dpp_old<kDppRowShr8, 0xF>(0u, b1 >= lane + 8 ? v : 0u));
    const uint32_t contrib = valid && lane == b1 ? v : 0u;
    ttft = pend + row_scan32(contrib) - contrib;
  }
  const uint32_t e2e = ttft + dec, x = kind == 0 ? ttft : (kind == 2 ? e2e : dec);
  lo = valid ? (e2e & 0xFFFFu) : 0u;
  hi = valid ? (e2e >> 16) : 0u;
  Seg<4>::template all2<OpAdd, OpAdd>(lo, hi, lane);
  return __ballot(valid && x <= s.T);
}

// One chain by one wave: record slot `chain`, Philox chain index `rng_chain`; n <= 16.
template <int LG, int OBJ>
__device__ void anneal_row16_body(const DevModel &m, const QueuePtrs &q, int chains, int chain, uint32_t rng_chain,
                                  int iters, double T0, double alpha, uint32_t key0, uint32_t key1, uint64_t swap_thr,
                                  const SearchParams &srch, unsigned char *ws) {
  const int n = m.n, B = m.B;
  const int lane = lane_id(), pos = lane & 15, row = lane >> 4;
  const bool valid = pos < n;
  const uint32_t d0 = (uint32_t)m.d0, d2 = (uint32_t)m.d2;
  const int b0 = valid ? lane - pos % B : lane, b1 = valid ? lane - pos + min(pos / B * B + B, n) - 1 : lane;
  const int maxb = min(B, n);
  const WsHeader *h = reinterpret_cast<const WsHeader *>(ws);
  const int64_t t_ref = h->t_ref;
  const int64_t allmet = h->allmet;
  const uint16_t *start = reinterpret_cast<const uint16_t *>(ws + ws_off_start());
  const size_t stride = ws_perm_stride(n);
  uint16_t *gbest = reinterpret_cast<uint16_t *>(ws + ws_off_best(n, chains)) + (size_t)chain * stride;
  uint16_t *gcur = reinterpret_cast<uint16_t *>(ws + ws_off_cur(n, chains)) + (size_t)chain * stride;
  // request `pos` in every row (zeros past the last: positions at or above n keep their own index)
  RegState req{0u, 0u, 0u, 0u};
  if (valid) {
    const uint32_t lin = q.in_len[pos], L = q.out_len[pos], kind = q.kind[pos], thr = q.thr[pos];
    const uint32_t e = (uint32_t)(2 * (m.d1 + m.d2 * lin) + m.d2);
    const uint64_t thr_l = (uint64_t)thr * L;
    req.A = L;
    req.E = e | (kind << 30);
    req.PF = (uint32_t)(m.p0 + m.p1 * lin);
    req.T = kind == 1 ? (uint32_t)min(thr_l, (uint64_t)0xFFFFFFFFu) : thr;
  }
  uint64_t ord = 0xFEDCBA9876543210ull;
  {
    const uint32_t r = valid ? start[pos] : (uint32_t)pos;
    if (lane < n) gbest[lane] = (uint16_t)r;
    for (int p = 0; p < n; ++p) ord = (ord & ~(uint64_t(15) << (4 * p))) | ((uint64_t)rl(r, p) << (4 * p));
  }
  // the lane's value of one of four per-row scalars
  auto by_row = [&](uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return row < 2 ? (row == 0 ? a : b) : (row == 2 ? c : d); };
  auto id_at = [&](uint64_t a, uint64_t b, uint64_t c, uint64_t d) {
    const uint32_t w = pos < 8 ? by_row((uint32_t)a, (uint32_t)b, (uint32_t)c, (uint32_t)d)
                               : by_row((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), (uint32_t)(d >> 32));
    return (w >> ((pos & 7) * 4)) & 15u;
  };
  int64_t cn = h->start_n;
  uint64_t ct = (uint64_t)h->start_t;
  int64_t bn = cn;
  uint64_t bt = ct;
  int64_t biter = -1, accepts = 0;
  uint64_t digest = kFnvOffset;
  Cooling cool{T0, alpha, srch.level_len, srch.level_len};
  ProposalStream ps;  // iterations kb .. kb + 63
  int kb = 0;
  const int iters_run = (srch.early_exit && allmet) ? 0 : iters;
  if (iters_run > 0) ps.refill(0, lane, n, rng_chain, key0, key1, swap_thr, 0);
  int k = 0;
  while (k < iters_run) {
    if (k + 3 - kb >= kWave) {
      kb = k;
      ps.refill(kb, lane, n, rng_chain, key0, key1, swap_thr, 0);
    }
    const uint64_t c0 = nib_move(ord, rl(ps.pk, k - kb));
    const uint64_t c1 = nib_move(c0, rl(ps.pk, k + 1 - kb));
    const uint64_t c2 = nib_move(c1, rl(ps.pk, k + 2 - kb));
    const uint64_t c3 = nib_move(c2, rl(ps.pk, k + 3 - kb));
    const int src = (int)(id_at(c0, c1, c2, c3) << 2);
    const RegState cand{from_lane(src, req.A), from_lane(src, req.E), from_lane(src, req.PF), from_lane(src, req.T)};
    const uint32_t w3 = from_lane((k - kb + row) << 2, ps.w3);
    uint32_t lo, hi;
    const uint64_t hit = row_replay<LG>(cand, valid, b0, b1, maxb, d0, d2, lane, lo, hi);
    const uint64_t t = (uint64_t)lo + ((uint64_t)hi << 16);
    const uint32_t n0 = (uint32_t)__builtin_popcount((uint32_t)hit & 0xFFFFu),
                   n1 = (uint32_t)__builtin_popcount((uint32_t)hit >> 16),
                   n2 = (uint32_t)__builtin_popcount((uint32_t)(hit >> 32) & 0xFFFFu),
                   n3 = (uint32_t)__builtin_popcount((uint32_t)(hit >> 48));
    const uint64_t t0 = rl64(t, 0), t1 = rl64(t, 16), t2 = rl64(t, 32), t3 = rl64(t, 48);
    // the key a row is judged against: the current one, or the row before's
    const uint32_t rn = by_row((uint32_t)cn, n0, n1, n2);
    const uint64_t rt =
        (uint64_t)by_row((uint32_t)ct, (uint32_t)t0, (uint32_t)t1, (uint32_t)t2) |
        ((uint64_t)by_row((uint32_t)(ct >> 32), (uint32_t)(t0 >> 32), (uint32_t)(t1 >> 32), (uint32_t)(t2 >> 32)) << 32);
    double T = cool.T;  // of the row's proposal
    if (cool.left <= 3) {
      Cooling c = cool;
      for (int d = 1; d < 4; ++d) {
        c.step();
        T = row >= d ? c.T : T;
      }
    }
    const uint64_t keep = __ballot(obj_accept<OBJ>((int64_t)rn, rt, (int64_t)by_row(n0, n1, n2, n3) - (int64_t)rn,
                                                   (int64_t)(t - rt), t_ref, T, w3));
    // proposals decided (up to the first rejection, at most those left) and kept
    const uint32_t bits = ((uint32_t)keep & 1u) | (((uint32_t)keep >> 15) & 2u) | (((uint32_t)(keep >> 32) << 2) & 4u) |
                          (((uint32_t)(keep >> 48) << 3) & 8u);
    const int run = __builtin_ctz(~bits), left = iters_run - k;
    const int kept = min(run, left), done = min(min(run + 1, 4), left);
    auto take = [&](int r, uint64_t c, uint32_t sn, uint64_t st) __attribute__((always_inline)) {
      ord = c;
      cn = (int64_t)sn;
      ct = st;
      digest = (digest ^ (uint64_t)(k + r)) * kFnvPrime;
      digest = (digest ^ (uint64_t)cn) * kFnvPrime;
      digest = (digest ^ ct) * kFnvPrime;
      if (obj_better<OBJ>(cn, ct, bn, bt)) {
        bn = cn;
        bt = ct;
        biter = k + r;
        const uint32_t id = id_at(c, c, c, c);
        if (lane < n) gbest[lane] = (uint16_t)id;
      }
    };
    if (kept > 0) {
      take(0, c0, n0, t0);
      if (kept > 1) {
        take(1, c1, n1, t1);
        if (kept > 2) {
          take(2, c2, n2, t2);
          if (kept > 3) take(3, c3, n3, t3);
        }
      }
    }
    accepts += kept;
    k += done;
    if (cool.left > done)
      cool.left -= done;
    else
      for (int d = 0; d < done; ++d) cool.step();
  }
  const uint32_t id = id_at(ord, ord, ord, ord);
  if (lane < n) gcur[lane] = (uint16_t)id;
  if (lane == 0) write_record(ws, n, chain, cn, ct, bn, bt, biter, accepts, digest, allmet);
}

// One wave per chain; blockDim / 64 chains per workgroup; no LDS.
template <int LG, int OBJ>
__global__ void __launch_bounds__(256) anneal_row16_kernel(DevModel m, QueuePtrs q, int chains, int iters, double T0,
                                                            double alpha, uint32_t key0, uint32_t key1,
                                                            uint64_t swap_thr, SearchParams srch, unsigned char *ws) {
  if (!gate_open(ws, m.gate, m.flags)) return;
  const int chain = uniform((int)blockIdx.x * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6));
  if (chain >= chains) return;
  anneal_row16_body<LG, OBJ>(m, q, chains, chain, (uint32_t)chain, iters, T0, alpha, key0, key1, swap_thr, srch, ws);
}

}  // namespace sa
