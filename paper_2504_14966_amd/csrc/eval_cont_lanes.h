// Evaluation of many orders under continuous admission: one order per lane (gfx950).
//
// The list-scheduling replay (device_cont.h) gives one order a wave: every admission is a
// serial step of four dependent instructions on a 64-lane list, and the prefix sums over the
// events follow. Here lane = order and the sorted list of running requests sits in CAP
// registers of the lane: popping the earliest finish and inserting the newcomer's is
// v[i] = median(v[i], v[i + 1], key) for every i, CAP independent instructions that serve 64
// orders. The timeline follows along, event by event, with no prefix sums:
//   keys   finish step << 6 | slot; the newcomer takes the popped request's slot (which of
//          two requests that finish at one step pops first changes no result);
//   slots  in LDS, [slot][lane]: the time below which the request meets its SLO when it
//          finishes, and its context at the end (l_in + l_out);
//   time   Tb, the clock at the current finish step before that step's admission group, and
//          Tend, after it: the step's first event adds the segment's cost to Tend and then the
//          prefills of the whole group, which the list already shows (the requests that finish
//          at this step are its first entries; the next three prefills are at hand in
//          registers, larger groups take a slower loop). So a newcomer's TTFT, Tend, is known
//          when it is admitted, and with it the limit its finish is compared with.
// Ids are staged in LDS 32 positions at a time (coalesced loads), records are gathered four
// events ahead. A bitmap per lane shows rows that are no permutation.
//
// 65536 orders of 256 requests, 32 running: 118 us, one order per wave 443 us. Bound by the
// issue and the LDS latency of a lone wave per SIMD (108 vector and 27 scalar instructions per
// event and 64 orders, 40 % of the cycles waiting); more rows than 64 per SIMD cost less each
// as long as the LDS and registers hold two waves (262144 rows of 256 requests, 16 running:
// 230 us, one order per wave 1642 us).
#pragma once
#include "anneal_static.h"
#include "lane_shape.h"

namespace sa {

__device__ __forceinline__ uint32_t med3_v(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

template <int CAP>
__global__ void __launch_bounds__(256) eval_cont_lanes_kernel(DevModel m, QueuePtrs q, const uint16_t *__restrict__ perms,
                                                               int64_t rows, int64_t *__restrict__ out) {
  extern __shared__ __align__(16) unsigned char lds[];
  const EvalRows span = eval_gate<true>(q, m, rows, out);
  if (span.end <= span.begin) return;
  const int n = m.n, n0 = min(m.B, n), nadm = n - n0, lane = lane_id();
  const uint32_t d0 = (uint32_t)m.d0, d1 = (uint32_t)m.d1, d2 = (uint32_t)m.d2;
  constexpr uint32_t kInf = 0xFFFFFFFFu;
  // by id: l_in | l_out << 16; prefill | TPOT << 31; limit at the finish (end to end: thr + 1;
  // TPOT: thr l_out + 1 past the TTFT; TTFT: 0); limit of the TTFT (TTFT: thr + 1, else 0)
  uint4 *rec = reinterpret_cast<uint4 *>(lds);
  for (int r = threadIdx.x; r < n; r += blockDim.x) {
    const uint32_t lin = q.in_len[r], L = q.out_len[r], kind = q.kind[r], thr = q.thr[r];
    const uint64_t tp = (uint64_t)thr * L;
    const uint32_t fin = kind == 0 ? 0u : (kind == 1 ? (uint32_t)min(tp, (uint64_t)0xFFFFFFFEu) + 1u : thr + 1u);
    rec[r] = make_uint4(lin | (L << 16), (uint32_t)(m.p0 + m.p1 * lin) | (kind == 1 ? 0x80000000u : 0u), fin,
                        kind == 0 ? thr + 1u : 0u);
  }
  __syncthreads();
  const int wave = uniform((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
  unsigned char *wb = lds + (size_t)n * 16 + (size_t)wave * cont_lane_wave_bytes(n, CAP);
  uint2 *slots = reinterpret_cast<uint2 *>(wb);                          // [slot][lane]
  uint32_t *seen = reinterpret_cast<uint32_t *>(slots + CAP * kWave);      // [word][lane]
  uint16_t *ids = reinterpret_cast<uint16_t *>(seen + ((n + 31) >> 5) * kWave);  // [lane][position]
  const int64_t tiles = (rows + kWave - 1) / kWave;
  for (int64_t tile = (int64_t)blockIdx.x * waves + wave; tile < tiles; tile += (int64_t)gridDim.x * waves) {
    const int64_t row0 = tile * kWave;
    // ids of positions [p, p + 32) of the 64 rows (out of range past the rows and the order)
    auto stage = [&](int p) __attribute__((always_inline)) {
      wave_sync_lds();
      const int col = lane & (kContStage - 1), sub = lane / kContStage;
#pragma unroll 4
      for (int r0 = 0; r0 < kWave; r0 += 8) {
        uint16_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = r0 + 2 * u + sub;
          const int64_t row = min(row0 + r, rows - 1);
          v[u] = perms[row * n + min(p + col, n - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) ids[(r0 + 2 * u + sub) * kContIdStride + col] = v[u];
      }
      wave_sync_lds();
    };
    // record of the lane's request at position p (uniform; none past the order)
    auto record = [&](int p, bool mark) __attribute__((always_inline)) {
      if (p >= n) return make_uint4(0u, 0u, 0u, 0u);
      if ((p & (kContStage - 1)) == 0) stage(p);
      const uint32_t id = ids[lane * kContIdStride + (p & (kContStage - 1))];
      // an id out of range reads as the last one, which leaves another bit of the map clear
      const uint32_t c = min(id, (uint32_t)n - 1u);
      if (mark) atomicOr(&seen[(c >> 5) * kWave + lane], id < (uint32_t)n ? 1u << (c & 31u) : 0u);
      return rec[c];
    };
    for (int w = 0; w < (n + 31) >> 5; ++w) seen[w * kWave + lane] = 0u;
    // initial group: its prefills first (they are every member's TTFT), then its members
    uint32_t Tend = 0;
    for (int p = 0; p < n0; ++p) Tend += record(p, false).y & 0x7FFFFFFFu;
    uint32_t Tb = 0, K = 0, C = 0, met = 0;
    uint64_t t = 0;
    uint32_t v[CAP];
#pragma unroll
    for (int i = 0; i < CAP; ++i) v[i] = kInf;
    // the newcomer r takes `slot`; its TTFT is Tend
    auto admit = [&](const uint4 &r, uint32_t slot) __attribute__((always_inline)) {
      met += Tend < r.w ? 1u : 0u;
      const uint32_t lim = add_sat(r.z, (uint32_t)((int32_t)r.y >> 31) & Tend);
      const uint32_t lin = r.x & 0xFFFFu, L = r.x >> 16;
      slots[slot * kWave + lane] = make_uint2(lim, lin + L);
      C += lin;
      return ((K + L) << 6) | slot;
    };
    for (int p = 0; p < n0; ++p) {
      const uint32_t key = admit(record(p, true), (uint32_t)p);
#pragma unroll
      for (int i = CAP - 1; i > 0; --i) v[i] = med3_v(v[i - 1], v[i], key);
      v[0] = min(v[0], key);
    }
    // event k (1 .. n): the earliest finish, and the admission of position n0 + k - 1. r is its
    // record, a1 .. a3 the next three, and r is refilled with the one four events ahead.
    auto event = [&](int k, uint4 &r, const uint4 &a1, const uint4 &a2, const uint4 &a3) __attribute__((always_inline)) {
      const uint32_t key = v[0], slot = key & 63u, f = key >> 6;
      const uint2 own = slots[slot * kWave + lane];
      const uint32_t b = (uint32_t)min(n0, n - k + 1);
      const uint32_t s = f - K;
      const bool adv = s != 0u;
      const uint32_t x = mad24_v(d2, C, d0 + d1 * b);
      const uint32_t tri = __umul24(s, s + 1u) >> 1;
      const uint32_t at = mad24_v(d2 * b, tri, mad24_v(s, x, Tend));
      K = f;
      Tb = adv ? at : Tb;
      C += __umul24(b, s) - own.y;
      met += Tb < own.x ? 1u : 0u;
      t += Tb;
      uint32_t nk = kInf;
      if (k <= nadm) {
        // the step's whole admission group, at its first event
        const bool e1 = (v[1] >> 6) == f, e2 = e1 && (v[2] >> 6) == f, e3 = e2 && (v[3] >> 6) == f;
        uint32_t grp = (r.y & 0x7FFFFFFFu) + (e1 ? a1.y & 0x7FFFFFFFu : 0u) + (e2 ? a2.y & 0x7FFFFFFFu : 0u) +
                       (e3 ? a3.y & 0x7FFFFFFFu : 0u);
        if (CAP > 4) {
          bool more = adv && e3 && (v[4] >> 6) == f;
          if (__ballot(more) != 0ull) {
            for (int j = 4; j < CAP && __ballot(more) != 0ull; ++j) {
              const int p = n0 + k - 1 + j;
              if (p >= n) break;
              uint32_t vj = kInf;
#pragma unroll
              for (int i = 4; i < CAP; ++i) vj = i == j ? v[i] : vj;
              more = more && (vj >> 6) == f;
              // (read from memory: the staged ids are the next four's)
              const uint32_t id = perms[min(row0 + lane, rows - 1) * n + p];
              grp += more ? rec[min(id, (uint32_t)n - 1u)].y & 0x7FFFFFFFu : 0u;
            }
          }
        }
        Tend = adv ? Tb + grp : Tend;
        nk = admit(r, slot);
        r = record(n0 + k + 3, true);
      } else {
        Tend = adv ? Tb : Tend;
      }
#pragma unroll
      for (int i = 0; i + 1 < CAP; ++i) v[i] = med3_v(v[i], v[i + 1], nk);
      v[CAP - 1] = max(v[CAP - 1], nk);
    };
    uint4 r0 = record(n0, true), r1 = record(n0 + 1, true), r2 = record(n0 + 2, true), r3 = record(n0 + 3, true);
    for (int k = 1; k <= n; k += 4) {
      event(k, r0, r1, r2, r3);
      if (k + 1 <= n) event(k + 1, r1, r2, r3, r0);
      if (k + 2 <= n) event(k + 2, r2, r3, r0, r1);
      if (k + 3 <= n) event(k + 3, r3, r0, r1, r2);
    }
    bool ok = true;  // every request seen
    for (int w = 0; w < (n + 31) >> 5; ++w) {
      const uint32_t all = n - 32 * w >= 32 ? 0xFFFFFFFFu : (1u << (n - 32 * w)) - 1u;
      ok &= seen[w * kWave + lane] == all;
    }
    if (row0 + lane < rows) {
      out[2 * (row0 + lane)] = ok ? (int64_t)met : -1;
      out[2 * (row0 + lane) + 1] = ok ? (int64_t)t : -1;
    }
  }
}

}  // namespace sa
