// Evaluation of many static-admission orders at once: one order per lane (gfx950).
//
// eval_static_kernel and eval_sized_kernel score one order per wave, and spend their time on
// the pair costs of each batch (B - 1 of them per member). Scoring 64 orders per wave, lane =
// order, makes the requests the wave-uniform loop: taken in ascending and then descending
// output length, every member's pair costs follow from three running sums of its batch.
// With h_j = w(j, L_j) / 2 (w the doubled pair cost of the delta kernels) and the members of
// i's batch split into those at least as long as i (already seen in descending order:
// E = sum of d1 + d2 l_j, cnt of them) and the rest, i included, the finish offset is
//   F_i = P + L_i d0 + sum_{rest} h_j + L_i E + cnt q_i,   q_i = d2 L_i (L_i + 1) / 2.
// Offsets grow with the output length, so the duration of a batch is the offset of its
// longest member, P + L_max d0 + sum of all h_j. Per 64 orders:
//   scatter     the ids of the 64 rows (contiguous in memory, 16-byte loads, four in flight)
//               turn into inv[request][order] = batch index, one byte (a request that never
//               appears keeps the spare index: the row is no permutation);
//   ascending   each request adds (h, prefill) to its batch's entry of the lane, one 64-bit
//               LDS add, and stores its output length (the last store is the longest);
//   starts      a serial pass over the batches: T0 = start + P, and the entry becomes
//               (U = sum of h, W = cnt << 24 | E = 0);
//   descending  one 64-bit LDS add with return per request reads (U, W) and moves the
//               request from the rest to the seen ones; F - P - L d0 = U + L E + cnt q.
// The LDS reads and adds of eight consecutive requests are in flight together (the adds
// commute, so nothing waits for an earlier request's result). Entries are [batch][lane]: no
// bank conflicts but those of the scatter (rows of 68 bytes spread it over the banks). The
// per-request constants come as 16-byte LDS broadcasts, which costs the least issue: v_readlane
// of the five fields and the scalar work on them took a third of the descending loop (302 us
// where this takes 250 us). Two orders per lane, which share that work, lose more by the halved
// occupancy (426 us against 302 us).
//
// 2^20 orders of 128 requests, batches of 16: 250 us, one order per wave 552 us; with layouts
// of about 15 batches 446 us against 1890 us. Bound by the LDS (its unit active 60 % of the
// cycles, 28 vector instructions per request and 64 orders issue in 40 %) at the two waves per
// SIMD that 15.7 KB per wave allow (layouts: one).
//
// Widths (kFlagEvalLaneSums, on top of the static widths and the 32-bit timeline): E of a
// batch and q below 2^24.
#pragma once
#include <type_traits>

#include "anneal_sized.h"
#include "lane_shape.h"

namespace sa {

constexpr int kLaneDepth = 8;  // requests whose LDS accesses are in flight together

// Start bits of the tile's layouts, their running counts per 32-position word, and the number
// of batches of the lane's row (0: not a valid layout).
__device__ __forceinline__ int lane_layouts(const uint8_t *__restrict__ src, int n, int B, int rows, uint32_t nmagic,
                                            uint32_t *bits, uint32_t *before, uint32_t *badrow) {
  const int lane = lane_id(), W = lane_words(n), words = (n + 31) >> 5;
  for (int w = 0; w < W; ++w) bits[w * kWave + lane] = 0u;
  badrow[lane] = 0u;
  wave_sync_lds();
  const int total = rows * n, chunks = total >> 4;
  // `len` flags from position x of the tile on (their low bits in `mask`), one row at a time,
  // at most two words each
  auto put = [&](int x, int len, uint32_t mask) {
    int o = (int)__umulhi((uint32_t)x, nmagic), p = x - o * n;
    while (len > 0) {
      const int c = min(len, n - p), w = p >> 5, sh = p & 31;
      const uint32_t part = mask & ((1u << c) - 1u);
      atomicOr(&bits[w + o * W], part << sh);
      if (sh + c > 32) atomicOr(&bits[w + 1 + o * W], part >> (32 - sh));
      mask >>= c;
      len -= c;
      p = 0;
      ++o;
    }
  };
  for (int c0 = 0; c0 < chunks; c0 += 4 * kWave) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = *reinterpret_cast<const uint4 *>(src + 16 * min(c0 + u * kWave + lane, chunks - 1));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * kWave + lane;
      if (c >= chunks) continue;
      // the low bits of four flags to four bits
      auto four = [](uint32_t w) { return ((w & 0x01010101u) * 0x10204080u) >> 28; };
      put(16 * c, 16, four(v[u].x) | (four(v[u].y) << 4) | (four(v[u].z) << 8) | (four(v[u].w) << 12));
      if ((v[u].x | v[u].y | v[u].z | v[u].w) & 0xFEFEFEFEu) {  // a flag above 1 makes its row invalid
        for (int i = 0; i < 16; ++i)
          if (src[16 * c + i] > 1u) badrow[(int)__umulhi((uint32_t)(16 * c + i), nmagic)] = 1u;
      }
    }
  }
  for (int x = 16 * chunks + lane; x < total; x += kWave) {  // a partial tile's last flags
    const uint32_t f = src[x];
    put(x, 1, f & 1u);
    if (f > 1u) badrow[(int)__umulhi((uint32_t)x, nmagic)] = 1u;
  }
  wave_sync_lds();
  // lane = row: counts before each word, and no B positions in a row without a start
  int count = 0, run = 0;
  bool bad = lane >= rows || badrow[lane] != 0u || (bits[lane * W] & 1u) == 0u;
  for (int w = 0; w < words; ++w) {
    const uint32_t v = bits[lane * W + w];
    const int len = min(32, n - 32 * w);
    before[lane * W + w] = (uint32_t)count;
    count += __popc(v);
    const int first = v ? __builtin_ctz(v) : len;
    bad |= run + first >= B;
    if (B <= 32) {
      // positions of the word without a start, and of them those that end B in a row
      uint32_t z = ~v & (len < 32 ? (1u << len) - 1u : 0xFFFFFFFFu);
      int have = 1;
      while (2 * have <= B) {
        z &= z >> have;
        have *= 2;
      }
      if (have < B) z &= z >> (B - have);
      bad |= z != 0u;
    }
    run = v ? len - 1 - (31 - __builtin_clz(v)) : run + len;
  }
  wave_sync_lds();
  return bad ? 0 : count;
}

template <bool LAYOUT>
__global__ void __launch_bounds__(256) eval_lanes_kernel(DevModel m, QueuePtrs q, const uint16_t *__restrict__ perms,
                                                          const uint8_t *__restrict__ starts, int64_t rows,
                                                          int64_t *__restrict__ out, int mcap) {
  extern __shared__ __align__(16) unsigned char lds[];
  const EvalRows span = eval_gate<true>(q, m, rows, out);
  if (span.end <= span.begin) return;
  const int n = m.n, B = m.B, lane = lane_id();
  const uint32_t d0 = (uint32_t)m.d0, d1 = (uint32_t)m.d1, d2 = (uint32_t)m.d2;
  // requests by ascending output length. ta: inv offset, h, prefill, L. tb: inv offset, the
  // 64-bit step (-h, +1 << 24 | e), limit. tc: L, q, masks of F and T0 in the compared time.
  uint4 *ta = reinterpret_cast<uint4 *>(lds), *tb = ta + n, *tc = tb + n;
  uint4 *req = tc + n;  // by id, layouts only
  uint32_t *by_id = reinterpret_cast<uint32_t *>(lds + lane_shared_bytes(n, LAYOUT));  // in the first wave's space
  for (int r = threadIdx.x; r < n; r += blockDim.x) by_id[r] = ((uint32_t)q.out_len[r] << 10) | (uint32_t)r;
  __syncthreads();
  for (int r = threadIdx.x; r < n; r += blockDim.x) {
    const uint32_t L = q.out_len[r], lin = q.in_len[r], kind = q.kind[r], thr = q.thr[r];
    const uint32_t key = (L << 10) | (uint32_t)r;
    int rank = 0;  // shorter requests, ties by id
    for (int j = 0; j < n; ++j) rank += by_id[j] < key ? 1 : 0;
    const uint32_t e = d1 + d2 * lin, tri = d2 * (uint32_t)(((uint64_t)L * (L + 1)) >> 1), h = L * e + tri;
    ta[rank] = make_uint4((uint32_t)(r * kLaneInvStride), h, (uint32_t)(m.p0 + m.p1 * lin), L);
    const uint64_t step = ((uint64_t)(e | (1u << 24)) << 32) - h;
    // met iff the compared time, without the request's own L d0 where F is in it, is below the
    // limit (a TPOT threshold of 2^32 - 1 or more always holds: F < 2^32 - 1)
    const uint64_t bound = (kind == 1 ? min((uint64_t)thr * L, (uint64_t)0xFFFFFFFEu) : (uint64_t)thr) + 1;
    const uint64_t own = kind == 0 ? 0ull : (uint64_t)L * d0;
    tb[rank] = make_uint4((uint32_t)(r * kLaneInvStride), (uint32_t)step, (uint32_t)(step >> 32),
                          bound > own ? (uint32_t)(bound - own) : 0u);
    tc[rank] = make_uint4(L, tri, kind == 0 ? 0u : ~0u, kind == 1 ? 0u : ~0u);
    if constexpr (LAYOUT) req[r] = make_uint4(lin | (L << 16), thr, kind, 0u);
  }
  __syncthreads();
  uint64_t own_sum = 0;  // sum of L d0
  for (int r = lane; r < n; r += kWave) own_sum += (uint64_t)ta[r].w * d0;
  own_sum = wave_sum_u64(own_sum);
  const int wave = uniform((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
  unsigned char *wb = lds + lane_shared_bytes(n, LAYOUT) + (size_t)wave * lane_wave_bytes(n, mcap, LAYOUT);
  const size_t inv_b = lane_inv_bytes(n);
  uint8_t *inv = wb;
  uint64_t *ent = reinterpret_cast<uint64_t *>(wb + inv_b);                       // [batch][order]
  uint32_t *t0 = reinterpret_cast<uint32_t *>(ent + (size_t)(mcap + 1) * kWave);  // [batch][order]
  uint32_t *bits = t0 + (size_t)(mcap + 1) * kWave, *before = bits + kWave * lane_words(n);
  uint32_t *badrow = before + kWave * lane_words(n);
  const int W = lane_words(n);
  const uint32_t nmagic = (uint32_t)((1ull << 32) / (uint32_t)n) + 1u;  // x / n for x < 2^16, n > 1
  const uint32_t bmagic = (65536u + (uint32_t)B - 1u) / (uint32_t)B;    // p / B for p B < 2^16
  const int64_t tiles = (rows + kWave - 1) / kWave;
  for (int64_t tile = (int64_t)blockIdx.x * waves + wave; tile < tiles; tile += (int64_t)gridDim.x * waves) {
    const int64_t row0 = tile * kWave;
    const int nr = (int)min((int64_t)kWave, rows - row0), total = nr * n, chunks = total >> 3;
    int M = (n + B - 1) / B;  // batches of the lane's order
    if constexpr (LAYOUT) M = lane_layouts(starts + row0 * n, n, B, nr, nmagic, bits, before, badrow);
    // every request in the spare batch, empty entries
    const uint32_t spare = (uint32_t)mcap * 0x01010101u;
    for (size_t x = (size_t)lane * 16; x < inv_b; x += kWave * 16)
      *reinterpret_cast<uint4 *>(inv + x) = make_uint4(spare, spare, spare, spare);
    for (size_t x = (size_t)lane * 16; x < (size_t)(mcap + 1) * (kWave * 12); x += kWave * 16)
      *reinterpret_cast<uint4 *>(reinterpret_cast<unsigned char *>(ent) + x) = make_uint4(0u, 0u, 0u, 0u);
    wave_sync_lds();
    const uint16_t *src = perms + row0 * n;
    // batch of position p of order o (bits and count of its word for layouts)
    auto batch_of = [&](int p, uint32_t wbits, uint32_t wcount) {
      if constexpr (LAYOUT)
        return min(wcount + (uint32_t)__popc(wbits & ((2u << (p & 31)) - 1u)) - 1u, (uint32_t)mcap);
      else
        return __umul24((uint32_t)p, bmagic) >> 16;
    };
    auto put = [&](uint32_t id, int o, uint32_t b) {
      inv[__umul24(min(id, (uint32_t)n), (uint32_t)kLaneInvStride) + (uint32_t)o] = (uint8_t)b;
    };
    for (int c0 = 0; c0 < chunks; c0 += 4 * kWave) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = *reinterpret_cast<const uint4 *>(src + 8 * min(c0 + u * kWave + lane, chunks - 1));
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = c0 + u * kWave + lane;
        if (c >= chunks) continue;
        int o = (int)__umulhi((uint32_t)(8 * c), nmagic), p = 8 * c - o * n;
        uint32_t wbits = 0, wcount = 0;
        auto word = [&]() {
          if constexpr (LAYOUT) {
            wbits = bits[o * W + (p >> 5)];
            wcount = before[o * W + (p >> 5)];
          }
        };
        const uint32_t ids[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
        word();
        if ((n & 7) == 0) {  // the eight positions lie in one row, and there in one 32-position word
          const bool one = !LAYOUT && (B & 7) == 0;  // and then in one batch of the maximum size
          const uint32_t b0 = batch_of(p, wbits, wcount);
#pragma unroll
          for (int i = 0; i < 8; ++i)
            put((i & 1) ? ids[i >> 1] >> 16 : ids[i >> 1] & 0xFFFFu, o, one ? b0 : batch_of(p + i, wbits, wcount));
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            if (i > 0 && (p & 31) == 0) word();
            put((i & 1) ? ids[i >> 1] >> 16 : ids[i >> 1] & 0xFFFFu, o, batch_of(p, wbits, wcount));
            if (++p == n) {
              p = 0;
              o = min(o + 1, kWave - 1);
            }
          }
        }
      }
    }
    for (int x = 8 * chunks + lane; x < total; x += kWave) {  // a partial tile's last ids
      const int o = (int)__umulhi((uint32_t)x, nmagic), p = x - o * n;
      uint32_t wbits = 0, wcount = 0;
      if constexpr (LAYOUT) {
        wbits = bits[o * W + (p >> 5)];
        wcount = before[o * W + (p >> 5)];
      }
      put(src[x], o, batch_of(p, wbits, wcount));
    }
    wave_sync_lds();
    // ascending output length: (h, prefill) sums and the longest member of every batch
    uint32_t bmax = 0u;
    auto ascend = [&](int s, auto count) {
      constexpr int C = decltype(count)::value;
      uint4 a[C];
      uint32_t b[C];
#pragma unroll
      for (int u = 0; u < C; ++u) a[u] = ta[s + u];
#pragma unroll
      for (int u = 0; u < C; ++u) b[u] = inv[a[u].x + (uint32_t)lane];
#pragma unroll
      for (int u = 0; u < C; ++u) {
        bmax = max(bmax, b[u]);
        const uint32_t at = b[u] * kWave + (uint32_t)lane;
        __hip_atomic_fetch_add(&ent[at], ((uint64_t)a[u].z << 32) | a[u].y, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WAVEFRONT);
        t0[at] = a[u].w;
      }
    };
    int s = 0;
    for (; s + kLaneDepth <= n; s += kLaneDepth) ascend(s, std::integral_constant<int, kLaneDepth>{});
    for (; s < n; ++s) ascend(s, std::integral_constant<int, 1>{});
    wave_sync_lds();
    const bool ok = lane < nr && bmax < (uint32_t)mcap && M > 0 && M <= mcap;
    // starts of the batches (empty ones past the lane's last have no duration)
    {
      uint32_t S = 0;
      for (int b = 0; b < mcap; ++b) {
        const uint64_t v = ent[b * kWave + lane];
        const uint32_t H = (uint32_t)v, P = (uint32_t)(v >> 32), L = t0[b * kWave + lane];
        ent[b * kWave + lane] = H;
        t0[b * kWave + lane] = S + P;
        S += P + H + L * d0;
      }
    }
    wave_sync_lds();
    // descending output length: latency and SLO of every request
    int met = 0;
    uint64_t t = own_sum;
    auto descend = [&](int s, auto count) {
      constexpr int C = decltype(count)::value;
      uint4 a[C], c[C];
      uint32_t b[C], T[C];
      uint64_t v[C];
#pragma unroll
      for (int u = 0; u < C; ++u) a[u] = tb[s - u];
#pragma unroll
      for (int u = 0; u < C; ++u) b[u] = inv[a[u].x + (uint32_t)lane];
#pragma unroll
      for (int u = 0; u < C; ++u) c[u] = tc[s - u];
#pragma unroll
      for (int u = 0; u < C; ++u) {
        const uint32_t at = b[u] * kWave + (uint32_t)lane;
        v[u] = __hip_atomic_fetch_add(&ent[at], ((uint64_t)a[u].z << 32) | a[u].y, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WAVEFRONT);
        T[u] = t0[at];
      }
#pragma unroll
      for (int u = 0; u < C; ++u) {
        const uint32_t w = (uint32_t)(v[u] >> 32);  // the product takes its low 24 bits
        const uint32_t f = mad24_v(c[u].x, w, mad24_v(w >> 24, c[u].y, (uint32_t)v[u]));
        met += (f & c[u].z) + (T[u] & c[u].w) < a[u].w ? 1 : 0;
        t += f;
      }
    };
    s = n - 1;
    for (; s + 1 >= kLaneDepth; s -= kLaneDepth) descend(s, std::integral_constant<int, kLaneDepth>{});
    for (; s >= 0; --s) descend(s, std::integral_constant<int, 1>{});
    wave_sync_lds();
    // every member's T0: the entries hold the batch sizes now
    for (int b = 0; b < mcap; ++b)
      t += (uint64_t)t0[b * kWave + lane] * (uint32_t)(ent[b * kWave + lane] >> 56);
    wave_sync_lds();
    if (lane < nr) {
      out[2 * (row0 + lane)] = ok ? (int64_t)met : -1;
      out[2 * (row0 + lane) + 1] = ok ? (int64_t)t : -1;
    }
    if constexpr (LAYOUT) {
      // valid layouts of more batches than the entries hold: one order at a time
      uint64_t more = __ballot(M > mcap);
      while (more) {
        const int64_t row = row0 + __builtin_ctzll(more);
        more &= more - 1;
        eval_sized_row<false>(m, req, perms + row * n, starts + row * n, wb, out + 2 * row, nullptr);
      }
      wave_sync_lds();
    }
  }
}

}  // namespace sa
