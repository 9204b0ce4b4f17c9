// Continuous admission with several proposals scored per round (speculation).
//
// Algorithm 1 scores one proposal at a time against the current order. Which order proposal
// k + d meets depends only on which of the d proposals before it are kept, so a round scores
// W proposals at once, one per wave of the chain's workgroup: wave 0 proposal k, every other
// wave a later proposal under one assumed outcome of the ones before it (a node of the tree
// of outcomes, kSpecTree). After a workgroup barrier all waves take the same decisions from
// the scores, node by node, until an outcome was not assumed by any wave. The trajectory,
// accept count, digest and best order are those of scoring one proposal at a time. The nodes
// are the W most probable ones for the chain's recent rate of acceptance (a running mean).
//
// The replay is the list-scheduling one with 32-bit times (the running requests in a sliding
// window when at most 32 run, else one pop per step from lane 0), restarted at the chunk of
// admissions holding the candidate's first change; it is bound by the latency and issue of
// its own serial steps, so the further waves of a chain work in issue slots that the SIMDs
// would otherwise leave empty. The waves meet once per round at the workgroup barrier, and
// once more when a move is accepted (the first wave applies the moves to the shared records
// before any wave replays again).
//
// Candidate records are read from the current order's records through a position map, so one
// copy of them serves all waves. LDS per
// chain: those records (16 B per position, request id above the kind bits), per wave four
// 32-bit arrays of n + 1 entries (prefill prefix sums, run starts, run-end prefills,
// segment-cost prefix sums, overwritten by the TTFTs), W + 1 sets of admission pops plus chunk-start keys (the
// current order's and one per wave), and the waves' scores in two slots used in alternate
// rounds. The request table is not staged in LDS: each chain reads its start order's records
// once from global memory.
#pragma once

#include "kernels.h"

namespace sa {

// Candidate position p reads current position src(p), without branches: position j reads
// i, and the positions in [rlo, rlo + rspan) read p + dir. An insert (remove at i,
// re-insert at j) shifts the positions between i and j by one towards i; a swap is the
// one-position range {i} reading j; the identity has no j and an empty range.
struct SrcMap {
  int j, ito, rlo, dir;
  uint32_t rspan;
  __device__ __forceinline__ int src(int p) const {
    const int shifted = (uint32_t)(p - rlo) < rspan ? p + dir : p;
    return p == j ? ito : shifted;
  }
};

__device__ __forceinline__ SrcMap src_map(int kind, int i, int j) {
  if (kind == 0 || i == j) return SrcMap{-1, 0, 0, 0, 0u};
  if (kind == 1) return SrcMap{j, i, i, j - i, 1u};
  if (i < j) return SrcMap{j, i, i, 1, (uint32_t)(j - i)};
  return SrcMap{j, i, j + 1, -1, (uint32_t)(i - j)};
}

// one wave's four arrays of n + 1 entries
__host__ __device__ __forceinline__ size_t spec_cand_bytes(int n) { return ((size_t)16 * (n + 1) + 15) / 16 * 16; }
// Admissions per chunk and running keys kept per chunk start: with at most 32 running, the
// sliding window's 64 - n0 admissions and 32 keys; with more, 64 admissions and n0 keys.
__host__ __device__ __forceinline__ int spec_chunk_len(int n0) { return n0 <= 32 ? 64 - n0 : 64; }
__host__ __device__ __forceinline__ int spec_snap_len(int n0) { return n0 <= 32 ? 32 : n0; }
// chunk-start keys of one order
__host__ __device__ __forceinline__ size_t spec_chunk_bytes(int n, int B) {
  const int n0 = n < B ? n : B, nadm = n - n0;
  const int S = spec_chunk_len(n0);
  return nadm > 0 ? (size_t)((nadm + S - 1) / S) * spec_snap_len(n0) * 4 : 0;
}
__host__ __device__ __forceinline__ size_t spec_pop_bytes(int n) { return ((size_t)4 * n + 15) / 16 * 16; }
// Nodes of the tree of outcomes, most probable first: proposal depth << 8 | outcomes of the
// proposals before it (bit d: proposal d kept), for acceptance rates around 0.1, 0.3, 0.5, 0.7
// and 0.9. Every prefix of a row holds its own ancestors, so the first W serve W waves. Mean
// proposals completed per round by 2, 4 and 8 waves: 1.9, 3.4 and 5.7 at 0.1 (and 0.9), 1.7, 2.5
// and 3.5 at 0.3 (and 0.7), 1.5, 2.25 and 3.1 at 0.5.
constexpr int kSpecWavesMax = 8;
__device__ __constant__ const uint16_t kSpecTree[5][kSpecWavesMax] = {
    {0x000, 0x100, 0x200, 0x300, 0x400, 0x500, 0x600, 0x700},
    {0x000, 0x100, 0x200, 0x300, 0x101, 0x400, 0x201, 0x202},
    {0x000, 0x100, 0x101, 0x200, 0x202, 0x201, 0x203, 0x300},
    {0x000, 0x101, 0x203, 0x307, 0x100, 0x40f, 0x202, 0x201},
    {0x000, 0x101, 0x203, 0x307, 0x40f, 0x51f, 0x63f, 0x77f}};

// scores exchanged per round: 2 slots x W waves x 32 B
__host__ __device__ __forceinline__ size_t spec_xch_bytes(int W) { return (size_t)64 * W; }
// LDS of one chain (one workgroup of W waves)
__host__ __device__ __forceinline__ size_t spec_chain_bytes(int n, int B, int W) {
  return spec_xch_bytes(W) + (size_t)16 * n + W * spec_cand_bytes(n) +
         (W + 1) * (spec_pop_bytes(n) + spec_chunk_bytes(n, B)) + (W > 2 ? (size_t)W * (((size_t)2 * n + 15) / 16 * 16) : 0);
}

// Two waves: the second one's candidate may stand on the first one's move.
struct SrcPair {
  SrcMap own, under;
  __device__ __forceinline__ int src(int p) const { return under.src(own.src(p)); }
};
// With more waves than two a candidate may stand on several moves: its positions map through
// an index array of its own (one more LDS read per lookup; maps in registers, one per move,
// cost seven instructions each and their scalars spill).
struct SrcIndex {
  const uint16_t *idx;
  __device__ __forceinline__ int src(int p) const { return (int)idx[p]; }
};

// One order's admission state: pops and chunk-start keys (whose first n0 entries are the
// initial group's sorted keys whenever a request waits), and the current order's initial
// group's prefill and context sums.
struct SpecCur {
  const uint32_t *ev, *snap;
  uint32_t pr0, c1;
};

// Score of one candidate of the current order. lo is the first position it changes:
// admissions before the window chunk holding it are the current order's. ev and snap
// receive the candidate's pops and chunk-start keys, sc holds its four arrays; pr0 and c1
// receive its initial group's sums. Every time fits 32 bits (checked on the device before
// the kernel runs).
template <class Map>
__device__ __forceinline__ Score spec_replay(const DevModel &m, const uint4 *__restrict__ posr, const Map &sm,
                                             const int lo, const SpecCur &cc, uint32_t *ev, uint32_t *snap,
                                             uint32_t *sc, uint32_t &pr0, uint32_t &c1) {
  const int lane = lane_id();
  const int N = m.n, B = m.B;
  const int n0 = min(B, N), nadm = N - n0;
  const uint32_t d0 = (uint32_t)m.d0, d1 = (uint32_t)m.d1, d2 = (uint32_t)m.d2;
  const int A = N + 1;
  uint32_t *preA = sc, *rsA = sc + A, *runpre = sc + 2 * A, *segA = sc + 3 * A;
  uint32_t *tta = segA;  // pass B leaves each event's TTFT in place of its segment-cost sum
  constexpr uint32_t kInf = 0xFFFFFFFFu;

  // initial group: positions 0 .. n0 - 1 start at step 0 (the current order's when the
  // candidate changes no position below n0)
  uint32_t list;
  if (lo >= n0) {
    list = lane < n0 ? cc.snap[lane] : kInf;
    pr0 = cc.pr0;
    c1 = cc.c1;
  } else {
    uint32_t key = kInf, lin0 = 0, pf0 = 0;
    if (lane < n0) {
      const uint4 rq = posr[sm.src(lane)];
      key = ((rq.x >> 16) << 10) | (uint32_t)lane;
      lin0 = rq.x & 0xFFFFu;
      pf0 = rq.w;
    }
    pr0 = wsum32(pf0);
    c1 = wsum32(lin0);
    int rank = 0;
    for (int u = 0; u < n0; ++u) rank += rl(key, u) < key ? 1 : 0;
    if (lane < n0) runpre[rank] = key;
    wave_sync_lds();
    list = lane < n0 ? runpre[lane] : kInf;
    wave_sync_lds();
  }

  // admissions before the chunk holding the first changed one are the current order's
  const int Sfull = spec_chunk_len(n0), SN = spec_snap_len(n0);
  const int cr = lo >= n0 ? (lo - n0) / Sfull : 0;
  int done = min(cr * Sfull, nadm);
  for (int x = lane; x < done; x += kWave) ev[x] = cc.ev[x];
  for (int x = lane; x < cr * SN; x += kWave) snap[x] = cc.snap[x];
  if (done > 0) list = lane < n0 ? cc.snap[cr * SN + lane] : kInf;
  if (n0 > 32) {
    // More than 32 running: the sorted keys fill lanes [0, n0), kInf above; a step pops
    // lane 0 and leaves lane i = max(list[i], min(list[i + 1], nk)); the pops enter lane 0
    // of a second register that moves up one lane per step.
    while (done < nadm) {
      const int cnt = min(kWave, nadm - done);
      if (lane < n0) snap[(done / kWave) * SN + lane] = list;
      uint32_t LP = 0;
      if (lane < cnt) {
        const int p = n0 + done + lane;
        LP = ((posr[sm.src(p)].x >> 16) << 10) | (uint32_t)p;
      }
      uint32_t evq = 0;
      uint32_t top = __builtin_amdgcn_readfirstlane(list);
      for (int t = 0; t < cnt; ++t) {
        const uint32_t nk = (top & ~1023u) + rl(LP, t);
        evq = dpp_old<kDppWaveShr1, 0xF>(list, evq);
        const uint32_t sh = dpp_old<kDppWaveShl1, 0xF>(kInf, list);
        list = max(list, min(sh, nk));
        top = __builtin_amdgcn_readfirstlane(list);
      }
      if (lane < cnt) ev[done + cnt - 1 - lane] = evq;
      done += cnt;
    }
  }
  // At most 32 running: a sliding window. Before step t of a chunk, lanes [0, t) hold the
  // keys popped so far and lanes [t, t + n0) the running keys, sorted, kInf above; popping
  // lane t and inserting key nk leaves lane i = median(list[i - 1], list[i], nk).
  while (done < nadm) {
    const int S = min(Sfull, nadm - done);
    if (lane < n0) snap[(done / Sfull) * 32 + lane] = list;
    uint32_t LP = 0;  // (l_out << 10) | position of the positions admitted in this chunk
    if (lane < S) {
      const int p = n0 + done + lane;
      LP = ((posr[sm.src(p)].x >> 16) << 10) | (uint32_t)p;
    }
    auto step = [&](int t) {
      const uint32_t nk = rl((list & ~1023u) + LP, t);
      const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)list, kDppWaveShr1, 0xF, 0xF, true);
      list = med3_u32(below, list, nk);
    };
    int t = 0;
    for (; t + 4 <= S; t += 4) {
      step(t);
      step(t + 1);
      step(t + 2);
      step(t + 3);
    }
    for (; t < S; ++t) step(t);
    if (lane < S) ev[done + lane] = list;
    const uint32_t moved = (uint32_t)__builtin_amdgcn_ds_bpermute((lane + S) << 2, (int)list);
    list = lane < n0 ? moved : kInf;
    done += S;
  }
  if (lane < n0) ev[nadm + lane] = list;
  if (lane == 0) preA[0] = 0u;
  wave_sync_lds();

  // pass A: segment costs, prefills, run starts and their prefix sums
  uint32_t fcarry = 0, Ccarry = c1, precarry = 0, rscarry = 0, segcarry = 0;
  for (int c0 = 0; c0 < N; c0 += kWave) {
    const int k = c0 + lane + 1;
    const bool v = k <= N;
    const uint32_t kk = v ? ev[k - 1] : 0u;
    const uint32_t f = kk >> 10;
    const int q = (int)(kk & 1023u);
    const uint32_t fprev = dpp_old<kDppWaveShr1, 0xF>(fcarry, f);
    const uint32_t s = v ? f - fprev : 0u;
    const uint32_t b = (uint32_t)min(n0, N - k + 1);
    const bool adm = v && k <= nadm;
    const uint4 rq = posr[sm.src(v ? q : 0)];
    const uint4 ra = posr[sm.src(adm ? n0 + k - 1 : 0)];
    const uint32_t outq = v ? (rq.x & 0xFFFFu) + (rq.x >> 16) : 0u;
    const uint32_t la = adm ? (ra.x & 0xFFFFu) : 0u, pfa = adm ? ra.w : 0u;
    const uint32_t dC = v ? b * s - outq + la : 0u;  // two's complement: a signed change
    const uint32_t dCi = scan_add32(dC);
    const uint32_t Ck = Ccarry + dCi - dC;
    const uint32_t seg = s * (d0 + d1 * b + d2 * Ck) + (d2 * b) * ((s * (s + 1u)) >> 1);
    const uint32_t SEG = segcarry + scan_add32(seg);
    const uint32_t PRE = precarry + scan_add32(pfa);
    const uint32_t rs = max(rscarry, scan_max32((v && (k == 1 || s != 0)) ? (uint32_t)k : 0u));
    const uint32_t fnext = k < N ? (ev[min(k, N - 1)] >> 10) : kInf;
    const int kw = v ? k : 0;
    preA[kw] = PRE;
    rsA[kw] = rs;
    segA[kw] = SEG;
    runpre[(v && (k == N || fnext != f)) ? rs : 0u] = PRE;
    fcarry = rl(f, kWave - 1);
    Ccarry += rl(dCi, kWave - 1);
    segcarry = rl(SEG, kWave - 1);
    precarry = rl(PRE, kWave - 1);
    rscarry = rl(rs, kWave - 1);
  }
  wave_sync_lds();

  // pass B: end-to-end latency of each finishing request, TTFT of each admitted one, SLOs
  uint64_t tsum = 0;
  int64_t nmet = 0;
  for (int c0 = 0; c0 < N; c0 += kWave) {
    const int k = c0 + lane + 1;
    const bool v = k <= N;
    const int kc = min(k, N);
    const uint32_t q = v ? (ev[kc - 1] & 1023u) : 0u, rsk = v ? rsA[kc] : 1u;
    const uint32_t SEG = v ? segA[kc] : 0u;
    const uint32_t e2e = pr0 + SEG + (rsk > 1 ? preA[max(rsk, 2u) - 1] : 0u);
    tta[(v && k <= nadm) ? k : 0] = pr0 + SEG + runpre[rsk];
    wave_sync_lds();
    const uint4 rq = posr[sm.src((int)q)];
    const uint32_t ttft = (int)q < n0 ? pr0 : tta[max((int)q - n0 + 1, 0)];
    const uint32_t kind = rq.z & 3u, thr = rq.y, L = rq.x >> 16;
    const bool met = v & (kind == 0 ? ttft <= thr
                                    : (kind == 2 ? e2e <= thr : (uint64_t)(e2e - ttft) <= (uint64_t)thr * L));
    tsum += v ? (uint64_t)e2e : 0ull;
    nmet += __popcll(__ballot(met));
  }
  wave_sync_lds();
  return Score{nmet, wave_sum_u64_dpp(tsum)};
}

// One chain by one workgroup of W waves: record slot `chain`, Philox chain index `rng_chain`.
template <int OBJ, int W>
__device__ void anneal_cont_spec_body(const DevModel &m, const QueuePtrs &q, unsigned char *lds, int chains, int chain,
                                      uint32_t rng_chain, int iters, double T0, double alpha, uint32_t key0,
                                      uint32_t key1, uint64_t swap_thr, const SearchParams &srch, unsigned char *ws) {
  const int n = m.n;
  const int w = uniform((int)(threadIdx.x >> 6));
  const int lane = lane_id();
  // scores of the waves, slot r & 1 in round r: {n, t, pr0 | c1 << 32, unused}
  uint64_t *xch = reinterpret_cast<uint64_t *>(lds);
  uint4 *posr = reinterpret_cast<uint4 *>(lds + spec_xch_bytes(W));
  unsigned char *base = lds + spec_xch_bytes(W) + (size_t)16 * n;
  uint32_t *sc = reinterpret_cast<uint32_t *>(base + (size_t)w * spec_cand_bytes(n));
  // W + 1 sets of pops and chunk-start keys: nibble w of `sets` is the set of wave w's
  // candidate, nibble W the current order's; accepting a candidate exchanges the two
  unsigned char *cb = base + W * spec_cand_bytes(n);
  const size_t evb = spec_pop_bytes(n), snb = spec_chunk_bytes(n, m.B);
  uint64_t sets = 0x876543210ull;
  auto set_ev = [&](int s) { return reinterpret_cast<uint32_t *>(cb + (size_t)((sets >> (4 * s)) & 15u) * evb); };
  auto set_snap = [&](int s) {
    return reinterpret_cast<uint32_t *>(cb + (W + 1) * evb + (size_t)((sets >> (4 * s)) & 15u) * snb);
  };
  auto accept_set = [&](int s) {
    const uint64_t x = ((sets >> (4 * s)) ^ (sets >> (4 * W))) & 15u;
    sets ^= (x << (4 * s)) | (x << (4 * W));
  };
  uint16_t *idx = reinterpret_cast<uint16_t *>(cb + (W + 1) * (evb + snb) + (size_t)w * (((size_t)2 * n + 15) / 16 * 16));
  if constexpr (W > 2)
    for (int p = lane; p < n; p += kWave) idx[p] = (uint16_t)p;
  const WsHeader *h = reinterpret_cast<const WsHeader *>(ws);
  const int64_t t_ref = h->t_ref;
  int64_t cn = h->start_n;
  uint64_t ct = (uint64_t)h->start_t;
  const int64_t allmet = h->allmet;
  const uint16_t *start = reinterpret_cast<const uint16_t *>(ws + ws_off_start());
  const size_t stride = ws_perm_stride(n);
  uint16_t *gbest = reinterpret_cast<uint16_t *>(ws + ws_off_best(n, chains)) + (size_t)chain * stride;
  uint16_t *gcur = reinterpret_cast<uint16_t *>(ws + ws_off_cur(n, chains)) + (size_t)chain * stride;
  // the start order's records by position, with the request id above the kind bits
  for (int p = (int)threadIdx.x; p < n; p += W * kWave) {
    const uint16_t r = start[p];
    gbest[p] = r;
    const uint32_t lin = q.in_len[r], lout = q.out_len[r];
    posr[p] = make_uint4(lin | (lout << 16), q.thr[r], (uint32_t)q.kind[r] | ((uint32_t)r << 2),
                         (uint32_t)(m.p0 + m.p1 * lin));
  }
  __syncthreads();
  // the start order's state: each wave replays it into its own buffers, the first wave's
  // become the current ones (all waves compute the same sums)
  uint32_t cur_pr0 = 0, cur_c1 = 0;
  {
    spec_replay(m, posr, src_map(0, 0, 0), 0, SpecCur{set_ev(W), set_snap(W), 0u, 0u}, set_ev(w), set_snap(w), sc, cur_pr0, cur_c1);
    accept_set(0);
  }
  __syncthreads();
  int64_t bn = cn;
  uint64_t bt = ct;
  int64_t biter = -1, accepts = 0;
  uint64_t digest = kFnvOffset;
  Cooling cool{T0, alpha, srch.level_len, srch.level_len};
  ProposalStream ps;  // iterations kb .. kb + 63
  int kb = 0, slot = 0;
  int rate = 3 << 14;  // running mean of the acceptances, of 2^16 (high at the start)
  const int iters_run = (srch.early_exit && allmet) ? 0 : iters;
  if (iters_run > 0) ps.refill(0, lane, n, rng_chain, key0, key1, swap_thr, 0);
  for (int k = 0; k < iters_run;) {
    if (k + W - 1 - kb >= kWave) {
      kb = k;
      ps.refill(kb, lane, n, rng_chain, key0, key1, swap_thr, 0);
    }
    // two waves: proposals k and k + 1, the second on the current order or, when most
    // proposals are accepted, on the first one's candidate
    const bool on_acc = rate >= 1 << 15;
    const uint16_t *tree = kSpecTree[W == 2 ? 0 : min((rate * 5) >> 16, 4)];
    const SpecCur cc{set_ev(W), set_snap(W), cur_pr0, cur_c1};
    uint32_t pr0, c1;
    Score s;
    if constexpr (W == 2) {
      auto map_of = [&](int d, int &lo) {
        const uint32_t pk = rl(ps.pk, k + d - kb);
        const int i = (int)(pk & 1023u), j = (int)((pk >> 10) & 1023u);
        lo = min(i, j);
        return src_map((int)((pk >> 20) & 1u) + 1, i, j);
      };
      int lo, lo0;
      const SrcMap own = map_of(w, lo);
      if (w == 1 && on_acc) {
        const SrcMap under = map_of(0, lo0);
        s = spec_replay(m, posr, SrcPair{own, under}, min(lo, lo0), cc, set_ev(w), set_snap(w), sc, pr0, c1);
      } else {
        s = spec_replay(m, posr, own, lo, cc, set_ev(w), set_snap(w), sc, pr0, c1);
      }
    } else {
      // this wave's node: its proposal on top of the moves it assumes kept
      const uint32_t node = (uint32_t)uniform((int)tree[w]);
      const uint32_t mask = (node & 0xFFu) | (1u << (node >> 8));
      int lo = n, hi = 0;
      for (uint32_t left = mask; left; left &= left - 1) {
        const uint32_t pk = rl(ps.pk, k + __builtin_ctz(left) - kb);
        const int i = (int)(pk & 1023u), j = (int)((pk >> 10) & 1023u);
        lo = min(lo, min(i, j));
        hi = max(hi, max(i, j));
        apply_move_lds(idx, i == j ? 0 : (int)((pk >> 20) & 1u) + 1, i, j, lane);
      }
      s = spec_replay(m, posr, SrcIndex{idx}, lo, cc, set_ev(w), set_snap(w), sc, pr0, c1);
      for (int p = lo + lane; p <= hi; p += kWave) idx[p] = (uint16_t)p;
    }
    uint64_t *mine = xch + (slot * W + w) * 4;
    if (lane == 0) {
      mine[0] = (uint64_t)s.n;
      mine[1] = s.t;
      mine[2] = (uint64_t)pr0 | ((uint64_t)c1 << 32);
    }
    __syncthreads();
    const uint64_t *x = xch + slot * W * 4;
    slot ^= 1;
    int last = -1;  // the last accepted node
    // decides proposal k, scored at `node`
    auto decide = [&](int node) __attribute__((always_inline)) {
      const int64_t sn = (int64_t)x[node * 4];
      const uint64_t st = x[node * 4 + 1];
      const bool acc = obj_accept<OBJ>(cn, ct, sn - cn, (int64_t)(st - ct), t_ref, cool.T, rl(ps.w3, k - kb));
      cool.step();
      rate += ((acc ? 1 << 16 : 0) - rate) >> 5;
      if (acc) {
        last = node;
        cn = sn;
        ct = st;
        ++accepts;
        digest = (digest ^ (uint64_t)k) * kFnvPrime;
        digest = (digest ^ (uint64_t)cn) * kFnvPrime;
        digest = (digest ^ ct) * kFnvPrime;
        const bool better = obj_better<OBJ>(cn, ct, bn, bt);
        if (better) {
          bn = cn;
          bt = ct;
          biter = k;
        }
        if (w == 0) {
          const uint32_t pk = rl(ps.pk, k - kb);
          const int i = (int)(pk & 1023u), j = (int)((pk >> 10) & 1023u);
          apply_move_lds(posr, i == j ? 0 : (int)((pk >> 20) & 1u) + 1, i, j, lane);
          if (better)
            for (int p = lane; p < n; p += kWave) gbest[p] = (uint16_t)(posr[p].z >> 2);
        }
      }
      ++k;
      return acc;
    };
    if constexpr (W == 2) {
      if (decide(0) == on_acc && k < iters_run) decide(1);
    } else {
      uint32_t pattern = 0;  // outcomes so far in this round
      for (int d = 0, node = 0; node >= 0; ++d) {
        pattern |= decide(node) ? 1u << d : 0u;
        if (k >= iters_run) break;
        const uint32_t next = ((uint32_t)(d + 1) << 8) | pattern;
        node = -1;
#pragma unroll
        for (int u = 1; u < W; ++u)
          if ((uint32_t)uniform((int)tree[u]) == next) node = u;
      }
    }
    if (last >= 0) {
      cur_pr0 = (uint32_t)x[last * 4 + 2];
      cur_c1 = (uint32_t)(x[last * 4 + 2] >> 32);
      accept_set(last);
      // every wave takes this branch: the records change before any replays again
      __syncthreads();
    }
  }
  if (w == 0) {
    for (int p = lane; p < n; p += kWave) gcur[p] = (uint16_t)(posr[p].z >> 2);
    if (lane == 0) {
      int64_t *rec = reinterpret_cast<int64_t *>(ws + ws_off_records(n)) + (size_t)chain * 8;
      rec[0] = cn;
      rec[1] = (int64_t)ct;
      rec[2] = bn;
      rec[3] = (int64_t)bt;
      rec[4] = biter;
      rec[5] = accepts;
      rec[6] = (int64_t)digest;
      rec[7] = allmet;
    }
  }
}

// One workgroup of W waves per chain.
template <int OBJ, int W>
__global__ void __launch_bounds__(W * kWave) anneal_cont_spec_kernel(DevModel m, QueuePtrs q, int chains, int iters,
                                                                      double T0, double alpha, uint32_t key0,
                                                                      uint32_t key1, uint64_t swap_thr,
                                                                      SearchParams srch, unsigned char *ws) {
  extern __shared__ __align__(16) unsigned char lds[];
  if (!gate_open(ws, m.gate, m.flags)) return;
  const int chain = (int)blockIdx.x;
  if (chain >= chains) return;
  anneal_cont_spec_body<OBJ, W>(m, q, lds, chains, chain, (uint32_t)chain, iters, T0, alpha, key0, key1, swap_thr, srch,
                                ws);
}

}  // namespace sa
