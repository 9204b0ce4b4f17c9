// Workgroup shapes of the annealing kernels and of the one-order-per-wave evaluation kernels, and
// which kernel of fixed-size batches pays. Host arithmetic only, with no HIP in it.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace sa {

struct LdsShape {
  int fit;    // chains per workgroup that the LDS holds, at most 16 (0: not even one)
  int waves;  // chains per workgroup of the launch
};

// The launch takes no more chains per workgroup than spread them evenly over the CUs in as many
// passes as the LDS makes necessary (1500 chains: 250 workgroups of 6; in 188 workgroups of 8 a
// quarter of the CUs idled).
inline LdsShape lds_shape(int chains, size_t shared, size_t per, int lim, int cus) {
  if (shared + per > (size_t)lim) return LdsShape{0, 0};
  const int64_t fit = std::min<int64_t>(16, ((int64_t)lim - (int64_t)shared) / (int64_t)per);
  const int64_t passes = (chains + fit * cus - 1) / (fit * cus);
  return LdsShape{(int)fit, (int)((chains + passes * cus - 1) / (passes * cus))};
}

// The same for the fitted-model chains, whose blocks are small: where one full workgroup per CU does
// not hold every chain and the LDS holds five of four chains, workgroups of four, one chain per
// SIMD. Two of ten on a CU can put six waves on one SIMD and four on another (5000 chains of 256
// requests in batches of 8: 1.07 times as long; 10000: 1.18 times).
inline LdsShape lds_shape_small(int chains, size_t shared, size_t per, int lim, int cus) {
  LdsShape s = lds_shape(chains, shared, per, lim, cus);
  if ((int64_t)s.fit * cus < chains && 5 * (shared + 4 * per) <= (size_t)lim) s.waves = 4;
  return s;
}

// Chains per workgroup of the register kernels, at most four (one per SIMD): one while the chains are
// at most two per CU, and beyond that as many as one workgroup per CU takes. Two workgroups of two
// can share two SIMDs of a CU and leave the others idle: 600 to 1023 chains took 10 to 27 % longer
// as twos, as long as 1024 do (64 requests in batches of 16: 323 against 276 us).
inline int reg_shape(int chains, int cus) {
  return chains > 2 * cus ? std::min(4, (chains + cus - 1) / cus) : 1;
}

// Whether the LDS gives the delta kernels of fixed-size batches enough chains at once: four per
// CU (one per SIMD), or every chain in one pass. What counts is what the LDS holds, not the
// spread: 1500 chains where five fit go as 500 workgroups of three.
inline bool lds_suffices(const LdsShape &s, int chains, int cus) {
  return s.fit >= 4 || (s.fit > 0 && (int64_t)s.fit * cus >= chains);
}

// Whether the register kernel's form for any batch size beats the LDS delta kernels: its cost
// grows with the batch (two lane gathers per member: 64 requests in batches of 3 take 2.6 ms
// against 6.0 ms, of 24 1.27 against 1.94 ms, of 33 1.31 against 1.27 ms), and when one batch
// holds every request no proposal needs a replay and neither wins (with several instances the
// mean size decides: 3500 chains on instances of 6 in batches of 9, 494 against 443 us). Two
// batches of 17 to 32 are one row of the delta kernel, which issues less: it takes 0.87 to 0.99 of
// the time while more than two waves share a SIMD and one pass holds every chain (`chains` 0: not
// known), 1.1 to 1.25 of it below and 0.9 to 1.25 beyond.
inline bool reg_any_pays(int n, int B, int chains = 0, int cus = 1) {
  if (B >= 17 && n <= 2 * B && chains > 8 * cus && chains <= 16 * cus) return false;
  return B <= 32 && n > B;
}

// One batch per wave with limit rows (timelines of 32 bits): batches of 17 and more, at most 32
// of them (the rows held in registers). Batches of 17 to 32 leave half the lanes idle, but the
// other kernel's rows of two batches cost it more than twice a limit row (bounds, recounts):
// 1500 chains of 389 requests in batches of 24 took 4.9 ms per 1000 proposals on it and 4.1 ms
// here (3.5 ms with the rows past the last batch left out); batches of 17: 3.4 against 2.8; 32: 3.2
// against 2.4 (1024 chains of 256 requests) and 3.2 against 2.8 (4096 of 1000). With four batches
// in one of its rows it wins: 500 requests in batches of 16: 2.2 against 2.9, in batches of 8 1.9
// against 2.8. (One or two batches of up to 32 are one of its rows: nothing to replay, 6 % longer
// with limit rows at 2000 chains of 2 to 30 requests, or the case above.)
inline bool rows_pay(int n, int B) { return B >= 17 && (B > 32 || n > 2 * B) && (n + B - 1) / B <= 32; }

// Workgroups of a one-order-per-wave evaluation. Each forms the verdict and stages the requests
// first, about 3 us, so no more than `held`, what the GPU holds at once, with every wave taking
// several rows: at 32768 rows of 10 requests, 8192 workgroups took 56 us and 2048 take 25 us.
// Workgroups all resident end unevenly over many rows, though, so from four rows per wave on one
// workgroup per 4 `waves` rows (at most 8192), which start as others end: 2^20 rows of 128
// requests take 678 us in 2048 workgroups, 551 us in 8192. Between the two, a count a little
// above `held` leaves a last pass nearly empty (4500 continuous rows of 700 requests in batches
// of 64, one workgroup per CU: 1125 workgroups 240 us, 281 352 us, 256 222 us; 32768 layouts of
// 400 requests in batches of up to 64, seven per CU: 8192 313 us, 2048 404 us, 1792 288 us): `beyond` times `held` must be passed.
// `per_simd` is what the kernel's registers allow; a CU has four SIMDs.
struct EvalShape {
  int per_simd;
  double beyond;
};
inline int eval_grid(int64_t rows, int waves, size_t lds, const EvalShape &k, int lim, int cus) {
  const int64_t per_cu =
      std::max<int64_t>(1, std::min<int64_t>(4 * k.per_simd / waves, (int64_t)lim / (int64_t)lds));
  const int64_t held = per_cu * cus, want = (rows + waves - 1) / waves;
  const int64_t more = std::min<int64_t>(8192, rows / (4 * waves));
  return (int)std::min<int64_t>(want, (double)more >= k.beyond * (double)held ? more : held);
}

}  // namespace sa
