// Truncated (top-k / top-p) sampling at temperature T, in refinement and in
// verification (the filtered form of the T > 0 sampling that speculative
// verification keeps lossless, section 3.1).
//
// On the scaled logits x_v = fl32(l_v * fl32(1/T)) of one row:
//   top-k keeps every v whose x_v is at least the k-th largest x (ties with it
//         stay);
//   top-p then orders the kept tokens by x descending, ties by lower index,
//         and keeps each token whose preceding mass in that order is below
//         p times the kept mass: the shortest prefix reaching p of it;
//   the kept tokens are sampled by inverse CDF in vocabulary order,
//         y = min{v : sum_{w <= v, kept} e^(x_w - m) > u Z}.
// A row's filter is a state (m, tk, tp, pidx, Z): v is kept iff
// key(x_v) >= tk and (key(x_v) > tp or (key(x_v) == tp and v <= pidx)), with
// key() the order-preserving 32-bit image of a float; Z is the kept mass.
//
// One workgroup of 16 waves per row, in one of two ways.
//
// Top-k rows (k up to kCandK and the number of vocabulary units): the row's
// unit maxima are at hand, from the softmax partials of the kernel that wrote
// the logits, or from k_row_units for the target's rows.  The k-th largest unit
// maximum (its leading 22 bits) is a bound that at least k tokens reach, and
// few more: only the units whose maximum reaches it are read, their tokens at
// or above it are listed in vocabulary order in LDS, and top-k, top-p, Z and
// the choice run on that list.  A row costs its unit maxima (2 K at most) and the
// tokens of about k units instead of seven passes over V = 151936 logits, two of
// them fp64 exponentials.  A unit has 64 tokens in a target row, at most 128 in the
// Read's rows and those of the LM-head GEMM, and a 256th of the vocabulary in the
// seed of the streamed LM heads (608 tokens).  A list that overflows kCand (many
// ties) falls back to the general way.  65 rows at k = 50, p = 0.9: 299 -> 23 us per pass, the seed
// 733 -> 45, the target rows 631 -> 17 + 39, the last token 229 -> 16 us.
//
// The general way (top-p alone): the row is re-read by every step:
//   1. m = max x;
//   2. top-k: radix select of the k-th largest key in digits of 11, 11 and 10
//      bits (bin counts in LDS: integer atomics, so the result does not depend
//      on their order);
//   3. top-p: the same radix select on masses, each token's e^(x - m) held as
//      a 64-bit fixed-point integer (2^-44 units; at most 2^18 tokens of at
//      most 2^44 each), again order-independent; tokens tied at the cut value
//      are kept in index order while the mass before them stays below p Z;
//   4. Z and the inverse-CDF choice in fp64 in a fixed order: each wave sums
//      a contiguous range of the vocabulary with in-order wave scans, the
//      wave totals are added in wave order, and the wave whose running total
//      passes u Z rescans its range for the crossing token.
// The list goes through the same steps 2 to 4.  One wave picks a digit's bin
// with a scan over the bins (one thread walking 256 of them took about 10 us a
// digit).  Everything is deterministic: two runs give the same tokens and
// states.
#include "xp_internal.h"

namespace xp {

constexpr int kFWaves = 16;
constexpr int kFThreads = kFWaves * kWave;
constexpr double kFixScale = 17592186044416.0;   // 2^44

// order-preserving key: x < y  <=>  key(x) < key(y); -0 and +0 map alike
__device__ __forceinline__ uint32_t okey(float x) {
  const uint32_t b = x == 0.f ? 0u : __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
__device__ __forceinline__ double fweight(float x, float m) { return exp((double)x - (double)m); }
__device__ __forceinline__ uint64_t fixw(float x, float m) {
  return (uint64_t)(fweight(x, m) * kFixScale);     // truncation; e^(x - m) <= 1
}
__device__ __forceinline__ bool fkept(uint32_t key, int v, const FState& s) {
  return key >= s.tk && (key > s.tp || (key == s.tp && v <= s.pidx));
}

__device__ __forceinline__ double fwave_scan(double x, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double y = __shfl_up(x, off, kWave);
    if (lane >= off) x += y;
  }
  return x;
}

constexpr int kBins = 2048;            // bins of a radix digit
constexpr int kDigits = 3;
__device__ __forceinline__ int digit_shift(int d) { return d == 0 ? 21 : d == 1 ? 10 : 0; }
__device__ __forceinline__ int digit_bins(int d) { return d == 2 ? 1024 : 2048; }
constexpr int kCandK = 1024;           // largest top-k taken by the candidate list
constexpr int kCand = 4096;            // tokens of the candidate list
constexpr int kCandUnits = 2048;       // vocabulary units that may hold candidates
constexpr int kUnitsMax = 4096;        // vocabulary units of a row

struct FShared {
  unsigned long long hist[kBins];      // counts (top-k) or fixed-point masses (top-p)
  uint32_t ck[kCand];                  // candidates in vocabulary order: key
  int32_t cv[kCand];                   //   and token
  int32_t ulist[kCandUnits], ucnt[kCandUnits];
  float wmax[kFWaves];
  unsigned long long wsum[kFWaves];
  double wtot[kFWaves];
  int32_t wcnt[kFWaves];
  uint32_t prefix;
  unsigned long long above, binmass;
  int pidx;
  int pick;
  double start;
};

__device__ __forceinline__ float block_max(float mx, FShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
  if (lane == 0) sh.wmax[wave] = mx;
  __syncthreads();
  float m = sh.wmax[0];
#pragma unroll
  for (int w = 1; w < kFWaves; ++w) m = fmaxf(m, sh.wmax[w]);
  __syncthreads();
  return m;
}

// Exclusive scan of one count per thread in thread order; *total for everyone.
__device__ __forceinline__ int block_scan(int c, int* total, FShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off, kWave);
    if (lane >= off) x += y;
  }
  if (lane == 63) sh.wcnt[wave] = x;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kFWaves; ++w) {
    if (w == wave) before = all;
    all += sh.wcnt[w];
  }
  __syncthreads();
  *total = all;
  return before + x - c;
}

__device__ __forceinline__ void zero_hist(int bins, FShared& sh) {
  for (int j = threadIdx.x; j < bins; j += kFThreads) sh.hist[j] = 0ull;
  __syncthreads();
}

// After the histogram of a digit: the highest bin whose content, with all above
// it and sh.above before that, satisfies reach(); the content above it goes to
// sh.above, its own to sh.binmass, the digit into sh.prefix.  By wave 0, lane l
// holding the bins / 64 bins from the top that follow lane l - 1's.  When no
// bin reaches (rounding), bin 0 with everything above it.
template <class RF>
__device__ void pick_bin(int bins, int shift, RF reach, FShared& sh) {
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x, per = bins / kWave, top = bins - 1 - lane * per;
    unsigned long long c = 0ull;
    for (int j = 0; j < per; ++j) c += sh.hist[top - j];
    unsigned long long x = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned long long y = __shfl_up(x, off, kWave);
      if (lane >= off) x += y;
    }
    const unsigned long long base = sh.above;
    const unsigned long long hit = __ballot(c != 0ull && reach(base + x));
    const int first = hit ? __ffsll((long long)hit) - 1 : kWave - 1;
    if (lane == first) {
      unsigned long long cum = base + x - c;
      int sel = 0;
      unsigned long long own = sh.hist[0];
      if (hit) {
        for (int j = 0; j < per; ++j) {
          const unsigned long long b = sh.hist[top - j];
          if (b != 0ull && reach(cum + b)) {
            sel = top - j;
            own = b;
            break;
          }
          cum += b;
        }
      } else {
        cum = base + x;
      }
      sh.above = cum;
      sh.binmass = own;
      sh.prefix |= (uint32_t)sel << shift;
    }
  }
  __syncthreads();
}

// f(i, x(i)) for i < n over the workgroup's threads, eight loads in flight per
// thread.
template <class XF, class F>
__device__ __forceinline__ void each(XF x, int n, F f) {
  constexpr int U = 8;
  int i = threadIdx.x;
  for (; i + (U - 1) * kFThreads < n; i += U * kFThreads) {
    float v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) v[j] = x(i + j * kFThreads);
#pragma unroll
    for (int j = 0; j < U; ++j) f(i + j * kFThreads, v[j]);
  }
  for (; i < n; i += kFThreads) f(i, x(i));
}

// The k-th largest of the n keys that keys(f) passes to f (1 <= k <= n), or its
// leading `digits` digits followed by zero bits.
template <class KF>
__device__ uint32_t select_key(KF keys, int k, int digits, FShared& sh) {
  if (threadIdx.x == 0) {
    sh.prefix = 0u;
    sh.above = 0ull;
  }
  for (int d = 0; d < digits; ++d) {
    const int bins = digit_bins(d), shift = digit_shift(d);
    const int hi = d == 0 ? 32 : digit_shift(d - 1);
    zero_hist(bins, sh);
    const uint32_t pre = d == 0 ? 0u : sh.prefix >> hi;
    keys([&](uint32_t key) {
      if (d == 0 || (key >> hi) == pre)
        atomicAdd(&sh.hist[(key >> shift) & (uint32_t)(bins - 1)], 1ull);
    });
    pick_bin(bins, shift, [&](unsigned long long c) { return c >= (unsigned long long)k; }, sh);
  }
  return sh.prefix;
}

// Top-p among the items i < n of value x(i) whose key reaches tk: the cut key
// s.tp and, where only some of the tokens tied at it stay, the last one kept
// (s.pidx, through tok(i), items being in token order).
template <class XF, class TF>
__device__ void select_mass(XF x, int n, TF tok, float p, FState& s, FShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float m = s.m;
  const uint32_t tk = s.tk;
  if (threadIdx.x == 0) {
    sh.prefix = 0u;
    sh.above = 0ull;
  }
  double target = 0.0;
  for (int d = 0; d < kDigits; ++d) {
    const int bins = digit_bins(d), shift = digit_shift(d);
    const int hi = d == 0 ? 32 : digit_shift(d - 1);
    zero_hist(bins, sh);
    const uint32_t pre = d == 0 ? 0u : sh.prefix >> hi;
    unsigned long long zl = 0ull;
    each(x, n, [&](int, float xv) {
      const uint32_t kv = okey(xv);
      if (kv >= tk && (d == 0 || (kv >> hi) == pre)) {
        const unsigned long long w = fixw(xv, m);
        if (d == 0) zl += w;
        atomicAdd(&sh.hist[(kv >> shift) & (uint32_t)(bins - 1)], w);
      }
    });
    if (d == 0) {
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) zl += __shfl_xor(zl, o, kWave);
      if (lane == 0) sh.wsum[wave] = zl;
      __syncthreads();
      unsigned long long Zk = 0ull;
#pragma unroll
      for (int w = 0; w < kFWaves; ++w) Zk += sh.wsum[w];
      target = (double)p * (double)Zk;
    }
    pick_bin(bins, shift, [&](unsigned long long c) { return (double)c >= target; }, sh);
  }
  s.tp = sh.prefix;
  // tokens tied at the cut value: keep them in index order while the mass
  // before them (all of equal weight wt) stays below p Zk
  const unsigned long long A = sh.above, wt = fixw(key_value(s.tp), m);
  const unsigned long long c = wt ? sh.binmass / wt : 1ull;
  unsigned long long nt = wt ? (unsigned long long)ceil((target - (double)A) / (double)wt) : 1ull;
  nt = nt < 1ull ? 1ull : (nt > c ? c : nt);
  while (nt > 1ull && (double)(A + (nt - 1ull) * wt) >= target) --nt;
  while (nt < c && (double)(A + nt * wt) < target) ++nt;
  if (nt < c) {
    // the nt-th tied token: one wave counts them in order
    if (wave == 0) {
      unsigned long long seen = 0ull;
      int found = n - 1;
      for (int base = 0; base < n; base += kWave) {
        const int i = base + lane;
        const bool t = i < n && okey(x(i)) == s.tp;
        const unsigned long long bal = __ballot(t);
        const unsigned long long cnt = __popcll(bal);
        if (seen + cnt >= nt) {
          unsigned long long b2 = bal;
          for (unsigned long long r = seen + 1ull; r < nt; ++r) b2 &= b2 - 1ull;
          found = base + __ffsll((long long)b2) - 1;
          break;
        }
        seen += cnt;
      }
      if (lane == 0) sh.pidx = tok(found);
    }
    __syncthreads();
    s.pidx = sh.pidx;
  }
  __syncthreads();
}

// The tokens of key >= thr in vocabulary order, into sh.ck / sh.cv: only the
// units (unit_lo(u) .. unit_lo(u + 1), u < U <= kUnitsMax) whose maximum
// reaches thr are read, a wave per unit: once to count, once to place.
// Returns their number, or -1 when a list would overflow or none reaches thr (a
// row with NaN: the maxima pass over it, a key does not).  um[j] is the maximum
// of unit (kUnitsMax / kFThreads) threadIdx.x + j.
constexpr int kUPT = kUnitsMax / kFThreads;
template <class XF, class UF>
__device__ int collect(XF x, int V, int U, UF unit_lo, const float (&um)[kUPT], uint32_t thr,
                       FShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int c = 0;
#pragma unroll
  for (int j = 0; j < kUPT; ++j) c += (kUPT * tid + j < U && okey(um[j]) >= thr) ? 1 : 0;
  int nu;
  int at = block_scan(c, &nu, sh);
  if (nu > kCandUnits) return -1;
#pragma unroll
  for (int j = 0; j < kUPT; ++j)
    if (kUPT * tid + j < U && okey(um[j]) >= thr) sh.ulist[at++] = kUPT * tid + j;
  __syncthreads();
  auto walk = [&](auto f) {                       // f(j, n-th tokens before, key, token, hit, ballot)
    for (int j = wave; j < nu; j += kFWaves) {
      const int u = sh.ulist[j], lo = unit_lo(u);
      const int hi = min(V, unit_lo(u + 1));
      int before = 0;
      for (int base = lo; base < hi; base += 2 * kWave) {
        const int v0 = base + lane, v1 = v0 + kWave;
        const float x0 = x(v0 < hi ? v0 : hi - 1), x1 = x(v1 < hi ? v1 : hi - 1);
        const uint32_t k0 = okey(x0), k1 = okey(x1);
        const unsigned long long h0 = __ballot(v0 < hi && k0 >= thr);
        const unsigned long long h1 = __ballot(v1 < hi && k1 >= thr);
        f(j, before, k0, v0, h0);
        before += __popcll(h0);
        f(j, before, k1, v1, h1);
        before += __popcll(h1);
      }
      if (lane == 0) sh.ucnt[j] = before;
    }
  };
  walk([](int, int, uint32_t, int, unsigned long long) {});
  __syncthreads();
  constexpr int UPT = kCandUnits / kFThreads;
  int mine[UPT], sum = 0;
#pragma unroll
  for (int j = 0; j < UPT; ++j) {
    mine[j] = UPT * tid + j < nu ? sh.ucnt[UPT * tid + j] : 0;
    sum += mine[j];
  }
  int n;
  int off = block_scan(sum, &n, sh);
  if (n > kCand || n == 0) return -1;
  // each unit's first place goes where its entry of the unit list was read from
  int place[UPT];
#pragma unroll
  for (int j = 0; j < UPT; ++j) {
    place[j] = off;
    off += mine[j];
  }
  __syncthreads();
  int32_t* first = reinterpret_cast<int32_t*>(sh.hist);        // free between selections
#pragma unroll
  for (int j = 0; j < UPT; ++j)
    if (UPT * tid + j < nu) first[UPT * tid + j] = place[j];
  __syncthreads();
  walk([&](int j, int before, uint32_t key, int v, unsigned long long hit) {
    if ((hit >> lane) & 1ull) {
      const int i = first[j] + before + __popcll(hit & ((1ull << lane) - 1ull));
      sh.ck[i] = key;
      sh.cv[i] = v;
    }
  });
  __syncthreads();
  return n;
}

// Block-wide filter state of the row x(v), v < V (every thread calls it; on
// return s holds m, tk, tp and pidx of the row; Z is filled by the caller).
// k = 0: no top-k; p >= 1: no top-p.  umax(u), u < U: the largest x of unit u.
// *list: the number of candidates in sh.ck / sh.cv when the state came from
// the candidate list (every kept token is in it), or -1.
template <class XF, class MF, class UF>
__device__ FState filter_state(XF x, int V, int U, MF umax, UF unit_lo, int k, float p, int* list,
                               FShared& sh) {
  const bool ka = k > 0 && k < V, pa = p < 1.f;
  float um[kUPT], mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < kUPT; ++j) {
    const int u = kUPT * threadIdx.x + j;
    um[j] = umax(u < U ? u : U - 1);
    mx = fmaxf(mx, um[j]);
  }
  FState s;
  s.m = block_max(mx, sh);
  s.tk = 0u;
  s.tp = 0u;
  s.pidx = 0x7FFFFFFF;
  s.Z = 0.0;
  *list = -1;
  if (ka && k <= kCandK && k <= U) {
    const uint32_t thr = select_key(
        [&](auto f) {
#pragma unroll
          for (int j = 0; j < kUPT; ++j)
            if (kUPT * (int)threadIdx.x + j < U) f(okey(um[j]));
        },
        k, 2, sh);
    *list = collect(x, V, U, unit_lo, um, thr, sh);
  }
  if (*list >= 0) {
    const int n = *list;
    auto cx = [&](int i) { return key_value(sh.ck[i]); };
    s.tk = select_key(
        [&](auto f) {
          for (int i = threadIdx.x; i < n; i += kFThreads) f(sh.ck[i]);
        },
        k, kDigits, sh);
    __syncthreads();
    if (pa) select_mass(cx, n, [&](int i) { return sh.cv[i]; }, p, s, sh);
    return s;
  }
  if (ka) {
    s.tk = select_key([&](auto f) { each(x, V, [&](int, float xv) { f(okey(xv)); }); }, k, kDigits,
                      sh);
    __syncthreads();
  }
  if (pa) select_mass(x, V, [](int i) { return i; }, p, s, sh);
  return s;
}

// Ordered fp64 sum of weight(v) over v < V: wave w sums the contiguous range
// [V w / 16, V (w + 1) / 16) with in-order scans; the wave totals are added in
// wave order.  Leaves each wave's total in sh.wtot.
template <class WF>
__device__ double ordered_sum(WF weight, int V, FShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lo = (int)((int64_t)V * wave / kFWaves), hi = (int)((int64_t)V * (wave + 1) / kFWaves);
  double carry = 0.0;
  for (int base = lo; base < hi; base += kWave) {
    const int v = base + lane;
    const double w = v < hi ? weight(v) : 0.0;
    carry += __shfl(fwave_scan(w, lane), 63, kWave);
  }
  __syncthreads();
  if (lane == 0) sh.wtot[wave] = carry;
  __syncthreads();
  double Z = 0.0;
#pragma unroll
  for (int w = 0; w < kFWaves; ++w) Z += sh.wtot[w];
  return Z;
}

// Inverse-CDF choice over weight(v) after ordered_sum() gave Z (its wave
// totals still in sh.wtot): the smallest v whose running sum exceeds u Z, in
// the same summation order; when rounding leaves no crossing, the last v of
// nonzero weight.  Returns the choice in every thread.
template <class WF>
__device__ int ordered_icdf(WF weight, int V, double Z, double u, FShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double target = u * Z;
  if (tid == 0) {
    double run = 0.0;
    int ws = -1;
    for (int w = 0; w < kFWaves; ++w) {
      if (run + sh.wtot[w] > target) {
        ws = w;
        break;
      }
      run += sh.wtot[w];
    }
    if (ws < 0) {                                   // no crossing: the last wave with mass
      ws = kFWaves - 1;
      while (ws > 0 && !(sh.wtot[ws] > 0.0)) --ws;
      run = 0.0;
      for (int w = 0; w < ws; ++w) run += sh.wtot[w];
    }
    sh.pick = ws;
    sh.start = run;
  }
  __syncthreads();
  if (wave == sh.pick) {
    const int lo = (int)((int64_t)V * wave / kFWaves), hi = (int)((int64_t)V * (wave + 1) / kFWaves);
    double cum = sh.start;
    int chosen = -1, last_nz = -1;
    for (int base = lo; base < hi; base += kWave) {
      const int v = base + lane;
      const double w = v < hi ? weight(v) : 0.0;
      const double tot = cum + fwave_scan(w, lane);
      const unsigned long long hit = __ballot(v < hi && tot > target);
      const unsigned long long nz = __ballot(v < hi && w > 0.0);
      if (nz) last_nz = base + 63 - __clzll((long long)nz);
      if (hit) {
        chosen = base + __ffsll((long long)hit) - 1;
        break;
      }
      cum = __shfl(tot, 63, kWave);
    }
    if (chosen < 0) chosen = last_nz >= 0 ? last_nz : lo;
    if (lane == 0) sh.pidx = chosen;                // reuses the slot: filter state is kept in s
  }
  __syncthreads();
  return sh.pidx;
}

// Per-sequence sampling parameters: filt[b] = the row samples and truncates;
// temp_nf[b] = the row samples without truncation (the untruncated sampler's
// rows); fk, fp the effective top-k (0 = none) and top-p (1 = none).  A
// negative k or a p that is not positive is an error (XP_DEVERR_FILTER) and
// is replaced by no truncation; k >= V and p >= 1 mean none.  Greedy rows
// ignore both.
__global__ void k_filter_params(int batch, int V, const uint8_t* __restrict__ temp,
                                const int32_t* __restrict__ top_k, const float* __restrict__ top_p,
                                uint8_t* __restrict__ filt, uint8_t* __restrict__ temp_nf,
                                int32_t* __restrict__ fk, float* __restrict__ fp,
                                uint32_t* __restrict__ err) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  const bool smp = temp != nullptr && temp[b] != 0;
  int k = top_k != nullptr ? top_k[b] : 0;
  float p = top_p != nullptr ? top_p[b] : 1.f;
  bool bad = false;
  if (k < 0) {
    bad = true;
    k = 0;
  }
  if (!(p > 0.f)) {                               // p <= 0 or NaN
    bad = true;
    p = 1.f;
  }
  if (k >= V) k = 0;
  if (!(p < 1.f)) p = 1.f;
  const bool f = smp && (k > 0 || p < 1.f);
  filt[b] = f ? 1 : 0;
  temp_nf[b] = (smp && !f) ? 1 : 0;
  fk[b] = k;
  fp[b] = p;
  if (smp && bad) atomicOr(err, XP_DEVERR_FILTER);
}

// Truncated sampling of one position per workgroup.  MODE 0: the seed Y^(0)
// from the base logits s (tile-major); with caller seed ids only the state is
// kept.  MODE 1: the selection of a Jacobi pass from the pass's logits
// (row-major, written by the Read stream).  The chosen token goes to Ynew for
// the selection kernel that follows; the state to fst for verification.
template <int MODE>
__global__ __launch_bounds__(kFThreads) void k_fsample(
    int B, int V, int M, const float* __restrict__ S, int Ms, const float* __restrict__ lf,
    const uint8_t* __restrict__ filt, const int32_t* __restrict__ fk, const float* __restrict__ fp,
    const float* __restrict__ invT, const float* __restrict__ u_draft,
    const int32_t* __restrict__ seed_ids, int32_t* __restrict__ Ynew, FState* __restrict__ fst,
    const int32_t* __restrict__ iters, int early_exit, const Stat* __restrict__ stats, int ntiles,
    int U) {
  const int p = blockIdx.x, b = p / B;
  if (!filt[b]) return;
  if (MODE == 1 && early_exit && iters[b] != 0) return;     // the sequence keeps Y^(j)
  __shared__ FShared sh;
  const float it = invT[b];
  auto x = [&](int v) -> float {
    return (MODE == 0 ? S[s_index(p, v, Ms)] : lf[(size_t)p * V + v]) * it;
  };
  int n;
  FState s = filter_state(
      x, V, U, [&](int u) { return stats[(size_t)p * U + u].m; },
      [&](int u) { return unit_tile_lo(u, ntiles, U) * kTile; }, fk[b], fp[b], &n, sh);
  const bool pick = !(MODE == 0 && seed_ids != nullptr);
  const double u01 = pick ? (double)u_draft[p] : 0.0;
  int y = 0;
  if (n >= 0) {                                     // workgroup-uniform
    auto w = [&](int i) -> double {
      return fkept(sh.ck[i], sh.cv[i], s) ? fweight(key_value(sh.ck[i]), s.m) : 0.0;
    };
    s.Z = ordered_sum(w, n, sh);
    if (pick) y = sh.cv[ordered_icdf(w, n, s.Z, u01, sh)];
  } else {
    auto w = [&](int v) -> double {
      const float xv = x(v);
      return fkept(okey(xv), v, s) ? fweight(xv, s.m) : 0.0;
    };
    s.Z = ordered_sum(w, V, sh);
    if (pick) y = ordered_icdf(w, V, s.Z, u01, sh);
  }
  if (pick && threadIdx.x == 0) Ynew[p] = y;
  if (threadIdx.x == 0) fst[p] = s;
}

// Unit maxima of the target rows of truncated sequences: units of kVUnit
// consecutive tokens, a workgroup taking kVUnitTok tokens of one row
// (blockIdx.y) of one sequence (blockIdx.z).  Bound by reading the rows once.
constexpr int kVUnit = 64, kVUnitTok = 4096;
__global__ __launch_bounds__(256) void k_row_units(int B, int V, const float* __restrict__ tl,
                                                   const uint8_t* __restrict__ filt,
                                                   const float* __restrict__ invT,
                                                   float* __restrict__ umax, int U) {
  const int b = blockIdx.z, k = blockIdx.y;
  if (!filt[b]) return;
  const float it = invT[b];
  const size_t r = (size_t)b * (B + 1) + k;
  const float* row = tl + r * V;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int N = kVUnitTok / 256;
  const int v0 = blockIdx.x * kVUnitTok + wave * (kVUnitTok / 4) + lane;
  float x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = row[min(v0 + kVUnit * i, V - 1)];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float m = v0 + kVUnit * i < V ? x[i] * it : -INFINITY;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
    const int u = (v0 - lane) / kVUnit + i;
    if (lane == 0 && u < U) umax[r * U + u] = m;
  }
}

// Filter state (with Z) of the target rows of truncated sequences, one
// workgroup per (row k = 0..B, sequence).
__global__ __launch_bounds__(kFThreads) void k_vfstate(
    int B, int V, const float* __restrict__ tl, const uint8_t* __restrict__ filt,
    const int32_t* __restrict__ fk, const float* __restrict__ fp, const float* __restrict__ invT,
    FState* __restrict__ tst, const float* __restrict__ umax, int U) {
  const int k = blockIdx.x, b = blockIdx.y;
  if (!filt[b]) return;
  __shared__ FShared sh;
  const float it = invT[b];
  const size_t r = (size_t)b * (B + 1) + k;
  const float* row = tl + r * V;
  auto x = [&](int v) -> float { return row[v] * it; };
  int n;
  FState s = filter_state(
      x, V, U, [&](int u) { return umax[r * U + u]; }, [&](int u) { return u * kVUnit; }, fk[b],
      fp[b], &n, sh);
  if (n >= 0)
    s.Z = ordered_sum(
        [&](int i) -> double {
          return fkept(sh.ck[i], sh.cv[i], s) ? fweight(key_value(sh.ck[i]), s.m) : 0.0;
        },
        n, sh);
  else
    s.Z = ordered_sum(
        [&](int v) -> double {
          const float xv = x(v);
          return fkept(okey(xv), v, s) ? fweight(xv, s.m) : 0.0;
        },
        V, sh);
  if (threadIdx.x == 0) tst[r] = s;
}

// Probability of token y under a truncated row: e^(x_y - m) / Z if kept.
__device__ __forceinline__ double fprob(float xv, int y, const FState& s) {
  return fkept(okey(xv), y, s) ? fweight(xv, s.m) / s.Z : 0.0;
}

// Logit of draft position p at token v: the last pass's (row-major) or, after
// K = 0 passes, the base logits (tile-major).
__device__ __forceinline__ float draft_logit(int k0, const float* __restrict__ lf,
                                             const float* __restrict__ S, int Ms, int V, int p,
                                             int v) {
  return k0 ? S[s_index(p, v, Ms)] : lf[(size_t)p * V + v];
}

// Accept scan of truncated sequences, one wave per sequence: accept y_k iff
// r_k q_k(y_k) <= p_k(y_k), both truncated.  vpos[b] = rejected position or B.
__global__ __launch_bounds__(64) void k_vfaccept(
    int B, int V, int k0, const int32_t* __restrict__ draft, const uint8_t* __restrict__ filt,
    const float* __restrict__ tl, const float* __restrict__ racc, const float* __restrict__ lf,
    const float* __restrict__ S, int Ms, const FState* __restrict__ fst,
    const FState* __restrict__ tst, const float* __restrict__ invT, int32_t* __restrict__ vpos,
    int32_t* __restrict__ out_n, uint32_t* __restrict__ err) {
  const int b = blockIdx.x;
  if (!filt[b] || threadIdx.x != 0) return;
  const float it = invT[b];
  int n = B, bad = 0;
  for (int k = 0; k < B; ++k) {
    const int p = b * B + k;
    int y = draft[p];
    if (y < 0 || y >= V) {
      bad = 1;
      y = 0;
    }
    const double q = fprob(draft_logit(k0, lf, S, Ms, V, p, y) * it, y, fst[p]);
    const double pt = fprob(tl[((size_t)b * (B + 1) + k) * V + y] * it, y,
                            tst[(size_t)b * (B + 1) + k]);
    if (!((double)racc[p] * q <= pt)) {
      n = k;
      break;
    }
  }
  out_n[b] = n;
  vpos[b] = n;
  if (bad) atomicOr(err, XP_DEVERR_TOKEN);
}

// Next token of truncated sequences, one workgroup per sequence: at the
// rejected position k the inverse-CDF sample of max(0, p_k - q_k) (of p_k if
// that has no mass), after B accepts the sample of p_{B+1}; at u_res.
__global__ __launch_bounds__(kFThreads) void k_vffinal(
    int B, int V, int k0, const uint8_t* __restrict__ filt, const float* __restrict__ tl,
    const float* __restrict__ lf, const float* __restrict__ S, int Ms,
    const FState* __restrict__ fst, const FState* __restrict__ tst,
    const float* __restrict__ invT, const int32_t* __restrict__ vpos,
    const float* __restrict__ ures, int32_t* __restrict__ out_next,
    const float* __restrict__ umax, int U) {
  const int b = blockIdx.x;
  if (!filt[b]) return;
  __shared__ FShared sh;
  const float it = invT[b];
  const int n = vpos[b];
  const size_t r = (size_t)b * (B + 1) + n;
  const float* trow = tl + r * V;
  const FState ts = tst[r];
  const bool resid = n < B;
  const int p = b * B + (resid ? n : 0);
  const FState qs = fst[p];
  const double u = (double)ures[b];
  auto xt = [&](int v) -> float { return trow[v] * it; };
  auto prob = [&](float xv, int v) -> double {
    return fkept(okey(xv), v, ts) ? fweight(xv, ts.m) / ts.Z : 0.0;
  };
  // max(0, p - q) where p has mass
  auto residual = [&](double pv, int v) -> double {
    if (!(pv > 0.0)) return 0.0;
    const float xq = draft_logit(k0, lf, S, Ms, V, p, v) * it;
    const double qv = fkept(okey(xq), v, qs) ? fweight(xq, qs.m) / qs.Z : 0.0;
    return pv > qv ? pv - qv : 0.0;
  };
  // both weights vanish outside the target's kept tokens: with few of them
  // (their keys reach max(tk, tp)) they are listed first
  int nc = -1;
  {
    float um[kUPT];
#pragma unroll
    for (int j = 0; j < kUPT; ++j) {
      const int uu = kUPT * threadIdx.x + j;
      um[j] = umax[r * U + (uu < U ? uu : U - 1)];
    }
    nc = collect(xt, V, U, [&](int uu) { return uu * kVUnit; }, um, ts.tk > ts.tp ? ts.tk : ts.tp,
                 sh);
  }
  const int m = nc >= 0 ? nc : V;
  auto tok = [&](int i) { return nc >= 0 ? sh.cv[i] : i; };
  auto wp = [&](int i) -> double {
    return nc >= 0 ? prob(key_value(sh.ck[i]), sh.cv[i]) : prob(xt(i), i);
  };
  auto wr = [&](int i) -> double { return residual(wp(i), tok(i)); };
  int i;
  if (resid) {
    const double Zr = ordered_sum(wr, m, sh);
    if (Zr > 0.0) {
      i = ordered_icdf(wr, m, Zr, u, sh);
    } else {
      const double Zp = ordered_sum(wp, m, sh);
      i = ordered_icdf(wp, m, Zp, u, sh);
    }
  } else {
    const double Zp = ordered_sum(wp, m, sh);
    i = ordered_icdf(wp, m, Zp, u, sh);
  }
  if (threadIdx.x == 0) out_next[b] = tok(i);
}

// ---------------------------------------------------------------------------
int target_units(int V) { return (V + kVUnit - 1) / kVUnit; }

hipError_t launch_filter_params(xp_handle* h, int batch, const uint8_t* temp, const int32_t* top_k,
                                const float* top_p, hipStream_t st) {
  hipLaunchKernelGGL(k_filter_params, dim3((batch + 255) / 256), dim3(256), 0, st, batch, h->V,
                     temp, top_k, top_p, h->ws.filt, h->ws.temp_nf, h->ws.fk, h->ws.fp,
                     h->ws.err);
  return hipGetLastError();
}

hipError_t launch_fsample(xp_handle* h, int batch, int pass, uint32_t flags,
                          const int32_t* seed_ids, const float* u_draft, hipStream_t st) {
  const int M = batch * h->B;
  int32_t* Ynew = h->ws.Y[(pass + 1) % 2];
  const int early = (flags & XP_EARLY_EXIT) ? 1 : 0;
  const int U = pass < 0 ? h->lm_units_cur : h->read_units;    // of the partials in stats
  if (pass < 0)
    hipLaunchKernelGGL((k_fsample<0>), dim3(M), dim3(kFThreads), 0, st, h->B, h->V, M, h->ws.s, M,
                       h->ws.lf, h->ws.filt, h->ws.fk, h->ws.fp, h->ws.invT, u_draft, seed_ids,
                       Ynew, h->ws.fst, h->ws.iters, early, h->ws.stats, h->ntiles, U);
  else
    hipLaunchKernelGGL((k_fsample<1>), dim3(M), dim3(kFThreads), 0, st, h->B, h->V, M, h->ws.s, M,
                       h->ws.lf, h->ws.filt, h->ws.fk, h->ws.fp, h->ws.invT, u_draft, nullptr,
                       Ynew, h->ws.fst, h->ws.iters, early, h->ws.stats, h->ntiles, U);
  return hipGetLastError();
}

hipError_t launch_vfilter(xp_handle* h, int batch, const int32_t* draft, const float* tl,
                          const float* racc, const float* ures, int32_t* out_n, int32_t* out_next,
                          hipStream_t st) {
  const int M = batch * h->B;
  const int k0 = h->state_k0 ? 1 : 0;
  const int U = target_units(h->V);
  hipLaunchKernelGGL(k_row_units, dim3((h->V + kVUnitTok - 1) / kVUnitTok, h->B + 1, batch),
                     dim3(256), 0, st, h->B, h->V, tl, h->ws.filt, h->ws.invT, h->ws.tumax, U);
  hipLaunchKernelGGL(k_vfstate, dim3(h->B + 1, batch), dim3(kFThreads), 0, st, h->B, h->V, tl,
                     h->ws.filt, h->ws.fk, h->ws.fp, h->ws.invT, h->ws.tst, h->ws.tumax, U);
  hipLaunchKernelGGL(k_vfaccept, dim3(batch), dim3(64), 0, st, h->B, h->V, k0, draft, h->ws.filt,
                     tl, racc, h->ws.lf, h->ws.s, M, h->ws.fst, h->ws.tst, h->ws.invT, h->ws.vpos,
                     out_n, h->ws.err);
  hipLaunchKernelGGL(k_vffinal, dim3(batch), dim3(kFThreads), 0, st, h->B, h->V, k0, h->ws.filt,
                     tl, h->ws.lf, h->ws.s, M, h->ws.fst, h->ws.tst, h->ws.invT, h->ws.vpos, ures,
                     out_next, h->ws.tumax, U);
  return hipGetLastError();
}

}  // namespace xp
