// A7: Read + Correct, l = s + W_r z (eqs. read, correct), fused with the first
// stage of token selection: per vocabulary unit the kernel leaves argmax keys
// (greedy rows) or (max, sum exp(l - max)) (sampled rows); no logit row is
// written on the fast path.
//
// W_r is streamed once per pass and 16-position block, tile by tile (16
// vocabulary rows), straight into MFMA operand registers.
#include <type_traits>

#include "xp_internal.h"
#include "xp_tiles.h"

namespace xp {

// Where a Read writes logit rows ([M][V] fp32, row-major): every position's to
// `out` (the caller's logits, written by the last pass only), those of rows
// that truncate (filt) to `lf` (the workspace rows their sampler reads, every
// pass).  Either may be null.  vec: V is a multiple of 4 and both are 16-byte
// aligned, so a lane's four consecutive rows go out as one 16-byte store and a
// tile's 16 rows of a position fill a 64-byte segment with one instruction.
// Six passes with the logits at V = 151936, against every pass storing them 4
// bytes at a time: a refine + verify step of 2048 positions 8.33 -> 5.10 ms,
// of 512 positions 2.17 -> 1.36 ms, of 128 positions 0.94 -> 0.74 ms.
struct LogitRows {
  float* out;
  float* lf;
  const uint8_t* filt;
  int vec;
};

__device__ __forceinline__ void put_rows(float* dst, size_t at, const floatx4& v, int row0, int V,
                                         bool vec) {
  if (vec) {
    if (row0 < V) *reinterpret_cast<floatx4*>(dst + at) = v;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (row0 + i < V) dst[at + i] = v[i];
  }
}

// ---------------------------------------------------------------------------
// A7: l = s + W_r z, r = 256.  Every wave streams its own unit of tiles with
// the full k range (one chain of MFMAs per tile, seeded with s); the position
// block's z fragments sit in LDS, shared by the waves.  A unit of at most
// kReadRes tiles (the common case) keeps all of them in registers: every W_r,
// s and z load of the wave is issued, unconditionally, before the first
// MFMA, so the whole unit is in flight at once (a short unit re-reads its
// last tile, which hits in L2).  Workgroups merge their waves' argmax keys;
// sampled rows write one (max, sum) per wave unit.
// ---------------------------------------------------------------------------
// ROWS: the launch writes logit rows (without them the kernel must not carry their
// tests: 17.4 against 17.0 us at V = 151936, six passes a step).
template <bool ROWS>
__global__ __launch_bounds__(kReadWaves * kWave) void k_read(
    const uint16_t* __restrict__ W, const uint16_t* __restrict__ Z, const float* __restrict__ S, int Ms, int V,
    int M, int ntiles, int U, uint64_t* __restrict__ keys, Stat* __restrict__ stats,
    const uint8_t* __restrict__ temp, int B, LogitRows rows, const int32_t* __restrict__ ctrl,
    int skip_when_done, const float* __restrict__ invT) {
  if (skip_when_done && ctrl[1]) return;          // every sequence is at its fixed point
  using T = uint16_t;
  constexpr int NU = ReadTile<T>::NU;
  constexpr int NR = 5;                           // resident tiles per wave (32 VGPRs each)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u = blockIdx.x * kReadWaves + wave, p0 = blockIdx.y * kTile;
  const int tlo = unit_tile_lo(u, ntiles, U), thi = unit_tile_lo(u + 1, ntiles, U);
  const int n = thi - tlo;
  __shared__ u32x4 zl[NU][64];
  __shared__ uint64_t kred[kReadWaves][kTile];
  // per-wave transpose tile (16 rows x 32 chunks, chunk XOR-swizzled by row:
  // conflict-free for the row-contiguous writes and the MFMA-order reads)
  __shared__ u32x4 tbuf[kReadWaves][16 * 32];

  const int p = p0 + (lane & 15);
  const bool act = p < M;
  const int pc = act ? p : M - 1;
  const float pit = invT[pc / B];               // sampled rows: softmax(l / T)
  const bool to_lf = ROWS && rows.lf != nullptr && act && rows.filt[pc / B] != 0;
  const bool to_out = ROWS && rows.out != nullptr && act;
  uint64_t best = kKeyMin;
  Stat st = stat_empty();
  bool sample = false;

  bool any_sample = false;                      // wave-uniform: some lane of the wave samples
  // Selection partials of one tile, without branches on the greedy path: the
  // key of every element is formed and kept or dropped by a select.
  auto epilogue = [&](const floatx4& acc, int t) {
    const int row0 = t * kTile + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool v = act && row0 + i < V && !sample;
      const uint64_t key = umax64(best, argmax_key(acc[i], (uint32_t)(row0 + i)));
      best = v ? key : best;
    }
    if (any_sample) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool v = act && row0 + i < V && sample;
        const Stat nx = stat_merge(st, Stat{acc[i] * pit, 1.f});
        st.m = v ? nx.m : st.m;
        st.s = v ? nx.s : st.s;
      }
    }
    if (to_out) put_rows(rows.out, (size_t)p * V + row0, acc, row0, V, rows.vec);
    if (to_lf) put_rows(rows.lf, (size_t)p * V + row0, acc, row0, V, rows.vec);
  };
  // z fragments, read once from LDS into registers after the barrier
  u32x4 zr[NU];
  auto fetch_z = [&]() {
#pragma unroll
    for (int i = 0; i < NU; ++i) zr[i] = zl[i][lane];
  };
  auto chain_lds = [&](const u32x4 (&a)[NU], floatx4 acc) {
#pragma unroll
    for (int i = 0; i < NU; ++i) acc = Mfma<T>::mma(a[i], zr[i], acc);
    return acc;
  };
  auto load_s = [&](int t) {
    const floatx4 v = *reinterpret_cast<const floatx4*>(S + s_index(pc, t * kTile + 4 * (lane >> 4), Ms));
    return act ? v : floatx4{0.f, 0.f, 0.f, 0.f};
  };
  // z fragments of the position block, one 16-byte chunk per thread
  constexpr int kZPer = (NU * 64 + kReadWaves * kWave - 1) / (kReadWaves * kWave);
  u32x4 zv[kZPer];
  auto load_z = [&]() {
#pragma unroll
    for (int j = 0; j < kZPer; ++j) {
      const int c = threadIdx.x + kReadWaves * kWave * j;
      const int zi = (c / 64) % NU, zlane = c % 64;
      const int zp = p0 + (zlane & 15);
      zv[j] = ld16(Z + (size_t)(zp < M ? zp : M - 1) * 256 + (zlane >> 4) * ReadTile<T>::EPB +
                   zi * ReadTile<T>::KU);
      if (zp >= M) zv[j] = u32x4{0u, 0u, 0u, 0u};
    }
  };
  static_assert(NU * 64 == kZPer * kReadWaves * kWave, "z chunks fill the workgroup exactly");
  auto put_z = [&]() {                          // no guard: a guarded store would sink its load
#pragma unroll
    for (int j = 0; j < kZPer; ++j) {
      const int c = threadIdx.x + kReadWaves * kWave * j;
      zl[c / 64][c % 64] = zv[j];
    }
  };

  if (n >= 1 && n <= NR) {
    // Line-complete loads: instruction i of a tile reads its rows 2i, 2i+1
    // (1 KB contiguous, non-temporal); each tile is then transposed through
    // the wave's LDS tile into the MFMA operand order of ReadTile::load_w,
    // so the chain sees exactly the operands of the rescans.
    // Issue order = use order (z, s, then the tiles): the vector-memory
    // counter drains in order, so tile j waits only for the loads before it.
    u32x4 a[NR][8];
    floatx4 c[NR];
    const int lrow = lane >> 5, lch = lane & 31;
    const int tv = load_flag(temp, pc / B, S);
    load_z();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < NR; ++j) c[j] = load_s(tlo + (j < n ? j : n - 1));
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int t = tlo + (j < n ? j : n - 1);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        int row = t * kTile + 2 * i + lrow;
        row = row < V ? row : V - 1;
        a[j][i] = ld16_nt(W + (size_t)row * 256 + lch * 8);
      }
    }
    sample = act && tv != 0;
    any_sample = __ballot(sample) != 0;
    put_z();
    lds_barrier();
    fetch_z();
    u32x4* tb = tbuf[wave];
    const int li = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      if (j < n) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int row = 2 * i + lrow;
          tb[row * 32 + (lch ^ row)] = a[j][i];
        }
        wave_lds_order();
        u32x4 m[NU];
#pragma unroll
        for (int i = 0; i < NU; ++i) m[i] = tb[li * 32 + ((4 * i + g) ^ li)];
        wave_lds_order();
        epilogue(chain_lds(m, c[j]), tlo + j);
      }
    }
  } else {
    load_z();
    const int tv = load_flag(temp, pc / B, S);
    sample = act && tv != 0;
    any_sample = __ballot(sample) != 0;
    put_z();
    __syncthreads();
    fetch_z();
    u32x4 a[NU];
    for (int t = tlo; t < thi; ++t) {
      ReadTile<T>::load_w(W, V, t, lane, a);
      epilogue(chain_lds(a, load_s(t)), t);
    }
  }
#pragma unroll
  for (int m = 16; m < 64; m <<= 1) {
    best = umax64(best, shfl_xor_u64(best, m));
    Stat o{__shfl_xor(st.m, m, kWave), __shfl_xor(st.s, m, kWave)};
    st = stat_merge(st, o);
  }
  if (lane < 16 && sample) stats[(size_t)p * U + u] = st;

  if (lane < 16) kred[wave][lane] = best;
  __syncthreads();
  if (threadIdx.x < kTile) {
    uint64_t b = kKeyMin;
    for (int w = 0; w < kReadWaves; ++w) b = umax64(b, kred[w][threadIdx.x]);
    const int pp = p0 + threadIdx.x;
    if (pp < M) keys[(size_t)blockIdx.x * M + pp] = b;
  }
}

// ---------------------------------------------------------------------------
// A7 in fp32: a wave takes the tiles of GS units, PB 16-position blocks per
// workgroup (their z in LDS).  A block at a time (the form before) read W_r once
// per 16 positions: 35.6 us a pass at 33 positions of V = 33001, bound by those
// reads and by one chain of dependent matrix operations per wave; PB interleaved
// chains share every tile.  Each chain is ReadTile::chain's, so the logits are those
// of the rescans.
//
// ONE: a wave's units hold one tile together at most (GS ntiles <= U).  Then no
// second tile's registers are kept and two workgroups fit a CU, one's loads under
// the other's matrix operations.  GS = 2 (vocabularies up to 16384 rows, whose units
// are at least half empty) keeps all eight waves of a workgroup at work where there
// are more workgroups than CUs.
//
// us a launch, event-timed, one block a workgroup column at a time / the form with
// one workgroup per CU, the flags behind the tile and no GS / now: V = 4000, 16 / 80 /
// 512 positions 14 / 12 / 9, 14 / 16 / 11, 43 / 39 / 19; V = 12000, 80 positions 24 /
// 32 / 16; V = 33001, 48 positions 36 / 25 / 20; V = 151936, 16 / 64 positions 30 /
// 34 / 33, 102 / 70 / 67.
// ---------------------------------------------------------------------------
template <int PB, int GS, bool ONE>
__global__ __launch_bounds__(kReadWaves * kWave) void k_read_f32(
    const float* __restrict__ W, const float* __restrict__ Z, const float* __restrict__ S, int Ms,
    int V, int M, int ntiles, int U, uint64_t* __restrict__ keys, Stat* __restrict__ stats,
    const uint8_t* __restrict__ temp, int B, LogitRows rows, const int32_t* __restrict__ ctrl,
    int skip_when_done, const float* __restrict__ invT) {
  if (skip_when_done && ctrl[1]) return;          // every sequence is at its fixed point
  using RT = ReadTile<float>;
  constexpr int NU = RT::NU;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the wave's units u0 .. u0 + GS - 1 (none past U) and their tiles
  const int u0 = (blockIdx.x * kReadWaves + wave) * GS, p0 = blockIdx.y * (kTile * PB);
  const int ub = u0 < U ? u0 : U, ue = u0 + GS < U ? u0 + GS : U;
  const int tlo = unit_tile_lo(ub, ntiles, U), thi = unit_tile_lo(ue, ntiles, U);
  const int tl = thi > tlo ? tlo : (tlo < ntiles ? tlo : ntiles - 1);   // an empty unit loads a tile it drops
  __shared__ u32x4 zl[PB][NU][64];
  __shared__ uint64_t kred[kReadWaves][PB * kTile];

  int pc[PB];
  bool act[PB], sample[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int p = p0 + kTile * pb + (lane & 15);
    act[pb] = p < M;
    pc[pb] = act[pb] ? p : M - 1;
  }
  auto load = [&](int t, u32x4 (&w)[NU], floatx4 (&s4)[PB]) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
      s4[pb] = *reinterpret_cast<const floatx4*>(S + s_index(pc[pb], t * kTile + 4 * (lane >> 4), Ms));
    RT::load_w(W, V, t, lane, w);
  };
  uint64_t best[PB];
  Stat st[PB];
  float pit[PB];
  // LONG: a unit of two tiles or more.  One block keeps its z in registers and takes
  // a tile at a time (V = 60000 16.6 us; two in flight 19.2 to 23.6: its waves wait
  // for memory, not for each other).  More blocks have two tiles in flight, in loops
  // whose loads are neither conditional (a wait past a join of both cases waits for
  // the later tile too) nor in vain; with four blocks that form spills, and the
  // short loop is the faster one (66.6 against 71.2 us at V = 151936).
  auto run = [&](auto longer) __attribute__((always_inline)) {
    constexpr bool LONG = decltype(longer)::value, kZReg = LONG && PB == 1;
    u32x4 a[NU], an[LONG ? NU : 1];
    floatx4 c[PB], cn[LONG ? PB : 1];
    // z fragments of the blocks, 16-byte chunks in turn over the threads; they and the
    // flags go out first, so that only they are waited for before the barrier
    constexpr int kZPer = PB * NU * 64 / (kReadWaves * kWave);
    u32x4 zv[kZPer];
#pragma unroll
    for (int j = 0; j < kZPer; ++j) {
      const int ch = threadIdx.x + kReadWaves * kWave * j;
      const int pb = ch / (NU * 64), zi = (ch / 64) % NU, zlane = ch % 64;
      const int zp = p0 + kTile * pb + (zlane & 15);
      zv[j] = ld16(Z + (size_t)(zp < M ? zp : M - 1) * 256 + (zlane >> 4) * RT::EPB + zi * RT::KU);
    }
    int tv[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      tv[pb] = load_flag(temp, pc[pb] / B, S);
      pit[pb] = invT[pc[pb] / B];
    }
    asm volatile("" ::: "memory");
    load(tl, a, c);
    if constexpr (LONG && PB > 1) load(tlo + 1, an, cn);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      sample[pb] = act[pb] && tv[pb] != 0;
      best[pb] = kKeyMin;
      st[pb] = stat_empty();
    }
#pragma unroll
    for (int j = 0; j < kZPer; ++j) {
      const int ch = threadIdx.x + kReadWaves * kWave * j;
      const int zp = p0 + kTile * (ch / (NU * 64)) + (ch & 15);
      zl[ch / (NU * 64)][(ch / 64) % NU][ch % 64] = zp < M ? zv[j] : u32x4{0u, 0u, 0u, 0u};
    }
    lds_barrier();
    u32x4 zr[kZReg ? NU : 1];                     // one block's z stays in registers
    if constexpr (kZReg) {
#pragma unroll
      for (int i = 0; i < NU; ++i) zr[i] = zl[0][i][lane];
    }
    auto tile = [&](const u32x4 (&w)[NU], const floatx4 (&s4)[PB], int t) {
      floatx4 acc[PB];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) acc[pb] = act[pb] ? s4[pb] : floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (kZReg) {
#pragma unroll
        for (int i = 0; i < NU; ++i) acc[0] = Mfma<float>::mma(w[i], zr[i], acc[0]);
      } else {
        // z one load unit ahead (all of it at once would not fit the registers)
        u32x4 z[2][PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) z[0][pb] = zl[pb][0][lane];
#pragma unroll
        for (int i = 0; i < NU; ++i) {
          if (i + 1 < NU) {
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) z[(i + 1) & 1][pb] = zl[pb][i + 1][lane];
          }
          asm volatile("" ::: "memory");
#pragma unroll
          for (int pb = 0; pb < PB; ++pb) acc[pb] = Mfma<float>::mma(w[i], z[i & 1][pb], acc[pb]);
        }
      }
      const int row0 = t * kTile + 4 * (lane >> 4);
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const int p = p0 + kTile * pb + (lane & 15);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool v = act[pb] && row0 + i < V;
          const uint64_t key = umax64(best[pb], argmax_key(acc[pb][i], (uint32_t)(row0 + i)));
          best[pb] = v && !sample[pb] ? key : best[pb];
          if (sample[pb] && v) st[pb] = stat_merge(st[pb], Stat{acc[pb][i] * pit[pb], 1.f});
        }
        if (act[pb] && rows.out) put_rows(rows.out, (size_t)p * V + row0, acc[pb], row0, V, rows.vec);
        if (act[pb] && rows.lf && rows.filt[pc[pb] / B])
          put_rows(rows.lf, (size_t)p * V + row0, acc[pb], row0, V, rows.vec);
      }
    };
    if constexpr (LONG && PB == 1) {
#pragma unroll 1
      for (int t = tlo; t < thi; ++t) {
        if (t > tlo) load(t, a, c);
        tile(a, c, t);
      }
    } else if constexpr (LONG && PB == 4) {
#pragma unroll 1
      for (int t = tlo; t < thi; t += 2) {
        tile(a, c, t);
        if (t + 1 >= thi) break;
        if (t + 2 < thi) load(t + 2, a, c);
        tile(an, cn, t + 1);
        if (t + 3 < thi) load(t + 3, an, cn);
      }
    } else if constexpr (LONG) {
      int t = tlo;
#pragma unroll 1
      for (; t + 3 < thi; t += 2) {
        tile(a, c, t);
        load(t + 2, a, c);
        tile(an, cn, t + 1);
        load(t + 3, an, cn);
      }
      if (t + 2 < thi) {
        tile(a, c, t);
        load(t + 2, a, c);
        tile(an, cn, t + 1);
        tile(a, c, t + 2);
      } else {
        tile(a, c, t);
        tile(an, cn, t + 1);
      }
    } else if (tlo < thi) {
      tile(a, c, tlo);
    }
  };
  if constexpr (ONE) {
    run(std::false_type{});
  } else {
    if (thi - tlo > 1)                            // wave-uniform
      run(std::true_type{});
    else
      run(std::false_type{});
  }
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
#pragma unroll
    for (int m = 16; m < 64; m <<= 1) {
      best[pb] = umax64(best[pb], shfl_xor_u64(best[pb], m));
      const Stat o{__shfl_xor(st[pb].m, m, kWave), __shfl_xor(st[pb].s, m, kWave)};
      st[pb] = stat_merge(st[pb], o);
    }
    if (lane < 16 && sample[pb]) {
#pragma unroll
      for (int q = 0; q < GS; ++q) {                // (ONE: the tile is in one of the units)
        const int u = u0 + q;
        if (u < U)
          stats[(size_t)(p0 + kTile * pb + lane) * U + u] =
              GS == 1 || unit_tile_lo(u + 1, ntiles, U) > unit_tile_lo(u, ntiles, U)
                  ? st[pb] : stat_empty();
      }
    }
    if (lane < 16) kred[wave][kTile * pb + lane] = best[pb];
  }
  __syncthreads();
  if (threadIdx.x < PB * kTile) {
    const int pp = p0 + threadIdx.x;
#pragma unroll
    for (int q = 0; q < GS; ++q) {                  // the key rows of GS read workgroups
      const int row = blockIdx.x * GS + q;
      uint64_t b = kKeyMin;
      for (int w = 0; w < kReadWaves / GS; ++w)
        b = umax64(b, kred[q * (kReadWaves / GS) + w][threadIdx.x]);
      if (pp < M && row * kReadWaves < U) keys[(size_t)row * M + pp] = b;
    }
  }
}

// ---------------------------------------------------------------------------
// A7 for many positions.  The stream kernel above re-reads W_r once per
// 16-position block; here a workgroup takes the tiles of one read workgroup
// (8 wave units) for 128 P positions: each wave keeps the z fragments of its
// 16 P positions in registers and runs through all the workgroup's tiles, so
// W_r is read once per 128 P positions and the pass is bound by reading s.
// The W_r tile and the s operands of every tile go through a ring of LDS
// stages filled by global-to-LDS loads three tiles ahead (each wave loads one
// 1 KB part of the W_r tile and the s of its own positions), so up to 100 KB
// per CU is in flight without staging registers.  Each (tile, 16 positions)
// product is the chain of matrix operations seeded with s used by the stream
// kernel and the sampling rescan (ReadTile), so all of them produce the same
// fp32 logits.  Outputs have the stream kernel's layout: one key row per
// workgroup, one (max, sum) per wave unit and position.
constexpr int kRmLds = 163840;                   // bytes of LDS the ring may take
constexpr int kRmMaxStages = 8;
constexpr int kRmMaxP = 4;                       // position blocks per wave (launch cap)
constexpr int kRmOutLd = 36;                     // floats per position of a store buffer (32 + pad)
constexpr int kRmOutWave = 16 * kRmOutLd;        // floats of a wave's store buffer

// W_r tile in LDS: 16 rows x 32 chunks of 16 bytes, chunk c of row r at slot
// 32 r + (c ^ r); s of 16 positions x 16 rows: chunk c (4 rows) of position q
// at slot 4 q + (c ^ (q / 4)).  The fragment reads (16 rows or positions, one
// chunk) then hit 16 different bank groups.
__device__ __forceinline__ int rm_wslot(int r, int c) { return 32 * r + (c ^ r); }
__device__ __forceinline__ int rm_sslot(int q, int c) { return 4 * q + ((c ^ (q >> 2)) & 3); }

// EE (early exit): a wave whose positions all belong to sequences at their
// fixed point is dead: its s loads go to one fixed address (every wave still
// issues the same number of loads per tile, which the waits count on, and its
// part of each W_r tile, which the other waves read), and its products,
// selection partials and outputs are skipped.
//
// WM: how logit rows are written (LogitRows).  0: not at all.  1: straight from
// the accumulators, 16 bytes per lane (rows.vec).  2: V or a pointer is not
// 16-byte aligned; two tiles' values of 16 positions pass through a per-wave
// LDS buffer, so that a store instruction writes 32 consecutive rows of two
// positions instead of 4 bytes in each of 64 places; the buffer takes 18 KB
// from the ring.  (V = 151935, H = 1024: the step at 2048 positions 8.52 ->
// 3.63 ms, at 512 positions 2.22 -> 0.97 ms, at 128 positions 0.71 -> 0.55 ms.)
// A wait count that leaves the stores of the later tiles outstanding too gained
// nothing (5.10 against 5.11 ms at 2048 positions).
template <int P, bool EE, int WM>
__global__ __launch_bounds__(kReadWaves * kWave) void k_read_multi(
    const uint16_t* __restrict__ W, const uint16_t* __restrict__ Z, const float* __restrict__ S,
    int Ms, int V, int M, int ntiles, int U, uint64_t* __restrict__ keys,
    Stat* __restrict__ stats, const uint8_t* __restrict__ temp, int B,
    LogitRows rows, const int32_t* __restrict__ ctrl, int skip_when_done,
    int nwg, int ny, int gs, const float* __restrict__ invT, const int32_t* __restrict__ iters) {
  static_assert(kReadWaves == 8, "one 1 KB load per wave fills a 16-row tile");
  if (skip_when_done && ctrl[1]) return;          // every sequence is at its fixed point
  using RT = ReadTile<uint16_t>;
  constexpr int NU = RT::NU;
  constexpr int WSL = 512, SSL = kReadWaves * P * 64;          // 16-byte slots per stage
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // A workgroup takes the gs consecutive read workgroups [g_lo, g_hi) (their
  // tiles in order, one key row per read workgroup) for position group py.
  // Workgroup b runs on XCD b % 8; the ny position groups of one group of
  // read workgroups sg are b = 8 (ny (sg / 8) + y) + sg % 8, y < ny: the
  // same XCD at about the same time, so W_r tiles read by the first come
  // from L2 for the others
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int sg = (slot / ny) * 8 + xcd, py = slot - (slot / ny) * ny;
  const int g_lo = sg * gs;
  if (g_lo >= nwg) return;                        // whole workgroup
  const int g_hi = min(nwg, g_lo + gs);
  const int u_lo = g_lo * kReadWaves, u_hi = g_hi * kReadWaves;
  const int t0 = unit_tile_lo(u_lo, ntiles, U), n = unit_tile_lo(u_hi, ntiles, U) - t0;
  const int pw = py * (kReadWaves * kTile * P) + wave * (kTile * P);
  // as many stages as fit: the deeper the ring, the more tiles are in flight
  constexpr int kOut = WM == 2 ? kReadWaves * kRmOutWave : 0;   // floats of the store buffers
  constexpr int NS0 = (kRmLds - 4 * kOut) / ((WSL + SSL) * 16);
  constexpr int kRmStages = NS0 < kRmMaxStages ? NS0 : kRmMaxStages;
  __shared__ u32x4 lds[kRmStages * (WSL + SSL) + kOut / 4];     // [stage][W tile | s], buffers
  if (EE) {
    // early exit: nothing to do when every sequence of the workgroup's
    // positions is at its fixed point (the flag lives in the first ring
    // slot, which no load has touched yet)
    const int P0 = py * (kReadWaves * kTile * P);
    const int P1 = min(M, P0 + kReadWaves * kTile * P);
    const int b0 = P0 / B, nb = (P1 - 1) / B - b0 + 1;
    bool live = false;
    for (int i = threadIdx.x; i < nb; i += kReadWaves * kWave) live |= iters[b0 + i] == 0;
    uint32_t* flag = reinterpret_cast<uint32_t*>(&lds[0]);
    if (threadIdx.x == 0) *flag = 0u;
    __syncthreads();
    if (live) *flag = 1u;
    __syncthreads();
    const bool any = *flag != 0u;
    __syncthreads();
    if (!any) return;                             // whole workgroup
  }

  u32x4 zf[P][NU];
#pragma unroll
  for (int pb = 0; pb < P; ++pb) RT::load_z(Z, M, pw + kTile * pb, lane, zf[pb]);
  bool act[P], sample[P], to_lf[P];
  float pit[P];                                   // sampled rows: softmax(l / T)
  bool any = false, live = false;
#pragma unroll
  for (int pb = 0; pb < P; ++pb) {
    const int p = pw + kTile * pb + (lane & 15);
    act[pb] = p < M;
    if (EE) live = live || (act[pb] && iters[(act[pb] ? p : M - 1) / B] == 0);
    sample[pb] = act[pb] && load_flag(temp, (act[pb] ? p : M - 1) / B, S) != 0;
    pit[pb] = invT[(act[pb] ? p : M - 1) / B];
    to_lf[pb] = WM != 0 && rows.lf != nullptr && act[pb] && rows.filt[(act[pb] ? p : 0) / B] != 0;
    any = any || sample[pb];
  }
  const bool any_sample = __ballot(any) != 0;    // wave-uniform
  const bool wdead = EE && __ballot(live) == 0;   // wave-uniform
  // per position block, wave-uniform: does any lane take the greedy maximum,
  // any the softmax partials?  (With B a multiple of 16 a block lies in one
  // sequence and does only one of the two.)
  bool do_max[P], do_sum[P];
#pragma unroll
  for (int pb = 0; pb < P; ++pb) {
    do_max[pb] = __ballot(act[pb] && !sample[pb]) != 0;
    do_sum[pb] = __ballot(sample[pb]) != 0;
  }
  // greedy rows: running maximum and its row (rows arrive in increasing order
  // in every lane, so a strict comparison keeps the lowest index of a tie;
  // -0 == +0 as in the key order).  Other rows start at +inf, which no value
  // exceeds, so they keep the empty key without a mask in the loop.
  float bv[P];
  uint32_t bi[P];
  Stat st[P];
#pragma unroll
  for (int pb = 0; pb < P; ++pb) {
    bv[pb] = (act[pb] && !sample[pb]) ? -INFINITY : INFINITY;
    bi[pb] = 0xFFFFFFFFu;
    st[pb] = stat_empty();
  }
  // the key row of every read workgroup that ends at or before tile boundary
  // tend, from the running maxima, which then restart
  int gc = g_lo, ge = unit_tile_lo((g_lo + 1) * kReadWaves, ntiles, U);
  auto flush_keys = [&](int tend) {
    while (gc < g_hi && ge <= tend) {             // wave-uniform
#pragma unroll
      for (int pb = 0; pb < P; ++pb) {
        uint64_t best = bi[pb] == 0xFFFFFFFFu ? kKeyMin : argmax_key(bv[pb], bi[pb]);
#pragma unroll
        for (int m = 16; m < 64; m <<= 1) best = umax64(best, shfl_xor_u64(best, m));
        const int p = pw + kTile * pb + (lane & 15);
        if (lane < 16 && act[pb] && !wdead) keys[(size_t)gc * M + p] = best;
        bv[pb] = (act[pb] && !sample[pb]) ? -INFINITY : INFINITY;
        bi[pb] = 0xFFFFFFFFu;
      }
      ++gc;
      ge = unit_tile_lo((gc + 1) * kReadWaves, ntiles, U);
    }
  };

  // loads of tile j (clamped into the range, so that every wave issues the
  // same number of loads per tile) into stage j % kRmStages
  const int wrow = (kWave * wave + lane) >> 5;
  const int wchunk = ((kWave * wave + lane) & 31) ^ wrow;
  const int sq = lane >> 2, sc = (lane & 3) ^ ((sq >> 2) & 3);
  const float* sbase[P];
#pragma unroll
  for (int pb = 0; pb < P; ++pb) {
    const int p = pw + kTile * pb + sq;
    sbase[pb] = S + s_index(p < M ? p : M - 1, 4 * sc, Ms);
    if (wdead) sbase[pb] = S + 4 * (lane & 3);    // fixed, in cache after the first tile
  }
  auto issue = [&](int j) {
    const int t = t0 + (j < n ? j : n - 1);
    int row = t * kTile + wrow;
    row = row < V ? row : V - 1;
    u32x4* stage = lds + (j % kRmStages) * (WSL + SSL);
    lds_dma16(W + (size_t)row * 256 + 8 * wchunk, stage + kWave * wave);
#pragma unroll
    for (int pb = 0; pb < P; ++pb)
      lds_dma16_nt(sbase[pb] + (wdead ? (size_t)0 : (size_t)t * Ms * kTile),
                stage + WSL + kWave * (P * wave + pb));
  };
  // (max, sum) of every unit that ends at or before tile boundary tend
  int uc = u_lo, ue = unit_tile_lo(u_lo + 1, ntiles, U);
  auto flush_until = [&](int tend) {
    while (uc < u_hi && ue <= tend) {             // wave-uniform
      if (any_sample) {
#pragma unroll
        for (int pb = 0; pb < P; ++pb) {
          Stat q = st[pb];
#pragma unroll
          for (int m = 16; m < 64; m <<= 1) {
            const Stat o{__shfl_xor(q.m, m, kWave), __shfl_xor(q.s, m, kWave)};
            q = stat_merge(q, o);
          }
          const int p = pw + kTile * pb + (lane & 15);
          if (lane < 16 && sample[pb] && !wdead) stats[(size_t)p * U + uc] = q;
          st[pb] = stat_empty();
        }
      }
      ++uc;
      ue = unit_tile_lo(uc + 1, ntiles, U);
    }
  };

  // WM 2: the 32 rows from row lo of the wave's positions, from the even
  // tile's values (lo, in c0) and the odd one's (c1); rows past hi - 1 are
  // not written
  float* obuf = reinterpret_cast<float*>(lds + kRmStages * (WSL + SSL)) + wave * kRmOutWave;
  auto put_pair = [&](const floatx4 (&c0)[P], const floatx4 (&c1)[P], int lo, int hi) {
    if constexpr (WM == 2) {
      const int q = lane & 15, r4 = 4 * (lane >> 4), half = lane >> 5, r = lane & 31;
      const uint32_t lane_at = (uint32_t)(half * V + r);
#pragma unroll
      for (int pb = 0; pb < P; ++pb) {
        const uint32_t lfm = (uint32_t)__ballot(lane < 16 && to_lf[pb]);
        *reinterpret_cast<floatx4*>(obuf + kRmOutLd * q + r4) = c0[pb];
        *reinterpret_cast<floatx4*>(obuf + kRmOutLd * q + 16 + r4) = c1[pb];
        wave_lds_order();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          // a wave-uniform address and one lane offset
          const int pi = pw + kTile * pb + 2 * i, qp = 2 * i + half;
          const size_t base = (size_t)pi * V + lo;
          const float v = obuf[kRmOutLd * qp + r];
          if (pi + half < M && lo + r < hi) {
            if (rows.out) (rows.out + base)[lane_at] = v;
            if ((lfm >> qp) & 1u) (rows.lf + base)[lane_at] = v;
          }
        }
        wave_lds_order();
      }
    }
  };
  floatx4 held[P];                                // WM 2: the even tile of a pair
#pragma unroll
  for (int pb = 0; pb < P; ++pb) held[pb] = floatx4{0.f, 0.f, 0.f, 0.f};

  flush_until(t0);                                // units without tiles
  flush_keys(t0);                                 // read workgroups without tiles
#pragma unroll
  for (int j = 0; j < kRmStages - 1; ++j) issue(j);
  constexpr int kPend = (kRmStages - 2) * (1 + P); // loads of the later tiles
  static_assert(kPend < 64, "vmcnt field");
  for (int j = 0; j < n; ++j) {
    // tile j's loads are done once only the later tiles' are outstanding;
    // the barrier then covers every wave's part of stage j, and every wave's
    // reads of the stage that the next issue overwrites (tile j - 1)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070 | (kPend & 15) | ((kPend >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(j + kRmStages - 1);
    if (wdead) continue;                           // wave-uniform
    const u32x4* stage = lds + (j % kRmStages) * (WSL + SSL);
    u32x4 a[NU];
#pragma unroll
    for (int i = 0; i < NU; ++i) a[i] = stage[rm_wslot(lane & 15, (lane >> 4) + 4 * i)];
    floatx4 c[P];
#pragma unroll
    for (int pb = 0; pb < P; ++pb)
      c[pb] = __builtin_bit_cast(floatx4, stage[WSL + kWave * (P * wave + pb) +
                                               rm_sslot(lane & 15, lane >> 4)]);
    const int t = t0 + j;
    const int row0 = t * kTile + 4 * (lane >> 4);
    const bool last = (t + 1) * kTile > V;         // wave-uniform: rows past V in this tile
    // the P chains interleaved (each is RT::chain's sequence of operations)
    floatx4 accs[P];
#pragma unroll
    for (int pb = 0; pb < P; ++pb) accs[pb] = c[pb];
#pragma unroll
    for (int i = 0; i < NU; ++i)
#pragma unroll
      for (int pb = 0; pb < P; ++pb) accs[pb] = Mfma<uint16_t>::mma(a[i], zf[pb][i], accs[pb]);
    if (last) {                                    // wave-uniform
      // rows past V become -inf: no maximum takes them, no sum counts them
#pragma unroll
      for (int pb = 0; pb < P; ++pb)
#pragma unroll
        for (int i = 0; i < 4; ++i) accs[pb][i] = row0 + i < V ? accs[pb][i] : -INFINITY;
    }
#pragma unroll
    for (int pb = 0; pb < P; ++pb) {
      const floatx4 acc = accs[pb];
      if (do_max[pb]) {                            // wave-uniform
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool take = acc[i] > bv[pb];
          bv[pb] = take ? acc[i] : bv[pb];
          bi[pb] = take ? (uint32_t)(row0 + i) : bi[pb];
        }
      }
      if (do_sum[pb]) {                            // wave-uniform
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = sample[pb] ? acc[i] * pit[pb] : -INFINITY;
        st[pb] = stat_add4(st[pb], x[0], x[1], x[2], x[3]);
      }
      if (WM == 1) {
        const size_t at = (size_t)(pw + kTile * pb + (lane & 15)) * V + row0;
        if (rows.out && act[pb]) put_rows(rows.out, at, acc, row0, V, true);
        if (to_lf[pb]) put_rows(rows.lf, at, acc, row0, V, true);
      }
    }
    if (WM == 2) {
      // pairs count from the workgroup's first tile; an odd last tile goes alone
      if (j & 1) {
        put_pair(held, accs, (t - 1) * kTile, min(V, (t + 1) * kTile));
      } else if (j == n - 1) {
        put_pair(accs, accs, t * kTile, min(V, (t + 1) * kTile));
      } else {
#pragma unroll
        for (int pb = 0; pb < P; ++pb) held[pb] = accs[pb];
      }
    }
    flush_until(t + 1);
    flush_keys(t + 1);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);             // the clamped loads past the end
}

// lf: the rows that truncate write their logits to the workspace; out: every
// row writes them there too (either may be off).
hipError_t launch_read(xp_handle* h, int batch, uint32_t flags, const uint8_t* temp, bool lf,
                       float* out, hipStream_t st) {
  const int M = batch * h->B;
  dim3 grid(h->read_wgs, (M + kTile - 1) / kTile), block(kReadWaves * kWave);
  const int skip = (flags & XP_EARLY_EXIT) ? 1 : 0;
  const LogitRows rows{out, lf ? h->ws.lf : nullptr, h->ws.filt,
                       h->V % 4 == 0 && (uintptr_t)out % 16 == 0};
  if (h->dtype == XP_BF16 && M > kTile) {
    // 16 P positions per wave, P = 1..4 (P = 4 from 512 positions on)
    const int per = kReadWaves * kTile;
    int P = (M + per - 1) / per;
    P = P < kRmMaxP ? P : kRmMaxP;
    const int ny = (M + per * P - 1) / (per * P);
    // one workgroup per CU and position group at most: a workgroup takes gs
    // read workgroups in a row, so that the launch runs in one round
    const int gs = ny;
    const int nsg = (h->read_wgs + gs - 1) / gs;
    grid = dim3((nsg + 7) / 8 * 8 * ny);
    const int wm = out == nullptr && !lf ? 0 : (rows.vec ? 1 : 2);
    const uint16_t* Wr = (const uint16_t*)h->W_r;
    const uint16_t* Zb = (const uint16_t*)h->ws.z;
#define XP_RM(PP, EEV, WMV)                                                                  \
  hipLaunchKernelGGL((k_read_multi<PP, EEV, WMV>), grid, block, 0, st, Wr, Zb, h->ws.s, M,     \
                     h->V, M, h->ntiles, h->read_units, h->ws.keys, h->ws.stats, temp, h->B,   \
                     rows, h->ws.ctrl, skip, h->read_wgs, ny, gs, h->ws.invT, h->ws.iters)
#define XP_RM_W(PP, EEV)                                                                     \
  do {                                                                                       \
    if (wm == 0) XP_RM(PP, EEV, 0);                                                          \
    else if (wm == 1) XP_RM(PP, EEV, 1);                                                     \
    else XP_RM(PP, EEV, 2);                                                                  \
  } while (0)
#define XP_RM_P(EEV)                                                                         \
  switch (P) {                                                                               \
    case 1: XP_RM_W(1, EEV); break;                                                          \
    case 2: XP_RM_W(2, EEV); break;                                                          \
    case 3: XP_RM_W(3, EEV); break;                                                          \
    default: XP_RM_W(4, EEV);                                                                \
  }
    if (skip) {
      XP_RM_P(true)
    } else {
      XP_RM_P(false)
    }
#undef XP_RM_P
#undef XP_RM_W
#undef XP_RM
    return hipGetLastError();
  }
  if (h->dtype == XP_BF16) {
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, block, 0, st, (const uint16_t*)h->W_r,
                         (const uint16_t*)h->ws.z, h->ws.s, M, h->V, M, h->ntiles,
                         h->read_units, h->ws.keys, h->ws.stats, temp, h->B, rows, h->ws.ctrl,
                         skip, h->ws.invT);
    };
    if (out != nullptr || lf)
      go(k_read<true>);
    else
      go(k_read<false>);
    return hipGetLastError();
  }
  // fp32: a wave takes two units where each is at least half empty and one apiece
  // would make more workgroups than CUs (V = 12000, 80 positions: 32 -> 16 us)
  const int nb = (M + kTile - 1) / kTile, cus = h->cus;
  const int GS = 2 * h->ntiles <= h->read_units && h->read_wgs * nb > cus ? 2 : 1;
  const int gx = (h->read_wgs + GS - 1) / GS;
  const bool one = GS * h->ntiles <= h->read_units;
  auto ny = [&](int pb) { return (nb + pb - 1) / pb; };
  // Position blocks per workgroup.  Units of one tile: the least of the launch's
  // times, which go with a + b ceil(workgroups / CUs) (us, event-timed, V = 1000 to
  // 32768 at 16 to 512 positions: what it picks is the fastest of the three there,
  // within 5%).  Longer units (one workgroup per CU): as many as four.
  int PB = 1;
  if (one) {
    constexpr float a[3] = {6.7f, 7.5f, 8.8f}, b[3] = {4.9f, 6.8f, 8.7f};
    float least = 0.f;
    for (int pb = 1; pb <= 3; ++pb) {
      const float t = a[pb - 1] + b[pb - 1] * (float)((gx * ny(pb) + cus - 1) / cus);
      if (pb == 1 || t < least) {
        PB = pb;
        least = t;
      }
    }
  } else {
    PB = nb < 4 ? nb : 4;
  }
  PB = (nb + ny(PB) - 1) / ny(PB);                // spread evenly
  grid = dim3(gx, ny(PB));
#define XP_RF(PP, GG, OO)                                                                     \
  hipLaunchKernelGGL((k_read_f32<PP, GG, OO>), grid, block, 0, st, (const float*)h->W_r,       \
                     (const float*)h->ws.z, h->ws.s, M, h->V, M, h->ntiles, h->read_units,     \
                     h->ws.keys, h->ws.stats, temp, h->B, rows, h->ws.ctrl, skip, h->ws.invT)
#define XP_RF_ONE(GG)                                                                         \
  switch (PB) {                                                                               \
    case 1: XP_RF(1, GG, true); break;                                                        \
    case 2: XP_RF(2, GG, true); break;                                                        \
    default: XP_RF(3, GG, true);                                                              \
  }
  if (one && GS == 1) {
    XP_RF_ONE(1)
  } else if (one) {
    XP_RF_ONE(2)
  } else {
    switch (PB) {
      case 1: XP_RF(1, 1, false); break;
      case 2: XP_RF(2, 1, false); break;
      case 3: XP_RF(3, 1, false); break;
      default: XP_RF(4, 1, false);
    }
  }
#undef XP_RF_ONE
#undef XP_RF
  return hipGetLastError();
}

}  // namespace xp
