// LM-head projection in front of acceptance, with the softmax statistics fused into its
// epilogue.  The verifying stage owns an LM head (Implementation); its logits are the target
// rows acceptance reads (Sec. 4, Related Work [sd]).  For bf16 h [M][d] and W [V][d]:
//   logits[m][v] = sum_j h[m][j] W[v][j]   (fp32 accumulation, fp32 output)
// and for every row and 128-column tile, at temperature T (c = log2(e)/T):
//   stats = (max_v x*c, sum_v 2^(x*c - max))   over the tile's columns v < V.
// Acceptance combines the tiles of a row into its normaliser without reading the row again.
//
// Work decomposition: one workgroup per (vocabulary tile of 256 columns, or 128 for narrow
// outputs), all of up to 128 rows of h (more rows take the kernels below, but for
// K splits); its four waves split the
// tile in a grid of waves (below), each holding 32x32 accumulator tiles of
// v_mfma_f32_32x32x16_bf16 (A operand: h rows, B operand: W rows).
//   * W, the stream that matters (V*d*2 bytes, read once), goes straight from HBM into each
//     wave's registers, DEPTH K-steps of 64 ahead.  It is packed (pack.hip) so that each operand
//     load of a wave reads 1 KB of contiguous memory; lane half h takes K = 32h + 8s .. +7 of
//     its column at MFMA step s (the contraction order over K is free as long as h uses the
//     same).
//   * h is shared by the four waves: it goes through LDS, one step per stage, fetched into
//     registers NA steps ahead (NA register sets).  Wait counts retire in issue order: the wait
//     for h step i+1 leaves the NA steps of W loaded after it in flight, and W runs DEPTH >=
//     NA + 2 steps ahead, so the compute of step i+1 never waits for its W.  Few row tiles leave
//     registers for NA = 4, DEPTH = 8 (one column tile per wave); two column tiles per wave and
//     the larger row groups use NA = 2, DEPTH = 4.
//   * Each XCD takes blocks of its vocabulary tiles x row groups (tile_of), so its resident
//     workgroups share the K-slices of h and W they read through its L2.
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace spexis {

namespace {

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;   // NaN
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }


// Waits until at most N LDS reads (or scalar loads) of the wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_lgkm() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
// One 16-byte LDS read, written as an instruction (byte address addr + off, off a constant).
template <int kOff>
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t addr) {
  static_assert(kOff >= 0 && kOff < 65536, "the instruction's offset field");
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(kOff) : "memory");
  return v;
}
// f(0), ..., f(N - 1) with compile-time indices.
template <typename F, int... I>
__device__ __forceinline__ void for_constants_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_constants(F&& f) {
  for_constants_impl(f, std::make_integer_sequence<int, N>{});
}
// Ties a register to the wait before it: no use of v moves above that wait.
__device__ __forceinline__ void tie(u32x4& v) { asm volatile("" : "+v"(v)); }
// A 16-byte-per-lane buffer load into LDS (lane l's bytes at lds + 16 l).  Kept out of the
// kernel templates: the host side of a template kernel cannot instantiate this builtin.
__device__ __forceinline__ void buffer_load_lds16(__amdgpu_buffer_rsrc_t rs, __attribute__((address_space(3))) void* lds,
                                                  int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, lds, 16, voff, soff, 0, 0);
}

__device__ __forceinline__ u32x4 buffer_ld16(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
}
__device__ __forceinline__ u32x4 buffer_ld16_nt(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 2);
}

// W rows are read once: non-temporal loads keep them from evicting h out of L2.
template <bool kStream>
__device__ __forceinline__ u32x4 ldw(const uint16_t* p) {
  if (kStream) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return *reinterpret_cast<const u32x4*>(p);
}

// Workgroup -> (vocabulary tile nt, row group mg).  Workgroup i runs on XCD i % 8, which takes
// the vocabulary tiles nt = 8 j + XCD; the XCD's workgroups, in launch order, walk blocks of
// kTileBlock of its tiles, and within a block the row groups in blocks of kGroupBlock, each
// (tiles x groups) block in tile-major order.  The XCD's resident workgroups (one per CU) then
// cover a few row groups of a few tiles at a time, so each K-step's slice of h and of W is
// fetched into the XCD's L2 once for several workgroups.
constexpr int kTileBlock = 8, kGroupBlock = 4;
__device__ __forceinline__ void tile_of(int bid, int ntiles, int groups, int& nt, int& mg) {
  const int xcd = bid & 7, local = bid >> 3;
  const int per_xcd = (ntiles + 7) / 8;                     // tiles of an XCD (the last may be absent)
  const int tb = local / (kTileBlock * groups), rem = local % (kTileBlock * groups);
  const int ctb = min(kTileBlock, per_xcd - tb * kTileBlock);   // tiles in this block
  const int full = groups / kGroupBlock * kGroupBlock;      // groups in whole group blocks
  int t, g;
  if (rem < ctb * full) {
    const int gb = rem / (ctb * kGroupBlock), r2 = rem % (ctb * kGroupBlock);
    t = r2 / kGroupBlock;
    g = gb * kGroupBlock + r2 % kGroupBlock;
  } else {
    const int r2 = rem - ctb * full, tail = groups - full;
    t = r2 / tail;
    g = full + r2 % tail;
  }
  nt = 8 * (tb * kTileBlock + t) + xcd;
  mg = g;
}

// A workgroup's accumulators to memory: fp32 logits (or K-split partials) at `out` and / or bf16
// outputs at y (+ residual), both with row stride V, from row m0 on.  One pointer per lane and
// column tile, which each store moves on by its accumulator's step in rows (uniform: 1, or 5 past
// every fourth); a group of whole 32-row tiles takes no row checks.  fp32 values are written once and
// read by a later kernel: non-temporal stores keep them from evicting the h and W lines the other
// workgroups still read through L2 (measured at 320 x 4096 @ 128256: 469 against 480 us; at 4608 x
// 3584 @ 152064: 5332 against 5684 us).
template <bool kFull, int RT>
__device__ __forceinline__ void store_column(const f32x16 (&acc)[RT], float* at, int64_t V, int left) {
  // kept apart from the next column's checks, or the compiler holds all their masks in (spilled) registers
  if (!kFull) asm volatile("" : "+v"(left));
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (kFull || 32 * t + 8 * (i >> 2) + (i & 3) < left) __builtin_nontemporal_store(acc[t][i], at);
      at += (i & 3) == 3 ? 5 * V : V;
    }
}
template <int RT, int CT, int WR, int WC>
__device__ __forceinline__ void store_epilogue(const f32x16 (&acc)[RT][CT], float* out, uint16_t* y, const uint16_t* res,
                                               int V, int m0, int n0, int rows, int wr, int wc, int lane) {
  const int col = lane & 31, half = lane >> 5;
  const bool full = rows == 32 * WR * RT;
  const int r0 = 32 * wr * RT + 4 * half;   // row of accumulator (t, i): r0 + 32 t + 8 (i / 4) + i % 4
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int v = n0 + 32 * (CT * wc + c) + col;
    if (v >= V) continue;
    if (out) {
      f32x16 col_acc[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) col_acc[t] = acc[t][c];
      float* at = out + (int64_t)(m0 + r0) * V + v;
      if (full) store_column<true>(col_acc, at, V, 0);
      else store_column<false>(col_acc, at, V, rows - r0);
    }
    if (y) {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int r = r0 + 32 * t + 8 * (i >> 2) + (i & 3);
          if (r < rows) {
            const int64_t at = (int64_t)(m0 + r) * V + v;
            y[at] = bf16_rne(res ? acc[t][c][i] + bf16_float(res[at]) : acc[t][c][i]);
          }
        }
    }
  }
}

// Row statistics of a workgroup's accumulators over its 128-column tiles, and the gathered logits
// (the epilogue of both kernels).  Waves form a WR x WC grid of RT x CT accumulator tiles; tile
// (t, c) of lane l, value i: row 32 (wr RT + t) + 8 (i / 4) + 4 (l / 32) + i % 4, column
// n0 + 32 (CT wc + c) + l % 32.  Each wave transposes one 32 x 32 tile at a time through its part of
// `scratch` (32 x 36 floats per wave); lane l then reduces 16 columns of row l % 32 (columns
// 16 (l / 32) ..), the two halves of a row combine in one cross-half lane swap, then the wave's CT
// tiles in order, and the waves of a 128-column tile in order at the end.  (Lanes 0 .. 31 reducing
// whole rows left half the wave idle in the exponentials: 3902 against 3801 us, statistics only, at
// 4608 x 3584 @ 152064.)
// Adds of two halves commute, so both halves of the wave hold the same row statistics.
template <int RT, int CT, int WR, int WC>
__device__ __forceinline__ void row_stats_epilogue(float* stats, float* gout, float scale, int V, int ntiles,
                                                   const f32x16 (&acc)[RT][CT], const int (&gcol)[RT],
                                                   int nt, int m0, int n0, int rows, int wr, int wc, int lane,
                                                   float* scratch, float (&sm_m)[WC][32 * WR * RT],
                                                   float (&sm_z)[WC][32 * WR * RT]) {
  constexpr int kStatTiles = 32 * WC * CT / kLmCols;   // 128-column statistics tiles of the workgroup
  constexpr int kTS = 36;   // floats per transposed row (16-byte aligned, padded)
  const int col = lane & 31, half = lane >> 5;
  float* tile = scratch + (wr * WC + wc) * 32 * kTS;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    float wm = -INFINITY, wz = 0.f;
    const int grow = 32 * (wr * RT + t) + col;   // this lane's row
    const int gc = gcol[t];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      // x c rounded once, then x c - max: no contraction into one fused operation
#pragma clang fp contract(off)
      const int cb = n0 + 32 * (CT * wc + c);   // the tile's first column
      const bool live = cb + col < V;
      wave_lds_fence();   // after the last tile's reads
#pragma unroll
      for (int i = 0; i < 16; ++i)
        tile[(8 * (i >> 2) + 4 * half + (i & 3)) * kTS + col] = live ? acc[t][c][i] : -INFINITY;
      wave_lds_fence();
      const float* mine = tile + col * kTS + 16 * half;   // 16 columns of this lane's row
      f32x4 x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const f32x4*>(mine + 4 * q) * scale;
      const int gl = gc - cb - 16 * half;
      if (gl >= 0 && gl < 16 && gc < V) gout[m0 + grow] = mine[gl];
      float mx = -INFINITY;
#pragma unroll
      for (int q = 0; q < 4; ++q) mx = fmaxf(fmaxf(mx, fmaxf(x[q][0], x[q][1])), fmaxf(x[q][2], x[q][3]));
      const auto rm = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(rm[0]), __uint_as_float(rm[1]));
      float e = 0.f;
      if (mx != -INFINITY) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 4; ++u) e += fast_exp2(x[q][u] - mx);
      }
      const auto re = __builtin_amdgcn_permlane32_swap(__float_as_uint(e), __float_as_uint(e), false, false);
      e = __uint_as_float(re[0]) + __uint_as_float(re[1]);
      if (c == 0) {
        wm = mx;
        wz = e;
      } else {
        const float M = fmaxf(wm, mx);
        wz = (wm != -INFINITY ? wz * fast_exp2(wm - M) : 0.f) + (mx != -INFINITY ? e * fast_exp2(mx - M) : 0.f);
        wm = M;
      }
    }
    if (half == 0) {
      sm_m[wc][grow] = wm;
      sm_z[wc][grow] = wz;
    }
  }
  __syncthreads();
  constexpr int kWavesPerStat = WC / kStatTiles;   // waves of a row within one statistics tile
  for (int q = threadIdx.x; q < rows * kStatTiles; q += 64 * WR * WC) {
    const int r = q % rows, st = q / rows, w0 = st * kWavesPerStat;
    const int stile = nt * kStatTiles + st;
    if (stile >= ntiles) continue;
    float M = sm_m[w0][r];
#pragma unroll
    for (int w = 1; w < kWavesPerStat; ++w) M = fmaxf(M, sm_m[w0 + w][r]);
    float Z = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerStat; ++w)
      if (sm_m[w0 + w][r] != -INFINITY) Z += sm_z[w0 + w][r] * fast_exp2(sm_m[w0 + w][r] - M);
    *reinterpret_cast<f32x2*>(stats + ((int64_t)(m0 + r) * ntiles + stile) * 2) = f32x2{M, Z};
  }
}

}  // namespace

// Waves form a WR x WC grid over the workgroup's (32 * WR * RT) rows x (32 * WC * CT) columns:
// wave (wr, wc) computes RT row tiles x CT column tiles.  The launched shapes put the four waves
// side by side (WR = 1) with two column tiles each (256 columns per workgroup): against one tile
// each, that halves the h fragments each wave reads from LDS per MFMA and the h rows staged per
// column.  (A 2 x 2 grid over 128 columns does the former but loads each W tile twice.)
// Statistics stay per 128-column tile: a 256-column workgroup writes two.
template <bool kStream, int RT, int CT, int WR, int NA, int DEPTH, int WPE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WPE)))
void lm_head_kernel(LmParams p) {
  static_assert(DEPTH >= NA + 2 && DEPTH % NA == 0 && DEPTH % 2 == 0, "pipeline shape");
  constexpr int WC = 4 / WR;
  constexpr int kCols = 32 * WC * CT;           // columns of the workgroup
  static_assert(WR * WC == 4 && (kCols == 128 || kCols == 256), "wave grid");
  constexpr int NRT = WR * RT;   // row tiles of the workgroup
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int wr = wave / WC, wc = wave % WC;
  const int wgcols = (p.V + kCols - 1) / kCols;
  int nt, mg;
  tile_of(blockIdx.x, wgcols, p.mgroups, nt, mg);
  if (nt >= wgcols) return;
  const int m0 = mg * 32 * NRT, n0 = nt * kCols;
  const int rows = min(32 * NRT, p.M - m0);
  // K split: workgroup row ks takes K values ks * klen .. +klen-1 (nsteps steps of 64)
  const int ks = blockIdx.y;
  const int klen = p.d / p.ksplit, nsteps = klen / kLmK;
  // column tile c of this wave is packed tile row n0 / 32 + CT wc + c (clamped for the columns
  // past V, whose results are dropped); lane l reads 16 contiguous bytes at s * 512 + 8 l of each
  // tile
  const uint16_t* wrow[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int wtile = min(n0 / 32 + CT * wc + c, (p.V + 31) / 32 - 1);
    wrow[c] = reinterpret_cast<const uint16_t*>(p.w) +
              ((int64_t)wtile * (p.d / kLmK) + (int64_t)ks * nsteps) * kPackTile + 8 * lane;
  }
  const uint16_t* hbase = reinterpret_cast<const uint16_t*>(p.h) + (int64_t)m0 * p.d + (int64_t)ks * klen;

  // h in LDS: stage x, row r, 16-byte chunk kc of the step stored at position kc ^ ((r >> 1) & 7),
  // so that the 16 rows one ds_read_b128 pass serves hit 16 distinct 16-byte bank groups.  Only
  // the workgroup's NRT row tiles are staged: 32 * NRT rows * 8 chunks = NRT chunks per thread.
  // (At least 72 rows: the epilogue transposes 4 x 32 x 36 floats through this space.)
  constexpr int kAChunks = NRT;
  constexpr int kStage = (32 * NRT > 72 ? 32 * NRT : 72) * 8;
  __shared__ u32x4 sm_a[2][kStage];
  u32x4 areg[NA][kAChunks];   // h chunks of the next NA steps, in flight
  auto load_a = [&](u32x4 (&dst)[kAChunks], int j) {
    j = min(j, nsteps - 1);   // past the end: re-read the last step (kept unconditional)
#pragma unroll
    for (int u = 0; u < kAChunks; ++u) {
      const int q = threadIdx.x + 256 * u;
      const int r = min(q >> 3, rows - 1), kc = q & 7;
      dst[u] = *reinterpret_cast<const u32x4*>(hbase + (int64_t)r * p.d + j * kLmK + 8 * kc);
    }
  };
  auto store_a = [&](const u32x4 (&src)[kAChunks], int stage) {
#pragma unroll
    for (int u = 0; u < kAChunks; ++u) {
      const int q = threadIdx.x + 256 * u;
      const int r = q >> 3, kc = q & 7;
      sm_a[stage][r * 8 + (kc ^ ((r >> 1) & 7))] = src[u];
    }
  };
  u32x4 wb[DEPTH][CT][4];
  auto load_w = [&](u32x4 (&dst)[CT][4], int j) {
    const int64_t off = (int64_t)min(j, nsteps - 1) * kPackTile;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) dst[c][s] = ldw<kStream>(wrow[c] + off + 512 * s);
  };

  f32x16 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][c][e] = 0.f;

  // prologue: h step 0 into stage 0, W steps 0 .. DEPTH-1, h steps 1 .. NA into registers
  load_a(areg[0], 0);
#pragma unroll
  for (int b = 0; b < DEPTH; ++b) load_w(wb[b], b);
  store_a(areg[0], 0);
#pragma unroll
  for (int a = 1; a <= NA; ++a) load_a(areg[a % NA], a);
  __syncthreads();

  // The A fragments of k-step s+1 are read from LDS while the MFMAs of k-step s run.
  auto frag = [&](int stage, int t, int s) {
    const int m = 32 * (wr * RT + t) + col;
    return sm_a[stage][m * 8 + ((4 * half + s) ^ ((m >> 1) & 7))];
  };
  auto compute = [&](const u32x4 (&w)[CT][4], int stage) {
    u32x4 fa[2][RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) fa[0][t] = frag(stage, t, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (s + 1 < 4) {
#pragma unroll
        for (int t = 0; t < RT; ++t) fa[(s + 1) & 1][t] = frag(stage, t, s + 1);
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const bf16x8 bop = as_bf16x8(w[c][s]);
#pragma unroll
        for (int t = 0; t < RT; ++t)
          acc[t][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fa[s & 1][t]), bop, acc[t][c], 0, 0, 0);
      }
    }
  };

  // step i: compute from stage i%2 and W buffer i%DEPTH; move h step i+1 (fetched NA steps ago)
  // into the other stage and fetch h step i+1+NA into the same registers; refill the W buffer
  // with step i+DEPTH
  for (int j = 0; j < nsteps; j += DEPTH) {
#pragma unroll
    for (int jj = 0; jj < DEPTH; ++jj) {
      if (j + jj < nsteps) compute(wb[jj], jj & 1);
      store_a(areg[(jj + 1) % NA], (jj + 1) & 1);
      load_a(areg[(jj + 1) % NA], j + jj + 1 + NA);
      load_w(wb[jj], j + jj + DEPTH);
      __syncthreads();
    }
  }

  // ---- epilogue: logits (or partials, or bf16 outputs), and each row's statistics over each of
  // this workgroup's 128-column statistics tiles.  The gather columns of the rows each lane reduces
  // in the statistics are loaded first: their latency passes under the stores.
  int gcol[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int grow = 32 * (wr * RT + t) + col;
    gcol[t] = p.gout && p.stats && grow < rows ? p.gcols[m0 + grow] : -1;
  }
  store_epilogue<RT, CT, WR, WC>(acc, p.logits ? p.logits + (int64_t)ks * p.M * p.V : nullptr,
                                 reinterpret_cast<uint16_t*>(p.y), reinterpret_cast<const uint16_t*>(p.res), p.V, m0, n0,
                                 rows, wr, wc, lane);
  if (!p.stats) return;
  // through the (now free) h stages
  __shared__ float sm_m[WC][32 * NRT], sm_z[WC][32 * NRT];
  row_stats_epilogue<RT, CT, WR, WC>(p.stats, p.gout, p.c, p.V, p.ntiles, acc, gcol, nt, m0, n0, rows, wr, wc, lane,
                                     reinterpret_cast<float*>(&sm_a[0][0]), sm_m, sm_z);
}

// More than 160 rows of a wide projection (an LM head's vocabulary): one workgroup of eight waves
// (two per SIMD) per (256-column tile, group of 64 RT rows; figures here are of 320), so that each
// K-slice of W crosses L2 once per group.  Both operands go through LDS: every K-step of 64 the
// workgroup copies h (320 rows, 40 KB) and W (eight packed 32-column tiles, 32 KB) from memory
// straight into one of two stages, a step ahead, and the waves read their fragments from the
// stage, those of the next MFMA step while the current step's MFMAs run.  Wave (wr, wc) of a
// 2 x 4 grid computes rows 160 wr .. +160 (five row tiles)
// by columns 64 wc .. +64 (two column tiles): 160 accumulators, within the 256 registers a wave
// has at two waves per SIMD.  Against four waves per 160-row x 256-column workgroup (two row
// groups, each reading W), the L2 serves about 2.35 GB instead of 3.4 GB at 320 x 4096 @ 128256.
// Epilogue as lm_head_kernel's: logits or bf16 outputs, then each row's statistics per
// 128-column tile.
template <int RT, int CT, int WR, int WC>
__global__ __launch_bounds__(64 * WR * WC) __attribute__((amdgpu_waves_per_eu(WR * WC / 4)))
void lm_head_wide_kernel(LmParams p) {
  constexpr int NRT = WR * RT;        // row tiles of the workgroup
  constexpr int kRows = 32 * NRT;     // rows of the group
  constexpr int kCols = 32 * WC * CT; // columns of the workgroup
  static_assert(kCols == 256 && WC % 2 == 0, "two 128-column statistics tiles, whole waves each");
  // the wave index wave-uniform (scalar), so the copies' LDS destinations are scalar sums
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int wr = wave / WC, wc = wave % WC;
  const int wgcols = (p.V + kCols - 1) / kCols;
  int nt, mg;
  tile_of(blockIdx.x, wgcols, p.mgroups, nt, mg);
  if (nt >= wgcols) return;
  const int n0 = nt * kCols, m0 = mg * kRows;
  const int rows = min(kRows, p.M - m0);
  const int nsteps = p.d / kLmK;
  const int wtiles = (p.V + 31) / 32;
  const uint16_t* hbase = reinterpret_cast<const uint16_t*>(p.h) + (int64_t)m0 * p.d;
  const uint16_t* wbase = reinterpret_cast<const uint16_t*>(p.w);

  // stage x of h: row r, chunk kc (8 K values) at r * 8 + (kc ^ ((r >> 1) & 7)) (the 16 rows of
  // one ds_read_b128 pass hit distinct bank groups); stage x of W: packed tile c (columns
  // n0 + 32 c ..), its 256 chunks in packed order.  One array: h stages 0 and 1, then W stages
  // 0 and 1.
  constexpr int kHStage = kRows * 8, kWStage = kCols / 32 * 256;
  __shared__ u32x4 sm[2 * kHStage + 2 * kWStage];
  static_assert(2 * kHStage >= WR * WC * 32 * 36 / 4, "the epilogue transposes a tile per wave through the h stages");
  // Copies go from memory straight into a stage (buffer loads to LDS, 1 KB per wave and
  // instruction, lane l's 16 bytes at slot 64 u + l): no staging registers, which leaves room
  // for two sets of operand fragments.  Buffer resources span the group's rows of h and the
  // workgroup's packed W tiles: loads past them (rows past M, columns past V) return zeros,
  // whose results are dropped.
  constexpr int kWaves = WR * WC;
  constexpr int kHCopies = kHStage / 64 / kWaves;   // copy instructions per wave and step
  constexpr int kWCopies = kWStage / 64 / kWaves;
  static_assert(kHStage % (64 * kWaves) == 0 && kWStage % (64 * kWaves) == 0, "copy split");
  const int wt0 = n0 / 32, wtn = min(kCols / 32, wtiles - wt0);
  const __amdgpu_buffer_rsrc_t hrs =
      __builtin_amdgcn_make_buffer_rsrc((void*)hbase, (short)0, rows * p.d * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(wbase + (int64_t)wt0 * (p.d / kLmK) * kPackTile), (short)0, wtn * (p.d / kLmK) * kPackTile * 2,
      0x00020000);
  int hoff[kHCopies], woff[kWCopies];   // byte offsets of the lane's chunks at step 0
#pragma unroll
  for (int u = 0; u < kHCopies; ++u) {
    const int q = (wave * kHCopies + u) * 64 + lane;
    const int r = q >> 3, kc = (q & 7) ^ ((r >> 1) & 7);
    hoff[u] = (r * p.d + 8 * kc) * 2;
  }
#pragma unroll
  for (int u = 0; u < kWCopies; ++u) {
    const int q = (wave * kWCopies + u) * 64 + lane;
    woff[u] = ((q >> 8) * (p.d / kLmK) * kPackTile + 8 * (q & 255)) * 2;
  }
  // copy instruction u of step j (the wave's h copies first, then its W copies)
  auto copy_one = [&](int j, int stage, int u) {
    if (u < kHCopies)
      buffer_load_lds16(hrs, (__attribute__((address_space(3))) void*)(sm + stage * kHStage + (wave * kHCopies + u) * 64),
                        hoff[u], j * kLmK * 2);
    else
      buffer_load_lds16(wrs,
                        (__attribute__((address_space(3))) void*)(sm + 2 * kHStage + stage * kWStage +
                                                                  (wave * kWCopies + u - kHCopies) * 64),
                        woff[u - kHCopies], j * kPackTile * 2);
  };
  constexpr int kCopies = kHCopies + kWCopies;
  auto copy_step = [&](int j, int stage) {
#pragma unroll
    for (int u = 0; u < kCopies; ++u) copy_one(j, stage, u);
  };

  f32x16 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][c][e] = 0.f;

  // Fragment reads are written as instructions: the compiler would make every LDS read wait for
  // all copies to LDS in flight (into either stage), which cancels the copies' prefetch.  The
  // reads of MFMA step s + 1 go out before step s's MFMAs, and each step waits for its own
  // fragments by count (LDS reads return in order).  Byte addresses: A fragment of row tile t at
  // step s, h stage + (32 (wr RT + t) + col) * 128 + ((4 half + s) ^ ((col >> 1) & 7)) * 16 (row
  // m's swizzle (m >> 1) & 7 is col's, 32 (wr RT + t) being a multiple of 16); B fragment of
  // column tile c, W stage + ((CT wc + c) * 256 + 64 s + lane) * 16.
  static_assert(RT + CT <= 15, "one lgkmcnt covers a step's fragment reads");
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4*)sm;   // LDS byte address
  uint32_t aaddr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    aaddr[s] = lds0 + (32 * wr * RT + col) * 128 + (((4 * half + s) ^ ((col >> 1) & 7)) << 4);
  const uint32_t baddr = lds0 + 2 * kHStage * 16 + (CT * wc * 256 + lane) * 16;
  u32x4 fa[2][RT], fb[2][CT];   // fragments of the current MFMA step and of the next one
  auto frags = [&](auto stage, auto step) {   // of MFMA step `step` of a stage, into set step % 2
    constexpr int st = decltype(stage)::value, sp = decltype(step)::value;
    for_constants<RT>([&](auto t) { fa[sp & 1][t] = lds_read_b128<st * kHStage * 16 + t * 4096>(aaddr[sp]); });
    for_constants<CT>([&](auto c) { fb[sp & 1][c] = lds_read_b128<st * kWStage * 16 + c * 4096 + sp * 1024>(baddr); });
  };
  // tie the fragments to the wait, so that no use of them moves above it
  auto tie_frags = [&](int x) {
#pragma unroll
    for (int t = 0; t < RT; ++t) tie(fa[x][t]);
#pragma unroll
    for (int c = 0; c < CT; ++c) tie(fb[x][c]);
  };
  auto mfma_one = [&](int x, int t, int c) {
    acc[t][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fa[x][t]), as_bf16x8(fb[x][c]), acc[t][c], 0, 0, 0);
  };

  // Step j: four MFMA steps from stage j % 2, the fragments of the next one read before the current
  // one's MFMAs.  Before the last one's MFMAs every wave has read all of the stage and waits for its
  // own copies of step j + 1 (issued a whole step ago); the barrier then makes that step visible and
  // frees the stage, so step j + 1's first fragments and, between the MFMAs, the copies of step
  // j + 2 go out while the last ten MFMAs run.  (With the barrier between two whole steps, both
  // waves of a SIMD read a step's first fragments with the matrix cores idle: 4612 against 4252 us
  // at 4608 x 3584 @ 152064, 344 against 322 us at 320 x 4096 @ 128256.)  Scheduling barriers keep
  // each group of MFMAs between its own wait and the next one; without them the compiler sank the
  // third group below the fourth's wait (4509 us).
  auto k_step = [&](auto stage, auto more, auto copy, int j) {
    constexpr int st = decltype(stage)::value;
    for_constants<3>([&](auto s) {
      frags(stage, std::integral_constant<int, s + 1>{});
      wait_lgkm<RT + CT>();   // this step's reads done; the next step's stay in flight
      tie_frags(s & 1);
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) mfma_one(s & 1, t, c);
      __builtin_amdgcn_sched_barrier(0);
    });
    wait_lgkm<0>();
    tie_frags(1);
    if constexpr (decltype(more)::value) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      frags(std::integral_constant<int, st ^ 1>{}, std::integral_constant<int, 0>{});
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < RT * CT || u < kCopies; ++u) {
      if (u < RT * CT) mfma_one(1, u / CT, u % CT);
      __builtin_amdgcn_sched_barrier(0);
      if (decltype(copy)::value && u < kCopies) copy_one(j + 2, st, u);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using Stage0 = std::integral_constant<int, 0>;
  using Stage1 = std::integral_constant<int, 1>;
  copy_step(0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  copy_step(1, 1);
  frags(Stage0{}, Stage0{});
  int j = 0;   // an even number of steps, at least four (d is a multiple of 256)
  for (; j + 2 < nsteps; j += 2) {
    k_step(Stage0{}, std::true_type{}, std::true_type{}, j);
    k_step(Stage1{}, std::true_type{}, std::true_type{}, j + 1);
  }
  k_step(Stage0{}, std::true_type{}, std::false_type{}, j);
  k_step(Stage1{}, std::false_type{}, std::false_type{}, j + 1);
  __syncthreads();   // the epilogue's transposes reuse the h stages

  // ---- epilogue (the gather columns first, as above)
  int gcol[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int grow = 32 * (wr * RT + t) + col;
    gcol[t] = p.gout && p.stats && grow < rows ? p.gcols[m0 + grow] : -1;
  }
  store_epilogue<RT, CT, WR, WC>(acc, p.logits, reinterpret_cast<uint16_t*>(p.y),
                                 reinterpret_cast<const uint16_t*>(p.res), p.V, m0, n0, rows, wr, wc, lane);
  if (!p.stats) return;
  __shared__ float sm_m[WC][kRows], sm_z[WC][kRows];   // the transposes: the (now free) h stages
  row_stats_epilogue<RT, CT, WR, WC>(p.stats, p.gout, p.c, p.V, p.ntiles, acc, gcol, nt, m0, n0, rows, wr, wc, lane, reinterpret_cast<float*>(&sm[0]),
                                     sm_m, sm_z);
}

// Many rows, in groups of 32 RT: half the waves and rows of lm_head_wide_kernel's workgroup and two
// workgroups per CU, so that one's epilogue (statistics, 320 of 4250 us at 4608 x 3584 @ 152064) and
// barriers pass under the other's MFMAs, and a row count is padded to groups half as tall.  h goes
// through LDS as there; the four waves lie side by side, so no two share a column of W, and W goes
// straight into registers.  Its bound is power: the matrix cores are busy 96% of the cycles of the K
// loop, at 1.46 GHz (lm_head_wide_kernel: 86% at 1.64 GHz, the same 1.4 PFLOP/s), so what is left to
// gain is what does not multiply.  A single group streams W past the caches (kStream: 202 against 221 us
// at 160 x 4096 @ 128256).
template <int RT, bool kStream>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void lm_head_pair_kernel(LmParams p) {
  constexpr int CT = 2, WC = 4;       // column tiles of a wave, waves
  constexpr int kRows = 32 * RT;      // rows of the group
  constexpr int kCols = 32 * WC * CT; // columns of the workgroup
  // the wave index wave-uniform (scalar), so the copies' LDS destinations are scalar sums
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int wgcols = (p.V + kCols - 1) / kCols;
  int nt, mg;
  tile_of(blockIdx.x, wgcols, p.mgroups, nt, mg);
  if (nt >= wgcols) return;
  const int n0 = nt * kCols, m0 = mg * kRows;
  const int rows = min(kRows, p.M - m0);
  const int nsteps = p.d / kLmK;
  const int wtiles = (p.V + 31) / 32;
  const uint16_t* hbase = reinterpret_cast<const uint16_t*>(p.h) + (int64_t)m0 * p.d;
  const uint16_t* wbase = reinterpret_cast<const uint16_t*>(p.w);

  // stage x of h: row r, chunk kc (8 K values) at r * 8 + (kc ^ ((r >> 1) & 7)), as above; copied from
  // memory straight into the stage (1 KB per wave and instruction).  Buffer resources span the group's
  // rows of h and the workgroup's packed W tiles: loads past them return zeros, whose results are dropped.
  constexpr int kHStage = kRows * 8;
  static_assert(2 * kHStage >= WC * 32 * 36 / 4, "the epilogue transposes a tile per wave through the stages");
  __shared__ u32x4 sm[2 * kHStage];
  constexpr int kCopies = kHStage / 64 / WC;   // copy instructions per wave and step
  static_assert(kHStage % (64 * WC) == 0, "copy split");
  const int wt0 = n0 / 32, wtn = min(kCols / 32, wtiles - wt0);   // the workgroup's packed tiles (a resource per wave spills registers)
  const __amdgpu_buffer_rsrc_t hrs =
      __builtin_amdgcn_make_buffer_rsrc((void*)hbase, (short)0, rows * p.d * 2, 0x00020000);
  const int wtile = nsteps * kPackTile;   // elements of a packed tile
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(wbase + (int64_t)wt0 * wtile), (short)0, wtn * wtile * 2, 0x00020000);
  int hoff[kCopies], woff[CT];   // byte offsets of the lane's chunks at step 0
#pragma unroll
  for (int u = 0; u < kCopies; ++u) {
    const int q = (wave * kCopies + u) * 64 + lane;
    const int r = q >> 3, kc = (q & 7) ^ ((r >> 1) & 7);
    hoff[u] = (r * p.d + 8 * kc) * 2;
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) woff[c] = (CT * wave + c) * wtile * 2 + lane * 16;
  // copy instruction u of step j
  auto copy_one = [&](int j, int stage, int u) {
    buffer_load_lds16(hrs, (__attribute__((address_space(3))) void*)(sm + stage * kHStage + (wave * kCopies + u) * 64),
                      hoff[u], j * kLmK * 2);
  };
  auto copy_step = [&](int j, int stage) {
#pragma unroll
    for (int u = 0; u < kCopies; ++u) copy_one(j, stage, u);
  };

  f32x16 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][c][e] = 0.f;

  // h fragments by instructions, as in lm_head_wide_kernel; W's by buffer loads, those of step j + 1 into
  // the registers whose MFMAs of step j have just been issued: in flight for three quarters of a step.
  static_assert(RT <= 15, "one lgkmcnt covers a step's fragment reads");
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4*)sm;   // LDS byte address
  uint32_t aaddr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    aaddr[s] = lds0 + col * 128 + (((4 * half + s) ^ ((col >> 1) & 7)) << 4);
  u32x4 fa[2][RT], fb[4][CT];
  auto load_w = [&](int j, int s) {
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int off = woff[c] + s * 1024;
      fb[s][c] = kStream ? buffer_ld16_nt(wrs, off, j * kPackTile * 2) : buffer_ld16(wrs, off, j * kPackTile * 2);
    }
  };
  auto frags = [&](auto stage, auto step) {   // of MFMA step `step` of a stage, into set step % 2
    constexpr int st = decltype(stage)::value, sp = decltype(step)::value;
    for_constants<RT>([&](auto t) { fa[sp & 1][t] = lds_read_b128<st * kHStage * 16 + t * 4096>(aaddr[sp]); });
  };
  // tie the fragments to the wait, so that no use of them moves above it
  auto tie_frags = [&](int x) {
#pragma unroll
    for (int t = 0; t < RT; ++t) tie(fa[x][t]);
  };
  auto mfma_one = [&](int x, int s, int t, int c) {
    acc[t][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fa[x][t]), as_bf16x8(fb[s][c]), acc[t][c], 0, 0, 0);
  };

  // Step j, its barrier and the copies as in lm_head_wide_kernel.  The copies of step j + 1 were issued
  // in step j - 1 before that step's last loads of W and this step's first three: those may stay in flight.
  auto k_step = [&](auto stage, auto more, auto copy, int j) {
    constexpr int st = decltype(stage)::value;
    for_constants<3>([&](auto s) {
      frags(stage, std::integral_constant<int, s + 1>{});
      wait_lgkm<RT>();   // this step's reads done; the next step's stay in flight
      tie_frags(s & 1);
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) mfma_one(s & 1, s, t, c);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(more)::value) load_w(j + 1, s);
      __builtin_amdgcn_sched_barrier(0);
    });
    wait_lgkm<0>();
    tie_frags(1);
    if constexpr (decltype(more)::value) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * CT) : "memory");
      __builtin_amdgcn_s_barrier();
      frags(std::integral_constant<int, st ^ 1>{}, std::integral_constant<int, 0>{});
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < RT * CT || u < kCopies; ++u) {
      if (u < RT * CT) mfma_one(1, 3, u / CT, u % CT);
      __builtin_amdgcn_sched_barrier(0);
      if (decltype(copy)::value && u < kCopies) copy_one(j + 2, st, u);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (decltype(more)::value) load_w(j + 1, 3);
    __builtin_amdgcn_sched_barrier(0);
  };
  using Stage0 = std::integral_constant<int, 0>;
  using Stage1 = std::integral_constant<int, 1>;
  copy_step(0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  copy_step(1, 1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < 4; ++s) load_w(0, s);
  __builtin_amdgcn_sched_barrier(0);
  frags(Stage0{}, Stage0{});
  int j = 0;   // an even number of steps, at least four (d is a multiple of 256)
  for (; j + 2 < nsteps; j += 2) {
    k_step(Stage0{}, std::true_type{}, std::true_type{}, j);
    k_step(Stage1{}, std::true_type{}, std::true_type{}, j + 1);
  }
  k_step(Stage0{}, std::true_type{}, std::false_type{}, j);
  k_step(Stage1{}, std::false_type{}, std::false_type{}, j + 1);
  __syncthreads();   // the epilogue's transposes reuse the h stages

  // ---- epilogue (the gather columns first, as above)
  int gcol[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) gcol[t] = p.gout && p.stats && 32 * t + col < rows ? p.gcols[m0 + 32 * t + col] : -1;
  store_epilogue<RT, CT, 1, WC>(acc, p.logits, reinterpret_cast<uint16_t*>(p.y),
                                reinterpret_cast<const uint16_t*>(p.res), p.V, m0, n0, rows, 0, wave, lane);
  if (!p.stats) return;
  __shared__ float sm_m[WC][kRows], sm_z[WC][kRows];   // the transposes: the (now free) h stages
  row_stats_epilogue<RT, CT, 1, WC>(p.stats, p.gout, p.c, p.V, p.ntiles, acc, gcol, nt, m0, n0, rows, 0, wave, lane,
                                    reinterpret_cast<float*>(&sm[0]), sm_m, sm_z);
}

template <int RT, int CT, int WR, int NA, int DEPTH, int WPE>
static hipError_t launch_lm_nrt(const LmParams& q, hipStream_t s) {
  // grid: tiles of 8 vocabulary tiles (one per XCD) x row groups of 32 WR RT rows, row groups
  // innermost; y: K split
  LmParams p = q;
  p.mgroups = (p.M + 32 * WR * RT - 1) / (32 * WR * RT);
  const int wgcols = (p.V + 32 * (4 / WR) * CT - 1) / (32 * (4 / WR) * CT);
  const int64_t grid = (int64_t)((wgcols + 7) / 8) * 8 * p.mgroups;
  const dim3 g((unsigned)grid, (unsigned)p.ksplit);
  if (p.mgroups == 1)
    hipLaunchKernelGGL((lm_head_kernel<true, RT, CT, WR, NA, DEPTH, WPE>), g, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((lm_head_kernel<false, RT, CT, WR, NA, DEPTH, WPE>), g, dim3(256), 0, s, p);
  return hipGetLastError();
}

// Up to 128 rows, 256-column workgroups when the columns alone give at least one workgroup per
// CU (an LM head's vocabulary); narrower outputs (hidden-size projections) keep 128 columns, whose
// twice as many workgroups the K split then fills the chip with.
static bool wide_columns(int64_t M, int64_t N) { return M > 128 || (N + 255) / 256 >= 256; }

// Workgroups of a launch, with the absent ones that round the column tiles up to the 8 XCDs.
int64_t launched_workgroups(int64_t N, int64_t groups) { return ((N + 255) / 256 + 7) / 8 * 8 * groups; }

// More than 128 rows: the kernel and the rows of its groups.  129 to 160 rows are one group of
// lm_head_pair_kernel, 161 to 320 one of lm_head_wide_kernel with the smallest of three heights that holds
// them (at 4096 @ 128256, against groups of 160 of lm_head_kernel, resp. one of 320: 199 against 228 us at
// 160 rows, 246 against 285 at 192, 280 against 305 at 256).  More rows take the least total of one
// group's measured time times the groups: 100 for 320 rows of the wide kernel, 51 and 42 for 160 and 128
// of the pair kernel (against lm_head_kernel or groups of 320: 395 against 464 us at 384 rows, 462 against
// 574 at 480, 507 against 561 at 512, 1018 against 1143 at 1024 x 3584 @ 152064, 4240 against 4303 at 4608
// rows there; 640 rows keep 320: 596, with 160 610).  Those are vocabularies whose columns alone fill the
// chip many times over; with few columns the rounds of workgroups over the CUs count (here and in
// one_round_of_rows).
struct RowGroups {
  bool wide;
  int rows;
};
static RowGroups row_groups(int64_t M, int64_t N) {
  if (M <= 160) return {false, 160};
  if (M <= 320) return {true, M <= 192 ? 192 : M <= 256 ? 256 : 320};
  const int64_t w320 = (M + 319) / 320 * 100, p160 = (M + 159) / 160 * 51, p128 = (M + 127) / 128 * 42;
  const int64_t pair = p160 <= p128 ? 160 : 128;
  if (w320 <= p160 && w320 <= p128) return {true, 320};
  // one round of the wide kernel (a workgroup a CU) against two of the pair kernel (two a CU): 120 against
  // 134 us at 832 x 3584 @ 20000
  if (launched_workgroups(N, (M + 319) / 320) <= 256 && launched_workgroups(N, (M + pair - 1) / pair) > 512)
    return {true, 320};
  return {false, (int)pair};
}

// The kernels of more than 128 rows address a workgroup's rows of h (up to 320) and its packed tiles of W
// (256 rows) by 32-bit byte offsets; a longer contraction keeps lm_head_kernel and its 64-bit addresses.
constexpr int kMaxOffsetDim = 1 << 21;
static_assert((int64_t)kMaxOffsetDim * 320 * 2 < (1ll << 31), "the rows of a group of 320");

// Row groups of lm_head_kernel, which keeps K splits (and their odd step counts): 192 rows (six tiles) when
// that pads M to at most 5% more rows than groups of 160 (five tiles), else 160.
int64_t group_rows(int64_t M) {
  const int64_t p160 = (M + 159) / 160 * 160, p192 = (M + 191) / 192 * 192;
  return p192 * 20 <= p160 * 21 ? 192 : 160;
}

// Few columns, where lm_head_kernel's groups are one workgroup for each CU and the pair kernel's are not two:
// some CUs then run two of its workgroups and the others wait (100 against 113 us at 352 x 3584 @ 32000, 95
// against 102 at 768 @ 16000; with two for each CU the pair kernel wins: 118 against 143 us at 480 @ 32000).
// Not with bf16 outputs, whose many small stores pass under the other workgroup's products: 106 against 83 us
// at 896 x 2048 @ 10240, 68 against 54 at 512 x 256 @ 18944.
static bool one_round_of_rows(int64_t M, int64_t N) {
  const RowGroups g = row_groups(M, N);
  if (g.wide || M <= 160 || launched_workgroups(N, (M + g.rows - 1) / g.rows) <= 256) return false;
  return launched_workgroups(N, (M + group_rows(M) - 1) / group_rows(M)) <= 256;
}

// The groups that a K split is sized by (one of 320 rows where those pad M little).
static bool wide_rows(int64_t M) {
  const int64_t g = group_rows(M);
  return M <= 320 || (M + 319) / 320 * 320 * 100 <= (M + g - 1) / g * g * 112;
}

int64_t projection_workgroups(int64_t M, int64_t N) {
  // one row group up to 128 rows
  const int64_t cols = wide_columns(M, N) ? (N + 255) / 256 : (N + kLmCols - 1) / kLmCols;
  if (M <= 128) return cols;
  if (M > 160 && wide_rows(M)) return cols * ((M + 319) / 320);
  return cols * ((M + group_rows(M) - 1) / group_rows(M));
}

hipError_t launch_projection(const LmParams& p, hipStream_t s) {
  // row tiles computed per workgroup: the smallest instantiated count covering the rows (a
  // group of fewer rows repeats its last row in the padding tiles, whose results are dropped).
  // Wide shapes are 256 columns: four waves across, each two column tiles of 32 (wide_columns).
  // Up to 64 rows, a hint of two waves per SIMD; more rows take more accumulators and one.
  // Every load -- h from L2, W from HBM -- is an L1 miss, and each CU's capacity for pending misses
  // bounds the streams, so wider tiles' fewer requests per MFMA pay: at 4096 @ 128256, 180 against 188 us for 128-column
  // workgroups at 32 rows, 190 against 205 at 64, 215 against 265 at 128.  Narrow outputs: 128
  // columns, one column tile per wave.
  const int need = (p.M + 31) / 32;
  if (!wide_columns(p.M, p.V)) {
    if (need <= 1) return launch_lm_nrt<1, 1, 1, 4, 8, 2>(p, s);
    if (need <= 2) return launch_lm_nrt<2, 1, 1, 4, 8, 2>(p, s);
    return launch_lm_nrt<4, 1, 1, 4, 8, 1>(p, s);
  }
  if (need <= 1) return launch_lm_nrt<1, 2, 1, 2, 4, 2>(p, s);
  if (need <= 2) return launch_lm_nrt<2, 2, 1, 2, 4, 2>(p, s);
  if (need <= 4) return launch_lm_nrt<4, 2, 1, 2, 4, 1>(p, s);
  if (p.ksplit > 1 || p.d > kMaxOffsetDim || (!p.y && one_round_of_rows(p.M, p.V)))
    return group_rows(p.M) == 192 ? launch_lm_nrt<6, 2, 1, 2, 4, 1>(p, s) : launch_lm_nrt<5, 2, 1, 2, 4, 1>(p, s);
  const RowGroups g = row_groups(p.M, p.V);
  LmParams q = p;
  q.mgroups = (p.M + g.rows - 1) / g.rows;
  const dim3 grid((unsigned)((p.V + 255) / 256 + 7) / 8 * 8 * q.mgroups);
  if (g.wide && g.rows == 192)
    hipLaunchKernelGGL((lm_head_wide_kernel<3, 2, 2, 4>), grid, dim3(512), 0, s, q);
  else if (g.wide && g.rows == 256)
    hipLaunchKernelGGL((lm_head_wide_kernel<4, 2, 2, 4>), grid, dim3(512), 0, s, q);
  else if (g.wide)
    hipLaunchKernelGGL((lm_head_wide_kernel<5, 2, 2, 4>), grid, dim3(512), 0, s, q);
  else if (q.mgroups == 1)
    hipLaunchKernelGGL((lm_head_pair_kernel<5, true>), grid, dim3(256), 0, s, q);
  else if (g.rows == 160)
    hipLaunchKernelGGL((lm_head_pair_kernel<5, false>), grid, dim3(256), 0, s, q);
  else
    hipLaunchKernelGGL((lm_head_pair_kernel<4, false>), grid, dim3(256), 0, s, q);
  return hipGetLastError();
}

}  // namespace spexis
