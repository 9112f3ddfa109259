// Linear layers of the drafting adapter (Implementation: a linear layer and an attention layer,
// then the LM head): y = x W^T (+ R) for bf16 x [M][K], a packed W [N][K], an optional bf16
// residual R [M][N], bf16 output y [M][N], fp32 accumulation.
//
// The adapter runs once per drafted token on the batch's exit hidden states: M is the batch (one to
// hundreds of rows).  Most of its layers run in linear_kernel below, K split over a workgroup's waves.
// Larger ones run on the projection kernel of the LM head (lm_head.hip), the K range split over
// workgroups until the chip is covered -- as long as the fp32 partials cost no more traffic than the
// weight; then a second kernel adds the partials in order, adds the residual and rounds to bf16;
// without a split the projection writes bf16 (with the residual) itself.  Several layers of one input
// (the attention layer's q, k, v) run as one layer of their stacked weights whose columns go each to
// their own output.
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace spexis {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;   // NaN
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Buffer loads (out-of-range lanes read zeros and fetch nothing); kept out of the kernel template, whose
// host side cannot instantiate these builtins.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 buffer_ld16(__amdgpu_buffer_rsrc_t rs, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
}
__device__ __forceinline__ u32x4 buffer_ld16_nt(__amdgpu_buffer_rsrc_t rs, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 2);
}

// Four consecutive outputs (row, c..c+3) of the layer: the residual added, rounded to bf16, stored to
// the output that owns the columns (with split outputs its bounds are multiples of 4).
__device__ __forceinline__ void put_outputs(const LinearParams& p, int64_t row, int c, f32x4 v) {
  uint16_t* y = reinterpret_cast<uint16_t*>(p.y) + row * p.N + c;
  if (p.nout > 0) {
    void* base = p.ys[0];
    int lo = 0, hi = p.off[1];
#pragma unroll
    for (int j = 1; j < kLinearMaxOutputs; ++j)
      if (j < p.nout && c >= p.off[j]) {
        base = p.ys[j];
        lo = p.off[j];
        hi = p.off[j + 1];
      }
    y = reinterpret_cast<uint16_t*>(base) + row * (hi - lo) + (c - lo);
  }
  const uint16_t* r = p.res ? reinterpret_cast<const uint16_t*>(p.res) + row * p.N + c : nullptr;
  if (p.vec4) {   // all four columns exist, 8-byte aligned
    if (r) {
      const u32x2 q = *reinterpret_cast<const u32x2*>(r);
      v[0] += __uint_as_float(q[0] << 16);
      v[1] += __uint_as_float(q[0] & 0xFFFF0000u);
      v[2] += __uint_as_float(q[1] << 16);
      v[3] += __uint_as_float(q[1] & 0xFFFF0000u);
    }
    u32x2 o;
    o[0] = (uint32_t)to_bf16(v[0]) | ((uint32_t)to_bf16(v[1]) << 16);
    o[1] = (uint32_t)to_bf16(v[2]) | ((uint32_t)to_bf16(v[3]) << 16);
    *reinterpret_cast<u32x2*>(y) = o;
  } else {
    for (int i = 0; i < 4 && c + i < p.N; ++i) y[i] = to_bf16(r ? v[i] + from_bf16(r[i]) : v[i]);
  }
}

}  // namespace

// y for up to 32 RT rows x 32 CT columns per workgroup, the whole of K inside it: its NW waves take equal
// contiguous parts of K, each computes the full tile from its part, and the partials are added in wave
// order through LDS.  So one launch gives the layer's bf16 output, no partials go through memory, and
// the tile loop has no barrier: x goes through each wave's own LDS (whose operations run in order).
// These layers are bound by the operand bytes a CU takes in (a workgroup reads its columns of W and
// its rows of x once, about 40 bytes a cycle; M x K of x comes from L2 once per column tile) and by
// one chain of launch, first loads and reduction of about 6 us, so the fewest launches and the
// smallest tile that still fills the chip in one go win.  Two steps of x and W in flight per wave:
// with four of W the registers leave one workgroup per CU instead of two (2 x 2 tiles: 34.3 against
// 27.9 us at 320 x 4096 x 4096).  The scheduling barriers keep the loads where they are written; the
// compiler gathers them at the loop's end otherwise and each wave waits for all of them.
template <int RT, int CT, int NW, bool kStream>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2)))
void linear_kernel(LinearParams p) {
  constexpr int DX = 2, DW = 2;   // steps of x and of W in flight
  constexpr int kRows = 32 * RT, kCols = 32 * CT;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int K = p.proj.d, tiles = (p.N + 31) / 32, ctiles = (tiles + CT - 1) / CT;
  const int groups = (p.M + kRows - 1) / kRows;
  const int local = blockIdx.x >> 3;
  const int g = local % groups, nt = (local / groups) * 8 + (blockIdx.x & 7);
  if (nt >= ctiles) return;
  const int m0 = g * kRows, rows = min(kRows, p.M - m0);
  // this wave's K-steps of 64
  const int nsteps = K / kLmK, s0 = wave * nsteps / NW, n = (wave + 1) * nsteps / NW - s0;
  const __amdgpu_buffer_rsrc_t xrs = buffer_of(
      reinterpret_cast<const uint16_t*>(p.proj.h) + (int64_t)m0 * K + s0 * kLmK, (rows * K - s0 * kLmK) * 2);
  const uint16_t* wbase = reinterpret_cast<const uint16_t*>(p.proj.w);
  int woff[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) woff[c] = lane * 16;
  __amdgpu_buffer_rsrc_t wrs[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int tile = min(nt * CT + c, tiles - 1);
    wrs[c] = buffer_of(wbase + ((int64_t)tile * nsteps + s0) * kPackTile, nt * CT + c < tiles ? n * kPackTile * 2 : 0);
  }

  // per wave: the staged step of x (row r, 16-byte chunk kc at r * 8 + (kc ^ ((r >> 1) & 7)), so that the
  // 16 rows of one ds_read_b128 pass hit distinct bank groups); at the end, its partial sums
  constexpr int kStage = kRows * 8, kPart = kRows * kCols / 4;   // 16-byte units
  __shared__ u32x4 sm[NW][kStage > kPart ? kStage : kPart];
  u32x4* const st = sm[wave];
  constexpr int kXL = kStage / 64;   // loads of an step of x per lane
  int xoff[kXL];
#pragma unroll
  for (int u = 0; u < kXL; ++u) {
    const int q = lane + 64 * u;
    xoff[u] = (q >> 3) * K * 2 + (q & 7) * 16;
  }
  u32x4 xreg[DX][kXL], wb[DW][CT][4];
  auto load_x = [&](u32x4 (&dst)[kXL], int i) {
    const int add = i < n ? i * (kLmK * 2) : 0x40000000;   // past the wave's steps: out of range
#pragma unroll
    for (int u = 0; u < kXL; ++u) dst[u] = buffer_ld16(xrs, xoff[u] + add);
  };
  auto load_w = [&](u32x4 (&dst)[CT][4], int i) {
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int off = woff[c] + s * 1024 + i * (kPackTile * 2);
        dst[c][s] = kStream ? buffer_ld16_nt(wrs[c], off) : buffer_ld16(wrs[c], off);
      }
  };
  f32x16 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][c][e] = 0.f;

#pragma unroll
  for (int i = 0; i < DX; ++i) load_x(xreg[i], i);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < DW; ++i) load_w(wb[i], i);
  __builtin_amdgcn_sched_barrier(0);
  for (int i = 0; i < n; i += DW) {
#pragma unroll
    for (int jj = 0; jj < DW; ++jj) {
      wave_lds_fence();   // this step's writes follow the last step's reads
#pragma unroll
      for (int u = 0; u < kXL; ++u) {
        const int q = lane + 64 * u, r = q >> 3, kc = q & 7;
        st[r * 8 + (kc ^ ((r >> 1) & 7))] = xreg[jj % DX][u];
      }
      wave_lds_fence();   // and its reads its writes
      load_x(xreg[jj % DX], i + jj + DX);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 a[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const int m = 32 * t + col;
          a[t] = st[m * 8 + ((4 * half + s) ^ ((m >> 1) & 7))];
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
          for (int t = 0; t < RT; ++t)
            acc[t][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a[t]), as_bf16x8(wb[jj][c][s]), acc[t][c], 0, 0, 0);
      }
      load_w(wb[jj], i + jj + DW);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // the waves' partials through LDS (over the wave's own last step), added in wave order
  wave_lds_fence();
  float* mine = reinterpret_cast<float*>(st);
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        mine[(32 * t + 8 * (e >> 2) + 4 * half + (e & 3)) * kCols + 32 * c + col] = acc[t][c][e];
  __syncthreads();
  const int n0 = nt * kCols;
  for (int q = threadIdx.x; q < kPart; q += 64 * NW) {
    const int r = q / (kCols / 4), c = (q % (kCols / 4)) * 4;
    if (r >= rows || n0 + c >= p.N) continue;
    f32x4 v = __builtin_bit_cast(f32x4, sm[0][q]);
#pragma unroll
    for (int w = 1; w < NW; ++w) v += __builtin_bit_cast(f32x4, sm[w][q]);
    put_outputs(p, m0 + r, n0 + c, v);
  }
}

// y = bf16(sum_s part[s] (in order) + R): 4 consecutive outputs per thread; with split outputs,
// each group of four goes to the output that owns its columns.
__global__ __launch_bounds__(kThreads) void linear_reduce_kernel(LinearParams p) {
  const int64_t total = (int64_t)p.M * p.N;
  const int64_t e0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
  if (e0 >= total) return;
  const int cnt = (int)min((int64_t)4, total - e0);
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (cnt == 4 && (total & 3) == 0) {   // 16-byte aligned in every partial
    // the partials in groups of 8, every load of a group issued together, added in order
    for (int s0 = 0; s0 < p.S; s0 += 8) {
      f32x4 x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        x[u] = *reinterpret_cast<const f32x4*>(p.part + (int64_t)min(s0 + u, p.S - 1) * total + e0);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < p.S)
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] += x[u][i];
    }
  } else {
    for (int s = 0; s < p.S; ++s)
      for (int i = 0; i < cnt; ++i) v[i] += p.part[(int64_t)s * total + e0 + i];
  }
  uint16_t* y = reinterpret_cast<uint16_t*>(p.y) + e0;
  if (p.nout > 0) {
    // split outputs: the four columns lie in one output (its bounds are multiples of 4)
    const int64_t row = e0 / p.N;
    const int c = (int)(e0 - row * p.N);
    void* base = p.ys[0];
    int lo = 0, hi = p.off[1];
#pragma unroll
    for (int j = 1; j < kLinearMaxOutputs; ++j)
      if (j < p.nout && c >= p.off[j]) {
        base = p.ys[j];
        lo = p.off[j];
        hi = p.off[j + 1];
      }
    y = reinterpret_cast<uint16_t*>(base) + row * (hi - lo) + (c - lo);
  }
  const uint16_t* r = p.res ? reinterpret_cast<const uint16_t*>(p.res) + e0 : nullptr;
  for (int i = 0; i < cnt; ++i) y[i] = to_bf16(r ? v[i] + from_bf16(r[i]) : v[i]);
}

// K split for a problem (the same choice in the workspace query and the launch): the smallest
// power of two up to 8 that gives at least 256 workgroups, while K / S stays a multiple of 64 and the
// partials (S M N fp32, written once and read once) stay within the weight's own traffic
// (2 S M N 4 <= 2 N K 2, i.e. 2 S M <= K).
int linear_split(int M, int N, int K) {
  const int64_t wgs = projection_workgroups(M, N);
  int S = 1;
  while (S < 8 && wgs * S < 256 && K % (kLmK * 2 * S) == 0 && (int64_t)2 * (2 * S) * M <= K) S *= 2;
  return S;
}

template <int RT, int CT, int NW>
static hipError_t launch_linear_t(const LinearParams& p, hipStream_t s) {
  const int64_t groups = (p.M + 32 * RT - 1) / (32 * RT), ctiles = ((p.N + 31) / 32 + CT - 1) / CT;
  const dim3 g((unsigned)((ctiles + 7) / 8 * 8 * groups));
  if (groups == 1)
    hipLaunchKernelGGL((linear_kernel<RT, CT, NW, true>), g, dim3(64 * NW), 0, s, p);
  else
    hipLaunchKernelGGL((linear_kernel<RT, CT, NW, false>), g, dim3(64 * NW), 0, s, p);
  return hipGetLastError();
}

// Microseconds of linear_kernel's shape 3 and of the projection with its reduce, for more than 128 rows.  Both go
// by whole rounds of workgroups over the CUs: a CU's time for one of linear_kernel's grows with K alone (two
// share it, so a round is one for each CU), and for one of the projection's with its part of K and its rows;
// the fp32 partials are written and read.  Fitted to 700 shapes of 2048 to 8192 x 256 to 28672 at 144 to 2048
// rows: the kernel taken was within 8% of the quicker one.  The longer K, the more a round and a bit costs: 54.3
// against 42.5 us at 320 x 4096 x 8192, 56.9 against 39.1 at 160 x 6144 x 8192, but 56.4 against 74.3 at 512 x 3584
// x 8192 and 29.5 against 32.7 at 320 x 4096 x 4096 (linear_kernel against the projection).
static double linear_us(int64_t M, int64_t N, int64_t K) {
  const int64_t wgs = ((N + 63) / 64 + 7) / 8 * 8 * ((M + 63) / 64);
  return 2 + 3.2 / 1024 * K * ((wgs + 255) / 256);
}
static double projection_us(int64_t M, int64_t N, int64_t K) {
  const int64_t S = linear_split((int)M, (int)N, (int)K), g = group_rows(M);
  if (S == 1) return INFINITY;   // narrow and without a split: a few CUs do it all
  const int64_t wgs = launched_workgroups(N, (M + g - 1) / g) * S;
  return 6 + 0.017 / 160 * g * K / S * ((wgs + 255) / 256) + 8.0 / 5e6 * M * N * S;
}

// The shape of linear_kernel for a problem, or 0 for the projection kernel (K split over workgroups,
// then the reduce): 1: 32 rows x 32 columns, 2: 64 x 32, 3: 64 x 64 per workgroup.  The smallest tile
// whose workgroups fit the 256 CUs at once, and one of 32 rows for up to 32.  Measured (weights from
// HBM, projection and reduce against linear_kernel): 13.4 against 10.1 us at 1 x 4096 x 4096, 17.8
// against 11.9 at 64 x 4096 x 4096 (shape 1; shape 2: 15.2), 25.1 against 16.1 at 64 x 6144 x 4096
// (shape 2; shape 1: 19.8), 36.2 against 21.2 at 128 x 6144 x 4096 (shape 3; shape 2: 25.3), 52.6
// against 26.9 at 512 x 3584 x 3584 (shape 3).  The projection is the quicker one
//   * for a long K and few workgroups, whose waves are one long chain each: 14.1 against 20.2 us at 32 x 1024 x
//     8192, 11.7 against 14.4 at 1 x 256 x 8192, 17.2 against 21.0 at 64 x 2048 x 8192 (15.1 against 14.2 at 64 x
//     2048 x 6144); 29.7 against 26.1 at 16 x 4096 x 14336;
//   * where its own tiles fill the chip: over 32640 columns, without a split, 7.7 against 10.0 us at 1 x 32768 x
//     256, 84.6 against 93.3 at 32 x 32768 x 8192 (but 12.4 against 9.9 at 33 x 32768 x 256); 101 against 152 us
//     at 2048 x 4096 x 4096, 73.4 against 75.5 at 128 x 28672 x 4096.  (62.9 against 59.1 at 1024 x 4096 x 4096;
//     past 1024 workgroups, to about 1400, some sizes would still gain by linear_kernel: 133 against 75 us at
//     1280 x 4096 x 4096);
//   * where linear_kernel's rounds are half empty (above; 63.4 against 68.2 us at 128 x 10240 x 8192).
static int linear_shape(int M, int N, int K) {
  if (K > 8192 || N > 32768) return 0;
  const int64_t tiles = (N + 31) / 32, g64 = (M + 63) / 64;
  if (M <= 32) {
    const bool chain = N <= 4096 && (int64_t)K * (M + 64) >= 300000 + 72 * (int64_t)N;
    return chain || (N > 32640 && (K < 512 || K > 4096)) ? 0 : 1;
  }
  if (tiles * ((M + 31) / 32) <= 256) return M <= 64 && N <= 3072 && K > 6144 ? 0 : 1;
  if (tiles * g64 <= 256) return 2;
  const int64_t wgs = (tiles + 1) / 2 * g64;
  if (M <= 64) return N > 32640 && K >= 4096 ? 0 : 3;
  if (M <= 128) return wgs > (K > 6144 ? 256 : 512) ? 0 : 3;
  return wgs <= 1024 && linear_us(M, N, K) <= projection_us(M, N, K) ? 3 : 0;
}

hipError_t launch_linear(const LinearParams& p, hipStream_t s) {
  switch (linear_shape(p.M, p.N, p.proj.d)) {
    case 1: return launch_linear_t<1, 1, 8>(p, s);
    case 2: return launch_linear_t<2, 1, 4>(p, s);
    case 3: return launch_linear_t<2, 2, 4>(p, s);
  }
  hipError_t e = launch_projection(p.proj, s);
  if (e != hipSuccess || (p.S == 1 && p.nout == 0)) return e;
  const int64_t quads = ((int64_t)p.M * p.N + 3) / 4;
  hipLaunchKernelGGL(linear_reduce_kernel, dim3((unsigned)((quads + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                     p);
  return hipGetLastError();
}

}  // namespace spexis
