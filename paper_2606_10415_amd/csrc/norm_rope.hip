// RMSNorm and rotary position embedding of the LLaMA-2 / Qwen2.5 decoder
// layers the paper evaluates (Sec. 6.1), forward and backward, gfx950.
//
// All four operations are elementwise or per-row reductions: HBM-bound.
//   * rmsnorm_fwd: one wave per token row; lane l owns the 16-byte chunks
//     l, l + 64, ... of the row (coalesced), the sum of squares is a wave
//     shuffle reduction; writes y = w * x * r (one rounding) and r.
//       r = (mean_j x_j^2 + eps)^(-1/2)
//   * rmsnorm_bwd: workgroups of 4 waves (at most 512), on one row at a time
//     (rows of up to 1024 columns: two or four rows side by side); per row
//       dx = r * w * g - r^3 * x / H * sum_j g_j w_j x_j   (+ residual R)
//     with g, x and R read once, into registers, one row ahead.  Every thread
//     keeps the FP32 partial of dw = sum_rows g * x * r for its columns; the
//     workgroup writes one partial row to the workspace, and rmsnorm_dw_sum
//     adds those rows in a fixed order (deterministic, no atomics).
//   * rope_table: cos / sin of p * base^(-2i/D) for p < S, i < D/2, with the
//     angle formed and reduced in FP64 (positions up to 10^4 and more keep
//     full FP32 accuracy), stored as FP32 pairs.
//   * rope: in place on `heads` consecutive heads of each token row
//     (the Q and K heads of the fused QKV buffer); rotate-half pairing
//     (i, i + D/2); inverse = rotation by the negated angle (the gradient).

#include "common.hpp"
#include "kernels.hpp"

namespace lt {
namespace {

constexpr int kRowsPerWg = 4;        // rmsnorm: one wave per row, 4 waves per workgroup

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// ---------------------------------------------------------------- forward
template <int MAXK>
__global__ void __launch_bounds__(64 * kRowsPerWg)
rmsnorm_fwd_kernel(const lt_half* __restrict__ X, int64_t ldx, const lt_half* __restrict__ W,
                   lt_half* __restrict__ Y, int64_t ldy, float* __restrict__ RSTD, int64_t T,
                   int H, float eps) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kRowsPerWg + (threadIdx.x >> 6);
  if (row >= T) return;                          // whole wave leaves together
  const int nch = H / 8;                         // 16-byte chunks per row
  const lt_half* x = X + row * ldx;
  half8 xv[MAXK];
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    const int c = lane + 64 * k;
    xv[k] = c < nch ? as_half8(ld16(x + c * 8)) : as_half8(u32x4{0, 0, 0, 0});
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += (float)xv[k][e] * (float)xv[k][e];
  }
  ss = wave_sum(ss);
  const float r = 1.f / sqrtf(ss / (float)H + eps);
  lt_half* y = Y + row * ldy;
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    const int c = lane + 64 * k;
    if (c < nch) {
      const half8 wv = as_half8(ld16(W + c * 8));
      half8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (_Float16)((float)wv[e] * ((float)xv[k][e] * r));
      st16(y + c * 8, as_u32x4(o));
    }
  }
  if (lane == 0) RSTD[row] = r;
}

// ---------------------------------------------------------------- backward
// Workgroups of kBwdWaves waves, the whole workgroup on one row at a time:
// thread t owns the 16-byte chunks t, t + 256, ... of every row, so its w and
// its FP32 dw partial stay in registers (KPT chunks) and the workgroup's
// partial row needs no further sum.  HBM-bound (g, x, R in, dx out): the next
// row's loads are in flight while the current row's dot product goes through
// the waves (one barrier a row, sums in wave order).  With one wave per row a
// row's 30 KB were loaded, reduced and written in turn by 8 waves a CU: 4096 x
// 5120 took 52 us (3.2 TB/s), now 41.
// Narrow rows would leave lanes idle: up to 512 (1024) columns a row takes one
// (two) of the four waves, the groups take rows side by side and add their dw
// partials through LDS at the end.
constexpr int kBwdWaves = kRmsBwdWaves;
constexpr int kBwdThreads = 64 * kBwdWaves;

// KPT chunks per thread, WR waves per row
template <int KPT, int WR>
__global__ void __launch_bounds__(kBwdThreads)
rmsnorm_bwd_kernel(const lt_half* __restrict__ dY, int64_t lddy, const lt_half* __restrict__ X,
                   int64_t ldx, const lt_half* __restrict__ W, const float* __restrict__ RSTD,
                   const lt_half* __restrict__ R, int64_t ldr, lt_half* __restrict__ dX,
                   int64_t lddx, float* __restrict__ part, int64_t T, int H) {
  constexpr int GT = 64 * WR;                      // threads of a row group
  constexpr int NG = kBwdWaves / WR;               // row groups
  static_assert(NG == 1 || KPT == 1, "groups: rows of one chunk per thread");
  __shared__ float red[2][kBwdWaves];
  const int wave = threadIdx.x >> 6;
  const int grp = wave / WR;
  const int tid = threadIdx.x % GT;                // within the row group
  const int nch = H / 8;
  const float inv_h = 1.f / (float)H;
  const u32x4 zero = {0, 0, 0, 0};

  half8 wv[KPT];
  float dw[KPT][8];
#pragma unroll
  for (int k = 0; k < KPT; ++k) {
    const int c = tid + GT * k;
    wv[k] = as_half8(c < nch ? ld16(W + c * 8) : zero);
#pragma unroll
    for (int e = 0; e < 8; ++e) dw[k][e] = 0.f;
  }

  struct Row {
    half8 g[KPT], x[KPT], r[KPT];
    float rstd;
  };
  auto load = [&](int64_t row, Row& v) __attribute__((always_inline)) {
    v.rstd = RSTD[row];
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      const int c = tid + GT * k;
      v.g[k] = v.x[k] = v.r[k] = as_half8(zero);
      if (c < nch) {
        v.g[k] = as_half8(ld16(dY + row * lddy + c * 8));
        v.x[k] = as_half8(ld16(X + row * ldx + c * 8));
        if (R) v.r[k] = as_half8(ld16(R + row * ldr + c * 8));
      }
    }
  };
  // every thread of the workgroup takes the same rows (barrier inside)
  auto finish = [&](int64_t row, const Row& v, int buf) __attribute__((always_inline)) {
    float dot = 0.f;
#pragma unroll
    for (int k = 0; k < KPT; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) dot += (float)v.g[k][e] * (float)wv[k][e] * (float)v.x[k][e];
    dot = wave_sum(dot);
    float sum = dot;
    if constexpr (WR > 1) {
      if ((tid & 63) == 0) red[buf][wave] = dot;
      __syncthreads();
      sum = 0.f;
#pragma unroll
      for (int q = 0; q < WR; ++q) sum += red[buf][grp * WR + q];
    }
    const float r = v.rstd;
    const float c3 = r * r * r * sum * inv_h;
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      const int c = tid + GT * k;
      half8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float g = (float)v.g[k][e], x = (float)v.x[k][e];
        dw[k][e] += g * x * r;
        o[e] = (_Float16)((float)v.r[k][e] + (r * (float)wv[k][e] * g - c3 * x));
      }
      if (c < nch && (NG == 1 || row < T)) st16(dX + row * lddx + c * 8, as_u32x4(o));
    }
  };

  // rows blockIdx.x, + gridDim.x, ...: the workgroups sweep the arrays together
  // (a contiguous range each: 43 us against 41 at 4096 x 5120; a third row in
  // flight changes nothing).  Two rows per trip: two register sets, two
  // reduction slots (a slot is written again only after the barrier of the row
  // between).
  // Groups run the same number of steps (barriers inside); a group without a
  // row left repeats its last one with nothing stored and zero g.
  const int64_t step = (int64_t)gridDim.x * NG;
  const int64_t first = (int64_t)blockIdx.x * NG;
  auto load_row = [&](int64_t base, Row& v) __attribute__((always_inline)) {
    const int64_t row = base + grp;
    load(row < T ? row : T - 1, v);
    if (NG > 1 && row >= T) {
#pragma unroll
      for (int k = 0; k < KPT; ++k) v.g[k] = as_half8(zero);
    }
  };
  if (first < T) {
    Row a, b;
    load_row(first, a);
    for (int64_t row = first; row < T; row += 2 * step) {
      if (row + step < T) load_row(row + step, b);
      finish(row + grp, a, 0);
      if (row + step >= T) break;
      if (row + 2 * step < T) load_row(row + 2 * step, a);
      finish(row + step + grp, b, 1);
    }
  }

  if constexpr (NG > 1) {
    // the other groups' partials, added in group order by the first
    __shared__ float acc[NG - 1][GT * 8];
    if (grp > 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[grp - 1][tid * 8 + e] = dw[0][e];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 0; g < NG - 1; ++g)
#pragma unroll
      for (int e = 0; e < 8; ++e) dw[0][e] += acc[g][tid * 8 + e];
  }

  float* dst = part + (int64_t)blockIdx.x * H;
#pragma unroll
  for (int k = 0; k < KPT; ++k) {
    const int c = tid + GT * k;
    if (c < nch) {
      *reinterpret_cast<float4*>(dst + c * 8) = make_float4(dw[k][0], dw[k][1], dw[k][2], dw[k][3]);
      *reinterpret_cast<float4*>(dst + c * 8 + 4) = make_float4(dw[k][4], dw[k][5], dw[k][6], dw[k][7]);
    }
  }
}

// dW[j] = sum over the partial rows; FP16 result.  Workgroup = 16 waves over
// 64 columns (lane = column, coalesced): wave v sums partial rows v, v + 16,
// ... in order (eight loads in flight at a time), then wave 0 adds the 16
// wave sums in order (deterministic).
constexpr int kSumWaves = 16;

__global__ void __launch_bounds__(64 * kSumWaves)
rmsnorm_dw_sum_kernel(const float* __restrict__ part, int nparts, int H, lt_half* __restrict__ dW) {
  __shared__ float red[kSumWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + lane;
  float s = 0.f;
  if (j < H) {
    // eight partial rows loaded together, added in row order
    for (int t = wave; t < nparts; t += 8 * kSumWaves) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int tu = t + u * kSumWaves;
        v[u] = tu < nparts ? part[(int64_t)tu * H + j] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && j < H) {
    float tot = 0.f;
#pragma unroll
    for (int v = 0; v < kSumWaves; ++v) tot += red[v][lane];
    reinterpret_cast<_Float16*>(dW)[j] = (_Float16)tot;
  }
}

// ---------------------------------------------------------------- rotary
__global__ void __launch_bounds__(256)
rope_table_kernel(float* __restrict__ CS, int S, int D, double base) {
  const int half = D / 2;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)S * half) return;
  const int p = (int)(idx / half);
  const int i = (int)(idx % half);
  const double theta = pow(base, -2.0 * (double)i / (double)D);
  const double a = fmod((double)p * theta, 6.283185307179586476925286766559);
  double s, c;
  sincos(a, &s, &c);
  CS[2 * idx] = (float)c;
  CS[2 * idx + 1] = (float)s;
}

// One thread: 8 consecutive pair indices i (and their partners i + D/2) of
// one head of one token.
__global__ void __launch_bounds__(256)
rope_kernel(lt_half* __restrict__ X, int64_t stride, int64_t T, int S, int heads, int D,
            const float* __restrict__ CS, float sign) {
  const int half = D / 2;
  const int gph = half / 8;                      // 8-pair groups per head
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= T * heads * gph) return;
  const int gi = (int)(idx % gph);
  const int64_t th = idx / gph;
  const int h = (int)(th % heads);
  const int64_t t = th / heads;                  // token row b*S + p
  const int p = (int)(t % S);
  lt_half* x = X + t * stride + (int64_t)h * D + gi * 8;
  const half8 x1 = as_half8(ld16(x));
  const half8 x2 = as_half8(ld16(x + half));
  const float4* cs = reinterpret_cast<const float4*>(CS + ((int64_t)p * half + gi * 8) * 2);
  half8 y1, y2;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = cs[q];                      // (cos, sin) of pairs 2q, 2q + 1
    const float cc[2] = {v.x, v.z};
    const float ss[2] = {sign * v.y, sign * v.w};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = 2 * q + u;
      const float a = (float)x1[e], b = (float)x2[e];
      y1[e] = (_Float16)(a * cc[u] - b * ss[u]);
      y2[e] = (_Float16)(b * cc[u] + a * ss[u]);
    }
  }
  st16(x, as_u32x4(y1));
  st16(x + half, as_u32x4(y2));
}

template <int MAXK>
hipError_t launch_rms_fwd(const lt_half* X, int64_t ldx, const lt_half* W, lt_half* Y, int64_t ldy,
                          float* RSTD, int64_t T, int64_t H, float eps, hipStream_t s) {
  const unsigned grid = (unsigned)((T + kRowsPerWg - 1) / kRowsPerWg);
  hipLaunchKernelGGL((rmsnorm_fwd_kernel<MAXK>), dim3(grid), dim3(64 * kRowsPerWg), 0, s, X, ldx,
                     W, Y, ldy, RSTD, T, (int)H, eps);
  return hipGetLastError();
}

template <int KPT, int WR>
hipError_t launch_rms_bwd(const RmsBwdArgs& a, hipStream_t s) {
  const int nblk = rmsnorm_bwd_blocks(a.T);
  hipLaunchKernelGGL((rmsnorm_bwd_kernel<KPT, WR>), dim3((unsigned)nblk), dim3(kBwdThreads), 0, s,
                     a.dY, a.lddy, a.X, a.ldx, a.W, a.RSTD, a.R, a.ldr, a.dX, a.lddx, a.part, a.T,
                     (int)a.H);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(rmsnorm_dw_sum_kernel, dim3((unsigned)((a.H + 63) / 64)), dim3(64 * kSumWaves),
                     0, s, a.part, nblk, (int)a.H, a.dW);
  return hipGetLastError();
}

}  // namespace

// H <= 8192 (validated by the caller): up to 16 chunks of 8 per lane.
hipError_t rmsnorm_fwd_launch(const lt_half* X, int64_t ldx, const lt_half* W, lt_half* Y,
                              int64_t ldy, float* RSTD, int64_t T, int64_t H, float eps,
                              hipStream_t s) {
  const int64_t k = (H / 8 + 63) / 64;
  if (k <= 4) return launch_rms_fwd<4>(X, ldx, W, Y, ldy, RSTD, T, H, eps, s);
  if (k <= 8) return launch_rms_fwd<8>(X, ldx, W, Y, ldy, RSTD, T, H, eps, s);
  return launch_rms_fwd<16>(X, ldx, W, Y, ldy, RSTD, T, H, eps, s);
}

hipError_t rmsnorm_bwd_launch(const RmsBwdArgs& a, hipStream_t s) {
  const int64_t nch = a.H / 8;
  if (nch <= 64) return launch_rms_bwd<1, 1>(a, s);
  if (nch <= 128) return launch_rms_bwd<1, 2>(a, s);
  switch ((nch + kBwdThreads - 1) / kBwdThreads) {   // chunks per thread: H <= 8192
    case 1: return launch_rms_bwd<1, 4>(a, s);
    case 2: return launch_rms_bwd<2, 4>(a, s);
    case 3: return launch_rms_bwd<3, 4>(a, s);
    default: return launch_rms_bwd<4, 4>(a, s);
  }
}

hipError_t rope_table_launch(float* CS, int S, int D, double base, hipStream_t s) {
  const int64_t n = (int64_t)S * (D / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, CS, S,
                     D, base);
  return hipGetLastError();
}

hipError_t rope_launch(lt_half* X, int64_t stride, int B, int S, int heads, int D, const float* CS,
                       int inverse, hipStream_t s) {
  const int64_t T = (int64_t)B * S;
  const int64_t n = T * heads * (D / 16);
  hipLaunchKernelGGL(rope_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, stride, T,
                     S, heads, D, CS, inverse ? -1.f : 1.f);
  return hipGetLastError();
}

}  // namespace lt
