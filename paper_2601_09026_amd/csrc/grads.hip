// Kernels of the parameter-gradient pass
//     dtheta_n = h * (dF/dtheta_n (Z_n))^T lambda_{n+1}            (paper section 3.1)
// that are not matrix products (those are launch_gemm_tn): the LayerNorm gain / shift gradients and sums
// over slots.  Sums over tokens are taken in two stages with a fixed order (no atomics): results are
// run-to-run identical.
#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace mg {

__global__ void __launch_bounds__(256) sum_slots_kernel(const float* in, int n, long elems, float* out, float scale) {
  const long i = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= elems) return;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < n; ++s) acc += *reinterpret_cast<const f32x4*>(in + (long)s * elems + i);
  *reinterpret_cast<f32x4*>(out + i) = scale * acc;
}

hipError_t launch_sum_slots(const float* in, int n, long elems, float* out, float scale, hipStream_t st) {
  if (n <= 0 || elems <= 0) return hipSuccess;
  if (elems % 4 != 0) return hipErrorInvalidValue;
  ProfScope ps(PC_ELEMENTWISE, 0.0, (double)(n + 1) * elems * 4, st);
  hipLaunchKernelGGL(sum_slots_kernel, dim3((unsigned)((elems / 4 + 255) / 256)), dim3(256), 0, st, in, n, elems, out,
                     scale);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// LayerNorm parameter gradients: dgamma[c] = sum_rows dy[r,c] * xhat[r,c], dbeta[c] = sum_rows
// dy[r,c], xhat recomputed from the LayerNorm input (state row + optional packed addend).
// One wavefront per row, a lane keeps the partial sums of its own columns in registers; the wavefronts
// of a block add theirs through LDS: partial[item][g][block] = [dgamma | dbeta] (2d floats), summed over the
// blocks by the second kernel.  All LayerNorms of a layer chunk go into one pair of launches.  Bound by
// reading its rows (10 bytes per element): 2 LayerNorms of one 4096 x 768 layer 20 + 5 us, of four layers
// 74 + 6 us (blocks of four wavefronts, 1024 over the launch: 20 + 8 and 74 + 10; 512 partial rows per group and one
// launch per LayerNorm: 2 x 47 + 4 x 8 us for the one layer).
// ---------------------------------------------------------------------------
constexpr int LNP_MAXV = 8;         // d <= 2048
constexpr int LNP_WAVES = 8;        // per block

// Blocks per (item, group): the two LayerNorms of a single layer give every CU one block, and a wavefront has at
// least 2 rows.  Their number follows from the rows alone: it decides the order of the sums, which must not depend on
// how many layers share the launch.
static int lnp_blocks(int T) {
  const int most = (T + 2 * LNP_WAVES - 1) / (2 * LNP_WAVES);
  return most < 128 ? most : 128;
}
size_t ln_param_partial_floats(int n_groups, int T, int d, int n_items) {
  return (size_t)n_items * n_groups * lnp_blocks(T) * 2 * d;
}

template <typename TO, int NV>
__global__ void __launch_bounds__(64 * LNP_WAVES) ln_param_partial_kernel(const LnParamArgs a, float* partial) {
  __shared__ __attribute__((aligned(16))) float red[LNP_WAVES - 1][NV * 256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = blockIdx.y, d = a.d;
  const LnParamItem it = a.item[blockIdx.z];
  f32x4 ag[NV], ab[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) { ag[i] = f32x4{0.f, 0.f, 0.f, 0.f}; ab[i] = ag[i]; }
  const TO* dyb = reinterpret_cast<const TO*>(it.dy) + it.dy_slots.of(g) * it.dy_slot_stride;
  const float* xb = a.X.at(g);
  const float* xab = it.xp ? it.xp + it.xp_slots.of(g) * it.xp_slot_stride : nullptr;
  for (int t = blockIdx.x * LNP_WAVES + wave; t < a.T; t += gridDim.x * LNP_WAVES) {
    const long ro = (long)t * d;
    f32x4 v[NV], dy[NV];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (i * 64 + lane) * 4;
      if (c < d) {
        v[i] = *reinterpret_cast<const f32x4*>(xb + ro + c);
        if (xab) v[i] += *reinterpret_cast<const f32x4*>(xab + ro + c);
        dy[i] = load4<TO>(dyb + ro + c);
        s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
      }
    }
    const float mu = wave_sum(s) / d;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if ((i * 64 + lane) * 4 < d) {
        v[i] = v[i] - mu;
        q += (v[i][0] * v[i][0] + v[i][1] * v[i][1]) + (v[i][2] * v[i][2] + v[i][3] * v[i][3]);
      }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / d + a.eps);
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if ((i * 64 + lane) * 4 < d) {
        ag[i] += dy[i] * (v[i] * rstd);
        ab[i] += dy[i];
      }
  }
  float* p = partial + (((long)blockIdx.z * gridDim.y + g) * gridDim.x + blockIdx.x) * 2 * d;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    f32x4(&acc)[NV] = half ? ab : ag;
    if (half) __syncthreads();
    if (wave > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) *reinterpret_cast<f32x4*>(&red[wave - 1][(i * 64 + lane) * 4]) = acc[i];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = (i * 64 + lane) * 4;
        f32x4 r[LNP_WAVES];
        r[0] = acc[i];
#pragma unroll
        for (int w = 1; w < LNP_WAVES; ++w) r[w] = *reinterpret_cast<const f32x4*>(&red[w - 1][c]);
#pragma unroll
        for (int n = LNP_WAVES / 2; n > 0; n /= 2)         // pairwise
#pragma unroll
          for (int w = 0; w < n; ++w) r[w] += r[w + n];
        if (c < d) *reinterpret_cast<f32x4*>(p + half * d + c) = r[0];
      }
    }
  }
}

// dgamma | dbeta of item z, group y: the partial rows summed, 64 columns per block; the rows are dealt to four
// wavefronts and their four sums added in a fixed order
__global__ void __launch_bounds__(256) ln_param_reduce_kernel(const LnParamArgs a, const float* partial, int n_rows) {
  __shared__ float red[4][64];
  const int g = blockIdx.y, d = a.d, l = threadIdx.x & 63, ph = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + l;                       // column of [dgamma | dbeta]
  float acc = 0.f;
  if (c < 2 * d) {
    const float* p = partial + ((long)blockIdx.z * gridDim.y + g) * n_rows * 2 * d + c;
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    int s = ph;
    for (; s + 12 < n_rows; s += 16) {
      a0 += p[(long)s * 2 * d]; a1 += p[(long)(s + 4) * 2 * d];
      a2 += p[(long)(s + 8) * 2 * d]; a3 += p[(long)(s + 12) * 2 * d];
    }
    for (; s < n_rows; s += 4) a0 += p[(long)s * 2 * d];
    acc = (a0 + a1) + (a2 + a3);
  }
  red[ph][l] = acc;
  __syncthreads();
  if (ph == 0 && c < 2 * d) {
    const LnParamItem it = a.item[blockIdx.z];
    float* o = reinterpret_cast<float*>(const_cast<char*>(a.out.at(g)) + (c < d ? it.gamma_off : it.beta_off));
    o[c < d ? c : c - d] = a.scale * ((red[0][l] + red[1][l]) + (red[2][l] + red[3][l]));
  }
}

template <typename TO>
static void lnp_dispatch(const LnParamArgs& a, float* partial, dim3 grid, hipStream_t st) {
  const int nv = (a.d + 255) / 256;
  if (nv <= 1) hipLaunchKernelGGL((ln_param_partial_kernel<TO, 1>), grid, dim3(64 * LNP_WAVES), 0, st, a, partial);
  else if (nv == 2) hipLaunchKernelGGL((ln_param_partial_kernel<TO, 2>), grid, dim3(64 * LNP_WAVES), 0, st, a, partial);
  else if (nv == 3) hipLaunchKernelGGL((ln_param_partial_kernel<TO, 3>), grid, dim3(64 * LNP_WAVES), 0, st, a, partial);
  else if (nv == 4) hipLaunchKernelGGL((ln_param_partial_kernel<TO, 4>), grid, dim3(64 * LNP_WAVES), 0, st, a, partial);
  else hipLaunchKernelGGL((ln_param_partial_kernel<TO, 8>), grid, dim3(64 * LNP_WAVES), 0, st, a, partial);
}

hipError_t launch_ln_param_grad(const LnParamArgs& a, float* partial, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0 || a.T <= 0 || a.n_items <= 0) return hipSuccess;
  if (a.d > 256 * LNP_MAXV || a.d % 4 != 0 || a.n_items > LN_PARAM_MAX) return hipErrorInvalidValue;
  double bytes = 0.0;
  for (int i = 0; i < a.n_items; ++i)
    bytes += (double)a.n_groups * a.T * a.d * ((is_bf16 ? 2 : 4) + 4 + (a.item[i].xp ? 4 : 0));
  ProfScope ps(PC_ELEMENTWISE, 0.0, bytes, st);
  const int nb = lnp_blocks(a.T);
  const dim3 grid(nb, a.n_groups, a.n_items);
  if (is_bf16) lnp_dispatch<bf16>(a, partial, grid, st);
  else lnp_dispatch<float>(a, partial, grid, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ln_param_reduce_kernel, dim3((2 * a.d + 63) / 64, a.n_groups, a.n_items), dim3(256), 0, st, a,
                     partial, nb);
  return hipGetLastError();
}

}  // namespace mg
