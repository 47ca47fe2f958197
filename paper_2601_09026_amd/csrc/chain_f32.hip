// The chains of chain.hip for fp32 layers 64 wide: what is local to a token row in one launch on either side of attention.
//
// Such layers come in few tokens and are bound by the number of dependent launches and, inside one, by trips to memory.  A
// block of four wavefronts owns 16 or 32 rows; a wavefront computes a quarter of each product's columns on the 16x16x4 MFMA
// and asks for all its weights (144 registers a lane for 256 hidden features) before it does anything else, so that a
// launch waits for memory once.  The rows pass from one product to the next through LDS, where LayerNorm takes 16 lanes a row.
// Whole layer steps launch by launch -> on chains, forward / adjoint with the cache pass, 256 hidden: 4 layers of 2 x 32
// tokens 31 / 59 -> 21 / 43 us, of 4 x 512 tokens 64 / 156 -> 48 / 128, 16 layers of 16 x 512 tokens 546 / 1460 -> 400 / 1230.
// What is left of the smallest: head and adjoint_head take 5 to 6 us, tail and adjoint_tail 10 to 11, of which the products are
// 1 to 2, the rest a launch's start, one trip to memory, the steps between the products and its end.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace mg {
namespace {

constexpr int D = 64, LD = D + 4;                          // row pitch: 16 rows of a 16-byte read fall on distinct slots

__device__ __forceinline__ f32x4 ld4(const float* p) { return ld_global(reinterpret_cast<const f32x4*>(p)); }
__device__ __forceinline__ void st4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ float sum16(float v) {          // over the 16 lanes of a row
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float sum4(f32x4 v) { return (v[0] + v[1]) + (v[2] + v[3]); }
__device__ __forceinline__ float dot4(f32x4 a, f32x4 b) { return (a[0] * b[0] + a[1] * b[1]) + (a[2] * b[2] + a[3] * b[3]); }
__device__ __forceinline__ void lds_barrier() {            // loads into registers stay in flight
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  bare_barrier();
}

// 16 features of 16 rows, features 4 lg + r of row l % 16 in lane l (lg = l / 16): w and x hold reduction indices
// 16 g + 4 lg + e of their row.
template <int KG> __device__ __forceinline__ f32x4 product(const f32x4 (&w)[KG], const f32x4 (&x)[KG]) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < KG; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[g][e], x[g][e], acc, 0, 0, 0);
  return acc;
}
// w: rows n0 .. n0 + 15 of a matrix of row length ld
template <int KG> __device__ __forceinline__ void weights(f32x4 (&w)[KG], const char* m, int n0, int ld, int lane) {
  const float* p = reinterpret_cast<const float*>(m) + (long)(n0 + (lane & 15)) * ld + 4 * (lane >> 4);
#pragma unroll
  for (int g = 0; g < KG; ++g) w[g] = ld4(p + 16 * g);
}
template <int KG> __device__ __forceinline__ void operand(f32x4 (&x)[KG], const float* lds, int pitch, int lane) {
  const float* p = lds + (lane & 15) * pitch + 4 * (lane >> 4);
#pragma unroll
  for (int g = 0; g < KG; ++g) x[g] = *reinterpret_cast<const f32x4*>(p + 16 * g);
}

// RT row tiles of 16: rows row0 .. ; the row a lane serves in a product (t) and in a LayerNorm (t)
template <int RT> struct Place {
  int g, row0, wave, lane, T;
  bool none;
  __device__ __forceinline__ Place(int T_, int tiles_m, int total, int per_xcd) : T(T_) {
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    none = tile >= total;
    g = __builtin_amdgcn_readfirstlane(tile / tiles_m);
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    row0 = __builtin_amdgcn_readfirstlane(tile - g * tiles_m) * 16 * RT;
  }
  __device__ __forceinline__ int clamp(int r) const { return r < T ? r : T - 1; }
  __device__ __forceinline__ int prow(int t) const { return row0 + 16 * t + (lane & 15); }
  __device__ __forceinline__ int lrow(int t) const { return 16 * t + 4 * wave + (lane >> 4); }   // inside the block
  __device__ __forceinline__ int lcol() const { return 4 * (lane & 15); }
};

struct Norm { f32x4 xn; float rstd; };
__device__ __forceinline__ Norm normalise(f32x4 v, float eps) {
  const float mu = sum16(sum4(v)) / D;
  v = v - mu;
  const float rstd = 1.0f / sqrtf(sum16(dot4(v, v)) / D + eps);
  return {v * rstd, rstd};
}
__device__ __forceinline__ f32x4 vjp(f32x4 dy, f32x4 gamma, f32x4 xh, float rstd) {
  const f32x4 w = dy * gamma;
  const float m1 = sum16(sum4(w)) / D, m2 = sum16(dot4(w, xh)) / D;
  return rstd * (w - m1 - xh * m2);
}

template <int RT>
__global__ void __launch_bounds__(256, 2) chain_f32_head_kernel(const ChainHeadArgs a, int tiles_m, int total, int per_xcd) {
  __shared__ __attribute__((aligned(16))) float us[RT * 16 * LD];
  const Place<RT> p(a.T, tiles_m, total, per_xcd);
  if (p.none) return;
  const int lane = p.lane, lg = lane >> 4;
  const char* pb = a.P.at(p.g);
  const float* X = a.X.at(p.g);
  f32x4 v[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) v[t] = ld4(X + (long)p.clamp(p.row0 + p.lrow(t)) * D + p.lcol());
  const f32x4 gamma = ld4(reinterpret_cast<const float*>(pb + a.g_off) + p.lcol());
  const f32x4 beta = ld4(reinterpret_cast<const float*>(pb + a.be_off) + p.lcol());
  f32x4 w[3][4], b[3];
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    weights(w[n], pb + a.w_off, 48 * p.wave + 16 * n, D, lane);
    b[n] = ld4(reinterpret_cast<const float*>(pb + a.b_off) + 48 * p.wave + 16 * n + 4 * lg);
  }
  __builtin_amdgcn_sched_barrier(0);
  const long cs = a.cs.of(p.g);
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const Norm n = normalise(v[t], a.eps);
    const f32x4 u = n.xn * gamma + beta;
    st4(us + p.lrow(t) * LD + p.lcol(), u);
    const int row = p.row0 + p.lrow(t);
    if (row < p.T) {
      const long at = (cs * p.T + row) * D + p.lcol();
      if (a.xhat) {
        st4(reinterpret_cast<float*>(a.xhat) + at, n.xn);
        if ((lane & 15) == 0) a.rstd[cs * p.T + row] = n.rstd;
      }
      if (a.u) st4(reinterpret_cast<float*>(a.u) + at, u);
    }
  }
  lds_barrier();
  float* out = reinterpret_cast<float*>(a.out) + a.out_slots.of(p.g) * p.T * 3 * D + 48 * p.wave + 4 * lg;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    f32x4 x[4];
    operand(x, us + 16 * t * LD, LD, lane);
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const f32x4 q = product(w[n], x) + b[n];
      if (p.prow(t) < p.T) st4(out + (long)p.prow(t) * 3 * D + 16 * n, q);
    }
  }
}

// MODE as in chain.hip; NF = hidden features / 64
template <int RT, int NF, int MODE>
__global__ void __launch_bounds__(256, 2) chain_f32_tail_kernel(const ChainTailArgs a, int tiles_m, int total, int per_xcd) {
  constexpr int F = 64 * NF, LDH = F + 4;
  __shared__ __attribute__((aligned(16))) float us[RT * 16 * LD], hs[RT * 16 * LDH];
  const Place<RT> p(a.T, tiles_m, total, per_xcd);
  if (p.none) return;
  const int lane = p.lane, lg = lane >> 4, n0 = 16 * p.wave + 4 * lg;
  const char* pb = a.P.at(p.g);
  auto vec = [&](long off, int c) { return ld4(reinterpret_cast<const float*>(pb + off) + c); };
  const float* o = reinterpret_cast<const float*>(a.o) + a.o_slots.of(p.g) * a.o_slot_stride;
  const float* X = a.X.at(p.g);
  f32x4 ox[RT][4], xin[RT], base[RT], wo[4], w1[NF][4], w2[4 * NF], b1[NF];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int row = p.clamp(p.prow(t));
#pragma unroll
    for (int g = 0; g < 4; ++g) ox[t][g] = ld4(o + (long)row * D + 16 * g + 4 * lg);
    xin[t] = ld4(X + (long)row * D + n0);
    if (a.base) base[t] = ld4(a.base + a.base_slots.of(p.g) * a.base_slot_stride + (long)row * D + n0);
  }
  weights(wo, pb + a.wo_off, 16 * p.wave, D, lane);
  const f32x4 bo = vec(a.bo_off, n0), gamma = vec(a.g_off, p.lcol()), beta = vec(a.be_off, p.lcol());
#pragma unroll
  for (int n = 0; n < NF; ++n) {
    weights(w1[n], pb + a.w1_off, 16 * NF * p.wave + 16 * n, D, lane);
    b1[n] = vec(a.b1_off, 16 * NF * p.wave + 16 * n + 4 * lg);
  }
  f32x4 b2 = {};
  if constexpr (MODE != 1) {
    weights(w2, pb + a.w2_off, 16 * p.wave, F, lane);
    b2 = vec(a.b2_off, n0);
  }
  __builtin_amdgcn_sched_barrier(0);

  const long cs = a.cs.of(p.g);
  f32x4 y[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {                           // ybar = o Wo^T + bo (+ base)
    y[t] = product(wo, ox[t]) + bo;
    if (a.base) y[t] += base[t];
    if (MODE && a.ybar && p.prow(t) < p.T) st4(a.ybar + (cs * p.T + p.prow(t)) * D + n0, y[t]);
    st4(us + (16 * t + (lane & 15)) * LD + n0, xin[t] + y[t]);
  }
  lds_barrier();
#pragma unroll
  for (int t = 0; t < RT; ++t) {                           // u = LN2(X + ybar), in place
    float* at = us + p.lrow(t) * LD + p.lcol();
    const Norm n = normalise(*reinterpret_cast<const f32x4*>(at), a.eps);
    const f32x4 u = n.xn * gamma + beta;
    st4(at, u);
    const int row = p.row0 + p.lrow(t);
    if (MODE && row < p.T) {
      const long c = (cs * p.T + row) * D + p.lcol();
      st4(reinterpret_cast<float*>(a.xhat) + c, n.xn);
      if ((lane & 15) == 0) a.rstd[cs * p.T + row] = n.rstd;
      if (a.u) st4(reinterpret_cast<float*>(a.u) + c, u);
    }
  }
  lds_barrier();
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    f32x4 x[4];
    operand(x, us + 16 * t * LD, LD, lane);
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      const f32x4 z = product(w1[n], x) + b1[n];
      const int c = 16 * NF * p.wave + 16 * n + 4 * lg;
      f32x4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = gelu_f(z[e]);
      if constexpr (MODE != 1) st4(hs + (16 * t + (lane & 15)) * LDH + c, h);
      if (MODE && p.prow(t) < p.T) {
        const long at = (cs * p.T + p.prow(t)) * F + c;
        f32x4 d;
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = gelu_prime_f(z[e]);
        st4(reinterpret_cast<float*>(a.dact) + at, d);
        if (a.act) st4(reinterpret_cast<float*>(a.act) + at, h);
      }
    }
  }
  if constexpr (MODE != 1) {
    lds_barrier();
    const float* RHS = a.RHS.present() ? a.RHS.at(p.g) : nullptr;
    float* OUT = a.OUT.at(p.g);
#pragma unroll
    for (int t = 0; t < RT; ++t) {                         // OUT = X + h (ybar + m) (+ rhs)
      f32x4 x[4 * NF];
      operand(x, hs + 16 * t * LDH, LDH, lane);
      const f32x4 m = product(w2, x) + b2 + y[t];
      if (p.prow(t) >= p.T) continue;
      const long at = (long)p.prow(t) * D + n0;
      f32x4 r = xin[t] + a.hstep * m;
      if (RHS) {
        const f32x4 rhs = ld4(RHS + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf(a.rhs_sign, r[e], rhs[e]);
      }
      st4(OUT + at, r);
    }
  }
}

template <int RT, int NF>
__global__ void __launch_bounds__(256, 2) chain_f32_adjoint_tail_kernel(const ChainAdjointArgs a, int tiles_m, int total, int per_xcd) {
  constexpr int F = 64 * NF, LDH = F + 4;
  __shared__ __attribute__((aligned(16))) float us[RT * 16 * LD], hs[RT * 16 * LDH];
  const Place<RT> p(a.T, tiles_m, total, per_xcd);
  if (p.none) return;
  const int lane = p.lane, lg = lane >> 4, n0 = 16 * p.wave + 4 * lg;
  const char *pb = a.P.at(p.g), *pt = a.PT.at(p.g);
  const long cs = a.cs.of(p.g), ls = a.loc.of(p.g);
  const float* C = a.c ? reinterpret_cast<const float*>(a.c) + a.c_slots.of(p.g) * p.T * D : a.IN.at(p.g);
  f32x4 cx[RT][4], crow[RT], dg[RT][NF], xh[RT], w2[NF][4], w1[4 * NF], wo[4];
  float rstd[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int row = p.clamp(p.prow(t)), lrow = p.clamp(p.row0 + p.lrow(t));
#pragma unroll
    for (int g = 0; g < 4; ++g) cx[t][g] = ld4(C + (long)row * D + 16 * g + 4 * lg);
#pragma unroll
    for (int n = 0; n < NF; ++n)
      dg[t][n] = ld4(reinterpret_cast<const float*>(a.dact) + (cs * p.T + row) * F + 16 * NF * p.wave + 16 * n + 4 * lg);
    crow[t] = ld4(C + (long)lrow * D + p.lcol());
    xh[t] = ld4(reinterpret_cast<const float*>(a.xhat) + (cs * p.T + lrow) * D + p.lcol());
    rstd[t] = a.rstd[cs * p.T + lrow];
  }
#pragma unroll
  for (int n = 0; n < NF; ++n) weights(w2[n], pt + a.w2_off, 16 * NF * p.wave + 16 * n, D, lane);
  weights(w1, pt + a.w1_off, 16 * p.wave, F, lane);
  weights(wo, pt + a.wo_off, 16 * p.wave, D, lane);
  const f32x4 gamma = ld4(reinterpret_cast<const float*>(pb + a.g_off) + p.lcol());
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (!a.c && a.c_out && p.row0 + p.lrow(t) < p.T)
      st4(reinterpret_cast<float*>(a.c_out) + (ls * p.T + p.row0 + p.lrow(t)) * D + p.lcol(), crow[t]);
#pragma unroll
    for (int n = 0; n < NF; ++n) {                         // dz = (c W2) gelu'(z)
      const f32x4 dz = product(w2[n], cx[t]) * dg[t][n];
      const int c = 16 * NF * p.wave + 16 * n + 4 * lg;
      st4(hs + (16 * t + (lane & 15)) * LDH + c, dz);
      if (a.dz && p.prow(t) < p.T) st4(reinterpret_cast<float*>(a.dz) + (ls * p.T + p.prow(t)) * F + c, dz);
    }
  }
  lds_barrier();
#pragma unroll
  for (int t = 0; t < RT; ++t) {                           // du = dz W1
    f32x4 x[4 * NF];
    operand(x, hs + 16 * t * LDH, LDH, lane);
    st4(us + (16 * t + (lane & 15)) * LD + n0, product(w1, x));
  }
  lds_barrier();
#pragma unroll
  for (int t = 0; t < RT; ++t) {                           // r = LN2^T du, ds = c + r, in place
    float* at = us + p.lrow(t) * LD + p.lcol();
    const f32x4 du = *reinterpret_cast<const f32x4*>(at);
    const f32x4 r = vjp(du, gamma, xh[t], rstd[t]), ds = crow[t] + r;
    st4(at, ds);
    const int row = p.row0 + p.lrow(t);
    if (row < p.T) {
      const long c = (ls * p.T + row) * D + p.lcol();
      st4(a.dx + c, r);
      if (a.du) st4(reinterpret_cast<float*>(a.du) + c, du);
      if (a.ds) st4(reinterpret_cast<float*>(a.ds) + c, ds);
    }
  }
  lds_barrier();
#pragma unroll
  for (int t = 0; t < RT; ++t) {                           // da = ds Wo
    f32x4 x[4];
    operand(x, us + 16 * t * LD, LD, lane);
    const f32x4 da = product(wo, x);
    if (p.prow(t) < p.T) st4(reinterpret_cast<float*>(a.da) + (ls * p.T + p.prow(t)) * D + n0, da);
  }
}

template <int RT>
__global__ void __launch_bounds__(256, 2) chain_f32_adjoint_head_kernel(const ChainAdjointArgs a, int tiles_m, int total, int per_xcd) {
  __shared__ __attribute__((aligned(16))) float us[RT * 16 * LD];
  const Place<RT> p(a.T, tiles_m, total, per_xcd);
  if (p.none) return;
  const int lane = p.lane, lg = lane >> 4, n0 = 16 * p.wave + 4 * lg;
  const char *pb = a.P.at(p.g), *pt = a.PT.at(p.g);
  const long cs = a.cs.of(p.g), ls = a.loc.of(p.g);
  const bool step = a.OUT.present();                       // else the gradients' du alone
  const float* Y = reinterpret_cast<const float*>(a.dqkv) + ls * p.T * 3 * D;
  const float* RHS = step && a.RHS.present() ? a.RHS.at(p.g) : nullptr;
  f32x4 yx[RT][12], w[12], xh[RT], dx[RT], c[RT], rhs[RT];
  float rstd[RT];
  weights(w, pt + a.wqkv_off, 16 * p.wave, 3 * D, lane);
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int row = p.clamp(p.prow(t)), lrow = p.clamp(p.row0 + p.lrow(t));
#pragma unroll
    for (int g = 0; g < 12; ++g) yx[t][g] = ld4(Y + (long)row * 3 * D + 16 * g + 4 * lg);
    if (step) {
      xh[t] = ld4(reinterpret_cast<const float*>(a.xhat) + (cs * p.T + lrow) * D + p.lcol());
      rstd[t] = a.rstd[cs * p.T + lrow];
      dx[t] = ld4(a.dx + (ls * p.T + lrow) * D + p.lcol());
      c[t] = ld4(a.IN.at(p.g) + (long)lrow * D + p.lcol());
      if (RHS) rhs[t] = ld4(RHS + (long)lrow * D + p.lcol());
    }
  }
  const f32x4 gamma = ld4(reinterpret_cast<const float*>(pb + a.g_off) + p.lcol());
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const f32x4 du = product(w, yx[t]);
    st4(us + (16 * t + (lane & 15)) * LD + n0, du);
    if (a.du && p.prow(t) < p.T) st4(reinterpret_cast<float*>(a.du) + (ls * p.T + p.prow(t)) * D + n0, du);
  }
  if (!step) return;
  lds_barrier();
#pragma unroll
  for (int t = 0; t < RT; ++t) {                           // OUT = c + h (dx + LN1^T du) (+ rhs)
    const f32x4 du = *reinterpret_cast<const f32x4*>(us + p.lrow(t) * LD + p.lcol());
    f32x4 r = c[t] + a.hstep * (vjp(du, gamma, xh[t], rstd[t]) + dx[t]);
    if (RHS) {
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf(a.rhs_sign, r[e], rhs[t][e]);
    }
    const int row = p.row0 + p.lrow(t);
    if (row < p.T) {
      st4(a.OUT.at(p.g) + (long)row * D + p.lcol(), r);
      if (a.out_cast) st4(reinterpret_cast<float*>(a.out_cast) + (a.oc_slots.of(p.g) * p.T + row) * D + p.lcol(), r);
    }
  }
}

template <int RT, typename K, typename A> hipError_t launch(K kern, const A& a, hipStream_t st) {
  const int tiles_m = (a.T + 16 * RT - 1) / (16 * RT), total = tiles_m * a.n_groups, per_xcd = (total + 7) / 8;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(256), 0, st, a, tiles_m, total, per_xcd);
  return hipGetLastError();
}
// Two tiles of rows in a block share its weights (147 KB from the L2) where there are blocks enough for all compute units.
bool many(int n_groups, int T) { return (long)n_groups * ((T + 15) / 16) >= 4 * compute_units(); }

template <int RT, int NF> hipError_t tail_of(const ChainTailArgs& a, int mode, hipStream_t st) {
  return mode == 0 ? launch<RT>(chain_f32_tail_kernel<RT, NF, 0>, a, st) : mode == 1 ? launch<RT>(chain_f32_tail_kernel<RT, NF, 1>, a, st)
                                                                        : launch<RT>(chain_f32_tail_kernel<RT, NF, 2>, a, st);
}
template <int RT> hipError_t tail_of(const ChainTailArgs& a, int mode, hipStream_t st) {
  return a.f == 64 ? tail_of<RT, 1>(a, mode, st) : a.f == 128 ? tail_of<RT, 2>(a, mode, st) : tail_of<RT, 4>(a, mode, st);
}
template <int RT> hipError_t adjoint_tail_of(const ChainAdjointArgs& a, hipStream_t st) {
  return a.f == 64 ? launch<RT>(chain_f32_adjoint_tail_kernel<RT, 1>, a, st)
                   : a.f == 128 ? launch<RT>(chain_f32_adjoint_tail_kernel<RT, 2>, a, st) : launch<RT>(chain_f32_adjoint_tail_kernel<RT, 4>, a, st);
}
}  // namespace

hipError_t launch_chain_f32_head(const ChainHeadArgs& a, hipStream_t st) {
  return many(a.n_groups, a.T) ? launch<2>(chain_f32_head_kernel<2>, a, st) : launch<1>(chain_f32_head_kernel<1>, a, st);
}
hipError_t launch_chain_f32_tail(const ChainTailArgs& a, int mode, hipStream_t st) {
  return many(a.n_groups, a.T) ? tail_of<2>(a, mode, st) : tail_of<1>(a, mode, st);
}
hipError_t launch_chain_f32_adjoint_tail(const ChainAdjointArgs& a, hipStream_t st) {
  return many(a.n_groups, a.T) ? adjoint_tail_of<2>(a, st) : adjoint_tail_of<1>(a, st);
}
hipError_t launch_chain_f32_adjoint_head(const ChainAdjointArgs& a, hipStream_t st) {
  return many(a.n_groups, a.T) ? launch<2>(chain_f32_adjoint_head_kernel<2>, a, st) : launch<1>(chain_f32_adjoint_head_kernel<1>, a, st);
}
bool chain_f32_ok(int d, int f) { return d == D && (f == 64 || f == 128 || f == 256); }

}  // namespace mg
