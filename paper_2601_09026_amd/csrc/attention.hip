// Fused softmax attention over all (group, sequence, head) triples of a batched layer
// step, forward and backward, without materialising the score matrix in HBM: the kernels for fp32
// operands and for bf16 heads that are not 64 or 128 wide (any d_head <= 128 that is a multiple of 4, any
// sequence length), every product on the 16x16x4 fp32 MFMA.
//
// Every product is D[i][j] = sum_k A[i][k] B[k][j] with the wavefront's own 16 rows (queries; keys in the
// dK/dV pass) on the j axis.  In the MFMA layout lane l holds A[l%16][l/16], B[l/16][l%16] and, in register
// r, D[4*(l/16) + r][l%16].  Consequences:
//   * softmax statistics are private to a lane plus exchanges between lanes 16 and 32 apart;
//   * register r of a score tile already IS the B operand of a k-step of the next product, the one over tile
//     rows 4*(l/16) + r; the A operand of that k-step is one float per lane of the row-major tile;
//   * reductions over features take four k-steps from one 16-byte LDS read (features 16s + 4*(l/16) + e).
// LDS rows of d_head (padded to 16 with zeros) + 4 floats: the 16-byte reads of 16 rows fall on distinct
// slots, and so do the four-row reads of the second kind, so no tile is ever transposed.
//
// Backward (no atomics, deterministic):
//   pass 1, per query row i : D_i = <dO_i, O_i>,  p_ij = exp(s_ij - lse_i),
//                             dA_ij = p_ij (dO_i.V_j - D_i),  dQ_i = scale * sum_j dA_ij K_j
//   pass 2, per key row j   : dV_j = sum_i p_ij dO_i,  dK_j = scale * sum_i dA_ij Q_i
// Sequences of at most 64 rows run both passes in one launch.
//
// What bounds them: the fp32 matrix rate (157 TFLOP/s) on long sequences, launch latency on short ones.
// The form before, one wavefront per row on the vector unit, fetched an operand from LDS for every FMA; whole
// layer steps with it and with this one: 8 layers of 10 bf16 heads of 32, 8 x 512 tokens, forward 2986 -> 372 us,
// transposed 19450 -> 1069; 4 layers of 8 fp32 heads of 64, 4 x 128 tokens, 292 -> 234 and 743 -> 460; of 2 fp32
// heads of 128, 2 x 1024 tokens, 1195 -> 312 and 5855 -> 785; of 4 fp32 heads of 16, 2 x 32 tokens, 116 -> 110 and
// 239 -> 231 (host time included).
#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace mg {

constexpr int AT_TILE = 64;    // rows staged at a time
constexpr int AT_ROWS = 64;    // rows owned by a block: 4 wavefronts x 16

template <typename T> struct Raw4;
template <> struct Raw4<float> { typedef f32x4 type; };
template <> struct Raw4<bf16> { typedef bf16x4 type; };
__device__ __forceinline__ f32x4 widen(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 widen(bf16x4 v) { return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]}; }
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// 64 rows of one operand: fetched into registers while the previous tile is in use, then written to LDS.
// Rows past the end and features past d_head are zeros.
template <typename T, int NC>
struct Tile {
  static constexpr int LD = 16 * NC + 4;
  typename Raw4<T>::type v[NC];
  __device__ __forceinline__ void load(const T* src, long row_stride, int row0, int nrows, int dh) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int item = threadIdx.x + 256 * j, r = row0 + item / (4 * NC), c = item % (4 * NC) * 4;
      v[j] = typename Raw4<T>::type{};
      if (r < nrows && c < dh) v[j] = *reinterpret_cast<const typename Raw4<T>::type*>(src + (long)r * row_stride + c);
    }
  }
  __device__ __forceinline__ void store(float* dst, float scale) const {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int item = threadIdx.x + 256 * j;
      *reinterpret_cast<f32x4*>(dst + item / (4 * NC) * LD + item % (4 * NC) * 4) = scale * widen(v[j]);
    }
  }
};

// one row's features as the B operand of the products over features: 16s + 4*(l/16) + e
template <typename T, int NC>
__device__ __forceinline__ void load_row(f32x4 (&f)[NC], const T* row, int lg, int dh, float scale) {
#pragma unroll
  for (int s = 0; s < NC; ++s) {
    const int c = 16 * s + 4 * lg;
    f[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (c < dh) f[s] = scale * load4<T>(row + c);
  }
}
template <typename T, int NC>
__device__ __forceinline__ void store_row(T* row, const f32x4 (&f)[NC], int lg, int dh, float scale) {
#pragma unroll
  for (int s = 0; s < NC; ++s)
    if (16 * s + 4 * lg < dh) store4<T>(row + 16 * s + 4 * lg, scale * f[s]);
}

// out[t][i][j] = sum over features of tile[16t + i][.] own[j][.] for the 16-row parts t with a set bit
template <int NC>
__device__ __forceinline__ void over_features(f32x4 (&out)[4], const float* tile, const f32x4 (&own)[NC], int lr, int lg,
                                              int parts) {
  constexpr int LD = 16 * NC + 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) out[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float* p = tile + lr * LD + 4 * lg;
  if (parts == 15) {
#pragma unroll
    for (int s = 0; s < NC; ++s) {
      f32x4 x[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = *reinterpret_cast<const f32x4*>(p + 16 * t * LD + 16 * s);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < 4; ++t) out[t] = mfma16(x[t][e], own[s][e], out[t]);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if ((parts >> t) & 1) {
#pragma unroll
        for (int s = 0; s < NC; ++s) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(p + 16 * t * LD + 16 * s);
#pragma unroll
          for (int e = 0; e < 4; ++e) out[t] = mfma16(x[e], own[s][e], out[t]);
        }
      }
  }
}

// out[f][i][j] += sum over tile rows of tile[row][16f + i] w[row][j]
template <int NC>
__device__ __forceinline__ void over_rows(f32x4 (&out)[NC], const float* tile, const f32x4 (&w)[4], int lr, int lg,
                                          int parts) {
  constexpr int LD = 16 * NC + 4;
  const float* p = tile + 4 * lg * LD + lr;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if ((parts >> t) & 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int f = 0; f < NC; ++f) out[f] = mfma16(p[(16 * t + r) * LD + 16 * f], w[t][r], out[f]);
    }
}

__device__ __forceinline__ float lanes_max(float v) {      // over the four lanes that share a column
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float lanes_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

template <typename T> struct Head {
  const T *Q, *K, *V, *O, *dO;
  T *Ow, *dQ, *dK, *dV;
  float *lse, *D;
  long kv_rs;
  __device__ __forceinline__ Head(const AttnArgs& a, int g, int b, int h) {
    const long col = (long)h * a.dh, stat = ((long)b * a.H + h) * a.Sq;
    Q = reinterpret_cast<const T*>(a.q) + a.q_slots.of(g) * a.q_slot_stride + (long)b * a.Sq * a.q_row_stride + col;
    K = reinterpret_cast<const T*>(a.k) + a.k_slots.of(g) * a.k_slot_stride + (long)b * a.Sk * a.k_row_stride + col;
    V = reinterpret_cast<const T*>(a.v) + a.k_slots.of(g) * a.v_slot_stride + (long)b * a.Sk * a.v_row_stride + col;
    Ow = reinterpret_cast<T*>(a.o) + a.o_slots.of(g) * a.o_slot_stride + (long)b * a.Sq * a.o_row_stride + col;
    O = Ow;
    lse = a.lse ? a.lse + a.lse_slots.of(g) * a.lse_slot_stride + stat : nullptr;
    dO = nullptr; dQ = dK = dV = nullptr; D = nullptr; kv_rs = 0;
    if (a.dO) {
      dO = reinterpret_cast<const T*>(a.dO) + a.do_slots.of(g) * a.do_slot_stride + (long)b * a.Sq * a.do_row_stride + col;
      D = a.D + a.D_slots.of(g) * a.D_slot_stride + stat;
      dQ = reinterpret_cast<T*>(a.dq) + a.dqkv_slots.of(g) * a.dqkv_slot_stride + (long)b * a.Sq * a.dqkv_row_stride + col;
      if (a.dk) {
        kv_rs = a.dkv_row_stride ? a.dkv_row_stride : a.dqkv_row_stride;
        const long base = a.dqkv_slots.of(g) * (a.dkv_slot_stride ? a.dkv_slot_stride : a.dqkv_slot_stride) +
                          (long)b * a.Sk * kv_rs + col;
        dK = reinterpret_cast<T*>(a.dk) + base;
        dV = reinterpret_cast<T*>(a.dv) + base;
      }
    }
  }
};

// The 16-row parts of a key tile at k0 that a wavefront's queries see.
__device__ __forceinline__ int key_parts(const AttnArgs& a, int k0, int q_last) {
  const int end = a.causal && q_last + 1 < a.Sk ? q_last + 1 : a.Sk, n = (end - k0 + 15) >> 4;
  return n <= 0 ? 0 : n >= 4 ? 15 : (1 << n) - 1;
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
template <typename T, int NC>
__global__ void __launch_bounds__(256) attn_fwd_f32_kernel(const AttnArgs a) {
  constexpr int LD = 16 * NC + 4;
  __shared__ __attribute__((aligned(16))) float Ks[AT_TILE * LD], Vs[AT_TILE * LD];
  const BlockTask bt = block_task(a.causal, true);
  const int b = bt.bh / a.H, h = bt.bh - b * a.H, dh = a.dh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const Head<T> P(a, bt.g, b, h);
  const int q0 = bt.tile * AT_ROWS, qw = q0 + 16 * wave, qi = qw + lr, qc = qi < a.Sq ? qi : a.Sq - 1;
  Tile<T, NC> tk, tv;
  tk.load(P.K, a.k_row_stride, 0, a.Sk, dh);
  tv.load(P.V, a.v_row_stride, 0, a.Sk, dh);
  f32x4 qf[NC], o[NC];
  load_row<T, NC>(qf, P.Q + (long)qc * a.q_row_stride, lg, dh, rsqrtf((float)dh));
#pragma unroll
  for (int f = 0; f < NC; ++f) o[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int k_end = a.causal ? min(a.Sk, min(q0 + AT_ROWS, a.Sq)) : a.Sk;
  for (int k0 = 0; k0 < k_end; k0 += AT_TILE) {
    __syncthreads();
    tk.store(Ks, 1.f);
    tv.store(Vs, 1.f);
    __syncthreads();
    if (k0 + AT_TILE < k_end) {
      tk.load(P.K, a.k_row_stride, k0 + AT_TILE, a.Sk, dh);
      tv.load(P.V, a.v_row_stride, k0 + AT_TILE, a.Sk, dh);
    }
    const int parts = qw < a.Sq ? key_parts(a, k0, qw + 15) : 0;
    if (parts == 0) continue;                            // wave-uniform
    f32x4 s[4];
    over_features<NC>(s, Ks, qf, lr, lg, parts);
    float mt = -INFINITY;                                // key 0 is valid for every query: finite after tile 0
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = k0 + 16 * t + 4 * lg + r;
        s[t][r] = key < a.Sk && (!a.causal || key <= qi) ? s[t][r] : -INFINITY;
        mt = fmaxf(mt, s[t][r]);
      }
    const float mn = fmaxf(m, lanes_max(mt)), corr = __expf(m - mn);
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[t][r] = __expf(s[t][r] - mn);
        sum += s[t][r];
      }
    l = l * corr + lanes_sum(sum);
    m = mn;
#pragma unroll
    for (int f = 0; f < NC; ++f) o[f] *= corr;
    over_rows<NC>(o, Vs, s, lr, lg, parts);
  }
  if (qi >= a.Sq) return;
  store_row<T, NC>(P.Ow + (long)qi * a.o_row_stride, o, lg, dh, 1.0f / l);
  if (P.lse && lg == 0) P.lse[qi] = m + __logf(l);
}

// ---------------------------------------------------------------------------
// backward pass 1: 64 query rows  ->  D, dQ
// ---------------------------------------------------------------------------
template <typename T, int NC>
__device__ __forceinline__ void dq_block(const AttnArgs& a, const Head<T>& P, float* Ks, float* Vs, int q0) {
  const int dh = a.dh, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const float scale = rsqrtf((float)dh);
  const int qw = q0 + 16 * wave, qi = qw + lr, qc = qi < a.Sq ? qi : a.Sq - 1;
  Tile<T, NC> tk, tv;
  tk.load(P.K, a.k_row_stride, 0, a.Sk, dh);
  tv.load(P.V, a.v_row_stride, 0, a.Sk, dh);
  f32x4 qf[NC], df[NC], dq[NC];
  load_row<T, NC>(qf, P.Q + (long)qc * a.q_row_stride, lg, dh, scale);
  load_row<T, NC>(df, P.dO + (long)qc * a.do_row_stride, lg, dh, 1.f);
  load_row<T, NC>(dq, P.O + (long)qc * a.o_row_stride, lg, dh, 1.f);
  const float lse = P.lse[qc];
  float D = 0.f;
#pragma unroll
  for (int s = 0; s < NC; ++s) {
#pragma unroll
    for (int e = 0; e < 4; ++e) D = fmaf(df[s][e], dq[s][e], D);
    dq[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  D = lanes_sum(D);
  if (qi < a.Sq && lg == 0) P.D[qi] = D;
  const int k_end = a.causal ? min(a.Sk, min(q0 + AT_ROWS, a.Sq)) : a.Sk;
  for (int k0 = 0; k0 < k_end; k0 += AT_TILE) {
    __syncthreads();
    tk.store(Ks, 1.f);
    tv.store(Vs, 1.f);
    __syncthreads();
    if (k0 + AT_TILE < k_end) {
      tk.load(P.K, a.k_row_stride, k0 + AT_TILE, a.Sk, dh);
      tv.load(P.V, a.v_row_stride, k0 + AT_TILE, a.Sk, dh);
    }
    const int parts = qw < a.Sq ? key_parts(a, k0, qw + 15) : 0;
    if (parts == 0) continue;                            // wave-uniform
    f32x4 s[4], dp[4];
    over_features<NC>(s, Ks, qf, lr, lg, parts);
    over_features<NC>(dp, Vs, df, lr, lg, parts);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = k0 + 16 * t + 4 * lg + r;
        const bool valid = key < a.Sk && (!a.causal || key <= qi);
        s[t][r] = valid ? __expf(s[t][r] - lse) * (dp[t][r] - D) : 0.f;     // dA
      }
    over_rows<NC>(dq, Ks, s, lr, lg, parts);
  }
  if (qi < a.Sq) store_row<T, NC>(P.dQ + (long)qi * a.dqkv_row_stride, dq, lg, dh, scale);
}

// ---------------------------------------------------------------------------
// backward pass 2: 64 key rows  ->  dK, dV
// ---------------------------------------------------------------------------
template <typename T, int NC>
__device__ __forceinline__ void dkv_block(const AttnArgs& a, const Head<T>& P, float* Qs, float* dOs, float* Ls,
                                          float* Ds, int j0) {
  const int dh = a.dh, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const float scale = rsqrtf((float)dh);
  const int kw = j0 + 16 * wave, kj = kw + lr, kc = kj < a.Sk ? kj : a.Sk - 1;
  const int i_begin = a.causal ? j0 : 0;                 // key j only sees queries i >= j (j0 is a multiple of 64)
  Tile<T, NC> tq, td;
  tq.load(P.Q, a.q_row_stride, i_begin, a.Sq, dh);
  td.load(P.dO, a.do_row_stride, i_begin, a.Sq, dh);
  f32x4 kf[NC], vf[NC], dk[NC], dv[NC];
  load_row<T, NC>(kf, P.K + (long)kc * a.k_row_stride, lg, dh, 1.f);
  load_row<T, NC>(vf, P.V + (long)kc * a.v_row_stride, lg, dh, 1.f);
#pragma unroll
  for (int f = 0; f < NC; ++f) dk[f] = dv[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = i_begin; i0 < a.Sq; i0 += AT_TILE) {
    __syncthreads();
    tq.store(Qs, scale);
    td.store(dOs, 1.f);
    if (threadIdx.x < AT_TILE) {
      const int qi = i0 + threadIdx.x;
      Ls[threadIdx.x] = qi < a.Sq ? P.lse[qi] : 0.f;
      Ds[threadIdx.x] = qi < a.Sq ? P.D[qi] : 0.f;
    }
    __syncthreads();
    if (i0 + AT_TILE < a.Sq) {
      tq.load(P.Q, a.q_row_stride, i0 + AT_TILE, a.Sq, dh);
      td.load(P.dO, a.do_row_stride, i0 + AT_TILE, a.Sq, dh);
    }
    int parts = 0;                                       // 16-query parts that exist and see the wavefront's keys
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (i0 + 16 * t < a.Sq && (!a.causal || i0 + 16 * t + 15 >= kw)) parts |= 1 << t;
    if (kw >= a.Sk) parts = 0;
    if (parts == 0) continue;                            // wave-uniform
    f32x4 p[4], da[4];
    over_features<NC>(p, Qs, kf, lr, lg, parts);
    over_features<NC>(da, dOs, vf, lr, lg, parts);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4 L = *reinterpret_cast<const f32x4*>(Ls + 16 * t + 4 * lg);
      const f32x4 Dq = *reinterpret_cast<const f32x4*>(Ds + 16 * t + 4 * lg);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qi = i0 + 16 * t + 4 * lg + r;
        const bool valid = qi < a.Sq && (!a.causal || kj <= qi);
        p[t][r] = valid ? __expf(p[t][r] - L[r]) : 0.f;
        da[t][r] = p[t][r] * (da[t][r] - Dq[r]);
      }
    }
    over_rows<NC>(dv, dOs, p, lr, lg, parts);
    over_rows<NC>(dk, Qs, da, lr, lg, parts);            // Qs is pre-scaled: includes 1/sqrt(dh)
  }
  if (kj >= a.Sk) return;
  store_row<T, NC>(P.dK + (long)kj * P.kv_rs, dk, lg, dh, 1.f);
  store_row<T, NC>(P.dV + (long)kj * P.kv_rs, dv, lg, dh, 1.f);
}

// PASS 1: dQ (and D), 2: dK and dV, 3: both, for sequences that fit one block (D is then handed over inside it)
template <typename T, int NC, int PASS>
__global__ void __launch_bounds__(256) attn_bwd_f32_kernel(const AttnArgs a) {
  constexpr int LD = 16 * NC + 4;
  __shared__ __attribute__((aligned(16))) float A[AT_TILE * LD], B[AT_TILE * LD], Ls[AT_TILE], Ds[AT_TILE];
  const BlockTask bt = block_task(a.causal, PASS == 1);
  const int b = bt.bh / a.H, h = bt.bh - b * a.H;
  const Head<T> P(a, bt.g, b, h);
  if constexpr (PASS & 1) dq_block<T, NC>(a, P, A, B, bt.tile * AT_ROWS);
  if constexpr (PASS == 3) __syncthreads();
  if constexpr (PASS & 2) dkv_block<T, NC>(a, P, A, B, Ls, Ds, bt.tile * AT_ROWS);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
bool attn_mfma_supported(const AttnArgs& a);
hipError_t attn_fwd_mfma(const AttnArgs& a, hipStream_t st);
hipError_t attn_bwd_mfma(const AttnArgs& a, hipStream_t st);

static int g_attn_force_simple = 0;
void attn_force_simple(int on) { g_attn_force_simple = on; }

template <typename T, int NC>
static hipError_t attn_fwd_f32(const AttnArgs& a, hipStream_t st) {
  const dim3 grid((a.Sq + AT_ROWS - 1) / AT_ROWS, a.B * a.H, a.n_groups);
  hipLaunchKernelGGL((attn_fwd_f32_kernel<T, NC>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

template <typename T, int NC>
static hipError_t attn_bwd_f32(const AttnArgs& a, hipStream_t st) {
  const dim3 gq((a.Sq + AT_ROWS - 1) / AT_ROWS, a.B * a.H, a.n_groups), gk((a.Sk + AT_ROWS - 1) / AT_ROWS, gq.y, gq.z);
  if (a.dk && gq.x == 1 && gk.x == 1) {
    hipLaunchKernelGGL((attn_bwd_f32_kernel<T, NC, 3>), gq, dim3(256), 0, st, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((attn_bwd_f32_kernel<T, NC, 1>), gq, dim3(256), 0, st, a);
  if (a.dk)                           // dK, dV pass (skipped when only dQ is wanted)
    hipLaunchKernelGGL((attn_bwd_f32_kernel<T, NC, 2>), gk, dim3(256), 0, st, a);
  return hipGetLastError();
}

// NC: d_head in units of 16 features (the last one may be partly zeros; 5 and 7 run as 6 and 8)
template <typename T>
static hipError_t attn_f32(const AttnArgs& a, bool bwd, hipStream_t st) {
  if (a.Sq <= 0 || a.Sk <= 0) return hipErrorInvalidValue;
  switch ((a.dh + 15) / 16) {
    case 1: return bwd ? attn_bwd_f32<T, 1>(a, st) : attn_fwd_f32<T, 1>(a, st);
    case 2: return bwd ? attn_bwd_f32<T, 2>(a, st) : attn_fwd_f32<T, 2>(a, st);
    case 3: return bwd ? attn_bwd_f32<T, 3>(a, st) : attn_fwd_f32<T, 3>(a, st);
    case 4: return bwd ? attn_bwd_f32<T, 4>(a, st) : attn_fwd_f32<T, 4>(a, st);
    case 5: case 6: return bwd ? attn_bwd_f32<T, 6>(a, st) : attn_fwd_f32<T, 6>(a, st);
    default: return bwd ? attn_bwd_f32<T, 8>(a, st) : attn_fwd_f32<T, 8>(a, st);
  }
}

hipError_t launch_attn_fwd(const AttnArgs& a, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0) return hipSuccess;
  if (a.dh > 128 || (a.dh & 3)) return hipErrorInvalidValue;
  const double heads = (double)a.n_groups * a.B * a.H, esz = is_bf16 ? 2 : 4;
  const double pairs = a.causal ? 0.5 * a.Sq * (a.Sk + 1.0) : (double)a.Sq * a.Sk;   // unmasked scores
  ProfScope ps(PC_ATTN_FWD, heads * pairs * a.dh * 4.0, heads * (2.0 * a.Sq + 2.0 * a.Sk) * a.dh * esz, st);
  if (is_bf16 && !g_attn_force_simple && attn_mfma_supported(a)) return attn_fwd_mfma(a, st);
  return is_bf16 ? attn_f32<bf16>(a, false, st) : attn_f32<float>(a, false, st);
}

hipError_t launch_attn_bwd(const AttnArgs& a, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0) return hipSuccess;
  if (a.dh > 128 || (a.dh & 3)) return hipErrorInvalidValue;
  const double heads = (double)a.n_groups * a.B * a.H, esz = is_bf16 ? 2 : 4;
  const double pairs = a.causal ? 0.5 * a.Sq * (a.Sk + 1.0) : (double)a.Sq * a.Sk;
  // recompute scores + dP, dV, dQ, dK: five contractions over the unmasked pairs
  ProfScope ps(PC_ATTN_BWD, heads * pairs * a.dh * 10.0, heads * (4.0 * a.Sq + 4.0 * a.Sk) * a.dh * esz, st);
  if (is_bf16 && !g_attn_force_simple && attn_mfma_supported(a)) return attn_bwd_mfma(a, st);
  return is_bf16 ? attn_f32<bf16>(a, true, st) : attn_f32<float>(a, true, st);
}

}  // namespace mg
