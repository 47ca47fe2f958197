// Shared device-side declarations of the MGRIT hot-path kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mg {

typedef __bf16 bf16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int WAVE = 64;

// ---------------------------------------------------------------------------
// Per-group addressing.  A batched launch works on `n` independent groups
// (coarse intervals).  Everything a group touches is found through device
// pointer tables indexed affinely by the group number, so that one launch can
// serve any sweep of the MGRIT driver without re-uploading pointers:
//   table entry of group g = tab[i0 + g*is]
// Packed intermediate buffers are indexed by "slot" = slot0 + g*slot_s.
// ---------------------------------------------------------------------------
struct Rows {                       // fp32 [T,d] states reached through a table
  const void* const* tab;           // device array of device pointers (may be null)
  int i0, is;
  long off;                         // element offset inside every state (a row range of a stacked state)
  __device__ __forceinline__ float* at(int g) const {
    return (float*)const_cast<void*>(tab[i0 + (long)g * is]) + off;
  }
  __host__ __device__ bool present() const { return tab != nullptr; }
};

struct Params {                     // packed parameter blocks reached through a table
  const void* const* tab;
  int i0, is;
  __device__ __forceinline__ const char* at(int g) const {
    return (const char*)tab[i0 + (long)g * is];
  }
};

struct Slots {
  int s0, ss;
  __host__ __device__ __forceinline__ long of(int g) const { return s0 + (long)g * ss; }
};

// ---------------------------------------------------------------------------
// scalar helpers
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ float to_f(T v);
template <> __device__ __forceinline__ float to_f<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f<bf16>(bf16 v) { return (float)v; }

template <typename T> __device__ __forceinline__ T from_f(float v);
template <> __device__ __forceinline__ float from_f<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f<bf16>(float v) { return (bf16)v; }   // RNE

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ float gelu_f(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752440f));
}
__device__ __forceinline__ float gelu_prime_f(float z) {
  const float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752440f));
  const float pdf = 0.39894228040143267794f * __expf(-0.5f * z * z);
  return cdf + z * pdf;
}

// Fast normal distribution function for the bf16 path: (1 + x P(x^2)) / 2 at x = z / sqrt(2), x P(x^2) the odd
// polynomial for erf fitted by least squares on Chebyshev nodes of |x| <= 2.8 and evaluated at the argument clamped
// to that range (erf(2.8) = 0.99992); absolute error at most 5.13e-5 everywhere (bf16 keeps 8 bits), no
// transcendental instruction.  The vector unit is what the bias+GELU epilogues wait for: the half is folded into the
// coefficients, which is exact, and the clamp is one instruction, 12 per GELU.  Folding 1 / sqrt(2) as well saves one
// more, but rounds differently where the terms cancel at the clamp (error 5.39e-5).
constexpr float SQRT_HALF = 0.70710678118654752440f, PHI_CLAMP = 2.8f;
constexpr float PHI_POLY[8] = {0.5f * -5.83171111e-07f, 0.5f * 2.22840511e-05f, 0.5f * -3.73322994e-04f, 0.5f * 3.65856420e-03f,
                               0.5f * -2.37276428e-02f, 0.5f * 1.09334266e-01f, 0.5f * -3.74316462e-01f, 0.5f * 1.12810103e+00f};
constexpr float PDF_SCALE = 0.39894228040143267794f, PDF_EXP2 = -0.72134752044448170f;   // pdf(z) = 1 / sqrt(2 pi) * 2^(-z^2 log2(e) / 2)
__device__ __forceinline__ float phi_fast(float z) {
  const float x = __builtin_amdgcn_fmed3f(z * SQRT_HALF, -PHI_CLAMP, PHI_CLAMP);
  const float t = x * x;
  float p = PHI_POLY[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) p = fmaf(p, t, PHI_POLY[i]);
  return fmaf(x, p, 0.5f);
}
__device__ __forceinline__ float gelu_fast(float z) { return z * phi_fast(z); }
__device__ __forceinline__ float gelu_prime_fast(float z) {
  const float e = __builtin_amdgcn_exp2f(z * z * PDF_EXP2);   // the bare exponential instruction
  return fmaf(z, PDF_SCALE * e, phi_fast(z));
}
template <typename T> __device__ __forceinline__ float gelu_t(float z);
template <> __device__ __forceinline__ float gelu_t<float>(float z) { return gelu_f(z); }
template <> __device__ __forceinline__ float gelu_t<bf16>(float z) { return gelu_fast(z); }
template <typename T> __device__ __forceinline__ float gelu_prime_t(float z);
template <> __device__ __forceinline__ float gelu_prime_t<float>(float z) { return gelu_prime_f(z); }
template <> __device__ __forceinline__ float gelu_prime_t<bf16>(float z) { return gelu_prime_fast(z); }

// Accesses with the non-temporal hint, for data a kernel touches once.  Only for pointers into
// device global memory (never LDS or scratch): they are issued as global, not flat, instructions,
// which do not count against the counter that LDS reads are waited for on.
template <typename V> __device__ __forceinline__ void st_stream(V* p, V v) {
  typedef __attribute__((address_space(1))) V* gptr;
  __builtin_nontemporal_store(v, (gptr)p);
}
template <typename V> __device__ __forceinline__ V ld_stream(const V* p) {
  typedef const __attribute__((address_space(1))) V* gptr;
  return __builtin_nontemporal_load((gptr)p);
}

// the same without the hint
template <typename V> __device__ __forceinline__ V ld_global(const V* p) {
  typedef const __attribute__((address_space(1))) V* gptr;
  return *(gptr)p;
}

// ---------------------------------------------------------------------------
// Global-to-LDS loads and the order of their tiles
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(1))) const void* gas_ptr;
typedef __attribute__((address_space(3))) void* las_ptr;

// Loads from global memory straight into LDS, 16 bytes per lane: lane l's bytes land at dst + 16*l.  As buffer loads
// (uniform base, 32-bit lane and scalar offsets in bytes): the compiler takes the global_load_lds form for a flat
// access that may touch LDS out of order, and then every wait on an LDS read in the loop waits for all reads in
// flight (lgkmcnt(0)) instead of for the one that is needed.
// The base is the same in every lane; readfirstlane says so where an index division went through vector registers (a
// base that may differ between lanes makes a loop over the lanes out of every load).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t lds_source(const void* base) {
  const unsigned long p = (unsigned long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)((unsigned long)hi << 32 | lo), 0, 0xffffffffu, 0x00020000);
}
template <bool STREAM = false>                             // non-temporal: read once, not to be kept in the caches
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t src, unsigned char* dst, int lane_offset,
                                            int scalar_offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, lane_offset,
                                           scalar_offset, 0, STREAM ? 2 : 0);
}

template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Block barrier that waits for nothing else.  __syncthreads() would first wait for every outstanding
// vector-memory operation of the wavefront, i.e. drain the whole ring of k-tiles in flight.
__device__ __forceinline__ void bare_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------
// Transposed fragments from row-major LDS tiles (ds_read_b64_tr_b16, bf16): in each group of 16 lanes, lane l
// addresses the 8 bytes at columns 4*(l%4).. of row l/4 of a 4 x 16 block and receives column l%16 of its 4 rows.
// The restrict-qualified parameter matters: without it the compiler's wait-count pass takes the read for one that
// may alias the global-to-LDS loads in flight and waits for all of them first, which empties the ring of k-tiles.
// The kernels order the two themselves (counted waits and block barriers).
// ---------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((address_space(3))) unsigned char lds_byte;
struct TrFrag { s16x4 lo, hi; };           // 4 + 4 consecutive reduction indices of this lane's column
__device__ __forceinline__ s16x4 tr_read4(const lds_byte* __restrict__ p) {
  typedef __attribute__((address_space(3))) s16x4* ptr;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr)p);
}
template <int LO, int HI> __device__ __forceinline__ void tr_read(TrFrag& f, const lds_byte* p) {
  f.lo = tr_read4(p + LO);
  f.hi = tr_read4(p + HI);
}
__device__ __forceinline__ void wait_lgkm() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// the fragment as an MFMA operand
__device__ __forceinline__ bf16x8 tr_value(const TrFrag& f) {
  const s16x8 v = {f.lo[0], f.lo[1], f.lo[2], f.lo[3], f.hi[0], f.hi[1], f.hi[2], f.hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// 16 bytes of an LDS tile that global-to-LDS loads fill (restrict: as above)
__device__ __forceinline__ bf16x8 lds_read16(const lds_byte* __restrict__ p) {
  typedef const __attribute__((address_space(3))) bf16x8* ptr;
  return *(ptr)p;
}

// load / store 4 consecutive elements as floats
template <typename T> __device__ __forceinline__ f32x4 load4(const T* p);
template <> __device__ __forceinline__ f32x4 load4<float>(const float* p) {
  return *reinterpret_cast<const f32x4*>(p);
}
template <> __device__ __forceinline__ f32x4 load4<bf16>(const bf16* p) {
  bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
  f32x4 r = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
  return r;
}
template <typename T> __device__ __forceinline__ void store4(T* p, f32x4 v);
template <> __device__ __forceinline__ void store4<float>(float* p, f32x4 v) {
  *reinterpret_cast<f32x4*>(p) = v;
}
template <> __device__ __forceinline__ void store4<bf16>(bf16* p, f32x4 v) {
  bf16x4 r = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
  *reinterpret_cast<bf16x4*>(p) = r;
}

// ---------------------------------------------------------------------------
// Attention grids.
// Which (row block, batch*head, group) a workgroup takes.  Workgroups are dispatched in linear order
// of their index (x fastest), consecutive ones to consecutive XCDs (8, each with an L2 of its own).
// Causal mask: the work of a row block grows (query blocks) or shrinks (key blocks) with its
// position, 4 : 1 between the two ends of a 512-token sequence, so in the natural order some XCDs get
// only heavy blocks.  The linear index is re-read as (rank of the row block, head), heaviest rank
// first: every XCD gets the same mix and the launch ends on its lightest blocks.
// No mask: all blocks are equal; the index is re-read so that the row blocks of one head go to ONE
// XCD one after the other (they run together and share the head's K and V, or Q and dO, in its L2).
struct BlockTask { int tile, bh, g; };
__device__ __forceinline__ BlockTask block_task(bool causal, bool last_tile_heaviest) {
  const int nx = gridDim.x, ny = gridDim.y;
  if (nx == 1) return {0, (int)blockIdx.y, (int)blockIdx.z};
  const int heads = ny * gridDim.z;
  const int lin = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
  int tile, head;
  if (causal) {
    const int rank = lin / heads;
    head = lin - rank * heads;
    tile = last_tile_heaviest ? nx - 1 - rank : rank;
  } else {
    const int whole = (heads >> 3) << 3;                  // heads that fill all 8 XCDs evenly
    if (lin < whole * nx) {
      const int s = lin >> 3, hs = s / nx;
      tile = s - hs * nx;
      head = (hs << 3) + (lin & 7);
    } else {
      const int rem = lin - whole * nx, hs = rem / nx;
      tile = rem - hs * nx;
      head = whole + hs;
    }
  }
  const int g = head / ny;
  return {tile, head - g * ny, g};
}

// ---------------------------------------------------------------------------
// GEMM epilogues:  C[m,n] = sum_k A[m,k] B[n,k]  (+ bias[n]), then
// ---------------------------------------------------------------------------
enum Epi : int {
  EPI_STORE = 0,        // out = acc + bias                               (packed, operand type)
  EPI_GELU = 1,         // out = gelu(acc + bias)
  EPI_RESID_INNER = 2,  // ybar[m,n] (fp32, packed) = [base +] acc + bias      (sum of attention sublayers)
  EPI_RESID_OUTER = 3,  // OUT[m,n] = X + h*(ybar + acc + bias) + rhs          (the Euler update)
  EPI_DGELU = 4,        // out = acc * g[m,n], g = the cached gelu'(z)          (adjoint of the activation)
  EPI_STORE_F32 = 5,    // out (fp32, packed) = hstep * (acc + bias)
  EPI_GELU_PRIME = 6,   // out = gelu'(acc + bias) (operand type): the linearisation cache holds the derivative,
                        // evaluated once per layer
  EPI_GELU_BOTH = 7     // out = gelu(acc + bias) and aux2 = gelu'(acc + bias): a forward step that also leaves its
                        // layer's entry of the linearisation cache
};

struct GemmArgs {
  int n_groups;
  int M, N, K;                 // per group: C is [M,N], reduction length K
  // A operand: packed [slot, M, K] of operand type; a_group_stride = 0 shares A between groups
  const void* A; long a_slot_stride; Slots a_slots;
  // B operand: inside the parameter block (or its transposed copy) at byte offset b_off, [N,K]
  Params B; long b_off;
  long bias_off;               // byte offset of fp32 bias[N] inside the parameter block, -1 = none
  Params bias;
  // outputs / epilogue operands
  void* out; long out_slot_stride; Slots out_slots;      // packed output (operand type or fp32)
  void* aux; long aux_slot_stride; Slots aux_slots;      // EPI_DGELU: g in; EPI_RESID_OUTER: ybar (fp32 packed)
  void* aux2; long aux2_slot_stride; Slots aux2_slots;   // EPI_GELU_BOTH: gelu'(z) out (operand type)
  Rows X;                      // EPI_RESID_OUTER: the step's input state
  const float* base; long base_slot_stride; Slots base_slots;   // EPI_RESID_INNER: optional packed fp32 addend
  Rows OUT;                    // EPI_RESID_OUTER: the step's output state
  Rows RHS;                    // EPI_RESID_OUTER: optional right-hand side
  float hstep;
  float rhs_sign;              // EPI_RESID_OUTER with RHS: OUT = RHS + rhs_sign * (X + h*(..)); +1 the step, -1 the
                               // coarse right-hand side g' = R - Phi'(w) formed in the step that evaluates Phi'
};

// Parameter gradients of one linear map per group, y = u W^T + b, from token-major operands (launch_gemm_tn):
//   dW[m,n] = scale * sum over K tokens of dY[t,m] U[t,n],   db[m] = scale * sum over tokens of dY[t,m]
struct GemmTnArgs {
  int n_groups;
  int M, N, K;                 // out features, in features, tokens
  const void* A; long a_slot_stride; Slots a_slots;      // dY, packed [slot, K, M] of operand type
  const void* B; long b_slot_stride; Slots b_slots;      // U, packed [slot, K, N]
  Params out;                  // the group's gradient block (fp32)
  long w_off, b_off;           // byte offsets of dW and db in it
  float scale;
  float* partial;              // scratch of gemm_tn_partial_floats() (null if that is 0)
};

}  // namespace mg
