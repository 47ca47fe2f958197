// Interval-batched grouped GEMM  C_g[m,n] = sum_k A_g[m,k] * W_g[n,k]  with fused
// epilogues, one launch for all groups of an F-/C-relaxation sweep; every group has
// its own weight matrix (the layer of its coarse interval), found through the
// parameter pointer table.
//
// The kernels:
//  * gemm_mfma    : bf16 operands, fp32 accumulate on the 32x32x16 MFMA of gfx950; operands
//                   stream global -> LDS directly through a ring of k-tiles, see below.
//  * gemm_mfma_dgelu_walk: the same with resident blocks that walk over the tiles of a multiply-by-GELU' launch.
//  * gemm_tn_mfma, gemm_tn_f32: token-major products of the parameter gradients.
//  * gemm_f32_mfma: fp32 operands on the 32x32x2 fp32 MFMA; gemm_f32_small: small and ragged launches on the 16x16x4.
//  * gemm_simple  : any operand type and shape, LDS-tiled FMA.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "lds_limit.h"
#include "prof.h"

namespace mg {

// ---------------------------------------------------------------------------
// Epilogue.  EpiPtrs holds the launch's epilogue operands resolved for one group; apply4
// finishes 4 consecutive columns n..n+3 of row m (idx = m*N + n) from the accumulated
// products `acc` (bias not yet added).
// ---------------------------------------------------------------------------
struct EpiPtrs {
  const float* bias;          // [N] or null
  void* out;                  // packed output (operand type or fp32)
  void* aux;                  // EPI_DGELU: gelu'(z) in; EPI_RESID_OUTER: ybar
  void* aux2;                 // EPI_GELU_BOTH: gelu'(z) out
  const float* base;          // EPI_RESID_INNER: optional addend
  const float* X;             // EPI_RESID_OUTER
  const float* RHS;           // EPI_RESID_OUTER, optional
  float* OUT;                 // EPI_RESID_OUTER
};

template <typename TO>
__device__ __forceinline__ EpiPtrs resolve_epi(const GemmArgs& a, int g, int epi) {
  EpiPtrs p;
  p.bias = a.bias_off >= 0 ? reinterpret_cast<const float*>(a.bias.at(g) + a.bias_off) : nullptr;
  const bool f32_out = epi == EPI_STORE_F32 || epi == EPI_RESID_INNER;
  const long osz = f32_out ? 4 : (long)sizeof(TO);
  p.out = a.out ? static_cast<char*>(a.out) + a.out_slots.of(g) * a.out_slot_stride * osz : nullptr;
  const long asz = epi == EPI_RESID_OUTER ? 4 : (long)sizeof(TO);
  p.aux = a.aux ? static_cast<char*>(a.aux) + a.aux_slots.of(g) * a.aux_slot_stride * asz : nullptr;
  p.aux2 = a.aux2 ? static_cast<char*>(a.aux2) + a.aux2_slots.of(g) * a.aux2_slot_stride * (long)sizeof(TO) : nullptr;
  p.base = a.base ? a.base + a.base_slots.of(g) * a.base_slot_stride : nullptr;
  p.X = a.X.present() ? a.X.at(g) : nullptr;
  p.RHS = a.RHS.present() ? a.RHS.at(g) : nullptr;
  p.OUT = a.OUT.present() ? a.OUT.at(g) : nullptr;
  return p;
}

// Epilogue operands and outputs are touched once per launch: they are moved with the
// non-temporal hint, so that they do not displace the operand panels that the tiles running
// on an XCD share through its L2.
template <typename T> __device__ __forceinline__ void estore4(T* p, f32x4 v);
template <> __device__ __forceinline__ void estore4<float>(float* p, f32x4 v) { st_stream(reinterpret_cast<f32x4*>(p), v); }
template <> __device__ __forceinline__ void estore4<bf16>(bf16* p, f32x4 v) {
  bf16x4 r = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
  st_stream(reinterpret_cast<bf16x4*>(p), r);
}
template <typename T> __device__ __forceinline__ f32x4 eload4(const T* p);
template <> __device__ __forceinline__ f32x4 eload4<float>(const float* p) { return ld_stream(reinterpret_cast<const f32x4*>(p)); }
template <> __device__ __forceinline__ f32x4 eload4<bf16>(const bf16* p) {
  bf16x4 v = ld_stream(reinterpret_cast<const bf16x4*>(p));
  f32x4 r = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
  return r;
}

// OPT: what is known at compile time about the optional operands of an epilogue: -1 nothing (tested
// per call), else bit 0 = the first one is there (ybar / base), bit 1 =
// RHS is there.  With OPT >= 0 a run of items is straight-line code.
template <int OPT> __device__ __forceinline__ bool has_opt(int bit, const void* p) {
  return OPT < 0 ? p != nullptr : ((OPT >> bit) & 1) != 0;
}

template <int EPI, typename TO, int OPT = -1>
__device__ __forceinline__ void apply4(TO* __restrict__ out_op, float* __restrict__ out_f32,
                                       const TO* __restrict__ z_in, TO* __restrict__ g_out,
                                       const float* __restrict__ base, const float* __restrict__ X,
                                       const float* __restrict__ ybar, const float* __restrict__ RHS,
                                       float* __restrict__ OUT, float hstep, float sgn, long idx, f32x4 acc) {
  if constexpr (EPI == EPI_STORE) {
    estore4<TO>(out_op + idx, acc);
  } else if constexpr (EPI == EPI_STORE_F32) {
    estore4<float>(out_f32 + idx, hstep * acc);
  } else if constexpr (EPI == EPI_GELU) {
    f32x4 y = {gelu_t<TO>(acc[0]), gelu_t<TO>(acc[1]), gelu_t<TO>(acc[2]), gelu_t<TO>(acc[3])};
    estore4<TO>(out_op + idx, y);
  } else if constexpr (EPI == EPI_GELU_PRIME) {
    f32x4 y = {gelu_prime_t<TO>(acc[0]), gelu_prime_t<TO>(acc[1]), gelu_prime_t<TO>(acc[2]),
               gelu_prime_t<TO>(acc[3])};
    estore4<TO>(out_op + idx, y);
  } else if constexpr (EPI == EPI_GELU_BOTH) {
    f32x4 y = {gelu_t<TO>(acc[0]), gelu_t<TO>(acc[1]), gelu_t<TO>(acc[2]), gelu_t<TO>(acc[3])};
    estore4<TO>(out_op + idx, y);
    f32x4 dy = {gelu_prime_t<TO>(acc[0]), gelu_prime_t<TO>(acc[1]), gelu_prime_t<TO>(acc[2]),
                gelu_prime_t<TO>(acc[3])};
    estore4<TO>(g_out + idx, dy);
  } else if constexpr (EPI == EPI_DGELU) {
    estore4<TO>(out_op + idx, acc * eload4<TO>(z_in + idx));
  } else if constexpr (EPI == EPI_RESID_INNER) {
    if (has_opt<OPT>(0, base)) acc += eload4<float>(base + idx);
    estore4<float>(out_f32 + idx, acc);
  } else if constexpr (EPI == EPI_RESID_OUTER) {
    f32x4 x = eload4<float>(X + idx);
    if (has_opt<OPT>(0, ybar)) acc += eload4<float>(ybar + idx);
    f32x4 r = x + hstep * acc;
    if (has_opt<OPT>(1, RHS)) {
      // sgn = 1: r + rhs; sgn = -1: rhs - r, each a single rounding of the exact value
      const f32x4 rhs = eload4<float>(RHS + idx);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf(sgn, r[e], rhs[e]);
    }
    estore4<float>(OUT + idx, r);
  }
}

// 8 consecutive columns of a bf16 output (the epilogues whose operands are all bf16)
__device__ __forceinline__ void store8(bf16* p, f32x4 a, f32x4 b) {
  bf16x8 r = {(bf16)a[0], (bf16)a[1], (bf16)a[2], (bf16)a[3], (bf16)b[0], (bf16)b[1], (bf16)b[2], (bf16)b[3]};
  st_stream(reinterpret_cast<bf16x8*>(p), r);
}
template <int EPI>
__device__ __forceinline__ void apply8(bf16* __restrict__ out, const bf16* __restrict__ z_in,
                                       bf16* __restrict__ g_out, long idx,
                                       f32x4 a, f32x4 b) {
  if constexpr (EPI == EPI_STORE) {
    store8(out + idx, a, b);
  } else if constexpr (EPI == EPI_GELU) {
#pragma unroll
    for (int r = 0; r < 4; ++r) { a[r] = gelu_fast(a[r]); b[r] = gelu_fast(b[r]); }
    store8(out + idx, a, b);
  } else if constexpr (EPI == EPI_GELU_PRIME) {
#pragma unroll
    for (int r = 0; r < 4; ++r) { a[r] = gelu_prime_fast(a[r]); b[r] = gelu_prime_fast(b[r]); }
    store8(out + idx, a, b);
  } else if constexpr (EPI == EPI_GELU_BOTH) {
    f32x4 da, db;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      da[r] = gelu_prime_fast(a[r]); db[r] = gelu_prime_fast(b[r]);
      a[r] = gelu_fast(a[r]); b[r] = gelu_fast(b[r]);
    }
    store8(out + idx, a, b);
    store8(g_out + idx, da, db);
  } else if constexpr (EPI == EPI_DGELU) {
    const bf16x8 g = ld_stream(reinterpret_cast<const bf16x8*>(z_in + idx));
#pragma unroll
    for (int r = 0; r < 4; ++r) { a[r] *= (float)g[r]; b[r] *= (float)g[4 + r]; }
    store8(out + idx, a, b);
  }
}

// one-off form for the generic kernel
template <int EPI, typename TO>
__device__ __forceinline__ void epilogue4(const EpiPtrs& p, float hstep, float sgn, int N, int m, int n, f32x4 acc) {
  if (p.bias) acc += *reinterpret_cast<const f32x4*>(p.bias + n);
  apply4<EPI, TO>(static_cast<TO*>(p.out), static_cast<float*>(p.out), static_cast<const TO*>(p.aux),
                  static_cast<TO*>(p.aux2), p.base, p.X,
                  static_cast<const float*>(p.aux), p.RHS, p.OUT, hstep, sgn, (long)m * N + n, acc);
}

constexpr int ce_gcd(int a, int b) { return b == 0 ? a : ce_gcd(b, a % b); }

// Whole-tile epilogue of one wavefront of the MFMA kernel.  All operand pointers are
// restrict-qualified parameters of this one function, so that the compiler may hoist the
// loads of later rows above the stores of earlier ones (outputs never alias inputs).
template <int EPI, typename TO, int TM, int TN, bool STAGED, bool RAGGED>
__device__ __forceinline__ void tile_epilogue(
    f32x16 (&acc)[TM][TN], unsigned char* ep, const float* __restrict__ bias, TO* __restrict__ out_op,
    float* __restrict__ out_f32, const TO* __restrict__ z_in, TO* __restrict__ g_out,
    const float* __restrict__ base, const float* __restrict__ X, const float* __restrict__ ybar,
    const float* __restrict__ RHS, float* __restrict__ OUT, float hstep, float sgn, int N, int M, int mrow0,
    int ncol0, int lane) {
  constexpr int WTN = TN * 32;
  const int lr = lane & 31, lh = lane >> 5;
  if constexpr (STAGED) {
    constexpr int EP_LD = WTN * 4 + 16;                  // bytes per staged row (padded)
    // A lane finishes CW consecutive columns at a time: 8 where the output is bf16 (16-byte
    // stores: four lanes fill a 64-byte sector, so the memory side never has to read a sector
    // back in order to merge a partial write), 4 where it is fp32.
    constexpr bool WIDE = sizeof(TO) == 2 && (EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_DGELU ||
                                              EPI == EPI_GELU_PRIME || EPI == EPI_GELU_BOTH);
    constexpr int CW = WIDE ? 8 : 4;
    constexpr int CI = WTN / CW;                         // items per row
    constexpr int NIT = 32 * CI / 64;                    // items per lane in a 32-row block
    static_assert(32 * CI % 64 == 0, "whole passes over a 32-row block");
    // item e = it*64 + lane is column group e % CI of row e / CI.  A lane's column group
    // repeats with period NB in `it` (1 when CI divides 64): one bias vector per phase.
    constexpr int NB = CI / ce_gcd(64, CI);
    f32x4 bv[NB][CW / 4];
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
      for (int h = 0; h < CW / 4; ++h) {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        int n = ncol0 + CW * ((p * 64 + lane) % CI) + 4 * h;
        if (RAGGED) n = n < N ? n : 0;
        bv[p][h] = bias ? ld_global(reinterpret_cast<const f32x4*>(bias + n)) : z;
      }
    // The bias vectors have landed before the first item uses them; saying so once, outside the
    // row guards below, keeps the per-item waits on them from also waiting for every earlier
    // store (stores count on the same counter), which would serialise the stores of a tile.
    if (bias) __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0)
    // GUARD: the wavefront's tile reaches past row M (ragged last tile of a group): per-row tests.
    // Otherwise the items of a 32-row block are straight-line code, whose operand loads the
    // compiler may issue ahead of the stores of earlier items (outputs never alias inputs).
    auto rows32 = [&](auto guard_tag, auto opt_tag, int i) {
      constexpr bool GUARD = decltype(guard_tag)::value;
      constexpr int OPT = decltype(opt_tag)::value;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *reinterpret_cast<f32x4*>(ep + lr * EP_LD + (32 * j + 8 * q + 4 * lh) * 4) = v;
        }
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int e = it * 64 + lane;
        const int row = e / CI, ci = e % CI;
        const unsigned char* src = ep + row * EP_LD + ci * CW * 4;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(src) + bv[it % NB][0];
        const int m = mrow0 + 32 * i + row;
        const int n = ncol0 + CW * ci;
        const long idx = (long)m * N + n;
        const bool inside = !GUARD || (m < M && (!RAGGED || n < N));   // N is a multiple of 8
        if constexpr (WIDE) {
          const f32x4 v1 = *reinterpret_cast<const f32x4*>(src + 16) + bv[it % NB][1];
          if (inside)
            apply8<EPI>(reinterpret_cast<bf16*>(out_op), reinterpret_cast<const bf16*>(z_in),
                        reinterpret_cast<bf16*>(g_out), idx, v0, v1);
        } else {
          if (inside)
            apply4<EPI, TO, OPT>(out_op, out_f32, z_in, g_out, base, X, ybar, RHS, OUT, hstep, sgn, idx, v0);
        }
      }
    };
    // which optional operands this launch has (uniform over the launch): resolved once, so that
    // the items carry no tests of their own
    constexpr int NOPT = EPI == EPI_RESID_OUTER ? 4 : EPI == EPI_RESID_INNER ? 2 : 1;
    const void* first = EPI == EPI_RESID_OUTER ? static_cast<const void*>(ybar) : static_cast<const void*>(base);
    const int opt = NOPT == 1 ? 0 : ((first ? 1 : 0) | (NOPT == 4 && RHS ? 2 : 0));
    auto all_rows = [&](auto guard_tag, auto opt_tag) {
#pragma unroll
      for (int i = 0; i < TM; ++i) rows32(guard_tag, opt_tag, i);
    };
    if (mrow0 + 32 * TM <= M && (!RAGGED || ncol0 + WTN <= N)) {   // wave-uniform
      if (opt == 0) all_rows(std::false_type{}, std::integral_constant<int, 0>{});
      else if (opt == 1) all_rows(std::false_type{}, std::integral_constant<int, NOPT >= 2 ? 1 : 0>{});
      else if (opt == 2) all_rows(std::false_type{}, std::integral_constant<int, NOPT == 4 ? 2 : 0>{});
      else all_rows(std::false_type{}, std::integral_constant<int, NOPT == 4 ? 3 : 0>{});
    } else {
      all_rows(std::true_type{}, std::integral_constant<int, -1>{});
    }
  } else {
    // acc[i][j] register 4q+r of lane l  =  C[m = 32i + l%32][n = 32j + 8q + 4*(l/32) + r]
    f32x4 bv[TN][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
        bv[j][q] = bias ? *reinterpret_cast<const f32x4*>(bias + ncol0 + j * 32 + q * 8 + lh * 4) : z;
      }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = mrow0 + i * 32 + lr;
      if (m < M) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = ncol0 + j * 32 + q * 8 + lh * 4;
            f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            apply4<EPI, TO>(out_op, out_f32, z_in, g_out, base, X, ybar, RHS, OUT, hstep, sgn,
                            (long)m * N + n, v + bv[j][q]);
          }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// MFMA kernel.  WM x WN wavefronts, each owning a (BM/WM) x (BN/WN) tile of the output.
//  * Operands go from global memory straight into LDS (buffer loads, 16 bytes per lane, no register
//    staging; the ragged form, whose zero chunk needs an address per lane, as global_load_lds) through a
//    ring of STAGES k-tiles of depth BK.  The buffer form lets the compiler wait for the fragment it needs
//    instead of for all LDS reads in flight and takes the address arithmetic off the vector unit: with 5
//    layers of 4096 rows 768 -> 2304 82 -> 78 us, 768 -> 3072 with GELU 116 -> 108, 3072 -> 768 84 -> 78;
//    one layer 27 -> 23, 36.5 -> 33.
//  * An LDS row holds the BK bf16 of one matrix row unpadded; its 16-byte chunks are XOR-swizzled by
//    the row number so that the 16-byte fragment reads of 32 consecutive rows are bank-conflict free.
//    A load instruction of a wavefront fills 1 KB = 8 consecutive rows; the lane that will
//    land at position p of row r fetches logical chunk p ^ f(r) of that row.
//  * MFMA fragments are double-buffered in registers: the LDS reads of k-step s+1 are spread between
//    the MFMAs of s, across the boundary of two k-tiles as well, and so are the loads that refill a stage.
//  * The barriers are bare: loads stay in flight across them, and each tile is waited for by count.
//    (__syncthreads() drains every outstanding load first, so that a deeper ring gains nothing: with it a
//    4096 x 768 product of reduction 3072 took 49 us with two, three or four stages of 128x128x64 tiles;
//    with counted waits 45, 41 and 38 us.)
//  * The weight fragment is the first MFMA operand: a lane then holds 4 consecutive output
//    columns per register quad.
//  * Epilogue: each wavefront transposes 32 rows at a time through a private padded LDS region and
//    walks them row-major, so every global access of the epilogue covers whole contiguous rows.
//  * RAGGED: N no multiple of BN or K no multiple of BK (both multiples of 8): weight rows are clamped,
//    columns guarded, and the chunks of the last k-tile that lie past K come from a zero chunk.
// What bounds it: large launches the matrix cores and then the epilogue, which moves 4 to 16 bytes per output
// element with the matrix cores idle (in the step at the GPT-2 shape they are busy for 55 % of a 256x256 launch
// with the plain store and for 37-46 % with the other epilogues: profiles/gpt2_small_fwd_adjoint_pmc_summary.txt);
// launches of up to one tile per CU the latency of first touches past the L2, which the deep ring covers.
// ---------------------------------------------------------------------------
// LDS has 64 four-byte banks (256 bytes per clock); a 16-byte read is served 16 lanes at a
// time, so 16 consecutive rows must land on 16 distinct 16-byte slots modulo 256 bytes.  Two of the
// 128-byte rows share a 256-byte bank row: swizzle by the row pair.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// Source of the chunks of a last k-tile that lie past K.
__device__ const __attribute__((aligned(16))) unsigned char g_zero_chunk[16] = {};

template <int BM, int BN, int BK, int STAGES, int OCC, bool RAGGED, int EPI, typename TO, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN, OCC * WM * WN / 4)
gemm_mfma_kernel(const GemmArgs a, int tiles_m, int tiles_n, int total_tiles, int per_xcd, int pm, int pn) {
  constexpr int NW = WM * WN;                            // wavefronts per block
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int RB = BK * 2;                             // bytes per LDS row
  constexpr int CPR = RB / 16;                           // 16-byte chunks per row
  constexpr int RPL = 1024 / RB;                         // rows per load instruction
  constexpr int KS = BK / 16;                            // MFMA k-steps per tile
  constexpr int A_BYTES = BM * RB, B_BYTES = BN * RB, STAGE = A_BYTES + B_BYTES;
  constexpr int A_LD = BM / RPL / NW, B_LD = BN / RPL / NW; // load instructions per wave per k-tile
  static_assert(BK == 64 && STAGES <= 4, "swz(), wait_tile()");
  static_assert(A_LD >= 1 && B_LD >= 1 && A_LD * RPL * NW == BM && B_LD * RPL * NW == BN, "tile/wave split");
  constexpr int PER_TILE = A_LD + B_LD;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem2[];

  // XCD-aware tile order: workgroup ids are dealt round-robin to the 8 XCDs, so give each
  // XCD one contiguous range of tiles.  Inside a group's tile grid the order runs over
  // pm x pn patches (pn = 0: plain row-major): the tiles an XCD runs at the same time then
  // share pm activation row panels and a pn-tile-wide slice of the weight matrix, which fit
  // that XCD's L2 together, and successive patches keep the row panels.
  const int pid = blockIdx.x;
  const int tile = (pid & 7) * per_xcd + (pid >> 3);
  if (tile >= total_tiles) return;
  const int tiles_per_group = tiles_m * tiles_n;
  const int g = __builtin_amdgcn_readfirstlane(tile / tiles_per_group);   // (the divisions go through vector registers)
  const int tg = tile - g * tiles_per_group;
  int tm, tn;
  if (pn > 0) {
    const int patch = pm * pn, patches_n = tiles_n / pn;
    const int b = tg / patch, w = tg - b * patch;
    const int bm = b / patches_n, bn = b - bm * patches_n;
    tm = bm * pm + w / pn;
    tn = bn * pn + w % pn;
  } else {
    tm = tg / tiles_n;
    tn = tg - tm * tiles_n;
  }
  const int m0 = __builtin_amdgcn_readfirstlane(tm) * BM, n0 = __builtin_amdgcn_readfirstlane(tn) * BN;

  const bf16* A = reinterpret_cast<const bf16*>(a.A) + a.a_slots.of(g) * a.a_slot_stride;
  const char* pblock = a.B.at(g);
  const bf16* B = reinterpret_cast<const bf16*>(pblock + a.b_off);
  const int K = a.K, M = a.M, N = a.N;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lr = lane & 31, lh = lane >> 5;
  const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;

  // global -> LDS: this lane's byte offsets from the tile's first rows (row clamped at the ragged tail of M)
  const int lrow = lane / CPR, lpos = lane % CPR;
  const char* Am = reinterpret_cast<const char*>(A + (long)m0 * K);
  const char* Bn = reinterpret_cast<const char*>(B + (long)n0 * K);
  const auto srcA = lds_source(Am), srcB = lds_source(Bn);
  int aoff[A_LD], boff[B_LD];
#pragma unroll
  for (int j = 0; j < A_LD; ++j) {
    const int row = (wave * A_LD + j) * RPL + lrow;            // row inside the tile
    aoff[j] = ((row < M - m0 ? row : M - 1 - m0) * K + (lpos ^ swz(row)) * 8) * 2;
  }
#pragma unroll
  for (int j = 0; j < B_LD; ++j) {
    const int row = (wave * B_LD + j) * RPL + lrow;
    boff[j] = ((RAGGED && row >= N - n0 ? N - 1 - n0 : row) * K + (lpos ^ swz(row)) * 8) * 2;
  }

  auto issue_one = [&](int stage, int k0, int idx) {
    unsigned char* sa = smem2 + stage * STAGE;
    const bool is_a = idx < A_LD;
    const int off = is_a ? aoff[idx < A_LD ? idx : 0] : boff[idx < A_LD ? 0 : idx - A_LD];
    unsigned char* dst = is_a ? sa + (wave * A_LD + idx) * 1024 : sa + A_BYTES + (wave * B_LD + idx - A_LD) * 1024;
    if constexpr (RAGGED) {
      // the last k-tile reaches past K: its 16-byte chunks from K on are zeros (K is a multiple of 8)
      const int row = is_a ? (wave * A_LD + idx) * RPL + lrow : (wave * B_LD + idx - A_LD) * RPL + lrow;
      const char* src = (is_a ? Am : Bn) + off + 2 * (long)k0;
      if (k0 + (lpos ^ swz(row)) * 8 >= K) src = reinterpret_cast<const char*>(g_zero_chunk);
      __builtin_amdgcn_global_load_lds((gas_ptr)src, (las_ptr)dst, 16, 0, 0);
    } else {
      load_to_lds(is_a ? srcA : srcB, dst, off, 2 * k0);
    }
  };
  auto issue = [&](int stage, int k0) {
#pragma unroll
    for (int idx = 0; idx < PER_TILE; ++idx) issue_one(stage, k0, idx);
  };

  // fragment byte offsets inside a tile region: row lr, swizzled chunk of k-step ks
  int foff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) foff[ks] = lr * RB + (((2 * ks + lh) ^ swz(lr)) << 4);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Ring: tile kt lives in stage kt % STAGES.  The fragments of the first k-step of tile kt+1 are read
  // during the last k-step of tile kt, so that step begins by making sure tile kt+1 has landed (own loads:
  // vmcnt, the others': barrier); from that barrier on nobody reads tile kt any more (its last fragments
  // are in registers), and its stage is refilled with tile kt+STAGES.
  const int KT = RAGGED ? (K + BK - 1) / BK : K / BK;
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < KT) issue(s, s * BK);
  auto wait_tile = [&](int kt, int issued) {               // own loads of tile kt have landed (issued: tiles so far)
    const int behind = issued - 1 - kt;
    if constexpr (STAGES >= 4) if (behind >= 3) { wait_vmcnt<3 * PER_TILE>(); return; }
    if constexpr (STAGES >= 3) if (behind >= 2) { wait_vmcnt<2 * PER_TILE>(); return; }
    if (behind >= 1) { wait_vmcnt<PER_TILE>(); return; }
    wait_vmcnt<0>();
  };
  const lds_byte* lds0 = (const lds_byte*)smem2;
  bf16x8 fa[2][TM], fb[2][TN];
  wait_tile(0, STAGES < KT ? STAGES : KT);
  bare_barrier();
#pragma unroll
  for (int j = 0; j < TN; ++j) fb[0][j] = lds_read16(lds0 + A_BYTES + (wn0 + j * 32) * RB + foff[0]);
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[0][i] = lds_read16(lds0 + (wm0 + i * 32) * RB + foff[0]);
  int cur = 0;
  auto tile_step = [&](int kt, auto loads_tag) {
    constexpr bool LOADS = decltype(loads_tag)::value;     // tile kt + STAGES exists
    const int nxt = cur + 1 == STAGES ? 0 : cur + 1;
    const int pk0 = (kt + STAGES) * BK;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int cb = ks & 1, nb = cb ^ 1;
      const bool last = ks == KS - 1;
      if (last) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr (LOADS) wait_vmcnt<(STAGES - 2) * PER_TILE>();
        else wait_tile(kt + 1, KT);
        bare_barrier();
      }
      const int rst = last ? nxt : cur, rks = last ? 0 : ks + 1;
      const lds_byte* sA = lds0 + rst * STAGE + wm0 * RB;
      const lds_byte* sB = lds0 + rst * STAGE + A_BYTES + wn0 * RB;
      // The fragment reads of the next k-step and the loads of the refilled stage are spread between
      // the matrix instructions, fenced so that the scheduler keeps them apart: a wavefront that has to
      // wait for its turn at the LDS or the load unit has matrix work queued meanwhile.
      constexpr int NM = TM * TN, RD = TM + TN;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int i = q / TN, j = q % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cb][j], fa[cb][i], acc[i][j], 0, 0, 0);
        const int r0 = (q * RD * 4 / 3 + NM - 1) / NM, r1 = ((q + 1) * RD * 4 / 3 + NM - 1) / NM;
#pragma unroll
        for (int u = 0; u < RD; ++u)
          if (u >= r0 && (u < r1 || q == NM - 1)) {
            if (u < TN) fb[nb][u] = lds_read16(sB + u * 32 * RB + foff[rks]);
            else fa[nb][u - TN] = lds_read16(sA + (u - TN) * 32 * RB + foff[rks]);
          }
        if (LOADS && last) {
          const int l0 = (q * PER_TILE + NM - 1) / NM, l1 = ((q + 1) * PER_TILE + NM - 1) / NM;
#pragma unroll
          for (int u = 0; u < PER_TILE; ++u)
            if (u >= l0 && u < l1) issue_one(cur, pk0, u);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    cur = nxt;
  };
  int kt = 0;
  for (; kt + STAGES < KT; ++kt) tile_step(kt, std::true_type{});
  for (; kt < KT; ++kt) tile_step(kt, std::false_type{});
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // (the reads ahead of a tile that does not exist)
  bare_barrier();

  // the staging regions reuse the (now idle) k-tile ring; the launcher sizes LDS for both
  constexpr int EP_BYTES = (32 * (WTN * 4 + 16) + 1023) / 1024 * 1024;
  const EpiPtrs P = resolve_epi<TO>(a, g, EPI);
  tile_epilogue<EPI, TO, TM, TN, true, RAGGED>(acc, smem2 + wave * EP_BYTES, P.bias, static_cast<TO*>(P.out),
                                         static_cast<float*>(P.out), static_cast<const TO*>(P.aux),
                                         static_cast<TO*>(P.aux2), P.base, P.X,
                                         static_cast<const float*>(P.aux), P.RHS, P.OUT, a.hstep, a.rhs_sign, a.N,
                                         M, m0 + wm0, n0 + wn0, lane);
}

// Pointer tables do not change while a kernel runs: read as constant memory, i.e. by scalar loads also behind stores
// (a vector load would be waited for together with every store before it).
__device__ __forceinline__ const char* table_entry(const void* const* tab, long i) {
  typedef const void* const __attribute__((address_space(4)))* cptr;
  return (const char*)((cptr)tab)[i];
}

typedef __attribute__((__vector_size__(16))) unsigned u32x4;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

// Epilogue of one wavefront of the kernel below: 128 x 64 outputs in pieces of 16 rows through 4 KB of LDS that the ring
// of k-tiles leaves free (the next tile's k-tiles are in it already), 16-byte chunks swizzled by the row instead of padded.
// Rows past M lie past the end of the buffers: their loads give zeros and their stores are dropped, so every tile issues
// the same operations.
__device__ __forceinline__ void dgelu_epilogue(f32x16 (&acc)[4][2], lds_byte* ep, const char* g_in, char* out, int N, int M,
                                               int mrow0, int ncol0, int lane) {
  const int lr = lane & 31, lh = lane >> 5, ci = lane & 7, rr = lane >> 3, r16 = lr & 15;
  const long first = 2 * ((long)mrow0 * N + ncol0);
  const unsigned left = M > mrow0 ? (unsigned)((M - mrow0) * N - ncol0) * 2u : 0u;
  auto buf = [&](const char* p) {
    const unsigned long b = (unsigned long)(p + first);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)((unsigned long)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(left), 0x00020000);
  };
  const auto bo = buf(out), bg = buf(g_in);
  const int off = 2 * (rr * N + 8 * ci);
  // the cached derivatives, fetched two pieces ahead: no wait for them then covers a store just issued
  constexpr int STREAM = 2;                                // non-temporal
  bf16x8 g[2][2];
  auto fetch = [&](int piece) {
#pragma unroll
    for (int it = 0; it < 2; ++it)
      g[piece & 1][it] = __builtin_bit_cast(
          bf16x8, __builtin_amdgcn_raw_buffer_load_b128(bg, off + 2 * N * (16 * piece + 8 * it), 0, STREAM));
  };
  fetch(0);
  fetch(1);
#pragma unroll
  for (int p = 0; p < 8; ++p) {                            // rows 16 p ..
    // the lanes read what others wrote: nothing may move across these two points, nor be taken into a branch
    __builtin_amdgcn_wave_barrier();
    if ((lr >> 4) == (p & 1)) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16& c = acc[p >> 1][j];
          const f32x4 v = {c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
          *(lds_f32x4*)(ep + r16 * 256 + (((8 * j + 2 * q + lh) ^ r16) << 4)) = v;
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int row = it * 8 + rr;
      const f32x4 x = *(const lds_f32x4*)(ep + row * 256 + (((2 * ci) ^ row) << 4));
      const f32x4 y = *(const lds_f32x4*)(ep + row * 256 + (((2 * ci + 1) ^ row) << 4));
      bf16x8 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r[e] = (bf16)(x[e] * (float)g[p & 1][it][e]);
        r[4 + e] = (bf16)(y[e] * (float)g[p & 1][it][4 + e]);
      }
      if (it == 1 && p + 2 < 8) fetch(p + 2);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, r), bo, off + 2 * N * (16 * p + 8 * it), 0, STREAM);
    }
  }
}

// ---------------------------------------------------------------------------
// Multiply-by-GELU' products of more than one round of whole 256x256 tiles: one block per CU walks the tiles of its XCD, and
// its ring of k-tiles runs on from one tile into the next.  What bounds such a launch besides the matrix cores is the time
// they stand still between two tiles: start of a block, pointer tables, first loads, and an epilogue that reads and
// writes the output's size.  Here the first two k-tiles of the next tile are on their way during the last two of this
// one, and the stores drain under its first products (waited for by count).  5 x 4096 rows, 768 -> 3072: 125 -> 119 us;
// 5 x 12608 rows, 384 -> 1536: 125 -> 117; 6 x 4096 rows, 512 -> 2048: 81 -> 77; training steps 0.7 % (GPT-2, ViT and MT
// shapes).  The other epilogues gained nothing in this form (store 79 -> 79 us, bias+GELU 110 -> 112).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(512, 2)
gemm_mfma_dgelu_walk_kernel(const GemmArgs a, int tiles_m, int tiles_n, int total_tiles, int per_xcd, int pm, int pn) {
  constexpr int BM = 256, BN = 256, BK = 64, WN = 4, WTM = 128, WTN = 64, TM = 4, TN = 2;
  constexpr int RB = BK * 2, CPR = RB / 16, RPL = 1024 / RB, KS = BK / 16;
  constexpr int A_BYTES = BM * RB, STAGE = A_BYTES + BN * RB, LD_ = 4, PER_TILE = 8, RING = 2 * STAGE;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem2[];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;
  const int K = a.K, M = a.M, KT = K / BK, per_group = tiles_m * tiles_n, walkers = gridDim.x >> 3;
  const int lrow = lane / CPR, lpos = lane % CPR;
  const int end = min(((int)(blockIdx.x & 7) + 1) * per_xcd, total_tiles);
  int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= end) return;

  struct Place { int g, m0, n0; __amdgpu_buffer_rsrc_t A, B; int aoff[LD_]; };
  auto locate = [&](Place& p, int t) {
    p.g = __builtin_amdgcn_readfirstlane(t / per_group);
    const int tg = t - p.g * per_group;
    int tm, tn;
    if (pn > 0) {
      const int patch = pm * pn, patches_n = tiles_n / pn, b = tg / patch, w = tg - b * patch, bm = b / patches_n;
      tm = bm * pm + w / pn;
      tn = (b - bm * patches_n) * pn + w % pn;
    } else {
      tm = tg / tiles_n;
      tn = tg - tm * tiles_n;
    }
    p.m0 = __builtin_amdgcn_readfirstlane(tm) * BM;
    p.n0 = __builtin_amdgcn_readfirstlane(tn) * BN;
    p.A = lds_source(reinterpret_cast<const bf16*>(a.A) + a.a_slots.of(p.g) * a.a_slot_stride + (long)p.m0 * K);
    p.B = lds_source(table_entry(a.B.tab, a.B.i0 + (long)p.g * a.B.is) + a.b_off + 2 * (long)p.n0 * K);
#pragma unroll
    for (int j = 0; j < LD_; ++j) {
      const int row = (wave * LD_ + j) * RPL + lrow;
      p.aoff[j] = ((row < M - p.m0 ? row : M - 1 - p.m0) * K + (lpos ^ swz(row)) * 8) * 2;
    }
  };
  int boff[LD_];
#pragma unroll
  for (int j = 0; j < LD_; ++j) {
    const int row = (wave * LD_ + j) * RPL + lrow;
    boff[j] = (row * K + (lpos ^ swz(row)) * 8) * 2;
  }
  auto issue_one = [&](const Place& p, int stage, int k0, int idx) {
    unsigned char* sa = smem2 + stage * STAGE + (idx < LD_ ? 0 : A_BYTES) + (wave * LD_ + (idx & (LD_ - 1))) * 1024;
    if (idx < LD_) load_to_lds(p.A, sa, p.aoff[idx & (LD_ - 1)], 2 * k0);
    else load_to_lds(p.B, sa, boff[idx & (LD_ - 1)], 2 * k0);
  };
  int foff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) foff[ks] = lr * RB + (((2 * ks + lh) ^ swz(lr)) << 4);
  const lds_byte* lds0 = (const lds_byte*)smem2;

  Place cur, nxt;
  locate(cur, tile);
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int u = 0; u < PER_TILE; ++u) issue_one(cur, s, s * BK, u);     // KT >= 2
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  wait_vmcnt<PER_TILE>();
  bare_barrier();
  bf16x8 fa[2][TM], fb[2][TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) fb[0][j] = lds_read16(lds0 + A_BYTES + (wn0 + j * 32) * RB + foff[0]);
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[0][i] = lds_read16(lds0 + (wm0 + i * 32) * RB + foff[0]);

  constexpr int EP_OPS = 16;                               // at least so many operations follow a tile's last loads
  int st = 0;                                              // stage of the k-tile at hand
  bool stores = false;                                     // the last epilogue's are in flight
  while (true) {
    const bool more = tile + walkers < end;
    nxt = cur;                                             // (after the last tile its own first k-tiles once more)
    if (more) locate(nxt, tile + walkers);
    int kt = 0;
    do {                                                   // KT >= 2
      const bool ahead = kt + 2 >= KT;                     // the loads are the next tile's
      const int k0 = (ahead ? kt + 2 - KT : kt + 2) * BK;
      Place from;
      from.A = ahead ? nxt.A : cur.A;
      from.B = ahead ? nxt.B : cur.B;
#pragma unroll
      for (int u = 0; u < LD_; ++u) from.aoff[u] = ahead ? nxt.aoff[u] : cur.aoff[u];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int cb = ks & 1, nb = cb ^ 1;
        const bool last = ks == KS - 1;
        if (last) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if (stores) wait_vmcnt<EP_OPS>();
          else wait_vmcnt<0>();
          stores = false;
          bare_barrier();
        }
        const int rst = last ? st ^ 1 : st, rks = last ? 0 : ks + 1;
        const lds_byte* sA = lds0 + rst * STAGE + wm0 * RB;
        const lds_byte* sB = lds0 + rst * STAGE + A_BYTES + wn0 * RB;
        constexpr int NM = TM * TN, RD = TM + TN;
#pragma unroll
        for (int q = 0; q < NM; ++q) {
          const int i = q / TN, j = q % TN;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cb][j], fa[cb][i], acc[i][j], 0, 0, 0);
          const int r0 = (q * RD * 4 / 3 + NM - 1) / NM, r1 = ((q + 1) * RD * 4 / 3 + NM - 1) / NM;
#pragma unroll
          for (int u = 0; u < RD; ++u)
            if (u >= r0 && (u < r1 || q == NM - 1)) {
              if (u < TN) fb[nb][u] = lds_read16(sB + u * 32 * RB + foff[rks]);
              else fa[nb][u - TN] = lds_read16(sA + (u - TN) * 32 * RB + foff[rks]);
            }
          if (last) issue_one(from, st, k0, q);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      st ^= 1;
    } while (++kt < KT);
    dgelu_epilogue(acc, (lds_byte*)smem2 + RING + wave * 4096,
                   static_cast<const char*>(a.aux) + 2 * a.aux_slots.of(cur.g) * a.aux_slot_stride,
                   static_cast<char*>(a.out) + 2 * a.out_slots.of(cur.g) * a.out_slot_stride, a.N, M, cur.m0 + wm0, cur.n0 + wn0,
                   lane);
    if (!more) break;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    stores = true;
    tile += walkers;
    cur = nxt;
  }
  wait_vmcnt<0>();                                         // (the loads behind the last tile)
}

// ---------------------------------------------------------------------------
// fp32 MFMA kernel (fp32 parameters and operands): 64x64 block tile, 4 wavefronts of 32x32 on
// the 32x32x2 fp32 MFMA, k-tiles of 16 staged through LDS.  As in the bf16 kernel the weight
// fragment is the first MFMA operand, so a lane ends up with 4 consecutive output columns of one
// row per register quad and the shared epilogue code applies.  Needs N % 64 == 0 and K % 16 == 0;
// M may be ragged (rows are clamped on load and guarded on store).
// ---------------------------------------------------------------------------
template <int EPI>
__global__ void __launch_bounds__(256)
gemm_f32_mfma_kernel(const GemmArgs a, int tiles_m, int tiles_n) {
  constexpr int BT = 64, BKF = 16, LD = BKF + 4;       // row pitch 20 floats: 16-byte aligned vector stores
  __shared__ __attribute__((aligned(16))) float As[BT * LD];
  __shared__ __attribute__((aligned(16))) float Bs[BT * LD];
  const int g = blockIdx.z;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
  const int m0 = tm * BT, n0 = tn * BT;
  const float* A = reinterpret_cast<const float*>(a.A) + a.a_slots.of(g) * a.a_slot_stride;
  const float* B = reinterpret_cast<const float*>(a.B.at(g) + a.b_off);
  const int M = a.M, K = a.K;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
  const int srow = tid >> 2, sk = (tid & 3) * 4;       // staging: one float4 of each operand per thread
  int am = m0 + srow;
  am = am < M ? am : M - 1;
  const float* ap = A + (long)am * K + sk;
  const float* bp = B + (long)(n0 + srow) * K + sk;
  f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
  f32x4 va = *reinterpret_cast<const f32x4*>(ap), vb = *reinterpret_cast<const f32x4*>(bp);
  for (int k0 = 0; k0 < K; k0 += BKF) {
    __syncthreads();                                   // the previous k-tile has been read by every wavefront
    *reinterpret_cast<f32x4*>(&As[srow * LD + sk]) = va;
    *reinterpret_cast<f32x4*>(&Bs[srow * LD + sk]) = vb;
    __syncthreads();
    if (k0 + BKF < K) {                                // next k-tile's loads fly while this one is multiplied
      va = *reinterpret_cast<const f32x4*>(ap + k0 + BKF);
      vb = *reinterpret_cast<const f32x4*>(bp + k0 + BKF);
    }
#pragma unroll
    for (int ks = 0; ks < BKF; ks += 2)
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(Bs[(wn0 + lr) * LD + ks + lh], As[(wm0 + lr) * LD + ks + lh],
                                                      acc[0][0], 0, 0, 0);
  }
  const EpiPtrs P = resolve_epi<float>(a, g, EPI);
  tile_epilogue<EPI, float, 1, 1, false, false>(acc, nullptr, P.bias, static_cast<float*>(P.out), static_cast<float*>(P.out),
                                         static_cast<const float*>(P.aux), static_cast<float*>(P.aux2), P.base, P.X,
                                         static_cast<const float*>(P.aux), P.RHS, P.OUT, a.hstep, a.rhs_sign, a.N, M,
                                         m0 + wm0, n0 + wn0, lane);
}

// ---------------------------------------------------------------------------
// fp32 MFMA kernel for launches that leave the kernel above fewer than two tiles per CU, and for ragged shapes:
// 32x32 block tile, four wavefronts of 16x16 on the 16x16x4 fp32 MFMA, k-tiles of 64.  What bounds such launches is
// one wavefront's serial chain, which a quarter tile on 32-cycle MFMAs makes four times shorter, and first touches:
// two k-tiles are in LDS and two more on their way in registers, and the one barrier per k-tile waits for LDS only.
// The fp32 MFMAs add their products one by one in the order of the reduction index, so with the operands in natural
// order this kernel, the one above and the FMA kernel give the same bits, and which of them a launch takes (it depends
// on how many layers share the launch) cannot show in a result.  Groups of 16 reduction indices lie in LDS as a
// transposed 4 x 4, so that a lane's 16-byte read is its operand of four MFMAs in that order; with the row pitch of 68
// floats the 16 rows of a read fall on 16 distinct 16-byte slots and the 4-byte writes of a wavefront on 64 banks.
// Any M; N and K multiples of 4: rows and columns past the edge are clamped, chunks past K become zeros.
// Whole layer steps on the kernel above and on this one: 512 wide, 100 tokens, one layer 138 -> 71 us, transposed
// 292 -> 165; 512 wide, 4 x 512 tokens 230 -> 213 and 472 -> 446; 200 wide, 600 hidden, 129 tokens (the FMA kernel
// before) 136 -> 55 and 257 -> 132.
// ---------------------------------------------------------------------------
template <int EPI, bool RAGGED>
__global__ void __launch_bounds__(256)
gemm_f32_small_kernel(const GemmArgs a, int tiles_n) {
  constexpr int BT = 32, BKF = 64, LD = BKF + 4;
  constexpr int CPR = BKF / 4, RPP = 256 / CPR;                  // 16-byte chunks per row; rows per pass of the block
  static_assert(2 * RPP == BT, "two chunks of each operand per thread");
  __shared__ __attribute__((aligned(16))) float As[2][BT * LD], Bs[2][BT * LD];
  const int g = blockIdx.z;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
  const int m0 = tm * BT, n0 = tn * BT;
  const float* A = reinterpret_cast<const float*>(a.A) + a.a_slots.of(g) * a.a_slot_stride;
  const float* B = reinterpret_cast<const float*>(a.B.at(g) + a.b_off);
  const int M = a.M, N = a.N, K = a.K, tiles_k = (K + BKF - 1) / BKF;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wm0 = (wave >> 1) * 16, wn0 = (wave & 1) * 16;
  const int srow = tid / CPR, sk = tid % CPR * 4;
  const int spos = (sk & ~15) + (sk >> 2 & 3);                   // of 16 reduction indices, 4e + j is kept at 4j + e
  const float *ap[2], *bp[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int am = m0 + srow + u * RPP, bn = n0 + srow + u * RPP;
    ap[u] = A + (long)(am < M ? am : M - 1) * K;
    bp[u] = B + (long)(bn < N ? bn : N - 1) * K;
  }
  struct Regs { f32x4 x[2], w[2]; };
  auto load = [&](Regs& v, int kt) {
    if (kt >= tiles_k) return;
    int k = kt * BKF + sk;
    if (RAGGED) k = k < K ? k : 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      v.x[u] = *reinterpret_cast<const f32x4*>(ap[u] + k);
      v.w[u] = *reinterpret_cast<const f32x4*>(bp[u] + k);
    }
  };
  auto store = [&](const Regs& v, int kt, int buf) {
    if (kt >= tiles_k) return;
    const bool inside = !RAGGED || kt * BKF + sk < K;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const f32x4 x = inside ? v.x[u] : z, w = inside ? v.w[u] : z;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        As[buf][(srow + u * RPP) * LD + spos + 4 * j] = x[j];
        Bs[buf][(srow + u * RPP) * LD + spos + 4 * j] = w[j];
      }
    }
  };
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int buf) {
    const float* pa = &As[buf][(wm0 + lr) * LD + 4 * lg];
    const float* pb = &Bs[buf][(wn0 + lr) * LD + 4 * lg];
#pragma unroll
    for (int k = 0; k < BKF; k += 16) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(pa + k), w = *reinterpret_cast<const f32x4*>(pb + k);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], x[e], acc, 0, 0, 0);
    }
  };
  auto lds_barrier = [&] {                               // loads into registers stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bare_barrier();
  };
  // k-tile kt in buffer kt % 2: buffer b is written again only after the barrier that ends its tile
  Regs r0, r1;
  load(r0, 0);
  load(r1, 1);
  store(r0, 0, 0);
  load(r0, 2);
  lds_barrier();
  for (int kt = 0; kt < tiles_k; kt += 2) {
    store(r1, kt + 1, 1);
    load(r1, kt + 3);
    multiply(0);
    lds_barrier();
    if (kt + 1 >= tiles_k) break;                        // uniform over the block
    store(r0, kt + 2, 0);
    load(r0, kt + 4);
    multiply(1);
    lds_barrier();
  }
  const int m = m0 + wm0 + lr, n = n0 + wn0 + 4 * lg;
  if (m < M && n < N) epilogue4<EPI, float>(resolve_epi<float>(a, g, EPI), a.hstep, a.rhs_sign, N, m, n, acc);
}

// ---------------------------------------------------------------------------
// Parameter gradients of a linear map:  dW_g[m,n] = scale * sum_t dY_g[t,m] U_g[t,n],  db_g[m] = scale *
// sum_t dY_g[t,m], both operands packed token-major.  The reduction runs over the rows of both, so the
// k-tiles are staged as they lie in memory ([token][feature], global -> LDS directly, the ring of the kernel
// above) and the fragments come out of LDS through the transposing read of gfx950 (ds_read_b64_tr_b16: 16
// lanes read 4 rows of 16 columns and each lane gets one column's 4 values).  16-byte chunks are
// XOR-swizzled by the row so that the 4 rows of a read fall on distinct banks; any token count works (rows
// past K come from a zero chunk), and so does any width that is a multiple of 8.
// The bias gradient is summed from the same fragments by the wavefronts of the first column of tiles, a k-tile at a
// time; the rounding errors of adding up the k-tiles and the slices are carried along.
// This replaces a transposition of both operands (2.8 TB/s, with GELU or a LayerNorm recomputed on the way)
// before a product of two reduction-contiguous operands.
// ---------------------------------------------------------------------------

// Sum that carries its rounding error along (Kahan): 16384 positive terms come out within 7e-8 of their sum, as a
// plain chain within 8e-7 to 3e-6, depending on their spread.  An infinite sum carries nothing, so it stays infinite.
struct CarrySum {
  float sum = 0.f, err = 0.f;
  __device__ __forceinline__ void add(float x) {
    const float y = x - err, t = sum + y;
    err = __builtin_isfinite(t) ? (t - sum) - y : 0.f;
    sum = t;
  }
};

template <int BM, int BN, int STAGES, int WM, int WN, bool TAIL>
__global__ void __launch_bounds__(64 * WM * WN, WM * WN / 4)
gemm_tn_mfma_kernel(const GemmTnArgs a, int tiles_m, int tiles_n, int splits, int total_tiles, int per_xcd) {
  constexpr int NW = WM * WN, BK = 64, KS = BK / 16;
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int RA = BM * 2, RB = BN * 2;                // bytes per LDS row (one token)
  constexpr int A_BYTES = BK * RA, B_BYTES = BK * RB, STAGE = A_BYTES + B_BYTES;
  constexpr int A_LD = A_BYTES / 1024 / NW, B_LD = B_BYTES / 1024 / NW, PER_TILE = A_LD + B_LD;
  static_assert(A_LD * 1024 * NW == A_BYTES && B_LD * 1024 * NW == B_BYTES, "tile/wave split");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem2[];
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= total_tiles) return;
  const int per_slice = tiles_m * tiles_n;
  const int gs = __builtin_amdgcn_readfirstlane(tile / per_slice), tg = tile - gs * per_slice;
  const int tm = __builtin_amdgcn_readfirstlane(tg / tiles_n), tn = tg - tm * tiles_n;
  const int g = __builtin_amdgcn_readfirstlane(gs / splits), sp = gs - g * splits;       // slice sp of the group's tokens
  const int m0 = tm * BM, n0 = tn * BN, M = a.M, N = a.N;
  const int all_tiles = (a.K + BK - 1) / BK;
  const int kt0 = (int)((long)all_tiles * sp / splits), kt1 = (int)((long)all_tiles * (sp + 1) / splits);
  const int K = (kt1 * BK < a.K ? kt1 * BK : a.K) - kt0 * BK;
  const bf16* A = reinterpret_cast<const bf16*>(a.A) + a.a_slots.of(g) * a.a_slot_stride + (long)kt0 * BK * M;
  const bf16* B = reinterpret_cast<const bf16*>(a.B) + a.b_slots.of(g) * a.b_slot_stride + (long)kt0 * BK * N;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;

  // row r keeps logical chunk c at position c ^ f(r): 256-byte rows (or longer) repeat the banks every row,
  // 128-byte rows every second one
  auto swz_of = [](int row_bytes, int r) { return row_bytes >= 256 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; };
  int aoff[A_LD], boff[B_LD];                            // element offsets inside a k-tile
#pragma unroll
  for (int j = 0; j < A_LD; ++j) {
    const int row = (wave * A_LD + j) * (1024 / RA) + lane / (RA / 16);
    int col = m0 + ((lane % (RA / 16)) ^ swz_of(RA, row)) * 8;
    col = col < M ? col : 0;                             // columns past the edge: never stored
    aoff[j] = row * M + col;
  }
#pragma unroll
  for (int j = 0; j < B_LD; ++j) {
    const int row = (wave * B_LD + j) * (1024 / RB) + lane / (RB / 16);
    int col = n0 + ((lane % (RB / 16)) ^ swz_of(RB, row)) * 8;
    col = col < N ? col : 0;
    boff[j] = row * N + col;
  }
  auto issue_one = [&](int stage, int k0, int idx) {
    const bool is_a = idx < A_LD;
    const int slot = is_a ? wave * A_LD + idx : wave * B_LD + idx - A_LD;
    unsigned char* dst = smem2 + stage * STAGE + (is_a ? 0 : A_BYTES) + slot * 1024;
    const bf16* tile = is_a ? A + (long)k0 * M : B + (long)k0 * N;
    const int off = is_a ? aoff[idx < A_LD ? idx : 0] : boff[idx < A_LD ? 0 : idx - A_LD];
    if constexpr (TAIL) {                                  // tokens past the last one are zeros
      const int row = is_a ? slot * (1024 / RA) + lane / (RA / 16) : slot * (1024 / RB) + lane / (RB / 16);
      const bf16* src = row < K - k0 ? tile + off : reinterpret_cast<const bf16*>(g_zero_chunk);
      __builtin_amdgcn_global_load_lds((gas_ptr)src, (las_ptr)dst, 16, 0, 0);
    } else {
      load_to_lds(lds_source(tile), dst, 2 * off, 0);
    }
  };
  auto issue = [&](int stage, int k0) {
#pragma unroll
    for (int idx = 0; idx < PER_TILE; ++idx) issue_one(stage, k0, idx);
  };
  // this lane's address inside a fragment: token 8*lh + (lane%16)/4 (+ 4 for the second half), 16 columns per
  // group of 16 lanes
  const int lh = lane >> 5, trow = 8 * lh + ((lane & 15) >> 2), low = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  int offa[TM], offb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    offa[i] = trow * RA + (((((wm0 + 32 * i) >> 3) + low) ^ swz_of(RA, trow)) << 4) + (lane & 1) * 8;
#pragma unroll
  for (int j = 0; j < TN; ++j)
    offb[j] = trow * RB + (((((wn0 + 32 * j) >> 3) + low) ^ swz_of(RB, trow)) << 4) + (lane & 1) * 8;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  CarrySum bsum[TM];
  float btile[TM];                                             // of the k-tile at hand
  const bool sums = tn == 0 && wn0 == 0;                       // wave-uniform

  const int KT = (K + BK - 1) / BK;
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < KT) issue(s, s * BK);
  auto wait_tile = [&](int kt, int issued) {
    const int behind = issued - 1 - kt;
    if constexpr (STAGES >= 4) if (behind >= 3) { wait_vmcnt<3 * PER_TILE>(); return; }
    if constexpr (STAGES >= 3) if (behind >= 2) { wait_vmcnt<2 * PER_TILE>(); return; }
    if (behind >= 1) { wait_vmcnt<PER_TILE>(); return; }
    wait_vmcnt<0>();
  };
  // Fragments are read DIST k-steps ahead of their products (1 where a step is long enough to hide the LDS
  // latency, else 2); the step that first needs the next tile begins with its wait and barrier.
  constexpr int NM = TM * TN, RD = TM + TN, DIST = NM >= 8 ? 1 : 2, BUFS = DIST == 1 ? 2 : 4;
  const lds_byte* lds0 = (const lds_byte*)smem2;
  TrFrag fa[BUFS][TM], fb[BUFS][TN];
  auto read = [&](auto ks_tag, unsigned stage_off, int u) {
    constexpr int ks = decltype(ks_tag)::value, nb = ks % BUFS;
    if (u < TN) tr_read<16 * ks * RB, (16 * ks + 4) * RB>(fb[nb][u < TN ? u : 0], lds0 + stage_off + A_BYTES + offb[u < TN ? u : 0]);
    else tr_read<16 * ks * RA, (16 * ks + 4) * RA>(fa[nb][u < TN ? 0 : u - TN], lds0 + stage_off + offa[u < TN ? 0 : u - TN]);
  };
  wait_tile(0, STAGES < KT ? STAGES : KT);
  bare_barrier();
#pragma unroll
  for (int u = 0; u < RD; ++u) read(std::integral_constant<int, 0>{}, 0, u);
  if constexpr (DIST == 2) {
#pragma unroll
    for (int u = 0; u < RD; ++u) read(std::integral_constant<int, 1>{}, 0, u);
  }
  // one k-step: its products, with the reads of the step DIST ahead and (LOADS) of the refilled stage's loads
  // in between
  auto step = [&](auto ks_tag, auto loads_tag, unsigned read_stage, int stage, int pk0) {
    constexpr int ks = decltype(ks_tag)::value, cb = ks % BUFS, rks = (ks + DIST) % KS;
    bf16x8 xa[TM], xb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) xa[i] = tr_value(fa[cb][i]);
#pragma unroll
    for (int j = 0; j < TN; ++j) xb[j] = tr_value(fb[cb][j]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      const int i = q / TN, j = q % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xb[j], xa[i], acc[i][j], 0, 0, 0);
      const int r0 = (q * RD * 4 / 3 + NM - 1) / NM, r1 = ((q + 1) * RD * 4 / 3 + NM - 1) / NM;
#pragma unroll
      for (int u = 0; u < RD; ++u)
        if (u >= r0 && (u < r1 || q == NM - 1)) read(std::integral_constant<int, rks>{}, read_stage, u);
      if constexpr (decltype(loads_tag)::value) {
        const int l0 = (q * PER_TILE + NM - 1) / NM, l1 = ((q + 1) * PER_TILE + NM - 1) / NM;
#pragma unroll
        for (int u = 0; u < PER_TILE; ++u)
          if (u >= l0 && u < l1) issue_one(stage, pk0, u);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (sums) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = (float)xa[i][e];
        const float u = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        btile[i] = ks == 0 ? u : btile[i] + u;
        if (ks == KS - 1) bsum[i].add(btile[i]);
      }
    }
  };
  int cur = 0;
  auto tile_step = [&](int kt, auto loads_tag) {
    const int nxt = cur + 1 == STAGES ? 0 : cur + 1;
    const unsigned so = cur * STAGE, sn = nxt * STAGE;
    auto handover = [&]() {                              // tile kt+1 is there, nobody reads tile kt any more
      wait_lgkm();
      wait_tile(kt + 1, kt + STAGES < KT ? kt + STAGES : KT);
      bare_barrier();
    };
    step(std::integral_constant<int, 0>{}, std::false_type{}, so, 0, 0);
    step(std::integral_constant<int, 1>{}, std::false_type{}, so, 0, 0);
    if constexpr (DIST == 2) handover();
    step(std::integral_constant<int, 2>{}, std::integral_constant<bool, DIST == 2 && decltype(loads_tag)::value>{},
         DIST == 2 ? sn : so, cur, (kt + STAGES) * BK);
    if constexpr (DIST == 1) handover();
    step(std::integral_constant<int, 3>{}, std::integral_constant<bool, DIST == 1 && decltype(loads_tag)::value>{}, sn,
         cur, (kt + STAGES) * BK);
    cur = nxt;
  };
  int kt = 0;
  for (; kt + STAGES < KT; ++kt) tile_step(kt, std::true_type{});
  for (; kt < KT; ++kt) tile_step(kt, std::false_type{});
  wait_lgkm();
  bare_barrier();
  // one slice: straight into the gradient block; several: unscaled into the slice's [M x N | M] of the scratch
  float *dW, *db, scale = a.scale;
  if (splits == 1) {
    char* out = const_cast<char*>(a.out.at(g));
    dW = reinterpret_cast<float*>(out + a.w_off);
    db = reinterpret_cast<float*>(out + a.b_off);
  } else {
    dW = a.partial + (long)gs * ((long)M * N + M);
    db = dW + (long)M * N;
    scale = 1.f;
  }
  if (sums) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const float t = bsum[i].sum + __shfl_xor(bsum[i].sum, 32, 64);   // the two k halves
      const int m = m0 + wm0 + 32 * i + (lane & 31);
      if (lh == 0 && m < M) db[m] = scale * t;
    }
  }
  constexpr int EP_BYTES = (32 * (WTN * 4 + 16) + 1023) / 1024 * 1024;
  tile_epilogue<EPI_STORE_F32, bf16, TM, TN, true, true>(
      acc, smem2 + wave * EP_BYTES, nullptr, static_cast<bf16*>(nullptr), dW, static_cast<const bf16*>(nullptr),
      static_cast<bf16*>(nullptr), nullptr, nullptr, nullptr, nullptr, nullptr, scale, 1.f, N, M, m0 + wm0, n0 + wn0,
      lane);
}

// sums of the slices, in order
__global__ void __launch_bounds__(256) gemm_tn_reduce_kernel(const GemmTnArgs a, int splits) {
  const int g = blockIdx.y;
  const long mn = (long)a.M * a.N, each = mn + a.M;            // M and N are multiples of 4
  const long i = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= each) return;
  const float* p = a.partial + (long)g * splits * each + i;
  CarrySum acc[4];
  for (int s = 0; s < splits; ++s) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + s * each);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e].add(v[e]);
  }
  char* out = const_cast<char*>(a.out.at(g));
  float* o = i < mn ? reinterpret_cast<float*>(out + a.w_off) + i : reinterpret_cast<float*>(out + a.b_off) + (i - mn);
  *reinterpret_cast<f32x4*>(o) = a.scale * f32x4{acc[0].sum, acc[1].sum, acc[2].sum, acc[3].sum};
}

// fp32 operands: 64x64 tile, 4 wavefronts of 32x32 on the 32x32x2 fp32 MFMA, 16 tokens per k-tile.  The
// fragments of this product are contiguous in the token-major tiles, so no transposition is involved.
__global__ void __launch_bounds__(256) gemm_tn_f32_kernel(const GemmTnArgs a, int tiles_n, int splits) {
  constexpr int BT = 64, BKF = 16, LD = BT + 4;
  __shared__ __attribute__((aligned(16))) float As[BKF * LD];
  __shared__ __attribute__((aligned(16))) float Bs[BKF * LD];
  const int g = blockIdx.z, tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n, sp = blockIdx.y;
  const int m0 = tm * BT, n0 = tn * BT, M = a.M, N = a.N;
  const int all_tiles = (a.K + BKF - 1) / BKF;
  const int kt0 = (int)((long)all_tiles * sp / splits), kt1 = (int)((long)all_tiles * (sp + 1) / splits);
  const int K = (kt1 * BKF < a.K ? kt1 * BKF : a.K) - kt0 * BKF;
  const float* A = reinterpret_cast<const float*>(a.A) + a.a_slots.of(g) * a.a_slot_stride + (long)kt0 * BKF * M;
  const float* B = reinterpret_cast<const float*>(a.B) + a.b_slots.of(g) * a.b_slot_stride + (long)kt0 * BKF * N;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
  const int srow = tid >> 4, sc = (tid & 15) * 4;              // one float4 of each operand per thread
  const int ac = m0 + sc < M ? m0 + sc : 0, bc = n0 + sc < N ? n0 + sc : 0;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
  CarrySum bsum;
  auto ld = [&](const float* p, int stride, int col, int k) {
    return k < K ? *reinterpret_cast<const f32x4*>(p + (long)k * stride + col) : zero;
  };
  f32x4 va = ld(A, M, ac, srow), vb = ld(B, N, bc, srow);
  for (int k0 = 0; k0 < K; k0 += BKF) {
    __syncthreads();
    *reinterpret_cast<f32x4*>(&As[srow * LD + sc]) = va;
    *reinterpret_cast<f32x4*>(&Bs[srow * LD + sc]) = vb;
    __syncthreads();
    if (k0 + BKF < K) { va = ld(A, M, ac, k0 + BKF + srow); vb = ld(B, N, bc, k0 + BKF + srow); }
#pragma unroll
    for (int ks = 0; ks < BKF; ks += 2)
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(Bs[(ks + lh) * LD + wn0 + lr], As[(ks + lh) * LD + wm0 + lr],
                                                      acc[0][0], 0, 0, 0);
    if (tn == 0 && tid < BT) {
      float t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float* p = As + 4 * k * LD + tid;
        t[k] = (p[0] + p[LD]) + (p[2 * LD] + p[3 * LD]);
      }
      bsum.add((t[0] + t[1]) + (t[2] + t[3]));
    }
  }
  float *W, *db, scale = a.scale;
  if (splits == 1) {
    char* out = const_cast<char*>(a.out.at(g));
    W = reinterpret_cast<float*>(out + a.w_off);
    db = reinterpret_cast<float*>(out + a.b_off);
  } else {
    W = a.partial + (long)(g * splits + sp) * ((long)M * N + M);
    db = W + (long)M * N;
    scale = 1.f;
  }
  if (tn == 0 && tid < BT && m0 + tid < M) db[m0 + tid] = scale * bsum.sum;
  const int m = m0 + wm0 + lr;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int n = n0 + wn0 + 8 * q + 4 * lh;
    const f32x4 v = {acc[0][0][4 * q], acc[0][0][4 * q + 1], acc[0][0][4 * q + 2], acc[0][0][4 * q + 3]};
    if (m < M && n < N) *reinterpret_cast<f32x4*>(W + (long)m * N + n) = scale * v;
  }
}

// ---------------------------------------------------------------------------
// generic kernel: 64x64x16 tile, 256 threads, 4x4 outputs per thread
// ---------------------------------------------------------------------------
template <typename TA, int EPI, typename TO>
__global__ void __launch_bounds__(256)
gemm_simple_kernel(const GemmArgs a, int tiles_m, int tiles_n) {
  constexpr int BT = 64, BKS = 16, LD = BT + 4;
  __shared__ float As[BKS][LD];
  __shared__ float Bs[BKS][LD];
  const int g = blockIdx.z;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
  const int m0 = tm * BT, n0 = tn * BT;
  const TA* A = reinterpret_cast<const TA*>(a.A) + a.a_slots.of(g) * a.a_slot_stride;
  const char* pblock = a.B.at(g);
  const TA* B = reinterpret_cast<const TA*>(pblock + a.b_off);
  const int M = a.M, N = a.N, K = a.K;
  const int tid = threadIdx.x;
  const int lrow = tid >> 2, lk = (tid & 3) * 4;
  const int ty = tid >> 4, tx = tid & 15;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += BKS) {
    f32x4 va = {0, 0, 0, 0}, vb = {0, 0, 0, 0};
    if (m0 + lrow < M && k0 + lk < K) va = load4<TA>(A + (long)(m0 + lrow) * K + k0 + lk);
    if (n0 + lrow < N && k0 + lk < K) vb = load4<TA>(B + (long)(n0 + lrow) * K + k0 + lk);
#pragma unroll
    for (int i = 0; i < 4; ++i) { As[lk + i][lrow] = va[i]; Bs[lk + i][lrow] = vb[i]; }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BKS; ++k) {
      f32x4 x = *reinterpret_cast<const f32x4*>(&As[k][ty * 4]);
      f32x4 y = *reinterpret_cast<const f32x4*>(&Bs[k][tx * 4]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(x[i], y[j], acc[i][j]);
    }
    __syncthreads();
  }
  const int n = n0 + tx * 4;
  if (n < N) {
    const EpiPtrs P = resolve_epi<TO>(a, g, EPI);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + ty * 4 + i;
      if (m < M) {
        f32x4 v = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
        epilogue4<EPI, TO>(P, a.hstep, a.rhs_sign, N, m, n, v);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static int g_force_simple = 0;
static int g_tile_cfg = 0;                 // 0 = choose by shape
static int g_grad_slices = 0;              // the same
void gemm_force_simple(int on) { g_force_simple = on; }
void gemm_set_tile_config(int cfg) { g_tile_cfg = cfg; }
bool gemm_forced() { return g_force_simple || g_tile_cfg; }
void gemm_set_grad_slices(int n) { g_grad_slices = n > 0 ? n : 0; }

// Compute units of the current device (256 if the query fails).
int compute_units() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8)
      cus = 256;
    n = cus;
  }
  return n;
}

template <int BM, int BN, int BK, int STAGES, int OCC, bool RAGGED, int EPI, int WM, int WN>
static hipError_t launch_mfma(const GemmArgs& a, hipStream_t st) {
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const int total = tiles_m * tiles_n * a.n_groups;
  const int per_xcd = (total + 7) / 8;
  const size_t ring = (size_t)STAGES * (BM + BN) * BK * 2;
  const size_t staging = (size_t)WM * WN * ((32 * (BN / WN * 4 + 16) + 1023) / 1024 * 1024);
  const size_t smem = ring > staging ? ring : staging;
  // patch shape of the tile order: 4 tiles wide, half of what one XCD runs at a time (two patches next
  // to each other are resident together; measured against whole-resident-set patches: the bias+GELU
  // launches 5 % faster at the GPT-2 and BERT shapes, the others unchanged)
  int pm = 0, pn = 0;
  const int resident = compute_units() / 8 * OCC;
  if (tiles_n > 4 && tiles_n % 4 == 0 && resident % 8 == 0 && tiles_m % (resident / 8) == 0) {
    pn = 4;
    pm = resident / 8;
  }
  auto kern = gemm_mfma_kernel<BM, BN, BK, STAGES, OCC, RAGGED, EPI, bf16, WM, WN>;
  static unsigned long raised = 0;
  if (const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), (int)smem, raised); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(64 * WM * WN), smem, st, a, tiles_m, tiles_n, total,
                     per_xcd, pm, pn);
  return hipGetLastError();
}

// The walking form of the 256x256 tile: more than one tile per CU, two k-tiles or more, byte offsets of 32 bits.
static bool dgelu_walks(const GemmArgs& a) {
  const long tiles = (long)((a.M + 255) / 256) * (a.N / 256) * a.n_groups;
  return tiles > compute_units() && a.K >= 128 && a.bias_off < 0 && (double)a.M * a.N < 2e9;
}
static hipError_t launch_dgelu_walk(const GemmArgs& a, hipStream_t st) {
  const int tiles_m = (a.M + 255) / 256, tiles_n = a.N / 256, total = tiles_m * tiles_n * a.n_groups, per_xcd = (total + 7) / 8;
  const int smem = 2 * 512 * 128 + 8 * 4096;               // ring and eight staging regions: all of a CU's LDS
  int pm = 0, pn = 0;                                      // as in launch_mfma
  if (tiles_n > 4 && tiles_n % 4 == 0 && compute_units() == 256 && tiles_m % 4 == 0) pm = pn = 4;
  static unsigned long raised = 0;
  if (const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(gemm_mfma_dgelu_walk_kernel), smem, raised); e != hipSuccess) return e;
  hipLaunchKernelGGL(gemm_mfma_dgelu_walk_kernel, dim3(compute_units() / 8 * 8), dim3(512), smem, st, a, tiles_m, tiles_n,
                     total, per_xcd, pm, pn);
  return hipGetLastError();
}

// Two 64x64 tiles per CU are where the larger tile takes over: whole steps of small launches are up to twice as fast
// on 32x32 tiles (1024 wide, 2 layers of 128 tokens: 171 us against 325), large ones lose up to 13 % to fetching each
// operand twice as often (1024 wide, 4 layers of 1024 tokens: 1191 us against 1052).  Between two and four tiles per CU
// the larger one takes as long as a whole number of them: a launch whose last round is at most a quarter full is faster on
// the smaller (large -> small, us: reduction 1280, 2.03 tiles per CU 90 -> 78 and, transposed, 83 -> 71; reduction 2048, 2.25:
// 154 -> 134, 140 -> 121; 4096, 3.12: 390 -> 343, 344 -> 304; 640, 3.05: 73 -> 63, 60 -> 54; of 320 and less, 17 to 35 us,
// within 8 % either way), one that fills it by half or more is not (2.62: 156 -> 164, 2.00: 107 -> 128).  Ragged shapes have
// no other matrix-core kernel.
inline bool large_f32_tile(long tiles, long cus) {
  const long rounds = tiles / cus, rest = tiles % cus;
  return rounds >= 4 || (rounds >= 2 && (rest == 0 || 4 * rest > cus));
}
template <int EPI>
static hipError_t launch_f32_mfma(const GemmArgs& a, hipStream_t st) {
  const int tiles_m = (a.M + 63) / 64, tiles_n = (a.N + 63) / 64;
  const bool large = g_tile_cfg ? g_tile_cfg < 8 : large_f32_tile((long)tiles_m * tiles_n * a.n_groups, compute_units());
  if (a.N % 64 == 0 && a.K % 16 == 0 && large) {
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI>), dim3(tiles_m * tiles_n, 1, a.n_groups), dim3(256), 0, st, a,
                       tiles_m, tiles_n);
    return hipGetLastError();
  }
  const dim3 grid((a.M + 31) / 32 * ((a.N + 31) / 32), 1, a.n_groups);
  if (a.K % 64) hipLaunchKernelGGL((gemm_f32_small_kernel<EPI, true>), grid, dim3(256), 0, st, a, (a.N + 31) / 32);
  else hipLaunchKernelGGL((gemm_f32_small_kernel<EPI, false>), grid, dim3(256), 0, st, a, (a.N + 31) / 32);
  return hipGetLastError();
}

template <typename TA, int EPI>
static hipError_t launch_simple(const GemmArgs& a, hipStream_t st) {
  const int tiles_m = (a.M + 63) / 64, tiles_n = (a.N + 63) / 64;
  hipLaunchKernelGGL((gemm_simple_kernel<TA, EPI, TA>), dim3(tiles_m * tiles_n, 1, a.n_groups), dim3(256), 0,
                     st, a, tiles_m, tiles_n);
  return hipGetLastError();
}

// algorithmic HBM bytes of one grouped GEMM launch: operands once, outputs once, epilogue operands once
template <int EPI>
static double gemm_bytes(const GemmArgs& a, double esz) {
  const double G = a.n_groups, MN = (double)a.M * a.N;
  double b = G * ((a.a_slot_stride ? 1.0 : 1.0 / G) * a.M * a.K * esz + (double)a.N * a.K * esz);
  if (EPI == EPI_STORE) b += G * MN * esz;
  if (EPI == EPI_GELU || EPI == EPI_GELU_PRIME) b += G * MN * esz;
  if (EPI == EPI_GELU_BOTH) b += G * MN * esz * 2;
  if (EPI == EPI_DGELU) b += G * MN * esz * 2;
  if (EPI == EPI_STORE_F32) b += G * MN * 4;
  if (EPI == EPI_RESID_INNER) b += G * MN * 4 * (a.base ? 2 : 1);
  if (EPI == EPI_RESID_OUTER) b += G * MN * 4 * (a.RHS.present() ? 4 : 3);
  return b;
}

// Tile configurations of the MFMA kernel (k-tiles of 64) and what a round of each takes on MI355X, in
// microseconds: fixed + per_ktile * (k-tiles).  A launch runs in rounds of (CUs x resident blocks) tiles
// whose time hardly depends on how full the round is.  The epilogue is not in the model: for the tile it picks it is
// 11 % off in the median and 66 % at worst (fp32 epilogues of reductions of 384), yet over 64 shapes its pick is 0.7 %
// slower than the best tile on average and 16 % at worst (profiles/gemm_tile_round_times.txt):
//  1: 256x256, 8 wavefronts of 128x64, two stages: most reuse, what large launches run on;
//  3: 256x192, 8 wavefronts of 64x96, two stages: where 256 columns leave a round much emptier;
//  4: 128x128, two stages, two blocks per CU (one block's epilogue under the other's k loop);
//  6: 128x128, four stages, one block per CU: launches of up to one tile per CU, which wait for memory
//     latency and not for bandwidth (4096 x 768, reduction 3072: 51 us with two stages, 37 with four);
//  8: 64x64, four stages, two blocks per CU, and 9: two stages, four blocks per CU: few rows or columns.
struct TileCfg { int id, bm, bn, per_cu; double fixed, per_ktile; };
static const TileCfg kTileCfgs[] = {{1, 256, 256, 1, 7.0, 1.60}, {3, 256, 192, 1, 5.5, 1.33}, {4, 128, 128, 2, 2.7, 1.07},
                                    {6, 128, 128, 1, 2.5, 0.55}, {8, 64, 64, 2, 2.5, 0.375}, {9, 64, 64, 4, 2.5, 0.75}};
static int choose_tile_config(int n_groups, int M, int N, int K, double* cost_out = nullptr) {
  const long cus = compute_units();
  const int ktiles = (K + 63) / 64;
  int best = 4;
  double best_cost = 1e30;
  for (const TileCfg& c : kTileCfgs) {
    if (c.id == 3 && (N % 192 != 0 || K % 64 != 0)) continue;            // no ragged form
    const long tiles = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * n_groups;
    const long rounds = (tiles + cus * c.per_cu - 1) / (cus * c.per_cu);
    const double cost = rounds * (c.fixed + c.per_ktile * ktiles);
    if (cost < best_cost) { best_cost = cost; best = c.id; }
  }
  if (cost_out) *cost_out = best_cost;
  return best;
}

// Modelled time of one grouped launch (the driver sizes its launch chunks with it).
double gemm_model_cost(int n_groups, int M, int N, int K) {
  double c = 0.0;
  choose_tile_config(n_groups, M, N, K, &c);
  return c;
}

// RAGGED: N or K is no multiple of the tile (columns are clamped and guarded, the last k-tile's chunks
// past K read as zeros).
template <int EPI, bool RAGGED>
static hipError_t launch_cfg(int cfg, const GemmArgs& a, hipStream_t st) {
  switch (cfg) {
    case 1:
      if constexpr (!RAGGED && EPI == EPI_DGELU)
        if (dgelu_walks(a)) return launch_dgelu_walk(a, st);
      return launch_mfma<256, 256, 64, 2, 1, RAGGED, EPI, 2, 4>(a, st);
    case 3:
      if constexpr (!RAGGED) return launch_mfma<256, 192, 64, 2, 1, false, EPI, 4, 2>(a, st);
      break;
    case 6: return launch_mfma<128, 128, 64, 4, 1, RAGGED, EPI, 4, 2>(a, st);
    case 8: return launch_mfma<64, 64, 64, 4, 2, RAGGED, EPI, 2, 2>(a, st);
    case 9: return launch_mfma<64, 64, 64, 2, 4, RAGGED, EPI, 2, 2>(a, st);
    default: break;
  }
  // two blocks per CU; long reductions: 8 wavefronts of 32x64 (four per SIMD) hide the k-loop's latencies
  // better than 4 of 64x64; short ones are all epilogue, where 4 do better
  if (RAGGED || a.K >= 512) return launch_mfma<128, 128, 64, 2, 2, RAGGED, EPI, 4, 2>(a, st);
  return launch_mfma<128, 128, 64, 2, 2, false, EPI, 2, 2>(a, st);
}

template <int EPI>
static hipError_t launch_epi(const GemmArgs& a, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0 || a.M <= 0) return hipSuccess;
  const double flops = 2.0 * a.n_groups * a.M * (double)a.N * a.K;
  // the MFMA kernel moves 16-byte chunks and needs 32-bit element offsets
  const bool mfma_ok = is_bf16 && !g_force_simple && (a.K % 8 == 0) && (a.N % 8 == 0) &&
                       (double)a.M * a.K < 4e9 && (double)a.N * a.K < 4e9;
  const int cls = mfma_ok ? (a.n_groups > 1 ? PC_GEMM_MFMA : PC_GEMM_MFMA_SINGLE) + EPI : PC_GEMM_SIMPLE;
  ProfScope ps(cls, flops, gemm_bytes<EPI>(a, is_bf16 ? 2 : 4), st);
  if (!is_bf16) {
    // fp32: the matrix cores, with 16-byte accesses of both operands and of the epilogue's
    if (!g_force_simple && a.N % 4 == 0 && a.K % 4 == 0) return launch_f32_mfma<EPI>(a, st);
    return launch_simple<float, EPI>(a, st);
  }
  if (!mfma_ok) return launch_simple<bf16, EPI>(a, st);
  const int cfg = g_tile_cfg ? g_tile_cfg : choose_tile_config(a.n_groups, a.M, a.N, a.K);
  const int bn = cfg == 1 ? 256 : cfg == 3 ? 192 : cfg == 8 || cfg == 9 ? 64 : 128;
  const bool ragged = a.N % bn != 0 || a.K % 64 != 0;
  if (ragged && cfg == 3) return launch_cfg<EPI, true>(4, a, st);
  return ragged ? launch_cfg<EPI, true>(cfg, a, st) : launch_cfg<EPI, false>(cfg, a, st);
}

template <int BM, int BN, int STAGES, int WM, int WN, bool TAIL>
static hipError_t launch_tn_tile(const GemmTnArgs& a, int splits, hipStream_t st) {
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const int total = tiles_m * tiles_n * a.n_groups * splits, per_xcd = (total + 7) / 8;
  const size_t ring = (size_t)STAGES * (BM + BN) * 128;
  const size_t staging = (size_t)WM * WN * ((32 * (BN / WN * 4 + 16) + 1023) / 1024 * 1024);
  const size_t smem = ring > staging ? ring : staging;
  auto kern = gemm_tn_mfma_kernel<BM, BN, STAGES, WM, WN, TAIL>;
  static unsigned long raised = 0;
  if (const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), (int)smem, raised); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(64 * WM * WN), smem, st, a, tiles_m, tiles_n, splits, total, per_xcd);
  return hipGetLastError();
}

// TAIL: the last 64-token k-tile is not whole
template <int BM, int BN, int STAGES, int WM, int WN>
static hipError_t launch_tn(const GemmTnArgs& a, int splits, hipStream_t st) {
  return a.K % 64 ? launch_tn_tile<BM, BN, STAGES, WM, WN, true>(a, splits, st)
                  : launch_tn_tile<BM, BN, STAGES, WM, WN, false>(a, splits, st);
}

// Tile and number of token slices of a parameter-gradient product.  Microseconds of a round as in
// kTileCfgs, 17 % off in the median over 384 to 4096 wide outputs of 2048 to 12608 tokens, the pick 0.8 % slower than
// the best tile on average and 9 % at worst (profiles/gemm_tile_round_times.txt); a fragment takes two transposing
// 8-byte reads here instead of one of 16, so a k-tile takes longer than there.  Few output tiles and many tokens (384 x 384
// from 12608 tokens: 9 tiles of 128x128) are cut into slices of at least 8 k-tiles, which costs writing and summing the
// slices' partial results.
// Slices change the order of the sums, so their number follows from the layer's sizes alone, as the best one for a
// launch of TN_GROUPS layers (the usual chunk): a gradient does not depend on how many layers share its launch.  The
// tile may follow from the launch: every tile adds a slice's tokens in the same order.
constexpr int TN_GROUPS = 4;
struct TnPlan { int cfg, splits; };
static TnPlan choose_tn(int n_groups, int M, int N, int K, bool is_bf16, int first, int last) {
  static const TileCfg bf[] = {{1, 256, 256, 1, 7.0, 2.05}, {6, 128, 128, 1, 3.0, 0.68}, {8, 64, 64, 2, 2.5, 0.50}};
  static const TileCfg fp[] = {{0, 64, 64, 4, 2.5, 2.2}};
  const long cus = compute_units();
  const int ktiles = (K + 63) / 64;
  TnPlan best = {6, first};
  double best_cost = 1e30;
  for (const TileCfg* c = is_bf16 ? bf : fp; c != (is_bf16 ? bf + 3 : fp + 1); ++c) {
    const long tiles = (long)((M + c->bm - 1) / c->bm) * ((N + c->bn - 1) / c->bn) * n_groups;
    for (int s = first; s <= last && (s == first || ktiles / s >= 8); s *= 2) {
      const long rounds = (tiles * s + cus * c->per_cu - 1) / (cus * c->per_cu);
      double cost = rounds * (c->fixed + c->per_ktile * ((ktiles + s - 1) / s));
      if (s > 1) cost += 4.0 + 2.0 * s * n_groups * (double)M * N * 4.0 / 3e6;         // us at 3 TB/s
      if (cost < best_cost) { best_cost = cost; best = {c->id, s}; }
    }
  }
  return best;
}
static TnPlan plan_tn(int n_groups, int M, int N, int K, bool is_bf16) {
  const int ktiles = (K + 63) / 64;
  const int s = !g_grad_slices ? choose_tn(TN_GROUPS, M, N, K, is_bf16, 1, 64).splits
                               : g_grad_slices < ktiles ? g_grad_slices : ktiles;
  TnPlan p = choose_tn(n_groups, M, N, K, is_bf16, s, s);
  if (g_tile_cfg) p.cfg = g_tile_cfg == 1 ? 1 : g_tile_cfg < 8 ? 6 : 8;
  return p;
}

size_t gemm_tn_partial_floats(int n_groups, int M, int N, int K, bool is_bf16) {
  const int s = plan_tn(n_groups, M, N, K, is_bf16).splits;
  return s == 1 ? 0 : (size_t)s * n_groups * ((size_t)M * N + M);
}

hipError_t launch_gemm_tn(const GemmTnArgs& a, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0 || a.K <= 0) return hipSuccess;
  const double esz = is_bf16 ? 2 : 4, G = a.n_groups;
  if (a.M % 8 != 0 || a.N % 8 != 0 || 64.0 * a.M > 4e9 || 64.0 * a.N > 4e9) return hipErrorInvalidValue;
  const TnPlan plan = plan_tn(a.n_groups, a.M, a.N, a.K, is_bf16);
  if (plan.splits > 1 && !a.partial) return hipErrorInvalidValue;
  ProfScope ps(is_bf16 ? (a.n_groups > 1 ? PC_GEMM_MFMA : PC_GEMM_MFMA_SINGLE) + EPI_STORE_F32 : PC_GEMM_SIMPLE,
               2.0 * G * a.M * (double)a.N * a.K,
               G * ((double)a.K * (a.M + a.N) * esz + 4.0 * a.M * a.N), st);
  hipError_t e;
  if (!is_bf16) {
    const int tiles_m = (a.M + 63) / 64, tiles_n = (a.N + 63) / 64;
    hipLaunchKernelGGL(gemm_tn_f32_kernel, dim3(tiles_m * tiles_n, plan.splits, a.n_groups), dim3(256), 0, st, a,
                       tiles_n, plan.splits);
    e = hipGetLastError();
  } else {
    switch (plan.cfg) {
      case 1: e = launch_tn<256, 256, 2, 2, 4>(a, plan.splits, st); break;
      case 8: e = launch_tn<64, 64, 4, 2, 2>(a, plan.splits, st); break;
      default: e = launch_tn<128, 128, 4, 4, 2>(a, plan.splits, st); break;
    }
  }
  if (e != hipSuccess || plan.splits == 1) return e;
  const long each = (long)a.M * a.N + a.M;
  hipLaunchKernelGGL(gemm_tn_reduce_kernel, dim3((unsigned)((each / 4 + 255) / 256), a.n_groups), dim3(256), 0, st, a,
                     plan.splits);
  return hipGetLastError();
}

hipError_t launch_gemm(const GemmArgs& a, int epi, bool is_bf16, hipStream_t st) {
  switch (epi) {
    case EPI_STORE: return launch_epi<EPI_STORE>(a, is_bf16, st);
    case EPI_GELU: return launch_epi<EPI_GELU>(a, is_bf16, st);
    case EPI_RESID_INNER: return launch_epi<EPI_RESID_INNER>(a, is_bf16, st);
    case EPI_RESID_OUTER: return launch_epi<EPI_RESID_OUTER>(a, is_bf16, st);
    case EPI_DGELU: return launch_epi<EPI_DGELU>(a, is_bf16, st);
    case EPI_STORE_F32: return launch_epi<EPI_STORE_F32>(a, is_bf16, st);
    case EPI_GELU_PRIME: return launch_epi<EPI_GELU_PRIME>(a, is_bf16, st);
    case EPI_GELU_BOTH: return a.aux2 ? launch_epi<EPI_GELU_BOTH>(a, is_bf16, st) : hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

}  // namespace mg
