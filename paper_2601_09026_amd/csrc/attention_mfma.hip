// Fused softmax attention on the 32x32x16 bf16 MFMA (d_head = 64 or 128), forward and backward.
//
// Every product is arranged as  D[i][j] = sum_k A[i][k] B[k][j]  with the wavefront's own 32
// rows (queries in the forward and dQ kernels, keys in the dK/dV kernel) on the j axis.  In
// the MFMA result layout lane l then owns column j = l%32 and its 16 registers hold rows
// i = 8q + 4*(l/32) + r  (q, r = 0..3).  Consequences:
//   * the softmax statistics of a query are private to a lane (plus one exchange between
//     lanes l and l+32): no cross-lane reductions over the score tile;
//   * a score / probability tile, converted to bf16, already IS the B operand of the next
//     product (registers 8t..8t+7 feed k-step t), provided the A operand enumerates the
//     reduction index the same way: k-slot (half, e) <-> row 16t + 8*(e/4) + 4*half + e%4,
//     which is what two transposing LDS reads of a row-major tile deliver;
//   * per-row scalars (running max, denominator, lse, D) scale whole accumulators in place.
// A operands come from LDS, B operands stay in registers for the whole kernel.
//
// Forward :  S^T = K Q^T,  P^T = exp2(c S^T - m),  O^T += V^T P^T           (online softmax)
// dQ pass :  S^T, dP^T = V dO^T,  dA^T = P^T (dP^T - D),  dQ^T += K^T dA^T
// dKV pass:  S = Q K^T, dP = dO V^T, P, dA;  dV^T += dO^T P,  dK^T += Q^T dA
// No atomics: dQ and dK/dV are separate passes, so results are bit-reproducible.
//
// What bounds them: the chain of a wavefront, scores - exponentials - products, with three wavefronts per SIMD (d_head 64;
// the plain forward loop four) or two (128).  In a step of 8 x 512 tokens, heads of 64, the vector unit issues for 60 % of
// the forward kernel's cycles (a 32 x 32 unit of scores is 16 exponentials of 8 clocks and about 130 other instructions
// of 4) and the matrix cores work for 21 %; in the backward passes 26-29 % and 20-24 %; with one head of 128 the matrix
// cores work for 42 / 51 / 53 % (forward, dQ, dK/dV).  (Counter summaries of the two shapes under profiles/, where
// the counter of issue cycles counts in fours.)  Sequences of 128 tokens and fewer wait for memory instead.  Hence tiles
// straight from memory to LDS in one layout that serves the plain and the transposing reads (no transposed copy, no
// registers in between), and no scores for halves of a tile that no pair is in.  Microseconds per launch, with tiles
// staged through registers and transposed in LDS -> now, forward / whole backward: 5 layers of 8 x 512 causal, 12 heads of
// 64: 40 -> 39 / 137 -> 116; 5 of 64 x 197, 6 of 64: 57 -> 49 / 228 -> 170; 5 of 32 x 128, 12 of 64: 27.5 -> 26 / 82 -> 63;
// 6 of 64 x 64, 8 of 64: 23 -> 23 / 64 -> 45; 4 of 8 x 2048, one of 128: 82 -> 78 / 262 -> 221.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace mg {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

// LDS tiles: rows of DH bf16 as they lie in memory (global -> LDS directly, 16 bytes per lane), the 16-byte chunks of
// a row XOR-swizzled by its number so that one layout serves both reads without bank conflicts (64 banks of 4
// bytes): 16 consecutive rows at one chunk (the 16-byte reads of a row-major fragment) fall on 16 distinct slots, and
// so do 4 rows at 4 chunks (the transposing 8-byte reads).
template <int DH> struct Lay {
  static constexpr int RB = DH * 2, CPR = DH / 8, RPI = 1024 / RB;      // bytes and chunks per row; rows per load
  static constexpr int TILE = 64 * RB;                                  // bytes of 64 rows
  __device__ static __forceinline__ int swz(int row) {
    return DH == 64 ? (((row >> 1) & 1) << 2) | ((row >> 2) & 3) : ((row & 3) << 2) | ((row >> 2) & 3);
  }
};

// Keeps a value where it is computed: the optimiser moves arithmetic out of loops and past branches otherwise.
template <typename T> __device__ __forceinline__ void pin(T& v) { asm volatile("" : "+v"(v)); }

// Loads of NW wavefronts for 64 rows from row `row0` on (rows past the end repeat the last one).
// AGAIN: the lane's offsets are formed at each use instead of kept in 3 registers per load, for the dK/dV pass at d_head
// 128: its accumulators and own rows take 192 of 256 registers, and with the offsets kept 13 or 20 went to scratch (whole
// backward, 4 layers of 8 x 2048, one head: 246 -> 221 us, causal 209 -> 183; 5 of 16 x 300, 6 heads: 178 -> 150).
template <int NW, int DH, bool AGAIN = false, bool STREAM = false> struct Stager {
  using L = Lay<DH>;
  static constexpr int N = L::TILE / 1024 / NW;          // load instructions per wavefront and tile
  static_assert(N >= 1, "one load or more per wavefront");
  int wave, lane;
  int rs;                                                // bytes per row of the source
  __device__ __forceinline__ Stager(long row_stride, int wave_, int lane_)
      : wave(wave_), lane(lane_), rs((int)row_stride * 2) {}
  __device__ __forceinline__ void issue(unsigned char* dst, const bf16* src, int row0, int nrows) const {
    const auto base = lds_source(reinterpret_cast<const char*>(src) + (long)row0 * rs);
    const int left = nrows - 1 - row0;
    int l = lane;
    if constexpr (AGAIN) pin(l);
    auto load = [&](int j, bool whole) {
      const int r = (wave * N + j) * L::RPI + l / L::CPR, chunk = ((l % L::CPR) ^ L::swz(r)) * 16;
      load_to_lds<STREAM>(base, dst + (wave * N + j) * 1024, (whole || r < left ? r : left) * rs + chunk, 0);
    };
    if (left >= 63) {                                    // block-uniform
#pragma unroll
      for (int j = 0; j < N; ++j) load(j, true);
    } else {
#pragma unroll
      for (int j = 0; j < N; ++j) load(j, false);
    }
  }
};

// A operand of a product that reduces over features: row 32*rt + lane%32 of the tile, k-step ks
template <int DH> struct Frags {
  using L = Lay<DH>;
  int plain, trans;                                      // this lane's byte offsets, see below
  __device__ __forceinline__ explicit Frags(int lane) {
    const int lr = lane & 31, lh = lane >> 5;
    plain = lr * L::RB + ((lh ^ L::swz(lr)) << 4);
    const int tr = 4 * lh + ((lane & 15) >> 2);
    trans = tr * L::RB + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ L::swz(tr)) << 4) + (lane & 1) * 8;
  }
  // row 32*rt + l%32, features 16*ks + 8*(l/32) ..
  __device__ __forceinline__ bf16x8 rows(const lds_byte* tile, int rt, int ks) const {
    return lds_read16(tile + (plain ^ (ks << 5)) + 32 * rt * L::RB);
  }
  // feature 32*dt + l%32, reduction over the tile's rows 32*rt + 16*t .. in the register-order enumeration
  __device__ __forceinline__ bf16x8 cols(const lds_byte* tile, int rt, int t, int dt) const {
    const int lo = trans ^ (dt << 6);
    TrFrag f;
    f.lo = tr_read4(tile + lo + (32 * rt + 16 * t) * L::RB);
    f.hi = tr_read4(tile + (lo ^ 32) + (32 * rt + 16 * t + 8) * L::RB);
    return tr_value(f);
  }
};

// registers 8t..8t+7 of a result tile as the bf16 B operand of k-step t
__device__ __forceinline__ bf16x8 regs_to_b(const f32x16& v, int t) {
  bf16x8 r = {(bf16)v[8 * t], (bf16)v[8 * t + 1], (bf16)v[8 * t + 2], (bf16)v[8 * t + 3],
              (bf16)v[8 * t + 4], (bf16)v[8 * t + 5], (bf16)v[8 * t + 6], (bf16)v[8 * t + 7]};
  return r;
}
__device__ __forceinline__ f32x16 splat16(float x) {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = x;
  return z;
}
// 2^x as the bare hardware instruction: the library routine wraps it in a range reduction for
// results below 2^-126, which a probability that small does not need (it is 0 in bf16 anyway)
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }
// combination of a value with that of the lane 32 apart, on the vector unit
__device__ __forceinline__ float half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Ring of tile sets (64 rows of two operands each) in dynamic LDS, waited for by count: ring_turn() leaves PER_SET of
// this wavefront's loads in flight (`more`) or none, and from its barrier on the set before those is complete.
//  * The pipelined forward loop needs set it+1 while it works on set it: three slots (set `it` in slot it % 3).  It turns
//    to set it+1 with nothing left in flight, and set it+2 then takes the slot of set it-1, which nobody reads any more.
//  * All other loops use a set at a time: two slots, set it+1 on its way meanwhile, and a barrier behind the last read of
//    a slot before it is filled again; or one slot, where more blocks per compute unit hide the wait better.
// Heads of fewer sets are launched with that many slots and never come round (launch_ring()).
constexpr int RING = 3;                                  // of the pipelined loop
template <int PER_SET> __device__ __forceinline__ void ring_turn(bool more) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if (more) wait_vmcnt<PER_SET>();
  else wait_vmcnt<0>();
  bare_barrier();
}

struct HeadPtrs {
  const bf16 *Q, *K, *V, *O, *dO;
  bf16 *Ow, *dQ, *dK, *dV;
  float *lse, *D;
};

__device__ __forceinline__ HeadPtrs head_ptrs(const AttnArgs& a, int g, int b, int h) {
  HeadPtrs p;
  const int dh = a.dh;
  p.Q = reinterpret_cast<const bf16*>(a.q) + a.q_slots.of(g) * a.q_slot_stride + (long)b * a.Sq * a.q_row_stride + h * dh;
  p.K = reinterpret_cast<const bf16*>(a.k) + a.k_slots.of(g) * a.k_slot_stride + (long)b * a.Sk * a.k_row_stride + h * dh;
  p.V = reinterpret_cast<const bf16*>(a.v) + a.k_slots.of(g) * a.v_slot_stride + (long)b * a.Sk * a.v_row_stride + h * dh;
  p.O = reinterpret_cast<const bf16*>(a.o) + a.o_slots.of(g) * a.o_slot_stride + (long)b * a.Sq * a.o_row_stride + h * dh;
  p.Ow = const_cast<bf16*>(p.O);
  p.lse = a.lse ? a.lse + a.lse_slots.of(g) * a.lse_slot_stride + ((long)b * a.H + h) * a.Sq : nullptr;
  p.dO = nullptr; p.dQ = p.dK = p.dV = nullptr; p.D = nullptr;
  if (a.dO) {
    p.dO = reinterpret_cast<const bf16*>(a.dO) + a.do_slots.of(g) * a.do_slot_stride + (long)b * a.Sq * a.do_row_stride + h * dh;
    const long base = a.dqkv_slots.of(g) * a.dqkv_slot_stride;
    p.dQ = reinterpret_cast<bf16*>(a.dq) + base + (long)b * a.Sq * a.dqkv_row_stride + h * dh;
    if (a.dk) {
      const long kv_rs = a.dkv_row_stride ? a.dkv_row_stride : a.dqkv_row_stride;
      const long kv_base = a.dqkv_slots.of(g) * (a.dkv_slot_stride ? a.dkv_slot_stride : a.dqkv_slot_stride);
      p.dK = reinterpret_cast<bf16*>(a.dk) + kv_base + (long)b * a.Sk * kv_rs + h * dh;
      p.dV = reinterpret_cast<bf16*>(a.dv) + kv_base + (long)b * a.Sk * kv_rs + h * dh;
    }
    p.D = a.D + a.D_slots.of(g) * a.D_slot_stride + ((long)b * a.H + h) * a.Sq;
  }
  return p;
}

// store [DH features][32 rows] accumulators (transposed result) as rows of DH bf16
template <int DH>
__device__ __forceinline__ void store_rows_T(bf16* dst, long row_stride, int row, const f32x16* acc, float mul,
                                             int lh) {
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v = {acc[dt][4 * q] * mul, acc[dt][4 * q + 1] * mul, acc[dt][4 * q + 2] * mul, acc[dt][4 * q + 3] * mul};
      store4<bf16>(dst + (long)row * row_stride + 32 * dt + 8 * q + 4 * lh, v);
    }
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
// Wavefronts per SIMD the register budget is set for: the accumulators grow with DH.  d_head 64 holds three (168
// registers); the dQ and dK/dV passes with both operands' fragments fetched ahead spill there and lose more than the
// earlier reads gain (5 layers of 8 x 512: whole backward 119 -> 126 to 163 us).
template <int DH, int NW> constexpr int fa_waves() { return DH == 64 && NW == 4 ? 3 : DH == 64 || NW == 8 ? 2 : NW / 2; }

// LONG: the pipelined loop over a ring of three sets (the next unit's scores are begun before this one's exponentials, so
// that the matrix and the vector unit work at the same time); without it a fourth wavefront per SIMD fits at d_head 64 and
// one or two sets do (`slots`).  Same operations on the same numbers in the same order: which of the two runs may
// follow from the launch (attn_fwd_mfma_dh()).  The running maximum is exact: rescaling only when it grew by more than a
// threshold is faster and loses 4 % of the output's precision.
// STREAM: keys and values with the non-temporal hint.
template <int NW, int DH, bool LONG, bool STREAM = false>
__global__ void __launch_bounds__(NW * 64, (DH == 64 && !LONG ? 4 : fa_waves<DH, NW>()))
attn_fwd_mfma_kernel(const AttnArgs a, int slots) {
  using L = Lay<DH>;
  constexpr int KS = DH / 16, DT = DH / 32;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];         // ring of K and V tiles
  const BlockTask bt = block_task(a.causal, true);
  const int g = bt.g;
  const int b = bt.bh / a.H, h = bt.bh - b * a.H;
  const int q0 = bt.tile * (NW * 32);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const HeadPtrs P = head_ptrs(a, g, b, h);
  const int q_first = q0 + wave * 32, qi = q_first + lr;
  const int qc = qi < a.Sq ? qi : a.Sq - 1;
  const int k_end = a.causal ? min(a.Sk, min(q0 + NW * 32, a.Sq)) : a.Sk;        // keys the block needs
  const int w_end = q_first >= a.Sq ? 0 : a.causal ? min(a.Sk, q_first + 32) : a.Sk;   // ... and the wavefront
  const int n_blk = (k_end + 63) >> 6;
  const Stager<NW, DH, false, STREAM> sk(a.k_row_stride, wave, lane), sv(a.v_row_stride, wave, lane);
  auto stage = [&](int slot, int it) {
    sk.issue(smem + slot * 2 * L::TILE, P.K, it * 64, a.Sk);
    sv.issue(smem + slot * 2 * L::TILE + L::TILE, P.V, it * 64, a.Sk);
  };
  auto refill = [&](int slot, int it) {                  // once the block has read it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bare_barrier();
    stage(slot, it);
  };
  stage(0, 0);
  if (LONG && n_blk > 1) stage(1, 1);
  __builtin_amdgcn_sched_barrier(0);                     // (else own rows before set 1: their wait leaves it in flight)
  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8*>(P.Q + (long)qc * a.q_row_stride + 16 * ks + 8 * lh);
  __builtin_amdgcn_sched_barrier(0);
  if (!LONG && n_blk > 1 && slots > 1) stage(1, 1);
  const Frags<DH> fr(lane);
  const lds_byte* lds = (const lds_byte*)smem;
  const float c = rsqrtf((float)DH) * LOG2E;
  const int limit = (a.causal ? min(qi, a.Sk - 1) : a.Sk - 1) - 4 * lh;   // last key of this lane's query
  float m = -INFINITY, l = 0.f;                          // running maximum and denominator
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = splat16(0.f);

  // Unit j: 32 keys.  Step j multiplies the probabilities of unit j with its values and forms the scores of unit j+1, one
  // stream of matrix instructions in fixed order with everything else placed between them: the fragment of each is
  // read RD instructions ahead, the exponentials of unit j stand under the scores of unit j+1 and the first products,
  // the maximum of unit j+1 under the last products.  Left to the compiler the two units ran one after the other.
  constexpr int RD = 4, NOPS = KS + 2 * DT;
  bf16x8 ring[RD];
  float ms = 0.f, corr = 1.f;                            // what the exponentials of the unit at hand refer to
  const lds_byte *Kc = lds, *Kn = lds;                   // key tiles of this set and the next
  auto new_max = [&](const f32x16& s) {                  // of the raw scores; the scale c is positive
    float x = fmaxf(s[0], s[1]);
#pragma unroll
    for (int i = 2; i < 16; ++i) x = fmaxf(x, s[i]);
    const float mn = fmaxf(m, half_max(x) * c);
    ms = mn == -INFINITY ? 0.f : mn;                     // fully masked so far: keep exp2 finite
    corr = exp2_raw(m - ms);
    m = mn;
  };
  auto step = [&](auto rt_tag, f32x16& s, f32x16& sn) {
    constexpr int rt = decltype(rt_tag)::value;
    const lds_byte* V = Kc + L::TILE;
    // fragment of instruction n of this step (from NOPS on: of the next step)
    auto read = [&](int n) {
      if (n < KS) return fr.rows(rt == 0 ? Kc : Kn, rt == 0 ? 1 : 0, n);
      if (n < NOPS) return fr.cols(V, rt, (n - KS) / DT, (n - KS) % DT);
      return fr.rows(Kn, rt == 0 ? 0 : 1, n - NOPS);
    };
    float t[2] = {0.f, 0.f};
    auto prob = [&](int i) {
      s[i] = exp2_raw(fmaf(s[i], c, -ms));
      t[i & 1] += s[i];
    };
#pragma unroll
    for (int n = 0; n < KS; ++n) {
      sn = MFMA(ring[n % RD], qf[n], n == 0 ? splat16(0.f) : sn);
      ring[n % RD] = read(n + RD);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (i >= 8 * n / KS && i < 8 * (n + 1) / KS) prob(i);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        if (dt >= DT * n / KS && dt < DT * (n + 1) / KS) o[dt] *= corr;
      __builtin_amdgcn_sched_barrier(0);
    }
    bf16x8 pb = regs_to_b(s, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = KS; n < NOPS; ++n) {
      const int dt = (n - KS) % DT;
      if (n == KS + DT) {
        pb = regs_to_b(s, 1);
        l = fmaf(l, corr, t[0] + t[1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      o[dt] = MFMA(ring[n % RD], pb, o[dt]);
      ring[n % RD] = read(n + RD);
      if (n < KS + DT) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (i >= 8 * dt / DT && i < 8 * (dt + 1) / DT) prob(8 + i);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (n == KS + DT) new_max(sn);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // iterations whose two steps only meet whole units of keys that every query of the wavefront attends to
  const int whole = a.causal ? min(w_end, q_first) >> 5 : w_end >> 5;
  const int fast = LONG && whole > 2 ? (whole - 1) >> 1 : 0;
  // first unit behind that loop, whose denominator is rounded once more: the other form does the same
  const int hand_over = !LONG && a.Sk > 128 && whole > 2 ? (whole - 1) & ~1 : -1;
  int slot = 0, it = 0;
  if (LONG) ring_turn<2 * Stager<NW, DH>::N>(n_blk > 1);           // set 0
  if (LONG && fast > 0) {
    f32x16 sa = splat16(0.f), sb;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) sa = MFMA(fr.rows(lds, 0, ks), qf[ks], sa);
    new_max(sa);
#pragma unroll
    for (int n = 0; n < RD; ++n) ring[n] = fr.rows(lds, 1, n);
    for (; it < fast; ++it) {                            // (set it+1 exists: unit 2*it+2 is in it)
      const int next = slot == RING - 1 ? 0 : slot + 1;
      ring_turn<0>(false);                               // set it+1
      if (it + 2 < n_blk) stage(next == RING - 1 ? 0 : next + 1, it + 2);
      Kc = lds + slot * 2 * L::TILE;
      Kn = lds + next * 2 * L::TILE;
      step(std::integral_constant<int, 0>{}, sa, sb);
      step(std::integral_constant<int, 1>{}, sb, sa);
      slot = next;
    }
    l *= corr;                                           // the next unit is formed once more below
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
  }
  for (; it < n_blk; ++it) {
    const int next = slot == (LONG ? RING : slots) - 1 ? 0 : slot + 1;
    if (LONG) {                                          // (in step with wavefronts that are still in the loop above)
      if (it + 1 < n_blk) ring_turn<0>(false);
      if (it + 2 < n_blk) stage(next == RING - 1 ? 0 : next + 1, it + 2);
    } else {
      ring_turn<2 * Stager<NW, DH>::N>(slots > 1 && it + 1 < n_blk);
    }
    const lds_byte* K = lds + slot * 2 * L::TILE;
    for (int rt = 0; rt < 2; ++rt) {
      const int k0 = it * 64 + 32 * rt;
      if (k0 >= w_end) break;
      const lds_byte *Kh = K + 32 * rt * L::RB, *Vh = Kh + L::TILE;
      f32x16 s = splat16(0.f);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = MFMA(fr.rows(Kh, 0, ks), qf[ks], s);
      // masked scores become -inf, whose exp2 is 0
      if (k0 + 32 > a.Sk || (a.causal && k0 + 31 > q_first)) {
        const int lim = limit - k0;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 8 * (i >> 2) + (i & 3) <= lim ? s[i] : -INFINITY;
      }
      new_max(s);
      float t[2] = {0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = exp2_raw(fmaf(s[i], c, -ms));
        t[i & 1] += s[i];
      }
      const float lu = t[0] + t[1];
      float two = l * corr;
      if (!LONG) pin(two);                               // (a product of its own)
      l = fmaf(l, corr, lu);
      if (!LONG && 2 * it + rt == hand_over) l = two + lu;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        const bf16x8 pb = regs_to_b(s, t2);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] = MFMA(fr.cols(Vh, 0, t2, dt), pb, o[dt]);
      }
    }
    if (!LONG && it + slots < n_blk) refill(slot, it + slots);
    slot = next;
  }
  l = half_sum(l);
  if (qi < a.Sq) {
    store_rows_T<DH>(P.Ow, a.o_row_stride, qi, o, 1.0f / l, lh);
    if (P.lse && lh == 0) P.lse[qi] = (m + log2f(l)) * LN2;
  }
}

// ---------------------------------------------------------------------------
// backward: the products of 32 own rows with 32 rows of a tile
// ---------------------------------------------------------------------------
// dQ pass: own queries (fragments qf, dof, scalars lse2 = lse * log2(e), neg_d = -D), key half `rt` of the tiles K, V.
// lim: last of the 32 keys this lane's query may attend to, less 4 * (lane / 32); masked: some pair is masked
template <int DH>
__device__ __forceinline__ void bwd_dq_half(const Frags<DH>& fr, const lds_byte* K, const lds_byte* V, int rt,
                                            const bf16x8 (&qf)[DH / 16], const bf16x8 (&dof)[DH / 16], float c, float lse2,
                                            float neg_d, bool masked, int lim, f32x16 (&dq)[DH / 32]) {
  f32x16 s = splat16(0.f), dp = splat16(neg_d);          // dP - D comes out of the matrix unit
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    s = MFMA(fr.rows(K, rt, ks), qf[ks], s);
    dp = MFMA(fr.rows(V, rt, ks), dof[ks], dp);
  }
  if (masked) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 8 * (i >> 2) + (i & 3) <= lim ? s[i] : -INFINITY;
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = exp2_raw(fmaf(s[i], c, -lse2)) * dp[i];      // dA^T
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bf16x8 ab = regs_to_b(s, t);
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) dq[dt] = MFMA(fr.cols(K, rt, t, dt), ab, dq[dt]);
  }
}

// dK/dV pass: own keys (fragments kf, vf), query half `rt` of the tiles Q, dO.  row_s, row_d: per query -lse / scale and
// -D, what the two products start from (rows that do not exist: -inf and 0, so that P = dA = 0).
// first: the first of the 32 queries that may attend to this lane's key, less 4 * (lane / 32)
template <int DH>
__device__ __forceinline__ void bwd_dkv_half(const Frags<DH>& fr, const lds_byte* Q, const lds_byte* dO, int rt,
                                             const float* row_s, const float* row_d, const bf16x8 (&kf)[DH / 16],
                                             const bf16x8 (&vf)[DH / 16], float c, bool masked, int first, int lh,
                                             f32x16 (&dk)[DH / 32], f32x16 (&dv)[DH / 32]) {
  f32x16 s, dp;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(row_s + 32 * rt + 8 * q + 4 * lh);
    const f32x4 y = *reinterpret_cast<const f32x4*>(row_d + 32 * rt + 8 * q + 4 * lh);
#pragma unroll
    for (int r = 0; r < 4; ++r) { s[4 * q + r] = x[r]; dp[4 * q + r] = y[r]; }
  }
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    s = MFMA(fr.rows(Q, rt, ks), kf[ks], s);
    dp = MFMA(fr.rows(dO, rt, ks), vf[ks], dp);
  }
  if (masked) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 8 * (i >> 2) + (i & 3) >= first ? s[i] : -INFINITY;
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    s[i] = exp2_raw(s[i] * c);                           // P
    dp[i] *= s[i];                                       // dA
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bf16x8 pb = regs_to_b(s, t), ab = regs_to_b(dp, t);
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) {
      dv[dt] = MFMA(fr.cols(dO, rt, t, dt), pb, dv[dt]);
      dk[dt] = MFMA(fr.cols(Q, rt, t, dt), ab, dk[dt]);
    }
  }
}

// D of this lane's query (both halves of the wavefront get the sum)
template <int DH>
__device__ __forceinline__ float row_dot(const bf16x8 (&dof)[DH / 16], const bf16* o, int lh) {
  float d = 0.f;
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    const bf16x8 of = *reinterpret_cast<const bf16x8*>(o + 16 * ks + 8 * lh);
#pragma unroll
    for (int e = 0; e < 8; ++e) d = fmaf((float)dof[ks][e], (float)of[e], d);
  }
  return half_sum(d);
}

template <int NW, int DH>
__global__ void __launch_bounds__(NW * 64, (fa_waves<DH, NW>())) attn_bwd_dq_mfma_kernel(const AttnArgs a) {
  using L = Lay<DH>;
  constexpr int KS = DH / 16, DT = DH / 32;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];         // ring of K and V tiles
  const BlockTask bt = block_task(a.causal, true);
  const int g = bt.g;
  const int b = bt.bh / a.H, h = bt.bh - b * a.H;
  const int q0 = bt.tile * (NW * 32);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const HeadPtrs P = head_ptrs(a, g, b, h);
  const int q_first = q0 + wave * 32, qi = q_first + lr;
  const int qc = qi < a.Sq ? qi : a.Sq - 1;
  const int k_end = a.causal ? min(a.Sk, min(q0 + NW * 32, a.Sq)) : a.Sk;
  const int w_end = q_first >= a.Sq ? 0 : a.causal ? min(a.Sk, q_first + 32) : a.Sk;
  const int n_blk = (k_end + 63) >> 6;
  const Stager<NW, DH> sk(a.k_row_stride, wave, lane), sv(a.v_row_stride, wave, lane);
  auto stage = [&](int slot, int it) {
    sk.issue(smem + slot * 2 * L::TILE, P.K, it * 64, a.Sk);
    sv.issue(smem + slot * 2 * L::TILE + L::TILE, P.V, it * 64, a.Sk);
  };
  auto refill = [&](int slot, int it) {                  // once the block has read it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bare_barrier();
    stage(slot, it);
  };
  stage(0, 0);
  if (n_blk > 1) stage(1, 1);
  bf16x8 qf[KS], dof[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qf[ks] = *reinterpret_cast<const bf16x8*>(P.Q + (long)qc * a.q_row_stride + 16 * ks + 8 * lh);
    dof[ks] = *reinterpret_cast<const bf16x8*>(P.dO + (long)qc * a.do_row_stride + 16 * ks + 8 * lh);
  }
  const float D = row_dot<DH>(dof, P.O + (long)qc * a.o_row_stride, lh);
  const float lse2 = P.lse[qc] * LOG2E;
  const Frags<DH> fr(lane);
  const lds_byte* lds = (const lds_byte*)smem;
  const float c = rsqrtf((float)DH) * LOG2E;
  const int limit = (a.causal ? min(qi, a.Sk - 1) : a.Sk - 1) - 4 * lh;
  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dq[dt] = splat16(0.f);
  int slot = 0;
  for (int it = 0; it < n_blk; ++it) {
    ring_turn<2 * Stager<NW, DH>::N>(it + 1 < n_blk);
    const lds_byte* K = lds + slot * 2 * L::TILE;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const int k0 = it * 64 + 32 * kt;
      if (k0 < w_end)                                    // wave-uniform
        bwd_dq_half<DH>(fr, K, K + L::TILE, kt, qf, dof, c, lse2, -D, k0 + 32 > a.Sk || (a.causal && k0 + 31 > q_first),
                        limit - k0, dq);
    }
    if (it + 2 < n_blk) refill(slot, it + 2);
    slot ^= 1;
  }
  if (qi < a.Sq) {
    if (lh == 0) P.D[qi] = D;                            // (not earlier: the first tile's wait would cover the store)
    store_rows_T<DH>(P.dQ, a.dqkv_row_stride, qi, dq, rsqrtf((float)DH), lh);
  }
}

template <int NW, int DH>
__global__ void __launch_bounds__(NW * 64, (fa_waves<DH, NW>())) attn_bwd_dkv_mfma_kernel(const AttnArgs a) {
  using L = Lay<DH>;
  constexpr int KS = DH / 16, DT = DH / 32;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];         // ring of Q and dO tiles
  __shared__ __attribute__((aligned(16))) float rows[2][2][64];               // -lse / scale and -D of their queries
  const BlockTask bt = block_task(a.causal, false);
  const int g = bt.g;
  const int b = bt.bh / a.H, h = bt.bh - b * a.H;
  const int j0 = bt.tile * (NW * 32);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const HeadPtrs P = head_ptrs(a, g, b, h);
  const int k_first = j0 + wave * 32, kj = k_first + lr;
  const int kc = kj < a.Sk ? kj : a.Sk - 1;
  bf16x8 kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    kf[ks] = *reinterpret_cast<const bf16x8*>(P.K + (long)kc * a.k_row_stride + 16 * ks + 8 * lh);
    vf[ks] = *reinterpret_cast<const bf16x8*>(P.V + (long)kc * a.v_row_stride + 16 * ks + 8 * lh);
  }
  constexpr bool AGAIN = DH == 128;
  const Stager<NW, DH, AGAIN> sq(a.q_row_stride, wave, lane), so(a.do_row_stride, wave, lane);
  auto stage = [&](int slot, int it) {
    sq.issue(smem + slot * 2 * L::TILE, P.Q, it * 64, a.Sq);
    so.issue(smem + slot * 2 * L::TILE + L::TILE, P.dO, it * 64, a.Sq);
  };
  auto refill = [&](int slot, int it) {                  // once the block has read it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bare_barrier();
    stage(slot, it);
  };
  float st_s = 0.f, st_d = 0.f;                          // on their way to `rows` (first wavefront)
  auto fetch_rows = [&](int it) {
    const int qq = it * 64 + lane;
    st_s = qq < a.Sq ? P.lse[qq] * -sqrtf((float)DH) : -INFINITY;
    st_d = qq < a.Sq ? -P.D[qq] : 0.f;
  };
  auto publish = [&](int slot) { rows[slot][0][lane] = st_s; rows[slot][1][lane] = st_d; };
  // causal: key j only receives from queries i >= j
  const int it0 = a.causal ? j0 >> 6 : 0, n_blk = (a.Sq + 63) >> 6;
  if (wave == 0) { fetch_rows(it0); publish(0); }
  if (it0 < n_blk) stage(0, it0);
  if (it0 + 1 < n_blk) stage(1, it0 + 1);
  if (wave == 0) fetch_rows(it0 + 1);
  const Frags<DH> fr(lane);
  const lds_byte* lds = (const lds_byte*)smem;
  const float c = rsqrtf((float)DH) * LOG2E;
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) { dk[dt] = splat16(0.f); dv[dt] = splat16(0.f); }
  int slot = 0;
  for (int it = it0; it < n_blk; ++it) {
    ring_turn<2 * Stager<NW, DH>::N>(it + 1 < n_blk);
    if (wave == 0 && it + 1 < n_blk) publish(slot ^ 1);  // before the barrier that opens set it+1
    if (wave == 0 && it + 2 < n_blk) fetch_rows(it + 2);
    const lds_byte* Q = lds + slot * 2 * L::TILE;
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const int i0 = it * 64 + 32 * qt;
      // wave-uniform: queries exist, one of them may attend to these keys, the keys exist
      if (i0 < a.Sq && (!a.causal || i0 + 31 >= k_first) && k_first < a.Sk)
        bwd_dkv_half<DH>(fr, Q, Q + L::TILE, qt, rows[slot][0], rows[slot][1], kf, vf, c, a.causal && i0 < k_first + 31,
                         kj - i0 - 4 * lh, lh, dk, dv);
    }
    if (it + 2 < n_blk) refill(slot, it + 2);
    slot ^= 1;
  }
  if (kj < a.Sk) {
    const long kv_rs = a.dkv_row_stride ? a.dkv_row_stride : a.dqkv_row_stride;
    store_rows_T<DH>(P.dK, kv_rs, kj, dk, rsqrtf((float)DH), lh);
    store_rows_T<DH>(P.dV, kv_rs, kj, dv, 1.0f, lh);
  }
}

// Sequences that fit one block (Sq, Sk <= 32 NW): both passes in one launch, the head's Q, K, V and dO in LDS as a
// whole, read from memory once; nothing waits between the two passes but the exchange of D.  Two wavefronts per SIMD at
// d_head 64: with three the dK/dV half spills.
template <int NW, int DH>
__global__ void __launch_bounds__(NW * 64, (DH == 64 ? 2 : 1)) attn_bwd_fused_mfma_kernel(const AttnArgs a) {
  using L = Lay<DH>;
  constexpr int KS = DH / 16, DT = DH / 32, TILES = NW / 2, OPND = TILES * L::TILE;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * OPND];        // K, V, Q, dO
  __shared__ __attribute__((aligned(16))) float rows[2][NW * 32];
  const int g = blockIdx.z, b = blockIdx.y / a.H, h = blockIdx.y - b * a.H;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const HeadPtrs P = head_ptrs(a, g, b, h);
  {
    const Stager<NW, DH> sk(a.k_row_stride, wave, lane), sv(a.v_row_stride, wave, lane), sq(a.q_row_stride, wave, lane),
        so(a.do_row_stride, wave, lane);
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      if (t * 64 < a.Sk) {
        sk.issue(smem + t * L::TILE, P.K, t * 64, a.Sk);
        sv.issue(smem + OPND + t * L::TILE, P.V, t * 64, a.Sk);
      }
      if (t * 64 < a.Sq) {
        sq.issue(smem + 2 * OPND + t * L::TILE, P.Q, t * 64, a.Sq);
        so.issue(smem + 3 * OPND + t * L::TILE, P.dO, t * 64, a.Sq);
      }
    }
  }
  const Frags<DH> fr(lane);
  const lds_byte* lK = (const lds_byte*)smem;
  const lds_byte *lV = lK + OPND, *lQ = lK + 2 * OPND, *lO = lK + 3 * OPND;
  const float c = rsqrtf((float)DH) * LOG2E;
  const int first = wave * 32, own = first + lr;         // this lane's query, then its key
  const int qc = own < a.Sq ? own : a.Sq - 1;
  bf16x8 of[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) of[ks] = *reinterpret_cast<const bf16x8*>(P.O + (long)qc * a.o_row_stride + 16 * ks + 8 * lh);
  const float lse = P.lse[qc];
  ring_turn<0>(false);
  bf16x8 fa[KS], fb[KS];
  if (first < a.Sq) {                                    // wave-uniform
    float D = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      fa[ks] = fr.rows(lQ, wave, ks);
      fb[ks] = fr.rows(lO, wave, ks);
#pragma unroll
      for (int e = 0; e < 8; ++e) D = fmaf((float)fb[ks][e], (float)of[ks][e], D);
    }
    D = half_sum(D);
    if (lh == 0) {
      rows[0][own] = own < a.Sq ? lse * -sqrtf((float)DH) : -INFINITY;
      rows[1][own] = own < a.Sq ? -D : 0.f;
    }
    const int w_end = a.causal ? min(a.Sk, first + 32) : a.Sk;
    const int limit = (a.causal ? min(own, a.Sk - 1) : a.Sk - 1) - 4 * lh;
    f32x16 dq[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) dq[dt] = splat16(0.f);
    for (int k0 = 0; k0 < w_end; k0 += 32)
      bwd_dq_half<DH>(fr, lK + k0 * L::RB, lV + k0 * L::RB, 0, fa, fb, c, lse * LOG2E, -D,
                      k0 + 32 > a.Sk || (a.causal && k0 + 31 > first), limit - k0, dq);
    if (own < a.Sq) store_rows_T<DH>(P.dQ, a.dqkv_row_stride, own, dq, rsqrtf((float)DH), lh);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  bare_barrier();                                        // every row's lse and D are there
  if (first >= a.Sk) return;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) { fa[ks] = fr.rows(lK, wave, ks); fb[ks] = fr.rows(lV, wave, ks); }
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) { dk[dt] = splat16(0.f); dv[dt] = splat16(0.f); }
  for (int i0 = a.causal ? first : 0; i0 < a.Sq; i0 += 32)
    bwd_dkv_half<DH>(fr, lQ + i0 * L::RB, lO + i0 * L::RB, 0, rows[0] + i0, rows[1] + i0, fa, fb, c,
                     a.causal && i0 < first + 31, own - i0 - 4 * lh, lh, dk, dv);
  if (own < a.Sk) {
    const long kv_rs = a.dkv_row_stride ? a.dkv_row_stride : a.dqkv_row_stride;
    store_rows_T<DH>(P.dK, kv_rs, own, dk, rsqrtf((float)DH), lh);
    store_rows_T<DH>(P.dV, kv_rs, own, dv, 1.0f, lh);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
bool attn_mfma_supported(const AttnArgs& a) {
  return (a.dh == 64 || a.dh == 128) && (a.q_row_stride % 8 == 0) && (a.k_row_stride % 8 == 0) &&
         (a.v_row_stride % 8 == 0) && (a.o_row_stride % 8 == 0);
}

// Blocks of 256 rows halve the K/V (Q/dO) bytes staged from L2 per flop.  Mask bits 0-2: forward, dQ pass, dK/dV pass
// at d_head = 128, from 129 tokens on; the two backward passes keep 128-row blocks when the last 256-row block would be at
// most half full.  Bits 4-6: the same at d_head = 64 from 512 tokens on.  Milliseconds of a training step of 8 x 2048
// tokens, one head of 128: all three 148.4; without the forward pass's 153.5, the dQ pass's 154.3, the dK/dV pass's 192.0,
// any 204.2.  8 x 512 tokens, 12 heads of 64 (three wavefronts per SIMD in 128-row blocks, two in these): none 179.0,
// forward 179.3, dQ 180.5, dK/dV 181.3, all 182.5.
int g_attn_wide = 7;
void attn_set_wide_blocks(int mask) { g_attn_wide = mask & 0x77; }
template <int DH> static bool attn_wide(int pass, int seq) {
  if (DH == 64) return seq >= 512 && ((g_attn_wide >> (4 + pass)) & 1);
  if (!((g_attn_wide >> pass) & 1) || seq <= 128) return false;
  const int tail = seq % 256;
  return pass == 0 || tail == 0 || tail > 128;
}

// Launch with a ring of as many tile sets as `seq` rows make, `most` at most.  fixed: bytes of LDS that the kernel
// declares itself; a block of more than 64 KB in all needs the limit of its dynamic part raised (two sets at d_head 128
// are 64 KB: the dK/dV kernel's rows come on top).
template <int DH, typename Kernel>
static hipError_t launch_ring(Kernel kern, int block_rows, int own_rows, int seq, const AttnArgs& a, hipStream_t st,
                              int most, size_t fixed = 0) {
  const int sets = (seq + 63) / 64, slots = sets < most ? sets : most;
  const size_t smem = (size_t)slots * 2 * Lay<DH>::TILE;
  if (smem + fixed > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((own_rows + block_rows - 1) / block_rows, a.B * a.H, a.n_groups), block(2 * block_rows);
  if constexpr (std::is_invocable_v<Kernel, AttnArgs, int>) hipLaunchKernelGGL(kern, grid, block, smem, st, a, slots);
  else hipLaunchKernelGGL(kern, grid, block, smem, st, a);
  return hipGetLastError();
}

template <int DH>
static hipError_t attn_fwd_mfma_dh(const AttnArgs& a, hipStream_t st) {
  if (a.Sq <= 0 || a.Sk <= 0) return hipErrorInvalidValue;
  if (attn_wide<DH>(0, a.Sq)) return launch_ring<DH>(attn_fwd_mfma_kernel<8, DH, true>, 256, a.Sq, a.Sk, a, st, RING);
  const int rows = a.Sq <= 64 ? 64 : 128;
  const long blocks = (long)((a.Sq + rows - 1) / rows) * a.B * a.H * a.n_groups;
  // How many sets a block gets decides how many blocks a compute unit holds (160 KB of LDS).  The pipelined loop hides the
  // chain of a block by itself and pays as long as all blocks run at once: 1024 keys, 64 queries, blocks of the launch
  // 256 / 512 / 1024, microseconds with one set -> three: d_head 64 27 -> 18, 32 -> 27, 49 -> 61; d_head 128 45 -> 36,
  // 63 -> 70, 115 -> 143.  Beyond that, one set: other blocks hide the waits.  Exceptions: 128 queries at d_head 64
  // have enough wavefronts in three blocks, and from about 450 keys on the pipelined loop is ahead there again (4096
  // blocks: 512 causal 74 -> 76 us, 512 not causal 103 -> 99, 2048 100 -> 95); d_head 128 with a few blocks more than fit
  // (512: 63 -> 59) or long memories keeps two.  Up to 128 keys, the whole head in two sets where that does not cost
  // blocks, or where a head is read from memory once (32 x 128 tokens, 12 heads, 5 layers: 27.5 -> 26.2; causal 27.6 with two,
  // 26.0 with one).
  auto at_once = [&](int sets) { return blocks <= compute_units() * (163840L / (sets * 2 * Lay<DH>::TILE)); };
  int sets;
  if (a.Sk <= 128) sets = at_once(2) || (DH == 64 && !a.causal && a.Sq <= 128) ? 2 : 1;
  else if (at_once(RING) || (DH == 64 && rows == 128 && (a.causal ? (a.Sk + 128) / 2 : a.Sk) > 448)) sets = RING;
  else sets = DH == 128 && (at_once(2) || (rows == 128 && a.Sk >= 512)) ? 2 : 1;
  const bool pipelined = sets == RING;
  // One block of queries per head reads its keys and values once.  Where they exceed the memory-side cache (256 MB) by far,
  // such launches are bound by HBM and faster if nothing is kept: 2048 heads of 64, 64 queries on 2048 keys (1.07 GB) 226 -> 201
  // us, 16 on 800 (0.42 GB) 85 -> 76; d_head 128, 1024 heads, 64 on 2048 213 -> 183.  At 0.27 GB 49 -> 50, below up to 30 % slower.
  const double kv_bytes = 4.0 * a.Sk * DH * a.B * a.H * a.n_groups;
  if (rows == 64 && !pipelined && kv_bytes > 300e6)
    return launch_ring<DH>(attn_fwd_mfma_kernel<2, DH, false, true>, 64, a.Sq, a.Sk, a, st, sets);
  if (rows == 64)
    return launch_ring<DH>(pipelined ? attn_fwd_mfma_kernel<2, DH, true> : attn_fwd_mfma_kernel<2, DH, false>, 64, a.Sq, a.Sk,
                           a, st, sets);
  return launch_ring<DH>(pipelined ? attn_fwd_mfma_kernel<4, DH, true> : attn_fwd_mfma_kernel<4, DH, false>, 128, a.Sq, a.Sk,
                         a, st, sets);
}

hipError_t attn_fwd_mfma(const AttnArgs& a, hipStream_t st) {
  return a.dh == 64 ? attn_fwd_mfma_dh<64>(a, st) : attn_fwd_mfma_dh<128>(a, st);
}

template <int DH>
static hipError_t attn_bwd_mfma_dh(const AttnArgs& a, hipStream_t st) {
  if (a.Sq <= 0 || a.Sk <= 0) return hipErrorInvalidValue;
  if (a.dk && a.Sq <= 128 && a.Sk <= 128) {
    dim3 grid(1, a.B * a.H, a.n_groups);
    if (a.Sq <= 64 && a.Sk <= 64) hipLaunchKernelGGL((attn_bwd_fused_mfma_kernel<2, DH>), grid, dim3(128), 0, st, a);
    else hipLaunchKernelGGL((attn_bwd_fused_mfma_kernel<4, DH>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
  }
  // Two sets: a third one gains nothing for a block (within 2 % at 64 to 2048 rows) and costs a resident block: 64 queries on
  // 192 keys, 1024 blocks, dQ pass 17.7 us with two, 20.4 with three at d_head 64; 19.1 and 25.3 at 128 (512 blocks).
  hipError_t e;
  if (a.Sq <= 64) e = launch_ring<DH>(attn_bwd_dq_mfma_kernel<2, DH>, 64, a.Sq, a.Sk, a, st, 2);
  else if (attn_wide<DH>(1, a.Sq)) e = launch_ring<DH>(attn_bwd_dq_mfma_kernel<8, DH>, 256, a.Sq, a.Sk, a, st, 2);
  else e = launch_ring<DH>(attn_bwd_dq_mfma_kernel<4, DH>, 128, a.Sq, a.Sk, a, st, 2);
  if (e != hipSuccess || !a.dk) return e;        // only dQ wanted (cross-attention: dK, dV feed the memory gradient)
  constexpr size_t rows = sizeof(float) * 2 * 2 * 64;      // the kernel's own
  if (a.Sk <= 64) return launch_ring<DH>(attn_bwd_dkv_mfma_kernel<2, DH>, 64, a.Sk, a.Sq, a, st, 2, rows);
  if (attn_wide<DH>(2, a.Sk)) return launch_ring<DH>(attn_bwd_dkv_mfma_kernel<8, DH>, 256, a.Sk, a.Sq, a, st, 2, rows);
  return launch_ring<DH>(attn_bwd_dkv_mfma_kernel<4, DH>, 128, a.Sk, a.Sq, a, st, 2, rows);
}

hipError_t attn_bwd_mfma(const AttnArgs& a, hipStream_t st) {
  return a.dh == 64 ? attn_bwd_mfma_dh<64>(a, st) : attn_bwd_mfma_dh<128>(a, st);
}

}  // namespace mg
