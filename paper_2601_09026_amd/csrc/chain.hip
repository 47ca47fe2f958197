// Row-local chains of a narrow layer (64 or 128 wide, bf16), one launch each:
//   head          LN1(X) and the Q | K | V projection
//   tail          output projection -> ybar -> LN2(X + ybar) -> both feed-forward products -> Euler update
//   adjoint_tail  transposes of the feed-forward products and of LN2, and of the output projection
//   adjoint_head  transposes of the Q | K | V projection and of LN1, and the Euler update
// What bounds these layers launch by launch is the traffic between the launches (a product of reduction 128 does 64
// flops a byte) and, with few tokens, the number of dependent launches.
//
// A wavefront owns 32 token rows and keeps them in registers from one end of the chain to the other: with the weights as
// the first MFMA operand a result has one row per lane, so that LayerNorm statistics are sums inside a lane and one exchange
// between the wavefront's halves, and a result becomes the next product's operand by packing and two half exchanges per
// 16 features.  The weights pass through a ring of 8 KB tiles in LDS that the wavefronts of a block share.
//
// 4 layers of 16384 tokens, 128 wide, 128 hidden, launch by launch -> chain: head 34 -> 22 us (84 MB, 3.8 TB/s), tail
// 65 -> 29 us (117 MB, 4.1 TB/s), adjoint_tail from fp32 cotangents 63 -> 28 us (117 MB, 4.1 TB/s), adjoint_head 53 -> 37 us
// (168 MB, 4.5 TB/s), where a copy reaches 5.8 TB/s.  What bounds them are their rows' traffic and its waits: the blocks of a
// launch start and end together, so that loads, products and stores hardly overlap, and two wavefronts a SIMD wait to issue
// for 39 to 73 % of their cycles with the matrix cores 7 to 13 % busy.
// With 512 hidden features (tail 48, adjoint_tail 43 us) the GELU, 14 vector instructions a value, takes as long as the traffic.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "lds_limit.h"
#include "prof.h"

namespace mg {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

// f(std::integral_constant<int, 0>) .. f(std::integral_constant<int, N - 1>)
template <int I, int N, typename F> __device__ __forceinline__ void each_from(F& f) {
  if constexpr (I < N) { f(std::integral_constant<int, I>{}); each_from<I + 1, N>(f); }
}
template <int N, typename F> __device__ __forceinline__ void each(F f) { each_from<0, N>(f); }
using ic0 = std::integral_constant<int, 0>;

__device__ __forceinline__ f32x4 lds_read4f(const lds_byte* __restrict__ p) {
  typedef const __attribute__((address_space(3))) f32x4* ptr;
  return *(ptr)p;
}
__device__ __forceinline__ unsigned pack2(float a, float b) {
  const bf16x2 r = {(bf16)a, (bf16)b};
  return __builtin_bit_cast(unsigned, r);
}
// 16 features of a lane's row: as a result they lie 0..3 and 8..11 in lanes 0..31, 4..7 and 12..15 in lanes 32..63; as an
// operand and in memory 0..7 and 8..15.  w0 .. w3 packed pairs in the order of either.
__device__ __forceinline__ u32x4 swap_halves(unsigned w0, unsigned w1, unsigned w2, unsigned w3) {
  const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
  return u32x4{a[0], b[0], a[1], b[1]};
}
__device__ __forceinline__ bf16x8 operand_of(f32x4 a, f32x4 b) {
  return __builtin_bit_cast(bf16x8, swap_halves(pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]), pack2(b[2], b[3])));
}
__device__ __forceinline__ float low_of(unsigned w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float high_of(unsigned w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
__device__ __forceinline__ void quads_of(bf16x8 o, f32x4& a, f32x4& b) {
  const u32x4 w = __builtin_bit_cast(u32x4, o);
  const u32x4 r = swap_halves(w[0], w[1], w[2], w[3]);
  a = f32x4{low_of(r[0]), high_of(r[0]), low_of(r[1]), high_of(r[1])};
  b = f32x4{low_of(r[2]), high_of(r[2]), low_of(r[3]), high_of(r[3])};
}
__device__ __forceinline__ f32x4 quad(const f32x16& c, int q) { return f32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]}; }
// keeps a value where it is computed: beside the products of that place
__device__ __forceinline__ void pin(float& a) { asm volatile("" : "+v"(a)); }
__device__ __forceinline__ void pin(unsigned& a) { asm volatile("" : "+v"(a)); }

// Packed bf16 rows of one group as a buffer whose end is the last row's: rows past it read as zeros, stores to them are dropped.
struct RowBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ RowBuf(const void* base, long bytes) {
    const unsigned long p = (unsigned long)base;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
    r = __builtin_amdgcn_make_buffer_rsrc((void*)((unsigned long)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane((unsigned)bytes),
                                          0x00020000);
  }
  __device__ __forceinline__ bf16x8 load(int off) const {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  }
  __device__ __forceinline__ void store(int off, bf16x8 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, 0);
  }
};

// ---------------------------------------------------------------------------
// Ring of weight tiles.  A tile is two blocks of 32 rows by 64 reduction indices (128-byte rows, 16-byte chunks swizzled by
// the row pair); a set of eight products takes its fragments block by block, k-step by k-step, six products ahead of
// their use.  Set i loads tile i + LEAD; every G-th set waits for the tiles of the next G sets, by count, and meets the
// block's other wavefronts, after which nobody reads the tiles before set i any more.
// Those counts (TILES, and LATER: loads and stores of rows behind the tiles) hold only while the compiler keeps every
// instruction that they count; tests/test_chain_waits.py reads the built kernels for it.
// ---------------------------------------------------------------------------
constexpr int RING_G = 2, RING_LEAD = 6, RING_R = RING_LEAD + RING_G, RING_BYTES = RING_R * 8192;
constexpr int RING_BEHIND = RING_LEAD - RING_G - 1;          // tiles asked for behind those waited for

// One matrix that tiles are taken from: 64 rows x 64 reduction indices, or (WIDE) 32 x 128.
template <int NW, bool WIDE> struct Matrix {
  static constexpr int LPT = 8 / NW;                       // load instructions of a wavefront per tile
  __amdgpu_buffer_rsrc_t src;
  int v[LPT];
  __device__ __forceinline__ Matrix(const void* base, int ld, int wave, int lane) : src(lds_source(base)) {
    const int lrow = lane >> 3, lpos = lane & 7;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int j = wave * LPT + i, r = 8 * (WIDE ? j & 3 : j) + lrow;
      v[i] = (r * ld + (WIDE ? j >> 2 : 0) * 64 + (lpos ^ ((r >> 1) & 7)) * 8) * 2;
    }
  }
  __device__ __forceinline__ void load(unsigned char* dst, int wave, int off) const {
#pragma unroll
    for (int i = 0; i < LPT; ++i) load_to_lds(src, dst + (wave * LPT + i) * 1024, v[i], off);
  }
};

template <int NW> struct Ring {
  static constexpr int LPT = 8 / NW;
  unsigned char *put, *first, *last;
  const lds_byte *cur, *nxt;
  int foff[4];
  bf16x8 fr[8];
  __device__ __forceinline__ void init(unsigned char* mem, int lane) {
    const int lr = lane & 31, lh = lane >> 5;
    first = put = mem;
    last = mem + RING_BYTES;
    cur = nxt = (const lds_byte*)mem;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) foff[ks] = lr * 128 + (((2 * ks + lh) ^ ((lr >> 1) & 7)) << 4);
  }
  __device__ __forceinline__ void step_put() { put = put + 8192 == last ? first : put + 8192; }
  __device__ __forceinline__ void read(int m, const lds_byte* from) { fr[m] = lds_read16(from + (m >> 2) * 4096 + foff[m & 3]); }
  __device__ __forceinline__ void prime() {
#pragma unroll
    for (int m = 0; m < 6; ++m) read(m, cur);
  }
  // Waits are by count, i.e. for all but the N youngest of the wavefront's loads and stores: TILES tiles and LATER others.
  template <int TILES, int LATER> __device__ __forceinline__ void wait() {
    wait_vmcnt<LPT * TILES + LATER>();
    bare_barrier();
  }
  // the first two of the first RING_LEAD tiles are there, the other loads behind these may not be
  template <int LATER = 0> __device__ __forceinline__ void start() {
    wait<RING_LEAD - 2, LATER>();
    prime();
  }
  // SYNC: the last of G sets.  TILES: tiles asked for behind those that the next G sets need.
  template <bool SYNC, int TILES, int LATER, typename L> __device__ __forceinline__ void turn(L load) {
    if constexpr (SYNC) wait<TILES, LATER>();
    load();
    step_put();
    const lds_byte* n = cur + 8192;
    nxt = n == (const lds_byte*)last ? (const lds_byte*)first : n;
    __builtin_amdgcn_sched_barrier(0);
  }
  template <bool SYNC, int TILES, int LATER, typename L, typename M, typename X>
  __device__ __forceinline__ void set(L load, M mul, X extra) {
    each<8>([&](auto mt) {
      constexpr int m = decltype(mt)::value;
      if constexpr (m == 2) turn<SYNC, TILES, LATER>(load);
      mul(mt, fr[m]);
      if constexpr (m + 6 < 8) read(m + 6, cur); else read(m - 2, nxt);
      extra(mt);
      __builtin_amdgcn_sched_barrier(0);
    });
    cur = nxt;
  }
  // a tile that is passed over (what was read ahead of it is dropped)
  template <bool SYNC, int LATER, typename L> __device__ __forceinline__ void pass(L load) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    turn<SYNC, RING_BEHIND, LATER>(load);
    cur = nxt;
  }
};
__device__ __forceinline__ void mfma(f32x16& c, bf16x8 w, bf16x8 x, bool fresh) {
  const f32x16 z = {};
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, fresh ? z : c, 0, 0, 0);
}

// fp32 vectors of a parameter block into LDS, 1 KB (of what follows the vector as well) per load; returns where the next goes
constexpr int vec_bytes(int n) { return (n * 4 + 1023) & ~1023; }
template <int NW> __device__ __forceinline__ unsigned char* vector_to_lds(unsigned char* dst, const char* src, int n, int wave, int lane) {
  const auto r = lds_source(src);
  const int bytes = vec_bytes(n);
  for (int o = wave * 1024; o < bytes; o += NW * 1024) load_to_lds(r, dst + o, lane * 16, o);
  return dst + bytes;
}
__device__ __forceinline__ float both_halves(float v) { return v + __shfl_xor(v, 32, 64); }

// The block's place in the launch: consecutive blocks of an XCD work on one layer.
struct Place { int g, row0, wave, lane; bool none; };
template <int NW> __device__ __forceinline__ Place place(int tiles_m, int total, int per_xcd) {
  Place p;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  p.none = tile >= total;
  p.g = __builtin_amdgcn_readfirstlane(tile / tiles_m);
  p.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  p.lane = threadIdx.x & 63;
  p.row0 = (__builtin_amdgcn_readfirstlane(tile - p.g * tiles_m) * NW + p.wave) * 32;
  return p;
}

// ---------------------------------------------------------------------------
// Activations between the two products: 32 hidden features of the wavefront's rows, two values at a time, in ITEMS
// parts of about four instructions that run beside the products; a fragment of 16 features is done after each half.
// ---------------------------------------------------------------------------
// GELU (gelu_fast of common.h, taken apart with its constants); BOTH: its derivative (gelu_prime_fast) as well
template <bool BOTH> struct Gelu {
  static constexpr int ST = BOTH ? 9 : 7, ITEMS = 8 * ST;
  static constexpr bool LAG = true;
  static constexpr int LATER = BOTH ? 3 : 0;               // its stores in a chunk's time, from the second chunk on
  const lds_byte* bias;                                    // of the features at hand, this half's quads
  f32x4 b, bn;
  float z0, z1, x0, x1, t0, t1, p0, p1, e0, e1;
  unsigned w[4], d[4];
  int col;                                                 // byte column of the features at hand in act / dact
  RowBuf act, dact;                                        // where to leave them
  bool keep;                                               // act is wanted
  int rowoff;
  __device__ __forceinline__ void begin() { bn = lds_read4f(bias); }
  __device__ __forceinline__ void next() { bias += 128; col += 64; }
  template <int it> __device__ __forceinline__ void item(const f32x16& acc, bf16x8* out) {
    constexpr int i = it / ST, st = it % ST, q = i >> 1, e = 2 * (i & 1);
    if constexpr (st == 0) {
      if constexpr (e == 0) { b = bn; if constexpr (q < 3) bn = lds_read4f(bias + (q + 1) * 32); }
      z0 = acc[4 * q + e] + b[e]; z1 = acc[4 * q + e + 1] + b[e + 1];
      x0 = z0 * SQRT_HALF; x1 = z1 * SQRT_HALF;
    } else if constexpr (st == 1) {
      x0 = __builtin_amdgcn_fmed3f(x0, -PHI_CLAMP, PHI_CLAMP); x1 = __builtin_amdgcn_fmed3f(x1, -PHI_CLAMP, PHI_CLAMP);
      t0 = x0 * x0; t1 = x1 * x1;
    } else if constexpr (st == 2) {
      two(PHI_POLY[0], PHI_POLY[1], PHI_POLY[2], true);
    } else if constexpr (st == 3) {
      two(0.f, PHI_POLY[3], PHI_POLY[4], false);
    } else if constexpr (st == 4) {
      two(0.f, PHI_POLY[5], PHI_POLY[6], false);
    } else if constexpr (st == 5) {
      p0 = fmaf(p0, t0, PHI_POLY[7]); p1 = fmaf(p1, t1, PHI_POLY[7]);
      p0 = fmaf(x0, p0, 0.5f); p1 = fmaf(x1, p1, 0.5f);
    } else if constexpr (st == 6) {
      w[i & 3] = pack2(z0 * p0, z1 * p1);
      if constexpr ((i & 3) == 3) {
        out[i >> 2] = __builtin_bit_cast(bf16x8, swap_halves(w[0], w[1], w[2], w[3]));
        if (BOTH && keep) act.store(rowoff + col + (i >> 2) * 32, out[i >> 2]);
      }
    } else if constexpr (st == 7) {
      e0 = __builtin_amdgcn_exp2f(z0 * z0 * PDF_EXP2); e1 = __builtin_amdgcn_exp2f(z1 * z1 * PDF_EXP2);
    } else {
      d[i & 3] = pack2(fmaf(z0, PDF_SCALE * e0, p0), fmaf(z1, PDF_SCALE * e1, p1));
      if constexpr ((i & 3) == 3) dact.store(rowoff + col + (i >> 2) * 32, __builtin_bit_cast(bf16x8, swap_halves(d[0], d[1], d[2], d[3])));
    }
  }
  __device__ __forceinline__ void two(float c0, float c1, float c2, bool first) {
    p0 = fmaf(first ? c0 : p0, t0, c1); p1 = fmaf(first ? c0 : p1, t1, c1);
    p0 = fmaf(p0, t0, c2); p1 = fmaf(p1, t1, c2);
  }
};

// Product with the cached derivative, read 64 features ahead.
template <int D> struct DGelu {
  static constexpr int ST = 2, ITEMS = 8 * ST;
  static constexpr bool LAG = false;
  static constexpr int LATER = D == 128 ? 4 : 8;           // its loads in the time of RING_LEAD - 2 sets
  RowBuf g, dz;
  bool keep;                                               // dz is wanted
  int rowoff, col;
  bf16x8 now[2], ahead[2], later[2];
  unsigned gw[4], w[4];
  float y0, y1;
  __device__ __forceinline__ void fetch(bf16x8* to, int c) {
#pragma unroll
    for (int k = 0; k < 2; ++k) to[k] = g.load(rowoff + c + 32 * k);
  }
  __device__ __forceinline__ void first() { col = 0; fetch(ahead, 0); fetch(later, 64); }
  __device__ __forceinline__ void begin() {
#pragma unroll
    for (int k = 0; k < 2; ++k) { now[k] = ahead[k]; ahead[k] = later[k]; }
    fetch(later, col + 128);                               // (past the last feature: another row's, or zeros)
  }
  __device__ __forceinline__ void next() { col += 64; }
  template <int it> __device__ __forceinline__ void item(const f32x16& acc, bf16x8* out) {
    constexpr int i = it / ST, st = it % ST, v = 2 * i;
    if constexpr (st == 0) {
      if constexpr ((i & 3) == 0) {
        const u32x4 n = __builtin_bit_cast(u32x4, now[i >> 2]);
        const u32x4 r = swap_halves(n[0], n[1], n[2], n[3]);
#pragma unroll
        for (int k = 0; k < 4; ++k) gw[k] = r[k];
      }
      y0 = acc[v] * low_of(gw[i & 3]); y1 = acc[v + 1] * high_of(gw[i & 3]);
      pin(y0); pin(y1);
    } else {
      w[i & 3] = pack2(y0, y1);
      pin(w[i & 3]);
      if constexpr ((i & 3) == 3) {
        out[i >> 2] = __builtin_bit_cast(bf16x8, swap_halves(w[0], w[1], w[2], w[3]));
        if (keep) dz.store(rowoff + col + (i >> 2) * 32, out[i >> 2]);
      }
    }
  }
};

// ---------------------------------------------------------------------------
// Two products with an activation between them:  acc += act(u A^T) B^T,  A [F, D], B [D, F], 64 hidden features (a chunk)
// at a time.  The tiles follow Q0 others in the ring and are followed by AFTER tiles of C [D, D] (those of A's form).
// LAG: the activation of a chunk, long as it is, runs beside the products of the next chunk with A and of the former one with
// B, which comes one chunk later in the ring; else beside the chunk's own.  DOWN = false: the first product and the
// activation alone.
// ---------------------------------------------------------------------------
template <int D, int NW, int Q0, bool DOWN, int AFTER, typename Act> struct Pair {
  static constexpr int SB = D / 64, PC = DOWN ? 2 * SB : SB;     // tiles per chunk: A's, then B's
  static constexpr bool WIDE = D == 128, LAG = DOWN && Act::LAG;
  static constexpr int STEP = WIDE ? 32 : 64;                    // features of a tile of A or C
  Matrix<NW, WIDE> A;
  Matrix<NW, false> B;
  __amdgpu_buffer_rsrc_t C;
  int P, F, wave;                                                // P chunks
  __device__ __forceinline__ Pair(const void* a, const void* b, const void* c, int f, int wave_, int lane)
      : A(a, D, wave_, lane), B(b, f, wave_, lane), C(lds_source(c)), P(f / 64), F(f), wave(wave_) {}
  __device__ __forceinline__ int last() const { return LAG ? P : P - 1; }
  // The tile `i` places after the first one of chunk p, or of C; behind the last one some tile again: a test whether there
  // is one would cut the products' code in pieces.  (With LAG A's of chunk P and B's of chunk -1 are loaded as well and
  // passed over.)
  __device__ __forceinline__ void tile(unsigned char* dst, int i, int p) const {
    const int np = p + i / PC, pos = i % PC;
    int off;
    if (pos < SB) {
      const int q = np < P ? np : P - 1;
      off = (q * 64 + pos * STEP) * D * 2;
    } else {
      const int q = LAG ? (np > 0 ? np <= P ? np - 1 : P - 1 : 0) : np < P ? np : P - 1;
      off = ((pos - SB) * 64 * F + q * 64) * 2;
    }
    if constexpr (AFTER == 0) {
      if (pos < SB) A.load(dst, wave, off);
      else B.load(dst, wave, off);
    } else {
      const bool over = np > last();
      const int q = (np - last() - 1) * PC + pos;
      if (over) off = (q < AFTER ? q : AFTER - 1) * STEP * D * 2;
#pragma unroll
      for (int k = 0; k < 8 / NW; ++k) {
        const int v = pos < SB || over ? A.v[k] : B.v[k];
        load_to_lds(over ? C : pos < SB ? A.src : B.src, dst + (wave * (8 / NW) + k) * 1024, v, off);
      }
    }
  }

  __device__ __forceinline__ void run(Ring<NW>& R, const bf16x8 (&U)[D / 16], f32x16 (&acc)[D / 32], Act& act) const {
    f32x16 ua[2];
    bf16x8 H[4], Hx[LAG ? 4 : 1];
    constexpr int I = Act::ITEMS;
    auto nothing = [](auto) {};
    // part `slot` of `slots` of items FIRST .. FIRST + N - 1
    auto some = [&](auto slot, auto slots, auto first, auto n, const f32x16& z, bf16x8* out) {
      constexpr int S = decltype(slot)::value, M = decltype(slots)::value, N = decltype(n)::value;
      constexpr int lo = S * N / M, hi = (S + 1) * N / M;
      each<hi - lo>([&](auto k) { act.template item<decltype(first)::value + lo + decltype(k)::value>(z, out); });
    };
    using Lo = ic0; using Hi = std::integral_constant<int, I / 2>; using Half = Hi; using Whole = std::integral_constant<int, I>;
    using In8 = std::integral_constant<int, 8>; using In4 = std::integral_constant<int, 4>; using In1 = std::integral_constant<int, 1>;
    using I1 = std::integral_constant<int, 1>;
    int p = 0;
    // late: other loads and stores behind the tiles waited for
    auto set = [&](auto post, auto late, auto mul, auto extra) {
      constexpr int pos = decltype(post)::value;
      R.template set<(Q0 + pos) % RING_G == RING_G - 1, RING_BEHIND, decltype(late)::value>([&] { tile(R.put, pos + RING_LEAD, p); }, mul, extra);
    };
    auto pass = [&](auto first, auto late) {
      each<SB>([&](auto k) {
        constexpr int pos = decltype(first)::value + decltype(k)::value;
        R.template pass<(Q0 + pos) % RING_G == RING_G - 1, decltype(late)::value>([&] { tile(R.put, pos + RING_LEAD, p); });
      });
      R.prime();
    };
    auto up = [&](auto h, auto late, auto extra) {               // WIDE: 32 features, else all 64
      if constexpr (WIDE) set(h, late, [&](auto m, bf16x8 w) { mfma(ua[decltype(h)::value], w, U[m], m == 0); }, extra);
      else set(h, late, [&](auto m, bf16x8 w) { mfma(ua[m >> 2], w, U[m & 3], (m & 3) == 0); }, extra);
    };
    auto down = [&](auto st, auto late, auto extra) {
      constexpr int s = decltype(st)::value;
      set(std::integral_constant<int, SB + s>{}, late, [&](auto m, bf16x8 w) { mfma(acc[2 * s + (m >> 2)], w, H[m & 3], false); }, extra);
    };
    auto on = [&] { act.next(); act.begin(); };
    using Late = std::integral_constant<int, Act::LATER>;
    act.begin();
    if constexpr (!DOWN) {
      auto chunk = [&](auto late, auto former) {
        if constexpr (WIDE) {
          up(ic0{}, late, former);
          up(I1{}, late, [&](auto m) { some(m, In8{}, Lo{}, Whole{}, ua[0], H); });
          on();
        } else {
          up(ic0{}, late, nothing);
          some(ic0{}, In1{}, Lo{}, Whole{}, ua[0], H); on();
          some(ic0{}, In1{}, Lo{}, Whole{}, ua[1], H); on();
        }
      };
      chunk(ic0{}, nothing);
      for (p = 1; p < P; ++p)
        chunk(Late{}, [&](auto m) {
          some(m, In8{}, Lo{}, Whole{}, ua[1], H);
          if constexpr (decltype(m)::value == 7) on();
        });
      if constexpr (WIDE) some(ic0{}, In1{}, Lo{}, Whole{}, ua[1], H);
    } else if constexpr (!LAG) {
      for (p = 0; p < P; ++p) {
        if constexpr (WIDE) {
          up(ic0{}, Late{}, nothing);
          up(I1{}, Late{}, [&](auto m) { some(m, In8{}, Lo{}, Whole{}, ua[0], H); });
        } else {
          up(ic0{}, Late{}, nothing);
          some(ic0{}, In1{}, Lo{}, Whole{}, ua[0], H);
        }
        on();
        some(ic0{}, In1{}, Lo{}, Whole{}, ua[1], H + 2);
        each<SB>([&](auto s) { down(s, Late{}, nothing); });
        on();
      }
    } else if constexpr (WIDE) {
      up(ic0{}, ic0{}, nothing);
      up(I1{}, ic0{}, [&](auto m) { some(m, In8{}, Lo{}, Half{}, ua[0], H); });
      some(ic0{}, In1{}, Hi{}, Half{}, ua[0], H);
      on();
      some(ic0{}, In1{}, Lo{}, Half{}, ua[1], H + 2);
      pass(std::integral_constant<int, SB>{}, ic0{});
      for (p = 1; p < P; ++p) {
        up(ic0{}, Late{}, [&](auto m) { some(m, In8{}, Hi{}, Half{}, ua[1], H + 2); });
        on();
        up(I1{}, Late{}, [&](auto m) { some(m, In8{}, Lo{}, Half{}, ua[0], Hx); });
        down(ic0{}, Late{}, [&](auto m) { some(m, In8{}, Hi{}, Half{}, ua[0], Hx); });
        on();
        down(I1{}, Late{}, [&](auto m) { some(m, In8{}, Lo{}, Half{}, ua[1], Hx + 2); });
#pragma unroll
        for (int k = 0; k < 3; ++k) H[k] = Hx[k];
      }
      some(ic0{}, In1{}, Hi{}, Half{}, ua[1], H + 2);
      pass(ic0{}, ic0{});
      down(ic0{}, ic0{}, nothing);
      down(I1{}, ic0{}, nothing);
    } else {
      up(ic0{}, ic0{}, nothing);
      some(ic0{}, In1{}, Lo{}, Whole{}, ua[0], H); on();
      some(ic0{}, In1{}, Lo{}, Whole{}, ua[1], H + 2);
      pass(I1{}, ic0{});
      for (p = 1; p < P; ++p) {
        on();
        up(ic0{}, Late{}, nothing);
        down(ic0{}, Late{}, [&](auto m) {
          constexpr int k = decltype(m)::value;
          if constexpr (k == 4) on();
          if constexpr (k < 4) some(m, In4{}, Lo{}, Whole{}, ua[0], Hx);
          else some(std::integral_constant<int, k - 4>{}, In4{}, Lo{}, Whole{}, ua[1], Hx + 2);
        });
#pragma unroll
        for (int k = 0; k < 4; ++k) H[k] = Hx[k];
      }
      pass(ic0{}, ic0{});
      down(ic0{}, ic0{}, nothing);
    }
  }
};

// ---------------------------------------------------------------------------
// tail.  MODE 0: the step alone; 1: the layer's entries of the linearisation cache, no state; 2: both.
// ---------------------------------------------------------------------------
template <int D, int NW, int MODE>
__global__ void __launch_bounds__(64 * NW, 2) chain_tail_kernel(const ChainTailArgs a, int tiles_m, int total, int per_xcd) {
  constexpr int SB = D / 64, NB = D / 32, KS = D / 16, NQ = D / 8, Q0 = SB * SB;
  constexpr bool KEEP_X = D == 64;
  using Ffn = Pair<D, NW, Q0, MODE != 1, 0, Gelu<MODE != 0>>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const Place pl = place<NW>(tiles_m, total, per_xcd);
  if (pl.none) return;
  const int lane = pl.lane, lr = lane & 31, lh = lane >> 5, g = pl.g, T = a.T, F = a.f;
  const int row = pl.row0 + lr, crow = row < T ? row : T - 1;
  const char* pb = a.P.at(g);
  const Matrix<NW, false> Wo(pb + a.wo_off, D, pl.wave, lane);
  const Ffn ffn(pb + a.w1_off, pb + a.w2_off, pb, F, pl.wave, lane);
  Ring<NW> R;
  R.init(smem, lane);
  auto load_at = [&](int i) {                                    // tile i: Wo's, then the chunks'
    if (i < Q0) Wo.load(R.put, pl.wave, (i / SB * 64 * D + i % SB * 64) * 2);
    else ffn.tile(R.put, i - Q0, 0);
  };

  bf16x8 U[KS];
  {
    const bf16* op = reinterpret_cast<const bf16*>(a.o) + a.o_slots.of(g) * a.o_slot_stride + (long)crow * D + 8 * lh;
#pragma unroll
    for (int k = 0; k < KS; ++k) U[k] = ld_global(reinterpret_cast<const bf16x8*>(op + 16 * k));
  }
  constexpr int V = vec_bytes(D);                                // bo, gamma, beta, b2, b1
  {
    unsigned char* v = smem + RING_BYTES;
    v = vector_to_lds<NW>(v, pb + a.bo_off, D, pl.wave, lane);
    v = vector_to_lds<NW>(v, pb + a.g_off, D, pl.wave, lane);
    v = vector_to_lds<NW>(v, pb + a.be_off, D, pl.wave, lane);
    v = vector_to_lds<NW>(v, pb + a.b2_off, D, pl.wave, lane);
    vector_to_lds<NW>(v, pb + a.b1_off, F, pl.wave, lane);
  }
  const lds_byte* vec = (const lds_byte*)smem + RING_BYTES + 16 * lh;
#pragma unroll
  for (int i = 0; i < RING_LEAD; ++i) { load_at(i); R.step_put(); }
  __builtin_amdgcn_sched_barrier(0);
  const float* xr = a.X.at(g) + (long)crow * D + 4 * lh;
  f32x4 v[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) v[i] = ld_global(reinterpret_cast<const f32x4*>(xr + 8 * i));
  __builtin_amdgcn_sched_barrier(0);
  R.template start<NQ>();

  f32x16 acc[NB];
  each<Q0>([&](auto qt) {                                        // o Wo^T
    constexpr int q = decltype(qt)::value;
    R.template set<q % RING_G == RING_G - 1, RING_BEHIND, NQ>([&] { load_at(q + RING_LEAD); }, [&](auto m, bf16x8 w) {
      mfma(acc[2 * (q / SB) + (m >> 2)], w, U[4 * (q % SB) + (m & 3)], q % SB == 0 && (m & 3) == 0);
    }, [](auto) {});
  });

  // u = LN2(X + ybar)
  f32x4 xk[KEEP_X ? NQ : 1];
  const long cs = a.cs.of(g);
  const RowBuf bxh(MODE ? (const bf16*)a.xhat + cs * T * D : nullptr, MODE ? 2L * T * D : 0);
  const RowBuf bu(MODE && a.u ? (const bf16*)a.u + cs * T * D : nullptr, MODE && a.u ? 2L * T * D : 0);
  {
    const float* br = a.base ? a.base + a.base_slots.of(g) * a.base_slot_stride + (long)crow * D + 4 * lh : nullptr;
    float* yr = MODE && a.ybar && row < T ? a.ybar + (cs * T + row) * D + 4 * lh : nullptr;
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      f32x4 y = quad(acc[i >> 2], i & 3) + lds_read4f(vec + 32 * i);
      if (br) y += ld_global(reinterpret_cast<const f32x4*>(br + 8 * i));
      if (MODE && yr) *reinterpret_cast<f32x4*>(yr + 8 * i) = y;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i >> 2][4 * (i & 3) + e] = y[e];
      if constexpr (KEEP_X) xk[i] = v[i];
      v[i] += y;
      part[i & 3] += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
    }
    const float mu = both_halves((part[0] + part[1]) + (part[2] + part[3])) / D;
    float sq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      v[i] = v[i] - mu;
      sq[i & 3] += (v[i][0] * v[i][0] + v[i][1] * v[i][1]) + (v[i][2] * v[i][2] + v[i][3] * v[i][3]);
    }
    const float rstd = 1.0f / sqrtf(both_halves((sq[0] + sq[1]) + (sq[2] + sq[3])) / D + a.eps);
    if (MODE && row < T && lh == 0) a.rstd[cs * T + row] = rstd;
    const int ro = row * D * 2 + 16 * lh;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      f32x4 w[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) w[h] = v[2 * k + h] * rstd;
      if constexpr (MODE != 0) bxh.store(ro + 32 * k, operand_of(w[0], w[1]));
#pragma unroll
      for (int h = 0; h < 2; ++h) w[h] = w[h] * lds_read4f(vec + V + 32 * (2 * k + h)) + lds_read4f(vec + 2 * V + 32 * (2 * k + h));
      U[k] = operand_of(w[0], w[1]);
      if (MODE != 0) if (a.u) bu.store(ro + 32 * k, U[k]);
    }
  }

  // m = gelu(u W1^T + b1) W2^T, added to ybar
  Gelu<MODE != 0> act{vec + 4 * V, {}, {}, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, {}, {}, 0,
                      RowBuf(MODE && a.act ? (const bf16*)a.act + cs * T * F : nullptr, MODE && a.act ? 2L * T * F : 0),
                      RowBuf(MODE ? (const bf16*)a.dact + cs * T * F : nullptr, MODE ? 2L * T * F : 0), MODE && a.act,
                      row * F * 2 + 16 * lh};
  ffn.run(R, U, acc, act);
  wait_vmcnt<0>();                                               // (tiles nobody reads)

  if constexpr (MODE != 1) {                                     // OUT = X + h (ybar + m) (+ rhs)
    if (row >= T) return;
    float* orow = a.OUT.at(g) + (long)row * D + 4 * lh;
    if constexpr (!KEEP_X) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) v[i] = ld_global(reinterpret_cast<const f32x4*>(xr + 8 * i));
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const f32x4 x = KEEP_X ? xk[KEEP_X ? i : 0] : v[i];
      v[i] = x + a.hstep * (quad(acc[i >> 2], i & 3) + lds_read4f(vec + 3 * V + 32 * i));
    }
    if (a.RHS.present()) {
      const float* rr = a.RHS.at(g) + (long)row * D + 4 * lh;
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const f32x4 rhs = ld_global(reinterpret_cast<const f32x4*>(rr + 8 * i));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = __builtin_fmaf(a.rhs_sign, v[i][e], rhs[e]);
      }
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) *reinterpret_cast<f32x4*>(orow + 8 * i) = v[i];
  }
}

// ---------------------------------------------------------------------------
// head: u = LN1(X), Q | K | V = u Wqkv^T + b
// ---------------------------------------------------------------------------
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2) chain_head_kernel(const ChainHeadArgs a, int tiles_m, int total, int per_xcd) {
  constexpr int KS = D / 16, NQ = D / 8, N = 3 * D;
  constexpr bool WIDE = D == 128;
  constexpr int FT = WIDE ? 32 : 64, NT = N / FT;                // features of a tile, tiles
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const Place pl = place<NW>(tiles_m, total, per_xcd);
  if (pl.none) return;
  const int lane = pl.lane, lr = lane & 31, lh = lane >> 5, g = pl.g, T = a.T;
  const int row = pl.row0 + lr, crow = row < T ? row : T - 1;
  const char* pb = a.P.at(g);
  const Matrix<NW, WIDE> W(pb + a.w_off, D, pl.wave, lane);
  Ring<NW> R;
  R.init(smem, lane);
  auto load_at = [&](int i) { if (i < NT) W.load(R.put, pl.wave, i * FT * D * 2); };
  const float* xr = a.X.at(g) + (long)crow * D + 4 * lh;
  f32x4 v[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) v[i] = ld_global(reinterpret_cast<const f32x4*>(xr + 8 * i));
  constexpr int V = vec_bytes(D);                                // gamma, beta, bias
  {
    unsigned char* m = smem + RING_BYTES;
    m = vector_to_lds<NW>(m, pb + a.g_off, D, pl.wave, lane);
    m = vector_to_lds<NW>(m, pb + a.be_off, D, pl.wave, lane);
    vector_to_lds<NW>(m, pb + a.b_off, N, pl.wave, lane);
  }
  const lds_byte* vec = (const lds_byte*)smem + RING_BYTES + 16 * lh;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < RING_LEAD; ++i) { load_at(i); R.step_put(); }
  wait_vmcnt<Ring<NW>::LPT*(NT < RING_LEAD ? NT : RING_LEAD)>();   // the rows and the vectors
  bare_barrier();

  bf16x8 U[KS];
  const long cs = a.cs.of(g);
  const RowBuf bxh(a.xhat ? (const bf16*)a.xhat + cs * T * D : nullptr, a.xhat ? 2L * T * D : 0);
  const RowBuf bu(a.u ? (const bf16*)a.u + cs * T * D : nullptr, a.u ? 2L * T * D : 0);
  {
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NQ; ++i) part[i & 3] += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
    const float mu = both_halves((part[0] + part[1]) + (part[2] + part[3])) / D;
    float sq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      v[i] = v[i] - mu;
      sq[i & 3] += (v[i][0] * v[i][0] + v[i][1] * v[i][1]) + (v[i][2] * v[i][2] + v[i][3] * v[i][3]);
    }
    const float rstd = 1.0f / sqrtf(both_halves((sq[0] + sq[1]) + (sq[2] + sq[3])) / D + a.eps);
    if (a.xhat && row < T && lh == 0) a.rstd[cs * T + row] = rstd;
    const int ro = row * D * 2 + 16 * lh;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      f32x4 w[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) w[h] = v[2 * k + h] * rstd;
      if (a.xhat) bxh.store(ro + 32 * k, operand_of(w[0], w[1]));
#pragma unroll
      for (int h = 0; h < 2; ++h) w[h] = w[h] * lds_read4f(vec + 32 * (2 * k + h)) + lds_read4f(vec + V + 32 * (2 * k + h));
      U[k] = operand_of(w[0], w[1]);
      if (a.u) bu.store(ro + 32 * k, U[k]);
    }
  }
  constexpr bool ALL = NT <= RING_LEAD;                          // all tiles are in the ring from the start
  R.template wait<ALL ? 0 : RING_LEAD - 2, 0>();
  R.prime();
  const RowBuf bo((const bf16*)a.out + a.out_slots.of(g) * T * N, 2L * T * N);
  const int oo = row * N * 2 + 16 * lh;
  constexpr int STORES = FT / 16;                                // of a set, behind its tile
  each<NT>([&](auto tt) {
    constexpr int t = decltype(tt)::value;
    constexpr int asked = t - 1 + RING_LEAD < NT ? t - 1 + RING_LEAD : NT - 1, behind = asked - (t + RING_G) > 0 ? asked - (t + RING_G) : 0;
    f32x16 c[FT / 32];
    R.template set<!ALL && t % RING_G == RING_G - 1, behind, STORES * (t < RING_LEAD - 2 ? t : RING_LEAD - 2)>(
        [&] { load_at(t + RING_LEAD); }, [&](auto m, bf16x8 w) {
          if constexpr (WIDE) mfma(c[0], w, U[m], m == 0);
          else mfma(c[m >> 2], w, U[m & 3], (m & 3) == 0);
        }, [](auto) {});
#pragma unroll
    for (int b = 0; b < FT / 32; ++b)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int f = t * FT + 32 * b + 16 * k;
        const lds_byte* bv = vec + 2 * V + f * 4;
        bo.store(oo + f * 2, operand_of(quad(c[b], 2 * k) + lds_read4f(bv), quad(c[b], 2 * k + 1) + lds_read4f(bv + 32)));
      }
  });
}

// ---------------------------------------------------------------------------
// adjoint_tail: dz = (c W2) gelu'(z), du = dz W1, r = LN2^T du, ds = c + r, da = ds Wo (matrices stored transposed)
// ---------------------------------------------------------------------------
// to the operand type and back: what the LayerNorm transposes are given (and the parameter gradients read)
template <int NB> __device__ __forceinline__ void round_all(f32x16 (&acc)[NB]) {
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = (float)(bf16)acc[i][e];
}
// r = LN^T dy for dy = acc; xh the normalised rows as operands
template <int D> __device__ __forceinline__ void ln_vjp(const f32x16 (&acc)[D / 32], bf16x8 (&xh)[D / 16], float rstd,
                                                        const lds_byte* gamma, f32x4 (&r)[D / 8]) {
  float s1[2] = {0.f, 0.f}, s2[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < D / 16; ++k) {
    f32x4 x[2];
    quads_of(xh[k], x[0], x[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = 2 * k + h;
      const f32x4 w = quad(acc[i >> 2], i & 3) * lds_read4f(gamma + 32 * i);
      s1[h] += (w[0] + w[1]) + (w[2] + w[3]);
      s2[h] += (w[0] * x[h][0] + w[1] * x[h][1]) + (w[2] * x[h][2] + w[3] * x[h][3]);
    }
  }
  const float m1 = both_halves(s1[0] + s1[1]) / D, m2 = both_halves(s2[0] + s2[1]) / D;
#pragma unroll
  for (int k = 0; k < D / 16; ++k) {
    f32x4 x[2];
    u32x4 again = __builtin_bit_cast(u32x4, xh[k]);          // unpacked once more: kept, the rows would take too many registers
    asm volatile("" : "+v"(again));
    xh[k] = __builtin_bit_cast(bf16x8, again);
    quads_of(xh[k], x[0], x[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = 2 * k + h;
      r[i] = rstd * (quad(acc[i >> 2], i & 3) * lds_read4f(gamma + 32 * i) - m1 - x[h] * m2);
    }
  }
}

template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2) chain_adjoint_tail_kernel(const ChainAdjointArgs a, int tiles_m, int total, int per_xcd) {
  constexpr int NB = D / 32, KS = D / 16, NQ = D / 8;
  constexpr bool WIDE = D == 128;
  constexpr int FT = WIDE ? 32 : 64, NR = D / FT;                // features of a tile of Wo, tiles
  using Ffn = Pair<D, NW, 0, true, NR, DGelu<D>>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const Place pl = place<NW>(tiles_m, total, per_xcd);
  if (pl.none) return;
  const int lane = pl.lane, lr = lane & 31, lh = lane >> 5, g = pl.g, T = a.T, F = a.f;
  const int row = pl.row0 + lr, crow = row < T ? row : T - 1;
  const char *pb = a.P.at(g), *pt = a.PT.at(g);
  const Ffn ffn(pt + a.w2_off, pt + a.w1_off, pt + a.wo_off, F, pl.wave, lane);
  Ring<NW> R;
  R.init(smem, lane);
  const long cs = a.cs.of(g), ls = a.loc.of(g);
  const int ro = row * D * 2 + 16 * lh;
  bf16x8 U[KS];
  if (a.c) {
    const RowBuf bc((const bf16*)a.c + a.c_slots.of(g) * T * D, 2L * T * D);
#pragma unroll
    for (int k = 0; k < KS; ++k) U[k] = bc.load(ro + 32 * k);
  } else {
    const RowBuf bc(a.c_out ? (bf16*)a.c_out + ls * T * D : nullptr, a.c_out ? 2L * T * D : 0);
    const float* cr = a.IN.at(g) + (long)crow * D + 4 * lh;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      U[k] = operand_of(ld_global(reinterpret_cast<const f32x4*>(cr + 16 * k)), ld_global(reinterpret_cast<const f32x4*>(cr + 16 * k + 8)));
      if (a.c_out) bc.store(ro + 32 * k, U[k]);
    }
  }
  const RowBuf bxh((const bf16*)a.xhat + cs * T * D, 2L * T * D);
  bf16x8 xh[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) xh[k] = bxh.load(ro + 32 * k);
  const float rstd = a.rstd[cs * T + crow];
  DGelu<D> act{RowBuf((const bf16*)a.dact + cs * T * F, 2L * T * F),
            RowBuf(a.dz ? (const bf16*)a.dz + ls * T * F : nullptr, a.dz ? 2L * T * F : 0), a.dz != nullptr, row * F * 2 + 16 * lh, 0,
            {}, {}, {}, {}, {}, 0.f, 0.f};
  vector_to_lds<NW>(smem + RING_BYTES, pb + a.g_off, D, pl.wave, lane);
  const lds_byte* vec = (const lds_byte*)smem + RING_BYTES + 16 * lh;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < RING_LEAD; ++i) { ffn.tile(R.put, i, 0); R.step_put(); }
  __builtin_amdgcn_sched_barrier(0);
  act.first();
  __builtin_amdgcn_sched_barrier(0);
  R.template start<4>();

  f32x16 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  ffn.run(R, U, acc, act);

  {
    if (a.du) {
      const RowBuf bd((const bf16*)a.du + ls * T * D, 2L * T * D);
#pragma unroll
      for (int k = 0; k < KS; ++k) bd.store(ro + 32 * k, operand_of(quad(acc[k >> 1], 2 * (k & 1)), quad(acc[k >> 1], 2 * (k & 1) + 1)));
    }
    round_all(acc);
    f32x4 r[NQ];
    ln_vjp<D>(acc, xh, rstd, vec, r);
    if (row < T) {
      float* dx = a.dx + (ls * T + row) * D + 4 * lh;
#pragma unroll
      for (int i = 0; i < NQ; ++i) *reinterpret_cast<f32x4*>(dx + 8 * i) = r[i];
    }
    const RowBuf bs(a.ds ? (const bf16*)a.ds + ls * T * D : nullptr, a.ds ? 2L * T * D : 0);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      f32x4 c0, c1;
      quads_of(U[k], c0, c1);
      U[k] = operand_of(c0 + r[2 * k], c1 + r[2 * k + 1]);
      if (a.ds) bs.store(ro + 32 * k, U[k]);
    }
  }
  const RowBuf bo((const bf16*)a.da + ls * T * D, 2L * T * D);
  each<NR>([&](auto qt) {
    constexpr int q = decltype(qt)::value;
    f32x16 c[FT / 32];
    R.template set<q % RING_G == RING_G - 1, 0, 0>([] {}, [&](auto m, bf16x8 w) {
      if constexpr (WIDE) mfma(c[0], w, U[m], m == 0);
      else mfma(c[m >> 2], w, U[m & 3], (m & 3) == 0);
    }, [](auto) {});
#pragma unroll
    for (int b = 0; b < FT / 32; ++b)
#pragma unroll
      for (int k = 0; k < 2; ++k) bo.store(ro + (q * FT + 32 * b + 16 * k) * 2, operand_of(quad(c[b], 2 * k), quad(c[b], 2 * k + 1)));
  });
  wait_vmcnt<0>();                                               // (tiles nobody reads)
}

// ---------------------------------------------------------------------------
// adjoint_head: du = dqkv Wqkv, r = dx + LN1^T du, OUT = c + h r (+ rhs)
// ---------------------------------------------------------------------------
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2) chain_adjoint_head_kernel(const ChainAdjointArgs a, int tiles_m, int total, int per_xcd) {
  constexpr int SB = D / 64, NB = D / 32, KS = D / 16, NQ = D / 8, K3 = 3 * SB, NT = SB * K3;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const Place pl = place<NW>(tiles_m, total, per_xcd);
  if (pl.none) return;
  const int lane = pl.lane, lr = lane & 31, lh = lane >> 5, g = pl.g, T = a.T;
  const int row = pl.row0 + lr, crow = row < T ? row : T - 1;
  const char *pb = a.P.at(g), *pt = a.PT.at(g);
  const Matrix<NW, false> W(pt + a.wqkv_off, 3 * D, pl.wave, lane);
  Ring<NW> R;
  R.init(smem, lane);
  auto load_at = [&](int i) { if (i < NT) W.load(R.put, pl.wave, (i / K3 * 64 * 3 * D + i % K3 * 64) * 2); };
  const long cs = a.cs.of(g), ls = a.loc.of(g);
  const int ro = row * D * 2 + 16 * lh;
  bf16x8 Y[3 * KS];
  {
    const RowBuf by((const bf16*)a.dqkv + ls * T * 3 * D, 6L * T * D);
#pragma unroll
    for (int k = 0; k < 3 * KS; ++k) Y[k] = by.load(row * 6 * D + 16 * lh + 32 * k);
  }
  const RowBuf bxh((const bf16*)a.xhat + cs * T * D, 2L * T * D);
  bf16x8 xh[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) xh[k] = bxh.load(ro + 32 * k);
  vector_to_lds<NW>(smem + RING_BYTES, pb + a.g_off, D, pl.wave, lane);
  const lds_byte* vec = (const lds_byte*)smem + RING_BYTES + 16 * lh;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < RING_LEAD; ++i) { load_at(i); R.step_put(); }
  constexpr bool ALL = NT <= RING_LEAD;
  R.template wait<ALL ? 0 : RING_LEAD - 2, 0>();
  R.prime();
  f32x16 acc[NB];
  each<NT>([&](auto qt) {
    constexpr int q = decltype(qt)::value;
    constexpr int asked = q - 1 + RING_LEAD < NT ? q - 1 + RING_LEAD : NT - 1, behind = asked - (q + RING_G) > 0 ? asked - (q + RING_G) : 0;
    R.template set<!ALL && q % RING_G == RING_G - 1, behind, 0>([&] { load_at(q + RING_LEAD); }, [&](auto m, bf16x8 w) {
      mfma(acc[2 * (q / K3) + (m >> 2)], w, Y[4 * (q % K3) + (m & 3)], q % K3 == 0 && (m & 3) == 0);
    }, [](auto) {});
  });
  if (a.du) {
    const RowBuf bd((const bf16*)a.du + ls * T * D, 2L * T * D);
#pragma unroll
    for (int k = 0; k < KS; ++k) bd.store(ro + 32 * k, operand_of(quad(acc[k >> 1], 2 * (k & 1)), quad(acc[k >> 1], 2 * (k & 1) + 1)));
  }
  if (!a.OUT.present()) return;                                  // gradients alone
  const float rstd = a.rstd[cs * T + crow];
  round_all(acc);
  f32x4 r[NQ];
  ln_vjp<D>(acc, xh, rstd, vec, r);
  const float* dx = a.dx + (ls * T + crow) * D + 4 * lh;
  const float* cr = a.IN.at(g) + (long)crow * D + 4 * lh;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    r[i] += ld_global(reinterpret_cast<const f32x4*>(dx + 8 * i));
    r[i] = ld_global(reinterpret_cast<const f32x4*>(cr + 8 * i)) + a.hstep * r[i];
  }
  if (a.RHS.present()) {
    const float* rr = a.RHS.at(g) + (long)crow * D + 4 * lh;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const f32x4 rhs = ld_global(reinterpret_cast<const f32x4*>(rr + 8 * i));
#pragma unroll
      for (int e = 0; e < 4; ++e) r[i][e] = __builtin_fmaf(a.rhs_sign, r[i][e], rhs[e]);
    }
  }
  if (a.out_cast) {
    const RowBuf bo((const bf16*)a.out_cast + a.oc_slots.of(g) * T * D, 2L * T * D);
#pragma unroll
    for (int k = 0; k < KS; ++k) bo.store(ro + 32 * k, operand_of(r[2 * k], r[2 * k + 1]));
  }
  if (row < T) {
    float* orow = a.OUT.at(g) + (long)row * D + 4 * lh;
#pragma unroll
    for (int i = 0; i < NQ; ++i) *reinterpret_cast<f32x4*>(orow + 8 * i) = r[i];
  }
}

template <auto kern, typename A>
hipError_t launch(const A& a, int nw, int vectors, hipStream_t st) {
  const int tiles_m = (a.T + 32 * nw - 1) / (32 * nw), total = tiles_m * a.n_groups, per_xcd = (total + 7) / 8;
  const int smem = RING_BYTES + vectors + 1024;            // (a bias is read one piece ahead)
  static unsigned long raised = 0;
  if (const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), 80 << 10, raised); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(64 * nw), smem, st, a, tiles_m, total, per_xcd);
  return hipGetLastError();
}
// two wavefronts a block where four would leave compute units without one
bool narrow(int n_groups, int T) { return (long)n_groups * ((T + 127) / 128) <= compute_units() / 2; }

template <int D, int MODE> hipError_t tail_of(const ChainTailArgs& a, hipStream_t st) {
  return narrow(a.n_groups, a.T) ? launch<chain_tail_kernel<D, 2, MODE>>(a, 2, 4 * vec_bytes(D) + vec_bytes(a.f), st)
                                 : launch<chain_tail_kernel<D, 4, MODE>>(a, 4, 4 * vec_bytes(D) + vec_bytes(a.f), st);
}
template <int D> hipError_t tail_of(const ChainTailArgs& a, int mode, hipStream_t st) {
  return mode == 0 ? tail_of<D, 0>(a, st) : mode == 1 ? tail_of<D, 1>(a, st) : tail_of<D, 2>(a, st);
}
}  // namespace

// Bytes reported for a launch: the rows that it reads and writes, of the operands that are there (e: bytes of an operand), the
// tail's second read of X included.
hipError_t launch_chain_tail(const ChainTailArgs& a, int d, int mode, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0) return hipSuccess;
  const double n = (double)a.n_groups * a.T, e = is_bf16 ? 2 : 4, f = a.f;
  const double step = mode == 1 ? 0 : (d == 128 ? 8.0 : 4.0) * d + (a.RHS.present() ? 4.0 * d : 0);
  const double kept = (mode ? e * (d + f) : 0) + (a.ybar ? 4.0 * d : 0) + (a.u ? e * d : 0) + (a.act ? e * f : 0);
  ProfScope ps(PC_CHAIN, n * (2.0 * d * d + (mode == 1 ? 2.0 : 4.0) * d * f),
               n * ((e + 4) * d + (a.base ? 4.0 * d : 0) + step + kept), st);
  if (!is_bf16) return launch_chain_f32_tail(a, mode, st);
  return d == 64 ? tail_of<64>(a, mode, st) : tail_of<128>(a, mode, st);
}
hipError_t launch_chain_head(const ChainHeadArgs& a, int d, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0) return hipSuccess;
  const double rows = (double)a.n_groups * a.T, e = is_bf16 ? 2 : 4;
  ProfScope ps(PC_CHAIN, rows * 6.0 * d * d, rows * d * (4 + 3 * e + (a.xhat ? e : 0) + (a.u ? e : 0)), st);
  if (!is_bf16) return launch_chain_f32_head(a, st);
  const bool n = narrow(a.n_groups, a.T);
  if (d == 64) return n ? launch<chain_head_kernel<64, 2>>(a, 2, 2 * vec_bytes(d) + vec_bytes(3 * d), st) : launch<chain_head_kernel<64, 4>>(a, 4, 2 * vec_bytes(d) + vec_bytes(3 * d), st);
  return n ? launch<chain_head_kernel<128, 2>>(a, 2, 2 * vec_bytes(d) + vec_bytes(3 * d), st) : launch<chain_head_kernel<128, 4>>(a, 4, 2 * vec_bytes(d) + vec_bytes(3 * d), st);
}
hipError_t launch_chain_adjoint_tail(const ChainAdjointArgs& a, int d, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0) return hipSuccess;
  const double rows = (double)a.n_groups * a.T, e = is_bf16 ? 2 : 4, f = a.f;
  const double kept = (a.c ? 0 : a.c_out ? e * d : 0) + (a.dz ? e * f : 0) + (a.du ? e * d : 0) + (a.ds ? e * d : 0);
  ProfScope ps(PC_CHAIN, rows * (2.0 * d * d + 4.0 * d * f), rows * ((a.c ? e : 4) * d + (2 * e + 4) * d + e * f + kept), st);
  if (!is_bf16) return launch_chain_f32_adjoint_tail(a, st);
  const bool n = narrow(a.n_groups, a.T);
  if (d == 64) return n ? launch<chain_adjoint_tail_kernel<64, 2>>(a, 2, vec_bytes(d), st) : launch<chain_adjoint_tail_kernel<64, 4>>(a, 4, vec_bytes(d), st);
  return n ? launch<chain_adjoint_tail_kernel<128, 2>>(a, 2, vec_bytes(d), st) : launch<chain_adjoint_tail_kernel<128, 4>>(a, 4, vec_bytes(d), st);
}
hipError_t launch_chain_adjoint_head(const ChainAdjointArgs& a, int d, bool is_bf16, hipStream_t st) {
  if (a.n_groups <= 0) return hipSuccess;
  const double rows = (double)a.n_groups * a.T, e = is_bf16 ? 2 : 4;
  const double step = a.OUT.present() ? e + 12 + (a.RHS.present() ? 4 : 0) + (a.out_cast ? e : 0) : 0;
  ProfScope ps(PC_CHAIN, rows * 6.0 * d * d, rows * d * (3 * e + (a.du ? e : 0) + step), st);
  if (!is_bf16) return launch_chain_f32_adjoint_head(a, st);
  const bool n = narrow(a.n_groups, a.T);
  if (d == 64) return n ? launch<chain_adjoint_head_kernel<64, 2>>(a, 2, vec_bytes(d), st) : launch<chain_adjoint_head_kernel<64, 4>>(a, 4, vec_bytes(d), st);
  return n ? launch<chain_adjoint_head_kernel<128, 2>>(a, 2, vec_bytes(d), st) : launch<chain_adjoint_head_kernel<128, 4>>(a, 4, vec_bytes(d), st);
}
// Whole layer steps launch by launch and on chains, forward / adjoint with the cache pass, in us (sequences of 64):
//   128 wide, 256 hidden: 1 x 64 tokens 28 / 62 and 26 / 58, 4 x 2048 tokens 40 / 82 and 32 / 70; 64 wide, 512 hidden: 1 x 64
//   tokens 29 / 58 and 23 / 53.  Never slower up to there.
// A wavefront's way through the hidden features takes a time of its own (128 wide, 2048 hidden: 70 us forward, 150 adjoint),
// which the launches it replaces take only where there are many tokens.  Wide hidden layers of a single layer:
//   128 wide, 384: 2048 tokens 32 / 66 and 31 / 67;  512: 2048 tokens 33 / 67 and 34 / 73, 3072 tokens 35 / 72 and 34 / 74, 6144
//   tokens 39 / 81 and 36 / 79;  768: 8192 tokens 45 / 90 and 43 / 95;  1024: 8192 tokens 46 / 93 and 49 / 108, 10240 tokens
//   57 / 113 and 51 / 110;  2048: 4096 tokens 46 / 89 and 70 / 153, 12288 tokens 75 / 150 and 75 / 161, 16384 tokens 84 / 181 and
//   76 / 167;
//   64 wide, 768: 2048 tokens 35 / 65 and 30 / 67;  1024: 4096 tokens 35 / 72 and 35 / 78, 6144 tokens 39 / 80 and 36 / 81;
//   2048: 4096 tokens 42 / 83 and 54 / 121, 12288 tokens 59 / 121 and 56 / 128, 16384 tokens 67 / 144 and 58 / 130.
// The lines lie where a training step of single layers (serial propagation, every launch one layer) is no slower on chains:
// within 1 % there, and a single transposed step alone up to 4 % slower, while launches of two layers gain up to 20 % and of
// four 10 to 45 %.  Cross attention adds as many launches on either path, so that decoders 128 wide gain less and need more
// tokens: 256 hidden, training steps of 16 layers on 2 levels, 64 tokens 3.20 -> 3.55 ms, 256 tokens 3.33 -> 3.51, 1024 tokens
// 3.83 -> 3.76;  384: 2048 tokens, step 56 / 109 -> 55 / 114 us, serial training step 2.30 -> 2.35 ms, 3072 tokens 57 / 115 ->
// 56 / 118, 2.41 both;  512: 4096 tokens 60 / 119 -> 60 / 127, 2.55 -> 2.62, 6144 tokens 66 / 130 -> 65 / 131, 2.78 -> 2.75.
// The rule follows from the model alone: how many layers share a launch cannot show in a result.
bool chain_ok(int d, int f, int T, bool cross, bool is_bf16) {
  if (!is_bf16) return chain_f32_ok(d, f);
  if ((d != 64 && d != 128) || f % 64 != 0 || f > 2048 || 2.0 * T * (f > 3 * d ? f : 3 * d) >= 2e9) return false;
  if (d == 64) return f <= 512 || T >= (f <= 768 ? 2048 : f <= 1024 ? 6144 : 16384);
  if (f > 512) return T >= (f <= 1024 ? 10240 : 16384);
  if (cross) return f <= 128 || T >= (f <= 256 ? 1024 : f <= 384 ? 3072 : 6144);
  return f <= 256 || T >= (f <= 384 ? 2048 : 3072);
}

}  // namespace mg
