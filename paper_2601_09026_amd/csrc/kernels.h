// Host-side launchers of the kernels (all enqueue on the given stream, none synchronises).
#pragma once
#include "common.h"

namespace mg {

// ---- gemm.hip ----------------------------------------------------------------
hipError_t launch_gemm(const GemmArgs& a, int epi, bool is_bf16, hipStream_t st);
hipError_t launch_gemm_tn(const GemmTnArgs& a, bool is_bf16, hipStream_t st);
size_t gemm_tn_partial_floats(int n_groups, int M, int N, int K, bool is_bf16);   // scratch floats of such a launch
void gemm_force_simple(int on);
void gemm_set_tile_config(int cfg);
void gemm_set_grad_slices(int n);
bool gemm_forced();                                         // a test hook chooses the products' kernels
double gemm_model_cost(int n_groups, int M, int N, int K);
int compute_units();                                        // of the current device
void attn_set_wide_blocks(int mask);

// ---- rowwise.hip -------------------------------------------------------------
struct LnFwdArgs {
  int n_groups, T, d;
  Rows X;                                   // LN input = X rows (optional) + packed addend (optional)
  const float* xp; long xp_slot_stride; Slots xp_slots;   // packed fp32 addend
  Params P; long gamma_off, beta_off;
  void* out; long out_slot_stride; Slots out_slots;       // packed, operand type
  float eps;
  // optional (linearisation cache): the normalised row xhat = (x - mean) * rstd, packed operand type with
  // the same row layout as `out`, and rstd, one float per row ([slot][T])
  void* xhat; long xhat_slot_stride; Slots xhat_slots;
  float* rstd;
};
hipError_t launch_ln_fwd(const LnFwdArgs& a, bool is_bf16, hipStream_t st);

struct LnBwdArgs {
  int n_groups, T, d;
  const void* dy; long dy_slot_stride; Slots dy_slots;    // packed operand type: cotangent of LN output
  Rows X;                                                 // LN input = X rows (optional) + addend (optional)
  const float* xp; long xp_slot_stride; Slots xp_slots;   // packed fp32 addend
  Params P; long gamma_off;
  const float* add; long add_slot_stride; Slots add_slots;   // optional packed fp32 added to the VJP
  float* out_f32; long of_slot_stride; Slots of_slots;       // optional: v = add + vjp
  Rows C;                                                     // cotangent rows c (required if out_op or OUT)
  void* out_op; long oo_slot_stride; Slots oo_slots;         // optional packed operand type: c + v
  Rows OUT; Rows RHS; float hstep;                           // optional: OUT = c + hstep*v (+ RHS)
  float rhs_sign;                                            // with RHS: OUT = RHS + rhs_sign * (c + hstep*v), +1 or -1
  float eps;
  // optional: the LN input given as cached xhat (packed operand type) and rstd ([slot][T]) instead of X / xp
  const void* xhat; long xhat_slot_stride; Slots xhat_slots;
  const float* rstd;
  // optional: c as a packed operand-type copy, used for out_op in place of the fp32 rows C
  const void* cop; long cop_slot_stride; Slots cop_slots;
  // optional (with OUT): the same values as OUT once more as a packed operand-type copy
  void* out_cast; long oc_slot_stride; Slots oc_slots;
};
hipError_t launch_ln_bwd(const LnBwdArgs& a, bool is_bf16, hipStream_t st);

// packed operand-type copy of fp32 rows
hipError_t launch_cast_rows(int n_groups, long elems, Rows X, void* out, long out_slot_stride, Slots out_slots,
                            bool is_bf16, hipStream_t st);
// packed operand-type copy of one fp32 array
hipError_t launch_cast_flat(const float* in, void* out, long elems, bool is_bf16, hipStream_t st);
// dst[g] = a[g] - b[g]  on fp32 rows
hipError_t launch_sub_rows(int n_groups, long elems, Rows A, Rows B, Rows D, hipStream_t st);
hipError_t launch_add_rows(int n_groups, long elems, Rows A, Rows B, Rows D, hipStream_t st);   // D = A (+ B)
// partial[block] = sum over the block's elements of (a-b)^2 in double; then out[0] = sqrt(sum partial)
hipError_t launch_resnorm(int n_groups, long elems, Rows A, Rows B, double* partial, int max_partial,
                          float* out, hipStream_t st);
// tab[i] = base + i*stride_bytes, i < n
hipError_t launch_fill_table(void** tab, char* base, long stride_bytes, int n, hipStream_t st);
// tab[i] = ptrs[i]: pointers travel as kernel arguments, 128 a launch (safe for any host memory, capturable)
hipError_t upload_pointers(void** tab, const void* const* host_ptrs, int n, hipStream_t st);
// n_src tables of n entries, one behind the other: a host list each, or (list = null) base + i*stride
struct PtrSource { const void* const* list; const char* base; long stride; };
hipError_t upload_tables(void** tab, const PtrSource* src, int n_src, int n, hipStream_t st);
// out_g[c, r] = in_g[r, c] for every group and every matrix of the list (at most 7 per block: byte offset, shape)
struct TransposeList { int n; int rows[7], cols[7], tiles[7]; long off[7]; };
hipError_t launch_transpose(int n_groups, Params in, Params out, const TransposeList& l, int elem_bytes, hipStream_t st);

// ---- chain.hip (bf16, d = 64 or 128), chain_f32.hip (d = 64) --------------------
struct ChainHeadArgs {
  int n_groups, T;
  Rows X;
  Params P; long g_off, be_off, w_off, b_off;
  void* out; Slots out_slots;                             // [slot, T, 3d]
  Slots cs; void* xhat; float* rstd; void* u;             // optional: cache entries (slots cs)
  float eps;
};
struct ChainTailArgs {
  int n_groups, T, f;
  const void* o; long o_slot_stride; Slots o_slots;       // attention output
  Rows X, OUT, RHS;
  const float* base; long base_slot_stride; Slots base_slots;   // optional fp32 addend of ybar
  Params P; long wo_off, bo_off, g_off, be_off, w1_off, b1_off, w2_off, b2_off;
  float hstep, rhs_sign, eps;
  Slots cs; void *xhat, *dact; float* rstd;               // modes 1, 2: cache entries (slots cs) ...
  float* ybar; void *u, *act;                             // ... and those that parameter gradients need, or null
};
// mode 0: the step; 1: the cache entries alone; 2: both
hipError_t launch_chain_tail(const ChainTailArgs& a, int d, int mode, bool is_bf16, hipStream_t st);
hipError_t launch_chain_head(const ChainHeadArgs& a, int d, bool is_bf16, hipStream_t st);
struct ChainAdjointArgs {
  int n_groups, T, f;
  const void* c; Slots c_slots;                           // tail: operand-type copy of IN, or null: formed here ...
  void* c_out;                                            // ... and left in slots loc
  Rows IN, OUT, RHS;                                      // head: without OUT du alone
  Params P, PT; long g_off, w1_off, w2_off, wo_off, wqkv_off;   // PT: matrices stored transposed
  Slots cs; const void *dact, *xhat; const float* rstd;   // cache entries
  Slots loc; void *dz, *du, *ds, *da; float* dx; const void* dqkv;   // work buffers; dz, du, ds may be null in the tail, du in the head
  void* out_cast; Slots oc_slots;
  float hstep, rhs_sign;
};
hipError_t launch_chain_adjoint_tail(const ChainAdjointArgs& a, int d, bool is_bf16, hipStream_t st);
hipError_t launch_chain_adjoint_head(const ChainAdjointArgs& a, int d, bool is_bf16, hipStream_t st);
bool chain_ok(int d, int f, int T, bool cross, bool is_bf16);
hipError_t launch_chain_f32_tail(const ChainTailArgs& a, int mode, hipStream_t st);      // (through the above)
hipError_t launch_chain_f32_head(const ChainHeadArgs& a, hipStream_t st);
hipError_t launch_chain_f32_adjoint_tail(const ChainAdjointArgs& a, hipStream_t st);
hipError_t launch_chain_f32_adjoint_head(const ChainAdjointArgs& a, hipStream_t st);
bool chain_f32_ok(int d, int f);

// ---- grads.hip ---------------------------------------------------------------
// LayerNorm gain / shift gradients of up to three LayerNorms of the same layers: sums over tokens of
// dy * xhat and dy, scaled
constexpr int LN_PARAM_MAX = 3;
struct LnParamItem {
  const void* dy; long dy_slot_stride; Slots dy_slots;    // packed operand type: cotangent of the LN output
  const float* xp; long xp_slot_stride; Slots xp_slots;   // LN input = X rows + optional packed fp32 addend
  long gamma_off, beta_off;                               // byte offsets of the fp32 results
};
struct LnParamArgs {
  int n_groups, T, d, n_items;
  Rows X;
  Params out;                                             // the group's output block
  float scale, eps;
  LnParamItem item[LN_PARAM_MAX];
};
// out[i] = scale * sum over s < n of in[s * elems + i]   (fixed order)
hipError_t launch_sum_slots(const float* in, int n, long elems, float* out, float scale, hipStream_t st);
size_t ln_param_partial_floats(int n_groups, int T, int d, int n_items);
hipError_t launch_ln_param_grad(const LnParamArgs& a, float* partial, bool is_bf16, hipStream_t st);

// ---- attention.hip -----------------------------------------------------------
struct AttnArgs {
  int n_groups, B, H, dh, Sq, Sk, causal;
  const void* q; long q_row_stride, q_slot_stride; Slots q_slots;    // operand type; head h at column h*dh
  const void* k; long k_row_stride, k_slot_stride; Slots k_slots;
  const void* v; long v_row_stride, v_slot_stride;                   // same slots as k
  void* o; long o_row_stride, o_slot_stride; Slots o_slots;          // forward output / backward input
  float* lse; long lse_slot_stride; Slots lse_slots;                 // [B,H,Sq] per slot (fwd: optional out)
  // backward only
  const void* dO; long do_row_stride, do_slot_stride; Slots do_slots;
  void* dq; void* dk; void* dv; long dqkv_row_stride, dqkv_slot_stride; Slots dqkv_slots;
  long dkv_row_stride, dkv_slot_stride;                              // dk, dv if laid out unlike dq (0: same)
  float* D; long D_slot_stride; Slots D_slots;                       // [B,H,Sq] scratch: rowsum(dO*O)
};
hipError_t launch_attn_fwd(const AttnArgs& a, bool is_bf16, hipStream_t st);
hipError_t launch_attn_bwd(const AttnArgs& a, bool is_bf16, hipStream_t st);
void attn_force_simple(int on);

}  // namespace mg
