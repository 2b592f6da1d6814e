// C ABI of libippd: argument validation, launch planning, kernel launches.
// Nothing here allocates, frees or synchronises; all work is enqueued on the
// caller's stream.
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <atomic>

#include "ippd.h"
#include "ippd_internal.h"
#include "plan.h"

namespace {

using ippd::check_batch;
using ippd::plan_prefill;
using ippd::plan_step;

thread_local int g_last_hip_error = 0;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Two-level fields of the kernel parameter blocks (S = 0 leaves positions unshifted).
template <typename P>
void set_instr_positions(const ippd_batch_t* bt, P* p) {
  p->S = bt->num_instr;
  p->instr_start = bt->num_instr > 0 ? bt->instr_start : nullptr;
  p->instr_len = bt->num_instr > 0 ? bt->instr_len : nullptr;
}

float softmax_scale(const ippd_batch_t* bt) {
  return bt->scale > 0.f ? bt->scale : 1.0f / sqrtf(static_cast<float>(bt->head_dim));
}

// theta_j = base^(-2j/D) in fp64, the rotation frequencies of pair j.
void fill_inv_freq(const ippd_batch_t* bt, double* out) {
  const int half = bt->head_dim / 2;
  for (int j = 0; j < ippd::kMaxHalfDim; ++j)
    out[j] = j < half ? pow(bt->rope_base, -2.0 * j / bt->head_dim) : 0.0;
}

ippd_status_t hip_status(hipError_t e) {
  if (e == hipSuccess) return IPPD_OK;
  g_last_hip_error = static_cast<int>(e);
  return IPPD_ERR_HIP;
}

// Shared body of the four decode entry points.  fused: q_new/k_new/v_new are
// raw token inputs that this launch rotates and appends (q_rot optional
// output); otherwise q_rot holds rotated queries and the segment already
// contains the step's token.
ippd_status_t decode(const ippd_batch_t* bt, bool shared, bool fused, const void* q_new,
                     const void* k_new, const void* v_new, const void* q_rot_in, void* q_rot_out,
                     const ippd_kv_cache_t* kv, float* out, float* lse, void* workspace,
                     size_t workspace_bytes, hipStream_t stream, bool dense = false) {
  ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  if (!kv || !out || !kv->ctx_k || !kv->ctx_vt || !kv->seg_k || !kv->seg_vt) return IPPD_ERR_NULL;
  if (fused ? (!q_new || !k_new || !v_new) : !q_rot_in) return IPPD_ERR_NULL;
  if (!aligned16(out) || !aligned16(kv->ctx_k) || !aligned16(kv->ctx_vt) || !aligned16(kv->seg_k) ||
      !aligned16(kv->seg_vt) || (lse && (reinterpret_cast<uintptr_t>(lse) & 3)))
    return IPPD_ERR_ALIGN;
  if (fused ? (!aligned16(q_new) || !aligned16(k_new) || !aligned16(v_new) || (q_rot_out && !aligned16(q_rot_out)))
            : !aligned16(q_rot_in))
    return IPPD_ERR_ALIGN;
  ippd::StepPlan pl;
  if (!plan_step(bt, shared, &pl, dense)) return IPPD_ERR_SHAPE;
  if (bt->num_questions == 0) return IPPD_OK;
  if (!workspace || workspace_bytes < pl.workspace_bytes) return IPPD_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return IPPD_ERR_ALIGN;

  ippd::StepParams p;
  p.q_new = q_new; p.k_new = k_new; p.v_new = v_new;
  p.q_rot_in = q_rot_in; p.q_rot_out = q_rot_out;
  p.ctx_k = kv->ctx_k; p.ctx_vt = kv->ctx_vt; p.seg_k = kv->seg_k; p.seg_vt = kv->seg_vt;
  p.ctx_off = bt->ctx_off; p.ctx_len = bt->ctx_len; p.q_start = bt->q_start;
  p.seg_len = bt->seg_len; p.active = bt->active; p.err_flag = bt->err_flag;
  p.out = out; p.lse = lse;
  char* ws = static_cast<char*>(workspace);
  p.part_acc = reinterpret_cast<float*>(ws + pl.off_acc);
  p.part_ml = reinterpret_cast<float*>(ws + pl.off_ml);
  p.pool = bt->ctx_pool_tokens;
  p.B = bt->num_prompts; p.Nt = bt->num_questions; p.Hq = bt->num_q_heads; p.Hkv = bt->num_kv_heads;
  p.G = bt->num_q_heads / bt->num_kv_heads; p.D = bt->head_dim; p.seg_cap = bt->seg_capacity;
  p.max_ctx_len = bt->max_ctx_len; p.max_questions = bt->max_questions;
  p.shared = pl.shared; p.fused = fused ? 1 : 0; p.nrg = pl.nrg; p.chunk = pl.chunk;
  p.max_chunks = pl.max_chunks; p.n_groups = pl.n_groups; p.ctx_blocks = pl.ctx_blocks;
  p.seg_tpu = pl.seg_tpu;
  p.instr_start = bt->num_instr > 0 ? bt->instr_start : nullptr;
  p.instr_off = bt->num_instr > 0 ? bt->instr_off : nullptr;
  p.instr_len = bt->num_instr > 0 ? bt->instr_len : nullptr;
  p.S = bt->num_instr; p.max_instr_len = bt->max_instr_len; p.max_instr_questions = bt->max_instr_questions;
  p.n_igroups = pl.n_igroups; p.nrg_i = pl.nrg_i; p.max_ichunks = pl.max_ichunks; p.instr_blocks = pl.instr_blocks;
  // merge: enough threads per item that each folds at most 8 of the
  // max_chunks + 1 partial states; items split over workgroups of kMergeThreads
  {
    int ph = 1;
    while (ph < 8 && (pl.max_chunks + 1 + pl.max_ichunks + ph - 1) / ph > 8) ph *= 2;
    const int items = bt->num_q_heads * (bt->head_dim / 8);
    const int per = ippd::kMergeThreads / ph;
    p.merge_phases = ph;
    p.merge_parts = (items + per - 1) / per;
  }
  p.scale = softmax_scale(bt);
  p.c = p.scale * 1.4426950408889634f;
  p.dense = pl.dense;
  fill_inv_freq(bt, p.inv_freq);
  if (pl.dense) return hip_status(ippd::launch_dense(bt->dtype, pl.waves, pl.rb, pl.grid, p, stream));
  return hip_status(ippd::launch_step(bt->dtype, pl.waves, pl.rb, pl.deep != 0, pl.grid, p, stream));
}

// Shared body of the two prefill entry points.
ippd_status_t prefill(const ippd_batch_t* bt, bool shared, int32_t max_q_tokens, const void* q_ctx,
                      const void* q_seg, const ippd_kv_cache_t* kv, float* out_ctx, float* out_seg,
                      hipStream_t stream) {
  ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  if (!q_ctx || !q_seg || !kv || !out_ctx || !out_seg || !kv->ctx_k || !kv->ctx_vt || !kv->seg_k || !kv->seg_vt)
    return IPPD_ERR_NULL;
  if (!aligned16(q_ctx) || !aligned16(q_seg) || !aligned16(out_ctx) || !aligned16(out_seg) ||
      !aligned16(kv->ctx_k) || !aligned16(kv->ctx_vt) || !aligned16(kv->seg_k) || !aligned16(kv->seg_vt))
    return IPPD_ERR_ALIGN;
  ippd::PrefillPlan pl;
  if (!plan_prefill(bt, shared, max_q_tokens, &pl)) return IPPD_ERR_SHAPE;
  if (pl.grid == 0) return IPPD_OK;
  ippd::PrefillParams p;
  p.q_ctx = q_ctx; p.q_seg = q_seg;
  p.ctx_k = kv->ctx_k; p.ctx_vt = kv->ctx_vt; p.seg_k = kv->seg_k; p.seg_vt = kv->seg_vt;
  p.ctx_off = bt->ctx_off; p.ctx_len = bt->ctx_len; p.q_start = bt->q_start; p.seg_len = bt->seg_len;
  p.err_flag = bt->err_flag;
  p.out_ctx = out_ctx; p.out_seg = out_seg;
  p.pool = bt->ctx_pool_tokens;
  p.B = bt->num_prompts; p.Nt = bt->num_questions; p.Hq = bt->num_q_heads; p.Hkv = bt->num_kv_heads;
  p.G = bt->num_q_heads / bt->num_kv_heads; p.D = bt->head_dim; p.seg_cap = bt->seg_capacity;
  p.max_ctx_len = bt->max_ctx_len;
  p.shared = pl.shared; p.tb = pl.tb; p.n_groups = pl.n_groups;
  p.kq = pl.kq; p.kc = pl.kc; p.q_blocks = pl.q_blocks;
  p.n_cgroups = pl.n_cgroups;
  p.S = bt->num_instr;
  p.max_instr_len = bt->num_instr > 0 ? bt->max_instr_len : 0;
  p.instr_start = bt->num_instr > 0 ? bt->instr_start : nullptr;
  p.instr_off = bt->num_instr > 0 ? bt->instr_off : nullptr;
  p.instr_len = bt->num_instr > 0 ? bt->instr_len : nullptr;
  p.c = softmax_scale(bt) * 1.4426950408889634f;
  fill_inv_freq(bt, p.inv_freq);
  return hip_status(ippd::launch_prefill(bt->dtype, bt->head_dim, pl.rb, pl.grid, p, stream));
}

// Per-device address of the no-allocation scratch array, looked up once per
// device (concurrent first calls look up the same address).
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_addr[kMaxDevices];

}  // namespace

// Partial softmax states of ippd_decode_step_noalloc: each GPU the library
// runs on holds its own copy until the process ends.  In host code this name
// is a stand-in, not a device address: kernels get the address looked up with
// hipGetSymbolAddress on the device concerned.
static __device__ __align__(256) unsigned char scratch[IPPD_NOALLOC_SCRATCH_BYTES];

extern "C" {

ippd_status_t ippd_load_context(const ippd_batch_t* bt, const void* k_raw, const void* v_raw,
                                const ippd_kv_cache_t* kv, hipStream_t stream) {
  ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  if (!k_raw || !v_raw || !kv || !kv->ctx_k || !kv->ctx_vt) return IPPD_ERR_NULL;
  if (!aligned16(k_raw) || !aligned16(v_raw) || !aligned16(kv->ctx_k) || !aligned16(kv->ctx_vt))
    return IPPD_ERR_ALIGN;
  ippd::LoadContextParams p;
  p.k_raw = k_raw; p.v_raw = v_raw; p.ctx_k = kv->ctx_k; p.ctx_vt = kv->ctx_vt;
  p.ctx_off = bt->ctx_off; p.ctx_len = bt->ctx_len; p.err_flag = bt->err_flag;
  p.pool = bt->ctx_pool_tokens; p.B = bt->num_prompts; p.Hkv = bt->num_kv_heads; p.D = bt->head_dim;
  p.max_ctx_len = bt->max_ctx_len;
  set_instr_positions(bt, &p);
  fill_inv_freq(bt, p.inv_freq);
  return hip_status(ippd::launch_load_context(bt->dtype, p, stream));
}

ippd_status_t ippd_load_instructions(const ippd_batch_t* bt, const void* k_raw, const void* v_raw,
                                     const ippd_kv_cache_t* kv, hipStream_t stream) {
  ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  if (bt->num_instr == 0) return IPPD_ERR_SHAPE;
  if (!k_raw || !v_raw || !kv || !kv->ctx_k || !kv->ctx_vt) return IPPD_ERR_NULL;
  if (!aligned16(k_raw) || !aligned16(v_raw) || !aligned16(kv->ctx_k) || !aligned16(kv->ctx_vt))
    return IPPD_ERR_ALIGN;
  // the context loader over the instruction blocks, at positions 0..len-1
  ippd::LoadContextParams p;
  p.k_raw = k_raw; p.v_raw = v_raw; p.ctx_k = kv->ctx_k; p.ctx_vt = kv->ctx_vt;
  p.ctx_off = bt->instr_off; p.ctx_len = bt->instr_len; p.err_flag = bt->err_flag;
  p.pool = bt->ctx_pool_tokens; p.B = bt->num_instr; p.Hkv = bt->num_kv_heads; p.D = bt->head_dim;
  p.max_ctx_len = bt->max_instr_len;
  p.S = 0; p.instr_start = nullptr; p.instr_len = nullptr;
  fill_inv_freq(bt, p.inv_freq);
  return hip_status(ippd::launch_load_context(bt->dtype, p, stream));
}

ippd_status_t ippd_load_segments(const ippd_batch_t* bt, const void* k_raw, const void* v_raw,
                                 const int32_t* init_len, const ippd_kv_cache_t* kv,
                                 hipStream_t stream) {
  ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  if (!k_raw || !v_raw || !init_len || !kv || !kv->seg_k || !kv->seg_vt) return IPPD_ERR_NULL;
  if (!aligned16(k_raw) || !aligned16(v_raw) || !aligned16(kv->seg_k) || !aligned16(kv->seg_vt))
    return IPPD_ERR_ALIGN;
  ippd::LoadSegmentsParams p;
  p.k_raw = k_raw; p.v_raw = v_raw; p.init_len = init_len; p.seg_k = kv->seg_k; p.seg_vt = kv->seg_vt;
  p.ctx_len = bt->ctx_len; p.q_start = bt->q_start; p.seg_len = bt->seg_len; p.err_flag = bt->err_flag;
  p.B = bt->num_prompts; p.Nt = bt->num_questions; p.Hkv = bt->num_kv_heads; p.D = bt->head_dim;
  p.seg_cap = bt->seg_capacity;
  set_instr_positions(bt, &p);
  fill_inv_freq(bt, p.inv_freq);
  return hip_status(ippd::launch_load_segments(bt->dtype, p, stream));
}

ippd_status_t ippd_append_kv(const ippd_batch_t* bt, const void* q_new, const void* k_new,
                             const void* v_new, void* q_rot, const ippd_kv_cache_t* kv,
                             hipStream_t stream) {
  ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  if (!q_new || !k_new || !v_new || !q_rot || !kv || !kv->seg_k || !kv->seg_vt) return IPPD_ERR_NULL;
  if (!aligned16(q_new) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(q_rot) ||
      !aligned16(kv->seg_k) || !aligned16(kv->seg_vt))
    return IPPD_ERR_ALIGN;
  ippd::AppendParams p;
  p.q_new = q_new; p.k_new = k_new; p.v_new = v_new; p.q_rot = q_rot;
  p.seg_k = kv->seg_k; p.seg_vt = kv->seg_vt;
  p.ctx_len = bt->ctx_len; p.q_start = bt->q_start; p.seg_len = bt->seg_len;
  p.active = bt->active; p.err_flag = bt->err_flag;
  p.B = bt->num_prompts; p.Nt = bt->num_questions; p.Hq = bt->num_q_heads; p.Hkv = bt->num_kv_heads;
  p.D = bt->head_dim; p.seg_cap = bt->seg_capacity;
  set_instr_positions(bt, &p);
  fill_inv_freq(bt, p.inv_freq);
  return hip_status(ippd::launch_append(bt->dtype, p, stream));
}

size_t ippd_decode_workspace_bytes(const ippd_batch_t* bt) {
  ippd::StepPlan pl;
  return plan_step(bt, true, &pl) ? pl.workspace_bytes : 0;
}

size_t standard_decode_workspace_bytes(const ippd_batch_t* bt) {
  ippd::StepPlan pl;
  return plan_step(bt, false, &pl) ? pl.workspace_bytes : 0;
}

ippd_status_t ippd_decode_attention(const ippd_batch_t* bt, const void* q_rot,
                                    const ippd_kv_cache_t* kv, float* out, float* lse,
                                    void* workspace, size_t workspace_bytes, hipStream_t stream) {
  return decode(bt, true, false, nullptr, nullptr, nullptr, q_rot, nullptr, kv, out, lse, workspace,
                workspace_bytes, stream);
}

ippd_status_t standard_decode_attention(const ippd_batch_t* bt, const void* q_rot,
                                        const ippd_kv_cache_t* kv, float* out, float* lse,
                                        void* workspace, size_t workspace_bytes,
                                        hipStream_t stream) {
  return decode(bt, false, false, nullptr, nullptr, nullptr, q_rot, nullptr, kv, out, lse, workspace,
                workspace_bytes, stream);
}

size_t dense_decode_workspace_bytes(const ippd_batch_t* bt) {
  ippd::StepPlan pl;
  return plan_step(bt, true, &pl, true) ? pl.workspace_bytes : 0;
}

ippd_status_t dense_decode_attention(const ippd_batch_t* bt, const void* q_rot, const ippd_kv_cache_t* kv,
                                     float* out, float* lse, void* workspace, size_t workspace_bytes,
                                     hipStream_t stream) {
  return decode(bt, true, false, nullptr, nullptr, nullptr, q_rot, nullptr, kv, out, lse, workspace,
                workspace_bytes, stream, true);
}

ippd_status_t ippd_decode_step(const ippd_batch_t* bt, const void* q_new, const void* k_new,
                               const void* v_new, void* q_rot, const ippd_kv_cache_t* kv, float* out,
                               float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  return decode(bt, true, true, q_new, k_new, v_new, nullptr, q_rot, kv, out, lse, workspace,
                workspace_bytes, stream);
}

ippd_status_t ippd_decode_step_noalloc(const ippd_batch_t* bt, const void* q_new, const void* k_new,
                                       const void* v_new, void* q_rot, const ippd_kv_cache_t* kv, float* out,
                                       float* lse, hipStream_t stream) {
  const ippd_status_t st = check_batch(bt);
  if (st != IPPD_OK) return st;
  ippd::StepPlan pl;
  if (!plan_step(bt, true, &pl)) return IPPD_ERR_SHAPE;
  if (pl.workspace_bytes > IPPD_NOALLOC_SCRATCH_BYTES) return IPPD_ERR_SCRATCH;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_status(e);
  if (dev < 0 || dev >= kMaxDevices) return hip_status(hipErrorInvalidDevice);
  void* ptr = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_status(e);
    if (ptr == nullptr || (reinterpret_cast<uintptr_t>(ptr) & 255u)) return hip_status(hipErrorInvalidSymbol);
    g_scratch_addr[dev].store(ptr, std::memory_order_release);
  }
  return decode(bt, true, true, q_new, k_new, v_new, nullptr, q_rot, kv, out, lse, ptr, IPPD_NOALLOC_SCRATCH_BYTES,
                stream);
}

ippd_status_t standard_decode_step(const ippd_batch_t* bt, const void* q_new, const void* k_new,
                                   const void* v_new, void* q_rot, const ippd_kv_cache_t* kv,
                                   float* out, float* lse, void* workspace, size_t workspace_bytes,
                                   hipStream_t stream) {
  return decode(bt, false, true, q_new, k_new, v_new, nullptr, q_rot, kv, out, lse, workspace,
                workspace_bytes, stream);
}

ippd_status_t ippd_prefill_attention(const ippd_batch_t* bt, int32_t max_prompt_question_tokens,
                                     const void* q_ctx, const void* q_seg, const ippd_kv_cache_t* kv,
                                     float* out_ctx, float* out_seg, hipStream_t stream) {
  return prefill(bt, true, max_prompt_question_tokens, q_ctx, q_seg, kv, out_ctx, out_seg, stream);
}

ippd_status_t standard_prefill_attention(const ippd_batch_t* bt, int32_t max_prompt_question_tokens,
                                         const void* q_ctx, const void* q_seg, const ippd_kv_cache_t* kv,
                                         float* out_ctx, float* out_seg, hipStream_t stream) {
  return prefill(bt, false, max_prompt_question_tokens, q_ctx, q_seg, kv, out_ctx, out_seg, stream);
}

const char* ippd_status_string(ippd_status_t s) {
  // a C caller may pass any int: read it as one (an out-of-range value of the
  // enum type itself would be undefined behaviour here)
  int code;
  static_assert(sizeof(code) == sizeof(s), "status codes are int-sized");
  memcpy(&code, &s, sizeof code);
  switch (code) {
    case IPPD_OK: return "ok";
    case IPPD_ERR_NULL: return "required pointer is NULL";
    case IPPD_ERR_SHAPE: return "inconsistent or unsupported sizes";
    case IPPD_ERR_DTYPE: return "unknown dtype";
    case IPPD_ERR_ALIGN: return "pointer not aligned (16 bytes; workspace 256 bytes)";
    case IPPD_ERR_WORKSPACE: return "workspace missing or too small";
    case IPPD_ERR_HIP: return "HIP call failed";
    case IPPD_ERR_SCRATCH: return "batch needs more partial-state scratch than the no-allocation step holds";
  }
  return "unknown status";
}

int ippd_last_hip_error(void) { return g_last_hip_error; }

int ippd_version(void) { return 700; }

}  // extern "C"
