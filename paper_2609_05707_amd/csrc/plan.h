// Argument checks and launch plans of the library's calls: host code only, a
// function of the batch fields, so that a workspace query and a launch agree.
#pragma once

#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "ippd.h"
#include "ippd_internal.h"

namespace ippd {

constexpr int kMinChunk = 256;
constexpr int kMaxChunk = 4096;

// Host-side checks of the batch sizes and device-array pointers.
inline ippd_status_t check_batch(const ippd_batch_t* bt) {
  if (bt == nullptr) return IPPD_ERR_NULL;
  if (bt->dtype != IPPD_DTYPE_F32 && bt->dtype != IPPD_DTYPE_BF16) return IPPD_ERR_DTYPE;
  if (bt->num_prompts < 1 || bt->num_questions < 0 || bt->num_q_heads < 1 || bt->num_kv_heads < 1)
    return IPPD_ERR_SHAPE;
  if (bt->num_q_heads % bt->num_kv_heads != 0) return IPPD_ERR_SHAPE;
  if (bt->num_q_heads / bt->num_kv_heads > kMaxGroup) return IPPD_ERR_SHAPE;
  if (bt->head_dim != 64 && bt->head_dim != 128) return IPPD_ERR_SHAPE;
  if (bt->ctx_pool_tokens < 0 || (bt->ctx_pool_tokens & 7)) return IPPD_ERR_SHAPE;
  if (bt->seg_capacity < 8 || (bt->seg_capacity & 7)) return IPPD_ERR_SHAPE;
  if (bt->max_ctx_len < 0 || bt->max_ctx_len > bt->ctx_pool_tokens) return IPPD_ERR_SHAPE;
  if (bt->max_questions < 1 || bt->max_questions > kMaxQuestionsPerPrompt) return IPPD_ERR_SHAPE;
  if (bt->chunk_tokens < 0 || (bt->chunk_tokens & 31)) return IPPD_ERR_SHAPE;
  if (bt->tile_rows != 0 && bt->tile_rows != 16 && bt->tile_rows != 32 && bt->tile_rows != 64 &&
      bt->tile_rows != 128 && bt->tile_rows != 256)
    return IPPD_ERR_SHAPE;
  if (bt->tile_rows == 256 && !(bt->dtype == IPPD_DTYPE_BF16 && bt->head_dim == 128)) return IPPD_ERR_SHAPE;
  if (!(bt->rope_base > 0.0) || !isfinite(bt->rope_base)) return IPPD_ERR_SHAPE;
  if (!isfinite(bt->scale)) return IPPD_ERR_SHAPE;
  if (!bt->ctx_off || !bt->ctx_len || !bt->q_start || !bt->seg_len || !bt->active || !bt->err_flag)
    return IPPD_ERR_NULL;
  if (bt->num_instr < 0) return IPPD_ERR_SHAPE;
  if (bt->num_instr > 0) {
    if (bt->num_instr > bt->num_prompts || bt->max_instr_len < 0 || bt->max_instr_len > bt->ctx_pool_tokens ||
        bt->max_instr_questions < 1)
      return IPPD_ERR_SHAPE;
    if (!bt->instr_start || !bt->instr_off || !bt->instr_len) return IPPD_ERR_NULL;
  }
  return IPPD_OK;
}

inline size_t round256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// Compute units the planner sizes grids for: the 256 of MI355X (gfx950).  A
// constant, not a device query, so that the plan (and with it the workspace
// size) depends on the batch fields only, the library holds no state, and a
// workspace query on one thread or device agrees with the launch on another.
// On a part with fewer compute units the plan is still correct, only sized
// for more of them.
constexpr int kPlanComputeUnits = 256;
inline int compute_units() { return kPlanComputeUnits; }

// Chunk of a small batch, whose units all run at once: a unit folds its tiles
// one after another (us a tile, the latency of its chain: bf16 0.75, fp32 1.6
// at D = 64 and 2.4 at D = 128), and the merge folds the n chunks' states (us
// a chunk: 0.03, and 0.36 per thousand rows).  n = sqrt(tile time * tiles /
// slot time) minimises the sum.  Measured over 32 .. 512 tokens, us a layer
// step at the former 256-token minimum, at this choice and at the best size:
// fp32 D = 64, 256 tokens x 4 questions 23.2, 11.9, 11.9; fp32 D = 128, 1024
// x 8 33.7, 19.1, 19.1; bf16 D = 128, 512 x 4 17.6, 13.0, 13.0, 1024 x 16
// 17.8, 15.6, 15.5, 4096 x 16 19.6, 18.8, 18.8.
inline int64_t small_chunk(const ippd_batch_t* bt, int max_ilen) {
  const double tile = bt->dtype == IPPD_DTYPE_BF16 ? 0.75 : (bt->head_dim == 64 ? 1.6 : 2.4);
  const double slot = 0.03 + 0.36e-3 * bt->num_questions * bt->num_q_heads;
  const double len = std::max(std::max(bt->max_ctx_len, max_ilen), 32);
  const double n = sqrt(tile * len / 32 / slot);
  return 32 * std::max<int64_t>(1, llround(len / n / 32));
}

// Launch plan of a decode call.  Depends only on host fields, so the
// workspace query and the launch agree.
inline bool plan_step(const ippd_batch_t* bt, bool shared, StepPlan* pl, bool dense = false) {
  if (check_batch(bt) != IPPD_OK) return false;
  // dense-mask baseline: one-level batches, up to 64 questions per prompt
  if (dense && (!shared || bt->num_instr > 0 || bt->max_questions > 64)) return false;
  const int G = bt->num_q_heads / bt->num_kv_heads;
  const int64_t max_rows = shared ? static_cast<int64_t>(bt->max_questions) * G : G;
  // rows per context unit: 16 * rb per wave; bf16 at D = 128 with more than
  // 64 rows takes the two-group unit of 128 or 256 rows.  (Dense-mask
  // baseline: two 16-row blocks a wave, 128 rows as 4 x 32, 256 as 8 x 32.)
  const bool two_blocks_ok = bt->dtype == IPPD_DTYPE_BF16 && bt->head_dim == 128;
  int rows = bt->tile_rows;
  const int S = bt->num_instr;
  const int64_t irows = shared ? static_cast<int64_t>(bt->max_instr_questions) * G : G;
  // context tokens to stream: one-level IPPD reads each prompt once, and the
  // prompts are packed in the pool, so its size bounds their sum (a ragged
  // batch is then sized by its total, not by B times the longest)
  const int64_t ctx_tokens = shared ? std::min<int64_t>(bt->ctx_pool_tokens,
                                                        static_cast<int64_t>(bt->num_prompts) * bt->max_ctx_len)
                                    : static_cast<int64_t>(bt->num_questions) * bt->max_ctx_len;
  if (rows == 0) {
    // a two-level batch's instruction rows (all questions behind it) favour at
    // least 64-row units (measured against 32 at 6 contexts per instruction)
    int64_t sized = max_rows;
    if (S > 0 && shared) sized = std::max(sized, std::min<int64_t>(irows, 64));
    if (two_blocks_ok && shared && !dense && sized <= 64) {
      // 64 rows at least: one or two waves are slow to issue the tiles' DMAs
      // (4 questions over 16384 tokens, us a layer step: 16 rows 30.2, 64
      // 26.4; over 512 tokens 13.5, 12.7).  128 where the streams are long
      // (256 tokens a compute unit and more): the paired unit's time a tile
      // is a third (16 questions over 16384 tokens: 32.7 at 64 rows, 28.6 at
      // 128; over 8192: 21.9, 24.0).
      const int64_t stream = (ctx_tokens + static_cast<int64_t>(S) * bt->max_instr_len * (irows > 64 ? 2 : 1)) *
                             bt->num_kv_heads;
      sized = stream >= 512ll * kPlanComputeUnits ? 128 : 64;
    }
    rows = sized <= 16 ? 16 : (sized <= 32 ? 32 : (sized <= 64 ? 64 : (sized <= 128 || !two_blocks_ok ? 128 : 256)));
  }
  const bool near_uniform = bt->ctx_pool_tokens * 10 >= static_cast<int64_t>(bt->num_prompts) * bt->max_ctx_len * 9;
  // bf16 at D = 128, 128 or 256 rows: the two-group unit, eight waves and one
  // workgroup per compute unit.
  const bool paired = two_blocks_ok && !dense && rows >= 128;
  // At 128 rows each group takes every other tile: half the steps a unit, so
  // that half the compute units can stream a short batch while the others
  // serve its segments (8192 tokens x 32 questions, 4 prompts, us a layer
  // step: 47.6, as 256-row units 54.6).  With more segment tasks than half
  // the chip holds (eight a compute unit) every compute unit streams and
  // memory bounds the units: as 256-row units they keep four tiles in flight
  // instead of three (8 such prompts 81.9, as 256-row units 81.0; 8 of 4096
  // x 32 62.3, 58.7; 16 of 4096 x 20 89.3, 88.0).
  const int64_t seg_tasks = static_cast<int64_t>(bt->num_questions) * bt->num_kv_heads;
  if (paired && rows == 128 && bt->tile_rows == 0 && shared && S == 0 && near_uniform && seg_tasks > 4 * kPlanComputeUnits)
    rows = 256;
  const int rb = two_blocks_ok && (paired ? rows == 256 : rows > 64) ? 2 : 1;
  int waves = paired ? 8 : rows / (16 * rb);
  // fp32 at D = 128: the operands of eight waves do not fit their registers
  if (bt->dtype == IPPD_DTYPE_F32 && bt->head_dim == 128 && waves > 4) waves = 4;
  const int unit_rows = 16 * rb * waves;
  const int nrg = static_cast<int>((max_rows + unit_rows - 1) / unit_rows);
  // workgroups resident per compute unit (eight waves of two row blocks use
  // the registers of two, and their ring the LDS of one)
  const int wg_per_cu = paired || (waves == 8 && rb == 2) ? 1 : 2;
  const int64_t n_groups = shared ? static_cast<int64_t>(bt->num_prompts) * bt->num_kv_heads
                                  : static_cast<int64_t>(bt->num_questions) * bt->num_kv_heads;
  // two-level batch: instruction groups, (instruction, kv head) or (question, kv head)
  const int64_t n_igroups = S == 0 ? 0 : (shared ? static_cast<int64_t>(S) : bt->num_questions) * bt->num_kv_heads;
  const int nrg_i = S == 0 ? 1 : static_cast<int>((irows + unit_rows - 1) / unit_rows);
  // segment tasks (question, kv head): up to `waves` per unit, each with a
  // wave's state in the unit's LDS, whichever ring depth is chosen below
  const int64_t state_bytes = static_cast<int64_t>(G) * segment_state_row(bt->head_dim);
  const int elem = bt->dtype == IPPD_DTYPE_BF16 ? 2 : 4;
  const int ring = ring_stages(elem, bt->head_dim, paired) * ring_stage_bytes(elem, bt->head_dim);
  const int64_t seg_lds = std::min(32768, segment_main_bytes(elem, bt->head_dim, waves, ring));
  int max_tpu = 1;
  // (few tasks under a chunk that the caller fixed: one a unit, so that a
  // prompt's sums are grouped alike whatever else the batch holds)
  if (paired || seg_tasks > compute_units() || bt->chunk_tokens == 0)
    while (max_tpu < waves && 2 * max_tpu * state_bytes <= seg_lds) max_tpu *= 2;
  auto seg_units = [&](int64_t tpu) { return (seg_tasks + tpu - 1) / tpu; };
  const int max_ilen = S ? bt->max_instr_len : 0;
  auto stream_units = [&](int64_t ch) {            // context and instruction units
    return 8 * (nrg * ((n_groups * ((bt->max_ctx_len + ch - 1) / ch) + 7) / 8) +
                nrg_i * ((n_igroups * ((max_ilen + ch - 1) / ch) + 7) / 8));
  };
  const int64_t cus = compute_units(), target = cus * wg_per_cu;
  int chunk = bt->chunk_tokens;
  if (chunk == 0) {
    const int64_t work = ctx_tokens * bt->num_kv_heads * nrg + n_igroups * nrg_i * max_ilen;
    int64_t ch = (work + target - 1) / target;
    ch = (ch + 31) / 32 * 32;
    ch = ch < kMinChunk ? kMinChunk : (ch > kMaxChunk ? kMaxChunk : ch);
    // a small batch: the first chunk from small_chunk on whose units all run
    // at once, one workgroup per compute unit if some chunk up to the minimum
    // allows it (4096 tokens x 16 questions, us a layer step: 192 tokens with
    // one workgroup per compute unit 19.4, with two 20.3; 256 with one 20.1)
    if (ch == kMinChunk) {
      auto resident = [&](int64_t c, int64_t at_once) { return stream_units(c) + seg_units(max_tpu) <= at_once; };
      const int64_t at_once = resident(kMinChunk, cus) ? cus : target;
      int64_t c = small_chunk(bt, max_ilen);
      while (c < kMinChunk && !resident(c, at_once)) c += 32;
      const int64_t states = ((bt->max_ctx_len + c - 1) / c + 1 + (max_ilen + c - 1) / c) *
                             static_cast<int64_t>(bt->num_questions) * bt->num_q_heads;
      if (c < kMinChunk && states * (bt->head_dim + 2) * 4 + 512 <= static_cast<int64_t>(IPPD_NOALLOC_SCRATCH_BYTES)) ch = c;
    }
    // work / target counts no partly filled last chunk: over contexts of
    // nearly one length that can leave a second round of a few units.  The
    // smallest chunk with one round (two-level batch of 12 contexts of 1024
    // behind 3 instructions of 2048: 384 -> 512 tokens, 44.1 -> 37.4 us).
    if (ch >= kMinChunk && near_uniform) {
      // Paired units leave room for the segment units beside them: they would
      // otherwise start only when a context unit ends (32768 tokens x 64
      // questions, us a layer step: 65.2 with 32 chunks and no room, 59.1 with 24).
      const int64_t segs = paired && 2 * seg_units(max_tpu) <= cus ? seg_units(max_tpu) : 0;
      int64_t c = ch;
      while (c < 2 * ch && stream_units(c) + segs > target) c += 32;
      if (stream_units(c) + segs <= target) ch = c;
    }
    chunk = static_cast<int>(ch);
  }
  const int64_t max_chunks = (bt->max_ctx_len + chunk - 1) / chunk;
  const int64_t ctx_blocks = 8 * nrg * ((n_groups * max_chunks + 7) / 8);
  const int64_t max_ichunks = (max_ilen + chunk - 1) / chunk;
  const int64_t instr_blocks = 8 * nrg_i * ((n_igroups * max_ichunks + 7) / 8);
  const int64_t streams = ctx_blocks + instr_blocks;
  // The deep ring (one workgroup per compute unit) if every unit fits the
  // chip with it, or if the context units do and have more tiles than it
  // holds (4 prompts of 2048 x 16 questions at 256 tokens: deep 26.8 us, two
  // workgroups per compute unit 21.7); paired units always.
  const bool all_fit = streams + seg_units(max_tpu) <= cus;
  const bool deep = wg_per_cu == 1 || all_fit || (streams <= cus && chunk > kMinChunk);
  const int64_t slots = cus * (deep ? 1 : 2);
  // Segment units: as few tasks per unit as keeps every unit resident from
  // the start, if that can be; else as keeps them within one round of their
  // own (they then run after the context units).
  const int64_t room = streams + seg_units(max_tpu) <= slots ? slots - streams : slots;
  int tpu = 1;
  while (tpu < max_tpu && seg_units(tpu) > room) tpu *= 2;
  // dense-mask baseline: segment units (prompt, kv head, segment chunk, row
  // group) split the prompt's concatenated segment tiles into chunks of
  // kDenseSegTiles tiles; chunk 0 writes the segment slot, chunks 1.. the
  // slots after it (where a two-level batch keeps its instruction chunks)
  const int64_t seg_tiles = static_cast<int64_t>(bt->max_questions) * ((bt->seg_capacity + 31) / 32);
  const int64_t seg_chunks = dense ? (seg_tiles + kDenseSegTiles - 1) / kDenseSegTiles : 0;
  const int64_t seg_blocks = dense ? n_groups * seg_chunks * nrg : seg_units(tpu);
  const int64_t dense_grid = n_groups * max_chunks * nrg + seg_blocks;
  const int64_t grid = ctx_blocks + instr_blocks + seg_blocks;
  if (grid > (1ll << 30) || n_groups * max_chunks > (1ll << 30) || n_igroups * max_ichunks > (1ll << 30)) return false;
  pl->shared = shared ? 1 : 0;
  pl->waves = waves;
  pl->rb = rb;
  pl->nrg = nrg;
  pl->chunk = chunk;
  pl->max_chunks = static_cast<int>(max_chunks);
  pl->n_groups = static_cast<int>(n_groups);
  pl->grid = static_cast<int>(dense ? dense_grid : grid);
  pl->ctx_blocks = static_cast<int>(ctx_blocks);
  pl->seg_blocks = static_cast<int>(seg_blocks);
  pl->seg_tpu = tpu;
  pl->deep = deep ? 1 : 0;
  pl->dense = dense ? 1 : 0;
  pl->n_igroups = static_cast<int>(n_igroups);
  pl->nrg_i = nrg_i;
  pl->max_ichunks = static_cast<int>(dense ? seg_chunks - 1 : max_ichunks);
  pl->instr_blocks = static_cast<int>(instr_blocks);
  pl->part_slots = static_cast<size_t>(max_chunks + 1 + pl->max_ichunks) * bt->num_questions * bt->num_q_heads;
  pl->off_acc = 0;
  pl->off_ml = pl->off_acc + round256(pl->part_slots * bt->head_dim * sizeof(float));
  pl->workspace_bytes = pl->off_ml + round256(pl->part_slots * 2 * sizeof(float));
  return true;
}

// Launch plan of a prefill call (host fields only).
inline bool plan_prefill(const ippd_batch_t* bt, bool shared, int32_t max_q_tokens, PrefillPlan* pl) {
  if (check_batch(bt) != IPPD_OK || max_q_tokens < 0) return false;
  int waves = 0, rb = 0;
  if (!prefill_variant(bt->dtype, bt->head_dim, &waves, &rb)) return false;
  const int G = bt->num_q_heads / bt->num_kv_heads;
  // 256-row units that would not fill the chip (an estimate from the host
  // bounds) are halved: twice the units, each K/V fragment serving one row
  // block.  tile_rows 128 or 256 fixes the choice.
  if (rb == 2 && bt->tile_rows == 128) {
    rb = 1;
  } else if (rb == 2 && bt->tile_rows != 256) {
    const int tb2 = 16 * rb * waves / G;
    const int64_t groups = static_cast<int64_t>(shared ? bt->num_prompts : bt->num_questions) * bt->num_kv_heads;
    const int64_t qt = shared ? max_q_tokens : (max_q_tokens < bt->seg_capacity ? max_q_tokens : bt->seg_capacity);
    const int64_t units = groups * ((qt + tb2 - 1) / tb2 + (static_cast<int64_t>(bt->max_ctx_len) + tb2 - 1) / tb2);
    if (units < compute_units()) rb = 1;
  }
  const int tb = 16 * rb * waves / G;
  const int64_t n_groups = static_cast<int64_t>(shared ? bt->num_prompts : bt->num_questions) * bt->num_kv_heads;
  const int64_t gps = (n_groups + 7) / 8;
  // two-level batch: instruction rows once per instruction (IPPD) or per question (baseline)
  const int S = bt->num_instr;
  const int64_t n_igroups = S == 0 ? 0 : static_cast<int64_t>(shared ? S : bt->num_questions) * bt->num_kv_heads;
  const int64_t n_cgroups = n_groups + n_igroups, gps_c = (n_cgroups + 7) / 8;
  const int64_t qtok = shared ? max_q_tokens : (max_q_tokens < bt->seg_capacity ? max_q_tokens : bt->seg_capacity);
  const int64_t rows_c = S > 0 && bt->max_instr_len > bt->max_ctx_len ? bt->max_instr_len : bt->max_ctx_len;
  const int64_t kq = (qtok + tb - 1) / tb, kc = (rows_c + tb - 1) / tb;
  const int64_t q_blocks = 8 * gps * kq, grid = q_blocks + 8 * gps_c * kc;
  if (grid > (1ll << 30)) return false;
  pl->shared = shared ? 1 : 0;
  pl->waves = waves;
  pl->rb = rb;
  pl->tb = tb;
  pl->n_groups = static_cast<int>(n_groups);
  pl->gps = static_cast<int>(gps);
  pl->n_cgroups = static_cast<int>(n_cgroups);
  pl->gps_c = static_cast<int>(gps_c);
  pl->kq = static_cast<int>(kq);
  pl->kc = static_cast<int>(kc);
  pl->q_blocks = static_cast<int>(q_blocks);
  pl->grid = static_cast<int>(grid);
  return true;
}

}  // namespace ippd
