// Argument checks and launch plans of the library's calls: host code only, a
// function of the batch fields, so that a workspace query and a launch agree.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#include "ippd.h"
#include "ippd_internal.h"

namespace ippd {

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
// size) depends on the batch fields only and a workspace query on one thread or
// device agrees with the launch on another.
// On a part with fewer compute units the plan is still correct, only sized
// for more of them.
constexpr int kPlanComputeUnits = 256;

// What every plan of a decode call has in common.
struct StepShape {
  const ippd_batch_t* bt;
  bool shared, dense, bf16;
  int elem, D, G, S, max_ilen;
  int64_t max_rows, irows;        // rows of the widest group; of the widest instruction group
  int64_t n_groups, n_igroups;    // (prompt or question, kv head); (instruction or question, kv head)
  int64_t seg_tasks;              // (question, kv head)
  double mean_len;                // context tokens of a group, on average
  bool uniform;                   // contexts of nearly one length
  double mean_rows, mean_irows;   // rows of a group, on average
  bool uniform_rows;              // prompts (and instructions) of nearly as many rows each
};

inline StepShape step_shape(const ippd_batch_t* bt, bool shared, bool dense) {
  StepShape s;
  s.bt = bt;
  s.shared = shared;
  s.dense = dense;
  s.bf16 = bt->dtype == IPPD_DTYPE_BF16;
  s.elem = s.bf16 ? 2 : 4;
  s.D = bt->head_dim;
  s.G = bt->num_q_heads / bt->num_kv_heads;
  s.S = bt->num_instr;
  s.max_ilen = s.S ? bt->max_instr_len : 0;
  s.max_rows = shared ? static_cast<int64_t>(bt->max_questions) * s.G : s.G;
  s.irows = shared ? static_cast<int64_t>(bt->max_instr_questions) * s.G : s.G;
  const int64_t hk = bt->num_kv_heads, nt = bt->num_questions;
  s.n_groups = (shared ? bt->num_prompts : nt) * hk;
  s.n_igroups = s.S == 0 ? 0 : (shared ? s.S : nt) * hk;
  s.seg_tasks = nt * hk;
  // one-level IPPD reads each prompt once, and the prompts are packed in the
  // pool, so its size bounds their sum (a ragged batch is then sized by its
  // total, not by B times the longest)
  const double mx = bt->max_ctx_len;
  const double in_pool = static_cast<double>(bt->ctx_pool_tokens) - static_cast<double>(s.S) * s.max_ilen;
  s.mean_len = std::max(std::min(mx, in_pool / bt->num_prompts), mx / bt->num_prompts);
  s.uniform = s.mean_len >= 0.9 * mx;
  s.mean_rows = shared ? static_cast<double>(nt) / bt->num_prompts * s.G : s.G;
  s.mean_irows = s.S == 0 ? 0.0 : (shared ? static_cast<double>(nt) / s.S * s.G : s.G);
  s.uniform_rows = s.mean_rows >= 0.9 * s.max_rows && (s.S == 0 || s.mean_irows >= 0.9 * s.irows);
  return s;
}

// Pieces of `size` that a group of `mean` parts into on average, where the
// largest parts into `most`.
inline double mean_pieces(double mean, bool uniform, double size, double most) {
  return uniform ? most : std::min(most, std::max(mean / size + 0.5, 1.0));
}

// Context and instruction units with tokens and rows, on average.
struct Streams {
  double most, ichunks;       // chunks of the longest context, and of the longest instruction
  double chunks;              // chunks of a context, on average
  double ctx, instr;          // units
};
inline Streams stream_units(const StepShape& s, int unit_rows, int nrg, int nrg_i, int chunk) {
  Streams u;
  const bool even = s.mean_rows >= 0.9 * s.max_rows, even_i = s.mean_irows >= 0.9 * s.irows;
  u.most = static_cast<double>((static_cast<uint32_t>(s.bt->max_ctx_len) + chunk - 1u) / chunk);
  u.ichunks = static_cast<double>((static_cast<uint32_t>(s.max_ilen) + chunk - 1u) / chunk);
  u.chunks = mean_pieces(s.mean_len, s.uniform, chunk, u.most);
  // (a chunk's row groups go to one of the 8 XCDs, which its units wait for)
  u.ctx = 8.0 * ceil(s.n_groups * u.chunks / 8) * mean_pieces(s.mean_rows, even, unit_rows, nrg);
  u.instr = s.S == 0 ? 0.0 : 8.0 * ceil(s.n_igroups * u.ichunks / 8) * mean_pieces(s.mean_irows, even_i, unit_rows, nrg_i);
  return u;
}

// Rows of a unit asked for as `rows`, and its waves.  bf16 at D = 128 with
// 128 or 256 rows is the two-group unit, eight waves and one workgroup per
// compute unit.  (Dense-mask baseline: two 16-row blocks a wave, 128 rows as
// 4 x 32, 256 as 8 x 32.)  Others: 16 rows a wave, two workgroups per compute
// unit, or for fp32 one with the deep ring (few units of many rows: 32 heads,
// 3 prompts of 4920 tokens x 16 questions 54 us, with two workgroups 77; bf16
// units never gained by it); fp32 at D = 128 four waves at most (the operands
// of eight do not fit their registers).
struct UnitKind {
  bool paired, deep;
  int rb, waves, rows;
  int at_once() const { return kPlanComputeUnits * (paired || deep ? 1 : 2); }   // units resident on the chip
};
inline UnitKind unit_kind(const StepShape& s, int rows, bool deep) {
  UnitKind k;
  k.deep = deep && !s.bf16 && !s.dense;
  const bool wide = s.bf16 && s.D == 128;
  k.paired = wide && !s.dense && rows >= 128;
  k.rb = wide && (k.paired ? rows == 256 : rows > 64) ? 2 : 1;
  k.waves = k.paired ? 8 : rows / (16 * k.rb);
  if (!s.bf16 && s.D == 128 && k.waves > 4) k.waves = 4;
  k.rows = 16 * k.rb * k.waves;
  return k;
}

// Segment tasks (question, kv head) per unit: up to one a wave, each with a
// wave's state in the unit's LDS; as few as keeps every unit resident beside
// the `streams` from the start, if that can be, else as keeps them within one
// round of their own (they then run after the context units; units past a
// context's end leave at once).  Few tasks under a chunk that the caller
// fixed: one a unit, so that a prompt's sums are grouped alike whatever else
// the batch holds.
inline int segment_tasks_per_unit(const StepShape& s, const UnitKind& k, double streams) {
  const int state_bytes = s.G * segment_state_row(s.D);
  const int ring = ring_stages(s.elem, s.D, k.paired || k.deep) * ring_stage_bytes(s.elem, s.D);
  const int lds = std::min(32768, segment_main_bytes(s.elem, s.D, k.waves, ring));
  int most = 1;
  if (k.paired || s.seg_tasks > kPlanComputeUnits || s.bt->chunk_tokens == 0)
    while (most < k.waves && 2 * most * state_bytes <= lds) most *= 2;
  const double slots = k.at_once();
  const double room = streams + (s.seg_tasks + most - 1) / most <= slots ? slots - streams : slots;
  int tpu = 1;
  while (tpu < most && (s.seg_tasks + tpu - 1) / tpu > room) tpu *= 2;
  return tpu;
}

// Launch plan with such units over chunks of `chunk` tokens.
inline bool make_step_plan(const StepShape& s, const UnitKind& k, int chunk, StepPlan* pl) {
  const ippd_batch_t* bt = s.bt;
  const int unit_rows = k.rows;
  const int nrg = static_cast<int>((s.max_rows + unit_rows - 1) / unit_rows);
  const int nrg_i = s.S == 0 ? 1 : static_cast<int>((s.irows + unit_rows - 1) / unit_rows);
  const int64_t max_chunks = (static_cast<int64_t>(bt->max_ctx_len) + chunk - 1) / chunk;
  const int64_t max_ichunks = (static_cast<int64_t>(s.max_ilen) + chunk - 1) / chunk;
  const int64_t ctx_blocks = 8 * nrg * ((s.n_groups * max_chunks + 7) / 8);
  const int64_t instr_blocks = 8 * nrg_i * ((s.n_igroups * max_ichunks + 7) / 8);
  const Streams u = stream_units(s, unit_rows, nrg, nrg_i, chunk);
  const int tpu = segment_tasks_per_unit(s, k, u.ctx + u.instr);
  // dense-mask baseline: segment units (prompt, kv head, segment chunk, row
  // group) split the prompt's concatenated segment tiles into chunks of
  // kDenseSegTiles tiles; chunk 0 writes the segment slot, chunks 1.. the
  // slots after it (where a two-level batch keeps its instruction chunks)
  const int64_t seg_tiles = static_cast<int64_t>(bt->max_questions) * ((bt->seg_capacity + 31) / 32);
  const int64_t seg_chunks = s.dense ? (seg_tiles + kDenseSegTiles - 1) / kDenseSegTiles : 0;
  const int64_t seg_blocks = s.dense ? s.n_groups * seg_chunks * nrg : (s.seg_tasks + tpu - 1) / tpu;
  const int64_t dense_grid = s.n_groups * max_chunks * nrg + seg_blocks;
  const int64_t grid = ctx_blocks + instr_blocks + seg_blocks;
  if (grid > (1ll << 30) || s.n_groups * max_chunks > (1ll << 30) || s.n_igroups * max_ichunks > (1ll << 30))
    return false;
  pl->shared = s.shared ? 1 : 0;
  pl->waves = k.waves;
  pl->rb = k.rb;
  pl->nrg = nrg;
  pl->chunk = chunk;
  pl->max_chunks = static_cast<int>(max_chunks);
  pl->n_groups = static_cast<int>(s.n_groups);
  pl->grid = static_cast<int>(s.dense ? dense_grid : grid);
  pl->ctx_blocks = static_cast<int>(ctx_blocks);
  pl->seg_blocks = static_cast<int>(seg_blocks);
  pl->seg_tpu = tpu;
  pl->deep = k.deep ? 1 : 0;
  pl->dense = s.dense ? 1 : 0;
  pl->n_igroups = static_cast<int>(s.n_igroups);
  pl->nrg_i = nrg_i;
  pl->max_ichunks = static_cast<int>(s.dense ? seg_chunks - 1 : max_ichunks);
  pl->instr_blocks = static_cast<int>(instr_blocks);
  pl->part_slots = static_cast<size_t>(max_chunks + 1 + pl->max_ichunks) * bt->num_questions * bt->num_q_heads;
  pl->off_acc = 0;
  pl->off_ml = pl->off_acc + round256(pl->part_slots * bt->head_dim * sizeof(float));
  pl->workspace_bytes = pl->off_ml + round256(pl->part_slots * 2 * sizeof(float));
  return true;
}

// The parts of a decode call's time, us.  Fitted to the times of 1407 batch
// shapes (1 to 32 prompts of 50 to 32768 tokens, 1 to 64 questions, uniform,
// ragged and two-level, five head shapes) at up to 27 chunks with every unit.
// The plan with the least estimated time took on average 1.03 times the best
// one measured, and 0.86 times the plan by a 256-token minimum and rows alone.
// No single part decides: 16 prompts of 1376 tokens x 3 questions take 31 us
// as 384 units of 32 rows, 35 as 128 of 128 rows (half the chip idle); 2 of
// 7000 and fewer x 21 questions 26 as 224 units, 41 as 94 of twice the chunk.
struct UnitCost {
  double start;               // a context unit's begin and end
  double tile, beside;        // a 32-token tile, alone on the compute unit and beside another unit
  double rate;                // MB/us at which many such units stream
};
struct StepCosts {
  UnitCost unit[6];           // of 32, 64 and 128 rows; bf16: of 256 with up to and with more than 128 in use;
                              // fp32: the first three again with the deep ring
  double seg_start, seg_tile; // a segment unit, and a 32-token tile of one of its waves
  double second;              // the first units beside others weigh so much of `beside`
  double last_round;          // an unfilled last round counts at least so much of a round
  double longest;             // ragged: the longest unit's share at the end
  double empty;               // a unit past its context's end or its prompt's rows
  double seg_last, seg_free;  // even batch: as last_round; share of a free compute unit's time that serves segments
  double seg_least, seg_share;             // ragged batch: rounds of segment units after the streams
  double seg_fill, seg_mb;    // share of the segments' capacity that streams beside; us/MB of it after
  double merge, merge_slot, merge_state;   // the merge, a chunk, a million state elements
};
constexpr double kStopped = 0.25;
inline const StepCosts& step_costs(const StepShape& s) {
  static constexpr StepCosts costs[] = {          // bf16 at D = 64 and 128, fp32 at 64 and 128
    {{{2.76, 0.49, 0.34, 6.54}, {2.27, 0.44, 0.40, 8.18}, {4.19, 0.35, 0.63, 7.84}},
     2.61, 1.49, 0.12, 0.22, 0.31, 1.69, 0.014, 1.00, 0.084, 0.067, 1.59, 0.16, 6.16, 0.029, 2.52},
    {{{4.09, 0.66, 0.64, 7.64}, {3.40, 0.63, 0.84, 7.91}, {10.03, 0.30, 0.30, 6.08},
      {7.07, 0.48, 0.48, 7.07}, {9.84, 0.42, 0.42, 6.69}},
     1.51, 3.15, 1.40, 0.95, 0.57, 6.10, 0.30, 0.20, 0.57, 0.81, 0.85, 0.052, 7.04, 0.033, 2.00},
    {{{4.20, 1.32, 1.08, 4.98}, {3.41, 1.16, 1.59, 6.11}, {4.24, 1.49, 1.79, 5.45},
      {2.90, 1.40, 1.40, 3.77}, {1.82, 1.43, 1.43, 3.78}, {4.10, 1.01, 1.01, 3.60}},
     0.81, 2.34, 1.43, 0.94, 0.58, 10.06, 1.00, 1.00, 0.70, 0.68, 1.73, 0.093, 6.67, 0.021, 5.03},
    {{{4.78, 2.77, 3.13, 7.77}, {5.58, 2.52, 3.83, 8.13}, {5.58, 2.52, 3.83, 8.13},
      {6.20, 2.54, 2.54, 4.23}, {5.81, 2.64, 2.64, 6.61}, {5.81, 2.64, 2.64, 6.61}},
     0.031, 3.66, 0.51, 0.58, 0.40, 3.13, 1.00, 1.00, 0.72, 0.96, 2.21, 0.004, 5.73, 0.034, 3.13}};
  return costs[(s.bf16 ? 0 : 2) + (s.D == 64 ? 0 : 1)];
}

// Estimated time of a decode call, us: the streams (their longest chain, or
// round by round where they need more than one, and the memory's time), the
// segment units beside or after them, and the merge.  The host knows how many
// tokens and questions a batch has, not which prompt has them; in a ragged
// batch a limit therefore counts as crossed by degrees.
inline double step_time(const StepShape& s, const UnitKind& k, int nrg, int nrg_i, int chunk, const Streams& u) {
  const StepCosts& c = step_costs(s);
  const int64_t widest = std::max(s.max_rows, s.S ? s.irows : 0);
  const UnitCost& uc = c.unit[k.rows == 256 ? (widest <= 128 ? 3 : 4)
                                       : (k.deep ? 3 : 0) + (k.rows <= 32 ? 0 : k.rows == 64 ? 1 : 2)];
  const double total = u.ctx + u.instr, cus = kPlanComputeUnits, slots = k.at_once();
  const int mx = s.bt->max_ctx_len;
  const bool sure = s.uniform && s.uniform_rows, even = s.uniform && s.S == 0;
  auto over = [&](double n, double limit) {
    return sure ? (n > limit ? 1.0 : 0.0) : std::min(1.0, std::max(0.0, (n / limit - 0.86) / 0.2));
  };
  auto both = [](double x, double y) { return sqrt(x * x + y * y); };
  // tiles of a unit: of an average one, of the longest, of an instruction's
  const double longest = s.uniform && u.most > 0 ? ceil(mx / (u.most * 32)) : std::min(chunk, mx) / 32.0;
  const double tiles = s.uniform ? longest : s.mean_len / u.chunks / 32.0;
  const double itiles = std::min(chunk, s.max_ilen) / 32.0;
  double tile = uc.tile;
  if (!k.paired && !k.deep)
    tile += (uc.beside - uc.tile) * over(total, cus) *
            (c.second + (1.0 - c.second) * std::min(1.0, std::max(0.0, (total - cus) / cus)));
  const double one = tiles * tile + uc.start, chain = std::max(longest, itiles) * tile + uc.start;
  const double mb = 2e-6 * s.elem * s.D;           // MB of a token's keys and values of one head
  const double stream_mb = mb * (s.n_groups * s.mean_len + static_cast<double>(s.n_igroups) * s.max_ilen);
  const double seg_mb = mb * s.seg_tasks * s.bt->seg_capacity;
  const double rounds = total / slots, whole = floor(rounds + 1e-9), part = std::max(0.0, rounds - whole);
  auto streams = [&](double bytes) {
    const double mem = bytes / uc.rate;
    if (even) {
      const double round = rounds > 0.0 ? mem / rounds : 0.0;
      const double last = part > 1e-6 ? both(one, part * round) : 0.0;
      return whole * both(one, round) + last * (whole > 0.0 ? c.last_round + (1.0 - c.last_round) * part : 1.0);
    }
    const double work = (u.ctx * one + u.instr * (itiles * tile + uc.start)) / slots;
    const double under = both(chain, mem), more = both(std::max(work + c.longest * chain, chain), mem);
    return under + over(total, slots) * (more - under);
  };
  const int tpu = segment_tasks_per_unit(s, k, total);
  const double segs = static_cast<double>((s.seg_tasks + tpu - 1) / tpu);
  const double seg = c.seg_start + c.seg_tile * std::max(1.0, s.bt->seg_capacity / 32.0 * tpu / k.waves);
  const double filled = std::max(streams(stream_mb + c.seg_fill * seg_mb), seg), alone = streams(stream_mb);
  double t;
  if (even) {
    // compute units that the last round leaves free serve segment units meanwhile
    const double vacant = slots * (std::max(1.0, ceil(rounds - 1e-9)) - rounds);
    const double left = std::max(0.0, segs - vacant * (1.0 + c.seg_free * std::max(0.0, (rounds <= 1.0 ? filled : one) / seg - 1.0)));
    const double q = left / slots;
    t = filled + seg * (q + c.seg_last * (ceil(q - 1e-9) - q));
  } else {
    const double after = alone + seg * std::max(c.seg_least, c.seg_share * segs / slots) + c.seg_mb * seg_mb;
    t = filled + over(total + segs, slots) * (after - filled);
  }
  // Questions stop one after another, and one plan serves them from the first
  // step to the last: part of the time is that of a step without segments.
  // (8 prompts of 8192 tokens x 32 questions, six in ten still answering: 192
  // units that leave room for the segments 87 us, 256 units 82.)
  t += kStopped * (alone - t);
  const double blocks = static_cast<double>(s.n_groups) * nrg * u.most + static_cast<double>(s.n_igroups) * nrg_i * u.ichunks;
  if (blocks > slots) t += std::max(0.0, blocks - total) * c.empty / slots;
  const double states = u.most + 1.0 + u.ichunks;
  return t + c.merge + c.merge_slot * states +
         c.merge_state * 1e-6 * states * s.bt->num_questions * s.bt->num_q_heads * s.D;
}

// Launch plan of a decode call.  Depends only on host fields, so the
// workspace query and the launch agree.
inline bool choose_step_plan(const ippd_batch_t* bt, bool shared, StepPlan* pl, bool dense) {
  // dense-mask baseline: one-level batches, up to 64 questions per prompt
  if (dense && (!shared || bt->num_instr > 0 || bt->max_questions > 64)) return false;
  const StepShape s = step_shape(bt, shared, dense);
  int rows = bt->tile_rows, chunk = bt->chunk_tokens;
  const bool wide = s.bf16 && s.D == 128;
  if (dense) {
    // its units serve all rows of a prompt, over the IPPD call's chunks, so
    // that its workspace holds that call's states too
    if (rows == 0) rows = s.max_rows <= 16 ? 16 : s.max_rows <= 32 ? 32 : s.max_rows <= 64 ? 64 : s.max_rows <= 128 || !wide ? 128 : 256;
    if (chunk == 0) {
      if (!choose_step_plan(bt, true, pl, false)) return false;
      chunk = pl->chunk;
    }
    return make_step_plan(s, unit_kind(s, rows, false), chunk, pl);
  }
  if (rows == 0 && chunk != 0)                     // by the prompt's rows alone: see segment_tasks_per_unit
    rows = wide ? (s.max_rows <= 64 ? 64 : s.max_rows <= 128 ? 128 : 256) : (s.max_rows <= 32 ? 32 : s.max_rows <= 64 ? 64 : 128);

  // The unit and chunk with the least estimated time.  A plan whose partial
  // states fit the no-allocation step's scratch goes before any that does not.
  static constexpr int kRows[] = {32, 64, 128, 256};
  static constexpr int kChunks[] = {32,  64,  96,  128,  160,  192,  224,  256,  320,  384,  448,  512,  640, 768,
                                    896, 1024, 1280, 1536, 1792, 2048, 2560, 3072, 3584, 4096, 5120, 6144, 8192};
  constexpr int kLast = sizeof kChunks / sizeof *kChunks - 1;
  const int longest = std::max(bt->max_ctx_len, s.max_ilen);
  const int64_t widest = std::max(s.max_rows, s.S ? s.irows : 0);
  const int largest = wide ? 256 : s.bf16 || s.D == 64 ? 128 : 64;
  const double state = static_cast<double>(bt->num_questions) * bt->num_q_heads * (s.D + 2) * 4;
  double best = INFINITY;
  bool best_fits = false;
  UnitKind best_kind = unit_kind(s, rows ? rows : largest, false);
  int best_chunk = chunk ? chunk : kChunks[kLast];
  auto consider_kind = [&](const UnitKind& k) {
    const double slots = k.at_once();
    const int nrg = static_cast<int>((s.max_rows + k.rows - 1) / k.rows);
    const int nrg_i = s.S == 0 ? 0 : static_cast<int>((s.irows + k.rows - 1) / k.rows);
    double least = INFINITY;                       // of this unit's chunks
    auto consider = [&](int ch, const Streams& u) {
      const bool fits = (u.most + 1.0 + u.ichunks) * state + 512 <= IPPD_NOALLOC_SCRATCH_BYTES;
      if (best_fits && !fits) return 0.0;
      const double t = step_time(s, k, nrg, nrg_i, ch, u);
      least = std::min(least, t);
      if (t < best || (fits && !best_fits)) {
        best = t;
        best_fits = fits;
        best_kind = k;
        best_chunk = ch;
      }
      return t;
    };
    if (chunk != 0) {
      consider(chunk, stream_units(s, k.rows, nrg, nrg_i, chunk));
      return;
    }
    for (int c = 0; c <= kLast; ++c) {
      const int ch = kChunks[c];
      const Streams u = stream_units(s, k.rows, nrg, nrg_i, ch);
      const bool more = c < kLast && ch < longest;   // a larger chunk gives fewer units
      if (more && u.ctx + u.instr > 4 * slots) continue;
      const double t = consider(ch, u);
      if (!more || t > 1.5 * least) break;           // past the least: fewer, longer chains
    }
    // the chunks with which the units fill one round exactly, with the segment
    // units beside them and without (32768 tokens x 64 questions: 24 chunks of
    // 1376 tokens 60 us, 26 of 1280 64, 22 of 1536 63)
    const Streams one = stream_units(s, k.rows, nrg, nrg_i, kChunks[kLast]);
    const double per_chunk = one.ctx / one.chunks;   // units of one chunk of every group
    for (const double room : {slots, slots - (s.seg_tasks + k.waves - 1) / k.waves}) {
      if (s.S > 0 || !(per_chunk > 0.0) || per_chunk > room) continue;
      const double len = s.uniform ? bt->max_ctx_len : s.mean_len;
      const double fit = 32.0 * ceil(len / floor(room / per_chunk) / 32);
      if (fit < 32.0 || fit > kChunks[kLast]) continue;
      const int ch = static_cast<int>(fit);
      consider(ch, stream_units(s, k.rows, nrg, nrg_i, ch));
    }
  };
  for (const int r : kRows) {
    if (rows != 0 ? r != 32 : r > largest) break;
    if (rows == 0 && (r < std::min(128, largest) ? 4 * r < s.max_rows : r == 256 && r >= 4 * widest)) continue;
    consider_kind(unit_kind(s, rows ? rows : r, false));
    if (!s.bf16) consider_kind(unit_kind(s, rows ? rows : r, true));
  }
  return make_step_plan(s, best_kind, best_chunk, pl);
}

// The same, through this thread's last plan: a decode loop asks for one plan
// at every layer and step, and choosing it takes about 2 us.  The key is the
// value of every field that a plan depends on.
inline bool plan_step(const ippd_batch_t* bt, bool shared, StepPlan* pl, bool dense = false) {
  if (check_batch(bt) != IPPD_OK) return false;
  const int64_t key[] = {shared, dense, bt->num_prompts, bt->num_questions, bt->num_q_heads, bt->num_kv_heads,
                         bt->head_dim, bt->dtype, bt->ctx_pool_tokens, bt->seg_capacity, bt->max_ctx_len,
                         bt->max_questions, bt->chunk_tokens, bt->tile_rows, bt->num_instr,
                         bt->num_instr ? bt->max_instr_len : 0, bt->num_instr ? bt->max_instr_questions : 0};
  static thread_local struct {
    int64_t of[sizeof key / sizeof *key];            // (no prompts: no plan yet)
    StepPlan plan;
  } last;
  if (memcmp(last.of, key, sizeof key) != 0) {
    StepPlan chosen;
    if (!choose_step_plan(bt, shared, &chosen, dense)) return false;
    last.plan = chosen;
    memcpy(last.of, key, sizeof key);
  }
  *pl = last.plan;
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
    if (units < kPlanComputeUnits) rb = 1;
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
  pl->n_cgroups = static_cast<int>(n_cgroups);
  pl->kq = static_cast<int>(kq);
  pl->kc = static_cast<int>(kc);
  pl->q_blocks = static_cast<int>(q_blocks);
  pl->grid = static_cast<int>(grid);
  return true;
}

}  // namespace ippd
