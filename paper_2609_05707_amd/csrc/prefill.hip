// IPPD stacked-prompt prefill attention on gfx950 (one launch per call).
//
// The prefill is the forward pass over the prompt header before any answer
// token exists (Sec. 4.1): every header token is a query row.  With the mask
// M_fin of the stacked prompt, a context token attends causally to its own
// context, and a question token attends to the whole context of its prompt
// and causally to its own question (M_ctx, M_qtn, M_caus with >=); every
// question's tokens start at the same virtual position, right after the
// context.  The IPPD form of this computation serves the rows of all
// questions of a prompt from one pass over the context (the shared keys and
// values come from memory once for the whole question set, Sec. 4.3, and
// App. A.2 for the prefill dimensions), and computes the context rows once.
// The standard baseline prefills every question's own prompt
// [context; question] (Sec. 3), so it streams the context and recomputes the
// context rows once per question.
//
// A group is (prompt b, kv head g) for IPPD or (question i, kv head g) for
// the baseline.  A unit serves tb query tokens x G heads (row r = token r / G,
// head g*G + r % G) and streams the keys its rows see as 32-key tiles through
// an LDS ring; a per-row limit hides the keys a row may not see.  Every unit
// sees all keys of its rows, so it writes normalised outputs directly: no
// split-K, no workspace.  bf16 units (256 or 128 rows) run the two wave
// groups of prefill_pingpong.h, fp32 units (128 or 64 rows) the decode
// kernels' ring and products (tile_attend.h).
//   question-row units  tokens k*tb .. of the group's questions (packed in
//                       question order): the whole context unmasked, then the
//                       tiles of each question present, visible to that
//                       question's rows up to their own token (causal);
//   context-row units   context tokens k*tb .. (k+1)*tb - 1: context tiles
//                       up to the block's last token, causal on the diagonal.
//   instruction-row units (two-level batch, Sec. 4.4) instruction tokens
//                       k*tb .., causal over the instruction alone.
// In a two-level batch every prompt behind instruction p is [p; c_b; x_i]:
// question-row and context-row units first stream p's tiles, all visible,
// and the positions of c_b and x_i move up by |p|.  IPPD computes p's rows
// once per instruction; the baseline recomputes them (and the context rows)
// once per question.
// Question-row units come first in the grid (each streams a whole context),
// then context-row and instruction-row units.  Unit u of either kind runs on
// XCD u & 7, which holds every unit of the groups 8j + (u & 7); there the
// units of a group follow each other, the longest causal block first, so the
// units that run at one time share a group's keys and values through that
// XCD's L2.  (With the blocks of all groups interleaved, a ragged batch of 8
// prompts kept 8 contexts in flight per XCD and fetched most tiles from
// beyond the L2: 1.90 ms against 1.38.)  Groups are numbered kv head minor,
// so each XCD gets its share of every prompt.
#include <limits.h>
#include <stddef.h>

#include "ippd.h"
#include "ippd_device.h"
#include "ippd_internal.h"
#include "prefill_pingpong.h"
#include "tile_attend.h"

namespace ippd {

template <typename T, int D, int NS>
struct PrefillLds {
  alignas(16) unsigned char ring[NS * Ring<T, D, NS>::STAGE];
  int pre[kMaxQuestionsPerPrompt + 1];   // question-row units: prefix sums of the group's question lengths
};

// Index j with pre[j] <= tau < pre[j + 1] (pre non-decreasing, pre[0] = 0 <= tau < pre[n]).
__device__ __forceinline__ int find_question(const int* pre, int n, int tau) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= tau) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// A unit's place in the grid: its group, row block and the key ranges its
// rows see.
struct Unit {
  bool qunit;                // question rows; else context (or instruction) rows
  int k;                     // row block of the group
  int g, qa, nq;             // kv head; first question and question count of the group
  int64_t coff, poff;        // pool offset of the rows' tokens; of the visible prefix before them
  int lc, lp;                // tokens of either
  int S;                     // question tokens of the group (question rows)
};

// Finds the workgroup's unit, and for question rows the prefix sums of the
// group's question lengths (into pre[0..nq]).  False if the unit has no rows
// or a broken layout (flagged); uniform over the workgroup.
template <int NW>
__device__ __forceinline__ bool find_unit(const PrefillParams& p, int* pre, int wave, int lane, Unit& un) {
  const int blk = static_cast<int>(blockIdx.x);
  const bool qunit = blk < p.q_blocks;
  const int ub = qunit ? blk : blk - p.q_blocks;
  const int slice = ub & 7, local = ub >> 3;
  const int nk = qunit ? p.kq : p.kc, gi = local / nk, kk = local - gi * nk, grp = 8 * gi + slice;
  if (grp >= (qunit ? p.n_groups : p.n_cgroups)) return false;
  const int k = qunit ? kk : p.kc - 1 - kk;
  const int TB = p.tb;
  // context-row groups past n_groups hold the rows of an instruction
  const bool irows = grp >= p.n_groups;
  const int gl = irows ? grp - p.n_groups : grp;

  int b, g, qa, nq, s = 0;
  int64_t off0 = 0;                               // the prompt's context, if its load can go out right away
  int len0 = 0;
  // kv head minor: the XCD slice (group % 8) cycles over kv heads, which
  // carry equal work, rather than over prompts of different lengths
  if (irows && p.shared) {
    s = gl / p.Hkv;
    g = gl - s * p.Hkv;
    b = 0;
    qa = 0;
    nq = 0;
  } else if (p.shared) {
    b = gl / p.Hkv;
    g = gl - b * p.Hkv;
    off0 = p.ctx_off[b];                          // all four in one round trip
    len0 = p.ctx_len[b];
    qa = p.q_start[b];
    nq = p.q_start[b + 1] - qa;
  } else {
    qa = gl / p.Hkv;
    g = gl - qa * p.Hkv;
    nq = 1;
    b = prompt_of(p.q_start, p.B, qa);
  }
  if (b >= p.B || qa < 0 || nq < 0 || nq > kMaxQuestionsPerPrompt || qa + nq > p.Nt || (irows && s >= p.S)) {
    if (threadIdx.x == 0 && k == 0) raise_flag(p.err_flag, kFlagBadLayout);
    return false;
  }
  if (p.S > 0 && !(irows && p.shared)) s = instr_of_prompt(p.instr_start, p.S, b);
  // this unit's rows: tokens coff .. coff+lc-1, after lp visible prefix tokens at poff
  int64_t coff, poff = 0;
  int lc, lp = 0;
  if (p.S > 0) {
    poff = p.instr_off[s];
    lp = p.instr_len[s];
    if (lp < 0 || lp > p.max_instr_len || (poff & 7) != 0 || poff < 0 || poff + lp > p.pool) {
      if (threadIdx.x == 0 && k == 0) raise_flag(p.err_flag, kFlagBadLayout);
      return false;
    }
  }
  if (irows) {
    coff = poff;
    lc = lp;
    poff = 0;
    lp = 0;
  } else {
    coff = p.shared ? off0 : p.ctx_off[b];
    lc = p.shared ? len0 : p.ctx_len[b];
    if (lc < 0 || lc > p.max_ctx_len || (coff & 7) != 0 || coff < 0 || coff + lc > p.pool) {
      if (threadIdx.x == 0 && k == 0) raise_flag(p.err_flag, kFlagBadLayout);
      return false;
    }
  }

  // question-row units: prefix sums of the group's question lengths
  int S = 0;                                      // question tokens of the group
  if (qunit) {
    for (int e = threadIdx.x; e < nq; e += 64 * NW) {
      int s = p.seg_len[qa + e];
      if (s < 0 || s > p.seg_cap) {
        raise_flag(p.err_flag, kFlagBadLayout);
        s = s < 0 ? 0 : p.seg_cap;
      }
      pre[e + 1] = s;
    }
    if (threadIdx.x == 0) pre[0] = 0;
    __syncthreads();
    if (wave == 0) {
      // lane l sums entries l*per+1 .. (l+1)*per, then an exclusive scan of the lane sums
      const int per = (nq + 63) / 64;
      int run = 0;
      for (int e = 0; e < per; ++e) {
        const int x = lane * per + e;
        run += x < nq ? pre[x + 1] : 0;
      }
      int incl = run;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(incl, d, 64);
        incl += lane >= d ? y : 0;
      }
      int acc = incl - run;
      for (int e = 0; e < per; ++e) {
        const int x = lane * per + e;
        if (x < nq) {
          acc += pre[x + 1];
          pre[x + 1] = acc;
        }
      }
    }
    __syncthreads();
    S = pre[nq];
    if (k == 0 && threadIdx.x == 0 && S > p.kq * TB) raise_flag(p.err_flag, kFlagBadLayout);
    if (k * TB >= S) return false;                // uniform: every thread read the same total
  } else if (k * TB >= lc) {
    return false;
  }
  un.qunit = qunit;
  un.k = k;
  un.g = g;
  un.qa = qa;
  un.nq = nq;
  un.coff = coff;
  un.poff = poff;
  un.lc = lc;
  un.lp = lp;
  un.S = S;
  return true;
}

// One query row: where its query comes from and its output goes, and which
// keys it sees.
struct QueryRow {
  int64_t at;                // element offset of the row in q_ctx / out_ctx or q_seg / out_seg
  int64_t pos;               // (virtual) position
  int lim;                   // context row: causal limit (context token); question row: own token
  int j;                     // question row: its question (relative); else -1
  bool valid;                // else the row repeats the block's first token and is not written
};

template <int D>
__device__ __forceinline__ QueryRow find_row(const PrefillParams& p, const Unit& un, const int* pre, int row) {
  QueryRow r;
  const int G = p.G, TB = p.tb;
  const int tr = row / G, h = un.g * G + row % G;
  const int t = un.k * TB + tr;
  r.valid = row < TB * G && t < (un.qunit ? un.S : un.lc);
  const int tc = r.valid ? t : un.k * TB;
  if (un.qunit) {
    r.j = un.nq == 1 ? 0 : find_question(pre, un.nq, tc);
    const int u = tc - pre[r.j];
    r.lim = u;
    r.pos = static_cast<int64_t>(un.lp) + un.lc + u;
    r.at = ((static_cast<int64_t>(un.qa + r.j) * p.seg_cap + u) * p.Hq + h) * D;
  } else {
    r.j = -1;
    r.lim = tc;
    r.pos = static_cast<int64_t>(un.lp) + tc;
    r.at = ((un.coff + tc) * p.Hq + h) * D;
  }
  return r;
}

// The keys of a unit in order, as regions of whole 32-key tiles: the
// instruction (two-level batch), the context up to kv_end, then the questions
// jlo .. jhi (relative to the group's first question).
struct KeySeq {
  int n;                     // tiles
  int jlo, nreg, lp, kv_end;
  const int* pre;
  __device__ __forceinline__ KeySeq(const PrefillParams& p, const Unit& un, const int* pre_) : pre(pre_) {
    const int TB = p.tb;
    lp = un.lp;
    kv_end = un.qunit ? un.lc : min(un.k * TB + TB, un.lc);
    jlo = 0;
    nreg = 2;
    int nst = 0;
    if (un.qunit) {
      jlo = un.nq == 1 ? 0 : find_question(pre, un.nq, un.k * TB);
      const int jhi = un.nq == 1 ? 0 : find_question(pre, un.nq, min(un.k * TB + TB, un.S) - 1);
      nreg = 3 + jhi - jlo;
      for (int j = jlo; j <= jhi; ++j) nst += (pre[j + 1] - pre[j] + 31) >> 5;
    }
    n = __builtin_amdgcn_readfirstlane(((lp + 31) >> 5) + ((kv_end + 31) >> 5) + nst);
    jlo = __builtin_amdgcn_readfirstlane(jlo);
    nreg = __builtin_amdgcn_readfirstlane(nreg);
  }
  __device__ __forceinline__ int tokens(int reg) const {
    if (reg < 2) return reg == 0 ? lp : kv_end;
    return __builtin_amdgcn_readfirstlane(pre[jlo + reg - 1] - pre[jlo + reg - 2]);
  }
};

// A place in the sequence: tile at token `at` of region `reg`, `rem` tokens
// of the region from there on.  A unit's sequence is never empty.
struct KeyCursor {
  int reg, at, rem;
  __device__ __forceinline__ void region(const KeySeq& ks, int first) {
    at = 0;
    for (reg = first;; ++reg) {
      rem = ks.tokens(reg);
      if (rem > 0 || reg + 1 >= ks.nreg) return;
    }
  }
  // the next tile; true if it begins a region (the last tile stays in place)
  __device__ __forceinline__ bool next(const KeySeq& ks) {
    if (rem > 32) {
      at += 32;
      rem -= 32;
      return false;
    }
    if (reg + 1 >= ks.nreg) return false;
    region(ks, reg + 1);
    return true;
  }
};

// Last key, relative to a region's first, that a row sees of it (-1: none).
__device__ __forceinline__ int region_limit(const Unit& un, const KeySeq& ks, const QueryRow& r, int reg) {
  if (reg >= 2) return r.j == ks.jlo + reg - 2 ? r.lim : -1;
  return reg == 0 || un.qunit ? INT_MAX : r.lim;
}

// fp32: 16 rows per wave, one 32-key tile per barrier (the decode kernels' ring).
template <int D, int NW, int NS>
__device__ __forceinline__ void prefill_unit(const PrefillParams& p, PrefillLds<float, D, NS>& sh, int wave, int lane) {
  using T = float;
  using RG = Ring<T, D, NS>;
  using M = Mfma<T>;
  constexpr int DS = D / 32, DPT = RG::BLOCKS / NW;
  static_assert(RG::NS >= 4, "the pipelined loop needs at least four stages");
  const int lr = lane & 15, lg = lane >> 4;
  Unit un;
  if (!find_unit<NW>(p, sh.pre, wave, lane, un)) return;
  // this lane's row: 16*w + lr
  const QueryRow row = find_row<D>(p, un, sh.pre, 16 * wave + lr);

  // queries, rotated at their (virtual) positions
  typename M::Frag qf[1][DS];
  const T* qsrc = static_cast<const T*>(un.qunit ? p.q_seg : p.q_ctx) + row.at;
#pragma unroll
  for (int ds = 0; ds < DS; ++ds) qf[0][ds] = M::load(qsrc + 32 * ds + 8 * lg);
#pragma unroll
  for (int ds = 0; ds < DS / 2; ++ds) {
    f32x8_t x = M::to_f32v(qf[0][ds]), y = M::to_f32v(qf[0][ds + DS / 2]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float cs, sn, xr, yr;
      rope_cos_sin(row.pos, p.inv_freq[32 * ds + 8 * lg + e], cs, sn);
      rope_rotate(x[e], y[e], cs, sn, xr, yr);
      x[e] = xr;
      y[e] = yr;
    }
    qf[0][ds] = M::from_f32(x);
    qf[0][ds + DS / 2] = M::from_f32(y);
  }

  const KeySeq ks(p, un, sh.pre);
  const int64_t kvoff = static_cast<int64_t>(un.g) * p.pool * D;
  const T* kctx = static_cast<const T*>(p.ctx_k) + kvoff;
  const T* vctx = static_cast<const T*>(p.ctx_vt) + kvoff;
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(sh.ring));
  TileOffsets<T, D, NW, NS> toff;
  toff.init(wave, lane);
  auto issue = [&](const KeyCursor& kc, uint32_t stage) {
    if (kc.reg < 2) {
      const int64_t t0 = (kc.reg == 0 ? un.poff : un.coff) + kc.at;
      issue_tile<T, D, NW, NS>(stage, kctx, vctx, t0, t0 + kc.rem, wave, lane, toff);
    } else {
      const int64_t so = (static_cast<int64_t>(un.qa + ks.jlo + kc.reg - 2) * p.Hkv + un.g) * p.seg_cap * D;
      issue_tile<T, D, NW, NS>(stage, static_cast<const T*>(p.seg_k) + so, static_cast<const T*>(p.seg_vt) + so,
                               kc.at, kc.at + kc.rem, wave, lane, toff);
    }
  };

  // every compiler-issued load has been consumed; from here the only vector
  // memory operations in flight are this wave's tile DMAs, which the waits count
  wait_vmcnt<0>();
  KeyCursor ti, tc;
  ti.region(ks, 0);
  tc = ti;
  const int last = ks.n - 1;
#pragma unroll
  for (int s = 0; s < RG::NS - 1; ++s) {
    if (s <= last) {
      issue(ti, lds + s * RG::STAGE);
      ti.next(ks);
    }
  }

  RowState<D> st[1];
  row_init(st[0]);
  const float c = p.c;
  f32x4_t sc[1][2], sn[1][2];
  wait_tiles<DPT, RG::NS - 2>(min(last, RG::NS - 2));
  __syncthreads();
  qk_tile<T, D, NS, 1>(sh.ring, qf, sc, lr, lg);
  int vis = region_limit(un, ks, row, tc.reg);     // last visible key, relative to tile t's region
  for (int t = 0; t <= last; ++t) {
    if (t < last) {
      wait_tiles<DPT, RG::NS - 3>(min(last - t - 1, RG::NS - 3));
      __syncthreads();                            // also: every wave is past iteration t-1
      if (t + RG::NS - 1 <= last) {
        issue(ti, lds + ((t + RG::NS - 1) % RG::NS) * RG::STAGE);
        ti.next(ks);
      }
    }
    // tile t: valid tokens and the row's visible limit (relative to the tile start)
    const int n = min(32, tc.rem);
    const int l = min(vis - tc.at, n - 1);
    const bool need = wave_any(l < 31);
    pipe_step_masked<T, D, NS, 1>(sh.ring + ((t + 1) % RG::NS) * RG::STAGE, sh.ring + (t % RG::NS) * RG::STAGE,
                                  qf, sc, sn, st, n, lr, lg, c, [&](f32x4_t (&s)[2], int) {
                                    if (need) mask_after(s, l, lg);
                                  });
    sc[0][0] = sn[0][0];
    sc[0][1] = sn[0][1];
    if (tc.next(ks)) vis = region_limit(un, ks, row, tc.reg);
  }
  wait_vmcnt<0>();                                // no LDS-DMA may outlive the workgroup

  if (!row.valid) return;
  const float inv = 1.f / st[0].ls[0];
  float* o = (un.qunit ? p.out_seg : p.out_ctx) + row.at + 4 * lg;
#pragma unroll
  for (int db = 0; db < D / 16; ++db) *reinterpret_cast<f32x4_t*>(o + 16 * db) = st[0].o[db] * inv;
}

template <int D, int NW, int NS>
__global__ __launch_bounds__(64 * NW, NW >= 8 ? 2 : 1) void prefill_kernel(PrefillParams p) {
  __shared__ PrefillLds<float, D, NS> sh;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  prefill_unit<D, NW, NS>(p, sh, wave, lane);
}

// ---------------------------------------------------------------------------
// bf16: 32 rows per wave, two wave groups half a step apart (prefill_pingpong.h).
// ---------------------------------------------------------------------------
// Values of a half tile past a unit's last key.
static __device__ __align__(16) uint16_t zero_half[32 * 128];

template <int D>
struct PingPongLds {
  alignas(16) unsigned char ring[PpRing<D>::BYTES];
  int pre[kMaxQuestionsPerPrompt + 1];
  float first[128];          // KS = 2: each row's offset after tile 0
};

// KS = 1: 256 rows; both groups work through the same 64-key tiles, group B
// (waves 4-7) half a step behind.  KS = 2: 128 rows; group A takes the even
// tiles and B the odd ones for the same rows, and their states are combined
// at the end: half the steps per unit, for calls too small to fill the chip
// with 256-row units.
//
// With phases counted between barriers, group A multiplies in even phases
// and B in odd ones.
//   KS = 1: tile t's keys are read in phases 2t (A) and 2t+1 (B), its values
//   in the product phases after.  In its product phase t a wave refills the
//   stages of K(t-1) and V(t-2) with tile t+3: the other group, one phase
//   behind, is past both.  When that phase ends its part of tile t+1 has
//   landed, so that after the next barrier the whole tile has.
//   KS = 2: tile t's keys are read in phase t, its values in phases t+1 (the
//   first fragments) and t+2.  In phase t its group refills the stages of
//   K(t-1) and V(t-3) with K(t+3) and V(t+2); what it issued two phases ago,
//   K(t+1) and V(t), has landed when the phase ends.
template <int D, int KS>
__device__ __forceinline__ void pingpong_unit(const PrefillParams& p, PingPongLds<D>& sh, int wave, int lane) {
  using T = uint16_t;
  using R = PpRing<D>;
  using F = PpFetch<D, 8 / KS>;
  constexpr int NK = R::NK, NV = R::NV, PER = F::PER;
  PpQuery<D> query;
  query.load_theta(p.inv_freq, lane);             // shares the layout loads' round trip
  Unit un;
  if (!find_unit<8>(p, sh.pre, wave, lane, un)) return;
  const int grp = wave >> 2, rw = KS == 1 ? wave : wave & 3;
  // this lane's row, 32*rw + lane % 32
  const QueryRow row = find_row<D>(p, un, sh.pre, 32 * rw + (lane & 31));
  query.load(static_cast<const T*>(un.qunit ? p.q_seg : p.q_ctx) + row.at, lane);
  const KeySeq ks(p, un, sh.pre);
  const int nh = ks.n;                            // 32-key halves
  const int steps = (nh + 2 * KS - 1) / (2 * KS); // steps of a group
  const int nt = steps * KS;                      // 64-key tiles, the last of them perhaps empty
  const int64_t kvoff = static_cast<int64_t>(un.g) * p.pool * D;
  const T* kctx = static_cast<const T*>(p.ctx_k) + kvoff;
  const T* vctx = static_cast<const T*>(p.ctx_vt) + kvoff;
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(sh.ring));
  KeyCursor ti, tc;
  ti.region(ks, 0);
  tc = ti;
  // the halves of a tile to be fetched; halves past the last repeat its keys
  // (masked) and take zeros for values: a weight of 0 times an infinity is NaN
  struct Half {
    const T *k, *v;
    int n;
  };
  Half ht[2], hv[2];                              // the tile located last; KS = 2: the one before it
  int hin = 0;
  auto locate = [&]() {
    if (ti.rem > 64 && ti.at > 0) {               // the common tile lies whole in the region of the last
      ht[0].k = ht[1].k + 32 * D;
      ht[0].v = ht[1].v + 32 * D;
      ht[1].k = ht[0].k + 32 * D;
      ht[1].v = ht[0].v + 32 * D;
      ht[0].n = ht[1].n = 32;
      ti.at += 64;
      ti.rem -= 64;
      hin += 2;
      return;
    }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      if (ti.reg < 2) {
        const int64_t t0 = ((ti.reg == 0 ? un.poff : un.coff) + ti.at) * D;
        ht[hf] = Half{kctx + t0, vctx + t0, min(32, ti.rem)};
      } else {
        const int64_t so = ((static_cast<int64_t>(un.qa + ks.jlo + ti.reg - 2) * p.Hkv + un.g) * p.seg_cap + ti.at) * D;
        ht[hf] = Half{static_cast<const T*>(p.seg_k) + so, static_cast<const T*>(p.seg_vt) + so, min(32, ti.rem)};
      }
      if (hin >= nh) ht[hf].v = zero_half;
      if (++hin < nh) ti.next(ks);
    }
  };
  F dma;
  dma.init(wave, lane);
  // stages of the tiles fetched next
  uint32_t kin = lds, vin = lds + R::VBASE;
  auto ahead = [&](uint32_t at, uint32_t base, int stages, int by) {
    at += by * R::STAGE;
    return at >= base + stages * R::STAGE ? at - stages * R::STAGE : at;
  };
  auto fetch_key = [&](const Half (&h)[2], int d, uint32_t on) {
    const int hf = F::half_of(d, wave);
    dma.key(d, h[hf].k, h[hf].n, kin + hf * R::HALF, on);
  };
  auto fetch_value = [&](const Half (&h)[2], int d, uint32_t on) {
    const int hf = F::half_of(d, wave);
    dma.value(d, h[hf].v, h[hf].n, vin + hf * R::HALF, on);
  };
  if constexpr (KS == 1) {
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
      if (t < nt) locate();
#pragma unroll
      for (int d = 0; d < PER; ++d) {
        fetch_key(ht, d, t < nt ? ~0u : 0u);
        fetch_value(ht, d, t < nt ? ~0u : 0u);
      }
      kin = ahead(kin, lds, NK, 1);
      vin = ahead(vin, lds + R::VBASE, NV, 1);
    }
  } else {
    // K(0), V(0), K(2) by group A, K(1), V(1) by B
#pragma unroll 1
    for (int t = 0; t < 3; ++t) {
      if (t < nt) locate();
      if ((t & 1) == grp && t < nt) {
#pragma unroll
        for (int d = 0; d < PER; ++d) fetch_key(ht, d, ~0u);
        if (t < 2) {
#pragma unroll
          for (int d = 0; d < PER; ++d) fetch_value(ht, d, ~0u);
        }
      }
      kin = ahead(kin, lds, NK, 1);
      vin = ahead(vin, lds + R::VBASE, NV, 1);
    }
  }

  bf16x8_t qf[D / 16];
  query.rotate(qf, p.inv_freq, row.pos, p.c, (p.G & 3) == 0, lane);
  PpState<D> st;
  pp_init(st);
  f32x16_t s[2];
  bf16x8_t pf[4];
  uint32_t kst = 0, vst = 0;                      // stages of K and V of the group's tile
  if constexpr (KS == 1) {
    wait_tiles<2 * PER, 3>(min(nt, 4) - 1);
  } else {
    // tiles this wave fetches in its first product phase: V(grp + 2), K(grp + 3)
    if (grp == 0) {
      hv[0] = ht[0];
      hv[1] = ht[1];
      vin = lds + R::VBASE + 2 * R::STAGE;
    } else {
      if (3 < nt) locate();
      hv[0] = ht[0];
      hv[1] = ht[1];
      kin = ahead(kin, lds, NK, 1);
      kst = vst = R::STAGE;
      if (nh > 1) tc.next(ks);                    // (the last half stays in place)
      if (nh > 2) tc.next(ks);
    }
    if (grp + 3 < nt) locate();
    wait_vmcnt<0>();
  }
  int vis = region_limit(un, ks, row, tc.reg);    // last key of the tile's region the row sees
  // keys of that region every row of the unit sees
  auto all_see = [&]() { return tc.reg >= 2 ? 0 : tc.reg == 1 && !un.qunit ? un.k * p.tb + 1 : INT_MAX; };
  int common = all_see();
  phase_barrier();
  if (grp == 1) phase_barrier();
  if constexpr (KS == 2) {
#pragma unroll
    for (int d = 0; d < PER; ++d) fetch_key(ht, d, grp + 3 < nt ? ~0u : 0u);
#pragma unroll
    for (int d = 0; d < PER; ++d) fetch_value(hv, d, grp + 2 < nt ? ~0u : 0u);
    kin = ahead(kin, lds, NK, 2);
    vin = ahead(vin, lds + R::VBASE, NV, 2);
  }
  pp_first_scores<D>(sh.ring + kst, qf, st, s, lane);
#pragma unroll 1
  for (int i = 0; i < steps; ++i) {
    const int t = KS * i + (KS == 2 ? grp : 0);   // the group's tile
    __builtin_amdgcn_s_setprio(0);
    wait_tiles<2 * PER / KS, 2>(max(min(nt - 2 - t, 2), 0));   // the younger fetches with lanes
    phase_barrier();
    unsigned char* vt = sh.ring + R::VBASE + vst;
    if (tc.rem > 64 * KS && tc.at + 64 <= common) {
      tc.at += 64 * KS;                           // a whole tile that every row sees
      tc.rem -= 64 * KS;
    } else {
#pragma unroll
      for (int hf = 0; hf < 2 * KS; ++hf) {
        if (hf < 2) {
          // tokens the half holds (0: it repeats the last), and those of them the row sees
          const int n = 2 * t + hf < nh ? min(32, tc.rem) : 0;
          const int l = min(vis - tc.at, n - 1);
          if (wave_any(l < 31)) pp_mask(s[hf], l, lane);
          if (n > 0 && n < 32) pp_clear_tail<D>(vt + hf * R::HALF, n, lane);
        }
        if (2 * t + hf + 1 < nh && tc.next(ks)) {
          vis = region_limit(un, ks, row, tc.reg);
          common = all_see();
        }
      }
    }
    if (KS == 2 && i == 0 && grp == 1) {
      // group B starts from the offsets that A took from tile 0 a phase ago:
      // a key's weight is then rounded alike in either group's tiles
      const float m = sh.first[32 * rw + (lane & 31)];
      const float d = m == -INFINITY ? 0.f : m;
      if (m > -INFINITY) st.thr = kRescaleLog2;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        st.negm[e] = -d;
        s[0][e] -= d;
        s[1][e] -= d;
      }
    }
    pp_softmax<D>(s, st, pf);
    if (KS == 2 && i == 0 && grp == 0 && lane < 32)
      sh.first[32 * rw + lane] = st.thr == -INFINITY ? -INFINITY : -st.negm[0];
    kst = ahead(kst, 0, NK, KS);
    vst = ahead(vst, 0, NV, KS);
    uint32_t kon, von;
    if constexpr (KS == 1) {
      kon = von = t + 4 < nt ? ~0u : 0u;
      if (t + 4 < nt) locate();
    } else {
      // next product phase t + 2: V(t + 4) and K(t + 5)
      von = t + 4 < nt ? ~0u : 0u;
      kon = t + 5 < nt ? ~0u : 0u;
      if (t + 4 < nt) locate();
      hv[0] = ht[0];
      hv[1] = ht[1];
      if (t + 5 < nt) locate();
    }
    bf16x8_t v0[kPpAhead];
#pragma unroll
    for (int f = 0; f < kPpAhead; ++f) v0[f] = pp_vfrag<D>(vt, f, lane);
    phase_barrier();
    // (after the last tile the scores are those of a stale stage, not used:
    // a way out of the loop before them would keep two sets of outputs live)
    __builtin_amdgcn_s_setprio(1);
    pp_products<D, 2 * PER>(v0, vt, sh.ring + kst, pf, qf, st, s, lane, [&](int d) {
      if (d < PER) fetch_key(ht, d, kon);
      else if constexpr (KS == 1) fetch_value(ht, d - PER, von);
      else fetch_value(hv, d - PER, von);
    });
    kin = ahead(kin, lds, NK, KS);
    vin = ahead(vin, lds + R::VBASE, NV, KS);
  }
  __builtin_amdgcn_s_setprio(0);
  if (grp == 0) phase_barrier();
  phase_barrier();                                // every wave is done with the ring

  float l = xor32_sum((st.l[0] + st.l[1]) + (st.l[2] + st.l[3]));
  constexpr int DB = D / 32 / KS;                 // 32-dim blocks a wave writes
  const int db0 = KS == 2 ? grp * DB : 0;
  f32x16_t o[DB];
  if constexpr (KS == 1) {
    const float inv = 1.f / l;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = st.o[db] * inv;
  } else {
    // each group finishes half of the dims: it gets the other's offset, sum
    // and values of them.  A row whose keys all went to the other group has
    // no offset (weight 0).
    f32x4_t* xo = reinterpret_cast<f32x4_t*>(sh.ring) + rw * (DB * 4 * 2 * 64) + lane;   // [group][piece][lane]
    float2* xm = reinterpret_cast<float2*>(sh.ring + 4 * DB * 4 * 2 * 1024) + rw * 128 + lane;
    const bool fresh = st.thr == -INFINITY;
    const float m = fresh ? -INFINITY : -st.negm[0];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4_t x;
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = grp == 0 ? st.o[DB + db][4 * i + v] : st.o[db][4 * i + v];
        xo[((1 - grp) * DB * 4 + db * 4 + i) * 64] = x;
      }
    xm[(1 - grp) * 64] = make_float2(m, l);
    __syncthreads();
    const float2 ml = xm[grp * 64];
    const float mn = fmaxf(m, ml.x);
    const float fa = fresh ? 0.f : fast_exp2(m - mn);
    const float fb = ml.x == -INFINITY ? 0.f : fast_exp2(ml.x - mn);
    const float inv = 1.f / (l * fa + ml.y * fb);
    const float ga = fa * inv, gb = fb * inv;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4_t y = xo[(grp * DB * 4 + db * 4 + i) * 64];
#pragma unroll
        for (int v = 0; v < 4; ++v)
          o[db][4 * i + v] = (grp == 0 ? st.o[db][4 * i + v] : st.o[DB + db][4 * i + v]) * ga + y[v] * gb;
      }
    __syncthreads();
  }

  // outputs through LDS (the ring's bytes, a region per 32 rows): whole rows
  // of D * 4 contiguous bytes per store
  constexpr int OROW = D * 4 + 16;                // padded: 16 rows' 16-byte pieces hit distinct banks
  unsigned char* ob = sh.ring + rw * (32 * OROW);
  {
    float* orow = reinterpret_cast<float*>(ob + (lane & 31) * OROW) + 4 * (lane >> 5) + 32 * db0;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4_t*>(orow + 32 * db + 8 * i) =
            f32x4_t{o[db][4 * i], o[db][4 * i + 1], o[db][4 * i + 2], o[db][4 * i + 3]};
  }
  // where the 32 rows go (-1: nowhere), after the output regions
  int64_t* at = reinterpret_cast<int64_t*>(sh.ring + 8 * 32 * OROW) + rw * 32;
  static_assert(8 * 32 * (OROW + 8) <= R::BYTES, "output rows and their places must fit the ring");
  if (lane < 32) at[lane] = row.valid ? row.at : -1;
  if (KS == 2) __syncthreads();                   // the two groups' halves of a row
  float* out = un.qunit ? p.out_seg : p.out_ctx;
  constexpr int LPR = D / 4, RPS = 64 / LPR;      // lanes per row, rows per store
#pragma unroll
  for (int it = 0; it < 32 / RPS / KS; ++it) {
    const int r = (it + (KS == 2 ? grp * (32 / RPS / KS) : 0)) * RPS + lane / LPR;
    const int64_t to = at[r];
    if (to >= 0)
      *reinterpret_cast<f32x4_t*>(out + to + (lane % LPR) * 4) =
          *reinterpret_cast<const f32x4_t*>(ob + r * OROW + (lane % LPR) * 16);
  }
}

template <int D, int KS>
__global__ __launch_bounds__(512, 2) void prefill_pingpong_kernel(PrefillParams p) {
  __shared__ PingPongLds<D> sh;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  pingpong_unit<D, KS>(p, sh, wave, lane);
}

// A unit's waves, and its rows as rb 16-row blocks per wave: bf16 units have
// eight waves and 256 rows (rb = 2; the planner halves them, rb = 1, to 128
// rows whose keys the two groups share), fp32 ones (operands twice as wide)
// one block per wave, and four waves at D = 128 (32 KB stages).
bool prefill_variant(int dtype, int head_dim, int* waves, int* rb) {
  const bool bf = dtype == IPPD_DTYPE_BF16;
  if (head_dim != 64 && head_dim != 128) return false;
  *waves = (!bf && head_dim == 128) ? 4 : 8;
  *rb = bf ? 2 : 1;
  return true;
}

hipError_t launch_prefill(int dtype, int head_dim, int rb, int grid, const PrefillParams& p, hipStream_t s) {
  const bool bf = dtype == IPPD_DTYPE_BF16;
  if (bf && head_dim == 128 && rb == 2) prefill_pingpong_kernel<128, 1><<<grid, 512, 0, s>>>(p);
  else if (bf && head_dim == 128) prefill_pingpong_kernel<128, 2><<<grid, 512, 0, s>>>(p);
  else if (bf && head_dim == 64 && rb == 2) prefill_pingpong_kernel<64, 1><<<grid, 512, 0, s>>>(p);
  else if (bf && head_dim == 64) prefill_pingpong_kernel<64, 2><<<grid, 512, 0, s>>>(p);
  else if (!bf && head_dim == 128) prefill_kernel<128, 4, 4><<<grid, 256, 0, s>>>(p);
  else if (!bf && head_dim == 64) prefill_kernel<64, 8, 8><<<grid, 512, 0, s>>>(p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace ippd
