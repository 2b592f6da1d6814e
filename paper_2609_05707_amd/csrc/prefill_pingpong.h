// bf16 attention unit of the prefill and of the decode step's wide context
// units on gfx950: eight waves in two groups of four that take
// turns on the matrix cores.
//
// Rows are columns of the products here: a wave owns 32 query rows and works
// on 64 keys per step with v_mfma_f32_32x32x16_bf16,
//   S^T (32 keys x 32 rows) = K Q^T - m    the running offset m enters as the
//                                          accumulator's start, and Q carries
//                                          the softmax scale and log2(e) from
//                                          its rotation on, so the scores come
//                                          out as exponents of two
//   P^T = exp2(S^T)                        in place, rounded to bf16
//   O^T (32 dims x 32 rows) += V^T P^T
// Key k of a 32-key half tile is row pi(k) of the product, pi exchanging bits
// 2 and 3 of the index: registers 8s .. 8s+7 of a lane are then 8 consecutive
// keys, the B operand of the next product, whose A operand (one 8-token value
// block of the cache) is 16 contiguous bytes.
//
// What bounds it: per 64 keys a wave issues 32 products (1024 matrix-core
// cycles) and the softmax's vector work (max, 32 exp2 at quarter rate,
// packing, row sums).  A SIMD holds two waves; if both do the same thing at
// the same time the two kinds of work add up.  So waves 0-3 and 4-7 (one of
// each group per SIMD) run half a step apart, separated by workgroup
// barriers: while one group multiplies, the other exponentiates.
#pragma once

#include "tile_attend.h"

namespace ippd {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// LDS ring: NK stages of keys and NV of values, a stage holding 64 keys as
// two 32-key halves.  Key rows keep token order; 16-byte chunk c of row r
// sits at chunk c ^ swizzle(r), so the 16 lanes of a read hit distinct banks.
// Values are as cached (8-token column blocks).
template <int D>
struct PpRing {
  static constexpr int ROWB = 2 * D;
  static constexpr int CPR = ROWB / 16;
  static constexpr int KSH = CPR >= 16 ? 0 : 1, KMASK = CPR - 1;
  static constexpr int HALF = 32 * ROWB;
  static constexpr int STAGE = 2 * HALF;
  static constexpr int NK = 4, NV = 5;
  static constexpr int BYTES = (NK + NV) * STAGE;
  static constexpr int VBASE = NK * STAGE;
  static constexpr int HB = HALF / 1024;              // 1 KB DMA blocks per half (keys; values the same)
};

// One 16-byte LDS-DMA as dma16s, issued with every lane (on = ~0) or none (0),
// so that the steps past the last fetch run the same code.  One without lanes
// moves nothing.  The waits allow for the younger fetches with lanes only, so
// they hold whether or not the others are counted as in flight: counting them
// can only make a wait longer.  No memory clobber: it
// fills stages that no LDS read of its phase touches, and its order against
// the barriers is that of any volatile asm.
__device__ __forceinline__ void dma16s_if(const void* sbase, uint32_t voff, uint32_t lds_block, uint32_t on) {
  asm volatile("s_mov_b32 exec_lo, %2\n\ts_mov_b32 exec_hi, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
               "s_mov_b64 exec, -1"
               :: "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(on)),
                  "{m0}"(__builtin_amdgcn_readfirstlane(lds_block)));
}

// A wave's DMAs of one 64-key tile's keys or values, shared by W waves (8: both
// groups fetch each tile together, 4: one group does): number d of
// PER = 2 * HB / W is block q + W * (d % BPH) of half d / BPH.  row and sub
// are the lane's key row and byte in it (vblk and vsub its value block and
// byte in that), so that a DMA costs a clamp and an address.
template <int D, int W>
struct PpFetch {
  using R = PpRing<D>;
  static constexpr int VBLK = 8 * R::ROWB;
  static constexpr int BPH = R::HB > W ? R::HB / W : 1;   // blocks of a half per wave
  static constexpr bool SPLIT = R::HB < W;                // waves 0-3 fetch the first half, 4-7 the second
  static constexpr int PER = SPLIT ? 1 : 2 * BPH;
  static_assert(!SPLIT || R::HB * 2 == W, "a wave fetches whole blocks");
  uint32_t blk;                                       // byte offset of this wave's first block in a half
  int krow, vblk;
  uint32_t ksub, vsub;
  __device__ __forceinline__ void init(int wave, int lane) {
    const int q = wave % (SPLIT ? R::HB : W);
    blk = static_cast<uint32_t>(q) * 1024u;
    krow = q * (64 / R::CPR) + lane / R::CPR;
    ksub = static_cast<uint32_t>(((lane % R::CPR) ^ ((krow >> R::KSH) & R::KMASK)) * 16);
    const int o = q * 1024 + lane * 16;
    vblk = o / VBLK;
    vsub = static_cast<uint32_t>(o % VBLK);
  }
  static __device__ __forceinline__ int half_of(int d, int wave) { return SPLIT ? (wave >= 4 ? 1 : 0) : d / BPH; }
  // keys (values) at src, n > 0 of the half's 32 tokens valid: tokens past them
  // are fetched from the last valid one (values: 8-token block)
  __device__ __forceinline__ void key(int d, const uint16_t* src, int n, uint32_t half, uint32_t on) const {
    const int b = SPLIT ? 0 : W * (d % BPH);
    dma16s_if(src, static_cast<uint32_t>(min(krow + b * (64 / R::CPR), n - 1) * R::ROWB) + ksub, half + blk + b * 1024u, on);
  }
  __device__ __forceinline__ void value(int d, const uint16_t* src, int n, uint32_t half, uint32_t on) const {
    const int b = SPLIT ? 0 : W * (d % BPH);
    dma16s_if(src, static_cast<uint32_t>(min(vblk + b * 1024 / VBLK, (n - 1) >> 3) * VBLK) + vsub,
              half + blk + b * 1024u, on);
  }
};

// Zeroes the values of a half tile past its n < 32 tokens (n = 0: a half that
// only repeats another): in the last block they may hold anything, the blocks
// after it are copies of that block, and a weight of 0 times NaN or infinity
// is NaN.  Each wave that will read them does it (all write the same zeros);
// if the last block is finite, and so are its copies, nothing has to be done.
// (Writing always cost a prefill of 3 questions of 8 tokens 1 of 33 us.)
template <int D>
__device__ __forceinline__ void pp_clear_tail(unsigned char* vhalf, int n, int lane) {
  if (n > 0) {
    bool any = false;
#pragma unroll
    for (int d = 0; d < D; d += 64) {
      const u16x8_t x = *reinterpret_cast<const u16x8_t*>(vhalf + ((n - 1) >> 3) * (16 * D) + (d + lane) * 16);
#pragma unroll
      for (int k = 0; k < 8; ++k) any = any || (x[k] & 0x7F80) == 0x7F80;
    }
    if (!wave_any(any)) return;
  }
#pragma unroll 1
  for (int b = n >> 3; b < 4; ++b) {
#pragma unroll
    for (int d = 0; d < D; d += 64) {
      u16x8_t* e = reinterpret_cast<u16x8_t*>(vhalf + b * (16 * D) + (d + lane) * 16);
      u16x8_t x = {0, 0, 0, 0, 0, 0, 0, 0};
      if (8 * b < n) {
        x = *e;
#pragma unroll
        for (int k = 1; k < 8; ++k) x[k] = 8 * b + k < n ? x[k] : 0;
      }
      *e = x;
    }
  }
}

// Softmax state and fragments of a wave's 32 rows.  Lane (hh, n) = (lane / 32,
// lane % 32) holds row n: of each 32-key half the 16 scores of keys
// 16*(i / 8) + 8*hh + i % 8, and the outputs of dims 32*db + 8*(i / 4) + 4*hh + i % 4.
template <int D>
struct PpState {
  f32x16_t o[D / 32];
  f32x16_t negm;           // minus the row's offset, in every element
  float l[4];              // this lane's part of the row sum, in four chains
  float thr;               // a score above it raises the offset: -inf until the row has one
};

template <int D>
__device__ __forceinline__ void pp_init(PpState<D>& st) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.o[db][i] = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) st.negm[i] = 0.f;
#pragma unroll
  for (int k = 0; k < 4; ++k) st.l[k] = 0.f;
  st.thr = -INFINITY;
}

__device__ __forceinline__ bf16x8_t lds_frag(const unsigned char* p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(p));
}

// Fragment f of a 64-key tile's values (16-key step f / (D / 32), dims
// 32 * (f % (D / 32))) and keys (dims 16 * (f / 2), half f % 2).
template <int D>
__device__ __forceinline__ bf16x8_t pp_vfrag(const unsigned char* vst, int f, int lane) {
  using R = PpRing<D>;
  const int s = f / (D / 32), db = f % (D / 32);
  return lds_frag(vst + (lane >> 5) * (8 * R::ROWB) + (lane & 31) * 16 + (s >> 1) * R::HALF +
                  2 * (s & 1) * (8 * R::ROWB) + db * 512);
}
template <int D>
__device__ __forceinline__ bf16x8_t pp_kfrag(const unsigned char* kst, int f, int lane) {
  using R = PpRing<D>;
  const int n = lane & 31, hh = lane >> 5;
  const int r = (n & 0x13) | ((n & 4) << 1) | ((n & 8) >> 1);      // pi: bits 2 and 3 exchanged
  const int sw = (r >> R::KSH) & R::KMASK;
  return lds_frag(kst + r * R::ROWB + (f & 1) * R::HALF + ((2 * (f >> 1) + hh) ^ sw) * 16);
}

// Product phase: O^T += V^T P^T over the previous tile, then S^T = K Q^T - m
// of this one.  A SIMD runs one wave's products at a time, so nothing else
// hides an LDS read's latency: the first kPpAhead value fragments are read
// at the end of the softmax phase, and the reads stay that far ahead of the
// products (the scheduling groups keep them there; left to itself the
// compiler issues each pair just before its use).  dma(i), i < ND, issues
// the wave's DMAs between the products, which hide them.
constexpr int kPpAhead = 8;

template <int D>
__device__ __forceinline__ void pp_first_scores(const unsigned char* kst, const bf16x8_t (&qf)[D / 16],
                                                const PpState<D>& st, f32x16_t (&s)[2], int lane) {
#pragma unroll
  for (int k = 0; k < D / 8; ++k)
    s[k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pp_kfrag<D>(kst, k, lane), qf[k >> 1],
                                                       k < 2 ? st.negm : s[k & 1], 0, 0, 0);
}

template <int D, int ND, typename Dma>
__device__ __forceinline__ void pp_products(const bf16x8_t (&v0)[kPpAhead], const unsigned char* vst,
                                            const unsigned char* kst, const bf16x8_t (&pf)[4],
                                            const bf16x8_t (&qf)[D / 16], PpState<D>& st, f32x16_t (&s)[2], int lane,
                                            Dma dma) {
  constexpr int N = D / 8, AH = kPpAhead;               // value fragments; key fragments the same
  bf16x8_t f[2 * N];
#pragma unroll
  for (int i = 0; i < 2 * N; ++i) f[i] = i < AH ? v0[i] : i < N ? pp_vfrag<D>(vst, i, lane) : pp_kfrag<D>(kst, i - N, lane);
#pragma unroll
  for (int i = 0; i < 2 * N; ++i) {
    if (i < N) {
      const int db = i % (D / 32);
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], pf[i / (D / 32)], st.o[db], 0, 0, 0);
    } else {
      const int k = i - N;
      s[k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], qf[k >> 1], k < 2 ? st.negm : s[k & 1], 0, 0, 0);
    }
    if (i % (2 * N / ND) == 2) dma(i / (2 * N / ND));
  }
#pragma unroll
  for (int i = AH; i < 2 * N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, AH, 0);
}

// Keys past a row's limit (relative to the half's first key) get -inf.
__device__ __forceinline__ void pp_mask(f32x16_t& s, int lim, int lane) {
  const int k0 = 8 * (lane >> 5);
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = 16 * (i >> 3) + (i & 7) + k0 > lim ? -INFINITY : s[i];
}

// Softmax of one 64-key tile.  The offset is raised only when a score lies
// more than kRescaleLog2 above it (then the sums and outputs are rescaled):
// weights below 2^kRescaleLog2 are harmless in fp32.  A row that has seen no
// key takes its first visible tile's max.  RAW: the queries do not carry the
// softmax scale, so scores and offsets are raw and an exponent is c times
// them (a query that is already rounded to bf16 would be rounded again by
// scaling it).
template <int D, bool RAW = false>
__device__ __forceinline__ void pp_softmax(f32x16_t (&s)[2], PpState<D>& st, bf16x8_t (&pf)[4], float c = 1.f) {
  float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
  for (int i = 1; i < 16; ++i) mx = fmaxf(fmaxf(mx, s[0][i]), s[1][i]);
  if (wave_any(mx > st.thr)) {
    const float m2 = xor32_max(mx);
    const bool fresh = st.thr == -INFINITY;
    const float d = fresh ? (m2 == -INFINITY ? 0.f : m2) : fmaxf(m2, 0.f);
    const float alpha = fresh ? 0.f : fast_exp2(RAW ? -d * c : -d);
    if (m2 > -INFINITY) st.thr = RAW ? kRescaleLog2 / c : kRescaleLog2;
#pragma unroll
    for (int k = 0; k < 4; ++k) st.l[k] *= alpha;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.o[db][i] *= alpha;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      st.negm[i] -= d;
      s[0][i] -= d;
      s[1][i] -= d;
    }
  }
  const bf16x2_t one = {static_cast<__bf16>(1.f), static_cast<__bf16>(1.f)};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f32x8_t p;
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = fast_exp2(RAW ? s[k >> 1][8 * (k & 1) + i] * c : s[k >> 1][8 * (k & 1) + i]);
    pf[k] = __builtin_convertvector(p, bf16x8_t);
    // the row sum adds the rounded weights, the ones the values are multiplied by
#pragma unroll
    for (int i = 0; i < 4; ++i)
      st.l[i] = __builtin_amdgcn_fdot2_f32_bf16(bf16x2_t{pf[k][2 * i], pf[k][2 * i + 1]}, one, st.l[i], false);
  }
}

// Query fragments of the lane's row (dims 16*ds + 8*hh + e): loaded raw, and,
// once the tile DMAs are out, rotated and scaled by c.  quad: lanes of a quad
// hold heads of one token (G a multiple of 4), so lane k of the quad
// evaluates the angles of pairs k and k + 4 and the quad exchanges the rest.
template <int D>
struct PpQuery {
  using M = Mfma<uint16_t>;
  static constexpr int DP = D / 32;               // fragment ds pairs with ds + DP
  bf16x8_t raw[2 * DP];
  double theta[DP][2];
  __device__ __forceinline__ void load_theta(const double* inv_freq, int lane) {
#pragma unroll
    for (int ds = 0; ds < DP; ++ds)
#pragma unroll
      for (int u = 0; u < 2; ++u) theta[ds][u] = inv_freq[16 * ds + 8 * (lane >> 5) + 4 * u + (lane & 3)];
  }
  __device__ __forceinline__ void load(const uint16_t* src, int lane) {
#pragma unroll
    for (int ds = 0; ds < 2 * DP; ++ds) raw[ds] = M::load(src + 16 * ds + 8 * (lane >> 5));
  }
  __device__ __forceinline__ void rotate(bf16x8_t (&qf)[D / 16], const double* inv_freq, int64_t pos, float c,
                                         bool quad, int lane) {
#pragma unroll
    for (int ds = 0; ds < DP; ++ds) {
      float cs[8], sn[8];
      if (quad) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float ca, sa;
          rope_cos_sin(pos, theta[ds][u], ca, sa);
          ca *= c;
          sa *= c;
          cs[4 * u] = quad_bcast<0>(ca); sn[4 * u] = quad_bcast<0>(sa);
          cs[4 * u + 1] = quad_bcast<1>(ca); sn[4 * u + 1] = quad_bcast<1>(sa);
          cs[4 * u + 2] = quad_bcast<2>(ca); sn[4 * u + 2] = quad_bcast<2>(sa);
          cs[4 * u + 3] = quad_bcast<3>(ca); sn[4 * u + 3] = quad_bcast<3>(sa);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          rope_cos_sin(pos, inv_freq[16 * ds + 8 * (lane >> 5) + e], cs[e], sn[e]);
          cs[e] *= c;
          sn[e] *= c;
        }
      }
      f32x8_t x = M::to_f32v(raw[ds]), y = M::to_f32v(raw[ds + DP]);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float xr, yr;
        rope_rotate(x[e], y[e], cs[e], sn[e], xr, yr);
        x[e] = xr;
        y[e] = yr;
      }
      qf[ds] = M::from_f32(x);
      qf[ds + DP] = M::from_f32(y);
    }
  }
};

__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace ippd
