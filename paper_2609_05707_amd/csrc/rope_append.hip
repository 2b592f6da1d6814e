// Rotary embedding at virtual positions: decode-step append and cache loaders.
//
// Positions follow the virtual-position rule of Sec. 4.1: a context token t
// sits at t (instruction folded into the context), segment slot t of a
// question of prompt b at ctx_len[b] + t, and the token fed at a decode step
// at ctx_len[b] + seg_len[i]; behind an instruction of a two-level batch all
// of them move up by its length.  theta_j = base^(-2j/D) comes from the host in
// fp64; cos/sin use the fp64-reduced angle (rope_cos_sin).
#include "ippd_device.h"
#include "ippd_internal.h"

namespace ippd {

// ---------------------------------------------------------------------------
// Decode-step append: one workgroup per question, one 16-byte vector per
// thread and item.  Item e of question i is
//   e < Hq*QP                 pairs [v*VE, v*VE + VE) of query head e / QP,
//                             rotated into q_rot (QP = D/2 / VE pair vectors),
//   e < (Hq + Hkv)*QP         the same pairs of key head (e - Hq*QP) / QP,
//                             rotated into segment slot s of (i, head),
//   e < (Hq + Hkv)*QP + Hkv*VG  dims [v*VE, v*VE + VE) of value head (e - ..) / VG,
//                             written into slot s of the transposed value cache
// (VE = 16 bytes / element size, VG = D / VE).  Every load is issued before
// the question's state is known; the prompt is found with one ballot over
// the prompts (lane l reads prompt l), so a question costs one round trip of
// loads and then its stores.  The D/2 (cos, sin) pairs of the question's
// position are evaluated once, into LDS; rotations use the same cos/sin and
// rounding as the fused decode step, so both give identical bits.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(1024) void append_kernel(AppendParams p) {
  constexpr int VE = 16 / static_cast<int>(sizeof(T));
  typedef T vec_t __attribute__((ext_vector_type(VE)));
  const int i = blockIdx.x;
  const int D = p.D, half = D / 2;
  const int QP = half / VE, VG = D / VE;
  const int nq = p.Hq * QP, nk = p.Hkv * QP, nitems = nq + nk + p.Hkv * VG;
  const int lane = threadIdx.x & 63;
  // the thread's items (a block covers a question in one pass when it can)
  constexpr int kMaxPass = 2;
  vec_t lo[kMaxPass], hi[kMaxPass];
  // every head of the question turns by the same D/2 angles: thread j < D/2
  // evaluates pair j's once into LDS (its frequency read first, with the
  // other loads, so that it shares their round trip)
  __shared__ float2 rot[kMaxHalfDim];
  const double theta = threadIdx.x < static_cast<unsigned>(half) ? p.inv_freq[threadIdx.x] : 0.0;
  // the question's state, and the first 64 prompts' question ends and
  // context lengths for the prompt lookup below, all loaded before any wait
  const bool act = p.active[i] != 0;
  const int s = p.seg_len[i];
  const int bl0 = lane < p.B ? lane : p.B - 1;
  const int q10 = p.q_start[bl0 + 1], cl0 = p.ctx_len[bl0];
  const T* __restrict__ qn = static_cast<const T*>(p.q_new);
  const T* __restrict__ kn = static_cast<const T*>(p.k_new);
  const T* __restrict__ vn = static_cast<const T*>(p.v_new);
  // one load site per pass (a value item reads its vector twice): loads
  // issued from separate branches into the same registers would each wait
  // for the one before
#pragma unroll
  for (int r = 0; r < kMaxPass; ++r) {
    const int e = threadIdx.x + r * blockDim.x;
    const T* src;
    int hoff;
    if (e < nq + nk) {
      const bool isq = e < nq;
      const int ee = isq ? e : e - nq;
      src = (isq ? qn + (static_cast<int64_t>(i) * p.Hq + ee / QP) * D
                 : kn + (static_cast<int64_t>(i) * p.Hkv + ee / QP) * D) + (ee % QP) * VE;
      hoff = half;
    } else {
      const int ev = e - nq - nk;
      src = vn + (static_cast<int64_t>(i) * p.Hkv + ev / VG) * D + (ev % VG) * VE;
      hoff = 0;
    }
    if (e < nitems) {
      lo[r] = *reinterpret_cast<const vec_t*>(src);
      hi[r] = *reinterpret_cast<const vec_t*>(src + hoff);
    }
  }
  // the question's prompt: the number of prompts whose questions all precede
  // i (windows of 64 prompts; the first was loaded above)
  int n = __popcll(__ballot(lane < p.B && q10 <= i));
  int b = n, len = __shfl(cl0, n < 64 ? n : 63, 64);
  for (int b0 = 64; n == 64 && b0 < p.B; b0 += 64) {
    const int bb = b0 + lane;
    const int bl = bb < p.B ? bb : p.B - 1;
    const int q1 = p.q_start[bl + 1], cl = p.ctx_len[bl];
    n = __popcll(__ballot(bb < p.B && q1 <= i));
    b = b0 + n;
    len = __shfl(cl, n < 64 ? n : 63, 64);
  }
  if (b >= p.B) {                                  // i past the last prompt's questions
    b = p.B - 1;
    len = p.ctx_len[b];
  }
  if (!act) return;
  if (s < 0 || s >= p.seg_cap) {
    if (threadIdx.x == 0) raise_flag(p.err_flag, s >= p.seg_cap ? kFlagSegmentFull : kFlagBadLayout);
    return;
  }
  const int64_t pos = instr_pos_base(p.instr_start, p.instr_len, p.S, b) + len + s;
  if (threadIdx.x < static_cast<unsigned>(half)) {
    float c, sn;
    rope_cos_sin(pos, theta, c, sn);
    rot[threadIdx.x] = make_float2(c, sn);
  }
  __syncthreads();                                 // act and s are the question's: every thread is here
  T* __restrict__ qr = static_cast<T*>(p.q_rot);
  T* __restrict__ sk = static_cast<T*>(p.seg_k);
  T* __restrict__ svt = static_cast<T*>(p.seg_vt);
#pragma unroll
  for (int r = 0; r < kMaxPass; ++r) {
    const int e = threadIdx.x + r * blockDim.x;
    if (e < nq + nk) {
      const bool isq = e < nq;
      const int ee = isq ? e : e - nq;
      const int j0 = (ee % QP) * VE;
      vec_t x, y;
#pragma unroll
      for (int u = 0; u < VE; ++u) {
        const float2 cs = rot[j0 + u];
        float xr, yr;
        rope_rotate(to_f32<T>(lo[r][u]), to_f32<T>(hi[r][u]), cs.x, cs.y, xr, yr);
        x[u] = from_f32<T>(xr);
        y[u] = from_f32<T>(yr);
      }
      T* dst = isq ? qr + (static_cast<int64_t>(i) * p.Hq + ee / QP) * D + j0
                   : sk + ((static_cast<int64_t>(i) * p.Hkv + ee / QP) * p.seg_cap + s) * D + j0;
      *reinterpret_cast<vec_t*>(dst) = x;
      *reinterpret_cast<vec_t*>(dst + half) = y;
    } else if (e < nitems) {
      const int ev = e - nq - nk;
      const int g = ev / VG, d0 = (ev % VG) * VE;
#pragma unroll
      for (int u = 0; u < VE; ++u)
        svt[vt_index(static_cast<int64_t>(i) * p.Hkv + g, p.seg_cap, D, s, d0 + u)] = lo[r][u];
    }
  }
  __syncthreads();   // every thread has read seg_len[i] before it moves
  if (threadIdx.x == 0) p.seg_len[i] = s + 1;
}

// ---------------------------------------------------------------------------
// Cache loaders: one workgroup of four waves per octet of tokens (one 8-token
// value block) of a context, instruction or segment, all kv heads.
//   waves 0, 1  keys: lane (token, 8 rotation pairs) evaluates its 8 angles
//               once and rotates the pairs of every second head with them, 16
//               bytes (fp32: 32) per load and store;
//   waves 2, 3  values: an item is (head, 8 dims) of the 8 tokens, transposed
//               in registers into 8 pieces of 8 tokens, 128 contiguous bytes
//               (fp32: 256).
// What bounds it is the copy itself, 4 bytes moved per byte of key: every
// byte is loaded and stored once in 16-byte pieces, and the angles (~35
// instructions each, fp64) are shared by the heads.  Contexts of
// 30.3k tokens of 8 heads x 128 (248 MB moved), bf16: 133 us with an angle, a
// 2-byte load and a 2-byte store per element, through LDS for the values; 62
// us (4.0 TB/s) so.  With 2.7k segment tokens, both calls: 149 and 85 us.
// ---------------------------------------------------------------------------
template <typename T> struct Oct { typedef T type __attribute__((ext_vector_type(8))); };

template <typename T>
struct OctetArgs {
  const T* k_raw; const T* v_raw;   // [rows][Hkv][D]
  T* k; T* vt;                      // regions of `region` tokens per head: [heads][region][D] and its blocked transpose
  int64_t src_row;                  // row of the octet's first token in k_raw / v_raw
  int64_t head0;                    // first token of head 0's region
  int64_t region;
  int64_t tok;                      // the octet's first token in the region (a multiple of 8)
  int64_t pos;                      // its position
  int n;                            // tokens of the octet: 1 .. 8
  int Hkv;
};

// The lane's 8 frequencies (waves 0, 1: pairs 8 * (lane % (D / 16)) ..).
template <int D>
__device__ __forceinline__ void octet_theta(double (&theta)[8], const double* inv_freq) {
  const double2* src = reinterpret_cast<const double2*>(inv_freq + (threadIdx.x % (D / 16)) * 8);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const double2 x = src[u];
    theta[2 * u] = x.x;
    theta[2 * u + 1] = x.y;
  }
}

template <typename T, int D>
__device__ __forceinline__ void load_octet(const OctetArgs<T>& a, const double (&theta)[8]) {
  typedef typename Oct<T>::type vec_t;
  constexpr int half = D / 2, P = half / 8;         // pieces of 8 pairs per row
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = static_cast<int64_t>(a.Hkv) * D;
  if (wave < 2) {
    constexpr int HPW = 64 / (8 * P);                // heads a wave holds at a time
    const int hs = lane / (8 * P), t = lane / P % 8, j0 = (lane % P) * 8;
    if (t >= a.n) return;
    const T* src = a.k_raw + (a.src_row + t) * row + j0;
    T* dst = a.k + (a.head0 + a.tok + t) * D + j0;
    float cs[8], sn[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) rope_cos_sin(a.pos + t, theta[u], cs[u], sn[u]);
#pragma unroll 4
    for (int g = wave * HPW + hs; g < a.Hkv; g += 2 * HPW) {
      const vec_t lo = *reinterpret_cast<const vec_t*>(src + g * D);
      const vec_t hi = *reinterpret_cast<const vec_t*>(src + g * D + half);
      vec_t x, y;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        float xr, yr;
        rope_rotate(to_f32<T>(lo[u]), to_f32<T>(hi[u]), cs[u], sn[u], xr, yr);
        x[u] = from_f32<T>(xr);
        y[u] = from_f32<T>(yr);
      }
      T* d = dst + g * a.region * D;
      *reinterpret_cast<vec_t*>(d) = x;
      *reinterpret_cast<vec_t*>(d + half) = y;
    }
    return;
  }
  for (int e = (wave - 2) * 64 + lane; e < a.Hkv * (D / 8); e += 128) {
    const int g = e / (D / 8), d0 = (e % (D / 8)) * 8;
    const T* src = a.v_raw + a.src_row * row + g * D + d0;
    T* dst = a.vt + (a.head0 + g * a.region + a.tok) * D + d0 * 8;
    vec_t v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = *reinterpret_cast<const vec_t*>(src + min(t, a.n - 1) * row);
    if (a.n == 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        vec_t w;
#pragma unroll
        for (int t = 0; t < 8; ++t) w[t] = v[t][u];
        *reinterpret_cast<vec_t*>(dst + u * 8) = w;
      }
    } else {                                         // tokens past the end are not the call's to write
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (t < a.n) dst[u * 8 + t] = v[t][u];
    }
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void load_context_kernel(LoadContextParams p, int blocks, int per) {
  const int b = blockIdx.x / blocks;
  const int blk = blockIdx.x - b * blocks;
  const int64_t off = p.ctx_off[b];
  const int len = p.ctx_len[b];
  double theta[8];
  octet_theta<D>(theta, p.inv_freq);
  if (off < 0 || (off & 7) || len < 0 || len > p.max_ctx_len || off + len > p.pool) {
    if (threadIdx.x == 0 && blk == 0) raise_flag(p.err_flag, kFlagBadLayout);
    return;
  }
  const int64_t base = instr_pos_base(p.instr_start, p.instr_len, p.S, b);
  for (int t0 = 8 * per * blk; t0 < min(8 * per * (blk + 1), len); t0 += 8) {
    const OctetArgs<T> a = {static_cast<const T*>(p.k_raw), static_cast<const T*>(p.v_raw), static_cast<T*>(p.ctx_k),
                            static_cast<T*>(p.ctx_vt), off + t0, 0, p.pool, off + t0, base + t0,
                            min(8, len - t0), p.Hkv};
    load_octet<T, D>(a, theta);
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void load_segments_kernel(LoadSegmentsParams p, int blocks, int per) {
  const int i = blockIdx.x / blocks;
  const int blk = blockIdx.x - i * blocks;
  const int lane = threadIdx.x & 63;
  // the question's length, its angles' frequencies and the first 64 prompts'
  // question ends and context lengths, in one round trip (a search of q_start
  // load by load made this small kernel 26 us)
  const int bl0 = lane < p.B ? lane : p.B - 1;
  const int q10 = p.q_start[bl0 + 1], cl0 = p.ctx_len[bl0];
  const int n = p.init_len[i];
  double theta[8];
  octet_theta<D>(theta, p.inv_freq);
  if (n < 0 || n > p.seg_cap) {
    if (threadIdx.x == 0 && blk == 0) raise_flag(p.err_flag, kFlagBadLayout);
    return;
  }
  if (threadIdx.x == 0 && blk == 0) p.seg_len[i] = n;
  if (8 * per * blk >= n) return;
  // the prompt holding question i: the number of prompts whose questions all precede it
  int k = __popcll(__ballot(lane < p.B && q10 <= i));
  int b = k, len = __shfl(cl0, k < 64 ? k : 63, 64);
  for (int b0 = 64; k == 64 && b0 < p.B; b0 += 64) {
    const int bb = b0 + lane, bl = bb < p.B ? bb : p.B - 1;
    const int q1 = p.q_start[bl + 1], cl = p.ctx_len[bl];
    k = __popcll(__ballot(bb < p.B && q1 <= i));
    b = b0 + k;
    len = __shfl(cl, k < 64 ? k : 63, 64);
  }
  if (b >= p.B) {                                  // i past the last prompt's questions
    b = p.B - 1;
    len = p.ctx_len[b];
  }
  const int64_t base = instr_pos_base(p.instr_start, p.instr_len, p.S, b) + len;
  for (int t0 = 8 * per * blk; t0 < min(8 * per * (blk + 1), n); t0 += 8) {
    const OctetArgs<T> a = {static_cast<const T*>(p.k_raw), static_cast<const T*>(p.v_raw), static_cast<T*>(p.seg_k),
                            static_cast<T*>(p.seg_vt), static_cast<int64_t>(i) * p.seg_cap + t0,
                            static_cast<int64_t>(i) * p.Hkv * p.seg_cap, p.seg_cap, t0, base + t0, min(8, n - t0),
                            p.Hkv};
    load_octet<T, D>(a, theta);
  }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
// Octets per workgroup: one, unless the workgroups of all ranges (n ranges
// of `octets`) would exceed 2^22 (a launch holds fewer than 2^32 threads).
static int octets_per_block(int64_t n, int octets) {
  int per = 1;
  while (n * ((octets + per - 1) / per) > (1 << 22) && per < octets) per *= 2;
  return per;
}

hipError_t launch_load_context(int dtype, const LoadContextParams& p, hipStream_t s) {
  const int octets = p.max_ctx_len / 8 + (p.max_ctx_len % 8 != 0);
  if (octets == 0 || p.B == 0) return hipSuccess;
  const int per = octets_per_block(p.B, octets), blocks = (octets + per - 1) / per;
  const unsigned grid = static_cast<unsigned>(p.B) * blocks;
  if (dtype == 0 && p.D == 64) load_context_kernel<float, 64><<<grid, 256, 0, s>>>(p, blocks, per);
  else if (dtype == 0) load_context_kernel<float, 128><<<grid, 256, 0, s>>>(p, blocks, per);
  else if (p.D == 64) load_context_kernel<uint16_t, 64><<<grid, 256, 0, s>>>(p, blocks, per);
  else load_context_kernel<uint16_t, 128><<<grid, 256, 0, s>>>(p, blocks, per);
  return hipGetLastError();
}

hipError_t launch_load_segments(int dtype, const LoadSegmentsParams& p, hipStream_t s) {
  const int octets = p.seg_cap / 8;
  if (p.Nt == 0) return hipSuccess;
  const int per = octets_per_block(p.Nt, octets), blocks = (octets + per - 1) / per;
  const unsigned grid = static_cast<unsigned>(p.Nt) * blocks;
  if (dtype == 0 && p.D == 64) load_segments_kernel<float, 64><<<grid, 256, 0, s>>>(p, blocks, per);
  else if (dtype == 0) load_segments_kernel<float, 128><<<grid, 256, 0, s>>>(p, blocks, per);
  else if (p.D == 64) load_segments_kernel<uint16_t, 64><<<grid, 256, 0, s>>>(p, blocks, per);
  else load_segments_kernel<uint16_t, 128><<<grid, 256, 0, s>>>(p, blocks, per);
  return hipGetLastError();
}

// One workgroup per question, as many threads (whole waves, at most 1024) as
// the question has items, or half of them when that exceeds 1024 (each
// thread then takes two: the kernel covers at most two passes).
hipError_t launch_append(int dtype, const AppendParams& p, hipStream_t s) {
  if (p.Nt == 0) return hipSuccess;
  const int ve = dtype == 0 ? 4 : 8;
  const int items = (p.Hq + p.Hkv) * (p.D / 2 / ve) + p.Hkv * (p.D / ve);
  int threads = (items + 63) / 64 * 64;
  if (threads > 1024) threads = ((items + 1) / 2 + 63) / 64 * 64;
  if (threads > 1024) return hipErrorInvalidValue;
  if (dtype == 0) append_kernel<float><<<p.Nt, threads, 0, s>>>(p);
  else append_kernel<uint16_t><<<p.Nt, threads, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace ippd
