// Prologue and epilogue kernels of the layer entry points: RoPE on the two
// relation projections (Sec. 3.1), Givens head-pair mixing of the information
// state (eq. 4, App. A.2.2-A.2.3), zero padding of the head width to the width
// the fused kernels tile, and the backward of all three.
//
// Each of these is a pass over [B, H, T, D] rows whose cost is linear in T,
// against the T^2 work of the fused kernels, so the rotation, the mixing and the
// padding run once per row here instead of once per key tile inside the fused
// kernels. They are bound by HBM: a thread moves chunks of VEC contiguous
// channels (16 bytes when the caller's layout allows it, in bf16 otherwise 8
// bytes on 4-byte boundaries), TPR threads (a power of two, at most 64) cover
// one row, and rows are contiguous in the padded layout. In the rotating
// kernels a thread holds the chunk of the first half and the one of the second
// half that RoPE turns it with, for q, k and v alike, so that every channel is
// read once and 8 to 12 loads are in flight per thread.
// Measured with rows of 60 channels (4 x 8 x 1999 rows): prologue 16.6 -> 12.3
// us (48 MB, 3.9 TB/s), row copies 7.9 -> 5.7 (16 MB), epilogue 18.0 -> 14.1,
// against 4-byte chunks with each half read by both halves' threads; with rows
// of 80 channels inside tokens of 640 (4 x 8 x 4096): prologue 37 -> 34.2 (138
// MB, 4.0 TB/s; 38.7 without a token's heads together), epilogue 39 -> 36.4.
//
// RoPE rotates channel d with channel d + D/2 by t * base^(-2d/D) (t zero-based),
// with cos and sin from a per-call [T, D/2] table evaluated in fp64.
// Givens mixing writes, for head h of pair p with partner head h':
//   I~_h = cos(theta_p) I_h + sigma_h sin(theta_p) I_h'
// where sigma_h = -1 for the pair's first head and +1 for its second.
#include "kernels.h"

namespace rel {

namespace {

constexpr int kLThreads = 256;
constexpr int kSumParts = 64;  // first-stage partial sums per dtheta segment
constexpr int kOneStage = 1024;  // threads that sum a short segment in one stage
constexpr int64_t kOneStageMax = 65536;

// VEC contiguous elements of type TI at p + i, as floats (i a multiple of VEC).
template <typename TI, int VEC>
struct Chunk;

template <>
struct Chunk<bf16, 8> {
  static __device__ __forceinline__ void load(const void* p, int64_t i, float (&x)[8]) {
    const uintx4 u = *reinterpret_cast<const uintx4*>((const bf16*)p + i);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      x[2 * t] = bf16_lo(u[t]);
      x[2 * t + 1] = bf16_hi(u[t]);
    }
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, const float (&x)[8]) {
    bf16x8 o;
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = (bf16)x[t];
    *reinterpret_cast<bf16x8*>((bf16*)p + i) = o;
  }
};

// 8 bytes on a 4-byte boundary, which the hardware's 8-byte accesses take.
template <>
struct Chunk<bf16, 4> {
  typedef unsigned int uintx2a4 __attribute__((ext_vector_type(2), aligned(4)));
  static __device__ __forceinline__ void load(const void* p, int64_t i, float (&x)[4]) {
    const uintx2a4 u = *reinterpret_cast<const uintx2a4*>((const bf16*)p + i);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      x[2 * t] = bf16_lo(u[t]);
      x[2 * t + 1] = bf16_hi(u[t]);
    }
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, const float (&x)[4]) {
    typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef float floatv4 __attribute__((ext_vector_type(4)));
    const bf16x4 o = __builtin_convertvector(floatv4{x[0], x[1], x[2], x[3]}, bf16x4);
    *reinterpret_cast<uintx2a4*>((bf16*)p + i) = __builtin_bit_cast(uintx2a4, o);
  }
};

template <>
struct Chunk<bf16, 2> {
  static __device__ __forceinline__ void load(const void* p, int64_t i, float (&x)[2]) {
    const unsigned int u = *reinterpret_cast<const unsigned int*>((const bf16*)p + i);
    x[0] = bf16_lo(u);
    x[1] = bf16_hi(u);
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, const float (&x)[2]) {
    typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 o;
    o[0] = (bf16)x[0];
    o[1] = (bf16)x[1];
    *reinterpret_cast<bf16x2*>((bf16*)p + i) = o;
  }
};

template <>
struct Chunk<float, 4> {
  static __device__ __forceinline__ void load(const void* p, int64_t i, float (&x)[4]) {
    const float4 u = *reinterpret_cast<const float4*>((const float*)p + i);
    x[0] = u.x; x[1] = u.y; x[2] = u.z; x[3] = u.w;
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, const float (&x)[4]) {
    *reinterpret_cast<float4*>((float*)p + i) = make_float4(x[0], x[1], x[2], x[3]);
  }
};

template <>
struct Chunk<float, 2> {
  static __device__ __forceinline__ void load(const void* p, int64_t i, float (&x)[2]) {
    const float2 u = *reinterpret_cast<const float2*>((const float*)p + i);
    x[0] = u.x; x[1] = u.y;
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, const float (&x)[2]) {
    *reinterpret_cast<float2*>((float*)p + i) = make_float2(x[0], x[1]);
  }
};

template <typename TI>
struct Chunk<TI, 1> {
  static __device__ __forceinline__ void load(const void* p, int64_t i, float (&x)[1]) {
    x[0] = Elem<TI>::load((const TI*)p + i);
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, const float (&x)[1]) {
    Elem<TI>::store((TI*)p + i, x[0]);
  }
};

// Pair index, partner head and sign sigma of head h in pairing 1 (A: (1,2),
// (3,4), ...) or 2 (B: (2,3), ..., (H,1)); heads are zero-based here.
__device__ __forceinline__ void givens_role(int h, int H, int mode, int& pair, int& partner,
                                            float& sigma) {
  if (mode == 1) {
    pair = h >> 1;
    partner = h ^ 1;
    sigma = (h & 1) ? 1.0f : -1.0f;
  } else if (h & 1) {
    pair = (h - 1) >> 1;
    partner = h + 1 == H ? 0 : h + 1;
    sigma = -1.0f;
  } else {
    const int hh = h == 0 ? H : h;
    pair = (hh >> 1) - 1;
    partner = hh - 1;
    sigma = 1.0f;
  }
}

// The row (b, h, t) a thread works on, and its position among the row's threads.
struct RowPos {
  int64_t row;  // (b H + h) T + t
  int t, h, b, lane;
  bool valid;
};

// The order of the rows over the grid. Where a token's heads lie side by side
// (views of [B, T, H, D]) a workgroup takes all heads of kTokens tokens after
// each other: rows of 160 bytes share their 128-byte lines with the next head's,
// which another workgroup, on another die with its own L2, would fetch again,
// and kTokens rows of a padded head still fill whole lines.
constexpr int kTokens = 4;
__host__ __device__ __forceinline__ bool by_token(const LayerArgs& a) { return a.sh < a.st; }

// n / d, in 32 bits where n fits (n >= 0).
__device__ __forceinline__ int64_t fast_div(int64_t n, int d) {
  return (n >> 32) == 0 ? (int64_t)((unsigned)n / (unsigned)d) : n / d;
}

template <int TPR>
__device__ __forceinline__ RowPos row_pos(const LayerArgs& a) {
  RowPos r;
  r.lane = threadIdx.x % TPR;
  const int64_t at = (int64_t)blockIdx.x * (kLThreads / TPR) + threadIdx.x / TPR;
  if (by_token(a)) {
    const int64_t rest = at / kTokens;
    const int64_t n = fast_div(rest, a.H);  // b, block of tokens
    const int blocks = (a.T + kTokens - 1) / kTokens;
    r.h = (int)(rest - n * a.H);
    const int64_t b = fast_div(n, blocks);
    r.t = (int)(n - b * blocks) * kTokens + (int)(at % kTokens);
    r.valid = b < a.B && r.t < a.T;
    r.b = (int)b;
  } else {
    const int64_t n = fast_div(at, a.T);
    r.t = (int)(at - n * a.T);
    const int64_t b = fast_div(n, a.H);
    r.h = (int)(n - b * a.H);
    r.valid = b < a.B;
    r.b = (int)b;
  }
  if (!r.valid) r.b = r.h = r.t = 0;
  r.row = ((int64_t)r.b * a.H + r.h) * a.T + r.t;
  return r;
}

// A row's channels as two runs [0, split) and [split, D): the halves that RoPE
// turns against each other, or without RoPE the first of whole chunks. Thread l
// takes the chunk at l VEC of both; a last chunk that would pass its run's end
// ends there instead and repeats channels of the chunk before it (the same
// values are stored twice).
template <int VEC>
__device__ __forceinline__ int split_of(const LayerArgs& a) {
  return a.rope ? a.D >> 1 : ((a.D + 1) / 2 + VEC - 1) / VEC * VEC;
}
struct ChunkPos {
  int lo, hi;  // hi: also without a chunk of its own in the second run (a repeated one, D >= VEC)
};
template <int VEC>
__device__ __forceinline__ ChunkPos chunk_pos(const LayerArgs& a, int split, int l) {
  ChunkPos c;
  c.lo = min(l * VEC, split - VEC);
  c.hi = min(split + c.lo, a.D - VEC);
  return c;
}

// Zeros in channels D .. DP - 1 of the padded row at dst.
template <typename TI, int VEC, int TPR>
__device__ __forceinline__ void pad_row(const LayerArgs& a, void* out, int64_t dst, int lane) {
  constexpr int PV = sizeof(TI) * VEC == 16 ? VEC : VEC > 1 ? 2 : 1;  // divides DP - D where VEC may not
  float zero[PV] = {};
  for (int c = a.D + lane * PV; c < a.DP; c += TPR * PV) Chunk<TI, PV>::store(out, dst + c, zero);
}

__global__ __launch_bounds__(256) void rope_table_kernel(float2* tab, int T, int D, double log_base) {
  const int half = D >> 1;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)T * half) return;
  const int t = (int)(idx / half), j = (int)(idx % half);
  const double ang = (double)t * exp(-2.0 * (double)j / (double)D * log_base);
  double s, c;
  sincos(ang, &s, &c);
  tab[idx] = make_float2((float)c, (float)s);
}

template <typename TI, int VEC, int TPR>
__global__ __launch_bounds__(kLThreads) void prologue_kernel(LayerArgs a) {
  const RowPos r = row_pos<TPR>(a);
  if (!r.valid) return;
  const int64_t src = r.b * a.sb + r.h * a.sh + (int64_t)r.t * a.st;
  const int64_t dst = r.row * a.DP;
  const int half = a.D >> 1;
  int pair = 0, partner = r.h;
  float sigma = 0.0f, cth = 1.0f, sth = 0.0f;
  if (a.givens) {
    givens_role(r.h, a.H, a.givens, pair, partner, sigma);
    sincosf(a.theta[pair], &sth, &cth);
  }
  const int64_t srcp = r.b * a.sb + partner * a.sh + (int64_t)r.t * a.st;
  const int split = split_of<VEC>(a);
  for (int l = r.lane; l * VEC < split; l += TPR) {
    const ChunkPos c = chunk_pos<VEC>(a, split, l);
    float q1[VEC], q2[VEC], k1[VEC], k2[VEC], v1[VEC], v2[VEC], p1[VEC], p2[VEC];
    Chunk<TI, VEC>::load(a.q, src + c.lo, q1);
    Chunk<TI, VEC>::load(a.q, src + c.hi, q2);
    Chunk<TI, VEC>::load(a.k, src + c.lo, k1);
    Chunk<TI, VEC>::load(a.k, src + c.hi, k2);
    Chunk<TI, VEC>::load(a.v, src + c.lo, v1);
    Chunk<TI, VEC>::load(a.v, src + c.hi, v2);
    if (a.givens) {
      Chunk<TI, VEC>::load(a.v, srcp + c.lo, p1);
      Chunk<TI, VEC>::load(a.v, srcp + c.hi, p2);
    }
    if (a.rope) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float2 cs = a.rope[(int64_t)r.t * half + c.lo + e];
        const float qa = q1[e], ka = k1[e];
        q1[e] = qa * cs.x - q2[e] * cs.y;
        q2[e] = qa * cs.y + q2[e] * cs.x;
        k1[e] = ka * cs.x - k2[e] * cs.y;
        k2[e] = ka * cs.y + k2[e] * cs.x;
      }
    }
    if (a.givens) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        v1[e] = cth * v1[e] + sigma * sth * p1[e];
        v2[e] = cth * v2[e] + sigma * sth * p2[e];
      }
    }
    Chunk<TI, VEC>::store(a.qr, dst + c.lo, q1);
    Chunk<TI, VEC>::store(a.kr, dst + c.lo, k1);
    Chunk<TI, VEC>::store(a.vt, dst + c.lo, v1);
    Chunk<TI, VEC>::store(a.qr, dst + c.hi, q2);
    Chunk<TI, VEC>::store(a.kr, dst + c.hi, k2);
    Chunk<TI, VEC>::store(a.vt, dst + c.hi, v2);
  }
  pad_row<TI, VEC, TPR>(a, a.qr, dst, r.lane);
  pad_row<TI, VEC, TPR>(a, a.kr, dst, r.lane);
  pad_row<TI, VEC, TPR>(a, a.vt, dst, r.lane);
}

// Copies rows between the caller's layout (true width D) and the contiguous
// padded layout (width DP): to_padded = 1 writes zeros in channels D .. DP-1.
template <typename TI, int VEC, int TPR>
__global__ __launch_bounds__(kLThreads) void repad_kernel(const void* src, void* dst, LayerArgs a,
                                                          int to_padded) {
  const RowPos r = row_pos<TPR>(a);
  if (!r.valid) return;
  const int64_t cl = r.b * a.sb + r.h * a.sh + (int64_t)r.t * a.st;
  const int64_t pd = r.row * a.DP;
  for (int l = r.lane; l * VEC < a.D; l += TPR) {
    const int c0 = min(l * VEC, a.D - VEC);
    float x[VEC];
    Chunk<TI, VEC>::load(src, (to_padded ? cl : pd) + c0, x);
    Chunk<TI, VEC>::store(dst, (to_padded ? pd : cl) + c0, x);
  }
  if (to_padded) pad_row<TI, VEC, TPR>(a, dst, pd, r.lane);
}

// Backward: gradients in the padded layout (gq, gk with respect to the rotated
// projections, gv with respect to I~) to the caller's tensors, and each row's
// term of dL/dtheta for the pair whose first head this row belongs to:
//   dL/dtheta_p += dI~_a . (-s I_a - c I_b) + dI~_b . (c I_a - s I_b).
// Threads past the last row still join the row reduction (they add zero).
template <typename TI, int VEC, int TPR>
__global__ __launch_bounds__(kLThreads) void epilogue_kernel(LayerArgs a) {
  const RowPos r = row_pos<TPR>(a);
  const int64_t cl = r.b * a.sb + r.h * a.sh + (int64_t)r.t * a.st;
  const int64_t pd = r.row * a.DP;
  const int half = a.D >> 1;
  int pair = 0, partner = r.h;
  float sigma = 0.0f, cth = 1.0f, sth = 0.0f;
  if (a.givens) {
    givens_role(r.h, a.H, a.givens, pair, partner, sigma);
    sincosf(a.theta[pair], &sth, &cth);
  }
  const int64_t pdp = (((int64_t)r.b * a.H + partner) * a.T + r.t) * a.DP;  // partner row, padded
  const int64_t clp = r.b * a.sb + partner * a.sh + (int64_t)r.t * a.st;    // partner row, caller
  const bool first = a.givens && sigma < 0.0f;
  float dth = 0.0f;
  const int split = split_of<VEC>(a);
  for (int l = r.lane; r.valid && l * VEC < split; l += TPR) {
    const ChunkPos c = chunk_pos<VEC>(a, split, l);
    float q1[VEC], q2[VEC], k1[VEC], k2[VEC], v1[VEC], v2[VEC];
    Chunk<TI, VEC>::load(a.gq, pd + c.lo, q1);
    Chunk<TI, VEC>::load(a.gq, pd + c.hi, q2);
    Chunk<TI, VEC>::load(a.gk, pd + c.lo, k1);
    Chunk<TI, VEC>::load(a.gk, pd + c.hi, k2);
    Chunk<TI, VEC>::load(a.gv, pd + c.lo, v1);
    Chunk<TI, VEC>::load(a.gv, pd + c.hi, v2);
    if (a.givens) {
      float p1[VEC], p2[VEC];
      Chunk<TI, VEC>::load(a.gv, pdp + c.lo, p1);
      Chunk<TI, VEC>::load(a.gv, pdp + c.hi, p2);
      if (first) {  // h = a, partner = b
        float a1[VEC], a2[VEC], b1[VEC], b2[VEC];
        Chunk<TI, VEC>::load(a.v, cl + c.lo, a1);
        Chunk<TI, VEC>::load(a.v, cl + c.hi, a2);
        Chunk<TI, VEC>::load(a.v, clp + c.lo, b1);
        Chunk<TI, VEC>::load(a.v, clp + c.hi, b2);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          // channels that a shortened chunk repeats are the chunk before's
          if (c.lo + e >= l * VEC)
            dth += v1[e] * (-sth * a1[e] - cth * b1[e]) + p1[e] * (cth * a1[e] - sth * b1[e]);
          if (c.hi + e >= split + l * VEC)
            dth += v2[e] * (-sth * a2[e] - cth * b2[e]) + p2[e] * (cth * a2[e] - sth * b2[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        v1[e] = cth * v1[e] - sigma * sth * p1[e];
        v2[e] = cth * v2[e] - sigma * sth * p2[e];
      }
    }
    if (a.rope) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float2 cs = a.rope[(int64_t)r.t * half + c.lo + e];
        const float qa = q1[e], ka = k1[e];
        q1[e] = qa * cs.x + q2[e] * cs.y;
        q2[e] = -qa * cs.y + q2[e] * cs.x;
        k1[e] = ka * cs.x + k2[e] * cs.y;
        k2[e] = -ka * cs.y + k2[e] * cs.x;
      }
    }
    Chunk<TI, VEC>::store(a.dq, cl + c.lo, q1);
    Chunk<TI, VEC>::store(a.dk, cl + c.lo, k1);
    Chunk<TI, VEC>::store(a.dv, cl + c.lo, v1);
    Chunk<TI, VEC>::store(a.dq, cl + c.hi, q2);
    Chunk<TI, VEC>::store(a.dk, cl + c.hi, k2);
    Chunk<TI, VEC>::store(a.dv, cl + c.hi, v2);
  }
  if (a.givens) {
    for (int o = TPR / 2; o >= 1; o >>= 1) dth += __shfl_xor(dth, o, 64);
    if (r.valid && first && r.lane == 0) a.dth_rows[((int64_t)pair * a.B + r.b) * a.T + r.t] = dth;
  }
}

// Fixed-order sums of nseg segments of seg_len floats: stage 1 (grid
// nseg x kSumParts) sums contiguous parts of each segment, stage 2 (grid nseg)
// sums a segment's kSumParts partials.
__device__ __forceinline__ float block_sum(float acc) {
  __shared__ float sh[256];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int hh = 128; hh >= 1; hh >>= 1) {
    if ((int)threadIdx.x < hh) sh[threadIdx.x] += sh[threadIdx.x + hh];
    __syncthreads();
  }
  return sh[0];
}

__global__ __launch_bounds__(256) void segment_parts_kernel(const float* x, int64_t seg_len, float* part) {
  const int seg = blockIdx.y, pi = blockIdx.x;
  const int64_t chunk = (seg_len + kSumParts - 1) / kSumParts;
  const int64_t i0 = pi * chunk, i1 = i0 + chunk < seg_len ? i0 + chunk : seg_len;
  const float* xs = x + (int64_t)seg * seg_len;
  float acc = 0.0f;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) acc += xs[i];
  acc = block_sum(acc);
  if (threadIdx.x == 0) part[seg * kSumParts + pi] = acc;
}

// A whole segment per workgroup, in a fixed order.
__global__ __launch_bounds__(kOneStage) void segment_sum_kernel(const float* x, int64_t seg_len, float* out) {
  __shared__ float sh[kOneStage / 64];
  const float* xs = x + (int64_t)blockIdx.x * seg_len;
  float acc[8] = {};
  int64_t i = threadIdx.x;
  for (; i + 7 * kOneStage < seg_len; i += 8 * kOneStage) {
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u] += xs[i + u * kOneStage];
  }
  for (; i < seg_len; i += kOneStage) acc[0] += xs[i];
  float s = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
    for (int w = 0; w < kOneStage / 64; ++w) t += sh[w];
    out[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(256) void segment_total_kernel(const float* part, float* out) {
  const float v = (int)threadIdx.x < kSumParts ? part[blockIdx.x * kSumParts + threadIdx.x] : 0.0f;
  const float s = block_sum(v);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

dim3 row_grid(const LayerArgs& a, int tpr) {
  const int64_t rows = (int64_t)a.B * a.H * (by_token(a) ? (a.T + kTokens - 1) / kTokens * kTokens : a.T);
  const int64_t per = kLThreads / tpr;
  return dim3((unsigned)((rows + per - 1) / per));
}

// Instantiates kernel K for (TI, VEC) with TPR = the power of two at or above
// the row's chunks of `run` channels, 4 to 64 (some threads of a row may stay
// idle, which keeps a row's loads in one pass and the row groups aligned within
// a wave).
#define REL_LAYER_DISPATCH(K, TI, VEC, ...)                                                           \
  do {                                                                                                \
    int tpr_ = 4;                                                                                     \
    while (tpr_ < 64 && tpr_ * (VEC) < run) tpr_ *= 2;                                                \
    if (tpr_ == 64)                                                                                   \
      hipLaunchKernelGGL((K<TI, VEC, 64>), row_grid(a, 64), dim3(kLThreads), 0, stream, __VA_ARGS__); \
    else if (tpr_ == 32)                                                                              \
      hipLaunchKernelGGL((K<TI, VEC, 32>), row_grid(a, 32), dim3(kLThreads), 0, stream, __VA_ARGS__); \
    else if (tpr_ == 16)                                                                              \
      hipLaunchKernelGGL((K<TI, VEC, 16>), row_grid(a, 16), dim3(kLThreads), 0, stream, __VA_ARGS__); \
    else if (tpr_ == 8)                                                                               \
      hipLaunchKernelGGL((K<TI, VEC, 8>), row_grid(a, 8), dim3(kLThreads), 0, stream, __VA_ARGS__);   \
    else                                                                                              \
      hipLaunchKernelGGL((K<TI, VEC, 4>), row_grid(a, 4), dim3(kLThreads), 0, stream, __VA_ARGS__);   \
  } while (0)

#define REL_LAYER_BY_TYPE(K, ...)                                         \
  do {                                                                    \
    if (dtype == 1) {                                                     \
      if (vec == 8) REL_LAYER_DISPATCH(K, bf16, 8, __VA_ARGS__);          \
      else if (vec == 4) REL_LAYER_DISPATCH(K, bf16, 4, __VA_ARGS__);     \
      else REL_LAYER_DISPATCH(K, bf16, 1, __VA_ARGS__);                   \
    } else {                                                              \
      if (vec == 4) REL_LAYER_DISPATCH(K, float, 4, __VA_ARGS__);         \
      else if (vec == 2) REL_LAYER_DISPATCH(K, float, 2, __VA_ARGS__);    \
      else REL_LAYER_DISPATCH(K, float, 1, __VA_ARGS__);                  \
    }                                                                     \
  } while (0)

bool vec_ok(int dtype, int vec) {
  return dtype == 1 ? (vec == 8 || vec == 4 || vec == 1) : (vec == 4 || vec == 2 || vec == 1);
}

}  // namespace

int layer_sum_parts() { return kSumParts; }

hipError_t launch_rope_table(float2* tab, int T, int D, double base, hipStream_t stream) {
  const int64_t n = (int64_t)T * (D / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, tab, T, D,
                     log(base));
  return hipGetLastError();
}

hipError_t launch_layer_prologue(const LayerArgs& a, int dtype, int vec, hipStream_t stream) {
  if (!vec_ok(dtype, vec)) return hipErrorInvalidValue;
  const int run = (a.D + 1) / 2;
  REL_LAYER_BY_TYPE(prologue_kernel, a);
  return hipGetLastError();
}

hipError_t launch_layer_repad(const void* src, void* dst, const LayerArgs& a, bool to_padded, int dtype,
                              int vec, hipStream_t stream) {
  if (!vec_ok(dtype, vec)) return hipErrorInvalidValue;
  const int tp = to_padded ? 1 : 0, run = a.D;
  REL_LAYER_BY_TYPE(repad_kernel, src, dst, a, tp);
  return hipGetLastError();
}

hipError_t launch_layer_epilogue(const LayerArgs& a, int dtype, int vec, hipStream_t stream) {
  if (!vec_ok(dtype, vec)) return hipErrorInvalidValue;
  const int run = (a.D + 1) / 2;
  REL_LAYER_BY_TYPE(epilogue_kernel, a);
  return hipGetLastError();
}

hipError_t launch_segment_sum(const float* x, int nseg, int64_t seg_len, float* part, float* out,
                              hipStream_t stream) {
  if (seg_len <= kOneStageMax) {  // 64 values per thread at most: 4.7 us, in two stages 4.8 + 4.6
    hipLaunchKernelGGL(segment_sum_kernel, dim3((unsigned)nseg), dim3(kOneStage), 0, stream, x, seg_len, out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(segment_parts_kernel, dim3(kSumParts, (unsigned)nseg), dim3(256), 0, stream, x, seg_len,
                     part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(segment_total_kernel, dim3((unsigned)nseg), dim3(256), 0, stream, (const float*)part, out);
  return hipGetLastError();
}

}  // namespace rel
