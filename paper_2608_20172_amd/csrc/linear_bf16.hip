// Linear Relation (Sec. 5.2, App. A.4) for bf16 inputs. The recurrence, the
// chunk formulas and the names are those at the top of linear.hip, which holds
// the fp32 kernels; b is kept here in log2 units.
//
// One workgroup of four waves per chunk of 64 tokens; wave w owns the 16 rows
// 16 w .. 16 w + 15. Lane (i, g) = (lane % 16, lane / 16) holds row i of its
// wave's block and, for every s < D / 32, the 8 channels 32 s + 8 g .. + 7: one
// 16-byte piece of a bf16 row. Every product runs on 16 x 16 matrix-core tiles
// with the transposed result (channels on tile rows, tokens on lanes): register
// v of tile m = 2 s + h is then channel 32 s + 8 g + 4 h + v of the lane's own
// row, the place where the row's own q, k and b are, so that results are scaled,
// summed and taken through S and the normalisation without leaving the lane,
// and a 16 x 16 block of scores is the operand of the next product as it stands
// in its registers. Only what other waves read goes through LDS, as bf16 rows
// of 16-byte pieces: row operands by 16-byte reads, operands that contract over
// rows by transpose reads.
//
// Decay. e^{b_t - b_j} over a 16 x 16 block is factored per channel: keys carry
// k e^{cK - b}, queries q e^{b - cQ} with a reference value per block. Inside a
// block both references are the middle of the block's range of b, so the
// factors lie within 2^+-90 when that range is at most 180 (kRange; kSteep where
// some S of the block is below kSmallS: an operand's lowest part, 2^-16 of it,
// then stays in the bf16 range either way); products of
// different blocks are accumulated in the order of the blocks and rescaled by
// e^{difference of the references} <= 1 on the way. A sum may be as large as
// 2^90 against its reference, so these factors are applied as the square of
// their root where ranges over kSteep occur: what underflows is then below 2^-126
// itself, not a factor that the sum's size makes up for. (Without such ranges
// the factors alone lose pairs below 2^-94 only.)
// A channel with a larger range takes one-sided references (factors <= 1)
// towards the other blocks, and the block's own pairs take it term by term, with
// the exact exponent, beside the matrix product over the other channels. Chunks
// without a range over kSteep, most of them where the gate retains, take a path
// that knows no such channels.
//
// Precision. Products that reach the decay gradient (dq, dk, C0, G) keep fp32
// accuracy: an fp32 operand is split as hi + mid + lo, three bf16 numbers that
// carry its 24 significant bits; against a bf16 input that is three exact
// products, against another split operand the six products above 2^-24. The
// scores, A V, Qe C0 and Kd G take operands rounded to bf16 once, except the
// scores of a block's own pairs in a chunk with a range over kSteep: those keep
// fp32 accuracy, by six products or term by term.
#include "kernels.h"
#include "lanes.h"

#include <type_traits>

namespace rel {

namespace {

constexpr int kL = 64;       // tokens per chunk
constexpr int kNT = 256;     // threads per workgroup
constexpr float kSteep = 64.0f;   // log2 units of decay over a block past which a chunk takes its kernel's path for steep channels
constexpr float kRange = 180.0f;  // log2 units over a block past which that path takes a channel term by term
constexpr float kSmallS = 0x1p-10f;  // S below which a block's q and k are small: kSteep is the limit there too

typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pk2(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
}
__device__ __forceinline__ uintx4 pack8(const float (&x)[8]) {
  return uintx4{pk2(x[0], x[1]), pk2(x[2], x[3]), pk2(x[4], x[5]), pk2(x[6], x[7])};
}
__device__ __forceinline__ void unpack8(const uintx4& u, float (&x)[8]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    x[2 * t] = bf16_lo(u[t]);
    x[2 * t + 1] = bf16_hi(u[t]);
  }
}
// x = hi + mid + lo in bf16 (24 significant bits)
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  h = pk2(a, b);
  const float a1 = a - bf16_lo(h), b1 = b - bf16_hi(h);
  m = pk2(a1, b1);
  l = pk2(a1 - bf16_lo(m), b1 - bf16_hi(m));
}
__device__ __forceinline__ void split8(const float (&x)[8], uintx4& h, uintx4& m, uintx4& l) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    unsigned hh, mm, ll;
    split_pair(x[2 * t], x[2 * t + 1], hh, mm, ll);
    h[t] = hh;
    m[t] = mm;
    l[t] = ll;
  }
}

// 16x16x32: A lane (i, g) holds A[i][8 g ..], B lane (i, g) B[8 g ..][i], register v of lane (i, g) C[4 g + v][i].
__device__ __forceinline__ floatx4 mm32(const uintx4& a, const uintx4& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}
// 16x16x16: A lane (i, g) holds A[i][4 g ..], B lane (i, g) B[4 g ..][i]; same C.
__device__ __forceinline__ floatx4 mm16(const uintx2& a, const uintx2& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(shortx4, a), __builtin_bit_cast(shortx4, b), c, 0,
                                                   0, 0);
}

// The same with fp32 operands, each as three bf16 parts: the six products above 2^-24.
__device__ __forceinline__ floatx4 mm32_split(const float (&a)[8], const float (&b)[8], floatx4 c) {
  uintx4 ah, am, al, bh, bm, bl;
  split8(a, ah, am, al);
  split8(b, bh, bm, bl);
  c = mm32(al, bh, c);
  c = mm32(ah, bl, c);
  c = mm32(am, bm, c);
  c = mm32(am, bh, c);
  c = mm32(ah, bm, c);
  return mm32(ah, bh, c);
}

// Byte offset of 16-byte piece ch of row `row` in a row-major bf16 array of RB
// bytes per row. Pieces are XOR-swizzled by row so that 16-byte reads of one
// piece over 8 consecutive rows, or over the rows {0-3, 8-11} + 4 h of a tile's
// channels, fill distinct banks.
template <int RB>
__device__ __forceinline__ int coff(int row, int ch) {
  const int f = RB == 64 ? (row >> 1) & 3 : ((row & 1) << 2) | (row & 2) | (((row >> 2) ^ (row >> 3)) & 1);
  return row * RB + ((ch ^ f) << 4);
}

struct LaneIx {
  int i, g;    // row in the block, group
  int e, cg;   // transpose reads: row and channel group this lane supplies
  int w;       // wave
  __device__ LaneIx() {
    const int lane = threadIdx.x & 63;
    i = lane & 15;
    g = lane >> 4;
    e = i >> 2;
    cg = i & 3;
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  }
};

// Transposed operand of tile m (its 16 channels) over 4 rows per lane group, `row` including this lane's e.
template <int RB>
__device__ __forceinline__ uintx2 tr_op(const unsigned char* arr, int row, int m, const LaneIx& L) {
  return lds_read_tr16(arr + coff<RB>(row, 4 * (m >> 1) + L.cg) + 8 * (m & 1));
}
template <int RB>
__device__ __forceinline__ uintx4 row_op(const unsigned char* arr, int row, int ch) {
  return *reinterpret_cast<const uintx4*>(arr + coff<RB>(row, ch));
}
template <int RB>
__device__ __forceinline__ void put_row(unsigned char* arr, int row, int ch, const uintx4& x) {
  *reinterpret_cast<uintx4*>(arr + coff<RB>(row, ch)) = x;
}

// Row shifts read zero past the row's ends (bound_ctrl), so that the move folds into the add.
template <int CTRL>
__device__ __forceinline__ float dpp_shift(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// Lane N of a row of 16 lanes, to all of them.
template <int N>
__device__ __forceinline__ float bcast16(float x) {
  return dpp_shift<0x150 + N>(x);
}
__device__ __forceinline__ float scan16(float x) {  // inclusive running sum over the 16 lanes
  x += dpp_shift<0x111>(x);
  x += dpp_shift<0x112>(x);
  x += dpp_shift<0x114>(x);
  x += dpp_shift<0x118>(x);
  return x;
}
__device__ __forceinline__ float rscan16(float x) {  // inclusive sum over this lane and the later ones
  x += dpp_shift<0x101>(x);
  x += dpp_shift<0x102>(x);
  x += dpp_shift<0x104>(x);
  x += dpp_shift<0x108>(x);
  return x;
}
__device__ __forceinline__ float sum_groups(float x) {  // over the four lane groups of a row
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

__device__ __forceinline__ void ld8f(const float* p, float (&x)[8]) {
  const floatx4 a = *reinterpret_cast<const floatx4*>(p), b = *reinterpret_cast<const floatx4*>(p + 4);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    x[t] = a[t];
    x[4 + t] = b[t];
  }
}
__device__ __forceinline__ void st8f(float* p, const float (&x)[8]) {
  *reinterpret_cast<floatx4*>(p) = floatx4{x[0], x[1], x[2], x[3]};
  *reinterpret_cast<floatx4*>(p + 4) = floatx4{x[4], x[5], x[6], x[7]};
}
// 8 consecutive values, on a 16-byte boundary with VEC
template <bool VEC>
__device__ __forceinline__ uintx4 ld_row(const bf16* p) {
  if (VEC) return *reinterpret_cast<const uintx4*>(p);
  const unsigned short* h = reinterpret_cast<const unsigned short*>(p);
  uintx4 u;
#pragma unroll
  for (int t = 0; t < 4; ++t) u[t] = (unsigned)h[2 * t] | ((unsigned)h[2 * t + 1] << 16);
  return u;
}
template <bool VEC>
__device__ __forceinline__ void st_row(bf16* p, const uintx4& u) {
  if (VEC) {
    *reinterpret_cast<uintx4*>(p) = u;
    return;
  }
  unsigned short* h = reinterpret_cast<unsigned short*>(p);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    h[2 * t] = (unsigned short)(u[t] & 0xffffu);
    h[2 * t + 1] = (unsigned short)(u[t] >> 16);
  }
}
template <bool VEC>
__device__ __forceinline__ void ld_f32(const float* p, float (&x)[8]) {
  if (VEC) {
    ld8f(p, x);
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = p[t];
  }
}

__device__ __forceinline__ int64_t head_off(const LinearArgs& a, int n) {
  return (int64_t)(n / a.H) * a.sb + (int64_t)(n % a.H) * a.sh;
}

// The lane's row as it comes from memory: NO pieces of the decay, all of the rest.
template <int D, bool DY, int NO = D / 32>
struct Raw {
  static constexpr int NS = D / 32;
  uintx4 p1[NS], p2[NS], v[NS], dy[DY ? NS : 1];
  float r[NO][8];
};

// Row t of head n (rows past the sequence read its last row; use_raw then
// counts them as zero). The rows of one head span less than 2 GiB (and those
// of the decay less than 4), so a lane's offset from the head is 32 bits.
template <int D, bool DY, bool VEC, int NO>
__device__ __forceinline__ void load_raw(const LinearArgs& a, int n, int t, int half, const LaneIx& L,
                                         Raw<D, DY, NO>& x) {
  const unsigned row = (unsigned)min(t, a.T - 1);
  const int64_t ho = head_off(a, n);
  const unsigned off = row * (unsigned)a.st + 8u * L.g;
  const bf16 *P1 = (const bf16*)a.p1 + ho, *P2 = (const bf16*)a.p2 + ho, *V = (const bf16*)a.v + ho,
             *DYp = DY ? (const bf16*)a.dy + ho : nullptr;
  const float* G = a.g + (int64_t)n * a.T * D + (NO < D / 32 ? 32 * NO * half : 0);
  const unsigned og = row * D + 8u * L.g;
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    x.p1[s] = ld_row<VEC>(P1 + (off + 32u * s));
    x.p2[s] = ld_row<VEC>(P2 + (off + 32u * s));
    x.v[s] = ld_row<VEC>(V + (off + 32u * s));
    if (DY) x.dy[s] = ld_row<VEC>(DYp + (off + 32u * s));
  }
#pragma unroll
  for (int s = 0; s < NO; ++s) ld_f32<VEC>(G + (og + 32u * s), x.r[s]);
}

// Channels of a row of the RoPE table: the turned ones, in whole pieces.
__host__ __device__ __forceinline__ int rope_width(int rope_half) { return (2 * rope_half + 7) & ~7; }

// (cos, +-sin) of the RoPE angle of position t at the 8 channels from c0: the
// table holds (cos, sin) per channel of the angle at every chunk start and at
// every offset inside a chunk (1, 0 at channels that are not turned), and the
// angle at t is their sum. The sign is that of the partner's term.
__device__ __forceinline__ void rope_cs(const LinearArgs& a, int t, int c0, bool transpose, float (&cs)[8],
                                        float (&sn)[8]) {
  const int W = rope_width(a.rope_half);
  const bool on = c0 < W;
  const int c = on ? c0 : 0;
  const floatx4* pa = reinterpret_cast<const floatx4*>(a.rope + ((unsigned)(t / kL) * W + c));
  const floatx4* pb = reinterpret_cast<const floatx4*>(a.rope + ((unsigned)(a.nchunks + t % kL) * W + c));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const floatx4 x = pa[i], y = pb[i];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int u = 2 * i + v;
      const float s = x[2 * v + 1] * y[2 * v] + x[2 * v] * y[2 * v + 1];
      cs[u] = on ? x[2 * v] * y[2 * v] - x[2 * v + 1] * y[2 * v + 1] : 1.0f;
      sn[u] = !on ? 0.0f : (c0 + u < a.rope_half) != transpose ? -s : s;
    }
  }
}

// Rotation of the lane's whole row in registers, for D >= 64 turned over its
// full width: a channel's partner is the same element of another piece.
template <int NS, bool WX = true>
__device__ __forceinline__ void rope_own(const LinearArgs& a, int t, const LaneIx& L, float (&x)[NS][8], float (&y)[NS][8],
                                         bool transpose) {
  constexpr int HS = NS / 2;
#pragma unroll
  for (int s = 0; s < HS; ++s) {
    float cs[8], sn[8];
    rope_cs(a, t, 32 * s + 8 * L.g, transpose, cs, sn);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (WX) {
        const float x0 = x[s][u], x1 = x[s + HS][u];
        x[s][u] = __builtin_fmaf(x1, sn[u], x0 * cs[u]);
        x[s + HS][u] = __builtin_fmaf(x0, -sn[u], x1 * cs[u]);
      }
      const float y0 = y[s][u], y1 = y[s + HS][u];
      y[s][u] = __builtin_fmaf(y1, sn[u], y0 * cs[u]);
      y[s + HS][u] = __builtin_fmaf(y0, -sn[u], y1 * cs[u]);
    }
  }
}

__device__ __forceinline__ int rope_partner(int c, int h) { return c < h ? c + h : c < 2 * h ? c - h : c; }

// The lane's 8 channels from c0 to their partners' places in its row of a bf16
// array in LDS (the reads are then whole pieces whatever rope_half is).
template <int RB>
__device__ __forceinline__ void put_partner(unsigned char* arr, int row, int c0, int h, const uintx4& x) {
  if (h % 8 == 0) {
    put_row<RB>(arr, row, rope_partner(c0, h) >> 3, x);
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int pc = rope_partner(c0 + u, h);
      *reinterpret_cast<unsigned short*>(arr + coff<RB>(row, pc >> 3) + 2 * (pc & 7)) =
          (unsigned short)(x[u >> 1] >> (16 * (u & 1)));
    }
  }
}

// q = S ^p1, k = S ^p2 (rotated), g log2(e) of NO pieces of the lane's row; S and the inverse norms.
template <int NO>
struct Own {
  float q[NO][8], k[NO][8], b[NO][8];
  float S, in1, in2;
};

// The gate of eq. 15 at the lane's elements: g = -exp(A_log) softplus(r +
// dt_bias) (softplus as max(x, 0) + ln(1 + e^-|x|): no overflow, and the
// logarithm's argument lies in (1, 2], where the hardware log2 is accurate) and
// dg/dr = -exp(A_log) sigmoid(r + dt_bias).
template <int NO>
struct Gate {
  float g[NO][8], d[NO][8];
};

// From the row as loaded; the pieces are those of channel half `half` when NO
// is half of them. WQ: q is wanted; GATE: the gate's values are kept. X1, X2:
// two bf16 [64][D] arrays in LDS whose row of this lane is free (the wave's own
// rows only are written and read, for RoPE partners on other lanes).
template <int D, int NO, bool DY, bool VEC, bool WQ, bool GATE = false>
__device__ __forceinline__ void use_raw(const LinearArgs& a, int n, int t, bool ok, int half, const LaneIx& L,
                                        unsigned char* X1, unsigned char* X2, Raw<D, DY, NO>& raw, Own<NO>& o,
                                        Gate<NO>* gate = nullptr) {
  constexpr int NS = D / 32;
  // formed here: in a walk over chunks the gate's parameters and the RoPE
  // table's offsets are loop invariants that would be held in registers
  int here = 0;
  asm volatile("" : "+v"(here));
  const bool whole = (__builtin_amdgcn_readfirstlane(t) | (kL - 1)) < a.T;  // every row of the chunk exists
  if (!whole && !ok) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      raw.p1[s] = raw.p2[s] = raw.v[s] = uintx4{0, 0, 0, 0};
      if (DY) raw.dy[s] = uintx4{0, 0, 0, 0};
    }
  }
  float s11 = 0.0f, s22 = 0.0f, s12 = 0.0f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    float x[8], y[8];
    unpack8(raw.p1[s], x);
    unpack8(raw.p2[s], y);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      s11 = __builtin_fmaf(x[u], x[u], s11);
      s22 = __builtin_fmaf(y[u], y[u], s22);
      s12 = __builtin_fmaf(x[u], y[u], s12);
    }
  }
  s11 = sum_groups(s11);
  s22 = sum_groups(s22);
  s12 = sum_groups(s12);
  o.S = 1.0f / (1.0f + expf(-s12 * a.scale * a.inv_tau));
  o.in1 = s11 > 0.0f ? rsqrtf(s11) : 0.0f;
  o.in2 = s22 > 0.0f ? rsqrtf(s22) : 0.0f;
#pragma unroll
  for (int s = 0; s < NO; ++s) {
    unpack8(NO < NS && half ? raw.p1[s + NS - NO] : raw.p1[s], o.q[s]);
    unpack8(NO < NS && half ? raw.p2[s + NS - NO] : raw.p2[s], o.k[s]);
  }
  const int ch0 = (NO < NS ? 32 * NO * half : 0) + 8 * L.g + here;  // first channel
  if (a.rope) {
    const int tc = min(t, a.T - 1) + here, h = a.rope_half;
    if (NO == NS && NS >= 2 && 2 * h == D) {
      rope_own<NO, WQ>(a, tc, L, o.q, o.k, false);
    } else {
      const int row = 16 * L.w + L.i;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (WQ) put_partner<2 * D>(X1, row, 32 * s + 8 * L.g, h, raw.p1[s]);
        put_partner<2 * D>(X2, row, 32 * s + 8 * L.g, h, raw.p2[s]);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int s = 0; s < NO; ++s) {
        const int c0 = ch0 + 32 * s;
        float cs[8], sn[8], y1[8], y2[8];
        rope_cs(a, tc, c0, false, cs, sn);
        if (WQ) unpack8(row_op<2 * D>(X1, row, c0 >> 3), y1);
        unpack8(row_op<2 * D>(X2, row, c0 >> 3), y2);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (WQ) o.q[s][u] = __builtin_fmaf(y1[u], sn[u], o.q[s][u] * cs[u]);
          o.k[s][u] = __builtin_fmaf(y2[u], sn[u], o.k[s][u] * cs[u]);
        }
        __builtin_amdgcn_sched_barrier(0);  // a piece at a time: the loads of all at once take too many registers
      }
    }
  }
  const float f1 = o.S * o.in1, f2 = o.S * o.in2;
#pragma unroll
  for (int s = 0; s < NO; ++s) {
    float al[8], dtb[8];
    if (a.a_log) {
      const unsigned pc = (unsigned)(n % a.H) * D + ch0 + 32 * s;
      ld_f32<VEC>(a.a_log + pc, al);
      ld_f32<VEC>(a.dt_bias + pc, dtb);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      o.q[s][u] *= f1;
      o.k[s][u] *= f2;
      float gg = raw.r[s][u];
      if (a.a_log) {
        const float ea = fast_exp2(al[u] * kLog2e), x = gg + dtb[u];
        const float e = fast_exp2(-fabsf(x) * kLog2e);
        gg = -ea * (fmaxf(x, 0.0f) + kLn2 * __builtin_amdgcn_logf(1.0f + e));
        if constexpr (GATE) {
          const float sg = fast_rcp(1.0f + e);
          gate->g[s][u] = gg;
          gate->d[s][u] = -ea * (x > 0.0f ? sg : e * sg);
        }
      }
      // 2^-512 counts as 0 wherever it is a factor; sums of b stay finite and as fine as that (NaN stays)
      const float b = gg * kLog2e;
      o.b[s][u] = b < -512.0f ? -512.0f : b;
    }
  }
  if (!whole && !ok) {
#pragma unroll
    for (int s = 0; s < NO; ++s)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        o.b[s][u] = 0.0f;
        if constexpr (GATE) gate->g[s][u] = gate->d[s][u] = 0.0f;
      }
  }
}

// Running sum of o.b down the chunk. tot [4][D] receives the blocks' totals
// (one barrier inside); off: the sum before the lane's block.
template <int D>  // D: channels of the pieces at hand
__device__ __forceinline__ void scan_b(Own<D / 32>& o, float (*tot)[D], const LaneIx& L, float (&off)[D / 32][8]) {
  constexpr int NS = D / 32;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int u = 0; u < 8; ++u) o.b[s][u] = scan16(o.b[s][u]);
    if (L.i == 15) st8f(&tot[L.w][32 * s + 8 * L.g], o.b[s]);
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int u = 0; u < 8; ++u) off[s][u] = 0.0f;
    for (int x = 0; x < L.w; ++x) {
      float y[8];
      ld8f(&tot[x][32 * s + 8 * L.g], y);
#pragma unroll
      for (int u = 0; u < 8; ++u) off[s][u] += y[u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) o.b[s][u] += off[s][u];
  }
}
// The chunk's last b at piece s of the lane.
template <int D>
__device__ __forceinline__ void last_b(const float (*tot)[D], int s, const LaneIx& L, float (&x)[8]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) x[u] = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float y[8];
    ld8f(&tot[w][32 * s + 8 * L.g], y);
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] += y[u];
  }
}

// Whether some channel of some block decays by more than 2^kSteep from the row
// before the block to its last (or by NaN): from the blocks' totals of scan_b, the
// same in every wave of the workgroup.
template <int D>
__device__ __forceinline__ bool chunk_steep(const float (*tot)[D]) {
  bool over = false;
#pragma unroll
  for (int x = 0; x < 4 * D / 64; ++x) over |= !(-(&tot[0][0])[64 * x + (int)(threadIdx.x & 63)] <= kSteep);
  return wave_any(over);
}

// Bit 8 s + u (wave-uniform): the block's range of b is over `limit` (or NaN) at
// element u of piece s in some lane group, four channels that then go term by term.
template <int D>
__device__ __forceinline__ unsigned block_over(const Own<D / 32>& o, float limit) {
  unsigned over = 0;
#pragma unroll
  for (int s = 0; s < D / 32; ++s)
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (wave_any(!(bcast16<0>(o.b[s][u]) - bcast16<15>(o.b[s][u]) <= limit))) over |= 1u << (8 * s + u);
  return __builtin_amdgcn_readfirstlane(over);
}
__device__ __forceinline__ bool is_over(unsigned over, int s, int u) { return (over >> (8 * s + u)) & 1; }

// Where the states of chunk c are. Within a segment of a.seg chunks the state
// kernel leaves every chunk's state from a zero start at the segment's first
// chunk; the state entering the segment joins with the retention in between:
//   C0_c = loc_c + pre_c in_seg      (loc: none in the segment's first chunk; in: none in the first segment)
// and in reverse for the gradient G of the state leaving the chunk.
struct StateRef {
  const float* loc;    // [D][D] or null
  const float* in;     // [D][D] or null
  const float* scale;  // [D]
};
template <int D>
__device__ __forceinline__ StateRef state_before(const LinearArgs& a, int n, int c) {
  const int s = c / a.seg;
  const int64_t at = (int64_t)n * a.nchunks + c;
  StateRef r;
  r.loc = c % a.seg ? a.cprev + at * D * D : nullptr;
  r.in = s ? a.segc + ((int64_t)n * a.nseg + s) * D * D : nullptr;
  r.scale = a.gpre + at * D;
  return r;
}
template <int D>
__device__ __forceinline__ StateRef grad_after(const LinearArgs& a, int n, int c) {
  const int s = c / a.seg;
  const int64_t at = (int64_t)n * a.nchunks + c;
  StateRef r;
  r.loc = (c + 1) % a.seg && c + 1 < a.nchunks ? a.gout + at * D * D : nullptr;
  r.in = s + 1 < a.nseg ? a.segp + ((int64_t)n * a.nseg + s) * D * D : nullptr;
  r.scale = a.gsuf + at * D;
  return r;
}
// 8 values of the state at row d, column e0.
template <int D>
__device__ __forceinline__ void ld_state(const StateRef& r, int d, int e0, float (&x)[8]) {
  const unsigned at = (unsigned)d * D + (unsigned)e0;
  float y[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) x[u] = 0.0f;
  if (r.loc) ld8f(r.loc + at, x);
  if (r.in) {
    ld8f(r.in + at, y);
    const float f = r.scale[(unsigned)d];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = __builtin_fmaf(f, y[u], x[u]);
  }
}

// ---------------------------------------------------------------------------
// Segment states. One workgroup walks the a.seg chunks of a segment with the
// state in registers (16 x 16 tiles, channels a on tile rows):
//   C <- e^{b_last} C + Kd^T v, Kd = k e^{b_last - b}
// and leaves, per chunk, the state before it from a zero start and, with more
// than one segment, the retention since the segment's start, and per segment
// the result and the retention. BWD: also P = Qe^T dY (Qe = q e^b) of every chunk, walked back to
// front at the end for the gradient of the state leaving each chunk. Bound by
// the rows' and the states' bytes.
// ---------------------------------------------------------------------------
constexpr int kMaxSeg = 8;

template <int D, bool BWD, bool VEC>
__global__ __launch_bounds__(kNT, D == 32 || (!BWD && D == 64) ? 3 : 2) void lin_state_kernel(LinearArgs a) {
  // at D = 128 two workgroups (blockIdx.z) share a segment, 64 of the state's
  // rows each: the registers of a whole one do not fit two waves per SIMD
  constexpr int DA = D < 64 ? D : 64;  // the workgroup's channels a
  constexpr int NS = D / 32, NO = DA / 32, RB = 2 * D, PS = kL * RB, RA = 2 * DA, PA = kL * RA, NP = BWD ? 3 : 1;
  constexpr int NE = D / 16;
  constexpr int AT = 1, ET = DA >= 64 ? NE : 1;  // tiles per wave: AT x ET
  __shared__ __attribute__((aligned(1024))) unsigned char K[NP * PA];
  __shared__ __attribute__((aligned(1024))) unsigned char V[PS];
  __shared__ float tot[4][DA];
  __shared__ float last[kMaxSeg][DA];  // b_last of the segment's chunks
  const LaneIx L;
  const int seg = blockIdx.x, n = blockIdx.y, half = DA < D ? blockIdx.z : 0, tid = threadIdx.x;
  const int a0 = DA * half;
  const int c0 = seg * a.seg, c1 = min(a.nchunks, c0 + a.seg);
  const int am = DA >= 64 ? L.w : L.w >> 1, em = DA >= 64 ? 0 : L.w & 1;  // first tile
  const int row = 16 * L.w + L.i;
  floatx4 C[AT][ET], P[AT][ET];
#pragma unroll
  for (int x = 0; x < AT; ++x)
#pragma unroll
    for (int y = 0; y < ET; ++y) C[x][y] = P[x][y] = floatx4{};
  float run = 0.0f;  // b since the segment's start, thread = channel
  // Rows are loaded a chunk ahead where the registers allow it (BWD, D = 64). At
  // D = 128 the spills cost more (930 against 868 us for a step of 32 heads x
  // 4096), and the forward is faster with a third workgroup per CU instead
  // (44 against 48 us for 16 heads x 3001 with the output kernel).
  constexpr bool kAhead = BWD && D == 64;
  Raw<D, BWD, NO> raw;
  if (kAhead) load_raw<D, BWD, VEC>(a, n, c0 * kL + row, half, L, raw);
  // RoPE partners on other lanes pass through V and (BWD, where K is the larger) K
  const bool turn = a.rope && !(NO == NS && NS >= 2 && 2 * a.rope_half == D);
  unsigned char* X1 = K;
  static_assert(!BWD || NP * PA >= PS, "a [64][D] array fits K");

  // acc += X^T Y over the chunk's 64 rows, X in NP parts
  auto gram = [&](floatx4 (&acc)[AT][ET]) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int r0 = 32 * ks + 4 * L.g + L.e;
      uintx4 xa[NP][AT];
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int x = 0; x < AT; ++x) {
          const uintx2 lo = lds_read_tr16(K + p * PA + coff<RA>(r0, 2 * (am + x) + (L.cg >> 1)) + 8 * (L.cg & 1));
          const uintx2 hi = lds_read_tr16(K + p * PA + coff<RA>(r0 + 16, 2 * (am + x) + (L.cg >> 1)) + 8 * (L.cg & 1));
          xa[p][x] = uintx4{lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
      for (int y = 0; y < ET; ++y) {
        const uintx2 lo = lds_read_tr16(V + coff<RB>(r0, 2 * (em + y) + (L.cg >> 1)) + 8 * (L.cg & 1));
        const uintx2 hi = lds_read_tr16(V + coff<RB>(r0 + 16, 2 * (em + y) + (L.cg >> 1)) + 8 * (L.cg & 1));
        const uintx4 yb = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
        for (int p = NP - 1; p >= 0; --p)
#pragma unroll
          for (int x = 0; x < AT; ++x) acc[x][y] = mm32(xa[p][x], yb, acc[x][y]);
      }
    }
  };
  auto scale_rows = [&](floatx4 (&acc)[AT][ET], const float* lb) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < AT; ++x) {
      const floatx4 l4 = *reinterpret_cast<const floatx4*>(lb + 16 * (am + x) + 4 * L.g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float f = fast_exp2(l4[v]);
#pragma unroll
        for (int y = 0; y < ET; ++y) acc[x][y][v] *= f;
      }
    }
  };
  auto store = [&](float* out, const floatx4 (&acc)[AT][ET]) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < AT; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int y = 0; y < ET; ++y) out[(a0 + 16 * (am + x) + 4 * L.g + v) * D + 16 * (em + y) + L.i] = acc[x][y][v];
  };

  for (int c = c0; c < c1; ++c) {
    const int t = c * kL + row;
    const bool ok = t < a.T;
    Own<NO> o;
    if (!kAhead) load_raw<D, BWD, VEC>(a, n, t, half, L, raw);
    if (turn) __syncthreads();  // everyone is past the products of the chunk before: K and V are free
    use_raw<D, NO, BWD, VEC, BWD>(a, n, t, ok, half, L, X1, V, raw, o);
    uintx4 v[NS], dy[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      v[s] = raw.v[s];
      if (BWD) dy[s] = raw.dy[s];
    }
    if (kAhead && c + 1 < c1) load_raw<D, BWD, VEC>(a, n, t + kL, half, L, raw);
    float off[NO][8];
    scan_b<DA>(o, tot, L, off);  // its barrier: everyone is past the products of the chunk before
#pragma unroll
    for (int s = 0; s < NO; ++s) {
      float lb[8], x[8];
      last_b<DA>(tot, s, L, lb);
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = o.k[s][u] * fast_exp2(lb[u] - o.b[s][u]);
      if constexpr (BWD) {
        uintx4 h, m, l;
        split8(x, h, m, l);
        put_row<RA>(K, row, 4 * s + L.g, h);
        put_row<RA>(K + PA, row, 4 * s + L.g, m);
        put_row<RA>(K + 2 * PA, row, 4 * s + L.g, l);
      } else {
        put_row<RA>(K, row, 4 * s + L.g, pack8(x));
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) put_row<RB>(V, row, 4 * s + L.g, v[s]);
    const int64_t at = (int64_t)n * a.nchunks + c;
    if (tid < DA) {
      const float lb = ((tot[0][tid] + tot[1][tid]) + tot[2][tid]) + tot[3][tid];
      last[c - c0][tid] = lb;
      if (a.nseg > 1) a.gpre[at * D + a0 + tid] = fast_exp2(run);
      run += lb;
    }
    if (c > c0) store(a.cprev + at * D * D, C);
    __syncthreads();
    scale_rows(C, last[c - c0]);
    gram(C);
    if constexpr (BWD) {
      __syncthreads();
#pragma unroll
      for (int s = 0; s < NO; ++s) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = o.q[s][u] * fast_exp2(o.b[s][u]);
        uintx4 h, m, l;
        split8(x, h, m, l);
        put_row<RA>(K, row, 4 * s + L.g, h);
        put_row<RA>(K + PA, row, 4 * s + L.g, m);
        put_row<RA>(K + 2 * PA, row, 4 * s + L.g, l);
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) put_row<RB>(V, row, 4 * s + L.g, dy[s]);
      __syncthreads();
#pragma unroll
      for (int x = 0; x < AT; ++x)
#pragma unroll
        for (int y = 0; y < ET; ++y) P[x][y] = floatx4{};
      gram(P);
      if (c + 1 < c1) store(a.gout + at * D * D, P);
    }
  }
  const int64_t sg = (int64_t)n * a.nseg + seg;
  if (a.nseg > 1) {
    store(a.segc + sg * D * D, C);
    if (tid < DA) a.segg[sg * D + a0 + tid] = fast_exp2(run);
  } else if (a.state_out) {
    store(a.state_out + (int64_t)n * D * D, C);
  }
  if constexpr (BWD) {
    // P holds the last chunk's: the gradient of the state before it, from a
    // zero start after the segment. Back to front, the chunk's stored P makes
    // way for the gradient of the state leaving it.
    float suf = 0.0f;
    if (a.nseg > 1 && tid < DA) {
      for (int c = c1 - 1; c >= c0; --c) {
        a.gsuf[((int64_t)n * a.nchunks + c) * D + a0 + tid] = fast_exp2(suf);
        suf += last[c - c0][tid];
      }
    }
    for (int c = c1 - 2; c >= c0; --c) {
      float* slot = a.gout + ((int64_t)n * a.nchunks + c) * D * D;
      floatx4 Q[AT][ET];
#pragma unroll
      for (int x = 0; x < AT; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int y = 0; y < ET; ++y) Q[x][y][v] = slot[(a0 + 16 * (am + x) + 4 * L.g + v) * D + 16 * (em + y) + L.i];
      store(slot, P);
      scale_rows(P, last[c - c0]);
#pragma unroll
      for (int x = 0; x < AT; ++x)
#pragma unroll
        for (int y = 0; y < ET; ++y) P[x][y] += Q[x][y];
    }
    if (a.nseg > 1) store(a.segp + sg * D * D, P);
  }
}

// The segments' results become the states entering them (z = 0; the state
// after the last token goes to state_out), and in reverse the gradients of the
// states leaving them (z = 1). A workgroup takes 64 state elements, wave w the
// segments 16 w .. 16 w + 15 of every 64: it loads them all before it walks
// them, the waves' results meet in LDS, and a second walk over the registers
// writes the entering states. (One thread per element over all segments took
// 7.5 us for 47 segments, three dependent rounds of loads.)
__global__ __launch_bounds__(kNT) void lin_scan_kernel(LinearArgs a) {
  constexpr int BT = 16;
  __shared__ float lc[2][4][64], lp[2][4][64];
  // up to 16 segments: a wave has all of them, and each wave elements of its own
  const bool solo = a.nseg <= BT;
  const int D = a.D, DD = D * D, e = threadIdx.x & 63, w = solo ? 0 : threadIdx.x >> 6;
  const int idx = solo ? (int)blockIdx.x * kNT + threadIdx.x : (int)blockIdx.x * 64 + e;  // D D is a multiple of both
  const int64_t n = blockIdx.y;
  const bool rev = blockIdx.z == 1;
  const float* gg = a.segg + n * a.nseg * D + idx / D;
  float* st = (rev ? a.segp : a.segc) + n * a.nseg * DD + idx;
  float carry = 0.0f;
  for (int r0 = 0, it = 0; r0 < a.nseg; r0 += 4 * BT, it ^= 1) {
    const int s0 = r0 + BT * w;
    float gv[BT], sv[BT];
#pragma unroll
    for (int k = 0; k < BT; ++k) {
      const int s = min(s0 + k, a.nseg - 1), at = rev ? a.nseg - 1 - s : s;
      gv[k] = gg[(int64_t)at * D];
      sv[k] = st[(int64_t)at * DD];
    }
    float C = 0.0f, prod = 1.0f;
#pragma unroll
    for (int k = 0; k < BT; ++k) {
      if (s0 + k < a.nseg) {
        C = __builtin_fmaf(gv[k], C, sv[k]);
        prod *= gv[k];
      }
    }
    if (solo) {
      carry = C;
      C = 0.0f;
    } else {
      lc[it][w][e] = C;
      lp[it][w][e] = prod;
      __syncthreads();  // two buffers: the next round writes the other one
      float run = carry;
      for (int x = 0; x < 4; ++x) {
        if (x == w) C = run;  // the state entering this wave's segments
        run = __builtin_fmaf(lp[it][x][e], run, lc[it][x][e]);
      }
      carry = run;
    }
#pragma unroll
    for (int k = 0; k < BT; ++k) {
      const int s = s0 + k, at = rev ? a.nseg - 1 - s : s;
      if (s < a.nseg) {
        st[(int64_t)at * DD] = C;
        C = __builtin_fmaf(gv[k], C, sv[k]);
      }
    }
  }
  if (!rev && a.state_out && w == 0) a.state_out[n * DD + idx] = carry;
}

// A block's own pairs, term by term, for one channel of the lane's row with
// exponent b: offset X + x, x < N, pairs the row with row i - X - x (or i + X + x,
// LATER) of the block, whose value `other` comes by a row shift. y = other
// e^{b_t - b_j}, 0 past the block's ends, goes to grad += d[x] y and P[x] += own y.
// Through ds_bpermute, and with a sum over the lane groups per channel and
// offset, a step of 16 heads x 4096 with every channel steep took 141, 309 and 767
// us at width 32, 64 and 128 (linear.hip's kernels: 118, 184, 729); so 79, 159, 492.
template <bool LATER, bool GRAD, bool SCORE, int X, int N, int x = 0>
__device__ __forceinline__ void exact_terms(int i, float own, float other, float b, const float (&d)[N], float& grad,
                                            float (&P)[N]) {
  constexpr int CTRL = (LATER ? 0x100 : 0x110) + X + x;  // row_shl, row_shr
  const float bx = dpp_shift<CTRL>(b);
  const float e = dpp_shift<CTRL>(other) * fast_exp2(LATER ? bx - b : b - bx);
  const float y = (LATER ? i < 16 - X - x : i >= X + x) ? e : 0.0f;
  if (GRAD) grad = __builtin_fmaf(d[x], y, grad);
  if (SCORE) P[x] = __builtin_fmaf(own, y, P[x]);
  if constexpr (x + 1 < N) exact_terms<LATER, GRAD, SCORE, X, N, x + 1>(i, own, other, b, d, grad, P);
}
// The same for every channel of `over`, offsets X .. 15 in runs of N: grad +=
// z' y with z' the block z (4 rows or columns per lane group) at the offset, r
// the scores' block. N = 0: a piece of eight channels and one offset at a time, in
// a loop that shifts the other rows on by one, for the width-128 gradient kernel,
// whose common path the registers of unrolled runs slow down (a step of 16 heads x
// 4096 without steep channels 450 us with runs of 3, 399 so).
template <bool LATER, bool GRAD, bool SCORE, int NS, int N, int X = 1>
__device__ __forceinline__ void exact_block(unsigned over, const LaneIx& L, const float (&own)[NS][8],
                                            const float (&other)[NS][8], const float (&b)[NS][8], const floatx4& z,
                                            float (&grad)[NS][8], floatx4& r) {
  static_assert(N == 0 || (16 - X) % N == 0, "whole runs");
  constexpr int M = N ? N : 1;
  auto pick = [&](int at) __attribute__((always_inline)) {  // z at the row's column (or row) `at`, to all its lane groups
    const float lo = at & 1 ? z[1] : z[0], hi = at & 1 ? z[3] : z[2];
    return __shfl(at & 2 ? hi : lo, L.i + 16 * ((at >> 2) & 3), 64);
  };
  auto put = [&](int at, float p) __attribute__((always_inline)) {
    const float sc = sum_groups(p);
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] += at == 4 * L.g + v ? sc : 0.0f;
  };
  float d[M], P[M];
  if constexpr (N == 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if ((over >> (8 * s)) & 255u) {  // the piece's eight channels together: their chains overlap
        float ox[8], bx[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          ox[u] = other[s][u];
          bx[u] = b[s][u];
        }
#pragma unroll 1
        for (int x = 1; x < 16; ++x) {
          const int at = LATER ? L.i + x : L.i - x;
          if (GRAD) d[0] = pick(at);
          P[0] = 0.0f;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            ox[u] = dpp_shift<(LATER ? 0x101 : 0x111)>(ox[u]);
            bx[u] = dpp_shift<(LATER ? 0x101 : 0x111)>(bx[u]);
            const float e = ox[u] * fast_exp2(LATER ? bx[u] - b[s][u] : b[s][u] - bx[u]);
            const float y = (at & 15) == at && is_over(over, s, u) ? e : 0.0f;
            if (GRAD) grad[s][u] = __builtin_fmaf(d[0], y, grad[s][u]);
            if (SCORE) P[0] = __builtin_fmaf(own[s][u], y, P[0]);
          }
          if (SCORE) put(at, P[0]);
        }
      }
  } else {
#pragma unroll
    for (int x = 0; x < M; ++x) {
      P[x] = 0.0f;
      if (GRAD) d[x] = pick(LATER ? L.i + X + x : L.i - X - x);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (is_over(over, s, u))
          exact_terms<LATER, GRAD, SCORE, X, N>(L.i, own[s][u], other[s][u], b[s][u], d, grad[s][u], P);
    if (SCORE) {
#pragma unroll
      for (int x = 0; x < M; ++x) put(LATER ? L.i + X + x : L.i - X - x, P[x]);
    }
    if constexpr (X + N < 16) exact_block<LATER, GRAD, SCORE, NS, N, X + N>(over, L, own, other, b, z, grad, r);
  }
}

// Per chunk: Y_t = v_t + sum_{j < t} A_tj v_j + Qe C0.
template <int D, bool VEC>
__global__ __launch_bounds__(kNT, D <= 64 ? 3 : 2) void lin_out_kernel(LinearArgs a) {
  constexpr int NS = D / 32, NM = D / 16, RB = 2 * D, PS = kL * RB;
  constexpr int NCT = D * D / 8 / kNT > 0 ? D * D / 8 / kNT : 1;  // pieces of C0 per thread
  __shared__ __attribute__((aligned(1024))) unsigned char KE[PS];    // k e^{b_end - b}, b_end: the block's last b
  __shared__ __attribute__((aligned(1024))) unsigned char V[PS];
  __shared__ __attribute__((aligned(1024))) unsigned char CS[D * RB];  // the state entering the chunk
  __shared__ float tot[4][D], bnd[4][D];
  const LaneIx L;
  const int c = blockIdx.x, n = blockIdx.y, tid = threadIdx.x;
  const int row = 16 * L.w + L.i, t = c * kL + row;
  const bool ok = t < a.T;
  Raw<D, false> raw;
  load_raw<D, false, VEC>(a, n, t, 0, L, raw);
  const StateRef sr = state_before<D>(a, n, c);
  const bool inter = c > 0;
  uintx4 c0r[NCT];  // the state, read under the row loads
  if (inter) {
#pragma unroll
    for (int x = 0; x < NCT; ++x) {
      const int task = tid + x * kNT;
      if (D * D / 8 >= kNT || task < D * D / 8) {
        float y[8];
        ld_state<D>(sr, task / (D / 8), 8 * (task % (D / 8)), y);
        c0r[x] = pack8(y);
      }
    }
  }
  Own<NS> o;
  use_raw<D, NS, false, VEC, true>(a, n, t, ok, 0, L, KE, V, raw, o);
  float off[NS][8];
  scan_b<D>(o, tot, L, off);
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    float x[8], e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      e[u] = bcast16<15>(o.b[s][u]);
      x[u] = o.k[s][u] * fast_exp2(e[u] - o.b[s][u]);
    }
    if (L.i == 0) st8f(&bnd[L.w][32 * s + 8 * L.g], e);
    put_row<RB>(KE, row, 4 * s + L.g, pack8(x));
    put_row<RB>(V, row, 4 * s + L.g, raw.v[s]);
  }
  if (inter) {
#pragma unroll
    for (int x = 0; x < NCT; ++x) {
      const int task = tid + x * kNT;
      if (D * D / 8 >= kNT || task < D * D / 8) put_row<RB>(CS, task / (D / 8), task % (D / 8), c0r[x]);
    }
  }
  __syncthreads();
  floatx4 acc[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
  auto add_block = [&](int jb, const floatx4& at) __attribute__((always_inline)) {
    const uintx2 p = {pk2(at[0], at[1]), pk2(at[2], at[3])};
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = mm16(tr_op<RB>(V, 16 * jb + 4 * L.g + L.e, m, L), p, acc[m]);
  };
  for (int jb = 0; jb < L.w; ++jb) {
    floatx4 at = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8], e[8];
      ld8f(&bnd[jb][32 * s + 8 * L.g], e);
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = o.q[s][u] * fast_exp2(o.b[s][u] - e[u]);
      at = mm32(row_op<RB>(KE, 16 * jb + L.i, 4 * s + L.g), pack8(x), at);
    }
    add_block(jb, at);
  }
  // the block's own pairs
  auto own_block = [&](auto steep) __attribute__((always_inline)) {
    constexpr bool STEEP = decltype(steep)::value;
    const unsigned over = STEEP ? block_over<D>(o, wave_any(o.S < kSmallS) ? kSteep : kRange) : 0;
    floatx4 at = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8], y[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float d = o.b[s][u] - 0.5f * (bcast16<0>(o.b[s][u]) + bcast16<15>(o.b[s][u]));
        x[u] = STEEP && is_over(over, s, u) ? 0.0f : o.q[s][u] * fast_exp2(d);
        y[u] = STEEP && is_over(over, s, u) ? 0.0f : o.k[s][u] * fast_exp2(-d);
      }
      at = STEEP ? mm32_split(y, x, at) : mm32(pack8(y), pack8(x), at);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) at[v] = 4 * L.g + v < L.i ? at[v] : 0.0f;
    if constexpr (STEEP) {
      if (over) exact_block<false, false, true, NS, D == 128 ? 3 : 15>(over, L, o.q, o.k, o.b, at, o.q, at);
    }
    add_block(L.w, at);
  };
  if (chunk_steep<D>(tot)) own_block(std::true_type{});
  else own_block(std::false_type{});
  if (inter) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = o.q[s][u] * fast_exp2(o.b[s][u]);
      const uintx4 qe = pack8(x);
      const int r0 = 32 * s + 8 * L.g + L.e;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const uintx2 lo = tr_op<RB>(CS, r0, m, L), hi = tr_op<RB>(CS, r0 + 4, m, L);
        acc[m] = mm32(uintx4{lo[0], lo[1], hi[0], hi[1]}, qe, acc[m]);
      }
    }
  }
  if (!ok) return;
  bf16* Y = (bf16*)a.out + head_off(a, n) + (int64_t)t * a.st + 8 * L.g;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    float x[8];
    unpack8(raw.v[s], x);
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] += acc[2 * s + (u >> 2)][u & 3];
    st_row<VEC>(Y + 32 * s, pack8(x));
  }
}

// The gate's values at the lane's elements, from memory once more.
template <int D, bool VEC>
__device__ __forceinline__ void gate_again(const LinearArgs& a, int n, int t, bool ok, const LaneIx& L,
                                           Gate<D / 32>& gate) {
  const float* G = a.g + (int64_t)n * a.T * D + ((unsigned)min(t, a.T - 1) * D + 8u * L.g);
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    float al[8], dtb[8], r8[8];
    const unsigned pc = (unsigned)(n % a.H) * D + 32 * s + 8 * L.g;
    ld_f32<VEC>(a.a_log + pc, al);
    ld_f32<VEC>(a.dt_bias + pc, dtb);
    ld_f32<VEC>(G + 32 * s, r8);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float ea = fast_exp2(al[u] * kLog2e), x = r8[u] + dtb[u];
      const float e = fast_exp2(-fabsf(x) * kLog2e), sg = fast_rcp(1.0f + e);
      gate.g[s][u] = ok ? -ea * (fmaxf(x, 0.0f) + kLn2 * __builtin_amdgcn_logf(1.0f + e)) : 0.0f;
      gate.d[s][u] = ok ? -ea * (x > 0.0f ? sg : e * sg) : 0.0f;
    }
  }
}

// ---------------------------------------------------------------------------
// Every input gradient of a chunk (the formulas are at the backward section of
// linear.hip). Four phases share one LDS region of three bf16 parts:
//   C0:  dq = e^b (dY C0^T)
//   K':  dA^T = V dY^T, dq += dA K'                       (blocks j <= own)
//   G:   dk = e^{b_last - b} (V G^T), dv = Kd G
//   Q':  dA = dY V^T, A, dk += dA^T Q', dv += A^T dY      (blocks t >= own)
// then db = q dq - k dk, its reverse running sum to dg, the gate, S and the
// normalisation, all on the lane's own row. The states are staged in column
// slabs of 64 so that the region holds D = 128 too.
// ---------------------------------------------------------------------------
template <int D, bool VEC>
__global__ __launch_bounds__(kNT, 2) void lin_grad_kernel(LinearArgs a) {
  constexpr int NS = D / 32, NM = D / 16, RB = 2 * D, PS = kL * RB;
  constexpr int ES = D < 64 ? D : 64, EB = 2 * ES, NSL = D / ES, NSE = ES / 32, EM = ES / 16;
  constexpr int NPC = D * ES / 8;                      // 16-byte pieces of a state slab
  constexpr int NCT = NPC / kNT > 0 ? NPC / kNT : 1;   // per thread
  static_assert(D * EB <= PS, "a state slab fits a part");
  __shared__ __attribute__((aligned(1024))) unsigned char R[4 * PS];  // three parts; V or dY
  __shared__ float tot[4][D], ck[4][D], cq[4][D], ek[3][D], eq[3][D], gm[D], pt[4][D], ex[4][D], lst[D];
  unsigned char* VY = R + 3 * PS;
  const LaneIx L;
  const int c = blockIdx.x, n = blockIdx.y, tid = threadIdx.x;
  const int row = 16 * L.w + L.i, t = c * kL + row;
  const bool ok = t < a.T;
  constexpr bool KEEP_G = D <= 64;  // the gate's values stay in registers to the end (else formed again)
  Gate<NS> gate;
  Own<NS> o;
  uintx4 vo[NS], dyo[NS];
  {
    Raw<D, true> raw;
    load_raw<D, true, VEC>(a, n, t, 0, L, raw);
    use_raw<D, NS, true, VEC, true, KEEP_G>(a, n, t, ok, 0, L, R, R + PS, raw, o, &gate);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      vo[s] = raw.v[s];
      dyo[s] = raw.dy[s];
    }
  }
  float off[NS][8];
  scan_b<D>(o, tot, L, off);
  auto rest = [&](auto steep) __attribute__((always_inline)) {
  constexpr bool STEEP = decltype(steep)::value;
  const unsigned over = STEEP ? block_over<D>(o, wave_any(o.S < kSmallS) ? kSteep : kRange) : 0;
  const bool fine = STEEP && (D < 128 || chunk_steep<D>(tot));  // the blocks' own scores keep fp32 accuracy
  {
    if (tid < D) lst[tid] = ((tot[0][tid] + tot[1][tid]) + tot[2][tid]) + tot[3][tid];  // b_last, as scan_b adds it
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float k8[8], q8[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float b0 = bcast16<0>(o.b[s][u]), b1 = bcast16<15>(o.b[s][u]);
        const float mid = 0.5f * (b0 + b1);
        k8[u] = STEEP && is_over(over, s, u) ? b1 : mid;
        q8[u] = STEEP && is_over(over, s, u) ? off[s][u] : mid;
      }
      if (L.i == 0) {
        st8f(&ck[L.w][32 * s + 8 * L.g], k8);
        st8f(&cq[L.w][32 * s + 8 * L.g], q8);
      }
    }
  }
  // q is not held through the last phases at D >= 64 (registers): it comes back
  // from its parts, or in a block with steep channels through memory
  float* qsave = a.qn + ((int64_t)n * a.T + min(t, a.T - 1)) * D + 8 * L.g;
  constexpr bool KEEP_Q = D < 64;
  if (STEEP && !KEEP_Q && over && ok) {
#pragma unroll
    for (int s = 0; s < NS; ++s) st8f(qsave + 32 * s, o.q[s]);
  }
  // a slab of a state, split in three, to the region
  const StateRef cref = state_before<D>(a, n, c), gref = grad_after<D>(a, n, c);
  const bool has_c = c > 0, has_g = c + 1 < a.nchunks;
  // rows d of tile m: channel 32 (m / 2) + 8 (i / 4) + 4 (m % 2) + i % 4
  auto drow = [&](int m) { return 32 * (m >> 1) + 8 * L.e + 4 * (m & 1) + L.cg; };

  float dq[NS][8];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int u = 0; u < 8; ++u) dq[s][u] = 0.0f;
  if (has_c) {
    floatx4 acc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) {
      if (sl) __syncthreads();
#pragma unroll
      for (int x = 0; x < NCT; ++x) {
        const int task = tid + x * kNT;
        if (NPC >= kNT || task < NPC) {
          const int d = task / (ES / 8), ch = task % (ES / 8);
          float y[8];
          ld_state<D>(cref, d, sl * ES + 8 * ch, y);
          uintx4 h, m, l;
          split8(y, h, m, l);
          put_row<EB>(R, d, ch, h);
          put_row<EB>(R + PS, d, ch, m);
          put_row<EB>(R + 2 * PS, d, ch, l);
        }
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int se = 0; se < NSE; ++se)
#pragma unroll
          for (int p = 2; p >= 0; --p)
            acc[m] = mm32(row_op<EB>(R + p * PS, drow(m), 4 * se + L.g), dyo[sl * NSE + se], acc[m]);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int u = 0; u < 8; ++u) dq[s][u] = acc[2 * s + (u >> 2)][u & 3] * fast_exp2(o.b[s][u]);
    __syncthreads();  // the region is free
  } else {
    __syncthreads();  // ck and cq are written
  }

  // x e^{+-(b - reference)} of the lane's row, split in three, to the region
  auto put_parts = [&](const float (&x)[NS][8], const float* ref, float sign) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float r8[8], y[8];
      ld8f(ref + 32 * s + 8 * L.g, r8);
#pragma unroll
      for (int u = 0; u < 8; ++u) y[u] = x[s][u] * fast_exp2(sign * (o.b[s][u] - r8[u]));
      uintx4 h, m, l;
      split8(y, h, m, l);
      put_row<RB>(R, row, 4 * s + L.g, h);
      put_row<RB>(R + PS, row, 4 * s + L.g, m);
      put_row<RB>(R + 2 * PS, row, 4 * s + L.g, l);
    }
  };
  // acc += X'^T (block blk's rows, in three parts) times a 16 x 16 block z, six products
  auto mul_block = [&](floatx4 (&acc)[NM], int blk, const floatx4& z) __attribute__((always_inline)) {
    uintx2 zh, zm, zl;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      unsigned hh, mm, ll;
      split_pair(z[2 * x], z[2 * x + 1], hh, mm, ll);
      zh[x] = hh;
      zm[x] = mm;
      zl[x] = ll;
    }
    const int r0 = 16 * blk + 4 * L.g + L.e;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const uintx2 xh = tr_op<RB>(R, r0, m, L), xm = tr_op<RB>(R + PS, r0, m, L), xl = tr_op<RB>(R + 2 * PS, r0, m, L);
      acc[m] = mm16(xl, zh, acc[m]);
      acc[m] = mm16(xh, zl, acc[m]);
      acc[m] = mm16(xm, zm, acc[m]);
      acc[m] = mm16(xm, zh, acc[m]);
      acc[m] = mm16(xh, zm, acc[m]);
      acc[m] = mm16(xh, zh, acc[m]);
    }
  };
  // e^x between blocks, held as its root in the path for steep channels, and x y with it
  auto factor = [](float x) __attribute__((always_inline)) { return fast_exp2(STEEP ? 0.5f * x : x); };
  auto times = [](float x, float f) __attribute__((always_inline)) { return STEEP ? x * f * f : x * f; };
  auto scale_tiles = [&](floatx4 (&acc)[NM], const float* f) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float f8[8];
      ld8f(f + 32 * s + 8 * L.g, f8);
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[2 * s + (u >> 2)][u & 3] = times(acc[2 * s + (u >> 2)][u & 3], f8[u]);
    }
  };

  // ---- K': dq over the keys of this and the earlier blocks
  put_parts(o.k, ck[L.w], -1.0f);
#pragma unroll
  for (int s = 0; s < NS; ++s) put_row<RB>(VY, row, 4 * s + L.g, vo[s]);
  for (int x = tid; x < 3 * D; x += kNT) {
    const int u = x / D, d = x % D;
    ek[u][d] = factor(ck[u + 1][d] - ck[u][d]);
    eq[u][d] = factor(cq[u + 1][d] - cq[u][d]);
  }
  __syncthreads();
  {
    floatx4 acc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
#pragma unroll 1
    for (int jb = 0; jb < L.w; ++jb) {
      if (jb) scale_tiles(acc, ek[jb - 1]);  // before z: a matrix result is first read in its own basic block
      floatx4 z = {};
#pragma unroll
      for (int s = 0; s < NS; ++s) z = mm32(row_op<RB>(VY, 16 * jb + L.i, 4 * s + L.g), dyo[s], z);
      mul_block(acc, jb, z);
    }
    if (L.w > 0) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        float r8[8];
        ld8f(&ck[L.w - 1][32 * s + 8 * L.g], r8);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          dq[s][u] += times(acc[2 * s + (u >> 2)][u & 3], factor(o.b[s][u] - r8[u]));
      }
    }
    floatx4 z = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) z = mm32(vo[s], dyo[s], z);
#pragma unroll
    for (int v = 0; v < 4; ++v) z[v] = 4 * L.g + v < L.i ? z[v] : 0.0f;
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
    mul_block(acc, L.w, z);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float r8[8];
      ld8f(&ck[L.w][32 * s + 8 * L.g], r8);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float f = STEEP && is_over(over, s, u) ? 0.0f : fast_exp2(o.b[s][u] - r8[u]);
        dq[s][u] = __builtin_fmaf(acc[2 * s + (u >> 2)][u & 3], f, dq[s][u]);
      }
    }
    if (STEEP && over) exact_block<false, true, false, NS, D == 128 ? 0 : 15>(over, L, o.q, o.k, o.b, z, dq, z);
  }
  __syncthreads();  // the region is free

  // ---- G: the state's gradient
  float dk[NS][8];
  floatx4 av[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) av[m] = floatx4{};
  if (has_g) {
    floatx4 acc[NM];
    uintx4 kd[NS];
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float lb[8], x[8];
      ld8f(lst + 32 * s + 8 * L.g, lb);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        dk[s][u] = fast_exp2(lb[u] - o.b[s][u]);
        x[u] = o.k[s][u] * dk[s][u];
      }
      kd[s] = pack8(x);
    }
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) {
      if (sl) __syncthreads();
#pragma unroll
      for (int x = 0; x < NCT; ++x) {
        const int task = tid + x * kNT;
        if (NPC >= kNT || task < NPC) {
          const int d = task / (ES / 8), ch = task % (ES / 8);
          float y[8], z[8];
          ld_state<D>(gref, d, sl * ES + 8 * ch, y);
          uintx4 h, m, l;
          split8(y, h, m, l);
          put_row<EB>(R, d, ch, h);
          put_row<EB>(R + PS, d, ch, m);
          put_row<EB>(R + 2 * PS, d, ch, l);
          // sum_e G C0 of row d, for the decay gradient: the ES / 8 pieces of a row are one lane group
          float dot = 0.0f;
          if (has_c) {
            ld_state<D>(cref, d, sl * ES + 8 * ch, z);
#pragma unroll
            for (int u = 0; u < 8; ++u) dot = __builtin_fmaf(y[u], z[u], dot);
          }
          dot = lane_group_sum<ES / 8>(dot);
          if (ch == 0) gm[d] = sl ? gm[d] + dot : dot;
        }
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int se = 0; se < NSE; ++se)
#pragma unroll
          for (int p = 2; p >= 0; --p)
            acc[m] = mm32(row_op<EB>(R + p * PS, drow(m), 4 * se + L.g), vo[sl * NSE + se], acc[m]);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int r0 = 32 * s + 8 * L.g + L.e;
#pragma unroll
        for (int m = 0; m < EM; ++m) {
          const uintx2 lo = tr_op<EB>(R, r0, m, L), hi = tr_op<EB>(R, r0 + 4, m, L);
          av[sl * EM + m] = mm32(uintx4{lo[0], lo[1], hi[0], hi[1]}, kd[s], av[sl * EM + m]);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        dk[s][u] *= acc[2 * s + (u >> 2)][u & 3];
        x[u] = group_sum<16>(dk[s][u] * o.k[s][u]);  // sum over the block's rows of dKd Kd
      }
      if (L.i == 0) st8f(&ex[L.w][32 * s + 8 * L.g], x);
    }
    __syncthreads();  // the region is free
  } else {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) dk[s][u] = x[u] = 0.0f;
      if (L.i == 0) st8f(&ex[L.w][32 * s + 8 * L.g], x);
    }
    if (tid < D) gm[tid] = 0.0f;
  }

  // ---- Q': dk and dv over the queries of this and the later blocks
  put_parts(o.q, cq[L.w], 1.0f);
#pragma unroll
  for (int s = 0; s < NS; ++s) put_row<RB>(VY, row, 4 * s + L.g, dyo[s]);
  __syncthreads();
  {
    floatx4 acc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
    auto add_dv = [&](int tb, const floatx4& s4) __attribute__((always_inline)) {
      const uintx2 p = {pk2(s4[0], s4[1]), pk2(s4[2], s4[3])};
#pragma unroll
      for (int m = 0; m < NM; ++m) av[m] = mm16(tr_op<RB>(VY, 16 * tb + 4 * L.g + L.e, m, L), p, av[m]);
    };
    // scores of block tb's queries with this block's keys (t on tile rows, j on lanes)
    auto scores = [&](int tb) __attribute__((always_inline)) {
      floatx4 s4 = {};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        float r8[8], x[8];
        ld8f(&cq[tb][32 * s + 8 * L.g], r8);
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = o.k[s][u] * fast_exp2(r8[u] - o.b[s][u]);
        s4 = mm32(row_op<RB>(R, 16 * tb + L.i, 4 * s + L.g), pack8(x), s4);
      }
      return s4;
    };
#pragma unroll 1
    for (int tb = 3; tb > L.w; --tb) {
      if (tb < 3) scale_tiles(acc, eq[tb]);
      floatx4 z = {};
#pragma unroll
      for (int s = 0; s < NS; ++s) z = mm32(row_op<RB>(VY, 16 * tb + L.i, 4 * s + L.g), vo[s], z);
      mul_block(acc, tb, z);
      add_dv(tb, scores(tb));
    }
    if (L.w < 3) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        float r8[8];
        ld8f(&cq[L.w + 1][32 * s + 8 * L.g], r8);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          dk[s][u] += times(acc[2 * s + (u >> 2)][u & 3], factor(r8[u] - o.b[s][u]));
      }
    }
    floatx4 z = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) z = mm32(dyo[s], vo[s], z);
#pragma unroll
    for (int v = 0; v < 4; ++v) z[v] = 4 * L.g + v > L.i ? z[v] : 0.0f;
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = floatx4{};
    mul_block(acc, L.w, z);
    floatx4 sf = {};  // the block's own scores with fp32 accuracy, six products
    if (fine) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        float r8[8], x[8];
        ld8f(&cq[L.w][32 * s + 8 * L.g], r8);
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = is_over(over, s, u) ? 0.0f : o.k[s][u] * fast_exp2(r8[u] - o.b[s][u]);
#pragma unroll
        for (int p = 0; p < 3; ++p) {  // x's parts one after the other: registers
          const uintx4 xp = pack8(x);
          float h[8];
          unpack8(xp, h);
#pragma unroll
          for (int y = 2 - p; y >= 0; --y) sf = mm32(row_op<RB>(R + y * PS, row, 4 * s + L.g), xp, sf);
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] -= h[u];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    floatx4 s4 = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float r8[8], x[8];
      ld8f(&cq[L.w][32 * s + 8 * L.g], r8);
      const uintx4 qh = row_op<RB>(R, row, 4 * s + L.g);
      float h[8], m[8], l[8];
      if constexpr (!KEEP_Q) {  // q back from its parts (the lane's own row)
        unpack8(qh, h);
        unpack8(row_op<RB>(R + PS, row, 4 * s + L.g), m);
        unpack8(row_op<RB>(R + 2 * PS, row, 4 * s + L.g), l);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float f = STEEP && is_over(over, s, u) ? 0.0f : fast_exp2(r8[u] - o.b[s][u]);
        x[u] = o.k[s][u] * f;
        dk[s][u] = __builtin_fmaf(acc[2 * s + (u >> 2)][u & 3], f, dk[s][u]);
        if constexpr (!KEEP_Q) o.q[s][u] = ((l[u] + m[u]) + h[u]) * f;
      }
      s4 = mm32(qh, pack8(x), s4);
    }
    if (fine) s4 = sf;
#pragma unroll
    for (int v = 0; v < 4; ++v) s4[v] = 4 * L.g + v > L.i ? s4[v] : 0.0f;
    if (STEEP && over) {
      if constexpr (!KEEP_Q) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          ld8f(qsave + 32 * s, o.q[s]);
#pragma unroll
          for (int u = 0; u < 8; ++u) o.q[s][u] = ok ? o.q[s][u] : 0.0f;
        }
      }
      exact_block<true, true, true, NS, D == 128 ? 0 : 15>(over, L, o.k, o.q, o.b, z, dk, s4);
    }
    add_dv(L.w, s4);
  }
  const int64_t at = head_off(a, n) + (int64_t)t * a.st + 8 * L.g;
  if (ok) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8];
      unpack8(dyo[s], x);  // Y = v + ...
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] += av[2 * s + (u >> 2)][u & 3];
      st_row<VEC>((bf16*)a.dv + at + 32 * s, pack8(x));
    }
  }

  // ---- dg: the reverse running sum of db = q dq - k dk, and what reaches every row through b_last
  float dg[NS][8];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int u = 0; u < 8; ++u) dg[s][u] = rscan16(o.q[s][u] * dq[s][u] - o.k[s][u] * dk[s][u]);
    if (L.i == 0) st8f(&pt[L.w][32 * s + 8 * L.g], dg[s]);
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int c0 = 32 * s + 8 * L.g;
    float lb[8], x[8];
    ld8f(lst + 32 * s + 8 * L.g, lb);
    ld8f(gm + c0, x);
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] *= fast_exp2(lb[u]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      float y[8];
      ld8f(&ex[w][c0], y);
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] += y[u];
    }
    for (int w = L.w + 1; w < 4; ++w) {
      float y[8];
      ld8f(&pt[w][c0], y);
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] += y[u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) dg[s][u] += x[u];
  }
  float* DG = a.dg + ((int64_t)n * a.T + t) * D + 8 * L.g;
  if (a.a_log) {
    // through the gate: dr = dg (-exp(A_log) sigmoid(r + dt_bias)) goes out in
    // place of dg; the chunk's sums of dg g and dr meet in LDS in a fixed order
    __syncthreads();  // pt and ex are read
    [[maybe_unused]] Gate<NS> again;
    if constexpr (!KEEP_G) gate_again<D, VEC>(a, n, t, ok, L, again);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float sa[8], sd[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        float gv, gd;
        if constexpr (KEEP_G) {
          gv = gate.g[s][u];
          gd = gate.d[s][u];
        } else {
          gv = again.g[s][u];
          gd = again.d[s][u];
        }
        sa[u] = group_sum<16>(dg[s][u] * gv);  // rows past the sequence have zeros in the gate
        dg[s][u] *= gd;
        sd[u] = group_sum<16>(dg[s][u]);
      }
      if (L.i == 0) {
        st8f(&pt[L.w][32 * s + 8 * L.g], sa);
        st8f(&ex[L.w][32 * s + 8 * L.g], sd);
      }
    }
    __syncthreads();
    if (tid < D) {
      float* P = a.gpart + ((int64_t)n * a.nchunks + c) * 2 * D;
      P[tid] = (pt[0][tid] + pt[1][tid]) + (pt[2][tid] + pt[3][tid]);
      P[D + tid] = (ex[0][tid] + ex[1][tid]) + (ex[2][tid] + ex[3][tid]);
    }
  }
  if (ok) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (VEC) {
        st8f(DG + 32 * s, dg[s]);
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) DG[32 * s + u] = dg[s][u];
      }
    }
  }

  // ---- back through the rotation
  if (a.rope) {
    const int tc = min(t, a.T - 1), h = a.rope_half;
    if (NS >= 2 && 2 * h == D) {
      rope_own<NS>(a, tc, L, dq, dk, true);
    } else {
      // the partner channels are on other lanes of the row, in the same wave:
      // through LDS (the region and VY hold two fp32 [64][D] arrays)
      __syncthreads();
      float* X1 = reinterpret_cast<float*>(R);
      float* X2 = X1 + kL * D;
      auto xi = [&](int cc) { return row * D + ((((cc >> 2) ^ (row & 7)) << 2) | (cc & 3)); };
      auto put4 = [&](float* X, int cc, const float* x) __attribute__((always_inline)) {  // to the partners' places
        if (h % 4 == 0) {
          *reinterpret_cast<floatx4*>(&X[xi(rope_partner(cc, h))]) = floatx4{x[0], x[1], x[2], x[3]};
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) X[xi(rope_partner(cc + u, h))] = x[u];
        }
      };
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int x = 0; x < 8; x += 4) {
          put4(X1, 32 * s + 8 * L.g + x, &dq[s][x]);
          put4(X2, 32 * s + 8 * L.g + x, &dk[s][x]);
        }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int c0 = 32 * s + 8 * L.g;
        float cs[8], sn[8];
        rope_cs(a, tc, c0, true, cs, sn);
#pragma unroll
        for (int x = 0; x < 8; x += 4) {
          const floatx4 y1 = *reinterpret_cast<const floatx4*>(&X1[xi(c0 + x)]);
          const floatx4 y2 = *reinterpret_cast<const floatx4*>(&X2[xi(c0 + x)]);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            dq[s][x + u] = __builtin_fmaf(y1[u], sn[x + u], dq[s][x + u] * cs[x + u]);
            dk[s][x + u] = __builtin_fmaf(y2[u], sn[x + u], dk[s][x + u] * cs[x + u]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // ---- through q = S ^p1, k = S ^p2, S = sigmoid(scale p1 . p2 / tau_S): the
  // rows once more, as S may be 0 and q and k then hold nothing of them
  {
    const unsigned off = (unsigned)min(t, a.T - 1) * (unsigned)a.st + 8u * L.g;
    const bf16 *P1 = (const bf16*)a.p1 + head_off(a, n), *P2 = (const bf16*)a.p2 + head_off(a, n);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      unpack8(ld_row<VEC>(P1 + (off + 32u * s)), o.q[s]);
      unpack8(ld_row<VEC>(P2 + (off + 32u * s)), o.k[s]);
    }
  }
  float h1 = 0.0f, h2 = 0.0f;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      h1 = __builtin_fmaf(o.q[s][u], dq[s][u], h1);
      h2 = __builtin_fmaf(o.k[s][u], dk[s][u], h2);
    }
  h1 = sum_groups(h1) * o.in1;  // ^p1 . dq
  h2 = sum_groups(h2) * o.in2;
  const float dU = (h1 + h2) * o.S * (1.0f - o.S) * a.scale * a.inv_tau;
  const float f1 = o.S * o.in1, f2 = o.S * o.in2;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float p1 = o.q[s][u], p2 = o.k[s][u];
      dq[s][u] = __builtin_fmaf(dU, p2, f1 * (dq[s][u] - p1 * o.in1 * h1));
      dk[s][u] = __builtin_fmaf(dU, p1, f2 * (dk[s][u] - p2 * o.in2 * h2));
    }
  if (ok) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      st_row<VEC>((bf16*)a.dp1 + at + 32 * s, pack8(dq[s]));
      st_row<VEC>((bf16*)a.dp2 + at + 32 * s, pack8(dk[s]));
    }
  }
  };
  // at D = 128 one path for all: two of them spill more (step of 32 heads x 128 x
  // 4096 887 -> 1085 us; at D = 64 two save 8 heads x 32K 2%)
  if (D == 128 || chunk_steep<D>(tot)) rest(std::true_type{});
  else rest(std::false_type{});
}

// The RoPE table of rope_cs: per channel (cos, sin) of t * base^(-2j/rope_dim),
// evaluated in fp64, for t at the chunk starts and the offsets inside a chunk.
// One workgroup per row, one thread per channel.
__global__ __launch_bounds__(128) void lin_rope_table_kernel(float2* tab, int nch, int h, double step) {
  const int row = blockIdx.x, c = threadIdx.x, W = blockDim.x;
  double sn = 0.0, cs = 1.0;
  if (c < 2 * h) {
    const double t = row < nch ? (double)row * kL : (double)(row - nch);
    sincos(t * exp((double)(c < h ? c : c - h) * step), &sn, &cs);
  }
  tab[(int64_t)row * W + c] = make_float2((float)cs, (float)sn);
}

hipError_t launch_scan(const LinearArgs& a, bool bwd, hipStream_t stream) {
  if (a.nseg == 1) return hipSuccess;
  const dim3 grid((unsigned)(a.D * a.D / (a.nseg <= 16 ? kNT : 64)), (unsigned)(a.B * a.H), bwd ? 2 : 1);
  hipLaunchKernelGGL(lin_scan_kernel, grid, dim3(kNT), 0, stream, a);
  return hipGetLastError();
}

template <int D, bool VEC>
hipError_t launch_fwd_d(const LinearArgs& a, hipStream_t stream) {
  const unsigned N = (unsigned)(a.B * a.H);
  hipLaunchKernelGGL((lin_state_kernel<D, false, VEC>), dim3((unsigned)a.nseg, N, D > 64 ? 2 : 1), dim3(kNT), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_scan(a, false, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((lin_out_kernel<D, VEC>), dim3((unsigned)a.nchunks, N), dim3(kNT), 0, stream, a);
  return hipGetLastError();
}

template <int D, bool VEC>
hipError_t launch_bwd_d(const LinearArgs& a, hipStream_t stream) {
  const unsigned N = (unsigned)(a.B * a.H);
  hipLaunchKernelGGL((lin_state_kernel<D, true, VEC>), dim3((unsigned)a.nseg, N, D > 64 ? 2 : 1), dim3(kNT), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_scan(a, true, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((lin_grad_kernel<D, VEC>), dim3((unsigned)a.nchunks, N), dim3(kNT), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

// Chunks per segment: long walks keep the per-segment states and the scan
// small, short ones keep the chip full (about two workgroups per CU).
int linear_bf16_segment(int64_t heads, int nchunks) {
  int s = kMaxSeg;
  while (s > 1 && (s / 2 >= nchunks || heads * ((nchunks + s - 1) / s) < 512)) s /= 2;
  return s;
}

// Which bf16 problems this file's kernels take; linear.hip's take the rest.
// Theirs share a chunk among more waves and scan up to 16 chunks a head in one
// launch; with few chunks in all that shorter chain is the whole time. The gate
// costs their width-128 backward a row pass, RoPE costs them barriers, and here
// RoPE over part of the width costs an exchange through LDS. Width 32 is
// faster here throughout. Measured with the gate (us per replayed graph of the
// call, linear.hip / this file; n/c: n chunks in all, c a head):
//   width 64 forward   10/5 20.4 / 20.9, 512/16 31.4 / 31.6, 1024/16 48.1 / 47.9, 36/18 23.3 / 21.6, 2/1 19.6 / 17.1
//     RoPE over 60     10/5 27.5 / 29.0, 1024/16 60.2 / 62.3, 36/18 30.6 / 29.9, 2/1 27.2 / 25.0; over 64 10/5 27.6 / 26.8
//   width 64 backward  36/18 40.3 / 38.7, 320/5 65.1 / 56.2; 128 and 256 chunks of up to 16 a head, with the forward and
//     not replayed, 48 / 52 and 51.6 / 55.9
//     RoPE over 60     10/5 45.2 / 48.9, 256/16 55.0 / 57.0, 36/18 50.8 / 49.8, 320/5 78.9 / 67.9, 2/1 44.7 / 41.1
//     over 64          64/8 46.1 / 45.3; channels that forget fast among them 20/5 48.7 / 51.1, 80/5 50.6 / 52.3,
//                      128/8 52.9 / 53.9, 128/2 55.4 / 53.0
//   width 128 forward  144/18 40.8 / 42.8, 64/32 34.0 / 36.2, 256/32 43.3 / 43.5, 288/18 64.4 / 56.1
//     RoPE over 80     10/5 35.5 / 38.9, 256/16 47.2 / 53.1, 144/18 49.7 / 53.0, 512/16 79.1 / 80.7, 64/1 47.1 / 32.1
//     over 128         256/16 49.4 / 51.1, 144/18 52.3 / 51.7
//   width 128 backward 64/2 80.7 / 87.3, 72/18 116.8 / 97.1, 256/16 without the gate 129 / 105
//     RoPE over 80     64/2 88.1 / 99.2, 64/16 96.9 / 106, 72/18 123 / 109, 64/1 86.6 / 69.9
bool linear_bf16_route(int64_t heads, int nchunks, int D, bool gated, int rope_dim, bool backward) {
  const int64_t chunks = heads * nchunks;
  const bool full = rope_dim == D, part = rope_dim > 0 && !full;
  const bool scan16 = nchunks > 1 && nchunks <= 16;  // linear.hip scans in one launch, and there is something to scan
  if (D == 32) return true;
  if (D == 128 && backward) return chunks > (!gated ? 160 : nchunks == 1 ? 32 : 64);
  if (D == 128) {
    if (chunks > 256) return true;
    if (nchunks <= 16) return nchunks == 1 && rope_dim > 0;
    return full || chunks > 160 || nchunks > 32;
  }
  if (!backward) return full || !scan16 || chunks > (part ? 1024 : 512);
  if (full) return nchunks <= 2 || nchunks > 8 || chunks > 80;
  if (part) return !scan16 || chunks > 256;
  return nchunks > 16 || chunks > 256;
}

int linear_bf16_rope_row(int rope_dim) { return rope_width(rope_dim / 2); }

hipError_t launch_linear_bf16_rope_table(float2* tab, int nchunks, int rope_dim, double base, hipStream_t stream) {
  const int h = rope_dim / 2;
  hipLaunchKernelGGL(lin_rope_table_kernel, dim3((unsigned)(nchunks + kL)), dim3((unsigned)rope_width(h)), 0, stream, tab,
                     nchunks, h, -2.0 / rope_dim * log(base));
  return hipGetLastError();
}

hipError_t launch_linear_bf16_fwd(const LinearArgs& a, hipStream_t stream) {
  switch (a.D) {
    case 32: return a.vec16 ? launch_fwd_d<32, true>(a, stream) : launch_fwd_d<32, false>(a, stream);
    case 64: return a.vec16 ? launch_fwd_d<64, true>(a, stream) : launch_fwd_d<64, false>(a, stream);
    case 128: return a.vec16 ? launch_fwd_d<128, true>(a, stream) : launch_fwd_d<128, false>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_linear_bf16_bwd(const LinearArgs& a, hipStream_t stream) {
  switch (a.D) {
    case 32: return a.vec16 ? launch_bwd_d<32, true>(a, stream) : launch_bwd_d<32, false>(a, stream);
    case 64: return a.vec16 ? launch_bwd_d<64, true>(a, stream) : launch_bwd_d<64, false>(a, stream);
    case 128: return a.vec16 ? launch_bwd_d<128, true>(a, stream) : launch_bwd_d<128, false>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rel
