// Decode step of the causal Full Relation operator: the one new row of every
// (b, h) against a KV cache, with the count correction at the token's absolute
// position i (eq. 2 with i = the cache length).
//
// The row is read-bound: every historical key and value is read once and used
// for one dot product and one weighted add. The history is split into slices
// of kSlice keys, one workgroup each, so that the chip has enough independent
// reads in flight; a workgroup leaves the Exchange scan state (m, l, z) of its
// slice (eq. 11). The merge kernel rescales the states of a row to their common
// maximum, adds them, and applies the epilogue of eqs. 12-13 with the Self
// entry (the token's own key and value, the last valid cache entry). The same
// merge serves a cache split over devices: each holds states of its shard.
//
// In the states kernel LPK lanes share one key: lane c of the group holds VEC
// channels of q (16 bytes of bf16 or fp32) and reads the same channels of the
// key and value rows; the dot product is finished by shuffles inside the group.
// Every lane group keeps its own running (m, l) and VEC channels of z, and the
// groups of a workgroup are merged at the end.
#include "kernels.h"
#include "lanes.h"

namespace rel {

namespace {

constexpr int kDT = 256;      // threads of the states kernel, and of the merge
constexpr int kDTFew = 1024;  // threads of the states kernel where workgroups are few
constexpr int kFewGroups = 512;
constexpr int kSlice = 256;   // keys per workgroup in relation_decode
constexpr int kUnroll = 2;    // keys per lane group whose loads are in flight together

template <typename TI, int VEC>
struct Row;

template <>
struct Row<bf16, 8> {
  static __device__ __forceinline__ void load(const bf16* p, float (&x)[8]) {
    const uintx4 u = *reinterpret_cast<const uintx4*>(p);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      x[2 * t] = bf16_lo(u[t]);
      x[2 * t + 1] = bf16_hi(u[t]);
    }
  }
};

template <>
struct Row<float, 4> {
  static __device__ __forceinline__ void load(const float* p, float (&x)[4]) {
    const float4 u = *reinterpret_cast<const float4*>(p);
    x[0] = u.x; x[1] = u.y; x[2] = u.z; x[3] = u.w;
  }
};

__device__ __forceinline__ float sigm(float x) { return fast_rcp(1.0f + fast_exp2(-x * kLog2e)); }

// The cache length of batch entry b, clamped to 1 .. Tmax so that every read
// stays inside the cache; the merge writes NaN for an entry outside that range.
__device__ __forceinline__ int clamp_len(const int32_t* lengths, int b, int Tmax) {
  const int n = lengths[b];
  return n < 1 ? 1 : (n > Tmax ? Tmax : n);
}
__device__ __forceinline__ bool len_valid(const int32_t* lengths, int b, int Tmax) {
  const int n = lengths[b];
  return n >= 1 && n <= Tmax;
}

// Merges state (mo, lo, zo) into (m, l, z); an empty state has m = -inf, l = 0.
template <int VEC>
__device__ __forceinline__ void merge_into(float& m, float& l, float (&z)[VEC], float mo, float lo,
                                           const float (&zo)[VEC]) {
  const float mn = fmaxf(m, mo);
  const float a = m == kNegInf ? 0.0f : fast_exp2((m - mn) * kLog2e);
  const float b = mo == kNegInf ? 0.0f : fast_exp2((mo - mn) * kLog2e);
  l = l * a + lo * b;
#pragma unroll
  for (int e = 0; e < VEC; ++e) z[e] = z[e] * a + zo[e] * b;
  m = mn;
}

// Exchange state of keys [j0, j1) of one (b, h) row, split into a.nsplit slices
// (grid: nsplit x B*H); keys at or after the row's own entry are never read.
//
// NT = kDT threads read a slice of 256 keys in several steps of the loop, which
// needs other workgroups on the CU to fill the waits. With fewer than
// kFewGroups workgroups (two per CU) NT = kDTFew: the same slice in one step or
// two. Whole steps (with the merge), 256 against 1024 threads: 9.3 and 8.4 us at
// 4 workgroups, 12.5 and 9.9 at 32 (D = 128), 17.4 and 13.0 at 256 (D = 128);
// 12.8 and 14.0 at 512 (D = 64), 15.4 and 20.2 at 768. (Four keys per lane
// group in flight instead of kUnroll: 139 -> 182 us at 12288 workgroups.)
template <typename TI, int VEC, int LPK, int NT>
__global__ __launch_bounds__(NT) void decode_states_kernel(DecodeArgs a) {
  constexpr int KPW = 64 / LPK;          // keys per wave and step
  constexpr int NW = NT / 64;
  __shared__ float red[NW][2 + 128];
  const int slice = blockIdx.x;
  const int n = blockIdx.y;              // b * H + h
  const int b = n / a.H, h = n % a.H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = lane % LPK, kg = lane / LPK;
  const int c0 = c * VEC;
  const bool chan = c0 < a.D;
  const int len = clamp_len(a.lengths, b, a.Tmax);
  const int hist_end = min(a.key1, len - 1);      // Exchange keys only: j < i - 1 (zero-based)
  const int span = a.key1 - a.key0;
  const int per = (span + a.nsplit - 1) / a.nsplit;
  const int s0 = a.key0 + slice * per;
  const int s1 = min(s0 + per, hist_end);

  float q[VEC];
  const TI* qrow = (const TI*)a.q + (int64_t)n * a.D;
#pragma unroll
  for (int e = 0; e < VEC; ++e) q[e] = 0.0f;
  if (chan) Row<TI, VEC>::load(qrow + c0, q);
  const int64_t hoff = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const TI* K = (const TI*)a.k + hoff;
  const TI* V = (const TI*)a.v + hoff;

  float m = kNegInf, l = 0.0f, z[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) z[e] = 0.0f;
  // kUnroll keys per lane group in flight: j = s0 + (kUnroll (it NW + w) + u) KPW + kg.
  // The loop runs on a wave-uniform base, so every lane reaches the shuffles.
  for (int base = s0 + kUnroll * w * KPW; base < s1; base += kUnroll * NW * KPW) {
    float kx[kUnroll][VEC], vx[kUnroll][VEC];
    bool ok[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int j = base + u * KPW + kg;
      ok[u] = j < s1;
#pragma unroll
      for (int e = 0; e < VEC; ++e) kx[u][e] = vx[u][e] = 0.0f;
      if (ok[u] && chan) {
        Row<TI, VEC>::load(K + (int64_t)j * a.st + c0, kx[u]);
        Row<TI, VEC>::load(V + (int64_t)j * a.st + c0, vx[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      float d = 0.0f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) d = __builtin_fmaf(q[e], kx[u][e], d);
      d = lane_group_sum<LPK>(d);
      if (ok[u]) {
        const float uu = d * a.scale;
        const float E = uu * sigm(uu);             // Exchange map, eq. (2)
        const float mn = fmaxf(m, E);
        const float cr = m == kNegInf ? 0.0f : fast_exp2((m - mn) * kLog2e);
        const float p = fast_exp2((E - mn) * kLog2e);
        l = l * cr + p;
#pragma unroll
        for (int e = 0; e < VEC; ++e) z[e] = __builtin_fmaf(p, vx[u][e], z[e] * cr);
        m = mn;
      }
    }
  }
  // merge the lane groups of a wave (lanes with equal c hold the same channels)
  auto merge_groups = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int o = LPK; o < 64; o <<= 1) {
      float zo[VEC];
      const float mo = __shfl_xor(m, o, 64), lo = __shfl_xor(l, o, 64);
#pragma unroll
      for (int e = 0; e < VEC; ++e) zo[e] = __shfl_xor(z[e], o, 64);
      merge_into<VEC>(m, l, z, mo, lo, zo);
    }
  };
  merge_groups();
  // then the waves, in a fixed order: group kg of the first wave takes waves kg, kg + KPW, ...
  if (kg == 0) {
    if (c == 0) {
      red[w][0] = m;
      red[w][1] = l;
    }
    if (chan) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) red[w][2 + c0 + e] = z[e];
    }
  }
  __syncthreads();
  if (w != 0) return;
  m = kNegInf;
  l = 0.0f;
#pragma unroll
  for (int e = 0; e < VEC; ++e) z[e] = 0.0f;
  for (int ow = kg; ow < NW; ow += KPW) {
    float zo[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) zo[e] = chan ? red[ow][2 + c0 + e] : 0.0f;
    merge_into<VEC>(m, l, z, red[ow][0], red[ow][1], zo);
  }
  merge_groups();
  if (kg == 0) {
    float* st = a.states + ((int64_t)slice * a.B * a.H + n) * (a.D + 2);
    if (c == 0) {
      st[0] = m;
      st[1] = l;
    }
    if (chan) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) st[2 + c0 + e] = z[e];
    }
  }
}

// One workgroup per (b, h) row: merge the row's a.nstates states, then Self
// and the count correction (eqs. 12-13) at i = the row's cache length. A lane
// holds a channel pair and G lanes a state, so that a state is read as one run
// of memory; lane group g takes the states g, g + kDT / G, ..., kBatch of them in
// flight, against its own running maximum, and the groups meet in LDS. Bound
// by latency: one round of reads for up to kBatch kDT / G states (64 at D = 64).
// With lanes over states and 32 channels each, whose sums met in 192 shuffles,
// the step took 12.6 us for 16 rows of 16 states and 34.6 us for 16 of 128;
// it takes 10.0 and 31.1 (256 threads in the states kernel).
template <typename TI, int G>
__global__ __launch_bounds__(kDT) void decode_merge_kernel(DecodeArgs a) {
  constexpr int NG = kDT / G, kBatch = 8;
  __shared__ float mls[NG][2];
  __shared__ float zsh[NG][2 * G];
  const int n = blockIdx.x;  // b * H + h
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int b = n / a.H, h = n % a.H;
  const int len = clamp_len(a.lengths, b, a.Tmax);
  const int64_t stride_s = (int64_t)a.B * a.H * (a.D + 2);
  const float* st0 = a.states + (int64_t)n * (a.D + 2);
  // the Self entry's reads first (the first wave), so that they overlap the states' reads
  const int64_t selfrow = (int64_t)b * a.sb + (int64_t)h * a.sh + (int64_t)(len - 1) * a.st;
  const TI* q = (const TI*)a.q + (int64_t)n * a.D;
  float d = 0.0f, vi0 = 0.0f, vi1 = 0.0f;
  if (w == 0) {
    if (lane < a.D) {
      d = Elem<TI>::load(q + lane) * Elem<TI>::load((const TI*)a.k + selfrow + lane);
      vi0 = Elem<TI>::load((const TI*)a.v + selfrow + lane);
    }
    if (lane + 64 < a.D) {
      d += Elem<TI>::load(q + lane + 64) * Elem<TI>::load((const TI*)a.k + selfrow + lane + 64);
      vi1 = Elem<TI>::load((const TI*)a.v + selfrow + lane + 64);
    }
  }
  const int grp = tid / G, c0 = 2 * (tid % G);
  const int cz = c0 < a.D ? c0 : 0;  // lanes past the width repeat the first pair; nobody reads theirs
  float m = kNegInf, l = 0.0f, z[2] = {0.0f, 0.0f};
  for (int s0 = grp; s0 < a.nstates; s0 += NG * kBatch) {
    float2 ml[kBatch], zz[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {  // slots past the end read the last state and count for nothing
      const float* st = st0 + min(s0 + k * NG, a.nstates - 1) * stride_s;
      ml[k] = *reinterpret_cast<const float2*>(st);  // 8-byte aligned: D + 2 and c0 even
      zz[k] = *reinterpret_cast<const float2*>(st + 2 + cz);
    }
    float mn = m;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      if (s0 + k * NG >= a.nstates) {
        ml[k] = float2{kNegInf, 0.0f};
        zz[k] = float2{0.0f, 0.0f};
      }
      mn = fmaxf(mn, ml[k].x);
    }
    const float f0 = m == kNegInf ? 0.0f : fast_exp2((m - mn) * kLog2e);
    l *= f0;
    z[0] *= f0;
    z[1] *= f0;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const float f = ml[k].x == kNegInf ? 0.0f : fast_exp2((ml[k].x - mn) * kLog2e);
      l = __builtin_fmaf(ml[k].y, f, l);
      z[0] = __builtin_fmaf(zz[k].x, f, z[0]);
      z[1] = __builtin_fmaf(zz[k].y, f, z[1]);
    }
    m = mn;
  }
  if (c0 == 0) {
    mls[grp][0] = m;
    mls[grp][1] = l;
  }
  *reinterpret_cast<float2*>(&zsh[grp][c0]) = float2{z[0], z[1]};
  __syncthreads();
  if (w != 0) return;  // the first wave finishes the row
  m = kNegInf;
#pragma unroll
  for (int x = 0; x < NG; ++x) m = fmaxf(m, mls[x][0]);
  l = 0.0f;
  float z0 = 0.0f, z1 = 0.0f;
#pragma unroll
  for (int x = 0; x < NG; ++x) {
    const float mx = mls[x][0], f = mx == kNegInf ? 0.0f : fast_exp2((mx - m) * kLog2e);
    l = __builtin_fmaf(mls[x][1], f, l);
    z0 = __builtin_fmaf(zsh[x][lane], f, z0);
    if (G > 32) z1 = __builtin_fmaf(zsh[x][64 + lane], f, z1);
  }
  // Self: U_ii = scale q . k_i, S = sigmoid(U_ii / tau_S)
  for (int o = 32; o >= 1; o >>= 1) d += __shfl_xor(d, o, 64);
  const float S = 1.0f / (1.0f + expf(-d * a.scale * a.inv_tau));
  const float ln_i = logf((float)len);
  const float lam = *a.lambda;
  float g = 0.0f, omg = 1.0f, zr0 = 0.0f, zr1 = 0.0f, lnZ = S;
  if (l > 0.0f) {
    const float A = m + logf(l) - lam * ln_i;       // A_i = L^E_i - lambda ln i (eq. 5)
    g = 1.0f / (1.0f + expf(S - A));                // g = sigmoid(A - S)
    omg = 1.0f / (1.0f + expf(A - S));              // 1 - g = sigmoid(S - A)
    const float il = 1.0f / l;
    zr0 = z0 * il;
    zr1 = z1 * il;
    lnZ = fmaxf(S, A) + log1pf(expf(-fabsf(S - A)));
  }
  // an entry whose cache length lies outside 1 .. Tmax gets NaN: the error is
  // visible in the output instead of a result at a clamped position
  const bool valid = len_valid(a.lengths, b, a.Tmax);
  const float nan = __builtin_nanf("");
  TI* o = (TI*)a.out + (int64_t)n * a.D;
  if (lane < a.D) Elem<TI>::store(o + lane, valid ? omg * vi0 + g * zr0 : nan);
  if (lane + 64 < a.D) Elem<TI>::store(o + lane + 64, valid ? omg * vi1 + g * zr1 : nan);
  if (lane == 0 && a.row_stat) a.row_stat[n] = valid ? lnZ + lam * ln_i : nan;
}

template <typename TI, int VEC, int LPK>
void launch_states_l(const DecodeArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)a.nsplit, (unsigned)(a.B * a.H));
  if ((int64_t)a.nsplit * a.B * a.H < kFewGroups)
    hipLaunchKernelGGL((decode_states_kernel<TI, VEC, LPK, kDTFew>), grid, dim3(kDTFew), 0, stream, a);
  else
    hipLaunchKernelGGL((decode_states_kernel<TI, VEC, LPK, kDT>), grid, dim3(kDT), 0, stream, a);
}

template <typename TI, int VEC>
hipError_t launch_states_t(const DecodeArgs& a, hipStream_t stream) {
  const int lanes = (a.D + VEC - 1) / VEC;
  if (lanes <= 4)
    launch_states_l<TI, VEC, 4>(a, stream);
  else if (lanes <= 8)
    launch_states_l<TI, VEC, 8>(a, stream);
  else if (lanes <= 16)
    launch_states_l<TI, VEC, 16>(a, stream);
  else
    launch_states_l<TI, VEC, 32>(a, stream);
  return hipGetLastError();
}

template <typename TI>
hipError_t launch_merge_t(const DecodeArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)(a.B * a.H));
  if (a.D <= 64)
    hipLaunchKernelGGL((decode_merge_kernel<TI, 32>), grid, dim3(kDT), 0, stream, a);
  else
    hipLaunchKernelGGL((decode_merge_kernel<TI, 64>), grid, dim3(kDT), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

int decode_slice_keys() { return kSlice; }

hipError_t launch_decode_states(const DecodeArgs& a, int dtype, hipStream_t stream) {
  return dtype == 1 ? launch_states_t<bf16, 8>(a, stream) : launch_states_t<float, 4>(a, stream);
}

hipError_t launch_decode_merge(const DecodeArgs& a, int dtype, hipStream_t stream) {
  return dtype == 1 ? launch_merge_t<bf16>(a, stream) : launch_merge_t<float>(a, stream);
}

}  // namespace rel
