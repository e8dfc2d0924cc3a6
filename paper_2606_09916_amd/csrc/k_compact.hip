// The compact apply path (Sec. 3.4: the standard compactors left-pack the kept rows
// and re-index RoPE; the Appendix layout ablation, Table 7, compares it with the
// dead-slot redirect). The t-th kept position j of a session moves to position t and
// to the caller's destination slot dst[t]: on every layer and KV head its key is
// re-rotated by t - j (Neox rotate-half: channel pair (i, i + D/2) turns by
// (t - j) * base^(-2i/D)) and its value copied.
//
//   k_compact_list  the kept positions in position order, and their count: a workgroup
//                   per span of positions counts the kept ones before it and lists its
//                   own (ballot prefix sums over 1024-position rounds);
//   k_compact_copy  a workgroup per kept index: the pair angles in float64 (they
//                   reach 1e5 radians at long distances), cos / sin in LDS, then every
//                   layer's key rows rotated in float32 and rounded once to the pool's
//                   type, value rows copied.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "ikv_internal.hpp"

namespace ikv {

constexpr int CL_THREADS = 1024;
constexpr int CL_WGS = 64;                       // workgroups per session at most
// One workgroup per session walked its rounds one after the other, a memory round trip and
// three barriers each: 47 to 56 us at 32,768 positions. Counting again what lies before the
// span costs a workgroup one sweep with CL_U loads in flight and needs no exchange.
constexpr int CL_U = 8;

__global__ void __launch_bounds__(CL_THREADS) k_compact_list(const ikv_session *__restrict__ sess,
                                                             const int32_t *__restrict__ slot_maps, int dead,
                                                             const uint8_t *__restrict__ keep,
                                                             int32_t *__restrict__ pos_list,
                                                             int32_t *__restrict__ n_keep, int span) {
  constexpr int NW = CL_THREADS / WAVE;
  __shared__ int wsum[NW];
  const int b = blockIdx.y;
  const ikv_session s = sess[b];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int p0 = int(blockIdx.x) * span, p1 = min(s.N, p0 + span);
  if (p0 >= s.N && p0 > 0) return;
  const int32_t *S = slot_maps + s.slot_off;
  const uint8_t *kp = keep + s.slot_off;
  int base = 0;
  if (p0 > 0) {
    int n = 0;
    for (int j0 = t; j0 < p0; j0 += CL_U * CL_THREADS) {
      int sv[CL_U];
      uint8_t kv[CL_U];
#pragma unroll
      for (int q = 0; q < CL_U; ++q) {
        const int j = min(j0 + q * CL_THREADS, p0 - 1);
        sv[q] = S[j];
        kv[q] = kp[j];
      }
#pragma unroll
      for (int q = 0; q < CL_U; ++q) n += j0 + q * CL_THREADS < p0 && kv[q] && sv[q] != dead;
    }
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) n += __shfl_xor(n, o, WAVE);
    if (lane == 0) wsum[w] = n;
    __syncthreads();
    for (int q = 0; q < NW; ++q) base += wsum[q];
    __syncthreads();
  }
  for (int j0 = p0; j0 < p1; j0 += CL_THREADS) {
    const int j = j0 + t;
    const bool k = j < p1 && kp[j] && S[j] != dead;
    const uint64_t m = __ballot(k);
    const int below = __popcll(m & ((uint64_t(1) << lane) - 1));
    if (lane == 0) wsum[w] = __popcll(m);
    __syncthreads();
    int off = base;
    for (int q = 0; q < w; ++q) off += wsum[q];
    if (k) pos_list[s.slot_off + off + below] = j;
    for (int q = 0; q < NW; ++q) base += wsum[q];
    __syncthreads();
  }
  if (t == 0 && p1 == s.N) n_keep[b] = base;
}

constexpr int CC_THREADS = 256;

// 16 bytes of a row: eight channels (bf16) or four (float32). Every row is read once and
// with the non-temporal hint; stores round to the pool's type (nearest even for bf16).
typedef unsigned int cc_u32x4 __attribute__((ext_vector_type(4)));
template <typename T> constexpr int CC_PP = 16 / int(sizeof(T));   // channel pairs per thread per step

__device__ __forceinline__ cc_u32x4 cc_ld(const void *p) {
  return __builtin_nontemporal_load(reinterpret_cast<const cc_u32x4 *>(p));
}
__device__ __forceinline__ void cc_st(void *p, cc_u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<cc_u32x4 *>(p));
}
__device__ __forceinline__ void cc_unpack(cc_u32x4 v, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __uint_as_float(v[i] << 16);
    x[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void cc_unpack(cc_u32x4 v, float (&x)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(v[i]);
}
__device__ __forceinline__ cc_u32x4 cc_pack(const float (&y)[8]) {
  cc_u32x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] = uint32_t(float_to_bf16_bits(y[2 * i])) | (uint32_t(float_to_bf16_bits(y[2 * i + 1])) << 16);
  return v;
}
__device__ __forceinline__ cc_u32x4 cc_pack(const float (&y)[4]) {
  cc_u32x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(y[i]);
  return v;
}

// A workgroup walks kept indices blockIdx.x, + gridDim.x, ... The registers hold three (bf16)
// or four (float32) workgroups per CU, 768 or 1024 on the chip; the hardware hands out the
// rest as they end. CC_WGS bounds the workgroups that come only to find no index, and is large
// enough to balance: 36 layers of 8 KV heads, 8192 of 32,768 kept, 471 us with 512, 472 with
// 1536 and 4096, 461 with 8192 and with one per position; 48 layers of 4, 16,000 of 60,000,
// 640, 632, 624 and 625 with 512, 4096, 8192 and one per position. U steps of 16-byte loads
// are in flight per thread, and the first are issued before the angles, whose float64 pow, cos
// and sin take about as long as a memory round trip.
constexpr int CC_WGS = 8192;

// Steps in flight (one, two or three) and threads of a workgroup, for the `steps` of an index
// (a step: 16 bytes of each half of a key row and of a value row): no more in flight than
// there are, and every turn about full. Lanes past the last step read its rows again. With
// three steps of 256 threads whatever the count, one layer of 2 KV heads (16 steps; 32
// sessions, 2000 of 8000 kept) took 290 us, 75 like this; two layers of 8 (128 steps) 330 and
// 171; from 36 layers of 8 (2304 steps) on the two are the same.
struct CopyShape {
  int u, threads;
};
inline CopyShape copy_shape(int64_t steps) {
  const int u = steps <= CC_THREADS ? 1 : steps <= 2 * CC_THREADS ? 2 : 3;
  const int64_t turns = cdiv(steps, u * CC_THREADS);
  return {u, int(cdiv(cdiv(steps, turns * u), WAVE)) * WAVE};
}

template <typename T, int U>
__global__ void __launch_bounds__(CC_THREADS) k_compact_copy(const ikv_session *__restrict__ sess, T *__restrict__ kp,
                                                             T *__restrict__ vp, int64_t num_slots, int L, int Hkv,
                                                             int D, const int32_t *__restrict__ slot_maps,
                                                             const int32_t *__restrict__ dst,
                                                             const int32_t *__restrict__ pos_list,
                                                             const int32_t *__restrict__ n_keep, double base) {
  constexpr int PP = CC_PP<T>;
  __shared__ __align__(16) float cs[64], sn[64];
  const int b = blockIdx.y;
  const ikv_session s = sess[b];
  const int h = D / 2, t = threadIdx.x, nt = blockDim.x;
  const int nk = n_keep[b];
  const int64_t row = int64_t(Hkv) * D;          // elements of one slot in one layer
  const int per = h / PP, groups = Hkv * per;    // pair groups per head and per layer
  const int steps = L * groups;
  for (int tk = blockIdx.x; tk < nk; tk += gridDim.x) {
    const int j = pos_list[s.slot_off + tk];
    const int64_t src = slot_maps[s.slot_off + j], dslot = dst[s.slot_off + tk];
    cc_u32x4 k1[U], k2[U], v1[U], v2[U];
    int64_t od[U];
    int q[U];
    // steps past the last are clamped: they read its rows again and store nothing
    auto load = [&](int g0) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = min(g0 + u * nt, steps - 1);
        const int l = g / groups, r = g - l * groups;
        const int hd = r / per;
        q[u] = (r - hd * per) * PP;
        const int64_t in = int64_t(hd) * D + q[u];
        const int64_t os = (int64_t(l) * num_slots + src) * row + in;
        od[u] = (int64_t(l) * num_slots + dslot) * row + in;
        k1[u] = cc_ld(kp + os);
        k2[u] = cc_ld(kp + os + h);
        v1[u] = cc_ld(vp + os);
        v2[u] = cc_ld(vp + os + h);
      }
    };
    load(t);
    if (t < h) {
      const double ang = double(tk - j) * pow(base, -2.0 * double(t) / double(D));
      cs[t] = float(cos(ang));
      sn[t] = float(sin(ang));
    }
    __syncthreads();
    for (int g0 = t;;) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (g0 + u * nt >= steps) continue;
        float x1[PP], x2[PP], y1[PP], y2[PP];
        cc_unpack(k1[u], x1);
        cc_unpack(k2[u], x2);
#pragma unroll
        for (int e = 0; e < PP; ++e) {
          const float c = cs[q[u] + e], sv = sn[q[u] + e];
          y1[e] = x1[e] * c - x2[e] * sv;
          y2[e] = x2[e] * c + x1[e] * sv;
        }
        cc_st(kp + od[u], cc_pack(y1));
        cc_st(kp + od[u] + h, cc_pack(y2));
        cc_st(vp + od[u], v1[u]);
        cc_st(vp + od[u] + h, v2[u]);
      }
      g0 += U * nt;
      if (g0 >= steps) break;
      load(g0);
    }
    __syncthreads();                             // the angles are read: the next index may write its own
  }
}

hipError_t launch_compact(const ikv_pool &pool, const ikv_session *sess_dev, int B, int maxN,
                          const int32_t *slot_maps, const uint8_t *keep, const int32_t *dst, double base,
                          int32_t *n_keep, int32_t *pos_list, hipStream_t st) {
  {
    KTimer kt_("k_compact_list", st);
    const int span = int(cdiv(maxN > 0 ? maxN : 1, int64_t(CL_THREADS) * CL_WGS)) * CL_THREADS;
    k_compact_list<<<dim3(unsigned(cdiv(maxN > 0 ? maxN : 1, span)), B), CL_THREADS, 0, st>>>(
        sess_dev, slot_maps, pool.dead_slot, keep, pos_list, n_keep, span);
  }
  if (maxN > 0) {
    KTimer kt_("k_compact_copy", st);
    const dim3 grid(unsigned(std::min(maxN, CC_WGS)), B);
    const bool bf = pool.kv_dtype == IKV_BF16;
    const CopyShape c = copy_shape(int64_t(pool.L) * pool.Hkv * (pool.D / 2 / (bf ? CC_PP<uint16_t> : CC_PP<float>)));
    auto run = [&](auto kernel, auto *kp, auto *vp) {
      kernel<<<grid, c.threads, 0, st>>>(sess_dev, kp, vp, pool.num_slots, pool.L, pool.Hkv, pool.D, slot_maps, dst,
                                         pos_list, n_keep, base);
    };
    auto pick = [&](auto *kp, auto *vp) {
      using T = std::remove_pointer_t<decltype(kp)>;
      if (c.u == 1) run(k_compact_copy<T, 1>, kp, vp);
      else if (c.u == 2) run(k_compact_copy<T, 2>, kp, vp);
      else run(k_compact_copy<T, 3>, kp, vp);
    };
    if (bf) pick(static_cast<uint16_t *>(pool.k_pool), static_cast<uint16_t *>(pool.v_pool));
    else pick(static_cast<float *>(pool.k_pool), static_cast<float *>(pool.v_pool));
  }
  return hipGetLastError();
}

}  // namespace ikv
