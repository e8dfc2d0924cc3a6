// Residual head of Eq. 4 with the features of Eq. 5 and the cross-attention of Eq. 6:
//   phi_j = [kbar_j, mbar, kbar_j * mbar, rule_j]
//   c_j   = 4-head attention (width 128, head width 32) of W_Q phi_j + b_Q over the
//           keys W_K kq + b_K and values W_V kq + b_V, kq = kbar at the live query
//           positions; c_j = 0 when the ablation flag is set or no query position is live
//   s_j   = rule_j + clip(alpha, -5, 5) * (w_2 . GELU(W_1 [phi_j ; c_j] + b_1) + b_2)
// All arithmetic is float32. The rule scores arrive in `scores` and are overwritten.
#include <math.h>

#include <type_traits>

#include "ikv_internal.hpp"
#include "res_setup.hpp"

namespace ikv {

int64_t residual_floats(int D) { return ResLayout(D).total; }

__global__ void __launch_bounds__(256) k_res_transpose(const float *__restrict__ blob, float *__restrict__ shared,
                                                       int D) {
  res_transpose_item(int64_t(blockIdx.x) * 256 + threadIdx.x, blob, shared, D);
}

// Per session: mbar and the live query positions (res_setup_body), one workgroup each.
template <int D>
__global__ void __launch_bounds__(256) k_res_setup(const ikv_session *__restrict__ sess,
                                                   const int32_t *__restrict__ slot_maps,
                                                   const int32_t *__restrict__ qpos, int dead, float *__restrict__ ws,
                                                   int L, int Hkv, bool mfma, bool pairs) {
  res_setup_body<D>(sess, int(blockIdx.x), slot_maps, qpos, dead, ws, L, Hkv, mfma, pairs);
}

// kq on the matrix-core path, where the second pass keeps kbar at the candidates only
// (a live query position in the query span is never one): row i of the kq block is the
// mean over the L Hkv units of the bf16 key row of the i-th live query position, summed
// layer-major in float32 and scaled by 1 / (L Hkv) as the second pass does. One
// workgroup per live row, thread = channel.
template <int D>
__global__ void __launch_bounds__(D) k_res_kq(const ikv_session *__restrict__ sess, const uint16_t *__restrict__ kpool,
                                              int64_t num_slots, int L, int Hkv,
                                              const int32_t *__restrict__ slot_maps, float *__restrict__ ws) {
  const int b = blockIdx.y;
  const ikv_session s = sess[b];
  if (s.N <= s.C) return;
  const int units = L * Hkv;
  const ScoreSizes z = score_sizes(s, L, units, D, true, true);
  float *base = ws + score_offset(sess, b, L, units, D, true, true);
  const int n = reinterpret_cast<const int *>(base + z.off_misc() + int64_t(MBAR_PARTS) * D)[D];
  const int i = blockIdx.x;
  if (i >= n) return;
  const int q = reinterpret_cast<const int *>(base + z.off_qlist())[i];
  const int64_t slot = slot_maps[s.slot_off + q];
  const int d = threadIdx.x;
  float a = 0.f;
  for (int u = 0; u < units; ++u) {
    const int l = u / Hkv, h = u - l * Hkv;
    a += bf16_bits_to_float(kpool[((int64_t(l) * num_slots + slot) * Hkv + h) * D + d]);
  }
  base[z.off_kq() + int64_t(i) * D + d] = a * (1.0f / float(units));
}

// K' = W_K kq + b_K and V' = W_V kq + b_V for four live query rows per workgroup,
// kq = kbar at the live query positions (from the second pass; on the matrix-core path
// the kq block of k_res_kq, row i for the i-th live row).
template <int D>
__device__ __forceinline__ void res_kv_body(int bx, const ikv_session *__restrict__ sess, const float *__restrict__ blob,
                                            float *__restrict__ ws, int L, int Hkv, bool mfma) {
  const int b = blockIdx.y;
  const ikv_session s = sess[b];
  if (s.N <= s.C) return;
  const int units = L * Hkv;
  const ResLayout lay(D);
  const ScoreSizes z = score_sizes(s, L, units, D, true, mfma);
  float *base = ws + score_offset(sess, b, L, units, D, true, mfma);
  const float *kbar = base + (mfma ? z.off_kq() : z.off_kbar());
  float *kp = base + z.off_kp();
  float *vp = base + z.off_vp();
  const int n = reinterpret_cast<const int *>(base + z.off_misc() + int64_t(MBAR_PARTS) * D)[D];
  const int *qlist = reinterpret_cast<const int *>(base + z.off_qlist());
  const int i0 = bx * 4;
  if (i0 >= n) return;
  __shared__ float kq[4][D];
  const int t = threadIdx.x;
  for (int e = t; e < 4 * D; e += 256) {
    const int r = e / D, d = e - r * D;
    const int i = min(i0 + r, n - 1);                  // a live row stands in past n
    const float v = kbar[int64_t(mfma ? i : qlist[i]) * D + d];
    kq[r][d] = (i0 + r < n) ? v : 0.f;
  }
  __syncthreads();
  const int o = t & (HC - 1);
  const bool isv = t >= HC;
  const float *W = blob + (isv ? lay.WV : lay.WK) + int64_t(o) * D;
  const float bias = blob[(isv ? lay.bV : lay.bK) + o];
  float a[4] = {bias, bias, bias, bias};
  constexpr int WB = 64;                              // weights in flight per thread
#pragma unroll 1
  for (int d0 = 0; d0 < D; d0 += WB) {
    float wv[WB];
#pragma unroll
    for (int d = 0; d < WB; ++d) wv[d] = W[d0 + d];
#pragma unroll
    for (int d = 0; d < WB; ++d)
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = fmaf(wv[d], kq[r][d0 + d], a[r]);
  }
  float *dst = isv ? vp : kp;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (i0 + r < n) dst[int64_t(i0 + r) * HC + o] = a[r];
}

template <int D>
__global__ void __launch_bounds__(256) k_res_kv(const ikv_session *__restrict__ sess, const float *__restrict__ blob,
                                                float *__restrict__ ws, int L, int Hkv, bool mfma) {
  res_kv_body<D>(int(blockIdx.x), sess, blob, ws, L, Hkv, mfma);
}

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// A workgroup takes TK candidates; every output's weights stream past them once, WB loads
// in flight per thread (one at a time, the loop waited out an L2 round trip per weight). 32
// candidates read the weights least often; few candidates take 8 or 16 each, so that their
// workgroups reach every CU. D = 64, 2016 candidates: 164 us at 32 without the batched
// loads, 63 workgroups. A candidate's sums have the same order at every TK.
template <int D, int TK>
__global__ void __launch_bounds__(256) k_residual(const ikv_session *__restrict__ sess,
                                                  const int32_t *__restrict__ slot_maps, int dead,
                                                  float *__restrict__ scores, const float *__restrict__ ws,
                                                  const float *__restrict__ shared, const float *__restrict__ blob,
                                                  int L, int Hkv, bool xattn, bool mfma) {
  constexpr int F = 3 * D + 1;
  constexpr int X = F + HC;
  constexpr int KC = 32;       // query keys per LDS chunk
  constexpr int WB = 16;       // weights in flight per thread
  __shared__ float xT[X][TK];          // [phi ; c] transposed: xT[i][k]
  __shared__ float ql[TK][HC + 4];     // W_Q phi + b_Q
  __shared__ float kvl[2][KC][HC];     // K', V' chunk
  __shared__ float red[4][TK];
  __shared__ int pos[TK];
  __shared__ int any;

  const int b = blockIdx.y;
  const ikv_session s = sess[b];
  if (s.N <= s.C) return;
  const int j0 = blockIdx.x * TK;
  if (j0 >= s.N) return;
  const int units = L * Hkv;
  const ResLayout lay(D);
  const ScoreSizes z = score_sizes(s, L, units, D, true, mfma);
  const float *base = ws + score_offset(sess, b, L, units, D, true, mfma);
  const float *kbar = base + z.off_kbar();
  const float *kp = base + z.off_kp();
  const float *vp = base + z.off_vp();
  const float *mbar = base + z.off_misc() + int64_t(MBAR_PARTS) * D;
  const int nql = reinterpret_cast<const int *>(mbar)[D];
  const float *wqT = shared;
  const float *w1T = shared + align64f(int64_t(F) * HC);
  float *out = scores + s.slot_off;
  const int t = threadIdx.x;

  if (t == 0) any = 0;
  __syncthreads();
  if (t < TK) {
    const int j = j0 + t;
    bool c = false;
    if (j < s.N) {
      const int slot = slot_maps[s.slot_off + j];
      c = slot != dead && !(j < s.pi || (j >= s.qs && j < s.qe));
    }
    pos[t] = c ? j : -1;
    if (c) atomicOr(&any, 1);
  }
  __syncthreads();
  if (!any) return;

  // phi
  for (int e = t; e < TK * F; e += 256) {
    const int i = e / TK, k = e - i * TK;
    const int j = pos[k];
    float v = 0.f;
    if (j >= 0) {
      if (i < D) v = kbar[int64_t(j) * D + i];
      else if (i < 2 * D) v = mbar[i - D];
      else if (i < 3 * D) v = kbar[int64_t(j) * D + (i - 2 * D)] * mbar[i - 2 * D];
      else v = out[j];
    }
    xT[i][k] = v;
  }
  __syncthreads();

  // acc[k] += sum over i < n of w[i * stride] * xT[i][k0 + k], i in order
  auto gemv = [&](auto &acc, const float *w, int64_t stride, int n, int k0) __attribute__((always_inline)) {
    constexpr int NK = sizeof(acc) / sizeof(float);
    auto add = [&](float wv, int i) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NK; k += 4) {
        const float4 xv = *reinterpret_cast<const float4 *>(&xT[i][k0 + k]);
        acc[k] = fmaf(xv.x, wv, acc[k]);
        acc[k + 1] = fmaf(xv.y, wv, acc[k + 1]);
        acc[k + 2] = fmaf(xv.z, wv, acc[k + 2]);
        acc[k + 3] = fmaf(xv.w, wv, acc[k + 3]);
      }
    };
    const int nb = n / WB * WB;
    float wv[WB];
#pragma unroll
    for (int q = 0; q < WB; ++q) wv[q] = w[q * stride];   // n >= 2 WB
    for (int i = 0; i < nb; i += WB) {
      float wn[WB];                                // the next batch, before this one is used
      const int in = min(i + WB, nb - WB);
#pragma unroll
      for (int q = 0; q < WB; ++q) wn[q] = w[(in + q) * stride];
#pragma unroll
      for (int q = 0; q < WB; ++q) add(wv[q], i + q);
#pragma unroll
      for (int q = 0; q < WB; ++q) wv[q] = wn[q];
    }
    for (int i = nb; i < n; ++i) add(w[i * stride], i);
  };

  // Q = W_Q phi + b_Q : thread -> output o, half of the candidates
  {
    constexpr int NK = TK / 2;
    const int o = t & (HC - 1), k0 = (t >> 7) * NK;
    float acc[NK];
    const float bq = blob[lay.bQ + o];
#pragma unroll
    for (int k = 0; k < NK; ++k) acc[k] = bq;
    gemv(acc, wqT + o, HC, F, k0);
#pragma unroll
    for (int k = 0; k < NK; ++k) ql[k0 + k][o] = acc[k];
  }
  __syncthreads();

  // cross-attention: thread -> (candidate k, head hh, half of the head's 32 channels)
  {
    const bool mine = t < 8 * TK;                  // the other threads only help to load
    const int k = mine ? t >> 3 : 0, hh = (t >> 1) & 3, half = t & 1;
    const int c0 = hh * 32 + half * 16;
    float q[16], o[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      q[c] = ql[k][c0 + c];
      o[c] = 0.f;
    }
    float m = -INFINITY, lsum = 0.f;
    const bool on = xattn && nql > 0;
    const float scale = 0.17677669529663688f;   // 1/sqrt(32)
    for (int p0 = 0; on && p0 < nql; p0 += KC) {
      const int np = min(KC, nql - p0);
      __syncthreads();
      for (int e = t; e < KC * HC; e += 256) {
        const int p = e / HC, c = e - p * HC;
        kvl[0][p][c] = p < np ? kp[int64_t(p0 + p) * HC + c] : 0.f;
        kvl[1][p][c] = p < np ? vp[int64_t(p0 + p) * HC + c] : 0.f;
      }
      __syncthreads();
      for (int p = 0; mine && p < np; ++p) {
        float x = 0.f;
#pragma unroll
        for (int c = 0; c < 16; ++c) x = fmaf(q[c], kvl[0][p][c0 + c], x);
        x += __shfl_xor(x, 1, WAVE);
        x *= scale;
        const float mn = fmaxf(m, x);
        const float corr = (m == -INFINITY) ? 0.f : expf(m - mn);
        const float w = expf(x - mn);
        lsum = lsum * corr + w;
#pragma unroll
        for (int c = 0; c < 16; ++c) o[c] = fmaf(w, kvl[1][p][c0 + c], o[c] * corr);
        m = mn;
      }
    }
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    if (mine)
#pragma unroll
      for (int c = 0; c < 16; ++c) xT[F + c0 + c][k] = o[c] * inv;
  }
  __syncthreads();

  // hidden layer: thread -> hidden unit o, every candidate
  {
    const int o = t;
    float acc[TK];
    const float b1 = blob[lay.b1 + o];
#pragma unroll
    for (int k = 0; k < TK; ++k) acc[k] = b1;
    gemv(acc, w1T + o, HIDDEN, X, 0);
    const float w2 = blob[lay.w2 + o];
    const int wave = t >> 6;
#pragma unroll
    for (int k = 0; k < TK; ++k) {
      const float y = wave_sum(gelu_erf(acc[k]) * w2);
      if ((t & 63) == 0) red[wave][k] = y;
    }
  }
  __syncthreads();
  if (t < TK && pos[t] >= 0) {
    const float alpha = fminf(fmaxf(blob[lay.alpha], -5.0f), 5.0f);
    const float y = ((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) + blob[lay.b2];
    const int j = pos[t];
    out[j] = out[j] + alpha * y;
  }
}

hipError_t launch_residual_mfma(const ScoreArgs &a, hipStream_t st);

template <int D>
static hipError_t launch_residual_t(const ScoreArgs &a, hipStream_t st) {
  const ikv_pool &p = a.pool;
  // on the vector-unit path k_score_rest has transposed the weights and left the partial sums
  // of mbar (on the matrix-core path k_msplit or the first pass leaves those)
  if (!a.mfma_resid && a.mfma)
    {
      KTimer kt_("k_res_transpose", st);
      k_res_transpose<<<unsigned(cdiv(res_transpose_items(D), 256)), 256, 0, st>>>(a.residual, a.ws_shared, D);
    }
  if (!a.mfma)   // on the matrix-core path the row-statistics launch did the set-up
    {
      KTimer kt_("k_res_setup<D>", st);
      k_res_setup<D><<<a.B, 256, 0, st>>>(a.sess_dev, a.slot_maps, a.qpos, p.dead_slot, a.ws, p.L, p.Hkv, a.mfma,
                                          a.stats);
    }
  if (a.maxNq > 0 && !a.mfma_resid && a.mfma)
    {
      KTimer kt_("k_res_kq<D>", st);
      k_res_kq<D><<<dim3(unsigned(a.maxNq), a.B), D, 0, st>>>(a.sess_dev, static_cast<const uint16_t *>(p.k_pool),
                                                              p.num_slots, p.L, p.Hkv, a.slot_maps, a.ws);
    }
  if (a.maxNq > 0 && !a.mfma_resid)
    {
      KTimer kt_("k_res_kv<D>", st);
      k_res_kv<D><<<dim3(unsigned(cdiv(a.maxNq, 4)), a.B), 256, 0, st>>>(a.sess_dev, a.residual, a.ws, p.L, p.Hkv,
                                                                         a.mfma);
    }
  // on the matrix-core path the row-statistics launch also folded the first layer and
  // built the K', V' fragments
  if (a.mfma_resid) return launch_residual_mfma(a, st);
  {
    KTimer kt_("k_residual<D>", st);
    auto run = [&](auto tk) {
      constexpr int TK = decltype(tk)::value;
      k_residual<D, TK><<<dim3(unsigned(cdiv(a.maxN, TK)), a.B), 256, 0, st>>>(
          a.sess_dev, a.slot_maps, p.dead_slot, a.scores, a.ws, a.ws_shared, a.residual, p.L, p.Hkv,
          (a.flags & IKV_NO_XATTN) == 0, a.mfma);
    };
    // the fewest candidates that keep within about two rounds of one workgroup per CU
    int64_t n = 0;
    for (int b = 0; b < a.B; ++b) n += a.sess_host[b].N > a.sess_host[b].C ? a.sess_host[b].N : 0;
    if (n <= 512 * 8) run(std::integral_constant<int, 8>{});
    else if (n <= 512 * 16) run(std::integral_constant<int, 16>{});
    else run(std::integral_constant<int, 32>{});
  }
  return hipGetLastError();
}

hipError_t launch_residual(const ScoreArgs &a, hipStream_t st) {
  return a.pool.D == 128 ? launch_residual_t<128>(a, st) : launch_residual_t<64>(a, st);
}

}  // namespace ikv
