// The position-major score passes of the matrix-core path (bf16 pool, D = 128, up to 128
// memory rows per KV head) in narrow tiles, for calls of few positions: the second pass of
// the two-pass form, and the one key pass of sessions of at most 16 memory rows.
//
// Both need a sum over every unit (layer, KV head) per position - the rule score of Eq. 3
// and, with the residual head, the mean key row of Eq. 5 - so a workgroup owns a tile of
// list entries and walks all units, one CU to itself (160 KB of LDS). The 128-entry passes
// (k_score_ws) leave CUs idle when there are fewer than 256 tiles: 4096 positions are 32
// tiles, 0.28 ms with 4 memory rows, most of it the same latency a unit whatever the
// tile. Here a tile is NG = 1 or 2 groups of 32 list entries, as long as those fit one
// round of CUs (narrow_tiles). Time per unit (36 layers, 8 KV heads, a full round) at 32,
// 64 and 128 entries: one key pass at 4 rows 0.44, 0.69, 1.26 us; second pass at 64 rows
// 0.80, 1.00, 1.58 us, at 128 rows 1.44, 1.67, 2.50 us (the memory rows, 32 or 64 KB a
// unit from L2, do not shrink with the tile). Measured per call: one key pass, 4096
// positions, 4 rows 278 -> 83 us; 12,000 positions 286 -> 179; second pass, 12,000
// positions, 64 rows 372 -> 300, 100 rows 609 -> 467 us.
//
// The arithmetic of a position does not depend on its tile: the order of its additions is
// that of the 128-entry passes, and every width gives the same bits.
//
// Producer and consumer waves, as in k_score_ws. Waves 4-7 (producers) issue every load and
// sum the mean key row on the VALU; waves 0-3 (consumers, one per SIMD) only read LDS, run
// the logit MFMAs and finish them. Narrow tiles leave room in LDS for more stages in
// flight; in the one key pass a stage holds UPS = 4 / NG units, one or two consumer waves
// each, so that a barrier still covers 32 KB of keys.
#include <algorithm>

#include "score_mfma.hpp"

namespace ikv {

constexpr int PW_THREADS = 512;
constexpr int PW_LDS = 160 * 1024;               // bytes
constexpr int PW_CUS = 256;                      // workgroups of one round

struct PosArgs {
  const uint16_t *kpool;
  int64_t num_slots;
  int L, Hkv, dead;
  const ikv_session *sess;
  const int32_t *slot_maps;
  float *ws;
  float *scores;
  bool resid;
  int CH;
  int ng;              // groups per tile
  bool fewer;          // take one group where that fits a round (one session: the count is known here)
};

// The groups of a tile (one or two): group j holds list entries at slots base .. base + ne - 1
// of the candidate list (chunk c of CH positions keeps its list at [c CH ...]). ident: a
// chunk whose every position is a candidate is its own list.
struct PosTile {
  int base[2], ne[2];
  bool ident[2];
};

// Groups of 32 entries of tile `tile`: the chunks' group counts are summed by a scan over
// the workgroup, 512 chunks at a time. Returns the groups per tile (0: no such tile).
__device__ __forceinline__ int pos_find(const PosArgs &a, const ikv_session &s, const int32_t *__restrict__ cc,
                                        int tile, int *__restrict__ scratch, PosTile &T) {
  int *wsum = scratch, *gi = scratch + 8;          // [8], [2][3]
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int nch = int(cdiv(s.N, a.CH));
  int cnt = 0, g = 0, excl = 0, tot = 0;
  auto scan = [&](int i0, int before) __attribute__((always_inline)) {
    const int i = i0 + t;
    cnt = i < nch ? cc[i] : 0;
    g = (cnt + 31) >> 5;
    int in = g;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int up = __shfl_up(in, o, WAVE);
      if (lane >= o) in += up;
    }
    if (lane == WAVE - 1) wsum[w] = in;
    __syncthreads();
    int off = before;
    tot = 0;
#pragma unroll
    for (int q = 0; q < PW_THREADS / WAVE; ++q) {
      const int v = wsum[q];
      off += q < w ? v : 0;
      tot += v;
    }
    excl = off + in - g;
    __syncthreads();
  };
  if (t < 6) gi[t] = 0;
  int groups = 0;
  for (int i0 = 0; i0 < nch; i0 += PW_THREADS) {
    scan(i0, groups);
    groups += tot;
  }
  groups = __builtin_amdgcn_readfirstlane(groups);
  const int ng = a.fewer && groups <= PW_CUS ? 1 : a.ng;
  const int g0 = tile * ng;
  if (g0 >= groups) return 0;
  int before = 0;
  for (int i0 = 0; i0 < nch; i0 += PW_THREADS) {
    if (nch > PW_THREADS) {                        // otherwise the only scan's values are still here
      scan(i0, before);
      before += tot;
    }
    for (int j = 0; j < ng; ++j) {
      const int q = g0 + j - excl;
      if (q >= 0 && q < g) {
        gi[3 * j] = (i0 + t) * a.CH + 32 * q;
        gi[3 * j + 1] = min(32, cnt - 32 * q);
        gi[3 * j + 2] = cnt == min(a.CH, s.N - (i0 + t) * a.CH);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    T.base[j] = __builtin_amdgcn_readfirstlane(gi[3 * j]);
    T.ne[j] = __builtin_amdgcn_readfirstlane(gi[3 * j + 1]);
    T.ident[j] = __builtin_amdgcn_readfirstlane(gi[3 * j + 2]) != 0;
  }
  __syncthreads();                                 // scratch lies in the ring
  return ng;
}

// RH row halves per unit: 1 for sessions of up to 64 memory rows; 2 for up to 128, where
// every unit's rows stream as two halves of 64 against the one key stage of the unit (a
// "virtual unit" is a half). A batch holding both kinds runs one launch of each.
template <int NG, bool KBAR, int RH, bool STASH>
__device__ __forceinline__ void pos_body(const PosArgs &a, const ikv_session &s, int b, const PosTile &T,
                                         uint16_t *__restrict__ lds) {
  constexpr int P = 32 * NG;                       // entries per tile
  constexpr int UPS = STASH ? 4 / NG : 1;          // units per stage
  constexpr int KU = P * MD;                       // bf16 of one unit's keys
  constexpr int KSZ = UPS * KU * 2;                // bytes of a key stage
  constexpr int KW = 2 * NG;                       // key loads (1 KB) per producer per unit
  constexpr int CPL = 2 * NG;                      // 8-channel chunks of the mean key row per lane
  const int units = a.L * a.Hkv, Hkv = a.Hkv;
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int R = s.R, R16 = pad16(R);
  const ScoreSizes z = score_sizes(s, a.L, units, MD, a.resid, true);
  float *base = a.ws + score_offset(a.sess, b, a.L, units, MD, a.resid, true);
  const int32_t *S = a.slot_maps + s.slot_off;
  const int32_t *lst = reinterpret_cast<const int32_t *>(base + z.off_clist());
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(lds));
  // entry tok of the tile: its list slot, whether it holds a candidate, the position
  auto pick = [&](const int (&v)[2], int j) __attribute__((always_inline)) {
    int r = v[0];
#pragma unroll
    for (int k = 1; k < NG; ++k) r = j == k ? v[k] : r;
    return r;
  };
  auto on_of = [&](int tok) __attribute__((always_inline)) { return (tok & 31) < pick(T.ne, tok >> 5); };
  auto pos_of = [&](int tok) __attribute__((always_inline)) {
    const int j = tok >> 5, e = pick(T.base, j) + (tok & 31);
    bool id = T.ident[0];
#pragma unroll
    for (int k = 1; k < NG; ++k) id = j == k ? T.ident[k] : id;
    return id ? e : lst[e];
  };

  // LDS: `ks` key stages from the start, `ms` memory-row stages at the end. The one key
  // pass keeps the R rows of its units (its pad rows' logits are never used), the two-pass
  // form the rows padded to slices (pad rows zero), up to 64 of them.
  const int mrow = STASH ? (R + 1) & ~1 : min(R16, 64);        // rows of a unit (half) in LDS
  const int MSZ = UPS * mrow * 512;                // bytes of a memory-row stage
  // Memory rows ma stages ahead of their use, keys kc. In issue order a key stage is waited
  // for with the memory rows issued a step after it, so keys gain nothing past ma + 1 ahead:
  // one row stage ahead where two would leave the keys fewer than three stages.
  const int ks3 = (PW_LDS - 3 * MSZ) / KSZ;
  const int ma = RH == 1 && ks3 >= 4 ? 2 : 1, ms = ma + 1;
  const int ks = ma == 2 ? 4 : min((PW_LDS - 2 * MSZ) / KSZ, 3), kc = ks - 1;
  const uint32_t mlds = uint32_t(PW_LDS - ms * MSZ);
  const int NS = (units + UPS - 1) / UPS;          // stages

  if (w >= 4) {
    // ---------------- producers: the rings' loads, and the mean key row
    const int pw = w - 4;
    const int64_t slot_stride = int64_t(Hkv) * MD;
    // key load k of producer pw: entries 4 (KW pw + k) .. + 3 of a unit, 16 lanes each,
    // 16-byte slot lane % 16 of the row, which holds chunk (lane % 16) ^ (entry % 16)
    const uint16_t *src[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int tok = (KW * pw + k) * 4 + (lane >> 4);
      const int slot = on_of(tok) ? S[pos_of(tok)] : a.dead;   // past the list: any valid row
      src[k] = a.kpool + int64_t(slot) * slot_stride + ((lane & 15) ^ (tok & 15)) * 8;
    }
#pragma unroll
    for (int k = 0; k < KW; ++k) asm volatile("" ::"v"(src[k]));   // complete before the first DMA
    // the units' keys are issued in order: where the next unit's rows lie, and its stage
    int ku = 0, kh = 0, kslot = 0;
    int64_t koff = 0;
    const int64_t layer_step = (a.num_slots - 1) * slot_stride + MD;   // last head of a layer to the next layer's first
    auto issue_k_piece = [&](int j, int k) __attribute__((always_inline)) {
      dma16_nt(src[k] + koff, __builtin_amdgcn_readfirstlane(lds0 + uint32_t(kslot * KSZ + j * KU * 2) +
                                                             uint32_t((KW * pw + k) * 1024)));
    };
    auto next_k = [&](int j) __attribute__((always_inline)) {   // after unit j of a stage
      ++ku;
      const bool wrap = ++kh == Hkv;
      koff += wrap ? layer_step : MD;
      kh = wrap ? 0 : kh;
      if (j == UPS - 1) kslot = kslot + 1 == ks ? 0 : kslot + 1;
    };
    // memory rows of a unit (half): 512 B each, two per 1-KB load, chunk slot c of row r
    // holding chunk c ^ (r & 15); producer pw takes loads pw, pw + 4, ...
    const uint16_t *msplit = reinterpret_cast<const uint16_t *>(base);
    int mu = 0, mslot = 0;                          // the next unit (RH = 1) to issue, its stage
    auto npc_of = [&](int hf) __attribute__((always_inline)) {
      return STASH ? (mrow / 2 - pw + 3) >> 2 : min(64, max(0, R16 - 64 * hf)) >> 3;
    };
    auto issue_m_piece = [&](int u, int j, int hf, int k) __attribute__((always_inline)) {
      const uint16_t *m0 = msplit + (int64_t(u) * R16 + 64 * hf) * 256;
      const int piece = pw + 4 * k;
      const int r = piece * 2 + (lane >> 5);
      const int sl = lane & 31;
      dma16(m0 + r * 256 + ((sl ^ (r & 15)) * 8),
            __builtin_amdgcn_readfirstlane(lds0 + mlds + uint32_t(mslot * MSZ + j * mrow * 512 + piece * 1024)));
    };
    auto next_m = [&]() __attribute__((always_inline)) { mslot = mslot + 1 == ms ? 0 : mslot + 1; };
    // mean key row: this lane's entry and first chunk of 8 channels
    const int pp = NG == 2 ? 32 * (pw & 1) + (lane & 31) : lane & 31;
    const int cg = (NG == 2 ? 2 * (pw >> 1) + (lane >> 5) : 2 * pw + (lane >> 5)) * CPL;
    float kb[8 * CPL];
#pragma unroll
    for (int i = 0; i < 8 * CPL; ++i) kb[i] = 0.f;
    uint4 kv[2];
    auto kbar_read = [&](const uint16_t *kr, int c) __attribute__((always_inline)) {
      kv[c & 1] = *reinterpret_cast<const uint4 *>(kr + (((cg + c) ^ (pp & 15)) * 8));
    };
    auto kbar_step = [&](int c) __attribute__((always_inline)) {
      const uint4 v = kv[c & 1];
      const uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {                  // bf16 -> float is exact: the high half of the word
        kb[8 * c + 2 * e] += __uint_as_float(q[e] << 16);
        kb[8 * c + 2 * e + 1] += __uint_as_float(q[e] & 0xffff0000u);
      }
    };
    // step v issues the memory rows of stage v + ma, then the keys of stage v + kc; the steps
    // before stage 0 fill the rings
    auto keys_of_stage = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < UPS; ++j) {
        if (ku >= units) break;
#pragma unroll
        for (int k = 0; k < KW; ++k) issue_k_piece(j, k);
        next_k(j);
      }
    };
    int rd = 0;                                      // the stage in use
    if constexpr (RH == 1) {
      for (int v = -max(ma, kc); v < 0; ++v) {
        if (v + ma >= 0) {
          for (int j = 0; j < UPS && mu < units; ++j, ++mu)
            for (int k = 0; k < npc_of(0); ++k) issue_m_piece(mu, j, 0, k);
          next_m();
        }
        if (v + kc >= 0) keys_of_stage();
      }
      constexpr int ST = CPL;                        // steps per unit
      for (int v = 0; v < NS; ++v) {
        // Outstanding at the top of stage v: what was issued after its rows and keys, that
        // is row stages v + 1 .. v + ma - 1 and key stages v + 1 .. v + kc - 1 (kc <= ma + 1).
        // Where one of them is the last, which may be short, or past it: everything waits
        // (the last stages are then in LDS together).
        if (v + max(ma, kc) > NS - 1) {
          vm_wait_c<0>();
        } else if (ma == 1) {
          if (kc == 2) vm_wait_c<UPS * KW>();
          else vm_wait_c<0>();
        } else {                                     // ma = 2, kc = 3
          constexpr int K2 = 2 * UPS * KW;
          if constexpr (STASH) {
            vm_wait_c<K2>();                         // at most two row loads a unit: not counted
          } else {
            switch (npc_of(0)) {
              case 8: vm_wait_c<K2 + 8>(); break;
              case 6: vm_wait_c<K2 + 6>(); break;
              case 4: vm_wait_c<K2 + 4>(); break;
              default: vm_wait_c<K2 + 2>(); break;   // R16 = 16
            }
          }
        }
        __syncthreads();
        const uint16_t *kr = lds + rd * (KSZ / 2) + pp * MD;
#pragma unroll
        for (int j = 0; j < UPS; ++j) {
          if (UPS > 1 && v * UPS + j >= units) break;
          if (KBAR) kbar_read(kr + j * KU, 0);
          const bool more = ku < units;
          // Rows before keys, as the counts above take them. Second pass: the row loads in
          // the first half of the unit's steps, its key loads in the second, among the
          // additions of the mean key row; one key pass: the few row loads of the whole stage
          // in its first step.
#pragma unroll
          for (int c = 0; c < ST; ++c) {
            if (KBAR && c + 1 < ST) kbar_read(kr + j * KU, c + 1);
            if (c < ST / 2) {
              if constexpr (STASH) {
                if (j == 0 && c == 0)
#pragma unroll
                  for (int q = 0; q < UPS; ++q)
                    if (mu + q < units)
#pragma unroll
                      for (int k = 0; k < 2; ++k)
                        if (k < npc_of(0)) issue_m_piece(mu + q, q, 0, k);
              } else {
                constexpr int MPS = 8 / (ST / 2);
                const int nn = mu < units ? npc_of(0) : 0;
#pragma unroll
                for (int k = MPS * c; k < MPS * c + MPS; ++k)
                  if (k < nn) issue_m_piece(mu, 0, 0, k);
              }
            } else if (more) {
              constexpr int KPS = (KW + ST / 2 - 1) / (ST / 2);
#pragma unroll
              for (int k = KPS * (c - ST / 2); k < KPS * (c - ST / 2) + KPS; ++k)
                if (k < KW) issue_k_piece(j, k);
            }
            if (KBAR) kbar_step(c);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (more) next_k(j);
        }
        mu += UPS;
        next_m();
        rd = rd + 1 == ks ? 0 : rd + 1;
      }
    } else {
      // Per half hf of unit u: the next half's rows, then half of the key loads of unit
      // u + kc; the mean key row takes half of its chunks. At the top of a half only the key
      // loads issued after its rows may be outstanding.
      keys_of_stage();
      for (int k = 0; k < npc_of(0); ++k) issue_m_piece(0, 0, 0, k);
      next_m();
      for (int v = 1; v < kc; ++v) keys_of_stage();
      constexpr int ST = CPL / 2;                    // steps per half
      for (int u = 0; u < units; ++u) {
        const uint16_t *kr = lds + rd * (KSZ / 2) + pp * MD;
        const bool more = ku < units;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          if (hf == 0 ? u > 0 && u - 1 + kc < units : more) vm_wait_c<KW / 2>();
          else vm_wait_c<0>();
          __syncthreads();
          if (KBAR) kbar_read(kr, hf * ST);
          const int mn = hf == 0 ? u : u + 1, mh = hf ^ 1, nn = mn < units ? npc_of(mh) : 0;
#pragma unroll
          for (int c = 0; c < ST; ++c) {
            if (KBAR && c + 1 < ST) kbar_read(kr, hf * ST + c + 1);
            // ST = 1: both kinds in the one step
            if (c < ST / 2 || ST == 1) {
              constexpr int MPS = ST == 1 ? 8 : 8 / (ST / 2);
#pragma unroll
              for (int k = MPS * c; k < MPS * c + MPS; ++k)
                if (k < nn) issue_m_piece(mn, 0, mh, k);
            }
            if ((c >= ST / 2 || ST == 1) && more) {
              constexpr int KH = KW / 2, SK = ST == 1 ? 1 : ST / 2, KPS = (KH + SK - 1) / SK;
              const int c0 = ST == 1 ? 0 : c - ST / 2;
#pragma unroll
              for (int k = KPS * c0; k < KPS * c0 + KPS; ++k)
                if (k < KH) issue_k_piece(0, hf * KH + k);
            }
            if (KBAR) kbar_step(hf * ST + c);
            __builtin_amdgcn_sched_barrier(0);
          }
          next_m();
        }
        if (more) next_k(0);
        rd = rd + 1 == ks ? 0 : rd + 1;
      }
    }
    __syncthreads();                                 // the ring is free (matches the consumers)
    // The mean key rows go out through LDS, so that each store writes two whole
    // 512-byte rows: stored straight from the lanes, every line would leave L2 in
    // 16-byte pieces. Rows of 132 floats keep the lanes' writes on distinct banks;
    // the region starts past the consumers' reduction buffer.
    float *kt = reinterpret_cast<float *>(lds) + 2 * 128;
    constexpr int KT_ROW = MD + 4;
    if (KBAR) {
      const float inv = 1.0f / float(units);
#pragma unroll
      for (int q = 0; q < 2 * CPL; ++q)
        *reinterpret_cast<float4 *>(kt + pp * KT_ROW + 8 * cg + 4 * q) =
            make_float4(kb[4 * q] * inv, kb[4 * q + 1] * inv, kb[4 * q + 2] * inv, kb[4 * q + 3] * inv);
    }
    __syncthreads();
    if (KBAR) {
      // producer pw stores entries 8 NG pw .. + 8 NG - 1: two rows (32 lanes x 16 B each) per instruction
#pragma unroll
      for (int q = 0; q < 4 * NG; ++q) {
        const int pr = 8 * NG * pw + 2 * q + (lane >> 5);
        const float4 v = *reinterpret_cast<const float4 *>(kt + pr * KT_ROW + 4 * (lane & 31));
        if (on_of(pr)) reinterpret_cast<float4 *>(base + z.off_kbar() + int64_t(pos_of(pr)) * MD)[lane & 31] = v;
      }
    }
    return;
  }

  if constexpr (STASH) {
    // ---------------- consumers, one key pass: a unit's logits of 32 entries to the stash
    // (log2 domain), and their (max, sum of exp2) per row, the partial of the entries'
    // quarter of a list tile; k_lse_mfma and k_score_stash finish the score. Consumer w
    // takes unit w UPS / 4 of a stage, group w % (4 / UPS) of the tile.
    constexpr int CPU = 4 / UPS;                     // consumers per unit
    const int cj = w / CPU, grp = w % CPU;
    const bool act = grp < NG && T.ne[grp < NG ? grp : 0] > 0;
    const int q0 = 32 * grp;
    const int gb = pick(T.base, grp), ne = pick(T.ne, grp);
    const int64_t NSt = stash_stride(s.N);
    float *stash = base + z.off_stash() + gb + 4 * g;
    float2 *pt = reinterpret_cast<float2 *>(base + z.off_part()) + int64_t(gb >> 5) * units * R;
    const int rl = min(r16, R - 1);                  // rows past R repeat the last one; never stored
    int rd = 0, md = 0;
    for (int v = 0; v < NS; ++v) {
      __syncthreads();                               // stage v in LDS
      const int u = v * UPS + cj;
      const uint16_t *kl = lds + rd * (KSZ / 2) + cj * KU;
      const uint16_t *mr = lds + (mlds + md * MSZ) / 2 + (cj * mrow + rl) * 256;
      rd = rd + 1 == ks ? 0 : rd + 1;
      md = md + 1 == ms ? 0 : md + 1;
      if (!act || u >= units) continue;
      bf16x8 mh[4], ml[4], ka[2][4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        mh[k] = *reinterpret_cast<const bf16x8 *>(mr + (((g * 8 + k * 2) ^ rl) * 8));
        ml[k] = *reinterpret_cast<const bf16x8 *>(mr + (((g * 8 + k * 2 + 1) ^ rl) * 8));
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
          ka[blk][k] = *reinterpret_cast<const bf16x8 *>(kl + (q0 + blk * 16 + r16) * MD + (((4 * k + g) ^ r16) * 8));
      }
      // lane (g, r16) of block blk: row r16 at entries q0 + 16 blk + 4 g + i
      f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
          acc[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[blk][k], mh[k], acc[blk], 0, 0, 0);
          acc[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[blk][k], ml[k], acc[blk], 0, 0, 0);
        }
      if (r16 < R) {
        float *o = stash + (int64_t(u) * R + r16) * NSt;
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)         // read once, by k_score_stash: non-temporal
          __builtin_nontemporal_store(acc[blk], reinterpret_cast<f32x4 *>(o + 16 * blk));
      }
      // the row's max and sum over the entries that hold a candidate
      float m = -INFINITY;
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (16 * blk + 4 * g + i >= ne) acc[blk][i] = -INFINITY;
          m = fmaxf(m, acc[blk][i]);
        }
      m = fmaxf(m, __shfl_xor(m, 16, WAVE));
      m = fmaxf(m, __shfl_xor(m, 32, WAVE));
      float zs = 0.f;
      if (m != -INFINITY)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
#pragma unroll
          for (int i = 0; i < 4; ++i) zs += ex2(acc[blk][i] - m);
      zs += __shfl_xor(zs, 16, WAVE);
      zs += __shfl_xor(zs, 32, WAVE);
      if (g == 0 && r16 < R) pt[int64_t(u) * R + r16] = make_float2(m, zs);
    }
    __syncthreads();                                 // matches the producers' "ring is free"
    __syncthreads();                                 // matches the producers' mean-key-row barrier
    return;
  }

  // ---------------- consumers, second pass: logits on the matrix cores, exp2 folded into the rule score
  // consumer w takes memory rows 32 (w & 1) .. + 31 against NG blocks of 16 entries from p0
  const int rh = w & 1, p0 = (w >> 1) * 16 * NG;
  const int nsl = R16 >> 4;
  const float *nl2 = base + z.off_nl2();
  float racc[NG][4];
#pragma unroll
  for (int blk = 0; blk < NG; ++blk)
#pragma unroll
    for (int i = 0; i < 4; ++i) racc[blk][i] = 0.f;
  f32x4 accp[2][NG];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl)
#pragma unroll
    for (int blk = 0; blk < NG; ++blk) accp[sl][blk] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  // step c (0-7) of the previous unit's epilogue: exp2 of NG of its 8 NG logits per lane
  auto epilogue_step = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      const int e = NG * c + k, sl = e / (4 * NG), blk = (e >> 2) % NG, i = e & 3;
      racc[blk][i] += ex2(accp[sl][blk][i]);
    }
  };
  // Seeds -(max + log2 Z) of the lane's two rows, loaded two (virtual) units ahead at
  // the end of a unit's MFMAs: issued right after the barrier, a load would queue behind
  // the producers' ring loads at the address unit. Rows past R take -inf against zero
  // fragments, so exp2 of their logits is 0. Virtual unit v is half v % RH of unit v / RH.
  auto rowv = [&](int v, int k) __attribute__((always_inline)) { return 64 * (v % RH) + 32 * rh + 16 * k + r16; };
  auto seed_ld = [&](int v, int k) __attribute__((always_inline)) { return nl2[int64_t(v / RH) * R + min(rowv(v, k), R - 1)]; };
  int rd = 0, md = 0;
  // one virtual unit: seeds s0, s1 as loaded (rows past R take -inf here)
  auto unit_step = [&](int v, float s0, float s1) __attribute__((always_inline)) {
    const int hf = v % RH;
    const float seed0 = rowv(v, 0) < R ? s0 : -INFINITY, seed1 = rowv(v, 1) < R ? s1 : -INFINITY;
    const bool act0 = 4 * hf + 2 * rh < nsl, act1 = 4 * hf + 2 * rh + 1 < nsl;   // slices within R
    __syncthreads();
    const uint16_t *kl = lds + rd * (KSZ / 2);
    const uint16_t *mb = lds + (mlds + md * MSZ) / 2;
    if (RH == 1 || hf == RH - 1) rd = rd + 1 == ks ? 0 : rd + 1;
    md = md + 1 == ms ? 0 : md + 1;
    // slices past R read the first one and take zeros
    const uint16_t *mr0 = mb + ((act0 ? 32 * rh : 0) + r16) * 256, *mr1 = mb + ((act1 ? 32 * rh + 16 : 0) + r16) * 256;
    // fragments of k-step k: memory rows (hi, lo) of both slices, the key blocks
    bf16x8 mh[2][4], ml[2][4], ka[NG][4];
    auto read_ks = [&](int k) __attribute__((always_inline)) {
      const int ch = ((g * 8 + k * 2) ^ r16) * 8, cl = ((g * 8 + k * 2 + 1) ^ r16) * 8;
      mh[0][k] = *reinterpret_cast<const bf16x8 *>(mr0 + ch);
      ml[0][k] = *reinterpret_cast<const bf16x8 *>(mr0 + cl);
      mh[1][k] = *reinterpret_cast<const bf16x8 *>(mr1 + ch);
      ml[1][k] = *reinterpret_cast<const bf16x8 *>(mr1 + cl);
      if (!act0) mh[0][k] = ml[0][k] = bf16x8{};
      if (!act1) mh[1][k] = ml[1][k] = bf16x8{};
#pragma unroll
      for (int blk = 0; blk < NG; ++blk)
        ka[blk][k] = *reinterpret_cast<const bf16x8 *>(kl + (p0 + blk * 16 + r16) * MD + (((4 * k + g) ^ r16) * 8));
    };
    read_ks(0);
    f32x4 acc[2][NG];
#pragma unroll
    for (int blk = 0; blk < NG; ++blk) {
      acc[0][blk] = f32x4{seed0, seed0, seed0, seed0};
      acc[1][blk] = f32x4{seed1, seed1, seed1, seed1};
    }
    // chunk c: the MFMAs of k-step c/2 (hi, then lo) for both slices, then step c of the
    // previous unit's epilogue; the fences keep the interleave
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int k = c >> 1;
      if ((c & 1) == 0 && k + 1 < 4) read_ks(k + 1);
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
#pragma unroll
        for (int blk = 0; blk < NG; ++blk)
          acc[sl][blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[blk][k], (c & 1) ? ml[sl][k] : mh[sl][k],
                                                                 acc[sl][blk], 0, 0, 0);
      epilogue_step(c);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int sl = 0; sl < 2; ++sl)
#pragma unroll
      for (int blk = 0; blk < NG; ++blk) accp[sl][blk] = acc[sl][blk];
  };
  // Even and odd virtual units keep their own seed registers (unrolled by two), so
  // that no register that a load is still filling has to be copied.
  const int V = units * RH;
  float a0 = seed_ld(0, 0), a1 = seed_ld(0, 1), b0 = 0.f, b1 = 0.f;
  if (V > 1) {
    b0 = seed_ld(1, 0);
    b1 = seed_ld(1, 1);
  }
  for (int v = 0; v < V; v += 2) {
    unit_step(v, a0, a1);
    if (v + 2 < V) {
      a0 = seed_ld(v + 2, 0);
      a1 = seed_ld(v + 2, 1);
    }
    if (v + 1 < V) {
      unit_step(v + 1, b0, b1);
      if (v + 3 < V) {
        b0 = seed_ld(v + 3, 0);
        b1 = seed_ld(v + 3, 1);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) epilogue_step(c);      // the last unit
  __syncthreads();                                   // the ring is free: reuse it for the reduction
  float *red = reinterpret_cast<float *>(lds);       // [2][128]
#pragma unroll
  for (int blk = 0; blk < NG; ++blk)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = racc[blk][i];                        // entry p0 + 16 blk + 4 g + i, row r16 of both slices
      v += __shfl_xor(v, 1, WAVE);
      v += __shfl_xor(v, 2, WAVE);
      v += __shfl_xor(v, 4, WAVE);
      v += __shfl_xor(v, 8, WAVE);
      if (r16 == 0) red[rh * 128 + p0 + blk * 16 + 4 * g + i] = v;
    }
  __syncthreads();
  if (t < P && on_of(t)) a.scores[s.slot_off + pos_of(t)] = red[t] + red[128 + t];
}

template <bool KBAR, int RH, bool STASH>
__global__ void __launch_bounds__(PW_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) k_score_narrow(PosArgs a) {
  __shared__ __align__(1024) uint16_t lds[PW_LDS / 2];
  const int b = blockIdx.y;
  const ikv_session s = a.sess[b];
  if (s.N <= s.C) return;
  if (!STASH && (RH == 2) != (s.R > 64)) return;   // the other launch's session
  const int units = a.L * a.Hkv;
  const ScoreSizes z = score_sizes(s, a.L, units, MD, a.resid, true);
  const float *base = a.ws + score_offset(a.sess, b, a.L, units, MD, a.resid, true);
  const int32_t *cc = reinterpret_cast<const int32_t *>(base + z.off_ccount(s.N));
  PosTile T;
  const int ng = pos_find(a, s, cc, int(blockIdx.x), reinterpret_cast<int *>(lds), T);
  if (ng == 1) pos_body<1, KBAR, RH, STASH>(a, s, b, T, lds);
  else if (ng == 2) pos_body<2, KBAR, RH, STASH>(a, s, b, T, lds);
}

// As narrow as the workgroups of all sessions fit one round of CUs, from the position
// counts (every position a candidate; with fewer, fewer workgroups). Beyond 512 groups the
// 128-entry passes win: two rounds of 64 entries take 1.38 to 3.3 us a unit, one of 128 1.26
// to 2.5.
int narrow_tiles(const ScoreArgs &a) {
  int64_t n[2] = {0, 0};
  for (int b = 0; b < a.B; ++b)
    if (a.sess_host[b].N > a.sess_host[b].C) {
      const int64_t g = cdiv(a.sess_host[b].N, 32);
      n[0] += g;
      n[1] += cdiv(g, 2);
    }
  return n[0] == 0 ? 0 : n[0] <= PW_CUS ? 1 : n[1] <= PW_CUS ? 2 : 0;
}

hipError_t launch_score_narrow(const ScoreArgs &a, int lch, int ng, hipStream_t st) {
  const ikv_pool &p = a.pool;
  const bool resid = (a.flags & IKV_RESIDUAL) != 0;
  PosArgs x;
  x.kpool = static_cast<const uint16_t *>(p.k_pool);
  x.num_slots = p.num_slots;
  x.L = p.L;
  x.Hkv = p.Hkv;
  x.dead = p.dead_slot;
  x.sess = a.sess_dev;
  x.slot_maps = a.slot_maps;
  x.ws = a.ws;
  x.scores = a.scores;
  x.resid = resid;
  x.CH = lch;
  x.ng = ng;
  x.fewer = a.B == 1;
  // one session: up to a round of workgroups, whichever width the kernel takes
  const int64_t tiles = a.B == 1 ? PW_CUS : cdiv(cdiv(a.maxN, 32), ng);
  const dim3 grid(unsigned(tiles), unsigned(a.B));
  KTimer kt_(a.stash ? "k_score_narrow_once" : resid ? "k_score_narrow<true>" : "k_score_narrow<false>", st);
  if (a.stash) {
    if (resid) k_score_narrow<true, 1, true><<<grid, PW_THREADS, 0, st>>>(x);
    else k_score_narrow<false, 1, true><<<grid, PW_THREADS, 0, st>>>(x);
    return hipGetLastError();
  }
  // one launch per kind of session (up to 64 rows, up to 128)
  if (a.minR <= 64) {
    if (resid) k_score_narrow<true, 1, false><<<grid, PW_THREADS, 0, st>>>(x);
    else k_score_narrow<false, 1, false><<<grid, PW_THREADS, 0, st>>>(x);
  }
  if (a.maxR > 64) {
    if (resid) k_score_narrow<true, 2, false><<<grid, PW_THREADS, 0, st>>>(x);
    else k_score_narrow<false, 2, false><<<grid, PW_THREADS, 0, st>>>(x);
  }
  return hipGetLastError();
}

}  // namespace ikv
