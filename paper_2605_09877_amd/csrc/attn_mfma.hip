// Fused prefill attention for bf16, head_dim 128 on the gfx950 matrix cores.
//
// A workgroup of NW waves owns 32*NW consecutive queries of one chunk for one query head; each
// wave owns 32 of them.  Keys are visited in 64-key tiles through three regions that share one
// online softmax ("Readout" equations of the paper): normalised state rows (scale tau_state,
// all visible), window tokens before the chunk (scale tau_bswa, all visible), and the chunk's
// own tokens (causal).  Per tile and wave:
//   QK : S^T[key, query] = K_tile . Q^T   16 MFMA 32x32x16, K from LDS, Q^T kept in registers
//   SM : online softmax down the key axis; a lane holds one query column, so the running max and
//        sum are per-lane scalars plus one exchange with lane^32
//   PV : O^T[d, query] += V_tile^T . P^T  16 MFMA; V^T fragments come out of the row-major V
//        tile through the transposing LDS read; P^T is S^T's own register layout, no shuffle
// K and V tiles go from HBM/L2 straight into LDS (16 B per lane, swizzled rows) ahead of use,
// one barrier per tile.  The mask is never materialised: it is the tile loop bounds plus a
// compare on diagonal tiles.
//
// The kernel runs NW = 4 (128 queries per workgroup, two workgroups per CU; the four tile buffers,
// two K and two V, fill 64 KiB of LDS).  Eight waves on 256 queries halve the tile bytes per flop
// but measured slower, both with one barrier per tile and with the two halves of the workgroup
// running half a tile apart: the waves of one workgroup then move in step and their matrix and
// softmax phases coincide instead of overlapping.
#include <type_traits>

#include "kvm_device.h"
#include "kvm_internal.h"
#include "kvm_mfma.h"
#include "kvm_score.h"

namespace kvm {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kXcds = 8;  // accelerator dies, each with its own L2

// One query (the lane's, half of its channels) over its visible keys one after the other, in fp32: what is left to do when
// a product with a masked key's value, 0 x something that is not finite, has spoilt the result.
struct KeyWalk {
  const char *khat, *vhat, *ring_k, *ring_v, *in_k, *in_v;   // (in_k, in_v: at the chunk's first position)
  uint32_t kst, vst;
  int m, wrel, t0rel, ring_slot0, L;
  float c_state, c_bswa;   // logit scales, signs included
};
template <int D>
__device__ __forceinline__ void attend_one_by_one(const KeyWalk &w, const char *qrow, int n_keys, int g, f32x16 (&oacc)[D / 32],
                                                  float &m_run, float &l) {
  constexpr int kNb = D / 32;
  // channels of a lane: 32 * dblk + 8 * vq + 4 * g .. + 3, as in the accumulators
  auto load4 = [&](const char *row, int dblk, int vq, float *f) {
    const uint2 x = *reinterpret_cast<const uint2 *>(row + 2 * (32 * dblk + 8 * vq + 4 * g));
    f[0] = __uint_as_float(x.x << 16);
    f[1] = __uint_as_float(x.x & 0xffff0000u);
    f[2] = __uint_as_float(x.y << 16);
    f[3] = __uint_as_float(x.y & 0xffff0000u);
  };
  float qf[kNb][16];
#pragma unroll
  for (int i = 0; i < 4 * kNb; ++i) load4(qrow, i >> 2, i & 3, &qf[i >> 2][4 * (i & 3)]);
#pragma unroll
  for (int i = 0; i < kNb; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[i][v] = 0.f;
  m_run = -INFINITY;
  l = 0.f;
#pragma unroll 1
  for (int n = 0; n < n_keys; ++n) {
    const char *kr, *vr;
    if (n < w.m) {
      kr = w.khat + (uint32_t)n * (D * 2);
      vr = w.vhat + (uint32_t)n * (D * 2);
    } else {
      const int prel = w.wrel + (n - w.m);
      if (prel >= w.t0rel) {
        kr = w.in_k + (int64_t)prel * (int64_t)w.kst;
        vr = w.in_v + (int64_t)prel * (int64_t)w.vst;
      } else {
        int slot = w.ring_slot0 + (n - w.m);
        slot = slot >= w.L ? slot - w.L : slot;
        kr = w.ring_k + (uint32_t)slot * (D * 2);
        vr = w.ring_v + (uint32_t)slot * (D * 2);
      }
    }
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < 4 * kNb; ++i) {
      float x[4];
      load4(kr, i >> 2, i & 3, x);
#pragma unroll
      for (int e = 0; e < 4; ++e) dot = fmaf(qf[i >> 2][4 * (i & 3) + e], x[e], dot);
    }
    const float t = xhalf_sum(dot) * (n < w.m ? w.c_state : w.c_bswa);
    const float m_new = fmaxf(m_run, t);
    if (m_new == -INFINITY) continue;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new), pr = __builtin_amdgcn_exp2f(t - m_new);
    m_run = m_new;
    l = fmaf(l, alpha, pr);
#pragma unroll
    for (int i = 0; i < 4 * kNb; ++i) {
      float x[4];
      load4(vr, i >> 2, i & 3, x);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        oacc[i >> 2][4 * (i & 3) + e] = fmaf(pr, x[e], oacc[i >> 2][4 * (i & 3) + e] * alpha);
    }
  }
}

template <int NW, int D>
__device__ __forceinline__ void attn_body(const Dev &dv, const AttnArgs &a, uint16_t *Ks, uint16_t *Vs) {
  static_assert((D == 128 || D == 64) && (D == 128 || NW == 4), "");
  constexpr int kKs = D / 16, kNb = D / 32;      // channel steps of the first product, channel blocks of the second
  constexpr int kTileE = kTileKeys * D;
  constexpr bool kSplitP = D == 64;              // P as the sum of three bf16 numbers (see the kernel)
  constexpr int kTileQ = 32 * NW;
  constexpr int kVBufs = 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
  const int g = lane >> 5, l32 = lane & 31;
  // Workgroup -> work item.  The tpc * Gq workgroups that read the same K and V (query tiles of one
  // chunk x query heads of one KV group) are given to one XCD, whose L2 then serves all but the
  // first read of every tile: consecutive workgroup ids go round-robin over the 8 XCDs, so id % 8
  // picks the XCD and id / 8 walks that XCD's own sequence of (group, member) pairs.
  // The workgroup's 32 * NW query rows: with grouped queries (NW query heads or a multiple per KV
  // head) the waves take the same 32 positions of NW different heads, so that all of them end at
  // the same causal tile (no wave idles at the barriers while another finishes the diagonal, and
  // the workgroup stops loading tiles a position block sooner); otherwise consecutive positions
  // of one head.
  const int Gq = dv.Hq / dv.Hkv;
  const bool by_head = Gq % NW == 0;
  const int span = by_head ? 32 : kTileQ;   // positions a workgroup covers
  const int hpw = by_head ? NW : 1;         // heads a workgroup covers
  const int tpc = (dv.C + span - 1) / span;
  const int per_group = tpc * (Gq / hpw);
  const int n_groups = a.n_chunks * dv.Hkv * dv.B;
  const int xcd = blockIdx.x % kXcds, seq = blockIdx.x / kXcds;
  const int group = (seq / per_group) * kXcds + xcd;
  if (group >= n_groups) return;
  const int member = seq % per_group;
  const int qt = member % tpc, gq = (member / tpc) * hpw + (by_head ? wave : 0);
  const int ci = group % a.n_chunks;
  const int hkv = (group / a.n_chunks) % dv.Hkv;
  const int b = group / (a.n_chunks * dv.Hkv);
  const int hq = __builtin_amdgcn_readfirstlane(hkv * Gq + gq);
  const int u = b * dv.Hkv + hkv;
  const int Q0 = (tpc - 1 - qt) * span;                                  // longest causal part first
  const int nq = ci == a.n_chunks - 1 ? a.nq_total - ci * dv.C : dv.C;  // queries of this chunk
  if (Q0 >= nq) return;
  const int64_t cs = a.s + (int64_t)ci * dv.C;                           // chunk start position
  const int64_t wb = cs + dv.C - dv.L > 0 ? cs + dv.C - dv.L : 0;        // first window position
  const int wq0 = by_head ? Q0 : Q0 + 32 * wave;
  const int myq = wq0 + l32;
  const int m = a.m[ci];

  // Q^T fragments: query myq, channels 16*ks + 8*g .. +7
  bf16x8 qreg[kKs];
  {
    const int qc = myq < nq ? myq : nq - 1;
    const uint16_t *qrow =
        (const uint16_t *)a.q + b * a.q_b + ((int64_t)ci * dv.C + qc) * a.q_t + hq * a.q_h;
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) {
      Frag8 f;
      f.q = *reinterpret_cast<const uint4 *>(qrow + 16 * ks + 8 * g);
      qreg[ks] = f.v;
    }
  }
  const float rs = kLog2e * rsqrtf((float)D);
  float c_state = (dv.tau_state ? dv.tau_state[hq] : 1.f) * rs;
  float c_bswa = (dv.tau_bswa ? dv.tau_bswa[hq] : 1.f) * rs;
  // The softmax below takes the row maximum on raw dot products and applies a positive scale
  // afterwards; for a negative temperature the region's dot products are negated, by flipping
  // the sign of Q^T when the tile loop enters the region (exact in bf16, and K . (-Q) = -(K . Q)
  // bit for bit).  Two bits of one wave-uniform scalar, so that the test is a scalar one.
  const int neg_bits = __builtin_amdgcn_readfirstlane((c_state < 0.f ? 1 : 0) | (c_bswa < 0.f ? 2 : 0));
  c_state = fabsf(c_state);
  c_bswa = fabsf(c_bswa);

  const int n_st = __builtin_amdgcn_readfirstlane((m + kTileKeys - 1) / kTileKeys);
  const int qend = (Q0 + span < nq) ? Q0 + span : nq;  // one past the last valid query here
  const int n_win = (int)((cs + qend - wb + kTileKeys - 1) / kTileKeys);
  const int n_tiles = __builtin_amdgcn_readfirstlane(n_st + n_win);

  // Tile sources, all wave-uniform: state rows of this chunk's version; window positions from the
  // call's own k/v (at or after t0) or from the ring (before t0).  Positions are kept relative
  // to the chunk start so that the per-tile arithmetic is 32-bit.
  // All of it is wave-uniform, which the compiler cannot see through the 64-bit divisions above:
  // each value is pinned to scalar registers once, so that the per-tile address arithmetic and
  // the loads' base operands are scalar instructions.
  auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  auto uni_ptr = [](const char *p_) {
    const uint64_t x = (uint64_t)p_;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return (const char *)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  const char *khat = uni_ptr((const char *)dv.khat + (a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D) * 2);
  const char *vhat = uni_ptr((const char *)dv.vhat + (a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D) * 2);
  const char *ring_k = uni_ptr((const char *)dv.winK + (int64_t)u * dv.L * D * 2);
  const char *ring_v = uni_ptr((const char *)dv.winV + (int64_t)u * dv.L * D * 2);
  const uint32_t kst_in = (uint32_t)uni((int)(a.in.k_t * 2)), vst_in = (uint32_t)uni((int)(a.in.v_t * 2));
  const char *in_k = uni_ptr((const char *)a.in.k + (b * a.in.k_b + hkv * a.in.k_h + (cs - a.t0) * a.in.k_t) * 2);
  const char *in_v = uni_ptr((const char *)a.in.v + (b * a.in.v_b + hkv * a.in.v_h + (cs - a.t0) * a.in.v_t) * 2);
  const int wrel = uni((int)(wb - cs));                              // first window position (<= 0)
  const int t0rel = uni(a.t0 - cs < -(1 << 30) ? -(1 << 30) : (int)(a.t0 - cs));
  const int ring_slot0 = uni((int)(wb % dv.L));
  const int last_rel = uni(nq - 1);

  // Per-lane fragment offsets (elements) from the start of the K / V buffers.  K has two buffers
  // and its offsets flip after every tile; V buffers are addressed by tile number.
  uint32_t koff[kKs], voff[kNb];
  const auto dl = [&] {
    if constexpr (D == 128) {
      ktile_offsets(lane, koff);
      vtile_offsets(lane, voff);
      return dma_lane(lane);
    } else {
      ktile_offsets64(lane, koff);
      vtile_offsets64(lane, voff);
      return dma_lane64(lane);
    }
  }();
  auto kfrag = [&](const uint16_t *t, int blk, int ks) {
    if constexpr (D == 128) return ktile_frag(t, koff, blk, ks);
    else return ktile_frag64(t, koff, blk, ks);
  };
  auto vfrag = [&](const uint16_t *t, int dblk, int ks) {
    if constexpr (D == 128) return vtile_frag(t, voff, dblk, ks);
    else return vtile_frag64(t, voff, dblk, ks);
  };
  const uint32_t ks_addr = lds_addr_of(Ks), vs_addr = lds_addr_of(Vs);

  struct TileSrc {
    const char *k, *v;
    uint32_t kst, vst;
    int valid;
  };
  auto tile_src = [&](int it) {
    TileSrc t;
    if (it < n_st) {
      const int row0 = it * kTileKeys;
      t.k = khat + (uint32_t)row0 * (D * 2);
      t.v = vhat + (uint32_t)row0 * (D * 2);
      t.kst = t.vst = D * 2;
      t.valid = m - row0;
    } else {
      const int w = it - n_st;
      const int prel = wrel + w * kTileKeys;
      t.valid = last_rel - prel + 1;
      if (prel >= t0rel) {
        t.k = in_k + (int64_t)prel * (int64_t)kst_in;
        t.v = in_v + (int64_t)prel * (int64_t)vst_in;
        t.kst = kst_in;
        t.vst = vst_in;
      } else {
        int slot = ring_slot0 + w * kTileKeys;
        slot = slot >= dv.L ? slot - dv.L : slot;   // a window is at most L long: one wrap
        t.k = ring_k + (uint32_t)slot * (D * 2);
        t.v = ring_v + (uint32_t)slot * (D * 2);
        t.kst = t.vst = D * 2;
      }
    }
    return t;
  };
  auto issue_tile = [&](int it) {
    const TileSrc t = tile_src(it);
    const uint32_t k_at = ks_addr + (uint32_t)(it & 1) * (kTileE * 2), v_at = vs_addr + (uint32_t)(it % kVBufs) * (kTileE * 2);
    if constexpr (D == 128) {
      tile_dma<false, NW>(t.k, t.kst, t.valid, k_at, wave, dl);
      tile_dma<true, NW>(t.v, t.vst, t.valid, v_at, wave, dl);
    } else {
      tile_dma64<false>(t.k, t.kst, t.valid, k_at, wave, dl);
      tile_dma64<true>(t.v, t.vst, t.valid, v_at, wave, dl);
    }
  };

  f32x16 oacc[kNb];
#pragma unroll
  for (int i = 0; i < kNb; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[i][v] = 0.f;
  float m_run = -INFINITY, l_part = 0.f;
  Frag8 pb[4];  // P^T of the tile just scored, packed for the second product
  [[maybe_unused]] Frag8 pl[kSplitP ? 4 : 1], pll[kSplitP ? 4 : 1];  // what the rounding of pb left, and of that

  // O^T += V^T . P^T for the tile whose P^T is in pb.  The first eight V^T fragments are asked
  // for ahead of the softmax (pv_fetch), so that their LDS latency is not waited for here.
  bf16x8 vf[8];
  auto pv_fetch = [&](auto parity) {
    const uint16_t *Vt = Vs + decltype(parity)::value * kTileE;
#pragma unroll
    for (int i = 0; i < 8; ++i) vf[i] = vfrag(Vt, i % kNb, i / kNb);
  };
  auto do_pv = [&](auto parity) {
    const uint16_t *Vt = Vs + decltype(parity)::value * kTileE;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int dblk = 0; dblk < kNb; ++dblk) {
        const int i = kNb * ks + dblk, slot = i & 7;
        oacc[dblk] = mfma32(vf[slot], pb[ks].v, oacc[dblk]);
        if constexpr (kSplitP) {
          oacc[dblk] = mfma32(vf[slot], pl[ks].v, oacc[dblk]);
          oacc[dblk] = mfma32(vf[slot], pll[ks].v, oacc[dblk]);
        }
        if (i + 8 < 4 * kNb) vf[slot] = vfrag(Vt, dblk, ks + 2);
      }
  };

  // S^T = K . Q^T and the online softmax for the tile in the current K buffer; leaves P^T in pb.
  auto do_qk_softmax = [&](bool is_state, int row0, int64_t p0, auto parity) {
    const uint16_t *Kt = Ks + decltype(parity)::value * kTileE;
    const float scale = is_state ? c_state : c_bswa;
    const bool need_mask = is_state ? (m - row0 < kTileKeys) : (p0 + kTileKeys - 1 > cs + wq0);
    f32x16 sacc[2];
    // a rolling window of eight K fragments in flight from LDS, so that a matrix instruction does
    // not wait for the read issued just before it
    {
      bf16x8 kf[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) kf[i] = kfrag(Kt, i & 1, i >> 1);
      const f32x16 zero = {0.f};
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks) {
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
          const int slot = (2 * ks + blk) & 7;
          sacc[blk] = mfma32(kf[slot], qreg[ks], ks == 0 ? zero : sacc[blk]);
          if (ks + 4 < kKs) kf[slot] = kfrag(Kt, blk, ks + 4);
        }
      }
      // pin that order: 8 LDS reads up front, then one read behind every matrix instruction
      __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
      if constexpr (kKs > 4) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
    }
    pv_fetch(parity);
    if (need_mask) {
      // keys up to `lim` (tile-local) are visible to this lane's query
      const int lim = is_state ? (m - row0 - 1) : (int)(cs + myq - p0);
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          sacc[blk][v] = (32 * blk + mfma_row(v, g)) <= lim ? sacc[blk][v] : -INFINITY;
    }
    float smax = sacc[0][0];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int v = 0; v < 16; ++v) smax = fmaxf(smax, sacc[blk][v]);
    smax = xhalf_max(smax);  // the other lane half holds the other 32 keys of the same query
    // m_run is the reference point of the exponentials rather than the running maximum itself: it
    // moves, and what is accumulated is rescaled, only when the maximum of some query of the wave
    // has risen more than kSlack (log2 units) above it.  Until then p = 2^(s - m_run) may exceed
    // 1, by at most 2^kSlack: harmless in fp32 and in bf16 (same relative precision at any
    // magnitude), and the division by the sum, taken against the same reference, is unchanged.
    // Some maximum among 32 queries creeps up in most tiles; a jump of this size is rare after
    // the first.
    constexpr float kSlack = 8.f;
    const float m_new = fmaxf(m_run, smax * scale);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run + kSlack) != 0) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_part *= alpha;
#pragma unroll
      for (int i = 0; i < kNb; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[i][v] *= alpha;
    }
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sacc[blk][v] = __builtin_amdgcn_exp2f(fmaf(sacc[blk][v], scale, -m_run));
      }
    // The row sum is taken over the probabilities as rounded to bf16 for the second product, two
    // per instruction (v_dot2c_f32_bf16 with a pair of ones): numerator and denominator of the
    // output then see the same rounded values.
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = sacc[ks >> 1][(ks & 1) * 8 + 2 * e], p1 = sacc[ks >> 1][(ks & 1) * 8 + 2 * e + 1];
        pb[ks].w[e] = pack_bf16(p0, p1);
        if constexpr (kSplitP) {
          auto rest = [](float x, float y, uint32_t w, float &rx, float &ry) {   // exact
            rx = x - __uint_as_float(w << 16);
            ry = y - __uint_as_float(w & 0xffff0000u);
          };
          float r0, r1;
          rest(p0, p1, pb[ks].w[e], r0, r1);
          pl[ks].w[e] = pack_bf16(r0, r1);
          rest(r0, r1, pl[ks].w[e], r0, r1);
          pll[ks].w[e] = pack_bf16(r0, r1);
          l_part += p0 + p1;
        } else {
          l_part = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pb[ks].w[e]), ones, l_part, false);
        }
      }
  };

  // One barrier per tile: it publishes tile `it` (every wave has waited for its own share of the
  // loads) and frees the buffers of tile it - 1 for the loads of tile it + 1.  (Measured and
  // dropped: a second barrier per tile that lets K and V loads run a tile and a half ahead, and
  // touching the lines of later tiles to pull them into L2 early; neither beat this loop.)
  bool q_negated = false;
  // Q^T is in registers from here on: said explicitly, or the compiler, which does not count the
  // tile loads, would wait for "its" loads inside the loop and drain the tile loads with them
  __builtin_amdgcn_s_waitcnt(0);
  issue_tile(0);
  // One tile; the buffer pair it lives in (tile number mod 2) is a compile-time constant, so
  // that the buffer's offset folds into the LDS instructions instead of costing address updates.
  auto tile_step = [&](int it, auto parity) {
    const bool is_state = it < n_st;
    if (((neg_bits & (is_state ? 1 : 2)) != 0) != q_negated) {
      asm volatile("" ::: "memory");  // stays a (rarely taken) branch
      q_negated = !q_negated;
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks) {
        Frag8 f;
        f.v = qreg[ks];
#pragma unroll
        for (int e = 0; e < 4; ++e) f.w[e] ^= 0x80008000u;
        qreg[ks] = f.v;
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (it + 1 < n_tiles) issue_tile(it + 1);
    const int64_t p0 = wb + (int64_t)(it - n_st) * kTileKeys;
    // skip tiles whose keys all lie after this wave's queries
    if (is_state || p0 <= cs + wq0 + 31) {
      do_qk_softmax(is_state, it * kTileKeys, p0, parity);
      do_pv(parity);
    }
  };
  for (int it = 0; it < n_tiles; it += 2) {
    tile_step(it, std::integral_constant<int, 0>{});
    if (it + 1 < n_tiles) tile_step(it + 1, std::integral_constant<int, 1>{});
  }
  float l = xhalf_sum(l_part);
  if constexpr (kSplitP) {
    // A key that a query does not see enters the second product with p = 0, and a value that is not finite makes that
    // NaN; so does the rest of a split p, 0, with a value the query sees.  A query whose result is not
    // finite is therefore done again, one visible key after the other, in fp32.
    float bad = 0.f * l;
#pragma unroll
    for (int i = 0; i < kNb; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) bad = fmaf(oacc[i][v], 0.f, bad);
    if (myq < nq && !(xhalf_sum(bad) == 0.f)) {
      KeyWalk w;
      w.khat = khat; w.vhat = vhat; w.ring_k = ring_k; w.ring_v = ring_v; w.in_k = in_k; w.in_v = in_v;
      w.kst = kst_in; w.vst = vst_in; w.m = m; w.wrel = wrel; w.t0rel = t0rel; w.ring_slot0 = ring_slot0; w.L = dv.L;
      w.c_state = neg_bits & 1 ? -c_state : c_state;
      w.c_bswa = neg_bits & 2 ? -c_bswa : c_bswa;
      const char *qrow = (const char *)((const uint16_t *)a.q + b * a.q_b + ((int64_t)ci * dv.C + myq) * a.q_t + hq * a.q_h);
      attend_one_by_one<D>(w, qrow, m + (int)(cs + myq - wb) + 1, g, oacc, m_run, l);
    }
  }
  if (myq < nq) {
    const float inv = 1.f / l;
    uint16_t *orow = (uint16_t *)a.out + b * a.o_b + ((int64_t)ci * dv.C + myq) * a.o_t + hq * a.o_h;
#pragma unroll
    for (int dblk = 0; dblk < kNb; ++dblk)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const uint32_t lo = pack_bf16(oacc[dblk][4 * vq] * inv, oacc[dblk][4 * vq + 1] * inv);
        const uint32_t hi = pack_bf16(oacc[dblk][4 * vq + 2] * inv, oacc[dblk][4 * vq + 3] * inv);
        *reinterpret_cast<uint2 *>(orow + 32 * dblk + 8 * vq + 4 * g) = make_uint2(lo, hi);
      }
    if (a.lse && g == 0)
      a.lse[b * a.lse_b + ((int64_t)ci * dv.C + myq) * a.lse_t + hq * a.lse_h] = (m_run + log2f(l)) * kLn2;
  }
}

// Static LDS: 2 K + 2 V tile buffers = 64 KiB, two workgroups per CU.
__global__ __launch_bounds__(256, 2) void attn_mfma_kernel_q128(Dev dv, AttnArgs a) {
  __shared__ __attribute__((aligned(32768))) uint16_t Ks[2 * kTileElems];
  __shared__ __attribute__((aligned(1024))) uint16_t Vs[2 * kTileElems];
  attn_body<4, 128>(dv, a, Ks, Vs);
}

// head_dim 64.  Probabilities enter the second product as three bf16 numbers, 3 x 8 bits = the 24 of an fp32
// significand, and their sum is taken in fp32: the row kernel, which these states used for prompts too,
// keeps p in fp32, and the result is as close to 64-bit arithmetic as that kernel's.  What bounds it
// at the sizes it is used for (a few heads, a launch per chunk) is the latency of the tile loop, so the extra matrix
// instructions hardly show.  Two prompts of 4173 tokens, 16 heads on 4, 256-token chunks:
// 19 us a chunk beside the folds (97 by the row kernel); the call 1.72 ms before, 0.90 now (scoring launches of the
// folds, 47 to 8 us, included).
__global__ __launch_bounds__(256, 2) void attn_mfma_kernel_d64(Dev dv, AttnArgs a) {
  __shared__ __attribute__((aligned(16384))) uint16_t Ks[kTileElems];
  __shared__ __attribute__((aligned(1024))) uint16_t Vs[kTileElems];
  attn_body<4, 64>(dv, a, Ks, Vs);
}

template <int N>
__device__ __forceinline__ void wait_loads() {   // until N of this wave's loads are under way
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// ------------------------------------------------------------------------------------------------
// head_dim 128, launches of few queries: the four waves of a workgroup take the same 32 queries of one head and four
// tiles of 64 keys at a time.  Each wave scores a tile (first product, maximum, exponentials) and leaves P^T in LDS in the
// second product's operand layout; then each wave adds all four tiles, in order, to a quarter of the channels.  The
// reference point of the exponentials moves tile by tile as in the tile kernel, decided by every wave from the
// tiles' maxima, and the sums are added up in the same order: the results have that kernel's bits, so a
// sequence's do not depend on the batch it is in.
// What bounds it: latencies, 1.2 us for four tiles where a workgroup of the tile kernel, alone on its compute unit, takes
// some 1.6 us for each.  A wave's K tile and its channels of the four V tiles are its own (no barrier
// but the two of the exchange); K of the next four is asked for as soon as the first product has read
// this one's, V as soon as the second has.
constexpr int kQuadK = 4 * kTileElems, kQuadV = 4 * 4 * kTileKeys * 32, kQuadP = 4 * 4 * 64 * 8;   // elements
constexpr int kQuadLds = (kQuadK + kQuadV + kQuadP) * 2 + 4 * 32 * 4;

__global__ __launch_bounds__(256, 2) void attn_quad_kernel_d128(Dev dv, AttnArgs a) {
  extern __shared__ __attribute__((aligned(1024))) uint16_t lds[];
  constexpr int D = 128;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  // workgroup -> work item as in the tile kernel, a member being 32 positions of one head
  const int Gq = dv.Hq / dv.Hkv, tpc = dv.C / 32;
  const int per_group = tpc * Gq;
  const int n_groups = a.n_chunks * dv.Hkv * dv.B;
  const int xcd = blockIdx.x % kXcds, seq = blockIdx.x / kXcds;
  const int group = (seq / per_group) * kXcds + xcd;
  if (group >= n_groups) return;
  const int member = seq % per_group;
  const int ci = group % a.n_chunks;
  const int hkv = (group / a.n_chunks) % dv.Hkv;
  const int b = group / (a.n_chunks * dv.Hkv);
  const int hq = __builtin_amdgcn_readfirstlane(hkv * Gq + member / tpc);
  const int u = b * dv.Hkv + hkv;
  const int Q0 = (tpc - 1 - member % tpc) * 32;                          // longest causal part first
  const int nq = ci == a.n_chunks - 1 ? a.nq_total - ci * dv.C : dv.C;
  if (Q0 >= nq) return;
  const int64_t cs = a.s + (int64_t)ci * dv.C;
  const int64_t wb = cs + dv.C - dv.L > 0 ? cs + dv.C - dv.L : 0;
  const int myq = Q0 + l32, m = a.m[ci];
  auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  auto uni_ptr = [](const char *p_) {
    const uint64_t x = (uint64_t)p_;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return (const char *)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  KeyWalk w;
  w.khat = uni_ptr((const char *)dv.khat + (a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D) * 2);
  w.vhat = uni_ptr((const char *)dv.vhat + (a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D) * 2);
  w.ring_k = uni_ptr((const char *)dv.winK + (int64_t)u * dv.L * D * 2);
  w.ring_v = uni_ptr((const char *)dv.winV + (int64_t)u * dv.L * D * 2);
  w.kst = (uint32_t)uni((int)(a.in.k_t * 2));
  w.vst = (uint32_t)uni((int)(a.in.v_t * 2));
  w.in_k = uni_ptr((const char *)a.in.k + (b * a.in.k_b + hkv * a.in.k_h + (cs - a.t0) * a.in.k_t) * 2);
  w.in_v = uni_ptr((const char *)a.in.v + (b * a.in.v_b + hkv * a.in.v_h + (cs - a.t0) * a.in.v_t) * 2);
  w.m = m;
  w.wrel = uni((int)(wb - cs));
  w.t0rel = uni(a.t0 - cs < -(1 << 30) ? -(1 << 30) : (int)(a.t0 - cs));
  w.ring_slot0 = uni((int)(wb % dv.L));
  w.L = dv.L;
  const int qend = Q0 + 32 < nq ? Q0 + 32 : nq;
  const int n_st = uni((m + kTileKeys - 1) / kTileKeys);
  const int n_tiles = uni(n_st + (qend - w.wrel + kTileKeys - 1) / kTileKeys);

  uint16_t *Kt = lds + wave * kTileElems;
  uint16_t *Vt = lds + kQuadK + wave * (4 * kTileKeys * 32);   // [tile][key][32 channels]
  uint16_t *Pt = lds + kQuadK + kQuadV;                        // [tile][16 keys][lane][8]
  float *tops = reinterpret_cast<float *>(lds + kQuadK + kQuadV + kQuadP);   // [tile][query]
  const uint32_t k_addr = lds_addr_of(Kt), v_addr = lds_addr_of(Vt);
  uint32_t koff[8];
  ktile_offsets(lane, koff);
  const DmaLane dl = dma_lane(lane);
  // where V^T fragments are read: row 4 g + j / 4 (+ 8), channels 16 half + 4 (j % 4); four rows are a bank cycle
  const uint32_t voff = (uint32_t)((4 * g + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
  struct TileSrc {
    const char *k, *v;
    uint32_t kst, vst;
    int valid;
  };
  auto tile_src = [&](int it) {
    TileSrc t;
    if (it < n_st) {
      t.k = w.khat + (uint32_t)(it * kTileKeys) * (D * 2);
      t.v = w.vhat + (uint32_t)(it * kTileKeys) * (D * 2);
      t.kst = t.vst = D * 2;
      t.valid = m - it * kTileKeys;
    } else {
      const int prel = w.wrel + (it - n_st) * kTileKeys;
      t.valid = nq - prel;
      if (prel >= w.t0rel) {
        t.k = w.in_k + (int64_t)prel * (int64_t)w.kst;
        t.v = w.in_v + (int64_t)prel * (int64_t)w.vst;
        t.kst = w.kst;
        t.vst = w.vst;
      } else {
        int slot = w.ring_slot0 + (it - n_st) * kTileKeys;
        slot = slot >= dv.L ? slot - dv.L : slot;   // a window is at most L long: one wrap
        t.k = w.ring_k + (uint32_t)slot * (D * 2);
        t.v = w.ring_v + (uint32_t)slot * (D * 2);
        t.kst = t.vst = D * 2;
      }
    }
    return t;
  };
  auto issue_k = [&](int it) {   // 16 loads
    const TileSrc t = tile_src(it);
#pragma unroll
    for (int q = 0; q < 4; ++q) tile_dma<false, 4>(t.k, t.kst, t.valid, k_addr, q, dl);
  };
  auto issue_v = [&](int it0) {   // 16 loads: this wave's channels of four tiles (of the last one, where there are fewer)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const TileSrc t = tile_src(it0 + i < n_tiles ? it0 + i : n_tiles - 1);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        int r = 16 * n + (lane >> 2);
        r = r < t.valid ? r : t.valid - 1;
        dma16(t.v, (uint32_t)r * t.vst + (uint32_t)(64 * wave + 16 * (lane & 3)), v_addr + (uint32_t)(4 * i + n) * 1024u);
      }
    }
  };
  issue_k(wave < n_tiles ? wave : n_tiles - 1);   // (a wave without a tile: loads to count, not read)
  issue_v(0);
  const char *qrow = (const char *)((const uint16_t *)a.q + b * a.q_b +
                                    ((int64_t)ci * dv.C + (myq < nq ? myq : nq - 1)) * a.q_t + hq * a.q_h);
  bf16x8 qreg[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    Frag8 f;
    f.q = *reinterpret_cast<const uint4 *>(qrow + 32 * ks + 16 * g);
    qreg[ks] = f.v;
  }
  const float rs = kLog2e * rsqrtf((float)D);
  w.c_state = (dv.tau_state ? dv.tau_state[hq] : 1.f) * rs;
  w.c_bswa = (dv.tau_bswa ? dv.tau_bswa[hq] : 1.f) * rs;
  const int neg_bits = uni((w.c_state < 0.f ? 1 : 0) | (w.c_bswa < 0.f ? 2 : 0));   // as in the tile kernel
  __builtin_amdgcn_s_waitcnt(0);   // no load that the compiler counts is under way in the loop

  f32x16 oacc = {0.f};
  float m_run = -INFINITY, l_part = 0.f;
  bool q_negated = false;
#pragma unroll 1
  for (int it0 = 0; it0 < n_tiles; it0 += 4) {
    const int it = it0 + wave;
    const bool mine = it < n_tiles, more = it0 + 4 < n_tiles, is_state = it < n_st;
    if (((neg_bits & (is_state ? 1 : 2)) != 0) != q_negated) {
      asm volatile("" ::: "memory");  // stays a (rarely taken) branch
      q_negated = !q_negated;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        Frag8 f;
        f.v = qreg[ks];
#pragma unroll
        for (int e = 0; e < 4; ++e) f.w[e] ^= 0x80008000u;
        qreg[ks] = f.v;
      }
    }
    wait_loads<16>();   // K is there; V, asked for after it, may still be under way
    f32x16 sacc[2];
    float smax = -INFINITY;
    const float scale = fabsf(is_state ? w.c_state : w.c_bswa);
    if (mine) {
      bf16x8 kf[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) kf[i] = ktile_frag(Kt, koff, i & 1, i >> 1);
      const f32x16 zero = {0.f};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) sacc[blk] = mfma32(kf[2 * ks + blk], qreg[ks], ks == 0 ? zero : sacc[blk]);
    }
    wait_lds();
    if (more) issue_k(it + 4 < n_tiles ? it + 4 : n_tiles - 1);
    if (mine) {
      const int row0 = it * kTileKeys, prel = w.wrel + (it - n_st) * kTileKeys;
      if (is_state ? m - row0 < kTileKeys : prel + kTileKeys - 1 > Q0) {
        const int lim = is_state ? m - row0 - 1 : myq - prel;   // keys up to it are visible to the lane's query
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
#pragma unroll
          for (int v = 0; v < 16; ++v) sacc[blk][v] = (32 * blk + mfma_row(v, g)) <= lim ? sacc[blk][v] : -INFINITY;
      }
      smax = sacc[0][0];
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int v = 0; v < 16; ++v) smax = fmaxf(smax, sacc[blk][v]);
      smax = xhalf_max(smax);
      if (g == 0) tops[wave * 32 + l32] = smax * scale;
    }
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // the reference point after each of the four tiles, and what is accumulated is multiplied by ahead of it
    constexpr float kSlack = 8.f;   // as in the tile kernel
    float alpha[4], m_mine = m_run;
    int moved = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      alpha[t] = 1.f;
      if (it0 + t < n_tiles) {
        const float m_new = fmaxf(m_run, tops[t * 32 + l32]);
        if (__builtin_amdgcn_ballot_w64(m_new > m_run + kSlack) != 0) {
          alpha[t] = __builtin_amdgcn_exp2f(m_run - m_new);
          m_run = m_new;
          moved |= 1 << t;
        }
      }
      if (t == wave) m_mine = m_run;
    }
    if (mine) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        Frag8 p;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int v = (ks & 1) * 8 + 2 * e;
          p.w[e] = pack_bf16(__builtin_amdgcn_exp2f(fmaf(sacc[ks >> 1][v], scale, -m_mine)),
                             __builtin_amdgcn_exp2f(fmaf(sacc[ks >> 1][v + 1], scale, -m_mine)));
        }
        *reinterpret_cast<uint4 *>(Pt + ((wave * 4 + ks) * 64 + lane) * 8) = p.q;
      }
    }
    if (more) wait_loads<16>(); else wait_loads<0>();   // V is there
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (it0 + t < n_tiles) {
        Frag8 p[4];
        bf16x8 vf[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          p[ks].q = *reinterpret_cast<const uint4 *>(Pt + ((t * 4 + ks) * 64 + lane) * 8);
          const uint16_t *vp = Vt + (t * kTileKeys + 16 * ks) * 32 + voff;
          Frag8 f;
          f.d[0] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(KVM_LDS_V4(vp)));
          f.d[1] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(KVM_LDS_V4(vp + 8 * 32)));
          vf[ks] = f.v;
        }
        if (moved & (1 << t)) {
          l_part *= alpha[t];
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[v] *= alpha[t];
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          oacc = mfma32(vf[ks], p[ks].v, oacc);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            l_part = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[ks].w[e]), ones, l_part, false);
        }
      }
    }
    wait_lds();
    if (more) issue_v(it0 + 4);
  }
  const float l = xhalf_sum(l_part);
  if (myq < nq) {
    const float inv = 1.f / l;
    uint16_t *orow = (uint16_t *)a.out + b * a.o_b + ((int64_t)ci * dv.C + myq) * a.o_t + hq * a.o_h;
#pragma unroll
    for (int vq = 0; vq < 4; ++vq)
      *reinterpret_cast<uint2 *>(orow + 32 * wave + 8 * vq + 4 * g) =
          make_uint2(pack_bf16(oacc[4 * vq] * inv, oacc[4 * vq + 1] * inv), pack_bf16(oacc[4 * vq + 2] * inv, oacc[4 * vq + 3] * inv));
    if (a.lse && wave == 0 && g == 0)
      a.lse[b * a.lse_b + ((int64_t)ci * dv.C + myq) * a.lse_t + hq * a.lse_h] = (m_run + log2f(l)) * kLn2;
  }
}

// ------------------------------------------------------------------------------------------------
// head_dim 64, launches of few queries: the four waves of a workgroup take the same 32 queries of one head and every
// fourth tile of 32 keys each, and put their results together at the end.  Four times as many
// workgroups as above, a quarter of the tiles in a row: what bounds such a launch is that chain (a wave alone on its SIMD
// takes two thirds of a 64-key tile's time for latencies).  A wave has its tiles to itself (no
// barriers in the loop), one K and one V buffer: K of the next tile is asked for as soon as the first
// product has read this one's, V as soon as the second has.
__device__ __forceinline__ void attn_split_d64(const Dev &dv, const AttnArgs &a, uint16_t *tiles, float2 *sh_ml, int *sh_bad) {
  constexpr int D = 64, kKs = D / 16, kNb = D / 32, kTK = 32, kTileE = kTK * D, kLoads = kTileE * 2 / 1024;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  // workgroup -> work item as above, a member being 32 positions of one head
  const int Gq = dv.Hq / dv.Hkv, tpc = dv.C / 32;
  const int per_group = tpc * Gq;
  const int n_groups = a.n_chunks * dv.Hkv * dv.B;
  const int xcd = blockIdx.x % kXcds, seq = blockIdx.x / kXcds;
  const int group = (seq / per_group) * kXcds + xcd;
  if (group >= n_groups) return;
  const int member = seq % per_group;
  const int ci = group % a.n_chunks;
  const int hkv = (group / a.n_chunks) % dv.Hkv;
  const int b = group / (a.n_chunks * dv.Hkv);
  const int hq = __builtin_amdgcn_readfirstlane(hkv * Gq + member / tpc);
  const int u = b * dv.Hkv + hkv;
  const int Q0 = (tpc - 1 - member % tpc) * 32;                          // longest causal part first
  const int nq = ci == a.n_chunks - 1 ? a.nq_total - ci * dv.C : dv.C;
  if (Q0 >= nq) return;
  const int64_t cs = a.s + (int64_t)ci * dv.C;
  const int64_t wb = cs + dv.C - dv.L > 0 ? cs + dv.C - dv.L : 0;
  const int myq = Q0 + l32, m = a.m[ci];
  auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  auto uni_ptr = [](const char *p_) {
    const uint64_t x = (uint64_t)p_;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return (const char *)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  KeyWalk w;
  w.khat = uni_ptr((const char *)dv.khat + (a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D) * 2);
  w.vhat = uni_ptr((const char *)dv.vhat + (a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D) * 2);
  w.ring_k = uni_ptr((const char *)dv.winK + (int64_t)u * dv.L * D * 2);
  w.ring_v = uni_ptr((const char *)dv.winV + (int64_t)u * dv.L * D * 2);
  w.kst = (uint32_t)uni((int)(a.in.k_t * 2));
  w.vst = (uint32_t)uni((int)(a.in.v_t * 2));
  w.in_k = uni_ptr((const char *)a.in.k + (b * a.in.k_b + hkv * a.in.k_h + (cs - a.t0) * a.in.k_t) * 2);
  w.in_v = uni_ptr((const char *)a.in.v + (b * a.in.v_b + hkv * a.in.v_h + (cs - a.t0) * a.in.v_t) * 2);
  w.m = m;
  w.wrel = uni((int)(wb - cs));
  w.t0rel = uni(a.t0 - cs < -(1 << 30) ? -(1 << 30) : (int)(a.t0 - cs));
  w.ring_slot0 = uni((int)(wb % dv.L));
  w.L = dv.L;
  const int qend = Q0 + 32 < nq ? Q0 + 32 : nq;
  const int n_st = uni((m + kTK - 1) / kTK);
  const int n_tiles = uni(n_st + (qend - w.wrel + kTK - 1) / kTK);

  uint32_t koff[kKs], voff[kNb];
  ktile_offsets64(lane, koff);
  vtile_offsets64(lane, voff);
  const DmaLane64 dl = dma_lane64(lane);
  uint16_t *Kt = tiles + wave * 2 * kTileE, *Vt = Kt + kTileE;
  const uint32_t k_addr = lds_addr_of(Kt), v_addr = lds_addr_of(Vt);
  // 32 rows of a tile, all of them by this wave; rows beyond the last repeat it
  auto load_tile = [&](const char *base, uint32_t stride, int valid, uint32_t at, auto vswz) {
    constexpr bool kV = decltype(vswz)::value;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      int r = 8 * n + (int)dl.rl;
      r = r < valid ? r : valid - 1;
      dma16(base, (uint32_t)r * stride + (kV ? dl.vcol : dl.kcol[n & 1]), at + (uint32_t)n * 1024u);
    }
  };
  auto issue = [&](int it, auto values) {
    constexpr bool kV = decltype(values)::value;
    const uint32_t at = kV ? v_addr : k_addr;
    if (it < n_st) {
      load_tile((kV ? w.vhat : w.khat) + (uint32_t)(it * kTK) * (D * 2), D * 2, m - it * kTK, at, values);
    } else {
      const int prel = w.wrel + (it - n_st) * kTK, valid = nq - prel;
      if (prel >= w.t0rel) {
        const uint32_t st = kV ? w.vst : w.kst;
        load_tile((kV ? w.in_v : w.in_k) + (int64_t)prel * (int64_t)st, st, valid, at, values);
      } else {
        int slot = w.ring_slot0 + (it - n_st) * kTK;
        slot = slot >= dv.L ? slot - dv.L : slot;   // a window is at most L long: one wrap
        load_tile((kV ? w.ring_v : w.ring_k) + (uint32_t)slot * (D * 2), D * 2, valid, at, values);
      }
    }
  };
  using Keys = std::integral_constant<bool, false>;
  using Values = std::integral_constant<bool, true>;
  if (wave < n_tiles) {   // the first tile and the queries travel together
    issue(wave, Keys{});
    issue(wave, Values{});
  }
  const char *qrow = (const char *)((const uint16_t *)a.q + b * a.q_b +
                                    ((int64_t)ci * dv.C + (myq < nq ? myq : nq - 1)) * a.q_t + hq * a.q_h);
  bf16x8 qreg[kKs];
#pragma unroll
  for (int ks = 0; ks < kKs; ++ks) {
    Frag8 f;
    f.q = *reinterpret_cast<const uint4 *>(qrow + 32 * ks + 16 * g);
    qreg[ks] = f.v;
  }
  const float rs = kLog2e * rsqrtf((float)D);
  w.c_state = (dv.tau_state ? dv.tau_state[hq] : 1.f) * rs;
  w.c_bswa = (dv.tau_bswa ? dv.tau_bswa[hq] : 1.f) * rs;
  const int neg_bits = uni((w.c_state < 0.f ? 1 : 0) | (w.c_bswa < 0.f ? 2 : 0));   // as above
  if (tid < 32) sh_bad[tid] = 0;
  __builtin_amdgcn_s_waitcnt(0);   // no load that the compiler counts is under way in the loop

  f32x16 oacc[kNb];
#pragma unroll
  for (int i = 0; i < kNb; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[i][v] = 0.f;
  float m_run = -INFINITY, l_part = 0.f;
  bool q_negated = false;
  for (int it = wave; it < n_tiles; it += 4) {
    const bool is_state = it < n_st, more = it + 4 < n_tiles;
    if (((neg_bits & (is_state ? 1 : 2)) != 0) != q_negated) {
      asm volatile("" ::: "memory");  // stays a (rarely taken) branch
      q_negated = !q_negated;
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks) {
        Frag8 f;
        f.v = qreg[ks];
#pragma unroll
        for (int e = 0; e < 4; ++e) f.w[e] ^= 0x80008000u;
        qreg[ks] = f.v;
      }
    }
    wait_loads<kLoads>();   // K is there; V, asked for after it, may still be under way
    f32x16 sacc = {0.f};
    {
      bf16x8 kf[kKs];
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks) kf[ks] = ktile_frag64(Kt, koff, 0, ks);
      wait_lds();
      if (more) issue(it + 4, Keys{});
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks) sacc = mfma32(kf[ks], qreg[ks], sacc);
    }
    const int prel = w.wrel + (it - n_st) * kTK;
    const int lim = is_state ? m - it * kTK - 1 : myq - prel;   // keys up to it are visible to the lane's query
    if (is_state ? m - it * kTK < kTK : prel + kTK - 1 > Q0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sacc[v] = mfma_row(v, g) <= lim ? sacc[v] : -INFINITY;
    }
    const float scale = fabsf(is_state ? w.c_state : w.c_bswa);
    float smax = sacc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) smax = fmaxf(smax, sacc[v]);
    smax = xhalf_max(smax);
    constexpr float kSlack = 8.f;   // as above
    const float m_new = fmaxf(m_run, smax * scale);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run + kSlack) != 0) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_part *= alpha;
#pragma unroll
      for (int i = 0; i < kNb; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[i][v] *= alpha;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[v] = __builtin_amdgcn_exp2f(fmaf(sacc[v], scale, -m_run));
    Frag8 pb[2], pl[2], pll[2];   // P as the sum of three bf16 numbers, as above
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = sacc[ks * 8 + 2 * e], p1 = sacc[ks * 8 + 2 * e + 1];
        auto rest = [](float x, float y, uint32_t ww, float &rx, float &ry) {   // exact
          rx = x - __uint_as_float(ww << 16);
          ry = y - __uint_as_float(ww & 0xffff0000u);
        };
        float r0, r1;
        pb[ks].w[e] = pack_bf16(p0, p1);
        rest(p0, p1, pb[ks].w[e], r0, r1);
        pl[ks].w[e] = pack_bf16(r0, r1);
        rest(r0, r1, pl[ks].w[e], r0, r1);
        pll[ks].w[e] = pack_bf16(r0, r1);
        l_part += p0 + p1;
      }
    if (more) wait_loads<kLoads>(); else wait_loads<0>();   // V is there
    bf16x8 vf[2][kNb];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dblk = 0; dblk < kNb; ++dblk) vf[ks][dblk] = vtile_frag64(Vt, voff, dblk, ks);
    wait_lds();
    if (more) issue(it + 4, Values{});
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dblk = 0; dblk < kNb; ++dblk) {
        oacc[dblk] = mfma32(vf[ks][dblk], pb[ks].v, oacc[dblk]);
        oacc[dblk] = mfma32(vf[ks][dblk], pl[ks].v, oacc[dblk]);
        oacc[dblk] = mfma32(vf[ks][dblk], pll[ks].v, oacc[dblk]);
      }
  }

  // The four results: a wave's own go where its tiles were (as many bytes: 32 x D floats), and every wave puts a
  // quarter of the channels together.
  float *mine = reinterpret_cast<float *>(Kt);
#pragma unroll
  for (int p = 0; p < 4 * kNb; ++p)
    *reinterpret_cast<float4 *>(mine + (p * 64 + lane) * 4) =
        make_float4(oacc[p >> 2][4 * (p & 3)], oacc[p >> 2][4 * (p & 3) + 1], oacc[p >> 2][4 * (p & 3) + 2],
                    oacc[p >> 2][4 * (p & 3) + 3]);
  {
    const float l_wave = xhalf_sum(l_part);
    if (g == 0) sh_ml[wave * 32 + l32] = make_float2(m_run, l_wave);
  }
  __syncthreads();
  float f[4], top = -INFINITY, l = 0.f;
#pragma unroll
  for (int o = 0; o < 4; ++o) top = fmaxf(top, sh_ml[o * 32 + l32].x);
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const float2 ml = sh_ml[o * 32 + l32];
    f[o] = __builtin_amdgcn_exp2f(ml.x - top);
    l = fmaf(ml.y, f[o], l);
  }
  float4 x[kNb];
#pragma unroll
  for (int i = 0; i < kNb; ++i) {
    const int p = wave * kNb + i;
    x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      const float4 y = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(tiles + o * 2 * kTileE) + (p * 64 + lane) * 4);
      x[i].x = fmaf(y.x, f[o], x[i].x);
      x[i].y = fmaf(y.y, f[o], x[i].y);
      x[i].z = fmaf(y.z, f[o], x[i].z);
      x[i].w = fmaf(y.w, f[o], x[i].w);
    }
  }
  uint16_t *orow = (uint16_t *)a.out + b * a.o_b + ((int64_t)ci * dv.C + myq) * a.o_t + hq * a.o_h;
  auto store4 = [&](int p, float x0, float x1, float x2, float x3, float inv) {
    *reinterpret_cast<uint2 *>(orow + 32 * (p >> 2) + 8 * (p & 3) + 4 * g) =
        make_uint2(pack_bf16(x0 * inv, x1 * inv), pack_bf16(x2 * inv, x3 * inv));
  };
  // a query whose result is not finite, as above: the first wave does it again
  float bad = 0.f * l;
#pragma unroll
  for (int i = 0; i < kNb; ++i) bad = fmaf(x[i].x, 0.f, fmaf(x[i].y, 0.f, fmaf(x[i].z, 0.f, fmaf(x[i].w, 0.f, bad))));
  if (!(bad == 0.f)) sh_bad[l32] = 1;
  __syncthreads();
  const bool again = sh_bad[l32] != 0;
  if (myq < nq && !again) {
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < kNb; ++i) store4(wave * kNb + i, x[i].x, x[i].y, x[i].z, x[i].w, inv);
  }
  if (wave == 0 && again && myq < nq) {
    attend_one_by_one<D>(w, qrow, m + myq - w.wrel + 1, g, oacc, top, l);
    const float inv = 1.f / l;
#pragma unroll
    for (int p = 0; p < 4 * kNb; ++p)
      store4(p, oacc[p >> 2][4 * (p & 3)], oacc[p >> 2][4 * (p & 3) + 1], oacc[p >> 2][4 * (p & 3) + 2],
             oacc[p >> 2][4 * (p & 3) + 3], inv);
  }
  if (a.lse && wave == 0 && g == 0 && myq < nq)
    a.lse[b * a.lse_b + ((int64_t)ci * dv.C + myq) * a.lse_t + hq * a.lse_h] = (top + log2f(l)) * kLn2;
}

__global__ __launch_bounds__(256, 2) void attn_split_kernel_d64(Dev dv, AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t tiles[4 * 2 * 32 * 64];
  __shared__ float2 ml[4 * 32];
  __shared__ int bad[32];
  attn_split_d64(dv, a, tiles, ml, bad);
}
// The same with the scores of the block that is folded after the chunk in further workgroups (attn_rows_score_kernel).  Here
// attention is the longer part and goes first: the call above 338 us, 365 the other way round.
__global__ __launch_bounds__(256, 2) void attn_split_score_kernel_d64(Dev dv, AttnArgs a, int n_att, int slot, int m) {
  __shared__ __attribute__((aligned(1024))) uint16_t tiles[4 * 2 * 32 * 64];
  __shared__ float2 ml[4 * 32];
  __shared__ int bad[32];
  if ((int)blockIdx.x < n_att) {
    attn_split_d64(dv, a, tiles, ml, bad);
  } else {
    const int id = (int)blockIdx.x - n_att, per_unit = (dv.C + 3) / 4;
    score_tokens<bf16_t, 64>(dv, slot, 0, m, 1, id % per_unit, id / per_unit);
  }
}

}  // namespace

// Launches of up to so many workgroups of the tile kernels go to the others: as many of theirs, four times the number, as find a
// place at once.  head_dim 128 (one per compute unit), us per call, tiles / four at a time: 64 workgroups: 3 x 8 heads on 2,
// 904 tokens 105 / 90; 4 heads, 4000 tokens 297 / 290; but 128: 2 x 16 heads, 612 tokens 41.7 / 44.4, 256: 8 x 8 heads on 2, 587 tokens
// 40 / 57.  head_dim 64 (two and more per compute unit; with the scores of the fold in the same launch), 4173 tokens: 64 workgroups: 2 x 16 heads on
// 4 655 / 338, 96: the same in 384-token blocks 519 / 387, 128: in 512-token blocks 495 / 375, 4 x 16 heads on 4 714 / 530, with 1000
// rows 1312 / 1059, 4 x 16 heads 1446 / 1270; but 256: 8 x 16 heads, 2000 tokens 470 / 483.
constexpr unsigned kQuadMost = 64, kSplitMost = 128;

// Workgroups of the tile kernels (four heads x 32 positions, or 128 positions of one head, each) and of the others.
static unsigned tile_workgroups(const Dev &dv, const AttnArgs &a, unsigned *of_32) {
  const int Gq = dv.Hq / dv.Hkv;
  const bool by_head = Gq % 4 == 0;
  const int span = by_head ? 32 : 128;
  const int per_group = ((dv.C + span - 1) / span) * (by_head ? Gq / 4 : Gq);
  const int n_groups = (a.n_chunks * dv.Hkv * dv.B + kXcds - 1) / kXcds * kXcds;
  *of_32 = (unsigned)(n_groups * (dv.C / 32) * Gq);
  return (unsigned)(n_groups * per_group);
}

bool attention_takes_scores(const Dev &dv, const AttnArgs &a, int m) {
  if (!attention_on_mfma(dv)) return attn_rows_take_scores(dv, a, m);
  unsigned of_32;
  return dv.d == 64 && tile_workgroups(dv, a, &of_32) <= kSplitMost;
}

hipError_t launch_attn_score(const Dev &dv, const AttnArgs &a, int slot, int m, hipStream_t st) {
  if (!attention_on_mfma(dv)) return launch_attn_rows_score(dv, a, slot, m, st);
  unsigned of_32;
  (void)tile_workgroups(dv, a, &of_32);
  const dim3 grid(of_32 + (unsigned)((dv.C + 3) / 4 * dv.U));
  hipLaunchKernelGGL(attn_split_score_kernel_d64, grid, dim3(256), 0, st, dv, a, (int)of_32, slot, m);
  return hipGetLastError();
}

hipError_t launch_attn_mfma(const Dev &dv, const AttnArgs &a, bool beside_folds, hipStream_t st) {
  static OncePerDevice<hipError_t> of_quad, of_beside;
  if (a.nq_total <= 0) return hipSuccess;
  unsigned of_32;
  const dim3 grid(tile_workgroups(dv, a, &of_32));
  if (dv.d == 128 && grid.x <= kQuadMost && !beside_folds) {
    if (const hipError_t e = allow_lds(of_quad, (const void *)attn_quad_kernel_d128, kQuadLds); e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_quad_kernel_d128, dim3(of_32), dim3(256), kQuadLds, st, dv, a);
  } else if (dv.d == 64 && grid.x <= kSplitMost) {
    hipLaunchKernelGGL(attn_split_kernel_d64, dim3(of_32), dim3(256), 0, st, dv, a);
  } else if (dv.d == 64) {
    hipLaunchKernelGGL(attn_mfma_kernel_d64, grid, dim3(256), 0, st, dv, a);
  } else {
    if (beside_folds)
      if (const hipError_t e = allow_lds(of_beside, (const void *)attn_mfma_kernel_q128, kBesideFoldLds); e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_mfma_kernel_q128, grid, dim3(256), beside_folds ? kBesideFoldLds : 0, st, dv, a);
  }
  return hipGetLastError();
}

}  // namespace kvm
