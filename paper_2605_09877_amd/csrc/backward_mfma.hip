// Attention part of the backward pass for bf16, head_dim 128 on the gfx950 matrix cores.
//
// One kernel body in two roles.  Each wave owns 32 "stationary" vectors and walks "streamed" tiles that
// come through LDS:
//   role dQ: stationary = 32 queries (q and dout rows, in registers as B operands), streamed = keys (64 state
//            rows of the visited version, then window tokens, at a time; K and V rows)   -> dq
//   role KV: stationary = 32 keys (K rows in registers, V rows in LDS), streamed = the chunk's queries, 32 at a
//            time, head after head of the group (q and dout rows)                        -> dk and dv
//            (or the adjoint of the state readout)
// Per 32 streamed rows and wave, with X the streamed "key-like" tile (K or q) and Y the streamed
// "value-like" tile (V or dout):
//   S^T  = X . staK^T           8 matrix instructions (32x32x16)    logits, transposed
//   dP^T = Y . staV^T           8
//   P^T  = exp(tau * scale * S^T - lse),  dS^T = P^T * (dP^T - D)   lse and D belong to the query:
//          to the lane's own column in role dQ, to the row in role KV (then they come from LDS)
//   O1^T += X^T . (tau dS^T)    8       dq^T resp. dk^T
//   O2^T += Y^T . P^T           8       dv^T (role KV)
// Both products that need a streamed tile transposed read it through the transposing LDS load
// from the one swizzled image that the first two products read row by row.  Tiles are filled by
// direct global -> LDS loads one tile ahead, one barrier per tile, like the forward kernel.
//
// What bounds it: matrix and LDS issue, two waves per SIMD.  Role KV carries two results (128 registers) at
// 256 registers a wave; the values moved to LDS, 32-row tiles and offsets made by exclusive or are what
// makes that fit without a spill in the loop.  Two kernels, dk and dv, each with the logits of its own,
// took 233 + 166 us a chunk of the bench workload (one after the other); so did three things inside the loops:
// a load of the temperature per tile, whose wait was a wait for the tile loads too; LDS fragments
// read just ahead of their use; and bank conflicts in every transposing read (half of all LDS cycles).
// Whole backward pass of the bench workload 44.5 ms before, 33.5 now (7 contractions at 790 TFLOP/s, undoing
// the folds included).
#include <type_traits>

#include "kvm_device.h"
#include "kvm_internal.h"
#include "kvm_mfma.h"

namespace kvm {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kXcds = 8;
constexpr int kStaPerWg = 128;                                      // stationary vectors per workgroup (4 waves)
constexpr int kRowScalars = 68;   // role KV, per stage: lse [32], D [32], temperature
constexpr int kBwdTileBytes = 4 * kTileElems * 2 + 2 * 2 * 64 * 4;  // 2 stages x 2 images + row scalars
constexpr int kBwdLdsBytes = kBwdTileBytes + 2 * 4 * kHeadDim * 4;  // + the LN_s parameter sums of role KV

// The tiles are read row by row and transposed: chunk q of row r sits in slot q ^ swz(r),
// swz(r) = 4 * (r & 3) + (r >> 2 & 3), which keeps both reads free of bank conflicts (r & 15, which
// serves the first alone, makes every transposing read take 8 cycles instead of 2).
__device__ __forceinline__ DmaLane dma_lane_both(int lane) {
  DmaLane d;
  const int rl = lane >> 4, c16 = lane & 15;
  d.rl = (uint32_t)rl;
#pragma unroll
  for (int n = 0; n < 4; ++n) d.kcol[n] = (uint32_t)(16 * (c16 ^ (4 * rl + n)));   // row 4 * n + rl (mod 16)
  d.vcol = 0;
  return d;
}
// Row fragments: lane = row lane%32, chunk 2*ks + lane/32 (as ktile_offsets).
__device__ __forceinline__ void rtile_offsets(int lane, uint32_t (&off)[8]) {
  const int l32 = lane & 31, swz = 4 * (l32 & 3) + ((l32 >> 2) & 3);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) off[ks] = (uint32_t)(l32 * kHeadDim + 8 * ((2 * ks + (lane >> 5)) ^ swz));
}
// Transposed (A-operand) fragment: lane gets channel 32*dblk + lane%32 and rows 16*ks + 4*g + {0..3},
// 16*ks + 8 + 4*g + {0..3}.  Lane j of a group of 16 addresses row 4*g + j/4 (+ 8 for the second read)
// and the 8 bytes at channel 32*dblk + 16*half + 4*(j%4).
__device__ __forceinline__ void ttile_offsets(int lane, uint32_t (&off)[4][2]) {
  const int j = lane & 15, t = j >> 2, c = j & 3;
  const int g = lane >> 5, half = (lane >> 4) & 1;
  const int x = 2 * half + (c >> 1);
#pragma unroll
  for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) {
      const int r = 8 * hi + 4 * g + t;
      const int slot = ((dblk ^ t) << 2) | (x ^ (2 * hi + g));
      off[dblk][hi] = (uint32_t)(r * kHeadDim + 8 * slot + 4 * (c & 1));
    }
}
__device__ __forceinline__ bf16x8 ttile_frag(const uint16_t *tile, const uint32_t (&off)[4][2], int dblk, int ks) {
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(KVM_LDS_V4(tile + off[dblk][0] + 16 * ks * kHeadDim));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(KVM_LDS_V4(tile + off[dblk][1] + 16 * ks * kHeadDim));
  Frag8 f;
  f.d[0] = __builtin_bit_cast(uint2, lo);
  f.d[1] = __builtin_bit_cast(uint2, hi);
  return f.v;
}

// Role KV has two results in registers and no room for offsets: both sets follow from one offset each by
// an exclusive or: chunk 2 * ks ^ .. of a row, block dblk ^ .. of a transposed fragment, whose second read lies eight
// rows further on with two chunks exchanged.  opaque(): computed where used.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}
// (addresses in LDS bytes; tiles are aligned to 8 KiB, so the exclusive or leaves `at` alone)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 ktile_frag_at(uint32_t addr0, int ks, uint32_t at) {
  return __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4 *)((addr0 ^ (uint32_t)(32 * ks)) + at));
}
__device__ __forceinline__ bf16x8 ttile_frag_at(uint32_t addr0, int dblk, int ks, uint32_t at) {
  at += (uint32_t)(2 * 16 * ks * kHeadDim);
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16 *)((addr0 ^ (uint32_t)(64 * dblk)) + at));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16 *)((addr0 ^ (uint32_t)(64 * dblk + 32)) + at + 2 * 8 * kHeadDim));
  Frag8 f;
  f.d[0] = __builtin_bit_cast(uint2, lo);
  f.d[1] = __builtin_bit_cast(uint2, hi);
  return f.v;
}

// Half of a query's D = dout . out (the lane's channels; the lane 32 away has the others).  One order of the sum
// for whoever forms D.
__device__ __forceinline__ float delta_half(const uint16_t *o_row, const bf16x8 (&dout)[8], int g) {
  float part = 0.f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    const uint4 ov = *reinterpret_cast<const uint4 *>(o_row + 16 * ks + 8 * g);
    Frag8 f;
    f.v = dout[ks];
    float of[8], df[8];
    unpack16<bf16_t>(ov, of);
    unpack16<bf16_t>(f.q, df);
#pragma unroll
    for (int e = 0; e < 8; ++e) part = fmaf(of[e], df[e], part);
  }
  return part;
}

// D of every query ahead of the walk: 32 queries per wave, two lanes each.
__global__ __launch_bounds__(256) void bwd_delta_mfma_kernel(const uint16_t *out, const uint16_t *dout, float *delta,
                                                             int64_t rows) {
  const int lane = threadIdx.x & 63, g = lane >> 5;
  const int64_t row = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32 + (lane & 31);
  const int64_t at = (row < rows ? row : rows - 1) * kHeadDim;
  bf16x8 d[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    Frag8 f;
    f.q = *reinterpret_cast<const uint4 *>(dout + at + 16 * ks + 8 * g);
    d[ks] = f.v;
  }
  const float sum = xhalf_sum(delta_half(out + at, d, g));
  if (row < rows && g == 0) delta[row] = sum;
}

struct MfmaChunk {
  int64_t cs, wb;   // chunk start, first window position
  int32_t nq, m;    // queries of the chunk, state rows it saw
  int32_t nq_ext;   // queries from the chunk start on that see the chunk's own tokens as window keys
  int32_t folded;   // the chunk's tokens were folded later on: their first gradient share is in the ring
  int32_t ring_row0;  // where in the ring ([U, ring rows, d]) the chunk's tokens have that share
  int32_t section;    // role KV: kSecBoth, or only the window-key / only the state-row workgroups
};


template <int kRole>
__device__ __forceinline__ void bwd_mfma_role(Bwd a, MfmaChunk c, int block) {   // (by reference the loops spill two registers more)
  constexpr bool kKeysSta = kRole != kRoleDQ;
  extern __shared__ __attribute__((aligned(1024))) uint16_t lds[];
  float *rowsc = reinterpret_cast<float *>(lds + 4 * kTileElems);  // [stage][lse * log2e | D][32]
  constexpr int D = kHeadDim;
  constexpr int kRows = kKeysSta ? 32 : kTileKeys;  // rows of a streamed tile
  constexpr int kTileE = kRows * D, kBlks = kRows / 32;
  const Dev &dv = a.dv;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  const int G = dv.Hq / dv.Hkv;
  const int n_keys_win = c.nq;  // role KV: the window keys of a launch are the chunk's own tokens
  const int n_st_wg = (c.m + kStaPerWg - 1) / kStaPerWg;
  const int tpc = (c.nq + kStaPerWg - 1) / kStaPerWg;
  // Consecutive workgroup ids go round-robin over the 8 XCDs: a unit's workgroups share one L2.
  // Role KV: the grid has two sections, the window-key workgroups of all units first and the
  // state-row workgroups after them.  The former stream a whole window of queries and the latter
  // one chunk: started first, the long ones are done when the short ones have had two rounds
  // (interleaved unit by unit, the last long ones would start after the first round of short ones).
  const int n_win_wg = (n_keys_win + kStaPerWg - 1) / kStaPerWg;
  const int groups8 = (dv.U + kXcds - 1) / kXcds * kXcds;
  int wg = block, per_group = G * tpc;
  bool section_state = false;
  if constexpr (kKeysSta) {
    section_state = c.section == kSecState || (c.section == kSecBoth && wg >= groups8 * n_win_wg);
    per_group = section_state ? n_st_wg : n_win_wg;
    if (section_state && c.section == kSecBoth) wg -= groups8 * n_win_wg;
  }
  const int xcd = wg % kXcds, seq = wg / kXcds;
  const int u = (seq / per_group) * kXcds + xcd;
  if (u >= dv.U) return;
  const int member = seq % per_group;
  const int b = u / dv.Hkv, h = u % dv.Hkv;
  const float scale = rsqrtf((float)D);

  // ---- stationary vectors
  bool col_ok;
  const uint16_t *sk_row;
  [[maybe_unused]] const uint16_t *sv_row = nullptr;
  int colq = 0;          // role dQ: the lane's query within the chunk
  int64_t kpos = -1;     // role KV, window keys: the lane's key position
  int hq_sta = 0, st_row = 0;
  bool sta_state = false;
  int wg_first = 0;      // role KV, window keys: first key position of the workgroup, relative to cs
  if constexpr (!kKeysSta) {
    const int qt = member % tpc, gq = member / tpc;
    hq_sta = __builtin_amdgcn_readfirstlane(h * G + gq);
    colq = kStaPerWg * qt + 32 * wave + l32;
    col_ok = colq < c.nq;
    const int qc = col_ok ? colq : c.nq - 1;
    const int64_t qrow = ((int64_t)b * a.T + c.cs + qc) * dv.Hq + hq_sta;
    sk_row = (const uint16_t *)a.q + qrow * D;
    sv_row = (const uint16_t *)a.dout + qrow * D;
  } else {
    sta_state = section_state;
    if (sta_state) {
      st_row = kStaPerWg * member + 32 * wave + l32;
      col_ok = st_row < c.m;
      const int64_t ro = ((int64_t)u * dv.Mcap + (col_ok ? st_row : c.m - 1)) * D;
      sk_row = (const uint16_t *)a.khat + ro;
    } else {
      const int64_t first = c.cs + (int64_t)kStaPerWg * member;
      wg_first = (int)(first - c.cs);
      kpos = first + 32 * wave + l32;
      col_ok = kpos < c.cs + c.nq;
      const int64_t tok = ((int64_t)b * a.T + (col_ok ? kpos : c.cs + c.nq - 1)) * dv.Hkv + h;
      sk_row = (const uint16_t *)a.k + tok * D;
    }
  }
  bf16x8 sk[8];
  [[maybe_unused]] bf16x8 sv[kKeysSta ? 1 : 8];
  float lse2_col = 0.f, d_col = 0.f;

  // ---- streamed tiles
  int n_st = 0, n_tiles, qt0 = 0, per_head = 1;
  int nq_str = c.nq;  // role KV: queries streamed, from the chunk start on
  if constexpr (!kKeysSta) {
    n_st = (c.m + kTileKeys - 1) / kTileKeys;
    const int qt = member % tpc;
    const int qend = kStaPerWg * (qt + 1) < c.nq ? kStaPerWg * (qt + 1) : c.nq;
    n_tiles = n_st + (int)((c.cs + qend - c.wb + kTileKeys - 1) / kTileKeys);
  } else {
    nq_str = sta_state ? c.nq : c.nq_ext;
    const int n_qt = (nq_str + kRows - 1) / kRows;
    qt0 = (!sta_state && wg_first > 0) ? wg_first / kRows : 0;
    per_head = n_qt - qt0;
    n_tiles = G * per_head;
    // Order of the streamed tiles: the last 64 queries first, for each 64 the heads of the group one after
    // the other, and a head's two tiles in ascending order (next_streamed).  The workgroups of a unit that share a stream differ in
    // where their first visible tile lies, not in where the last one does: walking backwards
    // they all start on the same tile and stay in step, so that one of them brings a tile into
    // the XCD's L2 and the others find it there (ascending, head by head, they ran up to six
    // tiles apart and the stream was fetched more than twice over).
  }
  n_tiles = __builtin_amdgcn_readfirstlane(n_tiles);
  // role KV: head and 32-query tile asked for last.  A tile without a partner (qt0 is even: workgroups start every 128
  // keys) comes first.  dk and dv are sums in this order: that of 64-query tiles, with the same bits.
  int str_gq = 0, str_qt = (qt0 + per_head - 1) & ~1;
  auto next_streamed = [&]() {
    if (!(str_qt & 1) && str_qt + 1 < qt0 + per_head) {
      ++str_qt;
    } else {
      str_qt &= ~1;
      if (++str_gq == G) {
        str_gq = 0;
        str_qt -= 2;
      }
    }
  };

  uint32_t koff[8], toff[4][2];
  rtile_offsets(lane, koff);
  ttile_offsets(lane, toff);
  const DmaLane dl = dma_lane_both(lane);
  const uint32_t lds_addr = lds_addr_of(lds);
  [[maybe_unused]] const uint32_t k_addr = lds_addr + 2 * koff[0], t_addr = lds_addr + 2 * toff[0][0];  // role KV

  auto issue_tile = [&](int it) {
    const char *xb, *yb;
    uint32_t stride;
    int valid;
    if constexpr (!kKeysSta) {
      if (it < n_st) {
        const int64_t ro = ((int64_t)u * dv.Mcap + (int64_t)it * kTileKeys) * D * 2;
        xb = (const char *)a.khat + ro;
        yb = (const char *)a.vhat + ro;
        stride = D * 2;
        valid = c.m - it * kTileKeys;
      } else {
        const int64_t p0 = c.wb + (int64_t)(it - n_st) * kTileKeys;
        const int64_t tok = ((int64_t)b * a.T + p0) * dv.Hkv + h;
        xb = (const char *)a.k + tok * D * 2;
        yb = (const char *)a.v + tok * D * 2;
        stride = (uint32_t)dv.Hkv * D * 2;
        valid = (int)(c.cs + c.nq - p0);
      }
    } else {
      const int64_t qrow = ((int64_t)b * a.T + c.cs + (int64_t)str_qt * kRows) * dv.Hq + h * G + str_gq;
      xb = (const char *)a.q + qrow * D * 2;
      yb = (const char *)a.dout + qrow * D * 2;
      stride = (uint32_t)dv.Hq * D * 2;
      valid = nq_str - str_qt * kRows;
    }
    const uint32_t at = lds_addr + (uint32_t)(2 * (it & 1)) * (kTileE * 2);
    if constexpr (kKeysSta) {
      // half a tile: the first four of eight waves' shares
      const DmaLane dl = dma_lane_both((int)opaque((uint32_t)lane));
      const int v = valid >= kRows ? kTileKeys : valid;
      tile_dma<false, 8>(xb, stride, v, at, wave, dl);
      tile_dma<false, 8>(yb, stride, v, at + kTileE * 2, wave, dl);
    } else {
      tile_dma<false, 4>(xb, stride, valid, at, wave, dl);
      tile_dma<false, 4>(yb, stride, valid, at + kTileE * 2, wave, dl);
    }
  };
  // role KV: lse and D of a tile's 32 query rows (a half of the wave each) and the head's temperature, asked for by
  // the first wave a tile ahead and put into LDS just before the barrier that publishes the tile.  Nothing
  // is done to the values before that: a use would wait for them, and for the tile loads with them.
  float rs = 0.f, rs_tau = 1.f;
  typedef const __attribute__((address_space(1))) float GlobalF32;
  GlobalF32 *taus = nullptr;
  if constexpr (kKeysSta) {   // wave-uniform, kept in scalar registers
    const uint64_t x = (uint64_t)(sta_state ? dv.tau_state : dv.tau_bswa);
    taus = (GlobalF32 *)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
                           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x));
  }
  auto fetch_rowsc = [&]() {
    if constexpr (kKeysSta) {
      if (wave == 0) {
        const int ln = (int)opaque((uint32_t)lane);
        int r = str_qt * kRows + (ln & 31);
        r = r < nq_str ? r : nq_str - 1;
        const int64_t qrow = ((int64_t)b * a.T + c.cs + r) * dv.Hq + h * G + str_gq;
        const float *src = ln < 32 ? a.lse : a.delta;
        rs = src[qrow];
        if (taus) rs_tau = taus[h * G + str_gq];
      }
    }
  };
  auto store_rowsc = [&](int it) {
    if constexpr (kKeysSta) {
      if (wave == 0) {
        rowsc[(it & 1) * kRowScalars + lane] = lane < 32 ? rs * kLog2e : rs;
        if (lane == 0) rowsc[(it & 1) * kRowScalars + 64] = rs_tau;
      }
    }
  };
  // role dQ: both temperatures of its one head
  float tau_st = 1.f, tau_bs = 1.f;
  if constexpr (!kKeysSta) {
    auto uni = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
    if (dv.tau_state) tau_st = uni(dv.tau_state[hq_sta]);
    if (dv.tau_bswa) tau_bs = uni(dv.tau_bswa[hq_sta]);
  }

  f32x16 o1[4];                               // dq^T or dk^T
  [[maybe_unused]] f32x16 o2[kKeysSta ? 4 : 1];  // role KV: dv^T
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      o1[i][v] = 0.f;
      if constexpr (kKeysSta) o2[i][v] = 0.f;
    }
  float tau_sum_state = 0.f, tau_sum_bswa = 0.f;  // role dQ: sum of dS * S over state / window keys

  auto tile_step = [&](int it, auto parity) {
    store_rowsc(it);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    [[maybe_unused]] const int qtile = str_qt;
    if (it + 1 < n_tiles) {
      if constexpr (kKeysSta) next_streamed();
      issue_tile(it + 1);
      fetch_rowsc();
    }
    const uint16_t *X = lds + (2 * decltype(parity)::value) * kTileE;
    const uint16_t *Y = X + kTileE;
    // what this tile is, and whether any of it is visible to this wave's columns
    bool tile_state;   // logits of this tile use the state temperature
    bool need_mask;    // wave-uniform: whether any pair of the tile is invisible to this wave
    int lim_lane = 0;  // role dQ: tile rows <= lim_lane are visible to the lane's query
    int lo_lane = 0, hi_row = 0;  // role KV: tile rows lo_lane .. hi_row are visible to the lane's key
    if constexpr (!kKeysSta) {
      tile_state = it < n_st;
      const int wave_q0 = kStaPerWg * (member % tpc) + 32 * wave;  // the wave's first query
      if (tile_state) {
        lim_lane = c.m - it * kTileKeys - 1;
        need_mask = lim_lane < kTileKeys - 1;
      } else {
        const int p0rel = (int)(c.wb - c.cs) + (it - n_st) * kTileKeys;
        if (p0rel > wave_q0 + 31) return;  // all keys after the wave's queries
        lim_lane = colq - p0rel;           // visible rows: p0rel + r <= colq
        need_mask = p0rel + kTileKeys - 1 > wave_q0;
      }
    } else {
      tile_state = sta_state;
      const int row_pos0 = qtile * kRows;  // the tile's first query, relative to the chunk start
      hi_row = nq_str - 1 - row_pos0;          // rows beyond the last query are padding
      need_mask = hi_row < kRows - 1;
      if (!sta_state) {
        const int wave_k0 = wg_first + 32 * wave;  // the wave's first key, relative to the chunk start
        if (wave_k0 > row_pos0 + kRows - 1) return;  // all queries before the wave's keys
        lo_lane = wave_k0 + l32 - row_pos0;              // visible rows: key position <= query position
        need_mask = need_mask || wave_k0 + 31 > row_pos0;
      }
    }
    float tau;
    if constexpr (kKeysSta)
      tau = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(rowsc[decltype(parity)::value * kRowScalars + 64])));
    else tau = tile_state ? tau_st : tau_bs;
    const float cexp = tau * scale * kLog2e;

    f32x16 sacc[kBlks], dacc[kBlks];
    [[maybe_unused]] Frag8 pP[2 * kBlks];
    Frag8 pS[2 * kBlks];
    float tsum = 0.f;
    // Role KV: P^T and dS^T are packed as they are made, four rows at a time, with the scalars of the next four
    // asked for: the registers that all of a tile's scalars would take at once are not there.
    auto elementwise = [&](auto masked, auto blk_c) {
      constexpr int blk = decltype(blk_c)::value;
      if constexpr (kKeysSta) {
        const float *rl = rowsc + decltype(parity)::value * kRowScalars + 4 * g;
        float4 x = *reinterpret_cast<const float4 *>(rl), y = *reinterpret_cast<const float4 *>(rl + 32);
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          const float lse4[4] = {x.x, x.y, x.z, x.w}, d4[4] = {y.x, y.y, y.z, y.w};
          if (v4 < 3) {
            x = *reinterpret_cast<const float4 *>(rl + 8 * v4 + 8);
            y = *reinterpret_cast<const float4 *>(rl + 8 * v4 + 40);
          }
          float p[4], ds[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int v = 4 * v4 + e, r = mfma_row(v, g);
            bool vis = true;
            if constexpr (decltype(masked)::value) vis = r >= lo_lane && r <= hi_row;
            p[e] = vis ? __builtin_amdgcn_exp2f(fmaf(sacc[0][v], cexp, -lse4[e])) : 0.f;
            ds[e] = p[e] * (dacc[0][v] - d4[e]) * tau;
          }
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            pP[v4 >> 1].w[2 * (v4 & 1) + i] = pack_bf16(p[2 * i], p[2 * i + 1]);
            pS[v4 >> 1].w[2 * (v4 & 1) + i] = pack_bf16(ds[2 * i], ds[2 * i + 1]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = 32 * blk + mfma_row(v, g);
          bool vis = true;
          if constexpr (decltype(masked)::value) vis = r <= lim_lane;
          const float s = sacc[blk][v];
          const float p = vis ? __builtin_amdgcn_exp2f(fmaf(s, cexp, -lse2_col)) : 0.f;
          const float ds = p * (dacc[blk][v] - d_col);
          tsum = fmaf(ds, s, tsum);
          dacc[blk][v] = ds * tau;
        }
#pragma unroll
        for (int ks = 2 * blk; ks < 2 * blk + 2; ++ks)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int v0 = (ks & 1) * 8 + 2 * e;
            pS[ks].w[e] = pack_bf16(dacc[blk][v0], dacc[blk][v0 + 1]);
          }
      }
    };
    // The products of 32 streamed rows.  Fragments are read from LDS four steps ahead of the matrix instruction that
    // takes them, and the first four of the second product while the first one ends; the order is pinned
    // (0x100: LDS reads, 0x008: matrix instructions), or the compiler, short of registers, reads every
    // fragment just before its use and each matrix instruction waits for LDS.
    bf16x8 tf[4];
    auto first_products = [&](auto blk_c) {
      __builtin_amdgcn_sched_barrier(0);
      constexpr int blk = decltype(blk_c)::value;
      const f32x16 zero = {0.f};
      bf16x8 xf[4], yf[4];
      if constexpr (kKeysSta) {
        const uint32_t k0 = opaque(k_addr), v0 = k0 + 4 * kTileE * 2 + (uint32_t)wave * (32 * D * 2), t0 = opaque(t_addr);
        constexpr uint32_t xa = decltype(parity)::value * (2 * kTileE * 2), ya = xa + kTileE * 2;
        constexpr int kAhead = 4;   // steps of the second chain, two fragments each: four do not fit the registers
        bf16x8 vf[kAhead];
#pragma unroll
        for (int i = 0; i < 4; ++i) xf[i] = ktile_frag_at(k0, i, xa);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          sacc[blk] = mfma32(xf[ks & 3], sk[ks], ks == 0 ? zero : sacc[blk]);
          if (ks < 4) xf[ks] = ktile_frag_at(k0, ks + 4, xa);
          if (ks >= 8 - kAhead) {
            yf[ks - (8 - kAhead)] = ktile_frag_at(k0, ks - (8 - kAhead), ya);
            vf[ks - (8 - kAhead)] = ktile_frag_at(v0, ks - (8 - kAhead), 0);
          }
        }
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          dacc[blk] = mfma32(yf[ks % kAhead], vf[ks % kAhead], ks == 0 ? zero : dacc[blk]);
          if (ks + kAhead < 8) {
            yf[ks % kAhead] = ktile_frag_at(k0, ks + kAhead, ya);
            vf[ks % kAhead] = ktile_frag_at(v0, ks + kAhead, 0);
          } else {
            tf[ks - (8 - kAhead)] = ttile_frag_at(t0, ks - (8 - kAhead), 0, ya);
          }
        }
#pragma unroll
        for (int i = kAhead; i < 4; ++i) tf[i] = ttile_frag_at(t0, i, 0, ya);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 - kAhead, 0);
#pragma unroll
        for (int i = 0; i < 8 + kAhead; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * (4 - kAhead), 0);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          xf[i] = ktile_frag(X, koff, blk, i);
          yf[i] = ktile_frag(Y, koff, blk, i);
        }
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          sacc[blk] = mfma32(xf[ks & 3], sk[ks], ks == 0 ? zero : sacc[blk]);
          dacc[blk] = mfma32(yf[ks & 3], sv[ks], ks == 0 ? zero : dacc[blk]);
          if (ks < 4) {
            xf[ks] = ktile_frag(X, koff, blk, ks + 4);
            yf[ks] = ktile_frag(Y, koff, blk, ks + 4);
          } else {
            tf[ks - 4] = ttile_frag(X, toff, ks - 4, 2 * blk);
          }
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto second_product = [&](auto blk_c) {
      constexpr int blk = decltype(blk_c)::value;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kKeysSta) {
        const uint32_t t0 = opaque(t_addr);
        constexpr uint32_t xa = decltype(parity)::value * (2 * kTileE * 2), ya = xa + kTileE * 2;
#pragma unroll
        for (int n = 0; n < 16; ++n) {   // eight of dv^T, then eight of dk^T
          const int ks = (n >> 2) & 1, dblk = n & 3;
          if (n < 8) o2[dblk] = mfma32(tf[dblk], pP[ks].v, o2[dblk]);
          else o1[dblk] = mfma32(tf[dblk], pS[ks].v, o1[dblk]);
          if (n < 12) tf[dblk] = ttile_frag_at(t0, dblk, ((n + 4) >> 2) & 1, n < 4 ? ya : xa);
        }
#pragma unroll
        for (int i = 0; i < 12; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      } else {
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          const int ks = 2 * blk + (n >> 2), dblk = n & 3;
          o1[dblk] = mfma32(tf[dblk], pS[ks].v, o1[dblk]);
          if (n < 4) tf[dblk] = ttile_frag(X, toff, dblk, ks + 1);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    using Masked = std::integral_constant<bool, true>;
    using Plain = std::integral_constant<bool, false>;
    auto rows32 = [&](auto blk) {
      first_products(blk);
      if (need_mask) elementwise(Masked{}, blk); else elementwise(Plain{}, blk);
      second_product(blk);
    };
    rows32(std::integral_constant<int, 0>{});
    if constexpr (kBlks == 2) rows32(std::integral_constant<int, 1>{});
    if constexpr (!kKeysSta) {
      if (tile_state) tau_sum_state += tsum; else tau_sum_bswa += tsum;
    }
  };

  // Role KV: the workgroup's 128 value rows go to LDS, in the layout of the tiles (a row block that
  // starts beyond the last key repeats that key; nothing of it is kept).
  if constexpr (kKeysSta) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int n_keys = sta_state ? c.m : c.nq;
      int row0 = kStaPerWg * member + 64 * half;
      row0 = row0 < n_keys ? row0 : n_keys - 1;
      const int64_t first = sta_state ? (int64_t)u * dv.Mcap + row0 : ((int64_t)b * a.T + c.cs + row0) * dv.Hkv + h;
      tile_dma<false, 4>((const char *)(sta_state ? a.vhat : (void *)a.v) + first * D * 2,
                         (uint32_t)(sta_state ? 1 : dv.Hkv) * D * 2, n_keys - row0,
                         lds_addr + 4 * kTileE * 2 + (uint32_t)half * (kTileElems * 2), wave, dl);
    }
  }
  // The first tile is asked for ahead of the stationary vectors, so that the two travel together
  // (short loops -- few streamed tiles per workgroup -- feel every round trip of the prologue).
  if (n_tiles > 0) {
    issue_tile(0);
    fetch_rowsc();
  }
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    Frag8 f;
    f.q = *reinterpret_cast<const uint4 *>(sk_row + 16 * ks + 8 * g);
    sk[ks] = f.v;
    if constexpr (!kKeysSta) {
      f.q = *reinterpret_cast<const uint4 *>(sv_row + 16 * ks + 8 * g);
      sv[ks] = f.v;
    }
  }
  if constexpr (!kKeysSta) {
    const int qc = col_ok ? colq : c.nq - 1;
    const int64_t qrow = ((int64_t)b * a.T + c.cs + qc) * dv.Hq + hq_sta;
    lse2_col = a.lse[qrow] * kLog2e;
    // D = dout . out of the lane's query: the lane has half of the dout row already.  Role KV, which
    // runs after this one when D is formed here, reads it from memory
    if (a.delta_ready) {
      d_col = a.delta[qrow];
    } else {
      d_col = xhalf_sum(delta_half((const uint16_t *)a.out + qrow * D, sv, g));
      if (col_ok && g == 0) a.delta[qrow] = d_col;
    }
  }

  // the stationary vectors are in registers from here on (the compiler does not count the tile
  // loads; said explicitly so that it does not wait for "its" loads inside the loop)
  __builtin_amdgcn_s_waitcnt(0);
  for (int it = 0; it < n_tiles; it += 2) {
    tile_step(it, std::integral_constant<int, 0>{});
    if (it + 1 < n_tiles) tile_step(it + 1, std::integral_constant<int, 1>{});
  }

  // ---- results (nothing of what follows is to be prepared, or kept in registers, during the loop)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!kKeysSta) {
    if (col_ok) {
      const int64_t qrow = ((int64_t)b * a.T + c.cs + colq) * dv.Hq + hq_sta;
      uint16_t *orow = (uint16_t *)a.dq + qrow * D;
#pragma unroll
      for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const uint32_t lo = pack_bf16(o1[dblk][4 * vq] * scale, o1[dblk][4 * vq + 1] * scale);
          const uint32_t hi = pack_bf16(o1[dblk][4 * vq + 2] * scale, o1[dblk][4 * vq + 3] * scale);
          *reinterpret_cast<uint2 *>(orow + 32 * dblk + 8 * vq + 4 * g) = make_uint2(lo, hi);
        }
    }
    const float ts = wave_sum(col_ok ? tau_sum_state : 0.f) * scale;
    const float tb = wave_sum(col_ok ? tau_sum_bswa : 0.f) * scale;
    if (lane == 0) {
      atomicAdd(a.par64 + 2 * dv.Hkv * D + hq_sta, (double)ts);
      atomicAdd(a.par64 + 2 * dv.Hkv * D + dv.Hq + hq_sta, (double)tb);
    }
  } else {
    if (col_ok) {
      // The chunk's own tokens as window keys: this launch has streamed every query that sees
      // them, so dk (which carries the logit scale) resp. dv is complete once the share the
      // token got when its fold was undone (kept in fp32 in a ring of the last window's blocks and one more)
      // is added, and goes out in the I/O dtype.
      if (!sta_state) {
        const int64_t tok = ((int64_t)b * a.T + kpos) * dv.Hkv + h;
        const int64_t ro = ((int64_t)u * a.ring_rows + c.ring_row0 + (int)(kpos - c.cs)) * D;
        auto finish = [&](const f32x16 (&o)[4], float os, void *out, const float *acc) {
          uint16_t *orow = (uint16_t *)out + tok * D;
          const float *ring = acc + ro;
#pragma unroll
          for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
              const int ch = 32 * dblk + 8 * vq + 4 * g;
              float4 x4 = c.folded ? *reinterpret_cast<const float4 *>(ring + ch) : make_float4(0.f, 0.f, 0.f, 0.f);
              x4.x += o[dblk][4 * vq] * os;
              x4.y += o[dblk][4 * vq + 1] * os;
              x4.z += o[dblk][4 * vq + 2] * os;
              x4.w += o[dblk][4 * vq + 3] * os;
              *reinterpret_cast<uint2 *>(orow + ch) = make_uint2(pack_bf16(x4.x, x4.y), pack_bf16(x4.z, x4.w));
            }
        };
        finish(o1, scale, a.dk, a.dk_acc);
        finish(o2, 1.f, a.dv_out, a.dv_acc);
      }
    }
    // State rows: the readout's adjoint goes straight on into the adjoint of the sums.  A lane
    // holds half of its row's channels (four at a time: 32*dblk + 8*vq + 4*g ..), the lane 32
    // away the other half, so a sum over the row is a sum over the lane's registers plus one
    // exchange between the wave's halves.
    if (sta_state) {
      const int64_t ro = ((int64_t)u * dv.Mcap + (col_ok ? st_row : 0)) * D;
      {
        // v-hat = rho * sV / max(|sV|, eps)
        float svr[4][16];
        float nn = 0.f, dot = 0.f;
#pragma unroll
        for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const float4 x4 = *reinterpret_cast<const float4 *>(a.wsV + ro + 32 * dblk + 8 * vq + 4 * g);
            const float xs[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              svr[dblk][4 * vq + e] = xs[e];
              nn += xs[e] * xs[e];
              dot += o2[dblk][4 * vq + e] * xs[e];
            }
          }
        const float nrm = sqrtf(xhalf_sum(nn));
        const float den = fmaxf(nrm, dv.norm_eps);
        dot = xhalf_sum(dot) / den;  // dv-hat . unit vector
        const float rho = dv.rho[(int64_t)u * dv.Mcap + (col_ok ? st_row : 0)];
        const float back = nrm > dv.norm_eps ? rho * dot / (den * den) : 0.f;
        if (col_ok) {
#pragma unroll
          for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
              const int ch = 32 * dblk + 8 * vq + 4 * g;
              float4 x4 = *reinterpret_cast<const float4 *>(a.dsV + ro + ch);
              x4.x += rho / den * o2[dblk][4 * vq] - back * svr[dblk][4 * vq];
              x4.y += rho / den * o2[dblk][4 * vq + 1] - back * svr[dblk][4 * vq + 1];
              x4.z += rho / den * o2[dblk][4 * vq + 2] - back * svr[dblk][4 * vq + 2];
              x4.w += rho / den * o2[dblk][4 * vq + 3] - back * svr[dblk][4 * vq + 3];
              *reinterpret_cast<float4 *>(a.dsV + ro + ch) = x4;
            }
          if (g == 0) a.drho[(int64_t)u * dv.Mcap + st_row] += dot;
        }
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      {
        // k-hat = LN_s(sK) * gamma + beta.  The standardised sums x-hat and 1 / sqrt(var + eps) of
        // the visited version are kept beside its readout, so everything the row needs is asked
        // for at once: one memory round trip, not a chain of them.
        const float rden = a.rden[(int64_t)u * dv.Mcap + (col_ok ? st_row : 0)];
        float xh[4][16], pg[4][16], pb[4][16];
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const int ch = 32 * dblk + 8 * vq + 4 * g;
            const float4 x4 = *reinterpret_cast<const float4 *>(a.xhat + ro + ch);
            const float4 g4 = dv.gamma ? *reinterpret_cast<const float4 *>(dv.gamma + h * D + ch) : make_float4(1.f, 1.f, 1.f, 1.f);
            const float xs[4] = {x4.x, x4.y, x4.z, x4.w}, gs[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float dkh = o1[dblk][4 * vq + e] * scale;
              xh[dblk][4 * vq + e] = xs[e];
              pb[dblk][4 * vq + e] = dkh * gs[e];  // dk-hat * gamma for now
              pg[dblk][4 * vq + e] = dkh;
              s1 += dkh * gs[e];
              s2 += dkh * gs[e] * xs[e];
            }
          }
        const float m1 = xhalf_sum(s1) / (float)D, m2 = xhalf_sum(s2) / (float)D;
        float *red = reinterpret_cast<float *>(reinterpret_cast<char *>(lds) + kBwdTileBytes);  // [gamma | beta][wave][D]
        // the adjoint of the sums; what the parameter gradients sum over the rows is kept:
        // pg = dk-hat * x-hat (dgamma), pb = dk-hat (dbeta), zero for rows beyond the state
#pragma unroll
        for (int dblk = 0; dblk < 4; ++dblk)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const int ch = 32 * dblk + 8 * vq + 4 * g;
            float add[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float dkh = pg[dblk][4 * vq + e], x = xh[dblk][4 * vq + e];
              add[e] = (pb[dblk][4 * vq + e] - m1 - x * m2) * rden;
              pg[dblk][4 * vq + e] = col_ok ? dkh * x : 0.f;
              pb[dblk][4 * vq + e] = col_ok ? dkh : 0.f;
            }
            if (col_ok) {
              float4 x4 = *reinterpret_cast<const float4 *>(a.dsK + ro + ch);
              x4.x += add[0]; x4.y += add[1]; x4.z += add[2]; x4.w += add[3];
              *reinterpret_cast<float4 *>(a.dsK + ro + ch) = x4;
            }
          }
        // Sums over the 32 rows (lanes) of this half of the wave, for 64 channels at once: a
        // butterfly in which every exchange also halves the number of channels a lane carries --
        // the lane whose bit is set keeps the upper half of its channels and hands the lower half
        // to its partner, and the other way round -- so that 62 exchanges do the work of 64 x 5.
        // Register i stands for channel 32*(i/16) + 8*((i%16)/4) + 4*g + i%4; after the five
        // steps a lane holds the sums of registers base, base + 1, base = 32*b0 + 16*b1 + 8*b2 +
        // 4*b3 + 2*b4 (b_k = bit k of its lane number).
        auto rows_sum = [&](float (&v)[4][16], int which) {
          float *f = &v[0][0];
#define KVM_BFLY(N, BIT, XCHG)                                  \
  {                                                             \
    const bool up = (lane & BIT) != 0;                          \
    _Pragma("unroll") for (int i = 0; i < N / 2; ++i) {         \
      const float send = up ? f[i] : f[i + N / 2];              \
      const float keep = up ? f[i + N / 2] : f[i];              \
      f[i] = keep + XCHG(send);                                 \
    }                                                           \
  }
#define KVM_X1(x) dpp_get<0xB1>(x)
#define KVM_X2(x) dpp_get<0x4E>(x)
#define KVM_X4(x) __uint_as_float(__builtin_amdgcn_ds_swizzle(__float_as_uint(x), 0x101F))
#define KVM_X8(x) __uint_as_float(__builtin_amdgcn_ds_swizzle(__float_as_uint(x), 0x201F))
#define KVM_X16(x) __uint_as_float(__builtin_amdgcn_ds_swizzle(__float_as_uint(x), 0x401F))
          KVM_BFLY(64, 1, KVM_X1)
          KVM_BFLY(32, 2, KVM_X2)
          KVM_BFLY(16, 4, KVM_X4)
          KVM_BFLY(8, 8, KVM_X8)
          KVM_BFLY(4, 16, KVM_X16)
#undef KVM_BFLY
#undef KVM_X1
#undef KVM_X2
#undef KVM_X4
#undef KVM_X8
#undef KVM_X16
          const int i0 = 32 * (lane & 1) + 16 * ((lane >> 1) & 1) + 8 * ((lane >> 2) & 1) + 4 * ((lane >> 3) & 1) +
                         2 * ((lane >> 4) & 1);
          const int ch0 = 32 * (i0 >> 4) + 8 * ((i0 & 15) >> 2) + 4 * g + (i0 & 3);
          red[(4 * which + wave) * D + ch0] = f[0];
          red[(4 * which + wave) * D + ch0 + 1] = f[1];
        };
        rows_sum(pg, 0);
        rows_sum(pb, 1);
        __syncthreads();
        {
          const int which = tid / D, ch = tid % D;
          const float sum4 = red[(4 * which) * D + ch] + red[(4 * which + 1) * D + ch] + red[(4 * which + 2) * D + ch] +
                             red[(4 * which + 3) * D + ch];
          if (sum4 != 0.f) atomicAdd(a.par64 + (which * dv.Hkv + h) * D + ch, (double)sum4);
        }
      }
    }
  }
}

template <int kRole>
__global__ __launch_bounds__(256, 2) void bwd_mfma_kernel(Bwd a, MfmaChunk c) {
  bwd_mfma_role<kRole>(a, c, blockIdx.x);
}
// Both roles of a chunk in one launch, n_dq workgroups of dQ first (D is there already): see launch_backward_mfma_both.
__global__ __launch_bounds__(256, 2) void bwd_mfma_both_kernel(Bwd a, MfmaChunk c, int n_dq) {
  if ((int)blockIdx.x < n_dq)
    bwd_mfma_role<kRoleDQ>(a, c, blockIdx.x);
  else
    bwd_mfma_role<kRoleKV>(a, c, (int)blockIdx.x - n_dq);
}

}  // namespace

bool backward_on_mfma(const Dev &dv) { return dv.io == 1 && dv.d == kHeadDim && dv.C % 64 == 0; }

hipError_t launch_delta_mfma(const Bwd &a, int64_t rows, hipStream_t st) {
  hipLaunchKernelGGL(bwd_delta_mfma_kernel, dim3((unsigned)((rows + 127) / 128)), dim3(256), 0, st, (const uint16_t *)a.out,
                     (const uint16_t *)a.dout, a.delta, rows);
  return hipGetLastError();
}

namespace {
OncePerDevice<hipError_t> g_dq, g_kv, g_both;   // more than 64 KiB of LDS per workgroup has to be asked for
MfmaChunk chunk_of(const Bwd &a, int64_t cs, int nq, int m, bool folded, int section) {
  const Dev &dv = a.dv;
  MfmaChunk c;
  c.cs = cs;
  c.wb = cs + dv.C - dv.L > 0 ? cs + dv.C - dv.L : 0;
  c.nq = nq;
  c.m = m;
  // the chunk's tokens are window keys for the queries of one window from the chunk start on
  const int64_t ext = a.T - cs < dv.L ? a.T - cs : dv.L;
  c.nq_ext = (int)ext;
  c.folded = folded ? 1 : 0;
  c.ring_row0 = (int)((cs / dv.C) % (a.ring_rows / dv.C)) * dv.C;
  c.section = section;
  return c;
}
struct Grids {
  unsigned dq, window, state;   // workgroups
};
Grids grids_of(const Dev &dv, int nq, int m) {
  const unsigned groups = (unsigned)((dv.U + kXcds - 1) / kXcds * kXcds);
  const unsigned n_win = (unsigned)((nq + kStaPerWg - 1) / kStaPerWg), n_st = (unsigned)((m + kStaPerWg - 1) / kStaPerWg);
  return {groups * (unsigned)(dv.Hq / dv.Hkv) * n_win, groups * n_win, groups * n_st};
}
}  // namespace

// The launches of one chunk: dq (and the temperature sums); dk and dv of its own tokens and of the state rows.
hipError_t launch_backward_mfma(const Bwd &a, int64_t cs, int nq, int m, bool folded, int role, int section,
                                hipStream_t st) {
  const MfmaChunk c = chunk_of(a, cs, nq, m, folded, section);
  const Grids g = grids_of(a.dv, nq, m);
  if (role == kRoleDQ) {
    if (const hipError_t e = allow_lds(g_dq, (const void *)bwd_mfma_kernel<kRoleDQ>, kBwdLdsBytes); e != hipSuccess) return e;
    hipLaunchKernelGGL((bwd_mfma_kernel<kRoleDQ>), dim3(g.dq), dim3(256), kBwdLdsBytes, st, a, c);
    return hipGetLastError();
  }
  const unsigned n = section == kSecBoth ? g.state + g.window : section == kSecState ? g.state : g.window;
  if (n == 0) return hipSuccess;
  if (const hipError_t e = allow_lds(g_kv, (const void *)bwd_mfma_kernel<kRoleKV>, kBwdLdsBytes); e != hipSuccess) return e;
  hipLaunchKernelGGL((bwd_mfma_kernel<kRoleKV>), dim3(n), dim3(256), kBwdLdsBytes, st, a, c);
  return hipGetLastError();
}

// All of them at once.
bool backward_fits_one_launch(const Dev &dv, int m) {
  const Grids g = grids_of(dv, dv.C, m);
  return g.dq + g.window + g.state <= (dv.Hq <= 2 * dv.Hkv ? kBwdOneLaunch : kBwdOneLaunchHeads);
}
hipError_t launch_backward_mfma_both(const Bwd &a, int64_t cs, int nq, int m, bool folded, hipStream_t st) {
  if (const hipError_t e = allow_lds(g_both, (const void *)bwd_mfma_both_kernel, kBwdLdsBytes); e != hipSuccess) return e;
  const Grids g = grids_of(a.dv, nq, m);
  hipLaunchKernelGGL(bwd_mfma_both_kernel, dim3(g.dq + g.window + g.state), dim3(256), kBwdLdsBytes, st, a,
                     chunk_of(a, cs, nq, m, folded, kSecBoth), (int)g.dq);
  return hipGetLastError();
}

}  // namespace kvm
