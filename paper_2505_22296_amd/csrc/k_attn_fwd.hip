// Attention forward for one SP rank's real heads on gfx950.
//
// One workgroup = 8 wavefronts = 256 query rows of one head (a work item from
// the host block-skip scheduler; KW = 1, see below for KW > 1); wavefront w
// owns rows q_begin + 32w .. +32.  The key loop walks 64-key tiles of the segment.  K and V tiles are
// copied global -> LDS by DMA into the blocked layout of dev_common.h (no
// padding, no transposed copy: V^T fragments come from transposing LDS
// reads), four tiles resident: while a pair of tiles is consumed the next
// pair lands, and the eight wavefronts meet at a barrier once per pair.  Each
// tile is shared by all eight wavefronts.
//
// Per 64-key tile and wavefront:
//   S^T = K Q^T      (32x32x16 bf16 MFMA; Q^T kept in registers as B operand)
//   online softmax   (fp32; the 32x32 C layout gives each lane one query row,
//                     16 keys per tile half; the row max needs one exchange
//                     with lane l^32)
//   O^T += V^T P^T   (V^T by ds_read_b64_tr_b16 from the V tile; P^T from the
//                     C registers directly: K rows are loaded in perm32 order
//                     so each lane half's C registers are 8 consecutive keys,
//                     i.e. a B operand k-slice)
// The running max is only raised when it grows by more than 2^8 (exact:
// the final normalisation uses the same max).  Masking is evaluated only on
// tiles that straddle a segment edge or the causal diagonal; a wavefront
// skips the arithmetic of tiles that lie wholly past its causal diagonal.
//
// Launches of few items (short sequences, few heads) leave CUs idle and last
// as long as their longest item's serial walk over the keys.  There the host
// splits every item over KW = 2 or 4 workgroups of 256 / KW rows whose
// wavefronts form KW key groups, each walking every KW-th tile; the groups'
// (m, l, O) meet in LDS at the end.  The walk is KW times shorter and KW times
// as many CUs work; each staged tile serves KW times fewer rows, which is why
// a full chip keeps KW = 1.  Measured, 4 heads on one causal sequence, D = 128,
// KW = 1 / 2 / 4: 1024 rows 29.7 / 23.2 / 18.1 us, 4096 rows 92.2 / 59.3 /
// 43.0 us, 16384 rows 381 / 293 / 362 us; 28 heads of 4096 rows 122 / 150 /
// 193 us.
//
// The ring variant (MERGE) folds the chunk's normalised (O_c, LSE_c) into
// float32 accumulators with the log-sum-exp rule in the epilogue.
#include "dev_common.h"
#include "launch.h"

namespace spk {

namespace {

constexpr int NW = kFwdWaves;         // wavefronts per workgroup
constexpr int NT = 64 * NW;
static_assert(kFwdBM == 32 * NW, "fwd tiling");

// LDS stage of the forward: for each of the KW key groups a K and a V tile
// [BN][D] in the blocked layout (D/32 sub-tiles [BN][32]), filled by DMA in
// 1 KB blocks by the RW wavefronts of the group.
template <int D, int KW>
struct FwdStage {
  static constexpr int RW = NW / KW;           // row groups of 32 rows
  // keys per tile: 32 where KW tiles of 64 keys would leave no room for the
  // next ones beside them
  static constexpr int BN = KW * D > 256 ? 32 : kFwdBN;
  static constexpr int NST = KW == 1 ? kFwdStages : 2;         // resident stages
  static constexpr int TPB = KW == 1 ? kFwdTilesPerSync : 1;   // stages per barrier
  static_assert(NST % TPB == 0 && NST >= 2 * TPB, "fwd pipeline");
  static constexpr int SUB = BN * 4;           // chunks per sub-tile
  static constexpr int KB = BN * (D / 8) / 64; // 1 KB blocks per tile
  static constexpr int NBK = KB / RW;          // blocks per wavefront and tile
  static_assert(KB % RW == 0, "DMA blocks per wavefront");
  static constexpr int OFF_V = KB * 64, TILE = 2 * KB * 64;  // 16-byte chunks
  static constexpr int STAGE = KW * TILE;
  // partial results of the key groups, exchanged through the same LDS: O^T of
  // every wavefront (quad i of 4 dims: 64 lanes x 16 bytes), then (m, l)
  static constexpr int NQ = D / 8, OFF_ML = NW * NQ * 64;
  static constexpr int XCH = KW > 1 ? OFF_ML + NW * 32 : 0;
  static constexpr int SMEM = NST * STAGE > XCH ? NST * STAGE : XCH;
};

// KW key groups of RW = 8 / KW wavefronts: row group w % RW owns 32 query
// rows, key group w / RW the tiles n * KW + w / RW.  An item's rows are split
// over KW workgroups (of 256 / KW rows each), all on the item's XCD, one
// after the other, the last rows (the longest under a causal mask) first.
// TWO: at most 128 VGPRs, so that two workgroups share a CU.
template <int D, bool MERGE, int KW, bool TWO>
__global__ __launch_bounds__(NT, TWO ? 4 : 1) void attn_fwd_kernel(FwdArgs a, ItemList list) {
  using S = FwdStage<D, KW>;
  constexpr int RW = S::RW, BN = S::BN, NST = S::NST, TPB = S::TPB;
  constexpr int KS = D / 16;   // MFMA k-steps over D
  constexpr int DB = D / 32;   // 32-dim blocks of O^T
  constexpr int G = BN / 32;   // 32-key halves of a tile
  constexpr int NBK = S::NBK, NBW = 2 * NBK, STAGE = S::STAGE, SUB = S::SUB;

  __shared__ u32x4 smem[S::SMEM];

  int pos, sub;
  if (!split_pos<KW>(blockIdx.x, a.n_items, pos, sub)) return;
  int32_t it[kItemInts];
  load_item(a.items, list, 0, pos, it);
  int q0 = it[0], q1 = it[1], k1 = it[3];
  const int k0 = it[2], delta = it[4], head = it[5], kvh = it[6];
  const int tid = threadIdx.x;
  if constexpr (KW > 1) {
    if (!split_rows<KW>(it[7] == kItemFillQ, 32 * RW, sub, q0, q1)) return;
    if (a.causal) k1 = max(k0, min(k1, q1 + delta));
  }
  if (it[7] == kItemFillQ) {
    // dummy slot: O = +0, LSE = -inf (ring: the accumulators' identity on the
    // first chunk, and +0 in the bf16 copy)
    if constexpr (!MERGE) {
      fill_rows_bf16(a.o, q0, q1, a.H, head, D, tid, NT);
      fill_span_f32(a.lse + (int64_t)head * a.T_q + q0, q1 - q0, neg_inf(), tid, NT);
    } else {
      if (a.init) {
        fill_rows_f32(a.o_acc, q0, q1, a.H, head, D, tid, NT);
        fill_span_f32(a.lse_acc + (int64_t)head * a.T_q + q0, q1 - q0, neg_inf(), tid, NT);
      }
      if (a.o_out) fill_rows_bf16(a.o_out, q0, q1, a.H, head, D, tid, NT);
    }
    return;
  }
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hh = lane >> 5, l32 = lane & 31;
  const int rg = KW > 1 ? w % RW : w, kg = KW > 1 ? w / RW : 0;
  const int wr0 = q0 + rg * 32;  // the wavefront's first row
  const int row = wr0 + l32;
  const bool row_ok = row < q1;
  // last key any row of this wavefront may see (tiles past it are skipped)
  const int wave_rows = min(32, q1 - wr0);
  const int wave_kmax = wave_rows <= 0 ? -1 : a.causal ? min(k1, wr0 + wave_rows + delta) : k1;

  // Q^T as B operand: lane holds query row `row`, dims ks*16 + hh*8 + [0..7].
  u32x4 qf[KS];
  {
    const uint16_t* qp = a.q + ((int64_t)(row_ok ? row : q0) * a.H + head) * D + hh * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qf[s] = *(const u32x4*)(qp + s * 16);
      if (!row_ok) qf[s] = u32x4{0u, 0u, 0u, 0u};
    }
  }

  f32x16 oacc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;
  float m_run = neg_inf(), l_part = 0.f;
  const float c2 = a.scale_log2;
  // Carried with the running max (they change only when it is raised):
  // msc = m_run * c2 (0 while m_run is -inf), and the score above which the
  // max is raised, m_run + 8 / c2 (-inf while m_run is -inf)
  const float raise_by = 8.f / c2;
  float msc = 0.f, m_thr = neg_inf();

  const int kt_first = k0 & ~7;
  // stages of KW tiles
  const int n_tiles = (k1 > k0) ? (k1 - kt_first + BN * KW - 1) / (BN * KW) : 0;

  // Per-lane, tile-independent element offsets of this wavefront's DMA
  // blocks rg + RW*j: the first NBK of them in the K tile, the rest in V;
  // both tiles have the same shape and source row stride.
  const int kstride = a.Hkv * D;
  int off[NBK], key_of[NBK];
#pragma unroll
  for (int j = 0; j < NBK; ++j) {
    const int t = (rg + RW * j) * 64 + lane;   // chunk slot within the tile
    const int ts = t % S::SUB, r = ts / 4;
    key_of[j] = r;
    off[j] = 2 * (r * kstride + (t / S::SUB) * 32 + blk_chunk(r, ts % 4) * 8);  // bytes
  }
  const uint16_t* kbase = a.k + (int64_t)kvh * D;
  const uint16_t* vbase = a.v + (int64_t)kvh * D;
  auto issue = [&](int n) {
    const int kt = kt_first + (n * KW + kg) * BN;
    if (KW > 1 && kt >= k1) return;  // the key group has no tile in the last stage
    u32x4* stg = smem + (n % NST) * STAGE + kg * S::TILE + rg * 64;
    const int64_t rowoff = (int64_t)kt * kstride;
    if (kt + BN <= k1) {
#pragma unroll
      for (int j = 0; j < NBK; ++j) {
        dma16s(kbase + rowoff, off[j], stg + RW * j * 64);
        dma16s(vbase + rowoff, off[j], stg + S::OFF_V + RW * j * 64);
      }
    } else {  // keys past k1 (masked) are clamped to k1-1
#pragma unroll
      for (int j = 0; j < NBK; ++j) {
        const int o = off[j] + 2 * (min(kt + key_of[j], k1 - 1) - kt - key_of[j]) * kstride;
        dma16s(kbase + rowoff, o, stg + RW * j * 64);
        dma16s(vbase + rowoff, o, stg + S::OFF_V + RW * j * 64);
      }
    }
  };
  // Lane-constant LDS offsets of the fragments.  K fragment (g, ks): tile row
  // g*32 + perm32(l32), logical chunk 2ks + hh -> sub-tile ks/2 (immediate)
  // and one of two lane bases (ks even / odd).  V^T fragments: transposing
  // reads at two lane offsets; dim block, k-step and stage are immediates.
  const int kr = perm32(l32);
  const int kf0 = kr * 4 + blk_chunk(kr, hh), kf1 = kr * 4 + blk_chunk(kr, 2 + hh);
  const int vt0 = S::OFF_V * 8 + blk_tr_off(lane), vt1 = S::OFF_V * 8 + blk_tr_off2(lane);

  for (int n = 0; n < NST - TPB && n < n_tiles; ++n) issue(n);

  for (int n0 = 0; n0 < n_tiles; n0 += NST) {
#pragma unroll
    for (int u = 0; u < NST; ++u) {
      const int n = n0 + u;
      if (n >= n_tiles) break;
      if (u % TPB == 0) {
        // stages n .. n+TPB-1 landed; every wavefront is done with the
        // memory of stages n-TPB .. n-1, which receives n+NST-TPB ..
        const int issued = min(n_tiles, n + NST - TPB);
        wait_batches<NBW, NST - 2 * TPB>(issued - min(n_tiles, n + TPB));
        __syncthreads();
        // KW = 4: a stage is consumed in one step, about as long as a copy
        // takes to land, so the next stage's copies go first
        if constexpr (KW == 4)
          if (n + 1 < n_tiles) issue(n + 1);
      }
      // stage n + NST - TPB was freed at the last barrier; its copy is issued
      // after this tile's first MFMAs (spreads the DMA burst)
      const bool pf = KW < 4 && n + NST - TPB < n_tiles;
      const int kt = kt_first + (n * KW + kg) * BN;
      if (kt >= wave_kmax) {  // wholly past this wavefront's rows
        if (pf) issue(n + NST - TPB);
        continue;
      }
      const u32x4* stg = smem + u * STAGE + kg * S::TILE;

      // ---- S^T = K Q^T for the 32-key halves of the tile.  The K
      // fragment reads are issued together ahead of the MFMAs; the compiler
      // places the MFMAs among them (measured faster than holding every
      // MFMA behind the last read).
      u32x4 kfr[G * KS];
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          kfr[g * KS + ks] = stg[(ks >> 1) * SUB + g * 128 + ((ks & 1) ? kf1 : kf0)];
      f32x16 s[G];
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[g][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int g = 0; g < G; ++g) s[g] = mfma32(kfr[g * KS + ks], qf[ks], s[g]);
      // V^T fragments of this tile, read while the softmax runs (TWO: after it,
      // for the 128 registers)
      const uint16_t* stg16 = (const uint16_t*)stg;
      u32x4 vfr[DB * 2 * G];
      auto read_v = [&](int ks0, int ks1) {
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int ks = ks0; ks < ks1; ++ks) {
            const int o = d * SUB * 8 + ks * 16 * 32;
            const u32x2 lo = lds_tr16(stg16 + vt0 + o), hi = lds_tr16(stg16 + vt1 + o);
            vfr[d * 2 * G + ks] = u32x4{lo[0], lo[1], hi[0], hi[1]};
          }
      };
      if constexpr (!TWO) {
        read_v(0, 2 * G);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (pf) issue(n + NST - TPB);

      // ---- mask (only on edge / diagonal tiles)
      const bool need_mask = (kt < k0) | (kt + BN > k1) | (a.causal & (kt + BN - 1 > wr0 + delta));
      if (need_mask) {
        // keys [lo, hi) of the lane half's, counted from kt + 8 hh
        const int lo = k0 - kt - hh * 8;
        const int hi = (a.causal ? min(k1, row + delta + 1) : k1) - kt - hh * 8;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = g * 32 + c_row_of(r, 0);
            if (key < lo || key >= hi) s[g][r] = neg_inf();
          }
      }

      // ---- online softmax (lazy rescale).  Row max of the lane's 32
      // scores (finite or -inf): four chains of three-input maxima, 18 VALU
      // operations (a wavefront's dependent VALU operations issue back to
      // back, so short chains buy nothing)
      float mx4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mx4[i] = max3_nonan(s[0][i], s[0][i + 4], s[0][i + 8]);
        if constexpr (G == 2) {
          mx4[i] = max3_nonan(mx4[i], s[0][i + 12], s[1][i]);
          mx4[i] = max3_nonan(mx4[i], s[1][i + 4], s[1][i + 8]);
        }
        mx4[i] = max3_nonan(mx4[i], s[G - 1][i + 12], s[G - 1][i + 12]);
      }
      const float mx = wave_max_xor32(max3_nonan(max3_nonan(mx4[0], mx4[1], mx4[2]), mx4[3], mx4[3]));
      const bool need = mx > m_thr;  // false while every score is -inf
      if (__ballot(need)) {
        float alpha = need ? exp2f((m_run - mx) * c2) : 1.f;
        if (need) {
          m_run = mx;
          msc = mx * c2;
          m_thr = mx + raise_by;
        }
        l_part *= alpha;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[d][r] *= alpha;
      }
      u32x4 pb[2 * G];
      float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g][r], c2, -msc));
          ps[r & 3] += p[r];
        }
        pb[2 * g] = pack_bf16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
        pb[2 * g + 1] = pack_bf16x8(p[8], p[9], p[10], p[11], p[12], p[13], p[14], p[15]);
      }
      l_part += (ps[0] + ps[1]) + (ps[2] + ps[3]);

      // ---- O^T += V^T P^T
      if constexpr (TWO) {
        __builtin_amdgcn_sched_barrier(0);
        read_v(0, 2 * G);
      }
#pragma unroll
      for (int ks = 0; ks < 2 * G; ++ks)
#pragma unroll
        for (int d = 0; d < DB; ++d) oacc[d] = mfma32(vfr[d * 2 * G + ks], pb[ks], oacc[d]);
    }
  }

  // ---- epilogue: quad i of the row (4 dims at (i >> 2) * 32 + (i & 3) * 8
  // + hh * 4); the key groups share out the quads of a row
  constexpr int NQW = S::NQ / KW;
  float l_tot = wave_sum_xor32(l_part);
  float la = neg_inf();  // ring: the row's accumulated LSE
  float acc[NQW][4];
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < NQW; ++i)
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[i][x] = oacc[i >> 2][(i & 3) * 4 + x];
  } else {
    // the groups' partial results meet in LDS (every copy has landed: the
    // last stage's barrier waited for it) and are summed in group order
    __syncthreads();
    f32x4* xo = (f32x4*)smem;
    f32x2* xml = (f32x2*)(smem + S::OFF_ML);
#pragma unroll
    for (int i = 0; i < S::NQ; ++i)
      xo[(w * S::NQ + i) * 64 + lane] = f32x4{oacc[i >> 2][(i & 3) * 4], oacc[i >> 2][(i & 3) * 4 + 1],
                                              oacc[i >> 2][(i & 3) * 4 + 2], oacc[i >> 2][(i & 3) * 4 + 3]};
    xml[w * 64 + lane] = f32x2{m_run, l_tot};
    if constexpr (MERGE) {
      // every group reads it before one of them writes it below: the value
      // has arrived (the empty asm consumes it) when the barrier is reached
      if (!a.init) la = a.lse_acc[(int64_t)head * a.T_q + (row_ok ? row : q0)];
      asm volatile("" : "+v"(la) : : "memory");
    }
    __syncthreads();
    f32x2 ml[KW];
#pragma unroll
    for (int p = 0; p < KW; ++p) ml[p] = xml[(rg + RW * p) * 64 + lane];
    m_run = ml[0][0];
#pragma unroll
    for (int p = 1; p < KW; ++p) m_run = fmaxf(m_run, ml[p][0]);
    l_tot = 0.f;
#pragma unroll
    for (int i = 0; i < NQW; ++i)
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[i][x] = 0.f;
#pragma unroll
    for (int p = 0; p < KW; ++p) {
      // a group that saw no key of the row weighs nothing
      const float wt = ml[p][0] == neg_inf() ? 0.f : exp2f((ml[p][0] - m_run) * c2);
      l_tot += wt * ml[p][1];
#pragma unroll
      for (int i = 0; i < NQW; ++i) {
        const f32x4 o = xo[((rg + RW * p) * S::NQ + kg * NQW + i) * 64 + lane];
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[i][x] += wt * o[x];
      }
    }
  }
  const bool has = l_tot > 0.f;
  const float inv = has ? 1.f / l_tot : 0.f;
  const float lse_v = has ? (m_run * c2 + __log2f(l_tot)) * kLn2 : neg_inf();
  if (!row_ok) return;
  const int64_t obase = ((int64_t)row * a.H + head) * D + hh * 4;
  // element offset of the wavefront's quad i
  auto dim = [&](int i) { return ((kg * NQW + i) >> 2) * 32 + ((kg * NQW + i) & 3) * 8; };
  if constexpr (!MERGE) {
#pragma unroll
    for (int i = 0; i < NQW; ++i)
      *(u32x2*)(a.o + obase + dim(i)) =
          pack_bf16x4(acc[i][0] * inv, acc[i][1] * inv, acc[i][2] * inv, acc[i][3] * inv);
    if (hh == 0 && kg == 0) a.lse[(int64_t)head * a.T_q + row] = lse_v;
  } else {
    // every accumulator value is loaded before the first store (the stores
    // could alias later loads for all the compiler knows, which would
    // serialize one memory round trip per 16 bytes), together with the
    // accumulated LSE
    float4 old[NQW];
#pragma unroll
    for (int i = 0; i < NQW; ++i)
      old[i] = a.init ? make_float4(0.f, 0.f, 0.f, 0.f) : *(const float4*)(a.o_acc + obase + dim(i));
    const int64_t li = (int64_t)head * a.T_q + row;
    if constexpr (KW == 1)
      if (!a.init) la = a.lse_acc[li];
    float wa = 0.f, wb = 0.f, L = neg_inf();
    const float m = fmaxf(la, lse_v);
    if (m != neg_inf()) {
      float ea = __expf(la - m), eb = __expf(lse_v - m);
      float ssum = ea + eb;
      L = m + __logf(ssum);
      wa = ea / ssum;
      wb = eb / ssum * inv;  // folds the chunk's 1/l normalisation
    }
#pragma unroll
    for (int i = 0; i < NQW; ++i) {
      const float4 o = old[i];
      float4 nv = make_float4(wa * o.x + wb * acc[i][0], wa * o.y + wb * acc[i][1],
                              wa * o.z + wb * acc[i][2], wa * o.w + wb * acc[i][3]);
      *(float4*)(a.o_acc + obase + dim(i)) = nv;
      if (a.o_out) *(u32x2*)(a.o_out + obase + dim(i)) = pack_bf16x4(nv.x, nv.y, nv.z, nv.w);
    }
    if (hh == 0 && kg == 0) a.lse_acc[li] = L;
  }
}

}  // namespace

template <int D, int KW, bool TWO>
static hipError_t launch_fwd(const FwdArgs& a, const ItemList& list, bool merge, hipStream_t st) {
  const dim3 grid(split_grid(a.n_items, KW)), block(NT);
  return merge ? sp_launch(kKFwd, attn_fwd_kernel<D, true, KW, TWO>, grid, block, st, a, list)
               : sp_launch(kKFwd, attn_fwd_kernel<D, false, KW, TWO>, grid, block, st, a, list);
}

hipError_t launch_attn_fwd(const FwdArgs& a, const ItemList& list, LaunchShape s, int D, bool merge,
                           hipStream_t st) {
  if (a.n_items <= 0) return hipSuccess;
  if (D == 128) {
    if (s.split == 4) return launch_fwd<128, 4, false>(a, list, merge, st);
    if (s.split == 2) return launch_fwd<128, 2, false>(a, list, merge, st);
    return launch_fwd<128, 1, false>(a, list, merge, st);
  }
  if (s.split == 4) return launch_fwd<64, 4, false>(a, list, merge, st);
  if (s.split == 2)
    return s.two ? launch_fwd<64, 2, true>(a, list, merge, st)
                 : launch_fwd<64, 2, false>(a, list, merge, st);
  if (s.two) return launch_fwd<64, 1, true>(a, list, merge, st);
  return launch_fwd<64, 1, false>(a, list, merge, st);
}

}  // namespace spk
