// Fused Ring Self-Attention backward (bf16, A = 64 or 128): the derivative of Eq. 1
// with the ring structure of section 3.2.2, without the score strip in memory.
// P is recomputed from Q, K and the forward's LSE: P = exp(s QK^T - LSE).
//
//   preprocess: the row terms -D = -rowsum(dO o O) and -LSE / s; a kernel of its own for the step-level entry
//     point, for heads of 128 and where both kinds of gradients share a grid (fused_bwd_both_kernel), else the
//     prologue of the dQ kernel.
//   Both kernels recompute P = exp2(s log2e (Q K^T - LSE / s)): the matrix core forms the bracket
//   from the caller's bf16 Q and K as they are (its accumulator starts from -LSE / s) and the
//   factor s log2e is applied to the fp32 result, one multiply per score.  Folding that factor
//   into a bf16 operand instead would save the multiply and round the operand a second time:
//   an error of 2^-9 per element that is the same for every score of a key (or query), adds up
//   coherently in dK (or dQ) and more than doubles their largest error.
//   dkdv kernel: a work-group owns 32 WK keys (WK waves) and walks the query tiles of every
//     simulated rank, starting with the rank that holds those keys (ring
//     order); the sum over ranks that the ring would all-reduce is its loop.
//       S' = Q K^T - LSE / s, dP' = dO V^T - D      (A: Q / dO rows from LDS; B: K / V registers;
//                                                    the row terms are the accumulators' start)
//       P = exp2(s log2e S'), dS = P o dP'
//       dV^T += dO^T P, dK^T += Q^T dS   (A operand: LDS transpose reads; B: P / dS registers)
//   dq kernel: a work-group owns RW*R query rows (RW waves) and walks the K/V tiles in ring
//     order (the paper's second K ring pass):
//       S'^T = K Q^T - LSE / s, P^T = exp2(s log2e S'^T),
//       dP'^T = V dO^T - D, dS^T = P^T o dP'^T, dQ^T += K^T dS^T
#include "rsa_fused_tile.h"
#include "rsa_kernels.h"

#include <type_traits>

namespace rsa {

// Which tile of which head the work-groups of a kernel take.
struct TileOrder {
  FastDiv by_tiles;  // tiles of a head
  int by_length;     // causal: order of the tiles over the work-groups (longest_first)
};
struct BwdArgs {
  const uint16_t *Q, *K, *V, *dO;
  const float *nL, *nD;                 // -LSE / scale and -D per query row
  // dQ kernel with the preprocess folded in: it forms the row terms from O and LSE
  // itself and leaves them in nL_out, nD_out for the dK/dV kernel that follows
  const uint16_t *O;
  const float *LSE;
  float *nL_out, *nD_out;
  uint16_t *dQ, *dK, *dV;
  // fp32 partial sums per split: dV then dK of the dK/dV kernel with a split query walk,
  // dQ of the dQ kernel with a split key walk
  float *part;
  uint16_t *strip;  // dS^T (strip_collect_keys_kernel)
  int64_t L, c, Lq;
  int64_t qs[3], ks[3], os[3];  // element strides (batch, head, row) of Q, dQ; K, V, dK, dV; O, dO
  RowMap map;  // local query row -> global token index
  int N;
  FastDiv by_heads, by_Z;  // heads, Z
  float cl2, scale, inv_scale;  // scale log2(e), scale, 1 / scale
};

// ------------------------------------------------------------- preprocess ---
// nD_i = -sum_a dO_ia O_ia and nL_i = -LSE_i / scale: 8 lanes per row, 8 elements of every 64 each.  Where rows are few it
// is a launch and one chain of latencies: a row's place by multiplications, its loads (LSE among them) in flight together,
// the sum over lanes without LDS.
__device__ __forceinline__ float sum_of_8_lanes(float x) {
  auto other = [](float y, auto ctrl) __attribute__((always_inline)) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, y), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  x += other(x, std::integral_constant<int, 0xB1>{});   // quad_perm 1 0 3 2
  x += other(x, std::integral_constant<int, 0x4E>{});   // quad_perm 2 3 0 1
  return x + other(x, std::integral_constant<int, 0x141>{});  // row_half_mirror: the other four
}
__global__ void __launch_bounds__(256) bwd_preprocess_kernel(const uint16_t *dO, const uint16_t *O,
                                                             const float *LSE, float *nD, float *nL,
                                                             int64_t rows, int A, float inv_scale,
                                                             OutLayout lay) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = gid >> 3;
  const int sub = (int)(gid & 7);
  if (row >= rows) return;  // (all eight lanes of a row)
  const int64_t off = lay.row_off(row) + sub * 8;
  auto at = [&](const uint16_t *p, int a) { return *reinterpret_cast<const u32x4 *>(p + off + a); };
  const u32x4 x0 = at(dO, 0), y0 = at(O, 0);
  u32x4 x1 = {0, 0, 0, 0}, y1 = x1;
  if (A > 64) { x1 = at(dO, 64); y1 = at(O, 64); }
  const float lse = LSE[row];
  float acc = 0.f;
  auto add = [&](const u32x4 &x, const u32x4 &y) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = fmaf(bf16_to_f32(x[e] & 0xffffu), bf16_to_f32(y[e] & 0xffffu), acc);
      acc = fmaf(bf16_to_f32(x[e] >> 16), bf16_to_f32(y[e] >> 16), acc);
    }
  };
  add(x0, y0);
  if (A > 64) add(x1, y1);
  acc = sum_of_8_lanes(acc);
  if (sub < 2) (sub == 0 ? nD : nL)[row] = sub == 0 ? -acc : -lse * inv_scale;
}

// ------------------------------------------------------------------ dK, dV ---
// Work-group: 4 waves x 32 keys.  K and V of a wave's keys stay in
// registers as B operands; the work-group walks the query rows in stages of NQ tiles of 64 rows
// of Q and dO, double-buffered in LDS and filled by direct global->LDS loads (no staging
// registers), one barrier per stage.
// The row terms of the softmax backward ride on the accumulator init of the MFMAs:
//   S'  = Q K^T - LSE / scale  (so P = exp2(scale log2e S') is one multiply and the exp2)
//   dP' = dO V^T - D           (so dS = P dP' is one multiply)
// and dK = scale * sum_i dS_ij Q_i.
// A head of 128 is two halves of 64 (AH = 2): two LDS tiles per 64 rows, S' and dP' contract over
// both, dV and dK have twice the accumulators, and the kernel runs one wave per SIMD.
// WK waves share the work-group's keys, 32 each; QS groups of such waves share the query rows: group g takes
// every QS-th stage of the walk and the groups' sums are added in LDS.
// id of ids: the work-group's place among those of this kind; buf0, buf1: the two stage buffers.
// STRIP: dS^T leaves as well, in the operand registers' own order.
template <int NQ, int AH>
struct DkdvStage {
  unsigned char Qt[NQ][AH][kTileBytes], dOs[NQ][AH][kTileBytes];
  float lse[NQ][64], d[NQ][64];
};
template <int NQ, bool CAUSAL, int AH, int WK, int QS, bool STRIP = false>
__device__ __forceinline__ void dkdv_body(const BwdArgs &a, const TileOrder &order, uint32_t id, uint32_t ids,
                                          unsigned char *buf0, unsigned char *buf1) {
  constexpr int KW = 32;       // keys per wave
  constexpr int BK = WK * KW;  // keys per work-group
  constexpr int A = 64 * AH;
  using Stage = DkdvStage<NQ, AH>;
  Stage *const stage0 = reinterpret_cast<Stage *>(buf0), *const stage1 = reinterpret_cast<Stage *>(buf1);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % WK;
  const int grp = QS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / WK;
  const int col = lane & 31, half = lane >> 5;
  uint32_t head_, kt_;  // under the causal mask the first keys are seen by the most rows
  if (CAUSAL && order.by_length) {
    longest_first(id, a.by_heads, head_, kt_);
  } else {
    const uint32_t wg = xcd_remap(id, ids);
    head_ = order.by_tiles(wg);
    kt_ = wg - head_ * order.by_tiles.d;
  }
  const int64_t head = settled(head_), kt = settled(kt_);
  const int key0 = (int)kt * BK;          // first key of the work-group
  const int wkey0 = key0 + wave * KW;     // first key of this wave

  const int64_t kv_off = head_offset((uint32_t)head, a.by_Z, a.ks);
  const uint16_t *Qh = a.Q + head_offset((uint32_t)head, a.by_Z, a.qs);
  const uint16_t *dOh = a.dO + head_offset((uint32_t)head, a.by_Z, a.os);
  const uint16_t *Kh = a.K + kv_off;
  const uint16_t *Vh = a.V + kv_off;
  const float *nLh = a.nL + head * a.Lq;
  const float *nDh = a.nD + head * a.Lq;
  const int64_t q_ld = a.qs[2], kv_ld = a.ks[2], o_ld = a.os[2];

  // K and V rows of this wave as B operands:
  // lane (col, half) holds row key = wkey0 + col, elements dk*16 + half*8 .. +8.
  bf16x8 kreg[4 * AH], vreg[4 * AH];
  {
    int64_t key = wkey0 + col;
    if (key >= a.L) key = a.L - 1;  // ragged tail: clamped here, not stored below
#pragma unroll
    for (int dk = 0; dk < 4 * AH; ++dk) {
      kreg[dk] = *reinterpret_cast<const bf16x8 *>(Kh + key * kv_ld + dk * 16 + half * 8);
      vreg[dk] = *reinterpret_cast<const bf16x8 *>(Vh + key * kv_ld + dk * 16 + half * 8);
    }
  }

  const TileLanes tl(lane);
  // the wave's block of 32 keys in the first of its strip's tiles
  const bool keys_here = wkey0 < a.L;
  uint16_t *const strip =
      STRIP ? a.strip + ((head * (a.L >> 6) + (wkey0 >> 6)) * (a.Lq >> 6)) * 4096 + ((wkey0 >> 5) & 1) * 2048 : nullptr;

  f32x16 dv[2 * AH], dk_[2 * AH];  // [db], transposed: rows = head dim, columns = keys
#pragma unroll
  for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) { dv[db][v] = 0.f; dk_[db][v] = 0.f; }

  // Stages of NQ query tiles in ring order: start at the rank that owns key0.  Under the causal mask the rows are taken in
  // the order of their tokens (see RowMap), from the first that sees key0 on.
  const int nqt = (int)(a.Lq >> 6);
  const int nst = (nqt + NQ - 1) / NQ;
  int start = 0;
  if (CAUSAL) {
    start = a.map.from_token(key0) / (64 * NQ);
  } else {
    const int r = (a.map.owner(key0) - a.map.rb) * (int)a.c;  // local row of that rank's first query
    if (r >= 0 && r < a.Lq) start = r / (64 * NQ);
  }
  auto st_of = [&](int i) { int q = start + i; return q >= nst ? q - nst : q; };
  // With few keys (Table 3's projected keys) the walk over the query stages is split over
  // gridDim.y work-groups, each writing fp32 partial sums that a second kernel adds up.
  int i_begin = 0, i_end = nst;
  if (gridDim.y > 1) {
    const int per_split = (nst + (int)gridDim.y - 1) / (int)gridDim.y;
    i_begin = (int)blockIdx.y * per_split;
    i_end = i_begin + per_split < nst ? i_begin + per_split : nst;
  }
  if (CAUSAL && nst - start < i_end) i_end = nst - start;

  const TileDMAT<WK> dma_q(wave, lane, (int)q_ld), dma_o(wave, lane, (int)o_ld);
  auto load_stage = [&](int i, Stage &sn) __attribute__((always_inline)) {
    const int st = st_of(i);
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      int qt = st * NQ + u;
      if (qt >= nqt) qt = nqt - 1;  // past the last tile: refetch it (never used)
      const int64_t r0 = CAUSAL ? a.map.row_at(qt * 64) : (int64_t)qt * 64;
#pragma unroll
      for (int ah = 0; ah < AH; ++ah) {
        dma_q.load(Qh + r0 * q_ld + ah * 64, sn.Qt[u][ah]);
        dma_o.load(dOh + r0 * o_ld + ah * 64, sn.dOs[u][ah]);
      }
      // the 64 row terms of the tile, one dword per lane: the group's first waves fetch -LSE / scale, its last -D
      if (WK < 4 || (wave & 1) == (u & 1)) {
        if (wave < (WK + 1) / 2) lds_dma4(nLh + r0 + lane, sn.lse[u]);
        if (wave >= WK / 2) lds_dma4(nDh + r0 + lane, sn.d[u]);
      }
    }
  };

  int i0 = i_begin;  // position of the walk: group 0's stage
  int i = i0 + grp;    // this group's stage
  if (i < i_end) load_stage(i, stage0[grp]);
  wait_vmem();
  __syncthreads();
  // one stage: start the loads of the next stage into sn, compute on sc
  auto stage = [&](Stage &sc, Stage &sn) __attribute__((always_inline)) {
    const int i0next = i0 + QS, inext = i + QS;
    if (inext < i_end) load_stage(inext, sn);

    // The 32 MFMAs of a tile go in four groups of eight -- S', dP' of rows 0..31 (G0) and of
    // rows 32..63 (G1), then dV, dK over rows 0..31 (H0) and 32..63 (H1) -- and the vector work
    // of each half (V0, V1) sits beside the next group: G0 | G1 + V0 | H0 + V1 | H1.  MFMA and
    // vector instructions of one wave overlap only when they alternate in its instruction
    // stream, and an LDS read costs its full latency unless issued a phase early, so the
    // phases are fenced, every read after the tile's first is issued one phase before its
    // use, and the compiler interleaves inside a phase.
    bf16x8 qa[2][4 * AH], ga[2][4 * AH];
    f32x16 sacc[2], dpacc[2];
    const int qt0 = st_of(i) * NQ;
    auto active = [&](int u) {
      const int qt = qt0 + u;
      return (QS == 1 || i < i_end) && qt < nqt && (!CAUSAL || a.map.token_at(qt * 64) + 63 >= wkey0);
    };
    auto fetch = [&](int u, int qb) __attribute__((always_inline)) {
      // accumulators start from -LSE / scale and -D of their rows (same for all lanes of a half)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 l4 = *reinterpret_cast<const f32x4 *>(&sc.lse[u][qb * 32 + g * 8 + half * 4]);
        const f32x4 d4 = *reinterpret_cast<const f32x4 *>(&sc.d[u][qb * 32 + g * 8 + half * 4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) { sacc[qb][g * 4 + e] = l4[e]; dpacc[qb][g * 4 + e] = d4[e]; }
      }
#pragma unroll
      for (int dk = 0; dk < 4 * AH; ++dk) {
        qa[qb][dk] = tl.read_rows(sc.Qt[u][dk >> 2], qb * 32, dk & 3);
        ga[qb][dk] = tl.read_rows(sc.dOs[u][dk >> 2], qb * 32, dk & 3);
      }
    };
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      if (active(u)) {
        const int qf = a.map.token_at((qt0 + u) * 64);  // token of the tile's first row
        const bool domask = CAUSAL && qf < wkey0 + KW - 1;
        bf16x8 pf[4], sf[4];  // [kk]: P and dS as B operands, k = query
        auto g12 = [&](int qb) __attribute__((always_inline)) {
#pragma unroll
          for (int dk = 0; dk < 4 * AH; ++dk) {
            sacc[qb] = mfma_32x32x16(qa[qb][dk], kreg[dk], sacc[qb]);
            dpacc[qb] = mfma_32x32x16(ga[qb][dk], vreg[dk], dpacc[qb]);
          }
        };
        auto softmax_bwd = [&](int qb) __attribute__((always_inline)) {
          f32x16 &sv = sacc[qb];
          const f32x16 &dp = dpacc[qb];
          if (domask) {
            // rows of the block of 32 that see the lane's key: all but the first n
            const uint32_t seen = ~low_bits(wkey0 + col - qf - qb * 32 - half * 4);
#pragma unroll
            for (int v = 0; v < 16; ++v) sv[v] = keep_bit(sv[v], seen, (v >> 2) * 8 + (v & 3));
          }
#pragma unroll
          for (int w2 = 0; w2 < 2; ++w2) {
            u32x4 w, x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float p0 = __builtin_amdgcn_exp2f(sv[w2 * 8 + 2 * e] * a.cl2);
              const float p1 = __builtin_amdgcn_exp2f(sv[w2 * 8 + 2 * e + 1] * a.cl2);
              w[e] = pack_bf16(p0, p1);
              x[e] = pack_bf16(p0 * dp[w2 * 8 + 2 * e], p1 * dp[w2 * 8 + 2 * e + 1]);
            }
            pf[qb * 2 + w2] = __builtin_bit_cast(bf16x8, w);
            sf[qb * 2 + w2] = __builtin_bit_cast(bf16x8, x);
            if constexpr (STRIP) {
              if (keys_here)
                *reinterpret_cast<u32x4 *>(strip + (int64_t)(qt0 + u) * 4096 + (qb * 2 + w2) * 512 + lane * 8) = x;
            }
          }
        };
        bf16x8 gt[2][2][2 * AH], qt2[2][2][2 * AH];  // [qb][kk & 1][db]: dO^T and Q^T fragments
        auto fetch_t = [&](int qb) __attribute__((always_inline)) {
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int db = 0; db < 2 * AH; ++db) {
              gt[qb][k2][db] = tl.read_cols(sc.dOs[u][db >> 1], (qb * 2 + k2) * 16, db & 1);
              qt2[qb][k2][db] = tl.read_cols(sc.Qt[u][db >> 1], (qb * 2 + k2) * 16, db & 1);
            }
        };
        auto g34 = [&](int qb) __attribute__((always_inline)) {
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int db = 0; db < 2 * AH; ++db) {
              dv[db] = mfma_32x32x16(gt[qb][k2][db], pf[qb * 2 + k2], dv[db]);
              dk_[db] = mfma_32x32x16(qt2[qb][k2][db], sf[qb * 2 + k2], dk_[db]);
            }
        };
        // without a mask the tiles of a stage are all walked, and the first reads of every tile
        // after the stage's first were issued beside the previous tile's last MFMA group
        if (CAUSAL || u == 0) fetch(u, 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch(u, 1);
        g12(0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_t(0);
        g12(1);
        softmax_bwd(0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_t(1);
        g34(0);
        softmax_bwd(1);
        __builtin_amdgcn_sched_barrier(0);
        // the first reads of the stage's next tile go beside this tile's last eight MFMAs
        // (their registers are free again), so that tile does not start by waiting for LDS
        // (past the end of the rows the tile is not walked and what was read is dropped)
        if (!CAUSAL && u + 1 < NQ) fetch(u + 1, 0);
        g34(1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    if constexpr (STRIP) {  // this stage's strip stores stay in flight: four a tile, behind the next stage's loads
      if (keys_here && active(0) && active(NQ - 1)) wait_loads_before_stores<4 * NQ>();
      else wait_vmem();
      barrier_lds();
    } else {
      wait_vmem();
      __syncthreads();
    }
    i = inext; i0 = i0next;
  };
  while (i0 < i_end) {
    stage(stage0[grp], stage1[grp]);
    if (i0 >= i_end) break;
    stage(stage1[grp], stage0[grp]);
  }

  if constexpr (QS > 1) {
    // groups 1 .. QS - 1 leave dV in the first stage buffers and dK in the second, group 0 adds them
    static_assert((QS - 1) * WK * 32 * A * 4 <= QS * (int)sizeof(Stage), "room for the groups' sums");
    auto slot = [&](unsigned char *o, int g, int db) {
      return reinterpret_cast<f32x4 *>(o + (((g - 1) * WK + wave) * 2 * AH + db) * 4096);
    };
    if (grp > 0) {
#pragma unroll
      for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          slot(buf0, grp, db)[g * 64 + lane] = f32x4{dv[db][g * 4], dv[db][g * 4 + 1], dv[db][g * 4 + 2], dv[db][g * 4 + 3]};
          slot(buf1, grp, db)[g * 64 + lane] = f32x4{dk_[db][g * 4], dk_[db][g * 4 + 1], dk_[db][g * 4 + 2], dk_[db][g * 4 + 3]};
        }
    }
    __syncthreads();
    if (grp == 0) {
      for (int q = 1; q < QS; ++q)
#pragma unroll
        for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 x = slot(buf0, q, db)[g * 64 + lane], y = slot(buf1, q, db)[g * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) { dv[db][g * 4 + e] += x[e]; dk_[db][g * 4 + e] += y[e]; }
          }
    }
    __syncthreads();  // the epilogue writes to the buffers that the other waves just read
    if (grp > 0) return;
  }

  if (gridDim.y > 1) {  // fp32 partial sums: [dV | dK][split][head][key][64]
    const int64_t heads = a.by_heads.d;
    const int64_t key = wkey0 + col;
    float *pv = a.part + (((int64_t)blockIdx.y * heads + head) * a.L + key) * A;
    float *pk = pv + (int64_t)gridDim.y * heads * a.L * A;
    if (key < a.L) {
#pragma unroll
      for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int off = db * 32 + g * 8 + half * 4;
          const f32x4 w = {dv[db][g * 4 + 0], dv[db][g * 4 + 1], dv[db][g * 4 + 2], dv[db][g * 4 + 3]};
          *reinterpret_cast<f32x4 *>(pv + off) = w;
          const f32x4 x = {dk_[db][g * 4 + 0] * a.scale, dk_[db][g * 4 + 1] * a.scale,
                           dk_[db][g * 4 + 2] * a.scale, dk_[db][g * 4 + 3] * a.scale};
          *reinterpret_cast<f32x4 *>(pk + off) = x;
        }
    }
    return;
  }

  // the wave's 32 x 64 blocks of dV and dK leave through its own LDS tile as whole 128-byte rows
  // (every wave is past the loop's last barrier and no load is in flight: the buffers are free)
  unsigned char *ot = wave < 2 ? (wave == 0 ? stage0[0].Qt[0][0] : stage1[0].Qt[0][0])
                               : (wave == 2 ? stage0[0].dOs[0][0] : stage1[0].dOs[0][0]);
#pragma unroll
  for (int ah = 0; ah < AH; ++ah) {  // one half of the head at a time through the wave's tile
    stage_block_T(ot, 0, dv[2 * ah], dv[2 * ah + 1], 1.0f, lane);
    stage_block_T(ot, 32, dk_[2 * ah], dk_[2 * ah + 1], a.scale, lane);
    flush_rows<32>(ot, 0, a.dV + kv_off + (int64_t)wkey0 * kv_ld + ah * 64, a.L - wkey0, lane, (int)kv_ld);
    flush_rows<32>(ot, 32, a.dK + kv_off + (int64_t)wkey0 * kv_ld + ah * 64, a.L - wkey0, lane, (int)kv_ld);
  }
}

template <int NQ, bool CAUSAL, int AH, int WK, int QS>
__global__ void __launch_bounds__(64 * WK * QS, AH == 2 ? 1 : 2) fused_bwd_dkdv_kernel(BwdArgs a, TileOrder order) {
  // The two stage buffers are separate objects, each addressed by name, so that the
  // compiler knows a direct load into one cannot alias the LDS reads of the other.
  __shared__ __attribute__((aligned(16))) unsigned char buf0[QS * sizeof(DkdvStage<NQ, AH>)], buf1[sizeof(buf0)];
  dkdv_body<NQ, CAUSAL, AH, WK, QS>(a, order, blockIdx.x, gridDim.x, buf0, buf1);
}

// The backward's first kernel in the two-pass layout: the same, and dS^T as a strip of 64 x 64 tiles, key tile by key
// tile (the layout of rsa_strip.hip with rows and keys changed over), for the pass that forms dQ.
template <bool CAUSAL, int AH, int WK, int QS>
__global__ void __launch_bounds__(64 * WK * QS, AH == 2 ? 1 : 2) strip_collect_keys_kernel(BwdArgs a, TileOrder order) {
  constexpr int NQ = QS == 1 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) unsigned char buf0[QS * sizeof(DkdvStage<NQ, AH>)], buf1[sizeof(buf0)];
  dkdv_body<NQ, CAUSAL, AH, WK, QS, true>(a, order, blockIdx.x, gridDim.x, buf0, buf1);
}

// ---------------------------------------------------------------------- dQ ---
// NK: key tiles per stage (one barrier per stage).  RW waves share the work-group's rows, R each; KS groups of
// such waves share the keys, as in the forward.
template <int AH, int NK>
struct DqStage { unsigned char K[NK][AH][kTileBytes], V[NK][AH][kTileBytes]; };
template <int R, bool CAUSAL, bool PRE, int AH, int NK, int RW, int KS>
__device__ __forceinline__ void dq_body(const BwdArgs &a, const TileOrder &order, uint32_t id, uint32_t ids,
                                        unsigned char *buf0, unsigned char *buf1) {
  constexpr int QB = R / 32;
  constexpr int BM = RW * R;
  constexpr int A = 64 * AH;  // a head of 128 is two halves of 64: two LDS tiles per 64 keys
  using Stage = DqStage<AH, NK>;
  Stage *const stage0 = reinterpret_cast<Stage *>(buf0), *const stage1 = reinterpret_cast<Stage *>(buf1);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % RW;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / RW;
  const int col = lane & 31, half = lane >> 5;
  uint32_t head_, qt_;  // (order: see the forward)
  if (CAUSAL && order.by_length) {
    longest_first(id, a.by_heads, head_, qt_);
  } else {
    const uint32_t wg = xcd_remap(id, ids, blockIdx.y);
    head_ = order.by_tiles(wg);
    qt_ = wg - head_ * order.by_tiles.d;
  }
  if (CAUSAL) qt_ = order.by_tiles.d - 1 - qt_;
  const int64_t head = settled(head_), qt = settled(qt_);
  const int64_t row0 = qt * BM;
  int n = CAUSAL ? a.map.rank_at((int)row0) : a.map.rb + (int)a.map.by_c((uint32_t)row0);  // rank that owns the first row (see the forward)
  if (n >= a.N) n %= a.N;
  // last token any row of the work-group may look at
  const int q_last = CAUSAL ? a.map.token_at((int)(row0 + BM < a.Lq ? row0 + BM : a.Lq) - 1) : 0;

  const int64_t kv_off = head_offset((uint32_t)head, a.by_Z, a.ks), q_off = head_offset((uint32_t)head, a.by_Z, a.qs);
  const int64_t o_off = head_offset((uint32_t)head, a.by_Z, a.os);
  const uint16_t *Qh = a.Q + q_off;
  const uint16_t *dOh = a.dO + o_off;
  const uint16_t *Kh = a.K + kv_off;
  const uint16_t *Vh = a.V + kv_off;
  const int64_t q_ld = a.qs[2], kv_ld = a.ks[2], o_ld = a.os[2];

  // Q and dO as B operands; -LSE / scale and -D of the lane's row, broadcast
  // over an accumulator, are what S'^T and dP'^T start from.
  bf16x8 qreg[QB][4 * AH], greg[QB][4 * AH];
  int64_t qrow[QB];
  int qtok[QB];      // global token index of the lane's row
  bool here[QB];
  f32x16 negl[QB], negd[QB];
  // this wave's rows (see the forward)
  const int64_t wblk = row0 + wave * R < a.Lq ? row0 + wave * R : a.Lq - R;
  const int64_t wrow = CAUSAL ? a.map.row_at((int)wblk) : wblk;
  const int wq_first = CAUSAL ? a.map.token_at((int)wblk) : 0, wq_last = wq_first + R - 1;

  const TileLanes tl(lane);

  f32x16 dq[2 * AH][QB];
#pragma unroll
  for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int v = 0; v < 16; ++v) dq[db][qb][v] = 0.f;

  // the ring walk, in stages of NK tiles, divided over gridDim.y work-groups (see the forward)
  const int nk = NK == 1 || ((int)(a.map.zigzag ? a.map.h : a.map.c) & (kTileKeys * NK - 1)) == 0 ? NK : 1;
  KeyWalk<CAUSAL> w, wg_;  // group 0's stage, this group's
  w.begin(a.map, n, a.N, nk == 2 ? 7 : 6, q_last, gridDim.y, blockIdx.y);
  const TileDMAT<RW> dma(wave, lane, (int)kv_ld);
  auto load_stage = [&](int64_t k0, Stage &sn) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NK; ++u) {
      if (u < nk) {
#pragma unroll
        for (int ah = 0; ah < AH; ++ah) {
          dma.load(Kh + (k0 + u * kTileKeys) * kv_ld + ah * 64, sn.K[u][ah]);
          dma.load(Vh + (k0 + u * kTileKeys) * kv_ld + ah * 64, sn.V[u][ah]);
        }
      }
    }
  };

  if (KS > 1) { wg_ = w; wg_.skip(grp); }
  KeyWalk<CAUSAL> &g = KS == 1 ? w : wg_;
  if (g.have) load_stage(g.key(), stage0[grp]);
  // The rows this wave keeps in registers are fetched after the first stage's tiles are on their
  // way, so that the two latencies overlap (short walks, e.g. a few hundred projected keys, are
  // mostly prologue).
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    int64_t blk = row0 + wave * R + qb * 32;  // the block of 32 rows is whole or absent
    here[qb] = blk < a.Lq;
    if (!here[qb]) blk = a.Lq - 32;
    qrow[qb] = (CAUSAL ? a.map.row_at((int)blk) : blk) + (here[qb] ? col : 31);  // (one row for all lanes: see the forward)
    qtok[qb] = CAUSAL ? a.map.token_at((int)blk) + col : 0;
#pragma unroll
    for (int dk = 0; dk < 4 * AH; ++dk) {
      qreg[qb][dk] = *reinterpret_cast<const bf16x8 *>(Qh + qrow[qb] * q_ld + dk * 16 + half * 8);
      greg[qb][dk] = *reinterpret_cast<const bf16x8 *>(dOh + qrow[qb] * o_ld + dk * 16 + half * 8);
    }
    float l2, dd;
    if (PRE) {
      // D = sum_a dO_a O_a: this lane holds half of the row's elements, the lane 32 away the rest
      float acc = 0.f;
#pragma unroll
      for (int dk = 0; dk < 4 * AH; ++dk) {
        const u32x4 x = __builtin_bit_cast(u32x4, greg[qb][dk]);
        const u32x4 y = *reinterpret_cast<const u32x4 *>(a.O + o_off + qrow[qb] * o_ld + dk * 16 + half * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc = fmaf(bf16_to_f32(x[e] & 0xffffu), bf16_to_f32(y[e] & 0xffffu), acc);
          acc = fmaf(bf16_to_f32(x[e] >> 16), bf16_to_f32(y[e] >> 16), acc);
        }
      }
      dd = -xhalf_sum(acc);
      l2 = -a.LSE[head * a.Lq + qrow[qb]] * a.inv_scale;
      if (here[qb] && blockIdx.y == 0 && grp == 0) {
        if (half == 0) {
          a.nD_out[head * a.Lq + qrow[qb]] = dd;
          a.nL_out[head * a.Lq + qrow[qb]] = l2;
        }
      }
    } else {
      l2 = a.nL[head * a.Lq + qrow[qb]];
      dd = a.nD[head * a.Lq + qrow[qb]];
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) { negl[qb][v] = l2; negd[qb][v] = dd; }
  }
  wait_vmem();
  __syncthreads();
  // one stage: start the loads of the next stage into sn, compute on sc
  auto stage = [&](Stage &sc, Stage &sn) __attribute__((always_inline)) {
    const int ks0 = g.key();
    const bool mine = KS == 1 || g.have;
    w.skip(KS);
    if (KS > 1) wg_.skip(KS);
    if (g.have) load_stage(g.key(), sn);

#pragma unroll
    for (int u = 0; u < NK; ++u) {
    const int k0 = ks0 + u * kTileKeys;
    if (mine && u < nk && (!CAUSAL || k0 <= wq_last)) {
      const bool domask = CAUSAL && k0 + kTileKeys - 1 > wq_first;
      bf16x8 sf[QB][4];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        f32x16 s[QB], dp[QB];
#pragma unroll
        for (int dk = 0; dk < 4 * AH; ++dk) {
          const bf16x8 ka = tl.read_rows(sc.K[u][dk >> 2], kb * 32, dk & 3);
          const bf16x8 va = tl.read_rows(sc.V[u][dk >> 2], kb * 32, dk & 3);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            s[qb] = mfma_32x32x16(ka, qreg[qb][dk], dk == 0 ? negl[qb] : s[qb]);
            dp[qb] = mfma_32x32x16(va, greg[qb][dk], dk == 0 ? negd[qb] : dp[qb]);
          }
        }
        if (domask) {  // uniform over the wave: only tiles on the diagonal pay for the mask
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            // keys of the block of 32 that the lane's row sees: the first n
            const uint32_t seen = low_bits(qtok[qb] + 1 - k0 - kb * 32 - half * 4);
#pragma unroll
            for (int v = 0; v < 16; ++v) s[qb][v] = keep_bit(s[qb][v], seen, (v >> 2) * 8 + (v & 3));
          }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
          for (int v = 0; v < 16; ++v) dp[qb][v] *= __builtin_amdgcn_exp2f(s[qb][v] * a.cl2);
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            u32x4 w = {pack_bf16(dp[qb][u * 8 + 0], dp[qb][u * 8 + 1]), pack_bf16(dp[qb][u * 8 + 2], dp[qb][u * 8 + 3]),
                       pack_bf16(dp[qb][u * 8 + 4], dp[qb][u * 8 + 5]), pack_bf16(dp[qb][u * 8 + 6], dp[qb][u * 8 + 7])};
            sf[qb][kb * 2 + u] = __builtin_bit_cast(bf16x8, w);
          }
        }
      }
#pragma unroll
      for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const bf16x8 ka = tl.read_cols(sc.K[u][db >> 1], kk * 16, db & 1);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) dq[db][qb] = mfma_32x32x16(ka, sf[qb][kk], dq[db][qb]);
        }
    }

    }

    wait_vmem();
    __syncthreads();
  };
  while (w.have) {
    stage(stage0[grp], stage1[grp]);
    if (!w.have) break;
    stage(stage1[grp], stage0[grp]);
  }

  if constexpr (KS > 1) {  // groups 1 .. KS - 1 leave their sums in the stage buffers, group 0 adds them
    static_assert(QB == 1, "32 rows per wave");
    constexpr int PARTS = 2 * AH;  // of 32 columns: 4 KiB per wave
    static_assert((PARTS * (KS - 1) + 1) / 2 * RW * 4096 <= KS * (int)sizeof(Stage), "room for the groups' sums");
    auto slot = [&](int g, int part) -> f32x4 * {
      const int i = (g - 1) * PARTS + part;
      return reinterpret_cast<f32x4 *>(((i & 1) ? buf1 : buf0) + ((i >> 1) * RW + wave) * 4096);
    };
    if (grp > 0) {
#pragma unroll
      for (int db = 0; db < PARTS; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          slot(grp, db)[g * 64 + lane] =
              f32x4{dq[db][0][g * 4 + 0], dq[db][0][g * 4 + 1], dq[db][0][g * 4 + 2], dq[db][0][g * 4 + 3]};
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int q = 1; q < KS; ++q)
#pragma unroll
        for (int db = 0; db < PARTS; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 x = slot(q, db)[g * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) dq[db][0][g * 4 + e] += x[e];
          }
    }
    __syncthreads();  // the epilogue writes to the buffers that the other waves just read
    if (grp > 0) return;
  }

  if (gridDim.y > 1) {  // fp32 partial sum of this split: [split][head][row][64]
    const int64_t heads = a.by_heads.d;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      if (here[qb]) {
        float *po = a.part + (((int64_t)blockIdx.y * heads + head) * a.Lq + qrow[qb]) * A + half * 4;
#pragma unroll
        for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 w = {dq[db][qb][g * 4 + 0] * a.scale, dq[db][qb][g * 4 + 1] * a.scale,
                             dq[db][qb][g * 4 + 2] * a.scale, dq[db][qb][g * 4 + 3] * a.scale};
            *reinterpret_cast<f32x4 *>(po + db * 32 + g * 8) = w;
          }
      }
    }
    return;
  }

  // the wave's R x 64 block of dQ leaves through its own LDS tile as whole 128-byte rows
  unsigned char *ot = ((wave & 1) ? buf1 : buf0) + (wave >> 1) * kTileBytes;
  const int64_t rows_here = a.Lq - (row0 + wave * R);
#pragma unroll
  for (int ah = 0; ah < AH; ++ah) {  // one half of the head at a time through the wave's tile
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) stage_block_T(ot, qb * 32, dq[2 * ah][qb], dq[2 * ah + 1][qb], a.scale, lane);
    flush_rows<R>(ot, 0, a.dQ + q_off + wrow * q_ld + ah * 64, rows_here, lane, (int)q_ld);
  }
}

template <int R, bool CAUSAL, bool PRE, int AH, int NK, int RW, int KS>
__global__ void __launch_bounds__(64 * RW * KS, R == 64 ? 1 : 2) fused_bwd_dq_kernel(BwdArgs a, TileOrder order) {
  // (two named stage buffers: see the dK/dV kernel)
  __shared__ __attribute__((aligned(16))) unsigned char buf0[KS * sizeof(DqStage<AH, NK>)], buf1[sizeof(buf0)];
  dq_body<R, CAUSAL, PRE, AH, NK, RW, KS>(a, order, blockIdx.x, gridDim.x, buf0, buf1);
}

// --------------------------------------------------------- dQ and dK, dV ---
// Both kernels in one grid, for sizes where each alone leaves the chip partly idle.
// Work-groups are dealt out in eights (one per XCD), the two kinds in turn in proportion to their numbers.
struct BothArgs {
  BwdArgs a;
  TileOrder kv, q;
  uint32_t kv_wgs, q_wgs, kv_eights;
  FastDiv by_eights;  // eights of both kinds
};
template <bool CAUSAL, int AH, int NQ, int WK, int QS, int NK, int RW, int KS>
__global__ void __launch_bounds__(64 * WK * QS, AH == 2 ? 1 : 2) fused_bwd_both_kernel(BothArgs b) {
  static_assert(WK * QS == RW * KS, "one block size");
  constexpr int KV = QS * (int)sizeof(DkdvStage<NQ, AH>), Q = KS * (int)sizeof(DqStage<AH, NK>);
  __shared__ __attribute__((aligned(16))) unsigned char buf0[KV > Q ? KV : Q], buf1[KV > Q ? KV : Q];
  const uint32_t e = blockIdx.x >> 3, x = blockIdx.x & 7, up = b.by_eights.d - 1;
  const uint32_t before = b.by_eights(e * b.kv_eights + up), upto = b.by_eights((e + 1) * b.kv_eights + up);
  if (upto > before) {
    const uint32_t id = before * 8 + x;
    if (id < b.kv_wgs) dkdv_body<NQ, CAUSAL, AH, WK, QS>(b.a, b.kv, id, b.kv_wgs, buf0, buf1);
  } else {
    const uint32_t id = (e - before) * 8 + x;
    if (id < b.q_wgs) dq_body<32, CAUSAL, false, AH, NK, RW, KS>(b.a, b.q, id, b.q_wgs, buf0, buf1);
  }
}

// out (bf16) = sum over the splits of part[s][i], in a fixed order; n4 groups of four per split
// (the partial sums are dense (head, row, A); `lay` says where a row of the output tensor lives).  A grid of two rows
// adds up two tensors, out1's sums behind out's: dV and dK in one launch (two: 3.9 us each where they are small).
__global__ void __launch_bounds__(kReduceBlock) qsplit_reduce_kernel(const float *part, uint16_t *out, uint16_t *out1,
                                                                     int64_t n4, int splits, int A, OutLayout lay) {
  if (blockIdx.y) {
    part += (int64_t)splits * n4 * 4;
    out = out1;
  }
  const int64_t i = (int64_t)blockIdx.x * kReduceBlock + threadIdx.x;
  if (i >= n4) return;
  const f32x4 *p = reinterpret_cast<const f32x4 *>(part) + i;
  const f32x4 s = sum_of_splits(splits, [&](int k) { return p[(int64_t)k * n4]; });
  const u32x2 w = {pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3])};
  const int64_t e = i * 4;  // (A is 64 or 128)
  *reinterpret_cast<u32x2 *>(out + lay.row_off(e >> (A == 64 ? 6 : 7)) + (e & (A - 1))) = w;
}

static BwdArgs make_bwd_args(const Dims &d, const void *dO, const void *Q, const void *K,
                             const void *V, const float *nL, const float *nD, void *dQ, void *dK,
                             void *dV) {
  BwdArgs a;
  a.Q = (const uint16_t *)Q;
  a.K = (const uint16_t *)K; a.V = (const uint16_t *)V;
  a.dO = (const uint16_t *)dO; a.nL = nL; a.nD = nD;
  a.dQ = (uint16_t *)dQ; a.dK = (uint16_t *)dK; a.dV = (uint16_t *)dV;
  a.part = nullptr; a.strip = nullptr;
  a.O = nullptr; a.LSE = nullptr; a.nL_out = nullptr; a.nD_out = nullptr;
  a.L = d.L; a.c = d.c; a.Lq = d.Lq; a.map = make_row_map(d);
  a.N = d.N; a.by_Z = make_fast_div(d.Z); a.by_heads = make_fast_div((int64_t)d.B * d.Z); a.cl2 = d.scale * kLog2e; a.scale = d.scale; a.inv_scale = 1.0f / d.scale;
  for (int k = 0; k < 3; ++k) { a.qs[k] = d.qs[k]; a.ks[k] = d.ks[k]; a.os[k] = d.os[k]; }
  return a;
}

hipError_t fused_bwd_preprocess(const Dims &d, const void *dO, const void *O, const float *LSE,
                                float *nD, float *nL, hipStream_t st) {
  const int64_t rows = (int64_t)d.B * d.Z * d.Lq;
  dim3 grid((unsigned)((rows * 8 + 255) / 256));
  hipLaunchKernelGGL(bwd_preprocess_kernel, grid, dim3(256), 0, st, (const uint16_t *)dO,
                     (const uint16_t *)O, LSE, nD, nL, rows, d.A, 1.0f / d.scale,
                     make_out_layout(d.os, d.Lq, d.Z));
  return hipGetLastError();
}

hipError_t qsplit_reduce(const float *part, void *out, void *out1, int64_t n4, int splits, int A, const OutLayout &lay,
                         hipStream_t st) {
  const dim3 grid(reduce_grid(n4).x, out1 ? 2 : 1);
  hipLaunchKernelGGL(qsplit_reduce_kernel, grid, dim3(kReduceBlock), 0, st, part, (uint16_t *)out, (uint16_t *)out1, n4,
                     splits, A, lay);
  return hipGetLastError();
}

// the order of a kernel whose work-groups own `own` of `n` rows (or keys) of every head
static TileOrder make_order(const Dims &d, int64_t n, int own, int splits) {
  TileOrder o;
  o.by_tiles = make_fast_div((n + own - 1) / own);
  o.by_length = order_by_length(d, splits, (int64_t)128 << 20);
  return o;
}

template <int NQ, int AH, int WK, int QS, int MASKS = kBothMasks>
static hipError_t launch_dkdv(const Dims &d, const BwdArgs &a, int splits, hipStream_t st) {
  const TileOrder o = make_order(d, d.L, 32 * WK, splits);
  const dim3 grid((unsigned)((int64_t)d.B * d.Z * o.by_tiles.d), (unsigned)splits), block(64 * WK * QS);
  if (!(MASKS & (d.causal ? kCausal : kNoMask))) return hipErrorInvalidValue;
  if constexpr (MASKS & kCausal)
    if (d.causal) hipLaunchKernelGGL((fused_bwd_dkdv_kernel<NQ, true, AH, WK, QS>), grid, block, 0, st, a, o);
  if constexpr (MASKS & kNoMask)
    if (!d.causal) hipLaunchKernelGGL((fused_bwd_dkdv_kernel<NQ, false, AH, WK, QS>), grid, block, 0, st, a, o);
  return hipGetLastError();
}

// dK/dV of few keys that many query rows see (projected keys): the waves per work-group, on WK blocks of 32 keys in QS
// groups, and the splits of the rows' walk with the least estimated time.  Work-groups run in rounds of `places`; a
// stage of a walk (two row tiles, or one per group) takes `alone` .. `full` us by how full the CUs are.  The constants
// were fitted to a sweep of 5 .. 96 heads of 896 .. 87808 rows and 64 .. 512 keys, heads of 64 and 128, all shapes and
// splits: what is picked is within 1 % of the best but for one call (4 %).  (Whole backward, us, splits of at least
// eight stages -> this: 2176 rows, 64 keys, 12 heads: 31.8 -> 20.6; 13824, 64, 5: 36.8 -> 28.6; 7488, 512, 15: 82.1 ->
// 76.8; 16384, 512, 64: 576 -> 553; heads of 128, 2048, 128, 12: 53.6 -> 33.6; 16384, 256, 64: 756 -> 706.)
struct DkdvPlan { int WK, QS, splits; };
static DkdvPlan plan_dkdv(const Dims &d) {
  struct Shape { int WK, QS, places; float fixed, alone, full; };
  static const Shape wide[] = {{4, 1, 256, 6.2f, 3.1f, 3.1f}, {2, 2, 256, 5.8f, 1.8f, 1.8f}};
  static const Shape narrow[] = {
      {4, 1, 512, 3.4f, 1.4f, 2.17f}, {1, 4, 256, 3.2f, 1.09f, 1.17f}, {2, 2, 512, 2.8f, 1.27f, 1.5f}};
  const int64_t heads = (int64_t)d.B * d.Z;
  DkdvPlan best{4, 1, 1};
  float least = 1e30f;
  for (int k = 0; k < (d.A == 128 ? 2 : 3); ++k) {
    const Shape &c = d.A == 128 ? wide[k] : narrow[k];
    const int64_t stages = c.QS == 1 ? (d.Lq / 64 + 1) / 2 : d.Lq / 64;
    for (int s = 1; s <= 64 && s <= stages; s *= 2) {
      const int64_t steps = ((stages + s - 1) / s + c.QS - 1) / c.QS;
      const float wgs = (float)(heads * ((d.L + 32 * c.WK - 1) / (32 * c.WK)) * s), rounds = wgs / (float)c.places;
      float fill = c.places == 512 ? wgs * (1.0f / 256) - 1.0f : rounds;
      fill = fill < 0.0f ? 0.0f : (fill > 1.0f ? 1.0f : fill);
      float us = (0.85f * ceilf(rounds) + 0.15f * fmaxf(rounds, 1.0f)) *
                 (c.fixed + (float)steps * (c.alone + (c.full - c.alone) * fill));
      if (s > 1) us += 1.6f + (float)s * (0.05f + (float)(heads * d.L * d.A) * (8.0f / 3.5e6f));
      if (us < least) { least = us; best = {c.WK, c.QS, s}; }
    }
  }
  return best;
}

static int both_groups(const Dims &d);
int fused_bwd_dkdv_splits(const Dims &d) { return both_groups(d) ? 1 : plan_dkdv(d).splits; }

hipError_t fused_bwd_dkdv(const Dims &d, const void *dO, const void *Q, const void *K,
                          const void *V, const float *nL, const float *nD, void *dK, void *dV,
                          hipStream_t st, float *part, int splits) {
  BwdArgs a = make_bwd_args(d, dO, Q, K, V, nL, nD, nullptr, dK, dV);
  a.part = part;
  if (!part) splits = 1;
  // Few work-groups of four waves (W: their number): fewer keys per work-group and several groups of waves on its
  // query rows, as in the forward (same sweep, forward + backward, us: W = 8: 29.4 -> 26.2; 96: 49.4 -> 44.9;
  // 252 causal: 104 -> 98).
  const int64_t W = (int64_t)d.B * d.Z * ((d.L + 127) / 128);
  hipError_t e;
  if (!d.causal && (splits > 1 || d.Lq > d.L)) {  // projected keys
    const DkdvPlan p = plan_dkdv(d);
    if (d.A == 128) {
      e = p.QS == 2 ? launch_dkdv<1, 2, 2, 2, kNoMask>(d, a, splits, st) : launch_dkdv<2, 2, 4, 1>(d, a, splits, st);
    } else if (p.QS == 4) {
      e = launch_dkdv<1, 1, 1, 4>(d, a, splits, st);
    } else {
      e = p.QS == 2 ? launch_dkdv<1, 1, 2, 2>(d, a, splits, st) : launch_dkdv<2, 1, 4, 1>(d, a, splits, st);
    }
  } else if (d.A == 128) e = launch_dkdv<2, 2, 4, 1>(d, a, 1, st);
  else if (W > (d.causal ? 256 : 128)) e = launch_dkdv<2, 1, 4, 1>(d, a, 1, st);
  else if (W <= 32) e = launch_dkdv<1, 1, 1, 4>(d, a, 1, st);
  else if (W <= 128) e = launch_dkdv<1, 1, 2, 4>(d, a, 1, st);
  else e = launch_dkdv<1, 1, 2, 2>(d, a, 1, st);
  if (e != hipSuccess || splits == 1) return e;
  const int64_t n4 = (int64_t)d.B * d.Z * d.L * (d.A / 4);
  return qsplit_reduce(part, dV, dK, n4, splits, d.A, make_out_layout(d.ks, d.L, d.Z), st);
}

template <int AH, int WK, int QS>
static hipError_t launch_collect_keys(const Dims &d, const BwdArgs &a, hipStream_t st) {
  const TileOrder o = make_order(d, d.L, 32 * WK, 1);
  const dim3 grid((unsigned)((int64_t)d.B * d.Z * o.by_tiles.d)), block(64 * WK * QS);
  if (d.causal) hipLaunchKernelGGL((strip_collect_keys_kernel<true, AH, WK, QS>), grid, block, 0, st, a, o);
  else hipLaunchKernelGGL((strip_collect_keys_kernel<false, AH, WK, QS>), grid, block, 0, st, a, o);
  return hipGetLastError();
}
hipError_t collect_keys(const Dims &d, const void *dO, const void *Q, const void *K, const void *V, const float *nL,
                        const float *nD, void *dK, void *dV, void *strip, int groups, hipStream_t st) {
  BwdArgs a = make_bwd_args(d, dO, Q, K, V, nL, nD, nullptr, dK, dV);
  a.strip = (uint16_t *)strip;
  if (d.A == 128) return groups > 1 ? launch_collect_keys<2, 2, 2>(d, a, st) : launch_collect_keys<2, 4, 1>(d, a, st);
  if (groups == 4) return launch_collect_keys<1, 2, 4>(d, a, st);
  return groups == 2 ? launch_collect_keys<1, 2, 2>(d, a, st) : launch_collect_keys<1, 4, 1>(d, a, st);
}

template <bool PRE, int AH, int NK, int RW, int KS, int MASKS = kBothMasks>
static hipError_t launch_dq_as(const Dims &d, const BwdArgs &a, int splits, hipStream_t st) {
  const TileOrder o = make_order(d, d.Lq, 32 * RW, splits);
  const dim3 grid((unsigned)((int64_t)d.B * d.Z * o.by_tiles.d), (unsigned)splits), block(64 * RW * KS);
  if (!(MASKS & (d.causal ? kCausal : kNoMask))) return hipErrorInvalidValue;
  if constexpr (MASKS & kCausal)
    if (d.causal) hipLaunchKernelGGL((fused_bwd_dq_kernel<32, true, PRE, AH, NK, RW, KS>), grid, block, 0, st, a, o);
  if constexpr (MASKS & kNoMask)
    if (!d.causal) hipLaunchKernelGGL((fused_bwd_dq_kernel<32, false, PRE, AH, NK, RW, KS>), grid, block, 0, st, a, o);
  return hipGetLastError();
}

// (PRE: heads of 64 only, see fused_backward)
template <bool PRE>
static hipError_t launch_dq(const Dims &d, const BwdArgs &a, int splits, hipStream_t st) {
  // (few work-groups: see the dK/dV kernel; W = 8: 29.4 -> 26.3, 96: 49.4 -> 44.1, 252 causal: 104 -> 94; heads
  // of 128, W = 64 causal: 100 -> 89, 256: 174 -> 162)
  const int64_t W = (int64_t)d.B * d.Z * ((d.Lq + 127) / 128);
  if constexpr (!PRE) {
    if (d.A == 128) {  // one key tile (two LDS tiles) per stage
      if (splits > 1 || W > 256) return launch_dq_as<PRE, 2, 1, 4, 1>(d, a, splits, st);
      if (d.causal || W <= 128) return launch_dq_as<PRE, 2, 1, 2, 2>(d, a, 1, st);
      return launch_dq_as<PRE, 2, 1, 4, 2, kNoMask>(d, a, 1, st);
    }
  }
  if (splits > 1 || W > 256) return launch_dq_as<PRE, 1, 2, 4, 1>(d, a, splits, st);
  if (W <= 32) return launch_dq_as<PRE, 1, 1, 1, 4>(d, a, 1, st);
  return launch_dq_as<PRE, 1, 1, 2, 2>(d, a, 1, st);
}

// dQ = sum of the split walks' partial sums
static hipError_t dq_reduce(const Dims &d, const float *part, void *dQ, int splits, hipStream_t st) {
  const int64_t n4 = (int64_t)d.B * d.Z * d.Lq * (d.A / 4);
  return qsplit_reduce(part, dQ, nullptr, n4, splits, d.A, make_out_layout(d.qs, d.Lq, d.Z), st);
}

hipError_t fused_bwd_dq(const Dims &d, const void *dO, const void *Q, const void *K, const void *V,
                        const float *nL, const float *nD, void *dQ, hipStream_t st, float *part,
                        int splits) {
  BwdArgs a = make_bwd_args(d, dO, Q, K, V, nL, nD, dQ, nullptr, nullptr);
  a.part = part;
  if (!part) splits = 1;
  hipError_t e = launch_dq<false>(d, a, splits, st);
  if (e != hipSuccess || splits == 1) return e;
  return dq_reduce(d, part, dQ, splits, st);
}

// The dQ kernel with the preprocess in its prologue: also writes -D and -LSE / scale.
hipError_t fused_bwd_dq_pre(const Dims &d, const void *dO, const void *Q, const void *K, const void *V,
                            const void *O, const float *LSE, float *nL, float *nD, void *dQ,
                            hipStream_t st, float *part, int splits) {
  BwdArgs a = make_bwd_args(d, dO, Q, K, V, nullptr, nullptr, dQ, nullptr, nullptr);
  a.O = (const uint16_t *)O; a.LSE = LSE; a.nL_out = nL; a.nD_out = nD;
  a.part = part;
  if (!part) splits = 1;
  hipError_t e = launch_dq<true>(d, a, splits, st);
  if (e != hipSuccess || splits == 1) return e;
  return dq_reduce(d, part, dQ, splits, st);
}

template <int AH, int NQ, int WK, int QS, int NK, int RW, int KS>
static hipError_t launch_both(const Dims &d, const BwdArgs &a, hipStream_t st) {
  BothArgs b;
  b.a = a;
  b.kv = make_order(d, d.L, 32 * WK, 1);
  b.q = make_order(d, d.Lq, 32 * RW, 1);
  const int64_t heads = (int64_t)d.B * d.Z;
  b.kv_wgs = (uint32_t)(heads * b.kv.by_tiles.d);
  b.q_wgs = (uint32_t)(heads * b.q.by_tiles.d);
  b.kv_eights = (b.kv_wgs + 7) / 8;
  b.by_eights = make_fast_div(b.kv_eights + (b.q_wgs + 7) / 8);
  const dim3 grid(8 * b.by_eights.d), block(64 * WK * QS);
  if (d.causal) hipLaunchKernelGGL((fused_bwd_both_kernel<true, AH, NQ, WK, QS, NK, RW, KS>), grid, block, 0, st, b);
  else hipLaunchKernelGGL((fused_bwd_both_kernel<false, AH, NQ, WK, QS, NK, RW, KS>), grid, block, 0, st, b);
  return hipGetLastError();
}

// Whether dQ and dK, dV go in one grid, behind the preprocess kernel: 0, or the groups of waves on a walk (then 128 / groups
// rows or keys per work-group).  One grid costs the preprocess launch (3 us and a second read of dO and O) and gives what
// two grids leave idle: half-filled rounds, prologues at HBM speed, under the causal mask the ends of the longest walks,
// which now lie beside the other kind's.  W: work-groups of 128 rows or keys per kind (512 places for A = 64, 256 for A =
// 128).  The lines are those of a sweep over 1 .. 1500 heads of 192 .. 65536 rows; backward, us, two grids -> one:
//   A = 64, four groups, W = 32: 512 rows 17.3 -> 13.9, 2048: 33.4 -> 19.6, 4096 causal: 69.5 -> 34.7;
//   two, W = 48: 512 rows 19.9 -> 14.1; causal W = 128: 20.8 -> 15.5, 4096 rows, W = 192: 103 -> 67, 32768, W = 256: 682 -> 607;
//   one, W = 128: 512 rows 20.8 -> 14.9, W = 384: 36.2 -> 32.2, 4096 rows: 208 -> 193, causal 167 -> 114, W = 768: 512 rows
//   63.6 -> 57.2; but 2048 rows, W = 512: 119 -> 124, W = 704: 180 -> 186, causal W = 1120: 164 -> 170 (whole rounds);
//   just above whole rounds each kind begins another, and one grid only one for both: 2048 rows, W = 544: 169 -> 149, 640: 172 ->
//   156, 672: 172 -> 177, 8192 rows, 576: 593 -> 563;
//   A = 128, two groups, W = 64: 512 rows 36.3 -> 18.5, 4096: 175 -> 74; one, W = 128: 512 rows 37.6 -> 25.4, 384: 78 -> 68,
//   causal 4096 rows, W = 256: 223 -> 148; but W = 192: 112 -> 129, 512: 142 -> 150.
static int both_groups(const Dims &d) {
  // (one rank's share of a longer sequence, or many rows of few keys: one kind's walks are far longer than the other's)
  const int64_t longer = d.L > d.Lq ? d.L : d.Lq, shorter = d.L > d.Lq ? d.Lq : d.L;
  if (longer > 2 * shorter && longer > 1024) return 0;
  const int64_t heads = (int64_t)d.B * d.Z, L = longer;
  const int64_t W = heads * ((d.L + 127) / 128 + (d.Lq + 127) / 128) / 2;
  if (d.A == 128) {
    if (W <= 64 || (d.causal && L > 512 && W <= 128)) return 2;
    if (W <= 128 || (d.causal ? W <= 460 : W > 256 && W <= 384)) return 1;
    return 0;
  }
  if (d.causal) {
    if (W <= 32 || (W <= 64 && L >= 2048)) return 4;
    if (W <= 128 || (W <= 224 && L >= 1024) || (W <= 256 && L >= 1536)) return 2;
    return W <= 640 || (W <= 768 && (L >= 4096 || L <= 512)) || (W <= 1536 && L <= 320) ? 1 : 0;
  }
  if (W <= 32) return 4;
  if (W <= 64) return 2;
  return (L <= 8192 && (W <= (L <= 2048 ? 460 : 384) || (W > 512 && W <= 640))) || (L <= 512 && W <= 1536) ? 1 : 0;
}

hipError_t fused_backward(const Dims &d, const void *dO, const void *Q, const void *K,
                          const void *V, const void *O, const float *LSE, void *dQ, void *dK,
                          void *dV, float *nD, float *nL, hipStream_t st, float *part,
                          int qsplits, int ksplits) {
  // the dQ kernel first: its prologue forms the row terms that the dK/dV kernel reads;
  // the two kernels' partial sums share `part`, one after the other.  (With heads of 128 the
  // prologue costs the dQ kernel more registers than it has: there the row terms come from
  // the preprocess kernel.)
  hipError_t e;
  // (dK, dV may lie over K, V: a dK/dV work-group has read its own keys by then and no other of its kind reads them, but the
  // dQ kind reads them all, and has to be done)
  const size_t kv = 2 * (size_t)((d.B - 1) * d.ks[0] + (d.Z - 1) * d.ks[1] + (d.L - 1) * d.ks[2] + d.A);
  const bool over = overlap(dK, kv, K, kv) || overlap(dK, kv, V, kv) || overlap(dV, kv, K, kv) || overlap(dV, kv, V, kv);
  if (const int groups = qsplits > 1 || over ? 0 : both_groups(d)) {
    e = fused_bwd_preprocess(d, dO, O, LSE, nD, nL, st);
    if (e != hipSuccess) return e;
    const BwdArgs a = make_bwd_args(d, dO, Q, K, V, nL, nD, dQ, dK, dV);
    if (d.A == 128) return groups == 2 ? launch_both<2, 1, 2, 2, 1, 2, 2>(d, a, st) : launch_both<2, 2, 4, 1, 1, 4, 1>(d, a, st);
    if (groups == 4) return launch_both<1, 1, 1, 4, 1, 1, 4>(d, a, st);
    return groups == 2 ? launch_both<1, 1, 2, 2, 1, 2, 2>(d, a, st) : launch_both<1, 2, 4, 1, 2, 4, 1>(d, a, st);
  }
  if (d.A == 128) {
    e = fused_bwd_preprocess(d, dO, O, LSE, nD, nL, st);
    if (e != hipSuccess) return e;
    e = fused_bwd_dq(d, dO, Q, K, V, nL, nD, dQ, st, part, ksplits);
  } else {
    e = fused_bwd_dq_pre(d, dO, Q, K, V, O, LSE, nL, nD, dQ, st, part, ksplits);
  }
  if (e != hipSuccess) return e;
  return fused_bwd_dkdv(d, dO, Q, K, V, nL, nD, dK, dV, st, part, qsplits);
}

}  // namespace rsa
