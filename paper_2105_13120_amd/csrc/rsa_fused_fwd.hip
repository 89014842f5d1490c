// Fused Ring Self-Attention forward (bf16, A = 64 or 128).
//
// One work-group owns RW*R query rows of one head (RW waves, R each) and walks the K/V chunks in
// ring order -- step t of rank n visits chunk j = (n - t) mod N, local chunk
// first (section 3.1) -- keeping a running row max and row sum, so the score
// strip S^n of Table 2 never reaches device memory.  The result is Eq. 1 /
// Eq. 3 exactly, up to summation order.
//
// K/V tiles reach LDS by direct global->LDS loads, two tiles per stage, double-buffered,
// one work-group barrier per stage.
//
// A head of 128 elements is handled as AH = 2 halves of 64: a 64-key tile is then two LDS tiles,
// the S^T contraction runs over both, and O^T has twice the accumulators.
//
// Data flow per 64-key tile and wave (R query rows):
//   S^T = K Q^T    A operand: K tile rows from LDS, B operand: Q^T in registers
//   softmax update on S^T: lane l owns query column l%32, so the row max and
//                  row sum are in-lane reductions plus one cross-half exchange
//   O^T += V^T P^T A operand: V^T through LDS transpose reads, B operand: P^T
//                  straight from the S^T accumulator registers (packed to bf16)
#include "rsa_fused_tile.h"
#include "rsa_kernels.h"

namespace rsa {

struct FwdArgs {
  const uint16_t *Q, *K, *V;
  uint16_t *O;
  float *LSE;
  int64_t L, c, Lq;
  int64_t qs[3], ks[3], os[3];  // element strides (batch, head, row) of Q; K and V; O
  RowMap map;            // local query row -> global token index
  int N;
  FastDiv by_tiles, by_heads, by_Z;  // row tiles of a head, heads, Z
  int by_length;         // causal: order of the row tiles over the work-groups (longest_first)
  float cl2;             // scale * log2(e)
  // split key walk (gridDim.y > 1): per split, head and row the unnormalised fp32 O and the pair
  // (stale max * cl2, row sum) it is relative to
  float *part_o, *part_ml;
};

// NK: key tiles per stage (one barrier per stage).  RW waves share the work-group's rows, R each; KS groups of
// such waves share its keys: group g takes every KS-th stage of the walk and the groups' results are merged in
// LDS.
// OWN (the two-pass layout, whose strip held them so): a tile's probabilities are rounded to bf16 against the tile's own
// maximum per row, its product with V is formed by itself and weighted, and sums are short and compensated.  The largest of
// a tile are then exact: RMS error of O against fp64, N(0, 1) inputs, 1e-3: 2.10 (576 rows), 1.99 (4096, causal), as the
// strip; 2.32, 2.12 against a common reference.  It costs a multiply-add per two scores (B8 Z16 L2048: 146 -> 159 us, 12 causal
// heads of 4096 44 -> 47, 128 of 512 13.4 -> 15.5).
template <int R, bool CAUSAL, int AH, int NK, int RW, int KS, bool OWN>
__global__ void __launch_bounds__(64 * RW * KS, (R == 32 && NK == 1 && AH == 1) ? 4 : 2) fused_fwd_kernel(FwdArgs a) {
  constexpr int QB = R / 32;
  constexpr int BM = RW * R;
  constexpr int A = 64 * AH;
  // The two stage buffers are separate objects, each addressed by name: the compiler then
  // knows that a direct load into one buffer cannot alias the LDS reads of the other and
  // does not wait for the load before them.
  __shared__ __attribute__((aligned(16))) unsigned char Ks0[KS][NK][AH][kTileBytes], Ks1[KS][NK][AH][kTileBytes];
  __shared__ __attribute__((aligned(16))) unsigned char Vs0[KS][NK][AH][kTileBytes], Vs1[KS][NK][AH][kTileBytes];

  // the walk's first maximum per row; every group's maximum and sum
  __shared__ float ref[KS == 1 ? 1 : RW][64], mls[KS == 1 ? 1 : KS][RW][2][64];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % RW;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / RW;
  const int col = lane & 31, half = lane >> 5;
  uint32_t head_, qt_;
  if (CAUSAL && a.by_length) {
    longest_first(blockIdx.x, a.by_heads, head_, qt_);
  } else {
    const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x, blockIdx.y);
    head_ = a.by_tiles(wg);
    qt_ = wg - head_ * a.by_tiles.d;
  }
  if (CAUSAL) qt_ = a.by_tiles.d - 1 - qt_;  // later rows see more keys
  const int64_t head = settled(head_), qt = settled(qt_);
  const int64_t row0 = qt * BM;  // first row of this work-group (causal: in the order of their tokens, see RowMap)
  // rank that owns the first row (modulo N: with projected keys, Table 3, the rows are not
  // tokens of the key sequence and any chunk may come first)
  int n = CAUSAL ? a.map.rank_at((int)row0) : a.map.rb + (int)a.map.by_c((uint32_t)row0);
  if (n >= a.N) n %= a.N;
  // last token any row of the work-group may look at
  const int q_last = CAUSAL ? a.map.token_at((int)(row0 + BM < a.Lq ? row0 + BM : a.Lq) - 1) : 0;

  const int64_t kv_off = head_offset((uint32_t)head, a.by_Z, a.ks);
  const uint16_t *Qh = a.Q + head_offset((uint32_t)head, a.by_Z, a.qs);
  const uint16_t *Kh = a.K + kv_off;
  const uint16_t *Vh = a.V + kv_off;
  const int64_t q_ld = a.qs[2], kv_ld = a.ks[2], o_ld = a.os[2];

  // Q^T operand: lane (col, half) holds Q[row][dk*16 + half*8 .. +8]
  bf16x8 qreg[QB][4 * AH];
  // The lane's row.  Of a block that is not there: the last of another, the same for all lanes, since products of equal rows
  // take less power (32 rows of it instead, us: 1150 heads of 192 rows, 1024 projected keys 100.4 -> 102.7, 1025 of 448 of 896 rows
  // 142 -> 145).
  int64_t qrow[QB];
  int qtok[QB];  // its global token index
  bool here[QB];     // (a block of 32 rows is whole or absent)
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    int64_t blk = row0 + wave * R + qb * 32;
    here[qb] = blk < a.Lq;
    if (!here[qb]) blk = a.Lq - 32;
    qrow[qb] = (CAUSAL ? a.map.row_at((int)blk) : blk) + (here[qb] ? col : 31);
    qtok[qb] = CAUSAL ? a.map.token_at((int)blk) + col : 0;
#pragma unroll
    for (int dk = 0; dk < 4 * AH; ++dk)
      qreg[qb][dk] = *reinterpret_cast<const bf16x8 *>(Qh + qrow[qb] * q_ld + dk * 16 + half * 8);
  }
  // this wave's rows, R of them in a run of tokens: the first one's place in the tensors, first and last token
  const int64_t wblk = row0 + wave * R < a.Lq ? row0 + wave * R : a.Lq - R;
  const int64_t wrow = CAUSAL ? a.map.row_at((int)wblk) : wblk;
  const int wq_first = CAUSAL ? a.map.token_at((int)wblk) : 0, wq_last = wq_first + R - 1;

  const TileLanes tl(lane);
  // A maximum as exponents are taken against it.  (OWN: the same rounded number in probabilities, weights and the LSE, and
  // not a product that the compiler contracts with the sum that it stands in: at scores of 60 the LSE erred twice as much.)
  auto ref_of = [&](float x) __attribute__((always_inline)) {
    float y = x * a.cl2;
    if constexpr (OWN) asm("" : "+v"(y));
    return y;
  };

  f32x16 o[2 * AH][QB];
  float m[QB], mc[QB], l[QB], l_err[OWN ? QB : 1];  // l_err: what the sum over tiles lost to rounding
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m[qb] = -INFINITY; mc[qb] = 0.f; l[qb] = 0.f;
    if (OWN) l_err[OWN ? qb : 0] = 0.f;
#pragma unroll
    for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[db][qb][v] = 0.f;
  }

  // Tiles are taken NK at a time; a stage never straddles runs of consecutive tokens of a chunk (the chunk, or its
  // half under zig-zag ownership) when their tiles divide by NK, otherwise NK falls to 1.
  const int nk = NK == 1 || ((int)(a.map.zigzag ? a.map.h : a.map.c) & (kTileKeys * NK - 1)) == 0 ? NK : 1;
  // With few work-groups the walk's stages are divided over gridDim.y work-groups, each leaving an unnormalised partial
  // result that a second kernel merges.
  KeyWalk<CAUSAL> w, wg_;  // group 0's stage, this group's
  w.begin(a.map, n, a.N, nk == 2 ? 7 : 6, q_last, gridDim.y, blockIdx.y);
  const TileDMAT<RW> dma(wave, lane, (int)kv_ld);
  auto load_stage = [&](int64_t k0, auto &Kn, auto &Vn) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NK; ++u) {
      if (u < nk) {
#pragma unroll
        for (int ah = 0; ah < AH; ++ah) {
          dma.load(Kh + (k0 + u * kTileKeys) * kv_ld + ah * 64, Kn[u][ah]);
          dma.load(Vh + (k0 + u * kTileKeys) * kv_ld + ah * 64, Vn[u][ah]);
        }
      }
    }
  };

  if (KS > 1) { wg_ = w; wg_.skip(grp); }
  KeyWalk<CAUSAL> &g = KS == 1 ? w : wg_;
  if (g.have) load_stage(g.key(), Ks0[grp], Vs0[grp]);
  wait_vmem();
  __syncthreads();
  bool first = true;
  // one stage: start the loads of the next stage into (Kn, Vn), compute on (Kc, Vc)
  auto stage = [&](auto &Kc, auto &Vc, auto &Kn, auto &Vn) __attribute__((always_inline)) {
    const int ks0 = g.key();
    const bool mine = KS == 1 || g.have;
    w.skip(KS);
    if (KS > 1) wg_.skip(KS);
    if (g.have) load_stage(g.key(), Kn, Vn);

#pragma unroll
    for (int u = 0; u < NK; ++u) {
    const int k0 = ks0 + u * kTileKeys;
    const bool work = mine && u < nk && (!CAUSAL || k0 <= wq_last);
    f32x16 s[2][QB];
    float tm[QB];
    auto scores = [&]() __attribute__((always_inline)) {
      // ---- S^T = K Q^T
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        bf16x8 ka[4 * AH];
#pragma unroll
        for (int dk = 0; dk < 4 * AH; ++dk) ka[dk] = tl.read_rows(Kc[u][dk >> 2], kb * 32, dk & 3);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
          for (int v = 0; v < 16; ++v) s[kb][qb][v] = 0.f;
#pragma unroll
          for (int dk = 0; dk < 4 * AH; ++dk) s[kb][qb] = mfma_32x32x16(ka[dk], qreg[qb][dk], s[kb][qb]);
        }
      }
      if (CAUSAL && k0 + kTileKeys - 1 > wq_first) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          // keys of the tile that the lane's row sees: the first n, less the lane half's offset
          const int n = qtok[qb] + 1 - k0 - half * 4;
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            const uint32_t seen = low_bits(n - kb * 32);
#pragma unroll
            for (int v = 0; v < 16; ++v) s[kb][qb][v] = keep_bit(s[kb][qb][v], seen, (v >> 2) * 8 + (v & 3));
          }
        }
      }
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        float x = s[0][qb][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) x = fmaxf(x, s[0][qb][v]);
#pragma unroll
        for (int v = 0; v < 16; ++v) x = fmaxf(x, s[1][qb][v]);
        tm[qb] = xhalf_max(x);
      }
    };
    auto accumulate = [&]() __attribute__((always_inline)) {
      // ---- running max; the accumulators are rescaled only when some row's max
      // grew by more than 2^8 in the exp2 domain (exact: l and O share the stale max)
      bool need = false;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) need |= (tm[qb] - m[qb]) * a.cl2 > 8.0f;
      if (__builtin_amdgcn_ballot_w64(need) != 0) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          // a row that has seen no key yet (a split walk can start right of it) keeps mc = 0
          const float mn = fmaxf(m[qb], tm[qb]);
          const bool seen = mn > -INFINITY;
          const float alpha = seen ? __builtin_amdgcn_exp2f(OWN ? ref_of(m[qb]) - ref_of(mn) : (m[qb] - mn) * a.cl2) : 1.0f;
          m[qb] = mn;
          mc[qb] = seen ? ref_of(mn) : 0.f;
          l[qb] *= alpha;
          if (OWN) l_err[OWN ? qb : 0] *= alpha;
#pragma unroll
          for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][qb][v] *= alpha;
        }
      }
      // ---- P^T = exp2(S^T cl2 - m cl2), packed to bf16 as the B operand
      bf16x8 pf[QB][4];
      float wt[QB];  // OWN: the tile's weight
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        float l4[OWN ? 4 : 1] = {};
        const float own = ref_of(tm[qb]), mt = !OWN ? mc[qb] : own > -INFINITY ? own : 0.f;
        wt[qb] = OWN ? __builtin_amdgcn_exp2f(own - mc[qb]) : 1.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          float p[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            p[v] = __builtin_amdgcn_exp2f(fmaf(s[kb][qb][v], a.cl2, -mt));
            l4[OWN ? v & 3 : 0] += p[v];
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            u32x4 w = {pack_bf16(p[u * 8 + 0], p[u * 8 + 1]), pack_bf16(p[u * 8 + 2], p[u * 8 + 3]),
                       pack_bf16(p[u * 8 + 4], p[u * 8 + 5]), pack_bf16(p[u * 8 + 6], p[u * 8 + 7])};
            pf[qb][kb * 2 + u] = __builtin_bit_cast(bf16x8, w);
          }
        }
        if constexpr (OWN) {
          const float x = fmaf(wt[qb], (l4[0] + l4[1]) + (l4[2] + l4[3]), -l_err[qb]), sum = l[qb] + x;
          l_err[qb] = (sum - l[qb]) - x;
          l[qb] = sum;
        } else {
          l[qb] += l4[0];
        }
      }
      // ---- O^T += V^T P^T
#pragma unroll
      for (int db = 0; db < 2 * AH; ++db) {
        f32x16 c[OWN ? QB : 1];
        if constexpr (OWN) {
#pragma unroll
          for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) c[qb][v] = 0.f;
        }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const bf16x8 va = tl.read_cols(Vc[u][db >> 1], kk * 16, db & 1);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            f32x16 &acc = OWN ? c[OWN ? qb : 0] : o[db][qb];
            acc = mfma_32x32x16(va, pf[qb][kk], acc);
          }
        }
        if constexpr (OWN) {
#pragma unroll
          for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][qb][v] = fmaf(wt[qb], c[qb][v], o[db][qb][v]);
        }
      }
    };
    if constexpr (KS == 1) {
      if (work) { scores(); accumulate(); }
    } else {
      if (work) scores();
      // all groups start from the maximum of the walk's first tile, as one group walking alone would
      if (first) {
        if (grp == 0) ref[wave][lane] = work ? tm[0] : -INFINITY;
        __syncthreads();
        m[0] = ref[wave][lane];
        mc[0] = m[0] > -INFINITY ? ref_of(m[0]) : 0.f;
        first = false;
      }
      if (work) accumulate();
    }
    }

    wait_vmem();
    __syncthreads();
  };
  while (w.have) {
    stage(Ks0[grp], Vs0[grp], Ks1[grp], Vs1[grp]);
    if (!w.have) break;
    stage(Ks1[grp], Vs1[grp], Ks0[grp], Vs0[grp]);
  }

  if constexpr (OWN) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l[qb] -= l_err[qb];
  }
  if constexpr (KS > 1) {
    // Groups 1 .. KS - 1 leave their sums in LDS (the stage buffers are free: group g takes one of the four
    // objects per 64 columns), group 0 brings them to a common maximum and adds them.
    static_assert(QB == 1, "32 rows per wave");
    constexpr int PARTS = 2 * AH;  // of 32 columns: 4 KiB per wave
    auto slot = [&](int g, int part) -> f32x4 * {
      // PARTS * (KS - 1) slots of RW waves x 4 KiB, dealt to the four objects
      const int i = (g - 1) * PARTS + part;
      unsigned char *o = (i & 3) == 0 ? &Ks0[0][0][0][0] : (i & 3) == 1 ? &Ks1[0][0][0][0]
                         : (i & 3) == 2 ? &Vs0[0][0][0][0] : &Vs1[0][0][0][0];
      return reinterpret_cast<f32x4 *>(o + ((i >> 2) * RW + wave) * 4096);
    };
    static_assert((PARTS * (KS - 1) + 3) / 4 * RW * 4096 <= KS * NK * AH * kTileBytes, "room for a group's sums");
    if (grp > 0) {
#pragma unroll
      for (int db = 0; db < PARTS; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          slot(grp, db)[g * 64 + lane] =
              f32x4{o[db][0][g * 4 + 0], o[db][0][g * 4 + 1], o[db][0][g * 4 + 2], o[db][0][g * 4 + 3]};
    }
    mls[grp][wave][0][lane] = m[0];
    mls[grp][wave][1][lane] = l[0];
    __syncthreads();
    if (grp == 0) {
      float M = m[0];
#pragma unroll
      for (int g = 1; g < KS; ++g) M = fmaxf(M, mls[g][wave][0][lane]);
      const bool seen = M > -INFINITY;
      auto weight = [&](float x) { return __builtin_amdgcn_exp2f(OWN ? ref_of(x) - ref_of(M) : (x - M) * a.cl2); };
      const float w0 = seen ? weight(m[0]) : 0.f;
      m[0] = M; mc[0] = seen ? ref_of(M) : 0.f; l[0] *= w0;
#pragma unroll
      for (int db = 0; db < PARTS; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][0][v] *= w0;
#pragma unroll
      for (int g = 1; g < KS; ++g) {
        const float w = seen ? weight(mls[g][wave][0][lane]) : 0.f;
        l[0] = fmaf(mls[g][wave][1][lane], w, l[0]);
#pragma unroll
        for (int db = 0; db < PARTS; ++db)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 x = slot(g, db)[q * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[db][0][q * 4 + e] = fmaf(x[e], w, o[db][0][q * 4 + e]);
          }
      }
    }
    __syncthreads();  // the epilogue writes to the buffers that the other waves just read
    if (grp > 0) return;
  }

  if (gridDim.y > 1) {  // partial result of this split
    const int64_t heads = a.by_heads.d;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float lt = xhalf_sum(l[qb]);
      if (here[qb]) {
        const int64_t pr = ((int64_t)blockIdx.y * heads + head) * a.Lq + qrow[qb];
        float *po = a.part_o + pr * A + half * 4;
#pragma unroll
        for (int db = 0; db < 2 * AH; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 w = {o[db][qb][g * 4 + 0], o[db][qb][g * 4 + 1], o[db][qb][g * 4 + 2], o[db][qb][g * 4 + 3]};
            *reinterpret_cast<f32x4 *>(po + db * 32 + g * 8) = w;
          }
        if (half == 0) {
          a.part_ml[pr * 2] = lt > 0.f ? mc[qb] : -INFINITY;
          a.part_ml[pr * 2 + 1] = lt;
        }
      }
    }
    return;
  }

  // ---- epilogue: O = O^T / l, LSE = s m + ln l.  The wave's R x 64 block of O goes through its
  // own LDS tile (every wave is past the loop's last barrier and no load is in flight, so the
  // stage buffers are free) and leaves as whole 128-byte rows.
  unsigned char *ot = wave == 0 ? Ks0[0][0][0] : (wave == 1 ? Ks1[0][0][0] : (wave == 2 ? Vs0[0][0][0] : Vs1[0][0][0]));
  float inv[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float lt = xhalf_sum(l[qb]);
    inv[qb] = 1.0f / lt;
    if (here[qb] && half == 0) {
      a.LSE[head * a.Lq + qrow[qb]] = OWN ? (float)(mc[qb] * 0.6931471805599453 + log((double)lt)) : (mc[qb] + __builtin_amdgcn_logf(lt)) * kLn2;
    }
  }
  const int64_t rows_here = a.Lq - (row0 + wave * R);
#pragma unroll
  for (int ah = 0; ah < AH; ++ah) {  // one half of the head at a time through the wave's tile
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) stage_block_T(ot, qb * 32, o[2 * ah][qb], o[2 * ah + 1][qb], inv[qb], lane);
    flush_rows<R>(ot, 0, a.O + head_offset((uint32_t)head, a.by_Z, a.os) + wrow * o_ld + ah * 64, rows_here, lane, (int)o_ld);
  }
}

// Merge of the split walks' partial results: with M the largest stale max of a row,
// O = sum_s 2^(mc_s - M) o_s / sum_s 2^(mc_s - M) l_s and LSE = (M + log2 of that denominator) ln 2.
// A split that saw no key of the row has mc = -inf and is left out.  A/4 lanes x 4 columns per row.
__global__ void __launch_bounds__(256) fwd_combine_kernel(const float *part_o, const float *part_ml,
                                                          uint16_t *O, float *LSE, int64_t rows, int splits,
                                                          int A, OutLayout lay) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lg = A == 64 ? 4 : 5;  // A / 4 lanes per row
  const int64_t row = gid >> lg;
  const int sub = (int)gid & ((1 << lg) - 1);
  if (row >= rows) return;
  float M = -INFINITY;
  for (int s = 0; s < splits; ++s) M = fmaxf(M, part_ml[((int64_t)s * rows + row) * 2]);
  float lsum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < splits; ++s) {
    const int64_t pr = (int64_t)s * rows + row;
    const float mc = part_ml[pr * 2];
    if (mc > -INFINITY) {
      const float w = __builtin_amdgcn_exp2f(mc - M);
      lsum = fmaf(w, part_ml[pr * 2 + 1], lsum);
      acc += *reinterpret_cast<const f32x4 *>(part_o + pr * A + sub * 4) * w;
    }
  }
  const float inv = 1.0f / lsum;
  const u32x2 w = {pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)};
  *reinterpret_cast<u32x2 *>(O + lay.row_off(row) + sub * 4) = w;
  if (sub == 0) LSE[row] = (M + __builtin_amdgcn_logf(lsum)) * kLn2;
}

template <bool OWN, int R, int AH, int NK, int RW, int KS, int MASKS = kBothMasks>
static hipError_t launch_fwd(const Dims &d, FwdArgs a, int64_t heads, int splits, hipStream_t st) {
  a.by_tiles = make_fast_div((d.Lq + RW * R - 1) / (RW * R));
  a.by_length = order_by_length(d, splits, (int64_t)400 << 20);
  dim3 grid((unsigned)(heads * a.by_tiles.d), (unsigned)splits);
  if (!(MASKS & (d.causal ? kCausal : kNoMask))) return hipErrorInvalidValue;
  if constexpr (MASKS & kCausal)
    if (d.causal) hipLaunchKernelGGL((fused_fwd_kernel<R, true, AH, NK, RW, KS, OWN>), grid, dim3(64 * RW * KS), 0, st, a);
  if constexpr (MASKS & kNoMask)
    if (!d.causal) hipLaunchKernelGGL((fused_fwd_kernel<R, false, AH, NK, RW, KS, OWN>), grid, dim3(64 * RW * KS), 0, st, a);
  return hipGetLastError();
}

// Whether a causal launch hands out its tiles by length (longest_first): when they differ by more than a
// factor of two, the walk is not split (splits turn the ranges over the XCDs instead, see xcd_remap), and what the
// walks of all heads read (K and V, or Q and dO) takes at most `most` bytes: all heads are then under way together, and
// what the caches cannot hold is fetched again and again.  Time in head order over time by length, by MB:
// forward 37 (70 heads): 1.18, 67: 1.37, 75: 1.41, 147: 1.10, 227: 1.00, 254: 1.05, 294: 1.11, 567: 0.92; backward 37:
// 1.15, 67: 1.14, 113: 1.10, 134: 1.04 and 0.98, 147: 1.00, 226: 0.97, 294: 0.94, 567: 0.89.
bool order_by_length(const Dims &d, int splits, int64_t most) {
  return d.causal && splits == 1 && (d.zigzag || 2 * d.rank_begin < d.rank_end) &&
         (int64_t)d.B * d.Z * d.L * d.A * 4 <= most;
}

// Splits of the key walk for a kernel whose work-groups own `rows_per_wg` query rows (two
// work-groups per CU make 512 slots): 1 when the rows alone fill the chip.  Otherwise the smallest count whose work-groups fill whole rounds of the 512 slots
// to 95 % -- a round that is half empty costs as much as a full one -- with at least 16 stages
// of 128 keys left per split (shorter walks lose more to their prologue and to the merge than
// the better fill gains).  Under the causal mask walks differ in length, so at least three
// rounds are wanted; under zig-zag ownership half of the row tiles see almost no keys and do
// not count.  When no count qualifies, the largest one allowed.
static int key_splits_for(const Dims &d, int rows_per_wg) {
  int64_t wgs = (int64_t)d.B * d.Z * ((d.Lq + rows_per_wg - 1) / rows_per_wg);
  if (wgs >= 1024) return 1;
  int64_t stages = d.L / 128;  // the longest walk of a row tile
  if (d.causal && !d.zigzag && (int64_t)d.rank_end * d.c / 128 < stages) stages = (int64_t)d.rank_end * d.c / 128;
  const int64_t smax = stages / 16 < 32 ? stages / 16 : 32;
  if (smax < 2) return 1;
  // The whole ring: splits in two, and those of walks of very different length, lose to groups of waves on a walk or
  // to plain work-groups (forward, split -> not, us, by 128-row work-groups: 4096 rows 32: 31.3 -> 25.3, 256: 50 -> 46, 768:
  // 124 -> 114; causal 4096 rows 192: 46 -> 28, 896: 118 -> 80, 8192 rows 256: 77 -> 57, 1024: 205 -> 165, 16384 rows 768:
  // 311 -> 254; but 8192 rows 128: 47 -> 50, 16384 rows 512: 188 -> 198).
  const int64_t W = (int64_t)d.B * d.Z * ((d.Lq + 127) / 128);
  if (d.Lq == d.L) {
    const bool wide = d.A == 128;  // (fewer work-groups on a CU: 4096 rows, W = 128: split 52, not 56)
    if (d.causal && ((d.L < 8192 && !(wide && W <= 128)) || W >= 640 || (d.L <= 8192 && W >= (wide ? 400 : 200)))) return 1;
    if (!d.causal && smax == 2 && (wide ? W > 128 : W <= 320 || W >= 400)) return 1;
  }
  if (d.causal && d.zigzag) wgs = (wgs + 1) / 2;
  const int64_t min_rounds = d.causal ? 3 : 1;
  for (int64_t s = 1; s <= smax; ++s) {
    const int64_t n = s * wgs, rounds = (n + 511) / 512;
    if (rounds >= min_rounds && n * 20 >= rounds * 512 * 19) return (int)s;
  }
  return (int)smax;
}

// the dQ kernel: 128 rows per work-group
int fused_key_splits(const Dims &d) { return key_splits_for(d, 128); }

// The forward: 64 rows per wave (256 per work-group) halve the LDS traffic per flop and are
// taken when their work-groups, times their splits, fill the 512 slots at least once; else 32
// rows per wave, which give twice the work-groups.  (A head of 128 elements takes 32 rows per
// wave and one key tile per stage: registers and LDS.)  Unsplit, a CU's two places for large work-groups, filled in turn, are
// compared with its four for small ones, which cost 5 % more per row where walks are longer than 512 keys (W, work-groups of
// 128 rows, small -> large, us: 1024 rows, 896: 41.2 -> 39.2, 1536: 61.9 -> 59.5, but 1200: 51 -> 57; 2048 rows, 1536: 117 ->
// 112) and less where they are shorter (512 rows, 1024: 25.6 -> 26.7, 256 rows: 17.3 -> 20.5).  Causal walks end one by one
// and fill places left over: large ones only for long walks on a full chip (8192 rows, 2048: 306 -> 299, 4096 rows: 160 -> 156;
// but 1888: 156 -> 166, 2048 rows, 3072: 129 -> 140, 1024 rows, 2048: 50.6 -> 53.6).
// Rows that are no multiple of 256 leave part of a head's last work-group idle: the rounds count that (whole ring: 4160
// rows, W = 1815: 290 -> 276, 3366: 510 -> 483; 2496 rows, 1820: 178 -> 169).  One rank's share and projected keys take large ones
// then only where 128 would leave as much (1472 rows of 2944, 2424: 265 -> 250; 960 rows, 1024 projected keys, 1536: 59.4 -> 58.2, but
// 1096: 48.5 -> 55.7; 832 of 6656, 1484: 372 -> 439), and not under the causal mask (last 1984 of 3968, 1392: 178 -> 193, 6000:
// 662 -> 675, first 448 of 1344, 1040: 20 -> 26; from 2040 on, of 4416 rows, 3 % either way).  One full round of either kind is shorter
// with the small ones (W = 512: 256 heads of 192 of 1536 rows 32.6 -> 34.3, 128 of 448 rows, 1024 projected keys, 23.7 -> 24.8, 64 whole
// rings of 960 21.9 -> 22.9, 32 of 1984 41.0 -> 42.0).
// A walk that would be split but has no room for partial results (the two-pass layout, projected keys) goes by the rounds as
// well, one rank's causal share by 512 large work-groups of its own: such as were to fill the chip times their splits left it half
// empty (two-pass, us, shape of the split -> this: 1 head of 16384 rows 337 -> 103, causal 341 -> 100; 4 of 8192 171 -> 98; 16 heads of
// 1024 of 16384 335 -> 104, 130 of 512 of 4096 139 -> 115; 160 heads of 512 rows, 4096 projected keys 123 -> 108; large ones as
// before: last 512 of 4096 causal, 256 heads, 166, not 173; 64 of 1024 of 8192 175, not 180).
void fused_fwd_plan(const Dims &d, bool may_split, bool *big, int *splits) {
  if (d.A == 64) {
    const int s = key_splits_for(d, 256);
    const int64_t heads = (int64_t)d.B * d.Z, wgs = heads * ((d.Lq + 255) / 256), W = heads * ((d.Lq + 127) / 128);
    const bool whole = d.Lq == d.L, even = d.Lq % 256 == 0;
    bool large = even && wgs * s >= 512;
    if (s == 1 ? whole || !even : !may_split) {
      if (d.causal) large = whole ? W >= 2000 && d.L >= 4096 : even && wgs >= 512;
      else large = (even ? W >= 512 : W > 512) && d.L > 512 && (whole || 2 * wgs == W) && (double)((wgs + 255) / 256) * 2 < (double)((W + 255) / 256) * 1.055;
    }
    if (large) {
      *big = true; *splits = may_split ? s : 1;
      return;
    }
  }
  *big = false; *splits = may_split ? key_splits_for(d, 128) : 1;
}

template <bool OWN>
static hipError_t forward_as(const Dims &d, const void *Q, const void *K, const void *V, void *O,
                         float *LSE, hipStream_t st, bool may_split, float *part, int64_t usual) {
  FwdArgs a;
  a.Q = (const uint16_t *)Q; a.K = (const uint16_t *)K; a.V = (const uint16_t *)V;
  a.O = (uint16_t *)O; a.LSE = LSE;
  a.L = d.L; a.c = d.c; a.Lq = d.Lq; a.map = make_row_map(d);
  a.N = d.N; a.by_Z = make_fast_div(d.Z); a.by_heads = make_fast_div((int64_t)d.B * d.Z);
  for (int k = 0; k < 3; ++k) { a.qs[k] = d.qs[k]; a.ks[k] = d.ks[k]; a.os[k] = d.os[k]; }
  a.cl2 = d.scale * kLog2e;
  const int64_t heads = (int64_t)d.B * d.Z;
  bool big;
  int splits;
  Dims call = d;  // what the shapes are chosen by
  if (usual) { call.B = 1; call.Z = (int)usual; }
  fused_fwd_plan(call, may_split, &big, &splits);
  const int64_t rows = heads * d.Lq;
  a.part_o = part;
  a.part_ml = part ? part + (int64_t)splits * rows * d.A : nullptr;
  // Few work-groups of four waves (W: their number): the chip is not full, and a work-group's walk is a serial chain.
  // Then fewer rows per work-group and several groups of waves on its keys (RW, KS in the kernel): the chain
  // shortens, at more tile loads per flop.  The lines are those of sweeps over 1 .. 2000 heads of 192 .. 32768 rows (us,
  // four waves -> chosen): W = 64: 9.4 -> 7.5; 128 (4096 rows): 49 -> 27; 256 (4096): 49 -> 46; causal 192 (4096): 59 -> 28;
  // 384 (4096): 61 -> 46; 512 (2048): 33 -> 30; 640 (8192): 133 -> 116; heads of 128, W = 256 (4096): 83 -> 72, causal
  // 512 (8192): 180 -> 149, but 400 (512): 18 -> 25.
  // The two-pass layout, whose strip went by what the rows see, takes one rank's causal rows by that where it is short (300 heads,
  // us: the first 64 of 1024 rows 10.7 -> 6.3, strip 9.0, heads of 128 13.2 -> 7.7, strip 10.4; 128 rows 15.9 -> 7.8, strip 12.6;
  // from 1000 keys on it would be slower: 38 heads, first 1024 of 4096, 16 -> 18.5).  Rows whose walks are about as long go by
  // the lines of walks without a mask (heads of 128, last 64 of 1024, 264 heads: 50 -> 37, strip 40; 64 of 1024 behind the first
  // 512, 420: 36 -> 25, strip 36; third 512 of 2048, 66: 62 -> 50, strip 58).
  const bool c = d.causal;
  const int64_t W = (usual ? usual : heads) * ((d.Lq + 127) / 128), walk = d.L / 64;
  const int64_t seen = c && !d.zigzag ? (int64_t)d.rank_end * d.c : d.L, L = OWN && seen <= 512 ? seen : d.L;
  const bool uneven = c && !(OWN && 2 * d.rank_begin >= d.rank_end);
  hipError_t e;
  if (big) e = launch_fwd<OWN, 64, 1, 2, 4, 1>(d, a, heads, splits, st);
  else if (d.A == 128) {
    if (splits > 1 || W > (uneven && L > 512 ? 512 : 256)) e = launch_fwd<OWN, 32, 2, 1, 4, 1>(d, a, heads, splits, st);
    else if (W > 128) e = launch_fwd<OWN, 32, 2, 1, 4, 2>(d, a, heads, 1, st);
    else e = launch_fwd<OWN, 32, 2, 1, 2, 2>(d, a, heads, 1, st);
  } else if (splits > 1) e = launch_fwd<OWN, 32, 1, 1, 4, 1>(d, a, heads, splits, st);
  else if (!OWN && W <= 64) e = launch_fwd<OWN, 32, 1, 1, 1, 4>(d, a, heads, 1, st);
  else if (W <= 128 || (c && W <= 300 && L >= 1536)) e = launch_fwd<OWN, 32, 1, 1, 2, 4>(d, a, heads, 1, st);
  else if (c && W <= (L >= 4096 ? 430 : 256)) e = launch_fwd<OWN, 32, 1, 1, 2, 2, kCausal>(d, a, heads, 1, st);
  else if (c ? (W <= 576 && L >= 1024) || (W <= 800 && L >= 4096) : W <= 256 && walk >= 16)
    e = launch_fwd<OWN, 32, 1, 1, 4, 2>(d, a, heads, 1, st);
  else e = launch_fwd<OWN, 32, 1, 1, 4, 1>(d, a, heads, 1, st);
  if (e != hipSuccess || splits == 1) return e;
  const OutLayout lay = make_out_layout(d.os, d.Lq, d.Z);
  hipLaunchKernelGGL(fwd_combine_kernel, dim3((unsigned)((rows * (d.A / 4) + 255) / 256)), dim3(256), 0, st,
                     a.part_o, a.part_ml, (uint16_t *)O, LSE, rows, splits, d.A, lay);
  return hipGetLastError();
}

hipError_t fused_forward(const Dims &d, const void *Q, const void *K, const void *V, void *O, float *LSE, hipStream_t st,
                         bool may_split, float *part) {
  return forward_as<false>(d, Q, K, V, O, LSE, st, may_split, part, 0);
}
hipError_t two_pass_forward(const Dims &d, const void *Q, const void *K, const void *V, void *O, float *LSE, int64_t usual,
                            hipStream_t st) {
  return forward_as<true>(d, Q, K, V, O, LSE, st, false, nullptr, usual);
}

}  // namespace rsa
