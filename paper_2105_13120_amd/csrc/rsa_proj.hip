// The two linear maps around Ring Self-Attention on a rank's rows (paper Table 2, sequence
// parallelism rows "Q/K/V" and "Linear") and their derivatives, bf16 with fp32 accumulation:
//   Q/K/V:  (B, rows, H) x (H, AZ) -> (B, Z, rows, A), written head-split as RSA reads it
//   Linear: (B, Z, rows, A) x (AZ, H) -> (B, rows, H), read head-split as RSA writes it
// One MFMA GEMM kernel serves all six products.  An operand is a "view": a matrix cut into
// 64 x 64 tiles that are either blocks of a plain row-major matrix or the (64 rows, 64 elements of
// one head) blocks of up to three (B, Z, rows, A) tensors, A = 64 or 128, so no tensor is ever
// re-laid out in memory.
//
// Work-group: 64 T x 64 T outputs, T = 4, 2 or 1 by the size of the product (plan_gemm), 2 T waves of 32 T x 64, k in
// slabs of 32 through a ring of four LDS buffers, one barrier per slab.  The product is formed transposed
// (accumulator rows = n, columns = m): a lane then owns one output row m and four consecutive n per register group;
// blocks leave through LDS as whole row segments of 128 (bf16) or 256 bytes.
#include "rsa_fused_tile.h"
#include "rsa_kernels.h"

#include <math.h>

namespace rsa {

// A bf16 matrix [R][C] served as 64 x 64 tiles.
struct MatView {
  const uint16_t *p[3];  // plain: p[0]; head-split: tensor cb / (Z * AH) holds column tile cb
  int64_t ld;            // row stride in elements (head-split: the head size A)
  int64_t rows;          // head-split: rows per (b, z) block (a multiple of 64)
  int Z;                 // head-split: heads per tensor
  int AH;                // head-split: column tiles per head (A / 64: 1 or 2), head-major order
  int split;             // 0: plain row-major; 1: (B, Z, rows, A) tensors, row index = b * rows + r
  FastDiv by_rows, by_tensor;  // rows; Z * AH
};

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// How the tiles of one operand move along k, slab by slab, with additions only (the divisions
// that place a head-split tile are done once, in TileCursor's constructor): `step` per slab, and
// after `period` steps an extra jump to the next batch element (mode 1) or to the next tensor of
// the view (mode 2: jump1 into tensor 1, jump2 into tensor 2).  With two column tiles per head
// (mode 3) a step is the 64 elements to the head's second half, every second step also jumps
// (jumpA) to the next head, and after Z heads comes the jump to the next tensor.
struct ViewWalk {
  int64_t ld, step, jump1, jump2, jumpA;
  int period, mode, Z;
  // krows: k runs over the row tiles of the view; else over its column tiles
  __device__ __forceinline__ ViewWalk(const MatView &v, bool krows) {
    jump1 = 0; jump2 = 0; jumpA = 0; period = 0x7fffffff; mode = 0; Z = v.Z;
    if (!v.split) {
      ld = v.ld;
      step = krows ? 64 * v.ld : 64;
    } else if (!krows) {  // k runs over heads, then over the tensors of the view
      ld = v.ld;
      const int64_t head = v.rows * v.ld;  // elements from one head to the next
      // after the last head of a tensor the pointer has moved Z heads; the next tensor starts over
      jump1 = (v.p[1] - v.p[0]) - (int64_t)v.Z * head;
      jump2 = (v.p[2] - v.p[1]) - (int64_t)v.Z * head;
      if (v.AH == 1) {
        step = head; period = v.Z; mode = 2;
      } else {
        step = 64; jumpA = head - 128; period = 2; mode = 3;
      }
    } else {  // k runs over the rows of a batch element, then over batch elements
      ld = v.ld;
      step = 64 * v.ld;
      jump1 = (int64_t)(v.Z - 1) * v.rows * v.ld;
      period = (int)(v.rows / 64); mode = 1;
    }
  }
};

struct TileCursor {
  const uint16_t *ptr;
  int cnt, which;  // which: tensor of the view; in mode 3 also the head inside it, times 4
  // krows: the tile index `fixed` selects columns and k (slab ks) selects rows; else the reverse
  __device__ __forceinline__ TileCursor(const MatView &v, bool krows, int64_t fixed, int64_t ks) {
    cnt = 0; which = 0;
    if (!v.split) {
      ptr = krows ? v.p[0] + ks * 64 * v.ld + fixed * 64 : v.p[0] + fixed * 64 * v.ld + ks * 64;
    } else {
      const uint32_t ct = (uint32_t)(krows ? fixed : ks), rt = (uint32_t)(krows ? ks : fixed);
      which = (int)v.by_tensor(ct);
      const uint32_t rem = ct - (uint32_t)which * v.by_tensor.d;
      const int64_t z = v.AH == 2 ? rem >> 1 : rem;
      const int ah = v.AH == 2 ? (int)(rem & 1) : 0;
      const uint32_t m0 = rt * 64u, b = v.by_rows(m0), r0 = m0 - b * v.by_rows.d;
      const uint16_t *t = which == 0 ? v.p[0] : (which == 1 ? v.p[1] : v.p[2]);
      ptr = t + (((int64_t)b * v.Z + z) * v.rows + r0) * v.ld + ah * 64;
      cnt = krows ? (int)(r0 / 64) : (v.AH == 1 ? (int)z : ah);
      if (!krows && v.AH == 2) which |= (int)z << 2;
    }
    ptr = reinterpret_cast<const uint16_t *>(uniform64(reinterpret_cast<int64_t>(ptr)));
    cnt = __builtin_amdgcn_readfirstlane(cnt);
    which = __builtin_amdgcn_readfirstlane(which);
  }
  template <bool WIDE>  // WIDE: some view of the product has two column tiles per head (mode 3)
  __device__ __forceinline__ void advance(const ViewWalk &w) {
    ptr += w.step;
    if (++cnt == w.period) {
      asm volatile("" ::: "memory");  // a real (rarely taken, uniform) branch instead of a chain of selects per slab
      cnt = 0;
      if (w.mode == 1) ptr += w.jump1;
      if (w.mode == 2) { ptr += which == 0 ? w.jump1 : w.jump2; ++which; }
      if (WIDE && w.mode == 3) {
        ptr += w.jumpA;
        which += 4;
        if ((which >> 2) == w.Z) { ptr += (which & 3) == 0 ? w.jump1 : w.jump2; which = (which & 3) + 1; }
      }
    }
  }
};

struct GemmArgs {
  MatView A, B;       // m-side and n-side operands
  int64_t M, N, K;    // multiples of 64
  int64_t kslabs;     // slabs of 64 k per split (split s takes slabs [s * kslabs, ...))
  int64_t chain;      // fp32 results: slabs of 64 k that one chain of additions may take (see plan_gemm)
  void *out[3];       // plain: out[0] (+ split * M * out_ld elements for a k split); head-split: 3 tensors
  int64_t out_ld, out_rows;
  int out_Z, out_AH, out_split;  // head-split output: (B, out_Z, out_rows, 64 * out_AH) tensors
  FastDiv by_out_rows, by_out_tensor;  // out_rows; out_Z * out_AH
  FastDiv by_ntiles;  // column tiles
  int part_heads;     // > 0: the partial sums of a k split lie in the rows of a (Zt, out_rows, A) bf16 tensor: A / 2
                      // columns per head, part_heads heads per split, and out_ld = A / 2
};

// Divisions by run-time sizes are multiplications by numbers that the host prepares, and a head-split result's are done once
// per 64 rows: as chains of vector instructions they stood in front of a work-group's first loads (five) and among its
// stores (sixteen a lane), 2 to 6 % of the Q/K/V map (52224 rows, 1536 -> 3072: 468 -> 459 us; 178112 rows of 448: 314 -> 294;
// 4096 rows of 768: 22.9 -> 22.1).

// A_KROWS / B_KROWS: the operand's tiles hold k along their rows (the view is [K][M] or [K][N])
// instead of along their columns ([M][K], [N][K]).
// Work-group: 2 T waves, 64 T (m) x 64 T (n) outputs; wave (wm, wn) of a 2 x T grid owns 32 T x 64 (T x 2 MFMA
// blocks).  Large products take T = 4, since a CU takes at most about 40 bytes per clock from global memory (measured,
// L2-resident data): 128 x 128 outputs need 32 KiB per 512 matrix-pipe cycles, 256 x 256 need 32 KiB per 1024.
// Products with few outputs take the smaller ones, which give more work-groups and a shorter chain per slab
// (a lone work-group's slab takes 0.61, 0.29, 0.20 us for T = 4, 2, 1).
// k goes in slabs of 32: 2 T half tiles, one half tile per wave, by direct global->LDS loads into a ring of
// four buffers, three slabs ahead of their use (T = 4: a slab takes 1600 cycles to arrive and 1024 to use).
// KG groups of such waves share the k of a work-group and are added in LDS at the end: where there are fewer
// work-groups than CUs, two slabs proceed side by side (T = 1: 0.155 us per slab).
constexpr int kHalfBytes = kTileBytes / 2;

// A half tile in LDS.  k along rows: 32 rows of 128 bytes, as the upper half of a tile.  k along columns: 64 rows
// (m or n) of 32 k = 64 bytes, the row's four 16-byte chunks permuted by c ^ ((row >> 2) & 3), so that the 16 rows
// of a phase of an operand read (four rows make 256 bytes) touch all banks once.
struct HalfLanes {
  int rows_off[2];     // [kk]: operand of rows 0 .. 31, slice kk
  int cols_off[2][2];  // [db][e]: operand of columns 32 db .. 32 db + 31
  __device__ __forceinline__ explicit HalfLanes(int lane) {
    const int col = lane & 31, half = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) rows_off[kk] = col * 64 + (((kk * 2 + half) ^ ((col >> 2) & 3)) << 4);
    const int g = lane >> 4, j = lane & 15;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int e = 0; e < 2; ++e)
        cols_off[db][e] = tile_off(half * 8 + e * 4 + (j >> 2), db * 4 + (g & 1) * 2 + ((j >> 1) & 1)) + (j & 1) * 8;
  }
  __device__ __forceinline__ bf16x8 read_rows(const unsigned char *t, int row_base, int kk) const {
    return *reinterpret_cast<const bf16x8 *>(t + row_base * 64 + rows_off[kk]);
  }
  // By transpose reads, k of slice kk in the order of read_rows: 16 kk + 8 half + e in element e.  (Unlike
  // TileLanes::read_cols, which takes k in the order of an accumulator's rows.)
  __device__ __forceinline__ bf16x8 read_cols(const unsigned char *t, int kk, int db) const {
    return read_cols_at(t, kk, cols_off[db]);
  }
  static __device__ __forceinline__ bf16x8 read_cols_at(const unsigned char *t, int kk, const int *off) {
    const u32x2 lo = lds_read_tr16(t + kk * 2048 + off[0]);
    const u32x2 hi = lds_read_tr16(t + kk * 2048 + off[1]);
    const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(bf16x8, w);
  }
};

// Longest row (elements) whose place in a tile of 64 fits the loads' unsigned 32-bit byte offset.
constexpr int64_t kMaxLd = (int64_t)1 << 25;

// The LDS of a work-group of KG groups, one object for every product that the kernel's branches form.
template <int N> struct GemmLds {
  unsigned char bytes[N * 8 * kHalfBytes];
  template <int KG, int T> __device__ __forceinline__ auto &as() {
    return *reinterpret_cast<unsigned char(*)[KG][4][2 * T][kHalfBytes]>(bytes);
  }
};
template <int N> __device__ __forceinline__ GemmLds<N> &gemm_lds() {
  __shared__ __attribute__((aligned(16))) GemmLds<N> lds;
  return lds;
}

// Work-group (bx, by) of (nx, splits).
// WIDE: heads of 128 elements somewhere in the product (an operand view or the output).
// LONG: an operand with rows of more than kMaxLd elements; its loads take 64-bit addresses per lane.
template <bool A_KROWS, bool B_KROWS, bool OUT_F32, bool WIDE, int T, int KG, bool LONG>
__device__ __forceinline__ void gemm_body(const GemmArgs g, uint32_t bx, uint32_t nx, uint32_t by) {
  constexpr int HT = 2 * T;         // half tiles per slab, and waves per group
  constexpr int BM = 64 * T, BN = 64 * T;
  // (The last word of A's divisors, asked for with the rest of the view: by a scalar load of its own, in front of a small map's
  // first tile, it cost 0.15 us.  Y of 384 rows of 4 heads, H = 1792: 4.64 -> 4.45 us, of 192 of 8, 576: 6.09 -> 5.89.  A view of 64
  // bytes, without the fields that plain ones do not need, did as much for these and made maps of 256 x 256 tiles 0.6 % slower.)
  if constexpr (!A_KROWS && B_KROWS && T == 1) asm volatile("" : : "s"(g.A.by_tensor.shift));
  auto &lds_ = gemm_lds<KG * T>().template as<KG, T>();  // [group][buffer][A.., B..]

  const int tid = threadIdx.x, lane = tid & 63;
  const int gw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KG == 1 ? 0 : gw / HT, wave = KG == 1 ? gw : gw % HT;
  const int wm = wave / T, wn = wave % T;
  const int col = lane & 31, half = lane >> 5;
  unsigned char(*lds)[HT][kHalfBytes] = lds_[grp];
  const uint32_t wg = xcd_remap(bx, nx);
  const uint32_t mt = g.by_ntiles(wg);
  const int64_t m0 = (int64_t)mt * BM, n0 = (int64_t)(wg - mt * g.by_ntiles.d) * BN;
  // slabs of 32 k of group `gr` of this split
  const int64_t per_grp = KG == 1 ? g.kslabs : (g.kslabs + KG - 1) / KG;
  auto slabs_of = [&](int gr, int64_t &begin) -> int {
    begin = (int64_t)by * g.kslabs + gr * per_grp;
    int64_t end = begin + per_grp;
    const int64_t split_end = (int64_t)(by + 1) * g.kslabs;
    if (KG > 1 && end > split_end) end = split_end;
    if (end > g.K / 64) end = g.K / 64;
    return end > begin ? (int)(end - begin) * 2 : 0;
  };
  int64_t ks_begin;
  const int ns0 = slabs_of(0, ks_begin);  // the first group has the most slabs
  const int ns = KG == 1 ? ns0 : slabs_of(grp, ks_begin);

  // Wave w < T brings A's half tile w of every slab, wave w >= T B's half tile w - T.  (A ragged edge refetches the
  // last tile; its outputs are never stored.)
  const bool is_b = wave >= T;
  const bool krows = is_b ? B_KROWS : A_KROWS;
  const int64_t edge = (is_b ? g.N : g.M) / 64 - 1, want = (is_b ? n0 : m0) / 64 + (is_b ? wave - T : wave);
  const int64_t tile = want > edge ? edge : want;
  ViewWalk walk = is_b ? ViewWalk(g.B, B_KROWS) : ViewWalk(g.A, A_KROWS);
  // (held in scalar registers: reloaded from the kernel arguments inside the loop, they make every wait for an LDS
  // read wait for all of them, since scalar loads share its counter and return out of order)
  asm volatile("" : "+s"(walk.step), "+s"(walk.jump1), "+s"(walk.jump2), "+s"(walk.jumpA), "+s"(walk.period),
                    "+s"(walk.mode), "+s"(walk.Z));
  TileCursor cur = is_b ? TileCursor(g.B, B_KROWS, tile, ks_begin) : TileCursor(g.A, A_KROWS, tile, ks_begin);
  const int64_t sub = krows ? 32 * walk.ld : 32;  // from a tile's first slab to its second
  uint32_t g_off[4];  // bytes; LONG: without the rows, which g_row has
  int64_t g_row[LONG ? 4 : 1];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = j * 64 + lane, r8 = p >> 3, r4 = p >> 2;
    const int row = krows ? r8 : r4, cc = krows ? (p & 7) ^ swz_rot(r8) : (p & 3) ^ ((r4 >> 2) & 3);
    g_off[j] = ((LONG ? 0u : (uint32_t)row * (uint32_t)walk.ld) + cc * 8) * 2;
    if constexpr (LONG) g_row[j] = row * walk.ld;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)&lds_[grp][0][wave][0];
  auto issue = [&](int i) __attribute__((always_inline)) {  // slab i (called for 0, 1, 2, ... in turn)
    const uint16_t *src = cur.ptr + ((i & 1) ? sub : 0);
    const uint32_t dst = lds0 + (uint32_t)(i & 3) * (HT * kHalfBytes);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (LONG) lds_dma16_unseen_far(src + g_row[j] + g_off[j] / 2, dst + j * 1024);
      else lds_dma16_unseen(src, (int)g_off[j], dst + j * 1024);
    }
    if (i & 1) cur.template advance<WIDE>(walk);
  };

  f32x16 acc[2][T];  // [nb][mb]: rows n, columns m
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int mb = 0; mb < T; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nb][mb][v] = 0.f;

  // fp32 results, and sums over rows, of the smaller tiles: longer sums are folded into a second set of accumulators, chain
  // by chain
  constexpr bool FOLD = (OUT_F32 || (A_KROWS && B_KROWS)) && T <= 2;
  f32x16 done[FOLD ? 2 : 1][FOLD ? T : 1];
  int left = FOLD ? (int)g.chain * 2 : 0;  // slabs to the next fold
  if constexpr (FOLD) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < T; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) done[nb][mb][v] = 0.f;
  }
  auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < T; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          done[nb][mb][v] += acc[nb][mb][v];
          acc[nb][mb][v] = 0.f;
        }
  };

  const HalfLanes hl(lane);
  int ca[T][2];  // transpose-read offsets of the wave's blocks of 32 m (which half of a tile: odd or even block)
#pragma unroll
  for (int mb = 0; mb < T; ++mb)
#pragma unroll
    for (int e = 0; e < 2; ++e) ca[mb][e] = (wm * T + mb) & 1 ? hl.cols_off[1][e] : hl.cols_off[0][e];
  bf16x8 af[2][T], bf[2][2];
  auto frags = [&](int i, int kk) __attribute__((always_inline)) {  // operands of slice kk of slab i
    const unsigned char(*sc)[kHalfBytes] = lds[i & 3];
#pragma unroll
    for (int mb = 0; mb < T; ++mb) {
      const int b32 = wm * T + mb;  // block of 32 m
      const unsigned char *ta = sc[b32 >> 1];
      af[kk][mb] = A_KROWS ? HalfLanes::read_cols_at(ta, kk, ca[mb]) : hl.read_rows(ta, (b32 & 1) * 32, kk);
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const unsigned char *tb = sc[T + wn];
      bf[kk][nb] = B_KROWS ? hl.read_cols(tb, kk, nb) : hl.read_rows(tb, nb * 32, kk);
    }
  };
  auto products = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < T; ++mb) acc[nb][mb] = mfma_32x32x16(bf[kk][nb], af[kk][mb], acc[nb][mb]);
  };

  // the next slice's reads beside the first MFMAs of this one, so that the last four cover their latency
  auto interleave = [&]() __attribute__((always_inline)) {
    constexpr int kReads = (A_KROWS ? 2 : 1) * T + (B_KROWS ? 4 : 2), kPer = (kReads + T - 1) / T;
#pragma unroll
    for (int k = 0; k < T; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, kPer, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, T, 0);
  };

  if (ns0 > 0) {  // uniform over the work-group; the numbers of slabs are even
    if (KG == 1 || ns > 0) {
      issue(0);
      issue(1);
      if (ns > 2) issue(2);
    }
    if (ns > 2) wait_loads<8>();
    else wait_loads<4>();
    barrier_only();
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): no scalar load is pending in the loop (see above)
    frags(0, 0);
    for (int i = 0; i < ns0; ++i) {
      // slab i + 1 has arrived (slab i + 2 may be in flight), and behind the barrier every wave is done with slab
      // i - 1, whose buffer takes slab i + 3
      if (i + 2 < ns) wait_loads<4>();
      else wait_loads<0>();
      barrier_only();
      if (KG > 1 && i >= ns) continue;  // (uniform over the wave)
      if (i + 3 < ns) issue(i + 3);
      frags(i, 1);
      products(0);
      interleave();
      __builtin_amdgcn_sched_barrier(0);
      frags(i + 1, 0);  // (past the last slab: some buffer's contents, not used)
      products(1);
      interleave();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (FOLD) {
        if (--left == 0) {
          asm volatile("" ::: "memory");  // a real branch
          fold();
          left = (int)g.chain * 2;
        }
      }
    }
  }
  if constexpr (FOLD) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < T; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][mb][v] += done[nb][mb][v];
  }
  __syncthreads();

  if constexpr (KG > 1) {  // groups 1 .. KG - 1 leave their sums in LDS, group 0 adds them in order
    static_assert((KG - 1) * HT * T * 2 * 4096 <= KG * 4 * HT * kHalfBytes, "room for the groups' sums");
    auto slot = [&](int gr, int nb, int mb) {
      return reinterpret_cast<f32x4 *>(&lds_[0][0][0][0] + ((((gr - 1) * HT + wave) * 2 + nb) * T + mb) * 4096);
    };
    if (grp > 0) {
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int mb = 0; mb < T; ++mb)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x16 &c = acc[nb][mb];
            slot(grp, nb, mb)[q * 64 + lane] = f32x4{c[q * 4], c[q * 4 + 1], c[q * 4 + 2], c[q * 4 + 3]};
          }
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int gr = 1; gr < KG; ++gr)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int mb = 0; mb < T; ++mb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x4 x = slot(gr, nb, mb)[q * 64 + lane];
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[nb][mb][q * 4 + e] += x[e];
            }
    }
    __syncthreads();  // the epilogue writes to what was just read
    if (grp > 0) return;
  }

  // lane (col, half) holds, for output row m, the columns n = nb*32 + grp*8 + half*4 .. +4
  if (!OUT_F32) {
    // bf16: the wave's block goes through LDS of its own (every wave is past
    // the loop's last barrier) and leaves as whole 128-byte row segments.
    unsigned char *t0 = &lds_[0][0][0][0] + wave * (T * kHalfBytes);
#pragma unroll
    for (int mb = 0; mb < T; ++mb) stage_block_T(t0, mb * 32, acc[0][mb], acc[1][mb], 1.0f, lane);
    const int64_t nw = n0 + wn * 64;  // the block's 64 columns: (half of) one head of a head-split output
    if (nw < g.N) {
      uint16_t *base = static_cast<uint16_t *>(g.out[0]);
      int64_t ld = g.out_ld, zoff = 0, aoff = nw;
      if (g.out_split) {
        const int out_AH = WIDE ? g.out_AH : 1;
        const uint32_t hb = (uint32_t)nw >> 6, which = g.by_out_tensor(hb), rem = hb - which * g.by_out_tensor.d;
        if (which) base = static_cast<uint16_t *>(which == 1 ? g.out[1] : g.out[2]);
        ld = 64 * out_AH;
        zoff = out_AH == 2 ? rem >> 1 : rem;
        aoff = out_AH == 2 ? (rem & 1) * 64 : 0;
      }
      constexpr int BLOCKS = T == 4 ? 2 : 1;  // of 64 rows (T = 1: half of one), which lie in one batch element
      const int64_t mw = m0 + wm * 32 * T;
#pragma unroll
      for (int blk = 0; blk < BLOCKS; ++blk) {
        int64_t r = mw + blk * 64;
        if (g.out_split) {
          const uint32_t b = g.by_out_rows((uint32_t)r);
          r = ((int64_t)b * g.out_Z + zoff) * g.out_rows + (r - (int64_t)b * g.out_rows);
        }
        uint16_t *const rows = base + r * ld + aoff;
#pragma unroll
        for (int it = 0; it < 4 * T / BLOCKS; ++it) {
          const int row = it * 8 + (lane >> 3), cc = lane & 7;
          if (mw + blk * 64 + row >= g.M) continue;
          const u32x4 w = *reinterpret_cast<const u32x4 *>(t0 + tile_off(blk * 64 + row, cc));
          *reinterpret_cast<u32x4 *>(rows + row * ld + cc * 8) = w;
        }
      }
    }
    return;
  }
  // fp32 (plain matrices): 32 rows of the wave's block at a time, through LDS of its own, as 256-byte row segments; row r's
  // 16-byte chunk c at c ^ rot(r), free of bank conflicts for both accesses.  (Stored from the accumulators, an instruction
  // touched 32 rows of 32 bytes.  us, projection along the sequence and its gradients, 48 heads of 114688 rows, Kp = 256: 217,
  // 444 -> 214, 435; 2 of 96768, 128: 22.3, 25.7 -> 22.2, 23.8; 11 of 128 of 8640, 192: 20.0, 22.2 -> 19.6, 21.5.)
  unsigned char *t0 = &lds_[0][0][0][0] + wave * 8192;
  static_assert(HT * 8192 <= KG * 4 * HT * kHalfBytes, "8 KiB a wave");
  auto place = [](int r, int c) { return r * 256 + ((c ^ ((r & 3) | ((r >> 1) & 4) | ((r & 4) << 1))) << 4); };
  const int64_t nw = n0 + wn * 64;
  if (nw >= g.N) return;
#pragma unroll
  for (int mb = 0; mb < T; ++mb) {
    const int64_t mw = m0 + wm * 32 * T + mb * 32;
    if (mw >= g.M) return;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x16 &c = acc[nb][mb];
        *reinterpret_cast<f32x4 *>(t0 + place(col, nb * 8 + q * 2 + half)) = f32x4{c[q * 4], c[q * 4 + 1], c[q * 4 + 2], c[q * 4 + 3]};
      }
    const int cc = lane & 15;
    int64_t off = ((int64_t)by * g.M + mw) * g.out_ld + nw + cc * 4;
    if (g.part_heads) {
      const uint32_t n = (uint32_t)nw + cc * 4, w = (uint32_t)g.out_ld, sh = w == 32 ? 5 : 6;  // (A / 2)
      off = ((int64_t)(by * (uint32_t)g.part_heads + (n >> sh)) * g.out_rows + mw) * g.out_ld + (n & (w - 1));
    }
    float *const out = static_cast<float *>(g.out[0]) + off;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int r = it * 4 + (lane >> 4);
      *reinterpret_cast<f32x4 *>(out + r * g.out_ld) = *reinterpret_cast<const f32x4 *>(t0 + place(r, cc));
    }
  }
}

template <bool A_KROWS, bool B_KROWS, bool OUT_F32, bool WIDE, int T, int KG, bool LONG>
__global__ void __launch_bounds__(128 * T * KG, 2) proj_gemm_kernel(GemmArgs g) {
  gemm_body<A_KROWS, B_KROWS, OUT_F32, WIDE, T, KG, LONG>(g, blockIdx.x, gridDim.x, blockIdx.y);
}

// Two products in one grid of work-groups of the same size (see plan_pair): the `cut` first work-groups form the product
// `first`.  GRAD_W: the gradients of a map of rows, by its input and, in fp32 and in k splits, by its weights; otherwise
// those of a projection along the sequence, dX = E dXp and dE = X dXp^T.
template <bool GRAD_W, bool WIDE, int T0, int K0, int T1, int K1>
__global__ void __launch_bounds__(128 * T0 * K0, 2) proj_gemm_pair_kernel(GemmArgs g0, GemmArgs g1, uint32_t cut,
                                                                          int first, uint32_t nx0, FastDiv by_nx1) {
  static_assert(T0 * K0 == T1 * K1, "one work-group size");
  const uint32_t id = blockIdx.x, own = id < cut ? id : id - cut;
  const uint32_t by1 = by_nx1(own), nx1 = by_nx1.d;
  if ((id < cut) == (first == 0))
    gemm_body<false, !GRAD_W, false, WIDE, T0, K0, false>(g0, own, nx0, 0);
  else
    gemm_body<GRAD_W, GRAD_W, true, WIDE, T1, K1, false>(g1, own - by1 * nx1, nx1, by1);
}

__global__ void __launch_bounds__(kReduceBlock) ksplit_reduce_kernel(const float *part, float *out, int64_t n4,
                                                                     int splits) {
  const int64_t i = (int64_t)blockIdx.x * kReduceBlock + threadIdx.x;
  if (i >= n4) return;
  const f32x4 *p = reinterpret_cast<const f32x4 *>(part) + i;
  reinterpret_cast<f32x4 *>(out)[i] = sum_of_splits<true>(splits, [&](int k) { return p[(int64_t)k * n4]; });
}

static MatView plain(const void *p, int64_t ld) {
  MatView v{};
  v.p[0] = static_cast<const uint16_t *>(p); v.ld = ld; v.split = 0; v.rows = 64; v.Z = 1; v.AH = 1;
  v.by_rows = make_fast_div(64); v.by_tensor = make_fast_div(1);
  return v;
}
static MatView heads(const void *p0, const void *p1, const void *p2, int64_t rows, int Z, int A = 64) {
  MatView v{};
  v.p[0] = static_cast<const uint16_t *>(p0); v.p[1] = static_cast<const uint16_t *>(p1);
  v.p[2] = static_cast<const uint16_t *>(p2); v.ld = A; v.rows = rows; v.Z = Z; v.AH = A / 64; v.split = 1;
  v.by_rows = make_fast_div(rows); v.by_tensor = make_fast_div((int64_t)Z * v.AH);
  return v;
}

static bool long_rows(const GemmArgs &g) { return g.A.ld > kMaxLd || g.B.ld > kMaxLd; }

static float tiles_of(int64_t M, int64_t N, int T) {
  const uint32_t t = 64 * (uint32_t)T;
  return (float)((((uint32_t)M + t - 1) / t) * (uint64_t)(((uint32_t)N + t - 1) / t));
}
static int next_splits(int s, int most) {
  const int next = s + (s < 4 ? 1 : (s < 8 ? 2 : (s < 16 ? 4 : (s < 32 ? 8 : 16))));
  return s < most && next > most ? most : next;
}
static float reduce_us(int64_t M, int64_t N, int s) {
  return s > 1 ? 3.0f + (float)s * (float)(M * N) * (4.0f / 5e6f) : 0.0f;
}

// Size of the work-groups' output tiles, groups per work-group and k splits: the candidate with the least estimated
// time (us).  n work-groups per CU (of which 1, 2, 4 are in flight) cost per slab of 32 k what was measured, and a round
// of them its prologue and epilogue; a split result is written and added up.  (Measured with M x N x K swept from
// 128 x 1856 x 28224 to 1664 x 5000 x 11520 and each T: the choice is within 10 % of the best on average.  T = 4 alone:
// 512 x 1408 x 1408: 31.7 us, now 10; 896 x 576 x 576: 15.8, now 6.)
// (Results in bf16: T = 4 as 62 products of 512 .. 50688 rows take it, and a last round of T = 2 that is partly empty for
// as much as it holds.  Q/K/V of 4096 rows of 2048: 127 -> 103 us with T = 4; of 8704 rows, 1088 -> 4608: 117 -> 99.)
// chain: where the result is kept in fp32, the slabs of 64 k that one chain of additions may take; its rounding error
// grows with the root of its length.  T = 4 has no registers for a second set of sums and takes as many splits as
// that asks for; the smaller tiles fold theirs.  (1024 x 1024 x 16384 in 4 splits, relative RMS error: one chain each
// 4.0e-7, folded at 1024 k 2.0e-7, as 16 splits give.)
// sum: the times of sums over many rows (weight gradients, projections along the sequence).
// Rows of more than kMaxLd elements: T = 4 (the only one with such loads) and all splits.
struct GemmPlan { int T, KG, splits, chain; float us; };
static GemmPlan plan_gemm(const GemmArgs &g, int max_splits, int chain = 1 << 29, bool sum = false) {
  const int64_t M = g.M, N = g.N, K = g.K;
  const int kslabs = (int)(K / 64);
  GemmPlan best{4, 1, max_splits, chain, 0.0f};
  if (long_rows(g)) return best;
  best.us = 1e30f;
  const float t4_full = sum ? 0.28f : 0.14f, last = sum ? 1.0f : 0.35f;
  for (int T = 4; T >= 1; T /= 2) {
    const float tiles = tiles_of(M, N, T);
    for (int s = 1; s <= max_splits; s = next_splits(s, max_splits)) {
      if (T == 4 && (kslabs + s - 1) / s > chain) continue;
      const float w = tiles * (float)s, n = ceilf(w * (1.0f / 256)), slabs = 2.0f * (float)((kslabs + s - 1) / s);
      float us;
      if (T == 4) us = n * (6.5f + slabs * (0.6f + t4_full * (w < 256 ? w * (1.0f / 256) : 1.0f)));
      else if (T == 2) us = n < 2 ? 4.0f + slabs * 0.29f
                            : 2.0f + (last * ceilf(n * 0.5f) + (1.0f - last) * fmaxf(1.0f, w * (1.0f / 512))) *
                                         (2.0f + slabs * 0.57f);
      else us = 2.0f + 1.5f * ceilf(n * 0.25f) + slabs * (n < 2 ? 0.20f : 0.13f * n);
      const float reduce = reduce_us(M, N, s);
      if (us + reduce < best.us) best = {T, 1, s, chain, us + reduce};
      if (T == 1) {
        const float second = n < 2 ? 0.0f : (w < 512 ? w * (1.0f / 256) - 1.0f : 1.0f);
        us = ceilf(n * 0.5f) * (4.5f + slabs * (0.15f + 0.05f * second));
        if (us + reduce < best.us) best = {1, 2, s, chain, us + reduce};
      }
    }
  }
  return best;
}

// The two products of a backward in one grid of work-groups of one size: where neither fills the chip, or fills it only
// in part of its last round, the other's work-groups take the CUs that are left, and one launch and its ramps go.
// (us, gradients of the Q/K/V and output maps, one launch each -> one grid: 128 rows, H = ZA = 768: 16.1 -> 11.6 and
// 10.0 -> 6.9; 1024 rows of 1024: 35.0 -> 25.0 and 18.7 -> 12.6; 4096 rows: 75.6 -> 59.9 and 36.7 -> 29.5; 16384 rows:
// 192 -> 188, and 88 either way; two launches stay where each is nearly full: 8192 rows of 1600, 254 against 289 in one
// grid.  Projection along the sequence, 5120 rows x 32 heads, Kp = 256: 30.2 -> 22.7; 87808 x 16, Kp = 192: 141 -> 137.)
// A work-group lasts fixed + slabs * r us, with r between that of a lone one and of a full chip (two of 256 threads per
// CU, one of 512).  The constants were fitted, those of the maps to 1400 timed launches of 65 pairs of 128 .. 50688 rows
// (off by 8 % RMS among the forms near the best; what is picked is 2 % above the best on average, and at most 1 % above
// two launches), those of the projections along the sequence, whose operands lie along the products' k, to 11 pairs.
struct WgTime {
  float fixed, alone, full;
  float operator()(int slabs, float fill) const {
    return fixed + (float)slabs * (alone + (full - alone) * (fill < 0.0f ? 0.0f : (fill > 1.0f ? 1.0f : fill)));
  }
};
static WgTime wg_time(int T, int KG, bool map) {
  if (T == 4) return map ? WgTime{8.5f, 0.47f, 0.74f} : WgTime{9.4f, 0.47f, 0.60f};
  if (T == 2 && KG == 2) return {7.2f, 0.19f, 0.265f};
  if (T == 2) return map ? WgTime{6.0f, 0.305f, 0.48f} : WgTime{5.1f, 0.30f, 0.41f};
  return map ? WgTime{2.7f, 0.15f, 0.24f} : WgTime{2.8f, 0.146f, 0.197f};
}
static int slabs_of(const GemmArgs &g, int splits) { return 2 * (int)((g.K / 64 + splits - 1) / splits); }

// A map's gradient alone in its launch, by the same constants.
static float launch_us(const GemmArgs &g, const GemmPlan &p) {
  const float per_cu = p.T == 4 ? 1.0f : (p.T == 1 && p.KG == 1 ? 4.0f : 2.0f);
  const float wgs = tiles_of(g.M, g.N, p.T) * (float)p.splits, rounds = wgs / (256.0f * per_cu);
  const int slabs = slabs_of(g, p.splits);
  const float each = p.T == 1 && p.KG == 1 ? 2.0f + (float)slabs * 0.2f
                                           : wg_time(p.T, p.KG, true)(slabs, wgs * (1.0f / 256) - (per_cu - 1.0f));
  return 2.5f + (0.7f * ceilf(rounds) + 0.3f * fmaxf(rounds, 1.0f)) * each + reduce_us(g.M, g.N, p.splits);
}

// The end of `na` work-groups of `ta` us, then `nb` of `tb`, each at the place that is free first; 0.3 of it by their sum,
// since they do not keep step.
static float both_us(int na, float ta, int nb, float tb, int places) {
  const int rounds = na / places, rest = na % places, free = places - rest;
  const float begin = (float)rounds * ta, sum = ((float)na * ta + (float)nb * tb) / (float)places;
  float end;
  if (rest == 0) {
    end = begin + (float)((nb + places - 1) / places) * tb;
  } else {
    // the least of begin + j tb and begin + ta + j tb by which all of the second kind are done
    auto done = [&](float t) {
      return free * (int)(t / tb + 1e-4f) + (t > ta ? rest * (int)((t - ta) / tb + 1e-4f) : 0) >= nb;
    };
    const float area = ((float)rest * ta + (float)nb * tb) / (float)places;
    int i = (int)(area / tb), j = area > ta ? (int)((area - ta) / tb) : 0;
    while (!done((float)i * tb)) ++i;
    while (!done(ta + (float)j * tb)) ++j;
    end = begin + fmaxf(ta, fminf((float)i * tb, ta + (float)j * tb));
  }
  return 0.7f * end + 0.3f * fmaxf(sum, fmaxf(ta, tb));
}

// Whether the work-groups of the second product are the longer ones, which the grid begins with.
static bool longer_first(int T0, int K0, int slabs0, int T1, int K1, int slabs1) {
  return (int64_t)slabs1 * T1 * T1 / K1 > (int64_t)slabs0 * T0 * T0 / K0;
}

struct PairPlan { GemmPlan p0, p1; float us; };
static PairPlan plan_pair(const GemmArgs &g0, const GemmArgs &g1, int max_splits, int chain, bool map) {
  static const int kinds[][4] = {{4, 1, 4, 1}, {2, 1, 2, 1}, {2, 1, 1, 2}, {1, 2, 1, 2}, {4, 1, 2, 2}, {1, 2, 2, 1}};
  PairPlan best{};
  best.us = 1e30f;
  for (int k = 0; k < (map ? 6 : 4); ++k) {
    const int *c = kinds[k], per_cu = c[0] == 4 ? 1 : 2;
    const WgTime t0 = wg_time(c[0], c[1], map), t1 = wg_time(c[2], c[3], map);
    const float n0 = tiles_of(g0.M, g0.N, c[0]), tiles1 = tiles_of(g1.M, g1.N, c[2]);
    if (n0 + tiles1 * (float)max_splits > 1e6f) continue;  // (far beyond where one grid gives anything)
    for (int s = 1; s <= max_splits; s = next_splits(s, max_splits)) {
      const int slabs0 = slabs_of(g0, 1), slabs1 = slabs_of(g1, s);
      if (c[2] == 4 && slabs1 > 2 * (int64_t)chain) continue;
      const float n1 = tiles1 * (float)s, fill = (n0 + n1) * (1.0f / 256) - (float)(per_cu - 1);
      const float ta = t0(slabs0, fill), tb = t1(slabs1, fill);
      float us = longer_first(c[0], c[1], slabs0, c[2], c[3], slabs1)
                     ? both_us((int)n1, tb, (int)n0, ta, 256 * per_cu)
                     : both_us((int)n0, ta, (int)n1, tb, 256 * per_cu);
      us += reduce_us(g1.M, g1.N, s);
      if (us < best.us) best = {{c[0], c[1], 1, 1 << 29, us}, {c[2], c[3], s, chain, us}, us};
    }
  }
  return best;
}

static bool wide_heads(const GemmArgs &g) {
  return (g.A.split && g.A.AH == 2) || (g.B.split && g.B.AH == 2) || (g.out_split && g.out_AH == 2);
}

// The fields of a product's arguments that its plan decides; returns the work-groups per split.
static uint32_t set_plan(GemmArgs &g, const GemmPlan &p) {
  const int64_t t = 64 * p.T;
  g.chain = p.chain;
  const int64_t ntiles = (g.N + t - 1) / t;
  g.by_ntiles = make_fast_div(ntiles);
  if (g.out_split) { g.by_out_rows = make_fast_div(g.out_rows); g.by_out_tensor = make_fast_div((int64_t)g.out_Z * g.out_AH); }
  g.kslabs = (g.K / 64 + p.splits - 1) / p.splits;
  return (uint32_t)(((g.M + t - 1) / t) * ntiles);
}

template <bool A_KROWS, bool B_KROWS, bool OUT_F32, int T, int KG>
static hipError_t launch_gemm_as(GemmArgs &g, const GemmPlan &p, hipStream_t st) {
  const uint32_t wgs = set_plan(g, p);
  const dim3 grid(wgs, (unsigned)p.splits), block(128 * T * KG);
  const bool wide = wide_heads(g);
  if constexpr (T == 4 && !(OUT_F32 && !A_KROWS)) {  // (dE's operands are rows of heads)
    if (long_rows(g)) {
      hipLaunchKernelGGL((proj_gemm_kernel<A_KROWS, B_KROWS, OUT_F32, true, T, KG, true>), grid, block, 0, st, g);
      return hipGetLastError();
    }
  }
  if (wide)
    hipLaunchKernelGGL((proj_gemm_kernel<A_KROWS, B_KROWS, OUT_F32, true, T, KG, false>), grid, block, 0, st, g);
  else
    hipLaunchKernelGGL((proj_gemm_kernel<A_KROWS, B_KROWS, OUT_F32, false, T, KG, false>), grid, block, 0, st, g);
  return hipGetLastError();
}
template <bool A_KROWS, bool B_KROWS, bool OUT_F32>
static hipError_t launch_gemm(GemmArgs &g, const GemmPlan &p, hipStream_t st) {
  if (p.T == 4) return launch_gemm_as<A_KROWS, B_KROWS, OUT_F32, 4, 1>(g, p, st);
  if (p.T == 2) return launch_gemm_as<A_KROWS, B_KROWS, OUT_F32, 2, 1>(g, p, st);
  if (p.KG == 2) return launch_gemm_as<A_KROWS, B_KROWS, OUT_F32, 1, 2>(g, p, st);
  return launch_gemm_as<A_KROWS, B_KROWS, OUT_F32, 1, 1>(g, p, st);
}

template <bool GRAD_W, int T0, int K0, int T1, int K1>
static hipError_t launch_pair_as(GemmArgs &g0, GemmArgs &g1, const GemmPlan &p0, const GemmPlan &p1, hipStream_t st) {
  const uint32_t nx0 = set_plan(g0, p0), nx1 = set_plan(g1, p1), n1 = nx1 * (uint32_t)p1.splits;
  const int first = longer_first(T0, K0, slabs_of(g0, p0.splits), T1, K1, slabs_of(g1, p1.splits));
  const dim3 grid(nx0 + n1), block(128 * T0 * K0);
  const uint32_t cut = first ? n1 : nx0;
  if (wide_heads(g0) || wide_heads(g1))
    hipLaunchKernelGGL((proj_gemm_pair_kernel<GRAD_W, true, T0, K0, T1, K1>), grid, block, 0, st, g0, g1, cut, first,
                       nx0, make_fast_div(nx1));
  else
    hipLaunchKernelGGL((proj_gemm_pair_kernel<GRAD_W, false, T0, K0, T1, K1>), grid, block, 0, st, g0, g1, cut, first,
                       nx0, make_fast_div(nx1));
  return hipGetLastError();
}
template <bool GRAD_W>
static hipError_t launch_pair(GemmArgs &g0, GemmArgs &g1, const PairPlan &p, hipStream_t st) {
  const GemmPlan &p0 = p.p0, &p1 = p.p1;
  if (p0.T == 4) {
    if (p1.T == 4) return launch_pair_as<GRAD_W, 4, 1, 4, 1>(g0, g1, p0, p1, st);
    if constexpr (GRAD_W) return launch_pair_as<GRAD_W, 4, 1, 2, 2>(g0, g1, p0, p1, st);
  }
  if (p0.T == 2) {
    if (p1.T == 2) return launch_pair_as<GRAD_W, 2, 1, 2, 1>(g0, g1, p0, p1, st);
    return launch_pair_as<GRAD_W, 2, 1, 1, 2>(g0, g1, p0, p1, st);
  }
  if constexpr (GRAD_W)
    if (p1.T == 2) return launch_pair_as<GRAD_W, 1, 2, 2, 1>(g0, g1, p0, p1, st);
  return launch_pair_as<GRAD_W, 1, 2, 1, 2>(g0, g1, p0, p1, st);
}

// Most k splits of a weight-gradient product (the workspace is sized by it): as many as still give every CU at most
// one work-group of T = 4.
int proj_wgrad_splits(int64_t Mout, int64_t Nout, int64_t K) {
  const int64_t tiles = ((Mout + 255) / 256) * ((Nout + 255) / 256);
  int64_t s = 256 / tiles;
  const int64_t slabs = K / 64;
  if (s > slabs / 4) s = slabs / 4;
  if (s < 1) s = 1;
  if (s > 64) s = 64;
  return (int)s;
}

// Slabs of 64 k of one chain of fp32 additions in such a product: what that many splits leave to each.
static int wgrad_chain(int64_t Mout, int64_t Nout, int64_t K) {
  const int s = proj_wgrad_splits(Mout, Nout, K);
  return (int)((K / 64 + s - 1) / s);
}
// ... after which the smaller tiles fold a gradient's: three quarters of it, since in few splits the folds are a chain as
// well, and 1024 k at the most.  (2304 rows, 640 -> 2880 weights, chain 320 k, relative RMS error in one split: 1.12e-7
// folded at the chain, 1.04 at three quarters; in two splits folded at it 1.06.)
static int grad_fold(int chain) { return chain > 21 ? 16 : (chain * 3 + 3) / 4; }

hipError_t proj_qkv(const Dims &d, int64_t H, const void *X, const void *W, void *Q, void *K, void *V,
                    hipStream_t st) {
  GemmArgs g{};
  g.M = (int64_t)d.B * d.Lq; g.N = 3LL * d.Z * d.A; g.K = H;
  g.A = plain(X, H);          // [M][K]
  g.B = plain(W, g.N);        // [K][N]
  g.out[0] = Q; g.out[1] = K; g.out[2] = V;
  g.out_split = 1; g.out_rows = d.Lq; g.out_Z = d.Z; g.out_AH = d.A / 64;
  return launch_gemm<false, true, false>(g, plan_gemm(g, 1), st);
}

hipError_t proj_out(const Dims &d, int64_t H, const void *O, const void *Wo, void *Y, hipStream_t st) {
  GemmArgs g{};
  g.M = (int64_t)d.B * d.Lq; g.N = H; g.K = (int64_t)d.Z * d.A;
  g.A = heads(O, nullptr, nullptr, d.Lq, d.Z, d.A);  // [M][K], column tile = (half of a) head
  g.B = plain(Wo, H);                           // [K][N]
  g.out[0] = Y; g.out_split = 0; g.out_ld = H;
  return launch_gemm<false, true, false>(g, plan_gemm(g, 1), st);
}

// The gradients of one of the maps, g0 that of its input and g1 that of its weights (kept in fp32, its sum over the
// rows in splits): in one grid where that is estimated to be faster and g1 does not lie over what g0 reads.
static hipError_t both_gradients(GemmArgs &g0, GemmArgs &g1, float *dW, float *part, const void *W, hipStream_t st) {
  const int most = proj_wgrad_splits(g1.M, g1.N, g1.K), chain = wgrad_chain(g1.M, g1.N, g1.K);
  const size_t n = (size_t)(g1.M * g1.N);
  const GemmPlan p0 = plan_gemm(g0, 1);
  GemmPlan p1 = plan_gemm(g1, most, chain, true);
  bool one_grid = !long_rows(g0) && !long_rows(g1) && !overlap(dW, n * 4, W, n * 2);
  PairPlan pair{};
  if (one_grid) {
    pair = plan_pair(g0, g1, most, chain, true);
    one_grid = pair.us < 0.92f * (launch_us(g0, p0) + launch_us(g1, p1));
  }
  p1.chain = pair.p1.chain = grad_fold(chain);
  const int splits = one_grid ? pair.p1.splits : p1.splits;
  g1.out[0] = splits > 1 ? part : dW;
  hipError_t e;
  if (one_grid) {
    e = launch_pair<true>(g0, g1, pair, st);
  } else {
    e = launch_gemm<false, false, false>(g0, p0, st);
    if (e == hipSuccess) e = launch_gemm<true, true, true>(g1, p1, st);
  }
  if (e != hipSuccess || splits == 1) return e;
  const int64_t n4 = (int64_t)n / 4;
  hipLaunchKernelGGL(ksplit_reduce_kernel, reduce_grid(n4), dim3(kReduceBlock), 0, st, part, dW, n4, splits);
  return hipGetLastError();
}

hipError_t proj_out_bwd(const Dims &d, int64_t H, const void *dY, const void *O, const void *Wo,
                        void *dO, float *dWo, float *part, hipStream_t st) {
  const int64_t M = (int64_t)d.B * d.Lq, ZA = (int64_t)d.Z * d.A;
  GemmArgs g{};  // dO = dY Wo^T, head-split
  g.M = M; g.N = ZA; g.K = H;
  g.A = plain(dY, H);   // [M][K]
  g.B = plain(Wo, H);   // [N][K]
  g.out[0] = dO; g.out_split = 1; g.out_rows = d.Lq; g.out_Z = d.Z; g.out_AH = d.A / 64;
  GemmArgs h{};  // dWo = O^T dY: contraction over the rows
  h.M = ZA; h.N = H; h.K = M;
  h.A = heads(O, nullptr, nullptr, d.Lq, d.Z, d.A);  // [K][M]
  h.B = plain(dY, H);                           // [K][N]
  h.out_split = 0; h.out_ld = H;
  return both_gradients(g, h, dWo, part, Wo, st);
}

hipError_t proj_qkv_bwd(const Dims &d, int64_t H, const void *dQ, const void *dK, const void *dV,
                        const void *X, const void *W, void *dX, float *dW, float *part,
                        hipStream_t st) {
  const int64_t M = (int64_t)d.B * d.Lq, N3 = 3LL * d.Z * d.A;
  GemmArgs g{};  // dX = [dQ | dK | dV] W^T
  g.M = M; g.N = H; g.K = N3;
  g.A = heads(dQ, dK, dV, d.Lq, d.Z, d.A);  // [M][K]
  g.B = plain(W, N3);                  // [N][K]
  g.out[0] = dX; g.out_split = 0; g.out_ld = H;
  GemmArgs h{};  // dW = X^T [dQ | dK | dV]
  h.M = H; h.N = N3; h.K = M;
  h.A = plain(X, H);                   // [K][M]
  h.B = heads(dQ, dK, dV, d.Lq, d.Z, d.A);  // [K][N]
  h.out_split = 0; h.out_ld = N3;
  return both_gradients(g, h, dW, part, W, st);
}

// ---- Linformer projections along the sequence (Table 3, row Projection) ----
// out (Zt, Kp, A) bf16 = sum over the k splits of part[s][k][zt*A + a], in a fixed order
__global__ void __launch_bounds__(kReduceBlock) ksplit_reduce_heads_kernel(const float *part, uint16_t *out,
                                                                           int64_t Kp, int64_t Zt, int splits, int A) {
  const uint32_t i = blockIdx.x * (uint32_t)kReduceBlock + threadIdx.x;  // one group of 4 columns
  const uint32_t n4 = (uint32_t)Zt * (uint32_t)(A / 4), total = (uint32_t)Kp * n4;
  if (i >= total) return;
  const uint32_t k = i / n4, c = (i - k * n4) * 4, sh = A == 64 ? 6 : 7;
  const f32x4 *p = reinterpret_cast<const f32x4 *>(part) + i;
  const f32x4 s = sum_of_splits(splits, [&](int j) { return p[(int64_t)j * total]; });
  const u32x2 w = {pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3])};
  *reinterpret_cast<u32x2 *>(out + ((((int64_t)(c >> sh)) * Kp + k) << sh) + (c & (uint32_t)(A - 1))) = w;
}
// dE (rows, Kp) from the partial sums that lie in dX's rows (see GemmArgs::part_heads)
__global__ void __launch_bounds__(kReduceBlock) de_reduce_kernel(const float *part, float *dE, int64_t n4, int64_t Kp,
                                                                 int64_t L, int splits, int part_heads, int w) {
  const int64_t i = (int64_t)blockIdx.x * kReduceBlock + threadIdx.x;
  if (i >= n4) return;
  const uint32_t kp4 = (uint32_t)Kp / 4, m = (uint32_t)i / kp4, n = ((uint32_t)i - m * kp4) * 4;
  const float *p = part + ((int64_t)(n / (uint32_t)w) * L + m) * w + n % (uint32_t)w;
  const int64_t stride = (int64_t)part_heads * L * w;
  reinterpret_cast<f32x4 *>(dE)[i] =
      sum_of_splits(splits, [&](int k) { return *reinterpret_cast<const f32x4 *>(p + k * stride); });
}

int linformer_splits(int64_t Kp, int64_t Zt, int64_t rows, int A) {
  return proj_wgrad_splits(Kp, Zt * A, rows);
}

// Xp (Zt, Kp, A) = E^T X over `rows` tokens: X (Zt, L, A) from token row0 on, E (rows, Kp) from row0 on
hipError_t linformer_project(int64_t Zt, int64_t L, int64_t rows, int64_t Kp, int A, const void *X,
                             const void *E, void *Xp, float *part, hipStream_t st) {
  GemmArgs g{};
  g.M = Kp; g.N = Zt * A; g.K = rows;
  g.A = plain(E, Kp);                               // [K = token][M = k]
  g.B = heads(X, nullptr, nullptr, L, (int)Zt, A);  // [K = token][N = (head, a)]; one "batch" of Zt heads
  const GemmPlan plan = plan_gemm(g, linformer_splits(Kp, Zt, rows, A), wgrad_chain(g.M, g.N, g.K), true);
  const size_t out_bytes = (size_t)(Zt * Kp * A) * 2;
  // One split leaves its sums in bf16, to the same bits, where Xp lies on nothing that other work-groups still read (us: 13 heads
  // of 448 rows, Kp = 512: 8.8 -> 6.1, 15 of 1280, 512: 12.0 -> 9.0, 160 of 1024, 512: 28.9 -> 19.7; 63 of 640, 3008: 39 -> 21).
  if (plan.splits == 1 && !overlap(Xp, out_bytes, X, (size_t)(((Zt - 1) * L + rows) * A) * 2) &&
      !overlap(Xp, out_bytes, E, (size_t)(rows * Kp) * 2)) {
    g.out[0] = Xp; g.out_split = 1; g.out_rows = Kp; g.out_Z = (int)Zt; g.out_AH = A / 64;
    return launch_gemm<true, true, false>(g, plan, st);
  }
  g.out[0] = part; g.out_split = 0; g.out_ld = g.N;
  hipError_t e = launch_gemm<true, true, true>(g, plan, st);
  if (e != hipSuccess) return e;
  const int64_t total = Kp * Zt * (A / 4);
  hipLaunchKernelGGL(ksplit_reduce_heads_kernel, reduce_grid(total), dim3(kReduceBlock), 0, st,
                     part, static_cast<uint16_t *>(Xp), Kp, Zt, plan.splits, A);
  return hipGetLastError();
}

// dX rows (Zt, L, A) from row0 on = E dXp, and dE (rows, Kp) fp32 = sum over heads of X dXp^T.
// dE first: with few rows its contraction over all heads is split, and the partial sums lie in the rows of dX that the
// second product then overwrites (A / 2 floats per row and head, so a split takes 2 Kp / A heads).  64 rows, Kp = 128,
// 180 heads of 128: one tile walked 23040 k in 427 us.  dE over E: dX, which reads E, comes first.
hipError_t linformer_project_bwd(int64_t Zt, int64_t L, int64_t rows, int64_t Kp, int A, const void *dXp,
                                 const void *X, const void *E, void *dX, float *dE, hipStream_t st) {
  const size_t x_bytes = (size_t)(((Zt - 1) * L + rows) * A) * 2;
  const bool dx_first = overlap(dE, (size_t)(rows * Kp) * 4, E, (size_t)(rows * Kp) * 2);
  GemmArgs x{};  // dX
  x.M = rows; x.N = Zt * A; x.K = Kp;
  x.A = plain(E, Kp);                                  // [M = token][K = k]
  x.B = heads(dXp, nullptr, nullptr, Kp, (int)Zt, A);  // [K = k][N = (head, a)]
  x.out[0] = dX; x.out_split = 1; x.out_rows = L; x.out_Z = (int)Zt; x.out_AH = A / 64;
  GemmArgs g{};  // dE
  g.M = rows; g.N = Kp; g.K = Zt * A;
  g.A = heads(X, nullptr, nullptr, L, (int)Zt, A);     // [M = token][K = (head, a)]
  g.B = heads(dXp, nullptr, nullptr, Kp, (int)Zt, A);  // [N = k][K = (head, a)]
  g.out[0] = dE; g.out_split = 0; g.out_ld = Kp;
  // (a gradient that overwrites X itself: X is read until dE is done, so its rows cannot hold partial sums, nor can
  // both be formed at once)
  const bool over = dx_first || overlap(X, x_bytes, dX, x_bytes);
  const bool by_heads = linformer_dx_supported(Kp, A);
  const int64_t part_heads = 2 * Kp / A;
  int64_t splits = Zt / part_heads;
  if (splits > g.K / 256) splits = g.K / 256;
  const int most = splits < 1 ? 1 : (splits > 64 ? 64 : (int)splits);
  // dE is kept in fp32, and its error grows with the root of its chains' length: T = 4 takes none longer than a sum that is
  // timed like the weight gradients' would be split into, and the smaller tiles fold theirs as those do.  (2048 rows, 32
  // heads of 64, Kp = 128, one grid, relative RMS error: chains of 1024 k 1.87e-7, folds of 192 0.93e-7, at 13.3 and 13.7 us.)
  const int slabs = (int)(g.K / 64), chain_splits = plan_gemm(g, most, slabs, true).splits;
  const int chain = (slabs + chain_splits - 1) / chain_splits, fold = grad_fold(wgrad_chain(g.M, g.N, g.K));
  GemmPlan plan = plan_gemm(g, most, chain), x_plan = plan_gemm(x, 1);
  PairPlan pair{};
  bool one_grid = !long_rows(g) && !long_rows(x);
  if (one_grid) {
    // (linformer_dx: its launch, E moved into registers, and dX written at 3.6 TB/s)
    const float dx_us = by_heads ? 2.5f + 0.015f * (float)Kp + (float)(rows * Zt * A) * (2.0f / 3.6e6f) : x_plan.us;
    pair = plan_pair(x, g, 1, chain, false);
    pair.p1.chain = fold;
    // (One grid moves X and dX at 3.6 TB/s at most, where the two launches' dX is a stream of its own: 16384 rows, 64 heads,
    // Kp = 128: 82 us, 68 in two launches, 80640 rows, 22 heads of 128: 293, 248; but 7296 rows, 27 heads, Kp = 256: 25.6, 36.5.
    // dE's folds are not in its estimate, hence the 3 %: of 260 calls of 128 .. 108864 rows and 2 .. 170 heads, the time of the slower
    // form where it is taken adds 0.6 % on average, 16 at most; with the line at 0.97 of two launches: 1.0 and 43.)
    const float one_us = fmaxf(pair.us, (float)(rows * Zt * A) * (4.0f / 3.6e6f));
    one_grid = one_us < 1.03f * (plan.us + dx_us);
  }
  if (one_grid && !over) return launch_pair<false>(x, g, pair, st);
  if (one_grid) x_plan = pair.p0;  // (dX's additions in the same order, wherever it lies)
  if (over) plan = plan_gemm(g, 1);
  plan.chain = fold;
  auto form_dx = [&]() -> hipError_t {
    if (by_heads && !one_grid) return linformer_dx(Zt, L, rows, Kp, A, dXp, E, dX, st);
    return launch_gemm<false, true, false>(x, x_plan, st);
  };
  if (dx_first) {
    hipError_t e = form_dx();
    if (e != hipSuccess) return e;
  }
  if (plan.splits > 1) {
    g.out[0] = dX; g.out_ld = A / 2; g.out_rows = L; g.part_heads = (int)part_heads;
  }
  hipError_t e = launch_gemm<false, false, true>(g, plan, st);
  if (e != hipSuccess) return e;
  if (plan.splits > 1) {
    const int64_t n4 = rows * Kp / 4;
    hipLaunchKernelGGL(de_reduce_kernel, reduce_grid(n4), dim3(kReduceBlock), 0, st, static_cast<const float *>(dX),
                       dE, n4, Kp, L, plan.splits, (int)part_heads, A / 2);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return dx_first ? hipSuccess : form_dx();
}

}  // namespace rsa
