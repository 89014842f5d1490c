// The two-pass layout of Ring Self-Attention (RSA_MODE_STAGED of rsa_forward and rsa_backward), bf16
// and fp32: the softmaxed strip S^n of Eq. 3 lives in device memory between the K ring pass and the
// V ring pass (section 3.1; Table 2, rows Ring-QK^T and Ring-AV).  A strip belongs to one head and a
// run of its query rows; the chunks that a rank's ring steps would bring one after the other are the
// strip's column tiles here, so a pass over them is one launch instead of N, and the ranks' rows are
// taken together as far as their strips fit the workspace.
//
//   forward    scores: S = Q K^T tile by tile, softmaxed against the tile's own row maximum:
//                strip tile = exp(S - m_t) (dtype), (m_t, l_t) per row and 64 keys
//              apply:  LSE from the pairs, O = sum_t exp(m_t - LSE) (strip tile) V
//   backward   scores: P = exp(S - LSE), dS = P o (dO V^T - D), both tiles written in dtype
//              apply:  dQ = s dS K;   collect: dV = P^T dO, dK = s dS^T Q
//
// Bytes per score: 2 es forward, 5 es backward (es: bytes of the dtype); every other operand is read
// from the caches.  The former version of this path kept S and dP as fp32 strips, softmaxed them in
// passes of their own and ran every product chunk by chunk: 12 (bf16) / 20 (fp32) bytes forward,
// 28 / 44 backward, and 10 N^2 launches.
//
// The tile kernels hold bf16 tiles in the layout of the fused kernels and fp32 tiles in one of their
// own; fp32 products run on v_mfma_f32_32x32x2_f32 (IEEE fp32 multiply-add, twice the rate of the
// vector unit).  All products are formed transposed: one lane owns one row of the result.
#include "rsa_fused_tile.h"
#include "rsa_kernels.h"

namespace rsa {
namespace {

// A 64 x 64 tile of T in LDS: how it is filled, read as MFMA operands and written as a result.
//   rows(t, rb, s):   operand whose row index runs over tile rows rb .. rb + 31, k over columns
//   rows_k(t, rb, s): the same with k in the order in which cols() delivers it
//   cols(t, s, cb):   operand whose row index runs over columns 32 cb .. 32 cb + 31, k over rows
// s: k slice of kSliceK; mfma() contracts one slice.
template <typename T> struct TileT;

template <> struct TileT<uint16_t> {
  typedef bf16x8 Frag;
  static constexpr int kBytes = kTileBytes, kSlices = 4, kSliceK = 16;
  TileLanes tl;
  __device__ __forceinline__ explicit TileT(int lane) : tl(lane) {}
  __device__ __forceinline__ Frag rows(const unsigned char *t, int rb, int s) const { return tl.read_rows(t, rb, s); }
  __device__ __forceinline__ Frag rows_k(const unsigned char *t, int rb, int s) const {
    return tl.read_rows_perm(t, rb, s);
  }
  __device__ __forceinline__ Frag cols(const unsigned char *t, int s, int cb) const {
    const int flip = cb << 6;  // the second column block: the other four of a row's eight chunks
    const u32x2 lo = lds_read_tr16(t + s * 2048 + (tl.cols_off[0][0] ^ flip));
    const u32x2 hi = lds_read_tr16(t + s * 2048 + (tl.cols_off[0][1] ^ flip));
    const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(Frag, w);
  }
  static __device__ __forceinline__ f32x16 mfma(Frag a, Frag b, f32x16 c) { return mfma_32x32x16(a, b, c); }
  static __device__ __forceinline__ float dot(Frag a, Frag b, float acc) {
    const u32x4 x = __builtin_bit_cast(u32x4, a), y = __builtin_bit_cast(u32x4, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = fmaf(bf16_to_f32(x[e] & 0xffffu), bf16_to_f32(y[e] & 0xffffu), acc);
      acc = fmaf(bf16_to_f32(x[e] >> 16), bf16_to_f32(y[e] >> 16), acc);
    }
    return acc;
  }
  static __device__ __forceinline__ void stage(unsigned char *t, const f32x16 &c0, const f32x16 &c1, float scale,
                                               int lane) {
    stage_block_T(t, 0, c0, c1, scale, lane);
  }
  static __device__ __forceinline__ void flush(const unsigned char *t, uint16_t *g, int64_t rows_valid, int lane,
                                               int64_t ld) {
    flush_rows<32>(t, 0, g, rows_valid, lane, (int)ld);
  }
  struct DMA {
    TileDMA d;
    __device__ __forceinline__ DMA(int wave, int lane, int64_t ld) : d(wave, lane, (int)ld) {}
    __device__ __forceinline__ void load(const uint16_t *g, unsigned char *t) const { d.load(g, t); }
  };
};

// fp32: row r occupies bytes [256 r, 256 r + 256), its 16-byte chunk cc sits at position cc ^ rot(r).
// rot takes bits 0, 1, 3, 2 of r to bits 0, 1, 2, 3: the 16 rows of a phase of a row read then
// touch 16 different positions, and the two lane halves of a column read (rows r and r + 4, eight
// chunks each) touch disjoint halves of the row: both are free of bank conflicts.
template <> struct TileT<float> {
  typedef f32x4 Frag;
  static constexpr int kBytes = 64 * 64 * 4, kSlices = 8, kSliceK = 8;
  int row0, col0;  // byte offsets of chunk `half` of row `col`, of element `col` of row 4 half
  static __device__ __forceinline__ int rot(int r) { return (r & 3) | ((r >> 1) & 4) | ((r & 4) << 1); }
  static __device__ __forceinline__ int off(int r, int cc) { return r * 256 + ((cc ^ rot(r)) << 4); }
  __device__ __forceinline__ explicit TileT(int lane) {
    const int col = lane & 31, half = lane >> 5;
    row0 = off(col, half);
    col0 = off(half * 4, col >> 2) + (col & 3) * 4;
  }
  // k of slice s: 8 s + 4 half + e in element e, both for rows and for columns
  __device__ __forceinline__ Frag rows(const unsigned char *t, int rb, int s) const {
    return *reinterpret_cast<const f32x4 *>(t + rb * 256 + (row0 ^ (s << 5)));
  }
  __device__ __forceinline__ Frag rows_k(const unsigned char *t, int rb, int s) const { return rows(t, rb, s); }
  __device__ __forceinline__ Frag cols(const unsigned char *t, int s, int cb) const {
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e)  // row 8 s + 4 half + e: its rot differs from that of row 4 half by these bits
      r[e] = *reinterpret_cast<const float *>(t + (s * 8 + e) * 256 + (col0 ^ (((cb << 3) ^ ((s & 1) << 2) ^ e) << 4)));
    return r;
  }
  static __device__ __forceinline__ f32x16 mfma(Frag a, Frag b, f32x16 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], c, 0, 0, 0);
    return c;
  }
  static __device__ __forceinline__ float dot(Frag a, Frag b, float acc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = fmaf(a[e], b[e], acc);
    return acc;
  }
  static __device__ __forceinline__ void stage(unsigned char *t, const f32x16 &c0, const f32x16 &c1, float scale,
                                               int lane) {
    const int col = lane & 31, half = lane >> 5;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      const f32x16 &c = db == 0 ? c0 : c1;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 w = {c[g * 4 + 0] * scale, c[g * 4 + 1] * scale, c[g * 4 + 2] * scale, c[g * 4 + 3] * scale};
        *reinterpret_cast<f32x4 *>(t + off(col, db * 8 + g * 2 + half)) = w;
      }
    }
  }
  static __device__ __forceinline__ void flush(const unsigned char *t, float *g, int64_t rows_valid, int lane,
                                               int64_t ld) {
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int row = it * 4 + (lane >> 4), cc = lane & 15;
      if (row < rows_valid)
        *reinterpret_cast<f32x4 *>(g + row * ld + cc * 4) = *reinterpret_cast<const f32x4 *>(t + off(row, cc));
    }
  }
  struct DMA {
    int g_off[4], l_off[4];
    __device__ __forceinline__ DMA(int wave, int lane, int64_t ld) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = (wave * 4 + j) * 64 + lane, row = p >> 4, cc = (p & 15) ^ rot(row);
        g_off[j] = row * (int)ld + cc * 4;
        l_off[j] = (wave * 4 + j) * 1024;
      }
    }
    __device__ __forceinline__ void load(const float *g, unsigned char *t) const {
#pragma unroll
      for (int j = 0; j < 4; ++j) lds_dma16(g + g_off[j], t + l_off[j]);
    }
  };
};

struct StripArgs {
  const void *Q, *K, *V, *dO, *O;  // first head of the group; Q, dO, O: first row of the group
  const float *LSE_in;
  float *LSE;                      // (head, Lq), first row of the group
  void *strip, *strip2;            // (head, rows, L): exp(S - m_t) or P; dS
  float *stats;                    // (head, L / 64, rows, 2): m_t and l_t, base-2 logarithm domain
  int64_t L, Lq, rows, q0;         // rows of the group; token of its first row
  int A, causal, rtiles, kblocks;  // 128-row tiles; key blocks
  float cl2, scale, inv_scale;
};

// Group of 64 rows that a wave's 32 rows belong to: a strip tile (64 rows x 64 keys) is written, and read,
// when its first key is visible to the last of its rows.
__device__ __forceinline__ bool tile_seen(const StripArgs &a, int64_t row, int64_t k0) {
  return !a.causal || k0 <= a.q0 + (row | 63);
}

// ---------------------------------------------------------------- scores ----
// Work-group: 128 rows (wave: 32, their Q as B operands in registers) x NKT tiles of 64 keys, whose K
// tiles are in LDS.  Nothing is pipelined inside a work-group: it is short (bound by the strip's stores
// in bf16, by the matrix pipe in fp32), and two to four of them share a compute unit.
template <typename T, int AH, int NKT>
__global__ void __launch_bounds__(256, AH <= 2 ? 2 : 1) strip_scores_fwd_kernel(StripArgs a) {
  typedef TileT<T> TT;
  constexpr int NS = TT::kSlices;
  __shared__ __attribute__((aligned(16))) unsigned char Kt[NKT][AH][TT::kBytes];
  __shared__ __attribute__((aligned(16))) unsigned char stg[4][TT::kBytes / 2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t key0 = (int64_t)(wg % (uint32_t)a.kblocks) * (64 * NKT);
  const uint32_t hr = wg / (uint32_t)a.kblocks;
  const int64_t head = hr / (uint32_t)a.rtiles, row0 = (int64_t)(hr % (uint32_t)a.rtiles) * 128;
  const int64_t row_last = (row0 + 128 < a.rows ? row0 + 128 : a.rows) - 1;
  if (!tile_seen(a, row_last, key0)) return;

  const T *Kh = static_cast<const T *>(a.K) + head * a.L * a.A;
  const typename TT::DMA dma(wave, lane, a.A);
#pragma unroll
  for (int u = 0; u < NKT; ++u)
    if (key0 + u * 64 < a.L)
#pragma unroll
      for (int ah = 0; ah < AH; ++ah) dma.load(Kh + (key0 + u * 64) * a.A + ah * 64, Kt[u][ah]);
  const int64_t wrow = row0 + wave * 32;  // (rows come in multiples of 64: a wave's rows are there or not)
  const bool rows_here = wrow < a.rows;
  typename TT::Frag q[AH * NS];
  if (rows_here) {
    const T *qp = static_cast<const T *>(a.Q) + (head * a.Lq + wrow + col) * a.A + half * (TT::kSliceK / 2);
#pragma unroll
    for (int i = 0; i < AH * NS; ++i)
      q[i] = *reinterpret_cast<const typename TT::Frag *>(qp + i * TT::kSliceK);
  }
  const TT tt(lane);
  wait_vmem();
  __syncthreads();
  if (!rows_here) return;
#pragma unroll
  for (int u = 0; u < NKT; ++u) {
    const int64_t k0 = key0 + u * 64;
    if (k0 >= a.L || !tile_seen(a, wrow, k0)) break;
    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int v = 0; v < 16; ++v) s[kb][v] = 0.f;
#pragma unroll
      for (int i = 0; i < AH * NS; ++i) s[kb] = TT::mfma(tt.rows(Kt[u][i / NS], kb * 32, i % NS), q[i], s[kb]);
    }
    if (a.causal && k0 + 63 > a.q0 + wrow) {  // last visible key of the lane's row, relative to the tile
      const int64_t d64 = a.q0 + wrow + col - k0 - half * 4;
      const int dlast = d64 > 64 ? 64 : (int)d64;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kb * 32 + (v >> 2) * 8 + (v & 3) > dlast) s[kb][v] = -INFINITY;
    }
    float m = s[0][0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m = fmaxf(m, s[0][v]);
#pragma unroll
    for (int v = 0; v < 16; ++v) m = fmaxf(m, s[1][v]);
    m = xhalf_max(m);
    const float mc = m > -INFINITY ? m * a.cl2 : 0.f;  // a row that sees none of these keys: all zeros
    float l = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[kb][v] = __builtin_amdgcn_exp2f(fmaf(s[kb][v], a.cl2, -mc));
        l += s[kb][v];
      }
    l = xhalf_sum(l);
    if (half == 0) {
      f32x2 p = {m > -INFINITY ? mc : -INFINITY, l};
      *reinterpret_cast<f32x2 *>(a.stats + ((head * (a.L / 64) + k0 / 64) * a.rows + wrow + col) * 2) = p;
    }
    TT::stage(stg[wave], s[0], s[1], 1.0f, lane);
    TT::flush(stg[wave], static_cast<T *>(a.strip) + (head * a.rows + wrow) * a.L + k0, 32, lane, a.L);
  }
}

template <typename T, int AH, int NKT>
__global__ void __launch_bounds__(256, sizeof(T) * AH <= 4 ? 2 : 1) strip_scores_bwd_kernel(StripArgs a) {
  typedef TileT<T> TT;
  constexpr int NS = TT::kSlices;
  __shared__ __attribute__((aligned(16))) unsigned char Kt[NKT][AH][TT::kBytes], Vt[NKT][AH][TT::kBytes];
  __shared__ __attribute__((aligned(16))) unsigned char stg[4][TT::kBytes / 2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t key0 = (int64_t)(wg % (uint32_t)a.kblocks) * (64 * NKT);
  const uint32_t hr = wg / (uint32_t)a.kblocks;
  const int64_t head = hr / (uint32_t)a.rtiles, row0 = (int64_t)(hr % (uint32_t)a.rtiles) * 128;
  const int64_t row_last = (row0 + 128 < a.rows ? row0 + 128 : a.rows) - 1;
  if (!tile_seen(a, row_last, key0)) return;

  const T *Kh = static_cast<const T *>(a.K) + head * a.L * a.A, *Vh = static_cast<const T *>(a.V) + head * a.L * a.A;
  const typename TT::DMA dma(wave, lane, a.A);
#pragma unroll
  for (int u = 0; u < NKT; ++u)
    if (key0 + u * 64 < a.L)
#pragma unroll
      for (int ah = 0; ah < AH; ++ah) {
        dma.load(Kh + (key0 + u * 64) * a.A + ah * 64, Kt[u][ah]);
        dma.load(Vh + (key0 + u * 64) * a.A + ah * 64, Vt[u][ah]);
      }
  const int64_t wrow = row0 + wave * 32;
  const bool rows_here = wrow < a.rows;
  typename TT::Frag q[AH * NS], g[AH * NS];
  float nl = 0.f, nd = 0.f;  // -LSE / scale and -D of the lane's row: what the accumulators start from
  if (rows_here) {
    const int64_t off = (head * a.Lq + wrow + col) * a.A + half * (TT::kSliceK / 2);
    const T *qp = static_cast<const T *>(a.Q) + off, *gp = static_cast<const T *>(a.dO) + off;
    const T *op = static_cast<const T *>(a.O) + off;
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < AH * NS; ++i) {
      q[i] = *reinterpret_cast<const typename TT::Frag *>(qp + i * TT::kSliceK);
      g[i] = *reinterpret_cast<const typename TT::Frag *>(gp + i * TT::kSliceK);
      acc = TT::dot(g[i], *reinterpret_cast<const typename TT::Frag *>(op + i * TT::kSliceK), acc);
    }
    nd = -xhalf_sum(acc);
    nl = -a.LSE_in[head * a.Lq + wrow + col] * a.inv_scale;
  }
  const TT tt(lane);
  wait_vmem();
  __syncthreads();
  if (!rows_here) return;
#pragma unroll
  for (int u = 0; u < NKT; ++u) {
    const int64_t k0 = key0 + u * 64;
    if (k0 >= a.L || !tile_seen(a, wrow, k0)) break;
    f32x16 s[2], dp[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int v = 0; v < 16; ++v) { s[kb][v] = nl; dp[kb][v] = nd; }
#pragma unroll
      for (int i = 0; i < AH * NS; ++i) {
        s[kb] = TT::mfma(tt.rows(Kt[u][i / NS], kb * 32, i % NS), q[i], s[kb]);
        dp[kb] = TT::mfma(tt.rows(Vt[u][i / NS], kb * 32, i % NS), g[i], dp[kb]);
      }
    }
    if (a.causal && k0 + 63 > a.q0 + wrow) {
      const int64_t d64 = a.q0 + wrow + col - k0 - half * 4;
      const int dlast = d64 > 64 ? 64 : (int)d64;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kb * 32 + (v >> 2) * 8 + (v & 3) > dlast) s[kb][v] = -INFINITY;
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[kb][v] = __builtin_amdgcn_exp2f(s[kb][v] * a.cl2);
        dp[kb][v] *= s[kb][v];
      }
    const int64_t o = (head * a.rows + wrow) * a.L + k0;
    TT::stage(stg[wave], s[0], s[1], 1.0f, lane);  // (LDS operations of a wave complete in order)
    TT::flush(stg[wave], static_cast<T *>(a.strip) + o, 32, lane, a.L);
    TT::stage(stg[wave], dp[0], dp[1], 1.0f, lane);
    TT::flush(stg[wave], static_cast<T *>(a.strip2) + o, 32, lane, a.L);
  }
}

// ----------------------------------------------------------------- apply ----
// out (row, A) = scale * sum over keys of strip(row, key) X(key, A).  Work-group: 128 rows (wave: 32) x
// 64 AHW columns, walking the key tiles; strip and X tiles reach LDS by direct loads, double-buffered,
// one barrier per tile.  WEIGHT (forward): the strip is exp(S - m_t); the weights exp(m_t - LSE) bring
// the tiles to one reference, and LSE is written here.
struct ApplyArgs {
  const void *strip, *X;
  void *out;
  const float *stats;
  float *LSE;
};

template <typename T, int AHW, bool WEIGHT>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? 1 : (AHW == 1 ? 3 : 2)) strip_apply_kernel(StripArgs a, ApplyArgs p) {
  typedef TileT<T> TT;
  constexpr int NS = TT::kSlices;
  struct Stage { unsigned char S[2][TT::kBytes], X[AHW][TT::kBytes]; };
  __shared__ __attribute__((aligned(16))) Stage st0, st1;  // separate objects: see the fused kernels
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t cblocks = (uint32_t)(a.A / (64 * AHW));
  const int a0 = (int)(wg % cblocks) * (64 * AHW);
  const uint32_t hr = wg / cblocks;
  // under the causal mask later rows see more keys: the long work-groups start first
  const uint32_t rt = hr % (uint32_t)a.rtiles;
  const int64_t head = hr / (uint32_t)a.rtiles, row0 = (int64_t)(a.causal ? a.rtiles - 1 - rt : rt) * 128;
  const int64_t row_last = (row0 + 128 < a.rows ? row0 + 128 : a.rows) - 1;
  const int ntiles = (int)(a.L / 64);
  int nt = ntiles;
  if (a.causal && (a.q0 + row_last) / 64 + 1 < nt) nt = (int)((a.q0 + row_last) / 64) + 1;

  const T *Sh = static_cast<const T *>(p.strip) + (head * a.rows + row0) * a.L;
  const int64_t second = row0 + 64 < a.rows ? 64 * a.L : 0;  // (no second half: refetch the first)
  const T *Xh = static_cast<const T *>(p.X) + head * a.L * a.A + a0;
  const typename TT::DMA dma_s(wave, lane, a.L), dma_x(wave, lane, a.A);
  auto load = [&](int t, Stage &st) __attribute__((always_inline)) {
    dma_s.load(Sh + t * 64, st.S[0]);
    dma_s.load(Sh + second + t * 64, st.S[1]);
#pragma unroll
    for (int ah = 0; ah < AHW; ++ah) dma_x.load(Xh + (int64_t)t * 64 * a.A + ah * 64, st.X[ah]);
  };
  load(0, st0);

  const int64_t wrow = row0 + wave * 32;
  const bool rows_here = wrow < a.rows;
  const float *stats = WEIGHT ? p.stats + ((head * ntiles) * a.rows + (rows_here ? wrow : row0) + col) * 2 : nullptr;
  float lse2 = 0.f;
  if (WEIGHT) {
    // LSE = log sum_t l_t exp(m_t): the two lane halves take every other tile of their row
    const int seen = a.causal ? (int)((a.q0 + ((rows_here ? wrow : row0) | 63)) / 64) + 1 : ntiles;
    const int n = seen < ntiles ? seen : ntiles;
    float M = -INFINITY, l = 0.f;
    for (int t = half; t < n; t += 2) {
      const f32x2 ml = *reinterpret_cast<const f32x2 *>(stats + (int64_t)t * a.rows * 2);
      const float mn = fmaxf(M, ml[0]);
      if (mn > -INFINITY)
        l = l * __builtin_amdgcn_exp2f(M - mn) + ml[1] * __builtin_amdgcn_exp2f(ml[0] - mn);
      M = mn;
    }
    const float MM = xhalf_max(M);  // finite: every row sees some key
    l = xhalf_sum(M > -INFINITY ? l * __builtin_amdgcn_exp2f(M - MM) : 0.f);
    lse2 = MM + __builtin_amdgcn_logf(l);
    if (rows_here && half == 0 && a0 == 0) p.LSE[head * a.Lq + wrow + col] = lse2 * kLn2;
  }
  const TT tt(lane);
  f32x16 o[2 * AHW];
#pragma unroll
  for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;

  int t = 0;
  wait_vmem();
  __syncthreads();
  auto step = [&](Stage &cur, Stage &nxt) __attribute__((always_inline)) {
    float w = 0.f;
    if (WEIGHT) w = __builtin_amdgcn_exp2f(stats[(int64_t)t * a.rows * 2] - lse2);
    if (t + 1 < nt) load(t + 1, nxt);
    if (rows_here && tile_seen(a, wrow, (int64_t)t * 64)) {
      const unsigned char *S = cur.S[wave >> 1];
      if constexpr (WEIGHT && sizeof(T) == 2) {
        // the weight cannot enter the bf16 operand without rounding it again: it goes to the tile's sum
        f32x16 c[2 * AHW];
#pragma unroll
        for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) c[db][v] = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const typename TT::Frag b = tt.rows_k(S, (wave & 1) * 32, s);
#pragma unroll
          for (int db = 0; db < 2 * AHW; ++db) c[db] = TT::mfma(tt.cols(cur.X[db >> 1], s, db & 1), b, c[db]);
        }
#pragma unroll
        for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[db][v] = fmaf(w, c[db][v], o[db][v]);
      } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          typename TT::Frag b = tt.rows_k(S, (wave & 1) * 32, s);
          if constexpr (WEIGHT) b *= w;
#pragma unroll
          for (int db = 0; db < 2 * AHW; ++db) o[db] = TT::mfma(tt.cols(cur.X[db >> 1], s, db & 1), b, o[db]);
        }
      }
    }
    wait_vmem();
    __syncthreads();
    ++t;
  };
  while (t < nt) {
    step(st0, st1);
    if (t >= nt) break;
    step(st1, st0);
  }
  if (!rows_here) return;
  unsigned char *ot = &st0.S[0][0] + wave * (TT::kBytes / 2);
  T *out = static_cast<T *>(p.out) + (head * a.Lq + wrow) * a.A + a0;
#pragma unroll
  for (int ah = 0; ah < AHW; ++ah) {
    TT::stage(ot, o[2 * ah], o[2 * ah + 1], WEIGHT ? 1.0f : a.scale, lane);
    TT::flush(ot, out + ah * 64, 32, lane, a.A);
  }
}

// --------------------------------------------------------------- collect ----
// out (key, A) = alpha * sum over the group's rows of strip(row, key) Y(row, A), two products per launch
// (dV from P and dO, dK from dS and Q).  Work-group: 128 keys (wave: 32) x 64 AHW columns, walking the row
// tiles.  With several row groups the sums pass through fp32 accumulators: `add` continues them, `keep`
// leaves them there instead of writing the result.
struct CollectArgs {
  const void *strip[2], *Y[2];
  void *out[2];
  float *acc[2];
  float alpha[2];
  int add, keep;
};

template <typename T, int AHW>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? 1 : (AHW == 1 ? 3 : 2)) strip_collect_kernel(StripArgs a, CollectArgs p) {
  typedef TileT<T> TT;
  constexpr int NS = TT::kSlices;
  struct Stage { unsigned char S[2][TT::kBytes], Y[AHW][TT::kBytes]; };
  __shared__ __attribute__((aligned(16))) Stage st0, st1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t cblocks = (uint32_t)(a.A / (64 * AHW));
  const int a0 = (int)(wg % cblocks) * (64 * AHW);
  wg /= cblocks;
  const bool which = wg & 1;
  wg >>= 1;
  const int64_t key0 = (int64_t)(wg % (uint32_t)a.kblocks) * 128;
  const int64_t head = wg / (uint32_t)a.kblocks;
  const int nt = (int)(a.rows / 64);
  int t = 0;
  if (a.causal && key0 > a.q0 + 63) {  // first row tile whose last row sees the block's first key
    const int64_t f = (key0 - a.q0) / 64;
    t = f < nt ? (int)f : nt;
  }
  const T *Sh = static_cast<const T *>(which ? p.strip[1] : p.strip[0]) + head * a.rows * a.L + key0;
  const int64_t second = key0 + 64 < a.L ? 64 : 0;
  const T *Yh = static_cast<const T *>(which ? p.Y[1] : p.Y[0]) + head * a.Lq * a.A + a0;
  const typename TT::DMA dma_s(wave, lane, a.L), dma_y(wave, lane, a.A);
  auto load = [&](int tt_, Stage &st) __attribute__((always_inline)) {
    const T *s = Sh + (int64_t)tt_ * 64 * a.L;
    dma_s.load(s, st.S[0]);
    dma_s.load(s + second, st.S[1]);
#pragma unroll
    for (int ah = 0; ah < AHW; ++ah) dma_y.load(Yh + (int64_t)tt_ * 64 * a.A + ah * 64, st.Y[ah]);
  };
  load(t < nt ? t : nt - 1, st0);  // (a block that no row sees: any tile)
  const int64_t wkey = key0 + wave * 32, wtile = key0 + (wave >> 1) * 64;
  const bool keys_here = wkey < a.L;
  const TT tt(lane);
  f32x16 o[2 * AHW];
#pragma unroll
  for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  wait_vmem();
  __syncthreads();
  auto step = [&](Stage &cur, Stage &nxt) __attribute__((always_inline)) {
    if (t + 1 < nt) load(t + 1, nxt);
    if (keys_here && tile_seen(a, (int64_t)t * 64, wtile)) {
      const unsigned char *S = cur.S[wave >> 1];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const typename TT::Frag b = tt.cols(S, s, wave & 1);
#pragma unroll
        for (int db = 0; db < 2 * AHW; ++db) o[db] = TT::mfma(tt.cols(cur.Y[db >> 1], s, db & 1), b, o[db]);
      }
    }
    wait_vmem();
    __syncthreads();
    ++t;
  };
  while (t < nt) {
    step(st0, st1);
    if (t >= nt) break;
    step(st1, st0);
  }
  if (!keys_here) return;
  if (p.add || p.keep) {
    float *acc = (which ? p.acc[1] : p.acc[0]) + (head * a.L + wkey + col) * a.A + a0 + half * 4;
#pragma unroll
    for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 *q = reinterpret_cast<f32x4 *>(acc + db * 32 + g * 8);
        f32x4 w = {o[db][g * 4 + 0], o[db][g * 4 + 1], o[db][g * 4 + 2], o[db][g * 4 + 3]};
        if (p.add) w += *q;
        if (p.keep) *q = w;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][g * 4 + e] = w[e];
      }
    if (p.keep) return;
  }
  const float alpha = which ? p.alpha[1] : p.alpha[0];
  unsigned char *ot = &st0.S[0][0] + wave * (TT::kBytes / 2);
  T *out = static_cast<T *>(which ? p.out[1] : p.out[0]) + (head * a.L + wkey) * a.A + a0;
#pragma unroll
  for (int ah = 0; ah < AHW; ++ah) {
    TT::stage(ot, o[2 * ah], o[2 * ah + 1], alpha, lane);
    TT::flush(ot, out + ah * 64, 32, lane, a.A);
  }
}

// ------------------------------------------------------------------ host ----
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// How the work is cut: `heads` heads and `rows` of their query rows per group of launches, and where a
// group's buffers lie in the workspace.
struct StripPlan {
  int64_t heads, rows;
  size_t strip, strip2, stats, acc_k, acc_v, total;
};

// The strips of a group fit into `kStripBytes`, or into what the strips of one rank take when every score
// has an fp32 and a dtype copy (per pass), whichever is more: the ranks' rows are then taken together
// whenever the sizes are ordinary.
constexpr size_t kStripBytes = (size_t)192 << 20;

StripPlan strip_plan(const Dims &d, int dtype, int pass) {
  const size_t es = dtype == RSA_BF16 ? 2 : 4, strips = pass == 1 ? 2 : 1;
  const int64_t heads = (int64_t)d.B * d.Z;
  const size_t one_rank = (size_t)heads * d.c * d.L * (4 + es) * strips;
  const size_t row = (size_t)d.L * es * strips;  // bytes of a head's row
  const size_t budget = row * d.Lq <= kStripBytes || one_rank <= kStripBytes ? kStripBytes : one_rank;
  StripPlan p{};
  if (row * d.Lq <= budget) {
    p.rows = d.Lq;
    p.heads = (int64_t)(budget / (row * d.Lq));
    if (p.heads > heads) p.heads = heads;
    const int64_t groups = (heads + p.heads - 1) / p.heads;
    p.heads = (heads + groups - 1) / groups;  // groups of equal size
  } else {
    p.heads = 1;
    p.rows = (int64_t)(budget / row) / 128 * 128;  // at least one rank's rows of every head: never 0
  }
  const size_t scores = (size_t)p.heads * p.rows * d.L;
  size_t off = 0;
  p.strip = off; off += align256(scores * es);
  if (pass == 1) {
    p.strip2 = off; off += align256(scores * es);
    if (p.rows < d.Lq) {
      p.acc_k = off; off += align256((size_t)p.heads * d.L * d.A * 4);
      p.acc_v = off; off += align256((size_t)p.heads * d.L * d.A * 4);
    }
  } else {
    p.stats = off; off += align256(scores / 64 * 8);
  }
  p.total = off;
  return p;
}

template <typename T>
hipError_t launch_scores(const StripArgs &a0, int64_t heads, int A, bool bwd, hipStream_t st) {
  StripArgs a = a0;
  // key tiles per work-group: two where LDS has room for them beside a second work-group's
#define RSA_SCORES(AH, NF, NB)                                                                     \
  case AH: {                                                                                       \
    constexpr int nf = NF, nb = NB;                                                                \
    const int nk = bwd ? nb : nf;                                                                  \
    a.kblocks = (int)((a.L / 64 + nk - 1) / nk);                                                   \
    const dim3 grid((unsigned)(heads * a.rtiles * a.kblocks));                                     \
    if (bwd) hipLaunchKernelGGL((strip_scores_bwd_kernel<T, AH, nb>), grid, dim3(256), 0, st, a);  \
    else hipLaunchKernelGGL((strip_scores_fwd_kernel<T, AH, nf>), grid, dim3(256), 0, st, a);      \
    break;                                                                                         \
  }
  constexpr bool bf = sizeof(T) == 2;
  switch (A / 64) {
    RSA_SCORES(1, 2, (bf ? 2 : 1))
    RSA_SCORES(2, (bf ? 2 : 1), 1)
    RSA_SCORES(3, 1, 1)
    default:
    RSA_SCORES(4, 1, 1)
  }
#undef RSA_SCORES
  return hipGetLastError();
}

template <typename T, bool WEIGHT>
hipError_t launch_apply(const StripArgs &a, const ApplyArgs &p, int64_t heads, hipStream_t st) {
  const bool wide = a.A % 128 == 0;
  const dim3 grid((unsigned)(heads * a.rtiles * (a.A / (wide ? 128 : 64))));
  if (wide) hipLaunchKernelGGL((strip_apply_kernel<T, 2, WEIGHT>), grid, dim3(256), 0, st, a, p);
  else hipLaunchKernelGGL((strip_apply_kernel<T, 1, WEIGHT>), grid, dim3(256), 0, st, a, p);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_collect(const StripArgs &a0, const CollectArgs &p, int64_t heads, hipStream_t st) {
  StripArgs a = a0;
  a.kblocks = (int)((a.L + 127) / 128);
  const bool wide = a.A % 128 == 0;
  const dim3 grid((unsigned)(heads * a.kblocks * 2 * (a.A / (wide ? 128 : 64))));
  if (wide) hipLaunchKernelGGL((strip_collect_kernel<T, 2>), grid, dim3(256), 0, st, a, p);
  else hipLaunchKernelGGL((strip_collect_kernel<T, 1>), grid, dim3(256), 0, st, a, p);
  return hipGetLastError();
}

#define RSA_TRY(expr)                       \
  do {                                      \
    hipError_t e_ = (expr);                 \
    if (e_ != hipSuccess) return e_;        \
  } while (0)

// The group of `heads` heads from h0 on and `rows` rows from r0 on.
template <typename T>
StripArgs group_args(const Dims &d, const StripPlan &pl, char *ws, int64_t h0, int64_t r0, int64_t rows,
                     const void *Q, const void *K, const void *V) {
  StripArgs a{};
  const int64_t q = (h0 * d.Lq + r0) * d.A, k = h0 * d.L * d.A;
  a.Q = static_cast<const T *>(Q) + q;
  a.K = static_cast<const T *>(K) + k; a.V = static_cast<const T *>(V) + k;
  a.strip = ws + pl.strip; a.strip2 = ws + pl.strip2;
  a.stats = reinterpret_cast<float *>(ws + pl.stats);
  a.L = d.L; a.Lq = d.Lq; a.rows = rows; a.q0 = (int64_t)d.rank_begin * d.c + r0;
  a.A = d.A; a.causal = d.causal; a.rtiles = (int)((rows + 127) / 128);
  a.cl2 = d.scale * kLog2e; a.scale = d.scale; a.inv_scale = 1.0f / d.scale;
  return a;
}

template <typename T>
hipError_t forward_t(const Dims &d, int dtype, const void *Q, const void *K, const void *V, void *O, float *LSE,
                     char *ws, hipStream_t st) {
  const StripPlan pl = strip_plan(d, dtype, 0);
  const int64_t heads = (int64_t)d.B * d.Z;
  for (int64_t h0 = 0; h0 < heads; h0 += pl.heads) {
    const int64_t nh = pl.heads < heads - h0 ? pl.heads : heads - h0;
    for (int64_t r0 = 0; r0 < d.Lq; r0 += pl.rows) {
      const int64_t nr = pl.rows < d.Lq - r0 ? pl.rows : d.Lq - r0;
      const StripArgs a = group_args<T>(d, pl, ws, h0, r0, nr, Q, K, V);
      RSA_TRY(launch_scores<T>(a, nh, d.A, false, st));
      const ApplyArgs p = {a.strip, a.V, static_cast<T *>(O) + (h0 * d.Lq + r0) * d.A, a.stats,
                           LSE + h0 * d.Lq + r0};
      RSA_TRY((launch_apply<T, true>(a, p, nh, st)));
    }
  }
  return hipSuccess;
}

template <typename T>
hipError_t backward_t(const Dims &d, int dtype, const void *dO, const void *Q, const void *K, const void *V,
                      const void *O, const float *LSE, void *dQ, void *dK, void *dV, char *ws, hipStream_t st) {
  const StripPlan pl = strip_plan(d, dtype, 1);
  const int64_t heads = (int64_t)d.B * d.Z;
  for (int64_t h0 = 0; h0 < heads; h0 += pl.heads) {
    const int64_t nh = pl.heads < heads - h0 ? pl.heads : heads - h0;
    for (int64_t r0 = 0; r0 < d.Lq; r0 += pl.rows) {
      const int64_t nr = pl.rows < d.Lq - r0 ? pl.rows : d.Lq - r0;
      StripArgs a = group_args<T>(d, pl, ws, h0, r0, nr, Q, K, V);
      const int64_t q = (h0 * d.Lq + r0) * d.A, k = h0 * d.L * d.A;
      a.dO = static_cast<const T *>(dO) + q; a.O = static_cast<const T *>(O) + q;
      a.LSE_in = LSE + h0 * d.Lq + r0;
      RSA_TRY(launch_scores<T>(a, nh, d.A, true, st));
      const ApplyArgs p = {a.strip2, a.K, static_cast<T *>(dQ) + q, nullptr, nullptr};
      RSA_TRY((launch_apply<T, false>(a, p, nh, st)));
      CollectArgs c{};
      c.strip[0] = a.strip; c.Y[0] = a.dO; c.out[0] = static_cast<T *>(dV) + k; c.alpha[0] = 1.0f;
      c.strip[1] = a.strip2; c.Y[1] = a.Q; c.out[1] = static_cast<T *>(dK) + k; c.alpha[1] = d.scale;
      c.acc[0] = reinterpret_cast<float *>(ws + pl.acc_v); c.acc[1] = reinterpret_cast<float *>(ws + pl.acc_k);
      c.add = r0 > 0; c.keep = r0 + nr < d.Lq;
      RSA_TRY(launch_collect<T>(a, c, nh, st));
    }
  }
  return hipSuccess;
}
#undef RSA_TRY

}  // namespace

size_t strip_workspace_bytes(const Dims &d, int dtype, int pass) { return strip_plan(d, dtype, pass).total; }

hipError_t strip_forward(const Dims &d, int dtype, const void *Q, const void *K, const void *V, void *O, float *LSE,
                         void *ws, hipStream_t st) {
  char *w = static_cast<char *>(ws);
  return dtype == RSA_BF16 ? forward_t<uint16_t>(d, dtype, Q, K, V, O, LSE, w, st)
                           : forward_t<float>(d, dtype, Q, K, V, O, LSE, w, st);
}

hipError_t strip_backward(const Dims &d, int dtype, const void *dO, const void *Q, const void *K, const void *V,
                          const void *O, const float *LSE, void *dQ, void *dK, void *dV, void *ws, hipStream_t st) {
  char *w = static_cast<char *>(ws);
  return dtype == RSA_BF16 ? backward_t<uint16_t>(d, dtype, dO, Q, K, V, O, LSE, dQ, dK, dV, w, st)
                           : backward_t<float>(d, dtype, dO, Q, K, V, O, LSE, dQ, dK, dV, w, st);
}

}  // namespace rsa
