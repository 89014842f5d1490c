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
//              (where rows are many, in fp32 also where walks are short: both in one kernel, and no strip; see
//              f32_forward_kernel and bf16_one_pass)
//   backward   by rows  scores: P = exp(S - LSE), dS = P o (dO V^T - D), both tiles written in dtype
//                       apply:  dQ = s dS K;   collect: dV = P^T dO, dK = s dS^T Q
//              by keys  (bf16, where work-groups that own 128 keys fill the chip: plan_by_keys)
//                       collect: dV and dK from P and dS in registers, dS^T written;   apply: dQ = s dS K
//
// In fp32 the backward's P is brought to its rows' own sums instead of relying on the LSE it is given, whose
// rounding (2^-25 |LSE|) every probability of the row would share: the scores kernel leaves each tile's row sums,
// apply adds them and scales its rows, collect scales the strips' rows as it reads them.  No accumulator starts
// from a row term (the contraction would be rounded at that term's size), and the fp32 sums over keys or rows are
// formed 32 at a time.  Relative RMS error against fp64, 1e-7, dQ | dK | dV | O, N(0, 1) inputs:
// A64 L512 2.0 | 2.0 | 1.6 | 1.6 (with products by the fp32 matrix instruction 3.5 | 3.5 | 3.2 | 3.2, with row terms in the
// accumulators and one chain per sum besides 12.5 | 12.2 | 12.1 | 5.8; the chunk-by-chunk steps of rsa_staged.hip, N4,
// 3.9 | 3.8 | 3.5 | 3.6); Q and K of N(0, 16), scores of 60: 14.8 | 14.8 | 5.4 | 5.4 (fp32 instruction 35 | 36 | 14 | 14).
//
// Bytes per score: 2 es forward, 5 es backward, by keys 2 es (es: bytes of the dtype); every other operand is read
// from the caches.  The former version of this path kept S and dP as fp32 strips, softmaxed them in
// passes of their own and ran every product chunk by chunk: 12 (bf16) / 16 (fp32) bytes forward,
// 28 / 40 backward, and 10 N^2 launches (B8 Z16 L2048 N8 bf16, forward and backward: 8.9 ms; now 0.71,
// forward 0.16, dK and dV 0.36 with one work-group to a CU, dQ 0.18, its strip read at 6 TB/s.  B16 Z12 L512 N4 fp32: 1.99 ms; with fp32
// matrix instructions 0.49, 55 to 70 % of their rate; now 0.37, the backward's 1.0 GB of strips at 3.4 to 3.6 TB/s).
//
// The tile kernels hold bf16 tiles in the layout of the fused kernels; fp32 products run on the bf16 matrix instructions
// over numbers split in three (TileT<float>).  All products are formed transposed: one lane owns one row of the result.
#include "rsa_fused_tile.h"
#include "rsa_kernels.h"

#include <type_traits>

namespace rsa {
namespace {

// A 64 x 64 tile of T in LDS: how it is filled, read as MFMA operands and written as a result.
//   rows(t, rb, s):   operand whose row index runs over tile rows rb .. rb + 31, k over columns
//   cols(t, s, cb):   operand whose row index runs over columns 32 cb .. 32 cb + 31, k over rows
// s: k slice of kSliceK; mfma() contracts one slice.
template <typename T> struct TileT;

template <> struct TileT<uint16_t> {
  typedef bf16x8 Frag, Piece;
  static constexpr int kBytes = kTileBytes, kPieces = 4;
  TileLanes tl;
  __device__ __forceinline__ explicit TileT(int lane) : tl(lane) {}
  __device__ __forceinline__ Frag rows(const unsigned char *t, int rb, int s) const { return tl.read_rows(t, rb, s); }
  __device__ __forceinline__ Frag cols(const unsigned char *t, int s, int cb) const {
    const int flip = cb << 6;  // the second column block: the other four of a row's eight chunks
    const u32x2 lo = lds_read_tr16(t + s * 2048 + (tl.cols_off[0][0] ^ flip));
    const u32x2 hi = lds_read_tr16(t + s * 2048 + (tl.cols_off[0][1] ^ flip));
    const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(Frag, w);
  }
  static __device__ __forceinline__ f32x16 mfma(Frag a, Frag b, f32x16 c) { return mfma_32x32x16(a, b, c); }
  static __device__ __forceinline__ void mfma(Frag a, Frag b, f32x16 &c, f32x16 &) { c = mfma_32x32x16(a, b, c); }
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
  // slice i of a transposed 32-row block (c0: its columns 0 .. 31, c1: 32 .. 63) as an operand
  static __device__ __forceinline__ Piece piece(const f32x16 &c0, const f32x16 &c1, int i) {
    const f32x16 &c = i < 2 ? c0 : c1;
    const int v = (i & 1) * 8;
    const u32x4 w = {pack_bf16(c[v + 0], c[v + 1]), pack_bf16(c[v + 2], c[v + 3]), pack_bf16(c[v + 4], c[v + 5]),
                     pack_bf16(c[v + 6], c[v + 7])};
    return __builtin_bit_cast(Frag, w);
  }
  // column (of 32) of a tile that holds strip fragments -> key: a fragment's eight elements are keys
  // 4 half .. + 3 and 8 + 4 half .. + 3 of its slice
  static __device__ __forceinline__ int key_of_col(int c) { return (c & 16) | ((c & 4) << 1) | ((c >> 1) & 4) | (c & 3); }
  template <int WAVES = 4> struct DMA {
    TileDMAT<WAVES> d;
    static constexpr int PER = TileDMAT<WAVES>::PER;
    __device__ __forceinline__ DMA(int wave, int lane, int64_t ld) : d(wave, lane, (int)ld) {}
    __device__ __forceinline__ void load_unseen(const uint16_t *g, uint32_t t) const {
#pragma unroll
      for (int j = 0; j < PER; ++j) lds_dma16_unseen(g, d.g_off[j] * 2, t + d.l_off[j]);
    }
    __device__ __forceinline__ void load(const uint16_t *g, unsigned char *t) const { d.load(g, t); }
  };
};

// Eight fp32 numbers as sums of three bf16 each, x = h + m + l to the last bit (8 + 8 + 8 bits of 24, each rest rounded to
// nearest; bf16 has the exponents of fp32).  A product of two such sums without its three smallest terms,
//   h l' + l h' + m m' + h m' + m h' + h h',
// is off by 2^-26 at most and takes six bf16 MFMAs of 16 k, 192 cycles, where v_mfma_f32_32x32x2_f32 takes 512.  The sums
// over k are rounded less often: RMS error of 32 x 32 blocks over 64 | 256 k of N(0, 1) numbers 1.10 | 2.37e-7, by the fp32
// instruction 1.44 | 2.88.  h and m are held to finite numbers: bf16 would round the largest to infinity, and the
// remainders are formed by a product over a pair, where an infinity or NaN (which l alone carries) would reach the neighbour.
// bf16 has subnormals down to 2^-133, so numbers below 2^-110 are held to 2^-134 instead of 2^-24 of themselves (dO of N(0, 1)
// times 2^-100, 2^-110, 2^-116, 512 rows, dV: errors of 2.4e-7, 2.4e-7, 2.3e-6 of it; dK, whose dS is smaller: 2.7e-7, 1.4e-6, 8.5e-5).
// (The two medians of m: 2 of 11 vector instructions a pair, 385 -> 390 us for forward and backward of 192 heads of 512 rows.)
struct Split { bf16x8 h, m, l; };
// x less the low (high) half of a pair of bf16: exact, one instruction.  (The pairs (-1, 0) and (0, -1) come from registers:
// as literals the compiler makes inline constants of them, which the instruction reads as other pairs.)
struct Minus {
  uint32_t lo, hi;
  __device__ __forceinline__ Minus() : lo(0x0000bf80u), hi(0xbf800000u) { asm("" : "+s"(lo), "+s"(hi)); }
  __device__ __forceinline__ float operator()(float x, uint32_t pair, bool high) const {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, high ? hi : lo), x, false);
  }
};
template <bool ANY = true>  // false: numbers of at most 1, or NaN that every result of their neighbours is as well
__device__ __forceinline__ Split split8(f32x4 a, f32x4 b) {
  const Minus minus;
  u32x4 h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = e < 2 ? a[2 * e] : b[2 * e - 4], y = e < 2 ? a[2 * e + 1] : b[2 * e - 3];
    constexpr float kMost = 3.3895314e38f;  // (a median with NaN is the lesser of the other two)
    auto pack = [](float x, float y) __attribute__((always_inline)) {
      return ANY ? pack_bf16(__builtin_amdgcn_fmed3f(x, -kMost, kMost), __builtin_amdgcn_fmed3f(y, -kMost, kMost)) : pack_bf16(x, y);
    };
    h[e] = pack(x, y);
    const float rx = minus(x, h[e], false), ry = minus(y, h[e], true);
    m[e] = pack(rx, ry);
    l[e] = pack_bf16(minus(rx, m[e], false), minus(ry, m[e], true));
  }
  return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// fp32: a tile lies in LDS as three bf16 tiles (of PLANE bytes) of its numbers' parts, and is split on its way there from
// registers.
template <> struct TileT<float> {
  typedef Split Frag;
  typedef f32x4 Piece;
  static constexpr int kBytes = 3 * kTileBytes, kPieces = 8;
  TileT<uint16_t> tb;
  __device__ __forceinline__ explicit TileT(int lane) : tb(lane) {}
  template <int PLANE = kTileBytes>
  __device__ __forceinline__ Frag rows(const unsigned char *t, int rb, int s) const {
    return {tb.rows(t, rb, s), tb.rows(t + PLANE, rb, s), tb.rows(t + 2 * PLANE, rb, s)};
  }
  template <int PLANE = kTileBytes>
  __device__ __forceinline__ Frag cols(const unsigned char *t, int s, int cb) const {
    return {tb.cols(t, s, cb), tb.cols(t + PLANE, s, cb), tb.cols(t + 2 * PLANE, s, cb)};
  }
  static __device__ __forceinline__ f32x16 mfma(const Frag &a, const Frag &b, f32x16 c) {
    c = mfma_32x32x16(a.h, b.l, c);
    c = mfma_32x32x16(a.l, b.h, c);
    c = mfma_32x32x16(a.m, b.m, c);
    c = mfma_32x32x16(a.h, b.m, c);
    c = mfma_32x32x16(a.m, b.h, c);
    return mfma_32x32x16(a.h, b.h, c);
  }
  // with the small terms in an accumulator of their own: 0.50 | 0.89e-7 in the comparison above.  (Scores are formed so, in
  // both passes: at scores of 60 the backward's dQ errs 15e-7, with all terms in one accumulator 38, by the fp32 instruction 35.)
  static __device__ __forceinline__ void mfma(const Frag &a, const Frag &b, f32x16 &c, f32x16 &small) {
    small = mfma_32x32x16(a.h, b.l, small);
    small = mfma_32x32x16(a.l, b.h, small);
    small = mfma_32x32x16(a.m, b.m, small);
    small = mfma_32x32x16(a.h, b.m, small);
    small = mfma_32x32x16(a.m, b.h, small);
    c = mfma_32x32x16(a.h, b.h, c);
  }
  static __device__ __forceinline__ float dot(f32x4 a, f32x4 b, float acc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = fmaf(a[e], b[e], acc);
    return acc;
  }
  // results: rows of 256 bytes, chunk cc of row r at cc ^ rot(r) (free of bank conflicts for both accesses)
  static __device__ __forceinline__ int off(int r, int cc) {
    return r * 256 + ((cc ^ ((r & 3) | ((r >> 1) & 4) | ((r & 4) << 1))) << 4);
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
  static __device__ __forceinline__ Piece piece(const f32x16 &c0, const f32x16 &c1, int i) {
    const f32x16 &c = i < 4 ? c0 : c1;
    const int v = (i & 3) * 4;
    return f32x4{c[v], c[v + 1], c[v + 2], c[v + 3]};
  }
  static __device__ __forceinline__ int key_of_col(int c) { return c; }
  // ROWS x 64 numbers of a matrix, from memory to registers (fetch) and from there, split, to LDS (put).
  // STRIP: instead, 32 rows of the CHUNKS chunks of eight keys from chunk `first` on of a strip tile (below), where a row's
  // chunk is two pieces 32 lanes apart.
  template <int ROWS, int WAVES, bool STRIP = false, int CHUNKS = 8> struct Tile {
    static constexpr int PER = ROWS * CHUNKS / (64 * WAVES);
    static_assert(!STRIP || ROWS == 32, "a block of a strip tile");
    uint32_t g_off[PER];  // bytes
    int l_off[PER];
    f32x4 r[PER][2];
    __device__ __forceinline__ Tile(int wave, int lane, int64_t ld, int first = 0) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int p = (wave * PER + j) * 64 + lane;
        const int row = STRIP ? p & 31 : p >> 3, cc = STRIP ? (p >> 5) + first : p & 7;
        g_off[j] = 4 * (uint32_t)(STRIP ? cc * 256 + row * 4 : row * (int)ld + cc * 8);
        l_off[j] = tile_off(row, cc);
      }
    }
    __device__ __forceinline__ void fetch(const float *g) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const char *p = reinterpret_cast<const char *>(g) + g_off[j];
        r[j][0] = *reinterpret_cast<const f32x4 *>(p);
        r[j][1] = *reinterpret_cast<const f32x4 *>(p + (STRIP ? 512 : 16));
      }
    }
    __device__ __forceinline__ void put(unsigned char *t, float factor = 1.f) const {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const Split x = STRIP ? split8(r[j][0] * factor, r[j][1] * factor) : split8(r[j][0], r[j][1]);
        *reinterpret_cast<bf16x8 *>(t + l_off[j]) = x.h;
        *reinterpret_cast<bf16x8 *>(t + ROWS * 128 + l_off[j]) = x.m;
        *reinterpret_cast<bf16x8 *>(t + 2 * ROWS * 128 + l_off[j]) = x.l;
      }
    }
  };
};
constexpr int kSlices = 4, kSliceK = 16;  // of a 64 x 64 tile's contraction

// How a strip lies in memory: 64 x 64 tiles, a head's tiles row tile by row tile; inside a tile its two blocks of
// 32 rows, and of a block the operand fragments in which the scores kernels hold it and the apply
// kernel wants it: [slice][lane][16 bytes].  A wave writes and reads a block as contiguous KiBs.
template <typename T> __device__ __forceinline__ int64_t strip_tile(int64_t head, int64_t rtiles64, int64_t rt, int64_t ktiles, int64_t kt) {
  return ((head * rtiles64 + rt) * ktiles + kt) * 4096;
}
// A wave's block of 32 rows, held transposed in c0, c1, into its place in the strip.
template <typename T>
__device__ __forceinline__ void strip_store(T *block, const f32x16 &c0, const f32x16 &c1, int lane) {
  typedef TileT<T> TT;
#pragma unroll
  for (int i = 0; i < TT::kPieces; ++i)
    *reinterpret_cast<typename TT::Piece *>(block + (i * 64 + lane) * (16 / (int)sizeof(T))) = TT::piece(c0, c1, i);
}
// Direct load of a bf16 strip tile into LDS as rows of 16-byte chunks (chunk 2 i + h of row r: the fragment of
// slice i that lane (r, h) holds), swizzled like every tile.
template <int WAVES> struct StripDMA {
  static constexpr int PER = kTileBytes / (1024 * WAVES);
  int g_off[PER], l_off[PER];
  __device__ __forceinline__ StripDMA(int wave, int lane) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int p = (wave * PER + j) * 64 + lane, row = p >> 3, cc = (p & 7) ^ swz_rot(row);
      g_off[j] = (row >> 5) * 2048 + ((cc >> 1) * 64 + (row & 31) + (cc & 1) * 32) * 8;
      l_off[j] = (wave * PER + j) * 1024;
    }
  }
  __device__ __forceinline__ void load_unseen(const uint16_t *tile, uint32_t t) const {
#pragma unroll
    for (int j = 0; j < PER; ++j) lds_dma16_unseen(tile, g_off[j] * 2, t + l_off[j]);
  }
};

// fp32 strips hold P to a factor per row (see on top).
template <typename T> constexpr bool kOwnSum = sizeof(T) == 4;

struct StripArgs {
  const void *Q, *K, *V, *dO, *O;  // first head of the group; Q, dO, O: first row of the group
  const float *LSE_in;
  float *LSE;                      // (head, Lq), first row of the group
  void *strip, *strip2;            // (head, rows, L) in tiles: exp(S - m_t) or P; dS
  float *stats;                    // forward: (head, L / 64, rows, 2), m_t and l_t, base-2 logarithm domain;
                                   // fp32 backward: (head, L / 64, rows), the tile's part of a row's sum
  int64_t L, Lq, rows, q0;         // rows of the group; token of its first row
  int A, causal, rtiles, kblocks, per;  // 128-row tiles; key blocks of `per` tiles
  float cl2, scale, inv_scale;
};

// Group of 64 rows that a wave's 32 rows belong to: a strip tile (64 rows x 64 keys) is written, and read,
// when its first key is visible to the last of its rows.
__device__ __forceinline__ bool tile_seen(const StripArgs &a, int64_t row, int64_t k0) {
  return !a.causal || k0 <= a.q0 + (row | 63);
}

// n slices of a contraction: the operands of slice i + 1 are read from LDS while slice i is on the matrix pipe
// (left to itself the compiler reads most of them right before their use).
template <int N, typename Read, typename Use>
__device__ __forceinline__ void pipelined(Read read, Use use) {
  read(0, 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + 1 < N) {
      read(i + 1, (i + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    use(i, i & 1);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ---------------------------------------------------------------- scores ----
// Work-group: 128 rows (wave: 32, their Q, and dO, as B operands in registers) walking `per` tiles of 64
// keys.  One LDS buffer: the next tile is requested as soon as every wave has the products of this one, so
// that its latency lies under this tile's exponentials and stores; two to four work-groups share a compute
// unit.  (With one tile pair per work-group, loads, products and stores of the work-groups of a unit ran in
// step, one after the other: the matrix pipe was busy 46 % in fp32.)
// The wait at a tile's end is for the next tile's loads alone, and its barrier for LDS alone: this tile's strip stores stay
// in flight (B8 Z16 L2048 bf16, forward and backward: 1657 -> 1641 us).
template <typename T, int AH, int NT>  // NT: tiles per key block (K, or K and V)
struct ScoreLds {
  unsigned char t[NT][AH][TileT<T>::kBytes];
};

// Position of a work-group in the grid of a scores kernel.
struct ScorePos {
  int64_t head, row0;
  int t0, t1;  // key tiles
  __device__ __forceinline__ explicit ScorePos(const StripArgs &a) {
    const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t hr = wg / (uint32_t)a.kblocks;
    head = hr / (uint32_t)a.rtiles;
    row0 = (int64_t)(hr % (uint32_t)a.rtiles) * 128;
    t0 = (int)(wg % (uint32_t)a.kblocks) * a.per;
    int n = (int)(a.L / 64);
    if (a.causal) {
      const int64_t row_last = (row0 + 128 < a.rows ? row0 + 128 : a.rows) - 1;
      const int64_t seen = (a.q0 + row_last) / 64 + 1;
      if (seen < n) n = (int)seen;
    }
    t1 = t0 + a.per < n ? t0 + a.per : n;
  }
};

// Scores of keys that the lane's row does not see: -inf.
__device__ __forceinline__ void mask_scores(const StripArgs &a, int64_t wrow, int64_t k0, int lane, f32x16 (&s)[2]) {
  if (!a.causal || k0 + 63 <= a.q0 + wrow) return;
  const int64_t d64 = a.q0 + wrow + (lane & 31) - k0 - (lane >> 5) * 4;  // last visible key, relative to the tile
  const int dlast = d64 > 64 ? 64 : (int)d64;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (kb * 32 + (v >> 2) * 8 + (v & 3) > dlast) s[kb][v] = -INFINITY;
}

// A work-group's rows of a matrix (wave: 32, lane: one) as B operands, from their fp32 pieces or as they are.
template <typename T, int AH> struct RowFrags {
  typedef TileT<T> TT;
  static constexpr bool kSplitNow = sizeof(T) == 4 && AH > 2;  // (no registers for the parts of wider heads: split at use)
  typename TT::Frag f[kSplitNow ? 1 : AH * kSlices];
  f32x4 raw[kSplitNow ? AH * kSlices * 2 : 1];
  // p: the lane's row, at element 8 half.  O: the same place in another matrix, whose dot product with the row is added to acc.
  template <bool DOT> __device__ __forceinline__ void load(const T *p, const T *O, float &acc) {
#pragma unroll
    for (int i = 0; i < AH * kSlices; ++i) {
      if constexpr (sizeof(T) == 2) {
        f[i] = *reinterpret_cast<const bf16x8 *>(p + i * kSliceK);
        if (DOT) acc = TT::dot(f[i], *reinterpret_cast<const bf16x8 *>(O + i * kSliceK), acc);
      } else {
        const f32x4 *x = reinterpret_cast<const f32x4 *>(p + i * kSliceK), *y = reinterpret_cast<const f32x4 *>(O + i * kSliceK);
        const f32x4 a = x[0], b = x[1];
        if (DOT) acc = TT::dot(b, y[1], TT::dot(a, y[0], acc));
        if constexpr (kSplitNow) { raw[2 * i] = a; raw[2 * i + 1] = b; }
        else f[i] = split8(a, b);
      }
    }
  }
  __device__ __forceinline__ typename TT::Frag get(int i) const {
    if constexpr (kSplitNow) return split8(raw[2 * i], raw[2 * i + 1]);
    else return f[i];
  }
};

// The key tiles of a scores kernel on their way to its one LDS buffer: bf16 by direct loads, fp32 through registers, which
// hold the tile after the requested one where there are enough (HOLD).
template <typename T, int AH, bool HOLD> struct KeyTiles;
template <int AH, bool HOLD> struct KeyTiles<uint16_t, AH, HOLD> {
  typename TileT<uint16_t>::template DMA<> dma;
  __device__ __forceinline__ KeyTiles(int wave, int lane, int64_t ld) : dma(wave, lane, ld) {}
  __device__ __forceinline__ void ask(const uint16_t *) {}
  __device__ __forceinline__ void bring(const uint16_t *g, unsigned char (*t)[kTileBytes]) {
#pragma unroll
    for (int ah = 0; ah < AH; ++ah) dma.load(g + ah * 64, t[ah]);
  }
};
template <int AH, bool HOLD> struct KeyTiles<float, AH, HOLD> {
  typename TileT<float>::template Tile<64, 4> tile;
  f32x4 held[HOLD ? AH - 1 : 0][2][2];
  __device__ __forceinline__ KeyTiles(int wave, int lane, int64_t ld) : tile(wave, lane, ld) {}
  __device__ __forceinline__ void ask(const float *g) {
    if constexpr (HOLD) {
#pragma unroll
      for (int ah = AH - 1; ah >= 0; --ah) {
        tile.fetch(g + ah * 64);
        if (ah > 0) {
#pragma unroll
          for (int j = 0; j < 2; ++j) { held[ah - 1][j][0] = tile.r[j][0]; held[ah - 1][j][1] = tile.r[j][1]; }
        }
      }
    }
  }
  __device__ __forceinline__ void bring(const float *g, unsigned char (*t)[TileT<float>::kBytes]) {
#pragma unroll
    for (int ah = 0; ah < AH; ++ah) {
      if constexpr (!HOLD) tile.fetch(g + ah * 64);
      else if (ah > 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) { tile.r[j][0] = held[ah - 1][j][0]; tile.r[j][1] = held[ah - 1][j][1]; }
      }
      tile.put(t[ah]);
    }
  }
};

template <typename T, int AH>
__global__ void __launch_bounds__(256, AH <= 2 ? (sizeof(T) * AH == 4 ? 3 : 2) : 1) strip_scores_fwd_kernel(StripArgs a) {
  typedef TileT<T> TT;
  constexpr int NS = kSlices;
  __shared__ __attribute__((aligned(16))) ScoreLds<T, AH, 1> lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const ScorePos pos(a);
  if (pos.t0 >= pos.t1) return;

  const T *Kh = static_cast<const T *>(a.K) + pos.head * a.L * a.A;
  auto at = [&](int t) { return Kh + (int64_t)t * 64 * a.A; };
  KeyTiles<T, AH, true> keys(wave, lane, a.A);
  keys.ask(at(pos.t0));
  keys.bring(at(pos.t0), lds.t[0]);
  if (pos.t0 + 1 < pos.t1) keys.ask(at(pos.t0 + 1));
  const int64_t wrow = pos.row0 + wave * 32;  // (rows come in multiples of 64: a wave's rows are there or not)
  const bool rows_here = wrow < a.rows;
  RowFrags<T, AH> q;
  if (rows_here) {
    const T *qp = static_cast<const T *>(a.Q) + (pos.head * a.Lq + wrow + col) * a.A + half * (kSliceK / 2);
    float none;
    q.template load<false>(qp, qp, none);
  }
  const TT tt(lane);
  if (sizeof(T) == 2) wait_vmem();
  barrier_lds();
  for (int t = pos.t0; t < pos.t1; ++t) {
    const int64_t k0 = (int64_t)t * 64;
    const bool work = rows_here && tile_seen(a, wrow, k0);
    f32x16 s[2];
    if (work) {
      f32x16 rest[2];  // fp32: the small terms' own sums (the row's LSE, sum and all, then errs less than with fp32 products)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) { s[kb][v] = 0.f; rest[kb][v] = 0.f; }
      // (a step: both 32-key blocks of a slice; fp32, whose operands are three times the registers: one of them)
      constexpr int KB = sizeof(T) == 4 ? 1 : 2, ST = 2 / KB;
      typename TT::Frag kf[2][KB];
      pipelined<AH * NS * ST>(
          [&](int u, int b) __attribute__((always_inline)) {
            const int i = u / ST;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) kf[b][kb] = tt.rows(lds.t[0][i / NS], (u % ST + kb) * 32, i % NS);
          },
          [&](int u, int b) __attribute__((always_inline)) {
            const typename TT::Frag qf = q.get(u / ST);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) TT::mfma(kf[b][kb], qf, s[u % ST + kb], rest[u % ST + kb]);
          });
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) s[kb][v] += rest[kb][v];
      }
    }
    barrier_lds();
    if (t + 1 < pos.t1) {
      keys.bring(at(t + 1), lds.t[0]);
      if (t + 2 < pos.t1) keys.ask(at(t + 2));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (work) {
      mask_scores(a, wrow, k0, lane, s);
      float m = s[0][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) m = fmaxf(m, s[0][v]);
#pragma unroll
      for (int v = 0; v < 16; ++v) m = fmaxf(m, s[1][v]);
      m = xhalf_max(m);
      const float mc = m > -INFINITY ? m * a.cl2 : 0.f;  // a row that sees none of these keys: all zeros
      float l[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          s[kb][v] = __builtin_amdgcn_exp2f(fmaf(s[kb][v], a.cl2, -mc));
          l[v & 3] += s[kb][v];
        }
      const float sum = xhalf_sum((l[0] + l[1]) + (l[2] + l[3]));
      if (half == 0) {
        f32x2 p = {m > -INFINITY ? mc : -INFINITY, sum};
        *reinterpret_cast<f32x2 *>(a.stats + ((pos.head * (a.L / 64) + t) * a.rows + wrow + col) * 2) = p;
      }
      strip_store(static_cast<T *>(a.strip) + strip_tile<T>(pos.head, a.rows / 64, wrow / 64, a.L / 64, t) +
                      (wave & 1) * 2048, s[0], s[1], lane);
      if (sizeof(T) == 2) wait_loads_before_stores<TT::kPieces>();
    } else if (sizeof(T) == 2) {
      wait_vmem();
    }
    barrier_lds();
  }
}

template <typename T, int AH>
__global__ void __launch_bounds__(256, sizeof(T) * AH <= 4 ? 2 : 1) strip_scores_bwd_kernel(StripArgs a) {
  typedef TileT<T> TT;
  constexpr int NS = kSlices;
  constexpr bool F = sizeof(T) == 4;
  constexpr bool ONE = sizeof(T) * AH == 16;  // fp32 heads of 256: K and V tiles take turns in LDS
  __shared__ __attribute__((aligned(16))) ScoreLds<T, AH, ONE ? 1 : 2> lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const ScorePos pos(a);
  if (pos.t0 >= pos.t1) return;

  const T *Kh = static_cast<const T *>(a.K) + pos.head * a.L * a.A;
  const T *Vh = static_cast<const T *>(a.V) + pos.head * a.L * a.A;
  KeyTiles<T, AH, true> keys(wave, lane, a.A);
  KeyTiles<T, AH, (AH <= 2)> vals(wave, lane, a.A);
  auto ask = [&](int t) __attribute__((always_inline)) {
    keys.ask(Kh + (int64_t)t * 64 * a.A);
    vals.ask(Vh + (int64_t)t * 64 * a.A);
  };
  auto bring = [&](int t) __attribute__((always_inline)) {
    keys.bring(Kh + (int64_t)t * 64 * a.A, lds.t[0]);
    if (!ONE) vals.bring(Vh + (int64_t)t * 64 * a.A, lds.t[ONE ? 0 : 1]);
  };
  ask(pos.t0);
  bring(pos.t0);
  if (pos.t0 + 1 < pos.t1) {
    if (ONE) keys.ask(Kh + (int64_t)(pos.t0 + 1) * 64 * a.A);
    else ask(pos.t0 + 1);
  }
  const int64_t wrow = pos.row0 + wave * 32;
  const bool rows_here = wrow < a.rows;
  RowFrags<T, AH> q, g;
  // bf16: -LSE / scale and -D of the lane's row, which the accumulators start from.  fp32: the reference of the row's
  // exponents, LSE less the logarithm of a power of two that brings likely scores near it (any value near LSE will
  // do; an exponent is rounded at its own size.  Scores beyond about 1e8 would leave its range), and D.
  float nl = 0.f, nd = 0.f;
  if (rows_here) {
    const int64_t off = (pos.head * a.Lq + wrow + col) * a.A + half * (kSliceK / 2);
    const T *gp = static_cast<const T *>(a.dO) + off;
    float acc = 0.f;
    q.template load<false>(static_cast<const T *>(a.Q) + off, gp, acc);
    g.template load<true>(gp, static_cast<const T *>(a.O) + off, acc);
    nd = -xhalf_sum(acc);
    const float lse = a.LSE_in[pos.head * a.Lq + wrow + col];
    if constexpr (kOwnSum<T>) {
      const float lse2 = lse * kLog2e;
      nl = fminf(fmaxf(rintf(lse2), 0.f), (float)(63 - __builtin_clzll((uint64_t)a.L))) - lse2;
    } else {
      nl = -lse * a.inv_scale;
    }
  }
  const TT tt(lane);
  if (sizeof(T) == 2) wait_vmem();
  barrier_lds();
  for (int t = pos.t0; t < pos.t1; ++t) {
    const int64_t k0 = (int64_t)t * 64;
    const bool work = rows_here && tile_seen(a, wrow, k0);
    f32x16 s[2], dp[2], rest[F ? 2 : 1];  // (rest: see the forward)
    if (work) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          s[kb][v] = kOwnSum<T> ? 0.f : nl; dp[kb][v] = kOwnSum<T> ? 0.f : nd;
          rest[F ? kb : 0][v] = 0.f;
        }
    }
    constexpr int KB = sizeof(T) == 4 ? 1 : 2, ST = 2 / KB;  // (see the forward)
    auto products = [&](auto K, auto V) __attribute__((always_inline)) {
      typename TT::Frag kf[2][KB], vf[2][KB];
      pipelined<AH * NS * ST>(
          [&](int u, int b) __attribute__((always_inline)) {
            const int i = u / ST;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
              if (K) kf[b][kb] = tt.rows(lds.t[0][i / NS], (u % ST + kb) * 32, i % NS);
              if (V) vf[b][kb] = tt.rows(lds.t[ONE ? 0 : 1][i / NS], (u % ST + kb) * 32, i % NS);
            }
          },
          [&](int u, int b) __attribute__((always_inline)) {
            typename TT::Frag qf, gf;
            if (K) qf = q.get(u / ST);
            if (V) gf = g.get(u / ST);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
              if (K) TT::mfma(kf[b][kb], qf, s[u % ST + kb], rest[F ? u % ST + kb : 0]);
              if (V) dp[u % ST + kb] = TT::mfma(vf[b][kb], gf, dp[u % ST + kb]);
            }
          });
    };
    if (work) products(std::true_type{}, std::integral_constant<bool, !F>{});
    if constexpr (F) {  // (S first, and its sums made one, so that their second set of registers is free for dP)
      if (work) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) s[kb][v] += rest[kb][v];
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (ONE) {
        barrier_lds();
        vals.bring(Vh + (int64_t)t * 64 * a.A, lds.t[0]);
        barrier_lds();
      }
      if (work) products(std::false_type{}, std::true_type{});
    }
    barrier_lds();
    if (t + 1 < pos.t1) {
      bring(t + 1);
      if (t + 2 < pos.t1) {
        if (ONE) keys.ask(Kh + (int64_t)(t + 2) * 64 * a.A);
        else ask(t + 2);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (work) {
      mask_scores(a, wrow, k0, lane, s);
      if constexpr (kOwnSum<T>) {
        float l[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            s[kb][v] = __builtin_amdgcn_exp2f(fmaf(s[kb][v], a.cl2, nl));
            dp[kb][v] = (dp[kb][v] + nd) * s[kb][v];
            l[v & 3] += s[kb][v];
          }
        const float sum = xhalf_sum((l[0] + l[1]) + (l[2] + l[3]));
        if (half == 0) a.stats[(pos.head * (a.L / 64) + t) * a.rows + wrow + col] = sum;
      } else {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            s[kb][v] = __builtin_amdgcn_exp2f(s[kb][v] * a.cl2);
            dp[kb][v] *= s[kb][v];
          }
      }
      const int64_t o = strip_tile<T>(pos.head, a.rows / 64, wrow / 64, a.L / 64, t) + (wave & 1) * 2048;
      strip_store(static_cast<T *>(a.strip) + o, s[0], s[1], lane);
      strip_store(static_cast<T *>(a.strip2) + o, dp[0], dp[1], lane);
      if (sizeof(T) == 2) wait_loads_before_stores<2 * TT::kPieces>();
    } else if (sizeof(T) == 2) {
      wait_vmem();
    }
    barrier_lds();
  }
}

// ----------------------------------------------------------------- apply ----
// out (row, A) = scale * sum over keys of strip(row, key) X(key, A).  Work-group: 128 rows (wave: 32) x
// 64 AHW columns, walking the key tiles; X tiles reach LDS by direct loads, the wave's strip fragments
// its registers, a tile ahead of their use; one barrier per tile.  A tile's product is formed by itself and then
// added, where it is weighted or fp32 (see on top).  WEIGHT (forward): the strip is exp(S - m_t); the weights
// exp(m_t - max m_t) bring the tiles to one reference, and the row's sum of weighted l_t normalises it and gives LSE.
// fp32 backward: the sum of the tiles' l_t does, and 1 / sum is left for collect.
struct ApplyArgs {
  const void *strip, *X;
  void *out;
  float *LSE;   // forward
  float *norm;  // fp32 backward: (head, rows)
};

// The tiles of X on their way to LDS.
template <typename T, int WAVES> struct XTile;
template <int WAVES> struct XTile<uint16_t, WAVES> { typedef typename TileT<uint16_t>::template DMA<WAVES> type; };
template <int WAVES> struct XTile<float, WAVES> { typedef typename TileT<float>::template Tile<64, WAVES> type; };
// RW waves share the work-group's rows, 32 each; KS groups of such waves share the key tiles, group g taking every
// KS-th, and their sums are added in LDS.
template <typename T, int AHW, bool WEIGHT, int RW, int KS>
__global__ void __launch_bounds__(64 * RW * KS, KS > 1 ? 1 : (AHW == 1 ? 3 : 2)) strip_apply_kernel(StripArgs a, ApplyArgs p) {
  typedef TileT<T> TT;
  constexpr int NS = kSlices, NP = TT::kPieces, BM = 32 * RW;
  constexpr bool F = sizeof(T) == 4;
  static_assert(!F || AHW == 1, "fp32: 64 columns");
  struct Stage { unsigned char X[AHW][TT::kBytes]; };
  // bf16: two stage buffers, separate objects (see the fused kernels); fp32: one, and the results' staging
  constexpr int kBuf = KS * (int)sizeof(Stage), kOut = RW * 8192;
  __shared__ __attribute__((aligned(16))) unsigned char buf0[F && kOut > kBuf ? kOut : kBuf], buf1[F ? 16 : kBuf];
  Stage *const st0 = reinterpret_cast<Stage *>(buf0), *const st1 = F ? st0 : reinterpret_cast<Stage *>(buf1);
  __shared__ float sums[KS == 1 ? 1 : KS][RW][2][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % RW;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / RW;
  const int col = lane & 31, half = lane >> 5;
  const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t cblocks = (uint32_t)(a.A / (64 * AHW));
  const int a0 = (int)(wg % cblocks) * (64 * AHW);
  const uint32_t hr = wg / cblocks;
  // under the causal mask later rows see more keys: the long work-groups start first
  const uint32_t rt = hr % (uint32_t)a.rtiles;
  const int64_t head = hr / (uint32_t)a.rtiles, row0 = (int64_t)(a.causal ? a.rtiles - 1 - rt : rt) * BM;
  const int64_t row_last = (row0 + BM < a.rows ? row0 + BM : a.rows) - 1;
  const int ntiles = (int)(a.L / 64);
  int nt = ntiles;
  if (a.causal && (a.q0 + row_last) / 64 + 1 < nt) nt = (int)((a.q0 + row_last) / 64) + 1;

  const int64_t wrow = row0 + wave * 32;
  const bool rows_here = wrow < a.rows;
  const int64_t rrow = rows_here ? wrow : row0;  // (a wave without rows reads the first wave's)
  const T *S = static_cast<const T *>(p.strip) + strip_tile<T>(head, a.rows / 64, rrow / 64, ntiles, 0) +
               (RW == 1 ? (int)(rrow >> 5) & 1 : wave & 1) * 2048;
  const T *Xh = static_cast<const T *>(p.X) + head * a.L * a.A + a0;
  typename XTile<T, RW>::type x_tile(wave, lane, a.A);
  typename TT::Piece s0[NP], s1[F ? 1 : NP];  // (fp32: a piece is fetched for the next tile as soon as it is used)
  constexpr bool kStats = WEIGHT || kOwnSum<T>;
  constexpr int kPer = WEIGHT ? 2 : 1;  // numbers per row and tile
  const float *stats = a.stats + ((head * ntiles) * a.rows + rrow) * kPer;  // (read at col)
  f32x2 ml0 = {0.f, 0.f}, ml1 = {0.f, 0.f};  // m_t (forward) and l_t of the lane's row
  auto piece = [&](int t, int i) __attribute__((always_inline)) {
    return *reinterpret_cast<const typename TT::Piece *>(reinterpret_cast<const char *>(S + (int64_t)t * 4096 + i * (1024 / (int)sizeof(T))) + (uint32_t)lane * 16);
  };
  auto load = [&](int t, Stage &st, auto &s, f32x2 &ml, auto pieces) __attribute__((always_inline)) {
    const float *p = stats + (int64_t)t * a.rows * kPer;
    if constexpr (WEIGHT) ml = reinterpret_cast<const f32x2 *>(p)[col];
    else if constexpr (kStats) ml[1] = p[col];
    if constexpr (!F) {
#pragma unroll
      for (int ah = 0; ah < AHW; ++ah) x_tile.load(Xh + (int64_t)t * 64 * a.A + ah * 64, st.X[ah]);
    }
    if constexpr (pieces) {
#pragma unroll
      for (int i = 0; i < NP; ++i) s[i] = piece(t, i);
    }
  };
  auto fetch_x = [&](int t) __attribute__((always_inline)) {  // fp32: to registers, a tile ahead of the strip's
    if constexpr (F) { if (t < nt) x_tile.fetch(Xh + (int64_t)t * 64 * a.A); }
  };
  auto put_x = [&](int t) __attribute__((always_inline)) {
    if constexpr (F) { if (t < nt) x_tile.put(st0[grp].X[0]); }
  };
  int t = grp;  // this group's tile
  fetch_x(t);
  if (KS == 1 || t < nt) load(t, st0[grp], s0, ml0, std::true_type{});
  put_x(t);
  fetch_x(t + KS);

  float M = -INFINITY;  // the row's largest m_t
  if (WEIGHT) {
    // the two lane halves take every other tile of their row, eight at a time, their loads in flight together
    const int seen = a.causal ? (int)((a.q0 + (rrow | 63)) / 64) + 1 : ntiles;
    const int n = seen < ntiles ? seen : ntiles;
    for (int t0 = half; t0 < n; t0 += 16) {
      float m[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = t0 + 2 * j < n ? t0 + 2 * j : t0;
        m[j] = stats[((int64_t)t * a.rows + col) * 2];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) M = fmaxf(M, m[j]);
    }
    M = xhalf_max(M);  // finite: every row sees some key
  }
  float l = 0.f, l_err = 0.f;  // the row's sum, and what its additions have lost so far
  const TT tt(lane);
  f32x16 o[2 * AHW];
#pragma unroll
  for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;

  wait_vmem();
#pragma unroll
  for (int i = 0; i < NP; ++i) asm volatile("" : "+v"(s0[i]));  // (keeps the first loads in front of this wait)
  asm volatile("" : "+v"(ml0));
  __syncthreads();
  auto step = [&](Stage &cur, auto &sc, f32x2 ml, Stage &nxt, auto &sn, f32x2 &mln) __attribute__((always_inline)) {
    if (t + KS < nt) load(t + KS, nxt, sn, mln, std::integral_constant<bool, !F>{});
    if (rows_here && (KS == 1 || t < nt) && tile_seen(a, wrow, (int64_t)t * 64)) {
      const float w = WEIGHT ? __builtin_amdgcn_exp2f(ml[0] - M) : 1.f;
      if constexpr (kStats) {
        const float x = fmaf(w, ml[1], -l_err), sum = l + x;
        l_err = (sum - l) - x;
        l = sum;
      }
      auto add = [&](f32x16 &sum, const f32x16 &c) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] = WEIGHT ? fmaf(w, c[v], sum[v]) : sum[v] + c[v];
      };
      if constexpr (F) {  // 32 keys at a time (LDS reads are hidden by the other waves: three fit a SIMD without a second set)
        f32x16 c[2];
        const int tn = t + KS < nt ? t + KS : t;  // (after the last tile: refetched, not used)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const typename TT::Frag pf = split8<!WEIGHT>(sc[2 * s], sc[2 * s + 1]);
          sc[2 * s] = piece(tn, 2 * s);
          sc[2 * s + 1] = piece(tn, 2 * s + 1);
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            if (s % 2 == 0) {
#pragma unroll
              for (int v = 0; v < 16; ++v) c[db][v] = 0.f;
            }
            c[db] = TT::mfma(tt.cols(cur.X[0], s, db), pf, c[db]);
            if (s % 2 == 1) add(o[db], c[db]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
        f32x16 c[WEIGHT ? 2 * AHW : 1];
        if constexpr (WEIGHT) {
#pragma unroll
          for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) c[db][v] = 0.f;
        }
        typename TT::Frag xf[2][2 * AHW];
        pipelined<NS>(
            [&](int s, int b) __attribute__((always_inline)) {
#pragma unroll
              for (int db = 0; db < 2 * AHW; ++db) xf[b][db] = tt.cols(cur.X[db >> 1], s, db & 1);
            },
            [&](int s, int b) __attribute__((always_inline)) {
#pragma unroll
              for (int db = 0; db < 2 * AHW; ++db) {
                f32x16 &acc = WEIGHT ? c[WEIGHT ? db : 0] : o[db];
                acc = TT::mfma(xf[b][db], sc[s], acc);
              }
            });
        if constexpr (WEIGHT) {
#pragma unroll
          for (int db = 0; db < 2 * AHW; ++db) add(o[db], c[db]);
        }
      }
    }
    if constexpr (F) {
      barrier_lds();
      put_x(t + KS);
      fetch_x(t + 2 * KS);
      barrier_lds();
    } else {
      wait_vmem();
      __syncthreads();
    }
    t += KS;
  };
  while (t - grp < nt) {
    step(st0[grp], s0, ml0, st1[grp], s1, ml1);
    if (t - grp >= nt) break;
    if constexpr (F) step(st0[grp], s0, ml1, st0[grp], s1, ml0);
    else step(st1[grp], s1, ml1, st0[grp], s0, ml0);
  }
  if constexpr (KS > 1) {
    // the groups' sums: bf16 in the second buffers, fp32 behind the epilogue's tiles
    static_assert(RW <= 2 && (F ? kBuf - 16384 : kBuf) >= (KS - 1) * RW * 2 * AHW * 4096, "room for the groups' sums");
    auto slot = [&](int g, int db) {
      return reinterpret_cast<f32x4 *>((F ? buf0 + 16384 : buf1) + (((g - 1) * RW + wave) * 2 * AHW + db) * 4096);
    };
    if (grp > 0) {
#pragma unroll
      for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) slot(grp, db)[g * 64 + lane] = f32x4{o[db][g * 4], o[db][g * 4 + 1], o[db][g * 4 + 2], o[db][g * 4 + 3]};
      sums[grp][wave][0][lane] = l; sums[grp][wave][1][lane] = l_err;
    }
    __syncthreads();
    if (grp > 0) return;
    for (int q = 1; q < KS; ++q) {
#pragma unroll
      for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 x = slot(q, db)[g * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[db][g * 4 + e] += x[e];
        }
      const float x = sums[q][wave][0][lane] - l_err, sum = l + x;
      l_err = ((sum - l) - x) + sums[q][wave][1][lane];
      l = sum;
    }
    l -= l_err;
  }
  if (!rows_here) return;
  const float norm = kStats ? 1.0f / l : 1.0f;
  if (half == 0 && a0 == 0) {
    if (WEIGHT) p.LSE[head * a.Lq + wrow + col] = fmaf(M, kLn2, logf(l));
    else if (kStats) p.norm[head * a.rows + wrow + col] = norm;
  }
  unsigned char *ot = F ? buf0 + wave * 8192 : (wave < 2 ? buf0 : buf1) + (wave & 1) * 4096;  // (free after the last barrier)
  T *out = static_cast<T *>(p.out) + (head * a.Lq + wrow) * a.A + a0;
#pragma unroll
  for (int ah = 0; ah < AHW; ++ah) {
    TT::stage(ot, o[2 * ah], o[2 * ah + 1], WEIGHT ? norm : a.scale * norm, lane);
    TT::flush(ot, out + ah * 64, 32, lane, a.A);
  }
}

// groups 1 .. QS - 1 leave their sums in LDS behind the first 16 KiB, which the epilogue takes, and group 0 adds them;
// false: the wave is done
template <int WK, int QS, int DB>
__device__ __forceinline__ bool add_groups(unsigned char *lds, f32x16 (&o)[DB], int grp, int wave, int lane) {
  auto slot = [&](int g, int db) { return reinterpret_cast<f32x4 *>(lds + 16384 + (((g - 1) * WK + wave) * DB + db) * 4096); };
  if (grp > 0) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) slot(grp, db)[g * 64 + lane] = f32x4{o[db][g * 4], o[db][g * 4 + 1], o[db][g * 4 + 2], o[db][g * 4 + 3]};
  }
  barrier_lds();
  if (grp > 0) return false;
  for (int q = 1; q < QS; ++q)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 x = slot(q, db)[g * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][g * 4 + e] += x[e];
      }
  return true;
}
// ------------------------------------------------- fp32 forward, one pass ----
// fp32 heads of 64: a step's 32 keys are scored, softmaxed and applied to V in registers, without the strip (whose write
// and read took as long as the products do now).  Work-group: as in apply; K and V of a step are split on their way to
// one LDS buffer per group.  A row's exponents are relative to a whole number (the ceiling of its maximum so far), so that
// bringing its sums to a new reference is exact; sums and products are formed as in scores and apply.
// With 32 rows to a work-group a wave walks its steps alone (ALONE): K goes from memory to operand registers, V through LDS
// of the wave's own, and nothing waits for a barrier; the splits, 1.2 us of a step where they came in front of the products, lie
// beside them.  us: 2 heads of 256 rows 9.9 -> 9.5, 16 of 512 17.2 -> 14.8, causal 10 of 832 26.9 -> 22.0, 12 of 1024 36.1 ->
// 30.5.  (Eight such waves: 512 rows 15.3, 256 rows 10.8.)  One step a wave has nothing to lie beside: up to 128 rows the waves
// fill LDS together (64 rows 6.9, 6.5; 128 rows 7.1, 6.7; 192 rows 9.5, 9.7), also where causal rows see no more (94 heads, the first 64
// of 1024 rows 7.1, 6.7).
struct PassArgs {
  const float *Q, *K, *V;
  float *O, *LSE;
  int64_t L, Lq, q0;
  int causal;
  FastDiv by_tiles;  // row tiles of a head
  float cl2;
};

template <int RW, int KS, bool ALONE>
__device__ __forceinline__ void f32_forward_body(const PassArgs &a) {
  typedef TileT<float> TT;
  constexpr int BM = 32 * RW, RT = 32, PL = RT * 128;
  static_assert(!ALONE || RW == 1, "a lone wave shares its keys with none");
  struct Stage { unsigned char K[ALONE ? 16 : 3 * PL], V[3 * PL]; };
  constexpr int kBuf = KS * (int)sizeof(Stage), kOut = RW * 8192;
  __shared__ __attribute__((aligned(16))) unsigned char buf[kBuf > kOut ? kBuf : kOut];
  __shared__ float sums[KS == 1 ? 1 : KS][RW][2][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % RW;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / RW;
  const int col = lane & 31, half = lane >> 5;
  Stage &st = reinterpret_cast<Stage *>(buf)[grp];
  const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x), head = a.by_tiles(wg);
  uint32_t rt = wg - head * a.by_tiles.d;
  if (a.causal) rt = a.by_tiles.d - 1 - rt;  // (the long work-groups first)
  const int row0 = (int)rt * BM, wrow = row0 + wave * 32, Lq = (int)a.Lq, q0 = (int)a.q0;
  const bool rows_here = wrow < Lq;
  int nt = (int)(a.L / RT);  // steps of 32 keys
  if (a.causal) {
    const int seen = (q0 + (row0 + BM < Lq ? row0 + BM : Lq) - 1) / RT + 1;
    nt = seen < nt ? seen : nt;
  }
  const float *Kh = a.K + (int64_t)head * a.L * 64, *Vh = a.V + (int64_t)head * a.L * 64;
  typename TT::template Tile<RT, RW> k_tile(wave, lane, 64), v_tile(wave, lane, 64);
  f32x4 key[ALONE ? 2 * kSlices : 1];  // a lone wave's step of K, as it multiplies it
  // (a lone wave past its last step fetches that again: a branch would part the splits from the products)
  auto fetch_k = [&](int t) __attribute__((always_inline)) {
    if (ALONE && t >= nt) t = nt - 1;
    if constexpr (ALONE) {
      const float *p = Kh + ((int64_t)t * RT + col) * 64 + half * (kSliceK / 2);
#pragma unroll
      for (int i = 0; i < 2 * kSlices; ++i) key[i] = *reinterpret_cast<const f32x4 *>(p + (i >> 1) * kSliceK + (i & 1) * 4);
    } else {
      k_tile.fetch(Kh + (int64_t)t * (RT * 64));
    }
  };
  auto fetch_v = [&](int t) __attribute__((always_inline)) {
    if (ALONE && t >= nt) t = nt - 1;
    v_tile.fetch(Vh + (int64_t)t * (RT * 64));
  };
  auto fetch = [&](int t) __attribute__((always_inline)) {
    if (!ALONE && t >= nt) return;
    fetch_k(t);
    fetch_v(t);
  };
  auto put = [&](int t) __attribute__((always_inline)) {
    if (ALONE || t >= nt) return;
    k_tile.put(st.K);
    v_tile.put(st.V);
  };
  int t = grp;  // this group's step
  RowFrags<float, 1> q;
  {
    const float *qp = a.Q + ((int64_t)head * Lq + (rows_here ? wrow : row0) + col) * 64 + half * (kSliceK / 2);
    if constexpr (ALONE) {
      f32x4 raw[2 * kSlices];  // (in front of the step's loads, under which it is split)
#pragma unroll
      for (int i = 0; i < 2 * kSlices; ++i) raw[i] = *reinterpret_cast<const f32x4 *>(qp + (i >> 1) * kSliceK + (i & 1) * 4);
      __builtin_amdgcn_sched_barrier(0);
      fetch(t);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kSlices; ++i) q.f[i] = split8(raw[2 * i], raw[2 * i + 1]);
    } else {
      fetch(t);
      float none;
      q.template load<false>(qp, qp, none);
    }
  }
  if (!ALONE) {
    put(t);
    fetch(t + KS);
  }
  const TT tt(lane);
  f32x16 o[2];
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  float M = -INFINITY;          // the row's reference, a whole number
  float l = 0.f, l_err = 0.f;   // the lane's share of the row's sum, and what its additions have lost so far
  if (!ALONE) barrier_lds();
  while (ALONE ? t < nt : t - grp < nt) {
    const int k0 = t * RT;
    if (ALONE || (rows_here && (KS == 1 || t < nt) && (!a.causal || k0 <= q0 + wrow + 31))) {
      f32x16 s, rest;
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = rest[v] = 0.f;
      if constexpr (ALONE) {  // (V is split beside the products; its place is the wave's own, which takes no barrier)
        typename TT::Frag kf[kSlices];
#pragma unroll
        for (int i = 0; i < kSlices; ++i) kf[i] = split8(key[2 * i], key[2 * i + 1]);
        fetch_k(t + KS);
#pragma unroll
        for (int i = 0; i < kSlices; ++i) TT::mfma(kf[i], q.get(i), s, rest);
        v_tile.put(st.V);
        fetch_v(t + KS);
#pragma unroll
        for (int i = 0; i < 6 * kSlices; ++i) {  // a lone wave's vector instructions in the shadow of its products
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 16, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int i = 0; i < kSlices; ++i) TT::mfma(tt.template rows<PL>(st.K, 0, i), q.get(i), s, rest);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] += rest[v];
      if (a.causal && k0 + 31 > q0 + wrow) {
        const uint32_t seen = low_bits(q0 + wrow + col + 1 - k0 - half * 4);
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = keep_bit(s[v], seen, (v >> 2) * 8 + (v & 3));
      }
      float m = s[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) m = fmaxf(m, s[v]);
      m = ceilf(xhalf_max(m) * a.cl2);
      if (__builtin_amdgcn_ballot_w64(m > M) != 0) {
        const float to = fmaxf(m, M);
        const int by = M > -INFINITY ? (int)fmaxf(M - to, -300.f) : 0;  // (2^-300 of a sum leaves nothing)
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[db][v] = __builtin_ldexpf(o[db][v], by);
        l = __builtin_ldexpf(l, by);
        l_err = __builtin_ldexpf(l_err, by);
        M = to;
      }
      const float ref = M > -INFINITY ? M : 0.f;  // (a row that has seen no key yet)
      float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], a.cl2, -ref));
        p[v & 3] += s[v];
      }
      const float x = ((p[0] + p[1]) + (p[2] + p[3])) - l_err, sum = l + x;
      l_err = (sum - l) - x;
      l = sum;
      typename TT::Frag pf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        pf[i] = split8<false>(f32x4{s[i * 8], s[i * 8 + 1], s[i * 8 + 2], s[i * 8 + 3]},
                              f32x4{s[i * 8 + 4], s[i * 8 + 5], s[i * 8 + 6], s[i * 8 + 7]});
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        f32x16 c;
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] = 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) c = TT::mfma(tt.template cols<PL>(st.V, i, db), pf[i], c);
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] += c[v];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (!ALONE) {
      barrier_lds();
      put(t + KS);
      fetch(t + 2 * KS);
      barrier_lds();
    }
    t += KS;
  }
  l = xhalf_sum(l - l_err);
  if constexpr (KS > 1) {  // to the largest of the groups' references, and together
    static_assert(RW <= 2 && kBuf >= 16384 + (KS - 1) * RW * 2 * 4096, "room for the groups' sums behind the epilogue's tiles");
    sums[grp][wave][0][lane] = M;
    barrier_lds();
    float top = M;
    for (int g = 0; g < KS; ++g) top = fmaxf(top, sums[g][wave][0][lane]);
    const int by = M > -INFINITY ? (int)fmaxf(M - top, -300.f) : 0;
    l = __builtin_ldexpf(l, by);
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[db][v] = __builtin_ldexpf(o[db][v], by);
    M = top;
    sums[grp][wave][1][lane] = l;
    if (!add_groups<RW, KS>(buf, o, grp, wave, lane)) return;
    for (int g = 1; g < KS; ++g) l += sums[g][wave][1][lane];
  }
  if (!rows_here) return;
  const int64_t row = (int64_t)head * Lq + wrow;
  if (half == 0) a.LSE[row + col] = fmaf(M, kLn2, logf(l));
  unsigned char *ot = buf + wave * 8192;  // (free after the last barrier)
  TT::stage(ot, o[0], o[1], 1.0f / l, lane);
  TT::flush(ot, a.O + row * 64, 32, lane, 64);
}
template <int RW, int KS>
__global__ void __launch_bounds__(64 * RW * KS, KS > 1 ? 1 : 3) f32_forward_kernel(PassArgs a) {
  f32_forward_body<RW, KS, RW == 1>(a);
}
// ... of walks of one step a wave
template <int RW, int KS>
__global__ void __launch_bounds__(64 * RW * KS, 1) f32_forward_step_kernel(PassArgs a) {
  f32_forward_body<RW, KS, false>(a);
}

// --------------------------------------------------------------- collect ----
// out (key, A) = alpha * sum over the group's rows of strip(row, key) Y(row, A), two products per launch
// (dV from P and dO, dK from dS and Q).  Work-group: 128 keys (wave: 32) x 64 AHW columns, walking the row
// tiles through a ring of DEPTH LDS buffers, DEPTH - 1 tiles requested ahead.  With several row groups the sums pass
// through fp32 accumulators: `add` continues them, `keep` leaves them there instead of writing the result.
struct CollectArgs {
  const void *strip[2], *Y[2];
  void *out[2];
  float *acc[2];
  const float *norm;  // fp32: (head, rows), the factors of the strips' rows
  float alpha[2];
  int add, keep;
};

// WK waves share the work-group's keys, 32 each; QS groups of such waves share the row tiles (see apply).
struct CollectPos {  // of a work-group of BK keys x 64 AHW columns
  int64_t head, key0;
  int a0;
  bool which;
  __device__ __forceinline__ CollectPos(const StripArgs &a, int BK, int AHW, bool dq = false) {
    uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t cblocks = (uint32_t)(a.A / (64 * AHW));
    a0 = (int)(wg % cblocks) * (64 * AHW);
    wg /= cblocks;
    which = !dq && (wg & 1);
    wg >>= dq ? 0 : 1;
    key0 = (int64_t)(wg % (uint32_t)a.kblocks) * BK;
    if (dq && a.causal) key0 = (int64_t)(a.kblocks - 1) * BK - key0;  // (the long walks first)
    head = wg / (uint32_t)a.kblocks;
  }
  // first tile of RT rows whose last row sees the block's first key
  __device__ __forceinline__ int first_tile(const StripArgs &a, int RT, int nt) const {
    if (!a.causal || key0 <= a.q0 + 63) return 0;
    const int64_t f = (key0 - a.q0) / 64 * (64 / RT);
    return f < nt ? (int)f : nt;
  }
};
// The wave's 32 keys from wkey on, column a0 on, become results or stay in the fp32 accumulators.
template <typename T, int AHW>
__device__ __forceinline__ void collect_out(const StripArgs &a, const CollectArgs &p, const CollectPos &pos, f32x16 (&o)[2 * AHW],
                                            int64_t wkey, unsigned char *ot, int lane) {
  typedef TileT<T> TT;
  const int col = lane & 31, half = lane >> 5;
  if (p.add || p.keep) {
    float *acc = (pos.which ? p.acc[1] : p.acc[0]) + (pos.head * a.L + wkey + TT::key_of_col(col)) * a.A + pos.a0 + half * 4;
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
  const float alpha = pos.which ? p.alpha[1] : p.alpha[0];
  T *out = static_cast<T *>(pos.which ? p.out[1] : p.out[0]) + (pos.head * a.L + wkey) * a.A + pos.a0;
#pragma unroll
  for (int ah = 0; ah < AHW; ++ah) {
    TT::stage(ot, o[2 * ah], o[2 * ah + 1], alpha, TT::key_of_col(col) + half * 32);
    TT::flush(ot, out + ah * 64, 32, lane, a.A);
  }
}

// DQ: the strip is dS^T, rows and keys change places, and the sums are dQ.
template <bool DQ, int AHW, int DEPTH, int WK, int QS>
__device__ __forceinline__ void collect_body(const StripArgs &a, const CollectArgs &p) {
  typedef uint16_t T;
  typedef TileT<T> TT;
  constexpr int BK = 32 * WK, KT = (WK + 1) / 2;  // keys, and the key tiles they lie in
  struct Stage { unsigned char S[KT][kTileBytes], Y[AHW][kTileBytes]; };  // 24 KiB leave room for three work-groups on a CU
  __shared__ __attribute__((aligned(16))) Stage st[QS * DEPTH];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % WK;
  const int grp = QS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / WK;
  const CollectPos pos(a, BK, AHW, DQ);
  const int tiles = (int)(a.rows / 64);
  int nt = tiles;
  if (DQ && a.causal) {
    const int64_t seen = (a.q0 + (pos.key0 + BK < a.L ? pos.key0 + BK : a.L) - 1) / 64 + 1;
    if (seen < nt) nt = (int)seen;
  }
  int t0 = DQ ? 0 : pos.first_tile(a, 64, nt);
  const int64_t ktiles = a.L / 64;
  const T *Sh = static_cast<const T *>(pos.which ? p.strip[1] : p.strip[0]) +
                strip_tile<T>(pos.head, tiles, 0, ktiles, pos.key0 / 64);
  const int64_t second = pos.key0 + 64 < a.L ? 4096 : 0;  // (no second key tile: refetch the first)
  const T *Yh = static_cast<const T *>(pos.which ? p.Y[1] : p.Y[0]) + pos.head * a.Lq * a.A + pos.a0;
  const StripDMA<WK> dma_s(wave, lane);
  const typename TT::template DMA<WK> dma_y(wave, lane, a.A);
  const uint32_t lds0 = lds_address(&st[grp * DEPTH]);
  constexpr int kLoads = KT * StripDMA<WK>::PER + AHW * TT::template DMA<WK>::PER;  // of a wave, per row tile
  auto load = [&](int tt_, int b) __attribute__((always_inline)) {  // row tile tt_ -> buffer b
    const T *s = Sh + tt_ * (ktiles * 4096);
    const uint32_t d = lds0 + (uint32_t)b * (uint32_t)sizeof(Stage);
    dma_s.load_unseen(s, d);
    if (KT == 2) dma_s.load_unseen(s + second, d + (uint32_t)sizeof(st[0].S[0]));
#pragma unroll
    for (int ah = 0; ah < AHW; ++ah)
      dma_y.load_unseen(Yh + (int64_t)tt_ * 64 * a.A + ah * 64, d + (uint32_t)(sizeof(st[0].S) + ah * sizeof(st[0].Y[0])));
  };
#pragma unroll
  for (int i = 0; i + 1 < DEPTH; ++i)
    if (t0 + grp + i * QS < nt) load(t0 + grp + i * QS, i);
  const int64_t wkey = pos.key0 + wave * 32, wtile = wkey & ~(int64_t)63;
  const int wcols = (int)(wkey >> 5) & 1;  // the wave's columns of the key tile
  const bool keys_here = wkey < a.L;
  const TT tt(lane);
  f32x16 o[2 * AHW];
#pragma unroll
  for (int db = 0; db < 2 * AHW; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  int b = 0;  // buffer of tile t
  for (; t0 < nt; t0 += QS) {
    const int t = t0 + grp;  // this group's tile
    // tile t has arrived, and behind the barrier every wave is done with the tile before, whose buffer takes the next one
    if (DEPTH == 3 && t + QS < nt) wait_loads<kLoads>();
    else wait_loads<0>();
    barrier_lds();
    if (t + (DEPTH - 1) * QS < nt) load(t + (DEPTH - 1) * QS, b == 0 ? DEPTH - 1 : b - 1);
    const Stage &cur = st[grp * DEPTH + b];
    const int64_t tile = (int64_t)t * 64;
    if (keys_here && (QS == 1 || t < nt) && (DQ ? tile_seen(a, wtile, tile) : tile_seen(a, tile, wtile))) {
      const unsigned char *S = cur.S[wave >> 1];
      typename TT::Frag sf[2], yf[2][2 * AHW];
      pipelined<kSlices>(
          [&](int s, int b) __attribute__((always_inline)) {
            sf[b] = tt.cols(S, s, wcols);
#pragma unroll
            for (int db = 0; db < 2 * AHW; ++db) yf[b][db] = tt.cols(cur.Y[db >> 1], s, db & 1);
          },
          [&](int s, int b) __attribute__((always_inline)) {
#pragma unroll
            for (int db = 0; db < 2 * AHW; ++db) o[db] = TT::mfma(yf[b][db], sf[b], o[db]);
          });
    }
    b = b + 1 < DEPTH ? b + 1 : 0;
  }
  barrier_lds();  // the epilogue writes to the buffers
  if constexpr (QS > 1) {
    static_assert(WK <= 2 && sizeof(st) >= 16384 + (QS - 1) * WK * 2 * AHW * 4096, "room for the groups' sums");
    if (!add_groups<WK, QS>(reinterpret_cast<unsigned char *>(st), o, grp, wave, lane)) return;
  }
  if (!keys_here) return;
  // (the buffers are free after the last barrier; a Stage holds at least two blocks of 32 x 64)
  collect_out<T, AHW>(a, p, pos, o, wkey, reinterpret_cast<unsigned char *>(&st[wave >> 1]) + (wave & 1) * 4096, lane);
}

template <int AHW, int DEPTH, int WK, int QS>
__global__ void __launch_bounds__(64 * WK * QS, QS > 1 ? 1 : (AHW == 1 && DEPTH == 2 ? 3 : 2)) strip_collect_kernel(StripArgs a, CollectArgs p) {
  collect_body<false, AHW, DEPTH, WK, QS>(a, p);
}
template <int AHW, int DEPTH, int WK, int QS>
__global__ void __launch_bounds__(64 * WK * QS, QS > 1 ? 1 : (AHW == 1 && DEPTH == 2 ? 3 : 2)) strip_apply_keys_kernel(StripArgs a, CollectArgs p) {
  collect_body<true, AHW, DEPTH, WK, QS>(a, p);
}

// fp32: 64 columns, 32 rows a step through registers; the strips' rows are scaled on their way to LDS.
template <int WK, int QS>
__global__ void __launch_bounds__(64 * WK * QS, QS > 1 ? 1 : 2) strip_collect_f32_kernel(StripArgs a, CollectArgs p) {
  typedef TileT<float> TT;
  constexpr int RT = 32, PL = RT * 128;                    // rows per step, bytes of a part's plane
  constexpr int BK = 32 * WK, KT = (WK + 1) / 2;           // (see above)
  constexpr int CH = WK == 1 ? 4 : 8;                      // chunks of eight keys per tile that the work-group needs
  struct Stage { unsigned char S[KT][3 * PL], Y[3 * PL]; };
  __shared__ __attribute__((aligned(16))) Stage st[QS];
  static_assert(sizeof(st) >= (QS > 1 ? 16384 + (QS - 1) * WK * 2 * 4096 : WK * 8192), "room for the groups' sums and the epilogue");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % WK;
  const int grp = QS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / WK;
  const CollectPos pos(a, BK, 1);
  const int nt = (int)(a.rows / RT);
  int t0 = pos.first_tile(a, RT, nt);
  const int64_t ktiles = a.L / 64;
  const float *Sh = static_cast<const float *>(pos.which ? p.strip[1] : p.strip[0]) +
                    strip_tile<float>(pos.head, a.rows / 64, 0, ktiles, pos.key0 / 64);
  const int64_t second = pos.key0 + 64 < a.L ? 4096 : 0;
  const float *Yh = static_cast<const float *>(pos.which ? p.Y[1] : p.Y[0]) + pos.head * a.Lq * a.A + pos.a0;
  const float *norms = p.norm + pos.head * a.rows + (lane & 31);
  const int64_t wkey = pos.key0 + wave * 32, wtile = wkey & ~(int64_t)63;
  const int wcols = (int)(wkey >> 5) & 1;
  const bool keys_here = wkey < a.L;
  typename TT::template Tile<RT, WK, true, CH> s_tile(wave, lane, 0, WK == 1 ? wcols * 4 : 0), s_tile2(wave, lane, 0);
  typename TT::template Tile<RT, WK> y_tile(wave, lane, a.A);
  float factor = 0.f;
  auto fetch = [&](int t) __attribute__((always_inline)) {
    if (t >= nt) return;
    const int row = t * RT;
    const float *s = Sh + (row >> 6) * (ktiles * 4096) + (row & 63) * 64;
    s_tile.fetch(s);
    if (KT == 2) s_tile2.fetch(s + second);
    y_tile.fetch(Yh + (int64_t)row * a.A);
    factor = norms[row];
  };
  auto put = [&](int t) __attribute__((always_inline)) {
    if (t >= nt) return;
    s_tile.put(st[grp].S[0], factor);
    if (KT == 2) s_tile2.put(st[grp].S[KT - 1], factor);
    y_tile.put(st[grp].Y);
  };
  fetch(t0 + grp);
  put(t0 + grp);
  fetch(t0 + grp + QS);
  const TT tt(lane);
  f32x16 o[2];
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  barrier_lds();
  for (; t0 < nt; t0 += QS) {
    const int t = t0 + grp;
    if (keys_here && (QS == 1 || t < nt) && tile_seen(a, (int64_t)t * RT, wtile)) {
      const unsigned char *S = st[grp].S[wave >> 1];
      typename TT::Frag sf[2], yf[2][2];
      f32x16 c[2];  // the step's own sum
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) c[db][v] = 0.f;
      pipelined<RT / kSliceK>(
          [&](int s, int b) __attribute__((always_inline)) {
            sf[b] = tt.template cols<PL>(S, s, wcols);
#pragma unroll
            for (int db = 0; db < 2; ++db) yf[b][db] = tt.template cols<PL>(st[grp].Y, s, db);
          },
          [&](int s, int b) __attribute__((always_inline)) {
#pragma unroll
            for (int db = 0; db < 2; ++db) c[db] = TT::mfma(yf[b][db], sf[b], c[db]);
          });
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] += c[db][v];
    }
    barrier_lds();
    put(t + QS);
    fetch(t + 2 * QS);
    barrier_lds();
  }
  if constexpr (QS > 1) {
    if (!add_groups<WK, QS>(reinterpret_cast<unsigned char *>(st), o, grp, wave, lane)) return;
  }
  if (!keys_here) return;
  collect_out<float, 1>(a, p, pos, o, wkey, reinterpret_cast<unsigned char *>(st) + wave * 8192, lane);
}

// ------------------------------------------------------------------ host ----
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Groups of waves on a walk of the fp32 forward in one pass (128 / groups rows per work-group), or 0: the strip, whose
// scores are shared by work-groups along the keys too, is better where rows are few and walks long.  us, strip -> one pass, by
// W, the work-groups of 128 rows: 64 (256 rows) 13.6 -> 9.6, 120 (320) 21.2 -> 15.8, 400 (512) 61.7 -> 51.4, 512 (512) 72.8 -> 53.5, 516
// (1536) 245 -> 193, causal 288 (1536) 75.7 -> 71.8, 96 (768) 30.4 -> 20.4; but 192 (2048) 117.3 -> 117.8, 64 (1024) with
// one or two groups 30.4 -> 61, 42.
// Short walks: a work-group alone on its CU takes 14.5, 22.8, 32.6 us (512 rows) with four, two, one group; a second one on the
// CU adds 13, 11, 18 us.  So as many groups as leave each work-group a CU; else two where they make one work-group per CU
// more of both kinds (320 rows, W = 288: two 23.7, one 33.6; but 512 rows: 50.2, 50.5), under the causal mask, whose short walks
// leave room, up to 720 of them (512 rows, W = 320: 38.7, 50.2; W = 400: 49.8, 50.7; 256 rows, W = 320: 29.5, 28.7).
// (Long walks of four groups with a CU to each work-group would be faster than the strip as well, 8 heads of 768 rows 24.1 -> 19.3,
// 3 of 2048 47.5 -> 43.4, 8 of 2048 causal 75.6 -> 49.3: only causal ones of up to 1024 rows have a line here.)
int f32_one_pass(const Dims &d) {
  if (d.A != 64) return 0;
  const int64_t heads = (int64_t)d.B * d.Z, W = heads * ((d.Lq + 127) / 128);
  if (d.L <= 512) {
    const int64_t by_two = heads * (d.Lq / 64), by_four = heads * (d.Lq / 32);
    if (by_four <= 256) return 4;
    return by_two <= (d.causal ? 720 : (W > 256 ? 512 : 256)) ? 2 : 1;
  }
  if (d.causal && d.L <= 1024 && W > 64 && W <= 128) return 4;
  if (d.causal && W >= 250 && W <= 400) return 2;
  return W >= 400 ? 1 : 0;
}

// The bf16 forward by the kernels that keep no strip (two_pass_forward), for heads of 64 and 128 with more
// than 64 work-groups of 128 rows (W); the strip, whose scores are shared by work-groups along the keys too, where rows are few.
// The strip was written and read at 4 to 5 TB/s, the products of one pass are bound by the matrix pipe and the exponentials.
// us, strip -> one pass: W = 128 (8 heads of 2048 rows) 33 -> 17, 512 (128 of 512) 37 -> 15.5, 1024 (128 of 1024) 139 -> 45, 2048
// (128 of 2048) 495 -> 159, causal 384 (12 of 4096) 113 -> 47; heads of 128: 80 (640 rows) 17.2 -> 14.3, causal 14.6 both, 512
// (512) 40 -> 27; but 64 (2048) 26.9 -> 32.1, 32 (2048) 18.8 -> 31.7.  Heads of 128 have at most two work-groups to a CU, each as long as
// the longest walk, where the strip's scores are shared along it: on long walks the line lies at more rows, under the causal mask, whose
// strip is half as long, at more again.  Over 9300 calls of 65 to 270 work-groups the time by these lines is 0.79 to 0.80 of the strip's on
// average and more than 1.04 of it in 79, by the 64 work-groups in 1690 (2 heads of 4608 rows 55.6 -> 66.1, causal 5 of 1600 22.9 ->
// 27.8, 2 of 8192 99 -> 117, 8 of the third 1280 of 5120 46.3 -> 57.5).  Heads of 64 lose later, with one or two heads of long rows (1
// of 1024 10.0 -> 11.1, 1 of 2048 14.7 -> 17.1), and gain at other W below the line (8 of 1024 14.0 -> 11.3, 4 of 2048 21.7 -> 17.2, 16 of
// 256 8.7 -> 6.8): they have no line of their own.  L >= A: all results then take no more room than strips.
int bf16_one_pass(const Dims &d) {
  const int64_t W = (int64_t)d.B * d.Z * ((d.Lq + 127) / 128);
  if (d.A > 128 || d.L < d.A || W <= 64) return 0;
  const int64_t walk = (d.causal ? d.rank_end * d.c : d.L) / 64;
  if (d.A == 64 || walk < 6) return 1;
  int64_t line = 40 + walk * 5 / 4, most = 110;  // in blocks of 128 rows
  if (d.causal) {
    const bool uneven = 2 * d.rank_begin < d.rank_end;  // walks of a few keys beside long ones
    line = 40 + walk * (uneven ? 3 : 2); most = uneven ? 180 : 130;
  }
  return (int64_t)d.B * d.Z * d.Lq > 128 * (line < most ? line : most);
}

// How the work is cut: `heads` heads and `rows` of their query rows per group of launches, and where a
// group's buffers lie in the workspace; out: results that may not be written yet (see apart_plan), of `chunk` heads.
// usual, one_pass: what kernels and their shapes are chosen by, the heads of a group and f32_one_pass or bf16_one_pass of the call
// as it is where its results lie beside its inputs, so that they round alike wherever they lie.
// keys: the groups of waves of collect_keys' work-groups, or 0 for the backward by rows; by_rows: what the latter would ask of
// every call.
struct StripPlan {
  int64_t heads, rows, chunk, usual;
  int one_pass, keys;
  size_t by_rows;
  size_t out[3];
  size_t terms, strip, strip2, stats, norm, acc_k, acc_v, total;
};

// Places a group's buffers from byte `off` of the workspace on (one pass: it has none).
void place_group(StripPlan &p, const Dims &d, int dtype, int pass, size_t off) {
  p.total = off;
  if (p.one_pass) return;
  if (p.keys) {
    p.terms = off; off += align256((size_t)p.chunk * d.Lq * 8);
    p.strip = off; off += align256((size_t)p.heads * p.rows * d.L * 2);
    p.total = off;
    return;
  }
  const size_t es = dtype == RSA_BF16 ? 2 : 4, scores = (size_t)p.heads * p.rows * d.L;
  p.strip = off; off += align256(scores * es);
  if (pass == 1) {
    p.strip2 = off; off += align256(scores * es);
    if (dtype == RSA_F32) {
      p.stats = off; off += align256(scores / 64 * 4);
      p.norm = off; off += align256((size_t)p.heads * p.rows * 4);
    }
    if (p.rows < d.Lq) {
      p.acc_k = off; off += align256((size_t)p.heads * d.L * d.A * 4);
      p.acc_v = off; off += align256((size_t)p.heads * d.L * d.A * 4);
    }
  } else {
    p.stats = off; off += align256(scores / 64 * 8);
  }
  p.total = off;
}

// Sizes of a group's strips.  All heads and rows at once where that is at most kStripBytes; else groups of
// heads of at most kCacheBytes, which the 256 MB infinity cache still holds when the next kernel reads them
// (bert_large-shaped, 12 groups: 1678 us; 5 groups of 512 MB 1946, one group 1689); else, for a single head with longer
// strips, groups of rows that fill kStripBytes or what one rank's strips take with an fp32 and a dtype copy
// of every score, whichever is more.
constexpr size_t kStripBytes = (size_t)512 << 20, kCacheBytes = (size_t)192 << 20;

StripPlan strip_plan_by_rows(const Dims &d, int dtype, int pass, bool strips_only = false) {
  const size_t es = dtype == RSA_BF16 ? 2 : 4, strips = pass == 1 ? 2 : 1;
  const int64_t heads = (int64_t)d.B * d.Z;
  const size_t one_rank = (size_t)heads * d.c * d.L * (4 + es) * strips;
  const size_t row = (size_t)d.L * es * strips, head = row * d.Lq;  // bytes of a head's row, of a head
  StripPlan p{};
  p.rows = d.Lq;
  p.heads = heads;
  p.one_pass = pass == 0 && !strips_only ? (dtype == RSA_F32 ? f32_one_pass(d) : bf16_one_pass(d)) : 0;
  if (head * heads > kStripBytes && !p.one_pass) {
    if (head <= kStripBytes) {
      const int64_t most = head < kCacheBytes ? (int64_t)(kCacheBytes / head) : 1;
      const int64_t groups = (heads + most - 1) / most;
      p.heads = (heads + groups - 1) / groups;  // groups of equal size
    } else {
      const size_t budget = one_rank > kStripBytes ? one_rank : kStripBytes;
      p.heads = 1;
      p.rows = (int64_t)(budget / row) / 128 * 128;  // at least 128: budget holds one rank's rows, 64 or more, twice
      if (p.rows > d.Lq) p.rows = d.Lq;
    }
  }
  p.usual = p.heads;
  p.chunk = heads;
  place_group(p, d, dtype, pass, 0);
  return p;
}

StripPlan strip_plan(const Dims &d, int dtype, int pass);
StripPlan apart_plan(const Dims &d, int dtype, int pass, StripPlan p, bool whole, size_t bytes);

// The bf16 backward by keys (collect_keys: dK, dV, and dS as the only strip, written once and read once) where its
// work-groups of 128 keys fill the chip, in no more workspace than the backward by rows takes (P and dS, five passes over a
// strip).  Wk, Wq: work-groups of 128 keys and of 128 rows (those of dQ) of a group of heads.  The lines are those of 1600 calls,
// whole rings of 64 .. 2048 rows and shares of 1/2 .. 1/16 of up to 4096: where it is taken it takes 0.76 of the time on average and
// 1.04 at most.  us, by rows -> by keys, heads of 64: 18 heads of 1024 rows (Wk = 144) 48 -> 38, 40 of 512 (160) 31.6 -> 25.4, 12 of 2048
// causal (192) 70 -> 51, 50 of 576 (250) 39 -> 30, 128 of 512 (512) 69 -> 46, 128 of 2048 (256, eight times) 1141 -> 545; but 24 heads of
// 384 of 1536 rows (168) 20 -> 21, 42 of 320 causal (126) 20.1 -> 20.7, 10 of 1280 causal (100) 36 -> 47.  One rank's rows leave dQ few
// work-groups on long walks: 9 heads of 512 of 2048 rows (Wq = 36) 33.6 -> 37.2, the last causal ones 33.8 -> 41.5, 62 of 64 of 512 16.5 ->
// 18.1; 16 of 512 of 2048 (64) 40.4 -> 36.4.  Heads of 128 fill a CU with one work-group: a round of 256 that is nearly empty costs as
// much as a full one (128 of 256, 256, 34.9 -> 30.3, 150 of 256, 300, 43.8 -> 43.7, 30 of 1088, 270, 100 -> 105), and two groups of waves on
// causal walks pay for long ones alone (41 of 768, 246, 53.2 -> 55.0, 85 of 320, 255, 32.6 -> 37.3; 32 of 1024, 256, 65.4 -> 58.1); 30 heads of
// 896 causal (210) 63 -> 59, 64 of 1024 (512) 189 -> 130; 62 of 64 of 512 20.7 -> 22.9, 125 of 128 of 1024, last causal, 62.7 -> 68.1.  Strips of
// all heads that the infinity cache cannot hold (64 M scores of P and dS) cost most: 21 of 1792 (294) 217 -> 160, 22 of 1024 of 4096, last
// causal, 264 -> 189.  Keys that no row sees are work-groups all the same: not the first of sixteen causal ranks (256, 400 heads of 64 of
// 1024 rows 25 -> 28, 32 -> 39); heads of 128, which lose more where fewer work-groups than CUs have rows, by 240 of all heads that see any
// (5 heads of 128, the first 2816 of 7040 rows, 110: 101 -> 142, 9 of 1984 of 3968, 139: 80 -> 106; 4700 such calls: 181 took more than 1.04
// of the time by rows, now 40) and, of smaller strips, from a third of the keys on (109 heads, the first 384 of 3072 rows, 79 -> 119, 121 of
// 448 of 2240 85 -> 112).
bool by_keys_pays(const Dims &d, int64_t heads) {
  const int64_t Wk = heads * ((d.L + 127) / 128), Wq = heads * ((d.Lq + 127) / 128), seen = d.causal ? d.rank_end * d.c : d.L;
  const bool whole = d.Lq == d.L, part = d.causal && !whole;
  if (16 * seen <= d.L) return false;
  if (d.A == 64) {
    if (Wk < 240 && (Wk < 128 || d.Lq < 512)) return false;
    if (Wq < 64 || Wk + Wq < (d.causal ? 260 : 240)) return false;
    return !d.causal || whole || d.Lq >= 128 || Wk >= 500;
  }
  if (Wk < 200) return false;
  if (d.Lq >= 512 && Wq >= 96 && (int64_t)d.B * d.Z * d.Lq * d.L >= (int64_t)64 << 20) return !part || (int64_t)d.B * d.Z * seen >= 240 * 128;
  if (part && 20 * seen < 7 * d.L) return false;
  if (!d.causal) return Wq >= 128 && (Wk <= 256 ? d.Lq >= 128 : Wk >= 320 && d.Lq >= 384);
  return Wk <= 256 ? d.Lq >= 960 && Wq >= 200 : Wk >= 300 && Wq >= 240 && d.Lq >= (whole ? 192 : 384);
}
bool plan_by_keys(const Dims &d, StripPlan &p) {
  if (d.A > 128) return false;
  const int64_t heads = (int64_t)d.B * d.Z, blocks = (d.L + 127) / 128;
  StripPlan k = p;
  k.rows = d.Lq; k.keys = 1;
  const size_t strip = (size_t)d.Lq * d.L * 2, terms = align256((size_t)heads * d.Lq * 8);
  if (p.total < terms + align256(strip)) return false;
  const int64_t most = (int64_t)((p.total - terms - 255) / strip);
  if (most < 1) return false;
  k.heads = heads;
  if (most < heads) {  // groups whose work-groups come in whole rounds of one to a CU; a group's launches cost a fifth of one
    float least = 1e30f;
    for (int64_t g = most; g > most / 2; g -= 1 + most / 64) {
      const int64_t n = (heads + g - 1) / g, last = heads - (n - 1) * g;
      auto rounds = [&](int64_t h) {  // (causal walks of several rounds even out)
        const float r = (float)(h * blocks) / 256;
        return d.causal ? fmaxf(r, 1.f) : ceilf(r);
      };
      const float cost = (float)(n - 1) * rounds(g) + rounds(last) + 0.2f * (float)n;
      if (cost < least) { least = cost; k.heads = g; }
    }
  }
  const int64_t W = k.heads * blocks;
  if (!by_keys_pays(d, k.heads)) return false;
  // groups of waves on the walks of uneven length (causal, heads of 64: 12 heads of 2048, W = 192: one 63, two 56, four 51;
  // 72 of 512, 288: 33.7, 31.2, 40.6; 52 of 1024, 416: 54.8, 53.2; 42 of 1344, 462: 67.4, 67.7; of 128: 21 of 1536, 252: 90, 82.5)
  if (d.causal) k.keys = d.A == 128 ? (W <= 256 ? 2 : 1) : (W <= 200 ? 4 : (W <= 360 ? 2 : 1));
  k.usual = k.heads;
  place_group(k, d, RSA_BF16, 1, 0);
  const size_t apart = apart_plan(d, RSA_BF16, 1, p, false, 0).total;
  k.by_rows = apart > p.total ? apart : p.total;
  if (apart_plan(d, RSA_BF16, 1, k, false, 0).total > k.by_rows) return false;
  p = k;
  return true;
}
StripPlan strip_plan(const Dims &d, int dtype, int pass) {
  StripPlan p = strip_plan_by_rows(d, dtype, pass);
  if (dtype == RSA_BF16 && pass == 1) plan_by_keys(d, p);
  return p;
}

// Bytes of one head of the pass's results (O and LSE, or dQ, dK and dV) and inputs (Q, K, V; dO, O, LSE).
struct HeadBytes {
  size_t out[3], in[6];
  HeadBytes(const Dims &d, int dtype, int pass) {
    const size_t es = dtype == RSA_BF16 ? 2 : 4, q = (size_t)d.Lq * d.A * es, k = (size_t)d.L * d.A * es, l = (size_t)d.Lq * 4;
    out[0] = q; out[1] = pass == 1 ? k : l; out[2] = pass == 1 ? k : 0;
    in[0] = q; in[1] = in[2] = k; in[3] = in[4] = q; in[5] = l;
  }
};

// The plan for results that lie over inputs: they stay in the workspace until these have been read, and are copied
// then.  Where each lies tensor over tensor, head over head, that is a group's results at a time; else (whole) those of
// all heads.  The groups take what is left of a workspace of `bytes`; 0: the least plan, one head's 128 rows at a time,
// by keys all of a head's rows, or, in one pass, heads whose work-groups fill the chip twice.  p: the call's plan beside its inputs.
StripPlan apart_plan(const Dims &d, int dtype, int pass, StripPlan p, bool whole, size_t bytes) {
  const HeadBytes hb(d, dtype, pass);
  const int64_t all = (int64_t)d.B * d.Z;
  auto place = [&](int64_t heads, int64_t rows) {
    p.heads = heads; p.rows = rows; p.chunk = whole ? all : heads;
    size_t off = 0;
    for (int i = 0; i < 3; ++i) { p.out[i] = off; off += align256(p.chunk * hb.out[i]); }
    place_group(p, d, dtype, pass, off);
    return p.total <= bytes;
  };
  for (int64_t h = p.usual; bytes > 0 && h > 0; h = h * 7 / 8)
    if (place(h, d.Lq)) return p;
  for (int64_t r = d.Lq / 128 * 128; !p.keys && bytes > 0 && r > 128; r = r * 7 / 8 / 128 * 128)
    if (place(1, r)) return p;
  const int64_t fill = (512 * 128 + d.Lq - 1) / d.Lq;
  if (p.one_pass) place(fill < all ? fill : all, d.Lq);
  else place(1, d.Lq < 128 || p.keys ? d.Lq : 128);
  return p;
}
// ... of the call as it is.  By keys the least plan holds all of a head's rows: beside all results, where a workspace that was
// asked for by rows holds no more than 128 of them, the call goes by rows (as it does where a head's rows are cut, it then rounds
// otherwise).
StripPlan apart_plan(const Dims &d, int dtype, int pass, bool whole, size_t bytes) {
  const StripPlan p = apart_plan(d, dtype, pass, strip_plan(d, dtype, pass), whole, bytes);
  if (!p.keys || !whole || p.total <= bytes) return p;
  const StripPlan rows = apart_plan(d, dtype, pass, strip_plan_by_rows(d, dtype, pass), whole, bytes);
  return bytes > 0 || rows.total < p.total ? rows : p;
}

template <typename T>
hipError_t launch_scores(const StripArgs &a0, int64_t heads, bool bwd, hipStream_t st) {
  StripArgs a = a0;
  // Key tiles per work-group: the count (at most 16) whose rounds of work-groups cost least, a work-group costing
  // its tiles and about two more for its prologue.
  const int64_t tiles = a.L / 64, slots = 256 * (bwd ? (sizeof(T) * a.A <= 256 ? 2 : 1) : (sizeof(T) * a.A <= 256 ? (sizeof(T) == 4 ? 3 : 4) : 2));
  double best = 1e30;
  for (int per = 1; per <= 16 && per <= tiles; ++per) {
    const int64_t wgs = heads * a.rtiles * ((tiles + per - 1) / per);
    const double cost = (double)((wgs + slots - 1) / slots) * (per + 2);
    if (cost < best) { best = cost; a.per = per; }
  }
  a.kblocks = (int)((tiles + a.per - 1) / a.per);
  const dim3 grid((unsigned)(heads * a.rtiles * a.kblocks));
#define RSA_SCORES(AH)                                                                          \
  case AH:                                                                                      \
    if (bwd) hipLaunchKernelGGL((strip_scores_bwd_kernel<T, AH>), grid, dim3(256), 0, st, a);   \
    else hipLaunchKernelGGL((strip_scores_fwd_kernel<T, AH>), grid, dim3(256), 0, st, a);       \
    break;
  switch (a.A / 64) { RSA_SCORES(1) RSA_SCORES(2) RSA_SCORES(3) RSA_SCORES(4) }
#undef RSA_SCORES
  return hipGetLastError();
}

template <typename T, int AHW, bool WEIGHT, int RW, int KS>
hipError_t launch_apply_as(StripArgs a, const ApplyArgs &p, int64_t heads, hipStream_t st) {
  a.rtiles = (int)((a.rows + 32 * RW - 1) / (32 * RW));
  const dim3 grid((unsigned)(heads * a.rtiles * (a.A / (64 * AHW))));
  hipLaunchKernelGGL((strip_apply_kernel<T, AHW, WEIGHT, RW, KS>), grid, dim3(64 * RW * KS), 0, st, a, p);
  return hipGetLastError();
}
// Few work-groups: their walks over the key tiles are serial chains on a partly idle chip, so groups of waves share them.
// The lines are those of a sweep over 2 .. 192 heads of 64 .. 256 elements, 256 .. 3072 rows; forward, us, by W:
//   fp32, one group -> four: 4 (256 rows) 16.0 -> 12.8, 24 (1536) 59 -> 35, 64 (A 128) 26 -> 19, 72 causal 71 -> 46;
//   one -> two: 96 45 -> 37, 192 67.8 -> 66, 288 causal 93 -> 82; but 300 77 -> 81, 400 causal 59.9 -> 61.2;
//   bf16, one -> four: 24 (1536 rows) 19.5 -> 13.6, 48 (3072) 40 -> 26; one -> two: 144 53 -> 47; but 288 47 -> 49.
template <typename T, bool WEIGHT>
hipError_t launch_apply(const StripArgs &a, const ApplyArgs &p, int64_t heads, int64_t usual, hipStream_t st) {
  const int64_t W = usual * a.rtiles * (a.A / 64);  // work-groups of 128 rows and 64 columns
  if (W <= 64 || (a.causal && W <= (sizeof(T) == 4 ? 96 : 144))) return launch_apply_as<T, 1, WEIGHT, 1, 4>(a, p, heads, st);
  const bool two = sizeof(T) == 4 ? W <= (a.causal ? 290 : 200) : W <= (a.causal ? 360 : 240);
  if (two) return launch_apply_as<T, 1, WEIGHT, 2, 2>(a, p, heads, st);
  if constexpr (sizeof(T) == 2)
    if (a.A % 128 == 0) return launch_apply_as<T, 2, WEIGHT, 4, 1>(a, p, heads, st);
  return launch_apply_as<T, 1, WEIGHT, 4, 1>(a, p, heads, st);
}

template <typename T, int AHW, int DEPTH, int WK, int QS>
hipError_t launch_collect_as(StripArgs a, const CollectArgs &p, int64_t heads, hipStream_t st) {
  a.kblocks = (int)((a.L + 32 * WK - 1) / (32 * WK));
  const dim3 grid((unsigned)(heads * a.kblocks * 2 * (a.A / (64 * AHW))));
  if constexpr (sizeof(T) == 4) hipLaunchKernelGGL((strip_collect_f32_kernel<WK, QS>), grid, dim3(64 * WK * QS), 0, st, a, p);
  else hipLaunchKernelGGL((strip_collect_kernel<AHW, DEPTH, WK, QS>), grid, dim3(64 * WK * QS), 0, st, a, p);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_collect(const StripArgs &a, const CollectArgs &p, int64_t heads, int64_t usual, hipStream_t st) {
  const int64_t W = usual * ((a.L + 127) / 128) * 2 * (a.A / 64);  // work-groups of 128 keys and 64 columns
  // Groups of waves on the row tiles of few work-groups, as in apply (same sweep, backward, us, by W): fp32, one group ->
  // four: 8 32 -> 26, 48 (1536 rows) 134 -> 100; one -> two: 96 80.9 -> 69.6, 192 87.8 -> 84.9, causal 288 175 -> 155; but
  // 512 102 -> 110; bf16: A = 128, 128 23.4 -> 21.7, causal 288 58 -> 50, but not causal 65 -> 68.
  if constexpr (sizeof(T) == 4) {
    if (W <= 64 || (a.causal && W <= 96)) return launch_collect_as<T, 1, 2, 1, 4>(a, p, heads, st);
    if (W <= (a.causal ? 480 : 400)) return launch_collect_as<T, 1, 2, 2, 2>(a, p, heads, st);
    return launch_collect_as<T, 1, 2, 4, 1>(a, p, heads, st);
  } else {
    if ((a.A % 128 == 0 && W <= 256) || (a.causal && W > 256 && W <= 400)) return launch_collect_as<T, 1, 2, 2, 2>(a, p, heads, st);
  }
  if constexpr (sizeof(T) == 2) {
    if (a.A % 128 == 0) return launch_collect_as<T, 2, 2, 4, 1>(a, p, heads, st);
    // bf16 strips come at the rate that requests in flight allow.  With at most one work-group on a compute unit its row
    // tiles are requested two steps ahead; several bring enough by themselves, and three fit where each takes two
    // buffers.  The whole backward with two | three buffers, us: 64 work-groups 33.5 | 30.4, 256: 45.4 | 40.8 and
    // 161.5 | 140.8, 384 (in groups): 1165 | 1180, 1536: 121 | 121.
    if (W <= 256) return launch_collect_as<T, 1, 3, 4, 1>(a, p, heads, st);
    return launch_collect_as<T, 1, 2, 4, 1>(a, p, heads, st);
  }
}

// dQ from dS^T: a.rows are the keys here, a.L the query rows.
template <int AHW, int DEPTH, int WK, int QS>
hipError_t launch_apply_keys_as(StripArgs a, const CollectArgs &p, int64_t heads, hipStream_t st) {
  a.kblocks = (int)((a.L + 32 * WK - 1) / (32 * WK));
  const dim3 grid((unsigned)(heads * a.kblocks * (a.A / (64 * AHW))));
  hipLaunchKernelGGL((strip_apply_keys_kernel<AHW, DEPTH, WK, QS>), grid, dim3(64 * WK * QS), 0, st, a, p);
  return hipGetLastError();
}
// W: the usual group's work-groups of 128 rows.  Two groups of waves share the walks of uneven length where W barely fills
// the CUs (19 heads of 2048 causal rows, W = 304: 263 -> 232 us for the whole backward; 5 of 3840, W = 150: 579, 586); a
// ring of three tiles beats one of two that lets three work-groups share a CU (W = 256, 512, 2048 of 2048 rows: 580, 564, 600
// against 637, 558, 606).
hipError_t launch_apply_keys(const StripArgs &a, const CollectArgs &p, int64_t heads, int64_t usual, hipStream_t st) {
  if (a.A == 128) return launch_apply_keys_as<2, 2, 4, 1>(a, p, heads, st);
  const int64_t W = usual * ((a.L + 127) / 128);
  if (a.causal && W > 256 && W <= 360) return launch_apply_keys_as<1, 2, 2, 2>(a, p, heads, st);
  return launch_apply_keys_as<1, 3, 4, 1>(a, p, heads, st);
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

template <int RW, int KS>
hipError_t launch_f32_forward(const Dims &d, PassArgs a, hipStream_t st) {
  a.by_tiles = make_fast_div((d.Lq + 32 * RW - 1) / (32 * RW));
  const dim3 grid((unsigned)((int64_t)d.B * d.Z * a.by_tiles.d));
  const int64_t seen = d.causal ? d.rank_end * d.c : d.L;
  if (RW == 1 && seen <= 32 * KS) hipLaunchKernelGGL((f32_forward_step_kernel<1, 4>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((f32_forward_kernel<RW, KS>), grid, dim3(64 * RW * KS), 0, st, a);
  return hipGetLastError();
}
hipError_t f32_forward(const Dims &d, const void *Q, const void *K, const void *V, void *O, float *LSE, int groups,
                       hipStream_t st) {
  PassArgs a{};
  a.Q = static_cast<const float *>(Q); a.K = static_cast<const float *>(K); a.V = static_cast<const float *>(V);
  a.O = static_cast<float *>(O); a.LSE = LSE;
  a.L = d.L; a.Lq = d.Lq; a.q0 = (int64_t)d.rank_begin * d.c; a.causal = d.causal; a.cl2 = d.scale * kLog2e;
  if (groups == 4) return launch_f32_forward<1, 4>(d, a, st);
  return groups == 2 ? launch_f32_forward<2, 2>(d, a, st) : launch_f32_forward<4, 1>(d, a, st);
}

template <typename T>
hipError_t forward_t(const Dims &d, const void *Q, const void *K, const void *V, void *O, float *LSE,
                     char *ws, const StripPlan &pl, hipStream_t st) {
  if constexpr (sizeof(T) == 4)
    if (pl.one_pass) return f32_forward(d, Q, K, V, O, LSE, pl.one_pass, st);
  if constexpr (sizeof(T) == 2)
    if (pl.one_pass) return two_pass_forward(d, Q, K, V, O, LSE, pl.usual, st);
  const int64_t heads = (int64_t)d.B * d.Z;
  for (int64_t h0 = 0; h0 < heads; h0 += pl.heads) {
    const int64_t nh = pl.heads < heads - h0 ? pl.heads : heads - h0;
    for (int64_t r0 = 0; r0 < d.Lq; r0 += pl.rows) {
      const int64_t nr = pl.rows < d.Lq - r0 ? pl.rows : d.Lq - r0;
      const StripArgs a = group_args<T>(d, pl, ws, h0, r0, nr, Q, K, V);
      RSA_TRY(launch_scores<T>(a, nh, false, st));
      const ApplyArgs p = {a.strip, a.V, static_cast<T *>(O) + (h0 * d.Lq + r0) * d.A, LSE + h0 * d.Lq + r0, nullptr};
      RSA_TRY((launch_apply<T, true>(a, p, nh, pl.usual, st)));
    }
  }
  return hipSuccess;
}

// bf16: dK and dV while the scores are in registers, and of the strips dS alone, which dQ is formed from.
hipError_t backward_by_keys(const Dims &d, const void *dO, const void *Q, const void *K, const void *V, const void *O,
                            const float *LSE, void *dQ, void *dK, void *dV, char *ws, const StripPlan &pl, hipStream_t st) {
  const int64_t heads = (int64_t)d.B * d.Z;
  float *nL = reinterpret_cast<float *>(ws + pl.terms), *nD = nL + heads * d.Lq;
  char *strip = ws + pl.strip;
  RSA_TRY(fused_bwd_preprocess(d, dO, O, LSE, nD, nL, st));
  for (int64_t h0 = 0; h0 < heads; h0 += pl.heads) {
    const int64_t nh = pl.heads < heads - h0 ? pl.heads : heads - h0, q = h0 * d.Lq * d.A, k = h0 * d.L * d.A;
    auto in = [](const void *p, int64_t n) { return static_cast<const uint16_t *>(p) + n; };
    auto out = [](void *p, int64_t n) { return static_cast<uint16_t *>(p) + n; };
    Dims dg = d;  // (the tensors are dense)
    dg.B = 1; dg.Z = (int)nh;
    RSA_TRY(collect_keys(dg, in(dO, q), in(Q, q), in(K, k), in(V, k), nL + h0 * d.Lq, nD + h0 * d.Lq, out(dK, k), out(dV, k),
                         strip, pl.keys, st));
    StripArgs a = group_args<uint16_t>(d, pl, ws, h0, 0, d.Lq, Q, K, V);
    a.rows = d.L; a.L = d.Lq; a.Lq = d.L;  // (keys for rows: collect_body)
    CollectArgs c{};
    c.strip[0] = strip; c.Y[0] = in(K, k); c.out[0] = out(dQ, q); c.alpha[0] = d.scale;
    RSA_TRY(launch_apply_keys(a, c, nh, pl.usual, st));
  }
  return hipSuccess;
}

template <typename T>
hipError_t backward_t(const Dims &d, const void *dO, const void *Q, const void *K, const void *V,
                      const void *O, const float *LSE, void *dQ, void *dK, void *dV, char *ws, const StripPlan &pl,
                      hipStream_t st) {
  const int64_t heads = (int64_t)d.B * d.Z;
  if constexpr (sizeof(T) == 2)
    if (pl.keys) return backward_by_keys(d, dO, Q, K, V, O, LSE, dQ, dK, dV, ws, pl, st);
  for (int64_t h0 = 0; h0 < heads; h0 += pl.heads) {
    const int64_t nh = pl.heads < heads - h0 ? pl.heads : heads - h0;
    for (int64_t r0 = 0; r0 < d.Lq; r0 += pl.rows) {
      const int64_t nr = pl.rows < d.Lq - r0 ? pl.rows : d.Lq - r0;
      StripArgs a = group_args<T>(d, pl, ws, h0, r0, nr, Q, K, V);
      const int64_t q = (h0 * d.Lq + r0) * d.A, k = h0 * d.L * d.A;
      a.dO = static_cast<const T *>(dO) + q; a.O = static_cast<const T *>(O) + q;
      a.LSE_in = LSE + h0 * d.Lq + r0;
      RSA_TRY(launch_scores<T>(a, nh, true, st));
      float *norm = reinterpret_cast<float *>(ws + pl.norm);
      const ApplyArgs p = {a.strip2, a.K, static_cast<T *>(dQ) + q, nullptr, norm};
      RSA_TRY((launch_apply<T, false>(a, p, nh, pl.usual, st)));
      CollectArgs c{};
      c.strip[0] = a.strip; c.Y[0] = a.dO; c.out[0] = static_cast<T *>(dV) + k; c.alpha[0] = 1.0f;
      c.strip[1] = a.strip2; c.Y[1] = a.Q; c.out[1] = static_cast<T *>(dK) + k; c.alpha[1] = d.scale;
      c.acc[0] = reinterpret_cast<float *>(ws + pl.acc_v); c.acc[1] = reinterpret_cast<float *>(ws + pl.acc_k);
      c.norm = norm;
      c.add = r0 > 0; c.keep = r0 + nr < d.Lq;
      RSA_TRY(launch_collect<T>(a, c, nh, pl.usual, st));
    }
  }
  return hipSuccess;
}

__global__ void __launch_bounds__(256) copy_kernel(const u32x4 *from, u32x4 *to, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) to[i] = from[i];
}
hipError_t copy(const void *from, void *to, size_t bytes, hipStream_t st) {  // bytes: a multiple of 16
  const int64_t n = (int64_t)(bytes / 16);
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, static_cast<const u32x4 *>(from),
                     static_cast<u32x4 *>(to), n);
  return hipGetLastError();
}

// Whether results lie over inputs: 0 none, 1 only tensor over tensor of the same size, 2 in some other way.
int results_over_inputs(const Dims &d, int dtype, int pass, const void *const (&in)[6], void *const (&out)[3]) {
  const HeadBytes hb(d, dtype, pass);
  const size_t heads = (size_t)d.B * d.Z;
  int over = 0;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 6; ++j) {
      if (!in[j] || !out[i] || !overlap(out[i], heads * hb.out[i], in[j], heads * hb.in[j])) continue;
      const int how = out[i] == in[j] && hb.out[i] == hb.in[j] ? 1 : 2;
      if (how > over) over = how;
    }
  return over;
}

template <typename T>
hipError_t pass_t(const Dims &d, int pass, const void *const (&in)[6], void *const (&out)[3], char *ws,
                  const StripPlan &pl, hipStream_t st) {
  if (pass == 0) return forward_t<T>(d, in[0], in[1], in[2], out[0], static_cast<float *>(out[1]), ws, pl, st);
  return backward_t<T>(d, in[3], in[0], in[1], in[2], in[4], static_cast<const float *>(in[5]), out[0], out[1], out[2],
                       ws, pl, st);
}

// A pass over the heads in chunks, each with its results in the workspace until it is done.
template <typename T>
hipError_t pass_apart(const Dims &d, int pass, const void *const (&in)[6], void *const (&out)[3], char *ws,
                      const StripPlan &pl, hipStream_t st) {
  const HeadBytes hb(d, sizeof(T) == 2 ? RSA_BF16 : RSA_F32, pass);
  const int64_t heads = (int64_t)d.B * d.Z;
  for (int64_t h0 = 0; h0 < heads; h0 += pl.chunk) {
    Dims dc = d;  // (the tensors are dense)
    dc.B = 1; dc.Z = (int)(pl.chunk < heads - h0 ? pl.chunk : heads - h0);
    const void *in_c[6];
    void *tmp[3];
    for (int j = 0; j < 6; ++j) in_c[j] = static_cast<const char *>(in[j]) + (in[j] ? h0 * hb.in[j] : 0);
    for (int i = 0; i < 3; ++i) tmp[i] = ws + pl.out[i];
    RSA_TRY(pass_t<T>(dc, pass, in_c, tmp, ws, pl, st));
    for (int i = 0; i < 3; ++i)
      if (hb.out[i]) RSA_TRY(copy(tmp[i], static_cast<char *>(out[i]) + h0 * hb.out[i], dc.Z * hb.out[i], st));
  }
  return hipSuccess;
}

hipError_t run_pass(const Dims &d, int dtype, int pass, const void *const (&in)[6], void *const (&out)[3], char *ws,
                    size_t ws_bytes, hipStream_t st) {
  const int over = results_over_inputs(d, dtype, pass, in, out);
  StripPlan pl = strip_plan(d, dtype, pass);
  // In one pass O may lie over Q as it is: a work-group has read its own rows when it writes them, and no other reads them.
  const HeadBytes hb(d, dtype, pass);
  const size_t heads = (size_t)d.B * d.Z;
  auto over_q_alone = [&]() {
    return over == 1 && !overlap(out[0], heads * hb.out[0], in[1], heads * hb.in[1]) &&
           !overlap(out[0], heads * hb.out[0], in[2], heads * hb.in[2]);
  };
  if (over && !(pl.one_pass && over_q_alone())) {
    pl = apart_plan(d, dtype, pass, over == 2, ws_bytes);
    return dtype == RSA_BF16 ? pass_apart<uint16_t>(d, pass, in, out, ws, pl, st)
                             : pass_apart<float>(d, pass, in, out, ws, pl, st);
  }
  return dtype == RSA_BF16 ? pass_t<uint16_t>(d, pass, in, out, ws, pl, st) : pass_t<float>(d, pass, in, out, ws, pl, st);
}
#undef RSA_TRY

}  // namespace

size_t strip_workspace_bytes(const Dims &d, int dtype, int pass) {
  const StripPlan pl = strip_plan(d, dtype, pass);
  size_t usual = pl.total;
  const size_t apart = apart_plan(d, dtype, pass, false, 0).total;
  if (pl.one_pass) {  // (room for all results, so that O may lie over K or V in any way, but no more than strips would take)
    const size_t results = apart_plan(d, dtype, pass, true, 0).total, strips = strip_plan_by_rows(d, dtype, pass, true).total;
    usual = results < strips ? results : strips;
  }
  if (pl.keys) {  // (room for all results where every call was asked for as much by rows)
    const size_t keys = apart_plan(d, dtype, pass, pl, true, 0).total, least = apart_plan(d, dtype, pass, true, 0).total;
    const size_t results = keys <= pl.by_rows ? keys : least;
    if (results <= pl.by_rows && results > usual) usual = results;
  }
  return usual > apart ? usual : apart;
}

size_t strip_workspace_bytes(const Dims &d, int dtype, int pass, const void *const (&in)[6], void *const (&out)[3]) {
  const size_t any = strip_workspace_bytes(d, dtype, pass);  // (what is asked of every call)
  if (results_over_inputs(d, dtype, pass, in, out) < 2) return any;
  const size_t whole = apart_plan(d, dtype, pass, true, 0).total;
  return whole > any ? whole : any;
}

hipError_t strip_pass(const Dims &d, int dtype, int pass, const void *const (&in)[6], void *const (&out)[3], void *ws,
                      size_t ws_bytes, hipStream_t st) {
  return run_pass(d, dtype, pass, in, out, static_cast<char *>(ws), ws_bytes, st);
}

}  // namespace rsa
