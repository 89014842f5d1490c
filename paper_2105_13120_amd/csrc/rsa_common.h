// Shared device helpers for the RSA kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rsa.h"

namespace rsa {

typedef __bf16 bf16_t;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// D = A(32x16) * B(16x32) + C on the matrix core.  Lane l supplies
// A[l%32][(l/32)*8 .. +8] and B[(l/32)*8 .. +8][l%32]; it receives
// C[(v/4)*8 + (l/32)*4 + v%4][l%32] in element v of the accumulator.
__device__ __forceinline__ f32x16 mfma_32x32x16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Two fp32 -> packed bf16 (round to nearest even), low half = x.
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
  f32x2 v = {x, y};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// LDS transpose read (ds_read_b64_tr_b16).  Within each group of 16 lanes,
// lane j passes the address of 4 consecutive 16-bit elements ("row j/4,
// columns (j%4)*4 .. +4" of a 4 x 16 block); lane i receives column i of that
// block: element k of the result is element i%4 of the row passed by lane
// 4*k + i/4.
__device__ __forceinline__ u32x2 lds_read_tr16(const void *lds_ptr) {
  typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
  typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
  s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_ptr));
  return __builtin_bit_cast(u32x2, r);
}

// Direct 16-byte global->LDS load (global_load_lds_dwordx4): lane l of the wave fetches
// 16 bytes from its own global address and the hardware writes them to LDS at
// lds_base + 16 l; lds_base must be the same for the whole wave.  Completion is tracked
// by vmcnt: wait_vmem() before the barrier that publishes the data.
__device__ __forceinline__ void lds_dma16(const void *gsrc, void *lds_base) {
  typedef __attribute__((address_space(1))) const void *gptr_t;
  typedef __attribute__((address_space(3))) void *lptr_t;
  __builtin_amdgcn_global_load_lds((gptr_t)gsrc, (lptr_t)lds_base, 16, 0, 0);
}
// Same, 4 bytes per lane: lane l's dword lands at lds_base + 4 l.
__device__ __forceinline__ void lds_dma4(const void *gsrc, void *lds_base) {
  typedef __attribute__((address_space(1))) const void *gptr_t;
  typedef __attribute__((address_space(3))) void *lptr_t;
  __builtin_amdgcn_global_load_lds((gptr_t)gsrc, (lptr_t)lds_base, 4, 0, 0);
}
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)
// Waits for the direct loads in flight when exactly `STORES` newer stores were issued behind them (vmcnt counts both, in
// order of issue).
template <int STORES> __device__ __forceinline__ void wait_loads_before_stores() {
  static_assert(STORES < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (STORES & 15) | ((STORES >> 4) << 14));
}
// Work-group barrier that orders LDS alone: __syncthreads() also waits for every global store in flight, a trip to HBM
// per step of a loop that writes its results as it goes.  Direct loads need their own wait in front of it.
__device__ __forceinline__ void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// A direct global->LDS load (16 bytes per lane, landing at lds_base + 16 lane) that the compiler does not see: it
// would wait for every such load in flight before the next LDS read where the buffers of a ring are one object.
// The kernel orders them itself (wait_loads before the barrier that publishes them).  lane_off: bytes, taken as unsigned.
__device__ __forceinline__ void lds_dma16_unseen(const void *g, int lane_off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               : : "v"(lane_off), "s"(g), "s"(lds_base) : "m0");
}
// Same, from an address of each lane's own.
__device__ __forceinline__ void lds_dma16_unseen_far(const void *g, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(lds_base) : "m0");
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}
template <int N> __device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void barrier_only() { asm volatile("s_barrier" : : : "memory"); }

// Exchange between the two lanes l and l^32 (the two halves of a 32x32
// accumulator column).  v_permlane32_swap a, b swaps a[32..63] with b[0..31];
// with a = b = x on entry, lanes 0-31 end with (a, b) = (x[l], x[l+32]) and
// lanes 32-63 with (x[l-32], x[l]).  Written as inline asm because the
// compiler's builtin for this instruction folds its two results into one when
// both operands carry the same value.  The s_nop covers the wait states the
// instruction needs after a VALU write of its operands.
__device__ __forceinline__ void xhalf_pair(float x, float &lo, float &hi) {
  uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  lo = __builtin_bit_cast(float, a);
  hi = __builtin_bit_cast(float, b);
}
// v_permlane32_swap a, b in general: lanes 32..63 of a change places with lanes 0..31 of b.
// (Not volatile: the compiler may place it anywhere between its operands and its uses.)
__device__ __forceinline__ void permlane32_swap(uint32_t &a, uint32_t &b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float xhalf_max(float x) {
  float lo, hi;
  xhalf_pair(x, lo, hi);
  return fmaxf(lo, hi);
}
__device__ __forceinline__ float xhalf_sum(float x) {
  float lo, hi;
  xhalf_pair(x, lo, hi);
  return lo + hi;
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// Sum of load(s) over the splits s, always in the same order: the deterministic end of a split walk.  Eight loads are in
// flight at a time (one after the other, 64 splits of a small result took 16 us).  TREE: these eight are added in pairs, which
// rounds less than one after the other does.
template <bool TREE = false, class F>
__device__ __forceinline__ f32x4 sum_of_splits(int splits, F load) {
  f32x4 s = load(0);
  for (int k = 1; k < splits; k += 8) {
    f32x4 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = load(k + j < splits ? k + j : splits - 1);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (TREE && j > 0 && k + j >= splits) x[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (!TREE && k + j < splits) s += x[j];
    }
    if (TREE) s += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
  }
  return s;
}
constexpr int kReduceBlock = 64;  // (one wave: a small result is spread over more CUs)
inline dim3 reduce_grid(int64_t n4) { return dim3((unsigned)((n4 + kReduceBlock - 1) / kReduceBlock)); }

// Causal masks as bits: the lowest n (clamped to 0 .. 32) bits set, and x where bit `bit` of `mask` is set, -inf
// elsewhere (a field extract and a bitwise select: compares would each hold a pair of scalar registers,
// 64 of them at once, and spill everything else).
__device__ __forceinline__ uint32_t low_bits(int n) {
  return n <= 0 ? 0u : (n >= 32 ? ~0u : (1u << n) - 1u);
}
__device__ __forceinline__ float keep_bit(float x, uint32_t mask, int bit) {
  const uint32_t t = (uint32_t)((int32_t)(mask << (31 - bit)) >> 31);
  return __builtin_bit_cast(float, (t & __builtin_bit_cast(uint32_t, x)) | (~t & 0xff800000u));
}

// Division of a uniform x < 2^31 by a number that the host knows: the high half of a product, an add and a shift (the
// round-up method of Granlund and Montgomery, "Division by invariant integers using multiplication", 1994).  The
// division itself is 40 dependent vector instructions, and the prologues of the fused kernels held six to eight of them.
struct FastDiv {
  uint32_t d, mul, shift;
  __host__ __device__ uint32_t operator()(uint32_t x) const {
    return ((uint32_t)(((uint64_t)x * mul) >> 32) + x) >> shift;
  }
};
inline FastDiv make_fast_div(int64_t d) {  // 1 <= d < 2^31
  FastDiv f;
  f.d = (uint32_t)d; f.shift = d > 1 ? 32 - __builtin_clz(f.d - 1) : 0;
  f.mul = (uint32_t)((((((uint64_t)1 << f.shift) - f.d)) << 32) / f.d + 1);
  return f;
}

// Work-group id remap for the 8 XCDs: hardware hands consecutive work-group
// ids to XCDs round-robin, so id i runs on XCD i % 8.  Returns a logical id
// such that each XCD gets one contiguous range of logical ids (work-groups
// that share K/V then share that XCD's L2).  `n` must be the grid size.
// `rot` turns the assignment of ranges to XCDs: with a second grid dimension that
// repeats the ids (splits of a walk), rot = blockIdx.y lets every XCD take every
// range in turn, so ranges of unequal work (causal mask) do not load the XCDs unequally.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t id, uint32_t n, uint32_t rot = 0) {
  const uint32_t per = n >> 3;
  if (per == 0 || id >= per * 8) return id;  // tail keeps its id
  return ((id + rot) & 7) * per + (id >> 3);
}

// (head, tile) of a work-group under the causal mask, where the tiles of a head differ in work: all heads' longest
// tiles first, so that the short ones fill the chip's last rounds.  (Head after head, longest first within
// a head, leaves the last heads' long tiles to the end: B8 Z16 L2048, forward, 148 us; in this order 97.)  With
// a multiple of 8 heads the heads stay on their XCDs, since id % heads and the XCD id % 8 agree.
// rank: the tile's place among the head's, 0 = the most work.
__device__ __forceinline__ void longest_first(uint32_t id, const FastDiv &heads, uint32_t &head, uint32_t &rank) {
  rank = heads(id);
  head = id - rank * heads.d;
}
// Ends the life of everything a uniform value was computed from (scalar registers are scarce in these kernels).
__device__ __forceinline__ uint32_t settled(uint32_t x) {
  x = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(x));
  return x;
}

// Derived sizes of a validated descriptor, shared by host code and kernels.
struct Dims {
  int B, Z, A, N, rank_begin, rank_end, causal;
  int mode;    // RSA_MODE_FUSED or RSA_MODE_STAGED
  int zigzag;  // 1: rank n owns half-chunks n and 2N-1-n (RSA_OWN_ZIGZAG)
  int64_t L, c, Lq;
  float scale;
  int deterministic;  // RSA_DETERMINISTIC was asked for (every path is deterministic already)
  // element strides of (batch, head, row) for Q/dQ, K/V/dK/dV and O/dO; strided = any not dense
  int64_t qs[3], ks[3], os[3];
  int strided;
};

// Element offset of row 0 of flat head index head = b * Z + z in a tensor whose batch, head and
// row strides are st[0], st[1], st[2].
__host__ __device__ inline int64_t head_offset(int64_t head, int Z, const int64_t *st) {
  const uint32_t h = (uint32_t)head, b = h / (uint32_t)Z;  // (32 bits: a 64-bit division is a hundred instructions)
  return (int64_t)b * st[0] + (int64_t)(h - b * (uint32_t)Z) * st[1];
}

__host__ __device__ inline int64_t head_offset(uint32_t h, const FastDiv &Z, const int64_t *st) {
  const uint32_t b = Z(h);
  return (int64_t)b * st[0] + (int64_t)(h - b * Z.d) * st[1];
}

// Where a row of a strided output tensor lives, for kernels that walk (head, row) pairs flat:
// flat_row = head * rows_per_head + row.
struct OutLayout {
  int64_t st[3];
  FastDiv by_rows, by_Z;  // rows per head (flat rows are below 2^31), Z
  __host__ __device__ int64_t row_off(int64_t flat_row) const {
    const uint32_t r = (uint32_t)flat_row, h = by_rows(r);
    return head_offset(h, by_Z, st) + (int64_t)(r - h * by_rows.d) * st[2];
  }
};
inline OutLayout make_out_layout(const int64_t *st, int64_t rows_per_head, int Z) {
  OutLayout l;
  for (int k = 0; k < 3; ++k) l.st[k] = st[k];
  l.by_rows = make_fast_div(rows_per_head); l.by_Z = make_fast_div(Z);
  return l;
}

// Which global token a local query row is.  Contiguous ownership (the paper, section 3.1):
// rank n owns rows [n c, (n+1) c).  Zig-zag ownership: the sequence is cut into 2N
// half-chunks of h = c/2 rows and rank n owns half-chunks n and 2N-1-n, stored in that
// order, so that under the causal mask every rank sees the same number of keys.
// h is a multiple of 64: the 64 rows of a tile are consecutive tokens in both layouts.
struct RowMap {
  int64_t q0, c, h;
  FastDiv by_c, by_h;
  int rb, last_half;  // first simulated rank; 2N - 1
  int zigzag;
  int first, q1, last_row;  // see row_at: rows of the first run, first token of the second; zig-zag: Lq - h
  // (rows and tokens are below 2^31: one head's K and V of that many would not fit the memory)
  __host__ __device__ int64_t operator()(int64_t r) const {
    if (!zigzag) return q0 + r;
    const uint32_t q = by_c((uint32_t)r);
    const int64_t rho = rb + (int64_t)q, w = r - (int64_t)q * c;
    return w < h ? rho * h + w : (last_half - rho) * h + (w - h);
  }
  // The rows in the order of their tokens, which the causal kernels take them in: the v-th row's token, its place in the
  // tensors, the rank that owns it.  Under zig-zag ownership the simulated ranks' earlier half-chunks are one run of
  // tokens and their later ones, in reverse, a second; 64 rows from a multiple of 64 on are rows of one half-chunk.
  // (Tiles cut from the rows as they lie straddle a rank's two half-chunks, one of few keys and one of many, and have no
  // order by length where h is no multiple of them.  Forward and backward, us: 36 heads of 7680 rows, h = 320, 1453 -> 1232;
  // 70 of 1536, h = 64, 176 -> 141; 70 of 384, h = 64, 28.8 -> 26.8.)
  __host__ __device__ int token_at(int v) const { return v < first ? (int)q0 + v : q1 + (v - first); }
  __host__ __device__ int64_t row_at(int v) const {
    if (!zigzag) return v;
    const int u = v < first ? v : v - first, hc = (int)by_h((uint32_t)u), w = u - hc * (int)h;
    return v < first ? (int64_t)hc * c + w : (int64_t)last_row - (int64_t)hc * c + w;
  }
  __host__ __device__ int rank_at(int v) const {
    if (!zigzag) return rb + (int)by_c((uint32_t)v);
    return v < first ? rb + (int)by_h((uint32_t)v) : last_half - (int)by_h((uint32_t)token_at(v));
  }
  // the first v of a token at or after g
  __host__ __device__ int from_token(int g) const {
    if (g < (int)q0 + first) return g > (int)q0 ? g - (int)q0 : 0;
    return zigzag && g > q1 ? first + (g - q1) : first;
  }
  // first key of the rows [w, ...) of the chunk (pair of half-chunks) that rank j owns
  __host__ __device__ int64_t key_of(int j, int64_t w) const {
    if (!zigzag) return (int64_t)j * c + w;
    return w < h ? (int64_t)j * h + w : (int64_t)(last_half - j) * h + (w - h);
  }
  // rank that owns global token g
  __host__ __device__ int owner(int64_t g) const {
    if (!zigzag) return (int)by_c((uint32_t)g);
    const int hc = (int)by_h((uint32_t)g);
    return hc <= last_half / 2 ? hc : last_half - hc;
  }
};
inline RowMap make_row_map(const Dims &d) {
  RowMap m;
  m.q0 = (int64_t)d.rank_begin * d.c; m.c = d.c; m.h = d.c / 2;
  m.by_c = make_fast_div(d.c); m.by_h = make_fast_div(m.h > 0 ? m.h : 1);
  m.rb = d.rank_begin; m.last_half = 2 * d.N - 1; m.zigzag = d.zigzag;
  const int64_t rows = (int64_t)(d.rank_end - d.rank_begin) * d.c;
  m.first = d.zigzag ? (int)(rows / 2) : 0x7fffffff - (int)m.q0; m.q1 = d.zigzag ? (int)((2 * d.N - d.rank_end) * m.h) : 0;
  m.last_row = (int)(rows - m.h);
  if (d.zigzag) m.q0 = (int64_t)d.rank_begin * m.h;
  return m;
}

// The ring walk of the forward and dQ kernels over a head's keys: ring step t of rank n visits chunk (n - t) mod N in
// stages of 2^lg keys, numbered t * spc + ks.  Only stages with a key at or before token q_last count under the
// causal mask; within a chunk they are its first `cnt`, since its keys (also the two half-chunks of zig-zag
// ownership) come in ascending order.  A walk is moved by adding to ks and, past cnt, going on to the next chunk: a
// few scalar instructions a step.  (Testing stage after stage took 1150 cycles of a stage's 3100 with four groups of
// waves, 300 of 2300 with two; forward and backward of 18 heads of 1728 causal rows 81.6 -> 71.8 us, of 2 heads of 512
// 27.7 -> 25.4, of one rank's 4096 rows against 65536 keys 3534 -> 3461.)
template <bool CAUSAL>
struct KeyWalk {
  int n, N, c, h, last_half, spc, sph, lg, q_last, f_end;  // (sph: stages of a chunk's first run of keys)
  int t, ks, cnt, lo, hi;  // lo, hi: key of stage ks is (ks < sph ? lo : hi) + (ks << lg)
  bool have;
  __host__ __device__ __forceinline__ int seen(int first, int most) const {  // stages of a run that starts at key `first`
    if (q_last < first) return 0;
    const int k = ((q_last - first) >> lg) + 1;
    return k < most ? k : most;
  }
  __host__ __device__ __forceinline__ void chunk() {
    int j = n - t;
    if (j < 0) j += N;
    if (h == 0) {
      lo = hi = j * c;
      cnt = CAUSAL ? seen(lo, spc) : spc;
    } else {
      lo = j * h;
      const int second = (last_half - j) * h;
      hi = second - h;
      cnt = CAUSAL ? seen(lo, sph) : spc;
      if (CAUSAL && cnt == sph) cnt += seen(second, spc - sph);
    }
    if (f_end - t * spc < cnt) cnt = f_end - t * spc;
  }
  // n_: rank of the first row; lg_: log2 of a stage's keys; splits, split: the share of the stages this walk takes
  __host__ __device__ __forceinline__ void begin(const RowMap &m, int n_, int N_, int lg_, int q_last_, int splits, int split) {
    n = n_; N = N_; lg = lg_; q_last = q_last_; last_half = m.last_half;
    // Rows of their ranks' tokens in one run see nothing behind the last row's chunk: the ring ends there, in the same order.
    // Going through the chunks behind it took 0.2 us each with few work-groups on a CU, 0.6 with many (forward of the first 64 of
    // 4096 rows, us: 64 heads 20.0 -> 5.5, 520 42.5 -> 9.3).  A split's stages are numbered over all chunks.
    if (CAUSAL && !m.zigzag && splits == 1) {
      const int last = (int)m.by_c((uint32_t)q_last);
      N = (last > n ? last : n) + 1;
    }
    c = (int)m.c; h = m.zigzag ? (int)m.h : 0;
    spc = c >> lg; sph = m.zigzag ? h >> lg : spc;
    t = 0; ks = 0; f_end = N * spc; have = true;
    if (splits > 1) {
      const int per = (int)((uint32_t)(f_end + splits - 1) / (uint32_t)splits), b = split * per;
      f_end = b + per < f_end ? b + per : f_end;
      t = (int)((uint32_t)b / (uint32_t)spc);
      ks = b - t * spc;
      have = b < f_end;
    }
    if (have) { chunk(); ks = ks < cnt ? ks : cnt; skip(0); }  // (a split may start behind a chunk's last stage)
  }
  __host__ __device__ __forceinline__ void skip(int stages) {  // that many stages further on; have: there is such a stage
    if (!have) return;
    ks += stages;
    while (ks >= cnt) {
      ks -= cnt; ++t;
      if (t * spc >= f_end) { have = false; return; }
      chunk();
    }
  }
  __host__ __device__ __forceinline__ int key() const { return (ks < sph ? lo : hi) + (ks << lg); }
};

}  // namespace rsa
