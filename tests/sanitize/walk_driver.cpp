// The scalar arithmetic of the fused kernels' walks, on the host: KeyWalk against the list of stages written out
// chunk by chunk, FastDiv against the division.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "rsa_common.h"

static std::mt19937_64 rng(1);
static int pick(int lo, int hi) { return lo + (int)(rng() % (uint64_t)(hi - lo + 1)); }

// first keys of the stages of one split, in the order of the walk
static std::vector<int> stages(const rsa::RowMap &m, int n, int N, int keys, int q_last, bool causal, int splits, int split) {
  const int spc = (int)m.c / keys, all = N * spc, per = (all + splits - 1) / splits;
  std::vector<int> out;
  for (int f = split * per; f < all && f < (split + 1) * per; ++f) {
    const int j = (n - f / spc + N) % N, k = (int)m.key_of(j, (int64_t)(f % spc) * keys);
    if (!causal || k <= q_last) out.push_back(k);
  }
  return out;
}

template <bool CAUSAL>
static int check_walk(const rsa::RowMap &m, int n, int N, int lg, int q_last, int splits, int split, int groups) {
  const std::vector<int> want = stages(m, n, N, 1 << lg, q_last, CAUSAL, splits, split);
  for (int g = 0; g < groups; ++g) {
    rsa::KeyWalk<CAUSAL> w;
    w.begin(m, n, N, lg, q_last, splits, split);
    w.skip(g);
    for (size_t i = g; i < want.size(); i += groups, w.skip(groups))
      if (!w.have || w.key() != want[i]) return 1;
    if (w.have) return 1;
    // chunks behind the last one that any row sees take no steps
    const int last = q_last / (int)m.c;
    if (CAUSAL && !m.zigzag && splits == 1 && w.N != (last > n ? last : n) + 1) return 1;
  }
  return 0;
}

// The rows in the order of their tokens: each once, 64 at a time in one run, as RowMap says whose token and rank they are.
static int check_row_order(const rsa::RowMap &m, const rsa::Dims &d) {
  const int rows = (d.rank_end - d.rank_begin) * (int)d.c;
  std::vector<char> seen((size_t)rows, 0);
  int last = -1;
  for (int v = 0; v < rows; ++v) {
    const int64_t r = m.row_at(v);
    if (r < 0 || r >= rows || seen[(size_t)r] || (v % 64 && r != m.row_at(v - 1) + 1)) return 1;
    seen[(size_t)r] = 1;
    const int g = m.token_at(v);
    if (g != (int)m(r) || g <= last || m.rank_at(v) != m.owner(g) || m.rank_at(v) != d.rank_begin + (int)(r / d.c)) return 1;
    for (int key = last + 1; key <= g; ++key)
      if (m.from_token(key) != v) return 1;
    last = g;
  }
  return m.from_token(last + 1) < rows;
}

int main() {
  int bad = 0;
  for (int it = 0; it < 20000 && !bad; ++it) {
    rsa::Dims d{};
    d.zigzag = pick(0, 1);
    d.N = pick(1, 12);
    d.c = 64 * pick(1, 10) * (d.zigzag ? 2 : 1);
    d.L = d.N * d.c;
    d.rank_begin = pick(0, d.N - 1); d.rank_end = pick(d.rank_begin + 1, d.N);
    const rsa::RowMap m = rsa::make_row_map(d);
    const int64_t run = d.zigzag ? d.c / 2 : d.c;
    const int lg = run % 128 == 0 ? pick(6, 7) : 6, n = pick(0, d.N - 1), splits = pick(0, 1) ? 1 : pick(1, 6);
    const int q_last = pick(0, (int)d.L - 1), split = pick(0, splits - 1), groups = 1 << pick(0, 2);
    if (it < 2000) bad |= check_row_order(m, d);
    bad |= check_walk<true>(m, n, d.N, lg, q_last, splits, split, groups);
    bad |= check_walk<false>(m, n, d.N, lg, q_last, splits, split, groups);
    if (bad) std::fprintf(stderr, "walk %d failed\n", it);
  }
  for (int it = 0; it < 200000 && !bad; ++it) {
    const uint32_t d = it < 4096 ? (uint32_t)it + 1 : (uint32_t)(rng() >> (33 + rng() % 28)) | 1;
    const rsa::FastDiv f = rsa::make_fast_div(d);
    const uint32_t r = (uint32_t)(rng() >> (33 + rng() % 28)), edge = (uint32_t)((0x7fffffffu / d) * (uint64_t)d);
    for (const uint32_t x : {0u, d - 1, d, r, r / d * d, r / d * d + d - 1, edge - 1, edge, 0x7fffffffu})
      if (x < 0x80000000u && f(x) != x / d) bad = 1;
    if (bad) std::fprintf(stderr, "division by %u failed\n", d);
  }
  std::printf(bad ? "WALKS_FAILED\n" : "WALKS_OK\n");
  return bad;
}
