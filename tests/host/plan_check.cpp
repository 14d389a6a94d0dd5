// Host-only property check of the planner (plan.cpp) and the bit allocation
// (alloc.cpp): packed layouts of random valid block lists, the statuses of
// invalid ones, the decode-GEMV work split (every chunk of a layer covered by
// exactly one wave, each wave inside one block and starting on one of its
// group boundaries, LDS within the work-group budget), the decode grid of a
// batch, the prefill launch's token tiles and splits, and the allocation's
// outputs (palette bit-widths, the budget never exceeded by waterfilling,
// counts on the quantum after matching, a permutation from clustering).
// Built with g++ and the address and undefined-behaviour sanitizers by
// tests/test_host_sanitizer.py; exits non-zero on the first violated
// property.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "internal.h"

namespace {

int g_fail = 0;

#define CHECK(cond, ...)                                  \
  do {                                                    \
    if (!(cond)) {                                        \
      fprintf(stderr, "FAIL %s:%d: %s: ", __FILE__, __LINE__, #cond); \
      fprintf(stderr, __VA_ARGS__);                       \
      fprintf(stderr, "\n");                              \
      ++g_fail;                                           \
      return;                                             \
    }                                                     \
  } while (0)

// splitmix64 (Steele, Lea and Flood 2014): a seeded, portable stream
struct Rng {
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  int uniform(int lo, int hi) { return lo + static_cast<int>(next() % static_cast<uint64_t>(hi - lo + 1)); }
};

const int kPalette[5] = {2, 3, 4, 8, 16};

// A random valid block list: a random ascending subset of the palette, each
// block a positive multiple of 32 channels.
int random_blocks(Rng& r, int max_units, polyq_block* b) {
  int nb = 0;
  for (int i = 0; i < 5; ++i)
    if (r.next() % 2) b[nb++] = polyq_block{kPalette[i], 0};
  if (nb == 0) b[nb++] = polyq_block{kPalette[r.uniform(0, 4)], 0};
  for (int i = 0; i < nb; ++i) b[i].len = 32 * r.uniform(1, max_units);
  return nb;
}

void check_layout(const polyq_layout& L, const polyq_block* b, int nb, int n, int k) {
  CHECK(L.n == n && L.k == k && L.nblocks == nb, "header");
  CHECK(L.n_tiles == (n + 63) / 64 && L.n_chunks == k / 32, "tiles %d chunks %d", L.n_tiles, L.n_chunks);
  int64_t off = 0, bits = 0;
  int k0 = 0, g0 = 0;
  for (int i = 0; i < nb; ++i) {
    const int64_t ng = (b[i].len + 127) / 128, nch = b[i].len / 32;
    const int64_t meta = b[i].bits <= 8 ? 256 : 0;
    CHECK(L.block[i].bits == b[i].bits && L.block[i].len == b[i].len, "block %d", i);
    CHECK(L.k_begin[i] == k0 && L.group_begin[i] == g0, "block %d begins", i);
    CHECK(L.block_offset[i] == off && off % 256 == 0, "block %d offset %lld", i, (long long)L.block_offset[i]);
    CHECK(L.tile_bytes[i] == ng * meta + nch * 64 * 4 * b[i].bits && L.tile_bytes[i] % 256 == 0,
          "block %d tile bytes %lld", i, (long long)L.tile_bytes[i]);
    off += static_cast<int64_t>(L.n_tiles) * L.tile_bytes[i];
    k0 += b[i].len;
    if (b[i].bits <= 8) g0 += static_cast<int>(ng);
    bits += static_cast<int64_t>(n) * b[i].bits * b[i].len;
  }
  CHECK(L.packed_bytes == off && L.n_groups == g0 && L.code_bits == bits, "totals");
  CHECK(L.weight_bytes == bits / 8 + static_cast<int64_t>(n) * g0 * 4, "weight bytes");
  CHECK(polyq::layout_is_valid(&L), "a planned layout is valid");
  polyq_layout bad = L;
  bad.packed_bytes += 256;
  CHECK(!polyq::layout_is_valid(&bad), "a changed layout is not valid");
}

// The decode split for m tokens: coverage, block and group alignment, budgets.
void check_gemv_plan(const polyq_layout& L, int m, int launch_tiles) {
  polyq::GemvPlan p;
  CHECK(polyq::plan_gemv(L, m, launch_tiles, &p) == 0, "no plan for k=%d m=%d", L.k, m);
  CHECK(p.W == 4 && p.S >= 1 && p.S * p.W <= polyq::kMaxSplitEntries, "S=%d W=%d", p.S, p.W);
  int sum = 0;
  for (int i = 0; i < L.nblocks; ++i) {
    CHECK(p.waves[i] >= 1, "block %d has no wave", i);
    sum += p.waves[i];
  }
  CHECK(sum <= p.S * p.W, "waves %d > %d", sum, p.S * p.W);
  const polyq::LayoutBlocks blk{&L, p.waves};
  std::vector<int> seen(L.n_chunks, 0), widest(L.nblocks, 0);
  int worst = 0;
  for (int w = 0; w < p.S * p.W; ++w) {
    int a = 0, b = 0, bi = -2;
    polyq::wave_range(w, L.nblocks, L.n_chunks, blk, &a, &b, &bi);
    CHECK(0 <= a && a <= b && b <= L.n_chunks, "wave %d range [%d, %d)", w, a, b);
    if (a == b) continue;
    CHECK(bi >= 0 && bi < L.nblocks, "wave %d block %d", w, bi);
    const int cb = L.k_begin[bi] / 32, ce = cb + L.block[bi].len / 32;
    CHECK(cb <= a && b <= ce, "wave %d leaves block %d", w, bi);
    CHECK((a - cb) % 4 == 0 && (b == ce || (b - cb) % 4 == 0), "wave %d not on group boundaries", w);
    for (int c = a; c < b; ++c) ++seen[c];
    worst = b - a > worst ? b - a : worst;
    widest[bi] = b - a > widest[bi] ? b - a : widest[bi];
  }
  // no wave has more of a block than an even split of its groups has to give
  // one of them; a single group too many is the partial one, where that saves more
  // than an eighth of the share
  for (int i = 0; i < L.nblocks; ++i) {
    const int nch = L.block[i].len / 32, groups = (nch + 3) / 4, q = groups / p.waves[i], r = groups % p.waves[i];
    const int partial = 4 * q + (nch + 3) % 4 + 1;
    const int most = r == 1 && 8 * (4 * (q + 1) - partial) > 4 * (q + 1) ? partial : r > 0 ? 4 * (q + 1) : 4 * q;
    CHECK(widest[i] <= most, "block %d of %d chunks over %d waves: %d chunks in one", i, nch, p.waves[i], widest[i]);
  }
  for (int c = 0; c < L.n_chunks; ++c) CHECK(seen[c] == 1, "chunk %d covered %d times (m=%d)", c, seen[c], m);
  CHECK(worst == p.lds_chunks, "lds_chunks %d, widest range %d", p.lds_chunks, worst);
  CHECK(polyq::gemv_lds_bytes(p, m) <= 80 * 1024, "LDS %zu", polyq::gemv_lds_bytes(p, m));
  const size_t ws = polyq_gemv_workspace_bytes(&L, m);
  CHECK(ws >= polyq::gemv_workspace_for(L, m, p) || launch_tiles != L.n_tiles, "workspace %zu", ws);
}

// The decode grid of a batch: every tile and split of every linear is reached by
// exactly one work-group, and no more are launched than `count` times the widest
// linear's (items of different n and k may not multiply each other's extremes).
void check_gemv_grid(Rng& r) {
  const int count = r.uniform(1, POLYQ_MAX_BATCH), m = r.uniform(1, 16);
  const int alike = r.uniform(0, 2);  // 1: equal linears, 2: of one input (n differs)
  std::vector<polyq_layout> L(count);
  int launch_tiles = 0;
  for (int i = 0; i < count; ++i) {
    if (i > 0 && alike) {
      CHECK(polyq_plan(alike == 1 ? L[0].n : r.uniform(1, 9000), L[0].k, L[0].block, L[0].nblocks, &L[i]) == POLYQ_OK, "plan");
    } else {
      polyq_block b[POLYQ_MAX_BLOCKS];
      const int nb = random_blocks(r, r.next() % 4 ? 8 : 300, b);
      int k = 0;
      for (int j = 0; j < nb; ++j) k += b[j].len;
      CHECK(polyq_plan(r.next() % 4 ? r.uniform(1, 700) : r.uniform(1, 30000), k, b, nb, &L[i]) == POLYQ_OK, "plan");
    }
    launch_tiles += L[i].n_tiles;
  }
  int32_t tiles[POLYQ_MAX_BATCH], splits[POLYQ_MAX_BATCH];
  int64_t widest = 0, all = 0;
  for (int i = 0; i < count; ++i) {
    polyq::GemvPlan p;
    CHECK(polyq::plan_gemv(L[i], m, launch_tiles, &p) == 0, "no plan");
    tiles[i] = L[i].n_tiles;
    splits[i] = p.S;
    widest = widest > static_cast<int64_t>(tiles[i]) * p.S ? widest : static_cast<int64_t>(tiles[i]) * p.S;
    all += static_cast<int64_t>(tiles[i]) * p.S;
  }
  const polyq::GemvGrid g = polyq::gemv_grid(tiles, splits, count);
  const int64_t launched = static_cast<int64_t>(g.x) * g.y * g.z;
  CHECK(g.x >= 1 && g.y == (g.joint ? 1 : count) && launched >= all && launched <= (g.joint ? all : g.z > 1 ? all + polyq::kCUs : widest * count),
        "grid %d x %d x %d for %lld work-groups, widest linear %lld", g.x, g.y, g.z, (long long)all, (long long)widest);
  for (int i = 0; i < count; ++i) {
    std::vector<int> seen(static_cast<size_t>(tiles[i]) * splits[i], 0);
    const uint32_t magic = polyq::div_magic(static_cast<uint32_t>(tiles[i]));
    for (int z = 0; z < g.z; ++z)
      for (int x0 = 0; x0 < g.x; ++x0) {
        int tile = -1, s = -1, x = x0;
        if (g.joint) {  // the last linear that begins at or before x
          int linear = 0;
          for (int j = 1; j < POLYQ_MAX_BATCH; ++j) linear += g.first_tile[j] <= x ? 1 : 0;
          if (linear != i) continue;
          CHECK((i > 0) == (x >= g.x_end[0]), "x %d, linear %d, x_end %d", x, i, g.x_end[0]);
          x -= g.first_tile[i];
        } else if (x >= g.x_end[i]) {
          continue;
        }
        polyq::gemv_place(static_cast<uint32_t>(x), static_cast<uint32_t>(z), magic, tiles[i], &tile, &s);
        CHECK(tile >= 0 && tile < tiles[i] && s >= 0 && s < splits[i], "tile %d of %d, split %d", tile, tiles[i], s);
        ++seen[static_cast<size_t>(s) * tiles[i] + tile];
      }
    for (size_t j = 0; j < seen.size(); ++j) CHECK(seen[j] == 1, "linear %d: place %zu reached %d times", i, j, seen[j]);
  }
}

// The grid form of the launches that tests/test_gpu_gemv.py runs (its GRIDS): rows of
// each linear, k, the form.
void check_grid_forms() {
  enum Form { kFlat, kBySplit, kJoint };
  struct {
    int count, n[3], k[3];
    Form form;
  } const cases[] = {
      {3, {4096, 1024, 1000}, {2048, 2048, 2048}, kJoint}, {3, {1000, 4096, 65}, {2048, 2048, 2048}, kJoint},
      {3, {2048, 2048, 2048}, {2048, 2048, 2048}, kBySplit}, {3, {400, 64, 30}, {2048, 2048, 2048}, kBySplit},
      {2, {13824, 13800, 0}, {1024, 1024, 0}, kFlat}, {3, {4096, 64, 130}, {1024, 20480, 2048}, kFlat},
  };
  for (const auto& c : cases)
    for (int m = 1; m <= 5; m += 4) {
      int32_t tiles[3], splits[3], launch_tiles = 0;
      polyq_layout L[3];
      for (int i = 0; i < c.count; ++i) {
        const int unit = (c.k[i] - 32) / 32, b2 = unit * 45 / 100 | 1, b3 = unit * 35 / 100 | 1, b4 = unit * 15 / 100 | 1;
        const polyq_block b[5] = {{2, 32 * b2}, {3, 32 * b3}, {4, 32 * b4}, {8, 32 * (unit - b2 - b3 - b4)}, {16, 32}};
        CHECK(polyq_plan(c.n[i], c.k[i], b, 5, &L[i]) == POLYQ_OK, "plan n=%d k=%d", c.n[i], c.k[i]);
        launch_tiles += L[i].n_tiles;
      }
      for (int i = 0; i < c.count; ++i) {
        polyq::GemvPlan p;
        CHECK(polyq::plan_gemv(L[i], m, launch_tiles, &p) == 0, "no plan");
        tiles[i] = L[i].n_tiles;
        splits[i] = p.S;
      }
      const polyq::GemvGrid g = polyq::gemv_grid(tiles, splits, c.count);
      const Form form = g.joint ? kJoint : g.z > 1 ? kBySplit : kFlat;
      CHECK(form == c.form, "n=%d, %d linears, m=%d: form %d, not %d", c.n[0], c.count, m, form, c.form);
    }
}

// Prefill launches: token tiles of a work-group and K splits.
struct GemmForm {
  int n, m, blocks;  // blocks: index into kGemmBlocks
  int nt;
  bool split;
};
const polyq_block kGemmBlocks[][5] = {{{2, 1440}, {3, 1472}, {4, 1504}, {8, 1536}, {16, 416}},
                                      {{2, 416}, {3, 448}, {4, 480}, {8, 512}, {16, 416}},
                                      {{2, 1376}, {3, 2048}, {4, 2400}, {8, 992}, {16, 64}},
                                      {{2, 160}, {3, 256}, {4, 288}, {8, 96}, {16, 32}}};
polyq::GemmShape gemm_shape_of(int n, int m, int blocks) {
  const polyq_block* b = kGemmBlocks[blocks];
  polyq_layout L;
  const polyq_layout* l = &L;
  if (polyq_plan(n, b[0].len + b[1].len + b[2].len + b[3].len + b[4].len, b, 5, &L) != POLYQ_OK) return {};
  return polyq::gemm_shape(&l, 1, m, polyq::kGemmMaxSplits);
}
// The forms that tests/test_gpu_gemm.py runs (its GEMM_FORMS).
void check_gemm_forms() {
  const GemmForm forms[] = {
      {2051, 11, 0, 1, true},  {1157, 183, 0, 2, true}, {1157, 337, 0, 3, true}, {2051, 374, 0, 4, true},
      {2051, 449, 0, 5, true}, {3205, 361, 0, 6, true}, {3205, 321, 0, 7, true}, {3205, 481, 0, 8, true},
      {40963, 3, 1, 1, false}, {3205, 577, 1, 2, false}, {5381, 401, 1, 3, false}, {5381, 529, 1, 4, false},
      {8195, 449, 1, 5, false}, {8195, 561, 1, 6, false}, {12805, 481, 1, 7, false}, {12805, 561, 1, 8, false}};
  for (const auto& f : forms) {
    const polyq::GemmShape s = gemm_shape_of(f.n, f.m, f.blocks);
    CHECK(s.nt == f.nt && (s.splits > 1) == f.split, "n=%d m=%d: %d token tiles, %d splits", f.n, f.m, s.nt, s.splits);
  }
  // Splits pay for the sum launch and their partial sums' way to memory and back: not
  // 13 of them for 111 tokens x 3149 rows x 6880 channels (45.3 us; 39.9 with the
  // kernel of one 256-token tile; 4 token tiles and 8 splits: less than either), and
  // none for 164 tokens x 14307 rows x 832 channels (35.0 us in two, 25.4 in one).
  polyq::GemmShape s = gemm_shape_of(3149, 111, 2);
  CHECK(s.splits > 1 && s.splits <= 8, "%d token tiles, %d splits", s.nt, s.splits);
  s = gemm_shape_of(14307, 164, 3);
  CHECK(s.splits == 1, "%d token tiles, %d splits", s.nt, s.splits);
}
// Any launch: its tokens covered by work-groups that all have some, no more splits than
// given or than half the groups, more than one only within one round.
void check_gemm_shape(Rng& r) {
  const int count = r.uniform(1, POLYQ_MAX_BATCH), m = r.next() % 2 ? r.uniform(1, 300) : r.uniform(1, 100000);
  const int most = r.uniform(1, polyq::kGemmMaxSplits);
  std::vector<polyq_layout> L(count);
  const polyq_layout* l[POLYQ_MAX_BATCH];
  int64_t rows = 0;
  int groups = 0;
  for (int i = 0; i < count; ++i) {
    polyq_block b[POLYQ_MAX_BLOCKS];
    const int nb = random_blocks(r, r.next() % 4 ? 8 : 300, b);
    int k = 0;
    for (int j = 0; j < nb; ++j) k += b[j].len;
    CHECK(polyq_plan(r.next() % 4 ? r.uniform(1, 700) : r.uniform(1, POLYQ_MAX_N), k, b, nb, &L[i]) == POLYQ_OK, "plan");
    l[i] = &L[i];
    rows += (L[i].n_tiles + 3) / 4;
    groups = std::max(groups, polyq::layout_groups(L[i]));
  }
  const polyq::GemmShape s = polyq::gemm_shape(l, count, m, most);
  const int64_t tiles = (static_cast<int64_t>(m) + 15) / 16;
  CHECK(s.nt >= 1 && s.nt <= polyq::kGemmMaxNT && s.nt * static_cast<int64_t>(s.m_tiles) >= tiles &&
            s.nt * (s.m_tiles - 1ll) < tiles, "m=%d: %d x %d token tiles", m, s.m_tiles, s.nt);
  CHECK(s.splits >= 1 && s.splits <= most && (s.splits == 1 || (2 * s.splits <= groups && rows * s.m_tiles * s.splits <= polyq::kCUs)),
        "%d splits of %d groups, %lld row blocks, %d token tiles", s.splits, groups, (long long)rows, s.m_tiles);
}

void check_invalid() {
  polyq_layout L;
  polyq_block ok[2] = {{2, 64}, {16, 64}};
  CHECK(polyq_plan(64, 128, nullptr, 2, &L) == POLYQ_ERR_ARG, "null blocks");
  CHECK(polyq_plan(64, 128, ok, 2, nullptr) == POLYQ_ERR_ARG, "null out");
  CHECK(polyq_plan(64, 128, ok, 0, &L) == POLYQ_ERR_ARG, "no blocks");
  CHECK(polyq_plan(64, 128, ok, POLYQ_MAX_BLOCKS + 1, &L) == POLYQ_ERR_ARG, "too many blocks");
  CHECK(polyq_plan(0, 128, ok, 2, &L) == POLYQ_ERR_SHAPE, "n = 0");
  CHECK(polyq_plan(POLYQ_MAX_N + 1, 128, ok, 2, &L) == POLYQ_ERR_SHAPE, "n too large");
  CHECK(polyq_plan(64, POLYQ_MAX_K + 32, ok, 2, &L) == POLYQ_ERR_SHAPE, "k too large");
  CHECK(polyq_plan(64, 160, ok, 2, &L) == POLYQ_ERR_SHAPE, "sum != k");
  polyq_block desc[2] = {{4, 64}, {2, 64}};
  CHECK(polyq_plan(64, 128, desc, 2, &L) == POLYQ_ERR_BITS, "descending bits");
  polyq_block dup[2] = {{4, 64}, {4, 64}};
  CHECK(polyq_plan(64, 128, dup, 2, &L) == POLYQ_ERR_BITS, "repeated bits");
  polyq_block five[1] = {{5, 128}};
  CHECK(polyq_plan(64, 128, five, 1, &L) == POLYQ_ERR_BITS, "5 bits");
  polyq_block odd[2] = {{2, 48}, {16, 80}};
  CHECK(polyq_plan(64, 128, odd, 2, &L) == POLYQ_ERR_QUANTUM, "not a multiple of 32");
  polyq_block neg[2] = {{2, -32}, {16, 160}};
  CHECK(polyq_plan(64, 128, neg, 2, &L) == POLYQ_ERR_QUANTUM, "negative length");
  for (int s = -2; s < 10; ++s) CHECK(polyq_status_str(static_cast<polyq_status>(s)) != nullptr, "status %d", s);
  CHECK(polyq_gemv_workspace_bytes(nullptr, 1) == 0, "null layout");
  polyq_block one[1] = {{3, 256}};
  CHECK(polyq_plan(64, 256, one, 1, &L) == POLYQ_OK, "plan");
  CHECK(polyq_gemv_workspace_bytes(&L, 0) == 0 && polyq_gemv_workspace_bytes(&L, POLYQ_MAX_M_GEMV + 1) == 0,
        "m out of range");
}

void check_alloc(Rng& r, int iter) {
  const int n = r.uniform(1, 40), k = 32 * r.uniform(1, 40);
  std::vector<float> w(static_cast<size_t>(n) * k), s(k);
  std::vector<double> x2(k), err(static_cast<size_t>(POLYQ_NUM_BITS) * k);
  for (auto& v : w) v = static_cast<float>((static_cast<int64_t>(r.next() % 2001) - 1000) * 2e-5);
  for (int j = 0; j < k; ++j) {
    x2[j] = 1.0 + static_cast<double>(r.next() % 1000);
    s[j] = 0.5f + static_cast<float>(r.next() % 100) / 50.0f;
  }
  CHECK(polyq_channel_error(w.data(), n, k, x2.data(), iter % 2 ? s.data() : nullptr, err.data()) == POLYQ_OK,
        "channel_error");
  for (int j = 0; j < k; ++j) CHECK(err[4 * static_cast<size_t>(k) + j] == 0.0 && err[j] >= 0.0, "E_16 = 0, E >= 0");
  const double budget = 2.0 + static_cast<double>(r.next() % 1400) / 100.0;
  std::vector<int32_t> bits(k), perm(k);
  CHECK(polyq_waterfill(err.data(), k, budget, bits.data()) == POLYQ_OK, "waterfill");
  int64_t sum = 0;
  for (int j = 0; j < k; ++j) sum += bits[j];
  CHECK(sum <= static_cast<int64_t>(nearbyint(budget * k)) || sum == 2 * k, "budget exceeded: %lld", (long long)sum);
  int32_t counts[POLYQ_NUM_BITS];
  CHECK(polyq_quanta_match(err.data(), k, 32, budget, bits.data(), counts) == POLYQ_OK, "quanta_match");
  int32_t total = 0;
  for (int i = 0; i < POLYQ_NUM_BITS; ++i) {
    CHECK(counts[i] % 32 == 0, "count %d off the quantum", counts[i]);
    total += counts[i];
  }
  CHECK(total == k, "counts sum to %d, k %d", total, k);
  polyq_block blocks[POLYQ_MAX_BLOCKS];
  int32_t nb = 0;
  CHECK(polyq_cluster(bits.data(), k, perm.data(), blocks, &nb) == POLYQ_OK, "cluster");
  std::vector<int> seen(k, 0);
  for (int j = 0; j < k; ++j) ++seen[perm[j]];
  for (int j = 0; j < k; ++j) CHECK(seen[j] == 1, "perm is not a permutation");
  polyq_layout L;
  CHECK(polyq_plan(n, k, blocks, nb, &L) == POLYQ_OK, "clustered blocks plan");
  // Eq. 8 scales on the final bit map: powers of two, 16-bit channels at 1
  std::vector<double> sal(k);
  for (int j = 0; j < k; ++j) sal[j] = 0.05 + static_cast<double>(r.next() % 4000) / 100.0;
  const float grid[4] = {0.0f, 0.3f, 0.7f, 1.0f};
  float alpha[POLYQ_NUM_BITS];
  CHECK(polyq_bit_scaling(w.data(), n, k, x2.data(), sal.data(), bits.data(), grid, 4, s.data(), alpha) ==
            POLYQ_OK, "bit_scaling");
  for (int j = 0; j < k; ++j) {
    int e = 0;
    CHECK(frexpf(s[j], &e) == 0.5f, "scale %g is not a power of two", static_cast<double>(s[j]));
    CHECK(bits[j] != 16 || s[j] == 1.0f, "16-bit channel scaled");
  }
  CHECK(alpha[POLYQ_NUM_BITS - 1] == 0.0f, "alpha_16 = 0");
  const float bad_grid[1] = {1.5f};
  CHECK(polyq_bit_scaling(w.data(), n, k, x2.data(), sal.data(), bits.data(), bad_grid, 1, s.data(), nullptr) ==
            POLYQ_ERR_ARG, "grid out of [0, 1] refused");
  CHECK(polyq_waterfill(err.data(), k, NAN, bits.data()) == POLYQ_ERR_ARG, "NaN budget refused");
  CHECK(polyq_quanta_match(err.data(), k, 7, budget, bits.data(), counts) ==
            (k % 7 ? POLYQ_ERR_QUANTUM : POLYQ_OK), "quantum check");
}

}  // namespace

int main(int argc, char** argv) {
  const uint64_t seed = argc > 1 ? strtoull(argv[1], nullptr, 10) : 1;
  const int iters = argc > 2 ? atoi(argv[2]) : 300;
  Rng r{seed};
  check_invalid();
  if (!g_fail) check_grid_forms();
  if (!g_fail) check_gemm_forms();
  for (int it = 0; it < iters && !g_fail; ++it) {
    polyq_block b[POLYQ_MAX_BLOCKS];
    // mostly short layers, some long ones up to the largest k
    const int max_units = it % 25 == 0 ? (POLYQ_MAX_K / 32) / 5 : (it % 5 == 0 ? 200 : 24);
    const int nb = random_blocks(r, max_units, b);
    int k = 0;
    for (int i = 0; i < nb; ++i) k += b[i].len;
    const int n = r.uniform(1, 5 * 64 + 7);
    polyq_layout L;
    const polyq_status st = polyq_plan(n, k, b, nb, &L);
    if (k > POLYQ_MAX_K) {
      if (st != POLYQ_ERR_SHAPE) { fprintf(stderr, "FAIL k=%d status %d\n", k, st); ++g_fail; }
      continue;
    }
    if (st != POLYQ_OK) { fprintf(stderr, "FAIL plan status %d (k=%d)\n", st, k); ++g_fail; break; }
    check_layout(L, b, nb, n, k);
    const int ms[4] = {1, 2, 5, 16};
    for (int j = 0; j < 4 && !g_fail; ++j) {
      check_gemv_plan(L, ms[j], L.n_tiles);
      check_gemv_plan(L, ms[j], L.n_tiles * r.uniform(1, 40));
    }
  }
  for (int it = 0; it < iters / 4 + 1 && !g_fail; ++it) check_gemv_grid(r);
  for (int it = 0; it < iters && !g_fail; ++it) check_gemm_shape(r);
  for (int it = 0; it < iters / 10 + 1 && !g_fail; ++it) check_alloc(r, it);
  if (g_fail) return 1;
  printf("plan_check ok: seed %llu, %d layouts\n", static_cast<unsigned long long>(seed), iters);
  return 0;
}
