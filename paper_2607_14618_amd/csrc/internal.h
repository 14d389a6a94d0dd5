// Internal definitions shared by the host planner and the HIP kernels of the
// mixed-bit linear-layer library.  Not part of the public ABI (include/polyq.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "polyq.h"

namespace polyq {

constexpr int kTileRows = POLYQ_TILE_ROWS;  // output rows per packed tile (one per lane)
constexpr int kChunk = POLYQ_QUANTUM;       // channels per chunk
constexpr int kGroup = POLYQ_GROUP;         // channels per quantization group
constexpr int kChunksPerGroup = kGroup / kChunk;
constexpr int kMetaBytes = kTileRows * 4;   // {fp16 s, fp16 z} per row of a tile

// Decode GEMV launch plan: the work-groups of one linear are n_tiles x S, each
// of W waves; wave w (0 <= w < S * W, across the tile's splits) covers the
// chunk range wave_range(w).  Every wave stays inside one block: block i gets
// waves[i] waves per tile.
constexpr int kMaxSplitEntries = 4096;  // S * W <= this
constexpr int kResidentWGs = 768;       // 256 CUs x 3 co-resident 4-wave work-groups (<= 168 VGPRs)

struct GemvPlan {
  int32_t S;                        // WG splits per 64-row tile
  int32_t W;                        // waves per WG
  int32_t waves[POLYQ_MAX_BLOCKS];  // waves per tile given to each block
  int32_t lds_chunks;               // largest chunk range of one wave
  int32_t lds_groups;               // most group records one wave stages (b <= 8 blocks)
};

// Exact floor(a / d) for 1 <= d and 0 <= a < 2^31 by a multiply and shifts
// (round-up multiplier, Granlund and Montgomery 1994): with l = floor(log2 d)
// and M = ceil(2^(32+l) / d), a M / 2^(32+l) = a / d + a e / (d 2^(32+l)) where
// e = M d - 2^(32+l) < d < 2^(l+1); since a e < 2^31 2^(l+1) = 2^(32+l) the
// excess stays below 1/d and cannot reach the next integer.  M < 2^32 unless d
// is a power of two, where div_magic returns 0 and the quotient is a >> l.
__host__ __device__ inline int div_log2(uint32_t d) { return d <= 1 ? 0 : 31 - __builtin_clz(d); }
__host__ __device__ inline uint32_t div_magic(uint32_t d) {
  if ((d & (d - 1)) == 0) return 0u;  // 0, 1 and powers of two
  return static_cast<uint32_t>(((1ull << (32 + div_log2(d))) + d - 1) / d);
}
__host__ __device__ inline uint32_t div_by_magic(uint32_t a, uint32_t magic, uint32_t d) {
  const uint32_t hi =
      magic == 0 ? a : static_cast<uint32_t>((static_cast<uint64_t>(a) * magic) >> 32);
  return hi >> div_log2(d);
}

// Grid of a decode launch: work-group (x, y, z), in one of three forms.
//   flat: linear y, x over its tiles x splits, tiles fastest (z = 0).  At most
//     `count` times the widest linear's work-groups, whatever the others look like.
//   split by split, where all linears have the same number of splits: linear y, tile
//     x, split z.
//   joint: the same with x over the tiles of all linears (first_tile) and y = 0.
// x_end: past it a work-group has nothing to do (flat, split by split), or belongs
// to a later linear than the first (joint).
// A CU's work-groups are about 256 apart in launch order and should be of different
// splits, that is of different bit-widths, so that all CUs take equally long.  Split
// by split they are, and in the flat order they are where one linear has about as
// many tiles as there are CUs; the flat one is the faster where a second round is
// begun and not half full.  Split by split / flat, one token: q/k/v of 5120 (720
// work-groups) 13.0 / 14.3 us, of 8192 (768) 24.9 / 29.7, gate/up of 12160 (760) 18.4
// / 19.0, of 13824 (864) 20.1 / 19.4, of 15360 (960) 21.4 / 19.5, of 25600 (1600)
// 38.0 / 39.5 (4 tokens 47.9 / 45.3, 16 tokens 74.3 / 76.2).
// Tiles that a narrow linear lacks cost about 2 ns each split by split; a joint
// launch has none, but its later linears wait for two more loads, 0.2 us.  Split by
// split / joint: 6 + 1 + 1 tiles 7.69 / 7.86 us, 48 + 12 + 12 (432 too many) 7.51 /
// 7.37, 64 + 16 + 16 (768) 11.1 / 8.6.  Linears without a common number of splits: in
// one box of the widest of each / flat, 131072 rows x 512 with 64 x 65536 (16
// tokens) 124 / 49.
constexpr int kCUs = 256;
struct GemvGrid {
  int32_t x, y, z;
  bool joint;
  int32_t x_end[POLYQ_MAX_BATCH];
  int32_t first_tile[POLYQ_MAX_BATCH];  // INT32_MAX past the last linear
};
inline GemvGrid gemv_grid(const int32_t* n_tiles, const int32_t* splits, int count) {
  GemvGrid g;
  bool same_splits = true;
  int widest = 0, most = 0, tiles = 0;  // work-groups and tiles of the widest linear, tiles of all
  for (int i = 0; i < POLYQ_MAX_BATCH; ++i) {
    g.x_end[i] = 0;
    g.first_tile[i] = i < count ? tiles : INT32_MAX;
    if (i >= count) continue;
    same_splits = same_splits && splits[i] == splits[0];
    widest = widest > n_tiles[i] * splits[i] ? widest : n_tiles[i] * splits[i];
    most = most > n_tiles[i] ? most : n_tiles[i];
    tiles += n_tiles[i];
  }
  const int64_t total = static_cast<int64_t>(tiles) * splits[0];
  const bool alternates = 3 * most > 2 * kCUs && 2 * most < 3 * kCUs;
  const bool by_split = same_splits && !(alternates && total > kResidentWGs && 2 * total < 3 * kResidentWGs);
  g.joint = by_split && static_cast<int64_t>(most) * count * splits[0] - total > kCUs;
  for (int i = 0; i < count; ++i) g.x_end[i] = by_split ? n_tiles[i] : n_tiles[i] * splits[i];
  g.x = g.joint ? tiles : by_split ? most : widest;
  g.y = g.joint ? 1 : count;
  g.z = by_split ? splits[0] : 1;
  return g;
}
// Tile and split of a linear's work-group (x counted from its first tile).
__host__ __device__ inline void gemv_place(uint32_t x, uint32_t z, uint32_t magic, int n_tiles, int* tile, int* split) {
  const int turn = static_cast<int>(div_by_magic(x, magic, static_cast<uint32_t>(n_tiles)));
  *tile = static_cast<int>(x) - turn * n_tiles;
  *split = turn + static_cast<int>(z);
}

// A block's groups over its nw waves: q = groups / nw each and one more for r =
// groups mod nw of them, the waves t .. t + r - 1; the first group of wave j is
// share_begin, it has q + share_extra.  The first waves take the rest (t = 0), but a
// single group too many goes to the last wave where the block's last group is a
// partial one and that makes the largest share smaller by more than an eighth: nine
// chunks over two waves are 4 + 5 and not 8 + 1 (512 channels x 2048 rows, one token:
// 4.29 us instead of 4.61).  A smaller saving does not pay (gate/up of 25600 rows at
// 6 bits, one token: 38.9 us instead of 38.3), and the rest for the last waves
// whatever r is made 16-token launches up to 5 % slower.
inline int share_first_extra(int chunks, int nw) {
  const int groups = (chunks + kChunksPerGroup - 1) / kChunksPerGroup;
  const int missing = groups * kChunksPerGroup - chunks;  // of the last group
  return groups % nw == 1 && 2 * missing > groups / nw + 1 ? nw - 1 : 0;
}
__host__ __device__ inline int share_begin(int q, int r, int t, int j) {
  const int past = j > t ? j - t : 0;
  return j * q + (past < r ? past : r);
}
__host__ __device__ inline int share_extra(int r, int t, int j) {
  return static_cast<unsigned>(j - t) < static_cast<unsigned>(r) ? 1 : 0;
}

// Chunk range [lo, hi) of wave w of every tile: waves are handed to the blocks
// in order (waves[i] to block i, starting at wave w0[i]) and a block's groups
// are split evenly among its waves (share_begin), so that every wave starts and
// ends on a group boundary of one block.  Waves past the last block get an empty
// range at the end of the layer.  `blk` gives, for block i, cb(i) / ce(i) (chunk
// range), w0(i) and nw(i).  The host planner's form; the kernel reads the same
// shares from its argument record.  `block` (optional) receives the block index
// i (or -1); the range is empty unless w < w0(i) + nw(i).
template <class Blk>
inline void wave_range(int w, int nblocks, int n_chunks, const Blk& blk, int* lo, int* hi, int* block = nullptr) {
  int i = -1;
  for (int b = 0; b < nblocks; ++b)
    if (blk.w0(b) <= w) i = b;
  *lo = *hi = n_chunks;
  if (block) *block = i;
  if (i < 0) return;
  const int w0 = blk.w0(i), nw = blk.nw(i);
  if (w >= w0 + nw) return;
  const int cb = blk.cb(i), nch = blk.ce(i) - cb;
  const int ngr = (nch + kChunksPerGroup - 1) / kChunksPerGroup, j = w - w0;
  const int q = ngr / nw, r = ngr % nw, t = share_first_extra(nch, nw);
  const int a = kChunksPerGroup * share_begin(q, r, t, j);
  const int b = a + kChunksPerGroup * (q + share_extra(r, t, j));
  *lo = cb + (a < nch ? a : nch);
  *hi = cb + (b < nch ? b : nch);
}

// Returns 0 on success.  Chooses S, W and the waves per block for `m` tokens;
// `launch_tiles` is the number of 64-row tiles of every linear that shares the
// launch (the splits are sized so that the launch fills the GPU about once).
int plan_gemv(const polyq_layout& L, int32_t m, int32_t launch_tiles, GemvPlan* p);

// Bytes of GEMV workspace needed for plan p (0 when S == 1): one uint32 counter
// per tile (padded to 256 B) followed by the partials [S][m][n_tiles*64] fp32.
size_t gemv_workspace_for(const polyq_layout& L, int32_t m, const GemvPlan& p);

// Prefill launch: a work-group multiplies kGemmTiles packed tiles by `nt` token
// tiles (kGemmTokens each), `m_tiles` work-groups cover the tokens and K is split
// into `splits` ranges of whole groups (at most `most`).
constexpr int kGemmTiles = 4;
constexpr int kGemmTokens = 16;
constexpr int kGemmMaxNT = 8;
constexpr int kGemmMaxSplits = 32;
struct GemmShape {
  int nt, splits;
  int32_t m_tiles;
};
GemmShape gemm_shape(const polyq_layout* const* layouts, int count, int32_t m, int most);

// Groups of a layout, of every bit-width (16 included).
int layout_groups(const polyq_layout& L);

// True when `L` is exactly what polyq_plan produces for its own n, k, blocks.
bool layout_is_valid(const polyq_layout* L);

// LDS bytes of one GEMV wave's staging region (x' of m tokens, then group
// metadata), the offset of the work-group's shared zero row (after the W wave
// regions) and the LDS of a work-group, for plan p and m tokens.
size_t gemv_wave_lds_bytes(const GemvPlan& p, int32_t m);
size_t gemv_zero_offset(const GemvPlan& p, int32_t m);
size_t gemv_lds_bytes(const GemvPlan& p, int32_t m);

// Validation and workspace size of a polyq_gemv_batch request: every check
// polyq_gemv_batch makes before it launches, except the workspace's own.
// need: total bytes; zero: the leading bytes that must be zero on entry.
polyq_status gemv_batch_workspace_status(const polyq_gemv_item* items, int32_t count, int32_t m,
                                         size_t* need, size_t* zero);

// One copy of the explicit activation shuffle (Eq. 9, with Eq. 8's channel
// factors): out[i][j] = x[i][perm[j]] * f[j] for m rows of k 2-byte
// activations.  perm NULL: the identity; an entry outside [0, k) yields 0;
// f NULL: no factors (the values are copied bit for bit); otherwise fp16
// factors, the product rounded to the activation type.
struct ShuffleJob {
  const int32_t* perm;
  const uint16_t* f;
  const uint16_t* x;
  uint16_t* out;
  int32_t k, pad;
};
// All `count` (<= POLYQ_MAX_BATCH) copies in one launch on `stream` (fp16
// activations, or bf16 when `bf16`); rows are staged in LDS when there are
// many and k and the alignments allow.  Launch only: the caller has validated
// the arguments.
void launch_shuffle(const ShuffleJob* jobs, int count, int32_t m, bool bf16, hipStream_t stream);

// Block accessor of a layout for wave_range (host side).
struct LayoutBlocks {
  const polyq_layout* L;
  const int32_t* waves;
  int cb(int i) const { return L->k_begin[i] / kChunk; }
  int ce(int i) const { return (L->k_begin[i] + L->block[i].len) / kChunk; }
  int w0(int i) const {
    int first = 0;
    for (int j = 0; j < i; ++j) first += waves[j];
    return first;
  }
  int nw(int i) const { return waves[i]; }
};

inline int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

}  // namespace polyq
