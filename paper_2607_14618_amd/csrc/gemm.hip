// Prefill GEMM over the mixed-bit clustered weight (Sec. 4.1-4.2), M tokens:
//   y[m][n] = sum_k' w_hat[n][k'] x'[m][k'],  x' = x[:, perm] (Eq. 9)
//
// Prefill is a dense contraction, so it runs on the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation).  A work-group of 8 waves owns
// four packed tiles (256 weight rows) x 16 NT tokens and walks K one
// 128-channel group at a time:
//   * wave (t, h) multiplies rows 32 h .. 32 h + 31 of packed tile t by all of
//     the work-group's tokens.  Its weights never pass through LDS: a packed
//     lane slice holds exactly the A fragments of that lane, so the wave loads
//     its half of each slice two groups ahead into registers, dequantizes the
//     group into eight fragments and multiplies them by every token tile;
//   * the activations of the group (16 NT tokens x 256 bytes) are the B operand
//     that all waves read from a two-stage LDS ring, loaded one group ahead.
// One barrier per group.  The two waves of a SIMD (h = 0 and h = 1) run half a
// group apart: one dequantizes behind the barrier, the other before it, so that
// the vector ALU work of one overlaps the matrix work of the other (without:
// 747 us instead of 681, gate/up of 2000 tokens x 13824 rows x 5120 channels).
//
// What bounds it: the issue slots and dependent chains of the two waves a SIMD
// holds (254 registers at NT = 8).  A group is 64 products and, per wave, 123 to 173
// vector instructions of dequantization (8 to 3 bits) and 64 of folds, one behind
// the other in a wave; a product takes two of its sixteen clocks' four issue slots.
// Loads are not it: with every load hitting the cache the launch is 3 % faster.
// Measured against the kernel before (256 tokens x 128 rows, both operands staged in
// LDS, whatever M is), packed size and mix as stated: 33 tokens through a 13B-class
// layer (4 launches, 4 bits) 306 -> 127 us, 512 tokens 543 -> 452 us (719 TFLOP/s),
// 2000 tokens of gate/up at 3 bits 771 -> 668 us (847 TFLOP/s).  Also tried: four
// waves per work-group and two work-groups per CU (734 us instead of 681 for the last),
// one loop for all bit-widths (735: the weights' loads then go one group ahead
// only), a second copy of the products for full groups or for the rare zero
// points (spills).
//
// Numerics.  The dequantized operand is (q - zi), zi the integer in [0, 255]
// nearest the zero point: of magnitude <= 255, which bf16 holds exactly.  Each
// 128-channel group accumulates into its own fp32 tile, which is then scaled
// by the row's fp16 scale s (fp32 FMA) into the output accumulator.  A code
// field at bit f of a half-word, OR-ed with the fp16 exponent field 25 - f,
// reads as the fp16 value 2^(10-f) + q (exact); converted to fp32 with
// -(2^(10-f) + zi) added in the same instruction it is q - zi exactly, and so is
// its upper half, the bf16 value.  Where a zero point of the wave's rows is not
// its zi, a second pass over the group with weights of 1 forms the sum of its
// activations and adds s (zi - z) times that, in fp32 (z - zi is exact): the
// weights are not read or unpacked again, and |q - zi| + |zi - z| <= 3 |q - z|
// bounds what the two parts round (every zero point fractional, 5120 rows x 5120
// channels at 4 bits: 22, 70 and 233 us for 33, 512 and 2000 tokens, against 19,
// 52 and 157 with integers; as hi + lo pairs re-read from memory 49, 135 and
// 585).  A 16-bit channel enters as the pair hi + lo of bf16 values (two passes),
// exact for an fp16 weight.
#include <hip/hip_runtime.h>

#include <string.h>

#include <algorithm>
#include <type_traits>

#include "codec.h"
#include "internal.h"

namespace polyq {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u3v __attribute__((ext_vector_type(3)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512;         // 8 waves
constexpr int kTilesWG = kGemmTiles;  // packed tiles per work-group (two waves each)
constexpr int kTok = kGemmTokens;     // tokens of one MFMA
constexpr int kMaxNT = kGemmMaxNT;    // token tiles per work-group (kernel instances 1 .. kMaxNT)

// One linear of a launch: 64 dwords, so that one vector load (a dword per lane)
// fetches it and v_readlane reads its fields at run-time indexes: scalar loads
// of it missed the scalar cache line by line, one round trip after the other
// (77 tokens x 1357 rows x 2976 channels: most of the launch).  Byte offsets
// fit 31 bits (the host refuses larger packed buffers).
struct GemmItem {
  const uint8_t* packed;
  const uint16_t* x;  // bf16 [m][k], clustered order
  float* y;           // fp32 [m][n]; splits > 1: the partial sums [splits][m][n]
  int32_t n, k, nblocks, n_tiles;
  int32_t groups;     // 128-channel groups (of every bit-width, 16 included)
  int32_t y_vec;      // rows of y can take 16-byte stores (n % 4 == 0, y 16-byte aligned)
  int32_t row_blocks; // ceil(n_tiles / kTilesWG)
  int32_t bits[POLYQ_MAX_BLOCKS];
  int32_t len[POLYQ_MAX_BLOCKS];   // channels
  int32_t k0[POLYQ_MAX_BLOCKS];    // first channel
  int32_t off[POLYQ_MAX_BLOCKS];   // byte offset of the block region
  int32_t tb[POLYQ_MAX_BLOCKS];    // bytes of one packed tile of the block
  int32_t pad[26];
};
static_assert(sizeof(GemmItem) == 256, "argument record");

// A launch: the linears' work-groups one after another (item i owns
// work-groups wg_begin[i] .. wg_begin[i + 1] - 1), all with the same m.  K is
// split into `splits` ranges of whole groups; with more than one, split s
// writes its sums to y[s][m][n] and a second kernel adds the splits in order.
struct GemmBatchArgs {
  GemmItem item[POLYQ_MAX_BATCH];
  int32_t count, m, m_tiles, splits;
  int32_t wg_begin[POLYQ_MAX_BATCH + 1];
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                           static_cast<int>(bytes), 0x00020000);
}

__host__ __device__ constexpr uint32_t exp_field(int e) { return (static_cast<uint32_t>(e) << 10) * 0x00010001u; }

// The fields at bits f and 16 + f of w (mask m2 covers both, already shifted
// to f) as the fp16 pair (2^(10-f) + q_even, 2^(10-f) + q_odd).
__device__ __forceinline__ uint32_t field_pair(uint32_t w, uint32_t m2, int f) {
  // one v_and_or_b32 (a VOP3 takes no literal: the mask in an SGPR, the exponent in a VGPR)
  uint32_t r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(m2), "v"(exp_field(25 - f)));
  return r;
}

// The 4 code pairs (channels 2j, 2j+1) of row sub-tile r of a lane slice, in
// the arrangement of codec.h, as fp16 pairs (off[j] + q) with off[j] =
// 2^(10 - f) for the field position f each pair is read at.  `w` holds the
// 16 bytes loaded at the sub-tile's offset (sub_offset); r is wave-uniform.
template <int B>
__device__ __forceinline__ void unpack_sub_tile(const u4v w, int r, uint32_t* hp) {
  if constexpr (B == 2) {  // word r/2 holds sub-tiles r & ~1 (bits 0..7) and r | 1 (8..15)
    const uint32_t u = w.x >> (8 * (r & 1));
    hp[0] = field_pair(u, 0x00030003u, 0);
    hp[1] = field_pair(u, 0x000C000Cu, 2);
    hp[2] = field_pair(u, 0x00300030u, 4);
    hp[3] = field_pair(u, 0x00C000C0u, 6);
  } else if constexpr (B == 4) {  // word r, pairs at 0, 4, 8, 12
    const uint32_t t = w.x >> 8;
    hp[0] = field_pair(w.x, 0x000F000Fu, 0);
    hp[1] = field_pair(w.x, 0x00F000F0u, 4);
    hp[2] = field_pair(t, 0x000F000Fu, 0);
    hp[3] = field_pair(t, 0x00F000F0u, 4);
  } else if constexpr (B == 8) {  // words 2r, 2r+1, pairs at bytes (0, 2) and (1, 3); 0x64 = exponent 25
    hp[0] = __builtin_amdgcn_perm(w.x, 0x64646464u, 0x00060004u);
    hp[1] = __builtin_amdgcn_perm(w.x, 0x64646464u, 0x00070005u);
    hp[2] = __builtin_amdgcn_perm(w.y, 0x64646464u, 0x00060004u);
    hp[3] = __builtin_amdgcn_perm(w.y, 0x64646464u, 0x00070005u);
  } else {  // B == 3: pair P = 4r + j in word P/5 at f3(P%5); fields at 10, 13 read after >> 10
    const uint32_t t0 = w.x >> 10, t1 = w.y >> 10, t2 = w.z >> 10;
    switch (r) {
      case 0:
        hp[0] = field_pair(w.x, 0x00070007u, 0);
        hp[1] = field_pair(w.x, 0x00380038u, 3);
        hp[2] = field_pair(w.x, 0x01C001C0u, 6);
        hp[3] = field_pair(t0, 0x00070007u, 0);
        break;
      case 1:
        hp[0] = field_pair(t0, 0x00380038u, 3);
        hp[1] = field_pair(w.y, 0x00070007u, 0);
        hp[2] = field_pair(w.y, 0x00380038u, 3);
        hp[3] = field_pair(w.y, 0x01C001C0u, 6);
        break;
      case 2:
        hp[0] = field_pair(t1, 0x00070007u, 0);
        hp[1] = field_pair(t1, 0x00380038u, 3);
        hp[2] = field_pair(w.z, 0x00070007u, 0);
        hp[3] = field_pair(w.z, 0x00380038u, 3);
        break;
      default:  // codes 30, 31: bit d of each in bits 9 and 25 of word d
        hp[0] = field_pair(w.z, 0x01C001C0u, 6);
        hp[1] = field_pair(t2, 0x00070007u, 0);
        hp[2] = field_pair(t2, 0x00380038u, 3);
        hp[3] = ((w.x >> 9) & 0x00010001u) | ((w.y >> 8) & 0x00020002u) | ((w.z >> 7) & 0x00040004u) |
                exp_field(25);
        break;
    }
  }
}

// off[j] of unpack_sub_tile for sub-tile r.
template <int B>
__device__ __forceinline__ void pair_offsets(int r, float* off) {
  if constexpr (B == 2) {
    off[0] = 1024.f; off[1] = 256.f; off[2] = 64.f; off[3] = 16.f;
  } else if constexpr (B == 4) {
    off[0] = 1024.f; off[1] = 64.f; off[2] = 1024.f; off[3] = 64.f;
  } else if constexpr (B == 8) {
    off[0] = off[1] = off[2] = off[3] = 1024.f;
  } else {
    const float t[4][4] = {{1024.f, 128.f, 16.f, 1024.f}, {128.f, 1024.f, 128.f, 16.f},
                           {1024.f, 128.f, 1024.f, 128.f}, {16.f, 1024.f, 128.f, 1024.f}};
    switch (r) {
      case 0: for (int j = 0; j < 4; ++j) off[j] = t[0][j]; break;
      case 1: for (int j = 0; j < 4; ++j) off[j] = t[1][j]; break;
      case 2: for (int j = 0; j < 4; ++j) off[j] = t[2][j]; break;
      default: for (int j = 0; j < 4; ++j) off[j] = t[3][j]; break;
    }
  }
}

__device__ __forceinline__ uint32_t hi_half_pair(float lo, float hi) {
  return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo),
                               0x07060302u);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

// Eight values as bf16: the nearest (hi), or the nearest to the remainder (lo).
__device__ __forceinline__ u4v bf16_part(const float* v, bool lo) {
  u4v r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = v[2 * i], b = v[2 * i + 1];
    uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, bf16x2));
    if (lo)
      h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a - __builtin_bit_cast(float, h << 16),
                                                                  b - __builtin_bit_cast(float, h & 0xFFFF0000u)}, bf16x2));
    r[i] = h;
  }
  return r;
}

// One group of one wave in flight: its half of four lane slices, the zero points of the
// lane's rows 16 (2h) + l%16 and 16 (2h+1) + l%16, and the scales of rows
// 16 r + 4 (l/16) + e.
struct Raw {
  uint32_t w[16];
  uint32_t z;
  u4v s;
};

template <int B>
__device__ __forceinline__ int slice_voff(int lane, int h) {
  return lane * 4 * B + (B == 2 ? 4 * h : B == 4 ? 8 * h : B == 8 ? 16 * h : B == 16 ? 32 * h : 0);
}

// Loads of the group at byte `rec` of the tile: `nch` chunks; absent ones
// re-read the last (their activations are zero).
template <int B>
__device__ __forceinline__ void issue_raw(Raw& r, __amdgpu_buffer_rsrc_t rs, int lane, int h, int rec, int nch) {
  const int voff = slice_voff<B>(lane, h);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int so = rec + (B <= 8 ? kMetaBytes : 0) + min(c, nch - 1) * 256 * B;
    if constexpr (B == 3) {
      const u3v v = __builtin_bit_cast(u3v, __builtin_amdgcn_raw_buffer_load_b96(rs, voff, so, 0));
      r.w[4 * c] = v.x; r.w[4 * c + 1] = v.y; r.w[4 * c + 2] = v.z;
    } else if constexpr (B == 4) {
      const u2v v = __builtin_bit_cast(u2v, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, so, 0));
      r.w[2 * c] = v.x; r.w[2 * c + 1] = v.y;
    } else if constexpr (B == 8) {
      const u4v v = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, so, 0));
      r.w[4 * c] = v.x; r.w[4 * c + 1] = v.y; r.w[4 * c + 2] = v.z; r.w[4 * c + 3] = v.w;
    } else {
      r.w[c] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, so, 0);
    }
  }
  if constexpr (B <= 8) {
    r.z = __builtin_amdgcn_raw_buffer_load_b32(rs, (lane & 15) * 8 + 4 * h, rec, 0);
    r.s = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(rs, 128 + (lane >> 4) * 32 + 16 * h, rec, 0));
  }
}

// The words of row sub-tile r of a chunk, as unpack_sub_tile takes them, out
// of the wave's half slice `w` (r = 2h or 2h + 1).
template <int B>
__device__ __forceinline__ u4v sub_words(const uint32_t* w, int rr) {
  if constexpr (B == 2) return u4v{w[0], 0u, 0u, 0u};
  else if constexpr (B == 4) return u4v{w[rr], 0u, 0u, 0u};
  else if constexpr (B == 8) return u4v{w[2 * rr], w[2 * rr + 1], 0u, 0u};
  else return u4v{w[0], w[1], w[2], 0u};
}
template <int B>
constexpr int chunk_words() { return B == 2 ? 1 : B == 4 ? 2 : 4; }

__device__ __forceinline__ float f16_of(uint32_t bits) {
  return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(bits)));
}

// The integer in [0, 255] nearest the zero point: q - zi is exact in bf16, and
// (zi - z) times the sum of the group's activations is added apart where z is
// not that integer itself.
__device__ __forceinline__ float z_int(float z) { return fminf(fmaxf(rintf(z), 0.f), 255.f); }

// The two halves of an fp16 pair plus c, in fp32 (v_fma_mix_f32 by 1.0: the
// conversion and the addition in one instruction each).
__device__ __forceinline__ float lo_plus(uint32_t pair, float c) {
  float d;
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(pair), "v"(c));
  return d;
}
__device__ __forceinline__ float hi_plus(uint32_t pair, float c) {
  float d;
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(pair), "v"(c));
  return d;
}

// The group's weights as bf16 A fragments (q - zi), a[rr][chunk].  H is the wave's
// half (3 bits: the positions of a sub-tile's codes depend on it; other widths take
// H = 0 for both).
template <int B, int H>
__device__ __forceinline__ void dequant(const Raw& raw, const float (&zi)[2], u4v (&a)[2][4]) {
  float nc[2][4];  // -(off + zi)
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {
    float off[4];
    pair_offsets<B>(2 * H + rr, off);
#pragma unroll
    for (int j = 0; j < 4; ++j) nc[rr][j] = -off[j] - zi[rr];
  }
  // A chunk in three stages of independent instructions (a dependent VALU
  // instruction waits about twice as long as an independent one; the fences
  // keep the compiler from chaining them pair by pair).
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t hp[2][4];
    float lo[2][4], hi[2][4];
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) unpack_sub_tile<B>(sub_words<B>(&raw.w[c * chunk_words<B>()], rr), 2 * H + rr, hp[rr]);
    __builtin_amdgcn_sched_barrier(0);
    // (off + q) - (off + zi) = q - zi exactly in fp32, and in its upper half
    // (bf16: |q - zi| <= 255)
#pragma unroll
    for (int rr = 0; rr < 2; ++rr)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lo[rr][j] = lo_plus(hp[rr][j], nc[rr][j]);
        hi[rr][j] = hi_plus(hp[rr][j], nc[rr][j]);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rr = 0; rr < 2; ++rr)
      a[rr][c] = u4v{hi_half_pair(lo[rr][0], hi[rr][0]), hi_half_pair(lo[rr][1], hi[rr][1]),
                     hi_half_pair(lo[rr][2], hi[rr][2]), hi_half_pair(lo[rr][3], hi[rr][3])};
  }
}

// Dword `dw` of a 64-dword argument record held one dword per lane, as a
// scalar (v_readlane; dw must be wave-uniform).
template <class T>
__device__ __forceinline__ T kfield(uint32_t kv, int dw) {
  if constexpr (sizeof(T) == 8) {
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(kv, dw));
    const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(kv, dw + 1));
    return __builtin_bit_cast(T, lo | (hi << 32));
  } else {
    return __builtin_bit_cast(T, static_cast<uint32_t>(__builtin_amdgcn_readlane(kv, dw)));
  }
}
#define ITEM(T, field) kfield<T>(kv, offsetof(GemmItem, field) / 4)
#define ITEM_AT(field, i) kfield<int32_t>(kv, offsetof(GemmItem, field) / 4 + (i))

template <int V>
using Int = std::integral_constant<int, V>;

template <int NT>
__global__ __launch_bounds__(kThreads) void gemm_kernel(const GemmBatchArgs a) {
  constexpr int kStage = NT * kTok * 256;                // bytes of one LDS stage
  constexpr int kPieces = (NT * 256 + kThreads - 1) / kThreads;  // 16-byte pieces per thread
  __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * kStage];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = wv >> 2;

  // Work-group order: each XCD (work-groups go to the eight XCDs in turn) takes
  // one contiguous stretch of the launch, token tile fastest, so that the
  // token tiles that share weight rows also share an L2.
  const int total = a.wg_begin[a.count];
  const int xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
  const int wg = xcd * per + min(xcd, rem) + static_cast<int>(blockIdx.x >> 3);
  int idx = 0;
#pragma unroll
  for (int i = 1; i < POLYQ_MAX_BATCH; ++i) idx += (i < a.count && wg >= a.wg_begin[i]) ? 1 : 0;
  static_assert(offsetof(GemmBatchArgs, item) == 0, "argument layout");
  const uint32_t* kargs = (const uint32_t*)(__builtin_amdgcn_kernarg_segment_ptr());
  const uint32_t kv = kargs[idx * 64 + lane];
  const uint8_t* packed = ITEM(const uint8_t*, packed);
  const int nblocks = ITEM(int32_t, nblocks);
  const int local = wg - a.wg_begin[idx];
  const int mt = local % a.m_tiles, rest = local / a.m_tiles;
  const int rb = rest % ITEM(int32_t, row_blocks), ks = rest / ITEM(int32_t, row_blocks);
  const int m0 = mt * (NT * kTok);
  const int groups = ITEM(int32_t, groups);
  const int g0 = groups * ks / a.splits, g1 = groups * (ks + 1) / a.splits;
  const int tile = rb * kTilesWG + (wv & 3);
  const bool tile_ok = tile < ITEM(int32_t, n_tiles);
  const int kdim = ITEM(int32_t, k);

  // ---- Activations: buffer over this token tile's rows (reads past row m - 1
  // return zero).  Stage layout: blocks of 8 tokens x 128 bytes (two chunks),
  // the 16-byte pieces of a token XOR-swizzled by token % 8, so that neither
  // the stores (8 lanes fill one row) nor the fragment reads (8 lanes read one
  // piece of 8 rows) conflict.
  const int rows = min(a.m - m0, NT * kTok);
  const __amdgpu_buffer_rsrc_t xrs =
      make_rsrc(ITEM(const uint16_t*, x) + static_cast<int64_t>(m0) * kdim, static_cast<uint32_t>(rows) * kdim * 2u);
  u4v xr[kPieces];
  // this thread's pieces: piece (tid & 7) of chunk pair (tid >> 6) & 1 of token
  // tid / 128 * 8 + tid / 8 % 8, and of the tokens 32, 64, .. further on
  const int xseg = ((tid >> 6) & 1) * 8 + (tid & 7);
  const int xvoff = (((tid >> 7) * 8 + ((tid >> 3) & 7)) * kdim + xseg * 8) * 2;
  // (`chan`: the group's first channel, nch: its chunks)
  auto load_x = [&](int chan, int nch) __attribute__((always_inline)) {
    // a chunk past the group's end reads zeros (an offset past the buffer)
    const int voff = (xseg >> 2) < nch ? xvoff : 0x40000000;
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
      xr[i] = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(xrs, voff + i * (64 * kdim), chan * 2, 0));
  };
  auto store_x = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int p = tid + i * kThreads;
      const int t8 = (p >> 3) & 7;
      const int at = (((p >> 6) & 1) * (NT * 2) + (p >> 7)) * 1024 + t8 * 128 + (((p & 7) ^ t8) * 16);
      if (NT % 2 == 0 || p < NT * 256) *reinterpret_cast<u4v*>(lds + stage * kStage + at) = xr[i];
    }
  };
  // this lane's piece of token l%16 of a token tile, chunk 0 (and, ^ 64, chunk 1)
  const int frag0 = ((lane >> 3) & 1) * 1024 + (lane & 7) * 128 + (((lane >> 4) ^ (lane & 7)) * 16);

  // ---- The walk over the groups [g0, g1): a position is a block, a group of
  // it and how many groups of the split follow; it stays on the split's last
  // group, so that the loads ahead of the multiplication are unconditional
  // (every wait then knows how many younger loads are in flight).
  struct Walk {
    int block, bits, chan, end, left;
  };
  auto enter = [&](Walk& w, int block, int g) __attribute__((always_inline)) {
    w.block = block;
    w.bits = ITEM_AT(bits, block);
    w.chan = ITEM_AT(k0, block) + g * kGroup;
    w.end = ITEM_AT(k0, block) + ITEM_AT(len, block);
  };
  auto advance = [&](Walk& w) __attribute__((always_inline)) {
    if (w.left == 0) return;
    --w.left;
    w.chan += kGroup;
    if (w.chan >= w.end) enter(w, w.block + 1, 0);
  };
  auto nch_of = [&](const Walk& w) __attribute__((always_inline)) { return min(kGroup, w.end - w.chan) / kChunk; };
  const int ng = g1 - g0;
  Walk wx, wr;  // the next group of the activations' loads and of the weights'
  int rec;      // byte of wr's group in its packed tile
  __amdgpu_buffer_rsrc_t wrs;
  auto locate = [&]() __attribute__((always_inline)) {
    rec = ((wr.chan - ITEM_AT(k0, wr.block)) / kGroup) * ((wr.bits <= 8 ? kMetaBytes : 0) + 1024 * wr.bits);
    wrs = make_rsrc(packed + ITEM_AT(off, wr.block) + static_cast<int64_t>(tile_ok ? tile : 0) * ITEM_AT(tb, wr.block),
                    tile_ok ? static_cast<uint32_t>(ITEM_AT(tb, wr.block)) : 0u);
  };
  auto advance_weights = [&]() __attribute__((always_inline)) {
    const int block = wr.block, chan = wr.chan;
    advance(wr);
    if (wr.block != block) locate();
    else if (wr.chan != chan) rec += (wr.bits <= 8 ? kMetaBytes : 0) + 1024 * wr.bits;
  };

  u4v af[2][4];
  f4 sc[2];
  f4 T[NT][2];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) T[j][rr] = f4{0.f, 0.f, 0.f, 0.f};

  // The second pass over a group with a zero point that is not an integer in
  // [0, 255]: weights of 1, so that the products are the sums of the activations,
  // and s (zi - z) for the scale.  (z and s re-read: the registers of the loads
  // ahead have taken their place, and a pair held over the products would spill.)
  auto rest_of_zero_points = [&](__amdgpu_buffer_rsrc_t rs, int rec) __attribute__((always_inline)) {
    int l = lane;
    asm volatile("" : "+v"(l));  // the addresses are formed here, not kept through the products
    uint32_t z[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      z[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, (4 * (l >> 4) + e) * 8 + 4 * h, rec, 0);
    const u4v s = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(rs, 128 + (l >> 4) * 32 + 16 * h, rec, 0));
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float zf = f16_of(rr ? z[e] >> 16 : z[e]);
        sc[rr][e] = f16_of(s[2 * rr + e / 2] >> (16 * (e & 1))) * (z_int(zf) - zf);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) af[rr][c] = u4v{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    }
  };
  // All products of one group, in sets of up to four token tiles: the set's
  // partial sums over the group's four chunks, then total += s * part, beside
  // the next set's first products.  The fragments of a step (one chunk of a
  // set) are read one step ahead; the fences keep the compiler from hoisting
  // every read to the front (the registers would not hold them).  The wave's
  // priority is raised meanwhile, so that the matrix pipe goes first and the
  // SIMD's other wave unpacks in the slots it leaves (gate/up of 2000 tokens:
  // 681 -> 676 us).
  auto multiply = [&](int stage) __attribute__((always_inline)) {
    constexpr int kSets = (NT + 3) / 4, kSteps = 4 * kSets;
    const uint8_t* b0 = lds + stage * kStage + frag0;
    const uint8_t* b1 = lds + stage * kStage + (frag0 ^ 64);
    bf16x8 bf[2][4];
    f4 P[4][2];
    auto read = [&](int st) __attribute__((always_inline)) {
      const int c = st & 3;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (st / 4 * 4 + u < NT)
          bf[st & 1][u] = *reinterpret_cast<const bf16x8*>((c & 1 ? b1 : b0) + (c >> 1) * (NT * 2048) + (st / 4 * 4 + u) * 2048);
    };
    auto fold = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int rr = 0; rr < 2; ++rr)
#pragma unroll
        for (int e = 0; e < 4; ++e) T[j][rr][e] = fmaf(sc[rr][e], P[j & 3][rr][e], T[j][rr][e]);
    };
    read(0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
      const int c = st & 3, j0 = st / 4 * 4;
      if (st + 1 < kSteps) read(st + 1);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (c == 0 && j0 > 0) fold(j0 - 4 + u);
        if (j0 + u < NT)
#pragma unroll
          for (int rr = 0; rr < 2; ++rr)
            P[u][rr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[rr][c]), bf[st & 1][u],
                                                               c == 0 ? f4{0.f, 0.f, 0.f, 0.f} : P[u][rr], 0, 0, 0);
      }
      // issue order of a step: the next step's reads, then the products (a
      // set's first step: each tile's fold before its products)
      const int nr = st + 1 < kSteps ? std::min(4, NT - (st + 1) / 4 * 4) : 0;
#pragma unroll
      for (int u = 0; u < nr; ++u) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (c == 0 && j0 > 0) __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
        if (j0 + u < NT) __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = (kSets - 1) * 4; j < NT; ++j) fold(j);
    __builtin_amdgcn_s_setprio(0);
  };

  // ---- Main loop.  Group i (of ng) sits in LDS stage i & 1; its activations
  // are loaded during group i - 1, its weights two groups ahead.  The barrier
  // of group i lets a wave read stage i & 1 and write the other one (every wave
  // has finished group i - 1).
  int i = 0;
  // The groups of one block of bit-width B from group i on (in the split).
  auto run_block = [&](auto b_tag) __attribute__((always_inline)) {
    constexpr int B = decltype(b_tag)::value;
    // the block's first two groups (the loads issued for them from the block
    // before only brought their lines into L2)
    const int block = wx.block;
    Walk cur = wx;  // group i
    if (i > 0) {
      wr = wx;
      locate();
    }
    Raw r0, r1;
    issue_raw<B>(r0, wrs, lane, h, rec, nch_of(wr));
    advance_weights();
    issue_raw<B>(r1, wrs, lane, h, rec, nch_of(wr));
    advance_weights();
    advance(wx);
    auto step = [&](Raw& raw) __attribute__((always_inline)) {
      if (h == 0) __syncthreads();
      const float z0 = f16_of(raw.z), z1 = f16_of(raw.z >> 16);
      float zi[2] = {z_int(z0), z_int(z1)};
      asm("" : "+v"(zi[0]), "+v"(zi[1]));  // formed once (the compiler would round in fp16 too)
      const bool exact = __all(z0 == zi[0] && z1 == zi[1]);
#pragma unroll
      for (int rr = 0; rr < 2; ++rr)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[rr][e] = f16_of(raw.s[2 * rr + e / 2] >> (16 * (e & 1)));
      if (B == 3 && h != 0) dequant<B, 1>(raw, zi, af);
      else dequant<B, 0>(raw, zi, af);
      load_x(wx.chan, nch_of(wx));
      issue_raw<B>(raw, wrs, lane, h, rec, nch_of(wr));
      advance_weights();
      if (h != 0) __syncthreads();
#pragma unroll 1
      for (int pass = 0;; ++pass) {
        if (__builtin_expect(pass != 0, 0)) {
          const int cb = cur.block;
          rest_of_zero_points(
              make_rsrc(packed + ITEM_AT(off, cb) + static_cast<int64_t>(tile_ok ? tile : 0) * ITEM_AT(tb, cb),
                        tile_ok ? static_cast<uint32_t>(ITEM_AT(tb, cb)) : 0u),
              ((cur.chan - ITEM_AT(k0, cb)) / kGroup) * (kMetaBytes + 1024 * B));
        }
        multiply(i & 1);
        if (exact || pass) break;
      }
      store_x((i + 1) & 1);
      ++i;
      cur = wx;
      if (i == ng || wx.block != block) return false;
      advance(wx);
      return true;
    };
    while (step(r0) && step(r1)) {
    }
  };
  // The groups of the 16-bit block: fp16 weights, hi then lo parts.  (Both
  // parts come from registers: re-reading the weights for each, with the
  // conversion in integer instructions, cost about 10 us per work-group.  The next
  // group's weights loaded behind the second part's products: 6394 rows x 18304
  // channels of 16 bits, 2047 tokens, 1200 us instead of 1146, since the loop of the two
  // parts then waits for every load; with the parts unrolled it spills from NT = 6 on.)
  auto run_block16 = [&]() __attribute__((always_inline)) {
    sc[0] = sc[1] = f4{1.f, 1.f, 1.f, 1.f};
    for (;;) {
      wr = wx;
      locate();
      const int nch = nch_of(wx);
      u4v w[2][4];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int rr = 0; rr < 2; ++rr)
          w[rr][c] = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(
              wrs, slice_voff<16>(lane, h) + 16 * rr, rec + min(c, nch - 1) * 4096, 0));
      advance(wx);
      load_x(wx.chan, nch_of(wx));
      __syncthreads();
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
        for (int rr = 0; rr < 2; ++rr)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = f16_of(w[rr][c][e / 2] >> (16 * (e & 1)));
            af[rr][c] = bf16_part(v, pass != 0);
          }
        multiply(i & 1);
      }
      store_x((i + 1) & 1);
      if (++i == ng) break;
    }
  };
  if (ng > 0) {
    int g = g0, b = 0;
    while (b + 1 < nblocks && g >= (ITEM_AT(len, b) + kGroup - 1) / kGroup) {
      g -= (ITEM_AT(len, b) + kGroup - 1) / kGroup;
      ++b;
    }
    enter(wx, b, g);
    wx.left = ng - 1;
    wr = wx;
    locate();
    load_x(wx.chan, nch_of(wx));
    store_x(0);
    // bit-widths ascend: one pass over the palette, straight-line code
    if (wx.bits == 2) run_block(Int<2>{});
    if (i < ng && wx.bits == 3) run_block(Int<3>{});
    if (i < ng && wx.bits == 4) run_block(Int<4>{});
    if (i < ng && wx.bits == 8) run_block(Int<8>{});
    if (i < ng && wx.bits == 16) run_block16();
  }

  // D layout: lane holds weight rows 16 rr + 4 (lane/16) + e of token 16 j + lane%16.
  if (!tile_ok) return;
  const int row0 = tile * kTileRows + 32 * h + 4 * (lane >> 4);
  const int n = ITEM(int32_t, n);
  const bool y_vec = ITEM(int32_t, y_vec) != 0;
  float* ybase = ITEM(float*, y) + static_cast<int64_t>(ks) * a.m * n;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int tok = m0 + kTok * j + (lane & 15);
    if (tok >= a.m) continue;
    float* yr = ybase + static_cast<int64_t>(tok) * n;
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
      const int row = row0 + 16 * rr;
      if (y_vec && row + 3 < n) {
        *reinterpret_cast<f4*>(yr + row) = T[j][rr];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (row + e < n) yr[row + e] = T[j][rr][e];
      }
    }
  }
}

// y = partial[0] + partial[1] + ... (in split order) of every linear of a
// launch (grid.y), `count` elements each, four consecutive elements per thread
// (16-byte accesses when count is a multiple of 4 and y is 16-byte aligned; the
// partials always are).
struct SumArgs {
  const float* partial[POLYQ_MAX_BATCH];
  float* y[POLYQ_MAX_BATCH];
  int64_t count[POLYQ_MAX_BATCH];
  int32_t splits;
};

__global__ __launch_bounds__(256) void sum_splits_kernel(const SumArgs a) {
  const float* __restrict__ partial = a.partial[blockIdx.y];
  float* __restrict__ y = a.y[blockIdx.y];
  const int64_t count = a.count[blockIdx.y];
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * 4;
  if (i >= count) return;
  if ((count & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0) {
    f4 v = *reinterpret_cast<const f4*>(partial + i);
    constexpr int kAhead = 8;  // loads in flight (one memory round trip for up to nine splits)
    for (int s0 = 1; s0 < a.splits; s0 += kAhead) {
      f4 w[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        w[u] = *reinterpret_cast<const f4*>(partial + std::min(s0 + u, a.splits - 1) * count + i);
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (s0 + u < a.splits) v += w[u];
    }
    *reinterpret_cast<f4*>(y + i) = v;
  } else {
    for (int64_t j = i; j < count && j < i + 4; ++j) {
      float v = partial[j];
      for (int s = 1; s < a.splits; ++s) v += partial[s * count + j];
      y[j] = v;
    }
  }
}

}  // namespace
}  // namespace polyq

using namespace polyq;

namespace {

size_t permuted_bytes(const polyq_layout& L, int32_t m) {
  return static_cast<size_t>(align_up(static_cast<int64_t>(m) * L.k * 2, 256));
}

struct GemmPlan {
  int64_t region[POLYQ_MAX_BATCH];   // workspace offset of item i's copy x', or -1
  size_t partial[POLYQ_MAX_BATCH];   // workspace offset of its partial sums (splits > 1)
  size_t total;
  GemmShape shape;
};

// Workspace of a batch: one clustered copy x' = x[:, perm] (times the channel
// factors of Eq. 8) per distinct (x, perm, factors) of the items with a
// permutation or factors, then the partial sums of every item (splits > 1).
// A batch (count > 1) is planned with the splits whose partial sums fit `room`
// bytes (one always does: it needs the copies alone); a single linear always
// with its own plan, which the caller's workspace has to hold.
polyq_status plan_gemm_batch(const polyq_gemv_item* items, int32_t count, int32_t m, size_t room, GemmPlan* p) {
  if (items == nullptr || count < 1 || m < 1) return POLYQ_ERR_ARG;
  if (count > POLYQ_MAX_BATCH) return POLYQ_ERR_CAPACITY;
  size_t off = 0;
  for (int i = 0; i < count; ++i) {
    if (!layout_is_valid(items[i].layout)) return POLYQ_ERR_ARG;
    if (static_cast<int64_t>(m) * items[i].layout->k * 2 > 0x7FFFFFFFll) return POLYQ_ERR_CAPACITY;
    p->region[i] = -1;
    if (items[i].perm == nullptr && items[i].xscale == nullptr) continue;
    for (int j = 0; j < i; ++j)
      if (p->region[j] >= 0 && items[j].perm == items[i].perm && items[j].x == items[i].x &&
          items[j].xscale == items[i].xscale && items[j].layout->k == items[i].layout->k) {
        p->region[i] = p->region[j];
        break;
      }
    if (p->region[i] < 0) {
      p->region[i] = static_cast<int64_t>(off);
      off += permuted_bytes(*items[i].layout, m);
    }
  }
  auto partial_bytes = [&](int i, int splits) {
    return static_cast<size_t>(align_up(static_cast<int64_t>(splits) * m * items[i].layout->n * 4, 256));
  };
  int most = kGemmMaxSplits;
  for (; count > 1 && most > 1; --most) {
    size_t need = off;
    for (int i = 0; i < count; ++i) need += partial_bytes(i, most);
    if (need <= room) break;
  }
  const polyq_layout* layouts[POLYQ_MAX_BATCH];
  for (int i = 0; i < count; ++i) layouts[i] = items[i].layout;
  p->shape = gemm_shape(layouts, count, m, most);
  for (int i = 0; i < count; ++i) {
    p->partial[i] = off;
    if (p->shape.splits > 1) off += partial_bytes(i, p->shape.splits);
  }
  p->total = off;
  return POLYQ_OK;
}

template <int NT>
void launch_gemm(int nt, int64_t wg, const GemmBatchArgs& a, hipStream_t st) {
  if (nt == NT)
    hipLaunchKernelGGL(gemm_kernel<NT>, dim3(static_cast<unsigned>(wg)), dim3(kThreads), 0, st, a);
  else if constexpr (NT < kMaxNT)
    launch_gemm<NT + 1>(nt, wg, a, st);
}

}  // namespace

extern "C" size_t polyq_gemm_batch_workspace_bytes(const polyq_gemm_item* items, int32_t count,
                                                   int32_t m) {
  GemmPlan p;
  if (plan_gemm_batch(items, count, m, SIZE_MAX, &p) != POLYQ_OK) return 0;
  return p.total;
}

extern "C" size_t polyq_gemm_workspace_bytes(const polyq_layout* layout, int32_t m, int perm_given) {
  if (!layout_is_valid(layout) || m < 1) return 0;
  const int32_t dummy = 0;
  const polyq_gemm_item item{layout, nullptr, perm_given ? &dummy : nullptr, nullptr, nullptr, nullptr};
  return polyq_gemm_batch_workspace_bytes(&item, 1, m);
}

extern "C" polyq_status polyq_gemm_batch(const polyq_gemm_item* items, int32_t count, int32_t m,
                                         void* workspace, size_t workspace_bytes, void* stream) {
  GemmPlan p;
  const size_t room = reinterpret_cast<uintptr_t>(workspace) % 16 == 0 && workspace != nullptr ? workspace_bytes : 0;
  const polyq_status pst = plan_gemm_batch(items, count, m, room, &p);
  if (pst != POLYQ_OK) return pst;
  if (p.total > 0 && (workspace == nullptr || workspace_bytes < p.total)) return POLYQ_ERR_CAPACITY;
  if (p.total > 0 && reinterpret_cast<uintptr_t>(workspace) % 16 != 0) return POLYQ_ERR_ARG;
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  GemmBatchArgs a;
  memset(&a, 0, sizeof(a));
  a.count = count;
  a.m = m;
  a.splits = p.shape.splits;
  a.m_tiles = p.shape.m_tiles;
  for (int i = 0; i < count; ++i) {
    const polyq_gemv_item& itm = items[i];
    const polyq_layout& L = *itm.layout;
    if (itm.packed == nullptr || itm.x == nullptr || itm.y == nullptr) return POLYQ_ERR_ARG;
    if (reinterpret_cast<uintptr_t>(itm.packed) % 256 != 0 || reinterpret_cast<uintptr_t>(itm.y) % 4 != 0)
      return POLYQ_ERR_ARG;
    if (L.packed_bytes > 0x7FFFFFFFll) return POLYQ_ERR_CAPACITY;
    if (itm.perm == nullptr && itm.xscale == nullptr && reinterpret_cast<uintptr_t>(itm.x) % 16 != 0)
      return POLYQ_ERR_ARG;  // clustered activations are read as 16-byte vectors
  }
  // Every check above and here comes before the first launch.
  int64_t wg = 0;
  for (int i = 0; i < count; ++i) {
    a.wg_begin[i] = static_cast<int32_t>(wg);
    a.item[i].row_blocks = (items[i].layout->n_tiles + kTilesWG - 1) / kTilesWG;
    wg += static_cast<int64_t>(a.item[i].row_blocks) * p.shape.m_tiles * p.shape.splits;
    if (wg > 0x7FFFFFFF) return POLYQ_ERR_CAPACITY;
  }
  for (int i = count; i <= POLYQ_MAX_BATCH; ++i) a.wg_begin[i] = static_cast<int32_t>(wg);
  // Permuted copies (one per distinct (x, perm, factors), all in one launch),
  // then the products.
  ShuffleJob jobs[POLYQ_MAX_BATCH];
  int njobs = 0;
  for (int i = 0; i < count; ++i) {
    if (p.region[i] < 0) continue;
    bool first = true;
    for (int j = 0; j < i; ++j) first = first && p.region[j] != p.region[i];
    if (first)
      jobs[njobs++] = ShuffleJob{items[i].perm, items[i].xscale, items[i].x,
                                 reinterpret_cast<uint16_t*>(ws + p.region[i]), items[i].layout->k, 0};
  }
  launch_shuffle(jobs, njobs, m, true, st);
  SumArgs sum;
  memset(&sum, 0, sizeof(sum));
  sum.splits = p.shape.splits;
  int64_t widest = 0;
  for (int i = 0; i < count; ++i) {
    const polyq_gemv_item& itm = items[i];
    const polyq_layout& L = *itm.layout;
    GemmItem& g = a.item[i];
    sum.partial[i] = reinterpret_cast<const float*>(ws + p.partial[i]);
    sum.y[i] = itm.y;
    sum.count[i] = static_cast<int64_t>(m) * L.n;
    widest = std::max(widest, sum.count[i]);
    g.packed = static_cast<const uint8_t*>(itm.packed);
    g.x = p.region[i] >= 0 ? reinterpret_cast<const uint16_t*>(ws + p.region[i]) : itm.x;
    g.y = p.shape.splits > 1 ? reinterpret_cast<float*>(ws + p.partial[i]) : itm.y;
    g.n = L.n;
    g.k = L.k;
    g.nblocks = L.nblocks;
    g.n_tiles = L.n_tiles;
    g.groups = layout_groups(L);
    g.y_vec = (L.n % 4 == 0 && reinterpret_cast<uintptr_t>(g.y) % 16 == 0) ? 1 : 0;
    for (int b = 0; b < L.nblocks; ++b) {
      g.bits[b] = L.block[b].bits;
      g.len[b] = L.block[b].len;
      g.k0[b] = L.k_begin[b];
      g.off[b] = static_cast<int32_t>(L.block_offset[b]);
      g.tb[b] = static_cast<int32_t>(L.tile_bytes[b]);
    }
  }
  launch_gemm<1>(p.shape.nt, wg, a, st);
  if (p.shape.splits > 1)
    hipLaunchKernelGGL(sum_splits_kernel, dim3(static_cast<unsigned>((widest + 1023) / 1024), count), dim3(256), 0, st,
                       sum);
  return hipGetLastError() == hipSuccess ? POLYQ_OK : POLYQ_ERR_DEVICE;
}

extern "C" polyq_status polyq_gemm(const polyq_layout* layout, const void* packed,
                                   const int32_t* perm, const uint16_t* x, int32_t m, float* y,
                                   void* workspace, size_t workspace_bytes, void* stream) {
  const polyq_gemm_item item{layout, packed, perm, x, y, nullptr};
  return polyq_gemm_batch(&item, 1, m, workspace, workspace_bytes, stream);
}
