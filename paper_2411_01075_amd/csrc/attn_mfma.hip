// Tiled attention forward and backward on the gfx950 matrix cores (bf16 operands, fp32 softmax
// and accumulation).  The S x S score matrix never reaches HBM: forward keeps a running row
// maximum and row sum (online softmax) and stores only the per-row log-sum-exp; backward
// recomputes the probabilities from Q, K and that log-sum-exp.
//
// Orientation.  v_mfma_f32_32x32x16_bf16 leaves each lane with ONE column of the 32x32 result
// (column lane%32) and 16 of its rows.  Every product is arranged so that the column is the
// index whose per-row statistics are needed and the rows are the index contracted next:
//   forward / dQ : S^T[t][q] = K Q^T  -> lane owns query q: max, sum, lse[q], rowsum(dO*O)[q] are
//                  lane scalars; the rows t feed the next product (O^T = V^T P^T, dQ^T = K^T dS^T)
//                  straight from registers as its B operand.
//   dK / dV      : S[q][t] = Q K^T    -> lane owns key t; rows q feed dV^T = dO^T P, dK^T = Q^T dS.
// The other operand of those second products (V^T, K^T, dO^T, Q^T: d-major views of row-major
// [token][d] tiles) is fetched from LDS with the transposing read ds_read_b64_tr_b16.
#include <type_traits>
#include <utility>
#include "kernels.h"
#include "reserve_lds.h"

namespace cephalo {
namespace {

typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))
typedef LDS_AS bf16 lds_bf16;

constexpr int kThreads = 256;
constexpr int TILE = 64;            // tokens per LDS tile
constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kLn2 = 0.69314718055994530942f;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// the same descriptor as four words (base, base high half with stride 0, extent, flags), for inline assembly
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 make_rsrc_words(const void* p, unsigned bytes) {
  const uint64_t addr = (uint64_t)(uintptr_t)p;
  return i32x4{(int)(unsigned)addr, (int)(unsigned)((addr >> 32) & 0xffffu), (int)bytes, 0x00020000};
}

// ROWS tokens by D values (D = 32, 64 or 128) of one operand in LDS, staged by THREADS threads straight from global memory.
//
// Rows are 2 D bytes without padding, so that a direct-to-LDS load of 16 bytes per lane fills 1 KiB = 512 / D whole rows at once; bank
// conflicts are avoided by permuting the 16-byte chunks of a row, chunk c of row r lives at chunk  c ^ swz(r);  the permutation is
// applied by the address each lane fetches.  16 consecutive rows put the same chunk on 16 different places of the 64 banks (fragment
// reads: 1, 2 or 4 rows share a line of all banks), and 4 consecutive rows put four neighbouring chunks on disjoint places
// (transposing reads):
//     D = 128   swz(r) = ((r & 7) << 1) | ((r >> 3) & 1)
//     D =  64   swz(r) = (((r >> 1) & 1) << 2) | ((r >> 2) & 3)
//     D =  32   swz(r) = (r >> 2) & 3
// (With padded rows only 4-byte-per-lane loads fit a row, and those run at a quarter of the rate; through registers, as the
// 64-wide tiles used to be staged, the loads cost 16 registers and an LDS write each.)
template <int D, int ROWS = TILE, int THREADS = kThreads> struct Tile {
  static constexpr int LD = D;
  static constexpr int ELEMS = ROWS * LD;
  __device__ static constexpr int swz(int r) {
    return D == 128 ? ((r & 7) << 1) | ((r >> 3) & 1) : D == 64 ? (((r >> 1) & 1) << 2) | ((r >> 2) & 3) : (r >> 2) & 3;
  }
  static constexpr int FLIP8 = D == 128 ? 1 : 2;          // swz(r + 8) = swz(r) ^ FLIP8 for r < 8

  // rsrc covers exactly one sample of the [*, ld_bytes/2] matrix, col_bytes is the head's
  // column offset.  Rows past the sample's end and chunks past the head's own width d are beyond the buffer's range
  // (every part of the address is in the range-checked offset): the hardware makes them zeros; callers mask such keys.
  // The loads are asynchronous: wait for vmcnt(0) and a workgroup barrier before reading the tile.
  static constexpr int NW = THREADS / 64, RPL = 512 / D, LOADS = ROWS / RPL, PER_WAVE = LOADS >= NW ? LOADS / NW : 1;      // RPL: rows per load
  static_assert(LOADS % NW == 0 || NW % LOADS == 0, "loads split evenly over the wavefronts");
  // the part of the offset that belongs to the lane (the same for every tile: the compiler keeps it out of the loops)
  // (wave: this wavefront's place among the THREADS / 64 that stage the tile; by default its place in the block)
  __device__ static unsigned stage_lane(int j, unsigned ld_bytes, int d, int wave = -1) {
    if (wave < 0) wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int row = (wave * PER_WAVE + j) * RPL + lane / (D / 8);
    const int c = (lane % (D / 8)) ^ swz(row);
    return c * 8 < d ? (unsigned)row * ld_bytes + (unsigned)c * 16 : 0x80000000u;
  }
  // The loads are issued behind the compiler's back: it tracks loads that write LDS, cannot tell one buffer from
  // another, and makes later LDS reads of the tile being multiplied wait for them (the whole memory latency, every
  // tile).  Callers wait (vmcnt(0)) and synchronise before they read what was staged.
  __device__ static void stage_one(i32x4 rsrc, int j, unsigned tile_bytes, unsigned ld_bytes, lds_bf16* lds, int d) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (LOADS < NW && wave >= LOADS) return;               // (a tile with fewer loads than wavefronts)
    const unsigned dst = (unsigned)(uintptr_t)(lds + (wave * PER_WAVE + j) * RPL * LD);
    const unsigned off = stage_lane(j, ld_bytes, d) + tile_bytes;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(off), "s"(rsrc) : "m0");
  }
  __device__ static void stage(i32x4 rsrc, unsigned col_bytes, unsigned ld_bytes, int row0, lds_bf16* lds, int d) {
#pragma unroll
    for (int j = 0; j < PER_WAVE; ++j) stage_one(rsrc, j, (unsigned)row0 * ld_bytes + col_bytes, ld_bytes, lds, d);
  }
  // operand with MFMA rows = tile rows [rb, rb+32), contraction over d in [kk, kk+16)   (rb: a multiple of 16 rows from
  // the tile's first row, so that a row's place in its group of 16 is the lane's)
  __device__ static bf16x8 frag_rows(const lds_bf16* lds, int rb, int kk) {
    const int lane = threadIdx.x & 63;
    // chunk (kk/8 + h) ^ swz = (kk/8) ^ (h ^ swz): the lane's part once, the fragment's part as an XOR of the byte address
    const unsigned own = (unsigned)(lane & 31) * (LD * 2) + (unsigned)(((lane >> 5) ^ swz(lane & 15)) << 4);
    return *reinterpret_cast<const LDS_AS bf16x8*>((const LDS_AS char*)lds + rb * (LD * 2) + (own ^ (unsigned)(kk * 2)));
  }
  // operand with MFMA rows = d in [db, db+32), contraction over 16 tile rows in the order the
  // accumulator of a preceding 32x32 product holds them: slot 4c+i of half-wave h is tile row
  // tb + 8c + 4h + i  (tb = first of the 16 rows, a multiple of 16 rows from the tile's first row)
  __device__ static bf16x8 frag_cols(const lds_bf16* lds, int db, int tb) {
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, i = lane & 15;
    // rows r and r + 8 (r < 8): the second read is the first with a chunk bit flipped
    const int r = 4 * (g >> 1) + (i >> 2);
    const unsigned own = (unsigned)r * (LD * 2) + (unsigned)(((2 * (g & 1) + ((i & 3) >> 1)) ^ swz(r)) << 4) + 8u * (i & 1);
    const LDS_AS char* p0 = (const LDS_AS char*)lds + tb * (LD * 2);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(p0 + (own ^ (unsigned)(db * 2))));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(p0 + 8 * (LD * 2) + ((own ^ (16u * FLIP8)) ^ (unsigned)(db * 2))));
    union { struct { s16x4 a, b; } s; bf16x8 v; } u;
    u.s.a = lo; u.s.b = hi;
    return u.v;
  }
};

// Which (tile pair, head, sample) a block works on.  Blocks are dealt round-robin to the 8 XCDs, each with an L2 of its
// own, and the blocks of one head (its query-tile pairs) all stream that head's keys and values: dealt out in launch
// order they land on 8 different XCDs, every XCD fetches every head's keys and values from memory and every staged
// tile pays the full memory latency.  Give each XCD a contiguous run of the (pair, head, sample) order instead, so the
// blocks of a head sit behind one L2: the first to ask for a tile brings it in, the others hit.
struct BlockCoords { int x, y, z; };
__device__ __forceinline__ BlockCoords block_coords(int l, int gx, int gy, int n) {      // (block l of n, gx tiles by gy heads by samples)
  l = (l & 7) * (n >> 3) + min(l & 7, n & 7) + (l >> 3);      // (the first n % 8 runs are one longer)
  // (the divisions run on the vector unit; readfirstlane tells the compiler that the results are uniform)
  return {__builtin_amdgcn_readfirstlane(l % gx), __builtin_amdgcn_readfirstlane((l / gx) % gy), __builtin_amdgcn_readfirstlane(l / (gx * gy))};
}
__device__ __forceinline__ int block_index() { return blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z); }
__device__ __forceinline__ BlockCoords block_coords() {
  const int gx = gridDim.x, gy = gridDim.y;
  return block_coords(block_index(), gx, gy, gx * gy * gridDim.z);
}

// The order in which a causal launch of the four-wavefront kernels takes its tiles (the work of a tile grows with the keys its queries see):
//   kSingle  one tile per block, the longest of a head first
//   kPaired  a block takes a tile and then its mirror image, so that every block does the same work
//   kByHead  one tile per block; each XCD has an eighth of the heads (some one more than others: y < 0, nothing to do) and takes the longest tiles of
//            all of them first (grid 8 * heads of an XCD * tiles)
// With several blocks on a compute unit pairs leave it idle at the end (600 pairs are 2.3 per compute unit); single tiles, the longest first, even
// out.  6 x 1024 tokens, 25 heads of 64, kPaired -> kByHead, us: forward 41.2 -> 35.5, backward 123 -> 102; 2048 tokens, 80 heads of 32: 50.0 -> 42.2
// and 122 -> 109; 4096 tokens, 50 heads of 64: backward 464 -> 411.
struct TileOrder { int kind, tiles, heads, blocks; };      // tiles: of a head, or pairs of them; blocks: of the whole order
enum { kSingle = 0, kPaired = 1, kByHead = 2 };
__device__ __forceinline__ BlockCoords ordered_coords(const TileOrder& order, int A, int l) {
  if (order.kind != kByHead) return block_coords(l, order.tiles, A, order.blocks);
  const int xcd = l & 7, i = l >> 3, per = (order.heads + 7) >> 3, at = i % per;
  const int first = (int)((int64_t)xcd * order.heads >> 3), count = (int)((int64_t)(xcd + 1) * order.heads >> 3) - first, head = first + at;
  return {__builtin_amdgcn_readfirstlane(i / per), __builtin_amdgcn_readfirstlane(at < count ? head % A : -1), __builtin_amdgcn_readfirstlane(head / A)};
}

// The LDS addresses of one lane's fragment reads (Tile::frag_rows / frag_cols) for two double-buffered tiles A and B that lie [A | B][A | B]: a register
// per constant that the permutation XORs in, everything else in the instruction's offset, and one XOR each to turn to the other buffer.
// (Left to itself the compiler keeps an address per constant and buffer, or forms one per read, an instruction beside every product.)
template <int D> struct FragAddr {
  typedef Tile<D> TL;
  static constexpr unsigned TILE_BYTES = TL::ELEMS * 2, STAGE = 2 * TILE_BYTES;
  unsigned r[D / 16], lo[D / 32], hi[D / 32];
  __device__ __forceinline__ explicit FragAddr(const lds_bf16* first) {
    // The XORs need a multiple of 2 * STAGE.  The tiles are the first of the dynamic LDS, which begins at 0 as long as the kernel has no static LDS: a test
    // of the compiled kernels sees to that.
    const unsigned base = (unsigned)(uintptr_t)first;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));                       // (formed here, not kept from pass to pass)
    const int g = lane >> 4, i = lane & 15, row = 4 * (g >> 1) + (i >> 2);
    const unsigned rows = (unsigned)(lane & 31) * (D * 2) + (unsigned)(((lane >> 5) ^ TL::swz(lane & 15)) << 4);
    const unsigned cols = (unsigned)row * (D * 2) + (unsigned)(((2 * (g & 1) + ((i & 3) >> 1)) ^ TL::swz(row)) << 4) + 8u * (i & 1);
#pragma unroll
    for (int k = 0; k < D / 16; ++k) r[k] = base + (rows ^ (unsigned)(k * 32));
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      lo[k] = base + (cols ^ (unsigned)(k * 64));
      hi[k] = base + (cols ^ (16u * TL::FLIP8) ^ (unsigned)(k * 64));
    }
  }
  __device__ __forceinline__ void flip() {
#pragma unroll
    for (int k = 0; k < D / 16; ++k) { r[k] ^= STAGE; asm volatile("" : "+v"(r[k])); }
#pragma unroll
    for (int k = 0; k < D / 32; ++k) { lo[k] ^= STAGE; hi[k] ^= STAGE; asm volatile("" : "+v"(lo[k]), "+v"(hi[k])); }
  }
  // rows [rb, rb + 32) of tile A (0) or B (1), contraction over d in [16 k, 16 k + 16)
  __device__ __forceinline__ bf16x8 rows(int tile, int rb, int k) const {
    return *(const LDS_AS bf16x8*)(uintptr_t)(r[k] + (unsigned)(tile * TILE_BYTES + rb * (D * 2)));
  }
  // d in [32 k, 32 k + 32), contraction over the 16 rows from tb on
  __device__ __forceinline__ bf16x8 cols(int tile, int k, int tb) const {
    const unsigned at = (unsigned)(tile * TILE_BYTES + tb * (D * 2));
    union { struct { s16x4 a, b; } s; bf16x8 v; } u;
    u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(uintptr_t)(lo[k] + at));
    u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(uintptr_t)(hi[k] + at + 8u * (D * 2)));
    return u.v;
  }
};

// fragment of 32 rows of a row-major [*, ld] matrix straight from global memory (rows = MFMA rows)
template <int D>
__device__ void load_row_frags(const bf16* __restrict__ g, int64_t ld, int row0, int nrows, bf16x8 (&f)[D / 16], int d) {
  const int lane = threadIdx.x & 63;
  const int row = row0 + (lane & 31);
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    bf16x8 val = {0, 0, 0, 0, 0, 0, 0, 0};
    const int c = kk * 16 + (lane >> 5) * 8;
    if (row < nrows && c < d) val = *reinterpret_cast<const bf16x8*>(g + (int64_t)row * ld + c);
    f[kk] = val;
  }
}

// Order hint for a run of N1 products whose LDS fragment is R1 ds_read instructions each, followed by N2 products
// with R2 reads each: the fragments of the first kAhead products are requested before the first product, then each
// product is followed by the request for the product kAhead places later.  (Left alone, the compiler waits for each
// fragment right before the product that uses it, and the matrix core idles for an LDS round trip every time.)
template <int N1, int R1, int N2 = 0, int R2 = 0>
__device__ __forceinline__ void lds_ahead_schedule() {
  constexpr int N = N1 + N2, kAhead = N1 < 4 ? N1 : 4;
  __builtin_amdgcn_sched_group_barrier(0x100, kAhead * R1, 0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (i + kAhead < N1) __builtin_amdgcn_sched_group_barrier(0x100, R1, 0);
    else if (i + kAhead < N) __builtin_amdgcn_sched_group_barrier(0x100, R2, 0);
  }
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int e0) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (bf16)v[e0 + i];
  return r;
}

// accumulator rows d (4 consecutive per group) of column token -> out[token][d0 + d], scaled
template <int D>
__device__ void store_transposed(const f32x16 (&acc)[D / 32], bf16* __restrict__ out, int64_t ld, int token, int ntokens, float mul, int d) {
  if (token >= ntokens) return;
  const int h = (threadIdx.x & 63) >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (bf16)(acc[dt][4 * j + i] * mul);
      const int d0 = dt * 32 + 8 * j + 4 * h;
      if (d0 < d) *reinterpret_cast<bf16x4*>(out + (int64_t)token * ld + d0) = v;      // (d is a multiple of 8: a group of 4 is in or out)
    }
}

// The same store for a gradient with respect to rotated queries or keys: each pair (2i, 2i+1) is first turned back by
// the angle of its position, rot[token][i] = (cos, sin), so that what is stored is the gradient before the rotation.
template <int D>
__device__ void store_transposed_unrotated(const f32x16 (&acc)[D / 32], bf16* __restrict__ out, int64_t ld, int token, int ntokens, float mul,
                                           const float* __restrict__ rot, int d) {
  asm volatile("" : "+v"(token));      // (the addresses are formed here: formed ahead, they are held through the whole pass and spill)
  if (token >= ntokens) return;
  const int h = (threadIdx.x & 63) >> 5;
  const f32x4* cs = reinterpret_cast<const f32x4*>(rot + (int64_t)token * d);      // d/2 pairs of (cos, sin) per position
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int d0 = dt * 32 + 8 * j + 4 * h;
      if (d0 >= d) continue;
      const f32x4 r = cs[d0 / 4];                                                   // pairs d0/2 and d0/2 + 1
      const float e0 = acc[dt][4 * j] * mul, o0 = acc[dt][4 * j + 1] * mul, e1 = acc[dt][4 * j + 2] * mul, o1 = acc[dt][4 * j + 3] * mul;
      bf16x4 v;
      v[0] = (bf16)(e0 * r[0] + o0 * r[1]);
      v[1] = (bf16)(o0 * r[0] - e0 * r[1]);
      v[2] = (bf16)(e1 * r[2] + o1 * r[3]);
      v[3] = (bf16)(o1 * r[2] - e1 * r[3]);
      *reinterpret_cast<bf16x4*>(out + (int64_t)token * ld + d0) = v;
    }
}

// f(0), f(1), .. f(N - 1) with the index as a type: products and what runs between them, unrolled whatever their number
template <typename F, int... I> __device__ __forceinline__ void static_steps_of(F& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F> __device__ __forceinline__ void static_steps(F f) { static_steps_of(f, std::make_integer_sequence<int, N>{}); }
// place AT of PLACES over which the work on 16 elements is spread
template <int AT, int PLACES, typename F> __device__ __forceinline__ void spread(F f) {
  if constexpr (AT >= 0 && AT < PLACES) {
#pragma unroll
    for (int e = AT * 16 / PLACES; e < (AT + 1) * 16 / PLACES; ++e) f(e);
  }
}

// Wavefronts per SIMD, that is blocks per compute unit, that the four-wavefront kernels are compiled for: as many as their registers allow without a
// spill.
template <int D, bool CAUSAL> constexpr int kFwdWaves = D == 128 ? 2 : D == 64 && CAUSAL ? 3 : 4;
template <int D> constexpr int kDqWaves = D == 32 ? 4 : D == 64 ? 3 : 2;
template <int D> constexpr int kDkvWaves = D == 32 ? 3 : 2;

// How the four-wavefront kernels (forward, dQ, and dK / dV of heads up to 64) run a tile.  What bounds them is three units in about equal measure: the
// matrix core, the vector unit (an exponential takes as long as half a 32x32x16 product) and waits for LDS and for one another.  A wavefront's products of a
// tile are one straight line, pinned product by product: fragments are asked for kAhead products early, and the exponentials of one block of 32
// scores go, a few after each product, between the products that do not need them.  Masking is a branch around a few selects (two copies of
// the whole tile, one masked, keep the accumulators in different registers: 64 moves and 130 spills), the tiles a wavefront has no work in are
// a loop of their own for the same reason, and fragment addresses are FragAddr's.  Eight wavefronts in step, their products and exponentials in phases of
// their own -> this form, us alone: forward 6 x 1024 tokens, 25 heads of 64, causal 45 -> 35; 2 x 1024, 8 heads of 128 26.5 -> 22.9; 8 x 512, 16 of 64 16.5 ->
// 15.5; backward 157 -> 104, 8 x 512, 16 of 64 54.7 -> 44.5, 16 x 197, 16 of 64 35.9 -> 29.0, 8 x 257, 16 of 104 60.1 -> 49.3, 2048, 80 of 32, causal 142 ->
// 112, 4 x 2048, 16 of 128, causal 286 -> 269 (dK / dV of 128, bound by LDS reads, did not gain by it and keeps its form).

// The sums of the two halves of a sample's keys, each relative to its own maximum, brought to a common one: rounded as the compiler rounds it in the
// eight-wavefront kernel (where, written like this, it would spill two registers); a test compares the bits of the two.
__device__ __forceinline__ float merged(float first, float a0, float second, float a1) { return __builtin_fmaf(first, a0, second * a1); }

// ------------------------------------------------------------------------------------ forward
template <int D, bool CAUSAL>
__global__ void __launch_bounds__(kThreads, (kFwdWaves<D, CAUSAL>))
attn_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ O, float* __restrict__ lse, int S, int H, int A, float scale, TileOrder order) {
  typedef Tile<D> TL;
  constexpr int NP = D / 16, DT = D / 32, N = 4 * NP, kAhead = 3;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_bf16* smem = (lds_bf16*)smem_raw;
  auto Ks = [&](int st) { return smem + st * 2 * TL::ELEMS; };
  auto Vs = [&](int st) { return smem + st * 2 * TL::ELEMS + TL::ELEMS; };

  const BlockCoords blk = ordered_coords(order, A, block_index());
  if (blk.y < 0) return;
  const int a = blk.y, n = blk.z;
  const int d = H / A;        // the head's own width: D, or less (a multiple of 8) with the tiles' further columns held at zero
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: tests on a wavefront's rows become real branches
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int64_t ld = 3 * (int64_t)H;
  const bf16* base = qkv + (int64_t)n * S * ld + a * d;
  const i32x4 rs_qkv = make_rsrc_words(qkv + (int64_t)n * S * ld, (unsigned)(S * ld * 2));
  const unsigned k_bytes = (unsigned)((H + a * d) * 2), v_bytes = (unsigned)((2 * H + a * d) * 2);
  const float c2 = scale * kLog2e;
  const int ntq = (S + 127) / 128;
  for (int pass = 0; pass < (CAUSAL && order.kind == kPaired ? 2 : 1); ++pass) {
  const int qt = pass == 0 && (order.kind == kPaired || !CAUSAL) ? blk.x : ntq - 1 - blk.x;
  if (pass == 1 && qt == blk.x) break;   // odd tile count: the middle tile is its own partner
  const int q0 = qt * 128 + wave * 32;             // this wavefront's 32 query rows
  const int q = q0 + (lane & 31);

  const int kv_end = CAUSAL ? min(S, qt * 128 + 128) : S;
  const int ntiles = (kv_end + TILE - 1) / TILE;
  bf16x8 qf[NP];
  load_row_frags<D>(base, ld, q0, S, qf, d);      // (before the staging: 16 x 197 tokens, 16 heads of 64 9.6 us, after it 10.3)
  TL::stage(rs_qkv, k_bytes, (unsigned)ld * 2, 0, Ks(0), d);
  TL::stage(rs_qkv, v_bytes, (unsigned)ld * 2, 0, Vs(0), d);
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wavefront's rows have landed
  __syncthreads();

  // Causal: the tiles of even index, then those of odd index, each half with a running maximum, sum and output of its own, as the eight-wavefront
  // form divides them between its groups: the same products in the same order, so the same bits.  (A probability is rounded to bf16 relative
  // to the maximum of its own half; relative to one maximum of all keys the rounding error is up to 5 % larger: 2048 tokens, heads of
  // 64, scores of standard deviation 5, 2.02e-3 against 1.92e-3 of the result.)
  const int nhalf = CAUSAL ? (ntiles + 1) / 2 : ntiles;      // tiles of the first half
  auto tile_of = [&](int i) { return !CAUSAL ? i : i < nhalf ? 2 * i : 2 * (i - nhalf) + 1; };
  FragAddr<D> at(smem);
  auto stage_after = [&](int i) {
    if (i + 1 >= ntiles) return;
    TL::stage(rs_qkv, k_bytes, (unsigned)ld * 2, tile_of(i + 1) * TILE, Ks((i + 1) & 1), d);
    TL::stage(rs_qkv, v_bytes, (unsigned)ld * 2, tile_of(i + 1) * TILE, Vs((i + 1) & 1), d);
  };
  auto close = [&] {
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
    __syncthreads();
  };
  const int mine = q0 >= S ? 0 : CAUSAL ? min(ntiles, (q0 + 31) / TILE + 1) : ntiles;      // (all, or all but the last of the second half)
  f32x16 o[DT], o_first[CAUSAL ? DT : 1];
  float m_run = -INFINITY, l_run = 0.f, m_first = -INFINITY, l_first = 0.f;
  int kt = 0;
  for (int half = 0; half < (CAUSAL ? 2 : 1); ++half) {
  if (half == 1) {
    m_first = m_run; l_first = l_run;
    m_run = -INFINITY; l_run = 0.f;
#pragma unroll
    for (int dt = 0; dt < (CAUSAL ? DT : 1); ++dt) o_first[dt] = o[dt];
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  for (const int upto = half == 0 ? min(nhalf, mine) : mine; kt < upto; ++kt) {
    const int t0 = tile_of(kt) * TILE;
    stage_after(kt);
    const bool mask = (CAUSAL && t0 + 63 > q0) || t0 + 64 > S;
    const int last = (CAUSAL ? min(q, S - 1) : S - 1) - t0 - 4 * h;
    // S^T of the two blocks of 32 keys, then O^T += V^T P^T of each
    auto fetch = [&](int i) -> bf16x8 {
      const int seg = i / NP, j = i % NP;
      if (seg < 2) return at.rows(0, seg * 32, j);
      return at.cols(1, j % DT, (seg - 2) * 32 + 16 * (j / DT));
    };
    bf16x8 f[kAhead], pf[2][2];
    f32x16 s[2], zero;
#pragma unroll
    for (int e = 0; e < 16; ++e) zero[e] = 0.f;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) f[i] = fetch(i);
    __builtin_amdgcn_sched_barrier(0);
    float psum = 0.f;
    float neg_m = 0.f;
    auto prob = [&](int b, int e) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][e], c2, neg_m));
      s[b][e] = p;
      psum += p;
    };
    static_steps<N>([&](auto step) {
      constexpr int i = decltype(step)::value, seg = i / NP, j = i % NP;
      if constexpr (seg < 2) s[seg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], qf[j], j == 0 ? zero : s[seg], 0, 0, 0);
      else o[j % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], pf[seg - 2][j / DT], o[j % DT], 0, 0, 0);
      if constexpr (i + kAhead < N) f[i % kAhead] = fetch(i + kAhead);
      if constexpr (i == 2 * NP - 1) {
        if (mask) {
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) s[b][e] = b * 32 + 8 * (e >> 2) + (e & 3) <= last ? s[b][e] : -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[b][e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;          // scores enter the exponent as s*c2 (c2 > 0)
        // Running maximum, in the log2 domain.  It is only raised when some row of the wavefront would otherwise see
        // an exponent above 8 (probabilities up to 2^8 are harmless in fp32 / bf16 and cancel in the final division);
        // raising it costs a pass over the output accumulators, and after the first tiles it is rarely needed.
        if (__any(mx > m_run + 8.0f)) {
          const float m_new = fmaxf(m_run, mx);
          const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
          l_run *= alpha;
          m_run = m_new;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
        }
        neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
#pragma unroll
        for (int e = 0; e < 16; ++e) prob(0, e);
        pf[0][0] = pack8(s[0], 0); pf[0][1] = pack8(s[0], 8);
      }
      spread<i - 2 * NP, NP>([&](int e) { prob(1, e); });
      if constexpr (i == 3 * NP - 1) { pf[1][0] = pack8(s[1], 0); pf[1][1] = pack8(s[1], 8); }
      __builtin_amdgcn_sched_barrier(0);
    });
    l_run += psum;
    at.flip();
    close();
  }
  }   // half
  for (; kt < ntiles; ++kt) {
    stage_after(kt);
    close();
  }
  if (CAUSAL) {
    const float m = fmaxf(m_first, m_run);
    const float a0 = (m_first == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_first - m);
    const float a1 = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] = merged(o_first[dt][e], a0, o[dt][e], a1);
    l_run = merged(l_first, a0, l_run, a1);
    m_run = m;
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = 1.0f / l_tot;
  store_transposed<D>(o, O + (int64_t)n * S * H + a * d, H, q, S, inv, d);
  if (h == 0 && q < S) lse[((int64_t)n * A + a) * S + q] = (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2;
  }   // pass
}

// ------------------------------------------------------------------------------------ forward, 8 wavefronts
// The same computation for launches of few blocks (heads of 64 or less, causal): 512 threads stage 128 keys per step, wavefronts 0-3 take the
// first 64 of them and wavefronts 4-7 the second 64, for the same four blocks of 32 queries.  Each half keeps its own
// running maximum, sum and output; at the end the second half hands them over through LDS and the first half merges
// (o = o0 2^(m0-m) + o1 2^(m1-m), likewise the sums).  While one wavefront of a SIMD runs its softmax on the vector
// unit the other's MFMAs keep the matrix core busy.
constexpr int kThreads8 = 512;
template <int D, bool CAUSAL>
__global__ void __launch_bounds__(kThreads8, 4)
attn_fwd8_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ O, float* __restrict__ lse, int S, int H, int A, float scale, int paired) {
  typedef Tile<D, 128, kThreads8> TL;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_bf16* smem = (lds_bf16*)smem_raw;
  auto Ks = [&](int st) { return smem + st * 2 * TL::ELEMS; };
  auto Vs = [&](int st) { return smem + st * 2 * TL::ELEMS + TL::ELEMS; };

  const BlockCoords blk = block_coords();
  const int a = blk.y, n = blk.z;
  const int d = H / A;        // the head's own width: D, or less (a multiple of 8) with the tiles' further columns held at zero
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: tests on a wavefront's rows become real branches
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int qsub = wave & 3, kh = wave >> 2;        // block of 32 queries, half of the staged keys
  const int64_t ld = 3 * (int64_t)H;
  const bf16* base = qkv + (int64_t)n * S * ld + a * d;
  const i32x4 rs_qkv = make_rsrc_words(qkv + (int64_t)n * S * ld, (unsigned)(S * ld * 2));
  const unsigned k_bytes = (unsigned)((H + a * d) * 2), v_bytes = (unsigned)((2 * H + a * d) * 2);
  const float c2 = scale * kLog2e;
  const int ntq = (S + 127) / 128;                  // causal, paired: query tile x, then its mirror tile (equal work per block)
  for (int pass = 0; pass < (CAUSAL && paired ? 2 : 1); ++pass) {
    const int qt = pass == 0 && (paired || !CAUSAL) ? blk.x : ntq - 1 - blk.x;      // (not paired: the longest first)
    if (pass == 1 && qt == blk.x) break;
    const int q0 = qt * 128 + qsub * 32;
    const int q = q0 + (lane & 31);

    bf16x8 qf[D / 16];
    load_row_frags<D>(base, ld, q0, S, qf, d);
    f32x16 o[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    const int kv_end = CAUSAL ? min(S, qt * 128 + 128) : S;
    const int ntiles = (kv_end + 127) / 128;
    TL::stage(rs_qkv, k_bytes, (unsigned)ld * 2, 0, Ks(0), d);
    TL::stage(rs_qkv, v_bytes, (unsigned)ld * 2, 0, Vs(0), d);
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): this wavefront's rows have landed
    __syncthreads();

    for (int kt = 0; kt < ntiles; ++kt) {
      const int cur = kt & 1;
      if (kt + 1 < ntiles) {                           // the next stage flies meanwhile
        TL::stage(rs_qkv, k_bytes, (unsigned)ld * 2, (kt + 1) * 128, Ks(cur ^ 1), d);
        TL::stage(rs_qkv, v_bytes, (unsigned)ld * 2, (kt + 1) * 128, Vs(cur ^ 1), d);
      }
      const int t0 = kt * 128 + kh * 64;            // this wavefront's 64 keys
      const lds_bf16* Kt = Ks(cur) + kh * 64 * TL::LD;
      const lds_bf16* Vt = Vs(cur) + kh * 64 * TL::LD;
      if (t0 < S && q0 < S && (!CAUSAL || t0 <= q0 + 31)) {
        f32x16 s[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
          for (int e = 0; e < 16; ++e) s[tb][e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
          for (int tb = 0; tb < 2; ++tb)     // the two key blocks accumulate in turn: no dependent accumulator back to back
            s[tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_rows(Kt, tb * 32, kk * 16), qf[kk], s[tb], 0, 0, 0);
        lds_ahead_schedule<D / 8, 1>();
        if ((CAUSAL && t0 + 63 > q0) || t0 + 64 > S) {      // diagonal or ragged end: per-element masking
#pragma unroll
          for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int t = t0 + tb * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
              if (t >= S || (CAUSAL && t > q)) s[tb][e] = -INFINITY;
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
          for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[tb][e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
        if (__any(mx > m_run + 8.0f)) {                       // lazy raise of the running maximum (log2 domain)
          const float m_new = fmaxf(m_run, mx);
          const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
          l_run *= alpha;
          m_run = m_new;
#pragma unroll
          for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
        }
        const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
        float psum = 0.f;
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[tb][e], c2, neg_m));
            s[tb][e] = p;
            psum += p;
          }
        l_run += psum;
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const bf16x8 pf = pack8(s[tb], 8 * jj);
#pragma unroll
            for (int dt = 0; dt < D / 32; ++dt)
              o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_cols(Vt, dt * 32, tb * 32 + 16 * jj), pf, o[dt], 0, 0, 0);
          }
        lds_ahead_schedule<D / 8, 2>();
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
      __syncthreads();
    }
    // merge the two key halves: [value index][lane] floats per block of queries, lanes contiguous
    constexpr int NV = D / 32 * 16 + 2;
    LDS_AS float* mrg = (LDS_AS float*)smem_raw + qsub * NV * 64 + lane;
    if (kh == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) mrg[(dt * 16 + e) * 64] = o[dt][e];
      mrg[(NV - 2) * 64] = m_run;
      mrg[(NV - 1) * 64] = l_run;
    }
    __syncthreads();
    if (kh == 0) {
      const float m1 = mrg[(NV - 2) * 64], l1 = mrg[(NV - 1) * 64];
      const float m = fmaxf(m_run, m1);
      const float a0 = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m);
      const float a1 = (m1 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m1 - m);
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = o[dt][e] * a0 + mrg[(dt * 16 + e) * 64] * a1;
      const float l = l_run * a0 + l1 * a1;
      const float l_tot = l + __shfl_xor(l, 32, 64);
      const float inv = 1.0f / l_tot;
      store_transposed<D>(o, O + (int64_t)n * S * H + a * d, H, q, S, inv, d);
      if (h == 0 && q < S) lse[((int64_t)n * A + a) * S + q] = (m + __builtin_amdgcn_logf(l_tot)) * kLn2;
    }
    __syncthreads();     // the merge area is staged over again by the next pass
  }
}

// The matrix-core step of one wavefront, written as an explicit pipeline: the LDS fragment of product i + kAhead is
// requested right after product i is issued, into the register product i just freed.  PV: the 16 products
// O^T += V^T P^T of the tile before (fragments by transposing reads); QK: the 16 products S^T = K Q^T of this tile.
// `between(i)` runs after product i is issued (the staging loads of the next tiles are dealt out there, a few at a time:
// issued in one bunch they hold the wavefront until the memory pipeline has taken them all).
template <int D, bool PV, bool QK, typename TL, typename Between>
__device__ __forceinline__ void turn_products(const lds_bf16* Vt, const lds_bf16* Kt, const bf16x8 (&pf)[2][2], const bf16x8 (&qf)[D / 16],
                                              f32x16 (&o)[D / 32], f32x16 (&s)[2], Between between) {
  static_assert(D == 128, "16 + 16 products");
  constexpr int NPV = PV ? 16 : 0, N = NPV + (QK ? 16 : 0), kAhead = 4;      // (3 to 8 ahead measure the same)
  auto fetch = [&](int i) -> bf16x8 {
    if (i < NPV) return TL::frag_cols(Vt, (i % 4) * 32, (i / 8) * 32 + 16 * ((i / 4) % 2));
    const int j = i - NPV;
    return TL::frag_rows(Kt, (j % 2) * 32, (j / 2) * 16);
  };
  bf16x8 f[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) f[i] = fetch(i);
  if (QK) {
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[tb][e] = 0.f;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i < NPV) {
      o[i % 4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], pf[i / 8][(i / 4) % 2], o[i % 4], 0, 0, 0);
    } else {
      const int j = i - NPV;
      s[j % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], qf[j / 2], s[j % 2], 0, 0, 0);
    }
    if (i + kAhead < N) f[i % kAhead] = fetch(i + kAhead);
    between(i);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ------------------------------------------------------------------------------------ forward, two groups in turns
// The eight-wavefront forward above leaves its two groups in step: the barrier of every key tile starts them together,
// so both multiply at the same time (sharing the matrix core) and then both run their softmax at the same time (sharing
// the vector unit) -- a tile costs the sum of the two, not the larger.  Here the groups take turns.  Time is cut into
// phases closed by a barrier; in a phase one group multiplies (the products of its softmax of the tile before, then the
// scores of the next tile) while the other runs its softmax, and in the next phase they swap:
//   step 2k   of a group:  O^T += V_{k-1}^T P_{k-1}^T ;  S_k^T = K_k Q^T        (matrix core, LDS reads)
//   step 2k+1 of a group:  P_k = softmax piece of S_k                            (vector unit)
// group 0 runs step p in phase p, group 1 runs step p-1.  K_{k+1} and V_k are staged during phases 2k and 2k+1 (V is
// wanted one tile later than K now) into the buffers that K_{k-1} and V_{k-2} left at the end of phase 2k-1: group 0
// issues the loads between the products of its step 2k and waits for them at the end of phase 2k+1.  The staging
// loads are issued behind the compiler's back (it would make the next transposing LDS read wait for them).
template <int D, bool CAUSAL>
__global__ void __launch_bounds__(kThreads8)
attn_fwd_turns_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ O, float* __restrict__ lse, int S, int H, int A, float scale, int paired) {
  typedef Tile<D, 128, kThreads8> TL;
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_bf16* smem = (lds_bf16*)smem_raw;
  auto Ks = [&](int st) { return smem + st * 2 * TL::ELEMS; };
  auto Vs = [&](int st) { return smem + st * 2 * TL::ELEMS + TL::ELEMS; };

  const BlockCoords blk = block_coords();
  const int a = blk.y, n = blk.z;
  const int d = H / A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int qsub = wave & 3, kh = wave >> 2;
  const int64_t ld = 3 * (int64_t)H;
  const bf16* base = qkv + (int64_t)n * S * ld + a * d;
  const unsigned ld_bytes = (unsigned)ld * 2;
  const unsigned k_bytes = (unsigned)((H + a * d) * 2), v_bytes = (unsigned)((2 * H + a * d) * 2);
  const i32x4 rsrc = make_rsrc_words(qkv + (int64_t)n * S * ld, (unsigned)(S * ld * 2));
  // Staging is group 0's job (its four wavefronts split a tile's 32 load instructions: 8 each per operand), dealt out
  // between the products of its matrix-core step.  Load q of a tile pair: q < 8 the keys, else the values.
  typedef Tile<D, 128, 256> TS;
  unsigned lane_part[TS::PER_WAVE];
#pragma unroll
  for (int j = 0; j < TS::PER_WAVE; ++j) lane_part[j] = kh == 0 ? TS::stage_lane(j, ld_bytes, d) : 0x80000000u;
  auto stage_one = [&](int j, unsigned col_bytes, int row0, lds_bf16* lds) {
    const unsigned dst = (unsigned)(uintptr_t)(lds + (wave * TS::PER_WAVE + j) * 4 * TL::LD);
    const unsigned off = lane_part[j] + ((unsigned)row0 * ld_bytes + col_bytes);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(off), "s"(rsrc) : "m0");
  };
  const float c2 = scale * kLog2e;
  const int ntq = (S + 127) / 128;
  for (int pass = 0; pass < (CAUSAL && paired ? 2 : 1); ++pass) {
    const int qt = pass == 0 && (paired || !CAUSAL) ? blk.x : ntq - 1 - blk.x;
    if (pass == 1 && qt == blk.x) break;
    const int q0 = qt * 128 + qsub * 32;
    const int q = q0 + (lane & 31);

    bf16x8 qf[D / 16];
    load_row_frags<D>(base, ld, q0, S, qf, d);
    f32x16 o[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    const int kv_end = CAUSAL ? min(S, qt * 128 + 128) : S;
    const int ntiles = (kv_end + 127) / 128;
    // this wavefront's 64 keys of tile k start at t0(k); the piece is skipped when it lies wholly past the queries
    auto first_key = [&](int k) { return k * 128 + kh * 64; };
    auto wanted = [&](int k) { const int t0 = first_key(k); return k < ntiles && t0 < S && (!CAUSAL || t0 <= q0 + 31); };

    if (kh == 0) {
#pragma unroll
      for (int j = 0; j < TS::PER_WAVE; ++j) stage_one(j, k_bytes, 0, Ks(0));
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
    __syncthreads();

    f32x16 s[2];
    bf16x8 pf[2][2];
    // the matrix-core step for tile k (products of tile k-1's probabilities, then tile k's scores)
    // (tile k's scores come from K buffer k & 1, tile k-1's values from V buffer (k - 1) & 1)
    auto Vprev = [&](int k) { return Vs((k + 1) & 1) + kh * 64 * TL::LD; };
    auto Kcur = [&](int k) { return Ks(k & 1) + kh * 64 * TL::LD; };
    // the vector-unit step for tile k
    auto soften = [&](int k) {
      if (!wanted(k)) {       // this wavefront's keys lie past its queries (or past the sequence): its products add nothing
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) pf[tb][jj] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        return;
      }
      const int t0 = first_key(k);
      if ((CAUSAL && t0 + 63 > q0) || t0 + 64 > S) {      // diagonal or ragged end: per-element masking
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int t = t0 + tb * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
            if (t >= S || (CAUSAL && t > q)) s[tb][e] = -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[tb][e]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
      if (__any(mx > m_run + 8.0f)) {                       // lazy raise of the running maximum (log2 domain)
        const float m_new = fmaxf(m_run, mx);
        const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
      }
      const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
      float psum = 0.f;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[tb][e], c2, neg_m));
          s[tb][e] = p;
          psum += p;
        }
      l_run += psum;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) pf[tb][jj] = pack8(s[tb], 8 * jj);
    };
    // load q (0..15) of the pair staged while tile k is multiplied: K of tile k+1, V of tile k
    auto stage_next = [&](int k, int q) {
      if (q < TS::PER_WAVE) { if (k + 1 < ntiles) stage_one(q, k_bytes, (k + 1) * 128, Ks((k + 1) & 1)); }
      else if (k < ntiles) stage_one(q - TS::PER_WAVE, v_bytes, k * 128, Vs(k & 1));
    };
    auto close_phase = [&](bool landed) {
      if (landed) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tiles staged in the phase before have landed
      __syncthreads();
    };
    // Every wavefront runs every product of the schedule (an unwanted piece multiplies zeros: it occurs only on the
    // diagonal tile), so the loop body is one straight line per group.
    auto nothing = [](int) {};
    if (kh == 0) {
      turn_products<D, false, true, TL>(nullptr, Kcur(0), pf, qf, o, s, [&](int i) { stage_next(0, i); });
      close_phase(false);
      soften(0);
      close_phase(true);
      for (int k = 1; k < ntiles; ++k) {
        turn_products<D, true, true, TL>(Vprev(k), Kcur(k), pf, qf, o, s, [&](int i) { if (i & 1) stage_next(k, i >> 1); });
        close_phase(false);
        soften(k);
        close_phase(true);
      }
      turn_products<D, true, false, TL>(Vprev(ntiles), nullptr, pf, qf, o, s, nothing);
      close_phase(false);
      close_phase(false);
    } else {
      close_phase(false);
      turn_products<D, false, true, TL>(nullptr, Kcur(0), pf, qf, o, s, nothing);
      close_phase(false);
      for (int k = 1; k < ntiles; ++k) {
        soften(k - 1);
        close_phase(false);
        turn_products<D, true, true, TL>(Vprev(k), Kcur(k), pf, qf, o, s, nothing);
        close_phase(false);
      }
      soften(ntiles - 1);
      close_phase(false);
      turn_products<D, true, false, TL>(Vprev(ntiles), nullptr, pf, qf, o, s, nothing);
      close_phase(false);
    }
    // merge the two key halves: [value index][lane] floats per block of queries, lanes contiguous
    constexpr int NV = D / 32 * 16 + 2;
    LDS_AS float* mrg = (LDS_AS float*)smem_raw + qsub * NV * 64 + lane;
    if (kh == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) mrg[(dt * 16 + e) * 64] = o[dt][e];
      mrg[(NV - 2) * 64] = m_run;
      mrg[(NV - 1) * 64] = l_run;
    }
    __syncthreads();
    if (kh == 0) {
      const float m1 = mrg[(NV - 2) * 64], l1 = mrg[(NV - 1) * 64];
      const float m = fmaxf(m_run, m1);
      const float a0 = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m);
      const float a1 = (m1 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m1 - m);
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = o[dt][e] * a0 + mrg[(dt * 16 + e) * 64] * a1;
      const float l = l_run * a0 + l1 * a1;
      const float l_tot = l + __shfl_xor(l, 32, 64);
      const float inv = 1.0f / l_tot;
      store_transposed<D>(o, O + (int64_t)n * S * H + a * d, H, q, S, inv, d);
      if (h == 0 && q < S) lse[((int64_t)n * A + a) * S + q] = (m + __builtin_amdgcn_logf(l_tot)) * kLn2;
    }
    __syncthreads();     // the merge area is staged over again by the next pass
  }
}

// rowsum(dO * O) of this lane's row (row0 + lane % 32), dO's row at hand
template <int D>
__device__ __forceinline__ float row_dot(const bf16* __restrict__ O, int64_t ld, int row0, int nrows, const bf16x8 (&dof)[D / 16], int d) {
  bf16x8 of[D / 16];
  load_row_frags<D>(O, ld, row0, nrows, of, d);
  float dv = 0.f;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e) dv = __builtin_fmaf((float)of[kk][e], (float)dof[kk][e], dv);
  return dv + __shfl_xor(dv, 32, 64);
}

// One wavefront's share of a key tile in the dQ kernel: 32 queries by 64 keys, as two blocks of 32 keys.
template <int D>
__device__ __forceinline__ void dq_tile(const FragAddr<D>& at, const bf16x8 (&qf)[D / 16], const bf16x8 (&dof)[D / 16], f32x16 (&dq)[D / 32],
                                        float c2, float lse2, float dv, bool mask, int last) {
  constexpr int NP = D / 16, N = 6 * NP, kAhead = 3, DT = D / 32;
  auto fetch = [&](int i) -> bf16x8 {
    const int seg = i / NP, j = i % NP;
    if (seg < 4) return at.rows(seg & 1, seg / 2 * 32, j);
    return at.cols(0, j % DT, (seg - 4) * 32 + 16 * (j / DT));
  };
  bf16x8 f[kAhead], df[2][2];
  f32x16 s[2], dp[2], zero;
#pragma unroll
  for (int e = 0; e < 16; ++e) zero[e] = 0.f;
#pragma unroll
  for (int i = 0; i < kAhead; ++i) f[i] = fetch(i);
  __builtin_amdgcn_sched_barrier(0);
  auto prob = [&](f32x16& s, int e) { s[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c2, -lse2)); };
  auto hide = [&](f32x16& s, int tb) {
    if (mask) {
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = tb * 32 + 8 * (e >> 2) + (e & 3) <= last ? s[e] : 0.f;
    }
  };
  static_steps<N>([&](auto step) {
    constexpr int i = decltype(step)::value, seg = i / NP, j = i % NP;
    if constexpr (seg == 0 || seg == 2) s[seg / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], qf[j], j == 0 ? zero : s[seg / 2], 0, 0, 0);
    else if constexpr (seg == 1 || seg == 3) dp[seg / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], dof[j], j == 0 ? zero : dp[seg / 2], 0, 0, 0);
    else dq[j % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], df[seg - 4][j / DT], dq[j % DT], 0, 0, 0);
    if constexpr (i + kAhead < N) f[i % kAhead] = fetch(i + kAhead);
    spread<i - NP - 1, NP>([&](int e) { prob(s[0], e); });
    spread<i - 2 * NP - 1, NP>([&](int e) { s[0][e] *= dp[0][e] - dv; });
    if constexpr (i == 3 * NP) { hide(s[0], 0); df[0][0] = pack8(s[0], 0); df[0][1] = pack8(s[0], 8); }
    spread<i - 3 * NP - 1, NP>([&](int e) { prob(s[1], e); });
    spread<i - 4 * NP - 1, NP - 1>([&](int e) { s[1][e] *= dp[1][e] - dv; });
    if constexpr (i == 5 * NP - 1) { hide(s[1], 1); df[1][0] = pack8(s[1], 0); df[1][1] = pack8(s[1], 8); }
    __builtin_amdgcn_sched_barrier(0);
  });
}

// ------------------------------------------------------------------------------------ dQ
// A block of four wavefronts owns 128 queries, 32 a wavefront, and walks the keys they see in tiles of 64.  (Eight wavefronts that split
// 128 keys, one block per compute unit, move in step between barriers: all multiply, then all run their exponentials.  Blocks that do not
// share a barrier drift apart.)
// The products are taken transposed (S^T = K Q^T, dP^T = V dO^T), so that a lane's 16 values belong to one query and
// its statistics are two scalars, and dS^T is at once the operand of dQ^T += K^T dS^T.
template <int D, bool CAUSAL, bool ROT>
__device__ __forceinline__ void dq_block(const bf16* __restrict__ qkv, const bf16* __restrict__ O, const bf16* __restrict__ dO, const float* __restrict__ lse,
                                         float* __restrict__ dvec, bf16* __restrict__ dqkv, int S, int H, int A, float scale,
                                         const float* __restrict__ rot, const BlockCoords& blk, bool paired) {
  typedef Tile<D> TL;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_bf16* smem = (lds_bf16*)smem_raw;
  auto Ks = [&](int st) { return smem + st * 2 * TL::ELEMS; };
  auto Vs = [&](int st) { return smem + st * 2 * TL::ELEMS + TL::ELEMS; };

  const int a = blk.y, n = blk.z;
  const int d = H / A;        // the head's own width: D, or less (a multiple of 8) with the tiles' further columns held at zero
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: tests on a wavefront's rows become real branches
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int64_t ld = 3 * (int64_t)H;
  const bf16* base = qkv + (int64_t)n * S * ld + a * d;
  const i32x4 rs_qkv = make_rsrc_words(qkv + (int64_t)n * S * ld, (unsigned)(S * ld * 2));
  const unsigned k_bytes = (unsigned)((H + a * d) * 2), v_bytes = (unsigned)((2 * H + a * d) * 2);
  const float c2 = scale * kLog2e;
  const int ntq = (S + 127) / 128;                 // causal, paired: query tiles x and ntq-1-x in turn (equal work per block)
  for (int pass = 0; pass < (CAUSAL && paired ? 2 : 1); ++pass) {
  const int qt = pass == 0 && (paired || !CAUSAL) ? blk.x : ntq - 1 - blk.x;      // (not paired: the longest first)
  if (pass == 1 && qt == blk.x) break;
  const int q0 = qt * 128 + wave * 32;
  const int q = q0 + (lane & 31);

  bf16x8 qf[D / 16], dof[D / 16];
  load_row_frags<D>(dO + (int64_t)n * S * H + a * d, H, q0, S, dof, d);
  const int64_t stat = ((int64_t)n * A + a) * S + q;
  const float dv = row_dot<D>(O + (int64_t)n * S * H + a * d, H, q0, S, dof, d);
  load_row_frags<D>(base, ld, q0, S, qf, d);
  const float lse2 = (q < S) ? lse[stat] * kLog2e : 0.f;
  if (h == 0 && q < S) dvec[stat] = dv;

  f32x16 dq[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[dt][e] = 0.f;

  const int kv_end = CAUSAL ? min(S, qt * 128 + 128) : S;
  const int ntiles = (kv_end + TILE - 1) / TILE;
  TL::stage(rs_qkv, k_bytes, (unsigned)ld * 2, 0, Ks(0), d);
  TL::stage(rs_qkv, v_bytes, (unsigned)ld * 2, 0, Vs(0), d);
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wavefront's rows have landed
  __syncthreads();

  FragAddr<D> at(smem);
  auto stage_after = [&](int kt) {                     // the next stage flies meanwhile
    if (kt + 1 >= ntiles) return;
    TL::stage(rs_qkv, k_bytes, (unsigned)ld * 2, (kt + 1) * TILE, Ks((kt + 1) & 1), d);
    TL::stage(rs_qkv, v_bytes, (unsigned)ld * 2, (kt + 1) * TILE, Vs((kt + 1) & 1), d);
  };
  auto close = [&] {
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
    __syncthreads();
  };
  // (the tiles whose keys the wavefront's queries see, then those it only helps to stage; one loop with the question inside copies the sums
  // from register to register every time)
  const int mine = q0 >= S ? 0 : CAUSAL ? min(ntiles, (q0 + 31) / TILE + 1) : ntiles;
  int kt = 0;
  for (; kt < mine; ++kt) {
    const int t0 = kt * TILE;
    stage_after(kt);
    dq_tile<D>(at, qf, dof, dq, c2, lse2, dv, (CAUSAL && t0 + 63 > q0) || t0 + 64 > S, (CAUSAL ? min(q, S - 1) : S - 1) - t0 - 4 * h);
    at.flip();
    close();
  }
  for (; kt < ntiles; ++kt) {
    stage_after(kt);
    close();
  }
  if (ROT) store_transposed_unrotated<D>(dq, dqkv + (int64_t)n * S * ld + a * d, ld, q, S, scale, rot, d);
  else store_transposed<D>(dq, dqkv + (int64_t)n * S * ld + a * d, ld, q, S, scale, d);
  }   // pass
}
template <int D, bool CAUSAL, bool ROT>
__global__ void __launch_bounds__(kThreads, kDqWaves<D>)
attn_dq_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ O, const bf16* __restrict__ dO, const float* __restrict__ lse,
               float* __restrict__ dvec, bf16* __restrict__ dqkv, int S, int H, int A, float scale,
               const float* __restrict__ rot, TileOrder order) {
  const BlockCoords blk = ordered_coords(order, A, block_index());
  if (blk.y < 0) return;
  dq_block<D, CAUSAL, ROT>(qkv, O, dO, lse, dvec, dqkv, S, H, A, scale, rot, blk, order.kind == kPaired);
}

// ------------------------------------------------------------------------------------ dK, dV
// A block owns 128 keys (causal: tile x, then its mirror tile) and walks the query tiles that see them.  Eight
// wavefronts: wavefront w takes the 32 keys of group w & 3 and, of every 64-query tile, the 32 queries of half w >> 2,
// so the two wavefronts of a SIMD work on different halves and one's exponentials run under the other's MFMAs.  Each
// half accumulates its own dK and dV; at the end of the pass the second half hands its sums over through LDS.
//
// The block's keys and values stay in LDS for the whole pass: held in registers (64 of them at D = 128) they push the
// kernel past 256 registers, where the accumulators move to the second register file and every score has to be copied
// back for the vector unit.  Query and dO tiles are double-buffered.
template <int D, bool CAUSAL, bool ROT>
__global__ void __launch_bounds__(kThreads8, 2)
attn_dkv_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dO, const float* __restrict__ lse,
                const float* __restrict__ dvec, bf16* __restrict__ dqkv, int S, int H, int A, float scale,
                const float* __restrict__ rot, int paired) {
  typedef Tile<D, TILE, kThreads8> TL;
  typedef Tile<D, 128, kThreads8> TKV;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_bf16* smem = (lds_bf16*)smem_raw;
  auto Qs = [&](int st) { return smem + st * 2 * TL::ELEMS; };
  auto dOs = [&](int st) { return smem + st * 2 * TL::ELEMS + TL::ELEMS; };
  lds_bf16* Ks = smem + 4 * TL::ELEMS;
  lds_bf16* Vs = Ks + TKV::ELEMS;
  LDS_AS float* stats = (LDS_AS float*)(Vs + TKV::ELEMS);   // [2 buffers][lse2 | dvec][64]

  const BlockCoords blk = block_coords();
  const int a = blk.y, n = blk.z;
  const int d = H / A;        // the head's own width: D, or less (a multiple of 8) with the tiles' further columns held at zero
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: tests on a wavefront's rows become real branches
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int kg = wave & 3, qh = wave >> 2;          // group of 32 keys, half of the query tile
  const int64_t ld = 3 * (int64_t)H;
  const bf16* base = qkv + (int64_t)n * S * ld + a * d;
  const bf16* dObase = dO + (int64_t)n * S * H + a * d;
  const i32x4 rs_qkv = make_rsrc_words(qkv + (int64_t)n * S * ld, (unsigned)(S * ld * 2));
  const i32x4 rs_do = make_rsrc_words(dO + (int64_t)n * S * H, (unsigned)((int64_t)S * H * 2));
  const unsigned col_bytes = (unsigned)(a * d * 2);
  const float* lse_base = lse + ((int64_t)n * A + a) * S;
  const float* dv_base = dvec + ((int64_t)n * A + a) * S;
  const float c2 = scale * kLog2e;
  const int ntk = (S + 127) / 128;                 // causal, paired: key tiles x and ntk-1-x in turn (early key tiles see the most queries)
  for (int pass = 0; pass < (CAUSAL && paired ? 2 : 1); ++pass) {
  const int tt = pass == 0 ? blk.x : ntk - 1 - blk.x;
  if (pass == 1 && tt == blk.x) break;
  const int t0 = tt * 128 + kg * 32;               // this wavefront's 32 keys
  const int t = t0 + (lane & 31);

  TKV::stage(rs_qkv, (unsigned)H * 2 + col_bytes, (unsigned)ld * 2, tt * 128, Ks, d);
  TKV::stage(rs_qkv, (unsigned)H * 4 + col_bytes, (unsigned)ld * 2, tt * 128, Vs, d);

  f32x16 dk[D / 32], dvv[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[dt][e] = 0.f; dvv[dt][e] = 0.f; }

  const int first = CAUSAL ? (tt * 128) / TILE : 0;    // first query tile that can see these keys
  const int ntiles = (S + TILE - 1) / TILE;
  float rstat = 0.f;                                   // threads 0..63: lse2, 64..127: dvec
  auto load_stats = [&](int row0) {
    rstat = 0.f;
    if (threadIdx.x < 128) {
      const int r = row0 + (threadIdx.x & 63);
      if (r < S) rstat = threadIdx.x < 64 ? lse_base[r] * kLog2e : dv_base[r];
    }
  };
  TL::stage(rs_qkv, col_bytes, (unsigned)ld * 2, first * TILE, Qs(0), d);
  TL::stage(rs_do, col_bytes, (unsigned)H * 2, first * TILE, dOs(0), d);
  load_stats(first * TILE);
  if (threadIdx.x < 128) stats[threadIdx.x] = rstat;
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wavefront's rows have landed
  __syncthreads();

  for (int it = first; it < ntiles; ++it) {
    const int cur = (it - first) & 1, qb0 = it * TILE;
    if (it + 1 < ntiles) {                             // the next tile flies into the other stage meanwhile
      TL::stage(rs_qkv, col_bytes, (unsigned)ld * 2, qb0 + TILE, Qs(cur ^ 1), d);
      TL::stage(rs_do, col_bytes, (unsigned)H * 2, qb0 + TILE, dOs(cur ^ 1), d);
      load_stats(qb0 + TILE);
    }
    const LDS_AS float* st = stats + cur * 128;
    const int q0 = qb0 + qh * 32;                      // this wavefront's 32 queries
    // (Without a mask, a wavefront whose queries or keys all lie past the end only stages.  Under the mask only the last query tile has
    // such, and asking in every tile costs more: 2 x 2048 tokens, 32 heads of 128, rotary 205 us instead of 195)
    if (CAUSAL ? q0 + 31 >= t0 : q0 < S && t0 < S) {
      constexpr int NP = D / 8;                        // products per phase
      // S and dP of the 32 queries x 32 keys
      f32x16 sc, dp;
#pragma unroll
      for (int e = 0; e < 16; ++e) { sc[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_rows(Qs(cur), qh * 32, kk * 16), TKV::frag_rows(Ks, kg * 32, kk * 16), sc, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_rows(dOs(cur), qh * 32, kk * 16), TKV::frag_rows(Vs, kg * 32, kk * 16), dp, 0, 0, 0);
      }
      lds_ahead_schedule<NP, 2>();
      __builtin_amdgcn_sched_barrier(0);
      // P = exp2(S c2 - lse2) and dS = P (dP - dvec) as bf16 operands.  They are not written back into the MFMA results.
      f32x16 pv, dsv;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = qh * 32 + 8 * j + 4 * h;         // 4 consecutive query rows
        const f32x4 l4 = *reinterpret_cast<const LDS_AS f32x4*>(st + r);
        const f32x4 d4 = *reinterpret_cast<const LDS_AS f32x4*>(st + 64 + r);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = 4 * j + i;
          pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], c2, -l4[i]));
          dsv[e] = dp[e] - d4[i];
        }
      }
      if ((CAUSAL && t0 + 31 > q0) || q0 + 32 > S) {    // diagonal or ragged end (wave-uniform): one branch around all the masking
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int qq = q0 + 8 * (e >> 2) + 4 * h + (e & 3);
          if (qq >= S || (CAUSAL && t > qq)) pv[e] = 0.f;
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) dsv[e] *= pv[e];
      // dV += P^T dO, dK += dS^T Q
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const bf16x8 pf = pack8(pv, 8 * jj), df = pack8(dsv, 8 * jj);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
          dvv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_cols(dOs(cur), dt * 32, qh * 32 + 16 * jj), pf, dvv[dt], 0, 0, 0);
          dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_cols(Qs(cur), dt * 32, qh * 32 + 16 * jj), df, dk[dt], 0, 0, 0);
        }
      }
      lds_ahead_schedule<NP, 2>();
    }
    if (it + 1 < ntiles && threadIdx.x < 128) stats[(cur ^ 1) * 128 + threadIdx.x] = rstat;
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
    __syncthreads();
  }
  // the second half's sums go through LDS ([key group][value][lane], lanes contiguous) and the first half stores
  constexpr int NV = D / 32 * 16 * 2;
  LDS_AS float* mrg = (LDS_AS float*)smem_raw + kg * NV * 64 + lane;
  if (qh == 1) {
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        mrg[(dt * 16 + e) * 64] = dk[dt][e];
        mrg[(NV / 2 + dt * 16 + e) * 64] = dvv[dt][e];
      }
  }
  __syncthreads();
  if (qh == 0) {
    bf16* out = dqkv + (int64_t)n * S * ld + a * d;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) dvv[dt][e] += mrg[(NV / 2 + dt * 16 + e) * 64];
    store_transposed<D>(dvv, out + 2 * H, ld, t, S, 1.0f, d);
    __builtin_amdgcn_sched_barrier(0);      // dv leaves its registers before dk's merge (and its rotary factors) need theirs
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) dk[dt][e] += mrg[(dt * 16 + e) * 64];
    if (ROT) store_transposed_unrotated<D>(dk, out + H, ld, t, S, scale, rot, d);
    else store_transposed<D>(dk, out + H, ld, t, S, scale, d);
  }
  __syncthreads();     // the merge area is staged over again by the next pass
  }   // pass
}

// ------------------------------------------------------------------------------------ dK, dV, heads of 64 or less
// Four wavefronts: a block owns 128 keys, each wavefront 32 of them, whose rows stay in its registers (at these widths they fit), and walks the
// query tiles of 64 that see them, as two blocks of 32 queries.
// OWN: the rows' statistics are formed here, kStatRows of them at a time and from O (dvec is not read), for a launch that runs beside the dQ blocks.
constexpr int kStatRows = 2048;
template <int D, bool CAUSAL, bool ROT, bool OWN>
__device__ __forceinline__ void dkv_block(const bf16* __restrict__ qkv, const bf16* __restrict__ O, const bf16* __restrict__ dO, const float* __restrict__ lse,
                                          const float* __restrict__ dvec, bf16* __restrict__ dqkv, int S, int H, int A, float scale,
                                          const float* __restrict__ rot, const BlockCoords& blk, bool paired) {
  typedef Tile<D> TL;
  constexpr int NP = D / 16, DT = D / 32, N = 8 * NP, kAhead = 3;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds_bf16* smem = (lds_bf16*)smem_raw;
  auto Qs = [&](int st) { return smem + st * 2 * TL::ELEMS; };
  auto dOs = [&](int st) { return smem + st * 2 * TL::ELEMS + TL::ELEMS; };
  LDS_AS float* stats = (LDS_AS float*)(smem + 4 * TL::ELEMS);      // [2 buffers][-lse / scale | -dvec][64], OWN: [-lse / scale | -dvec][kStatRows]

  const int a = blk.y, n = blk.z;
  const int d = H / A;        // the head's own width: D, or less (a multiple of 8) with the tiles' further columns held at zero
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: tests on a wavefront's rows become real branches
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int64_t ld = 3 * (int64_t)H;
  const bf16* base = qkv + (int64_t)n * S * ld + a * d;
  const i32x4 rs_qkv = make_rsrc_words(qkv + (int64_t)n * S * ld, (unsigned)(S * ld * 2));
  const i32x4 rs_do = make_rsrc_words(dO + (int64_t)n * S * H, (unsigned)((int64_t)S * H * 2));
  const unsigned col_bytes = (unsigned)(a * d * 2);
  const float* lse_base = lse + ((int64_t)n * A + a) * S;
  const float* dv_base = dvec + ((int64_t)n * A + a) * S;
  const float c2 = scale * kLog2e, per_scale = -1.0f / scale;
  const int ntk = (S + 127) / 128;                 // causal, paired: key tiles x and ntk-1-x in turn (early key tiles see the most queries)
  for (int pass = 0; pass < (CAUSAL && paired ? 2 : 1); ++pass) {
  const int tt = pass == 0 ? blk.x : ntk - 1 - blk.x;
  if (pass == 1 && tt == blk.x) break;
  const int t0 = tt * 128 + wave * 32;             // this wavefront's 32 keys
  const int t = t0 + (lane & 31);

  const int first = CAUSAL ? (tt * 128) / TILE : 0;    // first query tile that can see these keys
  const int ntiles = (S + TILE - 1) / TILE;
  float rstat = 0.f;                                   // threads 0..63: of lse, 64..127: of dvec
  auto load_stats = [&](int row0) {
    if (OWN) return;
    rstat = 0.f;
    if (threadIdx.x < 128) {
      const int r = row0 + (threadIdx.x & 63);
      if (r < S) rstat = threadIdx.x < 64 ? lse_base[r] * per_scale : -dv_base[r];
    }
  };
  TL::stage(rs_qkv, col_bytes, (unsigned)ld * 2, first * TILE, Qs(0), d);
  TL::stage(rs_do, col_bytes, (unsigned)H * 2, first * TILE, dOs(0), d);
  bf16x8 kf[NP], vf[NP];
  load_row_frags<D>(base + H, ld, t0, S, kf, d);
  load_row_frags<D>(base + 2 * H, ld, t0, S, vf, d);
  auto own_stats = [&](int row0, int end) {
    for (int r0 = row0 + wave * 32; r0 < end; r0 += 128) {
      const int r = r0 + (lane & 31), at = r % kStatRows;
      bf16x8 dof[NP];
      load_row_frags<D>(dO + (int64_t)n * S * H + a * d, H, r0, S, dof, d);
      const float dv = row_dot<D>(O + (int64_t)n * S * H + a * d, H, r0, S, dof, d), l = r < S ? lse_base[r] * per_scale : 0.f;
      if (h == 0) { stats[at] = l; stats[kStatRows + at] = -dv; }
    }
  };
  load_stats(first * TILE);
  if (!OWN && threadIdx.x < 128) stats[threadIdx.x] = rstat;

  f32x16 dk[DT], dvv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[dt][e] = 0.f; dvv[dt][e] = 0.f; }
  FragAddr<D> at(smem);
  auto stage_after = [&](int it) {                     // the next tile flies into the other stage meanwhile
    if (it + 1 >= ntiles) return;
    const int nxt = (it + 1 - first) & 1;
    TL::stage(rs_qkv, col_bytes, (unsigned)ld * 2, (it + 1) * TILE, Qs(nxt), d);
    TL::stage(rs_do, col_bytes, (unsigned)H * 2, (it + 1) * TILE, dOs(nxt), d);
    load_stats((it + 1) * TILE);
  };
  auto close = [&](int it) {
    if (!OWN && it + 1 < ntiles && threadIdx.x < 128) stats[((it + 1 - first) & 1) * 128 + threadIdx.x] = rstat;
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
    __syncthreads();
  };
  // (the tiles before the first whose queries see the wavefront's keys it only helps to stage; likewise all of them if its keys lie past the end)
  const int mine = t0 >= S ? ntiles : CAUSAL ? max(first, t0 / TILE) : first;
  int it = first;
  do {
  const int upto = OWN ? min(ntiles, (it / (kStatRows / TILE) + 1) * (kStatRows / TILE)) : ntiles;
  if (OWN) own_stats(it * TILE, upto * TILE);          // (those of the tiles before have been read: every tile ends with a barrier)
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wavefront's rows have landed
  __syncthreads();
  for (; it < min(mine, upto); ++it) {
    stage_after(it);
    at.flip();
    close(it);
  }
  for (; it < upto; ++it) {
    const int qb0 = it * TILE;
    stage_after(it);
    {
      const LDS_AS float* st = stats + (OWN ? qb0 % kStatRows : ((it - first) & 1) * 128) + 4 * h;
      constexpr int dvecs = OWN ? kStatRows : 64;
      // the products: S and dP of the first block and of the second, then dV and dK of each
      auto fetch = [&](int i) -> bf16x8 {
        const int seg = i / NP, j = i % NP;
        if (seg < 4) return at.rows(seg & 1, seg / 2 * 32, j);
        return at.cols(1 - (seg & 1), j % DT, (seg - 4) / 2 * 32 + 16 * (j / DT));
      };
      f32x16 s[2], dp[2];
      auto start = [&](f32x16& acc, int at) {           // a row's statistic is where its sums start
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 v = *reinterpret_cast<const LDS_AS f32x4*>(st + at + 8 * j);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[4 * j + i] = v[i];
        }
      };
      bf16x8 f[kAhead], pf[2][2], df[2][2];
      start(s[0], 0);
#pragma unroll
      for (int i = 0; i < kAhead; ++i) f[i] = fetch(i);
      start(dp[0], dvecs);
      __builtin_amdgcn_sched_barrier(0);
      const int seen = t - qb0 - 4 * h;                 // query rows from here on see the key
      auto hide = [&](f32x16& p, int b) {
        if (CAUSAL && t0 + 31 > qb0 + b * 32) {         // (the block touches the diagonal: wave-uniform)
#pragma unroll
          for (int e = 0; e < 16; ++e) p[e] = b * 32 + 8 * (e >> 2) + (e & 3) >= seen ? p[e] : 0.f;
        }
      };
      static_steps<N>([&](auto step) {
        constexpr int i = decltype(step)::value, seg = i / NP, j = i % NP;
        if constexpr (seg == 0 || seg == 2) s[seg / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], kf[j], s[seg / 2], 0, 0, 0);
        else if constexpr (seg == 1 || seg == 3) dp[seg / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], vf[j], dp[seg / 2], 0, 0, 0);
        else if constexpr (seg == 4 || seg == 6) dvv[j % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], pf[(seg - 4) / 2][j / DT], dvv[j % DT], 0, 0, 0);
        else dk[j % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kAhead], df[(seg - 4) / 2][j / DT], dk[j % DT], 0, 0, 0);
        if constexpr (i + kAhead < N) f[i % kAhead] = fetch(i + kAhead);
        if constexpr (i == NP) start(s[1], 32);
        if constexpr (i == 2 * NP) start(dp[1], dvecs + 32);
        // P = exp2(c2 (S - lse / scale)) and dS = P (dP - dvec)
        spread<i - NP - 1, NP>([&](int e) { s[0][e] = __builtin_amdgcn_exp2f(s[0][e] * c2); });
        if constexpr (i == 2 * NP) hide(s[0], 0);
        spread<i - 2 * NP - 1, NP - 1>([&](int e) { dp[0][e] *= s[0][e]; });
        if constexpr (i == 3 * NP - 1) {
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) { pf[0][jj] = pack8(s[0], 8 * jj); df[0][jj] = pack8(dp[0], 8 * jj); }
        }
        spread<i - 3 * NP, NP>([&](int e) { s[1][e] = __builtin_amdgcn_exp2f(s[1][e] * c2); });
        if constexpr (i == 4 * NP - 1) hide(s[1], 1);
        spread<i - 4 * NP - 1, NP - 1>([&](int e) { dp[1][e] *= s[1][e]; });
        if constexpr (i == 5 * NP - 1) {
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) { pf[1][jj] = pack8(s[1], 8 * jj); df[1][jj] = pack8(dp[1], 8 * jj); }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    at.flip();
    close(it);
  }
  } while (OWN && it < ntiles);
  bf16* out = dqkv + (int64_t)n * S * ld + a * d;
  store_transposed<D>(dvv, out + 2 * H, ld, t, S, 1.0f, d);
  if (ROT) store_transposed_unrotated<D>(dk, out + H, ld, t, S, scale, rot, d);
  else store_transposed<D>(dk, out + H, ld, t, S, scale, d);
  }   // pass
}
template <int D, bool CAUSAL, bool ROT>
__global__ void __launch_bounds__(kThreads, kDkvWaves<D>)
attn_dkv_narrow_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dO, const float* __restrict__ lse,
                       const float* __restrict__ dvec, bf16* __restrict__ dqkv, int S, int H, int A, float scale,
                       const float* __restrict__ rot, TileOrder order) {
  const BlockCoords blk = ordered_coords(order, A, block_index());
  if (blk.y < 0) return;
  dkv_block<D, CAUSAL, ROT, false>(qkv, nullptr, dO, lse, dvec, dqkv, S, H, A, scale, rot, blk, order.kind == kPaired);
}

// The whole backward of narrow heads in one launch, where two would not fill the chip: the dK / dV blocks first (they are the longer ones), then the dQ
// blocks, side by side instead of one after the other.  The statistics that the dK / dV kernel otherwise takes from the dQ kernel it forms itself,
// in the same order of additions, so that the choice does not show in the results.  Two launches -> one, heads of 64, us: 2 x 128 tokens, 4 heads 15.0 -> 9.1;
// 1024, 8 heads 41.7 -> 30.7; 4096, 8 132 -> 113.  Without a mask up to 512 tiles of short samples (16 x 197 tokens, 16 heads 29.7 -> 27.7) and 384 of
// longer ones (384 of 2048 112 -> 114, heads of 32 77 -> 66; 448 117 -> 137 and 80 -> 85).  Under a mask up to 512 tiles; from 257 on, of up to 16 tiles a head, by head (50 heads of 1024 tokens: two launches in
// pairs 57.6, by head 49.8, one by head 43.1, in pairs 45.2), of longer ones in pairs (16 heads of 4096: 158, 159, 148, 141).  Beyond, two launches win (64
// heads of 2048 142 and 161).
template <int D, bool CAUSAL, bool ROT>
__global__ void __launch_bounds__(kThreads, 2)
attn_bwd_small_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ O, const bf16* __restrict__ dO, const float* __restrict__ lse,
                      float* __restrict__ dvec, bf16* __restrict__ dqkv, int S, int H, int A, float scale, const float* __restrict__ rot, TileOrder order) {
  const bool second = (int)blockIdx.x >= order.blocks;
  const BlockCoords blk = ordered_coords(order, A, (int)blockIdx.x - (second ? order.blocks : 0));
  if (blk.y < 0) return;
  if (!second) dkv_block<D, CAUSAL, ROT, true>(qkv, O, dO, lse, nullptr, dqkv, S, H, A, scale, rot, blk, order.kind == kPaired);
  else dq_block<D, CAUSAL, ROT>(qkv, O, dO, lse, dvec, dqkv, S, H, A, scale, rot, blk, order.kind == kPaired);
}

// Causal launches of the eight-wavefront kernels: a block takes a tile and its mirror image (equal work per block) unless all tiles find a compute
// unit of their own at once: then the launch lasts as long as the longest tile, not as the longest and the shortest (8 heads of 80, 700 tokens, 48
// tiles: forward 22 -> 15 us, backward 61 -> 44).  Beyond that single tiles, longest first, lose (4 x 2048 tokens, 16 heads of 128).
inline bool pair_tiles(int nt, int A, int m) { return (int64_t)nt * A * m > 256; }
// a four-wavefront kernel's tiles in a given order, and the grid that goes with it.  By head only where no XCD has half as much again as it would at
// equal shares: 18 heads of 8192 tokens (three heads on an XCD, 2.25 at equal shares) 634 us by head, 674 in pairs; 9 heads (two, 1.1) 412 and 408.
inline dim3 tile_order(int kind, int nt, int A, int m, TileOrder* order) {
  const int64_t heads = (int64_t)A * m, per = (heads + 7) / 8;
  if (kind == kByHead && (2 * 8 * per > 3 * heads || 8 * per * nt >= (int64_t)1 << 31)) kind = kPaired;
  const int tiles = kind == kPaired ? (nt + 1) / 2 : nt;
  *order = {kind, tiles, (int)heads, (int)(kind == kByHead ? 8 * per * nt : heads * tiles)};
  return kind == kByHead ? dim3(order->blocks) : dim3(tiles, A, m);
}

// Forward.  Causal heads of 128: two groups that take turns.  Causal narrower heads: eight wavefronts, which split the keys between them and so
// halve the chain of a tile, where the launch consists of such chains, four where it has tiles enough to fill the chip with blocks of less; both give the
// same bits.  Us with eight and with four, heads of 64: 256 tiles of 1024 tokens 15.2 and 18.0, of 4096 42.6 and 55.7; 320 of 1024 19.6 and 18.7; 512 of
// 2048 28.8 and 32.7, 528 44.7 and 35.3 (eight: 256 pairs have a compute unit each, 257 do not); 640 of 4096 77.2 and 69.4, 1024 87.5 and 89.3, 1280 124
// and 108; 9 heads of 8192 141 and 151 (too few heads for four wavefronts' order), 18 227 and 221.
inline bool eight_wavefronts(int nt, int A, int m) {
  const int64_t tiles = (int64_t)nt * A * m;
  return tiles <= 256 || (nt > 8 && (tiles <= 512 || (int64_t)A * m < 16)) || (nt > 24 && tiles > 768 && tiles <= 1024);
}
template <int D, bool CAUSAL>
int fwd_cfg(const bf16* qkv, bf16* O, float* lse, int m, int S, int H, int A, hipStream_t s) {
  const int nt = (S + 127) / 128;
  const float scale = 1.0f / sqrtf((float)(H / A));
  if constexpr (CAUSAL) {
    if (D == 128 || eight_wavefronts(nt, A, m)) {
      const bool paired = pair_tiles(nt, A, m);
      dim3 grid(paired ? (nt + 1) / 2 : nt, A, m);
      const size_t staging = 4 * (size_t)Tile<D, 128, kThreads8>::ELEMS * sizeof(bf16), merge = (size_t)4 * (D / 32 * 16 + 2) * 64 * sizeof(float);
      const size_t lds = staging > merge ? staging : merge;
      constexpr auto kern = [] { if constexpr (D == 128) return attn_fwd_turns_kernel<D, CAUSAL>; else return attn_fwd8_kernel<D, CAUSAL>; }();
      int rc = reserve_lds<kern>("attention", lds);
      if (rc != CEPHALO_OK) return rc;
      kern<<<grid, kThreads8, lds, s>>>(qkv, O, lse, S, H, A, scale, paired);
      CEPHALO_CHECK_LAUNCH("attn_fwd_mfma");
      return CEPHALO_OK;
    }
  }
  if constexpr (!CAUSAL || D <= 64) {
    TileOrder order;
    const dim3 grid = tile_order(CAUSAL ? kByHead : kSingle, nt, A, m, &order);
    const size_t lds = 4 * (size_t)Tile<D>::ELEMS * sizeof(bf16);      // two stages of 64 keys and values
    constexpr auto kern = attn_fwd_kernel<D, CAUSAL>;
    int rc = reserve_lds<kern>("attention", lds);
    if (rc != CEPHALO_OK) return rc;
    kern<<<grid, kThreads, lds, s>>>(qkv, O, lse, S, H, A, scale, order);
  }
  CEPHALO_CHECK_LAUNCH("attn_fwd_mfma");
  return CEPHALO_OK;
}

template <int D, bool CAUSAL, bool ROT>
int bwd_cfg(const bf16* qkv, const bf16* O, const bf16* dO, const float* lse, float* dvec, bf16* dqkv,
            int m, int S, int H, int A, const float* rot, hipStream_t s) {
  const float scale = 1.0f / sqrtf((float)(H / A));
  const int nt = (S + 127) / 128;
  if constexpr (D <= 64) {
    const int64_t tiles = (int64_t)nt * A * m;
    if (tiles <= (CAUSAL || nt <= 4 ? 512 : 384)) {
      TileOrder order;
      (void)tile_order(!CAUSAL || tiles <= 256 ? kSingle : nt <= 16 ? kByHead : kPaired, nt, A, m, &order);
      const size_t lds = 4 * (size_t)Tile<D>::ELEMS * sizeof(bf16) + 2 * kStatRows * sizeof(float);
      constexpr auto kern = attn_bwd_small_kernel<D, CAUSAL, ROT>;
      int rc = reserve_lds<kern>("attention", lds);
      if (rc != CEPHALO_OK) return rc;
      kern<<<2 * order.blocks, kThreads, lds, s>>>(qkv, O, dO, lse, dvec, dqkv, S, H, A, scale, rot, order);
      CEPHALO_CHECK_LAUNCH("attn_bwd_mfma");
      return CEPHALO_OK;
    }
  }
  TileOrder order;
  // (heads of 128, whose dK / dV blocks have a compute unit each: dQ in pairs and by head, us of the whole backward: 12 heads of 4096 tokens 215 and 222, 64 of
  // 2048 268 and 268, 320 of 512 175 and 181, but 18 of 4096 408 and 396)
  const dim3 grid = tile_order(!CAUSAL ? kSingle : D <= 64 ? kByHead : pair_tiles(nt, A, m) ? kPaired : kSingle, nt, A, m, &order);
  {
    const size_t lds = 4 * (size_t)Tile<D>::ELEMS * sizeof(bf16);      // two stages of 64 keys and values
    constexpr auto kern = attn_dq_kernel<D, CAUSAL, ROT>;
    int rc = reserve_lds<kern>("attention", lds);
    if (rc != CEPHALO_OK) return rc;
    kern<<<grid, kThreads, lds, s>>>(qkv, O, dO, lse, dvec, dqkv, S, H, A, scale, rot, order);
  }
  if constexpr (D <= 64) {
    const size_t lds = 4 * (size_t)Tile<D>::ELEMS * sizeof(bf16) + 2 * 128 * sizeof(float);      // two stages of Q and dO and of the row statistics
    constexpr auto kern = attn_dkv_narrow_kernel<D, CAUSAL, ROT>;
    int rc = reserve_lds<kern>("attention", lds);
    if (rc != CEPHALO_OK) return rc;
    kern<<<grid, kThreads, lds, s>>>(qkv, dO, lse, dvec, dqkv, S, H, A, scale, rot, order);
  } else {
    // staging (2 stages of Q and dO, the keys, the values, the row statistics) or, at the end, the merge of the halves
    const size_t staging = (4 * (size_t)Tile<D>::ELEMS + 2 * (size_t)Tile<D, 128>::ELEMS) * sizeof(bf16) + 2 * 128 * sizeof(float);
    const size_t merge = (size_t)4 * (D / 32 * 16 * 2) * 64 * sizeof(float);
    const size_t lds = staging > merge ? staging : merge;
    constexpr auto kern = attn_dkv_kernel<D, CAUSAL, ROT>;
    int rc = reserve_lds<kern>("attention", lds);
    if (rc != CEPHALO_OK) return rc;
    kern<<<grid, kThreads8, lds, s>>>(qkv, dO, lse, dvec, dqkv, S, H, A, scale, rot, order.kind == kPaired);
  }
  CEPHALO_CHECK_LAUNCH("attn_bwd_mfma");
  return CEPHALO_OK;
}

template <int D>
int bwd_pick(const bf16* qkv, const bf16* O, const bf16* dO, const float* lse, float* dvec, bf16* dqkv,
             int m, int S, int H, int A, int causal, const float* rot, hipStream_t s) {
  if (rot) return causal ? bwd_cfg<D, true, true>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, rot, s)
                         : bwd_cfg<D, false, true>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, rot, s);
  return causal ? bwd_cfg<D, true, false>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, rot, s)
                : bwd_cfg<D, false, false>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, rot, s);
}

}  // namespace

int launch_attn_fwd_mfma(const bf16* qkv, bf16* O, float* lse, int m, int S, int H, int A, int causal, hipStream_t s) {
  const int D = A > 0 ? H / A : 0;
  if (H % 8 != 0 || !aligned16(qkv) || !aligned16(O)) return fail(CEPHALO_EINVAL, "attention: rows must be 16-byte aligned");
  if ((int64_t)S * 3 * H * 2 >= (int64_t)1 << 31)
    return fail(CEPHALO_EUNSUPPORTED, "attention: one sample of qkv (%lld bytes) exceeds the 2 GiB a buffer offset reaches", (long long)S * 3 * H * 2);
  // a head that is not 32, 64 or 128 wide runs on the next of these tiles with the further columns held at zero
  if (A <= 0 || H % A != 0 || D % 8 != 0 || D > 128)
    return fail(CEPHALO_EUNSUPPORTED, "attention (matrix-core kernel): head dim %d is not a multiple of 8 up to 128", A > 0 ? D : 0);
  if (D <= 32) return causal ? fwd_cfg<32, true>(qkv, O, lse, m, S, H, A, s) : fwd_cfg<32, false>(qkv, O, lse, m, S, H, A, s);
  if (D <= 64) return causal ? fwd_cfg<64, true>(qkv, O, lse, m, S, H, A, s) : fwd_cfg<64, false>(qkv, O, lse, m, S, H, A, s);
  return causal ? fwd_cfg<128, true>(qkv, O, lse, m, S, H, A, s) : fwd_cfg<128, false>(qkv, O, lse, m, S, H, A, s);
}

int launch_attn_bwd_mfma(const bf16* qkv, const bf16* O, const bf16* dO, const float* lse, float* dvec, bf16* dqkv,
                         int m, int S, int H, int A, int causal, hipStream_t s, const float* rot) {
  const int D = A > 0 ? H / A : 0;
  if (H % 8 != 0 || !aligned16(qkv) || !aligned16(O) || !aligned16(dO) || !aligned16(dqkv) || !aligned16(rot))
    return fail(CEPHALO_EINVAL, "attention: rows must be 16-byte aligned");
  if ((int64_t)S * 3 * H * 2 >= (int64_t)1 << 31)
    return fail(CEPHALO_EUNSUPPORTED, "attention: one sample of qkv (%lld bytes) exceeds the 2 GiB a buffer offset reaches", (long long)S * 3 * H * 2);
  if (A <= 0 || H % A != 0 || D % 8 != 0 || D > 128)
    return fail(CEPHALO_EUNSUPPORTED, "attention (matrix-core kernel): head dim %d is not a multiple of 8 up to 128", A > 0 ? D : 0);
  if (D <= 32) return bwd_pick<32>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, causal, rot, s);
  if (D <= 64) return bwd_pick<64>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, causal, rot, s);
  return bwd_pick<128>(qkv, O, dO, lse, dvec, dqkv, m, S, H, A, causal, rot, s);
}

}  // namespace cephalo
