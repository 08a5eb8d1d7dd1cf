// LayerNorm forward/backward and column sums (bias gradients): HBM-bound row kernels.
// Forward: one 64-lane wavefront owns a row; its lanes hold the row in registers as 16-byte
// vectors, and row statistics are wavefront reductions (no LDS, no block barrier).
// Backward: a team of one, two or four wavefronts shares each row (see ln_bwd_kernel).
// The residual stream (x, x1, y and their gradients) and the gradients entering LayerNorm's
// backward are fp32; LayerNorm outputs are in the activation type T.
#include "kernels.h"

namespace cephalo {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// N consecutive floats (N = 4 or 8) as 16-byte loads / stores
template <int N> __device__ __forceinline__ void load_f32(const float* p, float (&out)[N]) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int q = 0; q < N / 4; ++q) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + 4 * q);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[4 * q + i] = v[i];
  }
}
template <int N> __device__ __forceinline__ void store_f32(float* p, const float (&in)[N]) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int q = 0; q < N / 4; ++q) {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = in[4 * q + i];
    *reinterpret_cast<f32x4*>(p + 4 * q) = v;
  }
}

// RMS: root-mean-square norm instead (no mean subtraction, no beta: u = gamma * x / sqrt(mean(x^2) + eps)); the mean
// written is 0.
template <typename T, int MAXV, bool RMS>
__global__ void __launch_bounds__(kThreads)
ln_fwd_kernel(const float* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
              T* __restrict__ u, float* __restrict__ mean, float* __restrict__ rstd,
              int rows, int H, float eps) {
  constexpr int VN = Vec<T>::N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nv = H / VN;
  const float inv_h = 1.0f / (float)H;
  // Straight-line code: a lane whose 16-byte group lies past the row reads the row's first group instead and its
  // values are replaced by zeros; only the stores are predicated.  (With each group's loads under its own bounds
  // branch the compiler waited for one group before it asked for the next, and for every group's store before the next
  // group's gamma and beta: eight memory round trips in a row per row of the matrix.)
  typedef typename Vec<T>::raw RawT;
  for (int row = blockIdx.x * kWaves + wave; row < rows; row += gridDim.x * kWaves) {
    const float* xr = x + (int64_t)row * H;
    float vals[MAXV][VN];
    RawT gr[MAXV], br[MAXV];
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int v = lane + 64 * j, vc = v < nv ? v : 0;
      load_f32<VN>(xr + vc * VN, vals[j]);
    }
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const bool ok = lane + 64 * j < nv;
#pragma unroll
      for (int i = 0; i < VN; ++i) { vals[j][i] = ok ? vals[j][i] : 0.f; sum += vals[j][i]; }
    }
    const float mu = RMS ? 0.f : wave_sum(sum) * inv_h;
    // gamma and beta (in L2: every row reads the same) are asked for here, all at once, and arrive under the second
    // reduction; asked for with the row they cost 50 registers more and a third of the rows in flight per SIMD
    constexpr bool EARLY = MAXV <= 8;      // (the widest rows: no registers for that either, they load them group by group)
    if (EARLY) {
#pragma unroll
      for (int j = 0; j < MAXV; ++j) {
        const int v = lane + 64 * j;
        int vc = v < nv ? v : 0;
        asm volatile("" : "+v"(vc));      // (kept here: they do not depend on the row, and the compiler would move them above the row's own loads)
        gr[j] = *reinterpret_cast<const RawT*>(gamma + vc * VN);
        if (!RMS) br[j] = *reinterpret_cast<const RawT*>(beta + vc * VN);
      }
    }
    float sq = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const bool ok = lane + 64 * j < nv;
#pragma unroll
      for (int i = 0; i < VN; ++i) { const float d = ok ? vals[j][i] - mu : 0.f; sq += d * d; }
    }
    const float rs = 1.0f / sqrtf(wave_sum(sq) * inv_h + eps);
    T* ur = u + (int64_t)row * H;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int v = lane + 64 * j, vc = v < nv ? v : 0;
      if (!EARLY) {
        gr[j] = *reinterpret_cast<const RawT*>(gamma + vc * VN);
        if (!RMS) br[j] = *reinterpret_cast<const RawT*>(beta + vc * VN);
      }
      float o[VN];
#pragma unroll
      for (int i = 0; i < VN; ++i) o[i] = (float)gr[j][i] * ((vals[j][i] - mu) * rs) + (RMS ? 0.f : (float)br[j][i]);
      if (v < nv) store_vec<T>(ur + v * VN, o);
    }
    if (lane == 0) { mean[row] = mu; rstd[row] = rs; }
  }
}

constexpr int kLnBwdRowsPerBlock = 8;

// out = resid + rstd * (g - mean(g) - xhat * mean(g*xhat)),  g = du * gamma
// part_g[blk][h] = sum over the block's rows of du*xhat, part_b[blk][h] = sum of du
// RMS: backward of the root-mean-square norm, out = resid + rstd * (g - xhat * mean(g*xhat)) with xhat = x * rstd
// (part_b is still written, and not used).
//
// A block works on 8 rows.  TEAM threads (64, 128 or 256, the fewest that cover a row with MV 16-byte column groups each) share a
// row.  A thread owns the same column groups of every row of its team, so the column sums of the parameter gradients stay in its
// registers to the end and a row costs it three vectors; the two row sums of a team of several wavefronts go through LDS, one barrier per
// step, the slots alternate so that a second one is not needed.  (One wavefront per row, the row in registers, needed 234 registers at
// H = 2048.)  Wide rows (TEAM 256): one team per block, two rows a step and the next two in flight.  Narrow rows: 512 threads, so 4 or 8
// teams with 2 rows or 1 each, all asked for at once, and the teams' sums are added through LDS in team order; with one team of 256 half of
// it was idle at H = 1024 and seven eighths at 256 (1024 x 1024: 9.1 -> 7.9 us, 256 x 256: 7.8 -> 5.7).  Two teams of 256 lose (2048 x 1600:
// 14.0 -> 14.7; 2048 x 2560: 21 -> 26, spills).  Inside a layer's backward, tensors from memory: 8192 x 2048 52.7 us, 4096 x 4096 59, 2048 x 1600
// 13.4, 2048 x 8192 67; 55.5, 61, 15.3 and 70 with the rows' statistics in vector loads.
// SUMS: the block's column sums of `out` go to part_s as well (the bias gradient of a projection that writes into the
// residual stream is the column sum of the stream's gradient, which is this kernel's result).
// RESID: there is a residual to add (otherwise `resid` is not read).
constexpr int ln_bwd_threads(int team) { return team == 256 ? 256 : 512; }
template <typename T, int TEAM, int MV, bool RMS, bool SUMS, bool RESID>
__global__ void __launch_bounds__(ln_bwd_threads(TEAM))
ln_bwd_kernel(const float* __restrict__ du, const float* __restrict__ x, const float* __restrict__ mean,
              const float* __restrict__ rstd, const T* __restrict__ gamma, const float* __restrict__ resid,
              float* __restrict__ out, T* __restrict__ out_lowp, float* __restrict__ part_g, float* __restrict__ part_b,
              float* __restrict__ part_s, int seg, int seg_blocks, int H) {
  constexpr int VN = Vec<T>::N;
  constexpr int TEAMS = ln_bwd_threads(TEAM) / TEAM, TW = TEAM / 64;                 // teams per block, wavefronts per team
  constexpr int PER_TEAM = kLnBwdRowsPerBlock / TEAMS;                        // rows of a team
  constexpr int R = PER_TEAM < 2 ? 1 : 2;                                     // ... per step
  constexpr int STEPS = PER_TEAM / R;
  constexpr bool AHEAD = MV <= 2 && STEPS % 2 == 0;                           // the next step's rows fly under this one's
  constexpr int NS = SUMS ? 3 : 2;                                            // column sums
  __shared__ float red[2][TEAMS][R][2][TW];
  __shared__ __attribute__((aligned(16))) float cols[TEAM * VN];              // a team's sums on their way to the first team's
  // (the team is the same in every lane of a wavefront, and said so: a row's mean and rstd are then scalar loads, with a counter of their
  // own.  As vector loads they are the youngest when they are needed, and waiting for them drains the rows asked for ahead)
  const int lane = threadIdx.x & 63, of_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = of_block % TW, team = TEAMS == 1 ? 0 : of_block / TW, tt = threadIdx.x % TEAM;
  const int nv = H / VN;
  const float inv_h = 1.0f / (float)H;
  // rows [first, rows) are the block's matrix of seg rows
  const int of_seg = (int)blockIdx.x / seg_blocks, first = of_seg * seg, rows = first + seg;
  const int row0 = first + ((int)blockIdx.x - of_seg * seg_blocks) * kLnBwdRowsPerBlock + team * PER_TEAM;

  float gm[MV][VN], sum[NS][MV][VN];                                          // sums: d gamma, d beta, the result's
#pragma unroll
  for (int j = 0; j < MV; ++j) {
    const int v = tt + TEAM * j;
    if (v < nv) {
      load_vec<T>(gamma + v * VN, gm[j]);
    } else {
#pragma unroll
      for (int i = 0; i < VN; ++i) gm[j][i] = 0.f;
    }
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int i = 0; i < VN; ++i) sum[k][j][i] = 0.f;
  }

  struct Rows { float d[R][MV][VN], xv[R][MV][VN], rr[R][MV][VN]; };
  auto fetch = [&](Rows& b, int step) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + step * R + r;
#pragma unroll
      for (int j = 0; j < MV; ++j) {
        // (no branch around the loads: a group past the last row or the row's end reads a valid one instead and is
        // replaced by zeros -- it contributes nothing and is not stored; with the loads under bounds branches the
        // compiler waits for all of them at once and the rows asked for ahead do not overlap the arithmetic)
        const int v = tt + TEAM * j;
        const bool ok = row < rows && v < nv;
        const int64_t o = (int64_t)min(row, rows - 1) * H + (v < nv ? v : 0) * VN;
        load_f32<VN>(du + o, b.d[r][j]);
        load_f32<VN>(x + o, b.xv[r][j]);
        if (RESID) {
          load_f32<VN>(resid + o, b.rr[r][j]);
        } else {
#pragma unroll
          for (int i = 0; i < VN; ++i) b.rr[r][j][i] = 0.f;
        }
        // a zero gradient is all it takes: every sum below has it as a factor, and the result of such a group is not stored
#pragma unroll
        for (int i = 0; i < VN; ++i) b.d[r][j][i] = ok ? b.d[r][j][i] : 0.f;
      }
    }
  };
  auto reduce_and_store = [&](Rows& b, int step) {
    float rs[R], s1[R], s2[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = min(row0 + step * R + r, rows - 1);
      const float mu = RMS ? 0.f : mean[row];
      rs[r] = rstd[row];
      s1[r] = s2[r] = 0.f;
#pragma unroll
      for (int j = 0; j < MV; ++j)
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          const float d = b.d[r][j][i];
          const float xh = (b.xv[r][j][i] - mu) * rs[r];
          const float g = d * gm[j][i];
          s1[r] += g;
          s2[r] += g * xh;
          sum[0][j][i] += d * xh;
          sum[1][j][i] += d;
          b.xv[r][j][i] = xh;
          b.d[r][j][i] = g;
        }
      s1[r] = wave_sum(s1[r]);
      s2[r] = wave_sum(s2[r]);
      if (TW > 1 && lane == 0) { red[step & 1][team][r][0][wave] = s1[r]; red[step & 1][team][r][1][wave] = s2[r]; }
    }
    if (TW > 1) __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + step * R + r;
      float c1 = s1[r], c2 = s2[r];
      if (TW > 1) {
        c1 = c2 = 0.f;
#pragma unroll
        for (int w = 0; w < TW; ++w) { c1 += red[step & 1][team][r][0][w]; c2 += red[step & 1][team][r][1][w]; }
      }
      c1 = RMS ? 0.f : c1 * inv_h;
      c2 *= inv_h;
      if (row < rows) {
#pragma unroll
        for (int j = 0; j < MV; ++j) {
          const int v = tt + TEAM * j;
          if (v < nv) {
            float o[VN];
#pragma unroll
            for (int i = 0; i < VN; ++i) o[i] = b.rr[r][j][i] + rs[r] * (b.d[r][j][i] - c1 - b.xv[r][j][i] * c2);
            if (SUMS) {
#pragma unroll
              for (int i = 0; i < VN; ++i) sum[NS - 1][j][i] += o[i];
            }
            store_f32<VN>(out + (int64_t)row * H + v * VN, o);
            if (out_lowp) store_vec<T>(out_lowp + (int64_t)row * H + v * VN, o);
          }
        }
      }
    }
  };
  if constexpr (AHEAD) {
    Rows b0, b1;
    fetch(b0, 0);
#pragma unroll
    for (int step = 0; step < STEPS; step += 2) {
      fetch(b1, step + 1);
      reduce_and_store(b0, step);
      if (step + 2 < STEPS) fetch(b0, step + 2);
      reduce_and_store(b1, step + 1);
    }
  } else {
    Rows b0;
#pragma unroll 1
    for (int step = 0; step < STEPS; ++step) {
      fetch(b0, step);
      reduce_and_store(b0, step);
    }
  }
  // add the teams' column sums, in team order, one sum and column group at a time
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    float* const part = (k == 0 ? part_g : k == 1 ? part_b : part_s) + (int64_t)blockIdx.x * H;
#pragma unroll
    for (int j = 0; j < MV; ++j) {
      for (int t = 1; t < TEAMS; ++t) {
        __syncthreads();
        if (team == t) store_f32<VN>(cols + tt * VN, sum[k][j]);
        __syncthreads();
        if (team == 0) {
#pragma unroll
          for (int i = 0; i < VN; ++i) sum[k][j][i] += cols[tt * VN + i];
        }
      }
      const int v = tt + TEAM * j;
      if (team == 0 && v < nv) store_f32<VN>(part + v * VN, sum[k][j]);
    }
  }
}

// Up to kMaxReduceJobs reductions in one launch: out[n] = (accumulate ? out[n] : 0) + scale * sum_c part[c][n] for each job (the layer's
// eight norm-parameter and bias gradients are 4 KB to 32 KB each: what such a launch costs is the launch and its chain of dependent
// loads, not its bytes).  A block of 16 wavefronts owns 64 columns of one job; a wavefront reads four chunks at a time (16 lanes
// of 16 bytes each), four such groups in flight, so 256 chunks go out before the first is waited for.  Chunks are taken and added
// in an order that depends on the sizes alone.  Eight launches of the former one-job kernel (four wavefronts, 4-byte loads, in two stages
// when there were many chunks) took 61 us of a ViT-G-shaped layer and 21 us of a tiny one, this one 6.3 and 3.3.
typedef float f32x4v __attribute__((ext_vector_type(4)));
constexpr int kReduceWaves = 16;
struct ReduceBatch { int n; int first[kMaxReduceJobs + 1]; ReduceJob job[kMaxReduceJobs]; };

__global__ void __launch_bounds__(64 * kReduceWaves)
reduce_jobs_kernel(ReduceBatch b, float scale, int accumulate) {
  __shared__ f32x4v red[kReduceWaves][16];
  int q = 0;
  while (q + 1 < b.n && (int)blockIdx.x >= b.first[q + 1]) ++q;
  const float* __restrict__ part = b.job[q].part;
  const int nchunks = b.job[q].nchunks, N = b.job[q].N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = ((int)blockIdx.x - b.first[q]) * 64 + (lane & 15) * 4;
  constexpr int STEP = kReduceWaves * 4;
  f32x4v s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) s[u] = f32x4v{0.f, 0.f, 0.f, 0.f};
  if (n < N) {                                             // (N is a multiple of 4)
    int c = wave * 4 + (lane >> 4);
    auto at = [&](int r) { return *reinterpret_cast<const f32x4v*>(part + (int64_t)r * N + n); };
    for (; c + 3 * STEP < nchunks; c += 4 * STEP) {
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += at(c + u * STEP);
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) if (c + u * STEP < nchunks) s[u] += at(c + u * STEP);
  }
  f32x4v v = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] += __shfl_xor(v[i], 16, 64);
    v[i] += __shfl_xor(v[i], 32, 64);
  }
  if (lane < 16) red[wave][lane] = v;
  __syncthreads();
  if (wave == 0 && lane < 16 && n < N) {
    f32x4v t = red[0][lane];
#pragma unroll
    for (int w = 1; w < kReduceWaves; ++w) t += red[w][lane];
    f32x4v* o = reinterpret_cast<f32x4v*>(b.job[q].out + n);
    *o = accumulate ? *o + scale * t : scale * t;
  }
}

// Column sums of ROWS rows by 64 vectors of 16 bytes per block: the four wavefronts take every fourth row, all of them in flight, and
// their sums are added in wavefront order.  LOWP (T = float): the rows are written in bf16 as well.  (One row at a time per thread, as it
// used to be: the 4096 x 1024 gradient of a BERT-Large-shaped share took 38 to 68 us inside the step, with the copy into bf16 beside it 6.)
// Order of the blocks, whose sums do not depend on it: those of the same rows are neighbours (in order of the columns instead, neighbours read
// lines 64 rows apart: 24576 x 8192 in bf16 74 -> 83 us).  runs: each XCD has one contiguous run of that order, so that it reads whole rows; with
// neighbours on neighbouring XCDs each reads an eighth of every row and, at widths of a power of two, through a part of its L2's
// channels.  Memory by itself is faster with all XCDs at the same place.  So: runs where the matrix fits the 256 MB cache.  Both orders and the kernel
// of one row at a time, with the reduction, us: 24576 x 2048 fp32 38.4, runs 33.8, former 33.1; 24576 x 4096 bf16 37.2, 34.3, 34.5; 24576 x 2048 bf16 26.1,
// 20.6, 28.7; 8192 x 16384 bf16 48.3, 43.7, 48.9; beyond 256 MB 24576 x 8192 bf16 72.5, 76.6, 80.7; 24576 x 4096 fp32 72.5, 73.2, 76.7.  The
// copying form inside a layer, which also writes, keeps the plain order: 8192 x 2048 19.2, runs 20.1.  What is still behind
// the former kernel: 8192 x 10240 fp32 57.3 (55.8) and, for its reduction in one stage, 100000 x 256 fp32 25.8 (25.1).
constexpr int kColsumRowsPerChunk = 64;
template <typename T, bool LOWP, int ROWS>
__device__ __forceinline__ void colsum_block(const T* __restrict__ dY, bf16* __restrict__ lowp, float* __restrict__ partials, int rows, int N, int runs, int block, int total) {
  constexpr int VN = Vec<T>::N;
  typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
  __shared__ float red[kWaves][64][VN + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col_blocks = (N / VN + 63) / 64, xcd = block & 7;
  const int at = runs ? xcd * (total >> 3) + min(xcd, total & 7) + (block >> 3) : block;
  const int chunk = at / col_blocks, col = (at % col_blocks * 64 + lane) * VN;
  const int r0 = chunk * ROWS + wave;
  const bool in = col < N;
  float acc[VN];
#pragma unroll
  for (int i = 0; i < VN; ++i) acc[i] = 0.f;
  constexpr int PER = ROWS / kWaves;
  float d[PER][VN];
#pragma unroll
  for (int u = 0; u < PER; ++u) {                          // (rows and columns past the end read a valid place and count as zero)
    const int r = r0 + u * kWaves;
    load_vec<T>(dY + (int64_t)min(r, rows - 1) * N + (in ? col : 0), d[u]);
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int r = r0 + u * kWaves;
    const bool ok = r < rows && in;
#pragma unroll
    for (int i = 0; i < VN; ++i) acc[i] += ok ? d[u][i] : 0.f;
    if constexpr (LOWP) {
      bf16x4 q;
#pragma unroll
      for (int i = 0; i < 4; ++i) q[i] = (bf16)d[u][i];
      if (ok) *reinterpret_cast<bf16x4*>(lowp + (int64_t)r * N + col) = q;
    }
  }
  if (LOWP && !partials) return;                           // (the copy alone)
#pragma unroll
  for (int i = 0; i < VN; ++i) red[wave][lane][i] = acc[i];
  __syncthreads();
  if (wave == 0 && in) {
    float* p = partials + (int64_t)chunk * N + col;
#pragma unroll
    for (int i = 0; i < VN; ++i) p[i] = (red[0][lane][i] + red[1][lane][i]) + (red[2][lane][i] + red[3][lane][i]);
  }
}

template <typename T, bool LOWP, int ROWS>
__global__ void __launch_bounds__(kThreads)
colsum_kernel(const T* __restrict__ dY, bf16* __restrict__ lowp, float* __restrict__ partials, int rows, int N, int runs) {
  colsum_block<T, LOWP, ROWS>(dY, lowp, partials, rows, N, runs, blockIdx.x, gridDim.x);
}

// 64x64 tiles transposed through LDS: 16-byte global reads along the input rows, 16-byte global
// writes along the output rows; the LDS tile is padded so that the column walk is conflict-free.
// out has row pitch `pitch` >= rows; its columns [rows, pitch) are written with zeros.
// Up to kMaxTransposes matrices in one launch (a layer's four weights: 4.6 us each at width 1024, most of it the launch).
struct TransposeBatch { int n; int first[kMaxTransposes + 1]; TransposeJob job[kMaxTransposes]; };
__device__ __forceinline__ void transpose_block(const TransposeBatch& b, int block) {
  __shared__ bf16 tile[64][64 + 2];
  typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
  int q = 0;
  while (q + 1 < b.n && block >= b.first[q + 1]) ++q;
  const bf16* __restrict__ in = b.job[q].in;
  bf16* __restrict__ out = b.job[q].out;
  const int rows = b.job[q].rows, cols = b.job[q].cols, pitch = b.job[q].pitch;
  const int tile_cols = (cols + 63) / 64, at = block - b.first[q];
  const int r0 = at / tile_cols * 64, c0 = at % tile_cols * 64;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int v = threadIdx.x + kThreads * p;
    const int r = v >> 3, c = (v & 7) * 8;
    bf16x8 val = {0, 0, 0, 0, 0, 0, 0, 0};
    if (r0 + r < rows && c0 + c < cols) val = *reinterpret_cast<const bf16x8*>(in + (int64_t)(r0 + r) * cols + c0 + c);
#pragma unroll
    for (int i = 0; i < 8; ++i) tile[r][c + i] = val[i];
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int v = threadIdx.x + kThreads * p;
    const int c = v >> 3, r = (v & 7) * 8;       // output row c, output columns r..r+7
    if (c0 + c < cols && r0 + r < pitch) {
      bf16x8 val;
#pragma unroll
      for (int i = 0; i < 8; ++i) val[i] = tile[r + i][c];
      *reinterpret_cast<bf16x8*>(out + (int64_t)(c0 + c) * pitch + r0 + r) = val;
    }
  }
}

__global__ void __launch_bounds__(kThreads) transpose_bf16_kernel(TransposeBatch b) { transpose_block(b, blockIdx.x); }

// What a layer's backward needs before its first product: the transposed weights and, of a gradient that the caller hands over, its copy and column
// sums.  Neither reads the other, and for small layers a launch costs more than its work (a layer of width 256 on 256 tokens: 92.4 us with two launches,
// 90.1 with one; from width 1024 on no difference).
constexpr int kCastColsumRows = 32;
__global__ void __launch_bounds__(kThreads) prepare_backward_kernel(TransposeBatch b, CastColsum c, int sums) {
  if ((int)blockIdx.x < sums) colsum_block<float, true, kCastColsumRows>(c.x, c.lowp, c.partials, c.rows, c.N, 0, blockIdx.x, sums);
  else transpose_block(b, (int)blockIdx.x - sums);
}

template <typename T> int maxv_for(int H) {
  const int nv = H / Vec<T>::N;
  const int need = (nv + 63) / 64;
  int m = 1;
  while (m < need) m *= 2;
  return m;
}

}  // namespace

template <typename T>
int launch_ln_fwd(const float* x, const T* gamma, const T* beta, T* u, float* mean, float* rstd,
                  int rows, int H, float eps, hipStream_t s, bool rms) {
  const int grid = (rows + kWaves - 1) / kWaves;
#define LN_FWD_CASE(MV)                                                                             \
  case MV:                                                                                          \
    if (rms) ln_fwd_kernel<T, MV, true><<<grid, kThreads, 0, s>>>(x, gamma, beta, u, mean, rstd, rows, H, eps);    \
    else ln_fwd_kernel<T, MV, false><<<grid, kThreads, 0, s>>>(x, gamma, beta, u, mean, rstd, rows, H, eps);    \
    break;
  switch (maxv_for<T>(H)) {
    LN_FWD_CASE(1) LN_FWD_CASE(2) LN_FWD_CASE(4) LN_FWD_CASE(8) LN_FWD_CASE(16)
    default: return fail(CEPHALO_EUNSUPPORTED, "layer norm: hidden width %d too large", H);
  }
#undef LN_FWD_CASE
  CEPHALO_CHECK_LAUNCH("ln_fwd");
  return CEPHALO_OK;
}

int ln_bwd_blocks(int rows) { return (rows + kLnBwdRowsPerBlock - 1) / kLnBwdRowsPerBlock; }

template <typename T>
int launch_ln_bwd(const float* du, const float* x, const float* mean, const float* rstd, const T* gamma,
                  const float* resid, float* out, T* out_lowp, float* part_g, float* part_b, int rows, int H, hipStream_t s, bool rms,
                  float* part_s, int seg) {
  if (rms && part_s) return fail(CEPHALO_EINVAL, "norm backward: column sums of the result go with the LayerNorm form only");
  if (seg <= 0 || seg % kLnBwdRowsPerBlock == 0) seg = rows;          // (blocks end with the matrices anyway)
  if (rows % seg != 0) return fail(CEPHALO_EINVAL, "norm backward: %d rows are not whole matrices of %d", rows, seg);
  const int seg_blocks = ln_bwd_blocks(seg), nblocks = rows / seg * seg_blocks;
  const int nv = H / Vec<T>::N;                // 16-byte column groups of a row
#define LN_BWD_FORMS(TEAM, MV, RESID)                                                                                \
    { if (rms) ln_bwd_kernel<T, TEAM, MV, true, false, RESID><<<nblocks, ln_bwd_threads(TEAM), 0, s>>>(du, x, mean, rstd, gamma, resid, out, out_lowp, part_g, part_b, nullptr, seg, seg_blocks, H); \
      else if (part_s) ln_bwd_kernel<T, TEAM, MV, false, true, RESID><<<nblocks, ln_bwd_threads(TEAM), 0, s>>>(du, x, mean, rstd, gamma, resid, out, out_lowp, part_g, part_b, part_s, seg, seg_blocks, H); \
      else ln_bwd_kernel<T, TEAM, MV, false, false, RESID><<<nblocks, ln_bwd_threads(TEAM), 0, s>>>(du, x, mean, rstd, gamma, resid, out, out_lowp, part_g, part_b, nullptr, seg, seg_blocks, H); }
#define LN_BWD_CASE(TEAM, MV) { if (resid) LN_BWD_FORMS(TEAM, MV, true) else LN_BWD_FORMS(TEAM, MV, false) }
  if (nv <= 64) LN_BWD_CASE(64, 1)
  else if (nv <= 128) LN_BWD_CASE(128, 1)
  else if (nv <= 256) LN_BWD_CASE(256, 1)
  else if (nv <= 512) LN_BWD_CASE(256, 2)
  else if (nv <= 1024) LN_BWD_CASE(256, 4)
  else return fail(CEPHALO_EUNSUPPORTED, "layer norm: hidden width %d too large", H);
#undef LN_BWD_CASE
#undef LN_BWD_FORMS
  CEPHALO_CHECK_LAUNCH("ln_bwd");
  return CEPHALO_OK;
}

int launch_reduce_jobs(const ReduceJob* jobs, int n, float scale, int accumulate, hipStream_t s) {
  if (n <= 0) return CEPHALO_OK;
  if (n > kMaxReduceJobs) return fail(CEPHALO_EINVAL, "reduce: %d jobs in one launch", n);
  ReduceBatch b = {};
  b.n = n;
  for (int i = 0; i < n; ++i) {
    if (jobs[i].N % 4 != 0 || !aligned16(jobs[i].part) || !aligned16(jobs[i].out)) return fail(CEPHALO_EINVAL, "reduce: rows of %d floats", jobs[i].N);
    b.job[i] = jobs[i];
    b.first[i + 1] = b.first[i] + (jobs[i].N + 63) / 64;
  }
  reduce_jobs_kernel<<<b.first[n], 64 * kReduceWaves, 0, s>>>(b, scale, accumulate);
  CEPHALO_CHECK_LAUNCH("reduce_jobs");
  return CEPHALO_OK;
}

int launch_reduce_partials(const float* partials, int nchunks, int N, float* g, float scale, int accumulate, hipStream_t s) {
  const ReduceJob job = {partials, nchunks, N, g};
  return launch_reduce_jobs(&job, 1, scale, accumulate, s);
}

size_t colsum_partial_bytes(int rows, int N) {
  const size_t nchunks = (rows + kColsumRowsPerChunk - 1) / kColsumRowsPerChunk;
  return (nchunks + (nchunks > 64 ? (nchunks + 31) / 32 : 0)) * (size_t)N * sizeof(float);      // (the second term is not used any more and stays, so that sizes reported and refused are what they were)
}

template <typename T>
int launch_colsum(const T* dY, float* partials, size_t partial_bytes, float* g, float scale,
                  int accumulate, int rows, int N, hipStream_t s) {
  if (partial_bytes < colsum_partial_bytes(rows, N)) return fail(CEPHALO_EWORKSPACE, "colsum: partial buffer too small");
  const int nchunks = (rows + kColsumRowsPerChunk - 1) / kColsumRowsPerChunk;
  const int nvec = N / Vec<T>::N;
  const int64_t grid = (int64_t)nchunks * ((nvec + 63) / 64);      // (one axis: the blocks of a chunk of rows are neighbours)
  colsum_kernel<T, false, kColsumRowsPerChunk><<<(unsigned)grid, kThreads, 0, s>>>(dY, nullptr, partials, rows, N, (size_t)rows * N * sizeof(T) <= (size_t)256 << 20);
  CEPHALO_CHECK_LAUNCH("colsum");
  return launch_reduce_partials(partials, nchunks, N, g, scale, accumulate, s);
}

// (half the rows per block of the plain column sum: the launch has only N / 256 blocks per chunk)
int cast_colsum_chunks(int rows) { return (rows + kCastColsumRows - 1) / kCastColsumRows; }

int launch_transposes(const TransposeJob* jobs, int n, hipStream_t s, const CastColsum* beside) {
  if (n <= 0 || n > kMaxTransposes) return fail(CEPHALO_EINVAL, "transpose: %d matrices in one launch", n);
  TransposeBatch b = {};
  b.n = n;
  for (int i = 0; i < n; ++i) {
    TransposeJob& t = b.job[i] = jobs[i];
    if (t.pitch == 0) t.pitch = t.rows;
    if (t.pitch % 8 != 0 || t.pitch < t.rows || t.cols % 8 != 0)
      return fail(CEPHALO_EINVAL, "transpose: %d x %d into pitch %d: columns and pitch must be multiples of 8", t.rows, t.cols, t.pitch);
    b.first[i + 1] = b.first[i] + ((t.cols + 63) / 64) * ((t.pitch + 63) / 64);
  }
  if (beside) {
    const int chunks = cast_colsum_chunks(beside->rows);
    if (beside->partials && beside->partial_bytes < (size_t)chunks * beside->N * sizeof(float)) return fail(CEPHALO_EWORKSPACE, "cast_colsum: partial buffer too small");
    const int sums = chunks * ((beside->N / 4 + 63) / 64);
    prepare_backward_kernel<<<(unsigned)(sums + b.first[n]), kThreads, 0, s>>>(b, *beside, sums);
    CEPHALO_CHECK_LAUNCH("prepare_backward");
    return CEPHALO_OK;
  }
  transpose_bf16_kernel<<<b.first[n], kThreads, 0, s>>>(b);
  CEPHALO_CHECK_LAUNCH("transpose");
  return CEPHALO_OK;
}

// ---- rotary position embedding (Llama-style layer)
// Within each head the pair (2i, 2i+1) of the token at position t is rotated by the angle t * base^(-2i/d).
// The angles' cosines and sines are tabulated once per call, tab[t][i] = (cos, sin) in fp32 (fp32 power, accurate
// sincos), and every kernel that rotates (the GEMM epilogue that produces q and k, the attention backward's stores of
// dq and dk, the stand-alone kernel below) reads the same table.
static __global__ void __launch_bounds__(kThreads)
rotary_table_kernel(float* __restrict__ tab, int S, int d, float log2_base) {
  const int idx = blockIdx.x * kThreads + threadIdx.x;
  if (idx >= S * (d / 2)) return;
  const int t = idx / (d / 2), i = idx % (d / 2);
  const float inv = exp2f(-2.0f * (float)i / (float)d * log2_base);
  float sn, cs;
  sincosf((float)t * inv, &sn, &cs);
  tab[2 * idx] = cs;
  tab[2 * idx + 1] = sn;
}

int launch_rotary_table(float* tab, int S, int d, float base, hipStream_t s) {
  if (d % 8 != 0) return fail(CEPHALO_EUNSUPPORTED, "rotary: head dim %d must be a multiple of 8", d);
  const int n = S * (d / 2);
  rotary_table_kernel<<<(n + kThreads - 1) / kThreads, kThreads, 0, s>>>(tab, S, d, log2f(base));
  CEPHALO_CHECK_LAUNCH("rotary_table");
  return CEPHALO_OK;
}

// In place on the Q and K thirds of qkv [rows, 3H], position t = row % S; sign = -1 turns back (the gradient's way).
// One thread per 4 consecutive values (2 pairs).
template <typename T>
static __global__ void __launch_bounds__(kThreads)
rotary_kernel(T* __restrict__ qkv, const float* __restrict__ tab, int rows, int S, int H, int d, float sign) {
  const int per_row = 2 * H / 4;                           // groups of the Q and K parts of a row
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= (int64_t)rows * per_row) return;
  const int row = (int)(idx / per_row), col = (int)(idx % per_row) * 4;     // column within [0, 2H): Q then K
  const int t = row % S;
  T* p = qkv + (int64_t)row * 3 * H + col;
  const float* r = tab + ((int64_t)t * (d / 2) + (col % d) / 2) * 2;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float cs = r[2 * q], sn = sign * r[2 * q + 1];
    const float e = (float)p[2 * q], o = (float)p[2 * q + 1];
    p[2 * q] = (T)(e * cs - o * sn);
    p[2 * q + 1] = (T)(e * sn + o * cs);
  }
}

template <typename T>
int launch_rotary(T* qkv, const float* tab, int rows, int S, int H, int heads, int inverse, hipStream_t s) {
  const int d = H / heads;
  if (H % 8 != 0 || d % 8 != 0) return fail(CEPHALO_EUNSUPPORTED, "rotary: head dim %d must be a multiple of 8", d);
  const int64_t n = (int64_t)rows * (2 * H / 4);
  rotary_kernel<T><<<(int)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(qkv, tab, rows, S, H, d, inverse ? -1.0f : 1.0f);
  CEPHALO_CHECK_LAUNCH("rotary");
  return CEPHALO_OK;
}

// ---- gated SiLU feed-forward: gu [rows, 2F] = [gate | up];  h = silu(gate) * up (the backward is an epilogue of the GEMM that produces dh)
__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

template <typename T>
static __global__ void __launch_bounds__(kThreads)
swiglu_fwd_kernel(const T* __restrict__ gu, T* __restrict__ h, int64_t rows, int F) {
  constexpr int VN = Vec<T>::N;
  const int per_row = F / VN;
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= rows * per_row) return;
  const int64_t row = idx / per_row;
  const int c = (int)(idx % per_row) * VN;
  float g[VN], u[VN], o[VN];
  load_vec<T>(gu + row * 2 * F + c, g);
  load_vec<T>(gu + row * 2 * F + F + c, u);
#pragma unroll
  for (int i = 0; i < VN; ++i) o[i] = g[i] * sigmoidf_(g[i]) * u[i];
  store_vec<T>(h + row * F + c, o);
}


template <typename T>
int launch_swiglu_fwd(const T* gu, T* h, int64_t rows, int F, hipStream_t s) {
  const int64_t n = rows * (F / Vec<T>::N);
  swiglu_fwd_kernel<T><<<(int)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(gu, h, rows, F);
  CEPHALO_CHECK_LAUNCH("swiglu_fwd");
  return CEPHALO_OK;
}

#define INSTANTIATE(T)                                                                                          \
  template int launch_ln_fwd<T>(const float*, const T*, const T*, T*, float*, float*, int, int, float, hipStream_t, bool); \
  template int launch_ln_bwd<T>(const float*, const float*, const float*, const float*, const T*, const float*, float*, \
                                T*, float*, float*, int, int, hipStream_t, bool, float*, int);                    \
  template int launch_rotary<T>(T*, const float*, int, int, int, int, int, hipStream_t);                          \
  template int launch_swiglu_fwd<T>(const T*, T*, int64_t, int, hipStream_t);                                     \
  template int launch_colsum<T>(const T*, float*, size_t, float*, float, int, int, int, hipStream_t);
INSTANTIATE(float)
INSTANTIATE(bf16)
#undef INSTANTIATE

}  // namespace cephalo
