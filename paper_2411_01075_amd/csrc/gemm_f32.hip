// fp32 GEMM on the gfx950 matrix cores:  C[M,N] = sum_k A(m,k) B(n,k), any operand strides, ragged edges, the epilogues of
// GemmArgs.  v_mfma_f32_16x16x4_f32 multiplies and adds in full fp32 (256 flops per clock and compute unit, twice the
// vector unit's rate without packed forms).
//
// The fp32 workloads are small (a 256-wide layer on 256 tokens: outputs of 256 x 256 to 512 x 1024, contractions of 128 to
// 1024), so what bounds them is how much of the chip a launch reaches and how long its serial chain along k is.  Hence a
// 32 x 32 output tile (64 blocks where a 64 x 64 tile gives 16) and, inside the block, four groups of four wavefronts that
// take every fourth 32-wide piece of the contraction; the groups' sums are added through LDS in group order at the end (a
// fixed order: reproducible).  A block of 16 wavefronts brings in a slab of 128 k-values per barrier, one 16-byte load per
// thread and operand, with the next two slabs' loads in registers while one is multiplied.  Large outputs are bound by the
// matrix cores all the same: a slab is 1024 clocks of products against 512 clocks of tile traffic from L2.
// Measured at the tiny layer's shapes: 99 -> 8.6 us on average per launch against the former vector-FMA kernel (64 x 64 tiles, no
// load in flight during the arithmetic).
//
// Operand layout for the products: in step t a lane of group g = lane / 16 supplies k = 4 g + t of a piece of 16
// (the assignment of k to steps is free as long as A and B agree), so one 16-byte LDS read of four consecutive k-values
// feeds four products.  Both operands lie [row][k] in LDS with a pitch of 132 floats: 16 consecutive rows put a 16-byte
// chunk on 16 different bank groups.
#include "kernels.h"

namespace cephalo {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TB = 32;                 // tile rows and columns
constexpr int KG = 4;                  // groups of wavefronts along k
constexpr int SLAB = 32 * KG;          // k-values per slab
constexpr int PITCH = SLAB + 4;
constexpr int kThreads = 256 * KG;     // four wavefronts per group, a 16 x 16 piece of the tile each

// Four consecutive values of operand element (row, k) along its contiguous axis, as this thread's share of a slab: the slab
// holds 32 x 128 values, thread t takes the t-th group of four.  VEC: pitches, extents and base allow 16-byte loads.
template <bool VEC>
__device__ __forceinline__ f32x4 load_share(const float* __restrict__ p, int64_t rs, int64_t cs, int rows, int K, int row0, int k0) {
  const int t = threadIdx.x;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (cs == 1) {                                         // k-contiguous: row t / 32, k-values 4 (t % 32) ..
    const int r = row0 + (t >> 5), k = k0 + (t & 31) * 4;
    if (r < rows) {
      const float* q = p + (int64_t)r * rs + k;
      if (VEC) {
        if (k < K) v = *reinterpret_cast<const f32x4*>(q);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) if (k + i < K) v[i] = q[i];
      }
    }
  } else {                                               // row-contiguous: k-value t / 8, rows 4 (t % 8) ..
    const int k = k0 + (t >> 3), r = row0 + (t & 7) * 4;
    if (k < K) {
      const float* q = p + (int64_t)k * cs + (int64_t)r * rs;
      if (VEC) {
        if (r < rows) v = *reinterpret_cast<const f32x4*>(q);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) if (r + i < rows) v[i] = q[(int64_t)i * rs];
      }
    }
  }
  return v;
}
__device__ __forceinline__ void store_share(float* lds, bool kfast, f32x4 v) {
  const int t = threadIdx.x;
  if (kfast) {
    *reinterpret_cast<f32x4*>(lds + (t >> 5) * PITCH + (t & 31) * 4) = v;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[((t & 7) * 4 + i) * PITCH + (t >> 3)] = v[i];
  }
}

template <bool VEC>
__device__ __forceinline__ void gemm_f32_tile(const GemmArgs<float>& a, int tile_m, int tile_n) {
  __shared__ __attribute__((aligned(16))) float As[2][TB * PITCH];
  __shared__ __attribute__((aligned(16))) float Bs[2][TB * PITCH];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int group = wave >> 2;                           // which 32 k-values of a slab
  const int wm = (wave >> 1 & 1) * 16, wn = (wave & 1) * 16;
  const int m0 = tile_m * TB, n0 = tile_n * TB;
  const bool ak = a.a_cs == 1, bk = a.b_cs == 1;

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  f32x4 ra[2], rb[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {                          // (a slab past the end loads nothing: zeros)
    ra[s] = load_share<VEC>(a.A, a.a_rs, a.a_cs, a.M, a.K, m0, s * SLAB);
    rb[s] = load_share<VEC>(a.B, a.b_rs, a.b_cs, a.N, a.K, n0, s * SLAB);
  }
  const int fo = (lane & 15) * PITCH + group * 32 + (lane >> 4) * 4;
  const int nslab = (a.K + SLAB - 1) / SLAB;
  auto slab = [&](int s, int b) {                        // b = s & 1: LDS buffer and register set of slab s
    store_share(As[b], ak, ra[b]);
    store_share(Bs[b], bk, rb[b]);
    ra[b] = load_share<VEC>(a.A, a.a_rs, a.a_cs, a.M, a.K, m0, (s + 2) * SLAB);
    rb[b] = load_share<VEC>(a.B, a.b_rs, a.b_cs, a.N, a.K, n0, (s + 2) * SLAB);
    __syncthreads();       // (one per slab: buffer b was last read before the barrier of slab s - 1)
#pragma unroll
    for (int piece = 0; piece < 2; ++piece) {
      const f32x4 fa = *reinterpret_cast<const f32x4*>(&As[b][wm * PITCH + fo + piece * 16]);
      const f32x4 fb = *reinterpret_cast<const f32x4*>(&Bs[b][wn * PITCH + fo + piece * 16]);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[t], fa[t], acc, 0, 0, 0);
    }
  };
  for (int s = 0; s < nslab; s += 2) {
    slab(s, 0);
    if (s + 1 < nslab) slab(s + 1, 1);
  }

  // add the groups' sums, in group order
  __syncthreads();
  float* red = &As[0][0];                                // [group - 1][wavefront of the group][lane] of four floats
  if (group > 0) *reinterpret_cast<f32x4*>(red + (((group - 1) * 4 + (wave & 3)) * 64 + lane) * 4) = acc;
  __syncthreads();
  if (group > 0) return;
#pragma unroll
  for (int g = 0; g < KG - 1; ++g) acc += *reinterpret_cast<const f32x4*>(red + ((g * 4 + wave) * 64 + lane) * 4);

  // the operands went in exchanged: a lane owns row m and four consecutive columns
  const int m = m0 + wm + (lane & 15), nb = n0 + wn + (lane >> 4) * 4;
  if (m >= a.M) return;
  const int64_t row = (int64_t)m * (a.epi == EPI_GRAD || !a.ldc ? a.N : a.ldc);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = nb + j;
    if (n >= a.N) break;
    const int64_t o = row + n;
    const float v = acc[j];
    auto put = [&](float r) { if (a.Cf) a.Cf[o] = r; else a.C[o] = r; };
    switch (a.epi) {
      case EPI_NONE: case EPI_NONE_HEAD: put(v); break;
      case EPI_BIAS: put(v + a.bias[n]); break;
      case EPI_BIAS_RESID: put(v + (a.bias ? a.bias[n] : 0.f) + (a.Rf ? a.Rf[o] : a.R[o])); break;
      case EPI_BIAS_GELU: {
        const float z = v + a.bias[n];
        a.Z[o] = z;
        a.C[o] = gelu_f(z);
      } break;
      case EPI_DGELU: a.C[o] = v * gelu_grad_f(a.Z[o]); break;
      case EPI_BIAS_GELU_DERIV: {
        const float z = v + a.bias[n];
        a.Z[o] = gelu_grad_f(z);
        a.C[o] = gelu_f(z);
      } break;
      case EPI_MUL: a.C[o] = v * a.Z[o]; break;
      case EPI_ROPE: {      // the partner column's product sits in the same lane
        float r = v;
        if (n < a.rot_cols) {
          const float* cs = a.rot + ((int64_t)(m % a.rot_S) * (a.rot_d / 2) + (n % a.rot_d) / 2) * 2;
          r = (j & 1) ? acc[j ^ 1] * cs[1] + v * cs[0] : v * cs[0] - acc[j ^ 1] * cs[1];
        }
        put(r);
      } break;
      case EPI_DSWIGLU: {
        float dg, du;
        swiglu_grad(a.Z[o], a.Z[o + a.N], v, dg, du);
        a.C[o] = dg;
        a.C[o + a.N] = du;
      } break;
      case EPI_GRAD: a.G[o] = (a.accumulate ? a.G[o] : 0.f) + a.scale * v; break;
    }
  }
}

template <bool VEC>
__global__ void __launch_bounds__(kThreads) gemm_f32_kernel(GemmArgs<float> a) {
  const int tile_m = blockIdx.z * gridDim.y + blockIdx.y;
  if (tile_m * TB < a.M) gemm_f32_tile<VEC>(a, tile_m, blockIdx.x);
}

// Several products in one launch (a layer's weight gradients: four launches of 8.4 us each are one of 20).
struct F32Batch { int n; int first[kMaxGradGroup + 1]; int tiles_n[kMaxGradGroup]; GemmArgs<float> a[kMaxGradGroup]; };
template <bool VEC>
__global__ void __launch_bounds__(kThreads) gemm_f32_group_kernel(F32Batch b) {
  int q = 0;
  while (q + 1 < b.n && (int)blockIdx.x >= b.first[q + 1]) ++q;
  const GemmArgs<float> a = b.a[q];
  const int block = (int)blockIdx.x - b.first[q];
  gemm_f32_tile<VEC>(a, block / b.tiles_n[q], block % b.tiles_n[q]);
}

// 16-byte loads of an operand: base, pitch and extent along the contiguous axis are multiples of four floats
bool vec_ok(const float* p, int64_t rs, int64_t cs, int rows, int K) {
  if (!aligned16(p)) return false;
  return cs == 1 ? rs % 4 == 0 && K % 4 == 0 : rs == 1 && cs % 4 == 0 && rows % 4 == 0;
}

}  // namespace

int launch_gemm_f32(const GemmArgs<float>& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return fail(CEPHALO_EINVAL, "gemm: empty problem %dx%dx%d", a.M, a.N, a.K);
  const int tm = (a.M + TB - 1) / TB, ty = tm < 32768 ? tm : 32768;      // (a grid's second and third extents end at 65535)
  dim3 grid((a.N + TB - 1) / TB, ty, (tm + ty - 1) / ty);
  if (vec_ok(a.A, a.a_rs, a.a_cs, a.M, a.K) && vec_ok(a.B, a.b_rs, a.b_cs, a.N, a.K)) gemm_f32_kernel<true><<<grid, kThreads, 0, s>>>(a);
  else gemm_f32_kernel<false><<<grid, kThreads, 0, s>>>(a);
  CEPHALO_CHECK_LAUNCH("gemm_f32");
  return CEPHALO_OK;
}

int launch_gemm_f32_group(const GemmArgs<float>* a, int n, hipStream_t s) {
  if (n <= 0 || n > kMaxGradGroup) return fail(CEPHALO_EINVAL, "gemm: %d products in one launch", n);
  F32Batch b = {};
  b.n = n;
  bool vec = true;
  int64_t blocks = 0;
  for (int q = 0; q < n; ++q) {
    if (a[q].M <= 0 || a[q].N <= 0 || a[q].K <= 0) return fail(CEPHALO_EINVAL, "gemm: empty problem %dx%dx%d", a[q].M, a[q].N, a[q].K);
    b.a[q] = a[q];
    b.tiles_n[q] = (a[q].N + TB - 1) / TB;
    blocks += (int64_t)((a[q].M + TB - 1) / TB) * b.tiles_n[q];
    b.first[q + 1] = (int)blocks;
    vec = vec && vec_ok(a[q].A, a[q].a_rs, a[q].a_cs, a[q].M, a[q].K) && vec_ok(a[q].B, a[q].b_rs, a[q].b_cs, a[q].N, a[q].K);
  }
  if (blocks > (1 << 21)) {      // (a grid ends at 2^32 threads)
    for (int q = 0; q < n; ++q)
      if (const int rc = launch_gemm_f32(a[q], s); rc != CEPHALO_OK) return rc;
    return CEPHALO_OK;
  }
  if (vec) gemm_f32_group_kernel<true><<<(int)blocks, kThreads, 0, s>>>(b);
  else gemm_f32_group_kernel<false><<<(int)blocks, kThreads, 0, s>>>(b);
  CEPHALO_CHECK_LAUNCH("gemm_f32_group");
  return CEPHALO_OK;
}

}  // namespace cephalo
