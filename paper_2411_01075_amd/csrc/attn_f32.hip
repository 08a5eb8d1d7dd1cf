// fp32 attention forward / backward on the gfx950 matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums), any head width
// up to 128, online softmax.  It serves the fp32 workload, whose launches are small: 4 heads of 64, 2 x 128 tokens are 64 blocks.  What
// bounds them is the chain of dependent loads in a wavefront, so nothing is staged: a block owns 16 queries (dK / dV: 16 keys) of one head, its
// four wavefronts take every fourth block of 16 keys (queries), each keeps a running result of its own, and the four are merged
// through LDS at the end in wavefront order (reproducible).  The loop has no barrier, and all loads of a step are asked for at once.
// Forward 14.8 -> 12.8 us, dQ with rowsum(dO O) 19.2 -> 11.4, dK / dV 24.2 -> 14.9 at that size, and far more at larger ones, against one
// wavefront per row with scalar dot products.
//
// Operand layout.  A product D[i][j] = sum_k A[i][k] B[k][j] leaves lane l with column j = l % 16 and rows i = 4 (l / 16) .. + 3.  The
// contraction of a step of four products runs over 16 values, of which lane group g = l / 16 supplies 4 g + t in product t: for a product
// over the head's dimensions that is one 16-byte load of 4 consecutive values of a row; for a product over 16 keys (queries) the second operand
// is the four scores the lane itself holds, and the first is read from row 4 g + t of the value (key, query, gradient) matrix.
#include "kernels.h"

namespace cephalo {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kMaxHeadDim = 128;
constexpr int kMaxSeq = 7500;          // what the fp32 mode takes (nothing here grows with it; longer samples are the bf16 mode's)
constexpr int kWaves = 4;

// rows of a row-major [*, ld] matrix as an operand over the head's dimensions: row r0 + l % 16, dimensions 16 p + 4 g .. + 3 of piece p
// (rows past `rows` and dimensions past d are zero).  VEC: 16-byte loads (d and ld multiples of 4, aligned base).
template <int P, bool VEC>
__device__ __forceinline__ void load_rows(const float* __restrict__ m, int64_t ld, int r0, int rows, int d, f32x4 (&f)[P]) {
  const int lane = threadIdx.x & 63, r = r0 + (lane & 15), g = lane >> 4;
  const float* p = m + (int64_t)min(r, rows - 1) * ld;
  const bool ok = r < rows;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int c = 16 * q + 4 * g;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
      v = *reinterpret_cast<const f32x4*>(p + (c < d ? c : 0));
      f[q] = ok && c < d ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) if (ok && c + i < d) v[i] = p[c + i];
      f[q] = v;
    }
  }
}
// the same matrix as the first operand over 16 of its rows: element [t] of piece p is row r0 + 4 g + t, column 16 p + l % 16
template <int P>
__device__ __forceinline__ void load_cols(const float* __restrict__ m, int64_t ld, int r0, int rows, int d, f32x4 (&f)[P]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, c0 = lane & 15;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int r = r0 + 4 * g + t;
    const float* p = m + (int64_t)min(r, rows - 1) * ld;
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int c = 16 * q + c0;
      const float v = p[c < d ? c : 0];
      f[q][t] = r < rows && c < d ? v : 0.f;
    }
  }
}
// D[i][j] = sum over the dimensions of a[i] b[j], both from load_rows
template <int P>
__device__ __forceinline__ f32x4 dot_rows(const f32x4 (&a)[P], const f32x4 (&b)[P]) {
  f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};      // (two chains: no product waits for the one before)
#pragma unroll
  for (int q = 0; q < P; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) s[t & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][t], b[q][t], s[t & 1], 0, 0, 0);
  return s[0] + s[1];
}
// o[piece][i] (dimension 16 piece + 4 g + i of column j) += sum over the 16 rows of cols[..] w[row of the lane's scores]
template <int P>
__device__ __forceinline__ void add_weighted(f32x4 (&o)[P], const f32x4 (&cols)[P], f32x4 w) {
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int q = 0; q < P; ++q) o[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(cols[q][t], w[t], o[q], 0, 0, 0);
}
// The same for a block on the diagonal, where some of the 16 rows are masked for some columns: a weight of zero does not silence a row
// that holds an infinity or a NaN, so such a block (rare; one branch for the wavefront) is added value by value and masked rows are left
// out.  m: the matrix the rows come from; masked(r): row r0 + r does not count for this lane's column.
template <int P, typename Masked>
__device__ __forceinline__ void add_weighted_diagonal(f32x4 (&o)[P], const f32x4 (&cols)[P], f32x4 w, const float* __restrict__ m, int64_t ld, int r0, int rows, int d,
                                                      Masked masked) {
  bool bad = false;
#pragma unroll
  for (int q = 0; q < P; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) bad = bad || !(fabsf(cols[q][t]) < INFINITY);
  if (!__any(bad)) {
    add_weighted<P>(o, cols, w);
    return;
  }
  const int lane = threadIdx.x & 63, g = lane >> 4;
  for (int r = 0; r < 16 && r0 + r < rows; ++r) {
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) v = (r & 3) == i ? w[i] : v;
    v = __shfl(v, (r >> 2) * 16 + (lane & 15), 64);
    if (masked(r)) continue;
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 16 * q + 4 * g + i;
        if (c < d) o[q][i] += v * m[(int64_t)(r0 + r) * ld + c];
      }
  }
}
// sum over the four lane groups of a column
__device__ __forceinline__ float groups_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float groups_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
template <int P>
__device__ __forceinline__ void store_columns(float* __restrict__ out, int64_t ld, int row, int rows, int d, const f32x4 (&o)[P], float mul) {
  if (row >= rows) return;
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int q = 0; q < P; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 16 * q + 4 * g + i;
      if (c < d) out[(int64_t)row * ld + c] = o[q][i] * mul;
    }
}
// Adds the four wavefronts' `o` in wavefront order into wavefront 0's (red: kWaves - 1 images of P x 64 lanes x 4).
template <int P>
__device__ __forceinline__ void merge_sums(f32x4 (&o)[P], f32x4* red) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (wave > 0) {
#pragma unroll
    for (int q = 0; q < P; ++q) red[((wave - 1) * P + q) * 64 + lane] = o[q];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
      for (int q = 0; q < P; ++q) o[q] += red[(w * P + q) * 64 + lane];
  }
}

template <int P, bool VEC>
__global__ void __launch_bounds__(64 * kWaves)
attn_f32_fwd_kernel(const float* __restrict__ qkv, float* __restrict__ O, float* __restrict__ lse, int S, int H, int A, int causal) {
  __shared__ f32x4 red[(kWaves - 1) * P * 64];
  __shared__ float ml[kWaves][2][16];
  const int a = blockIdx.y, n = blockIdx.z, d = H / A;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4;
  const int q0 = blockIdx.x * 16, q = q0 + (lane & 15);
  const float scale = 1.0f / sqrtf((float)d);
  const int64_t ld = 3 * (int64_t)H;
  const float* base = qkv + (int64_t)n * S * ld + a * d;
  f32x4 qf[P], o[P];
  load_rows<P, VEC>(base, ld, q0, S, d, qf);
#pragma unroll
  for (int i = 0; i < P; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int end = causal ? min(S, q0 + 16) : S;
  for (int t0 = wave * 16; t0 < end; t0 += 16 * kWaves) {
    f32x4 kf[P], vf[P];
    load_rows<P, VEC>(base + H, ld, t0, S, d, kf);
    load_cols<P>(base + 2 * H, ld, t0, S, d, vf);
    f32x4 s = dot_rows<P>(kf, qf);                         // scores of keys t0 + 4 g + i with query q
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + 4 * g + i;
      s[i] = (t < S && (!causal || t <= q)) ? s[i] * scale : -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    const float m_new = fmaxf(m, groups_max(mx));          // (this wavefront's maximum of the column)
    const float shift = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m - shift);
    f32x4 p;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) { p[i] = expf(s[i] - shift); sum += p[i]; }
    l = l * alpha + sum;
    m = m_new;
#pragma unroll
    for (int i = 0; i < P; ++i) o[i] *= alpha;
    if (causal && t0 == q0) add_weighted_diagonal<P>(o, vf, p, base + 2 * H, ld, t0, S, d, [&](int r) { return t0 + r > q; });
    else add_weighted<P>(o, vf, p);
  }
  l = groups_sum(l);
  if (g == 0) { ml[wave][0][lane] = m; ml[wave][1][lane] = l; }
  __syncthreads();
  float mx = -INFINITY, sum = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, ml[w][0][lane & 15]);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) sum += ml[w][1][lane & 15] * expf(ml[w][0][lane & 15] - mx);
  const float mine = expf(m - mx);
#pragma unroll
  for (int i = 0; i < P; ++i) o[i] *= mine;
  merge_sums<P>(o, red);
  if (wave == 0) {
    store_columns<P>(O + (int64_t)n * S * H + a * d, H, q, S, d, o, 1.0f / sum);
    if (g == 0 && q < S) lse[((int64_t)n * A + a) * S + q] = mx + logf(sum);
  }
}

// o[r] . do[r] of row r = r0 + l % 16, in every lane of the column; dof: those rows of dO
template <int P, bool VEC>
__device__ __forceinline__ float row_dot(const float* __restrict__ O, int64_t ld, int r0, int rows, int d, const f32x4 (&dof)[P]) {
  f32x4 of[P];
  load_rows<P, VEC>(O, ld, r0, rows, d, of);
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) v = fmaf(of[i][e], dof[i][e], v);
  return groups_sum(v);
}

// dQ[s] = scale * sum_t dZ[s,t] K[t],  dZ = P (dP - dvec[s]),  dP[s,t] = dO[s] . V[t];  dvec[s] = dO[s] . O[s] on the way
template <int P, bool VEC>
__device__ __forceinline__ void dq_block(const float* __restrict__ qkv, const float* __restrict__ O, const float* __restrict__ dO, const float* __restrict__ lse,
                                         float* __restrict__ dvec, float* __restrict__ dqkv, int S, int H, int A, int causal, int block, f32x4* red) {
  const int a = blockIdx.y, n = blockIdx.z, d = H / A;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4;
  const int q0 = block * 16, q = q0 + (lane & 15);
  const float scale = 1.0f / sqrtf((float)d);
  const int64_t ld = 3 * (int64_t)H, stat = ((int64_t)n * A + a) * S;
  const float* base = qkv + (int64_t)n * S * ld + a * d;
  const int64_t orow = (int64_t)n * S * H + a * d;
  f32x4 qf[P], dof[P], dq[P];
  load_rows<P, VEC>(base, ld, q0, S, d, qf);
  load_rows<P, VEC>(dO + orow, H, q0, S, d, dof);
  const float dv = row_dot<P, VEC>(O + orow, H, q0, S, d, dof);
  if (wave == 0 && g == 0 && q < S) dvec[stat + q] = dv;
  const float l = lse[stat + min(q, S - 1)];
#pragma unroll
  for (int i = 0; i < P; ++i) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int end = causal ? min(S, q0 + 16) : S;
  for (int t0 = wave * 16; t0 < end; t0 += 16 * kWaves) {
    f32x4 kf[P], vf[P], kc[P];
    load_rows<P, VEC>(base + H, ld, t0, S, d, kf);
    load_rows<P, VEC>(base + 2 * H, ld, t0, S, d, vf);
    load_cols<P>(base + H, ld, t0, S, d, kc);
    const f32x4 s = dot_rows<P>(kf, qf), dp = dot_rows<P>(vf, dof);
    f32x4 dz;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + 4 * g + i;
      dz[i] = (t < S && (!causal || t <= q)) ? expf(s[i] * scale - l) * (dp[i] - dv) : 0.f;
    }
    if (causal && t0 == q0) add_weighted_diagonal<P>(dq, kc, dz, base + H, ld, t0, S, d, [&](int r) { return t0 + r > q; });
    else add_weighted<P>(dq, kc, dz);
  }
  merge_sums<P>(dq, red);
  if (wave == 0) store_columns<P>(dqkv + (int64_t)n * S * ld + a * d, ld, q, S, d, dq, scale);
}

// dV[t] = sum_s P[s,t] dO[s],  dK[t] = scale * sum_s dZ[s,t] Q[s].  OWN: forms dvec of the queries it meets itself, as the dQ blocks do.
template <int P, bool VEC, bool OWN>
__device__ __forceinline__ void dkv_block(const float* __restrict__ qkv, const float* __restrict__ O, const float* __restrict__ dO, const float* __restrict__ lse,
                                          const float* __restrict__ dvec, float* __restrict__ dqkv, int S, int H, int A, int causal, int block, f32x4* red) {
  const int a = blockIdx.y, n = blockIdx.z, d = H / A;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4;
  const int t0 = block * 16, t = t0 + (lane & 15);
  const float scale = 1.0f / sqrtf((float)d);
  const int64_t ld = 3 * (int64_t)H, stat = ((int64_t)n * A + a) * S;
  const float* base = qkv + (int64_t)n * S * ld + a * d;
  const float* dob = dO + (int64_t)n * S * H + a * d;
  f32x4 kf[P], vf[P], dk[P], dvv[P];
  load_rows<P, VEC>(base + H, ld, t0, S, d, kf);
  load_rows<P, VEC>(base + 2 * H, ld, t0, S, d, vf);
#pragma unroll
  for (int i = 0; i < P; ++i) { dk[i] = f32x4{0.f, 0.f, 0.f, 0.f}; dvv[i] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  for (int q0 = (causal ? t0 : 0) + wave * 16; q0 < S; q0 += 16 * kWaves) {
    f32x4 qf[P], dof[P], qc[P], doc[P];
    load_rows<P, VEC>(base, ld, q0, S, d, qf);
    load_rows<P, VEC>(dob, H, q0, S, d, dof);
    load_cols<P>(base, ld, q0, S, d, qc);
    load_cols<P>(dob, H, q0, S, d, doc);
    f32x4 l, dv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = min(q0 + 4 * g + i, S - 1);
      l[i] = lse[stat + q];
      if (!OWN) dv[i] = dvec[stat + q];
    }
    if (OWN) {
      const float own = row_dot<P, VEC>(O + (int64_t)n * S * H + a * d, H, q0, S, d, dof);
#pragma unroll
      for (int i = 0; i < 4; ++i) dv[i] = __shfl(own, 4 * g + i, 64);
    }
    const f32x4 s = dot_rows<P>(qf, kf), dp = dot_rows<P>(dof, vf);      // rows: queries q0 + 4 g + i, column: key t
    f32x4 p, dz;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = q0 + 4 * g + i;
      const bool ok = q < S && (!causal || t <= q);
      p[i] = ok ? expf(s[i] * scale - l[i]) : 0.f;
      dz[i] = ok ? p[i] * (dp[i] - dv[i]) : 0.f;
    }
    if (causal && q0 == t0) {
      add_weighted_diagonal<P>(dvv, doc, p, dob, H, q0, S, d, [&](int r) { return q0 + r < t; });
      add_weighted_diagonal<P>(dk, qc, dz, base, ld, q0, S, d, [&](int r) { return q0 + r < t; });
    } else {
      add_weighted<P>(dvv, doc, p);
      add_weighted<P>(dk, qc, dz);
    }
  }
  float* out = dqkv + (int64_t)n * S * ld + a * d;
  merge_sums<P>(dvv, red);
  if (wave == 0) store_columns<P>(out + 2 * H, ld, t, S, d, dvv, 1.0f);
  merge_sums<P>(dk, red);
  if (wave == 0) store_columns<P>(out + H, ld, t, S, d, dk, scale);
}

template <int P, bool VEC>
__global__ void __launch_bounds__(64 * kWaves)
attn_f32_dq_kernel(const float* __restrict__ qkv, const float* __restrict__ O, const float* __restrict__ dO, const float* __restrict__ lse,
                   float* __restrict__ dvec, float* __restrict__ dqkv, int S, int H, int A, int causal) {
  __shared__ f32x4 red[(kWaves - 1) * P * 64];
  dq_block<P, VEC>(qkv, O, dO, lse, dvec, dqkv, S, H, A, causal, blockIdx.x, red);
}
template <int P, bool VEC>
__global__ void __launch_bounds__(64 * kWaves)
attn_f32_dkv_kernel(const float* __restrict__ qkv, const float* __restrict__ dO, const float* __restrict__ lse,
                    const float* __restrict__ dvec, float* __restrict__ dqkv, int S, int H, int A, int causal) {
  __shared__ f32x4 red[(kWaves - 1) * P * 64];
  dkv_block<P, VEC, false>(qkv, nullptr, dO, lse, dvec, dqkv, S, H, A, causal, blockIdx.x, red);
}
// Both in one launch where they fit on the chip side by side: up to 512 blocks (256 for heads wider than 64, whose blocks have a compute unit each); the
// results are the same bits either way.  Two launches -> one, us: 2 x 128 tokens, 4 heads of 64 24.4 -> 14.3; 4 x 128, 8 heads, no mask (512 blocks) 26.6 -> 21.2;
// 2 x 512, 4 heads (512) 72.4 -> 57.1.  Beyond: 1024 blocks 178 -> 181, 2048 65.5 -> 75.6; heads of 128, 1024 blocks 259 -> 295.
template <int P, bool VEC>
__global__ void __launch_bounds__(64 * kWaves)
attn_f32_bwd_kernel(const float* __restrict__ qkv, const float* __restrict__ O, const float* __restrict__ dO, const float* __restrict__ lse,
                    float* __restrict__ dvec, float* __restrict__ dqkv, int S, int H, int A, int causal) {
  __shared__ f32x4 red[(kWaves - 1) * P * 64];
  const int tiles = (S + 15) / 16, b = blockIdx.x;
  if (b < tiles) dkv_block<P, VEC, true>(qkv, O, dO, lse, nullptr, dqkv, S, H, A, causal, b, red);
  else dq_block<P, VEC>(qkv, O, dO, lse, dvec, dqkv, S, H, A, causal, causal ? 2 * tiles - 1 - b : b - tiles, red);      // (the longest first)
}

int check_f32(int S, int H, int A) {
  if (H / A > kMaxHeadDim) return fail(CEPHALO_EUNSUPPORTED, "attention: head dim %d > %d", H / A, kMaxHeadDim);
  if (S > kMaxSeq) return fail(CEPHALO_EUNSUPPORTED, "attention (fp32): %d tokens a sample > %d", S, kMaxSeq);
  return CEPHALO_OK;
}

// pieces of 16 dimensions: 2, 4 or 8 (a head in between runs on the next with zeros)
#define ATTN_F32_FORMS(CALL)                                                                                      \
  const int pieces = (H / A + 15) / 16;                                                                           \
  if (vec) { if (pieces <= 2) { CALL(2, true) } else if (pieces <= 4) { CALL(4, true) } else { CALL(8, true) } }  \
  else { if (pieces <= 2) { CALL(2, false) } else if (pieces <= 4) { CALL(4, false) } else { CALL(8, false) } }
}  // namespace

int launch_attn_fwd_f32(const float* qkv, float* O, float* lse, int m, int S, int H, int A, int causal, hipStream_t s) {
  if (const int rc = check_f32(S, H, A); rc != CEPHALO_OK) return rc;
  const bool vec = (H / A) % 4 == 0 && aligned16(qkv);
  dim3 grid((S + 15) / 16, A, m);
#define CALL(P, V) attn_f32_fwd_kernel<P, V><<<grid, 64 * kWaves, 0, s>>>(qkv, O, lse, S, H, A, causal);
  ATTN_F32_FORMS(CALL)
#undef CALL
  CEPHALO_CHECK_LAUNCH("attn_fwd");
  return CEPHALO_OK;
}

int launch_attn_bwd_f32(const float* qkv, const float* O, const float* dO, const float* lse, float* dvec, float* dqkv,
                        int m, int S, int H, int A, int causal, hipStream_t s) {
  if (const int rc = check_f32(S, H, A); rc != CEPHALO_OK) return rc;
  const bool vec = (H / A) % 4 == 0 && aligned16(qkv) && aligned16(O) && aligned16(dO);
  dim3 grid((S + 15) / 16, A, m);
  if (2 * (int64_t)grid.x * A * m <= (H / A <= 64 ? 512 : 256)) {
    grid.x *= 2;
#define CALL(P, V) attn_f32_bwd_kernel<P, V><<<grid, 64 * kWaves, 0, s>>>(qkv, O, dO, lse, dvec, dqkv, S, H, A, causal);
    ATTN_F32_FORMS(CALL)
#undef CALL
    CEPHALO_CHECK_LAUNCH("attn_bwd");
    return CEPHALO_OK;
  }
#define CALL(P, V)                                                                                                \
  attn_f32_dq_kernel<P, V><<<grid, 64 * kWaves, 0, s>>>(qkv, O, dO, lse, dvec, dqkv, S, H, A, causal);            \
  attn_f32_dkv_kernel<P, V><<<grid, 64 * kWaves, 0, s>>>(qkv, dO, lse, dvec, dqkv, S, H, A, causal);
  ATTN_F32_FORMS(CALL)
#undef CALL
  CEPHALO_CHECK_LAUNCH("attn_bwd");
  return CEPHALO_OK;
}

}  // namespace cephalo
