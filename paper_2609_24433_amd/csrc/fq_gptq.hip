// GPTQ in the transformed coordinates (eq. (7), Sec. III-F): the offline rounding of
// four-bit folded weights against the second moment G = Z Z^T of calibration tokens taken
// in the runtime transform's coordinates, with diagonal damping.  Four stages, each a few
// kernels:
//   transform: the prologue's transform alone (fold-before multiplier, unnormalized
//     blockwise butterfly in the prologue's stage order, fold-after multiplier), fp32
//     rows out; it gives the calibration tokens Z and the folded weight rows;
//   second moment: G = sum_t z_t z_t^T in fp64 on the matrix cores, operands from registers;
//   factor: U upper triangular with (G + lambda I)^-1 = U^T U.  With the index reversal
//     P, the lower Cholesky factor L of A = P H P gives H = V V^T for the upper triangular
//     V = P L P, so U = V^-1 = P L^-1 P: a blocked Cholesky of one launch per 64 columns (panel,
//     trailing update and the next diagonal block's factor and inverse together) and a
//     triangular inverse that merges neighbouring diagonal blocks level by level, two launches
//     a level;
//   sweep: the lazy-batch column sweep in fp64, 128 columns per block: inside a block the
//     columns are rounded one at a time by a wave that holds its rows in registers; after the
//     block one fp64 product pushes the block's errors onto the later
//     columns.  Every operation and its order follow the fp64 contract of the sweep, so the
//     codes are reproducible bit for bit.
// The fp64 matrix instruction (42 TFLOP/s measured with four chains per wave) adds its four
// products one after the other with one rounding each, so a chain of instructions is the
// chain of fused multiply-adds that the contract asks for.  K = 1024, N = 1536, T = 2048: second
// moment 92 us (502 before), factor 0.52 ms (2.7: one wave per diagonal block, row-parallel solves
// with divisions, one launch per product), sweep 0.27 ms (1.2: barriers and a division per column).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fq_device.hpp"
#include "fq_launch.hpp"

namespace fq {

// ---------------------------------------------------------------------------------------
// transform

// One workgroup of E threads per E consecutive channels of a row (E = max(b, 128); K is
// a multiple of 128 and of b; grid x = rows, y = channel groups).  Stage h exchanges through LDS: the lower index of a pair
// gets a + c, the upper a - c, the same fp32 additions as the prologue's butterfly.
template <typename Tin, int E>
__global__ __launch_bounds__(E) void transform_kernel(const void *x, int64_t ldx, const float *pre,
                                                      const float *post, int K, int b, float *z) {
  __shared__ float buf[E];
  const int t = threadIdx.x;
  const int64_t row = blockIdx.x;
  const int c = blockIdx.y * E + t;
  float v;
  if constexpr (sizeof(Tin) == 2)
    v = bf16_lo(reinterpret_cast<const uint16_t *>(x)[row * ldx + c]);
  else
    v = reinterpret_cast<const float *>(x)[row * ldx + c];
  if (pre) v = v * pre[c];
  for (int h = 1; h < b; h *= 2) {
    buf[t] = v;
    __syncthreads();
    const float p = buf[t ^ h];
    v = (t & h) ? p - v : v + p;
    __syncthreads();
  }
  if (post) v = v * post[c];
  z[row * K + c] = v;
}

template <typename Tin>
static hipError_t launch_transform_t(const void *x, int64_t ldx, const float *pre, const float *post, int64_t M,
                                     int K, int b, float *z, hipStream_t s) {
  if (b <= 128) {
    hipLaunchKernelGGL((transform_kernel<Tin, 128>), dim3((unsigned)M, (unsigned)(K / 128)), dim3(128), 0, s, x,
                       ldx, pre, post, K, b, z);
  } else {
    hipLaunchKernelGGL((transform_kernel<Tin, 256>), dim3((unsigned)M, (unsigned)(K / 256)), dim3(256), 0, s, x,
                       ldx, pre, post, K, b, z);
  }
  return hipGetLastError();
}

hipError_t launch_transform(const void *x, bool x_is_f32, int64_t ldx, const float *pre, const float *post,
                            int64_t M, int K, int b, float *z, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (M > 2147483647) return hipErrorInvalidValue;
  return x_is_f32 ? launch_transform_t<float>(x, ldx, pre, post, M, K, b, z, s)
                  : launch_transform_t<uint16_t>(x, ldx, pre, post, M, K, b, z, s);
}

// ---------------------------------------------------------------------------------------
// fp64 product update: C (op)= sum_k A[i][k] B[k][j], every element's sum an fma chain in
// ascending k from +0, then C = C - sum, C = -sum or C = sum, on the fp64 matrix
// instruction.  A and B are addressed through element strides, so transposed operands need no
// copy.

enum : int { kSub = 0, kSetNeg = 1, kSet = 2 };

struct DProd {
  const double *a;
  int64_t a_si, a_sk;  // element strides of A: rows i, k
  const double *b;
  int64_t b_sk, b_sj;  // element strides of B: k, columns j
  double *c;
  int64_t ldc;
  int64_t m, n, kd;
  int mode;
  int kskip;  // B is lower triangular: tile column j0 sums k >= j0 only (the rest are zeros)
  int klow;   // A is lower triangular: tile row i0 sums k < i0 + 32 only
  // a batch of `batch` products (0 = one) at these element strides; m_last: rows of the last one
  // when it is narrower (else 0); kd_is_m: its k range shrinks with its rows
  int batch;
  int64_t a_sz, b_sz, c_sz, m_last;
  int kd_is_m;
};

typedef double v4d __attribute__((ext_vector_type(4)));
// 16 x 16 x 4 product update: lane l holds row (column) l % 16 and k = l / 16 of A (B); the result's
// lane l holds column l % 16 and rows l / 16 + 4 i.  Each element's four products are added in
// ascending k, each with one rounding (a chain of fused multiply-adds; checked on the card).
__device__ __forceinline__ v4d mfma_f64(double a, double b, v4d c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
#else
  return c;
#endif
}

// 32 x 32 tiles, each of 4 waves a 16 x 16 quarter (one chain of instructions); k in chunks of
// 32 through LDS, the next chunk's loads in flight while one is multiplied.  Several workgroups
// share a compute unit and cover each other's chains.
constexpr int kDT = 32;  // tile edge
__global__ __launch_bounds__(256) void dprod_kernel(DProd p) {
  constexpr int T = kDT, KC = 32, PER = T * KC / 256;
  __shared__ double as[KC][T + 2];
  __shared__ double bs[KC][T + 2];
  const int ti = blockIdx.y, tj = blockIdx.x, z = blockIdx.z;
  const int64_t m = p.m_last && z == (int)gridDim.z - 1 ? p.m_last : p.m;
  const int64_t kd = p.kd_is_m ? m : p.kd;
  const int64_t i0 = (int64_t)ti * T, j0 = (int64_t)tj * T;
  if (i0 >= m) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = (wave >> 1) * 16, wj = (wave & 1) * 16, l16 = lane & 15, l4 = lane >> 4;
  const double *A = p.a + z * p.a_sz, *Bm = p.b + z * p.b_sz;
  double *C = p.c + z * p.c_sz;
  v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
  const bool a_krun = p.a_sk == 1;  // consecutive lanes along k when k is the contiguous index
  const bool b_jrun = p.b_sj == 1;
  const int64_t kend = p.klow && i0 + T < kd ? i0 + T : kd;
  double va[PER], vb[PER];
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + 256 * u;
      const int64_t gi = i0 + (a_krun ? e / KC : e % T), gk = k0 + (a_krun ? e % KC : e / T);
      const int64_t gj = j0 + (b_jrun ? e % T : e / KC), gkb = k0 + (b_jrun ? e / T : e % KC);
      va[u] = gi < m && gk < kend ? A[gi * p.a_si + gk * p.a_sk] : 0.0;
      vb[u] = gj < p.n && gkb < kend ? Bm[gkb * p.b_sk + gj * p.b_sj] : 0.0;
    }
  };
  const int64_t kbeg = p.kskip ? j0 : 0;
  if (kbeg < kend) fetch(kbeg);
  for (int64_t k0 = kbeg; k0 < kend; k0 += KC) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + 256 * u;
      as[a_krun ? e % KC : e / T][a_krun ? e / KC : e % T] = va[u];
      bs[b_jrun ? e / T : e % KC][b_jrun ? e % T : e / KC] = vb[u];
    }
    __syncthreads();
    if (k0 + KC < kend) fetch(k0 + KC);
    // entries past kend are zeros: they add nothing
#pragma unroll
    for (int k = 0; k < KC; k += 4) acc = mfma_f64(as[k + l4][wi + l16], bs[k + l4][wj + l16], acc);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t gi = i0 + wi + 4 * q + l4, gj = j0 + wj + l16;
    if (gi >= m || gj >= p.n) continue;
    double *dst = C + gi * p.ldc + gj;
    switch (p.mode) {
      case kSub: *dst = *dst - acc[q]; break;
      case kSetNeg: *dst = -acc[q]; break;
      default: *dst = acc[q]; break;
    }
  }
}

// The grid's y extent holds 65535 tiles of rows (2 097 120 rows), so longer products (the sweep of
// as many weight rows; never a batch) go out in as many launches.
static hipError_t dprod(const DProd &p, hipStream_t s) {
  if (p.m <= 0 || p.n <= 0) return hipSuccess;
  constexpr int64_t kRows = (int64_t)65535 * kDT;
  const int64_t tn = (p.n + kDT - 1) / kDT;
  if (tn > 2147483647 || (p.batch > 0 && p.m > kRows)) return hipErrorInvalidValue;
  for (int64_t r0 = 0; r0 < p.m; r0 += kRows) {
    DProd q = p;
    q.a = p.a + r0 * p.a_si;
    q.c = p.c + r0 * p.ldc;
    q.m = p.m - r0 < kRows ? p.m - r0 : kRows;
    hipLaunchKernelGGL(dprod_kernel, dim3((unsigned)tn, (unsigned)((q.m + kDT - 1) / kDT), (unsigned)(p.batch > 0 ? p.batch : 1)),
                       dim3(256), 0, s, q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

__global__ __launch_bounds__(256) void fill_kernel(double *d, int64_t n, double v) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n) d[e] = v;
}

// G[i][j] (+)= sum_t z[t][i] z[t][j], lower 32 x 32 tiles mirrored.  The 4 waves of a workgroup take
// every fourth group of 32 tokens, operands straight from z into registers (fp32, widened exactly),
// and add up in wave order.  K = 1024, T = 2048: 528 tiles, two waves per SIMD.
__global__ __launch_bounds__(256) void second_moment_kernel(const float *z, int64_t ldz, int64_t T, int K, double *G,
                                                            int accumulate) {
  __shared__ double part[3][32][33];
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  const float *zi = z + ti * 32 + l16, *zj = z + tj * 32 + l16;
  v4d acc[2][2];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[r][c] = v4d{0.0, 0.0, 0.0, 0.0};
  float a[8][2], b[8][2];
  auto fetch = [&](int64_t t0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int64_t t = t0 + 4 * q + l4;
      const bool in = t < T;
      const int64_t o = (in ? t : T - 1) * ldz;
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const float x = zi[o + 16 * r], y = zj[o + 16 * r];
        a[q][r] = in ? x : 0.0f;
        b[q][r] = in ? y : 0.0f;
      }
    }
  };
  const int64_t groups = (T + 31) / 32;
  if (wave < groups) fetch((int64_t)wave * 32);
  for (int64_t g = wave; g < groups; g += 4) {
    float ca[8][2], cb[8][2];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        ca[q][r] = a[q][r];
        cb[q][r] = b[q][r];
      }
    if (g + 4 < groups) fetch((g + 4) * 32);
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[r][c] = mfma_f64((double)ca[q][r], (double)cb[q][c], acc[r][c]);
  }
  if (wave > 0)
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) part[wave - 1][16 * r + 4 * q + l4][16 * c + l16] = acc[r][c][q];
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int li = 16 * r + 4 * q + l4, lj = 16 * c + l16;
        const int64_t i = ti * 32 + li, j = tj * 32 + lj;
        if (j > i) continue;
        double v = acc[r][c][q] + part[0][li][lj];
        v += part[1][li][lj];
        v += part[2][li][lj];
        if (accumulate) v += G[i * K + j];
        G[i * K + j] = v;
        if (i != j) G[j * K + i] = v;
      }
}

hipError_t launch_gptq_hessian(const float *z, int64_t ldz, int64_t T, int K, double *G, bool accumulate,
                               hipStream_t s) {
  if (T <= 0) {
    if (accumulate) return hipSuccess;
    const int64_t n = (int64_t)K * K;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, G, n, 0.0);
    return hipGetLastError();
  }
  const unsigned t = (unsigned)(K / 32);
  hipLaunchKernelGGL(second_moment_kernel, dim3(t, t), dim3(256), 0, s, z, ldz, T, K, G, accumulate ? 1 : 0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// factor

// lambda = damp * mean(diag G), one workgroup; an all-zero diagonal gives lambda = 0,
// which the reversal kernel turns into the identity.
__global__ __launch_bounds__(256) void damp_kernel(const double *G, int K, double damp, double *lam) {
  __shared__ double part[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < K; i += 256) acc += G[(int64_t)i * K + i];
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) lam[0] = damp * (part[0] / (double)K);
}

// A = P (G + lambda I) P (index reversal), or the identity when lambda = 0; X = 0.
__global__ __launch_bounds__(256) void reverse_kernel(const double *G, int K, const double *lam, double *A,
                                                      double *X) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)K * K) return;
  const int64_t i = e / K, j = e % K;
  const double l = lam[0];
  double v;
  if (l == 0.0)
    v = i == j ? 1.0 : 0.0;
  else
    v = G[(K - 1 - i) * (int64_t)K + (K - 1 - j)] + (i == j ? l : 0.0);
  A[e] = v;
  X[e] = 0.0;
}

constexpr int kNb = 64;  // Cholesky / inverse block

// Factor and inverse of a 64 x 64 diagonal block in LDS (row stride kLd), by a workgroup of 512
// threads in four 16-wide steps: one wave factors the step's 16 columns with each lane holding
// its row of them in registers (the pivot row's values through scalar registers, 1 / sqrt of the
// pivot by two Newton steps on the hardware estimate, exact at 1), then the waves update the
// rest; the inverse follows from the 16-wide diagonal blocks' inverses (16-wide products on the
// matrix instruction).  a: the block (lower part), becomes L with zeros above; x: becomes L^-1.
// One wave's chain of 64 pivots bounds it (about 0.25 us each; the pivot row's values in scalar
// register pairs are more than there are, so the compiler keeps about 200 of them in vector lanes);
// the former wave-per-block factor and the row-parallel solves with fp64 divisions took 83 us a block.
constexpr int kLd = kNb + 1;
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// c + f S B over 16 channels by one wave: S = s[r0 + ..][c0 + ..], B = b[k0 + k][j0 + j], or with TR
// its transpose b[k0 + j][j0 + k]; the result in the matrix instruction's layout.
template <bool TR>
__device__ __forceinline__ v4d block16(const double *s, int r0, int c0, const double *b, int k0, int j0, v4d c, double f) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  double av[4], bv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    av[q] = f * s[(r0 + l16) * kLd + c0 + 4 * q + l4];
    bv[q] = TR ? b[(k0 + l16) * kLd + j0 + 4 * q + l4] : b[(k0 + 4 * q + l4) * kLd + j0 + l16];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) c = mfma_f64(av[q], bv[q], c);
  return c;
}
__device__ __forceinline__ void put16(double *d, int r0, int c0, v4d v) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) d[(r0 + 4 * q + l4) * kLd + c0 + l16] = v[q];
}
__device__ __forceinline__ void factor_block(double *a, double *x) {
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ double rdiag[kNb];
  for (int e = tid; e < kNb * kNb; e += 512) x[(e / kNb) * kLd + e % kNb] = 0.0;
  __syncthreads();
  for (int o = 0; o < kNb; o += 16) {
    const int nb = (kNb - o - 16) / 16;
    if (wave == 0) {
      double r[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) r[c] = a[lane * kLd + o + c];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double d = lane_value(r[j], o + j);
        double y = __builtin_amdgcn_rsq(d);
        y = __builtin_fma(0.5 * y, __builtin_fma(-d * y, y, 1.0), y);
        y = __builtin_fma(0.5 * y, __builtin_fma(-d * y, y, 1.0), y);
        if (lane == 0) rdiag[o + j] = y;  // 1 / l_jj
        r[j] = r[j] * y;
#pragma unroll
        for (int c = j + 1; c < 16; ++c) r[c] = __builtin_fma(-r[j], lane_value(r[j], o + c), r[c]);
      }
#pragma unroll
      for (int c = 0; c < 16; ++c) a[lane * kLd + o + c] = o + c <= lane ? r[c] : 0.0;
    }
    __syncthreads();
    // the rest: lower blocks (i, j) of nb x nb
    for (int e = wave; e < nb * (nb + 1) / 2; e += 8) {
      const int i = e >= 3 ? 2 : (e >= 1 ? 1 : 0), j = e - i * (i + 1) / 2;
      const int r0 = o + 16 + 16 * i, c0 = o + 16 + 16 * j;
      v4d v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = a[(r0 + 4 * q + l4) * kLd + c0 + l16];
      v = block16<true>(a, r0, o, a, c0, o, v, -1.0);
      put16(a, r0, c0, v);
    }
    __syncthreads();
  }
  // inverses of the 16-wide diagonal blocks, one wave each: lane i holds column i % 16,
  // x_m = (e_m - sum_{t < m} l_mt x_t) / l_mm
  if (wave < 4) {
    const int o = 16 * wave, i = l16;
    double r[16], xi[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) r[c] = a[(o + i) * kLd + o + c];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      double t = m == i ? 1.0 : 0.0;
#pragma unroll
      for (int q = 0; q < m; ++q) t = __builtin_fma(-xi[q], lane_value(r[q], m), t);
      xi[m] = t * rdiag[o + m];
    }
    if (lane < 16)
#pragma unroll
      for (int m = 0; m < 16; ++m) x[(o + m) * kLd + o + i] = m >= i ? xi[m] : 0.0;
  }
  __syncthreads();
  // X_ij = -X_ii sum_{j <= m < i} L_im X_mj for the 16-wide blocks, by distance from the diagonal,
  // one wave per block; the sum goes where the result will be, then the product replaces it
  for (int d = 1; d < 4; ++d) {
    if (wave < 4 - d) {
      const int i = (wave + d) * 16, j = wave * 16;
      v4d t = v4d{0.0, 0.0, 0.0, 0.0};
      for (int m = j; m < i; m += 16) t = block16<false>(a, i, m, x, m, j, t, 1.0);
      put16(x, i, j, t);
      wave_lds_fence();
      t = block16<false>(x, i, i, x, i, j, v4d{0.0, 0.0, 0.0, 0.0}, -1.0);
      wave_lds_fence();
      put16(x, i, j, t);
    }
    __syncthreads();
  }
}

__device__ __forceinline__ void store_block(double *dst, int64_t ld, const double *src) {
  for (int e = threadIdx.x; e < kNb * kNb; e += 512) dst[(e / kNb) * ld + e % kNb] = src[(e / kNb) * kLd + e % kNb];
}

// The first diagonal block: L_00 into A, its inverse into X.
__global__ __launch_bounds__(512) void chol_first_kernel(double *A, int K, double *X) {
  extern __shared__ double sm[];
  double *a = sm, *x = sm + kNb * kLd;
  for (int e = threadIdx.x; e < kNb * kNb; e += 512) a[(e / kNb) * kLd + e % kNb] = A[(int64_t)(e / kNb) * K + e % kNb];
  __syncthreads();
  factor_block(a, x);
  store_block(A, K, a);
  store_block(X, K, x);
}

// One 64-wide step of the Cholesky factor after its diagonal block (k0): workgroup (ti, tj), ti >=
// tj, forms the panel blocks L_i = A_i X_kk^T and L_j it needs itself (the panel is read where it
// was, below the diagonal, and its factor goes to the transposed place above it, so no
// workgroup waits for another) and updates its tile of the trailing matrix; workgroup (0, 0),
// whose tile is the next diagonal block, goes on to factor and invert it.
__global__ __launch_bounds__(512) void chol_step_kernel(double *A, int K, double *X, int k0) {
  extern __shared__ double sm[];
  double *s0 = sm, *s1 = sm + kNb * kLd, *s2 = sm + 2 * kNb * kLd;
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = (wave >> 2) * 32, wj = (wave & 3) * 16, l16 = lane & 15, l4 = lane >> 4;
  const int64_t ri = k0 + kNb + (int64_t)ti * kNb, rj = k0 + kNb + (int64_t)tj * kNb;
  for (int e = tid; e < kNb * kNb; e += 512) {
    const int r = e / kNb, c = e % kNb;
    s0[r * kLd + c] = A[(ri + r) * K + k0 + c];
    if (ti != tj) s1[r * kLd + c] = A[(rj + r) * K + k0 + c];
    s2[r * kLd + c] = X[(int64_t)(k0 + r) * K + k0 + c];
  }
  double old[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) old[r][q] = A[(ri + wi + 16 * r + 4 * q + l4) * K + rj + wj + l16];
  __syncthreads();
  // C (32 x 16 per wave) = S T^T over the first kn channels
  auto product = [&](const double *S, const double *Tt, int kn, v4d (&acc)[2]) {
    acc[0] = acc[1] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k = 0; k < kn; k += 4) {
      const double bv = Tt[(wj + l16) * kLd + k + l4];
#pragma unroll
      for (int r = 0; r < 2; ++r) acc[r] = mfma_f64(S[(wi + 16 * r + l16) * kLd + k + l4], bv, acc[r]);
    }
  };
  auto put = [&](double *S, const v4d (&v)[2]) {
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(wi + 16 * r + 4 * q + l4) * kLd + wj + l16] = v[r][q];
  };
  v4d li[2], lj[2], up[2];
  product(s0, s2, wj + 16, li);  // X_kk is lower triangular
  if (ti != tj) product(s1, s2, wj + 16, lj);
  __syncthreads();
  put(s0, li);
  if (ti != tj) put(s1, lj);
  __syncthreads();
  if (tj == 0)  // L_i^T above the diagonal
    for (int e = tid; e < kNb * kNb; e += 512) {
      const int c = e / kNb, r = e % kNb;
      A[(int64_t)(k0 + c) * K + ri + r] = s0[r * kLd + c];
    }
  product(s0, ti != tj ? s1 : s0, kNb, up);
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int gr = wi + 16 * r + 4 * q + l4, gc = wj + l16;
      const double v = old[r][q] - up[r][q];
      if (ti > 0 || tj > 0) A[(ri + gr) * K + rj + gc] = v;
      else s2[gr * kLd + gc] = v;
    }
  if (ti == 0 && tj == 0) {
    __syncthreads();
    factor_block(s2, s0);
    store_block(A + ri * K + ri, K, s2);
    store_block(X + ri * K + ri, K, s0);
  }
}

// U[i][j] = X[K-1-i][K-1-j] on and above the diagonal, 0 below.
__global__ __launch_bounds__(256) void unreverse_kernel(const double *X, int K, double *U) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)K * K) return;
  const int64_t i = e / K, j = e % K;
  U[e] = j >= i ? X[(K - 1 - i) * (int64_t)K + (K - 1 - j)] : 0.0;
}

size_t gptq_factor_ws_bytes(int K) {
  return ((size_t)2 * K * K + (size_t)(K / 2) * (K / 2)) * sizeof(double) + 256;
}

hipError_t launch_gptq_factor(const double *G, int K, double damp, double *U, void *ws, hipStream_t s) {
  double *A = static_cast<double *>(ws);
  double *X = A + (size_t)K * K;
  double *Tm = X + (size_t)K * K;  // B X_A of the inverse's merges, at most (K/2) x (K/2)
  double *lam = Tm + (size_t)(K / 2) * (K / 2);
  const int64_t n = (int64_t)K * K;
  const unsigned ge = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(damp_kernel, dim3(1), dim3(256), 0, s, G, K, damp, lam);
  hipLaunchKernelGGL(reverse_kernel, dim3(ge), dim3(256), 0, s, G, K, lam, A, X);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // blocked Cholesky A = L L^T: diagonal blocks in place, the rest of L transposed above the
  // diagonal; X gets the diagonal blocks' inverses
  constexpr size_t lds2 = 2 * (size_t)kNb * kLd * sizeof(double), lds3 = 3 * (size_t)kNb * kLd * sizeof(double);
  static std::atomic<uint64_t> attr2{0}, attr3{0};
  if ((e = allow_dynamic_lds(&chol_first_kernel, lds2, attr2)) != hipSuccess) return e;
  if ((e = allow_dynamic_lds(&chol_step_kernel, lds3, attr3)) != hipSuccess) return e;
  hipLaunchKernelGGL(chol_first_kernel, dim3(1), dim3(512), lds2, s, A, K, X);
  for (int k0 = 0; k0 + kNb < K; k0 += kNb) {
    const unsigned t = (unsigned)((K - k0) / kNb - 1);
    hipLaunchKernelGGL(chol_step_kernel, dim3(t, t), dim3(512), lds3, s, A, K, X, k0);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // X = L^-1: pairs of neighbouring diagonal blocks merged level by level (widths 64, 128,
  // 256, ...), every pair of a level in one launch: for A = block 2t, C = block 2t + 1
  // (possibly narrower at the end) and B the part of L below A and left of C,
  // X[C, A] = -X_C (B X_A).  Both products skip the zeros of their triangular operand.
  for (int n = kNb; n < K; n *= 2) {
    const int pairs = (K - n + 2 * n - 1) / (2 * n);
    const int64_t last = (int64_t)(pairs - 1) * 2 * n + n;  // first row of the last C
    const int64_t sz = (int64_t)2 * n * (K + 1), m_last = K - last < n ? K - last : 0;
    DProd p{};
    p.a = A + n;  // B[r][k] = L[n + r][k], kept at A[k][n + r]
    p.a_si = 1;
    p.a_sk = K;
    p.b = X;  // X_A[k][j]
    p.b_sk = K;
    p.b_sj = 1;
    p.c = Tm;
    p.ldc = n;
    p.m = n;
    p.n = n;
    p.kd = n;
    p.mode = kSet;
    p.kskip = 1;
    p.batch = pairs;
    p.a_sz = p.b_sz = sz;
    p.c_sz = (int64_t)n * n;
    p.m_last = m_last;
    if ((e = dprod(p, s)) != hipSuccess) return e;
    DProd q{};
    q.a = X + (int64_t)n * K + n;  // X_C[r][k]
    q.a_si = K;
    q.a_sk = 1;
    q.b = Tm;  // Tm[k][j]
    q.b_sk = n;
    q.b_sj = 1;
    q.c = X + (int64_t)n * K;
    q.ldc = K;
    q.m = n;
    q.n = n;
    q.kd = n;
    q.kd_is_m = 1;
    q.mode = kSetNeg;
    q.klow = 1;
    q.batch = pairs;
    q.a_sz = q.c_sz = sz;
    q.b_sz = (int64_t)n * n;
    q.m_last = m_last;
    if ((e = dprod(q, s)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(unreverse_kernel, dim3(ge), dim3(256), 0, s, X, K, U);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// sweep

constexpr int kSweepBlk = 128;  // columns per lazy batch
constexpr int kSweepRows = 2;   // rows per wave of the in-block sweep

// Per row: A = max |w| (fp32, exact), the fp32 scale, fp64 inv = q / A and step = A / q,
// and the fp64 working copy.  One workgroup per row.
__global__ __launch_bounds__(256) void sweep_init_kernel(const float *w, int64_t ldw, int K, int bits,
                                                         float scale_mult, float *scales, double *rowp,
                                                         double *w64) {
  __shared__ float red[256];
  const int64_t row = blockIdx.x;
  const float *src = w + row * ldw;
  float a = 0.0f;
  for (int c = threadIdx.x; c < K; c += 256) {
    a = fmaxf(a, fabsf(src[c]));
    w64[row * K + c] = (double)src[c];
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float A = red[0];
    const int q = (1 << (bits - 1)) - 1;
    scales[row] = A == 0.0f ? 0.0f : (A * scale_mult) / (float)q;
    rowp[2 * row] = A == 0.0f ? 0.0 : (double)q / (double)A;
    rowp[2 * row + 1] = (double)A / (double)q;
  }
}

// a / b, correctly rounded, from r = 1 / b correctly rounded: two residual corrections of a r
// (Markstein: a quotient within an ulp and the exact residual give the rounded quotient), for b
// far from the ends of the exponent range.
__device__ __forceinline__ double quotient(double a, double b, double r) {
  double q = a * r;
  q = __builtin_fma(__builtin_fma(-q, b, a), r, q);
  return __builtin_fma(__builtin_fma(-q, b, a), r, q);
}

// Columns [i1, i1 + 128) of 2 rows per wave, one column at a time: every lane holds columns l and
// 64 + l of the block in registers and forms the code and error of its own column; column c's
// error is lane c's, broadcast through scalar registers and pushed onto the later columns.  No
// LDS and no barrier: the chain of a column is about 15 dependent fp64 operations.  The rows of U
// are read eight columns ahead.  The errors go to e [N, 128] for the product update.
template <int H, bool PLAIN>
__device__ __forceinline__ void sweep_half(const double *ur, int K, int lane, double q, const double (&inv)[kSweepRows],
                                           const double (&step)[kSweepRows], double diag, double rdiag,
                                           double (&w)[kSweepRows][2], double (&code)[kSweepRows][2],
                                           double (&err)[kSweepRows][2]) {
  constexpr int PF = 8;
  double u0[PF], u1[PF];
  auto fetch = [&](int c) {  // rows 64 H + c .. of the block, this half's columns and the later half's
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const double *row = ur + (int64_t)(64 * H + c + i) * K;
      u0[i] = row[64 * H + lane];
      u1[i] = H == 0 ? row[64 + lane] : 0.0;
    }
  };
  fetch(0);
  for (int c0 = 0; c0 < 64; c0 += PF) {
    double v0[PF], v1[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      v0[i] = u0[i];
      v1[i] = u1[i];
    }
    if (c0 + PF < 64) fetch(c0 + PF);
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int c = c0 + i;
#pragma unroll
      for (int r = 0; r < kSweepRows; ++r) {
        double k = rint(w[r][H] * inv[r]);
        k = k > q ? q : k;
        k = k < -q ? -q : k;
        const double d = w[r][H] - k * step[r];
        const double ev = PLAIN ? d / diag : quotient(d, diag, rdiag);
        if (lane == c) {
          code[r][H] = k;
          err[r][H] = ev;
        }
        const double eb = lane_value(ev, c);
        const double n0 = __builtin_fma(-eb, v0[i], w[r][H]);
        w[r][H] = lane > c ? n0 : w[r][H];
        if constexpr (H == 0) w[r][1] = __builtin_fma(-eb, v1[i], w[r][1]);
      }
    }
  }
}

__global__ __launch_bounds__(256) void sweep_block_kernel(const double *U, int64_t N, int K, int bits, int i1,
                                                          const double *rowp, double *w64, int8_t *codes,
                                                          double *e) {
  const int lane = threadIdx.x & 63;
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kSweepRows;
  if (r0 >= N) return;
  const double q = (double)((1 << (bits - 1)) - 1);
  const double *ur = U + (int64_t)i1 * K + i1;
  double w[kSweepRows][2], inv[kSweepRows], step[kSweepRows], code[kSweepRows][2], err[kSweepRows][2];
#pragma unroll
  for (int r = 0; r < kSweepRows; ++r) {
    const int64_t row = r0 + r < N ? r0 + r : N - 1;  // a row past the end repeats the last one, unstored
    inv[r] = rowp[2 * row];
    step[r] = rowp[2 * row + 1];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      w[r][h] = w64[row * K + i1 + 64 * h + lane];
      code[r][h] = err[r][h] = 0.0;
    }
  }
  const double d0 = ur[(int64_t)lane * (K + 1)], d1 = ur[(int64_t)(64 + lane) * (K + 1)];
  // a diagonal entry near the ends of the exponent range (or not finite) divides plainly
  auto odd = [](double d) {
    const double m = fabs(d);
    return !(m > 0x1p-400 && m < 0x1p400);
  };
  const bool plain = __any(odd(d0) || odd(d1));
  if (plain) {
    sweep_half<0, true>(ur, K, lane, q, inv, step, d0, 0.0, w, code, err);
    sweep_half<1, true>(ur, K, lane, q, inv, step, d1, 0.0, w, code, err);
  } else {
    sweep_half<0, false>(ur, K, lane, q, inv, step, d0, 1.0 / d0, w, code, err);
    sweep_half<1, false>(ur, K, lane, q, inv, step, d1, 1.0 / d1, w, code, err);
  }
#pragma unroll
  for (int r = 0; r < kSweepRows; ++r) {
    if (r0 + r >= N) continue;
    // a row of zeros, or one whose maximum is infinite, has inv = 0: codes 0 and no error, whatever
    // the chain above made of its infinities
    const bool none = inv[r] == 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      codes[(r0 + r) * K + i1 + 64 * h + lane] = none ? (int8_t)0 : (int8_t)code[r][h];
      e[(r0 + r) * kSweepBlk + 64 * h + lane] = none ? 0.0 : err[r][h];
    }
  }
}

size_t gptq_sweep_ws_bytes(int64_t N, int K) {
  return (size_t)N * K * sizeof(double) + (size_t)N * kSweepBlk * sizeof(double) + (size_t)N * 2 * sizeof(double) +
         256;
}

hipError_t launch_gptq_sweep(const float *w, int64_t ldw, const double *U, int64_t N, int K, int bits,
                             float scale_mult, int8_t *codes, float *scales, void *ws, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  if (N > 2147483647) return hipErrorInvalidValue;
  double *w64 = static_cast<double *>(ws);
  double *e = w64 + (size_t)N * K;
  double *rowp = e + (size_t)N * kSweepBlk;
  hipLaunchKernelGGL(sweep_init_kernel, dim3((unsigned)N), dim3(256), 0, s, w, ldw, K, bits, scale_mult, scales,
                     rowp, w64);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const unsigned gb = (unsigned)((N + 4 * kSweepRows - 1) / (4 * kSweepRows));
  for (int i1 = 0; i1 < K; i1 += kSweepBlk) {
    hipLaunchKernelGGL(sweep_block_kernel, dim3(gb), dim3(256), 0, s, U, N, K, bits, i1, rowp, w64, codes, e);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    const int i2 = i1 + kSweepBlk;
    if (i2 < K) {
      // w64[:, i2:] -= e U[i1:i2, i2:], each element's sum an fma chain in ascending k
      DProd p{};
      p.a = e;
      p.a_si = kSweepBlk;
      p.a_sk = 1;
      p.b = U + (int64_t)i1 * K + i2;
      p.b_sk = K;
      p.b_sj = 1;
      p.c = w64 + i2;
      p.ldc = K;
      p.m = N;
      p.n = K - i2;
      p.kd = kSweepBlk;
      p.mode = kSub;
      if ((err = dprod(p, s)) != hipSuccess) return err;
    }
  }
  return hipSuccess;
}

}  // namespace fq
