#include <type_traits>

#include "fq_codes.hpp"
#include "fq_device.hpp"
#include "fq_launch.hpp"

namespace fq {

// Stored composite rotation (Sec. III-C, the action expert's optional transform in place of
// the block Hadamard): gather by a channel permutation, then per-block orthogonal b x b
// matrices, as two kernels through an fp32 workspace z [M, K]:
//   rot_mfma_kernel: blocks of 16 channels and more, on the matrix cores (below);
//   rot_transform_kernel: blocks of 1 to 8 channels.  A workgroup takes one block and R rows.  The
//     block's matrix goes to LDS transposed, the rows' gathered, pre-multiplied inputs
//     w_j = x[perm[kb + j]] * s_inv[perm[kb + j]] transposed as well and XOR-swizzled so that the
//     transposing writes are free of bank conflicts.  Thread (g, h) owns TR rows times TI outputs
//     and, for j = 0..b-1 ascending, reads TI matrix entries and TR inputs and advances each output's
//     fma chain Q[i][j] * w_j from +0.  Then the optional fold-after multiplier;
//   rot_quant_kernel: one workgroup per row: row absmax, eq. (5) with c_b = 1 (the
//     blocks are orthonormal), canonical packing.
// Permutation entries are clamped into [0, K): a bad permutation gives wrong codes, never
// an out-of-bounds read.

template <int B, int TR>
struct RotShape {
  static constexpr int TI = B < 4 ? B : 4;  // outputs per thread
  static constexpr int NI = B / TI;         // output groups per block
  static constexpr int R = 256 / NI * TR;   // rows per workgroup
};

template <typename Tin, int B, int TR>
__global__ __launch_bounds__(256) void rot_transform_kernel(const void *x, int64_t ldx, const int32_t *perm,
                                                            const float *blocks, const float *chan_mult,
                                                            const float *post_mult, int64_t M, int K, float *z) {
  using S = RotShape<B, TR>;
  constexpr int TI = S::TI, R = S::R;
  // input swizzle mask; with four rows per thread it keeps each thread's rows one aligned
  // 16-byte group
  constexpr int VSW = ((R < 32 ? R : 32) - 1) & (TR == 4 ? ~3 : ~0);
  // qt[j * B + i] = Q[i][j], vt[j * R + (r ^ (j & VSW))] = w_j of row r
  __shared__ __attribute__((aligned(16))) float qt[B * B], vt[B * R];
  const int tid = threadIdx.x;
  const int kblk = blockIdx.x;
  const int64_t row0 = (int64_t)blockIdx.y * R;
  // Thread (rr, j) gathers channel perm[kb + j] for rows rr, rr + 256/b, ...: one permutation
  // entry and multiplier per thread.  Every load goes out before the first LDS write, so the
  // matrix's round trip overlaps the permutation's and the gather's.
  constexpr int JR = 256 / B, NV = R / JR;
  const int j = tid % B, rr = tid / B;
  int src = perm ? perm[kblk * B + j] : kblk * B + j;
  const float qv = tid < B * B ? blocks[(int64_t)kblk * B * B + tid] : 0.0f;
  src = min(max(src, 0), K - 1);
  const float cm = chan_mult ? chan_mult[src] : 1.0f;
  // rows past M load row M - 1 (no branch, so every load is in flight at once) and store 0
  using Raw = typename std::conditional<sizeof(Tin) == 2, uint16_t, float>::type;
  Raw raw[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int64_t row = min(row0 + rr + JR * k, M - 1);
    raw[k] = reinterpret_cast<const Raw *>(x)[row * ldx + src];
  }
  __builtin_amdgcn_sched_barrier(0);  // every load above issues before the first use below
  if (tid < B * B) qt[(tid % B) * B + tid / B] = qv;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const bool in = row0 + rr + JR * k < M;
    float v;
    if constexpr (sizeof(Tin) == 2)
      v = bf16_lo(raw[k]);
    else
      v = raw[k];
    vt[j * R + ((rr + JR * k) ^ (j & VSW))] = in ? (chan_mult ? v * cm : v) : 0.0f;
  }
  __syncthreads();
  const int h = tid % S::NI, r0 = tid / S::NI * TR;
  float acc[TR][TI];
#pragma unroll
  for (int t = 0; t < TR; ++t)
#pragma unroll
    for (int c = 0; c < TI; ++c) acc[t][c] = 0.0f;
#pragma unroll
  for (int jj = 0; jj < B; ++jj) {
    float q[TI], w[TR];
#pragma unroll
    for (int c = 0; c < TI; ++c) q[c] = qt[jj * B + TI * h + c];
#pragma unroll
    for (int t = 0; t < TR; ++t) w[t] = vt[jj * R + (TR == 4 ? (r0 ^ (jj & VSW)) + t : r0 ^ (jj & VSW))];
#pragma unroll
    for (int t = 0; t < TR; ++t)
#pragma unroll
      for (int c = 0; c < TI; ++c) acc[t][c] = __builtin_fmaf(q[c], w[t], acc[t][c]);
  }
  const int c_out = kblk * B + h * TI;
  float pm[TI];
#pragma unroll
  for (int c = 0; c < TI; ++c) pm[c] = post_mult ? post_mult[c_out + c] : 1.0f;
#pragma unroll
  for (int t = 0; t < TR; ++t) {
    const int64_t row = row0 + r0 + t;
    if (row < M) {
      float v[TI];
#pragma unroll
      for (int c = 0; c < TI; ++c) v[c] = post_mult ? acc[t][c] * pm[c] : acc[t][c];
      if constexpr (TI == 4) {
        *reinterpret_cast<float4 *>(z + row * K + c_out) = float4{v[0], v[1], v[2], v[3]};
      } else {
#pragma unroll
        for (int c = 0; c < TI; ++c) z[row * K + c_out + c] = v[c];
      }
    }
  }
}

typedef float v4f __attribute__((ext_vector_type(4)));

// The 4 x 4 transpose over the wave's quarters: register p of quarter h <- register h of quarter p.
__device__ __forceinline__ float4 transpose_quarters(float4 f) {
  const uint32_t x = __float_as_uint(f.x), y = __float_as_uint(f.y), z = __float_as_uint(f.z), w = __float_as_uint(f.w);
  const auto xz = __builtin_amdgcn_permlane32_swap(x, z, false, false);
  const auto yw = __builtin_amdgcn_permlane32_swap(y, w, false, false);
  const auto lo = __builtin_amdgcn_permlane16_swap(xz[0], yw[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(xz[1], yw[1], false, false);
  return float4{__uint_as_float(lo[0]), __uint_as_float(lo[1]), __uint_as_float(hi[0]), __uint_as_float(hi[1])};
}

// Blocks of 16 channels and more, on the fp32 matrix instruction.  v_mfma_f32_16x16x4_f32 advances
// each output by its four products in ascending k, every step a rounded fma (bit-equal to the fma
// chain over 800 000 outputs of 128 steps, with denormals, overflow and infinities among them), so
// chaining it over the block from +0 is the same per-output chain as above.  A workgroup takes 128
// channels (128 / B blocks) and 16 RT rows; a wave 32 outputs of all its rows.
//   A = the matrix rows straight from memory to registers: lane (h, i) loads Q[i][16 s + 4 h ..],
//       and a 4 x 4 transpose over the lane quarters (four lane swaps) leaves k = 16 s + 4 p + h
//       in register p, what instruction p of group s wants.
//   B = the rows' gathered, pre-multiplied inputs through LDS: lanes gather along the channels of
//       one row, so a row's lines are fetched once and hit for its other channels; a pitch of 132
//       words puts both the writes (along channels) and the reads (16 rows by 4 channels) on
//       distinct banks.
// A lane ends with 4 consecutive channels of one row: one 16-byte store.  The next tile's gather
// is in flight under the products.  M = 816, K = 2048, b = 128: 14.4 us, against 17.5 for the
// register-tiled fma chains this replaced (bound by their LDS reads of both operands); M = 16 6.2
// against 7.4; b = 16 9.0 against 13.5.  What is left is mostly the gather (every 2-byte input is a lane
// address of its own: with b = 16, an eighth of the products and of the matrix, the kernel still takes
// 9 us), then the products (3.4 us at the fp32 rate).
constexpr int kRotPitch = 132;

template <typename Tin, int B, int RT>
__global__ __launch_bounds__(256) void rot_mfma_kernel(const void *x, int64_t ldx, const int32_t *perm,
                                                       const float *blocks, const float *chan_mult,
                                                       const float *post_mult, int64_t M, int K, int64_t tiles, float *z) {
  constexpr int R = 16 * RT, NS = B / 16, NV = R / 2;
  __shared__ float vt[2][R * kRotPitch];  // vt[.][r * pitch + j] = w_j of row r
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lh = lane >> 4;
  const int c0 = blockIdx.x * 128;
  const int j = tid & 127, rr = tid >> 7;
  int src = perm ? perm[c0 + j] : c0 + j;
  // blocks is [K / B][B][B], so output channel o's matrix row starts at o * B
  float4 q[2][NS];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int s = 0; s < NS; ++s)
      q[u][s] = *reinterpret_cast<const float4 *>(blocks + (int64_t)(c0 + 32 * wave + 16 * u + li) * B + 16 * s + 4 * lh);
  src = min(max(src, 0), K - 1);
  const float cm = chan_mult ? chan_mult[src] : 1.0f;
  using Raw = typename std::conditional<sizeof(Tin) == 2, uint16_t, float>::type;
  const int c_out = c0 + 32 * wave + 4 * lh;
  Raw raw[NV];
  // rows past M load row M - 1 (no branch, so every load is in flight at once) and store 0
  auto gather = [&](int64_t t) {
#pragma unroll
    for (int k = 0; k < NV; ++k) raw[k] = reinterpret_cast<const Raw *>(x)[min(t * R + rr + 2 * k, M - 1) * ldx + src];
  };
  auto stage = [&](int64_t t, float *dst) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      float v;
      if constexpr (sizeof(Tin) == 2)
        v = bf16_lo(raw[k]);
      else
        v = raw[k];
      dst[(rr + 2 * k) * kRotPitch + j] = t * R + rr + 2 * k < M ? (chan_mult ? v * cm : v) : 0.0f;
    }
  };
  gather(blockIdx.y);
  __builtin_amdgcn_sched_barrier(0);  // every load above issues before the first use below
  stage(blockIdx.y, vt[0]);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int s = 0; s < NS; ++s) q[u][s] = transpose_quarters(q[u][s]);
  int buf = 0;
  for (int64_t t = blockIdx.y; t < tiles; t += gridDim.y, buf ^= 1) {
    const int64_t row0 = t * R, next = t + gridDim.y;
    __syncthreads();  // this tile is staged, and the other buffer has been read
    if (next < tiles) gather(next);
    __builtin_amdgcn_sched_barrier(0);  // in flight under the products
    v4f acc[2][RT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[u][r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const float *vr = vt[buf] + li * kRotPitch + lh;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int jb = (32 * wave + 16 * u) / B * B;  // the block's first channel among the 128
            const float a = p == 0 ? q[u][s].x : p == 1 ? q[u][s].y : p == 2 ? q[u][s].z : q[u][s].w;
            acc[u][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, vr[16 * r * kRotPitch + jb + 16 * s + 4 * p], acc[u][r], 0, 0, 0);
          }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float pm[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) pm[i] = post_mult ? post_mult[c_out + 16 * u + i] : 1.0f;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int64_t row = row0 + 16 * r + li;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = post_mult ? acc[u][r][i] * pm[i] : acc[u][r][i];
        if (row < M) *reinterpret_cast<float4 *>(z + row * K + c_out + 16 * u) = float4{v[0], v[1], v[2], v[3]};
      }
    }
    if (next < tiles) stage(next, vt[buf ^ 1]);
  }
}

// One workgroup per row; thread t owns 16-channel chunks t, t + 256, ... (K <= 32768).
template <int CPT>
__global__ __launch_bounds__(256) void rot_quant_kernel(const float *z, int64_t M, int K, int bits, float clip_ratio,
                                                        uint8_t *codes, int64_t ld_codes, float *delta, int out_fmt) {
  __shared__ float red[4];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const int nchunks = K >> 4;
  const float *zr = z + row * K;
  float v[CPT][16];
  float amax = 0.0f;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    // chunks past the row's end reread its last chunk (no branch, so every load is in
    // flight at once) and are left out of the maximum
    const int j = min(c * 256 + tid, nchunks - 1);
    const float4 *s4 = reinterpret_cast<const float4 *>(zr + j * 16);
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const float4 t = s4[q4];
      v[c][4 * q4] = t.x; v[c][4 * q4 + 1] = t.y; v[c][4 * q4 + 2] = t.z; v[c][4 * q4 + 3] = t.w;
    }
  }
#pragma unroll
  for (int c = 0; c < CPT; ++c)
    if (c * 256 + tid < nchunks)
#pragma unroll
      for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(v[c][e]));
  amax = fmaxf(amax, lane_xor<1>(amax));
  amax = fmaxf(amax, lane_xor<2>(amax));
  amax = fmaxf(amax, lane_xor<4>(amax));
  amax = fmaxf(amax, lane_xor<8>(amax));
  amax = fmaxf(amax, lane_xor<16>(amax));
  amax = fmaxf(amax, __shfl_xor(amax, 32, kWave));
  if ((tid & 63) == 0) red[tid >> 6] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const int q = (1 << (bits - 1)) - 1;
  const float qf = (float)q;
  const bool zero = !(amax > 0.0f);
  const float rA = clip_ratio * amax;
  const float inv = zero ? 0.0f : qf / rA;
  if (tid == 0) delta[row] = zero ? 0.0f : (rA * 1.0f) / qf;
  uint8_t *row_out = codes + row * ld_codes;
  const float lim = qf + 0.49f;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int j = c * 256 + tid;
    if (j < nchunks) {
      int cc[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) cc[e] = quantize_bits(v[c][e], inv, lim);
      store_chunk_bits(row_out, j, cc, out_fmt);
    }
  }
}

template <typename Tin, int B, int TR>
static hipError_t launch_rot_tr(const void *x, int64_t ldx, const int32_t *perm, const float *blocks,
                                const float *chan_mult, const float *post_mult, int64_t M, int K, float *z,
                                hipStream_t s) {
  constexpr int R = RotShape<B, TR>::R;
  const int64_t gy = (M + R - 1) / R;
  if (gy > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL((rot_transform_kernel<Tin, B, TR>), dim3((unsigned)(K / B), (unsigned)gy), dim3(256), 0, s,
                     x, ldx, perm, blocks, chan_mult, post_mult, M, K, z);
  return hipGetLastError();
}

// Blocks of 1 to 8 channels: four rows per thread when that still gives a grid of at least one
// workgroup per compute unit, else one (small M: more workgroups).
template <typename Tin, int B>
static hipError_t launch_rot_b(const void *x, int64_t ldx, const int32_t *perm, const float *blocks,
                               const float *chan_mult, const float *post_mult, int64_t M, int K, float *z,
                               hipStream_t s) {
  constexpr int R = RotShape<B, 4>::R;
  return (K / B) * ((M + R - 1) / R) >= 256
             ? launch_rot_tr<Tin, B, 4>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s)
             : launch_rot_tr<Tin, B, 1>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
}

template <typename Tin, int B, int RT>
static hipError_t launch_rot_rt(const void *x, int64_t ldx, const int32_t *perm, const float *blocks,
                                const float *chan_mult, const float *post_mult, int64_t M, int K, float *z,
                                hipStream_t s) {
  const int64_t tiles = (M + 16 * RT - 1) / (16 * RT);
  const int64_t most = K / 128 < 512 ? 512 / (K / 128) : 1;
  hipLaunchKernelGGL((rot_mfma_kernel<Tin, B, RT>), dim3((unsigned)(K / 128), (unsigned)(RT == 1 || tiles < most ? tiles : most)),
                     dim3(256), 0, s, x, ldx, perm, blocks, chan_mult, post_mult, M, K, tiles, z);
  return hipGetLastError();
}

// 32 rows at a time, in at most two workgroups per compute unit that walk over the rows (each
// matrix row is loaded once a workgroup), when the grid of such tiles is well over one per
// compute unit; else 16 rows, one tile per workgroup.  At the line, b = 64: 352 tiles of 32 rows
// (M 333, K 4096) 12.6 us against 10.3 in tiles of 16; 416 (M 816, K 2048) 11.7 against 12.0, and
// 14.4 against 16.0 at b = 128.
template <typename Tin, int B>
static hipError_t launch_rot_m(const void *x, int64_t ldx, const int32_t *perm, const float *blocks,
                               const float *chan_mult, const float *post_mult, int64_t M, int K, float *z,
                               hipStream_t s) {
  if ((M + 4096 / B - 1) / (4096 / B) > 65535) return hipErrorInvalidValue;  // the range this entry takes
  return (K / 128) * ((M + 31) / 32) > 384 ? launch_rot_rt<Tin, B, 2>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s)
                                           : launch_rot_rt<Tin, B, 1>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
}

template <typename Tin>
static hipError_t launch_rot_t(const void *x, int64_t ldx, const int32_t *perm, const float *blocks,
                               const float *chan_mult, const float *post_mult, int64_t M, int K, int b,
                               float *z, hipStream_t s) {
  switch (b) {
    case 1: return launch_rot_b<Tin, 1>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 2: return launch_rot_b<Tin, 2>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 4: return launch_rot_b<Tin, 4>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 8: return launch_rot_b<Tin, 8>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 16: return launch_rot_m<Tin, 16>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 32: return launch_rot_m<Tin, 32>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 64: return launch_rot_m<Tin, 64>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    case 128: return launch_rot_m<Tin, 128>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, z, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rotate_quant(const void *x, bool x_is_f32, int64_t ldx, const int32_t *perm,
                               const float *blocks, const float *chan_mult, const float *post_mult,
                               int64_t M, int K, int b, int bits, float clip_ratio, uint8_t *codes,
                               int64_t ld_codes, float *delta, int out_fmt, float *z, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (K > 256 * 8 * 16 || M > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipError_t e = x_is_f32 ? launch_rot_t<float>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, b, z, s)
                          : launch_rot_t<uint16_t>(x, ldx, perm, blocks, chan_mult, post_mult, M, K, b, z, s);
  if (e != hipSuccess) return e;
  // chunks per thread: the fewest that cover the row (no thread rereads a chunk it does not own)
  const int nch = K / 16;
  if (nch <= 256)
    hipLaunchKernelGGL(rot_quant_kernel<1>, dim3((unsigned)M), dim3(256), 0, s, z, M, K, bits, clip_ratio, codes,
                       ld_codes, delta, out_fmt);
  else if (nch <= 512)
    hipLaunchKernelGGL(rot_quant_kernel<2>, dim3((unsigned)M), dim3(256), 0, s, z, M, K, bits, clip_ratio, codes,
                       ld_codes, delta, out_fmt);
  else if (nch <= 1024)
    hipLaunchKernelGGL(rot_quant_kernel<4>, dim3((unsigned)M), dim3(256), 0, s, z, M, K, bits, clip_ratio, codes,
                       ld_codes, delta, out_fmt);
  else
    hipLaunchKernelGGL(rot_quant_kernel<8>, dim3((unsigned)M), dim3(256), 0, s, z, M, K, bits, clip_ratio, codes,
                       ld_codes, delta, out_fmt);
  return hipGetLastError();
}

}  // namespace fq
