// Tiled INT4 GEMM for a few hundred to ~1000 tokens at long K (eq. (8) contraction and
// rescale), where larger output tiles would leave most compute units idle unless K is
// split across workgroups (and a second kernel adds the slices).
//
// Workgroup: 4 waves, one 128 x 64 output tile (4 x 2 tiles of 32 x 32); wave w owns the
// k steps w, w + 4, w + 8, ... of the whole of K, so the tile needs no split of K across
// workgroups and its four partial sums add up through LDS at the end (exact integers).
// Every wave streams its own operands straight from L2 into registers, three register sets
// deep, with buffer loads: one SGPR descriptor per operand, a fixed per-lane offset and a
// per-step scalar offset, so the loop carries no address arithmetic.  No operand goes through LDS.
// The products run on the FP6 matrix cores (fq_f6.hpp).  One wave per SIMD: the issue of the widening
// (128 operations a step, 144 on INT8 operands) and of the multiplies (28 against 64 instructions)
// bounds it.  M = 816, K 16384 -> N 2048: 27.7 us against 30.4 on INT8 operands; but 32.5 against 30.2
// at M = 896, the same grid without repeated rows in the last row tile.
#include "fq_device.hpp"
#include "fq_f6.hpp"
#include "fq_launch.hpp"

namespace fq {

namespace {

constexpr int kKgTI = 4;    // 32-row tiles per workgroup tile
constexpr int kKgTJ = 2;    // 32-column tiles per workgroup tile
constexpr int kKgWaves = 4; // k groups
constexpr int kKgSets = 3;  // operand register sets: loads run two k steps ahead
constexpr int kKgRows = 32 * kKgTI, kKgCols = 32 * kKgTJ;
constexpr size_t kKgPartLds = (size_t)kKgWaves * kKgTI * kKgTJ * 4096;  // the k groups' sums
constexpr int kKgOutStride = kKgCols * 2 + 16;                           // bf16 staging row, padded
constexpr size_t kKgSumOff = kKgPartLds + (size_t)kKgRows * kKgOutStride;
constexpr size_t kKgLds = kKgSumOff + (size_t)kKgWaves * (kKgRows + kKgCols) * 4;

__global__ __launch_bounds__(64 * kKgWaves) void gemm_kgroup_kernel(KgParams p) {
  constexpr int TI = kKgTI, TJ = kKgTJ, KG = kKgWaves, NB = TI * TJ;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntn = (p.N + kKgCols - 1) / kKgCols;
  const int tn = blockIdx.x % ntn, tm = blockIdx.x / ntn;
  const int m0 = tm * kKgRows, n0 = tn * kKgCols;
  const int ktot = p.K / kTileK;
  const uint32_t astep = (uint32_t)p.M * 64u;  // bytes of one k step of the codes
  const int u = lane >> 5, cl = lane & 31;

  // rows: 32-row blocks of the k-major codes, half h of a step at + 32 h
  uint32_t aoff[TI];
#pragma unroll
  for (int i = 0; i < TI; ++i) aoff[i] = row_offset(m0 + 32 * i, p.M, lane);
  // columns: lane l takes column l % 32 of a 32-column block and the k group 2 h + l / 32, 16
  // bytes of weight tile (column / 16) at lane 16 (2 h + l / 32) + column % 16 (tiles past N
  // re-read the last one, never stored)
  uint32_t boff[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
    boff[j] = (uint32_t)min(n0 / 16 + 2 * j + (cl >> 4), p.N / 16 - 1) * (uint32_t)ktot * 1024u +
              (uint32_t)(u * 16 + (cl & 15)) * 16u;
  const __amdgpu_buffer_rsrc_t arsrc = buffer_of(p.a, (int64_t)ktot * astep);
  const __amdgpu_buffer_rsrc_t brsrc = buffer_of(p.w, (int64_t)(p.N / 16) * ktot * 1024);

  v16f acc[TI][TJ];
  v4f rs[TI], cs[TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    rs[i] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  }
#pragma unroll
  for (int j = 0; j < TJ; ++j) cs[j] = v4f{0.f, 0.f, 0.f, 0.f};
  const v8i pat = f6_row_pattern(lane);
  constexpr int NSET = kKgSets;
  v4i ra[NSET][2][TI], rb[NSET][2][TJ];
  // the two halves of a row's 64 bytes by adjacent loads: they share cache lines, and with the other
  // blocks' loads between them the lines were fetched again (M = 896, K 16384 -> N 2048: 32.5 us
  // against 35.6)
  auto load = [&](v4i (&ra_)[2][TI], v4i (&rb_)[2][TJ], int ks) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) ra_[h][i] = __builtin_amdgcn_raw_buffer_load_b128(arsrc, aoff[i] + h * 32u, ks * astep, 0);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) rb_[h][j] = __builtin_amdgcn_raw_buffer_load_b128(brsrc, boff[j] + h * 512u, ks * 1024u, 0);
  };
  auto compute = [&](const v4i (&ra_)[2][TI], const v4i (&rb_)[2][TJ]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v8i fb[TJ];
#pragma unroll
      for (int j = 0; j < TJ; ++j) fb[j] = spread32(rb_[h][j]);
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const v8i fa = expand32(ra_[h][i]);
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = mfma_f6_32(fa, fb[j], acc[i][j]);
        rs[i] = mfma_f6_16(fa, pat, rs[i]);
      }
#pragma unroll
      for (int j = 0; j < TJ; ++j) cs[j] = mfma_f6_16(pat, fb[j], cs[j]);
    }
  };
  // NSET steps per loop trip, one per register set, each set's loads issued NSET - 1 steps
  // before its multiplies (the scheduling walls keep the compiler from sinking them); the
  // last nk mod NSET steps after the loop, so the accumulators flow through a single path
  // (a conditional trip end made the compiler copy them between AGPR sets every trip).  A
  // load past the wave's last step re-reads step K/128 - 1 (in bounds, never multiplied).
  const int nk = ktot > wave ? (ktot - wave + KG - 1) / KG : 0;
  const int klast = ktot - 1;
  int ks = wave;
#pragma unroll
  for (int q = 0; q < NSET - 1; ++q) load(ra[q], rb[q], min(ks + q * KG, klast));
  int t = 0;
  for (; t + NSET - 1 < nk; t += NSET) {
#pragma unroll
    for (int q = 0; q < NSET; ++q) {
      load(ra[(q + NSET - 1) % NSET], rb[(q + NSET - 1) % NSET], min(ks + (q + NSET - 1) * KG, klast));
      __builtin_amdgcn_sched_barrier(0);
      compute(ra[q], rb[q]);
      __builtin_amdgcn_sched_barrier(0);
    }
    ks += NSET * KG;
  }
#pragma unroll
  for (int q = 0; q < NSET - 1; ++q)
    if (t + q < nk) compute(ra[q], rb[q]);

  // ---- the k groups' sums: every wave leaves its 8 tiles (lane-major) and its sums of codes in
  // LDS, then wave w adds up and rescales row block w of all four ----
  v4f *part = reinterpret_cast<v4f *>(lds);
  int *rsum = reinterpret_cast<int *>(lds + kKgSumOff), *csum = rsum + KG * kKgRows;
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        part[((wave * NB + i * TJ + j) * 4 + e4) * 64 + lane] =
            v4f{acc[i][j][4 * e4], acc[i][j][4 * e4 + 1], acc[i][j][4 * e4 + 2], acc[i][j][4 * e4 + 3]};
  if ((lane & 15) < 2)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        rsum[wave * kKgRows + 32 * i + (lane & 1) * 16 + 4 * (lane >> 4) + r] = (int)(rs[i][r] * 8.0f);
  if (lane < 16)
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      csum[wave * kKgCols + 32 * j + lane] = (int)(cs[j][0] * 8.0f);
      csum[wave * kKgCols + 32 * j + 16 + lane] = (int)(cs[j][1] * 8.0f);
    }
  __syncthreads();
  static_assert(TI == KG, "one row block per wave in the final sum");
  uint8_t *out = lds + kKgPartLds;
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int col = 32 * j + cl, n = n0 + col, nc = min(n, p.N - 1);
    const float sw = p.w_scale[nc];
    const float bj = p.bias ? p.bias[nc] : 0.0f;
    int cc = 64 * p.K;
#pragma unroll
    for (int q = 0; q < KG; ++q) cc -= 8 * csum[q * kKgCols + col];
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      v4f s = part[((wave * TJ + j) * 4 + e4) * 64 + lane];
#pragma unroll
      for (int q = 1; q < KG; ++q) s += part[((q * NB + wave * TJ + j) * 4 + e4) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 32 * wave + 8 * e4 + 4 * u + e, m = m0 + row;
        int r = 0;
#pragma unroll
        for (int q = 0; q < KG; ++q) r += rsum[q * kKgRows + row];
        const int sum = (int)(s[e] * 64.0f) + cc - 8 * r;
        if (p.acc_out && m < p.M && n < p.N) p.acc_out[(int64_t)m * p.N + n] = sum;
        // rows past M read row M - 1's delta, never stored
        const float v = (float)sum * (sw * p.delta[min(m, p.M - 1)]) + bj;
        *reinterpret_cast<uint16_t *>(out + row * kKgOutStride + col * 2) = (uint16_t)f32_to_bf16(v);
      }
    }
  }
  // bf16 rows staged in LDS (after the partial sums) so that the tile leaves in 16-byte row chunks
  __syncthreads();
  constexpr int CPR = kKgCols / 8;  // 16-byte chunks per staged row
  for (int q = threadIdx.x; q < kKgRows * CPR; q += 64 * KG) {
    const int row = q / CPR, ch = q % CPR;
    const int m = m0 + row, nn = n0 + ch * 8;
    if (m < p.M && nn < p.N)
      *reinterpret_cast<uint4 *>(p.y + (int64_t)m * p.ldy + nn) = *reinterpret_cast<const uint4 *>(out + row * kKgOutStride + ch * 16);
  }
}

// Canonical nibble codes [M][K/2] -> the prologue's arrangement, k major, 16 bytes per thread.
// Thread u takes 16-byte chunk c = 16 kq + u % 16 of row r = (u / 16) % M, kq = u / (16 M):
// a wave reads 4 rows x 256 contiguous bytes (whole cache lines) and writes, for each of
// the 4 k steps those bytes hold, 4 consecutive rows x 64 bytes (256 contiguous bytes).
__global__ __launch_bounds__(256) void codes_major_kernel(const uint8_t *__restrict__ src, uint8_t *__restrict__ dst,
                                                          int M, int K) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int cpr = K / 32;  // 16-byte chunks per row (4 per k step)
  const int64_t rowunits = (int64_t)M * 16;
  const int kq = (int)(u / rowunits);
  const int rem = (int)(u - (int64_t)kq * rowunits);
  const int r = rem >> 4;
  const int c = 16 * kq + (rem & 15);
  if (c >= cpr) return;
  const uint4 x = *reinterpret_cast<const uint4 *>(src + (int64_t)r * (K / 2) + (int64_t)c * 16);
  const uint2 lo = rearrange16(x.x, x.y), hi = rearrange16(x.z, x.w);
  *reinterpret_cast<uint4 *>(dst + major_chunk(r, M, c)) = make_uint4(lo.x, lo.y, hi.x, hi.y);
}

}  // namespace

hipError_t launch_gemm_kgroup(const KgParams &p, const uint8_t *a_canonical, uint8_t *a_major, hipStream_t s,
                              bool go) {
  static std::atomic<uint64_t> attr{0};
  hipError_t e = allow_dynamic_lds(&gemm_kgroup_kernel, kKgLds, attr);
  if (e != hipSuccess || !go) return e;
  if (a_canonical) {
    const int64_t units = (int64_t)((p.K / 32 + 15) / 16) * p.M * 16;  // 16-chunk row groups, rounded up
    hipLaunchKernelGGL(codes_major_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s, a_canonical,
                       a_major, p.M, p.K);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int64_t tiles = ((int64_t)(p.M + kKgRows - 1) / kKgRows) * ((p.N + kKgCols - 1) / kKgCols);
  hipLaunchKernelGGL(gemm_kgroup_kernel, dim3((unsigned)tiles), dim3(64 * kKgWaves), kKgLds, s, p);
  return hipGetLastError();
}

}  // namespace fq
