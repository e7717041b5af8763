// Wide-tile GEMMs for many rows (eq. (8) contraction and rescale): one workgroup per compute unit
// owns a 256 x 128 output tile on 32 x 32 matrix instructions.
//
// What bounds them: the 128 x 128 LDS-ring kernel moves 64 operand bytes per clock and compute
// unit from L2 at W8A8's rate (a compute unit takes 52-58) and, for W4A4, issues 3 widening
// operations per multiply.  These tiles move 3/4 of the bytes, W4A4 multiplies on the FP6 matrix
// cores (fq_f6.hpp: twice the INT8 rate, and 2.5x fewer widening operations per product), and 32 x
// 32 instructions leave twice the issue slots between multiplies.  At full occupancy power
// bounds W8A8: at M = 4096, K 16384 -> N 2048 the clock is at most 1.8 GHz with the matrix pipe 60%
// busy.  W4A4 runs there at up to 2.2 GHz with the pipe 48% busy (counters under profiles/).
#include "fq_device.hpp"
#include "fq_f6.hpp"
#include "fq_launch.hpp"

namespace fq {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kBN = 128;  // columns of an output tile (256 rows)

// 16 bytes per lane from a buffer straight into LDS (lane l -> dst + 16 l).
__device__ __forceinline__ void buffer_to_lds16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, void *dst) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, voff, soff, 0, 0);
#else
  (void)r; (void)voff; (void)soff; (void)dst;
#endif
}

// Tile (tm, tn) of a workgroup.  The hardware hands workgroup p to XCD p % 8;
// consecutive logical ids go to one XCD, and ids run down kGroup row tiles before the next
// column tile, so the tiles an XCD works on at a time form a near-square block whose rows and
// columns its L2 serves repeatedly.
constexpr int kGroup = 4;
__device__ __forceinline__ void tile_of(int lin, int total, int ntm, int ntn, int &tm, int &tn) {
  const int x = lin & 7, q = total >> 3, r = total & 7;
  const int id = x * q + min(x, r) + (lin >> 3);
  const int grp = id / (kGroup * ntn);
  const int inner = id - grp * kGroup * ntn;
  const int gm = min(kGroup, ntm - grp * kGroup);
  tn = inner / gm;
  tm = grp * kGroup + (inner - tn * gm);
}

// A wave's 32 TI x 32 TJ part (rows rw, columns cw of the workgroup's tile) of the output.  Lane
// l holds column l % 32 and rows 8 (e / 4) + 4 (l / 32) + e % 4 of each 32 x 32 tile; `sums`
// gives the exact integer sum of (i, j, e).  The wave rescales, stages its bf16 rows in its own
// part of LDS and stores them in 16-byte chunks.  ACC: raw accumulators on request (the INT8 GEMM
// entry point; INT4 comes here only from the fused projection, which has none).
template <int TI, int TJ, bool ACC, typename F>
__device__ __forceinline__ void write_out(const WideParams &p, F sums, uint8_t *lds, const float *sdelta, int wave,
                                          int rw, int cw, int m0, int n0) {
  constexpr int STRIDE = 32 * TJ * 2 + 16;
  const int lane = threadIdx.x & 63;
  const int u = lane >> 5, cl = lane & 31;
  if (ACC && p.acc_out) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = m0 + rw + 32 * i + 8 * (e >> 2) + 4 * u + (e & 3), n = n0 + cw + 32 * j + cl;
          if (m < p.M && n < p.N) p.acc_out[(int64_t)m * p.N + n] = sums(i, j, e);
        }
  }
  uint8_t *out = lds + wave * 32 * TI * STRIDE;
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int n = min(n0 + cw + 32 * j + cl, p.N - 1);
    const float sw = p.w_scale[n];
    const float bj = p.bias ? p.bias[n] : 0.0f;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int row = 32 * i + 8 * e4 + 4 * u;
        const float4 dt = *reinterpret_cast<const float4 *>(sdelta + rw + row);
        const float d[4] = {dt.x, dt.y, dt.z, dt.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = (float)sums(i, j, 4 * e4 + e) * (sw * d[e]) + bj;
          *reinterpret_cast<uint16_t *>(out + (row + e) * STRIDE + (32 * j + cl) * 2) = (uint16_t)f32_to_bf16(v);
        }
      }
  }
  wave_lds_fence();  // lanes read what others wrote, in the wave's own part only
  constexpr int CPR = 32 * TJ / 8;
#pragma unroll
  for (int q = 0; q < 32 * TI * CPR / 64; ++q) {
    const int c = q * 64 + lane, row = c / CPR, ch = c % CPR;
    const int m = m0 + rw + row, n = n0 + cw + ch * 8;
    if (m < p.M && n < p.N)
      *reinterpret_cast<uint4 *>(p.y + (int64_t)m * p.ldy + n) =
          *reinterpret_cast<const uint4 *>(out + row * STRIDE + ch * 16);
  }
}


// ---------------- INT8 ----------------
// 4 x 1 waves of 64 x 128 (one per SIMD, 128 accumulators each), canonical codes.  Both operands go
// through a ring of k steps in LDS.  M = 4096, K 16384 -> N 2048: 123 us against 155 on the
// 128 x 128 tiles (2.2 against 1.8 POPS).  Measured and not kept: 8 waves of 64 x 64 (128-135 us,
// twice the LDS reads), rows straight into registers from a k-major copy written by the prologue
// (113 us, but the scattered 16-byte stores cost the prologue 14 us).
constexpr int k8Waves = 4, k8BM = 256, k8Stages = 3;
constexpr int k8A = k8BM * 128, k8W = kBN / 16 * 2048, k8Stage = k8A + k8W;  // bytes per k step
constexpr size_t k8Lds = (size_t)k8Stages * k8Stage + k8BM * 4;

__global__ __launch_bounds__(64 * k8Waves) void gemm_wide8_kernel(WideParams p) {
  constexpr int TI = 2, TJ = 4;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  float *sdelta = reinterpret_cast<float *>(lds + (size_t)k8Stages * k8Stage);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntm = (p.M + k8BM - 1) / k8BM, ntn = (p.N + kBN - 1) / kBN;
  int tm, tn;
  tile_of(blockIdx.x, gridDim.x, ntm, ntn, tm, tn);
  const int m0 = tm * k8BM, n0 = tn * kBN;
  const int ktot = p.K / kTileK;
  sdelta[tid] = p.delta[min(m0 + tid, p.M - 1)];

  // ring loads of one k step: wave w fills KBs [8 w, 8 w + 8) of the rows (8 rows x 128 bytes
  // each, 16-byte chunks XOR-swizzled by (row >> 1) & 7) and [4 w, 4 w + 4) of the weights (a
  // tile's chunk c at c ^ ((c >> 4) & 1): a wave reads every second chunk)
  constexpr int IA = k8A / 1024 / k8Waves, IB = k8W / 1024 / k8Waves, LPS = IA + IB;
  uint32_t avoff[IA], bvoff[IB];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int row = (wave * IA + i) * 8 + (lane >> 3);
    avoff[i] = (uint32_t)min(m0 + row, p.M - 1) * (uint32_t)p.K + ((lane & 7) ^ ((row >> 1) & 7)) * 16u;
  }
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int kb = wave * IB + i;
    bvoff[i] = (uint32_t)min(n0 / 16 + kb / 2, p.N / 16 - 1) * (uint32_t)ktot * 2048u + (kb & 1) * 1024u +
               (lane ^ ((lane >> 4) & 1)) * 16u;
  }
  const __amdgpu_buffer_rsrc_t ar = buffer_of(p.a, (int64_t)p.M * p.K);
  const __amdgpu_buffer_rsrc_t br = buffer_of(p.w, (int64_t)p.N * p.K);
  // load q of step ks (clamped to the last step: past it only slots that are never read fill)
  auto issue = [&](int ks, int slot, int q) {
    const uint32_t kc = (uint32_t)min(ks, ktot - 1);
    uint8_t *st = lds + slot * k8Stage;
    if (q < IA) buffer_to_lds16(ar, avoff[q], kc * 128u, st + (wave * IA + q) * 1024);
    else buffer_to_lds16(br, bvoff[q - IA], kc * 2048u, st + k8A + (wave * IB + q - IA) * 1024);
  };

  // operands of chunk q (32 channels): lane l takes row (or column) l % 32 and the 16 channels
  // 32 q + 16 (l / 32) + [0, 16)
  const int u = lane >> 5, r32 = lane & 31;
  const int abase = (wave * 64 + r32) * 128 + ((u ^ ((r32 >> 1) & 7)) * 16);
  const int bbase = k8A + (r32 >> 4) * 2048 + (((r32 & 15) * 2 + u) ^ ((r32 >> 3) & 1)) * 16;
  v4i ra[2][TI], rb[2][TJ];
  constexpr int NRD = TI + TJ;
  auto read = [&](int set, int slot, int q, int r) {  // in the order the multiplies want them
    const uint8_t *st = lds + slot * k8Stage;
    if (r == 0) rb[set][0] = *reinterpret_cast<const v4i *>(st + bbase + q * 512);
    else if (r <= TI) ra[set][r - 1] = *reinterpret_cast<const v4i *>(st + (abase ^ (q * 32)) + (r - 1) * 4096);
    else rb[set][r - TI] = *reinterpret_cast<const v4i *>(st + bbase + q * 512 + (r - TI) * 4096);
  };

  v16i acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

#pragma unroll
  for (int q = 0; q < LPS; ++q) issue(0, 0, q);
#pragma unroll
  for (int q = 0; q < LPS; ++q) issue(1, 1, q);
  wait_vmcnt<LPS>();
  lds_barrier();
#pragma unroll
  for (int r = 0; r < NRD; ++r) read(0, 0, 0, r);
#pragma unroll
  for (int q = 0; q < LPS / 2; ++q) issue(2, 2, q);

  int slot = 0;
  for (int ks = 0; ks < ktot; ++ks) {
    const int next = slot == k8Stages - 1 ? 0 : slot + 1;
    const int prev = slot == 0 ? k8Stages - 1 : slot - 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cur = q & 1;
      int r = 0, g = 0;
#pragma unroll
      for (int t = 0; t < TI * TJ; ++t) {
        const int i = t % TI, j = t / TI;
        __builtin_amdgcn_sched_barrier(0);
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ra[cur][i], rb[cur][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (q == 3 && t == 1) {
          // every read of this step's slot is done; the next step's loads have landed (step
          // ks + 2's are the LPS later ones)
          wait_vmcnt<LPS>();
          lds_barrier();
        }
        if (q < 3 || t >= 1) {
          // the next chunk's operands, two reads per multiply
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (r < NRD) {
              read(cur ^ 1, q == 3 ? next : slot, (q + 1) & 3, r);
              ++r;
            }
        }
        // step ks + 2's second half in chunk 0, step ks + 3's first half after the barrier
        if (q == 0 && g < LPS / 2) {
          issue(ks + 2, prev, LPS / 2 + g);
          ++g;
        }
        if (q == 3 && t >= 1 && g < LPS / 2) {
          issue(ks + 3, slot, g);
          ++g;
        }
      }
    }
    slot = next;
  }
  wait_vmcnt<0>();
  __syncthreads();  // the ring's trailing loads and reads are over: LDS is reused
  auto sums = [&](int i, int j, int e) -> int { return acc[i][j][e]; };
  write_out<TI, TJ, true>(p, sums, lds, sdelta, wave, wave * 64, 0, m0, n0);
}

// ---------------- INT4 on the FP6 matrix cores ----------------
// 8 x 1 waves (two per SIMD) of 32 x 128, k-major codes (kAF6Major).  A wave's 32 rows go straight
// into registers, four k steps ahead, and expand with 4 operations per 16 codes; each wave
// widens one of the 8 column tiles of a step (8 operations per 16 codes) into LDS, where all
// read it a step later.  M = 4096, K 16384 -> N 2048: 86 us against 127 on the 128 x 128 LDS-ring
// kernel (3.2 against 2.1 POPS); the multiplies alone take 55 us there.  Measured and not kept:
// four waves of 64 x 128 (117 us: one wave per SIMD issues 290 instructions a step at ~5 cycles
// each), rows through LDS (104 us), two workgroups of 128 rows per compute unit (113 us).
constexpr int k4Waves = 8, k4BM = 32 * k4Waves;
constexpr int k4W = kBN * 96;                              // widened weights of one k step, four in LDS
constexpr size_t k4Tail = (size_t)k4BM * (kBN * 2 + 16);   // the staged output is the larger use
static_assert(k4Tail >= 4 * (size_t)k4W, "LDS layout");
constexpr size_t k4Lds = k4Tail + k4BM * 8 + kBN * 4;      // + delta, row sums, column sums

__global__ __launch_bounds__(64 * k4Waves) void gemm_wide4_kernel(WideParams p) {
  constexpr int TJ = 4;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  float *sdelta = reinterpret_cast<float *>(lds + k4Tail);
  int *rsum = reinterpret_cast<int *>(lds + k4Tail + k4BM * 4);
  int *csum = rsum + k4BM;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntm = (p.M + k4BM - 1) / k4BM, ntn = (p.N + kBN - 1) / kBN;
  int tm, tn;
  tile_of(blockIdx.x, gridDim.x, ntm, ntn, tm, tn);
  const int m0 = tm * k4BM, n0 = tn * kBN;
  const int ktot = p.K / kTileK;
  if (tid < k4BM) sdelta[tid] = p.delta[min(m0 + tid, p.M - 1)];

  auto clamp_step = [&](int ks) -> uint32_t { return (uint32_t)min(ks, ktot - 1); };
  // activations: the wave's 32 rows straight into registers, one load per half step
  const __amdgpu_buffer_rsrc_t ar = buffer_of(p.a, (int64_t)p.M * (p.K / 2));
  const uint32_t aoff = row_offset(m0 + wave * 32, p.M, lane);
  auto load_a = [&](int ks, int h) -> v4i {
    return __builtin_amdgcn_raw_buffer_load_b128(ar, aoff + h * 32u, clamp_step(ks) * (uint32_t)p.M * 64u, 0);
  };
  // weights: wave w widens column tile w
  const __amdgpu_buffer_rsrc_t br = buffer_of(p.w, (int64_t)p.N * (p.K / 2));
  const uint32_t bvoff = (uint32_t)min(n0 / 16 + wave, p.N / 16 - 1) * (uint32_t)ktot * 1024u + lane * 16u;
  auto load_w = [&](int ks) -> v4i { return __builtin_amdgcn_raw_buffer_load_b128(br, bvoff, clamp_step(ks) * 1024u, 0); };
  const int u = lane >> 5, r32 = lane & 31;
  // lane (n = l % 16, g = l / 16) of column tile t holds k group g of column 16 t + n: lane
  // 32 (g % 2) + 16 (t % 2) + n of the operand of half g / 2, column block t / 2
  const int wslot = (wave >> 1) * 128 + (lane >> 5) * 64 + ((lane >> 4) & 1) * 32 + (wave & 1) * 16 + (lane & 15);
  v8i wf;  // the column tile of the current step, for the columns' sums
  auto put_w = [&](const v4i &raw, int buf) {
    wf = spread32(raw);
    uint8_t *b = lds + buf * k4W;
    *reinterpret_cast<v4i *>(b + wslot * 16) = v4i{wf[0], wf[1], wf[2], wf[3]};
    *reinterpret_cast<v2i *>(b + 8192 + wslot * 8) = v2i{wf[4], wf[5]};
  };
  auto operand = [&](int slot_, int buf) -> v8i {
    const uint8_t *b = lds + buf * k4W;
    const int s = slot_ * 64 + lane;
    const v4i a = *reinterpret_cast<const v4i *>(b + s * 16);
    const v2i c = *reinterpret_cast<const v2i *>(b + 8192 + s * 8);
    return v8i{a.x, a.y, a.z, a.w, c.x, c.y, 0, 0};
  };
  v8i bq[2][TJ];  // one set per half: each is read while the other is multiplied
  v8i fa[2];
  v16f acc[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
  const v8i ones = f6_ones(), pat = f6_row_pattern(lane);
  v4f rs = v4f{0.f, 0.f, 0.f, 0.f}, cs = v4f{0.f, 0.f, 0.f, 0.f};
  auto mul = [&](int h, int j) {
    acc[j] = mfma_f6_32(fa[h], bq[h][j], acc[j]);
  };

  // In flight before the loop: the rows of steps 0 .. 3 and the weights of steps 0 .. 4
  v4i wr[4], arw[4][2];
  const v4i w0 = load_w(0);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int h = 0; h < 2; ++h) arw[t][h] = load_a(t, h);
    wr[(t + 1) & 3] = load_w(t + 1);
  }
  __builtin_amdgcn_sched_barrier(0);
  put_w(w0, 0);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TJ; ++j) bq[0][j] = operand(j * 2, 0);
  fa[0] = expand32(arw[0][0]);

  auto step = [&](auto par, int ks) {
    constexpr int P = decltype(par)::value, Q = (P + 1) % 4;
    // the widened weights of step ks + 1, while half 0 is multiplied
    __builtin_amdgcn_sched_barrier(0);
    mul(0, 0);
    cs = mfma_f6_16(ones, wf, cs);
    mul(0, 1);
    put_w(wr[Q], Q);
    wr[Q] = load_w(ks + 5);
#pragma unroll
    for (int j = 0; j < 2; ++j) bq[1][j] = operand(j * 2 + 1, P);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, 6, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the rest of half 0; the rows of half 1
    mul(0, 2);
    mul(0, 3);
    rs = mfma_f6_16(fa[0], pat, rs);
#pragma unroll
    for (int j = 2; j < TJ; ++j) bq[1][j] = operand(j * 2 + 1, P);
    fa[1] = expand32(arw[P][1]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // half 1; the next step's first operands
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      mul(1, j);
      bq[0][j] = operand(j * 2, Q);
    }
    rs = mfma_f6_16(fa[1], pat, rs);
    fa[0] = expand32(arw[Q][0]);
#pragma unroll
    for (int h = 0; h < 2; ++h) arw[P][h] = load_a(ks + 4, h);
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  int ks = 0;
  for (; ks + 3 < ktot; ks += 4) {
    step(std::integral_constant<int, 0>{}, ks);
    step(std::integral_constant<int, 1>{}, ks + 1);
    step(std::integral_constant<int, 2>{}, ks + 2);
    step(std::integral_constant<int, 3>{}, ks + 3);
  }
  if (ks < ktot) step(std::integral_constant<int, 0>{}, ks);
  if (ks + 1 < ktot) step(std::integral_constant<int, 1>{}, ks + 1);
  if (ks + 2 < ktot) step(std::integral_constant<int, 2>{}, ks + 2);

  // the rows' sums sit in columns 0 and 1 of rs, the column tile's in every row of cs
  if ((lane & 15) < 2)
#pragma unroll
    for (int r = 0; r < 4; ++r) rsum[wave * 32 + (lane & 1) * 16 + 4 * (lane >> 4) + r] = (int)(rs[r] * 8.0f);
  if (lane < 16) csum[wave * 16 + lane] = (int)(cs[0] * 8.0f);
  __syncthreads();
  // sum a w = sum (a + 8)(w + 8) - 8 sum (a + 8) - 8 sum (w + 8) + 64 K
  int cc[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) cc[j] = 64 * p.K - 8 * csum[32 * j + r32];
  auto sums = [&](int, int j, int e) -> int {
    return (int)(acc[j][e] * 64.0f) + (cc[j] - 8 * rsum[wave * 32 + 8 * (e >> 2) + 4 * u + (e & 3)]);
  };
  write_out<1, TJ, false>(p, sums, lds, sdelta, wave, wave * 32, 0, m0, n0);
}

}  // namespace

hipError_t launch_gemm_wide(const WideParams &p, int bits, hipStream_t s, bool go) {
  static std::atomic<uint64_t> attr4{0}, attr8{0};
  const int64_t tiles = ((int64_t)(p.M + 255) / 256) * ((p.N + kBN - 1) / kBN);
  hipError_t e;
  if (bits == 4) {
    e = allow_dynamic_lds(&gemm_wide4_kernel, k4Lds, attr4);
    if (e != hipSuccess || !go) return e;
    hipLaunchKernelGGL(gemm_wide4_kernel, dim3((unsigned)tiles), dim3(64 * k4Waves), k4Lds, s, p);
  } else {
    e = allow_dynamic_lds(&gemm_wide8_kernel, k8Lds, attr8);
    if (e != hipSuccess || !go) return e;
    hipLaunchKernelGGL(gemm_wide8_kernel, dim3((unsigned)tiles), dim3(64 * k8Waves), k8Lds, s, p);
  }
  return hipGetLastError();
}

}  // namespace fq
