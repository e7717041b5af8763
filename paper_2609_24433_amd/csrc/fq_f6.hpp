// INT4 products on gfx950's FP6 matrix instructions, shared by the GEMMs that use them.
//
// The FP6 format E2M3 holds 0, 1/8, 2/8, .. 15/8 as the bit patterns 0 .. 15, so a six-bit field
// with code + 8 (1 .. 15 for codes -7 .. 7) in its low four bits is the number (code + 8) / 8
// exactly.  Products are integers over 64 of at most 225, and their fp32 sums stay exact: at most
// 225 * 32768 < 2^24 (tests cover the largest sum, and long sums of mixed codes to the last unit).
// The 32 x 32 x 64 instruction measured 8.4 PFLOP/s against 4.2 for INT8's 32 x 32 x 32 (small
// operands; under real codes the clock falls).  With both operands biased by 8,
//   sum a w = 64 sum (a+8)/8 (w+8)/8 - 8 sum (a+8) - 8 sum (w+8) + 64 K,
// the sums of codes coming from 16 x 16 x 128 instructions against patterns of ones.
#pragma once

#include "fq_device.hpp"
#include "fq_launch.hpp"

namespace fq {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, int64_t bytes) {
  const int n = bytes < 0x7fffffff ? (int)bytes : 0x7fffffff;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, n, 0x00020000);
}

// Byte offset of a wave's 32 rows in k-major codes: lane l reads chunk l / 32 (and, 32 bytes on,
// chunk 2 + l / 32) of a piece of row row0 + l % 32 (rows past M repeat row M - 1).
__device__ __forceinline__ uint32_t row_offset(int row0, int M, int lane) {
  return (uint32_t)min(row0 + (lane & 31), M - 1) * 64u + (uint32_t)(lane >> 5) * 16u;
}

// FP6 x FP6 products (a format selector of 2 is E2M3; six of the eight words are read).
__device__ __forceinline__ v16f mfma_f6_32(v8i a, v8i b, v16f c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, 0, 0, 0);
#else
  return c;
#endif
}
__device__ __forceinline__ v4f mfma_f6_16(v8i a, v8i b, v4f c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 2, 2, 0, 0, 0, 0);
#else
  return c;
#endif
}

// (a & b) ^ c
__device__ __forceinline__ uint32_t and_xor(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x6a);
#else
  return (a & b) ^ c;
#endif
}

// 16 nibble codes (words x and y, two's complement) -> 16 six-bit fields code + 8 in three
// words.
__device__ __forceinline__ void spread16(uint32_t x, uint32_t y, int *d) {
  const uint32_t x2 = x << 2;
  const uint32_t t = __builtin_amdgcn_alignbit(y, x, 30);
  d[0] = (int)and_xor(x2, 0xC03C03C0u, and_xor(x, 0x0F00F00Fu, 0x08208208u));
  d[1] = (int)and_xor(t, 0x03C03C03u, and_xor(y, 0xF00F00F0u, 0x82082082u));
  d[2] = (int)and_xor(t, 0x3C03C03Cu, and_xor(x, 0x00F00F00u, 0x20820820u));
}
__device__ __forceinline__ v8i spread32(const v4i &r) {
  int d[6];
  spread16((uint32_t)r.x, (uint32_t)r.y, d);
  spread16((uint32_t)r.z, (uint32_t)r.w, d + 3);
  return v8i{d[0], d[1], d[2], d[3], d[4], d[5], 0, 0};
}
// The prologue's arrangement (pack_chunk_f6) of 16 canonical nibble codes.
__device__ __forceinline__ uint2 rearrange16(uint32_t x, uint32_t y) {
  int d[3];
  spread16(x, y, d);
  return make_uint2((uint32_t)d[0] | ((uint32_t)d[2] & 0x30C30C30u), (uint32_t)d[1] | ((uint32_t)d[2] & 0x0C30C30Cu));
}
// The same fields from that arrangement: two words hold three words' fields in place.
__device__ __forceinline__ v8i expand32(const v4i &r) {
  const uint32_t x = (uint32_t)r.x, y = (uint32_t)r.y, z = (uint32_t)r.z, w = (uint32_t)r.w;
  return v8i{(int)(x & 0xCF3CF3CFu), (int)(y & 0xF3CF3CF3u), (int)((x & 0x30C30C30u) | (y & 0x0C30C30Cu)),
             (int)(z & 0xCF3CF3CFu), (int)(w & 0xF3CF3CF3u), (int)((z & 0x30C30C30u) | (w & 0x0C30C30Cu)), 0, 0};
}

// Operands of the code sums.  All ones (field 8 = 1.0).
__device__ __forceinline__ v8i f6_ones() {
  return v8i{0x08208208, (int)0x82082082u, 0x20820820, 0x08208208, (int)0x82082082u, 0x20820820, 0, 0};
}
// A 32-row operand of the 32 x 32 x 64 instruction, read as a 16-row one, has rows 0..15 in lane
// groups 0 and 2 and rows 16..31 in groups 1 and 3.  Against ones in groups 0, 2 of column 0 and
// groups 1, 3 of column 1, columns 0 and 1 of the product are the sums of rows 0..15 and 16..31
// (and with the pattern as the left operand rows 0 and 1 are those of the columns).
__device__ __forceinline__ v8i f6_row_pattern(int lane) {
  const int on = (lane & 15) == ((lane >> 4) & 1) ? -1 : 0;
  const v8i o = f6_ones();
  return v8i{o[0] & on, o[1] & on, o[2] & on, o[3] & on, o[4] & on, o[5] & on, 0, 0};
}

}  // namespace fq
