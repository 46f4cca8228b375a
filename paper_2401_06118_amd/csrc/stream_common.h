// Device helpers shared by the kernels that stream AQLM codes from HBM and
// look codewords up in LDS codebook copies (batch-1 and small-batch
// products).
#pragma once

#include "common.h"

namespace aqlm {

// How the rows of 8-bit codes end, a template parameter (ROWS) of the kernels
// that run them.  Codes past a row's end meet x = 0, but an infinite codeword
// would make NaN of that.  So in the wave's last K-slice
//   - a lane whose slot is past the end reads 16 zero bytes (a group of x past
//     the end) as every codeword, by the operands of its address permute;
//   - in a slot that is partly past the end, the codes after the last are set
//     to codes of finite codewords.
// Without the permute (few codebook copies) every code past the end takes the
// zero bytes by a select.
constexpr int kRowBytes = 0;  // any length, loaded byte by byte
constexpr int kRowSlots = 1;  // whole 16-byte slots (with the permute only)
constexpr int kRowPart = 2;   // loaded as whole slots (tiled codes of any length)
constexpr int kRowWhole = 3;  // whole K-slices: nothing is past the end

// The permute's selector in a lane past the row's end: its base as it is.
constexpr uint32_t kPermBase = 0x03020100u;

template <int B>
struct GCfg {
  static constexpr int kBpc = code_bytes(B);  // bytes per code
  static constexpr int kCPL = 16 / kBpc;      // codes per lane per item
  static constexpr int kKS = 4 * kCPL;        // codes per row per item
  static constexpr int kXL = (B == 8) ? 4 : 8;  // x staging loads per thread (groups <= kXL * 1024)
};

// Generic (unaligned-pitch) path: byte loads of the valid codes of a lane's
// 16-byte slot, zero past the row end.
template <int B>
__device__ __forceinline__ void load_codes_bytes(const uint8_t* __restrict__ row_ptr, uint32_t pitch, uint32_t off,
                                                 uint32_t (&w)[4]) {
  w[0] = w[1] = w[2] = w[3] = 0;
  const int nbytes = off < pitch ? (int)min(pitch - off, 16u) : 0;
#pragma unroll
  for (int b = 0; b < 16; ++b)
    if (b < nbytes) w[b / 4] |= (uint32_t)row_ptr[off + b] << (8 * (b % 4));
}

typedef __attribute__((address_space(3))) const u32x4_t lds_v4;

// 16-byte LDS load from an LDS byte address (ds_read_b128).
__device__ __forceinline__ uint4 lds_load16(uint32_t byte_addr) {
  const u32x4_t v = *(lds_v4*)(uintptr_t)byte_addr;
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Four code bytes (a whole number of groups) whose codewords are finite, from
// the interleaved copies at LDS address cb_base; a codebook without a finite
// codeword gives code 0.  Called by a whole wave.
template <int M, int COPIES>
__device__ __forceinline__ uint32_t finite_codes(uint32_t cb_base, int lane) {
  auto finite = [&](int m, int e) {
    const uint4 v = lds_load16(cb_base + (uint32_t)(e * 16 + m * COPIES + lane % COPIES) * 16u);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t bad = 0;  // (a half is finite if its exponent bits are not all ones)
#pragma unroll
    for (int i = 0; i < 4; ++i) bad |= ((w[i] & 0x7C007C00u) + 0x04000400u) & 0x80008000u;
    return __ballot(bad == 0);
  };
  uint64_t any[M];
#pragma unroll
  for (int m = 0; m < M; ++m) any[m] = finite(m, lane);
  uint32_t group = 0;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    uint32_t first = 0;
    while (__builtin_expect(any[m] == 0, 0) && first + kWave < 256) any[m] = finite(m, (int)(first += kWave) + lane);
    if (any[m] != 0) group |= (first + (uint32_t)__builtin_ctzll(any[m])) << (8 * m);
  }
  return M == 4 ? group : (M == 2 ? group * 0x10001u : group * 0x1010101u);
}

// The codes of a slot after its first `left`, replaced by those of `fill`.
__device__ __forceinline__ void fill_past_end(uint32_t (&w)[4], int left, uint32_t fill) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = left - 4 * i;
    const uint32_t keep = n >= 4 ? 0xFFFFFFFFu : (n <= 0 ? 0u : (1u << (8 * n)) - 1u);
    w[i] = (w[i] & keep) | (fill & ~keep);
  }
}

// LDS byte address of codeword `code` of codebook m for this lane's copy.
// With 16 copies and M <= 2 the address is (m << 16) | (code << 8) | (copy << 4),
// built from the code byte with a single v_perm_b32: byte 0 and byte 2 come
// from base_m = (m << 16) | (copy << 4), byte 1 is byte `k` of the code word.
template <int M, int COPIES>
__device__ __forceinline__ uint32_t cw_addr(uint32_t word, int k, uint32_t base_m, uint32_t copy_off, int m) {
  if constexpr (COPIES == 16 && M <= 2) {
    (void)copy_off;
    (void)m;
    return __builtin_amdgcn_perm(word, base_m, 0x0C020000u | ((uint32_t)(4 + k) << 8));
  } else {
    (void)base_m;
    const uint32_t code = (word >> (8 * k)) & 0xFFu;
    return ((uint32_t)(m * 256) + code) * (uint32_t)(COPIES * 16) + copy_off;
  }
}

}  // namespace aqlm
