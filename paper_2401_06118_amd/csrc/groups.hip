// Dequantization and the batch-1 product for groups of 16, 32 or 64 inputs
// (8-bit codes, up to 16 codebooks): the codebooks-versus-groups settings of
// the paper's ablation.  Eq. 2 is unchanged; only a codeword now spans g / 8
// chunks of 8 inputs, each chunk a 16-byte slice of the codeword.
//
// These formats have no GPU speed figure in the paper (its GPU kernels cover
// 1x16 and 2x8):
//   k_dequant_groups  one thread per 8-input chunk, codeword chunks gathered
//                     from L2 (up to 512 KiB of codebooks), fp32 sums in
//                     ascending m, one product with the scale, one rounding;
//   k_gemv_groups     one wave per output row; each lane adds the M codeword
//                     chunks of its input chunks in fp32 and multiplies them
//                     with x; a fixed-order wave sum, the scale, one rounding.
//                     The codebooks sit in LDS (one copy) when they fit
//                     (up to 128 KiB), else are gathered from L2 (15x8 gs64,
//                     480 KiB);
//   k_gemv_groups_mfma  batch 1 where the codebooks fit in LDS, M divides 16,
//                     x fits beside them and the layer is large enough
//                     (4x8 gs16, 8x8 gs32): matrix cores.
#include "common.h"
#include "groups.h"
#include "launch.h"
#include "lds_sync.h"

namespace aqlm {

namespace {

constexpr int kGrpThreads = 1024;
constexpr int kGrpWaves = kGrpThreads / kWave;
constexpr size_t kGrpCbLds = 128 * 1024;

__device__ __forceinline__ void add8(const uint4& v, float (&f)[8]) {
  f[0] += h2f(v.x & 0xFFFF); f[1] += h2f(v.x >> 16);
  f[2] += h2f(v.y & 0xFFFF); f[3] += h2f(v.y >> 16);
  f[4] += h2f(v.z & 0xFFFF); f[5] += h2f(v.z >> 16);
  f[6] += h2f(v.w & 0xFFFF); f[7] += h2f(v.w >> 16);
}

__device__ __forceinline__ void set8(const uint4& v, float (&f)[8]) {
  f[0] = h2f(v.x & 0xFFFF); f[1] = h2f(v.x >> 16);
  f[2] = h2f(v.y & 0xFFFF); f[3] = h2f(v.y >> 16);
  f[4] = h2f(v.z & 0xFFFF); f[5] = h2f(v.z >> 16);
  f[6] = h2f(v.w & 0xFFFF); f[7] = h2f(v.w >> 16);
}

__global__ __launch_bounds__(256) void k_dequant_groups(const GroupLayer L, uint32_t total, uint4* __restrict__ w) {
#pragma clang fp contract(off)
  const uint32_t k = (uint32_t)L.g / 8u;            // chunks per group
  const uint32_t G = (uint32_t)(L.d_in / L.g);      // groups per row
  const uint32_t per_row = (uint32_t)L.d_in / 8u;   // chunks per row
  const uint32_t M = (uint32_t)L.M;
  const uint4* __restrict__ cb = reinterpret_cast<const uint4*>(L.codebooks);
  const uint32_t stride = gridDim.x * 256u;
  for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < total; q += stride) {
    const uint32_t row = q / per_row;
    const uint32_t c = q - row * per_row;
    const uint32_t j = c / k, p = c - j * k;
    const uint8_t* __restrict__ code = L.codes + ((size_t)row * G + j) * M;
    float acc[8];
    set8(cb[(uint32_t)code[0] * k + p], acc);
    for (uint32_t m = 1; m < M; ++m) add8(cb[((m << 8) + (uint32_t)code[m]) * k + p], acc);
    const float s = h2f(L.scales[row]);
    uint32_t h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // the product keeps its own rounding step (no fused multiply-round)
      float t = acc[e] * s;
      asm volatile("" : "+v"(t));
      h[e] = f2h(t);
    }
    w[q] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
  }
}

// One row's product by a whole wave (codebooks `src`, codes `rc`): each lane adds
// the codeword chunks of its input chunks first, then multiplies them with x.
__device__ __forceinline__ float group_row_sum(const uint4* src, const uint8_t* __restrict__ rc,
                                               const uint4* __restrict__ x, uint32_t per_row, uint32_t k, uint32_t M,
                                               int lane) {
  float acc = 0.f;
  for (uint32_t c = (uint32_t)lane; c < per_row; c += kWave) {
    const uint32_t j = c / k, p = c - j * k;
    const uint8_t* __restrict__ code = rc + (size_t)j * M;
    float u[8];
    set8(src[(uint32_t)code[0] * k + p], u);
    for (uint32_t m = 1; m < M; ++m) add8(src[((m << 8) + (uint32_t)code[m]) * k + p], u);
    const uint4 xv = x[c];
    acc += u[0] * h2f(xv.x & 0xFFFF) + u[1] * h2f(xv.x >> 16) + u[2] * h2f(xv.y & 0xFFFF) +
           u[3] * h2f(xv.y >> 16) + u[4] * h2f(xv.z & 0xFFFF) + u[5] * h2f(xv.z >> 16) +
           u[6] * h2f(xv.w & 0xFFFF) + u[7] * h2f(xv.w >> 16);
  }
  return wave_sum(acc);
}

template <bool LDS>
__global__ __launch_bounds__(kGrpThreads) void k_gemv_groups(const GroupLayer L, const uint4* __restrict__ x,
                                                             uint16_t* __restrict__ y) {
  extern __shared__ uint4 cb_lds[];
  const uint32_t k = (uint32_t)L.g / 8u;
  const uint32_t G = (uint32_t)(L.d_in / L.g);
  const uint32_t per_row = (uint32_t)L.d_in / 8u;
  const uint32_t M = (uint32_t)L.M;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const uint4* __restrict__ cb = reinterpret_cast<const uint4*>(L.codebooks);
  if constexpr (LDS) {
    const uint32_t entries = M * 256u * k;
    for (uint32_t e = threadIdx.x; e < entries; e += kGrpThreads) cb_lds[e] = cb[e];
    __syncthreads();
  }
  const uint4* src = LDS ? cb_lds : cb;
  for (int32_t row = blockIdx.x * kGrpWaves + wave; row < L.d_out; row += gridDim.x * kGrpWaves) {
    const float sum = group_row_sum(src, L.codes + (size_t)row * G * M, x, per_row, k, M, lane);
    if (lane == 0) y[row] = f2h(h2f(L.scales[row]) * sum);
  }
}

// Batch 1 on the matrix cores.  A 16-byte chunk of a codeword is a lane's A
// fragment of v_mfma_f32_16x16x32_f16 (lane = row + 16 * slot), the matching
// chunk of x column 0 of B; a code takes G8 of them.  An item is 16 rows x 64
// code bytes: a lane's 16 codes (one 16-byte load at any alignment) are 16 / M
// whole groups.  Items go round-robin to the 16 waves of a workgroup, code
// loads two items ahead; a wave's sums move to LDS when its row block changes
// and are added over the waves in a fixed order.  Bound by the LDS gathers (16
// bytes per code chunk from kCopies codebook copies, lane l reads copy
// l % kCopies): 11008 x 4096 4x8 gs16 44 -> 14 us, 8x8 gs32 67 -> 23 us against
// one wave per row with byte loads of the codes and vector-ALU sums.
// A row's last, partial slot loads the row's last 16 bytes and skips the codes
// of the slot before; slots past the end read the row's first bytes against
// x = 0.  In an item with such slots (TAIL) their fragments are zero as well:
// an infinite codeword would make NaN of 0.
constexpr int kGmMaxRows = 2 * kWave;  // rows per workgroup (8 blocks; two waves store them)

template <int M, int G8>
struct GmCfg {
  static constexpr int kFit = 32 / (M * G8);  // copies that fit in 128 KiB (one copy: 4 KiB * M * G8)
  static constexpr int kCopies = kFit >= 16 ? 16 : (kFit >= 8 ? 8 : (kFit >= 4 ? 4 : (kFit >= 2 ? 2 : 1)));
  static constexpr size_t kCb = (size_t)M * 256 * G8 * kCopies * 16;
};

typedef uint32_t u32x4a1_t __attribute__((ext_vector_type(4), aligned(1)));

template <int M, int G8>
__global__ __launch_bounds__(kGrpThreads) void k_gemv_groups_mfma(const GroupLayer L, const uint4* __restrict__ x,
                                                                  uint16_t* __restrict__ y, int32_t rows_per_wg) {
  using C = GmCfg<M, G8>;
  constexpr int kCopies = C::kCopies, kGroups = 16 / M;  // whole groups per lane slot
  extern __shared__ uint4 lds[];
  uint4* const cb_lds = lds;  // [chunk][M][256][copies]
  uint4* const x_lds = lds + C::kCb / 16;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int r16 = lane & 15, slot = lane >> 4;
  const int32_t row0 = (int32_t)blockIdx.x * rows_per_wg;
  const int32_t rows = L.d_out - row0 < rows_per_wg ? L.d_out - row0 : rows_per_wg;
  const int32_t G = L.d_in / (8 * G8);
  const uint32_t pitch = (uint32_t)G * M;  // code bytes per row (at least 16)
  const int KS = (int)((pitch + 63u) / 64u);
  const int items = (rows + 15) / 16 * KS;
  const int xc = KS * 4 * kGroups * G8;    // x chunks staged, zero past the end
  const uint4* __restrict__ cb = reinterpret_cast<const uint4*>(L.codebooks);
  float* const part = reinterpret_cast<float*>(x_lds + xc);

  // this lane's slot of an item, and how many codes it starts before the slot
  auto slot_off = [&](int ks, int& back) -> uint32_t {
    const uint32_t off = (uint32_t)ks * 64u + (uint32_t)slot * 16u;
    back = 0;
    if (off >= pitch) return 0u;
    if (off + 16u > pitch) {
      back = (int)(off + 16u - pitch);
      return pitch - 16u;
    }
    return off;
  };
  auto load_codes = [&](int item, u32x4_t& w) {
    const int it = item < items ? item : items - 1;
    int back;
    int row = it / KS * 16 + r16;
    row = row < rows ? row : rows - 1;
    const uint8_t* p = L.codes + (size_t)(row0 + row) * pitch + slot_off(it % KS, back);
    w = __builtin_nontemporal_load(reinterpret_cast<const u32x4a1_t*>(p));
  };

  // small loads first, then the first items' codes
  constexpr int kCbLoads = M * 256 * G8 / kGrpThreads > 0 ? M * 256 * G8 / kGrpThreads : 1;
  uint4 cbv[kCbLoads];
#pragma unroll
  for (int i = 0; i < kCbLoads; ++i)
    if (tid + i * kGrpThreads < M * 256 * G8) cbv[i] = cb[tid + i * kGrpThreads];
  u32x4_t cw[2];
  load_codes(wave, cw[0]);
  load_codes(wave + kGrpWaves, cw[1]);
  const float sc = h2f(L.scales[row0 + (tid < rows ? tid : rows - 1)]);
  for (int e = tid; e < xc; e += kGrpThreads) x_lds[e] = e < G * G8 ? x[e] : make_uint4(0, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < kCbLoads; ++i) {
    const int q = tid + i * kGrpThreads;
    if (q < M * 256 * G8) {
#pragma unroll
      for (int c = 0; c < kCopies; ++c)
        cb_lds[((q % G8) * M * 256 + q / G8) * kCopies + ((c + lane) % kCopies)] = cbv[i];
    }
  }
  for (int e = tid; e < (rows + 15) / 16 * kGrpWaves * 16; e += kGrpThreads) part[e] = 0.f;
  __syncthreads();

  f4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  int cur = -1;
  auto flush = [&]() {
    if (cur >= 0 && r16 == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) part[(cur * kGrpWaves + wave) * 16 + 4 * slot + e] = acc0[e] + acc1[e];
    }
  };
  const uint4* const my_cb = cb_lds + lane % kCopies;
  for (int item = wave, u = 0; item < items; item += kGrpWaves, u ^= 1) {
    const u32x4_t w = u ? cw[1] : cw[0];
    // (the codes two items on: a select keeps both sets in registers)
    u32x4_t nw;
    load_codes(item + 2 * kGrpWaves, nw);
    const int rb = item / KS, ks = item % KS;
    if (rb != cur) {
      flush();
      acc0 = acc1 = f4_t{0.f, 0.f, 0.f, 0.f};
      cur = rb;
    }
    int back;
    slot_off(ks, back);
    // first chunk of the group of this lane's code 0
    const int c0 = ((ks * 4 + slot) * kGroups - back / M) * G8;
    auto products = [&](auto tail) __attribute__((always_inline)) {
      constexpr bool TAIL = decltype(tail)::value != 0;
      const bool past = (uint32_t)ks * 64u + (uint32_t)slot * 16u >= pitch;
#pragma unroll
      for (int q = 0; q < kGroups; ++q) {
        const bool valid = !TAIL || (!past && q * M >= back);
#pragma unroll
        for (int p = 0; p < G8; ++p) {
          uint4 xb = make_uint4(0, 0, 0, 0);
          if (r16 == 0 && valid) xb = x_lds[c0 + q * G8 + p];
          const h8_t xh = __builtin_bit_cast(h8_t, xb);
#pragma unroll
          for (int m = 0; m < M; ++m) {
            const int t = q * M + m;
            const uint32_t code = (w[t / 4] >> (8 * (t % 4))) & 0xFFu;
            uint4 av = my_cb[((p * M + m) * 256 + code) * kCopies];
            if (TAIL && !valid) av = make_uint4(0, 0, 0, 0);
            f4_t& a = (m + p) % 2 == 0 ? acc0 : acc1;
            a = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, av), xh, a, 0, 0, 0);
          }
        }
      }
    };
    if (__builtin_amdgcn_readfirstlane((uint32_t)ks * 64u + 64u) > pitch)
      products(IntC<1>{});
    else
      products(IntC<0>{});
    if (u)
      cw[1] = nw;
    else
      cw[0] = nw;
  }
  flush();
  __syncthreads();
  // Rows that come out as NaN are computed again as k_gemv_groups does: x_c
  // infinite makes infinities of both signs of a group's codewords, their sum only
  // one.  Their mask goes through the space of x, so that all waves share them.
  uint64_t* const nan = reinterpret_cast<uint64_t*>(x_lds);
  if (wave < kGmMaxRows / kWave) {
    float s = 0.f;
    if (tid < rows) {
#pragma unroll
      for (int v = 0; v < kGrpWaves; ++v) s += part[(tid / 16 * kGrpWaves + v) * 16 + tid % 16];
      if (s == s) y[row0 + tid] = f2h(sc * s);
    }
    const uint64_t bad = __ballot(s != s);
    if (lane == 0) nan[wave] = bad;
  }
  lds_barrier();
  const uint64_t bad0 = nan[0], bad1 = nan[1];
  if (__builtin_expect((bad0 | bad1) == 0, 1)) return;
  for (int r = wave; r < rows; r += kGrpWaves) {
    if ((((r < kWave ? bad0 : bad1) >> (r % kWave)) & 1) == 0) continue;
    const int32_t row = row0 + r;
    const float sum = group_row_sum(cb, L.codes + (size_t)row * pitch, x, (uint32_t)(G * G8), G8, M, lane);
    if (lane == 0) y[row] = f2h(h2f(L.scales[row]) * sum);
  }
}

template <int M, int G8>
size_t gm_lds(const GroupLayer& L, int rows) {
  const size_t KS = ((size_t)(L.d_in / L.g) * M + 63) / 64;
  return GmCfg<M, G8>::kCb + KS * 4 * (16 / M) * G8 * 16 + (size_t)((rows + 15) / 16) * kGrpWaves * 64;
}

// Whether the matrix-core kernel is the faster one.  It fills 128 KiB of LDS
// with codebook copies first and an item is a serial chain of 16 G8 gathers;
// k_gemv_groups copies each codebook once and takes about 0.2 + 0.17 M us per
// step of a row (64 chunks of 8 inputs) and row of a wave.  At equal rows and
// inputs, k_gemv_groups -> this kernel in us (4096 rows): one codebook g = 64
// 1024 inputs 3.8 -> 11.1, 8192 8.8 -> 11.0; 2x8 g = 16 1024 4.0 -> 4.7, 2048
// 5.0 -> 4.8; 4x8 g = 16 1024 4.8 -> 5.1, 2048 6.7 -> 5.7; 4x8 g = 64 2048 7.1 ->
// 9.4, 4096 10.5 -> 10.0; 16x8 g = 16 256 6.5 -> 5.4; and at 16384 rows 1x8
// g = 64 2048 9.4 -> 12.6, 4096 15.2 -> 10.7; 4x8 g = 16 256 7.3 -> 4.8.
bool groups_mfma_pays(const GroupLayer& L, int G8) {
  const int64_t cus = num_cus();
  const int64_t steps = (L.d_out + kGrpWaves * cus - 1) / (kGrpWaves * cus) * ((L.d_in + 511) / 512);
  return steps * L.M >= 4 * G8 && steps * (L.M + 1) >= 12;
}

// Launches the matrix-core kernel if it takes the layer.
template <int M, int G8>
bool try_groups_mfma(const GroupLayer& L, const uint16_t* x, uint16_t* y, hipStream_t s, hipError_t* e) {
  if constexpr (M * G8 > 32) {
    return false;
  } else {
    if ((int64_t)(L.d_in / L.g) * M < 16 || !groups_mfma_pays(L, G8)) return false;
    // rows split evenly over whole rounds of one workgroup per CU
    const int64_t cus = num_cus(), rounds = (L.d_out + kGmMaxRows * cus - 1) / (kGmMaxRows * cus);
    const int rows = (int)((L.d_out + rounds * cus - 1) / (rounds * cus));
    const size_t lds = gm_lds<M, G8>(L, rows);
    if (lds > 160 * 1024) return false;
    auto kern = k_gemv_groups_mfma<M, G8>;
    *e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), 160 * 1024);
    if (*e != hipSuccess) return true;
    hipLaunchKernelGGL(kern, dim3((uint32_t)((L.d_out + rows - 1) / rows)), dim3(kGrpThreads), lds, s, L,
                       reinterpret_cast<const uint4*>(x), y, rows);
    *e = hipGetLastError();
    return true;
  }
}

template <int M>
bool try_groups_mfma_g(const GroupLayer& L, const uint16_t* x, uint16_t* y, hipStream_t s, hipError_t* e) {
  switch (L.g) {
    case 16: return try_groups_mfma<M, 2>(L, x, y, s, e);
    case 32: return try_groups_mfma<M, 4>(L, x, y, s, e);
    case 64: return try_groups_mfma<M, 8>(L, x, y, s, e);
  }
  return false;
}

}  // namespace

hipError_t launch_dequant_groups(const GroupLayer& L, uint16_t* w, hipStream_t s) {
  const uint32_t total = (uint32_t)((int64_t)L.d_out * (L.d_in / 8));
  uint32_t blocks = (total + 255u) / 256u;
  const uint32_t cap = (uint32_t)num_cus() * 8u;
  if (blocks > cap) blocks = cap;
  hipLaunchKernelGGL(k_dequant_groups, dim3(blocks), dim3(256), 0, s, L, total, reinterpret_cast<uint4*>(w));
  return hipGetLastError();
}

hipError_t launch_gemv_groups(const GroupLayer& L, const uint16_t* x, uint16_t* y, hipStream_t s) {
  hipError_t me = hipSuccess;
  bool taken = false;
  switch (L.M) {
    case 1: taken = try_groups_mfma_g<1>(L, x, y, s, &me); break;
    case 2: taken = try_groups_mfma_g<2>(L, x, y, s, &me); break;
    case 4: taken = try_groups_mfma_g<4>(L, x, y, s, &me); break;
    case 8: taken = try_groups_mfma_g<8>(L, x, y, s, &me); break;
    case 16: taken = try_groups_mfma_g<16>(L, x, y, s, &me); break;
  }
  if (taken) return me;
  const size_t cb_bytes = (size_t)L.M * 256 * (size_t)L.g * 2;
  const int32_t row_blocks = (L.d_out + kGrpWaves - 1) / kGrpWaves;
  int32_t grid = num_cus();
  if (grid > row_blocks) grid = row_blocks;
  const uint4* xv = reinterpret_cast<const uint4*>(x);
  if (cb_bytes <= kGrpCbLds) {
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(k_gemv_groups<true>), (int)kGrpCbLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gemv_groups<true>, dim3(grid), dim3(kGrpThreads), cb_bytes, s, L, xv, y);
  } else {
    hipLaunchKernelGGL(k_gemv_groups<false>, dim3(grid), dim3(kGrpThreads), 0, s, L, xv, y);
  }
  return hipGetLastError();
}

}  // namespace aqlm
