// AQLM product for codebooks of 2^12 to 2^16 entries and 1 <= n <= 64
// activation rows (unpacked 16-bit codes, one or two codebooks):
//   Y[t][i] = fp16(s_i * sum_j sum_m <C_m[b_ijm], X[t, 8j:8j+8]>)   (Eq. 2)
//
// Bound.  A codebook of 2^15 or 2^16 entries does not fit in LDS, so each code
// fetches its codeword from L2, one 128-byte line per 16-byte codeword: 0.43-
// 0.45 gathers per clock per CU, whatever the cache policy of the load (probed:
// default, nontemporal, device and system scope), 21 us for the 5.6 million codes
// of a 7B gate or down projection.  The kernel's work is to keep that path
// busy and to make one gather serve every activation row: the gathered
// codeword is the A fragment of v_mfma_f32_16x16x32_f16 (lane = row + 16 *
// slot), and NB blocks of 16 rows of x are its B operands.
//
// Work split.  A workgroup of KW waves owns RB blocks of 16 rows; wave w takes
// the 64-byte K-slices w, w + KW, ... (one per round) of every block.  An item
// is one K-slice of one block: a lane's 8 codes (one 16-byte load at any
// alignment), 8 gathers, 8 NB MFMAs.  Gathers run one item ahead of their use
// and code loads two, across rounds, so the gather queue does not drain at the
// barriers.  x of a round (KW K-slices) sits in LDS, the next round's in
// registers.  The waves' partial sums are added in a fixed order at the end, so
// results are deterministic.
//
// Two 4096-entry codebooks (128 KiB) are copied into LDS instead and gathered
// there; four waves then suffice, and x of a round takes the remaining 32 KiB.
//
// Row ends.  A row's code bytes need not be a multiple of 16.  The slot that
// holds the row's last codes loads the row's last 16 bytes and shifts its x
// slices by as many groups, with zeros for the codes of the slot before; slots
// wholly past the end load the row's first bytes against x = 0.  Both kinds of
// codes get zero fragments too: an infinite codeword would make NaN of 0.
//
// Measured against the general tiled kernel (k_gemm_mfma, four waves per CU, two
// barriers per 32 codes; chunks of 16 rows) and, for one codebook from 33 rows,
// the prefill kernel; us at 5 / 16 / 32 / 64 / 128 rows:
//   1x16 4096 x 11008   49 / 61 / 120 / 270 / 281 -> 34 / 36 / 40 / 51 / 99
//   1x16 11008 x 4096   32 / 36 /  69 / 111 / 112 -> 31 / 31 / 35 / 40 / 78
//   2x16 4096 x 4096    34 / 35 /  68 / 142 / 150 -> 25 / 25 / 27 / 33 / 64
//   2x12 11008 x 4096   22 / 22 /  50 /  83 /  92 -> 18 / 19 / 23 / 47 / 91
//   2x12 4096 x 4096    21 / 22 /  43 /  65 /  91 -> 10 / 11 / 13 / 25 / 51
//   2x12 9000 x 7304    95 / 96 / 186 / 293 / 294 -> 29 / 31 / 38 / 76 / 150
// (One codebook, 17 to 32 rows and three row blocks: 10 registers spill.)
#include "common.h"
#include "launch.h"
#include "lds_sync.h"

namespace aqlm {

namespace {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef uint32_t u32x4a1_t __attribute__((ext_vector_type(4), aligned(1)));

constexpr size_t kGwLdsLimit = 160 * 1024;

struct GemmWideArgs {
  const uint8_t* codes;
  const uint4* cb;
  const uint16_t* scales;
  const uint4* x;  // [n][G] groups of 8 fp16
  uint16_t* y;     // [n][d_out]
  int32_t d_out;
  int32_t G;
  int32_t n;
  int32_t B;
  int32_t rows_per_wg;
};

// M codebooks; NB blocks of 16 activation rows; KW waves; RB blocks of 16
// weight rows; LDSCB: two 4096-entry codebooks in LDS.
template <int M, int NB, int KW, int RB, bool LDSCB>
__global__ __launch_bounds__(KW* kWave) void k_gemm_wide(const GemmWideArgs a) {
  constexpr int kThreads = KW * kWave;
  constexpr int kGS = 32 / M;                       // groups per K-slice
  constexpr int kXG = KW * kGS;                     // groups per round
  constexpr int kXV = NB * 16 * kXG / kThreads;     // x loads per thread and round
  constexpr int kSlotG = 8 / M;                     // groups per lane slot
  extern __shared__ uint4 lds[];
  uint4* const cb_lds = lds;
  uint4* const x_lds = lds + (LDSCB ? 2 * 4096 : 0);  // [tok][kXG], group position g ^ (tok % 16)
  float* const part = reinterpret_cast<float*>(x_lds);

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int r16 = lane & 15;
  const int slot = lane >> 4;
  const int32_t row0 = (int32_t)blockIdx.x * a.rows_per_wg;
  const int32_t rows = a.d_out - row0 < a.rows_per_wg ? a.d_out - row0 : a.rows_per_wg;
  const int32_t G = a.G, n = a.n;
  const uint32_t pitch = (uint32_t)G * M * 2u;  // code bytes per row (at least 16)
  const int KS = (int)((pitch + 63u) / 64u);
  const int R = (KS + KW - 1) / KW;
  const uint32_t mask = (1u << a.B) - 1u;
  const int cb_shift = a.B + 4;

  if constexpr (LDSCB) {
    for (int e = wave; e < 2 * 4096 / kWave; e += KW) {
#if defined(__HIP_DEVICE_COMPILE__)
      __builtin_amdgcn_global_load_lds(a.cb + e * kWave + lane, (lds_void_t*)(cb_lds + e * kWave), 16, 0, 0);
#endif
    }
  }

  // rows past the workgroup's last repeat it (their gathers fall on its lines,
  // their sums are not stored)
  const uint8_t* row_ptr[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int32_t row = rb * 16 + r16 < rows ? rb * 16 + r16 : rows - 1;
    row_ptr[rb] = a.codes + (size_t)(row0 + row) * pitch;
  }
  // Byte offset of this lane's slot of round j; `back` = groups the slot's
  // codes start before it (the row's last slot).
  auto slot_off = [&](int j, int& back) -> uint32_t {
    const int ks = wave + j * KW;
    const uint32_t off = (uint32_t)ks * 64u + (uint32_t)slot * 16u;
    back = 0;
    if (off >= pitch) return 0u;
    if (off + 16u > pitch) {
      back = (int)((off + 16u - pitch) / (2u * M));
      return pitch - 16u;
    }
    return off;
  };
  auto load_codes = [&](int j, const uint8_t* rp, uint32_t (&w)[4]) __attribute__((always_inline)) {
    int back;
    const uint32_t off = slot_off(j < R ? j : R - 1, back);
    const u32x4a1_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4a1_t*>(rp + off));
    w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
  };
  uint4 xv[kXV];
  auto load_x = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kXV; ++i) {
      const int e = tid + i * kThreads;
      const int t = e / kXG, g = j * kXG + e % kXG;
      xv[i] = make_uint4(0, 0, 0, 0);
      if (t < n && g < G) xv[i] = a.x[(size_t)t * G + g];
    }
  };
  auto gather = [&](bool live, const uint32_t (&w)[4], uint4 (&av)[8]) __attribute__((always_inline)) {
    // (a wave without a K-slice in the round fetches codeword 0 throughout:
    // one line)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint32_t code = live ? (w[t / 2] >> (16 * (t % 2))) & mask : 0u;
      if constexpr (LDSCB)
        av[t] = cb_lds[(t % M) * 4096 + code];
      else
        av[t] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.cb) +
                                                ((uint32_t)(t % M) << cb_shift) + (code << 4));
    }
  };

  f4_t acc[RB][NB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = f4_t{0.f, 0.f, 0.f, 0.f};

  // item it = round * RB + block; its codes are in cw[it % 2], its codewords
  // in av[it % 2]
  uint32_t cw[2][4];
  uint4 av[2][8];
  load_codes(0, row_ptr[0], cw[0]);
  load_codes(RB > 1 ? 0 : 1, row_ptr[RB > 1 ? 1 : 0], cw[1]);
  load_x(0);
  if constexpr (!LDSCB) gather(wave < KS, cw[0], av[0]);

  auto item = [&](int j, auto rbc, auto bufc) __attribute__((always_inline)) {
    constexpr int rb = decltype(rbc)::value, buf = decltype(bufc)::value;
    if constexpr (!LDSCB) {
      // the next item's gathers, then the codes of the one after it
      const int jn = rb + 1 < RB ? j : j + 1;
      gather(wave + jn * KW < KS && jn < R, cw[buf ^ 1], av[buf ^ 1]);
      load_codes(rb + 2 < RB ? j : (rb + 2 < 2 * RB ? j + 1 : j + 2), row_ptr[(rb + 2) % RB], cw[buf]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (rb == 0) {
      lds_barrier();  // the previous round's x fully read
#pragma unroll
      for (int i = 0; i < kXV; ++i) {
        const int e = tid + i * kThreads;
        const int t = e / kXG, g = e % kXG;
        x_lds[t * kXG + (g ^ (t & 15))] = xv[i];
      }
      if (j + 1 < R) load_x(j + 1);
      // (this wave's share of the codebooks has arrived; vmcnt 0)
      if (LDSCB && j == 0) __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
      lds_barrier();
    }
    if (wave + j * KW < KS) {
      int back;
      slot_off(j, back);
      const int g0 = wave * kGS + slot * kSlotG - back;
      if constexpr (LDSCB) gather(true, cw[buf], av[buf]);
      const uint32_t off = (uint32_t)(wave + j * KW) * 64u;
      if (off + 64u > pitch) {  // the row's last K-slice, partial
        const int skip = off + (uint32_t)slot * 16u >= pitch ? 8 : back * M;
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (t < skip) av[buf][t] = make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int t = 0; t < 8; t += M) {
        const bool valid = t / M >= back;
        h8_t bf[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int g = valid ? g0 + t / M : 0;
          uint4 v = x_lds[(nb * 16 + r16) * kXG + (g ^ r16)];
          if (!valid) v = make_uint4(0, 0, 0, 0);
          bf[nb] = __builtin_bit_cast(h8_t, v);
        }
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[rb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, av[buf][t + m]), bf[nb],
                                                                acc[rb][nb], 0, 0, 0);
      }
    }
    if constexpr (LDSCB) {
      load_codes(rb + 2 < RB ? j : (rb + 2 < 2 * RB ? j + 1 : j + 2), row_ptr[(rb + 2) % RB], cw[buf]);
    }
  };
  // two rounds per period when the block count is odd, so that the register
  // sets alternate
  auto round = [&](int j, auto first) __attribute__((always_inline)) {
    constexpr int f = decltype(first)::value;
    item(j, IntC<0>{}, IntC<f & 1>{});
    if constexpr (RB > 1) item(j, IntC<1 % RB>{}, IntC<(f + 1) & 1>{});
    if constexpr (RB > 2) item(j, IntC<2 % RB>{}, IntC<f & 1>{});
    if constexpr (RB > 3) item(j, IntC<3 % RB>{}, IntC<(f + 1) & 1>{});
  };
  if constexpr (RB % 2 == 0) {
    for (int j = 0; j < R; ++j) round(j, IntC<0>{});
  } else {
    int j = 0;
    for (; j + 2 <= R; j += 2) {
      round(j, IntC<0>{});
      round(j + 1, IntC<1>{});
    }
    if (j < R) round(j, IntC<0>{});
  }

  // every wave's 16 x 16 tiles (lane: token r16, rows 4 * slot + i), then the
  // sums over the waves in order
  lds_barrier();
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        part[((wave * RB + rb) * NB + nb) * 256 + (4 * slot + i) * 16 + r16] = acc[rb][nb][i];
  lds_barrier();
  for (int e = tid; e < RB * NB * 256; e += kThreads) {
    // row fastest over the threads: y is [token][row]
    const int rb = e / (NB * 256), nb = e / 256 % NB, tok = nb * 16 + (e >> 4) % 16, rr = e & 15;
    const int32_t row = row0 + rb * 16 + rr;
    if (tok < n && rb * 16 + rr < rows) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) s += part[((w * RB + rb) * NB + nb) * 256 + rr * 16 + (tok & 15)];
      a.y[(size_t)tok * a.d_out + row] = f2h(h2f(a.scales[row]) * s);
    }
  }
}

template <int M, int NB, int KW, int RB, bool LDSCB>
hipError_t run_wide(const GemmWideArgs& a, hipStream_t s) {
  constexpr size_t x_bytes = (size_t)NB * 16 * KW * (32 / M) * 16, part_bytes = (size_t)KW * RB * NB * 1024;
  constexpr size_t lds = (LDSCB ? 128 * 1024 : 0) + (x_bytes > part_bytes ? x_bytes : part_bytes);
  static_assert(lds <= kGwLdsLimit, "LDS budget");
  auto kern = k_gemm_wide<M, NB, KW, RB, LDSCB>;
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)kGwLdsLimit);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((uint32_t)((a.d_out + a.rows_per_wg - 1) / a.rows_per_wg)), dim3(KW * kWave), lds, s, a);
  return hipGetLastError();
}

template <int M, int NB, int KW, bool LDSCB>
hipError_t run_wide_rb(const GemmWideArgs& a, int rb, hipStream_t s) {
  switch (rb) {
    case 1: return run_wide<M, NB, KW, 1, LDSCB>(a, s);
    case 2: return run_wide<M, NB, KW, 2, LDSCB>(a, s);
    case 3: return run_wide<M, NB, KW, 3, LDSCB>(a, s);
    default: return run_wide<M, NB, KW, 4, LDSCB>(a, s);
  }
}

}  // namespace

// Rows per launch: 64, or 32 where two 4096-entry codebooks take the LDS.
int32_t gemm_wide_rows(const Layer& L) { return L.B == 12 ? 32 : 64; }

bool gemm_wide_supported(const Layer& L, int32_t n) {
  return L.B > 8 && !L.packed && (L.M == 1 || L.M == 2) && n >= 1 && n <= gemm_wide_rows(L) &&
         (int64_t)L.G * L.M * 2 >= 16;
}

hipError_t launch_gemm_wide(const Layer& L, int32_t n, const uint16_t* x, uint16_t* y, hipStream_t s) {
  if (!gemm_wide_supported(L, n)) return hipErrorInvalidValue;
  // Rows split evenly over whole rounds of one workgroup per CU, at most four
  // blocks each.
  const int64_t cus = num_cus();
  const int64_t rounds = (L.d_out + 64 * cus - 1) / (64 * cus);
  const int32_t rows = (int32_t)((L.d_out + rounds * cus - 1) / (rounds * cus));
  const int r = (rows + 15) / 16;
  const GemmWideArgs a{static_cast<const uint8_t*>(L.codes), reinterpret_cast<const uint4*>(L.codebooks), L.scales,
                       reinterpret_cast<const uint4*>(x), y, L.d_out, L.G, n, L.B, rows};
  if (L.B == 12) {
    if (n <= 16) return run_wide_rb<2, 1, 4, true>(a, r, s);
    return run_wide_rb<2, 2, 4, true>(a, r, s);
  }
  if (L.M == 1) {
    if (n <= 16) return run_wide_rb<1, 1, 8, false>(a, r, s);
    if (n <= 32) return run_wide_rb<1, 2, 8, false>(a, r, s);
    return run_wide_rb<1, 4, 4, false>(a, r, s);
  }
  if (n <= 16) return run_wide_rb<2, 1, 8, false>(a, r, s);
  if (n <= 32) return run_wide_rb<2, 2, 8, false>(a, r, s);
  return run_wide_rb<2, 4, 4, false>(a, r, s);
}

}  // namespace aqlm
