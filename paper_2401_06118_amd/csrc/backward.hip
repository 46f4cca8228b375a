// Gradients through Eq. 2: the backward pass of y = x W^T with W in AQLM form,
// for fine-tuning codebooks and scales (Sec. 3, "Phase 2" and "Phase 3";
// App. "End-to-end fine-tuning").
//
// With G[i][c] = sum_t dy[t][i] x[t][c] (the weight gradient) and u[i][c] the
// fp32 sum of the codewords of row i, group c / 8 (Eq. 2 before the scale):
//   dC_m[e][k] += sum over (i, j) with b_ijm = e of s_i * G[i][8j + k]
//   ds_i       += sum_c G[i][c] * u[i][c]
//
// The weight gradient is never stored.  A workgroup of 8 waves computes a
// BM x BN tile of G on the matrix cores (v_mfma_f32_16x16x32_f16, the
// reduction runs over the tokens), then reduces it in sub-tiles of 2048
// (row, group) pairs, and goes on to its next tile.
//
// Contraction.  Both operands are stored token-major (dy [n][d_out],
// x [n][d_in]) but an MFMA lane needs 8 consecutive tokens of one row.  Stages
// of 64 tokens go from global memory straight into LDS, token-major
// (global_load_lds_dwordx4), and the fragments are read with the transposing
// LDS load (ds_read_b64_tr_b16: 16 lanes read 4 tokens x 16 columns, lane i
// receives column i's 4 tokens).  A fragment is two such reads; its 16 token
// rows (4 per slot of 8 tokens) would start in the same banks, so the 32-byte
// column pairs of token t are permuted by XOR with (t & 3) + 4 * ((t >> 3) & 1),
// on the global side of the load.  Interval and barriers as in the dense
// product (gemm_f16.hip): the fragments of a half-step are read under the
// MFMAs of the one before.
//
// Codebook gradient.  Each code's sum over its pairs would be one LDS atomic
// per element (16384 M per 128 x 128 tile; the LDS adds about two a clock and
// this was half of the kernel's time).  Instead the pairs are sorted by code
// first: one integer atomic per pair and codebook counts the codes and returns
// each pair's rank, a scan turns the counts into offsets, the pairs are
// written in order, and the thread that owns (codebook, code) adds the 8
// values of each of its pairs from LDS into its registers, which it keeps over
// all of the workgroup's tiles.  One global atomic per entry and workgroup at
// the end.  Values are fp32 throughout, scaled by s_i as they are staged.
//
// Scale gradient.  u is needed in the accumulators' layout (row 4 slot + r,
// column r16).  An MFMA puts it there: the A fragment of lane (row, slot) is
// the codeword of group slot / 2 and codebook slot % 2 (one 16-byte LDS
// gather), B the constant that maps (slot, k) to column 8 (slot / 2) + k; so
// the sum over two codebooks comes out in fp32, exact up to its rounding.
// Then G * u is added over the tile's columns in registers.  B's zeros meet
// every codeword of two groups, those past the row (code 0) included, and 0 times
// an infinity is a NaN: infinities and NaNs are staged as zeros, and a workgroup
// that met any adds their products apart, from the staged s_i * G.
//
// Summation order: the order of a code's pairs and the global atomics vary, so
// dC and ds agree with the oracle to fp32 accuracy but are not
// bit-reproducible from run to run.
//
// Measured against the previous kernel (128 x 128 tiles, transposing LDS
// stores, fp32 LDS atomics): 11008 x 4096 2x8 at 2048 tokens 1095 -> 245-265 us by
// box, at 256 tokens 558 -> 93; 4096 x 11008 4x8 at 2048 1566 -> 279; 4096 x 4096 8x8
// at 512 794 -> 120; 2320 x 5112 1x8 at 1515 195 -> 77; 1024 x 1096 2x8 at 4096
// 160 -> 30; a layer of one group 8.5 -> 11.4 (outputs cleared in both).  The
// contraction runs at about 1.0 PFLOP/s (11008 x 4096 2x8 at 2048, 4096 and 8192
// tokens 266, 428 and 792 us; matrix cores and LDS reads are of equal length with
// 64 x 64 waves); the rest is about 15 us per 256 x 128 tile and CU with two
// codebooks (sort, gather and stores through LDS, five barriers per sub-tile).
// Five to eight codebooks spill 19 to 50 registers.
#include "common.h"
#include "launch.h"
#include "lds_sync.h"

namespace aqlm {

namespace {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef short s4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4_t lds_s4_t;

constexpr int kBwWaves = 8;
constexpr int kBwThreads = kBwWaves * kWave;
constexpr int kBwK = 64;         // tokens per stage
constexpr int kBwStages = 2;
constexpr int kBwPairs = 2048;   // (row, group) pairs of a sub-tile
constexpr int kBwOff = 260;      // offsets kept per codebook (257, padded)
constexpr int kBwOwn = 32;       // pairs of a class that its thread adds alone

struct BwArgs {
  const uint8_t* codes;  // [d_out][G][M]
  const uint4* cb;       // [M][256]
  const uint16_t* scales;
  const uint16_t* x;   // [n][d_in]
  const uint16_t* dy;  // [n][d_out]
  float* dcb;          // [M][256][8], accumulated
  float* ds;           // [d_out], accumulated
  int32_t d_out;
  int32_t d_in;
  int32_t n;
  int32_t tiles_r;
  int32_t tiles_c;
  int32_t full;       // tiles that take all tokens; the others are split
  int32_t items;      // full + (tiles - full) x splits
  int32_t split_len;  // tokens per split, a multiple of kBwK
};

// 256 x 128 tiles (rows x inputs), 4 x 2 waves of 64 x 64 in blocks of 16 x 16; a
// sub-tile takes FMS of every wave's row blocks.  Measured against it (11008 x
// 4096 2x8, 2048 / 256 tokens, when it took 274 / 99 us on the same box): 128 x 128
// with waves of 64 x 32 350 / 106 us; 256 x 256 with waves of 128 x 64 520 / 149 us
// (spills).
struct BwTile {
  static constexpr int BM = 256, BN = 128, WM = 4, WN = 2, FMS = 2;
  static constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
  static constexpr int Q = FM / FMS;             // sub-tiles
  static constexpr int SR = WM * 16 * FMS;       // rows of a sub-tile
  static constexpr int GT = BN / 8;              // groups of a tile
  static constexpr int kStage = kBwK * (BM + BN);  // halfs of a stage: dy, then x
  static constexpr int kDyInsts = BM / 8;        // load instructions (1 KiB) of a stage's dy part
  static constexpr int kPer = (BM + BN) / 8 / kBwWaves;  // per wave
  static_assert(WM * WN == kBwWaves && SR * GT == kBwPairs && Q * FMS == FM, "tile");
  static_assert((BM + BN) / 8 % kBwWaves == 0, "whole load instructions per wave");
};

template <int M>
struct BwLds {  // byte offsets
  using T = BwTile;
  static constexpr size_t kCb = 0;                                    // [M][256] codewords
  static constexpr size_t kScales = kCb + (size_t)M * 4096;           // [BM] fp32
  static constexpr size_t kFlags = kScales + (size_t)T::BM * 4;       // [waves]
  static constexpr size_t kUnion = kFlags + (size_t)kBwWaves * 4;
  // either the stages ...
  static constexpr size_t kStages = (size_t)kBwStages * T::kStage * 2;
  // ... or a sub-tile's values, codes, counts / offsets and sorted pairs
  static constexpr size_t kG = kUnion;                                // [pair][8] fp32
  static constexpr size_t kCodes = kG + (size_t)kBwPairs * 32;        // [row][GT][M]
  static constexpr size_t kCount = kCodes + (size_t)kBwPairs * M;     // [M][260] uint32
  static constexpr size_t kList = kCount + (size_t)M * kBwOff * 4;    // [M][2048] uint16
  static constexpr size_t kDs = kList + (size_t)M * kBwPairs * 2;     // [WN][SR] fp32
  static constexpr size_t kSub = kDs + (size_t)T::WN * T::SR * 4 - kUnion;
  static constexpr size_t kTotal = kUnion + (kStages > kSub ? kStages : kSub);
  static_assert(kTotal <= 160 * 1024, "LDS budget");
  static_assert((size_t)M * 8192 <= kStages, "the final exchange fits in the stages");
};

__device__ __forceinline__ void bw_load_to_lds(const uint16_t* g, uint16_t* l) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(g, (lds_void_t*)l, 16, 0, 0);
#else
  (void)g;
  (void)l;
#endif
}

__device__ __forceinline__ s4_t tr_read(const uint16_t* l) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t*)l);
#else
  (void)l;
  return s4_t{};
#endif
}

// Waits for all of this wave's vector-memory loads, and for its LDS reads.
__device__ __forceinline__ void wait_all_loads() { __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8)); }
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8)); }

// Barrier ordered for the compiler only (the waits are explicit).
__device__ __forceinline__ void bw_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The fragments of one 32-token half of a stage.  po: this lane's offsets (in
// halfs) of its column blocks within the stage part.
template <int F, int W>
__device__ __forceinline__ void bw_read(const uint16_t* part, const int (&po)[F], int h, h8_t (&f)[F]) {
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const uint16_t* l = part + po[i] + h * 32 * W;
    const s4_t lo = tr_read(l), hi = tr_read(l + 4 * W);
    f[i] = __builtin_bit_cast(h8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

template <int FM, int FN>
__device__ __forceinline__ void bw_mfma(const h8_t (&af)[FM], const h8_t (&bf)[FN], f4_t (&acc)[FM][FN]) {
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
      acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[fm], bf[fn], acc[fm][fn], 0, 0, 0);
}

// One stage interval.  `rd` and `wr` are different stages: restrict parameters
// of an inlined function, so that the fragment reads do not wait for the loads
// just issued.
template <typename T, typename Issue>
__device__ __forceinline__ void bw_interval(const uint16_t* __restrict__ rd, uint16_t* __restrict__ wr, Issue&& issue,
                                            const int (&pa)[T::FM], const int (&pb)[T::FN],
                                            f4_t (&acc)[T::FM][T::FN], h8_t (&a1)[T::FM], h8_t (&b1)[T::FN]) {
  issue(wr);
  h8_t a0[T::FM], b0[T::FN];
  bw_read<T::FM, T::BM>(rd, pa, 0, a0);
  bw_read<T::FN, T::BN>(rd + kBwK * T::BM, pb, 0, b0);
  __builtin_amdgcn_sched_barrier(0);
  bw_mfma<T::FM, T::FN>(a1, b1, acc);
  __builtin_amdgcn_sched_barrier(0);
  bw_read<T::FM, T::BM>(rd, pa, 1, a1);
  bw_read<T::FN, T::BN>(rd + kBwK * T::BM, pb, 1, b1);
  __builtin_amdgcn_sched_barrier(0);
  bw_mfma<T::FM, T::FN>(a0, b0, acc);
}

// Zeros the halfs of a word that are infinities or NaNs; nonzero if there are any.
__device__ __forceinline__ uint32_t zero_nonfinite(uint32_t& w) {
  const uint32_t bad = ((w & 0x7C00u) == 0x7C00u ? 0xFFFFu : 0u) | ((w & 0x7C000000u) == 0x7C000000u ? 0xFFFF0000u : 0u);
  w &= ~bad;
  return bad;
}

// The sum of G * (infinities and NaNs of the codewords) over a thread's `nv`
// groups of one row: g is s * G of the row's groups (group e at e ^ swz), and the
// sign of G that of s and s * G (a zero s leaves it in the sign of the zero).
template <int M>
__device__ float special_scale_grad(const uint16_t* cb, const uint8_t* codes, const float* g, int first, int swz,
                                    int nv, float s) {
  float sum = 0.f;
#pragma unroll 1
  for (int b = 0; b < nv * M * 8; ++b) {
    const int e = b / (8 * M), m = b / 8 % M, k = b % 8;
    const uint16_t h = cb[(m * 256 + codes[e * M + m]) * 8 + k];
    if ((h & 0x7C00u) == 0x7C00u) {
      float v = g[((first + e) ^ swz) * 8 + k];
      if (s == 0.f) v = __builtin_copysignf(1.f, v);
      sum += __builtin_copysignf(1.f, s) * v * h2f(h);
    }
  }
  return sum;
}

template <int M>
__global__ __launch_bounds__(kBwThreads) void k_grad_cb(const BwArgs a) {
  using T = BwTile;
  using L = BwLds<M>;
  constexpr int BM = T::BM, BN = T::BN, FM = T::FM, FN = T::FN, FMS = T::FMS, GT = T::GT, PER = T::kPer;
  constexpr int kClassV = (M * 256 + kBwThreads - 1) / kBwThreads;  // (codebook, code) classes per thread
  constexpr int kQuads = GT / 4;                                    // threads per row in the sort
  extern __shared__ uint4 lds_u4[];
  char* const lds = reinterpret_cast<char*>(lds_u4);
  const uint4* const cbl = reinterpret_cast<const uint4*>(lds + L::kCb);
  float* const tsc = reinterpret_cast<float*>(lds + L::kScales);
  uint16_t* const stg = reinterpret_cast<uint16_t*>(lds + L::kUnion);
  float* const gl = reinterpret_cast<float*>(lds + L::kG);
  uint8_t* const tcodes = reinterpret_cast<uint8_t*>(lds + L::kCodes);
  uint32_t* const count = reinterpret_cast<uint32_t*>(lds + L::kCount);
  uint16_t* const list = reinterpret_cast<uint16_t*>(lds + L::kList);
  float* const dsl = reinterpret_cast<float*>(lds + L::kDs);

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int r16 = lane & 15, slot = lane >> 4;
  const int wm = wave % T::WM, wn = wave / T::WM;
  const int32_t G = a.d_in / 8;

  uint32_t bad = 0;  // halfs with all exponent bits set
  for (int e = tid; e < M * 256; e += kBwThreads) {
    uint4 v = a.cb[e];
    bad |= zero_nonfinite(v.x) | zero_nonfinite(v.y) | zero_nonfinite(v.z) | zero_nonfinite(v.w);
    reinterpret_cast<uint4*>(lds + L::kCb)[e] = v;
  }
  // (one word per wave; read in the sub-tiles, barriers later)
  const uint4* const flags = reinterpret_cast<const uint4*>(lds + L::kFlags);
  if (const bool any = __any(bad != 0); lane == 0) reinterpret_cast<uint32_t*>(lds + L::kFlags)[wave] = any;

  // Fragment read offsets: token 8 slot + r16 / 4 of the half (and 4 more for
  // the second read), column pair p of the tile at position p ^ g.
  const int g = (r16 >> 2) + 4 * (slot & 1);
  int pa[FM], pb[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
    pa[i] = (8 * slot + (r16 >> 2)) * BM + ((wm * FM + i) ^ g) * 16 + (r16 & 3) * 4;
#pragma unroll
  for (int i = 0; i < FN; ++i)
    pb[i] = (8 * slot + (r16 >> 2)) * BN + ((wn * FN + i) ^ g) * 16 + (r16 & 3) * 4;

  // B operand that deals codeword (slot / 2: group, slot % 2: codebook) to
  // columns 8 (slot / 2) + k
  h8_t deal;
#pragma unroll
  for (int k = 0; k < 8; ++k) deal[k] = (slot >> 1) * 8 + k == r16 ? (_Float16)1.f : (_Float16)0.f;

  float cacc[kClassV][8];
#pragma unroll
  for (int v = 0; v < kClassV; ++v)
#pragma unroll
    for (int k = 0; k < 8; ++k) cacc[v][k] = 0.f;

  // Items are dealt so that each XCD (workgroup b on XCD b % 8) takes
  // neighbouring tiles, whose operands its L2 then shares.
  uint32_t first = blockIdx.x;
  {
    const uint32_t n = gridDim.x, q = n / 8, r = n % 8, xcd = first % 8;
    first = xcd * q + (xcd < r ? xcd : r) + first / 8;
  }
  const int32_t tiles = a.tiles_r * a.tiles_c;
  for (int32_t item = (int32_t)first; item < a.items; item += (int32_t)gridDim.x) {
    int32_t tile = item, t0 = 0, t1 = a.n;
    if (item >= a.full) {
      const int32_t rem = tiles - a.full;
      tile = a.full + (item - a.full) % rem;
      t0 = (item - a.full) / rem * a.split_len;
      t1 = a.n - t0 < a.split_len ? a.n : t0 + a.split_len;
    }
    const int32_t i0 = (tile / a.tiles_c) * BM, c0 = (tile % a.tiles_c) * BN;
    const int32_t steps = (t1 - t0 + kBwK - 1) / kBwK;

    // Load instruction q = wave * PER + i of a stage fills 1 KiB: tokens of dy
    // (BM columns each) or of x.  Columns past the end read valid ones (their
    // results are dropped); tokens past the end are stored as zeros.
    auto issue_stage = [&](uint16_t* st, int32_t step) {
      const int32_t left = t1 - t0 - step * kBwK;  // tokens from this stage on
      const bool partial = left < kBwK;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int q = wave * PER + i;
        const bool is_dy = q < T::kDyInsts;
        const int per_tok = is_dy ? BM / 8 : BN / 8;      // 16-byte chunks per token
        const int e = (is_dy ? q : q - T::kDyInsts) * 64 + lane;
        const int tl = e / per_tok, c = e % per_tok;
        const int gg = (tl & 3) + 4 * ((tl >> 3) & 1);
        const int32_t width = is_dy ? a.d_out : a.d_in;
        int32_t col = (is_dy ? i0 : c0) + ((((c >> 1) ^ gg) << 1) | (c & 1)) * 8;
        col = col < width ? col : width - 8;
        const int32_t t = t0 + step * kBwK + tl;
        uint16_t* dst = st + (is_dy ? 0 : kBwK * BM) + (is_dy ? q : q - T::kDyInsts) * 512;
        const uint16_t* src = (is_dy ? a.dy : a.x) + (size_t)t * width + col;
        if (!partial) {
          bw_load_to_lds(src, dst);
        } else if (tl < left) {
          bw_load_to_lds(src, dst);
        } else {
          reinterpret_cast<uint4*>(dst)[lane] = make_uint4(0, 0, 0, 0);
        }
      }
    };

    // The codes of this thread's 4 pairs in every sub-tile (4 M bytes each)
    // and the tile's scales: loaded now, used after the contraction.
    uint32_t cw[T::Q][M];
    int nv[T::Q];  // valid groups of the four
    const int lr = tid / kQuads, gq = (tid % kQuads) * 4;
#pragma unroll
    for (int q = 0; q < T::Q; ++q) {
      const int32_t i = i0 + (lr / (16 * FMS)) * (16 * FM) + q * 16 * FMS + lr % (16 * FMS);
      const int32_t j = c0 / 8 + gq;
      int v = i < a.d_out ? G - j : 0;
      v = v < 0 ? 0 : (v < 4 ? v : 4);
      nv[q] = v;
#pragma unroll
      for (int w = 0; w < M; ++w) cw[q][w] = 0;
      const uint8_t* cp = a.codes + ((size_t)i * G + j) * M;
      if (v == 4 && (G * M) % 4 == 0) {
#pragma unroll
        for (int w = 0; w < M; ++w) cw[q][w] = reinterpret_cast<const uint32_t*>(cp)[w];
      } else {
#pragma unroll
        for (int b = 0; b < 4 * M; ++b)
          if (b < v * M) cw[q][b / 4] |= (uint32_t)cp[b] << (8 * (b % 4));
      }
    }
    float scv = 0.f;
    if (tid < BM && i0 + tid < a.d_out) scv = h2f(a.scales[i0 + tid]);

    f4_t acc[FM][FN];
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = f4_t{0.f, 0.f, 0.f, 0.f};
    h8_t a1[FM], b1[FN];  // (the interval before the first: zeros)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) a1[fm] = h8_t{};
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) b1[fn] = h8_t{};

    lds_barrier();  // (the previous tile's last sub-tile has been read)
    issue_stage(stg, 0);
    if (tid < BM) tsc[tid] = scv;
    wait_all_loads();
    wait_lds();
    bw_barrier();
    for (int32_t k = 0; k < steps; ++k) {
      bw_interval<T>(
          stg + (k & 1) * T::kStage, stg + ((k + 1) & 1) * T::kStage,
          [&](uint16_t* st) {
            if (k + 1 < steps) issue_stage(st, k + 1);
          },
          pa, pb, acc, a1, b1);
      wait_all_loads();
      wait_lds();
      bw_barrier();
    }
    bw_mfma<FM, FN>(a1, b1, acc);

    const uint4 fl0 = flags[0], fl1 = flags[1];
    const int special =
        __builtin_amdgcn_readfirstlane((int)(fl0.x | fl0.y | fl0.z | fl0.w | fl1.x | fl1.y | fl1.z | fl1.w));
    // sub-tiles
#pragma unroll
    for (int q = 0; q < T::Q; ++q) {
      if (q > 0) {
        if (i0 + q * 16 * FMS >= a.d_out) break;  // (no rows in it, nor in the next)
        lds_barrier();                            // (the previous sub-tile has been read)
      }
      // 1. s_i * G into LDS: pair (row, group) of the sub-tile at
      // row * GT + (group ^ 2 (row / 4 % 4)), so that the four slots of a
      // store hit different banks; codes; counters to zero.
#pragma unroll
      for (int f = 0; f < FMS; ++f) {
        const int row = wm * 16 * FMS + f * 16 + 4 * slot;
        const f4_t s4 = *reinterpret_cast<const f4_t*>(tsc + wm * 16 * FM + (q * FMS + f) * 16 + 4 * slot);
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const int col = (wn * FN + fn) * 16 + r16;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            gl[((row + r) * GT + ((col >> 3) ^ (2 * slot))) * 8 + (col & 7)] = s4[r] * acc[q * FMS + f][fn][r];
        }
      }
      for (int e = tid; e < M * kBwOff; e += kBwThreads) count[e] = 0;
#pragma unroll
      for (int w = 0; w < M; ++w) reinterpret_cast<uint32_t*>(tcodes)[(lr * GT + gq) * M / 4 + w] = cw[q][w];
      lds_barrier();

      // 2. ranks of this thread's pairs within their codes
      uint32_t rank[M][4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int b = e * M + m;
          const uint32_t code = (cw[q][b / 4] >> (8 * (b % 4))) & 0xFFu;
          rank[m][e] = 0;
          if (e < nv[q]) rank[m][e] = atomicAdd(&count[m * kBwOff + code], 1u);
        }
      // scale gradients of the sub-tile's rows
#pragma unroll
      for (int f = 0; f < FMS; ++f) {
        f4_t dsum = {0.f, 0.f, 0.f, 0.f};
        const int row16 = wm * 16 * FMS + f * 16;
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          f4_t u = {0.f, 0.f, 0.f, 0.f};
          const int grp = (wn * FN + fn) * 2 + (slot >> 1);
#pragma unroll
          for (int m2 = 0; m2 < M; m2 += 2) {
            const int m = m2 + (slot & 1);
            uint4 cwd = make_uint4(0, 0, 0, 0);
            if (M % 2 == 0 || m < M) cwd = cbl[m * 256 + tcodes[((row16 + r16) * GT + grp) * M + m]];
            u = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, cwd), deal, u, 0, 0, 0);
          }
          // (columns past d_in: G there belongs to other columns)
          if (c0 + (wn * FN + fn) * 16 + r16 < a.d_in) {
#pragma unroll
            for (int r = 0; r < 4; ++r) dsum[r] += acc[q * FMS + f][fn][r] * u[r];
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float v = dsum[r];
          v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
          v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
          v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));
          v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));
          if (r16 == 0) dsl[wn * T::SR + row16 + 4 * slot + r] = v;
        }
      }
      // what the codewords' infinities and NaNs add to them
      if (__builtin_expect(special != 0, 0)) {
        const int row = (lr / (16 * FMS)) * (16 * FM) + q * 16 * FMS + lr % (16 * FMS);
        const float v = special_scale_grad<M>(reinterpret_cast<const uint16_t*>(a.cb), tcodes + (lr * GT + gq) * M,
                                              gl + lr * GT * 8, gq, 2 * ((lr >> 2) & 3), nv[q], tsc[row]);
        if (v != 0.f) atomicAdd(&a.ds[i0 + row], v);
      }
      lds_barrier();

      // 3. counts to offsets: wave m takes codebook m, four codes per lane
      if (wave < M) {
        uint4* cp = reinterpret_cast<uint4*>(count + wave * kBwOff) + lane;
        const uint4 c = *cp;
        const uint32_t own = c.x + c.y + c.z + c.w;
        uint32_t inc = own;
#pragma unroll
        for (int off = 1; off < kWave; off *= 2) {
          const uint32_t o = __shfl_up(inc, off);
          if (lane >= off) inc += o;
        }
        const uint32_t ex = inc - own;
        *cp = make_uint4(ex, ex + c.x, ex + c.x + c.y, ex + c.x + c.y + c.z);
        if (lane == kWave - 1) count[wave * kBwOff + 256] = inc;
      }
      // (one atomic per row for all of the tile's columns)
      if (tid >= kBwThreads - T::SR) {
        const int row = tid - (kBwThreads - T::SR);
        const int32_t i = i0 + (row / (16 * FMS)) * (16 * FM) + q * 16 * FMS + row % (16 * FMS);
        float v = dsl[row];
#pragma unroll
        for (int w = 1; w < T::WN; ++w) v += dsl[w * T::SR + row];
        if (i < a.d_out) atomicAdd(&a.ds[i], v);
      }
      lds_barrier();

      // 4. the pairs in code order
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int b = e * M + m;
          const uint32_t code = (cw[q][b / 4] >> (8 * (b % 4))) & 0xFFu;
          if (e < nv[q])
            list[m * kBwPairs + count[m * kBwOff + code] + rank[m][e]] =
                (uint16_t)(lr * GT + ((gq + e) ^ (2 * ((lr >> 2) & 3))));
        }
      lds_barrier();

      // 5. each class's pairs, two at a time (M = 1: a class's list is shared
      // by two threads).  A thread adds up to kBwOwn of them (evenly used codes
      // have 8 on average).
      auto class_list = [&](int cls, uint32_t& p, uint32_t& end) __attribute__((always_inline)) {
        const uint32_t* off = count + (cls >> 8) * kBwOff + (cls & 255);
        p = off[0], end = off[1];
        if constexpr (M == 1) {
          const uint32_t mid = (p + end) / 2;
          if (tid < 256)
            end = mid;
          else
            p = mid;
        }
      };
      uint32_t longs = 0;
#pragma unroll
      for (int v = 0; v < kClassV; ++v) {
        const int cls = M == 1 ? tid & 255 : tid + v * kBwThreads;
        if (cls < M * 256) {
          const int m = cls >> 8;
          uint32_t p, end;
          class_list(cls, p, end);
          if (end - p > (uint32_t)kBwOwn) {
            longs |= 1u << v;
            end = p + kBwOwn;
          }
          const uint16_t* lp = list + m * kBwPairs;
          // the sub-tile's sum on its own first (shorter chains of rounding)
          f4_t sum0 = {0.f, 0.f, 0.f, 0.f}, sum1 = {0.f, 0.f, 0.f, 0.f};
          for (; p < end; p += 2) {
            const uint32_t p1 = p + 1 < end ? p + 1 : p;
            const f4_t* v0 = reinterpret_cast<const f4_t*>(gl + (uint32_t)lp[p] * 8);
            const f4_t* v1 = reinterpret_cast<const f4_t*>(gl + (uint32_t)lp[p1] * 8);
            const f4_t x0 = v0[0], x1 = v0[1], y0 = v1[0], y1 = v1[1];
            sum0 += x0;
            sum1 += x1;
            if (p + 1 < end) {
              sum0 += y0;
              sum1 += y1;
            }
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            cacc[v][k] += sum0[k];
            cacc[v][4 + k] += sum1[k];
          }
        }
      }
      // The rest of long lists: the whole wave adds one list after the other
      // (lane: half of a pair's values).  A thread alone would follow a serial
      // chain of LDS reads: one code for all pairs, 1024 x 1024 2x8 at 64 tokens,
      // 431 -> 34 us, a tenth of them one code 57 -> 21.
      if (__builtin_expect(__ballot(longs != 0) != 0, 0)) {
#pragma unroll 1
        for (int v = 0; v < kClassV; ++v) {
          for (uint64_t rest = __ballot((longs >> v) & 1); rest != 0; rest &= rest - 1) {
            const int owner = __builtin_ctzll(rest);
            const int cls = (M == 1 ? (wave * kWave) & 255 : wave * kWave + v * kBwThreads) + owner;
            uint32_t p, end;
            class_list(cls, p, end);
            const uint16_t* lp = list + (cls >> 8) * kBwPairs;
            f4_t part = {0.f, 0.f, 0.f, 0.f};
            for (uint32_t i = p + kBwOwn + (lane >> 1); i < end; i += kWave / 2)
              part += reinterpret_cast<const f4_t*>(gl)[(uint32_t)lp[i] * 2 + (lane & 1)];
            for (int off = 2; off < kWave; off *= 2)
#pragma unroll
              for (int k = 0; k < 4; ++k) part[k] += __shfl_xor(part[k], off);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const float pk = part[k % 4];
              const float w =
                  __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pk), k / 4));
#pragma unroll
              for (int u = 0; u < kClassV; ++u)
                if (u == v && lane == owner) cacc[u][k] += w;
            }
          }
        }
      }
    }
  }

  // The class sums, exchanged through LDS so that the atomics of a wave fall
  // on consecutive entries.
  float* const fin = reinterpret_cast<float*>(stg);
  lds_barrier();
  if (M > 1 || tid < 256) {
#pragma unroll
    for (int v = 0; v < kClassV; ++v)
      if (tid + v * kBwThreads < M * 256)
#pragma unroll
        for (int k = 0; k < 8; ++k) fin[(tid + v * kBwThreads) * 8 + k] = cacc[v][k];
  }
  lds_barrier();
  if (M == 1) {
    if (tid >= 256)
#pragma unroll
      for (int k = 0; k < 8; ++k) fin[(tid - 256) * 8 + k] += cacc[0][k];
    lds_barrier();
  }
  for (int e = tid; e < M * 2048; e += kBwThreads) {
    const float v = fin[e];
    if (v != 0.f) atomicAdd(&a.dcb[e], v);
  }
}

template <int M>
hipError_t run_grad(BwArgs a, hipStream_t s) {
  using T = BwTile;
  auto kern = k_grad_cb<M>;
  constexpr size_t lds = BwLds<M>::kTotal;
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds);
  if (e != hipSuccess) return e;
  a.tiles_r = (a.d_out + T::BM - 1) / T::BM;
  a.tiles_c = (a.d_in + T::BN - 1) / T::BN;
  const int64_t tiles = (int64_t)a.tiles_r * a.tiles_c, cus = num_cus();
  if (tiles >= (int64_t(1) << 31) - 4096) return hipErrorInvalidValue;
  // Whole rounds of one tile per CU take all tokens.  The tiles of a last,
  // partly filled round are split over the tokens to fill it (both gradients
  // are sums over tokens), with at least four stages per split: below that
  // the reduction of the tile, paid per split, outweighs the contraction
  // (1024 x 1096, 4096 tokens, 36 tiles: 81 us unsplit, 53 with 2, 39 with 4,
  // 36 with 7 splits).
  const int64_t rem = tiles % cus, steps = ((int64_t)a.n + kBwK - 1) / kBwK;
  int64_t splits = rem > 0 ? cus / rem : 1;
  if (splits > steps / 4) splits = steps / 4 > 1 ? steps / 4 : 1;
  const int64_t len = (steps + splits - 1) / splits;
  splits = (steps + len - 1) / len;
  a.full = (int32_t)(splits > 1 ? tiles - rem : tiles);
  a.split_len = (int32_t)(len * kBwK < a.n ? len * kBwK : a.n);
  const int64_t items = a.full + (tiles - a.full) * splits;
  a.items = (int32_t)items;
  hipLaunchKernelGGL(kern, dim3((uint32_t)(items < cus ? items : cus)), dim3(kBwThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace

bool backward_supported(const Layer& L) { return L.B == 8 && L.M >= 1 && L.M <= 8 && L.d_out % 8 == 0; }

hipError_t launch_backward(const Layer& L, int32_t n, const uint16_t* x, const uint16_t* dy, float* dcb, float* ds,
                           hipStream_t s) {
  if (!backward_supported(L) || n < 1) return hipErrorInvalidValue;
  const BwArgs a{static_cast<const uint8_t*>(L.codes), reinterpret_cast<const uint4*>(L.codebooks), L.scales, x, dy,
                 dcb, ds, L.d_out, L.d_in, n, 0, 0, 0, 0, 0};
  switch (L.M) {
    case 1: return run_grad<1>(a, s);
    case 2: return run_grad<2>(a, s);
    case 3: return run_grad<3>(a, s);
    case 4: return run_grad<4>(a, s);
    case 5: return run_grad<5>(a, s);
    case 6: return run_grad<6>(a, s);
    case 7: return run_grad<7>(a, s);
    case 8: return run_grad<8>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace aqlm
