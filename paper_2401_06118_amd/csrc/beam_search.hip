// Phase 1 of AQLM: beam search over the codes (Sec. 3, "Phase 1: Beam search
// for codes").  Each output row is independent (the objective is additive
// over rows):
//   L(b) = (w - what) H (w - what)^T,  H = X X^T,
//   what[8j + t] = s * sum_m C_m[b_jm][t]   (exact reconstruction).
// A beam of at most k configurations of the row's codes starts as the row's
// current codes.  A step takes one position (j, m) (groups in order,
// codebooks in order within a group) and scores, for every configuration in
// the beam and every codeword e of codebook m, the configuration with code
// (j, m) set to e; the k distinct configurations of least loss form the next
// beam (ties: earlier beam entry, then smaller e).  The result is the best
// configuration after the given number of sweeps.
//
// Scores are incremental, as the paper describes: with h = H r kept per
// configuration (r = w - what), z = h_j and delta = s (C_e - C_o) on group j,
//   L' = L - 2 delta . z + delta H_jj delta^T.
// Expanded in C_e this is
//   L' = [L + 2 s C_o.z + s^2 C_o H_jj C_o] + s^2 q_e - 2 s C_e.(z + s H_jj C_o),
//   q_e = C_e H_jj C_e,
// so a candidate costs one 8-wide inner product, and q_e is shared by every
// row and entry.  The expansion cancels, so it is evaluated in fp64 (vector
// fp64 runs at the rate of unpacked fp32 here); the k winners' loss changes
// are then taken in the delta form, so keeping a code keeps the loss exactly.
//
// Work split: a workgroup of 8 waves searches up to 8 rows, one wave per row
// in the steps, all waves in the phases the rows share.  Per group j:
//   steps (one wave per row, no workgroup barrier): lane (b, t) holds
//     component t of entry b's z and of its change of the group; lane l
//     scores codewords l + 64 v.  A score carries its candidate's index in
//     its 11 lowest mantissa bits (relative 2^-41), so one 64-bit minimum
//     over the wave finds value and winner.
//   update (all waves): h of every entry takes its ancestor's h minus
//     H[:, group j] times the group's total change, one rank-8 product per
//     group on the matrix cores (v_mfma_f32_16x16x4_f32, fp32 in and out);
//     its result layout holds four consecutive inputs of one entry per lane,
//     so h moves as 16-byte LDS accesses, in place.  The group's rows of H
//     are loaded before the steps and shared by all rows of the workgroup.
//     q of the next group is computed in the same phase.
// Two LDS barriers per group.
//
// Which entries would produce equal configurations at a position is tracked
// exactly: lane (a, b) counts the positions at which entries a and b differ;
// they agree everywhere but at this position when the count without it is 0,
// and then the later entry's candidates repeat the earlier's.
//
// A step records (parent, code) per entry; the codes of the entries are
// traced back once per sweep.  Within a sweep an unvisited position still has
// the code of the entry's configuration at the sweep's start.
//
// Bound by vector instruction issue (about 2000 instructions per wave and
// group, two waves per SIMD).  Measured, one sweep, against one 256-thread
// workgroup per row scoring the delta form per candidate: 4096 x 1024 2x8 beam
// 4 38.8 -> 3.5 ms, 1193 x 472 4x8 beam 4 8.9 -> 1.2 ms, 4096 x 2048 2x8 beam
// 8 394 -> 37 ms, 512 x 4096 2x8 beam 4 108 -> 11 ms, 200 x 1024 1x8 beam 1
// 2.08 -> 0.71 ms.  The two exact losses take 0.74 of the 3.5 ms.  Rows that
// end on other codes than a search in 64 bits: 0.02-0.16 % where fp32 scores
// gave 0.1-0.6 %.
#include "common.h"
#include "launch.h"
#include "lds_sync.h"

namespace aqlm {

namespace {

constexpr int kBsWaves = 8;
constexpr int kBsThreads = kBsWaves * kWave;
constexpr int kBsMaxRows = kBsWaves;  // one wave per row in the steps
constexpr int kBsMaxBeam = 8;
constexpr size_t kBsLdsLimit = 160 * 1024;

struct BeamArgs {
  const float* w;       // [d_out][d_in]
  const float* h;       // [d_in][d_in]
  uint8_t* codes;       // [d_out][G][M], read and overwritten
  const uint16_t* cb;   // [M][256][8]
  const uint16_t* scales;
  float* loss;          // [d_out] (may be null)
  int32_t d_out;
  int32_t d_in;
  int32_t G;
  int32_t M;
  int32_t beam;
  int32_t sweeps;
  int32_t rows;  // rows per workgroup
};

// LDS of a workgroup (byte offsets, 16-byte aligned).  kp: the beam rounded
// up to a power of two.
struct BeamLds {
  uint32_t cb;     // [M][256] codewords, fp16
  uint32_t q;      // [M][256] fp64
  uint32_t hjj;    // [2][64] fp64, groups alternate
  uint32_t red;    // [waves][rows] fp64
  uint32_t h;      // [rows][slots][stride] fp32
  uint32_t hcode;  // [rows][ncode][kp] code chosen by entry n at a position
  uint32_t hpar;   // [rows][ncode] parents, packed (1 byte up to 4 entries, else 4)
  uint32_t cod;    // [rows][copies][ncode] codes at the start of the sweep
  uint32_t p;      // [rows][kp][8] fp64, 2 s (z + s H_jj C_o)
  uint32_t base;   // [rows][kp] fp64
  uint32_t delta;  // [rows][kp][8] fp32, minus the group's change
  uint32_t anc;    // [rows][kp] ancestor at the group's start, 0xFF: none
  uint32_t total;
  int32_t slots;   // h vectors per row (at least two: the second holds r while the losses are computed)
  int32_t stride;  // floats per h vector: 4 modulo 64, so that the entries of a tile start in different banks
};

__host__ __device__ inline BeamLds beam_lds(int d_in, int G, int M, int beam, int kp, int sweeps, int rows) {
  BeamLds L;
  const uint32_t ncode = (uint32_t)(G * M), R = (uint32_t)rows;
  const uint32_t copies = sweeps > 1 ? (uint32_t)beam : 1u;
  L.slots = beam > 1 ? beam : 2;
  L.stride = (d_in + 63) / 64 * 64 + 4;
  uint32_t o = 0;
  auto take = [&o](uint32_t bytes) {
    const uint32_t at = o;
    o += (bytes + 15u) & ~15u;
    return at;
  };
  L.cb = take((uint32_t)M * 4096u);
  L.q = take((uint32_t)M * 2048u);
  L.hjj = take(2u * 64u * 8u);
  L.red = take((uint32_t)kBsWaves * R * 8u);
  L.h = take(R * (uint32_t)L.slots * (uint32_t)L.stride * 4u);
  L.hcode = take(R * ncode * (uint32_t)kp);
  L.hpar = take(R * ncode * (kp > 4 ? 4u : 1u));
  L.cod = take(R * copies * ncode);
  L.p = take(R * (uint32_t)kp * 64u);
  L.base = take(R * (uint32_t)kp * 8u);
  L.delta = take(R * (uint32_t)kp * 32u);
  L.anc = take(R * (uint32_t)kp);
  L.total = o;
  return L;
}

int beam_kp(int beam) { return beam <= 1 ? 1 : (beam <= 2 ? 2 : (beam <= 4 ? 4 : 8)); }

// Wave-level ordering of LDS accesses between lanes (a wave's LDS operations
// execute in order; this keeps the compiler from caching across them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// min with a quiet NaN as "no value" (the instruction returns the other
// operand; of a signaling NaN it would make a NaN)
__device__ __forceinline__ double min64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

__device__ __forceinline__ double no_key() { return __builtin_bit_cast(double, 0x7FF8000000000000ull); }

template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double lane64(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Minimum over the wave, the same in every lane.
__device__ __forceinline__ double wave_min64(double v) {
  v = min64(v, dpp64<0xB1>(v));   // lanes xor 1
  v = min64(v, dpp64<0x4E>(v));   // xor 2
  v = min64(v, dpp64<0x141>(v));  // half rows of 8
  v = min64(v, dpp64<0x140>(v));  // rows of 16
  const double a = min64(lane64(v, 0), lane64(v, 16)), b = min64(lane64(v, 32), lane64(v, 48));
  return lane64(min64(a, b), 0);
}

// Sum over the 8 lanes that share an entry, the same in each of them.
__device__ __forceinline__ double sum8(double v) {
  v += dpp64<0xB1>(v);
  v += dpp64<0x4E>(v);
  v += dpp64<0x141>(v);
  return v;
}

__device__ __forceinline__ void codeword64(const uint4& v, double (&c)[8]) {
  c[0] = (double)h2f(v.x & 0xFFFF); c[1] = (double)h2f(v.x >> 16);
  c[2] = (double)h2f(v.y & 0xFFFF); c[3] = (double)h2f(v.y >> 16);
  c[4] = (double)h2f(v.z & 0xFFFF); c[5] = (double)h2f(v.z >> 16);
  c[6] = (double)h2f(v.w & 0xFFFF); c[7] = (double)h2f(v.w >> 16);
}

template <int KP>
__global__ __launch_bounds__(kBsThreads) void k_beam(const BeamArgs a) {
  constexpr int kTileRows = 16 / KP;                         // rows per 16-entry tile of the update
  constexpr int kTiles = (kBsMaxRows + kTileRows - 1) / kTileRows;
  constexpr int kPre = 8;                                    // 16-input tiles per wave loaded before the steps
  constexpr int kParBits = KP > 4 ? 4 : 2;                   // bits per parent in the history
  extern __shared__ uint4 lds_u4[];
  char* const lds = reinterpret_cast<char*>(lds_u4);
  const int d_in = a.d_in, G = a.G, M = a.M, beam = a.beam;
  const int ncode = G * M;
  const BeamLds L = beam_lds(d_in, G, M, beam, KP, a.sweeps, a.rows);
  const int copies = a.sweeps > 1 ? beam : 1;
  const uint4* const cbl = reinterpret_cast<const uint4*>(lds + L.cb);
  const uint16_t* const cbh = reinterpret_cast<const uint16_t*>(lds + L.cb);
  double* const ql = reinterpret_cast<double*>(lds + L.q);
  double* const hjj = reinterpret_cast<double*>(lds + L.hjj);
  double* const red = reinterpret_cast<double*>(lds + L.red);
  float* const hl = reinterpret_cast<float*>(lds + L.h);
  const int hrow_stride = L.slots * L.stride;

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int32_t row0 = (int32_t)blockIdx.x * a.rows;
  const int R = a.d_out - row0 < a.rows ? a.d_out - row0 : a.rows;

  for (int e = tid; e < M * 256; e += kBsThreads)
    reinterpret_cast<uint4*>(lds + L.cb)[e] = reinterpret_cast<const uint4*>(a.cb)[e];
  for (int r = 0; r < R; ++r)
    for (int e = tid; e < ncode; e += kBsThreads)
      reinterpret_cast<uint8_t*>(lds + L.cod)[r * copies * ncode + e] = a.codes[(size_t)(row0 + r) * ncode + e];
  lds_barrier();

  // Exact losses of the rows' configurations (codes in copy 0): r = w - what
  // into slot 1, h = H r accumulated in fp64 over the rows of H (H is
  // symmetric: row q holds column q, read contiguously and shared by the
  // workgroup's rows), written to slot 0 as fp32 when asked, and the loss
  // r . h in fp64, summed in a fixed order.
  auto exact_losses = [&](bool write_h) {
    for (int r = 0; r < R; ++r) {
      const uint8_t* cfg = reinterpret_cast<const uint8_t*>(lds + L.cod) + r * copies * ncode;
      const float s = h2f(a.scales[row0 + r]);
      float* rs = hl + r * hrow_stride + L.stride;
      for (int c = tid; c < d_in; c += kBsThreads) {
        const int j = c >> 3, t = c & 7;
        float u = 0.f;
        for (int m = 0; m < M; ++m) {
          const float v = h2f(cbh[(m * 256 + cfg[j * M + m]) * 8 + t]);
          u = (m == 0) ? v : u + v;
        }
        rs[c] = a.w[(size_t)(row0 + r) * d_in + c] - s * u;
      }
    }
    lds_barrier();
    // (NR: rows held in registers, the workgroup's rounded up to a power of
    // two; the reads of a row that does not exist repeat the last one's, so
    // that all reads of a step are in flight together)
    auto pass = [&](auto nr) {
      constexpr int NR = decltype(nr)::value;
      const float* rs[NR];
      double lpart[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        rs[r] = hl + (r < R ? r : R - 1) * hrow_stride + L.stride;
        lpart[r] = 0.0;
      }
      for (int cb = 0; cb < d_in; cb += 2 * kBsThreads) {
        const int c0 = cb + tid, c1 = c0 + kBsThreads;
        const int g0 = c0 < d_in ? c0 : d_in - 1, g1 = c1 < d_in ? c1 : d_in - 1;
        double acc0[NR], acc1[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) acc0[r] = acc1[r] = 0.0;
        // four rows of H at a time, the next four in flight meanwhile
        float x0[4], x1[4];
        auto load4 = [&](int q, float (&y0)[4], float (&y1)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            y0[i] = a.h[(size_t)(q + i) * d_in + g0];
            y1[i] = a.h[(size_t)(q + i) * d_in + g1];
          }
        };
        load4(0, x0, x1);
        for (int q = 0; q < d_in; q += 4) {
          float n0[4], n1[4];
          load4(q + 4 < d_in ? q + 4 : 0, n0, n1);
          f4_t rq[NR];
#pragma unroll
          for (int r = 0; r < NR; ++r) rq[r] = *reinterpret_cast<const f4_t*>(rs[r] + q);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double y0 = (double)x0[i], y1 = (double)x1[i];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
              acc0[r] = __builtin_fma(y0, (double)rq[r][i], acc0[r]);
              acc1[r] = __builtin_fma(y1, (double)rq[r][i], acc1[r]);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            x0[i] = n0[i];
            x1[i] = n1[i];
          }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          if (r < R) {
            float* h0 = hl + r * hrow_stride;
            if (c0 < d_in) {
              lpart[r] += (double)h0[L.stride + c0] * acc0[r];
              if (write_h) h0[c0] = (float)acc0[r];
            }
            if (c1 < d_in) {
              lpart[r] += (double)h0[L.stride + c1] * acc1[r];
              if (write_h) h0[c1] = (float)acc1[r];
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        double v = lpart[r];
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0 && r < R) red[wave * a.rows + r] = v;
      }
    };
    if (R > 4)
      pass(IntC<8>{});
    else if (R > 2)
      pass(IntC<4>{});
    else if (R > 1)
      pass(IntC<2>{});
    else
      pass(IntC<1>{});
    lds_barrier();
  };
  auto row_loss = [&](int r) {
    double v = red[r];
    for (int w = 1; w < kBsWaves; ++w) v += red[w * a.rows + r];
    return v;
  };

  exact_losses(true);

  // State of this wave's row.  Lane (b, t) = (lane / 8, lane % 8): entry b's
  // loss, its configuration at the sweep's start (root) and ancestor at the
  // group's start (anc), component t of z and of the group's change; lane
  // (x, y): the number of positions at which entries x and y differ.
  const bool has_row = wave < R;
  const int b8 = lane >> 3, t8 = lane & 7;
  const double s = has_row ? (double)h2f(a.scales[row0 + wave]) : 0.0;
  double loss = has_row ? row_loss(wave) : 0.0;
  double z = 0.0, change = 0.0;
  int root = 0, anc = 0, cnt = 0;
  int nb = has_row ? 1 : 0;
  uint8_t* const cod = reinterpret_cast<uint8_t*>(lds + L.cod) + wave * copies * ncode;
  uint8_t* const hcode = reinterpret_cast<uint8_t*>(lds + L.hcode) + (size_t)wave * ncode * KP;
  uint8_t* const hpar = reinterpret_cast<uint8_t*>(lds + L.hpar) + (size_t)wave * ncode * (KP > 4 ? 4 : 1);
  double* const pl = reinterpret_cast<double*>(lds + L.p) + wave * KP * 8;
  double* const bl = reinterpret_cast<double*>(lds + L.base) + wave * KP;
  float* const dl = reinterpret_cast<float*>(lds + L.delta) + wave * KP * 8;
  uint8_t* const al = reinterpret_cast<uint8_t*>(lds + L.anc) + wave * KP;

  // q of every codeword of every codebook for the group whose H_jj sits at `hb`
  auto group_q = [&](const double* hb) {
    for (int e = tid; e < M * 256; e += kBsThreads) {
      double c[8];
      codeword64(cbl[e], c);
      double q = 0.0;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) v = __builtin_fma(hb[t * 8 + u], c[u], v);
        q = __builtin_fma(c[t], v, q);
      }
      // A codeword that is not finite has a quiet NaN for q, so that its scores
      // are quiet NaNs and absent from every minimum.  An infinite score would
      // become a signaling NaN with its index in the mantissa, and take the
      // score it is compared with out of the minimum.
      ql[e] = __builtin_fabs(q) < __builtin_huge_val() ? q : no_key();
    }
  };
  // element tid of H_jj of group j (tid < 64)
  auto load_hjj = [&](int j) -> float {
    return a.h[(size_t)(8 * j + (tid >> 3)) * d_in + 8 * j + (tid & 7)];
  };
  float hj_next = 0.f;
  if (tid < 64) {
    hjj[tid] = (double)load_hjj(0);
    hj_next = load_hjj(G > 1 ? 1 : 0);
  }
  lds_barrier();
  group_q(hjj);
  lds_barrier();

  const int ctiles = (d_in + 15) / 16;
  const int etiles = (R + kTileRows - 1) / kTileRows;
  for (int sw = 0; sw < a.sweeps; ++sw) {
    for (int j = 0; j < G; ++j) {
      const int gi = sw * G + j;
      const double* const hb = hjj + (gi & 1) * 64;
      // The group's 8 rows of H for this wave's first input tiles (tile
      // wave + 8 i: lane (c, k) holds H[8j + k][c] and H[8j + 4 + k][c]),
      // in flight during the steps.
      float ha[kPre][2];
#pragma unroll
      for (int i = 0; i < kPre; ++i) {
        int c = (wave + kBsWaves * i) * 16 + (lane & 15);
        c = c < d_in ? c : d_in - 1;
        const float* hp = a.h + (size_t)(8 * j + (lane >> 4)) * d_in + c;
        ha[i][0] = hp[0];
        ha[i][1] = hp[(size_t)4 * d_in];
      }
      if (tid < 64) {
        hjj[((gi + 1) & 1) * 64 + tid] = (double)hj_next;
        hj_next = load_hjj(j + 2 < G ? j + 2 : (j + 2 - G) % G);
      }
      __builtin_amdgcn_sched_barrier(0);

      if (nb > 0) {
        double hrow[8];  // row t of H_jj
#pragma unroll
        for (int u = 0; u < 8; ++u) hrow[u] = hb[t8 * 8 + u];
        z = b8 < nb ? (double)hl[wave * hrow_stride + b8 * L.stride + 8 * j + t8] : 0.0;
        change = 0.0;
        anc = b8;
        for (int m = 0; m < M; ++m) {
          const int pos = j * M + m;
          // entry terms: the old codeword's, then p and the constant
          const int old = b8 < nb ? cod[root * ncode + pos] : 0;
          {
            double oc[8];
            codeword64(cbl[m * 256 + old], oc);
            double ho = 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) ho = __builtin_fma(hrow[u], oc[u], ho);
            const double ot = (double)h2f(cbh[(m * 256 + old) * 8 + t8]);
            const double cst = sum8(s * ot * (2.0 * z + s * ho));
            const double l0 = lane64(loss, 0);
            if (b8 < KP) {
              pl[b8 * 8 + t8] = 2.0 * s * (z + s * ho);
              if (t8 == 0) bl[b8] = (loss - l0) + cst;
            }
          }
          // entries whose candidates repeat an earlier entry's
          const int old_y = __shfl(old, t8 * 8);
          const int rest = cnt - (old != old_y ? 1 : 0);
          uint64_t dup = __ballot(b8 < t8 && t8 < nb && rest == 0);
          dup |= dup >> 32;
          dup |= dup >> 16;
          dup |= dup >> 8;
          wave_sync();

          // scores of codewords lane + 64 v against every entry
          double key[KP][4];
          {
            double c[4][8], sq[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              codeword64(cbl[m * 256 + v * 64 + lane], c[v]);
              sq[v] = s * s * ql[m * 256 + v * 64 + lane];
            }
#pragma unroll
            for (int b = 0; b < KP; ++b) {
              if (b < nb && !((dup >> b) & 1)) {
                double p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) p[u] = pl[b * 8 + u];
                const double base = bl[b];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  double k = base + sq[v];
#pragma unroll
                  for (int u = 0; u < 8; ++u) k = __builtin_fma(-c[v][u], p[u], k);
                  // the index, complemented under a negative value so that
                  // equal scores order by (entry, code)
                  uint64_t ku = __builtin_bit_cast(uint64_t, k);
                  const uint32_t neg = (uint32_t)((int32_t)(uint32_t)(ku >> 32) >> 31);
                  const uint32_t idx = (uint32_t)((b << 8) | (v << 6) | lane) ^ neg;
                  const uint32_t lo = ((uint32_t)ku & ~2047u) | (idx & 2047u);
                  key[b][v] = __builtin_bit_cast(double, (ku & 0xFFFFFFFF00000000ull) | lo);
                }
              } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) key[b][v] = no_key();
              }
            }
          }
          // the k least: one wave minimum each
          int mine = b8 << 8;  // (lanes of entries that do not exist keep themselves)
          uint64_t pcodes = 0;
          uint32_t ppar = 0;
          int nn = 0;
          // (least key per entry and lane; removing a winner touches one entry)
          double em[KP];
#pragma unroll
          for (int b = 0; b < KP; ++b) em[b] = min64(min64(key[b][0], key[b][1]), min64(key[b][2], key[b][3]));
          for (int n = 0; n < beam; ++n) {
            double lm = em[0];
#pragma unroll
            for (int b = 1; b < KP; ++b) lm = min64(lm, em[b]);
            const double w = wave_min64(lm);
            if (!(w < __builtin_huge_val())) break;  // fewer candidates than k
            const uint64_t wu = __builtin_bit_cast(uint64_t, w);
            const uint32_t neg = (uint32_t)((int32_t)(uint32_t)(wu >> 32) >> 31);
            const int widx = (int)(((uint32_t)wu ^ neg) & 2047u);
            if (b8 == n) mine = widx;
            pcodes |= (uint64_t)(widx & 255) << (8 * n);
            ppar |= (uint32_t)(widx >> 8) << (kParBits * n);
            ++nn;
#pragma unroll
            for (int b = 0; b < KP; ++b) {
              if (widx >> 8 == b) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  const uint64_t ku = __builtin_bit_cast(uint64_t, key[b][v]);
                  const uint32_t hi = key[b][v] == w ? 0x7FF80000u : (uint32_t)(ku >> 32);  // (a quiet NaN)
                  key[b][v] = __builtin_bit_cast(double, ((uint64_t)hi << 32) | (uint32_t)ku);
                }
                em[b] = min64(min64(key[b][0], key[b][1]), min64(key[b][2], key[b][3]));
              }
            }
          }
          nb = nn;
          if (nn == 0) break;  // (no finite score: the row keeps its codes)
          // the new entries, from their parents'
          const int par = mine >> 8, code = mine & 255;
          const int from = par * 8 + t8;
          const int oldp = __shfl(old, par * 8);
          double nc[8], oc[8];
          codeword64(cbl[m * 256 + code], nc);
          codeword64(cbl[m * 256 + oldp], oc);
          double hd = 0.0;
#pragma unroll
          for (int u = 0; u < 8; ++u) hd = __builtin_fma(hrow[u], s * (nc[u] - oc[u]), hd);
          const double dt = s * ((double)h2f(cbh[(m * 256 + code) * 8 + t8]) -
                                 (double)h2f(cbh[(m * 256 + oldp) * 8 + t8]));
          const double zp = __shfl(z, from);
          loss = __shfl(loss, from) + sum8(dt * (hd - 2.0 * zp));
          z = zp - hd;
          change = __shfl(change, from) + dt;
          root = __shfl(root, from);
          anc = __shfl(anc, from);
          const int par_y = __shfl(par, t8 * 8), code_y = __shfl(code, t8 * 8);
          cnt = __shfl(rest, par * 8 + par_y) + (code != code_y ? 1 : 0);
          if (lane < KP) hcode[(size_t)pos * KP + lane] = (uint8_t)(pcodes >> (8 * lane));
          if (lane == 0) {
            if constexpr (KP > 4)
              reinterpret_cast<uint32_t*>(hpar)[pos] = ppar;
            else
              hpar[pos] = (uint8_t)ppar;
          }
        }
      }
      if (has_row && b8 < KP) {
        dl[b8 * 8 + t8] = -(float)change;
        if (t8 == 0) al[b8] = b8 < nb ? (uint8_t)anc : (uint8_t)0xFF;
      }
      lds_barrier();

      // update: entry i of a tile is entry i % KP of row i / KP of the tile
      {
        float bd[kTiles][2];
        uint32_t src[kTiles], dst[kTiles];
        bool live[kTiles];
#pragma unroll
        for (int e = 0; e < kTiles; ++e) {
          const int r = e * kTileRows + (lane & 15) / KP, n = (lane & 15) % KP;
          live[e] = false;
          src[e] = dst[e] = 0;
          bd[e][0] = bd[e][1] = 0.f;
          if (e < etiles && r < R) {
            const float* dr = reinterpret_cast<const float*>(lds + L.delta) + (r * KP + n) * 8;
            const int an = reinterpret_cast<const uint8_t*>(lds + L.anc)[r * KP + n];
            if (an != 0xFF) {
              live[e] = true;
              bd[e][0] = dr[lane >> 4];
              bd[e][1] = dr[4 + (lane >> 4)];
              src[e] = (uint32_t)(r * hrow_stride + an * L.stride);
              dst[e] = (uint32_t)(r * hrow_stride + n * L.stride);
            }
          }
        }
        auto tile = [&](int ct, float h0, float h1) {
          const int c = ct * 16 + 4 * (lane >> 4);
#pragma unroll
          for (int e = 0; e < kTiles; ++e) {
            if (e < etiles) {
              const bool ok = live[e] && c < d_in;
              f4_t acc = {0.f, 0.f, 0.f, 0.f};
              if (ok) acc = *reinterpret_cast<const f4_t*>(hl + src[e] + c);
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(h0, bd[e][0], acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(h1, bd[e][1], acc, 0, 0, 0);
              // (every lane of the tile has read before any lane writes)
              if (ok) *reinterpret_cast<f4_t*>(hl + dst[e] + c) = acc;
            }
          }
        };
#pragma unroll
        for (int i = 0; i < kPre; ++i)
          if (wave + kBsWaves * i < ctiles) tile(wave + kBsWaves * i, ha[i][0], ha[i][1]);
        for (int ct = wave + kBsWaves * kPre; ct < ctiles; ct += kBsWaves) {
          int c = ct * 16 + (lane & 15);
          c = c < d_in ? c : d_in - 1;
          const float* hp = a.h + (size_t)(8 * j + (lane >> 4)) * d_in + c;
          tile(ct, hp[0], hp[(size_t)4 * d_in]);
        }
      }
      group_q(hjj + ((gi + 1) & 1) * 64);
      lds_barrier();
    }
    // Trace the entries' codes back (lane n: entry n; after the last sweep
    // only the best entry's are needed).
    if (nb > 0 && lane < (sw + 1 < a.sweeps ? nb : 1)) {
      int n = lane;
      for (int pos = ncode - 1; pos >= 0; --pos) {
        cod[lane * ncode + pos] = hcode[(size_t)pos * KP + n];
        uint32_t pp;
        if constexpr (KP > 4)
          pp = reinterpret_cast<const uint32_t*>(hpar)[pos];
        else
          pp = hpar[pos];
        n = (int)((pp >> (kParBits * n)) & ((1u << kParBits) - 1u));
      }
    }
    root = b8;
    wave_sync();
  }
  lds_barrier();
  for (int r = 0; r < R; ++r)
    for (int e = tid; e < ncode; e += kBsThreads)
      a.codes[(size_t)(row0 + r) * ncode + e] = reinterpret_cast<const uint8_t*>(lds + L.cod)[r * copies * ncode + e];
  // The exact loss of the result (the running losses add one change per step).
  if (a.loss) {
    exact_losses(false);
    if (tid < R) a.loss[row0 + tid] = (float)row_loss(tid);
  }
}

template <int KP>
hipError_t run_beam(const BeamArgs& a, size_t lds, hipStream_t s) {
  auto kern = k_beam<KP>;
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)kBsLdsLimit);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((uint32_t)((a.d_out + a.rows - 1) / a.rows)), dim3(kBsThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace

// The documented limit of the search (two generations of h and codes per
// entry within one workgroup's LDS).  The kernel keeps one generation, so
// every accepted size fits with at least one row per workgroup.
bool beam_search_fits(int32_t d_in, int32_t M, int32_t beam) {
  if (beam < 1 || beam > kBsMaxBeam || M < 1 || M > 8 || d_in > 4096) return false;
  const size_t k = (size_t)beam, state = 2 * k * d_in * 4 + (size_t)M * 4096 + 64 * 4 + k * 64 + k * 16 + k * 32 + 32 +
                                         k * 8 + 64 + 2 * k * ((size_t)d_in / 8) * M;
  return ((state + 15) & ~(size_t)15) <= kBsLdsLimit;
}

hipError_t launch_beam_search(const float* w, const float* h, uint8_t* codes, const uint16_t* codebooks,
                              const uint16_t* scales, int32_t d_out, int32_t d_in, int32_t M, int32_t beam,
                              int32_t sweeps, float* loss, hipStream_t s) {
  if (!beam_search_fits(d_in, M, beam)) return hipErrorInvalidValue;
  const int kp = beam_kp(beam), G = d_in / 8;
  // As many rows per workgroup as the LDS holds (they share the loads of H
  // and q), then no more than spread the rows over whole rounds of the CUs.
  int rows = kBsMaxRows;
  while (rows > 1 && beam_lds(d_in, G, M, beam, kp, sweeps, rows).total > kBsLdsLimit) --rows;
  const int64_t cus = num_cus();
  const int64_t rounds = (d_out + rows * cus - 1) / (rows * cus);
  rows = (int)((d_out + rounds * cus - 1) / (rounds * cus));
  const size_t lds = beam_lds(d_in, G, M, beam, kp, sweeps, rows).total;
  if (lds > kBsLdsLimit) return hipErrorInvalidValue;
  const BeamArgs a{w, h, codes, codebooks, scales, loss, d_out, d_in, G, M, beam, sweeps, rows};
  switch (kp) {
    case 1: return run_beam<1>(a, lds, s);
    case 2: return run_beam<2>(a, lds, s);
    case 4: return run_beam<4>(a, lds, s);
    default: return run_beam<8>(a, lds, s);
  }
}

}  // namespace aqlm
