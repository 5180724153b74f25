// FP64 forward body of the matrix-bound orders (Np = 56, 84, 120): D in
// registers, outputs stored straight from the accumulators.
//
// The product of a 16-column tile is formed with the columns as the matrix
// rows: A = u (lane (n, g): column n), B = D^T (lane (n, g): output node n of
// the tile), so lane (n, g) of a result holds node n of columns 4q + g.  Three
// tiles of one 16-node chunk (D_r, D_s, D_t) leave (D_r u, D_s u, D_t u) of a
// node in one lane: the combine with the geometric factors is lane-local, and
// a store of 16 consecutive nodes is a 128-byte run, which needs no staging
// through LDS and no barrier.  (With the columns in the lanes a store would be
// 16 runs of 32 bytes.)
//
// Np = 16 NFULL + NREM.  The last NREM nodes (8 or 4) of the three directions
// share remainder tiles: NREM = 8: D_r | D_s in one tile, D_t in a second;
// NREM = 4: D_r | D_s | D_t in one.  A row rotation (DPP) brings the three
// derivatives of a node together.
//
// The k order of the product is free as long as both operands agree: k-steps
// 2p and 2p + 1 take nodes 8p + 2g and 8p + 2g + 1, so that a lane reads both
// operands as 16-byte pairs (D from memory once per launch, u from LDS).
//
// Bound: the FP64 products (order 6: 84, order 7: 90 of 64 cycles per wave and
// column tile), with vector work, which does not overlap them, at about a
// tenth; at order 5 past the memory-side cache, the memory.  One barrier per
// iteration: u is double-buffered, and nothing else is shared (order 6: the
// exchanged tiles, used one iteration later).  No branch and no register
// spill may sit between the loads and their use: a spill's reload waits for
// every store in flight, which took order 6 from 328 back to 386 us.
//
// Measured against the chunk-register body it replaced (u staged, outputs
// assembled in LDS, two barriers per iteration), F = 3: order 6, K = 2^17
// 387 -> 326 us (67 % of the FP64 matrix peak; on another card, warmer, 389 ->
// 347), 3e6 nodal values 49.3 -> 35.6
// us, K = 157, F = 17 17.3 -> 10.5 us; order 7, K = 2^16 322 -> 294 us (75 %),
// 3e6 57.8 -> 51.2 us, K = 157, F = 1 18.0 -> 13.1 us.
#pragma once

#include <type_traits>

#include "dgvol_device.hpp"
#include "dgvol_forward.hpp"

namespace dgvol {

// The value of lane (l + R) % 16 of each row of 16 lanes (DPP row_ror by 16 - R).
template <int R>
__device__ __forceinline__ double row_rot_f64(double v) {
  static_assert(R > 0 && R < 16, "rotation within a row");
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned int)b, 0x120 + 16 - R, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned int)(b >> 32), 0x120 + 16 - R, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned int)hi << 32) | (unsigned int)lo);
}

// 16-byte pair at 8-byte alignment
typedef double f64x2_u __attribute__((ext_vector_type(2), aligned(8)));

template <int NP, int WAVES = 8>
struct DirectShape {
  static constexpr int WPB = WAVES;
  static constexpr int NTH = WAVE * WPB;
  static constexpr int NFULL = NP / 16;   // 16-node chunks
  static constexpr int NREM = NP % 16;    // remaining nodes
  static constexpr int KS = NP / 4;       // k-steps
  static constexpr int KP = KS / 2;       // pairs of k-steps
  static constexpr bool KODD = KS % 2 != 0;
  // Waves that share a column tile ("units").  Np = 120: units 0..6 take a
  // chunk each, unit 7 the remainder tiles.  Np = 56: units 0..2 a chunk, unit
  // 3 the remainder.  Np = 84: units 0..3 a chunk each plus one tile of the
  // last chunk or the remainder (XCH), so every wave carries 4 tiles.
  static constexpr int UNITS = NP == 120 ? 8 : 4;
  static constexpr bool XCH = NFULL == UNITS + 1;
  static constexpr int NT = XCH ? 4 : 3;  // tiles (of D operands) per wave
  static constexpr int HALVES = WPB / UNITS;
  static constexpr int LD = NP + 2;       // row stride of the staged u: pairs stay aligned, rows spread over banks
  static constexpr int GLD = 10;          // row stride of the staged geometric factors
  static constexpr int NGB = 4;           // buffers of them (the exchanged tiles use them one iteration later)
  static constexpr int XLD = 18;
  static constexpr int KL = KODD ? NT : 0;  // D operands per lane kept in LDS (the odd k-step)
  static_assert(NP % 4 == 0 && (NREM == 4 || NREM == 8), "nodes come in whole k-steps");
  static_assert(XCH ? NREM == 4 : NFULL == UNITS - 1, "units cover the chunks");
};

// Staging of u: a thread moves one 16-byte pair of a row per pass, RPP rows a
// pass, so that its LDS and memory offsets advance by constants.  Threads past
// RPP rows repeat the next pass's first row (the same words to the same
// place); rows past the iteration's columns land in rows of their own.
template <int NP, int WPB, int TILES>
struct DirectStage {
  using S = DirectShape<NP, WPB>;
  static constexpr int COLS = TILES * 16;
  static constexpr int RPP = S::NTH / (NP / 2);
  static constexpr int NLD = (COLS + RPP - 1) / RPP;
  static constexpr int ROWS = NLD * RPP + 1;
  static_assert((S::NTH - 1) / (NP / 2) <= RPP, "at most one repeated row");
  static constexpr int U = ROWS * S::LD;                          // doubles per u buffer
  static constexpr int G = COLS * S::GLD;                         // per buffer of geometric factors
  static constexpr int X = S::XCH ? TILES * 4 * 16 * S::XLD : 0;  // per buffer of exchanged tiles
  static constexpr int DL = S::KL * S::WPB * WAVE;                // D operands kept in LDS
};

// column tiles per iteration of the workgroup: TILES / HALVES per group of UNITS waves
template <int NP, int WPB, int TILES>
constexpr int fwd_f64_direct_lds() {
  using T = DirectStage<NP, WPB, TILES>;
  return (2 * T::U + T::S::NGB * T::G + 2 * T::X + T::DL) * 8;
}

template <int NP, int WPB, int TILES>
__device__ __forceinline__ void fwd_f64_direct_body(const FwdArgs<double>& p, uint32_t bid, uint32_t nblk, char* lds) {
  using S = DirectShape<NP, WPB>;
  using T = DirectStage<NP, WPB, TILES>;
  constexpr int KP = S::KP, NT = S::NT, LD = S::LD, GLD = S::GLD;
  constexpr int CT = TILES / S::HALVES;  // column tiles per wave per iteration
  static_assert(CT * S::HALVES == TILES, "whole tiles per group of waves");
  constexpr int COLS = T::COLS;
  constexpr int NG = (COLS * 9 + S::NTH - 1) / S::NTH;
  double* us = reinterpret_cast<double*>(lds);       // [2][ROWS][LD]
  double* gs = us + 2 * T::U;                        // [NGB][COLS][GLD]
  double* xch = gs + S::NGB * T::G;                  // [2][TILES][4][16][XLD]
  double* dl = xch + 2 * T::X;                       // [KL][WPB][WAVE]
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = w / S::UNITS;
  // Np = 56: the lighter unit 3 sits on another SIMD in the second half
  const int unit = (w % S::UNITS + (S::XCH ? 0 : h)) % S::UNITS;
  const bool rem = !S::XCH && unit == S::NFULL;  // this wave's tiles are the remainder tiles

  // ---- this wave's D operands, for the whole launch
  f64x2 dp[NT][KP];
  double* dlw = dl + w * WAVE + lane;  // operand x in LDS: dlw[x * WPB * WAVE]
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    int a, i;
    bool ok = true;
    if (t < 3 && !rem) {
      a = t;
      i = 16 * unit + n;
    } else if (S::XCH && unit < 3) {  // tile of the last chunk
      a = unit;
      i = 16 * (S::NFULL - 1) + n;
    } else {                          // remainder tile
      const int x = (S::XCH ? 0 : 16 * t) + n;
      a = x / S::NREM;
      i = 16 * S::NFULL + x % S::NREM;
      ok = a < 3;
    }
    const double* row = p.D + (int64_t)((ok ? a : 0) * NP + i) * NP;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
      const f64x2 v = *reinterpret_cast<const f64x2_u*>(row + 8 * q + 2 * g);
      dp[t][q] = ok ? v : f64x2{0.0, 0.0};
    }
    if constexpr (S::KODD) {
      const double v = row[4 * (S::KS - 1) + g];
      dlw[t * S::WPB * WAVE] = ok ? v : 0.0;  // read back by this lane only
    }
  }

  // ---- staging
  const uint32_t nsup = (p.ntiles + TILES - 1) / TILES;
  f64x2 ur[T::NLD];
  double gr[NG];
  const uint32_t F = p.F;
  const float invF = 1.0f / (float)F;
  auto load = [&](uint32_t s) __attribute__((always_inline)) {
    const bool any = s < nsup;
    const uint32_t c0 = any ? s * COLS : 0u;
    // (c0 is a column whatever s is: no guard that the subtraction's no-wrap flag could
    // come from, see cols_left, which costs order 7 0.7 %)
    const uint32_t left = min((uint32_t)COLS, p.ncols - c0);
    const uint32_t ncl = any ? left : 0u;
    const __amdgpu_buffer_rsrc_t ru = buffer_range(p.u + (int64_t)c0 * NP, ncl * NP * 8u);
    const int tid = opaque(threadIdx.x);
    const uint32_t off = (uint32_t)((tid / (NP / 2)) * NP + 2 * (tid % (NP / 2))) * 8u;
#pragma unroll
    for (int q = 0; q < T::NLD; ++q)
      ur[q] = __builtin_bit_cast(f64x2, buffer_load_vec<double, 2>(ru, off + (uint32_t)(q * T::RPP * NP) * 8u));
    const uint32_t k0 = c0 / F, r0 = c0 - k0 * F;
    const __amdgpu_buffer_rsrc_t rg = buffer_range(p.G + (int64_t)k0 * 9, any ? ((c0 + ncl - 1) / F - k0 + 1) * 72u : 0u);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const uint32_t x = (uint32_t)(tid + S::NTH * q);
      const uint32_t c = x / 9u;  // column of the iteration
      // its element, (r0 + c) / F: r0 < F, so at most one step for F >= COLS; exact in float below that
      const uint32_t e = F >= COLS ? (r0 + c >= F ? 1u : 0u) : (uint32_t)(((float)(r0 + c) + 0.5f) * invF);
      gr[q] = buffer_load_f64(rg, (e * 9u + x - 9u * c) * 8u);
    }
  };
  // unconditional writes: no branch, so the wait for the loads counts exactly
  // the stores issued after them
  auto stage = [&](uint32_t it) __attribute__((always_inline)) {
    const int tid = opaque(threadIdx.x);
    double* ub = us + (it & 1u) * T::U + (tid / (NP / 2)) * LD + 2 * (tid % (NP / 2));
#pragma unroll
    for (int q = 0; q < T::NLD; ++q) *reinterpret_cast<f64x2*>(ub + q * T::RPP * LD) = ur[q];
    double* gb = gs + (it % S::NGB) * T::G;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int x = tid + S::NTH * q;
      // words past the last column go to a pad word of some row
      gb[x < COLS * 9 ? (x / 9) * GLD + x % 9 : (x % COLS) * GLD + 9] = gr[q];
    }
  };

  // The three outputs of a node whose derivatives are (r, s, t): gk its column's
  // factors, off its byte offset in the tile of columns c0 .. c0 + ncl - 1 (past
  // the range: dropped).
  auto emit = [&](const __amdgpu_buffer_rsrc_t (&ro)[3], const double* gk, uint32_t off, double r, double s,
                  double t) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 3; ++b) buffer_store_f64(ro[b], off, gk[b] * r + gk[3 + b] * s + gk[6 + b] * t);
  };
  auto planes = [&](__amdgpu_buffer_rsrc_t (&ro)[3], uint32_t c0) __attribute__((always_inline)) {
    const uint32_t ncl = cols_left(p.ncols, c0, 16);
#pragma unroll
    for (int b = 0; b < 3; ++b) ro[b] = buffer_range(p.out + b * p.plane + (int64_t)c0 * NP, ncl * NP * 8u);
  };
  // exchanged tiles (last chunk, remainder) of iteration `it`, columns from col0
  auto emit_xch = [&](uint32_t it, uint32_t col0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int tp = h * CT + j;
      __amdgpu_buffer_rsrc_t ro[3];
      planes(ro, col0 + 16 * tp);
      const int l = opaque(lane);
      const double* xb = xch + (it & 1u) * T::X + tp * (4 * 16 * S::XLD);
      const double* gb = gs + (it % S::NGB) * T::G + tp * 16 * GLD;
      {
        const int col = 4 * unit + (l >> 4);
        const double* xr = xb + col * S::XLD + (l & 15);
        emit(ro, gb + col * GLD, (uint32_t)(col * NP + 16 * (S::NFULL - 1) + (l & 15)) * 8u, xr[0], xr[16 * S::XLD],
             xr[32 * S::XLD]);
      }
      if (unit == (int)(it & 3u)) {
        const int col = l >> 2, m = l & 3;
        const double* xr = xb + (48 + col) * S::XLD + m;
        emit(ro, gb + col * GLD, (uint32_t)(col * NP + 16 * S::NFULL + m) * 8u, xr[0], xr[4], xr[8]);
      }
    }
  };

  uint32_t it = 0;
  uint32_t st = bid;
  load(st);
  stage(0);
  for (; st < nsup; st += nblk, ++it) {
    const uint32_t col0 = st * COLS;
    __syncthreads();
    load(st + nblk);
    if constexpr (S::XCH) {
      if (it > 0) emit_xch(it - 1, col0 - nblk * COLS);
    }
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int tp = h * CT + j;
      const double* ub = us + (it & 1u) * T::U + tp * 16 * LD + n * LD + 2 * g;
      f64x4 acc[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
      auto run = [&](auto NTc) __attribute__((always_inline)) {
        constexpr int NTT = decltype(NTc)::value;
        f64x2 cur = *reinterpret_cast<const f64x2*>(ub);
        double tail = 0.0, dtl[NT];
#pragma unroll
        for (int q = 0; q < KP; ++q) {
          f64x2 nxt = cur;
          if (q + 1 < KP) {
            nxt = *reinterpret_cast<const f64x2*>(ub + 8 * (q + 1));
          } else if constexpr (S::KODD) {
            tail = (ub - g)[4 * (S::KS - 1)];
#pragma unroll
            for (int t = 0; t < NTT; ++t) dtl[t] = dlw[t * S::WPB * WAVE];
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) {
#pragma unroll
            for (int t = 0; t < NTT; ++t)
              acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[e], dp[t][q][e], acc[t], 0, 0, 0);
          }
          cur = nxt;
        }
        if constexpr (S::KODD) {
#pragma unroll
          for (int t = 0; t < NTT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(tail, dtl[t], acc[t], 0, 0, 0);
        }
      };
      __amdgpu_buffer_rsrc_t ro[3];
      planes(ro, col0 + 16 * tp);
      const int l = opaque(lane);
      const double* gk = gs + (it % S::NGB) * T::G + tp * 16 * GLD + (l >> 4) * GLD;
      const uint32_t off = (uint32_t)((l >> 4) * NP + (l & 15)) * 8u;
      if (rem) {
        run(std::integral_constant<int, 2>{});
        // lanes past the remainder: an offset past every range
        const uint32_t o = (l & 15) < S::NREM ? off + 16 * S::NFULL * 8u : 0x40000000u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          emit(ro, gk + 4 * q * GLD, o + (uint32_t)(4 * q * NP) * 8u, acc[0][q], row_rot_f64<8>(acc[0][q]), acc[1][q]);
      } else {
        run(std::integral_constant<int, NT>{});
        const uint32_t o = off + (uint32_t)(16 * unit) * 8u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          emit(ro, gk + 4 * q * GLD, o + (uint32_t)(4 * q * NP) * 8u, acc[0][q], acc[1][q], acc[2][q]);
        if constexpr (S::XCH) {
          double* xb = xch + (it & 1u) * T::X + (tp * 4 + unit) * (16 * S::XLD) + (l >> 4) * S::XLD + (l & 15);
#pragma unroll
          for (int q = 0; q < 4; ++q) xb[4 * q * S::XLD] = acc[NT - 1][q];
        }
      }
    }
    stage(it + 1);
  }
  if constexpr (S::XCH) {
    if (it > 0) {
      __syncthreads();
      emit_xch(it - 1, (st - nblk) * COLS);
    }
  }
}

}  // namespace dgvol
