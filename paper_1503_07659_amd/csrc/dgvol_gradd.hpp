// Cotangent of the reference differentiation matrices, FP64.
//
// The forward map is linear in D, so for a cotangent gout of the three output
// planes the cotangent of D is a sum over every element column c = (k, f):
//   W_a[c][i]   = sum_b G[k][3a+b] gout[b][c][i]
//   gD[a][i][j] = sum_c W_a[c][i] u[c][j]
// i.e. per direction one contraction [Np x ncols] . [ncols x Np] whose
// reduction runs over the (long) column axis.  It runs on the FP64 matrix
// cores with the columns as the MFMA k dimension, four per k-step:
//
//   * lane (n, g) of a wave owns column 4s + g of k-step s and nodes n, 16 + n,
//     ... of it, loads u and gout there (128-byte runs), forms W in its
//     registers and feeds both to the products as they are: the A operand of a
//     16-row tile is W at the lane's node of that tile, the B operand u.
//     Nothing passes through LDS, and waves meet no barrier until the end;
//   * the last Np mod 16 nodes do not pad a tile: they are held as quads of 4
//     (registers Q below) whose products run as v_mfma_f64_4x4x4f64 (four
//     4 x 4 blocks, 16 cycles against 64 for a 16 x 16 tile);
//   * loads run two k-steps ahead (u one, each register reloaded right after
//     its products, where registers are short: Np >= 84, and Np = 56 with the
//     rows split over two workgroups, where the second step's u spilled and
//     every other step waited for all loads in flight: 1e6 nodal values 20.9 ->
//     20.0 us, 1.8e6 25.8 -> 24.1); the 9 geometric factors of a column come as
//     one load (lane n of its 16-lane row takes factor n) and are handed to the
//     row by DPP broadcasts;
//   * the waves of a workgroup share its column range; a wave holds every
//     output (up to Np = 35) or those of a group of rows (Np = 56: 2 groups,
//     84: 4, 120: 8) in its accumulators.  Groups of rows, not directions:
//     gout is then read once and only u by every group.  (One workgroup per
//     direction read everything three times: order 5, K = 2^19 took 1049 us
//     instead of 632.)  At the end the waves of one group add their accumulators through
//     LDS in order, and the workgroup writes one partial sum to work[part]; a
//     second kernel adds the partial sums in a fixed order.
//
// The partition depends only on (K, F, Np), never on the device, and every
// sum runs in a fixed order, so the result is reproducible bit for bit.
//
// Bound: the memory up to Np = 35, the FP64 products from 56 (2400 / 5328 /
// 10848 matrix cycles per 4 columns at Np = 56 / 84 / 120, no padding), with
// W and the broadcasts beside them (a fifth at Np = 56).  Measured against the
// kernels it replaced (W and u staged through LDS, one barrier per 16 to 128
// columns; order 5: producer and consumer waves), F = 3, both kernels of a
// call: 2e7 nodal values, order 1 177 -> 157 us, 2 191 -> 149, 3 203 -> 140, 4
// 219 -> 129, 6 305 -> 209, 7 483 -> 281; order 5, K = 2^19 635 -> 632; 3e5
// values, order 4 17.4 -> 10.9, 5 20 -> 13, 6 29 -> 17, 7 33 -> 25.
#pragma once

#include <type_traits>

#include "dgvol_device.hpp"

namespace dgvol {

// Columns per partial sum, at least (the workspace holds one per GD_UNIT).
constexpr int GD_UNIT = 128;

// Bound on the number of partial sums the workspace holds (a function of Np only).
__host__ __device__ constexpr uint32_t gd_maxpart(int np) { return np <= 35 ? 1024u : 512u; }

template <int NP>
struct GdShape {
  // Np = 10: one padded tile; else whole 16-node tiles and up to two quads
  static constexpr int NF = NP == 10 ? 1 : NP / 16;
  static constexpr int NQ = NP == 10 ? 0 : (NP % 16 + 3) / 4;
  static_assert(NQ <= 2, "at most two quads");
  // Row groups of a workgroup's waves.  Np = 56: tiles 0, 1; tile 2 and the
  // quads.  Np = 84: tile g and one direction of tile 4 (g < 3), tile 3 and
  // the quad.  Np = 120: tile g (g < 7), the quads.  A workgroup is 4 waves, or
  // 8 (two per SIMD) with row groups.  More registers a wave (one per SIMD,
  // 512) would need fewer groups, but the compiler then moves accumulators
  // between the two register files around the products: 5 times slower.
  static constexpr int NRG = NP == 120 ? 8 : NP == 84 ? 4 : NP == 56 ? 2 : 1;
  static constexpr int WPB = NRG > 1 ? 8 : 4;
  static constexpr int SLICES = WPB / NRG;       // column slices
  static constexpr int NTH = WAVE * WPB;
  // Two kinds of groups: the last one (with the quads) and the others, which
  // differ by their first tile (and extra direction) only.  First tile of group
  // g; whole tiles, extra tile or -1, and quads of a kind.
  __host__ __device__ static constexpr int t0(int g) { return NP == 56 ? 2 * g : g; }
  static constexpr int nt(bool last) {
    return NP == 56 ? (last ? 1 : 2) : NP == 84 ? 1 : NP == 120 ? (last ? 0 : 1) : NF;
  }
  static constexpr int xt(bool last) { return NP == 84 && !last ? 4 : -1; }
  static constexpr bool rq(bool last) { return NQ > 0 && last; }
  // doubles per lane of a group's accumulators for nd directions
  static constexpr int acc(bool last, int nd) {
    return nd * nt(last) * (4 * NF + NQ) + (xt(last) >= 0 ? 4 * NF + NQ : 0) + (rq(last) ? nd * (NQ * NF + NQ) : 0);
  }
  // of them, those that pass through LDS at a time (Np = 84: all would be 166 KiB; 120: 90 KiB
  // let one wave a SIMD in, and the compiler then used both register files, see above)
  static constexpr int passes(int nd) { return NP >= 84 && nd == 3 ? 2 : 1; }
  static constexpr int acc_pass(bool last, int nd) { return (acc(last, nd) + passes(nd) - 1) / passes(nd); }
  static constexpr int lds_group(int nd) {
    return (acc_pass(true, nd) > acc_pass(false, nd) ? acc_pass(true, nd) : acc_pass(false, nd)) * WAVE;
  }
  // Column slices where rs workgroups share the row groups: at Np = 120 four workgroups
  // of two groups have a second slice each, so that their four waves have half the columns.
  static constexpr int slices(int rs) { return NP == 120 && rs == 4 ? 2 : SLICES; }
  // (each row group of a workgroup has its own)
  static constexpr int lds_doubles(int nd, int rs) { return slices(rs) > 1 ? NRG / rs * lds_group(nd) : 1; }
  // waves per SIMD the registers allow; partial sums: as many as run at once on
  // 256 CUs (a constant, not read from the device)
  static constexpr int WPS = NP <= 20 ? 4 : 2;
  static constexpr uint32_t MAXPART = 256u * 4u * WPS / WPB;
  static_assert(MAXPART <= gd_maxpart(NP), "the workspace holds every partial sum");
};

struct GdArgs {
  const double* G;
  const double* u;
  const double* gout;
  double* work;      // [npart][3][Np][Np]
  uint32_t ncols;    // K * F
  uint32_t F;
  int64_t plane;     // K * F * Np
  uint32_t npart;
};

template <int I, int N, typename Fn>
__device__ __forceinline__ void gd_static_for(Fn&& fn) {
  if constexpr (I < N) {
    fn(std::integral_constant<int, I>{});
    gd_static_for<I + 1, N>(fn);
  }
}

// A wave's share: row group rg_ (LAST: of the last kind), directions a0 .. a0 + ND - 1, over column
// slice `slice` of the part.
template <int NP, bool LAST, int ND, int RS>
__device__ __forceinline__ void gd_role(const GdArgs& p, uint32_t part, uint32_t slice, int rg_, int a0, double* lds) {
  using S = GdShape<NP>;
  constexpr int NF = S::NF, NQ = S::NQ;
  constexpr int NR = S::nt(LAST), XT = S::xt(LAST);
  constexpr bool X = XT >= 0;
  constexpr int NRQ = S::rq(LAST) ? NQ : 0;
  const int T0 = S::NRG > 1 ? S::t0(rg_) : 0;  // first tile
  const int XD = ND == 1 ? 0 : rg_;            // direction of the extra tile (past a0)
  const bool xon = ND == 3 || rg_ == 0;        // (one direction: the first group takes it)
  constexpr bool ONE = NP == 4;       // one quad, nothing else: 16 columns a k-step
  constexpr int CPS = ONE ? 16 : 4;   // columns per k-step
  constexpr int NG = NR + (X ? 1 : 0) + NRQ;  // gout registers per plane: tiles, extra tile, quads
  constexpr int NU = NF + NQ;                 // u registers: tiles, quads
  constexpr int DEPTH = 2;            // gout register sets
  constexpr int UD = NP >= 84 || (NP == 56 && ND == 3 && RS == 2) ? 1 : DEPTH;  // u register sets
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;

  // this wave's columns, from c_lo: its slice of the part's range, which comes
  // in units of a whole number of DEPTH k-steps per slice
  constexpr uint32_t SLICES = S::slices(RS);
  constexpr uint32_t UNIT = SLICES * DEPTH * CPS;
  static_assert(GD_UNIT % UNIT == 0, "every part has a unit");
  const uint32_t nunits = (p.ncols + UNIT - 1) / UNIT;
  const uint32_t u_lo = (uint32_t)((uint64_t)part * nunits / p.npart);
  const uint32_t u_hi = (uint32_t)((uint64_t)(part + 1) * nunits / p.npart);
  // (wave-uniform for certain: the buffer descriptors are built from them)
  const uint32_t per_wave = __builtin_amdgcn_readfirstlane((u_hi - u_lo) * (DEPTH * CPS));
  const uint32_t c_lo = __builtin_amdgcn_readfirstlane(u_lo * UNIT) + slice * per_wave;
  const uint32_t nsteps = per_wave / CPS;

  // The lane's byte offsets within a k-step's columns.  A quad register holds
  // node 16 NF + 4 q + (lane & 3) in lane group of 4 lanes b = (lane >> 2) & 3,
  // with q = 0 for one quad; for two, q = b & 1 in the first register and the
  // other quad in the second.  Nodes past Np: past every range.
  const int cl = ONE ? lane >> 2 : g;  // column within the k-step
  constexpr uint32_t OUT = 0x40000000u;
  uint32_t base_off = NP == 10 && n >= NP ? OUT : (uint32_t)(cl * NP + n) * 8u;  // tile t: + 128 t
  uint32_t tile_off = base_off + 128u * (uint32_t)T0;
  uint32_t qoff[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int node = 16 * NF + (NQ == 2 ? ((n & 7) ^ (4 * q)) : (n & 3));
    qoff[q] = node < NP ? (uint32_t)(cl * NP + node) * 8u : OUT;
  }

  // element (relative to the slice's first) and position in it of the lane's
  // column, advanced by CPS columns a step
  const uint32_t F = p.F;
  const uint32_t k_lo = c_lo / F;
  uint32_t ke, kr;
  {
    const uint32_t c = c_lo - k_lo * F + (uint32_t)cl;
    ke = c / F;
    kr = c - ke * F;
  }
  const uint32_t dk = CPS / F, dr = CPS % F;
  const uint32_t n_el = c_lo < p.ncols ? (min(c_lo + per_wave, p.ncols) - 1u) / F - k_lo + 1u : 0u;
  const __amdgpu_buffer_rsrc_t rG = buffer_range(p.G + (int64_t)k_lo * 9, n_el * 72u);
  const uint32_t gf = ND == 3 ? (uint32_t)min(n, 8) : (uint32_t)(3 * a0 + min(n, 2));  // lane n of a row takes factor 3 a0 + n

  double raw[DEPTH][3][NG], ru[UD][NU], rg[DEPTH][ONE ? 9 : 1];
  auto columns = [&](uint32_t s, int64_t& base, uint32_t& nb) __attribute__((always_inline)) {
    const uint32_t c0 = c_lo + s * CPS;
    const uint32_t ncl = s < nsteps ? cols_left(p.ncols, c0, CPS) : 0u;
    base = (int64_t)(ncl ? c0 : 0u) * NP;
    nb = ncl * NP * 8u;
  };
  auto range_u = [&](uint32_t s) __attribute__((always_inline)) {
    int64_t base;
    uint32_t nb;
    columns(s, base, nb);
    return buffer_range(p.u + base, nb);
  };
  auto load_u = [&](const __amdgpu_buffer_rsrc_t& bu, int d, int x) __attribute__((always_inline)) {
    ru[d][x] = buffer_load_f64(bu, x < NF ? base_off + 128u * x : qoff[x < NF ? 0 : x - NF]);
  };
  auto load_g = [&](uint32_t s, auto Dc) __attribute__((always_inline)) {
    constexpr int d = decltype(Dc)::value;
    int64_t base;
    uint32_t nb;
    columns(s, base, nb);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const __amdgpu_buffer_rsrc_t bg = buffer_range(p.gout + b * p.plane + base, nb);
#pragma unroll
      for (int t = 0; t < NR; ++t) raw[d][b][t] = buffer_load_f64(bg, tile_off + 128u * t);
      if constexpr (X) raw[d][b][NR] = buffer_load_f64(bg, base_off + 128u * XT);
#pragma unroll
      for (int q = 0; q < NRQ; ++q) raw[d][b][NG - NRQ + q] = buffer_load_f64(bg, qoff[q]);
    }
    if constexpr (ONE) {  // a row of 16 lanes holds 4 columns: no broadcast
#pragma unroll
      for (int c = 0; c < 9; ++c) rg[d][c] = buffer_load_f64(rG, (ke * 9u + (uint32_t)c) * 8u);
    } else {
      rg[d][0] = buffer_load_f64(rG, (ke * 9u + gf) * 8u);
    }
    ke += dk;
    kr += dr;
    if (kr >= F) {
      kr -= F;
      ++ke;
    }
  };

  // accumulators: tiles; C (row tile x quad columns), R (quad rows x column
  // tile), K (quad x quad); the extra tile's
  f64x4 accF[ND][NR > 0 ? NR : 1][NF > 0 ? NF : 1], accX[NF > 0 ? NF : 1];
  double accC[ND][NR > 0 ? NR : 1][NQ > 0 ? NQ : 1], accXC[NQ > 0 ? NQ : 1];
  double accR[ND][NRQ > 0 ? NRQ : 1][NF > 0 ? NF : 1], accK[ND][NQ > 0 ? NQ : 1];
#pragma unroll
  for (int a = 0; a < ND; ++a) {
#pragma unroll
    for (int t = 0; t < NR; ++t) {
#pragma unroll
      for (int j = 0; j < NF; ++j) accF[a][t][j] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < NQ; ++q) accC[a][t][q] = 0.0;
    }
#pragma unroll
    for (int q = 0; q < NRQ; ++q) {
#pragma unroll
      for (int j = 0; j < NF; ++j) accR[a][q][j] = 0.0;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) accK[a][q] = 0.0;
  }
#pragma unroll
  for (int j = 0; j < NF; ++j) accX[j] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < NQ; ++q) accXC[q] = 0.0;

  auto step = [&](uint32_t s, auto Dc) __attribute__((always_inline)) {
    constexpr int d = decltype(Dc)::value;
    // (the tiles' 128 t then fold into the loads, not into registers of their own)
    asm volatile("" : "+v"(base_off), "+v"(tile_off));
    // W of the k-step, then gout of step s + DEPTH into its registers
    double W[ND][NG], WX = 0.0, x0 = 0.0, x1 = 0.0, x2 = 0.0;
    gd_static_for<0, ND>([&](auto Ac) __attribute__((always_inline)) {
      constexpr int a = decltype(Ac)::value;
      double g0, g1, g2;
      if constexpr (ONE) {
        g0 = rg[d][3 * a];
        g1 = rg[d][3 * a + 1];
        g2 = rg[d][3 * a + 2];
      } else {
        g0 = row_bcast_f64<3 * a>(rg[d][0]);
        g1 = row_bcast_f64<3 * a + 1>(rg[d][0]);
        g2 = row_bcast_f64<3 * a + 2>(rg[d][0]);
      }
#pragma unroll
      for (int t = 0; t < NG; ++t) {
        if (X && t == NR) continue;
        W[a][t] = g0 * raw[d][0][t] + g1 * raw[d][1][t] + g2 * raw[d][2][t];
      }
      if constexpr (X) {
        if (a == 0 || XD == a) {  // (uniform)
          x0 = g0;
          x1 = g1;
          x2 = g2;
        }
      }
      if constexpr (NP >= 56) __builtin_amdgcn_sched_barrier(0);  // (else all 9 broadcasts are held at once)
    });
    if constexpr (X) WX = x0 * raw[d][0][NR] + x1 * raw[d][1][NR] + x2 * raw[d][2][NR];
    load_g(s + DEPTH, Dc);
    __builtin_amdgcn_sched_barrier(0);
    // u feeds the products directly: one register at a time, reloaded after its
    // products.  (Raised priority: products before another wave's vector work, -1 %.)
    __builtin_amdgcn_s_setprio(1);
    constexpr int ud = d % UD;
    const __amdgpu_buffer_rsrc_t bu = range_u(s + UD);
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const double U = ru[ud][j];
#pragma unroll
      for (int a = 0; a < ND; ++a) {
#pragma unroll
        for (int t = 0; t < NR; ++t)
          accF[a][t][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(W[a][t], U, accF[a][t][j], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < NRQ; ++q)
          accR[a][q][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(W[a][NG - NRQ + q], U, accR[a][q][j], 0, 0, 0);
      }
      if constexpr (X) {
        if (xon) accX[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(WX, U, accX[j], 0, 0, 0);
      }
      load_u(bu, ud, j);
      if constexpr (UD == 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const double U = ru[ud][NF + q];
#pragma unroll
      for (int a = 0; a < ND; ++a) {
#pragma unroll
        for (int t = 0; t < NR; ++t)
          accC[a][t][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(W[a][t], U, accC[a][t][q], 0, 0, 0);
        // the first quad register of W against every one of u covers every pair of quads
        if constexpr (NRQ > 0)
          accK[a][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(W[a][NG - NRQ], U, accK[a][q], 0, 0, 0);
      }
      if constexpr (X) {
        if (xon) accXC[q] = __builtin_amdgcn_mfma_f64_4x4x4f64(WX, U, accXC[q], 0, 0, 0);
      }
      load_u(bu, ud, NF + q);
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  load_g(0, I0{});
  load_g(1, I1{});
#pragma unroll
  for (int d = 0; d < UD; ++d) {
    const __amdgpu_buffer_rsrc_t bu = range_u((uint32_t)d);
#pragma unroll
    for (int x = 0; x < NU; ++x) load_u(bu, d, x);
  }
  for (uint32_t s = 0; s < nsteps; s += DEPTH) {
    step(s, I0{});
    step(s + 1, I1{});
    // The groups carry different loads; left alone they drift apart until the
    // columns one has read have left the caches before the other needs them
    // (order 5, K = 2^19: 702 us without, 662 at every 4 steps, 652 at 32).
    if constexpr (S::NRG > 1) {
      if (s % 32 == 30) __syncthreads();
    }
  }

  if constexpr (ONE) {  // the four blocks hold four sets of columns: add them first
#pragma unroll
    for (int a = 0; a < ND; ++a) {
      accK[a][0] += __shfl_xor(accK[a][0], 4);
      accK[a][0] += __shfl_xor(accK[a][0], 8);
    }
  }
  // fn(accumulator, index, lane's byte offset, common byte offset) for every
  // accumulator: rows and columns of its output; a lane without one has an
  // offset past the partial sum
  const int l = opaque(lane);
  const int n1 = l & 15, g1 = l >> 4, b4 = (l >> 2) & 3, x4 = l & 3;
  auto each = [&](auto&& fn) __attribute__((always_inline)) {
    int x = 0;
    uint32_t ot[4], oc[2], orr[2], ok[2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      ot[q] = NP != 10 || (4 * q + g1 < NP && n1 < NP) ? (uint32_t)(g1 * NP + n1) * 8u : OUT;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int nq = (NQ == 2 ? 4 * ((b4 & 1) ^ q) : 0);  // the quad's first node, past the tiles
      const int r0 = (NQ == 2 ? 4 * (b4 & 1) : 0) + g1;
      oc[q] = 16 * NF + nq + x4 < NP ? (uint32_t)((4 * b4 + g1) * NP + nq + x4) * 8u : OUT;
      orr[q] = 16 * NF + nq + g1 < NP ? (uint32_t)((nq + g1) * NP + 4 * b4 + x4) * 8u : OUT;
      ok[q] = 16 * NF + r0 < NP && 16 * NF + nq + x4 < NP && b4 < NQ ? (uint32_t)(r0 * NP + nq + x4) * 8u : OUT;
    }
    auto tile = [&](uint32_t row, const f64x4& v, int j) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) fn(v[q], x++, ot[q], ((row + 4 * q) * NP + 16 * j) * 8u);
    };
#pragma unroll
    for (int a = 0; a < ND; ++a) {
      const uint32_t rt = (uint32_t)((a0 + a) * NP + 16 * T0), rq = (uint32_t)((a0 + a) * NP + 16 * NF);
#pragma unroll
      for (int t = 0; t < NR; ++t) {
#pragma unroll
        for (int j = 0; j < NF; ++j) tile(rt + 16 * t, accF[a][t][j], j);
#pragma unroll
        for (int q = 0; q < NQ; ++q) fn(accC[a][t][q], x++, oc[q], ((rt + 16 * t) * NP + 16 * NF) * 8u);
      }
#pragma unroll
      for (int q = 0; q < NRQ; ++q) {
#pragma unroll
        for (int j = 0; j < NF; ++j) fn(accR[a][q][j], x++, orr[q], (rq * NP + 16 * j) * 8u);
      }
      if constexpr (NRQ > 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) fn(accK[a][q], x++, ok[q], (rq * NP + 16 * NF) * 8u);
      }
    }
    if constexpr (X) {
      if (!xon) return;
      const uint32_t rx = (uint32_t)((a0 + XD) * NP + 16 * XT);
#pragma unroll
      for (int j = 0; j < NF; ++j) tile(rx, accX[j], j);
#pragma unroll
      for (int q = 0; q < NQ; ++q) fn(accXC[q], x++, oc[q], (rx * NP + 16 * NF) * 8u);
    }
  };
  // add the slices' accumulators in order: the first writes, the next add theirs, the last adds and stores
  const __amdgpu_buffer_rsrc_t rw = buffer_range(p.work + (int64_t)part * 3 * NP * NP, 3u * NP * NP * 8u);
  auto store = [&](double v, uint32_t off, uint32_t common) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rw, (int)off, (int)common, 0);
  };
  if constexpr (SLICES == 1) {
    each([&](double v, int, uint32_t off, uint32_t common) __attribute__((always_inline)) { store(v, off, common); });
  } else {
    constexpr int PL = S::acc_pass(LAST, ND);
    double* mine = lds + l;
#pragma unroll
    for (int pass = 0; pass < S::passes(ND); ++pass) {
      const int x0 = pass * PL;
#pragma unroll 1
      for (uint32_t v = 0; v < SLICES; ++v) {
        if (slice == v) {
          if (v == 0)
            each([&](double a, int x, uint32_t, uint32_t) __attribute__((always_inline)) {
              if (x / PL == pass) mine[(x - x0) * WAVE] = a;
            });
          else if (v + 1 < SLICES)
            each([&](double a, int x, uint32_t, uint32_t) __attribute__((always_inline)) {
              if (x / PL == pass) mine[(x - x0) * WAVE] += a;
            });
          else
            each([&](double a, int x, uint32_t off, uint32_t common) __attribute__((always_inline)) {
              if (x / PL == pass) store(mine[(x - x0) * WAVE] + a, off, common);
            });
        }
        __syncthreads();
      }
    }
  }
}

// Forms: a workgroup per part (ND = 3, RS = 1); with few parts, RS = 2
// workgroups of half the row groups each (grid.z), or those for each direction
// (ND = 1, grid.y), so that the chain of products of a part is half or a sixth
// as long (a sum of 2 parts, orders 5 / 6 / 7: 17 / 24 / 27 -> 8 / 12 / 11 us); at
// Np = 120 also RS = 4 with two column slices, a quarter.
template <int NP, int ND, int RS>
constexpr int gd_threads() { return WAVE * GdShape<NP>::NRG / RS * GdShape<NP>::slices(RS); }

template <int NP, int ND, int RS>
__global__ __launch_bounds__((gd_threads<NP, ND, RS>())) __attribute__((amdgpu_waves_per_eu(ND == 1 ? 3 : GdShape<NP>::WPS, 8)))
void gd_partial_kernel(GdArgs p) {
  using S = GdShape<NP>;
  __shared__ double lds[S::lds_doubles(ND, RS)];
  const uint32_t w0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t slice, rg;
  if constexpr (S::NRG == 1) {
    slice = w0;
    rg = 0;
  } else if constexpr (RS > 1) {  // workgroup z has row groups z NRG / RS on
    constexpr uint32_t H = S::NRG / RS;
    slice = w0 / H;
    rg = w0 % H + blockIdx.z * H;
  } else {  // waves w and w + 4 share a SIMD: Np = 56: of the two groups; Np = 84: of neighbouring ones
    slice = S::NRG == 2 ? w0 & 3u : S::NRG == 4 ? w0 >> 2 : 0u;
    rg = S::NRG == 2 ? w0 >> 2 : S::NRG == 4 ? (w0 + slice) & 3u : w0;
  }
  double* mine = lds + (S::slices(RS) > 1 ? rg % (S::NRG / RS) * S::lds_group(ND) : 0);
  // (both kinds run the same number of workgroup barriers)
  if (S::NRG > 1 && rg + 1 < S::NRG)
    gd_role<NP, S::NRG == 1, ND, RS>(p, blockIdx.x, slice, (int)rg, (int)blockIdx.y, mine);
  else
    gd_role<NP, true, ND, RS>(p, blockIdx.x, slice, (int)rg, (int)blockIdx.y, mine);
}

// gD[x] = sum over parts of work[part][x], x < n, in a fixed order.
// Block: 16 consecutive x (whole cache lines) by GD_RED_PG part groups; part
// group g adds parts g, g + GD_RED_PG, ... in ascending order, and the group
// sums are then added in two ordered levels.  With 16 part groups of 64 x, one
// block of order 1 walked 64 parts in a chain (18 us; now 4).  With npart = 0
// it writes zeros.
constexpr int GD_RED_PG = 64;
constexpr int GD_RED_X = 16;

__global__ __launch_bounds__(GD_RED_X * GD_RED_PG) void gd_reduce_kernel(const double* __restrict__ work,
                                                                        double* __restrict__ gD, uint32_t npart,
                                                                        uint32_t n) {
  __shared__ double part_sum[GD_RED_PG][GD_RED_X];
  const int xi = threadIdx.x % GD_RED_X;
  const int g = threadIdx.x / GD_RED_X;
  const uint32_t x = blockIdx.x * GD_RED_X + xi;
  double s = 0.0;
  if (x < n) {
    for (uint32_t pt = g; pt < npart; pt += 4 * GD_RED_PG) {  // four reads in flight
      double v[4];
#pragma unroll
      for (uint32_t h = 0; h < 4; ++h) v[h] = work[(int64_t)min(pt + h * GD_RED_PG, npart - 1u) * n + x];
#pragma unroll
      for (uint32_t h = 0; h < 4; ++h) s += pt + h * GD_RED_PG < npart ? v[h] : 0.0;
    }
  }
  part_sum[g][xi] = s;
  __syncthreads();
  if (g < 8) {
    s = 0.0;
#pragma unroll
    for (int h = 0; h < 8; ++h) s += part_sum[8 * g + h][xi];
  }
  __syncthreads();
  if (g < 8) part_sum[g][xi] = s;
  __syncthreads();
  if (g == 0 && x < n) {
    double t = 0.0;
#pragma unroll
    for (int h = 0; h < 8; ++h) t += part_sum[h][xi];
    gD[x] = t;
  }
}

}  // namespace dgvol
