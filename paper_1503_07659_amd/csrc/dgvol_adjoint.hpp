// Adjoint kernels of the DG volume derivative (reverse mode w.r.t. u and G), Np <= 56.
//
//   W_a[i]      = sum_b G[3a+b] gout_b[i]
//   gu[j]       = sum_a sum_i D[a][i][j] W_a[i]          (transposed product)
//   gG[3a+b]    = sum_{f,i} gout_b[i] (D_a u)[i]          (D u recomputed)
#pragma once

#include "dgvol_device.hpp"

namespace dgvol {

// ------------------------------------------------------------------ adjoint FP64 (Np <= 56)
//
// A wave takes 16 columns (element, field) at a time.  Lane (n, g) owns column
// n and, of its nodes, those of lane group g: pairs 8p + 2g, 8p + 2g + 1, then
// one of the last Np mod 8.  It loads u and the three planes of gout at its
// own nodes (16-byte pairs, 64-byte runs over the four groups) straight into
// registers, one tile ahead, and never exchanges them:
//   * u is the B operand of R = D u as it is (k-step 2p + e takes node 8p + 2g
//     + e; the A rows are permuted so that lane (n, g) gets R at its own nodes);
//   * the gG partials gout_b R_a and W = G^T gout are lane-local;
//   * W is the A operand of gu = W^T D as it is, with the columns as the
//     matrix rows, so that a result lane holds 16 consecutive nodes'
//     neighbours of a column and gu is stored from the accumulators.
// Only the operand table of D and the gG sums live in LDS (with GG, u too: each
// lane's own values, read back for every chunk).
//
// Bound: the memory up to Np = 35 (and for gu alone), the FP64 products at Np
// = 56 with GG (266 of 64 and 112 of 16 cycles per tile, 80 % of the cycles
// busy; the 250 FP64 multiply-adds of W and gG do not overlap them).  Measured
// against the kernel it replaced (u, gout and gu exchanged through LDS, one
// 8-wave workgroup per 8 tiles), F = 3, 2e7 nodal values: order 1 315 -> 229
// us, order 2 214 -> 192, order 3 203 -> 187, order 4 242 -> 208; order 5,
// K = 2^19 1098 -> 1064 us; order 3, K = 13601, F = 17 61 -> 50 us; 1e6
// values: order 2 15.6 -> 11.5 us, order 3 14.7 -> 14.0, order 4 27.5 -> 15.6,
// order 5 49 -> 28; 3e5: order 4 24.5 -> 13.2, order 5 37.5 -> 25.9.  gu
// alone, 2e7 values: 135-160 us at orders 1-5.
//
// GG = false: gu alone (no u, no recomputed D u, no gG), tiles dealt to the
// waves in turn.  GG = true: each wave owns a contiguous run of whole elements
// and takes its columns as full 16-column tiles (only the run's last tile can
// be short); an element that continues past a tile carries its partial gG sum
// into the next one, so every element's gG sums finish in one wave, in a fixed
// order, with no cross-wave reduction.
template <int NP>
struct AdjShape {
  using Sh = Shape<NP>;
  static constexpr int KP = NP / 8;        // node pairs of a lane
  static constexpr int TRIP = Sh::TRIP;    // its nodes (2 KP, plus one of the last NP mod 8)
  static constexpr bool TAIL = NP % 8 != 0;
  static_assert(TRIP == 2 * KP + (TAIL ? 1 : 0) && NP % 8 <= 4, "nodes of a lane");
  static constexpr int KS = Sh::KS64;
  // Row quads of the last 16-row tile of D u, and node quads of the last tile
  // of gu.  At most two run as v_mfma_f64_4x4x4f64 each (16 cycles against 64).
  static constexpr int FQ = Sh::SLOTS - 4 * (Sh::MT - 1);
  static constexpr int JQ = (NP - 16 * (Sh::MTJ - 1) + 3) / 4;
  static constexpr bool FSPLIT = FQ <= 2, JSPLIT = JQ <= 2;
  static constexpr int MTJF = JSPLIT ? Sh::MTJ - 1 : Sh::MTJ;
  static constexpr int NJO = MTJF + (JSPLIT ? JQ : 0);  // products per slot of gu
  // doubles of the operand table: GG: the A rows of D u (read transposed for
  // gu too); else the B operands of gu, [slot][tile][lane], then [slot][quad][16]
  static constexpr int FTAB = Sh::MT * KS * WAVE;
  static constexpr int JTAB = Sh::SLOTS * (MTJF * WAVE + (JSPLIT ? JQ * 16 : 0));
};

// node -> the lane's node index tau and lane group g
template <int NP>
__device__ __forceinline__ void adj_split(int i, int& tau, int& g) {
  constexpr int KP = NP / 8;
  const bool pair = i < 8 * KP;
  tau = pair ? 2 * (i >> 3) + (i & 1) : 2 * KP;
  g = pair ? (i & 7) >> 1 : i - 8 * KP;
}

template <int NP, int WPB, bool GG>
struct AdjLds {
  using S = AdjShape<NP>;
  static constexpr int TAB = GG ? S::FTAB : S::JTAB;
  static constexpr int UP = GG ? S::TRIP * WAVE : 0;  // per wave: u, each lane's own values
  static constexpr int GK = 16 * 9;                   // per wave: geometric factors of the tile's elements
  static constexpr int RED = GG ? 16 * 9 + 10 : 0;    // per wave: gG sums per column, carry (even: u stays 16-byte aligned)
  static constexpr int BYTES = (TAB + WPB * (UP + GK + RED)) * 8;
};

// Sums of 9 values over the four lane groups: s[0], s[1] hold, in lane group g,
// value {0, 2, 1, 3}[g] and 4 + that; s[2] value 8 in every lane.  Each swap
// halves the registers (permlane32: rows 2, 3 of one against rows 0, 1 of the
// other; permlane16: odd rows against even rows).
__device__ __forceinline__ void swap_rows32(double& a, double& b) {
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
  u32x2_t x = __builtin_bit_cast(u32x2_t, a), y = __builtin_bit_cast(u32x2_t, b);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto r = __builtin_amdgcn_permlane32_swap(x[h], y[h], false, false);
    x[h] = r[0];
    y[h] = r[1];
  }
  a = __builtin_bit_cast(double, x);
  b = __builtin_bit_cast(double, y);
}
__device__ __forceinline__ void swap_rows16(double& a, double& b) {
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
  u32x2_t x = __builtin_bit_cast(u32x2_t, a), y = __builtin_bit_cast(u32x2_t, b);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto r = __builtin_amdgcn_permlane16_swap(x[h], y[h], false, false);
    x[h] = r[0];
    y[h] = r[1];
  }
  a = __builtin_bit_cast(double, x);
  b = __builtin_bit_cast(double, y);
}
__device__ __forceinline__ double sum_rows32(double a, double b) {
  swap_rows32(a, b);
  return a + b;
}
__device__ __forceinline__ double sum_rows16(double a, double b) {
  swap_rows16(a, b);
  return a + b;
}
__device__ __forceinline__ void sum_groups9(const double (&P)[9], double (&s)[3]) {
  s[0] = sum_rows16(sum_rows32(P[0], P[1]), sum_rows32(P[2], P[3]));
  s[1] = sum_rows16(sum_rows32(P[4], P[5]), sum_rows32(P[6], P[7]));
  const double t = sum_rows32(P[8], P[8]);
  s[2] = sum_rows16(t, t);
}

// waves per workgroup, and waves per SIMD the register budget must allow
constexpr int adj_wpb(int np, bool gg) { return np >= 56 || (np >= 35 && gg) ? 8 : 4; }
constexpr int adj_min_waves(int np, bool gg) { return np >= 56 ? 2 : np >= 35 ? (gg ? 2 : 3) : np >= 20 && gg ? 3 : 4; }

template <int NP, int WPB, bool GG>
__global__ __launch_bounds__(WAVE* WPB) __attribute__((amdgpu_waves_per_eu(adj_min_waves(NP, GG), 8))) void adj_f64_kernel(
    const double* __restrict__ D, const double* __restrict__ G, const double* __restrict__ u,
    const double* __restrict__ gout, double* __restrict__ gu, double* __restrict__ gG, uint32_t K, uint32_t F,
    int64_t plane, uint32_t nworkers) {
  using Sh = Shape<NP>;
  using S = AdjShape<NP>;
  using L = AdjLds<NP, WPB, GG>;
  constexpr int KS = S::KS, KP = S::KP, TRIP = S::TRIP, MTJF = S::MTJF, NJO = S::NJO;
  __shared__ __attribute__((aligned(16))) double lds[L::BYTES / 8];
  static_assert(L::BYTES <= 160 * 1024, "LDS budget");
  double* tab = lds;
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* mine = lds + L::TAB + wave * (L::UP + L::GK + L::RED);
  double* up = mine + lane * 2;         // u: pair p at up[p * 128], the last node at up_t
  double* up_t = mine + KP * 128 + lane;
  double* gks = mine + L::UP;
  double* red = gks + L::GK;
  double* cry = red + 16 * 9;

  // ---- operand table, from contiguous reads of D
  for (int x = threadIdx.x; x < L::TAB; x += WAVE * WPB) tab[x] = 0.0;
  __syncthreads();
  for (int x = threadIdx.x; x < 3 * NP * NP; x += WAVE * WPB) {
    const double v = D[x];
    const int r = x / NP, j = x - r * NP;
    const int a = r / NP, i = r - a * NP;
    int tau, gi;
    adj_split<NP>(i, tau, gi);
    const int sp = 3 * tau + a;
    if constexpr (GG) {
      int s, kk;
      adj_split<NP>(j, s, kk);
      tab[((sp >> 2) * KS + s) * WAVE + tswz(16 * kk + 4 * (sp & 3) + gi, s)] = v;
    } else {
      const int tj = j >> 4, nj = j & 15;
      if (S::JSPLIT && tj == MTJF)
        tab[Sh::SLOTS * MTJF * WAVE + (sp * S::JQ + (nj >> 2)) * 16 + 4 * gi + (nj & 3)] = v;
      else
        tab[(sp * MTJF + tj) * WAVE + 16 * gi + nj] = v;
    }
  }
  __syncthreads();

  // ---- this wave's tiles
  // Workers are numbered across the workgroups first, so that few tiles spread
  // over the CUs; with a tile for every wave, gu alone numbers them within the
  // workgroup first, so that its waves stream neighbouring tiles (2e7 nodal
  // values: order 1 165 -> 153 us, order 3 154 -> 143 us).
  const bool packed = !GG && nworkers == gridDim.x * WPB;
  const uint32_t gw = packed ? blockIdx.x * WPB + wave : wave * gridDim.x + blockIdx.x;
  if (gw >= nworkers) return;  // (no workgroup barrier follows)
  const uint32_t ncols = K * F;
  uint32_t c_lo, c_hi, step, nrun;
  if constexpr (GG) {
    // Short runs: the first K mod nworkers workers take the element more.  They are the
    // lowest waves of every workgroup, so that a SIMD has at most one of them before all
    // have one (spread evenly over the workers, order 5, K = 6178, F = 5 took 47.4 us, now
    // 38.1).  Past four tiles a run that gains nothing, and runs of one length can meet
    // the same memory channels: there they are spread (order 3, K = 27970, F = 17: 86 us
    // against 92).
    uint32_t e_lo, e_hi;
    const uint32_t q = K / nworkers;
    if (q * F < 64) {
      const uint32_t r = K - q * nworkers;
      e_lo = gw * q + min(gw, r);
      e_hi = e_lo + q + (gw < r ? 1u : 0u);
    } else {
      e_lo = (uint32_t)((uint64_t)gw * K / nworkers);
      e_hi = (uint32_t)((uint64_t)(gw + 1) * K / nworkers);
    }
    c_lo = e_lo * F;
    c_hi = e_hi * F;
    step = 16;
  } else {
    c_lo = gw * 16;
    c_hi = ncols;
    step = nworkers * 16;
  }
  nrun = c_lo < c_hi ? (c_hi - c_lo + step - 1) / step : 0u;

  // per-lane table offsets
  int fo[4], tb[4], tl[4];
  int fs = 0;
  if constexpr (GG) {
    const int s0 = 2 * (n >> 3) + (n & 1), k0 = (n & 7) >> 1;  // k-step (mod 4) and group of node n of a full tile
    int sl, kl;  // of this lane's node of the last tile (4x4x4: node lane & 3 of a quad; quad r adds 2 r 16 ...)
    const int nl = S::JSPLIT ? (lane & 3) : n;
    adj_split<NP>(min(16 * (Sh::MTJ - 1) + nl, NP - 1), sl, kl);
    sl -= 4 * (Sh::MTJ - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      fo[q] = tswz(lane, q);
      tb[q] = s0 * WAVE + tswz(16 * k0 + 4 * q + g, s0);
      tl[q] = sl * WAVE + tswz(16 * kl + 4 * q + g, sl);
    }
    fs = 16 * g + ((lane & 3) ^ g);
  }
  // a second quad of the last tile (nodes 4 on): group kl + 2 of the same k-step, so the
  // swizzled entry moves by 32 and flips bit 1 of the lane group
  // operand o of slot sp: 16 x 16 tiles o < MTJF, then the quads of the last tile
  auto jop = [&](int sp, int o) __attribute__((always_inline)) {
    if constexpr (GG) {
      if (o < MTJF && (o < Sh::MTJ - 1)) return tab[((sp >> 2) * KS + 4 * o) * WAVE + tb[sp & 3]];
      const int at = ((sp >> 2) * KS + 4 * (Sh::MTJ - 1)) * WAVE + tl[sp & 3];
      return o == Sh::MTJ - 1 ? tab[at] : tab[(at + 32) ^ 2];
    } else {
      if (o < MTJF) return tab[(sp * MTJF + o) * WAVE + lane];
      return tab[Sh::SLOTS * MTJF * WAVE + (sp * S::JQ + o - MTJF) * 16 + 4 * g + (lane & 3)];
    }
  };

  // ---- loads, one tile ahead, through buffer ranges of the tile's columns
  // (zero past them and for the padding nodes), so that no branch surrounds a
  // load and the waits count exactly
  const uint32_t loff = (uint32_t)(n * NP + 2 * g) * 8u;
  const uint32_t toff = 8 * KP + g < NP ? (uint32_t)(n * NP + 8 * KP + g) * 8u : 0x40000000u;
  f64x2 go[3][KP > 0 ? KP : 1], ur[KP > 0 ? KP : 1];
  double got[3], urt = 0.0, graw[3];
  struct Cols {
    uint32_t col0, ncol, k0, ne;
  };
  auto cols = [&](uint32_t t) __attribute__((always_inline)) {
    Cols c;
    c.ncol = t < nrun ? cols_left(c_hi, c_lo + t * step, 16) : 0u;
    c.col0 = t < nrun ? c_lo + t * step : 0u;
    c.k0 = c.col0 / F;
    c.ne = c.ncol ? (c.col0 + c.ncol - 1u) / F - c.k0 + 1u : 0u;
    return c;
  };
  auto range = [&](const double* base, const Cols& c) __attribute__((always_inline)) {
    return buffer_range(base + (int64_t)c.col0 * NP, c.ncol * NP * 8u);
  };
  auto load_pair = [&](const __amdgpu_buffer_rsrc_t& r, int p) __attribute__((always_inline)) {
    return __builtin_bit_cast(f64x2, buffer_load_vec<double, 2>(r, loff + (uint32_t)p * 64u));
  };
  auto load_u = [&](const Cols& c) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t r = range(u, c);
#pragma unroll
    for (int p = 0; p < KP; ++p) ur[p] = load_pair(r, p);
    if constexpr (S::TAIL) urt = buffer_load_f64(r, toff);
  };
  auto load_G = [&](const Cols& c) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t r = buffer_range(G + (int64_t)c.k0 * 9, c.ne * 72u);
#pragma unroll
    for (int q = 0; q < 3; ++q) graw[q] = buffer_load_f64(r, (uint32_t)(lane + WAVE * q) * 8u);
  };
  Cols cur = cols(0);
  if constexpr (GG) load_u(cur);
  load_G(cur);
  // nodes per step of the transposed product: a chunk of 4 with GG, a pair without
  constexpr int CHT = GG ? 4 : 2;
  constexpr int NCH = (TRIP + CHT - 1) / CHT;
  // gout of chunk ch's nodes
  auto load_go = [&](const __amdgpu_buffer_rsrc_t (&r)[3], int ch) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < CHT; ++x) {
      const int tau = CHT * ch + x;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (tau < 2 * KP && tau % 2 == 1) go[b][tau / 2] = load_pair(r[b], tau / 2);
        if (tau == 2 * KP && S::TAIL) got[b] = buffer_load_f64(r[b], toff);
      }
    }
  };
  // gout runs a whole tile ahead, each pair's registers reloaded right after
  // their use; at Np = 56 with GG, which has no registers for that, one chunk ahead
  constexpr bool AHEAD1 = GG && NP >= 56;
  {
    __amdgpu_buffer_rsrc_t r[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) r[b] = range(gout + b * plane, cur);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
      if (ch == 0 || !AHEAD1) load_go(r, ch);
  }
  // From Np = 20 in a scalar register: in a vector register it was the one that
  // spilled at Np = 56, and its reload in the loop waited for every memory
  // operation in flight (F = 3, 2e7 nodal values 269 -> 262 us, gu alone 156 ->
  // 153).  At Np = 10 the register saved let a seventh wave in, which made gu
  // alone slower (135 -> 137).
  float invF = 1.0f / (float)F;
  if constexpr (NP >= 20)
    invF = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(opaque(__builtin_bit_cast(int, invF))));
  for (uint32_t t = 0; t < nrun; ++t) {
    const Cols nxt = cols(t + 1);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int x = lane + WAVE * q;
      if (x < L::GK) gks[x] = graw[q];
    }
    load_G(nxt);
    if constexpr (GG) {
#pragma unroll
      for (int p = 0; p < KP; ++p) *reinterpret_cast<f64x2*>(up + p * 128) = ur[p];
      if constexpr (S::TAIL) *up_t = urt;
    }
    __amdgpu_buffer_rsrc_t rn[3], rc3[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      rn[b] = range(gout + b * plane, nxt);
      rc3[b] = range(gout + b * plane, cur);
    }
    wave_sync();
    // element of this lane's column within the tile, (col0 mod F + n) / F: one
    // step at most for F >= 16, else exact in float (+ 0.5 keeps a whole
    // quotient off its edge); a column past the tile takes the first element
    const uint32_t rc = cur.col0 - cur.k0 * F + (uint32_t)n;
    const uint32_t eq = F >= 16u ? (rc >= F ? 1u : 0u) : (uint32_t)(((float)rc + 0.5f) * invF);
    const double* ge = gks + ((uint32_t)n < cur.ncol ? eq : 0u) * 9;
    double gl[9];
    if constexpr (!GG) {
#pragma unroll
      for (int c = 0; c < 9; ++c) gl[c] = ge[c];
    }
    f64x4 accj[MTJF > 0 ? MTJF : 1];
    double accs[2] = {0.0, 0.0};
#pragma unroll
    for (int o = 0; o < MTJF; ++o) accj[o] = f64x4{0.0, 0.0, 0.0, 0.0};
    double P[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) P[c] = 0.0;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      if constexpr (AHEAD1) {
        if (ch + 1 < NCH)
          load_go(rc3, ch + 1);
        else
          load_go(rn, 0);
      }
      f64x4 acc[3];
      if constexpr (GG) {
        if (ch == (NCH > 1 ? NCH - 2 : 0)) load_u(nxt);
#pragma unroll
        for (int tt = 0; tt < 3; ++tt) acc[tt] = f64x4{0.0, 0.0, 0.0, 0.0};
        // operand o of a k-step: the chunk's 16 x 16 tiles, then the quads of the last tile
        const int ntile = Sh::MT - 3 * ch < 3 ? Sh::MT - 3 * ch : 3;
        const bool split = S::FSPLIT && 3 * ch + ntile == Sh::MT;
        const int nfull = split ? ntile - 1 : ntile;
        const int nop = nfull + (split ? S::FQ : 0);
        auto fop = [&](int s, int o) __attribute__((always_inline)) {
          if (o < nfull) return tab[((3 * ch + o) * KS + s) * WAVE + fo[s & 3]];
          return tab[((Sh::MT - 1) * KS + s) * WAVE + fs + 4 * ((o - nfull) ^ (s & 3))];
        };
        auto ub = [&](int s) __attribute__((always_inline)) { return s < 2 * KP ? up[(s / 2) * 128 + s % 2] : *up_t; };
        double ac[4], an[4], bc = ub(0), bn = 0.0;
#pragma unroll
        for (int o = 0; o < 4; ++o)
          if (o < nop) ac[o] = fop(0, o);
        __builtin_amdgcn_sched_barrier(0);
        // operands one k-step ahead, one read after each product
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          if (s + 1 < KS) bn = ub(s + 1);
#pragma unroll
          for (int o = 0; o < 4; ++o) {
            if (o >= nop) continue;
            if (s + 1 < KS) an[o] = fop(s + 1, o);
            if (o < nfull)
              acc[o] = __builtin_amdgcn_mfma_f64_16x16x4f64(ac[o], bc, acc[o], 0, 0, 0);
            else
              acc[nfull][o - nfull] = __builtin_amdgcn_mfma_f64_4x4x4f64(ac[o], bc, acc[nfull][o - nfull], 0, 0, 0);
          }
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
          for (int o = 0; o < 4; ++o) {
            if (o >= nop) continue;
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          bc = bn;
#pragma unroll
          for (int o = 0; o < 4; ++o) ac[o] = an[o];
        }
#pragma unroll
        for (int c = 0; c < 9; ++c) gl[c] = ge[c];
      }
      double W[3 * CHT];
#pragma unroll
      for (int x = 0; x < CHT; ++x) {
        const int tau = CHT * ch + x;
        if (tau >= TRIP) continue;
        double gv[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) gv[b] = tau < 2 * KP ? go[b][tau / 2][tau % 2] : got[b];
        if constexpr (GG) {
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const double R = acc[(3 * x + a) >> 2][(3 * x + a) & 3];
#pragma unroll
            for (int b = 0; b < 3; ++b) P[3 * a + b] += gv[b] * R;
          }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a)
          W[3 * x + a] = gl[3 * a] * gv[0] + gl[3 * a + 1] * gv[1] + gl[3 * a + 2] * gv[2];
      }
      if constexpr (!AHEAD1) load_go(rn, ch);  // these nodes' gout of the next tile
      // transposed product, operands one slot ahead (one read after each product)
      double tc[NJO], tn[NJO];
#pragma unroll
      for (int o = 0; o < NJO; ++o) tc[o] = jop(3 * CHT * ch, o);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int sl = 0; sl < 3 * CHT; ++sl) {
        const int sp = 3 * CHT * ch + sl;
        if (sp >= Sh::SLOTS) continue;
        const bool more = sl + 1 < 3 * CHT && sp + 1 < Sh::SLOTS;
#pragma unroll
        for (int o = 0; o < NJO; ++o) {
          if (more) tn[o] = jop(sp + 1, o);
          if (o < MTJF)
            accj[o] = __builtin_amdgcn_mfma_f64_16x16x4f64(W[sl], tc[o], accj[o], 0, 0, 0);
          else
            accs[o - MTJF] = __builtin_amdgcn_mfma_f64_4x4x4f64(W[sl], tc[o], accs[o - MTJF], 0, 0, 0);
        }
#pragma unroll
        for (int o = 0; o < NJO; ++o) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < NJO; ++o) tc[o] = tn[o];
      }
    }
    // gu.  Ordinary stores, which the L2 merges into whole lines; at Np <= 10 a
    // store instruction covers whole rows, and streaming stores measured better
    // (order 2, 2e7 nodal values: 143 -> 135 us; order 3 would lose 17 %).
    auto store = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t off, double v) __attribute__((always_inline)) {
      if constexpr (NP <= 10)
        buffer_store_stream_f64(r, off, v);
      else
        buffer_store_f64(r, off, v);
    };
    // rows (columns) 4q + g, nodes 16 o + n; quad r: column 4 b + g, node 4 r + (lane & 3)
    {
      const __amdgpu_buffer_rsrc_t ro = range(gu, cur);
#pragma unroll
      for (int o = 0; o < MTJF; ++o) {
        const uint32_t off = 16 * o + n < NP ? (uint32_t)(g * NP + 16 * o + n) * 8u : 0x40000000u;
#pragma unroll
        for (int q = 0; q < 4; ++q) store(ro, off + (uint32_t)(4 * q * NP) * 8u, accj[o][q]);
      }
      if constexpr (S::JSPLIT) {
#pragma unroll
        for (int r = 0; r < S::JQ; ++r) {
          const int j = 16 * MTJF + 4 * r + (lane & 3);
          store(ro, j < NP ? (uint32_t)((4 * ((lane >> 2) & 3) + g) * NP + j) * 8u : 0x40000000u, accs[r]);
        }
      }
    }
    if constexpr (GG) {
      // gG: sums over the lane groups, then lane (j, c) sums factor c of element k0 + j
      // over its columns in the tile in order, after the partial sum carried from the
      // previous tile when the element began there; written when the element ends in
      // this tile, else carried into the next one
      double s[3];
      sum_groups9(P, s);
      const int cg = (g >> 1) | ((g & 1) << 1);
      red[n * 9 + cg] = s[0];
      red[n * 9 + 4 + cg] = s[1];
      if (g == 0) red[n * 9 + 8] = s[2];
      wave_sync();
      double carry = 0.0;
      int carry_c = -1;  // factor whose sum this lane carries
      const __amdgpu_buffer_rsrc_t rgg = buffer_range(gG + (int64_t)cur.k0 * 9, cur.ne * 72u);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        if (WAVE * (uint32_t)r < cur.ne * 9u) {
          const uint32_t x = (uint32_t)lane + WAVE * (uint32_t)r;
          const uint32_t j = x / 9u, c = x - 9u * j;
          const uint32_t ke = cur.k0 + j;
          const bool mine_j = j < cur.ne;
          const uint32_t lo = max(ke * F, cur.col0) - cur.col0;
          const uint32_t hi = mine_j ? min((ke + 1u) * F, cur.col0 + cur.ncol) - cur.col0 : 0u;
          double sum = j == 0 && ke * F < cur.col0 ? cry[c] : 0.0;
          for (uint32_t m = lo; m < hi; m += 4) {  // four reads in flight
            double v[4];
#pragma unroll
            for (uint32_t h = 0; h < 4; ++h) v[h] = red[min(m + h, 15u) * 9 + c];
#pragma unroll
            for (uint32_t h = 0; h < 4; ++h) sum += m + h < hi ? v[h] : 0.0;
          }
          const bool ends = (ke + 1u) * F <= cur.col0 + cur.ncol;
          buffer_store_f64(rgg, mine_j && ends ? x * 8u : 0x40000000u, sum);
          if (mine_j && !ends) {  // (the tile's last element: one lane per factor)
            carry = sum;
            carry_c = (int)c;
          }
        }
      }
      wave_sync();  // the previous carry has been read
      if (carry_c >= 0) cry[carry_c] = carry;
    }
    wave_sync();
    cur = nxt;
  }
}

}  // namespace dgvol
