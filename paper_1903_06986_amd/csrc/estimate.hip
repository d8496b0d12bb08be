// The subtracted trace estimator (Sec. 5 Eq. (23); Sec. 6):
//   t_n[Theta][t] = sum_{x in timeslice t} eta_n(x)^+ Theta (x_n - xt_n)(x)
//   est[Theta][t] = (1/N) sum_n t_n[Theta][t] + Tr_t(Theta tilde-M^{-1})
// One pass over eta, x and xt per (timeslice, right-hand side) block; the
// lexicographic layout keeps each timeslice contiguous.  Standard errors are
// s / sqrt(N) with the unbiased sample variance, for Re and Im separately.
#include <cmath>
#include <mutex>
#include <type_traits>

#include "cplx.h"
#include "gamma.h"
#include "fields.h"
#include "pointsplit.h"

namespace lqcd {
namespace {

constexpr int kWaves = kBlock / 64;

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Up to kMaxVar subtracted vectors of one set of solutions are estimated
// together: variant v forms x - xt_v (xt_v null: x itself) with the same
// operations, in the same order, as a pass with that variant alone, so its
// sums equal that pass's bit for bit.  Both kernels read eta and x once for
// a group of variants.
constexpr int kMaxVar = 6;
// Partial-sum slots per (variant, right-hand side, timeslice, chunk): the
// nine operator codes, with code 8 (point-split in t) in two slots, 8 and
// 9, for its terms whose row site lies one timeslice below and above the
// site the kernel works on.
constexpr int kOpSlots = kNumOps + 1;
struct XtSet {
  const cx<double> *p[kMaxVar];
};

// Each timeslice is split over nch workgroups (blockIdx.x = t * nch + ch)
// so the launch fills the chip; partial sums of variant v0 + v go to
// out[(((v * nrhs + r) * kOpSlots + op) * Lt + t) * nch + ch] (re, im) and
// the host adds the chunks in a fixed order.
template <int NV>
__global__ void __launch_bounds__(kBlock)
    k_estimate(const cx<double> *__restrict__ eta, const cx<double> *__restrict__ x, XtSet xts, int v0,
               size_t V, int Vs, int Lt, int nch, double *__restrict__ out) {
  __shared__ double sh[NV * 2 * kNumTheta][kWaves];
  const int t = blockIdx.x / nch, ch = blockIdx.x % nch, r = blockIdx.y, nrhs = gridDim.y;
  const size_t base = (size_t(r) * V + size_t(t) * Vs) * 12;
  double acc[NV][2 * kNumTheta] = {};
  // lane = (site, colour c): it loads the four spins of colour c of eta, x
  // and each xt_v (loads of 16 bytes, three lanes cover a site's 192-byte
  // block) and forms every Theta's terms from registers, since each Theta
  // only permutes spins (with a phase) at fixed colour
  const size_t ne = size_t(Vs) * 3;
  for (size_t e = size_t(ch) * kBlock + threadIdx.x; e < ne; e += size_t(nch) * kBlock) {
    const size_t s0 = base + e / 3 * 12 + e % 3;  // (site, spin 0, colour c)
    cx<double> a[4], xs[4];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
      a[sp] = ldc(eta + s0 + 3 * sp);
      xs[sp] = ldc(x + s0 + 3 * sp);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const cx<double> *xt = xts.p[v];
      cx<double> d[4];
#pragma unroll
      for (int sp = 0; sp < 4; ++sp) d[sp] = xs[sp];
      if (xt)
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) d[sp] = d[sp] - ldc(xt + s0 + 3 * sp);
#pragma unroll
      for (int th = 0; th < kNumTheta; ++th)
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) {
          const cx<double> w = cmulc(a[sp], mk(kGamma[th].re[sp], kGamma[th].im[sp]) * d[kGamma[th].col[sp]]);
          acc[v][2 * th] += w.re;
          acc[v][2 * th + 1] += w.im;
        }
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int k = 0; k < 2 * kNumTheta; ++k) acc[v][k] = wave_sum(acc[v][k]);
  if (lane == 0)
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int k = 0; k < 2 * kNumTheta; ++k) sh[v * 2 * kNumTheta + k][wave] = acc[v][k];
  __syncthreads();
  if (threadIdx.x < NV * 2 * kNumTheta) {
    double sum = 0;
    for (int w = 0; w < kWaves; ++w) sum += sh[threadIdx.x][w];
    const int v = threadIdx.x / (2 * kNumTheta), k = threadIdx.x % (2 * kNumTheta);
    const int th = k / 2, part = k % 2;
    out[((((size_t(v0 + v) * nrhs + r) * kOpSlots + th) * Lt + t) * nch + ch) * 2 + part] = sum;
  }
}

// All nine operators at once, where a point-split one (codes 5..8) is asked
// for: t_n[mu][t] = sum_{x in t} eta_n(x)^+ (Theta(mu) (x_n - xt_n))(x),
// Theta(mu) = kappa [(1 + g_mu) U_mu(x - mu)^+ S_- - (1 - g_mu) U_mu(x) S_+]
// with S_-+ the shifts to x -+ mu.
//
// Every term is linear in d = x - xt at one site y, so at each y operator o is
// a 12-vector g_o(y) of eta and the links that is the same for all variants,
//   t[o][v] = sum_y g_o(y)^+ d_v(y):
// a matrix product of ten rows (the five local operators, x, y, z, and t in
// two rows: its forward terms belong to the timeslice below y's, its backward
// terms to the one above) with two columns per variant (real and imaginary
// part) over the 12 V components, summed on the matrix cores
// (v_mfma_f64_16x16x4, 4 components an instruction).  A column's sum depends
// on that column only, so a variant gives the same bits alone and in a group.
//
// g: (1 -+ g_mu) has rank 2 and squares to twice itself, and its lower half
// spinor is a unitary R times the upper one, so for any colour matrix W
//   a^+ (1 -+ g_mu) W b = sum_{s=0,1} (W^+ at_s)^+ h_s,
// where at and h are the upper halves of (1 -+ g_mu) a and (1 -+ g_mu) b:
// at_s = a_s + alpha_s a_{p(s)} with a spin partner p(s) in {2, 3} and a
// phase alpha_s in {+-1, +-i}.  The forward term of row x = y - mu is -kappa
// (U_mu(y - mu)^+ at)^+ h with at from eta(y - mu), the backward term of row x
// = y + mu is kappa (U_mu(y) at)^+ h with at from eta(y + mu), both with h
// from d(y).
//
// A workgroup takes 64 consecutive sites of one timeslice at a time.  Wave mu
// makes the rows of direction mu for them (lane = site), staging eta at the
// backward and then the forward neighbours through LDS (coalesced 16-byte
// loads; the rows take the same place afterwards, so no other wave waits for
// it), while eta at the sites, of which the local rows are permutations with
// phases, is staged by all.  Then each wave sums the products of 16 of the
// sites: the rows come from LDS, d straight from memory into registers (lane =
// half a complex number: 64 contiguous bytes of each variant an instruction).
//
// Bound by HBM (eta, x and each xt once): 24^3 x 32, 16 right-hand sides, six
// variants, one without xt, 7.9 ms (a local kernel for three variants a launch,
// and one that staged x - xt of every variant in LDS) -> 3.7 ms: 2.6 TB/s of
// links and fields, by the counters 1.64 times that (eta is gathered at the
// neighbours), 4.3 TB/s.
// Two workgroups a CU (LDS, registers) hide the latency of the two phases of
// each other only in part.
constexpr int kPsSites = 64;             // sites per chunk
constexpr int kPsStride = 13;            // LDS stride of a site: distinct banks across sites
constexpr int kPsRegion = kPsSites * kPsStride + 4;  // one staged field; consecutive ones 16 banks apart
constexpr int kPsRows = kNumTheta + kNumPS + 1;      // rows of the product
static_assert(kPsRows == kOpSlots && 2 * kMaxVar <= 16, "rows are slots, columns fit a tile");
static_assert(kNumPS == kWaves, "one direction per wave");

// Half spin HS of direction MU, forward (FWD: projector 1 - g_mu) or
// backward (1 + g_mu).
template <int MU, bool FWD, int HS>
struct PsHalf {
  // partner spin and phase of the forward projector (negated backward)
  static constexpr int PS = MU < 2 ? 3 - HS : 2 + HS;
  static constexpr double AR0 = MU == 1 ? (HS ? -1.0 : 1.0) : MU == 3 ? -1.0 : 0.0;
  static constexpr double AI0 = MU == 0 ? 1.0 : MU == 2 ? (HS ? -1.0 : 1.0) : 0.0;
  static constexpr double AR = FWD ? AR0 : -AR0, AI = FWD ? AI0 : -AI0;
  // p + alpha q with alpha in {+-1, +-i}
  __device__ static cx<double> proj(cx<double> p, cx<double> q) {
    return AR != 0.0 ? mk(p.re + AR * q.re, p.im + AR * q.im) : mk(p.re - AI * q.im, p.im + AI * q.re);
  }
  // conj(alpha) q
  __device__ static cx<double> phase(cx<double> q) {
    return AR != 0.0 ? mk(AR * q.re, AR * q.im) : mk(AI * q.im, -AI * q.re);
  }
  // at of a staged spinor
  __device__ static void at(const cx<double> *e, cx<double> a[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a[k] = proj(e[HS * 3 + k], e[PS * 3 + k]);
  }
};

// LDS operations of one wave are carried out in order; this keeps the
// compiler from moving them across the point where lanes exchange data.
__device__ inline void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// c = U^+ a (DAG) or U a.
template <bool DAG>
__device__ inline void ps_colour(const cx<double> u[9], const cx<double> a[3], cx<double> c[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const cx<double> w = u[DAG ? 3 * b + k : 3 * k + b];
      const double wi = DAG ? -w.im : w.im;
      re = fma(w.re, a[b].re, re);
      im = fma(w.re, a[b].im, im);
      re = fma(-wi, a[b].im, re);
      im = fma(wi, a[b].re, im);
    }
    c[k] = mk(re, im);
  }
}

// The rows of direction MU at the wave's 64 sites (lane = site, full index
// s of parity par; on: inside the timeslice, else the rows are zero) into
// reg.  sf, sb: index of the site's forward and backward neighbour.  mid() runs
// once the neighbours' registers are free.
template <int MU, class Mid>
__device__ inline void ps_rows(const cx<double> *__restrict__ U, size_t Vh, const cx<double> *__restrict__ eta,
                               double kappa, int s, int sf, int sb, int par, bool on, cx<double> *reg, Mid &&mid) {
  const int lane = threadIdx.x & 63;
  cx<double> vb[12], vf[12], ub[9], uf[9];
#pragma unroll
  for (int u = 0; u < 12; ++u) {  // piece j = lane + 64 u: complex j % 12 of site j / 12
    const int j = lane + 64 * (u % 3), site = j / 12 + 16 * (u / 3), k = j % 12;
    vb[u] = ldc(eta + size_t(__shfl(sb, site)) * 12 + k);
    vf[u] = ldc(eta + size_t(__shfl(sf, site)) * 12 + k);
  }
  const cx<double> *Ub = U + ((size_t(par ^ 1) * 4 + MU) * 9) * Vh + (sb >> 1);  // U_mu(y - mu)
  const cx<double> *Uf = U + ((size_t(par) * 4 + MU) * 9) * Vh + (s >> 1);       // U_mu(y)
#pragma unroll
  for (int e = 0; e < 9; ++e) ub[e] = ldc(Ub + e * Vh);
  cx<double> *own = reg + lane * kPsStride;
  cx<double> a0[3], a1[3], cf[2][3], cb[2][3];
  auto put = [&](const cx<double> *v) {
    wave_order();
#pragma unroll
    for (int u = 0; u < 12; ++u) {
      const int j = lane + 64 * (u % 3), site = j / 12 + 16 * (u / 3), k = j % 12;
      reg[site * kPsStride + k] = v[u];
    }
    wave_order();
  };
  put(vb);
#pragma unroll
  for (int e = 0; e < 9; ++e) uf[e] = ldc(Uf + e * Vh);
  PsHalf<MU, true, 0>::at(own, a0);
  PsHalf<MU, true, 1>::at(own, a1);
  ps_colour<true>(ub, a0, cf[0]);
  ps_colour<true>(ub, a1, cf[1]);
  put(vf);
  mid();
  PsHalf<MU, false, 0>::at(own, a0);
  PsHalf<MU, false, 1>::at(own, a1);
  ps_colour<false>(uf, a0, cb[0]);
  ps_colour<false>(uf, a1, cb[1]);
  wave_order();
  const double kp = on ? kappa : 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (MU == kNumPS - 1) {  // t: the upper halves of both rows (the lower ones differ by a sign)
        own[3 * h + k] = on ? -kp * cf[h][k] : mk(0.0, 0.0);
        own[6 + 3 * h + k] = on ? kp * cb[h][k] : mk(0.0, 0.0);
      } else {
        const cx<double> lo = -kp * (cf[h][k] + cb[h][k]);
        own[3 * h + k] = on ? kp * (cb[h][k] - cf[h][k]) : mk(0.0, 0.0);
        if (h == 0) own[PsHalf<MU, true, 0>::PS * 3 + k] = on ? PsHalf<MU, true, 0>::phase(lo) : mk(0.0, 0.0);
        else own[PsHalf<MU, true, 1>::PS * 3 + k] = on ? PsHalf<MU, true, 1>::phase(lo) : mk(0.0, 0.0);
      }
    }
}

// Where component k of a row's vector is found at a site (place in LDS, site
// 0) and the quarter turns to apply to it.
__device__ inline void row_piece(int row, int k, int *off, int *turns) {
  const int s = k / 3, c = k % 3;
  *off = k;
  *turns = 0;
#pragma unroll
  for (int th = 0; th < kNumTheta; ++th)  // (Theta d)_sp = val d_col: g_col = conj(val) eta_sp
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
      if (row == th && kGamma[th].col[sp] == s) {
        *off = 3 * sp + c;
        *turns = kGamma[th].re[sp] == 1.0 ? 0 : kGamma[th].im[sp] == -1.0 ? 1 : kGamma[th].re[sp] == -1.0 ? 2 : 3;
      }
  if (row >= kNumTheta && row < kPsRows - 2) *off = (row - kNumTheta + 1) * kPsRegion + k;
  if (row == kPsRows - 2 || row == kPsRows - 1) {
    *off = kNumPS * kPsRegion + (row == kPsRows - 1 ? 6 : 0) + 3 * (s & 1) + c;
    *turns = row == kPsRows - 2 && s >= 2 ? 2 : 0;
  }
}

// The value of the lane next to this one (lane ^ 1).
__device__ inline double swap_pair(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, int(b), 0xB1, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), 0xB1, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// A single variant (ONE) takes v_mfma_f64_4x4x4, whose four blocks are the row
// groups with the same four columns: a quarter of the products and the same bits
// (rows and components lie in the lanes alike, and both instructions round
// alike).  Its d goes through LDS, loaded in 1 KB runs while the rows are made:
// straight from memory a load brings 64 bytes of one variant, and those loads
// were half of the kernel's time.  24^3 x 32, 16 right-hand sides, all operators:
// 2.19 ms a call (a local and a point-split kernel 2.98, the 16-column form 3.16).
//
// Workgroup order: the right-hand side varies fastest within one XCD's
// contiguous range of logical workgroups (hardware workgroup h runs on XCD
// h % 8), so the nrhs workgroups of one chunk of sites run back to back on
// one XCD and read its links from that XCD's L2 (links are as many bytes as
// one right-hand side's three fields).
template <bool ONE>
__global__ void __launch_bounds__(kBlock, 2)
    k_estimate_all(Geom g, const cx<double> *__restrict__ U, double kappa, const cx<double> *__restrict__ eta,
                   const cx<double> *__restrict__ x, XtSet xts, int nv, int nch, int nrhs, int xq,
                   double *__restrict__ out) {
  typedef double d4 __attribute__((ext_vector_type(4)));
  using Acc = typename std::conditional<ONE, double, d4>::type;
  __shared__ cx<double> reg[(1 + kNumPS + ONE) * kPsRegion];
  const int L = int(blockIdx.x % 8) * xq + int(blockIdx.x / 8);
  if (L >= g.L[3] * nch * nrhs) return;  // whole workgroup: padding of the grid
  const int r = L % nrhs, tch = L / nrhs;
  const int t = tch / nch, ch = tch % nch;
  const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2], Lt = g.L[3];
  const int Vs = Lx * Ly * Lz;
  const size_t Vh = size_t(g.Vh), base = size_t(r) * size_t(g.V) * 12;
  eta += base;
  const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  // product: lane = row l % 16 and column l % 16 (ONE: l % 4), components l / 16
  // of groups of four;
  // gr, gi: places (in doubles) of the real and imaginary part of the row's
  // components and the signs they take
  const int l16 = lane & 15, kq = lane >> 4, lcol = ONE ? lane & 3 : l16;
  int gr[3], gi[3];
  unsigned sr[3], si[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    int off, turns;
    row_piece(l16, 4 * j + kq, &off, &turns);
    off += q * (kPsSites / kWaves) * kPsStride;
    gr[j] = 2 * off + (turns & 1);
    gi[j] = 2 * off + 1 - (turns & 1);
    sr[j] = turns == 1 || turns == 2 ? 0x80000000u : 0u;
    si[j] = turns >= 2 ? 0x80000000u : 0u;
  }
  const double *xp = reinterpret_cast<const double *>(x + base) + 2 * kq + (lcol & 1), *tp = nullptr;
#pragma unroll
  for (int v = 0; v < kMaxVar; ++v)
    if (v < nv && v == lcol >> 1) tp = reinterpret_cast<const double *>(xts.p[v]);
  const double minus = tp ? -1.0 : 0.0;
  tp = tp ? tp + 2 * base + 2 * kq + (lcol & 1) : xp;
  const unsigned odd = (lcol & 1) ? 0x80000000u : 0u;
  Acc tot = {};
  for (int i0 = ch * kPsSites; i0 < Vs; i0 += nch * kPsSites) {
    const int i = i0 + lane;
    const bool on = i < Vs;
    const int c4[4] = {i % Lx, (i / Lx) % Ly, i / (Lx * Ly), t};
    const int par = (c4[0] + c4[1] + c4[2] + t) & 1;
    const int s = on ? t * Vs + i : 0;
    const int st = q == 0 ? 1 : q == 1 ? Lx : q == 2 ? Lx * Ly : Vs;
    const int Lm = g.L[q], cm = c4[q];
    const int sf = on ? (cm + 1 == Lm ? s - st * (Lm - 1) : s + st) : 0;
    const int sb = on ? (cm == 0 ? s + st * (Lm - 1) : s - st) : 0;
    __syncthreads();  // the previous chunk's products are done
    {  // eta at the sites: piece j = thread + 256 u (past the end: site 0, dropped)
      cx<double> v[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int j = threadIdx.x + u * kBlock;
        v[u] = ldc(eta + (size_t(t) * Vs + i0) * 12 + (i0 + j / 12 < Vs ? j : 0));
      }
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int j = threadIdx.x + u * kBlock;
        reg[j / 12 * kPsStride + j % 12] = i0 + j / 12 < Vs ? v[u] : mk(0.0, 0.0);
      }
    }
    cx<double> *mine = reg + (1 + q) * kPsRegion;
    cx<double> xr[3], tr[3];  // ONE: x and xt at the sites, pieces as eta's
    const cx<double> *x1 = x + base, *t1 = ONE && xts.p[0] ? xts.p[0] + base : nullptr;
    auto mid = [&] {
      if constexpr (ONE)
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          const int j = threadIdx.x + u * kBlock;
          const size_t o = (size_t(t) * Vs + i0) * 12 + (i0 + j / 12 < Vs ? j : 0);
          xr[u] = ldc(x1 + o);
          tr[u] = t1 ? ldc(t1 + o) : mk(0.0, 0.0);
        }
    };
    if (q == 0) ps_rows<0>(U, Vh, eta, kappa, s, sf, sb, par, on, mine, mid);
    else if (q == 1) ps_rows<1>(U, Vh, eta, kappa, s, sf, sb, par, on, mine, mid);
    else if (q == 2) ps_rows<2>(U, Vh, eta, kappa, s, sf, sb, par, on, mine, mid);
    else ps_rows<3>(U, Vh, eta, kappa, s, sf, sb, par, on, mine, mid);
    constexpr int NS = kPsSites / kWaves, BS = 2;
    Acc acc0 = {}, acc1 = {};  // of this chunk: short chains of sums round less
    const double *rd = reinterpret_cast<const double *>(reg);
    auto product = [&](int site, int j, double d) {
      const double a0 = flip(rd[gr[j] + site], sr[j]), a1 = flip(rd[gi[j] + site], si[j]);
      const double e = flip(swap_pair(d), odd);
      if constexpr (ONE) {
        acc0 = __builtin_amdgcn_mfma_f64_4x4x4f64(a0, d, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_4x4x4f64(a1, e, acc1, 0, 0, 0);
      } else {
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, d, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, e, acc1, 0, 0, 0);
      }
    };
    if constexpr (ONE) {
      cx<double> *ds = reg + (1 + kNumPS) * kPsRegion;
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int j = threadIdx.x + u * kBlock;
        ds[j / 12 * kPsStride + j % 12] = i0 + j / 12 < Vs ? xr[u] - tr[u] : mk(0.0, 0.0);
      }
      __syncthreads();
      const double *dd = reinterpret_cast<const double *>(ds + q * NS * kPsStride) + 2 * kq + (lcol & 1);
#pragma unroll
      for (int u = 0; u < NS; ++u)
#pragma unroll
        for (int j = 0; j < 3; ++j) product(2 * u * kPsStride, j, dd[2 * u * kPsStride + 8 * j]);
    } else {
      // products of the wave's 16 sites, two at a time, the next ones' d in
      // flight (sites past the end, whose rows are zero, read the last one)
      double xv[2][3 * BS], tv[2][3 * BS];
      const int w0 = i0 + q * NS;
      auto fetch = [&](int b, double *px, double *pt) {
#pragma unroll
        for (int u = 0; u < BS; ++u) {
          const size_t o = (size_t(t) * Vs + std::min(w0 + BS * b + u, Vs - 1)) * 24;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            px[3 * u + j] = xp[o + 8 * j];
            pt[3 * u + j] = tp[o + 8 * j];
          }
        }
      };
      fetch(0, xv[0], tv[0]);
      __syncthreads();
#pragma unroll
      for (int b = 0; b < NS / BS; ++b) {
        if (b + 1 < NS / BS) fetch(b + 1, xv[(b + 1) & 1], tv[(b + 1) & 1]);
#pragma unroll
        for (int u = 0; u < BS; ++u)
#pragma unroll
          for (int j = 0; j < 3; ++j)
            product(2 * (BS * b + u) * kPsStride, j, fma(minus, tv[b & 1][3 * u + j], xv[b & 1][3 * u + j]));
      }
    }
    tot += acc0 + acc1;
  }
  // the four waves' sums, in order
  __syncthreads();
  double *sh = reinterpret_cast<double *>(reg);
  if constexpr (ONE) {
    sh[q * 256 + (4 * ((lane >> 2) & 3) + kq) * 16 + lcol] = tot;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) sh[q * 256 + (kq + 4 * u) * 16 + l16] = tot[u];
  }
  __syncthreads();
  const int row = threadIdx.x >> 4, col = threadIdx.x & 15, v = col >> 1;
  if (row < kPsRows && v < nv) {
    const int trow = row == kPsRows - 2 ? (t == 0 ? Lt - 1 : t - 1) : row == kPsRows - 1 ? (t + 1 == Lt ? 0 : t + 1) : t;
    double sum = sh[threadIdx.x];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) sum += sh[w * 256 + threadIdx.x];
    out[((((size_t(v) * nrhs + r) * kOpSlots + row) * Lt + trow) * nch + ch) * 2 + (col & 1)] = sum;
  }
}

// Scratch of the allocation-free entry point loop_estimate_noalloc: the
// per-workgroup partial sums, in a fixed device array (one copy per GPU,
// held until the process ends).  Host code reaches it only through the
// address hipGetSymbolAddress returns for the current device.
constexpr size_t kNoallocDoubles = size_t(1) << 19;  // 4 MiB
static __device__ __align__(256) double scratch[kNoallocDoubles];

constexpr int kMaxDevices = 64;
std::mutex noalloc_mu;
double *noalloc_ptr[kMaxDevices] = {};

// The scratch array's device address on the current device, looked up on
// the first call there.
double *noalloc_scratch() {
  int dev = 0;
  LQCD_HIP(hipGetDevice(&dev));
  LQCD_CHECK(dev >= 0 && dev < kMaxDevices, LQCD_EDEVICE, "loop_estimate_noalloc: device %d out of range", dev);
  std::lock_guard<std::mutex> lk(noalloc_mu);
  if (!noalloc_ptr[dev]) {
    void *p = nullptr;
    LQCD_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    noalloc_ptr[dev] = static_cast<double *>(p);
  }
  return noalloc_ptr[dev];
}

// Chunks per timeslice: about 2048 workgroups in all, at least one site
// block each, and at most cap_doubles of partial sums (0: no cap).
int estimate_chunks(const Geom &g, int nrhs, size_t cap_doubles) {
  const int Lt = g.L[3], Vs = g.V / Lt;
  int nch = std::max(1, std::min((Vs + kBlock / 4 - 1) / (kBlock / 4), (2048 + Lt * nrhs - 1) / (Lt * nrhs)));
  if (cap_doubles)
    nch = std::max(1, std::min<int>(nch, int(cap_doubles / (size_t(nrhs) * kOpSlots * Lt * 2))));
  return nch;
}

// Variants per launch of the local kernel: its per-lane sums grow by 10
// doubles per variant, and at 24^3 x 32 with 16 right-hand sides groups of
// three are fastest (2.0 ms for six variants, 2.6 in pairs, 2.4 all at once).
constexpr int kLocalGroup = 3;

template <int NV>
void launch_local(lqcd_ctx *c, const void *eta, const void *x, const XtSet &xts, int v0, int nrhs, double *d,
                  int nch) {
  const Geom &g = c->g;
  const int Lt = g.L[3], Vs = g.V / Lt;
  hipLaunchKernelGGL(k_estimate<NV>, dim3(Lt * nch, nrhs), dim3(kBlock), 0, c->stream,
                     static_cast<const cx<double> *>(eta), static_cast<const cx<double> *>(x), xts, v0, size_t(g.V),
                     Vs, Lt, nch, d);
  LQCD_HIP(hipGetLastError());
}

void launch_all(lqcd_ctx *c, const void *eta, const void *x, const XtSet &xts, int nv, int nrhs, double *d,
                int nch) {
  const Geom &g = c->g;
  const int xq = (g.L[3] * nch * nrhs + 7) / 8;  // logical workgroups per XCD (grid padded to 8 xq)
  hipLaunchKernelGGL(nv == 1 ? k_estimate_all<true> : k_estimate_all<false>, dim3(8 * xq), dim3(kBlock), 0, c->stream,
                     g, static_cast<const cx<double> *>(c->U64.ptr), c->kappa, static_cast<const cx<double> *>(eta),
                     static_cast<const cx<double> *>(x), xts, nv, nch, nrhs, xq, d);
  LQCD_HIP(hipGetLastError());
}

// The estimator of nvar variants (subtracted vectors xt[v], corrections
// corr[v]) with its partial sums in d (at least nvar * nrhs * kOpSlots * Lt
// * nch * 2 doubles of device memory).  Variant v's outputs start at
// est + v * nth * (Lt + 1) * 2, stderr_ + (same), samples + v * nrhs * nth
// * (Lt + 1) * 2.
void estimate_with(lqcd_ctx *c, const int *thetas, int nth, const void *eta, const void *x,
                   const void *const *xt, int nvar, int nrhs, const double *const *corr, double *est,
                   double *stderr_, double *samples, double *d, int nch) {
  bool any_ps = false;
  for (int a = 0; a < nth; ++a) any_ps = any_ps || thetas[a] >= kNumTheta;
  auto group = [&](int v0, int n) {
    XtSet xts{};
    for (int v = 0; v < n; ++v) xts.p[v] = static_cast<const cx<double> *>(xt[v0 + v]);
    return xts;
  };
  // local operators alone need neither links nor neighbours: their own kernel
  if (any_ps) launch_all(c, eta, x, group(0, nvar), nvar, nrhs, d, nch);
  else
    for (int v0 = 0; v0 < nvar; v0 += kLocalGroup) {
      const XtSet xts = group(v0, std::min(kLocalGroup, nvar - v0));
      switch (nvar - v0) {
        case 1: launch_local<1>(c, eta, x, xts, v0, nrhs, d, nch); break;
        case 2: launch_local<2>(c, eta, x, xts, v0, nrhs, d, nch); break;
        default: launch_local<kLocalGroup>(c, eta, x, xts, v0, nrhs, d, nch); break;
      }
    }
  const int Lt = c->g.L[3];
  std::vector<double> hc(size_t(nvar) * nrhs * kOpSlots * Lt * nch * 2);
  LQCD_HIP(hipMemcpyAsync(hc.data(), d, hc.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  LQCD_HIP(hipStreamSynchronize(c->stream));
  const int W = Lt + 1;
  for (int var = 0; var < nvar; ++var) {
    const double *hv = hc.data() + size_t(var) * nrhs * kOpSlots * Lt * nch * 2;
    const double *cv = corr ? corr[var] : nullptr;
    double *ev = est + size_t(var) * nth * W * 2, *sv = stderr_ + size_t(var) * nth * W * 2;
    std::vector<double> h(size_t(nrhs) * kOpSlots * Lt * 2, 0.0);
    for (size_t o = 0; o < h.size() / 2; ++o)
      for (int ch = 0; ch < nch; ++ch) {
        h[2 * o] += hv[(o * nch + ch) * 2];
        h[2 * o + 1] += hv[(o * nch + ch) * 2 + 1];
      }
    // samples [n][a][t], t = Lt the total
    std::vector<cdouble> smp(size_t(nrhs) * nth * W);
    for (int n = 0; n < nrhs; ++n)
      for (int a = 0; a < nth; ++a) {
        cdouble tot = 0;
        for (int t = 0; t < Lt; ++t) {
          size_t o = ((size_t(n) * kOpSlots + thetas[a]) * Lt + t) * 2;
          cdouble v(h[o], h[o + 1]);
          if (thetas[a] == kNumOps - 1) {  // point-split in t: its second slot
            const size_t o2 = ((size_t(n) * kOpSlots + kNumOps) * Lt + t) * 2;
            v += cdouble(h[o2], h[o2 + 1]);
          }
          smp[(size_t(n) * nth + a) * W + t] = v;
          tot += v;
        }
        smp[(size_t(n) * nth + a) * W + Lt] = tot;
      }
    for (int a = 0; a < nth; ++a)
      for (int t = 0; t < W; ++t) {
        cdouble mean = 0;
        for (int n = 0; n < nrhs; ++n) mean += smp[(size_t(n) * nth + a) * W + t];
        mean /= double(nrhs);
        double vr = 0, vi = 0;
        for (int n = 0; n < nrhs; ++n) {
          cdouble dv = smp[(size_t(n) * nth + a) * W + t] - mean;
          vr += dv.real() * dv.real();
          vi += dv.imag() * dv.imag();
        }
        double ser = 0, sei = 0;
        if (nrhs > 1) {
          ser = std::sqrt(vr / (nrhs - 1) / nrhs);
          sei = std::sqrt(vi / (nrhs - 1) / nrhs);
        }
        cdouble cr = 0;
        if (cv) {
          if (t < Lt) {
            cr = cdouble(cv[2 * (a * Lt + t)], cv[2 * (a * Lt + t) + 1]);
          } else {
            for (int s = 0; s < Lt; ++s) cr += cdouble(cv[2 * (a * Lt + s)], cv[2 * (a * Lt + s) + 1]);
          }
        }
        cdouble e = mean + cr;
        ev[2 * (a * W + t)] = e.real();
        ev[2 * (a * W + t) + 1] = e.imag();
        sv[2 * (a * W + t)] = ser;
        sv[2 * (a * W + t) + 1] = sei;
      }
    if (samples) {
      double *pv = samples + size_t(var) * nrhs * nth * W * 2;
      for (size_t i = 0; i < smp.size(); ++i) {
        pv[2 * i] = smp[i].real();
        pv[2 * i + 1] = smp[i].imag();
      }
    }
  }
}

void check_args(lqcd_ctx *c, const int *thetas, int nth, const void *eta, const void *x, int nrhs,
                const double *est, const double *stderr_, const char *who) {
  LQCD_CHECK(c && eta && x && est && stderr_, LQCD_EINVAL, "%s: null argument", who);
  LQCD_CHECK(nrhs >= 1, LQCD_EINVAL, "%s: need at least one noise vector", who);
  LQCD_CHECK(nth >= 1 && thetas, LQCD_EINVAL, "%s: no operator", who);
  for (int a = 0; a < nth; ++a)
    LQCD_CHECK(thetas[a] >= 0 && thetas[a] < kNumOps, LQCD_EINVAL, "%s: operator code %d outside 0..8", who,
               thetas[a]);
}

}  // namespace
}  // namespace lqcd

using namespace lqcd;

extern "C" lqcd_status loop_estimate(lqcd_ctx *c, const int *thetas, int nth, const void *eta,
                                     const void *x, const void *xt, int nrhs, const double *corr,
                                     double *est, double *stderr_, double *samples) {
  return guarded([&] {
    check_args(c, thetas, nth, eta, x, nrhs, est, stderr_, "loop_estimate");
    const int nch = estimate_chunks(c->g, nrhs, 0);
    double *d = static_cast<double *>(
        c->red.ensure(size_t(nrhs) * kOpSlots * c->g.L[3] * nch * 2 * sizeof(double)));
    estimate_with(c, thetas, nth, eta, x, &xt, 1, nrhs, &corr, est, stderr_, samples, d, nch);
  });
}

extern "C" lqcd_status loop_estimate_multi(lqcd_ctx *c, const int *thetas, int nth, const void *eta,
                                           const void *x, const void *const *xt_list, int nvar, int nrhs,
                                           const double *const *corr_list, double *est, double *stderr_,
                                           double *samples) {
  return guarded([&] {
    check_args(c, thetas, nth, eta, x, nrhs, est, stderr_, "loop_estimate_multi");
    LQCD_CHECK(xt_list && nvar >= 1 && nvar <= kMaxVar, LQCD_EINVAL,
               "loop_estimate_multi: %d variants (1..%d, with a list of subtracted vectors)", nvar, kMaxVar);
    const int nch = estimate_chunks(c->g, nrhs, 0);
    double *d = static_cast<double *>(
        c->red.ensure(size_t(nvar) * nrhs * kOpSlots * c->g.L[3] * nch * 2 * sizeof(double)));
    estimate_with(c, thetas, nth, eta, x, xt_list, nvar, nrhs, corr_list, est, stderr_, samples, d, nch);
  });
}

extern "C" lqcd_status loop_estimate_noalloc(lqcd_ctx *c, const int *thetas, int nth, const void *eta,
                                             const void *x, const void *xt, int nrhs, const double *corr,
                                             double *est, double *stderr_, double *samples) {
  return guarded([&] {
    check_args(c, thetas, nth, eta, x, nrhs, est, stderr_, "loop_estimate_noalloc");
    const size_t one = size_t(nrhs) * kOpSlots * c->g.L[3] * 2;
    LQCD_CHECK(one <= kNoallocDoubles, LQCD_EINVAL,
               "loop_estimate_noalloc: %d right-hand sides x %d timeslices need %zu partial sums, more than "
               "the fixed scratch of %zu (use loop_estimate)",
               nrhs, c->g.L[3], one, kNoallocDoubles);
    double *d = noalloc_scratch();
    const int nch = estimate_chunks(c->g, nrhs, kNoallocDoubles);
    estimate_with(c, thetas, nth, eta, x, &xt, 1, nrhs, &corr, est, stderr_, samples, d, nch);
  });
}
