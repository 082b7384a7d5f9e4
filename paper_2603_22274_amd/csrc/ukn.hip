// Cross-lambda reduced potentials u_k(x_n) for MBAR (section "Simulation
// protocol").  With ligand charges scaled by lambda_e (section "Double
// annihilation protocol") a window's potential is
//   U_k = U_env + lam_e E_LE + lam_e^2 E_LL + E_sc(lam_v) + lam_r U_B,
// U_env is lambda-independent and dropped (MBAR is invariant to it).
//   E_LE: ligand-environment real-space erfc Coulomb + reciprocal cross term
//         sum_{i in L} q_i phi_E(r_i) + background cross term;
//   E_LL: ligand-ligand real-space Coulomb over non-excluded pairs, minus
//         erf terms of excluded pairs, 1/2 sum_{i in L} q_i phi_L(r_i),
//         ligand self term, ligand background term;
//   E_sc: softcore LJ of every ligand pair (ligand-environment and
//         non-excluded ligand-ligand) at lambda_ij = lam_v;
//   U_B:  Boresch energy.
// The reciprocal parts need only the ligand's potential phi_L: the PME
// reciprocal energy is a symmetric bilinear form of two spread charge grids,
// so sum_{i in L} q_i phi_E(r_i) = sum_{j in E} q_j phi_L(r_j).  Each frame
// spreads its few ligand charges, two frames share one complex FFT (real and
// imaginary part), and phi_L is gathered at every atom: a read-only pass over
// the environment instead of scattering all of its charges.  Pair distances
// and the softcore LJ are FP64 (a frame evaluated at a state it was not
// sampled in can hold r^-12 overlaps of 1e6 kT), the erfc Coulomb FP32; pair
// sums run in FP64 per lane; block partials combine in a fixed order (pair
// terms) or in int64 fixed point (reciprocal terms).  Frames may each have
// their own box (NPT); with a pressure, u gains beta P V of the frame.
#include "felis_internal.h"
#include "erfc_coeffs.h"
#include "restraint.h"

#include <algorithm>

namespace felis {
namespace {

struct UknArgs {
  const float *fx, *fy, *fz;
  long long stride, f0;
  int nf, KV;
  int upk;                             // 1: one frame per complex grid (frames in their own boxes)
  float lamv[kMaxLamV];
  float asc[kMaxLamV];
};

constexpr int kUknAtoms = 256;       // atoms per block of k_ukn_pairs, one a thread
__host__ __device__ inline int ukn_pair_blocks(int n) { return (n + kUknAtoms - 1) / kUknAtoms; }

constexpr int kNU = 3 + kMaxLamV;    // accumulators per frame: LE, LL, UB, UT (slot 3; rest unused)

__device__ __forceinline__ float erfc_fit(float x, float* ex) {
  const float t = __builtin_amdgcn_rcpf(fmaf(FELIS_ERFC_P, x, 1.0f));
  float p = felis_erfc_c[0];
#pragma unroll
  for (int k = 1; k < FELIS_ERFC_NC; ++k) p = fmaf(p, t, felis_erfc_c[k]);
  const float e = __expf(-x * x);
  *ex = e;
  return p * t * e;
}

__device__ __forceinline__ void bspline4(float f, float* w) {
  const float f2 = f * f, f3 = f2 * f, g1 = 1.0f - f;
  w[0] = f3 * (1.0f / 6.0f);
  w[1] = (-3.0f * f3 + 3.0f * f2 + 3.0f * f + 1.0f) * (1.0f / 6.0f);
  w[2] = (3.0f * f3 - 6.0f * f2 + 4.0f) * (1.0f / 6.0f);
  w[3] = g1 * g1 * g1 * (1.0f / 6.0f);
}


__device__ __forceinline__ float3 min_img(const BoxW& B, float dx, float dy, float dz) {
  dx = fmaf(-B.Lf[0], rintf(dx * B.invLf[0]), dx);
  dy = fmaf(-B.Lf[1], rintf(dy * B.invLf[1]), dy);
  dz = fmaf(-B.Lf[2], rintf(dz * B.invLf[2]), dz);
  return make_float3(dx, dy, dz);
}

// The alchemical charge set B: the ligand atoms, then the alchemical-water
// atoms.  A window's charges are a + lambda_elec b: b is the ligand charge
// (minus the offset on an alchemical water, zero elsewhere) and a the
// environment charge plus the offset (zero on ligand atoms), so the
// electrostatic energy is E[a,a] + lambda_elec 2 E[a,b] + lambda_elec^2
// E[b,b]; E_LE = 2 E[a,b] and E_LL = E[b,b].
__device__ __forceinline__ int bset_atom(const LegDev& g, int t) {
  return t < g.nlig ? g.lig_idx[t] : g.aw_idx[t - g.nlig];
}
__device__ __forceinline__ float charge_b(const LegDev& g, int a) {
  return g.lig[a] ? g.q[a] : (g.aoff ? -g.aoff[a] : 0.0f);
}
__device__ __forceinline__ float charge_a(const LegDev& g, int a) {
  return g.lig[a] ? 0.0f : (g.aoff ? g.q[a] + g.aoff[a] : g.q[a]);
}

__device__ __forceinline__ void acc_add(const LegDev& g, int f, int slot, double e) {
  atomicAdd((unsigned long long*)&g.uacc[(size_t)f * kNU + slot],
            (unsigned long long)to_fixed(e, kEnergyScale, g.err, kSiteUkn, f));
}

// items: frame x atom of the alchemical charge set, 16 lanes per atom: the
// b charges of frame f into int64 grid f
__global__ __launch_bounds__(256) void k_ukn_spread(const LegDev* legs, UknArgs A) {
  const LegDev& g = legs[0];
  const int nB = g.nlig + g.naw;
  const long long local = (long long)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (local >= (long long)A.nf * nB) return;
  const int f = (int)(local / nB);
  const int a = bset_atom(g, (int)(local - (long long)f * nB));
  const int sub = threadIdx.x & 15, iy = sub & 3, iz = sub >> 2;
  const size_t o = (size_t)(A.f0 + f) * A.stride + a;
  float fxr, fyr, fzr, wx[4], wy[4], wz[4];
  const BoxW& B = g.ubox[f];
  const int bx = grid_base(A.fx[o], B.invL[0], g.K[0], &fxr);
  const int by = grid_base(A.fy[o], B.invL[1], g.K[1], &fyr);
  const int bz = grid_base(A.fz[o], B.invL[2], g.K[2], &fzr);
  bspline4(fxr, wx); bspline4(fyr, wy); bspline4(fzr, wz);
  int gy = by - iy; if (gy < 0) gy += g.K[1];
  int gz = bz - iz; if (gz < 0) gz += g.K[2];
  // int64 grids 2p, 2p+1 become the real and imaginary parts of complex grid
  // p: frame f takes grid f, or grid 2f (imaginary part left zero) when
  // every frame has a grid of its own
  long long* grid = g.grid64 + (size_t)(A.upk ? 2 * f : f) * g.Ktot + ((size_t)gz * g.K[1] + gy) * g.K[0];
  // the transform skips the rows and planes that no charge reaches
  const int nch = ukn_chunks(g.K[1]);
  int* flag = ukn_flags(g, A.upk ? f : f >> 1);
  flag[gz * nch + (gy >> 4)] = 1;
  flag[g.K[2] * nch + gz] = 1;
  const double qyz = (double)(charge_b(g, a) * wy[iy] * wz[iz]);
#pragma unroll
  for (int ix = 0; ix < 4; ++ix) {
    int gx = bx - ix; if (gx < 0) gx += g.K[0];
    const long long v = __double2ll_rn(qyz * (double)wx[ix] * kGridScale);
    if (v) atomicAdd((unsigned long long*)&grid[gx], (unsigned long long)v);
  }
}

// lane's value from lane `AXIS` of its quad
template <int AXIS>
__device__ __forceinline__ float quad_from(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), AXIS * 0x55, 0xf, 0xf, true));
}
template <int AXIS>
__device__ __forceinline__ int quad_from(int v) {
  return __builtin_amdgcn_update_dpp(0, v, AXIS * 0x55, 0xf, 0xf, true);
}
// items: frame x block of 256 atoms, 4 lanes per atom, 64 atoms per pass:
// phi_b of frame f (phi) at every atom;
// E_LE += a phi_b, E_LL += b phi_b / 2 over all atoms.  The FP64 grid position
// and the spline weights of an axis are the work here (an atom's 64 points are
// 64 FMAs): lane k of the quad makes those of axis k and the quad shares them.
// Lane k reads the points at x - k, so a quad reads 4 neighbours of one row at
// a time (a load of the wave touches 16 rows, not 64), a transpose within the
// quad hands lane k the rows of plane z - k, and it sums them.  42 frames of
// 70,527 atoms: 389 us with 16 lanes an atom, each making all three axes; 290
// us with lane k reading its own plane's rows of the complex grid, 181 us from
// phi's 128-byte lines.
__global__ __launch_bounds__(256) void k_ukn_gather(const LegDev* legs, UknArgs A) {
#pragma clang fp contract(off)
  const LegDev& g = legs[0];
  const int nb = (g.n + 255) / 256;
  const int f = blockIdx.x / nb;
  const int a0 = (blockIdx.x - f * nb) * 256 + (threadIdx.x >> 2);
  const int iz = threadIdx.x & 3;
  const PhiLines ln(g.K);
  const float* phi = g.phi + (size_t)(A.upk ? 2 * f : f) * ln.size;
  const BoxW& B = g.ubox[f];
  const size_t fo = (size_t)(A.f0 + f) * A.stride;
  const float* pos = iz == 0 ? A.fx : (iz == 1 ? A.fy : A.fz);
  const double invL = iz == 0 ? B.invL[0] : (iz == 1 ? B.invL[1] : B.invL[2]);
  const int Kx = g.K[0], Ky = g.K[1], Kz = g.K[2];
  const int Kd = iz == 0 ? Kx : (iz == 1 ? Ky : Kz);
  const bool b0 = iz & 1, b1 = iz & 2;
  double le = 0.0, ll = 0.0;
  float xp[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) xp[t] = pos[fo + min(a0 + 64 * t, g.n - 1)];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int a = a0 + 64 * t;
    const bool valid = a < g.n;                      // uniform over the quad
    const int ac = valid ? a : g.n - 1;
    float fr, w[4];
    const int b = grid_base(xp[t], invL, Kd, &fr);
    bspline4(fr, w);
    const int bx = quad_from<0>(b), by = quad_from<1>(b), bz = quad_from<2>(b);
    float wx[4], wy[4], wz[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      wx[k] = quad_from<0>(w[k]);
      wy[k] = quad_from<1>(w[k]);
      wz[k] = quad_from<2>(w[k]);
    }
    const float wzk = iz == 0 ? wz[0] : (iz == 1 ? wz[1] : (iz == 2 ? wz[2] : wz[3]));
    int gx = bx - iz; if (gx < 0) gx += Kx;
    int plane[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) { plane[m] = bz - m; if (plane[m] < 0) plane[m] += Kz; plane[m] = ln.z(plane[m]); }
    float r[4][4];
#pragma unroll
    for (int iy = 0; iy < 4; ++iy) {
      int gy = by - iy; if (gy < 0) gy += Ky;
      const int xy = ln.x(gx) + ln.y(gy);
#pragma unroll
      for (int m = 0; m < 4; ++m) r[iy][m] = phi[xy + plane[m]];
    }
    float p[4], wyz[4];
#pragma unroll
    for (int iy = 0; iy < 4; ++iy) {
      quad_transpose(r[iy], b0, b1);
      p[iy] = 0.f;
#pragma unroll
      for (int ix = 0; ix < 4; ++ix) p[iy] = fmaf(wx[ix], r[iy][ix], p[iy]);
      wyz[iy] = wy[iy] * wzk;
    }
    float ph = fmaf(p[0], wyz[0], p[1] * wyz[1]) + fmaf(p[2], wyz[2], p[3] * wyz[3]);
    ph += quad_xor1(ph);
    ph += quad_xor2(ph);
    if (iz == 0 && valid) {
      le += (double)charge_a(g, ac) * (double)ph;
      ll += 0.5 * (double)charge_b(g, ac) * (double)ph;
    }
  }
  le = wave_sum(le);
  ll = wave_sum(ll);
  __shared__ double s_r[2][4];
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { s_r[0][wv] = le; s_r[1][wv] = ll; }
  __syncthreads();
  if (threadIdx.x == 0) {
    acc_add(g, f, 0, ((s_r[0][0] + s_r[0][1]) + s_r[0][2]) + s_r[0][3]);
    acc_add(g, f, 1, ((s_r[1][0] + s_r[1][1]) + s_r[1][2]) + s_r[1][3]);
  }
}


// The softcore queue of one wave: pairs in range wait here until 64 are
// together, then the lanes share them out over the lambda_vdw values
struct ScQueue {
  double s6[128], r6[128], e4[128];
};

struct ScLane {                      // a lane's lambda_vdw value, its share of the queued pairs, its sum
  int group, groups;
  double lam, asc, sum;
};

// lanes 0 .. KV groups - 1 take value lane % KV and every groups-th pair
__device__ __forceinline__ ScLane sc_lane(const UknArgs& A, int lane) {
  ScLane L;
  L.groups = 64 / A.KV;
  L.group = lane / A.KV;
  const int v = lane - L.group * A.KV;
  L.lam = (double)A.lamv[v];
  L.asc = (double)A.asc[v];
  L.sum = 0.0;
  return L;
}

__device__ __forceinline__ void sc_eval(const ScQueue& Q, int first, int count, ScLane& L) {
  if (L.group < L.groups)
    for (int p = L.group; p < count; p += L.groups) {
      const double s6 = Q.s6[first + p];
      const double u = s6 / fma(L.asc, s6, Q.r6[first + p]);
      L.sum += L.lam * Q.e4[first + p] * fma(u, u, -u);
    }
}

// push the lanes with `in` set; evaluate when a wave's worth is queued
__device__ __forceinline__ void sc_push(ScQueue& Q, int& nq, bool in, double s6, double r6, double e4, int lane,
                                        ScLane& L) {
  const unsigned long long m = __ballot(in);
  if (in) {
    const int at = nq + __popcll(m & ((1ull << lane) - 1ull));
    Q.s6[at] = s6; Q.r6[at] = r6; Q.e4[at] = e4;
  }
  nq += __popcll(m);
  wave_lds_fence();
  if (nq >= 64) {
    nq -= 64;
    sc_eval(Q, nq, 64, L);
    wave_lds_fence();
  }
}

// the block's sums, one slot per lambda_vdw value (1 + v) and slot 0, in a
// fixed order (waves, then a wave's groups of lanes)
__device__ __forceinline__ void sc_flush(const UknArgs& A, double (*s_sum)[64], double* s_e0, double e0, const ScLane& L,
                                         double* out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  e0 = wave_sum(e0);
  __syncthreads();
  s_sum[wave][lane] = L.group < L.groups ? L.sum : 0.0;
  if (lane == 0) s_e0[wave] = e0;
  __syncthreads();
  for (int t = threadIdx.x; t < 1 + A.KV; t += blockDim.x) {
    double v = 0.0;
    if (t == 0) {
      v = ((s_e0[0] + s_e0[1]) + s_e0[2]) + s_e0[3];
    } else {
      for (int w = 0; w < 4; ++w)
        for (int k = 0; k < L.groups; ++k) v += s_sum[w][k * A.KV + t - 1];
    }
    out[t] = v;
  }
}

// Frame f's ligand block: pairs within the alchemical charge set (Coulomb of
// the b charges; softcore LJ between ligand atoms), excluded-pair corrections,
// the Boresch energy and the torsions; one partial row per frame (slot 0 E_LL
// real space, 1 + kv softcore LJ)
__device__ __forceinline__ void ukn_ligand(const LegDev& g, const UknArgs& A, int f, ScQueue& Q, double (*s_sum)[64],
                                           double* s_e0) {
  const size_t fo = (size_t)(A.f0 + f) * A.stride;
  const int nl = g.nlig + g.naw;                 // the alchemical charge set
  const int np = nl * (nl - 1) / 2;
  const int lane = threadIdx.x & 63;
  const float c_ke = (float)kKE;
  const BoxW& B = g.ubox[f];
  double ell = 0.0;
  int nq = 0;
  ScLane SL = sc_lane(A, lane);
  for (int base = 0; base < np; base += blockDim.x) {
    const int p = base + threadIdx.x;
    bool in = false;
    double r2s = 1.0, s6 = 0.0, e4 = 0.0;
    if (p < np) {
      // p -> (i, j), i < j, row-major over the upper triangle: row i starts at
      // i (2 nl - 1 - i) / 2; the FP32 root is within one row
      const float h = (float)(2 * nl - 1);
      int i = (int)(0.5f * (h - sqrtf(fmaxf(h * h - 8.0f * (float)p, 0.0f))));
      i = max(0, min(i, nl - 2));
      while (i > 0 && i * (2 * nl - 1 - i) / 2 > p) --i;
      while ((i + 1) * (2 * nl - 2 - i) / 2 <= p) ++i;
      const int jl = i + 1 + p - i * (2 * nl - 1 - i) / 2;
      const int a = bset_atom(g, i), b = bset_atom(g, jl);
      const bool both_lig = i < g.nlig && jl < g.nlig;   // softcore only between ligand atoms
      bool exc = false;
      for (int k = g.excl_ptr[a]; k < g.excl_ptr[a + 1]; ++k) exc |= (g.excl_idx[k] == b);
      double dxd = (double)A.fx[fo + b] - (double)A.fx[fo + a];
      double dyd = (double)A.fy[fo + b] - (double)A.fy[fo + a];
      double dzd = (double)A.fz[fo + b] - (double)A.fz[fo + a];
      dxd = fma(-B.L[0], rint(dxd * B.invL[0]), dxd);
      dyd = fma(-B.L[1], rint(dyd * B.invL[1]), dyd);
      dzd = fma(-B.L[2], rint(dzd * B.invL[2]), dzd);
      const double r2d = fma(dxd, dxd, fma(dyd, dyd, dzd * dzd));
      const float r2 = (float)r2d;
      const float qq = c_ke * charge_b(g, a) * charge_b(g, b);
      if (exc) {
        const float r = sqrtf(r2);
        ell -= (r > 1e-4f) ? (double)(qq * erff(g.alpha * r) / r)
                           : (double)(qq * 2.0f * g.alpha * 0.56418958354775628f);
      } else if (r2d < g.rc2d) {
        in = both_lig;
        r2s = r2d;
        const float rinv = __builtin_amdgcn_rsqf(r2);
        float ex;
        ell += (double)(qq * erfc_fit(g.alpha * r2 * rinv, &ex) * rinv);
        const double sg = 0.5 * ((double)g.sig[a] + (double)g.sig[b]);
        const double s2 = sg * sg;
        s6 = s2 * s2 * s2;
        e4 = 4.0 * sqrt((double)g.eps[a] * (double)g.eps[b]);
      }
    }
    sc_push(Q, nq, in, s6, r2s * r2s * r2s, e4, lane, SL);
  }
  sc_eval(Q, 0, nq, SL);
  sc_flush(A, s_sum, s_e0, ell, SL, g.lpart + (size_t)f * (1 + kMaxLamV));
  if (threadIdx.x == 0 && g.has_rest) {
    v3 p[6];
    const size_t o1 = fo + g.ranch[0];
    for (int t = 0; t < 6; ++t) {
      const size_t ot = fo + g.ranch[t];
      const float3 d = min_img(B, A.fx[ot] - A.fx[o1], A.fy[ot] - A.fy[o1], A.fz[ot] - A.fz[o1]);
      p[t] = mk(d.x, d.y, d.z);
    }
    acc_add(g, f, 2, boresch_eval(p, g.rg0, g.rk, nullptr));
  }
  if (threadIdx.x == 64 && g.ntors > 0) {
    // rotatable torsions, unscaled, in FP64 (slot 3)
    double ut = 0.0;
    for (int t = 0; t < g.ntors; ++t) {
      const size_t o0 = fo + g.tors[4 * t];
      double p[4][3];
      for (int s = 0; s < 4; ++s) {
        const size_t os = fo + g.tors[4 * t + s];
        double d[3] = {(double)A.fx[os] - (double)A.fx[o0], (double)A.fy[os] - (double)A.fy[o0],
                       (double)A.fz[os] - (double)A.fz[o0]};
        for (int c = 0; c < 3; ++c) p[s][c] = d[c] - B.L[c] * rint(d[c] * B.invL[c]);
      }
      ut += torsion_energy_fp64(p, (double)g.tors_k[t], g.tors_n[t], (double)g.tors_phase[t]);
    }
    acc_add(g, f, 3, ut);
  }
}

// The constants of E_LE / E_LL that depend only on charges: the self terms and
// the two background terms (one block of 256 threads, eight atoms a thread in
// flight)
__device__ __forceinline__ void ukn_const(const LegDev& g, double* out) {
  double qa = 0.0, qb = 0.0, qb2 = 0.0, qab = 0.0;
  const float* q = g.q;
  const float* off = g.aoff;
  const uint8_t* lig = g.lig;
  const int n = g.n;
  for (int a0 = threadIdx.x; a0 < n; a0 += 8 * 256) {
    float qv[8], ov[8];
    bool lv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int a = min(a0 + 256 * k, n - 1);
      qv[k] = q[a];
      lv[k] = lig[a] != 0;
      ov[k] = off ? off[a] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (a0 + 256 * k >= n) continue;
      const double ca = lv[k] ? 0.0 : (double)(qv[k] + ov[k]), cb = lv[k] ? (double)qv[k] : -(double)ov[k];
      qa += ca; qb += cb; qb2 += cb * cb; qab += ca * cb;
    }
  }
  __shared__ double r[4][4];
  qa = wave_sum(qa); qb = wave_sum(qb); qb2 = wave_sum(qb2); qab = wave_sum(qab);
  if ((threadIdx.x & 63) == 0) {
    const int w = threadIdx.x >> 6;
    r[0][w] = qa; r[1][w] = qb; r[2][w] = qb2; r[3][w] = qab;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t[4];
    for (int k = 0; k < 4; ++k) t[k] = ((r[k][0] + r[k][1]) + r[k][2]) + r[k][3];
    out[0] = 2.0 * t[0] * t[1];             // E_LE background / (-bg_pref)
    out[1] = t[1] * t[1];                   // E_LL background / (-bg_pref)
    out[2] = -g.self_pref * t[2];           // E_LL self term
    out[3] = -2.0 * g.self_pref * t[3];     // E_LE self term (atoms with both a and b charges)
  }
}

// items: frame x (blocks of kUknAtoms atoms, and one ligand block): pairs of
// the alchemical charge set with environment atoms within r_c (an alchemical
// water's own atoms: excluded-pair erf correction), softcore LJ for the
// ligand entries.  One block partial per frame, block and slot (slot 0
// Coulomb, 1 + kv softcore LJ at lamv[kv]), unbounded (a frame evaluated at a
// state it was not sampled in may carry enormous overlap energies) and summed
// in a fixed order by k_ukn_combine.
//
// A few percent of the atoms lie near the ligand, and a quarter of those are
// in range of a given ligand atom, so the block drops atoms in two steps: by
// the ligand's bounding sphere (and each alchemical-water atom) into a list in
// LDS, then the (listed atom, set entry) pairs are shared out over all lanes,
// and those in range are queued per wave for the softcore sums, where the
// lanes take one lambda_vdw value each.  The first block sums the charges'
// constants (a serial pass of its own otherwise).  42 frames of 70,527 atoms, 50 ligand
// atoms, 20 values: 525 + 45 us with a lane per atom looping over the ligand
// and the values; 120 us so, beside the transform on its own stream.
__global__ __launch_bounds__(256) void k_ukn_pairs(const LegDev* legs, UknArgs A, double* cst) {
  const LegDev& g = legs[0];
  if (blockIdx.x == 0) {                  // uniform
    ukn_const(g, cst);
    return;
  }
  const int nb = ukn_pair_blocks(g.n);
  const int f = (blockIdx.x - 1) / (nb + 1);
  const int blk = (int)blockIdx.x - 1 - f * (nb + 1);
  __shared__ ScQueue s_q[4];
  __shared__ double s_sum[4][64], s_e0[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blk == nb) {                        // uniform
    ukn_ligand(g, A, f, s_q[wave], s_sum, s_e0);
    return;
  }
  __shared__ float4 s_lx[kMaxLigand];     // x, y, z, b charge
  __shared__ float2 s_lp[kMaxLigand];     // sigma/2, eps (ligand entries)
  __shared__ int3 s_aw[kMaxLigand];       // alchemical-water entries: the atom and its two exclusion partners
  __shared__ float4 s_jx[kUknAtoms];      // listed atoms: x, y, z, a charge
  __shared__ float2 s_jp[kUknAtoms];      // sigma, eps
  __shared__ int s_jj[kUknAtoms];         // atom index
  __shared__ int s_cnt[4];
  const size_t fo = (size_t)(A.f0 + f) * A.stride;
  const BoxW& B = g.ubox[f];
  const int nB = g.nlig + g.naw;
  double* out = g.upart + (size_t)(f * nb + blk) * (1 + kMaxLamV);
  // an atom farther than r_c from the ligand's sphere is out of every ligand
  // atom's range (0.05 A covers the FP32 distances)
  const int j = blk * kUknAtoms + tid, jc = min(j, g.n - 1);
  const float xj = A.fx[fo + jc], yj = A.fy[fo + jc], zj = A.fz[fo + jc];
  const bool env = j < g.n && !g.lig[jc];
  const float4 sph = g.usph[f];
  const float rc = sqrtf((float)g.rc2d) + 0.05f;
  float3 d0 = min_img(B, xj - sph.x, yj - sph.y, zj - sph.z);
  const float reach = rc + sph.w;
  bool near = g.nlig && !(d0.x * d0.x + d0.y * d0.y + d0.z * d0.z > reach * reach);
  for (int t = g.nlig; t < nB; ++t) {     // alchemical-water atoms
    const int a = bset_atom(g, t);
    d0 = min_img(B, xj - A.fx[fo + a], yj - A.fy[fo + a], zj - A.fz[fo + a]);
    near |= !(d0.x * d0.x + d0.y * d0.y + d0.z * d0.z > rc * rc);
  }
  near &= env;
  const unsigned long long nm = __ballot(near);
  if (lane == 0) s_cnt[wave] = __popcll(nm);
  __syncthreads();
  const int nn = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
  if (nn == 0) {                          // uniform: nothing near
    for (int t = tid; t < 1 + A.KV; t += 256) out[t] = 0.0;
    return;
  }
  if (near) {
    int at = __popcll(nm & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) at += s_cnt[w];
    s_jx[at] = make_float4(xj, yj, zj, charge_a(g, j));
    s_jp[at] = make_float2(g.sig[j], g.eps[j]);
    s_jj[at] = j;
  }
  if (tid < nB) {                         // at most kMaxLigand = 256 entries
    const int a = bset_atom(g, tid);
    s_lx[tid] = make_float4(A.fx[fo + a], A.fy[fo + a], A.fz[fo + a], charge_b(g, a));
    s_lp[tid] = make_float2(0.5f * g.sig[a], g.eps[a]);
    if (tid >= g.nlig) {
      const int k = tid - g.nlig;
      s_aw[tid] = make_int3(a, g.aw_idx[g.naw + 2 * k], g.aw_idx[g.naw + 2 * k + 1]);
    }
  }
  __syncthreads();
  const double Lx = B.L[0], Ly = B.L[1], Lz = B.L[2], iLx = B.invL[0], iLy = B.invL[1], iLz = B.invL[2];
  const float c_ke = (float)kKE;
  double ec = 0.0;
  int nq = 0;
  ScLane SL = sc_lane(A, lane);
  const int total = nn * nB;              // at most 256 x 256
  const float inv = 1.0f / (float)nB;
  for (int base = 0; base < total; base += 256) {
    const int t = base + tid;
    bool in = false, soft = false;
    double s6 = 0.0, r6 = 1.0, e4 = 0.0;
    if (t < total) {
      int nj = (int)((float)t * inv);     // quotient within one, t < 2^22
      nj += (t - nj * nB < 0) ? -1 : (t - nj * nB >= nB ? 1 : 0);
      const int li = t - nj * nB;
      const float4 L = s_lx[li], J = s_jx[nj];
      const bool awe = li >= g.nlig;      // an alchemical-water entry (no softcore)
      // the distance in FP64 (minimum image included): a frame evaluated at a
      // state it was not sampled in can hold r^-12 overlaps of 1e6 kT, where
      // FP32 distances would lose six digits
      double dx = (double)J.x - (double)L.x, dy = (double)J.y - (double)L.y, dz = (double)J.z - (double)L.z;
      dx = fma(-Lx, rint(dx * iLx), dx);
      dy = fma(-Ly, rint(dy * iLy), dy);
      dz = fma(-Lz, rint(dz * iLz), dz);
      const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
      in = r2 < g.rc2d;
      bool exc = false;
      if (awe) {
        const int3 e3 = s_aw[li];
        const int jj = s_jj[nj];
        in = in && jj != e3.x;            // never the water's own atom
        exc = in && (jj == e3.y || jj == e3.z);  // its own water: excluded pair
      }
      if (in) {
        const float r2f = (float)r2;
        const float rinv = __builtin_amdgcn_rsqf(r2f);
        if (exc) {
          ec -= (double)(c_ke * L.w * J.w * erff(g.alpha * r2f * rinv) * rinv);
        } else {
          float ex;
          const float erfcv = erfc_fit(g.alpha * r2f * rinv, &ex);
          ec += (double)(c_ke * L.w * J.w * erfcv * rinv);
        }
      }
      soft = in && !awe;                  // an alchemical water keeps its LJ (no lambda dependence)
      if (soft) {
        const float2 jp = s_jp[nj], lp = s_lp[li];
        const double sg = (double)lp.x + 0.5 * (double)jp.x;
        const double s2 = sg * sg;
        s6 = s2 * s2 * s2;
        r6 = r2 * r2 * r2;
        e4 = 4.0 * sqrt((double)lp.y * (double)jp.y);
        soft = e4 != 0.0;                 // (water hydrogens have no LJ)
      }
    }
    sc_push(s_q[wave], nq, soft, s6, r6, e4, lane, SL);
  }
  sc_eval(s_q[wave], 0, nq, SL);
  sc_flush(A, s_sum, s_e0, ec, SL, out);
}

struct CombineArgs {
  double le[kMaxStates], lr[kMaxStates];
  unsigned char kv[kMaxStates];
  double pressure;                     // kcal/(mol A^3): u gains beta P V of the frame's box (NPT)
};

// one block per frame slot of the pass: its box (given edges, or the leg's
// box), its sums and the touched-row flags of its grid cleared, and the
// ligand's bounding sphere: the centre of its bounding box (images nearest its
// first atom) and the largest minimum-image distance from there
__global__ __launch_bounds__(256) void k_ukn_begin(const LegDev* legs, UknArgs A, const double* fbox) {
  const LegDev& g = legs[0];
  const int f = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ BoxW s_b;
  __shared__ float s_box[4][6];
  if (tid == 0) {                                                  // unused slots: the leg's box
    s_b = (fbox && f < A.nf) ? make_box(fbox + 3 * (A.f0 + f), (double)g.alpha) : g.box0;
    g.ubox[f] = s_b;
  }
  for (int t = tid; t < kNU; t += blockDim.x) g.uacc[(size_t)f * kNU + t] = 0;
  if (f < g.npair) {
    int* flag = ukn_flags(g, f);
    for (int t = tid; t < g.K[2] * (ukn_chunks(g.K[1]) + 1); t += blockDim.x) flag[t] = 0;
  }
  if (f >= A.nf || g.nlig == 0) return;                            // uniform
  const size_t fo = (size_t)(A.f0 + f) * A.stride;
  const int a0 = g.lig_idx[0], al = g.lig_idx[min(tid, g.nlig - 1)];       // at most kMaxLigand = 256
  const float ox = A.fx[fo + a0], oy = A.fy[fo + a0], oz = A.fz[fo + a0];
  const float x = A.fx[fo + al], y = A.fy[fo + al], z = A.fz[fo + al];
  __syncthreads();
  float3 d = min_img(s_b, x - ox, y - oy, z - oz);
  float lo[3] = {d.x, d.y, d.z}, hi[3] = {d.x, d.y, d.z};
  for (int c = 0; c < 3; ++c)
    for (int k = 32; k > 0; k >>= 1) {
      lo[c] = fminf(lo[c], __shfl_xor(lo[c], k, 64));
      hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], k, 64));
    }
  if (lane == 0)
    for (int c = 0; c < 3; ++c) { s_box[wave][c] = lo[c]; s_box[wave][3 + c] = hi[c]; }
  __syncthreads();
  float cen[3] = {ox, oy, oz};
  for (int c = 0; c < 3; ++c) {
    const float l = fminf(fminf(s_box[0][c], s_box[1][c]), fminf(s_box[2][c], s_box[3][c]));
    const float h = fmaxf(fmaxf(s_box[0][3 + c], s_box[1][3 + c]), fmaxf(s_box[2][3 + c], s_box[3][3 + c]));
    cen[c] += 0.5f * (l + h);
  }
  d = min_img(s_b, x - cen[0], y - cen[1], z - cen[2]);
  float r2 = d.x * d.x + d.y * d.y + d.z * d.z;
  for (int k = 32; k > 0; k >>= 1) r2 = fmaxf(r2, __shfl_xor(r2, k, 64));
  __syncthreads();
  if (lane == 0) s_box[wave][0] = r2;
  __syncthreads();
  if (tid == 0)
    g.usph[f] = make_float4(cen[0], cen[1], cen[2],
                            sqrtf(fmaxf(fmaxf(s_box[0][0], s_box[1][0]), fmaxf(s_box[2][0], s_box[3][0]))));
}

// one block per frame: the pair partials of every block of k_ukn_pairs summed
// per slot (one wave per slot, lanes over blocks, fixed tree), then u at every
// state
__global__ __launch_bounds__(1024) void k_ukn_combine(const LegDev* legs, UknArgs A, CombineArgs C,
                                                     const double* cst, int K, double beta, double* u,
                                                     long long u_stride) {
  const LegDev& g = legs[0];
  const int f = blockIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nb = g.nlig + g.naw > 0 ? ukn_pair_blocks(g.n) : 0;  // no alchemical charges: no pair partials
  __shared__ double s_p[1 + kMaxLamV];
  const double* pp = g.upart + (size_t)f * nb * (1 + kMaxLamV);
  const double* lp = g.lpart + (size_t)f * (1 + kMaxLamV);
  for (int slot = wv; slot < 1 + A.KV; slot += 16) {
    double v = 0.0;
    for (int t = lane; t < nb; t += 64) v += pp[(size_t)t * (1 + kMaxLamV) + slot];
    v = wave_sum(v);
    if (lane == 0) s_p[slot] = v;
  }
  __syncthreads();
  const long long* acc = g.uacc + (size_t)f * kNU;
  const double s = 1.0 / kEnergyScale;
  const bool has_l = g.nlig + g.naw > 0;
  const double bg = g.ubox[f].bg_pref;
  const double pv = C.pressure * g.ubox[f].vol;
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    const int kv = C.kv[k];
    const double ele = (double)acc[0] * s - bg * cst[0] + s_p[0] + cst[3];
    const double ell = (double)acc[1] * s + cst[2] - bg * cst[1] + (has_l ? lp[0] : 0.0);
    const double ub = (double)acc[2] * s;
    const double ut = (double)acc[3] * s;
    const double esc = s_p[1 + kv] + (has_l ? lp[1 + kv] : 0.0);
    const double le = C.le[k], lr = C.lr[k], lv = (double)A.lamv[kv];
    u[(long long)k * u_stride + A.f0 + f] = beta * (le * ele + le * le * ell + esc + lr * ub + lv * ut + pv);
  }
}

}  // namespace

int launch_ukn(hipStream_t s, hipStream_t side, hipEvent_t ev_fork, hipEvent_t ev_join, const LegDev* d, const LegHost& h, double sc_alpha, const double* lambdas,
               int K, const float* fx, const float* fy, const float* fz, long long frame_stride,
               long long n_frames, const double* frame_box, double pressure, double beta, double* u,
               long long u_stride, double* cst) {
  if (K < 1 || K > kMaxStates) return FELIS_E_UNSUPPORTED;
  const int nB = h.nlig + h.naw;
  if (nB > kMaxLigand) return FELIS_E_UNSUPPORTED;
  UknArgs A;
  CombineArgs C;
  A.fx = fx; A.fy = fy; A.fz = fz;
  A.stride = frame_stride;
  A.KV = 0;
  for (int k = 0; k < K; ++k) {
    const float lv = (float)lambdas[3 * k + 1];
    int found = -1;
    for (int t = 0; t < A.KV; ++t)
      if (A.lamv[t] == lv) found = t;
    if (found < 0) {
      if (A.KV == kMaxLamV) return FELIS_E_UNSUPPORTED;
      found = A.KV;
      A.lamv[A.KV] = lv;
      A.asc[A.KV] = (float)(sc_alpha * (1.0 - lambdas[3 * k + 1]));
      ++A.KV;
    }
    C.kv[k] = (unsigned char)found;
    C.le[k] = lambdas[3 * k];
    C.lr[k] = lambdas[3 * k + 2];
  }
  C.pressure = pressure;
  // two frames per complex grid (2 npair frames per pass) when they share the
  // leg's box; frames with boxes of their own take a grid each
  A.upk = frame_box ? 1 : 0;
  const int F = frame_box ? h.npair : 2 * h.npair;
  for (long long f0 = 0; f0 < n_frames; f0 += F) {
    const int nf = (int)std::min<long long>(F, n_frames - f0);
    const int nb = (h.n + 255) / 256;
    A.f0 = f0;
    A.nf = nf;
    hipLaunchKernelGGL(k_ukn_begin, dim3((unsigned)(2 * h.npair)), dim3(256), 0, s, d, A, frame_box);
    // the pair sums (arithmetic) run on the side stream beside the transform
    // (memory); (no alchemical charges: the constants' block alone)
    const long long np = nB ? (long long)nf * (ukn_pair_blocks(h.n) + 1) : 0;
    (void)hipEventRecord(ev_fork, s);
    (void)hipStreamWaitEvent(side, ev_fork, 0);
    hipLaunchKernelGGL(k_ukn_pairs, dim3((unsigned)(1 + np)), dim3(256), 0, side, d, A, cst);
    (void)hipEventRecord(ev_join, side);
    if (nB) {
      hipLaunchKernelGGL(k_ukn_spread, dim3((unsigned)(((long long)nf * nB + 15) / 16)), dim3(256), 0, s, d, A);
      launch_pme_fft(s, d, &h, 1, frame_box ? 2 : 1);
      hipLaunchKernelGGL(k_ukn_gather, dim3((unsigned)(nf * nb)), dim3(256), 0, s, d, A);
    }
    (void)hipStreamWaitEvent(s, ev_join, 0);
    hipLaunchKernelGGL(k_ukn_combine, dim3((unsigned)nf), dim3(1024), 0, s, d, A, C, (const double*)cst, K, beta,
                       u, u_stride);
  }
  return FELIS_OK;
}

}  // namespace felis
