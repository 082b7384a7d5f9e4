// Real-space alchemical pair kernel, Ewald corrections, bonds and the Boresch
// restraint.
//
// Pair terms follow section "Double annihilation protocol": ligand charges
// scaled by lambda_elec; Beutler softcore U = lam 4 eps (s6^2/s^2 - s6/s),
// s = alpha (1 - lam) s6 + r^6 (p = 1), lam = lambda_vdw for any pair touching
// the ligand and 1 otherwise; Lorentz-Berthelot mixing; everything cut at r_c
// (appendix B).  Real-space Coulomb is the Ewald direct term erfc(a r)/r.
//
// Pair kernel layout (gfx950, wave64): one wave per 8-atom i-cluster; a
// half-cluster's i-atoms are wave-uniform (scalar registers).  The cluster's two
// half-lists (partners of atoms 0-3, then of atoms 4-7) are swept in turn:
// each lane takes one listed j-atom per step and interacts it with the half's
// 4 i-atoms, so a j entry is loaded, decoded and imaged once for 4 pairs, and
// the next steps' entries and partner data are already in flight.  Each
// cluster lists all its partners (both directions), so every atom's pair force
// is summed by one wave in a fixed order and written once: no atomics and no
// cross-wave ordering.  FP32 arithmetic; energies summed in FP64 per lane and
// combined in int64 fixed point.
#include <type_traits>

#include "felis_internal.h"

#include "erfc_coeffs.h"
#include "erfc_coeffs_fp64.h"
#include "restraint.h"

namespace felis {
namespace {

// items: window x slot -- current coordinates (wrapped into the box) and
// scaled charges in sorted order, and each slot's PME stencil (grid base and
// B-spline offsets).  REBUILD (inside a list build): for windows being
// rebuilt also the sorted per-slot LJ parameters and each 8-slot cluster's
// bounding box of wrapped positions (8 consecutive lanes hold one cluster:
// N_pad is a multiple of 8).
template <bool REBUILD>
__global__ __launch_bounds__(256) void k_pack(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const long long i = (long long)(blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  const bool valid = i < (long long)g.W * g.npad;
  const long long ic = valid ? i : (long long)g.W * g.npad - 1;
  const int w = (int)(ic / g.npad);
  const int a = valid ? g.perm[ic] : -1;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (a >= 0) {
    // coordinates wrapped into the window's box [0, L): the pair kernel
    // needs no periodic shift for a cluster lying r_c inside every face
    const size_t o = (size_t)w * g.n + a;
    const float q = window_charge(g, a, g.lam[4 * w]);
    const BoxW& Bp = g.box[w];
    v = make_float4(wrapf(g.x[o], Bp.Lf[0], Bp.invLf[0]), wrapf(g.y[o], Bp.Lf[1], Bp.invLf[1]),
                    wrapf(g.z[o], Bp.Lf[2], Bp.invLf[2]), q * (float)sqrt(kKE));
  }
  if (valid) {
    g.xyzq[i] = v;
    // PME stencil of the slot (read by spreading and the gather)
    float f[3];
    const BoxW& B = g.box[w];
    const int bx = grid_base(v.x, B.invL[0], g.K[0], &f[0]);
    const int by = grid_base(v.y, B.invL[1], g.K[1], &f[1]);
    const int bz = grid_base(v.z, B.invL[2], g.K[2], &f[2]);
    g.gsten[i] = make_float4(f[0], f[1], f[2], pack_bases(bx, by, bz));
  }
  if (REBUILD) {
    const bool fl = valid && g.flag[w] != 0;
    if (fl) {
      // the ligand flag rides in the sign bit of 2 sqrt(eps) (-0 for a
      // ligand atom without LJ), so a partner's parameters are 8 bytes
      float2 p = make_float2(0.f, 0.f);
      if (a >= 0) {
        const float e2 = 2.0f * sqrtf(g.eps[a]);
        p = make_float2(0.5f * g.sig[a], g.lig[a] ? -e2 : e2);
      }
      g.prm[i] = p;
    }
    float lo[3] = {3.0e38f, 3.0e38f, 3.0e38f}, hi[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
    if (a >= 0) {
      const BoxW& B = g.box[w];
      const float r[3] = {wrapf(v.x, B.Lf[0], B.invLf[0]), wrapf(v.y, B.Lf[1], B.invLf[1]),
                          wrapf(v.z, B.Lf[2], B.invLf[2])};
      for (int d = 0; d < 3; ++d) { lo[d] = r[d]; hi[d] = r[d]; }
    }
    for (int k = 1; k < kClus; k <<= 1)
      for (int d = 0; d < 3; ++d) {
        lo[d] = fminf(lo[d], __shfl_xor(lo[d], k, 64));
        hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], k, 64));
      }
    if (fl && (i & (kClus - 1)) == 0) {
      g.bblo[i / kClus] = make_float4(lo[0], lo[1], lo[2], 0.f);
      g.bbhi[i / kClus] = make_float4(hi[0], hi[1], hi[2], 0.f);
    }
  }
}

__device__ __forceinline__ float3 min_img(const BoxW& B, float dx, float dy, float dz) {
  dx = fmaf(-B.Lf[0], rintf(dx * B.invLf[0]), dx);
  dy = fmaf(-B.Lf[1], rintf(dy * B.invLf[1]), dy);
  dz = fmaf(-B.Lf[2], rintf(dz * B.invLf[2]), dz);
  return make_float3(dx, dy, dz);
}

// The 4 i-atoms of a half-cluster, wave-uniform (held in scalar registers).
struct IHalf {
  float x[4], y[4], z[4], q[4], sig[4], eps[4];
};

__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Sums of four values over the wave, value k's in the 16 lanes of row k.  Half
// the wave's exchange and adds go away with each of the first two steps, which
// fold two values into one register; the steps pair lanes 32, 16, 8, 4, 2 and 1
// apart, in the order (and so with the rounding) of wave_sum.
__device__ __forceinline__ float wave_sum4(float v0, float v1, float v2, float v3) {
  auto swap32 = [](float& a, float& b) {         // a's upper half with b's lower half
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  auto swap16 = [](float& a, float& b) {         // a's odd rows with b's even rows
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  swap32(v0, v2);
  swap32(v1, v3);
  float a = v0 + v2, b = v1 + v3;                // rows 0, 1: values 0 (1); rows 2, 3: values 2 (3)
  swap16(a, b);
  a += b;                                        // row k: value k
  auto dpp = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  a += dpp(a, std::integral_constant<int, 0x128>{});   // 8 lanes on within the row
  a += dpp(a, std::integral_constant<int, 0x124>{});   // 4 (the row now repeats after 8)
  a += quad_xor2(a);
  a += quad_xor1(a);
  return a;
}

// lane `src`'s value (src wave-uniform), in a scalar register
__device__ __forceinline__ float lane_of(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

// a window's box edges held in scalar registers for a whole kernel
struct BoxF {
  float L[3], iL[3];
};

__device__ __forceinline__ BoxF box_f(const BoxW& B) {
  BoxF b;
  for (int d = 0; d < 3; ++d) { b.L[d] = uniform(B.Lf[d]); b.iL[d] = uniform(B.invLf[d]); }
  return b;
}

// The periodic image of a partner against a cluster, axis by axis and held in
// scalar registers: partners' coordinates are wrapped into [0, L), so the one
// nearest the cluster's first atom (at x0) is x - L for x > x0 + L/2 when x0 <
// L/2, and x + L for x < x0 - L/2 otherwise; none is needed on an axis where the
// cluster lies r_c inside both faces (every partner within r_c then has its
// wrapped coordinate as its nearest image, and any other image only lengthens
// the separation).
struct Image {
  float t[3];                               // x0 +- L/2
};

// A cluster's yes-or-no facts in one scalar register (a condition held across
// the sweep would take a register pair each)
constexpr int kFlagAxis = 0;                // + d: axis d needs the image
constexpr int kFlagLow = 3;                 // + d: x0 < L/2
constexpr int kFlagLig = 8;                 // + k: the half's atom k belongs to the ligand, in a softcore window
constexpr int kFlagLJ = 16;                 // + k: atom k has LJ
constexpr int kFlagSoft = 24;               // lambda_vdw < 1

__device__ __forceinline__ float image(float x, float t, float L, bool low) {    // low: uniform
  if (low) return x > t ? x - L : x;
  return x < t ? x + L : x;
}

// Sweep a cluster's j-list: lane = listed j, unrolled loop over the cluster's
// i-atoms.  IMG 1: the periodic image of j is chosen once against the
// cluster's first atom (exact when r_c + cluster extent < L/2 on every axis);
// IMG 0: every (i, j) takes its own minimum image.
template <int ENERGY, int IMG>
__device__ __forceinline__ void sweep(const LegDev& g, const BoxF B, const Image& P, const IHalf& I, gptr<unsigned> ent, int cnt,
                                      gptr<f32x4> xq, gptr<f32x2> pr, int lane,
                                      float lam_v, float a_sc, int flags, float (&fx)[4],
                                      float (&fy)[4], float (&fz)[4], double& ec, double& el) {
  const float Lx = B.L[0], Ly = B.L[1], Lz = B.L[2];
  const float iLx = B.iL[0], iLy = B.iL[1], iLz = B.iL[2];
  const float rc2 = g.rc2, alpha = g.alpha;
  const float c2a = 2.0f * alpha * 0.56418958354775628f;   // 2 alpha / sqrt(pi)
  const float pa = FELIS_ERFC_P * alpha;                    // fit variable t = 1 / (1 + P alpha r)
  const float kx2 = -alpha * alpha * 1.4426950408889634f;   // exp(-alpha^2 r^2) = 2^(kx2 r^2)
  // software pipeline: the entries two steps ahead and the partner data one
  // step ahead are in flight while a step computes
  unsigned e_next = lane < cnt ? ent[lane] : kListPartial;          // slot 0 with an empty mask
  unsigned e_next2 = 64 + lane < cnt ? ent[64 + lane] : kListPartial;
  f32x4 xj_next = xq[(int)(e_next >> 8)];
  f32x2 pj_next = pr[(int)(e_next >> 8)];
  for (int it = 0; it < cnt; it += 64) {
    const unsigned e = e_next;
    const f32x4 xj = xj_next;
    const f32x2 pj = pj_next;
    e_next = e_next2;
    const int nidx = it + 128 + lane;
    e_next2 = nidx < cnt ? ent[nidx] : kListPartial;
    xj_next = xq[(int)(e_next >> 8)];
    pj_next = pr[(int)(e_next >> 8)];
    const bool ligj = __float_as_uint(pj.y) >> 31;
    float jx = xj.x, jy = xj.y, jz = xj.z;
    int fl = flags;
    asm volatile("" : "+s"(fl));                          // tested afresh each step
    if (IMG == 1) {                                       // uniform branches
      if (fl & (1 << kFlagAxis)) { asm volatile(""); jx = image(jx, P.t[0], Lx, fl & (1 << kFlagLow)); }
      if (fl & (2 << kFlagAxis)) { asm volatile(""); jy = image(jy, P.t[1], Ly, fl & (2 << kFlagLow)); }
      if (fl & (4 << kFlagAxis)) { asm volatile(""); jz = image(jz, P.t[2], Lz, fl & (4 << kFlagLow)); }
    }
    // wave-uniform: does any lane hold an entry whose mask lacks a pair within
    // reach (an excluded pair, the atom itself) or none at all (past the end)?
    // Otherwise the masks say nothing that r < r_c does not: a pair missing
    // from a mask for its distance was beyond r_list when the list was made.
    // (An energy sum must not meet the padding atoms of the last cluster.)
    unsigned long long listed[4] = {~0ull, ~0ull, ~0ull, ~0ull};      // lanes that list the pair, per i-atom
    if (ENERGY || __ballot(e & kListPartial) != 0ull) {
      asm volatile("");                                   // a branch, not a select in every step
#pragma unroll
      for (int k = 0; k < 4; ++k) listed[k] = __ballot((e >> k) & 1u);
    }
    // wave-uniform: does any listed j of this step belong to the ligand?
    const bool jlig = (fl & (1 << kFlagSoft)) && __ballot(ligj) != 0ull;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float dx = jx - I.x[k], dy = jy - I.y[k], dz = jz - I.z[k];
      if (IMG == 0) {
        dx = fmaf(-Lx, rintf(dx * iLx), dx);
        dy = fmaf(-Ly, rintf(dy * iLy), dy);
        dz = fmaf(-Lz, rintf(dz * iLz), dz);
      }
      const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
      const unsigned long long in_lanes = __ballot(r2 < rc2) & listed[k];
      // wave-uniform: no lane's partner lies within r_c of this i-atom (the
      // list's entries are consecutive in the Hilbert order, so a wave's
      // partners are near one another and often all beyond r_c of one side
      // of the half-cluster); a skipped lane adds nothing, exactly as the
      // select below would.
      if (in_lanes == 0ull) continue;
      const bool in = __builtin_amdgcn_inverse_ballot_w64(in_lanes);
      // lanes outside (in == false) may compute inf or NaN below: every
      // result they feed is dropped by the selects on `in`
      const float r2s = r2;
      const float rinv = __builtin_amdgcn_rsqf(r2s);
      const float rinv2 = rinv * rinv;
      const float r = r2s * rinv;
      // erfc(alpha r) = t P(t) exp(-alpha^2 r^2), t = 1 / (1 + P alpha r): the
      // degree-6 fit of erfc_coeffs.h with alpha folded into its constants
      const float t = __builtin_amdgcn_rcpf(fmaf(pa, r, 1.0f));
      float pt = felis_erfc_c[0];
#pragma unroll
      for (int c = 1; c < FELIS_ERFC_NC; ++c) pt = fmaf(pt, t, felis_erfc_c[c]);
      pt *= t;
      const float ex = __builtin_amdgcn_exp2f(kx2 * r2s);
      const float qq = I.q[k] * xj.w;
      const float fc = qq * (ex * fmaf(pt, rinv, c2a)) * rinv2;
      float flj = 0.0f, elj = 0.0f;
      const bool ligi = fl & (1 << (kFlagLig + k));
      if (!(fl & (1 << (kFlagLJ + k)))) {
        // wave-uniform: an i-atom without LJ (a water hydrogen) contributes
        // exactly zero LJ force and energy with every partner
      } else if (const float sig = I.sig[k] + pj.x, eps4 = I.eps[k] * fabsf(pj.y);
                 (jlig || ligi) && __ballot(in && (ligi || ligj)) != 0ull) {
        const bool ligp = ligi || ligj;
        const float lam = ligp ? lam_v : 1.0f;
        const float a = ligp ? a_sc : 0.0f;
        const float s2 = sig * sig;
        const float s6 = s2 * s2 * s2;
        const float r4 = r2s * r2s;
        const float den = fmaf(a, s6, r4 * r2s);
        const float inv = __builtin_amdgcn_rcpf(den);
        const float u = s6 * inv;
        const float le = lam * eps4;
        flj = 6.0f * le * fmaf(2.0f, u, -1.0f) * u * inv * r4;
        if (ENERGY) elj = le * fmaf(u, u, -u);
      } else {
        const float s2 = sig * sig * rinv2;
        const float s6 = s2 * s2 * s2;
        flj = eps4 * fmaf(12.0f, s6, -6.0f) * s6 * rinv2;
        if (ENERGY) elj = eps4 * fmaf(s6, s6, -s6);
      }
      const float fs = in ? (fc + flj) : 0.0f;
      fx[k] = fmaf(-fs, dx, fx[k]);
      fy[k] = fmaf(-fs, dy, fy[k]);
      fz[k] = fmaf(-fs, dz, fz[k]);
      if (ENERGY && in) {
        ec += (double)(qq * (pt * ex) * rinv);
        el += (double)elj;
      }
    }
  }
}

// An excluded pair's reciprocal-space removal -KE q_a q_b erf(alpha r)/r in
// FP64 (its r -> 0 limit -KE q_a q_b 2 alpha / sqrt(pi) below 1e-6 A)
__device__ __attribute__((noinline)) double excl_energy_fp64(const LegDev& g, const BoxW& B, size_t oa, size_t ob,
                                                             double qa, double qb) {
#pragma clang fp contract(off)
  double dx = (double)g.x[ob] - (double)g.x[oa], dy = (double)g.y[ob] - (double)g.y[oa];
  double dz = (double)g.z[ob] - (double)g.z[oa];
  dx = dx - B.L[0] * rint(dx * B.invL[0]);
  dy = dy - B.L[1] * rint(dy * B.invL[1]);
  dz = dz - B.L[2] * rint(dz * B.invL[2]);
  const double r = sqrt((dx * dx + dy * dy) + dz * dz);
  const double qq = kKE * qa * qb;
  if (r < 1e-6) return -qq * 2.0 * g.alphad * 0.56418958354775628;
  return -qq * erf(g.alphad * r) / r;
}

// Vector issue bounds it: 1.2 wave instructions per SIMD and 4 cycles (the most
// seen here), some 38 a pair of a lane.  Hence masks only in the steps that need
// them, the image only on the axes that need it, conditions as lane masks and
// bits of one scalar register, and eight waves a SIMD (61 registers: one half's
// i-atoms at a time).  20 windows of 40,000 atoms: 684 us with masks and images
// in every step at five waves, 621 us.
template <int ENERGY>
__global__ __launch_bounds__(256, ENERGY ? 5 : 8) void k_pairs(const LegDev* legs, BlockMap map, int step) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const long long item = (long long)(blockIdx.x - map.start[leg]) * 4 + wave;
  if (item >= (long long)g.W * g.nclus) return;
  const int w = (int)(item / g.nclus);
  const int c = (int)(item - (long long)w * g.nclus);
  const gptr<f32x4> xq = as_global4(g.xyzq + (size_t)w * g.npad);
  const gptr<f32x2> pr = as_global2(g.prm + (size_t)w * g.npad);
  const BoxF B = box_f(g.box[w]);
  const float lam_v = g.lam[4 * w + 1];
  const float a_sc = g.lam[4 * w + 3];
  const bool soft_window = lam_v < 1.0f;

  // i-atoms, one in each of the first 8 lanes (repeated over the wave): images
  // nearest the cluster's first atom (always a real atom: padding only follows
  // the last atom), and the cluster's extent
  const f32x4 ia = xq[c * kClus + (lane & 7)];
  const f32x2 ip = pr[c * kClus + (lane & 7)];
  const float r0[3] = {uniform(ia.x), uniform(ia.y), uniform(ia.z)};
  float iv[3] = {ia.x, ia.y, ia.z}, ext[3];
  for (int d = 0; d < 3; ++d) {
    iv[d] = fmaf(-B.L[d], rintf((iv[d] - r0[d]) * B.iL[d]), iv[d]);
    ext[d] = c * kClus + (lane & 7) < g.n ? fabsf(iv[d] - r0[d]) : 0.0f;
    for (int k = 1; k < kClus; k <<= 1) ext[d] = fmaxf(ext[d], __shfl_xor(ext[d], k, 64));
    ext[d] = uniform(ext[d]);
  }
  // kept in LDS: in registers they would cost the sweep a wave of occupancy
  __shared__ float s_i[4][6][kClus];
  if (lane < kClus) {
    s_i[wave][0][lane] = iv[0]; s_i[wave][1][lane] = iv[1]; s_i[wave][2][lane] = iv[2];
    s_i[wave][3][lane] = ia.w; s_i[wave][4][lane] = ip.x; s_i[wave][5][lane] = fabsf(ip.y);
  }
  const unsigned ilig = soft_window ? (unsigned)__ballot(__float_as_uint(ip.y) >> 31) & 0xFFu : 0u;
  const unsigned ilj = (unsigned)__ballot(ip.y != 0.0f) & 0xFFu;
  int flags = soft_window ? 1 << kFlagSoft : 0;
  const float rc = sqrtf(g.rc2) + 0.01f;
  const bool shift = rc + ext[0] < 0.5f * B.L[0] && rc + ext[1] < 0.5f * B.L[1] && rc + ext[2] < 0.5f * B.L[2];
  Image P;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float x0 = r0[d];
    const bool inside = x0 - ext[d] - rc >= 0.0f && x0 + ext[d] + rc < B.L[d];
    const bool low = x0 < 0.5f * B.L[d];
    if (!inside) flags |= 1 << (kFlagAxis + d);
    if (low) flags |= 1 << (kFlagLow + d);
    P.t[d] = uniform(low ? x0 + 0.5f * B.L[d] : x0 - 0.5f * B.L[d]);
  }
  flags = __builtin_amdgcn_readfirstlane(flags);
  // the two half-cluster lists (partners of atoms 0-3, then of atoms 4-7);
  // each half's forces are reduced over the wave before the next half
  const gptr<unsigned> ent = as_global(g.lent + (size_t)item * 2 * g.cap);
  double ec = 0.0, el = 0.0;
  __shared__ float s_f[4][kClus][3];                  // per wave: the 8 atoms' pair forces
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    float fx[4] = {0.f, 0.f, 0.f, 0.f}, fy[4] = {0.f, 0.f, 0.f, 0.f}, fz[4] = {0.f, 0.f, 0.f, 0.f};
    const gptr<unsigned> eh = ent + half * g.cap;
    const int cnt = __builtin_amdgcn_readfirstlane(g.lcount[2 * item + half]);
    IHalf I;
    {
      wave_lds_fence();
      float v[6];
#pragma unroll
      for (int t = 0; t < 6; ++t) v[t] = s_i[wave][t][4 * half + (lane & 3)];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        I.x[k] = lane_of(v[0], k); I.y[k] = lane_of(v[1], k); I.z[k] = lane_of(v[2], k);
        I.q[k] = lane_of(v[3], k);
        I.sig[k] = lane_of(v[4], k);
        I.eps[k] = lane_of(v[5], k);
      }
    }
    const int fl = __builtin_amdgcn_readfirstlane(flags | (int)(ilig >> (4 * half) & 0xFu) << kFlagLig |
                                                  (int)(ilj >> (4 * half) & 0xFu) << kFlagLJ);
    if (shift) sweep<ENERGY, 1>(g, B, P, I, eh, cnt, xq, pr, lane, lam_v, a_sc, fl, fx, fy, fz, ec, el);
    else sweep<ENERGY, 0>(g, B, P, I, eh, cnt, xq, pr, lane, lam_v, a_sc, fl, fx, fy, fz, ec, el);
    // atom k's sums end up in the 16 lanes of row k
    const float sx = wave_sum4(fx[0], fx[1], fx[2], fx[3]);
    const float sy = wave_sum4(fy[0], fy[1], fy[2], fy[3]);
    const float sz = wave_sum4(fz[0], fz[1], fz[2], fz[3]);
    if ((lane & 15) == 0) {
      const int k = 4 * half + (lane >> 4);
      s_f[wave][k][0] = sx;
      s_f[wave][k][1] = sy;
      s_f[wave][k][2] = sz;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();

  // Excluded pairs: remove their reciprocal-space (erf) interaction, each
  // pair from both of its sides; lane = ii + 8 k takes the k-th exclusion of
  // i-atom ii (at most kMaxExcl = 8 per atom).
  const int ai = g.perm[(size_t)w * g.npad + c * kClus + (lane & 7)];
  float cx = 0.f, cy = 0.f, cz = 0.f;
  double ex = 0.0;
  if (ai >= 0) {
    const int e0 = g.excl_ptr[ai], ne = min(g.excl_ptr[ai + 1] - e0, kMaxExcl);
    const int k = lane >> 3;
    if (k < ne) {
      const int b = g.excl_idx[e0 + k];
      const float le = g.lam[4 * w];
      const float qa = window_charge(g, ai, le), qb = window_charge(g, b, le);
      const size_t oa = (size_t)w * g.n + ai, ob = (size_t)w * g.n + b;
      float3 d = make_float3(g.x[ob] - g.x[oa], g.y[ob] - g.y[oa], g.z[ob] - g.z[oa]);
      d.x = fmaf(-B.L[0], rintf(d.x * B.iL[0]), d.x);
      d.y = fmaf(-B.L[1], rintf(d.y * B.iL[1]), d.y);
      d.z = fmaf(-B.L[2], rintf(d.z * B.iL[2]), d.z);
      const float r2 = d.x * d.x + d.y * d.y + d.z * d.z;
      const float qq = (float)kKE * qa * qb;
      const float c2a = 2.0f * g.alpha * 0.56418958354775628f;
      float fs, en;
      if (r2 > 1e-8f) {
        const float r = sqrtf(r2), rinv = 1.0f / r;
        const float erfv = erff(g.alpha * r);
        en = -qq * erfv * rinv;
        fs = qq * (c2a * __expf(-g.alpha * g.alpha * r2) - erfv * rinv) * rinv * rinv;
      } else {
        en = -qq * c2a;
        fs = 0.f;
      }
      cx = -fs * d.x; cy = -fs * d.y; cz = -fs * d.z;      // F_i = fs (r_i - r_j)
      ex = 0.5 * (double)en;
    }
  }
  for (int o = 8; o < 64; o <<= 1) {
    cx += __shfl_xor(cx, o, 64);
    cy += __shfl_xor(cy, o, 64);
    cz += __shfl_xor(cz, o, 64);
  }
  float ox = cx, oy = cy, oz = cz;
  if (lane < kClus) { ox += s_f[wave][lane][0]; oy += s_f[wave][lane][1]; oz += s_f[wave][lane][2]; }
  if (lane < kClus) {
    const int a = ai;
    if (a >= 0) {
      const size_t o = (size_t)w * g.n + a;
      if (step && g.plain) {
        // the plain form: FP64 atomics into the leg's FP64 sums
        const size_t wn = (size_t)g.W * g.n;
        unsafeAtomicAdd(&g.fd[o], (double)ox);
        unsafeAtomicAdd(&g.fd[wn + o], (double)oy);
        unsafeAtomicAdd(&g.fd[2 * wn + o], (double)oz);
      } else {
        const int where = (w << 20) | a;
        g.fx[o] = to_fixed((double)ox, kForceScale, g.err, kSitePairs, where, g.leg_index);
        g.fy[o] = to_fixed((double)oy, kForceScale, g.err, kSitePairs, where, g.leg_index);
        g.fz[o] = to_fixed((double)oz, kForceScale, g.err, kSitePairs, where, g.leg_index);
      }
    }
  }
  if (ENERGY) {
    ec = wave_sum(ec);
    el = wave_sum(el);
    ex = wave_sum(ex);
    if (lane == 0) {
      long long* acc = g.eacc + (size_t)w * FELIS_NE;
      atomicAdd((unsigned long long*)&acc[FELIS_E_COUL_REAL],
                (unsigned long long)to_fixed(0.5 * ec, kEnergyScale, g.err, kSitePairsE, w));
      atomicAdd((unsigned long long*)&acc[FELIS_E_LJ],
                (unsigned long long)to_fixed(0.5 * el, kEnergyScale, g.err, kSitePairsE, w));
      atomicAdd((unsigned long long*)&acc[FELIS_E_EXCL],
                (unsigned long long)to_fixed(ex, kEnergyScale, g.err, kSitePairsE, w));
    }
  }
}

// FP64 energies of the real-space terms (felis_nonbonded with FELIS_ENERGY):
// every pair once, every term in FP64 from the raw (unwrapped) coordinates:
// the minimum-image distance d - L rint(d (1/L)) and d^2 = (dx^2 + dy^2) +
// dz^2 without contraction, the cutoff r < r_c on r = sqrt(d^2), the window's
// charges in FP64, Lorentz-Berthelot parameters from the packed (sigma/2,
// 2 sqrt(eps)) and the softcore form at lambda_vdw for pairs touching the
// ligand.
//
// One wave per cluster, as in the force sweep, but the FP64 arithmetic (some
// 200 instructions a pair) is the whole cost, so no lane may idle in it and
// no pair may be taken twice.  Both clusters of a pair list it: the pair is
// taken from cluster ci's list when ci < cj and ci + cj is odd or ci > cj and
// ci + cj is even (each list then gives half of its entries), within a cluster
// from its lower slot.  The entries kept are queued in LDS; 64 at a time, an
// FP32 distance with 0.01 A of room (the lists' own margin) drops what lies
// beyond the cutoff, and what is left is queued in turn and evaluated 64 pairs
// at a time.
// 20 windows of 7,540 atoms, 32 M pairs: 2.50 ms as a branch of the force sweep
// (both sides of every pair, half of the lanes idle, the library's erfc),
// 0.45 ms from one side with the queue of pairs alone, 0.39 ms with both queues.
constexpr int kEntQueue = 64 + 64;             // entries: less than a wave's worth kept, one step's pushes
constexpr int kPairQueue = 64 + 4 * 64;        // pairs, likewise

// 1/x and 1/sqrt(x) in FP64: the hardware estimates (some 2^-26) refined by two
// Newton steps to about one rounding (x normal and finite)
__device__ __forceinline__ double rcp_fp64(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double rsqrt_fp64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

struct EnergyAtoms {                           // a cluster's atoms (LDS, per wave)
  float x[kClus], y[kClus], z[kClus];          // raw coordinates
  float hs[kClus], e2[kClus];                  // packed LJ parameters
  double q[kClus];                             // the window's charges x KE
};

// a leg's arrays and constants the pair loop reads, held in registers
struct EnergyLeg {
  gptr<float> x, y, z, q, aoff;                  // coordinates of the window; topology
  gptr<uint8_t> lig;
  bool has_off;
  double L[3], iL[3], rc, alpha, sc_alpha, lam_e, lam_v;
};

__device__ __forceinline__ void pair_energy_fp64(const EnergyLeg& g, const EnergyAtoms& A, int ii, int aj, f32x2 pj,
                                                 double& ec, double& el) {
#pragma clang fp contract(off)
  // every load first: one wait covers them all
  const float xj = g.x[aj], yj = g.y[aj], zj = g.z[aj], q1 = g.q[aj];
  const uint8_t lj = g.lig[aj];
  const float off = g.has_off ? g.aoff[aj] : 0.f;
  double dx = (double)A.x[ii] - (double)xj, dy = (double)A.y[ii] - (double)yj;
  double dz = (double)A.z[ii] - (double)zj;
  dx = dx - g.L[0] * rint(dx * g.iL[0]);
  dy = dy - g.L[1] * rint(dy * g.iL[1]);
  dz = dz - g.L[2] * rint(dz * g.iL[2]);
  const double r2 = (dx * dx + dy * dy) + dz * dz;
  const double r = sqrt(r2);
  if (!(r < g.rc)) return;
  const double qj = (double)q1 * (lj ? g.lam_e : 1.0) + (1.0 - g.lam_e) * (double)off;
  // erfc(alpha r) by the fit of erfc_coeffs_fp64.h (fit 3e-16, evaluated in FP64
  // 1.4e-15, and an ulp or two more for the refined reciprocal; alpha r_c <= 3.5):
  // without the range branches of the library's erfc, which a wave of distances
  // from 1 to 10 A takes all of
  const double rinv = rsqrt_fp64(r2);
  const double xa = g.alpha * r;
  const double t = rcp_fp64(fma(FELIS_ERFC64_P, xa, 1.0));
  const double sv = fma(FELIS_ERFC64_A, t, FELIS_ERFC64_B);
  double pt = felis_erfc64_c[0];
#pragma unroll
  for (int k = 1; k < FELIS_ERFC64_NC; ++k) pt = fma(pt, sv, felis_erfc64_c[k]);
  ec += A.q[ii] * qj * (t * pt * exp(-xa * xa)) * rinv;
  const float e2i = A.e2[ii];
  const double eps = 0.25 * (double)fabsf(e2i) * (double)fabsf(pj.y);
  if (eps == 0.0) return;
  const double sig = (double)A.hs[ii] + (double)pj.x;
  const double lam = ((__float_as_uint(e2i) | __float_as_uint(pj.y)) >> 31) ? g.lam_v : 1.0;
  const double s2 = sig * sig, s6 = s2 * s2 * s2;
  const double u = s6 * rcp_fp64(g.sc_alpha * (1.0 - lam) * s6 + r2 * r2 * r2);
  el += lam * 4.0 * eps * (u * u - u);
}

__global__ __launch_bounds__(256) void k_pair_energy(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const long long item = (long long)(blockIdx.x - map.start[leg]) * 4 + wave;
  if (item >= (long long)g.W * g.nclus) return;
  const int w = (int)(item / g.nclus);
  const int c = (int)(item - (long long)w * g.nclus);
  const BoxW& B = g.box[w];
  const BoxF Bf = box_f(B);
  const double lam_e = (double)g.lam[4 * w];
  const size_t base = (size_t)w * g.n;
  const gptr<int> permw = as_global(g.perm + (size_t)w * g.npad);
  EnergyLeg G;
  G.x = as_global(g.x + base); G.y = as_global(g.y + base); G.z = as_global(g.z + base);
  G.q = as_global(g.q); G.lig = as_global(g.lig); G.aoff = as_global(g.aoff);
  G.has_off = g.aoff != nullptr;
  for (int d = 0; d < 3; ++d) { G.L[d] = B.L[d]; G.iL[d] = B.invL[d]; }
  G.rc = g.rcd; G.alpha = g.alphad; G.sc_alpha = g.sc_alphad;
  G.lam_e = lam_e; G.lam_v = (double)g.lam[4 * w + 1];
  const gptr<f32x4> xq = as_global4(g.xyzq + (size_t)w * g.npad);
  const gptr<f32x2> pr = as_global2(g.prm + (size_t)w * g.npad);
  __shared__ EnergyAtoms s_at[4];
  __shared__ unsigned s_ent[4][kEntQueue];       // partner's slot << 4 | 4-bit mask over the half's atoms
  __shared__ uint2 s_pair[4][kPairQueue];        // partner's slot << 3 | atom of the cluster; partner's atom index
  EnergyAtoms& A = s_at[wave];
  unsigned* eq = s_ent[wave];
  uint2* pq = s_pair[wave];
  if (lane < kClus) {
    const int a = permw[c * kClus + lane];
    const f32x2 p = pr[c * kClus + lane];
    A.x[lane] = a >= 0 ? g.x[base + a] : 0.f;
    A.y[lane] = a >= 0 ? g.y[base + a] : 0.f;
    A.z[lane] = a >= 0 ? g.z[base + a] : 0.f;
    A.q[lane] = a >= 0 ? kKE * window_charge_fp64(g, a, lam_e) : 0.0;
    A.hs[lane] = p.x;
    A.e2[lane] = p.y;
  }
  wave_lds_fence();
  const float rpre = (float)g.rcd + 0.01f, rpre2 = rpre * rpre;
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  double ec = 0.0, el = 0.0;
  int ne = 0, np = 0;                            // queued entries and pairs (the same in every lane)
  auto pairs = [&](int first, int count) {
    if (lane < count) {
      const uint2 v = pq[first + lane];
      pair_energy_fp64(G, A, (int)(v.x & 7u), (int)v.y, pr[v.x >> 3], ec, el);
    }
  };
  for (int half = 0; half < 2; ++half) {
    const gptr<unsigned> ent = as_global(g.lent + ((size_t)item * 2 + half) * g.cap);
    const int cnt = g.lcount[2 * item + half];
    float xi[4], yi[4], zi[4], ext[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x4 a = xq[c * kClus + 4 * half + k];
      xi[k] = uniform(a.x); yi[k] = uniform(a.y); zi[k] = uniform(a.z);
      if (k) {                                   // the images nearest the half's first atom
        xi[k] = fmaf(-Bf.L[0], rintf((xi[k] - xi[0]) * Bf.iL[0]), xi[k]);
        yi[k] = fmaf(-Bf.L[1], rintf((yi[k] - yi[0]) * Bf.iL[1]), yi[k]);
        zi[k] = fmaf(-Bf.L[2], rintf((zi[k] - zi[0]) * Bf.iL[2]), zi[k]);
        if (c * kClus + 4 * half + k < g.n) {
          ext[0] = fmaxf(ext[0], fabsf(xi[k] - xi[0]));
          ext[1] = fmaxf(ext[1], fabsf(yi[k] - yi[0]));
          ext[2] = fmaxf(ext[2], fabsf(zi[k] - zi[0]));
        }
      }
    }
    // one periodic image per entry, against the half's first atom, is the
    // nearest for all four when the cutoff and the half's extent fit in L/2
    const bool shift = rpre + 0.01f + ext[0] < 0.5f * Bf.L[0] && rpre + 0.01f + ext[1] < 0.5f * Bf.L[1] &&
                       rpre + 0.01f + ext[2] < 0.5f * Bf.L[2];
    // distances of 64 queued entries
    auto entries = [&](int first, int count) {
      const unsigned e = lane < count ? eq[first + lane] : 0u;       // slot 0 with an empty mask
      const int s = (int)(e >> 4);
      const f32x4 xj = xq[s];
      const unsigned aj = (unsigned)permw[s];
      float jx = xj.x, jy = xj.y, jz = xj.z;
      if (shift) {
        jx = fmaf(-Bf.L[0], rintf((jx - xi[0]) * Bf.iL[0]), jx);
        jy = fmaf(-Bf.L[1], rintf((jy - yi[0]) * Bf.iL[1]), jy);
        jz = fmaf(-Bf.L[2], rintf((jz - zi[0]) * Bf.iL[2]), jz);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float dx = jx - xi[k], dy = jy - yi[k], dz = jz - zi[k];
        if (!shift) {
          dx = fmaf(-Bf.L[0], rintf(dx * Bf.iL[0]), dx);
          dy = fmaf(-Bf.L[1], rintf(dy * Bf.iL[1]), dy);
          dz = fmaf(-Bf.L[2], rintf(dz * Bf.iL[2]), dz);
        }
        const bool in = ((e >> k) & 1u) && fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < rpre2;
        const unsigned long long m = __ballot(in);
        if (in) pq[np + __popcll(m & lt)] = make_uint2((unsigned)s << 3 | (unsigned)(4 * half + k), aj);
        np += __popcll(m);
      }
      wave_lds_fence();
      while (np >= 64) {
        np -= 64;
        pairs(np, 64);
      }
      wave_lds_fence();
    };
    for (int it = 0; it < cnt; it += 64) {
      const unsigned v = it + lane < cnt ? ent[it + lane] : 0u;
      const int s = (int)(v >> 8), cj = s >> 3;
      unsigned m = v & 0xFu;
      if (cj == c) {
        const int below = min(max((s & 7) - 4 * half, 0), 4);          // atoms of the half with a lower slot
        m &= (1u << below) - 1u;
      } else if ((((cj + c) & 1) != 0) != (cj > c)) {
        m = 0u;
      }
      const unsigned long long b = __ballot(m != 0u);
      if (m) eq[ne + __popcll(b & lt)] = (unsigned)s << 4 | m;
      ne += __popcll(b);
      wave_lds_fence();
      if (ne >= 64) {
        ne -= 64;
        entries(ne, 64);
      }
    }
    entries(0, ne);                              // the queue holds one half's entries: empty it
    ne = 0;
  }
  pairs(0, np);
  // excluded pairs, each from its lower atom: lane = ii + 8 k takes the k-th
  // exclusion of atom ii
  double ex = 0.0;
  const int ai = permw[c * kClus + (lane & 7)];
  if (ai >= 0) {
    const int e0 = g.excl_ptr[ai], ne = min(g.excl_ptr[ai + 1] - e0, kMaxExcl);
    const int k = lane >> 3;
    if (k < ne) {
      const int b = g.excl_idx[e0 + k];
      if (b > ai)
        ex = excl_energy_fp64(g, B, base + ai, base + b, window_charge_fp64(g, ai, lam_e),
                              window_charge_fp64(g, b, lam_e));
    }
  }
  ec = wave_sum(ec);
  el = wave_sum(el);
  ex = wave_sum(ex);
  if (lane == 0) {
    long long* acc = g.eacc + (size_t)w * FELIS_NE;
    atomicAdd((unsigned long long*)&acc[FELIS_E_COUL_REAL],
              (unsigned long long)to_fixed(ec, kEnergyScale, g.err, kSitePairsE, w));
    atomicAdd((unsigned long long*)&acc[FELIS_E_LJ],
              (unsigned long long)to_fixed(el, kEnergyScale, g.err, kSitePairsE, w));
    atomicAdd((unsigned long long*)&acc[FELIS_E_EXCL],
              (unsigned long long)to_fixed(ex, kEnergyScale, g.err, kSitePairsE, w));
  }
}

__device__ __forceinline__ void add_force(const LegDev& g, size_t o, float fx, float fy, float fz, int site) {
  const int where = (int)(((o / g.n) << 20) | (o % g.n));     // window << 20 | atom
  atomicAdd((unsigned long long*)&g.fx[o], (unsigned long long)to_fixed((double)fx, kForceScale, g.err, site, where, g.leg_index));
  atomicAdd((unsigned long long*)&g.fy[o], (unsigned long long)to_fixed((double)fy, kForceScale, g.err, site, where, g.leg_index));
  atomicAdd((unsigned long long*)&g.fz[o], (unsigned long long)to_fixed((double)fz, kForceScale, g.err, site, where, g.leg_index));
}

__device__ __forceinline__ void add_energy(const LegDev& g, int w, int comp, double e, int lane) {
  e = wave_sum(e);
  if (lane == 0)
    atomicAdd((unsigned long long*)&g.eacc[(size_t)w * FELIS_NE + comp],
              (unsigned long long)to_fixed(e, kEnergyScale, g.err, kSiteEnergy, comp));
}


// one block per window: Ewald self term and neutralising background
__global__ __launch_bounds__(256) void k_self(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int w = blockIdx.x - map.start[leg];
  const double le = (double)g.lam[4 * w];
  double s1 = 0.0, s2 = 0.0;
  for (int a = threadIdx.x; a < g.n; a += blockDim.x) {
    const double q = window_charge_fp64(g, a, le);
    s1 += q; s2 += q * q;
  }
  __shared__ double r1[256], r2[256];
  r1[threadIdx.x] = s1; r2[threadIdx.x] = s2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) { r1[threadIdx.x] += r1[threadIdx.x + s]; r2[threadIdx.x] += r2[threadIdx.x + s]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double e = -(double)g.self_pref * r2[0] - g.box[w].bg_pref * r1[0] * r1[0];
    atomicAdd((unsigned long long*)&g.eacc[(size_t)w * FELIS_NE + FELIS_E_SELF],
              (unsigned long long)to_fixed(e, kEnergyScale, g.err));
  }
}

__device__ __forceinline__ float3 vec(const LegDev& g, const BoxW& B, size_t ofrom, size_t oto) {
  return min_img(B, g.x[oto] - g.x[ofrom], g.y[oto] - g.y[ofrom], g.z[oto] - g.z[ofrom]);
}

// Torsion t's energy in FP64 from the raw coordinates (consistent images
// relative to its first atom)
__device__ __attribute__((noinline)) double torsion_energy_at(const LegDev& g, int w, int t) {
  const BoxW& B = g.box[w];
  const size_t base = (size_t)w * g.n, o0 = base + g.tors[4 * t];
  double p[4][3];
  for (int s = 0; s < 4; ++s) {
    const size_t os = base + g.tors[4 * t + s];
    double d[3] = {(double)g.x[os] - (double)g.x[o0], (double)g.y[os] - (double)g.y[o0],
                   (double)g.z[os] - (double)g.z[o0]};
    for (int c = 0; c < 3; ++c) p[s][c] = d[c] - B.L[c] * rint(d[c] * B.invL[c]);
  }
  return torsion_energy_fp64(p, (double)g.tors_k[t], g.tors_n[t], (double)g.tors_phase[t]);
}

// items: window x (bonds + torsions + 1): harmonic bonds, lambda_vdw-scaled
// rotatable torsions (section "Double annihilation protocol"); the last item
// of a window is the lambda_restraint-scaled Boresch restraint (section
// "Restraints").
// A bond's energy (k/2)(r - r0)^2 with r in FP64 from the raw coordinates
__device__ __attribute__((noinline)) double bond_energy_fp64(const LegDev& g, const BoxW& B, size_t oa, size_t ob,
                                                             int k) {
  double d[3] = {(double)g.x[oa] - (double)g.x[ob], (double)g.y[oa] - (double)g.y[ob],
                 (double)g.z[oa] - (double)g.z[ob]};
  for (int t = 0; t < 3; ++t) d[t] -= B.L[t] * rint(d[t] * B.invL[t]);
  const double dr = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) - (double)g.bond_r0[k];
  return 0.5 * (double)g.bond_k[k] * dr * dr;
}

// The unscaled Boresch energy in FP64 (anchor positions relative to P1, minimum image)
__device__ __attribute__((noinline)) double restraint_energy_fp64(const LegDev& g, int w) {
  const BoxW& B = g.box[w];
  const size_t base = (size_t)w * g.n, o1 = base + g.ranch[0];
  double p[6][3];
  for (int t = 0; t < 6; ++t) {
    const size_t ot = base + g.ranch[t];
    double d[3] = {(double)g.x[ot] - (double)g.x[o1], (double)g.y[ot] - (double)g.y[o1],
                   (double)g.z[ot] - (double)g.z[o1]};
    for (int c = 0; c < 3; ++c) p[t][c] = d[c] - B.L[c] * rint(d[c] * B.invL[c]);
  }
  return boresch_energy_fp64(p, g.rg0d, g.rkd);
}

template <int ENERGY>
__global__ __launch_bounds__(256) void k_bonded(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const long long i = (long long)(blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  const int per = g.nbonds + g.ntors + 1;
  const long long tot = (long long)g.W * per;
  const int lane = threadIdx.x & 63;
  double eb = 0.0, er = 0.0;
  const int w = (int)(min(i, tot - 1) / per);
  if (i < tot) {
    const int k = (int)(i - (long long)w * per);
    const size_t base = (size_t)w * g.n;
    if (k < g.nbonds) {
      const int a = g.bond_ij[2 * k], b = g.bond_ij[2 * k + 1];
      const float3 d = vec(g, g.box[w], base + b, base + a);          // r_a - r_b
      const float r = sqrtf(d.x * d.x + d.y * d.y + d.z * d.z);
      const float dr = r - g.bond_r0[k];
      const float fs = -g.bond_k[k] * dr / r;                // F_a = fs (r_a - r_b)
      add_force(g, base + a, fs * d.x, fs * d.y, fs * d.z, kSiteBonded);
      add_force(g, base + b, -fs * d.x, -fs * d.y, -fs * d.z, kSiteBonded);
      eb = ENERGY == 2 ? bond_energy_fp64(g, g.box[w], base + a, base + b, k)
                       : 0.5 * (double)g.bond_k[k] * (double)dr * (double)dr;
    } else if (k < g.nbonds + g.ntors) {
      const int t = k - g.nbonds;
      const float lv = g.lam[4 * w + 1];
      if (lv != 0.0f) {
        v3 p[4], F[4];
        const size_t o0 = base + g.tors[4 * t];
        for (int s = 0; s < 4; ++s) {
          const size_t os = base + g.tors[4 * t + s];
          const float3 d = min_img(g.box[w], g.x[os] - g.x[o0], g.y[os] - g.y[o0], g.z[os] - g.z[o0]);
          p[s] = mk(d.x, d.y, d.z);
        }
        const float e = torsion_eval(p, g.tors_k[t], g.tors_n[t], g.tors_phase[t], F);
        for (int s = 0; s < 4; ++s)
          add_force(g, base + g.tors[4 * t + s], lv * F[s].x, lv * F[s].y, lv * F[s].z, kSiteBonded);
        eb = (double)lv * (ENERGY == 2 ? torsion_energy_at(g, w, t) : (double)e);
      }
    } else if (g.has_rest && g.lam[4 * w + 2] != 0.0f) {
      const float lr = g.lam[4 * w + 2];
      v3 p[6], F[6];
      const size_t o1 = base + g.ranch[0];
      for (int t = 0; t < 6; ++t) {
        const size_t ot = base + g.ranch[t];
        const float3 d = min_img(g.box[w], g.x[ot] - g.x[o1], g.y[ot] - g.y[o1], g.z[ot] - g.z[o1]);
        p[t] = mk(d.x, d.y, d.z);
      }
      er = (double)lr * boresch_eval(p, g.rg0, g.rk, F);
      if (ENERGY == 2) er = (double)lr * restraint_energy_fp64(g, w);
      for (int t = 0; t < 6; ++t)
        add_force(g, base + g.ranch[t], lr * F[t].x, lr * F[t].y, lr * F[t].z, kSiteBonded);
    }
  }
  if (ENERGY) {
    const int w0 = __shfl(w, 0, 64);
    const bool same = __ballot(i < tot && w != w0) == 0ull;
    if (same) {
      add_energy(g, w0, FELIS_E_BOND, eb, lane);
      add_energy(g, w0, FELIS_E_RESTRAINT, er, lane);
    } else if (i < tot) {
      long long* acc = g.eacc + (size_t)w * FELIS_NE;
      atomicAdd((unsigned long long*)&acc[FELIS_E_BOND], (unsigned long long)to_fixed(eb, kEnergyScale, g.err));
      atomicAdd((unsigned long long*)&acc[FELIS_E_RESTRAINT], (unsigned long long)to_fixed(er, kEnergyScale, g.err));
    }
  }
}

// items: window -- zero energy accumulators [c0, c1)
__global__ void k_ezero(const LegDev* legs, BlockMap map, int c0, int c1) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int w = (blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  if (w >= g.W) return;
  for (int c = c0; c < c1; ++c) g.eacc[(size_t)w * FELIS_NE + c] = 0;
}

// items: window -- publish components [c0, c1) and the total
__global__ void k_efinish(const LegDev* legs, BlockMap map, int c0, int c1) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int w = (blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  if (w >= g.W) return;
  double* e = g.energy + (size_t)w * FELIS_NE;
  for (int c = c0; c < c1; ++c) e[c] = (double)g.eacc[(size_t)w * FELIS_NE + c] * (1.0 / kEnergyScale);
  double t = 0.0;
  for (int c = 0; c < FELIS_E_TOTAL; ++c) t += e[c];
  e[FELIS_E_TOTAL] = t;
}

inline int blocks_for(long long items, int per) { return (int)((items + per - 1) / per); }

}  // namespace

void launch_pack(hipStream_t s, const LegDev* d, const LegHost* h, int nl, bool rebuild) {
  BlockMap m;
  const int nb = make_map(m, nl, [&](int i) { return (int)(((long long)h[i].W * h[i].npad + 255) / 256); });
  if (!nb) return;
  if (rebuild) hipLaunchKernelGGL(k_pack<true>, dim3(nb), dim3(256), 0, s, d, m);
  else hipLaunchKernelGGL(k_pack<false>, dim3(nb), dim3(256), 0, s, d, m);
}

void launch_pairs(hipStream_t s, const LegDev* d, const LegHost* h, int nl, int energy, bool step) {
  BlockMap m;
  const int nb = make_map(m, nl, [&](int i) { return blocks_for((long long)h[i].W * h[i].nclus, 4); });
  if (!nb) return;
  const int st = step ? 1 : 0;
  if (energy == 1) hipLaunchKernelGGL(k_pairs<1>, dim3(nb), dim3(256), 0, s, d, m, 0);
  else hipLaunchKernelGGL(k_pairs<0>, dim3(nb), dim3(256), 0, s, d, m, st);
  if (energy == 2) hipLaunchKernelGGL(k_pair_energy, dim3(nb), dim3(256), 0, s, d, m);
}

void launch_corrections(hipStream_t s, const LegDev* d, const LegHost* h, int nl, bool energy) {
  BlockMap m;
  if (energy) {             // excluded-pair corrections are part of the pair kernel
    const int nb = make_map(m, nl, [&](int i) { return h[i].W; });
    if (nb) hipLaunchKernelGGL(k_self, dim3(nb), dim3(256), 0, s, d, m);
  }
}

void launch_bonded(hipStream_t s, const LegDev* d, const LegHost* h, int nl, int energy) {
  BlockMap m;
  const int nb = make_map(m, nl, [&](int i) { return blocks_for((long long)h[i].W * (h[i].nbonds + h[i].ntors + 1), 256); });
  if (!nb) return;
  if (energy == 2) hipLaunchKernelGGL(k_bonded<2>, dim3(nb), dim3(256), 0, s, d, m);
  else if (energy == 1) hipLaunchKernelGGL(k_bonded<1>, dim3(nb), dim3(256), 0, s, d, m);
  else hipLaunchKernelGGL(k_bonded<0>, dim3(nb), dim3(256), 0, s, d, m);
}

void launch_zero_energy(hipStream_t s, const LegDev* d, const LegHost* h, int nl, int c0, int c1) {
  BlockMap m;
  const int nb = make_map(m, nl, [&](int i) { return blocks_for(h[i].W, 64); });
  if (nb) hipLaunchKernelGGL(k_ezero, dim3(nb), dim3(64), 0, s, d, m, c0, c1);
}

void launch_finish_energy(hipStream_t s, const LegDev* d, const LegHost* h, int nl, int c0, int c1) {
  BlockMap m;
  const int nb = make_map(m, nl, [&](int i) { return blocks_for(h[i].W, 64); });
  if (nb) hipLaunchKernelGGL(k_efinish, dim3(nb), dim3(64), 0, s, d, m, c0, c1);
}

}  // namespace felis
