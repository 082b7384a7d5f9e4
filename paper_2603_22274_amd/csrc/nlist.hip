// Neighbour lists: displacement check, Hilbert cell sort, 8-atom clusters and
// per-cluster j-lists (appendix B cutoffs).
//
// A cluster lists every atom j that lies within r_list + 0.01 A (FP32
// minimum image) of at least one of its atoms i, with one bit per i; the
// margin is far above the FP32 error of d^2, so the listed pairs are a
// superset of the pairs within r_list.  The canonical list -- pairs with
// FP64 d^2 < r_list^2, d = x_j - x_i, d -= L * rint(d / L) as separate
// multiply and subtract, d^2 = (dx^2 + dy^2) + dz^2 -- is what the export
// applies to that superset; this unit is built with -ffp-contract=off so
// that sequence is exact as written.
#include "felis_internal.h"

namespace felis {
namespace {

constexpr int kBloomWords = 1024;             // 32-bit words of k_build's filter of own and excluded atoms
constexpr int kTabOf = 4096;                  // candidates per table window in k_build
// Most cluster pairs in a launch for four waves a pair: every wave repeats the
// pair's set-up and the round's (a sixth of a pair's work), so one wave does
// the least work and four end soonest where the pairs alone do not fill the
// chip.  One | four waves: 504 pairs 15.8 | 10.0 us, 9,440 (20 windows of 7,540
// atoms) 108 | 82, 39,000 245 | 290, 185,000 (42 windows of 70,527) 786 | 1418.
// Near the line, us a step: 7,540 atoms, 12,300 pairs 361 | 340, 16,500 441 | 431,
// 21,200 537 | 540; 70,527 atoms, 13,200 378 | 404, 17,600 469 | 487; 668 atoms, 8,400
// 244 | 254, 16,400 414 | 452
constexpr int kFewPairs = 16384;
constexpr float kFar = 1.0e30f;               // squared distance that no test passes

// a wave-uniform float moved to a scalar register
__device__ __forceinline__ float scalar(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Rows of 16 lanes.  out[k] holds v's row k in every row.
__device__ __forceinline__ void spread_rows(unsigned v, unsigned out[4]) {
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);       // rows 0 1 0 1 | 2 3 2 3
  const auto a = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
  out[0] = a[0];
  out[1] = a[1];
  out[2] = b[0];
  out[3] = b[1];
}
// v[k]'s row r to v[r]'s row k
__device__ __forceinline__ void transpose_rows(float v[4]) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  v[0] = __uint_as_float(c[0]);
  v[1] = __uint_as_float(c[1]);
  v[2] = __uint_as_float(d[0]);
  v[3] = __uint_as_float(d[1]);
}
// the value N lanes before in the row (0 at its start); the row's last value
template <int N>
__device__ __forceinline__ unsigned row_shr(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + N, 0xF, 0xF, true);
}
__device__ __forceinline__ unsigned row_last(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x15F, 0xF, 0xF, true);
}
__device__ __forceinline__ int cell_of(float v, float L, float invL, int n) {
  float u = wrapf(v, L, invL) * invL;
  int c = (int)(u * (float)n);
  return c < 0 ? 0 : (c >= n ? n - 1 : c);
}

// Largest squared displacement since the last build that keeps a window's
// lists and cells valid: (skin/2)^2, less what volume moves have used (a
// move by s changes a pair distance r by at most |s - 1| (r + 2 r_mol) and
// an atom's place in the scaled cell grid by |s - 1| (r_mol + drift)).
__device__ __forceinline__ float skin_threshold2(const LegDev& g, int w) {
  const float used = g.skin_used[w];
  if (used == 0.f) return g.skin_half2;
  if (!(used < g.skin)) return -1.f;             // nothing left: rebuild
  const float t = 0.5f * (g.skin - used);
  return t * t;
}

// Legs of kMovedAtoms atoms or more: the scan of the positions that starts a
// call, kMovedPer atoms a block, into the word that k_check reads (one block a
// window took 104 us for 70,527 atoms in one window, 148 us in each of 42).
// Legs that large have more than 64 units, so nothing else writes the word.
constexpr int kMovedAtoms = 8192;
constexpr int kMovedPer = 2048;

__global__ __launch_bounds__(256) void k_moved(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int parts = (g.n + kMovedPer - 1) / kMovedPer;
  const int b = blockIdx.x - map.start[leg], w = b / parts, a0 = (b - w * parts) * kMovedPer;
  const size_t o = (size_t)w * g.n;
  float m = 0.f;
#pragma unroll
  for (int k = 0; k < kMovedPer / 256; ++k) {
    const int a = a0 + k * 256 + (int)threadIdx.x;
    if (a < g.n) {
      const float dx = g.x[o + a] - g.xr[o + a], dy = g.y[o + a] - g.yr[o + a], dz = g.z[o + a] - g.zr[o + a];
      m = fmaxf(m, dx * dx + dy * dy + dz * dz);
    }
  }
  for (int k = 32; k > 0; k >>= 1) m = fmaxf(m, __shfl_xor(m, k, 64));
  if ((threadIdx.x & 63) == 0 && m > 0.f) atomicMax(&g.maxdisp[w], __float_as_uint(m));
}

// One block per window: rebuild flag = force || max displacement > skin/2;
// a window being rebuilt gets its per-cell counters zeroed.  FROM_WORD: the
// largest squared displacement was recorded by the previous step's
// integrator (same arithmetic as the scan below); either way the word is
// cleared for the next step.
template <bool FROM_WORD>
__global__ __launch_bounds__(1024) void k_check(const LegDev* legs, BlockMap map, int force) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int w = blockIdx.x - map.start[leg];
  const int tid = threadIdx.x;
  __shared__ float red[16];
  float m = 0.f;
  const float limit2 = skin_threshold2(g, w);    // (loaded beside the displacements)
  force |= g.rbforce[w];                         // a box change (barostat) since the last build
  if (FROM_WORD && g.units >= 64) {
    // integrator waves covering this window's units
    const long long u0 = (long long)w * g.units, u1 = u0 + g.units;
    for (long long q = (u0 >> 6) + tid; q <= ((u1 - 1) >> 6); q += blockDim.x) {
      const bool first = (q * 64) / g.units == w;           // this window is the wave's first
      m = fmaxf(m, __uint_as_float(g.wmax[2 * q + (first ? 0 : 1)]));
    }
  } else if (FROM_WORD || g.n >= kMovedAtoms) {
    m = __uint_as_float(g.maxdisp[w]);
  } else if (!force) {
    const size_t o = (size_t)w * g.n;
    for (int a = tid; a < g.n; a += blockDim.x) {
      const float dx = g.x[o + a] - g.xr[o + a], dy = g.y[o + a] - g.yr[o + a], dz = g.z[o + a] - g.zr[o + a];
      m = fmaxf(m, dx * dx + dy * dy + dz * dz);
    }
  }
  for (int k = 32; k > 0; k >>= 1) m = fmaxf(m, __shfl_xor(m, k, 64));
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();                                // (and every thread has read the word)
  for (int k = 0; k < 16; ++k) m = fmaxf(m, red[k]);
  const int f = (force || !(m <= limit2)) ? 1 : 0;          // the same in every thread
  if (tid == 0) {
    g.flag[w] = f;
    g.nbuild[w] += f;
    g.maxdisp[w] = 0u;
    g.rbforce[w] = 0;
    if (f) g.skin_used[w] = 0.f;
  }
  if (f) {
    int4* cur = reinterpret_cast<int4*>(g.cursor + (size_t)w * g.ncell);     // ncell is a power of 8
    for (int c = tid; c < g.ncell >> 2; c += blockDim.x) cur[c] = make_int4(0, 0, 0, 0);
  }
}

// items: window x atom -- Hilbert cell code, per-cell counts, reference positions
__global__ __launch_bounds__(256) void k_cells_count(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const long long i = (long long)(blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  if (i >= (long long)g.W * g.n) return;
  const int w = (int)(i / g.n);
  if (!g.flag[w]) return;
  const int nf = 1 << g.nbits;
  const BoxW& B = g.box[w];
  const float x = g.x[i], y = g.y[i], z = g.z[i];
  const unsigned c = g.hcell[(cell_of(x, B.Lf[0], B.invLf[0], nf) * nf + cell_of(y, B.Lf[1], B.invLf[1], nf)) * nf +
                            cell_of(z, B.Lf[2], B.invLf[2], nf)];
  g.cellcode[i] = (int)c;
  atomicAdd(&g.cursor[(size_t)w * g.ncell + c], 1);
  g.xr[i] = x; g.yr[i] = y; g.zr[i] = z;
}

// one block per window: exclusive scan of the counts into cellstart; reset
// cursor.  The cells go through LDS 16,384 at a time, read and written with
// consecutive lanes on consecutive cells; each thread scans 16 neighbouring
// counts (a word of padding after every 16: no bank conflicts), the block scans
// the threads' sums (wave shuffles, then the 16 wave totals), and a running
// total carries across the pieces.  Latency: 32,768 cells in pieces of 4,096
// took 22.5 us, 18.5 now.
__global__ __launch_bounds__(1024) void k_cells_scan(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int w = blockIdx.x - map.start[leg];
  if (!g.flag[w]) return;
  int* cnt = g.cursor + (size_t)w * g.ncell;
  int* st = g.cellstart + (size_t)w * (g.ncell + 1);
  constexpr int T = 1024, E = 16, TILE = T * E, NW = T / 64;
  __shared__ int s_v[TILE + TILE / E];
  auto at = [](int c) { return c + c / E; };
  __shared__ int s_wt[NW];
  __shared__ int s_tile;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nc = g.ncell;
  int carry = 0;                                  // counts before this piece (same in every thread)
  for (int t0 = 0; t0 < nc; t0 += TILE) {
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int c = t0 + k * T + tid;
      s_v[at(k * T + tid)] = c < nc ? cnt[c] : 0;
    }
    __syncthreads();
    int v[E], sum = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) { v[k] = s_v[at(tid * E + k)]; sum += v[k]; }
    int inc = sum;                                // inclusive scan over the wave
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(inc, o, 64);
      if (lane >= o) inc += u;
    }
    if (lane == 63) s_wt[wave] = inc;
    __syncthreads();
    if (wave == 0) {                              // exclusive scan of the wave totals; the piece's total
      const int t = lane < NW ? s_wt[lane] : 0;
      int ti = t;
      for (int o = 1; o < NW; o <<= 1) {
        const int u = __shfl_up(ti, o, 64);
        if (lane >= o) ti += u;
      }
      if (lane < NW) s_wt[lane] = ti - t;
      if (lane == NW - 1) s_tile = ti;
    }
    __syncthreads();
    int run = carry + s_wt[wave] + inc - sum;
#pragma unroll
    for (int k = 0; k < E; ++k) { s_v[at(tid * E + k)] = run; run += v[k]; }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int c = t0 + k * T + tid;
      if (c < nc) { st[c] = s_v[at(k * T + tid)]; cnt[c] = 0; }
    }
    carry += s_tile;
    __syncthreads();                              // s_v, s_wt and s_tile are rewritten next
  }
  if (tid == 0) st[nc] = carry;
}

// items: window x atom -- place each atom in its cell's range
__global__ __launch_bounds__(256) void k_cells_scatter(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const long long i = (long long)(blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  if (i >= (long long)g.W * g.n) return;
  const int w = (int)(i / g.n);
  if (!g.flag[w]) return;
  const int a = (int)(i - (long long)w * g.n);
  const int c = g.cellcode[i];
  const int slot = g.cellstart[(size_t)w * (g.ncell + 1) + c] + atomicAdd(&g.cursor[(size_t)w * g.ncell + c], 1);
  g.perm[(size_t)w * g.npad + slot] = a;
}

// items: window x cell -- order atoms within a cell by index (makes the sort
// deterministic), then write the padding slots
__global__ __launch_bounds__(256) void k_cells_order(const LegDev* legs, BlockMap map) {
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const long long i = (long long)(blockIdx.x - map.start[leg]) * blockDim.x + threadIdx.x;
  if (i >= (long long)g.W * g.ncell) return;
  const int w = (int)(i / g.ncell);
  if (!g.flag[w]) return;
  const int c = (int)(i - (long long)w * g.ncell);
  const int* st = g.cellstart + (size_t)w * (g.ncell + 1);
  int* p = g.perm + (size_t)w * g.npad;
  const int s0 = st[c], s1 = st[c + 1];
  for (int s = s0 + 1; s < s1; ++s) {
    int v = p[s], t = s - 1;
    while (t >= s0 && p[t] > v) { p[t + 1] = p[t]; --t; }
    p[t + 1] = v;
  }
  if (c == 0)
    for (int s = g.n; s < g.npad; ++s) p[s] = -1;
}

// Legs whose cell grid and atom count fit in LDS run the check and the whole
// cell sort in one block per window: Hilbert codes and per-cell counts in
// LDS, an exclusive scan into cellstart, placement by LDS atomics, then each
// cell's atoms in index order (the same deterministic order as the grid-wide
// kernels above).
constexpr int kSortCells = 4096;
constexpr int kSortAtoms = 12288;

template <bool FROM_WORD>
__global__ __launch_bounds__(1024) void k_check_sort(const LegDev* legs, BlockMap map, int force) {
  static_assert(kSortAtoms % 1024 == 0, "one block of 1024 threads sorts a window");
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int w = blockIdx.x - map.start[leg];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  __shared__ int s_cur[kSortCells];               // counts, then next free slot per cell
  __shared__ int s_st[kSortCells + 1];
  __shared__ unsigned short s_code[kSortAtoms];
  __shared__ int s_perm[kSortAtoms];
  __shared__ float s_red[16];
  __shared__ int s_wsum[16];
  __shared__ int s_flag;
  const size_t o = (size_t)w * g.n;
  float m = 0.f;
  const float limit2 = skin_threshold2(g, w);    // (loaded beside the displacements)
  force |= g.rbforce[w];                         // a box change (barostat) since the last build
  if (FROM_WORD) {
    if (g.units < 64) {
      if (tid == 0) m = __uint_as_float(g.maxdisp[w]);
    } else {
      const long long u0 = (long long)w * g.units, u1 = u0 + g.units;
      for (long long q = (u0 >> 6) + tid; q <= ((u1 - 1) >> 6); q += blockDim.x) {
        const bool first = (q * 64) / g.units == w;
        m = fmaxf(m, __uint_as_float(g.wmax[2 * q + (first ? 0 : 1)]));
      }
    }
  } else if (!force) {
    for (int a = tid; a < g.n; a += blockDim.x) {
      const float dx = g.x[o + a] - g.xr[o + a], dy = g.y[o + a] - g.yr[o + a], dz = g.z[o + a] - g.zr[o + a];
      m = fmaxf(m, dx * dx + dy * dy + dz * dz);
    }
  }
  for (int k = 32; k > 0; k >>= 1) m = fmaxf(m, __shfl_xor(m, k, 64));
  if (lane == 0) s_red[wave] = m;
  __syncthreads();
  if (tid == 0) {
    float r = s_red[0];
    for (int k = 1; k < (int)(blockDim.x >> 6); ++k) r = fmaxf(r, s_red[k]);
    s_flag = (force || !(r <= limit2)) ? 1 : 0;
  }
  __syncthreads();
  const int f = s_flag;                           // uniform over the block
  if (tid == 0) {
    g.flag[w] = f;
    g.nbuild[w] += f;
    g.maxdisp[w] = 0u;
    g.rbforce[w] = 0;
    if (f) g.skin_used[w] = 0.f;
  }
  if (!f) return;

  const int nc = g.ncell, n = g.n, nf = 1 << g.nbits;
  const float bL[3] = {g.box[w].Lf[0], g.box[w].Lf[1], g.box[w].Lf[2]};
  const float biL[3] = {g.box[w].invLf[0], g.box[w].invLf[1], g.box[w].invLf[2]};
  for (int c = tid; c < nc; c += blockDim.x) s_cur[c] = 0;
  // every position this thread sorts is loaded before any is used (at most
  // kSortAtoms / 1024 per thread), so the loads overlap
  constexpr int kPer = kSortAtoms / 1024;
  float px[kPer], py[kPer], pz[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int a = tid + k * 1024;
    if (a < n) { px[k] = g.x[o + a]; py[k] = g.y[o + a]; pz[k] = g.z[o + a]; }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int a = tid + k * 1024;
    if (a < n) {
      const unsigned c = g.hcell[(cell_of(px[k], bL[0], biL[0], nf) * nf + cell_of(py[k], bL[1], biL[1], nf)) *
                                     nf + cell_of(pz[k], bL[2], biL[2], nf)];
      s_code[a] = (unsigned short)c;
      atomicAdd(&s_cur[c], 1);
      g.xr[o + a] = px[k]; g.yr[o + a] = py[k]; g.zr[o + a] = pz[k];
    }
  }
  __syncthreads();
  // exclusive scan: each thread takes a run of consecutive cells
  const int per = (nc + (int)blockDim.x - 1) / (int)blockDim.x;
  const int c0 = min(nc, tid * per), c1 = min(nc, c0 + per);
  int sum = 0;
  for (int c = c0; c < c1; ++c) sum += s_cur[c];
  int inc = sum;
  for (int k = 1; k < 64; k <<= 1) {
    const int v = __shfl_up(inc, k, 64);
    if (lane >= k) inc += v;
  }
  if (lane == 63) s_wsum[wave] = inc;
  __syncthreads();
  int run = inc - sum;
  for (int k = 0; k < wave; ++k) run += s_wsum[k];
  int* cst = g.cellstart + (size_t)w * (nc + 1);
  for (int c = c0; c < c1; ++c) {
    const int cnt = s_cur[c];
    s_st[c] = run;
    cst[c] = run;
    s_cur[c] = run;
    run += cnt;
  }
  if (tid == 0) { s_st[nc] = n; cst[nc] = n; }
  __syncthreads();
  for (int a = tid; a < n; a += blockDim.x) s_perm[atomicAdd(&s_cur[s_code[a]], 1)] = a;
  __syncthreads();
  // index order within each cell: an atom's place is the count of smaller
  // indices in its cell
  int* p = g.perm + (size_t)w * g.npad;
  for (int a = tid; a < n; a += blockDim.x) {
    const int c = s_code[a], b0 = s_st[c], b1 = s_st[c + 1];
    int q = b0;
    for (int t = b0; t < b1; ++t) q += s_perm[t] < a ? 1 : 0;
    p[q] = a;
  }
  for (int q = n + tid; q < g.npad; q += blockDim.x) p[q] = -1;
}

bool sort_in_lds(const LegHost& h) { return h.ncell <= kSortCells && h.n <= kSortAtoms; }

// One workgroup per pair of consecutive clusters (16 atoms): sweep the coarse
// blocks (aligned 2x2x2 fine cells) within r_list of the pair's box, one block
// a lane and round, each trimmed to the Hilbert span of its fine cells within
// r_list, and list every atom j with at least one i of a half-cluster in
// range.  The waves take consecutive 64-candidate parts of each step and
// append in wave order, so the list order is fixed (cells in sweep order,
// slots ascending).
//
// The distance test is a contraction: with r relative to the pair's first
// atom, |r_j - r_i|^2 - (r_list + 0.01)^2 = (-2 r_i, 1) . (r_j, |r_j|^2 - inc2)
// + |r_i|^2, so one 16x16x4 FP32 matrix product tests 16 candidates against
// the 16 atoms, and it leaves a lane with exactly one half-cluster's four
// results (row 4 g + r: atom r of half-cluster g).  Four of them serve a
// wave's 64 candidates, which are brought from one lane a candidate to one row
// a component by four lane-row swaps.  Vector issue bounds it (0.83 wave
// instructions per SIMD and 4 cycles): about 115 instructions for 64
// candidates and 16 atoms, most of them to form masks and places of entries,
// 1,000 for a pair's set-up and rounds.  A list of every window of 42 x 70,527
// atoms takes 2.3 ms; it took 4.2 ms with one workgroup of two waves a
// cluster, eight tests of three FMAs a candidate, a byte table of the
// candidates' blocks and a search of the exclusions by each lane.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 1 ? 6 : 5) void k_build(const LegDev* legs, BlockMap map) {
  static_assert(WAVES <= 4, "a step's counts lie in one word a list");
  constexpr int kThreads = 64 * WAVES;
  const int leg = find_leg(map, blockIdx.x);
  const LegDev& g = legs[leg];
  const int npair = (g.nclus + 1) >> 1;
  const unsigned b = blockIdx.x - (unsigned)map.start[leg];
  const int w = (int)(b / (unsigned)npair);
  if (!g.flag[w]) return;                       // uniform over the block
  const int c = 2 * (int)(b - (unsigned)w * (unsigned)npair);    // the pair's first cluster
  const size_t item = (size_t)w * g.nclus + c;
  const int tid = threadIdx.x, wave = WAVES > 1 ? tid >> 6 : 0, lane = tid & 63;
  const int row = lane >> 4, col = lane & 15;   // matrix layout: half-cluster (or component), candidate

  __shared__ unsigned s_bloom[kBloomWords];     // filter of the pair's own and excluded atoms
  __shared__ unsigned long long s_bits[kTabOf / 64];  // candidates whose successor opens a new block
  __shared__ int s_delta[kThreads];             // per non-empty block of the round: slot - candidate
  __shared__ int s_wsum[WAVES], s_wblk[WAVES];
  __shared__ unsigned s_wc[2][4];               // entries of a step: byte per list and wave
  __shared__ float4 s_xi[16];
  __shared__ float s_ni[16];

  const size_t o = (size_t)w * g.npad;
  const gptr<int> perm = as_global(g.perm + o);
  const gptr<f32x4> xq = as_global4(g.xyzq + o);
  const int n = g.n, cap = g.cap, slot0 = c * kClus, nf = g.ncoarse, nbits = g.nbits;
  const gptr<int> cst = as_global(g.cellstart + (size_t)w * (g.ncell + 1));
  const gptr<unsigned> hcell = as_global(g.hcell);
  const bool two = c + 1 < g.nclus;
  const float4 lo0 = g.bblo[item], hi0 = g.bbhi[item], lo1 = g.bblo[item + two], hi1 = g.bbhi[item + two];
  // the four lists (halves of the first, then of the second cluster) lie one
  // after the other; each lane appends to its row's
  typedef __attribute__((address_space(1))) char gchar;
  gchar* const lists = (gchar*)(g.lent + item * 2 * cap);

  // box edges in scalar registers: read once, not again after every list store
  const BoxW& B = g.box[w];
  const float Lf[3] = {scalar(B.Lf[0]), scalar(B.Lf[1]), scalar(B.Lf[2])};
  const float iLf[3] = {scalar(B.invLf[0]), scalar(B.invLf[1]), scalar(B.invLf[2])};
  const float rlist = scalar((float)g.rlist), incl = rlist + 0.01f;
  const float inc2 = incl * incl;

  // the pair's atoms: atom col of the pair in every row
  const int si = slot0 + col;
  const f32x4 xi = xq[min(si, n - 1)];
  // exclusions: column i holds those of atom i, the first four in its four
  // rows and the others in the second register
  int ex[2] = {-1, -1}, own = -1;
  if (si < n) {
    own = perm[si];
    const int e0 = g.excl_ptr[own], ne = g.excl_ptr[own + 1] - e0;
    for (int h = 0; h < 2; ++h)
      if (4 * h + row < ne) ex[h] = g.excl_idx[e0 + 4 * h + row];
    if (ne > kMaxExcl && tid < 16) latch(g.err, kErrExcl, kSiteExclCount, (w << 20) | own, g.leg_index);
  }
  for (int k = tid; k < kBloomWords; k += kThreads) s_bloom[k] = 0u;
  if (tid < 8) s_wc[tid >> 2][tid & 3] = 0u;
  __syncthreads();
  if (wave == 0) {
    auto put = [&](int a) { atomicOr(&s_bloom[(a >> 5) & (kBloomWords - 1)], 1u << (a & 31)); };
    for (int h = 0; h < 2; ++h)
      if (ex[h] >= 0) put(ex[h]);
    if (row == 0 && si < n) put(own);
  }

  // positions relative to the first atom (always a real one), nearest image
  float ri[3], x0[3];
  bool near = true;
  for (int d = 0; d < 3; ++d) {
    x0[d] = scalar(xi[d]);
    const float v = xi[d] - x0[d];
    ri[d] = __fmaf_rn(-Lf[d], rintf(v * iLf[d]), v);
    // one periodic image per candidate (taken against the first atom) is the
    // nearest image for every i whenever extent + r_list + margin < L/2
    near = near && fabsf(ri[d]) + incl + 0.02f < 0.5f * Lf[d];
  }
  float ni = __fmaf_rn(ri[0], ri[0], __fmaf_rn(ri[1], ri[1], ri[2] * ri[2]));
  // The expanded form rounds by up to 27 2^-24 (|r_i| + r_list)^2 where it counts:
  // 7 roundings of |r_i|^2 and |r_j|^2, 5 of sums within (|r_i| + |r_j|)^2, |r_j| <
  // |r_i| + r_list.  Held below the margin of 0.01 A, 0.02 r_list A^2 (2^-18 (|r_i|^2
  // + r_list^2) is above that bound): |r_i| up to some 230 A at r_list = 10; wider
  // pairs, in sparse systems of large boxes, take the image per pair
  near = near && (ni + inc2) * 3.8146973e-6f < inc2 - rlist * rlist;
  const bool real = si < n && ni < kFar;        // false for a padding slot and for a NaN position
  const bool shift = __ballot(si < n && !near) == 0ull;
  ni = real ? ni : kFar;
  const float am = !real ? 0.f : row == 0 ? -2.0f * ri[0] : row == 1 ? -2.0f * ri[1] : row == 2 ? -2.0f * ri[2] : 1.0f;
  if (tid < 16) {
    s_xi[tid] = make_float4(xi[0], xi[1], xi[2], real ? 0.f : kFar);
    s_ni[tid] = ni;
  }
  __syncthreads();
  const f32x4 ci = {s_ni[4 * row], s_ni[4 * row + 1], s_ni[4 * row + 2], s_ni[4 * row + 3]};

  const float lo[3] = {scalar(fminf(lo0.x, lo1.x)), scalar(fminf(lo0.y, lo1.y)), scalar(fminf(lo0.z, lo1.z))};
  const float hi[3] = {scalar(fmaxf(hi0.x, hi1.x)), scalar(fmaxf(hi0.y, hi1.y)), scalar(fmaxf(hi0.z, hi1.z))};
  const float pre = rlist + 0.05f;
  const float pre2 = pre * pre;
  int r0[3], nC[3];
  bool full[3];
  float csd[3];
  for (int d = 0; d < 3; ++d) {
    float cen = 0.5f * (lo[d] + hi[d]), half = 0.5f * (hi[d] - lo[d]);
    if (!(half >= 0.f && half <= Lf[d])) { cen = 0.f; half = Lf[d]; }   // no valid atom
    // nf is a power of two: exact cell edge; the range ends use its inverse
    // (a rounding flip only adds or drops a cell whose nearest face lies
    // pre - r_list - 0.01 = 0.04 A beyond the list radius)
    const float cs = ldexpf(Lf[d], 1 - nbits);
    const float ics = ldexpf(iLf[d], nbits - 1);
    csd[d] = scalar(cs);
    const int a0 = (int)floorf((cen - half - pre) * ics);
    const int a1 = (int)floorf((cen + half + pre) * ics);
    full[d] = __builtin_amdgcn_readfirstlane(a1 - a0 + 1 >= nf);   // the range wraps onto itself: every cell, no gap test
    r0[d] = __builtin_amdgcn_readfirstlane(full[d] ? 0 : a0);
    nC[d] = __builtin_amdgcn_readfirstlane(full[d] ? nf : a1 - a0 + 1);
  }
  const unsigned first = (unsigned)row * (unsigned)cap * 4u, limit = first + (unsigned)cap * 4u;
  unsigned at = first;
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const unsigned below = wave ? ~0u >> (32 - 8 * wave) : 0u;             // bytes of the waves before this one
  const int ncells = nC[0] * nC[1] * nC[2];
  int par = 0;
  // block index ci -> (c0, c1, c2) by float-reciprocal quotients with one
  // correction (exact for ci < 2^22, with the hardware reciprocal too); a
  // block coordinate lies in (-nf, 2nf)
  // (the range is narrower than the box unless full), so one wrap suffices
  const int n12 = nC[1] * nC[2];
  const float inv12 = __builtin_amdgcn_rcpf((float)n12), inv2 = __builtin_amdgcn_rcpf((float)nC[2]);
  auto wrapc = [nf](int c) { return c < 0 ? c + nf : (c >= nf ? c - nf : c); };
  for (int cb = 0; cb < ncells; cb += kThreads) {
    const int cell = cb + tid;
    int s0 = 0, cnt = 0;
    if (cell < ncells) {
      int c0 = (int)((float)cell * inv12);
      c0 += (cell - c0 * n12 < 0) ? -1 : (cell - c0 * n12 >= n12 ? 1 : 0);
      const int rem = cell - c0 * n12;
      int c1 = (int)((float)rem * inv2);
      c1 += (rem - c1 * nC[2] < 0) ? -1 : (rem - c1 * nC[2] >= nC[2] ? 1 : 0);
      const int C[3] = {r0[0] + c0, r0[1] + c1, r0[2] + rem - c1 * nC[2]};
      float gap2 = 0.f;
      for (int d = 0; d < 3; ++d) {
        if (full[d]) continue;
        const float cs = csd[d];
        const float gp = fmaxf(0.f, fmaxf((float)C[d] * cs - hi[d], lo[d] - (float)(C[d] + 1) * cs));
        gap2 += gp * gp;
      }
      if (gap2 < pre2) {
        // the block's 8 fine cells hold 8 consecutive Hilbert indices: take
        // the span from the first to the last child that passes its own gap test
        float g2c[3][2];
        for (int d = 0; d < 3; ++d)
          for (int hh = 0; hh < 2; ++hh) {
            const float cf = 0.5f * csd[d];
            const int F = 2 * C[d] + hh;
            const float gp = fmaxf(0.f, fmaxf((float)F * cf - hi[d], lo[d] - (float)(F + 1) * cf));
            g2c[d][hh] = full[d] ? 0.f : gp * gp;
          }
        const int nff = 2 * nf, W0 = 2 * wrapc(C[0]), W1 = 2 * wrapc(C[1]), W2 = 2 * wrapc(C[2]);
        unsigned hc[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          hc[k] = hcell[((W0 + (k >> 2)) * nff + W1 + ((k >> 1) & 1)) * nff + W2 + (k & 1)];
        unsigned kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (g2c[0][k >> 2] + g2c[1][(k >> 1) & 1] + g2c[2][k & 1] < pre2) {
            kmin = min(kmin, hc[k]);
            kmax = max(kmax, hc[k]);
          }
        if (kmin <= kmax) {
          s0 = cst[kmin];
          cnt = cst[kmax + 1] - s0;
        }
      }
    }
    int inc = cnt;
    for (int k = 1; k < 64; k <<= 1) {
      const int v = __shfl_up(inc, k, 64);
      if (lane >= k) inc += v;
    }
    const unsigned long long held = __ballot(cnt > 0);
    if (lane == 63) { s_wsum[wave] = inc; s_wblk[wave] = __popcll(held); }
    __syncthreads();
    int pos = inc - cnt, blk = __popcll(held & lt), total = 0;
    for (int k = 0; k < WAVES; ++k) {
      if (k < wave) { pos += s_wsum[k]; blk += s_wblk[k]; }
      total += s_wsum[k];
    }
    total = __builtin_amdgcn_readfirstlane(total);
    if (cnt > 0) s_delta[blk] = s0 - pos;
    // candidate t belongs to the block whose number is the count of blocks
    // that open at 1..t: bit t - 1 marks an opening at t, kTabOf at a time
    int opened = 0;
    for (int T0 = 0; T0 < total; T0 += kTabOf) {
      for (int k = tid; k < kTabOf / 64; k += kThreads) s_bits[k] = 0ull;
      __syncthreads();
      if (cnt > 0 && pos > T0 && pos <= T0 + kTabOf)
        atomicOr((unsigned*)s_bits + ((pos - 1 - T0) >> 5), 1u << ((pos - 1 - T0) & 31));
      __syncthreads();
      const int T1 = min(total, T0 + kTabOf);
      // a lane's candidate of the step at t0, loaded a step ahead
      int s, a;
      f32x4 xj;
      auto fetch = [&](int t0) {
        unsigned long long mine = 0ull;
        int op = opened;
        for (int k = 0; k < WAVES; ++k) {
          const unsigned long long v = s_bits[((t0 - T0) >> 6) + k];
          const int ones = __popcll(v);
          if (k < wave) op += ones;
          if (k == wave) mine = v;
          opened += ones;
        }
        const int t = t0 + tid;
        const int blkno = __builtin_amdgcn_mbcnt_hi((unsigned)(mine >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mine, op));
        const int v = t + s_delta[blkno];
        s = t < T1 ? v : slot0;
        a = *(gptr<int>)((gptr<char>)perm + 4u * (unsigned)s);
        xj = *(gptr<f32x4>)((gptr<char>)xq + 16u * (unsigned)s);
      };
      fetch(T0);
      for (int t0 = T0; t0 < T1; t0 += kThreads) {
        const int tb = t0 + 64 * wave;                    // this wave's part
        unsigned m[4] = {0u, 0u, 0u, 0u}, ent[4];
        const int s_now = s, a_now = a;
        const f32x4 xj_now = xj;
        if (t0 + kThreads < T1) fetch(t0 + kThreads);
        if (tb < T1) {
          const int s = s_now, a = a_now;
          const f32x4 xj = xj_now;
          const bool in = tb + lane < T1;
          // possibly an own or excluded atom?  (settled below)
          const unsigned bit = (s_bloom[(a >> 5) & (kBloomWords - 1)] >> (a & 31)) & 1u;
          unsigned long long hits = __ballot(bit) & __ballot(in);
          spread_rows((unsigned)s << 8, ent);
          if (shift) {
            float r[3];
            for (int d = 0; d < 3; ++d) {
              const float v = xj[d] - x0[d];
              r[d] = __fmaf_rn(-Lf[d], rintf(v * iLf[d]), v);
            }
            float thr = __fmaf_rn(r[0], r[0], __fmaf_rn(r[1], r[1], r[2] * r[2])) - inc2;
            const bool ok = in && thr < kFar;
            if (__ballot(!ok)) {                    // past the end, or a NaN position: in no list
              asm volatile("");
              for (int d = 0; d < 3; ++d) r[d] = ok ? r[d] : 0.f;
              thr = ok ? thr : kFar;
            }
            float bm[4] = {r[0], r[1], r[2], thr};
            transpose_rows(bm);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(am, bm[k], ci, 0, 0, 0);
              unsigned v = __float_as_uint(d[3]) >> 31;           // bit r: atom r is in range (its sign)
              v = __builtin_amdgcn_alignbit(v, __float_as_uint(d[2]), 31);
              v = __builtin_amdgcn_alignbit(v, __float_as_uint(d[1]), 31);
              m[k] = __builtin_amdgcn_alignbit(v, __float_as_uint(d[0]), 31);
            }
          } else {
            // small boxes and wide cluster pairs: the nearest image per pair
            unsigned mask = 0;
#pragma unroll 4
            for (int ii = 0; ii < 16; ++ii) {
              const float4 p = s_xi[ii];
              float dx = xj[0] - p.x, dy = xj[1] - p.y, dz = xj[2] - p.z;
              dx = __fmaf_rn(-Lf[0], rintf(dx * iLf[0]), dx);
              dy = __fmaf_rn(-Lf[1], rintf(dy * iLf[1]), dy);
              dz = __fmaf_rn(-Lf[2], rintf(dz * iLf[2]), dz);
              const float d2 = __fmaf_rn(dx, dx, __fmaf_rn(dy, dy, __fmaf_rn(dz, dz, p.w)));
              mask |= d2 < inc2 ? 1u << ii : 0u;
            }
            unsigned v[4];
            spread_rows(in ? mask : 0u, v);
            for (int k = 0; k < 4; ++k) m[k] = (v[k] >> (4 * row)) & 0xFu;
          }
          if (hits) {
            // the pairs of these candidates that are an atom with itself or
            // excluded: 16 bits over the pair's atoms
            unsigned drop = 0;
            do {
              const int q = __builtin_ctzll(hits);
              hits &= hits - 1;
              const int aq = __builtin_amdgcn_readlane(a, q);
              unsigned long long x = __ballot(ex[0] == aq) | __ballot(ex[1] == aq) | __ballot(own == aq);
              x |= x >> 32;
              drop = lane == q ? (unsigned)(x | x >> 16) & 0xFFFFu : drop;
            } while (hits);
            unsigned v[4];
            spread_rows(drop, v);
            for (int k = 0; k < 4; ++k) {
              const unsigned x = (v[k] >> (4 * row)) & 0xFu;
              ent[k] |= (m[k] & x) ? kListPartial : 0u;
              m[k] &= ~x;
            }
          }
        }
        // place of each entry: the four parts' flags in the four bytes of a
        // word, summed along the row, then over the parts, then over the waves
        unsigned f = 0;
        for (int k = 0; k < 4; ++k) f |= min(m[k], 1u) << (8 * k);
        unsigned sum = f;
        sum += row_shr<1>(sum);
        sum += row_shr<2>(sum);
        sum += row_shr<4>(sum);
        sum += row_shr<8>(sum);
        unsigned tot = row_last(sum);
        tot += tot << 8;
        asm("" : "+v"(tot));                        // (else a multiplication, at a quarter of the rate)
        tot += tot << 16;
        asm("" : "+v"(tot));
        const unsigned place = sum - f + (tot << 8);
        unsigned o4 = at;
        if (WAVES > 1) {
          if (col == 0) ((unsigned char*)&s_wc[par][row])[wave] = (unsigned char)(tot >> 24);
          __syncthreads();
          const unsigned v = s_wc[par][row];
          o4 += 4u * __builtin_amdgcn_sad_u8(v & below, 0u, 0u);
          at += 4u * __builtin_amdgcn_sad_u8(v, 0u, 0u);
          par ^= 1;
        } else {
          at += 4u * (tot >> 24);
        }
        if (tb < T1) {
          unsigned p[4];
          for (int k = 0; k < 4; ++k) p[k] = o4 + 4u * ((place >> (8 * k)) & 0xFFu);
          if (__ballot(at > limit)) {               // past the capacity: counted, not stored
            asm volatile("");                       // (a branch: not selects on the way of every step)
            for (int k = 0; k < 4; ++k) m[k] = p[k] < limit ? m[k] : 0u;
          }
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (m[k]) *(__attribute__((address_space(1))) unsigned*)(lists + p[k]) = ent[k] | m[k];
        }
      }
      __syncthreads();                          // the table is rewritten next
    }
    __syncthreads();                            // the round's sums and blocks are rewritten next
  }
  if (wave == 0 && col == 0 && c + (row >> 1) < g.nclus) {
    const int count = (int)((at - first) >> 2);
    if (count > cap) {
      latch(g.err, kErrListCap, kSiteList, (w << 20) | max(perm[slot0], 0), g.leg_index);
      atomicMax(g.need, count);
    }
    g.lcount[2 * item + row] = min(count, cap);
  }
}

// Export pairs i < j with a set list bit and FP64 distance < r (both
// half-cluster lists).
__global__ __launch_bounds__(256) void k_export(const LegDev* legs, int leg, int w, double r2,
                                                int* pairs, long long cap,
                                                unsigned long long* count) {
  const LegDev& g = legs[leg];
  const int c = blockIdx.x;
  if (c >= g.nclus) return;
  const size_t item = (size_t)w * g.nclus + c;
  const int* perm = g.perm + (size_t)w * g.npad;
  const size_t o = (size_t)w * g.n;
  for (int half = 0; half < 2; ++half) {
    const unsigned* ent = g.lent + (item * 2 + half) * g.cap;
    const int cnt = g.lcount[item * 2 + half];
    for (int e = threadIdx.x; e < cnt; e += blockDim.x) {
      const unsigned v = ent[e];
      const unsigned m = v & 0xfu;
      if (!m) continue;
      const int aj = perm[v >> 8];
      for (int k = 0; k < 4; ++k) {
        if (!((m >> k) & 1u)) continue;
        const int ai = perm[c * kClus + 4 * half + k];
        if (ai >= aj) continue;
        double dx = (double)g.x[o + aj] - (double)g.x[o + ai];
        double dy = (double)g.y[o + aj] - (double)g.y[o + ai];
        double dz = (double)g.z[o + aj] - (double)g.z[o + ai];
        const BoxW& B = g.box[w];
        dx = dx - B.L[0] * rint(dx * B.invL[0]);
        dy = dy - B.L[1] * rint(dy * B.invL[1]);
        dz = dz - B.L[2] * rint(dz * B.invL[2]);
        const double d2 = (dx * dx + dy * dy) + dz * dz;
        if (!(d2 < r2)) continue;
        const unsigned long long k2 = atomicAdd(count, 1ull);
        if ((long long)k2 < cap) { pairs[2 * k2] = ai; pairs[2 * k2 + 1] = aj; }
      }
    }
  }
}

inline int blocks_for(long long items, int per) { return (int)((items + per - 1) / per); }

}  // namespace

void launch_check(hipStream_t s, const LegDev* d, const LegHost* h, int nl, int force, bool from_word) {
  BlockMap m;
  int nb = make_map(m, nl, [&](int i) { return sort_in_lds(h[i]) ? 0 : h[i].W; });
  if (nb) {
    if (!from_word && !force) {
      BlockMap mv;
      const int nm = make_map(mv, nl, [&](int i) {
        return sort_in_lds(h[i]) || h[i].n < kMovedAtoms ? 0 : h[i].W * blocks_for(h[i].n, kMovedPer);
      });
      if (nm) hipLaunchKernelGGL(k_moved, dim3(nm), dim3(256), 0, s, d, mv);
    }
    if (from_word) hipLaunchKernelGGL(k_check<true>, dim3(nb), dim3(1024), 0, s, d, m, force);
    else hipLaunchKernelGGL(k_check<false>, dim3(nb), dim3(1024), 0, s, d, m, force);
  }
  // small legs: the check and the whole cell sort in one launch
  nb = make_map(m, nl, [&](int i) { return sort_in_lds(h[i]) ? h[i].W : 0; });
  if (nb) {
    if (from_word) hipLaunchKernelGGL(k_check_sort<true>, dim3(nb), dim3(1024), 0, s, d, m, force);
    else hipLaunchKernelGGL(k_check_sort<false>, dim3(nb), dim3(1024), 0, s, d, m, force);
  }
}

void launch_sort_pack(hipStream_t s, const LegDev* d, const LegHost* h, int nl) {
  BlockMap m;
  // grid-wide cell sort for the legs that launch_check did not sort
  auto big = [&](int i) { return !sort_in_lds(h[i]); };
  int nb = make_map(m, nl, [&](int i) { return big(i) ? blocks_for((long long)h[i].W * h[i].n, 256) : 0; });
  if (nb) hipLaunchKernelGGL(k_cells_count, dim3(nb), dim3(256), 0, s, d, m);
  nb = make_map(m, nl, [&](int i) { return big(i) ? h[i].W : 0; });
  if (nb) hipLaunchKernelGGL(k_cells_scan, dim3(nb), dim3(1024), 0, s, d, m);
  nb = make_map(m, nl, [&](int i) { return big(i) ? blocks_for((long long)h[i].W * h[i].n, 256) : 0; });
  if (nb) hipLaunchKernelGGL(k_cells_scatter, dim3(nb), dim3(256), 0, s, d, m);
  nb = make_map(m, nl, [&](int i) { return big(i) ? blocks_for((long long)h[i].W * h[i].ncell, 256) : 0; });
  if (nb) hipLaunchKernelGGL(k_cells_order, dim3(nb), dim3(256), 0, s, d, m);
  // sorted coordinates every step; sorted parameters and cluster boxes for
  // the windows being rebuilt
  launch_pack(s, d, h, nl, true);
}

void launch_lists(hipStream_t s, const LegDev* d, const LegHost* h, int nl) {
  BlockMap m;
  const int nb = make_map(m, nl, [&](int i) { return h[i].W * ((h[i].nclus + 1) / 2); });
  if (nb > kFewPairs) hipLaunchKernelGGL(k_build<1>, dim3(nb), dim3(64), 0, s, d, m);
  else if (nb) hipLaunchKernelGGL(k_build<4>, dim3(nb), dim3(256), 0, s, d, m);
}

void launch_build(hipStream_t s, const LegDev* d, const LegHost* h, int nl) {
  launch_sort_pack(s, d, h, nl);
  launch_lists(s, d, h, nl);
}

void launch_export(hipStream_t s, const LegDev* d, const LegHost& h, int window, double r,
                   int* pairs, long long cap, unsigned long long* count) {
  if (h.nclus) hipLaunchKernelGGL(k_export, dim3(h.nclus), dim3(256), 0, s, d, 0, window, r * r, pairs, cap, count);
}

}  // namespace felis
