// MBAR (Shirts & Chodera 2008), named in section "Simulation protocol" as the
// estimator of each segment's free energy.  The free energies f solve
//   f_i = -ln sum_n exp(-u_in) / sum_k N_k exp(f_k - u_kn),
// the stationary point of the convex function
//   F(f) = sum_n logden_n(f) - sum_i N_i f_i,  logden_n = LSE_k(ln N_k + f_k - u_kn),
// with gradient g_i = N_i (sum_n W_in - 1) and Hessian
//   H_ij = delta_ij N_i sum_n W_in - N_i N_j sum_n W_in W_jn,
// W_in = exp(f_i - u_in - logden_n).  Newton steps on the sampled states
// (gauge: the first sampled state is held fixed), with a backtracking line
// search on F while steps are large (a change of F below its rounding level
// counts as no increase), and a self-consistent step
// f_i <- f_i - ln sum_n W_in when the Newton system is singular.  Unsampled
// states follow from the converged denominators.  Converged when the
// self-consistent update at the current iterate (the fixed-point iteration's
// own change, relative to the gauge state) or a full Newton step is within
// tol * max(1, max|f|); final gauge f_0 = 0.  Sums that are not finite (u holds
// a NaN, or a sample that no sampled state can hold), and a self-consistent
// step where the gauge state has no weight to take it from, end the iteration
// without a result.
//
// All device work is FP64 in a fixed summation order, so the result does not
// depend on launch timing.  Two forms of the same iteration:
//  - up to kFusedStates states: one kernel per evaluation (k_eval) reads u once
//    and makes the denominators, the weights and the curvature, a reduction
//    over its blocks, and one workgroup (k_newton) that solves the Newton
//    system and advances the iteration.  The host only enqueues rounds and
//    looks at the outcome after several of them.
//  - more states: logden per sample with per-block objective partials, the
//    weight matrix W [K][N], per-chunk partial sums of W rows and of the 16x16
//    tiles of W W^T, a fixed-order reduction over chunks, and the K x K Newton
//    system on the host.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "felis_internal.h"

namespace felis {
namespace {

constexpr int kChunk = 4096;      // samples per partial-sum chunk
constexpr int kTile = 16;         // Hessian tile edge
constexpr int kStage = 64;        // samples staged in LDS per tile step

inline size_t al256(size_t b) { return (b + 255) / 256 * 256; }

struct MbarWork {
  double* logden;   // [N]
  double* fpart;    // [ceil(N/256)] block sums of logden
  double* W;        // [K][N]
  double* gpart;    // [nch][K]
  double* hpart;    // [nch][K][K]
  double* G;        // [K] sum_n W_in
  double* H;        // [K][K] sum_n W_in W_jn
  double* f;        // [K]
  double* logN;     // [K] (-inf for N_k = 0)
};

MbarWork carve(void* work, int K, long long N) {
  const long long nch = (N + kChunk - 1) / kChunk, nb = (N + 255) / 256;
  char* p = (char*)work;
  MbarWork w;
  w.logden = (double*)p; p += al256(N * 8);
  w.fpart = (double*)p; p += al256(nb * 8);
  w.W = (double*)p; p += al256((size_t)K * N * 8);
  w.gpart = (double*)p; p += al256((size_t)nch * K * 8);
  w.hpart = (double*)p; p += al256((size_t)nch * K * K * 8);
  w.G = (double*)p; p += al256((size_t)K * 8);
  w.H = (double*)p; p += al256((size_t)K * K * 8);
  w.f = (double*)p; p += al256((size_t)K * 8);
  w.logN = (double*)p; p += al256((size_t)K * 8);
  return w;
}

// thread per sample: logden_n; block sums of logden (objective)
__global__ __launch_bounds__(256) void k_logden(const double* __restrict__ u, MbarWork w, int K, long long N) {
  __shared__ double s_b[512];
  __shared__ double red[256];
  for (int k = threadIdx.x; k < K; k += blockDim.x) s_b[k] = w.logN[k] + w.f[k];
  __syncthreads();
  const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double ld = 0.0;
  if (n < N) {
    double m = -INFINITY;
    for (int k = 0; k < K; ++k) m = fmax(m, s_b[k] - u[(long long)k * N + n]);
    double s = 0.0;
    for (int k = 0; k < K; ++k) s += exp(s_b[k] - u[(long long)k * N + n] - m);
    ld = m + log(s);
    w.logden[n] = ld;
  }
  red[threadIdx.x] = ld;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) w.fpart[blockIdx.x] = red[0];
}

// thread per (i, n): W_in
__global__ __launch_bounds__(256) void k_weights(const double* __restrict__ u, MbarWork w, int K, long long N) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)K * N) return;
  const int i = (int)(t / N);
  const long long n = t - (long long)i * N;
  w.W[t] = exp(w.f[i] - u[t] - w.logden[n]);
}

// block (chunk, tile i, tile j): partial sums over the chunk of W_in W_jn for a
// 16x16 tile (thread = one (i, j)); tiles on the diagonal also sum W_in
__global__ __launch_bounds__(256) void k_gram(MbarWork w, int K, long long N, int ntile) {
  const int per = ntile * ntile;
  const int c = blockIdx.x / per;
  const int tt = blockIdx.x - c * per;
  const int ti = tt / ntile, tj = tt - ti * ntile;
  const int a = threadIdx.x / kTile, b = threadIdx.x % kTile;
  const int i = ti * kTile + a, j = tj * kTile + b;
  const long long n0 = (long long)c * kChunk, n1 = min(N, n0 + kChunk);
  __shared__ double si[kTile][kStage + 1], sj[kTile][kStage + 1];
  double acc = 0.0, gs = 0.0;
  for (long long s0 = n0; s0 < n1; s0 += kStage) {
    const int len = (int)min((long long)kStage, n1 - s0);
    for (int e = threadIdx.x; e < kTile * kStage; e += blockDim.x) {
      const int r = e / kStage, q = e % kStage;
      const int ri = ti * kTile + r, rj = tj * kTile + r;
      si[r][q] = (q < len && ri < K) ? w.W[(long long)ri * N + s0 + q] : 0.0;
      sj[r][q] = (q < len && rj < K) ? w.W[(long long)rj * N + s0 + q] : 0.0;
    }
    __syncthreads();
    for (int q = 0; q < len; ++q) acc += si[a][q] * sj[b][q];
    if (ti == tj && b == 0)
      for (int q = 0; q < len; ++q) gs += si[a][q];
    __syncthreads();
  }
  if (i < K && j < K) w.hpart[((long long)c * K + i) * K + j] = acc;
  if (ti == tj && b == 0 && i < K) w.gpart[(long long)c * K + i] = gs;
}

// thread per (i, j): fixed-order sum over chunks
__global__ __launch_bounds__(256) void k_reduce(MbarWork w, int K, int nch) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= K * K) return;
  double s = 0.0;
  for (int c = 0; c < nch; ++c) s += w.hpart[(long long)c * K * K + t];
  w.H[t] = s;
  if (t < K) {
    double g = 0.0;
    for (int c = 0; c < nch; ++c) g += w.gpart[(long long)c * K + t];
    w.G[t] = g;
  }
}

struct Eval {
  double F;                      // objective
  std::vector<double> G, H;      // sum_n W_in, sum_n W_in W_jn
};

// Upload f, run the device passes, bring back what the host step needs.
int evaluate(hipStream_t s, const double* u, const MbarWork& w, int K, long long N, const std::vector<double>& f,
             const std::vector<double>& Nk, bool full, Eval& ev) {
  const long long nb = (N + 255) / 256;
  const int nch = (int)((N + kChunk - 1) / kChunk);
  const int ntile = (K + kTile - 1) / kTile;
  if (hipMemcpyAsync(w.f, f.data(), sizeof(double) * K, hipMemcpyHostToDevice, s) != hipSuccess) return FELIS_E_DEVICE;
  hipLaunchKernelGGL(k_logden, dim3((unsigned)nb), dim3(256), 0, s, u, w, K, N);
  std::vector<double> fp(nb);
  if (full) {
    hipLaunchKernelGGL(k_weights, dim3((unsigned)(((long long)K * N + 255) / 256)), dim3(256), 0, s, u, w, K, N);
    hipLaunchKernelGGL(k_gram, dim3((unsigned)(nch * ntile * ntile)), dim3(256), 0, s, w, K, N, ntile);
    hipLaunchKernelGGL(k_reduce, dim3((unsigned)((K * K + 255) / 256)), dim3(256), 0, s, w, K, nch);
    ev.G.resize(K);
    ev.H.resize((size_t)K * K);
    if (hipMemcpyAsync(ev.G.data(), w.G, sizeof(double) * K, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(ev.H.data(), w.H, sizeof(double) * K * K, hipMemcpyDeviceToHost, s) != hipSuccess)
      return FELIS_E_DEVICE;
  }
  if (hipMemcpyAsync(fp.data(), w.fpart, sizeof(double) * nb, hipMemcpyDeviceToHost, s) != hipSuccess)
    return FELIS_E_DEVICE;
  if (hipStreamSynchronize(s) != hipSuccess) return FELIS_E_DEVICE;
  double F = 0.0;
  for (long long b = 0; b < nb; ++b) F += fp[b];
  for (int i = 0; i < K; ++i)
    if (Nk[i] > 0) F -= Nk[i] * f[i];
  ev.F = F;
  return FELIS_OK;
}

// Solve A x = b (m x m, row-major, overwritten) by Gaussian elimination with
// partial pivoting; false if a pivot vanishes or the result is not finite.
bool solve(std::vector<double>& A, std::vector<double>& b, int m) {
  double scale = 0.0;
  for (double v : A) scale = std::fmax(scale, std::fabs(v));
  if (!(scale > 0.0)) return m == 0;
  for (int k = 0; k < m; ++k) {
    int p = k;
    for (int r = k + 1; r < m; ++r)
      if (std::fabs(A[(size_t)r * m + k]) > std::fabs(A[(size_t)p * m + k])) p = r;
    if (!(std::fabs(A[(size_t)p * m + k]) > 1e-14 * scale)) return false;
    if (p != k) {
      for (int c = 0; c < m; ++c) std::swap(A[(size_t)k * m + c], A[(size_t)p * m + c]);
      std::swap(b[k], b[p]);
    }
    for (int r = k + 1; r < m; ++r) {
      const double l = A[(size_t)r * m + k] / A[(size_t)k * m + k];
      if (l == 0.0) continue;
      for (int c = k; c < m; ++c) A[(size_t)r * m + c] -= l * A[(size_t)k * m + c];
      b[r] -= l * b[k];
    }
  }
  for (int k = m - 1; k >= 0; --k) {
    double v = b[k];
    for (int c = k + 1; c < m; ++c) v -= A[(size_t)k * m + c] * b[c];
    b[k] = v / A[(size_t)k * m + k];
    if (!std::isfinite(b[k])) return false;
  }
  return true;
}

// ---- the fused form

// Most states of the fused form: 5 tiles of 16, with which a wave of k_eval holds
// 20 states' values and 5 tiles' sums in registers, its weights take 41 KB of LDS
// and the Newton system of 79 free states 51 KB.  More take the general form
constexpr int kFusedStates = 80;
constexpr int kEvalBlocks = 512;  // two per CU: later rounds of a block keep its sums in registers
constexpr int kDirect = 4;        // up to this many blocks' sums k_newton adds up itself

enum : int { kPhFull = 0, kPhLine = 1, kPhFinal = 2, kPhDone = 3 };

struct IterState {
  int phase, it, done, code;      // code: FELIS_E_NOCONV when a step was not finite (no result)
  int ls, pad_;
  double F, t, slope, smax, f_round;
};

// What the host hands over by value: sample counts and the free states
struct FusedArgs {
  int nk[kFusedStates];
  unsigned char idx[kFusedStates];          // sampled states other than the gauge state
  int K, m, ref, nblk, max_iter;
  long long N;
  double tol;
};

struct FusedWork {
  IterState* st;
  double *f, *fe, *step, *G, *out;          // [K] accepted point, point to evaluate, step, G there, result
  double* red;                              // [E] sums over all samples: H [K][K], G [K], objective
  double* part;                             // [nblk][E]
};

inline size_t fused_elems(int K) { return (size_t)K * K + K + 1; }

// Lays the fused form's arrays out in `bytes` of workspace (the size the other
// form needs); false when not even one block's sums fit.  *nblk: blocks used.
bool carve_fused(void* work, size_t bytes, int K, long long N, FusedWork& w, int* nblk) {
  if (K > kFusedStates) return false;
  const size_t E = fused_elems(K), fixed = sizeof(IterState) / 8 + 5 * (size_t)K + E;
  static_assert(sizeof(IterState) % 8 == 0, "followed by doubles");
  const size_t have = bytes / 8;
  if (have < fixed + E) return false;
  const long long tiles = (N + 63) / 64;
  const long long per = (tiles + kEvalBlocks - 1) / kEvalBlocks;       // rounds of the busiest block
  *nblk = (int)std::min<long long>((tiles + per - 1) / per, (long long)((have - fixed) / E));
  w.st = (IterState*)work;
  double* p = (double*)work + sizeof(IterState) / 8;
  for (double** q : {&w.f, &w.fe, &w.step, &w.G, &w.out}) { *q = p; p += K; }
  w.red = p;
  w.part = p + E;
  return true;
}

__global__ __launch_bounds__(128) void k_fused_init(FusedWork w, FusedArgs a) {
  const int k = threadIdx.x;
  if (k < a.K) { w.f[k] = 0.0; w.fe[k] = 0.0; w.step[k] = 0.0; w.G[k] = 0.0; w.out[k] = 0.0; }
  if (k == 0) {
    IterState s;
    s.phase = kPhFull; s.it = 0; s.done = 0; s.code = 0; s.ls = 0; s.pad_ = 0;
    s.F = 0.0; s.t = 1.0; s.slope = 0.0; s.smax = 0.0; s.f_round = 0.0;
    *w.st = s;
  }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// One evaluation: per sample m = max_k(ln N_k + f_k - u_k), e_k = exp(f_k -
// u_k - m), s = sum_k N_k e_k, logden = m + ln s, W_k = e_k / s (one
// exponential per state and sample), then W W^T and the row sums of W.
//
// A block takes 64 samples at a time: lane = sample, each of the four waves a
// quarter of the states (held in registers between the maximum and the
// exponential).  The weights go to LDS as [sample][state], and the matrix
// cores multiply them: v_mfma_f64_16x16x4 takes A[i][n] and B[n][j] from lane
// i + 16 n (j + 16 n), i.e. 16 consecutive states of 4 samples, and the tiles
// of the upper triangle, with one column of ones per tile row for the row
// sums, are shared out over the waves.  Their sums stay in registers over the
// block's rounds.  A sample's states are stored at state ^ (sample & 15)
// within a tile and rows are an odd number of tiles long, so the writes (64
// samples, one state) meet in 2 of 32 bank pairs and the reads in none.
// Bound: reading u (8 K N bytes) and one FP64 exponential an element.  42 x
// 84,000: 43 us an evaluation with its reduction (separate denominators,
// weights and products through memory: 277 us), 27 us for k_newton.
template <int T>
__global__ __launch_bounds__(256) void k_eval(const double* __restrict__ u, FusedWork w, FusedArgs a) {
  if (w.st->phase == kPhDone) return;
  constexpr int NS = 4 * T;                      // states per wave
  constexpr int LD = 16 * (T | 1);
  constexpr int NT = T * (T + 1) / 2;            // tiles of the upper triangle
  constexpr int PW = (NT + T + 3) / 4;           // products per wave
  __shared__ double s_w[64 * LD];
  __shared__ double s_m[4][64], s_s[4][64];
  __shared__ double s_f[16 * T], s_n[16 * T], s_ln[16 * T];
  const int K = a.K, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int k = threadIdx.x; k < 16 * T; k += 256) {
    const double n = k < K ? (double)a.nk[k] : 0.0;
    s_f[k] = k < K ? w.fe[k] : 0.0;
    s_n[k] = n;
    s_ln[k] = n > 0.0 ? log(n) : -INFINITY;
  }
  int ti[PW], tj[PW];                            // this wave's products; tj == T: the row sums
#pragma unroll
  for (int q = 0; q < PW; ++q) {
    int p = wave + 4 * q;
    if (p < NT) {
      int r = 0;
      while (p >= T - r) { p -= T - r; ++r; }
      ti[q] = r; tj[q] = r + p;
    } else {
      ti[q] = p - NT; tj[q] = T;                 // ti >= T: none
    }
  }
  f64x4 acc[PW];
#pragma unroll
  for (int q = 0; q < PW; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
  double fsum = 0.0;
  const long long tiles = (a.N + 63) / 64;
  double un[NS];                                 // the next round's u, in flight during the products
  auto load = [&](long long tile) {
    const long long n = tile * 64 + lane;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const int k = wave * NS + q;
      un[q] = (n < a.N && k < K) ? u[(long long)k * a.N + n] : INFINITY;
    }
  };
  load(blockIdx.x);
  __syncthreads();
  for (long long tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const bool valid = tile * 64 + lane < a.N;
    double m = -INFINITY;
#pragma unroll
    for (int q = 0; q < NS; ++q) m = fmax(m, s_f[wave * NS + q] - un[q] + s_ln[wave * NS + q]);
    s_m[wave][lane] = m;
    __syncthreads();
    m = fmax(fmax(s_m[0][lane], s_m[1][lane]), fmax(s_m[2][lane], s_m[3][lane]));
    double e[NS], sum = 0.0;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const double nk = s_n[wave * NS + q];
      e[q] = nk > 0.0 ? exp(s_f[wave * NS + q] - un[q] - m) : 0.0;         // uniform
      sum += nk * e[q];
    }
    s_s[wave][lane] = sum;
    __syncthreads();
    sum = ((s_s[0][lane] + s_s[1][lane]) + s_s[2][lane]) + s_s[3][lane];
    const double inv = 1.0 / sum, ld = m + log(sum);
    if (wave == 0 && valid) fsum += ld;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const int k = wave * NS + q;
      double v = e[q] * inv;
      if (k < K && !(s_n[k] > 0.0)) v = exp(s_f[k] - un[q] - ld);          // an unsampled state (uniform)
      s_w[lane * LD + (k & ~15) + ((k ^ lane) & 15)] = valid && k < K ? v : 0.0;
    }
    load(tile + gridDim.x);
    __syncthreads();
    const int col = lane & 15, row = lane >> 4;
    for (int n0 = 0; n0 < 64; n0 += 4) {
      const double* r = s_w + (n0 + row) * LD + (col ^ ((n0 + row) & 15));
#pragma unroll
      for (int q = 0; q < PW; ++q) {
        if (ti[q] >= T) continue;                // uniform
        const double x = r[16 * ti[q]];
        const double y = tj[q] == T ? 1.0 : r[16 * tj[q]];
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[q], 0, 0, 0);
      }
    }
    __syncthreads();                             // s_w, s_m and s_s are rewritten next
  }
  // D[i][j]: register r of lane j + 16 g holds row i = 4 r + g
  double* out = w.part + (size_t)blockIdx.x * ((size_t)K * K + K + 1);
#pragma unroll
  for (int q = 0; q < PW; ++q) {
    if (ti[q] >= T) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * ti[q] + 4 * r + (lane >> 4);
      const int j = 16 * tj[q] + (lane & 15);
      if (i >= K) continue;
      if (tj[q] == T) {
        if ((lane & 15) == 0) out[K * K + i] = acc[q][r];
      } else if (j < K) {
        out[i * K + j] = acc[q][r];
        out[j * K + i] = acc[q][r];              // on the diagonal tile both triangles hold the same sums
      }
    }
  }
  if (wave == 0) {
    fsum = wave_sum(fsum);
    if (lane == 0) out[K * K + K] = fsum;
  }
}

// 32 elements per block: the evaluation blocks' sums added in a fixed order
// (each half-wave every 32nd block, then the 32 half-waves)
__global__ __launch_bounds__(1024) void k_eval_reduce(FusedWork w, FusedArgs a) {
  if (w.st->phase == kPhDone) return;
  const int E = a.K * a.K + a.K + 1;
  const int col = threadIdx.x & 31, row = threadIdx.x >> 5;
  const int e = blockIdx.x * 32 + col;
  __shared__ double s_p[32][33];
  double v = 0.0;
  if (e < E) {
#pragma unroll 4
    for (int b = row; b < a.nblk; b += 32) v += w.part[(size_t)b * E + e];
  }
  s_p[row][col] = v;
  __syncthreads();
  if (row == 0 && e < E) {
    for (int k = 1; k < 32; ++k) v += s_p[k][col];
    w.red[e] = v;
  }
}

// One workgroup: the sums at the evaluated point advance the iteration --
// line search, stopping rule, Newton step -- exactly as the host form below
// does, and set the next point to evaluate.  An accepted trial point of the
// line search is at once the next iterate (its sums are already here).
// The Newton matrix is a symmetric, diagonally dominant M-matrix (sum_j N_j
// W_jn = 1), so elimination keeps its diagonal pivots; Gauss-Jordan in LDS,
// one barrier a pivot.
__global__ __launch_bounds__(512) void k_newton(FusedWork w, FusedArgs a) {
  extern __shared__ double s_A[];                // [m][m + 1], the last column the right-hand side
  __shared__ double s_f[kFusedStates], s_step[kFusedStates], s_G[kFusedStates], s_col[kFusedStates];
  __shared__ double s_red[8], s_F;
  __shared__ int s_bad;
  if (w.st->phase == kPhDone) return;
  const int K = a.K, m = a.m, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  IterState st = *w.st;
  const double* sums = a.nblk <= kDirect ? w.part : w.red;
  const int nsum = a.nblk <= kDirect ? a.nblk : 1, E = K * K + K + 1;
  auto sum_of = [&](int e) {
    double v = sums[e];
    for (int b = 1; b < nsum; ++b) v += sums[(size_t)b * E + e];
    return v;
  };
  auto block_max = [&](double v) {               // over all threads; same value everywhere
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    __syncthreads();
    if (lane == 0) s_red[wave] = v;
    __syncthreads();
    v = s_red[0];
    for (int k = 1; k < 8; ++k) v = fmax(v, s_red[k]);
    return v;
  };
  auto block_sum = [&](double v) {
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) s_red[wave] = v;
    __syncthreads();
    v = s_red[0];
    for (int k = 1; k < 8; ++k) v += s_red[k];
    return v;
  };
  const bool mine = tid < K;
  const double nk = mine ? (double)a.nk[tid] : 0.0;
  double f = mine ? w.f[tid] : 0.0;              // thread k holds state k's numbers
  double step = mine ? w.step[tid] : 0.0;
  const double fe = mine ? w.fe[tid] : 0.0;
  const double G = mine ? sum_of(K * K + tid) : 0.0;
  const double F = sum_of(E - 1) - block_sum(nk > 0.0 ? nk * fe : 0.0);
  if (mine) s_G[tid] = G;
  __syncthreads();

  auto write_state = [&]() {
    if (tid == 0) *w.st = st;
  };
  auto finish = [&](int done) {                  // G holds the sums at f: unsampled states, gauge f_0 = 0
    if (mine && nk == 0.0) f -= log(G);
    if (mine) s_f[tid] = f;
    __syncthreads();
    if (mine) w.out[tid] = f - s_f[0];
    st.done = done;
    st.phase = kPhDone;
    write_state();
  };
  auto next = [&](double at, int phase) {        // evaluate `at` next
    if (mine) { w.f[tid] = f; w.step[tid] = step; w.fe[tid] = at; }
    st.phase = phase;
    write_state();
  };
  auto fail = [&]() {
    st.code = FELIS_E_NOCONV;
    st.phase = kPhDone;
    write_state();
  };
  // the self-consistent step from the sums g_k, relative to the gauge state;
  // false when that holds no weight
  auto sc_step = [&](double g) {
    if (mine) s_col[tid] = g;
    __syncthreads();
    const double gr = s_col[a.ref];
    step = (mine && nk > 0.0 && tid != a.ref) ? -log(g) + log(gr) : 0.0;
    return gr > 0.0;
  };
  // the step just taken: converged, out of iterations, or on
  auto after_step = [&]() {
    const double fmaxv = block_max(mine ? fabs(f) : 0.0);
    if (st.t == 1.0 && st.smax <= a.tol * fmax(1.0, fmaxv)) { st.done = 1; return true; }
    return st.it >= a.max_iter;
  };

  if (st.phase == kPhFinal) { finish(st.done); return; }
  if (st.phase == kPhLine) {
    if (!(F <= st.F + 1e-4 * st.t * st.slope + st.f_round)) {
      st.t *= 0.5;
      if (++st.ls < 30) { next(f + st.t * step, kPhLine); return; }
      // no decrease found: a self-consistent step from the iterate's own sums
      st.t = 1.0;
      if (!sc_step(mine ? w.G[tid] : 0.0)) { fail(); return; }
      st.smax = block_max(fabs(step));
      f += step;
      const bool end = after_step();
      next(f, end ? kPhFinal : kPhFull);
      return;
    }
    f = fe;
    if (after_step()) { finish(st.done); return; }
  }
  // sums at the iterate f; the maxima below drop a NaN, so it is asked for by
  // itself (a sample's logden is finite where its sampled states' weights are)
  if (!isfinite(F)) { fail(); return; }
  ++st.it;
  st.t = 1.0;
  const double fscale = block_max(mine ? fmax(1.0, fabs(f)) : 1.0);
  const double gref = s_G[a.ref];
  if (gref > 0.0) {
    const double dl = (mine && nk > 0.0 && tid != a.ref) ? log(G) - log(gref) : 0.0;
    // a non-finite change says the test does not hold
    const double sc = block_max(isfinite(dl) ? fabs(dl) : INFINITY);
    if (sc <= a.tol * fscale) { finish(1); return; }
  }
  const int ld = m + 1;
  double amax = 0.0;
  for (int e = tid; e < m * m; e += 512) {
    const int r = e / m, c = e - r * m;
    const int i = a.idx[r], j = a.idx[c];
    const double ni = (double)a.nk[i], nj = (double)a.nk[j];
    const double v = (i == j ? ni * s_G[i] : 0.0) - ni * nj * sum_of(i * K + j);
    s_A[r * ld + c] = v;
    amax = fmax(amax, fabs(v));
  }
  for (int r = tid; r < m; r += 512) {
    const int i = a.idx[r];
    s_A[r * ld + m] = -(double)a.nk[i] * (s_G[i] - 1.0);
  }
  const double scale = block_max(amax);          // (its barriers order the writes above)
  bool newton = scale > 0.0 || m == 0;
  const double b0 = tid < m ? s_A[tid * ld + m] : 0.0;        // -gradient
  for (int k = 0; newton && k < m; ++k) {
    const double piv = s_A[k * ld + k];
    if (!(fabs(piv) > 1e-14 * scale)) { newton = false; break; }         // uniform
    double ip = __builtin_amdgcn_rcp(piv);                     // refined to FP64 by two Newton steps
    ip = fma(fma(-piv, ip, 1.0), ip, ip);
    ip = fma(fma(-piv, ip, 1.0), ip, ip);
    for (int r = tid >> 3; r < m; r += 64) {                   // 8 lanes a row
      if (r == k) continue;
      const double l = s_A[r * ld + k] * ip;                   // column k is left as it is
      for (int c = k + 1 + (tid & 7); c < ld; c += 8) s_A[r * ld + c] -= l * s_A[k * ld + c];
    }
    __syncthreads();
  }
  if (tid == 0) s_bad = 0;
  if (mine) s_step[tid] = 0.0;
  __syncthreads();
  double slope = 0.0;
  if (newton) {
    double x = 0.0;
    if (tid < m) {
      x = s_A[tid * ld + m] / s_A[tid * ld + tid];
      s_step[a.idx[tid]] = x;
      if (!isfinite(x)) s_bad = 1;
    }
    slope = block_sum(-b0 * x);
    newton = s_bad == 0 && (slope < 0.0 || m == 0);            // (after block_sum's barriers)
  }
  __syncthreads();
  if (newton) step = mine ? s_step[tid] : 0.0;
  else if (!sc_step(G)) { fail(); return; }
  if (tid == 0) s_bad = 0;
  __syncthreads();
  if (mine && !isfinite(step)) s_bad = 1;
  st.smax = block_max(fabs(step));
  if (s_bad) { fail(); return; }
  if (newton && st.smax > 1e-3) {                // backtracking on F while the step is large
    st.F = F;
    st.slope = slope;
    st.ls = 0;
    st.f_round = 1e-12 * (fabs(F) + block_sum(nk * fabs(f)));
    if (mine) w.G[tid] = G;
    next(f + step, kPhLine);
    return;
  }
  f += step;
  const bool end = after_step();
  next(f, end ? kPhFinal : kPhFull);
}

template <int T>
void launch_eval(hipStream_t s, const double* u, const FusedWork& w, const FusedArgs& a) {
  hipLaunchKernelGGL(k_eval<T>, dim3((unsigned)a.nblk), dim3(256), 0, s, u, w, a);
}

int fused_mbar(hipStream_t s, const double* u, const FusedWork& w, const FusedArgs& a, double* f_out, int* iters) {
  hipLaunchKernelGGL(k_fused_init, dim3(1), dim3(128), 0, s, w, a);
  const size_t lds = (size_t)a.m * (a.m + 1) * sizeof(double);
  const unsigned nred = (unsigned)((fused_elems(a.K) + 31) / 32);
  struct { IterState st; double v[5 * kFusedStates]; } back;               // the state and the arrays behind it
  const size_t nback = sizeof(IterState) + 5 * (size_t)a.K * sizeof(double);
  // most solves take 6 to 9 evaluations; one that is over leaves at once
  for (int rounds = 7;; rounds = 4) {
    for (int r = 0; r < rounds; ++r) {
      switch ((a.K + 15) / 16) {
        case 1: launch_eval<1>(s, u, w, a); break;
        case 2: launch_eval<2>(s, u, w, a); break;
        case 3: launch_eval<3>(s, u, w, a); break;
        case 4: launch_eval<4>(s, u, w, a); break;
        default: launch_eval<5>(s, u, w, a); break;
      }
      if (a.nblk > kDirect) hipLaunchKernelGGL(k_eval_reduce, dim3(nred), dim3(1024), 0, s, w, a);
      hipLaunchKernelGGL(k_newton, dim3(1), dim3(512), lds, s, w, a);
    }
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&back, w.st, nback, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return FELIS_E_DEVICE;
    if (back.st.phase == kPhDone) break;
  }
  if (back.st.code) return back.st.code;
  for (int k = 0; k < a.K; ++k) f_out[k] = back.v[4 * a.K + k];
  if (iters) *iters = back.st.it;
  for (int k = 0; k < a.K; ++k)
    if (!std::isfinite(f_out[k])) return FELIS_E_NOCONV;
  return back.st.done ? FELIS_OK : FELIS_E_NOCONV;
}

}  // namespace

size_t mbar_work_bytes(int K, long long N) {
  const long long nch = (N + kChunk - 1) / kChunk, nb = (N + 255) / 256;
  return al256(N * 8) + al256(nb * 8) + al256((size_t)K * N * 8) + al256((size_t)nch * K * 8) +
         al256((size_t)nch * K * K * 8) + al256((size_t)K * 8) + al256((size_t)K * K * 8) + 2 * al256((size_t)K * 8);
}

int launch_mbar(hipStream_t s, const double* u, const int* N_k, int K, long long N, double tol, int max_iter,
                double* f_out, int* iters, void* work, size_t work_bytes) {
  if (K < 2 || K > 512 || N < 1 || !u || !N_k || !f_out || !work || !(tol > 0) || max_iter < 1)
    return FELIS_E_INVAL;
  if (work_bytes < mbar_work_bytes(K, N)) return FELIS_E_INVAL;
  long long tot = 0;
  for (int k = 0; k < K; ++k) {
    if (N_k[k] < 0) return FELIS_E_INVAL;
    tot += N_k[k];
  }
  if (tot != N) return FELIS_E_INVAL;
  {
    FusedWork fw;
    FusedArgs fa;
    // (laid out for the size asked for, not the size given: both entry points sum in the same order)
    if (carve_fused(work, mbar_work_bytes(K, N), K, N, fw, &fa.nblk)) {
      fa.K = K; fa.N = N; fa.tol = tol; fa.max_iter = max_iter;
      fa.m = 0; fa.ref = -1;
      for (int k = 0; k < K; ++k) {
        fa.nk[k] = N_k[k];
        if (N_k[k] > 0) {
          if (fa.ref < 0) fa.ref = k;
          else fa.idx[fa.m++] = (unsigned char)k;
        }
      }
      return fused_mbar(s, u, fw, fa, f_out, iters);
    }
  }
  MbarWork w = carve(work, K, N);
  std::vector<double> Nk(K), logN(K);
  std::vector<int> idx;                 // sampled states other than the gauge state
  int ref = -1;
  for (int k = 0; k < K; ++k) {
    Nk[k] = N_k[k];
    logN[k] = N_k[k] > 0 ? std::log((double)N_k[k]) : -INFINITY;
    if (N_k[k] > 0) {
      if (ref < 0) ref = k;
      else idx.push_back(k);
    }
  }
  if (hipMemcpyAsync(w.logN, logN.data(), sizeof(double) * K, hipMemcpyHostToDevice, s) != hipSuccess)
    return FELIS_E_DEVICE;
  const int m = (int)idx.size();
  std::vector<double> f(K, 0.0), step(K), ftry(K);
  Eval ev, trial;
  bool done = false;
  int it = 0;
  while (it < max_iter) {
    int rc = evaluate(s, u, w, K, N, f, Nk, true, ev);
    if (rc) return rc;
    if (!std::isfinite(ev.F)) return FELIS_E_NOCONV;
    ++it;
    // the self-consistent update at this iterate, -ln(sum_n W_in) relative
    // to the gauge state: the change of f the fixed-point iteration would
    // make, which is the stopping rule's quantity
    double fscale = 1.0;
    for (int k = 0; k < K; ++k) fscale = std::fmax(fscale, std::fabs(f[k]));
    if (ev.G[ref] > 0.0) {
      double sc = 0.0;
      bool finite = true;
      for (int r = 0; r < m; ++r) {
        const double d = std::log(ev.G[idx[r]]) - std::log(ev.G[ref]);
        finite = finite && std::isfinite(d);
        sc = std::fmax(sc, std::fabs(d));
      }
      if (finite && sc <= tol * fscale) { done = true; break; }
    }
    // gradient of F on the free states and the Newton system H d = -g
    std::vector<double> A((size_t)m * m), b(m);
    for (int r = 0; r < m; ++r) {
      const int i = idx[r];
      b[r] = -Nk[i] * (ev.G[i] - 1.0);
      for (int c = 0; c < m; ++c) {
        const int j = idx[c];
        A[(size_t)r * m + c] = (i == j ? Nk[i] * ev.G[i] : 0.0) - Nk[i] * Nk[j] * ev.H[(size_t)i * K + j];
      }
    }
    std::vector<double> g(b);            // -gradient
    std::fill(step.begin(), step.end(), 0.0);
    bool newton = solve(A, b, m);
    double slope = 0.0;                  // g . d (negative for a descent direction)
    if (newton) {
      for (int r = 0; r < m; ++r) { step[idx[r]] = b[r]; slope -= g[r] * b[r]; }
      newton = slope < 0.0 || m == 0;
    }
    if (!newton) {                       // self-consistent step
      if (!(ev.G[ref] > 0.0)) return FELIS_E_NOCONV;
      std::fill(step.begin(), step.end(), 0.0);
      for (int r = 0; r < m; ++r) step[idx[r]] = -std::log(ev.G[idx[r]]) + std::log(ev.G[ref]);
    }
    double smax = 0.0;
    for (int k = 0; k < K; ++k) {
      if (!std::isfinite(step[k])) return FELIS_E_NOCONV;
      smax = std::fmax(smax, std::fabs(step[k]));
    }
    double t = 1.0;
    if (newton && smax > 1e-3) {         // backtracking on F while the step is large
      // F is a sum over every sample: a change below its rounding level
      // (far from the optimum's curvature along flat directions) is no increase
      double fabs_sum = std::fabs(ev.F);
      for (int k = 0; k < K; ++k) fabs_sum += Nk[k] * std::fabs(f[k]);
      const double f_round = 1e-12 * fabs_sum;
      bool ok = false;
      for (int ls = 0; ls < 30 && !ok; ++ls) {
        for (int k = 0; k < K; ++k) ftry[k] = f[k] + t * step[k];
        rc = evaluate(s, u, w, K, N, ftry, Nk, false, trial);
        if (rc) return rc;
        ok = trial.F <= ev.F + 1e-4 * t * slope + f_round;
        if (!ok) t *= 0.5;
      }
      if (!ok) {                         // no decrease found: self-consistent step instead
        if (!(ev.G[ref] > 0.0)) return FELIS_E_NOCONV;
        t = 1.0;
        smax = 0.0;
        std::fill(step.begin(), step.end(), 0.0);
        for (int r = 0; r < m; ++r) {
          step[idx[r]] = -std::log(ev.G[idx[r]]) + std::log(ev.G[ref]);
          smax = std::fmax(smax, std::fabs(step[idx[r]]));
        }
      }
    }
    double fmaxv = 0.0;
    for (int k = 0; k < K; ++k) {
      f[k] += t * step[k];
      fmaxv = std::fmax(fmaxv, std::fabs(f[k]));
    }
    // or converged when the full (undamped) step is within the tolerance: a
    // step the line search cut short says nothing about the distance left
    if (t == 1.0 && smax <= tol * std::fmax(1.0, fmaxv)) { done = true; break; }
  }
  // unsampled states from the final denominators, then the gauge f_0 = 0
  int rc = evaluate(s, u, w, K, N, f, Nk, true, ev);
  if (rc) return rc;
  for (int k = 0; k < K; ++k)
    if (Nk[k] == 0) f[k] -= std::log(ev.G[k]);
  const double f0 = f[0];
  for (int k = 0; k < K; ++k) f_out[k] = f[k] - f0;
  if (iters) *iters = it;
  for (int k = 0; k < K; ++k)
    if (!std::isfinite(f_out[k])) return FELIS_E_NOCONV;
  return done ? FELIS_OK : FELIS_E_NOCONV;
}

// ---- allocation-free MBAR
//
// Workspace in a file-scope device array, for callers that cannot allocate
// device memory.  Host code never passes `scratch` itself to a kernel (in
// host code the name is a stand-in, not a device address): its device
// address is looked up once per device with hipGetSymbolAddress at context
// creation and kept in g_scratch[device].  Every region of the workspace is
// written by a kernel before any kernel reads it, so nothing needs clearing
// between calls; calls that overlap on one device share the array and race.

static __device__ __align__(256) unsigned char scratch[kMbarStaticBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};
}  // namespace

int mbar_scratch_setup(int device) {
  if (device < 0 || device >= kMaxDevices) return FELIS_E_INVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[device]) return FELIS_OK;
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FELIS_E_DEVICE;
  g_scratch[device] = p;
  return FELIS_OK;
}

int launch_mbar_noalloc(int device, hipStream_t s, const double* u, const int* N_k, int K, long long N, double tol,
                        int max_iter, double* f_out, int* iters) {
  if (K < 2 || K > 512 || N < 1) return FELIS_E_INVAL;
  if (mbar_work_bytes(K, N) > kMbarStaticBytes) return FELIS_E_CAPACITY;
  void* p = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (device >= 0 && device < kMaxDevices) p = g_scratch[device];
  }
  if (!p) return FELIS_E_DEVICE;
  return launch_mbar(s, u, N_k, K, N, tol, max_iter, f_out, iters, p, kMbarStaticBytes);
}

}  // namespace felis
