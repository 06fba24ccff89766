// pisa_block_heterogeneity: M_j = || H_j - Hbar ||, Hbar = (1/N) sum_j H_j, and the column
// bias log(M_j + eps) of the covariance-aware selection score (Methodology,
// "Covariance-Aware Block Selection"; H_j from "Global First-Order Correction").
//
// Everything here is fp64: the bias is added to fp64 pooled logits and has to keep their
// accuracy.  Two passes over K and V, no per-block matrices in memory:
//   (1) hsum64_kernel   one workgroup per chunk of blocks accumulates sum_j H_j on the fp64
//                       matrix cores; the partial sums are added in chunk order and divided
//                       by N (hbar64_kernel).  A caller that accepts Hbar at fp32 accuracy hands
//                       in the hsum of the statistics pass instead and saves this pass;
//   (2) hetero_kernel   one workgroup per block rebuilds H_j the same way on top of -Hbar, so that
//                       D_j = H_j - Hbar ends up in the accumulators, and takes its norm from
//                       there: the Frobenius norm, or the largest singular value by a Lanczos
//                       iteration on D^T D that never leaves the registers but for two short vectors.
#include <hip/hip_bf16.h>

#include "common.h"

namespace pisa {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kRows = 64;    // tokens staged at a time

// Four waves share a D x D matrix by rows: wave w owns key channels (D/4) w .. (D/4) w + D/4 - 1 and all value
// channels, as TA x TB accumulator tiles of v_mfma_f64_16x16x4_f64.  Lane (i = lane % 16, kk = lane / 16)
// supplies token 4 s + kk of contraction step s, key channels (D/4) w + TA i + a and value channels TB i + b: K and V
// stay in LDS as they came (bf16 or fp32), a lane's channels are neighbours (one or two reads a step) and the
// block mean it subtracts is a register.  The result is
//   acc[a][b][e] <-> key channel (D/4) w + TA (4 e + kk) + a, value channel TB i + b.
template <int D> struct Geo {
  static constexpr int TA = D / 64;        // key tiles per wave
  static constexpr int TB = D / 16;        // value tiles
  static constexpr int NY = 4 * TA;        // rows of the matrix a lane has elements of
  static constexpr int NQ = TB / 4;        // entries of a D-vector a lane holds when a wave spreads it over its lanes
  // Partial sums lie in memory in the order of the accumulators, a pair acc[a][b][e], acc[a][b + 1][e] (b even) of thread
  // tid at pair_at: every store of a wave is 1 KB in one piece.  (As rows and columns a lane's 16 bytes lay 64 apart: sum
  // over 19 heads of 10 blocks 21.7 us in bf16 and 22.4 in fp32, now 15.6 and 16.3.)
  __device__ static inline int pair_at(int a, int e, int b, int tid) { return ((a * 4 + e) * (TB / 2) + b / 2) * 256 + tid; }
  // The same place by row (key channel) and even column (value channel).
  __device__ static inline int pair_of(int row, int col) {
    const int w = row / (D / 4), r = row % (D / 4), a = r % TA, kk = r / TA % 4, e = r / TA / 4;
    return pair_at(a, e, col % TB, 64 * w + 16 * kk + col / TB);
  }
};

// N neighbouring channels as they lie in LDS, and widened to fp64.
template <typename T, int N> struct Raw {
  static constexpr int WORDS = (N * (int)sizeof(T) + 3) / 4;
  unsigned w[WORDS];
  __device__ inline void load(const T* p) {
    if constexpr (WORDS >= 4) {
#pragma unroll
      for (int c = 0; c < WORDS; c += 4) {
        const uint4 x = reinterpret_cast<const uint4*>(p)[c / 4];
        w[c] = x.x; w[c + 1] = x.y; w[c + 2] = x.z; w[c + 3] = x.w;
      }
    } else if constexpr (WORDS == 2) {
      const uint2 x = *reinterpret_cast<const uint2*>(p);
      w[0] = x.x; w[1] = x.y;
    } else if constexpr (N * sizeof(T) == 4) {
      w[0] = *reinterpret_cast<const unsigned*>(p);
    } else {
      w[0] = *reinterpret_cast<const unsigned short*>(p);
    }
  }
  __device__ inline double get(int c) const {
    if constexpr (sizeof(T) == 4) return (double)__uint_as_float(w[c]);
    else return (double)__uint_as_float((c & 1) ? w[c / 2] & 0xffff0000u : w[c / 2] << 16);
  }
};

// The rows of up to kRows tokens of K and V, 16 bytes per lane and load.
template <typename T, int D> struct Staged {
  static constexpr int CPR = D * (int)sizeof(T) / 16;      // 16-byte chunks per row
  static constexpr int NLD = kRows * CPR / 256;            // loads per lane and tensor
  uint4 k[NLD], v[NLD];
};
template <typename T, int D>
__device__ inline void load_rows(Staged<T, D>& st, const T* kh, const T* vh, int row0, int rows) {
  constexpr int CPR = Staged<T, D>::CPR;
#pragma unroll
  for (int u = 0; u < Staged<T, D>::NLD; ++u) {
    const int n = (u * 256 + (int)threadIdx.x) / CPR, c = (u * 256 + (int)threadIdx.x) % CPR;
    st.k[u] = st.v[u] = make_uint4(0u, 0u, 0u, 0u);        // rows past the block: v = 0 makes them count nothing
    if (n < rows) {
      st.k[u] = reinterpret_cast<const uint4*>(kh + (size_t)(row0 + n) * D)[c];
      st.v[u] = reinterpret_cast<const uint4*>(vh + (size_t)(row0 + n) * D)[c];
    }
  }
}
template <typename T, int D>
__device__ inline void store_rows(const Staged<T, D>& st, T (*ks)[D], T (*vs)[D]) {
  constexpr int CPR = Staged<T, D>::CPR;
#pragma unroll
  for (int u = 0; u < Staged<T, D>::NLD; ++u) {
    const int n = (u * 256 + (int)threadIdx.x) / CPR, c = (u * 256 + (int)threadIdx.x) % CPR;
    reinterpret_cast<uint4*>(ks[n])[c] = st.k[u];
    reinterpret_cast<uint4*>(vs[n])[c] = st.v[u];
  }
}

// acc += sum over the staged tokens of (k_n - mean)^T v_n.
template <typename T, int D>
__device__ inline void add_products(f64x4 (&acc)[Geo<D>::TA][Geo<D>::TB], const T (*ks)[D], const T (*vs)[D],
                                    const double (&mean)[Geo<D>::TA], int rows) {
  constexpr int TA = Geo<D>::TA, TB = Geo<D>::TB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, kk = lane >> 4;
  const T* kp = &ks[kk][(D / 4) * wave + TA * i];
  const T* vp = &vs[kk][TB * i];
  // G steps at a time: their reads go out together, and the scheduling fences keep the conversions of a step
  // behind the products of the one before (all at once they would not fit the registers).
  constexpr int G = sizeof(T) * D > 256 ? 2 : 4;
  auto steps_together = [&](int s0) {
    Raw<T, TA> kr[G];
    Raw<T, TB> vr[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      kr[u].load(kp + 4 * (s0 + u) * D);
      vr[u].load(vp + 4 * (s0 + u) * D);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < G; ++u) {
      double af[TA], bf[TB];
#pragma unroll
      for (int a = 0; a < TA; ++a) af[a] = kr[u].get(a) - mean[a];
#pragma unroll
      for (int b = 0; b < TB; ++b) bf[b] = vr[u].get(b);
#pragma unroll
      for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[a], bf[b], acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll 1
  for (int s = 0; s < (rows + 3) / 4; s += G) steps_together(s);   // staged rows past the block have v = 0
}

// The block's means of this lane's key channels; held back until they have arrived, so that the loads issued
// after them are not waited for along with them.
template <int D>
__device__ inline void load_means(double (&mean)[Geo<D>::TA], const double* kmean) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int a = 0; a < Geo<D>::TA; ++a) mean[a] = kmean[(D / 4) * wave + Geo<D>::TA * (lane & 15) + a];
#pragma unroll
  for (int a = 0; a < Geo<D>::TA; ++a) asm volatile("" : "+v"(mean[a]));
}

// (1) The sum of H_j over a chunk of blocks.  The rows of the next 64 tokens are in flight while the products of
// the current ones run.  Bound by the fp64 matrix instruction: 2 D^2 flop per token at 128 flop per clock and CU.
template <typename T, int D>
__global__ __launch_bounds__(256, 2) void hsum64_kernel(const T* __restrict__ k, const T* __restrict__ v,
                                                     const double* __restrict__ kbar64,
                                                     double* __restrict__ partial, int L, int B, int N,
                                                     int chunk_blocks, int n_chunks) {
  constexpr int TA = Geo<D>::TA, TB = Geo<D>::TB;
  __shared__ __attribute__((aligned(16))) T ks[kRows][D];
  __shared__ __attribute__((aligned(16))) T vs[kRows][D];
  const int chunk = blockIdx.x;
  const size_t bh = blockIdx.y;
  const T* kh = k + bh * (size_t)L * D;
  const T* vh = v + bh * (size_t)L * D;
  f64x4 acc[TA][TB];
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int first = chunk * chunk_blocks * B, last = min(L, min(N, (chunk + 1) * chunk_blocks) * B);
  Staged<T, D> st;
  load_rows(st, kh, vh, first, min(kRows, last - first));
  for (int row0 = first; row0 < last; row0 += kRows) {       // kRows divides B: 64 tokens lie in one block
    double mean[TA];
    load_means<D>(mean, kbar64 + (bh * N + row0 / B) * D);
    __syncthreads();
    store_rows(st, ks, vs);
    __syncthreads();
    if (row0 + kRows < last) load_rows(st, kh, vh, row0 + kRows, min(kRows, last - row0 - kRows));
    add_products<T, D>(acc, ks, vs, mean, min(kRows, last - row0));
  }
  f64x2* ph = reinterpret_cast<f64x2*>(partial + (bh * n_chunks + chunk) * (size_t)D * D);
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int b = 0; b < TB; b += 2)
        ph[Geo<D>::pair_at(a, e, b, threadIdx.x)] = f64x2{acc[a][b][e], acc[a][b + 1][e]};
}

// hbar64[bh][e] = hsum[bh][e] / N from the fp32 sum the statistics pass has already produced.
__global__ __launch_bounds__(256) void hbar_from_hsum_kernel(const float* __restrict__ hsum,
                                                             double* __restrict__ hbar64, size_t total, int N) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e < total) hbar64[e] = (double)hsum[e] / (double)N;
}

// hbar64[bh] = (sum over chunks, in chunk order, of partial[bh][chunk]) / N, row-major: a thread per pair of columns (a
// wave writes 1 KB in one piece and reads pieces of 256 bytes).
template <int D>
__global__ __launch_bounds__(256) void hbar64_kernel(const double* __restrict__ partial,
                                                     double* __restrict__ hbar64, int n_chunks, int N) {
  constexpr int pairs = D * D / 2;
  const size_t bh = blockIdx.y;
  const int n = blockIdx.x * 256 + threadIdx.x;              // the grid covers them exactly
  const f64x2* p = reinterpret_cast<const f64x2*>(partial) + bh * n_chunks * (size_t)pairs +
                   Geo<D>::pair_of(n / (D / 2), n % (D / 2) * 2);
  f64x2 acc = {0.0, 0.0};
#pragma unroll 8
  for (int c = 0; c < n_chunks; ++c) acc += p[(size_t)c * pairs];
  reinterpret_cast<f64x2*>(hbar64)[bh * pairs + n] = f64x2{acc[0] / (double)N, acc[1] / (double)N};
}

// ---- lane exchanges on the vector ALU ----
template <int CTRL> __device__ inline double dpp(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Partner lanes inside a row of 16: together these four pairings span the row.
constexpr int kMirror = 0x140, kHalfMirror = 0x141, kXor2 = 0x4e, kXor1 = 0xb1;

// Lanes 32..63 of a change places with lanes 0..31 of b (odd 16-lane rows of a with even rows of b): afterwards
// a + b holds the pair sums of the old a in the lower half (even rows), those of the old b in the upper (odd).
__device__ inline void swap32(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a), y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
  b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ inline void swap16(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a), y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
  b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ inline double sum_rows(double x) {            // over the four lanes that share lane % 16
  double y = x;
  swap16(x, y);
  x += y;
  y = x;
  swap32(x, y);
  return x + y;
}
__device__ inline double sum_in_row(double x) {          // over the 16 lanes of a row
  x += dpp<kMirror>(x);
  x += dpp<kHalfMirror>(x);
  x += dpp<kXor2>(x);
  return x + dpp<kXor1>(x);
}
// One halving step of a transposing sum: of the 2 H values a lane keeps H (the upper ones if `upper`) and adds
// its partner's.
template <int CTRL, int H, int N> __device__ inline void halve(double (&x)[N], bool upper) {
#pragma unroll
  for (int c = 0; c < H; ++c) {
    const double keep = upper ? x[c + H] : x[c], send = upper ? x[c] : x[c + H];
    x[c] = keep + dpp<CTRL>(send);
  }
}

__device__ inline double reciprocal(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(fma(-d, y, 1.0), y, y);
  return fma(fma(-d, y, 1.0), y, y);
}
__device__ inline double reciprocal_sqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * fma(-0.5 * x * y, y, 1.5);
  return y * fma(-0.5 * x * y, y, 1.5);
}
__device__ inline double read_lane(double x, int lane /* uniform */) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double max_over_wave(double x) {
  x = fmax(x, dpp<kMirror>(x));
  x = fmax(x, dpp<kHalfMirror>(x));
  x = fmax(x, dpp<kXor2>(x));
  x = fmax(x, dpp<kXor1>(x));
  double y = x;
  swap16(x, y);
  x = fmax(x, y);
  y = x;
  swap32(x, y);
  return fmax(x, y);
}
// Orders this wave's LDS traffic: writes before it are visible to every lane after it.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Largest eigenpair of the m x m tridiagonal Lanczos matrix T (diagonal alpha, off-diagonal beta), by one wave.
// The eigenvector's recurrence  beta_c s_{c+1} = (lambda - alpha_c) s_c - beta_{c-1} s_{c-1},  s_1 = 1, has no division
// (1 / beta_c is computed beforehand, a lane per row) and s_{m+1}(lambda) is the characteristic polynomial but for a
// constant.
// theta: kept between `lo` and `hi`, a pass looks at 64 points of the interval at once, one a lane.  The lowest of
// them without a sign change along s is still above the spectrum (`above_root`); the next one below is the new lo, and
// Laguerre's step from it (monotone from above, with cubic convergence where the root is simple; first and second
// derivative along the same recurrence) the new hi.  Where rounding carries that step below the root (a dominant
// root: the step is exact, whatever the distance, and lands an ulp to either side), no point of the next pass is above the
// spectrum: the root then lies between hi and `above_root`, and the passes go on in there.
// residual: s satisfies all rows of T - theta above the one it is cut at, so the Krylov vector with the
// coefficients s_1 .. s_c has |A x - theta x|^2 = beta_c^2 (s_c^2 + s_{c+1}^2) / (s_1^2 + .. + s_c^2); the least over
// c is taken (past convergence rounding makes the later entries grow again).
// decay4: how much s shrank over the last four entries in front of that c (squared).
struct RitzPair {
  double theta, residual, decay4;
};
struct RitzRow {
  double alpha, inv_beta, ratio, pad;            // ratio = beta_{c-1} / beta_c
};
__device__ inline RitzPair largest_ritz_pair(const double* alpha, const double* beta2, RitzRow* rows, int m,
                                             double lo, double hi) {
  const int lane = threadIdx.x & 63;
  double bound = 0.0;
  for (int c = lane; c < m; c += 64) {
    // beta = 0 (the last one, an exact end of the Krylov space): s_{m+1} is a multiple of the polynomial with any factor
    const double inv = beta2[c] > 0.0 ? reciprocal_sqrt(beta2[c]) : 1.0, b = beta2[c] * inv;
    const double a = c > 0 ? beta2[c - 1] * reciprocal_sqrt(beta2[c - 1]) : 0.0;
    rows[c].alpha = alpha[c];
    rows[c].inv_beta = inv;
    rows[c].ratio = a * inv;
    bound = fmax(bound, alpha[c] + a + (c + 1 < m ? b : 0.0));      // Gershgorin
  }
  bound = max_over_wave(bound) * 1.001;
  wave_lds_sync();
  if (!(hi < bound)) hi = bound;                 // no estimate given, or no better one
  const double n = (double)m;
  double above_root = INFINITY;                  // lowest point known to be above the spectrum
  for (int it = 0; it < 100; ++it) {
    const double lam = hi - (hi - lo) * (0.015625 * (double)lane);
    double s0 = 0.0, s1 = 1.0, p0 = 0.0, p1 = 0.0, q0 = 0.0, q1 = 0.0;     // s, s', s'' of the last two rows
    bool above = true;
    RitzRow next = rows[0];
#pragma unroll 4
    for (int c = 0; c < m; ++c) {
      const RitzRow row = next;
      next = rows[c + 1];                        // one row past the end is read, and not used
      const double a = (lam - row.alpha) * row.inv_beta;
      const double s2 = fma(a, s1, -row.ratio * s0);
      const double p2 = fma(a, p1, fma(row.inv_beta, s1, -row.ratio * p0));
      const double q2 = fma(a, q1, fma(2.0 * row.inv_beta, p1, -row.ratio * q0));
      above = above && s2 > 0.0;
      s0 = s1; s1 = s2;
      p0 = p1; p1 = p2;
      q0 = q1; q1 = q2;
    }
    const unsigned long long not_above = ~__ballot(above);
    const int n_above = not_above ? __builtin_ctzll(not_above) : 64;       // lanes 0 .. n_above - 1
    if (n_above == 0) {
      if (above_root < INFINITY) {               // Laguerre's step fell below the root by rounding
        lo = fmax(lo, hi);
        hi = above_root;
        if (hi - lo < 1e-15 * hi) break;
        continue;
      }
      if (hi < bound) {                          // the estimate handed in was no upper bound
        hi = bound;
        continue;
      }
      break;                                     // no point above the spectrum at all: not a number, or a zero matrix
    }
    const double inv = reciprocal(s1), g = p1 * inv, h = fma(g, g, -q1 * inv);
    const double disc = fmax(1e-300, (n - 1.0) * fma(n, h, -g * g));
    const double my_step = n * reciprocal(fma(disc, reciprocal_sqrt(disc), g));
    const double from = read_lane(lam, n_above - 1), step = read_lane(my_step, n_above - 1);
    // how far the other roots are: 0: the root alone; 1: as if it were double
    const double crowd = read_lane(g * g * reciprocal(h), n_above - 1) - 1.0;
    if (n_above < 64) lo = fmax(lo, read_lane(lam, n_above));
    above_root = from;
    if (!(step > 0.0)) {
      hi = from;
      break;
    }
    hi = fmax(lo, from - step);
    // the distance left after a Laguerre step is about step * crowd^2
    if (step * crowd * crowd < 1e-15 * hi || hi - lo < 1e-15 * hi) break;
  }
  const double lam = hi;
  double s0 = 0.0, s1 = 1.0, sum = 0.0, best = 1.0, best_sum = 0.0, decay = 1.0;
  double back[4] = {1.0, 1.0, 1.0, 1.0};         // squared entries before s_c
  RitzRow next = rows[0];
  double next_b2 = beta2[0];
#pragma unroll 4
  for (int c = 0; c < m; ++c) {
    const RitzRow row = next;
    const double b2 = next_b2;
    next = rows[c + 1];
    next_b2 = beta2[c + 1];
    const double s2 = fma((lam - row.alpha) * row.inv_beta, s1, -row.ratio * s0), sq = s1 * s1;
    sum += sq;
    const double res = b2 * fma(s2, s2, sq);
    if (c == 0 || res * best_sum < best * sum) { // res / sum < best / best_sum
      best = res;
      best_sum = sum;
      decay = sq * reciprocal(back[0]);
    }
    back[0] = back[1];
    back[1] = back[2];
    back[2] = back[3];
    back[3] = sq;
    s0 = s1;
    s1 = s2;
  }
  return RitzPair{lam, sqrt(best / best_sum), decay};
}

// (2) One workgroup per block.  Spectral norm: Golub-Kahan-Lanczos written as Lanczos on A = D^T D,
//   y = D v,  alpha = |y|^2,  w = D^T y - alpha v - beta v_prev,  beta = |w|,  v_next = w / beta,
// from a fixed start vector until the residual of the largest Ritz pair is below kRelResidual of its value.
// A wave owns rows of D, so the y it needs for its part of D^T y are its own: the only exchange between waves is
// the sum of the four partial D^T y (one barrier a step; every wave then holds all of w, two entries a lane, and
// does the vector work redundantly).  The sums over lanes are transposing ones: in a row of 16 lanes by DPP, over
// the rows by lane swaps.  No reorthogonalisation: the largest Ritz value does not need it.
// 24 x 72 blocks of 64 x 128, bf16: 1 309 us with a three-term eigenvalue iteration behind 16 barriers a step and a
// 3 x 3 eigenproblem in every thread; 224 us now, of which the fp64 products of the rebuild take about 80 and
// 19.5 Lanczos steps a block (400 vector instructions a wave each, issue-bound with two workgroups on a CU) and
// 1.5 looks the rest.
// The Ritz pair is looked at by one wave after kFirstLook steps and then when its decay says it should be there.
constexpr int kFirstLook = 20;
template <typename T, int D, bool SPECTRAL>
__global__ __launch_bounds__(256, 2) void hetero_kernel(const T* __restrict__ k, const T* __restrict__ v,
                                                     const double* __restrict__ kbar64,
                                                     const double* __restrict__ hbar64,
                                                     double* __restrict__ log_m, int L, int B, int N,
                                                     int max_steps, double eps) {
  constexpr int TA = Geo<D>::TA, TB = Geo<D>::TB, NY = Geo<D>::NY, NQ = Geo<D>::NQ;
  // the staging area of the rebuild and the scratch of the iteration share their memory
  constexpr int kMaxRows = kSpectralMaxSteps + 1;          // (one row past the end is read)
  union Scratch {
    struct {
      T ks[kRows][D], vs[kRows][D];
    } in;
    struct {
      double zpart[2][4][D];                     // partial D^T y by step parity and wave
      double ysum[4][4 * NY];                    // wave-private: y by lane row
      RitzRow ritz[kMaxRows];
      double alpha[kMaxRows], beta2[kMaxRows];
    } it;
  };
  __shared__ __attribute__((aligned(16))) Scratch sh;
  __shared__ double apart[2][4];
  __shared__ double theta_s;
  __shared__ int look_s;                         // next step to look at the Ritz pair, 0: done
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, kk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = blockIdx.x;
  const size_t bh = blockIdx.y;
  const T* kh = k + bh * (size_t)L * D;
  const T* vh = v + bh * (size_t)L * D;
  const int first = j * B, last = min(L, first + B);
  Staged<T, D> st;
  load_rows(st, kh, vh, first, min(kRows, last - first));
  double mean[TA];
  load_means<D>(mean, kbar64 + (bh * N + j) * D);
  f64x4 acc[TA][TB];
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f64x2* row = reinterpret_cast<const f64x2*>(
          hbar64 + bh * (size_t)D * D + (size_t)((D / 4) * wave + TA * (4 * e + kk) + a) * D + TB * i);
#pragma unroll
      for (int b = 0; b < TB; b += 2) {
        const f64x2 hb = row[b / 2];
        acc[a][b][e] = -hb[0];
        acc[a][b + 1][e] = -hb[1];
      }
    }
  for (int row0 = first; row0 < last; row0 += kRows) {
    __syncthreads();
    store_rows(st, sh.in.ks, sh.in.vs);
    __syncthreads();
    if (row0 + kRows < last) load_rows(st, kh, vh, row0 + kRows, min(kRows, last - row0 - kRows));
    add_products<T, D>(acc, sh.in.ks, sh.in.vs, mean, min(kRows, last - row0));
  }

  if (!SPECTRAL) {
    double ss = 0.0;
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) ss = fma(acc[a][b][e], acc[a][b][e], ss);
    ss = sum_rows(sum_in_row(ss));
    if (lane == 0) apart[0][wave] = ss;
    __syncthreads();
    if (tid == 0) log_m[bh * N + j] = log(sqrt((apart[0][0] + apart[0][1]) + (apart[0][2] + apart[0][3])) + eps);
    return;
  }

  __syncthreads();                               // the staging area is used up
  // Vectors of value channels: spread over a wave (entries NQ (4 i + kk) + u of lane (i, kk)): vq, vq_prev; and in
  // full as the lane's columns TB i + b: vc.
  double vq[NQ], vq_prev[NQ], vc[TB];
  auto spread_to_columns = [&]() {
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      double e0 = vq[u], e1 = vq[u];
      swap16(e0, e1);                            // lane rows 0, 1 (2, 3)
      double e2 = e0, e3 = e1;
      swap32(e0, e2);                            // e0: row 0, e2: row 2
      swap32(e1, e3);
      vc[u] = e0;
      vc[NQ + u] = e1;
      vc[2 * NQ + u] = e2;
      vc[3 * NQ + u] = e3;
    }
  };
  auto norm2 = [&](const double (&x)[NQ]) {
    double n2 = 0.0;
#pragma unroll
    for (int u = 0; u < NQ; ++u) n2 = fma(x[u], x[u], n2);
    return sum_rows(sum_in_row(n2));
  };
#pragma unroll
  for (int u = 0; u < NQ; ++u) {                 // fixed, generic start
    vq[u] = 1.0 + 0.5 * sin(1.0 + 0.37 * (double)(NQ * (4 * i + kk) + u));
    vq_prev[u] = 0.0;
  }
  {
    const double inv = 1.0 / sqrt(norm2(vq));
#pragma unroll
    for (int u = 0; u < NQ; ++u) vq[u] *= inv;
  }
  double beta = 0.0, alpha_max = 0.0;
  int look = min(kFirstLook, max_steps);
  double theta_below = 0.0, theta_above = INFINITY;   // wave 0: where theta lies, from the last look (Ritz values only grow)
  for (int m = 1;; ++m) {
    const int par = m & 1;
    spread_to_columns();
    double y[NY];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double s0 = 0.0;
#pragma unroll
        for (int b = 0; b < TB; ++b) s0 = fma(acc[a][b][e], vc[b], s0);
        y[4 * a + e] = s0;
      }
    // sum over the 16 lanes of a row, value (side bits) left in each lane
    if constexpr (NY == 8) {
      halve<kMirror, 4>(y, (i & 8) != 0);
      halve<kHalfMirror, 2>(y, (i & 4) != 0);
      halve<kXor2, 1>(y, (i & 2) != 0);
      y[0] += dpp<kXor1>(y[0]);
      sh.it.ysum[wave][NY * kk + (i >> 1)] = y[0];     // lanes 2 c, 2 c + 1 hold the same value
    } else {
      halve<kMirror, 2>(y, (i & 8) != 0);
      halve<kHalfMirror, 1>(y, (i & 4) != 0);
      y[0] += dpp<kXor2>(y[0]);
      y[0] += dpp<kXor1>(y[0]);
      sh.it.ysum[wave][NY * kk + (i >> 2)] = y[0];
    }
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < NY; c += 2) {
      const f64x2 x = *reinterpret_cast<const f64x2*>(&sh.it.ysum[wave][NY * kk + c]);
      y[c] = x[0];
      y[c + 1] = x[1];
    }
    double a_mine = 0.0;
#pragma unroll
    for (int c = 0; c < NY; ++c) a_mine = fma(y[c], y[c], a_mine);
    a_mine = sum_rows(a_mine);
    double z[TB];
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      double s0 = 0.0;
#pragma unroll
      for (int c = 0; c < NY; ++c) s0 = fma(acc[c / 4][b][c % 4], y[c], s0);
      z[b] = s0;
    }
#pragma unroll
    for (int b = 0; b < TB / 2; ++b) {           // sum over the lane rows: halves, then quarters
      swap32(z[b], z[b + TB / 2]);
      z[b] += z[b + TB / 2];
    }
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
      swap16(z[b], z[b + NQ]);
      z[b] += z[b + NQ];
      sh.it.zpart[par][wave][NQ * (4 * i + kk) + b] = z[b];
    }
    if (lane == 0) apart[par][wave] = a_mine;
    __syncthreads();
    const double alpha = (apart[par][0] + apart[par][1]) + (apart[par][2] + apart[par][3]);
    double w[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const int o = NQ * (4 * i + kk) + u;
      w[u] = (sh.it.zpart[par][0][o] + sh.it.zpart[par][1][o]) + (sh.it.zpart[par][2][o] + sh.it.zpart[par][3][o]);
      w[u] -= fma(alpha, vq[u], beta * vq_prev[u]);
    }
    const double b2 = norm2(w);
    alpha_max = fmax(alpha_max, alpha);
    if (wave == 0 && lane == 0) {
      sh.it.alpha[m - 1] = alpha;
      sh.it.beta2[m - 1] = b2;
    }
    // |w| alone bounds the residual: below the bar the Krylov space is exhausted (ends on D = 0 and on NaN too)
    const double bar = kRelResidual * alpha_max;
    const bool exhausted = !(b2 > bar * bar);
    if (exhausted || m == look) {
      if (wave == 0) {
        wave_lds_sync();
        const RitzPair p = largest_ritz_pair(sh.it.alpha, sh.it.beta2, sh.it.ritz, m, theta_below, theta_above);
        theta_below = fmax(0.0, p.theta * (1.0 - 1e-14));
        theta_above = p.theta + p.residual;
        if (lane == 0) {
          theta_s = p.theta;
          int next = 0;
          if (!exhausted && m < max_steps && p.residual > kRelResidual * p.theta) {
            // steps still missing at the rate at which the Ritz vector decayed (1 .. 8)
            const float rate = 0.125f * __builtin_amdgcn_logf((float)p.decay4);        // log2 per step
            const float gap = __builtin_amdgcn_logf((float)(kRelResidual * p.theta / p.residual));
            const float steps = rate < -0.05f ? ceilf(gap / rate) : 8.f;
            next = min(max_steps, m + max(1, min(8, (int)steps)));
          }
          look_s = next;
        }
      }
      __syncthreads();
      look = look_s;
      if (look == 0) break;                      // look_s is written again only after the next barrier
    }
    const double r = reciprocal_sqrt(b2);
    beta = b2 * r;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      vq_prev[u] = vq[u];
      vq[u] = w[u] * r;
    }
  }
  if (tid == 0) log_m[bh * N + j] = log((theta_s > 0.0 ? sqrt(theta_s) : theta_s == theta_s ? 0.0 : theta_s) + eps);
}

}  // namespace

size_t hetero_workspace_bytes(const Dims& dm) {
  const StatsPlan plan = matrix_bound_plan(dm);
  return (size_t)dm.bh() * (plan.n_chunks + 1) * dm.d * dm.d * sizeof(double);
}

hipError_t launch_block_heterogeneity(const Dims& dm, const void* k, const void* v, const double* kbar64,
                                      const float* hsum, int spectral, int n_iter, double eps, double* log_m,
                                      double* workspace, hipStream_t stream) {
  const StatsPlan plan = matrix_bound_plan(dm);
  const int dd = dm.d * dm.d;
  double* partial = workspace;
  double* hbar = workspace + (size_t)dm.bh() * plan.n_chunks * dd;
  const dim3 g1(plan.n_chunks, dm.bh()), g2(dd / 512, dm.bh()), g3(dm.N, dm.bh());
#define PISA_HET(T, DD)                                                                                \
  do {                                                                                                  \
    if (hsum) {                                                                                         \
      const size_t total = (size_t)dm.bh() * dd;                                                        \
      hipLaunchKernelGGL(hbar_from_hsum_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, \
                         hsum, hbar, total, dm.N);                                                      \
    } else {                                                                                            \
      hipLaunchKernelGGL((hsum64_kernel<T, DD>), g1, dim3(256), 0, stream, (const T*)k, (const T*)v,    \
                         kbar64, partial, dm.L, dm.B, dm.N, plan.chunk_blocks, plan.n_chunks);          \
      hipLaunchKernelGGL(hbar64_kernel<DD>, g2, dim3(256), 0, stream, partial, hbar, plan.n_chunks, dm.N); \
    }                                                                                                   \
    if (spectral)                                                                                       \
      hipLaunchKernelGGL((hetero_kernel<T, DD, true>), g3, dim3(256), 0, stream, (const T*)k, (const T*)v, \
                         kbar64, hbar, log_m, dm.L, dm.B, dm.N, n_iter, eps);                           \
    else                                                                                                \
      hipLaunchKernelGGL((hetero_kernel<T, DD, false>), g3, dim3(256), 0, stream, (const T*)k, (const T*)v, \
                         kbar64, hbar, log_m, dm.L, dm.B, dm.N, n_iter, eps);                           \
  } while (0)
  if (dm.dtype == PISA_BF16 && dm.d == 64)
    PISA_HET(__hip_bfloat16, 64);
  else if (dm.dtype == PISA_BF16)
    PISA_HET(__hip_bfloat16, 128);
  else if (dm.d == 64)
    PISA_HET(float, 64);
  else
    PISA_HET(float, 128);
#undef PISA_HET
  return hipGetLastError();
}

}  // namespace pisa
