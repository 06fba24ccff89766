// pisa_block_stats for bf16 inputs, head_dim 128 or 64, block 64 or 128: one streaming pass
// (Alg. 1, "Prepare" step).  Written out for head_dim 128; the differences at 64 are noted where they occur.
//
// Grid (n_chunks, batch*heads); a workgroup of 8 waves walks `chunk_blocks` consecutive
// blocks of one head.  Per 64-token (sub-)block:
//   * wave w loads rows 8w..8w+7 of the Q, K and V tiles, one 4-byte channel pair per
//     lane (a wave-load is one 256-byte row), one sub-block ahead of their use, and adds
//     them in fp64 (exact for bf16 data);
//     the waves' partial column sums meet in LDS and are added in wave order;
//   * K is centred on the block mean in registers, split into bf16 hi + lo parts and
//     written to LDS together with V (rows swizzled for conflict-free transposed reads);
//   * H += Kc^T V on the matrix cores: wave w owns 32 key channels and 64 value
//     channels (two 32x32 accumulators); both operands are contracted over
//     tokens, so both come from ds_read_b64_tr_b16.
// The partial H of the chunk goes to scratch; partials are added in chunk order by the
// caller's reduction kernel, so hsum is run-to-run identical.
#include "common.h"

namespace pisa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
#define LDS_PTR(T) __attribute__((address_space(3))) T*


__device__ inline unsigned int pack_bf16(float lo, float hi) {
  f32x2 f = {lo, hi};
  bf16x2 b = __builtin_convertvector(f, bf16x2);
  return __builtin_bit_cast(unsigned int, b);
}

// Swizzle of a staged [token][channel] tile: the 32-byte chunk index of row n is XORed with
// this value, which makes the transposed reads below bank-conflict free (256-byte rows: a
// 3-bit pattern; 128-byte rows, two to a bank line: bit 1 flipped for every other row pair).
template <int D> __device__ inline int swz3(int n) {
  return D == 128 ? (((n & 3) << 1) | ((n >> 2) & 1)) : (((n >> 1) & 1) << 1);
}

// Byte address of channel pair `c2` (channels 2 c2, 2 c2 + 1) of row n in a swizzled tile.
template <int D> __device__ inline int swz_pair(int n, int c2) {
  const int byte = c2 * 4;
  return n * (2 * D) + ((((byte >> 5) ^ swz3<D>(n)) << 5) | (byte & 31));
}

// A / B operand of v_mfma_f32_32x32x16_bf16 for contraction step `step` (16 tokens) and
// channel tile `ct` (32 channels), read transposed from a swizzled [token][channel] tile.
template <int D>
__device__ inline bf16x8 read_operand(LDS_PTR(const unsigned char) tile, int lane, int step, int ct) {
  constexpr int ROWB = 2 * D;
  const int j16 = lane & 15, h = lane >> 5, lhalf = (lane >> 4) & 1;
  const int kq = 4 * h + (j16 >> 2);
  const int off = (16 * step + kq) * ROWB + 8 * (j16 & 3) + (((2 * ct + lhalf) ^ swz3<D>(kq)) << 5);
  LDS_PTR(unsigned char) p = const_cast<LDS_PTR(unsigned char)>(tile) + off;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_PTR(s16x4)>(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_PTR(s16x4)>(p + 8 * ROWB));
  const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
  const u32x4 w = {l2.x, l2.y, h2.x, h2.y};
  return __builtin_bit_cast(bf16x8, w);
}

// TPB = tiles (64-token sub-blocks) per block: 1 for block 64, 2 for block 128.  With two
// sub-blocks each is centred on its OWN mean c_s for the matrix-core contraction, and the
// block's H_j follows from  sum_n (k_n - c_s)^T v_n = sum_n (k_n - kbar_j)^T v_n + (kbar_j - c_s)^T Vhat_s :
//   H_j = sum_s [ A_s + (c_s - kbar_j)^T Vhat_s ],
// a small rank-one correction per sub-block (c_s is close to kbar_j, so nothing cancels).
// Head_dim 64: four waves, a 256-byte wave-load is two rows (lane = row parity x channel pair), a
// lane holds 8 rows per tensor, the two row parities are added with one lane
// exchange, and the 64 x 64 matrix H is four 32 x 32 tiles, one per wave.
//
// HETERO: the same walk used for the covariance-aware score instead of the statistics: every
// block's H_j is rebuilt exactly as above (same centring, same hi/lo split, same products, so
// the same bits that went into hsum), kept per block instead of summed over the chunk, and
// reduced to log(||H_j - hsum / N||_F + eps); nothing else is written and Q is not read.
//
// Waves per workgroup.  The launch is bound by memory (input rows, and the partial H it writes), but
// with four waves at two workgroups per CU a SIMD had two waves for a chain of three barriers, 190 fp64
// instructions and 32 MFMAs per 64 rows, and 39 % of their time went into waiting.  At head_dim 128 eight
// waves halve the chain (2 heads of 1 000 tokens 9.2 -> 7.3 us, 24 heads of 4 608 31.3 -> 28.8 us,
// 40 heads of 75 600 598 -> 571 us = 4.1 TB/s); at 64 a wave has half the rows and an eighth of the MFMAs,
// and there are only four 32 x 32 tiles of H to hand out: four waves.
constexpr int stats_waves(int d) { return d == 128 ? 8 : 4; }
constexpr int kNormBlocks = 8;      // (head_dim 128, block 128: two workgroups fill the LDS to the byte)

// Sum over the wave by lane permutations on the vector ALU.
template <int CTRL> __device__ inline double add_dpp(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
  return x + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double wave_sum(double x) {
  x = add_dpp<0xb1>(x);              // lane ^ 1
  x = add_dpp<0x4e>(x);              // lane ^ 2
  x = add_dpp<0x141>(x);             // mirrored inside 8 lanes
  x = add_dpp<0x140>(x);             // mirrored inside 16 lanes: every lane has its row's sum
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

template <int D, int TPB, bool HETERO>
__global__ __launch_bounds__(64 * stats_waves(D), D == 128 ? 4 : 2) void stats_bf16_kernel(
    const unsigned int* __restrict__ q, const unsigned int* __restrict__ k, const unsigned int* __restrict__ v,
    float* __restrict__ qbar, float* __restrict__ kbar, float* __restrict__ vsum,
    double* __restrict__ qbar64, double* __restrict__ kbar64, float* __restrict__ partial_h,
    unsigned short* __restrict__ kcen, unsigned short* __restrict__ vbar, int npad,
    int L, int N, int chunk_blocks, int n_chunks,
    const float* __restrict__ hsum, double eps, double* __restrict__ log_m) {
  constexpr int B = TPB * kTile;
  constexpr int TILEB = kTile * 2 * D;
  constexpr int LPR = D / 2;            // lanes per row (one channel pair each)
  constexpr int RPW = 64 / LPR;         // rows per wave-load
  constexpr int NW = stats_waves(D);
  constexpr int RW = kTile / NW;        // rows per wave
  constexpr int NR = RW / RPW;          // loads per lane and tensor
  constexpr int NB = D / 32 / 2;        // value tiles per wave: 2, or 1
  __shared__ __attribute__((aligned(1024))) unsigned char khi_s[TILEB];
  __shared__ __attribute__((aligned(1024))) unsigned char klo_s[TILEB];
  __shared__ __attribute__((aligned(1024))) unsigned char v_s[TILEB];
  __shared__ __attribute__((aligned(16))) double red[3][NW][D];
  __shared__ double tot[3][D];          // block totals over the sub-blocks (q, k, v)
  __shared__ double csub[2][D];         // sub-block key means c_s
  __shared__ float vsub[2][D];          // sub-block value sums Vhat_s
  __shared__ float dks[2][D];           // c_s - kbar_j
  __shared__ float kmean_s[D];
  __shared__ double hnorm_s[HETERO ? kNormBlocks : 1][NW];         // HETERO: per-wave sums of squares

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: row addresses stay scalar
  const int chunk = blockIdx.x;
  const size_t bh = blockIdx.y;
  const size_t head_words = (size_t)L * (D / 2);
  const unsigned int* qh = q + bh * head_words;
  const unsigned int* kh = k + bh * head_words;
  const unsigned int* vh = v + bh * head_words;
  LDS_PTR(unsigned char) khi = (LDS_PTR(unsigned char))khi_s;
  LDS_PTR(unsigned char) klo = (LDS_PTR(unsigned char))klo_s;
  LDS_PTR(unsigned char) vt = (LDS_PTR(unsigned char))v_s;
  const int lam = lane & 31, h = lane >> 5;
  const int rp = lane / LPR, cp = lane % LPR;        // row parity inside a wave-load, channel pair
  const int ktile = wave & (D / 32 - 1);             // this wave's 32 key channels of H
  const int vtile0 = NB * (wave / (D / 32));         // its first 32-value-channel tile
  const int grp = tid / D, ch = tid % D;             // block sums: tensor (0 q, 1 k, 2 v; 3 idle) and channel

  f32x16 acc[NB];
#pragma unroll
  for (int bt = 0; bt < NB; ++bt) acc[bt] = (f32x16){0};

  // HETERO: 1 / N, and the elements of this head's hsum at this lane's accumulator positions (see the store at the end).
  // Kept in registers; read per block from L2 (16 at a time) only at head_dim 128 with two sub-blocks, where they do not fit
  // (40 heads of 20 000 tokens 163 us with every block reading them, 135 kept).
  constexpr bool KEEP_HSUM = !(D == 128 && TPB == 2);
  const float inv_n = 1.f / (float)N;
  const float* hs_head = HETERO ? hsum + bh * (size_t)D * D : nullptr;
  float hb[HETERO && KEEP_HSUM ? NB : 1][16];
  auto load_hsum = [&](const float* hp, unsigned off, int bt, float (&x)[16]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = (hp + (32 * ktile + (r / 4) * 8 + (r % 4)) * D + 32 * (vtile0 + bt))[off];
  };
  if (HETERO && KEEP_HSUM)
#pragma unroll
    for (int bt = 0; bt < NB; ++bt) load_hsum(hs_head, 4 * h * D + lam, bt, hb[bt]);

  // Optional second form of the block outputs, for the attention kernel's centroid phase: the
  // key mean and the value mean of block j as bf16 rows of tiles [bh][npad][D] (the fp32
  // values just written, rounded to nearest even; rows N .. npad - 1 are zero).  Called by
  // the threads of the k group and of the v group, each for its own tensor.
  auto centroid_row = [&](unsigned short* dst, int j, float mean) {
    if (!dst) return;
    dst[(bh * (size_t)npad + j) * D + ch] = (unsigned short)pack_bf16(mean, 0.f);
    if (j == N - 1)
      for (int jj = N; jj < npad; ++jj) dst[(bh * (size_t)npad + jj) * D + ch] = 0;
  };

  // This wave's RW rows of one 64-token sub-block, one channel pair per lane.  Rows past the
  // end repeat the last valid row (the users mask them), so the loads carry no conditions.
  auto load_rows = [&](const unsigned int* src, int row0, int rows, unsigned int (&x)[NR]) {
    if (rows <= 0) return;
#pragma unroll
    for (int i = 0; i < NR; ++i)
      x[i] = src[(size_t)(row0 + min(RW * wave + RPW * i + rp, rows - 1)) * (D / 2) + cp];
  };

  const int j_begin = chunk * chunk_blocks;
  const int j_end = min(N, j_begin + chunk_blocks);
  // The rows of sub-block t + 1 are requested while sub-block t is worked on (K and V at its
  // start into a second register set, Q into its own registers once its sums are taken), so a
  // wave always has 4 to 6 KB of loads in flight (8 waves; twice that with four).
  unsigned int kx[NR] = {}, vx[NR] = {}, qx[NR] = {}, kn[NR] = {}, vn[NR] = {};
  if (j_begin < j_end) {
    const int rows = min(kTile, L - j_begin * B);
    if (!HETERO) load_rows(qh, j_begin * B, rows, qx);
    load_rows(kh, j_begin * B, rows, kx);
    load_rows(vh, j_begin * B, rows, vx);
  }
  for (int j = j_begin; j < j_end; ++j) {
    const int block_rows = min(B, L - j * B);
    int n_sub = 0;
    for (int sub = 0; sub < TPB; ++sub) {
      const int row0 = j * B + sub * kTile;
      const int rows = min(kTile, L - row0);
      if (rows <= 0) break;                       // uniform: the block ends inside its first half
      n_sub = sub + 1;
      // Head_dim 128: LDS addresses are made again per sub-block from this copy; hoisted, they cost more
      // registers than eight waves a workgroup leave.
      int ln = lane;
      if (D == 128) asm volatile("" : "+v"(ln));
      const int cpn = ln % LPR, rpn = ln / LPR;
      int next_row0, next_rows;
      {
        int nj = j, ns = sub + 1;
        if (ns == TPB || j * B + ns * kTile >= L) {
          nj = j + 1;
          ns = 0;
        }
        next_row0 = nj * B + ns * kTile;
        next_rows = nj < j_end ? min(kTile, L - next_row0) : 0;
        load_rows(kh, next_row0, next_rows, kn);
        load_rows(vh, next_row0, next_rows, vn);
      }
      // ---- fp64 column sums of the wave's rows (absent rows are zeroed first) ----
      double sq0 = 0, sq1 = 0, sk0 = 0, sk1 = 0, sv0 = 0, sv1 = 0;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        if (RW * wave + RPW * i + rp >= rows) {   // uniform at head_dim 128
          qx[i] = kx[i] = vx[i] = 0u;
        }
        sq0 += (double)__uint_as_float(qx[i] << 16);
        sq1 += (double)__uint_as_float(qx[i] & 0xffff0000u);
        sk0 += (double)__uint_as_float(kx[i] << 16);
        sk1 += (double)__uint_as_float(kx[i] & 0xffff0000u);
        sv0 += (double)__uint_as_float(vx[i] << 16);
        sv1 += (double)__uint_as_float(vx[i] & 0xffff0000u);
      }
      if (RPW == 2) {                             // the other row parity of the same channels
        sq0 += __shfl_xor(sq0, 32); sq1 += __shfl_xor(sq1, 32);
        sk0 += __shfl_xor(sk0, 32); sk1 += __shfl_xor(sk1, 32);
        sv0 += __shfl_xor(sv0, 32); sv1 += __shfl_xor(sv1, 32);
      }
      if (lane < LPR) {
        *reinterpret_cast<f64x2*>(&red[0][wave][2 * cp]) = (f64x2){sq0, sq1};
        *reinterpret_cast<f64x2*>(&red[1][wave][2 * cp]) = (f64x2){sk0, sk1};
        *reinterpret_cast<f64x2*>(&red[2][wave][2 * cp]) = (f64x2){sv0, sv1};
      }
      if (!HETERO) load_rows(qh, next_row0, next_rows, qx);    // Q(t) is used up
      __syncthreads();
      if (grp < 3) {
        double sum = red[grp][0][ch];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += red[grp][w][ch];
        const double mean = sum / (double)rows;
        if (TPB == 1) {
          if (!HETERO) {
            const size_t o = (bh * N + j) * D + ch;
            if (grp == 0) {
              qbar[o] = (float)mean;
              if (qbar64) qbar64[o] = mean;
            } else if (grp == 1) {
              kbar[o] = (float)mean;
              if (kbar64) kbar64[o] = mean;
              centroid_row(kcen, j, (float)mean);
            } else {
              vsum[o] = (float)sum;
              centroid_row(vbar, j, (float)sum * (1.f / (float)rows));
            }
          }
        } else {
          tot[grp][ch] = sub == 0 ? sum : tot[grp][ch] + sum;
          if (grp == 1) csub[sub][ch] = mean;
          if (grp == 2) vsub[sub][ch] = (float)sum;
        }
        if (grp == 1) kmean_s[ch] = (float)mean;
      }
      __syncthreads();
      // ---- centre K on the sub-block mean, split hi/lo, stage with V ----
      {
        const float m0 = kmean_s[2 * cpn], m1 = kmean_s[2 * cpn + 1];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          const int n = RW * wave + RPW * i + rpn;
          unsigned int hi = 0u, lo = 0u;
          if (n < rows) {
            const float c0 = __uint_as_float(kx[i] << 16) - m0;
            const float c1 = __uint_as_float(kx[i] & 0xffff0000u) - m1;
            hi = pack_bf16(c0, c1);
            lo = pack_bf16(c0 - __uint_as_float(hi << 16), c1 - __uint_as_float(hi & 0xffff0000u));
          }
          const int a = swz_pair<D>(n, cpn);
          *reinterpret_cast<LDS_PTR(unsigned int)>(khi + a) = hi;
          *reinterpret_cast<LDS_PTR(unsigned int)>(klo + a) = lo;
          *reinterpret_cast<LDS_PTR(unsigned int)>(vt + a) = vx[i];
        }
      }
      __syncthreads();
      // ---- H[32 ktile .. +32][this wave's value tiles] += Kc^T V over the 64 tokens ----
#pragma unroll
      for (int step = 0; step < 4; ++step) {
        const bf16x8 ahi = read_operand<D>(khi, ln, step, ktile);
        const bf16x8 alo = read_operand<D>(klo, ln, step, ktile);
#pragma unroll
        for (int bt = 0; bt < NB; ++bt) {
          const bf16x8 b = read_operand<D>(vt, ln, step, vtile0 + bt);
          acc[bt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, b, acc[bt], 0, 0, 0);
          acc[bt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, b, acc[bt], 0, 0, 0);
        }
      }
      // the next sub-block's LDS writes are separated from these reads by its two barriers
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        kx[i] = kn[i];
        vx[i] = vn[i];
      }
    }
    if (TPB == 2) {
      // ---- block outputs from the sub-block totals, then the rank-one corrections ----
      if (grp < 3) {
        const double sum = tot[grp][ch], mean = sum / (double)block_rows;
        if (!HETERO) {
          const size_t o = (bh * N + j) * D + ch;
          if (grp == 0) {
            qbar[o] = (float)mean;
            if (qbar64) qbar64[o] = mean;
          } else if (grp == 1) {
            kbar[o] = (float)mean;
            if (kbar64) kbar64[o] = mean;
            centroid_row(kcen, j, (float)mean);
          } else {
            vsum[o] = (float)sum;
            centroid_row(vbar, j, (float)sum * (1.f / (float)block_rows));
          }
        }
        if (grp == 1)
          for (int sub = 0; sub < n_sub; ++sub) dks[sub][ch] = (float)(csub[sub][ch] - mean);
      }
      __syncthreads();
      for (int sub = 0; sub < n_sub; ++sub) {
#pragma unroll
        for (int bt = 0; bt < NB; ++bt) {
          const float vb = vsub[sub][32 * (vtile0 + bt) + lam];
#pragma unroll
          for (int r = 0; r < 16; ++r)
            acc[bt][r] = fmaf(dks[sub][32 * ktile + (r / 4) * 8 + 4 * h + (r % 4)], vb, acc[bt][r]);
        }
      }
      __syncthreads();                            // dks / vsub / tot are rewritten by the next block
    }
    if (HETERO) {
      // acc holds H_j
      double ss = 0.0;
      const float* hp = hs_head;
      unsigned hoff = 4 * h * D + lam;
      if (!KEEP_HSUM) {             // the loads and their addresses stay inside the block loop (hoisted, they spill)
        asm volatile("" : "+s"(hp));
        asm volatile("" : "+v"(hoff));
      }
#pragma unroll
      for (int bt = 0; bt < NB; ++bt) {
        float (&hx)[16] = hb[KEEP_HSUM ? bt : 0];
        if (!KEEP_HSUM) load_hsum(hp, hoff, bt, hx);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const double dlt = (double)fmaf(-hx[r], inv_n, acc[bt][r]);   // both terms carry fp32 rounding already
          ss = fma(dlt, dlt, ss);
          acc[bt][r] = 0.f;
        }
      }
      ss = wave_sum(ss);
      // The norms are finished kNormBlocks at a time, a thread per block.  (What goes by the thread is made here: kept over the
      // block, it spills, but for the one kernel that has registers to spare.)
      int t = tid;
      if (!(D == 64 && TPB == 2)) asm volatile("" : "+v"(t));
      const int at = __builtin_amdgcn_readfirstlane((j - j_begin) % kNormBlocks);
      if (t % 64 == 0) hnorm_s[at][wave] = ss;
      if (at == kNormBlocks - 1 || j == j_end - 1) {
        __syncthreads();
        if (t <= at) {
          double sum = hnorm_s[t][0];
#pragma unroll
          for (int w = 1; w < NW; ++w) sum += hnorm_s[t][w];
          log_m[bh * N + j - at + t] = log(sqrt(sum) + eps);
        }
        // hnorm_s is written again only after the next block's barriers
      }
    }
  }
  if (HETERO) return;
  // acc[bt][r] = H[32 ktile + (r/4)*8 + 4h + r%4][32 (vtile0 + bt) + lam]
  float* ph = partial_h + (bh * n_chunks + chunk) * (size_t)D * D;
#pragma unroll
  for (int bt = 0; bt < NB; ++bt)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      ph[(size_t)(32 * ktile + (r / 4) * 8 + 4 * h + (r % 4)) * D + 32 * (vtile0 + bt) + lam] = acc[bt][r];
}

}  // namespace

hipError_t launch_block_stats_bf16(const Dims& dm, const void* q, const void* k, const void* v,
                                   float* qbar, float* kbar, float* vsum,
                                   double* qbar64, double* kbar64, float* partial_h,
                                   void* kcen, void* vbar, const StatsPlan& plan, hipStream_t stream) {
  const int npad = ((dm.N + kTile - 1) / kTile) * kTile;
  const dim3 grid(plan.n_chunks, dm.bh());
#define PISA_STATS_BF16(DD, TPB)                                                                           \
  hipLaunchKernelGGL((stats_bf16_kernel<DD, TPB, false>), grid, dim3(64 * stats_waves(DD)), 0, stream, (const unsigned int*)q, \
                     (const unsigned int*)k, (const unsigned int*)v, qbar, kbar, vsum, qbar64, kbar64,     \
                     partial_h, (unsigned short*)kcen, (unsigned short*)vbar, npad, dm.L, dm.N,                \
                     plan.chunk_blocks, plan.n_chunks, nullptr, 0.0, nullptr)
  if (dm.d == 128 && dm.B == kTile) PISA_STATS_BF16(128, 1);
  else if (dm.d == 128) PISA_STATS_BF16(128, 2);
  else if (dm.B == kTile) PISA_STATS_BF16(64, 1);
  else PISA_STATS_BF16(64, 2);
#undef PISA_STATS_BF16
  return hipGetLastError();
}

// log(||H_j - hsum / N||_F + eps) per block with H_j rebuilt on the bf16 matrix cores (fp32-level
// accuracy, the accuracy hsum itself has).
hipError_t launch_block_heterogeneity_fast(const Dims& dm, const void* k, const void* v, const float* hsum,
                                           double eps, double* log_m, hipStream_t stream) {
  StatsPlan plan = stats_plan(dm);
  // No partial sums are written here, so up to few_blocks a block of 64 has a workgroup to itself.  In twos, which save every other
  // read of hsum, / one by one, us: 4 heads of 1 000 tokens 8.7 / 6.1, 48 of 1 000 16.8 / 13.8, 24 of 4 608 24.1 / 22.4, head_dim
  // 64 6.1 / 4.5, 7.5 / 6.3, 10.4 / 11.0.  Blocks of 128 go as 512 workgroups (24 of 4 608 24.3, one by one 26.4).
  if (few_blocks(dm)) {
    const int chunk = dm.B == kTile ? 1 : chunk_for(dm, 512);
    plan = {chunk, (dm.N + chunk - 1) / chunk};
  }
  const dim3 grid(plan.n_chunks, dm.bh());
#define PISA_HET_FAST(DD, TPB)                                                                              \
  hipLaunchKernelGGL((stats_bf16_kernel<DD, TPB, true>), grid, dim3(64 * stats_waves(DD)), 0, stream, nullptr,               \
                     (const unsigned int*)k, (const unsigned int*)v, nullptr, nullptr, nullptr, nullptr,    \
                     nullptr, nullptr, nullptr, nullptr, 0, dm.L, dm.N, plan.chunk_blocks, plan.n_chunks,   \
                     hsum, eps, log_m)
  if (dm.d == 128 && dm.B == kTile) PISA_HET_FAST(128, 1);
  else if (dm.d == 128) PISA_HET_FAST(128, 2);
  else if (dm.B == kTile) PISA_HET_FAST(64, 1);
  else PISA_HET_FAST(64, 2);
#undef PISA_HET_FAST
  return hipGetLastError();
}

}  // namespace pisa
