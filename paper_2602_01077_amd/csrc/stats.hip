// pisa_block_stats: block means of Q and K, block sums of V, and the global
// first-order statistic  hsum = sum_j sum_n (k_{j,n} - kbar_j)^T v_{j,n}
// (Alg. 1, "Prepare" step; H_j as defined in the "Global First-Order Correction" paragraph).
//
// Grid: (n_chunks, batch*heads).  A workgroup walks `chunk_blocks` consecutive
// blocks of one head, keeps its share of H in registers, and writes one partial
// d x d matrix; a second kernel adds the partials in chunk order, so hsum is
// bit-identical from run to run.
#include "common.h"
#include "reduce_h.h"

namespace pisa {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
#define LDS_PTR(T) __attribute__((address_space(3))) T*

// Statistics of fp32 inputs (bf16 inputs have a kernel of their own) on v_mfma_f32_16x16x4_f32.
// A workgroup of 4 waves holds the K and V rows of a whole block (TPB tiles of 64 rows) in registers, 16
// bytes of a row per lane and load, so every input is read once: column sums in fp64, one exchange over
// LDS, then tile by tile K centred on the block mean goes to LDS beside V and the registers take the
// loads of the next block, which are in flight during the products.
//   H += Kc^T V: lane (i = lane % 16, g = lane / 16) of contraction step s takes token 4 s + g; 16-byte
//   reads of a V row feed four 16-channel tiles (tile t of half hf <-> channels 64 hf + 4 i + t); of the key
//   channels each wave owns D / 4: channels 64 (w / 2) + 4 i + 2 (w % 2) + {0, 1} (head_dim 64: 4 i + w).
// 8 heads of 4 500 tokens, head_dim 128: 63 us as a vector-ALU kernel that read K and V twice in 4-byte
// pieces, 25.7 us now (55 MB of inputs and 13 MB of partial H; 192 workgroups of three blocks, so this is the
// latency of the first loads plus 3 x 3.4 us of products and the stores; 33 us with two blocks to a workgroup, where
// some compute units had two workgroups).
// 2 heads of 1 024 tokens, head_dim 64: 11.1 us, now 5.6 us.
template <int D, int TPB>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2) void stats_fp32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ qbar, float* __restrict__ kbar, float* __restrict__ vsum,
    double* __restrict__ qbar64, double* __restrict__ kbar64, float* __restrict__ partial_h,
    int L, int N, int chunk_blocks, int n_chunks) {
  constexpr int B = TPB * kTile;
  constexpr int LPR = D / 4;                // lanes per row
  constexpr int RPP = 256 / LPR;            // rows per pass of the workgroup
  constexpr int NR = kTile / RPP;           // loads per lane, tensor and tile
  constexpr int NA = D / 64;                // 16-channel key tiles per wave
  constexpr int NB = D / 16;                // 16-channel value tiles
  __shared__ __attribute__((aligned(16))) float kc[kTile][D];
  __shared__ __attribute__((aligned(16))) float vs[kTile][D];
  __shared__ __attribute__((aligned(16))) double red[3][4][D];
  __shared__ __attribute__((aligned(16))) double kmean[D];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int r0 = tid / LPR, c0 = (tid % LPR) * 4;      // this lane's first row of a tile, its channels
  const int chunk = blockIdx.x;
  const size_t bh = blockIdx.y;
  const float* qh = q + bh * (size_t)L * D;
  const float* kh = k + bh * (size_t)L * D;
  const float* vh = v + bh * (size_t)L * D;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

  // One tile's rows of one tensor; rows past the end of the sequence are zero.
  auto load_tile = [&](const float* src, int row0, f32x4 (&x)[NR]) {
    const float* tile = src + (size_t)row0 * D;              // uniform
    if (row0 + kTile <= L) {
#pragma unroll
      for (int n = 0; n < NR; ++n) x[n] = *reinterpret_cast<const f32x4*>(tile + (unsigned)((r0 + RPP * n) * D + c0));
    } else {
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        x[n] = zero;
        if (row0 + r0 + RPP * n < L) x[n] = *reinterpret_cast<const f32x4*>(tile + (unsigned)((r0 + RPP * n) * D + c0));
      }
    }
  };

  f32x4 acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = zero;

  f32x4 qx[TPB][NR], kx[TPB][NR], vx[TPB][NR];
  const int j_begin = chunk * chunk_blocks, j_end = min(N, j_begin + chunk_blocks);
#pragma unroll
  for (int t = 0; t < TPB; ++t) {
    load_tile(qh, j_begin * B + t * kTile, qx[t]);
    load_tile(kh, j_begin * B + t * kTile, kx[t]);
    load_tile(vh, j_begin * B + t * kTile, vx[t]);
  }
  for (int j = j_begin; j < j_end; ++j) {
    const int rows = min(B, L - j * B);
    // ---- column sums in fp64 ----
    double sum[3][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) sum[0][c] = sum[1][c] = sum[2][c] = 0.0;
#pragma unroll
    for (int t = 0; t < TPB; ++t)
#pragma unroll
      for (int n = 0; n < NR; ++n)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          sum[0][c] += (double)qx[t][n][c];
          sum[1][c] += (double)kx[t][n][c];
          sum[2][c] += (double)vx[t][n][c];
        }
#pragma unroll
    for (int x = 0; x < 3; ++x) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (LPR == 16) sum[x][c] += __shfl_xor(sum[x][c], 16);
        sum[x][c] += __shfl_xor(sum[x][c], 32);
      }
      if (lane < LPR) {
        *reinterpret_cast<f64x2*>(&red[x][wave][c0]) = (f64x2){sum[x][0], sum[x][1]};
        *reinterpret_cast<f64x2*>(&red[x][wave][c0 + 2]) = (f64x2){sum[x][2], sum[x][3]};
      }
    }
#pragma unroll
    for (int t = 0; t < TPB; ++t)
      if (j + 1 < j_end) load_tile(qh, (j + 1) * B + t * kTile, qx[t]);
    __syncthreads();
    if (tid < D) {
      double s[3];
#pragma unroll
      for (int x = 0; x < 3; ++x) s[x] = ((red[x][0][tid] + red[x][1][tid]) + red[x][2][tid]) + red[x][3][tid];
      const double qm = s[0] / (double)rows, km = s[1] / (double)rows;
      const size_t o = (bh * N + j) * D + tid;
      qbar[o] = (float)qm;
      kbar[o] = (float)km;
      vsum[o] = (float)s[2];
      if (qbar64) qbar64[o] = qm;
      if (kbar64) kbar64[o] = km;
      kmean[tid] = km;
    }
    __syncthreads();
    double mean[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) mean[c] = kmean[c0 + c];
#pragma unroll
    for (int t = 0; t < TPB; ++t) {
      if (t > 0) __syncthreads();             // the products of the first tile have been read
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        const int row = r0 + RPP * n;
        f32x4 kv = zero;
        if (t * kTile + row < rows) {
#pragma unroll
          for (int c = 0; c < 4; ++c) kv[c] = (float)((double)kx[t][n][c] - mean[c]);
        }
        *reinterpret_cast<f32x4*>(&kc[row][c0]) = kv;
        *reinterpret_cast<f32x4*>(&vs[row][c0]) = vx[t][n];
      }
      if (j + 1 < j_end) {
        load_tile(kh, (j + 1) * B + t * kTile, kx[t]);
        load_tile(vh, (j + 1) * B + t * kTile, vx[t]);
      }
      __syncthreads();
#pragma unroll 2
      for (int s = 0; s < kTile / 4; ++s) {
        const int n = 4 * s + g;
        float a[NA];
        if constexpr (D == 128) {
          const f32x2 av = *reinterpret_cast<const f32x2*>(&kc[n][64 * (wave >> 1) + 4 * i + 2 * (wave & 1)]);
          a[0] = av[0];
          a[1] = av[1];
        } else {
          a[0] = kc[n][4 * i + wave];
        }
#pragma unroll
        for (int hf = 0; hf < NB / 4; ++hf) {
          const f32x4 bv = *reinterpret_cast<const f32x4*>(&vs[n][64 * hf + 4 * i]);
#pragma unroll
          for (int x = 0; x < NA; ++x)
#pragma unroll
            for (int u = 0; u < 4; ++u)
              acc[x][4 * hf + u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[x], bv[u], acc[x][4 * hf + u], 0, 0, 0);
        }
      }
    }
    // the next block's writes to kc, vs and red come after its own barriers
  }
  // acc[x][4 hf + u][r] = H[key channel (4 g + r) of this wave's tile x][64 hf + 4 i + u]
  float* ph = partial_h + (bh * n_chunks + chunk) * (size_t)D * D;
#pragma unroll
  for (int x = 0; x < NA; ++x)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = D == 128 ? 64 * (wave >> 1) + 4 * (4 * g + r) + 2 * (wave & 1) + x : 4 * (4 * g + r) + wave;
#pragma unroll
      for (int hf = 0; hf < NB / 4; ++hf) {
        const f32x4 w = {acc[x][4 * hf][r], acc[x][4 * hf + 1][r], acc[x][4 * hf + 2][r], acc[x][4 * hf + 3][r]};
        *reinterpret_cast<f32x4*>(&ph[(size_t)a * D + 64 * hf + 4 * i]) = w;
      }
    }
}

// hsum (and, if asked for, its packed bf16 split) from the per-chunk partial sums: one thread
// per matrix element.
__global__ __launch_bounds__(256) void reduce_h_kernel(const float* __restrict__ partial_h,
                                                       float* __restrict__ hsum,
                                                       unsigned short* __restrict__ hpack, int n_chunks, int D) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= D * D) return;
  reduce_h_element(partial_h, hsum, hpack, n_chunks, D, blockIdx.y, e);
}

}  // namespace

hipError_t launch_block_stats_bf16(const Dims& dm, const void* q, const void* k, const void* v,
                                       float* qbar, float* kbar, float* vsum,
                                       double* qbar64, double* kbar64, float* partial_h,
                                       void* kcen, void* vbar, const StatsPlan& plan, hipStream_t stream);

hipError_t launch_block_stats(const Dims& dm, const void* q, const void* k, const void* v,
                              float* qbar, float* kbar, float* vsum, float* hsum,
                              double* qbar64, double* kbar64, float* partial_h,
                              const StatsExtras& extra, hipStream_t stream) {
  const StatsPlan plan = stats_plan(dm);
  dim3 grid(plan.n_chunks, dm.bh());
#define PISA_STATS(DD, TPB)                                                                            \
  hipLaunchKernelGGL((stats_fp32_kernel<DD, TPB>), grid, dim3(256), 0, stream, (const float*)q,       \
                     (const float*)k, (const float*)v, qbar, kbar, vsum, qbar64, kbar64, partial_h, dm.L, \
                     dm.N, plan.chunk_blocks, plan.n_chunks)
  if (dm.dtype == PISA_BF16) {
    hipError_t e = launch_block_stats_bf16(dm, q, k, v, qbar, kbar, vsum, qbar64, kbar64,
                                           partial_h, extra.kcen, extra.vbar, plan, stream);
    if (e != hipSuccess) return e;
  } else if (dm.d == 64 && dm.B == kTile) {
    PISA_STATS(64, 1);
  } else if (dm.d == 64) {
    PISA_STATS(64, 2);
  } else if (dm.B == kTile) {
    PISA_STATS(128, 1);
  } else {
    PISA_STATS(128, 2);
  }
#undef PISA_STATS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (extra.defer_reduce) return hipSuccess;   // the caller reduces the partial sums in a later launch
  const int dd = dm.d * dm.d;
  hipLaunchKernelGGL(reduce_h_kernel, dim3((dd + 255) / 256, dm.bh()), dim3(256), 0, stream,
                     partial_h, hsum, (unsigned short*)extra.hpack, plan.n_chunks, dm.d);
  return hipGetLastError();
}

}  // namespace pisa
