// fp32 attention path (dense and PISA) on the fp32 matrix instruction v_mfma_f32_16x16x4_f32.
//
// Workgroup = 8 wavefronts = RG row groups of 16 query rows x KG key groups.  Keys are walked in
// pieces of 16 rows; a trip stages KG consecutive pieces of K and V in LDS and each wave takes its
// row group against its own piece, with a running maximum, row sum and output of its own; the KG
// partial results of a row meet in LDS at the end.  As in the bf16 kernels everything is transposed:
//     S^T (keys x queries) = K_piece (keys x d) * Q^T,    O^T (d x queries) = V_piece^T * P^T
// so that a lane owns one query column and the S^T accumulator is already the B operand of the
// second product: lane (i = lane % 16, g = lane / 16) holds keys 4 g .. 4 g + 3 of query i, and
// contraction step r of the second product takes key 4 g + r of every g.  Both A operands come from
// ds_read_b128: four channels of K feed four contraction steps (K rows XOR their 16-byte chunk index
// with the row, so the 16 rows of a read hit different banks), four channels of V feed four 16-channel
// tiles of O^T (tile t <-> channels 4 i + t; a row is read in one contiguous line).
//
// Stages are filled global -> LDS without registers.  Double buffered (NBUF = 2) the loads of trip t + 1
// are in flight during all of trip t, one barrier a trip; where two buffers do not fit (NBUF = 1) K and V
// take turns: V of trip t is in flight while S^T of trip t is computed, K of trip t + 1 while O^T is, two
// barriers a trip.
//
// Bound by the fp32 matrix instruction (256 flop per clock and CU) and, on sequences of a few thousand
// tokens, by how evenly the workgroups divide over the CUs.  8 heads of 4 500 tokens, head_dim 128, r = 0.85:
// 1 080 us as a vector-ALU kernel (four threads per row, keys and probabilities through LDS), 221 us now;
// 2 heads of 1 024, head_dim 64, r = 0.75: 69 us, now 12 us.
//
// The three phases of Alg. 1 run inside one running-max softmax:
//   Phase 1  pieces of the selected blocks S_i (all of the sequence for dense attention)
//   Phase 2  pieces of 16 centroids: logit s q.kbar_j + ln B_j, selected columns and columns past N
//            masked; values vsum_j, whose 1 / B_j goes into the probability; the same mass is l_tail
//   Phase 3  O^T += hsum^T (w Q)^T, the second product with hsum's rows in the place of V's and Q's
//            registers in the place of P's
#include "common.h"

namespace pisa {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
#define LDS_PTR(T) __attribute__((address_space(3))) T*

constexpr int kPiece = 16;      // keys per piece
constexpr int kWaves = 8;       // wavefronts per workgroup

struct P32 {
  const float* q;
  const float* k;
  const float* v;
  const float* kbar;
  const float* vsum;
  const float* hsum;
  const int32_t* idx;
  float* out;
  float* lse;
  int L, B, N, k_top, n_groups, total;    // n_groups: row groups of a head per workgroup; total: workgroups with work
  float scale;
  int dense;
};

__device__ inline void wait_async_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Largest of the four lanes that share lane % 16 (row swaps on the vector ALU instead of LDS shuffles).
__device__ inline float max_over_g(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// One LDS-DMA instruction: 64 lanes x 16 bytes from per-lane addresses to 1 KB at `lds` (wave-uniform).
// Inline asm keeps the compiler from waiting on it before unrelated LDS reads; a stage is read only
// after wait_async_loads() + barrier.  (M0 needs one wait state before the instruction reads it.)
__device__ inline void dma_1kb(const float* src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds), "v"(src)
               : "memory", "m0");
}

template <int D, int RG, int KG, int NBUF>
__global__ __launch_bounds__(64 * kWaves, NBUF * KG * D > 512 ? 2 : 4) void attn_fp32_kernel(P32 p) {
  static_assert(RG * KG == kWaves, "eight wavefronts");
  constexpr int NS = D / 16;              // 16-channel slices
  constexpr int NT = D / 16;              // O^T tiles of 16 channels
  constexpr int PIECE_F = kPiece * D;     // floats per piece
  constexpr int STAGE_F = KG * PIECE_F;   // floats per stage (K or V)
  constexpr int NLD = STAGE_F * 4 / 1024 / kWaves;   // 1 KB loads per wave and stage
  constexpr int RPL = 1024 / (D * 4);     // rows per load
  __shared__ __attribute__((aligned(1024))) float stage[2 * NBUF * STAGE_F];    // (K | V) x NBUF
  __shared__ unsigned short list[kMaxBlocks];
  __shared__ unsigned int chosen[kMaxBlocks / 32];
  __shared__ float part_s[3][KG][RG * 16];   // m, l, l_tail of every key group

  // Each XCD gets a contiguous range of (head, row group) items, so that its L2 serves one head.
  const int per_xcd = (p.total + 7) / 8;
  if ((int)blockIdx.x / 8 >= per_xcd) return;
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (item >= p.total) return;
  const size_t bh = item / p.n_groups;
  const int row0 = (item % p.n_groups) * (RG * 16);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave % RG, kg = wave / RG;
  const int i = lane & 15, g = lane >> 4;
  const int L = p.L, N = p.N;
  const float* kh = p.k + bh * (size_t)L * D;
  const float* vh = p.v + bh * (size_t)L * D;
  const int q_row = row0 + 16 * rg + i;
  const int tpb = p.B / kTile;
  LDS_PTR(float) ks = (LDS_PTR(float)) & stage[0];
  const unsigned lds_addr = (unsigned)(unsigned long long)ks;

  // ---- Q^T operand: channels 16 s + 4 g + u of this lane's row ----
  f32x4 q[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    q[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (q_row < L) q[s] = *reinterpret_cast<const f32x4*>(p.q + (bh * (size_t)L + q_row) * D + 16 * s + 4 * g);
  }

  // ---- index row: list in LDS, bitmask for Phase 2 ----
  if (!p.dense) {
    const int32_t* row = p.idx + (bh * N + row0 / p.B) * (size_t)p.k_top;
    if (tid < kMaxBlocks / 32) chosen[tid] = 0u;
    __syncthreads();
    for (int t = tid; t < p.k_top; t += 64 * kWaves) {
      const int j = row[t];
      const bool ok = (unsigned)j < (unsigned)N;        // entries outside [0, N) are ignored
      list[t] = ok ? (unsigned short)j : (unsigned short)0xffff;
      if (ok) atomicOr(&chosen[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
  }

  // Key row at which piece `pc` of Phase 1 starts, or -1 (an ignored entry, or past the end).
  const int n_exact = (p.dense ? (L + kTile - 1) / kTile : p.k_top * tpb) * (kTile / kPiece);
  const int block_shift = tpb == 1 ? 2 : 3;                       // pieces per block: 4 or 8
  auto exact_row = [&](int pc) -> int {
    if (pc >= n_exact) return -1;
    if (p.dense) return pc * kPiece < L ? pc * kPiece : -1;
    const int j = __builtin_amdgcn_readfirstlane((int)list[pc >> block_shift]);
    if (j == 0xffff) return -1;
    const int r = j * p.B + (pc & ((1 << block_shift) - 1)) * kPiece;
    return r < L ? r : -1;
  };

  // This wave's share of a stage (K or V of buffer `buf`): 1 KB loads NLD wave .. NLD wave + NLD - 1, RPL
  // rows each.  Rows past the end of the source repeat its last row (the reader masks them).
  auto load_stage = [&](const float* src, int first_pc, int n_rows, bool kfmt, bool by_list, int buf) {
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int srow = (wave * NLD + u) * RPL;                    // first stage row of this load
      const int pc = first_pc + srow / kPiece;
      const int base = by_list ? exact_row(pc) : pc * kPiece;
      const int r_in = srow % kPiece + lane / (64 / RPL);         // row inside the piece
      const int ch = lane % (64 / RPL);                           // 16-byte chunk of the row in LDS
      const int row = min(max(base, 0) + r_in, n_rows - 1);
      const int src_ch = kfmt ? ch ^ r_in : ch;
      dma_1kb(src + (size_t)row * D + 4 * src_ch,
              lds_addr + ((2 * buf + (kfmt ? 0 : 1)) * STAGE_F + srow * D) * 4);
    }
  };

  f32x4 o[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) o[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f, l_tail = 0.f;     // log2 domain; l, l_tail: this lane's keys only
  // scale * log2(e) in two fp32 parts, so that the base-2 logit is the scaled product to fp32 rounding; both
  // positive, so that an infinite product stays what it is
  const double c = (double)p.scale * 1.4426950408889634074;
  float c_hi = (float)c;
  if ((double)c_hi >= c) c_hi = __uint_as_float(__float_as_uint(c_hi) - 1u);
  const float c_lo = (float)(c - (double)c_hi);

  // S^T of this wave's staged piece: element r = key 4 g + r.
  auto scores = [&](int buf) -> f32x4 {
    LDS_PTR(const float) kr = ks + 2 * buf * STAGE_F + (kPiece * kg + i) * D;
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0, kv, kn = *reinterpret_cast<LDS_PTR(const f32x4)>(kr + 4 * (g ^ i));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      kv = kn;                               // one read ahead of the products
      if (s + 1 < NS) kn = *reinterpret_cast<LDS_PTR(const f32x4)>(kr + 4 * ((4 * (s + 1) + g) ^ i));
      a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[0], q[s][0], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[1], q[s][1], a1, 0, 0, 0);
      a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[2], q[s][2], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[3], q[s][3], a1, 0, 0, 0);
    }
    return a0 + a1;
  };
  // O^T += (staged rows)^T b, b = B operand of the piece's 16 rows.
  auto add_values = [&](const f32x4 b, int buf) {
    LDS_PTR(const float) v0 = ks + (2 * buf + 1) * STAGE_F + (kPiece * kg + 4 * g) * D + 4 * i;
    constexpr int NR = NT;                   // reads: row r of the four, half hf of its channels
    f32x4 vv, vn = *reinterpret_cast<LDS_PTR(const f32x4)>(v0);
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      const int r = n / (NT / 4), hf = n % (NT / 4);
      vv = vn;
      if (n + 1 < NR)
        vn = *reinterpret_cast<LDS_PTR(const f32x4)>(v0 + (n + 1) / (NT / 4) * D + 64 * ((n + 1) % (NT / 4)));
#pragma unroll
      for (int t = 0; t < 4; ++t)
        o[4 * hf + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[t], b[r], o[4 * hf + t], 0, 0, 0);
    }
  };
  // Clears what add_values would read of a piece's rows from `rows` on: copies of the last row there is, whose
  // probability of 0 would make a NaN of an infinity.  (Waves that share the piece write the same zeros.)
  auto clear_absent = [&](int rows, int buf) {
    int ln = lane;
    asm volatile("" : "+v"(ln));               // the addresses are made here, not kept in registers all along
    LDS_PTR(float) v0 = ks + (2 * buf + 1) * STAGE_F + (kPiece * kg + 4 * (ln >> 4)) * D + 4 * (ln & 15);
#pragma unroll 1
    for (int r = 0; r < 4; ++r) {
      if (4 * (ln >> 4) + r >= rows)
#pragma unroll
        for (int hf = 0; hf < NT / 4; ++hf)
          *reinterpret_cast<LDS_PTR(f32x4)>(v0 + r * D + 64 * hf) = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
  };
  // Running maximum takes in the logits x (bias included, log2 domain up to the bias); returns the
  // probabilities and adds their sum to l.
  bool far = false;                          // uniform: some row's maximum lies beyond +-2^20
  auto softmax = [&](const f32x4 s, const f32x4 bias) -> f32x4 {
    f32x4 z;
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] = fmaf(s[r], c_hi, bias[r]);
    const float t = max_over_g(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
    const float m_new = fmaxf(m, t);
    const float m_safe = m_new == -INFINITY ? 0.f : m_new;
    if (__any(m_new != m)) {
      const float corr = __builtin_amdgcn_exp2f(m - m_safe);
      l *= corr;
      l_tail *= corr;
#pragma unroll
      for (int t2 = 0; t2 < NT; ++t2) o[t2] *= corr;
      m = m_new;
      far = __any(!(fabsf(m_new) <= 0x1p20f));
    }
    f32x4 e;
    if (!far) {
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_hi, fmaf(s[r], c_lo, bias[r] - m_safe)));
    } else {
      // There the rounding of the maximum itself is no longer small against 1 (keys masked by a huge negative
      // channel, for one): the same rounded product is subtracted from it, so that the largest key keeps weight 1.
#pragma clang fp contract(off)
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(s[r] * c_hi - (m_safe - bias[r]));
    }
    l += (e[0] + e[1]) + (e[2] + e[3]);
    return e;
  };

  // The walk over `n` pieces of (src_k, src_v): `absorb(pc, buf, e)` turns this wave's staged K piece into the B
  // operand e of the second product and returns the rows the piece has, 0 if the wave has nothing in this trip.
  auto walk = [&](const float* src_k, const float* src_v, int n, int n_rows, bool by_list, auto absorb) {
    load_stage(src_k, 0, n_rows, true, by_list, 0);
    if (NBUF == 2) load_stage(src_v, 0, n_rows, false, by_list, 0);
    int buf = 0;
    for (int pc = 0; pc < n; pc += KG) {
      wait_async_loads();
      __syncthreads();                       // this trip's K (and V, if double buffered) has landed
      f32x4 e = {0.f, 0.f, 0.f, 0.f};
      if (NBUF == 2) {
        if (pc + KG < n) {                   // the other buffer was used up before the barrier
          load_stage(src_k, pc + KG, n_rows, true, by_list, buf ^ 1);
          load_stage(src_v, pc + KG, n_rows, false, by_list, buf ^ 1);
        }
        const int rows = absorb(pc + kg, buf, e);
        if (rows > 0) {
          if (rows < kPiece) clear_absent(rows, buf);
          add_values(e, buf);
        }
        buf ^= 1;
      } else {
        load_stage(src_v, pc, n_rows, false, by_list, 0);
        const int rows = absorb(pc + kg, 0, e);
        wait_async_loads();
        __syncthreads();                     // V has landed; K is used up
        if (pc + KG < n) load_stage(src_k, pc + KG, n_rows, true, by_list, 0);
        if (rows > 0) {
          if (rows < kPiece) clear_absent(rows, 0);
          add_values(e, 0);
        }
      }
    }
  };

  // ---- Phase 1: exact pieces ----
  if (n_exact > 0)
    walk(kh, vh, n_exact, L, true, [&](int pc, int buf, f32x4& e) -> int {
      const int first = exact_row(pc);
      if (first < 0) return 0;
      f32x4 bias;
#pragma unroll
      for (int r = 0; r < 4; ++r) bias[r] = first + 4 * g + r < L ? 0.f : -INFINITY;
      e = softmax(scores(buf), bias);
      return L - first;
    });

  // ---- Phase 2: centroid pieces ----
  const bool approx = !p.dense && p.k_top < N && p.kbar != nullptr;
  if (approx) {
    const int last_rows = L - (N - 1) * p.B;
    const float b_full = log2f((float)p.B), b_last = log2f((float)last_rows);
    const float inv_full = 1.f / (float)p.B, inv_last = 1.f / (float)last_rows;
    const int n_cen = (N + kPiece - 1) / kPiece;
    __syncthreads();                         // every wave is done with the stages
    walk(p.kbar + bh * (size_t)N * D, p.vsum + bh * (size_t)N * D, n_cen, N, false,
         [&](int pc, int buf, f32x4& e) -> int {
           if (pc >= n_cen) return 0;
           const int j0 = pc * kPiece + 4 * g;          // this lane's first centroid
           const unsigned bits = chosen[j0 >> 5] >> (j0 & 31);
           f32x4 bias;
#pragma unroll
           for (int r = 0; r < 4; ++r)
             bias[r] = (j0 + r >= N || ((bits >> r) & 1u)) ? -INFINITY : (j0 + r == N - 1 ? b_last : b_full);
           e = softmax(scores(buf), bias);
           l_tail += (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
           for (int r = 0; r < 4; ++r) e[r] *= j0 + r == N - 1 ? inv_last : inv_full;
           return N - pc * kPiece;
         });
  }

  // ---- the key groups of a row agree on one maximum ----
  const bool first_order = approx && p.hsum != nullptr;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  l_tail += __shfl_xor(l_tail, 16);
  l_tail += __shfl_xor(l_tail, 32);
  if (g == 0) {
    part_s[0][kg][16 * rg + i] = m;
    part_s[1][kg][16 * rg + i] = l;
    part_s[2][kg][16 * rg + i] = l_tail;
  }
  __syncthreads();                           // also: every wave is done with the stages
  if (first_order) load_stage(p.hsum + bh * (size_t)D * D, 0, D, false, false, 0);
  float m_all = -INFINITY;
#pragma unroll
  for (int u = 0; u < KG; ++u) m_all = fmaxf(m_all, part_s[0][u][16 * rg + i]);
  float l_all = 0.f, tail_all = 0.f;
  // a group that met no key at all (maximum still -inf) holds zeros
  auto weight = [&](float m_part) { return m_part == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_part - m_all); };
#pragma unroll
  for (int u = 0; u < KG; ++u) {
    const float f = weight(part_s[0][u][16 * rg + i]);
    l_all += part_s[1][u][16 * rg + i] * f;
    tail_all += part_s[2][u][16 * rg + i] * f;
  }
  {
    const float f = weight(m);
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t] *= f;
  }

  // ---- Phase 3: hsum's rows as values, w Q as probabilities ----
  if (first_order) {
    const float w = tail_all / (float)L * p.scale;
#pragma unroll
    for (int s0 = 0; s0 < NS; s0 += KG) {
      wait_async_loads();
      __syncthreads();
#pragma unroll
      for (int u = 0; u < KG && s0 + u < NS; ++u)
        if (kg == u) add_values(q[s0 + u] * w, 0);        // uniform over the wave
      if (s0 + KG < NS) {
        __syncthreads();
        load_stage(p.hsum + bh * (size_t)D * D, s0 + KG, D, false, false, 0);
      }
    }
  }

  // ---- sum over the key groups, normalise, store ----
  __syncthreads();
  LDS_PTR(f32x4) board = (LDS_PTR(f32x4))ks;
  static_assert((KG - 1) * RG * NT * 64 * 16 <= 2 * NBUF * STAGE_F * 4, "the partial outputs must fit the stages");
  if (kg > 0) {
#pragma unroll
    for (int t = 0; t < NT; ++t) board[(((kg - 1) * RG + rg) * NT + t) * 64 + lane] = o[t];
  }
  __syncthreads();
  if (kg > 0) return;
#pragma unroll
  for (int u = 0; u < KG - 1; ++u)
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t] += board[((u * RG + rg) * NT + t) * 64 + lane];
  if (q_row < L) {
    // o[4 hf + t][r] = channel 64 hf + 4 (4 g + r) + t
    const float inv_l = 1.f / l_all;
    float* orow = p.out + (bh * (size_t)L + q_row) * D;
#pragma unroll
    for (int hf = 0; hf < NT / 4; ++hf)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4 w = {o[4 * hf][r] * inv_l, o[4 * hf + 1][r] * inv_l, o[4 * hf + 2][r] * inv_l,
                         o[4 * hf + 3][r] * inv_l};
        *reinterpret_cast<f32x4*>(orow + 64 * hf + 16 * g + 4 * r) = w;
      }
    if (p.lse && g == 0) p.lse[bh * (size_t)L + q_row] = (m_all + log2f(l_all)) * 0.69314718055994530942f;
  }
}

template <int D, int RG, int KG, int NBUF> void launch(P32& p, const Dims& dm, hipStream_t stream) {
  p.n_groups = (dm.L + 16 * RG - 1) / (16 * RG);
  p.total = p.n_groups * dm.bh();
  hipLaunchKernelGGL((attn_fp32_kernel<D, RG, KG, NBUF>), dim3(8 * ((p.total + 7) / 8)), dim3(64 * kWaves), 0, stream, p);
}

template <int D> void launch_d(P32& p, const Dims& dm, hipStream_t stream) {
  // Query rows per workgroup.  Fewer rows per workgroup fill more of the chip and balance it better, more
  // rows read K and V less often (a 16-row workgroup asks L2 for 8.4 TB/s, which is what it gives).
  // Measured, us per call (statistics and selection included), 16 / 32 / 64 rows: 32 tiles at head_dim 64
  // 29.7 / 32.3 / 38.5; at head_dim 128 128 tiles 71.7 / 59.5 / 67.2, 568 tiles 388 / 278 / 283, 1136 tiles
  // 732 / 465 / 448.
  const long long tiles = (long long)((dm.L + kTile - 1) / kTile) * dm.bh();
  if (tiles <= 64) launch<D, 1, 8, D == 128 ? 1 : 2>(p, dm, stream);
  else if (tiles <= 768) launch<D, 2, 4, D == 128 ? 1 : 2>(p, dm, stream);
  else launch<D, 4, 2, 2>(p, dm, stream);
}

}  // namespace

hipError_t launch_attention_fp32(const Dims& dm, const AttnArgs& a, hipStream_t stream) {
  P32 p;
  p.q = (const float*)a.q;
  p.k = (const float*)a.k;
  p.v = (const float*)a.v;
  p.kbar = a.kbar;
  p.vsum = a.vsum;
  p.hsum = a.hsum;
  p.idx = a.idx;
  p.out = (float*)a.out;
  p.lse = a.lse;
  p.L = dm.L;
  p.B = dm.B;
  p.N = dm.N;
  p.k_top = a.k_top;
  p.scale = dm.scale;
  p.dense = a.dense ? 1 : 0;
  if (dm.d == 64) launch_d<64>(p, dm, stream);
  else launch_d<128>(p, dm, stream);
  return hipGetLastError();
}

}  // namespace pisa
