// fp32 attention path (dense and PISA) on the fp32 matrix instruction v_mfma_f32_16x16x4_f32.
//
// Workgroup = 4 or 8 wavefronts on 32 (or 16) query rows.  Keys are walked in pieces of 16 rows: wave w takes pieces
// w, w + KG, ... against all of the workgroup's rows, with a running maximum, row sum and output of its own; the KG
// partial results of a row meet in LDS at the end.  As in the bf16 kernels everything is transposed:
//     S^T (keys x queries) = K_piece (keys x d) * Q^T,    O^T (d x queries) = V_piece^T * P^T
// so that a lane owns one query column per 16 rows and the S^T accumulator is already the B operand of the
// second product: lane (i = lane % 16, g = lane / 16) holds keys 4 g .. 4 g + 3 of query i, and
// contraction step r of the second product takes key 4 g + r of every g.  Both A operands come from
// ds_read_b128, each read serving both 16-row tiles: four channels of K feed four contraction steps (K rows XOR their
// 16-byte chunk index with the row, so the 16 rows of a read hit different banks), four channels of V feed four
// 16-channel tiles of O^T (tile t <-> channels 4 i + t; a row is read in one contiguous line).
//
// A wave fills its stages (one K piece, one V piece) itself, global -> LDS without registers, and nobody else reads them:
// the walk has no barriers, a wave waits for its own loads only.  V of a piece is in flight while S^T is computed, the
// next K while O^T is.  The centroids' pieces follow the exact ones in the same walk.
//
// Bound by the fp32 matrix instruction (256 flop per clock and CU), by what a workgroup does once (index row, first
// loads, merge: 9 us) and by how evenly the workgroups divide over the CUs.  8 heads of 4 500 tokens, head_dim 128,
// r = 0.85, us for the attention step: 201 with stages shared by eight waves (two barriers a trip, 16 rows to a wave), 184
// with stages of a wave's own, 170 with the last row groups in halves (dense 899, 820, 749); 2 heads of 1 024, head_dim 64,
// r = 0.75: 11.8, now 11.3, at head_dim 128 19.1, now 14.5.  With the loads taken out the first takes 167 instead of
// 184, without the softmax 170.
//
// The three phases of Alg. 1 run inside one running-max softmax:
//   Phase 1  pieces of the selected blocks S_i (all of the sequence for dense attention)
//   Phase 2  pieces of 16 centroids: logit s q.kbar_j + ln B_j, selected columns and columns past N
//            masked; values vsum_j, whose 1 / B_j goes into the probability; the same mass is l_tail
//   Phase 3  O^T += hsum^T (w Q)^T, the second product with hsum's rows in the place of V's and Q's
//            registers in the place of P's
#include <type_traits>

#include "common.h"

namespace pisa {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
#define LDS_PTR(T) __attribute__((address_space(3))) T*

constexpr int kPiece = 16;      // keys per piece
constexpr int kCusPerXcd = 32;
typedef __attribute__((address_space(4))) int32_t ConstInt;

// Wavefronts per SIMD: what registers allow at 32 rows a workgroup, in workgroups that fit the LDS.
constexpr int waves_per_simd(int d, int kg) { return d == 128 || kg == 8 ? 2 : 3; }

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
  int L, B, N, k_top, n_groups, total;    // n_groups: row groups of a head; total: of all heads
  int per_xcd, n_whole;                   // groups per XCD; how many of them a workgroup takes whole
  float scale;
  int dense;
};

// s_waitcnt vmcnt(N) / lgkmcnt(0) with the other counters left alone (gfx9 encoding).
template <int N> __device__ inline void wait_loads() {
  static_assert(N >= 0 && N < 16, "low four bits of vmcnt");
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | N);
  asm volatile("" : : : "memory");
}
__device__ inline void wait_lds() {
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  asm volatile("" : : : "memory");
}

// Largest of the four lanes that share lane % 16 (row swaps on the vector ALU instead of LDS shuffles).
__device__ inline float max_over_g(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// One LDS-DMA instruction: 64 lanes x 16 bytes, global (base + voff + IMM) -> LDS (M0 + IMM + 16 lane).
// Inline asm keeps the compiler from waiting on it before unrelated LDS reads; a stage is read only after wait_loads().
// (M0 needs one wait state before the instruction reads it.)
__device__ inline void set_dma_lds_base(unsigned lds /* wave-uniform */) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(lds) : "memory", "m0");
}
template <int IMM> __device__ inline void dma_1kb(unsigned voff, const float* base /* wave-uniform */) {
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(voff), "s"(base), "n"(IMM) : "memory");
}
__device__ inline void dma_1kb_far(const float* src) {
  asm volatile("global_load_lds_dwordx4 %0, off" : : "v"(src) : "memory");
}

// One workgroup's work: RT * 16 query rows from row0 of head bh.
template <int D, int RT, int KG>
__device__ __forceinline__ void attend_rows(const P32& p, const size_t bh, const int row0, float* stage_mem,
                                            unsigned int* chosen, float (*part_s)[KG][32]) {
  constexpr int NS = D / 16;              // 16-channel slices
  constexpr int NT = D / 16;              // O^T tiles of 16 channels
  constexpr int PIECE_F = kPiece * D;     // floats per piece
  constexpr int NLD = PIECE_F * 4 / 1024; // 1 KB loads per piece
  constexpr int RPL = 1024 / (D * 4);     // rows per load
  constexpr int LPR = 64 / RPL;           // lanes (16-byte chunks) per row
  constexpr int WAVE_F = 2 * PIECE_F;     // a wave's own stages: K | V
  const int tid = threadIdx.x, lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int L = p.L, N = p.N;
  const bool approx = !p.dense && p.k_top < N && p.kbar != nullptr;
  const bool first_order = approx && p.hsum != nullptr;
  LDS_PTR(float) ks = (LDS_PTR(float))stage_mem + kg * WAVE_F;
  const unsigned lds_addr = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)ks);

  // The index row is read through the scalar cache, an entry at a time, by the wave that needs it.
  const ConstInt* idx_row = nullptr;
  int j_mine = -1;
  if (!p.dense) {
    const int32_t* row = p.idx + (bh * N + row0 / p.B) * (size_t)p.k_top;
    idx_row = (const ConstInt*)(unsigned long long)row;
    if (tid < p.k_top) j_mine = row[tid];
  }

  // ---- Q^T operand: channels 16 s + 4 g + u of this lane's rows ----
  f32x4 q[RT][NS];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int q_row = row0 + 16 * rt + i;
      q[rt][s] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (q_row < L) q[rt][s] = *reinterpret_cast<const f32x4*>(p.q + (bh * (size_t)L + q_row) * D + 16 * s + 4 * g);
    }

  // ---- the pieces of the walk: those of the exact blocks, then those of the centroids; wave kg takes kg, kg + KG, ... ----
  const int shift = p.B == kTile ? 2 : 3;                         // pieces per block: 4 or 8
  const int n_exact = p.dense ? (L + kPiece - 1) / kPiece : p.k_top << shift;
  const int n_all = n_exact + (approx ? (N + kPiece - 1) / kPiece : 0);
  // First row of piece pc in its source (keys or centroids), or -1: an ignored entry, or rows past the end.
  auto first_row = [&](int pc) -> int {
    if (pc >= n_exact) return (pc - n_exact) * kPiece;
    if (p.dense) return pc * kPiece;
    const int j = idx_row[pc >> shift];
    if ((unsigned)j >= (unsigned)N) return -1;
    const int r = j * p.B + (pc & ((1 << shift) - 1)) * kPiece;
    return r < L ? r : -1;
  };
  // Loads of one piece (16 rows from `row` of a matrix of n_rows) to `dst` in LDS: K format if KF.  Rows past the
  // end repeat the last one (the reader masks them).
  const unsigned voff_v = (unsigned)lane * 16, voff_k = (unsigned)(lane / LPR * LPR + ((lane % LPR) ^ (lane / LPR))) * 16;
  auto load_rows = [&](const float* src, int row, int n_rows, auto kf_tag, unsigned dst) {
    constexpr bool KF = decltype(kf_tag)::value;
    row = __builtin_amdgcn_readfirstlane(max(row, 0));
    if (row + kPiece <= n_rows) {
      const float* base = src + (size_t)row * D;
      unsigned vo = KF ? voff_k : voff_v;
      asm volatile("" : "+v"(vo));           // the variants below are made here, not kept in registers all along
#pragma unroll
      for (int u0 = 0; u0 < NLD; u0 += 4) {                       // the immediate offset reaches 4 KB
        set_dma_lds_base(dst + u0 * 1024);
        const float* b = base + u0 * 256;
        dma_1kb<0>(KF ? vo ^ (u0 * RPL * 16) : vo, b);
        dma_1kb<1024>(KF ? vo ^ ((u0 + 1) * RPL * 16) : vo, b);
        dma_1kb<2048>(KF ? vo ^ ((u0 + 2) * RPL * 16) : vo, b);
        dma_1kb<3072>(KF ? vo ^ ((u0 + 3) * RPL * 16) : vo, b);
      }
    } else {
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll 1
      for (int u = 0; u < NLD; ++u) {
        const int r_in = u * RPL + ln / LPR, ch = ln % LPR;
        set_dma_lds_base(dst + u * 1024);
        dma_1kb_far(src + (size_t)min(row + r_in, n_rows - 1) * D + 4 * (KF ? ch ^ r_in : ch));
      }
    }
  };
  const float* kh = p.k + bh * (size_t)L * D;
  const float* vh = p.v + bh * (size_t)L * D;
  const float* kc = p.kbar + (approx ? bh * (size_t)N * D : 0);
  const float* vc = p.vsum + (approx ? bh * (size_t)N * D : 0);
  auto load_k = [&](int pc, int row) {
    if (pc < n_exact) load_rows(kh, row, L, std::true_type{}, lds_addr);
    else load_rows(kc, row, N, std::true_type{}, lds_addr);
  };
  auto load_v = [&](int pc, int row) {
    if (pc < n_exact) load_rows(vh, row, L, std::false_type{}, lds_addr + PIECE_F * 4);
    else load_rows(vc, row, N, std::false_type{}, lds_addr + PIECE_F * 4);
  };
  int pc = kg, row = -1;
  if (pc < n_all) {
    row = first_row(pc);
    load_k(pc, row);
    load_v(pc, row);
  }

  // ---- bitmask of the index row, for the centroids ----
  if (approx) {
    for (int w = tid; w < kMaxBlocks / 32; w += 64 * KG) chosen[w] = 0u;
    __syncthreads();
    for (int t = tid, j = j_mine; t < p.k_top; t += 64 * KG) {
      if (t != tid) j = p.idx[(bh * N + row0 / p.B) * (size_t)p.k_top + t];
      if ((unsigned)j < (unsigned)N) atomicOr(&chosen[j >> 5], 1u << (j & 31));   // entries outside [0, N) are ignored
    }
    __syncthreads();
  }

  f32x4 o[RT][NT];
  float m[RT], l[RT], l_tail[RT];            // log2 domain; l, l_tail: this lane's keys only
  bool far[RT];                              // uniform: some row's maximum lies beyond +-2^20
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int t = 0; t < NT; ++t) o[rt][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    m[rt] = -INFINITY;
    l[rt] = l_tail[rt] = 0.f;
    far[rt] = false;
  }
  // scale * log2(e) in two fp32 parts, so that the base-2 logit is the scaled product to fp32 rounding; both
  // positive, so that an infinite product stays what it is
  const double c = (double)p.scale * 1.4426950408889634074;
  float c_hi = (float)c;
  if ((double)c_hi >= c) c_hi = __uint_as_float(__float_as_uint(c_hi) - 1u);
  const float c_lo = (float)(c - (double)c_hi);

  // S^T of the staged piece: element r = key 4 g + r.
  auto scores = [&](f32x4 (&sc)[RT]) {
    LDS_PTR(const float) kr = ks + i * D;
    f32x4 a[RT][2], kv, kn = *reinterpret_cast<LDS_PTR(const f32x4)>(kr + 4 * (g ^ i));
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) a[rt][0] = a[rt][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      kv = kn;                               // one read ahead of the products
      if (s + 1 < NS) kn = *reinterpret_cast<LDS_PTR(const f32x4)>(kr + 4 * ((4 * (s + 1) + g) ^ i));
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          a[rt][u & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[u], q[rt][s][u], a[rt][u & 1], 0, 0, 0);
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) sc[rt] = a[rt][0] + a[rt][1];
  };
  // O^T += (staged rows)^T b, b = B operand of the piece's 16 rows.
  auto add_values = [&](const f32x4 (&b)[RT], LDS_PTR(const float) piece) {
    LDS_PTR(const float) v0 = piece + 4 * g * D + 4 * i;
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
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          o[rt][4 * hf + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[t], b[rt][r], o[rt][4 * hf + t], 0, 0, 0);
    }
  };
  // Clears what add_values would read of a piece's rows from `rows` on: copies of the last row there is, whose
  // probability of 0 would make a NaN of an infinity.
  auto clear_absent = [&](int rows) {
    int ln = lane;
    asm volatile("" : "+v"(ln));               // the addresses are made here, not kept in registers all along
    LDS_PTR(float) v0 = ks + PIECE_F + 4 * (ln >> 4) * D + 4 * (ln & 15);
#pragma unroll 1
    for (int r = 0; r < 4; ++r) {
      if (4 * (ln >> 4) + r >= rows)
#pragma unroll
        for (int hf = 0; hf < NT / 4; ++hf)
          *reinterpret_cast<LDS_PTR(f32x4)>(v0 + r * D + 64 * hf) = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
  };
  // Running maximum of row tile rt takes in the logits s * c + bias (log2 domain); returns the probabilities.
  auto softmax = [&](int rt, const f32x4 s, const f32x4 bias) -> f32x4 {
    f32x4 z;
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] = fmaf(s[r], c_hi, bias[r]);
    const float t = max_over_g(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
    const float m_new = fmaxf(m[rt], t);
    const float m_safe = m_new == -INFINITY ? 0.f : m_new;
    if (__any(m_new != m[rt])) {
      const float corr = __builtin_amdgcn_exp2f(m[rt] - m_safe);
      l[rt] *= corr;
      l_tail[rt] *= corr;
#pragma unroll
      for (int t2 = 0; t2 < NT; ++t2) o[rt][t2] *= corr;
      m[rt] = m_new;
      far[rt] = __any(!(fabsf(m_new) <= 0x1p20f));
    }
    f32x4 e;
    if (!far[rt]) {
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c_hi, fmaf(s[r], c_lo, bias[r] - m_safe)));
    } else {
      // There the rounding of the maximum itself is no longer small against 1 (keys masked by a huge negative
      // channel, for one): the same rounded product is subtracted from it, so that the largest key keeps weight 1.
#pragma clang fp contract(off)
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(s[r] * c_hi - (m_safe - bias[r]));
    }
    return e;
  };

  const int last_rows = L - (N - 1) * p.B;
  const float b_full = log2f((float)p.B), b_last = log2f((float)last_rows);
  const float inv_full = 1.f / (float)p.B, inv_last = 1.f / (float)last_rows;

  // ---- Phases 1 and 2 ----
  // No barriers: the stages are the wave's own.  A load may overwrite a stage once this wave's reads of it have returned.
  wait_loads<0>();                           // Q, and the first piece
  while (pc < n_all) {
    const int pc_n = pc + KG;
    const bool more = pc_n < n_all;
    const int row_n = more ? first_row(pc_n) : -1;
    if (row < 0) {                           // nothing to attend here
      wait_loads<0>();
      if (more) {
        load_k(pc_n, row_n);
        load_v(pc_n, row_n);
      }
    } else {
      f32x4 e[RT], bias, wt = {1.f, 1.f, 1.f, 1.f};
      wait_loads<NLD>();                     // K has landed; V may be on its way
      scores(e);
      wait_lds();
      if (more) load_k(pc_n, row_n);
      const bool cen = pc >= n_exact;
      const int rows = (cen ? N : L) - row;
      if (!cen) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bias[r] = 4 * g + r < rows ? 0.f : -INFINITY;
      } else {
        const int j0 = row + 4 * g;          // this lane's first centroid
        const unsigned bits = chosen[j0 >> 5] >> (j0 & 31);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          bias[r] = (j0 + r >= N || ((bits >> r) & 1u)) ? -INFINITY : (j0 + r == N - 1 ? b_last : b_full);
          wt[r] = j0 + r == N - 1 ? inv_last : inv_full;
        }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        e[rt] = softmax(rt, e[rt], bias);
        const float sum = (e[rt][0] + e[rt][1]) + (e[rt][2] + e[rt][3]);
        l[rt] += sum;
        l_tail[rt] += cen ? sum : 0.f;
        e[rt] *= wt;
      }
      if (more) wait_loads<NLD>();           // V has landed; the next K may be on its way
      else wait_loads<0>();
      if (rows < kPiece) clear_absent(rows);
      add_values(e, ks + PIECE_F);
      wait_lds();
      if (more) load_v(pc_n, row_n);
    }
    pc = pc_n;
    row = row_n;
  }

  // ---- the waves of a row agree on one maximum ----
  // This wave's pieces of hsum are on their way meanwhile
  const float* hs = p.hsum + bh * (size_t)D * D;
  // (where a wave has two, the second goes where its K pieces went)
  constexpr int HP = (NS + KG - 1) / KG;       // pieces of hsum per wave
  static_assert(HP <= 2, "two stages hold a wave's pieces of hsum");
  if (first_order) {
    if (kg < NS) load_rows(hs, kPiece * kg, D, std::false_type{}, lds_addr + PIECE_F * 4);
    if (HP == 2) load_rows(hs, kPiece * (KG + kg), D, std::false_type{}, lds_addr);
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    l[rt] += __shfl_xor(l[rt], 16);
    l[rt] += __shfl_xor(l[rt], 32);
    l_tail[rt] += __shfl_xor(l_tail[rt], 16);
    l_tail[rt] += __shfl_xor(l_tail[rt], 32);
    if (g == 0) {
      part_s[0][kg][16 * rt + i] = m[rt];
      part_s[1][kg][16 * rt + i] = l[rt];
      part_s[2][kg][16 * rt + i] = l_tail[rt];
    }
  }
  __syncthreads();
  float m_all[RT], l_all[RT], tail_all[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_all[rt] = -INFINITY;
#pragma unroll
    for (int u = 0; u < KG; ++u) m_all[rt] = fmaxf(m_all[rt], part_s[0][u][16 * rt + i]);
    l_all[rt] = tail_all[rt] = 0.f;
    // a wave that met no key at all (maximum still -inf) holds zeros
    auto weight = [&](float m_part) { return m_part == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_part - m_all[rt]); };
#pragma unroll
    for (int u = 0; u < KG; ++u) {
      const float f = weight(part_s[0][u][16 * rt + i]);
      l_all[rt] += part_s[1][u][16 * rt + i] * f;
      tail_all[rt] += part_s[2][u][16 * rt + i] * f;
    }
    const float f = weight(m[rt]);
#pragma unroll
    for (int t = 0; t < NT; ++t) o[rt][t] *= f;
  }

  // ---- Phase 3: hsum's rows as values, w Q as probabilities ----
  if (first_order) {
    wait_loads<0>();
#pragma unroll
    for (int s1 = 0; s1 < NS; ++s1)
      if (kg == s1 % KG) {                              // uniform over the wave
        f32x4 b[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) b[rt] = q[rt][s1] * (tail_all[rt] / (float)L * p.scale);
        add_values(b, s1 < KG ? ks + PIECE_F : ks);
      }
  }

  // ---- sum over the waves, normalise, store ----
  // o[rt][4 hf + t][r] = channel 64 hf + 4 (4 g + r) + t: unit (rt, hf, r) is 16 bytes a lane, and a wave sums up the units
  // kg, kg + KG, ... over all waves.  Each wave lays its own out in its own stages, which nobody else reads before the barrier.
  constexpr int UNITS = RT * NT;
  static_assert(UNITS * 256 <= WAVE_F, "a wave's output must fit its stages");
  wait_loads<0>();
  wait_lds();
  LDS_PTR(f32x4) board = (LDS_PTR(f32x4))stage_mem;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int hf = 0; hf < NT / 4; ++hf)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        board[kg * (WAVE_F / 4) + ((rt * (NT / 4) + hf) * 4 + r) * 64 + lane] =
            (f32x4){o[rt][4 * hf][r], o[rt][4 * hf + 1][r], o[rt][4 * hf + 2][r], o[rt][4 * hf + 3][r]};
  __syncthreads();
  for (int n = kg; n < UNITS; n += KG) {
    f32x4 sum = board[n * 64 + lane];
#pragma unroll
    for (int u = 1; u < KG; ++u) sum += board[u * (WAVE_F / 4) + n * 64 + lane];
    const int r = n % 4, hf = n / 4 % (NT / 4), rt = n / NT;
    const int q_row = row0 + 16 * rt + i;
    const float lr = RT == 2 && rt == 1 ? l_all[RT - 1] : l_all[0];
    if (q_row < L)
      *reinterpret_cast<f32x4*>(p.out + (bh * (size_t)L + q_row) * D + 64 * hf + 16 * g + 4 * r) = sum * (1.f / lr);
  }
  if (p.lse && g == 0 && kg == 0)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int q_row = row0 + 16 * rt + i;
      if (q_row < L) p.lse[bh * (size_t)L + q_row] = (m_all[rt] + log2f(l_all[rt])) * 0.69314718055994530942f;
    }
}

template <int D, int KG>
__global__ __launch_bounds__(64 * KG, waves_per_simd(D, KG)) void attn_fp32_kernel(P32 p) {
  __shared__ __attribute__((aligned(1024))) float stage[KG * 2 * kPiece * D];
  __shared__ unsigned int chosen[kMaxBlocks / 32];
  __shared__ float part_s[3][KG][32];        // m, l, l_tail of every wave
  // Each XCD gets a contiguous range of (head, row group) items, so that its L2 serves one head; the first n_whole are
  // taken by a workgroup each, the rest by two.
  const int xcd = blockIdx.x % 8, j = blockIdx.x / 8;
  const int nth = j < p.n_whole ? j : p.n_whole + (j - p.n_whole) / 2;
  const int item = xcd * p.per_xcd + nth;
  if (nth >= p.per_xcd || item >= p.total) return;
  const int row0 = item % p.n_groups * 32;
  if (j < p.n_whole) {
    attend_rows<D, 2, KG>(p, item / p.n_groups, row0, stage, chosen, part_s);
  } else {
    const int half0 = row0 + 16 * ((j - p.n_whole) & 1);
    if (half0 < p.L) attend_rows<D, 1, KG>(p, item / p.n_groups, half0, stage, chosen, part_s);
  }
}

template <int D> void launch_d(P32& p, const Dims& dm, hipStream_t stream) {
  p.n_groups = (dm.L + 31) / 32;
  p.total = p.n_groups * dm.bh();
  p.per_xcd = (p.total + 7) / 8;
  // Row groups per XCD, of 32 CUs.  Up to one a CU, eight waves share a group's keys; up to half of that, each half of a
  // group has a CU of its own.  Above, two (head_dim 128) or three workgroups of four waves share a CU, and the groups past
  // the last full round of CUs are taken in halves where both halves of all of them find a CU, because the dispatcher puts
  // the last workgroups on whatever CU is free first, two on one and none on another.  Measured over 110 sizes from 4 to 24
  // heads of 700 to 4 000 rows: with halves 9-13 % faster (r = 0.85) and 11-16 % (dense) where up to 16 groups are left over,
  // slower from there on.  At head_dim 128 all of up to 32 groups past a round of 64 workgroups are halved: 17 .. 32 groups
  // 5 % faster (at head_dim 64, where a CU holds three workgroups, 13 % slower).
  // Eight waves against four, us for the attention step: 2 heads of 2 200 rows 28.6 / 30.4 (dense 88 / 103); past one group a
  // CU 8 of 1 500 38.7 / 31.6 (102 / 94).  Where up to one group a CU walks few pieces, what a workgroup does once is most of its
  // time, and two workgroups of four waves on a CU, half a group each, hide each other's (8 of 700, r = 0.85, nine pieces, eight
  // waves 20.3, four 18.9, four on halves 17.1; 25 pieces 28.8, 30.7, 27.7; 32 28.6 / 28.4; 36 34.8 / 35.9).
  const bool approx = !p.dense && p.k_top < dm.N && p.kbar != nullptr;
  const int pieces = (p.dense ? dm.N : p.k_top) * (dm.B / kPiece) + (approx ? (dm.N + kPiece - 1) / kPiece : 0);
  if (2 * p.per_xcd > kCusPerXcd && p.per_xcd <= kCusPerXcd && pieces <= 32) {
    p.n_whole = 0;
    hipLaunchKernelGGL((attn_fp32_kernel<D, 4>), dim3(8 * 2 * p.per_xcd), dim3(256), 0, stream, p);
  } else if (p.per_xcd <= kCusPerXcd) {
    p.n_whole = 2 * p.per_xcd <= kCusPerXcd ? 0 : p.per_xcd;
    hipLaunchKernelGGL((attn_fp32_kernel<D, 8>), dim3(8 * (2 * p.per_xcd - p.n_whole)), dim3(512), 0, stream, p);
  } else {
    int over = p.per_xcd % kCusPerXcd;
    if (D == 128 && 2 * over > kCusPerXcd) over = p.per_xcd % (2 * kCusPerXcd);
    p.n_whole = over <= (D == 128 ? kCusPerXcd : kCusPerXcd / 2) ? p.per_xcd - over : p.per_xcd;
    hipLaunchKernelGGL((attn_fp32_kernel<D, 4>), dim3(8 * (2 * p.per_xcd - p.n_whole)), dim3(256), 0, stream, p);
  }
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
