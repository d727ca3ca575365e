// Vector-ALU kernels of the Flash-LoRA-Attention library: a partial-attention kernel,
// one workgroup per row and key share, for any dtype, and the split merge +
// epilogue kernel every decode path ends with.
//
// Partial kernel: Alg. 1 (LRAgent, Sec. 3.3) for one query row and one range of
// keys, with the key-side reordering of App. D.1:
//     s_j  = scale * ( q . K_base[j] + (q B_K^T) . L[j] )
//     m, l = online softmax statistics,  O += p_j V_base[j],  O_lr += p_j L[j]
// The epilogue O += O_lr B_V and the division by l (the last two steps of Alg. 1) happen in
// the merge kernel, after the per-split states are combined.
#include <type_traits>

#include "lra_common.h"
#include "lra_decode_util.h"
#include "lra_plan.h"

namespace lra {

// row . vec, the row read in 16-byte pieces where its length and address allow (every lane of these kernels walks
// a row of its own, so a piece is one cache-line touch instead of four or eight)
template <typename T>
__device__ __forceinline__ float dot_row(const T* __restrict__ row, const float* __restrict__ vec, int len) {
  constexpr int PER = 16 / static_cast<int>(sizeof(T));  // elements per piece: 4 (fp32) or 8 (bf16)
  float acc = 0.f;
  if (len % PER == 0 && (reinterpret_cast<uintptr_t>(row) & 15) == 0) {
    for (int c = 0; c < len; c += PER) {
      const uint4 piece = *reinterpret_cast<const uint4*>(row + c);
      const uint32_t w[4] = {piece.x, piece.y, piece.z, piece.w};
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        float x;
        if constexpr (sizeof(T) == 4) x = __uint_as_float(w[e]);
        else x = __uint_as_float((e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
        acc = fmaf(x, vec[c + e], acc);
      }
    }
    return acc;
  }
  for (int c = 0; c < len; ++c) acc = fmaf(to_f32<T>(row[c]), vec[c], acc);
  return acc;
}

// Sequence of query `tok`: the last t with seq_query_start[t] <= tok.
__device__ __forceinline__ int sequence_of_query(const Params& p, int tok) {
  int lo = 0, hi = p.n_seqs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (p.seq_query_start[mid] <= tok) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The elements of a 16-byte piece as floats.
template <typename T, int E>
__device__ __forceinline__ void unpack_piece(uint4 v, float (&x)[E]) {
  static_assert(E * sizeof(T) == 16, "a piece is 16 bytes");
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if constexpr (sizeof(T) == 4) x[e] = __uint_as_float(w[e]);
    else x[e] = __uint_as_float((e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
  }
}

// Lane exchanges on the vector unit: an LDS permute (__shfl) costs its round trip through LDS at every step of a chain.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <typename F>
__device__ __forceinline__ float over_16_lanes(float v, F op) {
  v = op(v, dpp_f32<0x128>(v));  // row_ror:8, 4, 2, 1
  v = op(v, dpp_f32<0x124>(v));
  v = op(v, dpp_f32<0x122>(v));
  return op(v, dpp_f32<0x121>(v));
}
__device__ __forceinline__ float from_lane(float v, int lane) {  // (lane: uniform)
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
// op over the first N lanes' rows of sixteen (N = 16, 32 or 64), in every lane
template <int N, typename F>
__device__ __forceinline__ float over_lanes(float v, F op) {
  v = over_16_lanes(v, op);
  float x = from_lane(v, 0);
#pragma unroll
  for (int i = 16; i < N; i += 16) x = op(x, from_lane(v, i));
  return x;
}

// sum over a quad of lanes, in each of them
__device__ __forceinline__ float sum_quad(float v) {
  v += dpp_f32<0xb1>(v);         // quad_perm [1,0,3,2]
  return v + dpp_f32<0x4e>(v);   // quad_perm [2,3,0,1]
}

// kv_offset / l_offset with the layout known
template <bool PAGED>
__device__ __forceinline__ int64_t kv_row(const Params& p, int t, int j, int h) {
  if constexpr (PAGED) {
    const int blk = p.block_table[static_cast<int64_t>(t) * p.max_blocks_per_seq + (j >> 4)];
    return static_cast<int64_t>(blk) * p.kv_block_stride + static_cast<int64_t>(h) * p.kv_head_stride +
           static_cast<int64_t>(j & 15) * p.kv_token_stride;
  } else {
    return static_cast<int64_t>(j) * p.kv_token_stride + static_cast<int64_t>(h) * p.kv_head_stride;
  }
}
template <bool PAGED>
__device__ __forceinline__ int64_t l_row(const Params& p, int t, int j, int a) {
  const int64_t base = static_cast<int64_t>(a) * p.l_adapter_stride;
  if constexpr (PAGED) {
    const int blk = p.block_table[static_cast<int64_t>(t) * p.max_blocks_per_seq + (j >> 4)];
    return base + (static_cast<int64_t>(blk) * 16 + (j & 15)) * p.l_row_stride;
  } else {
    return base + static_cast<int64_t>(j) * p.l_row_stride;
  }
}

// idx / n for rows of any plan: below 2^23 (and n of at most 4096 heads) a short division
__device__ __forceinline__ int row_div(int idx, int n) {
  if (__builtin_expect(idx >= (1 << 23), 0)) return idx / n;
  return static_cast<int>((static_cast<uint32_t>(idx) & 0x7fffffu) / (static_cast<uint32_t>(n) & 0x1fffu));
}

// (a grid dimension holds fewer than 2^32 threads: rows beyond 2^23 go on in z)
constexpr int kGenericRowBits = 23;

// One workgroup of four waves per (query row, share of the keys), 64 keys per step, sixteen to a wave.  Calls of this
// kernel (fp32, odd ranks) cost round trips and chains of instructions, not bytes.  A wave is on its own from the first
// key to the last: four lanes share a K row (16-byte pieces dealt round robin) and add up by DPP, the wave keeps its own
// softmax reference, a lane sums a column piece of V over every KGW-th of the wave's keys and the ranks of its own L
// pieces over its own key, and only behind the last step do lanes, then waves (in LDS, one barrier) meet.  One barrier
// before the loop hands Qt = q B_K^T round.  The K and L rows of a step are requested under the sums of the one before,
// its V rows as soon as those of the one before are used up, so that three workgroups fit the registers of a compute unit.
// Parameter block, adapter id and length come in one round trip each, the layout and the rank's bound are template
// arguments (13 KB of code otherwise, of which a small call executes a third).  With scores, weights and L rows through LDS
// (two barriers a step, 18 dependent LDS permutes) two agents on 512 fp32 keys took 6.23 us in this kernel, 3.82 so
// (a captured call less its merge; traced by itself 4.5); 1024 new fp32 tokens at 32 heads of 128 1353, 739; 8192 fp32
// keys, 4 agents, 91, 59; 700 new bf16 tokens of rank 12 578, 294.
// K and V rows are 16-byte aligned (bases and strides are checked); L rows of a rank that is no multiple of four
// are not, and are read element by element.
template <typename T, int D, bool PAGED, int RB>
__global__ __launch_bounds__(256, 3) void generic_partial_kernel(Params p) {
  constexpr int E = 16 / static_cast<int>(sizeof(T));  // elements per piece
  constexpr int CG = D / E;                            // pieces per row
  constexpr int PK = CG / 4;                           // pieces of a K row per lane; V rows per lane and step
  constexpr int KGW = 64 / CG;                         // V rows of one request of a wave
  constexpr bool Q_IN_REGS = D == 64;
  constexpr bool L_EARLY = RB == 16;  // (L rows of a step under the sums of the one before; at higher ranks behind them, for the registers)
  constexpr int LN = RB / 4;  // L elements per lane
  // (the large forms: the scheduler kept to one part at a time, or it asks for more registers than three workgroups leave)
  auto part_end = []() __attribute__((always_inline)) {
    if constexpr (RB > 16 && D == 128) __builtin_amdgcn_sched_barrier(0);
  };
  // the parameter block in one round trip (left alone the compiler fetches it piece by piece behind each use)
  asm volatile("" ::"s"(p.q), "s"(p.k_base), "s"(p.v_base), "s"(p.l), "s"(p.b_k), "s"(p.seq_lens), "s"(p.query_adapter));
  asm volatile("" ::"s"(p.kv_token_stride), "s"(p.kv_head_stride), "s"(p.l_row_stride), "s"(p.l_adapter_stride), "s"(p.part_ml), "s"(p.part_o),
               "s"(p.part_lr), "s"(p.part_adapter));
  asm volatile("" ::"s"(p.n_q_heads), "s"(p.n_kv_heads), "s"(p.group), "s"(p.rank), "s"(p.max_seq_len), "s"(p.n_seqs), "s"(p.n_queries),
               "s"(p.n_adapters), "s"(p.n_new), "s"(p.is_prefill), "s"(p.split_keys), "s"(p.n_splits), "s"(p.scale));
  const int split = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Hq = p.n_q_heads, r = p.rank;
  // workgroup -> row: the kv head runs fastest, so that with 8 kv heads an XCD takes the rows of one (200 new tokens
  // on 1200 fp32 keys: 1206 -> 966 us); the longest rows of a prefill come first, so that no long one is left for
  // the end (1024 new tokens, bf16, rank 12: 1140 -> 1103 us)
  const int idx = (static_cast<int>(blockIdx.z) << kGenericRowBits) + static_cast<int>(blockIdx.x);
  if (idx >= (p.is_prefill ? p.n_new : p.n_queries) * Hq) return;
  const int rest = row_div(idx, p.n_kv_heads), h = idx - rest * p.n_kv_heads;
  const int tok_up = row_div(rest, p.group), tok = p.is_prefill ? p.n_new - 1 - tok_up : tok_up;
  const int row = tok * Hq + h * p.group + (rest - tok_up * p.group);

  // (scalar loads, both requested before either is waited for)
  int t, a, n_vis;
  if (p.is_prefill) {
    t = p.seq_index;
    a = p.adapter_index;
    n_vis = min(CONST_I32(p.seq_lens)[t], p.max_seq_len) - p.n_new + tok + 1;
  } else {
    t = p.n_seqs > 1 ? sequence_of_query(p, tok) : 0;
    const int a_raw = CONST_I32(p.query_adapter)[tok], n_t = CONST_I32(p.seq_lens)[t];
    a = min(max(a_raw, 0), p.n_adapters - 1);  // ids are device data: kept inside the table
    n_vis = min(n_t, p.max_seq_len);
  }
  const int64_t slot = static_cast<int64_t>(row) * p.n_splits + split;
  const int j0 = split * p.split_keys;
  const int j1 = min(j0 + p.split_keys, n_vis);
  if (j0 >= j1) {  // nothing visible: (-inf, 0), rows that the merge does not read
    if (tid == 0) {
      p.part_ml[slot * 2 + 0] = -INFINITY;
      p.part_ml[slot * 2 + 1] = 0.f;
      if (split == 0) p.part_adapter[row] = a;
    }
    return;
  }

  __shared__ __align__(16) T q_s[Q_IN_REGS ? 1 : D];
  __shared__ float qt_s[64];
  __shared__ __align__(16) float o_s[4][D];
  __shared__ float olr_s[4][64];
  __shared__ float m_s[4], ell_s[4];

  const T* kb = static_cast<const T*>(p.k_base);
  const T* vb = static_cast<const T*>(p.v_base);
  const T* lr = static_cast<const T*>(p.l);
  const int quarter = lane & 3, key_k = 16 * wave + (lane >> 2);  // score part: this lane's K row of the step, and its quarter
  const int cg = lane % CG, kg = lane / CG;                       // sum part: column piece, first of the wave's keys (kg, kg + KGW, ...)

  uint4 kp[PK], vp[PK];
  T lv[LN];
  // (rows past the end: the last one again, weighted zero)
  auto request_v = [&](int jb) __attribute__((always_inline)) {
    int jk = jb + 16 * wave + kg;
    if constexpr (RB > 16) asm volatile("" : "+v"(jk));  // (row numbers formed again in each step, not held in registers)
#pragma unroll
    for (int i = 0; i < PK; ++i)
      vp[i] = reinterpret_cast<const uint4*>(vb + kv_row<PAGED>(p, t, min(jk + KGW * i, j1 - 1), h))[cg];
  };
  auto request_k = [&](int jb) __attribute__((always_inline)) {
    const uint4* krow = reinterpret_cast<const uint4*>(kb + kv_row<PAGED>(p, t, min(jb + key_k, j1 - 1), h));
#pragma unroll
    for (int i = 0; i < PK; ++i) kp[i] = krow[quarter + 4 * i];
  };
  auto request_l = [&](int jb) __attribute__((always_inline)) {
    const T* lrow = lr + l_row<PAGED>(p, t, min(jb + key_k, j1 - 1), a);
    int q4 = quarter;
    if constexpr (!L_EARLY) asm volatile("" : "+v"(q4));  // (sixteen offsets formed again in each step, not held in registers)
#pragma unroll
    for (int i = 0; i < LN; ++i) {
      lv[i] = lrow[min(4 * i + q4, r - 1)];  // (ranks beyond the last: zeroed below)
      if ((i & 3) == 3) part_end();
    }
  };
  const uint4* qrow = reinterpret_cast<const uint4*>(static_cast<const T*>(p.q) + static_cast<int64_t>(row) * D);
  uint4 qp[PK];
#pragma unroll
  for (int i = 0; i < PK; ++i) qp[i] = qrow[quarter + 4 * i];
  uint4 bp[PK];
  request_k(j0);
  part_end();
  request_l(j0);
  // row key_k of B_K for this kv head, a quarter of it (without a key-side adapter: q again, times zero below)
  const bool has_bk = p.b_k != nullptr;
  {
    const T* base = has_bk ? static_cast<const T*>(p.b_k) + (static_cast<int64_t>(a) * r * p.n_kv_heads + h) * D : reinterpret_cast<const T*>(qrow);
    int64_t ld = has_bk ? static_cast<int64_t>(p.n_kv_heads) * D : 0;
    asm volatile("" : "+s"(base), "+s"(ld));  // (otherwise the loads of the two cases are told apart, under a branch and with waits)
    const auto* brow = (const __attribute__((address_space(1))) u32x4*)(base + min(key_k, r - 1) * ld);
#pragma unroll
    for (int i = 0; i < PK; ++i) bp[i] = __builtin_bit_cast(uint4, u32x4(brow[quarter + 4 * i]));
  }
  request_v(j0);
  part_end();
  auto dot_pieces = [&](const uint4 (&pc)[PK], auto q_piece) __attribute__((always_inline)) -> float {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < PK; ++i) {
      float x[E], y[E];
      unpack_piece<T, E>(pc[i], x);
      unpack_piece<T, E>(q_piece(i), y);
#pragma unroll
      for (int e = 0; e < E; ++e) acc = fmaf(x[e], y[e], acc);
      if ((i & 3) == 3) part_end();
    }
    return acc;
  };
  if constexpr (!Q_IN_REGS) {
    if (tid < 4) {
#pragma unroll
      for (int i = 0; i < PK; ++i) reinterpret_cast<uint4*>(q_s)[quarter + 4 * i] = qp[i];
    }
  }
  {
    const float qt = sum_quad(dot_pieces(bp, [&](int i) { return qp[i]; }));
    if (quarter == 0) qt_s[key_k] = has_bk && key_k < r ? qt : 0.f;
  }
  __syncthreads();

  float m = -INFINITY, ell = 0.f, o[E], olr[LN];  // (ell, o, olr: this lane's part)
#pragma unroll
  for (int e = 0; e < E; ++e) o[e] = 0.f;
#pragma unroll
  for (int i = 0; i < LN; ++i) olr[i] = 0.f;
  for (int jb = j0; jb < j1; jb += kWave) {
    const int cnt = j1 - jb - 16 * wave;  // this wave's keys of the step (sixteen and more: all)
    if (cnt <= 0) break;
    const bool mine = (lane >> 2) < cnt;
    int q4 = quarter;
    if constexpr (RB > 16) asm volatile("" : "+v"(q4));  // (q and Qt read from LDS in each step, not held in registers)
    float part = dot_pieces(kp, [&](int i) {
      if constexpr (Q_IN_REGS) return qp[i];
      else return reinterpret_cast<const uint4*>(q_s)[q4 + 4 * i];
    });
    T x[LN];  // this lane's L elements, zero past the end and past the rank (the next rows take lv under the sums)
#pragma unroll
    for (int i = 0; i < LN; ++i) {
      if (!(4 * i + q4 < r && mine)) lv[i] = T(0);
      if constexpr (L_EARLY) x[i] = lv[i];
      part = fmaf(to_f32<T>(lv[i]), qt_s[4 * i + q4], part);
    }
    part = p.scale * sum_quad(part);
    asm volatile("" : "+v"(part));  // (or the whole product moves under a branch on the lanes whose key exists)
    part_end();
    const float s = mine ? part : -INFINITY;
    const bool more = jb + kWave < j1;
    if (more) request_k(jb + kWave);
    if (more && L_EARLY) request_l(jb + kWave);
    part_end();
    const float m_new = fmaxf(m, over_lanes<64>(s, [](float u, float v) { return fmaxf(u, v); }));
    const float alpha = (m == -INFINITY) ? 0.f : expf(m - m_new);
    // past the end: zero; a score of minus infinity likewise, also where all sixteen are and m_new with them (NaN stays NaN)
    const float pj = s == -INFINITY ? 0.f : expf(s - m_new);
    ell = fmaf(alpha, ell, quarter == 0 ? pj : 0.f);
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] *= alpha;
    if (cnt < 16) {  // (a row requested again stays out of the sums, whatever it holds)
#pragma unroll
      for (int i = 0; i < PK; ++i)
        if (kg >= cnt - KGW * i) vp[i] = make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int i = 0; i < PK; ++i) {
      const float pk = __shfl(pj, 4 * (kg + KGW * i), kWave);
      float v[E];
      unpack_piece<T, E>(vp[i], v);
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = fmaf(pk, v[e], o[e]);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) asm volatile("" : "+v"(o[e]));  // (or the sums sink behind the requests, with a copy of every row)
    part_end();
    if (more) request_v(jb + kWave);
    part_end();
#pragma unroll
    for (int i = 0; i < LN; ++i) olr[i] = fmaf(alpha, olr[i], pj * to_f32<T>(L_EARLY ? x[i] : lv[i]));
    if (more && !L_EARLY) request_l(jb + kWave);
    part_end();
    m = m_new;
  }

  // ---- lanes of a wave, then the waves ----
  auto over_rows = [&](float v) __attribute__((always_inline)) -> float {  // over the lanes with the same index mod 16
    return sum_over_lane_groups(v);
  };
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if constexpr (CG == 8) o[e] += dpp_f32<0x128>(o[e]);  // row_ror:8
    if constexpr (CG <= 16) o[e] = over_rows(o[e]);
    else {
      float other = o[e];
      permlane32_swap(o[e], other);
      o[e] += other;
    }
  }
  part_end();
  if (lane < CG) {
#pragma unroll
    for (int e = 0; e < E; ++e) o_s[wave][cg * E + e] = o[e];
  }
#pragma unroll
  for (int i = 0; i < LN; ++i)
    if (RB == 16 || 4 * i < r) {  // (uniform)
      float v = olr[i];
      v += dpp_f32<0x124>(v);  // row_ror:4, 8: the keys of a row of sixteen lanes
      v += dpp_f32<0x128>(v);
      v = over_rows(v);
      if (lane < 4) olr_s[wave][4 * i + lane] = v;
    }
  ell = over_lanes<64>(ell, [](float u, float v) { return u + v; });
  if (lane == 0) {
    m_s[wave] = m;
    ell_s[wave] = ell;
  }
  __syncthreads();
  const float m_all = fmaxf(fmaxf(m_s[0], m_s[1]), fmaxf(m_s[2], m_s[3]));
  float f[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) f[w] = m_s[w] == -INFINITY ? 0.f : expf(m_s[w] - m_all);
  if (tid < D) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) v = fmaf(f[w], o_s[w][tid], v);
    p.part_o[slot * D + tid] = v;
  }
  const int rho = tid - (256 - 64);  // (the last wave, which has no columns at d = 128)
  if (rho >= 0 && rho < r) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) v = fmaf(f[w], olr_s[w][rho], v);
    p.part_lr[slot * r + rho] = v;
  }
  if (tid == 128) {
    float l_all = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) l_all = fmaf(f[w], ell_s[w], l_all);
    p.part_ml[slot * 2 + 0] = m_all;
    p.part_ml[slot * 2 + 1] = l_all;
    if (split == 0) p.part_adapter[row] = a;
  }
}

// The same for the rotary key side (App. D.1 with the rotation in place: LoRA on the key
// projection of a model with rotary embeddings).  K_j = K_base,j + RoPE_j(L_j B_K): the
// rotation sits between L_j B_K and the score, so (q B_K^T) . L_j no longer applies.  With
// rotate-half pairs (i, i + h), h = d/2, and c_i, s_i the cosine and sine of j * theta^(-2i/d),
//     q . RoPE_j(L_j B) = sum_i  c_i (L_j . U_i) + s_i (L_j . W_i),
//     U_i[rho] = q_i B[rho][i] + q_{i+h} B[rho][i+h],   W_i[rho] = q_{i+h} B[rho][i] - q_i B[rho][i+h],
// r-vectors per pair that depend on the query row only.  The wave forms U and W once in LDS,
// stages the L rows of its 64 keys there as well, and every lane (one key) sums over the
// pairs.  r * d multiply-adds per (row, key) instead of d + r: the price of the rotation
// without materialising the keys.  Angles as in the cache-append producer: rates in double
// precision and revolutions, fractional part, v_sin_f32 / v_cos_f32.
template <typename T>
__global__ __launch_bounds__(kWave) void generic_partial_rope_kernel(Params p) {
  const int row = blockIdx.x;
  const int split = blockIdx.y;
  const int lane = threadIdx.x;
  const int Hq = p.n_q_heads, d = p.head_dim, r = p.rank, half = d / 2;
  const int tok = row / Hq;
  const int g = row - tok * Hq;
  const int h = g / p.group;

  int t, a, n_vis;
  if (p.is_prefill) {
    t = p.seq_index;
    a = p.adapter_index;
    const int n_t = min(p.seq_lens[t], p.max_seq_len);
    n_vis = n_t - p.n_new + tok + 1;
  } else {
    t = sequence_of_query(p, tok);
    a = min(max(p.query_adapter[tok], 0), p.n_adapters - 1);  // ids are device data: kept inside the table
    n_vis = min(p.seq_lens[t], p.max_seq_len);
  }
  const int j0 = split * p.split_keys;
  const int j1 = min(j0 + p.split_keys, n_vis);

  __shared__ float q_s[128];
  __shared__ float u_s[64 * 64];   // [rho][i], i < d/2
  __shared__ float w_s[64 * 64];
  __shared__ float l_s[64 * 65];   // [key of the step][rho], rows padded to 65 floats
  __shared__ double rate_s[64];    // revolutions per position of pair i
  const T* q = static_cast<const T*>(p.q) + static_cast<int64_t>(row) * d;
  for (int c = lane; c < d; c += kWave) q_s[c] = to_f32<T>(q[c]);
  if (lane < half)
    rate_s[lane] = exp2(-2.0 * lane / d * log2(static_cast<double>(p.key_rope_theta))) * 0.15915494309189533577;
  __syncthreads();
  {
    const T* bk = static_cast<const T*>(p.b_k) + static_cast<int64_t>(a) * r * (static_cast<int64_t>(p.n_kv_heads) * d) + h * d;
    for (int e = lane; e < r * half; e += kWave) {
      const int rho = e / half, i = e - rho * half;
      const float b_lo = to_f32<T>(bk[static_cast<int64_t>(rho) * p.n_kv_heads * d + i]);
      const float b_hi = to_f32<T>(bk[static_cast<int64_t>(rho) * p.n_kv_heads * d + i + half]);
      u_s[rho * 64 + i] = q_s[i] * b_lo + q_s[i + half] * b_hi;
      w_s[rho * 64 + i] = q_s[i + half] * b_lo - q_s[i] * b_hi;
    }
  }
  __syncthreads();

  const T* kb = static_cast<const T*>(p.k_base);
  const T* vb = static_cast<const T*>(p.v_base);
  const T* lr = static_cast<const T*>(p.l);

  float m = -INFINITY, ell = 0.f, o0 = 0.f, o1 = 0.f, olr = 0.f;
  for (int jb = j0; jb < j1; jb += kWave) {
    const int j = jb + lane;
    const bool valid = j < j1;
    // this lane's L row, as floats, where the lane can index it with a loop variable
    if (valid) {
      const T* lrow = lr + l_offset(p, t, j, a);
      for (int rho = 0; rho < r; ++rho) l_s[lane * 65 + rho] = to_f32<T>(lrow[rho]);
    }
    __syncthreads();  // one wave: orders the staging against the other lanes' reads below
    float s = -INFINITY;
    if (valid) {
      const float sk = dot_row<T>(kb + kv_offset(p, t, j, h), q_s, d);
      float sl = 0.f;
      for (int i = 0; i < half; ++i) {
        float u = 0.f, w = 0.f;
        for (int rho = 0; rho < r; ++rho) {
          const float lv = l_s[lane * 65 + rho];
          u = fmaf(lv, u_s[rho * 64 + i], u);
          w = fmaf(lv, w_s[rho * 64 + i], w);
        }
        double rev = static_cast<double>(j) * rate_s[i];
        rev -= floor(rev);
        const float fr = static_cast<float>(rev);
        sl = fmaf(__builtin_amdgcn_cosf(fr), u, fmaf(__builtin_amdgcn_sinf(fr), w, sl));
      }
      s = p.scale * (sk + sl);
    }
    const float m_new = fmaxf(m, wave_max(s));  // finite: lane 0 is always valid here
    const float alpha = (m == -INFINITY) ? 0.f : expf(m - m_new);
    const float pj = valid ? expf(s - m_new) : 0.f;
    ell = alpha * ell + wave_sum(pj);
    o0 *= alpha;
    o1 *= alpha;
    olr *= alpha;
    // (as in generic_partial_kernel: the V rows of eight keys requested before the first is used)
    const int cnt = min(kWave, j1 - jb);
    const int c0 = min(lane, d - 1), c1 = min(lane + kWave, d - 1);
    for (int jj0 = 0; jj0 < cnt; jj0 += 8) {
      float v0[8], v1[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const T* v = vb + kv_offset(p, t, jb + min(jj0 + u, cnt - 1), h);
        v0[u] = to_f32<T>(v[c0]);
        v1[u] = to_f32<T>(v[c1]);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (jj0 + u < cnt) {  // (uniform)
          const float pjj = __shfl(pj, jj0 + u, kWave);
          o0 = fmaf(pjj, v0[u], o0);
          o1 = fmaf(pjj, v1[u], o1);
          if (lane < r) olr = fmaf(pjj, l_s[(jj0 + u) * 65 + lane], olr);
        }
      }
    }
    m = m_new;
    __syncthreads();  // before the next step overwrites the staged rows
  }

  const int64_t slot = static_cast<int64_t>(row) * p.n_splits + split;
  if (lane == 0) {
    p.part_ml[slot * 2 + 0] = m;  // a split past the row's last visible key leaves (-inf, 0)
    p.part_ml[slot * 2 + 1] = ell;
    if (split == 0) p.part_adapter[row] = a;
  }
  if (lane < d) p.part_o[slot * d + lane] = o0;
  if (lane + kWave < d) p.part_o[slot * d + lane + kWave] = o1;
  if (lane < r) p.part_lr[slot * r + lane] = olr;
}

// Flash-decoding merge of the per-split states followed by Alg. 1's epilogue:
//   M = max_s m_s, w_s = exp(m_s - M), l = sum w_s l_s, O = sum w_s O_s,
//   O_lr = sum w_s O_lr,s ;  out = (O + O_lr B_V) / l.
// One workgroup of 128 x kMergeGroups threads per query row.  Thread (c, g) owns
// column c of the splits s = g, g + kMergeGroups, ... and, for the epilogue, the
// B_V rows rho = g, g + kMergeGroups, ...  All of a thread's global loads (split
// statistics, partial rows, B_V) are issued before the first one is consumed, so
// the kernel costs about two memory round trips.  Groups are added in a fixed
// order: the result does not depend on which workgroup of the first kernel
// finished first.
constexpr int kMergeUnroll = 8;  // splits per thread and pass

#ifdef LRA_TIMING
#define LRA_MSTAMP(k) do { unsigned long long t_; asm volatile("s_waitcnt lgkmcnt(0)\n\ts_memrealtime %0\n\ts_waitcnt lgkmcnt(0)" : "=s"(t_)); mt[k] = t_; } while (0)
#else
#define LRA_MSTAMP(k)
#endif

template <typename T, int kMergeGroups>
__global__ __launch_bounds__(128 * kMergeGroups) void merge_kernel(Params p) {
#ifdef LRA_TIMING
  unsigned long long mt[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#endif
  LRA_MSTAMP(0);
  // Workgroups go round-robin over the XCDs; numbering them kv head first puts the rows of
  // kv head h on the XCD(s) where the streaming kernel wrote that head's partial states.
  const int Hq = p.n_q_heads, d = p.head_dim, r = p.rank;
  const int h = blockIdx.x % p.n_kv_heads;
  const int rest = blockIdx.x / p.n_kv_heads;
  const int tok = rest / p.group;
  const int g = h * p.group + rest % p.group;
  const int row = tok * Hq + g;
  const int c = threadIdx.x, gq = threadIdx.y;
  const int tid = gq * 128 + c;
  // Everything this kernel needs was left in the workspace by the first kernel: the row's
  // adapter, and a zero row sum in every split that had no visible key (its O and O_lr rows
  // were never written and are ignored below).  No sequence table is read here.
  const int ns = p.n_splits;
  // (clamped: whatever the workspace holds, the B_V rows read below exist)
  const int a = min(max(p.part_adapter[row], 0), p.n_adapters - 1);
#ifdef LRA_TIMING
  asm volatile("" ::"v"(a));
#endif
  LRA_MSTAMP(1);
  const int64_t slot0 = static_cast<int64_t>(row) * p.n_splits;
  const float2* ml = reinterpret_cast<const float2*>(p.part_ml) + slot0;
  const float* po = p.part_o + slot0 * d + c;
  const float* pl = p.part_lr + slot0 * r + c;
  const bool col_o = c < d, col_l = c < r;

  __shared__ float red[2 * kMergeGroups];
  __shared__ float o_sh[kMergeGroups][128];
  __shared__ float olr_sh[kMergeGroups][64];
  __shared__ float ell_sh[kMergeGroups];

  // ---- issue: statistics for the row maximum, first pass of partial rows, B_V rows ----
  float big = -INFINITY;
  for (int s = tid; s < ns; s += 128 * kMergeGroups) {
    const float2 v = ml[s];
    if (v.y > 0.f) big = fmaxf(big, v.x);
  }
  float2 st[kMergeUnroll];
  float xo[kMergeUnroll], xl[kMergeUnroll];
#pragma unroll
  for (int i = 0; i < kMergeUnroll; ++i) {
    const int s = i * kMergeGroups + gq;
    const bool ok = s < ns;
    st[i] = ok ? ml[s] : make_float2(0.f, 0.f);
    xo[i] = (ok && col_o) ? po[static_cast<int64_t>(s) * d] : 0.f;
    xl[i] = (ok && col_l) ? pl[static_cast<int64_t>(s) * r] : 0.f;
  }
  float bvv[64 / kMergeGroups];
  {
    const int64_t ld = static_cast<int64_t>(p.n_kv_heads) * d;
    const T* bv = static_cast<const T*>(p.b_v) + static_cast<int64_t>(a) * r * ld + h * d + c;
#pragma unroll
    for (int i = 0; i < 64 / kMergeGroups; ++i) {
      const int rho = i * kMergeGroups + gq;
      bvv[i] = (p.b_v != nullptr && col_o && rho < r) ? to_f32<T>(bv[rho * ld]) : 0.f;
    }
  }

  LRA_MSTAMP(2);
  big = wave_max(big);
  if ((tid & 63) == 0) red[tid >> 6] = big;
  __syncthreads();
  LRA_MSTAMP(3);
  big = red[0];
#pragma unroll
  for (int i = 1; i < 2 * kMergeGroups; ++i) big = fmaxf(big, red[i]);

  float ell = 0.f, o = 0.f, olr = 0.f;
#pragma unroll
  for (int i = 0; i < kMergeUnroll; ++i) {
    const bool live = st[i].y > 0.f;
    const float w = live ? expf(st[i].x - big) : 0.f;
    ell = fmaf(w, st[i].y, ell);
    o = fmaf(w, live ? xo[i] : 0.f, o);
    olr = fmaf(w, live ? xl[i] : 0.f, olr);
  }
  // further passes, only for more than kMergeGroups * kMergeUnroll splits
  for (int s = kMergeGroups * kMergeUnroll + gq; s < ns; s += kMergeGroups) {
    const float2 v = ml[s];
    const float x = col_o ? po[static_cast<int64_t>(s) * d] : 0.f;
    const float y = col_l ? pl[static_cast<int64_t>(s) * r] : 0.f;
    const bool live = v.y > 0.f;
    const float w = live ? expf(v.x - big) : 0.f;
    ell = fmaf(w, v.y, ell);
    o = fmaf(w, live ? x : 0.f, o);
    olr = fmaf(w, live ? y : 0.f, olr);
  }
  if (c < 64) olr_sh[gq][c] = olr;
  if (c == 0) ell_sh[gq] = ell;
  LRA_MSTAMP(4);
  __syncthreads();
  // epilogue O += O_lr B_V: group g contributes its rows rho = g, g + kMergeGroups, ...
#pragma unroll
  for (int i = 0; i < 64 / kMergeGroups; ++i) {
    const int rho = i * kMergeGroups + gq;
    if (rho < r) {
      float x = olr_sh[0][rho];
#pragma unroll
      for (int k = 1; k < kMergeGroups; ++k) x += olr_sh[k][rho];
      o = fmaf(x, bvv[i], o);
    }
  }
  o_sh[gq][c] = o;
  __syncthreads();
  if (gq == 0 && col_o) {
    o = o_sh[0][c];
    ell = ell_sh[0];
#pragma unroll
    for (int k = 1; k < kMergeGroups; ++k) {
      o += o_sh[k][c];
      ell += ell_sh[k];
    }
    static_cast<T*>(p.out)[static_cast<int64_t>(row) * d + c] = from_f32<T>(o / ell);
  }
  LRA_MSTAMP(5);
#ifdef LRA_TIMING
  if (p.timing && (tid & 63) == 0) {
    unsigned long long* o_ = p.timing + 4096 * 128 + static_cast<size_t>(blockIdx.x) * 64 + (tid >> 6) * 8;
    for (int i_ = 0; i_ < 6; ++i_) o_[i_] = mt[i_];
  }
#endif
}

// The same merge for the common case (head dimension 64 or 128, rank a multiple of 4, at most 64 splits): one workgroup
// of four waves per query row.  The launch is a chain of latencies (parameter block, the row's adapter id, the loads, one
// barrier), so nothing may stand between them:
//   - the parameter block is fetched in one round trip (left alone the compiler fetches it piece by piece behind each
//     use), the grid is (kv head, q head of the group, query) so that no index needs a division, and every load is
//     unconditional from a clamped index (a load under a condition, with zero as the other value, makes the compiler
//     wait for it on the spot); what a clamped index fetched in vain gets weight zero;
//   - wave w sums the splits w, w + 4, ...: addresses and weights are scalars (v_readlane), lane = column (pair at d = 128);
//   - lane = split for the statistics, every wave forms the weights w_s on its own by DPP, without LDS;
//   - the waves' sums meet in LDS behind the only barrier; then a wave finishes a quarter of the columns, sixteen lanes of
//     which each take a quarter of the ranks, with their B_V elements in registers since before the barrier.
// With weights by ds_bpermute (24 dependent ones), a branch per split and three barriers the launch took 3.57 us behind the
// headline decode's first kernel, 2.40 so (3.09 and 2.11 behind the fp32 one); a launch that only adds the same parts takes 2.2
// (all of captured calls, with the merge less without; traced by itself the kernel takes 3.6 and 2.7, its start and end included).
// NS, RB: bounds of splits and rank (16, 32 or 64).  Every sum runs in a fixed order, so the result does not depend on
// which workgroup of the first kernel finished first.
template <typename T, int D, int NS, int RB>
__global__ __launch_bounds__(256) void merge_rows_kernel(Params p) {
  constexpr int CPL = D / 64;  // columns per lane
  constexpr int OPW = NS / 4;  // splits per wave
  constexpr int RPT = RB / 4;  // ranks per thread of the epilogue
  asm volatile("" ::"s"(p.part_adapter), "s"(p.part_ml), "s"(p.part_o), "s"(p.part_lr), "s"(p.b_v), "s"(p.out));
  asm volatile("" ::"s"(p.n_q_heads), "s"(p.n_kv_heads), "s"(p.group), "s"(p.head_dim), "s"(p.rank), "s"(p.n_splits),
               "s"(p.n_adapters));
  const int Hq = p.n_q_heads, r = p.rank, ns = p.n_splits;
  const int h = blockIdx.x;
  const int row = static_cast<int>(blockIdx.z) * Hq + h * p.group + static_cast<int>(blockIdx.y);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t slot0 = static_cast<int64_t>(row) * ns;

  __shared__ __align__(16) float o_sh[4][D];
  __shared__ __align__(16) float lr_sh[64][4];  // [rank][wave]

  // the row's adapter first: the B_V rows depend on it (requested here by hand and waited for where the B_V addresses are
  // formed: left to the compiler the request sinks below the vector loads, and its round trip is then paid after theirs)
  int a_raw;
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(a_raw) : "s"(p.part_adapter + row));

  // ---- issue everything ----
  const float2 st_raw = reinterpret_cast<const float2*>(p.part_ml)[slot0 + min(lane, ns - 1)];
  float xo[OPW][CPL], xl[OPW];
#pragma unroll
  for (int k = 0; k < OPW; ++k) {
    const float* po = p.part_o + (slot0 + min(wave + 4 * k, ns - 1)) * D;
    if constexpr (CPL == 2) {
      const float2 v = reinterpret_cast<const float2*>(po)[lane];
      xo[k][0] = v.x;
      xo[k][CPL - 1] = v.y;
    } else {
      xo[k][0] = po[lane];
    }
  }
  const int rl = min(lane, r - 1);  // (lanes beyond the rank: sums that are never read)
#pragma unroll
  for (int k = 0; k < OPW; ++k) xl[k] = (p.part_lr + (slot0 + min(wave + 4 * k, ns - 1)) * r)[rl];
  // epilogue: columns c .. c + CPL - 1 of this wave's quarter, ranks rq, rq + 4, ...
  const int c = wave * (D / 4) + (lane & 15) * CPL, rq = lane >> 4;
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(a_raw));
  const int a = min(max(a_raw, 0), p.n_adapters - 1);  // (clamped: whatever the workspace holds, the rows read below exist)
  typedef typename std::conditional<sizeof(T) * CPL == 8, float2, typename std::conditional<sizeof(T) * CPL == 4, uint32_t, T>::type>::type BvPiece;
  BvPiece bvp[RPT];
  // (Requesting the slices of all adapters of a small table next to the partial rows, to pick the row's
  // own when its id arrives, takes one dependent round trip off the path and was measured 0.8 us slower.)
  const bool has_bv = p.b_v != nullptr;  // (uniform)
  if (has_bv) {
    const int64_t ld = static_cast<int64_t>(p.n_kv_heads) * D;
    const T* bv = static_cast<const T*>(p.b_v) + static_cast<int64_t>(a) * r * ld + h * D;
    const uint32_t ldb = static_cast<uint32_t>(ld);
#pragma unroll
    for (int i = 0; i < RPT; ++i)  // (ranks beyond the last: fetched again, left out below)
      bvp[i] = *reinterpret_cast<const BvPiece*>(bv + (static_cast<uint32_t>(min(4 * i + rq, r - 1)) * ldb + static_cast<uint32_t>(c)));
  }

  // ---- weights (per wave, lane = split) ----
  // (a share without a visible key left a zero row sum; its rows were never written)
  const bool live = lane < ns && st_raw.y > 0.f;
  const float big = over_lanes<NS>(live ? st_raw.x : -INFINITY, [](float x, float y) { return fmaxf(x, y); });
  const float w = live ? expf(st_raw.x - big) : 0.f;
  const float ell = over_lanes<NS>(lane < ns ? w * st_raw.y : 0.f, [](float x, float y) { return x + y; });  // (a share's NaN is the row's)

  // ---- weighted sums of this wave's splits ----
  float o[CPL], olr = 0.f;
#pragma unroll
  for (int e = 0; e < CPL; ++e) o[e] = 0.f;
#pragma unroll
  for (int k = 0; k < OPW; ++k) {
    const float wk = from_lane(w, wave + 4 * k);
    const bool in = wk > 0.f;  // also keeps whatever an unwritten row holds out of the sums
#pragma unroll
    for (int e = 0; e < CPL; ++e) o[e] = fmaf(wk, in ? xo[k][e] : 0.f, o[e]);
    olr = fmaf(wk, in ? xl[k] : 0.f, olr);
  }
#pragma unroll
  for (int e = 0; e < CPL; ++e) o_sh[wave][lane * CPL + e] = o[e];
  lr_sh[lane][wave] = lane < r ? olr : 0.f;
  __syncthreads();

  // ---- O += O_lr B_V, division, store ----
  float x[CPL];
#pragma unroll
  for (int e = 0; e < CPL; ++e) x[e] = o_sh[rq][c + e];  // (each quarter of the lanes brings one wave's sums)
  if (has_bv) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      if (4 * i >= r) break;  // (uniform; a fetched-again row of infinities stays out)
      const float4 l4 = *reinterpret_cast<const float4*>(lr_sh[4 * i + rq]);
      const float lv = (l4.x + l4.y) + (l4.z + l4.w);
      if constexpr (sizeof(T) * CPL == 8) {
        x[0] = fmaf(lv, bvp[i].x, x[0]);
        x[CPL - 1] = fmaf(lv, bvp[i].y, x[CPL - 1]);
      } else if constexpr (sizeof(T) == 2 && CPL == 2) {
        x[0] = fmaf(lv, __uint_as_float(bvp[i] << 16), x[0]);
        x[CPL - 1] = fmaf(lv, __uint_as_float(bvp[i] & 0xffff0000u), x[CPL - 1]);
      } else if constexpr (sizeof(T) == 2) {
        x[0] = fmaf(lv, bf16_to_f32(static_cast<bf16_t>(bvp[i])), x[0]);
      } else {
        x[0] = fmaf(lv, __builtin_bit_cast(float, bvp[i]), x[0]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < CPL; ++e) {
    float lo = x[e], hi = x[e];
    permlane16_swap(lo, hi);
    lo += hi;
    hi = lo;
    permlane32_swap(lo, hi);
    x[e] = (lo + hi) / ell;
  }
  if (rq == 0) {
    T* out = static_cast<T*>(p.out) + static_cast<int64_t>(row) * D + c;
    if constexpr (sizeof(T) == 2 && CPL == 2) {
      *reinterpret_cast<uint32_t*>(out) = pack_bf16x2(x[0], x[CPL - 1]);
    } else {
#pragma unroll
      for (int e = 0; e < CPL; ++e) out[e] = from_f32<T>(x[e]);
    }
  }
}

// The same merge for calls with many rows: one wave per row (four rows, q heads of one kv
// head, per workgroup), no LDS and no barrier, so that a CU holds twenty rows' worth of loads
// in flight instead of four.  Lane = split for the statistics (at most 64 splits), lane =
// column (pair of columns at d = 128) for the rows; the weight of a split and the entries of
// O_lr travel by v_readlane.  Splits are added in index order, four or eight requested at a time, up to the last
// one that holds a visible key (in a ragged batch most rows have fewer shares than the grid).
template <typename T, int D, int RB, int U>
__global__ __launch_bounds__(256) void merge_wave_kernel(Params p) {
  constexpr int CPL = D / 64;   // columns per lane: c = CPL * lane + k
  constexpr int SPL = 64 / RB;  // splits whose O_lr entries one load brings: four, or one above rank 16
  static_assert(SPL == 4 || SPL == 1, "how their lanes are added up");
  // (as in merge_rows_kernel: the parameter block in one round trip, a grid (kv head, group of four q
  // heads, query) without divisions, the adapter id requested by hand ahead of the vector loads, and
  // unconditional loads from clamped indices)
  asm volatile("" ::"s"(p.part_adapter), "s"(p.part_ml), "s"(p.part_o), "s"(p.part_lr), "s"(p.b_v), "s"(p.out));
  asm volatile("" ::"s"(p.n_q_heads), "s"(p.n_kv_heads), "s"(p.group), "s"(p.head_dim), "s"(p.rank), "s"(p.n_splits),
               "s"(p.n_adapters));
  const int Hq = p.n_q_heads, r = p.rank, G = p.group;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = blockIdx.x;
  const int gq = static_cast<int>(blockIdx.y) * 4 + wave;
  if (gq >= G) return;
  const int row = static_cast<int>(blockIdx.z) * Hq + h * G + gq;
  const int ns = p.n_splits;
  const int64_t slot0 = static_cast<int64_t>(row) * ns;
  int a_raw;
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(a_raw) : "s"(p.part_adapter + row));
  const float2 st_raw = reinterpret_cast<const float2*>(p.part_ml)[slot0 + min(lane, ns - 1)];

  const float* po = p.part_o + slot0 * D;
  const float* pl = p.part_lr + slot0 * r + min(lane % RB, r - 1);  // (lanes beyond the rank: sums that are never read)
  const int y_split = lane / RB;
  float x[U][CPL], y[U / SPL];
  auto request = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int sidx = min(s0 + u, ns - 1);
      if constexpr (CPL == 2) {
        const float2 v = reinterpret_cast<const float2*>(po + sidx * D)[lane];
        x[u][0] = v.x;
        x[u][CPL - 1] = v.y;
      } else {
        x[u][0] = (po + sidx * D)[lane];
      }
    }
#pragma unroll
    for (int k = 0; k < U / SPL; ++k) y[k] = pl[min(s0 + k * SPL + y_split, ns - 1) * r];
  };
  request(0);
  // this wave's column pairs of B_V, requested behind the first partial rows
  typedef typename std::conditional<sizeof(T) * CPL == 8, float2, typename std::conditional<sizeof(T) * CPL == 4, uint32_t, T>::type>::type BvPiece;
  constexpr int BN = RB < 32 ? RB : 32;  // rows at a time
  BvPiece bvp[BN];
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(a_raw));
  const int a = min(max(a_raw, 0), p.n_adapters - 1);
  const bool has_bv = p.b_v != nullptr;  // (uniform)
  const int64_t ld = static_cast<int64_t>(p.n_kv_heads) * D;
  const T* bv = static_cast<const T*>(p.b_v) + static_cast<int64_t>(a) * r * ld + h * D;
  auto request_bv = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < BN; ++i)  // (ranks beyond the last: fetched again, left out below)
      bvp[i] = reinterpret_cast<const BvPiece*>(bv + min(r0 + i, r - 1) * ld)[lane];
  };
  if (has_bv) request_bv(0);

  // (a share without a visible key left a zero row sum; its rows were never written)
  const bool live = lane < ns && st_raw.y > 0.f;
  const float big = over_lanes<64>(live ? st_raw.x : -INFINITY, [](float u, float v) { return fmaxf(u, v); });
  const float w = live ? expf(st_raw.x - big) : 0.f;
  const float ell = over_lanes<64>(lane < ns ? w * st_raw.y : 0.f, [](float u, float v) { return u + v; });  // (a share's NaN is the row's)
  const uint64_t live_mask = __ballot(w > 0.f);
  const int ns_live = 64 - __builtin_clzll(live_mask | 1);

  float o[CPL], olr = 0.f;
#pragma unroll
  for (int k = 0; k < CPL; ++k) o[k] = 0.f;
  for (int s0 = 0; s0 < ns_live; s0 += U) {
    if (s0 > 0) request(s0);
#pragma unroll
    for (int k = 0; k < U / SPL; ++k) {
      const int s = s0 + k * SPL;
      const float wy = SPL == 1 ? from_lane(w, s & 63) : __shfl(w, (s + y_split) & 63, kWave);
      olr = fmaf(wy, wy > 0.f ? y[k] : 0.f, olr);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float wu = from_lane(w, (s0 + u) & 63);  // (splits beyond the last: lanes without a weight)
      const bool in = wu > 0.f;                      // keeps whatever an unwritten row holds out of the sums
#pragma unroll
      for (int k = 0; k < CPL; ++k) o[k] = fmaf(wu, in ? x[u][k] : 0.f, o[k]);
    }
  }
  if constexpr (SPL == 4) olr = sum_over_lane_groups(olr);
  // epilogue O += O_lr B_V
  if (has_bv) {
    for (int r0 = 0; r0 < r; r0 += BN) {
      if (r0 > 0) request_bv(r0);
#pragma unroll
      for (int i = 0; i < BN; ++i) {
        if (r0 + i < r) {  // (uniform)
          const float xr = from_lane(olr, r0 + i);
          if constexpr (sizeof(T) * CPL == 8) {
            o[0] = fmaf(xr, bvp[i].x, o[0]);
            o[CPL - 1] = fmaf(xr, bvp[i].y, o[CPL - 1]);
          } else if constexpr (sizeof(T) == 2 && CPL == 2) {
            o[0] = fmaf(xr, __uint_as_float(bvp[i] << 16), o[0]);
            o[CPL - 1] = fmaf(xr, __uint_as_float(bvp[i] & 0xffff0000u), o[CPL - 1]);
          } else {
            o[0] = fmaf(xr, to_f32<T>(__builtin_bit_cast(T, bvp[i])), o[0]);
          }
        }
      }
    }
  }
  T* out = static_cast<T*>(p.out) + static_cast<int64_t>(row) * D + CPL * lane;
  if constexpr (sizeof(T) == 2 && CPL == 2) {
    *reinterpret_cast<uint32_t*>(out) = pack_bf16x2(o[0] / ell, o[CPL - 1] / ell);
  } else {
#pragma unroll
    for (int k = 0; k < CPL; ++k) out[k] = from_f32<T>(o[k] / ell);
  }
}

// The same merge for the rows of a long prefill, which share one adapter: a wave takes four rows of a kv head, reads a
// piece of 16 bytes per lane, two rows (d = 64: four) with one load, and the B_V slice once for its rows.  Statistics: the
// sixteen lanes of a DPP row hold sixteen shares of the row that their loads belong to, and hand a weight round by a DPP
// broadcast.  What bounds it is the states' bytes, which the caches behind the L2s hand over at 2.5 to 2.7 TB/s, launch included (10240 rows of 32 q heads
// over 8, 5 shares, rank 32: 33 MB in 12.1 us, 12.6 with a wave per row, 17.6 with a workgroup per row; rank 64: 39 MB in 15.6, 20.2
// and 22.8: the other forms load B_V once per rank and row).
template <int D>
__global__ __launch_bounds__(256) void merge_tokens_kernel(Params p) {
  constexpr int RPL = 256 / D;        // rows of one load
  constexpr int NL = 4 / RPL;         // loads that cover the wave's four rows
  constexpr int LPR = 64 / RPL;       // lanes per row
  constexpr int YN = 64 / LPR;        // loads that cover 64 ranks
  constexpr int U = 8;                // shares in flight
  constexpr int kShares = kMergeTokenShares;
  __shared__ __align__(16) float olr_sh[4][4][64];
  asm volatile("" ::"s"(p.part_ml), "s"(p.part_o), "s"(p.part_lr), "s"(p.b_v), "s"(p.out));
  asm volatile("" ::"s"(p.n_q_heads), "s"(p.n_kv_heads), "s"(p.group), "s"(p.rank), "s"(p.n_splits), "s"(p.n_new), "s"(p.adapter_index));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane / LPR, c = lane % LPR, l16 = lane & 15;
  const int h = blockIdx.x, G = p.group, r = p.rank, ns = p.n_splits;
  const int n_rows = p.n_new * G;  // of this kv head: (new token, q head), the q head fastest
  const int i0 = (static_cast<int>(blockIdx.y) * 4 + wave) * 4;
  if (i0 >= n_rows) return;
  int row[NL];
  bool live_row[NL];
  float2 st[NL][kShares / 16];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int i = i0 + k * RPL + sub;
    live_row[k] = i < n_rows;
    const int ic = min(i, n_rows - 1), tok = ic / G;
    row[k] = tok * p.n_q_heads + h * G + (ic - tok * G);
    const float2* ml = reinterpret_cast<const float2*>(p.part_ml) + static_cast<int64_t>(row[k]) * ns;
#pragma unroll
    for (int j = 0; j < kShares / 16; ++j) st[k][j] = ml[min(16 * j + l16, ns - 1)];
  }
  // the first sixteen rows of B_V (the next ones, at larger ranks, follow the sums)
  const int64_t ld = static_cast<int64_t>(p.n_kv_heads) * D;
  const bf16_t* bv = static_cast<const bf16_t*>(p.b_v) + static_cast<int64_t>(p.adapter_index) * r * ld + h * D + 4 * c;
  uint2 b[16];
  auto fetch_bv = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      b[i] = *reinterpret_cast<const uint2*>(bv + min(r0 + i, r - 1) * ld);
      if (r0 + i >= r) b[i] = make_uint2(0u, 0u);  // (fetched again, and no rank)
    }
  };
  if (p.b_v != nullptr) fetch_bv(0);

  // ---- weights of the shares ----
  float w[NL][kShares / 16], ell[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    float big = -INFINITY;
#pragma unroll
    for (int j = 0; j < kShares / 16; ++j) {
      if (16 * j + l16 >= ns) st[k][j] = make_float2(-INFINITY, 0.f);
      // (a share without a visible key left a zero row sum; its rows were never written)
      big = fmaxf(big, st[k][j].y > 0.f ? st[k][j].x : -INFINITY);
    }
    big = over_16_lanes(big, [](float a, float x) { return fmaxf(a, x); });
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < kShares / 16; ++j) {
      w[k][j] = st[k][j].y > 0.f ? expf(st[k][j].x - big) : 0.f;
      sum = fmaf(w[k][j], st[k][j].y, sum);  // (a share's NaN is the row's)
    }
    ell[k] = over_16_lanes(sum, [](float a, float x) { return a + x; });
  }

  // ---- weighted sums, shares in index order ----
  float4 o[NL];
  float olr[NL][YN];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    o[k] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int y = 0; y < YN; ++y) olr[k][y] = 0.f;
  }
  auto shares = [&](auto s0_c) __attribute__((always_inline)) {
    constexpr int S0 = decltype(s0_c)::value;
    if (S0 >= ns) return;
    float4 x[NL][U];
    float y[NL][U][YN];
#pragma unroll
    for (int k = 0; k < NL; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t slot = static_cast<int64_t>(row[k]) * ns + min(S0 + u, ns - 1);
        x[k][u] = *reinterpret_cast<const float4*>(p.part_o + slot * D + 4 * c);
#pragma unroll
        for (int q = 0; q < YN; ++q)
          if (q * LPR < r) y[k][u][q] = p.part_lr[slot * r + min(q * LPR + c, r - 1)];
      }
    __builtin_amdgcn_sched_barrier(0);
    auto add = [&](int k, int u, float wu) __attribute__((always_inline)) {
      // (weight zero: whatever an unwritten row holds stays out of the sums)
      const bool in = wu > 0.f;
      o[k].x = fmaf(wu, in ? x[k][u].x : 0.f, o[k].x);
      o[k].y = fmaf(wu, in ? x[k][u].y : 0.f, o[k].y);
      o[k].z = fmaf(wu, in ? x[k][u].z : 0.f, o[k].z);
      o[k].w = fmaf(wu, in ? x[k][u].w : 0.f, o[k].w);
#pragma unroll
      for (int q = 0; q < YN; ++q)
        if (q * LPR < r) olr[k][q] = fmaf(wu, in ? y[k][u][q] : 0.f, olr[k][q]);
    };
    constexpr int J = S0 / 16, B = 0x150 + (S0 & 15);  // row_newbcast of the share's lane
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      add(k, 0, dpp_f32<B + 0>(w[k][J]));
      add(k, 1, dpp_f32<B + 1>(w[k][J]));
      add(k, 2, dpp_f32<B + 2>(w[k][J]));
      add(k, 3, dpp_f32<B + 3>(w[k][J]));
      add(k, 4, dpp_f32<B + 4>(w[k][J]));
      add(k, 5, dpp_f32<B + 5>(w[k][J]));
      add(k, 6, dpp_f32<B + 6>(w[k][J]));
      add(k, 7, dpp_f32<B + 7>(w[k][J]));
    }
  };
  // (shares behind the last have weight zero: lanes that hold none)
  shares(std::integral_constant<int, 0>{});
  shares(std::integral_constant<int, 8>{});

  // ---- O += O_lr B_V ----
  if (p.b_v != nullptr) {
#pragma unroll
    for (int k = 0; k < NL; ++k)
#pragma unroll
      for (int q = 0; q < YN; ++q) olr_sh[wave][k * RPL + sub][q * LPR + c] = q * LPR + c < r ? olr[k][q] : 0.f;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int r0 = 0; r0 < r; r0 += 16) {
      if (r0 > 0) fetch_bv(r0);
#pragma unroll
      for (int k = 0; k < NL; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 l4 = *reinterpret_cast<const float4*>(&olr_sh[wave][k * RPL + sub][r0 + 4 * q]);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint2 w = b[4 * q + e];
            o[k].x = fmaf(lv[e], __uint_as_float(w.x << 16), o[k].x);
            o[k].y = fmaf(lv[e], __uint_as_float(w.x & 0xffff0000u), o[k].y);
            o[k].z = fmaf(lv[e], __uint_as_float(w.y << 16), o[k].z);
            o[k].w = fmaf(lv[e], __uint_as_float(w.y & 0xffff0000u), o[k].w);
          }
        }
    }
  }
#pragma unroll
  for (int k = 0; k < NL; ++k)
    if (live_row[k]) {
      bf16_t* out = static_cast<bf16_t*>(p.out) + static_cast<int64_t>(row[k]) * D + 4 * c;
      const bf16_t v[4] = {from_f32<bf16_t>(o[k].x / ell[k]), from_f32<bf16_t>(o[k].y / ell[k]), from_f32<bf16_t>(o[k].z / ell[k]),
                           from_f32<bf16_t>(o[k].w / ell[k])};
      *reinterpret_cast<uint2*>(out) = make_uint2(v[0] | static_cast<uint32_t>(v[1]) << 16, v[2] | static_cast<uint32_t>(v[3]) << 16);
    }
}

static void launch_merge_tokens(const Params& p, hipStream_t s) {
  const dim3 grid(p.n_kv_heads, static_cast<unsigned>((static_cast<int64_t>(p.n_new) * p.group + 15) / 16));
  if (p.head_dim == 128) hipLaunchKernelGGL((merge_tokens_kernel<128>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((merge_tokens_kernel<64>), grid, dim3(256), 0, s, p);
}

template <typename T>
static void launch_merge_wave(const Params& p, int rows, hipStream_t s) {
  const dim3 grid(p.n_kv_heads, (p.group + 3) / 4, rows / p.n_q_heads);
  auto launch = [&](auto rb_c, auto u_c) {
    constexpr int RB = decltype(rb_c)::value, U = decltype(u_c)::value;
    if (p.head_dim == 128) hipLaunchKernelGGL((merge_wave_kernel<T, 128, RB, U>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((merge_wave_kernel<T, 64, RB, U>), grid, dim3(256), 0, s, p);
  };
  // (bound 64 for rank 16 1.02 to 1.27 times as long, a bound of 32 for ranks 17 to 32 0.99 to 1.02; eight shares requested at a time where
  // there are three 1.03 to 1.07)
  auto by_rank = [&](auto u_c) {
    if (p.rank <= 16) launch(std::integral_constant<int, 16>{}, u_c);
    else launch(std::integral_constant<int, 64>{}, u_c);
  };
  if (p.n_splits <= 4) by_rank(std::integral_constant<int, 4>{});
  else by_rank(std::integral_constant<int, 8>{});
}

template <typename T>
static void launch_merge_rows(const Params& p, int rows, hipStream_t s) {
  // (kv head, q head of the group, query): workgroups go round-robin over the XCDs, so with 8 kv heads
  // the rows of a head are merged on one XCD
  const dim3 grid(p.n_kv_heads, p.group, rows / p.n_q_heads);
  auto launch = [&](auto ns_c, auto rb_c) {
    constexpr int NS = decltype(ns_c)::value, RB = decltype(rb_c)::value;
    if (p.head_dim == 128) hipLaunchKernelGGL((merge_rows_kernel<T, 128, NS, RB>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((merge_rows_kernel<T, 64, NS, RB>), grid, dim3(256), 0, s, p);
  };
  // (a bound of 64 for 3, 16 and 32 shares 1.24 to 1.45, 1.19 to 1.31 and 1.07 to 1.15 times as long, for ranks 16 and 32 1.04 to
  // 1.09 and 1.03 to 1.05)
  auto by_rank = [&](auto ns_c) {
    if (p.rank <= 16) launch(ns_c, std::integral_constant<int, 16>{});
    else if (p.rank <= 32) launch(ns_c, std::integral_constant<int, 32>{});
    else launch(ns_c, std::integral_constant<int, 64>{});
  };
  if (p.n_splits <= 16) by_rank(std::integral_constant<int, 16>{});
  else if (p.n_splits <= 32) by_rank(std::integral_constant<int, 32>{});
  else by_rank(std::integral_constant<int, 64>{});
}

hipError_t launch_generic_partials(const Params& p, bool is_bf16, int rows, hipStream_t s) {
  const dim3 grid(rows, p.n_splits), block(kWave);
  if (p.key_rope_theta > 0.f && p.b_k != nullptr) {
    if (is_bf16) hipLaunchKernelGGL(generic_partial_rope_kernel<bf16_t>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(generic_partial_rope_kernel<float>, grid, block, 0, s, p);
    return hipGetLastError();
  }
  const int x = rows < (1 << kGenericRowBits) ? rows : (1 << kGenericRowBits);
  const dim3 rgrid(x, p.n_splits, (rows + x - 1) / x);
  auto launch = [&](auto paged_c, auto rb_c) {
    constexpr bool PAGED = decltype(paged_c)::value;
    constexpr int RB = decltype(rb_c)::value;
    if (p.head_dim == 128) {
      if (is_bf16) hipLaunchKernelGGL((generic_partial_kernel<bf16_t, 128, PAGED, RB>), rgrid, dim3(256), 0, s, p);
      else hipLaunchKernelGGL((generic_partial_kernel<float, 128, PAGED, RB>), rgrid, dim3(256), 0, s, p);
    } else {
      if (is_bf16) hipLaunchKernelGGL((generic_partial_kernel<bf16_t, 64, PAGED, RB>), rgrid, dim3(256), 0, s, p);
      else hipLaunchKernelGGL((generic_partial_kernel<float, 64, PAGED, RB>), rgrid, dim3(256), 0, s, p);
    }
  };
  auto by_rank = [&](auto paged_c) {
    if (p.rank <= 16) launch(paged_c, std::integral_constant<int, 16>{});
    else launch(paged_c, std::integral_constant<int, 64>{});
  };
  if (p.block_size != 0) by_rank(std::true_type{});
  else by_rank(std::false_type{});
  return hipGetLastError();
}

template <typename T>
static void launch_merge_t(const Params& p, bool is_bf16, int rows, hipStream_t s) {
  switch (merge_form(is_bf16, p.head_dim, p.rank, p.n_q_heads, p.n_kv_heads, p.n_splits, p.is_prefill != 0, rows)) {
    case MergeForm::kRows: return launch_merge_rows<T>(p, rows, s);
    case MergeForm::kWave: return launch_merge_wave<T>(p, rows, s);
    case MergeForm::kTokens: return launch_merge_tokens(p, s);
    case MergeForm::kColumns: break;
  }
  // enough 128-thread groups that one pass of kMergeUnroll splits per thread covers the splits
  const int groups = (p.n_splits + kMergeUnroll - 1) / kMergeUnroll;
  dim3 grid(rows);
  if (groups <= 1)
    hipLaunchKernelGGL((merge_kernel<T, 1>), grid, dim3(128, 1), 0, s, p);
  else if (groups <= 2)
    hipLaunchKernelGGL((merge_kernel<T, 2>), grid, dim3(128, 2), 0, s, p);
  else if (groups <= 4)
    hipLaunchKernelGGL((merge_kernel<T, 4>), grid, dim3(128, 4), 0, s, p);
  else
    hipLaunchKernelGGL((merge_kernel<T, 8>), grid, dim3(128, 8), 0, s, p);
}

hipError_t launch_merge(const Params& p, bool is_bf16, int rows, hipStream_t s) {
  if (is_bf16)
    launch_merge_t<bf16_t>(p, true, rows, s);
  else
    launch_merge_t<float>(p, false, rows, s);
  return hipGetLastError();
}

}  // namespace lra
