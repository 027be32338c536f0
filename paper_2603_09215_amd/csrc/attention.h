// Grouped-query attention of a few query rows over the paged KV cache (decode, flush, prefill
// chunks).  Row r attends cache entries 0..pos_r of its own sequence; since the projection step
// has already written K/V of every row of the pass, this is causal inside a batch of pending
// positions as well (the "length-K causal mask" of Sec. IV-B.3).
//
// Few KV heads cannot fill 256 CUs, so the context is cut into slices of 64 tokens: one task per
// (slice, kv head, row) produces an unnormalised partial (max, sum, weighted values) for all the
// query heads of the group, and the workgroup that finishes last for a (row, kv head) merges the
// slices (arrival counter, device-scope accesses), so no second launch is needed.  Inside a task a
// token's key (and value) vector is spread over LPT consecutive lanes, 16 bytes each, so a wave
// reads 64/LPT whole rows per instruction; all K and V loads of the slice are issued before any
// use.
#pragma once
#include <limits.h>

#include "device_common.h"

namespace spark {

constexpr int ATTN_THREADS = 256;
constexpr int ATTN_SLICE = 64;      // tokens per task
constexpr int ATTN_MAX_GROUP = 16;  // query heads per KV head
static_assert(ATTN_SLICE == 64, "the softmax step maps one token to one lane of a wave");

// Synchronise the NT threads that execute a task: a workgroup barrier, or, when a single wave runs
// the task inside a larger workgroup, only the memory ordering (a wave is in lockstep already).
template <int NT> __device__ __forceinline__ void task_sync() {
  if (NT == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// floats of LDS one task needs with NT threads: scores, softmax statistics, per-wave sums
template <int HD, int G, int NT> constexpr int attn_lds_floats() {
  return G * ATTN_SLICE + G * 2 + (NT / 64) * G * HD + 4;
}

// for the MFMA output projection: the largest magnitude of what each wave has written of row r
template <int NT> __device__ __forceinline__ void put_wave_max(const RowMax &row_max, int r, uint32_t big) {
  if (!row_max.list) return;
  const int tid = threadIdx.x % NT;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) big = max(big, (uint32_t)__shfl_xor((int)big, o, 64));
  if ((tid & 63) == 0) row_max.put(r, blockIdx.y * (NT / 64) + tid / 64, big);
}

// partial layout: part[((r*nq + hq)*n_splits + split)*(HD+4)] = {o[HD], m, l, pad, pad}
//
// Second half of a task, executed by all NT threads that produced the partial of one slice for
// query heads hq0 .. hq0 + g_count - 1 of row r: count the slice as done; the workgroup that
// arrives last for this (row, group of heads) merges the slices,
// out = sum_s exp(m_s - M) o_s / sum_s exp(m_s - M) l_s.
template <int HD, int NT, bool PARTS>
__device__ __forceinline__ void attn_merge(const RowDesc &rd, int r, int hq0, int g_count, int nq,
                                           int n_splits, int slice_tokens, const float *__restrict__ part,
                                           int *__restrict__ cnt, const RowOut &out,
                                           const RowMax &row_max, int *s_last) {
  constexpr int PS = HD + 4;
  const int tid = threadIdx.x % NT;
  // Partials are written through to memory (device-scope stores) and counted with a device-scope
  // atomic; the merging workgroup drops its stale cache lines once and then reads them normally.
  const int used = rd.pos / slice_tokens + 1;   // slices that intersect the context
  wait_memory_ops();                                      // partials written before the count
  task_sync<NT>();
  if (tid == 0) {
    const int prev = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_last = prev == used - 1;
    if (*s_last) {
      __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next layer
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // one cache invalidate for the workgroup
    }
  }
  task_sync<NT>();
  if (!*s_last) return;

  // every thread merges four output elements of one head over all slices in one pass (running
  // maximum, rescaled sums), eight slices' loads in flight at a time
  uint32_t big = 0u;
  for (int i = tid; i < g_count * (HD / 4); i += NT) {
    const int g = i / (HD / 4), c = (i - g * (HD / 4)) * 4;
    const float *p = part + (size_t)(r * nq + hq0 + g) * n_splits * PS;
    float M = -INFINITY, L = 0.f;
    float4 acc4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < used; s0 += 8) {
      float2 ml8[8];
      float4 o8[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int sl = min(s0 + k, used - 1);
        ml8[k] = *(const float2 *)(p + (size_t)sl * PS + HD);
        o8[k] = *(const float4 *)(p + (size_t)sl * PS + c);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (s0 + k < used) {
          const float Mn = fmaxf(M, ml8[k].x);
          const float so = expf(M - Mn), sn = expf(ml8[k].x - Mn);   // exp(-inf) = 0 on the first slice
          acc4.x = acc4.x * so + o8[k].x * sn; acc4.y = acc4.y * so + o8[k].y * sn;
          acc4.z = acc4.z * so + o8[k].z * sn; acc4.w = acc4.w * so + o8[k].w * sn;
          L = L * so + ml8[k].y * sn;
          M = Mn;
        }
      }
    }
    const float inv = 1.0f / L;
    out.put<PARTS>(r, (hq0 + g) * HD + c, make_float4(acc4.x * inv, acc4.y * inv, acc4.z * inv, acc4.w * inv));
    const uint32_t m01 = max(magnitude_bits(acc4.x * inv), magnitude_bits(acc4.y * inv));
    const uint32_t m23 = max(magnitude_bits(acc4.z * inv), magnitude_bits(acc4.w * inv));
    big = max(big, max(m01, m23));
  }
  put_wave_max<NT>(row_max, r, big);
}

// One task, executed by all NT threads of a workgroup: query heads hq0 .. hq0 + g_count - 1
// (g_count <= G, all sharing KV head hk) of row r over one slice; `cnt` counts the slices of this
// (row, group of heads) that are done.
template <typename KT, int HD, int G, int NT, bool PARTS>
__device__ __forceinline__ void attn_task(const RowDesc &rd, int r, int hk, int hq0, int g_count,
                                          int split, const float *__restrict__ qbuf, const KVView &kv,
                                          int layer, int nq, int n_splits, float scale,
                                          float *__restrict__ part, int *__restrict__ cnt,
                                          const RowOut &out, const RowMax &row_max, float *lds) {
  constexpr int VEC = Elem<KT>::VEC;
  constexpr int LPT = HD / VEC;                   // lanes per token
  constexpr int TPI = NT / LPT;                   // tokens per iteration of the workgroup
  constexpr int ITERS = (ATTN_SLICE + TPI - 1) / TPI;
  constexpr int WAVES = NT / 64;
  constexpr int PS = HD + 4;
  float *sc = lds;                                // [G][ATTN_SLICE] scores, then probabilities
  float *ml = sc + G * ATTN_SLICE;                // [G][2]
  float *ored = ml + G * 2;                       // [WAVES][G][HD]
  int *s_last = (int *)(lds + attn_lds_floats<HD, G, NT>() - 4);

  const int ctx = rd.pos + 1;
  const int t0 = split * ATTN_SLICE;
  const int n_tok = min(ATTN_SLICE, ctx - t0);
  const int tid = threadIdx.x % NT, lane = tid & 63, wave = tid >> 6;
  const int tg = tid / LPT, dc = tid % LPT;       // token slot in an iteration, 16-byte chunk of the row

  // issue every K and V load of the slice
  uint4 kraw[ITERS], vraw[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int t = it * TPI + tg;
    if (t < n_tok) {
      const KT *kp = (const KT *)kv.pool + kv_elem_offset(kv, rd.seq, t0 + t, layer, 0, hk) + dc * VEC;
      const KT *vp = (const KT *)kv.pool + kv_elem_offset(kv, rd.seq, t0 + t, layer, 1, hk) + dc * VEC;
      kraw[it] = *(const uint4 *)kp;
      vraw[it] = *(const uint4 *)vp;
    } else {
      kraw[it] = make_uint4(0, 0, 0, 0);
      vraw[it] = make_uint4(0, 0, 0, 0);
    }
  }

  // this lane's chunk of every query head of the group, pre-scaled
  float q[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float *qp = qbuf + (size_t)r * nq * HD + (hq0 + min(g, g_count - 1)) * HD + dc * VEC;
#pragma unroll
    for (int e = 0; e < VEC; e += 2) {
      float2 v = *(const float2 *)(qp + e);
      q[g][e] = v.x * scale; q[g][e + 1] = v.y * scale;
    }
  }

  // scores
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int t = it * TPI + tg;
    float kf[VEC];
    Elem<KT>::unpack(kraw[it], kf);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) s += q[g][e] * kf[e];
#pragma unroll
      for (int o = LPT / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (dc == 0 && t < ATTN_SLICE) sc[g * ATTN_SLICE + t] = t < n_tok ? s : -INFINITY;
    }
  }
  task_sync<NT>();

  // softmax statistics of the slice, one wave per query head at a time (lane = token)
  for (int g = wave; g < g_count; g += WAVES) {
    float s = sc[g * ATTN_SLICE + lane];
    float mx = wave_max(s);
    float p = lane < n_tok ? expf(s - mx) : 0.f;
    sc[g * ATTN_SLICE + lane] = p;
    float sum = wave_sum(p);
    if (lane == 0) { ml[g * 2] = mx; ml[g * 2 + 1] = sum; }
  }
  task_sync<NT>();

  // weighted values: acc[g][e] over this thread's tokens, then over the token slots of the wave
  float acc[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[g][e] = 0.f;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int t = it * TPI + tg;
    if (t < ATTN_SLICE) {
      float vf[VEC];
      Elem<KT>::unpack(vraw[it], vf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float p = sc[g * ATTN_SLICE + t];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[g][e] += p * vf[e];
      }
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      float a = acc[g][e];
#pragma unroll
      for (int o = LPT; o < 64; o <<= 1) a += __shfl_xor(a, o, 64);
      if (lane < LPT) ored[(wave * G + g) * HD + dc * VEC + e] = a;
    }
  task_sync<NT>();
  if (rd.pos < ATTN_SLICE) {
    // the whole context is this slice: nothing to hand over and nobody to wait for (a small fp32
    // model's contexts of 16 to 80 tokens: 7.3 -> 6.2 us a layer on average, 4.7 without the hand-over)
    uint32_t big = 0u;
    for (int i = tid; i < g_count * HD; i += NT) {
      const int g = i / HD, c = i - g * HD;
      float o = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) o += ored[(w * G + g) * HD + c];
      const float inv = 1.0f / ml[g * 2 + 1], y = o * inv;
      out.put<PARTS>(r, (hq0 + g) * HD + c, y);
      big = max(big, magnitude_bits(y));
    }
    put_wave_max<NT>(row_max, r, big);
    return;
  }
  for (int i = tid; i < g_count * HD; i += NT) {
    const int g = i / HD, c = i - g * HD;
    float o = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) o += ored[(w * G + g) * HD + c];
    store_device_scope(part + ((size_t)(r * nq + hq0 + g) * n_splits + split) * PS + c, o);
  }
  if (tid < g_count * 2) {
    const int g = tid >> 1, w = tid & 1;
    store_device_scope(part + ((size_t)(r * nq + hq0 + g) * n_splits + split) * PS + HD + w,
                       ml[g * 2 + w]);
  }
  attn_merge<HD, NT, PARTS>(rd, r, hq0, g_count, nq, n_splits, ATTN_SLICE, part, cnt, out, row_max, s_last);
}

// stand-alone launch: one workgroup per (slice, group of G query heads, row).  A KV head's `group`
// query heads are dealt to ceil(group / G) workgroups: with few rows and few KV heads that is what
// gives the chip enough workgroups, at the price of reading the slice's K and V once per group.
template <typename KT, int HD, int G, bool PARTS>
__global__ void __launch_bounds__(ATTN_THREADS)
attn_rows_k(const RowDesc *__restrict__ rows, const float *__restrict__ qbuf, KVView kv,
            int layer, int nq, int group, int n_splits, float scale, float *__restrict__ part,
            int *__restrict__ arrivals, RowOut out, RowMax row_max) {
  __shared__ float lds[attn_lds_floats<HD, G, ATTN_THREADS>()];
  const int n_groups = (group + G - 1) / G;
  const int split = blockIdx.x, hk = blockIdx.y / n_groups, gi = blockIdx.y - hk * n_groups, r = blockIdx.z;
  const RowDesc rd = rows[r];
  if (split * ATTN_SLICE > rd.pos) return;        // slice beyond the row's context
  attn_task<KT, HD, G, ATTN_THREADS, PARTS>(rd, r, hk, hk * group + gi * G, min(G, group - gi * G), split,
                                            qbuf, kv, layer, nq, n_splits, scale, part,
                                            arrivals + r * gridDim.y + blockIdx.y, out, row_max, lds);
}

// ------------------------------------------------------------------ the same task on the MFMA units
//
// bf16 cache, head_dim 128, up to 16 query heads per KV head, one workgroup (4 waves) per
// (slice, KV head or half of its query heads, row); a slice is one or several 64-token pieces,
// taken one after the other.  Of a piece wave w takes tokens 16w .. 16w+15, from the scores to the weighted values, with
// a maximum and sums of its own, so that the waves wait for each other at the slice's end only:
//   scores   S^T[token][head] = K[token][:] . Q[head][:]   v_mfma_f32_16x16x32_bf16: the K
//            rows go from memory straight into the A operand (lane l: token l%16, eight
//            consecutive elements at 8*(l/16) of each 32-wide step), the scaled queries, split into
//            three bf16 parts that add up to the fp32 value (once per workgroup, handed to the
//            waves through LDS), are the B operand;
//   values   O^T[hd][head] = V[token][hd] . P[token][head]   v_mfma_f32_16x16x16_bf16: the probabilities (two
//            bf16 parts) are the B operand in the registers where the scores have left them, V is
//            staged in the wave's piece of LDS as it lies in the cache (token-major) and read with the transposing
//            LDS load, four tokens of one hd a lane.
// (The waves used to share a piece's maximum, P and V: three barriers a piece.  A launch of 8 rows of 8192 tokens, 2 KV heads,
// 26.5 -> 24.0 us, of 48 rows of 256 to 2048 tokens, 4 KV heads, 41.2 -> 39.5, of 32 28.2 -> 27.5; 8 rows 14.8 and one row 8.8, level.
// What bounds it is the K and V that few bytes in flight per workgroup fetch: the old one without its arithmetic took nine
// tenths of its time, 113 MB in 31 us.)
// The partial it leaves and the merge are those of the vector task.
typedef __attribute__((ext_vector_type(8))) __bf16 attn_bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float attn_f32x4_t;
typedef unsigned int attn_u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int attn_u32x2_t __attribute__((ext_vector_type(2)));
typedef short attn_s16x4_t __attribute__((ext_vector_type(4)));

constexpr int AM_VPITCH = 132;   // bf16 elements per V row in LDS: 4 * 66 dwords lie between the four token groups of a gather, eight banks apart
constexpr int AM_OPITCH = 132;   // floats per head of a wave's sums in LDS
constexpr int AM_QPITCH = 136;   // elements per Q row in LDS (16-byte aligned rows, 4 dwords of skew)

struct AttnPiece {
  attn_u32x4_t v[4];
  attn_bf16x8_t k[4];
};

// loads of a wave's 16 tokens of a 64-token piece that begins with token t0 and reaches n_tok: V as the wave stages it, K as
// its A operand
template <int HD, bool ONE_PAGE>
__device__ __forceinline__ void attn_piece_load(AttnPiece &pc, const KVView &kv, const bf16_t *pool, int seq,
                                                int layer, int hk, int t0, int n_tok, int lane, int wave) {
  // tokens beyond the context read token t0 instead (it exists) and are masked later.  With pages
  // of a multiple of 64 tokens the piece lies inside one page: one address for the workgroup.
  const int col = lane & 15, quad = lane >> 4;
  const size_t piece_k = ONE_PAGE ? kv_elem_offset(kv, seq, t0, layer, 0, hk) : 0;
  const size_t piece_v = ONE_PAGE ? piece_k + (size_t)kv.n_kv_heads * kv.page_tokens * HD : 0;
  const int t = 16 * wave + col, tt = t < n_tok ? t : 0;
  const size_t o = ONE_PAGE ? piece_k + (size_t)tt * HD : kv_elem_offset(kv, seq, t0 + tt, layer, 0, hk);
  const bf16_t *kp = pool + o + quad * 8;
#pragma unroll
  for (int s = 0; s < 4; ++s) pc.k[s] = __builtin_bit_cast(attn_bf16x8_t, *(const attn_u32x4_t *)(kp + 32 * s));
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int t = 16 * wave + 4 * it + quad, tt = t < n_tok ? t : 0;
    const size_t o = ONE_PAGE ? piece_v + (size_t)tt * HD : kv_elem_offset(kv, seq, t0 + tt, layer, 1, hk);
    pc.v[it] = *(const attn_u32x4_t *)(pool + o + col * 8);
  }
}

// `pieces` 64-token pieces per workgroup (slice = 64 * pieces tokens): a workgroup's life is mostly
// dependent round trips (row descriptor, page table, K/V, partial, arrival), so with many rows it
// pays to put several pieces behind one such chain; the pieces are folded with a running maximum.
// TEAMS = 2: two teams of four waves take the even and the odd pieces and are combined at the end.
// ONE_PAGE: pages hold a multiple of 64 tokens.  Known when the kernel is compiled: with both ways of finding
// an address in the loop a piece had 400 vector instructions, forty of them 32-bit products (batch of 32, contexts of 256 to
// 2048: 27.1 -> 23.4 us a launch, of 8 15.0 -> 13.7, one row of 512 tokens 8.5 -> 8.3).
// A piece is a chain of about 3 us, and long contexts make as few workgroups as CUs
// (more of them leave more partial results to one workgroup's merge): a step of eight sequences of 8192
// tokens 18.63 ms with one team and eight pieces, 17.89 with two teams and ten.
template <int HD, int TEAMS, bool PARTS, bool ONE_PAGE>
__global__ void __launch_bounds__(ATTN_THREADS * TEAMS)
attn_rows_mfma_k(const RowDesc *__restrict__ rows, const float *__restrict__ qbuf, KVView kv, int layer,
                 int nq, int kv_group, int heads_per_wg, int n_splits, int pieces, float scale,
                 float *__restrict__ part, int *__restrict__ arrivals, RowOut out, RowMax row_max) {
  static_assert(HD == 128, "four 32-wide steps per key row, eight operands of 16 value columns a wave");
  constexpr int PS = HD + 4;
  constexpr int WAVES = ATTN_THREADS / 64 * TEAMS, VS = 16 * AM_VPITCH, V_BYTES = WAVES * VS * 2;
  constexpr int USED = V_BYTES + 3 * 16 * AM_QPITCH * 2, O_BYTES = 4 * 16 * AM_OPITCH * 4;
  // the waves' V and the queries; in the end, when nobody reads those any more, the sums of four waves
  __shared__ __align__(16) char s_mem[USED > O_BYTES ? USED : O_BYTES];
  __shared__ float s_max[WAVES * 16], s_sum[WAVES * 16], s_total[16];
  __shared__ int s_last;
  bf16_t *s_q = (bf16_t *)(s_mem + V_BYTES);
  const int team = TEAMS == 1 ? 0 : threadIdx.x / ATTN_THREADS;
  // blockIdx.y = (KV head, part of its query heads): with few rows and few KV heads the query
  // heads of a KV head are dealt to several workgroups, which shortens each one's merge
  const int wg_per_kv = (kv_group + heads_per_wg - 1) / heads_per_wg;
  const int split = blockIdx.x, hk = blockIdx.y / wg_per_kv, r = blockIdx.z;
  const int h_first = (blockIdx.y - hk * wg_per_kv) * heads_per_wg;
  const int group = min(heads_per_wg, kv_group - h_first);   // query heads of this workgroup
  const RowDesc rd = rows[r];
  const int span = ATTN_SLICE * pieces;
  if (split * span > rd.pos) return;              // slice beyond the row's context
  const int tid = threadIdx.x % ATTN_THREADS, lane = tid & 63, wave = tid >> 6;   // in the team
  const int col = lane & 15, quad = lane >> 4;    // operand column / row, and which eight of a 32-wide step
  bf16_t *s_v = (bf16_t *)s_mem + (threadIdx.x >> 6) * VS;   // this wave's 16 tokens
  const int hq0 = hk * kv_group + h_first;
  const bf16_t *pool = (const bf16_t *)kv.pool;
  const int n_pieces = min(pieces, (rd.pos - split * span) / ATTN_SLICE + 1);   // pieces the context reaches

  const int trips = (n_pieces + TEAMS - 1) / TEAMS;
  // (a team without a piece left loads the last one again and leaves it)
  auto load_piece = [&](AttnPiece &pc, int j) {
    const int t0 = split * span + min(j, n_pieces - 1) * ATTN_SLICE;
    attn_piece_load<HD, ONE_PAGE>(pc, kv, pool, rd.seq, layer, hk, t0, min(ATTN_SLICE, rd.pos + 1 - t0), lane, wave);
  };
  AttnPiece cur;
  load_piece(cur, team);

  // the scaled queries as three bf16 parts that add up to the fp32 value (each part keeps the
  // upper 8 significant bits of what the parts before it left: truncation, exact remainders):
  // split once by the workgroup, eight elements per thread, and handed to the waves through LDS
  if (team == 0) {
    const int h = tid >> 4, e0 = (tid & 15) * 8;
    attn_u32x4_t ph = {0u, 0u, 0u, 0u}, pm = ph, pl = ph;
    if (h < group) {
      const float *qp = qbuf + ((size_t)r * nq + hq0 + h) * HD + e0;
      const float4 q0 = *(const float4 *)qp, q1 = *(const float4 *)(qp + 4);
      const float qf[8] = {q0.x * scale, q0.y * scale, q0.z * scale, q0.w * scale,
                           q1.x * scale, q1.y * scale, q1.z * scale, q1.w * scale};
      unsigned hi[8], mi[8], lo[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        hi[e] = __float_as_uint(qf[e]) & 0xffff0000u;
        const float r1 = qf[e] - __uint_as_float(hi[e]);
        mi[e] = __float_as_uint(r1) & 0xffff0000u;
        lo[e] = __float_as_uint(r1 - __uint_as_float(mi[e]));   // at most 8 significant bits are left
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ph[e] = (hi[2 * e] >> 16) | hi[2 * e + 1];
        pm[e] = (mi[2 * e] >> 16) | mi[2 * e + 1];
        pl[e] = (lo[2 * e] >> 16) | (lo[2 * e + 1] & 0xffff0000u);
      }
    }
    *(attn_u32x4_t *)(s_q + (0 * 16 + h) * AM_QPITCH + e0) = ph;
    *(attn_u32x4_t *)(s_q + (1 * 16 + h) * AM_QPITCH + e0) = pm;
    *(attn_u32x4_t *)(s_q + (2 * 16 + h) * AM_QPITCH + e0) = pl;
  }

  __syncthreads();

  // this wave's running state, of head `col`.  Score layout: lane = (head col, tokens 4*quad + i of the wave's 16);
  // output layout: lane = (head col, hd 16*t + 4*quad + i).
  float run_max = -INFINITY, run_sum = 0.f;
  attn_f32x4_t oacc[HD / 16];
#pragma unroll
  for (int t = 0; t < HD / 16; ++t) oacc[t] = attn_f32x4_t{0.f, 0.f, 0.f, 0.f};

  for (int trip = 0; trip < trips; ++trip) {
    const int j = trip * TEAMS + team;
    const int t0 = split * span + j * ATTN_SLICE;
    const int n_tok = j < n_pieces ? min(ATTN_SLICE, rd.pos + 1 - t0) : 0;   // 0: every token is masked
    // V into LDS as it lies in the cache
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      attn_u32x2_t *dst = (attn_u32x2_t *)(s_v + (4 * it + quad) * AM_VPITCH + col * 8);
      dst[0] = attn_u32x2_t{cur.v[it][0], cur.v[it][1]};
      dst[1] = attn_u32x2_t{cur.v[it][2], cur.v[it][3]};
    }
    attn_bf16x8_t ka[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) ka[s] = cur.k[s];
    if (trip + 1 < trips) load_piece(cur, j + TEAMS);   // the next piece's loads fly during this one's arithmetic

    // scores of this wave's 16 tokens
    attn_f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const attn_bf16x8_t qb = __builtin_bit_cast(
            attn_bf16x8_t, *(const attn_u32x4_t *)(s_q + (p * 16 + col) * AM_QPITCH + 32 * s + 8 * quad));
        sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[s], qb, sc, 0, 0, 0);
      }
    const int tok0 = 16 * wave + 4 * quad;
    float mw = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (tok0 + i >= n_tok) sc[i] = -INFINITY;
      mw = fmaxf(mw, sc[i]);
    }
    mw = fmaxf(mw, __shfl_xor(mw, 16, 64));
    mw = fmaxf(mw, __shfl_xor(mw, 32, 64));
    const float new_max = fmaxf(run_max, mw), base = new_max > -INFINITY ? new_max : 0.f;   // (-inf: the wave has had no token)
    const float alpha = expf(run_max - base);          // exp(-inf) = 0 on the first piece
    float pr[4], lw = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pr[i] = tok0 + i < n_tok ? expf(sc[i] - base) : 0.f;
      lw += pr[i];
    }
    lw += __shfl_xor(lw, 16, 64);
    lw += __shfl_xor(lw, 32, 64);
    run_sum = run_sum * alpha + lw;
    // probabilities as two bf16 parts (16 significant bits)
    unsigned h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = __float_as_uint(pr[i]) & 0xffff0000u;
      l[i] = __float_as_uint(pr[i] - __uint_as_float(h[i])) & 0xffff0000u;
    }
    const attn_s16x4_t ph = __builtin_bit_cast(attn_s16x4_t, attn_u32x2_t{(h[0] >> 16) | h[1], (h[2] >> 16) | h[3]});
    const attn_s16x4_t pl = __builtin_bit_cast(attn_s16x4_t, attn_u32x2_t{(l[0] >> 16) | l[1], (l[2] >> 16) | l[3]});

    // weighted values on top of the rescaled sums of the earlier pieces
    if (__any(new_max > run_max)) {
#pragma unroll
      for (int t = 0; t < HD / 16; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) oacc[t][i] *= alpha;
    }
    run_max = new_max;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (other lanes of the wave have stored what this one reads)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < HD / 16; ++t) {
      // 16 lanes read 16 elements of four tokens, four of one token a lane, and get one element of all four each
      const attn_s16x4_t va = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) attn_s16x4_t *)(s_v + (4 * quad + (col >> 2)) * AM_VPITCH + 4 * (col & 3) + 16 * t));
      oacc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, ph, oacc[t], 0, 0, 0);
      oacc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, pl, oacc[t], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  // the slice's partial: the waves' weighted values brought to one maximum and added up
  const int w_all = threadIdx.x >> 6;
  if (quad == 0) { s_max[w_all * 16 + col] = run_max; s_sum[w_all * 16 + col] = run_sum; }
  __syncthreads();                        // (and every wave is past its last piece)
  auto slice_max = [&](int g) {           // (the first token's wave has had it: finite)
    float m = s_max[g];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) m = fmaxf(m, s_max[w * 16 + g]);
    return m;
  };
  auto slice_sum = [&](int g) {
    const float m = slice_max(g);
    float y = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) y += s_sum[w * 16 + g] * expf(s_max[w * 16 + g] - m);
    return y;
  };
  // (once per head: found by each of its 128 elements, an exponential per wave every time, it made prompts of 66 and 100
  // tokens, 16 heads per KV head, a quarter of the layers, 3034 -> 3055 and 3517 -> 3555 us)
  if (threadIdx.x < 16) s_total[threadIdx.x] = slice_sum(threadIdx.x);
  float *s_o = (float *)s_mem + (w_all & 3) * 16 * AM_OPITCH + col * AM_OPITCH + 4 * quad;
  {
    const float f = expf(run_max - slice_max(col));
#pragma unroll
    for (int t = 0; t < HD / 16; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) oacc[t][i] *= f;
  }
  if constexpr (TEAMS == 2) {
    // the odd pieces' team first
    if (team == 1) {
#pragma unroll
      for (int t = 0; t < HD / 16; ++t) *(attn_f32x4_t *)(s_o + 16 * t) = oacc[t];
    }
    __syncthreads();
    if (team == 0) {
#pragma unroll
      for (int t = 0; t < HD / 16; ++t) {
        const attn_f32x4_t other = *(const attn_f32x4_t *)(s_o + 16 * t);
#pragma unroll
        for (int i = 0; i < 4; ++i) oacc[t][i] += other[i];
      }
    }
  }
  if (team == 0) {   // (a lane writes where it has read)
#pragma unroll
    for (int t = 0; t < HD / 16; ++t) *(attn_f32x4_t *)(s_o + 16 * t) = oacc[t];
  }
  __syncthreads();
  auto value = [&](int i) {   // element i of the group's heads, the waves in their order
    const float *p = (const float *)s_mem + (i / HD) * AM_OPITCH + i % HD;
    return p[0] + p[16 * AM_OPITCH] + p[2 * 16 * AM_OPITCH] + p[3 * 16 * AM_OPITCH];
  };
  if (rd.pos < span) {   // the whole context is this slice: nothing to hand over and nobody to wait for
    uint32_t big = 0u;
    for (int i = threadIdx.x; i < group * HD; i += 64 * WAVES) {
      const float y = value(i) * (1.0f / s_total[i / HD]);
      out.put<PARTS>(r, hq0 * HD + i, y);
      big = max(big, magnitude_bits(y));
    }
    put_wave_max<ATTN_THREADS * TEAMS>(row_max, r, big);
    return;
  }
  for (int i = threadIdx.x; i < group * HD; i += 64 * WAVES)
    store_device_scope(part + ((size_t)(r * nq + hq0 + i / HD) * n_splits + split) * PS + i % HD, value(i));
  if ((int)threadIdx.x < group * 2) {
    const int g = threadIdx.x >> 1;
    store_device_scope(part + ((size_t)(r * nq + hq0 + g) * n_splits + split) * PS + HD + (threadIdx.x & 1),
                       (threadIdx.x & 1) ? s_total[g] : slice_max(g));
  }
  attn_merge<HD, ATTN_THREADS * TEAMS, PARTS>(rd, r, hq0, group, nq, n_splits, span, part,
                                              arrivals + r * gridDim.y + blockIdx.y, out, row_max, &s_last);
}

// ------------------------------------------------------------------ prompt passes
//
// The rows of a prompt pass are consecutive positions of one sequence, so they share their K and V:
// a workgroup takes one KV head and as many rows as make 128 (row, query head) pairs (8 rows of 16
// heads, 18 of 7), and reads every K and V row of the context once for all of them.  With one
// workgroup per row, as above, a prompt of 8192 tokens reads its cache from L2 for every row again
// (8 MB per row and layer at two KV heads), which is what bounded it.
//
// Eight waves: wave w takes the pairs 32 (w % 4) .. + 31, and of the context's 64-token tiles the
// even ones (w < 4) or the odd ones; the two halves are combined at the end.  Two waves share a
// SIMD, so that one's softmax runs under the other's MFMAs.  v_mfma_f32_32x32x16_bf16 twice:
//   scores  S^T[token][pair] = K . Q^T   A: token l % 32, eight elements at 16 s + 8 (l / 32);
//           B: the pair's scaled query, three bf16 parts that add up to the fp32 value, in
//           registers for the whole context.
//   values  O^T[hd][pair] = V^T . P^T    a lane holds 16 of a block's 32 scores of its own pair (tokens
//           8 i + 4 (l / 32) + 0..3), and since a sum over tokens may take them in any order, those
//           are its B operand as they are: the probabilities (two bf16 parts, rounded to nearest)
//           never leave the lane.  A: V^T, staged transposed in LDS, in the same order of tokens.
// Maximum and sum of a pair live in its two lanes.  K and V of the next tile are on their way in
// registers while a tile is computed; two LDS buffers per half, one barrier per tile.
constexpr int AP_PAIRS = 128;                       // (row, query head) pairs of a workgroup
constexpr int AP_THREADS = 512;
// rows in LDS, padded so that the 16 lanes of an access meet different banks (and, unlike turned
// columns, so that every address of a tile is one register and a constant)
constexpr int AP_KPITCH = 128 + 8, AP_VPITCH = ATTN_SLICE + 4;
constexpr int AP_K_ELEMS = ATTN_SLICE * AP_KPITCH, AP_V_ELEMS = 128 * AP_VPITCH, AP_BUF_ELEMS = AP_K_ELEMS + AP_V_ELEMS;
constexpr size_t AP_LDS_BYTES = sizeof(bf16_t) * 2 * 2 * AP_BUF_ELEMS;   // halves, buffers
typedef __attribute__((ext_vector_type(16))) float attn_f32x16_t;

typedef __attribute__((ext_vector_type(2))) __bf16 attn_bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float attn_f32x2_t;
__device__ __forceinline__ unsigned pack_bf16_rn(float a, float b) {   // (one instruction)
  const attn_f32x2_t f = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f, attn_bf16x2_t));
}

template <int HD, bool PARTS>
__global__ void __launch_bounds__(AP_THREADS, 2)
attn_prompt_k(const RowDesc *__restrict__ rows, int m_rows, const float *__restrict__ qbuf, KVView kv, int layer, int nq,
              int group, int rows_per_wg, int n_row_tiles, float scale, RowOut out, RowMax row_max) {
  static_assert(HD == 128, "tiles and swizzles are for 128 elements");
  extern __shared__ uint4 ap_smem[];
  __shared__ int s_bad;   // the first token whose values were left out for not being finite
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave >> 2, hl = lane >> 5, col = lane & 31;
  const int hk = blockIdx.x % kv.n_kv_heads;
  // the longest contexts first
  const int tile_row = n_row_tiles - 1 - blockIdx.x / kv.n_kv_heads;
  const int row0 = tile_row * rows_per_wg, n_rows = min(rows_per_wg, m_rows - row0);
  const int seq = rows[row0].seq, pos0 = rows[row0].pos;          // the pass's rows are consecutive positions
  const int n_tiles = (pos0 + n_rows - 1) / ATTN_SLICE + 1, trips = (n_tiles + 1) / 2;
  const bf16_t *pool = (const bf16_t *)kv.pool;
  bf16_t *s_k = (bf16_t *)ap_smem + half * 2 * AP_BUF_ELEMS, *s_v = s_k + AP_K_ELEMS;   // + AP_BUF_ELEMS: the other buffer

  // this lane's pair; pairs past the last row repeat a valid one and are not stored
  const int pair = (wave & 3) * 32 + col;
  const bool live = pair / group < n_rows;
  const int row = live ? pair / group : 0, head = hk * group + (live ? pair % group : 0);
  const int pos = pos0 + row;

  // staging: this thread's share of a tile (of its half): four 16-byte pieces of K (one column of the
  // tokens kt + 16 i), four of V (one column of the tokens 4 kt .. + 3)
  const int st = threadIdx.x & 255, kt = st >> 4, kc = st & 15;
  const bool one_page = (kv.page_tokens & (ATTN_SLICE - 1)) == 0;
  attn_u32x4_t kv_r[4];   // of K or of V: K of the next tile goes to LDS before its V is asked for
  auto load_kv = [&](int t, int which) {
    const int t0 = min(t, n_tiles - 1) * ATTN_SLICE, last = pos0 + n_rows - 1;   // tokens past the last row: that one, masked
    const size_t tile = one_page ? kv_elem_offset(kv, seq, t0, layer, which, hk) : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tok = min(t0 + (which ? 4 * kt + i : kt + 16 * i), last);
      const size_t at = one_page ? tile + (size_t)(tok - t0) * HD : kv_elem_offset(kv, seq, tok, layer, which, hk);
      kv_r[i] = *(const attn_u32x4_t *)(pool + at + kc * 8);
    }
  };
  auto store_k = [&](int buf) {
    bf16_t *d = s_k + buf * AP_BUF_ELEMS + kt * AP_KPITCH + kc * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) *(attn_u32x4_t *)(d + 16 * i * AP_KPITCH) = kv_r[i];
  };
  // The values of a token meet the zero probabilities of the rows before it, and zero times infinity is
  // NaN: in tiles that reach past the first row, a token that not all rows attend goes in as zeros if it
  // is not finite, and what the rows from it on get is set to NaN at the end (which is what their next
  // projection would make of one such element).
  auto store_v = [&](int t, int buf) {
    const int t0 = min(t, n_tiles - 1) * ATTN_SLICE, last = pos0 + n_rows - 1;
    if (t0 + ATTN_SLICE - 1 > pos0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tok = min(t0 + 4 * kt + i, last);
        bool bad = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= (kv_r[i][e] & 0x7f80u) == 0x7f80u || (kv_r[i][e] & 0x7f800000u) == 0x7f800000u;
        if (bad && tok > pos0) {
          kv_r[i] = attn_u32x4_t{0u, 0u, 0u, 0u};
          atomicMin(&s_bad, tok);
        }
      }
    }
    bf16_t *d = s_v + buf * AP_BUF_ELEMS + 8 * kc * AP_VPITCH + 4 * kt;
#pragma unroll
    for (int e = 0; e < 8; ++e) {   // element 8 kc + e of four tokens
      const unsigned sel = (e & 1) ? 0x07060302u : 0x05040100u;
      const attn_u32x2_t w = {__builtin_amdgcn_perm(kv_r[1][e >> 1], kv_r[0][e >> 1], sel),
                              __builtin_amdgcn_perm(kv_r[3][e >> 1], kv_r[2][e >> 1], sel)};
      *(attn_u32x2_t *)(d + e * AP_VPITCH) = w;
    }
  };
  load_kv(half, 0);
  if (threadIdx.x == 0) s_bad = INT_MAX;
  __syncthreads();
  store_k(0);
  load_kv(half, 1);
  store_v(half, 0);
  __builtin_amdgcn_sched_barrier(0);

  // the scaled query, three bf16 parts (truncation, exact remainders)
  attn_bf16x8_t qp[3][HD / 16];
  {
    const float *q = qbuf + ((size_t)(row0 + row) * nq + head) * HD + 8 * hl;
#pragma unroll
    for (int s = 0; s < HD / 16; ++s) {
      const float4 a = *(const float4 *)(q + 16 * s), b = *(const float4 *)(q + 16 * s + 4);
      const float f[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale, b.x * scale, b.y * scale, b.z * scale, b.w * scale};
      unsigned hi[8], mi[8], lo[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        hi[e] = __float_as_uint(f[e]) & 0xffff0000u;
        const float r1 = f[e] - __uint_as_float(hi[e]);
        mi[e] = __float_as_uint(r1) & 0xffff0000u;
        lo[e] = __float_as_uint(r1 - __uint_as_float(mi[e]));
      }
      attn_u32x4_t ph, pm, pl;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ph[e] = (hi[2 * e] >> 16) | hi[2 * e + 1];
        pm[e] = (mi[2 * e] >> 16) | mi[2 * e + 1];
        pl[e] = (lo[2 * e] >> 16) | (lo[2 * e + 1] & 0xffff0000u);
      }
      qp[0][s] = __builtin_bit_cast(attn_bf16x8_t, ph);
      qp[1][s] = __builtin_bit_cast(attn_bf16x8_t, pm);
      qp[2][s] = __builtin_bit_cast(attn_bf16x8_t, pl);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();

  float run_max = -INFINITY, run_sum = 0.f;   // the sum: over this lane's tokens
  attn_f32x16_t o[HD / 32];
#pragma unroll
  for (int b = 0; b < HD / 32; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[b][r] = 0.f;

  for (int it = 0; it < trips; ++it) {
    const int t = 2 * it + half, buf = it & 1;
    const bool more = it + 1 < trips;
    const bf16_t *bk = s_k + buf * AP_BUF_ELEMS + col * AP_KPITCH + 8 * hl, *bv = s_v + buf * AP_BUF_ELEMS + col * AP_VPITCH + 4 * hl;
    if (more) load_kv(t + 2, 0);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {              // 32 tokens at a time
      if (t < n_tiles) {
        attn_f32x16_t sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < HD / 16; ++s) {
          const attn_bf16x8_t ka = __builtin_bit_cast(attn_bf16x8_t, *(const attn_u32x4_t *)(bk + 32 * tb * AP_KPITCH + 16 * s));
#pragma unroll
          for (int p = 2; p >= 0; --p) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qp[p][s], sc, 0, 0, 0);
        }
        const int t0 = t * ATTN_SLICE + 32 * tb;
        if (t0 + 31 > pos0) {                     // the tokens reach past the first row
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (t0 + (r >> 2) * 8 + 4 * hl + (r & 3) > pos) sc[r] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float new_max = fmaxf(run_max, mx);
        // (a pair of the odd half may have no token yet: nothing to add, and nothing to rescale)
        const float base = new_max == -INFINITY ? 0.f : new_max;
        const float alpha = expf(run_max - base);
        run_max = new_max;
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sc[r] = expf(sc[r] - base);
          sum += sc[r];
        }
        run_sum = run_sum * alpha + sum;
        if (__any(alpha != 1.f)) {
#pragma unroll
          for (int b = 0; b < HD / 32; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {             // 16 tokens of them
          attn_u32x4_t ph, pl;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p0 = sc[8 * j + 2 * e], p1 = sc[8 * j + 2 * e + 1];
            ph[e] = pack_bf16_rn(p0, p1);
            pl[e] = pack_bf16_rn(p0 - __uint_as_float(ph[e] << 16), p1 - __uint_as_float(ph[e] & 0xffff0000u));
          }
#pragma unroll
          for (int b = 0; b < HD / 32; ++b) {
            const bf16_t *v = bv + 32 * b * AP_VPITCH + 32 * tb + 16 * j;
            const attn_u32x2_t v0 = *(const attn_u32x2_t *)v, v1 = *(const attn_u32x2_t *)(v + 8);
            const attn_u32x4_t va = {v0.x, v0.y, v1.x, v1.y};
            const attn_bf16x8_t a = __builtin_bit_cast(attn_bf16x8_t, va);
            o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(attn_bf16x8_t, pl), o[b], 0, 0, 0);
            o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(attn_bf16x8_t, ph), o[b], 0, 0, 0);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
        if (tb == 0) { store_k(buf ^ 1); load_kv(t + 2, 1); }
        else store_v(t + 2, buf ^ 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  }

  // the odd half hands its share to the even one
  run_sum += __shfl_xor(run_sum, 32, 64);
  float *s_o = (float *)ap_smem;                  // [4 waves][64 registers + maximum, sum][64 lanes]
  float *mine = s_o + (wave & 3) * 66 * 64 + lane;
  if (half == 1) {
#pragma unroll
    for (int b = 0; b < HD / 32; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(b * 16 + r) * 64] = o[b][r];
    mine[64 * 64] = run_max;
    mine[65 * 64] = run_sum;
  }
  __syncthreads();
  if (half == 1) return;
  const float other_max = mine[64 * 64], M = fmaxf(run_max, other_max);   // (token 0 is everybody's: finite)
  const float f0 = expf(run_max - M), f1 = expf(other_max - M);
  const float inv = pos >= s_bad ? NAN : 1.0f / (run_sum * f0 + mine[65 * 64] * f1);
  uint32_t big = 0u;
#pragma unroll
  for (int b = 0; b < HD / 32; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = (o[b][4 * i + e] * f0 + mine[(b * 16 + 4 * i + e) * 64] * f1) * inv;
        big = max(big, magnitude_bits(y[e]));
      }
      if (live) out.put<PARTS>(row0 + row, head * HD + 32 * b + 8 * i + 4 * hl, make_float4(y[0], y[1], y[2], y[3]));
    }
  if (row_max.list) {
    big = max(big, (uint32_t)__shfl_xor((int)big, 32, 64));
    if (live && hl == 0) row_max.put(row0 + row, head, big);
  }
}

}  // namespace spark
