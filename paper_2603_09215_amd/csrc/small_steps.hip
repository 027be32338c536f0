// The kernel of small_steps.h, a translation unit of its own (it holds all the operations of a step).
#include "small_steps.h"

#include "gemv.h"

namespace spark {

__device__ __forceinline__ const SmallSteps &fresh_args() { return kernel_args<SmallSteps>(); }
// the thread's number, made anew too
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// LDS of a workgroup beside the staged rows: its own copy of the sequences' counters (all workgroups
// advance them alike), their page tables and the row lists of the step
struct SmallShared {
  int seq[SMALL_SEQS], st[SMALL_SEQS][ST_WORDS], is_text[SMALL_SEQS], full[SMALL_SEQS];
  RowDesc lower[SMALL_SEQS], upper[SMALL_ROWS], ee[SMALL_SEQS], full_rows[SMALL_SEQS];
  int upper_seq[SMALL_ROWS];                              // index of the row's sequence in the call
  int lower_first[SMALL_SEQS], upper_first[SMALL_ROWS];   // position of the first row that the pass has of the row's sequence
  int lower_row0[SMALL_SEQS], upper_row0[SMALL_ROWS];     // and that row
  int page[SMALL_SEQS][SMALL_CTX / 16];
  int n_upper, n_ee, n_full, broken;
  u64 best[SMALL_SEQS], key[SMALL_SEQS];
  float score[SMALL_CTX + 64], red[SMALL_WAVES * 128];
};

// ------------------------------------------------------------------ words handed over

// The last tag that was waited for, and whether some wait of this wave has run out of polls: then it asks for nothing any
// more, and what it hands on it hands on, so that the others need not run out as well
struct SmallLine {
  unsigned tag;
  bool broken;
  int max_polls;
};
// N neighbouring words with tag `tag`, all lanes of the wave together (on: whether this lane asks)
template <int N>
__device__ __forceinline__ void take_words(SmallLine &line, const u64 *p, unsigned tag, bool on, float *v) {
  u64 w[N];
  for (int polls = 0;; ++polls) {
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = on ? peek_word(p + i) : (u64)tag << 32;
    bool ok = true;
#pragma unroll
    for (int i = 0; i < N; ++i) ok = ok && (unsigned)(w[i] >> 32) == tag;
    if (__all((int)ok) || line.broken) break;
    if (polls == line.max_polls) line.broken = true;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = on ? __uint_as_float((unsigned)w[i]) : 0.f;
}

// The largest logit of a workgroup's, or the token drawn, as an arg-max key whose lower half holds the step beside the
// index: order key (32), step + 1 (16), 0xffff - index (16).  0: no logit.
__device__ __forceinline__ u64 small_key(u64 key, int step) {
  const unsigned index = 0xffffffffu - (unsigned)key;
  return (key & 0xffffffff00000000ull) | (u64)((unsigned)(step + 1) << 16) | (u64)(key ? (0xffffu - index) & 0xffffu : 0u);
}
// (a wait that has run out: 0 for all lanes, as keys of some workgroups alone would not belong to the logits)
__device__ __forceinline__ u64 take_key(SmallLine &line, const u64 *p, int step) {
  u64 k;
  bool ok;
  for (int polls = 0;; ++polls) {
    k = peek_word(p);
    ok = __all((int)(((unsigned)k >> 16) == (unsigned)(step + 1)));
    if (ok || line.broken) break;
    if (polls == line.max_polls) line.broken = true;
  }
  return ok && k >> 32 ? (k & 0xffffffff00000000ull) | (u64)(0xffffffffu - (0xffffu - ((unsigned)k & 0xffffu))) : 0ull;
}

// Totals over the wave of a[0..3] and b[0..3]: lane l of the last eight has that of b (l odd) or a of (l >> 1) & 3
__device__ __forceinline__ float eight_totals(const float (&a)[4], const float (&b)[4], int lane) {
#define SPARK_DPP(v, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false))
  float t[4], u[2];
  // quad_perm [1 0 3 2], then [2 3 0 1]: the neighbours at distance 1 and 2
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float keep = lane & 1 ? b[j] : a[j], give = lane & 1 ? a[j] : b[j];
    t[j] = keep + SPARK_DPP(give, 0xb1);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {   // bit 1: rows 1, 3 or 0, 2
    const float keep = lane & 2 ? t[2 * j + 1] : t[2 * j], give = lane & 2 ? t[2 * j] : t[2 * j + 1];
    u[j] = keep + SPARK_DPP(give, 0x4e);
  }
  // bit 2: rows 2, 3 or 0, 1; the neighbour at distance 4 is the one of row_shl 4 or row_shr 4 in a row of 16
  const float keep = lane & 4 ? u[1] : u[0], give = lane & 4 ? u[0] : u[1];
  const float up = SPARK_DPP(give, 0x104), down = SPARK_DPP(give, 0x114);   // of lane + 4, of lane - 4
  float v = keep + (lane & 4 ? down : up);
  v += SPARK_DPP(v, 0x128);   // row_ror 8: over the row of 16
#undef SPARK_DPP
  v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401f));   // lane ^ 16
  v += __shfl_xor(v, 32, 64);
  return v;
}
__device__ __forceinline__ float4 load_device_scope4(const float *p) {   // p 8-byte aligned
  const float2 a = load_device_scope2(p), b = load_device_scope2(p + 2);
  return make_float4(a.x, a.y, b.x, b.y);
}

// Where the rows that a projection reads come from: words with a tag, or floats in memory that the step does not
// write any more (the embedding, hidden rows of earlier steps)
struct SmallRow {
  const u64 *words;      // nullptr: floats
  const float *floats;
};

// One projection phase of `n_tasks` pairs of weight rows on m rows: workgroup w takes its share of the tasks, a
// wave one piece of SMALL_CHUNK elements of a task's two rows at a time for all rows of the tile; the pieces'
// sums meet in LDS and one thread per (task, row) finishes, or, for a single row in one piece, the wave itself.
//   src(r): the row;  tag: of its words;  gamma: RMSNorm before the product, or nullptr
//   old(task, r): what finish(task, r, y0, y1, old) needs besides the sums and may be read ahead of the rows
template <typename Weights, typename Src, typename Old, typename Finish>
__device__ __forceinline__ void small_projection(SmallLine &line, float *lds, const SmallPhase &ph, int m, float eps, const float *gamma,
                                                 unsigned tag, const Weights &weight_rows, const Src &src, const Old &old, const Finish &finish) {
  float *xs = lds, *part = xs + SMALL_X_FLOATS, *squares = part + SMALL_PART_FLOATS;
  const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_in = ph.n_in, chunks = ph.chunks, chunk_bits = ph.chunk_bits, pitch = chunks * SMALL_CHUNK;
  const int t0 = (int)((unsigned)blockIdx.x * (unsigned)ph.n_tasks / SMALL_WGS);
  const int nt = (int)((unsigned)(blockIdx.x + 1) * (unsigned)ph.n_tasks / SMALL_WGS) - t0;
  const int units = nt << chunk_bits;   // (pieces past the row are skipped)
  const bool alone = m == 1 && chunks == 1;
  constexpr int PRE = 2;   // units of a wave whose weights are fetched ahead of the rows
  float4 pa[PRE], pb[PRE];
  decltype(old(0, 0)) o = decltype(old(0, 0)){};
  auto load_unit = [&](int u, float4 &a, float4 &b) {
    const int k = ((u & ((1 << chunk_bits) - 1)) * SMALL_CHUNK) + lane * 4;
    const float *r0, *r1;
    weight_rows(t0 + (u >> chunk_bits), r0, r1);
    const int ko = k < n_in ? k : 0;   // (meets zeros)
    a = *(const float4 *)(r0 + ko);
    b = *(const float4 *)(r1 + ko);
  };
  auto inverse_rms = [&](int r) {
    if (!gamma) return 1.0f;
    float ss = 0.f;
    for (int c = 0; c < chunks; ++c) ss += squares[r * SMALL_NORM_CHUNKS + c];
    return 1.0f / sqrtf(ss / (float)n_in + eps);
  };
  // (a single row in one piece: its last addition and this product round once, which puts the logits 1 to 2 % closer to 64 bits)
  auto normalised = [](double total, float inv) { return (float)(total * (double)inv); };
  // the thread's own (task, row); a single row in one piece: lane i finishes the wave's unit i
  const int f_task = alone ? t0 + min(wave + (lane & (PRE - 1)) * SMALL_WAVES, max(nt - 1, 0)) : t0 + min(tid & ((1 << ph.task_bits) - 1), max(nt - 1, 0));
  const int f_row = alone ? 0 : tid >> ph.task_bits;
  const bool f_mine = alone || (tid & ((1 << ph.task_bits) - 1)) < nt;
  if (wave < units || (f_row < m && !alone)) {   // (a wave with nothing to do does not take the others' issue slots)
#pragma unroll
    for (int i = 0; i < PRE; ++i) {
      const int u = wave + i * SMALL_WAVES;
      pa[i] = pb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (u < units) load_unit(u, pa[i], pb[i]);
    }
    if (f_row < m) o = old(f_task, f_row);
  }
  for (int r0 = 0; r0 < m; r0 += ph.tile) {
    const int mt = min(ph.tile, m - r0);
    for (int u = wave; u < mt << chunk_bits; u += SMALL_WAVES) {
      const int r = u >> chunk_bits, c = u & ((1 << chunk_bits) - 1), k = c * SMALL_CHUNK + lane * 4, ko = k < n_in ? k : 0;
      if (c >= chunks) continue;
      const SmallRow row = src(r0 + r);
      float4 g = make_float4(1.f, 1.f, 1.f, 1.f);
      if (gamma) g = *(const float4 *)(gamma + ko);
      float v[4];
      if (row.words) {
        take_words<4>(line, row.words + ko, tag, k < n_in, v);
      } else {
        const float4 f = load_device_scope4(row.floats + ko);
        const bool on = k < n_in;
        v[0] = on ? f.x : 0.f; v[1] = on ? f.y : 0.f; v[2] = on ? f.z : 0.f; v[3] = on ? f.w : 0.f;
      }
      *(float4 *)(xs + r * pitch + k) = make_float4(v[0] * g.x, v[1] * g.y, v[2] * g.z, v[3] * g.w);
      if (gamma) {   // RMSNorm is linear in 1 / rms, which the sums are multiplied by
        const float ss = wave_total_last(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]);
        if (lane == 63) squares[r * SMALL_NORM_CHUNKS + c] = ss;
      }
    }
    __syncthreads();
    if (alone) {
      if (wave < units) {
        const float4 v = *(const float4 *)(xs + lane * 4);
        const float inv = inverse_rms(0);
        float s0[PRE], s1[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
          s0[i] = normalised(wave_total64(pa[i].x * v.x + pa[i].y * v.y + pa[i].z * v.z + pa[i].w * v.w), inv);
          s1[i] = normalised(wave_total64(pb[i].x * v.x + pb[i].y * v.y + pb[i].z * v.z + pb[i].w * v.w), inv);
        }
        if (lane < PRE && wave + lane * SMALL_WAVES < units) finish(f_task, 0, lane ? s0[1] : s0[0], lane ? s1[1] : s1[0], o);
        for (int u = wave + PRE * SMALL_WAVES; u < units; u += SMALL_WAVES) {
          float4 a, b;
          load_unit(u, a, b);
          const float y0 = normalised(wave_total64(a.x * v.x + a.y * v.y + a.z * v.z + a.w * v.w), inv);
          const float y1 = normalised(wave_total64(b.x * v.x + b.y * v.y + b.z * v.z + b.w * v.w), inv);
          if (lane == 0) finish(t0 + u, 0, y0, y1, old(t0 + u, 0));
        }
      }
      __syncthreads();
      return;
    }
    int i = 0;
    for (int u = wave; u < units; u += SMALL_WAVES, ++i) {
      const int c = u & ((1 << chunk_bits) - 1);
      if (c >= chunks) continue;
      float4 a = pa[0], b = pb[0];
      if (i == 1) { a = pa[1]; b = pb[1]; }
      if (i >= PRE) load_unit(u, a, b);
      const float *x = xs + c * SMALL_CHUNK + lane * 4;
      if (mt == 1) {
        const float4 v = *(const float4 *)x;
        const float s0 = wave_total_last(a.x * v.x + a.y * v.y + a.z * v.z + a.w * v.w);
        const float s1 = wave_total_last(b.x * v.x + b.y * v.y + b.z * v.z + b.w * v.w);
        if (lane == 63) *(float2 *)(part + 2 * u) = make_float2(s0, s1);
        continue;
      }
      for (int rg = 0; rg < mt; rg += 4) {
        float s0[4], s1[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 v = *(const float4 *)(x + min(rg + j, mt - 1) * pitch);
          s0[j] = a.x * v.x + a.y * v.y + a.z * v.z + a.w * v.w;
          s1[j] = b.x * v.x + b.y * v.y + b.z * v.z + b.w * v.w;
        }
        // eight sums over the wave: halved three times, lanes that differ in one bit each keeping half of them
        // (8 + 4 + 2 additions and three more for the one sum left, where eight sums one by one take 48)
        const float total = eight_totals(s0, s1, lane);
        if (lane >= 56) {
          const int j = (lane >> 1) & 3;
          if (rg + j < mt) part[2 * (u * mt + rg + j) + (lane & 1)] = total;
        }
      }
    }
    __syncthreads();
    const int r = r0 + f_row;
    if (f_mine && f_row < mt) {
      const int t = f_task - t0;
      float2 y = make_float2(0.f, 0.f);
      for (int c = 0; c < chunks; ++c) {
        const float2 p = *(const float2 *)(part + 2 * (((t << chunk_bits) + c) * mt + f_row));
        y.x += p.x; y.y += p.y;
      }
      if (r0 > 0) o = old(f_task, r);
      const float inv = inverse_rms(f_row);
      finish(f_task, r, y.x * inv, y.y * inv, o);
    }
    if (r0 + ph.tile < m) __syncthreads();   // the next tile takes the rows' place
  }
}

// Attention of (row, query head) tasks, one per workgroup at a time.  Cache entries older than the pass are requested
// ahead of the rows' own words, IT * TPT of them; the keys and values of the pass come as words.
// qkv: words of the pass, [row][query heads, key heads, value heads][HD]
template <int HD>
__device__ __forceinline__ void small_attention(SmallLine &line, SmallShared &sh, bool upper, int m, int layer, unsigned tag,
                                                const SmallSteps &a) {
  constexpr int LPT = HD / 4, TPW = 64 / LPT, TPT = SMALL_WAVES * TPW;   // lanes of a token, tokens of a wave and of a trip
  constexpr int IT = 2;                                                  // trips whose loads are in flight together
  const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slot = wave * TPW + lane / LPT, at = lane % LPT * 4;
  const float scale = 1.0f / sqrtf((float)HD);
  const int tasks = m * a.nq, group = a.nq / a.nkv, heads = a.nq + 2 * a.nkv;
  const u64 *qkv = a.qkv_words;
  for (int t = blockIdx.x; t < tasks; t += SMALL_WGS) {
    const int r = t / a.nq, h = t % a.nq;
    const RowDesc rd = upper ? sh.upper[r] : sh.lower[r];
    const int who = upper ? sh.upper_seq[r] : r, row0 = upper ? sh.upper_row0[r] : r;
    const int ctx = rd.pos + 1, old_ctx = upper ? sh.upper_first[r] : sh.lower_first[r], hk = h / group;
    const int pt = a.kv.page_tokens;
    auto entry = [&](int which, int tok) {
      const size_t o = (((size_t)sh.page[who][tok / pt] * a.kv.n_layers + layer) * 2 + which) * a.nkv + hk;
      return (const float *)a.kv.pool + (o * pt + tok % pt) * HD + at;
    };
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 k[IT], v[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int tok = min(i * TPT + slot, max(old_ctx - 1, 0));
      k[i] = v[i] = zero;
      if (i * TPT < old_ctx) { k[i] = load_device_scope4(entry(0, tok)); v[i] = load_device_scope4(entry(1, tok)); }
    }
    // the rows of the pass, one per group of LPT lanes (a sequence has at most 2 * SPARK_MAX_PERIOD of them)
    const int own = ctx - old_ctx;
    const bool have_own = wave * TPW < own, own_on = slot < own;
    float qf[4], kf[4], vf[4];
    {
      const u64 *pq = qkv + ((size_t)r * heads + h) * HD + at;
      const u64 *pk = have_own ? qkv + ((size_t)(row0 + (own_on ? slot : 0)) * heads + a.nq + hk) * HD + at : pq;
      const u64 *pv = have_own ? pk + (size_t)a.nkv * HD : pq;
      u64 wq[4], wk[4], wv[4];
      for (int polls = 0;; ++polls) {
        bool ok = true;
#pragma unroll
        for (int i = 0; i < 4; ++i) { wq[i] = peek_word(pq + i); if (have_own) { wk[i] = peek_word(pk + i); wv[i] = peek_word(pv + i); } else wk[i] = wv[i] = (u64)tag << 32; }
#pragma unroll
        for (int i = 0; i < 4; ++i) ok = ok && (unsigned)(wq[i] >> 32) == tag && (unsigned)(wk[i] >> 32) == tag && (unsigned)(wv[i] >> 32) == tag;
        if (__all((int)ok) || line.broken) break;
        if (polls == line.max_polls) line.broken = true;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) { qf[i] = __uint_as_float((unsigned)wq[i]); kf[i] = __uint_as_float((unsigned)wk[i]); vf[i] = __uint_as_float((unsigned)wv[i]); }
    }
    const float4 q = make_float4(qf[0] * scale, qf[1] * scale, qf[2] * scale, qf[3] * scale);
    auto score = [&](int tok, const float4 &kk, bool on) {
      float s = row16_total(q.x * kk.x + q.y * kk.y + q.z * kk.z + q.w * kk.w);
      if (LPT == 32) s += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(s), 0x401f));   // lane ^ 16
      if (at == 0 && on) sh.score[tok] = s;
    };
#pragma unroll
    for (int i = 0; i < IT; ++i) score(i * TPT + slot, k[i], i * TPT + slot < old_ctx);
    for (int b = IT * TPT; b < old_ctx; b += IT * TPT) {
      float4 kk[IT];
#pragma unroll
      for (int i = 0; i < IT; ++i) kk[i] = load_device_scope4(entry(0, min(b + i * TPT + slot, old_ctx - 1)));
#pragma unroll
      for (int i = 0; i < IT; ++i) score(b + i * TPT + slot, kk[i], b + i * TPT + slot < old_ctx);
    }
    if (have_own) score(old_ctx + slot, make_float4(kf[0], kf[1], kf[2], kf[3]), own_on);
    __syncthreads();
    // every wave finds the maximum and the sum for itself
    float mx = -INFINITY, sum = 0.f;
    for (int i = lane; i < ctx; i += 64) mx = fmaxf(mx, sh.score[i]);
    mx = wave_largest(mx);
    for (int i = lane; i < ctx; i += 64) sum += expf(sh.score[i] - mx);
    sum = wave_total(sum);
    float4 acc = zero;
    auto add = [&](int tok, const float4 &vv, bool on) {
      const float p = on ? expf(sh.score[on ? tok : 0] - mx) : 0.f;
      acc.x += p * vv.x; acc.y += p * vv.y; acc.z += p * vv.z; acc.w += p * vv.w;
    };
#pragma unroll
    for (int i = 0; i < IT; ++i)
      if (i * TPT < old_ctx) add(i * TPT + slot, v[i], i * TPT + slot < old_ctx);
    for (int b = IT * TPT; b < old_ctx; b += IT * TPT) {
      float4 vv[IT];
#pragma unroll
      for (int i = 0; i < IT; ++i) vv[i] = load_device_scope4(entry(1, min(b + i * TPT + slot, old_ctx - 1)));
#pragma unroll
      for (int i = 0; i < IT; ++i) add(b + i * TPT + slot, vv[i], b + i * TPT + slot < old_ctx);
    }
    if (have_own) add(old_ctx + slot, make_float4(vf[0], vf[1], vf[2], vf[3]), own_on);
#pragma unroll
    for (int o = LPT; o < 64; o <<= 1) {
      acc.x += __shfl_xor(acc.x, o, 64); acc.y += __shfl_xor(acc.y, o, 64);
      acc.z += __shfl_xor(acc.z, o, 64); acc.w += __shfl_xor(acc.w, o, 64);
    }
    if (lane < LPT) *(float4 *)(sh.red + wave * HD + at) = acc;
    __syncthreads();
    if (tid < HD) {
      float p[SMALL_WAVES];   // added pairwise: one after the other, they put the logits 1 to 3 % further from 64 bits
#pragma unroll
      for (int w = 0; w < SMALL_WAVES; ++w) p[w] = sh.red[w * HD + tid];
#pragma unroll
      for (int o = SMALL_WAVES / 2; o > 0; o >>= 1)
#pragma unroll
        for (int w = 0; w < o; ++w) p[w] += p[w + o];
      put_word(a.attn_words + ((size_t)r * a.nq + h) * HD + tid, p[0] / sum, tag);
    }
    if (t + SMALL_WGS < tasks) __syncthreads();
  }
}

template <int HD>
__global__ void __launch_bounds__(SMALL_THREADS)
small_steps_k(SmallSteps) {
  extern __shared__ float4 smem4[];
  float *lds = (float *)smem4;
  __shared__ SmallShared sh;
  const int n = fresh_args().n, steps = fresh_args().steps;
  SmallLine line{0u, false, fresh_args().max_polls};
  {
    const SmallSteps &a = fresh_args();
    const int tid = threadIdx.x;
    if (tid < n) {
      sh.seq[tid] = a.seq_ids[tid];
      for (int i = 0; i < ST_WORDS; ++i) sh.st[tid][i] = a.state[sh.seq[tid] * ST_WORDS + i];
      if (blockIdx.x == 0 && !sh.st[tid][ST_ACTIVE]) atomicOr(a.plan + PL_ERR, ERR_INACTIVE);
    }
    __syncthreads();
    for (int i = tid; i < n * (SMALL_CTX / 16); i += SMALL_THREADS) {
      const int b = i / (SMALL_CTX / 16), p = i % (SMALL_CTX / 16);
      sh.page[b][p] = p < a.kv.max_pages ? a.kv.page_table[sh.seq[b] * a.kv.max_pages + p] : 0;
    }
    // a call that has to run again needs the pending rows, which its full-depth steps complete in place
    for (int i = blockIdx.x; i < n * a.kept_rows; i += SMALL_WGS) {
      const int b = i / a.kept_rows, r = i % a.kept_rows;
      if (r < sh.st[b][ST_NPENDING])
        for (int k = tid; k < a.d; k += SMALL_THREADS) a.kept[(size_t)i * a.d + k] = load_device_scope(a.hidden + (size_t)(sh.seq[b] * a.sp.rmax + r) * a.d + k);
    }
    // what an earlier launch has left in the words is not to be taken for a tag
    const int me = blockIdx.x * SMALL_THREADS + tid;
    for (int w = 0; w < 2; ++w) {
      u64 *p = w ? a.words_b : a.words_a;
      const int count = w ? a.count_b : a.count_a;
      for (int i = me; i < count; i += SMALL_WGS * SMALL_THREADS) __hip_atomic_store(p + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (me < n * SMALL_WGS) __hip_atomic_store(a.wg_best + (size_t)(me / SMALL_WGS) * SAMPLE_CAP + me % SMALL_WGS, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (me < n) __hip_atomic_store(a.best + me, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_memory_ops();
    __syncthreads();
    if (tid == 0) __hip_atomic_store(a.flags + blockIdx.x, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid < 64) {
      int polls = 0;
      while (!__all((int)(__hip_atomic_load(a.flags + (tid & (SMALL_WGS - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch)) && ++polls < a.first_polls) {}
      if (tid == 0) sh.broken = polls >= a.first_polls;
    }
    __syncthreads();
    if (sh.broken) {   // (a workgroup that has yet to start would copy pending rows that this one has completed)
      if (tid == 0) atomicOr(a.plan + PL_ERR, ERR_STALLED);
      return;
    }
  }

  for (int step = 0; step < steps; ++step) {
    {
    const SmallSteps &a = fresh_args();
    const int tid = fresh_tid();
    // ---- the step's rows, as next_step_k lists them; every workgroup for itself
    if (tid < n) {
      int *st = sh.st[tid];
      const SchedParams sp = a.sp;
      schedule_decide(sp, st[ST_G], st[ST_OFFSET], st[ST_JSTREAM], st[ST_TEXTBUDGET], st[ST_PHASE], sh.is_text[tid], sh.full[tid]);
      sh.lower[tid] = RowDesc{sh.seq[tid] * a.sp.rmax + st[ST_NPENDING], sh.seq[tid], st[ST_LEN], tid};
      sh.lower_first[tid] = st[ST_LEN];
      sh.lower_row0[tid] = tid;
      if (blockIdx.x == 0) a.out_depth[step * n + tid] = sh.full[tid] ? a.sp.n_layers : a.sp.exit_layer;
    }
    __syncthreads();
    if (tid < n) {
      int u = 0, ne = 0, nf = 0;   // rows of the sequences before this one
      for (int b = 0; b < tid; ++b) {
        const int full = sh.full[b];
        u += full ? sh.st[b][ST_NPENDING] + 1 : 0;
        nf += full;
        ne += !full;
      }
      const int np = sh.st[tid][ST_NPENDING], len = sh.st[tid][ST_LEN], seq = sh.seq[tid];
      if (sh.full[tid]) {
        for (int r = 0; r <= np; ++r) {
          sh.upper[u + r] = RowDesc{seq * a.sp.rmax + r, seq, len - np + r, r == np ? tid : -1};
          sh.upper_seq[u + r] = tid;
          sh.upper_first[u + r] = len - np;
          sh.upper_row0[u + r] = u;
        }
        sh.full_rows[nf] = RowDesc{u + np, seq, len, tid};   // (x_slot: row of the pass)
        u += np + 1; ++nf;
      } else {
        sh.ee[ne++] = RowDesc{tid, seq, len, tid};
      }
      if (tid == n - 1) { sh.n_upper = u; sh.n_ee = ne; sh.n_full = nf; }
    }
    __syncthreads();
    }

    unsigned x_tag = 0;   // of the hidden rows' words
    for (int pass = 0; pass < 2; ++pass) {
      const RowDesc *rows = pass ? sh.upper : sh.lower;
      const int m = __builtin_amdgcn_readfirstlane(pass ? sh.n_upper : n), hm = __builtin_amdgcn_readfirstlane(pass ? sh.n_full : sh.n_ee);
      const RowDesc *head_rows = pass ? sh.full_rows : sh.ee;
      if (pass && !hm) break;
      for (int l = pass ? fresh_args().sp.exit_layer : 0; l < (pass ? fresh_args().sp.n_layers : fresh_args().sp.exit_layer); ++l) {
        const SmallSteps &a = fresh_args();
        const int d = a.d;
        const int qw = a.nq * HD, kvw = a.nkv * HD, heads = a.nq + 2 * a.nkv;
        const int x_row0 = pass ? n : 0;   // (the upper pass begins while some still read the rows of the lower one)
        const bool lowest = l == 0, entered = pass && l == a.sp.exit_layer;
        EpiQKV<float, true> eq;
        eq.wq = a.wq + (size_t)l * qw * d; eq.wk = a.wk + (size_t)l * kvw * d; eq.wv = a.wv + (size_t)l * kvw * d;
        eq.d = d; eq.nq = a.nq; eq.nkv = a.nkv; eq.hd = HD; eq.layer = l;
        // a pass begins with rows of the embedding, or with the rows that wait for the upper layers and the lower pass' own
        auto hidden_row = [&](int r) {
          const RowDesc rd = rows[r];
          if (lowest) return SmallRow{nullptr, a.embed + (size_t)sh.st[rd.out_idx][ST_NEXT] * d};
          if (entered && rd.out_idx < 0) return SmallRow{nullptr, a.hidden + (size_t)rd.x_slot * d};
          return SmallRow{a.x_words + (size_t)(entered ? rd.out_idx : x_row0 + r) * d, nullptr};
        };
        const unsigned t_qkv = ++line.tag;
        const float2 *rope = a.rope;
        small_projection(line, lds, a.qkv, m, a.eps, a.attn_norm + (size_t)l * d, x_tag,
              [&](int t, const float *&r0, const float *&r1) { eq.weight_rows(t, r0, r1); }, hidden_row,
              [&](int t, int r) { return t / (HD / 2) < a.nq + a.nkv ? rope[(size_t)rows[r].pos * (HD / 2) + t % (HD / 2)] : make_float2(1.f, 0.f); },
              [&](int t, int r, float y0, float y1, const float2 &cs) {
                const int head = t / (HD / 2), i = t % (HD / 2);
                if (head < a.nq + a.nkv) {
                  const float u0 = y0 * cs.x - y1 * cs.y, u1 = y1 * cs.x + y0 * cs.y;
                  y0 = u0; y1 = u1;
                }
                u64 *w = a.qkv_words + ((size_t)r * heads + head) * HD + i;
                put_word(w, y0, t_qkv);
                put_word(w + HD / 2, y1, t_qkv);
                if (head >= a.nq) {   // key heads, then value heads, page_tokens apart
                  const RowDesc rd = rows[r];
                  const int pt = a.kv.page_tokens, who = pass ? sh.upper_seq[r] : r;
                  const size_t e = (((size_t)sh.page[who][rd.pos / pt] * a.kv.n_layers + l) * 2 * a.nkv + (head - a.nq)) * pt + rd.pos % pt;
                  float *dst = (float *)a.kv.pool + e * HD + i;
                  store_device_scope(dst, y0);
                  store_device_scope(dst + HD / 2, y1);
                }
              });
        small_attention<HD>(line, sh, pass, m, l, t_qkv, a);
        // a hidden value is read and written by one workgroup alone, o's and down's tasks being dealt alike
        auto residual_rows = [&](const float *w, int n_in) {
          return [w, n_in](int t, const float *&r0, const float *&r1) { r0 = w + (size_t)(2 * t) * n_in; r1 = r0 + n_in; };
        };
        auto old_hidden = [&](int t, int r) {
          return lowest ? *(const float2 *)(a.embed + (size_t)sh.st[rows[r].out_idx][ST_NEXT] * d + 2 * t)
                        : load_device_scope2(a.hidden + (size_t)rows[r].x_slot * d + 2 * t);
        };
        const unsigned t_o = ++line.tag;
        auto store_hidden = [&](unsigned tag) {
          return [&, tag](int t, int r, float y0, float y1, const float2 &o) {
            const float2 h = make_float2(o.x + y0, o.y + y1);
            u64 *w = a.x_words + (size_t)(x_row0 + r) * d + 2 * t;
            put_word(w, h.x, tag);
            put_word(w + 1, h.y, tag);
            store_device_scope2(a.hidden + (size_t)rows[r].x_slot * d + 2 * t, h);
          };
        };
        small_projection(line, lds, a.o, m, a.eps, nullptr, t_qkv, residual_rows(a.wo + (size_t)l * d * qw, qw),
              [&](int r) { return SmallRow{a.attn_words + (size_t)r * qw, nullptr}; }, old_hidden, store_hidden(t_o));
        const unsigned t_act = ++line.tag;
        const float *wg = a.wg + (size_t)l * a.F * d, *wu = a.wu + (size_t)l * a.F * d;
        wait_memory_ops();   // (cache entries and hidden values of this workgroup are in memory before what follows from the next words)
        small_projection(line, lds, a.gateup, m, a.eps, a.mlp_norm + (size_t)l * d, t_o,
              [&](int t, const float *&r0, const float *&r1) { r0 = wg + (size_t)t * d; r1 = wu + (size_t)t * d; },
              [&](int r) { return SmallRow{a.x_words + (size_t)(x_row0 + r) * d, nullptr}; }, [&](int, int) { return 0; },
              [&](int t, int r, float y0, float y1, int) { put_word(a.act_words + (size_t)r * a.F + t, y0 / (1.0f + expf(-y0)) * y1, t_act); });
        x_tag = ++line.tag;
        small_projection(line, lds, a.down, m, a.eps, nullptr, t_act, residual_rows(a.wd + (size_t)l * d * a.F, a.F),
              [&](int r) { return SmallRow{a.act_words + (size_t)r * a.F, nullptr}; },
              [&](int t, int r) { return load_device_scope2(a.hidden + (size_t)rows[r].x_slot * d + 2 * t); }, store_hidden(x_tag));
      }
      if (!hm) continue;
      // ---- the head of this depth
      const SmallSteps &a = fresh_args();
      const int d = a.d, tid = fresh_tid();
      const int head_row0 = a.sp.exit_layer < a.sp.n_layers ? n : 0;   // (no upper layers: the rows are the lower pass' own)
      unsigned h_tag = x_tag;
      if (!pass) {
        const unsigned t_u = ++line.tag;
        small_projection(line, lds, a.lens, hm, a.eps, nullptr, x_tag,
              [&](int t, const float *&r0, const float *&r1) { r0 = a.lens_a + (size_t)(2 * t) * d; r1 = r0 + d; },
              [&](int r) { return SmallRow{a.x_words + (size_t)head_rows[r].x_slot * d, nullptr}; },
              [&](int t, int r) {   // (this workgroup's own hidden values)
                const float2 b = *(const float2 *)(a.lens_b + 2 * t), h = load_device_scope2(a.hidden + (size_t)rows[head_rows[r].x_slot].x_slot * d + 2 * t);
                return make_float4(h.x, h.y, b.x, b.y);
              },
              [&](int t, int r, float y0, float y1, const float4 &o) {
                u64 *w = a.u_words + (size_t)r * d + 2 * t;
                put_word(w, o.x + y0 + o.z, t_u);
                put_word(w + 1, o.y + y1 + o.w, t_u);
              });
        h_tag = t_u;
      }
      EpiVocab<float> ev{pass ? a.lm_head : a.lens_head, d, a.V, a.logits, nullptr};
      if (tid < SMALL_SEQS) sh.best[tid] = 0ull;
      __syncthreads();
      small_projection(line, lds, a.vocab, hm, a.eps, pass ? a.final_norm : a.lens_norm, h_tag,
            [&](int t, const float *&r0, const float *&r1) { ev.weight_rows(t, r0, r1); },
            [&](int r) { return SmallRow{pass ? a.x_words + (size_t)(head_row0 + head_rows[r].x_slot) * d : a.u_words + (size_t)r * d, nullptr}; },
            [&](int, int) { return 0; },
            [&](int t, int r, float y0, float y1, int) {
              float *lg = a.logits + (size_t)head_rows[r].out_idx * a.V + 2 * t;
              store_device_scope(lg, y0);
              if (2 * t + 1 < a.V) store_device_scope(lg + 1, y1);
              EpiVocab<float>::State s{0ull};
              ev.consider(t, y0, y1, s);
              ev.reduce_local(s, &sh.best[r]);
            });
      wait_memory_ops();   // the logits are in memory before the keys
      __syncthreads();
      // (an index of the vocabulary leaves room for the step's number in the key)
      if (tid < hm) __hip_atomic_store(a.wg_best + (size_t)head_rows[tid].out_idx * SAMPLE_CAP + blockIdx.x, small_key(sh.best[tid], step), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- tokens: the largest key of the workgroups', or the draw of one workgroup per sequence
    const SmallSteps &a = fresh_args();
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < n) {
      u64 k = take_key(line, a.wg_best + (size_t)wave * SAMPLE_CAP + (lane & (SMALL_WGS - 1)), step);
#pragma unroll
      for (int o = SMALL_WGS / 2; o > 0; o >>= 1) {
        const u64 other = __shfl_xor(k, o, 64);
        k = other > k ? other : k;
      }
      if (lane == 0) sh.key[wave] = k;
    }
    __syncthreads();
    if (a.words) {
      const int row = blockIdx.x;
      if (row < n) {
        if (tid == 0) sh.best[0] = sh.key[row];
        __syncthreads();
        sample_pick<true, true>(0, 0, 1, a.logits + (size_t)row * a.V, a.V, a.temperature, a.top_p, a.words[(size_t)step * n + row], sh.key[row],
                                nullptr, nullptr, nullptr, nullptr, nullptr, &sh.best[0]);
        __syncthreads();
        if (tid == 0) __hip_atomic_store(a.best + row, small_key(sh.best[0], step), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (wave == 0) {
        const u64 k = take_key(line, a.best + (lane < n ? lane : 0), step);
        if (lane < n) sh.key[lane] = k;
      }
      __syncthreads();
    }
    // ---- the sequences advance, as emit_one does it
    if (tid < n) {
      int *st = sh.st[tid];
      const u64 key = sh.key[tid];
      const int tok = max(0, min((int)(0xffffffffu - (uint32_t)(key & 0xffffffffull)), a.V - 1));
      const int f = a.forced ? a.forced[(size_t)step * n + tid] : -1;
      if (blockIdx.x == 0) {
        if ((uint32_t)(key >> 32) == 0xffffffffu || key == 0ull) atomicOr(a.plan + PL_ERR, ERR_NAN);
        a.out_tokens[(size_t)step * n + tid] = tok;
      }
      st[ST_LEN] += 1;
      st[ST_G] += 1;
      if (!sh.is_text[tid]) st[ST_JSTREAM] += 1;
      st[ST_NPENDING] = sh.full[tid] ? 0 : st[ST_NPENDING] + 1;
      st[ST_NEXT] = f >= 0 ? f : tok;
      st[ST_LASTFULL] = sh.full[tid];
    }
    __syncthreads();
  }
  const SmallSteps &a = fresh_args();
  const int tid = threadIdx.x;
  if (line.broken && (tid & 63) == 0) atomicOr(a.plan + PL_ERR, ERR_STALLED);
  if (blockIdx.x == 0 && tid < n)
    for (int i = 0; i < ST_WORDS; ++i) a.state[sh.seq[tid] * ST_WORDS + i] = sh.st[tid][i];
}

namespace {
const void *kernel_for(int head_dim) { return head_dim == 64 ? (const void *)small_steps_k<64> : (const void *)small_steps_k<128>; }
}  // namespace

bool small_steps_fit(int head_dim) {
  const void *kern = kernel_for(head_dim);
  int per_cu = 0;
  return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_LDS) == hipSuccess &&
         hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, SMALL_THREADS, SMALL_LDS) == hipSuccess && per_cu > 0;
}

hipError_t launch_small_steps(const SmallSteps &a, int head_dim, hipStream_t stream) {
  void *args[] = {(void *)&a};
  return hipLaunchCooperativeKernel(kernel_for(head_dim), dim3(SMALL_WGS), dim3(SMALL_THREADS), args, SMALL_LDS, stream);
}

}  // namespace spark
