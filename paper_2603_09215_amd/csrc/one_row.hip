// The kernel of one_row.h, a translation unit of its own.
//
// What bounds it: the hand-overs.  A layer of the Step shape takes 86 us (20 layers 1 715, 28 layers 2 418, by
// rocprofv3; a launch per operation: 101), 68 of them the bytes at the rate of a plain read.  Of the rest a hand-over costs 2 to 4 us from the last workgroup's sums to the next
// phase's first product, attention's three together 8, of which the units fetched meanwhile (up to ten a wave,
// 40 MB in all) win back the larger part; and the workgroups reach the end of a phase up to 5 us apart.
#include "one_row.h"

#include <type_traits>

#include "sched.h"

namespace spark {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(1))) const char global_char;

constexpr int UNIT_BYTES = 2048;   // of a unit's place in the ring
constexpr int PHASES = 3 + ROW_PARTS;   // with weights, of a layer: q/k/v, o, the pieces of gate/up, down
constexpr int PH_QKV = 0, PH_O = 1, PH_GATEUP = 2, PH_DOWN = PHASES - 1;

__device__ __forceinline__ void barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ... of the other waves alone, which do attention while the streaming ones fetch on: a count in LDS
__device__ __forceinline__ void aux_barrier(unsigned *count, unsigned &target) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  target += ROW_AUX_WAVES;
  while ((int)(__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - target) < 0) {}
  asm volatile("" ::: "memory");
}

// Whether some wait of this wave has run out of polls: then it asks for nothing any more, and what it hands on it hands
// on, so that the others need not run out as well.  Nothing is read or written where it would not be otherwise.
struct Patience {
  bool broken;
  int max_polls;
};
// N words, the i-th at at(i); all lanes of the wave together
template <int N, typename At>
__device__ __forceinline__ void take_words(Patience &wait, const row_word *p, unsigned tag, const At &at, float (&v)[N]) {
  row_word w[N];
  unsigned todo = (1u << N) - 1u;   // what has come for the whole wave is not asked for again
#pragma unroll
  for (int i = 0; i < N; ++i) w[i] = 0ull;
  for (int polls = 0;; ++polls) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (todo >> i & 1u) w[i] = peek_word(p + at(i));
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (__all((int)((unsigned)(w[i] >> 32) == tag))) todo &= ~(1u << i);
    if (todo == 0u || wait.broken) break;
    if (polls == wait.max_polls) wait.broken = true;
    __builtin_amdgcn_s_sleep(1);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = __uint_as_float((unsigned)w[i]);
}

// where element k of a row lies in LDS (floats): a lane's eight as two vectors 1 KiB apart
__device__ __forceinline__ int x_pos(int k) { return (k & ~511) + ((k >> 2) & 1) * 256 + ((k & 511) >> 3) * 4 + (k & 3); }

__device__ __forceinline__ int share(int n, int w) { return (int)((unsigned)n * (unsigned)w / ROW_WGS); }

// A workgroup's pairs of weight rows in a phase: first .. first + n - 1, of a k of `k` in `segs` pieces of 512
struct Share { int first, n, k, segs; };
__device__ __forceinline__ Share share_of(const OneRow &a, int ph, int wg) {
  Share s;
  if (ph == PH_QKV || ph == PH_O || ph == PH_DOWN) {
    const int pairs = ph == PH_QKV ? (a.nq + 2 * a.nkv) * (ROW_HD / 2) : a.d / 2;
    s.first = share(pairs, wg);
    s.n = share(pairs, wg + 1) - s.first;
    s.k = ph == PH_QKV ? a.d : ph == PH_O ? a.nq * ROW_HD : a.F;
  } else {
    const int f0 = share(a.F, wg), n = share(a.F, wg + 1) - f0, b = ph - PH_GATEUP;
    s.first = f0 + n * b / ROW_PARTS;
    s.n = f0 + n * (b + 1) / ROW_PARTS - s.first;
    s.k = a.d;
  }
  s.segs = (s.k + 511) >> 9;
  return s;
}
__device__ __forceinline__ void weight_rows(const OneRow &a, int ph, int layer, int pair, const bf16_t *&r0, const bf16_t *&r1) {
  if (ph == PH_QKV) {
    constexpr int half = ROW_HD / 2;
    int head = pair / half;
    const int i = pair - head * half;
    const bf16_t *w;
    int heads;
    if (head < a.nq) { w = a.wq; heads = a.nq; }
    else if (head < a.nq + a.nkv) { w = a.wk; heads = a.nkv; head -= a.nq; }
    else { w = a.wv; heads = a.nkv; head -= a.nq + a.nkv; }
    r0 = w + ((size_t)(layer * heads + head) * ROW_HD + i) * a.d;
    r1 = r0 + (size_t)half * a.d;
  } else if (ph == PH_O) {
    r0 = a.wo + ((size_t)layer * a.d + 2 * pair) * (size_t)(a.nq * ROW_HD);
    r1 = r0 + a.nq * ROW_HD;
  } else if (ph == PH_DOWN) {
    r0 = a.wd + ((size_t)layer * a.d + 2 * pair) * (size_t)a.F;
    r1 = r0 + a.F;
  } else {
    const size_t at = ((size_t)layer * a.F + pair) * (size_t)a.d;
    r0 = a.wg + at;
    r1 = a.wu + at;
  }
}

// A wave's units of a phase, walked pair by pair
struct Walk {
  int layer, ph, u, end, seg, pair, segs, k;
  __device__ __forceinline__ void begin(const OneRow &a, int wg, int wave) {
    const Share s = share_of(a, ph, wg);
    const int units = s.n * s.segs;
    u = units * wave / ROW_STREAM_WAVES;
    end = units * (wave + 1) / ROW_STREAM_WAVES;
    const int p = u / s.segs;
    seg = u - p * s.segs;
    pair = s.first + p;
    segs = s.segs;
    k = s.k;
  }
};

// The slice of the context that a workgroup attends to, for `heads` query heads from `head` on, all of KV head `kv`.
// While there are workgroups enough slices are short, and the query heads of a KV head are dealt to several.
struct Slice { int kv, head, heads, index, count, size, first; bool mine; };
__device__ __forceinline__ Slice slice_of(const OneRow &a, int pos, int wg) {
  Slice s;
  s.size = ROW_SLICE / 2;
  if (a.nkv * (pos / s.size + 1) > ROW_WGS) s.size = ROW_SLICE;
  s.count = pos / s.size + 1;
  const int group = a.nq / a.nkv;
  int deal = 0;   // workgroups per KV head and slice, as a power of two
  while (deal < 2 && (2 << deal) <= group && a.nkv * s.count * (2 << deal) <= ROW_WGS) ++deal;
  const int most = (group + (1 << deal) - 1) >> deal, id = wg / s.count;
  s.mine = id < a.nkv << deal;
  s.kv = s.mine ? id >> deal : 0;
  const int g0 = s.mine ? (id & ((1 << deal) - 1)) * most : 0;
  s.head = s.kv * group + g0;
  s.heads = min(most, group - g0);
  s.index = s.mine ? wg - id * s.count : 0;
  s.first = s.index * s.size;
  return s;
}

// The waves that had some of pair t's pieces, a bit each, and the sum over them
__device__ __forceinline__ unsigned summed_waves(int t, const Share &s) {
  const int units = s.n * s.segs, lo = t * s.segs, hi = lo + s.segs;
  unsigned who = 0;
#pragma unroll
  for (int w = 0; w < ROW_STREAM_WAVES; ++w) {
    const int u0 = units * w / ROW_STREAM_WAVES, u1 = units * (w + 1) / ROW_STREAM_WAVES;
    if (max(u0, lo) < min(u1, hi)) who |= 1u << w;
  }
  return who;
}
__device__ __forceinline__ float2 sums(const OneRow &a, const char *lds, int t, int set, unsigned who) {
  const float4 *part = (const float4 *)((const float2 *)(lds + a.lds_part) + (set * a.pairs + t) * ROW_STREAM_WAVES);
  float2 y = make_float2(0.f, 0.f);
#pragma unroll
  for (int w = 0; w < ROW_STREAM_WAVES; w += 2) {
    const float4 v = part[w / 2];
    y.x += who >> w & 1u ? v.x : 0.f; y.y += who >> w & 1u ? v.y : 0.f;
    y.x += who >> w & 2u ? v.z : 0.f; y.y += who >> w & 2u ? v.w : 0.f;
  }
  return y;
}
__device__ __forceinline__ float inverse_rms(const OneRow &a, const char *lds) {
  const float *squares = (const float *)(lds + a.lds_misc);
  float ss = 0.f;
#pragma unroll
  for (int w = 0; w < ROW_AUX_WAVES; ++w) ss += squares[w];
  return 1.0f / sqrtf(ss / (float)a.d + a.eps);
}
// A row of n into LDS; under a norm times gamma, and its squares (RMSNorm is linear in 1 / rms, which the sums are
// multiplied by)
__device__ __forceinline__ void put_row(const OneRow &a, char *lds, int t, const float (&v)[8], const float (&g)[8], int n, bool norm) {
  float *x = (float *)(lds + a.lds_x);
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int k = i * ROW_AUX + t;
    if (k < ((n + 511) & ~511)) {
      const float e = k < n ? v[i] : 0.f;
      ss += e * e;
      x[x_pos(k)] = k < n ? e * g[i] : 0.f;
    }
  }
  if (norm) {
    ss = wave_total_last(ss);
    if ((t & 63) == 63) ((float *)(lds + a.lds_misc))[t >> 6] = ss;
  }
}
__device__ __forceinline__ void gather_row(const OneRow &a, char *lds, int t, Patience &wait, const row_word *words, int n, const float *gamma, unsigned tag, bool wait_words = false) {
  float g[8], v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) g[i] = gamma ? gamma[min(i * ROW_AUX + t, n - 1)] : 1.f;
  if (wait_words) {   // for a while yet nothing will have come: one word of eight is asked for
    float first[1];
    take_words<1>(wait, words, tag, [&](int) { return (unsigned)min((t >> 6) * ROW_AUX + t, n - 1); }, first);
  } else {
    __builtin_amdgcn_s_sleep(ROW_NAP);
  }
  take_words<8>(wait, words, tag, [&](int i) { return (unsigned)min(i * ROW_AUX + t, n - 1); }, v);
  put_row(a, lds, t, v, g, n, gamma != nullptr);
}

}  // namespace

__device__ __forceinline__ const OneRow &fresh_args() { return kernel_args<OneRow>(); }
// the thread's number, made anew too
__device__ __forceinline__ int fresh_aux() {
  int t = threadIdx.x - 64 * ROW_STREAM_WAVES;
  asm volatile("" : "+v"(t));
  return t;
}

__global__ void __launch_bounds__(ROW_THREADS) one_row_k(OneRow) {
  extern __shared__ float4 smem4[];
  char *lds = (char *)smem4;
  const int wg = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  if (wave < ROW_STREAM_WAVES) {
    // ------------------------------------------------------------ the streaming waves
    // Their loads are the only memory operations they have under way, so that a wait can name how many may be
    // left.  All their LDS accesses are written out: the compiler would wait for every load before each.
    const OneRow &a = fresh_args();
    lds_char *ring = (lds_char *)lds + wave * (ROW_DEPTH * UNIT_BYTES);
    const unsigned ring_at = (unsigned)(uintptr_t)ring + lane * 16;
    const unsigned x_at = (unsigned)(uintptr_t)((lds_char *)lds + a.lds_x) + lane * 16;
    const unsigned act_at = (unsigned)(uintptr_t)((lds_char *)lds + a.lds_act) + lane * 16;
    const unsigned part_at = (unsigned)(uintptr_t)((lds_char *)lds + a.lds_part);
    Walk in;
    in.layer = a.l0; in.ph = 0;
    in.begin(a, wg, wave);
    const bf16_t *r0, *r1;
    weight_rows(a, in.ph, in.layer, in.pair, r0, r1);
    bool more = true;
    auto next_phase = [&] {   // the next that has units for this wave; behind the last one the first rows again
      const OneRow &a = fresh_args();
      while (in.u >= in.end) {
        if (++in.ph == PHASES) { in.ph = 0; ++in.layer; }
        if (in.layer >= a.l1) {
          more = false;
          in.k = a.d; in.seg = 0;
          r0 = r1 = a.wq;
          return;
        }
        in.begin(a, wg, wave);
      }
      weight_rows(a, in.ph, in.layer, in.pair, r0, r1);
    };
    if (in.u >= in.end) next_phase();
    int to_slot = 0;
    auto issue = [&] {
      const int k = in.seg * 512 + lane * 8, ko = k < in.k ? k : 0;   // (meets zeros)
      lds_char *to = ring + to_slot * UNIT_BYTES;
      to_slot = to_slot == ROW_DEPTH - 1 ? 0 : to_slot + 1;
      __builtin_amdgcn_global_load_lds((global_char *)(r0 + ko), to, 16, 0, 2);
      __builtin_amdgcn_global_load_lds((global_char *)(r1 + ko), to + 1024, 16, 0, 2);
      if (!more) return;
      ++in.u;
      if (in.u >= in.end) {
        next_phase();
      } else if (++in.seg == in.segs) {
        in.seg = 0;
        ++in.pair;
        if (in.ph == PH_QKV && in.pair % (ROW_HD / 2) == 0) {
          weight_rows(fresh_args(), in.ph, in.layer, in.pair, r0, r1);   // the next head
        } else {
          const int step = in.ph == PH_O || in.ph == PH_DOWN ? 2 * in.k : in.k;
          r0 += step;
          r1 += step;
        }
      }
    };
#pragma unroll 1
    for (int i = 0; i < ROW_DEPTH; ++i) issue();
    int slot = 0, set = 0;
    const int l1 = a.l1;
    for (int layer = a.l0; layer < l1; ++layer) {
      for (int ph = 0; ph < PHASES; ++ph) {
        const OneRow &a = fresh_args();
        Walk w;
        w.layer = layer; w.ph = ph;
        w.begin(a, wg, wave);
        const int first = share_of(a, ph, wg).first;
        const unsigned xs = ph == PH_DOWN ? act_at : x_at;
        float s0 = 0.f, s1 = 0.f;
        auto multiply = [&](const u4 &wa, const u4 &wb, const f4 &x0, const f4 &x1) {
          float fa[8], fb[8];
          Elem<bf16_t>::unpack(make_uint4(wa.x, wa.y, wa.z, wa.w), fa);
          Elem<bf16_t>::unpack(make_uint4(wb.x, wb.y, wb.z, wb.w), fb);
          s0 += fa[0] * x0.x + fa[1] * x0.y + fa[2] * x0.z + fa[3] * x0.w;
          s1 += fb[0] * x0.x + fb[1] * x0.y + fb[2] * x0.z + fb[3] * x0.w;
          s0 += fa[4] * x1.x + fa[5] * x1.y + fa[6] * x1.z + fa[7] * x1.w;
          s1 += fb[4] * x1.x + fb[5] * x1.y + fb[6] * x1.z + fb[7] * x1.w;
          ++w.u;
          if (++w.seg == w.segs || w.u == w.end) {   // the wave's part of a pair is complete
            const float2 t = make_float2(wave_total_last(s0), wave_total_last(s1));
            const unsigned to = part_at + (unsigned)(((set * a.pairs + (w.pair - first)) * ROW_STREAM_WAVES + wave) * 8);
            if (lane == 63) asm volatile("ds_write_b64 %0, %1" ::"v"(to), "v"(t) : "memory");
            s0 = s1 = 0.f;
            if (w.seg == w.segs) { w.seg = 0; ++w.pair; }
          }
        };
        constexpr int behind = 2 * (ROW_DEPTH - ROW_SPARE - 1);   // loads that may be under way before another is issued
        if (ph <= PH_GATEUP || ph == PH_DOWN) {
          // until the row is there, the first units wait in registers, so that memory goes on filling the ring
          u4 pa[ROW_PARKED], pb[ROW_PARKED];
          const int parked = min(ROW_PARKED, w.end - w.u);
#pragma unroll
          for (int i = 0; i < ROW_PARKED; ++i) {
            pa[i] = pb[i] = u4{0u, 0u, 0u, 0u};
            if (i < parked) {
              asm volatile("s_waitcnt vmcnt(%3)\n\t"
                           "ds_read_b128 %0, %2\n\t"
                           "ds_read_b128 %1, %2 offset:1024\n\t"
                           "s_waitcnt lgkmcnt(0)"
                           : "=&v"(pa[i]), "=&v"(pb[i])
                           : "v"(ring_at + slot * UNIT_BYTES), "i"(0)
                           : "memory");
              if (i >= ROW_SPARE) issue();
              slot = slot == ROW_DEPTH - 1 ? 0 : slot + 1;
            }
          }
          barrier();
#pragma unroll 1
          for (int i = 0; i < min(parked, ROW_SPARE); ++i) issue();
#pragma unroll
          for (int i = 0; i < ROW_PARKED; ++i) {
            if (i < parked) {
              f4 x0, x1;
              asm volatile("ds_read_b128 %0, %2\n\t"
                           "ds_read_b128 %1, %2 offset:1024\n\t"
                           "s_waitcnt lgkmcnt(0)"
                           : "=&v"(x0), "=&v"(x1)
                           : "v"(xs + w.seg * 2048)
                           : "memory");
              multiply(pa[i], pb[i], x0, x1);
            }
          }
        }
        while (w.u < w.end) {
          u4 wa, wb;
          f4 x0, x1;
          asm volatile("s_waitcnt vmcnt(%6)\n\t"
                       "ds_read_b128 %0, %4\n\t"
                       "ds_read_b128 %1, %4 offset:1024\n\t"
                       "ds_read_b128 %2, %5\n\t"
                       "ds_read_b128 %3, %5 offset:1024\n\t"
                       "s_waitcnt lgkmcnt(0)"
                       : "=&v"(wa), "=&v"(wb), "=&v"(x0), "=&v"(x1)
                       : "v"(ring_at + slot * UNIT_BYTES), "v"(xs + w.seg * 2048), "i"(behind)
                       : "memory");
          issue();
          slot = slot == ROW_DEPTH - 1 ? 0 : slot + 1;
          multiply(wa, wb, x0, x1);
        }
        barrier();   // the sums are there
        set ^= 1;
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the ring is this workgroup's until nothing is under way to it)
    return;
  }

  // -------------------------------------------------------------- the other waves
  Patience wait{false, fresh_args().max_polls};
  int set = 0;
  float2 h = make_float2(0.f, 0.f);   // the thread's pair of the hidden state
  unsigned arrived = 0;
  auto aux_barrier_ = [&] { aux_barrier((unsigned *)(lds + fresh_args().lds_misc) + ROW_AUX_WAVES, arrived); };
  {
    const OneRow &a = fresh_args();
    const int t = fresh_aux();
    if (t == 0) *((unsigned *)(lds + a.lds_misc) + ROW_AUX_WAVES) = 0u;   // (a barrier comes before its first use)
    const Share s = share_of(a, PH_O, wg);
    if (t < s.n) h = *(const float2 *)(a.hidden + (size_t)a.row->x_slot * a.d + 2 * (s.first + t));
  }
  const int l0 = fresh_args().l0, l1 = fresh_args().l1;
  for (int layer = l0; layer < l1; ++layer) {
    // ---- q/k/v
    if (layer == l0) {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const float *row = a.hidden + (size_t)a.row->x_slot * a.d, *gamma = a.attn_norm + (size_t)layer * a.d;
      float g[8], v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = min(i * ROW_AUX + t, a.d - 1);
        g[i] = gamma[k];
        v[i] = row[k];
      }
      put_row(a, lds, t, v, g, a.d, true);
    } else {
      const OneRow &a = fresh_args();
      gather_row(a, lds, fresh_aux(), wait, a.h1, a.d, a.attn_norm + (size_t)layer * a.d, a.tag + (unsigned)(layer - l0) - 1u);
    }
    barrier();
    // the slice of attention that this workgroup has: its old keys and values, and what the epilogue needs, are fetched
    // under the stream.  16 threads have a token of each half of the slice, eight elements of it.
    uint4 kr[2], vr[2];
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const RowDesc rd = *a.row;
      const Slice sl = slice_of(a, rd.pos, wg);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int at_tok = sl.first + e * (ROW_SLICE / 2) + (t >> 4);
        const int p = sl.mine && at_tok < rd.pos ? at_tok : 0;   // (the others' are not used)
        kr[e] = *(const uint4 *)((const bf16_t *)a.kv.pool + kv_elem_offset(a.kv, rd.seq, p, layer, 0, sl.kv) + (t & 15) * 8);
        vr[e] = *(const uint4 *)((const bf16_t *)a.kv.pool + kv_elem_offset(a.kv, rd.seq, p, layer, 1, sl.kv) + (t & 15) * 8);
      }
    }
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const RowDesc rd = *a.row;
      const unsigned tag = a.tag + (unsigned)(layer - l0);
      const Share s = share_of(a, PH_QKV, wg);
      constexpr int half = ROW_HD / 2;
      const int pair = s.first + t, head = pair / half, i = pair - head * half;
      float2 cs = make_float2(1.f, 0.f);
      size_t kv_at = 0;
      if (t < s.n) {
        const int which = head < a.nq + a.nkv ? 0 : 1;
        if (head < a.nq + a.nkv) cs = a.rope[(size_t)rd.pos * half + i];
        if (head >= a.nq) kv_at = kv_elem_offset(a.kv, rd.seq, rd.pos, layer, which, head - a.nq - which * a.nkv) + i;
      }
      const unsigned who = summed_waves(t, s);
      const float inv = inverse_rms(a, lds);
      barrier();
      if (t < s.n) {
        const float2 y = sums(a, lds, t, set, who);
        float y0 = y.x * inv, y1 = y.y * inv;
        if (head < a.nq + a.nkv) {
          const float u = y0 * cs.x - y1 * cs.y, v = y1 * cs.x + y0 * cs.y;
          y0 = u; y1 = v;
        }
        if (head >= a.nq) {
          const bf16_t b0 = f32_to_bf16(y0), b1 = f32_to_bf16(y1);
          bf16_t *dst = (bf16_t *)a.kv.pool + kv_at;
          dst[0] = b0; dst[half] = b1;
          y0 = bf16_to_f32(b0); y1 = bf16_to_f32(b1);
        }
        put_word(a.qkv + head * ROW_HD + i, y0, tag);
        put_word(a.qkv + head * ROW_HD + i + half, y1, tag);
      }
      set ^= 1;
    }
    // ---- attention; its scratch lies where the MLP's activations will
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const unsigned tag = a.tag + (unsigned)(layer - l0);
      const int pos = a.row->pos;
      const Slice sl = slice_of(a, pos, wg);
      const int ch = t & 15;
      const bool mine = sl.mine;
      float *qs = (float *)(lds + a.lds_act), *sc = qs + ROW_MAX_GROUP * ROW_HD, *vs = sc + ROW_MAX_GROUP * ROW_SLICE;
      float *kn = vs + ROW_SLICE * ROW_HD;   // the new token's key
      if (mine) {
        const int n = sl.heads * ROW_HD;
        const bool last = pos < sl.first + sl.size;   // the slice has the new token: its key and value are words as well
        float q[5];
        const unsigned new_at = last ? (unsigned)((a.nq + (t & ROW_HD ? a.nkv : 0) + sl.kv) * ROW_HD + (t & (ROW_HD - 1))) : (unsigned)(sl.head * ROW_HD);
        take_words<5>(wait, a.qkv, tag, [&](int i) { return i < 4 ? (unsigned)(sl.head * ROW_HD + min(i * ROW_AUX + t, n - 1)) : new_at; }, q);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i * ROW_AUX + t < n) qs[i * ROW_AUX + t] = q[i] * a.scale;
        if (last && t < 2 * ROW_HD) (t < ROW_HD ? kn : vs + (pos - sl.first - 1) * ROW_HD)[t] = q[4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int tok = e * (ROW_SLICE / 2) + (t >> 4), at_tok = sl.first + tok;
          float vf[8];
          Elem<bf16_t>::unpack(vr[e], vf);
          if (tok < sl.size && at_tok != pos)
#pragma unroll
            for (int i = 0; i < 8; i += 4)
              *(f4 *)(vs + tok * ROW_HD + ch * 8 + i) = at_tok < pos ? f4{vf[i], vf[i + 1], vf[i + 2], vf[i + 3]} : f4{0.f, 0.f, 0.f, 0.f};
        }
      }
      aux_barrier_();
      if (mine) {
        float kf[2][8];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          Elem<bf16_t>::unpack(kr[e], kf[e]);
          if (sl.first + e * (ROW_SLICE / 2) + (t >> 4) == pos)
#pragma unroll
            for (int i = 0; i < 8; i += 4) {
              const f4 v = *(const f4 *)(kn + ch * 8 + i);
              kf[e][i] = v.x; kf[e][i + 1] = v.y; kf[e][i + 2] = v.z; kf[e][i + 3] = v.w;
            }
        }
        for (int g0 = 0; g0 < sl.heads; g0 += 4) {
          float s[4][2];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float *q = qs + min(g0 + j, sl.heads - 1) * ROW_HD + ch * 8;
            s[j][0] = s[j][1] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; i += 4) {
              const f4 v = *(const f4 *)(q + i);
#pragma unroll
              for (int e = 0; e < 2; ++e) s[j][e] += kf[e][i] * v.x + kf[e][i + 1] * v.y + kf[e][i + 2] * v.z + kf[e][i + 3] * v.w;
            }
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 2; ++e) s[j][e] = row16_total(s[j][e]);
          if (ch == 0)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (g0 + j < sl.heads)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  const int tok = e * (ROW_SLICE / 2) + (t >> 4);
                  sc[(g0 + j) * ROW_SLICE + tok] = tok < sl.size && sl.first + tok <= pos ? s[j][e] : -INFINITY;
                }
        }
      }
      aux_barrier_();
    }
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const unsigned tag = a.tag + (unsigned)(layer - l0);
      const Slice sl = slice_of(a, a.row->pos, wg);
      const int dim = t & (ROW_HD - 1), quarter = __builtin_amdgcn_readfirstlane(t >> 7);
      float *sc = (float *)(lds + a.lds_act) + ROW_MAX_GROUP * ROW_HD, *vs = sc + ROW_MAX_GROUP * ROW_SLICE, *red = vs + ROW_SLICE * ROW_HD;
      if (sl.mine) {   // a quarter of the threads (two waves) takes every fourth head; thread: one dimension
        row_word *to = a.part + ((size_t)sl.head * sl.count + sl.index) * (ROW_HD + 2);
        auto weigh = [&](auto heads) {
          constexpr int HEADS = decltype(heads)::value;
          float p[HEADS], o[HEADS], m[HEADS], l[HEADS];
#pragma unroll
          for (int j = 0; j < HEADS; ++j) p[j] = sc[min(quarter + 4 * j, sl.heads - 1) * ROW_SLICE + lane];
#pragma unroll
          for (int j = 0; j < HEADS; ++j) m[j] = wave_largest(p[j]);
#pragma unroll
          for (int j = 0; j < HEADS; ++j) p[j] = expf(p[j] - m[j]);   // (a slice has at least one token)
#pragma unroll
          for (int j = 0; j < HEADS; ++j) {
            l[j] = wave_total(p[j]);
            o[j] = 0.f;
          }
          for (int k0 = 0; k0 < sl.size; k0 += 32) {
            float v[32];
#pragma unroll
            for (int k = 0; k < 32; ++k) v[k] = vs[(k0 + k) * ROW_HD + dim];
#pragma unroll
            for (int k = 0; k < 32; ++k)
#pragma unroll
              for (int j = 0; j < HEADS; ++j) o[j] += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p[j]), k0 + k)) * v[k];
          }
#pragma unroll
          for (int j = 0; j < HEADS; ++j) {
            const int g = quarter + 4 * j;
            if (g < sl.heads) {
              row_word *w = to + g * sl.count * (ROW_HD + 2);
              put_word(w + dim, o[j], tag);
              if (dim < 2) put_word(w + ROW_HD + dim, dim ? l[j] : m[j], tag);
            }
          }
        };
        if (sl.heads <= 4) weigh(std::integral_constant<int, 1>());
        else if (sl.heads <= 8) weigh(std::integral_constant<int, 2>());
        else weigh(std::integral_constant<int, ROW_MAX_GROUP / 4>());
      }
      // the slices of a head meet at two of the last workgroups, half of its dimensions at each
      constexpr int width = ROW_HD / 2, groups = ROW_AUX / width;
      const int id = ROW_WGS - 1 - wg, head = id >> 1, d0 = (id & 1) * width + (t & (width - 1));
      if (head < a.nq) {
        float M = -INFINITY, L = 0.f, O = 0.f;
        const row_word *p = a.part + (size_t)head * sl.count * (ROW_HD + 2);
        constexpr int N = 6;   // slices that a thread asks for at a time
        for (int b = 0; b < sl.count; b += N * groups) {
          const int s0 = b + t / width;
          float v[3 * N];
          take_words<3 * N>(wait, p, tag, [&](int i) {
            const int s = min(s0 + groups * (i / 3), sl.count - 1), e = i % 3;
            return (unsigned)(s * (ROW_HD + 2) + (e == 0 ? d0 : ROW_HD - 1 + e));
          }, v);
#pragma unroll
          for (int i = 0; i < N; ++i) {
            if (s0 + groups * i < sl.count) {
              const float Mn = fmaxf(M, v[3 * i + 1]);
              const float f0 = expf(M - Mn), f1 = expf(v[3 * i + 1] - Mn);
              O = O * f0 + v[3 * i] * f1;
              L = L * f0 + v[3 * i + 2] * f1;
              M = Mn;
            }
          }
        }
        red[t] = O;
        red[ROW_AUX + t] = M;
        red[2 * ROW_AUX + t] = L;
      }
      aux_barrier_();
      if (head < a.nq && t < width) {
        float M = -INFINITY, L = 0.f, O = 0.f;
#pragma unroll 4
        for (int i = 0; i < groups; ++i) M = fmaxf(M, red[ROW_AUX + i * width + t]);
#pragma unroll 4
        for (int i = 0; i < groups; ++i) {
          const float f = expf(red[ROW_AUX + i * width + t] - M);
          O += red[i * width + t] * f;
          L += red[2 * ROW_AUX + i * width + t] * f;
        }
        put_word(a.attn + head * ROW_HD + d0, O * (1.0f / L), tag);
      }
    }
    // ---- o
    {
      const OneRow &a = fresh_args();
      gather_row(a, lds, fresh_aux(), wait, a.attn, a.nq * ROW_HD, nullptr, a.tag + (unsigned)(layer - l0), true);
    }
    barrier();
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const unsigned tag = a.tag + (unsigned)(layer - l0);
      const Share s = share_of(a, PH_O, wg);
      const unsigned who = summed_waves(t, s);
      barrier();
      if (t < s.n) {
        const float2 y = sums(a, lds, t, set, who);
        h.x += y.x; h.y += y.y;
        put_word(a.h0 + 2 * (s.first + t), h.x, tag);
        put_word(a.h0 + 2 * (s.first + t) + 1, h.y, tag);
      }
      set ^= 1;
    }
    // ---- gate/up, in pieces; a piece's activations are gathered under the stream of the next
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      gather_row(a, lds, t, wait, a.h0, a.d, a.mlp_norm + (size_t)layer * a.d, a.tag + (unsigned)(layer - l0));
      float *act = (float *)(lds + a.lds_act);
      for (int k = a.F + t; k < ((a.F + 511) & ~511); k += ROW_AUX) act[x_pos(k)] = 0.f;   // (meets weights)
    }
    barrier();
    for (int b = 0; b < ROW_PARTS; ++b) {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const unsigned tag = a.tag + (unsigned)(layer - l0);
      float *act = (float *)(lds + a.lds_act);
      const int slots = row_slots(a.F);
      const Share s = share_of(a, PH_GATEUP + b, wg);
      const unsigned who = summed_waves(t, s);
      const float inv = inverse_rms(a, lds);
      barrier();
      if (t < s.n) {
        const float2 y = sums(a, lds, t, set, who);
        const float g = y.x * inv, u = y.y * inv;
        put_word(a.act + (b * ROW_WGS + wg) * slots + t, g / (1.0f + expf(-g)) * u, tag);
      }
      set ^= 1;
      if (b + 1 < ROW_PARTS) __builtin_amdgcn_s_sleep(ROW_PIECE_NAP);
      constexpr int N = ROW_ACT_WORDS;
      for (int i0 = 0; i0 < ROW_WGS * slots; i0 += N * ROW_AUX) {
        float v[N];
        int from[N], at[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int idx = min(i0 + i * ROW_AUX + t, ROW_WGS * slots - 1), w = idx / slots;
          const Share o = share_of(a, PH_GATEUP + b, w);
          const int j = min(idx - w * slots, o.n - 1);   // (a slot that is not used: the one before it)
          from[i] = (b * ROW_WGS + w) * slots + j;
          at[i] = x_pos(o.first + j);
        }
        take_words<N>(wait, a.act, tag, [&](int i) { return (unsigned)from[i]; }, v);
#pragma unroll
        for (int i = 0; i < N; ++i) act[at[i]] = v[i];
      }
    }
    // ---- down
    barrier();
    {
      const OneRow &a = fresh_args();
      const int t = fresh_aux();
      const unsigned tag = a.tag + (unsigned)(layer - l0);
      const Share s = share_of(a, PH_DOWN, wg);
      const unsigned who = summed_waves(t, s);
      barrier();
      if (t < s.n) {
        const float2 y = sums(a, lds, t, set, who);
        h.x += y.x; h.y += y.y;
        if (layer + 1 < l1) {
          put_word(a.h1 + 2 * (s.first + t), h.x, tag);
          put_word(a.h1 + 2 * (s.first + t) + 1, h.y, tag);
        } else {
          *(float2 *)(a.hidden + (size_t)a.row->x_slot * a.d + 2 * (s.first + t)) = h;
        }
      }
      set ^= 1;
    }
  }
  if (wait.broken && lane == 0) atomicOr(fresh_args().error, ERR_STALLED);
}

size_t one_row_lds(OneRow &a) {
  const int wide = a.d > a.nq * ROW_HD ? a.d : a.nq * ROW_HD;
  size_t at = (size_t)ROW_STREAM_WAVES * ROW_DEPTH * UNIT_BYTES;
  a.lds_x = (int)at;
  at += sizeof(float) * (size_t)((wide + 511) & ~511);
  a.lds_act = (int)at;
  const size_t attn = sizeof(float) * (ROW_MAX_GROUP * ROW_HD + ROW_MAX_GROUP * ROW_SLICE + ROW_SLICE * ROW_HD + 12 * ROW_HD);
  const size_t act = sizeof(float) * (size_t)((a.F + 511) & ~511);
  at += act > attn ? act : attn;
  a.lds_part = (int)at;
  a.pairs = row_pairs((a.nq + 2 * a.nkv) * (ROW_HD / 2));
  for (int n : {row_pairs(a.d / 2), row_slots(a.F)}) a.pairs = n > a.pairs ? n : a.pairs;
  at += 2 * (size_t)a.pairs * ROW_STREAM_WAVES * sizeof(float2);
  a.lds_misc = (int)at;
  at += sizeof(float) * ROW_AUX_WAVES + sizeof(unsigned);
  return at <= 160 * 1024 && a.pairs <= ROW_AUX ? at : 0;
}

bool one_row_fit() {
  int per_cu = 0;
  return hipFuncSetAttribute((const void *)one_row_k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess &&
         hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, one_row_k, ROW_THREADS, 160 * 1024) == hipSuccess && per_cu > 0;
}

hipError_t launch_one_row(const OneRow &a, size_t lds, hipStream_t stream) {
  void *args[] = {(void *)&a};
  return hipLaunchCooperativeKernel((const void *)one_row_k, dim3(ROW_WGS), dim3(ROW_THREADS), args, lds, stream);
}

}  // namespace spark
