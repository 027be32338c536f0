// Projections for 5 and more activation rows at once (prompt chunks, batched decoding) on the MFMA
// units.  With that many rows a projection is a real dense contraction: every weight element is
// used many times, so the vector kernel that serves a handful of rows would be ALU-bound.
//
// Weights are bf16, activations fp32, and the MFMA takes 16-bit operands: an activation goes through
// it in parts that add up to the fp32 value, which keeps the result at fp32 accuracy instead of
// rounding the activations to 8 bits of mantissa.  Three kernels run the contraction:
//
//   mfma_tiled_k and, for at most 48 rows, mfma_direct_k (further down), which a context with the
//   memory for it runs, take their weights from a copy in fp16 and in MFMA operand order, written when the context was created.  A bf16
//   weight scaled by a power of two per row is an fp16 number (exact down to 2^-31 of the row's
//   largest weight), so the activations are fp16 parts too, and fp16
//   has 11 bits of mantissa: two parts hold 23 of the 24 bits that three of bf16 hold.  A third of the
//   MFMA work, and at the clock the chip holds under MFMA load a third of the time of a prompt's
//   projections, is not done.
//   mfma_rows_k, described next, takes the caller's row-major bf16 weights, for contexts without
//   that copy: three bf16 parts (3 x 8 bits), which the producers of the rows write.
//
// (Two bf16 parts leave 2^-17 relative error per element; re-rounded to bf16 in the KV cache that
// is enough to double the deviation from the oracle.)
//
// v_mfma_f32_32x32x16: A is 32 weight rows x 16 k, B is 16 k x 32 activation rows; lane l
// supplies 8 consecutive k of row (l % 32), k-block (l / 32); of the 16 results in a lane,
// register r belongs to weight row (r/4)*8 + (l/32)*4 + r%4 and activation row l % 32.
//
// A workgroup of eight waves owns 256 "tasks" (the same pairs of weight rows the vector kernel
// uses, so the epilogues are shared: rotary pairs, gate/up pairs, adjacent rows), 32 per wave, and
// all rows of one tile of 32 or 64 activation rows; more rows are further tiles (grid.z), whose
// workgroups read the same weights at about the same time.  The k range may be split over
// blockIdx.y; partial sums then go to a buffer and a second kernel finishes them, which is what
// fills 256 CUs when a matrix has only a few thousand rows.
//
// HBM delivers its bandwidth only to loads that cover whole 128-byte lines of a row in one
// instruction (measured: 6.3 TB/s, against 2.6 TB/s when a wave instruction takes 32 bytes from
// each of 32 rows, which is what loading straight into the A-operand layout does).  So a wave
// loads its 64 weight rows eight lanes per row, 128 bytes per row and instruction, and turns the
// result into the A-operand layout through a private piece of LDS: written as (row, 16-byte
// segment), read back as (lane % 32 = row, lane / 32 = segment of the MFMA step).
#pragma once
#include <type_traits>
#include "cover.h"
#include "device_common.h"
#include "gemv.h"

namespace spark {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef _Float16 f16_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int MG_THREADS = 512;
constexpr int MG_WAVES = 8;
constexpr int MG_ROWPAD = MG_KC + 8;   // bf16 per staged row (a 16-byte skew per row keeps the operand reads conflict-free)
constexpr int MG_TASKS_PER_WAVE = 32;
constexpr int MG_TASKS_PER_BLOCK = MG_WAVES * MG_TASKS_PER_WAVE;
constexpr int MG_MAX_MTILES = 2;       // activation rows per workgroup: 32 or 64
// bf16 parts of an activation that meet bf16 weights: all three, so that every product is the
// exact product of the fp32 activation and the bf16 weight, as in the vector kernel
constexpr int MG_PARTS = 3;
// weight chunks a wave has in registers, on their way from HBM
constexpr int MG_W_DEPTH = 2;
// dynamic LDS of mfma_rows_k: per wave 64 padded weight rows of one chunk; two buffers of three
// parts of 32*MTILES padded activation rows
constexpr size_t mg_lds_bytes(int mtiles, int waves = MG_WAVES) {
  return sizeof(bf16_t) * (waves * 64 * MG_ROWPAD + 2 * MG_PARTS * 32 * mtiles * MG_ROWPAD);
}

// ------------------------------------------------------------------ activation preparation

// x[r][k] = src row (plain) or RMSNorm(hidden[x_slot_r]; gamma), and the row's largest
// magnitude: the input of a projection that no finishing launch
// before it has prepared
__global__ void __launch_bounds__(256)
prep_rows_k(const RowDesc *__restrict__ rows, const float *__restrict__ src, int stride, int indirect,
            const float *__restrict__ gamma, float eps, int n, RowOut x, RowMax row_max) {
  __shared__ float red[4];
  __shared__ uint32_t big[4];
  const int r = blockIdx.x;
  const float *row = src + (size_t)(indirect ? rows[r].x_slot : r) * stride;
  uint32_t amax = 0u;
  auto put = [&](int k, float4 f) {
    if (x.part_units) x.put<true>(r, k, f);
    else x.put<false>(r, k, f);
    amax = max(amax, max(max(magnitude_bits(f.x), magnitude_bits(f.y)), max(magnitude_bits(f.z), magnitude_bits(f.w))));
  };
  auto finish = [&]() {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, o, 64));
    if ((threadIdx.x & 63) == 0) big[threadIdx.x >> 6] = amax;
    __syncthreads();
    if (threadIdx.x == 0 && row_max.list) row_max.put(r, 0, max(max(big[0], big[1]), max(big[2], big[3])));
  };
  if (n <= 4096) {
    // the row and the gains in registers: every load is issued before the first is used (one
    // memory round trip instead of one per loop trip of two passes)
    constexpr int NI = 4;
    float4 v[NI], g[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = threadIdx.x * 4 + i * 1024;
      v[i] = *(const float4 *)(row + (k < n ? k : 0));
      if (gamma) g[i] = *(const float4 *)(gamma + (k < n ? k : 0));
    }
    float inv = 1.0f;
    if (gamma) {
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (threadIdx.x * 4 + i * 1024 < n) ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
      ss = wave_sum(ss);
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
      __syncthreads();
      inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)n + eps);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = threadIdx.x * 4 + i * 1024;
      if (k < n)
        put(k, gamma ? make_float4(v[i].x * inv * g[i].x, v[i].y * inv * g[i].y, v[i].z * inv * g[i].z, v[i].w * inv * g[i].w)
                     : v[i]);
    }
    finish();
    return;
  }
  float inv = 1.0f;
  if (gamma) {
    float ss = 0.f;
    for (int k = threadIdx.x * 4; k < n; k += 1024) {
      const float4 v = *(const float4 *)(row + k);
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)n + eps);
  }
  for (int k = threadIdx.x * 4; k < n; k += 1024) {
    float4 v = *(const float4 *)(row + k);
    if (gamma) {
      const float4 g = *(const float4 *)(gamma + k);
      v = make_float4(v.x * inv * g.x, v.y * inv * g.y, v.z * inv * g.z, v.w * inv * g.w);
    }
    put(k, v);
  }
  finish();
}

// The input of a projection: fp32 rows `stride` elements apart (or in operand order, see RowOut) and
// the lists of their magnitudes; and words that are to be zero for the launches after this one.
struct ProjIn {
  const float *x;
  int stride, part_units;   // (as in RowOut; parts for the kernel on the caller's weights)
  RowMax row_max;
  uint4 *zero;
  int n_zero;   // 16-byte units
};
__device__ __forceinline__ void clear_words(const ProjIn &in) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < in.n_zero; i += gridDim.x * blockDim.x)
    in.zero[i] = make_uint4(0, 0, 0, 0);
}
// Largest exponent in the list of row r, found by LANES (a power of two) neighbouring lanes of which
// this is number `l`, in two halves: the first loads, issued before the weights' (memory answers in
// order, and the weights come from further away), and the rest.
template <int LANES> struct RowExponent {
  static constexpr int U = 5, SPAN = 16 * LANES * U;   // bytes per trip: an MLP of 20480 in one
  const uint8_t *p;
  int n, l;
  uint4 v[U];
  __device__ __forceinline__ void load(int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + (u * LANES + l) * 16;
      v[u] = *(const uint4 *)(p + (i < n ? i : 0));
    }
  }
  __device__ __forceinline__ RowExponent(const RowMax &rm, int r, int l_) : p(rm.list + (size_t)r * rm.stride), n(rm.n), l(l_) { load(0); }
  __device__ __forceinline__ int get() {
    uint32_t even = 0u, odd = 0u;   // of the bytes 0, 2 and 1, 3 of every word
    for (int i0 = 0;;) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + (u * LANES + l) * 16;
        const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int left = n - (i + 4 * e);   // bytes past the end of the list are not anybody's
          const uint32_t word = left >= 4 ? w[e] : left > 0 ? w[e] & ((1u << (8 * left)) - 1u) : 0u;
          const uint32_t a = word & 0x00ff00ffu, b = (word >> 8) & 0x00ff00ffu;
          even = max(even & 0xffffu, a & 0xffffu) | max(even & 0xff0000u, a & 0xff0000u);
          odd = max(odd & 0xffffu, b & 0xffffu) | max(odd & 0xff0000u, b & 0xff0000u);
        }
      }
      i0 += SPAN;
      if (i0 >= n) break;
      load(i0);
    }
    int big = (int)max(max(even & 0xffu, even >> 16), max(odd & 0xffu, odd >> 16));
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) big = max(big, __shfl_xor(big, o, 64));
    return big;
  }
};

// ------------------------------------------------------------------ the contraction

// A workgroup takes one tile of 256 (or 128) tasks, one k range and one tile of 32*MTILES activation rows.
// SPLIT: write partial sums part[split][task][2][m_pad] instead of running the epilogue.
//
// The loop over 64-wide chunks of k is software-pipelined.  Weights: a wave has MG_W_DEPTH chunks
// of its 64 rows on their way in registers; the oldest is written to the wave's LDS piece, read
// back as A operands and its registers are reloaded with the chunk MG_W_DEPTH ahead (LDS
// operations of one wave execute in order, so the piece needs no barrier).  Activations: two LDS
// buffers shared by the workgroup; while the MFMAs read one, the next chunk (loaded into
// registers one iteration earlier) is written to the other and the chunk after that is requested:
// one workgroup barrier per chunk and no load whose latency is exposed.  All loads are
// unconditional (rows, tasks and chunks past the end are clamped to valid addresses and their
// products skipped or discarded), which lets the compiler wait for exactly the loads a step needs;
// loads return in issue order, so inside an iteration the activation loads are issued before the
// weight loads and the order of the steps is pinned.
// WAVES: 8, or 4 for matrices of few rows, whose launches then have twice as many workgroups
template <int MTILES, typename Epi, bool SPLIT, int WAVES = MG_WAVES>
__global__ void __launch_bounds__(64 * WAVES)
mfma_rows_k(Epi epi, const RowDesc *__restrict__ rows, int m_rows, ProjIn in, int n_in, int n_tasks,
            int chunks_per_split, float *__restrict__ part, int m_pad, int n_task_tiles, int n_splits, int n_row_tiles,
            int xcd_groups) {
  static_assert(MTILES <= MG_MAX_MTILES, "accumulators and LDS are sized for 64 rows");
  clear_words(in);
  // Workgroup -> (task tile, k range, row tile).  Consecutive workgroup ids go to consecutive
  // XCDs, each with its own L2: the row tiles of one (task tile, k range) read the same weights,
  // so they get ids 8 apart (same XCD, launched together) and the weights cross HBM once for them.
  // Ids are dealt in groups of 8 * n_row_tiles: 8 tiles, one per XCD, times their row tiles.
  // (xcd_groups: chosen by the launch; measured to pay for few, long k ranges: gate/up of a prompt
  // pass 191 -> 169 us, while down with its many short ranges lost, 101 -> 116 us.)
  int bx, by, bz;
  if (!xcd_groups) {   // task tiles fastest, then k ranges, then row tiles
    const int tiles = n_task_tiles * n_splits;
    bz = blockIdx.x / tiles;
    const int tile = blockIdx.x - bz * tiles;
    if (bz >= n_row_tiles) return;
    by = tile / n_task_tiles;
    bx = tile - by * n_task_tiles;
  } else {
    const int per_group = 8 * n_row_tiles;
    const int group = blockIdx.x / per_group, r = blockIdx.x - group * per_group;
    const int tile = group * 8 + (r & 7);
    if (tile >= n_task_tiles * n_splits) return;
    bz = r >> 3;
    by = tile / n_task_tiles;
    bx = tile - by * n_task_tiles;
  }
  constexpr int MROWS = 32 * MTILES;
  constexpr int WD = MG_W_DEPTH;
  constexpr int XPOS = MROWS * (MG_KC / 8);                  // 16-byte vectors of one part of a chunk
  constexpr int XV = (XPOS + (64 * WAVES) - 1) / (64 * WAVES);   // of them per thread
  // Every thread stages XV vectors, wrapping around when the workgroup has more threads than a
  // chunk has vectors (32 rows in an eight-wave workgroup: two threads then write the same data to
  // the same place).  A store under a condition would take its load with it: the compiler sinks a
  // load whose only use is conditional into that branch, next to the store, and the wave then
  // waits out the whole memory latency once per chunk instead of having the data a chunk ahead.
  static_assert(XPOS % (64 * WAVES) == 0 || (64 * WAVES) % XPOS == 0, "the staging wraps evenly");
  constexpr int PART_ELEMS = MROWS * MG_ROWPAD;
  constexpr int WI = 8;                                      // load instructions per chunk: 8 rows x 128 bytes each
  extern __shared__ uint4 mg_smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bf16_t *s_w = (bf16_t *)mg_smem + wave * 64 * MG_ROWPAD;             // this wave's [64][MG_ROWPAD]
  bf16_t *s_x = (bf16_t *)mg_smem + WAVES * 64 * MG_ROWPAD;         // [2][3][MROWS * MG_ROWPAD]
  const int row0 = bz * MROWS;
  const int task0 = bx * (WAVES * MG_TASKS_PER_WAVE) + wave * MG_TASKS_PER_WAVE;
  const int n_chunks = (n_in + MG_KC - 1) / MG_KC;   // the last one may be short: activations are zero-padded
  const int c_begin = by * chunks_per_split;
  const int c_end = min(n_chunks, c_begin + chunks_per_split);
  if (c_begin >= c_end) return;

  // Load instruction i covers the wave's rows 8i..8i+7 (rows 0..31: first weight row of tasks
  // task0.., rows 32..63: their second weight row); this lane takes segment lane % 8 of row
  // 8i + lane / 8.
  const bf16_t *wrow[WI];
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    const int q = 8 * i + (lane >> 3);
    const int task = task0 + (q & 31);
    const bf16_t *a, *b;
    epi.weight_rows(task < n_tasks ? task : 0, a, b);
    wrow[i] = q < 32 ? a : b;
  }
  const int w_seg = (lane & 7) * 8;   // this lane's k inside a chunk
  const int w_dst = (lane >> 3) * MG_ROWPAD + (lane & 7) * 8;          // + 8 i rows
  const int koff = (lane >> 5) * 8;                                    // this lane's k-block inside an MFMA step
  const int a_off = (lane & 31) * MG_ROWPAD + koff;                    // + 32 rows for the second tile, + 16 s

  f32x16_t acc0[MTILES], acc1[MTILES];
#pragma unroll
  for (int c = 0; c < MTILES; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc0[c][r] = acc1[c][r] = 0.f;

  u32x4_t wr[WD][WI];   // (a native vector type: arrays of it are kept in registers)
  // this thread's vectors of the three parts of a chunk's activations (beyond the row's end: zeros)
  const bf16_t *parts = (const bf16_t *)in.x;
  const size_t part_stride = (size_t)in.part_units * 64;
  const int x_pitch = n_chunks * MG_KC;
  int x_src[XV], x_dst[XV];
#pragma unroll
  for (int i = 0; i < XV; ++i) {
    const int pos = ((int)threadIdx.x + i * (64 * WAVES)) % XPOS;
    const int m = pos / (MG_KC / 8), x_k = (pos - m * (MG_KC / 8)) * 8;
    x_src[i] = min(row0 + m, m_rows - 1) * x_pitch + x_k;    // rows past the end repeat the last one
    x_dst[i] = m * MG_ROWPAD + x_k;
  }
  u32x4_t xr[XV][MG_PARTS];
  auto load_x = [&](int chunk) {
    const int k = min(chunk, c_end - 1) * MG_KC;
#pragma unroll
    for (int i = 0; i < XV; ++i)
#pragma unroll
      for (int p = 0; p < MG_PARTS; ++p) xr[i][p] = *(const u32x4_t *)(parts + p * part_stride + k + x_src[i]);
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int i = 0; i < XV; ++i)
#pragma unroll
      for (int p = 0; p < MG_PARTS; ++p) *(u32x4_t *)(s_x + (buf * MG_PARTS + p) * PART_ELEMS + x_dst[i]) = xr[i][p];
  };

  load_x(c_begin);
  __builtin_amdgcn_sched_barrier(0);
  store_x(0);
  __builtin_amdgcn_sched_barrier(0);
  load_x(c_begin + 1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < WD; ++j) {
    int k_ = min(c_begin + j, c_end - 1) * MG_KC + w_seg;
    k_ = k_ < n_in ? k_ : 0;   // past the row's end: any finite weights, they meet zero activations
#pragma unroll
    for (int i = 0; i < WI; ++i) wr[j][i] = __builtin_nontemporal_load((const u32x4_t *)(wrow[i] + k_));
  }
  __syncthreads();

  for (int base = c_begin; base < c_end; base += WD) {
#pragma unroll
    for (int j = 0; j < WD; ++j) {
      const int chunk = base + j;
      const int buf = j & 1;   // WD is even, so a chunk's buffer is its slot's parity
      // weights of this chunk into the wave's LDS piece (the MFMAs of the previous chunk have
      // issued their reads of it: one wave's LDS operations stay in order)
#pragma unroll
      for (int i = 0; i < WI; ++i) *(u32x4_t *)(s_w + 8 * i * MG_ROWPAD + w_dst) = wr[j][i];
      __builtin_amdgcn_sched_barrier(0);
      // activations of chunk + 1, requested one iteration ago, into the other buffer
      store_x(buf ^ 1);
      __builtin_amdgcn_sched_barrier(0);
      load_x(chunk + 2);
      __builtin_amdgcn_sched_barrier(0);
      {
        int k_ = min(chunk + WD, c_end - 1) * MG_KC + w_seg;
        k_ = k_ < n_in ? k_ : 0;
#pragma unroll
        for (int i = 0; i < WI; ++i) wr[j][i] = __builtin_nontemporal_load((const u32x4_t *)(wrow[i] + k_));
      }
      __builtin_amdgcn_sched_barrier(0);
      if (chunk < c_end) {
        const bf16_t *xb = s_x + buf * MG_PARTS * PART_ELEMS + a_off;
#pragma unroll
        for (int s = 0; s < MG_KC / 16; ++s) {
          const bf16x8_t a0 = __builtin_bit_cast(bf16x8_t, *(const u32x4_t *)(s_w + a_off + s * 16));
          const bf16x8_t a1 = __builtin_bit_cast(bf16x8_t, *(const u32x4_t *)(s_w + 32 * MG_ROWPAD + a_off + s * 16));
          // smallest part first, so that the large terms are added last; consecutive MFMAs go to
          // different accumulators
#pragma unroll
          for (int p = MG_PARTS - 1; p >= 0; --p) {
#pragma unroll
            for (int c = 0; c < MTILES; ++c) {
              const bf16x8_t b = __builtin_bit_cast(
                  bf16x8_t, *(const u32x4_t *)(xb + p * PART_ELEMS + c * 32 * MG_ROWPAD + s * 16));
              acc0[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b, acc0[c], 0, 0, 0);
              acc1[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b, acc1[c], 0, 0, 0);
            }
          }
        }
      }
      __syncthreads();
    }
  }

  // results: register r <-> task (r/4)*8 + (lane/32)*4 + r%4 of this wave, activation row lane%32
  if constexpr (!SPLIT && !EpiHasLocalReduce<Epi>::value) {
    // The epilogue runs here, and what it writes runs along the tasks (consecutive elements of a
    // row of the hidden state, of q, of the cache, of the split activations), while a lane's
    // registers hold 16 tasks of ONE row: stored as they lie, every store instruction would put
    // 64 single elements into 64 different rows (measured on the gate/up projection of a prompt
    // pass: 178 -> 163 us).  So each 32 x 32 tile is turned in the wave's own piece of LDS (free
    // now; the wave's LDS operations execute in order, no barrier) and the epilogue is called with
    // the tasks across the lanes: 32 consecutive elements per half-wave.
    float *s_t = (float *)s_w;   // [2][32 tasks][33]
    typename Epi::State st;      // (what it gathers about a row is for contexts with tiled weights)
    epi.init(st);
    const int tl = lane & 31, rh = (lane >> 5) * 16;
#pragma unroll
    for (int c = 0; c < MTILES; ++c) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        s_t[t * 33 + (lane & 31)] = acc0[c][r];
        s_t[32 * 33 + t * 33 + (lane & 31)] = acc1[c][r];
      }
      const int task = task0 + tl;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int m = row0 + c * 32 + rh + i;
        const float y0 = s_t[tl * 33 + rh + i], y1 = s_t[32 * 33 + tl * 33 + rh + i];
        if (task < n_tasks && m < m_rows) epi.finish(task, m, rows[m], y0, y1, st);
      }
    }
    return;
  }
  typename Epi::State st;
  epi.init(st);
#pragma unroll
  for (int c = 0; c < MTILES; ++c) {
    const int m = row0 + c * 32 + (lane & 31);
    const bool m_ok = m < m_rows;
    RowDesc rd = rows[m_ok ? m : 0];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int task = task0 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
      if (task < n_tasks) {
        if (SPLIT) {
          float *p = part + (((size_t)by * n_tasks + task) * 2) * m_pad + m;
          if (m < m_pad) { p[0] = acc0[c][r]; p[m_pad] = acc1[c][r]; }
        } else if (m_ok) {
          epi.finish(task, m, rd, acc0[c][r], acc1[c][r], st);
        }
      }
    }
    if (!SPLIT && MTILES == 1 && m_ok) epi.end(m, rd, st);
  }
}

// ------------------------------------------------------------------ the contraction on tiled weights
//
// A context that owns enough memory keeps a second copy of every bf16 projection matrix as fp16 and
// in the order the MFMA consumes it: for each block of 16 tasks (rows 0..15 of the operand: their
// first weight rows, rows 16..31: their second) and for each 64-wide chunk of k, one 4 KiB tile
// [step 0..3][lane 0..63][8 elements], lane l of step s holding row l % 32, elements
// 64 c + 16 s + 8 (l / 32) .. + 7.  A wave then loads a whole A operand with one fully coalesced
// instruction (64 lanes x 16 bytes, consecutive) straight into registers: the weights never touch
// LDS, which leaves LDS to the activations, and a wave can hold several A tiles, so that every B
// operand it reads feeds several MFMAs.  Both weight rows of a task end up in one lane: result
// registers r and r + 8 (r < 8) are task (r/4)*8 + (l/32)*4 + r%4 of the block.
// Every row has a power of two that brings its largest weight just below 2^15 (`wdown`, 32 words a
// block, undoes it).  A bf16 weight has 8 significant bits and fp16 a least unit of 2^-24, so a weight
// is exact down to 2^-31 of its row's largest and off by at most 2^-39 of that below.  Both are written
// once, when the context is created, from the same weight_rows() of the epilogue that the kernels use.
constexpr int TG_TILE = 32 * MG_KC;   // elements of one A tile of one chunk
constexpr int TG_PARTS = 2;           // fp16 parts of an activation
constexpr int TG_FOLD_CHUNKS = 10;    // chunks that go into one set of sums

constexpr size_t tg_tiled_elems(int n_tasks, int n_in) {
  return (size_t)((n_tasks + TG_TASKS - 1) / TG_TASKS) * ((n_in + MG_KC - 1) / MG_KC) * TG_TILE;
}
constexpr size_t tg_blocks(int n_tasks) { return (size_t)((n_tasks + TG_TASKS - 1) / TG_TASKS); }

// Writes the tiles of eight operand rows of a block and what undoes their scales.  A wave takes the
// eight rows eight elements at a time, so that it reads 128 bytes of a row and writes 128 bytes of a tile
// in one piece.  (Infinities and NaN have no part in a row's largest magnitude.)
//
// HELD vectors a thread keeps between the two passes over its rows: inputs of up to 1024 HELD elements are
// read once (a second read of them from memory cost a third of the time: 28 layers of d 3584, FFN 18944
// 11.4 ms, 6.9 with one).  HELD 0: any input, read twice.
constexpr int TW_THREADS = 1024, TW_ROWS = 8, TW_HELD = 20;
template <typename Epi, int HELD>
__global__ void __launch_bounds__(TW_THREADS)
tile_weights_k(Epi epi, int n_tasks, int n_in, int n_chunks, float *__restrict__ wdown, f16_t *__restrict__ dst) {
  constexpr int STRIDE = TW_THREADS / TW_ROWS;   // vectors of eight elements from trip to trip
  __shared__ uint32_t s_max[TW_THREADS / 64][TW_ROWS];
  const int block = blockIdx.x / (32 / TW_ROWS), r = threadIdx.x % TW_ROWS;
  const int op_row = blockIdx.x % (32 / TW_ROWS) * TW_ROWS + r, task = block * TG_TASKS + op_row % TG_TASKS;
  const bf16_t *a, *b;
  epi.weight_rows(task < n_tasks ? task : 0, a, b);
  const bf16_t *row = op_row < TG_TASKS ? a : b;
  const int vec0 = threadIdx.x / TW_ROWS, n_vecs = n_chunks * (MG_KC / 8);
  auto load = [&](int vec) {   // beyond the matrix: zeros
    const bool real = task < n_tasks && vec * 8 < n_in;
    const u32x4_t v = *(const u32x4_t *)(row + (real ? vec * 8 : 0)), zero = {0u, 0u, 0u, 0u};
    return real ? v : zero;
  };
  uint32_t m = 0u;
  auto consider = [&](const u32x4_t &v) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t u = (h ? v[e] & 0xffff0000u : v[e] << 16) & 0x7fffffffu;
        m = max(m, u < 0x7f800000u ? u : 0u);
      }
  };
  u32x4_t held[HELD > 0 ? HELD : 1];
  if constexpr (HELD > 0) {
#pragma unroll
    for (int i = 0; i < HELD; ++i) held[i] = load(vec0 + i * STRIDE);   // (beyond the last: zeros)
#pragma unroll
    for (int i = 0; i < HELD; ++i) consider(held[i]);
  } else {
    for (int vec = vec0; vec < n_vecs; vec += STRIDE) consider(load(vec));
  }
#pragma unroll
  for (int o = 32; o >= TW_ROWS; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  if ((threadIdx.x & 63) < TW_ROWS) s_max[threadIdx.x >> 6][r] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < TW_THREADS / 64; ++w) m = max(m, s_max[w][r]);
  const int E = scale_exponent(m >> 23);
  const float up = scale_up(E);
  if (vec0 == 0) wdown[block * 32 + op_row] = scale_down(E);
  auto store = [&](int vec, const u32x4_t &v) {
    f16x8_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[2 * e] = (f16_t)(__uint_as_float(v[e] << 16) * up);
      o[2 * e + 1] = (f16_t)(__uint_as_float(v[e] & 0xffff0000u) * up);
    }
    *(f16x8_t *)(dst + ((size_t)block * n_chunks + vec / 8) * TG_TILE + vec % 8 / 2 * 512 + (op_row + vec % 2 * 32) * 8) = o;
  };
  if constexpr (HELD > 0) {
#pragma unroll
    for (int i = 0; i < HELD; ++i)
      if (vec0 + i * STRIDE < n_vecs) store(vec0 + i * STRIDE, held[i]);
  } else {
    for (int vec = vec0; vec < n_vecs; vec += STRIDE) store(vec, load(vec));
  }
}

// Tile -> (task tile, row tile).  Consecutive workgroup ids go to consecutive XCDs, each with its
// own L2: the row tiles of one task tile read the same weights, so they get ids 8 apart (same XCD,
// launched together) and the weights cross HBM once for them.  (xcd_groups: chosen by the launch;
// measured to pay for few, long k ranges: gate/up of a prompt pass 191 -> 169 us, while down with
// its many short ranges lost, 101 -> 116 us.)
__device__ __forceinline__ void tile_place(const TileCover &tc, int t, int &bx, int &bz) {
  if (!tc.xcd_groups) {
    bz = t / tc.n_task_tiles;
    bx = t - bz * tc.n_task_tiles;
    return;
  }
  const int even = tc.n_task_tiles / 8 * 8;          // task tiles in whole groups of eight
  const int per_group = 8 * tc.n_row_tiles, group = t / per_group;
  if (group * 8 < even) {
    const int r = t - group * per_group;
    bx = group * 8 + (r & 7);
    bz = r >> 3;
  } else {
    const int r = t - even * tc.n_row_tiles, rest = tc.n_task_tiles - even;
    bz = r / rest;
    bx = even + r - bz * rest;
  }
}

// dynamic LDS of mfma_tiled_k: three buffers of two parts of 32*MTILES padded activation rows, or
// the four waves' pieces for turning the result tiles, whichever is larger; the activation rows' scales and
// arg-max keys, the weight rows' scales, what the epilogue needs of the rows
constexpr int TG_BUFS = 3;
constexpr int TG_TPITCH = 36;   // floats of a row of a turned tile: 32 tasks and a skew of one 16-byte word
constexpr size_t tg_scales_at(int mtiles) {
  const size_t x = sizeof(f16_t) * TG_BUFS * TG_PARTS * 32 * mtiles * MG_ROWPAD;
  const size_t t = sizeof(float) * TG_WAVES * 2 * 32 * TG_TPITCH;
  return x > t ? x : t;
}
constexpr size_t tg_rows_at(int mtiles, int tb) {
  return tg_scales_at(mtiles) + (sizeof(float) + sizeof(unsigned long long)) * 32 * mtiles + sizeof(float) * 64 * TG_WAVES * tb;
}
constexpr size_t tg_lds_bytes(int mtiles, int tb) { return tg_rows_at(mtiles, tb) + sizeof(RowFacts) * 32 * mtiles; }

// A workgroup of four waves takes 128 * TB tasks (wave w: 2 * TB A tiles of 16 tasks),
// one k range and one tile of 32 * MTILES activation rows.  WHOLE: the launch has tiles that end in
// the epilogue here (others only write partial sums and the epilogue's code is left out).
//
// The loop over the chunks is written MFMA by MFMA in the order it is to execute, with a scheduling
// barrier after each: the MFMAs of one B operand (2 * TB of them) form a group, and between them
// issue the LDS read of the B operand PD groups ahead, a reload of weights whose last use has just
// been issued, and pieces of the staging of the next chunk's activations (an fp32 load, two
// elements cut into fp16 parts, an LDS write).  Left to itself the compiler puts each LDS read next
// to its use and the loads at the end of the chunk, and the MFMA pipe then idles half the time.
// Activations go through three LDS buffers, so that one barrier per chunk, placed before the first
// read of the next chunk, is enough: a wave writes the buffer two chunks ahead of what the slowest
// wave can still read.
//
// Every MFMA rounds the running sum to 32 bits, and what K / 8 of them leave grows with the root of
// their number: 5.4e-7 of the result for the 448 of a k of 3584.  So the sums of TG_FOLD_CHUNKS chunks
// are added to a second set of registers and begin at zero again (error of the heads' logits against 64
// bits, k of 3584: 2.4e-7, and 2.5e-7 to 3.2e-7 as three bf16 parts with k cut into ranges; steps of 48
// and 96 sequences take under 1 % longer for it).  64 tasks a wave have no registers for that; they
// serve gate/up, whose k is d_model (MLP of 18944, 49 to 256 rows: 5.3e-7 to 8.7e-7; three bf16 parts 6.7e-7
// to 1.16e-6).
//
// A tile that ends here turns its results in LDS, eight rows of four tasks a lane and store, and finds what the
// epilogue needs of a row (its scale, its cache entries' place) once per workgroup, at the start: with single
// words and a chain of loads per row the epilogue took 10 to 15 us of a round of 185 (q/k/v of 1023 rows, d 4096:
// 134 -> 116 us).
template <int MTILES, int TB, typename Epi, bool WHOLE>
__device__ __forceinline__ void
tiled_tile(const Epi &epi, const f16_t *__restrict__ tiled, const float *__restrict__ wdown, const RowDesc *__restrict__ rows, int m_rows,
           const ProjIn &in, int n_in, int n_tasks, const TileCover &tc, float *__restrict__ part, uint4 *tg_smem,
           int bx, int row0, bool whole, int split, int cut_tile) {
  static_assert(MTILES * TB <= 6 && MTILES <= 4 && TB <= 2, "accumulators take at most 192 registers");
  constexpr int MROWS = 32 * MTILES;
  constexpr int NT = 64 * TG_WAVES;
  constexpr int XV = MROWS * (MG_KC / 8) / NT;      // vectors of eight activations a thread stages per chunk
  static_assert(XV == MTILES, "every thread stages the same number of vectors");
  constexpr int PART_ELEMS = MROWS * MG_ROWPAD;
  constexpr int STEPS = MG_KC / 16;
  constexpr int QT = 2 * TB;                        // A tiles per wave
  constexpr int NB = TG_PARTS * MTILES;             // B operands (and groups of QT MFMAs) per step
  constexpr int GROUPS = STEPS * NB;
  constexpr int W = 4, PD = W - 1;                  // window of B operands in registers, and how far ahead they are read
  static_assert(GROUPS % W == 0 && NB >= 2, "an operand keeps its place in the window from chunk to chunk");
  constexpr int BAR = GROUPS - PD;                  // group before which the next chunk's activations must be visible
  static_assert(BAR >= 2 * NB, "the staging of the next chunk ends two steps into this one");
  constexpr int PER = (QT + NB - 1) / NB;           // weight loads per group
  constexpr int BUF_ELEMS = TG_PARTS * PART_ELEMS;
  constexpr int TASKS = 32 * TG_WAVES * TB;
  constexpr bool FOLD = TB == 1;
  constexpr int SEGMENT = FOLD ? TG_FOLD_CHUNKS : 1 << 20;   // chunks that are added up before they are folded
  static_assert(SEGMENT % 2 == 0, "whole turns of the ring of chunks");
  constexpr size_t SCALE_AT = tg_scales_at(MTILES);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (known to be uniform: addresses of weights stay scalar)
  f16_t *s_x = (f16_t *)tg_smem;                    // [3][2][MROWS * MG_ROWPAD]
  float *s_down = (float *)((char *)tg_smem + SCALE_AT);   // per activation row: what undoes its scale
  float *s_wdown = (float *)((char *)tg_smem + SCALE_AT + (sizeof(float) + sizeof(unsigned long long)) * MROWS);   // and per weight row
  RowFacts *s_rows = (RowFacts *)((char *)tg_smem + tg_rows_at(MTILES, TB));   // what the epilogue needs of the rows

  const int n_chunks = (n_in + MG_KC - 1) / MG_KC;
  const int c_begin = whole ? 0 : split * tc.chunks_per_split;
  const int c_end = whole ? n_chunks : min(n_chunks, c_begin + tc.chunks_per_split);
  const int n_blocks = (n_tasks + TG_TASKS - 1) / TG_TASKS;
  const int tb0 = (bx * TG_WAVES + wave) * TB;       // this wave's first 32 tasks

  const f16_t *abase[QT];   // A tile q: block 2 tb0 + q (past the end: the last one)
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int block = min(2 * tb0 + q, n_blocks - 1);
    abase[q] = tiled + (size_t)block * n_chunks * TG_TILE + lane * 8;
  }
  const int a_off = (lane & 31) * MG_ROWPAD + (lane >> 5) * 8;

  f32x16_t acc[QT][MTILES];
#pragma unroll
  for (int q = 0; q < QT; ++q)
#pragma unroll
    for (int c = 0; c < MTILES; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[q][c][r] = 0.f;
  f32x16_t folded[FOLD ? QT : 1][FOLD ? MTILES : 1];
  if constexpr (FOLD)
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
      for (int c = 0; c < MTILES; ++c) folded[q][c] = acc[q][c];

  // chunks of weights in registers, slot = (chunk - c_begin) % RING
  constexpr int RING = 2;
  u32x4_t wr[RING][QT][STEPS];
  // all loads are unconditional (chunks past the range are clamped to its last one) so that the
  // compiler waits for exactly the loads a step needs; a chunk past the range is staged as zeros
  auto load_a1 = [&](int slot, int q, int s, int chunk) {
    wr[slot][q][s] = __builtin_nontemporal_load(
        (const u32x4_t *)(abase[q] + (size_t)min(chunk, c_end - 1) * TG_TILE + s * 512));
  };

  int x_src[XV];
  float x_up[XV];
  const int x_kv = ((int)threadIdx.x & 7) * 8;       // k of this thread's vectors inside a chunk
#pragma unroll
  for (int n = 0; n < XV; ++n) {
    const int m = ((int)threadIdx.x + n * NT) >> 3;
    x_src[n] = min(row0 + m, m_rows - 1) * in.stride;                 // rows past the end repeat the last one
  }
  const int x_dst = ((int)threadIdx.x >> 3) * MG_ROWPAD + x_kv;         // + 32 rows from vector to vector
  float4 xr[XV][2];
  auto load_x1 = [&](int n, int half, int chunk) {
    const int k = min(chunk, c_end - 1) * MG_KC + x_kv;
    xr[n][half] = *(const float4 *)(in.x + x_src[n] + (k < n_in ? k : 0) + half * 4);
  };
  // elements 2 e and 2 e + 1 of vector n: two fp16 parts each, zeros where there is nothing to
  // multiply; every second call writes four elements to the buffer at `at`
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  u32x2_t xh, xl;
  auto cut_x2 = [&](int n, int e, int at, bool real) {
    const float4 v = xr[n][e >> 1];
    const float f0 = ((e & 1) ? v.z : v.x) * x_up[n], f1 = ((e & 1) ? v.w : v.y) * x_up[n];
    const f16_t h0 = (f16_t)f0, h1 = (f16_t)f1;
    const f16_t l0 = (f16_t)(f0 - (float)h0), l1 = (f16_t)(f1 - (float)h1);
    const uint32_t h = (uint32_t)__builtin_bit_cast(uint16_t, h0) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
    const uint32_t l = (uint32_t)__builtin_bit_cast(uint16_t, l0) | ((uint32_t)__builtin_bit_cast(uint16_t, l1) << 16);
    xh[e & 1] = real ? h : 0u;
    xl[e & 1] = real ? l : 0u;
    if (e & 1) {
      *(u32x2_t *)(s_x + at + x_dst + n * 32 * MG_ROWPAD + 2 * (e - 1)) = xh;
      *(u32x2_t *)(s_x + at + PART_ELEMS + x_dst + n * 32 * MG_ROWPAD + 2 * (e - 1)) = xl;
    }
  };
  // B operand i of step s of a buffer: the smaller part first (the large terms are added last), row tiles inside
  auto load_b1 = [&](int i, int at, int s) -> u32x4_t {
    const int p = TG_PARTS - 1 - i / MTILES, c = i % MTILES;
    return *(const u32x4_t *)(s_x + at + p * PART_ELEMS + c * 32 * MG_ROWPAD + s * 16 + a_off);
  };

  // the first loads: the rows' magnitudes (of a row per eight lanes) and activations, then the weights
  constexpr int LPR = MG_KC / 8;
  const int xr0 = (int)threadIdx.x >> 3;
  RowExponent<LPR> mag0(in.row_max, min(row0 + xr0, m_rows - 1), threadIdx.x & 7);
  RowFacts facts;
  if constexpr (WHOLE && EpiFacts<Epi>::value) {
    const int r = min(row0 + min((int)threadIdx.x, MROWS - 1), m_rows - 1);
    if (whole) facts = epi.row_facts(r, rows[r]);
  }
  float wd[TB];             // of weight row threadIdx.x + NT u of the workgroup's 64 TG_WAVES TB
#pragma unroll
  for (int u = 0; u < TB; ++u) {
    const int r = (int)threadIdx.x + NT * u;
    wd[u] = wdown[(size_t)min(bx * (2 * TG_WAVES * TB) + r / 32, n_blocks - 1) * 32 + r % 32];
  }
#pragma unroll
  for (int n = 0; n < XV; ++n) { load_x1(n, 0, c_begin); load_x1(n, 1, c_begin); }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < RING; ++j)
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int q = 0; q < QT; ++q) load_a1(j, q, s, c_begin + j);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < XV; ++n) {
    const int m = xr0 + n * (NT / LPR);
    const int E = scale_exponent(n == 0 ? mag0.get() : RowExponent<LPR>(in.row_max, min(row0 + m, m_rows - 1), threadIdx.x & 7).get());
    x_up[n] = scale_up(E);
    if (x_kv == 0) s_down[((int)threadIdx.x + n * NT) >> 3] = scale_down(E);
  }
#pragma unroll
  for (int u = 0; u < TB; ++u) s_wdown[(int)threadIdx.x + NT * u] = wd[u];
  if constexpr (WHOLE && EpiFacts<Epi>::value) {
    if (whole && (int)threadIdx.x < MROWS) s_rows[threadIdx.x] = facts;
  }
#pragma unroll
  for (int n = 0; n < XV; ++n) {
#pragma unroll
    for (int e = 0; e < 4; ++e) cut_x2(n, e, 0, c_begin * MG_KC + x_kv < n_in);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < XV; ++n) { load_x1(n, 0, c_begin + 1); load_x1(n, 1, c_begin + 1); }
  __syncthreads();
  u32x4_t bw[W];
#pragma unroll
  for (int o = 0; o < PD; ++o) bw[o] = load_b1(o % NB, 0, o / NB);

  int cur = 0, nxt = BUF_ELEMS, aft = 2 * BUF_ELEMS;   // LDS buffers of this chunk, the next, the one after
  for (int seg = c_begin; seg < c_end; seg += SEGMENT) {
    const int seg_end = min(c_end, seg + SEGMENT);
    for (int base = seg; base < seg_end; base += RING) {
#pragma unroll
      for (int j = 0; j < RING; ++j) {
        const int chunk = base + j;
        const bool next_real = chunk + 1 < c_end && (chunk + 1) * MG_KC + x_kv < n_in;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int o = s * NB + i;
            if (o == BAR) __syncthreads();
#pragma unroll
            for (int q = 0; q < QT; ++q) {
              acc[q][i % MTILES] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, wr[j][q][s]),
                                                                          __builtin_bit_cast(f16x8_t, bw[o % W]),
                                                                          acc[q][i % MTILES], 0, 0, 0);
              if (q == 0) {
                const int n = o + PD;
                bw[n % W] = n < GROUPS ? load_b1(n % NB, cur, n / NB) : load_b1((n - GROUPS) % NB, nxt, (n - GROUPS) / NB);
              }
              if (q == 1 % QT) {
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                  const int qq = i * PER + e;
                  if (qq < QT) {
                    if (s == 0) load_a1((j + RING - 1) % RING, qq, STEPS - 1, chunk - 1 + RING);   // last step of the chunk before
                    else load_a1(j, qq, s - 1, chunk + RING);
                  }
                }
              }
              if (q == QT - 1) {
                // vector i / 2 of the next chunk: four pieces of two elements over the groups of steps 0 and 1
                if (s < 2) cut_x2(i / 2, (i & 1) + 2 * s, nxt, next_real);
                if (s == 2) load_x1(i / 2, i & 1, chunk + 2);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
        const int old = cur;
        cur = nxt;
        nxt = aft;
        aft = old;
      }
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int q = 0; q < QT; ++q)
#pragma unroll
        for (int c = 0; c < MTILES; ++c) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            folded[q][c][r] += acc[q][c][r];
            acc[q][c][r] = 0.f;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    }
  }

  // number r (0..15) of what a lane holds of 32 tasks jb and row tile c: task 32 (tb0 + jb) + task_of(r),
  // activation row lane % 32, sums y_of(0 / 1, jb, c, r) of its two weight rows
  auto task_of = [&](int r) { return (r >> 3) * TG_TASKS + ((r >> 2) & 1) * 8 + (lane >> 5) * 4 + (r & 3); };
  auto y_of = [&](int which, int jb, int c, int r) { return acc[2 * jb + (r >> 3)][c][(r & 7) + 8 * which]; };
  // (one factor after the other: their product may lie outside the range of an fp32 where the result does not)
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const float4 *w4 = (const float4 *)(s_wdown + (wave * QT + q) * 32 + 4 * (lane >> 5));   // operand rows 8 j + 4 (lane / 32) + 0..3
    float w[16];
#pragma unroll
    for (int j = 0; j < 4; ++j) *(float4 *)(w + 4 * j) = w4[2 * j];
#pragma unroll
    for (int c = 0; c < MTILES; ++c) {
      const float xd = s_down[c * 32 + (lane & 31)];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if constexpr (FOLD) acc[q][c][r] = folded[q][c][r];
        acc[q][c][r] = acc[q][c][r] * xd * w[r];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (!whole) {
    float *base = part + ((size_t)split * tc.n_cut + cut_tile) * TASKS * 2 * tc.m_pitch;
#pragma unroll
    for (int jb = 0; jb < TB; ++jb)
#pragma unroll
      for (int c = 0; c < MTILES; ++c) {
        const int m = c * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int tl = (wave * TB + jb) * 32 + task_of(r);
          if (m < tc.m_pitch) {
            float *p = base + (size_t)tl * 2 * tc.m_pitch + m;
            p[0] = y_of(0, jb, c, r);
            p[tc.m_pitch] = y_of(1, jb, c, r);
          }
        }
      }
    return;
  }
  if constexpr (WHOLE) {
    // the epilogue's stores run along the tasks: each 32 x 32 tile is turned in the wave's piece of
    // LDS (the buffers are free once every wave has left the loop)
    __syncthreads();
    float *s_t = (float *)tg_smem + wave * 2 * 32 * TG_TPITCH;
    const int tl = lane & 31, rh = (lane >> 5) * 16;
    if constexpr (EpiHasLocalReduce<Epi>::value) {
      // a running state per activation row (the heads' arg-max): formed while a lane holds tasks of one
      // row, combined over the workgroup in LDS, so that one atomic per row and workgroup reaches memory
      unsigned long long *s_best = (unsigned long long *)((char *)tg_smem + SCALE_AT + sizeof(float) * MROWS);
      if (threadIdx.x < MROWS) s_best[threadIdx.x] = 0ull;
      __syncthreads();
#pragma unroll
      for (int c = 0; c < MTILES; ++c) {
        typename Epi::State st;
        epi.init(st);
#pragma unroll
        for (int jb = 0; jb < TB; ++jb) {
          const int t0 = (tb0 + jb) * 32;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int tt = task_of(r);
            if (t0 + tt < n_tasks) epi.consider(t0 + tt, y_of(0, jb, c, r), y_of(1, jb, c, r), st);
            s_t[tt * 33 + (lane & 31)] = y_of(0, jb, c, r);
            s_t[32 * 33 + tt * 33 + (lane & 31)] = y_of(1, jb, c, r);
          }
          // (a few at a time: all sixteen in flight, times the tiles, is more than the registers hold)
#pragma unroll 4
          for (int i = 0; i < 16; ++i) {
            const int m = row0 + c * 32 + rh + i;
            if (t0 + tl < n_tasks && m < m_rows)
              epi.store_pair(t0 + tl, rows[m], s_t[tl * 33 + rh + i], s_t[32 * 33 + tl * 33 + rh + i]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        epi.reduce_local(st, s_best + c * 32 + (lane & 31));
      }
      __syncthreads();
      const int m = row0 + (int)threadIdx.x;
      if (threadIdx.x < MROWS && m < m_rows && s_best[threadIdx.x]) epi.end_reduced(rows[m], s_best[threadIdx.x]);
    } else if constexpr (EpiRow<Epi>::max) {
      // one value per pair of weight rows: it is formed while a lane still holds 16 tasks of one row,
      // so that the row's scale is one per lane and its largest magnitude stays in the lane
#pragma unroll
      for (int c = 0; c < MTILES; ++c) {
        const int mine = row0 + c * 32 + (lane & 31);
        const float inv = s_rows[c * 32 + (lane & 31)].inv;
        typename Epi::State st;
        epi.init(st);
#pragma unroll
        for (int jb = 0; jb < TB; ++jb) {
          const int t0 = (tb0 + jb) * 32;
          if (tc.max_words > 1) epi.init(st);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int r = 4 * j + e;
              v[e] = epi.value(inv, y_of(0, jb, c, r), y_of(1, jb, c, r));
              if (t0 + task_of(r) < n_tasks) st.amax = max(st.amax, magnitude_bits(v[e]));
            }
            *(float4 *)(s_t + (lane & 31) * TG_TPITCH + task_of(4 * j)) = make_float4(v[0], v[1], v[2], v[3]);
            __builtin_amdgcn_sched_barrier(0);   // (registers: sixteen exponentials at once are too many)
          }
          // eight rows a store, four tasks a lane
          float4 out[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) out[i] = *(const float4 *)(s_t + ((lane >> 3) + 8 * i) * TG_TPITCH + (lane & 7) * 4);
          const int task = t0 + (lane & 7) * 4;   // (the number of tasks is a multiple of four)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int m = row0 + c * 32 + (lane >> 3) + 8 * i;
            if (task < n_tasks && m < m_rows) epi.store_values(task, m, out[i]);
          }
          if (tc.max_words > 1 || jb == TB - 1) {
            st.amax = max(st.amax, (uint32_t)__shfl_xor((int)st.amax, 32, 64));
            const int word = tc.max_words > 1 ? tb0 + jb : bx * TG_WAVES + wave;
            if (lane < 32 && mine < m_rows && (tc.max_words > 1 ? t0 : tb0 * 32) < n_tasks) epi.put_row(mine, word, st);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else if constexpr (EpiFacts<Epi>::value) {
      // pairs, four tasks of a row a lane: 32 tasks lie in one head, and what depends on the row is in LDS
#pragma unroll
      for (int jb = 0; jb < TB; ++jb) {
        const int task = (tb0 + jb) * 32 + (lane & 7) * 4;
#pragma unroll
        for (int c = 0; c < MTILES; ++c) {
#pragma unroll
          for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              *(float4 *)(s_t + (32 * w + (lane & 31)) * TG_TPITCH + task_of(4 * j)) =
                  make_float4(y_of(w, jb, c, 4 * j), y_of(w, jb, c, 4 * j + 1), y_of(w, jb, c, 4 * j + 2), y_of(w, jb, c, 4 * j + 3));
          typename Epi::Turn turn[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) turn[i] = epi.load_turn(task, s_rows[c * 32 + (lane >> 3) + 8 * i]);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int rl = (lane >> 3) + 8 * i, m = row0 + c * 32 + rl;
            const float *p = s_t + rl * TG_TPITCH + (lane & 7) * 4;
            if (task < n_tasks && m < m_rows)
              epi.finish4(task, m, s_rows[c * 32 + rl], *(const float4 *)p, *(const float4 *)(p + 32 * TG_TPITCH), turn[i]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
      typename Epi::State st;
      epi.init(st);
#pragma unroll
      for (int jb = 0; jb < TB; ++jb) {
#pragma unroll
        for (int c = 0; c < MTILES; ++c) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int tt = task_of(r);
            s_t[tt * 33 + (lane & 31)] = y_of(0, jb, c, r);
            s_t[32 * 33 + tt * 33 + (lane & 31)] = y_of(1, jb, c, r);
          }
          const int task = (tb0 + jb) * 32 + tl;
#pragma unroll 2
          for (int i = 0; i < 16; ++i) {
            const int m = row0 + c * 32 + rh + i;
            const float y0 = s_t[tl * 33 + rh + i], y1 = s_t[32 * 33 + tl * 33 + rh + i];
            if (task < n_tasks && m < m_rows) epi.finish(task, m, rows[m], y0, y1, st);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
}

template <int MTILES, int TB, typename Epi, bool WHOLE>
__global__ void __launch_bounds__(64 * TG_WAVES)
mfma_tiled_k(Epi epi, const f16_t *__restrict__ tiled, const float *__restrict__ wdown,
             const RowDesc *__restrict__ rows, int m_rows, ProjIn in, int n_in, int n_tasks, TileCover tc,
             float *__restrict__ part) {
  extern __shared__ uint4 tg_smem[];
  clear_words(in);
  int t, split = 0, bx, bz;
  const bool whole = WHOLE && (int)blockIdx.x < tc.n_whole;
  if (whole) {
    t = blockIdx.x;
  } else {
    const int i = blockIdx.x - tc.n_whole;
    split = i / tc.n_cut;
    t = tc.n_whole + i - split * tc.n_cut;
  }
  tile_place(tc, t, bx, bz);
  tiled_tile<MTILES, TB, Epi, WHOLE>(epi, tiled, wdown, rows, m_rows, in, n_in, n_tasks, tc, part, tg_smem, bx, bz * 32 * MTILES, whole, split,
                                     t - tc.n_whole);
}

// Whole tiles of three and of two blocks of rows in one launch (see MixedCover): the higher ones first.
// (gate/up of 18944 tasks, 511 rows: 308 -> 285 us.)
template <int TB, typename Epi>
__global__ void __launch_bounds__(64 * TG_WAVES)
mfma_tiled_mixed_k(Epi epi, const f16_t *__restrict__ tiled, const float *__restrict__ wdown,
                   const RowDesc *__restrict__ rows, int m_rows, ProjIn in, int n_in, int n_tasks, MixedCover mc) {
  extern __shared__ uint4 tg_smem[];
  clear_words(in);
  int t = blockIdx.x, k = 0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (k == i && t >= mc.part[i].n_task_tiles * mc.part[i].n_row_tiles) {
      t -= mc.part[i].n_task_tiles * mc.part[i].n_row_tiles;
      k = i + 1;
    }
  TileCover tc = mc.part[0];
#pragma unroll
  for (int i = 1; i < 4; ++i)
    if (k == i) tc = mc.part[i];
  int bx, bz;
  tile_place(tc, t, bx, bz);
  if (k & 1) bx += mc.part[0].n_task_tiles;   // (0, 1: the higher tiles of the first and of the other task tiles; 2, 3: the lower ones)
  if (k < 2) tiled_tile<3, TB, Epi, true>(epi, tiled, wdown, rows, m_rows, in, n_in, n_tasks, tc, nullptr, tg_smem, bx, bz * 96, true, 0, 0);
  else tiled_tile<2, TB, Epi, true>(epi, tiled, wdown, rows, m_rows, in, n_in, n_tasks, tc, nullptr, tg_smem, bx,
                                    (k == 2 ? mc.part[0].n_row_tiles : mc.part[1].n_row_tiles) * 96 + bz * 64, true, 0, 0);
}

// ------------------------------------------------------------------ finishing

// Where the partial sums of (task, row) lie, one range of k after the other `stride` floats apart.
// Both kernels cut a projection into tiles for this purpose; mfma_rows_k into a single one.
struct PartialSums {
  const float *part;
  int n_split, m_pitch, tasks_per_tile, rows_per_tile;
  TileCover tc;
  __device__ __forceinline__ size_t stride() const { return (size_t)tc.n_cut * tasks_per_tile * 2 * m_pitch; }
};

// The partial sums of one (task, row) over the k ranges, added in the order of the ranges.  All
// loads are issued before the first is used: a loop that loads and adds pays a memory round trip
// per trip, and a projection with few tiles has up to MG_MAX_SPLIT ranges.
// MAXS: the most ranges this instance adds (8 or MG_MAX_SPLIT): the loads live in 2 * MAXS
// registers, and a finishing launch with hundreds of workgroups wants two of them on a CU
template <int MAXS>
__device__ __forceinline__ void sum_splits(const float *__restrict__ p, size_t stride, int n_split, int m_pitch,
                                           float &y0, float &y1) {
  float a[MAXS], b[MAXS];
#pragma unroll
  for (int i = 0; i < MAXS; ++i) { const int s = i < n_split ? i : 0; a[i] = p[s * stride]; b[i] = p[s * stride + m_pitch]; }
#pragma unroll
  for (int i = 0; i < MAXS; ++i) if (i < n_split) { y0 += a[i]; y1 += b[i]; }
}

// sums the k-split partials and runs the epilogue: one thread per activation row and group of
// `tasks_per_thread` consecutive tasks, for epilogues that keep a running state worth reducing
// before it goes to memory (the arg-max of the vocabulary heads).  The running states of a
// workgroup's threads that serve the same activation row are combined in LDS (64-bit maximum), so
// that one atomic per row and workgroup reaches memory; with that the groups can be small (eight
// tasks: every thread issues all loads of a k range at once and the launch has thousands of
// waves; with 64 tasks per thread a head of 158 497 rows was 620 waves that each walked 32 dependent
// round trips, 59 us).
template <typename Epi>
__global__ void __launch_bounds__(256)
mfma_finish_k(Epi epi, const RowDesc *__restrict__ rows, int m_rows, int n_tasks, int n_split,
              const float *__restrict__ part, int m_pad, int tasks_per_thread) {
  __shared__ unsigned long long s_best[256];   // per activation row of this workgroup (m_pad <= 256)
  s_best[threadIdx.x] = 0ull;
  __syncthreads();
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int group = idx / m_pad, m = idx - group * m_pad;
  const int t_begin = group * tasks_per_thread;
  if (t_begin < n_tasks && m < m_rows) {
    const int t_end = min(n_tasks, t_begin + tasks_per_thread);
    typename Epi::State st;
    epi.init(st);
    const RowDesc rd = rows[m];
    // eight tasks at a time: the loads of their partial sums of one k range are issued together
    // (a thread that takes its tasks one by one pays a round trip per task and range); every task's
    // ranges are still added in their order
    constexpr int G = 8;
    const size_t stride = (size_t)n_tasks * 2 * m_pad;
    for (int task = t_begin; task < t_end; task += G) {
      float y0[G], y1[G];
#pragma unroll
      for (int i = 0; i < G; ++i) y0[i] = y1[i] = 0.f;
      for (int s = 0; s < n_split; ++s) {
        float a[G], b[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
          const float *p = part + s * stride + ((size_t)min(task + i, t_end - 1) * 2) * m_pad + m;
          a[i] = p[0];
          b[i] = p[m_pad];
        }
#pragma unroll
        for (int i = 0; i < G; ++i) { y0[i] += a[i]; y1[i] += b[i]; }
      }
#pragma unroll
      for (int i = 0; i < G; ++i)
        if (task + i < t_end) epi.finish(task + i, m, rd, y0[i], y1[i], st);
    }
    epi.reduce_local(st, s_best + m);
  }
  __syncthreads();
  if ((int)threadIdx.x < m_rows && s_best[threadIdx.x]) epi.end_reduced(rows[threadIdx.x], s_best[threadIdx.x]);
}

// What an epilogue needs besides the sums, requested before they are ready, if `wanted` (a finishing launch
// for eight rows has four times as many threads as pairs: q/k/v 6.2 us with the others' requests, 5.3 without)
template <typename Epi> __device__ __forceinline__ auto load_old(const Epi &epi, int task, int m, const RowDesc &rd, bool wanted) {
  if constexpr (EpiReadsOld<Epi>::value) {
    typename Epi::Old o{};
    if (wanted) o = epi.load_old(task, m, rd);
    return o;
  } else {
    return 0;
  }
}
// What an epilogue gathers about a row, combined over the LANES neighbouring lanes that have finished
// tasks of it (shuffles: a fixed order) and handed on by the first of them as part `i`
template <int LANES, typename Epi>
__device__ __forceinline__ void hand_on_row(const Epi &epi, int m, bool row_live, typename Epi::State st, int i) {
  if constexpr (EpiRow<Epi>::sum || EpiRow<Epi>::max) {
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) {
      if constexpr (EpiRow<Epi>::sum) st.ssq += __shfl_xor(st.ssq, o, 64);
      if constexpr (EpiRow<Epi>::max) st.amax = max(st.amax, (uint32_t)__shfl_xor((int)st.amax, o, 64));
    }
    if ((threadIdx.x & (LANES - 1)) == 0 && row_live) epi.put_row(m, i, st);
  }
}
template <typename Epi, typename Old>
__device__ __forceinline__ void finish_pair(const Epi &epi, int task, int m, const RowDesc &rd, float y0, float y1, const Old &old,
                                            typename Epi::State &st) {
  if constexpr (EpiReadsOld<Epi>::value) epi.finish_old(task, m, rd, y0, y1, old, st);
  else epi.finish(task, m, rd, y0, y1, st);
}

// The same for the other epilogues, with the stores in mind: a workgroup of 1024 threads takes 32
// tasks x 32 activation rows, one pair per thread.  It sums the k ranges with the rows fastest
// across threads (the order in which the partials lie), turns the tile in LDS, and runs the
// epilogue with the tasks fastest, so that what the epilogue writes (consecutive elements of a row
// of the hidden state, of q, of the cache, of the activations) leaves a wave as whole segments
// instead of single words 7 KB apart.  grid (cut tiles * blocks of 32 tasks in a tile, blocks of 32
// rows in a tile).
template <typename Epi, int MAXS>
__global__ void __launch_bounds__(1024)
mfma_finish_tile_k(Epi epi, const RowDesc *__restrict__ rows, int m_rows, int n_tasks, PartialSums ps) {
  __shared__ float s_y[2][32][33];
  const int per_tile = (ps.tasks_per_tile + 31) / 32;
  const int tile = blockIdx.x / per_tile, tb = blockIdx.x - tile * per_tile;   // cut tile, block of tasks in it
  int bx, bz;
  tile_place(ps.tc, ps.tc.n_whole + tile, bx, bz);
  const int task0 = bx * ps.tasks_per_tile + tb * 32, row0 = bz * ps.rows_per_tile + blockIdx.y * 32;
  if (task0 >= n_tasks || row0 >= m_rows) return;
  // what the epilogue will need besides the sums is requested first: the row's descriptor, and
  // through it the old value of a residual projection; both round trips run under the loads of
  // the partial sums
  const int tl = threadIdx.x & 31, ml = threadIdx.x >> 5, task = task0 + tl, m = row0 + ml;
  const bool live = task < n_tasks && m < m_rows;
  const RowDesc rd = rows[m < m_rows ? m : 0];
  const auto old = load_old(epi, task, m, rd, live);
  {
    const int ml_ = blockIdx.y * 32 + (threadIdx.x & 31);                     // row and task inside the tile
    const int tl_ = min(tb * 32 + (int)(threadIdx.x >> 5), ps.tasks_per_tile - 1);
    float y0 = 0.f, y1 = 0.f;
    if (ml_ < ps.m_pitch)
      sum_splits<MAXS>(ps.part + ((size_t)tile * ps.tasks_per_tile + tl_) * 2 * ps.m_pitch + ml_, ps.stride(), ps.n_split,
                       ps.m_pitch, y0, y1);
    s_y[0][threadIdx.x >> 5][threadIdx.x & 31] = y0;
    s_y[1][threadIdx.x >> 5][threadIdx.x & 31] = y1;
  }
  __syncthreads();
  typename Epi::State st;
  epi.init(st);
  if (live) finish_pair(epi, task, m, rd, s_y[0][tl][ml], s_y[1][tl][ml], old, st);
  hand_on_row<32>(epi, m, m < m_rows, st, task0 / 32);
}

// ------------------------------------------------------------------ at most 48 rows
//
// Batched decoding: the projection is a stream of weights again, only with more arithmetic per
// weight.  A workgroup of four waves takes NT A tiles (16 NT tasks) and one range of k, a quarter
// of it for each wave; the waves' sums meet in LDS at the end.  Weights and activations go from
// memory straight into registers, both in operand order, so the loop has no LDS traffic and no
// barrier: every wave runs on its own behind its own loads, RING steps ahead (memory answers in
// order: a shorter ring for the activations would empty the weights' longer one), and the
// activations are cut into fp16 parts by the wave that multiplies them.
//
// v_mfma_f32_16x16x32_f16, COLS = 16, 32 or 48 activation rows as one to three B operands: with 32-wide
// operands a pass of 16 rows would fetch and cut as many activations as one of 32.  What bounds the short
// launches is what a CU has to fetch, activations (from L2, 4 COLS bytes per k) as much as weights:
// q/k/v of 8 rows, k 3584, 33 MB: 11.0 us with the activations' loads left out, 16.2 with 32 columns, 11.9
// with 16.
// More in flight is not better: the same launch takes 12.5, 11.9, 12.3, 19 us with rings of 3, 4, 6 and 14 steps,
// and 13 to 16 with eight or sixteen waves; gate/up of 271 MB 46.7 us with four waves and one tile,
// 53 with eight and five (237 workgroups that all start, and all finish, together).
// So: few loads in flight per wave, four waves, and for at most 8 rows one tile a workgroup, several
// workgroups on a CU, whose starts and ends run under the others' streaming.  From 9 rows on fetching all
// activations in every workgroup costs more than that gains (gate/up of 16 rows 52.4 us with one tile, 49.0 with
// five): then NT makes one round of CUs, or as few as can be, of about equal size.  Either way a workgroup
// takes all of k, and there are no partial sums.
// Where that leaves CUs idle k is cut (CUT): a long one with few tasks (down) into as many ranges as fill the chip, and
// that of o in two from 9 rows on.  The last workgroup to arrive adds the ranges up; a launch that did so took 5 us (down
// of 136 MB: 8 rows 24.5 and 4.9 us in two launches, 27.6 in one; 48 rows 40.5 and 5.2, 45.6, but the next
// launch no longer waits for a small one to start and drain).
//
// (48 rows: gate/up of 271 MB 58 us, where mfma_tiled_k and its finishing launch take 58 and 12; a quarter of the heads 61
// against 87; down 37 and 5 against 40 and 8; q/k/v and o level.  With 64 the sums of five tiles spill.)
// Loads are buffer loads: the lane's place is one register for all of them, step and tile are scalars.  No load
// leaves the matrix or the activations (direct_x_step, direct_x_quad, direct_w_tile): whether a scalar offset takes part in
// the check of a buffer's end is not something to rely on.
constexpr int td_ring(int nt) { return nt == 1 ? 4 : 2; }
// Every MFMA rounds its running sums to 32 bits, and a quarter of k in one chain leaves 2.8e-7 of the heads'
// logits (k 3584, against 64 bits): the sums of a few steps are added to a second set and begin at zero again,
// and where there are registers for it the activations' lower parts have sums of their own.  1.3e-7 without
// the latter, 1.2e-7 with them (vector kernel: 1.1e-7); MLP blocks 2.6e-7 and 2.3e-7 (vector kernels 2.5e-7).
constexpr bool td_fine(int nt, int cols) { return nt * cols <= 32; }   // (what the registers of four waves a SIMD allow)
constexpr int td_fold_steps(int nt, int cols) { return td_fine(nt, cols) || nt * cols > 160 ? 2 : 4; }   // steps of 32 k whose products go into one set of sums (240: four spill)

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t buffer_of(const void *p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)(bytes < 0xfffffff0ull ? bytes : 0xfffffff0ull), 0x00027000);
}
template <bool ONCE> __device__ __forceinline__ u32x4_t load_buffer16(buffer_t b, int lane_at, int at) {   // ONCE: non-temporal
  return __builtin_amdgcn_raw_buffer_load_b128(b, lane_at, at, ONCE ? 2 : 0);
}

template <int NT, int COLS, typename Epi, bool CUT>
__global__ void __launch_bounds__(64 * TD_WAVES, 1)
mfma_direct_k(Epi epi, const f16_t *__restrict__ tiled, const float *__restrict__ wdown,
              const RowDesc *__restrict__ rows, int m_rows, ProjIn in, int n_in, int n_tasks, int n_groups,
              int chunks_per_split, float *__restrict__ part, int *__restrict__ arrivals) {
  static_assert(COLS % 16 == 0 && COLS <= OP_ROWS, "operands of 16 activation rows");
  constexpr int CG = COLS / 16, KS = 32, STEPS = MG_KC / KS, RING = td_ring(NT), THREADS = 64 * TD_WAVES;
  extern __shared__ uint4 td_smem[];
  float *s_t = (float *)td_smem;                             // [waves][NT][COLS][TD_PITCH]
  float *s_wdown = s_t + TD_WAVES * NT * COLS * TD_PITCH;    // [NT][32 operand rows]
  int *s_exp = (int *)((char *)td_smem + td_exp_at(NT, COLS));   // [THREADS / LPR], the first COLS are needed
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, kq = lane >> 4;   // operand row / column, and which eight of the step's 32 k
  clear_words(in);
  const int split = CUT ? blockIdx.x / n_groups : 0, group = blockIdx.x - split * n_groups;
  const int n_chunks = (n_in + MG_KC - 1) / MG_KC, n_blocks = (n_tasks + TG_TASKS - 1) / TG_TASKS;
  const int c_begin = CUT ? split * chunks_per_split : 0;
  const int c_end = CUT ? min(n_chunks, c_begin + chunks_per_split) : n_chunks;

  // this wave's steps [s_begin, s_end) of the range
  const int per_wave = ((c_end - c_begin) * STEPS + TD_WAVES - 1) / TD_WAVES;
  const int s_begin = min(c_begin * STEPS + wave * per_wave, c_end * STEPS), s_end = min(s_begin + per_wave, c_end * STEPS);
  const int s_last = max(s_end - 1, 0);   // steps past the end read this one and are multiplied with zeros
  const size_t tile_bytes = sizeof(f16_t) * TG_TILE, first = (size_t)group * NT * n_chunks;
  const buffer_t w_buf = buffer_of(tiled + first * TG_TILE, ((size_t)n_blocks * n_chunks - first) * tile_bytes);
  const int op_rows = -in.stride;
  const buffer_t x_buf = buffer_of(in.x, sizeof(float) * op_rows * (size_t)n_in);
  // of a tile's chunk: operand rows 16 h + col, elements 32 step + 8 kq .. + 7
  const int w_at = (int)sizeof(f16_t) * ((kq >> 1) * 512 + (col + 32 * (kq & 1)) * 8);
  u32x4_t wr[RING][NT][2], xr[RING][CG][2];
  auto load_w = [&](int u, int step) {
    const int at = min(step, s_last) * (32 * KS * (int)sizeof(f16_t));
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        wr[u][q][h] = load_buffer16<true>(w_buf, w_at + h * 256, at + direct_w_tile(q, group * NT, n_blocks) * n_chunks * (int)tile_bytes);
  };
  int x_row[CG];   // (columns past the last row repeat it)
#pragma unroll
  for (int g = 0; g < CG; ++g) x_row[g] = min(16 * g + col, m_rows - 1) * 16;
  auto load_x = [&](int u, int step) {
    const int s = direct_x_step(min(step, s_last), n_in), at = s * (KS * (int)sizeof(float)) * op_rows;
    const int quad = direct_x_quad(kq, s, n_in) * 16 * op_rows;
#pragma unroll
    for (int g = 0; g < CG; ++g)
#pragma unroll
      for (int i = 0; i < 2; ++i) xr[u][g][i] = load_buffer16<false>(x_buf, quad + x_row[g], at + i * 16 * op_rows);
  };
  // (finishing, a thread has task t of every tile and the rows m0 + 16 g)
  const int t = threadIdx.x & (TG_TASKS - 1), m0 = threadIdx.x >> 4;
  constexpr int EARLY = CG <= 2 ? CG : 0;   // descriptors requested now (registers)
  RowDesc early[EARLY > 0 ? EARLY : 1];
#pragma unroll
  for (int g = 0; g < EARLY; ++g) early[g] = rows[min(m0 + 16 * g, m_rows - 1)];
  constexpr int LPR = td_lanes_per_row(COLS);   // neighbouring lanes that find a row's largest exponent
  static_assert(THREADS % LPR == 0 && THREADS / LPR >= COLS && td_exp_at(NT, COLS) + sizeof(int) * (THREADS / LPR) <= td_lds_bytes(NT, COLS),
                "every row's exponent, also those of rows that nobody asks for, has its place in LDS");
  RowExponent<LPR> mag(in.row_max, min((int)threadIdx.x / LPR, m_rows - 1), threadIdx.x & (LPR - 1));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < RING; ++u) { load_w(u, s_begin + u); load_x(u, s_begin + u); }
  __builtin_amdgcn_sched_barrier(0);
  static_assert(NT * 32 <= THREADS, "a thread fetches one weight row's scale at most");
  const int wd_row = min((int)threadIdx.x, NT * 32 - 1);   // (needed last, and from far away)
  const float wd = wdown[(size_t)min(group * NT + wd_row / 32, n_blocks - 1) * 32 + wd_row % 32];
  __builtin_amdgcn_sched_barrier(0);
  {
    const int e = mag.get();
    if ((threadIdx.x & (LPR - 1)) == 0) s_exp[threadIdx.x / LPR] = scale_exponent(e);   // (rows past the last repeat it)
  }
  __syncthreads();
  float x_up[CG];
#pragma unroll
  for (int g = 0; g < CG; ++g) x_up[g] = scale_up(s_exp[16 * g + col]);

  const f32x4_t none = {0.f, 0.f, 0.f, 0.f};
  constexpr bool FINE = td_fine(NT, COLS);
  constexpr int FOLD = td_fold_steps(NT, COLS), TURN = RING > FOLD ? RING : FOLD;
  static_assert(TURN % RING == 0 && TURN % FOLD == 0, "whole turns of the ring, whole sets of sums");
  f32x4_t acc[NT][CG][2], folded[NT][CG][2], small[FINE ? NT : 1][CG][2];   // small: of the lower parts, if kept apart
#pragma unroll
  for (int q = 0; q < NT; ++q)
#pragma unroll
    for (int g = 0; g < CG; ++g)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        folded[q][g][h] = none;
        if constexpr (FINE) small[q][g][h] = none;
      }
  auto mm = [](const u32x4_t &w, const f16x8_t &x, const f32x4_t &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, w), x, c, 0, 0, 0);
  };
  for (int s0 = s_begin; s0 < s_end; s0 += TURN) {
#pragma unroll
    for (int i = 0; i < TURN; ++i) {
      const int step = s0 + i, u = i % RING;
#pragma unroll
      for (int g = 0; g < CG; ++g) {
        const float up = step < s_end ? x_up[g] : 0.f;
        f16x8_t hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float f = __uint_as_float(xr[u][g][e >> 2][e & 3]);
          hi[e] = (f16_t)(f * up);
          lo[e] = (f16_t)__builtin_fmaf(f, up, -(float)hi[e]);   // (up is a power of two: the product is exact)
        }
#pragma unroll
        for (int q = 0; q < NT; ++q)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if constexpr (FINE) small[q][g][h] = mm(wr[u][q][h], lo, small[q][g][h]);
            else acc[q][g][h] = mm(wr[u][q][h], lo, i % FOLD == 0 ? none : acc[q][g][h]);
          }
#pragma unroll
        for (int q = 0; q < NT; ++q)
#pragma unroll
          for (int h = 0; h < 2; ++h) acc[q][g][h] = mm(wr[u][q][h], hi, FINE && i % FOLD == 0 ? none : acc[q][g][h]);
      }
      load_w(u, step + RING);
      load_x(u, step + RING);
      if (i % FOLD == FOLD - 1) {
#pragma unroll
        for (int q = 0; q < NT; ++q)
#pragma unroll
          for (int g = 0; g < CG; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) folded[q][g][h] += acc[q][g][h];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (FINE) {
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int g = 0; g < CG; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h) folded[q][g][h] += small[q][g][h];
  }

  // the waves' sums, [activation row][weight row]: a lane has four neighbouring weight rows of one activation row
  if (threadIdx.x < NT * 32) s_wdown[threadIdx.x] = wd;
#pragma unroll
  for (int q = 0; q < NT; ++q)
#pragma unroll
    for (int g = 0; g < CG; ++g)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *(f32x4_t *)(s_t + ((wave * NT + q) * COLS + 16 * g + col) * TD_PITCH + 16 * h + 4 * kq) = folded[q][g][h];
  __syncthreads();
  // the sum of an operand row, always in the order of the waves, without its scales
  // (one factor after the other: their product may lie outside the range of an fp32 where the result does not)
  auto sum = [&](int q, int row, int m, float x_down) {
    float y = s_t[(q * COLS + m) * TD_PITCH + row];
#pragma unroll
    for (int w = 1; w < TD_WAVES; ++w) y += s_t[((w * NT + q) * COLS + m) * TD_PITCH + row];
    return y * x_down * s_wdown[q * 32 + row];
  };
  // 16 lanes finish a row's tasks of one tile after the other
  auto task_of = [&](int q) { return (group * NT + q) * TG_TASKS + t; };
  typedef decltype(load_old(epi, 0, 0, RowDesc{}, true)) Old;
  // (requested together: the stores between them would hold them back)
  auto load_olds = [&](int m, const RowDesc &rd, Old *old) {
#pragma unroll
    for (int q = 0; q < NT; ++q) old[q] = load_old(epi, m < m_rows && task_of(q) < n_tasks ? task_of(q) : 0, min(m, m_rows - 1), rd, true);
  };
  auto hand_on = [&](int m, const RowDesc &rd, const typename Epi::State &st) {
    const bool row_live = m < m_rows;
    if constexpr (EpiHasLocalReduce<Epi>::value) {
      // the heads' arg-max: one atomic per row and workgroup
      unsigned long long best = st.best;
#pragma unroll
      for (int o = TG_TASKS / 2; o > 0; o >>= 1) {
        const unsigned long long other =
            ((unsigned long long)(uint32_t)__shfl_xor((int)(best >> 32), o, 64) << 32) | (uint32_t)__shfl_xor((int)best, o, 64);
        if (other > best) best = other;
      }
      if (t == 0 && row_live) epi.end_reduced(rd, best);
    } else {
      hand_on_row<TG_TASKS>(epi, m, row_live, st, group);
    }
  };
  if constexpr (CUT) {
    // This range's sums go to memory, written through; the workgroup that arrives last adds up the ranges, in
    // their order, and runs the epilogue.
    const int n_split = gridDim.x / n_groups;
    auto place = [&](int s, int q, int m) { return part + (((size_t)(s * n_groups + group) * COLS + m) * NT + q) * 32 + t; };
    RowDesc rd[CG];
    Old old[CG][NT];
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      const int m = m0 + 16 * g;
      const float x_down = scale_down(s_exp[m]);
#pragma unroll
      for (int q = 0; q < NT; ++q)
        if (m < m_rows) {
          store_device_scope(place(split, q, m), sum(q, t, m, x_down));
          store_device_scope(place(split, q, m) + TG_TASKS, sum(q, TG_TASKS + t, m, x_down));
        }
      rd[g] = EARLY > 0 ? early[EARLY > 0 ? g : 0] : rows[min(m, m_rows - 1)];
      load_olds(m, rd[g], old[g]);
    }
    wait_memory_ops();
    __syncthreads();
    if (threadIdx.x == 0) {
      const int last = __hip_atomic_fetch_add(arrivals + group, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_split - 1;
      if (last) {
        __hip_atomic_store(arrivals + group, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      s_exp[0] = last;
    }
    __syncthreads();
    if (!s_exp[0]) return;
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      const int m = m0 + 16 * g, m_read = min(m, m_rows - 1);
      typename Epi::State st;
      epi.init(st);
      float y0[NT], y1[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) y0[q] = y1[q] = 0.f;
      for (int s0 = 0; s0 < n_split; s0 += 4) {   // four ranges' loads at a time
        float a[4][NT], b[4][NT];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < NT; ++q) {
            const float *p = place(min(s0 + i, n_split - 1), q, m_read);
            a[i][q] = p[0];
            b[i][q] = p[TG_TASKS];
          }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < NT; ++q)
            if (s0 + i < n_split) { y0[q] += a[i][q]; y1[q] += b[i][q]; }
      }
#pragma unroll
      for (int q = 0; q < NT; ++q)
        if (m < m_rows && task_of(q) < n_tasks) finish_pair(epi, task_of(q), m, rd[g], y0[q], y1[q], old[g][q], st);
      hand_on(m, rd[g], st);
    }
  } else {
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      const int m = m0 + 16 * g;
      const RowDesc rd = EARLY > 0 ? early[EARLY > 0 ? g : 0] : rows[min(m, m_rows - 1)];
      const float x_down = scale_down(s_exp[m]);
      typename Epi::State st;
      epi.init(st);
      Old old[NT];
      load_olds(m, rd, old);
#pragma unroll
      for (int q = 0; q < NT; ++q)
        if (m < m_rows && task_of(q) < n_tasks)
          finish_pair(epi, task_of(q), m, rd, sum(q, t, m, x_down), sum(q, TG_TASKS + t, m, x_down), old[q], st);
      hand_on(m, rd, st);
    }
  }
}

}  // namespace spark
