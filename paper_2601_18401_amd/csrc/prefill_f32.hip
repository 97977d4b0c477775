// Prefill span-attention in fp32 on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums).
//
// The row-stationary kernel reads every key and value row once per query row and slot through the L1: 4096 rows x 4 heads,
// D = 64, spans of 64, top-4 is 2.4 GB of reads and as many vector instructions (the vector units busy 79 % of 82 us) for
// 1.2 GFLOP.  Here the rows that attend a span share it: 46 us, of which 35 span_tiles_f32 (its MFMAs alone take 9;
// 1900 workgroups in two and a half rounds of three per compute unit, each a chain of loads, look through, products; at
// this bound of three two registers spill) and 11 window_f32.  D = 128 165 -> 79, top-8 141 -> 64, 32 heads x 1024 rows
// behind 65536 tokens in spans of 256 8400 -> 716.
//
//   span_tiles_f32       one workgroup per (kv head, span, chunk of query rows) looks through the chunk's index lists
//                        for its span (no bucketing launches: the lists are a few KB), stages the span in LDS and
//                        takes the rows found 16 at a time per wavefront; partial (o, m, l) per (row, slot)
//   window_f32           sixteen rows of a head per wavefront: their local windows on the matrix cores, and the merge with
//                        their partials.  Keys and values behind a row's query are loaded and have weight 0; where a
//                        value is not finite the rows go one by one, by vector instructions, which touch none of them
//
// S^T = K Q^T and O^T += V^T P^T, so that a lane owns a query column: with 16x16x4, lane l of a result holds column l % 16
// and rows 4 (l / 16) + r.  The contraction may run over the dimensions and the kv rows in any order: QK takes d = 16 j +
// 4 (l / 16) + x in step (j, x), PV takes kv = 16 t + 4 (l / 16) + r in step (t, r), whose P is accumulator r of tile t as
// it stands, and the rows of V^T are d = 4 (l % 16) + dt: every operand is a component of a 16-byte read.
#include <mutex>

#include "kernels.h"
#include "stream_attend.h"

namespace sl {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kListItems = 2048;  // query heads of a group x rows of a chunk at most: a row has one place (see the look through)

// Which workgroup takes what.  Rows at position p choose topk of p / A spans, so the further back a row stands the more
// rows it takes for a span to find a tile's worth: the rows go in segments over which the position grows by half (at most),
// and a segment in equal chunks, each with a workgroup for every span that is a candidate at the segment's end.  (With
// equal chunks throughout, the first spans' workgroups had ten times the average's rows and were the kernel's time.)
struct F32Segment {
  unsigned block;  // first workgroup (of a kv head)
  int row, rows;   // first row, rows per chunk
  int spans;
};
struct F32Plan {
  static constexpr int kMost = 64;  // a lane each
  F32Segment seg[kMost];
  int count;
  int64_t blocks;  // of a kv head
};

// kv rows staged at a time (spans of ceil(sqrt(L)) tokens are whole up to L = 6400 at D = 64)
template <int D>
struct F32Tiles {
  static constexpr int kRows = D == 64 ? 80 : 64, kLd = D + 4;  // padded: 16 rows fall into distinct banks
  static constexpr int kBytes = 2 * kRows * kLd * (int)sizeof(float) + kListItems * (int)sizeof(int);
};

template <int D>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void span_tiles_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const int32_t* __restrict__ idx, float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t Lq,
    int64_t q_pos0, int G, int S, int A, int topk, const F32Plan plan, float scale_log2e, int64_t qsh,
    int64_t qst, int64_t kvsh, int64_t kvst) {
  using T = F32Tiles<D>;
  constexpr int LD = T::kLd, NT = T::kRows / 16, NJ = D / 16, PPR = D / 4;
  extern __shared__ __align__(16) float s_mem[];
  float* const sK = s_mem;
  float* const sV = s_mem + T::kRows * LD;
  int* const s_list = reinterpret_cast<int*>(s_mem + 2 * T::kRows * LD);
  __shared__ int s_count;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i16 = lane & 15, g = lane >> 4;
  const unsigned at_block = blockIdx.x;
  const int kv = blockIdx.y;
  const bool mine = lane < plan.count && plan.seg[lane < F32Plan::kMost ? lane : 0].block <= at_block;
  const int sg = __builtin_popcountll(__builtin_amdgcn_ballot_w64(mine)) - 1;  // (their first workgroups ascend)
  const F32Segment seg = plan.seg[sg];
  const unsigned in_seg = at_block - seg.block, chunk = in_seg / (unsigned)seg.spans;
  const int j = (int)(in_seg - chunk * (unsigned)seg.spans);
  const int64_t ra = seg.row + (int64_t)chunk * seg.rows, stop = sg + 1 < plan.count ? plan.seg[sg + 1].row : Lq;
  const int64_t rb = ra + seg.rows < stop ? ra + seg.rows : stop;
  const int chunk_rows = seg.rows;
  const int64_t end = (int64_t)(j + 1) * A, begin = end - S > 0 ? end - S : 0;
  if (end > q_pos0 + rb - 1) return;  // candidate of no row: j < (q_pos0 + r) / A  <=>  (j + 1) A <= q_pos0 + r
  const float* const Kh = K + kv * kvsh;
  const float* const Vh = V + kv * kvsh;
  const int len = (int)(end - begin);
  const bool whole = len <= T::kRows;

  // the first kv rows are asked for before the index lists are looked through
  constexpr int NLD = T::kRows * PPR / 256;
  static_assert(T::kRows * PPR % 256 == 0, "a whole number of pieces per thread");
  uint4 kr[NLD], vr[NLD];
  auto fetch = [&](int64_t t0) {
    const int rows = end - t0 < T::kRows ? (int)(end - t0) : T::kRows;
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int row = (tid + 256 * u) / PPR, c = (tid + 256 * u) % PPR;
      kr[u] = vr[u] = make_uint4(0, 0, 0, 0);
      if (row < rows) {
        kr[u] = load16(Kh + (t0 + row) * kvst + 4 * c);
        vr[u] = load16(Vh + (t0 + row) * kvst + 4 * c);
      }
    }
  };
  auto put = [&]() {
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int row = (tid + 256 * u) / PPR, c = (tid + 256 * u) % PPR;
      *reinterpret_cast<uint4*>(&sK[row * LD + 4 * c]) = kr[u];
      *reinterpret_cast<uint4*>(&sV[row * LD + 4 * c]) = vr[u];
    }
  };
  fetch(begin);
  if (tid == 0) s_count = 0;
  __syncthreads();
  const int per_head = (int)(rb - ra) * topk;
  // A row that lists the span more than once (its own result is anyone's guess) must not cost another row its place:
  // where the places do not suffice, only the first such slot of a row takes one, and its partial goes to the others too.
  auto look_through = [&](auto first_only) {
    for (int hl = 0; hl < G; ++hl) {
      const int32_t* const list = idx + ((int64_t)(kv * G + hl) * Lq + ra) * topk;
      for (int e0 = tid; e0 < per_head; e0 += 1024) {
        int v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = e0 + 256 * u < per_head ? list[e0 + 256 * u] : -1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (v[u] != j) continue;
          const int r = (e0 + 256 * u) / topk, slot = (e0 + 256 * u) % topk;
          if (end > q_pos0 + ra + r) continue;  // not a candidate of this row
          if constexpr (decltype(first_only)::value) {
            bool again = false;
            for (int s = 0; s < slot; ++s) again |= list[r * topk + s] == j;
            if (again) continue;
          }
          const int at = atomicAdd(&s_count, 1);
          if (at < kListItems) s_list[at] = (hl * chunk_rows + r) << 5 | slot;  // (the order does not matter: a row's arithmetic is its own)
        }
      }
    }
  };
  look_through(std::false_type{});
  put();
  __syncthreads();
  const bool repeated = s_count > kListItems;
  if (repeated) {
    __syncthreads();
    if (tid == 0) s_count = 0;
    __syncthreads();
    look_through(std::true_type{});
    __syncthreads();
  }
  const int count = s_count, tiles = (count + 15) / 16;
  if (count == 0) return;

#pragma unroll 1
  for (int tile = wave; tile < (whole ? tiles : (tiles + 3) / 4 * 4); tile += 4) {  // (not whole: all wavefronts stage)
    const int at = tile * 16 + i16;
    const int item = s_list[at < count ? at : 0], slot = item & 31;
    const int hl = (item >> 5) / chunk_rows;
    const int64_t r = ra + (item >> 5) % chunk_rows;
    const int h = kv * G + hl;
    const float* const qp = Q + h * qsh + r * qst + 4 * g;
    f32x4 q[NJ];
#pragma unroll
    for (int x = 0; x < NJ; ++x) q[x] = *reinterpret_cast<const f32x4*>(qp + 16 * x);
    f32x4 o[NJ];
#pragma unroll
    for (int x = 0; x < NJ; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
#pragma unroll 1
    for (int64_t t0 = begin; t0 < end; t0 += T::kRows) {
      if (!whole && !(t0 == begin && tile < 4)) {
        __syncthreads();  // every wavefront is done with the rows staged before
        fetch(t0);
        put();
        __syncthreads();
      }
      const int rows = end - t0 < T::kRows ? (int)(end - t0) : T::kRows;
      auto attend = [&](auto count_of) {
        constexpr int N = decltype(count_of)::value;  // 16-row tiles
        // Four sums of a quarter of the dimensions each: one sum of all of them is a chain of D roundings, where the
        // row-stationary kernel adds in a tree (error against 64 bits 2.9e-7, with four sums 1.9e-7 as there).
        f32x4 s[N];
        constexpr int GT = 3;  // tiles at a time: what the registers hold
#pragma unroll
        for (int ta = 0; ta < N; ta += GT) {
          f32x4 part[4][GT];
#pragma unroll
          for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int t = 0; t < GT; ++t) part[x][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int x = 0; x < NJ; ++x) {
            f32x4 k[GT];
#pragma unroll
            for (int t = 0; t < GT; ++t)
              if (ta + t < N) k[t] = *reinterpret_cast<const f32x4*>(&sK[(16 * (ta + t) + i16) * LD + 16 * x + 4 * g]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int t = 0; t < GT; ++t)
                if (ta + t < N)
                  part[x & 3][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[t][e], q[x][e], part[x & 3][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);  // (left alone, the compiler reads the whole stage ahead and spills)
          }
#pragma unroll
          for (int t = 0; t < GT; ++t)
            if (ta + t < N) s[ta + t] = (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s[t][e] = 16 * t + 4 * g + e < rows ? s[t][e] * scale_log2e : -INFINITY;
            mx = fmaxf(mx, s[t][e]);
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        // Rows whose scores are all -inf have no weight, whatever their values hold: m stays -inf and l 0 (a score
        // that is NaN shows in l), and o starts anew behind them.
        const float m_new = fmaxf(m, mx), base = m_new > -INFINITY ? m_new : 0.f;
        if (t0 > begin) {
          const bool some = m > -INFINITY;
          const float corr = fast_exp2(m - base);
          l *= corr;
#pragma unroll
          for (int x = 0; x < NJ; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[x][e] = some ? o[x][e] * corr : 0.f;
        }
        m = m_new;
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s[t][e] = fast_exp2(s[t][e] - base);
            l += s[t][e];
          }
        // (16 kv rows at a time, for the same reason)
#pragma unroll
        for (int t = 0; t < N; t += 2) {
#pragma unroll
          for (int half = 0; half < D / 64; ++half) {
            f32x4 w[2][4];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
#pragma unroll
              for (int dt = 0; dt < 4; ++dt) w[y][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
              if (t + y >= N) continue;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(&sV[(16 * (t + y) + 4 * g + e) * LD + 64 * half + 4 * i16]);
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
                  w[y][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[dt], s[t + y][e], w[y][dt], 0, 0, 0);
              }
            }
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) o[4 * half + dt] += t + 1 < N ? w[0][dt] + w[1][dt] : w[0][dt];
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      if (rows > 64) attend(std::integral_constant<int, NT>{});
      else if (rows > 48) attend(std::integral_constant<int, 4>{});
      else if (rows > 16) attend(std::integral_constant<int, 3>{});
      else attend(std::integral_constant<int, 1>{});
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (at < count) {
      const bool some = m > -INFINITY;
      const int64_t rec = ((int64_t)h * Lq + r) * topk + slot;
      float* const po = part_o + rec * D;
#pragma unroll
      for (int half = 0; half < D / 64; ++half)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f32x4 w;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) w[dt] = some ? o[4 * half + dt][e] : 0.f;
          *reinterpret_cast<f32x4*>(po + 64 * half + 16 * g + 4 * e) = w;
        }
      if (g == 0) part_ml[rec] = make_float2(m, l);
    }
  }
  if (!repeated) return;
#pragma unroll 1
  for (int at = wave * 16 + i16; at < count; at += 64) {  // a lane copies what it has written
    const int item = s_list[at], slot = item & 31;
    const int64_t rec = ((int64_t)(kv * G + (item >> 5) / chunk_rows) * Lq + ra + (item >> 5) % chunk_rows) * topk + slot;
    for (int s = 1; s < topk - slot; ++s) {
      if (idx[rec + s] != j) continue;
#pragma unroll
      for (int x = 0; x < NJ; ++x) {
        const int at_d = 64 * (x / 4) + 16 * g + 4 * (x % 4);
        *reinterpret_cast<f32x4*>(part_o + (rec + s) * D + at_d) = *reinterpret_cast<const f32x4*>(part_o + rec * D + at_d);
      }
      if (g == 0) part_ml[rec + s] = part_ml[rec];
    }
  }
}

// Sum over the row groups of a wavefront (lanes with equal lane % LPR).
template <int LPR>
__device__ __forceinline__ float sum_groups(float x) {
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// The local window [cA, i] of every row, and the merge with its slots' partials: one joint softmax, or (COMBINED,
// Section 3.4) per slot the softmax over span and window, gated by the softmax of the search scores.

// One row, by vector instructions: what lies behind the query is never touched.  The row groups of the wavefront take
// the slots in turn.
struct WindowArgs {
  const float *Q, *K, *V;
  const int32_t* idx;
  const float *gate, *part_o;
  const float2* part_ml;
  float *O, *LSE;
  int64_t Lq, q_pos0;
  int Hq, G, A, topk;
  float scale_log2e;
  int64_t qsh, qst, kvsh, kvst;
};

template <int D, bool COMBINED>
__device__ void window_row(const WindowArgs& a, int h, int64_t r, int lane) {
  const float *const Q = a.Q, *const K = a.K, *const V = a.V, *const gate = a.gate, *const part_o = a.part_o;
  const int32_t* const idx = a.idx;
  const float2* const part_ml = a.part_ml;
  float *const O = a.O, *const LSE = a.LSE;
  const int G = a.G, A = a.A, topk = a.topk;
  const float scale_log2e = a.scale_log2e;
  const int64_t qsh = a.qsh, qst = a.qst, kvsh = a.kvsh, kvst = a.kvst;
  using RL = RowLayout<float, D>;
  constexpr int LPR = RL::LPR, RPW = RL::RPW;
  const int64_t row = (int64_t)h * a.Lq + r, i = a.q_pos0 + r;
  const int kv = h / G;
  const int64_t c = i / A;
  const int lr = lane % LPR, g = lane / LPR;
  float q2[4];
  Elem<float>::unpack(load16(Q + h * qsh + r * qst + lr * 4), q2);
#pragma unroll
  for (int e = 0; e < 4; ++e) q2[e] *= scale_log2e;

  // this group's first slots, asked for before the window
  constexpr int PRE = 2;
  const int64_t rec0 = row * topk;
  bool ok[PRE];
  float2 ml[PRE];
  uint4 po[PRE];
  auto slot_data = [&](int slot, bool& valid, float2& a, uint4& b) {
    const int64_t jj = slot < topk ? idx[rec0 + slot] : -1;
    valid = jj >= 0 && jj < c;
    a = valid ? part_ml[rec0 + slot] : make_float2(-INFINITY, 0.f);
    b = valid ? load16(part_o + (rec0 + slot) * D + lr * 4) : make_uint4(0, 0, 0, 0);
  };
#pragma unroll
  for (int u = 0; u < PRE; ++u) slot_data(g + u * RPW, ok[u], ml[u], po[u]);

  AttendState<float, D> st;
  st.init();
  attend_range<float, D, 4>(q2, K + kv * kvsh, V + kv * kvsh, kvst, c * A, i + 1, lane, st);

  if constexpr (!COMBINED) {
    auto add = [&](const float2& a, const uint4& b) {
      float f[4];
      Elem<float>::unpack(b, f);
      const float M = fmaxf(st.m, a.x);
      const float ws = st.m > -INFINITY ? fast_exp2(st.m - M) : 0.f, wp = a.x > -INFINITY ? fast_exp2(a.x - M) : 0.f;
      st.m = M;
      st.l = st.l * ws + a.y * wp;
#pragma unroll
      for (int e = 0; e < 4; ++e) st.o[e] = st.o[e] * ws + f[e] * wp;
    };
#pragma unroll
    for (int u = 0; u < PRE; ++u)
      if (ok[u]) add(ml[u], po[u]);
    for (int slot = g + PRE * RPW; slot < topk; slot += RPW) {
      bool v;
      float2 a;
      uint4 b;
      slot_data(slot, v, a, b);
      if (v) add(a, b);
    }
  }
  merge_row_groups<float, D>(st);
  float out[4];
  if constexpr (!COMBINED) {
    const float inv = 1.f / st.l;  // the local window always holds the query's own token: l > 0
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = st.o[e] * inv;
    if (lane == 0) LSE[row] = (st.m + __log2f(st.l)) * kLn2;
  } else {
    float smax = -INFINITY;
    for (int slot = 0; slot < topk; ++slot) {
      const int64_t jj = idx[rec0 + slot];
      if (jj >= 0 && jj < c) smax = fmaxf(smax, gate[rec0 + slot]);
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f}, asum = 0.f;
    auto add = [&](const float2& s, const uint4& b, int slot) {
      float f[4];
      Elem<float>::unpack(b, f);
      const float M = fmaxf(s.x, st.m);
      const float wa = fast_exp2(s.x - M), wb = fast_exp2(st.m - M);
      const float a = __expf(gate[rec0 + slot] - smax);
      const float w = a / (s.y * wa + st.l * wb);
      asum += a;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(w, f[e] * wa + st.o[e] * wb, acc[e]);
    };
#pragma unroll
    for (int u = 0; u < PRE; ++u)
      if (ok[u]) add(ml[u], po[u], g + u * RPW);
    for (int slot = g + PRE * RPW; slot < topk; slot += RPW) {
      bool v;
      float2 a;
      uint4 b;
      slot_data(slot, v, a, b);
      if (v) add(a, b, slot);
    }
    asum = sum_groups<LPR>(asum);
    const bool any = asum > 0.f;
    const float inv = any ? 1.f / asum : 1.f / st.l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = sum_groups<LPR>(acc[e]);
      out[e] = (any ? x : st.o[e]) * inv;
    }
  }
  if (g == 0) *reinterpret_cast<float4*>(O + row * D + lr * 4) = make_float4(out[0], out[1], out[2], out[3]);
}


// Sixteen rows of a head per wavefront, operands straight from memory (each is used once).  A value behind a row's query
// has weight 0 there, and 0 times what is not finite is not 0: where one of the values is not finite, the rows go one by
// one.  One wavefront per row took 27 us where this takes 11 (16384 rows, D = 64, windows of up to 64).
template <int D, bool COMBINED>
__global__ __launch_bounds__(256, 2) void window_f32_kernel(const WindowArgs a) {
  constexpr int NJ = D / 16, N = D == 64 ? 4 : 2, ROWS = 16 * N;
  const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
  const int64_t tiles = (a.Lq + 15) / 16, tile = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (tile >= a.Hq * tiles) return;
  const int h = (int)(tile / tiles), kv = h / a.G;
  const int64_t r0 = tile % tiles * 16, rl = r0 + 15 < a.Lq ? r0 + 15 : a.Lq - 1, r = r0 + i16 < rl ? r0 + i16 : rl;
  const bool real = r0 + i16 < a.Lq;
  const int64_t i = a.q_pos0 + r, c = i / a.A, begin = (a.q_pos0 + r0) / a.A * a.A, last = a.q_pos0 + rl;
  const float* const Kh = a.K + kv * a.kvsh;
  const float* const Vh = a.V + kv * a.kvsh;
  const int64_t rec0 = ((int64_t)h * a.Lq + r) * a.topk;
  f32x4 q[NJ], o[NJ];
#pragma unroll
  for (int x = 0; x < NJ; ++x) {
    q[x] = *reinterpret_cast<const f32x4*>(a.Q + h * a.qsh + r * a.qst + 16 * x + 4 * g);
    o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY, l = 0.f;
  const int lo = (int)(c * a.A - begin), hi = (int)(i - begin);  // the row's own keys, counted from the first
  unsigned largest = 0u;
#pragma unroll 1
  for (int t0 = 0; t0 <= (int)(last - begin); t0 += ROWS) {
    const int most = (int)(last - begin);
    f32x4 v[N][4][D / 64];
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = min(t0 + 16 * t + 4 * g + e, most);
#pragma unroll
        for (int half = 0; half < D / 64; ++half)
          v[t][e][half] = *reinterpret_cast<const f32x4*>(Vh + (begin + row) * a.kvst + 64 * half + 4 * i16);
      }
    f32x4 part[4][N];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int t = 0; t < N; ++t) part[x][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < NJ; ++x) {
      f32x4 k[N];
#pragma unroll
      for (int t = 0; t < N; ++t)
        k[t] = *reinterpret_cast<const f32x4*>(Kh + (begin + min(t0 + 16 * t + i16, most)) * a.kvst + 16 * x + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < N; ++t)
          part[x & 3][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[t][e], q[x][e], part[x & 3][t], 0, 0, 0);
    }
    f32x4 s[N];
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < N; ++t) {
      s[t] = (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int at = t0 + 16 * t + 4 * g + e;
        s[t][e] = at >= lo && at <= hi ? s[t][e] * a.scale_log2e : -INFINITY;
        mx = fmaxf(mx, s[t][e]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx), base = m_new > -INFINITY ? m_new : 0.f;  // (no key of the row's so far)
    const float corr = fast_exp2(m - base);
    l *= corr;
#pragma unroll
    for (int x = 0; x < NJ; ++x) o[x] *= corr;
    m = m_new;
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[t][e] = fast_exp2(s[t][e] - base);
        l += s[t][e];
      }
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
      for (int half = 0; half < D / 64; ++half) {
        f32x4 w[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) w[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) {
            largest = max(largest, __float_as_uint(v[t][e][half][dt]) & 0x7fffffffu);
            w[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[t][e][half][dt], s[t][e], w[dt], 0, 0, 0);
          }
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[4 * half + dt] += w[dt];
      }
  }
  if (__builtin_amdgcn_ballot_w64(largest >= 0x7f800000u) != 0ull) {
    for (int64_t x = r0; x <= rl; ++x) window_row<D, COMBINED>(a, h, x, lane);
    return;
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);

  // the row's partials: lane (row, g) holds dimensions 64 half + 16 g + 4 e + dt in o[4 half + dt][e]
  float smax = -INFINITY, asum = 0.f;
  f32x4 acc[NJ];
  if constexpr (COMBINED) {
    for (int slot = 0; slot < a.topk; ++slot) {
      const int64_t jj = a.idx[rec0 + slot];
      if (jj >= 0 && jj < c) smax = fmaxf(smax, a.gate[rec0 + slot]);
    }
#pragma unroll
    for (int x = 0; x < NJ; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  constexpr int B = D == 64 ? 4 : 2;  // slots at a time
  for (int s0 = 0; s0 < a.topk; s0 += B) {
    bool ok[B];
    float2 ml[B];
    float gt[B];
    f32x4 p[B][D / 64][4];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int64_t jj = s0 + u < a.topk ? a.idx[rec0 + s0 + u] : -1;
      ok[u] = jj >= 0 && jj < c;
      const int64_t rec = ok[u] ? rec0 + s0 + u : 0;
      ml[u] = ok[u] ? a.part_ml[rec] : make_float2(-INFINITY, 0.f);
      gt[u] = COMBINED && ok[u] ? a.gate[rec] : 0.f;
#pragma unroll
      for (int half = 0; half < D / 64; ++half)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[u][half][e] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (ok[u]) p[u][half][e] = *reinterpret_cast<const f32x4*>(a.part_o + rec * D + 64 * half + 16 * g + 4 * e);
        }
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (!ok[u]) continue;
      const float M = fmaxf(m, ml[u].x), at = COMBINED || M > -INFINITY ? M : 0.f;  // (joint: a list may begin with -inf alone)
      const float ww = fast_exp2(m - at), wp = fast_exp2(ml[u].x - at);
      if constexpr (!COMBINED) {
        m = M;
        l = l * ww + ml[u].y * wp;
#pragma unroll
        for (int half = 0; half < D / 64; ++half)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
              o[4 * half + dt][e] = o[4 * half + dt][e] * ww + p[u][half][e][dt] * wp;
      } else {
        const float w = __expf(gt[u] - smax), f = w / (ml[u].y * wp + l * ww);
        asum += w;
#pragma unroll
        for (int half = 0; half < D / 64; ++half)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
              acc[4 * half + dt][e] = fmaf(f, p[u][half][e][dt] * wp + o[4 * half + dt][e] * ww, acc[4 * half + dt][e]);
      }
    }
  }
  if (!real) return;
  const int64_t row = (int64_t)h * a.Lq + r;
  const bool any = COMBINED && asum > 0.f;
  const float inv = any ? 1.f / asum : 1.f / l;
#pragma unroll
  for (int half = 0; half < D / 64; ++half)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f32x4 w;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        if constexpr (COMBINED) w[dt] = (any ? acc[4 * half + dt][e] : o[4 * half + dt][e]) * inv;
        else w[dt] = o[4 * half + dt][e] * inv;
      }
      *reinterpret_cast<f32x4*>(a.O + row * D + 64 * half + 16 * g + 4 * e) = w;
    }
  if (!COMBINED && g == 0) a.LSE[row] = (m + __log2f(l)) * kLn2;
}

// A span finds about 64 rows in a chunk, a tile for each wavefront; more where there are workgroups enough, since each
// stages the span.
F32Plan f32_plan(const Problem& pb) {
  F32Plan plan;
  const int64_t most = kListItems / pb.G;  // a place for every row
  for (int64_t target = 64;; target *= 2) {
    plan.count = 0;
    plan.blocks = 0;
    for (int64_t r = 0; r < pb.Lq;) {
      const int64_t p = pb.q_pos0 + r, c = p / pb.A;
      // rows with no more spans than they take, and those before the first span's end, are one segment each
      int64_t stop = c < 1 ? pb.A : c < pb.topk ? (int64_t)pb.topk * pb.A : p + (p + 1) / 2;
      stop = (plan.count == F32Plan::kMost - 1 || stop > pb.q_pos0 + pb.Lq) ? pb.Lq : stop - pb.q_pos0;
      const int64_t end_c = (pb.q_pos0 + stop - 1) / pb.A;
      if (end_c > 0) {
        int64_t rows = target * (c > pb.topk ? c : pb.topk) / ((int64_t)pb.topk * pb.G);
        rows = rows < 1 ? 1 : rows > most ? most : rows;
        const int64_t chunks = (stop - r + rows - 1) / rows;
        rows = (stop - r + chunks - 1) / chunks;  // all alike
        plan.seg[plan.count++] = {(unsigned)plan.blocks, (int)r, (int)rows, (int)end_c};
        plan.blocks += chunks * end_c;
      }
      r = stop;
    }
    if (plan.blocks * pb.Hkv <= 16384 || target >= 512) return plan;
  }
}

size_t f32_bytes(const Problem& pb) {
  return align_up((size_t)pb.Hq * pb.Lq * pb.topk * sizeof(float2), 256) + (size_t)pb.Hq * pb.Lq * pb.topk * pb.D * sizeof(float);
}

constexpr size_t kF32MaxScratch = (size_t)4 << 30;

Problem f32_part(const Problem& pb, int kv_heads) {
  Problem q = pb;
  q.Hkv = kv_heads;
  q.Hq = kv_heads * pb.G;
  return q;
}

int f32_heads(const Problem& pb) {  // kv heads per pass: as many as fit the scratch limit
  int h = pb.Hkv;
  while (h > 1 && f32_bytes(f32_part(pb, h)) > kF32MaxScratch) --h;
  return h;
}

// The kernel's LDS at D = 128 is more than the 64 KB that it gets without asking.
bool f32_setup() {
  static std::mutex mu;
  static bool done[64];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  std::lock_guard<std::mutex> lock(mu);
  if (!done[dev])
    done[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(span_tiles_f32_kernel<128>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, F32Tiles<128>::kBytes) == hipSuccess;
  return done[dev];
}

template <int D>
sl_status f32_pass(const Problem& pb, const float* Q, const float* K, const float* V, const int32_t* idx, float* O,
                   float* LSE, char* ws, hipStream_t st) {
  using T = F32Tiles<D>;
  float2* const part_ml = reinterpret_cast<float2*>(ws);
  float* const part_o = reinterpret_cast<float*>(ws + align_up((size_t)pb.Hq * pb.Lq * pb.topk * sizeof(float2), 256));
  const F32Plan plan = f32_plan(pb);
  const dim3 grid((unsigned)plan.blocks, (unsigned)pb.Hkv);
  if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
  if (plan.blocks > 0)
    hipLaunchKernelGGL((span_tiles_f32_kernel<D>), grid, dim3(256), T::kBytes, st, Q, K, V, idx, part_o, part_ml, pb.Lq,
                     pb.q_pos0, pb.G, pb.S, pb.A, pb.topk, plan, pb.scale * kLog2e, pb.qsh, pb.qst, pb.kvsh,
                     pb.kvst);
  if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  const WindowArgs w = {Q, K, V, idx, pb.gate, part_o, part_ml, O, LSE, pb.Lq, pb.q_pos0, pb.Hq, pb.G, pb.A, pb.topk,
                        pb.scale * kLog2e, pb.qsh, pb.qst, pb.kvsh, pb.kvst};
  const dim3 wgrid((unsigned)((pb.Hq * ((pb.Lq + 15) / 16) + 3) / 4));
  if (pb.combined) hipLaunchKernelGGL((window_f32_kernel<D, true>), wgrid, dim3(256), 0, st, w);
  else hipLaunchKernelGGL((window_f32_kernel<D, false>), wgrid, dim3(256), 0, st, w);
  return hipGetLastError() == hipSuccess ? SL_OK : SL_ERR_LAUNCH;
}

// Estimated us of the two forms; the call takes this one where it is the faster.  Fitted to 6500 shapes of 1 to 128 heads, 1
// to 100000 rows, spans of 1 to 2048 tokens, top-1 to top-32, both forms measured: each sum is within a fifth of the time
// for eight shapes in ten.  A call of few rows is one chain of latencies, and there the estimates err most, so it needs a
// lead.  Of the 6500, this form runs 2807, 94 of them more than 2 % and 50 more than 10 % slower than by rows; all 6500
// take 1.0 % longer than the faster form each, by rows throughout 45 %.  (The size of the scratch is asked for without
// saying which softmax it is for, so the rule does not look at that: the gated rows take 0.4 us a slot more.)
// What counts, us, rows -> this form (heads, D, rows of a prompt of L, spans, top-k):
//   the lists: a workgroup looks through those of its whole chunk, for every span of it: 64:4, 128, 5986 of 19015, spans of
//     4, top-24 3530 -> 32300; 64:4, 128, 1372, spans of 1, top-32 673 -> 3080; 8:1, 128, 300 of 1241, spans of 6 21 -> 64;
//   the window: one wavefront takes 16 rows' keys, 64 (D = 128: 32) at a time, one behind the other: 2:1, 64, 27 of 1223,
//     spans of 896, top-1 38 -> 76; 16:1, 128, 16 of 2111, spans of 1432, top-12 131 -> 234 (a span of several stages, too);
//   a wavefront of the other form has all slots' keys behind one another, and past the L2 every row reads its own from
//     memory: 8:4, 128, 1 of 25613, spans of 982, top-12 1250 -> 129; 64:8, 128, 1000 of 59212, 64, top-12 6590 -> 1350;
//   4:4, 64, 4096, 64, top-4 82 -> 46, top-8 141 -> 62, D = 128 165 -> 79; 32:4, 128, 1024 of 65536, 256, top-8 8400 -> 716.
bool f32_is_faster(const Problem& pb, const F32Plan& plan) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t q0 = pb.q_pos0, first = q0 / pb.A, last = (q0 + pb.Lq - 1) / pb.A;
  const double rows = (double)pb.Hq * pb.Lq, d = pb.D / 64, k = pb.topk, key = pb.D / 4096.0;
  // slots in use: the most, and a row's mean (the candidates grow evenly until there are topk)
  const double most = last < k ? last : k;
  double slots = k;
  if (last <= k) slots = 0.5 * (first + last);
  else if (first < k) slots = k - (k * pb.A - q0) / (double)pb.Lq * (k - 0.5 * (first + k));
  // window lengths: the longest, and their mean
  const int64_t at = q0 % pb.A, head = pb.Lq < pb.A - at ? pb.Lq : pb.A - at, rest = pb.Lq - head;
  const int64_t longest = rest >= pb.A ? pb.A : at + head > rest ? at + head : rest, part = rest % pb.A;
  const double window = (head * (at + 0.5 * (head + 1)) + 0.5 * (rest - part) * (pb.A + 1) + 0.5 * part * (part + 1)) / pb.Lq;

  const int64_t at_once = 1024 / pb.D;  // keys that a wavefront of the row-stationary kernel takes at a time
  const double keys = slots * pb.S + window, group = (double)pb.G * pb.Lq;  // keys of a row, rows of a kv head
  // reads that miss the 4 MB of an XCD's L2: keys read for the first time there, and what the kv heads in flight do not leave
  const double visible = (double)(q0 + pb.Lq), in_flight = 8192 / group, heads = in_flight < 1 ? 1 : in_flight > pb.Hkv ? pb.Hkv : in_flight;
  const double fresh = 8 * visible / (group * keys), evicted = 1 - (4 << 20) / (heads * visible * pb.D * 8);
  const double miss = fresh > 1 || evicted > 1 ? 1 : fresh > evicted ? fresh : evicted;
  const double chain_rows = most * up(pb.S, at_once) + up(longest, at_once);
  const double by_rows = 3.5 + (0.387 + 0.159 * miss) * chain_rows + 0.2 * most +
                         rows * (2.31e-4 * (slots * up(pb.S, at_once) + window / at_once + 0.5) + 0.95e-4 * slots +
                                 1.77e-3 * slots * pb.S * key * miss);

  const int64_t stage = pb.D == 64 ? F32Tiles<64>::kRows : F32Tiles<128>::kRows, over = pb.S % stage, wkeys = pb.D == 64 ? 64 : 32;
  const double computed = pb.S - over + (over == 0 ? 0 : over <= 16 ? 16 : over <= 48 ? 48 : over <= 64 ? 64 : 80);
  double scan = 0, chain = 0, scans = 0, tiles = 0;
  for (int x = 0; x < plan.count; ++x) {
    const F32Segment& g = plan.seg[x];
    const double blocks = (x + 1 < plan.count ? plan.seg[x + 1].block : (double)plan.blocks) - g.block;
    const double looks = (double)pb.G * up((int64_t)g.rows * pb.topk, 1024);
    const double c = (double)((q0 + g.row) / pb.A), of = c < 1 ? 1 : c;
    const double items = (double)pb.G * g.rows * (of < k ? 1 : k / of);
    const double many = up(pb.S, stage) * up(up((int64_t)(items + 2 * std::sqrt(items)) + 1, 16), 4);
    scan = looks > scan ? looks : scan;
    chain = many > chain ? many : chain;
    scans += blocks * looks;
    tiles += blocks * (items / 16 + 0.5);
  }
  const double waves = (double)pb.Hq * up(pb.Lq, 16);
  const double by_tiles = 5.3 + 5.18 * up(longest, wkeys) + 2.61 * up((int64_t)most, pb.D == 64 ? 4 : 2) + 0.273 * scan + 1.68 * d * chain +
                          waves * d * (7.9e-4 * d * ((window + 8) / wkeys + 0.5) + 2.54e-3 * slots) +
                          pb.Hkv * (6.6e-4 * scans + 7e-3 * plan.blocks * pb.S * key + 7.3e-4 * tiles * computed * key);
  return (rows < 4096 ? 1.1 * by_tiles + 1 : by_tiles) < by_rows;
}

}  // namespace

bool prefill_attention_f32_supported(const Problem& pb) {
  if (pb.dtype != SL_F32 || pb.topk < 1 || pb.G > kListItems || pb.Hkv >= 65536 || pb.S >= (1 << 30) ||
      pb.n >= ((int64_t)1 << 31) || pb.Lq >= ((int64_t)1 << 31) || f32_bytes(f32_part(pb, 1)) > kF32MaxScratch)
    return false;
  const F32Plan plan = f32_plan(pb);
  return plan.blocks < ((int64_t)1 << 31) && f32_is_faster(pb, plan);
}

size_t prefill_attention_f32_ws_bytes(const Problem& pb) { return f32_bytes(f32_part(pb, f32_heads(pb))); }

// Spans of a row that overlap in one joint softmax (A < S) are clipped per row: the row-stationary kernels.
sl_status prefill_attention_f32(const Problem& pb, const void* Q, const void* K, const void* V, const int32_t* idx,
                                void* O, float* LSE, void* ws, hipStream_t st) {
  if (pb.A < pb.S && !pb.combined) return prefill_attention_rows(pb, Q, K, V, idx, O, LSE, st);
  if (pb.D == 128 && !f32_setup()) return SL_ERR_LAUNCH;
  const int step = f32_heads(pb);
  for (int kv = 0; kv < pb.Hkv; kv += step) {
    Problem q = f32_part(pb, pb.Hkv - kv < step ? pb.Hkv - kv : step);
    if (kv > 0) q.prof_start = nullptr;
    if (kv + step < pb.Hkv) q.prof_stop = nullptr;
    const int64_t h = (int64_t)kv * pb.G, row = h * pb.Lq;
    if (pb.gate) q.gate = pb.gate + row * pb.topk;
    const float* const qp = static_cast<const float*>(Q) + h * pb.qsh;
    const float* const kp = static_cast<const float*>(K) + kv * pb.kvsh;
    const float* const vp = static_cast<const float*>(V) + kv * pb.kvsh;
    float* const op = static_cast<float*>(O) + row * pb.D;
    float* const lp = LSE ? LSE + row : nullptr;
    const sl_status s = pb.D == 64 ? f32_pass<64>(q, qp, kp, vp, idx + row * pb.topk, op, lp, static_cast<char*>(ws), st)
                                   : f32_pass<128>(q, qp, kp, vp, idx + row * pb.topk, op, lp, static_cast<char*>(ws), st);
    if (s != SL_OK) return s;
  }
  return SL_OK;
}

}  // namespace sl
