// Prefill span-search on the matrix cores (bf16, D = 128).
//
// Scores (eq. (2)) are computed transposed, S^T[span][query] = Ks[span][:] . Qs[query][:], so
// that after v_mfma_f32_32x32x16_bf16 a lane owns one query column: lane l holds query l%32 and
// the 16 spans 8*(r/4) + 4*(l/32) + r%4 of a 32-span tile.  Each lane keeps the running top-k
// (eq. (3)) of the spans it sees: scores with their span's number in the low bits, in one walk over the candidates,
// or, where the scores are returned too or the spans are many, their values alone, which give a threshold that a
// second walk applies (see the kernel).  Scores never leave the chip.
//
// Ties: among the spans whose score equals the threshold, the lower indices are kept.
#include "kernels.h"

namespace sl {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int HD = 128;
constexpr int TMQ = 128;        // query rows per workgroup (4 wavefronts x 32 columns)
// Span keys per staged chunk and their bytes: DIRECT, two buffers of 32 keys filled by direct global -> LDS loads;
// otherwise one of 64, through registers (LDS rows padded by 16 bytes: conflict-free 16-byte reads).
template <bool DIRECT>
struct Stages {
  static constexpr int kKeys = DIRECT ? 32 : 64, kStride = DIRECT ? HD : HD + 8;
  static constexpr int kBytes = (DIRECT ? 2 : 1) * kKeys * kStride * (int)sizeof(bf16_t);
};
constexpr int kEmpty = 0x7fffffff;

// Running top-K VALUES of the candidates a lane has seen, sorted descending.  Inserting x is one
// median-of-three per slot: new v[e] = med3(x, v[e-1], v[e]) (x above v[e-1]: v[e-1] moves down;
// x between: x lands here; x below v[e]: unchanged), and v[0] = max(x, v[0]).
template <int KMAX>
struct TopVals {
  float v[KMAX];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int e = 0; e < KMAX; ++e) v[e] = -INFINITY;
  }
  __device__ __forceinline__ void push(float x) {
#pragma unroll
    for (int e = KMAX - 1; e >= 1; --e) v[e] = __builtin_amdgcn_fmed3f(x, v[e - 1], v[e]);
    v[0] = fmaxf(x, v[0]);
  }
};

// Ascending order of N whole numbers (N a power of two): Batcher's odd-even merge exchange.
template <int N, int P = 1, int K = 1>
__device__ __forceinline__ void sort_ascending(int (&x)[N]) {
#pragma unroll
  for (int a = K % P; a + K < N; ++a)
    if ((a - K % P) % (2 * K) < K && a / (2 * P) == (a + K) / (2 * P)) {
      const int lo = min(x[a], x[a + K]), hi = max(x[a], x[a + K]);
      x[a] = lo;
      x[a + K] = hi;
    }
  if constexpr (K > 1) sort_ascending<N, P, K / 2>(x);
  else if constexpr (2 * P < N) sort_ascending<N, 2 * P, 2 * P>(x);
}

// The value that lane l ^ 32 holds (both, in an order that depends on the half: the one that is not this lane's own).
__device__ __forceinline__ float of_other_half(float x) {
  const int own = __float_as_int(x);
  auto a = __builtin_amdgcn_permlane32_swap(own, own, false, false);
  return __int_as_float(a[0] == own ? a[1] : a[0]);
}

// The candidate spans of 128 query rows (4 wavefronts x 32 columns), scored by the matrix cores and selected in one
// of two ways.  Both are bound by their vector instructions, not by loads or MFMAs: for 65536 rows x 256 spans, top-8,
// the vector units were busy 78 % of the time, the matrix pipes 19 %, so instructions are what counts.
//
// One walk (no scores wanted, up to `packed` candidates): a lane keeps its KMAX + 1 best scores with the span's
// number in place of their lowest bits, a median instruction per list entry and score; the two lanes of a column merge
// their lists.  Cutting a score towards zero keeps the order of scores that differ after it, so where the k'-th and
// the next one do, the first k' entries are the selection, and no index had to be carried beside the scores.  Where
// they agree in the bits that are left (one column in a thousand at 256 spans), and no third one does, those entries'
// scores are computed again, by the same MFMAs on their own keys, and the lowest is dropped.  For longer runs the
// workgroup walks a second time and keeps, of the scores that agree with the k'-th one, the bits that the number took and
// the number, as one whole number each: equal scores everywhere take two walks, as in the other way.  Scores come into a
// finite range first; a column whose k'-th score lies outside it goes the other way, and its workgroup with it.
//
// Two walks:
//   pass 1  keeps, per lane, only the VALUES of the top-k scores it has seen (a lane sees half of
//           its column's spans); the two lanes of a column are merged at the end, which gives the
//           column's threshold T = k'-th largest score, k' = min(topk, c), and the number of
//           scores above it;
//   pass 2  recomputes the scores and appends every span with score > T, and up to
//           need = k' - #(> T) spans per lane with score == T (its lowest-index ones), to the column's list in LDS;
//   finish  one lane per column keeps the spans above T plus the `need` lowest-index spans at T
//           (ties go to the lower index), and writes them in ascending span order.
// WS: the scores of the selected spans are written too (their list costs LDS, which limits the
// resident workgroups; most callers only want the indices).
// DIRECT: stages of 32 span keys by direct global -> LDS loads into two buffers, one barrier each: while one is
// scored the next is on its way.  Otherwise 64 keys through registers with two barriers.  The launch says which is
// taken where.  Slower than both: stages of 64 in two buffers and three buffers of 32.  Lists of at most 4 spans have
// their own KMAX: half of the median instructions.
//
// Two walks -> one, us, 32 heads: 65536 rows x 256 spans top-4 264 -> 166, top-8 315 -> 200, top-16 549 -> 302, top-32
// 1320 -> 607; 16384 rows x 1024 spans, top-8 380 -> 238, x 2048 694 -> 507, x 4096 (where the second look at
// agreeing scores is needed in most wavefronts) 1326 -> 1020; 500 rows x 256 23.4 -> 10.8; 3000 x 46 14.1 -> 8.8.  Where
// all scores are equal one walk becomes two: 20000 x 156, top-4 68 -> 83, top-8 99 -> 103, top-32 740 -> 332.

template <int KMAX, bool WS, bool DIRECT>
__global__ __launch_bounds__(256, (KMAX <= 4 || (KMAX == 8 && !WS)) ? 4 : KMAX == 32 && !WS ? 2 : 1) void prefill_search_mfma_kernel(
    const bf16_t* __restrict__ Qs, const bf16_t* __restrict__ K, const bf16_t* __restrict__ Ks,
    int32_t* __restrict__ idx, float* __restrict__ scores, int64_t Lq, int64_t q_pos0, int G, int S,
    int topk, int64_t n, int packed, int64_t qsh, int64_t qst, int64_t kvsh, int64_t kvst) {
  constexpr int CAP = 3 * KMAX;  // list entries per column: < KMAX above T, <= KMAX at T from each lane
  using St = Stages<DIRECT>;
  constexpr int TNS = St::kKeys;
  // Dynamic: for a static array that direct loads are filling the compiler waits for all of
  // them in front of the next read of it, other stage or not.
  extern __shared__ __align__(16) char s_stage[];
  bf16_t* const s_k = reinterpret_cast<bf16_t*>(s_stage);
  __shared__ int s_way;
  __shared__ int s_cnt[TMQ];
  __shared__ int s_j[TMQ][CAP + 1];  // odd row stride: the lanes of a wavefront read their own rows
  __shared__ float s_x[WS ? TMQ : 1][CAP + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int qc = lane & 31, hf = lane >> 5;
  const int col = wave * 32 + qc;
  const int tiles_per_head = (int)((Lq + TMQ - 1) / TMQ);
  const int h = blockIdx.x / tiles_per_head;
  const int64_t r0 = (int64_t)(blockIdx.x % tiles_per_head) * TMQ;
  const int kv = h / G;
  const int64_t r = r0 + col;
  const int64_t rc = r < Lq ? r : Lq - 1;
  auto spans_below = [&](int64_t i) {  // (a 64-bit division by a variable takes four times the instructions)
    return i < ((int64_t)1 << 31) ? (int)((uint32_t)i / (uint32_t)S) : (int)(i / S);
  };
  const int c_q = spans_below(q_pos0 + rc);  // candidates of this lane's query: spans [0, c_q)
  const int64_t r_last = (r0 + TMQ - 1 < Lq ? r0 + TMQ - 1 : Lq - 1);
  const int c_max = __builtin_amdgcn_readfirstlane(spans_below(q_pos0 + r_last));
  const int c_lo = __builtin_amdgcn_readfirstlane(c_q);  // rows ascend with the lane: lane 0 has the lowest c

  bf16x8 qf[8];
  {
    const bf16_t* qp = Qs + h * qsh + rc * qst;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16 + hf * 8);
  }
  const bf16_t* const key0 = Ks ? Ks + (int64_t)kv * n * HD : K + kv * kvsh + (S - 1) * kvst;
  const int64_t key_step = Ks ? HD : S * kvst;
  auto key = [&](int j) { return key0 + j * key_step; };

  // Walks the candidate spans in tiles of 32 and hands the lane's 16 scores of a tile to f(scores, first span of the
  // tile, whether the tile reaches beyond the lowest c of the wavefront): score e is that of span 8 (e / 4) + 4 hf + e % 4 of it.
  auto walk = [&](auto f) {
    // 16 lanes x 16 bytes per key; DIRECT: 1 KB per load, pieces swizzled for the operand reads.  The lane's keys move
    // on by one addition per stage; only the last stage looks for keys past the last candidate (that one again).
    constexpr int NLD = DIRECT ? TNS / 16 : 4;
    const bf16_t* src[NLD];
    auto row_of = [&](int i) { return DIRECT ? (uwave * NLD + i) * 4 + (lane >> 4) : (tid >> 4) + 16 * i; };
    auto piece_of = [&](int i) { return (DIRECT ? (lane & 15) ^ (row_of(i) & 15) : tid & 15) * 8; };
#pragma unroll
    for (int i = 0; i < NLD; ++i) src[i] = key(row_of(i)) + piece_of(i);
    auto next_stage = [&](int j0) {
      if (j0 + TNS > c_max) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) src[i] = key(min(j0 + row_of(i), c_max - 1)) + piece_of(i);
      }
    };
    auto advance = [&]() {
#pragma unroll
      for (int i = 0; i < NLD; ++i) src[i] += TNS * key_step;
    };
    auto stage = [&](int j0, int buf) {
      next_stage(j0);
#pragma unroll
      for (int i = 0; i < NLD; ++i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src[i],
                                         (__attribute__((address_space(3))) void*)(s_k + buf * TNS * HD + (uwave * NLD + i) * 512), 16, 0, 0);
      advance();
    };
    uint4 pre[DIRECT ? 1 : 4];
    auto fetch = [&](int j0) {
      next_stage(j0);
#pragma unroll
      for (int i = 0; i < (DIRECT ? 0 : 4); ++i) pre[i] = load16(src[i]);
      advance();
    };
    if (c_max > 0) {
      if constexpr (DIRECT) stage(0, 0);
      else fetch(0);
    }
    int buf = 0;
    for (int j0 = 0; j0 < c_max; j0 += TNS) {
      if constexpr (DIRECT) {
        // every wavefront is done with the other buffer, and this one's loads have arrived
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        if (j0 + TNS < c_max) stage(j0 + TNS, buf ^ 1);
      } else {
        if (j0 > 0) __syncthreads();  // every wavefront is done with the stage
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<uint4*>(&s_k[((tid >> 4) + 16 * i) * St::kStride + (tid & 15) * 8]) = pre[i];
        __syncthreads();
        if (j0 + TNS < c_max) fetch(j0 + TNS);
      }
      const bf16_t* const cur = s_k + (DIRECT ? buf * TNS * HD : 0);
#pragma unroll
      for (int sub = 0; sub < TNS / 32; ++sub) {
        if (j0 + 32 * sub < c_max) {  // uniform over the workgroup
          f32x16 s;
#pragma unroll
          for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
          for (int kk = 0; kk < 8; ++kk) {
            const bf16x8 ka =
                *reinterpret_cast<const bf16x8*>(
                    &cur[(32 * sub + qc) * St::kStride + (((2 * kk + hf) ^ (DIRECT ? qc & 15 : 0)) << 3)]);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[kk], s, 0, 0, 0);
          }
          f(s, j0 + 32 * sub, j0 + 32 * sub + 32 > c_lo);
        }
      }
      buf ^= 1;
    }
    __syncthreads();  // the next walk (or the lists' readers) may touch what this one used
  };
  // The two-walk form's view: f(score, span index); scores of spans >= c_q (causal: only complete spans below the
  // query's own) come as -inf.
  auto for_each_candidate = [&](auto f) {
    walk([&](const f32x16& s, int j0, bool edge) {
      if (!edge) {
#pragma unroll
        for (int e = 0; e < 16; ++e) f(s[e], j0 + 8 * (e >> 2) + 4 * hf + (e & 3));
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = j0 + 8 * (e >> 2) + 4 * hf + (e & 3);
          f(j < c_q ? s[e] : -INFINITY, j);
        }
      }
    });
  };
  const int kq = topk < c_q ? topk : c_q;  // spans to select for this column

  if constexpr (!WS) {
    if (c_max <= packed) {
      constexpr float kMasked = -3e38f, kNone = -3.3e38f;
      const int number = (1 << (32 - __builtin_clz(c_max > 32 ? c_max - 1 : 31))) - 1;  // the bits of a span's number
      int keep = ~number;
      asm volatile("" : "+v"(keep));  // (in a vector register: an instruction takes one scalar operand, the number)
      auto cut = [&](float x) { return __int_as_float(__float_as_int(x) & keep); };
      if (tid == 0) s_way = 0;  // (the walk ends with a barrier)
      TopVals<KMAX + 1> own;
#pragma unroll
      for (int e = 0; e <= KMAX; ++e) own.v[e] = cut(kNone);
      // Scores come into this range before they are numbered: an infinite one with a number in its low bits is a NaN, and
      // a signalling one, which would unsettle the list.  (What is not a number becomes the lowest one.)
      float infinity = INFINITY, high = 2.9e38f, low = -2.9e38f;
      asm volatile("" : "+v"(infinity), "+v"(high), "+v"(low));
      auto numbered = [&](float x, int j) {
        asm volatile("" : "+s"(j));  // one v_and_or
        return (__float_as_int(x) & keep) | j;
      };
      auto push = [&](int p) {
        const float f = __int_as_float(p);
#pragma unroll
        for (int e = KMAX; e >= 1; --e) own.v[e] = __builtin_amdgcn_fmed3f(f, own.v[e - 1], own.v[e]);
        own.v[0] = __builtin_amdgcn_fmed3f(f, own.v[0], infinity);  // (a maximum that makes no numbers canonical first)
      };
      walk([&](const f32x16& s, int j0, bool edge) {
        const int left = c_q - j0 - 4 * hf;
        auto tile = [&](auto score) {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int u = 8 * (e >> 2) + (e & 3);
            push(numbered(score(__builtin_amdgcn_fmed3f(s[e], low, high), u), j0 + u));
          }
        };
        if (edge) tile([&](float x, int u) { return u < left ? x : kMasked; });
        else tile([](float x, int) { return x; });
      });
      // bit 2 of a span's number is the lane's half
      TopVals<KMAX + 2> top;
      top.v[KMAX + 1] = cut(kNone);
#pragma unroll
      for (int e = 0; e <= KMAX; ++e) top.v[e] = own.v[e] = __int_as_float(__float_as_int(own.v[e]) | (hf << 2));
#pragma unroll
      for (int e = 0; e <= KMAX; ++e) own.v[e] = of_other_half(own.v[e]);
      const float own_last = top.v[KMAX], other_last = own.v[KMAX];
#pragma unroll
      for (int e = 0; e <= KMAX; ++e) top.push(own.v[e]);
      float kth = INFINITY, next = kNone, third = kNone;
#pragma unroll
      for (int e = 0; e < KMAX; ++e)
        if (e == kq - 1) {
          kth = top.v[e];
          next = top.v[e + 1];
          third = top.v[e + 2];
        }
      const float at = cut(kth);
      bool close = kq > 0 && next > 0.5f * kMasked && cut(next) == at;
      const bool lost = close && (cut(third) == at || cut(own_last) == at || cut(other_last) == at);
      const bool other_way = kq > 0 && !(kth > 0.5f * kMasked && at < cut(high));
      const int mine = (__builtin_amdgcn_ballot_w64(lost) != 0ull ? 1 : 0) | (__builtin_amdgcn_ballot_w64(other_way) != 0ull ? 2 : 0);
      if (mine != 0 && lane == 0) atomicOr(&s_way, mine);
      __syncthreads();
      const int way = __builtin_amdgcn_readfirstlane(s_way);
      if ((way & 2) == 0) {
        if (way != 0) {
          // A second walk over the scores that agree with the k'-th one: the bits that the number took and the number,
          // lower ones first, are all that is left to order them by, and make a whole number of at most 25 bits
          // (the exponent makes it a float that nothing flushes).  Those above the k'-th are in `top`.
          const float wanted = lost ? at : __builtin_nanf("");
          const int bits = __builtin_popcount(number);
          constexpr int kNothing = 0x20000000, kAbove = 0x30000000;
#pragma unroll
          for (int e = 0; e <= KMAX; ++e) own.v[e] = __int_as_float(kNothing);
          walk([&](const f32x16& s, int j0, bool) {
            if ((mine & 1) == 0) return;
            const int left = c_q - j0 - 4 * hf;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int u = 8 * (e >> 2) + (e & 3), x = __float_as_int(s[e]), part = x & number;
              const int key = (((x < 0 ? -part : part) + number + 1) << bits) | (number - (j0 + u)) | kNothing;
              push(cut(s[e]) == wanted && u < left ? key : kNothing);
            }
          });
          TopVals<KMAX + 1> other;
#pragma unroll
          for (int e = 0; e <= KMAX; ++e) {
            own.v[e] = __int_as_float(__float_as_int(own.v[e]) & ~(hf << 2));
            other.v[e] = of_other_half(own.v[e]);
          }
#pragma unroll
          for (int e = 0; e <= KMAX; ++e) push(__float_as_int(other.v[e]));
#pragma unroll
          for (int e = 0; e < KMAX; ++e) {
            const int j = __float_as_int(top.v[e]) & number;
            push(e < kq && cut(top.v[e]) > at ? kAbove | (number - j) : kNothing);
          }
#pragma unroll
          for (int e = 0; e < KMAX; ++e)
            top.v[e] = lost ? __int_as_float(number - (__float_as_int(own.v[e]) & number)) : top.v[e];
        }
        close = close && !lost;
        if (__builtin_amdgcn_ballot_w64(close) != 0ull) {
          // the entries that agree with the k'-th one, entry by entry: the column's own key as row qc of a product
          // with all columns, of which the diagonal is taken
          float worst = INFINITY;
          int worst_j = -1, worst_e = KMAX;
          for (int e = 0; e <= KMAX; ++e) {
            float entry = top.v[0];
#pragma unroll
            for (int x = 1; x <= KMAX; ++x) entry = x == e ? top.v[x] : entry;
            const bool in = close && e <= kq && cut(entry) == at;
            if (__builtin_amdgcn_ballot_w64(in) == 0ull) continue;
            const int j = in ? __float_as_int(entry) & number : 0;
            const bf16_t* const kp = key(j) + hf * 8;
            f32x16 s;
#pragma unroll
            for (int x = 0; x < 16; ++x) s[x] = 0.f;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
              s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kp + kk * 16), qf[kk], s, 0, 0, 0);
            float x = -INFINITY;  // row qc of column qc lies in the half (qc / 4) % 2
#pragma unroll
            for (int y = 0; y < 16; ++y) x = (y == 4 * (qc >> 3) + (qc & 3) && hf == ((qc >> 2) & 1)) ? s[y] : x;
            x = fmaxf(x, of_other_half(x));
            if (in && (x < worst || (x == worst && j > worst_j))) {
              worst = x;
              worst_j = j;
              worst_e = e;
            }
          }
#pragma unroll
          for (int e = 0; e < KMAX; ++e) top.v[e] = close && e == worst_e ? next : top.v[e];
        }
        int j[KMAX];
#pragma unroll
        for (int e = 0; e < KMAX; ++e) j[e] = e < kq ? __float_as_int(top.v[e]) & number : kEmpty;
        sort_ascending(j);
        int32_t* const oi = idx + ((int64_t)h * Lq + r) * topk;
        // the column's lanes take four entries each in turn (picked by masks: a select between two array elements
        // becomes one of their addresses, and the array goes to memory)
        const int upper = -hf;
#pragma unroll
        for (int g = 0; g < KMAX / 4; g += 2) {
          int w4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int up = 4 * g + 4 + e < KMAX ? 4 * g + 4 + e : 4 * g + e;
            w4[e] = (j[4 * g + e] & ~upper) | (j[up] & upper);
            w4[e] = w4[e] == kEmpty ? -1 : w4[e];
          }
          const int4 w = make_int4(w4[0], w4[1], w4[2], w4[3]);
          const int e0 = 4 * (g + hf);
          if (r < Lq && e0 < topk && g + hf < KMAX / 4) {
            if ((topk & 3) == 0) *reinterpret_cast<int4*>(oi + e0) = w;
            else {
              oi[e0] = w.x;
              if (e0 + 1 < topk) oi[e0 + 1] = w.y;
              if (e0 + 2 < topk) oi[e0 + 2] = w.z;
              if (e0 + 3 < topk) oi[e0 + 3] = w.w;
            }
          }
        }
        return;
      }
    }
  }
  if (tid < TMQ) s_cnt[tid] = 0;  // (read and added to after the first walk's barriers)

  // ---- pass 1: the column's top-k values
  TopVals<KMAX> top;
  top.init();
  for_each_candidate([&](float x, int) { top.push(x); });
  {
    float pv[KMAX];
#pragma unroll
    for (int e = 0; e < KMAX; ++e) pv[e] = of_other_half(top.v[e]);
#pragma unroll
    for (int e = 0; e < KMAX; ++e) top.push(pv[e]);
  }
  float thr = INFINITY;                    // kq == 0: nothing passes
  int n_gt = 0;
#pragma unroll
  for (int e = 0; e < KMAX; ++e) thr = (e == kq - 1) ? top.v[e] : thr;
#pragma unroll
  for (int e = 0; e < KMAX; ++e) n_gt += (e < kq && top.v[e] > thr) ? 1 : 0;
  const int need_eq = kq - n_gt;           // >= 1 when kq >= 1

  // ---- pass 2: collect the spans at or above the threshold
  int n_eq = 0;  // spans at the threshold this lane has listed
  for_each_candidate([&](float x, int j) {
    if (x >= thr) {  // rare: at most k' + ties of the column's candidates
      const bool eq = x == thr;
      if (!eq || n_eq < need_eq) {
        const int pos = atomicAdd(&s_cnt[col], 1);
        s_j[col][pos] = eq ? (j | 0x40000000) : j;
        if (WS) s_x[col][pos] = x;
        n_eq += eq ? 1 : 0;
      }
    }
  });
  __syncthreads();

  // ---- finish: the column's two lanes share its list entries.  An entry at the threshold is
  // kept if fewer than need_eq such entries have a lower index; the kept ones below an entry are
  // then the entries above the threshold plus min(#at-threshold below it, need_eq).
  if (r < Lq) {
    const int cnt = s_cnt[col];
    int32_t* oi = idx + ((int64_t)h * Lq + r) * topk;
    float* os = WS ? scores + ((int64_t)h * Lq + r) * topk : nullptr;
    for (int u = hf; u < cnt; u += 2) {
      const int eu = s_j[col][u], ju = eu & 0x3fffffff;
      int lower_gt = 0, lower_eq = 0;
      for (int w = 0; w < cnt; ++w) {
        const int ew = s_j[col][w];
        const bool below = (ew & 0x3fffffff) < ju;
        lower_eq += (below && (ew & 0x40000000) != 0) ? 1 : 0;
        lower_gt += (below && (ew & 0x40000000) == 0) ? 1 : 0;
      }
      if ((eu & 0x40000000) == 0 || lower_eq < need_eq) {
        const int rank = lower_gt + (lower_eq < need_eq ? lower_eq : need_eq);
        oi[rank] = ju;
        if (WS) os[rank] = s_x[col][u];
      }
    }
  }
  if (hf == 0 && r < Lq) {
    int32_t* oi = idx + ((int64_t)h * Lq + r) * topk;
    float* os = WS ? scores + ((int64_t)h * Lq + r) * topk : nullptr;
    for (int e = kq; e < topk; ++e) {
      oi[e] = -1;
      if (os) os[e] = -INFINITY;
    }
  }
}

// Up to how many candidates a workgroup goes one walk.  Long runs of agreeing scores become eight times as frequent
// with twice the spans (at 4096, one workgroup in 30), and each such workgroup walks twice: of many workgroups one in
// 30 does not show, but where all run at once the slowest is the call's time.  us, two walks -> one, top-8, mean of 8
// inputs: 1024 spans, 256 workgroups 63 -> 31, 1000: 116 -> 81; 2048 spans, 32 workgroups 110 -> 48, 256: 108 -> 81, 512:
// 134 -> 117, 1000: 209 -> 170, 2000: 377 -> 269; 4096 spans, 32 workgroups 197 -> 170, 128: 194 -> 216, 512: 244 -> 267,
// 1000: 392 -> 371, 2000: 717 -> 571.  Above 4096 spans too few bits of the score are left.
constexpr int kFewWorkgroups = 1536;

int one_walk_spans(int64_t grid) {
  return grid > kFewWorkgroups ? 4096 : 2048;
}

template <int KMAX, bool WS, bool DIRECT>
void launch_as(const Problem& pb, int grid, const void* Qs, const void* K, const void* Ks, int32_t* idx, float* scores,
               hipStream_t st) {
  hipLaunchKernelGGL((prefill_search_mfma_kernel<KMAX, WS, DIRECT>), dim3(grid), dim3(256), Stages<DIRECT>::kBytes, st,
                     static_cast<const bf16_t*>(Qs), static_cast<const bf16_t*>(K), static_cast<const bf16_t*>(Ks), idx,
                     scores, pb.Lq, pb.q_pos0, pb.G, pb.S, pb.topk, pb.n, one_walk_spans(grid), pb.qsh, pb.qst, pb.kvsh, pb.kvst);
}

// Through registers -> direct, us, 32 heads.  One walk: 65536 rows x 256 spans top-4 165.7 -> 169.4, top-8 200.1 ->
// 201.7, top-16 343 -> 302; 8000 x 125, top-12, 38.5 -> 35.7; top-32 621 -> 614 (no second instantiation for that);
// 4000 x 62, top-8, 11.8 -> 12.7.  Two walks with scores: top-4 65536 x 256 376 -> 288, 20000 x 156, top-2, 68.9 -> 66.5,
// 64 rows x 4096 spans 185 -> 169; top-8 419 -> 429, top-16 765 -> 773, top-32 2410 -> 2425.
template <int KMAX>
sl_status launch(const Problem& pb, const void* Qs, const void* K, const void* Ks, int32_t* idx,
                 float* scores, hipStream_t st) {
  const int grid = pb.Hq * (int)((pb.Lq + TMQ - 1) / TMQ);
  if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
  if (scores) launch_as<KMAX, true, KMAX <= 4>(pb, grid, Qs, K, Ks, idx, scores, st);
  else launch_as<KMAX, false, KMAX == 16>(pb, grid, Qs, K, Ks, idx, scores, st);
  if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  return hipGetLastError() == hipSuccess ? SL_OK : SL_ERR_LAUNCH;
}

}  // namespace

bool prefill_search_mfma_supported(const Problem& pb) {
  return pb.dtype == SL_BF16 && pb.D == HD && (int64_t)pb.Hq * ((pb.Lq + TMQ - 1) / TMQ) < ((int64_t)1 << 31);
}

sl_status prefill_search_mfma(const Problem& pb, const void* Qs, const void* K, const void* Ks,
                              int32_t* idx, float* scores, hipStream_t st) {
  // A list of four in lanes of five: one column in 16 whose fourth and fifth score agree has all five in one lane, which
  // then cannot tell whether a sixth does.  Longer lanes' lists instead where one such workgroup is the call's time and one
  // walk is taken: 500 rows x 1024 spans, top-4, two walks 55.5 us, lanes of five 43.7, of nine 27.2; x 2048 97, 90, 48.4.
  const int64_t grid = pb.Hq * ((pb.Lq + TMQ - 1) / TMQ), spans = (pb.q_pos0 + pb.Lq - 1) / pb.S;
  const bool longer = pb.topk == 4 && !scores && grid <= kFewWorkgroups && spans > 512 && spans <= one_walk_spans(grid);
  if (pb.topk <= 4 && !longer) return launch<4>(pb, Qs, K, Ks, idx, scores, st);
  if (pb.topk <= 8) return launch<8>(pb, Qs, K, Ks, idx, scores, st);
  if (pb.topk <= 16) return launch<16>(pb, Qs, K, Ks, idx, scores, st);
  return launch<32>(pb, Qs, K, Ks, idx, scores, st);
}

}  // namespace sl
