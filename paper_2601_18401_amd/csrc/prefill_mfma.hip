// Prefill span-attention on the matrix cores (bf16, D = 128, S a multiple of 64).
//
// Every (head, query) row picks its own spans, so a query-stationary tile has no shared K
// operand.  Following the bucketing idea of Section 4.3 (group (query, span) pairs by the key
// blocks they touch; on the fixed span grid a bucket is simply (kv head, span)), the routed part
// makes the SPAN stationary:
//
//   bucket (count) / unit_scan / scan / tiles / bucket (fill)   invert idx into per-(kv, span)
//                                   lists of query rows (integer work, LDS histograms)
//   span_flash_wide                 persistent workgroups take tiles of 256 (or 128) rows of a bucket:
//                                   gathered Q rows against the span's K/V tiles staged through
//                                   LDS, flash softmax, MFMA QK^T and PV; writes a normalised
//                                   partial (o, lse) per (row, slot)
//   span_window_wide                the local window [c*S, i]: regular tiles of as many columns
//                                   with the causal mask; joint form with topk <= 8: merges
//                                   the row's routed partials in its epilogue (log-sum-exp) and
//                                   writes O and LSE; otherwise writes the row's last partial
//   span_fine / span_fine_window    the same two with fp32 softmax weights and partials (spans of
//                                   any length, D = 64)
//   merge_partials / merge_combined streaming merge of the <= topk + 1 partials of every row
//                                   (topk > 8, and the gated combination of Section 3.4)
//
// MFMA formulation.  Both products are computed transposed so that a lane owns a query column:
//   S^T[kv][q] = K[kv][:] . Q[q][:]      A = K tile (LDS), B = Q rows (registers)
//   O^T[d][q] += V^T[d][kv] . P^T[kv][q] A = V tile (LDS, transposing reads), B = P^T straight from
//                                         the S^T accumulators (no shuffle: the K rows of a tile
//                                         are fed in an order that makes a lane's 8 consecutive
//                                         accumulators 8 consecutive kv positions)
// With v_mfma_f32_32x32x16_bf16, lane l of the 32x32 result holds column l%32 and rows
// 8*(r/4) + 4*(l/32) + r%4 for accumulator r = 0..15.
#include <mutex>

#include "kernels.h"

namespace sl {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

constexpr int TG = 128;            // rows of a tile of the fp32-weight kernels (4 wavefronts x 32 columns)
constexpr int TM = 256;            // rows of a tile of the kernels with bf16 weights (4 wavefronts x 64 columns)
constexpr int TN = 64;             // kv positions per staged tile
constexpr int HD = 128;            // head dimension of the kernels with bf16 weights

// LDS of the flash kernels (dynamic).  Main loop: two stages of the K and of the V tile, filled
// by direct global->LDS loads (16 bytes per lane, a wavefront instruction fills 1 KB
// contiguously); rows are unpadded and their 16-byte pieces XOR-swizzled so that the MFMA
// operand reads of 16 consecutive lanes hit 16 distinct bank groups:
//   K tile [64][128]: piece p of row r at position p ^ (r & 15)
//   V tile [64][128]: piece p of row r at position p ^ ((r & 3) << 2): the four rows that 16 lanes read
//                     64 bytes of (with the 16 lanes beside them) lie in different bank groups
// V is staged as it lies in memory and transposed by the LDS reads (ds_read_b64_tr_b16): a transposed
// copy of V in the workspace cost a pass over the whole cache per call, however few the rows (63 us for
// 4000 new rows behind 196000 tokens).
// Output rows go out through LDS in swizzled pieces, over stages that are dead by then.
#define SL_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// Direct global->LDS loads go through buffer instructions: base is wave-uniform, `bytes` bounds the
// offsets (a lane past it stores zeros).  The flat form (global_load_lds) counts as an LDS operation
// too, and the compiler then waits for every LDS read with lgkmcnt(0): the fragment reads that run four
// MFMAs ahead were drained at every fourth MFMA.  With the buffer form those waits are lgkmcnt(3).
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
__device__ __forceinline__ BufferRsrc buffer_of(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Two transposing LDS reads: the lane's column of kv rows 0..3 and 4..7 behind p (its own block address).  (Without
// __restrict__ the compiler knows nothing of what the reads may alias and waits for the next tile's staging loads in front of
// the products: the paper's geometry at 48K 3.55 -> 3.51 ms, 4000 rows behind 196000 tokens 845 -> 833 us.)
template <int D>
__device__ __forceinline__ bf16x8 transposed8(const bf16_t* __restrict__ p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) s16x4* LdsPtr;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)p);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)(p + 4 * D));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int D>
__device__ __forceinline__ bf16x8 transposed8(uint32_t at) {  // at: address in LDS
  return transposed8<D>((const bf16_t*)(const __attribute__((address_space(3))) bf16_t*)(uintptr_t)at);
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

__device__ __forceinline__ float pair_max(float x) {
  // lanes l and l^32 hold the two halves of a query column
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return fmaxf(__int_as_float(r[0]), __int_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}

// The paper's geometry: token range [lo, hi) that slot anchor t contributes for the query at i
// (S_t minus the window, Algorithm 1's DedupConcat(S_t, W) being that range followed by W).
// ell = l(i).  valid: t is an anchor of this query at all; the range may still be empty.
struct AnchorSpan {
  int64_t lo, hi;
  bool valid;
};
__device__ __forceinline__ AnchorSpan anchor_span_of(int64_t i, int64_t t, int64_t ell, int64_t window, int ab,
                                                     int af) {
  AnchorSpan r;
  r.valid = t >= 0 && t <= i;
  const int64_t wlo = window > 0 ? (i - window + 1 > 0 ? i - window + 1 : 0) : i + 1;
  r.lo = t - ab * ell > 0 ? t - ab * ell : 0;
  const int64_t e1 = t + af * ell < i ? t + af * ell : i;
  r.hi = (e1 < wlo - 1 ? e1 : wlo - 1) + 1;
  if (r.hi < r.lo || !r.valid) r.hi = r.lo;
  return r;
}

// ------------------------------------------------------------------ bucketing
// Inverts idx into per-(kv head, bucket) lists of (row, slot) items without a sort and without
// global atomics.  The rows of a head are cut into units of `rows` (64 .. 1024) consecutive rows, one
// wavefront each, with a histogram of its own in LDS:
//   bucket_kernel<false>      counts the unit's items per bucket -> cnt[kv][order of the unit][bucket]
//   bucket_unit_scan_kernel   per (kv head, bucket): exclusive scan of cnt over the units, in place; the
//                             total goes to g_count
//   bucket_scan_kernel / bucket_tiles_kernel   bucket offsets and tile records
//   bucket_kernel<true>       loads the unit's bases into its histogram and scatters the items
// The unit order is the item order inside a bucket.  On the grid it is (head of the group, row); on the
// paper's geometry (row, head of the group), so that the rows of a tile have nearly the same span length.
//
// Both passes are bound by the latency of idx (a row is read 16 bytes at a time, two rows per lane in
// flight) and by LDS atomics that meet in one counter (hence the rotated slots), so units are made short
// enough for four wavefronts on every SIMD.  4000 rows x 32 heads x 16
// slots: 40 + 103 us with blocks of 4096 rows that counted twice, 8 + 17 us; 262144 rows x 8 slots
// with planted needles: 226 + 456 us, 80 + 255 us.

// Grid: an entry is a span, its bucket the span itself.
struct GridItems {
  static constexpr bool kRotate = true;
  int S;  // anchor spacing
  struct Row {
    int c;  // candidates: spans [0, c)
  };
  __device__ __forceinline__ Row row(int64_t i) const {
    return {i < ((int64_t)1 << 31) ? (int)((uint32_t)i / (uint32_t)S) : (int)(i / S)};
  }
  __device__ __forceinline__ int bucket(const Row& r, int j) const { return j >= 0 && j < r.c ? j : -1; }
  __device__ __forceinline__ bool empty(const Row&, int) const { return false; }
};

// The paper's geometry: an entry is an anchor token (positions fit 32 bits); an item is a (row, slot)
// whose anchor is valid and whose span minus the window is not empty; its bucket is the block of E tokens
// that holds the span's last token.
struct AnchorItems {
  static constexpr bool kRotate = false;  // a bucket is worth computing once, and neighbours' anchors differ
  int64_t window;
  int ab, af, aroot, E;
  struct Row {
    int64_t i, ell;
  };
  __device__ __forceinline__ Row row(int64_t i) const { return {i, span_base_length(i, aroot)}; }
  __device__ __forceinline__ int bucket(const Row& r, int t) const {
    const AnchorSpan sp = anchor_span_of(r.i, t, r.ell, window, ab, af);
    return sp.hi > sp.lo ? (int)((uint32_t)(sp.hi - 1) / (uint32_t)E) : -1;
  }
  __device__ __forceinline__ bool empty(const Row& r, int t) const { return t >= 0 && t <= r.i; }
};

// j[x] = j[(x + BY) % 8] where `on`.
template <int BY>
__device__ __forceinline__ void rotate8(int (&j)[8], bool on) {
  int t[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) t[x] = on ? j[(x + BY) & 7] : j[x];
#pragma unroll
  for (int x = 0; x < 8; ++x) j[x] = t[x];
}

struct BucketPlan {
  int rows;    // rows per unit
  int units;   // units per head
  int unit_h, unit_u;  // place of unit u of head hl in its kv head's order: hl * unit_h + u * unit_u
};

// FILL: the marks of valid anchors with an empty span (lse = -inf in their partial) are written too.
template <bool FILL, typename Items>
__global__ __launch_bounds__(256) void bucket_kernel(const int32_t* __restrict__ idx, int* __restrict__ cnt,
                                                     const int* __restrict__ g_cursor, int* __restrict__ items,
                                                     float* __restrict__ part_lse, int64_t Lq, int64_t q_pos0,
                                                     int G, int topk, int n, const BucketPlan plan, const Items it) {
  extern __shared__ int s_hist[];  // [wavefronts of the block][n]
  const int h = blockIdx.y, kv = h / G, hl = h % G;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int u = blockIdx.x * (blockDim.x >> 6) + wave;
  if (u >= plan.units) return;  // (no barrier below: a unit is one wavefront's)
  int* const hist = s_hist + wave * n;
  int* const mine = cnt + ((int64_t)kv * G * plan.units + (int64_t)hl * plan.unit_h + (int64_t)u * plan.unit_u) * n;
  for (int b = lane; b < n; b += 64) hist[b] = FILL ? g_cursor[kv * n + b] + mine[b] : 0;
  __builtin_amdgcn_wave_barrier();  // (LDS operations of one wavefront complete in issue order)
  const int64_t r0 = (int64_t)u * plan.rows;
  const int64_t r1 = r0 + plan.rows < Lq ? r0 + plan.rows : Lq;
  const bool quads = (topk & 3) == 0;
  // two rows per lane at a time, eight slots of each
  for (int64_t rb = r0 + lane; rb < r1; rb += 128) {
    typename Items::Row rw[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) rw[e] = it.row(q_pos0 + rb + 64 * e);
    for (int s0 = 0; s0 < topk; s0 += 8) {
      int j[2][8];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int64_t r = rb + 64 * e;
        const int32_t* row = idx + ((int64_t)h * Lq + r) * topk + s0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          int4 v = make_int4(-1, -1, -1, -1);
          if (r < r1 && s0 + 4 * q < topk) {
            if (quads) v = *reinterpret_cast<const int4*>(row + 4 * q);
            else {
              v.x = row[4 * q];
              if (s0 + 4 * q + 1 < topk) v.y = row[4 * q + 1];
              if (s0 + 4 * q + 2 < topk) v.z = row[4 * q + 2];
              if (s0 + 4 * q + 3 < topk) v.w = row[4 * q + 3];
            }
          }
          j[e][4 * q] = v.x;
          j[e][4 * q + 1] = v.y;
          j[e][4 * q + 2] = v.z;
          j[e][4 * q + 3] = v.w;
        }
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int64_t r = rb + 64 * e;
        // neighbouring rows tend to list the same span in the same slot: lane l starts with slot l % 8
        constexpr bool kRotate = Items::kRotate;
        if (kRotate) {
          rotate8<1>(j[e], lane & 1);
          rotate8<2>(j[e], lane & 2);
          rotate8<4>(j[e], lane & 4);
        }
        if (r >= r1) continue;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int s = s0 + ((kRotate ? x + lane : x) & 7);
          if (!kRotate && s >= topk) break;
          const int b = s < topk ? it.bucket(rw[e], j[e][x]) : -1;
          if (b >= 0) {
            const int at = atomicAdd(&hist[b], 1);
            if (FILL) items[at] = (int)(((hl * Lq + r) << 5) | s);
          } else if (FILL && s < topk && it.empty(rw[e], j[e][x])) {
            part_lse[((int64_t)h * Lq + r) * (topk + 1) + s] = -INFINITY;
          }
        }
      }
    }
  }
  if (!FILL) {
    __builtin_amdgcn_wave_barrier();
    for (int b = lane; b < n; b += 64) mine[b] = hist[b];
  }
}

// grid (ceil(n / 32), Hkv), 1024 threads = 32 buckets x 32 segments of the E units of a kv head:
// exclusive scan in place, total to g_count.
__global__ __launch_bounds__(1024) void bucket_unit_scan_kernel(int* __restrict__ cnt, int* __restrict__ g_count,
                                                                int E, int n) {
  __shared__ int s_tot[32][32];
  const int bl = threadIdx.x & 31, seg = threadIdx.x >> 5;
  const int b = blockIdx.x * 32 + bl, kv = blockIdx.y;
  const int per = (E + 31) / 32, e0 = min(E, seg * per), e1 = min(E, e0 + per);
  int* const col = cnt + (int64_t)kv * E * n + b;
  int sum = 0;
  if (b < n) {
    for (int e = e0; e < e1; e += 8) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = e + u < e1 ? col[(int64_t)(e + u) * n] : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += v[u];
    }
  }
  s_tot[seg][bl] = sum;
  __syncthreads();
  if (b >= n) return;
  int run = 0;
  for (int s2 = 0; s2 < seg; ++s2) run += s_tot[s2][bl];
  for (int e = e0; e < e1; e += 8) {
    int v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = e + u < e1 ? col[(int64_t)(e + u) * n] : 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (e + u < e1) col[(int64_t)(e + u) * n] = run;
      run += v[u];
    }
  }
  if (seg == 31) g_count[kv * n + b] = run;
}

// One workgroup: exclusive scans of the item counts and of the tile counts over the B buckets.
// item_off[B] / tile_off[B] receive the totals.  The item list is laid out tile by tile, tm
// entries per tile (a bucket's last tile is padded), so that the items of tile t start at t*tm
// whatever its record says: cursor[b] = tile_off[b] * tm for the fill pass.
__global__ __launch_bounds__(1024) void bucket_scan_kernel(const int* __restrict__ g_count,
                                                           int* __restrict__ item_off,
                                                           int* __restrict__ tile_off,
                                                           int* __restrict__ g_cursor, int B, int tm,
                                                           int* __restrict__ flag, int* __restrict__ claims) {
  __shared__ int s_items[1024], s_tiles[1024];
  const int tid = threadIdx.x;
  if (flag && tid == 0) *flag = 0;
  if (tid < 8) claims[32 * tid] = 0;
  const int per = (B + 1023) / 1024;
  const int b0 = tid * per, b1 = min(B, b0 + per);
  int ni = 0, nt = 0;
  for (int b = b0; b < b1; ++b) {
    const int cnt = g_count[b];
    ni += cnt;
    nt += (cnt + tm - 1) / tm;
  }
  s_items[tid] = ni;
  s_tiles[tid] = nt;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {  // Hillis-Steele inclusive scan
    const int a = tid >= off ? s_items[tid - off] : 0;
    const int t = tid >= off ? s_tiles[tid - off] : 0;
    __syncthreads();
    s_items[tid] += a;
    s_tiles[tid] += t;
    __syncthreads();
  }
  int io = s_items[tid] - ni, to = s_tiles[tid] - nt;
  for (int b = b0; b < b1; ++b) {
    const int cnt = g_count[b];
    item_off[b] = io;
    tile_off[b] = to;
    g_cursor[b] = to * tm;
    io += cnt;
    to += (cnt + tm - 1) / tm;
  }
  if (tid == 1023) {
    item_off[B] = s_items[1023];
    tile_off[B] = s_tiles[1023];
  }
}

// One workgroup per bucket writes the record of each of its tiles,
// {bucket, first item = t*tm, number of items (1..tm), unused}, and fills the padding of the
// bucket's last tile with item 0 (row 0, slot 0 of the kv head's first query head: a valid row to
// read, whose result the flash kernel drops because the lane lies beyond the tile's item count).
__global__ __launch_bounds__(256) void bucket_tiles_kernel(const int* __restrict__ tile_off,
                                                           const int* __restrict__ item_off,
                                                           int4* __restrict__ tile_info,
                                                           int* __restrict__ items, int tm) {
  const int b = blockIdx.x;
  const int t0 = tile_off[b], t1 = tile_off[b + 1];
  const int cnt = item_off[b + 1] - item_off[b];
  for (int t = t0 + threadIdx.x; t < t1; t += 256)
    tile_info[t] = make_int4(b, t * tm, min(tm, cnt - (t - t0) * tm), 0);
  if (t1 > t0) {
    const int last = cnt - (t1 - 1 - t0) * tm;  // items of the last tile, 1..tm
    for (int e = last + threadIdx.x; e < tm; e += 256) items[(int64_t)(t1 - 1) * tm + e] = 0;
  }
}

// ------------------------------------------------------------------ flash tile
struct FlashArgs {
  const bf16_t* Q;
  const bf16_t* K;
  const bf16_t* V;
  const int32_t* idx;
  // routed
  const int* tile_off;
  const int4* tile_info;
  const int* items;
  int* claims;      // [8][32]: tiles taken of each XCD's share
  bf16_t* part_o;   // bf16 partials
  float* part_of;   // fp32 partials (fp32-weight kernels)
  float* part_lse;
  // local + merge
  bf16_t* O;
  float* LSE;
  int64_t L, Lq, q_pos0;
  int Hq, G, S, A, topk, n;  // A: anchor spacing (= S on the disjoint grid); n = ceil(L / A)
  // The paper's own geometry (Section 3.3, Algorithm 1) instead of the grid: idx holds anchor
  // TOKENS; window > 0 marks this mode.  Span of anchor t for the query at i:
  // [max(0, t - ab*l(i)), min(i, t + af*l(i))] minus the window [i - window + 1, i], l = ceil(i^(1-1/aroot)).
  // Buckets are (kv head, end block): block e holds the spans whose last token lies in
  // [e*E, (e+1)*E), E a multiple of 64 (the key-block bucketing of Section 4.3); n = ceil(L / E).
  int64_t window;
  int ab, af, aroot;
  int clip;  // fp32-weight kernels: overlapping spans in one joint softmax
  float scale_log2e;
  int64_t qsh, qst, kvsh, kvst;
};

// The kernel's arguments (its only parameter is a FlashArgs), read anew where they are used once per tile:
// kept in scalar registers across the kv loop, they fill those, and the scheduler then gives up the
// ordering of the loop's LDS reads and MFMAs.
typedef const __attribute__((address_space(4))) FlashArgs* ArgsPtr;
__device__ __forceinline__ ArgsPtr args_anew() {
  ArgsPtr p = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// Swizzle keys of the staged rows: the 16-byte pieces of the rows that 16 lanes read together fall into
// distinct bank groups (D = 64: two rows share 256 bytes).
template <int D>
__device__ __forceinline__ int k_swizzle(int row) {
  return D == 128 ? row & 15 : (row >> 1) & 7;
}
template <int D>
__device__ __forceinline__ int v_swizzle(int row) {
  return D == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2;
}

__device__ __forceinline__ int perm_row(int rho) {
  // swap bits 2 and 3: accumulator order <-> consecutive kv positions
  return (rho & 0x13) | ((rho & 4) << 1) | ((rho & 8) >> 1);
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ tiles of the kernels with bf16 weights
// A wavefront has CB blocks of 32 query columns, a workgroup four wavefronts; two workgroups share a compute unit, so that one's
// tile ends run beside the other's kv loop and their softmax and matrix phases take turns by themselves.
//
// What bounds them.  With one block of columns a product needs a fragment of 1 KB from the LDS, the LDS's whole rate; with two
// blocks half of that, and what is left is the power: the matrix pipes are busy half the time at 1.80 GHz, where a dense bf16
// product of 8192^3 reaches 1170 to 1230 TFLOP/s and spans of 2048 tokens 1050 to 1200 here, by card (980 with eight wavefronts of one block in two
// phase-shifted groups, one workgroup per compute unit).  A tile costs 1.65 us per kv step of 64 tokens and 5 us around them (2.0
// and 6 then): the gathered queries, the output.  Beside the other workgroup's products an instruction takes 8 cycles, an
// exponential 13, of which a step has what a lane's 64 scores need and little else.
// Routed part of 262144 rows, top-8, spans of 512 21.4 -> 18.4 ms; of 4000 rows x 16 spans of 512 behind 196000 tokens 724 -> 640
// us; of 49157 rows on the paper's geometry 2450 -> 2250 (eight wavefronts of one block -> this, the same card in turn).
//
// Two blocks of columns leave no register for what can be had again: values that only address things are derived anew where
// they are used.
__device__ __forceinline__ int anew(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int lane_anew() {
  int x;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(x));
  return x;
}
struct WideLds {
  static constexpr int kStage = TN * HD;          // K and V tile of a stage, one after the other
  static constexpr int kAhead = 4 * kStage * 2;   // per wavefront: the next tile's record (256 bytes) and items
  static constexpr int kRow = kAhead + 4 * 512;   // per wavefront: int row[2][64], int q[64], float lse[64], ranges
  static constexpr int kRange = kRow + 4 * 2048;  // int2[2][4]
  static constexpr int kClaim = kRange + 64;
  static constexpr int kBytes = kClaim + 16;
};

struct Range {  // of a tile; the last four: over the rows of a wavefront
  int kv, begin, end;
  int live;              // rows of the tile from the wavefront's first on: none if not positive
  int any_lo, any_last;  // the first and last token that any of its rows attends
  int all_lo, all_last;  // the range that all of them attend
  // kv rows that no row of the wavefront attends are passed over
  template <bool MASKED, int ROWS>
  __device__ __forceinline__ bool attended(int t0) const {
    return live > 0 && (!MASKED || (t0 + ROWS - 1 >= any_lo && t0 <= any_last));
  }
};

// The state and the steps of a wavefront's columns.
template <int CB>
struct WideTile {
  // kv rows at a time: 64 for one block of columns, 32 for two
  static constexpr int KB = 2 / CB, kRows = 32 * KB;
  bf16x8 qf[CB][8];
  f32x16 o[CB][4], s[CB][2];
  float m[CB];
  f32x4 l[CB];
  bf16x8 pb[CB][4];
  int kbase, vbase;
  float sc;

  __device__ __forceinline__ void setup(float scale) {
    sc = scale;
    const int lane = lane_anew();
    const int qc = lane & 31, hf = lane >> 5;
    const int krow = perm_row(qc);
    kbase = 2 * (krow * HD + ((hf ^ k_swizzle<HD>(krow)) << 3));
    const int vrow = (lane & 15) >> 2;
    vbase = 2 * ((8 * hf + vrow) * HD + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ v_swizzle<HD>(vrow)) << 3) + 4 * (lane & 1));
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) m[cb] = -INFINITY;
    clear_sums();
  }
  __device__ __forceinline__ void clear_sums() {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      l[cb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[cb][dt][r] = 0.f;
    }
  }
  // row_q: element offsets of the wavefront's queries
  __device__ __forceinline__ void load_q(const bf16_t* Q, const int* row_q) {
    const int ln = lane_anew(), hf = ln >> 5;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const bf16_t* const qp = Q + (uint32_t)row_q[cb * 32 + (ln & 31)] + hf * 8;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) qf[cb][kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
    }
  }
  template <int HALVES = KB>
  __device__ __forceinline__ void qk(const bf16_t* kt) {
    const uint32_t at = lds_address(kt) + anew(kbase);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int kb = 0; kb < HALVES; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[cb][kb][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
#pragma unroll
      for (int kb = 0; kb < HALVES; ++kb) {
        const bf16x8 ka = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>((at ^ (kk << 5)) + 64 * HD * kb);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) s[cb][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[cb][kk], s[cb][kb], 0, 0, 0);
      }
    // fragment reads run four MFMAs ahead (0x100 = LDS read, 0x008 = MFMA)
    __builtin_amdgcn_sched_group_barrier(0x100, 4 / CB, 0);
#pragma unroll
    for (int i = 0; i < 8 * HALVES - 4 / CB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, CB, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  }
  // Weights are taken against a bound of the column's scores (log2 units), which moves when a score passes it and is looked at
  // every 32 kv rows.  Weights lie in [0, 1]; the clamp that makes sure of it also keeps what is not a number out of the row
  // sums, whose product mixes columns.  A score that is not a number makes the bound one, and with it the column's output.
  //
  // The bound moves to a maximum + 8, so that the weight of that maximum, the heaviest, is a power of two and not rounded.  Where
  // the first 32 rows of a step of 64 move it, it is the maximum of all 64: with that of the 32 alone, a heavier weight, rounded,
  // is among the second 32 half the time, and the error of lse against 64 bits was 1.12 times as large at spans of 64 tokens, 1.04
  // at 128 and 1.02 at 512; 2.2 at spans of 64 with scores twice as steep.  One block of columns has the scores of both halves at
  // hand.  Two have them in a tile's first step, where the sums' registers are free; otherwise (a row's range begins later, or a
  // score passes its bound, which is rare) the second half's maxima are computed ahead.  The rule is the column's own, so that a
  // row's result does not depend on the form that takes it.
  __device__ __forceinline__ float highest(int cb, int kb) const {
    float mx = s[cb][kb][0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = __builtin_elementwise_maximum(mx, s[cb][kb][r]);
    auto pair = __builtin_amdgcn_permlane32_swap(__float_as_int(mx), __float_as_int(mx), false, false);
    return __builtin_elementwise_maximum(__int_as_float(pair[0]), __int_as_float(pair[1])) * sc;
  }
  __device__ __forceinline__ bool passed(const float (&mx)[CB]) const {
    bool any = !(mx[0] <= m[0]);
    if (CB == 2) any = any || !(mx[CB - 1] <= m[CB - 1]);
    return __builtin_amdgcn_ballot_w64(any) != 0ull;
  }
  // Columns whose mx passes their bound: to top + 8.
  __device__ __forceinline__ void move_bounds(const float (&mx)[CB], const float (&top)[CB]) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const bool grow = !(mx[cb] <= m[cb]);
      const float to = grow ? top[cb] + 8.f : m[cb];
      const float alpha = grow ? fast_exp2(m[cb] - to) : 1.f;
      m[cb] = to;
      l[cb][0] *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[cb][dt][r] *= alpha;
    }
  }
  __device__ __forceinline__ void weights(int kb) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const float nm = m[cb] == -INFINITY ? 0.f : -m[cb];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        f32x8 p;
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_fmed3f(fast_exp2(fmaf(s[cb][kb][8 * ks + e], sc, nm)), 0.f, 1.f);
        pb[cb][2 * kb + ks] = __builtin_convertvector(p, bf16x8);
      }
    }
  }
  // Row sums of the rounded weights, as a product with ones: the columns of a 16x16x32 product are columns n and n + 16 of the
  // weights, the latter as kv rows 8 .. 15 and 24 .. 31; row 0 and 8 of A ask for the former, row 4 and 12 for the latter, so that
  // the first accumulator of every lane is its own column's sum, of both halves.  (Two-element dot instructions run on the
  // matrix pipe too and take 22 cycles each beside the other workgroup's products, 350 of the 1500 that 32 kv rows took.)
  template <int B>  // block of 32 kv rows
  __device__ __forceinline__ void pv(const bf16_t* vt) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    uint64_t with = 0x1010010110100101ull;  // the lanes that hold ones: l % 4 = 0, l / 4 and l / 16 both even or both odd
    asm volatile("" : "+s"(with));
    const uint32_t x = __builtin_amdgcn_inverse_ballot_w64(with) ? 0x3f803f80u : 0u;
    const bf16x8 ones = __builtin_bit_cast(bf16x8, (u32x4){x, x, x, x});
#pragma unroll
    for (int ks = 2 * B; ks < 2 * B + 2; ++ks)  // (while the first fragments are on their way)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) l[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[cb][ks], l[cb], 0, 0, 0);
    const uint32_t at = lds_address(vt) + anew(vbase);
#pragma unroll
    for (int ks = 2 * B; ks < 2 * B + 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 va = transposed8<HD>((at ^ (dt << 6)) + 32 * ks * HD);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) o[cb][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[cb][ks], o[cb][dt], 0, 0, 0);
      }
    __builtin_amdgcn_sched_group_barrier(0x100, 8 / CB, 1);
#pragma unroll
    for (int i = 0; i < 8 - 4 / CB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, CB, 1);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 1);
  }
  // per-row ranges: only where not all rows attend
  template <bool MASKED, int HALVES = KB>
  __device__ __forceinline__ void mask(int t0, const Range& r, const int* row_range) {
    if (MASKED && (t0 < r.all_lo || t0 + 32 * HALVES - 1 > r.all_last)) {
      const int ln = lane_anew();
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int lo = row_range[32 * cb + (ln & 31)], last = row_range[128 + 32 * cb + (ln & 31)];
        const uint32_t width = last >= lo ? (uint32_t)(last - lo) : 0u;
        const uint32_t u = last >= lo ? (uint32_t)(t0 + 8 * (ln >> 5) - lo) : 0x80000000u;
#pragma unroll
        for (int kb = 0; kb < HALVES; ++kb)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            s[cb][kb][e] = u + (uint32_t)(32 * kb + 16 * (e >> 3) + (e & 7)) <= width ? s[cb][kb][e] : -INFINITY;
      }
    }
  }
  // Two blocks of columns: the maxima of 32 kv rows, scores and all.
  template <bool MASKED>
  __device__ __forceinline__ void maxima(int t0, const Range& r, const int* row_range, const bf16_t* kt, float (&mx)[CB]) {
    qk(kt);
    mask<MASKED>(t0, r, row_range);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) mx[cb] = highest(cb, 0);
  }
  // What follows the scores of the kv rows from t0 on: masks, weights, O^T += V^T P^T.  The vector instructions compete for
  // issue slots with the products of the SIMD's other wavefront; that one needs a slot every 32 cycles, this one most.
  template <bool MASKED>
  __device__ __forceinline__ void attend(int t0, const Range& r, const int* row_range, const bf16_t* vt) {
    static_assert(CB == 1);
    __builtin_amdgcn_s_setprio(3);
    mask<MASKED>(t0, r, row_range);
    const float first[CB] = {highest(0, 0)}, second[CB] = {highest(0, KB - 1)};
    const float both[CB] = {__builtin_elementwise_maximum(first[0], second[0])};
    const bool any = passed(both);  // rare: both halves' weights are there before the first product otherwise
    if (any && passed(first)) move_bounds(first, both);
    weights(0);
    if (!any) weights(KB - 1);
    __builtin_amdgcn_s_setprio(0);
    pv<0>(vt);
    if (any) {
      if (passed(second)) move_bounds(second, second);
      weights(KB - 1);
    }
    pv<KB - 1>(vt);
  }
  // The same for two blocks of columns, 32 kv rows, whose keys lie at kt.  first: of a step's 64; second: then the maxima of the
  // other 32, if they are known.
  template <bool MASKED>
  __device__ __forceinline__ void attend(int t0, const Range& r, const int* row_range, const bf16_t* kt, const bf16_t* vt, bool first,
                                         bool known, const float (&second)[CB]) {
    static_assert(CB == 2);
    __builtin_amdgcn_s_setprio(3);
    mask<MASKED>(t0, r, row_range);
    float mx[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) mx[cb] = highest(cb, 0);
    if (passed(mx)) {
      float top[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) top[cb] = second[cb];
      if (first && !known) {
        maxima<MASKED>(t0 + 32, r, row_range, kt + 32 * HD, top);
        maxima<MASKED>(t0, r, row_range, kt, mx);
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) top[cb] = __builtin_elementwise_maximum(mx[cb], top[cb]);
      move_bounds(mx, top);
    }
    weights(0);
    __builtin_amdgcn_s_setprio(0);
    pv<0>(vt);
  }
  // A tile's first 64 kv rows, two blocks of columns: there are no sums yet, whose registers hold the second half's scores.
  // (Computed ahead here too, the maxima cost 262144 rows with spans of 512 3.5 %.)  `ask` follows the scores.
  template <bool MASKED, typename Ask>
  __device__ __forceinline__ void begin(int t0, const Range& r, const int* row_range, const bf16_t* kt, Ask&& ask) {
    qk<2>(kt);
    ask();
    __builtin_amdgcn_s_setprio(3);
    mask<MASKED, 2>(t0, r, row_range);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const float mx = __builtin_elementwise_maximum(highest(cb, 0), highest(cb, 1));
      m[cb] = mx <= -INFINITY ? -INFINITY : mx + 8.f;
    }
    weights(0);
    weights(1);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    clear_sums();
    pv<0>(kt + WideLds::kStage);
    __builtin_amdgcn_sched_barrier(0);
    pv<1>(kt + WideLds::kStage);
  }
  // One block of columns, 64 kv rows from t0 on between the first and the last token that the wavefront's rows attend: whether none
  // attends any of them.  That takes rows without a token in common, in end blocks longer than a span: those of the paper's geometry
  // far behind a prompt's start, a few rows to a tile (8 rows of 8 heads behind 178499 tokens, spans of 424: 135 -> 104 us).  Blocks
  // with enough rows for tiles of two blocks of columns are shorter.
  __device__ __forceinline__ bool between(int t0, const Range& r, const int* row_range) const {
    if (r.all_lo <= r.all_last) return false;
    const int ln = lane_anew() & 31, lo = row_range[ln], last = row_range[128 + ln];
    return __builtin_amdgcn_ballot_w64(lo <= (last < t0 + 63 ? last : t0 + 63) && last >= t0) == 0ull;
  }
  // Two blocks of columns: whether a column without a score yet attends any of the 32 kv rows from t0 on.
  __device__ __forceinline__ bool begins(int t0, const int* row_range) const {
    const int ln = lane_anew();
    bool any = false;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) any = any || (m[cb] == -INFINITY && row_range[32 * cb + (ln & 31)] < t0 + 32);
    return __builtin_amdgcn_ballot_w64(any) != 0ull;
  }
  // A step's 64 kv rows.  `ask` follows the scores of the last ones.
  template <bool MASKED, typename Ask>
  __device__ __forceinline__ void step(int t0, const Range& r, const int* row_range, const bf16_t* kt, Ask&& ask) {
    const bf16_t* const vt = kt + WideLds::kStage;
    if constexpr (CB == 1) {
      if (!r.template attended<MASKED, 64>(t0) || (MASKED && between(t0, r, row_range))) return;
      qk(kt);
      ask();
      attend<MASKED>(t0, r, row_range, vt);
    } else {
      float second[CB] = {-INFINITY, -INFINITY};
      const bool ahead = MASKED && t0 <= r.all_lo && begins(t0, row_range);
      if (ahead && r.template attended<MASKED, 32>(t0 + 32)) maxima<MASKED>(t0 + 32, r, row_range, kt + 32 * HD, second);
#pragma unroll 1
      for (int at = 0; at < 64; at += 32) {
        if (!r.template attended<MASKED, 32>(t0 + at)) continue;
        qk(kt + at * HD);
        if (at != 0) ask();
        attend<MASKED>(t0 + at, r, row_range, kt + at * HD, vt + at * HD, at == 0, ahead, second);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) second[cb] = -INFINITY;
      }
    }
  }
  // The normalised output of 32 columns to LDS, [32][HD] bf16 with swizzled 16-byte pieces, and their lse.
  __device__ __forceinline__ void stage_output(int cb, bf16_t* ost, float* row_lse) {
    const int ln = lane_anew(), qc = ln & 31, hf = ln >> 5;
    const float lt = l[cb][0];
    const float inv = 1.f / lt;
    if (hf == 0) row_lse[cb * 32 + qc] = (m[cb] + __log2f(lt)) * kLn2;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int unit = (4 * dt + g4) ^ (qc & 15);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[cb][dt][4 * g4 + e] * inv;
        *reinterpret_cast<bf16x4*>(&ost[qc * HD + unit * 8 + 4 * hf]) = __builtin_convertvector(v, bf16x4);
      }
    __builtin_amdgcn_wave_barrier();
  }
  // staged output rows -> their partials: out = record of each row, -1 = none
  __device__ __forceinline__ void write_output(int cb, const bf16_t* ost, const int* out, bf16_t* part_o) {
    const int ln = lane_anew(), piece = ln & 15;
#pragma unroll
    for (int ub = 0; ub < 8; ub += 4) {
      int outs[4];
      bf16x8 vals[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = (ub + u) * 4 + (ln >> 4);
        outs[u] = out[cb * 32 + row];
        vals[u] = *reinterpret_cast<const bf16x8*>(&ost[row * HD + ((piece ^ (row & 15)) << 3)]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (outs[u] >= 0) store16_stream(part_o + (int64_t)outs[u] * HD + piece * 8, __builtin_bit_cast(uint4, vals[u]));
    }
    __builtin_amdgcn_wave_barrier();
  }
};

// (LDS operations only: a fence would wait for the stores)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Direct global -> LDS loads of a K and a V tile of 64 rows by four wavefronts, K at dst, V behind it.  BOUNDED: rows may lie
// behind the end of the sequence (zeros).  ANEW: offsets and arguments are derived where they are used (two blocks of columns).
template <bool BOUNDED, bool ANEW>
struct WideStage {
  BufferRsrc kr, vr;
  uint32_t row, kp, vp, step;
  __device__ __forceinline__ WideStage(int wave, int kvh, int t0) {
    const ArgsPtr a = ANEW ? args_anew() : (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int rows = __builtin_amdgcn_readfirstlane(a->L - t0 < TN ? (int)(a->L - t0) : TN);
    const int64_t first = uniform64((int64_t)kvh * a->kvsh + t0 * a->kvst);
    const uint32_t bytes = (uint32_t)(((rows - 1) * a->kvst + HD) * sizeof(bf16_t));
    kr = buffer_of(a->K + first, bytes);
    vr = buffer_of(a->V + first, bytes);
    // block i of the wavefront holds rows 16 * wave + 4 * i + lane / 16: what depends on i is scalar, but for K's swizzle
    const int ln = ANEW ? lane_anew() : (int)(threadIdx.x & 63);
    step = 4 * (uint32_t)a->kvst * (uint32_t)sizeof(bf16_t);
    row = (uint32_t)(wave * 16 + ln / 16) * ((uint32_t)a->kvst * (uint32_t)sizeof(bf16_t));
    kp = ((ln ^ (ln >> 4)) & 15) << 4;
    vp = row + (((ln & 15) ^ ((ln >> 4) << 2)) << 4);
  }
  __device__ __forceinline__ void issue(bf16_t* dst, int wave) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, SL_LDS_PTR(dst + (wave * 4 + i) * 512), 16,
                                               row + (kp ^ (i << 6)) + (BOUNDED ? i * step : 0), BOUNDED ? 0 : i * step, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, SL_LDS_PTR(dst + WideLds::kStage + (wave * 4 + i) * 512), 16,
                                               vp + (BOUNDED ? i * step : 0), BOUNDED ? 0 : i * step, 0, 0);
    }
  }
};

// Routed spans: XCD x (workgroups with blockIdx % 8 == x) owns the contiguous chunk [x*T/8, (x+1)*T/8) of the tile list, so that at
// any moment its workgroups sit on neighbouring tiles -- the same one or two buckets -- and share the span through that
// XCD's L2.  The record and the items of a workgroup's next tile are requested in a tile's first kv step, by direct
// global->LDS loads into the wavefront's own 512 bytes (the items of tile t sit at t * rows, so the two do not depend on each
// other), and turned into addresses in its second; its queries are asked for when the last scores are there.
//   kWhole    the grid's spans
//   kClipped  overlapping spans (anchor spacing A < S) in one joint softmax: a row's range in span j starts behind the end of the
//             nearest lower span that the row lists, so that every token of the union counts once
//   kAnchor   the paper's geometry, tiles of a (kv head, end block) bucket: every row has its own range, ending inside the
//             bucket's block; the tile walks from the lowest to the highest token of its rows
enum class Spans { kWhole, kClipped, kAnchor };

template <Spans MODE, int CB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, CB == 1 ? 2 : 8))) void span_flash_wide_kernel(const FlashArgs a) {
  constexpr bool kMasked = MODE != Spans::kWhole;
  constexpr int kCols = 32 * CB, kRows = 4 * kCols;  // columns of a wavefront, rows of a tile
  using Lds = WideLds;
  extern __shared__ __align__(16) char lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t T = a.tile_off[a.Hq / a.G * a.n];
  const int NWL = gridDim.x / 8;
  const int xcd = blockIdx.x % 8, wl = blockIdx.x / 8;
  const int c_begin = (int)(T * xcd / 8), t_begin = c_begin + wl, t_end = (int)(T * (xcd + 1) / 8);
  if (t_begin >= t_end) return;
  bf16_t* const ldsK = reinterpret_cast<bf16_t*>(lds);  // stage b: K at 2 * b * kStage, V behind it
  int* const ahead = reinterpret_cast<int*>(lds + Lds::kAhead) + wave * 128;
  int* const row_out = reinterpret_cast<int*>(lds + Lds::kRow) + wave * 512;
  int* const row_q = row_out + 128;
  float* const row_lse = reinterpret_cast<float*>(row_out + 192);
  int* const row_range = row_out + 256;  // kMasked: int lo[2][64], last[2][64]
  int2* const s_range = reinterpret_cast<int2*>(lds + Lds::kRange);
  int* const s_claim = reinterpret_cast<int*>(lds + Lds::kClaim);

  // what a tile's record and items say: its kv range, and, per row, where its query and its partial are (to LDS)
  auto describe = [&](int bucket, int count, const int* items, int turn) {
    const ArgsPtr a = args_anew();
    const int lane = lane_anew(), ln = lane & (kCols - 1);  // (anew: what the exchanges below address is not kept)
    Range r = {};
    r.kv = bucket / a->n;
    r.live = count - wave * kCols;
    const int j = bucket % a->n;
    r.end = (j + 1) * a->A;
    r.begin = r.end - a->S > 0 ? r.end - a->S : 0;
    const int item = items[ln];
    const int rowid = item >> 5, slot = item & 31;
    const int hl = (uint32_t)rowid / (uint32_t)a->Lq;
    const int row = rowid - hl * (int)a->Lq;
    const int h = r.kv * a->G + hl;
    const bool real = wave * kCols + ln < count;
    row_q[ln] = (int)(h * a->qsh + row * a->qst);
    row_out[64 * turn + ln] = real ? (h * (int)a->Lq + row) * (a->topk + 1) + slot : -1;
    if constexpr (kMasked) {
      int lo = r.begin, last = r.end - 1;
      const int32_t* const irow = a->idx + ((int64_t)h * a->Lq + row) * a->topk;
      if constexpr (MODE == Spans::kClipped) {
        const int c = (int)((uint32_t)(a->q_pos0 + row) / (uint32_t)a->A);  // (positions lie below 2^24)
        for (int s2 = 0; s2 < a->topk; ++s2) {
          const int jj = irow[s2];
          if (jj >= 0 && jj < c && jj < j && (jj + 1) * a->A > lo) lo = (jj + 1) * a->A;
        }
      } else {
        const int64_t i = a->q_pos0 + row;
        const AnchorSpan sp = anchor_span_of(i, irow[slot], span_base_length(i, a->aroot), a->window, a->ab, a->af);
        lo = (int)sp.lo;
        last = (int)sp.hi - 1;
      }
      row_range[64 * turn + ln] = real ? lo : INT32_MAX;  // (padding attends nothing)
      row_range[128 + 64 * turn + ln] = real ? last : -1;
      const bool some = real && last >= lo;
      r.any_lo = some ? lo : INT32_MAX;
      r.all_lo = some ? lo : 0;
      r.any_last = some ? last : -1;
      r.all_last = some ? last : INT32_MAX;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        const int from = (lane ^ off) << 2;
        r.any_lo = min(r.any_lo, __builtin_amdgcn_ds_bpermute(from, r.any_lo));
        r.all_lo = max(r.all_lo, __builtin_amdgcn_ds_bpermute(from, r.all_lo));
        r.any_last = max(r.any_last, __builtin_amdgcn_ds_bpermute(from, r.any_last));
        r.all_last = min(r.all_last, __builtin_amdgcn_ds_bpermute(from, r.all_last));
      }
      r.any_lo = __builtin_amdgcn_readfirstlane(r.any_lo);
      r.all_lo = __builtin_amdgcn_readfirstlane(r.all_lo);
      r.any_last = __builtin_amdgcn_readfirstlane(r.any_last);
      r.all_last = __builtin_amdgcn_readfirstlane(r.all_last);
      if (MODE == Spans::kAnchor && ln == 0) s_range[4 * turn + wave] = make_int2(r.any_lo, r.any_last);
    }
    return r;
  };
  // kAnchor: from the lowest token to the highest of the tile's rows, behind a barrier
  auto whole_range = [&](Range& r, int turn) {
    if constexpr (MODE == Spans::kAnchor) {
      int lo = INT32_MAX, last = -1;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int2 x = s_range[4 * turn + w];
        lo = min(lo, x.x);
        last = max(last, x.y);
      }
      lo = __builtin_amdgcn_readfirstlane(last < lo ? 0 : lo);
      last = __builtin_amdgcn_readfirstlane(last < 0 ? 0 : last);
      r.begin = lo / TN * TN;
      r.end = (last / TN + 1) * TN;
    }
  };
  WideTile<CB> tile;
  auto stage = [&](int kvh, int t0, int b) { WideStage<kMasked, CB == 2>(wave, kvh, t0).issue(ldsK + 2 * b * Lds::kStage, wave); };
  auto load_q = [&] { tile.load_q(args_anew()->Q, row_q); };

  int b = 0, turn = 0;
  Range cur;
  {
    const int4 info = a.tile_info[t_begin];
    cur = describe(info.x, info.z, a.items + (int64_t)t_begin * kRows + wave * kCols, 0);
    if (MODE == Spans::kAnchor) {
      lds_barrier();
      whole_range(cur, 0);
    }
    load_q();
    stage(cur.kv, cur.begin, b);
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }
  int claimed = 0;
  // Tiles are claimed one by one, from a counter of the XCD's (equal shares: 12 % of the time without a tile at the end): a
  // workgroup has its second one from the start, and asks for the one after its next while it ends a tile.
  for (bool first = true;; first = false) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    if (!first && wave == 0 && lane_anew() == 0) *s_claim = claimed;
    claimed = 0;
    tile.setup(args_anew()->scale_log2e);
    lds_barrier();
    const int next = first ? t_begin + NWL : c_begin + 2 * NWL + __builtin_amdgcn_readfirstlane(*s_claim);
    const bool has_next = next < t_end;
    Range nxt = cur;
    // what comes before a step's scores: the next step's rows, and word of the next tile
    auto arrive = [&](int t0) {
      if (t0 + TN < cur.end) stage(cur.kv, t0 + TN, b ^ 1);
      if (!has_next) return;
      if (t0 == cur.begin) {
        const ArgsPtr a = args_anew();
        const int ln = lane_anew();
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(a->tile_info + next, 16), SL_LDS_PTR(ahead), 4, (ln & 3) * 4, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(a->items + (int64_t)next * kRows + wave * kCols, kCols * 4),
                                                 SL_LDS_PTR(ahead + 64), 4, ln * 4, 0, 0, 0);
      }
      const bool last = t0 + TN >= cur.end;
      if (t0 == cur.begin + TN || (last && t0 == cur.begin)) {
        if (last) __builtin_amdgcn_s_waitcnt(0x0F70);  // (one step: they are not here yet)
        nxt = describe(__builtin_amdgcn_readfirstlane(ahead[0]), __builtin_amdgcn_readfirstlane(ahead[2]), ahead + 64, turn ^ 1);
      }
    };
    int t0 = cur.begin;
    arrive(t0);
    tile.clear();
    // the queries are needed no more once the scores of the tile's last kv rows are there
    bool asked = !has_next;
    auto ask = [&] {
      if (asked || t0 + TN < cur.end) return;
      load_q();
      asked = true;
    };
    if (CB == 2 && cur.attended<kMasked, 32>(t0) && cur.attended<kMasked, 32>(t0 + 32)) {
      tile.template begin<kMasked>(t0, cur, row_range + 64 * turn, ldsK + 2 * b * Lds::kStage, ask);
      b ^= 1;
      t0 += TN;
    }
    auto next_step = [&](auto&& ask) {
      if (t0 != cur.begin) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        lds_barrier();
        arrive(t0);
      }
      tile.template step<kMasked>(t0, cur, row_range + 64 * turn, ldsK + 2 * b * Lds::kStage, ask);
      b ^= 1;
      t0 += TN;
    };
    // Loads of queries inside the loop make the compiler wait for the next kv rows behind the first products of every step: 0.3 %
    // of a long prompt, but a quarter of a call whose tiles are too few to fill the chip.  The paper's geometry with two blocks of
    // columns, which only large calls have, has no registers for the last step's own code (44 of 256 would go to memory).
    constexpr bool kOwnLast = CB == 1 || MODE != Spans::kAnchor;
#pragma unroll 1
    while (t0 + (kOwnLast ? TN : 0) < cur.end) {
      if constexpr (kOwnLast) next_step([] {});
      else next_step(ask);
    }
    if (kOwnLast && t0 < cur.end) next_step(ask);
    ask();  // (a wavefront none of whose rows attends the last ones)
    lds_barrier();
    if (has_next && wave == 0 && lane_anew() == 0)
      claimed = (int)__builtin_amdgcn_atomic_inc32((uint32_t*)&args_anew()->claims[32 * xcd], 0xffffffffu, __ATOMIC_RELAXED, "agent");
    if (has_next) {
      whole_range(nxt, turn ^ 1);
      stage(nxt.kv, nxt.begin, b);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // the other stage is dead until the next tile's first barrier
    bf16_t* const ost = ldsK + 2 * (b ^ 1) * Lds::kStage + wave * 4096;
    const int* const out = row_out + 64 * turn;
    const ArgsPtr pa = args_anew();
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      tile.stage_output(cb, ost, row_lse);
      tile.write_output(cb, ost, out, pa->part_o);
    }
    {
      const int ln = lane_anew(), to = out[ln & (kCols - 1)];
      if (ln < kCols && to >= 0) __builtin_nontemporal_store(row_lse[ln], &pa->part_lse[to]);
    }
    if (!has_next) break;
    cur = nxt;
    turn ^= 1;
  }
}

// A window tile's columns (128 or 256) are `heads` query heads of one kv head, which attend the same keys, times columns / heads rows:
// the fewer rows, the shorter the kv range that the tile walks beyond what each of its rows attends.  Heads: the largest
// power of two that divides the group, up to 8.  Tiles of 128 rows of one head -> 16 rows of 8, us, 32:4 heads: 20011 rows,
// spans of 142 (fp32 weights) 181 -> 140; 4000 rows, spans of 512 47 -> 43.
__host__ __device__ inline int local_heads(int G) {
  const int p = G & -G;
  return p < 8 ? p : 8;
}
// Row tiles and their grouping into chunks of `tps` tiles (the tiles of one span when S is a multiple of the tile height).
struct LocalMap {
  int shift, rows;         // rows of a tile, a power of two: what depends on it is shifted, not divided
  int tiles, tps, chunks;  // tiles of a kv head (and group of `heads` heads)
};
__host__ __device__ inline LocalMap local_map(int64_t Lq, int S, int G, int columns) {
  LocalMap m;
  m.shift = __builtin_ctz(columns / local_heads(G));
  m.rows = 1 << m.shift;
  m.tiles = (int)((Lq + m.rows - 1) >> m.shift);
  // No more than an eighth of the tiles in a run: the paper's geometry, whose runs are 1024 tokens long, 1024 rows behind
  // 48133 tokens 407 -> 285 us, 4096 530 -> 444, a prompt of 3000 253 -> 161.
  const int each = (m.tiles + 7) / 8;
  m.tps = (S >> m.shift) < each ? S >> m.shift : each;
  m.tps = m.tps > 0 ? m.tps : 1;
  m.chunks = (m.tiles + m.tps - 1) / m.tps;
  return m;
}
// Blocks to launch: 8 x the largest per-XCD share.
inline unsigned local_grid(int64_t Lq, int S, int Hkv, int G, int columns) {
  const LocalMap m = local_map(Lq, S, G, columns);
  int best = 0;
  for (int x = 0; x < 8; ++x) {
    const int cx = (m.chunks - x + 7) / 8;
    const bool lx = m.chunks > 0 && (m.chunks - 1) % 8 == x;
    const int tx = cx * m.tps - (lx ? m.chunks * m.tps - m.tiles : 0);
    best = tx > best ? tx : best;
  }
  return (unsigned)(8 * Hkv * best * (G / local_heads(G)));
}

// Workgroup -> (heads, row tile) of a window kernel, XCD-aware: blocks are dealt round-robin to the 8 XCDs, each
// with its own L2.  A run of `tps` consecutive row tiles (one span's worth) goes to one XCD,
// and inside an XCD the groups of heads of a kv head take the same row tile back to back, so the
// window's K/V tiles are fetched from HBM about once.
struct LocalTile {
  bool any;  // the grid is padded to 8 * the largest share
  int kv, tile, head0;
};
__device__ __forceinline__ LocalTile local_tile(const LocalMap& lm, int columns, int Hkv, int G) {
  const int heads = columns >> lm.shift, sets = G / heads;
  const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const int chunks_x = (lm.chunks - xcd + 7) / 8;                 // chunks xcd, xcd+8, ... of a kv head
  const bool has_last = lm.chunks > 0 && (lm.chunks - 1) % 8 == xcd;  // the only chunk that may be short
  const int tiles_x = chunks_x * lm.tps - (has_last ? lm.chunks * lm.tps - lm.tiles : 0);
  LocalTile t;
  t.any = slot < Hkv * tiles_x * sets;
  if (!t.any) return t;
  t.kv = slot / (tiles_x * sets);
  const int rem = slot % (tiles_x * sets), tile_local = rem / sets;
  t.tile = (xcd + 8 * (tile_local / lm.tps)) * lm.tps + tile_local % lm.tps;
  t.head0 = t.kv * G + rem % sets * heads;
  return t;
}

// ------------------------------------------------------------------ tiles of the kernels with fp32 weights
// Tiles of 128 rows, one block of 32 query columns per wavefront, the kv rows 32 at a time; spans of any length at any offset.
// Every softmax weight is split into three bf16 parts, which hold the 24 bits of its mantissa between them, and V is
// multiplied with all three; the row sum is taken over the unsplit weights, partials are written in fp32.
//
// What bounds them: a step of 32 kv rows is 32 products (D = 128), and 39000 tiles take 103 us for each (spans of 78 to 238 tokens
// lie on a line; 72 at D = 64), 1.6 PFLOP/s, where a dense product reaches 1.2: a measured cost, not a limit that is known.  A
// tile's 64 KB of partials take 490 us in all at what scattered 512-byte rows are written at (5.2 TB/s), its gathered queries 190
// at least.  Routed part, kernels of 64 kv rows at a time -> these, us: 20011 rows, top-8, 32:4 heads, spans of 142 1250 -> 930 (D = 64:
// 690 -> 555); 6400 rows with spans of 80 306 -> 210; 2500 with 50 92 -> 76.  What gave it:
//   - steps of 32 instead of 64 kv rows, so that three workgroups share a compute unit (D = 64: four) and a span of 142 is 160
//     rows' work instead of 192's;
//   - the next tile's record, queries and first stage are asked for before a tile's output leaves, and its stores are not waited
//     for: what is older than they are is (vector memory completes in order);
//   - the split by cutting, not rounding: 11 instructions for two weights instead of 15;
//   - lse stored through the caches, next to the row's other slots' (past them, 4 bytes at a time, 2500 rows: 98 us; the bf16
//     partials' kernel is the other way round: 8192 rows, spans of 64 201 past them, 216 through).
// Measured and not taken: whole rows of 256 bytes per store instruction (+1 %), records two tiles ahead, fragment reads in a
// fixed order (+-1 %), a workgroup per tile (+4 %).
constexpr int fine_blocks(int D, int TT) { return TT * D == 4096 ? (D == 128 ? 3 : 4) : 2; }  // workgroups per compute unit

template <int D, int TT>  // TT: tokens of a staged K and V tile
struct FineLds {
  static constexpr int kStage = TT * D;
  static constexpr int kAhead = 4 * kStage * 2;          // per wavefront: the next tile's record (256 bytes) and items
  static constexpr int kRow = kAhead + 4 * 512;          // per wavefront: int row[2][32], int q[32], int lo[2][32], last[2][32]
  static constexpr int kClaim = kRow + 4 * 896;
  static constexpr int kBytes = kClaim + 16;
};

// p = hi + mid + low exactly: 8 bits of the mantissa each.
__device__ __forceinline__ void split24(f32x8 p, bf16x8* hi, bf16x8* mid, bf16x8* low) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 part[3];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    float x = p[e], y = p[e + 1];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      part[i][e / 2] = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);  // the upper halves of x and y
      x -= __uint_as_float(__float_as_uint(x) & 0xffff0000u);
      y -= __uint_as_float(__float_as_uint(y) & 0xffff0000u);
    }
  }
  *hi = __builtin_bit_cast(bf16x8, part[0]);
  *mid = __builtin_bit_cast(bf16x8, part[1]);
  *low = __builtin_bit_cast(bf16x8, part[2]);
}

// fp32 partials of a pass: less than 4 GiB of them (kFineMaxScratch holds the lists, too), so that 32-bit offsets reach all.
struct FlashPartials {
  float* o;
  float* lse;
  uint32_t records;
};
constexpr uint32_t kNoRecord = 0xffff0000u;

template <int D>
struct FineTile {
  static constexpr int NDT = D / 32, NKK = D / 16;
  bf16x8 qf[NKK];
  f32x16 o[NDT], s;
  float m, l;  // m in log2 units of the scaled logit; l of the lane's half of the kv rows
  int kbase, vbase;
  float sc;

  __device__ __forceinline__ void setup(float scale) {
    sc = scale;
    const int lane = threadIdx.x & 63, qc = lane & 31, hf = lane >> 5;
    const int krow = perm_row(qc);
    kbase = 2 * (krow * D + ((hf ^ k_swizzle<D>(krow)) << 3));
    const int vrow = (lane & 15) >> 2;
    vbase = 2 * ((8 * hf + vrow) * D + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ v_swizzle<D>(vrow)) << 3) + 4 * (lane & 1));
  }
  __device__ __forceinline__ void clear() {
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  }
  __device__ __forceinline__ void load_q(const bf16_t* Q, const int* row_q) {
    const int ln = lane_anew();
    const bf16_t* const qp = Q + (uint32_t)row_q[ln & 31] + (ln >> 5) * 8;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
  }
  __device__ __forceinline__ void qk(const bf16_t* kt) {
    const uint32_t at = lds_address(kt) + kbase;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      const bf16x8 ka = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(at ^ (kk << 5));
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[kk], s, 0, 0, 0);
    }
  }
  // What follows the scores of the 32 kv rows from t0 on.  fresh: the tile's first; masked: not all rows of the wavefront attend
  // them all.
  __device__ __forceinline__ void attend(int t0, bool fresh, bool masked, const int* row_range, const bf16_t* vt) {
    __builtin_amdgcn_s_setprio(3);
    if (masked) {
      const int ln = lane_anew();
      const int lo = row_range[ln & 31], last = row_range[64 + (ln & 31)];
      const uint32_t width = last >= lo ? (uint32_t)(last - lo) : 0u;
      const uint32_t u = last >= lo ? (uint32_t)(t0 + 8 * (ln >> 5) - lo) : 0x80000000u;
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = u + (uint32_t)(16 * (e >> 3) + (e & 7)) <= width ? s[e] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = pair_max(mx) * sc;
    // Lazy rescale, decided per column: a column's running maximum only moves when that column grew by more than 2^8; until
    // then its exponentials are taken against the old maximum (p <= 256).  The branch is per wavefront, the arithmetic of a
    // column does not depend on the columns it shares the wavefront with.
    const bool grow = mx > m + 8.f || (m == -INFINITY && mx > -INFINITY);
    if (__builtin_amdgcn_ballot_w64(grow) != 0ull) {
      const float alpha = grow ? fast_exp2(m - mx) : 1.f;  // m = -inf: 0, and l and o are still 0
      m = grow ? mx : m;
      if (!fresh) {
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      }
    }
    const float nm = m > -INFINITY ? -m : 0.f;  // whole column masked so far: exponentials are 0 anyway
    const uint32_t at = lds_address(vt) + vbase;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      f32x8 p;
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = fast_exp2(fmaf(s[8 * ks + e], sc, nm));
#pragma unroll
      for (int e = 0; e < 8; ++e) l += p[e];
      bf16x8 hi, mid, low;
      split24(p, &hi, &mid, &low);
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const bf16x8 va = transposed8<D>((at ^ (dt << 6)) + 32 * ks * D);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, hi, o[dt], 0, 0, 0);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, mid, o[dt], 0, 0, 0);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, low, o[dt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
  }
  // The normalised output in fp32, 32 columns of o at a time through 4 KB of LDS (swizzled 16-byte pieces), 8 lanes a row.
  // Written past the caches: the partials are gigabytes, the K/V tiles keep the L2.  D / 8 + 1 stores, whatever rows there
  // are: those of a row without a record (out = -1) lie out of the buffer's range and are dropped.
  __device__ __forceinline__ void write_output(float* ost, const int* out, const FlashPartials& to) {
    const int ln = lane_anew(), qc = ln & 31, hf = ln >> 5, piece = ln & 7;
    const float lt = pair_sum(l), inv = 1.f / lt;
    const BufferRsrc ob = buffer_of(to.o, to.records * (D * 4)), lb = buffer_of(to.lse, to.records * 4);
    constexpr int kNt = 2;
    {
      // The bound is the first 32 kv rows', so that sums grow; the logarithm of one is taken in two parts, of which only the
      // small one is rounded by the instruction (20011 rows, spans of 142: lse is 2.05e-7 off, 2.87e-7 otherwise).
      const float whole = (float)__builtin_amdgcn_frexp_expf(lt), rest = __log2f(__builtin_amdgcn_frexp_mantf(lt)) * kLn2;
      const float lse = fmaf(m, kLn2, fmaf(whole, kLn2, rest));
      const int at = out[qc];
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(lse), lb, at >= 0 && hf == 0 ? (uint32_t)at * 4u : kNoRecord, 0, 0);
    }
    uint32_t to_row[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int at = out[8 * u + (ln >> 3)];
      to_row[u] = at >= 0 ? (uint32_t)at * (D * 4u) + 16 * piece : kNoRecord;
    }
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[dt][4 * g4 + e] * inv;
        *reinterpret_cast<f32x4*>(&ost[qc * 32 + (((2 * g4 + hf) ^ (qc & 7)) << 2)]) = v;
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const int row = 8 * u + (ln >> 3);
        const f32x4 v = *reinterpret_cast<const f32x4*>(&ost[row * 32 + ((piece ^ (row & 7)) << 2)]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ob, to_row[u] + 128 * dt, 0, kNt);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
};

__device__ __forceinline__ void stage_block(bf16_t* dst, BufferRsrc from, uint32_t off) {  // 1 KB, global -> LDS
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, SL_LDS_PTR(dst), 16, off, 0, 0, 0);
}

// Direct global -> LDS loads of a staged K and V tile, K at dst, V behind it; rows from `end` on are zeros.
template <int D, int TT>
struct FineStage {
  static constexpr int kBlocks = TT * D / 2048;  // of 1 KB, per wavefront
  BufferRsrc kr, vr;
  uint32_t koff[kBlocks], voff[kBlocks];
  __device__ __forceinline__ FineStage(int wave, int kvh, int t0, int end) {
    constexpr int PPR = D / 8, RPB = 64 / PPR;  // 16-byte pieces per row, rows per 1 KB block
    const ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int rows = __builtin_amdgcn_readfirstlane(end - t0 < TT ? end - t0 : TT);
    const int64_t first = uniform64((int64_t)kvh * a->kvsh + t0 * a->kvst);
    const uint32_t bytes = (uint32_t)(((rows - 1) * a->kvst + D) * sizeof(bf16_t));
    kr = buffer_of(a->K + first, bytes);
    vr = buffer_of(a->V + first, bytes);
    const int ln = lane_anew();
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
      const int row = (wave * kBlocks + i) * RPB + ln / PPR, pc = ln % PPR;
      koff[i] = (uint32_t)((row * a->kvst + (pc ^ k_swizzle<D>(row)) * 8) * sizeof(bf16_t));
      voff[i] = (uint32_t)((row * a->kvst + (pc ^ v_swizzle<D>(row)) * 8) * sizeof(bf16_t));
    }
  }
  __device__ __forceinline__ void issue(bf16_t* dst, int wave) const {
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
      stage_block(dst + (wave * kBlocks + i) * 512, kr, koff[i]);
      stage_block(dst + TT * D + (wave * kBlocks + i) * 512, vr, voff[i]);
    }
  }
};

// Routed spans of the fp32-weight kernels: tiles shared out and claimed as in span_flash_wide_kernel.  a.clip: spans of a row
// overlap in one joint softmax, and a row's range starts behind the end of the nearest lower span that it lists.
template <int D, int TT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TT * D > 4096 ? 2 : D == 128 ? 3 : 4, TT * D > 4096 ? 2 : D == 128 ? 3 : 4)))
void span_fine_kernel(const FlashArgs a) {
  using Lds = FineLds<D, TT>;
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t T = a.tile_off[a.Hq / a.G * a.n];
  const int NWL = gridDim.x / 8;
  const int xcd = blockIdx.x % 8, wl = blockIdx.x / 8;
  const int c_begin = (int)(T * xcd / 8), t_begin = c_begin + wl, t_end = (int)(T * (xcd + 1) / 8);
  if (t_begin >= t_end) return;
  bf16_t* const stages = reinterpret_cast<bf16_t*>(lds);  // stage b: K at 2 * b * kStage, V behind it
  int* const ahead = reinterpret_cast<int*>(lds + Lds::kAhead) + wave * 128;
  int* const row_out = reinterpret_cast<int*>(lds + Lds::kRow) + wave * 224;
  int* const row_q = row_out + 64;
  int* const row_range = row_out + 96;  // int lo[2][32], last[2][32]
  int* const s_claim = reinterpret_cast<int*>(lds + Lds::kClaim);

  struct Span {
    int kv, begin, end, live, all_lo;  // all_lo: where the last of the wavefront's rows starts
  };
  auto describe = [&](int bucket, int count, const int* items, int turn) {
    const ArgsPtr p = args_anew();
    const int ln = lane & 31;
    Span r;
    r.kv = bucket / p->n;
    r.live = wave * 32 < count;
    const int j = bucket % p->n;
    r.end = (j + 1) * p->A;
    r.begin = r.end - p->S > 0 ? r.end - p->S : 0;
    const int item = items[ln];
    const int rowid = item >> 5, slot = item & 31;
    const int hl = (uint32_t)rowid / (uint32_t)p->Lq;
    const int row = rowid - hl * (int)p->Lq;
    const int h = r.kv * p->G + hl;
    row_q[ln] = (int)(h * p->qsh + row * p->qst);
    row_out[32 * turn + ln] = wave * 32 + ln < count ? (h * (int)p->Lq + row) * (p->topk + 1) + slot : -1;
    int lo = r.begin;
    r.all_lo = r.begin;
    if (p->clip) {
      const int c = (int)((uint32_t)(p->q_pos0 + row) / (uint32_t)p->A);  // (positions lie below 2^24)
      const int32_t* irow = p->idx + ((int64_t)h * p->Lq + row) * p->topk;
      for (int s2 = 0; s2 < p->topk; ++s2) {
        const int jj = irow[s2];
        if (jj >= 0 && jj < c && jj < j && (jj + 1) * p->A > lo) lo = (jj + 1) * p->A;
      }
      int most = lo;
#pragma unroll
      for (int off = 16; off >= 1; off >>= 1) most = max(most, __shfl_xor(most, off, 64));
      r.all_lo = __builtin_amdgcn_readfirstlane(most);
    }
    row_range[32 * turn + ln] = lo;
    row_range[64 + 32 * turn + ln] = r.end - 1;
    return r;
  };

  FineTile<D> tile;
  tile.setup(a.scale_log2e);
  int b = 0, turn = 0;
  Span cur;
  {
    const int4 info = a.tile_info[t_begin];
    cur = describe(info.x, info.z, a.items + (int64_t)t_begin * TG + wave * 32, 0);
    FineStage<D, TT>(wave, cur.kv, cur.begin, cur.end).issue(stages, wave);
    tile.load_q(a.Q, row_q);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  }
  int claimed = 0;
  for (bool first = true;; first = false) {
    if (!first && threadIdx.x == 0) *s_claim = claimed;
    lds_barrier();
    const int next = first ? t_begin + NWL : c_begin + 2 * NWL + __builtin_amdgcn_readfirstlane(*s_claim);
    const bool has_next = next < t_end;
    Span nxt = cur;
    tile.clear();
    const int final = cur.begin + (cur.end - cur.begin - 1) / 32 * 32;  // the span's last 32 kv rows, or fewer
#pragma unroll 1
    for (int t0 = cur.begin; t0 < cur.end; t0 += TT) {
      if (t0 != cur.begin) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        lds_barrier();
      }
      const bool last = t0 + TT >= cur.end;
      if (!last) FineStage<D, TT>(wave, cur.kv, t0 + TT, cur.end).issue(stages + 2 * (b ^ 1) * Lds::kStage, wave);
      if (has_next && t0 == cur.begin) {
        const ArgsPtr p = args_anew();
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(p->tile_info + next, 16), SL_LDS_PTR(ahead), 4, (lane & 3) * 4, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(p->items + (int64_t)next * TG + wave * 32, 128), SL_LDS_PTR(ahead + 64), 4,
                                                 lane * 4, 0, 0, 0);
      }
      const bf16_t* const kt = stages + 2 * b * Lds::kStage;
      const int until = t0 + TT < final ? t0 + TT : final;
      if (cur.live) {
#pragma unroll 1
        for (int at = t0; at < until; at += 32) {
          tile.qk(kt + (at - t0) * D);
          tile.attend(at, at == cur.begin, at < cur.all_lo, row_range + 32 * turn, kt + Lds::kStage + (at - t0) * D);
        }
      }
      b ^= 1;
    }
    if (has_next) {
      if (cur.end - cur.begin <= TT) __builtin_amdgcn_s_waitcnt(0x0F70);  // (one stage: they may not be here yet)
      nxt = describe(__builtin_amdgcn_readfirstlane(ahead[0]), __builtin_amdgcn_readfirstlane(ahead[2]), ahead + 64, turn ^ 1);
    }
    // the span's last kv rows: the queries are needed no more once their scores are there
    const bf16_t* const kt = stages + (2 * (b ^ 1) * Lds::kStage + (final - cur.begin) % TT * D);
    tile.qk(kt);
    if (has_next) {
      tile.load_q(args_anew()->Q, row_q);
      if (threadIdx.x == 0)
        claimed = (int)__builtin_amdgcn_atomic_inc32((uint32_t*)&args_anew()->claims[32 * xcd], 0xffffffffu, __ATOMIC_RELAXED, "agent");
    }
    tile.attend(final, final == cur.begin, final < cur.all_lo || final + 32 > cur.end, row_range + 32 * turn, kt + Lds::kStage);
    lds_barrier();
    if (has_next) FineStage<D, TT>(wave, nxt.kv, nxt.begin, nxt.end).issue(stages + 2 * b * Lds::kStage, wave);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // the other stage is dead until the next tile's first barrier
    const ArgsPtr pa = args_anew();
    tile.write_output(reinterpret_cast<float*>(stages + 2 * (b ^ 1) * Lds::kStage + wave * 2048), row_out + 32 * turn,
                      FlashPartials{pa->part_of, pa->part_lse, (uint32_t)(pa->Hq * (int)pa->Lq * (pa->topk + 1))});
    // What is older than the output's last D / 8 stores: the next tile's queries and its first stage.
    __builtin_amdgcn_s_waitcnt(D == 128 ? 0x4F70 : 0x0F78);
    if (!has_next) break;
    cur = nxt;
    turn ^= 1;
  }
}

// Local window [c*S, i] of the fp32-weight kernels: tiles of 128 columns with the causal mask; writes the window's partial into
// the row's last slot.
template <int D, int TT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TT * D > 4096 ? 2 : D == 128 ? 3 : 4, TT * D > 4096 ? 2 : D == 128 ? 3 : 4)))
void span_fine_window_kernel(const FlashArgs a) {
  using Lds = FineLds<D, TT>;
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bf16_t* const stages = reinterpret_cast<bf16_t*>(lds);
  int* const row_out = reinterpret_cast<int*>(lds + Lds::kRow) + wave * 224;
  int* const row_q = row_out + 64;
  int* const row_range = row_out + 96;
  const LocalMap lm = local_map(a.Lq, a.A, a.G, TG);
  const LocalTile lt = local_tile(lm, TG, a.Hq / a.G, a.G);
  if (!lt.any) return;
  const int r0 = lt.tile << lm.shift;
  auto window_of = [&](int i) { return (int)((uint32_t)i / (uint32_t)a.A) * a.A; };  // (positions lie below 2^24)
  auto pos = [&](int r) { return (int)(a.q_pos0 + (r < (int)a.Lq ? r : (int)a.Lq - 1)); };
  {
    const int ln = lane & 31, col = wave * 32 + ln;
    const int h = lt.head0 + (col >> lm.shift);
    const int r = r0 + (col & (lm.rows - 1));
    const int rc = r < (int)a.Lq ? r : (int)a.Lq - 1;
    row_q[ln] = (int)(h * a.qsh + rc * a.qst);
    row_out[ln] = r < (int)a.Lq ? (h * (int)a.Lq + r) * (a.topk + 1) + a.topk : -1;
    row_range[ln] = window_of(pos(r));
    row_range[64 + ln] = pos(r);
  }
  // rows of the wavefront: a run of the tile's (all of them where a tile has no more than a wavefront columns)
  const int f = lm.rows > 32 ? wave * 32 & (lm.rows - 1) : 0, n = lm.rows > 32 ? 32 : lm.rows;
  const int any_lo = window_of(pos(r0 + f)), all_lo = window_of(pos(r0 + f + n - 1));
  const int all_last = pos(r0 + f), any_last = r0 + f < (int)a.Lq ? pos(r0 + f + n - 1) : -1;
  const int begin = window_of(pos(r0)), end = pos(r0 + lm.rows - 1) + 1;
  FineTile<D> t;
  t.setup(a.scale_log2e);
  int b = 0;
  FineStage<D, TT>(wave, lt.kv, begin, end).issue(stages, wave);
  t.load_q(a.Q, row_q);
  t.clear();
#pragma unroll 1
  for (int t0 = begin; t0 < end; t0 += TT) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    lds_barrier();
    if (t0 + TT < end) FineStage<D, TT>(wave, lt.kv, t0 + TT, end).issue(stages + 2 * (b ^ 1) * Lds::kStage, wave);
    const bf16_t* const kt = stages + 2 * b * Lds::kStage;
    const int until = t0 + TT < any_last + 1 ? t0 + TT : any_last + 1;
#pragma unroll 1
    for (int at = t0; at < until; at += 32) {
      if (at + 31 < any_lo) continue;
      t.qk(kt + (at - t0) * D);
      t.attend(at, at == begin, at < all_lo || at + 31 > all_last, row_range, kt + Lds::kStage + (at - t0) * D);
    }
    b ^= 1;
  }
  lds_barrier();
  t.write_output(reinterpret_cast<float*>(stages) + wave * 1024, row_out,
                 FlashPartials{a.part_of, a.part_lse, (uint32_t)(a.Hq * (int)a.Lq * (a.topk + 1))});
}

// Windows: regular tiles of 128 or 256 columns with the causal / window mask.
// FUSED = false: writes the window's partial into the row's last slot (a merge kernel follows).
// FUSED = true (joint softmax, topk <= 8): merges the row's routed partials in the epilogue and
// writes the final output, which takes the merge's HBM traffic off the critical path of a
// separate kernel and saves the window partial's round trip.
template <bool FUSED, int CB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, CB == 1 ? 2 : 8))) void span_window_wide_kernel(const FlashArgs a) {
  using Lds = WideLds;
  constexpr int kCols = 32 * CB, kTile = 4 * kCols;
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bf16_t* const ldsK = reinterpret_cast<bf16_t*>(lds);
  int* const row_out = reinterpret_cast<int*>(lds + Lds::kRow) + wave * 512;
  int* const row_q = row_out + 128;
  float* const row_lse = reinterpret_cast<float*>(row_out + 192);
  int* const row_range = row_out + 256;
  const LocalMap lm = local_map(a.Lq, a.A, a.G, kTile);
  const LocalTile lt = local_tile(lm, kTile, a.Hq / a.G, a.G);
  if (!lt.any) return;
  const int kvh = lt.kv;
  const int r0 = lt.tile << lm.shift;
  auto window_of = [&](int64_t i) {
    if (a.window > 0) return i - a.window + 1 > 0 ? (int)(i - a.window + 1) : 0;
    return (int)((uint32_t)i / (uint32_t)a.A) * a.A;  // (positions lie below 2^24)
  };
  {
    const int ln = lane & (kCols - 1), col = wave * kCols + ln;
    const int h = lt.head0 + (col >> lm.shift);
    const int r = r0 + (col & (lm.rows - 1));
    const int rc = r < (int)a.Lq ? r : (int)a.Lq - 1;
    row_q[ln] = (int)(h * a.qsh + rc * a.qst);
    row_out[ln] = r < (int)a.Lq ? (FUSED ? h * (int)a.Lq + r : (h * (int)a.Lq + r) * (a.topk + 1) + a.topk) : -1;
    row_range[ln] = window_of(a.q_pos0 + rc);
    row_range[128 + ln] = (int)(a.q_pos0 + rc);
  }
  // rows of the wavefront: a run of the tile's (all of them where a tile has no more than a wavefront columns)
  const int f = lm.rows > kCols ? wave * kCols & (lm.rows - 1) : 0, n = lm.rows > kCols ? kCols : lm.rows;
  auto pos = [&](int r) { return (int)(a.q_pos0 + (r < (int)a.Lq ? r : (int)a.Lq - 1)); };
  Range cur;
  cur.kv = kvh;
  cur.live = (int)a.Lq - (r0 + f);
  cur.any_lo = window_of(pos(r0 + f));
  cur.all_lo = window_of(pos(r0 + f + n - 1));
  cur.all_last = pos(r0 + f);
  cur.any_last = pos(r0 + f + n - 1);
  cur.begin = window_of(pos(r0)) / TN * TN;
  cur.end = (pos(r0 + lm.rows - 1) / TN + 1) * TN;

  WideTile<CB> t;
  t.setup(a.scale_log2e);
  int b = 0;
  WideStage<true, CB == 2>(wave, kvh, cur.begin).issue(ldsK, wave);
  t.load_q(a.Q, row_q);
  auto arrive = [&](int t0) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    lds_barrier();
    if (t0 + TN < cur.end) WideStage<true, CB == 2>(wave, kvh, t0 + TN).issue(ldsK + 2 * (b ^ 1) * Lds::kStage, wave);
  };
  int t0 = cur.begin;
  arrive(t0);
  t.clear();
  if (CB == 2 && cur.attended<true, 32>(t0) && cur.attended<true, 32>(t0 + 32)) {
    t.template begin<true>(t0, cur, row_range, ldsK + 2 * b * Lds::kStage, [] {});
    b ^= 1;
    t0 += TN;
  }
#pragma unroll 1
  for (; t0 < cur.end; t0 += TN) {
    if (t0 != cur.begin) arrive(t0);
    t.template step<true>(t0, cur, row_range, ldsK + 2 * b * Lds::kStage, [] {});
    b ^= 1;
  }
  lds_barrier();
  // the stages are dead: 64 rows of 256 bytes per wavefront
  bf16_t* const ost = ldsK + wave * CB * 4096;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) t.stage_output(cb, ost + cb * 4096, row_lse);
  if constexpr (!FUSED) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) t.write_output(cb, ost + cb * 4096, row_out, a.part_o);
    if (lane < kCols && row_out[lane] >= 0) a.part_lse[row_out[lane]] = row_lse[lane];
  } else {
    // The merge (topk <= 8): the lane that would store 16 bytes of the window's partial instead loads the same 16 bytes of the
    // row's routed partials (written by the routed kernel, which ran before on the stream), does the log-sum-exp merge and
    // stores the final output.  Every load is issued before the first dependent use; slots that take no part may hold
    // anything and are discarded by selects, never by arithmetic.  Partials are read and outputs written past the caches, which
    // are left to the queries (read by eight spans' tiles) and the keys and values: 8192 rows, 32:4 heads, top-8, spans of 64
    // 386 -> 357 us (routed 201 -> 186, this kernel 148 -> 137), 16384 with 128 800 -> 735, 262144 with 512 24.57 -> 24.48 ms.
    const int topk = a.topk, nslot = topk + 1;
#pragma unroll 1
    for (int ub = 0; ub < kCols; ub += 16) {
      int64_t outs[4];
      int js[4][8];
      float ls[4][8];
      uint4 ov[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = ub + u * 4 + (lane >> 4), piece = lane & 15;
        outs[u] = row_out[row];
        const int64_t rg = outs[u] >= 0 ? outs[u] : 0;
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
          const bool in = sl < topk;
          js[u][sl] = in ? a.idx[rg * topk + sl] : -1;
          ls[u][sl] = in ? a.part_lse[rg * nslot + sl] : 0.f;
          ov[u][sl] = in ? load16_stream(a.part_o + (rg * nslot + sl) * HD + piece * 8) : make_uint4(0, 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = ub + u * 4 + (lane >> 4), piece = lane & 15;
        const int cq = row_range[128 + row] / a.A;
        const float lw = row_lse[row];
        float M = lw;
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
          // a slot takes part if its span is a candidate and no earlier slot lists the same span
          bool ok = js[u][sl] >= 0 && js[u][sl] < cq;
#pragma unroll
          for (int v = 0; v < sl; ++v) ok = ok && js[u][v] != js[u][sl];
          ls[u][sl] = ok ? ls[u][sl] : -INFINITY;
          M = fmaxf(M, ls[u][sl]);
        }
        float acc[8], f[8];
        float wsum = __expf(lw - M);
        Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(&ost[row * HD + ((piece ^ (row & 15)) << 3)]), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = wsum * f[e];
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
          const bool ok = ls[u][sl] > -INFINITY;
          const float w = ok ? __expf(ls[u][sl] - M) : 0.f;
          wsum += w;
          Elem<bf16_t>::unpack(ok ? ov[u][sl] : make_uint4(0, 0, 0, 0), f);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf(w, f[e], acc[e]);
        }
        const float winv = 1.f / wsum;
        uint4 res;
        res.x = (uint32_t)f32_to_bf16(acc[0] * winv) | ((uint32_t)f32_to_bf16(acc[1] * winv) << 16);
        res.y = (uint32_t)f32_to_bf16(acc[2] * winv) | ((uint32_t)f32_to_bf16(acc[3] * winv) << 16);
        res.z = (uint32_t)f32_to_bf16(acc[4] * winv) | ((uint32_t)f32_to_bf16(acc[5] * winv) << 16);
        res.w = (uint32_t)f32_to_bf16(acc[6] * winv) | ((uint32_t)f32_to_bf16(acc[7] * winv) << 16);
        if (outs[u] >= 0) {
          store16_stream(a.O + outs[u] * HD + piece * 8, res);
          if (piece == 0) a.LSE[outs[u]] = M + __logf(wsum);
        }
      }
    }
  }
}

// ------------------------------------------------------------------ merge
// A lane's 16 bytes of a partial: 8 bf16 (P = bf16_t) or 4 fp32 (P = float) columns.
// Past the caches, as in the window kernel: 20011 rows, top-8, spans of 142 1609 -> 1538 us, of 66 1428 -> 1323, in calls that
// follow each other.
template <typename P>
__device__ __forceinline__ void store_columns(bf16_t* p, const float* v) {
  uint32_t w[Elem<P>::EPL / 2];
#pragma unroll
  for (int e = 0; e < Elem<P>::EPL / 2; ++e)
    w[e] = (uint32_t)f32_to_bf16(v[2 * e]) | ((uint32_t)f32_to_bf16(v[2 * e + 1]) << 16);
  if constexpr (Elem<P>::EPL == 8) store16_stream(p, make_uint4(w[0], w[1], w[2], w[3]));
  else __builtin_nontemporal_store((uint64_t)w[1] << 32 | w[0], reinterpret_cast<uint64_t*>(p));
}

// fp32 partials: an output that is not finite marks the call (see rerun_flag).
template <typename P>
__device__ __forceinline__ void mark_not_finite(const float* v, int* flag) {
  if constexpr (Elem<P>::EPL == 4) {
    bool bad = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) bad = bad || !(fabsf(v[e]) < INFINITY);
    if (bad) *flag = 1;
  }
}

// Log-sum-exp merge of a row's partials: up to topk routed slots plus the local window (slot
// topk).  16 bytes per lane, D * sizeof(P) / 16 lanes per row; every load of a lane is issued before the
// first dependent use, so the kernel streams at HBM rate.
template <int KMAX, typename P = bf16_t, int D = HD>
__global__ __launch_bounds__(256) void merge_partials_kernel(
    const int32_t* __restrict__ idx, const P* __restrict__ part_o,
    const float* __restrict__ part_lse, bf16_t* __restrict__ O, float* __restrict__ LSE,
    int64_t rows, int64_t Lq, int64_t q_pos0, int S, int topk, int* __restrict__ flag) {
  constexpr int E = Elem<P>::EPL, LPRW = D / E;
  const int64_t row = (int64_t)blockIdx.x * (256 / LPRW) + threadIdx.x / LPRW;
  const int piece = threadIdx.x % LPRW;
  if (row >= rows) return;
  const int64_t r = row % Lq;
  const int c = (int)((q_pos0 + r) / S);
  const int nslot = topk + 1;
  const int32_t* irow = idx + row * topk;
  const float* lrow = part_lse + row * nslot;
  const P* orow = part_o + row * nslot * D + piece * E;

  int js[KMAX];
  float ls[KMAX + 1];
  uint4 ov[KMAX + 1];
#pragma unroll
  for (int s = 0; s < KMAX; ++s) js[s] = s < topk ? irow[s] : -1;
#pragma unroll
  for (int s = 0; s < KMAX; ++s) {
    // a slot takes part if its span is a candidate and no earlier slot lists the same span
    bool ok = js[s] >= 0 && js[s] < c;
#pragma unroll
    for (int u = 0; u < s; ++u) ok = ok && js[u] != js[s];
    ls[s] = ok ? lrow[s] : -INFINITY;
    ov[s] = ok ? load16_stream(orow + (int64_t)s * D) : make_uint4(0, 0, 0, 0);
  }
  ls[KMAX] = lrow[topk];
  ov[KMAX] = load16_stream(orow + (int64_t)topk * D);

  float M = ls[KMAX];
#pragma unroll
  for (int s = 0; s < KMAX; ++s) M = fmaxf(M, ls[s]);
  float acc[E], f[E];
  float wsum = __expf(ls[KMAX] - M);
  Elem<P>::unpack(ov[KMAX], f);
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = wsum * f[e];
#pragma unroll
  for (int s = 0; s < KMAX; ++s) {
    const float w = ls[s] > -INFINITY ? __expf(ls[s] - M) : 0.f;
    wsum += w;
    Elem<P>::unpack(ov[s], f);
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = fmaf(w, f[e], acc[e]);
  }
  const float winv = 1.f / wsum;
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] *= winv;
  mark_not_finite<P>(acc, flag);
  store_columns<P>(O + row * D + piece * E, acc);
  if (piece == 0) LSE[row] = M + __logf(wsum);
}


// Combination form of the merge (Section 3.4, eq. (5)-(6); Algorithm 1): per valid slot t,
// A_t = log-sum-exp merge of the slot's partial with the local window's partial (the attention
// over span t and the window with its own softmax); O = sum_t alpha_t A_t with alpha = softmax of
// the slots' search scores; no valid slot: the window's partial.
// ANCHOR: the paper's geometry.  idx holds anchor tokens, a slot is valid if its anchor is one of
// the row's (0 <= t <= i); a valid slot whose span minus the window is empty has lse = -inf and
// A_t is then the window's attention alone.
template <int KMAX, bool ANCHOR, typename P = bf16_t, int D = HD>
__global__ __launch_bounds__(256) void merge_combined_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ gate,
    const P* __restrict__ part_o, const float* __restrict__ part_lse, bf16_t* __restrict__ O,
    int64_t rows, int64_t Lq, int64_t q_pos0, int S, int topk, int64_t full_from, int* __restrict__ flag) {
  constexpr int E = Elem<P>::EPL, LPRW = D / E;
  const int64_t row = (int64_t)blockIdx.x * (256 / LPRW) + threadIdx.x / LPRW;
  const int piece = threadIdx.x % LPRW;
  if (row >= rows) return;
  const int64_t r = row % Lq;
  const int64_t limit = ANCHOR ? q_pos0 + r + 1 : (q_pos0 + r) / S;  // valid entries lie in [0, limit)
  const int nslot = topk + 1;
  const int32_t* irow = idx + row * topk;
  const float* grow = gate + row * topk;
  const float* lrow = part_lse + row * nslot;
  const P* orow = part_o + row * nslot * D + piece * E;

  // Rows from full_from on have candidates for all their slots: every load is issued before the first use, whatever
  // the row's list says; what an empty slot's record holds is dropped by selects.  (Asking for a partial only after
  // its lse had come, and for that only after the list entry, took three memory round trips: a gated call of 4000
  // rows x 32 heads x 16 slots 935 -> 890 us.)  Earlier rows ask for the partials of the slots in use, a second round
  // trip: what the empty slots' records hold need not be read (4096 rows x 16 slots, at most 3 in use: 337 -> 292).
  // Lists of up to 32 take their partials eight at a time: with all of them in registers a SIMD holds one wavefront
  // (20000 rows x 32 slots, at most 19 in use: the call 5684 -> 4774; one slot after the other 5429).
  constexpr int BK = KMAX > 16 ? 8 : KMAX;
  const bool full = q_pos0 + r >= full_from;
  int js[KMAX];
  float ls[KMAX], gs[KMAX];
  uint4 ov[BK];
#pragma unroll
  for (int s = 0; s < KMAX; ++s) {
    const bool in = s < topk;
    js[s] = in ? irow[s] : -1;
    ls[s] = in ? lrow[s] : -INFINITY;
    gs[s] = in ? grow[s] : -INFINITY;
    if (s < BK) ov[s] = in && full ? load16_stream(orow + (int64_t)s * D) : make_uint4(0, 0, 0, 0);
  }
  const float lw = lrow[topk];
  const uint4 ow = load16_stream(orow + (int64_t)topk * D);
  float gmax = -INFINITY;
  unsigned okmask = 0u;
#pragma unroll
  for (int s = 0; s < KMAX; ++s) {
    bool ok = js[s] >= 0 && js[s] < limit;
    if (!ANCHOR) {
#pragma unroll
      for (int u = 0; u < s; ++u) ok = ok && js[u] != js[s];
    }
    ls[s] = ok ? ls[s] : -INFINITY;
    gs[s] = ok ? gs[s] : -INFINITY;
    gmax = fmaxf(gmax, gs[s]);
    okmask |= ok ? (1u << s) : 0u;
  }
  float acc[E], fw[E], f[E];
  Elem<P>::unpack(ow, fw);
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;
  float asum = 0.f;
#pragma unroll
  for (int b = 0; b < KMAX; b += BK) {
    if (b > 0 || !full) {
#pragma unroll
      for (int x = 0; x < BK; ++x)
        if (okmask & (1u << (b + x))) ov[x] = load16_stream(orow + (int64_t)(b + x) * D);
    }
#pragma unroll
    for (int x = 0; x < BK; ++x) {
      const int s = b + x;
      if (okmask & (1u << s)) {  // valid slot
        // an empty span has lse = -inf.  (fp32 partials: an lse that is NaN, from a key that is not finite, goes
        // on into the output, which then marks the call.)
        const bool has = sizeof(P) == 4 ? !(ls[s] == -INFINITY) : ls[s] > -INFINITY;
        const float M = fmaxf(ls[s], lw);
        const float wa = has ? __expf(ls[s] - M) : 0.f, wb = __expf(lw - M);
        const float a = __expf(gs[s] - gmax);
        const float fa = a * wa / (wa + wb), fb = a * wb / (wa + wb);
        asum += a;
        Elem<P>::unpack(has ? ov[x] : make_uint4(0, 0, 0, 0), f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = fmaf(fa, f[e], fmaf(fb, fw[e], acc[e]));
      }
    }
  }
  const bool any = asum > 0.f;
  const float inv = any ? 1.f / asum : 1.f;
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = (any ? acc[e] : fw[e]) * inv;
  mark_not_finite<P>(acc, flag);
  store_columns<P>(O + row * D + piece * E, acc);
}

// ------------------------------------------------------------------ workspace carving
struct MfmaWs {
  int tm;  // rows of a tile
  size_t counts, claims, unit_cnt, item_off, tile_off, cursor, tile_info, items, part_lse, part_o, flag, total;
  BucketPlan plan;
  int B, max_tiles;
  int64_t max_items;
};

using One = std::integral_constant<int, 1>;
using Two = std::integral_constant<int, 2>;

// Per-device facts, looked up on the first call with that device current: compute units, and whether the
// flash kernels were granted more dynamic LDS than the 64 KB a kernel gets by default.
struct DeviceSetup {
  int grid = 0;     // compute units, rounded up to a multiple of 8; 0 = not looked up yet
  bool lds_ok = false;
};
constexpr int kMaxDevices = 64;
std::mutex g_setup_mu;
DeviceSetup g_setup[kMaxDevices];

bool device_setup(DeviceSetup* out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::lock_guard<std::mutex> lock(g_setup_mu);
  DeviceSetup& d = g_setup[dev];
  if (d.grid == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    auto allow = [](auto kernel) {
      return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, WideLds::kBytes) ==
             hipSuccess;
    };
    auto allow_both = [&](auto columns) {
      constexpr int CB = decltype(columns)::value;
      return allow(span_flash_wide_kernel<Spans::kWhole, CB>) && allow(span_flash_wide_kernel<Spans::kClipped, CB>) &&
             allow(span_flash_wide_kernel<Spans::kAnchor, CB>) && allow(span_window_wide_kernel<false, CB>) &&
             allow(span_window_wide_kernel<true, CB>);
    };
    d.lds_ok = allow_both(One{}) && allow_both(Two{});
    d.grid = (cus + 7) / 8 * 8;
  }
  *out = d;
  return true;
}

// Rows per bucketing unit: 64, doubled (to 1024) while that leaves 4096 units, four wavefronts on each
// of 1024 SIMDs, or while the unit holds fewer items than it has counters to clear, write and scan.
BucketPlan bucket_plan(const Problem& pb) {
  BucketPlan p;
  p.rows = 64;
  while (p.rows < 1024 && ((pb.Lq + 2 * p.rows - 1) / (2 * p.rows) * pb.Hq >= 4096 || (int64_t)p.rows * pb.topk < pb.n))
    p.rows <<= 1;
  p.units = (int)((pb.Lq + p.rows - 1) / p.rows);
  p.unit_h = p.units;
  p.unit_u = 1;
  return p;
}

// Slots of its list that a row has candidates for, on average: the row at position i has i / A.
double grid_slots(const Problem& pb) {
  const double full = (double)pb.topk * pb.A;
  auto before = [&](double i) { return i < full ? 0.5 * i * i / pb.A : pb.topk * (i - 0.5 * full); };
  return (before((double)(pb.q_pos0 + pb.Lq)) - before((double)pb.q_pos0)) / pb.Lq;
}

// Columns of a wavefront of the kernels with bf16 weights, in blocks of 32.  With two a fragment of K or V feeds two products,
// and the long prompt's routed kernel runs at 1050 to 1150 TFLOP/s where one reaches 970 to 1040; but a tile that is mostly
// empty, or that alone keeps the call waiting, takes twice the time.  460 random calls (1 to 64 heads, 1 to 150000 rows, grid
// and paper's geometry, two -> one): from 1024 tiles of 256 rows and 500 items a bucket on 0.86 to 1.10, geometric mean 0.97;
// below 256 tiles 1.0 to 1.6, mean 1.15.  With these two numbers the calls are within 0.3 % of the faster form each (0.7 % with
// one block throughout, 0.8 % with two from 512 tiles on, whatever the buckets hold).  `slots` of its list are in use by a row, on the
// grid those it has candidates for: with lists of 8 taken as full 850 rows of 64:8 heads behind 655, anchors every 1024, took 126 us and not 102.
int routed_blocks(const Problem& pb, double slots) {
  const double spans = fmin((double)pb.n, fmax(1, (double)((pb.q_pos0 + pb.Lq) / pb.A)));
  const double items = (double)pb.Hq * pb.Lq * slots, buckets = fmin(items, pb.Hkv * spans);
  return items >= 500 * buckets && items / 256 + 0.5 * buckets >= 1024 ? 2 : 1;
}
// Windows (tokens: how many a row's has on average) by workgroups of 256 rows: where they are not two a compute unit, one block is
// faster (up to 32 two -> one 1.17, up to 256 1.05); from there on two win where windows are long: 384000 rows and windows of
// 1088 tokens 692 us the call with one block, 634 with two, 1.6 million 3.15 ms, 3.04; 8.4 million, spans of 512, with the
// merge 5.0 ms, 4.8.  Up to 2048 workgroups of half spans of 512 tokens and less 1.00 to 1.02.
int window_blocks(const Problem& pb, double tokens) {
  const double rows = (double)pb.Hq * pb.Lq;
  return rows >= 512 * 256 && rows * tokens >= 2048.0 * 256 * 256 ? 2 : 1;
}

MfmaWs carve(const Problem& pb, int tm, size_t part_elem = sizeof(bf16_t)) {
  MfmaWs w;
  w.tm = tm;
  w.B = pb.Hkv * (int)pb.n;
  w.max_items = (int64_t)pb.Hq * pb.Lq * pb.topk;
  w.max_tiles = (int)((w.max_items + tm - 1) / tm) + w.B;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes, 256);
    return at;
  };
  w.counts = take((size_t)w.B * sizeof(int));
  w.claims = take(8 * 32 * sizeof(int));
  w.plan = bucket_plan(pb);
  w.unit_cnt = take((size_t)pb.Hq * w.plan.units * pb.n * sizeof(int));
  w.item_off = take((size_t)(w.B + 1) * sizeof(int));
  w.tile_off = take((size_t)(w.B + 1) * sizeof(int));
  w.cursor = take((size_t)w.B * sizeof(int));
  w.tile_info = take((size_t)w.max_tiles * sizeof(int4));
  w.items = take((size_t)w.max_tiles * tm * sizeof(int));  // tile by tile, tm entries each
  const size_t nparts = (size_t)pb.Hq * pb.Lq * (pb.topk + 1);  // routed slots + the local window
  w.part_lse = take(nparts * sizeof(float));
  w.part_o = take(nparts * pb.D * part_elem);
  w.flag = take(256);
  w.total = off;
  return w;
}

// The bucketing passes.  Blocks hold as many units as their histograms fit into 64 KB of LDS (n <= 4096).
template <typename Items>
bool launch_buckets(const Problem& pb, const MfmaWs& w, const int32_t* idx, int* unit_cnt, int* counts,
                    int* item_off, int* tile_off, int* cursor, int4* tile_info, int* items, float* part_lse,
                    const Items& it, int* flag, int* claims, hipStream_t st) {
  const int n = (int)pb.n;
  const int per_block = 4;  // 4 * 4096 counters = 64 KB
  const dim3 grid((unsigned)((w.plan.units + per_block - 1) / per_block), pb.Hq);
  const size_t lds = (size_t)per_block * n * sizeof(int);
  hipLaunchKernelGGL((bucket_kernel<false, Items>), grid, dim3(64 * per_block), lds, st, idx, unit_cnt, cursor,
                     items, part_lse, pb.Lq, pb.q_pos0, pb.G, pb.topk, n, w.plan, it);
  hipLaunchKernelGGL(bucket_unit_scan_kernel, dim3((n + 31) / 32, pb.Hkv), dim3(1024), 0, st, unit_cnt, counts,
                     pb.G * w.plan.units, n);
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(1024), 0, st, counts, item_off, tile_off, cursor, w.B,
                     w.tm, flag, claims);
  hipLaunchKernelGGL(bucket_tiles_kernel, dim3(w.B), dim3(256), 0, st, tile_off, item_off, tile_info, items, w.tm);
  hipLaunchKernelGGL((bucket_kernel<true, Items>), grid, dim3(64 * per_block), lds, st, idx, unit_cnt, cursor,
                     items, part_lse, pb.Lq, pb.q_pos0, pb.G, pb.topk, n, w.plan, it);
  return hipGetLastError() == hipSuccess;
}

}  // namespace

// Longer sequences stay with the row-stationary kernels, whose softmax weights are fp32.
constexpr int64_t kMaxTokens = ((int64_t)1 << 24) - 64;

bool prefill_attention_mfma_supported(const Problem& pb) {
  return pb.dtype == SL_BF16 && pb.D == HD && pb.S % TN == 0 && pb.A % TN == 0 && pb.n <= 4096 &&
         (int64_t)pb.G * pb.Lq < ((int64_t)1 << 26) &&  // item = (row id << 5) | slot
         pb.L <= kMaxTokens &&
         // staging uses 32-bit byte offsets inside a 64-row tile
         64 * pb.kvst * 2 < ((int64_t)1 << 31) &&
         (int64_t)pb.Hq * pb.Lq * (pb.topk + 1) < ((int64_t)1 << 31) &&
         // 32-bit positions in the tile-by-tile item list
         (int64_t)pb.Hq * pb.Lq * pb.topk + ((int64_t)pb.Hkv * pb.n + 1) * TM < ((int64_t)1 << 31) &&
         // row_q holds 32-bit element offsets into Q
         (int64_t)pb.Hq * pb.qsh + pb.Lq * pb.qst < ((int64_t)1 << 31);
}

// Enough for either form, so that it does not depend on where the rows stand.
size_t prefill_attention_mfma_ws_bytes(const Problem& pb) {
  const size_t one = carve(pb, 128).total, two = carve(pb, 256).total;
  return one > two ? one : two;
}

sl_status prefill_attention_mfma(const Problem& pb, const void* Q, const void* K, const void* V,
                                 const int32_t* idx, void* O, float* LSE, void* ws,
                                 hipStream_t st) {
  const int blocks = routed_blocks(pb, grid_slots(pb));
  const MfmaWs w = carve(pb, 128 * blocks);
  DeviceSetup dev;
  if (!device_setup(&dev) || !dev.lds_ok) return SL_ERR_LAUNCH;
  char* base = static_cast<char*>(ws);
  int* counts = reinterpret_cast<int*>(base + w.counts);
  int* unit_cnt = reinterpret_cast<int*>(base + w.unit_cnt);
  int* item_off = reinterpret_cast<int*>(base + w.item_off);
  int* tile_off = reinterpret_cast<int*>(base + w.tile_off);
  int* cursor = reinterpret_cast<int*>(base + w.cursor);
  int4* tile_info = reinterpret_cast<int4*>(base + w.tile_info);
  int* items = reinterpret_cast<int*>(base + w.items);
  float* part_lse = reinterpret_cast<float*>(base + w.part_lse);
  bf16_t* part_o = reinterpret_cast<bf16_t*>(base + w.part_o);
  const int n = (int)pb.n;

  FlashArgs a;
  a.Q = static_cast<const bf16_t*>(Q);
  a.K = static_cast<const bf16_t*>(K);
  a.V = static_cast<const bf16_t*>(V);
  a.idx = idx;
  a.tile_off = tile_off;
  a.tile_info = tile_info;
  a.items = items;
  a.claims = reinterpret_cast<int*>(base + w.claims);
  a.part_o = part_o;
  a.part_of = nullptr;
  a.part_lse = part_lse;
  a.O = static_cast<bf16_t*>(O);
  a.LSE = LSE;
  a.L = pb.L;
  a.Lq = pb.Lq;
  a.q_pos0 = pb.q_pos0;
  a.Hq = pb.Hq;
  a.G = pb.G;
  a.S = pb.S;
  a.A = pb.A;
  a.window = 0;
  a.ab = a.af = 0;
  a.aroot = 2;
  a.clip = 0;
  a.topk = pb.topk;
  a.n = n;
  a.scale_log2e = pb.scale * kLog2e;
  a.qsh = pb.qsh;
  a.qst = pb.qst;
  a.kvsh = pb.kvsh;
  a.kvst = pb.kvst;

  if (pb.topk > 0) {
    if (!launch_buckets(pb, w, idx, unit_cnt, counts, item_off, tile_off, cursor, tile_info, items, part_lse,
                        GridItems{pb.A}, nullptr, a.claims, st))
      return SL_ERR_LAUNCH;
    if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
    auto routed = [&](auto columns) {
      constexpr int CB = decltype(columns)::value;
      const dim3 grid(2 * dev.grid), block(256);
      if (pb.A < pb.S && !pb.combined)  // overlapping spans in one joint softmax: per-row clipping
        hipLaunchKernelGGL((span_flash_wide_kernel<Spans::kClipped, CB>), grid, block, WideLds::kBytes, st, a);
      else
        hipLaunchKernelGGL((span_flash_wide_kernel<Spans::kWhole, CB>), grid, block, WideLds::kBytes, st, a);
    };
    if (blocks == 1) routed(One{});
    else routed(Two{});
    if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  }
  const bool fused = !pb.combined && pb.topk <= 8;  // the window kernel merges and writes the final output
  auto window = [&](auto columns) {
    constexpr int CB = decltype(columns)::value;
    const dim3 grid(local_grid(pb.Lq, pb.A, pb.Hkv, pb.G, 128 * CB)), block(256);
    if (fused) hipLaunchKernelGGL((span_window_wide_kernel<true, CB>), grid, block, WideLds::kBytes, st, a);
    else hipLaunchKernelGGL((span_window_wide_kernel<false, CB>), grid, block, WideLds::kBytes, st, a);
  };
  if (window_blocks(pb, 0.5 * pb.A) == 1) window(One{});
  else window(Two{});
  if (fused) return hipGetLastError() == hipSuccess ? SL_OK : SL_ERR_LAUNCH;
  const int64_t rows = (int64_t)pb.Hq * pb.Lq;
  const dim3 mgrid((unsigned)((rows + 15) / 16));
#define SL_MERGE(KM)                                                                             \
  do {                                                                                           \
    if (pb.combined)                                                                                 \
      hipLaunchKernelGGL((merge_combined_kernel<KM, false>), mgrid, dim3(256), 0, st, idx, pb.gate, \
                         part_o, part_lse, a.O, rows, pb.Lq, pb.q_pos0, pb.A, pb.topk, (int64_t)pb.topk * pb.A,      \
                         static_cast<int*>(nullptr));                                              \
    else                                                                                         \
      hipLaunchKernelGGL(merge_partials_kernel<KM>, mgrid, dim3(256), 0, st, idx, part_o,        \
                         part_lse, a.O, LSE, rows, pb.Lq, pb.q_pos0, pb.A, pb.topk, static_cast<int*>(nullptr));             \
  } while (0)
  if (pb.topk == 0) SL_MERGE(1);
  else if (pb.topk <= 8) SL_MERGE(8);
  else if (pb.topk <= 16) SL_MERGE(16);
  else SL_MERGE(32);
#undef SL_MERGE
  return hipGetLastError() == hipSuccess ? SL_OK : SL_ERR_LAUNCH;
}

// ------------------------------------------------------------------ any span length, fp32 weights
// bf16 inputs that the kernels above do not take -- spans that are no multiple of 64 tokens, D = 64 -- on
// the matrix cores without giving up the row-stationary kernels' precision: every product of the weights
// with V is taken three times, with the weight's leading bf16 part, with that of what it leaves, and with the rest;
// partials are fp32.  Error against 64 bits: the row-stationary kernels' to all seven digits looked at (1.641783e-3
// of a bf16 output of 20011 rows, nearly all of it the rounding of the output; with two parts, 16 to 17 bits,
// 1.641784e-3 at 7 to 10 % less time; with bf16 weights and partials 2.4e-3).
//
// Measured (32:4 heads, top-8, D = 128 unless said otherwise; row-stationary -> this form, us):
//   20011 rows, spans of 142: 16400 -> 1605; at D = 64: 8320 -> 860; 2500 rows, spans of 50: 791 -> 172;
//   200 rows behind 60000 tokens, spans of 245: 589 -> 82; 8 rows there: 157 -> 60.
// Calls without a workspace, or with one too small, take the row-stationary kernels as before.
namespace {

// Tiles that the routed part has at most: one that is not full for every span with a row, and the full ones.
double fine_tiles(const Problem& pb) {
  const double items = (double)pb.Hq * pb.Lq * pb.topk;
  return fmin(items, (double)pb.Hkv * pb.n) + items / TG;
}

// Estimated us of the two forms in calls that follow each other; the call takes the smaller.
//
// Row-stationary, 16 keys (D = 64: 32) at a time: one row's chain of loads, 0.5 us each and up to 2.5 times that where the keys and
// values that the rows touch leave the L2, and what all rows take, by key and by slot in use; neither hides behind the other entirely.
// Spans that overlap are looked up in the whole list each, to be clipped, and cover no more than the cache.  (One rule for both
// softmaxes: the scratch is asked for without saying which.)
// This form: nine launches, some of them over all buckets; routed tiles of 6.3 us and a step cost, on as many workgroups as are resident;
// windows; partials written and read.
//
// 60667 random calls (1 to 20000 rows of 1 to 64 heads behind up to 200000 tokens, spans of 4 to 900, lists of 1 to 32, one in five
// with overlapping spans, both D, both softmaxes), 40000 of them fitted: of the others the estimates choose the slower form in 3.2 %,
// which costs 0.4 % over all calls, and more than 30 % in 0.3 %.  (With one figure a key for the chain, wherever the keys lie, and
// nothing for looking through lists 6.8, 1.8 and 2.7 %, calls of 50 to 150 us at twice their time among them.)
bool fine_is_faster(const Problem& pb) {
  const double end = (double)(pb.q_pos0 + pb.Lq), rows = (double)pb.Hq * pb.Lq, window = 0.5 * fmin(pb.A, end);
  const double slots = grid_slots(pb), items = rows * slots, most = fmin(pb.topk, floor(end / pb.A));
  const bool half = pb.D == 64, overlap = pb.A < pb.S;
  const double span = overlap ? fmin(pb.S, fmax(pb.A, end / fmax(1, most))) : pb.S;
  const double touched = fmin(pb.Hkv * end, items * span + rows * window) * pb.D * 4, far = touched / (touched + 23e6);
  const double at_once = half ? 32 : 16, look = overlap ? pb.topk : 0;
  const double chain = 0.5 * (1 + 1.5 * far) * (most * ceil(span / at_once) + ceil(window / at_once)) + most * (0.07 + 0.063 * look);
  const double key = (half ? 7.9e-6 : 15.5e-6) * (1 + 1.36 * far);
  const double all = rows * (key * (slots * span + window) + slots * (3.1e-4 + 1.3e-5 * look) + 4.7e-4);
  const double by_rows = 9 + pow(pow(chain, 1.5) + pow(all, 1.5), 2.0 / 3);
  const double workgroups = half ? 1024 : 768, step = half ? 0.9 : 1.4;
  const double tiles = fmin(items, (double)pb.Hkv * pb.n) + items / TG;
  const double routed = (6.3 + step * ((pb.S + 31) / 32)) * fmax(1, tiles / workgroups);
  const double windows = rows / TG / workgroups * (15 + step * (window / 32 + 1));
  return 29 + 0.002 * pb.Hkv * pb.n + routed + windows + (items + rows) * pb.D * 8 / 7.5e6 < by_rows;
}

constexpr size_t kFineMaxScratch = (size_t)4 << 30;

Problem fine_part(const Problem& pb, int kv_heads) {  // the first kv_heads kv heads and their query heads
  Problem q = pb;
  q.Hkv = kv_heads;
  q.Hq = kv_heads * pb.G;
  return q;
}

size_t fine_bytes(const Problem& pb) {
  return carve(pb, TG, sizeof(float)).total;
}

// kv heads per pass: as many as fit the scratch limit
int fine_heads(const Problem& pb) {
  int h = pb.Hkv;
  while (h > 1 && fine_bytes(fine_part(pb, h)) > kFineMaxScratch) --h;
  return h;
}

// Stages of twice the tokens, two workgroups per compute unit: where these take all tiles at once, a call lasts as long as one
// tile's chain of stages.  D = 128, us: 57 tiles, spans of 838 79 -> 73, 54 of 525 74 -> 71, 117 of 191 56 -> 54, 488 of 867
// 151 -> 148; 667 of 864 152 -> 166, more up to 13 % slower.  At D = 64 a stage holds 64 tokens as it is, and 128 were never faster.
bool long_stages(const Problem& pb, const DeviceSetup& dev, double tiles) { return pb.D == 128 && tiles <= 2 * dev.grid; }

template <int D>
bool fine_setup(DeviceSetup* out) {
  static std::mutex mu;
  static bool done[kMaxDevices];
  int dev = -1;
  if (!device_setup(out) || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::lock_guard<std::mutex> lock(mu);
  auto allow = [](auto routed, auto window, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(routed), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(window), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
  };
  constexpr int kShort = 4096 / D, kLong = 64;  // tokens of a stage; D = 64 has one length
  if (!done[dev])
    done[dev] = allow(span_fine_kernel<D, kShort>, span_fine_window_kernel<D, kShort>, FineLds<D, kShort>::kBytes) &&
                allow(span_fine_kernel<D, kLong>, span_fine_window_kernel<D, kLong>, FineLds<D, kLong>::kBytes);
  return done[dev];
}

template <int D>
sl_status fine_pass(const Problem& pb, const DeviceSetup& dev, const bf16_t* Q, const bf16_t* K, const bf16_t* V,
                    const int32_t* idx, bf16_t* O, float* LSE, char* base, hipStream_t st) {
  const MfmaWs w = carve(pb, TG, sizeof(float));
  int* item_off = reinterpret_cast<int*>(base + w.item_off);
  int* tile_off = reinterpret_cast<int*>(base + w.tile_off);
  int4* tile_info = reinterpret_cast<int4*>(base + w.tile_info);
  int* items = reinterpret_cast<int*>(base + w.items);
  float* part_lse = reinterpret_cast<float*>(base + w.part_lse);
  float* part_o = reinterpret_cast<float*>(base + w.part_o);
  int* flag = reinterpret_cast<int*>(base + w.flag);
  FlashArgs a = {};
  a.Q = Q;
  a.K = K;
  a.V = V;
  a.idx = idx;
  a.tile_off = tile_off;
  a.tile_info = tile_info;
  a.items = items;
  a.claims = reinterpret_cast<int*>(base + w.claims);
  a.part_of = part_o;
  a.part_lse = part_lse;
  a.O = O;
  a.LSE = LSE;
  a.L = pb.L;
  a.Lq = pb.Lq;
  a.q_pos0 = pb.q_pos0;
  a.Hq = pb.Hq;
  a.G = pb.G;
  a.S = pb.S;
  a.A = pb.A;
  a.clip = pb.A < pb.S && !pb.combined;
  a.aroot = 2;
  a.topk = pb.topk;
  a.n = (int)pb.n;
  a.scale_log2e = pb.scale * kLog2e;
  a.qsh = pb.qsh;
  a.qst = pb.qst;
  a.kvsh = pb.kvsh;
  a.kvst = pb.kvst;
  if (!launch_buckets(pb, w, idx, reinterpret_cast<int*>(base + w.unit_cnt), reinterpret_cast<int*>(base + w.counts),
                      item_off, tile_off, reinterpret_cast<int*>(base + w.cursor), tile_info, items, part_lse,
                      GridItems{pb.A}, flag, a.claims, st))
    return SL_ERR_LAUNCH;
  if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
  const unsigned lgrid = local_grid(pb.Lq, pb.A, pb.Hkv, pb.G, TG);
  constexpr int kShort = 4096 / D, kLong = 64;  // tokens of a stage; D = 64 has one length
  auto launch = [&](void (*kernel)(FlashArgs), unsigned grid, int bytes) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), bytes, st, a);
  };
  if (long_stages(pb, dev, fine_tiles(pb))) launch(span_fine_kernel<D, kLong>, fine_blocks(D, kLong) * dev.grid, FineLds<D, kLong>::kBytes);
  else launch(span_fine_kernel<D, kShort>, fine_blocks(D, kShort) * dev.grid, FineLds<D, kShort>::kBytes);
  if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  if (long_stages(pb, dev, lgrid)) launch(span_fine_window_kernel<D, kLong>, lgrid, FineLds<D, kLong>::kBytes);
  else launch(span_fine_window_kernel<D, kShort>, lgrid, FineLds<D, kShort>::kBytes);
  const int64_t rows = (int64_t)pb.Hq * pb.Lq;
  constexpr int kRowsPerBlock = 256 / (D / 4);
  const dim3 mgrid((unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock));
#define SL_MERGE(KM)                                                                                       \
  do {                                                                                                     \
    if (pb.combined)                                                                                       \
      hipLaunchKernelGGL((merge_combined_kernel<KM, false, float, D>), mgrid, dim3(256), 0, st, idx, pb.gate, \
                         part_o, part_lse, O, rows, pb.Lq, pb.q_pos0, pb.A, pb.topk, (int64_t)pb.topk * pb.A, flag); \
    else                                                                                                   \
      hipLaunchKernelGGL((merge_partials_kernel<KM, float, D>), mgrid, dim3(256), 0, st, idx, part_o,      \
                         part_lse, O, LSE, rows, pb.Lq, pb.q_pos0, pb.A, pb.topk, flag);                   \
  } while (0)
  if (pb.topk <= 8) SL_MERGE(8);
  else if (pb.topk <= 16) SL_MERGE(16);
  else SL_MERGE(32);
#undef SL_MERGE
  if (hipGetLastError() != hipSuccess) return SL_ERR_LAUNCH;
  // A V row that is not finite meets zero weights of rows that do not attend it (the later rows of a window
  // tile, the rows of clipped spans): where any output is not finite the row-stationary kernels, which
  // never touch such a row, compute the pass again.
  Problem again = pb;
  again.prof_start = again.prof_stop = nullptr;  // (the events hold the routed kernel)
  return prefill_attention_rows(again, Q, K, V, idx, O, LSE, st, flag);
}

template <int D>
sl_status fine_all(const Problem& pb, const void* Q, const void* K, const void* V, const int32_t* idx, void* O,
                   float* LSE, void* ws, hipStream_t st) {
  DeviceSetup dev;
  if (!fine_setup<D>(&dev)) return SL_ERR_LAUNCH;
  const int step = fine_heads(pb);
  for (int kv = 0; kv < pb.Hkv; kv += step) {
    Problem q = fine_part(pb, pb.Hkv - kv < step ? pb.Hkv - kv : step);
    if (kv > 0) q.prof_start = nullptr;
    if (kv + step < pb.Hkv) q.prof_stop = nullptr;
    const int64_t h = (int64_t)kv * pb.G, row = h * pb.Lq;
    if (pb.gate) q.gate = pb.gate + row * pb.topk;
    const sl_status s = fine_pass<D>(q, dev, static_cast<const bf16_t*>(Q) + h * pb.qsh,
                                     static_cast<const bf16_t*>(K) + kv * pb.kvsh,
                                     static_cast<const bf16_t*>(V) + kv * pb.kvsh, idx + row * pb.topk,
                                     static_cast<bf16_t*>(O) + row * D, LSE ? LSE + row : nullptr,
                                     static_cast<char*>(ws), st);
    if (s != SL_OK) return s;
  }
  return SL_OK;
}

}  // namespace

bool prefill_attention_fine_supported(const Problem& pb) {
  if (pb.dtype != SL_BF16 || prefill_attention_mfma_supported(pb) || pb.topk < 1 || pb.n > 4096) return false;
  const int64_t rows = (int64_t)pb.Hq * pb.Lq;
  return fine_is_faster(pb) && (int64_t)pb.G * pb.Lq < ((int64_t)1 << 26) && pb.L <= kMaxTokens && 64 * pb.kvst * 2 < ((int64_t)1 << 31) &&
         rows * (pb.topk + 1) < ((int64_t)1 << 31) &&
         rows * pb.topk + ((int64_t)pb.Hkv * pb.n + 1) * TM < ((int64_t)1 << 31) &&
         pb.Hq * pb.qsh + pb.Lq * pb.qst < ((int64_t)1 << 31) &&
         fine_bytes(fine_part(pb, 1)) <= kFineMaxScratch;
}

size_t prefill_attention_fine_ws_bytes(const Problem& pb) { return fine_bytes(fine_part(pb, fine_heads(pb))); }

sl_status prefill_attention_fine(const Problem& pb, const void* Q, const void* K, const void* V, const int32_t* idx,
                                 void* O, float* LSE, void* ws, hipStream_t st) {
  return pb.D == 64 ? fine_all<64>(pb, Q, K, V, idx, O, LSE, ws, st)
                    : fine_all<128>(pb, Q, K, V, idx, O, LSE, ws, st);
}

// ------------------------------------------------------------------ the paper's geometry on the matrix cores
namespace {

Problem anchor_view(const Problem& pb, int E) {
  Problem q = pb;
  q.A = E;
  q.n = (pb.L + q.A - 1) / q.A;
  return q;
}

// 4096 blocks per kv head (their histograms), 32-bit positions in the tile-by-tile item list.
bool anchor_blocks_fit(const Problem& pb, int E) {
  const int64_t n = (pb.L + E - 1) / E;
  return n <= 4096 && (int64_t)pb.Hq * pb.Lq * pb.topk + ((int64_t)pb.Hkv * n + 1) * TM < ((int64_t)1 << 31);
}

// End-block size E of the buckets, a power-of-two multiple of 64 tokens, at most 4096 blocks per kv head.  A tile walks E
// tokens and the length of a span; smaller blocks leave more tiles that are not full.  With x items per token and kv head the
// tokens walked are (x E / rows + 1/2) (E + span) for every E of them, least at E^2 = rows * span / 2x.  Where that leaves
// compute units without a tile the call lasts as long as its longest tile, so blocks are halved while there are fewer.
int anchor_block_tokens(const Problem& pb, double span, int tile_rows) {
  const double x = (double)pb.G * pb.Lq * pb.topk / pb.L, best = sqrt(0.5 * tile_rows * span / x);
  int64_t E = 64;
  while (E < 4096 && E * 1.4142 < best) E <<= 1;
  while (E > 64 && pb.Hkv * (pb.L / (double)E + x * pb.L / tile_rows) < 256) E >>= 1;
  while (!anchor_blocks_fit(pb, (int)E)) E <<= 1;
  return (int)E;
}

}  // namespace

bool prefill_anchor_mfma_supported(const Problem& pb, int64_t window) {
  return window >= 1 && pb.topk >= 1 && pb.dtype == SL_BF16 && pb.D == HD && anchor_blocks_fit(pb, 4096) &&
         (int64_t)pb.G * pb.Lq < ((int64_t)1 << 26) &&
         pb.L <= kMaxTokens &&
         64 * pb.kvst * 2 < ((int64_t)1 << 31) &&
         (int64_t)pb.Hq * pb.Lq * (pb.topk + 1) < ((int64_t)1 << 31) &&
         (int64_t)pb.Hq * pb.qsh + pb.Lq * pb.qst < ((int64_t)1 << 31);
}

// Enough for every block size, so that it does not depend on the spans' length.
size_t prefill_anchor_mfma_ws_bytes(const Problem& pb) {
  size_t most = 0;
  for (int E = 64; E <= 4096; E <<= 1)
    if (anchor_blocks_fit(pb, E)) {
      const Problem q = anchor_view(pb, E);
      for (int blocks = 1; blocks <= 2; ++blocks) {
        const size_t bytes = carve(q, 128 * blocks).total;
        most = bytes > most ? bytes : most;
      }
    }
  return most;
}

// Span-attention and combination on the paper's geometry (Section 3.3-3.4, Algorithm 1), matrix-core
// form following Section 4.3's bucketing by key-block footprint: (row, slot) pairs are bucketed by
// the block that holds their span's last token, a bucket's rows share one sliding K/V range with
// per-row masks, the sliding window is a banded flash kernel, and the gated merge combines them.
sl_status prefill_anchor_attention_mfma(const Problem& pb, int64_t window, int b, int f, int root,
                                        const void* Q, const void* K, const void* V,
                                        const int32_t* anchors, void* O, void* ws, hipStream_t st) {
  const int64_t mid = pb.q_pos0 + pb.Lq / 2, reach = (int64_t)(b + f) * span_base_length(mid, root);
  const double span = (double)(reach < mid ? reach : mid) + 1;
  Problem q = anchor_view(pb, anchor_block_tokens(pb, span, 256));
  const int blocks = routed_blocks(q, q.topk);
  if (blocks == 1) q = anchor_view(pb, anchor_block_tokens(pb, span, 128));
  const MfmaWs w = carve(q, 128 * blocks);
  DeviceSetup dev;
  if (!device_setup(&dev) || !dev.lds_ok) return SL_ERR_LAUNCH;
  char* base = static_cast<char*>(ws);
  int* counts = reinterpret_cast<int*>(base + w.counts);
  int* unit_cnt = reinterpret_cast<int*>(base + w.unit_cnt);
  int* item_off = reinterpret_cast<int*>(base + w.item_off);
  int* tile_off = reinterpret_cast<int*>(base + w.tile_off);
  int* cursor = reinterpret_cast<int*>(base + w.cursor);
  int4* tile_info = reinterpret_cast<int4*>(base + w.tile_info);
  int* items = reinterpret_cast<int*>(base + w.items);
  float* part_lse = reinterpret_cast<float*>(base + w.part_lse);
  bf16_t* part_o = reinterpret_cast<bf16_t*>(base + w.part_o);
  const int n = (int)q.n;

  FlashArgs a;
  a.Q = static_cast<const bf16_t*>(Q);
  a.K = static_cast<const bf16_t*>(K);
  a.V = static_cast<const bf16_t*>(V);
  a.idx = anchors;
  a.tile_off = tile_off;
  a.tile_info = tile_info;
  a.items = items;
  a.claims = reinterpret_cast<int*>(base + w.claims);
  a.part_o = part_o;
  a.part_of = nullptr;
  a.part_lse = part_lse;
  a.O = static_cast<bf16_t*>(O);
  a.LSE = nullptr;
  a.L = pb.L;
  a.Lq = pb.Lq;
  a.q_pos0 = pb.q_pos0;
  a.Hq = pb.Hq;
  a.G = pb.G;
  a.S = 1024;  // only groups the window kernel's row tiles per XCD
  a.A = 1024;
  a.topk = pb.topk;
  a.n = n;
  a.window = window;
  a.ab = b;
  a.af = f;
  a.aroot = root;
  a.clip = 0;
  a.scale_log2e = pb.scale * kLog2e;
  a.qsh = pb.qsh;
  a.qst = pb.qst;
  a.kvsh = pb.kvsh;
  a.kvst = pb.kvst;

  MfmaWs wa = w;
  wa.plan.unit_h = 1;  // items of a bucket by row, then by head
  wa.plan.unit_u = pb.G;
  if (!launch_buckets(q, wa, anchors, unit_cnt, counts, item_off, tile_off, cursor, tile_info, items, part_lse,
                      AnchorItems{window, b, f, root, q.A}, nullptr, a.claims, st))
    return SL_ERR_LAUNCH;
  if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
  if (blocks == 1)
    hipLaunchKernelGGL((span_flash_wide_kernel<Spans::kAnchor, 1>), dim3(2 * dev.grid), dim3(256), WideLds::kBytes, st, a);
  else
    hipLaunchKernelGGL((span_flash_wide_kernel<Spans::kAnchor, 2>), dim3(2 * dev.grid), dim3(256), WideLds::kBytes, st, a);
  if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  if (window_blocks(pb, (double)(window < pb.L ? window : pb.L)) == 1)
    hipLaunchKernelGGL((span_window_wide_kernel<false, 1>), dim3(local_grid(pb.Lq, a.A, pb.Hkv, pb.G, 128)), dim3(256), WideLds::kBytes, st, a);
  else
    hipLaunchKernelGGL((span_window_wide_kernel<false, 2>), dim3(local_grid(pb.Lq, a.A, pb.Hkv, pb.G, 256)), dim3(256), WideLds::kBytes, st, a);
  const int64_t rows = (int64_t)pb.Hq * pb.Lq;
  const dim3 mgrid((unsigned)((rows + 15) / 16));
  // the first position with topk anchors outside the window: stride indices floor(window^(1/root)) and up
  const int64_t full_from = ipow_root(iroot_floor(window, root) + pb.topk, root) - 1;
  if (pb.topk <= 8)
    hipLaunchKernelGGL((merge_combined_kernel<8, true>), mgrid, dim3(256), 0, st, anchors, pb.gate, part_o,
                       part_lse, a.O, rows, pb.Lq, pb.q_pos0, 1, pb.topk, full_from, static_cast<int*>(nullptr));
  else if (pb.topk <= 16)
    hipLaunchKernelGGL((merge_combined_kernel<16, true>), mgrid, dim3(256), 0, st, anchors, pb.gate, part_o,
                       part_lse, a.O, rows, pb.Lq, pb.q_pos0, 1, pb.topk, full_from, static_cast<int*>(nullptr));
  else
    hipLaunchKernelGGL((merge_combined_kernel<32, true>), mgrid, dim3(256), 0, st, anchors, pb.gate, part_o,
                       part_lse, a.O, rows, pb.Lq, pb.q_pos0, 1, pb.topk, full_from, static_cast<int*>(nullptr));
  return hipGetLastError() == hipSuccess ? SL_OK : SL_ERR_LAUNCH;
}

}  // namespace sl
