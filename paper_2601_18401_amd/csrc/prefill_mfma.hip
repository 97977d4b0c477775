// Prefill span-attention on the matrix cores (bf16, D = 128, S a multiple of 64).
//
// Every (head, query) row picks its own spans, so a query-stationary tile has no shared K
// operand.  Following the bucketing idea of Section 4.3 (group (query, span) pairs by the key
// blocks they touch; on the fixed span grid a bucket is simply (kv head, span)), the routed part
// makes the SPAN stationary:
//
//   bucket (count) / unit_scan / scan / tiles / bucket (fill)   invert idx into per-(kv, span)
//                                   lists of query rows (integer work, LDS histograms)
//   span_flash_routed               persistent workgroups walk the (bucket, 256-row tile) list:
//                                   gathered Q rows against the span's K/V tiles staged through
//                                   LDS, flash softmax, MFMA QK^T and PV; writes a normalised
//                                   partial (o, lse) per (row, slot)
//   span_flash_local                the local window [c*S, i]: regular 128-row tiles of one
//                                   head with the causal mask; joint form with topk <= 8: merges
//                                   the row's routed partials in its epilogue (log-sum-exp) and
//                                   writes O and LSE; otherwise writes the row's last partial
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

constexpr int TG = 128;            // rows of one wavefront group (4 wavefronts x 32 columns)
constexpr int TN = 64;             // kv positions per staged tile
// Of the kernels with fp32 weights, too; at D = 64 tiles of 32 leave room (registers, LDS) for a third workgroup per
// compute unit and end closer to a span's end: 20011 rows in spans of 142 1213 -> 1098 us, 8000 in spans of 90, top-4, 260 ->
// 221 (short_routed_tiles: not where the tiles are few).  At D = 128 the registers of a third do not suffice: 2000 ->
// 2164.  (Nor does it help there to ask for the next tile's first stages, queries and record before a tile's output leaves,
// over the stages of its last kv tile: 1929 -> 2015.)
constexpr int fine_blocks(int tile) { return tile == 32 ? 3 : 2; }  // workgroups per compute unit
constexpr int HD = 128;            // head dimension of the kernels with bf16 weights

// LDS of the flash kernels (dynamic).  Main loop: stages of the V tile and of the K tile, filled
// by direct global->LDS loads (16 bytes per lane, a wavefront instruction fills 1 KB
// contiguously); rows are unpadded and their 16-byte pieces XOR-swizzled so that the MFMA
// operand reads of 16 consecutive lanes hit 16 distinct bank groups:
//   K tile [64][128]: piece p of row r at position p ^ (r & 15)
//   V tile [64][128]: piece p of row r at position p ^ ((r & 3) << 2): the four rows that 16 lanes read
//                     64 bytes of (with the 16 lanes beside them) lie in different bank groups
// V is staged as it lies in memory and transposed by the LDS reads (ds_read_b64_tr_b16): a transposed
// copy of V in the workspace cost a pass over the whole cache per call, however few the rows: 63 us for
// 4000 new rows behind 196000 tokens (0.945 -> 0.931 ms in all, the twice as many LDS reads take back part
// of it), 22 us at 48K on the paper's geometry (4.45 -> 4.41 ms); with all 262144 rows, where the copy was
// 87 us of 25.8 ms, the attention takes 26.0 ms.
// Epilogue: each wavefront group stages its output tile [128][128] bf16 (piece p of row r at
// p ^ (r & 15)).
//   NG = 2 (routed, 512 threads, 256 rows, one workgroup per compute unit, 154624 bytes): two K
//     and three V stages (the late group reads a V tile one step after the early group); the
//     output region is separate, so the first K/V tile of the next 256-row tile can be fetched
//     while the current one is written out.
//   NG = 1 (local window, 256 threads, 128 rows, 67072 bytes: two workgroups per compute unit, so
//     one's epilogue runs beside the other's main loop): two stages each; the output region
//     lies over the V stages, which are dead by then.
//   fp32-weight kernels: a wavefront's 32 rows go out in fp32, 64 columns at a time, through a slice of the
//     same size (32 x 64 fp32 = 32 x 128 bf16); at D = 64 the V stages are too small to lie under it.
template <int NG, int D = HD, int TNK = TN>
struct FlashLds {
  static constexpr int kStageElems = TNK * D;  // D = 128: 8192 bf16 = 16 KB
  static constexpr int kStagesK = 2, kStagesV = NG == 2 ? 3 : 2;
  static constexpr int kV = 0;
  static constexpr int kK = kStagesV * kStageElems * 2;
  static constexpr int kStagesEnd = (kStagesV + kStagesK) * kStageElems * 2;
  static constexpr bool kOver = NG == 1 && D == 128;  // the output region lies over the V stages
  static constexpr int kOutBytes = NG * TG * 256;
  static constexpr int kOut = kOver ? 0 : kStagesEnd;                               // [NG][TG][256 bytes]
  static constexpr int kRowOut = kOver ? kStagesEnd : kOut + kOutBytes;             // int64[NG][TG]
  static constexpr int kRowLse = kRowOut + NG * TG * 8;                             // float[NG][TG]
  // NG = 2: per wavefront 256 bytes for the next tile's record and 256 for its items, fetched by
  // direct global->LDS loads while the current tile runs (they hold no registers meanwhile)
  static constexpr int kAhead = kRowLse + NG * TG * 4;
  static constexpr int kBytes = kAhead + (NG == 2 ? 8 * 512 : 0);
  static constexpr int kThreads = NG * 256;
  static constexpr int kRows = NG * TG;  // query rows per workgroup
  static constexpr int kBlocksPerWave = kStageElems * 2 / 1024 / (4 * NG);  // 1 KB blocks of a staged tile per wavefront
};
constexpr int TM = FlashLds<2>::kRows;  // rows of a routed tile

#define SL_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// Direct global->LDS loads go through buffer instructions: base is wave-uniform, `bytes` bounds the
// offsets (a lane past it stores zeros).  The flat form (global_load_lds) counts as an LDS operation
// too, and the compiler then waits for every LDS read with lgkmcnt(0): the fragment reads that run four
// MFMAs ahead were drained at every fourth MFMA.  With the buffer form those waits are lgkmcnt(3).
// Measured: attention of a 256K prompt 27.09 -> 26.86 ms, the paper's geometry at 48K 4.75 -> 4.56 ms (its
// masked kernel no longer spills); the long kernel is held to 1.93 GHz by its power, so stalls cost it little.
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
__device__ __forceinline__ BufferRsrc buffer_of(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Two transposing LDS reads: the lane's column of kv rows 0..3 and 4..7 behind p (its own block address).
template <int D>
__device__ __forceinline__ bf16x8 transposed8(const bf16_t* p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) s16x4* LdsPtr;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)p);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)(p + 4 * D));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
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
                                                           int* __restrict__ flag) {
  __shared__ int s_items[1024], s_tiles[1024];
  const int tid = threadIdx.x;
  if (flag && tid == 0) *flag = 0;
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
  const int* item_off;
  const int* tile_off;
  const int4* tile_info;
  const int* items;
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
  int ab, af, aroot, E;
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

// One tile (256 rows, 128 of the window and fp32-weight kernels) as seen by a lane: the kv head and kv range [kv_begin,
// kv_end) shared by the workgroup (walked in kv tiles; what lies behind its end is masked or zero), and the lane's own
// query column.
struct TileDesc {
  int kv;
  int64_t kv_begin, kv_end;
  int64_t q_off;      // element offset of the lane's Q vector
  int64_t row_out;    // partial record index of the lane's column (fused merge: its row index
                      // h*Lq + r), -1 = no row
  int64_t first_pos;  // fused merge: position of the tile's first row; column x holds row x & row_mask of the tile
  int row_mask;
  int64_t i_q, lo_q;  // LOCAL: query position and start of its window
};

// State a workgroup carries from one tile to the next: the rotating stage indices, whether the
// tile's first K/V stage and Q fragments were already fetched by the previous tile's tail, and
// the Q fragments themselves.
struct FlashCarry {
  int kb, vb;
  bool primed;
  bool pending;  // the previous tile's output still sits in LDS (routed tiles write it out a step later)
  bf16x8 qf[8];
};

// Writes a wavefront's staged output rows (normalised partial o as bf16, lse) of a routed tile
// from the group's LDS region to the partial buffers: 16 lanes per row, 16 bytes per lane.
// Called when no direct global->LDS load is in flight (the compiler orders an LDS read after all
// outstanding vector-memory operations once such loads exist).
__device__ __forceinline__ void flush_routed_output(char* lds, int grp, int w4, int lane) {
  using Lds = FlashLds<2>;
  const ArgsPtr a = args_anew();
  const bf16_t* const ost = reinterpret_cast<const bf16_t*>(lds + Lds::kOut) + grp * TG * HD;
  const int64_t* const row_out = reinterpret_cast<const int64_t*>(lds + Lds::kRowOut) + grp * TG;
  const float* const row_lse = reinterpret_cast<const float*>(lds + Lds::kRowLse) + grp * TG;
  const int piece = lane & 15;
  // two rows per lane at a time: the tile's accumulators are live here, registers are scarce
#pragma unroll
  for (int ub = 0; ub < 8; ub += 2) {
    int64_t outs[2];
    uint4 vals[2];
    float lses[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = w4 * 32 + (ub + u) * 4 + (lane >> 4);
      outs[u] = row_out[row];
      lses[u] = row_lse[row];
      vals[u] = *reinterpret_cast<const uint4*>(&ost[row * HD + ((piece ^ (row & 15)) << 3)]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (outs[u] >= 0) {
        // streamed past the caches: the partials (gigabytes) are read back by a later kernel, and
        // the K/V tiles keep the L2
        store16_stream(a->part_o + outs[u] * HD + piece * 8, vals[u]);
        if (piece == 0) __builtin_nontemporal_store(lses[u], &a->part_lse[outs[u]]);
      }
    }
  }
}

// One tile of NG*128 rows.  All threads call.  If has_next, request_next() issues the caller's
// loads for the tile this workgroup processes afterwards and describe_next() turns them into
// `next`: the first is called right after the first kv step's barrier (next to that step's K/V
// loads, so the wait before the second step covers it), the second after the kv loop.
//
// The eight wavefronts form two groups of four (each group owns 128 rows, a wavefront 32
// columns); SIMD s hosts wavefront s of both groups.  Both groups consume the same staged K/V
// tiles, but the late group runs its PV product one kv tile behind:
//     early, per kv tile i:   QK(i)    softmax(i)  PV(i)
//     late,  per kv tile i:   PV(i-1)  QK(i)       softmax(i)          (+ PV(last) after the loop)
// so that between two barriers the softmax arithmetic of one group runs in the shadow of the
// other group's MFMAs instead of both groups asking for the matrix pipe at the same time.
// When the kv loop is over, the first K/V stage and the Q fragments of the next tile are
// requested before the output tile is normalised and staged in LDS; a routed tile's staged
// output goes to HBM during the next tile's first kv step (c.pending), a window tile's at once.
//
// FINE: the softmax weights keep fp32 precision: each is split into three bf16 parts, which hold the 24 bits of its
// mantissa between them, and V is multiplied with all three; the row sum is taken over the unsplit weights, partials
// are written in fp32, and the output of a tile goes to HBM before the next one starts.
template <int NG, bool LOCAL, bool FUSED, bool CLIP, int D = HD, bool FINE = false, int TT = TN, typename RequestNext,
          typename DescribeNext>
__device__ __forceinline__ void flash_tile(const FlashArgs& a, char* lds, const TileDesc& cur,
                                           TileDesc& next, bool has_next, RequestNext&& request_next,
                                           DescribeNext&& describe_next, FlashCarry& c) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int grp = wave >> 2, w4 = wave & 3;  // grp 0 = early, 1 = late
  const int qc = lane & 31, hf = lane >> 5;
  const int srow = w4 * 32 + qc;             // row inside the group's 128-row half tile
  static_assert(NG == 1 || !FINE, "fp32 partials leave with their tile: one group's output region");
  constexpr bool kMasked = LOCAL || CLIP;
  using Lds = FlashLds<NG, D, TT>;
  constexpr int kStageElems = Lds::kStageElems;
  constexpr int PPR = D / 8, RPB = 64 / PPR;  // 16-byte pieces per staged row, rows per 1 KB block
  constexpr int NDT = D / 32, NKK = D / 16;   // 32-row output tiles, 16-deep steps of the QK product
  constexpr int kStagesK = Lds::kStagesK, kStagesV = Lds::kStagesV, BPW = Lds::kBlocksPerWave;
  bf16_t* const ldsV = reinterpret_cast<bf16_t*>(lds + Lds::kV);
  bf16_t* const ldsK = reinterpret_cast<bf16_t*>(lds + Lds::kK);

  // Direct global -> LDS staging of one (K, V) tile pair in 1 KB blocks (4 rows each at D = 128); lane L
  // of a block lands at byte 16*L.
  // Per-lane byte offsets are loop-invariant 32-bit values; the kv head and the tile position
  // go into the wave-uniform base pointer.
  uint32_t koff[BPW], voff[BPW];
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    const int row = (wave * BPW + i) * RPB + lane / PPR, pc = lane % PPR;
    koff[i] = (uint32_t)((row * a.kvst + (pc ^ k_swizzle<D>(row)) * 8) * sizeof(bf16_t));
    voff[i] = (uint32_t)((row * a.kvst + (pc ^ v_swizzle<D>(row)) * 8) * sizeof(bf16_t));
  }
  // wavefront w fills blocks w*BPW .. w*BPW + BPW-1 of both tiles
  auto stage = [&](int kvh, int64_t t0, int64_t t_end, int kb, int vb) {
    // rows past the end of the sequence (FINE: of the tile's range) lie beyond the buffer: zeros in LDS
    // (masked later)
    const int64_t stop = FINE ? t_end : a.L;
    const int rows = __builtin_amdgcn_readfirstlane(stop - t0 < TT ? (int)(stop - t0) : TT);
    const int64_t first = uniform64((int64_t)kvh * a.kvsh + t0 * a.kvst);
    const uint32_t bytes = (uint32_t)(((rows - 1) * a.kvst + D) * sizeof(bf16_t));
    const BufferRsrc kr = buffer_of(a.K + first, bytes), vr = buffer_of(a.V + first, bytes);
#pragma unroll
    for (int i = 0; i < BPW; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, SL_LDS_PTR(ldsK + kb * kStageElems + (uwave * BPW + i) * 512), 16,
                                               koff[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < BPW; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, SL_LDS_PTR(ldsV + vb * kStageElems + (uwave * BPW + i) * 512), 16,
                                               voff[i], 0, 0, 0);
  };
  // Q row of a lane's column, as the B operand of S^T = K Q^T
  auto load_q = [&](int64_t q_off) {
    const bf16_t* qp = a.Q + q_off;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) c.qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16 + hf * 8);
  };
  if (!c.primed) {
    stage(cur.kv, cur.kv_begin, cur.kv_end, c.kb, c.vb);
    load_q(cur.q_off);
  }

  f32x16 o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m = -INFINITY, l = 0.f;  // m in log2 units of the scaled logit
  constexpr int NS = TT / 32, NP = TT / 16;  // 32-row score tiles, weight fragments
  bf16x8 pb[NP];                 // P^T fragments; the late group carries them to the next kv tile
#pragma unroll
  for (int ks = 0; ks < NP; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) pb[ks][e] = (__bf16)0.f;
  bf16x8 pl[FINE ? NP : 1], pm[FINE ? NP : 1];  // FINE: what pb leaves of the weights, and what that leaves

  const int krow = perm_row(qc);
  const int kswz = k_swizzle<D>(krow);  // swizzle key of this lane's K rows (32*sub does not change it)
  // V^T fragments come from transposing reads: 16 lanes read a [4 kv][16 d] block, 8 bytes each, and lane
  // i of them receives column i.  Lane offset (elements) of the block for d tile dt, kv rows 8*hf .. 8*hf+3.
  const int vrow = (lane & 15) >> 2;
  int vlane[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
    vlane[dt] = (8 * hf + vrow) * D +
                (((4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ v_swizzle<D>(vrow)) << 3) + 4 * (lane & 1);
  const float sc = a.scale_log2e;
  // the lane's own range [lo_q, i_q] as 32-bit offsets from the tile's first token
  auto offset_of = [&](int64_t t) {
    const int64_t d = t - cur.kv_begin;
    return (int)(d < -1 ? -1 : d > (1 << 30) ? (1 << 30) : d);
  };
  const int lo_r = kMasked ? offset_of(cur.lo_q) : 0, hi_r = kMasked ? offset_of(cur.i_q) : 0;

  // S^T = K Q^T (two 32-row halves of the tile), mask, running maximum, exponentials -> pb.
  // LDS fragment reads run four MFMAs ahead (0x100 = LDS read, 0x008 = MFMA).
  // base: the kv tile's offset from the tile's first token.
  auto qk_softmax = [&](const bf16_t* kt, int base) {
    f32x16 s[NS];
#pragma unroll
    for (int sub = 0; sub < NS; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sub][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
      for (int sub = 0; sub < NS; ++sub) {
        const bf16x8 ka = *reinterpret_cast<const bf16x8*>(
            &kt[(32 * sub + krow) * D + (((2 * kk + hf) ^ kswz) << 3)]);
        s[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, c.qf[kk], s[sub], 0, 0, 0);
      }
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < NS * NKK - 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    // The softmax arithmetic below competes for issue slots with the MFMA stream of the SIMD's
    // other wavefront; that one needs a slot every 32 cycles, this one needs most of them.
    __builtin_amdgcn_s_setprio(3);

    // Per-row ranges (the causal window, a span clipped behind a lower one, an anchor's span): only the
    // tiles at the ends of a wavefront's ranges are masked, one unsigned compare per score.  (With two
    // 64-bit compares per score on every tile the paper's geometry at 48K took 4.50 ms, now 3.68.)
    if (kMasked && __builtin_amdgcn_ballot_w64(lo_r > base || hi_r < base + TT - 1) != 0ull) {
      const uint32_t width = hi_r >= lo_r ? (uint32_t)(hi_r - lo_r) : 0u;
      const uint32_t u = hi_r >= lo_r ? (uint32_t)(base + 8 * hf - lo_r) : 0x80000000u;
#pragma unroll
      for (int sub = 0; sub < NS; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          s[sub][r] = u + (uint32_t)(32 * sub + 16 * (r >> 3) + (r & 7)) <= width ? s[sub][r] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < NS; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sub][r]);
    mx = pair_max(mx) * sc;
    // Lazy rescale, decided per column: a column's running maximum only moves when that column
    // grew by more than 2^8; until then its exponentials are taken against the old maximum
    // (p <= 256).  The branch is per wavefront, the arithmetic of a column does not depend on the
    // columns it shares the wavefront with (so a row's result does not depend on its tile-mates).
    const bool grow = mx > m + 8.f || (m == -INFINITY && mx > -INFINITY);
    if (__builtin_amdgcn_ballot_w64(grow) != 0ull) {
      const float alpha = grow ? fast_exp2(m - mx) : 1.f;  // m = -inf: 0, and l and o are still 0
      m = grow ? mx : m;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
    const float nm = m > -INFINITY ? -m : 0.f;  // whole column masked so far: exponentials are 0 anyway
#pragma unroll
    for (int ks = 0; ks < NP; ++ks) {
      f32x8 p;
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = fast_exp2(fmaf(s[ks >> 1][8 * (ks & 1) + e], sc, nm));
      pb[ks] = __builtin_convertvector(p, bf16x8);
      if constexpr (FINE) {
        const f32x8 rest = p - __builtin_convertvector(pb[ks], f32x8);
        pl[ks] = __builtin_convertvector(rest, bf16x8);
        pm[ks] = __builtin_convertvector(rest - __builtin_convertvector(pl[ks], f32x8), bf16x8);
#pragma unroll
        for (int e = 0; e < 8; ++e) l += p[e];
        continue;
      }
      // the row sum is taken over the rounded weights, the ones the PV product uses
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 pr = {pb[ks][e], pb[ks][e + 1]};
        const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
        l = __builtin_amdgcn_fdot2_f32_bf16(pr, one, l, false);
      }
    }
    __builtin_amdgcn_s_setprio(0);
  };
  // O^T += V^T P^T with the P^T fragments in pb
  auto pv = [&](const bf16_t* vt) {
#pragma unroll
    for (int ks = 0; ks < NP; ++ks)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const bf16x8 va = transposed8<D>(vt + vlane[dt] + 16 * ks * D);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[ks], o[dt], 0, 0, 0);
        if constexpr (FINE) {
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pl[ks], o[dt], 0, 0, 0);
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pm[ks], o[dt], 0, 0, 0);
        }
      }
    constexpr int kPer = FINE ? 3 : 1;  // MFMAs per fragment
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 1);
#pragma unroll
    for (int i = 0; i < NP * NDT - 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, kPer, 1);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4 * kPer, 1);
  };

  // a kv tile that none of the wavefront's rows attends is passed over (its weights would all be 0)
  auto attends = [&](int base) {
    return !kMasked || __builtin_amdgcn_ballot_w64(lo_r <= base + TT - 1 && hi_r >= base && hi_r >= lo_r) != 0ull;
  };
  int kb = c.kb, vb = c.vb, vb_prev = c.vb;
  // The late group of a bucket's last tile often has no row at all: it then only stages.  (4000 rows x 16
  // slots, six tiles a bucket: 885 -> 850 us for the call.  The same test in the early group, per
  // wavefront, cost the long prompt 1 %.)
  const bool idle = NG == 2 && grp == 1 && __builtin_amdgcn_ballot_w64(cur.row_out >= 0) == 0ull;
  bool owes_pv = false;  // late group: the previous kv tile's PV product is still to be taken
  for (int64_t t0 = cur.kv_begin; t0 < cur.kv_end; t0 += TT) {
    // After the barrier the tile of this iteration is visible to every wavefront, every wavefront
    // is done with the K stage of the previous tile and the late group with the V stage before
    // that: exactly the stages that the next tile goes into.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    const int kb1 = kb == kStagesK - 1 ? 0 : kb + 1, vb1 = vb == kStagesV - 1 ? 0 : vb + 1;
    if (NG == 2 && !LOCAL && c.pending) {
      // the previous tile's output: written out here, a step after it was staged, so that the wait
      // at the top of this tile did not have to cover its stores
      flush_routed_output(lds, grp, w4, lane);
      c.pending = false;
    }
    if (t0 + TT < cur.kv_end) stage(cur.kv, t0 + TT, cur.kv_end, kb1, vb1);
    if (NG == 2 && has_next && t0 == cur.kv_begin) request_next();
    const int base = (int)(t0 - cur.kv_begin);
    const bool mine = attends(base);
    if (grp == 0) {
      if (mine) {
        qk_softmax(ldsK + kb * kStageElems, base);
        pv(ldsV + vb * kStageElems);
      }
    } else if (!idle) {
      if (owes_pv) pv(ldsV + vb_prev * kStageElems);
      if (mine) qk_softmax(ldsK + kb * kStageElems, base);
      owes_pv = mine;
    }
    vb_prev = vb;
    kb = kb1;
    vb = vb1;
  }
  // Every wavefront is past its last QK: all K stages and the Q fragments are dead, and so is
  // every V stage except the last tile's (the late group still owes its PV).  Request the next
  // tile's first stage and Q fragments now; they land while this tile is written out.
  __syncthreads();
  c.kb = kb;
  c.vb = vb;
  c.primed = NG == 2 && has_next;  // NG = 1: the output region lies over the stages, nothing is fetched ahead
  if (NG == 2 && has_next) {
    next = describe_next();
    stage(next.kv, next.kv_begin, next.kv_end, kb, vb);
    load_q(next.q_off);
  }
  // From here to the end of the tile the late group is the critical path (it still owes a PV):
  // its wavefronts go first wherever both groups want an issue slot.
  if (NG == 2 && grp == 1) __builtin_amdgcn_s_setprio(2);
  if (grp == 1 && owes_pv) pv(ldsV + vb_prev * kStageElems);  // the late group's last PV

  // epilogue, wavefront-local (no workgroup barrier): normalise, stage the wavefront's 32 rows as
  // [row][d] bf16 in its own slice of the group's LDS region (swizzled 16-byte pieces), then
  // write 16 lanes per row, 16 bytes per lane.  LDS operations of one wavefront complete in
  // issue order, so the reads below see the writes of the other lanes.
  const float lt = pair_sum(l);
  const float inv = 1.f / lt;
  bf16_t* const ost = reinterpret_cast<bf16_t*>(lds + Lds::kOut) + grp * TG * HD;  // 256 bytes per row
  int64_t* const row_out = reinterpret_cast<int64_t*>(lds + Lds::kRowOut) + grp * TG;
  float* const row_lse = reinterpret_cast<float*>(lds + Lds::kRowLse) + grp * TG;
  if (hf == 0) {
    row_lse[srow] = (m + __log2f(lt)) * kLn2;
    row_out[srow] = cur.row_out;
  }
  if constexpr (FINE) {
    // fp32 partial, 64 columns at a time: 16 lanes per row, 16 bytes per lane
    float* const fst = reinterpret_cast<float*>(ost);
    const ArgsPtr b = args_anew();
    const int piece = lane & 15;
#pragma unroll
    for (int half = 0; half < D / 64; ++half) {
#pragma unroll
      for (int dd = 0; dd < 2; ++dd)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = o[2 * half + dd][4 * g4 + e] * inv;
          *reinterpret_cast<f32x4*>(&fst[srow * 64 + (((8 * dd + 2 * g4 + hf) ^ (srow & 15)) << 2)]) = v;
        }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int row = w4 * 32 + u * 4 + (lane >> 4);
        const int64_t at = row_out[row];
        const uint4 v = *reinterpret_cast<const uint4*>(&fst[row * 64 + ((piece ^ (row & 15)) << 2)]);
        if (at >= 0) {
          // past the caches, like the bf16 partials: they are gigabytes, the K/V tiles keep the L2
          store16_stream(b->part_of + at * D + half * 64 + piece * 4, v);
          if (half == 0 && piece == 0) b->part_lse[at] = row_lse[row];
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_s_setprio(0);
    return;
  }
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int unit = (4 * dt + g4) ^ (srow & 15);
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[dt][4 * g4 + e] * inv;
      const bf16x4 w = __builtin_convertvector(v, bf16x4);
      *reinterpret_cast<bf16x4*>(&ost[srow * HD + unit * 8 + 4 * hf]) = w;
    }
  __builtin_amdgcn_wave_barrier();
  if constexpr (FUSED) {
    // Local-window tile with the merge fused in (topk <= 8): the lane that would store 16 bytes
    // of the window's partial instead loads the same 16 bytes of the row's routed partials
    // (written by the routed kernel, which ran before on the stream), does the log-sum-exp merge
    // and stores the final output.  Every load is issued before the first dependent use; slots
    // that take no part may hold anything and are discarded by selects, never by arithmetic.
    const int topk = a.topk, nslot = topk + 1;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      int64_t outs[4];
      int js[4][8];
      float ls[4][8];
      uint4 ov[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = w4 * 32 + (half * 4 + u) * 4 + (lane >> 4), piece = lane & 15;
        outs[u] = row_out[row];
        const int64_t rg = outs[u] >= 0 ? outs[u] : 0;
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
          const bool in = sl < topk;
          js[u][sl] = in ? a.idx[rg * topk + sl] : -1;
          ls[u][sl] = in ? a.part_lse[rg * nslot + sl] : 0.f;
          ov[u][sl] = in ? load16(a.part_o + (rg * nslot + sl) * HD + piece * 8) : make_uint4(0, 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = w4 * 32 + (half * 4 + u) * 4 + (lane >> 4), piece = lane & 15;
        const int cq = (int)((cur.first_pos + (row & cur.row_mask)) / a.A);
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
          *reinterpret_cast<uint4*>(a.O + outs[u] * HD + piece * 8) = res;
          if (piece == 0) a.LSE[outs[u]] = M + __logf(wsum);
        }
      }
    }
  } else if (NG == 2 && !LOCAL) {
    c.pending = true;  // written out during the next tile's first kv step, or by the caller after the last tile
  } else {
    // Every LDS read comes before the first store, and the values are pinned there: the compiler
    // orders an LDS read after all outstanding vector-memory operations once direct global->LDS
    // loads are in flight (the next tile's), so a read between two stores would wait for the
    // earlier store to be acknowledged.
    int64_t outs[8];
    uint4 vals[8];
    float lses[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int row = w4 * 32 + u * 4 + (lane >> 4), piece = lane & 15;
      outs[u] = row_out[row];
      lses[u] = row_lse[row];
      vals[u] = *reinterpret_cast<const uint4*>(&ost[row * HD + ((piece ^ (row & 15)) << 3)]);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      asm volatile("" : "+v"(vals[u].x), "+v"(vals[u].y), "+v"(vals[u].z), "+v"(vals[u].w), "+v"(lses[u]),
                   "+v"(outs[u]));
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int piece = lane & 15;
      if (outs[u] >= 0) {
        store16_stream(a.part_o + outs[u] * HD + piece * 8, vals[u]);
        if (piece == 0) a.part_lse[outs[u]] = lses[u];
      }
    }
  }
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_wave_barrier();
  // No trailing barrier: a wavefront's output slice is private to it, and the K/V stages are
  // handed over through c.kb / c.vb.
}

// Routed spans: persistent workgroups walk the tile list.  XCD x (workgroups with
// blockIdx % 8 == x) owns the contiguous chunk [x*T/8, (x+1)*T/8) of the tile list; its
// workgroups walk the chunk interleaved, so at any moment they sit on neighbouring tiles -- the
// same one or two buckets -- and share the span through that XCD's L2.  The record and the item
// of a workgroup's next tile are fetched while its current tile is computed.
// CLIP (overlapping spans, anchor spacing A < S, joint softmax): a row's range in span j starts behind
// the end of the nearest lower span that the row lists, so that every token of the union counts once.
// FINE (with CLIP): fp32 weights and partials, spans of any length at any offset; a row's range is its whole
// span unless a->clip says that spans of a row overlap in one softmax.  Tiles of 128 rows, two workgroups per
// compute unit: one's tile ends run beside the other's kv loop.
template <bool CLIP, int D = HD, bool FINE = false, int TT = TN, int NG = FINE ? 1 : 2>
__global__ __launch_bounds__(NG * 256, NG == 2 ? 1 : FINE ? fine_blocks(TT) : 2) void span_flash_routed_kernel(
    const FlashArgs a) {
  using Lds = FlashLds<NG, D, TT>;
  constexpr int TM = Lds::kRows;
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qrow = (wave >> 2) * TG + (wave & 3) * 32 + (lane & 31);
  const int64_t T = a.tile_off[a.Hq / a.G * a.n];
  const int NWL = gridDim.x / 8;  // workgroups per XCD (the grid is a multiple of 8)
  const int xcd = blockIdx.x % 8, wl = blockIdx.x / 8;
  const int64_t c_begin = T * xcd / 8, c_end = T * (xcd + 1) / 8;
  const int64_t t_begin = c_begin + wl, t_end = c_end;
  if (t_begin >= t_end) return;

  auto describe = [&](const int4& info, int item) {
    const ArgsPtr a = args_anew();
    TileDesc d;
    d.kv = info.x / a->n;
    const int j = info.x % a->n;
    d.kv_end = (int64_t)(j + 1) * a->A;
    d.kv_begin = d.kv_end - a->S > 0 ? d.kv_end - a->S : 0;
    const int rowid = item >> 5, slot = item & 31;
    const int hl = rowid / (int)a->Lq;
    const int64_t r = rowid - (int64_t)hl * a->Lq;
    const int h = d.kv * a->G + hl;
    d.q_off = h * a->qsh + r * a->qst;
    d.row_out = qrow < info.z ? ((int64_t)h * a->Lq + r) * (a->topk + 1) + slot : -1;
    d.i_q = d.kv_end - 1;
    d.lo_q = d.kv_begin;
    if (FINE ? a->clip : CLIP) {
      const int64_t c = (a->q_pos0 + r) / a->A;
      const int32_t* irow = a->idx + ((int64_t)h * a->Lq + r) * a->topk;
      for (int s2 = 0; s2 < a->topk; ++s2) {
        const int64_t jj = irow[s2];
        if (jj >= 0 && jj < c && jj < j && (jj + 1) * a->A > d.lo_q) d.lo_q = (jj + 1) * a->A;
      }
    }
    d.first_pos = 0;
    d.row_mask = 0;
    return d;
  };
  FlashCarry carry;
  carry.kb = carry.vb = 0;
  carry.primed = false;
  carry.pending = false;
  if constexpr (NG == 1) {
    for (int64_t t = t_begin; t < t_end; t += NWL) {
      TileDesc cur = describe(a.tile_info[t], a.items[t * TM + qrow]), unused = cur;
      flash_tile<1, false, false, CLIP, D, FINE, TT>(a, lds, cur, unused, false, [] {}, [&] { return cur; }, carry);
      __syncthreads();  // the next tile's stages lie over the output slices of all wavefronts
    }
  } else {
    // The record and the items of a workgroup's next tile are requested during the current tile's
    // first kv step as direct global->LDS loads into the wavefront's own 512 bytes (the items of tile t sit
    // at t*TM, so the two do not depend on each other) and read back at its tail.
    int* const ahead = reinterpret_cast<int*>(lds + Lds::kAhead) + __builtin_amdgcn_readfirstlane(wave) * 128;
    const int4 info0 = a.tile_info[t_begin];
    TileDesc cur = describe(info0, a.items[t_begin * TM + qrow]);
    for (int64_t t = t_begin; t < t_end; t += NWL) {
      const bool has_next = t + NWL < t_end;
      TileDesc nxt = cur;
      flash_tile<2, false, false, CLIP>(
          a, lds, cur, nxt, has_next,
          [&] {
            const ArgsPtr a = args_anew();
            const int uw = __builtin_amdgcn_readfirstlane(wave);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(a->tile_info + (t + NWL), 16), SL_LDS_PTR(ahead), 4,
                                                     (lane & 3) * 4, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(a->items + (t + NWL) * TM + uw * 32, 128),
                                                     SL_LDS_PTR(ahead + 64), 4, (lane & 31) * 4, 0, 0, 0);
          },
          [&] {
            const int4 ninfo = make_int4(ahead[0], ahead[1], ahead[2], 0);
            return describe(ninfo, ahead[64 + lane]);
          },
          carry);
      cur = nxt;
    }
    // the last tile's output (its epilogue ended with the wavefront's own LDS writes)
    if (carry.pending) flush_routed_output(lds, wave >> 2, wave & 3, lane);
  }
}

// The paper's geometry: routed tiles of a (kv head, end block) bucket.  Every row of a tile has
// its own token range [lo, hi) (hi inside the bucket's block); the tile walks the kv range from
// the lowest lo to the highest hi of its rows (rounded to whole 64-token tiles) with per-row masks.
__global__ __launch_bounds__(FlashLds<2>::kThreads, 1) void span_flash_anchor_kernel(const FlashArgs a) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int64_t s_lo[8], s_hi[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qrow = (wave >> 2) * TG + (wave & 3) * 32 + (lane & 31);
  const int64_t T = a.tile_off[a.Hq / a.G * a.n];
  const int NWL = gridDim.x / 8;
  const int xcd = blockIdx.x % 8, wl = blockIdx.x / 8;
  const int64_t c_begin = T * xcd / 8, c_end = T * (xcd + 1) / 8;
  const int64_t t_begin = c_begin + wl, t_end = c_end;
  if (t_begin >= t_end) return;

  // all threads call (two barriers inside)
  auto describe = [&](const int4& info, int item) {
    const ArgsPtr a = args_anew();
    TileDesc d;
    d.kv = info.x / a->n;
    const int rowid = item >> 5, slot = item & 31;
    const int hl = rowid / (int)a->Lq;
    const int64_t r = rowid - (int64_t)hl * a->Lq;
    const int h = d.kv * a->G + hl;
    const int64_t i = a->q_pos0 + r;
    const bool real = qrow < info.z;
    const int64_t t = a->idx[((int64_t)h * a->Lq + r) * a->topk + slot];
    const AnchorSpan sp = anchor_span_of(i, t, span_base_length(i, a->aroot), a->window, a->ab, a->af);
    d.q_off = h * a->qsh + r * a->qst;
    d.row_out = real ? ((int64_t)h * a->Lq + r) * (a->topk + 1) + slot : -1;
    d.lo_q = sp.lo;
    d.i_q = sp.hi - 1;
    d.first_pos = 0;
    d.row_mask = 0;
    // the tile's kv range: from the lowest lo to the highest hi of its rows
    int64_t lo = real && sp.hi > sp.lo ? sp.lo : INT64_MAX, hi = real && sp.hi > sp.lo ? sp.hi : 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const int64_t lo2 = __shfl_xor(lo, off, 64), hi2 = __shfl_xor(hi, off, 64);
      lo = lo2 < lo ? lo2 : lo;
      hi = hi2 > hi ? hi2 : hi;
    }
    __syncthreads();  // earlier readers of s_lo / s_hi are done
    if (lane == 0) {
      s_lo[wave] = lo;
      s_hi[wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      lo = s_lo[w] < lo ? s_lo[w] : lo;
      hi = s_hi[w] > hi ? s_hi[w] : hi;
    }
    if (hi <= lo) lo = hi = 0;  // cannot happen for a tile with items; keeps the range sane
    d.kv_begin = lo / TN * TN;
    d.kv_end = (hi + TN - 1) / TN * TN;
    return d;
  };
  FlashCarry carry;
  carry.kb = carry.vb = 0;
  carry.primed = false;
  carry.pending = false;
  int* const ahead = reinterpret_cast<int*>(lds + FlashLds<2>::kAhead) + __builtin_amdgcn_readfirstlane(wave) * 128;
  const int4 info0 = a.tile_info[t_begin];
  TileDesc cur = describe(info0, a.items[t_begin * TM + qrow]);
  for (int64_t t = t_begin; t < t_end; t += NWL) {
    const bool has_next = t + NWL < t_end;
    TileDesc nxt = cur;
    flash_tile<2, false, false, true>(
        a, lds, cur, nxt, has_next,
        [&] {
          const ArgsPtr a = args_anew();
          const int uw = __builtin_amdgcn_readfirstlane(wave);
          __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(a->tile_info + (t + NWL), 16), SL_LDS_PTR(ahead), 4,
                                                   (lane & 3) * 4, 0, 0, 0);
          __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer_of(a->items + (t + NWL) * TM + uw * 32, 128),
                                                   SL_LDS_PTR(ahead + 64), 4, (lane & 31) * 4, 0, 0, 0);
        },
        [&] {
          const int4 ninfo = make_int4(ahead[0], ahead[1], ahead[2], 0);
          return describe(ninfo, ahead[64 + lane]);
        },
        carry);
    cur = nxt;
  }
  if (carry.pending) flush_routed_output(lds, wave >> 2, wave & 3, lane);
}

// A window tile's 128 columns are `heads` query heads of one kv head, which attend the same keys, times 128 / heads rows:
// the fewer rows, the shorter the kv range that the tile walks beyond what each of its rows attends.  Heads: the largest
// power of two that divides the group, up to 8.  Tiles of 128 rows of one head -> 16 rows of 8, this kernel, us, 32:4
// heads: 20011 rows, spans of 142 (fp32 weights) 181 -> 140; 49157 rows, windows of 1088 tokens 990 -> 970; 4000 rows, spans
// of 512 47 -> 43; 262144 rows, spans of 512, with the merge (bound by the partials) 5000 -> 4960.
__host__ __device__ inline int local_heads(int G) {
  const int p = G & -G;
  return p < 8 ? p : 8;
}
// Row tiles and their grouping into chunks of `tps` tiles (the tiles of one span when S is a multiple of the tile height).
struct LocalMap {
  int shift, rows;         // rows of a tile, a power of two: what depends on it is shifted, not divided
  int tiles, tps, chunks;  // tiles of a kv head (and group of `heads` heads)
};
__host__ __device__ inline LocalMap local_map(int64_t Lq, int S, int G) {
  LocalMap m;
  m.shift = __builtin_ctz(FlashLds<1>::kRows / local_heads(G));
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
inline unsigned local_grid(int64_t Lq, int S, int Hkv, int G) {
  const LocalMap m = local_map(Lq, S, G);
  int best = 0;
  for (int x = 0; x < 8; ++x) {
    const int cx = (m.chunks - x + 7) / 8;
    const bool lx = m.chunks > 0 && (m.chunks - 1) % 8 == x;
    const int tx = cx * m.tps - (lx ? m.chunks * m.tps - m.tiles : 0);
    best = tx > best ? tx : best;
  }
  return (unsigned)(8 * Hkv * best * (G / local_heads(G)));
}

// Local window [c*S, i]: regular tiles of 128 columns with the causal / window mask.
// FUSED = false: writes the window's partial into the row's last slot (a merge kernel follows).
// FUSED = true (joint softmax, topk <= 8): merges the row's routed partials in the epilogue and
// writes the final output, which takes the merge's HBM traffic off the critical path of a
// separate kernel and saves the window partial's round trip.
template <bool FUSED, int D = HD, bool FINE = false, int TT = TN>
__global__ __launch_bounds__(FlashLds<1>::kThreads, FINE ? fine_blocks(TT) : 2) void span_flash_local_kernel(const FlashArgs a) {
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qrow = wave * 32 + (lane & 31);
  // Workgroup -> (heads, row tile), XCD-aware: blocks are dealt round-robin to the 8 XCDs, each
  // with its own L2.  A run of `tps` consecutive row tiles (one span's worth) goes to one XCD,
  // and inside an XCD the groups of heads of a kv head take the same row tile back to back, so the
  // window's K/V tiles are fetched from HBM about once.
  const LocalMap lm = local_map(a.Lq, a.A, a.G);
  const int heads = FlashLds<1>::kRows >> lm.shift, sets = a.G / heads;
  const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const int chunks_x = (lm.chunks - xcd + 7) / 8;                 // chunks xcd, xcd+8, ... of a kv head
  const bool has_last = lm.chunks > 0 && (lm.chunks - 1) % 8 == xcd;  // the only chunk that may be short
  const int tiles_x = chunks_x * lm.tps - (has_last ? lm.chunks * lm.tps - lm.tiles : 0);
  if (slot >= (a.Hq / a.G) * tiles_x * sets) return;  // uniform: the grid is padded to 8 * the largest share
  const int kvh = slot / (tiles_x * sets), rem = slot % (tiles_x * sets);
  const int tile_local = rem / sets;
  const int tile = (xcd + 8 * (tile_local / lm.tps)) * lm.tps + tile_local % lm.tps;
  const int h = kvh * a.G + rem % sets * heads + (qrow >> lm.shift);
  const int64_t r0 = (int64_t)tile << lm.shift;
  const int64_t r = r0 + (qrow & (lm.rows - 1));
  const int64_t rc = r < a.Lq ? r : a.Lq - 1;
  TileDesc d;
  d.kv = kvh;
  d.q_off = h * a.qsh + rc * a.qst;
  d.first_pos = a.q_pos0 + r0;
  d.row_mask = lm.rows - 1;
  if (FUSED) d.row_out = r < a.Lq ? (int64_t)h * a.Lq + r : -1;
  else d.row_out = r < a.Lq ? ((int64_t)h * a.Lq + r) * (a.topk + 1) + a.topk : -1;
  d.i_q = a.q_pos0 + rc;
  const int64_t i_first = a.q_pos0 + r0;
  const int64_t i_last = min(a.q_pos0 + r0 + lm.rows - 1, a.q_pos0 + a.Lq - 1);
  if (a.window > 0) {  // the paper's geometry: a sliding window [i - window + 1, i] per row
    d.lo_q = d.i_q - a.window + 1 > 0 ? d.i_q - a.window + 1 : 0;
    const int64_t first_lo = i_first - a.window + 1 > 0 ? i_first - a.window + 1 : 0;
    d.kv_begin = first_lo / TN * TN;
  } else {
    d.lo_q = (d.i_q / a.A) * a.A;
    d.kv_begin = (i_first / a.A) * a.A;
  }
  d.kv_end = FINE ? i_last + 1 : d.kv_begin + ((i_last - d.kv_begin) / TN + 1) * TN;
  FlashCarry carry;
  carry.kb = carry.vb = 0;
  carry.primed = false;
  carry.pending = false;
  TileDesc unused = d;
  flash_tile<1, true, FUSED, false, D, FINE, TT>(a, lds, d, unused, false, [] {}, [&] { return d; }, carry);
}

// ------------------------------------------------------------------ merge
// A lane's 16 bytes of a partial: 8 bf16 (P = bf16_t) or 4 fp32 (P = float) columns.
template <typename P>
__device__ __forceinline__ void store_columns(bf16_t* p, const float* v) {
  uint32_t w[Elem<P>::EPL / 2];
#pragma unroll
  for (int e = 0; e < Elem<P>::EPL / 2; ++e)
    w[e] = (uint32_t)f32_to_bf16(v[2 * e]) | ((uint32_t)f32_to_bf16(v[2 * e + 1]) << 16);
  if constexpr (Elem<P>::EPL == 8) *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
  else *reinterpret_cast<uint2*>(p) = make_uint2(w[0], w[1]);
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
  size_t counts, unit_cnt, item_off, tile_off, cursor, tile_info, items, part_lse, part_o, flag, total;
  BucketPlan plan;
  int B, max_tiles;
  int64_t max_items;
};

// Per-device facts, looked up on the first call with that device current: the grid of the
// persistent kernel (one resident workgroup of eight wavefronts per compute unit) and whether the
// flash kernels were granted more dynamic LDS than the 64 KB a kernel gets by default.
struct DeviceSetup {
  int grid = 0;     // 0 = not looked up yet
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
    d.lds_ok =
        hipFuncSetAttribute(reinterpret_cast<const void*>(span_flash_routed_kernel<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FlashLds<2>::kBytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(span_flash_routed_kernel<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FlashLds<2>::kBytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(span_flash_anchor_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FlashLds<2>::kBytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(span_flash_local_kernel<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FlashLds<1>::kBytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(span_flash_local_kernel<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FlashLds<1>::kBytes) == hipSuccess;
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

MfmaWs carve(const Problem& pb, int tm = TM, size_t part_elem = sizeof(bf16_t)) {
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
                    const Items& it, int* flag, hipStream_t st) {
  const int n = (int)pb.n;
  const int per_block = 4;  // 4 * 4096 counters = 64 KB
  const dim3 grid((unsigned)((w.plan.units + per_block - 1) / per_block), pb.Hq);
  const size_t lds = (size_t)per_block * n * sizeof(int);
  hipLaunchKernelGGL((bucket_kernel<false, Items>), grid, dim3(64 * per_block), lds, st, idx, unit_cnt, cursor,
                     items, part_lse, pb.Lq, pb.q_pos0, pb.G, pb.topk, n, w.plan, it);
  hipLaunchKernelGGL(bucket_unit_scan_kernel, dim3((n + 31) / 32, pb.Hkv), dim3(1024), 0, st, unit_cnt, counts,
                     pb.G * w.plan.units, n);
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(1024), 0, st, counts, item_off, tile_off, cursor, w.B,
                     w.tm, flag);
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

size_t prefill_attention_mfma_ws_bytes(const Problem& pb) { return carve(pb).total; }

sl_status prefill_attention_mfma(const Problem& pb, const void* Q, const void* K, const void* V,
                                 const int32_t* idx, void* O, float* LSE, void* ws,
                                 hipStream_t st) {
  const MfmaWs w = carve(pb);
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
  a.item_off = item_off;
  a.tile_off = tile_off;
  a.tile_info = tile_info;
  a.items = items;
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
  a.E = 0;
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
                        GridItems{pb.A}, nullptr, st))
      return SL_ERR_LAUNCH;
    if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
    if (pb.A < pb.S && !pb.combined)  // overlapping spans in one joint softmax: per-row clipping
      hipLaunchKernelGGL(span_flash_routed_kernel<true>, dim3(dev.grid), dim3(FlashLds<2>::kThreads),
                         FlashLds<2>::kBytes, st, a);
    else
      hipLaunchKernelGGL(span_flash_routed_kernel<false>, dim3(dev.grid), dim3(FlashLds<2>::kThreads),
                         FlashLds<2>::kBytes, st, a);
    if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  }
  const unsigned lgrid = local_grid(pb.Lq, pb.A, pb.Hkv, pb.G);
  if (!pb.combined && pb.topk <= 8) {  // the window kernel merges and writes the final output
    hipLaunchKernelGGL(span_flash_local_kernel<true>, dim3(lgrid), dim3(FlashLds<1>::kThreads),
                       FlashLds<1>::kBytes, st, a);
    return hipGetLastError() == hipSuccess ? SL_OK : SL_ERR_LAUNCH;
  }
  hipLaunchKernelGGL(span_flash_local_kernel<false>, dim3(lgrid), dim3(FlashLds<1>::kThreads),
                     FlashLds<1>::kBytes, st, a);
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
//   20011 rows, spans of 142: 16400 -> 1940; at D = 64: 8320 -> 1210; 2500 rows, spans of 50: 791 -> 191;
//   200 rows behind 60000 tokens, spans of 245: 589 -> 83; 8 rows there: 157 -> 72.
// 128-row tiles, two workgroups per compute unit, three at D = 64 (one's tile ends beside the other's kv loop): a span of
// 142 tokens is three kv tiles, and 256-row tiles with one workgroup took 1381 us for the routed part where
// these take 1288.
// Calls without a workspace, or with one too small, take the row-stationary kernels as before.
namespace {

// Tiles that the routed part has at most: one that is not full for every span with a row, and the full ones.
double fine_tiles(const Problem& pb) {
  const double items = (double)pb.Hq * pb.Lq * pb.topk;
  return fmin(items, (double)pb.Hkv * pb.n) + items / TG;
}

// Estimated us of the two forms; the call takes the smaller.  Row-stationary: 0.02 ns per row and key, with
// about 13 keys' worth of latency per slot, and no less than one row's own chain of loads.  This form: nine
// launches, tiles of 4 us plus 2.6 us per kv tile on 512 workgroups (a bucket's last tile is padded),
// partials written and read.  Of 22 measured calls (2 to 20000 rows, spans of 4 to 245 tokens) the estimates
// choose the faster form in 18; the other four stay with the row kernels and lose 5 to 15 us, or half of
// 415 us (1000 rows behind 60000 tokens in spans of 30, buckets a quarter full).
bool fine_is_faster(const Problem& pb) {
  const double rows = (double)pb.Hq * pb.Lq, items = rows * pb.topk, keys = (double)pb.topk * pb.S + pb.A / 2;
  const double d = pb.D / 128.0;
  const double by_rows = fmax(0.075 * keys, 2e-5 * d * rows * (keys + 13.0 * pb.topk));
  const double steps = (double)((pb.S + TN - 1) / TN);
  return 45 + fine_tiles(pb) * (4 + 2.6 * steps) / 512 + (items + rows) * pb.D * 8 / 4.5e6 < by_rows;
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

// D = 64: kv tiles of 32 tokens, three workgroups per compute unit, pay where there are tiles for a second round.  Where two
// workgroups per compute unit take them all at once, the call lasts as long as one tile's chain of kv steps, and half as
// many steps of 64 are shorter; so they are over long spans.  500 calls of 1 to 64 heads, 64 -> 32 tokens, time of the call
// (means): up to 512 tiles, spans of up to 64 1.00, 256 1.03, 512 1.06, longer ones 1.11 (2253 tokens, 24:4 heads, one row
// 110 -> 133 us); 1024 to 2048 tiles 0.96, 0.97, 0.97, 1.06; more 0.93, 0.94, 0.98, 1.03.
// The window alone: up to a workgroup per compute unit 1.01 (spans beyond 512 tokens 1.03), from two on 0.98.
bool short_routed_tiles(const Problem& pb, const DeviceSetup& dev) {
  return pb.D == 64 && fine_tiles(pb) > 2 * dev.grid && pb.S <= 512;
}
bool short_window_tiles(const Problem& pb, const DeviceSetup& dev, unsigned grid) {
  return pb.D == 64 && grid > (unsigned)dev.grid;
}

template <int D>
bool fine_setup(DeviceSetup* out) {
  static std::mutex mu;
  static bool done[kMaxDevices];
  int dev = -1;
  if (!device_setup(out) || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::lock_guard<std::mutex> lock(mu);
  auto allow = [](auto routed, auto local, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(routed), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(local), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
  };
  if (!done[dev]) {
    done[dev] = allow(span_flash_routed_kernel<true, D, true>, span_flash_local_kernel<false, D, true>, FlashLds<1, D>::kBytes);
    if constexpr (D == 64)
      done[dev] = done[dev] && allow(span_flash_routed_kernel<true, D, true, 32>, span_flash_local_kernel<false, D, true, 32>, FlashLds<1, D, 32>::kBytes);
  }
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
  a.item_off = item_off;
  a.tile_off = tile_off;
  a.tile_info = tile_info;
  a.items = items;
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
                      GridItems{pb.A}, flag, st))
    return SL_ERR_LAUNCH;
  if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
  const unsigned lgrid = local_grid(pb.Lq, pb.A, pb.Hkv, pb.G);
  auto routed = [&](auto tile) {
    constexpr int TT = decltype(tile)::value;
    hipLaunchKernelGGL((span_flash_routed_kernel<true, D, true, TT>), dim3(fine_blocks(TT) * dev.grid), dim3(256),
                       (FlashLds<1, D, TT>::kBytes), st, a);
  };
  auto local = [&](auto tile) {
    constexpr int TT = decltype(tile)::value;
    hipLaunchKernelGGL((span_flash_local_kernel<false, D, true, TT>), dim3(lgrid), dim3(256),
                       (FlashLds<1, D, TT>::kBytes), st, a);
  };
  using Short = std::integral_constant<int, D == 64 ? 32 : TN>;
  using Long = std::integral_constant<int, TN>;
  if (short_routed_tiles(pb, dev)) routed(Short{});
  else routed(Long{});
  if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  if (short_window_tiles(pb, dev, lgrid)) local(Short{});
  else local(Long{});
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

// End-block size E of the buckets: the smallest power-of-two multiple of 64 tokens that gives a
// bucket about two 256-row tiles of items on average, and at most 4096 blocks per kv head.
int anchor_block_tokens(const Problem& pb) {
  const int64_t items = (int64_t)pb.G * pb.Lq * (pb.topk > 0 ? pb.topk : 1);
  int64_t E = 64;
  while (E < 4096 && (items * E < 512 * pb.L || (pb.L + E - 1) / E > 4096)) E <<= 1;
  return (int)E;
}

Problem anchor_view(const Problem& pb) {
  Problem q = pb;
  q.A = anchor_block_tokens(pb);
  q.n = (pb.L + q.A - 1) / q.A;
  return q;
}

}  // namespace

bool prefill_anchor_mfma_supported(const Problem& pb, int64_t window) {
  const Problem q = anchor_view(pb);
  return window >= 1 && pb.topk >= 1 && pb.dtype == SL_BF16 && pb.D == HD && q.n <= 4096 &&
         (int64_t)pb.G * pb.Lq < ((int64_t)1 << 26) &&
         pb.L <= kMaxTokens &&
         64 * pb.kvst * 2 < ((int64_t)1 << 31) &&
         (int64_t)pb.Hq * pb.Lq * (pb.topk + 1) < ((int64_t)1 << 31) &&
         (int64_t)pb.Hq * pb.Lq * pb.topk + ((int64_t)pb.Hkv * q.n + 1) * TM < ((int64_t)1 << 31) &&
         (int64_t)pb.Hq * pb.qsh + pb.Lq * pb.qst < ((int64_t)1 << 31);
}

size_t prefill_anchor_mfma_ws_bytes(const Problem& pb) { return carve(anchor_view(pb)).total; }

// Span-attention and combination on the paper's geometry (Section 3.3-3.4, Algorithm 1), matrix-core
// form following Section 4.3's bucketing by key-block footprint: (row, slot) pairs are bucketed by
// the block that holds their span's last token, a bucket's rows share one sliding K/V range with
// per-row masks, the sliding window is a banded flash kernel, and the gated merge combines them.
sl_status prefill_anchor_attention_mfma(const Problem& pb, int64_t window, int b, int f, int root,
                                        const void* Q, const void* K, const void* V,
                                        const int32_t* anchors, void* O, void* ws, hipStream_t st) {
  const Problem q = anchor_view(pb);
  const MfmaWs w = carve(q);
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
  a.item_off = item_off;
  a.tile_off = tile_off;
  a.tile_info = tile_info;
  a.items = items;
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
  a.E = q.A;
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
                      AnchorItems{window, b, f, root, a.E}, nullptr, st))
    return SL_ERR_LAUNCH;
  if (pb.prof_start) (void)hipEventRecord(pb.prof_start, st);
  hipLaunchKernelGGL(span_flash_anchor_kernel, dim3(dev.grid), dim3(FlashLds<2>::kThreads),
                     FlashLds<2>::kBytes, st, a);
  if (pb.prof_stop) (void)hipEventRecord(pb.prof_stop, st);
  const unsigned lgrid = local_grid(pb.Lq, a.A, pb.Hkv, pb.G);
  hipLaunchKernelGGL(span_flash_local_kernel<false>, dim3(lgrid), dim3(FlashLds<1>::kThreads),
                     FlashLds<1>::kBytes, st, a);
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
