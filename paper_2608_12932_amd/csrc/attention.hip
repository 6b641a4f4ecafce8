// Streaming prefill attention (FlashDrive Sec. 3.1 and Fig. 3).
//
// When the camera window advances by one frame, only the tokens of the
// frame that just arrived need fresh attention rows: they form the query
// set here, while the keys and values come from the whole window's cache
// (older frames kept from earlier steps plus the arrival, ordered view by
// view).  The cache stores keys without their rotary embedding; this
// kernel rotates each key at the position it occupies in the window now,
// so sliding the window changes only the position array.  Key j may be
// seen by query i exactly when pos_k[j] <= pos_q[i], i.e. causally in the
// view-major order of the window.
//
// A first kernel rotates the window's keys once per call, at the
// positions they occupy now (every query head of a kv head reads them),
// records each 32-key tile's smallest and largest position, and (one more
// workgroup) deals the attention's work items to workgroup ids so that the
// CUs get even shares: a query block late in the window sees many more key
// tiles than an early one.  Then one workgroup per (64 queries, head, key
// split), 2 query halves by 2 key halves of waves.  The workgroup lists the
// key tiles that some query of it can see; a split none of them sees ends
// the workgroup before its queries are rotated.  Per listed tile:
//   - rotated keys and values go from memory straight into LDS ([key][d],
//     rows swizzled), a stage of two tiles ahead of their use;
//   - a wave forms S^T = K Q^T with v_mfma_f32_32x32x16_bf16 (its 32 rotated
//     queries are the B operand, held in registers), so a lane holds one
//     query's scores for 16 keys;
//   - online softmax in fp32: base-2 hardware exponentials of
//     score * (scale log2 e) - running maximum as one fused multiply-add
//     (weights below 2^-126 of the largest may flush to 0), the per-score
//     position test only on tiles that straddle a query of the wave;
//   - the weights rounded to bf16 as the B operand of O^T += V^T P^T; the
//     keys a lane holds are the reduction indices of its lane half, and V^T
//     comes out of LDS in the same key order through transposing reads.
// Rotations are fp32 IEEE operations rounded to bf16, as a bf16 model holds
// its rotated operands.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "device.h"
#include "attention.h"
#include "kernels.h"

namespace w4a8 {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short v4s_t __attribute__((ext_vector_type(4)));

constexpr int kD = 128;          // head dimension
constexpr int kHalf = kD / 2;    // rotate-half pairing (d, d + 64)
constexpr int kQPerWave = 32;
constexpr int kAttnWaves = 4;    // two query halves by two key halves
constexpr int kQPerBlock = 2 * kQPerWave;
constexpr int kKeys = 32;        // keys per tile

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8_t, u); }

// Maximum over the lane pair (l, l ^ 32) with the gfx950 row swap (no LDS
// round trip): the swap hands a lane its partner's value in one of the two
// results and its own in the other.  Scores are never NaN.
__device__ __forceinline__ float max_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
  return a > b ? a : b;
}

// The rotated pair chunks (8 values each at d and d + 64) of one row at
// position pos, as bf16 words: lo = a cos - b sin, hi = b cos + a sin.
__device__ __forceinline__ void rotate_chunks(uint4 a8, uint4 b8, const float* cs, const float* sn, uint4& lo,
                                              uint4& hi) {
  // three roundings per output (two products, then the sum), as in plain
  // fp32 arithmetic: no contraction into fused multiply-adds (the _rn
  // intrinsics are ordinary operators in their own scope and would be
  // contracted)
#pragma clang fp contract(off)
  const uint32_t aw[4] = {a8.x, a8.y, a8.z, a8.w}, bw[4] = {b8.x, b8.y, b8.z, b8.w};
  uint32_t lw[4], hw[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float a0 = bf16_lo(aw[e]), a1 = bf16_hi(aw[e]);
    const float b0 = bf16_lo(bw[e]), b1 = bf16_hi(bw[e]);
    const float c0 = cs[2 * e], c1 = cs[2 * e + 1], s0 = sn[2 * e], s1 = sn[2 * e + 1];
    lw[e] = bf16x2_bits(a0 * c0 - b0 * s0, a1 * c1 - b1 * s1);
    hw[e] = bf16x2_bits(b0 * c0 + a0 * s0, b1 * c1 + a1 * s1);
  }
  lo = make_uint4(lw[0], lw[1], lw[2], lw[3]);
  hi = make_uint4(hw[0], hw[1], hw[2], hw[3]);
}

// Limits of the dispatch schedule (larger calls keep the plain order).
constexpr int kSchedMaxClasses = 256;  // (query block, split) pairs
constexpr int kSchedMaxTiles = 1024;   // 32-key tiles

// The order in which the attention's workgroups take their work items.
// Workgroup ids are dealt to the CUs in rounds of C consecutive ids (id mod
// C picks the CU in the first two rounds, which are resident together), so a
// CU runs one item of each side by side; later ids go where a workgroup has
// ended.  The items are ranked by their number of
// visible key tiles (the same for every head of a (query block, split)
// pair) and dealt heaviest first, every second round in reverse: a CU that
// gets one of the heaviest items of a round gets one of the lightest of the
// next.  sched[id] = (query block * S + split) * H + head.
__device__ void build_schedule(const AttnArgs& a) {
  __shared__ int s_qmax[kSchedMaxClasses];
  __shared__ int s_tmin[kSchedMaxTiles];
  __shared__ int s_vis[kSchedMaxClasses];
  __shared__ int s_class_of_rank[kSchedMaxClasses];
  const int tid = threadIdx.x;
  const int X = (a.Nq + kQPerBlock - 1) / kQPerBlock, ntiles = (a.Nk + kKeys - 1) / kKeys;
  const int S = a.S, n = X * S, H = a.H;
  // Each block's largest query position and each tile's smallest key
  // position: 16 lanes fold a block's 64 and 8 lanes a tile's 32 (four each)
  // with shuffles.  (One LDS atomic per position took 5.6 us of the 9 us
  // that this kernel took on the 4 x 4 x 192 window.)
  auto load4 = [](const int* p, int i, int n, int none) {
    return make_int4(i < n ? p[i] : none, i + 1 < n ? p[i + 1] : none, i + 2 < n ? p[i + 2] : none,
                     i + 3 < n ? p[i + 3] : none);
  };
  const int span = max(X * 16, ntiles * 8);
  for (int i0 = tid; i0 < span; i0 += 256 * 4) {
    int4 q4[4], k4[4];  // every load of a batch goes out first
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = (i0 + 256 * b) * 4;
      q4[b] = load4(a.pos_q, i, a.Nq, INT_MIN);
      k4[b] = load4(a.pos_k, i, a.Nk, INT_MAX);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = i0 + 256 * b;
      int mx = max(max(q4[b].x, q4[b].y), max(q4[b].z, q4[b].w)), mn = min(min(k4[b].x, k4[b].y), min(k4[b].z, k4[b].w));
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) mx = max(mx, __shfl_xor(mx, off, 64));
#pragma unroll
      for (int off = 4; off >= 1; off >>= 1) mn = min(mn, __shfl_xor(mn, off, 64));
      if ((tid & 15) == 0 && i / 16 < X) s_qmax[i / 16] = mx;
      if ((tid & 7) == 0 && i / 8 < ntiles) s_tmin[i / 8] = mn;
    }
  }
  __syncthreads();
  // visible tiles of each (block, split) class, 8 lanes to a class
  const int tps = a.tiles_per_split;
  for (int i0 = 0; i0 < n * 8; i0 += 256) {
    const int c = (i0 + tid) >> 3;
    int cnt = 0;
    if (c < n) {
      const int qm = s_qmax[c / S], t0 = (c % S) * tps, t1 = min(t0 + tps, ntiles);
#pragma unroll 4
      for (int t = t0 + (tid & 7); t < t1; t += 8) cnt += s_tmin[t] <= qm ? 1 : 0;
    }
#pragma unroll
    for (int off = 4; off >= 1; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    if ((tid & 7) == 0 && c < n) s_vis[c] = cnt;
  }
  __syncthreads();
  // a block whose keys only one split sees: that split writes the output
  // itself and the merge skips the block's rows
  for (int x = tid; x < X; x += 256) {
    int only = -1, cnt = 0;
    for (int z = 0; z < S; ++z)
      if (s_vis[x * S + z] > 0) {
        ++cnt;
        only = z;
      }
    a.solo[x] = cnt == 1 ? only : -1;
  }
  // rank of each class: heavier first, ties in class order
  for (int c = tid; c < n; c += 256) {
    const int vc = s_vis[c];
    int r = 0;
#pragma unroll 8
    for (int c2 = 0; c2 < n; ++c2) {
      const int v2 = s_vis[c2];
      r += (v2 > vc || (v2 == vc && c2 < c)) ? 1 : 0;
    }
    s_class_of_rank[r] = c;
  }
  __syncthreads();
  // item k of the ranked list is class s_class_of_rank[k / H], head k % H
  const int G = n * H, C = a.sched_cus;
  for (int k = tid; k < G; k += 256) {
    const int r = k / H, h = k - r * H;
    const int round = k / C, p = k - round * C;
    const bool reversed = (round & 1) && (round + 1) * C <= G;  // a partial last round keeps its order
    a.sched[round * C + (reversed ? C - 1 - p : p)] = s_class_of_rank[r] * H + h;
  }
}

constexpr int kRotHeads = 2;  // kv heads per thread of the key rotation

// The keys rotated at their window positions: k_rot[hk][j] from k[hk][j]
// and pos_k[j], one 16-byte pair of chunks (d = 8 c .., 64 + 8 c ..) of
// kRotHeads kv heads per thread (one read of the table row), 32 keys per
// workgroup.  Rotating each key once here instead of in every workgroup
// that stages it (all query blocks of the kv head's query heads) took
// 21 us off the bench workload's 114 us.  The first row of workgroups also
// records each tile's key-position bounds, and one more workgroup, past
// the last tile, builds the dispatch schedule.
__global__ __launch_bounds__(256) void rotate_keys(const AttnArgs a) {
  const int tid = threadIdx.x, hk = blockIdx.y;
  if ((int)blockIdx.x * kKeys >= a.Nk) {  // the column past the last tile: the schedule
    if (hk == 0) build_schedule(a);
    return;
  }
  if (hk == 0 && tid < 64) {
    // the tile's smallest and largest key positions (keys past Nk count as
    // unseen), read by every workgroup of the attention for its skip and
    // mask tests
    const int jj = blockIdx.x * kKeys + (tid & (kKeys - 1));
    int mn = jj < a.Nk ? a.pos_k[jj] : INT_MAX, mx = mn;
#pragma unroll
    for (int off = kKeys / 2; off >= 1; off >>= 1) {
      mn = min(mn, __shfl_xor(mn, off, 64));
      mx = max(mx, __shfl_xor(mx, off, 64));
    }
    if (tid == 0) a.tile_bounds[blockIdx.x] = make_int2(mn, mx);
  }
  const int j = blockIdx.x * kKeys + (tid >> 3), c = tid & 7;
  if (j >= a.Nk) return;
  const int P = a.n_pos, p = a.pos_k[j];
  const int pc = p < 0 ? 0 : (p >= P ? P - 1 : p);  // table reads stay in bounds
  // kRotHeads kv heads per thread share one read of the table row
  const int h0 = hk * kRotHeads, nh = min(kRotHeads, a.Hkv - h0);
  uint4 x0[kRotHeads], x1[kRotHeads];
#pragma unroll
  for (int i = 0; i < kRotHeads; ++i)
    if (i < nh) {
      const uint16_t* src = a.k + ((size_t)(h0 + i) * a.Nk + j) * kD;
      x0[i] = *reinterpret_cast<const uint4*>(src + 8 * c);
      x1[i] = *reinterpret_cast<const uint4*>(src + kHalf + 8 * c);
    }
  float cs[8], sn[8];
  {
    const float4* cp = reinterpret_cast<const float4*>(a.rope_cos + (size_t)pc * kHalf + 8 * c);
    const float4* sp = reinterpret_cast<const float4*>(a.rope_sin + (size_t)pc * kHalf + 8 * c);
    const float4 c0 = cp[0], c1 = cp[1], s0 = sp[0], s1 = sp[1];
    cs[0] = c0.x; cs[1] = c0.y; cs[2] = c0.z; cs[3] = c0.w; cs[4] = c1.x; cs[5] = c1.y; cs[6] = c1.z; cs[7] = c1.w;
    sn[0] = s0.x; sn[1] = s0.y; sn[2] = s0.z; sn[3] = s0.w; sn[4] = s1.x; sn[5] = s1.y; sn[6] = s1.z; sn[7] = s1.w;
  }
#pragma unroll
  for (int i = 0; i < kRotHeads; ++i)
    if (i < nh) {
      uint4 lo, hi;
      rotate_chunks(x0[i], x1[i], cs, sn, lo, hi);
      uint16_t* dst = a.k_rot + ((size_t)(h0 + i) * a.Nk + j) * kD;
      *reinterpret_cast<uint4*>(dst + 8 * c) = lo;
      *reinterpret_cast<uint4*>(dst + kHalf + 8 * c) = hi;
    }
}

// Key tiles of a split whose visible ones are listed (longer splits visit
// every tile and test every score).
constexpr int kMaxSkipTiles = 512;

constexpr int kStageTiles = 2;                     // key tiles per LDS stage, one per key group of waves
constexpr int kTileBytes = kKeys * kD * 2;         // one tile of keys or values, 8 KiB
constexpr int kStageKV = kStageTiles * kTileBytes; // a stage's keys (or values)
constexpr int kPosBytes = 256;                     // a wave's copy of its tile's key positions (128 bytes; one load fills 256)
// LDS: the keys of two stages, their values, their key positions, then the
// list of visible tiles; the halves' merge reuses the keys and values.
constexpr int kLdsV = 2 * kStageKV, kLdsPos = 2 * kLdsV, kLdsList = kLdsPos + 2 * kAttnWaves * kPosBytes;
constexpr int kLdsAttn = kLdsList + kMaxSkipTiles * 2;
static_assert(kMaxSkipTiles <= 512, "a list entry holds 9 bits of tile number");

// One workgroup per (64 queries, head, key split), 4 waves: a wave owns the
// 32 queries of half qh and every second visible key tile (kh); the two key
// halves meet in LDS at the end.  What bounds it is feeding the operands
// (the L2-to-LDS fill reaches ~60 GB/s per CU beside matrix instructions;
// LDS serves 128 bytes a clock) and the vector instructions of the softmax,
// which take 4 cycles each while a matrix instruction runs.  So a key or
// value fragment read from LDS feeds 32 queries, the tiles go from memory
// straight into the LDS stage (no registers), and the softmax rescales
// only where a maximum moves (below).  The 4 x 4 x 192 window with 32 heads took
// 65.7 us with 16 queries a wave and values transposed through registers and
// 50.6 us so, in two key splits with a merge of 5.1 us; 49.8 us with the
// queries rotated once a workgroup, without splits.  (Two heads of a kv head
// per workgroup of 8 waves halve the fill and took 43 us: one workgroup per
// CU, whose waves all wait at once.)
// Rows are swizzled by the fetching lanes:
//   keys    16-byte chunk c of key j at c ^ (j & 15): the 16 keys that an
//           operand read touches at once lie on 16 distinct chunks;
//   values  chunk c of key j at c ^ 4 (j & 3): the transposed read takes 4
//           chunks of 4 consecutive keys at once.
// The values' operand (d by key) comes out of the row-major tile with the
// transposing LDS read.  The scores of the next stage are formed under this
// stage's softmax, so the keys run one stage ahead of the values.
__global__ __launch_bounds__(kAttnWaves * 64, 2) void stream_attention(const AttnArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ int l_qmax[2], l_qmin[2];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qh = wave & 1, kh = wave >> 1;  // query half, key half
  int xb = blockIdx.x, h = blockIdx.y, split = blockIdx.z;  // this workgroup's item
  if (a.sched) {  // a 1-D grid dealt by the schedule
    // Ids go round robin over the 8 XCDs: within a run of H ids (the heads
    // of one class) id t takes the head of id (t % 8) (H / 8) + t / 8, so
    // that an XCD works on neighbouring heads, whose keys its L2 then holds
    // once.
    int id = blockIdx.x;
    if ((a.H & 7) == 0) {
      const int t = id % a.H;
      id += (t & 7) * (a.H >> 3) + (t >> 3) - t;
    }
    const int code = a.sched[id], c = code / a.H;
    h = code % a.H;
    xb = c / a.S;
    split = c % a.S;
  }
  // this split alone sees keys of the block: it writes the output itself
  const bool final_out = a.S == 1 || (a.sched && a.solo[xb] == split);
  const int hk = h / (a.H / a.Hkv);
  const int l32 = lane & 31, hi = lane >> 5;
  const int P = a.n_pos;
  auto clamp_pos = [&](int p) { return p < 0 ? 0 : (p >= P ? P - 1 : p); };  // table reads stay in bounds

  // ---- this lane's query
  const int qi = xb * kQPerBlock + qh * kQPerWave + l32;
  const bool q_ok = qi < a.Nq;
  // Everything that the item alone decides is requested at once: the query's
  // position, the split's first tile bounds, the query.
  const int pq = q_ok ? a.pos_q[qi] : INT_MIN;
  const int ntiles_all = (a.Nk + kKeys - 1) / kKeys;
  const int t_begin = split * a.tiles_per_split;
  const int t_end = min(ntiles_all, t_begin + a.tiles_per_split);
  const int2 bounds0 = a.tile_bounds[min(t_begin + lane, ntiles_all - 1)];
  // The workgroup rotates its 64 queries once, 4 threads to a query, the
  // pairs of chunks (8 p, 64 + 8 p), p = c and c + 4, to thread c, and hands
  // them round through LDS: loaded by each wave as its operands, the table
  // rows and queries took twice the loads, each over 32 rows.  Rows past Nq
  // and keys past Nk are out-of-range buffer offsets, which read zeros.
  const __amdgpu_buffer_rsrc_t qres = make_rsrc(a.q + (size_t)h * a.Nq * kD, (uint32_t)((size_t)a.Nq * kD * 2));
  const int rq = tid >> 2, rch = tid & 3;  // this thread's row and chunk in the rotation
  const int rqi = xb * kQPerBlock + rq;
  const int rpos = rqi < a.Nq ? clamp_pos(a.pos_q[rqi]) : 0;
  uint4 qraw[2][2];  // rotated once the block is known to see a key
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int e = 0; e < 2; ++e)
      qraw[u][e] = buf_load16(qres, rqi < a.Nq ? (uint32_t)((rqi * kD + 8 * (rch + 4 * u) + kHalf * e) * 2) : kOOB);
  float4 rc[2][2], rs[2][2];  // the table row (requested before the list is made)
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const size_t at = (size_t)rpos * kHalf + 8 * (rch + 4 * u) + 4 * e;
      rc[u][e] = *reinterpret_cast<const float4*>(a.rope_cos + at);
      rs[u][e] = *reinterpret_cast<const float4*>(a.rope_sin + at);
    }

  // ---- this workgroup's key tiles (its split of the key range): the list
  // of those that some query of the block sees (a tile whose smallest key
  // position lies above the largest query position is left out); bits 0-8
  // the tile within the split, bit 9 + q: every key of it is seen by every
  // query of half q (never of the tile that the cache ends in: the keys past
  // Nk have the largest position, which a query may have too)
  const bool listed = t_end - t_begin <= kMaxSkipTiles;
  uint16_t* list = reinterpret_cast<uint16_t*>(lds + kLdsList);
  {
    int qm = pq, qn = q_ok ? pq : INT_MAX;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) {
      qm = max(qm, __shfl_xor(qm, off, 64));
      qn = min(qn, __shfl_xor(qn, off, 64));
    }
    if (lane == 0 && kh == 0) {
      l_qmax[qh] = qm;
      l_qmin[qh] = qn;  // INT_MAX when the half has no query
    }
  }
  lds_barrier();
  const int wg_qmax = max(l_qmax[0], l_qmax[1]), qmin0 = l_qmin[0], qmin1 = l_qmin[1];
  int n_vis = t_end - t_begin;
  if (listed) {
    n_vis = 0;
    for (int t0 = t_begin; t0 < t_end; t0 += 64) {  // every wave counts; each fourth batch is one wave's to write
      const int t = t0 + lane;
      const int2 bd = t0 == t_begin ? bounds0 : a.tile_bounds[min(t, ntiles_all - 1)];
      const bool vis = t < t_end && bd.x <= wg_qmax;
      const uint64_t m = __ballot(vis);
      const bool whole = (t + 1) * kKeys <= a.Nk;
      if (vis && wave == ((t0 - t_begin) >> 6) % kAttnWaves)
        list[n_vis + __popcll(m & ((1ull << lane) - 1))] =
            (uint16_t)((t - t_begin) | (whole && bd.y <= qmin0 ? 512 : 0) | (whole && bd.y <= qmin1 ? 1024 : 0));
      n_vis += (int)__popcll(m);
    }
    n_vis = __builtin_amdgcn_readfirstlane(n_vis);
  }
  if (a.S > 1 && n_vis == 0) {
    // no query of the block sees a key of this split: an empty partial
    // (the merge reads only its maximum)
    if (q_ok && hi == 0 && kh == 0)
      *reinterpret_cast<float2*>(a.part_ml + (((size_t)split * a.H + h) * a.Nq + qi) * 2) = make_float2(-INFINITY, 0.0f);
    return;
  }
  lds_barrier();  // the list

  // ---- staging.  A stage takes the next two listed tiles, kh = 0 and 1 of
  // them computed by the waves of that key half, and the waves of a key half
  // fetch its tile: kRows rows each of the keys and of the values, 4 rows
  // (1 KiB of LDS) per instruction: lane l is row l / 16's chunk l % 16 of
  // LDS.
  constexpr int kRows = kKeys / 2, kLoads = kRows / 4;
  static_assert(kLoads == 4, "a stage deals its loads one to a slot");
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  const u32x4 k_res = make_rsrc_words(a.k_rot + (size_t)hk * a.Nk * kD, (uint32_t)((size_t)a.Nk * kD * 2));
  const u32x4 v_res = make_rsrc_words(a.v + (size_t)hk * a.Nk * kD, (uint32_t)((size_t)a.Nk * kD * 2));
  const int r4 = lane >> 4, c16 = lane & 15;
  const int row0 = kRows * qh;  // first row of the tile that this wave fetches
  uint32_t k_voff[kLoads];
#pragma unroll
  for (int n = 0; n < kLoads; ++n) {
    const int row = row0 + 4 * n + r4;
    k_voff[n] = (uint32_t)(row * 256 + ((c16 ^ (row & 15)) << 4));
  }
  const uint32_t v_voff = (uint32_t)((row0 + r4) * 256 + ((c16 ^ (4 * r4)) << 4));
  // The wave's tile of the stage of visible tiles i, i + 1, as listed (a
  // value every lane holds; made scalar where it is used, a stage later, so
  // that nothing waits for the LDS read).
  const int last_entry = max(min(n_vis, kMaxSkipTiles) - 1, 0);
  auto tile_at = [&](int i) {
    const int e = list[min(i + kh, last_entry)];  // read in any case: no branch
    return listed ? e : i + kh;
  };
  auto scalar = [](int e) { return (int)__builtin_amdgcn_readfirstlane(e); };
  auto tile_of = [&](int e) { return t_begin + (listed ? e & 511 : e); };
  const int full_bit = listed ? 512 << qh : 0;
  const u32x4 pos_res = make_rsrc_words(a.pos_k, (uint32_t)(a.Nk * 4));
  // Byte offset of the tile's rows in the head's keys and values.  Rows past
  // Nk lie past the buffers and read zeros; so do all rows of a tile past
  // the last visible one, without traffic.
  auto tile_off = [&](int i, int e) { return i + kh < n_vis ? (uint32_t)(tile_of(e) * kTileBytes) : kOOB; };
  const uint32_t my_rows = lds_base + (uint32_t)(kh * kTileBytes + row0 * 256);
  auto issue_keys = [&](int b, int n, uint32_t off) {
    lds_dma16(k_res, my_rows + (uint32_t)(b * kStageKV + n * 1024), k_voff[n] + off, 0);
  };
  auto issue_values = [&](int b, int n, uint32_t off) {
    lds_dma16(v_res, my_rows + (uint32_t)(kLdsV + b * kStageKV + n * 1024), v_voff + n * 1024 + off, 0);
  };
  auto issue_pos = [&](int b, uint32_t off) {
    lds_dma4(pos_res, lds_base + (uint32_t)(kLdsPos + (kAttnWaves * b + wave) * kPosBytes),
             hi == 0 ? (off == kOOB ? kOOB : off / (kTileBytes / (kKeys * 4))) + l32 * 4 : kOOB, 0);
  };

  int cur = scalar(tile_at(0)), nxt = scalar(tile_at(kStageTiles)), ahead = tile_at(2 * kStageTiles);
#pragma unroll
  for (int n = 0; n < kLoads; ++n) issue_keys(0, n, tile_off(0, cur));

  // The rotated queries, laid out as two tiles of keys, where the second
  // stage's values come later (the scale's sign goes into the rotation's
  // factors: 1 and -1 are exact, and with 0 every score of finite operands
  // is 0).
  uint8_t* l_q = lds + kLdsV + kStageKV;
  static_assert(kQPerBlock * kD * 2 <= kStageKV, "the queries fit a stage's values");
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float cs[8] = {rc[u][0].x, rc[u][0].y, rc[u][0].z, rc[u][0].w, rc[u][1].x, rc[u][1].y, rc[u][1].z, rc[u][1].w};
    float sn[8] = {rs[u][0].x, rs[u][0].y, rs[u][0].z, rs[u][0].w, rs[u][1].x, rs[u][1].y, rs[u][1].z, rs[u][1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      cs[e] *= a.q_sign;
      sn[e] *= a.q_sign;
    }
    uint4 lo, hi4;
    rotate_chunks(qraw[u][0], qraw[u][1], cs, sn, lo, hi4);
    const int ch = rch + 4 * u, sw = rq & 15;
    *reinterpret_cast<uint4*>(l_q + rq * 256 + ((ch ^ sw) << 4)) = lo;
    *reinterpret_cast<uint4*>(l_q + rq * 256 + (((ch + 8) ^ sw) << 4)) = hi4;
  }

  // This lane's query as the B operand of S^T = K Q^T (query l32,
  // d = 16 i + 8 hi .. for MFMA i), read behind the first keys' barrier.
  bf16x8_t qf[8];
  f32x16_t acc[kD / 32];
#pragma unroll
  for (int t = 0; t < kD / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
  float m = -INFINITY, tmax = -INFINITY;
  float ls[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // the weights' total, in four chains
  // (in a vector register: a scalar operand halves the rate of an fma)
  float sl2 = a.scale_log2e;
  asm volatile("" : "+v"(sl2));

  // LDS read addresses within a stage: key l32's chunks 2 i + hi; the
  // transposed value read of (32 t, 16 j + 8 u): lane k of a 16-lane group
  // addresses row k / 4 of its four keys (16 j + 8 u + 4 hi + ..) and d
  // chunk k % 4 of its sixteen d (32 t + 16 (group & 1) + ..), and receives
  // the four keys of d = 32 t + l32.
  uint32_t k_rd[4];  // MFMAs i and i + 4 are 8 chunks apart
#pragma unroll
  for (int i = 0; i < 4; ++i) k_rd[i] = (uint32_t)(kh * kTileBytes + l32 * 256 + (((2 * i + hi) ^ (l32 & 15)) << 4));
  const int vr = (lane & 15) >> 2;                                    // key row of the four
  const int vch = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);          // 16-byte chunk within 32 t's four
  __attribute__((address_space(3))) uint8_t* v_rd[kD / 32];
#pragma unroll
  for (int t = 0; t < kD / 32; ++t)
    v_rd[t] = (__attribute__((address_space(3))) uint8_t*)lds + kLdsV + kh * kTileBytes + (4 * hi + vr) * 256 +
              ((4 * (t ^ vr) + vch) << 4) + 8 * (lane & 1);

  // Fragment i of the keys of stage b (a constant: the immediate offset)
  auto key_frag = [&](int b, int i) {
    return as_bf16x8(*reinterpret_cast<const uint4*>(lds + (i < 4 ? k_rd[i & 3] : k_rd[i & 3] ^ 128u) + b * kStageKV));
  };
  // Stage b holds visible tiles i, i + 1, whose scores are in s: score 4 q +
  // r is key 8 q + 4 hi + r of the wave's tile, raw (the scale is applied
  // inside the exponent).  Unless it is the last, the next stage's scores
  // are formed into sn.  One barrier per stage: the wait and the barrier
  // publish this stage's values and the next stage's keys (every wave's
  // share has landed) and say that the last stage's values and this stage's
  // keys are no longer read, so their refills go out under this stage's
  // compute.
  // The waves pass their phases together, so each wave's own matrix
  // instructions are dealt out between its vector instructions (slots kept
  // apart by scheduling barriers): the next scores' and the first half of
  // the values' under the exponentials, the rest under the next maximum.
  // In one block each the two units took turns: 43 % and 24 % busy, 1470
  // cycles a tile and wave pair.
  // The running maximum m is the offset of the exponents.  The sums are
  // rescaled only where some query of the wave has a new one: 64 multiplies,
  // a quarter of a tile's vector cycles, and none for most tiles once the
  // maxima have settled.  (Letting scores exceed m by up to 2^8 before it
  // moves took 3 us off the 4 x 4 x 192 window, but the largest weights then
  // lie anywhere in their binade and not just below a power of two: the
  // bf16 weights' error grew, 2.2e-3 to 2.3e-3 of the output.)
  auto max16 = [](const f32x16_t& s) {  // three levels deep: a dependent instruction costs 8 cycles
    auto max3 = [](float x, float y, float z) { return fmaxf(fmaxf(x, y), z); };
    const float u0 = max3(s[0], s[1], s[2]), u1 = max3(s[3], s[4], s[5]), u2 = max3(s[6], s[7], s[8]),
                u3 = max3(s[9], s[10], s[11]), u4 = max3(s[12], s[13], s[14]);
    return fmaxf(max3(u0, u1, u2), max3(u3, u4, s[15]));
  };
  auto stage_step = [&](auto b_c, auto last_c, int i, f32x16_t& s, f32x16_t& sn) {
    constexpr int b = decltype(b_c)::value;
    constexpr bool last = decltype(last_c)::value;
    wait_vmcnt<0>();
    lds_barrier();
    const int nxt2 = scalar(ahead);
    const uint32_t v_off = tile_off(i + kStageTiles, nxt), k_off = tile_off(i + 2 * kStageTiles, nxt2);
    const bool on = i + kh < n_vis;  // the last stage may hold one tile
    if (!(on && (cur & full_bit))) {
      // the position test per score only where some key of the tile lies
      // beyond some query of the wave (or past Nk)
      const int* pos = reinterpret_cast<const int*>(lds + kLdsPos + (kAttnWaves * b + wave) * kPosBytes);
      const int left = on ? a.Nk - tile_of(cur) * kKeys : 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int4 p4 = *reinterpret_cast<const int4*>(pos + 8 * q + 4 * hi);
        const int pp[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (pp[r] > pq || 8 * q + 4 * hi + r >= left) s[4 * q + r] = -INFINITY;
      }
      tmax = max16(s);
    }
    bf16x8_t kf[8];
    if constexpr (!last) {
#pragma unroll
      for (int q = 0; q < 8; ++q) kf[q] = key_frag(b ^ 1, q);
      issue_pos(b ^ 1, v_off);
    }
    // ---- online softmax over this lane's query (its 16 keys here, the
    // other 16 in lane ^ 32), in scaled base-2 units: sl2 is positive, so
    // the largest raw score gives the largest scaled one and -inf stays -inf
    const float top = max_xor32(tmax) * sl2;
    if (__any(top > m)) {
      const float mnew = fmaxf(m, top);
      // (while nothing is visible yet m stays -inf and all sums are 0)
      const float alpha = mnew == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - mnew);
#pragma unroll
      for (int r = 0; r < 4; ++r) ls[r] *= alpha;
#pragma unroll
      for (int t4 = 0; t4 < kD / 32; ++t4)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t4][r] *= alpha;
      m = mnew;
    }
    // exponent offset: while nothing is visible yet the masked scores
    // (-inf) must still give 0
    const float mb = m == -INFINITY ? 0.0f : m;
    if constexpr (!last) ahead = tile_at(i + 3 * kStageTiles);
    // The weights go through three steps a slot or more apart, so that none
    // waits for the one before: exponent (fma), exponential, then the sum
    // and the rounding to bf16.
    uint32_t pw[8];  // weights, two to a word
    auto expo = [&](int r) { s[r] = __builtin_fmaf(s[r], sl2, -mb); };
    auto weigh = [&](int r) { s[r] = __builtin_amdgcn_exp2f(s[r]); };
    auto close = [&](int w) {
      ls[(2 * w) & 3] += s[2 * w];
      ls[(2 * w + 1) & 3] += s[2 * w + 1];
      pw[w] = bf16x2_bits(s[2 * w], s[2 * w + 1]);
    };
    union { v4s_t h[2]; bf16x8_t v; } vf[kD / 32][2];
    auto next_score = [&](int q) {
      if constexpr (!last) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[q], qf[q], q == 0 ? f32x16_t{} : sn, 0, 0, 0);
    };
    auto value_frag = [&](int t4, int j) {  // d block t4, keys 16 j + 8 u + 4 hi ..
#pragma unroll
      for (int u = 0; u < 2; ++u)
        vf[t4][j].h[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) v4s_t*)(v_rd[t4] + (b * kStageKV + (16 * j + 8 * u) * 256)));
    };
#pragma unroll
    for (int r = 0; r < 6; ++r) expo(r);
    weigh(0);
    weigh(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // weights 0 - 7
      next_score(q);
      if constexpr (!last)
        issue_values(b ^ 1, q, v_off);
      value_frag(q, 0);
      weigh(2 * q + 2);
      weigh(2 * q + 3);
      expo(2 * q + 6);
      expo(2 * q + 7);
      close(q);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- O^T += V^T P^T: the weights are the B operand of MFMA j: elements
    // 0-3 are keys 16 j + 4 hi .., 4-7 keys 16 j + 8 + 4 hi ..
    const bf16x8_t pb0 = as_bf16x8(make_uint4(pw[0], pw[1], pw[2], pw[3]));
    expo(14);
    expo(15);
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // weights 8 - 15
      next_score(4 + q);
      if constexpr (!last)
        issue_keys(b, q, k_off);
      if (q < 3) weigh(10 + 2 * q);
      if (q > 0) close(3 + q);
      __builtin_amdgcn_sched_barrier(0);
      acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[q][0].v, pb0, acc[q], 0, 0, 0);
      value_frag(q, 1);
      if (q < 3) weigh(11 + 2 * q);
      if (q == 3) close(7);
      __builtin_amdgcn_sched_barrier(0);
    }
    const bf16x8_t pb1 = as_bf16x8(make_uint4(pw[4], pw[5], pw[6], pw[7]));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[q][1].v, pb1, acc[q], 0, 0, 0);
      if constexpr (!last)
        if (q == 2) {
          tmax = max16(sn);
          asm volatile("" : "+v"(tmax));  // here, under the matrix instructions
        }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) asm volatile("" : "+v"(ls[r]));
    cur = nxt;
    nxt = nxt2;
  };
  if (n_vis > 0) {
    constexpr std::integral_constant<int, 0> b0{};
    constexpr std::integral_constant<int, 1> b1{};
    f32x16_t s0, s1;
    wait_vmcnt<0>();
    lds_barrier();  // the first keys and the queries are there
#pragma unroll
    for (int i = 0; i < 8; ++i)
      qf[i] = as_bf16x8(*reinterpret_cast<const uint4*>(l_q + (qh * kQPerWave + l32) * 256 + (((2 * i + hi) ^ (l32 & 15)) << 4)));
#pragma unroll
    for (int n = 0; n < kLoads; ++n) {
      issue_values(0, n, tile_off(0, cur));
      issue_keys(1, n, tile_off(kStageTiles, nxt));
    }
    issue_pos(0, tile_off(0, cur));
#pragma unroll
    for (int q = 0; q < 8; ++q)
      s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(key_frag(0, q), qf[q], q == 0 ? f32x16_t{} : s0, 0, 0, 0);
    tmax = max16(s0);
    int i = 0;
    for (; i + 2 * kStageTiles < n_vis; i += 2 * kStageTiles) {
      stage_step(b0, std::false_type{}, i, s0, s1);
      stage_step(b1, std::false_type{}, i + kStageTiles, s1, s0);
    }
    if (i + kStageTiles < n_vis) {
      stage_step(b0, std::false_type{}, i, s0, s1);
      stage_step(b1, std::true_type{}, i + kStageTiles, s1, s0);
    } else {
      stage_step(b0, std::true_type{}, i, s0, s1);
    }
  }

  // ---- the two key halves of each query group meet: wave kh finishes d
  // blocks 2 kh, 2 kh + 1 and hands the others, with its maximum and weight
  // total, to its partner through the idle stages
  float lsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
  lsum += __shfl_xor(lsum, 32, 64);
  wait_vmcnt<0>();
  lds_barrier();  // every wave is done with the stages
  float* xo = reinterpret_cast<float*>(lds) + wave * (32 * 64);  // 8 KiB per wave
  float* xml = reinterpret_cast<float*>(lds + kAttnWaves * 8192);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) xo[(16 * u + r) * 64 + lane] = kh == 0 ? acc[2 + u][r] : acc[u][r];
  if (hi == 0) *reinterpret_cast<float2*>(xml + (wave * 32 + l32) * 2) = make_float2(m, lsum);
  lds_barrier();
  const int other = wave ^ 2;
  const float2 ml2 = *reinterpret_cast<const float2*>(xml + (other * 32 + l32) * 2);
  const float mt = fmaxf(m, ml2.x), mtb = mt == -INFINITY ? 0.0f : mt;
  const float w0 = __builtin_amdgcn_exp2f(m - mtb), w1 = __builtin_amdgcn_exp2f(ml2.x - mtb);
  const float l = lsum * w0 + ml2.y * w1;
  const float* xr = reinterpret_cast<const float*>(lds) + other * (32 * 64);
  float o[2][16];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[u][r] = (kh == 0 ? acc[u][r] : acc[2 + u][r]) * w0 + xr[(16 * u + r) * 64 + lane] * w1;

  // ---- O = O^T / l: lane holds query l32, d = 32 (2 kh + u) + 8 q + 4 hi + r
  if (!q_ok) return;
  if (!final_out) {
    // a split's partial result: the unnormalized sum, its running maximum
    // (base 2, scaled scores) and weight total; attn_combine merges them
    const size_t row = ((size_t)split * a.H + h) * a.Nq + qi;
    float* po = a.part_o + row * kD + 64 * kh + 4 * hi;
    if (mt != -INFINITY)  // the merge reads no sum of a split that saw nothing
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(po + 32 * u + 8 * q) = make_float4(o[u][4 * q], o[u][4 * q + 1], o[u][4 * q + 2], o[u][4 * q + 3]);
    if (hi == 0 && kh == 0) *reinterpret_cast<float2*>(a.part_ml + row * 2) = make_float2(mt, l);
    return;
  }
  const float inv = l > 0.0f ? __fdiv_rn(1.0f, l) : 0.0f;  // a query that sees no key gets 0
  uint16_t* orow = a.o + ((size_t)h * a.Nq + qi) * kD + 64 * kh + 4 * hi;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint2 w = make_uint2(bf16x2_bits(o[u][4 * q] * inv, o[u][4 * q + 1] * inv),
                                 bf16x2_bits(o[u][4 * q + 2] * inv, o[u][4 * q + 3] * inv));
      *reinterpret_cast<uint2*>(orow + 32 * u + 8 * q) = w;
    }
}

// Merge of the splits' partial results: thread per (head, query, 8 of d).
__global__ __launch_bounds__(256) void attn_combine(const AttnArgs a) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t rows = (size_t)a.H * a.Nq;
  if (idx >= rows * (kD / 8)) return;
  const size_t row = idx / (kD / 8);
  const int c = (int)(idx % (kD / 8));
  if (a.sched && a.solo[(int)(row % (size_t)a.Nq) / kQPerBlock] >= 0) return;  // written by its only split
  float mmax = -INFINITY;
  for (int s = 0; s < a.S; ++s) mmax = fmaxf(mmax, a.part_ml[((size_t)s * rows + row) * 2]);
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, l = 0.0f;
  if (mmax != -INFINITY) {
    for (int s = 0; s < a.S; ++s) {
      const float2 ml = *reinterpret_cast<const float2*>(a.part_ml + ((size_t)s * rows + row) * 2);
      if (ml.x == -INFINITY) continue;  // the split saw no key of this query
      const float wgt = exp2f(ml.x - mmax);
      l += ml.y * wgt;
      const float4* po = reinterpret_cast<const float4*>(a.part_o + ((size_t)s * rows + row) * kD + 8 * c);
      const float4 u0 = po[0], u1 = po[1];
      o[0] += u0.x * wgt; o[1] += u0.y * wgt; o[2] += u0.z * wgt; o[3] += u0.w * wgt;
      o[4] += u1.x * wgt; o[5] += u1.y * wgt; o[6] += u1.z * wgt; o[7] += u1.w * wgt;
    }
  }
  const float inv = l > 0.0f ? __fdiv_rn(1.0f, l) : 0.0f;
  *reinterpret_cast<uint4*>(a.o + row * kD + 8 * c) =
      make_uint4(bf16x2_bits(o[0] * inv, o[1] * inv), bf16x2_bits(o[2] * inv, o[3] * inv),
                 bf16x2_bits(o[4] * inv, o[5] * inv), bf16x2_bits(o[6] * inv, o[7] * inv));
}

}  // namespace

// Key-range splits (1, 2, 4 or 8, of at least 8 tiles): the heaviest workgroups, whose queries see
// the whole window, otherwise run every tile in series; each split costs a
// prologue and its partial sums' way through memory.  The least of, in ns,
//   the longer of 400 a tile of the heaviest workgroup and 1 a tile of all
//   (256 CUs, the two workgroups that fit one, ~60 % of the keys visible),
//   and with splits 1000 for the merge and 20 a workgroup.
// Fitted to S = 1, 2, 4, 8 of 80 windows (1 - 6 views, 2 - 6 frames, 16 - 256
// tokens, 8 - 32 heads): 0.8 % above the best S on average, 8 % at most.
// (Splitting up to 4 workgroups a CU, as when that many fitted, took 8 %
// more.)  us at S = 1, 2, 4, 8: 4 x 4 x 192 on 32 heads (384 blocks, 96
// tiles) 51.8 54.2 61.0 80.1; 2 x 4 x 192 on 32 (192, 48) 30.5 31.2 37.5
// 45.8; 4 x 6 x 128 on 32 (256, 96) 54.8 42.4 51.5 59.8; 4 x 4 x 192 on 8
// (96, 96) 48.1 35.5 31.6 35.9; 1 x 16 x 256 on 8 (32, 128) 65.0 42.8 31.4
// 28.6.
int stream_attention_splits(int H, int Nq, int Nk) {
  const int64_t blocks = (int64_t)((Nq + kQPerBlock - 1) / kQPerBlock) * H, ntiles = (Nk + kKeys - 1) / kKeys;
  int best = 1;
  int64_t least = INT64_MAX;
  for (int S = 1; S <= 8 && (S == 1 || ntiles / S >= 8); S *= 2) {
    const int64_t cost = std::max(400 * ntiles / S, blocks * ntiles) + (S > 1 ? 1000 + 20 * blocks * S : 0);
    if (cost < least) {
      least = cost;
      best = S;
    }
  }
  return best;
}

// Workspace, past the counter region shared with the linear calls'
// workspaces (left untouched here): the rotated keys (room for H kv heads,
// the most a call with H query heads has), then the split partials.
size_t rotated_keys_bytes(int H, int Nk) { return ((size_t)H * Nk * kD * 2 + 255) / 256 * 256; }
size_t tile_bounds_bytes(int Nk) { return ((size_t)(Nk + kKeys - 1) / kKeys * sizeof(int2) + 255) / 256 * 256; }
// The splits a call uses (the split rule, without empty trailing splits).
int used_splits(int H, int Nq, int Nk, int* tiles_per_split) {
  const int ntiles = (Nk + kKeys - 1) / kKeys;
  const int S = stream_attention_splits(H, Nq, Nk);
  const int tps = (ntiles + S - 1) / S;
  if (tiles_per_split) *tiles_per_split = tps;
  return (ntiles + tps - 1) / tps;
}
// Bytes of the dispatch schedule (0 for calls past its limits).
size_t schedule_bytes(int H, int Nq, int Nk) {
  const long classes = (long)((Nq + kQPerBlock - 1) / kQPerBlock) * used_splits(H, Nq, Nk, nullptr);
  if (classes > kSchedMaxClasses || (Nk + kKeys - 1) / kKeys > kSchedMaxTiles) return 0;
  const size_t blocks = (size_t)(Nq + kQPerBlock - 1) / kQPerBlock;
  return (((size_t)classes * H + blocks) * sizeof(int) + 255) / 256 * 256;  // the schedule, then the solo table
}
size_t stream_attention_workspace(int H, int Nq, int Nk) {
  const int S = stream_attention_splits(H, Nq, Nk);
  return kCounterRegionBytes + rotated_keys_bytes(H, Nk) + tile_bounds_bytes(Nk) + schedule_bytes(H, Nq, Nk) +
         (S > 1 ? (size_t)S * H * Nq * (kD + 2) * sizeof(float) : 0);
}

// Compute units of the current device (looked up once per device).
int compute_units() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

hipError_t launch_stream_attention(const AttnArgs& a0, hipStream_t stream) {
  if (a0.Nq == 0) return hipSuccess;
  AttnArgs a = a0;
  const int ntiles = (a.Nk + kKeys - 1) / kKeys;
  a.S = used_splits(a.H, a.Nq, a.Nk, &a.tiles_per_split);
  uint8_t* ws = static_cast<uint8_t*>(a.workspace) + kCounterRegionBytes;
  a.k_rot = reinterpret_cast<uint16_t*>(ws);
  a.tile_bounds = reinterpret_cast<int2*>(ws + rotated_keys_bytes(a.H, a.Nk));
  const size_t sched_bytes = schedule_bytes(a.H, a.Nq, a.Nk);
  // Calls of at most one workgroup per CU go without a schedule: their order
  // cannot matter, and making it is the longest chain of the first kernel,
  // reading it the first of the second.  us a call with / without: 1 x 2 x 16
  // on 8 heads 10.5 / 8.7, 2 x 2 x 40 on 16 13.5 / 11.7, 1 x 2 x 256 on 16
  // 19.2 / 17.1.
  const int64_t items = (int64_t)((a.Nq + kQPerBlock - 1) / kQPerBlock) * a.S * a.H;
  a.sched = sched_bytes && items > 256 ? reinterpret_cast<int*>(ws + rotated_keys_bytes(a.H, a.Nk) + tile_bounds_bytes(a.Nk)) : nullptr;
  a.sched_cus = compute_units();
  a.solo = a.sched ? a.sched + (size_t)((a.Nq + kQPerBlock - 1) / kQPerBlock) * a.S * a.H : nullptr;
  if (a.S > 1) {
    a.part_o = reinterpret_cast<float*>(ws + rotated_keys_bytes(a.H, a.Nk) + tile_bounds_bytes(a.Nk) + sched_bytes);
    a.part_ml = a.part_o + (size_t)a.S * a.H * a.Nq * kD;
  }
  rotate_keys<<<dim3((unsigned)(ntiles + (a.sched ? 1 : 0)), (unsigned)((a.Hkv + kRotHeads - 1) / kRotHeads)), dim3(256), 0,
                stream>>>(a);
  const unsigned X = (unsigned)((a.Nq + kQPerBlock - 1) / kQPerBlock);
  // scheduled calls (at most kSchedMaxClasses x 4096 items) take a 1-D grid
  const dim3 grid = a.sched ? dim3(X * (unsigned)a.H * (unsigned)a.S) : dim3(X, (unsigned)a.H, (unsigned)a.S);
  stream_attention<<<grid, dim3(kAttnWaves * 64), kLdsAttn, stream>>>(a);
  if (a.S > 1) {
    const size_t threads = (size_t)a.H * a.Nq * (kD / 8);
    attn_combine<<<dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream>>>(a);
  }
  return hipGetLastError();
}

}  // namespace w4a8
