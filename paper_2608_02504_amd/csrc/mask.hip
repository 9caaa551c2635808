// Token-radius block mask (App. C.1, Alg. 1) and the heaviest-first row order.
//
// One workgroup of four waves per query-block row (batch, head, u).  For a key
// column j of block v, c_j counts the valid queries i of u whose radius covers j
// (Eq. 15):
//     (x_i - x_j)^2 + (y_i - y_j)^2 <= thr[n_i][|f_i - f_j|].
// Alg. 1 evaluates every (i, j) pair and the vote needs a column with 3 c_j >
// n_u, that is c_j >= k = floor(n_u / 3) + 1 (the union rule: k = 1).  Here the
// key blocks pass three filters; each only skips work whose outcome is already
// known, so the counts -- and the mask -- are exactly Alg. 1's:
//   1. one lane per key block, bounding box of u against bounding box of v (App.
//      C.1 uses such boxes to reject whole block pairs): if the k-th largest
//      threshold of u's queries at the nearest frames does not reach the boxes'
//      distance, fewer than k queries touch v and it is dropped; if at the
//      farthest frames it covers the boxes' farthest points, k queries cover all
//      of v and it is kept (thresholds are monotone in the radius, so one query
//      is the k-th at every frame distance);
//   2. one lane per undecided block, a loop over u's queries: each query's
//      position against v's box gives the queries that cover all of v and those
//      that reach it, which decide most of the rest;
//   3. the blocks left are tested pair by pair.  2-D: E_ij = T_i(frame of j) -
//      D_ij is bilinear in per-query and per-key vectors of 8 small integers, so
//      a 32 x 32 tile of the test is one v_mfma_f32_32x32x8_f16 (exact: integers
//      of magnitude <= 2048, partial sums below 2^24; the key vectors are the
//      plan's, those of the token-level attention), the 0/1 results come from
//      v_cvt_pknorm_u16_f32 of E + 1 (clamps to [0, 1]: 0xFFFF iff E >= 0), two
//      queries an instruction, and are counted in packed 16-bit lanes.  That is
//      one vector instruction per pair and lane, where testing two partial queries
//      at a time with packed 16-bit arithmetic took 3.5 and the list of them more.
// Everything is integer arithmetic in effect.  Bound: vector instructions (the
// outputs are 68 MB at 75,600 tokens x 40 heads).  Measured there, lists at 12 % of
// the block pairs: 4.35 -> 2.05 ms; of a row's 591 blocks filter 1 leaves 219 and
// filter 2 100.  (Box tests per 32 keys before filter 3 would halve its pairs but
// cost more than that; sorting the queries by radius skips 14 % of its tiles.)
//
// Sequence-distance ablation (DIST = TRA_DIST_1D, App. C.1): a query covers
// key j iff |i - j| <= thr1[n_i][|f_i - f_j|] on raster indices; the box of a
// block is then its raster-index range, and the same arguments hold because thr1
// is non-increasing in delta and monotone in n too; its pairs, and those of blocks
// that span more than two frames, are tested one query at a time.
//
// Joint text-video attention (Sec. 3.2; Alg. 1's u >= B_v or v >= B_v branch):
// a block holding any text token is retained in every row, and the row of such
// a block retains every key block.
#include <climits>
#include <mutex>

#include "tra_internal.h"

namespace tra {
namespace {

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ int popc(uint64_t m) { return __popcll(m); }

// Distance of a token pair from its position difference: squared Euclidean
// (x, y) for 2-D, |raster difference| (carried in the first component) for 1-D.
// (Coordinate differences are below 1024 in magnitude, so 24-bit multiplies
// are exact.)
template <int DIST>
__device__ __forceinline__ int metric(int da, int db) {
  if constexpr (DIST == TRA_DIST_1D) return abs(da);
  else return __mul24(da, da) + __mul24(db, db);
}

// Position of a packed coordinate in the metric's space.
template <int DIST>
__device__ __forceinline__ void position(int32_t c, int H, int W, int* a, int* b, int* f) {
  *f = coord_f(c);
  if constexpr (DIST == TRA_DIST_1D) {
    *a = (*f * H + coord_x(c)) * W + coord_y(c);
    *b = 0;
  } else {
    *a = coord_x(c);
    *b = coord_y(c);
  }
}

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWaves = 4;

// Key block v's box in the metric's space and its counts (kBlockInfo layout).
struct Box {
  int fmin, fmax, amin, amax, bmin, bmax, n_video, n_text;
};
template <int DIST>
__device__ __forceinline__ Box load_box(const int32_t* __restrict__ binfo, int v) {
  const int32_t* bi = binfo + (size_t)v * kBlockInfo;
  constexpr bool one_d = DIST == TRA_DIST_1D;
  return Box{bi[0], bi[1], one_d ? bi[7] : bi[2], one_d ? bi[8] : bi[3], one_d ? 0 : bi[4], one_d ? 0 : bi[5],
             bi[6], bi[9]};
}

// (T - x^2 - y^2) of a query as the two f16 components (h, l) of 2048 h + l, 0 <=
// l < 2048; a query covering every key gets T = 2^22, beyond any squared
// distance on a 1023 x 1023 frame.
__device__ __forceinline__ uint32_t threshold_word(int T, int sq) {
  const int a = min(T, 1 << 22) - sq;
  const f16x2 w = {(_Float16)(a >> 11), (_Float16)(a & 2047)};
  return __builtin_bit_cast(uint32_t, w);
}

// Pair test of key block v, one query at a time (any distance, any number of
// frames): the row's queries as lanes, each first classified against v's box, then
// the partial ones broadcast to this wave's keys.  Returns Alg. 1's decision.
template <int B, int RULE, int DIST>
__device__ bool test_block_by_query(const Box& bx, int v, const int32_t* __restrict__ coord, const int32_t* s_T,
                                    const int32_t* s_c, int FS, int n_u, int H, int W, int lane) {
  constexpr int QPL = B / 64;  // queries (and keys) per lane
  int qx[QPL], qy[QPL], qf[QPL], kx[QPL], ky[QPL], kf[QPL], c[QPL];
  bool kvalid[QPL];
  uint64_t part_m[QPL];
  int n_all = 0;
#pragma unroll
  for (int s = 0; s < QPL; ++s) {
    const int qi = lane + 64 * s;
    position<DIST>(s_c[qi], H, W, &qx[s], &qy[s], &qf[s]);
    const int dxn = max(0, max(bx.amin - qx[s], qx[s] - bx.amax));
    const int dyn = max(0, max(bx.bmin - qy[s], qy[s] - bx.bmax));
    const int dxf = max(qx[s] - bx.amin, bx.amax - qx[s]);
    const int dyf = max(qy[s] - bx.bmin, bx.bmax - qy[s]);
    const int dmin = max(0, max(bx.fmin - qf[s], qf[s] - bx.fmax));
    const int dmax = max(qf[s] - bx.fmin, bx.fmax - qf[s]);
    const bool in = qi < n_u && metric<DIST>(dxn, dyn) <= s_T[qi * FS + dmin];
    const bool all = in && metric<DIST>(dxf, dyf) <= s_T[qi * FS + dmax];
    n_all += popc(ballot(all));
    part_m[s] = ballot(in && !all);
    const int j = lane + 64 * s;
    kvalid[s] = j < bx.n_video;
    position<DIST>(kvalid[s] ? coord[(size_t)v * B + j] : 0, H, W, &kx[s], &ky[s], &kf[s]);
  }
#pragma unroll
  for (int s = 0; s < QPL; ++s) c[s] = n_all;
#pragma unroll
  for (int s2 = 0; s2 < QPL; ++s2) {
    uint64_t m = part_m[s2];
    while (m) {
      const int l = __ffsll((unsigned long long)m) - 1;
      m &= m - 1;
      const int px = __builtin_amdgcn_readlane(qx[s2], l);
      const int py = __builtin_amdgcn_readlane(qy[s2], l);
      const int pf = __builtin_amdgcn_readlane(qf[s2], l);
      const int32_t* Tp = s_T + (l + 64 * s2) * FS;
#pragma unroll
      for (int s = 0; s < QPL; ++s)
        c[s] += (metric<DIST>(px - kx[s], py - ky[s]) <= Tp[abs(pf - kf[s])]) ? 1 : 0;
      if (RULE == TRA_MASK_UNION) {
        bool hit = false;
#pragma unroll
        for (int s = 0; s < QPL; ++s) hit |= kvalid[s] && c[s] > 0;
        if (ballot(hit) != 0) return true;  // one covered key decides the union
      }
    }
  }
  int nonempty = 0, high = 0;
#pragma unroll
  for (int s = 0; s < QPL; ++s) {
    nonempty += popc(ballot(kvalid[s] && c[s] > 0));
    high += popc(ballot(kvalid[s] && 3 * c[s] > n_u));
  }
  return RULE == TRA_MASK_VOTE ? (nonempty > 0 && 10 * high > 6 * nonempty) : nonempty > 0;
}

// Pair test of key block v (2-D, at most two frames) on the matrix cores.  Tile
// (qt, kt): rows the queries 32 qt.., columns the keys 32 kt..; lane half h
// holds components 4h..4h+3 of both vectors: a query's (h, l of its threshold for
// the block's first frame, h, l for its second | 2048, 1, 2x, 2y), see threshold_word.
// A wave's 64 lanes then hold counts of 32 keys, half of the queries in each
// half.  Decided after every 64 keys where the rest cannot change the vote.
template <int B, int RULE>
__device__ bool test_block_by_tile(const Box& bx, int v, const uint16_t* __restrict__ kfeat, const uint32_t* s_A,
                                   const int (&qf)[B / 32], const uint32_t (&qxy)[B / 32], int FS, int n_u,
                                   int lane) {
  constexpr int QT = B / 32;
  const int col = lane & 31, half = lane >> 5;
  const uint2* kv = (const uint2*)(kfeat + (size_t)v * B * kKeyFeat) + half * B + col;
  f16x4 kb[QT];
#pragma unroll
  for (int kt = 0; kt < QT; ++kt) kb[kt] = __builtin_bit_cast(f16x4, kv[32 * kt]);
  const f16x2 one2 = {(_Float16)2048, (_Float16)1};
  f16x4 qa[QT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const uint32_t* row = s_A + (32 * qt + col) * FS;
    const uint32_t lo = row[abs(qf[qt] - bx.fmin)], hi = row[abs(qf[qt] - bx.fmax)];
    qa[qt] = __builtin_bit_cast(f16x4, make_uint2(half ? __builtin_bit_cast(uint32_t, one2) : lo, half ? qxy[qt] : hi));
  }
  f32x16 one;
#pragma unroll
  for (int e = 0; e < 16; ++e) one[e] = 1.f;
  int nonempty = 0, high = 0;
#pragma unroll
  for (int k2 = 0; k2 < QT; k2 += 2) {
    ushort2_t c[2] = {{0, 0}, {0, 0}};
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      f32x16 e1[2];  // E + 1, the two key tiles in flight together
#pragma unroll
      for (int s = 0; s < 2; ++s) e1[s] = __builtin_amdgcn_mfma_f32_32x32x8f16(qa[qt], kb[k2 + s], one, 0, 0, 0);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 16; e += 2)
          c[s] -= __builtin_bit_cast(ushort2_t, __builtin_amdgcn_cvt_pknorm_u16(e1[s][e], e1[s][e + 1]));
    }
    int c2[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int n = (int)c[s][0] + (int)c[s][1];
      c2[s] = n + __shfl_xor(n, 32);
    }
    // lane half s takes key tile k2 + s
    const int n = half ? c2[1] : c2[0];
    const bool kvalid = 32 * k2 + lane < bx.n_video;
    nonempty += popc(ballot(kvalid && n > 0));
    high += popc(ballot(kvalid && 3 * n > n_u));
    if (RULE == TRA_MASK_UNION) {
      if (nonempty > 0) return true;
    } else {
      const int rest = max(0, bx.n_video - 32 * (k2 + 2));  // keys not tested yet
      if (10 * high > 6 * (nonempty + rest)) return true;
      if (10 * (high + rest) <= 6 * (nonempty + rest)) return false;
    }
  }
  return false;  // (the last pass has decided: rest = 0)
}

template <int B, int RULE, int DIST>
__global__ __launch_bounds__(64 * kWaves) void block_mask_kernel(
    const int32_t* __restrict__ radius_sq, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ coord, const int32_t* __restrict__ thr,
    const int32_t* __restrict__ binfo, const uint16_t* __restrict__ kfeat, uint8_t* __restrict__ mask,
    int32_t* __restrict__ cnt, int32_t* __restrict__ cols, int S, int NB, int F, int H, int W, int n_cap) {
  // thresholds of query q by frame distance at s_T[q * FS + delta] (INT_MAX: covers
  // every key, -1: no query), FS odd so that lanes reading one distance of
  // consecutive queries hit different banks; 2-D: their two f16 components at s_A
  extern __shared__ int32_t s_T[];
  const int FS = F | 1;
  uint32_t* s_A = (uint32_t*)(s_T + B * FS);
  __shared__ int32_t s_c[B];  // packed coordinate of query q
  __shared__ __attribute__((aligned(16))) int32_t s_n[B];  // its radius, n_cap + 1 for the full one, -1 for no query
  __shared__ uint8_t s_keep[kMaxBlocks];
  __shared__ uint16_t s_list[kWaves][kMaxBlocks / kWaves];  // undecided key blocks of each wave
  __shared__ int s_fend[kMaxFrames];       // one past the last query of u's i-th frame
  __shared__ int s_kth;

  const int row = blockIdx.x;
  const int bh = row / NB, u = row - bh * NB;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const Box ub = load_box<DIST>(binfo, u);
  // a block's tokens fill its first n_video + n_text positions
  const int n_u = ub.n_video;

  if (ub.n_text > 0) {
    // a text block's row keeps every key block
    for (int v = t; v < NB; v += blockDim.x) {
      if (mask) mask[(size_t)row * NB + v] = 1;
      cols[(size_t)row * NB + v] = v;
    }
    if (t == 0) cnt[row] = NB;
    return;
  }

  // (this lane's first key block of filter 1, requested before the row's own chain
  // of loads: on small grids the kernel is one such chain after another)
  const Box first_box = load_box<DIST>(binfo, min(wave + kWaves * lane, NB - 1));
  for (int qi = t; qi < B; qi += blockDim.x) {
    int n = -1;
    int32_t c = 0;
    if (qi < n_u) {
      n = radius_sq[(size_t)bh * S + perm[u * B + qi]];
      n = n > n_cap ? n_cap + 1 : max(n, 0);  // TRA_RADIUS_FULL and anything above the cap
      c = coord[u * B + qi];
    }
    s_n[qi] = n;
    s_c[qi] = c;
    // (a block's queries come frame by frame)
    if (qi < n_u && (qi == n_u - 1 || coord_f(coord[u * B + qi + 1]) != coord_f(c))) s_fend[coord_f(c) - ub.fmin] = qi + 1;
  }
  __syncthreads();
  {
    // blockDim / B threads per query share its thresholds
    constexpr int TPQ = 64 * kWaves / B;
    const int qi = t / TPQ;
    const int n = s_n[qi];
    const int32_t c = s_c[qi];
    const int sq = coord_x(c) * coord_x(c) + coord_y(c) * coord_y(c);
    for (int d = t % TPQ; d < F; d += TPQ) {
      const int T = n < 0 ? -1 : n > n_cap ? INT_MAX : thr[(size_t)n * F + d];  // -1 covers nothing: D >= 0
      s_T[qi * FS + d] = T;
      if (DIST == TRA_DIST_2D) s_A[qi * FS + d] = threshold_word(T, sq);
    }
  }
  {
    // the query of the k-th largest radius (equal ones ranked by position)
    constexpr int TPQ = 64 * kWaves / B;
    const int qi = t / TPQ, n = s_n[qi];
    int rank = 0;
#pragma unroll 4
    for (int j = 4 * (t % TPQ); j < B; j += 4 * TPQ) {
      const int4 o = *(const int4*)(s_n + j);
      rank += o.x > n - (j < qi) ? 1 : 0;
      rank += o.y > n - (j + 1 < qi) ? 1 : 0;
      rank += o.z > n - (j + 2 < qi) ? 1 : 0;
      rank += o.w > n - (j + 3 < qi) ? 1 : 0;
    }
#pragma unroll
    for (int x = 1; x < TPQ; x <<= 1) rank += __shfl_xor(rank, x);
    if (t % TPQ == 0 && rank == (RULE == TRA_MASK_VOTE ? n_u / 3 : 0)) s_kth = qi;
  }
  __syncthreads();

  // Key block v belongs to wave v mod 4 through all three filters (the blocks left
  // undecided are neighbours, so this spreads them evenly), which keeps them in
  // a list of its own: a wave's 64 lanes append and drop entries by ballot.
  uint16_t* list = s_list[wave];
  auto rank_in = [](uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  };
  int n_open = 0;

  // 1. box against box, one key block per lane
  const int32_t* Tk = s_T + s_kth * FS;
  for (int v0 = wave; v0 < NB; v0 += 64 * kWaves) {
    const int v = v0 + kWaves * lane;
    bool keep = false, open = false;
    if (v < NB) {
      const Box b = v0 == wave ? first_box : load_box<DIST>(binfo, v);
      if (v == u || b.n_text > 0) {
        keep = true;  // every query keeps its own key; text keys stay visible
      } else {
        const int an = max(0, max(b.amin - ub.amax, ub.amin - b.amax));
        const int bn = max(0, max(b.bmin - ub.bmax, ub.bmin - b.bmax));
        const int af = max(ub.amax - b.amin, b.amax - ub.amin);
        const int bf = max(ub.bmax - b.bmin, b.bmax - ub.bmin);
        const int dn = max(0, max(b.fmin - ub.fmax, ub.fmin - b.fmax));
        const int df = max(ub.fmax - b.fmin, b.fmax - ub.fmin);
        keep = metric<DIST>(af, bf) <= Tk[df];
        open = !keep && metric<DIST>(an, bn) <= Tk[dn];
      }
      if (!open) s_keep[v] = keep ? 1 : 0;
    }
    const uint64_t m = ballot(open);
    if (open) list[n_open + rank_in(m)] = (uint16_t)v;
    n_open += popc(m);
  }
  __syncthreads();

  // 2. each query against the box, one key block per lane.  A column is covered
  // by the queries that reach the block with a positive threshold, and by those
  // whose threshold there is 0 only at their own (x, y): at most one per frame of
  // u, so no column counts more than n_in + the frames of u.
  // (A pass costs about as much as eight pair tests, so a wave with no more
  // blocks than that goes straight to them.)
  constexpr int kFewOpen = 8;
  const int u_frames = ub.fmax - ub.fmin + 1;
  int n_test = n_open <= kFewOpen ? n_open : 0;
  for (int i0 = n_test; i0 < n_open; i0 += 64) {
    const bool have = i0 + lane < n_open;
    const int v = list[min(i0 + lane, n_open - 1)];
    const Box b = load_box<DIST>(binfo, v);
    int n_all = 0, n_in = 0;
    int q = 0;
    for (int qf = ub.fmin; qf <= ub.fmax; ++qf) {
      const int32_t* Tn = s_T + max(0, max(b.fmin - qf, qf - b.fmax));  // nearest frame
      const int32_t* Tf = s_T + max(qf - b.fmin, b.fmax - qf);          // farthest
      const int q_end = __builtin_amdgcn_readfirstlane(s_fend[qf - ub.fmin]);
      auto count = [&](int qq, int32_t cw) {
        int qx, qy, f;
        position<DIST>(__builtin_amdgcn_readfirstlane(cw), H, W, &qx, &qy, &f);
        const int a0 = b.amin - qx, a1 = qx - b.amax, b0 = b.bmin - qy, b1 = qy - b.bmax;
        const int near = metric<DIST>(max(0, max(a0, a1)), max(0, max(b0, b1)));
        const int far = metric<DIST>(min(a0, a1), min(b0, b1));  // (squared, or |.|: the sign does not matter)
        n_in += (RULE == TRA_MASK_VOTE ? max(near, 1) : near) <= Tn[qq * FS] ? 1 : 0;
        n_all += far <= Tf[qq * FS] ? 1 : 0;
      };
      for (; q + 4 <= q_end; q += 4)  // four queries' LDS reads in flight
#pragma unroll
        for (int j = 0; j < 4; ++j) count(q + j, s_c[q + j]);
      for (; q < q_end; ++q) count(q, s_c[q]);
    }
    const bool keep = RULE == TRA_MASK_VOTE ? 3 * n_all > n_u : n_all > 0;
    const bool drop = RULE == TRA_MASK_VOTE ? 3 * (n_in + u_frames) <= n_u : n_in == 0;
    const bool open = have && !keep && !drop;
    if (have && !open) s_keep[v] = keep ? 1 : 0;
    const uint64_t m = ballot(open);
    if (open) list[n_test + rank_in(m)] = (uint16_t)v;  // (in place: at or before the entries just read)
    n_test += popc(m);
  }
  __syncthreads();

  // 3. pair by pair, the wave's undecided blocks in turn
  [[maybe_unused]] int qf[B / 32];        // this lane's query of each 32-query tile: frame,
  [[maybe_unused]] uint32_t qxy[B / 32];  // and (2x, 2y) as f16
#pragma unroll
  for (int qt = 0; qt < B / 32; ++qt) {
    const int32_t cw = s_c[32 * qt + (lane & 31)];
    const f16x2 xy = {(_Float16)(2 * coord_x(cw)), (_Float16)(2 * coord_y(cw))};
    qf[qt] = coord_f(cw);
    qxy[qt] = __builtin_bit_cast(uint32_t, xy);
  }
  for (int i = 0; i < n_test; ++i) {
    const int v = __builtin_amdgcn_readfirstlane((int)list[i]);
    const Box b = load_box<DIST>(binfo, v);
    bool keep;
    if (DIST == TRA_DIST_2D && b.fmax - b.fmin <= 1)
      keep = test_block_by_tile<B, RULE>(b, v, kfeat, s_A, qf, qxy, FS, n_u, lane);
    else
      keep = test_block_by_query<B, RULE, DIST>(b, v, coord, s_T, s_c, FS, n_u, H, W, lane);
    if (lane == 0) s_keep[v] = keep ? 1 : 0;
  }
  __syncthreads();

  // Compact the retained key blocks of this row in ascending order.
  if (mask)
    for (int v = t; v < NB; v += blockDim.x) mask[(size_t)row * NB + v] = s_keep[v];
  if (wave == 0) {
    int base = 0;
    for (int v0 = 0; v0 < NB; v0 += 64) {
      const int v = v0 + lane;
      const bool k = v < NB && s_keep[v];
      const uint64_t bm = ballot(k);
      const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)bm, 0u));
      if (k) cols[(size_t)row * NB + base + rank] = v;
      base += popc(bm);
    }
    for (int i = base + lane; i < NB; i += 64) cols[(size_t)row * NB + i] = -1;
    if (lane == 0) cnt[row] = base;
  }
}

// ------------------------------------------------ heaviest-first row order
// Stable counting sort of rows by key NB - cnt (so larger cnt first, ties by
// row index): per-chunk histograms; per key, the exclusive scan over its chunks
// (one wave a key, coalesced) with the key's total left in its first entry,
// whose scan is 0; then a scatter whose workgroups each scan the totals and rank
// equal keys inside their chunk by row index.  (One workgroup scanning all keys x
// chunks took 0.10 of the sort's 0.11 ms at 23,640 rows x 592 keys; the sort now
// takes 0.02.)

__global__ __launch_bounds__(kSortChunk) void order_hist_kernel(const int32_t* __restrict__ cnt,
                                                                int32_t* __restrict__ ws, int rows,
                                                                int NB, int chunks) {
  __shared__ int32_t h[kMaxBlocks + 1];
  for (int i = threadIdx.x; i <= NB; i += blockDim.x) h[i] = 0;
  __syncthreads();
  const int r = blockIdx.x * kSortChunk + threadIdx.x;
  if (r < rows) atomicAdd(&h[NB - min(max(cnt[r], 0), NB)], 1);
  __syncthreads();
  for (int k = threadIdx.x; k <= NB; k += blockDim.x) ws[(size_t)k * chunks + blockIdx.x] = h[k];
}

__global__ __launch_bounds__(256) void order_scan_kernel(int32_t* __restrict__ ws, int keys, int chunks) {
  const int lane = threadIdx.x & 63, key = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (key >= keys) return;
  int32_t* row = ws + (size_t)key * chunks;
  int run = 0;
  for (int c0 = 0; c0 < chunks; c0 += 64) {
    const int c = c0 + lane;
    const int x = c < chunks ? row[c] : 0;
    int s = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(s, o);
      if (lane >= o) s += y;
    }
    if (c < chunks && c > 0) row[c] = run + s - x;
    run += __shfl(s, 63);
  }
  if (lane == 0) row[0] = run;
}

__global__ __launch_bounds__(kSortChunk) void order_scatter_kernel(const int32_t* __restrict__ cnt,
                                                                   const int32_t* __restrict__ ws,
                                                                   int32_t* __restrict__ order,
                                                                   int rows, int NB, int chunks) {
  __shared__ int32_t keys[kSortChunk];
  __shared__ int32_t first[kMaxBlocks + 1];  // rows of smaller keys
  __shared__ int32_t part[kSortChunk];
  const int t = threadIdx.x;
  const int r = blockIdx.x * kSortChunk + t;
  const int key = r < rows ? NB - min(max(cnt[r], 0), NB) : -1;
  keys[t] = key;
  for (int k = t; k <= NB; k += kSortChunk) first[k] = ws[(size_t)k * chunks];
  __syncthreads();
  // exclusive scan of the totals: each thread its run of keys, then the threads
  const int per = (NB + kSortChunk) / kSortChunk, k0 = min(NB + 1, t * per), k1 = min(NB + 1, k0 + per);
  int sum = 0;
  for (int k = k0; k < k1; ++k) sum += first[k];
  part[t] = sum;
  __syncthreads();
  for (int o = 1; o < kSortChunk; o <<= 1) {
    const int y = t >= o ? part[t - o] : 0;
    __syncthreads();
    part[t] += y;
    __syncthreads();
  }
  int run = part[t] - sum;
  for (int k = k0; k < k1; ++k) {
    const int x = first[k];
    first[k] = run;
    run += x;
  }
  __syncthreads();
  if (r < rows) {
    int rank = 0;
    for (int s = 0; s < t; ++s) rank += keys[s] == key;
    order[first[key] + (blockIdx.x ? ws[(size_t)key * chunks + blockIdx.x] : 0) + rank] = r;
  }
}

}  // namespace

template <int B, int RULE, int DIST>
void launch_mask_variant(const tra_plan_s& p, const int32_t* radius_sq, uint8_t* mask, int32_t* cnt,
                         int32_t* cols, hipStream_t s) {
  const int32_t* thr = DIST == TRA_DIST_1D ? p.d_thr1 : p.d_thr;
  const size_t lds = (size_t)B * (p.cfg.frames | 1) * sizeof(int32_t) * (DIST == TRA_DIST_2D ? 2 : 1);
  hipLaunchKernelGGL((block_mask_kernel<B, RULE, DIST>), dim3(p.rows), dim3(64 * kWaves), lds, s, radius_sq,
                     p.d_perm, p.d_coord, thr, p.d_blocks, p.d_kfeat, mask, cnt, cols, p.S, p.NB, p.cfg.frames,
                     p.cfg.height, p.cfg.width, p.n_cap);
}

template <int B, int RULE>
void launch_mask_dist(const tra_plan_s& p, const int32_t* radius_sq, uint8_t* mask, int32_t* cnt,
                      int32_t* cols, hipStream_t s) {
  if (p.cfg.distance == TRA_DIST_1D) launch_mask_variant<B, RULE, TRA_DIST_1D>(p, radius_sq, mask, cnt, cols, s);
  else launch_mask_variant<B, RULE, TRA_DIST_2D>(p, radius_sq, mask, cnt, cols, s);
}

template <int B>
void launch_mask_rule(const tra_plan_s& p, const int32_t* radius_sq, uint8_t* mask, int32_t* cnt,
                      int32_t* cols, hipStream_t s) {
  if (p.cfg.rule == TRA_MASK_VOTE) launch_mask_dist<B, TRA_MASK_VOTE>(p, radius_sq, mask, cnt, cols, s);
  else launch_mask_dist<B, TRA_MASK_UNION>(p, radius_sq, mask, cnt, cols, s);
}

hipError_t launch_block_mask(const tra_plan_s& p, const int32_t* radius_sq, uint8_t* mask,
                             int32_t* cnt, int32_t* cols, hipStream_t s) {
  if (p.cfg.block == 128) launch_mask_rule<128>(p, radius_sq, mask, cnt, cols, s);
  else launch_mask_rule<64>(p, radius_sq, mask, cnt, cols, s);
  return hipGetLastError();
}

hipError_t launch_row_order_ws(const tra_plan_s& p, const int32_t* cnt, int32_t* order, int32_t* ws,
                               hipStream_t s) {
  const int chunks = p.sort_chunks;
  hipLaunchKernelGGL(order_hist_kernel, dim3(chunks), dim3(kSortChunk), 0, s, cnt, ws, p.rows, p.NB, chunks);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(order_scan_kernel, dim3((p.NB + 4) / 4), dim3(256), 0, s, ws, p.NB + 1, chunks);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(order_scatter_kernel, dim3(chunks), dim3(kSortChunk), 0, s, cnt, ws, order, p.rows, p.NB,
                     chunks);
  return hipGetLastError();
}

hipError_t launch_row_order(const tra_plan_s& p, const int32_t* cnt, int32_t* order, hipStream_t s) {
  return launch_row_order_ws(p, cnt, order, p.d_sort_ws, s);
}

// ------------------------------------------------ no-allocation entry point
// The counting-sort workspace of tra_build_block_mask_noalloc: a device array
// of the library itself, one copy per GPU, held until the process ends.  In
// host code `scratch` only names the symbol; its device address on each GPU
// comes from hipGetSymbolAddress (resolve_noalloc_scratch) and only that
// address is handed to kernels.  Every order kernel writes each workspace
// entry it later reads, so no clearing is needed between calls.
static __device__ __align__(256) int32_t scratch[kNoAllocScratchInts];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t resolve_noalloc_scratch(int device, int32_t** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    int32_t* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = ptr;
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

hipError_t launch_row_order_noalloc(const tra_plan_s& p, const int32_t* cnt, int32_t* order, hipStream_t s) {
  int32_t* ws = nullptr;
  const hipError_t e = resolve_noalloc_scratch(p.device, &ws);
  if (e != hipSuccess) return e;
  return launch_row_order_ws(p, cnt, order, ws, s);
}

}  // namespace tra
