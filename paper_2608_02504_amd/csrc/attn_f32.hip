// fp32 attention family (dense, block-sparse, token-level sparse, entropy with
// or without the output) for fp32 workloads, on the fp32 matrix instructions
// (v_mfma_f32_32x32x2_f32: fp32 inputs, products and sums throughout).
//
// Work decomposition.  One workgroup of 8 waves takes 32 queries of a
// query-block row; the waves split the row's key tiles (32 keys each, tile i to
// wave i mod 8), each with its own running softmax state, and merge their states
// through LDS at the end.  Splitting the keys inside the workgroup is what fills
// the chip at the sizes fp32 calls have: 256 tokens x 2 heads are 16 workgroups
// of one tile per wave.
//
// Bound.  A 32x32x2 MFMA holds a SIMD's matrix pipe for 64 cycles, so a tile at
// head_dim 128 (64 MFMAs for S^T = K Q^T, 64 for O^T += V^T P^T) takes 8,192
// cycles for 32 KB of K and V: the matrix pipe is the bound, and every operand
// can come straight from memory into registers.  No LDS staging of K and V and
// no barrier in the loop: a lane's float4 of K (four consecutive components of
// one key) feeds four QK^T steps, its float4 of V (four consecutive components
// of one key) one step of each of the four 32-wide output tiles; the contraction
// order over d and the row order of O^T are chosen to make them so.  V loads are
// issued before the tile's QK^T and the next tile's K loads before its softmax,
// so each has a matrix phase to land in; two waves per SIMD overlap one's softmax
// with the other's MFMAs.  Q stays in LDS (one ds_read_b128 per four MFMAs),
// which keeps the wave inside 256 registers.
//
// Measured (MI355X), against one thread per query and scalar FMAs: entropy with
// output at 4 heads x 3,510 tokens x 128, 13.69 -> 0.276 ms (1.8 -> 91 TFLOP/s; a
// large fp32 GEMM reaches 155 here, and 440 workgroups on 256 CUs are two rounds
// of one, which bounds it at 0.19); the whole chain on 256 tokens x 2 heads x 64,
// 1,018 -> 41 us.  Error against fp64: 4.5e-6 -> 1.6e-6 (2-norm, relative).
//
// Online softmax with the entropy accumulator of Alg. 2 (App. C.2), kept
// relative to the running maximum m: per query l = sum_j e^{s_j - m} and
// a = sum_j e^{s_j - m} (s_j - m); when m grows to m', l <- e^{m-m'} l and
// a <- e^{m-m'} (a + l (m - m')).  At the end H = log l - a / l, which equals
// log Z - sum_j p_j s_j (the fused-entropy identity of App. C.2), and
// lse = m + log l.  The token-level variant (Eq. 16 with the token mask of Eq.
// 15 inside the listed blocks) tests every (query, key) pair with the plan's
// integer thresholds, as the block-mask kernel does.
#include <algorithm>
#include <cmath>

#include "tra_internal.h"

namespace tra {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct F32Params {
  const float* q;
  const float* k;
  const float* v;
  float* o;
  float* lse;
  float* entropy;
  const int32_t* perm;
  const int32_t* coord;  // packed (f, x, y) per position (token-level attention)
  const int32_t* cnt;
  const int32_t* cols;
  const int32_t* order;
  const int32_t* bcount;  // tokens of each block (tile-aligned layout), NULL: packed
  int N, NB, rows, B;  // B: tokens per block (64 or 128)
  float alpha;
  // token-level attention only
  const int32_t* radius_sq;
  const int32_t* thr;  // [(n_cap + 1) * F], 2-D or 1-D thresholds per the plan
  int Nv, F, n_cap;
  int first;  // the launch's first query tile (see launch_f32_d)
};

constexpr int kWaves = 8;
constexpr int kF32Threads = 64 * kWaves;
constexpr int kTile = 32;  // queries per workgroup, keys per tile

// v of the lane whose index is lane4 / 4 (0..31, in this wave's lower half).
__device__ __forceinline__ int from_lane(int v, int lane4) { return __builtin_amdgcn_ds_bpermute(lane4, v); }

// Key (of a 32-key tile) of element e of this lane's scores, less 4 half.
__device__ __forceinline__ constexpr int key_of(int e) { return 8 * (e >> 2) + (e & 3); }

// Hides a value from the optimiser: indexes derived from it are formed next to
// their use instead of being hoisted out of the tile loop into registers.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// max / sum over the two lane halves (lanes l and l ^ 32)
__device__ __forceinline__ float max_halves(float x) { return fmaxf(x, __shfl_xor(x, 32)); }
__device__ __forceinline__ float sum_halves(float x) { return x + __shfl_xor(x, 32); }

// Does the query (position word cw_i, raster index i, radius n) cover the video
// key (cw_j, j)?  TOK 1: 2-D squared distance, 2: |i - j|.
template <int TOK>
__device__ __forceinline__ bool covers(const F32Params& P, int32_t cw_i, int i, int n, int32_t cw_j, int j) {
  int dist;
  if constexpr (TOK == 2) {
    dist = abs(i - j);
  } else {
    const int dx = coord_x(cw_i) - coord_x(cw_j), dy = coord_y(cw_i) - coord_y(cw_j);
    dist = dx * dx + dy * dy;
  }
  return dist <= P.thr[(size_t)n * P.F + abs(coord_f(cw_i) - coord_f(cw_j))];
}

// TOK: 0 block-granular, 1 token mask with 2-D distance, 2 with 1-D distance.
template <int D, bool SPARSE, bool PV, bool ENT, int TOK = 0>
__global__ __launch_bounds__(kF32Threads, 2) void attn_f32_kernel(F32Params P) {
  constexpr int KC = D / 8;    // float4 chunks of a key per lane (half h: components 8g + 4h ..+3)
  constexpr int DT = D / 32;   // 32-wide output tiles; a lane's V load holds one component of each
  constexpr int QP = D + 4;    // pitch of a query in LDS: rows on distinct bank groups
  typedef float vecv __attribute__((ext_vector_type(DT)));
  __shared__ __attribute__((aligned(16))) float sQ[kTile * QP];
  __shared__ __attribute__((aligned(16))) float sO[PV ? kWaves / 2 : 1][PV ? D * kTile : 4];
  __shared__ float sStat[kWaves / 2][3][kTile];

  const int subs = P.B / kTile;  // query tiles per row, key tiles per block
  int idx = blockIdx.x;
  if (!(SPARSE && P.order)) {
    // workgroup b runs on XCD b mod 8: give each XCD a contiguous range of
    // query tiles, so that those in flight share a head's K and V in its L2
    const int x = idx & 7, per = (int)gridDim.x / 8, rem = (int)gridDim.x % 8;
    idx = x * per + min(x, rem) + (idx >> 3);
  }
  idx += P.first;
  int r = idx / subs;
  const int qsub = idx - r * subs;
  if (SPARSE && P.order) {
    r = P.order[r];
    if (r < 0 || r >= P.rows) return;  // whole workgroup leaves together
  }
  const int bh = r / P.NB, u = r - bh * P.NB;
  // a block's tokens fill its first positions: nothing to do past them
  if (P.perm[u * P.B + qsub * kTile] < 0) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int col = lane & 31, half = lane >> 5;
  const size_t head_off = (size_t)bh * P.N * D;
  const float* Kh = P.k + head_off;
  const float* Vh = PV ? P.v + head_off : nullptr;

  const int qpos = u * P.B + qsub * kTile + col;
  const int qtok = P.perm[qpos];  // -1 at a padding position
  const bool qvalid = qtok >= 0;
  // stage the 32 queries (zeros at padding)
  for (int i = t; i < kTile * (D / 4); i += kF32Threads) {
    const int qi = i / (D / 4), c = i - qi * (D / 4);
    const int tok = P.perm[u * P.B + qsub * kTile + qi];
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tok >= 0) x = *(const float4*)(P.q + head_off + (size_t)tok * D + 4 * c);
    *(float4*)(sQ + qi * QP + 4 * c) = x;
  }
  // token mask: a text query (or a FULL radius) covers every key
  [[maybe_unused]] int n_i = 0;
  [[maybe_unused]] int32_t cw_i = 0;
  [[maybe_unused]] bool all_keys = true;
  if constexpr (TOK != 0) {
    if (qvalid && qtok < P.Nv) {
      n_i = P.radius_sq[(size_t)bh * P.N + qtok];
      all_keys = n_i > P.n_cap;
      n_i = max(n_i, 0);
      cw_i = P.coord[qpos];
    }
  }
  __syncthreads();

  const int count = SPARSE ? min(max(P.cnt[r], 0), P.NB) : P.NB;
  const int32_t* colp = SPARSE ? P.cols + (size_t)r * P.NB : nullptr;
  // Tile i: keys [32 (i % subs), +32) of block list[i / subs].  Returns the
  // first tile >= i of this wave (step 8) that holds a token, its first position
  // and its tokens (a block's tokens fill its first positions); total if none.
  const int n_tiles = count * subs;
  auto next_tile = [&](int i, int* pos, int* ns) -> int {
    for (; i < n_tiles; i += kWaves) {
      const int c = i / subs, sub = i - c * subs;
      const int vb = SPARSE ? colp[c] : c;
      if (vb < 0 || vb >= P.NB) continue;
      const int nv = (P.bcount ? P.bcount[vb] : min(P.B, P.N - vb * P.B)) - sub * kTile;
      if (nv <= 0) continue;
      *pos = vb * P.B + sub * kTile;
      *ns = min(nv, kTile);
      return i;
    }
    return n_tiles;
  };
  // the token of this lane's key of a tile (a tile's keys past its last token repeat that one)
  auto key_token = [&](int pos, int ns) { return P.perm[pos + min(col, ns - 1)]; };

  f32x16 oacc[PV ? DT : 1];
  float m, l, a;
  // (TOK) A query takes nothing from a tile of which it covers no key, but 0 times an
  // infinite or NaN value is NaN: a wave whose output is not finite goes over its
  // tiles once more, carefully, putting such queries' sums back after each.
  [[maybe_unused]] bool careful = false;
again:
#pragma unroll
  for (int i = 0; i < (PV ? DT : 1); ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[i][e] = 0.f;
  m = -INFINITY;
  l = a = 0.f;

  // buf: the current tile's K (16 / KC entries per chunk); as a chunk of it is
  // consumed by QK^T, rows of the tile's V take its place, and as those are
  // consumed by PV, chunks of the next tile's K: every load is in flight for
  // about one matrix phase, and K and V together need one tile's registers.
  constexpr int CE = 16 / KC;  // entries per chunk, CE * DT = 4 components
  vecv buf[16];
  auto load_chunk = [&](int tok, int g) {
    const float4 x = *(const float4*)(Kh + (size_t)tok * D + 4 * half + 8 * g);
    const float w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) buf[g * CE + c / DT][c % DT] = w[c];
  };

  int pos = 0, ns = 0, pos_n = 0, ns_n = 0, tok_n = 0;
  int i = next_tile(wave, &pos, &ns);
  int tok = 0;
  if (i < n_tiles) {
    tok = key_token(pos, ns);
#pragma unroll
    for (int g = 0; g < KC; ++g) load_chunk(tok, g);
  }
  const float* qrow = sQ + col * QP + 4 * half;
  while (i < n_tiles) {
    const int i_n = next_tile(i + kWaves, &pos_n, &ns_n);
    tok_n = i_n < n_tiles ? key_token(pos_n, ns_n) : tok;  // (after the last tile its K is loaded once more)
    [[maybe_unused]] int32_t cw = 0;
    if constexpr (TOK != 0) cw = P.coord[pos + min(col, ns - 1)];

    const int half16 = opaque(16 * half);  // 4 (4 half)
    f32x16 s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
    float4 qv = *(const float4*)qrow;
#pragma unroll
    for (int g = 0; g < KC; ++g) {
      const float4 q0 = qv;
      if (g + 1 < KC) qv = *(const float4*)(qrow + 8 * (g + 1));
      const float qc[4] = {q0.x, q0.y, q0.z, q0.w};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[g * CE + c / DT][c % DT], qc[c], s, 0, 0, 0);
      if constexpr (PV) {
        // element e of this half's scores is key 8 (e / 4) + 4 half + e % 4
#pragma unroll
        for (int e = g * CE; e < (g + 1) * CE; ++e)
          buf[e] = *(const vecv*)(Vh + (size_t)from_lane(tok, half16 + 4 * key_of(e)) * D + DT * col);
      } else {
        load_chunk(tok_n, g);
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    float mc = -INFINITY;
    [[maybe_unused]] bool some = false;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      bool keep = half16 + 4 * key_of(e) < 4 * ns;
      if constexpr (TOK != 0) {
        const int tok_j = from_lane(tok, half16 + 4 * key_of(e));
        const int32_t cw_j = from_lane(cw, half16 + 4 * key_of(e));
        if (keep && !all_keys && tok_j < P.Nv) keep = covers<TOK>(P, cw_i, qtok, n_i, cw_j, tok_j);
      }
      if (TOK != 0) some = some || keep;
      s[e] = keep ? s[e] * P.alpha : -INFINITY;
      mc = fmaxf(mc, s[e]);
    }
    // (TOK) the queries that cover a key of the tile
    [[maybe_unused]] uint64_t takes = ~0ull;
    if constexpr (TOK != 0) {
      takes = __ballot(some);
      takes |= takes >> 32 | takes << 32;
    }
    mc = max_halves(mc);
    const float mn = fmaxf(m, mc);
    const float mr = mn > -INFINITY ? mn : 0.f;  // (TOK) a query with no covered key yet: every weight is 0
    const float sc = expf(m - mr);               // 0 on the first tile (m = -inf)
    if (ENT) a = l > 0.f ? sc * (a + l * (m - mr)) : 0.f;
    l *= sc;
    if constexpr (PV) {
      if (__ballot(sc != 1.f) != 0) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[dt][e] *= sc;
      }
    }
    float ls = 0.f, as = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float x = s[e] - mr;
      const float p = expf(x);
      ls += p;
      // (a masked key has p = 0 and x = -inf: its p x is 0)
      if (ENT) as += p > 0.f ? p * x : p;
      s[e] = p;
    }
    l += ls;
    if (ENT) a += as;
    m = mn;
    if constexpr (PV) {
      if (ns < kTile) {  // rows past the last token: 0 times the repeated one would be NaN where it is infinite
        const int left = opaque(ns - 4 * half);
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (key_of(e) >= left) buf[e] = vecv(0.f);
      }
      const bool apart = TOK != 0 && careful && takes != ~0ull;
      float old[TOK != 0 ? 16 * DT : 1];
      if (apart) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) old[16 * dt + e] = oacc[dt][e];
        asm volatile("" : : "v"(&old[0]) : "memory");  // (in scratch memory, not in registers)
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[e][dt], s[e], oacc[dt], 0, 0, 0);
        if (e % CE == CE - 1) load_chunk(tok_n, e / CE);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (apart && !(takes >> lane & 1)) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[dt][e] = old[16 * dt + e];
      }
    }
    i = i_n;
    pos = pos_n;
    ns = ns_n;
    tok = tok_n;
  }

  if constexpr (TOK != 0) {
    float z = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) z = fmaf(oacc[dt][e], 0.f, z);  // NaN where a sum is not finite
    if (!careful && __ballot(z != 0.f) != 0) {
      careful = true;
      goto again;
    }
  }

  // ---- merge the waves' states: waves s..2s-1 into waves 0..s-1, s = 4, 2, 1
  l = sum_halves(l);
  if (ENT) a = sum_halves(a);
#pragma unroll
  for (int st = kWaves / 2; st > 0; st >>= 1) {
    if (wave >= st && wave < 2 * st) {
      if constexpr (PV) {
        float4* dst = (float4*)sO[wave - st];
#pragma unroll
        for (int j = 0; j < 4 * DT; ++j)
          dst[j * 64 + lane] = make_float4(oacc[j >> 2][4 * (j & 3)], oacc[j >> 2][4 * (j & 3) + 1],
                                           oacc[j >> 2][4 * (j & 3) + 2], oacc[j >> 2][4 * (j & 3) + 3]);
      }
      if (half == 0) {
        sStat[wave - st][0][col] = m;
        sStat[wave - st][1][col] = l;
        sStat[wave - st][2][col] = a;
      }
    }
    __syncthreads();
    if (wave < st) {
      const float m1 = sStat[wave][0][col], l1 = sStat[wave][1][col], a1 = sStat[wave][2][col];
      const float mn = fmaxf(m, m1);
      // a state that saw no key has m = -inf and weight 0
      const float s0 = m > -INFINITY ? expf(m - mn) : 0.f, s1 = m1 > -INFINITY ? expf(m1 - mn) : 0.f;
      if (ENT) a = (l > 0.f ? s0 * (a + l * (m - mn)) : 0.f) + (l1 > 0.f ? s1 * (a1 + l1 * (m1 - mn)) : 0.f);
      l = s0 * l + s1 * l1;
      m = mn;
      if constexpr (PV) {
        const float4* src = (const float4*)sO[wave];
#pragma unroll
        for (int j = 0; j < 4 * DT; ++j) {
          const float4 x = src[j * 64 + lane];
          f32x16& acc = oacc[j >> 2];
          const int e = 4 * (j & 3);
          acc[e] = s0 * acc[e] + s1 * x.x;
          acc[e + 1] = s0 * acc[e + 1] + s1 * x.y;
          acc[e + 2] = s0 * acc[e + 2] + s1 * x.z;
          acc[e + 3] = s0 * acc[e + 3] + s1 * x.w;
        }
      }
    }
    __syncthreads();
  }
  if (wave != 0 || !qvalid) return;
  const size_t tok_o = (size_t)bh * P.N + qtok;
  if constexpr (PV) {
    const float inv = l > 0.f ? 1.f / l : 0.f;
    // row 8 (e / 4) + 4 half + e % 4 of output tile dt is component DT row + dt
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      vecv x;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) x[dt] = oacc[dt][e] * inv;
      *(vecv*)(P.o + tok_o * D + DT * (8 * (e >> 2) + 4 * half + (e & 3))) = x;
    }
  }
  if (half == 0) {
    if (ENT) P.entropy[tok_o] = logf(l) - a / l;
    if (P.lse) P.lse[tok_o] = l > 0.f ? m + logf(l) : -INFINITY;
  }
}

template <int D>
hipError_t launch_f32_d(const tra_plan_s& p, const AttnArgs& a, hipStream_t s) {
  const bool one_d = p.cfg.distance == TRA_DIST_1D;
  F32Params P{(const float*)a.q, (const float*)a.k, (const float*)a.v, (float*)a.o, a.lse,
              a.entropy, p.d_perm, p.d_coord, a.cnt, a.cols, a.order,
              a.sparse && p.cfg.block_layout == TRA_BLOCKS_TILES ? p.d_bcount : nullptr, p.S, p.NB, p.rows,
              p.cfg.block, 1.0f / sqrtf((float)D), a.radius_sq, one_d ? p.d_thr1 : p.d_thr, p.N,
              p.cfg.frames, p.n_cap, 0};
  // (a launch holds fewer than 2^32 threads: a plan of many short rows, all padding but
  // a few tokens, has more query tiles than that)
  constexpr int kMostTiles = 1 << 22;
  const int tiles = p.rows * (p.cfg.block / kTile);
  const dim3 block(kF32Threads);
  if (a.ev_start) (void)hipEventRecord(a.ev_start, s);
  for (P.first = 0; P.first < tiles; P.first += kMostTiles) {
    const dim3 grid(std::min(tiles - P.first, kMostTiles));
    if (a.sparse && a.radius_sq && one_d)
      hipLaunchKernelGGL((attn_f32_kernel<D, true, true, false, 2>), grid, block, 0, s, P);
    else if (a.sparse && a.radius_sq)
      hipLaunchKernelGGL((attn_f32_kernel<D, true, true, false, 1>), grid, block, 0, s, P);
    else if (a.sparse)
      hipLaunchKernelGGL((attn_f32_kernel<D, true, true, false>), grid, block, 0, s, P);
    else if (a.entropy && a.o)
      hipLaunchKernelGGL((attn_f32_kernel<D, false, true, true>), grid, block, 0, s, P);
    else if (a.entropy)
      hipLaunchKernelGGL((attn_f32_kernel<D, false, false, true>), grid, block, 0, s, P);
    else
      hipLaunchKernelGGL((attn_f32_kernel<D, false, true, false>), grid, block, 0, s, P);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.ev_stop) (void)hipEventRecord(a.ev_stop, s);
  return hipSuccess;
}

}  // namespace

hipError_t launch_attention_f32(const tra_plan_s& p, const AttnArgs& a, hipStream_t s) {
  return p.cfg.head_dim == 64 ? launch_f32_d<64>(p, a, s) : launch_f32_d<128>(p, a, s);
}

}  // namespace tra
