// k_score_docs.hip - document scoring of a batch by document (Sec. 3.2
// document scoring, Sec. 4.2 aggregation; the same F^ as k_score.hip).
//
// The candidates of a batch of queries overlap: with 1024 queries that keep
// 8192 of 1M documents, half of the (query, document) visits go to 35,000
// documents that over 64 queries keep.  k_score.hip goes query by query: it
// decodes a document's codes for every visit and adds the centroid part from
// a per-query table of centroid scores S^T (one 128-byte row gathered per
// token and visit, 34 MB per query at 262,144 centroids), which the probe
// has to write first.  Here the visits are sorted by document, each
// document's tokens are decoded once into LDS as centroid + residual, and
// every visiting query multiplies them straight from there: no S^T, no
// gather and no decoding per visit, only the matrix product.
//
// The decoded token c + w[code] is held in fp16.  On the value grid its
// components are multiples of 2^-11, and fp16 holds every such multiple up
// to 1 in magnitude exactly, so the sum is exact whenever max |c_d| + max |w|
// <= 1 (f16_tokens_exact; the caller checks it once per index and keeps to
// k_score.hip otherwise).  Query components are bf16 grid values, exact in
// fp16 as well (the norm bound of exact scores, 4 / (max |c| + sqrt(128) max
// |w|), is at most 8192 as soon as one c or w is not 0), and the products are
// summed in fp32, exact in any order under that bound.  The scores are the
// same bits.
//
// Steps: k_visit_count takes each visit's rank within its document (one
// atomic per visit), k_visit_alloc gives every document a slice of the visit
// array, k_visit_fill writes the visits there, k_doc_score scores them.
//
// k_doc_score is bound by the matrix cores and the power they draw: 8 MFMA
// 32x32x16 (256 cycles of a SIMD) per 32 document tokens and 32 query tokens.
// A wave keeps 64 query columns in registers, so each 8 KB tile read from LDS
// feeds 16 MFMA (64 bytes per clock and CU, half of what LDS delivers).
// Measured with 1024 queries of 16,384 candidates on 2.2M documents: 20.5 ms
// against 29.1 ms by query, 1.05 PFLOP/s, the matrix cores 61% busy; 128
// queries of 64 tokens and 32,768 candidates on 250,000 documents of 320
// tokens (4-bit codes): 26.8 ms against 67.0 ms, 1.16 PFLOP/s (a loop of
// nothing but these MFMA reaches 1.6 to 1.76 PFLOP/s here).  The probe, which
// no longer writes S^T, falls from 10.0 to 7.6 ms in the first (4.0 ms since,
// the centroids in operand order).
// Also tried, all slower for short documents: one query's columns per wave
// with eight waves a workgroup (LDS reads double), 16 lanes to a token in the
// decoder (fewer cache lines per load, a longer chain), documents decoded into
// one wave's registers without LDS tiles (the operands of a visit are then
// loaded once per four tiles; vector memory limits it).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "internal.h"

namespace chimera {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

static uint16_t f16_of_grid_k(int32_t k) {
  return __builtin_bit_cast(uint16_t, (_Float16)((float)k / 2048.0f));  // exact for |k| <= 2048
}

bool f16_tokens_exact(const uint16_t *cent, int64_t n, const uint16_t *weights, int nweights) {
  int32_t cmax = 0, wmax = 0;
  for (int64_t i = 0; i < n; ++i) cmax = std::max(cmax, std::abs(grid_k_of_float(float_of_bf16(cent[i]))));
  for (int u = 0; u < nweights; ++u) wmax = std::max(wmax, std::abs(grid_k_of_float(float_of_bf16(weights[u]))));
  // (all zero: such an index bounds no query's norm, whose components then need not fit fp16)
  return cmax + wmax > 0 && cmax + wmax <= 2048;
}

void f16_of_bf16_grid(const uint16_t *src, int64_t n, uint16_t *dst) {
  for (int64_t i = 0; i < n; ++i) dst[i] = f16_of_grid_k(grid_k_of_float(float_of_bf16(src[i])));
}

// -------------------------------------------------------- visits by document
// A visit is a slot p = q * ncand + i of cand_ids with i < n_valid[q].

// rank[p] = the number of visits of p's document counted before p (any order)
__global__ __launch_bounds__(256) void k_visit_count(const int32_t *__restrict__ cand_ids,
                                                     const int32_t *__restrict__ n_valid, int ncand,
                                                     uint32_t *__restrict__ cnt, uint32_t *__restrict__ rank) {
  const int64_t q = blockIdx.y;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_valid[q]) return;
  const int64_t p = q * ncand + i;
  rank[p] = atomicAdd(&cnt[cand_ids[p]], 1u);
}

// A segment of VISIT_SEG documents takes one contiguous part of the visit
// array (in the order the segments' atomics arrive); within it, documents
// ascend.  cnt and first hold whole segments.
constexpr int VISIT_SEG = 4096;

__global__ __launch_bounds__(256) void k_visit_alloc(const uint32_t *__restrict__ cnt, uint32_t *__restrict__ first,
                                                     uint32_t *__restrict__ total) {
  __shared__ uint32_t wsum[4];
  __shared__ uint32_t s_base;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t d = (int64_t)blockIdx.x * VISIT_SEG + threadIdx.x * 16;
  uint4 x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = ((const uint4 *)(cnt + d))[i];
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) sum += x[i].x + x[i].y + x[i].z + x[i].w;
  uint32_t incl = sum;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const uint32_t y = __shfl_up(incl, m, 64);
    if (lane >= m) incl += y;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  if (threadIdx.x == 0) s_base = atomicAdd(total, wsum[0] + wsum[1] + wsum[2] + wsum[3]);
  __syncthreads();
  uint32_t at = s_base + incl - sum;
  for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint4 y;
    y.x = at;
    y.y = y.x + x[i].x;
    y.z = y.y + x[i].y;
    y.w = y.z + x[i].z;
    at = y.w + x[i].w;
    ((uint4 *)(first + d))[i] = y;
  }
}

__global__ __launch_bounds__(256) void k_visit_fill(const int32_t *__restrict__ cand_ids,
                                                    const int32_t *__restrict__ n_valid, int ncand,
                                                    const uint32_t *__restrict__ first,
                                                    const uint32_t *__restrict__ rank, uint32_t *__restrict__ visit) {
  const int64_t q = blockIdx.y;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_valid[q]) return;
  const int64_t p = q * ncand + i;
  visit[first[cand_ids[p]] + rank[p]] = (uint32_t)p;
}

// ------------------------------------------------------------------ queries
// The rounded queries as MFMA column operands in fp16: element i of lane l in
// step s of column block cb of query q, at ((q NCB + cb) 8 + s) 512 + 8 l + i,
// is dimension 64 (l / 32) + 8 s + i of query token 32 cb + l % 32, so a
// step's operand is one contiguous KB.
__global__ __launch_bounds__(256) void k_query_operand(const uint16_t *__restrict__ Qs, int64_t n8,
                                                       uint16_t *__restrict__ Qf) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;  // one 16-byte group of Qf
  if (e >= n8) return;
  const int l = (int)(e & 63), s = (int)((e >> 6) & 7);
  const int64_t block = e >> 9;  // q * NCB + cb: 32 rows of Qs
  const uint4 x = *(const uint4 *)(Qs + (block * 32 + (l & 31)) * 128 + 64 * (l >> 5) + 8 * s);
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
  f16x8 y;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    y[2 * i] = (_Float16)__uint_as_float(w[i] << 16);
    y[2 * i + 1] = (_Float16)__uint_as_float(w[i] & 0xFFFF0000u);
  }
  *(f16x8 *)(Qf + e * 8) = y;
}

// ------------------------------------------------------------------ scoring
// Tiles (32 tokens, 8 KB) of LDS per workgroup: 48 KB or 40 KB, so that three
// workgroups share a CU and one decodes while the others multiply.
template <int NCB>
constexpr int ds_tiles() { return NCB == 1 ? 6 : 5; }
// Jobs per wave whose running maxima are kept while a document longer than
// the LDS tiles goes through in pieces.
template <int NCB>
constexpr int ds_long_jobs() { return NCB == 1 ? 2 : 8; }

// sum over the 32 lanes of each half wave, in lanes 31 and 63
__device__ __forceinline__ int ds_half_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);  // row_half_mirror
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row_mirror
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
  return v;
}

__device__ __forceinline__ int rl(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ int64_t rl64(int64_t v, int lane) {
  return (int64_t)(((uint64_t)(uint32_t)rl((int)((uint64_t)v >> 32), lane) << 32) | (uint32_t)rl((int)v, lane));
}

// Workgroup b scores the visits of documents [b * ndb, (b + 1) * ndb), ndb
// <= 64: lane l of every wave holds document l's slice of visits, tokens and
// tiles.  Documents with visits are taken in bundles of at most TL tiles.  A
// bundle is decoded by the four waves together (units of half a tile: 32
// tokens x 64 dimensions), then its jobs are dealt to the waves: a job is 64
// query columns against one document, two visits (NCB = 1) or one (NCB = 2).
// Tile rows past a document repeat its last token, which leaves the maximum
// as it is.  A document of more than TL tiles goes through LDS in pieces for
// every JW jobs of a wave, the running maxima kept in LDS.
template <int NBITS, int NCB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_doc_score(
    const uint16_t *__restrict__ Qf, int Tq, int ncand, const uint16_t *__restrict__ cent16,
    const int64_t *__restrict__ doc_off, const int32_t *__restrict__ cid, const uint8_t *__restrict__ codes,
    uint4 w_lo, uint4 w_hi, int64_t ndocs, int ndb, const uint32_t *__restrict__ cnt,
    const uint32_t *__restrict__ first, const uint32_t *__restrict__ visit, int32_t *__restrict__ fhat) {
  constexpr int TL = ds_tiles<NCB>(), JW = ds_long_jobs<NCB>();
  constexpr int CB = 16 * NBITS;                  // code bytes per token
  constexpr int MAXU = (2 * TL + 3) / 4;          // decode units per wave
  __shared__ f16x8 At[TL * 8 * 64];               // [tile][step][lane]
  __shared__ uint2 lut2[NBITS == 2 ? 256 : 1];    // code byte -> 4 weights
  __shared__ uint32_t lut4[NBITS == 4 ? 256 : 1];  // code byte -> 2 weights
  __shared__ float run[4][JW][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  {
    const uint32_t w8[8] = {w_lo.x, w_lo.y, w_lo.z, w_lo.w, w_hi.x, w_hi.y, w_hi.z, w_hi.w};
    auto w = [&](int u) {  // constant indices only: the words stay in registers
      uint32_t x = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) x = (u >> 1) == i ? w8[i] : x;
      return (u & 1) ? x >> 16 : x & 0xFFFFu;
    };
    const int e = threadIdx.x;
    if (NBITS == 2)
      lut2[e] = make_uint2(w(e & 3) | (w((e >> 2) & 3) << 16), w((e >> 4) & 3) | (w((e >> 6) & 3) << 16));
    else
      lut4[e] = w(e & 15) | (w(e >> 4) << 16);
  }
  const int64_t d = (int64_t)blockIdx.x * ndb + lane;
  int nv = 0, nt = 0, len = 0, vo = 0;
  int64_t beg = 0;
  if (lane < ndb && d < ndocs) nv = (int)cnt[d];
  if (nv > 0) {
    vo = (int)first[d];
    beg = doc_off[d];
    len = (int)(doc_off[d + 1] - beg);
    nt = (len + 31) >> 5;
  }
  const int nj = NCB == 1 ? (nv + 1) >> 1 : nv;
  unsigned long long todo = __ballot(nv > 0 && len > 0);

  // A wave's decode units (half a tile: 32 tokens x 64 dimensions) of the T
  // tiles of a bundle: lane l's tiles are those of `mine` lanes, at tile
  // slots ts .. ts + n - 1, from the document's tile t0 on.
  struct Units {
    int64_t tok[MAXU];
    int c[MAXU];
  };
  auto unit_ids = [&](Units &U, bool mine, int ts, int n, int t0, int T) {
#pragma unroll
    for (int k = 0; k < MAXU; ++k) {
      const int u = wave + 4 * k;
      U.tok[k] = 0;
      U.c[k] = 0;
      if (u >= 2 * T) continue;  // wave-uniform
      const int t = u >> 1;
      const int e = __builtin_ctzll(__ballot(mine && ts <= t && t < ts + n));
      const int row = 32 * (t0 + t - rl(ts, e)) + (lane & 31);
      U.tok[k] = rl64(beg, e) + min(row, rl(len, e) - 1);
      U.c[k] = cid[U.tok[k]];
    }
  };
  // Loads the units' centroid rows and codes, waits until every wave has read
  // the tiles before, then writes the decoded tokens.
  auto decode = [&](const Units &U, int T) {
    f16x8 cv[MAXU][4];
    uint32_t cw[MAXU][4];
    const int h = lane >> 5;
#pragma unroll
    for (int k = 0; k < MAXU; ++k) {
      const int u = wave + 4 * k, sh = u & 1;
      if (u >= 2 * T) continue;
      // steps 4 sh .. 4 sh + 3: dimensions 64 h + 32 sh .. + 31
      const f16x8 *cp = (const f16x8 *)(cent16 + (int64_t)U.c[k] * 128 + 64 * h + 32 * sh);
#pragma unroll
      for (int s = 0; s < 4; ++s) cv[k][s] = cp[s];
      const uint8_t *kp = codes + U.tok[k] * CB + (CB / 2) * h + (CB / 4) * sh;
      if (NBITS == 2) {
        const uint2 x = *(const uint2 *)kp;
        cw[k][0] = x.x;
        cw[k][1] = x.y;
      } else {
        const uint4 x = *(const uint4 *)kp;
        cw[k][0] = x.x;
        cw[k][1] = x.y;
        cw[k][2] = x.z;
        cw[k][3] = x.w;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < MAXU; ++k) {
      const int u = wave + 4 * k, sh = u & 1;
      if (u >= 2 * T) continue;
      f16x8 *out = At + ((u >> 1) * 8 + 4 * sh) * 64 + lane;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint4 x;
        if (NBITS == 2) {
          const uint32_t word = cw[k][s >> 1] >> (16 * (s & 1));
          const uint2 lo = lut2[word & 255u], hi = lut2[(word >> 8) & 255u];
          x = make_uint4(lo.x, lo.y, hi.x, hi.y);
        } else {
          const uint32_t word = cw[k][s];
          x = make_uint4(lut4[word & 255u], lut4[(word >> 8) & 255u], lut4[(word >> 16) & 255u], lut4[word >> 24]);
        }
        out[64 * s] = cv[k][s] + __builtin_bit_cast(f16x8, x);  // exact (see above)
      }
    }
  };
  // This wave's jobs of a batch, one per lane: job jbase + wave + 4 * lane.
  // Its visits p0 and p1 (p1 = p0 for a single one), where their query
  // operands start in Qf (16-byte units), and its tile slots.
  struct Jobs {
    uint32_t p0, p1, g0, g1;
    int ta, tb;
  };
  auto jobs_of = [&](unsigned long long set, int ts, int js, int jbase) {
    Jobs L;
    const int jx = jbase + wave + 4 * lane;
    uint32_t v = 0;
    bool two = false, found = false;
    L.ta = L.tb = 0;
    for (unsigned long long m = set; m; m &= m - 1) {
      // (other lanes are read outside of divergent code, where a lane that is
      // switched off need not hold its value)
      const int e = __builtin_ctzll(m);
      const int nve = rl(nv, e), nje = rl(nj, e), tse = rl(ts, e), nte = rl(nt, e);
      const uint32_t voe = (uint32_t)rl(vo, e);
      const int k = jx - rl(js, e);
      const bool in = k >= 0 && k < nje;
      v = in ? voe + (NCB == 1 ? 2 * k : k) : v;
      two = in ? NCB == 1 && 2 * k + 1 < nve : two;
      L.ta = in ? tse : L.ta;
      L.tb = in ? tse + nte : L.tb;
      found = found || in;
    }
    L.p0 = L.p1 = 0;
    if (found) {
      L.p0 = visit[v];
      L.p1 = two ? visit[v + 1] : L.p0;
    }
    L.g0 = L.p0 / (uint32_t)ncand * (NCB * 512);
    L.g1 = NCB == 1 ? L.p1 / (uint32_t)ncand * 512 : L.g0 + 512;
    return L;
  };
  f16x8 b0[8], b1[8];  // the query operand of the current job
  auto load_b = [&](const Jobs &L, int i) {
    const f16x8 *g0 = (const f16x8 *)Qf + rl((int)L.g0, i) + lane, *g1 = (const f16x8 *)Qf + rl((int)L.g1, i) + lane;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      b0[s] = g0[64 * s];
      b1[s] = g1[64 * s];
    }
  };
  float m0, m1;
  // One tile against the job's 64 columns; NEXT: the operand of job i of L
  // is loaded as the steps finish with the current one.
  auto tile = [&](int t, const Jobs *next, int i) {
    const f16x8 *a = At + t * 512 + lane;
    f32x16 x0, x1;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      x0[v] = 0.f;
      x1[v] = 0.f;
    }
    if (!next) {
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const f16x8 av = a[64 * s];
        x0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, b0[s], x0, 0, 0, 0);
        x1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, b1[s], x1, 0, 0, 0);
      }
    } else {
      const f16x8 *g0 = (const f16x8 *)Qf + rl((int)next->g0, i) + lane;
      const f16x8 *g1 = (const f16x8 *)Qf + rl((int)next->g1, i) + lane;
      f16x8 av[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) av[s] = a[64 * s];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        x0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[s], b0[s], x0, 0, 0, 0);
        x1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[s], b1[s], x1, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        b0[s] = g0[64 * s];
        b1[s] = g1[64 * s];
      }
    }
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      m0 = fmaxf(fmaxf(m0, x0[v]), x0[v + 1]);
      m1 = fmaxf(fmaxf(m1, x1[v]), x1[v + 1]);
    }
  };
  // Maxima of job i's 64 columns over tile slots ta .. tb - 1, with job i + 1
  // (of n) loaded on the way: lane l holds column l (NCB = 1: column l % 32 of
  // visit l / 32).
  auto multiply = [&](const Jobs &L, int i, int n, int ta, int tb) {
    m0 = m1 = -INFINITY;
    for (int t = ta; t < tb - 1; ++t) tile(t, nullptr, 0);
    if (i + 1 < n) tile(tb - 1, &L, i + 1);
    else tile(tb - 1, nullptr, 0);
    // the half waves hold the maxima of different rows: after the swap the
    // low half has both of column block 0, the high half both of block 1
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(m0), __float_as_uint(m1), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  auto put = [&](const Jobs &L, int i, float m) {
    const bool in = NCB == 1 ? (lane & 31) < Tq : lane < Tq;
    const int key = ds_half_sum(in ? to_key(m) : 0);
    const uint32_t p0 = (uint32_t)rl((int)L.p0, i);
    if (NCB == 1) {
      const uint32_t p1 = (uint32_t)rl((int)L.p1, i);
      if (lane == 31) fhat[p0] = key;
      if (lane == 63 && p1 != p0) fhat[p1] = key;
    } else {
      const int low = rl(key, 31);
      if (lane == 63) fhat[p0] = key + low;
    }
  };
  auto share = [&](int jobs) { return max(0, (jobs - wave + 3) >> 2); };  // of `jobs`, this wave's

  while (todo) {
    const int e0 = __builtin_ctzll(todo);
    const int nt0 = rl(nt, e0);
    if (nt0 > TL) {  // a long document, in pieces
      todo &= todo - 1;
      const int J = rl(nj, e0);
      for (int jb = 0; jb < J; jb += 4 * JW) {
        const Jobs L = jobs_of(1ull << e0, 0, 0, jb);
        const int n = share(min(J - jb, 4 * JW));
        for (int t0 = 0; t0 < nt0; t0 += TL) {
          const int T = min(TL, nt0 - t0);
          Units U;
          unit_ids(U, lane == e0, 0, T, t0, T);
          decode(U, T);
          load_b(L, 0);  // also without a job, so that no older operand stays live
          __syncthreads();
          for (int i = 0; i < n; ++i) {
            float m = multiply(L, i, n, 0, T);
            if (t0 > 0) m = fmaxf(m, run[wave][i][lane]);
            if (t0 + TL < nt0) run[wave][i][lane] = m;
            else put(L, i, m);
          }
        }
      }
      continue;
    }
    // a bundle: documents from e0 on while their tiles fit
    bool mine = false;
    int ts = 0, js = 0, T = 0, J = 0;
    unsigned long long m = todo;
    while (m) {
      const int e = __builtin_ctzll(m);
      const int te = rl(nt, e);
      if (T + te > TL) break;
      if (lane == e) {
        mine = true;
        ts = T;
        js = J;
      }
      T += te;
      J += rl(nj, e);
      m &= m - 1;
    }
    const unsigned long long set = todo & ~m;
    todo = m;
    Units U;
    unit_ids(U, mine, ts, nt, 0, T);
    Jobs L = jobs_of(set, ts, js, 0);
    decode(U, T);
    for (int jb = 0; jb < J; jb += 256) {
      const int n = share(min(J - jb, 256));
      if (jb > 0) L = jobs_of(set, ts, js, jb);
      load_b(L, 0);  // also without a job, so that no older operand stays live
      if (jb == 0) __syncthreads();
      for (int i = 0; i < n; ++i) put(L, i, multiply(L, i, n, rl(L.ta, i), rl(L.tb, i)));
    }
  }
}

// ------------------------------------------------------------ RaBitQ scoring
// The same from the 1-bit RaBitQ codes (k_rabitq.hip has the formula): a
// document's bits become fp16 zeros and ones in LDS once, and a visiting
// query's rotated token x is the sum of two fp16 values, hi = fp16(x) and lo =
// x - hi, both exact (x is a multiple of 2^-11 below 32 in magnitude for
// tokens of norm below 2.8, so hi rounds at 2^-6 or finer and lo has at most 5
// bits).  Their products with the bits add up in one fp32 accumulator that
// starts at -sum(x) / 2: <x, b> - sum(x) / 2 is a multiple of 2^-12 below 2^12,
// exact in any order.  One multiply by the token's factor g1 is the one
// rounding, as before.  With the document's tokens as rows, the maximum over
// tokens stays in a lane's registers.  Going query by query, the bits were
// expanded for every visit and the three 7-bit limbs of X chained by shifts:
// 12 int8 MFMA and about 250 vector instructions per 32 x 32 tile, the latter
// the bound; here 16 MFMA and 24, and the 16 KB of a visit's operand take as
// long to load (64 bytes per clock and CU).  256 queries of 4096 candidates on
// 20,000 documents of 64 tokens: 1500 us against 1859 us.

// One wave per query row: x = H diag(signs) q by the fast transform in fp32
// (lane l holds dimensions 2l and 2l + 1), its hi and lo parts in operand
// order (block q * NCB + cb: 512 groups of hi, then 512 of lo), and sum(x) / 2.
__global__ __launch_bounds__(256) void k_rq_operand(const uint16_t *__restrict__ Qs, int64_t rows,
                                                    const int8_t *__restrict__ signs, uint16_t *__restrict__ Qf,
                                                    float *__restrict__ half_sum) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const uint32_t w = ((const uint32_t *)(Qs + row * 128))[lane];
  float x0 = __uint_as_float(w << 16) * (float)signs[2 * lane];
  float x1 = __uint_as_float(w & 0xFFFF0000u) * (float)signs[2 * lane + 1];
  const float a = x0 + x1, b = x0 - x1;
  x0 = a;
  x1 = b;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const float y0 = __shfl_xor(x0, m, 64), y1 = __shfl_xor(x1, m, 64);
    x0 = lane & m ? y0 - x0 : x0 + y0;
    x1 = lane & m ? y1 - x1 : x1 + y1;
  }
  const _Float16 h0 = (_Float16)x0, h1 = (_Float16)x1;
  const _Float16 l0 = (_Float16)(x0 - (float)h0), l1 = (_Float16)(x1 - (float)h1);
  // dimensions 2l, 2l + 1: half d / 64, step d % 64 / 8, element d % 8
  const int d = 2 * lane;
  uint32_t *o = (uint32_t *)(Qf + (row >> 5) * 8192 + ((d & 63) >> 3) * 512 + (32 * (d >> 6) + (int)(row & 31)) * 8 + (d & 7));
  o[0] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | (uint32_t)__builtin_bit_cast(uint16_t, h1) << 16;
  o[2048] = (uint32_t)__builtin_bit_cast(uint16_t, l0) | (uint32_t)__builtin_bit_cast(uint16_t, l1) << 16;
  float sum = x0 + x1;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
  if (lane == 0) half_sum[row] = 0.5f * sum;
}

// Bundles and jobs as k_doc_score; a job is one visit, its column blocks one
// after the other.
template <int NCB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_doc_score_rq(
    const uint16_t *__restrict__ Qf, const float *__restrict__ half_sum, int Tq, int ncand,
    const int64_t *__restrict__ doc_off, const uint8_t *__restrict__ bits, const float *__restrict__ g1, int64_t ndocs,
    int ndb, const uint32_t *__restrict__ cnt, const uint32_t *__restrict__ first, const uint32_t *__restrict__ visit,
    int32_t *__restrict__ fhat) {
  constexpr int TL = 6, MAXU = 3;
  constexpr int JW = NCB == 1 ? 2 : 1;            // visits per wave of a long document at a time
  __shared__ f16x8 At[TL * 8 * 64];               // [tile][step][lane]
  __shared__ __align__(16) float gt[TL * 32];     // the rows' factors
  __shared__ float run[4][JW * NCB][32];
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t d = (int64_t)blockIdx.x * ndb + lane;
  int nv = 0, nt = 0, len = 0, vo = 0;
  int64_t beg = 0;
  if (lane < ndb && d < ndocs) nv = (int)cnt[d];
  if (nv > 0) {
    vo = (int)first[d];
    beg = doc_off[d];
    len = (int)(doc_off[d + 1] - beg);
    nt = (len + 31) >> 5;
  }
  unsigned long long todo = __ballot(nv > 0 && len > 0);

  // (as k_doc_score: units of half a tile, loads before the barrier)
  auto decode = [&](bool mine, int ts, int n, int t0, int T) {
    uint32_t w[MAXU];
    float g[MAXU];
#pragma unroll
    for (int k = 0; k < MAXU; ++k) {
      const int u = wave + 4 * k;
      w[k] = 0;
      g[k] = 0.f;
      if (u >= 2 * T) continue;  // wave-uniform
      const int t = u >> 1;
      const int e = __builtin_ctzll(__ballot(mine && ts <= t && t < ts + n));
      const int row = 32 * (t0 + t - rl(ts, e)) + (lane & 31);
      const int64_t tok = rl64(beg, e) + min(row, rl(len, e) - 1);
      // steps 4 sh .. 4 sh + 3: dimensions 64 h + 32 sh .. + 31
      w[k] = *(const uint32_t *)(bits + tok * 16 + 8 * h + 4 * (u & 1));
      g[k] = g1[tok];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < MAXU; ++k) {
      const int u = wave + 4 * k, sh = u & 1;
      if (u >= 2 * T) continue;
      f16x8 *out = At + ((u >> 1) * 8 + 4 * sh) * 64 + lane;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t y = w[k] >> (8 * s);
        uint4 x;  // bit i of the byte as fp16 0 or 1
        x.x = (y & 1u) * 0x3C00u | (y >> 1 & 1u) * 0x3C000000u;
        x.y = (y >> 2 & 1u) * 0x3C00u | (y >> 3 & 1u) * 0x3C000000u;
        x.z = (y >> 4 & 1u) * 0x3C00u | (y >> 5 & 1u) * 0x3C000000u;
        x.w = (y >> 6 & 1u) * 0x3C00u | (y >> 7 & 1u) * 0x3C000000u;
        out[64 * s] = __builtin_bit_cast(f16x8, x);
      }
      if (sh == 0 && h == 0) gt[32 * (u >> 1) + lane] = g[k];
    }
    __syncthreads();
  };
  // Largest estimate of each of a block's 32 columns over tile slots ta .. tb
  // - 1, in both half waves; g is the block's first group of Qf.
  auto block_max = [&](uint32_t g, float hs, int ta, int tb) {
    f16x8 b0[8], b1[8];
    const f16x8 *gp = (const f16x8 *)Qf + g + lane;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      b0[s] = gp[64 * s];
      b1[s] = gp[512 + 64 * s];
    }
    float m = -INFINITY;
    for (int t = ta; t < tb; ++t) {
      const f16x8 *a = At + t * 512 + lane;
      f32x16 x;
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = -hs;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const f16x8 av = a[64 * s];
        x = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, b0[s], x, 0, 0, 0);
        x = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, b1[s], x, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; v += 4) {
        // registers v .. v + 3 hold rows 8 (v / 4) + 4 h .. + 3
        const float4 gv = *(const float4 *)(gt + 32 * t + 2 * v + 4 * h);
        m = fmaxf(fmaxf(m, gv.x * x[v]), gv.y * x[v + 1]);
        m = fmaxf(fmaxf(m, gv.z * x[v + 2]), gv.w * x[v + 3]);
      }
    }
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  // the columns' keys rint(m 2^22) summed in two 32-bit halves (a key is below
  // 2^40 in magnitude), in lane 31
  auto key_sum = [&](const float (&m)[NCB]) {
    long long total = 0;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const float r = rintf(m[cb] * KEY_SCALE), hi = floorf(r * (1.0f / 65536.0f));
      const bool in = 32 * cb + (lane & 31) < Tq;
      const int sh = ds_half_sum(in ? (int)hi : 0), sl = ds_half_sum(in ? (int)(r - hi * 65536.0f) : 0);
      total += (long long)sh * 65536 + sl;
    }
    return (int32_t)std::min<long long>(INT32_MAX, std::max<long long>(-INT32_MAX, total));
  };

  while (todo) {
    const int e0 = __builtin_ctzll(todo);
    const int nt0 = rl(nt, e0);
    if (nt0 > TL) {  // a long document, in pieces
      todo &= todo - 1;
      const int J = rl(nv, e0);
      const uint32_t v0 = (uint32_t)rl(vo, e0);
      for (int jb = 0; jb < J; jb += 4 * JW) {
        for (int t0 = 0; t0 < nt0; t0 += TL) {
          const int T = min(TL, nt0 - t0);
          decode(lane == e0, 0, T, t0, T);
          for (int i = 0; i < JW; ++i) {
            const int jx = jb + wave + 4 * i;
            if (jx >= J) break;
            const uint32_t p = visit[v0 + jx], q = p / (uint32_t)ncand;
            float m[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
              m[cb] = block_max((q * NCB + cb) * 1024, half_sum[(q * NCB + cb) * 32 + (lane & 31)], 0, T);
              float *r = &run[wave][i * NCB + cb][lane & 31];
              if (t0 > 0) m[cb] = fmaxf(m[cb], *r);
              if (t0 + TL < nt0) *r = m[cb];
            }
            if (t0 + TL >= nt0) {
              const int32_t key = key_sum(m);
              if (lane == 31) fhat[p] = key;
            }
          }
        }
      }
      continue;
    }
    bool mine = false;
    int ts = 0, js = 0, T = 0, J = 0;
    unsigned long long m = todo;
    while (m) {
      const int e = __builtin_ctzll(m);
      const int te = rl(nt, e), je = rl(nv, e);
      if (T + te > TL) break;
      mine = lane == e ? true : mine;
      ts = lane == e ? T : ts;
      js = lane == e ? J : js;
      T += te;
      J += je;
      m &= m - 1;
    }
    todo = m;
    decode(mine, ts, nt, 0, T);
    for (int jx = wave; jx < J; jx += 4) {
      const int e = __builtin_ctzll(__ballot(mine && js <= jx && jx < js + nv));
      const uint32_t p = visit[(uint32_t)rl(vo, e) + (uint32_t)(jx - rl(js, e))], q = p / (uint32_t)ncand;
      const int ta = rl(ts, e), tb = ta + rl(nt, e);
      float mm[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        mm[cb] = block_max((q * NCB + cb) * 1024, half_sum[(q * NCB + cb) * 32 + (lane & 31)], ta, tb);
      const int32_t key = key_sum(mm);
      if (lane == 31) fhat[p] = key;
    }
  }
}

// ------------------------------------------------------------------ host
static int64_t visit_docs(int64_t ndocs) { return (ndocs + VISIT_SEG - 1) / VISIT_SEG * VISIT_SEG; }

// Scratch: the query operand (256 bytes a row, 516 for RaBitQ's two parts and
// sums), a count and a first visit per document (whole segments) with the
// running total, and the visits.
size_t doc_score_scratch_bytes(int64_t nq, int TQP, int64_t ndocs, int ncand, bool rq) {
  return (size_t)nq * TQP * (rq ? 516 : 256) + (size_t)(2 * visit_docs(ndocs) + 64) * 4 + (size_t)nq * ncand * 4 + 1024;
}

// Sorts the visits of the kept candidates by document; ranks are taken in
// fhat, which the scoring writes afterwards.
struct Visits {
  uint32_t *cnt, *first, *visit;
  unsigned blocks;  // workgroups of ndb documents each
  int ndb;
};
static Visits sort_visits(int64_t nq, int64_t ndocs, const int32_t *cand_ids, const int32_t *n_valid, int ncand,
                          uint32_t *scratch, int32_t *fhat, hipStream_t s) {
  const int64_t nd = visit_docs(ndocs);
  Visits V;
  V.cnt = scratch;
  uint32_t *total = V.cnt + nd;
  V.first = total + 64;
  V.visit = V.first + nd;
  const dim3 gv((unsigned)((ncand + 255) / 256), (unsigned)nq);
  launch_fill_zero(V.cnt, (size_t)(nd + 64) * 4, s);
  hipLaunchKernelGGL(k_visit_count, gv, dim3(256), 0, s, cand_ids, n_valid, ncand, V.cnt, (uint32_t *)fhat);
  hipLaunchKernelGGL(k_visit_alloc, dim3((unsigned)(nd / VISIT_SEG)), dim3(256), 0, s, V.cnt, V.first, total);
  hipLaunchKernelGGL(k_visit_fill, gv, dim3(256), 0, s, cand_ids, n_valid, ncand, V.first, (const uint32_t *)fhat,
                     V.visit);
  // documents per workgroup: 64, fewer while that leaves under about 6144
  // workgroups
  V.ndb = 64;
  while (V.ndb > 1 && (ndocs + V.ndb - 1) / V.ndb < 6144) V.ndb >>= 1;
  V.blocks = (unsigned)((ndocs + V.ndb - 1) / V.ndb);
  return V;
}

// Whether a batch goes by document.  Both ways were timed (probe and scoring,
// as by query the probe also writes S^T) on 20,000 to 2.2M documents, with 4 to
// 1024 queries of 4 to 64 tokens and 0.5 to 42 visits a document.  Within about
// a tenth they take, in ns,
//   by query     30e3 + 0.044 nq ncent B + b V L
//   by document  78e3 + 0.022 nq ncent B + d D L + 0.0108 B V L + 0.83 ndocs + P
// for V visits, D documents with a visit, L tokens a document and B blocks of
// 32 query tokens.  b is 0.013 at 4 and 0.019 at 32 query tokens (a row of S^T
// that several tokens share is read once), 0.034 at 64; with 4-bit codes a tenth
// more, and 0.025 a block where a query's S^T is past an L2; d, the decoding,
// 0.020 and 0.033.  So few query tokens and few
// visits a document go by query: by document takes 1.5 times as long with 64
// queries of 4 tokens and 4096 candidates on 100,000 documents, 1.3 times with
// 256 and 8192 on 1M, where 32 tokens take 0.96 and 1024 queries 0.73.
//
// A visit here is a kept candidate: no more than the probed lists hold, where
// the lists are about even.
//
// With dense lists some documents are kept by many queries, in small
// collections by nearly all (p, taken as 16 ncand / ndocs), and the workgroups
// that score them are busy for 8 B p nq L together: P is what that is above half
// of the other workgroups' time (the terms of D, V and ndocs).  938 queries of 51
// tokens on 2,211 documents, 4-bit codes: probe and scoring 0.98 ms by document
// and 0.56 by query with 87 candidates, 1.64 and 1.25 with 400.
//
// One workgroup scores a document, so a document far longer than the others
// keeps the rest of the chip waiting: with 256 queries of 4096 candidates on
// 100,000 documents of 64 tokens, one of them of 600, 1200, 8000 and 40,000,
// by document takes 1.18, 1.66, 5.6 and 26.6 ms, by query 1.34, 1.35, 1.4 and
// 2.1.  Its chain is as long as its tokens, the rest's share of the chip as
// long as ncand L / 256; it is left aside below 0.4 of that (0.7 of RaBitQ's,
// whose scoring by query is slower: a document of 2,400 and 16,384 candidates,
// 0.93 of the time by query; of 600 and 4096, 0.87; of 2,400 and 4096, 1.72).
//
// Besides, by document has to have 2^16 visits, 36 tokens a document (1,000 of
// 32 tokens and 256 visits each: 0.167 against 0.157 ms) and 7 visits a
// document of 64 tokens, 2 where there are dense lists.  (Below that line it
// was up to a third slower with 256 queries and fewer and up to a third faster
// with 512 and more; those stay by query.)
//
// The RaBitQ scoring has no S^T.  By document it takes 0.74 to 0.94 of the
// time above the same line, but 1.04 to 1.07 with 512 queries of 512
// candidates: with many queries of 32 tokens their operands no longer stay in
// an L2, and few candidates each do not make up for it.
bool doc_score_grouped(int64_t nq, int Tq, int nprobe, int ncand, int64_t ndocs, int64_t ntok, int64_t nnz,
                       int max_doc_len, int ncent, int ndense, int nbits, bool rq) {
  if (ndocs <= 0 || ntok < 36 * ndocs) return false;
  const double n = (double)ndocs, L = (double)ntok / n;
  const double line = (ndense > 0 ? 2 : 7) * 64 * n / L;
  if ((double)nq * ncand < (1 << 16) || (double)nq * ncand < line) return false;
  double kept = ncand;
  if (ndense == 0) kept = std::min(kept, (double)Tq * nprobe * (double)nnz / ncent);
  if (max_doc_len > 4 * L && max_doc_len > (rq ? 0.7 : 0.4) * kept * L / 256) return false;
  if (rq) return ncand >= 1024 || (Tq > 32 && ndense == 0);
  const double B = Tq > 32 ? 2 : 1, V = (double)nq * kept;
  const double D = n * (1 - std::exp(-(ndense > 0 ? 0.5 : 1.0) * V / n));
  const double b2 = 0.0127 + 0.0093 * (B - 1) + 0.000185 * Tq;
  const double b = nbits != 4 ? b2 : (double)ncent * B < 32768 ? 1.1 * b2 : 0.025 + 0.022 * (B - 1);
  const double by_query = 30e3 + 0.044 * (double)nq * ncent * B + b * V * L;
  const double spread = (nbits == 4 ? 0.033 : 0.020) * D * L + 0.0108 * B * V * L + 0.83 * n;
  const double p = std::min(1.0, 16.0 * ncand / n);
  const double popular = ndense > 0 ? std::max(0.0, 8 * B * p * (double)nq * L - 0.5 * spread) : 0.0;
  const double by_doc = 78e3 + 0.022 * (double)nq * ncent * B + spread + popular;
  // (20 us in its favour: in small batches it was measured closer than that)
  return by_doc - 20e3 < by_query;
}

void launch_doc_score(const uint16_t *Qs, int64_t nq, int Tq, int TQP, const uint16_t *cent16,
                      const int64_t *doc_off, const int32_t *cid, const uint8_t *codes, int nbits,
                      const uint16_t *weights_host, int64_t ndocs, const int32_t *cand_ids, const int32_t *n_valid,
                      int ncand, void *scratch, int32_t *fhat, hipStream_t s) {
  if (nq <= 0 || ncand <= 0) return;
  uint16_t *Qf = (uint16_t *)scratch;
  uint32_t w[8] = {0};
  const int B = 1 << nbits;
  for (int u = 0; u < B; ++u)
    w[u >> 1] |= (uint32_t)f16_of_grid_k(grid_k_of_float(float_of_bf16(weights_host[u]))) << (16 * (u & 1));
  const uint4 w_lo = make_uint4(w[0], w[1], w[2], w[3]), w_hi = make_uint4(w[4], w[5], w[6], w[7]);
  const int64_t n8 = nq * TQP * 16;
  hipLaunchKernelGGL(k_query_operand, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s, Qs, n8, Qf);
  const Visits V = sort_visits(nq, ndocs, cand_ids, n_valid, ncand, (uint32_t *)(Qf + (size_t)nq * TQP * 128), fhat, s);
#define CHIMERA_DS(NB, NC)                                                                                            \
  hipLaunchKernelGGL((k_doc_score<NB, NC>), dim3(V.blocks), dim3(256), 0, s, Qf, Tq, ncand, cent16, doc_off, cid, codes, \
                     w_lo, w_hi, ndocs, V.ndb, V.cnt, V.first, V.visit, fhat)
  if (nbits == 2 && TQP == 32) CHIMERA_DS(2, 1);
  else if (nbits == 2) CHIMERA_DS(2, 2);
  else if (TQP == 32) CHIMERA_DS(4, 1);
  else CHIMERA_DS(4, 2);
#undef CHIMERA_DS
}

void launch_doc_score_rq(const uint16_t *Qs, int64_t nq, int Tq, int TQP, const int8_t *signs, const int64_t *doc_off,
                         const uint8_t *bits, const float *g1, int64_t ndocs, const int32_t *cand_ids,
                         const int32_t *n_valid, int ncand, void *scratch, int32_t *fhat, hipStream_t s) {
  if (nq <= 0 || ncand <= 0) return;
  const int64_t rows = nq * TQP;
  uint16_t *Qf = (uint16_t *)scratch;
  float *half_sum = (float *)(Qf + (size_t)rows * 256);
  hipLaunchKernelGGL(k_rq_operand, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, Qs, rows, signs, Qf, half_sum);
  const Visits V = sort_visits(nq, ndocs, cand_ids, n_valid, ncand, (uint32_t *)(half_sum + rows), fhat, s);
  if (TQP == 32)
    hipLaunchKernelGGL((k_doc_score_rq<1>), dim3(V.blocks), dim3(256), 0, s, Qf, half_sum, Tq, ncand, doc_off, bits, g1,
                       ndocs, V.ndb, V.cnt, V.first, V.visit, fhat);
  else
    hipLaunchKernelGGL((k_doc_score_rq<2>), dim3(V.blocks), dim3(256), 0, s, Qf, half_sum, Tq, ncand, doc_off, bits, g1,
                       ndocs, V.ndb, V.cnt, V.first, V.visit, fhat);
}

}  // namespace chimera
