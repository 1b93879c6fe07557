// k_prune.hip - candidate generation and candidate refinement.
//
// Candidate set (Sec. 3.2, the set S): documents with a token in a probed
// posting list.  Partial score (Sec. 3.2, the F' definition; Alg. 2):
//   F'(V) = sum_j max{ S[j][c] : c in C_j, V in list(c) }   (0 if none).
// The max is taken by visiting each query token's probed lists in rank
// order (C_j is sorted by S descending): the first list of rank r that holds
// V carries the maximum, so one atomic OR on a per-(query, doc) bit mask
// detects the first hit and one integer atomic add accumulates F'.  Integer
// atomics make the result independent of scheduling.  This plays the role of
// the paper's fused atomic aggregation (Sec. 4.2, Alg. 4) with one update
// per (doc, query token) instead of an atomic max per retrieved token, and
// with the score table held in LDS one document range at a time.
#include <algorithm>
#include <climits>

#include "device_common.h"
#include "internal.h"

namespace chimera {

__global__ __launch_bounds__(256) void k_fill_zero(uint4 *__restrict__ p, size_t n16) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
    p[i] = make_uint4(0, 0, 0, 0);
}

void launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
  // scratch carve-outs are 256-byte aligned and sized in 256-byte steps
  size_t n16 = (bytes + 15) / 16;
  if (!n16) return;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, s, (uint4 *)p, n16);
}

// Workgroup (query q, group g): the document ranges [d0, d0 + R) of a
// contiguous group of ranges, one after the other, in one of two ways.
//
// Through chains and a table, where walk_by_chains says so and the query has at
// most WALK_TAB_BITS dense groups (below): F' is a maximum per query token, so
// it needs no order.  The dense groups' own F' is a table of 2^g sums, built
// once per workgroup, that a document looks up by the bits of its dense mask.
// Every posting entry of the range is linked into its document's chain in LDS;
// documents with a chain (about a quarter on Zipf-popular corpora) are listed
// and taken one a lane: up to four entries are sorted by rank and each corrects
// the table's sum for the tokens that no better entry or dense group holds;
// longer chains are taken by the whole wave, a query token a lane.  Three
// barriers a range (the chains are complete; the range has been read; the entry
// counter is cleared), where the other way has one a rank and more; the group's
// histogram is kept in LDS and added once.  1024 queries x 2.2M documents, 16
// ranks: 23.8 -> 20.3 ms; 1M documents, 8 ranks: 10.0 ms either way.
//
// Rank by rank, else, and from the first range on that holds more entries than
// the chains take (WALK_NODES).  The state of a range
// (per document: the mask of query tokens already credited, and F') lives in
// LDS, so the updates are LDS atomics and each document's F' is written to
// HBM once.  Query tokens that probe the same centroid at the same rank form
// a group whose list is walked once, with the group's token mask and score
// sum (on the Zipf-popular corpora this halves the entries walked).  Ranks
// are applied in order, one barrier apart, so the first rank whose list
// holds a document gives each token its maximum: one atomic OR of the
// group's mask tells which tokens see the document for the first time.
//
// Every list's next entries wait in registers, loaded a range ahead:
//  * a short list (a few entries per range, the usual case) belongs to one
//    thread for the workgroup's lifetime, with a window of its next WIN
//    entries;
//  * a long list (more than WALK_LONG entries expected per range) belongs to
//    one wave, with a window of its next 64 entries (one per lane);
//  * a dense list (see dense_lists) is not walked: each thread applies it to
//    the documents it owns from their 64-bit masks, loaded a range ahead.
// At the start of a range the windows' entries inside it are copied into
// per-rank buckets in LDS and the windows are refilled; the ranks then run
// over the buckets, so they wait on no memory.  Only a list with more
// entries in one range than its window holds goes on through memory, at its
// rank.  The workgroup then writes F' (or NO_HIT for documents outside S_Q)
// and adds the range's histogram of the top 12 bits of the order key to the
// query's histogram, the first pass of the refinement select.  Workgroup b
// runs on XCD b % 8: with 8 or more queries all groups of query q run on XCD
// q % 8, with fewer they spread over every XCD.
constexpr int WALK_THREADS = 512;
constexpr int WALK_WAVES = WALK_THREADS / 64;
constexpr int WALK_LONG = 4;        // expected entries per range above which a list belongs to a wave
constexpr int WALK_LONG_SLOTS = 4;  // lists per wave
constexpr int WALK_MAX_LONG = WALK_LONG_SLOTS * WALK_WAVES;  // beyond that, lists stay with threads
constexpr int WALK_MAX_LISTS = 4 * WALK_THREADS;              // Tq * nprobe
constexpr int WALK_SHORT_ENTRIES = 4096;                      // short-list windows in all
constexpr int WALK_BUCKET = WALK_SHORT_ENTRIES + WALK_MAX_LONG * 64;
constexpr int WALK_DOC_BITS = 13;   // a bucket entry: list index << 13 | document in the range

// Dense groups of a query up to which a range is walked through their table of
// sums (see k_cand_walk), and the entries such a range holds at most.
constexpr int WALK_TAB_BITS = 11;
constexpr int WALK_NODES = 4096;
constexpr int WALK_HITS = (WALK_BUCKET - WALK_NODES) / WALK_WAVES;  // documents with entries a wave lists at a time

// Window of a thread's short list: WIN = 8, 4 or 2 entries as a thread owns
// 1, 2 or 4 lists (WALK_SHORT_ENTRIES in all).
template <int LPT>
constexpr int walk_win() {
  return WALK_SHORT_ENTRIES / (LPT * WALK_THREADS);
}

// Documents per range: 4096 with 32-bit token masks, 2048 with 64-bit masks
// (two workgroups per compute unit; 8192 needs one, measured 4x slower).
static inline int walk_range_docs(int TQP, int, int) { return TQP == 32 ? 4096 : 2048; }

// LDS cursor of a wave's list: entries ivf_doc[beg .. beg + len), pos the
// first entry not yet credited; t its list index r * Tq + j.
struct LongList {
  int64_t beg;
  int32_t pos, len, t, rank, n, off;  // n, off: entries in the current range and their bucket offset
};

// Register state of a thread's short list: entries lp[0 .. len); e[i] holds
// lp[pos0 + i] for i < avail; e[0 .. c) are credited.  rank < 0: no list.
template <int WIN>
struct ShortList {
  const int32_t *lp;
  int32_t len, pos0, avail, c, rank, t;
  int32_t e[WIN];
};

// Credits the group (gmask, gsum) to document v of the range: the tokens of
// the group not yet seen there add their scores.
template <typename MaskT>
__device__ __forceinline__ void credit(MaskT *smask, int32_t *sfp, int v, MaskT gmask, int32_t gsum,
                                       const int32_t *keys) {
  const MaskT fresh = gmask & ~atomicOr(&smask[v], gmask);
  if (fresh == gmask) {
    atomicAdd(&sfp[v], gsum);
  } else if (fresh) {
    int32_t add = 0;
    for (MaskT m = fresh; m; m &= m - 1) add += keys[__builtin_ctzll((unsigned long long)m)];
    atomicAdd(&sfp[v], add);
  }
}

// One wave walks a list from pos up to the range's end d1, U blocks of 64
// entries per step; leaves pos at the first entry >= d1.
template <int U, typename MaskT>
__device__ __forceinline__ void walk_list(const int32_t *__restrict__ list, int32_t len, int64_t d0, int64_t d1,
                                          MaskT gmask, int32_t gsum, const int32_t *keys, int lane, MaskT *smask,
                                          int32_t *sfp, int32_t &pos) {
  bool done = false;
  while (!done) {
    int32_t doc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t p = pos + 64 * u + lane;
      doc[u] = p < len ? list[p] : INT32_MAX;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = doc[u] < d1;
      if (in && !done) credit(smask, sfp, (int)(doc[u] - d0), gmask, gsum, keys);
      const unsigned long long out = __ballot(!in);  // lanes at or past the range's end
      if (out && !done) {
        pos += 64 * u + (__ffsll((long long)out) - 1);
        done = true;
      }
    }
    if (!done) pos += 64 * U;
  }
}

// Entries lp[pos .. pos + n) of a window, every load issued (indices past
// the list read its last entry and are not used), so each range issues the
// same loads.
template <int N>
__device__ __forceinline__ void load_window(const int32_t *lp, int32_t pos, int32_t len, int32_t (&e)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = lp[min(pos + i, len - 1)];
}

// Byte offsets of the walk's LDS arrays (each 16-byte aligned).
struct WalkLds {
  size_t smask, sfp, bucket, ll, lmask, lsum, skey, scid, dcount, bcnt, bbase, dgm, dgs, dls, nlong, dtab, dtok, dgrp,
      total;
};
__host__ __device__ inline WalkLds walk_lds_layout(int R, int mask_bytes, int nprobe, int Tq, bool tab) {
  const size_t nl = (size_t)nprobe * Tq;
  WalkLds L;
  size_t o = 0;
  auto take = [&o](size_t bytes) {
    const size_t at = o;
    o += (bytes + 15) / 16 * 16;
    return at;
  };
  L.smask = take((size_t)R * mask_bytes);
  L.sfp = take((size_t)R * 4);
  L.bucket = take((size_t)WALK_BUCKET * 4);
  L.ll = take(WALK_MAX_LONG * sizeof(LongList));
  L.lmask = take(nl * mask_bytes);
  L.lsum = take(nl * 4);
  L.skey = take(nl * 4);
  L.dcount = take((size_t)nprobe * 4);
  L.bcnt = take((size_t)nprobe * 4);
  L.bbase = take((size_t)nprobe * 4);
  // the table takes the place of what its ranges do not read, so that a query
  // that had two workgroups a CU (640 to 928 lists: with 8 KB more, one) keeps them
  L.dtab = o;
  L.scid = take(nl * 4);
  L.dgm = take(nl * mask_bytes);
  L.dgs = take(nl * 4);
  L.dls = take(nl);
  if (tab) o = o > L.dtab + (4u << WALK_TAB_BITS) ? o : L.dtab + (4u << WALK_TAB_BITS);
  L.nlong = take(12);
  L.dtok = take(tab ? 64 * 2 : 0);
  L.dgrp = take(tab ? WALK_TAB_BITS * 8 : 0);
  L.total = o;
  return L;
}

// TAB: the walk through chains and a table, with the other way for the queries
// and ranges that it does not take; else every range rank by rank.  (With 128
// registers, two workgroups a CU; rank by rank with two lists a thread and all
// the registers it asks for: 186.2 against 190.2 ms for 1024 queries of 32
// tokens, 1M documents and 32 ranks, where the others gain up to 6%.)
template <typename MaskT, int R, int LPT, bool TAB>
__global__ __launch_bounds__(WALK_THREADS) __attribute__((amdgpu_waves_per_eu(TAB || LPT != 2 ? 4 : 1))) void k_cand_walk(
    const int32_t *__restrict__ cent_ids, const int32_t *__restrict__ cent_keys, int64_t nq, int Tq, int TQP,
    int nprobe, const int64_t *__restrict__ ivf_off, const int32_t *__restrict__ ivf_doc, int64_t ndocs, int ncent,
    int ndense, const int8_t *__restrict__ dense_slot, const uint64_t *__restrict__ doc_dense,
    const uint64_t *__restrict__ deleted, int nranges, int G, int M, int32_t *__restrict__ fp,
    uint32_t *__restrict__ hist) {
  constexpr int DPT = R / WALK_THREADS;  // documents of a range each thread owns in the dense phase
  constexpr int WIN = walk_win<LPT>();
  static_assert(R * sizeof(MaskT) >= SEL_BINS * 4, "the histogram reuses the mask array");
  static_assert(R <= (1 << WALK_DOC_BITS), "a bucket entry holds the document in 13 bits");
  extern __shared__ __align__(16) unsigned char walk_lds[];
  const int nl = nprobe * Tq;
  const WalkLds lay = walk_lds_layout(R, (int)sizeof(MaskT), nprobe, Tq, TAB);
  MaskT *smask = (MaskT *)(walk_lds + lay.smask);        // [R] tokens already credited, per document
  int32_t *sfp = (int32_t *)(walk_lds + lay.sfp);        // [R] F' accumulators
  uint32_t *bucket = (uint32_t *)(walk_lds + lay.bucket);  // [WALK_BUCKET] the range's entries, by rank
  LongList *LL = (LongList *)(walk_lds + lay.ll);        // [WALK_MAX_LONG]
  MaskT *lmask = (MaskT *)(walk_lds + lay.lmask);        // [nl] group token masks
  int32_t *lsum = (int32_t *)(walk_lds + lay.lsum);      // [nl] group score sums
  int32_t *skey = (int32_t *)(walk_lds + lay.skey);      // [nl] S[j][c] keys, index r * Tq + j
  int32_t *scid = (int32_t *)(walk_lds + lay.scid);      // [nl] centroid ids
  int32_t *dcount = (int32_t *)(walk_lds + lay.dcount);  // [nprobe] dense groups per rank
  int32_t *bcnt = (int32_t *)(walk_lds + lay.bcnt);      // [nprobe] bucket entries per rank
  int32_t *bbase = (int32_t *)(walk_lds + lay.bbase);    // [nprobe] first bucket entry of each rank
  // the dense groups of rank r: k < dcount[r] at r * Tq + k
  MaskT *dgm = (MaskT *)(walk_lds + lay.dgm);            // [nl] token masks
  int32_t *dgs = (int32_t *)(walk_lds + lay.dgs);        // [nl] score sums
  int8_t *dls = (int8_t *)(walk_lds + lay.dls);          // [nl] dense slots
  int32_t *nlong = (int32_t *)(walk_lds + lay.nlong);    // [3] wave-owned lists, dense groups, entries of the range
  int32_t *dtab = (int32_t *)(walk_lds + lay.dtab);      // [2^g] F' of the dense groups alone, by their hits, on scid .. dls
  uint16_t *dtok = (uint16_t *)(walk_lds + lay.dtok);    // [Tq] the dense groups that hold a token
  int2 *dgrp = (int2 *)(walk_lds + lay.dgrp);            // [g] dense groups by rank: list index r * Tq + j, slot
  // workgroup b runs on XCD b % 8: with 8 or more queries, the groups of
  // query q run on XCD q % 8; fewer queries spread over every XCD
  const int b = blockIdx.x;
  const int64_t q = nq >= 8 ? (b & 7) + 8 * (int64_t)((b >> 3) / G) : b / G;
  const int g = nq >= 8 ? (b >> 3) % G : b % G;
  if (q >= nq) return;
  const int rg0 = g * M, rg1 = min(nranges, rg0 + M);
  if (rg0 >= rg1) return;  // uniform, before any barrier
  const int64_t dstart = (int64_t)rg0 * R;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int t = threadIdx.x; t < nl; t += WALK_THREADS) {
    const int r = t / Tq, j = t - r * Tq;
    const int64_t e = (q * TQP + j) * nprobe + r;
    scid[t] = cent_ids[e];
    skey[t] = cent_keys[e];
  }
  for (int r = threadIdx.x; r < nprobe; r += WALK_THREADS) dcount[r] = 0;
  if (threadIdx.x < 3) nlong[threadIdx.x] = 0;
  __syncthreads();
  // classify list t = threadIdx.x + WALK_THREADS * i: group head or not,
  // dense, long or short; a short list stays with this thread (slot i)
  ShortList<WIN> S[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int t = threadIdx.x + WALK_THREADS * i;
    S[i].rank = -1;
    S[i].avail = 0;
    S[i].lp = ivf_doc;  // a readable entry for slots without a list
    S[i].len = 1;
    S[i].pos0 = 0;
    S[i].c = 0;
    if (t >= nl) continue;
    const int r = t / Tq, j = t - r * Tq;
    const int32_t c = scid[t];
    // one pass over the rank's centroids: is j the group's first token, and
    // the group's mask and score sum
    bool head = (uint32_t)c < (uint32_t)ncent;
    MaskT gm = 0;
    int32_t gs = 0;
    for (int u = 0; u < Tq; ++u) {
      const bool same = scid[r * Tq + u] == c;
      head = head && !(same && u < j);
      gm |= same ? (MaskT)1 << u : (MaskT)0;
      gs += same ? skey[r * Tq + u] : 0;
    }
    lmask[t] = gm;
    lsum[t] = gs;
    if (!head) continue;
    if (ndense > 0 && dense_slot[c] >= 0) {
      // a dense list: applied from the documents' masks, never walked
      const int k = atomicAdd(&dcount[r], 1);
      dls[r * Tq + k] = dense_slot[c];
      dgm[r * Tq + k] = gm;
      dgs[r * Tq + k] = gs;
      if (TAB) {
        const int d = atomicAdd(&nlong[1], 1);
        if (d < WALK_TAB_BITS) ((int2 *)bucket)[d] = make_int2(t, dense_slot[c]);
      }
      continue;
    }
    const int64_t beg = ivf_off[c], end = ivf_off[c + 1];
    const int64_t p = dstart > 0 ? lower_bound_i32(ivf_doc, beg, end, dstart) : beg;
    const int32_t len = (int32_t)(end - beg), pos = (int32_t)(p - beg);
    if (pos >= len) continue;  // nothing left in the group's documents
    if ((int64_t)(len - pos) * R > (int64_t)WALK_LONG * (ndocs - dstart)) {
      const int k = atomicAdd(nlong, 1);
      if (k < WALK_MAX_LONG) {
        LongList w;
        w.beg = beg;
        w.pos = pos;
        w.len = len;
        w.t = t;
        w.rank = r;
        LL[k] = w;
        continue;
      }
    }
    S[i].lp = ivf_doc + beg;
    S[i].len = len;
    S[i].pos0 = pos;
    S[i].c = 0;
    S[i].rank = r;
    S[i].t = t;
    S[i].avail = min(WIN, len - pos);
    load_window(S[i].lp, pos, len, S[i].e);
  }
  __syncthreads();
  // the dense groups in rank order, the groups of each token, and the table:
  // entry x is the sum of the best keys of the tokens that the groups of x hold
  const int ng = TAB ? nlong[1] : 0;
  bool tab = TAB && ng <= WALK_TAB_BITS;  // uniform
  if (tab) {
    if ((int)threadIdx.x < ng) {
      const int2 me = ((const int2 *)bucket)[threadIdx.x];
      int at = 0;
      for (int k = 0; k < ng; ++k) {
        const int t = ((const int2 *)bucket)[k].x;
        at += t < me.x ? 1 : 0;
      }
      dgrp[at] = me;
    }
    __syncthreads();
    if ((int)threadIdx.x < Tq) {
      int m = 0;
      for (int k = 0; k < ng; ++k) m |= (int)((lmask[dgrp[k].x] >> threadIdx.x) & 1) << k;
      dtok[threadIdx.x] = (uint16_t)m;
    }
    for (int x = threadIdx.x; x < (1 << ng); x += WALK_THREADS) {
      MaskT seen = 0;
      int32_t f = 0;
      for (int k = 0; k < ng; ++k) {
        if (!((x >> k) & 1)) continue;
        const int t = dgrp[k].x;
        const MaskT gm = lmask[t], fresh = gm & ~seen;
        seen |= gm;
        if (fresh == gm) {
          f += lsum[t];
        } else {
          const int32_t *keys = skey + (t - __builtin_ctzll((unsigned long long)gm));
          for (MaskT m = fresh; m; m &= m - 1) f += keys[__builtin_ctzll((unsigned long long)m)];
        }
      }
      dtab[x] = f;
    }
    // the histogram of the group's ranges, and the documents' chains
    for (int i = threadIdx.x; i < SEL_BINS; i += WALK_THREADS) ((uint32_t *)smask)[i] = 0;
    for (int v = threadIdx.x; v < R; v += WALK_THREADS) sfp[v] = 0;
    __syncthreads();
  }
  // lane k: the dense group k's slot
  const int slots = tab && lane < ng ? dgrp[lane].y : 0;
  // the wave's lists and their windows: slot i is list wave + WALK_WAVES * i
  const int nlw = min(*nlong, WALK_MAX_LONG);
  // (lane l holds entry pos + l, loaded as is: lanes past the list's end hold
  // its last entry and are masked where the window is read)
  int32_t lw[WALK_LONG_SLOTS];
#pragma unroll
  for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
    const int k = wave + WALK_WAVES * i;
    if (k < nlw) {
      const LongList w = LL[k];
      lw[i] = ivf_doc[w.beg + min(w.pos + lane, w.len - 1)];
    }
  }
  // dense-list masks of the documents this thread owns (tid + WALK_THREADS * i),
  // loaded at the end of the previous range
  uint64_t dm[DPT];
#pragma unroll
  for (int i = 0; i < DPT; ++i) {
    const int64_t v = dstart + threadIdx.x + WALK_THREADS * i;
    dm[i] = ndense > 0 && v < ndocs ? doc_dense[v] : 0;
  }
  for (int rg = rg0; rg < rg1; ++rg) {
    const int64_t d0 = (int64_t)rg * R;
    const int64_t d1 = min(ndocs, d0 + R);
    const int nd = (int)(d1 - d0);
    if (tab) {  // uniform
      // ---- the range through chains of entries and the dense groups' table
      uint32_t *hsh = (uint32_t *)smask;    // [SEL_BINS] the histogram of the group's ranges so far
      uint32_t *chain = (uint32_t *)sfp;    // [R] 1 + a document's last entry, 0: none
      int32_t *nent = nlong + 2;
      // every list's entries in the range: list index << 16 | 1 + the document's entry before
      auto link = [&](int node, int t, int v) {
        if (node < WALK_NODES) bucket[node] = (uint32_t)t << 16 | atomicExch(&chain[v], (uint32_t)node + 1);
      };
      int snew[LPT];
      int32_t spos[LPT];
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        int mt = 0;
#pragma unroll
        for (int u = 0; u < WIN; ++u) mt += (u < S[i].avail && S[i].e[u] < d1) ? 1 : 0;
        snew[i] = mt;
        spos[i] = S[i].pos0 + mt;
        const uint32_t incl = wave_incl_scan((uint32_t)mt);
        const int all = __builtin_amdgcn_readlane((int)incl, 63);
        if (all == 0) continue;  // wave-uniform
        int base = 0;
        if (lane == 0) base = atomicAdd(nent, all);
        base = __builtin_amdgcn_readfirstlane(base) + (int)incl - mt;
        // (the exchanges are issued together, their results used afterwards)
        uint32_t before[WIN];
#pragma unroll
        for (int u = 0; u < WIN; ++u) {
          before[u] = 0;
          if (u < mt && base + u < WALK_NODES)
            before[u] = atomicExch(&chain[(int)(S[i].e[u] - d0)], (uint32_t)(base + u) + 1);
        }
#pragma unroll
        for (int u = 0; u < WIN; ++u)
          if (u < mt && base + u < WALK_NODES) bucket[base + u] = (uint32_t)S[i].t << 16 | before[u];
        // a list with more entries in the range than its window goes on through memory
        if (mt == S[i].avail && mt > 0) {
          while (spos[i] < S[i].len) {
            const int32_t dd = S[i].lp[spos[i]];
            if (dd >= d1) break;
            link(atomicAdd(nent, 1), S[i].t, (int)(dd - d0));
            ++spos[i];
          }
        }
      }
      int lnew[WALK_LONG_SLOTS];  // wave-uniform
#pragma unroll
      for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
        lnew[i] = 0;
        const int k = wave + WALK_WAVES * i;
        if (k >= nlw) continue;  // wave-uniform
        const LongList w = LL[k];
        int32_t doc = w.pos + lane < w.len ? lw[i] : INT32_MAX;
        for (;;) {
          const bool in = doc < d1;
          const unsigned long long ins = __ballot(in);  // a prefix of the lanes: the list ascends
          const int n = __popcll(ins);
          if (n > 0) {
            int base = 0;
            if (lane == 0) base = atomicAdd(nent, n);
            base = __builtin_amdgcn_readfirstlane(base);
            if (in) link(base + lane, w.t, (int)(doc - d0));
          }
          lnew[i] += n;
          if (n < 64) break;
          const int32_t p = w.pos + lnew[i] + lane;
          doc = p < w.len ? ivf_doc[w.beg + p] : INT32_MAX;
        }
      }
      __syncthreads();  // the chains are complete
      if (*nent <= WALK_NODES) {  // uniform
        // each wave takes the documents its threads own, four of a thread at a
        // time: without entries F' is the table's; the others are listed and
        // taken one a lane
        uint32_t *hl = bucket + WALK_NODES + wave * WALK_HITS;
        constexpr int HALF = DPT < 4 ? DPT : 4;
        static_assert(HALF * 64 <= WALK_HITS, "a wave lists every document of a step");
#pragma unroll
        for (int i0 = 0; i0 < DPT; i0 += HALF) {
          int32_t x[HALF];
          bool hit[HALF];
          int nh = 0;  // wave-uniform
          uint32_t bits[HALF];
#pragma unroll
          for (int i = 0; i < HALF; ++i) bits[i] = 0;
          for (int k = 0; k < ng; ++k) {
            const int sl = __builtin_amdgcn_readlane(slots, k);
#pragma unroll
            for (int i = 0; i < HALF; ++i) {
              const uint32_t w = sl < 32 ? (uint32_t)dm[i0 + i] : (uint32_t)(dm[i0 + i] >> 32);
              bits[i] |= ((w >> (sl & 31)) & 1u) << k;
            }
          }
#pragma unroll
          for (int i = 0; i < HALF; ++i) {
            const int v = threadIdx.x + WALK_THREADS * (i0 + i);
            const int idx = (int)bits[i];
            hit[i] = chain[v] != 0;
            x[i] = idx ? dtab[idx] : NO_HIT;
            const unsigned long long hs = __ballot(hit[i]);
            if (hit[i]) hl[nh + __popcll(hs & ((1ull << lane) - 1))] = (uint32_t)v << 16 | (uint32_t)idx;
            nh += __popcll(hs);
          }
          for (int b0 = 0; b0 < nh; b0 += 64) {
            const bool on = b0 + lane < nh;
            const uint32_t h = on ? hl[b0 + lane] : 0;
            const int v = (int)(h >> 16), idx = (int)(h & 0xFFFFu);
            // the document's entries in rank order (list indexes ascend with the rank)
            uint32_t a[4] = {0xFFFFu, 0xFFFFu, 0xFFFFu, 0xFFFFu};
            uint32_t e = on ? chain[v] : 0;
            int n = 0;
            while (e && n <= 4) {
              const uint32_t y = bucket[e - 1];
              uint32_t t = y >> 16;
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const uint32_t lo = min(a[u], t);
                t = max(a[u], t);
                a[u] = lo;
              }
              e = y & 0xFFFFu;
              ++n;
            }
            if (on && n <= 4) {
              // the tokens of an entry's group that no better entry has credited
              // take its key where no dense group of a better rank holds them,
              // in place of a worse one's
              int32_t f = dtab[idx];
              MaskT seen = 0;
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                if (a[u] == 0xFFFFu) continue;
                const MaskT gm = lmask[a[u]];
                const int rb = (int)a[u] - __builtin_ctzll((unsigned long long)gm);  // r * Tq: the head is the first token
                for (MaskT m = gm & ~seen; m; m &= m - 1) {
                  const int j = __builtin_ctzll((unsigned long long)m);
                  const int dk = idx & dtok[j];
                  if (dk) {
                    const int td = dgrp[__builtin_ctz(dk)].x;
                    const int db = td - __builtin_ctzll((unsigned long long)lmask[td]);
                    if (db > rb) f += skey[rb + j] - skey[db + j];
                  } else {
                    f += skey[rb + j];
                  }
                }
                seen |= gm;
              }
              chain[v] = (uint32_t)f;
            }
            // a document with more entries: the wave takes it, a token a lane,
            // each the largest of its keys
            for (unsigned long long big = __ballot(on && n > 4); big; big &= big - 1) {
              const int l = __builtin_ctzll(big);
              const int bv = __builtin_amdgcn_readlane(v, l), bidx = __builtin_amdgcn_readlane(idx, l);
              int32_t best = INT_MIN;
              auto take = [&](int t) {
                const MaskT gm = lmask[t];
                if (lane < Tq && ((gm >> lane) & 1)) best = max(best, skey[t - __builtin_ctzll((unsigned long long)gm) + lane]);
              };
              uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)chain[bv]);
              while (c) {
                const uint32_t y = (uint32_t)__builtin_amdgcn_readfirstlane((int)bucket[c - 1]);
                take((int)(y >> 16));
                c = y & 0xFFFFu;
              }
              for (int k = 0; k < ng; ++k)
                if ((bidx >> k) & 1) take(dgrp[k].x);
              const uint32_t sum = wave_incl_scan(best == INT_MIN ? 0u : (uint32_t)best);
              if (lane == 63) chain[bv] = sum;
            }
          }
          int32_t *f = fp + q * ndocs + d0;
#pragma unroll
          for (int i = 0; i < HALF; ++i) {
            const int v = threadIdx.x + WALK_THREADS * (i0 + i);
            if (hit[i]) {
              x[i] = (int32_t)chain[v];
              chain[v] = 0;
            }
            if (v < nd) {
              if (deleted && ((deleted[(d0 + v) >> 6] >> ((d0 + v) & 63)) & 1)) x[i] = NO_HIT;
              f[v] = x[i];
              if (x[i] != NO_HIT) atomicAdd(&hsh[fp_key(x[i]) >> 20], 1u);
            }
          }
        }
        // the next range's inputs
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
          S[i].pos0 = spos[i];
          S[i].avail = S[i].rank < 0 ? 0 : min(WIN, S[i].len - S[i].pos0);
          load_window(S[i].lp, S[i].pos0, S[i].len, S[i].e);
        }
#pragma unroll
        for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
          const int k = wave + WALK_WAVES * i;
          if (k < nlw) {  // wave-uniform
            const LongList w = LL[k];
            const int32_t pos = w.pos + lnew[i];
            lw[i] = ivf_doc[w.beg + min(pos + lane, w.len - 1)];
            if (lane == 0) LL[k].pos = pos;
          }
        }
        if (rg + 1 < rg1) {
#pragma unroll
          for (int i = 0; i < DPT; ++i) {
            const int64_t v = d1 + threadIdx.x + WALK_THREADS * i;
            dm[i] = ndense > 0 && v < ndocs ? doc_dense[v] : 0;
          }
        }
        __syncthreads();  // the range has been read
        if (threadIdx.x == 0) *nent = 0;
        __syncthreads();
        continue;
      }
      // more entries than the chains hold: the histogram so far goes out, and
      // the range (and the group's others) are walked rank by rank, with the
      // dense groups' arrays back in the table's place
      uint32_t *hq = hist + q * SEL_BINS;
      for (int i = threadIdx.x; i < SEL_BINS; i += WALK_THREADS)
        if (hsh[i]) atomicAdd(&hq[i], hsh[i]);
      if ((int)threadIdx.x < ng) {
        const int2 me = dgrp[threadIdx.x];
        const int r = me.x / Tq;
        int k = 0;
        for (int b = 0; b < (int)threadIdx.x; ++b) k += dgrp[b].x / Tq == r ? 1 : 0;
        dls[r * Tq + k] = (int8_t)me.y;
        dgm[r * Tq + k] = lmask[me.x];
        dgs[r * Tq + k] = lsum[me.x];
      }
      tab = false;
      __syncthreads();
    }
    for (int v = threadIdx.x; v < R; v += WALK_THREADS) {
      smask[v] = 0;
      sfp[v] = 0;
    }
    for (int r = threadIdx.x; r < nprobe; r += WALK_THREADS) bcnt[r] = 0;
    __syncthreads();  // the range is cleared; the previous range's reads are done

    // the windows' entries inside the range: count them per rank and reserve
    // their places in the rank's bucket
    int snew[LPT], soff[LPT];
    bool sovf[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      snew[i] = 0;
      soff[i] = 0;
      sovf[i] = false;
      if (S[i].avail == 0) continue;
      int mt = 0;
#pragma unroll
      for (int u = 0; u < WIN; ++u) mt += (u < S[i].avail && S[i].e[u] < d1) ? 1 : 0;
      snew[i] = mt - S[i].c;
      sovf[i] = mt == S[i].avail && S[i].pos0 + S[i].avail < S[i].len;
      if (snew[i] > 0) soff[i] = atomicAdd(&bcnt[S[i].rank], snew[i]);
    }
#pragma unroll
    for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
      const int k = wave + WALK_WAVES * i;
      if (k >= nlw) continue;  // wave-uniform
      const LongList w = LL[k];
      const int n = __popcll(__ballot(w.pos + lane < w.len && lw[i] < d1));
      if (lane == 0) {
        LL[k].n = n;
        if (n > 0) LL[k].off = atomicAdd(&bcnt[LL[k].rank], n);
      }
    }
    __syncthreads();
    if (wave == 0) {  // bucket base of each rank: exclusive prefix sum (nprobe <= 64)
      const int x = lane < nprobe ? bcnt[lane] : 0;
      int incl = x;
#pragma unroll
      for (int dd = 1; dd < 64; dd <<= 1) {
        const int y = __shfl_up(incl, dd, 64);
        if (lane >= dd) incl += y;
      }
      if (lane < nprobe) bbase[lane] = incl - x;
    }
    __syncthreads();
    // copy the entries into the buckets, then move every window forward;
    // the refills are needed a range later
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      if (S[i].avail == 0) continue;
      if (snew[i] > 0) {
        uint32_t *bk = bucket + bbase[S[i].rank] + soff[i] - S[i].c;
#pragma unroll
        for (int u = 0; u < WIN; ++u)
          if (u >= S[i].c && u < S[i].c + snew[i])
            bk[u] = (uint32_t)S[i].t << WALK_DOC_BITS | (uint32_t)(S[i].e[u] - d0);
      }
      S[i].c += snew[i];
    }
#pragma unroll
    for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
      const int k = wave + WALK_WAVES * i;
      if (k >= nlw) continue;  // wave-uniform
      const LongList w = LL[k];
      const int n = w.n;
      if (n == 0) continue;
      if (lane < n) bucket[bbase[w.rank] + w.off + lane] = (uint32_t)w.t << WALK_DOC_BITS | (uint32_t)(lw[i] - d0);
      if (n < 64 && lane == 0) LL[k].pos = w.pos + n;  // a full window goes on through memory at its rank
    }
    __syncthreads();  // the buckets are complete

    for (int r = 0; r < nprobe; ++r) {
      const int ndg = dcount[r];
      const int32_t *keys = skey + r * Tq;
      // the rank's bucket, spread over every thread
      const int e1 = bbase[r] + bcnt[r];
      for (int e = bbase[r] + threadIdx.x; e < e1; e += WALK_THREADS) {
        const uint32_t x = bucket[e];
        const int t = (int)(x >> WALK_DOC_BITS);
        credit(smask, sfp, (int)(x & ((1u << WALK_DOC_BITS) - 1)), lmask[t], lsum[t], keys);
      }
      // lists with more entries in the range than their window held
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        if (!sovf[i] || S[i].rank != r) continue;
        int32_t p = S[i].pos0 + S[i].avail;
        const MaskT gm = lmask[S[i].t];
        const int32_t gs = lsum[S[i].t];
        while (p < S[i].len) {
          const int32_t d = S[i].lp[p];
          if (d >= d1) break;
          credit(smask, sfp, (int)(d - d0), gm, gs, keys);
          ++p;
        }
        S[i].pos0 = p;
        S[i].c = 0;
      }
#pragma unroll
      for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
        const int k = wave + WALK_WAVES * i;
        if (k >= nlw) continue;  // wave-uniform
        const LongList w = LL[k];
        if (w.rank != r || w.n != 64) continue;
        int32_t pos = w.pos + 64;
        walk_list<8>(ivf_doc + w.beg, w.len, d0, d1, lmask[w.t], lsum[w.t], keys, lane, smask, sfp, pos);
        if (lane == 0) LL[k].pos = pos;
      }
      if (ndg > 0) {  // uniform
        // dense lists of rank r: each thread applies them to the documents it
        // owns from their masks.  The groups of one rank hold disjoint
        // tokens, so a document's hits add up to one token mask and one
        // score sum; the groups are visited in the same order by every lane.
        // They are credited with the same atomics as the rank's other lists,
        // whose tokens they do not share, so the two need no barrier between
        // them: only the earlier ranks must be complete.
        MaskT nb[DPT];
        int32_t sall[DPT];
#pragma unroll
        for (int i = 0; i < DPT; ++i) {
          nb[i] = 0;
          sall[i] = 0;
        }
        for (int k = 0; k < ndg; ++k) {
          const int sl = dls[r * Tq + k];
          const MaskT gm = dgm[r * Tq + k];
          const int32_t gs = dgs[r * Tq + k];
#pragma unroll
          for (int i = 0; i < DPT; ++i) {
            const bool hit = (dm[i] >> sl) & 1;
            nb[i] |= hit ? gm : (MaskT)0;
            sall[i] += hit ? gs : 0;
          }
        }
#pragma unroll
        for (int i = 0; i < DPT; ++i)
          if (nb[i]) credit(smask, sfp, threadIdx.x + WALK_THREADS * i, nb[i], sall[i], keys);
      }
      __syncthreads();  // rank r's LDS updates complete before rank r+1's
    }
    // the next range's inputs, loaded now and first read a range from now:
    // every window at its list's new position (its lines are cached), and
    // the dense masks
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      S[i].pos0 += S[i].c;
      S[i].c = 0;
      S[i].avail = S[i].rank < 0 ? 0 : min(WIN, S[i].len - S[i].pos0);
      load_window(S[i].lp, S[i].pos0, S[i].len, S[i].e);
    }
#pragma unroll
    for (int i = 0; i < WALK_LONG_SLOTS; ++i) {
      const int k = wave + WALK_WAVES * i;
      if (k < nlw) {  // wave-uniform
        const LongList w = LL[k];
        lw[i] = ivf_doc[w.beg + min(w.pos + lane, w.len - 1)];
      }
    }
    if (rg + 1 < rg1) {
#pragma unroll
      for (int i = 0; i < DPT; ++i) {
        const int64_t v = d1 + threadIdx.x + WALK_THREADS * i;
        dm[i] = ndense > 0 && v < ndocs ? doc_dense[v] : 0;
      }
    }
    // documents outside S_Q, and deleted ones, get NO_HIT
    for (int v = threadIdx.x; v < nd; v += WALK_THREADS)
      if (smask[v] == 0 || (deleted && ((deleted[(d0 + v) >> 6] >> ((d0 + v) & 63)) & 1))) sfp[v] = NO_HIT;
    __syncthreads();
    uint32_t *sh = (uint32_t *)smask;  // the masks are no longer needed
    for (int i = threadIdx.x; i < SEL_BINS; i += WALK_THREADS) sh[i] = 0;
    __syncthreads();
    int32_t *f = fp + q * ndocs + d0;
    for (int v = threadIdx.x; v < nd; v += WALK_THREADS) {
      const int32_t x = sfp[v];
      f[v] = x;
      if (x != NO_HIT) atomicAdd(&sh[fp_key(x) >> 20], 1u);
    }
    __syncthreads();
    uint32_t *hq = hist + q * SEL_BINS;
    for (int i = threadIdx.x; i < SEL_BINS; i += WALK_THREADS)
      if (sh[i]) atomicAdd(&hq[i], sh[i]);
    __syncthreads();  // sh (the mask array) is cleared by the next range
  }
  if (tab) {
    uint32_t *hq = hist + q * SEL_BINS;
    const uint32_t *hsh = (const uint32_t *)smask;
    for (int i = threadIdx.x; i < SEL_BINS; i += WALK_THREADS)
      if (hsh[i]) atomicAdd(&hq[i], hsh[i]);
  }
}

size_t walk_lds_bytes(int TQP, int nprobe, int Tq) {
  if ((size_t)nprobe * Tq > (size_t)WALK_MAX_LISTS) return SIZE_MAX;
  // either walk may run (k_walk_lists.hip takes indexes without dense lists)
  return std::max(walk_lds_layout(walk_range_docs(TQP, nprobe, Tq), TQP == 32 ? 4 : 8, nprobe, Tq, false).total,
                  list_walk_lds_bytes(TQP, nprobe, Tq));
}

// Whether the walk through chains and a table pays, for workgroups of M ranges
// and lists of nnz entries in all.  It saves a barrier and more per rank and range, but its table is
// built once per workgroup, and costs more the more dense groups a query has:
// at 1M documents and one range a workgroup (128 queries) it takes 0.86, 0.97
// and 1.11 of the time rank by rank at 8 ranks with 4, 16 and 32 query tokens,
// 0.74, 0.84 and 0.93 at 16; with eight ranges (1024 queries) 0.71, 0.76 and
// 0.99 at 8 ranks, 0.80, 0.87 and 1.03 at 4.  Queries of more than
// WALK_TAB_BITS dense groups gain nothing: with 64 tokens most have them (1.00
// to 1.07 at every rank count on 1M and 2.2M documents), and with few centroids
// the lower ranks add groups to the tokens' own, about (nprobe - 1) Tq ndense /
// ncent.  Nor do ranges with more entries than the chains hold; the lower ranks'
// lists bring about 4096 (nprobe - 1) Tq nnz / (ndocs ncent).  (100,000
// documents, 16,384 centroids, 32 tokens: 1.01 at 16 ranks, 1.05 at 32; 1M,
// 65,536 centroids, 64 ranks: 1.13, where 32 ranks take 0.82; 313,900 and 15,644,
// 26 tokens, 22 ranks: 1.17; but 4,676 and 4,904, 13 tokens, 12 ranks: 0.44.)
bool walk_by_chains(int Tq, int TQP, int nprobe, int64_t ndocs, int64_t nnz, int ncent, int ndense, int M) {
  const double lower = (double)(nprobe - 1) * Tq / ncent;
  if (TQP != 32 || lower * ndense > 2 || 4096 * lower * (double)nnz > (double)WALK_NODES * (double)ndocs) return false;
  if (Tq > 16) return nprobe >= 16 || (nprobe >= 8 && M >= 3);
  return M * nprobe >= (Tq > 8 ? 12 : 8);
}

template <typename MaskT, int R, int LPT, bool TAB>
static void launch_walk_t(const int32_t *cent_ids, const int32_t *cent_keys, int64_t nq, int Tq, int TQP, int nprobe,
                          const int64_t *ivf_off, const int32_t *ivf_doc, int64_t ndocs, int ncent, int ndense,
                          const int8_t *dense_slot, const uint64_t *doc_dense, const uint64_t *deleted, int nranges,
                          int G, int M, int32_t *fp, uint32_t *hist, hipStream_t s) {
  const int64_t blocks = (nq >= 8 ? (nq + 7) / 8 * 8 : nq) * G;
  if (blocks == 0 || nranges == 0) return;
  const size_t lds = walk_lds_layout(R, (int)sizeof(MaskT), nprobe, Tq, TAB).total;
  static bool attr = [] {
    return hipFuncSetAttribute((const void *)k_cand_walk<MaskT, R, LPT, TAB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               160 * 1024) == hipSuccess;
  }();
  (void)attr;
  hipLaunchKernelGGL((k_cand_walk<MaskT, R, LPT, TAB>), dim3((unsigned)blocks), dim3(WALK_THREADS), lds, s, cent_ids,
                     cent_keys, nq, Tq, TQP, nprobe, ivf_off, ivf_doc, ndocs, ncent, ndense, dense_slot, doc_dense,
                     deleted, nranges, G, M, fp, hist);
}

template <typename MaskT, int R, bool TAB>
static void launch_walk_r(const int32_t *cent_ids, const int32_t *cent_keys, int64_t nq, int Tq, int TQP, int nprobe,
                          const int64_t *ivf_off, const int32_t *ivf_doc, int64_t ndocs, int ncent, int ndense,
                          const int8_t *dense_slot, const uint64_t *doc_dense, const uint64_t *deleted, int nranges,
                          int G, int M, int32_t *fp, uint32_t *hist, hipStream_t s) {
  const int lpt = (nprobe * Tq + WALK_THREADS - 1) / WALK_THREADS;  // at most 4 (walk_lds_bytes)
  auto *launch = lpt <= 1   ? launch_walk_t<MaskT, R, 1, TAB>
                 : lpt <= 2 ? launch_walk_t<MaskT, R, 2, TAB>
                            : launch_walk_t<MaskT, R, 4, TAB>;
  launch(cent_ids, cent_keys, nq, Tq, TQP, nprobe, ivf_off, ivf_doc, ndocs, ncent, ndense, dense_slot, doc_dense,
         deleted, nranges, G, M, fp, hist, s);
}

void launch_cand_walk(const int32_t *cent_ids, const int32_t *cent_keys, int64_t nq, int Tq, int TQP, int nprobe,
                      const int64_t *ivf_off, const int32_t *ivf_doc, int64_t ndocs, int64_t nnz, int ncent, int ndense,
                      const int8_t *dense_slot, const uint64_t *doc_dense, const uint64_t *deleted, int32_t *fp, uint32_t *hist,
                      hipStream_t s) {
  if (nq <= 0) return;
  // without dense lists the centroids are used about evenly: each probed list
  // is walked from memory at its rank (k_walk_lists.hip); measured 2x faster
  // there than the bucketed walk, which wins on skewed (Zipf) lists
  if (ndense == 0) {
    launch_list_walk(cent_ids, cent_keys, nq, Tq, TQP, nprobe, ivf_off, ivf_doc, ndocs, ncent, deleted, fp, hist, s);
    return;
  }
  const int R = walk_range_docs(TQP, nprobe, Tq);
  const int nranges = (int)((ndocs + R - 1) / R);
  // ranges per workgroup: enough groups per query for about 32768 workgroups
  // (measured at 8.8M and 1M: shorter workgroups leave fewer CUs idle at a
  // launch's end than fewer, longer ones; 8.8M walk 403 -> 383 ms, 1M 12.1
  // -> 10.0 ms, against about 4096)
  int G = (int)std::min<int64_t>(nranges, std::max<int64_t>(1, (32768 + nq - 1) / nq));
  const int M = (nranges + G - 1) / std::max(1, G);
  G = (nranges + M - 1) / std::max(1, M);
  auto *launch = TQP != 32 ? launch_walk_r<unsigned long long, 2048, false>
                 : walk_by_chains(Tq, TQP, nprobe, ndocs, nnz, ncent, ndense, M)
                     ? launch_walk_r<uint32_t, 4096, true>
                     : launch_walk_r<uint32_t, 4096, false>;
  launch(cent_ids, cent_keys, nq, Tq, TQP, nprobe, ivf_off, ivf_doc, ndocs, ncent, ndense, dense_slot, doc_dense,
         deleted, nranges, G, M, fp, hist, s);
}

// ------------------------------------------------------- block helpers
constexpr int SEL_THREADS = 1024;
constexpr int SEL_ITEMS = 4;
constexpr int SEL_UNROLL = 8;       // independent F' loads per thread in a histogram pass
constexpr int SEL_COMPACT_ITEMS = 16;  // consecutive documents per thread in k_select's compaction

// Exclusive prefix sum over the block; thread 0 leaves the block total in
// *total (shared), readable by every thread once the call returns.
__device__ __forceinline__ long long block_exclusive_scan(long long x, long long *wsum, long long *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  long long incl = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const long long y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long acc = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      const long long t = wsum[w];
      wsum[w] = acc;
      acc += t;
    }
    *total = acc;
  }
  __syncthreads();
  const long long res = wsum[wave] + incl - x;
  __syncthreads();  // wsum is reused by the next call
  return res;
}

// Radix-select step: over bins[0..nbins) taken from the highest bin down,
// find the bin b where the running count reaches rem.  Leaves b in *s_bin
// and the count of the bins above b in *s_above.
__device__ __forceinline__ void select_bin(const uint32_t *bins, int nbins, long long rem, long long *wsum,
                                           long long *s_tot, int *s_bin, long long *s_above) {
  const int per = (nbins + (int)blockDim.x - 1) / (int)blockDim.x;
  const int top = nbins - 1 - (int)threadIdx.x * per;  // this thread's bins: top, top-1, ... (descending)
  long long local = 0;
  for (int i = 0; i < per; ++i)
    if (top - i >= 0) local += bins[top - i];
  const long long excl = block_exclusive_scan(local, wsum, s_tot);
  if (excl < rem && excl + local >= rem) {
    long long cum = excl;
    for (int i = 0; i < per; ++i) {
      const int bb = top - i;
      if (bb < 0) break;
      if (cum + bins[bb] >= rem) {
        *s_bin = bb;
        *s_above = cum;
        break;
      }
      cum += bins[bb];
    }
  }
  __syncthreads();
}

// Per-query selection of the ncand best hits by (F' desc, doc asc), written
// in ascending doc order.  The first radix pass (top 12 key bits) comes from
// the walk's histogram; two more passes over F' (12 and 8 bits) give the
// exact threshold key T and how many documents with key T to keep (the
// lowest ids first).  MODE 1 lists every hit at offsets[q] (the candidate-set
// tap).
template <int MODE>
__global__ __launch_bounds__(SEL_THREADS) void k_select(const int32_t *__restrict__ fp,
                                                        const uint32_t *__restrict__ hist1, int64_t ndocs, int ncand,
                                                        const int64_t *__restrict__ offsets,
                                                        int32_t *__restrict__ out_ids, int32_t *__restrict__ out_keys,
                                                        int32_t *__restrict__ n_valid) {
  __shared__ uint32_t hist[SEL_BINS];
  __shared__ long long wsum[SEL_THREADS / 64];
  __shared__ long long s_tot, s_above;
  __shared__ int s_bin;
  const int64_t q = blockIdx.x;
  const int32_t *f = fp + q * ndocs;

  uint32_t T = 0;
  long long need = 0;  // hits with key == T still to take
  bool take_all = true;
  if (MODE == 0) {
    long long local = 0;
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) {
      hist[i] = hist1[q * SEL_BINS + i];
      local += hist[i];
    }
    block_exclusive_scan(local, wsum, &s_tot);
    const long long nhit = s_tot;
    take_all = nhit <= ncand;
    if (!take_all) {
      long long rem = ncand;
      // pass 1 (histogram from the walk): key bits 31..20
      select_bin(hist, SEL_BINS, rem, wsum, &s_tot, &s_bin, &s_above);
      const uint32_t b1 = (uint32_t)s_bin;
      rem -= s_above;
      // pass 2: key bits 19..8 among keys with top bits b1
      for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) hist[i] = 0;
      __syncthreads();
      for (int64_t v0 = threadIdx.x; v0 < ndocs; v0 += SEL_THREADS * SEL_UNROLL) {
        int32_t x[SEL_UNROLL];
#pragma unroll
        for (int i = 0; i < SEL_UNROLL; ++i) {
          const int64_t v = v0 + (int64_t)i * SEL_THREADS;
          x[i] = v < ndocs ? f[v] : NO_HIT;
        }
#pragma unroll
        for (int i = 0; i < SEL_UNROLL; ++i) {
          const uint32_t u = fp_key(x[i]);
          if (x[i] != NO_HIT && (u >> 20) == b1) atomicAdd(&hist[(u >> 8) & 4095u], 1u);
        }
      }
      __syncthreads();
      select_bin(hist, SEL_BINS, rem, wsum, &s_tot, &s_bin, &s_above);
      const uint32_t p2 = (b1 << 12) | (uint32_t)s_bin;
      rem -= s_above;
      // pass 3: key bits 7..0 among keys with top bits p2
      for (int i = threadIdx.x; i < 256; i += SEL_THREADS) hist[i] = 0;
      __syncthreads();
      for (int64_t v0 = threadIdx.x; v0 < ndocs; v0 += SEL_THREADS * SEL_UNROLL) {
        int32_t x[SEL_UNROLL];
#pragma unroll
        for (int i = 0; i < SEL_UNROLL; ++i) {
          const int64_t v = v0 + (int64_t)i * SEL_THREADS;
          x[i] = v < ndocs ? f[v] : NO_HIT;
        }
#pragma unroll
        for (int i = 0; i < SEL_UNROLL; ++i) {
          const uint32_t u = fp_key(x[i]);
          if (x[i] != NO_HIT && (u >> 8) == p2) atomicAdd(&hist[u & 255u], 1u);
        }
      }
      __syncthreads();
      select_bin(hist, 256, rem, wsum, &s_tot, &s_bin, &s_above);
      T = (p2 << 8) | (uint32_t)s_bin;
      need = rem - s_above;
    }
  }

  // --- ordered compaction
  const int64_t base_out = MODE == 1 ? offsets[q] : q * (int64_t)ncand;
  long long written = 0, ties_seen = 0;
  const int64_t chunk = (int64_t)SEL_THREADS * SEL_COMPACT_ITEMS;
  for (int64_t c0 = 0; c0 < ndocs; c0 += chunk) {
    const int64_t v0 = c0 + (int64_t)threadIdx.x * SEL_COMPACT_ITEMS;
    int take_flags = 0, tie_flags = 0, ntie = 0;
    int32_t xs[SEL_COMPACT_ITEMS];
#pragma unroll
    for (int i = 0; i < SEL_COMPACT_ITEMS; ++i) {
      const int64_t v = v0 + i;
      xs[i] = v < ndocs ? f[v] : NO_HIT;
      if (xs[i] != NO_HIT) {
        if (MODE == 1 || take_all) {
          take_flags |= 1 << i;
        } else {
          const uint32_t u = fp_key(xs[i]);
          if (u > T) take_flags |= 1 << i;
          else if (u == T) { tie_flags |= 1 << i; ++ntie; }
        }
      }
    }
    long long tie_total = 0, tie_rank = 0;
    if (MODE == 0 && !take_all) {
      tie_rank = block_exclusive_scan(ntie, wsum, &s_tot);
      tie_total = s_tot;
    }
#pragma unroll
    for (int i = 0; i < SEL_COMPACT_ITEMS; ++i)
      if (tie_flags & (1 << i)) {
        if (ties_seen + tie_rank < need) take_flags |= 1 << i;
        ++tie_rank;
      }
    long long pos = block_exclusive_scan(__popc(take_flags), wsum, &s_tot);
    const long long take_total = s_tot;
#pragma unroll
    for (int i = 0; i < SEL_COMPACT_ITEMS; ++i)
      if (take_flags & (1 << i)) {
        if (MODE == 1 || written + pos < ncand) {
          out_ids[base_out + written + pos] = (int32_t)(v0 + i);
          if (MODE == 0) out_keys[base_out + written + pos] = xs[i];
        }
        ++pos;
      }
    written += take_total;
    ties_seen += tie_total;
  }
  if (MODE == 0) {
    for (int64_t i = written + threadIdx.x; i < ncand; i += SEL_THREADS) {
      out_ids[base_out + i] = -1;
      out_keys[base_out + i] = 0;
    }
    if (threadIdx.x == 0) n_valid[q] = (int32_t)(written < ncand ? written : ncand);
  }
}

// ---------------------------------------------------------------------
// Refinement select split over P chunks of documents per query, so that a
// launch with few queries still fills the chip, and long F' rows are read by
// many workgroups (with 128 queries or more over fewer than 2^19 documents,
// k_select runs one workgroup per query instead).  A radix select on the order
// key u = fp_key(F') finds the ncand-th largest key T and how many documents
// with key T to keep (the lowest ids): bits 31..20 come from the walk's
// histogram, bits 19..8 and 7..0 from two histogram passes over the chunks
// (global atomics, only documents whose higher bits match count).  The middle
// pass reads F' and lists each chunk's documents at or above the 12-bit
// prefix, which the last pass reads instead of F'.  The last
// pass also records, per chunk, how many keys lie above the 24-bit prefix and
// the chunk's own histogram of the low 8 bits, so that once T is known every
// chunk's kept and tied counts follow without another pass; the counts are
// scanned per query, and each chunk that keeps documents writes its part of
// the candidate list in ascending doc order.
// SelState per query: the bins found so far, the count still to place, T and
// the ties to keep.
struct SelState {
  long long rem;     // candidates still to place below the bins fixed so far
  uint32_t prefix;   // key bits fixed so far
  uint32_t T;        // threshold key (0: keep every hit)
  long long need;    // documents with key T to keep
  long long total;   // candidates written
};
constexpr int SPLIT_THREADS = 256;

// Documents per chunk of the split select: a multiple of 16, so that chunks
// start 16-byte aligned within an F' row.
__host__ __device__ inline int64_t sel_chunk_docs(int64_t ndocs, int P) { return ((ndocs + P - 1) / P + 15) / 16 * 16; }


// Per query: bin of bits 31..20 from the walk's histogram; clears the
// histograms of the next passes.
__global__ __launch_bounds__(SPLIT_THREADS) void k_sel_first(const uint32_t *__restrict__ hist1, int ncand,
                                                             uint32_t *__restrict__ hist2, uint32_t *__restrict__ hist3,
                                                             SelState *__restrict__ st) {
  __shared__ long long wsum[SPLIT_THREADS / 64];
  __shared__ long long s_tot, s_above;
  __shared__ int s_bin;
  const int64_t q = blockIdx.x;
  const uint32_t *h = hist1 + q * SEL_BINS;
  long long local = 0;
  for (int i = threadIdx.x; i < SEL_BINS; i += SPLIT_THREADS) {
    local += h[i];
    hist2[q * SEL_BINS + i] = 0;
  }
  for (int i = threadIdx.x; i < 256; i += SPLIT_THREADS) hist3[q * 256 + i] = 0;
  block_exclusive_scan(local, wsum, &s_tot);
  const long long nhit = s_tot;
  if (nhit <= ncand) {
    if (threadIdx.x == 0) st[q] = SelState{0, 0, 0, 0, 0};
    return;
  }
  select_bin(h, SEL_BINS, ncand, wsum, &s_tot, &s_bin, &s_above);
  if (threadIdx.x == 0) st[q] = SelState{ncand - s_above, (uint32_t)s_bin, 1, 0, 0};
}

// Per query: the next bin from a pass's histogram; after the last pass, the
// threshold key T and the ties to keep.
template <int BITS, bool LAST>
__global__ __launch_bounds__(SPLIT_THREADS) void k_sel_next(const uint32_t *__restrict__ hin, SelState *__restrict__ st) {
  __shared__ long long wsum[SPLIT_THREADS / 64];
  __shared__ long long s_tot, s_above;
  __shared__ int s_bin;
  const int64_t q = blockIdx.x;
  const SelState s0 = st[q];
  if (s0.T == 0) return;
  select_bin(hin + q * (1 << BITS), 1 << BITS, s0.rem, wsum, &s_tot, &s_bin, &s_above);
  if (threadIdx.x == 0) {
    SelState s1 = s0;
    s1.prefix = (s0.prefix << BITS) | (uint32_t)s_bin;
    s1.rem = s0.rem - s_above;
    if (LAST) {
      s1.T = s1.prefix;
      s1.need = s1.rem;
    }
    st[q] = s1;
  }
}

// Last histogram pass over one chunk (bits 7..0 under the 24-bit prefix),
// over the middle pass's list of the chunk (or its F' when that list was not
// kept), plus the chunk's own record: chunk_hist [256] of those keys and
// chunk_above, the number of keys above the prefix (every hit when all are
// kept).
// The last histogram pass also lists, per chunk and in document order, the
// documents whose 24-bit key prefix reaches the bin being resolved (those
// above it and those in it), so that the write pass reads these lists
// instead of F' again.  A list longer than cap is not kept (the write pass
// then reads the chunk's F').
constexpr int SEL_LAST_ITEMS = 16;  // contiguous F' entries per thread and step
constexpr uint32_t SEL_NO_LIST = 0xFFFFFFFFu;

__host__ __device__ inline int sel_list_cap(int64_t ndocs, int P, int ncand) {
  const int64_t per = sel_chunk_docs(ndocs, P);
  return (int)std::min<int64_t>(per, 4 * ((int64_t)ncand / P) + 1024);
}

// The middle histogram pass over one chunk (bits 19..8 under the 12-bit
// prefix), which also lists, in document order, the chunk's documents whose
// top 12 key bits reach the prefix (those above the prefix's bin and those in
// it: every document the select can keep), so that the last pass reads these
// lists instead of F'.  A list longer than cap is not kept (clen = SEL_NO_LIST;
// the last pass then reads the chunk's F').
__global__ __launch_bounds__(SPLIT_THREADS) void k_sel_mid(const int32_t *__restrict__ fp, int64_t ndocs, int P,
                                                           const SelState *__restrict__ st,
                                                           uint32_t *__restrict__ hout, int cap,
                                                           int2 *__restrict__ clist, uint32_t *__restrict__ clen) {
  __shared__ uint32_t h[SEL_BINS];
  __shared__ long long wsum[SPLIT_THREADS / 64];
  __shared__ long long s_tot;
  const int64_t q = blockIdx.x / P;
  const int c = blockIdx.x % P;
  if (st[q].T == 0) return;  // uniform: every hit is kept
  const uint32_t prefix = st[q].prefix;
  for (int i = threadIdx.x; i < SEL_BINS; i += SPLIT_THREADS) h[i] = 0;
  __syncthreads();
  const int64_t per = sel_chunk_docs(ndocs, P), v0 = min(ndocs, c * per), v1 = min(ndocs, v0 + per);
  const int32_t *f = fp + q * ndocs;
  int2 *L = clist + ((int64_t)q * P + c) * cap;
  long long nlist = 0;  // uniform
  const int64_t step = (int64_t)SPLIT_THREADS * SEL_LAST_ITEMS;
  const bool vec = ((uintptr_t)f & 15) == 0 && (v0 & 3) == 0;
  for (int64_t vb = v0; vb < v1; vb += step) {
    const int64_t vt = vb + (int64_t)threadIdx.x * SEL_LAST_ITEMS;
    int32_t x[SEL_LAST_ITEMS];
    if (vec && vt + SEL_LAST_ITEMS <= v1) {
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; i += 4) {
        const int4 y = *(const int4 *)(f + vt + i);
        x[i] = y.x;
        x[i + 1] = y.y;
        x[i + 2] = y.z;
        x[i + 3] = y.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; ++i) x[i] = vt + i < v1 ? f[vt + i] : NO_HIT;
    }
    int flags = 0;
#pragma unroll
    for (int i = 0; i < SEL_LAST_ITEMS; ++i) {
      if (x[i] == NO_HIT) continue;
      const uint32_t u = fp_key(x[i]);
      if ((u >> 20) > prefix) {
        flags |= 1 << i;
      } else if ((u >> 20) == prefix) {
        atomicAdd(&h[(u >> 8) & (SEL_BINS - 1)], 1u);
        flags |= 1 << i;
      }
    }
    long long pos = block_exclusive_scan(__popc(flags), wsum, &s_tot);
    const long long tot = s_tot;
#pragma unroll
    for (int i = 0; i < SEL_LAST_ITEMS; ++i)
      if (flags & (1 << i)) {
        if (nlist + pos < cap) L[nlist + pos] = make_int2((int)(vt + i), x[i]);
        ++pos;
      }
    nlist += tot;
  }
  __syncthreads();
  uint32_t *o = hout + q * SEL_BINS;
  for (int i = threadIdx.x; i < SEL_BINS; i += SPLIT_THREADS)
    if (h[i]) atomicAdd(&o[i], h[i]);
  if (threadIdx.x == 0) clen[(int64_t)q * P + c] = nlist <= cap ? (uint32_t)nlist : SEL_NO_LIST;
}

__global__ __launch_bounds__(SPLIT_THREADS) void k_sel_last(const int32_t *__restrict__ fp, int64_t ndocs, int P,
                                                            const SelState *__restrict__ st,
                                                            uint32_t *__restrict__ hout,
                                                            uint32_t *__restrict__ chunk_hist,
                                                            uint32_t *__restrict__ chunk_above, int cap,
                                                            const int2 *__restrict__ mlist,
                                                            const uint32_t *__restrict__ mlen,
                                                            int2 *__restrict__ clist, uint32_t *__restrict__ clen) {
  __shared__ uint32_t h[256];
  __shared__ uint32_t s_above;
  __shared__ long long wsum[SPLIT_THREADS / 64];
  __shared__ long long s_tot;
  const int64_t q = blockIdx.x / P;
  const int c = blockIdx.x % P;
  const bool all = st[q].T == 0;  // uniform: every hit is kept (no list: the write pass reads F')
  const uint32_t prefix = st[q].prefix;
  for (int i = threadIdx.x; i < 256; i += SPLIT_THREADS) h[i] = 0;
  if (threadIdx.x == 0) s_above = 0;
  __syncthreads();
  const int64_t per = sel_chunk_docs(ndocs, P), v0 = min(ndocs, c * per), v1 = min(ndocs, v0 + per);
  const int32_t *f = fp + q * ndocs;
  int2 *L = clist + ((int64_t)q * P + c) * cap;
  uint32_t above = 0;
  long long nlist = 0;  // uniform
  const int64_t step = (int64_t)SPLIT_THREADS * SEL_LAST_ITEMS;
  // the middle pass's list of the chunk (documents with the 12-bit prefix or
  // above, with their F'), when it kept one; else F' itself
  const uint32_t ml = all ? SEL_NO_LIST : mlen[(int64_t)q * P + c];
  const bool from_list = ml != SEL_NO_LIST;  // uniform
  const int2 *M = mlist + ((int64_t)q * P + c) * cap;
  const int64_t b0 = from_list ? 0 : v0, b1 = from_list ? (int64_t)ml : v1;
  // 16-byte loads where the row allows it (every F' row starts 16-byte
  // aligned when ndocs is a multiple of 4, and chunks start at multiples of 16)
  const bool vec = !from_list && ((uintptr_t)f & 15) == 0 && (v0 & 3) == 0;
  for (int64_t vb = b0; vb < b1; vb += step) {
    const int64_t vt = vb + (int64_t)threadIdx.x * SEL_LAST_ITEMS;
    int32_t x[SEL_LAST_ITEMS], d[SEL_LAST_ITEMS];
    if (from_list) {
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; ++i) {
        const int2 e = vt + i < b1 ? M[vt + i] : make_int2(0, NO_HIT);
        d[i] = e.x;
        x[i] = e.y;
      }
    } else if (vec && vt + SEL_LAST_ITEMS <= v1) {
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; i += 4) {
        const int4 y = *(const int4 *)(f + vt + i);
        x[i] = y.x;
        x[i + 1] = y.y;
        x[i + 2] = y.z;
        x[i + 3] = y.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; ++i) x[i] = vt + i < v1 ? f[vt + i] : NO_HIT;
    }
    if (!from_list) {
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; ++i) d[i] = (int)(vt + i);
    }
    int flags = 0;
#pragma unroll
    for (int i = 0; i < SEL_LAST_ITEMS; ++i) {
      if (x[i] == NO_HIT) continue;
      const uint32_t u = fp_key(x[i]);
      if (all || (u >> 8) > prefix) {
        ++above;
        flags |= 1 << i;
      } else if ((u >> 8) == prefix) {
        atomicAdd(&h[u & 255u], 1u);
        flags |= 1 << i;
      }
    }
    if (!all) {
      long long pos = block_exclusive_scan(__popc(flags), wsum, &s_tot);
      const long long tot = s_tot;
#pragma unroll
      for (int i = 0; i < SEL_LAST_ITEMS; ++i)
        if (flags & (1 << i)) {
          if (nlist + pos < cap) L[nlist + pos] = make_int2(d[i], x[i]);
          ++pos;
        }
      nlist += tot;
    }
  }
  atomicAdd(&s_above, above);
  __syncthreads();
  uint32_t *o = hout + q * 256, *ch = chunk_hist + ((int64_t)q * P + c) * 256;
  for (int i = threadIdx.x; i < 256; i += SPLIT_THREADS) {
    ch[i] = h[i];
    if (h[i]) atomicAdd(&o[i], h[i]);
  }
  if (threadIdx.x == 0) {
    chunk_above[(int64_t)q * P + c] = s_above;
    clen[(int64_t)q * P + c] = !all && nlist <= cap ? (uint32_t)nlist : SEL_NO_LIST;
  }
}

// Per query: every chunk's kept (key > T) and tied (key == T) counts from its
// record, then (in order) its output offset, ties before it and the number it
// keeps [3 per chunk], the number of candidates, and the padding of the
// unused slots.
__global__ __launch_bounds__(SPLIT_THREADS) void k_sel_scan(int P, int ncand, SelState *__restrict__ st,
                                                            const uint32_t *__restrict__ chunk_hist,
                                                            const uint32_t *__restrict__ chunk_above,
                                                            long long *__restrict__ counts, int32_t *__restrict__ out_ids,
                                                            int32_t *__restrict__ out_keys,
                                                            int32_t *__restrict__ n_valid) {
  __shared__ long long wsum[SPLIT_THREADS / 64];
  __shared__ long long s_tot;
  const int64_t q = blockIdx.x;
  const uint32_t T = st[q].T;
  const long long need = st[q].need;
  const int b3 = (int)(T & 255u);
  // thread t owns chunks [c0, c1): two block scans (ties before each chunk,
  // then output offsets) instead of one thread walking every chunk
  const int per = (P + SPLIT_THREADS - 1) / SPLIT_THREADS;
  const int c0 = min(P, (int)threadIdx.x * per), c1 = min(P, c0 + per);
  long long my_ties = 0;
  for (int c = c0; c < c1; ++c) {
    const uint32_t *ch = chunk_hist + ((int64_t)q * P + c) * 256;
    long long above = chunk_above[(int64_t)q * P + c], ties = 0;
    if (T != 0) {
      for (int b = b3 + 1; b < 256; ++b) above += ch[b];
      ties = ch[b3];
    }
    counts[3 * (q * P + c)] = above;
    counts[3 * (q * P + c) + 1] = ties;
    my_ties += ties;
  }
  long long tb = block_exclusive_scan(my_ties, wsum, &s_tot);
  long long my_take = 0;
  for (int c = c0; c < c1; ++c) {
    long long *cc = counts + 3 * (q * P + c);
    const long long a = cc[0], t = cc[1];
    const long long take = a + max(0ll, min(t, need - tb));
    cc[1] = tb;
    cc[2] = take;
    tb += t;
    my_take += take;
  }
  long long off = block_exclusive_scan(my_take, wsum, &s_tot);
  const long long n = min(s_tot, (long long)ncand);
  for (int c = c0; c < c1; ++c) {
    long long *cc = counts + 3 * (q * P + c);
    cc[0] = off;
    off += cc[2];
  }
  if (threadIdx.x == 0) {
    st[q].total = n;
    n_valid[q] = (int32_t)n;
  }
  for (long long i = n + threadIdx.x; i < ncand; i += SPLIT_THREADS) {
    out_ids[q * ncand + i] = -1;
    out_keys[q * ncand + i] = 0;
  }
}

// ---------------------------------------------------------------------
// The select of a small batch: the same result in three launches instead of
// seven, for chunks of SEL_CHUNK documents where nq chunks of a query are no
// more than the split select would make (launch_select).  Its time is
// launches and the latency of each launch's chain, not bytes.
//  k_keep_list  per chunk: the bin of bits 31..20 from the walk's histogram
//               (every workgroup finds it for itself), and the chunk's
//               documents whose top 12 bits reach it, in document order, at a
//               place of the query's list reserved by one atomic;
//  k_keep_cut   T and the ties to keep (bits 19..8, then 7..0), each chunk's
//               kept and tied counts, their prefix sums, the number of
//               candidates and the padding;
//  k_sel_write  per chunk, as in the split select.
// How long a query's list gets is up to the data: the bins of the first pass
// are 0.25 wide in F', so that few query tokens, or many ties, put most
// documents into the bin that is cut.  A list of at most keep_short entries
// is cut by one workgroup, from registers.  For a longer one every pass stays
// spread over the chunks: k_keep_list adds the histogram of bits 19..8,
// k_keep_cut has a workgroup for every four chunks, which record their counts
// and the histogram of bits 7..0, and the one that arrives last finds T and
// sums the chunks' counts.  (Lists of more than cap entries are not kept: F'
// is read instead.)
// One query of 100,000 documents: 54 us in seven launches before, now 22 us;
// of 2.2M documents 116 us, now 45 us; 16 queries of 1,000 documents 60 us,
// now 17 us (the list in registers and the prefix sums by DPP are half of
// that: 35, 61 and 31 us without them).  Long lists, 1M documents: one query of
// four tokens 58 us (1,600 us when one workgroup read F' three times, 76 us in
// seven launches), 16 of them 136 us (1,660 and 138), 64 of them 385 us (2,750
// and 325); one query of 262,144 candidates 48 us (311 and 68).
constexpr int SEL_CHUNK = 4096;
constexpr int SEL_MAX_CHUNKS = 3072;  // of a query: their counts are in LDS, 57 KB with the bins

// Entries of the list a thread of k_keep_cut keeps in registers over the passes.
constexpr int KEEP_REGS = 24;
constexpr int CUT_CHUNKS = SEL_THREADS / SPLIT_THREADS;  // of a workgroup of k_keep_cut

// Entries that the list of a query in K chunks holds: as many as both of the
// split select's lists, in whose scratch it is.
__host__ inline int64_t keep_cap(int64_t ndocs, int64_t K, int ncand) {
  return std::min<int64_t>(ndocs, 2 * K * sel_list_cap(ndocs, (int)K, ncand));
}
// Entries up to which one workgroup cuts a list.
__host__ __device__ inline uint32_t keep_short(int64_t cap) {
  return (uint32_t)std::min<int64_t>(cap, KEEP_REGS * SEL_THREADS);
}

// Scratch of the small batch's select, in this order: the arrays that are zero
// on entry (select_zero_bytes), then the others.
struct SmallSel {
  uint32_t *hist2, *hist3;     // [nq][4096], [nq][256] bits 19..8 and 7..0 of long lists
  uint32_t *nlist, *arrived;   // [nq] list lengths; [nq] workgroups of k_keep_cut that are done
  SelState *st;                // [nq]
  long long *counts;           // [nq][K][3]
  uint2 *part;                 // [nq][K] where a chunk's entries start in the list, and how many they are
  uint32_t *rec;               // [nq][K][2] a chunk's documents above the 24-bit prefix, and in it
  uint32_t *rows;              // [nq][K][128] a chunk's histogram of bits 7..0, two counts a word
  int2 *list;                  // [nq][cap] document, F'
};
__host__ inline SmallSel small_sel(void *scratch, int64_t nq, int64_t K) {
  SmallSel x;
  x.hist2 = (uint32_t *)scratch;
  x.hist3 = x.hist2 + nq * SEL_BINS;
  x.nlist = x.hist3 + nq * 256;
  x.arrived = x.nlist + nq;
  x.st = (SelState *)(x.arrived + nq);
  x.counts = (long long *)(x.st + nq);
  x.part = (uint2 *)(x.counts + 3 * nq * K);
  x.rec = (uint32_t *)(x.part + nq * K);
  x.rows = x.rec + 2 * nq * K;
  x.list = (int2 *)(x.rows + 128 * nq * K);
  return x;
}
static size_t small_sel_bytes(int64_t nq, int64_t K, int64_t cap) {
  return (size_t)((char *)(small_sel(nullptr, nq, K).list + nq * cap) - (char *)nullptr);
}

// F' of documents v0 .. v0 + 15 (those below v1; NO_HIT past it).
__device__ __forceinline__ void load_fp16(const int32_t *f, int64_t v0, int64_t v1, int32_t (&x)[16]) {
  if (((uintptr_t)f & 15) == 0 && v0 + 16 <= v1) {  // (v0 is a multiple of 16)
#pragma unroll
    for (int i = 0; i < 16; i += 4) {
      const int4 y = *(const int4 *)(f + v0 + i);
      x[i] = y.x;
      x[i + 1] = y.y;
      x[i + 2] = y.z;
      x[i + 3] = y.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = v0 + i < v1 ? f[v0 + i] : NO_HIT;
  }
}

__global__ __launch_bounds__(SPLIT_THREADS) void k_keep_list(const int32_t *__restrict__ fp,
                                                             const uint32_t *__restrict__ hist1, int64_t ndocs, int P,
                                                             int ncand, int64_t cap, SmallSel S) {
  constexpr int W = SPLIT_THREADS / 64;
  __shared__ uint32_t wsum[2][W];
  __shared__ uint3 s_bin;
  __shared__ uint32_t s_at;
  __shared__ uint32_t h[SEL_BINS];
  const int64_t q = blockIdx.x / P;
  const int c = blockIdx.x % P;
  const int64_t v0 = (int64_t)c * SEL_CHUNK + threadIdx.x * 16, v1 = min(ndocs, (int64_t)(c + 1) * SEL_CHUNK);
  int32_t x[16];
  load_fp16(fp + q * ndocs, v0, v1, x);
  const uint32_t nhit = find_bin<W, SEL_BINS / SPLIT_THREADS>(hist1 + q * SEL_BINS, (uint32_t)ncand, wsum[0], &s_bin);
  const bool all = nhit <= (uint32_t)ncand;  // no more hits than candidates: all are listed
  const uint32_t b1 = all ? 0 : s_bin.x;
  // the whole list's length
  const uint32_t nl = all ? nhit : s_bin.y + s_bin.z;
  uint32_t n = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) n += x[i] != NO_HIT && (fp_key(x[i]) >> 20) >= b1;
  uint32_t tot;
  uint32_t pos = block_scan<W>(n, wsum[1], tot);
  if (threadIdx.x == 0) {
    s_at = tot ? atomicAdd(&S.nlist[q], tot) : 0;
    S.part[q * P + c] = make_uint2(s_at, tot);
  }
  const bool hist = nl > keep_short(cap) && !all && tot > 0;  // uniform
  if (hist)
    for (int i = threadIdx.x; i < SEL_BINS; i += SPLIT_THREADS) h[i] = 0;
  __syncthreads();
  if (nl <= (uint64_t)cap) {  // uniform
    pos += s_at;
    int2 *L = S.list + q * cap;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (x[i] != NO_HIT && (fp_key(x[i]) >> 20) >= b1) {
        if (pos < (uint64_t)cap) L[pos] = make_int2((int)(v0 + i), x[i]);
        ++pos;
      }
  }
  if (!hist) return;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (x[i] != NO_HIT && (fp_key(x[i]) >> 20) == b1) atomicAdd(&h[(fp_key(x[i]) >> 8) & 4095u], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < SEL_BINS; i += SPLIT_THREADS)
    if (h[i]) atomicAdd(&S.hist2[q * SEL_BINS + i], h[i]);
}

// Words that one workgroup writes and another of the same launch reads: agent
// scope goes past the XCDs' caches, so the writer needs no write-back of its
// whole L2 (a __threadfence in every wave cost 25 ns each: 0.9 of 1.3 ms for 64
// queries of 1M documents), only its own stores to be done (wait_stores).
__device__ __forceinline__ uint32_t load_agent(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(uint32_t *p, uint32_t x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_stores() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);  // every counter at zero: stores and atomics are done
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Workgroup b < nq: query b's list, when it is short.  Workgroup nq + q PB + g:
// chunks CUT_CHUNKS g .. of query q (256 threads each), when its list is long.
__global__ __launch_bounds__(SEL_THREADS) void k_keep_cut(const int32_t *__restrict__ fp,
                                                          const uint32_t *__restrict__ hist1, int64_t nq,
                                                          int64_t ndocs, int P, int PB, int ncand, int64_t cap,
                                                          SmallSel S, int32_t *__restrict__ out_ids,
                                                          int32_t *__restrict__ out_keys,
                                                          int32_t *__restrict__ n_valid) {
  constexpr int W = SEL_THREADS / 64, PER = SEL_BINS / SEL_THREADS;
  __shared__ __align__(16) uint32_t hist[2][SEL_BINS];
  __shared__ uint32_t wsum[5][W];
  __shared__ uint3 s_bin[3];
  __shared__ uint32_t s_cnt[CUT_CHUNKS][2], s_done;
  extern __shared__ uint32_t chunk_n[];  // [P] kept, [P] tied
  const bool one = (int64_t)blockIdx.x < nq;  // the whole list by this workgroup
  const int64_t b = (int64_t)blockIdx.x - nq, q = one ? blockIdx.x : b / PB;
  const uint32_t nl = S.nlist[q];
  if (one != (nl <= keep_short(cap))) return;  // uniform
  int2 r[KEEP_REGS];
  if (one) {
    const int2 *L = S.list + q * cap;
#pragma unroll
    for (int u = 0; u < KEEP_REGS; ++u) {
      const uint32_t i = threadIdx.x + u * SEL_THREADS;
      r[u] = i < nl ? L[i] : make_int2(0, NO_HIT);
    }
  }
  for (int i = threadIdx.x; i < 2 * SEL_BINS; i += SEL_THREADS) hist[0][i] = 0;
  if (threadIdx.x < 2 * CUT_CHUNKS) s_cnt[0][threadIdx.x] = 0;
  const uint32_t nhit = find_bin<W, PER>(hist1 + q * SEL_BINS, (uint32_t)ncand, wsum[0], &s_bin[0]);
  const bool cut = nhit > (uint32_t)ncand;  // uniform
  const uint32_t b1 = cut ? s_bin[0].x : 0, rem1 = (uint32_t)ncand - (cut ? s_bin[0].y : 0);
  uint32_t T = 0, need = 0;
  // ties before each chunk, then output offsets, from the chunks' kept and
  // tied counts in chunk_n (a thread reads those of its own chunks)
  const int per = (P + SEL_THREADS - 1) / SEL_THREADS;
  const int c0 = min(P, (int)threadIdx.x * per), c1 = min(P, c0 + per);
  auto finish = [&]() {
    uint32_t my = 0, all;
    for (int c = c0; c < c1; ++c) my += chunk_n[P + c];
    uint32_t tb = block_scan<W>(my, wsum[3], all);
    my = 0;
    for (int c = c0; c < c1; ++c) {
      const uint32_t t = chunk_n[P + c], take = chunk_n[c] + (tb < need ? min(t, need - tb) : 0);
      S.counts[3 * (q * P + c) + 1] = tb;
      S.counts[3 * (q * P + c) + 2] = take;
      chunk_n[c] = take;
      tb += t;
      my += take;
    }
    uint32_t off = block_scan<W>(my, wsum[4], all);
    for (int c = c0; c < c1; ++c) {
      S.counts[3 * (q * P + c)] = off;
      off += chunk_n[c];
    }
    const uint32_t kept = min(all, (uint32_t)ncand);
    if (threadIdx.x == 0) {
      S.st[q] = SelState{0, 0, T, (long long)need, (long long)kept};
      n_valid[q] = (int32_t)kept;
    }
    for (uint32_t i = kept + threadIdx.x; i < (uint32_t)ncand; i += SEL_THREADS) {
      out_ids[q * ncand + i] = -1;
      out_keys[q * ncand + i] = 0;
    }
  };

  if (one) {
    // g(document, key) of every entry
    auto each = [&](auto &&g) {
#pragma unroll
      for (int u = 0; u < KEEP_REGS; ++u)
        if (r[u].y != NO_HIT) g(r[u].x, fp_key(r[u].y));
    };
    for (int i = threadIdx.x; i < 2 * P; i += SEL_THREADS) chunk_n[i] = 0;
    if (cut) {
      each([&](int, uint32_t u) {
        if ((u >> 20) == b1) atomicAdd(&hist[0][(u >> 8) & 4095u], 1u);
      });
      __syncthreads();
      find_bin<W, PER>(hist[0], rem1, wsum[1], &s_bin[1]);
      const uint32_t p2 = (b1 << 12) | s_bin[1].x, rem2 = rem1 - s_bin[1].y;
      each([&](int, uint32_t u) {
        if ((u >> 8) == p2) atomicAdd(&hist[1][u & 255u], 1u);
      });
      __syncthreads();
      find_bin<W, PER>(hist[1], rem2, wsum[2], &s_bin[2]);
      T = (p2 << 8) | s_bin[2].x;
      need = rem2 - s_bin[2].y;
    }
    __syncthreads();  // chunk_n is zero
    each([&](int d, uint32_t u) {
      if (u > T) atomicAdd(&chunk_n[d / SEL_CHUNK], 1u);
      else if (u == T) atomicAdd(&chunk_n[P + d / SEL_CHUNK], 1u);
    });
    __syncthreads();
    finish();
    return;
  }

  // a long list: this workgroup's chunks, from their part of the list or F'
  uint32_t p2 = 0, rem2 = 0;
  if (cut) {
    find_bin<W, PER>(S.hist2 + q * SEL_BINS, rem1, wsum[1], &s_bin[1]);
    p2 = (b1 << 12) | s_bin[1].x;
    rem2 = rem1 - s_bin[1].y;
    const int g = threadIdx.x / SPLIT_THREADS, t = threadIdx.x % SPLIT_THREADS;
    const int c = (int)(b % PB) * CUT_CHUNKS + g;
    uint32_t *h = hist[0] + 256 * g;  // this chunk's histogram of bits 7..0
    uint32_t above = 0, in = 0;
    auto count = [&](int32_t x) {
      if (x == NO_HIT) return;
      const uint32_t u = fp_key(x);
      if ((u >> 8) > p2) ++above;
      else if ((u >> 8) == p2) ++in, atomicAdd(&h[u & 255u], 1u);
    };
    if (c < P) {
      if (nl <= (uint64_t)cap) {  // uniform
        const uint2 pt = S.part[q * P + c];
        const int2 *L = S.list + q * cap + pt.x;
        for (uint32_t i = t; i < pt.y; i += SPLIT_THREADS) count(L[i].y);
      } else {
        int32_t x[16];
        load_fp16(fp + q * ndocs, (int64_t)c * SEL_CHUNK + t * 16, min(ndocs, (int64_t)(c + 1) * SEL_CHUNK), x);
#pragma unroll
        for (int i = 0; i < 16; ++i) count(x[i]);
      }
    }
    above = wave_incl_scan(above);
    in = wave_incl_scan(in);
    if (lane_id() == 63) {
      atomicAdd(&s_cnt[g][0], above);
      atomicAdd(&s_cnt[g][1], in);
    }
    __syncthreads();
    if (c < P) {
      if (t < 2) store_agent(S.rec + 2 * (q * P + c) + t, s_cnt[g][t]);
      if (s_cnt[g][1]) {  // (a chunk's counts are at most 4096)
        if (t < 128) store_agent(S.rows + (q * P + c) * 128 + t, h[2 * t] | h[2 * t + 1] << 16);
        if (h[t]) atomicAdd(&S.hist3[q * 256 + t], h[t]);
      }
    }
    // the query's last workgroup to get here finds every chunk's record
    wait_stores();
    __syncthreads();
    if (threadIdx.x == 0) s_done = atomicAdd(&S.arrived[q], 1u);
    __syncthreads();
    if (s_done != (uint32_t)PB - 1) return;  // uniform
    if (threadIdx.x < 256) hist[1][threadIdx.x] = load_agent(&S.hist3[q * 256 + threadIdx.x]);
    __syncthreads();
    find_bin<W, PER>(hist[1], rem2, wsum[2], &s_bin[2]);
    T = (p2 << 8) | s_bin[2].x;
    need = rem2 - s_bin[2].y;
    const uint32_t b3 = T & 255u;
    // 16 lanes a chunk, 16 of its 256 counts each
    const uint32_t sub = threadIdx.x & 15;
    for (int k0 = 0; k0 < P; k0 += SEL_THREADS / 16) {
      const int k = k0 + (int)(threadIdx.x / 16);
      uint32_t more = 0, ties = 0;
      if (k < P) {
        const uint32_t *rec = S.rec + 2 * (q * P + k), *row = S.rows + (q * P + k) * 128 + 8 * sub;
        const uint32_t n = load_agent(rec + 1);
        if (sub == 0) more = load_agent(rec);
        if (n) {
          uint32_t y[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) y[i] = load_agent(row + i);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t lo = 16 * sub + 2 * i;
            more += (lo > b3 ? y[i] & 0xFFFFu : 0) + (lo + 1 > b3 ? y[i] >> 16 : 0);
            ties += lo == b3 ? y[i] & 0xFFFFu : lo + 1 == b3 ? y[i] >> 16 : 0;
          }
        }
      }
#pragma unroll
      for (int m = 1; m < 16; m <<= 1) {
        more += shfl_xor(more, m);
        ties += shfl_xor(ties, m);
      }
      if (k < P && sub == 0) {
        chunk_n[k] = more;
        chunk_n[P + k] = ties;
      }
    }
    __syncthreads();
  } else {
    // every hit is kept: the chunks' counts are those of the first pass
    if (b % PB != 0) return;  // uniform
    for (int k = c0; k < c1; ++k) {
      chunk_n[k] = S.part[q * P + k].y;
      chunk_n[P + k] = 0;
    }
  }
  finish();
}

// Per chunk: the ordered compaction of its kept documents, from the chunk's
// list when the last pass kept one, else from F'.
__global__ __launch_bounds__(SPLIT_THREADS) void k_sel_write(const int32_t *__restrict__ fp, int64_t ndocs, int P,
                                                             int ncand, const SelState *__restrict__ st,
                                                             const long long *__restrict__ counts, int cap,
                                                             const int2 *__restrict__ clist,
                                                             const uint32_t *__restrict__ clen,
                                                             const uint32_t *__restrict__ nlist, int64_t qcap,
                                                             const uint2 *__restrict__ part,
                                                             int32_t *__restrict__ out_ids,
                                                             int32_t *__restrict__ out_keys) {
  __shared__ long long wsum[SPLIT_THREADS / 64];
  __shared__ long long s_tot;
  const int64_t q = blockIdx.x / P;
  const int c = blockIdx.x % P;
  const uint32_t T = st[q].T;
  const long long need = st[q].need;
  const long long *cc = counts + 3 * (q * P + c);
  if (cc[2] == 0 || cc[0] >= ncand) return;  // uniform: the chunk keeps nothing that fits
  long long written = cc[0], ties_seen = cc[1];
  // the chunk's list: its own (the split select), or its part of the query's
  const uint2 pt = part ? part[q * P + c] : make_uint2(0, 0);
  const uint32_t nl = !part ? clen[q * P + c] : nlist[q] <= qcap ? pt.y : SEL_NO_LIST;
  const bool from_list = nl != SEL_NO_LIST;  // uniform
  const int2 *L = part ? clist + q * qcap + pt.x : clist + (q * P + c) * (int64_t)cap;
  const int64_t per = part ? SEL_CHUNK : sel_chunk_docs(ndocs, P);
  const int64_t vb = min(ndocs, c * per), ve = min(ndocs, vb + per);
  const int64_t b0 = from_list ? 0 : vb, b1 = from_list ? (int64_t)nl : ve;
  const int32_t *f = fp + q * ndocs;
  const int64_t step = (int64_t)SPLIT_THREADS * SEL_ITEMS;
  for (int64_t c0 = b0; c0 < b1; c0 += step) {
    const int64_t j0 = c0 + (int64_t)threadIdx.x * SEL_ITEMS;
    int take_flags = 0, tie_flags = 0, ntie = 0;
    int32_t xs[SEL_ITEMS], vs[SEL_ITEMS];
#pragma unroll
    for (int i = 0; i < SEL_ITEMS; ++i) {
      const int64_t j = j0 + i;
      if (from_list) {
        const int2 e = j < b1 ? L[j] : make_int2(-1, NO_HIT);
        vs[i] = e.x;
        xs[i] = e.y;
      } else {
        vs[i] = (int32_t)j;
        xs[i] = j < b1 ? f[j] : NO_HIT;
      }
      if (xs[i] != NO_HIT) {
        const uint32_t u = fp_key(xs[i]);
        if (u > T) take_flags |= 1 << i;
        else if (u == T) { tie_flags |= 1 << i; ++ntie; }
      }
    }
    long long tie_rank = block_exclusive_scan(ntie, wsum, &s_tot);
    const long long tie_total = s_tot;
#pragma unroll
    for (int i = 0; i < SEL_ITEMS; ++i)
      if (tie_flags & (1 << i)) {
        if (ties_seen + tie_rank < need) take_flags |= 1 << i;
        ++tie_rank;
      }
    long long pos = block_exclusive_scan(__popc(take_flags), wsum, &s_tot);
    const long long take_total = s_tot;
#pragma unroll
    for (int i = 0; i < SEL_ITEMS; ++i)
      if (take_flags & (1 << i)) {
        if (written + pos < ncand) {
          out_ids[q * ncand + written + pos] = vs[i];
          out_keys[q * ncand + written + pos] = xs[i];
        }
        ++pos;
      }
    written += take_total;
    ties_seen += tie_total;
  }
}

// Chunks per query of the split select: about 16384 workgroups over the
// batch (measured at 8.8M: 34 ms per step against 55 ms for 2048), each
// chunk at least 4096 documents.
int select_chunks(int64_t nq, int64_t ndocs) {
  const int64_t by_q = (16384 + nq - 1) / std::max<int64_t>(1, nq);
  const int64_t by_docs = (ndocs + 4095) / 4096;
  return (int)std::max<int64_t>(1, std::min(by_q, by_docs));
}

// Enough queries to fill the chip with one workgroup each, over short enough
// F' rows: k_select, one launch (measured faster than the split passes at
// 100,000 documents, slower at 1M; at 256 queries of 100,000 documents 115 us
// against 150 us for the small batch's three launches).
static bool select_by_query(int64_t nq, int64_t ndocs) { return nq >= 128 && ndocs < (1 << 19); }

// Chunks of the small batch's select, 0 where it is not used: as long as a
// chunk of SEL_CHUNK documents is no smaller than the split select's.
static int keep_chunks(int64_t nq, int64_t ndocs) {
  if (select_by_query(nq, ndocs)) return 0;
  const int64_t P = (ndocs + SEL_CHUNK - 1) / SEL_CHUNK;
  return P <= SEL_MAX_CHUNKS && nq * P <= 16384 ? (int)P : 0;
}

// The split select's size whichever is used, so that what fits a fixed scratch
// does not depend on the choice (the small batch's never needs more).
size_t select_scratch_bytes(int64_t nq, int64_t ndocs, int ncand) {
  const int P = select_chunks(nq, ndocs);
  const size_t cap = (size_t)sel_list_cap(ndocs, P, ncand);
  const size_t split = (size_t)nq * (sizeof(SelState) + (SEL_BINS + 256) * 4 +
                                     (size_t)P * (24 + 256 * 4 + 4 + 4 + cap * 8)) + (size_t)nq * P * (4 + cap * 8) + 1024;
  const int64_t K = keep_chunks(nq, ndocs);
  return K ? std::max(split, small_sel_bytes(nq, K, keep_cap(ndocs, K, ncand))) : split;
}

size_t select_zero_bytes(int64_t nq, int64_t ndocs) {
  return keep_chunks(nq, ndocs) ? (size_t)nq * (SEL_BINS + 256 + 2) * 4 : 0;
}

void launch_select(const int32_t *fp, const uint32_t *hist, int64_t nq, int64_t ndocs, int ncand, void *scratch,
                   int32_t *cand_ids, int32_t *cand_keys, int32_t *n_valid, hipStream_t s) {
  if (nq <= 0) return;
  if (const int K = keep_chunks(nq, ndocs)) {
    const int64_t cap = keep_cap(ndocs, K, ncand);
    const SmallSel x = small_sel(scratch, nq, K);
    const int PB = (K + CUT_CHUNKS - 1) / CUT_CHUNKS;
    const dim3 gc((unsigned)(nq * K)), tb(SPLIT_THREADS);
    hipLaunchKernelGGL(k_keep_list, gc, tb, 0, s, fp, hist, ndocs, K, ncand, cap, x);
    hipLaunchKernelGGL(k_keep_cut, dim3((unsigned)(nq * (1 + PB))), dim3(SEL_THREADS), (size_t)K * 8, s, fp, hist, nq,
                       ndocs, K, PB, ncand, cap, x, cand_ids, cand_keys, n_valid);
    hipLaunchKernelGGL(k_sel_write, gc, tb, 0, s, fp, ndocs, K, ncand, x.st, x.counts, 0, x.list,
                       (const uint32_t *)nullptr, x.nlist, cap, x.part, cand_ids, cand_keys);
    return;
  }
  if (select_by_query(nq, ndocs)) {
    hipLaunchKernelGGL((k_select<0>), dim3((unsigned)nq), dim3(SEL_THREADS), 0, s, fp, hist, ndocs, ncand,
                       (const int64_t *)nullptr, cand_ids, cand_keys, n_valid);
    return;
  }
  const int P = select_chunks(nq, ndocs);
  SelState *st = (SelState *)scratch;
  uint32_t *hist2 = (uint32_t *)(st + nq);
  uint32_t *hist3 = hist2 + nq * SEL_BINS;
  long long *counts = (long long *)(((uintptr_t)(hist3 + nq * 256) + 15) & ~(uintptr_t)15);
  uint32_t *chunk_hist = (uint32_t *)(counts + 3 * nq * P);
  uint32_t *chunk_above = chunk_hist + (size_t)nq * P * 256;
  uint32_t *clen = chunk_above + (size_t)nq * P;
  const int cap = sel_list_cap(ndocs, P, ncand);
  int2 *clist = (int2 *)(((uintptr_t)(clen + (size_t)nq * P) + 15) & ~(uintptr_t)15);
  uint32_t *mlen = (uint32_t *)(clist + (size_t)nq * P * cap);
  int2 *mlist = (int2 *)(((uintptr_t)(mlen + (size_t)nq * P) + 15) & ~(uintptr_t)15);
  const dim3 gq((unsigned)nq), gc((unsigned)(nq * P)), tb(SPLIT_THREADS);
  hipLaunchKernelGGL(k_sel_first, gq, tb, 0, s, hist, ncand, hist2, hist3, st);
  hipLaunchKernelGGL(k_sel_mid, gc, tb, 0, s, fp, ndocs, P, st, hist2, cap, mlist, mlen);
  hipLaunchKernelGGL((k_sel_next<12, false>), gq, tb, 0, s, hist2, st);
  hipLaunchKernelGGL(k_sel_last, gc, tb, 0, s, fp, ndocs, P, st, hist3, chunk_hist, chunk_above, cap, mlist, mlen,
                     clist, clen);
  hipLaunchKernelGGL((k_sel_next<8, true>), gq, tb, 0, s, hist3, st);
  hipLaunchKernelGGL(k_sel_scan, gq, tb, 0, s, P, ncand, st, chunk_hist, chunk_above, counts, cand_ids, cand_keys,
                     n_valid);
  hipLaunchKernelGGL(k_sel_write, gc, tb, 0, s, fp, ndocs, P, ncand, st, counts, cap, clist, clen,
                     (const uint32_t *)nullptr, (int64_t)0, (const uint2 *)nullptr, cand_ids, cand_keys);
}

__global__ __launch_bounds__(256) void k_count_hits(const int32_t *__restrict__ fp, int64_t ndocs,
                                                    int64_t *__restrict__ counts) {
  __shared__ unsigned long long acc;
  if (threadIdx.x == 0) acc = 0;
  __syncthreads();
  const int32_t *f = fp + (int64_t)blockIdx.x * ndocs;
  unsigned long long local = 0;
  for (int64_t v = threadIdx.x; v < ndocs; v += 256) local += f[v] != NO_HIT;
  atomicAdd(&acc, local);
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = (int64_t)acc;
}

void launch_count_hits(const int32_t *fp, int64_t nq, int64_t ndocs, int64_t *counts, hipStream_t s) {
  hipLaunchKernelGGL(k_count_hits, dim3((unsigned)nq), dim3(256), 0, s, fp, ndocs, counts);
}

void launch_list_hits(const int32_t *fp, int64_t nq, int64_t ndocs, const int64_t *offsets, int32_t *doc_ids,
                      hipStream_t s) {
  hipLaunchKernelGGL((k_select<1>), dim3((unsigned)nq), dim3(SEL_THREADS), 0, s, fp, (const uint32_t *)nullptr, ndocs,
                     0, offsets, doc_ids, (int32_t *)nullptr, (int32_t *)nullptr);
}

}  // namespace chimera
