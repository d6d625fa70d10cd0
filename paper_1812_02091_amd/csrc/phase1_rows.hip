// Phase 1 of LC-ACT (Sec. 4, Phase 1) with float32 keys, lists of up to 32
// entries.  Table modes: per (vocabulary row, query) the nearest query words
// of Alg. 3 and their capacities.  Pair mode (Q2D of a candidate pair): the
// query's words as rows against the database row's words, and the transfers
// of the query's mass summed per block of rows.
//
// Bound: the float32 MFMA (157 TFLOP/s; 134-150 in a loop of nothing but
// MFMAs and their LDS reads; here 113 on lists of 4, 110 on lists of 8).
// Float32 MFMAs and vector instructions hardly run side by side on a SIMD, so
// every vector instruction adds to the contraction's time, and keeping them
// few is what this kernel is about.
//
// Contraction: a workgroup of four waves takes 128 vocabulary rows; wave w
// owns rows 32w .. 32w + 31.  The rows are the MFMA's N operand (each lane
// reads its row's dims straight from global memory, a 32-dim slice ahead),
// the queries' words its M operand (a slice of two or three tiles of 32
// staged in LDS for the four waves), so that after a pass a lane holds 32 or
// 48 keys of its own row -- words 32 t + 8 (r / 4) + 4 (lane / 32) + r % 4 --
// in its accumulators.
//
// Queries: an item takes up to eight, their words end to end, so that tiles
// are full (a query alone wastes half a tile, 13 % at 118 words) and the next
// query's slices are in flight while a query ends.  The tile in which a
// query ends is selected from once per query that has words there, the
// others' keys masked.  18,000 documents of ~118 words x 5,300 words of 61
// others and back, RWMD: items of one query 54.8 ms, of eight 48.7; 500
// queries over a 70,000-word vocabulary, k = 16: 29.1 -> 26.3 ms.
//
// Selection: in registers.  A key and its word's position make one 64-bit
// number that orders by (key, position), compared as float64 (the key's bits
// on top; positions complemented under negative keys): a compare-exchange is
// v_min_f64 + v_max_f64.  Each 16 keys go through a sorting network and are
// merged into the lane's sorted list, the two lanes of a row merge theirs at
// the end.  No branch, no LDS, and the list is exactly the row's LK smallest:
// nothing has to be certified or redone but ICT rows deeper than the list.
// The kernel this replaced put every key through LDS (two barriers per 64
// words) and merged lists held there entry by entry with a band for quantised
// keys.  Against it, tables: the RWMD matrix above 75 -> 48.7 ms, the 500
// queries 42.7 -> 26.3, 784 grid words x 20,000 images, k = 8, 7.7 -> 2.6.
//
// Distances: |v|^2 + key unless cancellation could bite (below a quarter of
// |v|^2 + |c|^2), where it is recomputed by direct differences.  Most of
// those are a word against itself, which is 0 without a look at its dims
// (the loop over 300 dims was 9 % of the RWMD matrix above: in most items
// some row meets its own word).
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace lcemd {

typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int kFR = 128;        // rows per workgroup
constexpr int kFStride = 144;   // bytes per staged word slice (128 + 16 pad: conflict-free 16-byte reads)
constexpr int kFCat = 2 * LCEMD_MAX_HIST;  // words of an item's queries in LDS at a time
constexpr float kFGuard = 0.25f;
// No key: above every key, also +inf (a word whose squared norm is beyond
// float32 is the farthest word, not a missing one) and the NaN that arithmetic
// gives (0x7fc00000, between two such words); itself a quiet NaN, which a sum
// hands on as it is, but not yet one as the high half of a float64.
constexpr uint32_t kNoKey = 0x7fe00000u;

// Tiles per pass at most, and workgroups per CU.  Two tiles bring a wave of
// lists of up to 8 entries near 168 registers (tables of 1, 2, 4 and 8 spill
// 8, 9, 11 and 22), three workgroups per CU, which hide each other's
// latencies: lists of 1, items of eight queries, two tiles and three
// workgroups 48.7 ms, three and two 50.3, four and two 52.0 (the RWMD matrix
// above).  Longer lists spill too much there (k = 16: 30.2 ms against 26.4 with
// three tiles and two workgroups, 28.0 with four).  Lists of 32 spill 116
// registers at two workgroups and are still the faster way: 64 queries against
// 18,000 documents of a 70,000-word vocabulary, k = 17 / 24 / 32, 6.2 / 6.2 /
// 6.2 ms a call, 11.8 / 12.2 / 12.3 on the kernel this replaced.  The pair mode
// has one short segment per item, for which two workgroups of wider passes are
// the faster (2.1 against 2.3 ms over 500 queries; lists of 16 spill 14).  Embeddings of at most 28
// dims (SMALL) have one slice and little to contract, so what counts there is
// how many waves hide the set-up and the selection (four workgroups, at 128
// registers, spill: 20,000 images x 784 words, k = 8, 2.9 against 2.6 ms).
template <int MODE, int LK, bool SMALL>
constexpr int max_tiles() { return SMALL || (MODE != P1_PAIR && LK <= 8) ? 2 : 3; }
template <int MODE, int LK, bool SMALL>
constexpr int groups_per_cu() { return LK <= 8 && (SMALL || MODE != P1_PAIR) ? 3 : 2; }

template <int MODE, int LK, bool SMALL>
struct F32Smem {
  unsigned char st[SMALL ? 1 : 2][32 * max_tiles<MODE, LK, SMALL>() * kFStride];  // word slices, double-buffered
  float rcost[kFR];       // pair mode: the rows' costs
  int cid[kFCat + 32 * max_tiles<MODE, LK, SMALL>()];   // zero_word past the queries' words, up to a pass's end
  float cap[kFCat + 32 * max_tiles<MODE, LK, SMALL>()];
  float qn[kFCat + 32 * max_tiles<MODE, LK, SMALL>()];  // kNoKey there, and with a zero dot product the key too
};

// queries per item group: 8, or 32 over vocabularies of at least 2^18 used
// words, where a row block's vectors are reused by more items before they
// leave L2 (1M words: phase 1 -2 %; 70,000 words: 8 keeps a group's query
// vectors within an XCD's L2)
__host__ __device__ inline int f32_group_log2(int64_t v_used) { return v_used >= (int64_t(1) << 18) ? 5 : 3; }

// Table modes over embeddings of more than 28 dims take several queries per
// item, their words end to end.  (SMALL: with next to nothing to contract the
// selection over all tiles at once, unrolled, is worth more: 2.6 ms against
// 2.9 on the images above.)
template <int MODE, bool SMALL>
constexpr bool streams() { return MODE != P1_PAIR && !SMALL; }
constexpr int kStreamLog2 = 3;

__device__ __forceinline__ double dmin(double a, double b) {
  double d;
  asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double dmax(double a, double b) {
  double d;
  asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ void cas(double& a, double& b) {
  const double x = a, y = b;
  a = dmin(x, y);
  b = dmax(x, y);
}

// Batcher's odd-even merge sort of N (a power of two) keys at k[0 .. N)
template <int N>
__device__ __forceinline__ void net_sort(double* k) {
#pragma unroll
  for (int p = 1; p < N; p <<= 1)
#pragma unroll
    for (int q = p; q >= 1; q >>= 1)
#pragma unroll
      for (int j = q % p; j + q < N; j += 2 * q)
#pragma unroll
        for (int i = 0; i < q; ++i)
          if (i + j + q < N && (i + j) / (2 * p) == (i + j + q) / (2 * p)) cas(k[i + j], k[i + j + q]);
}

// a (ascending, LK) := the LK smallest of a and b (ascending, NB <= LK)
template <int LK, int NB>
__device__ __forceinline__ void net_merge(double* a, const double* b) {
#pragma unroll
  for (int i = 0; i < NB; ++i) a[LK - 1 - i] = dmin(a[LK - 1 - i], b[i]);
  // bitonic now
#pragma unroll
  for (int h = LK >> 1; h > 0; h >>= 1)
#pragma unroll
    for (int i = 0; i < LK; ++i)
      if ((i & h) == 0) cas(a[i], a[i + h]);
}

// The tile's 16 keys into the lane's list.
template <int LK>
__device__ __forceinline__ void take16(double (&lst)[LK], double (&k)[16]) {
  if constexpr (LK == 1) {
#pragma unroll
    for (int h = 8; h > 0; h >>= 1)
#pragma unroll
      for (int i = 0; i < h; ++i) k[i] = dmin(k[i], k[i + h]);
    lst[0] = dmin(lst[0], k[0]);
  } else if constexpr (LK >= 16) {
    net_sort<16>(k);
    net_merge<LK, 16>(lst, k);
  } else {
#pragma unroll
    for (int i = 0; i < 16; i += LK) net_sort<LK>(k + i);
#pragma unroll
    for (int w = LK; w < 16; w <<= 1)
#pragma unroll
      for (int i = 0; i < 16; i += 2 * w) net_merge<LK, LK>(k + i, k + i + w);
    net_merge<LK, LK>(lst, k);
  }
}

// Squared distance by direct differences over the m4 float4 groups that
// hold the real dims.  FOUR: four partial sums over pairs of groups (at most
// 28 dims), else one sum.
template <bool FOUR>
__device__ __forceinline__ float f32_exact_d2(const float* __restrict__ V, int m_pad, int m4, int a, int b,
                                              float an) {
  const float4* x = (const float4*)(V + (size_t)a * m_pad);
  const float4* y = (const float4*)(V + (size_t)b * m_pad);
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  if (a == b && an < INFINITY) return 0.f;  // (an = |a|^2: a row of finite numbers against itself)
  const int n4 = FOUR ? (m4 + 1) & ~1 : m4;  // (m_pad / 4 is even; the padding adds exact zeros)
#pragma unroll 4
  for (int d = 0; d < n4; ++d) {
    const float4 p = x[d], q = y[d];
    const float e0 = p.x - q.x, e1 = p.y - q.y, e2 = p.z - q.z, e3 = p.w - q.w;
    if constexpr (FOUR) {
      s0 = fmaf(e0, e0, s0);
      s1 = fmaf(e1, e1, s1);
      s2 = fmaf(e2, e2, s2);
      s3 = fmaf(e3, e3, s3);
    } else {
      s0 = fmaf(e0, e0, s0);
      s0 = fmaf(e1, e1, s0);
      s0 = fmaf(e2, e2, s0);
      s0 = fmaf(e3, e3, s0);
    }
  }
  return FOUR ? (s0 + s1) + (s2 + s3) : s0;
}

// One staged slice on NT 32-word tiles (NT fixed at compile time so the
// MFMAs issue back to back without branches); the first njq of its four
// groups of MFMAs (the others hold no real dims and would add exact zeros).
template <int NT, bool FULL, int MAXT>
__device__ __forceinline__ void f32_slice(floatx16 (&acc)[MAXT], const float4 (&rows)[4], const unsigned char* st, int li,
                                          int lh, int njq) {
  // lane half lh supplies dims [16 lh, 16 lh + 16) of the 32-dim slice
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (!FULL && j >= njq) break;
    float4 wv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
      wv[t] = *(const float4*)(st + (32 * t + li) * kFStride + lh * 64 + j * 16);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[t].x, rows[j].x, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[t].y, rows[j].y, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[t].z, rows[j].z, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[t].w, rows[j].w, acc[t], 0, 0, 0);
  }
}

// What a thread has in flight: the lane's row's next slice, and the pieces of
// the words' next slice that it stages (word 32 it + tid / 8, piece tid % 8).
struct Flight {
  const unsigned char* rptr;
  const unsigned char* wptr[3];
  float4 r[4];
  float4 w[3];
  template <int NT>
  __device__ __forceinline__ void words(const unsigned char* vb, size_t rowbytes, const int* cid, int tid) {
#pragma unroll
    for (int it = 0; it < NT; ++it) wptr[it] = vb + (size_t)cid[32 * it + (tid >> 3)] * rowbytes + (tid & 7) * 16;
  }
  __device__ __forceinline__ void load_rows(int sl) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = *(const float4*)(rptr + sl * 128 + i * 16);
  }
  template <int NT>
  __device__ __forceinline__ void load_words(int sl) {
#pragma unroll
    for (int it = 0; it < NT; ++it) w[it] = *(const float4*)(wptr[it] + sl * 128);
  }
  template <int NT>
  __device__ __forceinline__ void load(int sl) {
    load_rows(sl);
    load_words<NT>(sl);
  }
};

// One pass: the dot products of NT tiles of words from c0 on, all slices
// (live: the wave has rows; it stages words either way).  A pass is a
// function of its own tile count so that the accumulators stay in the same
// registers throughout (a switch inside the slice loop had them copied, 200
// moves a slice).
template <int NT, int MODE, int LK, bool SMALL>
__device__ __forceinline__ void f32_pass(F32Smem<MODE, LK, SMALL>& sm, Flight& fl, floatx16 (&acc)[max_tiles<MODE, LK, SMALL>()], int c0,
                                         bool more, bool live, int nsl, int last_njq, const unsigned char* vb,
                                         size_t rowbytes, int tid) {
  const int lane = tid & 63, li = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  auto stage = [&](int buf) {
#pragma unroll
    for (int it = 0; it < NT; ++it)
      *(float4*)(sm.st[buf] + (32 * it + (tid >> 3)) * kFStride + (tid & 7) * 16) = fl.w[it];
  };
  // (one barrier a slice; two, with one buffer, took the same time)
  __syncthreads();  // the previous pass's slices are consumed
  stage(0);
  if constexpr (!SMALL) {
    if (nsl > 1) fl.load_words<NT>(1);
    __syncthreads();
    for (int sl = 0; sl < nsl - 1; ++sl) {
      stage((sl + 1) & 1);  // (last read a slice ago, before the barrier)
      if (sl + 2 < nsl) fl.load_words<NT>(sl + 2);
      if (live) f32_slice<NT, true>(acc, fl.r, sm.st[sl & 1], li, lh, 4);
      fl.load_rows(sl + 1);
      __syncthreads();
    }
  } else {
    __syncthreads();
  }
  if (more) {  // the next pass's first slice (it has at most NT tiles)
    fl.words<NT>(vb, rowbytes, sm.cid + c0 + 32 * NT, tid);
    fl.load_words<NT>(0);
  }
  if (live) f32_slice<NT, false>(acc, fl.r, sm.st[SMALL ? 0 : (nsl - 1) & 1], li, lh, last_njq);
  if (more) fl.load_rows(0);
}

// The lane's row.
struct RowInfo {
  int64_t r;    // table modes: table row
  int id;       // word
  float vn;     // |v|^2
  float bound;  // table modes: largest database weight; pair mode: weight
  bool ok;
};

// A finished list (merged over the row's two lanes): distances and cut.
// Both lanes of a row do the same arithmetic.
template <int MODE, int LK, bool SMALL>
struct Cut {
  float z[LK], w[LK];
  int pos[LK];  // in the item's words
  int D = 0;
  bool covered = false;
  __device__ __forceinline__ Cut(const P1Args& a, const F32Smem<MODE, LK, SMALL>& sm, double (&lst)[LK], const RowInfo& row,
                                 int h) {
    constexpr bool kCapStop = MODE != P1_TABLE_FULL;
    {
      double other[LK];
#pragma unroll
      for (int i = 0; i < LK; ++i)
        other[i] = __hiloint2double(__shfl_xor(__double2hiint(lst[i]), 32), __shfl_xor(__double2loint(lst[i]), 32));
      net_merge<LK, LK>(lst, other);
    }
    int kef;
    if constexpr (MODE == P1_TABLE_FULL) {
      kef = min(a.k, h);
    } else {
      if (a.method == LCEMD_ICT) kef = h;
      else if (a.method == LCEMD_OMR) kef = min(2, h);
      else if (a.method == LCEMD_RWMD) kef = 1;
      else kef = min(a.k, h);
    }
    float Pc = 0.f;
#pragma unroll
    for (int l = 0; l < LK; ++l) {
      z[l] = 0.f;
      w[l] = 0.f;
      pos[l] = 0;
      const int bits = __double2hiint(lst[l]);
      const bool live = row.ok && !covered && bits != (int)kNoKey;
      if (!__any(live)) continue;
      if (live) {
        pos[l] = __double2loint(lst[l]) ^ (bits >> 31);
        const float qn = sm.qn[pos[l]];
        float d2 = row.vn + __int_as_float(bits);
        bool need = !(d2 >= kFGuard * (row.vn + qn));
        if (kCapStop && a.method == LCEMD_OMR && l == 0) need = true;
        if (need) d2 = f32_exact_d2<SMALL>(a.V, a.m_pad, a.m4, row.id, sm.cid[pos[l]], row.vn);
        z[l] = sqrtf(fmaxf(d2, 0.f));
        w[l] = sm.cap[pos[l]];
        ++D;
        Pc += w[l];
        covered = D >= kef;
        if (kCapStop) covered = covered || Pc >= row.bound || (a.method == LCEMD_OMR && l == 0 && d2 != 0.f);
      }
    }
  }
};

// Table modes: a row's list for the query at words [seg, seg + h) of the
// item, out.  The two lanes of a row share the stores.
template <int MODE, int LK, bool SMALL>
__device__ __forceinline__ void f32_store(const P1Args& a, const F32Smem<MODE, LK, SMALL>& sm, double (&lst)[LK],
                                          const RowInfo& row, int64_t qi, int seg, int h, int lh) {
  const Cut<MODE, LK, SMALL> c(a, sm, lst, row, h);
  if (!row.ok) return;
  // an ICT row deeper than the list: redone exactly by k_fix_rows while the
  // redo list has room, else the launch reports overflow.  So is a row with keys
  // that are no numbers (+inf - inf: words whose squared norms are beyond float32,
  // against the row of one),
  // which come first in the list, by position; where the redo list is full it
  // keeps that order.
  const bool deeper = !c.covered && c.D < h;
  const uint32_t first = (uint32_t)__double2hiint(lst[0]);
  const bool unordered = (first << 1) > 0xff000000u && first != kNoKey;
  if ((deeper || unordered) && lh == 0) {
    bool listed = false;
    if (a.fix_list) {
      const int slot = atomicAdd(a.fix_count, 1);
      listed = slot < a.fix_cap;
      if (listed) a.fix_list[slot] = qi * a.v_used + row.r;
    }
    if (!listed && deeper && a.overflow) a.overflow[0] = 1;
  }
  if constexpr (MODE == P1_TABLE) {
    if (c.D > a.KT && a.overflow) a.overflow[0] = 1;
#pragma unroll
    for (int l = 0; l < LK; l += 2) {
      if (((l >> 1) & 1) == lh && l < c.D && l < a.KT) {
        constexpr int kOdd = LK > 1 ? 1 : 0;  // (LK = 1: a row has one entry)
        const bool two = kOdd && l + 1 < c.D && l + 1 < a.KT;
        *zw_pair(a.ZW, a.zw_nq, a.KT, qi, row.r, l >> 1) =
            make_float4(c.z[l], l == c.D - 1 ? INFINITY : c.w[l], two ? c.z[l + kOdd] : 0.f,
                        two ? (l + 1 == c.D - 1 ? INFINITY : c.w[l + kOdd]) : 0.f);
      }
    }
  } else {
    const int64_t o0 = (qi * a.v_used + row.r) * (int64_t)a.k;
#pragma unroll
    for (int l = 0; l < LK; ++l) {
      if ((l & 1) == lh && l < a.k) {
        const bool in = l < c.D;
        a.S[o0 + l] = in ? c.pos[l] - seg : -1;
        a.Z[o0 + l] = in ? c.z[l] : 0.f;
        a.W[o0 + l] = in ? c.w[l] : 0.f;
      }
    }
  }
}

// The words in LDS (n of them) against the lanes' rows.  Streams: they are
// those of the queries qs .. qe - 1 of the launch, the first of which starts
// at word s0 of the batch, and each query's list is stored where its words
// end, inside the last tile that has some.  Else they are one query's (pair
// mode: the database row's), and lst is left to the caller.
template <int MODE, int LK, bool SMALL>
__device__ __forceinline__ void f32_words(const P1Args& a, F32Smem<MODE, LK, SMALL>& sm, double (&lst)[LK], const RowInfo& row,
                                          int n, int64_t qs, int64_t qe, int64_t s0, int tid) {
  constexpr bool kStream = streams<MODE, SMALL>();
  const int lh = (tid & 63) >> 5;
  const bool live = __any(row.ok);  // the wave has rows
  const size_t rowbytes = (size_t)a.m_pad * 4;
  const int nsl = SMALL ? 1 : (a.m4 + 7) >> 3;  // 32-dim slices that hold real dims
  const int last_njq = min(4, a.m4 - 8 * (nsl - 1));
  const unsigned char* vb = (const unsigned char*)a.V;
  auto reset = [&]() {
#pragma unroll
    for (int i = 0; i < LK; ++i) lst[i] = __hiloint2double((int)kNoKey, 0);
  };
  // the query whose words are being taken, and where they begin and end
  int64_t qi = qs;
  int b = 0, e = n;
  auto next = [&]() {  // the next query that has words (fixed-size batches have empty slots)
    do {
      b = e;
      if (++qi >= qe) break;
      e = (int)(a.qptr[a.q0 + qi + 1] - s0);
    } while (e == b);
  };
  if constexpr (kStream) {
    qi = qs - 1;
    e = 0;
    next();
  }
  // the lane's i-th key of the tile of words from j0 on: its word and bits
  auto at = [&](int j0, int i) { return j0 | (lh << 2) | (8 * (i >> 2) + (i & 3)); };
  auto keys = [&](const floatx16& acc, int j0, int (&bits)[16]) {
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const float4 qn = *(const float4*)(sm.qn + j0 + 8 * rq + 4 * lh);
      const float qv[4] = {qn.x, qn.y, qn.z, qn.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) bits[4 * rq + i] = __float_as_int(qv[i] - 2.f * acc[4 * rq + i]);
    }
  };
  auto take = [&](int j0, const int (&bits)[16]) {
    double k[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) k[i] = __hiloint2double(bits[i], (bits[i] >> 31) ^ at(j0, i));
    take16<LK>(lst, k);
  };
  reset();
  // passes of at most kNT tiles, as even as they come (a pass of one tile
  // costs its barriers and latencies like one of four), longer ones first
  constexpr int kNT = max_tiles<MODE, LK, SMALL>();
  const int nt = (n + 31) >> 5, npass = (nt + kNT - 1) / kNT, base = nt / npass, extra = nt % npass;
  Flight fl;
  fl.rptr = vb + (size_t)row.id * rowbytes + lh * 64;
  fl.words<kNT>(vb, rowbytes, sm.cid, tid);
  fl.load<kNT>(0);
  int c0 = 0;
#pragma unroll 1
  for (int p = 0; p < npass; ++p) {
    const int tiles = base + (p < extra ? 1 : 0);
    const bool more = p + 1 < npass;
    floatx16 acc[kNT];
    auto pass = [&](auto nt_) {
      f32_pass<decltype(nt_)::value, MODE, LK, SMALL>(sm, fl, acc, c0, more, live, nsl, last_njq, vb, rowbytes, tid);
    };
    if (tiles == 1) pass(std::integral_constant<int, 1>());
    else if (kNT == 2 || tiles == 2) pass(std::integral_constant<int, 2>());
    else pass(std::integral_constant<int, kNT>());
    // ---- selection: 16 keys of the lane's row per tile ----
    if constexpr (!kStream) {
      if (live) {
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          if (t >= tiles) break;
          int bits[16];
          keys(acc[t], c0 + 32 * t, bits);
          take(c0 + 32 * t, bits);
        }
      }
    } else if (live) {
      // per query of the tile; one copy of the code for all tiles (the next
      // one's sums move to acc[0])
#pragma unroll 1
      for (int t = 0; t < tiles; ++t) {
        const int j0 = c0 + 32 * t, j1 = j0 + 32;
#pragma unroll 1
        while (qi < qe) {
          int bits[16];
          keys(acc[0], j0, bits);
          if (b > j0 || e < j1) {  // not the other queries' words
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if ((unsigned)(at(j0, i) - b) >= (unsigned)(e - b)) bits[i] = (int)kNoKey;
          }
          take(j0, bits);
          if (e > j1) break;
          f32_store<MODE, LK, SMALL>(a, sm, lst, row, qi, b, e - b, lh);
          reset();
          next();
          if (b >= j1) break;
        }
#pragma unroll
        for (int i = 0; i + 1 < kNT; ++i) acc[i] = acc[i + 1];
      }
    }
    c0 += 32 * tiles;
  }
}

// One work item: (up to 2^glog queries, 128-row block) in the table modes,
// (candidate pair, 128-row block of the query's words) in pair mode.  Returns
// early (uniformly) for empty items.
template <int MODE, int LK, bool SMALL>
__device__ __forceinline__ void f32_task(const P1Args& a, F32Smem<MODE, LK, SMALL>& sm, int64_t item, int lg, int glog) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 31, lh = lane >> 5;
  constexpr int kPad = 32 * max_tiles<MODE, LK, SMALL>();  // (past the words: a pass's)
  RowInfo row;
  double lst[LK];
  if constexpr (MODE == P1_PAIR) {
    // partial sums of 128 rows, or 64 (SMALL: two per item)
    const int nblk = SMALL ? (a.rb_max + 1) >> 1 : a.rb_max;
    const int64_t pair = item / nblk;
    const int blk = (int)(item % nblk);
    const int part = SMALL ? 2 * blk : blk;  // the first partial sum here
    const int64_t qr = pair / a.cand_use, b = a.qlist ? (int64_t)a.qlist[qr] : qr;
    const int64_t u = (int64_t)(uint32_t)a.cand[qr * a.cand_ld + pair % a.cand_use];
    const int64_t q0 = a.qptr[b] + blk * kFR;
    const int nrows = (int)min((int64_t)kFR, a.qptr[b + 1] - q0);
    if (nrows <= 0 || u >= a.n) {
      if (tid == 0) a.partial[pair * a.rb_max + part] = 0.f;
      if (SMALL && tid == 0 && part + 1 < a.rb_max) a.partial[pair * a.rb_max + part + 1] = 0.f;
      return;
    }
    row.ok = 32 * wave + li < nrows;
    const int64_t i = q0 + (row.ok ? 32 * wave + li : 0);
    row.id = a.qcol[i];
    row.bound = row.ok ? a.qval[i] : 0.f;
    const int64_t s0 = a.xptr[u];
    const int h = (int)(a.xptr[u + 1] - s0);
    for (int c = tid; c < h + kPad; c += kThreads) {
      const int w = c < h ? a.xcol[s0 + c] : a.zero_word;
      sm.cid[c] = w;
      sm.cap[c] = c < h ? __int_as_float(a.xcv[s0 + c].y) : 0.f;
      sm.qn[c] = c < h ? a.vnorm[w] : __uint_as_float(kNoKey);
    }
    row.vn = a.vnorm[row.id];
    __syncthreads();
    f32_words<MODE, LK, SMALL>(a, sm, lst, row, h, 0, 1, 0, tid);
    const Cut<MODE, LK, SMALL> c(a, sm, lst, row, h);
    // the transfers of the row's mass (the last entry takes the rest), then
    // the rows' sum in order
    if (!c.covered && c.D < h && row.ok && a.overflow) a.overflow[0] = 1;  // a list too short
    if (lh == 0) {
      float rem = row.bound, cost = 0.f;
#pragma unroll
      for (int l = 0; l < LK; ++l) {
        if (l < c.D) {
          const float t = l == c.D - 1 ? rem : fminf(rem, c.w[l]);
          rem -= t;
          cost = fmaf(t, c.z[l], cost);
        }
      }
      sm.rcost[32 * wave + li] = cost;
    }
    __syncthreads();
    constexpr int kPart = SMALL ? 64 : kFR;
    if (tid % kPart == 0 && tid < kFR && part + tid / kPart < a.rb_max) {
      float tot = 0.f;
      for (int i = tid; i < min(tid + kPart, nrows); ++i) tot += sm.rcost[i];
      a.partial[pair * a.rb_max + part + tid / kPart] = tot;
    }
  } else {
    // items run query-fastest within a group of queries, then row block, then
    // group: an XCD's contiguous range of items keeps a group's query vectors
    // and a row block's vectors in its L2
    const int64_t nrb = (a.v_used + kFR - 1) / kFR;
    const int64_t t0 = item >> (lg - glog);
    const int64_t rblk = t0 % nrb;
    int64_t qs = ((t0 / nrb) << lg) + ((item & ((int64_t(1) << (lg - glog)) - 1)) << glog);
    const int64_t qend = min(qs + (int64_t(1) << glog), a.nq);
    const int64_t r0 = rblk * kFR;
    row.r = r0 + 32 * wave + li;  // the lane's row (both halves)
    row.ok = row.r < a.v_used;
    row.id = row.ok ? a.used[row.r] : a.used[r0];
    row.bound = MODE == P1_TABLE ? (row.ok ? a.xmax[row.r] : 0.f) : INFINITY;
    row.vn = a.vnorm[row.id];
#pragma unroll 1
    while (qs < qend) {
      // as many of the queries as LDS holds
      const int64_t s0 = a.qptr[a.q0 + qs];
      int64_t qe = qs + 1;
      while (streams<MODE, SMALL>() && qe < qend && a.qptr[a.q0 + qe + 1] - s0 <= kFCat) ++qe;
      const int n = (int)(a.qptr[a.q0 + qe] - s0);
      if (n > 0) {
        __syncthreads();  // the words before are done with
        for (int c = tid; c < n + kPad; c += kThreads) {
          const int w = c < n ? a.qcol[s0 + c] : a.zero_word;
          sm.cid[c] = w;
          sm.cap[c] = c < n ? a.qval[s0 + c] : 0.f;
          sm.qn[c] = c < n ? a.vnorm[w] : __uint_as_float(kNoKey);
        }
        __syncthreads();
        f32_words<MODE, LK, SMALL>(a, sm, lst, row, n, qs, qe, s0, tid);
        if constexpr (!streams<MODE, SMALL>()) f32_store<MODE, LK, SMALL>(a, sm, lst, row, qs, 0, n, lh);
      }
      qs = qe;
    }
  }
}

// Persistent grid: as many workgroups as stay resident, each pulling items
// from the counter of its XCD (workgroup i runs on XCD i % 8), which walks a
// contiguous eighth of the items; the counter is read one item ahead.  Every
// workgroup exits once its counter passes the end of its range.
template <int MODE, int LK, bool SMALL>
__global__ __launch_bounds__(kThreads, (groups_per_cu<MODE, LK, SMALL>())) void k_phase1_rows(P1Args a, int64_t total,
                                                                                      int lg, int glog) {
  __shared__ F32Smem<MODE, LK, SMALL> sm;
  __shared__ int64_t s_item;
  // no more items than workgroups: one each, no counter (and none to clear;
  // the streams' registers are full, and large launches are what they are for)
  const bool once = !streams<MODE, SMALL>() && total <= (int64_t)gridDim.x;
  const int xcd = blockIdx.x & 7;
  const int64_t lo = total * xcd / 8, hi = once ? total : total * (xcd + 1) / 8;
  unsigned long long nxt = 0;
  if (threadIdx.x == 0 && !once) nxt = atomicAdd(&a.work_ctr[xcd], 1ull);
  int64_t item = blockIdx.x;
  while (true) {
    if (!once) {
      __syncthreads();  // the previous item is done with LDS and s_item
      if (threadIdx.x == 0) {
        s_item = lo + (int64_t)nxt;
        if (lo + (int64_t)nxt < hi) nxt = atomicAdd(&a.work_ctr[xcd], 1ull);
      }
      __syncthreads();
      item = s_item;
    }
    if (item >= hi) break;
    f32_task<MODE, LK, SMALL>(a, sm, item, lg, glog);
    if (once) break;
  }
}

template <int MODE, int LK, bool SMALL>
hipError_t launch_f32_one(const P1Args& a, hipStream_t s) {
  int64_t total;
  int lg = f32_group_log2(a.v_used), glog = 0;
  const void* fn = (const void*)k_phase1_rows<MODE, LK, SMALL>;
  const int resident = persistent_grid(fn, kThreads, 0, int64_t(1) << 40);
  if (resident <= 0) return hipErrorInvalidConfiguration;
  if (MODE == P1_PAIR) {
    total = a.npairs * (SMALL ? (a.rb_max + 1) / 2 : a.rb_max);
  } else {
    const int64_t nrb = (a.v_used + kFR - 1) / kFR;
    while (lg > 0 && (int64_t(1) << (lg - 1)) >= a.nq) --lg;  // (no empty items in a small batch)
    // several queries per item as long as every resident workgroup still
    // gets three items (16 queries of a 70,000-word vocabulary, 2160 items of
    // two: 1.24 ms a call; items of one 1.30, of eight 1.45)
    auto items = [&](int g) { return ((a.nq + (int64_t(1) << lg) - 1) >> lg) * nrb << (lg - g); };
    if (streams<MODE, SMALL>())
      while (glog < kStreamLog2 && glog < lg && items(glog + 1) >= 3 * resident) ++glog;
    total = items(glog);
  }
  if (total <= 0) return hipSuccess;
  if (!a.work_ctr) return hipErrorInvalidValue;
  const int grid = persistent_grid(fn, kThreads, 0, total);
  if (grid <= 0) return hipErrorInvalidConfiguration;
  if (streams<MODE, SMALL>() || total > grid) {
    const hipError_t e = launch_zero_ints((int*)a.work_ctr, 16, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_phase1_rows<MODE, LK, SMALL>), dim3(grid), dim3(kThreads), 0, s, a, total, lg, glog);
  return hipGetLastError();
}

template <int MODE, bool SMALL>
hipError_t launch_f32_list(const P1Args& a, int depth, hipStream_t s) {
  if (depth <= 1) return launch_f32_one<MODE, 1, SMALL>(a, s);
  if (depth <= 2) return launch_f32_one<MODE, 2, SMALL>(a, s);
  if (depth <= 4) return launch_f32_one<MODE, 4, SMALL>(a, s);
  if (depth <= 8) return launch_f32_one<MODE, 8, SMALL>(a, s);
  if (depth <= 16) return launch_f32_one<MODE, 16, SMALL>(a, s);
  if (depth <= 32) return launch_f32_one<MODE, 32, SMALL>(a, s);
  return hipErrorInvalidValue;
}

// embeddings of at most 28 dims: one slice
bool phase1_rows_small(const P1Args& a) { return a.m4 <= 7; }

template <int MODE>
hipError_t launch_f32_mode(const P1Args& a, int depth, hipStream_t s) {
  return phase1_rows_small(a) ? launch_f32_list<MODE, true>(a, depth, s) : launch_f32_list<MODE, false>(a, depth, s);
}

}  // namespace

int phase1_rows_partials(const P1Args& a, int row_hmax) {
  const int rows = phase1_rows_small(a) ? 64 : kFR;
  return (row_hmax + rows - 1) / rows;
}

hipError_t launch_phase1_rows(const P1Args& a, int mode, int depth, hipStream_t s) {
  if (mode == P1_TABLE) return launch_f32_mode<P1_TABLE>(a, depth, s);
  if (mode == P1_TABLE_FULL) return launch_f32_mode<P1_TABLE_FULL>(a, depth, s);
  if (mode == P1_PAIR && a.cand) return launch_f32_mode<P1_PAIR>(a, depth, s);
  return hipErrorInvalidValue;
}

}  // namespace lcemd
