// Phase 1 of LC-ACT (Sec. 4, Phase 1) with bfloat16 keys, table modes:
// per (vocabulary row, query) the nearest query words of Alg. 3 (and their
// capacities), selected on bfloat16 contractions and finished with float32
// distances recomputed from the float32 embeddings.
//
// Work item: one query against a block of 256 used vocabulary rows, a
// workgroup of eight waves, wave w owning rows 32w .. 32w + 31.  The
// contraction runs on the 32x32x16 bf16 MFMA with the vocabulary rows as its
// N operand (each lane reads its row's dims straight from global memory, a
// 64-dim slice ahead) and the query's words as its M operand (a slice of 64
// words staged in LDS for the eight waves, double-buffered), so that after a
// pass a lane holds 32 keys of its own row in its accumulators: words 32 t +
// 8 (r / 4) + 4 (lane / 32) + r % 4.
//
// Keys are approximate squared distances.  The bf16 rows (built at load)
// hold -2 v in their first m dims, 1 in the next three and a three-piece
// bf16 split of |v|^2 in the three after (three bf16 significands hold a
// float32 one exactly); the query form of a word holds v, the split of its
// |q|^2 and three ones.  One contraction then gives |v|^2 + |q|^2 -
// 2 <v_b, q_b> with float32 accumulation.
//
// Error band.  With e_v = v - v_b: <v,q> - <v_b,q_b> = <e_v, q> + <v_b, e_q>,
// so by Cauchy-Schwarz the key is off the exact squared distance by at
// most eps = 2 (|e_v| |q| + |v_b| |e_q|) plus the float32 accumulation of
// K + 6 terms (|e_v| is stored per row at load, rounded up).  A row keeps
// every candidate whose key is within band = 2 eps (plus the rounding of
// the packed keys) of its cut key: a word outside that band is farther,
// exactly, than every word up to the cut, so it can never be needed.
//
// Selection, in registers: packed keys (position in the 9 low bits) go 16 at
// a time through a sorting network and into the lane's sorted list, the two
// lanes of a row merge theirs at the end.  The list is the row's LK smallest
// keys; what it leaves out is no nearer than its last entry, and the row is
// redone exactly unless every used entry is provably nearer than that.
//
// Exact distances.  Every listed candidate gets a float32 dot product with
// the float32 row: the query's float32 vectors are staged through LDS W dims
// at a time, and of every RD = 64 dims (32 for queries of more than 256
// words) each of a row's two lanes sums one half over all chunks; the halves
// are added in a fixed order.  Where cancellation could bite the distance is
// taken by direct differences (identical words: exactly 0).  The list is
// re-sorted by (distance, position) and cut as Alg. 3 / the capacity bound
// say.
//
// Bound: the recompute, half of an item's time: its LDS reads (a dot product
// reads the whole float32 word, 1.2 KB at 300 dims, from rows that no order
// makes conflict-free) and its FMAs take about half of a CU's cycles each.
// Reading a second list entry's words during the first one's sums took the
// same time, with the registers for it (128 let two workgroups share a CU).
//
// Measured on ACT k = 8 tables of 300-dim words, CU cycles per query x 256
// rows.  The form before this one (rows and words both staged in LDS, keys
// inserted into LDS lists one at a time, queue merges): 76 k at 32 words,
// 88 k at 64, 110 k at 128; this one: 47 k, 51 k, 68 k (192 queries of about
// 118 words over 485 k rows: 69 ms, now 44 ms).  Workgroups of four waves and
// passes of up to 128 words, three to a CU, were slower (57 ms against 55 at
// the time, and an item of half the rows stages the same words); the row's
// dims all in registers and a tile of 32 words at a time: 68 ms.
// What is computed from the thread's index is kept from being hoisted out of
// the item and stage loops (fresh): 46 registers spilled, and a reload waits
// for every load in flight before it, the next stage's words (55 -> 44 ms;
// lists of 16 still spill 3).
#include <algorithm>

#include "internal.h"
#include "launch_sizes.h"

namespace lcemd {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

namespace {

constexpr int kBT = 512;              // threads per workgroup
constexpr int kBR = 256;              // rows per item (8 waves x 32)
constexpr int kBW = 64;               // query words per pass
constexpr int kBStride = 144;         // bytes per staged word slice (128 + 16 pad: conflict-free 16-byte reads)
constexpr int kBMaxMb = kBf16MaxDims; // bf16 row width
constexpr int kBSeg = kSegShort;      // query words per item
constexpr int kBGroupLog2 = 5;        // queries per item group (query-fastest): a row block stays in L2 for 32 items
                                      // (8: 48.3 ms, 16: 46.2, 32: 43.2, 64: 42.9 on the 192 queries above)
constexpr uint32_t kNone = 0xffffffffu;
constexpr uint32_t kPosMask = 511u;   // 9 position bits (words < 512)
// twice the largest relative rounding of a packed key: 2 * 2^(9 - 23)
constexpr float kQuant = 1.f / 8192.f;
constexpr float kGuard = 0.25f;       // cancellation guard of the float32 form
// no listed word: above every squared distance, also +inf and the NaN that
// arithmetic gives, and not a float64 NaN as the high half of one
constexpr uint32_t kNoD2 = 0x7fe00000u;

// LDS of a workgroup: a union of the contraction's word slice, the lists
// on their way to the recompute's lanes and its staged float32 words; then
// the query's words and the rows.
struct BfLds {
  unsigned char* st;   // [2][kBW][kBStride]
  uint32_t* lst;       // [kBR][LK + 1]
  float* qf;           // [h][W + 4]
  int* cid;            // [hp]
  float* cap;
  float* qn;
  int* rid;            // [kBR] each
  float* rbound;
  float* rvn;
  float* reps;
  uint32_t* rdrop;
  int* rkey;           // length and row, for the order of length
  int* rflag;          // the merged list has its cut
  int* rorder;         // rows by list length (the recompute's row of each lane pair)
};
// dims staged at a time for the recompute: what four pieces a thread hold
__host__ __device__ inline int bf_stage(int h) { return h <= 256 ? 32 : 16; }
__host__ __device__ inline int bf_words(int hmax) { return hmax + kBW; }
__host__ __device__ inline size_t bf_union(int hmax, int LK) {
  const size_t a = 2 * (size_t)kBW * kBStride, b = sizeof(uint32_t) * kBR * (LK + 1);
  const int h32 = hmax < 256 ? hmax : 256;
  const size_t c = sizeof(float) * (h32 * 36 > hmax * 20 ? h32 * 36 : hmax * 20);
  const size_t m = a > b ? (a > c ? a : c) : (b > c ? b : c);
  return (m + 15) / 16 * 16;
}
__host__ __device__ inline size_t bf_bytes(int hmax, int LK) {
  return bf_union(hmax, LK) + 12 * (size_t)bf_words(hmax) + 4 * (size_t)kBR * 8;
}
__device__ __forceinline__ BfLds bf_lds(unsigned char* base, int hmax, int LK) {
  BfLds s;
  s.st = base;
  s.lst = (uint32_t*)base;
  s.qf = (float*)base;
  // (the rows first: rkey is read 16 bytes at a time)
  int* p = (int*)(base + bf_union(hmax, LK));
  s.rid = p;
  s.rbound = (float*)(p + kBR);
  s.rvn = (float*)(p + 2 * kBR);
  s.reps = (float*)(p + 3 * kBR);
  s.rdrop = (uint32_t*)(p + 4 * kBR);
  s.rkey = p + 5 * kBR;
  s.rflag = p + 6 * kBR;
  s.rorder = p + 7 * kBR;
  p += 8 * kBR;
  const int hp = bf_words(hmax);
  s.cid = p;
  s.cap = (float*)(p + hp);
  s.qn = (float*)(p + 2 * hp);
  return s;
}

// x, as a value of its own: what is computed from it is computed where it
// stands, instead of ahead of a loop and spilled there
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ float pk_key(uint32_t k) { return __uint_as_float(k & ~kPosMask); }
__device__ __forceinline__ int pk_pos(uint32_t k) { return (int)(k & kPosMask); }

// compare-exchange of packed keys and of exact (distance, position) pairs:
// both order as unsigned 32 / 64-bit numbers, the latter (never negative)
// also as float64
__device__ __forceinline__ uint32_t kmin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t kmax(uint32_t a, uint32_t b) { return a < b ? b : a; }
__device__ __forceinline__ double kmin(double a, double b) {
  double d;
  asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double kmax(double a, double b) {
  double d;
  asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
template <typename T>
__device__ __forceinline__ void cas(T& a, T& b) {
  const T x = a, y = b;
  a = kmin(x, y);
  b = kmax(x, y);
}

// Batcher's odd-even merge sort of N (a power of two) keys
template <int N, typename T>
__device__ __forceinline__ void net_sort(T* k) {
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
__device__ __forceinline__ void net_merge(uint32_t* a, const uint32_t* b) {
#pragma unroll
  for (int i = 0; i < NB; ++i) a[LK - 1 - i] = kmin(a[LK - 1 - i], b[i]);
#pragma unroll
  for (int h = LK >> 1; h > 0; h >>= 1)
#pragma unroll
    for (int i = 0; i < LK; ++i)
      if ((i & h) == 0) cas(a[i], a[i + h]);
}

// Cut of an ascending list (Alg. 3 / Lemma 1-2): the first entry where
// k_eff entries are listed or the listed capacities reach the row's bound.
// Returns the cut entry (kNone if none).
template <int LK, bool CAPSTOP>
__device__ __forceinline__ uint32_t list_cut(const uint32_t (&a)[LK], const float* cap, int kef, float bound) {
  // the capacities of the first entries are read together (one LDS round
  // trip instead of one per entry); lists are cut within a few entries
  constexpr int kPre = LK < 8 ? LK : 8;
  float c[kPre];
#pragma unroll
  for (int i = 0; i < kPre; ++i) c[i] = (CAPSTOP && a[i] != kNone) ? cap[pk_pos(a[i])] : 0.f;
  float P = 0.f;
  uint32_t K0 = kNone;
#pragma unroll
  for (int i = 0; i < LK; ++i) {
    const bool live = K0 == kNone && a[i] != kNone;
    if (!__any(live)) break;
    if (live) {
      if (CAPSTOP) P += i < kPre ? c[i] : cap[pk_pos(a[i])];
      if (i + 1 >= kef || (CAPSTOP && P >= bound)) K0 = a[i];
    }
  }
  return K0;
}

__device__ __forceinline__ float exact_d2(const float* __restrict__ V, int m_pad, int m4, int a, int b, float an) {
  if (a == b && an < INFINITY) return 0.f;  // (an = |a|^2: a row of finite numbers against itself)
  const float4* x = (const float4*)(V + (size_t)a * m_pad);
  const float4* y = (const float4*)(V + (size_t)b * m_pad);
  float s = 0.f;
  for (int d = 0; d < m4; ++d) {
    const float4 p = x[d], q = y[d];
    const float e0 = p.x - q.x, e1 = p.y - q.y, e2 = p.z - q.z, e3 = p.w - q.w;
    s = fmaf(e0, e0, s);
    s = fmaf(e1, e1, s);
    s = fmaf(e2, e2, s);
    s = fmaf(e3, e3, s);
  }
  return s;
}

// What a thread has in flight for the contraction: the lane's row's next
// slice, and the pieces of the words' next slice that it stages.
struct BfFlight {
  const unsigned char* rptr;
  const unsigned char* wptr;
  uint4 r[4];
  uint4 w;
  __device__ __forceinline__ void words(const uint16_t* vbq, size_t rowbytes, const int* cid, int tid) {
    wptr = (const unsigned char*)vbq + (size_t)cid[tid >> 3] * rowbytes + (tid & 7) * 16;
  }
  __device__ __forceinline__ void load_rows(int sl) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = *(const uint4*)(rptr + sl * 128 + i * 16);
  }
  __device__ __forceinline__ void load_words(int sl) { w = *(const uint4*)(wptr + sl * 128); }
};

// One pass: the 64 words from c0 on, all slices, then their keys into the
// list.
template <int LK>
__device__ __forceinline__ void bf16_pass(const BfLds& sm, BfFlight& fl, uint32_t (&lst)[LK], int c0, int h, int nsl,
                                          const uint16_t* vbq, size_t rowbytes, int tid) {
  constexpr int NT = kBW / 32;
  const int lane = tid & 63, li = lane & 31, lh = lane >> 5;
  floatx16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  const bool more = c0 + kBW < h;
#pragma unroll 1
  for (int sl = 0; sl < nsl; ++sl) {
    unsigned char* st = sm.st + (sl & 1) * (kBW * kBStride);  // (last read two slices ago, before a barrier)
    *(uint4*)(st + (tid >> 3) * kBStride + (tid & 7) * 16) = fl.w;
    if (sl + 1 < nsl) {
      fl.load_words(sl + 1);
    } else if (more) {  // the next pass's first slice
      fl.words(vbq, rowbytes, sm.cid + c0 + kBW, tid);
      fl.load_words(0);
    }
    __syncthreads();
    // lane half lh supplies dims [32 lh, 32 lh + 32) of the 64-dim slice
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bf16x8 rv = *reinterpret_cast<const bf16x8*>(&fl.r[s]);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *(const bf16x8*)(st + (32 * t + li) * kBStride + lh * 64 + s * 16), rv, acc[t], 0, 0, 0);
    }
    // (into the registers just read: a second set would cost a workgroup per CU)
    if (sl + 1 < nsl) fl.load_rows(sl + 1);
    else if (more) fl.load_rows(0);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int j0 = c0 + 32 * t;
    if (j0 >= h) break;
    const int jb = j0 | (lh << 2);
    uint32_t k[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      // d2 >= 0: its bits order like the values; the 9 low bits give way to the position
      k[r] = (__float_as_uint(fmaxf(acc[t][r], 0.f)) & ~kPosMask) | (uint32_t)jb | (uint32_t)(8 * (r >> 2) + (r & 3));
    if (j0 + 32 > h) {  // words past the query's
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((jb | (8 * (r >> 2) + (r & 3))) >= h) k[r] = kNone;
    }
    net_sort<16>(k);
    net_merge<LK, 16>(lst, k);
  }
  // (an odd slice count: the next pass starts on the buffer that was read last)
  if (nsl & 1) __syncthreads();
}

// Float32 dot products of row xr's listed words (a row's two lanes, sub): of
// every RD dims lane sub takes [sub RD / 2, (sub + 1) RD / 2), in order,
// staged W dims (W / 2 of each half) at a time.  off[e]: the word's staged
// row in floats.  The row's dims are loaded a stage ahead, the words' while
// the stage before them is worked on (up to 4 pieces a thread).
template <int W, int LK>
__device__ __forceinline__ void recompute(const P1Args& a, const BfLds& sm, int h, int dims, int RD, int rid, int sub,
                                          int wlen, const int (&off)[LK], float (&dot)[LK]) {
  constexpr int WS = W + 4;    // floats per staged word
  constexpr int Q = W / 8;     // float4 of a lane's half of a stage
  constexpr int N4 = W / 4;    // float4 per staged word
  constexpr int kAhead = 4;
  const int tid = threadIdx.x;
  const int pieces = h * N4;
  const int per = RD / W;      // stages per chunk of RD dims (1, 2 or 4)
  const int nst = (dims + RD - 1) / RD * per;
  // a stage's first dim of either half
  auto dim0 = [&](int i, int half) { return i / per * RD + half * (RD / 2) + i % per * (W / 2); };
  auto put1 = [&](int f, const float4& x) {
    if (f < pieces) *(float4*)(&sm.qf[f / N4 * WS + f % N4 * 4]) = x;
  };
  float4 nx[kAhead], vn[Q];
  const float* vrow = a.V + (size_t)rid * a.m_pad;
  // (stages end within m_pad, a multiple of 64; the rows are 0 past their dims)
  auto fetch = [&](int i) {
    const int t = fresh(tid);
    const int d = dim0(i, t % N4 / Q) + 4 * (t % Q);
    int id[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) id[k] = sm.cid[min(t + k * kBT, pieces - 1) / N4];
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      nx[k] = t + k * kBT < pieces ? *(const float4*)(a.V + (size_t)id[k] * a.m_pad + d)
                                   : make_float4(0.f, 0.f, 0.f, 0.f);
    const int dr = dim0(i, sub);
#pragma unroll
    for (int q = 0; q < Q; ++q) vn[q] = *(const float4*)(vrow + dr + 4 * q);
  };
  fetch(0);
#pragma unroll 1
  for (int i = 0; i < nst; ++i) {
    __syncthreads();  // the previous stage (at first: the lists) is consumed
    const int t = fresh(tid);
#pragma unroll
    for (int k = 0; k < kAhead; ++k) put1(t + k * kBT, nx[k]);
    float4 vc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) vc[q] = vn[q];
    __syncthreads();
    if (i + 1 < nst) fetch(i + 1);
#pragma unroll
    for (int e = 0; e < LK; ++e) {
      if (e < wlen) {  // uniform (a loop exit would have off[] and dot[] indexed at run time)
        const float* qp = sm.qf + off[e] + sub * (W / 2);
        float4 qv[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) qv[q] = *(const float4*)(qp + 4 * q);
        float t = dot[e];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          t = fmaf(vc[q].x, qv[q].x, t);
          t = fmaf(vc[q].y, qv[q].y, t);
          t = fmaf(vc[q].z, qv[q].z, t);
          t = fmaf(vc[q].w, qv[q].w, t);
        }
        dot[e] = t;
      }
    }
  }
}

template <int MODE, int LK>
__device__ __forceinline__ void bf16_task(const P1Args& a, const BfLds& sm, int64_t item, int glog) {
  static_assert(LK == 16 || LK == 32, "list sizes 16 or 32");
  const int tid = fresh(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  const int li = lane & 31, lh = lane >> 5;
  constexpr bool kCapStop = MODE != P1_TABLE_FULL;

  // ---------------- item decode ----------------
  const int64_t nsb = (a.v_used + kBR - 1) / kBR;
  const int64_t qin = item & ((int64_t(1) << glog) - 1), t0 = item >> glog;
  const int64_t sb = t0 % nsb, g = t0 / nsb;
  const int64_t qi = (g << glog) + qin;
  if (qi >= a.nq) return;
  const int64_t r0 = sb * kBR;
  const int64_t b = a.q0 + qi;
  const int nrows = (int)min((int64_t)kBR, a.v_used - r0);
  const int64_t s0 = a.qptr[b];
  const int h = (int)(a.qptr[b + 1] - s0);
  if (h <= 0) return;  // padding slot of a fixed-size batch

  // one 16-byte record per row and per query word (built per call by
  // k_bf16_info): word id, bound / weight, |v|^2, |v - bf16(v)|
  const int row = 32 * wave + li;
  const bool row_ok = row < nrows;
  const float4 ri = a.rinfo[r0 + (row_ok ? row : 0)];
  for (int c = tid; c < h + kBW; c += kBT) {
    const float4 q = c < h ? a.qinfo[s0 + c] : make_float4(0.f, 0.f, 0.f, 0.f);  // (word 0 past the query's)
    sm.cid[c] = __float_as_int(q.x);
    sm.cap[c] = q.y;
    sm.qn[c] = q.z;
  }
  const float2 mx = a.qmx[qi];  // the query's largest |q|^2 and |q - bf16(q)| (k_bf16_qmax)
  const float bound = row_ok ? (MODE == P1_TABLE ? ri.y : INFINITY) : 0.f;
  float eps, band;
  {
    const float qm = sqrtf(mx.x) * 1.0001f, nv = sqrtf(ri.z) * 1.0001f;
    // |v_b| <= |v| (1 + 2^-8); K + 6 float32 accumulation steps
    eps = 2.02f * (ri.w * qm + nv * mx.y) +
          (float)(a.mb + 8) * 6.0e-8f * (ri.z + qm * qm + 2.f * nv * qm) * 1.1f + 1e-30f;
    band = 2.f * eps + kQuant * (ri.z + qm * qm + 2.f * nv * qm);
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
  __syncthreads();

  // ---------------- contraction and selection ----------------
  uint32_t lst[LK];
#pragma unroll
  for (int i = 0; i < LK; ++i) lst[i] = kNone;
  {
    const size_t rowbytes = (size_t)a.mb * 2;
    const int nsl = a.mb >> 6;  // 64-dim slices
    BfFlight fl;
    fl.rptr = (const unsigned char*)a.Vb + (size_t)__float_as_int(ri.x) * rowbytes + lh * 64;
    fl.words(a.Vbq, rowbytes, sm.cid, tid);
    fl.load_rows(0);
    fl.load_words(0);
#pragma unroll 1
    for (int c0 = 0; c0 < h; c0 += kBW) bf16_pass<LK>(sm, fl, lst, c0, h, nsl, a.Vbq, rowbytes, tid);
    __syncthreads();  // every wave is done with the word slices
  }
  {  // the row's list: merge of its two lanes
    uint32_t other[LK];
#pragma unroll
    for (int i = 0; i < LK; ++i) other[i] = (uint32_t)__shfl_xor((int)lst[i], 32);
    net_merge<LK, LK>(lst, other);
  }
  {
    const uint32_t K0 = list_cut<LK, kCapStop>(lst, sm.cap, kef, bound);
    const float lim = K0 != kNone ? pk_key(K0) * (1.f + kQuant) + band : INFINITY;
    int len = 0;
#pragma unroll
    for (int i = 0; i < LK; ++i)
      if (lst[i] != kNone && pk_key(lst[i]) <= lim) len = i + 1;
    uint32_t* L = sm.lst + row * (LK + 1);
    // both lanes hold the same list: each writes half of it
#pragma unroll
    for (int i = 0; i < LK; ++i)
      if ((i >= LK / 2) == (lh == 1)) L[i] = lst[i];
    if (lh == 0) {
      sm.rid[row] = __float_as_int(ri.x);
      sm.rbound[row] = bound;
      sm.rvn[row] = ri.z;
      sm.reps[row] = eps;
      // words left out of a full list have keys of at least its last entry
      sm.rdrop[row] = h > LK ? lst[LK - 1] : kNone;
      sm.rflag[row] = K0 != kNone ? 1 : 0;
      sm.rkey[row] = (row_ok ? len : 0) * kBR + (kBR - 1 - row);
    }
  }
  __syncthreads();

  // ---------------- exact float32 distances of the listed words ----------------
  // rows by list length, longest first (a row's rank: how many keys are
  // larger), so that the lanes of a wave have lists of similar lengths
  if (tid < kBR) {
    const int me = sm.rkey[tid];
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < kBR; i += 4) {
      const int4 o = *(const int4*)(sm.rkey + i);
      rank += (o.x > me) + (o.y > me) + (o.z > me) + (o.w > me);
    }
    sm.rorder[rank] = tid;
  }
  __syncthreads();
  const int xr = sm.rorder[tid >> 1], sub = tid & 1;
  const int len = sm.rkey[xr] / kBR, xid = sm.rid[xr];
  // the longest list of the wave bounds its (uniform) entry loop; shorter
  // lists compute on word 0 and drop the result
  const int wlen = __builtin_amdgcn_readfirstlane(len);  // (the wave's first row has its longest list)
  const int W = bf_stage(h), ws = W + 4;
  int off[LK];  // the listed words' staged rows
  float dot[LK];
#pragma unroll
  for (int e = 0; e < LK; ++e) {
    off[e] = e < len ? pk_pos(sm.lst[xr * (LK + 1) + e]) * ws : 0;
    dot[e] = 0.f;
  }
  const int dims = 4 * a.m4 <= a.m_pad ? a.m4 * 4 : a.m_pad;  // real dims rounded up to 4
  const int RD = h <= 256 ? 64 : 32;
  if (W == 32) recompute<32, LK>(a, sm, h, dims, RD, xid, sub, wlen, off, dot);
  else recompute<16, LK>(a, sm, h, dims, RD, xid, sub, wlen, off, dot);

  // ---------------- re-sort, cut, certificate, outputs ----------------
  // both lanes of a row do the same arithmetic and share the stores
  const float vn = sm.rvn[xr];
  double ex[LK];
  uint32_t need = 0;  // entries that cancellation could have hurt
#pragma unroll
  for (int e = 0; e < LK; ++e) {
    uint32_t bits = kNoD2;
    const int pos = W == 32 ? (int)((uint32_t)off[e] / 36u) : (int)((uint32_t)off[e] / 20u);
    if (e < wlen) {
      const float full = dot[e] + __shfl_xor(dot[e], 1);  // (the sum of the halves, either way round)
      const float sq = vn + sm.qn[pos];
      const float d2 = sq - 2.f * full;
      if (e < len) {
        bits = __float_as_uint(d2);
        if (!(d2 >= kGuard * sq)) need |= 1u << e;
      }
    }
    ex[e] = __hiloint2double((int)bits, pos);
  }
  // (rare: one copy of the loop over the dims, entry by entry)
  while (need) {
    const int e = __ffs(need) - 1;
    need &= need - 1;
    int pos = 0;
#pragma unroll
    for (int i = 0; i < LK; ++i) pos = i == e ? __double2loint(ex[i]) : pos;
    const float d2 = exact_d2(a.V, a.m_pad, a.m4, xid, sm.cid[pos], vn);
#pragma unroll
    for (int i = 0; i < LK; ++i) ex[i] = i == e ? __hiloint2double(__float_as_int(d2), pos) : ex[i];
  }
  net_sort<LK>(ex);
  if (xr >= nrows) return;  // (no barrier past this point)
  const float xb = sm.rbound[xr];
  float z[LK], w[LK];
  int pos[LK];
  int D = 0;
  bool covered = false;
  float Pc = 0.f, last = 0.f;
#pragma unroll
  for (int l = 0; l < LK; ++l) {
    z[l] = 0.f;
    w[l] = 0.f;
    pos[l] = 0;
    const uint32_t bits = (uint32_t)__double2hiint(ex[l]);
    const bool live = !covered && bits != kNoD2;
    if (!__any(live)) continue;
    if (live) {
      const float d2 = __uint_as_float(bits);
      pos[l] = __double2loint(ex[l]);
      z[l] = sqrtf(fmaxf(d2, 0.f));
      w[l] = sm.cap[pos[l]];
      last = d2;
      ++D;
      Pc += w[l];
      covered = D >= kef;
      if (kCapStop) covered = covered || Pc >= xb || (a.method == LCEMD_OMR && l == 0 && d2 != 0.f);
    }
  }
  // the merge cut this list (k_eff or capacity reached in key order); a
  // shortfall after the exact re-sort is a rounding residue of the
  // capacity sum, which the last entry absorbs
  // (a row without entries, whose band has no number, is written by the redo)
  if (!covered && sm.rflag[xr]) covered = D > 0;
  const int64_t r = r0 + xr;
  if (sub == 0) {
    bool redo = !covered && D < h;
    // a word left out of a full list has an exact squared distance of at
    // least its key minus eps: every used entry must be nearer
    const uint32_t dr = sm.rdrop[xr];
    if (dr != kNone && D > 0 && !(last < pk_key(dr) - sm.reps[xr])) redo = true;
    if (redo) {
      bool listed = false;
      if (a.fix_list) {
        const int slot = atomicAdd(a.fix_count, 1);
        listed = slot < a.fix_cap;
        if (listed) a.fix_list[slot] = qi * a.v_used + r;
      }
      if (!listed && a.overflow) a.overflow[0] = 1;
    }
  }
  if constexpr (MODE == P1_TABLE) {
    if (D > a.KT && a.overflow) a.overflow[0] = 1;
#pragma unroll
    for (int l = 0; l < LK; l += 2) {
      if (((l >> 1) & 1) == sub && l < D && l < a.KT) {
        const bool two = l + 1 < D && l + 1 < a.KT;
        *zw_pair(a.ZW, a.zw_nq, a.KT, qi, r, l >> 1) =
            make_float4(z[l], l == D - 1 ? INFINITY : w[l], two ? z[l + 1] : 0.f,
                        two ? (l + 1 == D - 1 ? INFINITY : w[l + 1]) : 0.f);
      }
    }
  } else {
    const int64_t o0 = (qi * a.v_used + r) * (int64_t)a.k;
#pragma unroll
    for (int l = 0; l < LK; ++l) {
      if ((l & 1) == sub && l < a.k) {
        const bool in = l < D;
        a.S[o0 + l] = in ? pos[l] : -1;
        a.Z[o0 + l] = in ? z[l] : 0.f;
        a.W[o0 + l] = in ? w[l] : 0.f;
      }
    }
  }
}

// Persistent grid: as many workgroups as stay resident pull items from the
// counter of their XCD (workgroup i runs on XCD i % 8), which walks a
// contiguous eighth of the items; the counter is read one item ahead.  Every
// workgroup exits once its counter passes its range.
template <int MODE, int LK>
__global__ __launch_bounds__(kBT, LK == 16 ? 4 : 2) void k_phase1_bf16(P1Args a, int64_t total, int hmax, int glog) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int64_t s_item;
  const BfLds sm = bf_lds(smem_raw, hmax, LK);
  // no more items than workgroups: one each, no counter (and none to clear)
  const bool once = total <= (int64_t)gridDim.x;
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
    bf16_task<MODE, LK>(a, sm, item, glog);
    if (once) break;
  }
}

template <int MODE, int LK>
hipError_t launch_bf16_one(const P1Args& a, int seg_hmax, hipStream_t s) {
  const int hmax = bf16_layout_words(seg_hmax, kBSeg);
  const size_t shmem = bf_bytes(hmax, LK);
  const void* fn = (const void*)k_phase1_bf16<MODE, LK>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bf_bytes(kBSeg, LK));
  if (e != hipSuccess) return e;
  const int64_t nsb = (a.v_used + kBR - 1) / kBR;
  // (a smaller batch has smaller groups: every empty item costs its workgroup a
  // counter's round trip, 31 of 32 for one query over 70 k rows: 0.20 -> 0.07 ms)
  int glog = kBGroupLog2;
  while (glog > 0 && (int64_t(1) << (glog - 1)) >= a.nq) --glog;
  const int64_t total = ((a.nq + (int64_t(1) << glog) - 1) >> glog) * nsb << glog;
  if (total <= 0) return hipSuccess;
  if (!a.work_ctr) return hipErrorInvalidValue;
  const int grid = persistent_grid(fn, kBT, shmem, total);
  if (grid <= 0) return hipErrorInvalidConfiguration;
  if (total > grid) {
    e = launch_zero_ints((int*)a.work_ctr, 16, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_phase1_bf16<MODE, LK>), dim3(grid), dim3(kBT), shmem, s, a, total, hmax, glog);
  return hipGetLastError();
}

// Row and query-word records for the bf16 kernel: rinfo[r] = (word id bits,
// largest database weight, |v|^2, |v - bf16(v)|) for the used words of the
// rows, qinfo[i] = (word id bits, weight, |v|^2, |v - bf16(v)|) for the
// non-zeros i of the launch's queries (qptr[q0] <= i < qptr[q0 + nq]).
__global__ __launch_bounds__(kThreads) void k_bf16_info(P1Args a) {
  const int64_t qlo = a.qptr[a.q0], qhi = a.qptr[a.q0 + a.nq];
  const int64_t n = max(a.v_used, qhi - qlo);
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    if (i < a.v_used) {
      const int w = a.used[i];
      a.rinfo[i] = make_float4(__int_as_float(w), a.xmax ? a.xmax[i] : INFINITY, a.vnorm[w], a.vres[w]);
    }
    if (i < qhi - qlo) {
      const int64_t j = qlo + i;
      const int w = a.qcol[j];
      a.qinfo[j] = make_float4(__int_as_float(w), a.qval[j], a.vnorm[w], a.vres[w]);
    }
  }
}

// Per query of the launch, the largest |q|^2 and |q - bf16(q)| over its
// words (from qinfo): one wave per query.
__global__ __launch_bounds__(kThreads) void k_bf16_qmax(P1Args a) {
  const int64_t qi = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (qi >= a.nq) return;
  const int64_t s0 = a.qptr[a.q0 + qi], s1 = a.qptr[a.q0 + qi + 1];
  float mq = 0.f, me = 0.f;
  for (int64_t j = s0 + lane; j < s1; j += 64) {
    const float4 q = a.qinfo[j];
    mq = fmaxf(mq, q.z);
    me = fmaxf(me, q.w);
  }
  for (int o = 32; o > 0; o >>= 1) {
    mq = fmaxf(mq, __shfl_xor(mq, o));
    me = fmaxf(me, __shfl_xor(me, o));
  }
  if (lane == 0) a.qmx[qi] = make_float2(mq, me);
}

}  // namespace

bool phase1_bf16_fits(int mb, int seg_hmax, int depth) {
  return mb <= kBMaxMb && mb % 64 == 0 && seg_hmax <= kBSeg && depth + 8 <= 32;
}

hipError_t launch_phase1_bf16(const P1Args& a, int mode, int depth, int seg_hmax, hipStream_t s) {
  if (!a.Vb || !a.Vbq || !a.vres || !a.rinfo || !a.qinfo || !a.qmx || a.mb % 64 != 0 || a.mb > kBMaxMb ||
      a.mb < a.m + 6 || seg_hmax < 1 || seg_hmax > kBSeg)
    return hipErrorInvalidValue;
  {
    // grid-stride over the rows and the launch's query words (at most qnnz)
    const int64_t n = std::max<int64_t>(a.v_used, a.qnnz);
    const unsigned g = (unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, 8192);
    hipLaunchKernelGGL(k_bf16_info, dim3(g), dim3(kThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.nq > 0) {
      hipLaunchKernelGGL(k_bf16_qmax, dim3((unsigned)((a.nq + kThreads / 64 - 1) / (kThreads / 64))), dim3(kThreads),
                         0, s, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  const bool small = depth + 8 <= 16;
  if (mode == P1_TABLE)
    return small ? launch_bf16_one<P1_TABLE, 16>(a, seg_hmax, s) : launch_bf16_one<P1_TABLE, 32>(a, seg_hmax, s);
  if (mode == P1_TABLE_FULL)
    return small ? launch_bf16_one<P1_TABLE_FULL, 16>(a, seg_hmax, s)
                 : launch_bf16_one<P1_TABLE_FULL, 32>(a, seg_hmax, s);
  return hipErrorInvalidValue;
}

}  // namespace lcemd
