// Phase 1 of LC-ACT (Sec. 4, Phase 1) with fp8 keys, table modes, lists of up
// to 32 entries: 128 rows per workgroup and up to 128 columns per MFMA pass;
// and the exact redo of single table rows (every precision).
//
// Contraction: wave w owns rows [32w, 32w+32).  Its row operand (32 rows x
// one 128-byte slice of dims) is read straight from global memory into
// registers -- no other wave needs it -- while the column slice (128
// columns) is staged once in LDS for all four waves.  Each wave keeps four
// 32x32 accumulators (one per 32-column tile) and issues them interleaved.
// The next slice is prefetched into registers during the MFMAs, so a slice
// costs one LDS store and two barriers.
//
// Selection: after a pass the keys |c|^2 - 2 <v, c> go to LDS 64 columns at
// a time and two lanes per row merge them into the row's sorted candidate
// list (packed key | position; position breaks ties; each lane first sorts
// its 32 keys in registers and the merge takes from their heads), cut at
// k_eff = min(k, h) (Alg. 3; 1 for RWMD, 2 for OMR) or as soon as the listed
// capacities reach the row's bound (Lemma 1/2: no transfer of at most that
// much mass passes this point).
//
// Exact distances: the list keeps, past the cut, every candidate within a
// statistical band of the cut key.  All listed candidates then get float32
// distances -- |v|^2 + |c|^2 - 2<v, c> with the dot product accumulated in
// float32 over the original vectors (staged through LDS a chunk of dims at a
// time), or by direct differences where cancellation could bite -- and are
// re-sorted and cut again.
#include <algorithm>

#include "internal.h"

namespace lcemd {

typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int kWR = 128;        // rows per workgroup
constexpr int kWC = 128;        // columns per MFMA pass
constexpr int kStride = 144;    // bytes per staged column slice (128 + 16 pad)
constexpr int kCK = 66;         // floats per key row (64 columns + 2 pad)
constexpr int kQSCap = kWR * kCK;  // floats of the staging area (the key buffer's size)
constexpr int kSeg = kSegShort;            // segment words held in LDS
constexpr int kSegLong = LCEMD_MAX_HIST;   // longest segment of the exact redo
constexpr int kWGroupLog2 = 3;  // queries per item group (table modes; 32 was 3 % slower at 1M words)
constexpr float kGuardW = 0.25f;
// fp8 (e4m3, 3 mantissa bits): a statistical band, not a worst-case one --
// about six standard deviations of the key error of a few-hundred-term dot
// product with independent relative rounding errors of at most 2^-4
constexpr float kBandFP8 = 0.04f;

__device__ __forceinline__ uint32_t w_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ uint64_t w_pack(float f, uint32_t pos) {
  return ((uint64_t)w_bits(f) << 32) | (uint64_t)pos;
}
__device__ __forceinline__ float w_unpack(uint64_t k) {
  const uint32_t o = (uint32_t)(k >> 32);
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
// Selection keys: the key's 9 low bits give way to the position (segments of
// up to 512 words), one 32-bit word, rounded down in value by at most 2^-14
// of the key's magnitude; lists keep every entry within twice that band past
// their cut and are re-sorted afterwards by the recomputed distances.
constexpr uint32_t kWNone = 0xffffffffu;
constexpr uint32_t kWPos = 511u;
constexpr float kWRound = 1.f / 8192.f;  // twice the largest relative rounding of a key
__device__ __forceinline__ uint32_t wk_pack(float f, uint32_t pos) { return (w_bits(f) & ~kWPos) | pos; }
__device__ __forceinline__ float wk_key(uint32_t k) {
  const uint32_t o = k & ~kWPos;
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
__device__ __forceinline__ uint32_t wk_pos(uint32_t k) { return k & kWPos; }

// Squared distance by direct differences over the m4 float4 groups that
// hold the real dims (the zero padding would add exact zeros).
__device__ __forceinline__ float w_exact_d2(const float* __restrict__ V, int m_pad, int m4, int a, int b, float an) {
  if (a == b && an < INFINITY) return 0.f;  // (an = |a|^2: a row of finite numbers against itself)
  const float4* x = (const float4*)(V + (size_t)a * m_pad);
  const float4* y = (const float4*)(V + (size_t)b * m_pad);
  float s = 0.f;
  const int n4 = m4;
  for (int d = 0; d < n4; ++d) {
    const float4 p = x[d], q = y[d];
    const float e0 = p.x - q.x, e1 = p.y - q.y, e2 = p.z - q.z, e3 = p.w - q.w;
    s = fmaf(e0, e0, s);
    s = fmaf(e1, e1, s);
    s = fmaf(e2, e2, s);
    s = fmaf(e3, e3, s);
  }
  return s;
}

// One staged slice on NT 32-column tiles (NT fixed at compile time so the
// MFMAs issue back to back without branches).
template <int NT>
__device__ __forceinline__ void slice_fp8(floatx16 (&acc)[4], const uint4 (&a_cur)[4],
                                          const unsigned char* st, int li, int lh) {
  // lane half lh supplies dims [64 lh + 8 s, +8) of the 128-dim slice
  const long* ap = reinterpret_cast<const long*>(a_cur);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    long bv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) bv[t] = *(const long*)(st + (32 * t + li) * kStride + lh * 64 + s * 8);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(ap[s], bv[t], acc[t], 0, 0, 0);
  }
}

__device__ __forceinline__ void slice_mfma(int ntile, floatx16 (&acc)[4], const uint4 (&a_cur)[4],
                                           const unsigned char* st, int li, int lh) {
  switch (ntile) {
    case 1: slice_fp8<1>(acc, a_cur, st, li, lh); break;
    case 2: slice_fp8<2>(acc, a_cur, st, li, lh); break;
    case 3: slice_fp8<3>(acc, a_cur, st, li, lh); break;
    default: slice_fp8<4>(acc, a_cur, st, li, lh); break;
  }
}

template <int KL>
struct WideSmem {
  static constexpr int KLS = KL + 1;  // list row stride (spreads rows over banks)
  union {
    unsigned char st[kWC * kStride];  // staged column slice
    float ck[kWR * kCK];              // keys of 64 columns of a pass
    float qs[kQSCap];  // segment vectors, a chunk of dims (exact recompute)
    float zb[kWR * KLS];              // exact squared distances of the lists
  } u;
  uint32_t lst[2][kWR * KLS];
  int cid[kSeg];
  float cap[kSeg];
  float qn[kSeg];
  int rid[kWR];
  float rbound[kWR];
  float rvn[kWR];
  int rlen[kWR];
  float rdrop[kWR];  // smallest key dropped because the list was full
  int rcut[kWR];     // the last merge reached k_eff or the row's bound
  float qmax;
  float rsc[kWR];   // fp8 row scales
  float csc[kSeg];  // fp8 column scales
};

// Float32 dot products <v_row, c_pos> of a thread's listed candidates
// (ex[e] for list entry sub + 2e), D dims at a time: the row's D dims are
// loaded into registers before the barrier, the segment's vectors are
// staged in LDS (row stride D + 4 floats).  Dims are accumulated in order.
template <int D, int KH>
__device__ __forceinline__ void wide_dots(float (&ex)[KH], const int (&ps)[KH], int len, int sub,
                                          bool row_ok, const float* __restrict__ vr,
                                          const P1Args& a, float* qs, const int* cid, int h,
                                          int tid) {
  constexpr int D4 = D / 4, QS = D + 4;
  for (int d0 = 0; d0 < a.m_pad; d0 += D) {
    float4 v[D4];
#pragma unroll
    for (int q = 0; q < D4; ++q) v[q] = row_ok ? *(const float4*)(vr + d0 + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    for (int f = tid; f < h * D4; f += kThreads) {
      const int c = f / D4, q = f % D4;
      *(float4*)(&qs[c * QS + q * 4]) = *(const float4*)(a.V + (size_t)cid[c] * a.m_pad + d0 + q * 4);
    }
    __syncthreads();
    if (row_ok) {
#pragma unroll
      for (int e = 0; e < KH; ++e) {
        if (sub + 2 * e < len) {
          const float* cp = &qs[ps[e] * QS];
          float s = ex[e];
#pragma unroll
          for (int q = 0; q < D4; ++q) {
            const float4 c = *(const float4*)(cp + 4 * q);
            s = fmaf(v[q].x, c.x, s);
            s = fmaf(v[q].y, c.y, s);
            s = fmaf(v[q].z, c.z, s);
            s = fmaf(v[q].w, c.w, s);
          }
          ex[e] = s;
        }
      }
    }
  }
}

}  // namespace

// One work item: (query, 128-row block).  Returns early (uniformly) for empty
// items.
template <int MODE, int KL>
__device__ __forceinline__ void wide_task(const P1Args& a, unsigned char* smem_raw, int64_t item) {
  using Sm = WideSmem<KL>;
  constexpr int KLS = Sm::KLS;
  Sm& sm = *reinterpret_cast<Sm*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // ---------------- task decode ----------------
  int nrows = 0, h = 0;
  int64_t out_row0 = 0;
  {
    // items run query-fastest within a group of queries, then row
    // block, then group: an XCD's contiguous range of items keeps a group's
    // query vectors and a row block's vectors in its L2
    const int64_t nrb = (a.v_used + kWR - 1) / kWR;
    const int64_t work = item;
    constexpr int lg = kWGroupLog2;
    const int64_t qin = work & ((int64_t(1) << lg) - 1), t = work >> lg;
    const int64_t rblk = t % nrb, g = t / nrb;
    const int64_t qi = (g << lg) + qin;
    if (qi >= a.nq) return;
    const int64_t r0 = rblk * kWR;
    const int64_t b = a.q0 + qi;
    nrows = (int)min((int64_t)kWR, a.v_used - r0);
    out_row0 = qi * a.v_used + r0;
    if (tid < kWR) {
      const bool ok = tid < nrows;
      const int w = ok ? a.used[r0 + tid] : 0;
      sm.rid[tid] = w;
      sm.rbound[tid] = ok ? (MODE == P1_TABLE ? a.xmax[r0 + tid] : INFINITY) : 0.f;
      sm.rvn[tid] = a.vnorm[w];
      sm.rsc[tid] = a.vscale[w];
      sm.rlen[tid] = 0;
      sm.rdrop[tid] = INFINITY;
    }
    const int64_t s0 = a.qptr[b];
    h = (int)(a.qptr[b + 1] - s0);
    if (h <= 0) return;  // padding slot of a fixed-size batch
    for (int c = tid; c < h; c += kThreads) {
      const int w = a.qcol[s0 + c];
      sm.cid[c] = w;
      sm.cap[c] = a.qval[s0 + c];
      sm.qn[c] = a.vnorm[w];
      sm.csc[c] = a.vscale[w];
    }
  }
  if (tid == 0) sm.qmax = 0.f;
  __syncthreads();
  if (tid < 64) {
    float mx = 0.f;
    for (int c = tid; c < h; c += 64) mx = fmaxf(mx, sm.qn[c]);
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if (tid == 0) sm.qmax = sqrtf(mx);
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
  constexpr bool kCapStop = MODE != P1_TABLE_FULL;

  // ---------------- contraction ----------------
  const unsigned char* base = a.V8;
  const size_t rowbytes = (size_t)a.m8;
  // 128-byte slices that hold real dims (the zero padding past them would
  // add exact zeros)
  const int nsl = min((int)(rowbytes / 128), (4 * a.m4 + 127) / 128);
  const int li = lane & 31, lh = lane >> 5;
  const int arow = 32 * wave + li;
  const bool arow_ok = arow < nrows;
  const unsigned char* aptr = base + (size_t)sm.rid[arow] * rowbytes + lh * 64;

  uint4 a_cur[4], a_nxt[4], b_nxt[4];
  auto load_a = [&](int sl) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a_nxt[i] = arow_ok ? *(const uint4*)(aptr + sl * 128 + i * 16) : make_uint4(0, 0, 0, 0);
  };
  // column operand: the 4 (column, 16-byte piece) addresses this thread
  // stages are fixed for a pass; only the slice offset moves
  const unsigned char* bptr[4];
  auto set_b = [&](int c0) {
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int f = tid + it * kThreads;
      const int cc = c0 + (f >> 3);
      bptr[it] = cc < h ? base + (size_t)sm.cid[cc] * rowbytes + (f & 7) * 16 : nullptr;
    }
  };
  auto load_b = [&](int sl) {
#pragma unroll
    for (int it = 0; it < 4; ++it)
      b_nxt[it] = bptr[it] ? *(const uint4*)(bptr[it] + sl * 128) : make_uint4(0, 0, 0, 0);
  };

  const int row = tid >> 1, sub = tid & 1;
  const bool row_ok = row < nrows;
  const float bound = row_ok ? sm.rbound[row] : 0.f;
  int par = 0;

  load_a(0);
  set_b(0);
  load_b(0);
  for (int c0 = 0; c0 < h; c0 += kWC) {
    const int ntile = min(4, (h - c0 + 31) >> 5);
    floatx16 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    for (int sl = 0; sl < nsl; ++sl) {
      __syncthreads();
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int f = tid + it * kThreads;
        *(uint4*)(sm.u.st + (f >> 3) * kStride + (f & 7) * 16) = b_nxt[it];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) a_cur[i] = a_nxt[i];
      __syncthreads();
      if (sl + 1 < nsl) {
        load_a(sl + 1);
        load_b(sl + 1);
      } else if (c0 + kWC < h) {
        load_a(0);
        set_b(c0 + kWC);
        load_b(0);
      }
      slice_mfma(ntile, acc, a_cur, sm.u.st, li, lh);
    }

    // ---- selection: 64 columns at a time ----
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int cb = c0 + 64 * half;
      if (cb >= h) break;
      __syncthreads();
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const int t = 2 * half + tt;
        const int c = cb + 32 * tt + li;
        const float qc = c < h ? sm.qn[c] : 0.f;
        const float csc = c < h ? sm.csc[c] : 1.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = 32 * wave + 8 * (r >> 2) + 4 * lh + (r & 3);
          sm.u.ck[i * kCK + 32 * tt + li] = qc - 2.f * (sm.rsc[i] * csc) * acc[t][r];
        }
      }
      __syncthreads();
      // this thread's 32 contiguous columns, read without branches (the
      // buffer is fully allocated; columns past h are masked afterwards)
      uint32_t kk[32];
      const float2* krow = (const float2*)&sm.u.ck[row * kCK + 32 * sub];
#pragma unroll
      for (int j2 = 0; j2 < 16; ++j2) {
        const float2 kv = krow[j2];
        const int c = cb + 32 * sub + 2 * j2;
        const uint32_t m0 = (row_ok && c < h) ? 0u : kWNone;
        const uint32_t m1 = (row_ok && c + 1 < h) ? 0u : kWNone;
        kk[2 * j2] = wk_pack(kv.x, (uint32_t)c) | m0;
        kk[2 * j2 + 1] = wk_pack(kv.y, (uint32_t)(c + 1)) | m1;
      }
      // the thread's 32 keys are sorted once (bitonic network in registers)
      // and the merge takes from their head
#pragma unroll
      for (int kb = 2; kb <= 32; kb <<= 1) {
#pragma unroll
        for (int jb = kb >> 1; jb > 0; jb >>= 1) {
#pragma unroll
          for (int i = 0; i < 32; ++i) {
            const int l2 = i ^ jb;
            if (l2 > i) {
              const uint32_t x = kk[i], y = kk[l2];
              const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
              const bool up = (i & kb) == 0;
              kk[i] = up ? lo : hi;
              kk[l2] = up ? hi : lo;
            }
          }
        }
      }
      const uint32_t* cur = &sm.lst[par][row * KLS];
      uint32_t* nxt = &sm.lst[par ^ 1][row * KLS];
      const int len = row_ok ? sm.rlen[row] : 0;
      // approximate keys: the error band plus the rounding of 32-bit keys
      const float band = kBandFP8 * sqrtf(sm.rvn[row]) * sm.qmax +
                         kWRound * (sm.qmax * sm.qmax + 2.f * sqrtf(sm.rvn[row]) * sm.qmax);
      int ptr = 0, w = 0;
      float P = 0.f, K0 = 0.f;
      bool cut = false;
      bool act = row_ok;
      while (__any(act)) {
        const uint32_t mine = act ? kk[0] : kWNone;
        const uint32_t o = (uint32_t)__shfl_xor((int)mine, 1);
        const uint32_t best = o < mine ? o : mine;
        if (act) {
          const uint32_t lc = ptr < len ? cur[ptr] : kWNone;
          const uint32_t take = lc < best ? lc : best;
          if (take == kWNone) {
            act = false;
          } else if (cut && wk_key(take) > K0 + band) {
            act = false;
          } else if (w >= KL) {
            // the list is full: remember the smallest key left out; the
            // final lists are certified against it after the exact re-sort
            act = false;
            if (sub == 0) sm.rdrop[row] = fminf(sm.rdrop[row], wk_key(take));
          } else {
            if (lc < best) {
              ++ptr;
            } else if (mine == best) {  // this thread's head was taken
#pragma unroll
              for (int j = 0; j < 31; ++j) kk[j] = kk[j + 1];
              kk[31] = kWNone;
            }
            if (sub == 0) nxt[w] = take;
            ++w;
            if (!cut) {
              P += sm.cap[wk_pos(take)];
              if (w >= kef || (kCapStop && P >= bound)) {
                cut = true;
                K0 = wk_key(take);
              }
            }
          }
        }
      }
      __syncthreads();
      if (sub == 0 && row_ok) {
        sm.rlen[row] = w;
        sm.rcut[row] = cut ? 1 : 0;
      }
      par ^= 1;
    }
  }
  __syncthreads();

  // ---------------- exact distances of the final lists ----------------
  const int len = row_ok ? sm.rlen[row] : 0;
  const auto* L = &sm.lst[par][row * KLS];
  {
    constexpr int KH = (KL + 1) / 2;
    float ex[KH];
    int ps[KH];
#pragma unroll
    for (int e = 0; e < KH; ++e) {
      ex[e] = 0.f;
      const int l = sub + 2 * e;
      ps[e] = l < len ? (int)wk_pos(L[l]) : 0;
    }
    const float* vr = a.V + (size_t)sm.rid[row] * a.m_pad;
    // chunks of D dims of all h segment vectors per LDS pass, as wide as
    // the staging area allows (fewer passes and barriers)
    if (h * 68 <= kQSCap && a.m_pad % 64 == 0)
      wide_dots<64, KH>(ex, ps, len, sub, row_ok, vr, a, sm.u.qs, sm.cid, h, tid);
    else if (h * 36 <= kQSCap && a.m_pad % 32 == 0)
      wide_dots<32, KH>(ex, ps, len, sub, row_ok, vr, a, sm.u.qs, sm.cid, h, tid);
    else if (h * 20 <= kQSCap && a.m_pad % 16 == 0)
      wide_dots<16, KH>(ex, ps, len, sub, row_ok, vr, a, sm.u.qs, sm.cid, h, tid);
    else
      wide_dots<8, KH>(ex, ps, len, sub, row_ok, vr, a, sm.u.qs, sm.cid, h, tid);
    // squared distances from the float32 dot products; where cancellation
    // could bite, by direct differences (as for float32 keys)
#pragma unroll
    for (int e = 0; e < KH; ++e) {
      if (row_ok && sub + 2 * e < len) {
        const float qn = sm.qn[ps[e]];
        float d2 = (sm.rvn[row] + qn) - 2.f * ex[e];
        if (!(d2 >= kGuardW * (sm.rvn[row] + qn)))
          d2 = w_exact_d2(a.V, a.m_pad, a.m4, sm.rid[row], sm.cid[ps[e]], sm.rvn[row]);
        ex[e] = d2;
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < KH; ++e) {
      const int l = sub + 2 * e;
      if (l < len) sm.u.zb[row * KLS + l] = ex[e];
    }
  }
  __syncthreads();

  if (sub == 0 && row_ok) {
    auto* Lw = &sm.lst[par][row * KLS];
    float* Z2 = &sm.u.zb[row * KLS];
    {
      // exact re-sort by (squared distance, position); the list then holds
      // positions
      for (int i = 0; i < len; ++i) Lw[i] = wk_pos(Lw[i]);
      for (int i = 1; i < len; ++i) {
        const uint64_t e = w_pack(Z2[i], (uint32_t)Lw[i]);
        int j = i - 1;
        while (j >= 0 && w_pack(Z2[j], (uint32_t)Lw[j]) > e) {
          Lw[j + 1] = Lw[j];
          Z2[j + 1] = Z2[j];
          --j;
        }
        Lw[j + 1] = (uint32_t)e;
        Z2[j + 1] = w_unpack(e);
      }
    }
    int D = 0;
    bool covered = false;
    {
      float Pc = 0.f;
      for (int l = 0; l < len; ++l) {
        ++D;
        Pc += sm.cap[(uint32_t)Lw[l]];
        if (D >= kef) { covered = true; break; }
        if (kCapStop) {
          if (Pc >= bound) { covered = true; break; }
          if (a.method == LCEMD_OMR && l == 0 && Z2[0] != 0.f) { covered = true; break; }
        }
      }
    }
    // the merge cut this list (k_eff or capacity reached in key order); a
    // shortfall after the exact re-sort is a rounding residue of the
    // capacity sum, which the last entry absorbs
    if (!covered && sm.rcut[row]) covered = true;
    // rows redone exactly by k_fix_rows (while their list has
    // room; otherwise the launch reports overflow): a list that ran out
    // before the row's bound was covered (an ICT row deeper than the list;
    // the table may hold up to KT entries), or a cut that is not certified
    const bool can_redo = a.fix_list != nullptr;
    bool redo = false;
    if (!covered && D < h) {
      if (can_redo) redo = true;
      else if (a.overflow) a.overflow[0] = 1;
    }
    // a candidate left out of a full list has a key >= rdrop - half a band
    // (fp8 keys): the used entries must all be nearer
    if (D > 0 && sm.rdrop[row] < INFINITY && a.overflow) {
      const float half_band = 0.5f * kBandFP8 * sqrtf(sm.rvn[row]) * sm.qmax;
      const float last_key = Z2[D - 1] - sm.rvn[row];
      const bool certified = last_key < sm.rdrop[row] - half_band - 1e-6f * (sm.rvn[row] + sm.qmax * sm.qmax);
      if (!certified) {
        if (can_redo) redo = true;
        else a.overflow[0] = 1;
      }
    }
    if (redo) {
      const int slot = atomicAdd(a.fix_count, 1);
      if (slot < a.fix_cap) a.fix_list[slot] = out_row0 + row;
      else if (a.overflow) a.overflow[0] = 1;
    }
    if constexpr (MODE == P1_TABLE) {
      const int64_t flat = out_row0 + row;
      zw_write_row(a.ZW, a.zw_nq, a.KT, flat / a.v_used, flat % a.v_used, D,
                   [&](int l) { return sqrtf(fmaxf(Z2[l], 0.f)); },
                   [&](int l) { return l == D - 1 ? INFINITY : sm.cap[(uint32_t)Lw[l]]; });
      if (D > a.KT && a.overflow) a.overflow[0] = 1;
    } else {
      const int64_t o0 = (out_row0 + row) * (int64_t)a.k;
      for (int l = 0; l < a.k; ++l) {
        if (l < D) {
          const int pos = (int)(uint32_t)Lw[l];
          a.S[o0 + l] = pos;
          a.Z[o0 + l] = sqrtf(fmaxf(Z2[l], 0.f));
          a.W[o0 + l] = sm.cap[pos];
        } else {
          a.S[o0 + l] = -1;
          a.Z[o0 + l] = 0.f;
          a.W[o0 + l] = 0.f;
        }
      }
    }
  }
}

// Persistent grid: as many workgroups as stay resident, each pulling items
// from the counter of its XCD (workgroup i runs on XCD i % 8), which walks a
// contiguous eighth of the items.  No workgroup waits on another; each
// exits once its counter passes the end of its range.
template <int MODE, int KL>
__global__ __launch_bounds__(kThreads, 2) void k_phase1_wide(P1Args a, int64_t total) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int64_t s_item;
  const int xcd = blockIdx.x & 7;
  const int64_t lo = total * xcd / 8, hi = total * (xcd + 1) / 8;
  while (true) {
    __syncthreads();  // the previous item is done with LDS and s_item
    if (threadIdx.x == 0) s_item = lo + (int64_t)atomicAdd(&a.work_ctr[xcd], 1ull);
    __syncthreads();
    const int64_t item = s_item;
    if (item >= hi) break;
    wide_task<MODE, KL>(a, smem_raw, item);
  }
}

template <int MODE, int KL>
static hipError_t launch_wide_one(const P1Args& a, hipStream_t s) {
  const size_t shmem = sizeof(WideSmem<KL>);
  const void* fn = (const void*)k_phase1_wide<MODE, KL>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
  if (e != hipSuccess) return e;
  const int64_t nrb = (a.v_used + kWR - 1) / kWR;
  const int64_t gw = int64_t(1) << kWGroupLog2;
  const int64_t total = (a.nq + gw - 1) / gw * nrb * gw;
  if (total <= 0) return hipSuccess;
  if (!a.work_ctr) return hipErrorInvalidValue;
  e = launch_zero_ints((int*)a.work_ctr, 16, s);
  if (e != hipSuccess) return e;
  const int grid = persistent_grid(fn, kThreads, shmem, total);
  if (grid <= 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((k_phase1_wide<MODE, KL>), dim3(grid), dim3(kThreads), shmem, s, a, total);
  return hipGetLastError();
}

template <int MODE>
static hipError_t launch_wide_mode(const P1Args& a, int KL, hipStream_t s) {
  if (KL <= 16) return launch_wide_one<MODE, 16>(a, s);  // (depth + 8 entries)
  if (KL <= 32) return launch_wide_one<MODE, 32>(a, s);
  return hipErrorInvalidValue;
}

// Exact redo of single table rows (rows whose selection certificate
// failed): one wave per row computes float32 squared distances to all of the
// query's words by direct differences (16 columns per lane in registers),
// then takes them in ascending (distance, position) order by repeated wave
// minimum -- at most KT + 1 of them -- with the same cut and outputs as the
// table modes.
template <int MODE>
__global__ __launch_bounds__(kThreads) void k_fix_rows(P1Args a, const int64_t* __restrict__ list) {
  constexpr int kCols = kSegLong / 64;  // columns per lane
  constexpr int kTake = 64;             // entries a row can take; deeper rows are flagged as overflow
  __shared__ uint64_t taken[kThreads / 64][kTake];
  const int count = min(*a.fix_count, a.fix_cap);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (a.fix_total && blockIdx.x == 0 && threadIdx.x == 0 && count > 0) atomicAdd(a.fix_total, (unsigned long long)count);
  const int nw = gridDim.x * (kThreads / 64);
  uint64_t* tk = taken[wv];
  for (int item = blockIdx.x * (kThreads / 64) + wv; item < count; item += nw) {
    const int64_t flat = list[item];
    const int64_t qi = flat / a.v_used, r = flat % a.v_used;
    const int64_t b = a.q0 + qi;
    const int64_t s0 = a.qptr[b];
    const int h = (int)(a.qptr[b + 1] - s0);
    const float* vrow = a.V + (size_t)a.used[r] * a.m_pad;
    uint64_t key[kCols];
#pragma unroll
    for (int j = 0; j < kCols; ++j) {
      const int c = lane + 64 * j;
      key[j] = ~0ull;
      if (c < h) {
        const float4* q = (const float4*)(a.V + (size_t)a.qcol[s0 + c] * a.m_pad);
        float d2 = 0.f;
        // eight float4 of each vector (one 128-byte line) are loaded together
        // and then added in the same order as one at a time (indices past
        // the end are clamped and their values unused); the zero padding
        // adds exact zeros
        for (int d0 = 0; d0 < a.m4; d0 += 8) {
          float4 y[8], x[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int d = min(d0 + i, a.m4 - 1);
            y[i] = q[d];
            x[i] = *(const float4*)(vrow + 4 * d);
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            if (d0 + i < a.m4) {
              float e;
              e = x[i].x - y[i].x; d2 = fmaf(e, e, d2);
              e = x[i].y - y[i].y; d2 = fmaf(e, e, d2);
              e = x[i].z - y[i].z; d2 = fmaf(e, e, d2);
              e = x[i].w - y[i].w; d2 = fmaf(e, e, d2);
            }
          }
        }
        key[j] = w_pack(d2, (uint32_t)c);
      }
    }
    int kef;
    const float bound = MODE == P1_TABLE ? a.xmax[r] : INFINITY;
    if (MODE == P1_TABLE_FULL) kef = min(a.k, h);
    else if (a.method == LCEMD_ICT) kef = h;
    else if (a.method == LCEMD_OMR) kef = min(2, h);
    else if (a.method == LCEMD_RWMD) kef = 1;
    else kef = min(a.k, h);
    const int limit = min(MODE == P1_TABLE ? min(h, a.KT + 1) : min(h, a.k), kTake);
    int D = 0;
    float Pc = 0.f;
    bool done = false;  // a cut was reached
    for (int l = 0; l < limit; ++l) {
      uint64_t m = ~0ull;
#pragma unroll
      for (int j = 0; j < kCols; ++j) m = key[j] < m ? key[j] : m;
#pragma unroll
      for (int sh = 32; sh >= 1; sh >>= 1) {
        int lo = (int)(uint32_t)m, hi = (int)(uint32_t)(m >> 32);
        lo = __shfl_xor(lo, sh);
        hi = __shfl_xor(hi, sh);
        const uint64_t o = ((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo;
        m = o < m ? o : m;
      }
#pragma unroll
      for (int j = 0; j < kCols; ++j)
        if (key[j] == m) key[j] = ~0ull;  // keys are distinct (position bits)
      if (lane == 0) tk[l] = m;
      ++D;
      Pc += a.qval[s0 + (uint32_t)m];
      done = D >= kef || D == h;
      if (MODE == P1_TABLE)
        done = done || Pc >= bound || (a.method == LCEMD_OMR && l == 0 && w_unpack(m) != 0.f);
      if (done) break;
    }
    if (lane == 0) {  // the lane that recorded the taken entries
      if (MODE == P1_TABLE) {
        if (D > a.KT || !done) {  // deeper than the table, or than kTake entries
          a.overflow[0] = 1;
        } else {
          zw_write_row(a.ZW, a.zw_nq, a.KT, qi, r, D,
                       [&](int l) { return sqrtf(fmaxf(w_unpack(tk[l]), 0.f)); },
                       [&](int l) { return l == D - 1 ? INFINITY : a.qval[s0 + (uint32_t)tk[l]]; });
        }
      } else {
        const int64_t o0 = flat * (int64_t)a.k;
        for (int l = 0; l < a.k; ++l) {
          if (l < D) {
            const int pos = (int)(uint32_t)tk[l];
            a.S[o0 + l] = pos;
            a.Z[o0 + l] = sqrtf(fmaxf(w_unpack(tk[l]), 0.f));
            a.W[o0 + l] = a.qval[s0 + pos];
          } else {
            a.S[o0 + l] = -1;
            a.Z[o0 + l] = 0.f;
            a.W[o0 + l] = 0.f;
          }
        }
      }
    }
  }
}

hipError_t launch_fix_rows(const P1Args& a, int mode, int count, hipStream_t s) {
  // `count` bounds the grid; the kernel reads the live count from a.fix_count
  if (count <= 0) return hipSuccess;
  if (mode == P1_TABLE_FULL && a.k > 64) return hipErrorInvalidValue;
  const int per = kThreads / 64;
  const unsigned grid = (unsigned)std::min<int64_t>((count + per - 1) / per, 65536);
  if (mode == P1_TABLE)
    hipLaunchKernelGGL(k_fix_rows<P1_TABLE>, dim3(grid), dim3(kThreads), 0, s, a, a.fix_list);
  else if (mode == P1_TABLE_FULL)
    hipLaunchKernelGGL(k_fix_rows<P1_TABLE_FULL>, dim3(grid), dim3(kThreads), 0, s, a, a.fix_list);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_phase1_wide(const P1Args& a, int mode, int KL, hipStream_t s) {
  if (!a.V8 || !a.vscale || a.m8 % 128 != 0) return hipErrorInvalidValue;
  if (mode == P1_TABLE) return launch_wide_mode<P1_TABLE>(a, KL, s);
  if (mode == P1_TABLE_FULL) return launch_wide_mode<P1_TABLE_FULL>(a, KL, s);
  return hipErrorInvalidValue;
}

}  // namespace lcemd
