// Phase 2/3 of LC-ACT (Sec. 4, Eq. 6-9) for small vocabularies and tables of
// one or two entries per row: the tables of 16 queries live in LDS.
//
// k_phase2_persistent reads a 16-byte table pair per (non-zero, query) from
// L1/L2, and that path's 64 bytes per CU and clock bound it (784-word image
// tables, one transfer: 31.9 TB/s, 81 % of the path).  LDS gives twice the
// bytes per clock, and there a row is cut to what the measure reads: one
// distance (KT = 1) or (z0, w0, z1) (KT = 2; the last entry's capacity is
// never read: it takes the rest).  The kernel is then bound by its vector
// instructions (about eight per non-zero and 64 queries, 77 % of the issue
// cycles busy; the row broadcasts among them cost two).  60,000 images x
// 3,000 queries, 784 words: KT = 2 14.6 -> 8.7 ms, KT = 1 14.6 -> 4.6 ms.
// Measured without gain: windows of 256 with the results in registers (8.74
// ms), table reads issued a group ahead (8.9), records loaded by every lane
// instead of broadcast (9.1; KT = 1 8.0), 12-byte entries behind one address
// (9.3).
//
// Split: a workgroup of 16 waves (one per CU, it owns the LDS) stages the
// tables of 16 queries once and takes windows of 128 documents; units (query
// group, window) are divided evenly and in order over the grid, so a
// workgroup changes tables once or twice in a large batch.  A DPP row of 16
// lanes is one document x 16 queries: the row's lanes load 16 records
// together and hand them on by row broadcast, which costs no LDS bandwidth.
// The four documents of a wave are neighbours in their window's order of
// length; a wave's two turns in a window are its w-th and (31 - w)-th
// quadruple, so that the waves end together, and the window's results leave
// through LDS as whole lines (stored one by one, every 4 bytes cost a 32-byte
// write).
//
// Deeper tables stay with k_phase2_persistent: with only their first pair in
// LDS (8 queries), packing the walks that go on (16 % of them) into full
// waves cost more instructions than the loads it saved (20,000 images x 501
// queries, KT = 8: 3.46 ms against 2.36 ms).
//
// Every (query, document) sum is the one of k_phase2_persistent: eight-term
// trees in CSR order, Kahan across groups -- the same bits.
#include <algorithm>

#include "internal.h"
#include "launch_sizes.h"
#include "phase2_step.h"

namespace lcemd {

namespace {

constexpr int kLT = 1024;           // threads: 16 waves, one workgroup per CU
constexpr int kWin = 128;           // documents of a window (the order of length is made per window)
constexpr int kG = 16;              // queries per workgroup
constexpr int kOutLd = kWin + 4;    // floats per query of the window's staged results
constexpr size_t kLdsMax = 160 * 1024;

// bytes of a table row: KT = 1: z; KT = 2: (z0, w0) pairs, then z1
template <int KT>
constexpr int row_bytes() { return KT == 1 ? 64 : 192; }

// the value of the row's lane K (0-15) in every lane of a 16-lane row
template <int K>
__device__ __forceinline__ int row_bcast(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x150 + K, 0xf, 0xf, true);
}
struct Kahan {
  float t = 0.f, comp = 0.f;
  __device__ __forceinline__ void add(float g) {
    const float y = g - comp;
    const float tt = t + y;
    comp = (tt - t) - y;
    t = tt;
  }
};

// LDS by byte address (one register per address; row broadcasts then fold
// into the address additions)
using lds_u32 = uint32_t;
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ lds_u32 lds_addr(const void* p) {
  return (lds_u32)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
template <typename T>
__device__ __forceinline__ T lds_read(lds_u32 a) {
  return *(const __attribute__((address_space(3))) T*)(uintptr_t)a;
}

// The sum of the costs of the row's records B .. B + 7 against the
// lane's query.  roff / wbits: the lane's own record (its word's row offset,
// its weight); ta, tb: the lane's addresses of (z0, w0) (or z) and z1 in
// table row 0.  All reads are issued before the first use.  Padding records
// have weight 0: cost 0 (but see doc_by_records).
template <int KT, int B>
__device__ __forceinline__ float group_cost(lds_u32 ta, lds_u32 tb, int roff, int wbits) {
  float a[8];
  if constexpr (KT == 1) {
    float z[8];
    z[0] = lds_read<float>(row_bcast<B + 0>(roff) + ta);
    z[1] = lds_read<float>(row_bcast<B + 1>(roff) + ta);
    z[2] = lds_read<float>(row_bcast<B + 2>(roff) + ta);
    z[3] = lds_read<float>(row_bcast<B + 3>(roff) + ta);
    z[4] = lds_read<float>(row_bcast<B + 4>(roff) + ta);
    z[5] = lds_read<float>(row_bcast<B + 5>(roff) + ta);
    z[6] = lds_read<float>(row_bcast<B + 6>(roff) + ta);
    z[7] = lds_read<float>(row_bcast<B + 7>(roff) + ta);
    __builtin_amdgcn_sched_barrier(0);
    // (written as the step's own fma: a plain product would contract with
    // the sums)
    a[0] = fmaf(__int_as_float(row_bcast<B + 0>(wbits)), z[0], 0.f);
    a[1] = fmaf(__int_as_float(row_bcast<B + 1>(wbits)), z[1], 0.f);
    a[2] = fmaf(__int_as_float(row_bcast<B + 2>(wbits)), z[2], 0.f);
    a[3] = fmaf(__int_as_float(row_bcast<B + 3>(wbits)), z[3], 0.f);
    a[4] = fmaf(__int_as_float(row_bcast<B + 4>(wbits)), z[4], 0.f);
    a[5] = fmaf(__int_as_float(row_bcast<B + 5>(wbits)), z[5], 0.f);
    a[6] = fmaf(__int_as_float(row_bcast<B + 6>(wbits)), z[6], 0.f);
    a[7] = fmaf(__int_as_float(row_bcast<B + 7>(wbits)), z[7], 0.f);
  } else {
    floatx2 zw[8];
    float z1[8];
    zw[0] = lds_read<floatx2>(row_bcast<B + 0>(roff) + ta), z1[0] = lds_read<float>(row_bcast<B + 0>(roff) + tb);
    zw[1] = lds_read<floatx2>(row_bcast<B + 1>(roff) + ta), z1[1] = lds_read<float>(row_bcast<B + 1>(roff) + tb);
    zw[2] = lds_read<floatx2>(row_bcast<B + 2>(roff) + ta), z1[2] = lds_read<float>(row_bcast<B + 2>(roff) + tb);
    zw[3] = lds_read<floatx2>(row_bcast<B + 3>(roff) + ta), z1[3] = lds_read<float>(row_bcast<B + 3>(roff) + tb);
    zw[4] = lds_read<floatx2>(row_bcast<B + 4>(roff) + ta), z1[4] = lds_read<float>(row_bcast<B + 4>(roff) + tb);
    zw[5] = lds_read<floatx2>(row_bcast<B + 5>(roff) + ta), z1[5] = lds_read<float>(row_bcast<B + 5>(roff) + tb);
    zw[6] = lds_read<floatx2>(row_bcast<B + 6>(roff) + ta), z1[6] = lds_read<float>(row_bcast<B + 6>(roff) + tb);
    zw[7] = lds_read<floatx2>(row_bcast<B + 7>(roff) + ta), z1[7] = lds_read<float>(row_bcast<B + 7>(roff) + tb);
    __builtin_amdgcn_sched_barrier(0);
    auto cost = [](int xbits, const floatx2& e, float z) {
      const float x = __int_as_float(xbits);
      const float r = __uint_as_float(min((uint32_t)xbits, __float_as_uint(e.y)));
      return fmaf(x - r, z, fmaf(r, e.x, 0.f));
    };
    a[0] = cost(row_bcast<B + 0>(wbits), zw[0], z1[0]);
    a[1] = cost(row_bcast<B + 1>(wbits), zw[1], z1[1]);
    a[2] = cost(row_bcast<B + 2>(wbits), zw[2], z1[2]);
    a[3] = cost(row_bcast<B + 3>(wbits), zw[3], z1[3]);
    a[4] = cost(row_bcast<B + 4>(wbits), zw[4], z1[4]);
    a[5] = cost(row_bcast<B + 5>(wbits), zw[5], z1[5]);
    a[6] = cost(row_bcast<B + 6>(wbits), zw[6], z1[6]);
    a[7] = cost(row_bcast<B + 7>(wbits), zw[7], z1[7]);
  }
  return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}

// The document's sum again, from its records alone, where it came out without
// a number: a padding record's mass of 0 times an infinite distance of word 0
// has none.
template <int KT>
__device__ __forceinline__ Kahan doc_by_records(const int2* __restrict__ rp, int len, lds_u32 ta, lds_u32 tb) {
  Kahan s;
#pragma unroll 1
  for (int e = 0; e < len; e += 8) {
    float pair = 0.f, quad = 0.f, g = 0.f;  // group_cost's tree
#pragma unroll 1
    for (int k = 0; k < 8; ++k) {
      float a = 0.f;
      if (e + k < len) {
        const int2 rec = rp[e + k];
        const lds_u32 ro = rec.x * row_bytes<KT>();
        if constexpr (KT == 1) {
          a = fmaf(__int_as_float(rec.y), lds_read<float>(ro + ta), 0.f);
        } else {
          const floatx2 zw = lds_read<floatx2>(ro + ta);
          const float r = __uint_as_float(min((uint32_t)rec.y, __float_as_uint(zw.y)));
          a = fmaf(__int_as_float(rec.y) - r, lds_read<float>(ro + tb), fmaf(r, zw.x, 0.f));
        }
      }
      pair = k & 1 ? pair + a : a;
      if (k & 1) quad = k & 2 ? quad + pair : pair;
      if ((k & 3) == 3) g = k & 4 ? g + quad : quad;
    }
    s.add(g);
  }
  return s;
}

template <int KT>
__global__ __launch_bounds__(kLT) void k_phase2_lds(const int64_t* __restrict__ xptr, const int2* __restrict__ xcv,
                                                    int64_t n, const int32_t* __restrict__ perm,
                                                    const float4* __restrict__ ZP, int64_t zw_nq, int64_t nq,
                                                    int v_used, float* __restrict__ out, int64_t ld) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int RB = row_bytes<KT>();
  unsigned char* tab = smem;
  float* ob = (float*)(smem + (size_t)v_used * RB);  // kG x kOutLd
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l = lane & 15, row = lane >> 4;  // l: the lane's query and its record of 16
  const lds_u32 ta = lds_addr(tab) + (KT == 1 ? 4 : 8) * l;
  const lds_u32 tb = lds_addr(tab) + 128 + 4 * l;  // KT = 2
  // the grid is a multiple of 8 and workgroup i runs on XCD i % 8: an XCD's
  // workgroups take neighbouring ranges of units
  const int64_t nr = gridDim.x, id = (int64_t)(blockIdx.x & 7) * (nr >> 3) + (blockIdx.x >> 3);
  const int64_t nwin = (n + kWin - 1) / kWin, units = (nq + kG - 1) / kG * nwin;
  int64_t have = -1;
  for (int64_t unit = units * id / nr; unit < units * (id + 1) / nr; ++unit) {
    const int64_t g = unit / nwin, w0 = unit % nwin * kWin;
    if (g != have) {
      __syncthreads();  // every wave is done with the previous tables
      have = g;
      // lanes past the batch get the last query's tables; their results are
      // not written
      for (int i = tid; i < v_used * kG; i += kLT) {
        const int r = i / kG, t = i % kG;
        const float4 e = ZP[(int64_t)r * zw_nq + min(g * kG + t, nq - 1)];  // one pair per row
        unsigned char* p = tab + (size_t)r * RB;
        if constexpr (KT == 1) {
          *(float*)(p + 4 * t) = e.x;
        } else {
          *(float2*)(p + 8 * t) = make_float2(e.x, e.y);
          *(float*)(p + 128 + 4 * t) = e.z;
        }
      }
      __syncthreads();
    }
    const int cnt = (int)min((int64_t)kWin, n - w0);
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      const int at = 4 * (half ? kWin / 4 - 1 - wave : wave) + row;
      if (at < cnt) {
        const int64_t u = perm[w0 + at];
        const int64_t e0 = xptr[u];
        const int len = (int)(xptr[u + 1] - e0);
        const int2* rp = xcv + e0;
        Kahan s;
        int2 rec = l < len ? rp[l] : make_int2(0, 0);
        for (int e = 0; e < len; e += 16) {
          const int ro = rec.x * RB, wb = rec.y;
          // the next 16 records, in flight through this step
          rec = e + 16 + l < len ? rp[e + 16 + l] : make_int2(0, 0);
          s.add(group_cost<KT, 0>(ta, tb, ro, wb));
          if (e + 8 < len) s.add(group_cost<KT, 8>(ta, tb, ro, wb));
        }
        if (__any(s.t != s.t)) s = doc_by_records<KT>(rp, len, ta, tb);
        ob[l * kOutLd + (int)(u - w0)] = s.t;
      }
    }
    __syncthreads();
    for (int i = tid; i < kG * kWin; i += kLT) {
      const int t = i / kWin, d = i % kWin;
      if (d < cnt && g * kG + t < nq) out[(g * kG + t) * ld + w0 + d] = ob[t * kOutLd + d];
    }
    __syncthreads();  // written before the next window's results come in
  }
}

size_t lds_bytes(int64_t v_used, int KT) {
  return (size_t)v_used * (KT == 1 ? row_bytes<1>() : row_bytes<2>()) + sizeof(float) * kG * kOutLd;
}

template <int KT>
hipError_t launch_lds(const int64_t* xptr, const int2* xcv, int64_t n, const int32_t* perm, int64_t v_used,
                      const float2* ZW, int64_t zw_nq, int64_t nq, float* out, int64_t ld, hipStream_t s) {
  const void* fn = (const void*)k_phase2_lds<KT>;
  const size_t sh = lds_launch_bytes(lds_bytes(v_used, KT), kLdsMax);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
  if (e != hipSuccess) return e;
  const int64_t units = (nq + kG - 1) / kG * ((n + kWin - 1) / kWin);
  const int grid = persistent_grid(fn, kLT, sh, units);
  if (grid <= 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_phase2_lds<KT>, dim3(grid), dim3(kLT), sh, s, xptr, xcv, n, perm, (const float4*)ZW, zw_nq, nq,
                     (int)v_used, out, ld);
  return hipGetLastError();
}

}  // namespace

bool phase2_lds_fits(int64_t n, int64_t v_used, int KT, int64_t nq) {
  if (KT > 2 || v_used < 1 || v_used > 2048 || lds_bytes(v_used, KT) > kLdsMax) return false;
  // Up to 32 queries k_phase2_small takes about 1.65 ps per (non-zero, query);
  // here every round of 256 windows takes about 0.15 us per word of a
  // document, whatever the queries: the line is n nq = 91,000 a round (784
  // words, KT = 2: 60,000 documents x 8: 0.165 -> 0.069 ms, x 1: 0.068 against
  // 0.070; 3,000 x 32: 0.040 -> 0.035, x 16: 0.025 against 0.034).  Larger
  // batches always run here: k_phase2_persistent was slower down to nine
  // units (300 x 33: 0.054 -> 0.033 ms).  The line was fitted to 784 words at
  // KT = 2; over 100 to 2,000 words, both depths, 300 to 18,000 documents, 1 to
  // 200 queries and the reverse direction (1 to 33 documents x as many
  // queries) the calls it sends here took 0.10-0.93 of the time of the
  // per-document kernels, one document x 18,000 queries 32-39 us against 42.
  const int64_t units = (nq + kG - 1) / kG * ((n + kWin - 1) / kWin);
  return nq > 32 || n * nq > 91000 * ((units + 255) / 256);
}

hipError_t launch_phase2_lds(const int64_t* xptr, const int2* xcv, int64_t n, const int32_t* perm, int64_t v_used,
                             const float2* ZW, int64_t zw_nq, int KT, int64_t nq, float* out, int64_t ld,
                             hipStream_t s) {
  if (!perm || !phase2_lds_fits(n, v_used, KT, nq)) return hipErrorInvalidValue;
  return KT == 1 ? launch_lds<1>(xptr, xcv, n, perm, v_used, ZW, zw_nq, nq, out, ld, s)
                 : launch_lds<2>(xptr, xcv, n, perm, v_used, ZW, zw_nq, nq, out, ld, s);
}

}  // namespace lcemd
