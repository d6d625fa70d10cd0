// Phase 2/3 of LC-ACT (Sec. 4, Eq. 6-9): for every non-zero X_ui of the
// database, the capacity-limited transfers of its mass against the query's
// table row for word i, summed per database row (document).
//
// Each table row holds (z, w) pairs in ascending distance order; its last
// valid entry carries w = +inf, so the walk below is Eq. (6)-(8) followed by
// Eq. (9) (the rest of the mass at the last distance) and always ends.
//
// Layout and mapping: batches of more than 32 queries take 64 consecutive
// queries in a wave's lanes and one document at a time (k_phase2_persistent);
// smaller ones QL queries (a power of two) beside several lanes that share a
// document's non-zeros and, below 8 queries, several documents in order of
// length within windows of 128 (a permutation made when the database is
// loaded), so that the lanes of a wave finish together while its outputs stay
// close (k_phase2_small).  A non-zero's table row is one contiguous run for the
// queries of a wave (16 bytes each, the interleaved layout), and every (query,
// document) sum has one fixed order: groups of eight consecutive non-zeros
// summed as a binary tree, the groups accumulated in order with Kahan
// compensation (the error stays a few ulps for rows of any length) -- the same
// bits whatever the split, the batch or the launch.
#include <algorithm>
#include <climits>
#include <mutex>
#include <vector>

#include "internal.h"
#include "phase2_step.h"

namespace lcemd {

constexpr int kUnroll = 8;       // non-zeros whose table loads are in flight together
constexpr int kItemSlots = 16;   // document slots per lane and work item
static_assert(kItemSlots % 4 == 0, "results are stored four at a time");

// doc_cost entry by entry and only while mass is left: no padding slot and no
// entry past a walk's end is looked at.  doc_cost multiplies those by a mass of
// 0, which is 0 unless the distance is infinite; it takes a document whose sum
// came out without a number again here, so that an infinite distance reaches
// only the documents that move mass to it, and the same ones whatever the batch
// (k_phase2_small and the word-major walk step like this).  The second entry
// of a row's first pair is the exception in all of them (phase2_step.h).
// (Asked per document: asked per group, it was 2 % of the LDS kernel's time.)
__device__ __forceinline__ float doc_by_steps(int64_t e0, int64_t e1, const int2* __restrict__ xcv,
                                              const char* __restrict__ ZP, uint32_t lane, uint32_t rbytes,
                                              uint32_t pbytes, int KP) {
  float t = 0.f, comp = 0.f;
#pragma unroll 1
  for (int64_t e = e0; e < e1; e += kUnroll) {
    float pair = 0.f, quad = 0.f, g = 0.f;  // doc_cost's tree over eight terms
#pragma unroll 1
    for (int k = 0; k < kUnroll; ++k) {
      float rem = 0.f, acc = 0.f;
      if (e + k < e1) {
        const int2 r = xcv[e + k];
        const char* base = ZP + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(r.x) * rbytes + lane;
        rem = __int_as_float(r.y);
#pragma unroll 1
        for (int p = 0; p < KP && rem > 0.f; ++p) {
          const float4 f = *(const float4*)(base + p * pbytes);
          step(rem, acc, f.x, f.y);
          if (p == 0 || rem > 0.f) step(rem, acc, f.z, f.w);
        }
      }
      pair = k & 1 ? pair + acc : acc;
      if (k & 1) quad = k & 2 ? quad + pair : pair;
      if ((k & 3) == 3) g = k & 4 ? g + quad : quad;
    }
    const float y = g - comp;
    const float tt = t + y;
    comp = (tt - t) - y;
    t = tt;
  }
  return t;
}

// Cost of document [e0, e1) against a lane's query (64 consecutive queries a
// wave): the non-zeros in order, kUnroll at a time with their first table
// pairs loaded together.  Every lane of the wave is on this document, so its
// records and the table rows' addresses are wave-uniform: ZP (the tables)
// plus the word's row in scalar registers, `lane` (the query's byte offset)
// in one vector register.  rbytes / pbytes: from one word's / pair's run to
// the next.
//
// DEEP (KT > 2): the second pairs are loaded with the first ones (some lane
// goes on for four of five non-zeros, and the walk then waits once, not
// twice).  Their values count only for lanes with mass left -- a row that
// ended in its first pair has no second one written.  Further pairs are
// loaded for the lanes that need them; the others step over the pair they
// hold, which changes nothing without mass.
// Bound: the vector-memory path (2.6 loads of 16 bytes per non-zero and
// query for image tables at KT = 8) beside as much scalar work, which is why
// a row's address is one 64-bit product and sum and nothing but the further
// pairs' loads branches.  Against the walk that loaded pair by pair and
// tested the mass before every step: 20,000 images x 501 queries, KT = 8,
// 3.47 -> 2.36 ms; 6,000 x 100 with background, KT = 16, 8.2 -> 1.32 ms, ICT
// 56.6 -> 9.6 ms; text 18,000 x 500, KT = 16, 4.01 -> 3.50 ms.
template <bool DEEP>
__device__ __forceinline__ float doc_cost(int64_t e0, int64_t e1, const int2* __restrict__ xcv,
                                          const char* __restrict__ ZP, uint32_t lane, uint32_t rbytes,
                                          uint32_t pbytes, int KP) {
  static_assert(kUnroll == 8, "the group sum below is a tree over 8 terms");
  e0 = uniform64(e0);
  e1 = uniform64(e1);
  float t = 0.f, comp = 0.f;
  auto records = [&](int64_t e, int2(&cv)[kUnroll]) {
    if (e + kUnroll <= e1) {
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) cv[k] = xcv[e + k];
    } else {
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) cv[k] = e + k < e1 ? xcv[e + k] : make_int2(0, 0);
    }
  };
  int2 nx[kUnroll];
  records(e0, nx);
  for (int64_t e = e0; e < e1; e += kUnroll) {
    const char* base[kUnroll];
    float4 f[kUnroll], f2[DEEP ? kUnroll : 1];
    float rem[kUnroll], acc[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      // padding slots read word 0's run: their mass is 0
      base[k] = ZP + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(nx[k].x) * rbytes;
      rem[k] = __int_as_float(nx[k].y);
      f[k] = *(const float4*)(base[k] + lane);
      if constexpr (DEEP) f2[k] = *(const float4*)(base[k] + (lane + pbytes));
    }
    records(e + kUnroll, nx);  // the next group's, in flight through this one
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      acc[k] = 0.f;
      step(rem[k], acc[k], f[k].x, f[k].y);
      step(rem[k], acc[k], f[k].z, f[k].w);
    }
    if constexpr (DEEP) {
      float left = 0.f;
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const bool on = rem[k] > 0.f;
        f[k] = make_float4(on ? f2[k].x : 0.f, f2[k].y, on ? f2[k].z : 0.f, f2[k].w);
        step(rem[k], acc[k], f[k].x, f[k].y);
        step(rem[k], acc[k], f[k].z, f[k].w);
        left = fmaxf(left, rem[k]);
      }
      for (int p = 2; p < KP && __any(left > 0.f); ++p) {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k)
          if (rem[k] > 0.f) f[k] = *(const float4*)(base[k] + (lane + p * pbytes));
        left = 0.f;
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
          step(rem[k], acc[k], f[k].x, f[k].y);
          step(rem[k], acc[k], f[k].z, f[k].w);
          left = fmaxf(left, rem[k]);
        }
      }
    }
    // padding slots hold exact zeros
    const float g = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    const float y = g - comp;
    const float tt = t + y;
    comp = (tt - t) - y;
    t = tt;
  }
  if (__any(t != t)) t = doc_by_steps(e0, e1, xcv, ZP, lane, rbytes, pbytes, KP);
  return t;
}

// Batches of more than 32 queries.  Persistent grid: waves pull (64
// queries, `slots` documents) items from eight work counters, one per XCD,
// each walking a contiguous eighth of the items, query group major (an XCD
// keeps one group's slice of the tables hot in its L2).  For fixed-shape
// batches the live query count is read from device memory, and the launcher
// issues one kernel per lane width: the one whose band holds the live count
// works, the others return at once (so a batch with few live queries does
// not pay for the lanes of its empty slots).  Every wave exits once its
// counter passes the end of its range.
//
// slots (4, 8 or kItemSlots consecutive documents) is the host's: a lane's
// results leave as 16-byte stores, so long items write whole sectors, but
// one 64-query group of 18,000 documents is only 1,125 items of 16 -- about
// one wave per SIMD, each alone with its loads' latency.  The launcher
// shortens items until the chip holds about 16 waves per CU (ICT, 64
// queries: 1,355 -> 520 us) and an XCD's waves stay with one group's tables
// (501 documents x 20,000 queries, KT = 8: 5.7 -> 3.6 ms).
template <bool DEEP>
__global__ __launch_bounds__(kThreads) void k_phase2_persistent(
    const int64_t* __restrict__ xptr, const int2* __restrict__ xcv, int64_t n,
    const float4* __restrict__ ZP, int64_t zw_nq, int KP, int64_t nq_arg, const int* __restrict__ nq_dev,
    int slots, float* __restrict__ out, int64_t ld, unsigned long long* __restrict__ counters) {
  constexpr int QL = 64;
  const int lane = threadIdx.x & 63;
  const int xcd = blockIdx.x & 7;
  const int64_t nq = nq_dev ? (int64_t)*nq_dev : nq_arg;
  if (nq_dev && (nq > nq_arg || 2 * nq <= QL)) return;  // another width's band
  const int64_t nd = (n + slots - 1) / slots;
  const int64_t total = (nq + QL - 1) / QL * nd;
  const int64_t lo = total * xcd / 8, hi = total * (xcd + 1) / 8;
  const uint32_t pbytes = (uint32_t)zw_nq * 16u, rbytes = (uint32_t)KP * pbytes;  // (the launcher checks)
  while (true) {
    unsigned long long it = 0;
    if (lane == 0) it = atomicAdd(&counters[xcd], 1ull);
    const int64_t item = uniform64(lo + (int64_t)__shfl((long long)it, 0));
    if (item >= hi) break;
    // lanes past the batch walk the last query's table and write nothing
    const int64_t q = (item / nd) * QL + lane;
    const bool qok = q < nq;
    const uint32_t zq = (uint32_t)(qok ? q : nq - 1) * 16u;
    const int64_t d0 = (item % nd) * slots;
    // one document at a time for all 64 lanes: each lane's results are
    // consecutive in its query's row, so they are staged in the wave's own
    // LDS rows (lane-private slots: no barrier) and written together,
    // 16-byte stores where aligned
    __shared__ float st[kThreads / 64][kItemSlots][64];
    float(*sw)[64] = st[threadIdx.x >> 6];
    int cnt = 0;
    for (int j = 0; j < slots; ++j) {
      const int64_t i = d0 + j;
      if (i >= n) break;
      sw[j][lane] = doc_cost<DEEP>(xptr[i], xptr[i + 1], xcv, (const char*)ZP, zq, rbytes, pbytes, KP);
      ++cnt;
    }
    if (qok && cnt > 0) {
      float* o = out + q * ld + d0;
      if (cnt == slots && (reinterpret_cast<uintptr_t>(o) & 15) == 0) {
        for (int t = 0; t < slots; t += 4)
          *reinterpret_cast<float4*>(o + t) = make_float4(sw[t][lane], sw[t + 1][lane], sw[t + 2][lane], sw[t + 3][lane]);
      } else {
        for (int t = 0; t < cnt; ++t) o[t] = sw[t][lane];
      }
    }
  }
}

// Batches of up to 32 queries: a wave's lanes are QL queries (fastest, so a
// non-zero's table run is one contiguous read) x NL non-zeros of one group
// of eight x S documents (S > 1 only below 8 queries; then taken in order of
// length within windows of 128).  Lane j of a document's NL holds non-zeros
// j, j + NL, ... of every group, NL groups a step, so a lane has eight table
// loads in flight as in doc_cost; the group sums cross the lanes as the same
// eight-term tree and every lane of the document runs the same Kahan chain:
// the bits of doc_cost.
//
// Bound: the table gather's latency and the L1/L2 request rate.  The former
// split (documents side by side, 16 slots each, work counters) put 18,000
// documents x 1 query on 18 waves: 1,813 us, and x 16 queries on 281:
// 1,043 us.  Spreading a document's non-zeros over lanes gives 8x the waves
// and coalesced record reads: 35 us and 133 us (ACT, k = 8 and 4, 2.1 M
// non-zeros, 70,000 words).
// Waves take documents at a fixed stride (a counter's atomics, about 0.2 us
// each on one address, cost more than the walk of a short document).
template <int QL>
__global__ __launch_bounds__(kThreads) void k_phase2_small(
    const int64_t* __restrict__ xptr, const int2* __restrict__ xcv, int64_t n,
    const int32_t* __restrict__ perm, const float4* __restrict__ ZP, int64_t zw_nq, int KP,
    int64_t nq_arg, const int* __restrict__ nq_dev, float* __restrict__ out, int64_t ld) {
  constexpr int NL = QL >= 8 ? 64 / QL : 8;  // lanes of a group of eight non-zeros
  constexpr int S = 64 / (QL * NL);          // documents side by side
  constexpr int PER = kUnroll / NL;          // non-zeros of a group per lane
  constexpr int G = NL;                      // groups a step: PER * G = 8 loads in flight
  const int64_t nq = nq_dev ? (int64_t)*nq_dev : nq_arg;
  if (nq_dev && (nq > nq_arg || (QL > 1 ? 2 * nq <= QL : nq < 1))) return;  // another width's band
  const int lane = threadIdx.x & 63, qs = lane % QL, j = lane / QL % NL, ds = lane / (QL * NL);
  // lanes past the batch walk the last query's table and write nothing
  const bool qok = qs < nq;
  const float4* Zq = ZP + (qok ? qs : nq - 1);
  const int64_t rstride = (int64_t)KP * zw_nq;  // float4s from one word's run to the next
  const int64_t wave = (int64_t)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t items = (n + S - 1) / S, nw = (int64_t)gridDim.x * (kThreads / 64);
  for (int64_t item = wave; item < items; item += nw) {
    const int64_t i = min(item * S + ds, n - 1);  // past the end: the last document again, not written
    const int64_t u = S > 1 ? (int64_t)perm[i] : i;
    int64_t e0 = xptr[u], e1 = xptr[u + 1];
    if constexpr (S == 1) {
      e0 = uniform64(e0);
      e1 = uniform64(e1);
    }
    float t = 0.f, comp = 0.f;
    for (int64_t e = e0; e < e1; e += kUnroll * G) {
      const int left = (int)min((int64_t)(kUnroll * G), e1 - e);
      float rem[kUnroll], acc[kUnroll];
      const float4* base[kUnroll];
      int2 cv[kUnroll];
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {  // k = PER * group + non-zero of the lane
        const int at = kUnroll * (k / PER) + j + NL * (k % PER);
        cv[k] = at < left ? xcv[e + at] : make_int2(0, 0);
      }
      float4 f[kUnroll];
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const int at = kUnroll * (k / PER) + j + NL * (k % PER);
        base[k] = Zq + (int64_t)cv[k].x * rstride;
        f[k] = at < left ? base[k][0] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      bool any = false;
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        rem[k] = __int_as_float(cv[k].y);  // 0 for the padding slots
        acc[k] = 0.f;
        step(rem[k], acc[k], f[k].x, f[k].y);
        step(rem[k], acc[k], f[k].z, f[k].w);
        any = any || rem[k] > 0.f;
      }
      for (int p = 1; any && p < KP; ++p) {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k)
          if (rem[k] > 0.f) f[k] = base[k][p * zw_nq];
        any = false;
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
          if (rem[k] > 0.f) {
            step(rem[k], acc[k], f[k].x, f[k].y);
            if (rem[k] > 0.f) step(rem[k], acc[k], f[k].z, f[k].w);
            any = any || rem[k] > 0.f;
          }
        }
      }
      // group sums: ((a0 + a1) + (a2 + a3)) + ((a4 + a5) + (a6 + a7)), the
      // terms of one lane NL apart, the others across lanes (a sum of two is
      // the same bits either way round); groups past the document add +0
      // to a state they leave unchanged, so they are skipped
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float a[PER];
#pragma unroll
        for (int r = 0; r < PER; ++r) {
          a[r] = acc[PER * g + r];
#pragma unroll
          for (int o = 1; o < NL; o <<= 1) a[r] += __shfl_xor(a[r], o * QL);
        }
        float s;
        if constexpr (PER == 1) s = a[0];
        else if constexpr (PER == 2) s = a[0] + a[1];
        else s = (a[0] + a[1]) + (a[2] + a[3]);
        if (kUnroll * g < left) {
          const float y = s - comp;
          const float tt = t + y;
          comp = (tt - t) - y;
          t = tt;
        }
      }
    }
    if (j == 0 && qok && item * S + ds < n) out[(int64_t)qs * ld + u] = t;
  }
}

__global__ void k_zero_ints(int* p, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0;
}

hipError_t launch_zero_ints(int* p, int count, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_ints, dim3((count + 63) / 64), dim3(64), 0, s, p, count);
  return hipGetLastError();
}

namespace {
struct OccEntry {
  const void* fn;
  size_t shmem;
  int device;
  int per_cu;
};
// a fixed table (no allocation at launch time); once full, further
// kernels are queried at every launch
constexpr int kOccCap = 512;
std::mutex g_occ_mu;
OccEntry g_occ[kOccCap];
int g_nocc = 0;
int g_cus[64] = {0};
}  // namespace

int persistent_grid(const void* fn, int threads, size_t shmem, int64_t items) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -1;
  int per_cu = -1;
  {
    std::lock_guard<std::mutex> g(g_occ_mu);
    for (int i = 0; i < g_nocc; ++i)
      if (g_occ[i].fn == fn && g_occ[i].shmem == shmem && g_occ[i].device == dev) per_cu = g_occ[i].per_cu;
    if (!g_cus[dev] && hipDeviceGetAttribute(&g_cus[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return -1;
    if (per_cu < 0) {
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, shmem) != hipSuccess) return -1;
      if (g_nocc < kOccCap) g_occ[g_nocc++] = OccEntry{fn, shmem, dev, per_cu};
    }
  }
  if (per_cu < 1) return -1;
  int64_t grid = (int64_t)per_cu * g_cus[dev];
  grid = std::min<int64_t>(grid, (items + 7) / 8 * 8);
  grid = std::max<int64_t>(8, (grid + 7) / 8 * 8);
  return (int)grid;
}

template <bool DEEP>
static hipError_t launch_p2_wide(const int64_t* xptr, const int2* xcv, int64_t n, const float2* ZW, int64_t zw_nq,
                                 int KT, int64_t nq, const int* nq_dev, float* out, int64_t ld,
                                 unsigned long long* counters, hipStream_t s) {
  // the kernel's 32-bit offsets (tiles hold at most 16,384 queries and 512 pairs)
  if (zw_pairs(KT) * zw_nq * 16 >= (int64_t(1) << 32)) return hipErrorInvalidValue;
  // documents per item: the longest of 16, 8, 4 that leaves about 16 waves
  // per CU (256 CUs), and, an XCD holding about 512 waves, no more than one
  // query group's tables in use on an XCD at a time
  int slots = kItemSlots;
  while (slots > 4 && ((nq + 63) / 64 * ((n + slots - 1) / slots) < 4096 || (n + slots - 1) / slots < 512)) slots /= 2;
  // waves needed at most (bounds the grid)
  const int64_t items = (nq + 63) / 64 * ((n + slots - 1) / slots);
  const int grid = persistent_grid((const void*)k_phase2_persistent<DEEP>, kThreads, 0, (items + 3) / 4);
  if (grid <= 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_phase2_persistent<DEEP>, dim3(grid), dim3(kThreads), 0, s, xptr, xcv, n, (const float4*)ZW, zw_nq,
                     (int)zw_pairs(KT), nq, nq_dev, slots, out, ld, counters);
  return hipGetLastError();
}

template <int QL>
static hipError_t launch_p2_small(const int64_t* xptr, const int2* xcv, int64_t n, const int32_t* perm,
                                  const float2* ZW, int64_t zw_nq, int KT, int64_t nq, const int* nq_dev,
                                  float* out, int64_t ld, hipStream_t s) {
  constexpr int kDocs = QL >= 8 ? 1 : 8 / QL;  // documents of a wave
  const int64_t items = (n + kDocs - 1) / kDocs;
  const int grid = persistent_grid((const void*)k_phase2_small<QL>, kThreads, 0, (items + 3) / 4);
  if (grid <= 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_phase2_small<QL>, dim3(grid), dim3(kThreads), 0, s, xptr, xcv, n, perm, (const float4*)ZW,
                     zw_nq, (int)zw_pairs(KT), nq, nq_dev, out, ld);
  return hipGetLastError();
}

hipError_t launch_phase2_persistent(const int64_t* xptr, const int2* xcv, int64_t n, const int32_t* perm,
                                    const float2* ZW, int64_t zw_nq, int KT, int64_t nq,
                                    const int* nq_dev, float* out, int64_t ld,
                                    unsigned long long* counters, hipStream_t s) {
  // nq: the batch size, or with nq_dev the largest live count
  if (n <= 0 || nq <= 0) return hipSuccess;
  if (nq <= 32 && !perm) return hipErrorInvalidValue;
  // lane width: the smallest power of two >= the queries (at most 64); with
  // a device-side live count, every width up to that one (each works only
  // for live counts in its band)
  int top = 1;
  while (top < 64 && top < nq) top *= 2;
  hipError_t e;
  if (top == 64) {
    e = launch_zero_ints((int*)counters, 16, s);
    if (e != hipSuccess) return e;
  }
  for (int ql = top; ql >= (nq_dev ? 1 : top); ql /= 2) {
    const int64_t qmax = ql == top ? nq : std::min<int64_t>(nq, ql);  // the most queries this width takes
    switch (ql) {
      case 64:
        e = KT > 2 ? launch_p2_wide<true>(xptr, xcv, n, ZW, zw_nq, KT, qmax, nq_dev, out, ld, counters, s)
                   : launch_p2_wide<false>(xptr, xcv, n, ZW, zw_nq, KT, qmax, nq_dev, out, ld, counters, s);
        break;
      case 32: e = launch_p2_small<32>(xptr, xcv, n, perm, ZW, zw_nq, KT, qmax, nq_dev, out, ld, s); break;
      case 16: e = launch_p2_small<16>(xptr, xcv, n, perm, ZW, zw_nq, KT, qmax, nq_dev, out, ld, s); break;
      case 8: e = launch_p2_small<8>(xptr, xcv, n, perm, ZW, zw_nq, KT, qmax, nq_dev, out, ld, s); break;
      case 4: e = launch_p2_small<4>(xptr, xcv, n, perm, ZW, zw_nq, KT, qmax, nq_dev, out, ld, s); break;
      case 2: e = launch_p2_small<2>(xptr, xcv, n, perm, ZW, zw_nq, KT, qmax, nq_dev, out, ld, s); break;
      default: e = launch_p2_small<1>(xptr, xcv, n, perm, ZW, zw_nq, KT, qmax, nq_dev, out, ld, s); break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Word-major phase 2 for large vocabularies.  When a query group's tables
// are far larger than the caches, the per-document walk above re-reads a
// word's table run from HBM for every document that holds the word.  Here
// the same transfers run in two passes over one group of 64 queries:
//  A. the database's non-zeros word by word (their weights grouped by word,
//     made at load): a wave keeps the 64 queries' table run of the current
//     word in registers (pairs loaded as some lane's walk first needs them)
//     and writes each non-zero's 64 costs as one 256-byte row, in the same
//     by-word order (a sequential stream);
//  B. the documents in order: every (query, document) sum takes the costs
//     of its non-zeros in CSR order (each non-zero's by-word index from a
//     map made at load) with the grouping and compensation of doc_cost
//     (eight-term trees, Kahan across groups).
// The walk in A is the same sequence of step() calls as in doc_cost, so
// the results are the same bits whichever phase 2 ran.
constexpr int kWmSpan = 2048;  // non-zeros per pass-A wave (a fixed range: no work counter)

// Pass A.  Wave w takes the by-word records [w kWmSpan, (w + 1) kWmSpan),
// which may span many words; a lane per query.  The next two words' first
// table pairs and end offsets are in flight while the current word runs,
// and the next 64 weights while the current 64 are walked.
template <int KPM>
__global__ __launch_bounds__(kThreads) void k_p2_word_costs(
    const int64_t* __restrict__ wptr, const float* __restrict__ wwt, int64_t nnz, int64_t v_used,
    const float4* __restrict__ ZP, int64_t zw_nq, int KP, float* __restrict__ cost) {
  const int lane = threadIdx.x & 63;
  // the wave's index, made visibly wave-uniform (its range, offsets and
  // counts then live in scalar registers)
  const int64_t gw = (int64_t)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t e0 = gw * kWmSpan, e1 = min(nnz, e0 + kWmSpan);
  if (e0 >= e1) return;
  // the word of e0: the last p with wptr[p] <= e0 (wave-uniform search)
  int64_t lo = 0, hi = v_used;  // wptr[lo] <= e0 < wptr[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (uniform64(wptr[mid]) <= e0) lo = mid;
    else hi = mid;
  }
  int64_t word = lo;
  int64_t wend = uniform64(wptr[word + 1]);
  // indices past the last word are clamped to it: those loads are never used
  // (no record lies past the last word), and plain loads of valid rows keep
  // the compiler from selecting between pointers
  const int64_t lastw = v_used - 1;
  int64_t nend = uniform64(wptr[min(word + 2, v_used)]);
  int64_t nend2 = uniform64(wptr[min(word + 3, v_used)]);
  const int64_t rs = (int64_t)KP * zw_nq;  // float4s from one word's run to the next
  const float4* run = ZP + word * rs + lane;
  float4 f[KPM];
  f[0] = run[0];
  float4 fn = ZP[min(word + 1, lastw) * rs + lane];
  float4 fn2 = ZP[min(word + 2, lastw) * rs + lane];
  int loaded = 1;
  // weights come 64 at a time, one per lane (the next 64 in flight while
  // these are walked), and are read out to every lane by readlane
  float wcur = e0 + lane < e1 ? wwt[e0 + lane] : 0.f, wnext = 0.f;
  for (int64_t e = e0; e < e1; e += kUnroll) {
    const int cnt = (int)min((int64_t)kUnroll, e1 - e);
    const int off = (int)((e - e0) & 63);
    if (off == 0 && e + 64 < e1) wnext = e + 64 + lane < e1 ? wwt[e + 64 + lane] : 0.f;
    const float wcur0 = wcur;  // this batch's block of weights
    float rec[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k)
      rec[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wcur), off + k));
    if (off + kUnroll == 64) wcur = wnext;
    float* cb = cost + e * 64 + lane;  // this batch's cost rows (offsets k * 256 bytes)
    if (e + cnt <= wend) {
      // the whole batch on the current word: the eight walks side by side,
      // pair by pair (the same steps per walk as one at a time)
      float rem[kUnroll], acc[kUnroll];
      bool any = false;
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        rem[k] = rec[k];  // 0 past the range: the weight blocks hold 0 there
        acc[k] = 0.f;
        step(rem[k], acc[k], f[0].x, f[0].y);
        step(rem[k], acc[k], f[0].z, f[0].w);
        any = any || rem[k] > 0.f;
      }
#pragma unroll
      for (int p = 1; p < KPM; ++p) {
        if (p >= KP || !__any(any)) break;
        if (p >= loaded) {
          f[p] = run[p * zw_nq];
          loaded = p + 1;
        }
        any = false;
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
          if (rem[k] > 0.f) {
            step(rem[k], acc[k], f[p].x, f[p].y);
            if (rem[k] > 0.f) step(rem[k], acc[k], f[p].z, f[p].w);
            any = any || rem[k] > 0.f;
          }
        }
      }
      if (cnt == kUnroll) {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) cb[k * 64] = acc[k];
      } else {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k)
          if (k < cnt) cb[k * 64] = acc[k];
      }
      continue;
    }
    // the batch crosses into later words: one walk at a time
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      if (k >= cnt) break;
      const int64_t ee = e + k;
      if (ee >= wend) {  // the next word (wave-uniform)
        ++word;
        if (ee < nend) {
          f[0] = fn;
          fn = fn2;
          wend = nend;
          nend = nend2;
        } else {  // words without records (none in a loaded database): search on
          while (uniform64(wptr[word + 1]) <= ee) ++word;
          wend = uniform64(wptr[word + 1]);
          f[0] = ZP[word * rs + lane];
          fn = ZP[min(word + 1, lastw) * rs + lane];
          nend = uniform64(wptr[min(word + 2, v_used)]);
        }
        run = ZP + word * rs + lane;
        loaded = 1;
        nend2 = uniform64(wptr[min(word + 3, v_used)]);
        fn2 = ZP[min(word + 2, lastw) * rs + lane];
      }
      float rem = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wcur0), off + k)), acc = 0.f;
      step(rem, acc, f[0].x, f[0].y);
      step(rem, acc, f[0].z, f[0].w);
#pragma unroll
      for (int p = 1; p < KPM; ++p) {
        if (p >= KP || !__any(rem > 0.f)) break;
        if (p >= loaded) {  // the first walk to reach this pair loads it for the wave
          f[p] = run[p * zw_nq];
          loaded = p + 1;
        }
        if (rem > 0.f) {
          step(rem, acc, f[p].x, f[p].y);
          if (rem > 0.f) step(rem, acc, f[p].z, f[p].w);
        }
      }
      cb[k * 64] = acc;
    }
  }
}

// Pass B: one wave per kItemSlots consecutive documents, a lane per query.
__global__ __launch_bounds__(kThreads) void k_p2_doc_sums(const int64_t* __restrict__ xptr, int64_t n,
                                                          const uint32_t* __restrict__ winv,
                                                          const float* __restrict__ cost, float* __restrict__ out,
                                                          int64_t ld, unsigned long long* __restrict__ counters) {
  __shared__ float st[kThreads / 64][kItemSlots][64];
  float(*sw)[64] = st[threadIdx.x >> 6];
  const int lane = threadIdx.x & 63;
  const int xcd = blockIdx.x & 7;
  const int64_t total = (n + kItemSlots - 1) / kItemSlots;
  const int64_t lo = total * xcd / 8, hi = total * (xcd + 1) / 8;
  while (true) {
    unsigned long long it = 0;
    if (lane == 0) it = atomicAdd(&counters[8 + xcd], 1ull);
    const int64_t item = uniform64(lo + (int64_t)__shfl((long long)it, 0));
    if (item >= hi) break;
    const int64_t d0 = item * kItemSlots;
    int cnt = 0;
    for (int j = 0; j < kItemSlots; ++j) {
      const int64_t u = d0 + j;
      if (u >= n) break;
      const int64_t e0 = uniform64(xptr[u]), e1 = uniform64(xptr[u + 1]);
      float t = 0.f, comp = 0.f;
      int wv = 0;  // 64 by-word indices at a time, one per lane
      for (int64_t e = e0; e < e1; e += kUnroll) {
        const int c8 = (int)min((int64_t)kUnroll, e1 - e);
        const int off = (int)((e - e0) & 63);
        if (off == 0) wv = e + lane < e1 ? (int)winv[e + lane] : 0;
        float x[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
          const uint32_t wi = (uint32_t)__builtin_amdgcn_readlane(wv, off + k);
          x[k] = k < c8 ? cost[(int64_t)wi * 64 + lane] : 0.f;
        }
        const float g = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        const float y = g - comp;
        const float tt = t + y;
        comp = (tt - t) - y;
        t = tt;
      }
      sw[j][lane] = t;
      ++cnt;
    }
    float* o = out + (int64_t)lane * ld + d0;
    if (cnt == kItemSlots && (reinterpret_cast<uintptr_t>(o) & 15) == 0) {
#pragma unroll
      for (int t = 0; t < kItemSlots; t += 4)
        *reinterpret_cast<float4*>(o + t) = make_float4(sw[t][lane], sw[t + 1][lane], sw[t + 2][lane], sw[t + 3][lane]);
    } else {
      for (int t = 0; t < cnt; ++t) o[t] = sw[t][lane];
    }
  }
}

hipError_t launch_phase2_wordmajor(const int64_t* xptr, int64_t n, const int64_t* wptr, const float* wwt,
                                   const uint32_t* winv, int64_t nnz, int64_t v_used, const float2* ZW,
                                   int64_t zw_nq, int KT, float* cost, float* out, int64_t ld,
                                   unsigned long long* counters, hipStream_t s) {
  // one group of 64 queries: ZW and out start at the group's first query
  const int KP = (int)zw_pairs(KT);
  if (n <= 0 || nnz <= 0 || v_used <= 0) return hipSuccess;
  if (KP > 8 || nnz > 0xffffffffLL) return hipErrorInvalidValue;
  hipError_t e = launch_zero_ints((int*)counters, 32, s);
  if (e != hipSuccess) return e;
  const int64_t waves = (nnz + kWmSpan - 1) / kWmSpan;
  const dim3 ga((unsigned)((waves + kThreads / 64 - 1) / (kThreads / 64)));
  if (KP <= 4)
    hipLaunchKernelGGL(k_p2_word_costs<4>, ga, dim3(kThreads), 0, s, wptr, wwt, nnz, v_used, (const float4*)ZW,
                       zw_nq, KP, cost);
  else
    hipLaunchKernelGGL(k_p2_word_costs<8>, ga, dim3(kThreads), 0, s, wptr, wwt, nnz, v_used, (const float4*)ZW,
                       zw_nq, KP, cost);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t itemsB = (n + kItemSlots - 1) / kItemSlots;
  const int gb = persistent_grid((const void*)k_p2_doc_sums, kThreads, 0, (itemsB + 3) / 4);
  if (gb <= 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_p2_doc_sums, dim3(gb), dim3(kThreads), 0, s, xptr, n, winv, cost, out, ld, counters);
  return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void k_max_inplace(float* a, const float* b, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < count) a[i] = fmaxf(a[i], b[i]);
}

hipError_t launch_max_inplace(float* a, const float* b, int64_t count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_max_inplace, dim3((unsigned)((count + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, a, b, count);
  return hipGetLastError();
}

}  // namespace lcemd
