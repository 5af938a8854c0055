// Many instances with few clusters, solved level by level: each step of a
// pass (score, apply, commit) is one launch over all of them, whatever
// their sizes, so that a few instances fill the chip as well as thousands.
//
// One partition's slice of an instance's contingency table is small here, so
// the counts a pass reads are gathered from LDS: the scorer walks the
// partitions, a group of slices at a time in LDS, with one vertex a thread
// and its candidates' sums in registers.  Labels are read as the caller
// laid them out (partition-major, so neighbouring threads read neighbouring
// words), label values serve as table rows, and the distinct candidate
// clusters of a vertex are the bits of a mask: no transposed rows, no hash
// sets, no alignment.
//
// Measured against one workgroup an instance (the persistent launch): 4096
// SBM instances of 200 to 20 000 vertices 155 -> 30 ms, 24 of them
// 48.4 -> 0.90 ms; against the general pass kernels, 1000 vertices alone
// 0.55 -> 0.14 ms, 30 000 with 150 clusters 5.2 to 7.6 -> 1.5 to 2.4 ms (the
// pass count differs between inputs).
#include "multi.h"

namespace mcc {

namespace {

constexpr int32_t kNone = -1;
constexpr int64_t kGainBias = (int64_t)1 << 33;
constexpr int kLeader = 1024;  // threads of the one-workgroup-per-instance kernels

__device__ inline uint64_t owner_key(int64_t gain, int64_t v) {
  return ((uint64_t)(gain + kGainBias) << 31) | (uint64_t)v;
}

// Sum over the workgroup of B threads, valid in every thread.
template <int B, typename T>
__device__ inline T wg_sum(T x) {
  __shared__ T part[B / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
  __syncthreads();
  T r = 0;
#pragma unroll
  for (int j = 0; j < B / 64; ++j) r += part[j];
  return r;
}

// Exclusive scan over the workgroup of B threads.
template <int B>
__device__ inline int32_t wg_excl_scan(int32_t x, int32_t* total) {
  __shared__ int32_t wsum[B / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t v = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  __syncthreads();
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  int32_t off = 0, tot = 0;
#pragma unroll
  for (int j = 0; j < B / 64; ++j) {
    if (j < w) off += wsum[j];
    tot += wsum[j];
  }
  *total = tot;
  return off + v - x;
}

// Addition to a table entry that returns its previous value.  Two int16
// counts share a 32-bit word; an atomic addition to one of them adds to the
// word, shifted to its half: a count never passes 2^15 - 1 or drops below 0
// (an instance has fewer vertices), so no carry or borrow reaches the other.
template <typename T>
__device__ inline int32_t table_add(T* p, int32_t d) {
  if constexpr (sizeof(T) == 4) {
    return atomicAdd(reinterpret_cast<int32_t*>(p), d);
  } else {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    const int sh = (a & 2) ? 16 : 0;
    const int32_t old = atomicAdd(reinterpret_cast<int32_t*>(a & ~(uintptr_t)3),
                                  (int32_t)((uint32_t)d << sh));
    return (int32_t)(int16_t)((uint32_t)old >> sh);
  }
}

// ---------------------------------------------------------------------------
// Clusters and label ranges.  An instance's initial ids are marked in a
// bitmap in LDS; an id's dense cluster index is its rank among the marked
// ones (order of the ids, so tie-breaks are unchanged).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kLeader) void k_multi_ranges(MultiArgs a, const MultiItem* labels) {
  const int t = threadIdx.x;
  if ((int)blockIdx.x >= a.count) {  // one partition's label range
    const MultiItem it = labels[blockIdx.x - a.count];
    const MultiInst& m = a.inst[it.inst];
    const int32_t* p = m.labels[it.part];
    const int64_t n = m.n;
    int32_t hi = -1, lo = 0;
    constexpr int U = 8;
    for (int64_t v = t; v < n; v += U * kLeader) {
      int32_t x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = p[min(v + u * kLeader, n - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        hi = max(hi, x[u]);
        lo = min(lo, x[u]);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      hi = max(hi, __shfl_xor(hi, o, 64));
      lo = min(lo, __shfl_xor(lo, o, 64));
    }
    __shared__ int32_t s_hi, s_lo;
    if (t == 0) {
      s_hi = -1;
      s_lo = 0;
    }
    __syncthreads();
    if ((t & 63) == 0) {
      atomicMax(&s_hi, hi);
      atomicMin(&s_lo, lo);
    }
    __syncthreads();
    if (t == 0) {
      atomicMax(&a.ctl[it.inst].lmax, s_hi);
      if (s_lo < 0) atomicOr(&a.ctl[it.inst].err, kErrNegLabel);
    }
    return;
  }
  constexpr int kWords = (int)(kMultiVertices / 32);
  extern __shared__ uint32_t bits[];  // a bit an id
  __shared__ int32_t rank[kWords];    // marked ids before the word
  const MultiInst& m = a.inst[blockIdx.x];
  MultiCtl& ctl = a.ctl[blockIdx.x];
  const int64_t n = m.n;
  if (!m.init) {
    for (int64_t v = t; v < n && n <= kMultiVertices; v += kLeader) {
      m.C[v] = (uint16_t)v;
      m.rawid[v] = (int32_t)v;
    }
    if (t == 0) ctl.K0 = (int32_t)n;
    return;
  }
  const int words = (int)((n + 31) >> 5);
  for (int j = t; j < words; j += kLeader) bits[j] = 0;
  __syncthreads();
  constexpr int U = 4;
  bool bad = false;
  for (int64_t v = t; v < n; v += U * kLeader) {
    int32_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = m.init[min(v + u * kLeader, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (x[u] < 0 || x[u] >= n) {
        bad = true;
        continue;
      }
      const uint32_t b = 1u << (x[u] & 31);
      if (!(bits[x[u] >> 5] & b)) atomicOr(&bits[x[u] >> 5], b);
    }
  }
  if (__syncthreads_or(bad)) {
    if (t == 0) atomicOr(&ctl.err, kErrInitRange);
    return;
  }
  if (n > kMultiVertices) {  // counted only
    int32_t c = 0;
    for (int j = t; j < words; j += kLeader) c += __popc(bits[j]);
    c = wg_sum<kLeader>(c);
    if (t == 0) ctl.K0 = c;
    return;
  }
  constexpr int W = kWords / kLeader;  // words a thread
  int32_t cnt = 0;
#pragma unroll
  for (int j = 0; j < W; ++j) cnt += t * W + j < words ? __popc(bits[t * W + j]) : 0;
  int32_t total;
  int32_t run = wg_excl_scan<kLeader>(cnt, &total);
#pragma unroll
  for (int j = 0; j < W; ++j) {
    const int w = t * W + j;
    if (w >= words) break;
    rank[w] = run;
    uint32_t b = bits[w];
    while (b) {
      m.rawid[run++] = w * 32 + __ffs(b) - 1;
      b &= b - 1;
    }
  }
  if (t == 0) ctl.K0 = total;
  __syncthreads();
  for (int64_t v = t; v < n; v += U * kLeader) {
    int32_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = m.init[min(v + u * kLeader, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t below = (1u << (x[u] & 31)) - 1;
      if (v + u * kLeader < n)
        m.C[v + u * kLeader] = (uint16_t)(rank[x[u] >> 5] + __popc(bits[x[u] >> 5] & below));
    }
  }
}

// ---------------------------------------------------------------------------
// The slice of one partition: counted in LDS, stored once; the objective's
// terms from the same counts, and from partition 0's also the sizes.  Bound by
// LDS atomics on counts that many labels share (of 4096 instances: LDS busy
// half of the time, 93 % of it conflicts).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_multi_build(MultiArgs a, const MultiItem* parts) {
  extern __shared__ int32_t h[];
  const MultiItem it = parts[blockIdx.x];
  const MultiInst& m = a.inst[it.inst];
  MultiCtl& ctl = a.ctl[it.inst];
  const int t = threadIdx.x;
  const int32_t K0 = m.K0, Ls = m.Ls, cells = K0 * Ls;
  for (int32_t j = t; j < cells; j += kBlock) h[j] = 0;
  __syncthreads();
  const int64_t n = m.n;
  const int32_t* p = m.labels[it.part];
  const uint16_t* C = m.C;
  constexpr int U = 8;
  for (int64_t v0 = t; v0 < n; v0 += U * kBlock) {
    int32_t l[U], c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t v = min(v0 + u * kBlock, n - 1);
      l[u] = p[v];
      c[u] = C[v];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v0 + u * kBlock < n) atomicAdd(&h[l[u] * K0 + c[u]], 1);
  }
  __syncthreads();
  int64_t acc = 0;
  T* N = static_cast<T*>(m.N) + (int64_t)it.part * m.cs;
  for (int32_t j = t; j < cells; j += kBlock) {
    const int32_t c = h[j], l = j / K0;
    N[l * m.rs + (j - l * K0)] = (T)c;
    acc -= 2 * (int64_t)c * c;
  }
  for (int32_t l = t; l < Ls; l += kBlock) {  // label sizes
    int64_t z = 0;
    for (int32_t x = 0; x < K0; ++x) z += h[l * K0 + x];
    acc += z * z;
  }
  if (it.part == 0)
    for (int32_t x = t; x < K0; x += kBlock) {  // cluster sizes
      int64_t z = 0;
      for (int32_t l = 0; l < Ls; ++l) z += h[l * K0 + x];
      m.s[x] = (int32_t)z;
      acc += (int64_t)m.k * z * z;
    }
  acc = wg_sum<kBlock>(acc);
  if (t == 0) atomicAdd((unsigned long long*)&ctl.O, (unsigned long long)acc);
}

// ---------------------------------------------------------------------------
// Score one tile of TB vertices, one a thread.
//  1. Arcs, spread over all threads: the head's cluster sets a bit of the
//     tail's mask (the own cluster, and with it self-loops, left out).
//  2. The agreement sums, over the partitions with a group of table slices
//     at a time in LDS (MODE kRows*, kGather) or from memory (kDirect).
//     kRows*: the thread adds the whole row of its label, the counts of all
//     of up to KX clusters, eight to a 16-byte read; the int16 counts are
//     added as packed halves over two partitions, or four when the instance
//     is small enough for their sum to fit a half, and then into 32-bit sums.
//     kGather, kDirect: one count per candidate, kCand candidates in
//     registers; vertices with more take further rounds over the partitions,
//     from memory.
//  3. The smallest (gain, cluster id); the proposals are appended to the
//     instance's list.
// A label costs 2 K0 bytes of LDS reads in the row modes (a row starts four
// banks after the one before: row strides are odd in 16-byte units), against
// one conflicting read of 64 lanes a candidate of the wave's largest set in
// the gather mode.  Bound by latency with a third to a half of the vector
// issue (rows of 32 and 64 clusters over 1.7 M vertices, tiles of 1024: 0.54
// and 1.33 ms a pass; a wave waits 74 % of its time, the vector units are busy
// 48 and 35 % of theirs, LDS 21 and 17, 7 to 9 % of that conflicts; 27 and 14
// waves a compute unit).
// ---------------------------------------------------------------------------
constexpr int kCand = 16;
enum ScoreMode { kGather = 0, kDirect = kMultiDirect, kRows32 = 2, kRows64 = 3 };

// Copies n16 16-byte words to LDS, four in flight a thread.
template <int TB>
__device__ inline void copy_slices(const int4* __restrict__ src, int4* dst, int32_t n16) {
  for (int32_t j = threadIdx.x; j < n16; j += 4 * TB) {
    int4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = src[min(j + u * TB, n16 - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j + u * TB < n16) dst[j + u * TB] = v[u];
  }
}

template <typename T, int TB, int MODE>
__global__ __launch_bounds__(TB) void k_multi_score(MultiArgs a, const MultiItem* tiles, int words,
                                                    int slice_bytes) {
  extern __shared__ __align__(16) unsigned char smem[];
  int32_t* s_off = reinterpret_cast<int32_t*>(smem);            // TB + 4
  int32_t* s_sz = s_off + TB + 4;                               // kMultiClusters
  uint32_t* s_mask = reinterpret_cast<uint32_t*>(s_sz + kMultiClusters);  // words * TB
  uint16_t* s_c = reinterpret_cast<uint16_t*>(s_mask + words * TB);       // TB
  T* s_tab = reinterpret_cast<T*>(s_c + TB);                    // slice_bytes
  __shared__ int32_t s_base;
  const MultiItem it = tiles[blockIdx.x];
  MultiCtl& ctl = a.ctl[it.inst];
  if (ctl.done || ctl.stage) return;
  const MultiInst& m = a.inst[it.inst];
  const int t = threadIdx.x;
  const int64_t n = m.n, v0 = (int64_t)it.part * TB;
  const int nv = (int)min((int64_t)TB, n - v0);
  const int32_t k = m.k, K0 = m.K0, rs = m.rs;
  const uint16_t* C = m.C;
  const int64_t a0 = m.row_ptr[v0];
  s_off[min(t, nv)] = (int32_t)(m.row_ptr[v0 + min(t, nv)] - a0);
  if (t == 0) s_off[nv] = (int32_t)(m.row_ptr[v0 + nv] - a0);
  const int32_t cv = t < nv ? C[v0 + t] : 0;
  s_c[t] = (uint16_t)cv;
  const int W = (K0 + 31) >> 5;  // at most `words`
  for (int w = 0; w < W; ++w) s_mask[w * TB + t] = 0;
  for (int x = t; x < K0; x += TB) s_sz[x] = m.s[x];
  __syncthreads();
  // ---- candidates ----
  const int32_t A = s_off[nv];
  const int32_t* col = m.col + a0;
  constexpr int U = 4;
  int32_t hn[U];  // the next chunk's heads, loaded while this one is processed
#pragma unroll
  for (int r = 0; r < U; ++r) hn[r] = t * U + r < A ? col[t * U + r] : 0;
  for (int32_t cb = 0; cb < A; cb += TB * U) {
    const int32_t j0 = cb + t * U;
    int32_t hd[U], cu[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      hd[r] = hn[r];
      const int32_t jn = j0 + TB * U + r;
      hn[r] = jn < A ? col[jn] : 0;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) cu[r] = j0 + r < A ? C[hd[r]] : 0;
    if (j0 >= A) continue;
    int lo = 0, hi = nv - 1;  // tail: the last vertex whose row starts at or before j0
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_off[mid] <= j0) lo = mid;
      else hi = mid - 1;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      if (j0 + r >= A) break;
      while (s_off[lo + 1] <= j0 + r) ++lo;
      const int32_t x = cu[r];
      if (x == s_c[lo]) continue;
      uint32_t* w = &s_mask[(x >> 5) * TB + lo];
      const uint32_t b = 1u << (x & 31);
      if (!(*w & b)) atomicOr(w, b);
    }
  }
  __syncthreads();
  int32_t nc = 0;
  for (int w = 0; w < W; ++w) nc += __popc(s_mask[w * TB + t]);
  // ---- sums ----
  const int32_t cs = m.cs;
  const int P = max(1, min(k, (int32_t)(slice_bytes / (int)sizeof(T)) / cs));  // slices a load
  const T* N = static_cast<const T*>(m.N);
  const bool literal = a.literal != 0;
  int32_t bx = kNone;
  int64_t bd = 0;
  const int64_t vt = v0 + min(t, nv - 1);
  constexpr int G = 4;  // partitions whose labels are in flight
  if constexpr (MODE == kRows32 || MODE == kRows64) {
    constexpr int KX = MODE == kRows32 ? 32 : 64;
    const bool any = __any(nc > 0);  // of the wave
    const int units = (K0 + 7) >> 3;
    uint32_t acc[KX];
#pragma unroll
    for (int x = 0; x < KX; ++x) acc[x] = 0;
    int32_t ln[G];
#pragma unroll
    for (int q = 0; q < G; ++q) ln[q] = (nc && q < k) ? m.labels[q][vt] : 0;
    const bool four = n < (1 << 14);  // four counts of at most n fit a half
    for (int32_t i0 = 0; i0 < k; i0 += P) {
      const int32_t np = min(P, k - i0);
      if (i0) __syncthreads();
      copy_slices<TB>(reinterpret_cast<const int4*>(N + (int64_t)i0 * cs),
                      reinterpret_cast<int4*>(s_tab), np * cs / 8);
      __syncthreads();
      if (!any) continue;
      for (int32_t g = 0; g < np; g += G) {
        int32_t l[G];
#pragma unroll
        for (int q = 0; q < G; ++q) l[q] = ln[q];
        const int32_t left = np - g, nx = i0 + g + min(G, left);
#pragma unroll
        for (int q = 0; q < G; ++q) ln[q] = (nc && nx + q < k) ? m.labels[nx + q][vt] : 0;
        const uint4* row[G];
#pragma unroll
        for (int q = 0; q < G; ++q)
          row[q] = reinterpret_cast<const uint4*>(s_tab + (g + min(q, left - 1)) * cs + l[q] * rs);
#pragma unroll
        for (int j = 0; j < KX / 8; ++j) {
          if (j < units) {
          auto flush = [&](const uint4& p) {
            acc[8 * j + 0] += p.x & 0xffff;
            acc[8 * j + 1] += p.x >> 16;
            acc[8 * j + 2] += p.y & 0xffff;
            acc[8 * j + 3] += p.y >> 16;
            acc[8 * j + 4] += p.z & 0xffff;
            acc[8 * j + 5] += p.z >> 16;
            acc[8 * j + 6] += p.w & 0xffff;
            acc[8 * j + 7] += p.w >> 16;
          };
          uint4 p = row[0][j];
          if (left > 1) {
            const uint4 r = row[1][j];
            p.x += r.x; p.y += r.y; p.z += r.z; p.w += r.w;
          }
          if (left > 2) {
            uint4 r = row[2][j];
            if (left > 3) {
              const uint4 z = row[3][j];
              r.x += z.x; r.y += z.y; r.z += z.z; r.w += z.w;
            }
            if (four) {
              p.x += r.x; p.y += r.y; p.z += r.z; p.w += r.w;
            } else {
              flush(r);
            }
          }
          flush(p);
          }
        }
      }
    }
    uint32_t own = 0;
#pragma unroll
    for (int x = 0; x < KX; ++x) own = x == cv ? acc[x] : own;
    const uint32_t m0 = s_mask[t], m1 = (KX > 32 && W > 1) ? s_mask[TB + t] : 0u;
#pragma unroll
    for (int x = 0; x < KX; ++x) {
      if (((x < 32 ? m0 >> (x & 31) : m1 >> (x & 31)) & 1)) {  // only clusters below K0
        int64_t d = 2 * ((int64_t)own - acc[x]) + (int64_t)k * ((int64_t)s_sz[x] - s_sz[cv] - 1);
        if (literal) d += k;
        if (bx == kNone || d < bd) {
          bd = d;
          bx = x;
        }
      }
    }
  } else {
    int32_t s_own = 0;
    int cw = 0;                // the mask word the thread is at
    uint32_t cb = s_mask[t];   // and its bits not taken yet
    for (int32_t done = 0;; done += kCand) {
      const bool lds = MODE == kGather && done == 0;
      if (!lds && !__any(done < nc)) break;
      const int32_t mine = max(0, min(kCand, nc - done));
      int32_t xs[kCand], S[kCand];
#pragma unroll
      for (int c = 0; c < kCand; ++c) {
        xs[c] = cv;
        S[c] = 0;
        if (c < mine) {
          while (!cb) cb = s_mask[++cw * TB + t];
          xs[c] = cw * 32 + __ffs(cb) - 1;
          cb &= cb - 1;
        }
      }
      int32_t most = mine;  // of the wave
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
      most = __builtin_amdgcn_readfirstlane(most);
      int32_t own = 0;
      int32_t ln[G];
#pragma unroll
      for (int q = 0; q < G; ++q) ln[q] = (mine && q < k) ? m.labels[q][vt] : 0;
      const int step = lds ? P : k;
      for (int32_t i0 = 0; i0 < k; i0 += step) {
        const int32_t np = min(step, k - i0);
        if (lds) {
          if (i0) __syncthreads();
          copy_slices<TB>(reinterpret_cast<const int4*>(N + (int64_t)i0 * cs),
                          reinterpret_cast<int4*>(s_tab), np * cs / (int32_t)(16 / sizeof(T)));
          __syncthreads();
        }
        if (!most) continue;
        for (int32_t g = 0; g < np; g += G) {
          int32_t l[G];
#pragma unroll
          for (int q = 0; q < G; ++q) l[q] = ln[q];
          const int32_t left = np - g, nx = i0 + g + min(G, left);
#pragma unroll
          for (int q = 0; q < G; ++q) ln[q] = (mine && nx + q < k) ? m.labels[nx + q][vt] : 0;
          // one partition's counts at a time, all of them in flight
          // (32-bit byte offsets from a uniform base, so that a lane holds one
          // register an address)
          auto add = [&](const T* tab, uint32_t row) {
            const char* base = reinterpret_cast<const char*>(tab);
            auto at = [&](int32_t x) -> int32_t {
              return *reinterpret_cast<const T*>(base + (row + (uint32_t)x) * (uint32_t)sizeof(T));
            };
            int32_t got[kCand + 1];
            got[kCand] = at(cv);
#pragma unroll
            for (int c = 0; c < kCand; ++c) got[c] = c < most ? at(xs[c]) : 0;
            own += got[kCand];
#pragma unroll
            for (int c = 0; c < kCand; ++c) S[c] += got[c];
          };
#pragma unroll
          for (int q = 0; q < G; ++q) {
            if (q < left) {
              const uint32_t row = (uint32_t)l[q] * (uint32_t)rs;
              if (lds) add(s_tab + (g + q) * cs, row);
              else add(N + (int64_t)(i0 + g + q) * cs, row);
              __builtin_amdgcn_sched_barrier(0);  // registers of one partition's counts
            }
          }
        }
      }
      if (done == 0) s_own = own;
#pragma unroll
      for (int c = 0; c < kCand; ++c) {
        if (c >= mine) break;
        int64_t d = 2 * ((int64_t)s_own - S[c]) +
                    (int64_t)k * ((int64_t)s_sz[xs[c]] - s_sz[cv] - 1);
        if (literal) d += k;
        if (bx == kNone || d < bd) {  // candidates come in increasing id
          bd = d;
          bx = xs[c];
        }
      }
    }
  }
  const bool p = bx != kNone && bd < 0;
  int32_t total;
  const int32_t off = wg_excl_scan<TB>(p ? 1 : 0, &total);
  const int32_t evals = wg_sum<TB>(nc);  // at most TB * 256
  const int32_t bnd = wg_sum<TB>(nc > 0 ? 1 : 0);
  if (t == 0) {
    s_base = total ? atomicAdd(&ctl.nprop, total) : 0;
    if (evals) atomicAdd((unsigned long long*)&ctl.pass_evals, (unsigned long long)evals);
    if (bnd) atomicAdd((unsigned long long*)&ctl.pass_boundary, (unsigned long long)bnd);
  }
  __syncthreads();
  if (p) {
    m.plist[s_base + off] = make_int2((int32_t)(v0 + t), bx);
    m.dprop[s_base + off] = bd;
  }
}

// ---------------------------------------------------------------------------
// The owner of every cluster that a proposal touches: its smallest
// (gain, vertex) proposer, elected in LDS by the whole workgroup of B
// threads.  Only a key below the one that is there asks for the word.
// ---------------------------------------------------------------------------
template <int B>
__device__ inline void elect_owners(const MultiInst& m, int32_t np, uint64_t* s_owner) {
  for (int x = threadIdx.x; x < m.K0; x += B) s_owner[x] = ~0ull;
  __syncthreads();
  for (int32_t e = threadIdx.x; e < np; e += B) {
    const int2 q = m.plist[e];
    const uint64_t key = owner_key(m.dprop[e], q.x);
    const int32_t pair[2] = {(int32_t)m.C[q.x], q.y};
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (key < s_owner[pair[j]])
        atomicMin((unsigned long long*)&s_owner[pair[j]], (unsigned long long)key);
  }
  __syncthreads();
}

// Whether proposal e (vertex q.x from `from` to q.y) owns both its clusters.
__device__ inline bool owns_both(const MultiInst& m, const uint64_t* s_owner, int32_t e,
                                 const int2& q, int32_t from) {
  const uint64_t key = owner_key(m.dprop[e], q.x);
  return s_owner[from] == key && s_owner[q.y] == key;
}

// ---------------------------------------------------------------------------
// Apply the proposals to one partition's slice, which the workgroup owns:
// the changes gathered in LDS and added once, or, when they are few against
// the slice, added directly.  A net change d of a count whose previous value
// is `old` changes its square by 2 old d + d^2; partition 0's workgroup
// does the sizes.  In the second slot of a pass that falls back the proposals
// that do not own both their clusters are taken out again in the same way.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_multi_apply(MultiArgs a, const MultiItem* parts) {
  extern __shared__ int32_t h[];
  __shared__ int32_t s_d[kMultiClusters];
  __shared__ uint64_t s_owner[kMultiClusters];
  const MultiItem it = parts[blockIdx.x];
  MultiCtl& ctl = a.ctl[it.inst];
  if (ctl.done) return;
  const int32_t np = ctl.nprop;
  if (np == 0) return;
  const MultiInst& m = a.inst[it.inst];
  const int t = threadIdx.x;
  const bool undo = ctl.stage != 0;
  const int32_t K0 = m.K0, rs = m.rs, cells = K0 * m.Ls;
  const int32_t* lab = m.labels[it.part];
  T* N = static_cast<T*>(m.N) + (int64_t)it.part * m.cs;
  const bool sizes = it.part == 0;
  int64_t dn2 = 0, ds2 = 0;
  if (undo) elect_owners<kBlock>(m, np, s_owner);
  const bool few = np < cells / 64;
  if (!few)
    for (int32_t j = t; j < cells; j += kBlock) h[j] = 0;
  if (sizes)
    for (int x = t; x < K0; x += kBlock) s_d[x] = 0;
  __syncthreads();
  const int32_t d = undo ? -1 : 1;
  constexpr int U = 4;  // proposals in flight a thread
  for (int32_t e0 = t; e0 < np; e0 += U * kBlock) {
    int2 q[U];
    int32_t from[U], l[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = m.plist[min(e0 + u * kBlock, np - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      from[u] = m.C[q[u].x];
      l[u] = lab[q[u].x];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t e = e0 + u * kBlock;
      if (e >= np || (undo && owns_both(m, s_owner, e, q[u], from[u]))) continue;
      const int32_t to = q[u].y;
      if (few) {
        const int32_t o1 = table_add(N + l[u] * rs + to, d),
                      o2 = table_add(N + l[u] * rs + from[u], -d);
        dn2 += 2 * (int64_t)o1 * d + 1 - 2 * (int64_t)o2 * d + 1;
      } else {
        atomicAdd(&h[l[u] * K0 + to], d);
        atomicAdd(&h[l[u] * K0 + from[u]], -d);
      }
      if (sizes) {
        atomicAdd(&s_d[to], d);
        atomicAdd(&s_d[from[u]], -d);
      }
    }
  }
  __syncthreads();
  if (!few)
    for (int32_t j = t; j < cells; j += kBlock) {
      const int32_t c = h[j];
      if (!c) continue;
      const int32_t x = j / K0;
      T* cell = N + x * rs + (j - x * K0);
      const int32_t old = *cell;
      *cell = (T)(old + c);
      dn2 += 2 * (int64_t)old * c + (int64_t)c * c;
    }
  if (sizes)
    for (int x = t; x < K0; x += kBlock) {
      const int32_t c = s_d[x];
      if (!c) continue;
      const int32_t old = m.s[x];
      m.s[x] = old + c;
      ds2 += 2 * (int64_t)old * c + (int64_t)c * c;
    }
  dn2 = wg_sum<kBlock>(dn2);
  if (t == 0 && dn2) atomicAdd((unsigned long long*)&ctl.dN2, (unsigned long long)dn2);
  if (sizes) {
    ds2 = wg_sum<kBlock>(ds2);
    if (t == 0) ctl.dS2 += ds2;
  }
}

// ---------------------------------------------------------------------------
// End of an instance's slot, by one workgroup: keep the batch if it lowered
// the objective, else leave it to a second slot, whose apply takes out the
// proposals that do not own both their clusters and which commits the others;
// account the pass; write the output of a finished instance.
//
// The batch is taken out by all workgroups of the apply: by this one alone a
// pass of 20 000 vertices and 256 partitions that fell back took 26 ms, with
// the second slot 0.28.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kLeader) void k_multi_commit(MultiArgs a, const int32_t* ids) {
  __shared__ uint64_t s_owner[kMultiClusters];
  const int32_t id = ids[blockIdx.x];
  MultiCtl& ctl = a.ctl[id];
  if (ctl.done) return;
  const MultiInst& m = a.inst[id];
  const int t = threadIdx.x;
  const int32_t np = ctl.nprop;
  const int32_t passes = ctl.passes + 1;
  const bool fell = ctl.stage != 0;
  const int64_t dO = (int64_t)m.k * ctl.dS2 - 2 * ctl.dN2;
  const int64_t O0 = ctl.O;
  int64_t O = O0, moved = 0;
  __syncthreads();  // the counters are read
  if (np > 0 && dO >= 0 && !fell) {
    if (t == 0) ctl.stage = 1;
    return;
  }
  if (fell) {
    elect_owners<kLeader>(m, np, s_owner);
    int32_t com = 0;
    for (int32_t e = t; e < np; e += kLeader) {
      const int2 q = m.plist[e];
      if (!owns_both(m, s_owner, e, q, m.C[q.x])) continue;
      m.C[q.x] = (uint16_t)q.y;
      ++com;
    }
    moved = wg_sum<kLeader>(com);
    O += dO;
  } else if (np > 0) {
    for (int32_t e = t; e < np; e += kLeader) {
      const int2 q = m.plist[e];
      m.C[q.x] = (uint16_t)q.y;
    }
    O += dO;
    moved = np;
  }
  const bool done = np == 0 || passes >= a.max_rounds;
  int32_t clusters = 0;
  if (done) {
    __syncthreads();
    for (int64_t v = t; v < m.n; v += kLeader) m.out[v] = m.rawid[m.C[v]];
    for (int32_t x = t; x < m.K0; x += kLeader)
      clusters += __hip_atomic_load(&m.s[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0;
    clusters = wg_sum<kLeader>(clusters);
  }
  __syncthreads();
  if (t == 0) {
    if (ctl.passes == 0) ctl.O0 = O0;
    if (a.trace) {
      int64_t* r = a.trace + (int64_t)(passes - 1) * 4;
      r[0] = np;
      r[1] = moved;
      r[2] = fell;
      r[3] = O;
    }
    ctl.passes = passes;
    ctl.evals += ctl.pass_evals;
    ctl.boundary += ctl.pass_boundary;
    ctl.moves += moved;
    ctl.fallback_rounds += fell;
    ctl.O = O;
    ctl.nprop = 0;
    ctl.stage = 0;
    ctl.pass_evals = 0;
    ctl.pass_boundary = 0;
    ctl.dN2 = 0;
    ctl.dS2 = 0;
    if (np == 0) ctl.converged = 1;
    if (done) {
      ctl.clusters = clusters;
      ctl.done = 1;
    }
  }
}

// ---------------------------------------------------------------------------
// Evaluation of one small partition.
// ---------------------------------------------------------------------------
__device__ inline double xlogx(int32_t c) { return c > 0 ? (double)c * log((double)c) : 0.0; }

// Sum over a workgroup of kBlock threads as the comparison kernels take it
// (the order fixes the bits of a floating-point sum).
__device__ inline double block_total(double x, double* part) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
  __syncthreads();
  double t = 0;
#pragma unroll
  for (int j = 0; j < kBlock / 64; ++j) t += part[j];
  __syncthreads();
  return t;
}

// sum over j < len of f(j) in the order of a grid of len / (4 kBlock)
// workgroups striding over len, their sums then added up by one workgroup:
// the same bits as the general comparison gives
template <typename F>
__device__ inline double grid_order_sum(int64_t len, F&& f, double* part) {
  const int t = threadIdx.x;
  const int nb = (int)max((int64_t)1, min((int64_t)2048, (len + 4 * kBlock - 1) / (4 * kBlock)));
  double mine = 0.0;  // thread t adds the sums of the grid's workgroups t, t + kBlock, ...
  for (int b = 0; b < nb; ++b) {
    double acc = 0.0;
    for (int64_t j = (int64_t)b * kBlock + t; j < len; j += (int64_t)nb * kBlock) acc += f(j);
    acc = block_total(acc, part);
    if (b % kBlock == t) mine += acc;
  }
  return block_total(mine, part);
}

// Label values that do not occur are left out, as the general comparison's
// dense ids leave them out (compared there instead, a small call with gaps in
// its labels took 0.47 ms, 0.36 before this kernel, and takes 0.09 here).
__global__ __launch_bounds__(kBlock) void k_multi_compare(MultiArgs a, MultiCompare* out) {
  __shared__ double part[kBlock / 64];
  extern __shared__ int32_t s_col[];  // Ls sums, then the Ls values that occur
  const MultiInst& m = a.inst[0];
  const int t = threadIdx.x;
  const int32_t K0 = m.K0, Ls = m.Ls, rs = m.rs;
  const bool wide = m.n >= (1 << 15);
  auto at = [&](int32_t x, int32_t l) -> int32_t {
    return wide ? static_cast<const int32_t*>(m.N)[l * rs + x]
                : (int32_t)static_cast<const int16_t*>(m.N)[l * rs + x];
  };
  int64_t rowmax = 0, colmax = 0;
  for (int32_t x = t; x < K0; x += kBlock) {
    int32_t best = 0;
    for (int32_t l = 0; l < Ls; ++l) best = max(best, at(x, l));
    rowmax += best;
  }
  uint16_t* s_val = reinterpret_cast<uint16_t*>(s_col + Ls);
  for (int32_t l = t; l < Ls; l += kBlock) {
    int32_t best = 0, sum = 0;
    for (int32_t x = 0; x < K0; ++x) {
      const int32_t c = at(x, l);
      best = max(best, c);
      sum += c;
    }
    colmax += best;
    s_col[l] = sum;
  }
  __syncthreads();
  int32_t Lb = 0;  // values that occur
  for (int32_t l0 = 0; l0 < Ls; l0 += kBlock) {
    const int32_t l = l0 + t;
    const bool occurs = l < Ls && s_col[l] > 0;
    int32_t total;
    const int32_t e = wg_excl_scan<kBlock>(occurs ? 1 : 0, &total);
    if (occurs) s_val[Lb + e] = (uint16_t)l;
    Lb += total;
  }
  __syncthreads();
  rowmax = wg_sum<kBlock>(rowmax);
  colmax = wg_sum<kBlock>(colmax);
  const double cells = grid_order_sum(
      (int64_t)K0 * Lb,
      [&](int64_t j) {
        const int32_t x = (int32_t)(j / Lb);
        return xlogx(at(x, s_val[j - (int64_t)x * Lb]));
      },
      part);
  const double rows = grid_order_sum(K0, [&](int64_t x) { return xlogx(m.s[x]); }, part);
  const double cols = grid_order_sum(Lb, [&](int64_t l) { return xlogx(s_col[s_val[l]]); }, part);
  if (t == 0) *out = MultiCompare{rowmax, colmax, cells, rows, cols, Lb, 0};
}

// The smallest vertex of every id is found in LDS; then the vertices are
// walked in order, those that are the first of their id counted by a scan,
// and an id's entry becomes the complement of its rank (negative, so that it
// is no vertex).
__global__ __launch_bounds__(kLeader) void k_multi_canonical(const int32_t* in, int32_t n,
                                                             int32_t* out, int32_t* total) {
  extern __shared__ int32_t first[];  // n
  const int t = threadIdx.x;
  for (int32_t x = t; x < n; x += kLeader) first[x] = 0x7fffffff;
  __syncthreads();
  bool bad = false;
  for (int32_t v = t; v < n; v += kLeader) {
    const int32_t x = in[v];
    if (x < 0 || x >= n) bad = true;
    else if (first[x] > v) atomicMin(&first[x], v);
  }
  if (__syncthreads_or(bad)) {
    if (t == 0) *total = -1;
    return;
  }
  int32_t seen = 0;
  for (int32_t v0 = 0; v0 < n; v0 += kLeader) {
    const int32_t v = v0 + t, x = v < n ? in[v] : 0;
    const bool lead = v < n && first[x] == v;
    int32_t tot;
    const int32_t e = wg_excl_scan<kLeader>(lead ? 1 : 0, &tot);
    if (lead) first[x] = ~(seen + e);
    seen += tot;
    __syncthreads();
  }
  for (int32_t v = t; v < n; v += kLeader) out[v] = ~first[in[v]];
  if (t == 0) *total = seen;
}

}  // namespace

void launch_multi_compare(const MultiArgs& a, int32_t Ls, MultiCompare* out, hipStream_t st) {
  k_multi_compare<<<1, kBlock, 6 * (size_t)Ls, st>>>(a, out);
}

void launch_multi_canonical(const int32_t* in, int64_t n, int32_t* out, int32_t* total,
                            hipStream_t st) {
  k_multi_canonical<<<1, kLeader, 4 * (size_t)n, st>>>(in, (int32_t)n, out, total);
}

size_t multi_score_lds(int tile, int words, size_t slice_bytes) {
  return 4 * (size_t)(tile + 4) + 4 * (size_t)kMultiClusters + 4 * (size_t)words * tile +
         2 * (size_t)tile + slice_bytes;
}

void launch_multi_ranges(const MultiArgs& a, const MultiItem* labels, int32_t nlabels,
                         int64_t n_max, hipStream_t st) {
  const size_t lds = 4 * (size_t)((n_max + 31) / 32);
  k_multi_ranges<<<a.count + nlabels, kLeader, lds, st>>>(a, labels);
}

void launch_multi_build(const MultiArgs& a, const MultiItem* parts, int32_t nparts, bool wide,
                        int32_t cells_max, hipStream_t st) {
  if (nparts <= 0) return;
  const size_t lds = 4 * (size_t)cells_max;
  if (wide) k_multi_build<int32_t><<<nparts, kBlock, lds, st>>>(a, parts);
  else k_multi_build<int16_t><<<nparts, kBlock, lds, st>>>(a, parts);
}

template <typename T, int TB>
static void launch_score_mode(const MultiArgs& a, const MultiItem* tiles, int32_t ntiles, int mode,
                              int words, size_t slice_bytes, hipStream_t st) {
  const size_t lds = multi_score_lds(TB, words, slice_bytes);
  const int sb = (int)slice_bytes;
  if (mode == kDirect) {
    k_multi_score<T, TB, kDirect><<<ntiles, TB, lds, st>>>(a, tiles, words, sb);
  } else if (mode == kGather) {
    k_multi_score<T, TB, kGather><<<ntiles, TB, lds, st>>>(a, tiles, words, sb);
  } else if constexpr (sizeof(T) == 2) {
    if (mode == kRows32)
      k_multi_score<T, TB, kRows32><<<ntiles, TB, lds, st>>>(a, tiles, words, sb);
    else
      k_multi_score<T, TB, kRows64><<<ntiles, TB, lds, st>>>(a, tiles, words, sb);
  }
}

// How an instance is scored.  Rows while a row has at most 64 int16 counts.
// Else gathers: from LDS where a slice is small against its tile (up to
// 64 KiB for 1024 vertices, 8 KiB for 256), from memory above that.
int multi_score_mode(int32_t K0, int32_t cs, bool wide, int tile) {
  const size_t slice = (size_t)cs * (wide ? 4 : 2);
  if (slice > (tile == 1024 ? (size_t)65536 : (size_t)8192)) return kDirect;
  if (wide || K0 > 64) return kGather;
  return K0 <= 32 ? kRows32 : kRows64;
}

void launch_multi_score(const MultiArgs& a, const MultiItem* tiles, int32_t ntiles, bool wide,
                        int mode, int tile, int words, size_t slice_bytes, hipStream_t st) {
  if (ntiles <= 0) return;
  if (tile == 256) {
    if (wide) launch_score_mode<int32_t, 256>(a, tiles, ntiles, mode, words, slice_bytes, st);
    else launch_score_mode<int16_t, 256>(a, tiles, ntiles, mode, words, slice_bytes, st);
  } else {
    if (wide) launch_score_mode<int32_t, 1024>(a, tiles, ntiles, mode, words, slice_bytes, st);
    else launch_score_mode<int16_t, 1024>(a, tiles, ntiles, mode, words, slice_bytes, st);
  }
}

void launch_multi_apply(const MultiArgs& a, const MultiItem* parts, int32_t nparts, bool wide,
                        int32_t cells_max, hipStream_t st) {
  if (nparts <= 0) return;
  const size_t lds = 4 * (size_t)cells_max;
  if (wide) k_multi_apply<int32_t><<<nparts, kBlock, lds, st>>>(a, parts);
  else k_multi_apply<int16_t><<<nparts, kBlock, lds, st>>>(a, parts);
}

void launch_multi_commit(const MultiArgs& a, const int32_t* ids, int32_t nids, hipStream_t st) {
  if (nids > 0) k_multi_commit<<<nids, kLeader, 0, st>>>(a, ids);
}

}  // namespace mcc
