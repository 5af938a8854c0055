// One synchronous pass of the greedy consensus (Methods, "Graph-aware
// consensus clustering" and "Parallel algorithm"):
//
//   score      every vertex, against the frozen partition, finds the
//              neighbour cluster with the smallest (gain, cluster id) and
//              proposes it when the gain is negative (Eq. objective3/4)
//   props      list the proposals; its last workgroup counts the pass and
//              stops the solve if there are none
//   apply      apply every proposal to sizes and counts, measuring the exact
//              change of the objective on the way; its last workgroup keeps
//              the batch if the objective dropped, else lets it fall back
//   commit     write the new cluster ids, or (fallback) undo the batch and
//              elect an owner per touched cluster; its last workgroup
//              accounts the pass and enforces the pass cap
//
// A pass that falls back takes a second slot of the same launches, in which
// only fallback and commit work: fallback applies the proposals that own both
// their clusters, commit releases the owners and writes the committed cluster
// ids.
//
// Every kernel returns at once when the control block says the solve is
// done, so the host may enqueue slots ahead of the device.  The control
// steps ride on the last workgroup of a kernel (a ticket counter: nothing
// waits) because a launch of its own costs about 4 us each.
//
// Gain of moving v from c to x (exact, the pair (v, v) left out):
//   2 (S_c(v) - S_x(v)) + k (s_x - s_c - 1),  S_y(v) = sum_i N_i(y, P_i(v)),
// obtained from Eq. objective3 by summing (k - 2 delta_uv) over the members
// of a cluster: delta_uv = k - #partitions agreeing on u, v, so the sum over
// y is 2 S_y(v) - k s_y.
//
// Objective bookkeeping: O = k sum_x s_x^2 + sum_i sum_l |P_i l|^2
// - 2 sum_i sum_(x,l) N_i(x,l)^2.  Each +-1 atomic update of a counter that
// returns the previous value `old` changes that counter's square by
// 2 old d + 1; summed over all updates of a pass this telescopes to the
// exact change of the sum of squares whatever order the atomics land in, so
// the batch's objective change is exact and deterministic.
#include <algorithm>

#include "impl.h"

namespace mcc {

namespace {

constexpr int32_t kNone = -1;
constexpr int64_t kGainBias = (int64_t)1 << 33;

__device__ inline uint64_t owner_key(int64_t gain, int64_t v) {
  // (gain, vertex) ordered lexicographically; gain lies in (-2^33, 0) and
  // v in [0, 2^31)
  return ((uint64_t)(gain + kGainBias) << 31) | (uint64_t)v;
}

template <int G>
__device__ inline int32_t group_min(int32_t x) {
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) x = min(x, __shfl_xor(x, o, G));
  return x;
}

template <int G>
__device__ inline int32_t group_sum(int32_t x) {
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, G);
  return x;
}

// Exclusive prefix sum over the wave's lanes; *total: the wave's sum.
__device__ inline int32_t wave_excl_scan(int32_t x, int32_t* total) {
  const int lane = threadIdx.x & 63;
  int32_t s = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(s, o, 64);
    if (lane >= o) s += y;
  }
  *total = __shfl(s, 63, 64);
  return s - x;
}

__device__ inline int64_t wave_sum64(int64_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

__device__ inline int32_t wave_sum32(int32_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Add the workgroup's totals of the pass counters (all threads call; one
// atomic per counter and workgroup).
template <int B = kBlock>
__device__ inline void flush_counts(const PassArgs& a, int64_t evals, int64_t nprop,
                                    int64_t boundary, int64_t skipped, int64_t wide = 0) {
  __shared__ int64_t red[kPassCounters][B / 64];
  const int64_t v[kPassCounters] = {evals, nprop, boundary, skipped, wide};
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < kPassCounters; ++c) {
    const int64_t x = wave_sum64(v[c]);
    if (lane == 0) red[c][w] = x;
  }
  __syncthreads();
  if (threadIdx.x < kPassCounters) {
    int64_t tot = 0;
#pragma unroll
    for (int j = 0; j < B / 64; ++j) tot += red[threadIdx.x][j];
    if (tot) atomicAdd((unsigned long long*)&a.pc[threadIdx.x * kCounterStride],
                       (unsigned long long)tot);
  }
}

// ---------------------------------------------------------------------------
// score: G lanes per vertex.  A lane keeps R neighbour cluster ids and the
// labels of up to KR partitions in registers; larger degrees or k fall back
// to re-reading memory.  Candidates are enumerated in increasing id by
// repeated group minima, so duplicates vanish and ties resolve to the
// smallest id without any sort.
// ---------------------------------------------------------------------------
constexpr int kMaxLdsPart = 256;  // partitions whose table geometry sits in LDS
// Candidates a vertex above which a pass counts as one for the wave-per-vertex
// scorer (three quarters of the 32 that the key sets of 64-vertex tiles hold).
constexpr int kTileCandAvg = 24;
constexpr int kCandSetBits = 8;   // deferred vertex: LDS set of its candidate clusters
constexpr int kCandSet = 1 << kCandSetBits;

// Ids that agree in 16 bytes of two compact label rows: zero bytes (halves)
// of the exclusive or.
__device__ inline int32_t zeros8(uint32_t x) {
  return __popc(~((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) | 0x7f7f7f7fu));
}
__device__ inline int32_t zeros16(uint32_t x) {
  return __popc(~((((x & 0x7fff7fffu) + 0x7fff7fffu) | x) | 0x7fff7fffu));
}
__device__ inline int32_t agree8(const uint4& a, const uint4& b) {
  return zeros8(a.x ^ b.x) + zeros8(a.y ^ b.y) + zeros8(a.z ^ b.z) + zeros8(a.w ^ b.w);
}
__device__ inline int32_t agree16(const uint4& a, const uint4& b) {
  return zeros16(a.x ^ b.x) + zeros16(a.y ^ b.y) + zeros16(a.z ^ b.z) + zeros16(a.w ^ b.w);
}

// MEM: hashed tables, whose small clusters are scored from member rows.
template <int G, bool LIST, bool MEM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_score(PassArgs a) {
  if (a.ctl->done || a.ctl->stage) return;
  // LIST: the vertices the tiled or list scorer deferred or, in a dense pass
  // the tiled scorer leaves to this kernel (defer_all), every vertex to
  // score: the rescoring list, or all vertices when there is none
  const bool all = LIST && a.ctl->defer_all && !(a.st && a.ctl->rescore_count <= a.sparse_max);
  const int64_t count =
      !LIST ? a.n : (all ? (a.st ? (int64_t)a.ctl->rescore_count : a.n) : (int64_t)a.ctl->heavy_count);
  if (LIST && count == 0) return;
  // arcs per lane held in registers; the deferred-vertex scorer (one wave
  // per vertex) holds 512, for the highest degrees
  constexpr int R = (LIST && G == 64) ? 8 : ((128 / G) < 16 ? ((128 / G) > 1 ? (128 / G) : 1) : 16);
  constexpr int KR = (64 / G) > 1 ? (64 / G) : 1;  // labels held per lane
  constexpr int32_t kInf = 0x7fffffff;
  __shared__ int64_t s_toff[kMaxLdsPart];
  __shared__ int32_t s_L[kMaxLdsPart];
  // deferred-vertex scorer, per wave: items' first member pair, sums, member
  // list starts, clusters, and the items of clusters without member lists
  constexpr int kW = (LIST && G == 64) ? kBlock / 64 : 1;
  constexpr int kI = (LIST && G == 64 && MEM) ? 130 : 1;
  __shared__ int32_t s_ioff[kW][kI], s_imst[kW][kI], s_iy[kW][kI], s_ilarge[kW][kI];
  __shared__ int32_t s_isum[kW][(LIST && G == 64) ? kCandSet + 2 : 1];
  __shared__ __align__(8) int32_t s_vrow[kW][(LIST && G == 64 && MEM) ? 64 : 2];
  __shared__ int32_t s_cset[kW][(LIST && G == 64) ? kCandSet : 1];
  __shared__ int32_t s_cnb[kW][(LIST && G == 64) ? kCandSet : 1];  // a neighbour in the cluster
  __shared__ int32_t s_clist[kW][(LIST && G == 64) ? kCandSet : 1];
  __shared__ int32_t s_cnbl[kW][(LIST && G == 64) ? 128 : 1];
  __shared__ int32_t s_ccount[kW];
  const int lane = threadIdx.x & (G - 1);
  const int64_t group = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G;
  const int64_t ngroups = ((int64_t)gridDim.x * kBlock) / G;
  const int32_t k = a.k;
  const bool kfits = k <= KR * G;
  for (int i = threadIdx.x; i < k && i < kMaxLdsPart; i += kBlock) {
    s_toff[i] = a.t.interleaved ? 0 : a.t.toff[i];  // no offsets when interleaved
    s_L[i] = a.t.L[i];
  }
  __syncthreads();
  const bool lds_geom = k <= kMaxLdsPart;

  int64_t evals = 0;
  int32_t nprop = 0, boundary = 0, wide = 0;
  for (int64_t idx = group; idx < count; idx += ngroups) {
    const int64_t v = !LIST ? idx : (all ? (a.st ? (int64_t)a.rlist[idx] : idx) : (int64_t)a.heavy[idx]);
    const int32_t cv = a.C[v];
    const int64_t beg = a.row_ptr[v], end = a.row_ptr[v + 1];
    const bool fits = end - beg <= (int64_t)G * R;
    int32_t x[R];
    if (fits) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        int64_t j = beg + r * G + lane;
        x[r] = kInf;
        if (j < end) {
          // a self-loop points at v's own cluster and drops out with it
          const int32_t cu = a.ac ? a.ac[j] : cn_load(a, a.col[j]);
          if (cu != cv) x[r] = cu;
        }
      }
    }
    // the label row is read only once the vertex has a candidate: interior
    // vertices (every neighbour in their own cluster) never touch it
    const int32_t* row = a.Lvm + v * k;
    int32_t lab[KR];
    bool have_row = false;
    auto load_row = [&]() {
      if (kfits && !have_row) {
#pragma unroll
        for (int t = 0; t < KR; ++t) {
          int i = lane + t * G;
          lab[t] = i < k ? row[i] : 0;
        }
      }
      have_row = true;
    };
    // S_y(v) summed over the group's lanes
    auto agree = [&](int32_t y) -> int32_t {
      int32_t sum = 0;
      if (MEM && a.s[y] <= a.msum_max) {
        // S_y(v) = sum over members u of y of the partitions agreeing on u, v;
        // the member ids are read once, one per lane, and broadcast
        const int32_t cnt = a.s[y], b = a.mstart[y];
        for (int32_t m0 = 0; m0 < cnt; m0 += G) {
          const int32_t mid = m0 + lane < cnt ? a.members[b + m0 + lane] : 0;
          const int32_t mc = min(G, cnt - m0);
          for (int32_t j = 0; j < mc; ++j) {
          const int32_t* ru = a.Lvm + (int64_t)__shfl(mid, j, G) * k;
          if (kfits) {
#pragma unroll
            for (int t = 0; t < KR; ++t) {
              int i = lane + t * G;
              if (i < k) sum += ru[i] == lab[t];
            }
          } else {
            for (int i = lane; i < k; i += G) sum += ru[i] == row[i];
          }
          }
        }
      } else if (a.t.hashed) {
        const uint64_t ky = (uint64_t)(uint32_t)y << 32;
        if (kfits && a.t.rows) {
#pragma unroll
          for (int t = 0; t < KR; ++t) {
            int i = lane + t * G;
            if (i < k) sum += hcount(a.t, i, y, lab[t]);
          }
        } else if (kfits) {  // implies lds_geom
#pragma unroll
          for (int t = 0; t < KR; ++t) {
            int i = lane + t * G;
            if (i < k) sum += hget(a.t, ky | (uint64_t)(s_toff[i] + lab[t]));
          }
        } else {
          for (int i = lane; i < k; i += G) sum += count_of(a.t, i, y, row[i]);
        }
      } else if (a.t.interleaved) {
        const int64_t base = (int64_t)y * a.t.Lmax;
        if (kfits) {
#pragma unroll
          for (int t = 0; t < KR; ++t) {
            int i = lane + t * G;
            if (i < k) sum += a.t.N[(base + lab[t]) * k + i];
          }
        } else {
          for (int i = lane; i < k; i += G) sum += a.t.N[(base + row[i]) * k + i];
        }
      } else if (kfits) {  // implies lds_geom
#pragma unroll
        for (int t = 0; t < KR; ++t) {
          int i = lane + t * G;
          if (i < k) sum += a.t.N[s_toff[i] + (int64_t)y * s_L[i] + lab[t]];
        }
      } else if (lds_geom) {
        for (int i = lane; i < k; i += G)
          sum += a.t.N[s_toff[i] + (int64_t)y * s_L[i] + row[i]];
      } else {
        for (int i = lane; i < k; i += G)
          sum += a.t.N[a.t.toff[i] + (int64_t)y * a.t.L[i] + row[i]];
      }
      return group_sum<G>(sum);
    };

    if constexpr (LIST && G == 64) {
      if (fits && kfits) {
        // a deferred vertex: its distinct candidate clusters collected in a
        // per-wave LDS hash set and compacted (lane j holds candidates j and
        // 64 + j, in no particular order: every argmin breaks ties by
        // cluster id), then its own cluster and the candidates scored, and
        // the smallest (gain, cluster id) taken by a wave reduction
        const int w = threadIdx.x >> 6;
        int32_t* cset = s_cset[w];
        int32_t* cnb = s_cnb[w];
        for (int j = lane; j < kCandSet; j += 64) cset[j] = -1;
        if (lane == 0) s_ccount[w] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int32_t y = x[r];
          if (y == kInf) continue;
          uint32_t h = ((uint32_t)y * 2654435761u) >> (32 - kCandSetBits);
          for (int q = 0; q < kCandSet; ++q) {  // bounded: a full set ends it
            int32_t cur = cset[h];
            if (cur == -1) {
              cur = atomicCAS(&cset[h], -1, y);
              if (cur == -1) {
                // the arc's head: a candidate of one vertex has it as its
                // only member
                cnb[h] = a.col[beg + r * 64 + lane];
                atomicAdd(&s_ccount[w], 1);
                break;
              }
            }
            if (cur == y) break;
            h = (h + 1) & (kCandSet - 1);
          }
        }
        __builtin_amdgcn_wave_barrier();
        int32_t nc = s_ccount[w];
        // more than 128 candidates (with member lists), or as many as the set
        // holds: the general path below
        const bool many = MEM ? nc > 128 : nc >= kCandSet;
        int32_t cand_lo = kInf, cand_hi = kInf;
        if (!many) {
          int32_t mine = 0, keys[kCandSet / 64];
#pragma unroll
          for (int q = 0; q < kCandSet / 64; ++q) {
            keys[q] = cset[lane + 64 * q];
            mine += keys[q] != -1;
          }
          int32_t total;
          int32_t pos = wave_excl_scan(mine, &total);
          int32_t* clist = s_clist[w];
          int32_t* cnbl = s_cnbl[w];
#pragma unroll
          for (int q = 0; q < kCandSet / 64; ++q)
            if (keys[q] != -1) {
              if (pos < 128) cnbl[pos] = cnb[lane + 64 * q];
              clist[pos++] = keys[q];
            }
          __builtin_amdgcn_wave_barrier();
          cand_lo = lane < nc ? clist[lane] : kInf;
          cand_hi = 64 + lane < nc ? clist[64 + lane] : kInf;
          __builtin_amdgcn_wave_barrier();
        }
        if (!many) {
          if (a.dirty) {  // the candidate set, cached for later passes
            if (lane < min(nc, kCacheCand)) a.ccache[v * kCacheCand + lane] = cand_lo;
            if (lane == 0) a.cnum[v] = nc;
          }
          if (nc == 0) {
            if (lane == 0) a.prop[v] = kNone;
            continue;
          }
          const int sg = lane >> 4, sl = lane & 15;
          int32_t lb[4];  // labels of partitions sl + 16 q
#pragma unroll
          for (int q = 0; q < 4; ++q) lb[q] = sl + 16 * q < k ? row[sl + 16 * q] : 0;
          int32_t s_lo = 0, s_hi = 0, s_v = 0;
          const int nitems = nc + 1;  // item 0: the own cluster; item c + 1: candidate c
          if constexpr (MEM) {
            // Small clusters (member lists) are scored by their members' label
            // rows, every member row of every small item in flight at once:
            // four lanes per (item, member) pair, sixteen pairs a step, the
            // pair sums added into the item's LDS slot.  The other items
            // probe the table, one per 16-lane group.
            int32_t* ioff = s_ioff[w];
            int32_t* isum = s_isum[w];
            int32_t* imst = s_imst[w];
            int32_t* iy = s_iy[w];
            int32_t* ilarge = s_ilarge[w];
            // this lane's items: lane, 64 + lane and, for lane 0, 128
            const int32_t lo_prev = __shfl(cand_lo, (lane + 63) & 63, 64);
            const int32_t hi_prev = __shfl(cand_hi, (lane + 63) & 63, 64);
            const int32_t yA = lane == 0 ? cv : lo_prev;
            const int32_t yB = lane == 0 ? lo_prev : hi_prev;
            const int32_t yC = hi_prev;
            const bool vA = lane < nitems, vB = 64 + lane < nitems, vC = lane == 0 && 128 < nitems;
            // a member of each item: v for its own cluster, else the head of
            // an arc into the candidate (candidate c is item c + 1)
            const int32_t* cnbl = s_cnbl[w];
            const int32_t uA = lane == 0 ? (int32_t)v : (vA ? cnbl[lane - 1] : -1);
            const int32_t uB = vB ? cnbl[63 + lane] : -1;
            const int32_t uC = vC ? cnbl[127] : -1;
            const int32_t zA = vA ? a.s[yA] : 0, zB = vB ? a.s[yB] : 0, zC = vC ? a.s[yC] : 0;
            const bool smA = vA && zA <= a.msum_max, smB = vB && zB <= a.msum_max,
                       smC = vC && zC <= a.msum_max;
            // member list start, or ~u for a cluster whose one member u is known
            auto mlist = [&](bool sm, int32_t z, int32_t u, int32_t y) -> int32_t {
              return !sm ? 0 : ((z == 1 && u >= 0) ? ~u : a.mstart[y]);
            };
            const int32_t mA = mlist(smA, zA, uA, yA), mB = mlist(smB, zB, uB, yB),
                          mC = mlist(smC, zC, uC, yC);
            int32_t totA, totB, lgA, lgB;
            const int32_t exA = wave_excl_scan(smA ? zA : 0, &totA);
            const int32_t exB = wave_excl_scan(smB ? zB : 0, &totB);
            const int32_t gA = wave_excl_scan((vA && !smA) ? 1 : 0, &lgA);
            const int32_t gB = wave_excl_scan((vB && !smB) ? 1 : 0, &lgB);
            const int32_t cC = __shfl(smC ? zC : 0, 0, 64);
            const int32_t P = totA + totB + cC;  // member pairs
            ioff[lane] = exA;
            ioff[64 + lane] = totA + exB;
            isum[lane] = 0;
            isum[64 + lane] = 0;
            imst[lane] = mA;
            imst[64 + lane] = mB;
            iy[lane] = yA;
            iy[64 + lane] = yB;
            if (vA && !smA) ilarge[gA] = lane;
            if (vB && !smB) ilarge[lgA + gB] = 64 + lane;
            if (lane == 0) {
              ioff[128] = totA + totB;
              ioff[129] = P;
              isum[128] = 0;
              imst[128] = mC;
              iy[128] = yC;
              if (vC && !smC) ilarge[lgA + lgB] = 128;
            }
            const int32_t NL = lgA + lgB + __shfl((vC && !smC) ? 1 : 0, 0, 64);
            __builtin_amdgcn_wave_barrier();
            // the item of pair p: the last item whose first pair is at or
            // before p (items without pairs share their successor's offset)
            auto item_of = [&](int32_t p) {
              int lo = 0, hi = 128;
              while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (ioff[mid] <= p) lo = mid;
                else hi = mid - 1;
              }
              return lo;
            };
            const int li = lane & 3, pq = lane >> 2;
            int32_t* vrow = s_vrow[w];  // the vertex's row, read by every pair
            vrow[lane] = lane < k ? row[lane] : 0;
            __builtin_amdgcn_wave_barrier();
            if (a.Lc) {  // compact rows: four lanes read 64 bytes of a member's row
              const uint4* L4 = reinterpret_cast<const uint4*>(a.Lc);
              const int q4 = a.lc_stride >> 4;  // 16-byte words a row
              const bool bytes = a.lc_width == 1;
              const int32_t pad = (a.lc_stride / a.lc_width) - k;  // zeros that agree
              constexpr int E = 4;
              for (int32_t p0 = 0; p0 < P; p0 += 16 * E) {
                int32_t its[E], us[E], sums[E];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                  const int32_t p = p0 + 16 * e + pq;
                  its[e] = -1;
                  us[e] = 0;
                  sums[e] = 0;
                  if (p < P) {
                    const int it = item_of(p);
                    its[e] = it;
                    const int32_t ms = imst[it];
                    us[e] = ms < 0 ? ~ms : a.members[ms + (p - ioff[it])];
                  }
                }
                for (int c = li; c < q4; c += 4) {
                  const uint4 o = L4[v * q4 + c];
                  uint4 r[E];
#pragma unroll
                  for (int e = 0; e < E; ++e)
                    r[e] = its[e] >= 0 ? L4[(int64_t)us[e] * q4 + c] : o;
#pragma unroll
                  for (int e = 0; e < E; ++e)
                    sums[e] += bytes ? agree8(r[e], o) : agree16(r[e], o);
                }
#pragma unroll
                for (int e = 0; e < E; ++e) {
                  sums[e] += __shfl_xor(sums[e], 1, 4);
                  sums[e] += __shfl_xor(sums[e], 2, 4);
                  if (li == 0 && its[e] >= 0) atomicAdd(&isum[its[e]], sums[e] - pad);
                }
              }
            } else if ((k & 1) == 0) {  // rows 8-byte aligned: two partitions a load
              const int h = k >> 1;
              const int2* vl = reinterpret_cast<const int2*>(vrow);
              for (int32_t p0 = 0; p0 < P; p0 += 32) {
                int32_t sums[2], its[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  const int32_t p = p0 + 16 * e + pq;
                  sums[e] = 0;
                  its[e] = -1;
                  if (p < P) {
                    const int it = item_of(p);
                    its[e] = it;
                    const int32_t ms = imst[it];
                    const int32_t u = ms < 0 ? ~ms : a.members[ms + (p - ioff[it])];
                    const int2* ru = reinterpret_cast<const int2*>(a.Lvm + (int64_t)u * k);
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                      if (li + 4 * t < h) {
                        const int2 q = ru[li + 4 * t], r = vl[li + 4 * t];
                        sums[e] += (q.x == r.x) + (q.y == r.y);
                      }
                  }
                }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  sums[e] += __shfl_xor(sums[e], 1, 4);
                  sums[e] += __shfl_xor(sums[e], 2, 4);
                  if (li == 0 && its[e] >= 0) atomicAdd(&isum[its[e]], sums[e]);
                }
              }
            } else {  // odd k: one partition a load
              for (int32_t p0 = 0; p0 < P; p0 += 16) {
                const int32_t p = p0 + pq;
                int32_t sum = 0, it = -1;
                if (p < P) {
                  it = item_of(p);
                  const int32_t ms = imst[it];
                  const int32_t u = ms < 0 ? ~ms : a.members[ms + (p - ioff[it])];
                  const int32_t* ru = a.Lvm + (int64_t)u * k;
#pragma unroll
                  for (int t = 0; t < 16; ++t)
                    if (li + 4 * t < k) sum += ru[li + 4 * t] == vrow[li + 4 * t];
                }
                sum += __shfl_xor(sum, 1, 4);
                sum += __shfl_xor(sum, 2, 4);
                if (li == 0 && it >= 0) atomicAdd(&isum[it], sum);
              }
            }
            // items of larger clusters: table probes, four items a step
            for (int32_t j0 = 0; j0 < NL; j0 += 4) {
              const int32_t jj = j0 + sg;
              int32_t sum = 0, it = -1;
              if (jj < NL) {
                it = ilarge[jj];
                const int32_t y = iy[it];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                  if (sl + 16 * q < k) sum += count_of(a.t, sl + 16 * q, y, lb[q]);
              }
              sum = group_sum<16>(sum);
              if (sl == 0 && it >= 0) isum[it] = sum;
            }
            __builtin_amdgcn_wave_barrier();
            s_v = isum[0];
            s_lo = isum[1 + lane];
            s_hi = isum[65 + lane];
            __builtin_amdgcn_wave_barrier();
          } else {
            // table probes, eight items a step and group, the sums of a lane's
            // items kept in LDS (the latency of a probe, not the sums, is what
            // a step costs: a hub's forty candidates took ten dependent steps)
            constexpr int D = 8;
            int32_t* isum = s_isum[w];
            const int32_t* clist = s_clist[w];
            for (int j0 = 0; j0 < nitems; j0 += 4 * D) {
              int32_t sum[D];
#pragma unroll
              for (int e = 0; e < D; ++e) {
                const int it = j0 + 4 * e + sg;
                sum[e] = 0;
                if (it < nitems) {
                  const int32_t y = it == 0 ? cv : clist[it - 1];
#pragma unroll
                  for (int q = 0; q < 4; ++q)
                    if (sl + 16 * q < k) sum[e] += count_of(a.t, sl + 16 * q, y, lb[q]);
                }
              }
#pragma unroll
              for (int e = 0; e < D; ++e) {
                const int it = j0 + 4 * e + sg;
                const int32_t x = group_sum<16>(sum[e]);
                if (sl == 0 && it < nitems) isum[it] = x;
              }
            }
            __builtin_amdgcn_wave_barrier();
            s_v = isum[0];
          }
          const int64_t scv = a.s[cv];
          int64_t bd = INT64_MAX;
          int32_t bx = kInf;
          auto consider = [&](int32_t xc, int32_t sx) {
            int64_t d = 2 * ((int64_t)s_v - sx) + (int64_t)k * ((int64_t)a.s[xc] - scv - 1);
            if (a.literal) d += k;
            if (d < bd || (d == bd && xc < bx)) {
              bd = d;
              bx = xc;
            }
          };
          if constexpr (MEM) {
            if (lane < nc) consider(cand_lo, s_lo);
            if (lane + 64 < nc) consider(cand_hi, s_hi);
          } else {
            for (int c = lane; c < nc; c += 64) consider(s_clist[w][c], s_isum[w][c + 1]);
            __builtin_amdgcn_wave_barrier();
          }
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) {
            const int64_t od = __shfl_xor(bd, o, 64);
            const int32_t ox = __shfl_xor(bx, o, 64);
            if (od < bd || (od == bd && ox < bx)) {
              bd = od;
              bx = ox;
            }
          }
          if (lane == 0) {
            evals += nc;
            boundary += 1;
            wide += nc > kTileCandAvg;
            const bool p = bd < 0;
            a.prop[v] = p ? bx : kNone;
            if (p) {
              a.dprop[v] = bd;
              ++nprop;
            }
            if (a.slack) a.slack[v] = p ? -1 : (int32_t)min(bd, (int64_t)INT32_MAX);
          }
          continue;
        }
        // the arc registers again, for the general path
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int64_t j = beg + r * G + lane;
          x[r] = kInf;
          if (j < end) {
            const int32_t cu = a.ac ? a.ac[j] : cn_load(a, a.col[j]);
            if (cu != cv) x[r] = cu;
          }
        }
      }
    }

    int32_t last = -1, ncand = 0, bestx = kNone;
    int64_t bestd = 0, s_own = -1;
    const int64_t sc = a.s[cv];
    for (;;) {
      int32_t m = kInf;
      if (fits) {
#pragma unroll
        for (int r = 0; r < R; ++r) m = min(m, x[r]);
      } else {
        for (int64_t j = beg + lane; j < end; j += G) {
          const int32_t cu = a.ac ? a.ac[j] : cn_load(a, a.col[j]);
          if (cu != cv && cu > last && cu < m) m = cu;
        }
      }
      m = group_min<G>(m);
      if (m == kInf) break;
      if (s_own < 0) {
        load_row();
        s_own = agree(cv);
      }
      const int64_t sx = agree(m);
      int64_t d = 2 * (s_own - sx) + (int64_t)k * ((int64_t)a.s[m] - sc - 1);
      if (a.literal) d += k;
      if (ncand == 0 || d < bestd) {
        bestd = d;
        bestx = m;
      }
      ++ncand;
      last = m;
      if (fits) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (x[r] == m) x[r] = kInf;
      }
    }
    if (lane == 0) {
      evals += ncand;
      boundary += ncand > 0;
      wide += ncand > kTileCandAvg;
      if (LIST && a.dirty) {  // nothing kept: scored anew next pass
        a.cnum[v] = -1;
        a.slack[v] = -1;
      }
      const bool p = ncand > 0 && bestd < 0;
      a.prop[v] = p ? bestx : kNone;
      if (p) {
        a.dprop[v] = bestd;
        ++nprop;
      }
    }
  }
  flush_counts(a, evals, nprop, boundary, 0, wide);
}

// ---------------------------------------------------------------------------
// Tiled scorer.  A workgroup owns a tile of TV consecutive vertices:
//  1. the tile's row offsets and clusters go to LDS;
//  2. its arcs are walked in chunks, every thread taking consecutive arcs
//     with independent loads; each arc whose head lies in another cluster
//     inserts the key (tail, head cluster) into a tile-wide LDS hash set and
//     the first insertion of a key counts a candidate for the tail (a
//     self-loop points at the own cluster and drops out with it);
//  3. the set is compacted into one run of pairs per boundary vertex, its
//     own cluster first, then its candidate clusters;
//  4. groups of kProbeLanes lanes probe the flat list of pairs, lanes spread
//     over the partitions, with the next batch's label rows in flight while
//     the current batch probes (consecutive pairs of one vertex share one
//     load of its label row);
//  5. one thread per vertex takes the smallest (gain, cluster id).
// A vertex whose key finds no slot in the set is deferred to a list that
// the group scorer finishes in the same pass, so results never depend on
// the set's capacity.
//
// Bound by the latency of the chain arcs -> clusters -> set -> rows -> table
// lines at 16 waves a compute unit, so the tile is sized to give every unit
// its four workgroups (launch_tile), and a lane holds ceil(k / 16) labels
// (NR; 0: any k) of four pairs, of eight where that is two or fewer: the
// loads in flight, not the arithmetic, set the pace.
// ---------------------------------------------------------------------------
constexpr int kArcChunk = 1024;
constexpr int kSetSlots = 2048;
constexpr int kSetProbe = 64;
constexpr int kProbeLanes = 16;
constexpr int64_t kSmallTileMax = (int64_t)1 << 18;  // vertices scored by tiles of 64
constexpr int64_t kSmallTileFew = (int64_t)5 << 15;  // the same with at most 256 clusters
static_assert(kMemberSumMax <= kProbeLanes, "member ids of a small cluster fit one probe group");

// Clusters at the heads of a thread's arcs (-1 where the tail is -1): one
// uniform branch on the width of the narrow copy, all loads of a width in
// flight together.
template <int U>
__device__ inline void tile_clusters(const PassArgs& a, const int (&tl)[U], const int32_t (&hd)[U],
                                     int32_t (&cu)[U]) {
  if (a.ac) {  // the per-arc cache: the clusters themselves were streamed
#pragma unroll
    for (int r = 0; r < U; ++r) cu[r] = tl[r] >= 0 ? hd[r] : -1;
  } else if (a.cn_bytes == 1) {
#pragma unroll
    for (int r = 0; r < U; ++r) cu[r] = tl[r] >= 0 ? (int32_t)((const uint8_t*)a.Cn)[hd[r]] : -1;
  } else if (a.cn_bytes == 2) {
#pragma unroll
    for (int r = 0; r < U; ++r) cu[r] = tl[r] >= 0 ? (int32_t)((const uint16_t*)a.Cn)[hd[r]] : -1;
  } else {
#pragma unroll
    for (int r = 0; r < U; ++r) cu[r] = tl[r] >= 0 ? ((const int32_t*)a.Cn)[hd[r]] : -1;
  }
}

template <int TK, int TV, int NR>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8)))
void k_score_tile(PassArgs a) {
  if (a.ctl->done || a.ctl->stage) return;
  constexpr int kPairMax = kSetSlots + TV;  // every candidate plus one own pair per vertex
  constexpr int kProbeRegs = NR > 0 ? NR : 1;       // labels per lane when k <= 16 NR
  // pairs in flight (hashed lookups hold more registers a pair)
  constexpr int kProbeBatch = TK == kHashed ? (NR > 2 ? 2 : 4) : (NR > 2 || NR == 0 ? 4 : 8);
  __shared__ int32_t s_off[TV + 1];
  __shared__ int32_t s_c[TV];
  __shared__ int32_t s_nc[TV];    // candidates of each vertex
  __shared__ int32_t s_def[TV];   // 1: vertex deferred to the group scorer
  __shared__ int32_t s_cur[TV];   // fill cursor of the vertex's run
  __shared__ int32_t s_clean[TV]; // 1: candidate set taken from the cache
  __shared__ int32_t s_np;            // pairs that fit the pair arrays
  __shared__ int32_t s_nq;            // hashed tables: pairs left for the table
  __shared__ int32_t s_set[kSetSlots];
  __shared__ int32_t s_cl[kPairMax];   // pair keys (vertex << 24 | cluster), run per vertex
  __shared__ int32_t s_S[kPairMax];    // agreement sum of each pair
  const int t = threadIdx.x;
  const int32_t k = a.k;
  const int g = t / kProbeLanes, lane = t % kProbeLanes;
  int64_t evals = 0;
  int32_t nprop = 0, boundary = 0, wide = 0;
  const int64_t ntiles = (a.n + TV - 1) / TV;
  // passes with few vertices to rescore are left to the list scorer, and
  // passes whose vertices mostly have more candidates than a tile holds to
  // the wave-per-vertex scorer
  if (a.st && a.ctl->rescore_count <= a.sparse_max) return;
  if (a.ctl->defer_all) return;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t v0 = tile * TV;
    const int nv = (int)min((int64_t)TV, a.n - v0);
    const int32_t cv = t < nv ? a.C[v0 + t] : -1;
    if (t < TV) s_c[t] = cv;
    // candidates of a vertex that need not be found again (from the status
    // pass: 0 also for a vertex already settled), -1: walk its arcs
    int32_t cached = -1;
    if (a.st && t < nv) {
      const int32_t stv = a.st[v0 + t];
      cached = stv < 0 ? 0 : (stv > 0 ? stv : -1);
    }
    if (t < TV) {
      s_clean[t] = cached >= 0;
      s_nc[t] = cached > 0 ? cached : 0;
      s_def[t] = 0;
    }
    for (int j = t; j < kSetSlots; j += kBlock) s_set[j] = -1;
    // the arcs are walked only when some vertex of the tile needs them
    const int walk = __syncthreads_or(t < nv && cached < 0);
    int64_t a0 = 0;
    if (walk) {
      a0 = a.row_ptr[v0];
      for (int j = t; j <= nv; j += kBlock) s_off[j] = (int32_t)(a.row_ptr[v0 + j] - a0);
    } else if (t == 0) {
      s_off[nv] = 0;
    }
    __syncthreads();
    const int32_t A = s_off[nv];
    // each thread takes U consecutive arcs of every chunk, read as one
    // 16-byte load from an aligned arc index (the tile's arcs are walked from
    // the aligned index at or before its first arc): one search for the tail
    // of the first, then a walk along the row offsets
    constexpr int U = kArcChunk / kBlock;
    static_assert(U == 4, "one int4 load per thread and chunk");
    const int32_t sh = a.arcs_aligned ? (int32_t)(a0 & 3) : 0;
    const int64_t base = a0 - sh;
    const int32_t* src = a.ac ? a.ac : a.col;  // heads, or the per-arc clusters
    for (int32_t cb = 0; cb < A + sh; cb += kArcChunk) {
      const int32_t jt = cb + t * U - sh;  // tile-relative index of the thread's first arc
      int32_t hd[U];
      if (jt + U > 0 && jt < A) {
        const int64_t gi = base + cb + t * U;
        if (a.arcs_aligned && gi + U <= a.nnz) {
          const int4 q4 = *reinterpret_cast<const int4*>(src + gi);
          hd[0] = q4.x;
          hd[1] = q4.y;
          hd[2] = q4.z;
          hd[3] = q4.w;
        } else {
#pragma unroll
          for (int r = 0; r < U; ++r) {
            const int32_t j = jt + r;
            hd[r] = (j >= 0 && j < A) ? src[a0 + j] : 0;
          }
        }
      }
      int lo = 0;
      const int32_t j0 = max(jt, 0);
      if (j0 < A) {
        int hi = nv - 1;  // tail: the last vertex whose row starts at or before j0
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (s_off[mid] <= j0) lo = mid;
          else hi = mid - 1;
        }
      }
      // tails of the thread's arcs; clean tails skip the gather
      int tl[U];
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const int32_t j = jt + r;
        tl[r] = -1;
        if (j < 0 || j >= A) continue;
        while (s_off[lo + 1] <= j) ++lo;
        if (!s_clean[lo]) tl[r] = lo;
      }
      int32_t cu[U];
      tile_clusters<U>(a, tl, hd, cu);
      int32_t prev = -1;  // the last key this thread placed: repeats skip the set
#pragma unroll
      for (int r = 0; r < U; ++r) {
        if (tl[r] < 0) continue;
        lo = tl[r];
        const int32_t x = cu[r];
        if (x == s_c[lo] || s_def[lo]) continue;  // a deferred vertex needs no more keys
        const int32_t key = (lo << 24) | x;
        if (key == prev) continue;
        prev = key;
        uint32_t h = ((uint32_t)key * 2654435761u) >> 21;  // 11 bits: kSetSlots
        bool placed = false;
        for (int q = 0; q < kSetProbe; ++q) {
          int32_t cur = s_set[h];
          if (cur == -1) cur = atomicCAS(&s_set[h], -1, key);
          if (cur == -1) {  // first sighting of (lo, x)
            atomicAdd(&s_nc[lo], 1);
            placed = true;
            break;
          }
          if (cur == key) {
            placed = true;
            break;
          }
          h = (h + 1) & (kSetSlots - 1);
        }
        if (!placed) s_def[lo] = 1;
      }
    }
    __syncthreads();
    const int nc = t < nv ? s_nc[t] : 0;
    bool def = t < nv && s_def[t];
    bool is_b = t < nv && nc > 0 && !def;
    // one run per boundary vertex: its own cluster, then its candidates.
    // Candidates taken from the key set number at most kSetSlots, but cached
    // sets bypass it: a run that would pass the end of the pair arrays
    // defers its vertex (and the runs after it) to the group scorer.
    int32_t npairs;
    const int32_t coff = block_exclusive_scan(is_b ? nc + 1 : 0, &npairs);
    if (t == 0) s_np = npairs;
    __syncthreads();
    if (is_b && coff + nc + 1 > kPairMax) {
      is_b = false;
      def = true;
      s_def[t] = 1;
      atomicMin(&s_np, coff);
    }
    if (t < nv) {
      const int64_t v = v0 + t;
      if (def) {
        const int32_t slot = atomicAdd(&a.ctl->heavy_count, 1);
        a.heavy[slot] = (int32_t)v;
        if (a.slack) a.slack[v] = -1;
      } else if (nc == 0) {
        a.prop[v] = kNone;
      } else {
        evals += nc;
        boundary += 1;
        wide += nc > kTileCandAvg;
      }
    }
    if (t < TV) s_cur[t] = coff + 1;
    if (is_b) {
      s_cl[coff] = (t << 24) | s_c[t];
      if (s_clean[t])
        for (int j = 0; j < nc; ++j)
          s_cl[coff + 1 + j] = (t << 24) | a.ccache[(v0 + t) * kCacheCand + j];
    }
    __syncthreads();
    npairs = s_np;
    for (int h = t; h < kSetSlots; h += kBlock) {
      const int32_t key = s_set[h];
      if (key == -1) continue;
      const int tv = (int)((uint32_t)key >> 24);
      if (s_def[tv]) continue;
      s_cl[atomicAdd(&s_cur[tv], 1)] = key;
    }
    __syncthreads();
    // cache the sets found this pass (interior vertices cache "none")
    if (a.dirty && t < nv && !s_clean[t]) {
      const int64_t v = v0 + t;
      if (def) {
        a.cnum[v] = -1;
      } else {
        if (nc <= kCacheCand)
          for (int j = 0; j < nc; ++j)
            a.ccache[v * kCacheCand + j] = s_cl[coff + 1 + j] & 0xffffff;
        a.cnum[v] = nc;
      }
    }
    // Hashed tables with compact rows: clusters of up to msum_max members are
    // scored from their members' rows, four lanes a pair and four members at
    // a time (a 64-byte line each, against about ten lines of a table lookup);
    // the pairs of the others are listed (in the key set, which is done with)
    // for the probes below.
    int nprobe = npairs;
    uint16_t* plist = reinterpret_cast<uint16_t*>(s_set);
    const bool by_rows = TK == kHashed && a.Lc != nullptr;
    if (by_rows) {
      if (t == 0) s_nq = 0;
      __syncthreads();
      const uint4* L4 = reinterpret_cast<const uint4*>(a.Lc);
      const int q4 = a.lc_stride >> 4, li = t & 3;
      const bool bytes = a.lc_width == 1;
      const int32_t pad = a.lc_stride / a.lc_width - k;  // zeros that agree
      for (int p = t >> 2; p < npairs; p += kBlock / 4) {
        const int32_t key = s_cl[p], x = key & 0xffffff;
        const int64_t v = v0 + (int)((uint32_t)key >> 24);
        const int32_t cnt = a.s[x];
        if (cnt > a.msum_max) {
          if (li == 0) plist[atomicAdd(&s_nq, 1)] = (uint16_t)p;
          continue;
        }
        const int32_t b = a.mstart[x];
        int32_t sum = 0;
        for (int32_t m = 0; m < cnt; m += 4) {
          const int32_t mid = m + li < cnt ? a.members[b + m + li] : -1;
          int32_t u[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) u[j] = __shfl(mid, j, 4);
          for (int c = li; c < q4; c += 4) {
            const uint4 o = L4[v * q4 + c];
            uint4 r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = L4[(int64_t)max(u[j], 0) * q4 + c];
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (u[j] >= 0) sum += bytes ? agree8(r[j], o) : agree16(r[j], o);
          }
        }
        sum += __shfl_xor(sum, 1, 4);
        sum += __shfl_xor(sum, 2, 4);
        if (li == 0) s_S[p] = sum - cnt * pad;
      }
      __syncthreads();
      nprobe = s_nq;
    }
    constexpr int kStride = (kBlock / kProbeLanes) * kProbeBatch;
    auto pair_of = [&](int p) { return by_rows ? (int)plist[p] : p; };
    auto pair_at = [&](int p, int32_t& x, uint32_t& row) {
      x = -1;
      row = 0;
      if (p < nprobe) {
        const int32_t key = s_cl[pair_of(p)];
        x = key & 0xffffff;
        row = (uint32_t)(v0 + (int)((uint32_t)key >> 24)) * (uint32_t)k;
      }
    };
    // label rows of a batch; a pair of the same vertex as the one before it
    // takes that pair's registers instead of loading again
    auto load_rows = [&](const int32_t* xq, const uint32_t* vq, int32_t (*lq)[kProbeRegs]) {
#pragma unroll
      for (int q = 0; q < kProbeBatch; ++q) {
        const bool same = q > 0 && xq[q - 1] >= 0 && vq[q] == vq[q - 1];
#pragma unroll
        for (int r = 0; r < kProbeRegs; ++r) {
          const int i = lane + r * kProbeLanes;
          lq[q][r] = (xq[q] >= 0 && i < k && !same) ? a.Lvm[vq[q] + i] : 0;
        }
      }
#pragma unroll
      for (int q = 1; q < kProbeBatch; ++q)
        if (xq[q - 1] >= 0 && vq[q] == vq[q - 1]) {
#pragma unroll
          for (int r = 0; r < kProbeRegs; ++r) lq[q][r] = lq[q - 1][r];
        }
    };
    if constexpr (NR > 0) {
      int32_t xs[kProbeBatch], lab[kProbeBatch][kProbeRegs];
      uint32_t vs[kProbeBatch];
      int p0 = g * kProbeBatch;
#pragma unroll
      for (int q = 0; q < kProbeBatch; ++q) pair_at(p0 + q, xs[q], vs[q]);
      load_rows(xs, vs, lab);
      for (; p0 < nprobe; p0 += kStride) {
        int32_t xn[kProbeBatch], labn[kProbeBatch][kProbeRegs];
        uint32_t vn[kProbeBatch];
#pragma unroll
        for (int q = 0; q < kProbeBatch; ++q) pair_at(p0 + kStride + q, xn[q], vn[q]);
        load_rows(xn, vn, labn);
        int32_t sums[kProbeBatch];
#pragma unroll
        for (int q = 0; q < kProbeBatch; ++q) {
          int32_t sum = 0;
          if (TK == kHashed && !by_rows && xs[q] >= 0 && a.s[xs[q]] <= a.msum_max) {
            const int32_t cnt = a.s[xs[q]];  // <= kProbeLanes: one member id per lane
            const int32_t mid = lane < cnt ? a.members[a.mstart[xs[q]] + lane] : 0;
            for (int32_t m = 0; m < cnt; ++m) {
              const uint32_t ru = (uint32_t)__shfl(mid, m, kProbeLanes) * (uint32_t)k;
#pragma unroll
              for (int r = 0; r < kProbeRegs; ++r) {
                const int i = lane + r * kProbeLanes;
                if (i < k) sum += a.Lvm[ru + i] == lab[q][r];
              }
            }
          } else {
#pragma unroll
            for (int r = 0; r < kProbeRegs; ++r) {
              const int i = lane + r * kProbeLanes;
              if (xs[q] >= 0 && i < k) sum += count_t<TK>(a.t, i, xs[q], lab[q][r]);
            }
          }
          sums[q] = sum;
        }
#pragma unroll
        for (int q = 0; q < kProbeBatch; ++q) {
          const int32_t sq = group_sum<kProbeLanes>(sums[q]);
          if (lane == 0 && xs[q] >= 0) s_S[pair_of(p0 + q)] = sq;
        }
#pragma unroll
        for (int q = 0; q < kProbeBatch; ++q) {
          xs[q] = xn[q];
          vs[q] = vn[q];
#pragma unroll
          for (int r = 0; r < kProbeRegs; ++r) lab[q][r] = labn[q][r];
        }
      }
    } else {
      for (int p0 = g * kProbeBatch; p0 < nprobe; p0 += kStride) {
#pragma unroll
        for (int q = 0; q < kProbeBatch; ++q) {
          int32_t x;
          uint32_t ro;
          pair_at(p0 + q, x, ro);
          int32_t sum = 0;
          if (x >= 0) {
            const int32_t* row = a.Lvm + ro;
            if (TK == kHashed && !by_rows && a.s[x] <= a.msum_max) {
              const int32_t cnt = a.s[x];
              const int32_t mid = lane < cnt ? a.members[a.mstart[x] + lane] : 0;
              for (int32_t m = 0; m < cnt; ++m) {
                const int32_t* ru = a.Lvm + (int64_t)__shfl(mid, m, kProbeLanes) * k;
                for (int i = lane; i < k; i += kProbeLanes) sum += ru[i] == row[i];
              }
            } else {
              for (int i = lane; i < k; i += kProbeLanes) sum += count_t<TK>(a.t, i, x, row[i]);
            }
          }
          const int32_t sq = group_sum<kProbeLanes>(sum);
          if (lane == 0 && x >= 0) s_S[pair_of(p0 + q)] = sq;
        }
      }
    }
    __syncthreads();
    if (is_b) {
      const int64_t v = v0 + t;
      const int32_t c = s_c[t];
      const int64_t s_own = s_S[coff];
      const int64_t scz = a.s[c];
      int64_t bestd = 0;
      int32_t bestx = kNone;
      for (int j = coff + 1; j <= coff + nc; ++j) {
        const int32_t x = s_cl[j] & 0xffffff;
        int64_t d = 2 * (s_own - (int64_t)s_S[j]) + (int64_t)k * ((int64_t)a.s[x] - scz - 1);
        if (a.literal) d += k;
        if (bestx == kNone || d < bestd || (d == bestd && x < bestx)) {
          bestd = d;
          bestx = x;
        }
      }
      const bool p = bestd < 0;
      a.prop[v] = p ? bestx : kNone;
      if (p) {
        a.dprop[v] = bestd;
        ++nprop;
      }
      if (a.slack) a.slack[v] = p ? -1 : (int32_t)min(bestd, (int64_t)INT32_MAX);
    }
    __syncthreads();
  }
  flush_counts(a, evals, nprop, boundary, 0, wide);
}

// ---------------------------------------------------------------------------
// Slice scorer: few clusters and many vertices, where four partitions'
// slices of the table fit half of the LDS.  k_slices writes the interleaved
// table as one slice a partition (half a megabyte for 51 clusters and 50
// partitions); a workgroup scores a tile of 1024 vertices of the rescoring
// list, one a thread:
//  1. arcs, spread over all threads: the head's cluster sets a bit of the
//     tail's mask (cached candidate sets set theirs without arcs);
//  2. the vertices are put in order of their candidates;
//  3. the agreement sums: two or more slices at a time in LDS, the counts of
//     the own cluster and of up to 11 candidates a round added in registers,
//     labels read as words of four partitions.  Vertices with more candidates
//     take further rounds, or, where they are few in the tile, go to the
//     wave-per-vertex scorer;
//  4. the smallest (gain, cluster id).
// The counts of a candidate come from LDS where the tiled scorer gathers them
// from L2, sixteen lanes a pair.  Bound by latency, about 40 us a tile for
// the arcs (columns from HBM, then clusters) and 55 us for the sums (label
// words from HBM, slices from L2) with two workgroups a compute unit: waves
// wait on memory 46 % and for issue 43 % of their time, LDS is busy 20 to 29 %
// (half of it conflicts), the vector units 20 to 32 %.  2 M kNN vertices, 51
// clusters, 50 partitions, a pass over all of them 1.22 -> 0.55 ms, over half
// 0.66 -> 0.30, over a twentieth 0.17 -> 0.11 (from the list scorer); solves of
// seven inputs 5.3 to 9.2 -> 4.0 to 6.7 ms.
// One workgroup a compute unit with all of its LDS: 0.68 ms; slices through
// registers instead of straight to LDS: 0.59; eight lanes a vertex for the
// arcs: 0.69.
// ---------------------------------------------------------------------------
constexpr int kSliceTile = 1024;
constexpr int kSliceItems = 12;     // the own cluster and the candidates of a round
constexpr int kSliceStatic = 1024;  // bytes of the kernel's own arrays, at most

__global__ __launch_bounds__(kBlock) void k_slices(PassArgs a) {
  const Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  if (a.st && ctl->rescore_count <= a.sparse_max) return;
  const int32_t k = a.k, Lmax = a.t.Lmax;
  const int32_t cells = (int32_t)a.cells;
  for (int32_t j = blockIdx.x * kBlock + threadIdx.x; j < cells; j += gridDim.x * kBlock) {
    const int32_t row = j / k, i = j - row * k;
    const int32_t x = row / Lmax, l = row - x * Lmax;
    a.slices[(int64_t)i * a.slice_cells + l * a.slice_row + x] = a.t.N[j];
  }
}

__global__ __launch_bounds__(kSliceTile) __attribute__((amdgpu_waves_per_eu(8, 8)))
void k_score_slices(PassArgs a) {
  constexpr int TB = kSliceTile, U = 8;
  const Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  if (a.st && ctl->rescore_count <= a.sparse_max) return;
  if (ctl->defer_all) return;
  extern __shared__ __align__(16) unsigned char smem[];
  const int W = (a.K0 + 31) >> 5;
  uint32_t* s_mask = reinterpret_cast<uint32_t*>(smem);               // W * TB
  int32_t* s_sz = reinterpret_cast<int32_t*>(s_mask + W * TB);        // K0, to a multiple of 4
  unsigned char* s_tab = reinterpret_cast<unsigned char*>(s_sz + ((a.K0 + 3) & ~3));
  // until the slices take their place:
  int32_t* s_off = reinterpret_cast<int32_t*>(s_tab);  // TB + 1: arcs to walk of the vertices before
  int32_t* s_d = s_off + TB + 4;                       // TB: position of a vertex's arc j less j
  uint8_t* s_c = reinterpret_cast<uint8_t*>(s_d + TB); // TB: clusters
  int32_t* s_v = s_off;                                // TB + 1, after the arcs: vertices
  int32_t* s_perm = s_d;                               // TB, after the arcs: their order
  __shared__ int32_t s_hist[kSliceItems];
  __shared__ int32_t s_more;
  const int t = threadIdx.x;
  const int32_t k = a.k, K0 = a.K0;
  const int64_t n = a.n, v0 = (int64_t)blockIdx.x * TB;
  // the vertices to rescore, in the order of their list unless that is all
  const int64_t count = a.st ? ctl->rescore_count : n;
  if (v0 >= count) return;
  const int nv = (int)min((int64_t)TB, count - v0);
  const int64_t v = t >= nv ? -1 : (count < n ? a.rlist[v0 + t] : v0 + t);
  const int32_t cv = t < nv ? a.C[v] : 0;
  // candidates that need not be found again (see k_score_tile)
  int32_t cached = t < nv ? -1 : 0;
  if (a.st && t < nv) {
    const int32_t stv = a.st[v];
    if (stv > 0) cached = stv;
  }
  s_c[t] = (uint8_t)cv;
  for (int w = 0; w < W; ++w) s_mask[w * TB + t] = 0;
  for (int j = 0; j < cached; j += 4) {
    const int4 q = *reinterpret_cast<const int4*>(a.ccache + v * kCacheCand + j);
    const int32_t x[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (j + r < cached) s_mask[(x[r] >> 5) * TB + t] |= 1u << (x[r] & 31);
  }
  for (int x = t; x < K0; x += TB) s_sz[x] = a.s[x];
  if (t == 0) s_more = 0;
  if (t < kSliceItems) s_hist[t] = 0;
  int32_t beg = 0, deg = 0;
  if (cached < 0) {
    beg = (int32_t)a.row_ptr[v];
    deg = (int32_t)a.row_ptr[v + 1] - beg;
  }
  int32_t A;
  const int32_t off = block_exclusive_scan<TB>(deg, &A);
  s_off[t] = off;
  s_d[t] = beg - off;
  if (t == 0) s_off[TB] = A;
  __syncthreads();
  const uint8_t* Cn = static_cast<const uint8_t*>(a.Cn);
  for (int32_t j0 = t * U; j0 < A; j0 += TB * U) {
    int lo = 0, hi = TB - 1;  // tail: the last vertex whose arcs start at or before j0
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_off[mid] <= j0) lo = mid;
      else hi = mid - 1;
    }
    int tl[U];
    int32_t hd[U], ch[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      while (j0 + r < A && s_off[lo + 1] <= j0 + r) ++lo;
      tl[r] = lo;
      hd[r] = a.col[s_d[lo] + min(j0 + r, A - 1)];
    }
#pragma unroll
    for (int r = 0; r < U; ++r) ch[r] = Cn[hd[r]];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int32_t x = ch[r];
      if (x == s_c[tl[r]]) continue;
      uint32_t* w = &s_mask[(x >> 5) * TB + tl[r]];
      const uint32_t b = 1u << (x & 31);
      if (!(*w & b)) atomicOr(w, b);
    }
  }
  __syncthreads();
  int32_t nc = 0;
  for (int w = 0; w < W; ++w) nc += __popc(s_mask[w * TB + t]);
  // keep the sets found this pass
  const bool found = a.dirty && t < nv && cached < 0;
  if (found && nc <= kCacheCand) {
    int j = 0;
    for (int w = 0; w < W; ++w)
      for (uint32_t b = s_mask[w * TB + t]; b; b &= b - 1)
        a.ccache[v * kCacheCand + j++] = w * 32 + __ffs(b) - 1;
  }
  constexpr int kRound = kSliceItems - 1;
  const uint64_t more = __ballot(nc > kRound);
  if ((t & 63) == 0 && more) atomicAdd(&s_more, (int32_t)__popcll(more));
  __syncthreads();
  const bool def = nc > kRound && s_more <= TB / 16;
  if (def) a.heavy[atomicAdd(&a.ctl->heavy_count, 1)] = (int32_t)v;
  if (found) a.cnum[v] = def ? -1 : nc;
  if (def && a.slack) a.slack[v] = -1;
  const int32_t cnt = def ? 0 : nc;
  if (t < nv && !def && cnt == 0) a.prop[v] = kNone;
  // The threads take the vertices in order of their candidates, so that a
  // wave's work is that of its vertices and not of the largest among 64.
  const int32_t key = min(cnt, kRound);
  const int32_t rank = atomicAdd(&s_hist[key], 1);
  s_v[t] = (int32_t)v;
  __syncthreads();
  int32_t at = rank;
  for (int j = 0; j < key; ++j) at += s_hist[j];
  s_perm[at] = t;
  __syncthreads();
  const int p = s_perm[t];
  const int64_t own = s_v[p];
  const int32_t cu = s_c[p];
  int32_t mine = 0;
  for (int w = 0; w < W; ++w) mine += __popc(s_mask[w * TB + p]);
  if (t < s_hist[0]) mine = 0;  // no candidate, or deferred
  // ---- sums ----
  int64_t bd = 0;
  int32_t bx = kNone;
  int cw = 0;               // the mask word the thread is at
  uint32_t cb = s_mask[p];  // and its bits not taken yet
  for (int32_t done = 0; __syncthreads_or(done < mine); done += kRound) {
    const int32_t here = max(0, min(kRound, mine - done));
    // byte offsets of the items in a row, two a register; the own cluster
    // first, and in the places of the candidates that are not there
    uint32_t xp[kSliceItems / 2];
    int32_t S[kSliceItems];
#pragma unroll
    for (int c = 0; c < kSliceItems; ++c) {
      uint32_t x = (uint32_t)cu;
      if (c > 0 && c <= here) {
        while (!cb) cb = s_mask[++cw * TB + p];
        x = (uint32_t)(cw * 32 + __ffs(cb) - 1);
        cb &= cb - 1;
      }
      S[c] = 0;
      if (c & 1) xp[c >> 1] |= x << 18;
      else xp[c >> 1] = x << 2;
    }
    const bool any = __any(here > 0);  // of the wave
    const uint32_t step = (uint32_t)a.slice_cells * 4, rb = (uint32_t)a.slice_row * 4;
    uint32_t lw = 0, ln = here ? a.Lp[own] : 0;
    // Straight to LDS, the next slices while these are read: no registers,
    // and one barrier a group of slices.
    auto fetch = [&](int32_t i0, uint32_t buf) {
      const int4* src = reinterpret_cast<const int4*>(a.slices + (int64_t)i0 * a.slice_cells);
      const int32_t n16 = min(a.slice_load, k - i0) * a.slice_cells / 4;
      const int w0 = __builtin_amdgcn_readfirstlane(t & ~63), lane = t & 63;
      for (int32_t j = w0; j < n16; j += TB)
        if (j + lane < n16)
          __builtin_amdgcn_global_load_lds(
              (const __attribute__((address_space(1))) void*)(src + j + lane),
              (__attribute__((address_space(3))) void*)(s_tab + buf + 16 * j), 16, 0, 0);
    };
    const uint32_t half = (uint32_t)a.slice_load * step;
    uint32_t buf = 0;
    fetch(0, 0);
    for (int32_t i0 = 0; i0 < k; i0 += a.slice_load, buf ^= half) {
      const int32_t np = min(a.slice_load, k - i0);
      // this wave's slices have arrived; after the barrier everyone's have,
      // and the other half has been read
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (i0 + a.slice_load < k) fetch(i0 + a.slice_load, buf ^ half);
      if (!any) continue;
      for (int32_t g = 0; g < np; g += 2) {  // i0 + g is even
        if (((i0 + g) & 3) == 0) {
          lw = ln;
          const int32_t nx = i0 + g + 4;
          if (nx < k) ln = here ? a.Lp[(int64_t)(nx >> 2) * n + own] : 0;
        }
        const uint32_t l0 = lw & 255, l1 = (lw >> 8) & 255;
        lw >>= 16;
        if (!here) continue;
        const bool two = g + 1 < np;
        const uint32_t r0 = buf + g * step + l0 * rb, r1 = two ? r0 + step + (l1 - l0) * rb : r0;
        const int32_t m1 = two ? -1 : 0;
        // the offsets stay packed: unpacked ahead of the loop they would take
        // the registers of the counts in flight
#pragma unroll
        for (int c = 0; c < kSliceItems / 2; ++c) asm("" : "+v"(xp[c]));
#pragma unroll
        for (int c = 0; c < kSliceItems; c += 4) {
          if (c > here) break;
          int32_t g0[4], g1[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint32_t x = (c + u) & 1 ? xp[(c + u) >> 1] >> 16 : xp[(c + u) >> 1] & 0xffff;
            g0[u] = *reinterpret_cast<const int32_t*>(s_tab + (r0 + x));
            g1[u] = *reinterpret_cast<const int32_t*>(s_tab + (r1 + x));
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) S[c + u] += g0[u] + (g1[u] & m1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (here) {
      const int32_t szc = s_sz[cu];
#pragma unroll
      for (int c = 1; c < kSliceItems; ++c) {
        if (c > here) break;
        const int32_t x = (int32_t)(c & 1 ? xp[c >> 1] >> 18 : (xp[c >> 1] & 0xffff) >> 2);
        int64_t d = 2 * ((int64_t)S[0] - S[c]) + (int64_t)k * ((int64_t)s_sz[x] - szc - 1);
        if (a.literal) d += k;
        if (bx == kNone || d < bd) {  // candidates come in increasing id
          bd = d;
          bx = x;
        }
      }
    }
  }
  const bool move = bx != kNone && bd < 0;
  if (mine > 0) {
    a.prop[own] = move ? bx : kNone;
    if (move) a.dprop[own] = bd;
    if (a.slack) a.slack[own] = move ? -1 : (int32_t)min(bd, (int64_t)INT32_MAX);
  }
  flush_counts<TB>(a, mine, move ? 1 : 0, mine > 0 ? 1 : 0, 0, mine > kTileCandAvg ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Dirty marks where the graph is not known to be symmetric: eight lanes a
// vertex look up whether it or one of its neighbours moved in the previous
// pass (a bit a vertex: 125 KiB for 1 M vertices), unless more than an eighth
// of the vertices moved.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_pull(PassArgs a) {
  const Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  const int64_t n = a.n;
  if ((int64_t)ctl->last_moves * 8 > n) return;  // k_status takes all as dirty
  constexpr int G = 8;
  const int lane = threadIdx.x & (G - 1);
  const int64_t ngroups = (int64_t)gridDim.x * kBlock / G;
  for (int64_t v = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G; v < n; v += ngroups) {
    const int64_t beg = a.row_ptr[v], end = a.row_ptr[v + 1];
    int32_t hit = lane == 0 ? (int32_t)(a.moved[v >> 5] >> (v & 31)) & 1 : 0;
    for (int64_t j = beg + lane; j < end; j += 2 * G) {
      const int32_t u = a.col[j], w = a.col[j + G < end ? j + G : j];
      hit |= (int32_t)((a.moved[u >> 5] >> (u & 31)) | (a.moved[w >> 5] >> (w & 31))) & 1;
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) hit |= __shfl_xor(hit, o, G);
    if (lane == 0) a.dirty[v] = hit;
  }
}

// ---------------------------------------------------------------------------
// Status of every vertex at the start of a pass (with the candidate cache),
// one thread per vertex.  A vertex is settled here when it has no candidate
// (a clean vertex whose cached set is empty) or when the bound on the
// change of its gains since its last exact scoring cannot make any of them
// negative (it would not propose: its decision is written and its
// candidates counted as scored, as the method scores them).  Every other
// vertex goes to the rescoring list.  Also clears this pass's dirty marks
// and the per-cluster move counts the coming apply fills.
// ---------------------------------------------------------------------------
template <int V>  // vertices per thread and chunk: v = c0 + j kBlock + t
__global__ __launch_bounds__(kBlock) void k_status(PassArgs a) {
  Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  __shared__ int32_t s_base;
  const int par = ctl->passes & 1;
  const int32_t* churn = a.churn + (int64_t)par * a.K0;
  int32_t* next = a.churn + (int64_t)(par ^ 1) * a.K0;
  const int32_t churn_max = ctl->churn_max;
  const bool all_dirty = (int64_t)ctl->last_moves * 8 > a.n;
  const int t = threadIdx.x;
  const int64_t t0 = (int64_t)blockIdx.x * kBlock + t, T = (int64_t)gridDim.x * kBlock;
  for (int64_t x = t0; x < a.K0; x += T) next[x] = 0;
  if (a.moved)
    for (int64_t w = t0; w < (a.n + 31) / 32; w += T) a.moved[w] = 0;
  const int32_t k = a.k;
  constexpr int64_t kChunk = (int64_t)V * kBlock;
  int64_t evals = 0, skipped = 0, boundary = 0;
  for (int64_t c0 = (int64_t)blockIdx.x * kChunk; c0 < a.n; c0 += (int64_t)gridDim.x * kChunk) {
    int32_t d[V], cn[V], sl[V], cv[V], stv[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int64_t v = c0 + j * kBlock + t;
      d[j] = 1;
      cn[j] = -1;
      sl[j] = -1;
      cv[j] = 0;
      if (v < a.n) {
        d[j] = all_dirty ? 1 : a.dirty[v];
        cn[j] = a.cnum[v];
        sl[j] = a.slack[v];
        cv[j] = a.C[v];
      }
    }
    int32_t mine = 0;
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int64_t v = c0 + j * kBlock + t;
      stv[j] = -1;
      if (v >= a.n) continue;
      if (d[j]) a.dirty[v] = 0;  // this pass's moves mark it again
      const int32_t known = d[j] ? -1 : cn[j];
      if (known == 0) {
        a.prop[v] = kNone;
      } else if (known > 0) {
        stv[j] = known <= kListLanes ? known : 0;
        if (sl[j] >= 0) {
          // the candidates' largest move count, by the cheap bound first
          const int64_t own = churn[cv[j]];
          int64_t bound = (int64_t)k * (own + churn_max);
          if ((int64_t)sl[j] < bound && known <= kCacheCand) {
            const int4* cc = reinterpret_cast<const int4*>(a.ccache + v * kCacheCand);
            int32_t mx = 0;
            for (int q = 0; 4 * q < known; ++q) {
              const int4 c = cc[q];
              const int32_t left = known - 4 * q;
              mx = max(mx, churn[c.x]);
              if (left > 1) mx = max(mx, churn[c.y]);
              if (left > 2) mx = max(mx, churn[c.z]);
              if (left > 3) mx = max(mx, churn[c.w]);
            }
            bound = (int64_t)k * (own + mx);
          }
          if ((int64_t)sl[j] >= bound) {  // no candidate's gain can have become negative
            a.slack[v] = (int32_t)(sl[j] - bound);
            a.prop[v] = kNone;
            evals += known;
            skipped += known;
            boundary += 1;
            stv[j] = -1;
          }
        }
      } else {
        stv[j] = 0;
      }
      a.st[v] = stv[j];
      mine += stv[j] >= 0;
    }
    // the chunk's vertices left for scoring, appended with one atomic
    int32_t total;
    int32_t off = block_exclusive_scan(mine, &total);
    if (t == 0 && total) s_base = atomicAdd(&ctl->rescore_count, total);
    __syncthreads();
    if (total) {
      off += s_base;
#pragma unroll
      for (int j = 0; j < V; ++j)
        if (stv[j] >= 0) a.rlist[off++] = (int32_t)(c0 + j * kBlock + t);
    }
    __syncthreads();
  }
  flush_counts(a, evals, 0, boundary, skipped);
}

// ---------------------------------------------------------------------------
// List scorer: the vertices of the rescoring list, in passes where they are
// few, kListLanes lanes per vertex.  A vertex's candidates come from its
// cache or from its arcs (distinct neighbour clusters, in increasing id, one
// per lane); its own cluster and the candidates are then probed eight at a
// time (four in hashed tables) with all their probes issued together.
// Vertices with more candidates than lanes, a degree beyond the arc registers
// or k beyond the label registers go to the deferred list (the
// wave-per-vertex scorer).
// ---------------------------------------------------------------------------

template <int CN, int TK>
__global__ __launch_bounds__(kBlock) void k_score_list(PassArgs a) {
  Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  const int32_t count = ctl->rescore_count;
  if (count == 0 || count > a.sparse_max) return;  // the tiled scorer takes dense passes
  constexpr int G = kListLanes;
  constexpr int R = 8;               // arcs per lane in registers: degree <= 128
  constexpr int KR = 64 / G;         // labels per lane: k <= 64
  constexpr int32_t kInf = 0x7fffffff;
  const int lane = threadIdx.x & (G - 1);
  const int64_t group = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G;
  const int64_t ngroups = ((int64_t)gridDim.x * kBlock) / G;
  const int32_t k = a.k;
  int64_t evals = 0;
  int32_t nprop = 0, boundary = 0, wide = 0;
  for (int64_t idx = group; idx < count; idx += ngroups) {
    const int64_t v = a.rlist[idx];
    const int32_t cv = a.C[v];
    const int32_t stv = a.st[v];
    int32_t cand = kInf, nc = 0;
    bool defer = k > KR * G;
    if (!defer && stv > 0) {
      nc = stv;
      if (lane < nc) cand = a.ccache[v * kCacheCand + lane];
    } else if (!defer) {
      const int64_t beg = a.row_ptr[v], end = a.row_ptr[v + 1];
      if (end - beg > (int64_t)G * R) {
        defer = true;
      } else {
        int32_t x[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int64_t j = beg + r * G + lane;
          x[r] = kInf;
          if (j < end) {
            const int32_t cu = cn_load_t<CN>(a, j, CN ? a.col[j] : 0);
            if (cu != cv) x[r] = cu;
          }
        }
        for (;;) {  // distinct clusters in increasing id, candidate j on lane j
          int32_t m = kInf;
#pragma unroll
          for (int r = 0; r < R; ++r) m = min(m, x[r]);
          m = group_min<G>(m);
          if (m == kInf) break;
          if (nc == G) {
            defer = true;
            break;
          }
          if (lane == nc) cand = m;
          ++nc;
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (x[r] == m) x[r] = kInf;
        }
        if (!defer) {  // the set found, cached for later passes
          if (lane < min(nc, kCacheCand)) a.ccache[v * kCacheCand + lane] = cand;
          if (lane == 0) a.cnum[v] = nc;
        }
      }
    }
    if (defer) {
      if (lane == 0) {
        a.heavy[atomicAdd(&ctl->heavy_count, 1)] = (int32_t)v;
        a.cnum[v] = -1;
        a.slack[v] = -1;
      }
      continue;
    }
    if (nc == 0) {
      if (lane == 0) {
        a.prop[v] = kNone;
        a.slack[v] = -1;
      }
      continue;
    }
    int32_t lab[KR];
    const int32_t* row = a.Lvm + v * k;
#pragma unroll
    for (int t = 0; t < KR; ++t) {
      const int i = lane + t * G;
      lab[t] = i < k ? row[i] : 0;
    }
    const int64_t scv = a.s[cv];
    int64_t s_own = 0, bd = 0;
    int32_t bx = kNone;
    constexpr int D = TK == kHashed ? 4 : 8;  // items in flight
    for (int i0 = 0; i0 <= nc; i0 += D) {  // item 0: own cluster; item j: candidate j - 1
      int32_t part[D], ys[D];
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const int it = i0 + q;
        const int32_t yc = __shfl(cand, it > 0 ? (it - 1) & (G - 1) : 0, G);
        ys[q] = it == 0 ? cv : (it <= nc ? yc : -1);
        part[q] = 0;
        if (ys[q] >= 0) {
#pragma unroll
          for (int t = 0; t < KR; ++t) {
            const int i = lane + t * G;
            if (i < k) part[q] += count_t<TK>(a.t, i, ys[q], lab[t]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const int64_t sum = group_sum<G>(part[q]);
        if (ys[q] < 0) continue;
        if (i0 + q == 0) {
          s_own = sum;
          continue;
        }
        int64_t d = 2 * (s_own - sum) + (int64_t)k * ((int64_t)a.s[ys[q]] - scv - 1);
        if (a.literal) d += k;
        if (bx == kNone || d < bd || (d == bd && ys[q] < bx)) {
          bd = d;
          bx = ys[q];
        }
      }
    }
    if (lane == 0) {
      evals += nc;
      boundary += 1;
      wide += nc > kTileCandAvg;
      const bool p = bd < 0;
      a.prop[v] = p ? bx : kNone;
      if (p) {
        a.dprop[v] = bd;
        ++nprop;
      }
      a.slack[v] = p ? -1 : (int32_t)min(bd, (int64_t)INT32_MAX);
    }
  }
  flush_counts(a, evals, nprop, boundary, 0, wide);
}

// True in every thread of the last of `total` workgroups to get here (each
// calls it once, after its last global update; `which`: the ticket).  Every
// wave waits until its updates have been performed (the barrier alone does
// not wait for global memory); what the other workgroups added with atomics
// is then read with atomics (now()), so no cache is flushed or invalidated.
__device__ inline bool last_workgroup(const PassArgs& a, int which, int32_t total) {
  __shared__ int32_t s_last;
  int32_t* ticket =
      reinterpret_cast<int32_t*>(a.pc + (kPassCounters + which) * kCounterStride);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    s_last = atomicAdd(ticket, 1) == total - 1;
    if (s_last) atomicExch(ticket, 0);
  }
  __syncthreads();
  return s_last;
}

template <typename T>
__device__ inline T now(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The pass's counters folded into the control block (one thread).
__device__ inline void pass_begin(const PassArgs& a) {
  Ctl* ctl = a.ctl;
  int64_t c[kPassCounters];
#pragma unroll
  for (int j = 0; j < kPassCounters; ++j) {
    c[j] = a.pc[j * kCounterStride];
    a.pc[j * kCounterStride] = 0;
  }
  ctl->nprop = (int32_t)c[1];
  ctl->boundary += c[2];
  ctl->skipped += c[3];
  // most boundary vertices had more candidates than the tiles hold, and
  // many on average (the counts fall fast once clusters merge): the next
  // pass skips the tiled scorer and scores every vertex by the wave
  ctl->defer_all = (2 * c[4] > c[2] && c[0] > kTileCandAvg * c[2]) ? 1 : 0;
  ctl->passes += 1;
  ctl->evals += c[0];
  ctl->dS2 = 0;
  ctl->dN2 = 0;
  ctl->churn_max = 0;
  if (c[1] == 0) {
    ctl->converged = 1;
    ctl->done = 1;
    ctl->slots += 1;
    if (ctl->trace) {
      int64_t* r = ctl->trace + (int64_t)(ctl->passes - 1) * 4;
      r[0] = 0; r[1] = 0; r[2] = 0; r[3] = ctl->O;
    }
  }
  if (!a.hflag) return;
  // Hashed tables: before the batch is applied, rebuild the table from the
  // partition (the counts are a function of C alone) if the keys the batch
  // may add could take it beyond half full (rows: three quarters; the second
  // pass of 2 M singletons then needs no rebuild, 4 ms, and few passes read a
  // row table before a dense one takes over).  Keys: the batch adds at most k
  // keys per proposal; the table holds 4 n k slots or more and at most n k
  // live keys, so after a rebuild there is always room.  Rows: a proposal
  // adds at most its vertex's distinct label ids, at most T0 in all, over at
  // most T0 live rows, in more than 2 T0 rows.  The first pass's table is the
  // one just built (no key without a count), so a rebuild would not change it.
  const int64_t adds = a.t.rows ? now(&ctl->prop_rows) : (int64_t)a.k * c[1];
  const bool need = c[1] > 0 && ctl->passes > 1 &&
                    (int64_t)*a.t.hocc + adds > (int64_t)(a.t.rows ? 3 * ((a.t.hmask + 1) / 4)
                                                                 : (a.t.hmask + 1) / 2);
  *a.hflag = need ? 1 : 0;
  if (need) *a.t.hocc = 0;
}

// Keep the applied batch if it lowered the objective, else fall back (one
// thread).
__device__ inline void pass_decide(Ctl* ctl) {
  const int64_t dO = (int64_t)ctl->k * now(&ctl->dS2) - 2 * now(&ctl->dN2);
  ctl->dS2 = 0;
  ctl->dN2 = 0;
  if (dO < 0) {
    ctl->fallback = 0;
    ctl->O += dO;
    ctl->committed = ctl->nprop;
  } else {
    ctl->fallback = 1;
    ctl->fallback_rounds += 1;
    ctl->committed = 0;
  }
}

// End of a slot (one thread): a batch that fell back goes on in the next
// one, else the pass is accounted.
__device__ inline void pass_end(Ctl* ctl) {
  ctl->slots += 1;
  if (ctl->fallback && !ctl->stage) {
    ctl->stage = 1;
    return;
  }
  ctl->stage = 0;
  if (ctl->fallback) ctl->O += (int64_t)ctl->k * ctl->dS2 - 2 * ctl->dN2;
  ctl->moves += ctl->committed;
  if (ctl->trace) {
    int64_t* r = ctl->trace + (int64_t)(ctl->passes - 1) * 4;
    r[0] = ctl->nprop;
    r[1] = ctl->committed;
    r[2] = ctl->fallback;
    r[3] = ctl->O;
  }
  ctl->last_moves = ctl->committed;
  ctl->nprop = 0;
  ctl->committed = 0;
  ctl->fallback = 0;
  ctl->heavy_count = 0;
  ctl->rescore_count = 0;
  ctl->plist_count = 0;
  ctl->prop_rows = 0;
  ctl->dS2 = 0;
  ctl->dN2 = 0;
  if (ctl->passes >= ctl->max_rounds) ctl->done = 1;
}

// Apply the move of v (from -> to) with sign d (+1 apply, -1 undo) to the
// sizes and counts; lanes of the wave take the partitions.  Returns this
// lane's share of the change of the sums of squares (N part; the size part
// is added by lane 0 to *ds2).
__device__ inline int64_t move_counts(const PassArgs& a, int64_t v, int32_t from, int32_t to,
                                      int32_t d, int lane, int64_t* ds2) {
  int64_t acc = 0;
  const int32_t* row = a.Lvm + v * a.k;
  int32_t claimed = 0;  // these keys exist already (k_apply_all added them)
  for (int i = lane; i < a.k; i += 64) {
    const int32_t l = row[i];
    int32_t o1 = atomicAdd(counter(a.t, cell_upd(a.t, i, to, l, claimed)), d);
    int32_t o2 = atomicAdd(counter(a.t, cell_upd(a.t, i, from, l, claimed)), -d);
    acc += 2 * (int64_t)o1 * d + 1 - 2 * (int64_t)o2 * d + 1;
  }
  if (claimed) atomicAdd(a.t.hocc, claimed);
  if (lane == 0) {
    int32_t o1 = atomicAdd(&a.s[to], d);
    int32_t o2 = atomicAdd(&a.s[from], -d);
    *ds2 += 2 * (int64_t)o1 * d + 1 - 2 * (int64_t)o2 * d + 1;
  }
  return acc;
}

// More than an eighth of the vertices moved in the pass: nearly all are
// dirty, so none is marked and the next pass takes all as dirty (2 M kNN
// vertices that all moved: 0.85 ms of scattered marks).
__device__ inline bool mass_move(const PassArgs& a) {
  return (int64_t)a.ctl->committed * 8 > a.n;
}

// Vertex w moved: it and its out-neighbours (its in-neighbours, the graph
// being symmetric) recompute their candidate sets next pass.
__device__ inline void mark_dirty(const PassArgs& a, int64_t w, int lane, bool mass) {
  if (!a.dirty) return;
  if (a.moved) {  // looked up by k_pull
    if (lane == 0) atomicOr(&a.moved[w >> 5], 1u << (w & 31));
    return;
  }
  if (mass) return;
  if (lane == 0) a.dirty[w] = 1;
  const int64_t b = a.row_ptr[w], e = a.row_ptr[w + 1];
  for (int64_t p = b + lane; p < e; p += 64) a.dirty[a.col[p]] = 1;
}

// Vertex w now sits in cluster c: every arc pointing at w learns it.
__device__ inline void relabel_in_arcs(const PassArgs& a, int64_t w, int32_t c, int lane) {
  if (!a.ac) return;
  const int32_t b = a.in_ptr[w], e = a.in_ptr[w + 1];
  for (int32_t p = b + lane; p < e; p += 64) a.ac[a.in_pos[p]] = c;
}

// The apply-type kernels walk the vertices 64 at a time per wave: one
// coalesced load of the proposals, a ballot, then the wave serves each
// selected vertex with its lanes spread over the partitions.
enum ApplyMode { kCommitOrElect = 1, kFallbackCommit = 2, kFallbackFinish = 3 };

template <int MODE>
__device__ inline void apply_walk(const PassArgs& a, int64_t wave, int64_t nwaves) {
  Ctl* ctl = a.ctl;
  const bool fb = ctl->fallback, mass = mass_move(a);
  const int lane = threadIdx.x & 63;
  int64_t dn2 = 0, ds2 = 0;
  int32_t committed = 0;
  for (int64_t v0 = wave * 64; v0 < a.n; v0 += nwaves * 64) {
    const int64_t v = v0 + lane;
    int32_t p = v < a.n ? a.prop[v] : kNone;
    bool sel;
    if (MODE == kFallbackFinish) sel = p != kNone;  // committed (>= 0) or not (<= -2)
    else sel = p >= 0;
    uint64_t mask = __ballot(sel);
    while (mask) {
      const int b = __ffsll((unsigned long long)mask) - 1;
      mask &= mask - 1;
      const int64_t w = v0 + b;
      const int32_t pw = __shfl(p, b, 64);
      const int32_t from = a.C[w];
      if (MODE == kCommitOrElect) {
        if (!fb) {
          if (lane == 0) {
            a.C[w] = pw;
            cn_store(a, w, pw);
          }
          relabel_in_arcs(a, w, pw, lane);
          mark_dirty(a, w, lane, mass);
        } else {
          move_counts(a, w, from, pw, -1, lane, &ds2);  // undo the batch
          if (lane == 0) {
            const uint64_t key = owner_key(a.dprop[w], w);
            atomicMin((unsigned long long*)&a.owner[from], (unsigned long long)key);
            atomicMin((unsigned long long*)&a.owner[pw], (unsigned long long)key);
          }
        }
      } else if (MODE == kFallbackCommit) {
        const uint64_t key = owner_key(a.dprop[w], w);
        const bool own = a.owner[from] == key && a.owner[pw] == key;
        if (own) {
          dn2 += move_counts(a, w, from, pw, +1, lane, &ds2);
          if (lane == 0) ++committed;
        } else if (lane == 0) {
          a.prop[w] = -2 - pw;  // proposal kept out of this pass
        }
      } else {  // kFallbackFinish
        const int32_t to = pw >= 0 ? pw : -2 - pw;
        if (lane == 0) {
          a.owner[from] = ~0ull;
          a.owner[to] = ~0ull;
          if (pw >= 0) {
            a.C[w] = pw;
            cn_store(a, w, pw);
          }
        }
        if (pw >= 0) {
          relabel_in_arcs(a, w, pw, lane);
          mark_dirty(a, w, lane, mass);
        }
      }
    }
  }
  if (MODE == kFallbackCommit) {
    dn2 = wave_sum64(dn2);
    ds2 = wave_sum64(ds2);
    committed = wave_sum32(committed);
    if (lane == 0) {
      if (dn2) atomicAdd((unsigned long long*)&ctl->dN2, (unsigned long long)dn2);
      if (ds2) atomicAdd((unsigned long long*)&ctl->dS2, (unsigned long long)ds2);
      if (committed) atomicAdd(&ctl->committed, committed);
    }
  }
}

// ---------------------------------------------------------------------------
// Apply every proposal with per-workgroup aggregation.  Updates are keyed by
// table cell (sizes use keys cells + cluster) and summed in an LDS hash
// before one global atomic per distinct key.  Once half the slots hold keys
// the table takes no new ones (probe runs stay short when a workgroup sees
// many distinct keys, as on a first pass): a key not in it, or that finds no
// free slot within kHashProbe steps, goes straight to the global counter.
// A net update d on a counter whose previous value is `old` changes its
// square by 2 old d + d^2, so the flush measures the objective change
// exactly, whichever updates of a key went where.
// ---------------------------------------------------------------------------
constexpr int kHashSlots = 4096;
constexpr int kHashOpen = kHashSlots / 2;  // keys the table takes
constexpr int kHashProbe = 32;

// The changes of the sums of squares caused by one global update: the
// contingency part (n) and the size part (s).  Returned by value: pointers
// to the caller's accumulators would keep them in scratch memory.
struct Sq2 {
  int64_t n, s;
  int32_t churn;  // a cluster's move count after the update, else 0
};

// Keys: [0, cells) table cells, [cells, cells + K0) cluster sizes,
// [cells + K0, cells + 2 K0) per-cluster move counts (churn_w).
__device__ __attribute__((always_inline)) inline Sq2 agg_add(int32_t* hkey, int32_t* hval,
                                                           int32_t* fill, const PassArgs& a,
                                                           int32_t* churn_w, int64_t key,
                                                           int32_t d) {
  const int32_t k32 = (int32_t)key;
  uint32_t h = ((uint32_t)k32 * 2654435761u) >> 20;  // 12 bits: kHashSlots
#pragma unroll 1
  for (int q = 0; q < kHashProbe; ++q) {
    int32_t cur = hkey[h];
    if (cur == -1) {
      if (*fill >= kHashOpen) break;  // the key is not in the table
      cur = atomicCAS(&hkey[h], -1, k32);
      if (cur == -1) {
        atomicAdd(fill, 1);
        cur = k32;
      }
    }
    if (cur == k32) {
      atomicAdd(&hval[h], d);
      return Sq2{0, 0, 0};
    }
    h = (h + 1) & (kHashSlots - 1);
  }
  if (key < a.cells) {
    const int32_t old = atomicAdd(counter(a.t, (uint32_t)key), d);
    return Sq2{2 * (int64_t)old * d + 1, 0, 0};
  }
  if (key < a.cells + a.K0) {
    const int32_t old = atomicAdd(&a.s[key - a.cells], d);
    return Sq2{0, 2 * (int64_t)old * d + 1, 0};
  }
  return Sq2{0, 0, atomicAdd(&churn_w[key - a.cells - a.K0], d) + d};
}

// The proposers of the pass, in plist (order irrelevant): one atomic per
// chunk of V kBlock vertices.
__global__ __launch_bounds__(kBlock) void k_props(PassArgs a) {
  Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) {
    if (a.hflag && blockIdx.x == 0 && threadIdx.x == 0) *a.hflag = 0;
    return;
  }
  __shared__ int32_t s_base;
  constexpr int V = 4;
  constexpr int64_t kChunk = (int64_t)V * kBlock;
  const int t = threadIdx.x;
  int64_t rows = 0;  // hashed rows: the rows the proposals can add
  for (int64_t c0 = (int64_t)blockIdx.x * kChunk; c0 < a.n; c0 += (int64_t)gridDim.x * kChunk) {
    bool pr[V];
    int32_t mine = 0;
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int64_t v = c0 + j * kBlock + t;
      pr[j] = v < a.n && a.prop[v] >= 0;
      mine += pr[j];
      if (pr[j] && a.rdist) rows += a.rdist[v];
    }
    int32_t total;
    int32_t off = block_exclusive_scan(mine, &total);
    if (t == 0 && total) s_base = atomicAdd(&ctl->plist_count, total);
    __syncthreads();
    if (total) {
      off += s_base;
#pragma unroll
      for (int j = 0; j < V; ++j)
        if (pr[j]) a.plist[off++] = (int32_t)(c0 + j * kBlock + t);
    }
    __syncthreads();
  }
  if (a.rdist) {  // one atomic per workgroup
    __shared__ int64_t s_rows[kBlock / 64];
    rows = wave_sum64(rows);
    if ((t & 63) == 0) s_rows[t >> 6] = rows;
    __syncthreads();
    if (t == 0) {
      int64_t tot = 0;
      for (int j = 0; j < kBlock / 64; ++j) tot += s_rows[j];
      if (tot) atomicAdd((unsigned long long*)&ctl->prop_rows, (unsigned long long)tot);
    }
  }
  if (last_workgroup(a, 0, (int32_t)gridDim.x) && t == 0) pass_begin(a);
}

__global__ __launch_bounds__(kBlock) void k_apply_all(PassArgs a) {
  Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  const int lane = threadIdx.x & 63;
  __shared__ int32_t hkey[kHashSlots];
  __shared__ int32_t hval[kHashSlots];
  __shared__ int32_t fill;
  // the workgroup's share of the listed proposals: one per group of 16 lanes
  // at least (late passes move vertices between few clusters: updates merged
  // in LDS spare the counters they share), the lanes of a group spread over
  // the partitions
  constexpr int kApplyLanes = 16, kGroups = kBlock / kApplyLanes;
  const int64_t count = ctl->plist_count;
  const int64_t per = max((int64_t)kGroups, (count + gridDim.x - 1) / gridDim.x);
  const int64_t eb = blockIdx.x * per, ee = min(count, eb + per);
  if (eb < ee) {
    for (int j = threadIdx.x; j < kHashSlots; j += kBlock) {
      hkey[j] = -1;
      hval[j] = 0;
    }
    if (threadIdx.x == 0) fill = 0;
    __syncthreads();
    int64_t dn2 = 0, ds2 = 0;
    int32_t claimed = 0, cmax = 0;
    // moves per cluster, read by the next pass's scorer (counted over every
    // proposal: a fallback pass commits fewer, so the count is an upper bound)
    int32_t* churn_w = a.churn ? a.churn + (int64_t)(ctl->passes & 1) * a.K0 : nullptr;
    const int gl = lane % kApplyLanes;
    for (int64_t e = eb + threadIdx.x / kApplyLanes; e < ee; e += kGroups) {
      const int64_t w = a.plist[e];
      const int32_t to = a.prop[w], from = a.C[w];
      const int32_t* row = a.Lvm + w * a.k;
      for (int i = gl; i < a.k; i += kApplyLanes) {
        const int32_t l = row[i];
        const Sq2 up =
            agg_add(hkey, hval, &fill, a, churn_w, cell_upd(a.t, i, to, l, claimed), +1);
        const Sq2 dn =
            agg_add(hkey, hval, &fill, a, churn_w, cell_upd(a.t, i, from, l, claimed), -1);
        dn2 += up.n + dn.n;
      }
      if (gl == 0) {
        const Sq2 up = agg_add(hkey, hval, &fill, a, churn_w, a.cells + to, +1);
        const Sq2 dn = agg_add(hkey, hval, &fill, a, churn_w, a.cells + from, -1);
        ds2 += up.s + dn.s;
      } else if (gl == 1 && churn_w) {
        cmax = max(cmax, agg_add(hkey, hval, &fill, a, churn_w, a.cells + a.K0 + to, +1).churn);
        cmax = max(cmax, agg_add(hkey, hval, &fill, a, churn_w, a.cells + a.K0 + from, +1).churn);
      }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < kHashSlots; j += kBlock) {
      const int32_t key = hkey[j], d = hval[j];
      if (key < 0 || d == 0) continue;
      if (key < a.cells) {
        const int32_t old = atomicAdd(counter(a.t, (uint32_t)key), d);
        dn2 += 2 * (int64_t)old * d + (int64_t)d * d;
      } else if (key < a.cells + a.K0) {
        const int32_t old = atomicAdd(&a.s[key - a.cells], d);
        ds2 += 2 * (int64_t)old * d + (int64_t)d * d;
      } else {
        cmax = max(cmax, atomicAdd(&churn_w[key - a.cells - a.K0], d) + d);
      }
    }
    if (a.t.hashed) flush_claims(a.t, claimed);
    dn2 = wave_sum64(dn2);
    ds2 = wave_sum64(ds2);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cmax = max(cmax, __shfl_xor(cmax, o, 64));
    if (lane == 0) {
      if (dn2) atomicAdd((unsigned long long*)&ctl->dN2, (unsigned long long)dn2);
      if (ds2) atomicAdd((unsigned long long*)&ctl->dS2, (unsigned long long)ds2);
      if (cmax) atomicMax(&ctl->churn_max, cmax);
    }
  }
  if (last_workgroup(a, 1, (int32_t)gridDim.x) && threadIdx.x == 0) pass_decide(ctl);
}

// ---------------------------------------------------------------------------
// Batch apply for dense tables whose per-partition slice fits in LDS.  The
// grid is (slices, k): workgroup (p, i) takes slice p of the listed
// proposals and histograms partition i's count changes in LDS, +1 at
// (to, l) and -1 at (from, l) with l the mover's label in partition i; then
// it adds every nonzero change to the table with one atomic, whose returned
// value gives the cell's exact share of the change of the sum of squares
// (2 old d + d^2 for each addition, which sums to the exact change whatever
// the order).  The workgroups of partition 0 do the same for the cluster
// sizes and count the moves per cluster (churn).  Late passes, whose few
// proposals mostly move between the same clusters, run one slice: each
// counter then receives one atomic.
// ---------------------------------------------------------------------------
constexpr int kDeltaPerSlice = 2048;  // proposals per slice of the list
constexpr int kDeltaUnroll = 4;

template <bool IL>
__global__ __launch_bounds__(kBlock) void k_apply_delta(PassArgs a) {
  extern __shared__ int32_t sh[];
  Ctl* ctl = a.ctl;
  if (ctl->done || ctl->stage) return;
  const int p = blockIdx.x, i = blockIdx.y, t = threadIdx.x;
  const int64_t count = ctl->plist_count;
  const int64_t active = min((int64_t)gridDim.x,
                             max((int64_t)1, (count + kDeltaPerSlice - 1) / kDeltaPerSlice));
  if (p >= active) return;
  const int32_t k = a.k, K0 = a.K0;
  const int32_t Li = IL ? a.t.Lmax : a.t.L[i];
  const int32_t cells = K0 * Li;  // fits in LDS (checked by the host)
  const bool sizes = i == 0;
  int32_t* hd = sh;
  int32_t* hs = sh + cells;
  int32_t* hc = hs + K0;
  const int32_t zero_len = sizes ? cells + 2 * K0 : cells;
  for (int32_t j = t; j < zero_len; j += kBlock) sh[j] = 0;
  __syncthreads();
  const int64_t per = (count + active - 1) / active;
  const int64_t eb = (int64_t)p * per, ee = min(count, eb + per);
  for (int64_t e0 = eb + t; e0 < ee; e0 += (int64_t)kDeltaUnroll * kBlock) {
    int32_t vv[kDeltaUnroll], to[kDeltaUnroll], fr[kDeltaUnroll], lb[kDeltaUnroll];
#pragma unroll
    for (int q = 0; q < kDeltaUnroll; ++q) {
      const int64_t e = e0 + (int64_t)q * kBlock;
      vv[q] = e < ee ? a.plist[e] : -1;
    }
#pragma unroll
    for (int q = 0; q < kDeltaUnroll; ++q) {
      if (vv[q] < 0) continue;
      to[q] = a.prop[vv[q]];
      fr[q] = a.C[vv[q]];
      lb[q] = a.Lvm[(int64_t)vv[q] * k + i];
    }
#pragma unroll
    for (int q = 0; q < kDeltaUnroll; ++q) {
      if (vv[q] < 0) continue;
      atomicAdd(&hd[to[q] * Li + lb[q]], 1);
      atomicAdd(&hd[fr[q] * Li + lb[q]], -1);
      if (sizes) {
        atomicAdd(&hs[to[q]], 1);
        atomicAdd(&hs[fr[q]], -1);
        atomicAdd(&hc[to[q]], 1);
        atomicAdd(&hc[fr[q]], 1);
      }
    }
  }
  __syncthreads();
  int64_t dn2 = 0, ds2 = 0;
  int32_t cmax = 0;
  const int64_t toff = IL ? 0 : a.t.toff[i];
  for (int32_t j0 = t; j0 < cells; j0 += kDeltaUnroll * kBlock) {
    int32_t d[kDeltaUnroll], old[kDeltaUnroll];
#pragma unroll
    for (int q = 0; q < kDeltaUnroll; ++q) {
      const int32_t j = j0 + q * kBlock;
      d[q] = j < cells ? hd[j] : 0;
      old[q] = 0;
      if (d[q]) {
        const int32_t x = j / Li, l = j - x * Li;
        const uint32_t c = IL ? ((uint32_t)x * (uint32_t)Li + (uint32_t)l) * (uint32_t)k + i
                              : (uint32_t)toff + (uint32_t)j;
        old[q] = atomicAdd(&a.t.N[c], d[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < kDeltaUnroll; ++q)
      dn2 += 2 * (int64_t)old[q] * d[q] + (int64_t)d[q] * d[q];
  }
  if (sizes) {
    int32_t* churn_w = a.churn ? a.churn + (int64_t)(ctl->passes & 1) * K0 : nullptr;
    for (int32_t x = t; x < K0; x += kBlock) {
      const int32_t d = hs[x];
      if (d) {
        const int32_t old = atomicAdd(&a.s[x], d);
        ds2 += 2 * (int64_t)old * d + (int64_t)d * d;
      }
      if (churn_w && hc[x]) cmax = max(cmax, atomicAdd(&churn_w[x], hc[x]) + hc[x]);
    }
  }
  if (sizes && a.churn) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cmax = max(cmax, __shfl_xor(cmax, o, 64));
    if ((t & 63) == 0 && cmax) atomicMax(&ctl->churn_max, cmax);
  }
  dn2 = wave_sum64(dn2);
  ds2 = wave_sum64(ds2);
  __shared__ int64_t red[2][kBlock / 64];
  if ((t & 63) == 0) {
    red[0][t >> 6] = dn2;
    red[1][t >> 6] = ds2;
  }
  __syncthreads();
  if (t == 0) {
    int64_t n2 = 0, s2 = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
      n2 += red[0][w];
      s2 += red[1][w];
    }
    if (n2) atomicAdd((unsigned long long*)&ctl->dN2, (unsigned long long)n2);
    if (s2) atomicAdd((unsigned long long*)&ctl->dS2, (unsigned long long)s2);
  }
  if (last_workgroup(a, 1, (int32_t)active * a.k) && t == 0) pass_decide(ctl);
}

// The second slot's apply (a kernel of its own: inside the apply kernels its
// registers cost them a third of their speed).
__global__ __launch_bounds__(kBlock) void k_fallback(PassArgs a) {
  if (a.ctl->done || !a.ctl->stage) return;
  apply_walk<kFallbackCommit>(a, ((int64_t)blockIdx.x * kBlock + threadIdx.x) / 64,
                              ((int64_t)gridDim.x * kBlock) / 64);
}

__global__ __launch_bounds__(kBlock) void k_commit(PassArgs a) {
  Ctl* ctl = a.ctl;
  if (ctl->done) return;
  const int64_t wave = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / 64;
  const int64_t nwaves = ((int64_t)gridDim.x * kBlock) / 64;
  if (ctl->stage) apply_walk<kFallbackFinish>(a, wave, nwaves);
  else apply_walk<kCommitOrElect>(a, wave, nwaves);
  if (last_workgroup(a, 2, (int32_t)gridDim.x) && threadIdx.x == 0) pass_end(ctl);
}

__global__ __launch_bounds__(kBlock) void k_hash_reset(PassArgs a) {
  if (!*a.hflag) return;
  if (a.t.rows) {  // empty keys, zero counts
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j <= (int64_t)a.t.hmask;
         j += (int64_t)gridDim.x * kBlock)
      a.t.rkeys[j] = kHashEmpty;
    const int64_t cells = ((int64_t)a.t.hmask + 1) * a.k;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < cells;
         j += (int64_t)gridDim.x * kBlock)
      a.t.N[j] = 0;
    return;
  }
  uint4* H = reinterpret_cast<uint4*>(a.t.N);
  const uint4 empty = make_uint4(0xffffffffu, 0xffffffffu, 0u, 0u);
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j <= (int64_t)a.t.hmask;
       j += (int64_t)gridDim.x * kBlock)
    H[j] = empty;
}

__global__ __launch_bounds__(kBlock) void k_hash_refill(PassArgs a) {
  if (!*a.hflag) return;
  if (a.t.rows) {
    flush_claims(a.t, rows_count(a.t, a.C, a.Lvm, a.n, a.k,
                                 (int64_t)blockIdx.x * kBlock + threadIdx.x,
                                 (int64_t)gridDim.x * kBlock));
    return;
  }
  const int64_t total = a.n * a.k;
  int32_t claimed = 0;
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < total;
       j += (int64_t)gridDim.x * kBlock) {
    const int64_t v = j / a.k;
    const int i = (int)(j - v * a.k);
    atomicAdd(counter(a.t, cell_upd(a.t, i, a.C[v], a.Lvm[j], claimed)), 1);
  }
  flush_claims(a.t, claimed);
}

// Member lists of the clusters at the start of the pass (mstart holds the
// exclusive scan of the sizes, mcnt is zeroed): a counting sort of C.
__global__ __launch_bounds__(kBlock) void k_member_fill(PassArgs a) {
  if (a.ctl->done) return;
  for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < a.n;
       v += (int64_t)gridDim.x * kBlock) {
    const int32_t x = a.C[v];
    if (a.s[x] <= a.msum_max)  // larger clusters are probed, not listed
      a.members[a.mstart[x] + atomicAdd(&a.mcnt[x], 1)] = (int32_t)v;
  }
}

__global__ void k_ctl_init(Ctl* ctl, const int64_t* acc, int32_t n, int32_t k, int32_t max_rounds,
                           int64_t* trace, int32_t defer_all) {
  Ctl c = {};
  c.k = k;
  c.max_rounds = max_rounds;
  c.trace = trace;
  c.last_moves = n;
  c.defer_all = defer_all;
  c.O = (int64_t)k * acc[0] + acc[1] - 2 * acc[2];
  *ctl = c;
}

template <int G>
void launch_score(const PassArgs& a, int grid, hipStream_t st) {
  if (a.members) k_score<G, false, true><<<grid, kBlock, 0, st>>>(a);
  else k_score<G, false, false><<<grid, kBlock, 0, st>>>(a);
}

template <int TK, int TV>
void launch_tile_v(const PassArgs& a, hipStream_t st) {
  // as many workgroups as tiles, eight per compute unit at most
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((a.n + TV - 1) / TV, a.tile_grid));
  if (a.k <= 16) k_score_tile<TK, TV, 1><<<grid, kBlock, 0, st>>>(a);
  else if (a.k <= 32) k_score_tile<TK, TV, 2><<<grid, kBlock, 0, st>>>(a);
  else if (a.k <= 64) k_score_tile<TK, TV, 4><<<grid, kBlock, 0, st>>>(a);
  else k_score_tile<TK, TV, 0><<<grid, kBlock, 0, st>>>(a);
}

template <int TK>
void launch_list(const PassArgs& a, int grid, hipStream_t st) {
  if (!a.st) return;
  if (a.ac) k_score_list<0, TK><<<grid, kBlock, 0, st>>>(a);
  else if (a.cn_bytes == 1) k_score_list<1, TK><<<grid, kBlock, 0, st>>>(a);
  else if (a.cn_bytes == 2) k_score_list<2, TK><<<grid, kBlock, 0, st>>>(a);
  else k_score_list<4, TK><<<grid, kBlock, 0, st>>>(a);
}

template <int TK>
void launch_tile(const PassArgs& a, int grid, hipStream_t st) {
  // Vertices a tile: up to 2^18 vertices, tiles of 64 (a launch of 256 would
  // leave compute units without a tile: 15 passes over 100 000 vertices of
  // an LFR graph 5.9 ms against 9.3, 24 over 30 000 3.5 against 7.9).  Above,
  // tiles of 128, whose key set holds 16 candidates a vertex (1 M LFR
  // vertices, ten candidates each, all passes dense: 49.6 ms against 51.4 with
  // 256 and 54.7 with 64).  At most 256 clusters keep the candidates few, and
  // tiles of 256 pay from 2.5 of them a compute unit (kNN shape, 42 partitions,
  // tiles of 64 and 256: 120 000 vertices 0.74 and 0.78 ms, 160 000 1.82 and
  // 1.79, 200 000 2.19 and 2.05, 250 000 2.29 and 2.10; 2 M scored by tiles 8.8
  // with 128, 8.2 with 256).
  // Tiles of 64 also where the candidates are many: with hashed tables, whose
  // starts have one for most arcs, and after a pass with more than twelve.
  const bool few = a.K0 <= 256;
  if (TK == kHashed || a.tile_small || a.n <= (few ? kSmallTileFew : kSmallTileMax))
    launch_tile_v<TK, 64>(a, st);
  else if (few)
    launch_tile_v<TK, 256>(a, st);
  else
    launch_tile_v<TK, 128>(a, st);
  launch_list<TK>(a, grid, st);
}

// Taken (slice_shape) from 2^19 vertices, two tiles for every compute unit
// (320 000 vertices, 42 partitions: 2.72 ms, 2.62 with tiles of 256; 530 000:
// 2.98 against 3.18), where two buffers of two slices fit beside the candidate masks in half of
// the LDS (4480 cells for up to 64 clusters: 2 M vertices of 51 clusters and
// 75 label ids), the ids fit a byte, and the labels were transposed by tiles.
// Passes over up to 65536 vertices keep the list scorer: 21 us over 10 000,
// 140 to 177 us over 100 000 to 250 000, which the slices take in 100 us.
void launch_slices(const PassArgs& a, int grid, hipStream_t st) {
  k_slices<<<(int)std::min<int64_t>((a.cells + kBlock - 1) / kBlock, 1024), kBlock, 0, st>>>(a);
  k_score_slices<<<(unsigned)((a.n + kSliceTile - 1) / kSliceTile), kSliceTile, a.slice_lds,
                   st>>>(a);
  launch_list<kInterleaved>(a, grid, st);
}

}  // namespace

bool slice_shape(int64_t n, int32_t k, int64_t K0, int64_t Lmax, PassArgs* a) {
  if (n < kSliceVertices || K0 > 256 || Lmax > 256) return false;
  const int64_t row = K0 | 1;  // odd: a label's rows spread over the banks
  const int64_t cells = (row * Lmax + 3) & ~(int64_t)3;
  const int64_t words = (K0 + 31) / 32;
  const int64_t fixed = 4 * ((K0 + 3) & ~(int64_t)3) + 4 * words * kSliceTile;
  int64_t load = std::min<int64_t>((kSliceLds - kSliceStatic - fixed) / (8 * cells), k + 1) & ~1;
  if (load < 2) return false;
  a->slice_row = (int32_t)row;
  a->slice_cells = (int32_t)cells;
  a->slice_load = (int32_t)load;
  a->slice_lds = (int32_t)(fixed + std::max<int64_t>(8 * load * cells, 9 * kSliceTile + 16));
  return true;
}

bool score_lanes_ok(int lanes) {
  return lanes == 0 || lanes == 4 || lanes == 8 || lanes == 16 || lanes == 32 || lanes == 64;
}

void launch_ctl_init(Ctl* ctl, const int64_t* acc, int64_t n, int32_t k, int32_t max_rounds,
                     int64_t* trace, bool defer_all, hipStream_t st) {
  k_ctl_init<<<1, 1, 0, st>>>(ctl, acc, (int32_t)n, k, max_rounds, trace, defer_all ? 1 : 0);
}

void enqueue_pass(const PassArgs& a, int lanes, int grid_score, int grid_apply, hipStream_t st,
                  hipEvent_t score_begin, hipEvent_t score_end) {
  if (a.members) {
    launch_scan(a.s, a.mstart, a.K0, a.mscan_tmp, st);
    launch_fill_i32(a.mcnt, a.K0, 0, st);
    k_member_fill<<<grid_apply, kBlock, 0, st>>>(a);
  }
  if (score_begin) (void)hipEventRecord(score_begin, st);
  switch (lanes) {
    case 0:
      if (a.moved)
        k_pull<<<(int)std::min<int64_t>((a.n * 8 + kBlock - 1) / kBlock, a.tile_grid), kBlock, 0,
                 st>>>(a);
      // one vertex a thread until that fills the chip
      if (a.st && a.n <= kSmallTileMax) k_status<1><<<grid_apply, kBlock, 0, st>>>(a);
      else if (a.st) k_status<4><<<grid_apply, kBlock, 0, st>>>(a);
      if (a.Lp) launch_slices(a, grid_score, st);
      else if (a.t.hashed) launch_tile<kHashed>(a, grid_score, st);
      else if (a.t.interleaved) launch_tile<kInterleaved>(a, grid_score, st);
      else launch_tile<kBlocked>(a, grid_score, st);
      // deferred vertices: one per wave, as many waves as the chip holds
      if (a.members) k_score<64, true, true><<<grid_score, kBlock, 0, st>>>(a);
      else k_score<64, true, false><<<grid_score, kBlock, 0, st>>>(a);
      break;
    case 4: launch_score<4>(a, grid_score, st); break;
    case 8: launch_score<8>(a, grid_score, st); break;
    case 16: launch_score<16>(a, grid_score, st); break;
    case 32: launch_score<32>(a, grid_score, st); break;
    default: launch_score<64>(a, grid_score, st); break;
  }
  if (score_end) (void)hipEventRecord(score_end, st);
  // Two workgroups a compute unit: each takes a ticket at the end, one after
  // another (300 000 vertices: 7 us with 512 workgroups, 12 with 1024).  The
  // commit needs four where many of 2^20 vertices or more move (106 us against
  // 137 for 290 000 moves of 2 M), below two (13 against 15 us).
  const int grid_end = std::min(grid_apply, std::max(1, a.tile_grid / 4));
  k_props<<<grid_end, kBlock, 0, st>>>(a);
  if (a.t.hashed) {
    k_hash_reset<<<grid_apply, kBlock, 0, st>>>(a);
    k_hash_refill<<<grid_apply, kBlock, 0, st>>>(a);
  }
  if (a.delta_lds > 0) {
    const dim3 grid((unsigned)a.delta_slices, (unsigned)a.k);
    if (a.t.interleaved) k_apply_delta<true><<<grid, kBlock, a.delta_lds, st>>>(a);
    else k_apply_delta<false><<<grid, kBlock, a.delta_lds, st>>>(a);
  } else {
    k_apply_all<<<grid_apply, kBlock, 0, st>>>(a);
  }
  k_fallback<<<grid_apply, kBlock, 0, st>>>(a);
  k_commit<<<a.n < (1 << 20) ? grid_end : grid_apply, kBlock, 0, st>>>(a);
}

}  // namespace mcc
