// Candidate drain on the device: the entries emitted in arbitrary order (atomics) are put
// into key order (search, segment, sky, spindown index, bin) before they are copied out.
// Count -> offsets -> write, as the paper's candidate output is organised (Sect. 3.2):
//   1. count the entries of every template (one atomic per entry, which also gives the
//      entry its rank among its template's entries in arrival order);
//   2. exclusive scan of the counts: each template's offset in the output;
//   3. write every entry to its template's range (template order);
//   4. order each template's range by bin (bins within a template are distinct, so an
//      entry's place is the number of entries of its template with a smaller bin);
//   5. form the records and keys for the copy out.
// Templates are numbered search by search (searches since the previous drain), then
// segment, sky, spindown: t = base[search] + (segment * nsky + sky) * nfdot + fdot_idx.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fstat_kernels.hpp"

namespace fstat {

struct DrainSearch {
  long long base;     // number of the search's first template
  int nsky, nfdot;
};

constexpr int DRAIN_NT = 256;
constexpr int SCAN_TILE = 4096;                 // counts per workgroup of the scan (16 per thread)
constexpr int DRAIN_SEG_MAX = 4096;             // longest template range ordered by counting (longer: bitmap)

__device__ __forceinline__ long long drain_template(const CandEntry& c, const DrainSearch* __restrict__ s,
                                                    int nsearch, int search0, int nseg, unsigned* bad) {
  const int r = c.search - search0;
  if (r < 0 || r >= nsearch) {
    atomicOr(bad, 1u);
    return -1;
  }
  const DrainSearch d = s[r];
  if (c.segment < 0 || c.segment >= nseg || c.sky < 0 || c.sky >= d.nsky || c.fdot_idx < 0 || c.fdot_idx >= d.nfdot) {
    atomicOr(bad, 1u);
    return -1;
  }
  return d.base + ((long long)c.segment * d.nsky + c.sky) * d.nfdot + c.fdot_idx;
}

__global__ void k_drain_zero(unsigned* __restrict__ a, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    a[i] = 0u;
}

// 1. per-template counts; rank[i] = the entry's place among its template's entries so far.
// A template's entries arrive together, so a wavefront first groups its lanes by template
// (up to eight groups; with many templates of few entries the rest go singly) and each group
// counts with one atomic: with one per entry, all on a few cache lines, 13000 entries of 128
// templates took 20 us.
__global__ void __launch_bounds__(DRAIN_NT) k_drain_count(const CandEntry* __restrict__ cand, long long n, const DrainSearch* __restrict__ s,
                              int nsearch, int search0, int nseg, unsigned* __restrict__ counts,
                              unsigned* __restrict__ rank, unsigned* bad) {
  const int lane = threadIdx.x & 63;
  for (long long i0 = (long long)blockIdx.x * DRAIN_NT + (threadIdx.x & ~63); i0 < n;
       i0 += (long long)gridDim.x * DRAIN_NT) {   // whole wavefronts
    const long long i = i0 + lane;
    const long long t = i < n ? drain_template(cand[i], s, nsearch, search0, nseg, bad) : -1;
    bool todo = t >= 0;
    int leader = lane;
    unsigned place = 0, many = 1;
    for (int k = 0; k < 8; ++k) {
      const unsigned long long left = __ballot(todo);
      if (!left) break;
      const int first = __ffsll(left) - 1;
      const long long t0 = __shfl(t, first, 64);
      const unsigned long long same = __ballot(todo && t == t0);
      if (todo && t == t0) {
        leader = first;
        place = (unsigned)__popcll(same & ((1ull << lane) - 1ull));
        many = (unsigned)__popcll(same);
        todo = false;
      }
    }
    unsigned base = 0;
    if (t >= 0 && lane == leader) base = atomicAdd(&counts[t], many);
    base = __shfl(base, leader, 64);
    if (i < n) rank[i] = t < 0 ? 0u : base + place;
  }
}

// Sum of 16 consecutive counts per thread, then of the workgroup's 4096.
__device__ __forceinline__ unsigned long long tile_thread_sum(const unsigned* __restrict__ a, long long n,
                                                              long long i0) {
  unsigned long long v = 0;
  for (int k = 0; k < SCAN_TILE / DRAIN_NT; ++k) {
    const long long i = i0 + k;
    if (i < n) v += a[i];
  }
  return v;
}

// Inclusive scan over the workgroup of one 64-bit value per thread (wavefront shuffles,
// then the wavefront totals through LDS); *total gets the workgroup's sum.
__device__ __forceinline__ unsigned long long block_inclusive_scan_u64(unsigned long long v,
                                                                       unsigned long long* total) {
  __shared__ unsigned long long wsum[DRAIN_NT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned long long u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  if (lane == 63) wsum[wv] = v;
  __syncthreads();
  unsigned long long before = 0, all = 0;
  for (int w = 0; w < DRAIN_NT / 64; ++w) {
    if (w < wv) before += wsum[w];
    all += wsum[w];
  }
  __syncthreads();
  *total = all;
  return v + before;
}

// 2a. workgroup sums of tiles of SCAN_TILE counts
__global__ void __launch_bounds__(DRAIN_NT) k_scan_tile_sums(const unsigned* __restrict__ a, long long n,
                                                             unsigned long long* __restrict__ sums) {
  const long long base = (long long)blockIdx.x * SCAN_TILE + (long long)threadIdx.x * (SCAN_TILE / DRAIN_NT);
  unsigned long long tot;
  (void)block_inclusive_scan_u64(tile_thread_sum(a, n, base), &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// 2b. exclusive scan of the tile sums in place, by one workgroup walking them in order
__global__ void __launch_bounds__(DRAIN_NT) k_scan_sums(unsigned long long* __restrict__ sums, long long ntiles) {
  unsigned long long carry = 0;
  for (long long j0 = 0; j0 < ntiles; j0 += DRAIN_NT) {
    const long long j = j0 + threadIdx.x;
    const unsigned long long v = j < ntiles ? sums[j] : 0ull;
    unsigned long long tot;
    const unsigned long long inc = block_inclusive_scan_u64(v, &tot);
    if (j < ntiles) sums[j] = carry + inc - v;
    carry += tot;
  }
}

// 2c. off[i] = sum of counts before i (i < n), off[n] = the total: each workgroup scans its
// tile (sums null: there is one tile, and this is the whole scan)
__global__ void __launch_bounds__(DRAIN_NT) k_scan_apply(const unsigned* __restrict__ a, long long n,
                                                         const unsigned long long* __restrict__ sums,
                                                         unsigned long long* __restrict__ off) {
  constexpr int PER = SCAN_TILE / DRAIN_NT;
  const long long i0 = (long long)blockIdx.x * SCAN_TILE + (long long)threadIdx.x * PER;
  unsigned long long tot;
  const unsigned long long own = tile_thread_sum(a, n, i0);
  const unsigned long long before = sums ? sums[blockIdx.x] : 0ull;
  unsigned long long run = before + block_inclusive_scan_u64(own, &tot) - own;
  for (int k = 0; k < PER; ++k) {
    const long long i = i0 + k;
    if (i < n) {
      off[i] = run;
      run += a[i];
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == DRAIN_NT - 1) off[n] = before + tot;
}

// 3. every entry to its template's range, in arrival order
__global__ void k_drain_scatter(const CandEntry* __restrict__ cand, long long n, const DrainSearch* __restrict__ s,
                                int nsearch, int search0, int nseg, const unsigned long long* __restrict__ off,
                                const unsigned* __restrict__ rank, CandEntry* __restrict__ grouped, unsigned* bad) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const CandEntry c = cand[i];
    const long long t = drain_template(c, s, nsearch, search0, nseg, bad);
    if (t >= 0) grouped[off[t] + rank[i]] = c;
  }
}

// 4. each template's range ordered by bin, one workgroup per template (grid-stride over
// templates).  Ranges of at most DRAIN_SEG_MAX entries: an entry's place is the number of
// entries of its template with a smaller bin (the bins in LDS); longer ranges are left to
// k_drain_order_long.
__global__ void __launch_bounds__(DRAIN_NT) k_drain_order(const CandEntry* __restrict__ grouped,
                                                          const unsigned long long* __restrict__ off, long long ntpl,
                                                          CandEntry* __restrict__ out, const unsigned* bad) {
  __shared__ int sbin[DRAIN_SEG_MAX];
  if (*bad) return;   // a key outside its search: the entries stay as they are
  for (long long t = blockIdx.x; t < ntpl; t += gridDim.x) {
    const unsigned long long a = off[t], c = off[t + 1] - a;
    if (c == 0 || c > (unsigned long long)DRAIN_SEG_MAX) continue;
    const int m = (int)c;
    __syncthreads();
    for (int j = threadIdx.x; j < m; j += DRAIN_NT) sbin[j] = grouped[a + j].bin;
    __syncthreads();
    for (int j = threadIdx.x; j < m; j += DRAIN_NT) {
      const int b = sbin[j];
      int r = 0;
      for (int k = 0; k < m; ++k) r += (sbin[k] < b) | ((sbin[k] == b) & (k < j));
      out[a + r] = grouped[a + j];
    }
  }
}

// 4b. ranges longer than DRAIN_SEG_MAX (thresholds low enough that a good share of a
// template's bins cross): a bitmap of the template's bins in LDS (up to 2^20 bins, the
// longest transform), popcounts of 32-word blocks scanned across the workgroup, and each
// entry's place = the set bits below its bin.  Bins of one template are distinct: a
// repeated one, or a range wider than the bitmap, sets *bad (bad[-1]: a key outside its
// search, as above).
constexpr int DRAIN_LONG_NT = 1024;
constexpr int DRAIN_BITMAP_WORDS = (1 << 20) / 32;
__global__ void __launch_bounds__(DRAIN_LONG_NT) k_drain_order_long(const CandEntry* __restrict__ grouped,
                                                                    const unsigned long long* __restrict__ off,
                                                                    long long ntpl, CandEntry* __restrict__ out,
                                                                    unsigned* bad) {
  __shared__ unsigned bits[DRAIN_BITMAP_WORDS];
  __shared__ unsigned bpre[DRAIN_BITMAP_WORDS / 32];
  __shared__ int rmin[DRAIN_LONG_NT / 64], rmax[DRAIN_LONG_NT / 64];
  __shared__ unsigned wsum[DRAIN_LONG_NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (bad[-1]) return;
  for (long long t = blockIdx.x; t < ntpl; t += gridDim.x) {
    const unsigned long long a = off[t], c = off[t + 1] - a;
    if (c <= (unsigned long long)DRAIN_SEG_MAX) continue;
    // the template's bin range
    int lo = 0x7fffffff, hi = -0x7fffffff - 1;
    for (unsigned long long j = tid; j < c; j += DRAIN_LONG_NT) {
      const int b = grouped[a + j].bin;
      lo = min(lo, b);
      hi = max(hi, b);
    }
    for (int d = 32; d >= 1; d >>= 1) {
      lo = min(lo, __shfl_xor(lo, d, 64));
      hi = max(hi, __shfl_xor(hi, d, 64));
    }
    __syncthreads();   // the previous template's readers of the shared arrays are done
    if (lane == 0) {
      rmin[wv] = lo;
      rmax[wv] = hi;
    }
    __syncthreads();
    lo = rmin[0];
    hi = rmax[0];
    for (int k = 1; k < DRAIN_LONG_NT / 64; ++k) {
      lo = min(lo, rmin[k]);
      hi = max(hi, rmax[k]);
    }
    if ((long long)hi - lo >= (long long)DRAIN_BITMAP_WORDS * 32) {
      if (tid == 0) atomicOr(bad, 1u);
      continue;
    }
    const int nw = ((hi - lo) >> 5) + 1, nb = (nw + 31) >> 5;
    for (int w = tid; w < nw; w += DRAIN_LONG_NT) bits[w] = 0u;
    __syncthreads();
    for (unsigned long long j = tid; j < c; j += DRAIN_LONG_NT) {
      const int d = grouped[a + j].bin - lo;
      const unsigned m = 1u << (d & 31);
      if (atomicOr(&bits[d >> 5], m) & m) atomicOr(bad, 1u);
    }
    __syncthreads();
    // exclusive scan of the 32-word blocks' popcounts (one block per thread, nb <= 1024)
    unsigned v = 0;
    if (tid < nb)
      for (int k = 0; k < 32; ++k) {
        const int w = tid * 32 + k;
        if (w < nw) v += __popc(bits[w]);
      }
    unsigned inc = v;
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned u = __shfl_up(inc, d, 64);
      if (lane >= d) inc += u;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    unsigned before = 0;
    for (int k = 0; k < wv; ++k) before += wsum[k];
    if (tid < nb) bpre[tid] = before + inc - v;
    __syncthreads();
    for (unsigned long long j = tid; j < c; j += DRAIN_LONG_NT) {
      const CandEntry e = grouped[a + j];
      const int d = e.bin - lo, w = d >> 5;
      unsigned r = bpre[w >> 5];
      for (int u = w & ~31; u < w; ++u) r += __popc(bits[u]);
      r += __popc(bits[w] & ((1u << (d & 31)) - 1u));
      out[a + r] = e;
    }
  }
}

// 5. the records and keys of the ordered entries (none if the ordering refused one: bad, which
// goes to page-locked `flags` for the host), formed as the host would form them (the
// paper's five numbers from the search's lists, the integer key, the vetting score), for a
// copy straight into the caller's arrays
struct DrainList {
  const double* v;   // device copy: alpha[nsky], delta[nsky], then fdot[nfdot] (explicit
                     // list) or w_freq[nsky], w_spin[nsky] (lattice grid)
  int nsky, lattice, s_lo;
  double m10, m11;
};
struct DrainSeg {
  double f_off, dt;
  int nfft;
};

// A search call's lists, kept on the device for the records of its candidates:
// alpha[nsky], delta[nsky], then c[nc] and d[nd] to dst.
__global__ void __launch_bounds__(DRAIN_NT) k_record_lists(const double* __restrict__ alpha,
                                                           const double* __restrict__ delta, int nsky,
                                                           const double* __restrict__ c, int nc,
                                                           const double* __restrict__ d, int nd,
                                                           double* __restrict__ dst) {
  const long long n = 2LL * nsky + nc + nd;
  for (long long i = (long long)blockIdx.x * DRAIN_NT + threadIdx.x; i < n; i += (long long)gridDim.x * DRAIN_NT) {
    long long k = i;
    double v;
    if (k < nsky) v = alpha[k];
    else if ((k -= nsky) < nsky) v = delta[k];
    else if ((k -= nsky) < nc) v = c[k];
    else v = d[k - nc];
    dst[i] = v;
  }
}

__device__ __forceinline__ fstat_candidate_key drain_key(const CandEntry& c, int scored) {
  fstat_candidate_key k;
  k.search = c.search;
  k.segment = c.segment;
  k.sky = c.sky;
  k.fdot_idx = c.fdot_idx;
  k.bin = c.bin;
  k.vet_score = __int_as_float(scored ? c.score : NO_SCORE);
  return k;
}

__device__ __forceinline__ fstat_candidate drain_record(const CandEntry& c, const DrainList& L, const DrainSeg& sg) {
#pragma clang fp contract(off)
  fstat_candidate r;
  if (L.lattice) {
    // the template's frequency shift and spindown, as the search kernels formed them
    const int s = L.s_lo + c.fdot_idx;
    const double u = lattice_shift_bins(lattice_w(s, L.m10, L.v[2 * L.nsky + c.sky]), (double)sg.nfft / (2.0 * M_PI));
    r.f_hz = sg.f_off + ((double)c.bin + u) / ((double)sg.nfft * sg.dt);
    r.fdot = lattice_w(s, L.m11, L.v[3 * L.nsky + c.sky]) / (M_PI * sg.dt * sg.dt);
  } else {
    r.f_hz = sg.f_off + (double)c.bin / ((double)sg.nfft * sg.dt);
    r.fdot = L.v[2 * L.nsky + c.fdot_idx];
  }
  r.alpha = L.v[c.sky];
  r.delta = L.v[L.nsky + c.sky];
  r.twoF = c.twoF;
  return r;
}

__global__ void k_drain_records(const CandEntry* __restrict__ ent, long long n, const DrainList* __restrict__ lists,
                                int search0, const DrainSeg* __restrict__ segs, int scored,
                                fstat_candidate* __restrict__ out, fstat_candidate_key* __restrict__ keys,
                                const unsigned* __restrict__ bad, unsigned* flags) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    flags[0] = bad[0];
    flags[1] = bad[1];
    __threadfence_system();
  }
  if (bad[0]) return;   // an entry outside its search has no list to form a record from
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const CandEntry c = ent[i];
    if (keys) keys[i] = drain_key(c, scored);
    if (out) out[i] = drain_record(c, lists[c.search - search0], segs[c.segment]);
  }
}

// ---- small drains: one launch
// Up to SMALL_CAP crossings of up to SMALL_SEARCHES searches: one workgroup reads the count,
// sorts the entries' keys in LDS (template number, bin and entry packed into 63 bits) and
// writes head, records and keys straight to page-locked host memory.  The general drain's
// ten launches, three synchronous copies each way and per-search page-locked lists took
// 250 us of a search that itself takes 150.
constexpr int SMALL_CAP = 4096, SMALL_SEARCHES = 4, SMALL_NT = 1024;
struct SmallDrain {
  int nsearch, search0, nseg, scored, want;   // want: 0 count only, else records and keys
  long long capacity, buffer;                 // entries asked for; entries of the device buffer
  DrainSearch s[SMALL_SEARCHES];
  DrainList l[SMALL_SEARCHES];
};
struct SmallHead {
  unsigned long long count;
  unsigned bad, done;                          // done: drained here (the count is reset)
  unsigned flags[2], pad[2];                   // the general drain's flags
};

__global__ void k_drain_reset(unsigned long long* __restrict__ count) { *count = 0ull; }

__global__ void __launch_bounds__(SMALL_NT) k_drain_small(SmallDrain a, const CandEntry* __restrict__ cand,
                                                          unsigned long long* __restrict__ count,
                                                          const DrainSeg* __restrict__ segs, SmallHead* head,
                                                          fstat_candidate* out, fstat_candidate_key* keys) {
  __shared__ unsigned long long key[SMALL_CAP];
  __shared__ unsigned bad;
  const int tid = threadIdx.x;
  const unsigned long long found = *count;
  if (tid == 0) bad = 0u;
  __syncthreads();   // every thread has the count before it is reset
  const bool small = a.want && found <= (unsigned long long)SMALL_CAP && (long long)found <= a.buffer;
  if (small && found > 0) {
    const int n = (int)found;
    int n2 = 2;
    while (n2 < n) n2 <<= 1;
    for (int i = tid; i < n2; i += SMALL_NT) {
      unsigned long long k = ~0ull;
      if (i < n) {
        const CandEntry c = cand[i];
        const long long t = drain_template(c, a.s, a.nsearch, a.search0, a.nseg, &bad);
        if (t >= 0) k = ((((unsigned long long)t << 20) | (unsigned)c.bin) << 12) | (unsigned)i;
      }
      key[i] = k;
    }
    __syncthreads();
    for (int size = 2; size <= n2; size <<= 1)
      for (int step = size >> 1; step > 0; step >>= 1) {
        for (int p = tid; p < n2 / 2; p += SMALL_NT) {
          const int lo = 2 * p - (p & (step - 1)), hi = lo + step;
          const unsigned long long x = key[lo], y = key[hi];
          if ((x > y) == ((lo & size) == 0)) {
            key[lo] = y;
            key[hi] = x;
          }
        }
        __syncthreads();
      }
    if (!bad) {
      const int nout = (int)min((long long)n, a.capacity);
      for (int r = tid; r < nout; r += SMALL_NT) {
        const CandEntry c = cand[key[r] & (SMALL_CAP - 1)];
        keys[r] = drain_key(c, a.scored);
        out[r] = drain_record(c, a.l[c.search - a.search0], segs[c.segment]);
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    const unsigned done = !a.want || (small && !bad);
    head->count = found;
    head->bad = bad;
    head->done = done;
    if (done) *count = 0ull;
    __threadfence_system();
  }
}

}  // namespace fstat
