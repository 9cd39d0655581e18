// k_bin.hip -- pointing preprocessing: bin samples by interpolation anchor.
//
// The interpolation stencil of a pointing starts at the grid node
// (row0, col0) = (floor(theta / h_theta), floor(phi / h_phi)) in map storage
// coordinates; every sample with the same anchor reads the same W x W x ncomp
// block of the component maps.  A counting sort groups the samples by anchor
// so that the gather can stage one block in LDS and reuse it for all of them:
//
//   k_bin_keys     anchor key and rank within the key per sample (counts
//                  aggregated per workgroup in LDS, one global atomic per key)
//   k_scan_*       exclusive scan of (samples, work items) per key, in two or three kernels
//   k_bin_scatter  sample records in key order: fractional offsets and psi
//                  (FP64) and the original index, 32 bytes each
//   k_bin_items    work items (key, first sorted sample, count <= the plan's bin chunk);
//                  anchors of at most BIN_SHORT samples for the split gather, BIN_SHORT_SC64
//                  for the FP64 scatter, are listed apart, from the end of the item array down
//   k_bin_small    all of it in one workgroup, for passes of at most BIN_SMALL samples
//
// Integer index arithmetic is exact; the fractional offsets u - floor(u) are
// kept in FP64 (the FP32 gather rounds them when it forms its weights).
#include <algorithm>

#include "sc_common.h"

namespace {

__global__ void k_fill_int(int *a, int64_t n, int v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = v;
}

__device__ __forceinline__ void anchor_of(const double *ptg, int64_t s, const BinGeom &g, int &row0, int &col0,
                                          double &fu, double &fv, double &psi) {
    const double two_pi = 6.283185307179586477;
    const double th = ptg[3 * s], ph = ptg[3 * s + 1], ps = ptg[3 * s + 2];
    double u = th * g.inv_hth;
    u = fmin(fmax(u, 0.0), 0.5 * (double)g.n2os);  // also maps NaN to 0
    double v = (ph - two_pi * floor(ph / two_pi)) * g.inv_hph;
    if (!(v < (double)g.nphi) || v < 0.0) v = 0.0;
    const double flu = floor(u), flv = floor(v);
    row0 = (int)flu;
    col0 = (int)flv;
    fu = u - flu;
    fv = v - flv;
    psi = ps - two_pi * floor(ps / two_pi);
    if (!(psi >= 0.0 && psi < two_pi)) psi = 0.0;
}

// Anchor key and rank within the key.  A scan crosses about one anchor cell per
// sample but retraces nearly the same cells on consecutive spin circles, so a
// workgroup's span of consecutive samples hits each of its keys several times.
// The workgroup counts its keys in an LDS hash table (local ranks from LDS
// atomics), then reserves one global range per distinct key (one global atomic
// per key instead of per sample): rank = global base + local rank.  Keys that find
// no free slot within the probe limit take a global rank directly.  Ranges of
// different workgroups, and direct ranks, are disjoint by construction.
// SPT samples per thread: long passes take spans of 16384 samples (about 8 scan
// circles), so a scan's keys are counted mostly in LDS; with spans of 4096 or 1024 the
// global atomics of retraced cells cost more than the idle CUs (lmax 512, 1e7 scan
// samples, whole interpolation: 1.03 ms against 1.21 and 1.52 ms).  Passes below 2^19
// samples take 4096 and below 2^17 1024: their few workgroups are what bounds them (2e5
// scan samples at lmax 128: 74 against 81 us).  Samples that are spread evenly overflow
// the table: the short probe limit sends them to the global counter early (1e5 uniform
// pointings: this kernel 193 us in spans of 16384 with 64 probes, 8 us now).
constexpr int KEYS_NT = 1024;        // threads per workgroup
constexpr int KEYS_HT = 8192;        // hash slots
constexpr int KEYS_PROBE = 8;       // linear-probe limit
constexpr int KEYS_EMPTY = -1;

template <int KEYS_SPT>
__global__ void __launch_bounds__(KEYS_NT) k_bin_keys(const double *__restrict__ ptg, int64_t n, BinGeom g,
                                                      int *__restrict__ key, int *__restrict__ rank,
                                                      int *__restrict__ count) {
    __shared__ int hkey[KEYS_HT];
    __shared__ int hcnt[KEYS_HT];  // local count, then the key's global base
    const int tid = threadIdx.x;
    for (int i = tid; i < KEYS_HT; i += KEYS_NT) {
        hkey[i] = KEYS_EMPTY;
        hcnt[i] = 0;
    }
    __syncthreads();
    const int64_t s0 = (int64_t)blockIdx.x * (KEYS_NT * KEYS_SPT);
    int kk[KEYS_SPT], slot[KEYS_SPT], lr[KEYS_SPT];
#pragma unroll
    for (int i = 0; i < KEYS_SPT; ++i) {  // all keys first: the pointing loads overlap
        const int64_t s = s0 + tid + (int64_t)i * KEYS_NT;
        kk[i] = -1;
        if (s < n) {
            int r0, c0;
            double fu, fv, psi;
            anchor_of(ptg, s, g, r0, c0, fu, fv, psi);
            kk[i] = r0 * g.nkc + c0;
            key[s] = kk[i];
        }
    }
#pragma unroll
    for (int i = 0; i < KEYS_SPT; ++i) {
        const int k = kk[i];
        slot[i] = -1;
        lr[i] = 0;
        if (k >= 0) {
            int h = (int)(((unsigned)k * 2654435761u) >> 19) & (KEYS_HT - 1);
            for (int q = 0; q < KEYS_PROBE; ++q) {
                int cur = hkey[h];
                if (cur == KEYS_EMPTY) cur = atomicCAS(&hkey[h], KEYS_EMPTY, k);
                if (cur == KEYS_EMPTY || cur == k) {
                    slot[i] = h;
                    lr[i] = atomicAdd(&hcnt[h], 1);
                    break;
                }
                h = (h + 1) & (KEYS_HT - 1);
            }
            if (slot[i] < 0) lr[i] = atomicAdd(&count[k], 1);  // table full along the probe path
        }
    }
    __syncthreads();
    for (int i = tid; i < KEYS_HT; i += KEYS_NT) {
        const int k = hkey[i];
        if (k != KEYS_EMPTY) hcnt[i] = atomicAdd(&count[k], hcnt[i]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KEYS_SPT; ++i) {
        const int64_t s = s0 + tid + (int64_t)i * KEYS_NT;
        if (s < n) rank[s] = slot[i] >= 0 ? hcnt[slot[i]] + lr[i] : lr[i];
    }
}

// --- exclusive scan of int2 (x: samples per key, y: items per key) ------------
constexpr int SCAN_NT = 256;
constexpr int SCAN_PER = 16;
constexpr int SCAN_BLOCK = SCAN_NT * SCAN_PER;

__device__ __forceinline__ int2 key_pair(const int *count, int64_t i, int64_t nkeys, int chunk, int shortn) {
    if (i >= nkeys) return make_int2(0, 0);
    const int c = count[i];
    return make_int2(c, c <= shortn ? 0 : (c + chunk - 1) / chunk);  // short anchors are listed apart
}

// block-wide exclusive scan of one int2 per thread; returns the block total.  In registers
// within a wave (through LDS with a barrier per step it took 2 us of a small scan's 7).
__device__ int2 block_scan(int2 v, int2 *sh, int &excl_x, int &excl_y) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int2 incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_up(incl.x, off), y = __shfl_up(incl.y, off);
        if (lane >= off) {
            incl.x += x;
            incl.y += y;
        }
    }
    if (lane == 63) sh[wv] = incl;
    __syncthreads();
    int2 tot = make_int2(0, 0);
    excl_x = incl.x - v.x;
    excl_y = incl.y - v.y;
#pragma unroll
    for (int w = 0; w < SCAN_NT / 64; ++w) {
        const int2 t = sh[w];
        if (w < wv) {
            excl_x += t.x;
            excl_y += t.y;
        }
        tot.x += t.x;
        tot.y += t.y;
    }
    __syncthreads();
    return tot;
}

__global__ void __launch_bounds__(SCAN_NT) k_scan_reduce(const int *__restrict__ count, int64_t nkeys,
                                                         int2 *__restrict__ sums, int chunk, int shortn) {
    __shared__ int2 sh[SCAN_NT / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + (int64_t)threadIdx.x * SCAN_PER;
    int2 acc = make_int2(0, 0);
    for (int q = 0; q < SCAN_PER; ++q) {
        const int2 v = key_pair(count, base + q, nkeys, chunk, shortn);
        acc.x += v.x;
        acc.y += v.y;
    }
    int ex, ey;
    const int2 tot = block_scan(acc, sh, ex, ey);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// single block: exclusive scan of the per-block sums; writes totals
__global__ void __launch_bounds__(SCAN_NT) k_scan_sums(int2 *__restrict__ sums, int nblk, int *__restrict__ totals) {
    __shared__ int2 sh[SCAN_NT / 64];
    int2 carry = make_int2(0, 0);
    for (int base = 0; base < nblk; base += SCAN_NT) {
        const int i = base + threadIdx.x;
        const int2 v = i < nblk ? sums[i] : make_int2(0, 0);
        int ex, ey;
        const int2 tot = block_scan(v, sh, ex, ey);
        if (i < nblk) sums[i] = make_int2(carry.x + ex, carry.y + ey);
        carry.x += tot.x;
        carry.y += tot.y;
    }
    if (threadIdx.x == 0) {
        totals[0] = carry.x;  // samples
        totals[1] = carry.y;  // work items
        totals[2] = 0;        // work-queue cursor of the gather
        totals[3] = 0;        // short items
    }
}

// OWN: sums are the per-block sums as k_scan_reduce left them; every block adds up those before
// its own, the last one writes the totals, and k_scan_sums need not run (a launch of 4 us; with
// up to SCAN_OWN blocks, 4.2e6 anchors, they read 8 KB each at most).
constexpr int SCAN_OWN = 1024;
template <bool OWN>
__global__ void __launch_bounds__(SCAN_NT) k_scan_apply(const int *__restrict__ count, int64_t nkeys,
                                                        const int2 *__restrict__ sums, int2 *__restrict__ offs,
                                                        int chunk, int shortn, int *__restrict__ totals) {
    __shared__ int2 sh[SCAN_NT / 64];
    int2 bo = make_int2(0, 0);
    if (OWN) {
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += SCAN_NT) {
            bo.x += sums[i].x;
            bo.y += sums[i].y;
        }
        int ex, ey;
        bo = block_scan(bo, sh, ex, ey);
    } else {
        bo = sums[blockIdx.x];
    }
    const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + (int64_t)threadIdx.x * SCAN_PER;
    int2 v[SCAN_PER];
    int2 acc = make_int2(0, 0);
    for (int q = 0; q < SCAN_PER; ++q) {
        v[q] = key_pair(count, base + q, nkeys, chunk, shortn);
        acc.x += v[q].x;
        acc.y += v[q].y;
    }
    int ex, ey;
    const int2 tot = block_scan(acc, sh, ex, ey);
    if (OWN && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        totals[0] = bo.x + tot.x;
        totals[1] = bo.y + tot.y;
        totals[2] = 0;
        totals[3] = 0;
    }
    int2 run = make_int2(bo.x + ex, bo.y + ey);
    for (int q = 0; q < SCAN_PER; ++q) {
        if (base + q < nkeys) offs[base + q] = run;
        run.x += v[q].x;
        run.y += v[q].y;
    }
}

// The four 8-byte words of a sample's record: BinRec, or with y the adjoint layout.
struct RecWords {
    double w[4];
};
__device__ __forceinline__ double word2(int lo, int hi) {
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ RecWords make_rec(double fu, double fv, double psi, int s, const float *__restrict__ y) {
    if (!y) return RecWords{{fu, fv, psi, word2(s, 0)}};
    double sn, cs;
    sincos(psi, &sn, &cs);
    return RecWords{{word2(__float_as_int((float)fu), __float_as_int((float)fv)), cs, sn, word2(__float_as_int(y[s]), s)}};
}

// Sample records in anchor order.  Lane pairs write the two 16-byte halves of one
// record in the same instruction (one 32-byte run per sample, not four partial
// writes); the values come from the sample's own lane by shuffles.  (Blocks are
// whole waves.)  Samples of one key within a span of consecutive samples have
// consecutive ranks, so their records are neighbours: the blocks of a span run on
// one XCD, whose L2 merges those partial-line writes.
__global__ void k_bin_scatter(const double *__restrict__ ptg, int64_t n, BinGeom g, const int *__restrict__ key,
                              const int *__restrict__ rank, const int2 *__restrict__ offs, BinSorted out,
                              const float *__restrict__ y) {
    const int64_t s = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const bool valid = s < n;
    int pos = -1;
    RecWords rw = {{0.0, 0.0, 0.0, 0.0}};
    if (valid) {
        int r0, c0;
        double fu, fv, psi;
        anchor_of(ptg, s, g, r0, c0, fu, fv, psi);
        pos = offs[key[s]].x + rank[s];
        rw = make_rec(fu, fv, psi, (int)s, y);
    }
    const int lane = threadIdx.x & 63;
    const int hi = lane & 1;
    double2 *rec2 = (double2 *)out.rec;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int src = (lane >> 1) + 32 * half;  // the wave lane whose sample this lane writes
        const int p = __shfl(pos, src);
        const double w0 = __shfl(rw.w[0], src), w1 = __shfl(rw.w[1], src);
        const double w2 = __shfl(rw.w[2], src), w3 = __shfl(rw.w[3], src);
        if (p >= 0) {
            const double2 v = hi ? make_double2(w2, w3) : make_double2(w0, w1);
            rec2[2 * (size_t)p + hi] = v;
        }
    }
}

// A workgroup lists 256 PER anchors; the short ones among them get one reservation, so
// neighbouring anchors stay neighbours and the counter sees one atomic per workgroup (8 ns each:
// with one per wave of 64 anchors they took 0.35 ms of a pass of 1e5 uniform pointings at lmax
// 512).  PER = 16 from 2^20 anchors on, 4 from 2^18 on, else 1: few workgroups with many items
// each take long (lmax 32, 2e6 scan samples: 12 us at 4, 5 at 1).
constexpr int ITEMS_NT = 256;
template <int ITEMS_PER>
__global__ void __launch_bounds__(ITEMS_NT)
k_bin_items(const int *__restrict__ count, const int2 *__restrict__ offs, int64_t nkeys, int4 *__restrict__ items,
            int chunk, int shortn, int64_t cap, int *__restrict__ totals) {
    constexpr int NWV = ITEMS_NT / 64;
    static_assert(NWV * ITEMS_PER <= 64, "one wave scans the counts of every wave and step");
    __shared__ int before[NWV * ITEMS_PER];  // short anchors ahead of a wave's step
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t k0 = (int64_t)blockIdx.x * (ITEMS_NT * ITEMS_PER) + threadIdx.x;
    int c[ITEMS_PER];
#pragma unroll
    for (int q = 0; q < ITEMS_PER; ++q) {
        const int64_t k = k0 + q * ITEMS_NT;
        c[q] = k < nkeys ? count[k] : 0;
    }
    if (shortn > 0) {
#pragma unroll
        for (int q = 0; q < ITEMS_PER; ++q) {
            const unsigned long long mask = __ballot(c[q] > 0 && c[q] <= shortn);
            if (lane == 0) before[q * NWV + wv] = __popcll(mask);
        }
        __syncthreads();
        if (wv == 0) {
            const int n = lane < NWV * ITEMS_PER ? before[lane] : 0;
            int incl = n;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int t = __shfl_up(incl, off);
                if (lane >= off) incl += t;
            }
            int base = 0;
            if (lane == 63 && incl > 0) base = atomicAdd(&totals[3], incl);
            base = __shfl(base, 63);
            if (lane < NWV * ITEMS_PER) before[lane] = base + incl - n;
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < ITEMS_PER; ++q) {
        const int64_t k = k0 + q * ITEMS_NT;
        const bool is = c[q] > 0 && c[q] <= shortn;
        const unsigned long long mask = __ballot(is);
        if (c[q] == 0) continue;
        const int2 o = offs[k];
        if (is) {
            items[cap - 1 - (before[q * NWV + wv] + __popcll(mask & ((1ull << lane) - 1)))] =
                make_int4((int)k, o.x, c[q], 0);
        } else {
            for (int i = 0; i * chunk < c[q]; ++i) {
                const int cnt = c[q] - i * chunk < chunk ? c[q] - i * chunk : chunk;
                items[o.y + i] = make_int4((int)k, o.x + i * chunk, cnt, 0);
            }
        }
    }
}

// A pass of at most BIN_SMALL samples in one workgroup: an LDS hash table of the keys gives
// each sample its rank within its anchor, a scan over the slots the first record and work
// item of each anchor, and the records and items follow.  (Anchors come in slot order, not
// key order.)  The six or seven kernels of the general path cost a launch each, which is all that
// such a pass takes (1950 samples at lmax 256, interpolation with kmax 8: 66 us
// through the general path, 18 us, 9 of them here).
constexpr int SMALL_NT = 1024;
constexpr int SMALL_SPT = BIN_SMALL / SMALL_NT;
constexpr int SMALL_HT = 2 * BIN_SMALL;  // slots: at most half of them used, so every probe ends
constexpr int SMALL_HPT = SMALL_HT / SMALL_NT;

// SPLIT: anchors of at most shortn samples go to the short list (the FP64 scatter); otherwise it
// takes every item if shortn > 0 (the split gather).
template <bool SPLIT>
__global__ void __launch_bounds__(SMALL_NT)
k_bin_small(const double *__restrict__ ptg, int n, BinGeom g, BinSorted out, const float *__restrict__ y,
            int4 *__restrict__ items, int chunk, int shortn, int64_t cap, int *__restrict__ totals) {
    __shared__ int nshort;  // SPLIT only
    __shared__ int hkey[SMALL_HT];
    __shared__ int hcnt[SMALL_HT];  // samples of the slot's key, then its first record
    __shared__ unsigned sh[SMALL_NT / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
#pragma unroll
    for (int i = 0; i < SMALL_HPT; ++i) {
        hkey[tid + i * SMALL_NT] = KEYS_EMPTY;
        hcnt[tid + i * SMALL_NT] = 0;
    }
    if (SPLIT && tid == 0) nshort = 0;
    double fu[SMALL_SPT], fv[SMALL_SPT], psi[SMALL_SPT];
    int key[SMALL_SPT], slot[SMALL_SPT], rank[SMALL_SPT];
#pragma unroll
    for (int q = 0; q < SMALL_SPT; ++q) {
        const int s = tid + q * SMALL_NT;
        key[q] = -1;
        if (s < n) {
            int r0, c0;
            anchor_of(ptg, s, g, r0, c0, fu[q], fv[q], psi[q]);
            key[q] = r0 * g.nkc + c0;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SMALL_SPT; ++q) {
        const int k = key[q];
        if (k < 0) continue;
        int h = (int)(((unsigned)k * 2654435761u) >> 19) & (SMALL_HT - 1);
        for (;;) {  // ends: the table has more slots than keys
            int cur = hkey[h];
            if (cur == KEYS_EMPTY) cur = atomicCAS(&hkey[h], KEYS_EMPTY, k);
            if (cur == KEYS_EMPTY || cur == k) break;
            h = (h + 1) & (SMALL_HT - 1);
        }
        slot[q] = h;
        rank[q] = atomicAdd(&hcnt[h], 1);
    }
    __syncthreads();
    // exclusive scan over the slots of (items << 16 | samples); both stay below 2^13
    unsigned v[SMALL_HPT], sum = 0;
#pragma unroll
    for (int i = 0; i < SMALL_HPT; ++i) {
        const int c = hcnt[SMALL_HPT * tid + i];
        const int listed = SPLIT && c <= shortn ? 0 : (c + chunk - 1) / chunk;
        v[i] = ((unsigned)listed << 16) | (unsigned)c;
        sum += v[i];
    }
    unsigned incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
    }
    if (lane == 63) sh[wv] = incl;
    __syncthreads();
    unsigned run = incl - sum;
    for (int w = 0; w < wv; ++w) run += sh[w];
#pragma unroll
    for (int i = 0; i < SMALL_HPT; ++i) {
        const int c = (int)(v[i] & 0xffff), first = (int)(run & 0xffff), it = (int)(run >> 16);
        if (c) {
            const int k = hkey[SMALL_HPT * tid + i];
            hcnt[SMALL_HPT * tid + i] = first;
            if (SPLIT && c <= shortn)
                items[cap - 1 - atomicAdd(&nshort, 1)] = make_int4(k, first, c, 0);
            else
                for (int q = 0; q * chunk < c; ++q)
                    items[!SPLIT && shortn > 0 ? cap - 1 - (it + q) : it + q] =
                        make_int4(k, first + q * chunk, c - q * chunk < chunk ? c - q * chunk : chunk, 0);
        }
        run += v[i];
    }
    if (SPLIT) __syncthreads();  // nshort is complete
    if (tid == SMALL_NT - 1) {
        const int nit = (int)(run >> 16);
        totals[0] = n;
        totals[1] = !SPLIT && shortn > 0 ? 0 : nit;
        totals[2] = 0;
        totals[3] = SPLIT ? nshort : shortn > 0 ? nit : 0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SMALL_SPT; ++q) {
        if (key[q] < 0) continue;
        const RecWords rw = make_rec(fu[q], fv[q], psi[q], tid + q * SMALL_NT, y);
        double2 *dst = (double2 *)(out.rec + hcnt[slot[q]] + rank[q]);
        dst[0] = make_double2(rw.w[0], rw.w[1]);
        dst[1] = make_double2(rw.w[2], rw.w[3]);
    }
}

template <typename T>
__global__ void k_count_nonfinite(const T *__restrict__ x, int64_t n, int *count) {
    int c = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        c += isfinite(x[i]) ? 0 : 1;
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(count, c);
}

__global__ void k_zero_words(uint4 *a, int64_t nw) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void k_zero_bytes(unsigned char *a, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0;
}

}  // namespace

// Zero a device buffer with a kernel (no memset node if the caller captures a graph).
hipError_t sc_launch_zero(void *dst, size_t bytes, hipStream_t stream) {
    const int64_t nw = (int64_t)(bytes / 16);
    if (nw > 0) hipLaunchKernelGGL(k_zero_words, dim3(2048), dim3(256), 0, stream, (uint4 *)dst, nw);
    const int64_t tail = (int64_t)(bytes - 16 * (size_t)nw);
    if (tail > 0) hipLaunchKernelGGL(k_zero_bytes, dim3(1), dim3(64), 0, stream, (unsigned char *)dst + 16 * nw, tail);
    return hipGetLastError();
}

hipError_t sc_launch_count_nonfinite(const void *x, int64_t n, int f32, int *count, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    int64_t nb = (n + 255) / 256;
    if (nb > 4096) nb = 4096;
    if (f32)
        hipLaunchKernelGGL(k_count_nonfinite<float>, dim3((unsigned)nb), dim3(256), 0, stream, (const float *)x, n, count);
    else
        hipLaunchKernelGGL(k_count_nonfinite<double>, dim3((unsigned)nb), dim3(256), 0, stream, (const double *)x, n,
                           count);
    return hipGetLastError();
}

hipError_t sc_launch_binning(sc_plan *p, const double *ptg, int64_t n, const float *y, BinUse use) {
    BinWork &w = p->bw;
    w.last_n = n;
    const BinGeom g = sc_bin_geom(p);
    const int64_t nkeys = (int64_t)g.nkr * g.nkc;
    const int bs = 256;
    const unsigned gs = (unsigned)((n + bs - 1) / bs);
    int chunk = p->bin_chunk;
    if (p->prec == SC_FP64) chunk = std::min(chunk, use == SC_BIN_SCATTER ? BIN_CHUNK_SC64 : BIN_CHUNK_64);
    const int shortn = use == SC_BIN_GATHER && sc_short_items(p, n) ? BIN_SHORT
                       : use == SC_BIN_SCATTER && sc_short_items64(p) ? BIN_SHORT_SC64
                                                                      : 0;
    // (the deterministic scatter reads the per-anchor tables of the general path)
    w.small = n <= BIN_SMALL && !(use == SC_BIN_SCATTER && p->det_adjoint);
    if (w.small) {
        const bool split = use == SC_BIN_SCATTER && shortn > 0;
        hipLaunchKernelGGL(split ? k_bin_small<true> : k_bin_small<false>, dim3(1), dim3(SMALL_NT), 0, p->stream, ptg,
                           (int)n, g, w.sorted, y, w.items,
                           !split && shortn > 0 ? shortn : std::min(chunk, BIN_CHUNK), shortn, w.cap, w.totals);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_fill_int, dim3(1024), dim3(256), 0, p->stream, w.count, nkeys, 0);
    const int spt = n >= (1 << 19) ? 16 : n >= (1 << 17) ? 4 : 1;
    const unsigned gk = (unsigned)((n + KEYS_NT * spt - 1) / (KEYS_NT * spt));
    auto keys = spt == 16 ? k_bin_keys<16> : spt == 4 ? k_bin_keys<4> : k_bin_keys<1>;
    hipLaunchKernelGGL(keys, dim3(gk), dim3(KEYS_NT), 0, p->stream, ptg, n, g, w.key, w.rank, w.count);
    const int nblk = (int)((nkeys + SCAN_BLOCK - 1) / SCAN_BLOCK);
    hipLaunchKernelGGL(k_scan_reduce, dim3(nblk), dim3(SCAN_NT), 0, p->stream, w.count, nkeys, w.sums, chunk, shortn);
    const bool own = nblk <= SCAN_OWN;
    if (!own) hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(SCAN_NT), 0, p->stream, w.sums, nblk, w.totals);
    hipLaunchKernelGGL(own ? k_scan_apply<true> : k_scan_apply<false>, dim3(nblk), dim3(SCAN_NT), 0, p->stream, w.count,
                       nkeys, w.sums, w.offs, chunk, shortn, w.totals);
    hipLaunchKernelGGL(k_bin_scatter, dim3(gs), dim3(bs), 0, p->stream, ptg, n, g, w.key, w.rank, w.offs, w.sorted, y);
    const int q = nkeys >= (1 << 20) ? 16 : nkeys >= (1 << 18) ? 4 : 1;
    const int64_t per = ITEMS_NT * q;
    hipLaunchKernelGGL(q == 16 ? k_bin_items<16> : q == 4 ? k_bin_items<4> : k_bin_items<1>,
                       dim3((unsigned)((nkeys + per - 1) / per)), dim3(ITEMS_NT), 0, p->stream, w.count, w.offs, nkeys,
                       w.items, chunk, shortn, w.cap, w.totals);
    return hipGetLastError();
}
