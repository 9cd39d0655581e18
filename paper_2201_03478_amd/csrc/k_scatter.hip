// k_scatter.hip -- adjoint of the interpolation + k-sum (scatter to gradient maps).
//
// The gather computes c_t = sum_{taps} w_t(tap) sum_c basis_c(psi_t) M_c[tap]
// (k_gather.hip).  Its adjoint for a TOD gradient y is
//     GM_c[p] = sum_t y_t w_t(p) basis_c(psi_t)
// over the samples whose stencil covers map pixel p.  Different samples and
// anchors add into the same pixels, so the result is accumulated with
// hardware floating-point atomics (order-dependent rounding, Z15).
//
//  * k_scatter_mfma (FP32 maps, W = 8): per work item (samples of one anchor,
//    k_bin.hip) the 64 x ncomp patch gradient PG[t][c] = sum_s w_s(t) V[s][c],
//    V[s][c] = y_s basis_c(psi_s), is a v_mfma_f32_16x16x4_f32 product summed
//    over all chunks of the item, then added to the maps with one atomic per
//    (tap, component).  Each sample's record (the binning's adjoint layout, with
//    e^{i psi} and the TOD gradient) is read once, by one thread, and the tap
//    weight w_s(t) = w_theta(t / 8) w_phi(t % 8) is formed from the 1-d weights
//    in LDS as the matrix operand is read.  The atomics are not what limits it:
//    without them the kernel takes within 2% of the time.
//  * k_scatter_mfma64 (FP64 maps): the same product in FP64 for every even W; anchors of at
//    most four samples go to k_scatter_short64, one wave each.
//  * k_scatter_direct (FP32 maps with W != 8; FP64 passes too small to pay for the binning, or
//    without its workspace; the forced per-sample path): one wave per sample, lanes over
//    components, one atomic per (tap, component, sample).
#include <algorithm>

#include "sc_common.h"

typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

// exp(beta (sqrt(1 - z^2) - 1)) without the cancellation next to z = 0
template <typename T>
__device__ __forceinline__ T es_w(T z, T beta) {
    const T z2 = z * z, q = (T)1 - z2;
    return q > (T)0 ? exp(-beta * z2 / ((T)1 + sqrt(q))) : (T)0;
}

__device__ __forceinline__ void atomic_add(float *p, float v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void atomic_add(double *p, double v) { unsafeAtomicAdd(p, v); }

__device__ __forceinline__ double2 cpow_int(double2 z, int n) {
    double2 r = make_double2(1.0, 0.0);
    while (n) {
        if (n & 1) r = cmul(r, z);
        z = cmul(z, z);
        n >>= 1;
    }
    return r;
}

template <typename T>
__global__ void __launch_bounds__(256)
k_scatter_direct(const double *__restrict__ ptg, int64_t n, const T *__restrict__ y, T *__restrict__ gmaps, int cols,
                 int ncp, int ncomp, int W, double beta, double inv_hth, double inv_hph, int n2os, int nphi) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int half = W / 2;
    const double two_pi = 6.283185307179586477;
    for (int64_t s = wave; s < n; s += nwaves) {
        const double th = ptg[3 * s], ph = ptg[3 * s + 1], ps = ptg[3 * s + 2];
        double u = th * inv_hth;
        u = fmin(fmax(u, 0.0), 0.5 * (double)n2os);
        const int r0 = (int)floor(u) - half + 1;
        double v = (ph - two_pi * floor(ph / two_pi)) * inv_hph;
        if (!(v < (double)nphi) || v < 0.0) v = 0.0;
        const int q0 = (int)floor(v) - half + 1;
        T w = (T)0;
        if (lane < W)
            w = es_w<T>((T)((u - (double)(r0 + lane)) / half), (T)beta);
        else if (lane < 2 * W)
            w = es_w<T>((T)((v - (double)(q0 + lane - W)) / half), (T)beta);
        const double psr = ps - two_pi * floor(ps / two_pi);
        const T ys = y[s];
        T val[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int c = lane + 64 * t;
            T bas = (T)0;
            if (c < ncomp) {
                double sn, cs;
                sincos((double)(c >> 1) * psr, &sn, &cs);
                bas = (T)((c & 1) ? sn : cs);
            }
            val[t] = ys * bas;
        }
        const int row0 = r0 + half - 1, col0 = q0 + half - 1;
        for (int i = 0; i < W; ++i) {
            const T wi = __shfl(w, i);
            for (int j = 0; j < W; ++j) {
                const T wij = wi * __shfl(w, W + j);
                T *base = gmaps + ((size_t)(row0 + i) * cols + (col0 + j)) * ncp;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = lane + 64 * t;
                    if (c < ncomp && c != 1) atomic_add(base + c, wij * val[t]);  // basis_1 = sin 0 = 0
                }
            }
        }
    }
}

constexpr int W1ROW = 65;  // row stride of the 1-d weights: the 8 phi rows of one sample in distinct banks

template <int CT>
struct ScatterLds {
    static constexpr int NC = 16 * CT;
    static constexpr size_t bytes = sizeof(float) * (64 * NC + 16 * W1ROW) + 64 * (sizeof(double2) + sizeof(float2) +
                                                                                    sizeof(float));
};

// Work items come from the binning's queue; each chunk's samples (AdjRec, written
// by the binning with e^{i psi} and the TOD gradient) are staged by one thread each.
template <int CT, bool DET>
__global__ void __launch_bounds__(256)
k_scatter_mfma(const int4 *__restrict__ items, int *__restrict__ totals, const AdjRec *__restrict__ rec,
               const int *__restrict__ perm, float *__restrict__ gmaps, float *__restrict__ pg, int cols, int ncp,
               int ncomp, int nkc, double beta) {
    constexpr int NC = 16 * CT;
    extern __shared__ __attribute__((aligned(16))) double smem_d[];  // 16-byte operands
    float *Vsh = (float *)smem_d;                // [64 samples][NC]
    float *W1 = Vsh + 64 * NC;                   // [16][W1ROW]: theta weights (rows 0-7), phi weights (8-15)
    double2 *E1 = (double2 *)(W1 + 16 * W1ROW);  // [64] e^{i psi} (64 NC + 1040 floats: 16-byte aligned)
    float2 *UV = (float2 *)(E1 + 64);            // [64] (u - floor u, v - floor v)
    float *Ys = (float *)(UV + 64);              // [64]
    __shared__ int item_sh;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int r = lane & 15, grp = lane >> 4;
    const int nitems = totals[1];
    const float nbl = -(float)beta * 1.44269504088896341f;  // -beta log2(e)
    // with many items (over ~64 per workgroup) they are taken in runs of consecutive
    // ones, one queue atomic per run (the single counter is contended otherwise)
    int run = nitems / (64 * (int)gridDim.x);
    run = run < 1 ? 1 : (run > 32 ? 32 : run);
    for (;;) {
        if (tid == 0) item_sh = atomicAdd(&totals[2], run);
        __syncthreads();
        const int i0 = __builtin_amdgcn_readfirstlane(item_sh);  // read before the first barrier below
        if (i0 >= nitems) break;
        const int iend = i0 + run < nitems ? i0 + run : nitems;
        for (int it = i0; it < iend; ++it) {
            const int4 item = items[it];
            const int row0 = item.x / nkc, col0 = item.x - (item.x / nkc) * nkc;
            floatx4 acc[CT];
    #pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int ch = 0; ch < item.z; ch += 64) {
                const int ns = item.z - ch < 64 ? item.z - ch : 64;
                if (tid < 64) {
                    double2 e1 = make_double2(1.0, 0.0);
                    float2 uv = make_float2(0.f, 0.f);
                    float yy = 0.f;
                    if (tid < ns) {
                        const int pos = DET ? perm[item.y + ch + tid] : item.y + ch + tid;
                        const AdjRec q = rec[pos];
                        e1 = make_double2(q.cps, q.sps);
                        uv = make_float2(q.fu, q.fv);
                        yy = q.y;
                    }
                    E1[tid] = e1;
                    UV[tid] = uv;
                    Ys[tid] = yy;
                }
                __syncthreads();
                for (int e = tid; e < 64 * 16; e += 256) {
                    const int q = e >> 6, sl = e & 63;
                    float w = 0.f;
                    if (sl < ns) {
                        const float2 uv = UV[sl];
                        w = es_weight_f32(((q < 8 ? uv.x : uv.y) + (float)(3 - (q & 7))) * 0.25f, nbl);
                    }
                    W1[q * W1ROW + sl] = w;
                }
                {
                    // V[s][c] = y_s basis_c(psi_s): 4 lanes per sample, NC/4 components each
                    const int sl = tid >> 2, qq = tid & 3;
                    constexpr int PER = NC / 4;
                    const int c0 = qq * PER;
                    const double2 e1 = E1[sl];
                    const float yy = Ys[sl];
                    int kc = c0 >> 1;  // PER is even: the range starts on a cos/sin pair
                    double2 z = cpow_int(e1, kc);
                    float *vrow = Vsh + sl * NC;
                    for (int j = 0; j < PER; ++j) {
                        const int c = c0 + j;
                        float vv = 0.f;
                        if (c < ncomp) {
                            if ((c >> 1) > kc) {
                                z = cmul(z, e1);
                                ++kc;
                            }
                            vv = yy * (float)((c & 1) ? z.y : z.x);
                        }
                        vrow[c] = vv;
                    }
                }
                __syncthreads();
                // PG[tap][c] += sum_s W[tap][s] V[s][c] with W[tap][s] = w_theta_s(tap / 8) w_phi_s(tap % 8)
                // formed from the 1-d weights as the operand is read; wave wv owns taps 16 wv .. 16 wv + 15
                const int tap = 16 * wv + r;
                const float *wth = W1 + (tap >> 3) * W1ROW + grp;  // A[i = tap r][k = sample grp]
                const float *wph = W1 + (8 + (tap & 7)) * W1ROW + grp;
                const float *vb = Vsh + grp * NC + r;               // B[k = sample grp][j = comp r]
    #pragma unroll 4
                for (int ks = 0; ks < 16; ++ks) {
                    const float a = wth[4 * ks] * wph[4 * ks];
    #pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, vb[4 * ks * NC + 16 * ct], acc[ct], 0, 0, 0);
                }
                __syncthreads();
            }
            // D[i][j] in lane j + 16 (i/4), register i%4: tap 16 wv + 4 grp + v, component 16 ct + r
    #pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = 16 * wv + 4 * grp + v;
                if constexpr (DET) {
                    // the item's patch gradient, summed per pixel in a fixed order by k_scatter_reduce
                    float *dst = pg + ((size_t)it * 64 + t) * NC;
    #pragma unroll
                    for (int ct = 0; ct < CT; ++ct) dst[16 * ct + r] = acc[ct][v];
                } else {
                    float *base = gmaps + ((size_t)(row0 + (t >> 3)) * cols + (col0 + (t & 7))) * ncp;
    #pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int c = 16 * ct + r;
                        if (c < ncomp && c != 1) atomic_add(base + c, acc[ct][v]);  // basis_1 = sin 0 = 0
                    }
                }
            }
        }
    }
}

// Split products (the default): the same patch gradients from
// v_mfma_f32_16x16x32_f16, to FP32 accuracy.  Operands are written as two FP16
// parts, x = hi + lo with hi = fp16(x), lo = fp16(x - hi) (|x - hi - lo| <= 2^-22 |x|),
// and PG ~ Wh Vh + Wh Vl + Wl Vh (the omitted Wl Vl is below 2^-22 of the product):
// three FP16 products per 16 x 16 x 32 block, 3/16 of the matrix time of the FP32
// form.  Ranges: tap weights (in [0, 1]) are scaled by 2^14, the chunk's V by
// 2^(14 - e) with 2^e above its largest |y|; each chunk's product goes to a
// temporary accumulator that is added, unscaled, into the item's sums.  The
// operand layout of the 16x16x32 instruction: A[i][k] in lane i + 16 (k / 8),
// element k % 8; B[k][j] in lane j + 16 (k / 8), element k % 8; D as in the FP32 form.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

template <int CT>
struct SplitScatterLds {
    static constexpr size_t bytes = 2 * (2 * (size_t)CT * 64 * sizeof(half8)) + sizeof(float) * 16 * W1ROW +
                                    64 * (sizeof(double2) + sizeof(float2) + sizeof(float));
};

template <int CT, bool DET>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CT <= 5 ? 5 : 3)))
k_scatter_split(const int4 *__restrict__ items, int *__restrict__ totals, const AdjRec *__restrict__ rec,
                const int *__restrict__ perm, float *__restrict__ gmaps, float *__restrict__ pg, int cols, int ncp,
                int ncomp, int nkc, double beta) {
    constexpr int NC = 16 * CT;
    extern __shared__ __attribute__((aligned(16))) double smem_d[];
    half8 *Bhi = (half8 *)smem_d;                // [2 sample halves][CT][64 lanes]
    half8 *Blo = Bhi + 2 * CT * 64;
    float *W1 = (float *)(Blo + 2 * CT * 64);    // [16][W1ROW]: theta weights (rows 0-7), phi weights (8-15)
    double2 *E1 = (double2 *)(W1 + 16 * W1ROW);  // [64] e^{i psi} (1040 floats after 16-byte blocks: aligned)
    float2 *UV = (float2 *)(E1 + 64);            // [64] (u - floor u, v - floor v)
    float *Ys = (float *)(UV + 64);              // [64] y 2^(14 - e)
    __shared__ int item_sh;
    __shared__ float osc_sh;  // 2^(e - 28): undoes both scalings

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int r = lane & 15, grp = lane >> 4;
    const int nitems = totals[1];
    const float nbl = -(float)beta * 1.44269504088896341f;  // -beta log2(e)
    // with many items (over ~64 per workgroup) they are taken in runs of consecutive
    // ones, one queue atomic per run (the single counter is contended otherwise)
    int run = nitems / (64 * (int)gridDim.x);
    run = run < 1 ? 1 : (run > 32 ? 32 : run);
    for (;;) {
        if (tid == 0) item_sh = atomicAdd(&totals[2], run);
        __syncthreads();
        const int i0 = __builtin_amdgcn_readfirstlane(item_sh);  // read before the first barrier below
        if (i0 >= nitems) break;
        const int iend = i0 + run < nitems ? i0 + run : nitems;
        for (int it = i0; it < iend; ++it) {
            const int4 item = items[it];
            const int row0 = item.x / nkc, col0 = item.x - (item.x / nkc) * nkc;
            floatx4 acc[CT];
    #pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int ch = 0; ch < item.z; ch += 64) {
                const int ns = item.z - ch < 64 ? item.z - ch : 64;
                if (tid < 64) {  // one wave: one sample per lane
                    double2 e1 = make_double2(1.0, 0.0);
                    float2 uv = make_float2(0.f, 0.f);
                    float yy = 0.f;
                    if (tid < ns) {
                        const int pos = DET ? perm[item.y + ch + tid] : item.y + ch + tid;
                        const AdjRec q = rec[pos];
                        e1 = make_double2(q.cps, q.sps);
                        uv = make_float2(q.fu, q.fv);
                        yy = q.y;
                    }
                    float m = fabsf(yy);
    #pragma unroll
                    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
                    int e = 0;
                    if (m > 0.f) (void)frexpf(m, &e);  // m < 2^e
                    E1[tid] = e1;
                    UV[tid] = uv;
                    Ys[tid] = ldexpf(yy, 14 - e);  // exact
                    if (tid == 0) osc_sh = ldexpf(1.f, e - 28);
                }
                __syncthreads();
                for (int e = tid; e < 64 * 16; e += 256) {
                    const int q = e >> 6, sl = e & 63;
                    float w = 0.f;
                    if (sl < ns) {
                        const float2 uv = UV[sl];
                        w = es_weight_f32(((q < 8 ? uv.x : uv.y) + (float)(3 - (q & 7))) * 0.25f, nbl);
                    }
                    W1[q * W1ROW + sl] = w;
                }
                {
                    // V[s][c] = y_s basis_c(psi_s) (scaled), split and written in the B layout:
                    // sample s -> half s / 32, lane group (s % 32) / 8, element s % 8; component c ->
                    // tile c / 16, lane c % 16.  4 lanes per sample; lane qq takes the orders
                    // k = qq + 4 j (components 2k, 2k + 1: tile j / 2, lanes 2 qq + 8 (j % 2) and
                    // the next), so its offsets are compile-time after the base, and steps the
                    // phase by e^{4 i psi}.
                    const int sl = tid >> 2, qq = tid & 3;
                    const double2 e1 = E1[sl];
                    const double2 e2 = cmul(e1, e1), e4 = cmul(e2, e2);
                    double2 z = qq == 0 ? make_double2(1.0, 0.0) : qq == 1 ? e1 : qq == 2 ? e2 : cmul(e2, e1);
                    const float yy = Ys[sl];
                    const int base = ((sl >> 5) * CT * 64 + 16 * ((sl & 31) >> 3)) * 8 + (sl & 7) + 16 * qq;
                    _Float16 *bh = (_Float16 *)Bhi + base, *bl = (_Float16 *)Blo + base;
    #pragma unroll
                    for (int j = 0; j < 2 * CT; ++j) {
                        const int k = qq + 4 * j;
                        const float vc = 2 * k < ncomp ? yy * (float)z.x : 0.f;
                        const float vs = 2 * k + 1 < ncomp ? yy * (float)z.y : 0.f;
                        const int o = (j >> 1) * 512 + 64 * (j & 1);
                        const _Float16 hc = (_Float16)vc, hs = (_Float16)vs;
                        bh[o] = hc;
                        bl[o] = (_Float16)(vc - (float)hc);
                        bh[o + 8] = hs;
                        bl[o + 8] = (_Float16)(vs - (float)hs);
                        z = cmul(z, e4);
                    }
                }
                __syncthreads();
                {
                    // A: wave wv's taps 16 wv + r, samples 32 kh + 8 grp + q
                    const int tap = 16 * wv + r;
                    const float *wth = W1 + (tap >> 3) * W1ROW + 8 * grp;
                    const float *wph = W1 + (8 + (tap & 7)) * W1ROW + 8 * grp;
                    half8 ah[2], al[2];
    #pragma unroll
                    for (int kh = 0; kh < 2; ++kh)
    #pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const float w = wth[32 * kh + q] * wph[32 * kh + q] * 16384.f;
                            const _Float16 h = (_Float16)w;
                            ah[kh][q] = h;
                            al[kh][q] = (_Float16)(w - (float)h);
                        }
                    const float osc = osc_sh;
    #pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        floatx4 t = floatx4{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
                        for (int kh = 0; kh < 2; ++kh) {
                            const half8 bh = Bhi[(kh * CT + ct) * 64 + lane], bl = Blo[(kh * CT + ct) * 64 + lane];
                            t = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[kh], bh, t, 0, 0, 0);
                            t = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[kh], bl, t, 0, 0, 0);
                            t = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[kh], bh, t, 0, 0, 0);
                        }
    #pragma unroll
                        for (int v = 0; v < 4; ++v) acc[ct][v] = fmaf(t[v], osc, acc[ct][v]);
                    }
                }
                __syncthreads();
            }
            // D[i][j] in lane j + 16 (i/4), register i%4: tap 16 wv + 4 grp + v, component 16 ct + r
    #pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = 16 * wv + 4 * grp + v;
                if constexpr (DET) {
                    // the item's patch gradient, summed per pixel in a fixed order by k_scatter_reduce
                    float *dst = pg + ((size_t)it * 64 + t) * NC;
    #pragma unroll
                    for (int ct = 0; ct < CT; ++ct) dst[16 * ct + r] = acc[ct][v];
                } else {
                    float *base = gmaps + ((size_t)(row0 + (t >> 3)) * cols + (col0 + (t & 7))) * ncp;
    #pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int c = 16 * ct + r;
                        if (c < ncomp && c != 1) atomic_add(base + c, acc[ct][v]);  // basis_1 = sin 0 = 0
                    }
                }
            }
        }
    }
}

// FP64 plans: the patch gradients as v_mfma_f64_16x16x4_f64 products (FP64 products and
// accumulation).  PG[t][c] = sum_s w_s(t) V[s][c] with a tile of 16 taps (16 columns of
// one row of the stencil, two rows at W <= 8, four at W = 4) x 16 components; operand
// layout A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k, D[i][j] in lane
// j + 16 (i % 4), element i / 4.  A workgroup takes items of at most S64 samples: their
// 1-d weights stay in LDS for every sweep over two component tiles, V is formed 64
// samples at a time, and wave w owns tap tiles w, w + 4, ...  One FP64 atomic per
// (tap, component, item): the sample-by-sample form (k_scatter_direct) issues one per
// (tap, component, sample) and is bound by them.  lmax 128, kmax 8, W = 14, 2e5 scan
// samples: 6.23 ms sample by sample (7.1e8 atomics), 0.13 ms here.
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int S64 = BIN_CHUNK_SC64;  // samples per item
constexpr int S64R = S64 + 4; // row stride of the weights: eight tap rows x four samples in distinct banks

template <int W>
struct Sc64 {
    static constexpr int RPT = W <= 4 ? 4 : W <= 8 ? 2 : 1;  // stencil rows per tap tile
    static constexpr int NT = (W + RPT - 1) / RPT;           // tap tiles
    static constexpr int TW = (NT + 3) / 4;                  // per wave
    static constexpr int NVS = 48;                           // row stride of V (two tiles + padding)
    static constexpr size_t lds() {
        return sizeof(double) * (2 * W * S64R + 64 * NVS + S64) + sizeof(double2) * S64;
    }
};

template <int W, int N>
__device__ __forceinline__ void scatter64_sweep(const double *Wt, double *V, const double2 *E1, const double *Ys, int ns,
                                                int cbase, double *__restrict__ gm, int cols, int ncp, int ncomp) {
    using C = Sc64<W>;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 15, grp = lane >> 4;
    const int tr = r / W, tc = r - tr * W;  // tap r of a tile: row tr, column tc
    const bool on = tr < C::RPT && r < C::RPT * W;
    const double *wph = Wt + (W + (on ? tc : 0)) * S64R + grp;
    const double *wth[C::TW];
#pragma unroll
    for (int q = 0; q < C::TW; ++q) {
        const int row = (wv + 4 * q) * C::RPT + (on ? tr : 0);
        wth[q] = Wt + (row < W ? row : W - 1) * S64R + grp;  // past the stencil: left out below
    }
    doublex4 acc[C::TW][N];
#pragma unroll
    for (int q = 0; q < C::TW; ++q)
#pragma unroll
        for (int c = 0; c < N; ++c) acc[q][c] = doublex4{0.0, 0.0, 0.0, 0.0};
    for (int s0 = 0; s0 < ns; s0 += 64) {
        __syncthreads();  // V's readers (and, first, the weights' writers) are done
        {
            // V[s][c] = y_s basis_c(psi_s): 4 lanes per sample, 2 N orders each; zero past ns
            const int sl = tid >> 2, k0 = (cbase >> 1) + 2 * N * (tid & 3);
            const bool in = s0 + sl < ns;
            const double2 e1 = in ? E1[s0 + sl] : make_double2(0.0, 0.0);
            const double yy = in ? Ys[s0 + sl] : 0.0;
            double2 z = cpow_int(e1, k0);
            double *v = V + sl * C::NVS + 4 * N * (tid & 3);
#pragma unroll
            for (int j = 0; j < 2 * N; ++j) {
                v[2 * j] = yy * z.x;
                v[2 * j + 1] = yy * z.y;
                z = cmul(z, e1);
            }
            if (!in)
#pragma unroll
                for (int j = 0; j < 4 * N; ++j) v[j] = 0.0;
        }
        __syncthreads();
        const int nk = (ns - s0 < 64 ? ns - s0 + 3 : 64) >> 2;
        const double *vb = V + grp * C::NVS + r;
#pragma unroll 2
        for (int ks = 0; ks < nk; ++ks) {
            double b[N];
#pragma unroll
            for (int c = 0; c < N; ++c) b[c] = vb[4 * ks * C::NVS + 16 * c];
            const double wf = wph[s0 + 4 * ks];
#pragma unroll
            for (int q = 0; q < C::TW; ++q) {
                const double a = wth[q][s0 + 4 * ks] * wf;
#pragma unroll
                for (int c = 0; c < N; ++c) acc[q][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[c], acc[q][c], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < C::TW; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int t = 4 * v + grp;  // tap of the tile
            const int row = (wv + 4 * q) * C::RPT + t / W, col = t - (t / W) * W;
            if (t >= C::RPT * W || row >= W) continue;
            double *base = gm + ((size_t)row * cols + col) * ncp;
#pragma unroll
            for (int c = 0; c < N; ++c) {
                const int cc = cbase + 16 * c + r;
                if (cc < ncomp && cc != 1) atomic_add(base + cc, acc[q][c][v]);  // basis_1 = sin 0 = 0
            }
        }
}

template <int W>
__global__ void __launch_bounds__(256)
k_scatter_mfma64(const int4 *__restrict__ items, const int *__restrict__ totals, const BinRec *__restrict__ rec,
                 const double *__restrict__ y, double *__restrict__ gmaps, int cols, int ncp, int ncomp, int nkc,
                 double beta) {
    extern __shared__ __attribute__((aligned(16))) double smem_d[];
    double2 *E1 = (double2 *)smem_d;         // [S64] e^{i psi}
    double *Ys = (double *)(E1 + S64);       // [S64]
    double *Wt = Ys + S64;                   // [2 W][S64R]: theta weights, then phi weights
    double *V = Wt + 2 * W * S64R;           // [64][NVS]
    const int tid = threadIdx.x;
    const int nitems = totals[1];
    const int nct = (ncomp + 15) >> 4;
    for (int it = xcd_remap(blockIdx.x, gridDim.x); it < nitems; it += gridDim.x) {
        const int4 item = items[it];
        const int row0 = item.x / nkc, col0 = item.x - (item.x / nkc) * nkc;
        double *gm = gmaps + ((size_t)row0 * cols + col0) * ncp;
        for (int ch = 0; ch < item.z; ch += S64) {
            const int ns = item.z - ch < S64 ? item.z - ch : S64;
            const BinRec *rc = rec + item.y + ch;
            if (tid < ns) {
                double sn, cs;
                sincos(rc[tid].psi, &sn, &cs);
                E1[tid] = make_double2(cs, sn);
                Ys[tid] = y[rc[tid].idx];
            }
            const int nsp = (ns + 3) & ~3;  // whole steps of four samples
            for (int e = tid; e < 2 * W * S64; e += 256) {
                const int node = e / S64, sl = e - node * S64;
                if (sl < nsp) {
                    double w = 0.0;
                    if (sl < ns) {
                        const bool th = node < W;
                        const double f = th ? rc[sl].fu : rc[sl].fv;
                        w = es_w<double>((f + (double)(W / 2 - 1 - (th ? node : node - W))) / (double)(W / 2), beta);
                    }
                    Wt[node * S64R + sl] = w;
                }
            }
            int ct = 0;
            for (; ct + 2 <= nct; ct += 2) scatter64_sweep<W, 2>(Wt, V, E1, Ys, ns, 16 * ct, gm, cols, ncp, ncomp);
            if (ct < nct) scatter64_sweep<W, 1>(Wt, V, E1, Ys, ns, 16 * ct, gm, cols, ncp, ncomp);
            __syncthreads();  // weights and phases are rewritten by the next samples
        }
    }
}

__device__ __forceinline__ double read_lane(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Anchors of at most BIN_SHORT_SC64 samples, one wave each: the sum over the samples in
// registers, one atomic per (tap, component), 64 of them at a time: CW components of 64 / CW
// neighbouring columns of one row, which share sectors (a column of 64 / CW rows instead: 1.6
// times the time at kmax 0), and whose theta weight is the same for the whole wave (read from a
// lane).  The matrix form costs such an item its barriers and LDS fills, about as much as the
// atomics of four samples: 1e5 uniform pointings, W = 14, lmax 512, kmax 0: 1.70 ms with it,
// 0.47 here, 0.92 sample by sample; kmax 8: 3.2, 2.3 and 2.6.
template <int W, int NS, int CW>
__device__ __forceinline__ void scatter64_samples(const BinRec *__restrict__ rc, int ns, const double *__restrict__ y,
                                                  double *__restrict__ gm, int cols, int ncp, int ncomp, double beta,
                                                  int lane) {
    constexpr int CP = 64 / CW, NG = (W + CP - 1) / CP;  // columns at a time, groups of them
    double w[NS], ys[NS];
    double2 e1[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        w[s] = ys[s] = 0.0;
        e1[s] = make_double2(0.0, 0.0);
        if (s < ns) {
            const BinRec q = rc[s];
            sincos(q.psi, &e1[s].y, &e1[s].x);
            ys[s] = y[q.idx];
            const bool th = lane < W;
            if (lane < 2 * W)
                w[s] = es_w<double>(((th ? q.fu : q.fv) + (double)(W / 2 - 1 - (th ? lane : lane - W))) / (double)(W / 2),
                                    beta);
        }
    }
    for (int c0 = 0; c0 < ncomp; c0 += CW) {
        const int c = c0 + lane % CW;
        double val[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const double2 z = cpow_int(e1[s], c >> 1);
            val[s] = ys[s] * ((c & 1) ? z.y : z.x);
        }
        const bool on = c < ncomp && c != 1;  // basis_1 = sin 0 = 0
        double vj[NG][NS];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int j = g * CP + lane / CW;
#pragma unroll
            for (int s = 0; s < NS; ++s) vj[g][s] = __shfl(w[s], W + (j < W ? j : 0)) * val[s];
        }
        for (int i = 0; i < W; ++i) {
            double wi[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) wi[s] = read_lane(w[s], i);
            double *row = gm + (size_t)i * cols * ncp + c;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int j = g * CP + lane / CW;
                double a = 0.0;
#pragma unroll
                for (int s = 0; s < NS; ++s) a = fma(wi[s], vj[g][s], a);
                if (on && j < W) atomic_add(row + (size_t)j * ncp, a);
            }
        }
    }
}
template <int W, int NS>
__device__ __forceinline__ void scatter64_short(const BinRec *__restrict__ rc, int ns, const double *__restrict__ y,
                                                double *__restrict__ gm, int cols, int ncp, int ncomp, double beta,
                                                int lane) {
    if (ncomp <= 4)
        scatter64_samples<W, NS, 4>(rc, ns, y, gm, cols, ncp, ncomp, beta, lane);
    else if (ncomp <= 16)
        scatter64_samples<W, NS, 16>(rc, ns, y, gm, cols, ncp, ncomp, beta, lane);
    else
        scatter64_samples<W, NS, 32>(rc, ns, y, gm, cols, ncp, ncomp, beta, lane);
}

template <int W>
__global__ void __launch_bounds__(256)
k_scatter_short64(const int4 *__restrict__ items, const int *__restrict__ totals, int64_t cap,
                  const BinRec *__restrict__ rec, const double *__restrict__ y, double *__restrict__ gmaps, int cols,
                  int ncp, int ncomp, int nkc, double beta) {
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nitems = totals[3];
    for (int it = xcd_remap(blockIdx.x, gridDim.x) * 4 + wv; it < nitems; it += gridDim.x * 4) {
        const int4 item = items[cap - 1 - it];
        const int row0 = item.x / nkc, col0 = item.x - (item.x / nkc) * nkc;
        double *gm = gmaps + ((size_t)row0 * cols + col0) * ncp;
        const BinRec *rc = rec + item.y;
        if (item.z == 1)
            scatter64_short<W, 1>(rc, 1, y, gm, cols, ncp, ncomp, beta, lane);
        else if (item.z == 2)
            scatter64_short<W, 2>(rc, 2, y, gm, cols, ncp, ncomp, beta, lane);
        else
            scatter64_short<W, BIN_SHORT_SC64>(rc, item.z, y, gm, cols, ncp, ncomp, beta, lane);
    }
}

template <int W>
hipError_t launch_scatter_mfma64(sc_plan *p, const double *y, double *gmaps) {
    const int nkc = sc_bin_geom(p).nkc;
    if (sc_short_items64(p)) {
        auto shrt = k_scatter_short64<W>;
        const int sgrid = (int)std::min<int64_t>(sc_persistent_grid((const void *)shrt, 256, 0, 0), (p->bw.last_n + 3) / 4);
        hipLaunchKernelGGL(shrt, dim3(sgrid), dim3(256), 0, p->stream, p->bw.items, p->bw.totals, p->bw.cap,
                           p->bw.sorted.rec, y, gmaps, p->cols, p->ncp, p->ncomp, nkc, p->beta);
    }
    const size_t lds = Sc64<W>::lds();
    auto kern = k_scatter_mfma64<W>;
    hipError_t e = sc_set_lds_attr((const void *)kern, lds);
    if (e != hipSuccess) return e;
    const int grid = sc_persistent_grid((const void *)kern, 256, lds, p->gather_wgs_per_cu);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, p->stream, p->bw.items, p->bw.totals, p->bw.sorted.rec, y, gmaps,
                       p->cols, p->ncp, p->ncomp, nkc, p->beta);
    return hipGetLastError();
}

// Deterministic mode, sample order.  The binning ranks the samples of an anchor in
// the order its atomics happen to run, so the same samples can land in different
// 64-sample chunks from run to run.  In this mode every anchor is one work item and
// this kernel sorts the item's samples by their index (a bitonic sort of (index,
// position) pairs in LDS, one workgroup per item of at most DET_MAXN samples), writing
// perm[first + i] = the sorted position of the i-th sample in index order; the scatter
// reads its records through perm.  It also records the largest item (totals[3]).
constexpr int DET_MAXN = 8192;

__global__ void __launch_bounds__(256)
k_det_order(const int4 *__restrict__ items, const int *__restrict__ totals, const AdjRec *__restrict__ rec,
            int *__restrict__ perm, int *__restrict__ maxn) {
    __shared__ unsigned key[DET_MAXN], val[DET_MAXN];
    const int it = blockIdx.x;
    if (it >= totals[1]) return;
    const int4 item = items[it];
    const int n = item.z, tid = threadIdx.x;
    if (tid == 0) atomicMax(maxn, n);
    if (n > DET_MAXN) return;  // the host splits the pass and bins again
    int np = 64;
    while (np < n) np <<= 1;
    for (int i = tid; i < np; i += 256) {
        key[i] = i < n ? (unsigned)rec[item.y + i].idx : 0xffffffffu;
        val[i] = (unsigned)(item.y + i);
    }
    __syncthreads();
    for (int k = 2; k <= np; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < np; i += 256) {
                const int l = i ^ j;
                if (l > i) {
                    const bool up = (i & k) == 0;
                    const unsigned a = key[i], b = key[l];
                    if ((a > b) == up) {
                        key[i] = b;
                        key[l] = a;
                        const unsigned t = val[i];
                        val[i] = val[l];
                        val[l] = t;
                    }
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < n; i += 256) perm[item.y + i] = (int)val[i];
}

// Deterministic mode: gmaps[R][C] += sum over the anchors (R - i, C - j), i, j < 8, in that
// order, and over each anchor's items in order, of the items' patch gradients at tap
// (i, j).  One workgroup per 8 x 8 pixel tile; the item ranges of the tile's 15 x 15
// anchors go to LDS first (an anchor's items are consecutive: ceil(count / chunk) of
// them from offs[key].y).  Thread (pixel, part) sums CT float4s of its pixel (the map
// record holds ncp <= 16 CT floats; the patch gradients 16 CT).
template <int CT>
__global__ void __launch_bounds__(256)
k_scatter_reduce(const float4 *__restrict__ pg, const int *__restrict__ count, const int2 *__restrict__ offs,
                 float *__restrict__ gmaps, int rows, int cols, int ncp, int nkr, int nkc, int chunk) {
    constexpr int NC4 = 4 * CT;  // float4s per tap
    __shared__ int2 rng[15 * 15];
    const int tiles_c = (cols + 7) / 8;
    const int R0 = 8 * (blockIdx.x / tiles_c), C0 = 8 * (blockIdx.x - (blockIdx.x / tiles_c) * tiles_c);
    const int tid = threadIdx.x;
    if (tid < 225) {
        const int ar = R0 - 7 + tid / 15, ac = C0 - 7 + tid % 15;
        int2 v = make_int2(0, 0);
        if (ar >= 0 && ar < nkr && ac >= 0 && ac < nkc) {
            const int64_t k = (int64_t)ar * nkc + ac;
            const int c = count[k];
            if (c > 0) v = make_int2(offs[k].y, (c + chunk - 1) / chunk);
        }
        rng[tid] = v;
    }
    __syncthreads();
    const int pix = tid >> 2, part = tid & 3;
    const int pr = pix >> 3, pc = pix & 7;
    const int R = R0 + pr, C = C0 + pc;
    if (R >= rows || C >= cols) return;
    float4 acc[CT];
#pragma unroll
    for (int q = 0; q < CT; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = 0; i < 8; ++i)
        for (int j = 0; j < 8; ++j) {
            const int2 g = rng[(pr + 7 - i) * 15 + (pc + 7 - j)];
            for (int it = g.x; it < g.x + g.y; ++it) {
                const float4 *src = pg + ((size_t)it * 64 + 8 * i + j) * NC4 + part * CT;
#pragma unroll
                for (int q = 0; q < CT; ++q) {
                    const float4 v = src[q];
                    acc[q].x += v.x;
                    acc[q].y += v.y;
                    acc[q].z += v.z;
                    acc[q].w += v.w;
                }
            }
        }
    float4 *dst = (float4 *)(gmaps + ((size_t)R * cols + C) * ncp) + part * CT;
#pragma unroll
    for (int q = 0; q < CT; ++q) {
        if (4 * (part * CT + q) >= ncp) break;  // CT may round the map's tile count up
        float4 o = dst[q];
        o.x += acc[q].x;
        o.y += acc[q].y;
        o.z += acc[q].z;
        o.w += acc[q].w;
        dst[q] = o;
    }
}

template <int CT>
hipError_t launch_scatter_split(sc_plan *p, void *gmaps) {
    const size_t lds = SplitScatterLds<CT>::bytes;
    auto kern = p->det_adjoint ? k_scatter_split<CT, true> : k_scatter_split<CT, false>;
    hipError_t e = sc_set_lds_attr((const void *)kern, lds);
    if (e != hipSuccess) return e;
    const int grid = sc_persistent_grid((const void *)kern, 256, lds, p->gather_wgs_per_cu);
    const BinGeom g = sc_bin_geom(p);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, p->stream, p->bw.items, p->bw.totals,
                       (const AdjRec *)p->bw.sorted.rec, p->bw.key, (float *)gmaps, p->pg, p->cols, p->ncp, p->ncomp,
                       g.nkc,
                       p->beta);
    return hipGetLastError();
}

template <int CT>
hipError_t launch_scatter_mfma(sc_plan *p, void *gmaps) {
    const size_t lds = ScatterLds<CT>::bytes;
    auto kern = p->det_adjoint ? k_scatter_mfma<CT, true> : k_scatter_mfma<CT, false>;
    hipError_t e = sc_set_lds_attr((const void *)kern, lds);
    if (e != hipSuccess) return e;
    const int grid = sc_persistent_grid((const void *)kern, 256, lds, p->gather_wgs_per_cu);
    const BinGeom g = sc_bin_geom(p);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, p->stream, p->bw.items, p->bw.totals,
                       (const AdjRec *)p->bw.sorted.rec, p->bw.key, (float *)gmaps, p->pg, p->cols, p->ncp, p->ncomp,
                       g.nkc,
                       p->beta);
    return hipGetLastError();
}

hipError_t launch_scatter_mfma_any(sc_plan *p, void *gmaps) {
    const int ct = (p->ncomp + 15) / 16;
    if (p->gather_mma == 1) {  // split FP16 products (the plan's product form, as for the gather)
        if (ct <= 1) return launch_scatter_split<1>(p, gmaps);
        if (ct <= 2) return launch_scatter_split<2>(p, gmaps);
        if (ct <= 3) return launch_scatter_split<3>(p, gmaps);
        if (ct <= 5) return launch_scatter_split<5>(p, gmaps);
        if (ct <= 9) return launch_scatter_split<9>(p, gmaps);
        if (ct <= 13) return launch_scatter_split<13>(p, gmaps);
        return launch_scatter_split<16>(p, gmaps);
    }
    if (ct <= 1) return launch_scatter_mfma<1>(p, gmaps);
    if (ct <= 2) return launch_scatter_mfma<2>(p, gmaps);
    if (ct <= 3) return launch_scatter_mfma<3>(p, gmaps);
    if (ct <= 5) return launch_scatter_mfma<5>(p, gmaps);
    if (ct <= 9) return launch_scatter_mfma<9>(p, gmaps);
    if (ct <= 13) return launch_scatter_mfma<13>(p, gmaps);
    return launch_scatter_mfma<16>(p, gmaps);
}

template <int CT>
hipError_t launch_reduce(sc_plan *p, void *gmaps) {
    const BinGeom g = sc_bin_geom(p);
    const int tiles = ((p->rows + 7) / 8) * ((p->cols + 7) / 8);
    hipLaunchKernelGGL(k_scatter_reduce<CT>, dim3(tiles), dim3(256), 0, p->stream, (const float4 *)p->pg,
                       p->bw.count, p->bw.offs, (float *)gmaps, p->rows, p->cols, p->ncp, g.nkr, g.nkc, p->bin_chunk);
    return hipGetLastError();
}

}  // namespace

bool sc_scatter_binned_supported(const sc_plan *p) {
    return p->prec != SC_FP64 && p->W == 8 && p->ncomp <= 256 && !p->gather_direct;
}

// Deterministic mode, after the binning (one item per anchor): the sample order of
// every item into the binning's key buffer (free after the binning), and the largest
// item into totals[3] (to be read back: above DET_MAXN the pass must be split).
hipError_t sc_launch_det_order(sc_plan *p, int nitems) {
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_det_order, dim3((unsigned)nitems), dim3(256), 0, p->stream, p->bw.items, p->bw.totals,
                       (const AdjRec *)p->bw.sorted.rec, p->bw.key, p->bw.totals + 3);
    return hipGetLastError();
}
int sc_det_max_items() { return DET_MAXN; }

// Deterministic mode, after the scatter of a pass has written its patch gradients (the
// reduction's tile count must match the scatter's: the same (ncomp + 15) / 16 rounding).
hipError_t sc_launch_scatter_reduce(sc_plan *p, void *gmaps) {
    const int ct = (p->ncomp + 15) / 16;
    if (ct <= 1) return launch_reduce<1>(p, gmaps);
    if (ct <= 2) return launch_reduce<2>(p, gmaps);
    if (ct <= 3) return launch_reduce<3>(p, gmaps);
    if (ct <= 5) return launch_reduce<5>(p, gmaps);
    if (ct <= 9) return launch_reduce<9>(p, gmaps);
    if (ct <= 13) return launch_reduce<13>(p, gmaps);
    return launch_reduce<16>(p, gmaps);
}

// FP64 plans: the binned scatter of one pass (after sc_launch_binning in adjoint form without y).
bool sc_scatter64_supported(const sc_plan *p) {
    return p->prec == SC_FP64 && p->W >= 4 && p->W <= 16 && (p->W & 1) == 0 && p->ncomp <= 256 && !p->gather_direct;
}
// Whether binning a pass of n samples pays.  Sample by sample the scatter is bound by its
// atomics, one request per tap and 64-byte sector of a pixel's components at 45 ps (W = 14, 2e4
// to 4e5 samples: 8.8 ns a sample up to kmax 3, 17 up to 7, 26 at 8, 53 at 20; W = 8: 3.3).  The
// binning costs a launch of 12 us up to BIN_SMALL samples, from there six or seven kernels and
// 10.5 ps per anchor (34 us at lmax 64, 56 at 512, 132 at 1024), and only samples that share
// anchors give it back: spread evenly, the same atomics remain, save that the columns of a row of
// one- or two-component pixels share sectors (k_scatter_short64).  So it runs where it is at most
// half of the per-sample form's time, or 1 / 1.2 of it with such pixels.  Near the line (samples
// evenly spread | a scan; sample by sample, binned, us): lmax 64, kmax 4, 5000: 113, 118 | 145, 74;
// kmax 0, 2500: 41, 38 | 69, 41; 5000: 73, 67 | 125, 60; lmax 512, 10,000, kmax 0: 120, 128 | 182,
// 114, kmax 2: 130, 185 | 165, 138; lmax 1024, 20,000, kmax 0: 251, 313 | 319, 230.
bool sc_scatter64_pays(const sc_plan *p, int64_t n) {
    const BinGeom g = sc_bin_geom(p);
    const double direct = 45e-6 * (double)n * p->W * p->W * ((p->ncomp + 7) / 8);
    const double bin = n <= BIN_SMALL ? 12.0 : 34.0 + 10.5e-6 * (double)g.nkr * (double)g.nkc;
    return direct > (p->ncomp <= 2 ? 1.2 : 2.0) * bin;
}
hipError_t sc_launch_scatter64(sc_plan *p, const double *y, double *gmaps) {
    switch (p->W) {
        case 4: return launch_scatter_mfma64<4>(p, y, gmaps);
        case 6: return launch_scatter_mfma64<6>(p, y, gmaps);
        case 8: return launch_scatter_mfma64<8>(p, y, gmaps);
        case 10: return launch_scatter_mfma64<10>(p, y, gmaps);
        case 12: return launch_scatter_mfma64<12>(p, y, gmaps);
        case 14: return launch_scatter_mfma64<14>(p, y, gmaps);
        case 16: return launch_scatter_mfma64<16>(p, y, gmaps);
        default: return hipErrorInvalidValue;
    }
}

// Scatter of one pass (binned: binning with the pass's TOD gradient already done).
hipError_t sc_launch_scatter_binned(sc_plan *p, void *gmaps) { return launch_scatter_mfma_any(p, gmaps); }

hipError_t sc_launch_scatter(sc_plan *p, const double *ptg, int64_t n, const void *y, void *gmaps) {
    const double two_pi = 6.283185307179586477;
    const double inv_hth = (double)p->n2os / two_pi, inv_hph = (double)p->nphi / two_pi;
    int64_t nblk = (n + 3) / 4;
    if (nblk > 65536) nblk = 65536;
    if (p->prec == SC_FP64)
        hipLaunchKernelGGL(k_scatter_direct<double>, dim3((unsigned)nblk), dim3(256), 0, p->stream, ptg, n,
                           (const double *)y, (double *)gmaps, p->cols, p->ncp, p->ncomp, p->W, p->beta, inv_hth,
                           inv_hph, p->n2os, p->nphi);
    else
        hipLaunchKernelGGL(k_scatter_direct<float>, dim3((unsigned)nblk), dim3(256), 0, p->stream, ptg, n,
                           (const float *)y, (float *)gmaps, p->cols, p->ncp, p->ncomp, p->W, p->beta, inv_hth,
                           inv_hph, p->n2os, p->nphi);
    return hipGetLastError();
}
