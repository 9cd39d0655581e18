// k_gather64.hip -- FP64 interpolation + k-sum on the matrix cores (FP64 plans).
//
// The convolution at a pointing is (Galloway et al. 2022, Sec. 2.1, Eq. 8 with the
// finite-resolution maps and interpolation that follow the two-step algorithm)
//     c = sum_c basis_c(psi) X[c],   X[c] = sum_{i,j < W} w_theta(i) w_phi(j) M_c[r0 + i][q0 + j],
// basis_{2k} = cos k psi, basis_{2k+1} = sin k psi.  For the samples of one
// interpolation anchor (a work item of the binning, k_bin.hip) the inner sums are a
// matrix product over the W^2 taps:
//     X[c][s] = sum_t P[t][c] w_s(t),   w_s(t) = w_theta_s(i) w_phi_s(j),
// which runs here as v_mfma_f64_16x16x4_f64 (FP64 products and accumulation), so the
// result keeps the FP64 form's accuracy (1e-12 at W = 14).
//
// One wave per work item, no workgroup barriers.  The items hold at most 64 samples
// (four 16-sample tiles; one or two when 32 or fewer are left), and the map values go
// from L2 straight into the A operand: one 8-byte load per lane (four columns x 16
// components) feeds a matrix instruction per sample tile.  Each tile holds the matrix
// pipe for 64 cycles, so four tiles leave the caches 256 cycles per 512-byte operand
// (two tiles measured 1.15, one 2.0 ms where four take 0.91 ms).  The weights and phases
// of the item's samples are in the wave's LDS.  Staging the block in LDS for 256-sample
// passes instead held a CU to one workgroup (118 KB at W = 14), whose four waves waited
// on each other, and computed 256 samples whatever the item held.  At W = 14: lmax 384,
// kmax 45, 1e6 scan samples (about 125 per anchor) 1.55 -> 0.91 ms, 42 TFLOP/s of useful
// products (63% of what a large FP64 matrix product reaches); lmax 64, kmax 4, 1e5
// uniform samples (3 per anchor) 3.17 -> 0.16 ms.
//
// Operand layout of the 16x16x4 FP64 instruction (checked on the device): A[i][k] in
// lane i + 16 k, B[k][j] in lane j + 16 k, D[i][j] in lane j + 16 (i % 4), element
// i / 4.  A is the map block (16 components x 4 taps, row i holding component
// 4 (i % 4) + i / 4 of the tile), B the tap weights (4 taps x 16 samples), so lane
// (r = lane % 16, grp = lane / 16) ends with components 16 ct + 4 grp + v (v < 4) of
// sample r: the cos/sin pairs of orders k0 = 8 ct + 2 grp and k0 + 1.  Its part of
// the k-sum is Re[e^{2 i grp psi} sum_ct (A_ct + B_ct e^{i psi}) e^{8 i ct psi}] with
// A_ct = X[c0] - i X[c0 + 1], B_ct = X[c0 + 2] - i X[c0 + 3] (c0 = 16 ct + 4 grp),
// evaluated by Horner's rule in e^{8 i psi} from the highest tile down; the four
// lanes of a sample then add their parts.
//
// The four taps of a step are four columns of one row when W is a multiple of 4.
// For W = 6, 10 and 14 the steps cover pairs of rows (2 W taps, a multiple of 4): in
// the middle step the lanes of groups 2 and 3 read the first two columns of the
// second row.  Either way no step holds a padded tap.
#include "sc_common.h"

typedef double doublex4 __attribute__((ext_vector_type(4)));

namespace {

// exp(beta (sqrt(1 - z^2) - 1)) without the cancellation next to z = 0
__device__ __forceinline__ double es_weight64(double z, double beta) {
    const double z2 = z * z, q = 1.0 - z2;
    return q > 0.0 ? exp(-beta * z2 / (1.0 + sqrt(q))) : 0.0;
}

// Orders one wave's LDS writes before its other lanes' reads (and those before later writes).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int W>
struct G64 {
    static constexpr int RP = (W & 3) ? 2 : 1;   // rows per group of steps
    static constexpr int NG = W / RP;            // groups
    static constexpr int NS = W * RP / 4;        // steps per group
    static constexpr int TS = 4;                 // sample tiles of a full item
    static constexpr int WR = 16 * TS + 1;       // row stride of the weights in LDS
    static constexpr int NWV = 4;                // waves per workgroup (independent)
    static constexpr int CTC = 2;                // component tiles per sweep over the taps
};

// One wave's LDS: tap weights (theta nodes, then phi nodes) and phases of its samples.
template <int W>
struct Wave64 {
    double w[2 * W * G64<W>::WR];
    double2 e1[16 * G64<W>::TS], e8[16 * G64<W>::TS];  // e^{i psi}, e^{8 i psi}
};

// One sweep: component tiles ct0 .. ct0 + N - 1 of every sample tile, then their Horner
// steps.  The next group's map values are loaded during the current group's products.
template <int W, int T, int N>
__device__ __forceinline__ void sweep(const char *__restrict__ blk, size_t rowb, const unsigned (&off)[G64<W>::NS],
                                      int ct0, int nct, int ncomp, unsigned dlast, const Wave64<W> &sh, int r, int grp,
                                      double2 (&qh)[T]) {
    using G = G64<W>;
    const unsigned dl = ct0 + N == nct ? dlast : 0u;
    blk += (size_t)ct0 * 1024;
    // wave-uniform base plus a 32-bit lane offset; only the sweep's top tile can be the last one
    auto load = [&](const char *base, int s, int c) {
        const unsigned o = c == N - 1 ? off[s] + dl : off[s];
        return *(const double *)(base + c * 1024 + o);
    };
    doublex4 acc[T][N];
#pragma unroll
    for (int h = 0; h < T; ++h)
#pragma unroll
        for (int c = 0; c < N; ++c) acc[h][c] = doublex4{0.0, 0.0, 0.0, 0.0};
    const double *Wth = sh.w + r;                     // theta node i at row i
    const double *Wph = sh.w + (W + grp) * G::WR + r; // phi node 4 s + grp at row 4 s
    double a[G::NS][N];
#pragma unroll
    for (int s = 0; s < G::NS; ++s)
#pragma unroll
        for (int c = 0; c < N; ++c) a[s][c] = load(blk, s, c);
#pragma unroll 1
    for (int g = 0; g < G::NG; ++g) {
        const char *nb = blk + (size_t)(g + 1 < G::NG ? g + 1 : g) * G::RP * rowb;  // last group: a harmless re-read
        double w0[T], w1[T], wf[T];
#pragma unroll
        for (int h = 0; h < T; ++h) {
            w0[h] = Wth[(G::RP * g) * G::WR + 16 * h];
            w1[h] = G::RP == 2 ? Wth[(2 * g + 1) * G::WR + 16 * h] : 0.0;
            wf[h] = Wph[16 * h];
        }
#pragma unroll
        for (int s = 0; s < G::NS; ++s) {
            double b[T];
#pragma unroll
            for (int h = 0; h < T; ++h) {
                double wt = w0[h];
                if (G::RP == 2 && s == G::NS / 2) wt = grp < 2 ? w0[h] : w1[h];
                if (G::RP == 2 && s > G::NS / 2) wt = w1[h];
                b[h] = wt * wf[h];
            }
            if (s + 1 < G::NS) {
                // the next step's phi weights: column 4 (s + 1) + grp, less W in the second row of a pair
                const int s1 = s + 1;
                const bool second = G::RP == 2 && (s1 > G::NS / 2 || (s1 == G::NS / 2 && grp >= 2));
                const double *wp = Wph + (second ? 4 * s1 - W : 4 * s1) * G::WR;
#pragma unroll
                for (int h = 0; h < T; ++h) wf[h] = wp[16 * h];
            }
#pragma unroll
            for (int c = 0; c < N; ++c) {
#pragma unroll
                for (int h = 0; h < T; ++h)
                    acc[h][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][c], b[h], acc[h][c], 0, 0, 0);
                a[s][c] = load(nb, s, c);
            }
            // keep the steps apart: hoisting a group's LDS reads and loads would spill
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int h = 0; h < T; ++h) {
        const double2 e1 = sh.e1[16 * h + r], e8 = sh.e8[16 * h + r];
        double2 q = qh[h];
#pragma unroll
        for (int c = N - 1; c >= 0; --c) {
            doublex4 x = acc[h][c];
            if (c == N - 1) {  // components past ncomp (the last tile only)
                const int c0 = 16 * (ct0 + c) + 4 * grp;
                if (c0 >= ncomp) x[0] = x[1] = 0.0;
                if (c0 + 2 >= ncomp) x[2] = x[3] = 0.0;
            }
            // C = A + B e1 with A = x0 - i x1, B = x2 - i x3; q = q e8 + C
            const double cx = fma(x[2], e1.x, fma(x[3], e1.y, x[0]));
            const double cy = fma(x[2], e1.y, fma(-x[3], e1.x, -x[1]));
            const double qx = fma(q.x, e8.x, fma(-q.y, e8.y, cx));
            const double qy = fma(q.x, e8.y, fma(q.y, e8.x, cy));
            q = make_double2(qx, qy);
        }
        qh[h] = q;
    }
}

// The samples pos0 .. pos0 + ns - 1 (ns <= 16 T) of one anchor.
template <int W, int T>
__device__ __forceinline__ void samples64(const BinRec *__restrict__ rec, int pos0, int ns,
                                          const char *__restrict__ blk, size_t rowb, const unsigned (&off)[G64<W>::NS],
                                          int nct, int ncomp, unsigned dlast, Wave64<W> &sh, int lane, double beta,
                                          double *__restrict__ tod) {
    using G = G64<W>;
    constexpr int HALF = W / 2;
    const int r = lane & 15, grp = lane >> 4;
    // Weight of node e / 2^lp for sample e % 2^lp (theta nodes, then phi nodes), 2^lp >= ns.
    // Columns past ns are left as they are: they reach only the unused outputs of their own
    // sample slot.
    const int lp = ns > 1 ? 32 - __builtin_clz((unsigned)(ns - 1)) : 0;
#pragma unroll 1
    for (int e = lane; e < (2 * W) << lp; e += 64) {
        const int node = e >> lp, sl = e & ((1 << lp) - 1);
        if (sl < ns) {
            const bool th = node < W;
            const double f = th ? rec[pos0 + sl].fu : rec[pos0 + sl].fv;
            sh.w[node * G::WR + sl] =
                es_weight64((f + (double)(HALF - 1 - (th ? node : node - W))) / (double)HALF, beta);
        }
    }
    int idx = -1;
    if (lane < ns) {
        idx = rec[pos0 + lane].idx;
        double sn, cs;
        sincos(rec[pos0 + lane].psi, &sn, &cs);
        const double2 e1 = make_double2(cs, sn);
        const double2 e2 = cmul(e1, e1), e4 = cmul(e2, e2);
        sh.e1[lane] = e1;
        sh.e8[lane] = cmul(e4, e4);
    }
    wave_lds_sync();
    double2 q[T];
#pragma unroll
    for (int h = 0; h < T; ++h) q[h] = make_double2(0.0, 0.0);
    // tiles from the highest down: the remainder first, then CTC at a time
    int ct = nct;
    if (nct % G::CTC) {
        static_assert(G::CTC == 2, "the remainder is one tile");
        ct -= 1;
        sweep<W, T, 1>(blk, rowb, off, ct, nct, ncomp, dlast, sh, r, grp, q);
    }
    while (ct > 0) {
        ct -= G::CTC;
        sweep<W, T, G::CTC>(blk, rowb, off, ct, nct, ncomp, dlast, sh, r, grp, q);
    }
    // part = Re[e^{2 i grp psi} q], summed over the sample's four lane groups
#pragma unroll
    for (int h = 0; h < T; ++h) {
        const double2 e1 = sh.e1[16 * h + r];
        const double2 e2 = cmul(e1, e1), e4 = cmul(e2, e2);
        const double2 z0 = grp == 0 ? make_double2(1.0, 0.0) : grp == 1 ? e2 : grp == 2 ? e4 : cmul(e4, e2);
        double part = z0.x * q[h].x - z0.y * q[h].y;
        part += __shfl_xor(part, 16);
        part += __shfl_xor(part, 32);
        const int ix = __shfl(idx, 16 * h + r);
        if (grp == 0 && ix >= 0) tod[ix] = part;
    }
    wave_lds_sync();  // the weights and phases are rewritten by the next samples
}

template <int W>
__global__ void __launch_bounds__(64 * G64<W>::NWV) __attribute__((amdgpu_waves_per_eu(2)))
k_gather_mfma64(const int4 *__restrict__ items, const int *__restrict__ totals, BinSorted srt,
                const double *__restrict__ maps, double *__restrict__ tod, int cols, int ncp, int ncomp, int nkc,
                double beta) {
    using G = G64<W>;
    __shared__ Wave64<W> wsh[G::NWV];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, grp = lane >> 4;
    const int nitems = totals[1];
    const int nct = (ncomp + 15) >> 4;
    const size_t rowb = (size_t)sc_map_ntile(cols) * (size_t)(ncp >> 1) * 128;  // bytes of one map row
    const int tileb = (ncp >> 1) * 128;                                         // bytes of one column tile
    // the lane's component within a tile; past ncomp in the last tile it reads the tile's
    // first component instead (left out of the k-sum)
    const int comp = 4 * (r & 3) + (r >> 2);
    const int compb = (comp >> 1) * 128 + (comp & 1) * 8;
    const unsigned dlast = 16 * (nct - 1) + comp < ncomp ? 0u : 0u - (unsigned)compb;
    // Items in a fixed stride over the waves (a shared queue counter would serialise the
    // short ones); at any time one XCD works on a run of consecutive anchors, whose blocks
    // overlap in its L2.
    const int nw = gridDim.x * G::NWV;
    for (int it = xcd_remap(blockIdx.x, gridDim.x) * G::NWV + wv; it < nitems; it += nw) {
        const int4 item = items[it];
        const int row0 = item.x / nkc, col0 = item.x - (item.x / nkc) * nkc;
        const char *blk = (const char *)maps + (size_t)row0 * rowb;
        unsigned off[G::NS];
#pragma unroll
        for (int s = 0; s < G::NS; ++s) {
            const int t = 4 * s + grp, j = t < W ? t : t - W;
            const int c = col0 + j;
            off[s] = (c >> 3) * tileb + (c & 7) * 16 + compb + (t < W ? 0u : (unsigned)rowb);
        }
        for (int ch = 0; ch < item.z; ch += 16 * G::TS) {
            const int left = item.z - ch;
            if (left > 32)
                samples64<W, 4>(srt.rec, item.y + ch, left < 64 ? left : 64, blk, rowb, off, nct, ncomp, dlast, wsh[wv],
                                lane, beta, tod);
            else if (left > 16)
                samples64<W, 2>(srt.rec, item.y + ch, left, blk, rowb, off, nct, ncomp, dlast, wsh[wv], lane, beta, tod);
            else
                samples64<W, 1>(srt.rec, item.y + ch, left, blk, rowb, off, nct, ncomp, dlast, wsh[wv], lane, beta, tod);
        }
    }
}

template <int W>
hipError_t launch64(sc_plan *p, void *tod) {
    using G = G64<W>;
    auto kern = k_gather_mfma64<W>;
    const int grid = sc_persistent_grid((const void *)kern, 64 * G::NWV, 0, p->gather_wgs_per_cu);
    const BinGeom g = sc_bin_geom(p);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * G::NWV), 0, p->stream, p->bw.items, p->bw.totals, p->bw.sorted,
                       (const double *)p->maps, (double *)tod, p->cols, p->ncp, p->ncomp, g.nkc, p->beta);
    return hipGetLastError();
}

}  // namespace

// Kernel widths with an instantiation (every even width the plans accept).
bool sc_gather_mfma64_supported(int W) { return W >= 4 && W <= 16 && (W & 1) == 0; }

hipError_t sc_launch_gather_mfma64(sc_plan *p, void *tod) {
    switch (p->W) {
        case 4: return launch64<4>(p, tod);
        case 6: return launch64<6>(p, tod);
        case 8: return launch64<8>(p, tod);
        case 10: return launch64<10>(p, tod);
        case 12: return launch64<12>(p, tod);
        case 14: return launch64<14>(p, tod);
        case 16: return launch64<16>(p, tod);
        default: return hipErrorInvalidValue;
    }
}
