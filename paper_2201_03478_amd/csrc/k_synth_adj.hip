// k_synth_adj.hip -- adjoint of the ring sums (gradient w.r.t. the sky a_lm).
//
// The forward ring sums are (k_synth.hip)
//     F_k(theta_j, m)      = sum_l a_lm conj(b_lk) d^l_mk(theta_j)
//     F_k(pi - theta_j, -m) = sum_l (-1)^{l+k+m} conj(a_lm) conj(b_lk) d^l_mk(theta_j),
// the inner sums of Eqs. 7/9 of Galloway et al. (2022, Sec. 2.1).  Given the
// ring-sum gradients F_adj (from the adjoint transforms), with the real inner
// product Re sum conj(u) v, the gradient g = dL/dRe a_lm + i dL/dIm a_lm is
//     Q+(l) = sum_j d^l_mk(theta_j) F_adj_k(theta_j, m),
//     Q-(l) = sum_j d^l_mk(theta_j) F_adj_k(pi - theta_j, -m),
//     g_lm  = sum_k [ Q+ b_lk + (-1)^{l+k+m} conj(Q- b_lk) ]      (m > 0),
//     g_l0  = sum_k Re(Q+ b_lk)                                  (m = 0).
// The d values come from the same recursions and start values as the forward
// kernel, on northern rings only: lanes 0-31 run the column (m, k) (R+) for the
// rings theta_j <= pi/2, lanes 32-63 the column (-m, k) (R-) on the same rings,
// which by d^l_mk(pi - theta) = (-1)^{l+k} d^l_{-m,k}(theta) gives the southern
// rings.  R- runs on (-1)^l d^l_{-m,k}, whose recursion has the coefficient
// -((alpha + beta) - alpha y) and the same gamma, so that its products with the
// ring-sum gradients (times (-1)^k, folded into them at load) add to the same
// per-l sums as R+'s:
//     Q+(l) = sum_{j north} [d^l_mk(theta_j) F_adj(theta_j, m) + (-1)^k dt F_adj(pi - theta_j, m)],
//     Q-(l) = sum_{j north} [d^l_mk(theta_j) F_adj(pi - theta_j, -m) + (-1)^k dt F_adj(theta_j, -m)],
// dt = (-1)^l d^l_{-m,k}(theta_j).  The recursion is the forward kernel's, on
// u^l = d^l / S_l with the plan's coefficient table, and S_l multiplies the finished sums.
//
// The sums over rings are reductions across lanes for every l.  A lane holds up to nine
// northern rings and adds their products, 4 real partials per l, in registers; the 64 lanes
// then halve the partials of 16 consecutive l against each other (at every level a lane
// keeps one of two values and adds its partner's copy of it), so that after 63 exchanges
// each lane holds one finished (l, value) sum.  The exchanges over 32 and 16 lanes are
// single swap instructions, those inside a row are DPP moves: about 16 instructions per l
// and wave beside 6 FMAs per ring, no LDS round trip.  With all of the 270 northern rings of
// lmax 512 in one wave, lmax 512, kmax 32 takes 0.84 ms, 33 TFLOP/s (2.21 ms when the
// partials of every l went through a padded LDS buffer, 8 l at a time, three rings per lane).
// Waves of a workgroup are the ring groups of one (k, m) and are combined in LDS.
// Per-k contributions go to GA[k][alm index]; a second kernel sums over k in a
// fixed order (deterministic).  Columns with more than 2048 rings are split into
// slabs of rings, one workgroup each, whose partial sums go to separate copies of
// GA and are added by the same fixed-order reduction (no atomics).
//
// The same Q+- give the gradient with respect to the beam (BEAM = true): the
// TOD is bilinear, and with the sky gradient above L = Re sum conj(g_lm) a_lm
// is, as a function of b,
//     L = Re sum_{l,k,m>0} [conj(b_lk) conj(Q+) a_lm + b_lk (-1)^{l+k+m} Q- a_lm]
//       + Re sum_{l,k} b_lk Q+(m = 0) a_l0,
// so h_lk = dL/dRe b_lk + i dL/dIm b_lk = sum_m [conj(Q+) a_lm +
// (-1)^{l+k+m} conj(Q- a_lm)] (the Q- term for m > 0), real for k = 0.  Per-m
// contributions go to GB[m][blm index] and are summed over m in a fixed order.
#include "wigner_rec.h"

namespace {

using namespace wrec;

constexpr int ADJ_MAXR = 9;  // rings per lane
constexpr int ADJ_MAXW = 4;  // waves per workgroup: at most 1024 northern rings
constexpr int ADJ_GRP = 16;  // l steps per reduction

__device__ __forceinline__ double dbl(int lo, int hi) { return __hiloint2double(hi, lo); }

// One level of the reduction over lane pairs 32 (or 16) apart: lanes of the lower half (even
// rows) get a's pair sum, the others b's.
template <bool ROWS>
__device__ __forceinline__ double fold_swap(double a, double b) {
    typedef unsigned uint2v __attribute__((ext_vector_type(2)));
    const unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
    const unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
    uint2v l, h;
    if constexpr (ROWS) {
        l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
        h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    } else {
        l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    }
    return dbl((int)l[0], (int)h[0]) + dbl((int)l[1], (int)h[1]);
}

// One level inside a row of 16 lanes: partner lane by the DPP control (an involution that
// flips the lane bit `hi` tells); lanes with hi = false get a's pair sum, the others b's.
template <int CTRL>
__device__ __forceinline__ double fold_dpp(double a, double b, bool hi) {
    const double keep = hi ? b : a, send = hi ? a : b;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(send), CTRL, 0xf, 0xf, true);
    const int up = __builtin_amdgcn_mov_dpp(__double2hiint(send), CTRL, 0xf, 0xf, true);
    return keep + dbl(lo, up);
}
constexpr int DPP_ROR8 = 0x128;      // lane ^ 8
constexpr int DPP_HALF_MIRROR = 0x141;  // lane ^ 7
constexpr int DPP_XOR2 = 0x4e;       // quad_perm 2, 3, 0, 1
constexpr int DPP_XOR1 = 0xb1;       // quad_perm 1, 0, 3, 2

// The 4 partials of one l to one value per lane: rows 0 .. 3 hold values 0, 2, 1, 3.
__device__ __forceinline__ double fold_values(const double (&p)[4]) {
    return fold_swap<true>(fold_swap<false>(p[0], p[1]), fold_swap<false>(p[2], p[3]));
}

// Rings of one lane.
template <int RPT>
struct AdjRings {
    double x[RPT], u[RPT], up[RPT];
    double2 fa[RPT], fm[RPT];
    int e[RPT];
};

// One l: partial sums of the lane's rings (scaled rings, e != 0, are below 2^-600 and add
// nothing) and the recursion step.
template <int RPT, bool MASK>
__device__ __forceinline__ void adj_step(double a, double b, AdjRings<RPT> &R, double (&p)[4]) {
    p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const double v = MASK && R.e[r] != 0 ? 0.0 : R.u[r];
        p[0] = fma(v, R.fa[r].x, p[0]);
        p[1] = fma(v, R.fa[r].y, p[1]);
        p[2] = fma(v, R.fm[r].x, p[2]);
        p[3] = fma(v, R.fm[r].y, p[3]);
        const double un = fma(fma(a, R.x[r], b), R.u[r], -R.up[r]);
        R.up[r] = R.u[r];
        R.u[r] = un;
    }
}

// ADJ_GRP steps; returns the lane's finished sum: value (row 0 .. 3: 0, 2, 1, 3) of step
// b3 + 2 b2 + 4 b1 + 8 b0 for lane bits b3 .. b0.
template <int RPT, bool MASK>
__device__ __forceinline__ double adj_group(const double *cA, const double *cB, AdjRings<RPT> &R, int lane) {
    double q3 = 0.0, q2 = 0.0, q1 = 0.0, q0 = 0.0;  // first halves waiting at each level
    double res = 0.0;
#pragma unroll
    for (int t = 0; t < ADJ_GRP; ++t) {
        double p[4];
        adj_step<RPT, MASK>(cA[t], cB[t], R, p);
        double v = fold_values(p);
        if ((t & 1) == 0) {
            q3 = v;
        } else {
            v = fold_dpp<DPP_ROR8>(q3, v, lane & 8);
            if ((t & 2) == 0) {
                q2 = v;
            } else {
                v = fold_dpp<DPP_HALF_MIRROR>(q2, v, lane & 4);
                if ((t & 4) == 0) {
                    q1 = v;
                } else {
                    v = fold_dpp<DPP_XOR2>(q1, v, lane & 2);
                    if ((t & 8) == 0)
                        q0 = v;
                    else
                        res = fold_dpp<DPP_XOR1>(q0, v, lane & 1);
                }
            }
        }
        if (t & 1) __builtin_amdgcn_sched_barrier(0);  // keep the coefficient reads near their steps
    }
    return res;
}

template <int RPT, bool BEAM>
__global__ void __launch_bounds__(64 * ADJ_MAXW) __attribute__((amdgpu_waves_per_eu(2)))
k_ring_sums_adjoint(const double2 *__restrict__ FA, const double2 *__restrict__ coefs, double2 *__restrict__ GA,
                    const double *__restrict__ sbin_m, const int *__restrict__ sbin_e,
                    const double *__restrict__ rtab, const double2 *__restrict__ rroot,
                    const double4 *__restrict__ ctab, const long long *__restrict__ ctab_off, int lmax, int kmax,
                    int nring, int alm_lmax, int nslab, int per) {
    // coefs: the beam b_lk (sky gradient into GA[k]) or, with BEAM, the sky a_lm
    // in the alm_lmax layout (beam gradient into GA[m], blm layout)
    __shared__ double cA[64], cB[2 * 64], cS[64];
    __shared__ double Qw[ADJ_MAXW][64][4];
    const int nw = blockDim.x >> 6;
    const int slab = blockIdx.x % nslab;  // rings [slab per, slab per + per)
    const int b = blockIdx.x / nslab;
    const int k = b % (kmax + 1);
    const int m = b / (kmax + 1);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tp = lane >> 5, sub = lane & 31;  // recursion R+ (0) or R- (1); northern ring slot
    const int nh = (nring + 1) / 2;
    const int l0 = m > k ? m : k;
    const int mn = m < k ? m : k;
    const int nm = 2 * lmax + 1;
    const size_t aoff = (size_t)m * (2 * lmax + 1 - m) / 2;
    const size_t nalm = (size_t)(lmax + 1) * (lmax + 2) / 2;
    const size_t boff = (size_t)k * (2 * lmax + 1 - k) / 2;
    const size_t nblm = (size_t)(kmax + 1) * (2 * lmax + 2 - kmax) / 2;
    // output column: (l, m) of GA[k] for the sky gradient, (l, k) of GA[m] for the beam
    double2 *gk = BEAM ? GA + ((size_t)slab * (lmax + 1) + m) * nblm + boff
                       : GA + ((size_t)slab * (kmax + 1) + k) * nalm + aoff;
    // orders below l0 have no d^l_mk: their contribution is zero
    for (int l = (BEAM ? k : m) + tid; l < l0 && l <= lmax; l += blockDim.x) gk[l] = make_double2(0.0, 0.0);
    if (l0 > lmax) return;

    AdjRings<RPT> R;
    const XN pref = {sbin_m[l0 * (kmax + 1) + mn], sbin_e[l0 * (kmax + 1) + mn]};
    const double pfe = (double)pref.e, pfm = log2(pref.m);  // log2 of the start prefactor
    const double sk = (k & 1) ? -1.0 : 1.0;
    bool scaled = false;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int jl = (w * RPT + r) * 32 + sub;  // northern ring within the slab
        const int j = slab * per + jl, js = nring - 1 - j;
        R.up[r] = 0.0;
        R.fa[r] = make_double2(0.0, 0.0);
        R.fm[r] = make_double2(0.0, 0.0);
        R.x[r] = 0.0;
        R.u[r] = 0.0;
        R.e[r] = 0;
        if (jl < per && j < nh && (tp == 0 || js != j)) {  // R- skips the equator ring of an odd count
            start_value(rtab + 5 * j, m, k, pfe, pfm, R.x[r], R.u[r], R.e[r], tp == 1);
            if (tp == 0) {
                R.x[r] = -R.x[r];  // y' = -y (k_synth.hip)
                R.fa[r] = FA[((size_t)k * nm + (m + lmax)) * nring + j];
                if (m > 0) R.fm[r] = FA[((size_t)k * nm + (lmax - m)) * nring + js];
            } else {
                if (l0 & 1) R.u[r] = -R.u[r];  // (-1)^l u^l_{-m,k} at l = l0
                R.fa[r] = cscale(FA[((size_t)k * nm + (m + lmax)) * nring + js], sk);
                if (m > 0) R.fm[r] = cscale(FA[((size_t)k * nm + (lmax - m)) * nring + j], sk);
            }
        }
        scaled |= R.e[r] != 0;
    }
    bool fast = !__any(scaled);

    const double4 *ccol = ctab ? ctab + ctab_off[m * (kmax + 1) + k] : nullptr;
    double s_prev = 1.0, s_cur = 1.0;
    // the finished sum a lane holds after each group: value tv of step tl
    const int tv = ((lane >> 5) & 1) | ((lane >> 3) & 2);
    const int tl = ((lane >> 3) & 1) | ((lane >> 1) & 2) | ((lane << 1) & 4) | ((lane << 3) & 8);
    for (int lc = l0; lc <= lmax; lc += 64) {
        __syncthreads();  // previous chunk's coefficients and Qw are consumed
        if (w == 0) {
            // (zero past lmax: those steps' sums are not used)
            const ChunkCoef c = ctab ? chunk_coefs_tab(ccol, lc, lane, l0, lmax)
                                     : chunk_coefs(lc, lane, l0, lmax, m, k, rroot, s_prev, s_cur);
            cA[lane] = c.a;
            cB[lane] = c.b;
            cB[64 + lane] = -c.bn;
            cS[lane] = c.sl;
        }
        __syncthreads();
        const int nl = (lmax - lc + 1) < 64 ? (lmax - lc + 1) : 64;
        const double *cBt = cB + 64 * tp;
        for (int t0 = 0; t0 < nl; t0 += ADJ_GRP) {
            Qw[w][t0 + tl][tv] = fast ? adj_group<RPT, false>(cA + t0, cBt + t0, R, lane)
                                      : adj_group<RPT, true>(cA + t0, cBt + t0, R, lane);
            if (fast || !(t0 & ADJ_GRP)) continue;
            // rescaling every 32 steps (k_synth.hip)
            bool low = false;
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                if (fabs(R.u[r]) > REC_BIG) {
                    R.u[r] = rec_down(R.u[r]);
                    R.up[r] = rec_down(R.up[r]);
                    R.e[r] += 1;
                }
                low |= R.e[r] != 0;
            }
            fast = !__any(low);
        }
        __syncthreads();
        if (tid < nl) {
            const int l = lc + tid;
            double q0 = 0.0, q1 = 0.0, q2 = 0.0, q3 = 0.0;
            for (int ww = 0; ww < nw; ++ww) {
                const double *qq = Qw[ww][tid];
                q0 += qq[0];
                q1 += qq[1];
                q2 += qq[2];
                q3 += qq[3];
            }
            const double sl = cS[tid];
            q0 *= sl;
            q1 *= sl;
            q2 *= sl;
            q3 *= sl;
            const double sg = ((l + k + m) & 1) ? -1.0 : 1.0;
            double2 g;
            if constexpr (BEAM) {
                double2 aa = coefs[(size_t)m * (2 * alm_lmax + 1 - m) / 2 + l];
                if (m == 0) aa.y = 0.0;
                g = cmul(make_double2(q0, -q1), aa);  // conj(Q+) a
                if (m > 0) {
                    const double2 t = cmul(make_double2(q2, q3), aa);  // Q- a
                    g.x += sg * t.x;
                    g.y -= sg * t.y;
                }
            } else {
                double2 bb = coefs[boff + l];
                if (k == 0) bb.y = 0.0;
                const double2 gp = cmul(make_double2(q0, q1), bb);
                if (m == 0) {
                    g = make_double2(gp.x, 0.0);
                } else {
                    const double2 gm = cmul(make_double2(q2, q3), bb);
                    g = make_double2(gp.x + sg * gm.x, gp.y - sg * gm.y);
                }
            }
            gk[l] = g;
        }
    }
}

// grad[i] = sum over slabs and m of GB[slab][m][i], in a fixed order, over the blm layout;
// the k = 0 column (entries i <= lmax) is real.  A workgroup takes 16 entries with 16 slices
// of the sum each: one thread per entry left a serial chain of loads (lmax 128, kmax 8, 129
// terms on five workgroups: 34 us).
__global__ void __launch_bounds__(256) k_reduce_over_m(const double2 *__restrict__ GB, double2 *__restrict__ grad,
                                                       int64_t nblm, int lmax, int nslab) {
    __shared__ double2 part[256];
    const int e = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int64_t i = (int64_t)blockIdx.x * 16 + e;
    double2 s = make_double2(0.0, 0.0);
    if (i < nblm) {
#pragma unroll 4
        for (int q = sl; q < nslab * (lmax + 1); q += 16) s = cadd(s, GB[(size_t)q * nblm + i]);
    }
    part[threadIdx.x] = s;
    __syncthreads();
    if (sl > 0 || i >= nblm) return;
    for (int q = 1; q < 16; ++q) s = cadd(s, part[16 * q + e]);
    if (i <= lmax) s.y = 0.0;
    grad[i] = s;
}

// grad[i] = sum over slabs and k of GA[slab][k][i] in that fixed order (entries with
// k > l are zero).
__global__ void k_reduce_over_k(const double2 *__restrict__ GA, double2 *__restrict__ grad, int64_t nalm,
                                int kmax, int nslab) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nalm) return;
    double2 s = make_double2(0.0, 0.0);
    for (int q = 0; q < nslab * (kmax + 1); ++q) {
        const double2 v = GA[(size_t)q * nalm + i];
        s.x += v.x;
        s.y += v.y;
    }
    grad[i] = s;
}

}  // namespace

// Ring slabs per (k, m) column, northern rings per slab, waves per workgroup and rings per
// lane: a workgroup holds at most 1024 northern rings, longer columns are split into equal
// slabs.  A wave takes up to 32 ADJ_MAXR rings (fewest waves: the reduction is per wave).
static void adj_layout(int nring, int *rpt, int *nw, int *nslab, int *per) {
    const int nh = (nring + 1) / 2;
    *nslab = (nh + 1023) / 1024;
    *per = (nh + *nslab - 1) / *nslab;
    *nw = (*per + 32 * ADJ_MAXR - 1) / (32 * ADJ_MAXR);
    *rpt = (*per + 32 * *nw - 1) / (32 * *nw);
}

int sc_adjoint_slabs(const sc_plan *p) { return ((p->nring + 1) / 2 + 1023) / 1024; }

template <int RPT>
static hipError_t launch_adj(sc_plan *p, const double *coefs, double2 *out, bool beam, int rpt, int nw, int nslab,
                             int per) {
    if constexpr (RPT < ADJ_MAXR)
        if (rpt > RPT) return launch_adj<RPT + 1>(p, coefs, out, beam, rpt, nw, nslab, per);
    const int nblk = (p->lmax + 1) * (p->kmax + 1) * nslab;
    auto kern = beam ? k_ring_sums_adjoint<RPT, true> : k_ring_sums_adjoint<RPT, false>;
    hipLaunchKernelGGL(kern, dim3(nblk), dim3(64 * nw), 0, p->stream, p->F, (const double2 *)coefs, out, p->sbin_m,
                       p->sbin_e, p->rtab, p->rroot, p->ctab, p->ctab_off, p->lmax, p->kmax, p->nring, p->alm_lmax,
                       nslab, per);
    return hipGetLastError();
}

static hipError_t ring_sums_adjoint(sc_plan *p, const double *coefs, double2 *out, bool beam) {
    int rpt, nw, nslab, per;
    adj_layout(p->nring, &rpt, &nw, &nslab, &per);
    return launch_adj<1>(p, coefs, out, beam, rpt, nw, nslab, per);
}

hipError_t sc_launch_ring_sums_adjoint(sc_plan *p, const double *blm, double *grad) {
    hipError_t e = ring_sums_adjoint(p, blm, p->GA, false);
    if (e != hipSuccess) return e;
    const int64_t nalm = (int64_t)(p->lmax + 1) * (p->lmax + 2) / 2;
    hipLaunchKernelGGL(k_reduce_over_k, dim3((unsigned)((nalm + 255) / 256)), dim3(256), 0, p->stream, p->GA,
                       (double2 *)grad, nalm, p->kmax, sc_adjoint_slabs(p));
    return hipGetLastError();
}

hipError_t sc_launch_ring_sums_adjoint_beam(sc_plan *p, const double *alm, double *grad) {
    hipError_t e = ring_sums_adjoint(p, alm, p->GB, true);
    if (e != hipSuccess) return e;
    const int64_t nblm = (int64_t)(p->kmax + 1) * (2 * p->lmax + 2 - p->kmax) / 2;
    hipLaunchKernelGGL(k_reduce_over_m, dim3((unsigned)((nblm + 15) / 16)), dim3(256), 0, p->stream, p->GB,
                       (double2 *)grad, nblm, p->lmax, sc_adjoint_slabs(p));
    return hipGetLastError();
}
