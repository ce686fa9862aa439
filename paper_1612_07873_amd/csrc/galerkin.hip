// Galerkin coarse operator Mhat = P^+ M P (Sec. 3.4 step 4), keeping the
// nearest-neighbour form of Eq. (3) at every level (the recursion of Sec. 3.4).
//
// With Pf(x) the dof x N slice of P at fine site x (nonzero only where the
// chirality of the row matches that of the column), D(x) the on-site block
// and H_d(x) the hop block of the parent towards x' = x + hop_d:
//   Y_d(xc) = sum over x in xc with x' outside xc of Pf(x)^+ H_d(x) Pf(x')
//   X(xc)   = sum over x in xc of Pf(x)^+ D(x) Pf(x)
//           + sum over hops x -> x' that stay inside xc of Pf(x)^+ H_d(x) Pf(x').
// The parent is the fine Wilson-clover operator (D = 4 + m0 + A, H_d from the
// spin projectors and links) or a coarse operator (D = X, H_d = Y_d).
//
// Work decomposition: one work-group per (coarse site, term), 17 terms: the
// eight Y_d, and X split into its eight inside-hop sums and the on-site sum
// (written to separate slots and added in a fixed order afterwards, so the
// build is deterministic and needs no atomics).  A coarse parent (and a fine one
// with more than 32 vectors) goes site by site: the work-group forms the
// parent's block H (dof x dof) in LDS, then W = H Pf(x') in LDS, then each
// thread adds Pf(x)^+ W to the N x N entries it owns.  The fine parent's form is
// k_galerkin_fine below.  All arithmetic is FP64.  This is setup work, done once
// per hierarchy.
#include "handles.h"

#include <type_traits>
#include <vector>

namespace qmg {

constexpr int GAL_MAXE = 16;  // output entries per thread

struct Proj {  // spin matrices (1 - gamma_mu) [fwd] and (1 + gamma_mu) [bwd], 4x4 complex
    double p[8][4][4][2];
};

template <typename R>
__device__ __forceinline__ cpx<double> fine_link(const cpx<R>* U, int mu, int e, int64_t x, int64_t V) {
    const cpx<R> u = U[((int64_t)mu * 9 + e) * V + x];
    return {(double)u.re, (double)u.im};
}

// H[f][g] of the fine parent for term (d or diag) at fine site x.
template <typename R>
__device__ cpx<double> fine_H(const qmg_fine_op_s& op, const cpx<R>* U, const R* clov, const Proj& P,
                              int term, int64_t x, int64_t xn, int f, int g) {
    const int s = f / 3, a = f % 3, t = g / 3, b = g % 3;
    if (term == 8) {  // 4 + m0 + A(x)
        cpx<double> v = {f == g ? 4.0 + op.m0 : 0.0, 0.0};
        if (op.csw != 0.0 && (s / 2) == (t / 2)) {
            const int chi = s / 2, i = f - 6 * chi, j = g - 6 * chi;
            const R* A = clov + (int64_t)chi * 36 * op.V + x;
            if (i == j) v.re += (double)A[i * op.V];
            else {
                const int r = i < j ? i : j, c = i < j ? j : i;
                const int k = r * 6 - r * (r + 1) / 2 + (c - r - 1);
                const double re = (double)A[(6 + 2 * k) * op.V], im = (double)A[(7 + 2 * k) * op.V];
                v.re += re;
                v.im += i < j ? im : -im;
            }
        }
        return v;
    }
    const int mu = term / 2;
    const double pr = P.p[term][s][t][0], pi = P.p[term][s][t][1];
    if (pr == 0.0 && pi == 0.0) return {0.0, 0.0};
    cpx<double> u;
    if ((term & 1) == 0) u = fine_link(U, mu, a * 3 + b, x, op.V);  // U_mu(x)
    else {                                                        // U_mu(x - mu)^+
        const cpx<double> w = fine_link(U, mu, b * 3 + a, xn, op.V);
        u = {w.re, -w.im};
    }
    return {-0.5 * (pr * u.re - pi * u.im), -0.5 * (pr * u.im + pi * u.re)};
}

template <typename R>
__device__ __forceinline__ cpx<double> coarse_H(const qmg_coarse_op_s& op, const R* L, int term, int64_t x,
                                                int f, int g) {
    // element (row f, col g) of X (term 8) or Y_term in the chunked layout
    constexpr int cpc = sizeof(R) == 8 ? 1 : 2;
    const int blk = term == 8 ? 0 : term + 1;
    const int e = blk * op.N + g;
    const int j = e / cpc, q = e % cpc;
    const R* c = L + (((int64_t)x * op.J + j) * op.N + f) * 2 * cpc;
    return {(double)c[2 * q], (double)c[2 * q + 1]};
}

template <bool FINE, typename R, bool ST>
__global__ __launch_bounds__(1024) void k_galerkin(double2* __restrict__ Yout, double2* __restrict__ Xpart,
                                                   qmg_fine_op_s fop, qmg_coarse_op_s cop,
                                                   const void* __restrict__ parent_a,
                                                   const void* __restrict__ parent_b,
                                                   const int* __restrict__ nbr, const double2* __restrict__ B,
                                                   const int* __restrict__ members, const int* __restrict__ owner,
                                                   int64_t Vc, int dof, int nvec, int bsites, Proj P) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = 2 * nvec, half = dof / 2;
    cpx<double>* W = reinterpret_cast<cpx<double>*>(smem);  // [dof][N]
    // ST: the parent's block and the two basis blocks are staged in LDS
    cpx<double>* H = W + dof * N;                           // [dof][dof]
    cpx<double>* Px = H + dof * dof;                        // Pf(x) [dof][nvec]
    cpx<double>* Pn = Px + dof * nvec;                      // Pf(x') [dof][nvec]
    const int64_t xc = blockIdx.x / 17;
    const int term = (int)(blockIdx.x % 17);
    const bool isY = term < 8;
    const int hterm = isY ? term : term - 8;  // 0..7 hops, 8 = on-site
    const int T = blockDim.x;
    cpx<double> acc[GAL_MAXE];
#pragma unroll
    for (int i = 0; i < GAL_MAXE; ++i) acc[i] = {0.0, 0.0};

    for (int b = 0; b < bsites; ++b) {
        const int64_t x = members[xc * bsites + b];
        int64_t xn = x;
        if (hterm < 8) {
            xn = nbr[x * 8 + hterm];
            const bool inside = owner[xn] == xc;
            if (isY == inside) continue;  // Y wants hops leaving the aggregate, X the ones inside
        }
        // the parent's block H[f][g] for this (x, term), once (when it fits
        // in LDS; otherwise each element is formed where it is used)
        auto Hfg = [&](int f, int g) {
            return FINE ? fine_H<R>(fop, (const cpx<R>*)parent_a, (const R*)parent_b, P, hterm, x, xn, f, g)
                        : coarse_H<R>(cop, (const R*)parent_a, hterm, x, f, g);
        };
        __syncthreads();
        if constexpr (ST) {
            for (int e = threadIdx.x; e < dof * dof; e += T) H[e] = Hfg(e / dof, e % dof);
            for (int e = threadIdx.x; e < dof * nvec; e += T) {   // coalesced loads of both basis blocks
                const double2 a = B[x * dof * nvec + e], c = B[xn * dof * nvec + e];
                Px[e] = cpx<double>{a.x, a.y};
                Pn[e] = cpx<double>{c.x, c.y};
            }
            __syncthreads();
        }
        // W[f][m] = sum_{g in chi(m)} H[f][g] Pf(xn)[g][m'] ; Pf(xn)[g][m'] = B[xn][g][m']
        for (int e = threadIdx.x; e < dof * N; e += T) {
            const int f = e / N, m = e % N;
            const int chi = m / nvec, mp = m - chi * nvec;
            cpx<double> w = {0.0, 0.0};
            for (int gg = 0; gg < half; ++gg) {
                const int g = chi * half + gg;
                cpx<double> h, bv;
                if constexpr (ST) {
                    h = H[f * dof + g];
                    bv = Pn[g * nvec + mp];
                } else {
                    h = Hfg(f, g);
                    const double2 b2 = B[(xn * dof + g) * nvec + mp];
                    bv = cpx<double>{b2.x, b2.y};
                }
                cmac(w.re, w.im, h.re, h.im, bv.re, bv.im);
            }
            W[e] = w;
        }
        __syncthreads();
        // acc[n][m] += sum_{f in chi(n)} conj(Pf(x)[f][n']) W[f][m]
#pragma unroll
        for (int i = 0; i < GAL_MAXE; ++i) {
            const int e = threadIdx.x + i * T;
            if (e >= N * N) break;
            const int n = e / N, m = e % N;
            const int chi = n / nvec, np = n - chi * nvec;
            for (int ff = 0; ff < half; ++ff) {
                const int f = chi * half + ff;
                cpx<double> bv;
                if constexpr (ST) bv = Px[f * nvec + np];
                else {
                    const double2 b2 = B[(x * dof + f) * nvec + np];
                    bv = cpx<double>{b2.x, b2.y};
                }
                const cpx<double> w = W[f * N + m];
                cmac_conj(acc[i].re, acc[i].im, bv.re, bv.im, w.re, w.im);
            }
        }
    }
    double2* out = isY ? Yout + ((int64_t)term * Vc + xc) * N * N : Xpart + ((int64_t)hterm * Vc + xc) * N * N;
#pragma unroll
    for (int i = 0; i < GAL_MAXE; ++i) {
        const int e = threadIdx.x + i * T;
        if (e >= N * N) break;
        out[e] = make_double2(acc[i].re, acc[i].im);
    }
}

// ------------------------------------------------ fine parent on the matrix cores
// The fine parent's product as dense FP64 products.  A hop's block is
// -1/2 (1 -+ gamma_mu) (x) U, whose chirality blocks are the unit matrix and one
// entry per row and column, so per contributing site only Z = U Pf(x') is
// formed, 3x3 per spin and vector: for the rows f of one chirality the columns
// of the same chirality multiply Z itself, those of the other one Z with its two
// spins exchanged or not and a phase of +-1 or +-i.  (The on-site term has only
// the first kind.)  What is left, Pf(x)^+ W summed over the sites of the term,
// is per (chirality, kind) one real product of depth 6 per site,
//   S(i, j) = sum over (x, f) of Pf(x)(f, i) W(x)(f, j),  i = (n, re/im), j = (m, re/im),
// on v_mfma_f64_16x16x4_f64, one wave each, and then
//   T(n, m) = S(n re, m re) + S(n im, m im) + i [S(n re, m im) - S(n im, m re)].
// A work-group takes one (coarse site, term); it first lists the sites that
// contribute, then four of its waves stage the next CS of them in LDS (loads,
// Z, phases) while the other four multiply the ones before, one barrier per CS
// sites.  The work-groups of kGalGroup coarse sites run next to each other on
// one XCD, the terms with the most sites first.
// The staging waves keep FP64 products to the 36 of Z: FP64 vector instructions
// share their unit with the matrix ones and wait for the 64 cycles of each
// (leaving the phases and the -1/2 to sign bits and the end: 3.9 -> 3.45 ms).
// Bound: the FP64 matrix rate.  16^3x32, nvec 24: 123 GFLOP, 1.9 ms at 64
// TFLOP/s; 14.4 ms in the form above, which multiplies the dense 12x12 block on
// the vector unit, 6.9 ms with the four waves staging and multiplying in turn,
// 3.45 ms now (36 TFLOP/s, the matrix cores busy 45 % of the time; the rest is
// Z's own products, the on-site term's idle waves and the barriers).
constexpr int kGalList = 4096;   // most sites of an aggregate this form lists
constexpr int kGalGroup = 16;    // coarse sites (3 to 6: as fast at 16^3x32, where they share more of the L2, but
                                 // up to 1.4x slower below 128 coarse sites, the long terms of the last group ending alone)

struct HopSpin {   // W of spin `to[t]` gets (re + i im) times Z of spin t, per hop
    signed char to[8][4], re[8][4], im[8][4];
};

template <typename R, int RT, int CS>
__global__ __launch_bounds__(512, RT <= 3 ? 4 : 2) void k_galerkin_fine(
    double2* __restrict__ Yout, double2* __restrict__ Xpart, const cpx<R>* __restrict__ U, const R* __restrict__ clov,
    double diag, int use_clover, const int* __restrict__ nbr, const double2* __restrict__ B,
    const int* __restrict__ members, const int* __restrict__ owner, int64_t V, int64_t Vc, int nvec, int bsites,
    uint32_t rec, HopSpin hs) {
    typedef double V4 __attribute__((ext_vector_type(4)));
    constexpr int LD = 16 * RT + 8;      // doubles per LDS row (the four row groups of a read in different banks)
    constexpr int ROWS = 6 * CS;         // rows of a chunk and chirality, a multiple of the depth 4
    constexpr int BUF = 6 * ROWS * LD;   // Pf(x) [2][ROWS][LD], then W [2][2][ROWS][LD]: same and other chirality
    constexpr int PI = (CS * 12 * 8 * RT + 255) / 256;   // entries of Pf(x) per staging thread
    static_assert(ROWS % 4 == 0, "whole products");
    static_assert(CS * 4 * 8 * RT <= 256, "one entry of Z per staging thread");
    extern __shared__ __align__(16) unsigned char smem[];
    double* bufs = reinterpret_cast<double*>(smem);   // two
    int* list = reinterpret_cast<int*>(bufs + 2 * BUF);   // [2][bsites]: x, x'
    __shared__ int wsum[8], total;
    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nx = (int)((Vc + 7) >> 3), seq = blockIdx.x >> 3;
    const int g0 = seq / (17 * kGalGroup) * kGalGroup, gn = nx - g0 < kGalGroup ? nx - g0 : kGalGroup;
    const int order = (seq - 17 * g0) / gn;
    const int64_t xc = (int64_t)(g0 + (seq - 17 * g0) % gn) * 8 + (blockIdx.x & 7);
    if (xc >= Vc) return;
    const bool isY = order > 8;
    const int hterm = isY ? order - 9 : order == 0 ? 8 : order - 1;
    const int N = 2 * nvec;
    // contributing sites, in the aggregate's order
    if (tid == 0) total = 0;
    __syncthreads();
    for (int b0 = 0; b0 < bsites; b0 += 512) {
        const int b = b0 + tid;
        bool take = false;
        int x = 0, xn = 0;
        if (b < bsites) {
            x = members[xc * bsites + b];
            if (hterm < 8) xn = nbr[(int64_t)x * 8 + hterm];
            take = hterm == 8 || (owner[xn] == xc) != isY;
        }
        const unsigned long long mask = __ballot(take);
        if (l == 0) wsum[w] = __popcll(mask);
        __syncthreads();
        int at = total + __popcll(mask & ((1ull << l) - 1));
        for (int q = 0; q < w; ++q) at += wsum[q];
        if (take) {
            list[at] = x;
            list[bsites + at] = xn;
        }
        __syncthreads();
        if (tid == 0)
            for (int q = 0; q < 8; ++q) total += wsum[q];
        __syncthreads();
    }
    const int nsites = total;
    // staging waves: `load` takes a chunk's inputs into registers, from the last
    // site where the chunk runs past it, and `write` forms W and puts both into
    // LDS, zeros past the last site; the loads of one chunk fly while the chunk
    // before is multiplied
    const int pt = tid - 256;
    auto stage = [&](auto hop_c) {
        constexpr bool HOP = decltype(hop_c)::value;
        const bool back = hterm & 1;
        const int wq = (int)((pt * rec) >> 20), wk = pt - wq * nvec;   // this thread's entry of W
        const int ws = HOP ? wq >> 2 : wq >> 1, wt = HOP ? wq & 3 : wq & 1;
        const bool has = pt < CS * (HOP ? 4 : 2) * nvec;
        const int to = HOP ? hs.to[hterm][wt] : 0;
        // the phase without FP64 products, which would wait for the matrix
        // products on the same unit: (+-i) z exchanges the parts
        const int fr = HOP ? hs.re[hterm][wt] : 0, fi = HOP ? hs.im[hterm][wt] : 0;
        const bool turn = fr == 0;
        const unsigned nre = fr < 0 || fi > 0 ? 0x80000000u : 0, nim = fr < 0 || fi < 0 ? 0x80000000u : 0;
        auto flip = [](double d, unsigned sign) {
            return __hiloint2double((int)((unsigned)__double2hiint(d) ^ sign), __double2loint(d));
        };
        int bo[PI], ps[PI], po[PI];   // this thread's entries of Pf(x)
#pragma unroll
        for (int q = 0; q < PI; ++q) {
            const int e0 = pt + 256 * q, e = e0 < CS * 12 * nvec ? e0 : 0;
            const int fs = (int)((e * rec) >> 20), k = e - fs * nvec, f = fs % 12;
            ps[q] = fs / 12;
            bo[q] = f * nvec + k;
            po[q] = e0 < CS * 12 * nvec ? ((f / 6) * ROWS + ps[q] * 6 + f % 6) * LD + 2 * k : -1;
        }
        double2 pv[PI], v[HOP ? 3 : 6];
        cpx<R> u[9];
        auto at = [&](int c) { return c < nsites ? c : nsites - 1; };
        auto load = [&](int c0) {
#pragma unroll
            for (int q = 0; q < PI; ++q) pv[q] = B[(int64_t)list[at(c0 + ps[q])] * 12 * nvec + bo[q]];
            if (has) {
                if constexpr (HOP) {
                    const int x = list[at(c0 + ws)], xn = list[bsites + at(c0 + ws)], xl = back ? xn : x;
#pragma unroll
                    for (int b = 0; b < 3; ++b) v[b] = B[((int64_t)xn * 12 + 3 * wt + b) * nvec + wk];
#pragma unroll
                    for (int e = 0; e < 9; ++e) u[e] = U[(int64_t)((hterm >> 1) * 9 + e) * V + xl];
                } else {
                    const int x = list[at(c0 + ws)];
#pragma unroll
                    for (int b = 0; b < 6; ++b) v[b] = B[((int64_t)x * 12 + 6 * wt + b) * nvec + wk];
                }
            }
        };
        auto write = [&](int c0, double* buf) {
            double* Wb = buf + 2 * ROWS * LD;
            auto put = [&](double* to_, bool ok, double re, double im) {
                *reinterpret_cast<double2*>(to_) = ok ? make_double2(re, im) : make_double2(0, 0);
            };
            const bool ok = c0 + ws < nsites;
            if (has) {
                if constexpr (HOP) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        cpx<double> z = {0, 0};
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            // U_mu(x), or U_mu(x - mu)^+
                            const cpx<R> h = back ? cpx<R>{u[3 * b + a].re, -u[3 * b + a].im} : u[3 * a + b];
                            cmac(z.re, z.im, (double)h.re, (double)h.im, v[b].x, v[b].y);
                        }
                        put(Wb + ((wt >> 1) * 2 * ROWS + ws * 6 + (wt & 1) * 3 + a) * LD + 2 * wk, ok, z.re, z.im);
                        put(Wb + ((to >> 1) * 2 * ROWS + ROWS + ws * 6 + (to & 1) * 3 + a) * LD + 2 * wk, ok,
                            flip(turn ? z.im : z.re, nre), flip(turn ? z.re : z.im, nim));
                    }
                } else {   // (diag + A) Pf(x), one chirality block
                    cpx<double> t[6];
#pragma unroll
                    for (int i = 0; i < 6; ++i) t[i] = {diag * v[i].x, diag * v[i].y};
                    if (use_clover) {
                        const R* A = clov + (int64_t)wt * 36 * V + list[at(c0 + ws)];
                        int o = 0;
#pragma unroll
                        for (int a = 0; a < 6; ++a) {
                            const double d = (double)A[a * V];
                            t[a].re = fma(d, v[a].x, t[a].re);
                            t[a].im = fma(d, v[a].y, t[a].im);
#pragma unroll
                            for (int b = a + 1; b < 6; ++b, ++o) {
                                const double re = (double)A[(6 + 2 * o) * V], im = (double)A[(7 + 2 * o) * V];
                                cmac(t[a].re, t[a].im, re, im, v[b].x, v[b].y);
                                cmac_conj(t[b].re, t[b].im, re, im, v[a].x, v[a].y);
                            }
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 6; ++i)
                        put(Wb + (wt * 2 * ROWS + ws * 6 + i) * LD + 2 * wk, ok, t[i].re, t[i].im);
                }
            }
#pragma unroll
            for (int q = 0; q < PI; ++q)
                if (po[q] >= 0) put(buf + po[q], c0 + ps[q] < nsites, pv[q].x, pv[q].y);
        };
        load(0);
        for (int c0 = 0; c0 < nsites; c0 += CS) {
            write(c0, bufs + ((c0 / CS) & 1) * BUF);
            load(c0 + CS);
            __syncthreads();
        }
    };
    const int chi = (w & 3) >> 1, cross = w & 1;
    const int i16 = l & 15, g = l >> 4;
    if (w >= 4) {
        __builtin_amdgcn_s_setprio(3);
        if (nsites) {
            if (hterm < 8) stage(std::true_type{});
            else stage(std::false_type{});
        }
        return;
    }
    V4 acc[RT][RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j) acc[i][j] = V4{0, 0, 0, 0};
    for (int c0 = 0; c0 < nsites; c0 += CS) {
        __syncthreads();   // chunk c0 is staged; the one before it has been read by all
        if (!(cross && hterm == 8)) {
            const double* buf = bufs + ((c0 / CS) & 1) * BUF;
            const double* pa = buf + (chi * ROWS + g) * LD + i16;
            const double* wb = buf + 2 * ROWS * LD + ((chi * 2 + cross) * ROWS + g) * LD + i16;
#pragma unroll
            for (int s = 0; s < ROWS / 4; ++s) {
                double a[RT], b[RT];
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    a[i] = pa[4 * s * LD + 16 * i];
                    b[i] = wb[4 * s * LD + 16 * i];
                }
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < RT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    // element q of a lane: row g + 4 q, column i16 of its tile; the hops' -1/2 is left to here
    const double scale = hterm < 8 ? -0.5 : 1.0;
    double2* out = isY ? Yout + ((int64_t)hterm * Vc + xc) * N * N : Xpart + ((int64_t)hterm * Vc + xc) * N * N;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double v = acc[i][j][q];
                const double rc = __shfl(v, (l + 1) & 63, 64), cr = __shfl(v, (l + 16) & 63, 64), cc = __shfl(v, (l + 17) & 63, 64);
                const int n = (16 * i + g + 4 * q) >> 1, m = (16 * j + i16) >> 1;
                if (!((g | i16) & 1) && n < nvec && m < nvec)
                    out[(int64_t)(chi * nvec + n) * N + (cross ? 1 - chi : chi) * nvec + m] = make_double2(scale * (v + cc), scale * (rc - cr));
            }
}

static Proj projectors() {
    Proj P{};
    for (int mu = 0; mu < 4; ++mu) {
        double g[4][4][2];
        gamma_matrix(mu, g);
        for (int r = 0; r < 4; ++r)
            for (int c = 0; c < 4; ++c) {
                const double id = r == c ? 1.0 : 0.0;
                P.p[2 * mu][r][c][0] = id - g[r][c][0];
                P.p[2 * mu][r][c][1] = -g[r][c][1];
                P.p[2 * mu + 1][r][c][0] = id + g[r][c][0];
                P.p[2 * mu + 1][r][c][1] = g[r][c][1];
            }
    }
    return P;
}

// where the other chirality's columns of (1 -+ gamma_mu) take each spin's Z, and with which phase
static HopSpin hop_spins(const Proj& P) {
    HopSpin h{};
    for (int d = 0; d < 8; ++d)
        for (int t = 0; t < 4; ++t)
            for (int s = 0; s < 4; ++s) {
                if (s / 2 == t / 2 || (P.p[d][s][t][0] == 0.0 && P.p[d][s][t][1] == 0.0)) continue;
                h.to[d][t] = (signed char)s;
                h.re[d][t] = (signed char)P.p[d][s][t][0];
                h.im[d][t] = (signed char)P.p[d][s][t][1];
            }
    return h;
}

template <typename R, int RT>
static qmg_status launch_galerkin_fine(qmg_transfer t, qmg_fine_op fine, double2* Y, double2* Xp, const HopSpin& hs,
                                       hipStream_t s) {
    constexpr int CS = RT == 1 ? 4 : 2;
    const size_t lds = sizeof(double) * 2 * 6 * 6 * CS * (16 * RT + 8) + sizeof(int) * 2 * t->bsites;
    // e / nvec as (e * rec) >> 20, exact for the e < 2048 of a chunk
    // (rec nvec - 2^20 < nvec, so the quotient is at most e / 2^20 too large, under 1 / nvec)
    const uint32_t rec = ((1u << 20) + t->nvec - 1) / t->nvec;
    auto kern = k_galerkin_fine<R, RT, CS>;
    if (lds > 65536) QMG_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3((unsigned)((t->Vc + 7) / 8 * 8 * 17)), dim3(512), lds, s, Y, Xp, (const cpx<R>*)fine->U,
                       (const R*)fine->clov, 4.0 + fine->m0, fine->csw != 0.0 ? 1 : 0, fine->nbr, t->basis64, t->members,
                       t->owner, t->V, t->Vc, t->nvec, t->bsites, rec, hs);
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}
template <typename R>
static qmg_status galerkin_fine(qmg_transfer t, qmg_fine_op fine, double2* Y, double2* Xp, const HopSpin& hs,
                                hipStream_t s) {
    if (t->nvec <= 8) return launch_galerkin_fine<R, 1>(t, fine, Y, Xp, hs, s);
    if (t->nvec <= 16) return launch_galerkin_fine<R, 2>(t, fine, Y, Xp, hs, s);
    if (t->nvec <= 24) return launch_galerkin_fine<R, 3>(t, fine, Y, Xp, hs, s);
    return launch_galerkin_fine<R, 4>(t, fine, Y, Xp, hs, s);
}

__global__ void k_sum_xparts(double2* __restrict__ X, const double2* __restrict__ Xpart, int64_t n) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    double re = 0, im = 0;
    for (int t = 0; t < 9; ++t) {  // hops 0..7, then the on-site term
        re += Xpart[t * n + g].x;
        im += Xpart[t * n + g].y;
    }
    X[g] = make_double2(re, im);
}

}  // namespace qmg

using namespace qmg;

extern "C" qmg_status qmg_build_coarse_op(qmg_transfer t, qmg_fine_op fine, qmg_coarse_op parent,
                                          qmg_prec storage, void* stream, qmg_coarse_op* out) {
    if (!out) return fail(QMG_ERR_ARG, "build_coarse_op: out is NULL");
    *out = nullptr;
    if (!t) return fail(QMG_ERR_ARG, "build_coarse_op: transfer is NULL");
    if ((fine == nullptr) == (parent == nullptr))
        return fail(QMG_ERR_ARG, "build_coarse_op: give exactly one of fine / parent");
    const int* pdims = fine ? fine->dims : parent->dims;
    const int pdof = fine ? 12 : parent->N;
    for (int m = 0; m < 4; ++m)
        if (pdims[m] != t->fdims[m])
            return fail(QMG_ERR_SHAPE, "build_coarse_op: transfer lattice does not match the parent");
    if (pdof != t->dof) return fail(QMG_ERR_SHAPE, "build_coarse_op: transfer dof %d != parent dof %d", t->dof, pdof);
    const int N = 2 * t->nvec;
    if (pdof * N > 4096)
        return fail(QMG_ERR_SHAPE, "build_coarse_op: parent dof x N = %d exceeds 4096", pdof * N);
    if (storage != QMG_C128 && storage != QMG_C64)
        return fail(QMG_ERR_PREC, "build_coarse_op: storage %d not supported", (int)storage);
    const qmg_prec from = fine ? fine->storage : parent->storage;
    if (from != QMG_C128 && from != QMG_C64)
        return fail(QMG_ERR_PREC, "build_coarse_op: the parent operator must use complex128 or complex64 storage");
    if (fine && fine->link_reals != 18)
        return fail(QMG_ERR_PREC, "build_coarse_op: the fine operator must store all 18 link reals");
    hipStream_t s = as_stream(stream);
    const int64_t Vc = t->Vc;
    const size_t blk = (size_t)Vc * N * N;
    double2 *Y = nullptr, *Xp = nullptr, *X = nullptr;
    hipError_t e = hipMalloc(&Y, sizeof(double2) * 8 * blk);
    if (e == hipSuccess) e = hipMalloc(&Xp, sizeof(double2) * 9 * blk);
    if (e == hipSuccess) e = hipMalloc(&X, sizeof(double2) * blk);
    auto cleanup = [&]() {
        if (Y) (void)hipFree(Y);
        if (Xp) (void)hipFree(Xp);
        if (X) (void)hipFree(X);
    };
    if (e != hipSuccess) {
        cleanup();
        return fail(QMG_ERR_NOMEM, "build_coarse_op: %s", hipGetErrorString(e));
    }
    int threads = 256;
    while ((int64_t)threads * GAL_MAXE < (int64_t)N * N) threads += 64;
    if (threads > 1024) {
        cleanup();
        return fail(QMG_ERR_SHAPE, "build_coarse_op: N=%d too large", N);
    }
    // W [pdof][N]; with the parent's block H [pdof][pdof] and the two basis
    // blocks [pdof][nvec] staged too when all of it fits in 64 KiB (the fine
    // parent: 21 KiB).  A larger staging area would cost more in occupancy
    // than it saves (measured on a 48 -> 64 coarse parent: 2.2 ms unstaged,
    // 2.75 ms with H staged).
    const size_t lds_st = sizeof(cpx<double>) * ((size_t)pdof * N + (size_t)pdof * pdof + 2 * (size_t)pdof * t->nvec);
    const bool st_lds = lds_st <= 65536;
    const size_t lds = st_lds ? lds_st : sizeof(cpx<double>) * (size_t)pdof * N;
    const dim3 grid((unsigned)(Vc * 17));
    const Proj P = projectors();
    qmg_fine_op_s fop{};
    qmg_coarse_op_s cop{};
#define QMG_GAL(FINE, R, ST, A, B_)                                                                            \
    hipLaunchKernelGGL((k_galerkin<FINE, R, ST>), grid, dim3(threads), lds, s, Y, Xp, fop, cop, A, B_,           \
                       FINE ? fine->nbr : parent->nbr, t->basis64, t->members, t->owner, Vc, pdof, t->nvec,     \
                       t->bsites, P)
    // a fine parent goes to the matrix cores up to 32 vectors (four 16-column
    // tiles) and aggregates whose site list fits beside the staged rows
    if (fine && t->nvec <= 32 && t->bsites <= kGalList) {
        const HopSpin hs = hop_spins(P);
        const qmg_status gst = fine->storage == QMG_C128 ? galerkin_fine<double>(t, fine, Y, Xp, hs, s)
                                                         : galerkin_fine<float>(t, fine, Y, Xp, hs, s);
        if (gst != QMG_OK) {
            cleanup();
            return gst;
        }
    } else if (fine) {
        fop = *fine;
        const bool d = fine->storage == QMG_C128;
        if (st_lds) {
            if (d) QMG_GAL(true, double, true, fine->U, fine->clov);
            else QMG_GAL(true, float, true, fine->U, fine->clov);
        } else {
            if (d) QMG_GAL(true, double, false, fine->U, fine->clov);
            else QMG_GAL(true, float, false, fine->U, fine->clov);
        }
    } else {
        cop = *parent;
        const bool d = parent->storage == QMG_C128;
        if (st_lds) {
            if (d) QMG_GAL(false, double, true, parent->links, nullptr);
            else QMG_GAL(false, float, true, parent->links, nullptr);
        } else {
            if (d) QMG_GAL(false, double, false, parent->links, nullptr);
            else QMG_GAL(false, float, false, parent->links, nullptr);
        }
    }
#undef QMG_GAL
    hipLaunchKernelGGL(k_sum_xparts, dim3((unsigned)((blk + 255) / 256)), dim3(256), 0, s, X, Xp, (int64_t)blk);
    e = hipGetLastError();
    if (e != hipSuccess) {
        cleanup();
        return fail(QMG_ERR_HIP, "build_coarse_op: launch: %s", hipGetErrorString(e));
    }
    qmg_status st = qmg_coarse_op_create(t->cdims, N, X, Y, storage, stream, out);
    // the create call packs X, Y on the same stream; wait before freeing them
    e = hipStreamSynchronize(s);
    cleanup();
    if (st != QMG_OK) return st;
    if (e != hipSuccess) {
        qmg_coarse_op_destroy(*out);
        *out = nullptr;
        return fail(QMG_ERR_HIP, "build_coarse_op: %s", hipGetErrorString(e));
    }
    return QMG_OK;
}
