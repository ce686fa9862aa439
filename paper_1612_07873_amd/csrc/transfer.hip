// Transfer operators (Sec. 3.4 step 3 and Sec. 6.6).
//
// Setup: the near-null vectors are cut into hypercubic aggregates; within
// each aggregate the two chirality halves of every vector (fine level: spins
// {0,1} vs {2,3}; coarse parent: components n < N/2 vs n >= N/2) are
// orthonormalised separately by modified Gram-Schmidt in vector order, every
// projection done twice, normalised so that R has a real positive diagonal.
// One work-group per (aggregate, chirality), FP64, working set in global
// memory (it is read from L2).
//
// Apply, for all members of a batch together:
//   prolong  (P u)(x)_f = sum_k V(x)_{f,k} u(xc(x))_{chi(f)*Nvec + k}
//   restrict (R psi)(xc)_{chi*Nvec + k} = sum_{x in xc, chi(f) = chi} conj(V(x)_{f,k}) psi(x)_f
// both as dense products per (aggregate, chirality), on the matrix cores or for
// few members on the vector unit, every sum in one fixed order: no atomics,
// bitwise repeatable, and a member of a batch equals the single call bitwise.
// The basis is kept as [V][dof][Nvec] (row f of site x holds the Nvec
// coefficients of its chirality) in the storage precision, plus an FP64 copy
// for the Galerkin build.  The 16-bit storage keeps each complex entry as an
// FP16 pair with no scale: the columns are orthonormal within an aggregate,
// so no entry exceeds 1 in modulus.
#include "codes16.h"
#include "handles.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace qmg {

__device__ __forceinline__ double block_sum(double v, double* red) {
    // sum over the work-group; result returned to every thread
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    double t = 0;
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) t += red[i];
    return t;
}

// gather vecs [nvec][V][dof] -> W [Vc][2][nvec][Lb]  (Lb = bsites*dof/2)
__global__ void k_gather_blocks(double2* __restrict__ W, const double2* __restrict__ vecs,
                                const int* __restrict__ members, int64_t V, int64_t Vc, int dof,
                                int nvec, int bsites) {
    const int half = dof / 2;
    const int64_t Lb = (int64_t)bsites * half;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = Vc * 2 * nvec * Lb;
    if (g >= total) return;
    const int64_t p = g % Lb;
    int64_t t = g / Lb;
    const int k = (int)(t % nvec);
    t /= nvec;
    const int chi = (int)(t % 2);
    const int64_t xc = t / 2;
    const int64_t x = members[xc * bsites + p / half];
    const int f = chi * half + (int)(p % half);
    W[g] = vecs[((int64_t)k * V + x) * dof + f];
}

// MGS on one (aggregate, chirality) per work-group.
__global__ __launch_bounds__(256) void k_block_mgs(double2* __restrict__ W, int nvec, int64_t Lb,
                                                    double rank_tol, int* __restrict__ rank_fail) {
    __shared__ double red[8];
    double2* Wb = W + (int64_t)blockIdx.x * nvec * Lb;
    for (int k = 0; k < nvec; ++k) {
        double2* wk = Wb + (int64_t)k * Lb;
        double s = 0;
        for (int64_t i = threadIdx.x; i < Lb; i += blockDim.x) s += wk[i].x * wk[i].x + wk[i].y * wk[i].y;
        const double before = sqrt(block_sum(s, red));
        for (int pass = 0; pass < 2; ++pass)
            for (int j = 0; j < k; ++j) {
                const double2* wj = Wb + (int64_t)j * Lb;
                double cr = 0, cim = 0;
                for (int64_t i = threadIdx.x; i < Lb; i += blockDim.x) {
                    cr += wj[i].x * wk[i].x + wj[i].y * wk[i].y;    // conj(wj) * wk
                    cim += wj[i].x * wk[i].y - wj[i].y * wk[i].x;
                }
                cr = block_sum(cr, red);
                cim = block_sum(cim, red);
                for (int64_t i = threadIdx.x; i < Lb; i += blockDim.x) {
                    const double2 a = wj[i];
                    wk[i].x -= cr * a.x - cim * a.y;
                    wk[i].y -= cr * a.y + cim * a.x;
                }
                __syncthreads();
            }
        s = 0;
        for (int64_t i = threadIdx.x; i < Lb; i += blockDim.x) s += wk[i].x * wk[i].x + wk[i].y * wk[i].y;
        const double nrm = sqrt(block_sum(s, red));
        if (!(nrm >= rank_tol * before) || nrm == 0.0) {
            if (threadIdx.x == 0) rank_fail[0] = 1;
        }
        const double inv = nrm > 0 ? 1.0 / nrm : 0.0;
        for (int64_t i = threadIdx.x; i < Lb; i += blockDim.x) {
            wk[i].x *= inv;
            wk[i].y *= inv;
        }
        __syncthreads();
    }
}

// W [Vc][2][nvec][Lb] -> basis [V][dof][nvec]
__global__ void k_scatter_basis(double2* __restrict__ B, const double2* __restrict__ W,
                                const int* __restrict__ members, int64_t Vc, int dof, int nvec,
                                int bsites) {
    const int half = dof / 2;
    const int64_t Lb = (int64_t)bsites * half;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= Vc * 2 * nvec * Lb) return;
    const int64_t p = g % Lb;
    int64_t t = g / Lb;
    const int k = (int)(t % nvec);
    t /= nvec;
    const int chi = (int)(t % 2);
    const int64_t xc = t / 2;
    const int64_t x = members[xc * bsites + p / half];
    const int f = chi * half + (int)(p % half);
    B[(x * dof + f) * nvec + k] = W[g];
}

__global__ void k_to_c64(float2* __restrict__ o, const double2* __restrict__ i, int64_t n) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n) o[g] = make_float2((float)i[g].x, (float)i[g].y);
}
__global__ void k_to_h16(uint32_t* __restrict__ o, const double2* __restrict__ i, int64_t n, unsigned* __restrict__ nf) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    note_nonfinite(nf, !(isfinite(i[g].x) && isfinite(i[g].y)));
    o[g] = enc_pair<FMT_H16>((float)i[g].x, (float)i[g].y);
}

// Both directions run on the matrix cores, in the arithmetic precision of the
// fields (v_mfma_f32_16x16x4_f32 / v_mfma_f64_16x16x4_f64: one real per lane
// and operand, products and sums in that precision).  Per aggregate and
// chirality the transfer is one dense product with the aggregate's block of
// the basis, a real matrix of rows (site, f) and 2 nvec columns (k, re/im);
// the fields' columns are (member, re/im), so 8 members fill a tile of 16
// columns and the basis is read once for up to 32 members.  The bound is the
// basis stream: complex64, 16^3x32, nvec 24, twelve members, 302 MB of basis
// and 151 MB of fields.  One kernel per member (each re-reading the basis)
// took 524 us (restriction) and 673 us (prolongation); these take 83 and 113
// (one call repeated; in turn, as a solve makes them, 108 and 108, the bytes moved
// 1.00 and 1.10 times these).
// Every column of a product is summed in the same order whatever the number of
// members, and the forms for few members below keep that order, so a member of
// a batch equals the single call bitwise with every storage of the basis.
template <typename R> struct Mm;
template <> struct Mm<float> {
    typedef float V4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V4 mac(float a, float b, V4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // row of a lane's element q (column lane % 16), g = lane / 16
    static __device__ __forceinline__ int row(int g, int q) { return 4 * g + q; }
};
template <> struct Mm<double> {
    typedef double V4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V4 mac(double a, double b, V4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int q) { return 4 * q + g; }
};

// The (aggregate, chirality) of work-group i: work-groups are dealt to the 8
// XCDs round-robin, and the two chiralities of an aggregate, whose rows of a
// field share cache lines, go to the same one.  -1 past the last aggregate.
__device__ __forceinline__ int64_t agg_of(int64_t i, int64_t Vc, int& chi) {
    const int64_t xc = (i >> 4) * 8 + (i & 7);
    chi = (int)(i >> 3) & 1;
    return xc < Vc ? xc : -1;
}
static int64_t agg_grid(int64_t Vc) { return (Vc + 7) / 8 * 16; }

// n reals of a basis row as stored (ST: the storage's real type), decoded only
// when they are used: a conversion next to the load would wait for it and end
// the prefetch.  FP16 is kept as words of two.  Plain reals are read by scalar
// loads, which the compiler joins into the widest that stay inside the n (a
// three-element vector type would be read as four, past the end of the basis).
template <typename ST, int n> struct Raw {
    ST v[n];
    template <typename R> __device__ __forceinline__ R get(int i) const { return (R)v[i]; }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = 0;
    }
};
template <int n> struct Raw<_Float16, n> {
    uint32_t v[(n + 1) / 2];
    template <typename R> __device__ __forceinline__ R get(int i) const {
        return (R)h16_to_f32((uint16_t)(i & 1 ? v[i >> 1] >> 16 : v[i >> 1] & 0xffffu));
    }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < (n + 1) / 2; ++i) v[i] = 0;
    }
};

// The T columns of a basis row that lane i of 16 holds in the restriction:
// T i + t, so that a lane's columns are contiguous; with FP16 the pairs
// 2 i, 2 i + 1 of each 32 columns and then, for an odd T, column 16 (T - 1) + i,
// which keeps every word aligned.
template <typename ST, int T> __device__ __forceinline__ int basis_col(int i, int t) {
    if constexpr (sizeof(ST) == 2) return T % 2 && t == T - 1 ? 16 * t + i : 32 * (t >> 1) + 2 * i + (t & 1);
    else return T * i + t;
}
// Those columns of a row (non-temporal: read once per application); past
// the last column, the last one or pair again.
template <bool FULL, typename ST, int T>
__device__ __forceinline__ void ld_cols(Raw<ST, T>& v, const ST* row, int i, int cols) {
    if constexpr (sizeof(ST) == 2) {
        const uint32_t* w = reinterpret_cast<const uint32_t*>(row);
#pragma unroll
        for (int t = 0; t < T / 2; ++t) {
            const int c = 16 * t + i;
            v.v[t] = __builtin_nontemporal_load(w + (FULL ? c : min(c, (cols >> 1) - 1)));
        }
        if constexpr (T % 2) {
            const int c = 16 * (T - 1) + i;
            v.v[T / 2] = __builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(row) + (FULL ? c : min(c, cols - 1)));
        }
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t) v.v[t] = __builtin_nontemporal_load(row + (FULL ? T * i + t : min(T * i + t, cols - 1)));
    }
}
// The columns of a basis row that lane group g of 4 holds in the prolongation:
// runs of L consecutive ones, run q at 4 L q + L g.  Zero past the last column.
template <bool FULL, int L, typename ST, int n>
__device__ __forceinline__ void ld_runs(Raw<ST, n>& v, const ST* row, int g, int cols) {
#pragma unroll
    for (int s = 0; s < n; s += L) {
        const int c0 = 4 * s + L * g;
        if constexpr (sizeof(ST) == 2) {
            const uint32_t* w = reinterpret_cast<const uint32_t*>(row + c0);
#pragma unroll
            for (int i = 0; i < L / 2; ++i) v.v[s / 2 + i] = FULL || c0 + 2 * i < cols ? w[i] : 0u;
        } else {
#pragma unroll
            for (int i = 0; i < L; ++i) v.v[s + i] = FULL || c0 + i < cols ? row[c0 + i] : ST(0);
        }
    }
}

// Orders a wave's own LDS accesses in the program: the hardware completes them
// in order, the fences (no instructions at this scope) keep the compiler from
// moving them past each other.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Restriction: S(m, n) = sum over the rows r of an (aggregate, chirality) of
// basis(r, m) field(r, n), m = (k, re/im), n = (member, re/im); the coarse
// component is then S(k re, j re) + S(k im, j im) + i [S(k re, j im) - S(k im, j re)].
// One work-group per (aggregate, chirality); its wave w takes the chunks of 16
// rows w, w + 8, ...  Each chunk's sum (four products of depth four) is added
// to the wave's total and the waves' totals are added in LDS, all in a fixed
// order.  A lane holds T consecutive columns of its row (T = 3 at nvec 24: a
// wave reads four whole rows, 768 contiguous bytes, per load), so tile t of S
// covers the columns basis_col(i, t).  A chunk's fields pass through the wave's own
// part of LDS as [row][n]; no wave waits for another before the end, and the
// next chunk's basis rows (non-temporal) and fields are in flight while this
// one is multiplied.  (Chunks of 128 rows staged by the whole work-group, two
// barriers each, took 139 us against 108 for twelve members, complex64.)
// FULL: the 16 T columns are all there (nvec a multiple of 8, at most 32);
// otherwise, and for the blocks of 32 vectors of a larger nvec (grid dimension
// z), columns past the last one read it again and are not stored.
constexpr int kRestrictWaves = 8;
constexpr int restrict_ld(int NT) { return NT == 1 ? 16 : 16 * NT + 16; }   // LDS row of a chunk: the four row groups of a read in different banks

template <typename R, typename ST, int T, int NT, bool FULL>
__global__ __launch_bounds__(64 * kRestrictWaves, T <= 3 && NT <= 2 && sizeof(R) == 4 ? 4 : 2) void k_restrict(
    cpx<R>* __restrict__ out, const ST* __restrict__ B, const cpx<R>* __restrict__ in, const int* __restrict__ members,
    int dof, int nvec, int bsites, int64_t V, int64_t Vc, int nrhs) {
    using V4 = typename Mm<R>::V4;
    constexpr int W = kRestrictWaves, U = 4, LDF = restrict_ld(NT), P = 2 * NT;
    extern __shared__ __align__(16) unsigned char smem[];
    R* sh = reinterpret_cast<R*>(smem);                // [wave][16][LDF], then [wave][16 T][16]
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int i16 = l & 15, g = l >> 4;
    int chi;
    const int64_t xc = agg_of(blockIdx.x, Vc, chi);
    if (xc < 0) return;   // the whole work-group
    const int half = dof >> 1;
    const int k0 = (int)blockIdx.z * 32;
    const int cols = 2 * (FULL ? nvec : (nvec - k0 < 32 ? nvec - k0 : 32));
    const int j0 = (int)blockIdx.y * 8 * NT;
    const int nj = nrhs - j0 < 8 * NT ? nrhs - j0 : 8 * NT;
    const int* mem = members + xc * bsites;
    const int rows = bsites * half;
    R* mine = sh + w * 16 * LDF;
    V4 tot[T][NT];
#pragma unroll
    for (int r = 0; r < T; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) tot[r][t] = V4{0, 0, 0, 0};
    // row i16 of the wave's current chunk: (site, f), stepped by 16 W rows
    int site = (16 * w + i16) / half, f = 16 * w + i16 - site * half;
    const int dsite = 16 * W / half, df = 16 * W - dsite * half;
    int x = mem[site < bsites ? site : bsites - 1];    // lattice site of the row (any for a row past the end)
    constexpr int NB = 2;   // chunks in flight, one included
    Raw<ST, T> a[NB][U];
    cpx<R> fv[NB][P];
    // Basis rows 4 u + g and this lane's field entries (row i16, members g + 4 p) of the current chunk,
    // then the site of the next chunk's row.  Rows past the end read a row of the last site, members past
    // the last one that one.
    auto load = [&](Raw<ST, T> (&d)[U], cpx<R> (&v)[P]) {
        const int64_t row = (int64_t)x * dof + chi * half + f;
#pragma unroll
        for (int u = 0; u < U; ++u)
            ld_cols<FULL>(d[u], B + ((int64_t)__shfl((long long)row, 4 * u + g, 64) * nvec + k0) * 2, i16, cols);
#pragma unroll
        for (int p = 0; p < P; ++p) v[p] = in[(int64_t)(j0 + min(g + 4 * p, nj - 1)) * V * dof + row];
        site += dsite;
        f += df;
        if (f >= half) { f -= half; ++site; }
        x = mem[site < bsites ? site : bsites - 1];
    };
    auto step = [&](Raw<ST, T> (&d)[U], cpx<R> (&v)[P], int c, bool more) {
        const bool live = 16 * c + i16 < rows;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            mine[i16 * LDF + 2 * (g + 4 * p)] = live ? v[p].re : R(0);
            mine[i16 * LDF + 2 * (g + 4 * p) + 1] = live ? v[p].im : R(0);
        }
        if (16 * c + 16 > rows) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (16 * c + 4 * u + g >= rows) d[u].zero();
        }
        wave_lds_sync();   // its lanes read what others wrote
        V4 acc[T][NT];
#pragma unroll
        for (int r = 0; r < T; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[r][t] = V4{0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            R b[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) b[t] = mine[(4 * u + g) * LDF + 16 * t + i16];
#pragma unroll
            for (int r = 0; r < T; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[r][t] = Mm<R>::mac(d[u].template get<R>(r), b[t], acc[r][t]);
        }
        wave_lds_sync();   // the next chunk overwrites it
#pragma unroll
        for (int r = 0; r < T; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) tot[r][t] += acc[r][t];
        if (more) load(d, v);   // the chunk NB steps on
    };
#pragma unroll
    for (int k = 0; k < NB; ++k)
        if (16 * (w + k * W) < rows) load(a[k], fv[k]);
    int c = w;
    // whole rounds first, whose loads are unconditional: a load under a
    // condition makes the next wait one for all loads before it
    for (; 16 * (c + (2 * NB - 1) * W) < rows; c += NB * W) {
#pragma unroll
        for (int k = 0; k < NB; ++k) step(a[k], fv[k], c + k * W, true);
    }
    for (; 16 * c < rows; c += NB * W) {
#pragma unroll
        for (int k = 0; k < NB; ++k)
            if (16 * (c + k * W) < rows) step(a[k], fv[k], c + k * W, 16 * (c + (k + NB) * W) < rows);
    }
    constexpr int M = 16 * T, LD = 16;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (8 * t >= nj) break;                        // the whole work-group
        __syncthreads();
#pragma unroll
        for (int r = 0; r < T; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) sh[(w * M + basis_col<ST, T>(Mm<R>::row(g, q), r)) * LD + i16] = tot[r][t][q];
        __syncthreads();
        for (int e = threadIdx.x; e < 8 * (cols >> 1); e += 64 * W) {
            const int jj = e / (cols >> 1), k = e - jj * (cols >> 1);
            if (8 * t + jj >= nj) continue;
            R re = 0, im = 0;
#pragma unroll
            for (int v = 0; v < W; ++v) {
                const R* p = sh + (v * M + 2 * k) * LD + 2 * jj;
                re += p[0] + p[LD + 1];
                im += p[1] - p[LD];
            }
            const int64_t o = (int64_t)(j0 + 8 * t + jj) * Vc + xc;
            out[o * 2 * nvec + chi * nvec + k0 + k] = cpx<R>{re, im};
        }
    }
}

// Prolongation: row r of an (aggregate, chirality) times the coarse columns,
//   P(r, j re) = sum_k W(k re) c(k, j).re - W(k im) c(k, j).im,
//   P(r, j im) = sum_k W(k re) c(k, j).im + W(k im) c(k, j).re.
// A work-group takes up to kProlongTiles tiles of 16 rows (grid dimension z
// divides an aggregate's tiles evenly), whose places in a fine field it first
// puts in LDS.  The coarse operand stays in registers while a wave walks its
// tiles; lane group g (of 16 lanes) holds KS columns of its rows in runs of L
// (ld_runs), and the next tile's are loaded while this one is multiplied.  A
// product of depth four takes one column of each lane group.  D neighbouring ones
// are added up in one chain (D = 1: one chain each, the chains of a pair added),
// these chains in order, then the runs: one chain over all columns had 1.6 times
// the error at nvec 24 (prolong_t chooses D).  Lanes of the two parts of a
// member exchange halves, so that each stores whole complex numbers (16 bytes
// where the rows of a chirality are even in number and `out` is so aligned:
// `wide`).  FULL: 2 nvec = 4 KS.
template <typename R> constexpr int kProlongTiles = sizeof(R) == 4 ? 16 : 32;   // complex64 66 (32 tiles) -> 63 us, complex128 132 (32) against 147 (16)

// Waves per SIMD, by the bytes of coarse operand a lane holds.  (Two or more
// also keep the accumulators where the vector unit can add them.)
constexpr int prolong_waves(int NT, int bytes) {
    return NT <= 2 && bytes <= 128 ? (NT == 1 ? 4 : 3) : bytes <= 256 ? 2 : 1;
}

template <typename R, typename ST, int KS, int L, int D, int NT, bool FULL>
__global__ __launch_bounds__(256, prolong_waves(NT, KS * NT * (int)sizeof(R))) void k_prolong(
    cpx<R>* __restrict__ out, const ST* __restrict__ B, const cpx<R>* __restrict__ uc, const int* __restrict__ members,
    int dof, int nvec, int bsites, int64_t V, int64_t Vc, int nrhs, int wide) {
    using V4 = typename Mm<R>::V4;
    __shared__ int64_t at[16 * kProlongTiles<R>];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int i16 = l & 15, g = l >> 4, odd = l & 1;
    int chi;
    const int64_t xc = agg_of(blockIdx.x, Vc, chi);
    if (xc < 0) return;   // the whole work-group
    const int half = dof >> 1;
    const int j0 = (int)blockIdx.y * 8 * NT;
    const int rows = bsites * half;
    const int tiles = (rows + 15) >> 4;
    const int t0 = (int)((int64_t)tiles * blockIdx.z / gridDim.z), t1 = (int)((int64_t)tiles * (blockIdx.z + 1) / gridDim.z);
    const int cols = 2 * nvec;
    for (int e = threadIdx.x; e < 16 * (t1 - t0); e += 256) {
        const int q = 16 * t0 + e;
        const int site = q / half;
        // -1 past the last row
        at[e] = q < rows ? (int64_t)members[xc * bsites + site] * dof + chi * half + (q - site * half) : -1;
    }
    R b[KS][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int j = j0 + 8 * t + (i16 >> 1);
        if (j >= nrhs) j = nrhs - 1;
        const cpx<R>* c = uc + ((int64_t)j * Vc + xc) * cols + chi * nvec;
#pragma unroll
        for (int s = 0; s < KS; s += 2) {
            const int e = 4 * (s - s % L) + L * g + s % L;
            cpx<R> v = {0, 0};
            if (FULL || e < cols) v = c[e >> 1];
            b[s][t] = odd ? v.im : v.re;
            b[s + 1][t] = odd ? v.re : -v.im;
        }
    }
    __syncthreads();
    auto load = [&](Raw<ST, KS>& a, int tile) {
        int64_t x = at[16 * tile + i16];
        if (x < 0) x = at[16 * tile];   // rows past the end: the tile's first row, not stored
        ld_runs<FULL, L>(a, B + x * cols, g, cols);
    };
    const int n = t1 - t0;
    auto step = [&](Raw<ST, KS>& a, int tile) {
        // this lane's two rows: elements 0 and 1 (even lanes) or 2 and 3 (odd lanes)
        const int64_t o0 = at[16 * tile + Mm<R>::row(g, 2 * odd)], o1 = at[16 * tile + Mm<R>::row(g, 2 * odd + 1)];
        V4 acc[NT], run[NT];
#pragma unroll
        for (int s = 0; s < KS; s += 2) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const V4 zero = {0, 0, 0, 0};
                V4 c = Mm<R>::mac(a.template get<R>(s), b[s][t], D == 4 && s % 4 ? run[t] : zero);
                V4 d = Mm<R>::mac(a.template get<R>(s + 1), b[s + 1][t], D == 1 ? zero : c);
                if constexpr (D == 1) d = c + d;
                run[t] = D == 4 || s % L == 0 ? d : run[t] + d;
                if ((s + 2) % L == 0) acc[t] = s >= L ? acc[t] + run[t] : run[t];
                if (sizeof(R) == 8) __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);   // else more products are started than there are registers for
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const R x0 = odd ? acc[t][0] : acc[t][2], x1 = odd ? acc[t][1] : acc[t][3];
            const R y0 = __shfl_xor(x0, 1, 64), y1 = __shfl_xor(x1, 1, 64);
            const cpx<R> v0 = odd ? cpx<R>{y0, acc[t][2]} : cpx<R>{acc[t][0], y0};
            const cpx<R> v1 = odd ? cpx<R>{y1, acc[t][3]} : cpx<R>{acc[t][1], y1};
            const int j = j0 + 8 * t + (i16 >> 1);
            if (j >= nrhs) continue;
            cpx<R>* o = out + (int64_t)j * V * dof;
            if (sizeof(R) == 4 && wide) {
                if (o0 >= 0) *reinterpret_cast<float4*>(o + o0) = make_float4(v0.re, v0.im, v1.re, v1.im);
            } else {
                if (o0 >= 0) o[o0] = v0;
                if (o1 >= 0) o[o1] = v1;
            }
        }
    };
    // NB tiles in flight, one included; whole rounds first, whose loads are
    // unconditional (a load under a condition makes the next wait one for all
    // loads before it)
    constexpr int NB = KS * NT * sizeof(R) <= 256 ? 2 : 1;
    Raw<ST, KS> a[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k)
        if (w + 4 * k < n) load(a[k], w + 4 * k);
    int tile = w;
    for (; tile + 4 * (2 * NB - 1) < n; tile += 4 * NB) {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            step(a[k], tile + 4 * k);
            load(a[k], tile + 4 * (k + NB));
        }
    }
    for (; tile < n; tile += 4 * NB) {
#pragma unroll
        for (int k = 0; k < NB; ++k)
            if (tile + 4 * k < n) {
                step(a[k], tile + 4 * k);
                if (tile + 4 * (k + NB) < n) load(a[k], tile + 4 * (k + NB));
            }
    }
}

// ----------------------------------------------------- on the vector unit
// One field fills 2 of the matrix cores' 16 columns, and with few vectors
// their tiles are mostly padding.  The same products on the vector unit, each
// member reading the basis for itself.  A matrix product of depth four is a
// chain of multiply-adds in the order of its depth, so these kernels form the
// sums above term by term: a field's result does not depend on the form, and
// the choice between them (transfer_prolong, transfer_restrict) is one of speed
// alone.  Bound: the basis stream.  One member, 16^3x32, nvec 24, restriction and
// prolongation: FP32 51 and 55 us (302 MB each; on the matrix cores 57 and 62),
// FP16 29 and 31 (48 and 37), FP64 103 and 118 us (122 and 127).  32^3x64: FP32
// 756 and 1020 us, FP16 426 and 562 us (2.4 GB each).
// BT: the stored entry, cpx<R> or a 32-bit FP16 pair.
template <typename R> __device__ __forceinline__ cpx<R> bval(const cpx<R>& b) { return b; }
template <typename R> __device__ __forceinline__ cpx<R> bval(const uint32_t& w) { return dec_pair<FMT_H16>(w); }
__device__ __forceinline__ float fma_r(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) { return __builtin_fma(a, b, c); }

// P consecutive entries in one load.  NT: non-temporal, so that the basis
// stream does not push the fine vector being restricted out of the caches (the
// prolongation, which reads the small coarse vector, is slower with them).
template <bool NT, int P, typename BT>
__device__ __forceinline__ void ld_entries(BT* b, const BT* p) {
    constexpr int words = (int)sizeof(BT) * P / 4;
    if constexpr (words == 1) {
        const int* w = reinterpret_cast<const int*>(p);
        const int v = NT ? __builtin_nontemporal_load(w) : *w;
        __builtin_memcpy(b, &v, 4);
    } else {
        static_assert(words == 2 || words == 4, "4, 8 or 16 bytes");
        typedef int vec __attribute__((ext_vector_type(words)));
        const vec* w = reinterpret_cast<const vec*>(p);
        const vec v = NT ? __builtin_nontemporal_load(w) : *w;
        __builtin_memcpy(b, &v, sizeof(v));
    }
}

// The sum of a run for one row: entry h of lane group g at H g + h, GN groups.
template <int H, int GN, int D, typename R, typename BT>
__device__ __forceinline__ cpx<R> run_sum(const BT* b, const cpx<R>* u) {
    cpx<R> sum = {0, 0};
    R x1 = 0, y1 = 0;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        // the entries' real parts, then their imaginary ones: a chain per product, both in one, or on from the entry before
        R x = D == 4 ? x1 : R(0), y = D == 4 ? y1 : R(0);
#pragma unroll
        for (int g = 0; g < GN; ++g) {
            const cpx<R> w = bval<R>(b[H * g + h]), v = u[H * g + h];
            x = fma_r(w.re, v.re, x);
            y = fma_r(w.re, v.im, y);
        }
        x1 = D == 1 ? R(0) : x;
        y1 = D == 1 ? R(0) : y;
#pragma unroll
        for (int g = 0; g < GN; ++g) {
            const cpx<R> w = bval<R>(b[H * g + h]), v = u[H * g + h];
            x1 = fma_r(w.im, -v.im, x1);
            y1 = fma_r(w.im, v.re, y1);
        }
        if (D == 1) {
            x1 = x + x1;
            y1 = y + y1;
        }
        sum = h && D != 4 ? cpx<R>{sum.re + x1, sum.im + y1} : cpx<R>{x1, y1};
    }
    return sum;
}

// Prolongation: a lane takes a run of 4 L columns (2 L entries), keeps its part
// of the coarse vector and walks the rows of a slab of an (aggregate, chirality),
// one slab per wave; the lanes of a row add their runs in order.  The next row's
// entries are in flight while one is multiplied.  Loads of P entries, which
// divides nvec; FULL: 2 L does.
constexpr int kProlongRows = 256;   // most rows of a slab

template <typename R, typename BT, int L, int D, int P, bool FULL>
__global__ __launch_bounds__(256) void k_prolong_vec(cpx<R>* __restrict__ out, const BT* __restrict__ B,
                                                     const cpx<R>* __restrict__ uc, const int* __restrict__ members,
                                                     int dof, int nvec, int bsites, int64_t V, int64_t Vc, int slabs) {
    constexpr int E = 2 * L;
    __shared__ int64_t places[4 * kProlongRows];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int64_t unit = 4 * (int64_t)blockIdx.x + w, agg = unit / slabs;
    if (agg >= 2 * Vc) return;   // the whole wave; no barrier below
    const int slab = (int)(unit - agg * slabs);
    const int64_t xc = agg >> 1;
    const int chi = (int)(agg & 1);
    const int half = dof >> 1, rows = bsites * half;
    const int r0 = (int)((int64_t)rows * slab / slabs), n = (int)((int64_t)rows * (slab + 1) / slabs) - r0;
    int64_t* at = places + w * kProlongRows;
    for (int e = l; e < n; e += 64) {
        const int site = (r0 + e) / half;
        at[e] = (int64_t)members[xc * bsites + site] * dof + chi * half + (r0 + e - site * half);
    }
    const int gpr = (nvec + E - 1) / E;        // runs of a row, lanes next to each other
    const int rpw = 64 / gpr;                  // rows of a turn
    const int lr = l / gpr, q = l - lr * gpr;
    const bool mine = lr < rpw;
    cpx<R> u[E];
    {
        const cpx<R>* c = uc + ((int64_t)blockIdx.y * Vc + xc) * 2 * nvec + chi * nvec;
#pragma unroll
        for (int i = 0; i < E; ++i) u[i] = FULL || E * q + i < nvec ? c[E * q + i] : cpx<R>{0, 0};
    }
    out += (int64_t)blockIdx.y * V * dof;
    wave_lds_sync();
    // a row past the end is the last one again, not stored
    auto load = [&](BT (&b)[E], int r) {
        const BT* p = B + at[mine && r < n ? r : n - 1] * nvec;
#pragma unroll
        for (int i = 0; i < E; i += P) {
            const bool ok = FULL || E * q + i < nvec;
            ld_entries<false, P>(b + i, p + (ok ? E * q + i : 0));
            if (!ok)
#pragma unroll
                for (int k = 0; k < P; ++k) b[i + k] = BT{};
        }
    };
    auto row = [&](const BT (&b)[E], int r) {
        const cpx<R> v = run_sum<L / 2, 4, D, R>(b, u);
        cpx<R> sum = v;
        for (int k = 1; k < gpr; ++k) {
            sum.re += __shfl(v.re, (l + k) & 63, 64);
            sum.im += __shfl(v.im, (l + k) & 63, 64);
        }
        if (mine && q == 0 && r < n) out[at[r]] = sum;
    };
    BT b0[E], b1[E];
    load(b0, lr);
    for (int r = lr, k = 0; k < n; r += 2 * rpw, k += 2 * rpw) {   // every lane takes the same number of turns
        load(b1, r + rpw);
        row(b0, r);
        load(b0, r + 2 * rpw);
        row(b1, r + rpw);
    }
}

// The same where nvec is at most L: a thread per row, in lattice order, four
// rows of a thread in flight, the members one after another.
template <typename R, typename BT, int L, int D, int P>
__global__ __launch_bounds__(256) void k_prolong_few(cpx<R>* __restrict__ out, const BT* __restrict__ B,
                                                     const cpx<R>* __restrict__ uc, const int* __restrict__ owner,
                                                     int dof, int nvec, int64_t V, int64_t Vc, int nb) {
    constexpr int U = 4;
    const int64_t rows = V * dof, r0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
    BT b[U][L];
    int64_t c[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int64_t r = r0 + 256 * j < rows ? r0 + 256 * j : rows - 1;
        const int64_t x = r / dof;
        const int chi = (int)(r - x * dof) >= (dof >> 1);
        c[j] = ((int64_t)owner[x] * 2 + chi) * nvec;
#pragma unroll
        for (int i = 0; i < L; i += P) {
            const bool ok = i < nvec;   // P divides nvec
            ld_entries<false, P>(&b[j][i], B + r * nvec + (ok ? i : 0));
            if (!ok)
#pragma unroll
                for (int k = 0; k < P; ++k) b[j][i + k] = BT{};
        }
    }
    for (int m = 0; m < nb; ++m, uc += Vc * 2 * nvec, out += rows) {
        cpx<R> u[U][L];
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int i = 0; i < L; ++i) u[j][i] = i < nvec ? uc[c[j] + i] : cpx<R>{0, 0};
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const cpx<R> v = run_sum<L / 2, 2, D, R>(b[j], u[j]);
            if (r0 + 256 * j < rows) out[r0 + 256 * j] = v;
        }
    }
}

// Restriction: the sums of the chunks of 16 rows, one thread per chunk and P
// vectors, go to LDS and are then added in the order of the waves of the form
// above.  A work-group first puts the field and the place of every row it takes
// into LDS (read by the threads where they use them, the lines of the fields and
// of the site lists push those of the basis out of the L1: FP16 nvec 24, with
// non-temporal loads, 42 us against 38).  It takes M (aggregate, chirality) units
// where one has few chunks, and G chunks of a unit at a time where all do not fit
// LDS (then a multiple of 8, and M = 1).  half_rec: ceil(2^32 / half); V dof fits
// an int, bsites half^2 32 bits.
template <typename R, typename BT, int P, bool NT>
__global__ __launch_bounds__(256) void k_restrict_vec(cpx<R>* __restrict__ out, const BT* __restrict__ B,
                                                      const cpx<R>* __restrict__ in, const int* __restrict__ members,
                                                      int dof, int nvec, int bsites, int64_t V, int64_t Vc, int G, int M,
                                                      uint32_t half_rec) {
    struct Sum { R rr, ii, ri, ir; };
    extern __shared__ __align__(16) unsigned char smem[];
    const int half = dof >> 1, rows = bsites * half, nch = (rows + 15) >> 4;
    const bool one = nch <= G;                  // all chunks at once
    Sum* part = reinterpret_cast<Sum*>(smem);   // [M][G][nvec]
    Sum* tot = one ? part : part + G * nvec;    // the eight totals of a unit: in place, or carried
    cpx<R>* fld = reinterpret_cast<cpx<R>*>(part + (M * G + (one ? 0 : 8)) * nvec);   // [M][G][17]
    int* at = reinterpret_cast<int*>(fld + M * G * 17);                                // [M][G][17]
    const int tid = threadIdx.x;
    constexpr int T = 256;
    int64_t unit0 = (int64_t)blockIdx.x * M;
    if (M == 1) {                  // the two chiralities of an aggregate on one XCD, as above
        int chi;
        const int64_t xc = agg_of(blockIdx.x, Vc, chi);
        unit0 = xc < 0 ? 2 * Vc : 2 * xc + chi;
    }
    if (unit0 >= 2 * Vc) return;   // the whole work-group
    const int mu = (int)(2 * Vc - unit0 < M ? 2 * Vc - unit0 : M);
    const int cpr = nvec / P;
    const int nv = nch < 8 ? nch : 8;
    in += (int64_t)blockIdx.y * V * dof;
    for (int c0 = 0; c0 < nch; c0 += G) {
        const int ng = nch - c0 < G ? nch - c0 : G;
        for (int e0 = tid; e0 < mu * 16 * ng; e0 += T) {
            const int m = e0 / (16 * ng), e = e0 - m * 16 * ng;
            const int64_t unit = unit0 + m;
            const int r = 16 * c0 + e < rows ? 16 * c0 + e : rows - 1;   // past the end the last row, not used
            const int site = half == 1 ? r : (int)__umulhi((uint32_t)r, half_rec);
            const int x = members[(unit >> 1) * bsites + site] * dof + (int)(unit & 1) * half + (r - site * half);
            at[(m * G + (e >> 4)) * 17 + (e & 15)] = x;
            fld[(m * G + (e >> 4)) * 17 + (e & 15)] = in[x];
        }
        __syncthreads();
        const int items = ng * cpr;
        for (int it = tid; it < mu * items; it += T) {
            const int m = it / items, j = it - m * items;
            const int cl = j / cpr, k0 = (j - cl * cpr) * P;
            const int left = rows - 16 * (c0 + cl);      // rows of the chunk, 16 or more if whole
            const int* a16 = at + (m * G + cl) * 17;
            const cpx<R>* f16 = fld + (m * G + cl) * 17;
            BT b[16][P];
#pragma unroll
            for (int r = 0; r < 16; ++r) ld_entries<NT, P>(b[r], B + (int64_t)a16[r] * nvec + k0);
            Sum a[P];
#pragma unroll
            for (int i = 0; i < P; ++i) a[i] = Sum{0, 0, 0, 0};
            __builtin_amdgcn_sched_barrier(0);   // all loads first
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const cpx<R> fv = r < left ? f16[r] : cpx<R>{0, 0};
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const cpx<R> wv = bval<R>(r < left ? b[r][i] : BT{});
                    a[i].rr = fma_r(wv.re, fv.re, a[i].rr);
                    a[i].ii = fma_r(wv.im, fv.im, a[i].ii);
                    a[i].ri = fma_r(wv.re, fv.im, a[i].ri);
                    a[i].ir = fma_r(wv.im, fv.re, a[i].ir);
                }
                if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // else every entry is decoded before the first product
            }
#pragma unroll
            for (int i = 0; i < P; ++i) part[(m * G + cl) * nvec + k0 + i] = a[i];
        }
        __syncthreads();
        if (nch > 8) {
            for (int o = tid; o < mu * 8 * nvec; o += T) {
                const int m = o / (8 * nvec), vk = o - m * 8 * nvec;   // (class, vector)
                Sum t = c0 ? tot[vk] : Sum{0, 0, 0, 0};
                for (int e = vk; e < ng * nvec; e += 8 * nvec) {
                    const Sum p = part[m * G * nvec + e];
                    t = Sum{t.rr + p.rr, t.ii + p.ii, t.ri + p.ri, t.ir + p.ir};
                }
                tot[m * G * nvec + vk] = t;   // (M = 1 unless in place)
            }
            __syncthreads();
        }
    }
    for (int o = tid; o < mu * nvec; o += T) {
        const int m = o / nvec, k = o - m * nvec;
        R re = 0, im = 0;
        for (int v = 0; v < nv; ++v) {
            const Sum t = tot[(m * G + v) * nvec + k];
            re += t.rr + t.ii;
            im += t.ri - t.ir;
        }
        out[((int64_t)blockIdx.y * 2 * Vc + unit0 + m) * nvec + k] = cpx<R>{re, im};
    }
}

}  // namespace qmg

using namespace qmg;

extern "C" void qmg_transfer_destroy(qmg_transfer t) {
    if (!t) return;
    if (t->basis && t->basis != (void*)t->basis64) (void)hipFree(t->basis);
    if (t->basis64) (void)hipFree(t->basis64);
    if (t->members) (void)hipFree(t->members);
    if (t->owner) (void)hipFree(t->owner);
    delete t;
}

namespace {

// Validation, aggregate tables and the FP64 basis buffer shared by
// qmg_transfer_create and qmg_transfer_import; `what` prefixes the messages.
qmg_status transfer_shell(const char* what, const int fine_dims[4], int fine_dof, const int block[4], int nvec,
                          const void* vecs, qmg_prec storage, hipStream_t s, qmg_transfer_s** out) {
    QMG_TRY(check_dims(fine_dims, 2, what));
    if (!block || !vecs) return fail(QMG_ERR_ARG, "%s: NULL argument", what);
    if (fine_dof < 2 || (fine_dof & 1) || fine_dof > 128)
        return fail(QMG_ERR_SHAPE, "%s: fine_dof %d must be even in [2,128]", what, fine_dof);
    if (nvec < 1 || 2 * nvec > 128) return fail(QMG_ERR_SHAPE, "%s: nvec %d outside [1,64]", what, nvec);
    if (storage != QMG_C128 && storage != QMG_C64 && storage != QMG_H16)
        return fail(QMG_ERR_PREC, "%s: storage %d not supported", what, (int)storage);
    int cd[4];
    int64_t bs = 1;
    for (int m = 0; m < 4; ++m) {
        if (block[m] < 1 || fine_dims[m] % block[m])
            return fail(QMG_ERR_SHAPE, "%s: block %d does not divide extent %d (dim %d)", what, block[m],
                        fine_dims[m], m);
        cd[m] = fine_dims[m] / block[m];
        if (cd[m] < 2) return fail(QMG_ERR_SHAPE, "%s: coarse extent %d < 2 in dim %d", what, cd[m], m);
        bs *= block[m];
    }
    if ((int64_t)nvec > bs * (fine_dof / 2))
        return fail(QMG_ERR_SHAPE, "%s: nvec %d exceeds aggregate dimension %lld", what, nvec,
                    (long long)(bs * (fine_dof / 2)));
    auto* t = new qmg_transfer_s();
    for (int m = 0; m < 4; ++m) { t->fdims[m] = fine_dims[m]; t->block[m] = block[m]; t->cdims[m] = cd[m]; }
    t->V = volume(fine_dims);
    t->Vc = volume(cd);
    t->dof = fine_dof;
    t->nvec = nvec;
    t->bsites = (int)bs;
    t->storage = storage;

    // aggregate tables on the host
    std::vector<int> members(t->V), owner(t->V), fill(t->Vc, 0);
    for (int64_t i = 0; i < t->V; ++i) {
        int64_t r = i;
        int x[4];
        for (int m = 0; m < 4; ++m) { x[m] = (int)(r % fine_dims[m]); r /= fine_dims[m]; }
        const int64_t xc = x[0] / block[0] + (int64_t)cd[0] * (x[1] / block[1] + (int64_t)cd[1] * (x[2] / block[2] + (int64_t)cd[2] * (x[3] / block[3])));
        owner[i] = (int)xc;
        members[xc * bs + fill[xc]++] = (int)i;
    }
    const size_t nb = (size_t)t->V * fine_dof * nvec;
    hipError_t e = hipMalloc(&t->members, sizeof(int) * t->V);
    if (e == hipSuccess) e = hipMalloc(&t->owner, sizeof(int) * t->V);
    if (e == hipSuccess) e = hipMalloc(&t->basis64, sizeof(double2) * nb);
    if (e == hipSuccess) e = hipMemcpyAsync(t->members, members.data(), sizeof(int) * t->V, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(t->owner, owner.data(), sizeof(int) * t->V, hipMemcpyHostToDevice, s);
    // the host tables are released on return: the copies must have landed
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        qmg_transfer_destroy(t);
        return fail(e == hipErrorOutOfMemory ? QMG_ERR_NOMEM : QMG_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
    }
    *out = t;
    return QMG_OK;
}

// The storage-precision copy of the FP64 basis (the same buffer for QMG_C128).
qmg_status transfer_finish(const char* what, qmg_transfer_s* t, hipStream_t s) {
    const size_t nb = (size_t)t->V * t->dof * t->nvec;
    if (t->storage == QMG_C128) {
        t->basis = t->basis64;
        return QMG_OK;
    }
    const bool h16 = t->storage == QMG_H16;
    const hipError_t e = hipMalloc(&t->basis, (h16 ? sizeof(uint32_t) : sizeof(float2)) * nb);
    if (e != hipSuccess) return fail(QMG_ERR_NOMEM, "%s: %s", what, hipGetErrorString(e));
    if (h16) {
        unsigned* nf = nullptr;
        QMG_TRY(nonfinite_flag(&nf));
        hipLaunchKernelGGL(k_to_h16, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, (uint32_t*)t->basis,
                           t->basis64, (int64_t)nb, nf);
        QMG_LAUNCH_CHECK();
        return take_nonfinite(s, what);
    } else
        hipLaunchKernelGGL(k_to_c64, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, (float2*)t->basis,
                           t->basis64, (int64_t)nb);
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}

}  // namespace

extern "C" qmg_status qmg_transfer_create(const int fine_dims[4], int fine_dof, const int block[4],
                                          int nvec, const void* nullvecs, qmg_prec storage,
                                          void* stream, qmg_transfer* out) {
    if (!out) return fail(QMG_ERR_ARG, "transfer_create: out is NULL");
    *out = nullptr;
    hipStream_t s = as_stream(stream);
    qmg_transfer_s* t = nullptr;
    QMG_TRY(transfer_shell("transfer_create", fine_dims, fine_dof, block, nvec, nullvecs, storage, s, &t));
    const int64_t Lb = (int64_t)t->bsites * (fine_dof / 2);
    const size_t wbytes = sizeof(double2) * (size_t)t->Vc * 2 * nvec * Lb;
    double2* W = nullptr;
    int* flag = nullptr;
    hipError_t e = hipMalloc(&W, wbytes);
    if (e == hipSuccess) e = hipMalloc(&flag, sizeof(int));
    if (e == hipSuccess) e = hipMemsetAsync(flag, 0, sizeof(int), s);
    if (e != hipSuccess) {
        if (W) (void)hipFree(W);
        if (flag) (void)hipFree(flag);
        qmg_transfer_destroy(t);
        return fail(e == hipErrorOutOfMemory ? QMG_ERR_NOMEM : QMG_ERR_HIP, "transfer_create: %s", hipGetErrorString(e));
    }
    const int64_t total = t->Vc * 2 * nvec * Lb;
    const unsigned g1 = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(k_gather_blocks, dim3(g1), dim3(256), 0, s, W, (const double2*)nullvecs, t->members,
                       t->V, t->Vc, fine_dof, nvec, t->bsites);
    hipLaunchKernelGGL(k_block_mgs, dim3((unsigned)(t->Vc * 2)), dim3(256), 0, s, W, nvec, Lb, 1e-10, flag);
    hipLaunchKernelGGL(k_scatter_basis, dim3(g1), dim3(256), 0, s, t->basis64, W, t->members, t->Vc,
                       fine_dof, nvec, t->bsites);
    e = hipGetLastError();
    int hflag = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(W);
    (void)hipFree(flag);
    if (e != hipSuccess) {
        qmg_transfer_destroy(t);
        return fail(QMG_ERR_HIP, "transfer_create: %s", hipGetErrorString(e));
    }
    if (hflag) {
        qmg_transfer_destroy(t);
        return fail(QMG_ERR_ARG, "transfer_create: near-null vectors are linearly dependent within an aggregate");
    }
    const qmg_status st = transfer_finish("transfer_create", t, s);
    if (st != QMG_OK) {
        qmg_transfer_destroy(t);
        return st;
    }
    *out = t;
    return QMG_OK;
}

extern "C" qmg_status qmg_transfer_import(const int fine_dims[4], int fine_dof, const int block[4], int nvec,
                                          const void* basis, qmg_prec storage, void* stream, qmg_transfer* out) {
    if (!out) return fail(QMG_ERR_ARG, "transfer_import: out is NULL");
    *out = nullptr;
    hipStream_t s = as_stream(stream);
    qmg_transfer_s* t = nullptr;
    QMG_TRY(transfer_shell("transfer_import", fine_dims, fine_dof, block, nvec, basis, storage, s, &t));
    qmg_status st = QMG_OK;
    if (hipMemcpyAsync(t->basis64, basis, sizeof(double2) * (size_t)t->V * fine_dof * nvec, hipMemcpyDeviceToDevice,
                       s) != hipSuccess)
        st = fail(QMG_ERR_HIP, "transfer_import: basis copy failed");
    if (st == QMG_OK) st = transfer_finish("transfer_import", t, s);
    if (st == QMG_OK && hipStreamSynchronize(s) != hipSuccess) st = fail(QMG_ERR_HIP, "transfer_import: sync");
    if (st != QMG_OK) {
        qmg_transfer_destroy(t);
        return st;
    }
    *out = t;
    return QMG_OK;
}

extern "C" qmg_status qmg_transfer_coarse_dims(qmg_transfer t, int cdims[4], int* N) {
    if (!t || !cdims || !N) return fail(QMG_ERR_ARG, "transfer_coarse_dims: NULL argument");
    for (int m = 0; m < 4; ++m) cdims[m] = t->cdims[m];
    *N = 2 * t->nvec;
    return QMG_OK;
}

extern "C" qmg_status qmg_transfer_export(qmg_transfer t, void* basis, void* stream) {
    if (!t || !basis) return fail(QMG_ERR_ARG, "transfer_export: NULL argument");
    QMG_HIP(hipMemcpyAsync(basis, t->basis64, sizeof(double2) * (size_t)t->V * t->dof * t->nvec,
                           hipMemcpyDeviceToDevice, as_stream(stream)));
    return QMG_OK;
}

namespace qmg {
template <typename R, typename ST, int KS, int L, int D, int NT>
static void prolong_nt(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    const int tiles = (t->bsites * (t->dof / 2) + 15) / 16;
    // work-groups per (aggregate, chirality): at most kProlongTiles tiles each,
    // fewer (but one per wave) where that leaves the chip without 2048 of them
    int64_t slabs = (tiles + kProlongTiles<R> - 1) / kProlongTiles<R>;
    const int64_t fill = (2048 + 2 * t->Vc - 1) / (2 * t->Vc);
    if (slabs < fill) slabs = fill < (tiles + 3) / 4 ? fill : (tiles + 3) / 4;
    const dim3 grid((unsigned)agg_grid(t->Vc), (unsigned)((nb + 8 * NT - 1) / (8 * NT)), (unsigned)slabs);
    // the rows of a pair share a site, and pairs start at even components
    const int wide = (t->dof / 2) % 2 == 0 && (uintptr_t)out % 16 == 0;
    if (2 * t->nvec == 4 * KS)
        hipLaunchKernelGGL((k_prolong<R, ST, KS, L, D, NT, true>), grid, dim3(256), 0, s, (cpx<R>*)out, (const ST*)B,
                           (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, t->V, t->Vc, nb, wide);
    else
        hipLaunchKernelGGL((k_prolong<R, ST, KS, L, D, NT, false>), grid, dim3(256), 0, s, (cpx<R>*)out, (const ST*)B,
                           (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, t->V, t->Vc, nb, wide);
}

template <typename R, typename BT, int L, int D, int P, bool FULL>
static void prolong_vec_t(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    const int gpr = (t->nvec + 2 * L - 1) / (2 * L), rows = t->bsites * (t->dof / 2);
    const int per = 4 * (64 / gpr);   // rows of a slab: four turns of a wave
    const int64_t slabs = (rows + per - 1) / per;
    const dim3 grid((unsigned)((2 * t->Vc * slabs + 3) / 4), (unsigned)nb);
    hipLaunchKernelGGL((k_prolong_vec<R, BT, L, D, P, FULL>), grid, dim3(256), 0, s, (cpx<R>*)out, (const BT*)B,
                       (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, t->V, t->Vc, (int)slabs);
}

// The forms of the prolongation for one shape of its sums (KS columns per lane
// group in runs of L, D).
template <typename R, typename ST, int KS, int L, int D>
static void prolong_form(qmg_transfer t, const void* B, const void* in, void* out, int nb, bool vec, hipStream_t s) {
    if (!vec) {
        // column tiles per wave: the coarse operand takes KS x NT registers
        if (nb <= 8) return prolong_nt<R, ST, KS, L, D, 1>(t, B, in, out, nb, s);
        if constexpr (KS * sizeof(R) <= (D > 1 ? 64 : 32))
            if (nb > 16) return prolong_nt<R, ST, KS, L, D, 4>(t, B, in, out, nb, s);
        return prolong_nt<R, ST, KS, L, D, 2>(t, B, in, out, nb, s);
    }
    using BT = std::conditional_t<sizeof(ST) == 2, uint32_t, cpx<R>>;
    constexpr int most = 16 / sizeof(BT);   // entries of a 16-byte load
    const int nv = t->nvec;
    if constexpr (KS == 4)
        if (nv <= L) {
            auto go = [&](auto p) {
                hipLaunchKernelGGL((k_prolong_few<R, BT, L, D, decltype(p)::value>),
                                   dim3((unsigned)((t->V * t->dof + 1023) / 1024)), dim3(256), 0, s, (cpx<R>*)out, (const BT*)B,
                                   (const cpx<R>*)in, t->owner, t->dof, nv, t->V, t->Vc, nb);
            };
            return nv == L ? go(std::integral_constant<int, most < L ? most : L>{}) : go(std::integral_constant<int, 1>{});
        }
    if (nv % (2 * L) == 0) return prolong_vec_t<R, BT, L, D, most, true>(t, B, in, out, nb, s);
    if (nv % most == 0) return prolong_vec_t<R, BT, L, D, most, false>(t, B, in, out, nb, s);
    if constexpr (most > 2)
        if (nv % 2 == 0) return prolong_vec_t<R, BT, L, D, 2, false>(t, B, in, out, nb, s);
    if constexpr (most > 1) prolong_vec_t<R, BT, L, D, 1, false>(t, B, in, out, nb, s);
}

// The shape of the sums is a function of the number of vectors and of the
// storage alone.  A run is 16 bytes of a lane group's row where its columns
// divide so (FP16: from 25 vectors on).  D, the products in one chain, is as
// large (faster, fewer registers) as leaves the error no larger than that of one
// chain per two entries (FP32; FP16 up to four, FP64 one) and these chains added
// in order.  The squared error of that order, in units of one rounding of the
// result, and of two and one product: FP32 nvec 6 4.2, 4.5 and 4.0; 8 4.8, 5.5
// and 4.5; 10 5.3, 5.9 and 5.2; 12 5.8 and 5.8; 24 8.9 and 7.2; 32 10.9 and 7.8.
template <typename R, typename ST>
static qmg_status prolong_t(qmg_transfer t, const void* B, const void* in, void* out, int nb, bool vec, hipStream_t s) {
    const int nv = t->nvec;
    constexpr bool f64 = sizeof(ST) == 8;
    constexpr int L = f64 ? 2 : 4, LW = sizeof(ST) == 2 ? 8 : L;
    if (!f64 && nv <= 2) prolong_form<R, ST, 4, L, f64 ? 2 : 4>(t, B, in, out, nb, vec, s);
    else if (f64 ? nv >= 2 && nv <= 5 : nv == 6 || nv == 8) prolong_form<R, ST, 4, L, 1>(t, B, in, out, nb, vec, s);
    else if (nv <= 8) prolong_form<R, ST, 4, L, 2>(t, B, in, out, nb, vec, s);
    else if (!f64 && nv == 10) prolong_form<R, ST, 8, L, f64 ? 2 : 1>(t, B, in, out, nb, vec, s);
    else if (nv <= 16) prolong_form<R, ST, 8, L, 2>(t, B, in, out, nb, vec, s);
    else if (nv <= 24) prolong_form<R, ST, 12, L, 2>(t, B, in, out, nb, vec, s);
    else if (nv <= 32) prolong_form<R, ST, 16, LW, 2>(t, B, in, out, nb, vec, s);
    else prolong_form<R, ST, 32, LW, 2>(t, B, in, out, nb, vec, s);
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}

template <typename R, typename ST, int T, int NT>
static void restrict_nt(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    // the split of the rows is not a function of the number of members, which keep one order of summation
    const size_t lds = sizeof(R) * kRestrictWaves * 16 * std::max(restrict_ld(NT), 16 * T);
    const dim3 grid((unsigned)agg_grid(t->Vc), (unsigned)((nb + 8 * NT - 1) / (8 * NT)), (unsigned)((t->nvec + 31) / 32));
    if (t->nvec == 8 * T)
        hipLaunchKernelGGL((k_restrict<R, ST, T, NT, true>), grid, dim3(64 * kRestrictWaves), lds, s, (cpx<R>*)out,
                           (const ST*)B, (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, t->V, t->Vc, nb);
    else
        hipLaunchKernelGGL((k_restrict<R, ST, T, NT, false>), grid, dim3(64 * kRestrictWaves), lds, s, (cpx<R>*)out,
                           (const ST*)B, (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, t->V, t->Vc, nb);
}

template <typename R, typename ST, int T>
static void restrict_tt(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    if (nb <= 8) return restrict_nt<R, ST, T, 1>(t, B, in, out, nb, s);
    if constexpr (sizeof(R) == 4)
        if (nb > 16) return restrict_nt<R, ST, T, 4>(t, B, in, out, nb, s);
    restrict_nt<R, ST, T, 2>(t, B, in, out, nb, s);
}

template <typename R, typename ST>
static qmg_status restrict_t(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    const int nv = t->nvec;
    if (nv <= 8) restrict_tt<R, ST, 1>(t, B, in, out, nb, s);
    else if (nv <= 16) restrict_tt<R, ST, 2>(t, B, in, out, nb, s);
    else if (nv <= 24) restrict_tt<R, ST, 3>(t, B, in, out, nb, s);
    else restrict_tt<R, ST, 4>(t, B, in, out, nb, s);
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}

template <typename R, typename BT, int P, bool NT>
static qmg_status restrict_vec_t(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    const int half = t->dof / 2, nch = (t->bsites * half + 15) / 16, cpr = t->nvec / P;
    const int sums = (int)(4 * sizeof(R)) * t->nvec, chunk = sums + 17 * (int)(sizeof(cpx<R>) + sizeof(int));   // LDS bytes
    constexpr int budget = 32768;   // of LDS: five work-groups on a CU (four: 32^3x64, nvec 24, FP16 434 us against 426)
    int G = nch, M = 1;
    if (nch <= budget / chunk) {    // units that give every thread a chunk and P vectors
        M = std::max(1, std::min(budget / chunk / nch, 256 / (nch * cpr)));
    } else {
        const int fit = std::max(8, (budget - 8 * sums) / chunk / 8 * 8);
        const int passes = (nch + fit - 1) / fit;
        G = ((nch + passes - 1) / passes + 7) / 8 * 8;
    }
    const size_t lds = (size_t)chunk * G * M + (G < nch ? 8 * sums : 0);
    const dim3 grid((unsigned)(M == 1 ? agg_grid(t->Vc) : (2 * t->Vc + M - 1) / M), (unsigned)nb);
    hipLaunchKernelGGL((k_restrict_vec<R, BT, P, NT>), grid, dim3(256), lds, s, (cpx<R>*)out, (const BT*)B,
                       (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, t->V, t->Vc, G, M,
                       (uint32_t)((0x100000000ull + half - 1) / half));
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}
template <typename R, typename BT, int P>
static qmg_status restrict_vec(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    // Non-temporal loads of a basis that the last-level cache (256 MB) does not hold, where rows neither share a
    // 64-byte sector nor are shorter than a cache line (one member, 4^4 blocks, with and without: 24^3x48 FP32 16
    // vectors 159 and 181 us, 24 246 and 268; 16^3x32 FP32 32, 403 MB, 65 and 75).  Elsewhere the cache serves what
    // it holds, to repeated calls (8^3x16 FP32 24 16.1 and 12.4 us) and to the prolongation after this one (in a
    // solve on 16^3x32, FP32 24, 302 MB: restriction 57 and 68 us, prolongation 72 and 53); and sectors that rows
    // share would be fetched again (24^3x48 FP32 20, 160 bytes, 246 and 221 us, FP16 24, 96 bytes, 176 and 145).
    const int row = t->nvec * (int)sizeof(BT);
    return row >= 128 && row % 64 == 0 && t->V * t->dof * row > 320000000 ? restrict_vec_t<R, BT, P, true>(t, B, in, out, nb, s)
                                                                          : restrict_vec_t<R, BT, P, false>(t, B, in, out, nb, s);
}

// One member goes to the vector unit, as do up to four with so few vectors that a
// thread holds a row: 16^3x32, FP32, prolongation on the vector unit / the matrix
// cores in us, nvec 24: one member 55 / 62, two 104 / 68; nvec 4: two 17 / 25, four
// 25 / 27, six 32 / 30.
static bool prolong_on_vector_unit(bool f64, int nvec, int nb) { return nb == 1 || (nb <= 4 && nvec <= (f64 ? 2 : 4)); }
// One member, and two with at most four vectors: restriction, FP32, nvec 24: one
// member 51 / 57, two 99 / 53; nvec 4: two 26 / 29, three 37 / 29.
// (The bounds: a row's place is kept as an int, and its site is found by a
// product with ceil(2^32 / half), exact while rows x half stays below 2^32.)
static bool restrict_on_vector_unit(const qmg_transfer_s* t, int nb) {
    const int64_t half = t->dof / 2;
    return (nb == 1 || (nb == 2 && t->nvec <= 4)) && t->V * t->dof <= INT32_MAX && t->bsites * half * half <= UINT32_MAX;
}

qmg_status transfer_prolong(qmg_transfer t, const void* in, void* out, qmg_prec p, int nb, hipStream_t s) {
    const bool vec = prolong_on_vector_unit(p == QMG_C128, t->nvec, nb);
    if (p == QMG_C128) return prolong_t<double, double>(t, t->basis64, in, out, nb, vec, s);
    if (t->storage == QMG_H16) return prolong_t<float, _Float16>(t, t->basis, in, out, nb, vec, s);
    return prolong_t<float, float>(t, t->basis, in, out, nb, vec, s);
}

qmg_status transfer_restrict(qmg_transfer t, const void* in, void* out, qmg_prec p, int nb, hipStream_t s) {
    const bool h16 = t->storage == QMG_H16;
    if (restrict_on_vector_unit(t, nb)) {
        const int nv = t->nvec;
        if (p == QMG_C128) return restrict_vec<double, cpx<double>, 1>(t, t->basis64, in, out, nb, s);
        if (h16 && nv % 2 == 0) return restrict_vec<float, uint32_t, 2>(t, t->basis, in, out, nb, s);
        if (h16) return restrict_vec<float, uint32_t, 1>(t, t->basis, in, out, nb, s);
        if (nv % 2 == 0) return restrict_vec<float, cpx<float>, 2>(t, t->basis, in, out, nb, s);
        return restrict_vec<float, cpx<float>, 1>(t, t->basis, in, out, nb, s);
    }
    if (p == QMG_C128) return restrict_t<double, double>(t, t->basis64, in, out, nb, s);
    if (h16) return restrict_t<float, _Float16>(t, t->basis, in, out, nb, s);
    return restrict_t<float, float>(t, t->basis, in, out, nb, s);
}
}  // namespace qmg

static qmg_status check_transfer_prec(qmg_transfer t, qmg_prec p, const char* what) {
    if (p != QMG_C128 && p != QMG_C64) return fail(QMG_ERR_PREC, "%s: precision %d not supported", what, (int)p);
    if (p == QMG_C64 && t->storage != QMG_C64 && t->storage != QMG_H16)
        return fail(QMG_ERR_PREC, "%s: complex64 fields need a transfer created with complex64 or FP16 storage", what);
    return QMG_OK;
}

extern "C" qmg_status qmg_prolong(qmg_transfer t, const void* coarse_in, void* fine_out, int nrhs, qmg_prec p,
                                  void* stream) {
    if (!t || !coarse_in || !fine_out) return fail(QMG_ERR_ARG, "prolong: NULL argument");
    if (nrhs < 1 || nrhs > kMaxFieldBatch) return fail(QMG_ERR_ARG, "prolong: nrhs %d not in [1, %d]", nrhs, kMaxFieldBatch);
    QMG_TRY(check_transfer_prec(t, p, "prolong"));
    return transfer_prolong(t, coarse_in, fine_out, p, nrhs, as_stream(stream));
}

extern "C" qmg_status qmg_restrict(qmg_transfer t, const void* fine_in, void* coarse_out, int nrhs, qmg_prec p,
                                   void* stream) {
    if (!t || !fine_in || !coarse_out) return fail(QMG_ERR_ARG, "restrict: NULL argument");
    if (nrhs < 1 || nrhs > kMaxFieldBatch) return fail(QMG_ERR_ARG, "restrict: nrhs %d not in [1, %d]", nrhs, kMaxFieldBatch);
    QMG_TRY(check_transfer_prec(t, p, "restrict"));
    return transfer_restrict(t, fine_in, coarse_out, p, nrhs, as_stream(stream));
}
