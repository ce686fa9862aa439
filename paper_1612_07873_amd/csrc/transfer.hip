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
// both as dense products per (aggregate, chirality) on the matrix cores, every
// sum in a fixed order: no atomics, bitwise repeatable.
// The basis is kept as [V][dof][Nvec] (row f of site x holds the Nvec
// coefficients of its chirality) in the storage precision, plus an FP64 copy
// for the Galerkin build.  The 16-bit storage keeps each complex entry as an
// FP16 pair with no scale: the columns are orthonormal within an aggregate,
// so no entry exceeds 1 in modulus.
#include "codes16.h"
#include "handles.h"

#include <algorithm>
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
// took 559 us (restriction) and 752 us (prolongation); these take 108 and 117.
// Every column of a product is summed in the same order whatever the number of
// members, so with a complex64 basis a member of a batch equals the single call
// bitwise.
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

// ------------------------------------------ one member, FP16 or FP64 basis
// A single field does not fill the matrix cores (2 of 16 columns).  With an
// FP16 basis (half the bytes) or in FP64 one thread per 16-byte chunk of the
// basis is faster there: 16^3x32, nvec 24, both directions, FP16 65 us against
// 85, FP64 230 against 248.  (With a complex64 basis 116 against 114: one form
// for every number of members.)  BT: the stored entry, cpx<double> or a 32-bit
// FP16 pair.
template <typename R> __device__ __forceinline__ cpx<R> bval(const cpx<R>& b) { return b; }
template <typename R> __device__ __forceinline__ cpx<R> bval(const uint32_t& w) { return dec_pair<FMT_H16>(w); }

// CPC consecutive basis entries, read once per application: non-temporal
// loads, so the basis stream does not push the fine vector being restricted
// out of the caches (the prolongation, which reads the small coarse vector,
// was slower with them and keeps plain loads).
template <typename BT, int CPC>
__device__ __forceinline__ void ld_basis(BT (&b)[CPC], const BT* p) {
    constexpr int words = (int)sizeof(BT) * CPC / 4;
    if constexpr (words == 1) {
        const int v = __builtin_nontemporal_load(reinterpret_cast<const int*>(p));
        __builtin_memcpy(b, &v, 4);
    } else {
        typedef int vec __attribute__((ext_vector_type(words)));
        static_assert(words == 2 || words == 4, "basis chunks of 4, 8 or 16 bytes");
        const vec v = __builtin_nontemporal_load(reinterpret_cast<const vec*>(p));
        __builtin_memcpy(b, &v, sizeof(v));
    }
}

// Prolongation: one thread per 16-byte chunk of the basis ([x][f][k] row
// major, so a wave reads one contiguous span).  A work-group covers RPT
// consecutive spans of rows_per_wg rows; each thread issues its RPT chunk
// loads before any arithmetic so that enough bytes are in flight to cover
// HBM latency.  The `cpr` chunks of a row (x, f) are then summed in LDS in a
// fixed order, one thread per row.
template <typename R, typename BT, int CPC, int RPT>
__global__ __launch_bounds__(256) void k_prolong_one(cpx<R>* __restrict__ out, const BT* __restrict__ B,
                                                 const cpx<R>* __restrict__ uc, const int* __restrict__ owner,
                                                 int64_t V, int dof, int nvec, int rows_per_wg) {
    constexpr int cpc = CPC;
    __shared__ cpx<R> part[RPT][256];
    const int cpr = nvec / cpc;                    // chunks per row
    const int t = threadIdx.x;
    const int lr = t / cpr, kc = t - (t / cpr) * cpr;
    const int64_t rows = V * dof;
    const int64_t base = (int64_t)blockIdx.x * rows_per_wg * RPT;
    BT b[RPT][cpc];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int64_t row = base + (int64_t)j * rows_per_wg + lr;
        if (lr < rows_per_wg && row < rows) {
#pragma unroll
            for (int q = 0; q < cpc; ++q) b[j][q] = B[row * nvec + kc * cpc + q];
        }
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int64_t row = base + (int64_t)j * rows_per_wg + lr;
        R ar = 0, ai = 0;
        if (lr < rows_per_wg && row < rows) {
            const int64_t x = row / dof;
            const int f = (int)(row - x * dof);
            const int chi = f / (dof / 2);
            const cpx<R>* u = uc + (int64_t)owner[x] * 2 * nvec + chi * nvec + kc * cpc;
#pragma unroll
            for (int q = 0; q < cpc; ++q) {
                const cpx<R> bq = bval<R>(b[j][q]);
                cmac(ar, ai, bq.re, bq.im, u[q].re, u[q].im);
            }
        }
        part[j][t] = cpx<R>{ar, ai};
    }
    __syncthreads();
    for (int rr = t; rr < rows_per_wg * RPT; rr += 256) {
        const int j = rr / rows_per_wg, r = rr - j * rows_per_wg;
        const int64_t row = base + rr;
        if (row < rows) {
            R sr = 0, si = 0;
            for (int q = 0; q < cpr; ++q) {
                sr += part[j][r * cpr + q].re;
                si += part[j][r * cpr + q].im;
            }
            out[row] = cpx<R>{sr, si};
        }
    }
}

// Restriction: one work-group per aggregate.  Thread (slice, q) owns chunk q
// of the per-site basis block (dof x nvec, contiguous) and accumulates
// conj(V) psi over the aggregate's sites slice, slice + S, ...; the S slices
// and then the dof/2 rows of each chirality are summed in LDS in a fixed
// order.  No atomics; bitwise repeatable.  With S = 1 the threads stride over
// the chunks instead (blocks with more chunks than threads).
template <typename R, typename BT, int CPC>
__global__ __launch_bounds__(1024) void k_restrict_one(cpx<R>* __restrict__ out, const BT* __restrict__ B,
                                                   const cpx<R>* __restrict__ in, const int* __restrict__ members,
                                                   int dof, int nvec, int bsites, int S) {
    constexpr int cpc = CPC;
    extern __shared__ __align__(16) unsigned char smem[];
    cpx<R>* acc_l = reinterpret_cast<cpx<R>*>(smem);   // [S][dof][nvec]
    const int64_t xc = blockIdx.x;
    const int* mem = members + xc * bsites;
    const int cpr = nvec / cpc;
    const int nchunk = dof * cpr;
    const int slice = S > 1 ? (int)threadIdx.x / nchunk : 0;
    const int q0 = S > 1 ? (int)threadIdx.x - slice * nchunk : (int)threadIdx.x;
    const int qstep = S > 1 ? nchunk : (int)blockDim.x;
    if (slice < S) {
        cpx<R>* acc_s = acc_l + (int64_t)slice * dof * nvec;
        for (int q = q0; q < nchunk; q += qstep) {
            const int f = q / cpr, kc = q - (q / cpr) * cpr;
            R ar[cpc], ai[cpc];
#pragma unroll
            for (int c = 0; c < cpc; ++c) ar[c] = ai[c] = 0;
            int b = slice;
            for (; b + 3 * S < bsites; b += 4 * S) {
                int64_t x[4];
                cpx<R> v[4];
                BT bb[4][cpc];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[j] = mem[b + j * S];
                    v[j] = in[x[j] * dof + f];
                    ld_basis<BT, cpc>(bb[j], B + (x[j] * dof + f) * nvec + kc * cpc);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < cpc; ++c) {
                        const cpx<R> bq = bval<R>(bb[j][c]);
                        cmac_conj(ar[c], ai[c], bq.re, bq.im, v[j].re, v[j].im);
                    }
            }
            for (; b < bsites; b += S) {
                const int64_t x = mem[b];
                const cpx<R> v = in[x * dof + f];
                BT bv[cpc];
                ld_basis<BT, cpc>(bv, B + (x * dof + f) * nvec + kc * cpc);
#pragma unroll
                for (int c = 0; c < cpc; ++c) {
                    const cpx<R> bq = bval<R>(bv[c]);
                    cmac_conj(ar[c], ai[c], bq.re, bq.im, v.re, v.im);
                }
            }
#pragma unroll
            for (int c = 0; c < cpc; ++c) acc_s[f * nvec + kc * cpc + c] = cpx<R>{ar[c], ai[c]};
        }
    }
    __syncthreads();
    const int half = dof / 2;
    const int64_t sstride = (int64_t)dof * nvec;
    for (int n = threadIdx.x; n < 2 * nvec; n += blockDim.x) {
        const int chi = n / nvec, k = n - chi * nvec;
        R sr = 0, si = 0;
        for (int ff = 0; ff < half; ++ff)
            for (int sl = 0; sl < S; ++sl) {
                const cpx<R> a = acc_l[sl * sstride + (chi * half + ff) * nvec + k];
                sr += a.re;
                si += a.im;
            }
        out[xc * 2 * nvec + n] = cpx<R>{sr, si};
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

// The prolongation for one shape of its sums (KS columns per lane group in runs
// of L, D).
template <typename R, typename ST, int KS, int L, int D>
static void prolong_form(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    // column tiles per wave: the coarse operand takes KS x NT registers
    if (nb <= 8) return prolong_nt<R, ST, KS, L, D, 1>(t, B, in, out, nb, s);
    if constexpr (KS * sizeof(R) <= (D > 1 ? 64 : 32))
        if (nb > 16) return prolong_nt<R, ST, KS, L, D, 4>(t, B, in, out, nb, s);
    prolong_nt<R, ST, KS, L, D, 2>(t, B, in, out, nb, s);
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
static qmg_status prolong_t(qmg_transfer t, const void* B, const void* in, void* out, int nb, hipStream_t s) {
    const int nv = t->nvec;
    constexpr bool f64 = sizeof(ST) == 8;
    constexpr int L = f64 ? 2 : 4, LW = sizeof(ST) == 2 ? 8 : L;
    if (!f64 && nv <= 2) prolong_form<R, ST, 4, L, f64 ? 2 : 4>(t, B, in, out, nb, s);
    else if (f64 ? nv >= 2 && nv <= 5 : nv == 6 || nv == 8) prolong_form<R, ST, 4, L, 1>(t, B, in, out, nb, s);
    else if (nv <= 8) prolong_form<R, ST, 4, L, 2>(t, B, in, out, nb, s);
    else if (!f64 && nv == 10) prolong_form<R, ST, 8, L, f64 ? 2 : 1>(t, B, in, out, nb, s);
    else if (nv <= 16) prolong_form<R, ST, 8, L, 2>(t, B, in, out, nb, s);
    else if (nv <= 24) prolong_form<R, ST, 12, L, 2>(t, B, in, out, nb, s);
    else if (nv <= 32) prolong_form<R, ST, 16, LW, 2>(t, B, in, out, nb, s);
    else prolong_form<R, ST, 32, LW, 2>(t, B, in, out, nb, s);
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

template <typename R, typename BT, int CPC>
static qmg_status prolong_one(qmg_transfer t, const void* B, const void* in, void* out, hipStream_t s) {
    constexpr int RPT = 4;
    const int cpr = t->nvec / CPC;
    const int rows_per_wg = 256 / cpr;
    const int64_t rows = t->V * t->dof;
    const int64_t per_wg = (int64_t)rows_per_wg * RPT;
    const unsigned nblk = (unsigned)((rows + per_wg - 1) / per_wg);
    hipLaunchKernelGGL((k_prolong_one<R, BT, CPC, RPT>), dim3(nblk), dim3(256), 0, s, (cpx<R>*)out, (const BT*)B,
                       (const cpx<R>*)in, t->owner, t->V, t->dof, t->nvec, rows_per_wg);
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}

template <typename R, typename BT, int CPC>
static qmg_status restrict_one(qmg_transfer t, const void* B, const void* in, void* out, hipStream_t s) {
    const int nchunk = t->dof * (t->nvec / CPC);
    const size_t lds1 = sizeof(cpx<R>) * t->dof * t->nvec;
    // site slices per aggregate: as many as fit in 1024 threads and 64 KiB of
    // LDS, at most 8 and at most the aggregate's sites
    int S = 1024 / nchunk;
    if (S > 8) S = 8;
    if (S > t->bsites) S = t->bsites;
    while (S > 1 && (size_t)S * lds1 > 65536) --S;
    if (S < 1) S = 1;
    int threads = S > 1 ? S * nchunk : nchunk;
    threads = ((threads + 63) / 64) * 64;
    if (threads > 1024) threads = 1024;
    const size_t lds = lds1 * S;
    if (lds > 65536)
        QMG_HIP(hipFuncSetAttribute((const void*)k_restrict_one<R, BT, CPC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    hipLaunchKernelGGL((k_restrict_one<R, BT, CPC>), dim3((unsigned)t->Vc), dim3(threads), lds, s, (cpx<R>*)out,
                       (const BT*)B, (const cpx<R>*)in, t->members, t->dof, t->nvec, t->bsites, S);
    QMG_LAUNCH_CHECK();
    return QMG_OK;
}

// one member in FP64 or with an FP16 basis (16-byte chunks of four pairs where
// nvec allows, else 8 or 4 bytes); every other call goes to the dense products
static bool one_member(qmg_transfer t, qmg_prec p, int nb) { return nb == 1 && (p == QMG_C128 || t->storage == QMG_H16); }

qmg_status transfer_prolong(qmg_transfer t, const void* in, void* out, qmg_prec p, int nb, hipStream_t s) {
    if (one_member(t, p, nb)) {
        if (p == QMG_C128) return prolong_one<double, cpx<double>, 1>(t, t->basis64, in, out, s);
        if (t->nvec % 4 == 0) return prolong_one<float, uint32_t, 4>(t, t->basis, in, out, s);
        if (t->nvec % 2 == 0) return prolong_one<float, uint32_t, 2>(t, t->basis, in, out, s);
        return prolong_one<float, uint32_t, 1>(t, t->basis, in, out, s);
    }
    if (p == QMG_C128) return prolong_t<double, double>(t, t->basis64, in, out, nb, s);
    if (t->storage == QMG_H16) return prolong_t<float, _Float16>(t, t->basis, in, out, nb, s);
    return prolong_t<float, float>(t, t->basis, in, out, nb, s);
}

qmg_status transfer_restrict(qmg_transfer t, const void* in, void* out, qmg_prec p, int nb, hipStream_t s) {
    if (one_member(t, p, nb)) {
        if (p == QMG_C128) return restrict_one<double, cpx<double>, 1>(t, t->basis64, in, out, s);
        if (t->nvec % 4 == 0) return restrict_one<float, uint32_t, 4>(t, t->basis, in, out, s);
        if (t->nvec % 2 == 0) return restrict_one<float, uint32_t, 2>(t, t->basis, in, out, s);
        return restrict_one<float, uint32_t, 1>(t, t->basis, in, out, s);
    }
    if (p == QMG_C128) return restrict_t<double, double>(t, t->basis64, in, out, nb, s);
    if (t->storage == QMG_H16) return restrict_t<float, _Float16>(t, t->basis, in, out, nb, s);
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
