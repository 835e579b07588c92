// HIP kernels (gfx950) of the black-box multigrid V-cycle: discretisation,
// set-up (operator-induced interpolation, Galerkin coarse operators, coarsest
// LDL^T factor) and the per-level cycle steps (four-colour Gauss-Seidel,
// residual, restriction, interpolation, norms).
//
// All floating-point expressions are written in one fixed order and the
// library is compiled with -ffp-contract=off, so every point's result is the
// correctly rounded value of that expression sequence (IEEE division
// included); schedules that respect the colour dependencies produce the same
// bits.
//
// Level arrays are (n+2) rows of `ld` elements, row j (north) after row j-1,
// element (i,j) at j*ld + i; rows/columns 0 and n+1 are the Dirichlet ring and
// hold zeros.  Stencils are symmetric-compact: O, W, S on every level plus SW,
// NW on nine-point levels; the east / north / north-east / south-east entries
// of point p are W(p+1), S(p+ld), SW(p+ld+1), NW(p+1-ld).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace bmg {

template <typename T>
struct Lev {
    int n;   // interior points per side
    int ld;  // row pitch (elements)
    T *u, *b, *r;
    T *O, *W, *S, *SW, *NW;  // SW, NW null on five-point levels
};

// Weights between a fine level and the next coarser one: 8 planes
// (LNE, LA, LNW, LR, LL, LSE, LB, LSW) of the coarse level's shape.
template <typename T>
struct Wts {
    T *p;
    int ld;       // coarse row pitch
    size_t ps;    // plane stride (elements)
    __device__ __forceinline__ T at(int plane, size_t c) const { return p[plane * ps + c]; }
};

enum : int { LNE = 0, LA = 1, LNW = 2, LR = 3, LL = 4, LSE = 5, LB = 6, LSW = 7 };

// validation / breakdown flag bits
enum : int {
    F_NONFINITE = 1, F_DIAG = 2, F_BOUNDARY = 4, F_ASYM = 8,
    F_BREAK_INTERP = 16, F_BREAK_COARSE = 32, F_BREAK_LINE = 64
};

__device__ __forceinline__ bool stopped(const int *stop) { return stop && *stop; }

// --------------------------------------------------------------- discretise
// Vertex-centred five-point operator of -div(k grad u) = f, cell-constant k:
// coupling = -(mean of the two cells sharing the grid edge), centre = minus the
// sum of the four couplings (before the boundary couplings are zeroed),
// right-hand side h^2 f.  Output [n][n][5] = S, W, O, E, N.
static __global__ void k_discretize(const double *__restrict__ k, const double *__restrict__ f,
                             int n, double h2, double *__restrict__ st,
                             double *__restrict__ rhs)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int j = blockIdx.y * blockDim.y + threadIdx.y + 1;
    if (i > n || j > n) return;
    const size_t lk = (size_t)n + 1;
    const double kSW = k[(size_t)(j - 1) * lk + (i - 1)];
    const double kSE = k[(size_t)(j - 1) * lk + i];
    const double kNW = k[(size_t)j * lk + (i - 1)];
    const double kNE = k[(size_t)j * lk + i];
    double aW = -0.5 * (kSW + kNW);
    double aE = -0.5 * (kSE + kNE);
    double aS = -0.5 * (kSW + kSE);
    double aN = -0.5 * (kNW + kNE);
    const double aO = -(((aW + aE) + aS) + aN);
    if (i == 1) aW = 0.0;
    if (i == n) aE = 0.0;
    if (j == 1) aS = 0.0;
    if (j == n) aN = 0.0;
    const size_t q = (size_t)(j - 1) * n + (i - 1);
    double *o = st + q * 5;
    o[0] = aS; o[1] = aW; o[2] = aO; o[3] = aE; o[4] = aN;
    rhs[q] = h2 * f[q];
}

// ------------------------------------------------------------ import stencil
__device__ __forceinline__ bool asym(double a, double b)
{
    const double d = fabs(a - b), m = fmax(fabs(a), fabs(b));
    return !(d <= 1e-14 * m);
}

// [n][n][K] user stencil -> compact level-0 planes, with validation.
static __global__ void k_import_stencil(const double *__restrict__ st, int K, Lev<double> L,
                                 int *__restrict__ flags)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int j = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int n = L.n;
    if (i > n || j > n) return;
    const size_t q = ((size_t)(j - 1) * n + (i - 1)) * K;
    const size_t p = (size_t)j * L.ld + i;
    int bad = 0;
    double e[9];
    // e[] in the order SW, S, SE, W, O, E, NW, N, NE
    if (K == 5) {
        e[0] = 0.0; e[1] = st[q + 0]; e[2] = 0.0; e[3] = st[q + 1]; e[4] = st[q + 2];
        e[5] = st[q + 3]; e[6] = 0.0; e[7] = st[q + 4]; e[8] = 0.0;
    } else {
#pragma unroll
        for (int t = 0; t < 9; ++t) e[t] = st[q + t];
    }
#pragma unroll
    for (int t = 0; t < 9; ++t)
        if (!isfinite(e[t])) bad |= F_NONFINITE;
    if (!(e[4] > 0.0)) bad |= F_DIAG;
    if (i == 1 && (e[0] != 0.0 || e[3] != 0.0 || e[6] != 0.0)) bad |= F_BOUNDARY;
    if (i == n && (e[2] != 0.0 || e[5] != 0.0 || e[8] != 0.0)) bad |= F_BOUNDARY;
    if (j == 1 && (e[0] != 0.0 || e[1] != 0.0 || e[2] != 0.0)) bad |= F_BOUNDARY;
    if (j == n && (e[6] != 0.0 || e[7] != 0.0 || e[8] != 0.0)) bad |= F_BOUNDARY;
    // symmetry against the neighbours' west / south / south-west / north-west
    if (i < n) {
        const size_t qe = q + K;
        if (asym(e[5], K == 5 ? st[qe + 1] : st[qe + 3])) bad |= F_ASYM;
    }
    if (j < n) {
        const size_t qn = q + (size_t)n * K;
        if (asym(e[7], K == 5 ? st[qn + 0] : st[qn + 1])) bad |= F_ASYM;
    }
    if (K == 9) {
        if (i < n && j < n && asym(e[8], st[q + ((size_t)n + 1) * K + 0])) bad |= F_ASYM;
        if (i < n && j > 1 && asym(e[2], st[q - ((size_t)n - 1) * K + 6])) bad |= F_ASYM;
    }
    L.O[p] = e[4];
    L.W[p] = e[3];
    L.S[p] = e[1];
    if (L.SW) {
        L.SW[p] = e[0];
        L.NW[p] = e[6];
    }
    if (bad) atomicOr(flags, bad);
}

// ------------------------------------------------- interpolation weights
// Row p of a compact stencil: SW, S, SE, W, O, E, NW, N, NE (a five-point
// stencil has no SW and NW planes: its corners are zero).
template <bool NINE>
__device__ __forceinline__ void row_of(const Lev<double> &L, size_t p, double a[9])
{
    const size_t ld = L.ld;
    a[0] = NINE ? L.SW[p] : 0.0;
    a[1] = L.S[p];
    a[2] = NINE ? L.NW[p + 1 - ld] : 0.0;
    a[3] = L.W[p];
    a[4] = L.O[p];
    a[5] = L.W[p + 1];
    a[6] = NINE ? L.NW[p] : 0.0;
    a[7] = L.S[p + ld];
    a[8] = NINE ? L.SW[p + ld + 1] : 0.0;
}

// Positive off-diagonals moved onto the diagonal (SW,S,SE,W,E,NW,N,NE order).
__device__ __forceinline__ void lump_row(double a[9])
{
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        if (e == 4) continue;
        if (a[e] > 0.0) {
            a[4] = a[4] + a[e];
            a[e] = 0.0;
        }
    }
}

// Edge weights: x-edge X(I,J) = (2I-1, 2J) for I <= nc+1, J <= nc collapses the
// lumped stencil along y (west, east); y-edge Y(I,J) = (2I, 2J-1) for I <= nc,
// J <= nc+1 collapses along x (south, north).  An edge that does not exist has
// the weights zero.
struct EdgeWeights {
    double lo, hi;   // LL, LR or LB, LA
    bool there;
};
template <bool NINE>
__device__ __forceinline__ EdgeWeights x_edge(const Lev<double> &F, int nc, int I, int J, int &bad)
{
    const bool there = J >= 1 && J <= nc;
    double a[9];
    row_of<NINE>(F, (size_t)(2 * min(max(J, 1), nc)) * F.ld + (2 * I - 1), a);
    lump_row(a);
    const double D = (a[4] + a[7]) + a[1];
    if (there && !(D > 0.0)) bad = F_BREAK_INTERP;
    const double lo = -((a[3] + a[6]) + a[0]) / D, hi = -((a[5] + a[8]) + a[2]) / D;
    return {there ? lo : 0.0, there ? hi : 0.0, there};
}
template <bool NINE>
__device__ __forceinline__ EdgeWeights y_edge(const Lev<double> &F, int nc, int I, int J, int &bad)
{
    const bool there = I >= 1 && I <= nc;
    double a[9];
    row_of<NINE>(F, (size_t)(2 * J - 1) * F.ld + 2 * min(max(I, 1), nc), a);
    lump_row(a);
    const double D = (a[4] + a[3]) + a[5];
    if (there && !(D > 0.0)) bad = F_BREAK_INTERP;
    const double lo = -((a[1] + a[0]) + a[2]) / D, hi = -((a[7] + a[6]) + a[8]) / D;
    return {there ? lo : 0.0, there ? hi : 0.0, there};
}

// All weights of coarse point (I, J), I, J <= nc+1: its two edges and its
// cell centre Z(I,J) = (2I-1, 2J-1), which takes the weights of the edges
// around it, the lumped stencil's couplings to them and to the four corners.
// The two edges of the south and west neighbours are formed again here: their
// rows are in the cache, and one pass over the level takes 188 us (4095^2,
// five-point) where edges and then centres took 137 + 126.
template <bool NINE>
static __global__ void k_weights(Lev<double> F, Wts<double> C, int nc, int *__restrict__ flags)
{
    const int I = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int J = blockIdx.y * blockDim.y + threadIdx.y + 1;
    if (I > nc + 1 || J > nc + 1) return;
    const size_t c = (size_t)J * C.ld + I;
    int bad = 0;
    const EdgeWeights n = x_edge<NINE>(F, nc, I, J, bad), s = x_edge<NINE>(F, nc, I, J - 1, bad);
    const EdgeWeights e = y_edge<NINE>(F, nc, I, J, bad), w = y_edge<NINE>(F, nc, I - 1, J, bad);
    double a[9];
    row_of<NINE>(F, (size_t)(2 * J - 1) * F.ld + (2 * I - 1), a);
    lump_row(a);
    if (!(a[4] > 0.0)) bad = F_BREAK_INTERP;
    if (n.there) {
        C.p[LL * C.ps + c] = n.lo;
        C.p[LR * C.ps + c] = n.hi;
    }
    if (e.there) {
        C.p[LB * C.ps + c] = e.lo;
        C.p[LA * C.ps + c] = e.hi;
    }
    C.p[LNE * C.ps + c] = -((a[8] + a[7] * n.hi) + a[5] * e.hi) / a[4];
    C.p[LNW * C.ps + c] = -((a[6] + a[7] * n.lo) + a[3] * w.hi) / a[4];
    C.p[LSE * C.ps + c] = -((a[2] + a[1] * s.hi) + a[5] * e.lo) / a[4];
    C.p[LSW * C.ps + c] = -((a[0] + a[1] * s.lo) + a[3] * w.lo) / a[4];
    if (bad) atomicOr(flags, bad);
}

// --------------------------------------------------------- Galerkin RAP
// Weight of coarse basis function K = (KI,KJ) at fine point 2K + (di,dj).
__device__ __forceinline__ double basis_weight(const Wts<double> &C, int KI, int KJ, int di, int dj)
{
    const size_t c = (size_t)KJ * C.ld + KI;
    if (dj == 0) {
        if (di == 0) return 1.0;
        return di < 0 ? C.at(LR, c) : C.at(LL, c + 1);
    }
    if (dj < 0) {
        if (di == 0) return C.at(LA, c);
        return di < 0 ? C.at(LNE, c) : C.at(LNW, c + 1);
    }
    if (di == 0) return C.at(LB, c + C.ld);
    return di < 0 ? C.at(LSE, c + C.ld) : C.at(LSW, c + C.ld + 1);
}

// A_c(I,J;d) = sum_p P(p;IJ) sum_q A(p,q) P(q;IJ+d), d = O, W, S, SW, NW, p over
// the fine 3x3 patch of (2I,2J) (rows south to north, west to east inside a
// row), q over p's neighbours SW..NE inside the support of basis IJ+d; both
// sums start from zero.  Couplings to ring coarse points are zero: their sums
// are formed with the weights of the nearest interior point (so every load
// is in range and none waits behind a branch) and then replaced by zero.
template <bool NINE>
static __global__ __launch_bounds__(128) void k_rap(Lev<double> F, Wts<double> C, Lev<double> Cl)
{
    const int I = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int J = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int nc = Cl.n;
    if (I > nc || J > nc) return;
    constexpr int offI[5] = {0, -1, 0, -1, -1};
    constexpr int offJ[5] = {0, 0, -1, -1, 1};
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    bool live[5];
    int KI[5], KJ[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) {
        const int ki = I + offI[d], kj = J + offJ[d];
        live[d] = ki >= 1 && kj >= 1 && kj <= nc;
        KI[d] = ki < 1 ? 1 : ki;
        KJ[d] = kj < 1 ? 1 : kj > nc ? nc : kj;
    }
#pragma unroll
    for (int jj = -1; jj <= 1; ++jj) {
#pragma unroll
        for (int ii = -1; ii <= 1; ++ii) {
            const int pi = 2 * I + ii, pj = 2 * J + jj;
            double a[9];
            row_of<NINE>(F, (size_t)pj * F.ld + pi, a);
            const double wp = basis_weight(C, I, J, ii, jj);
#pragma unroll
            for (int d = 0; d < 5; ++d) {
                double t = 0.0;
#pragma unroll
                for (int e = 0; e < 9; ++e) {
                    // q - 2(IJ+d), the same for the clamped point's support
                    const int di = ii + (e % 3) - 1 - 2 * offI[d], dj = jj + (e / 3) - 1 - 2 * offJ[d];
                    if (di < -1 || di > 1 || dj < -1 || dj > 1) continue;
                    t = t + a[e] * basis_weight(C, KI[d], KJ[d], di, dj);
                }
                acc[d] = acc[d] + wp * t;
            }
        }
    }
    const size_t c = (size_t)J * Cl.ld + I;
    Cl.O[c] = acc[0];
    Cl.W[c] = live[1] ? acc[1] : 0.0;
    Cl.S[c] = live[2] ? acc[2] : 0.0;
    Cl.SW[c] = live[3] ? acc[3] : 0.0;
    Cl.NW[c] = live[4] ? acc[4] : 0.0;
}

// The set-up kernels of one level pair, for a five- or nine-point fine stencil.
static inline void launch_weights(const Lev<double> &F, const Wts<double> &C, int nc, int *flags, dim3 grid,
                                  dim3 blk, hipStream_t st)
{
    if (F.SW) hipLaunchKernelGGL(k_weights<true>, grid, blk, 0, st, F, C, nc, flags);
    else hipLaunchKernelGGL(k_weights<false>, grid, blk, 0, st, F, C, nc, flags);
}

static inline void launch_rap(const Lev<double> &F, const Wts<double> &C, const Lev<double> &Cl, hipStream_t st)
{
    const dim3 blk(32, 4), grid((Cl.n + 31) / 32, (Cl.n + 3) / 4);
    if (F.SW)
        hipLaunchKernelGGL(k_rap<true>, grid, blk, 0, st, F, C, Cl);
    else
        hipLaunchKernelGGL(k_rap<false>, grid, blk, 0, st, F, C, Cl);
}

// ------------------------------------------------ coarsest level: band LDL^T
// The coarsest level (nc points per side, 3 <= nc <= 63) is solved directly.
// Its unknowns in lexicographic order k = (i-1) + nc (j-1) give a band matrix
// of half-bandwidth w = nc + 1 <= 64, whose square-root-free Cholesky factor
// L D L^T stays inside the band.  Set-up keeps
//   Lb[i w + (k - i + w)] = L_ik  (k = i-w .. i-1, zero for k < 0), D[i];
// and, for the solve, the same entries rearranged by the lane that uses them
// (BandSolve below).
constexpr int BAND_MAX_NC = 63;

// A(i, i - d) of the coarsest level's matrix, d = 0 .. w, from its compact
// stencil: d = 1 W, nc - 1 SE (the NW entry of the point below-right), nc S,
// nc + 1 SW; couplings to points outside the grid are zero.
__device__ inline double band_entry(const Lev<double> &L, int i, int d)
{
    const int nc = L.n;
    const int ii = i % nc + 1, jj = i / nc + 1;
    const size_t p = (size_t)jj * L.ld + ii;
    if (d == 0) return L.O[p];
    if (d == 1) return ii > 1 ? L.W[p] : 0.0;
    if (d == nc - 1) return (ii < nc && jj > 1 && L.NW) ? L.NW[p + 1 - L.ld] : 0.0;
    if (d == nc) return jj > 1 ? L.S[p] : 0.0;
    if (d == nc + 1) return (ii > 1 && jj > 1 && L.SW) ? L.SW[p] : 0.0;
    return 0.0;
}

// A workgroup barrier that orders LDS only: loads from global memory stay in
// flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// v of lane `lane`, on every lane.
__device__ __forceinline__ double readlane_d(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The factor in one workgroup, in right-looking form by panels of
// BAND_PANEL columns.  Once column k is final (D_k = a_kk, L_ik = a_ik / D_k,
// v_j = L_jk D_k), every entry of the trailing window takes its term,
// a_ij <- a_ij - L_ik v_j (k < j <= i <= k + w).  An entry thus receives its
// terms in order of increasing k, each the same product of the same operands
// as in the column-by-column sums of the definition
//   D_j = A_jj - sum_k L_jk v_k,  L_ij = (A_ij - sum_k L_ik v_k) / D_j,
// so the factor is the same to the bit.  A panel's columns are finished by
// wave 0 alone in registers, one after the other, together with the terms
// they give to the panel's own later columns (each lane holds two rows of
// the panel; the diagonal and the v values come from their rows' lanes by
// readlane); then every thread applies the panel's terms, in column order,
// to its entries of the trailing triangle and writes the panel's L and D to
// memory: two barriers per panel instead of two per column.  One wave's
// column chain is what the factor waits on, so that part is straight-line
// code with one division per lane and column and no stores to memory (at
// 63^2: 2.04 ms; 2.81 ms with predicated updates and the stores in wave 0,
// 2.92 ms by columns).  The window's rows live in an LDS ring (row i,
// column j at slot i mod RR, offset j - i + w); the B rows a panel adds to the
// window enter during the previous panel's trailing update, their entries of
// A requested from memory two panels ahead (registers, then a staging
// buffer), so no panel waits on memory.
constexpr int BAND_FACTOR_THREADS = 1024;
constexpr int BAND_NNZ = 5;   // lower-band entries of a row of A: distances 0, 1, nc - 1, nc, nc + 1
#ifndef BMG_BAND_PANEL
#define BMG_BAND_PANEL 8
#endif
constexpr int BAND_PANEL = BMG_BAND_PANEL;
static_assert(BAND_PANEL * (BAND_MAX_NC + 2) <= BAND_FACTOR_THREADS && BAND_PANEL <= 64,
              "the rows a panel adds take one thread per entry, and wave 0 holds the panel's rows");

__device__ inline int band_nz_dist(int e, int nc) { return e == 0 ? 0 : e == 1 ? 1 : e == 2 ? nc - 1 : e == 3 ? nc : nc + 1; }

static __global__ __launch_bounds__(BAND_FACTOR_THREADS) void k_band_factor(Lev<double> L, double *__restrict__ Lb,
                                                                             double *__restrict__ D,
                                                                             int *__restrict__ flags)
{
    constexpr int B = BAND_PANEL, RW = BAND_MAX_NC + 2, RR = BAND_MAX_NC + 1 + B;
    __shared__ double ring[RR * RW];
    __shared__ double Lp[B][RW], vp[B][RW];           // the panel's columns: L(k + d, k), v at offset d
    __shared__ double stage[2][B * BAND_NNZ];
    __shared__ double Dpan[B];
    const int nc = L.n, m = nc * nc, w = nc + 1, t = threadIdx.x;
    const int npanel = (m + B - 1) / B;
    auto at = [&](int i, int j) -> double & { return ring[(i % RR) * RW + (j - i + w)]; };
    // the rows panel q adds to the window: q B + w .. q B + w + B - 1; entry u
    // of its staging buffer is row q B + w + u / NNZ at distance nz(u % NNZ)
    auto entering = [&](int q, int u) -> double {
        const int i = q * B + w + u / BAND_NNZ;
        return i < m ? band_entry(L, i, band_nz_dist(u % BAND_NNZ, nc)) : 0.0;
    };
    // rows 0 .. w + B - 1 of A (the window of panel 0)
    for (int e = t; e < (w + B) * (w + 1); e += blockDim.x) {
        const int i = e / (w + 1), off = e % (w + 1), j = i - w + off;
        if (i < m) at(i, j) = j >= 0 ? band_entry(L, i, i - j) : 0.0;
    }
    const bool loader = t < B * BAND_NNZ;
    if (loader) stage[1] [t] = entering(1, t);
    double pf = loader ? entering(2, t) : 0.0;        // panel 2's rows, in flight
    // this thread's entries of the trailing triangle, e = t + s * blockDim.x
    const int ntri = w * (w + 1) / 2;
    int di[3], dj[3];
#pragma unroll
    for (int s2 = 0; s2 < 3; ++s2) {
        const int e = t + s2 * BAND_FACTOR_THREADS;
        int d = (int)((1.0f + sqrtf(8.0f * (float)e + 1.0f)) * 0.5f);
        while (d > 1 && d * (d - 1) / 2 > e) --d;
        while ((d + 1) * d / 2 <= e) ++d;
        di[s2] = e < ntri ? d : 0;
        dj[s2] = e - d * (d - 1) / 2 + 1;
    }
    // this thread's entry of the rows entering the window: row b, offset off
    const int eb = t / (w + 1), eoff = t % (w + 1);
    const bool enters = t < B * (w + 1);
    int eu = -1;   // its index in the staging buffer (-1: a zero of the band)
    if (enters) {
#pragma unroll
        for (int e = 0; e < BAND_NNZ; ++e)
            if (w - eoff == band_nz_dist(e, nc)) eu = eb * BAND_NNZ + e;
    }
    int bad = 0;
    lds_barrier();
    for (int p = 0; p < npanel; ++p) {
        const int k0 = p * B;
        if (t < 64) {
            // wave 0: the panel's columns, in registers.  Lane l holds the
            // panel entries of rows k0 + l and k0 + 64 + l.  The band rows
            // below the diagonal of column k = k0 + b are k + 1 .. k + 64:
            // the first row of lanes l > b and the second row of lanes
            // l <= b, so every lane divides once per column.  The diagonal
            // and the v of a later panel column come from the lane of its
            // row.  A row outside a column's band holds zeros there, and
            // rows past the matrix act as rows of the identity (D = 1, no
            // terms), so the work is the same straight-line code for every
            // panel; a lane's first row takes terms in every later panel
            // column (those right of its diagonal are never read again),
            // its second row only once it is the lane's row of the column
            const int r0 = k0 + t, r1 = k0 + 64 + t;
            double a0[B], a1[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int k = k0 + b;
                a0[b] = r0 >= m ? (r0 == k ? 1.0 : 0.0) : (r0 >= k && r0 - k <= w) ? at(r0, k) : 0.0;
                a1[b] = (r1 < m && r1 - k <= w) ? at(r1, k) : 0.0;
            }
            double dg = 0.0;   // D of the lane's own panel column
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const double Dk = readlane_d(a0[b], b);
                dg = t == b ? a0[b] : dg;
                const bool first = t > b;
                const double l = (first ? a0[b] : a1[b]) / Dk;
                const double v = l * Dk;
                const int d = first ? t - b : 64 + t - b;   // the lane's row of the column is k + d
                if (d <= w) {
                    Lp[b][d] = l;
                    vp[b][d] = v;
                }
                const double l1 = first ? 0.0 : l;
                // the terms of column k in the panel's later columns
#pragma unroll
                for (int jb = b + 1; jb < B; ++jb) {
                    const double vj = readlane_d(v, jb);   // v(k0 + jb, k), the lane of row k0 + jb
                    a0[jb] = a0[jb] - l * vj;
                    a1[jb] = a1[jb] - l1 * vj;
                }
            }
            if (t < B) Dpan[t] = dg;
        }
        lds_barrier();
        // the panel's columns go to memory, a row's B entries side by side
        if (t < (w + B - 1) * B) {
            const int r = k0 + 1 + t / B, b = t % B, d = r - k0 - b;
            if (d >= 1 && d <= w && r < m) Lb[(size_t)r * w + (w - d)] = Lp[b][d];
        }
        if (t >= BAND_FACTOR_THREADS - B) {
            const int b = t - (BAND_FACTOR_THREADS - B);
            if (k0 + b < m) {
                const double Dk = Dpan[b];
                D[k0 + b] = Dk;
                if (!(Dk > 0.0)) bad = 1;
            }
        }
        // the panel's terms in the trailing triangle (rows and columns
        // k0 + B .. k0 + B - 1 + w), in column order
#pragma unroll
        for (int s2 = 0; s2 < 3; ++s2) {
            const int i = k0 + B - 1 + di[s2], j = k0 + B - 1 + dj[s2];
            if (di[s2] > 0 && i < m) {
                double a = at(i, j);
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const int k = k0 + b;
                    if (i - k <= w && k < m) a = a - Lp[b][i - k] * vp[b][j - k];
                }
                at(i, j) = a;
            }
        }
        // the rows of panel p + 1 enter (their slots are those of panel p's
        // rows); the staging buffer of panel p + 2 is filled from the
        // registers and panel p + 3's entries are requested
        if (enters) {
            const int i = (p + 1) * B + w + eb;
            if (i < m) at(i, i - w + eoff) = eu >= 0 ? stage[(p + 1) & 1][eu] : 0.0;
        }
        if (loader) {
            stage[p & 1][t] = pf;
            pf = entering(p + 3, t);
        }
        lds_barrier();
    }
    if (bad) atomicOr(flags, F_BREAK_COARSE);
}

// The factor as the one-wave solve reads it.  Unknowns are padded to M, a
// multiple of 64, and taken in blocks of 16 (block p: unknowns 16p .. 16p+15).
// While block p is being finished, every 16-lane row of the wave holds the
// block's pending values (`cur`, unknown 16p + i in lane i of each row), and
// `pend` holds the pending values of the four blocks that come next, block b in
// row b mod 4: w <= 64, so a step touches nothing further away.  A step then
// takes its final value from lane t of each row by the row broadcast of the
// multiply-add itself (DPP), without a trip through scalar registers.
// Row of step s = 16p + t (CF forward, CG backward), 64 doubles, lane l = 16r + i:
//   CF: r == p mod 4:  i > t:  -L(16p + i, s)          (cur)
//                      i <= t: -L(16(p + 4) + i, s)    (pend)
//       else, b the block of p+1 .. p+3 with b mod 4 == r: -L(16b + i, s);
//   CG: r == p mod 4:  i < t:  -L(s, 16p + i)          (cur)
//                      i >= t: -L(s, 16(p - 4) + i)    (pend)
//       else, b the block of p-1 .. p-3 with b mod 4 == r: -L(s, 16b + i);
// (-)zero wherever the entry lies outside the band or the matrix; Dp = D
// padded with ones.  Two consecutive steps in the order they run (CG: t
// descending) lie side by side per lane, so one 16-byte access per lane reads
// both; the 64 rows of 4 blocks are contiguous (32 KB).
struct BandSolve {
    const double *CF, *CG, *Dp;
    int m, M, nc;
};

__host__ __device__ inline int band_padded(int m) { return (m + 63) & ~63; }

// Step s of a factor given by its entries Lf(i, k) of the forward and
// Ub(k, i) of the backward substitution (the multiple of the final value of
// unknown s that the pending value of unknown i loses), written by lane l.
template <typename Fwd, typename Bwd>
__device__ __forceinline__ void band_expand_step(int s, int l, double *CF, double *CG, Fwd &&fwd, Bwd &&bwd)
{
    const int p = s >> 4, t = s & 15, r = l >> 4, i = l & 15, e = 15 - t;
    const int f = r == (p & 3) ? (i > t ? p : p + 4) : p + ((r - p) & 3);
    const int g = r == (p & 3) ? (i < t ? p : p - 4) : p - ((p - r) & 3);
    CF[((size_t)(p * 8 + (t >> 1)) * 64 + l) * 2 + (t & 1)] = -fwd(16 * f + i, s);
    CG[((size_t)(p * 8 + (e >> 1)) * 64 + l) * 2 + (e & 1)] = -bwd(16 * g + i, s);
}

static __global__ void k_band_expand(int nc, const double *__restrict__ Lb, const double *__restrict__ D,
                                     double *__restrict__ CF, double *__restrict__ CG, double *__restrict__ Dp)
{
    const int m = nc * nc, w = nc + 1, M = band_padded(m);
    const int l = threadIdx.x & 63;
    const int s = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);   // step
    if (s >= M) return;
    // L(i, k) for 0 <= i - w <= k < i < m, else 0
    auto Lik = [&](int i, int k) -> double {
        return (i < m && k >= 0 && k < i && i - k <= w) ? Lb[(size_t)i * w + (k - i + w)] : 0.0;
    };
    band_expand_step(s, l, CF, CG, [&](int i, int k) { return Lik(i, k); }, [&](int i, int k) { return Lik(k, i); });
    if (l == 0) Dp[s] = s < m ? D[s] : 1.0;
}

typedef double band_v2d __attribute__((ext_vector_type(2)));

// Eight steps of a block, H = 0 the first half: the final value y of lane t of
// each row is broadcast within the row and y L is removed from the pending
// values, each update one fused multiply-add rounded once (c, p hold -L for cur
// and pend, two steps each; t ascending for DIR > 0, else descending).  A lane
// whose entry is zero keeps its value (up to the sign of a zero).  A DPP operand
// must not be read within two wait states of the vector instruction that
// wrote it, and the compiler does not look into the block (it may even copy
// cur just before it, hence the first wait): `cur` takes its own update first,
// and `pend` reads its broadcast from a copy of cur as the previous step left
// it (%2 and %3 in turn), so a step's copy and its update of pend are the two
// instructions between a write of cur and its next use; waiting in their
// place costs a slot more per step.
template <int DIR, int H>
__device__ __forceinline__ void band_steps(double &cur, double &pend, const band_v2d *c, const band_v2d *p)
{
    double copy = cur, mid;
    constexpr int T0 = DIR > 0 ? 8 * H : 15 - 8 * H;
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %0, %4 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %3, %0\n\t"
                 "v_fmac_f64_dpp %1, %2, %12 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %5 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %2, %0\n\t"
                 "v_fmac_f64_dpp %1, %3, %13 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %6 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %3, %0\n\t"
                 "v_fmac_f64_dpp %1, %2, %14 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %7 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %2, %0\n\t"
                 "v_fmac_f64_dpp %1, %3, %15 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %8 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %3, %0\n\t"
                 "v_fmac_f64_dpp %1, %2, %16 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %9 row_newbcast:%25 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %2, %0\n\t"
                 "v_fmac_f64_dpp %1, %3, %17 row_newbcast:%25 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %10 row_newbcast:%26 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %3, %0\n\t"
                 "v_fmac_f64_dpp %1, %2, %18 row_newbcast:%26 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %0, %0, %11 row_newbcast:%27 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mov_b64 %2, %0\n\t"
                 "v_fmac_f64_dpp %1, %3, %19 row_newbcast:%27 row_mask:0xf bank_mask:0xf"
                 : "+v"(cur), "+v"(pend), "+v"(copy), "=&v"(mid)
                 : "v"(c[0].x), "v"(c[0].y), "v"(c[1].x), "v"(c[1].y), "v"(c[2].x), "v"(c[2].y), "v"(c[3].x),
                   "v"(c[3].y), "v"(p[0].x), "v"(p[0].y), "v"(p[1].x), "v"(p[1].y), "v"(p[2].x), "v"(p[2].y),
                   "v"(p[3].x), "v"(p[3].y), "n"(T0), "n"(T0 + DIR), "n"(T0 + 2 * DIR), "n"(T0 + 3 * DIR),
                   "n"(T0 + 4 * DIR), "n"(T0 + 5 * DIR), "n"(T0 + 6 * DIR), "n"(T0 + 7 * DIR));
}

// Row R of v in every row of the wave: two copies swap their rows 16 lanes
// apart, (0, 0, 2, 2) and (1, 1, 3, 3), then two copies of the one that holds
// row R their halves.  v may come straight from band_steps, and a swap must not
// read a register within two wait states of its write: the compiler, which
// does not look into that block and would wait for each half in turn, is kept
// out of it.
template <int R>
__device__ __forceinline__ double row_to_all(double v)
{
    double a, b;
    asm volatile("v_mov_b64 %0, %2\n\t"
                 "v_mov_b64 %1, %2\n\t"
                 "s_nop 1" : "=&v"(a), "=&v"(b) : "v"(v));
    auto swap = [](double &x, double &y, bool half) {
        const long long p = __double_as_longlong(x), q = __double_as_longlong(y);
        unsigned h[2][2] = {{(unsigned)p, (unsigned)(p >> 32)}, {(unsigned)q, (unsigned)(q >> 32)}};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const auto t = half ? __builtin_amdgcn_permlane32_swap(h[0][k], h[1][k], false, false)
                                : __builtin_amdgcn_permlane16_swap(h[0][k], h[1][k], false, false);
            h[0][k] = t[0];
            h[1][k] = t[1];
        }
        x = __longlong_as_double(((long long)h[0][1] << 32) | h[0][0]);
        y = __longlong_as_double(((long long)h[1][1] << 32) | h[1][0]);
    };
    swap(a, b, false);
    double c = (R & 1) ? b : a, d;
    asm volatile("v_mov_b64 %0, %1\n\t"
                 "s_nop 1" : "=&v"(d), "+v"(c));
    swap(c, d, true);
    return (R >> 1) ? d : c;
}

// The coarsest solve x = L^-T D^-1 L^-1 b, in the order of the oracle's
// column form: y_i takes its terms over increasing j, z_i = y_i / D_i, x_i
// takes its terms over decreasing k.  Run by one wave (lanes l = 0..63),
// reading the step rows from global memory (the persistent small-level
// kernel, whose coarsest level is small).  Blocks of padding unknowns (index
// >= m) change nothing and are skipped.  get(k): right-hand side of unknown
// k < m as FP64; put(k, x): the result; z: M doubles of scratch.
template <typename Get, typename Put>
__device__ void band_solve_direct(const BandSolve &B, Get get, Put put, double *z)
{
    const int l = threadIdx.x & 63, i = l & 15, r = l >> 4, m = B.m, nb = (m + 15) >> 4;
    auto rhs = [&](int k) -> double { return k < m ? get(k) : 0.0; };
    // the factors of a block: each half's registers take the next block's half
    // once they are used, so its loads run behind the rest of the block
    band_v2d fc[8], fp[8];
    auto load = [&](const double *rows, int p, int k) {
        const band_v2d *g = reinterpret_cast<const band_v2d *>(rows) + (size_t)(p * 8 + k) * 64;
        fp[k] = g[l];
        fc[k] = g[(p & 3) * 16 + i];
    };
    auto start = [&](const double *rows, int p) {
#pragma unroll
        for (int k = 0; k < 8; ++k) load(rows, p, k);
    };
    // half h of the block, each entry zero where it belongs to the other of
    // cur and pend; then the same half of block pn is requested
    auto half = [&](auto dir, auto h, bool own, const double *rows, int pn, double &cur, double &pend) {
        constexpr bool fwd = dir.value > 0;
        band_v2d c[4], f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = 4 * h.value + u, ta = fwd ? 2 * k : 15 - 2 * k, tb = fwd ? 2 * k + 1 : 14 - 2 * k;
            const bool ca = fwd ? i > ta : i < ta, cb = fwd ? i > tb : i < tb;
            c[u].x = ca ? fc[k].x : -0.0;
            c[u].y = cb ? fc[k].y : -0.0;
            f[u].x = own && ca ? -0.0 : fp[k].x;
            f[u].y = own && cb ? -0.0 : fp[k].y;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) load(rows, pn, 4 * h.value + u);
        band_steps<dir.value, h.value>(cur, pend, c, f);
    };
    using Up = std::integral_constant<int, 1>;
    using Down = std::integral_constant<int, -1>;
    using First = std::integral_constant<int, 0>;
    using Second = std::integral_constant<int, 1>;
    auto next_cur = [](int rr, double pend) {
        return rr == 0 ? row_to_all<0>(pend) : rr == 1 ? row_to_all<1>(pend)
             : rr == 2 ? row_to_all<2>(pend) : row_to_all<3>(pend);
    };
    // rows 1..3 hold blocks 1..3, row 0 block 4
    start(B.CF, 0);
    double cur = rhs(i), pend = rhs(r == 0 ? 64 + i : l);
    for (int p = 0; p < nb; ++p) {
        const double nx = rhs(16 * (p + 5) + i);
        const bool own = r == (p & 3);
        const int pn = p + 1 < nb ? p + 1 : p;
        half(Up{}, First{}, own, B.CF, pn, cur, pend);
        half(Up{}, Second{}, own, B.CF, pn, cur, pend);
        if (r == 0) z[16 * p + i] = cur / B.Dp[16 * p + i];
        const int rr = (p + 1) & 3;
        cur = next_cur(rr, pend);
        pend = r == rr ? nx : pend;
    }
    auto zed = [&](int k) -> double { return k >= 0 ? z[k] : 0.0; };
    start(B.CG, nb - 1);
    // block b of nb-2 .. nb-5 in row b mod 4
    cur = zed(16 * (nb - 1) + i);
    pend = zed(16 * (nb - 2 - ((nb - 2 - r) & 3)) + i);
    for (int p = nb - 1; p >= 0; --p) {
        const double nx = zed(16 * (p - 5) + i);
        const bool own = r == (p & 3);
        const int pn = p > 0 ? p - 1 : p;
        half(Down{}, First{}, own, B.CG, pn, cur, pend);
        half(Down{}, Second{}, own, B.CG, pn, cur, pend);
        if (r == 0 && 16 * p + i < m) put(16 * p + i, cur);
        const int rr = (p - 1) & 3;
        cur = next_cur(rr, pend);
        pend = r == rr ? nx : pend;
    }
}

// The coarsest solve as a kernel of its own (the coarsest level is larger
// than the persistent small-level kernel handles, or the basic path runs).
// Wave 0 runs the chain of steps, 64 (four blocks) per phase, reading the
// factors from LDS, so a step is two fused multiply-adds, a copy and half a
// pair of 16-byte reads.  The loader waves split the rows of a phase into the
// entries of `cur` and of `pend` (8 KB + 32 KB) in one of three LDS slots, two
// phases ahead, so the chain's reads run ahead across the end of a phase; the
// global loads of the phases after that are already in flight in the loaders'
// registers (BAND_INFLIGHT sets), so memory latency stays behind the chain.
// The right-hand side is staged in LDS first (z).  Phases run forward through
// the blocks, then backward: nch = M / 32 phases.  Workgroup k solves
// right-hand side k (its arrays ks elements, its stop flag kstop ints after
// the first's).
constexpr int BAND_LOADERS = 8;
constexpr int BAND_SOLVE_THREADS = 64 * (1 + BAND_LOADERS);
constexpr int BAND_INFLIGHT = 4;
constexpr int BAND_PER_LANE = 64 * 64 / 2 / (64 * BAND_LOADERS);   // double pairs per loader lane per phase
constexpr int BAND_SLOT = 64 * 64 + 64 * 16;                       // doubles of a phase in LDS

// Phases the loaders write: one past the last (its slot is read ahead), in
// whole rounds of the loaders' register sets; every wave passes one barrier
// after each of them but the first.
__host__ __device__ inline int band_phases(int nch) { return (nch + BAND_INFLIGHT) / BAND_INFLIGHT * BAND_INFLIGHT; }

__host__ __device__ inline size_t band_solve_lds(int M) { return ((size_t)M + 3 * BAND_SLOT) * sizeof(double); }

// The factors of a block's eight pairs of steps, in running order.
struct BandFactors {
    band_v2d c[8], p[8];
};

// Pair k of a phase from its slot: `pend` entries per lane, then `cur` entries
// per lane of a row.
__device__ __forceinline__ void band_read(const double *slot, int l, int k, band_v2d &c, band_v2d &p)
{
    p = reinterpret_cast<const band_v2d *>(slot)[k * 64 + l];
    c = reinterpret_cast<const band_v2d *>(slot + 64 * 64)[k * 16 + (l & 15)];
}

// The four blocks of a phase.  The next block's factors are requested at the
// start of a block (the scheduling barriers keep them there: left to itself
// the scheduler reads a row just before its step to save registers, and the
// read's latency joins the chain) and waited for at its end: an instruction
// of any kind costs the lone wave about 5 clocks, a wait per pair as much as a
// step's multiply-add.  nx, nx2: the pending values that enter as
// blocks finish.  Returns the final values of the phase, lane l = unknown l of
// the 64.
template <int DIR>
__device__ __forceinline__ double band_phase(double &cur, double &pend, BandFactors &A, const double *slot,
                                             const double *next, int l, double nx, const double &nx2)
{
    const int r = l >> 4;
    double fin = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        BandFactors N;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            band_read(b < 3 ? slot : next, l, b < 3 ? 8 * (b + 1) + u : u, N.c[u], N.p[u]);
        __builtin_amdgcn_sched_barrier(0);
        band_steps<DIR, 0>(cur, pend, A.c, A.p);
        band_steps<DIR, 1>(cur, pend, A.c + 4, A.p + 4);
        __builtin_amdgcn_sched_barrier(0);
        const int s = DIR > 0 ? b : 3 - b, rr = DIR > 0 ? (s + 1) & 3 : (s + 3) & 3;
        fin = r == s ? cur : fin;
        cur = rr == 0 ? row_to_all<0>(pend) : rr == 1 ? row_to_all<1>(pend)
            : rr == 2 ? row_to_all<2>(pend) : row_to_all<3>(pend);
        pend = r == rr ? (b < 3 ? nx : nx2) : pend;
        __builtin_amdgcn_s_waitcnt(0xc07f);   // LDS reads only
#pragma unroll
        for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(N.c[k]), "+v"(N.p[k]));
        A = N;
    }
    return fin;
}

template <typename T>
static __global__ __launch_bounds__(BAND_SOLVE_THREADS) void k_coarse_solve(Lev<T> Cl, BandSolve B, size_t ks,
                                                                               const int *stop, int kstop)
{
    const int rk = blockIdx.x;
    extern __shared__ double band_sm[];
    double *z = band_sm, *slots = band_sm + B.M;
    const int nb = B.M >> 6, nch = 2 * nb;
    const int l = threadIdx.x & 63;
    const int nc = B.nc, m = B.m;
    if (threadIdx.x >= 64) {
        // loaders.  Phase c: the 64 unknowns q, forward for c < nb, backward
        // after; its rows are contiguous in CF or CG.
        const int t0 = threadIdx.x - 64;
        // the loads are unconditional (a phase past the last reads the last)
        // and so are the phases, and the requests keep their order, so that
        // the wait for a set covers that set's loads only and the other sets
        // stay in flight
        band_v2d buf[BAND_INFLIGHT][BAND_PER_LANE];
        auto request = [&](band_v2d(&v)[BAND_PER_LANE], int c) {
            const int cc = min(c, nch - 1);
            const bool fwd = cc < nb;
            const int q = fwd ? cc : nch - 1 - cc;
            const band_v2d *g = reinterpret_cast<const band_v2d *>((fwd ? B.CF : B.CG) + (size_t)q * 4096);
#pragma unroll
            for (int e = 0; e < BAND_PER_LANE; ++e) v[e] = g[t0 + e * 64 * BAND_LOADERS];
            __builtin_amdgcn_sched_barrier(0);
        };
        // the right-hand side and the first rows are requested before the stop
        // flag is known, so that their latencies overlap.  Unknown k sits at
        // point (k mod nc, k div nc).
        constexpr int NZ = BAND_MAX_NC * BAND_MAX_NC / (64 * BAND_LOADERS) + 1;
        double zv[NZ];
        {
            const T *bv = Cl.b + (size_t)rk * ks;
            int j = t0 / nc, i = t0 - j * nc;
            const int dj = 64 * BAND_LOADERS / nc, di = 64 * BAND_LOADERS - dj * nc;
#pragma unroll
            for (int e = 0; e < NZ; ++e) {
                const bool in = t0 + e * 64 * BAND_LOADERS < m;
                const double v = (double)bv[in ? (size_t)(j + 1) * Cl.ld + i + 1 : 0];
                zv[e] = in ? v : 0.0;
                i += di;
                j += dj;
                if (i >= nc) {
                    i -= nc;
                    ++j;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < BAND_INFLIGHT; ++u) request(buf[u], u);
        if (stopped(stop ? stop + rk * kstop : stop)) return;
#pragma unroll
        for (int e = 0; e < NZ; ++e)
            if (t0 + e * 64 * BAND_LOADERS < B.M) z[t0 + e * 64 * BAND_LOADERS] = zv[e];
        // phase c: its rows go into slot c mod 3 (one that is no longer read),
        // block by block in the order they run; the set then requests phase
        // c + BAND_INFLIGHT.  Wave k holds pair k of each block, e = 0 .. 3:
        // the `cur` entries of block e are in its row e, so the four blocks'
        // are gathered into one write (an instruction costs a wave about 5
        // clocks here, and the loaders have to keep up with the chain)
        static_assert(BAND_LOADERS == 8 && BAND_PER_LANE == 4, "a loader wave holds one pair of each block");
        const int k = __builtin_amdgcn_readfirstlane(t0 >> 6), i = l & 15, r = l >> 4;
        const bool upx = i > 2 * k, upy = i > 2 * k + 1, dnx = i < 15 - 2 * k, dny = i < 14 - 2 * k;
        double *dst = slots;
        auto phase = [&](band_v2d(&v)[BAND_PER_LANE], int c) {
            const bool fwd = c < nb;
            const bool cx = fwd ? upx : dnx, cy = fwd ? upy : dny;   // an entry of cur, in the own row
            band_v2d g = v[0];
            band_v2d *pd = reinterpret_cast<band_v2d *>(dst) + k * 64 + l;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                band_v2d f = v[e];
                const bool own = r == e;
                if (e > 0) g = own ? f : g;
                f.x = own && cx ? -0.0 : f.x;
                f.y = own && cy ? -0.0 : f.y;
                pd[(fwd ? e : 3 - e) * 8 * 64] = f;
            }
            g.x = cx ? g.x : -0.0;
            g.y = cy ? g.y : -0.0;
            reinterpret_cast<band_v2d *>(dst + 64 * 64)[((fwd ? r : 3 - r) * 8 + k) * 16 + i] = g;
            dst = dst == slots + 2 * BAND_SLOT ? slots : dst + BAND_SLOT;
            request(v, c + BAND_INFLIGHT);
            if (c > 0) lds_barrier();
        };
        for (int c0 = 0; c0 < band_phases(nch); c0 += BAND_INFLIGHT) {
#pragma unroll
            for (int u = 0; u < BAND_INFLIGHT; ++u) phase(buf[u], c0 + u);
        }
        return;
    }
    // wave 0: forward through the blocks, then backward.  Unknown 64q + l of
    // the next and the next but one 64 enter as blocks finish (zero outside).
    // At barrier c the slots of phases c and c + 1 are filled.  The barrier
    // between phases orders the loaders' later writes after this wave's reads
    // of a slot, whose values have all been used by then, so the reads ahead
    // stay in flight across it.
    T *uv = Cl.u + (size_t)rk * ks;
    const double *cs = slots, *ns = slots + BAND_SLOT;
    auto turn = [&]() {
        cs = ns;
        ns = ns == slots + 2 * BAND_SLOT ? slots : ns + BAND_SLOT;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    double d = B.Dp[l];
    if (stopped(stop ? stop + rk * kstop : stop)) return;
    __builtin_amdgcn_s_setprio(3);                  // before the loaders on the same SIMD
    lds_barrier();                                  // phases 0 and 1 and b are in LDS
    BandFactors A;
#pragma unroll
    for (int k = 0; k < 8; ++k) band_read(cs, l, k, A.c[k], A.p[k]);
    auto zq = [&](int q) -> double { return q >= 0 && q < nb ? z[64 * q + l] : 0.0; };
    double cur = z[l & 15], nx = zq(1), pend = l < 16 ? nx : z[l];
    for (int q = 0; q < nb; ++q) {
        const double nx2 = zq(q + 2), dn = B.Dp[64 * min(q + 1, nb - 1) + l];
        const double fin = band_phase<1>(cur, pend, A, cs, ns, l, nx, nx2);
        z[64 * q + l] = fin / d;                    // b of these unknowns is no longer needed
        nx = nx2;
        d = dn;
        turn();
    }
    cur = z[64 * (nb - 1) + 48 + (l & 15)];
    nx = zq(nb - 2);
    pend = l >= 48 ? nx : z[64 * (nb - 1) + l];
    // unknown k = 64q + l at point (k mod nc, k div nc), walked down with q
    int k = 64 * (nb - 1) + l, j = k / nc, i = k - j * nc;
    const int dj = 64 / nc, di = 64 - dj * nc;
    for (int q = nb - 1; q >= 0; --q) {
        const double nx2 = zq(q - 2);
        const double x = band_phase<-1>(cur, pend, A, cs, ns, l, nx, nx2);
        if (k < m) uv[(size_t)(j + 1) * Cl.ld + i + 1] = (T)x;
        k -= 64;
        j -= dj;
        i -= di;
        if (i < 0) {
            i += nc;
            --j;
        }
        nx = nx2;
        if (q > 0) turn();
    }
    for (int c = nch; c < band_phases(nch) - 1; ++c) lds_barrier();   // the loaders' last phases
}

// ------------------------------------------------------ basic cycle steps
// One colour of four-colour Gauss-Seidel: colour(i,j) = (i mod 2) + 2 (j mod 2).
// s = b; s -= A_d u_d for d = SW, S, SE, W, E, NW, N, NE; u = s / A_O.
template <typename T, bool NINE>
__device__ __forceinline__ T gs_point(const Lev<T> &L, size_t p)
{
    const size_t ld = L.ld;
    const T *u = L.u;
    T s = L.b[p];
    if (NINE) s -= L.SW[p] * u[p - ld - 1];
    s -= L.S[p] * u[p - ld];
    if (NINE) s -= L.NW[p + 1 - ld] * u[p - ld + 1];
    s -= L.W[p] * u[p - 1];
    s -= L.W[p + 1] * u[p + 1];
    if (NINE) s -= L.NW[p] * u[p + ld - 1];
    s -= L.S[p + ld] * u[p + ld];
    if (NINE) s -= L.SW[p + ld + 1] * u[p + ld + 1];
    return s / L.O[p];
}

template <typename T, bool NINE>
static __global__ void k_gs_colour(Lev<T> L, int colour, const int *stop)
{
    if (stopped(stop)) return;
    const int i = ((colour & 1) ? 1 : 2) + 2 * (int)(blockIdx.x * blockDim.x + threadIdx.x);
    const int j = ((colour >> 1) ? 1 : 2) + 2 * (int)(blockIdx.y * blockDim.y + threadIdx.y);
    if (i > L.n || j > L.n) return;
    const size_t p = (size_t)j * L.ld + i;
    L.u[p] = gs_point<T, NINE>(L, p);
}

// r = b - A u, the centre term last.
template <typename T, bool NINE>
__device__ __forceinline__ T residual_point(const Lev<T> &L, const T *u, size_t p)
{
    const size_t ld = L.ld;
    T s = L.b[p];
    if (NINE) s -= L.SW[p] * u[p - ld - 1];
    s -= L.S[p] * u[p - ld];
    if (NINE) s -= L.NW[p + 1 - ld] * u[p - ld + 1];
    s -= L.W[p] * u[p - 1];
    s -= L.W[p + 1] * u[p + 1];
    if (NINE) s -= L.NW[p] * u[p + ld - 1];
    s -= L.S[p + ld] * u[p + ld];
    if (NINE) s -= L.SW[p + ld + 1] * u[p + ld + 1];
    s -= L.O[p] * u[p];
    return s;
}

template <typename T, bool NINE>
static __global__ void k_residual(Lev<T> L, const int *stop)
{
    if (stopped(stop)) return;
    const int i = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int j = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    if (i > L.n || j > L.n) return;
    const size_t p = (size_t)j * L.ld + i;
    L.r[p] = residual_point<T, NINE>(L, L.u, p);
}

// b_c(I,J) = P^T r in the term order of Fig. restrict_kernel; u_c = 0.
template <typename T>
static __global__ void k_restrict(const T *__restrict__ r, int ldf, Wts<T> C, Lev<T> Cl, const int *stop)
{
    if (stopped(stop)) return;
    const int I = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int J = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    if (I > Cl.n || J > Cl.n) return;
    const size_t c = (size_t)J * C.ld + I;
    const size_t f = (size_t)(2 * J) * ldf + 2 * I;
    const size_t cn = c + C.ld;
    T s = C.at(LNE, c) * r[f - ldf - 1];
    s = s + C.at(LA, c) * r[f - ldf];
    s = s + C.at(LNW, c + 1) * r[f - ldf + 1];
    s = s + C.at(LR, c) * r[f - 1];
    s = s + r[f];
    s = s + C.at(LL, c + 1) * r[f + 1];
    s = s + C.at(LSE, cn) * r[f + ldf - 1];
    s = s + C.at(LB, cn) * r[f + ldf];
    s = s + C.at(LSW, cn + 1) * r[f + ldf + 1];
    Cl.b[c] = s;
    Cl.u[c] = (T)0;
}

// Correction e = P e_c at fine (i,j); e_c is zero on the ring.
template <typename T>
__device__ __forceinline__ T interp_point(const Wts<T> &C, const T *ec, int i, int j)
{
    const int ldc = C.ld;
    if (!(i & 1) && !(j & 1)) return ec[(size_t)(j >> 1) * ldc + (i >> 1)];
    if ((i & 1) && !(j & 1)) {
        const size_t c = (size_t)(j >> 1) * ldc + ((i + 1) >> 1);
        return C.at(LL, c) * ec[c - 1] + C.at(LR, c) * ec[c];
    }
    if (!(i & 1)) {
        const size_t c = (size_t)((j + 1) >> 1) * ldc + (i >> 1);
        return C.at(LB, c) * ec[c - ldc] + C.at(LA, c) * ec[c];
    }
    const size_t c = (size_t)((j + 1) >> 1) * ldc + ((i + 1) >> 1);
    T e = C.at(LSW, c) * ec[c - ldc - 1] + C.at(LSE, c) * ec[c - ldc];
    e = e + C.at(LNW, c) * ec[c - 1];
    e = e + C.at(LNE, c) * ec[c];
    return e;
}

// u += P e_c by coarse cells: thread (I, J) takes the fine points
// (2I-1, 2J-1), (2I, 2J-1), (2I-1, 2J), (2I, 2J), I, J = 1 .. nc+1, whose
// terms all use the weights and e_c around coarse index c = J ldc + I (the
// expressions of interp_point), so a wave runs no divergent paths; fine
// points on the ring (column or row n+1) are skipped.
template <typename T>
static __global__ void k_interp_add(Lev<T> L, Wts<T> C, const T *__restrict__ ec, const int *stop)
{
    if (stopped(stop)) return;
    const int I = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int J = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    const int n = L.n, nc = (n - 1) / 2;
    if (I > nc + 1 || J > nc + 1) return;
    const int ldc = C.ld;
    const size_t c = (size_t)J * ldc + I;
    const T e00 = ec[c], e01 = ec[c - 1], e10 = ec[c - ldc], e11 = ec[c - ldc - 1];
    const size_t p = (size_t)(2 * J - 1) * L.ld + (2 * I - 1);   // the odd-odd point
    const bool east = 2 * I <= n, north = 2 * J <= n;
    {
        T e = C.at(LSW, c) * e11 + C.at(LSE, c) * e10;
        e = e + C.at(LNW, c) * e01;
        e = e + C.at(LNE, c) * e00;
        L.u[p] = L.u[p] + e;
    }
    if (east) L.u[p + 1] = L.u[p + 1] + (C.at(LB, c) * e10 + C.at(LA, c) * e00);
    if (north) L.u[p + L.ld] = L.u[p + L.ld] + (C.at(LL, c) * e01 + C.at(LR, c) * e00);
    if (east && north) L.u[p + L.ld + 1] = L.u[p + L.ld + 1] + e00;
}

// k_interp_add over the coarse cells of fine level F.
template <typename T>
static inline void launch_interp_add(const Lev<T> &F, const Wts<T> &C, const T *ec, const int *stop, hipStream_t st)
{
    const int cells = (F.n - 1) / 2 + 1;
    const dim3 blk(64, 4), grid((cells + 63) / 64, (cells + 3) / 4);
    hipLaunchKernelGGL((k_interp_add<T>), grid, blk, 0, st, F, C, ec, stop);
}

// ------------------------------------------------------------ reductions
// Wave64 + LDS block reduction of a double (up to 16 waves) through 16
// doubles of LDS at `part`; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *part)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) part[wid] = v;
    __syncthreads();
    if (wid == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        v = lane < nw ? part[lane] : 0.0;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    }
    return v;
}

__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double part[16];
    return block_sum(v, part);
}

// Per-block partial sums of squares of the residual (r_mode = 1: recompute
// b - A u; 0: of the array x itself) over the interior, grid-stride over rows.
template <typename T, bool NINE, bool RES>
static __global__ void k_sumsq_partial(Lev<T> L, const T *__restrict__ x, double *__restrict__ part,
                                const int *stop)
{
    if (stopped(stop)) return;
    double acc = 0.0;
    const int n = L.n;
    for (int j = 1 + blockIdx.x; j <= n; j += gridDim.x) {
        for (int i = 1 + threadIdx.x; i <= n; i += blockDim.x) {
            const size_t p = (size_t)j * L.ld + i;
            const double v = RES ? (double)residual_point<T, NINE>(L, L.u, p) : (double)x[p];
            acc += v * v;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// Partial sums of s_p^2 with s_p = |b_p| + sum_d |A_d(p)| |x_(p+d)| (the
// nine entries of the row, centre included): eps * sqrt(sum) / ||b|| bounds
// the relative residual that rounding the exact solution to FP64 can leave,
// the floor below which no FP64 vector's residual reliably goes.  An estimate
// only, summed in plain FP64.
template <bool NINE>
static __global__ void k_floor_partial(Lev<double> L, const double *__restrict__ B, const double *__restrict__ X,
                                       double *__restrict__ part)
{
    double acc = 0.0;
    const int n = L.n;
    const size_t ld = L.ld;
    for (int j = 1 + blockIdx.x; j <= n; j += gridDim.x) {
        for (int i = 1 + threadIdx.x; i <= n; i += blockDim.x) {
            const size_t p = (size_t)j * ld + i;
            double s = fabs(B[p]);
            s += fabs(L.S[p]) * fabs(X[p - ld]) + fabs(L.W[p]) * fabs(X[p - 1]);
            s += fabs(L.O[p]) * fabs(X[p]);
            s += fabs(L.W[p + 1]) * fabs(X[p + 1]) + fabs(L.S[p + ld]) * fabs(X[p + ld]);
            if (NINE) {
                s += fabs(L.SW[p]) * fabs(X[p - ld - 1]) + fabs(L.NW[p + 1 - ld]) * fabs(X[p - ld + 1]);
                s += fabs(L.NW[p]) * fabs(X[p + ld - 1]) + fabs(L.SW[p + ld + 1]) * fabs(X[p + ld + 1]);
            }
            acc += s * s;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// Several right-hand sides in one launch (block solves): the launch serves
// those whose mode[] equals `want`; right-hand side z's level-0 u, b are kl
// elements after the first's, its B, XH, XL planes kx after, its partial sums
// kpart doubles, scalars kscal doubles, history khist doubles and (count, stop)
// pair kcnt ints after.
struct RhsFan {
    int nrhs;
    const int *mode;
    int want;
    size_t kl, kx;
    int kpart, kscal, khist, kcnt;
};

// Final sum of the partials (fixed order) -> out[0].  With `hist` given (and
// the solve not stopped), this also records rel = sqrt(sum)/bnorm[0] into hist[*count], advances the count,
// and raises *stop: 1 once rel <= tol, 2 if rel is not finite or exceeds
// 1e3 times the initial relative residual bnorm[1], 3 when maxc entries exist,
// 4 once rel <= refine (refine > 0): the solve switches to refinement.
__device__ __forceinline__ void sumsq_final_body(const double *__restrict__ part, int np, double *__restrict__ out,
                                                 double *hist, int *count, int *stop, const double *bnorm,
                                                 double tol, int maxc, double refine)
{
    double v = 0.0;
    for (int t = threadIdx.x; t < np; t += blockDim.x) v += part[t];
    v = block_sum(v);
    if (threadIdx.x == 0) {
        out[0] = v;
        if (hist) {
            const int k = *count;
            const double rel = sqrt(v) / bnorm[0];
            hist[k] = rel;
            *count = k + 1;
            int s = 0;
            if (rel <= tol) s = 1;
            else if (!isfinite(rel) || rel > 1e3 * bnorm[1]) s = 2;
            else if (k + 1 >= maxc) s = 3;
            else if (refine > 0.0 && rel <= refine) s = 4;
            if (s) *stop = s;
        }
    }
}

static __global__ void k_sumsq_final(const double *__restrict__ part, int np, double *__restrict__ out,
                              double *hist, int *count, int *stop, const double *bnorm,
                              double tol, int maxc, double refine)
{
    if (hist && stopped(stop)) return;   // a finished solve records nothing more
    sumsq_final_body(part, np, out, hist, count, stop, bnorm, tol, maxc, refine);
}

// The same for the right-hand sides F selects (one workgroup each): out and
// bnorm are the first right-hand side's, count its (count, stop) pair.
static __global__ void k_sumsq_final_fan(const double *__restrict__ part, int np, double *out, double *hist,
                                         int *count, const double *bnorm, double tol, int maxc, double refine,
                                         RhsFan F)
{
    const int z = blockIdx.x;
    int *cz = count + z * F.kcnt;
    if (F.mode[z] != F.want || stopped(cz + 1)) return;
    sumsq_final_body(part + (size_t)z * F.kpart, np, out + z * F.kscal, hist + (size_t)z * F.khist, cz, cz + 1,
                     bnorm + z * F.kscal, tol, maxc, refine);
}

// ---------------------------------------------------- layout conversions
// [n][n] user array <-> padded level array.
template <typename TI, typename TO>
static __global__ void k_pack_in(const TI *__restrict__ src, int n, TO *__restrict__ dst, int ld)
{
    const int i = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int j = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    if (i > n || j > n) return;
    dst[(size_t)j * ld + i] = (TO)src[(size_t)(j - 1) * n + (i - 1)];
}

template <typename TI, typename TO>
static __global__ void k_pack_out(const TI *__restrict__ src, int ld, int n, TO *__restrict__ dst)
{
    const int i = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int j = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    if (i > n || j > n) return;
    dst[(size_t)(j - 1) * n + (i - 1)] = (TO)src[(size_t)j * ld + i];
}

// Rounded copy of a padded array (the FP32 hierarchy from the FP64 set-up).
static __global__ void k_round_f32(const double *__restrict__ src, float *__restrict__ dst, size_t count)
{
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < count;
         t += (size_t)gridDim.x * blockDim.x)
        dst[t] = (float)src[t];
}

// Up to ROUND_MAX arrays rounded to FP32 in one launch (a hierarchy's
// planes): blockIdx.y selects the array.
constexpr int ROUND_MAX = 96;
struct RoundList {
    int n;
    const double *src[ROUND_MAX];
    float *dst[ROUND_MAX];
    size_t count[ROUND_MAX];
};

static __global__ void k_round_f32_list(RoundList R)
{
    const int a = blockIdx.y;
    if (a >= R.n) return;
    const double *__restrict__ src = R.src[a];
    float *__restrict__ dst = R.dst[a];
    const size_t count = R.count[a];
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < count;
         t += (size_t)gridDim.x * blockDim.x)
        dst[t] = (float)src[t];
}

// -------------------------------------------- FP64 iterative refinement
// Maximum over the block (up to 16 waves); result valid in thread 0.
__device__ __forceinline__ double block_max(double m)
{
    __shared__ double sm[16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_down(m, o, 64));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, sm[w]);
    return m;
}

// Largest of np partial maxima of |r| -> out[0] (a maximum: the same value in
// any order of reduction).
static __global__ void k_absmax_final(const double *__restrict__ part, int np, double *__restrict__ out,
                               const int *stop)
{
    if (stopped(stop)) return;
    double m = 0.0;
    for (int t = threadIdx.x; t < np; t += blockDim.x) m = fmax(m, part[t]);
    m = block_max(m);
    if (threadIdx.x == 0) out[0] = m;
}

// Exponent e of the scale 2^e: the least power of two >= rmax (1 for rmax = 0).
__device__ __forceinline__ int ir_exponent(double rmax)
{
    int e = 0;
    const double fr = frexp(rmax, &e);  // rmax = fr 2^e, fr in [1/2, 1)
    if (fr == 0.5) e -= 1;
    if (fr == 0.0) e = 0;
    return e;
}

// s = the smallest power of two >= ||r||_inf (1 if r = 0); the FP32 right-hand
// side is fl32(r / s) (an exact scaling, then one rounding) and u32 = 0.
static __global__ void k_ir_scale(Lev<double> L, Lev<float> F, const double *__restrict__ rmax,
                           double *__restrict__ scale, const int *stop)
{
    if (stopped(stop)) return;
    const int e = ir_exponent(*rmax);
    const double inv = ldexp(1.0, -e);
    const int i = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int j = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    if (i == 1 && j == 1) scale[0] = ldexp(1.0, e);
    if (i > L.n || j > L.n) return;
    const size_t p = (size_t)j * L.ld + i;
    F.b[p] = (float)(L.r[p] * inv);
    F.u[p] = 0.0f;
}

// ------------------------------------------------ double-FP64 iterate
__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e)
{
    const double x = a + b, z = x - a;
    s = x;
    e = (a - (x - z)) + (b - z);
}

// Accurate residual r = B - A (XH + XL) (XL nullable) on the fine level: the
// plain residual's terms in its order (SW, S, SE, W, E, NW, N, NE, centre),
// each product split into value and exact error by fma, each subtraction by
// TwoSum, the errors summed apart, then the XL products, one final rounding.
// MODE 0: sum of squares only; 1: also r -> rout; 2: also r -> L.b and 0 -> L.u
// (the next refinement cycle starts from zero on the right-hand side r).


// Row block rb of nrb (rows 1 + rb, 1 + rb + nrb, ...): the sum of squares of
// r into part[rb] and, with MODE 1 (the refinement of the FP32 cycle, which
// scales r by its largest magnitude next), max |r| into part[nrb + rb].
template <bool NINE, int MODE>
__device__ __forceinline__ void resid_dd_rows(Lev<double> L, const double *__restrict__ B,
                                              const double *__restrict__ XH, const double *__restrict__ XL,
                                              double *__restrict__ rout, double *__restrict__ part, int rb, int nrb)
{
    const size_t ld = L.ld;
    const int n = L.n;
    double acc = 0.0, mx = 0.0;
    for (int j = 1 + rb; j <= n; j += nrb) {
        for (int i = 1 + threadIdx.x; i <= n; i += blockDim.x) {
            const size_t p = (size_t)j * ld + i;
            double a[9];
            size_t q[9] = {p - ld - 1, p - ld, p - ld + 1, p - 1, p + 1, p + ld - 1, p + ld, p + ld + 1, p};
            a[0] = NINE ? L.SW[p] : 0.0;
            a[1] = L.S[p];
            a[2] = NINE ? L.NW[p + 1 - ld] : 0.0;
            a[3] = L.W[p];
            a[4] = L.W[p + 1];
            a[5] = NINE ? L.NW[p] : 0.0;
            a[6] = L.S[p + ld];
            a[7] = NINE ? L.SW[p + ld + 1] : 0.0;
            a[8] = L.O[p];
            double s = B[p], c = 0.0, ns, se;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                if (!NINE && (t == 0 || t == 2 || t == 5 || t == 7)) continue;
                const double x = XH[q[t]];
                const double pr = a[t] * x;
                const double pe = fma(a[t], x, -pr);
                two_sum(s, -pr, ns, se);
                s = ns;
                c = c + (se - pe);
            }
            if (XL) {
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    if (!NINE && (t == 0 || t == 2 || t == 5 || t == 7)) continue;
                    two_sum(s, -(a[t] * XL[q[t]]), ns, se);
                    s = ns;
                    c = c + se;
                }
            }
            const double r = s + c;
            if (MODE == 1) {
                rout[p] = r;
                mx = fmax(mx, fabs(r));
            }
            if (MODE == 2) {
                L.b[p] = r;
                L.u[p] = 0.0;
            }
            acc += r * r;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) part[rb] = acc;
    if (MODE == 1) {
        mx = block_max(mx);
        if (threadIdx.x == 0) part[nrb + rb] = mx;
    }
}

template <bool NINE, int MODE>
static __global__ void k_resid_dd(Lev<double> L, const double *__restrict__ B, const double *__restrict__ XH,
                           const double *__restrict__ XL, double *__restrict__ rout,
                           double *__restrict__ part, const int *stop)
{
    if (stopped(stop)) return;
    resid_dd_rows<NINE, MODE>(L, B, XH, XL, rout, part, blockIdx.x, gridDim.x);
}

// The same for the right-hand sides F selects: work item w serves right-hand
// side w % nrhs and row block w / nrhs.  Consecutive workgroups are dealt
// round-robin to the 8 XCDs, so w regroups them (grids that are a multiple of
// 8) to give each XCD a contiguous run: the right-hand sides of a row block run
// side by side on one XCD and share its operator rows through that L2.
template <bool NINE, int MODE>
static __global__ void k_resid_dd_fan(Lev<double> L, const double *__restrict__ B, const double *__restrict__ XH,
                                      const double *__restrict__ XL, double *__restrict__ part, const int *stop,
                                      RhsFan F)
{
    const int g = gridDim.x;
    const int w = (g & 7) ? (int)blockIdx.x : (int)(blockIdx.x & 7) * (g >> 3) + (int)(blockIdx.x >> 3);
    const int z = w % F.nrhs;
    if (F.mode[z] != F.want || stopped(stop + z * F.kcnt)) return;
    L.u += z * F.kl;
    L.b += z * F.kl;
    resid_dd_rows<NINE, MODE>(L, B + z * F.kx, XH + z * F.kx, XL ? XL + z * F.kx : XL, nullptr,
                              part + (size_t)z * F.kpart, w / F.nrhs, g / F.nrhs);
}

// (xh, xl) += d: TwoSum, add the low part, renormalise with Dekker's fast
// TwoSum.
__device__ __forceinline__ void dd_add_point(double *XH, double *XL, size_t p, double d)
{
    double s, e;
    two_sum(XH[p], d, s, e);
    e = e + XL[p];
    const double hi = s + e;
    XL[p] = e - (hi - s);
    XH[p] = hi;
}

// (XH, XL) += d in double-FP64 with d = L.u (FP64 inner cycle) or
// d = scale * (double)U32 (FP32 inner cycle): TwoSum, add the low part,
// renormalise with Dekker's fast TwoSum.
__device__ __forceinline__ void dd_update_point(const Lev<double> &L, double *__restrict__ XH,
                                                double *__restrict__ XL, const float *__restrict__ U32,
                                                const double *__restrict__ scale)
{
    const int i = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    const int j = 1 + blockIdx.y * blockDim.y + threadIdx.y;
    if (i > L.n || j > L.n) return;
    const size_t p = (size_t)j * L.ld + i;
    dd_add_point(XH, XL, p, U32 ? scale[0] * (double)U32[p] : L.u[p]);
}

static __global__ void k_dd_update(Lev<double> L, double *__restrict__ XH, double *__restrict__ XL,
                            const float *__restrict__ U32, const double *__restrict__ scale,
                            const int *stop)
{
    if (stopped(stop)) return;
    dd_update_point(L, XH, XL, U32, scale);
}

// FP64 inner cycle, the right-hand sides F selects (blockIdx.z).
static __global__ void k_dd_update_fan(Lev<double> L, double *__restrict__ XH, double *__restrict__ XL,
                                       const int *stop, RhsFan F)
{
    const int z = blockIdx.z;
    if (F.mode[z] != F.want || stopped(stop + z * F.kcnt)) return;
    L.u += z * F.kl;
    dd_update_point(L, XH + z * F.kx, XL + z * F.kx, nullptr, nullptr);
}

}  // namespace bmg
