// Fused passes as streams of single waves.
//
// A wave owns a strip of 128 grid columns, two neighbours (even, odd) per lane,
// and a block of rows, and streams upward through it two rows at a time like
// the workgroups of bmg_fused.hpp: the same row pipeline, warm-up rows, halo
// columns and expressions, so the same results to the bit.  What differs is
// where the values live.  The iterate, the right-hand side and the couplings
// read in their own column (O, S) stay in registers, in a ring of rows whose
// slots are compile-time constants (the step loop is unrolled over one turn of
// the ring, so nothing shifts); a neighbour in the other lane comes by a
// one-lane wave shift; W, SW and NW, read at the next column too, sit in an LDS
// ring that only this wave touches.  So no phase waits at a barrier, no value
// of the iterate goes through LDS, and every lane has a point to update in
// every colour phase (with one column per lane half of them idle).
//
// Measured in a 4095^2 solve (FP64, V(2,1)), against the workgroup passes:
// nine-point 2047^2 pre 142 -> 81 us, post 97 -> 71, 1023^2 66 -> 32 and
// 34 -> 25; the cross-cycle pass of the fine level 444 -> 295, 1.48 GB at 5.0
// TB/s (a copy reaches 4.9).  The 2047^2 passes are bound by
// memory: 452 MB for the pre pass, 5 TB/s, while both neighbours of a tile
// streamed the same way (91 us); streaming every other row of tiles downward
// lets two tiles share the rows at their border.
//
// The ring holds two rows more than a step's window: the rows of the next step
// are requested straight into their slots while this step computes.  Points
// on the grid's ring, and beyond it, carry zero couplings, b = 0 and O = 1, so
// that the update leaves them at zero without a test.
#pragma once

#include "bmg_fused.hpp"

namespace bmg {

constexpr int WAVE_COLS = 128;

// Stencils: five-point, nine-point (both symmetric, half of the couplings
// stored), and five-point nonsymmetric, all four couplings of a row stored
// with it: S and W in their planes, E in the one of SW and N in the one of NW.
enum : int { FIVE = 0, NINE = 1, FIVE_NS = 2 };

// Tiles of a wave-stream pass over n^2 points for nrhs right-hand sides, hx halo
// columns on each side of a strip, of `rows` rows (0: chosen).  An FP64 pre pass
// takes more than 256 registers, one wave per SIMD: the height is the least that
// leaves all tiles in one round of 1024.  Tiles of half that height (a round of
// 2048, which FP32 and the post passes could hold) re-read more rows: nine-point
// FP64, two sweeps before and one after, 2047^2 79 + 69 us against 87 + 78, 1023^2
// 29 + 18 against 40 + 24, the cross-cycle pass of 4095^2 299 against 324; in FP32
// 2047^2 42 + 29 either way, 1023^2 20.6 + 11.8 against 20.8 + 10.8.
constexpr int WAVE_SLOTS = 1024;
inline TileGeo wave_geo(int n, int hx, int rows, int nrhs)
{
    const int useful = WAVE_COLS - 2 * hx, strips = (n + useful) / useful;
    if (rows <= 0) {
        const int blocks = std::max(1, WAVE_SLOTS / (strips * nrhs));
        rows = std::max(2, ((n + blocks - 1) / blocks + 1) & ~1);
    }
    TileGeo g;
    g.hx = hx;
    g.ht = std::max(2, std::min(rows, (n + 2) & ~1));
    g.tiles_x = strips;
    g.ntiles = strips * ((n + g.ht - 1) / g.ht);
    g.nrhs = nrhs;
    return g;
}

// Value of the lane to the west (lane 0: zero) or east (lane 63: zero).
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename T>
__device__ __forceinline__ T from_west(T v) { return lane_shift<0x138>(v); }   // wave_shr:1
template <typename T>
__device__ __forceinline__ T from_east(T v) { return lane_shift<0x130>(v); }   // wave_shl:1

// Orders this wave's LDS accesses (its lanes read what their neighbours wrote;
// to the compiler those are unrelated addresses).  No instruction.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <typename T>
struct Pair {
    typedef T vec __attribute__((ext_vector_type(2)));
};

// LDS ring of a wave: W and on nine-point levels SW, NW (FIVE_NS: E), RX rows of
// 128 columns (and two elements that the last lane's read of "the next column"
// may touch).
template <typename T, int KIND, int NU>
struct WaveLds {
    static constexpr int RX = 2 * NU + 6;
    T W[RX * WAVE_COLS], SW[KIND != FIVE ? RX * WAVE_COLS : 0], NW[KIND == NINE ? RX * WAVE_COLS : 0], pad[2];
};

// What both passes share: geometry, the ring and the point update.  A tile is
// streamed upward (DIR = 1) or downward (DIR = -1): the colours' order, even
// rows before odd ones, is the same seen from either side.  Slot of row
// e + DIR d at turn M of the unrolled loop (e = es + 2 M DIR mod RX).
template <typename T, int KIND, int NU, int DIR>
struct WaveTile {
    static constexpr int RX = 2 * NU + 6;
    using V = typename Pair<T>::vec;
    template <int M>
    static constexpr int at(int d) { return ((2 * M + d) % RX + RX) % RX; }

    T u[RX][2], b[RX][2], O[RX][2], S[RX][2];
    T N[KIND == FIVE_NS ? RX : 1][2];
    T *sW, *sSW, *sNW;         // this lane's pair in ring row 0
    int n, ld, i0, i0c, y0, y1;
    bool in0, in1, own;        // columns interior, pair owned

    __device__ __forceinline__ void place(const Lev<T> &L, const TileGeo &G, int tid, WaveLds<T, KIND, NU> &lds)
    {
        n = L.n;
        ld = L.ld;
        const int lane = threadIdx.x, useful = WAVE_COLS - 2 * G.hx;
        const int tx = tid % G.tiles_x, ty = tid / G.tiles_x;
        const int xo = tx * useful;                 // first owned column (0: the ring)
        i0 = xo - G.hx + 2 * lane;
        i0c = i0 >= 0 && i0 <= n + 1 ? i0 : n + 1;   // beyond the grid: the ring and the zeros past it
        in0 = i0 >= 1 && i0 <= n;
        in1 = i0 + 1 >= 1 && i0 + 1 <= n;
        own = i0 >= xo && i0 < xo + useful && i0 < n;
        y0 = 1 + ty * G.ht;
        y1 = min(y0 + G.ht, n + 1);
        sW = lds.W + 2 * lane;
        sSW = lds.SW + 2 * lane;
        sNW = lds.NW + 2 * lane;
    }
    __device__ __forceinline__ int rowc(int row) const { return row >= 0 && row <= n + 1 ? row : n + 1; }
    template <typename E>
    __device__ __forceinline__ typename Pair<E>::vec load(const E *a, int row) const
    {
        return *reinterpret_cast<const typename Pair<E>::vec *>(a + (size_t)rowc(row) * ld + i0c);
    }
    template <typename E>
    __device__ __forceinline__ void store(E *a, int row, E v0, E v1) const
    {
        E *p = a + (size_t)row * ld + i0;
        if (i0 > 0) *reinterpret_cast<typename Pair<E>::vec *>(p) = typename Pair<E>::vec{v0, v1};
        else p[1] = v1;
    }
    // the couplings of a row that go through LDS
    struct Couplings {
        V w, sw, nw;
    };
    __device__ __forceinline__ Couplings couplings(const Lev<T> &L, int row) const
    {
        Couplings c;
        c.w = load(L.W, row);
        if constexpr (KIND != FIVE) c.sw = load(L.SW, row);
        if constexpr (KIND == NINE) c.nw = load(L.NW, row);
        return c;
    }
    __device__ __forceinline__ void next_couplings(const Lev<T> &L, int e, Couplings (&c)[2]) const
    {
        c[0] = couplings(L, e);
        c[1] = couplings(L, e + DIR);
    }
    template <int SL>
    __device__ __forceinline__ void put_couplings(const Couplings &c)
    {
        *reinterpret_cast<V *>(sW + SL * WAVE_COLS) = c.w;
        if constexpr (KIND != FIVE) *reinterpret_cast<V *>(sSW + SL * WAVE_COLS) = c.sw;
        if constexpr (KIND == NINE) *reinterpret_cast<V *>(sNW + SL * WAVE_COLS) = c.nw;
    }
    // b, O, S of a row into its slot
    template <int SL, bool WITH_B = true>
    __device__ __forceinline__ void request(const Lev<T> &L, int row)
    {
        if constexpr (WITH_B) {
            const V vb = load(L.b, row);
            b[SL][0] = vb.x; b[SL][1] = vb.y;
        }
        const V vo = load(L.O, row), vs = load(L.S, row);
        O[SL][0] = vo.x; O[SL][1] = vo.y;
        S[SL][0] = vs.x; S[SL][1] = vs.y;
        if constexpr (KIND == FIVE_NS) {
            const V vn = load(L.NW, row);
            N[SL][0] = vn.x; N[SL][1] = vn.y;
        }
    }
    // a row that has arrived: O = 1 where there is no equation
    template <int SL>
    __device__ __forceinline__ void arrived(int row)
    {
        const bool ok = row >= 1 && row <= n;
        O[SL][0] = ok && in0 ? O[SL][0] : (T)1;
        O[SL][1] = ok && in1 ? O[SL][1] : (T)1;
    }
    // b minus the couplings at column C of the row in slot S0 (SD below, SU
    // above), in the order of gs_lds
    template <int C, int SD, int S0, int SU>
    __device__ __forceinline__ T offdiag() const
    {
        if constexpr (KIND != NINE) {
            const T uw = C ? u[S0][0] : from_west(u[S0][1]), ue = C ? from_east(u[S0][0]) : u[S0][1];
            T s = b[S0][C];
            s -= S[S0][C] * u[SD][C];
            s -= sW[S0 * WAVE_COLS + C] * uw;
            s -= (KIND == FIVE_NS ? sSW[S0 * WAVE_COLS + C] : sW[S0 * WAVE_COLS + C + 1]) * ue;
            if constexpr (KIND == FIVE_NS) s -= N[S0][C] * u[SU][C];
            else s -= S[SU][C] * u[SU][C];
            return s;
        }
        const T uwd = C ? u[SD][0] : from_west(u[SD][1]), ued = C ? from_east(u[SD][0]) : u[SD][1];
        const T uw0 = C ? u[S0][0] : from_west(u[S0][1]), ue0 = C ? from_east(u[S0][0]) : u[S0][1];
        const T uwu = C ? u[SU][0] : from_west(u[SU][1]), ueu = C ? from_east(u[SU][0]) : u[SU][1];
        T s = b[S0][C];
        s -= sSW[S0 * WAVE_COLS + C] * uwd;
        s -= S[S0][C] * u[SD][C];
        s -= sNW[SD * WAVE_COLS + C + 1] * ued;
        s -= sW[S0 * WAVE_COLS + C] * uw0;
        s -= sW[S0 * WAVE_COLS + C + 1] * ue0;
        s -= sNW[S0 * WAVE_COLS + C] * uwu;
        s -= S[SU][C] * u[SU][C];
        s -= sSW[SU * WAVE_COLS + C + 1] * ueu;
        return s;
    }
    template <int M, int D, int C>
    __device__ __forceinline__ void relax()
    {
        constexpr int SD = at<M>(D - DIR), S0 = at<M>(D), SU = at<M>(D + DIR);
        u[S0][C] = offdiag<C, SD, S0, SU>() / O[S0][C];
    }
    template <int M, int D, int C>
    __device__ __forceinline__ T resid() const
    {
        constexpr int SD = at<M>(D - DIR), S0 = at<M>(D), SU = at<M>(D + DIR);
        T s = offdiag<C, SD, S0, SU>();
        s -= O[S0][C] * u[S0][C];
        return s;
    }
    // square of the accurate residual at column C of the row in slot S0 (the
    // terms of post_tile; FIVE_NS: of the plain residual)
    template <int C, int SD, int S0, int SU>
    __device__ __forceinline__ double resid2() const
    {
        if constexpr (KIND == FIVE_NS) {
            T s = offdiag<C, SD, S0, SU>();
            s -= O[S0][C] * u[S0][C];
            return s * s;
        }
        constexpr int N = KIND == NINE ? 9 : 5;
        double a[N], x[N];
        int q = 0;
        auto term = [&](double ai, double xi) {
            a[q] = ai;
            x[q++] = xi;
        };
        if constexpr (KIND == NINE) term(sSW[S0 * WAVE_COLS + C], C ? u[SD][0] : from_west(u[SD][1]));
        term(S[S0][C], u[SD][C]);
        if constexpr (KIND == NINE) term(sNW[SD * WAVE_COLS + C + 1], C ? from_east(u[SD][0]) : u[SD][1]);
        term(sW[S0 * WAVE_COLS + C], C ? u[S0][0] : from_west(u[S0][1]));
        term(sW[S0 * WAVE_COLS + C + 1], C ? from_east(u[S0][0]) : u[S0][1]);
        if constexpr (KIND == NINE) term(sNW[S0 * WAVE_COLS + C], C ? u[SU][0] : from_west(u[SU][1]));
        term(S[SU][C], u[SU][C]);
        if constexpr (KIND == NINE) term(sSW[SU * WAVE_COLS + C + 1], C ? from_east(u[SU][0]) : u[SU][1]);
        term(O[S0][C], u[S0][C]);
        double s = b[S0][C], cc = 0.0, ns, se;
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const double pr = a[t] * x[t];
            const double pe = fma(a[t], x[t], -pr);
            two_sum(s, -pr, ns, se);
            s = ns;
            cc = cc + (se - pe);
        }
        const double r = s + cc;
        return r * r;
    }
    // the owned points of row e + DIR D (in window row D) into the norm's sum
    template <int M, int D>
    __device__ __forceinline__ void norm(int row, double &acc) const
    {
        constexpr int SD = at<M>(D - DIR), S0 = at<M>(D), SU = at<M>(D + DIR);
        const double q0 = resid2<0, SD, S0, SU>(), q1 = resid2<1, SD, S0, SU>();
        if (own && row >= y0 && row < y1) {
            acc += q0;
            acc += q1;
        }
    }
    // sweep s of the step: colours 0, 1 on the even row 2s behind e, then 2, 3
    // on the odd row behind that
    template <int M, int SW_, int END>
    __device__ __forceinline__ void sweeps()
    {
        if constexpr (SW_ < END) {
            relax<M, -2 * SW_, 0>();
            relax<M, -2 * SW_, 1>();
            relax<M, -2 * SW_ - 1, 0>();
            relax<M, -2 * SW_ - 1, 1>();
            sweeps<M, SW_ + 1, END>();
        }
    }
    // the two rows of sweep SW_ are final: the owned ones go out
    template <int M, int SW_ = NU - 1>
    __device__ __forceinline__ void write(T *out, int e) const
    {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row = e - DIR * (2 * SW_ + t);
            if (row < y0 || row >= y1 || !own) continue;
            const T *v = u[at<M>(-2 * SW_ - t)];
            store(out, row, v[0], v[1]);
        }
    }
};

// Tiles of odd rows of tiles stream downward, so that two tiles that share a
// border are there at the same time, both at their start or both at their end,
// and the warm-up rows of one are fetched while the other's L2 still has them.
__device__ __forceinline__ bool wave_up(const TileGeo &G, int tid) { return !((tid / G.tiles_x) & 1); }

// nu sweeps, residual and restriction (results as pre_tile).  zero_u: the
// iterate is known to be zero (a coarse level's first visit in a cycle).  IRIN
// (see IrArgs): b is the scaled FP64 residual, also stored as the FP32
// right-hand side.
template <typename T, int KIND, int NU, int DIR, bool IRIN = false>
struct WavePre : WaveTile<T, KIND, NU, DIR> {
    using B = WaveTile<T, KIND, NU, DIR>;
    using V = typename B::V;
    static constexpr int RX = B::RX;
    T pr0[2], pr1[2];          // residual of the coarse row's f and of the odd row behind it
    T w[8];                    // restriction weights of the next step's coarse row
    bool rest;
    int I, nc;
    Pair<double>::vec res[2];  // IRIN: the FP64 residual of the next step's rows
    const double *r;
    double inv;

    __device__ __forceinline__ void run(const Lev<T> &L, T *__restrict__ uout, const Wts<T> &Cw, const Lev<T> &Cl,
                                        const TileGeo &G, int tid, WaveLds<T, KIND, NU> &lds, bool zero_u,
                                        const IrArgs &ir = {})
    {
        B::place(L, G, tid, lds);
        if constexpr (IRIN) {
            const int ex = ir_exponent(*ir.rmax);
            inv = ldexp(1.0, -ex);
            r = ir.r;
            if (tid == 0 && threadIdx.x == 0) ir.scale[0] = ldexp(1.0, ex);
        }
        nc = Cl.n;
        I = this->i0 >> 1;
        rest = this->own && I >= 1 && I <= nc;
        const int y0 = this->y0, y1 = this->y1;
        // warm-up rows before the owned ones as in pre_tile; the last step
        // restricts the last owned coarse row
        const int es = DIR > 0 ? (y0 - 2 * NU) & ~1 : (y1 + 2 * NU) & ~1;
        const int elast = DIR > 0 ? 2 * ((y1 - 1) >> 1) + 2 * NU + 2 : 2 * ((y0 + 1) >> 1) - 2 * NU - 2;
        // the rows behind es, and the request of es and the next
        fill<-2 * NU - 2>(L, es, zero_u);
        typename B::Couplings c[2];
        B::next_couplings(L, es, c);
        want<0>(L, es, zero_u);
        weights(Cw, (es - DIR * (2 * NU + 2)) >> 1);
        pr0[0] = pr0[1] = pr1[0] = pr1[1] = (T)0;
        for (int e = es; DIR * (elast - e) >= 0; e += DIR * RX)
            turn<0>(L, uout, Cw, Cl, e, elast, zero_u, c);
    }

private:
    template <int D>
    __device__ __forceinline__ void fill(const Lev<T> &L, int es, bool zero_u)
    {
        if constexpr (D < 0) {
            constexpr int SL = B::template at<0>(D);
            const int row = es + DIR * D;
            const V vu = zero_u ? V{(T)0, (T)0} : B::load(L.u, row);
            this->u[SL][0] = vu.x;
            this->u[SL][1] = vu.y;
            B::template request<SL, !IRIN>(L, row);
            if constexpr (IRIN) scaled<SL>(B::load(r, row));
            B::template put_couplings<SL>(B::couplings(L, row));
            B::template arrived<SL>(row);
            fill<D + 1>(L, es, zero_u);
        }
    }
    // request turn M's two rows into their slots
    template <int M>
    __device__ __forceinline__ void want(const Lev<T> &L, int e, bool zero_u)
    {
        constexpr int S0 = B::template at<M>(0), S1 = B::template at<M>(1);
        const V u0 = zero_u ? V{(T)0, (T)0} : B::load(L.u, e), u1 = zero_u ? V{(T)0, (T)0} : B::load(L.u, e + DIR);
        this->u[S0][0] = u0.x; this->u[S0][1] = u0.y;
        this->u[S1][0] = u1.x; this->u[S1][1] = u1.y;
        B::template request<S0, !IRIN>(L, e);
        B::template request<S1, !IRIN>(L, e + DIR);
        if constexpr (IRIN) {
            res[0] = B::load(r, e);
            res[1] = B::load(r, e + DIR);
        }
    }
    template <int SL>
    __device__ __forceinline__ void scaled(Pair<double>::vec v)
    {
        this->b[SL][0] = (T)(v.x * inv);
        this->b[SL][1] = (T)(v.y * inv);
    }
    // every owned row arrives once: keep its FP32 right-hand side
    template <int SL>
    __device__ __forceinline__ void scaled(const Lev<T> &L, Pair<double>::vec v, int row)
    {
        scaled<SL>(v);
        if (this->own && row >= this->y0 && row < this->y1) B::store(L.b, row, this->b[SL][0], this->b[SL][1]);
    }
    __device__ __forceinline__ void weights(const Wts<T> &C, int J)
    {
        const bool ok = J >= 1 && J <= nc;
        const size_t c = (size_t)(ok ? J : 1) * C.ld + (rest ? I : 1), cn = c + C.ld;
        w[0] = C.at(LNE, c);
        w[1] = C.at(LA, c);
        w[2] = C.at(LNW, c + 1);
        w[3] = C.at(LR, c);
        w[4] = C.at(LL, c + 1);
        w[5] = C.at(LSE, cn);
        w[6] = C.at(LB, cn);
        w[7] = C.at(LSW, cn + 1);
    }
    template <int M>
    __device__ __forceinline__ void turn(const Lev<T> &L, T *__restrict__ uout, const Wts<T> &Cw, const Lev<T> &Cl,
                                         int e, int elast, bool zero_u, typename B::Couplings (&c)[2])
    {
        if constexpr (M < RX / 2) {
            if (DIR * (e - elast) > 0) return;
            constexpr int S0 = B::template at<M>(0), S1 = B::template at<M>(1);
            wave_lds_order();
            B::template put_couplings<S0>(c[0]);
            B::template put_couplings<S1>(c[1]);
            wave_lds_order();
            B::template arrived<S0>(e);
            B::template arrived<S1>(e + DIR);
            if constexpr (IRIN) {
                scaled<S0>(L, res[0], e);
                scaled<S1>(L, res[1], e + DIR);
            }
            T wc[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) wc[q] = w[q];
            // the next step's data
            const int en2 = e + 2 * DIR;
            B::next_couplings(L, en2, c);
            want<(M + 1) % (RX / 2)>(L, en2, zero_u);
            weights(Cw, (en2 - DIR * (2 * NU + 2)) >> 1);
            B::template sweeps<M, 0, NU>();
            B::template write<M>(uout, e);
            // residual of the two rows behind the last sweep, restriction of f
            T r0[2], r1[2];
            r0[0] = B::template resid<M, -2 * NU, 0>();
            r0[1] = B::template resid<M, -2 * NU, 1>();
            r1[0] = B::template resid<M, -2 * NU - 1, 0>();
            r1[1] = B::template resid<M, -2 * NU - 1, 1>();
            const int f = e - DIR * (2 * NU + 2), J = f >> 1;
            // rows f - 1 and f + 1: the odd rows of the previous step and of this one
            const T *rd = DIR > 0 ? pr1 : r1, *ru = DIR > 0 ? r1 : pr1;
            const T dw = from_west(rd[1]), mw = from_west(pr0[1]), uw = from_west(ru[1]);
            if (rest && J >= 1 && J <= nc && f >= this->y0 && f < this->y1) {
                const size_t p = (size_t)J * Cw.ld + I;
                T s = wc[0] * dw;
                s = s + wc[1] * rd[0];
                s = s + wc[2] * rd[1];
                s = s + wc[3] * mw;
                s = s + pr0[0];
                s = s + wc[4] * pr0[1];
                s = s + wc[5] * uw;
                s = s + wc[6] * ru[0];
                s = s + wc[7] * ru[1];
                Cl.b[p] = s;
                Cl.u[p] = (T)0;
            }
            pr0[0] = r0[0]; pr0[1] = r0[1];
            pr1[0] = r1[0]; pr1[1] = r1[1];
            turn<M + 1>(L, uout, Cw, Cl, en2, elast, zero_u, c);
        }
    }
};

template <typename T, int KIND, int NU, bool ZU>
__global__ __launch_bounds__(64, 1) void k_pre_wave(Lev<T> L, T *__restrict__ uout, Wts<T> C, Lev<T> Cl, TileGeo G,
                                                    const int *stop)
{
    int tid, k;
    if (!tile_work(G, tid, k)) return;
    if (stopped(stop ? stop + k * G.kstop : stop)) return;
    L.u += k * G.ksf; L.b += k * G.ksf; uout += k * G.ksf;
    Cl.u += k * G.ksc; Cl.b += k * G.ksc;
    __shared__ WaveLds<T, KIND, NU> S;
    if (wave_up(G, tid)) {
        WavePre<T, KIND, NU, 1> P;
        P.run(L, uout, C, Cl, G, tid, S, ZU);
    } else {
        WavePre<T, KIND, NU, -1> P;
        P.run(L, uout, C, Cl, G, tid, S, ZU);
    }
}

// The fine pre pass of an FP32 refinement step (one or two sweeps), at the rate
// of memory: 8191^2, two sweeps, 537 us for 38 bytes per point, 4.7 TB/s (as
// workgroups 631).
template <int NU>
__global__ __launch_bounds__(64, 1) void k_pre_ir_wave(Lev<float> L, float *__restrict__ uout, Wts<float> C,
                                                       Lev<float> Cl, TileGeo G, const int *stop, IrArgs ir)
{
    int tid, k;
    if (!tile_work(G, tid, k)) return;
    if (stopped(stop)) return;
    __shared__ WaveLds<float, false, NU> S;
    if (wave_up(G, tid)) {
        WavePre<float, false, NU, 1, true> P;
        P.run(L, uout, C, Cl, G, tid, S, true, ir);
    } else {
        WavePre<float, false, NU, -1, true> P;
        P.run(L, uout, C, Cl, G, tid, S, true, ir);
    }
}

// A tile whose rows enter as u + P e_c.
template <typename T, int KIND, int NU, int DIR>
struct WaveInterp : WaveTile<T, KIND, NU, DIR> {
    using B = WaveTile<T, KIND, NU, DIR>;
    using V = typename B::V;
    T e0, w[8];                // e_c of row e / 2 at I; the next step's weights
    T en;                      // e_c of the coarse row after it
    int Ic, nc, ldc;

    __device__ __forceinline__ T crow(const T *ec, int J) const
    {
        return ec[(size_t)(J >= 0 && J <= nc + 1 ? J : nc + 1) * ldc + Ic];
    }
    // weights of rows e (even) and e + DIR: LL, LR at (I + 1, J0), LB, LA at
    // (I, J1) and LSW, LSE, LNW, LNE at (I + 1, J1)
    __device__ __forceinline__ void weights(const Wts<T> &C, int e)
    {
        const int J0 = e >> 1, J1 = DIR > 0 ? J0 + 1 : J0;
        const size_t c0 = (size_t)(J0 >= 0 && J0 <= nc + 1 ? J0 : nc + 1) * ldc + Ic;
        const size_t c1 = (size_t)(J1 >= 0 && J1 <= nc + 1 ? J1 : nc + 1) * ldc + Ic;
        w[0] = C.at(LL, c0 + 1);
        w[1] = C.at(LR, c0 + 1);
        w[2] = C.at(LB, c1);
        w[3] = C.at(LA, c1);
        w[4] = C.at(LSW, c1 + 1);
        w[5] = C.at(LSE, c1 + 1);
        w[6] = C.at(LNW, c1 + 1);
        w[7] = C.at(LNE, c1 + 1);
    }
    // u += P e_c on rows e and e + DIR (slots S0, S1); ee, eo: e_c of row e / 2
    // and of the one on the odd row's other side
    template <int S0, int S1>
    __device__ __forceinline__ void correct(int e, T ee, T eo)
    {
        const T eee = from_east(ee), eoe = from_east(eo);
        const T el = DIR > 0 ? ee : eo, ele = DIR > 0 ? eee : eoe;   // below the odd row
        const T eu = DIR > 0 ? eo : ee, eue = DIR > 0 ? eoe : eee;   // above it
        const int n = this->n;
        if (e >= 1 && e <= n) {
            if (this->in0) this->u[S0][0] = this->u[S0][0] + ee;
            if (this->in1) {
                const T c = w[0] * ee + w[1] * eee;
                this->u[S0][1] = this->u[S0][1] + c;
            }
        }
        if (e + DIR >= 1 && e + DIR <= n) {
            if (this->in0) {
                const T c = w[2] * el + w[3] * eu;
                this->u[S1][0] = this->u[S1][0] + c;
            }
            if (this->in1) {
                T c = w[4] * el + w[5] * ele;
                c = c + w[6] * eu;
                c = c + w[7] * eue;
                this->u[S1][1] = this->u[S1][1] + c;
            }
        }
    }
    // place() and the rows behind es, interpolated; es and the next requested
    __device__ __forceinline__ void begin(const Lev<T> &L, const Wts<T> &Cw, const T *ec, int es,
                                          typename B::Couplings (&c)[2])
    {
        e0 = crow(ec, (es - DIR * (2 * NU + 2)) >> 1);
        fill<-2 * NU - 2>(L, Cw, ec, es);
        B::next_couplings(L, es, c);
        want<0>(L, es);
        en = crow(ec, (es >> 1) + DIR);
        weights(Cw, es);
    }
    __device__ __forceinline__ void coarse(const Wts<T> &Cw)
    {
        nc = (this->n - 1) >> 1;
        ldc = Cw.ld;
        Ic = this->i0c >> 1;
    }
    template <int D>
    __device__ __forceinline__ void fill(const Lev<T> &L, const Wts<T> &Cw, const T *ec, int es)
    {
        if constexpr (D < 0) {
            constexpr int S0 = B::template at<0>(D), S1 = B::template at<0>(D + 1);
            const int row = es + DIR * D;
            request_u<S0, S1>(L, row);
            const T e1 = crow(ec, (row >> 1) + DIR);
            weights(Cw, row);
            B::template request<S0>(L, row);
            B::template request<S1>(L, row + DIR);
            B::template put_couplings<S0>(B::couplings(L, row));
            B::template put_couplings<S1>(B::couplings(L, row + DIR));
            correct<S0, S1>(row, e0, e1);
            B::template arrived<S0>(row);
            B::template arrived<S1>(row + DIR);
            e0 = e1;
            fill<D + 2>(L, Cw, ec, es);
        }
    }
    template <int S0, int S1>
    __device__ __forceinline__ void request_u(const Lev<T> &L, int row)
    {
        const V u0 = B::load(L.u, row), u1 = B::load(L.u, row + DIR);
        this->u[S0][0] = u0.x; this->u[S0][1] = u0.y;
        this->u[S1][0] = u1.x; this->u[S1][1] = u1.y;
    }
    template <int M>
    __device__ __forceinline__ void want(const Lev<T> &L, int e)
    {
        constexpr int S0 = B::template at<M>(0), S1 = B::template at<M>(1);
        request_u<S0, S1>(L, e);
        B::template request<S0>(L, e);
        B::template request<S1>(L, e + DIR);
    }
    // the rows of step e take their places, interpolated, and the next step's
    // data is requested
    template <int M>
    __device__ __forceinline__ void enter(const Lev<T> &L, const Wts<T> &Cw, const T *ec, int e,
                                          typename B::Couplings (&c)[2])
    {
        constexpr int S0 = B::template at<M>(0), S1 = B::template at<M>(1);
        B::template arrived<S0>(e);
        B::template arrived<S1>(e + DIR);
        correct<S0, S1>(e, e0, en);
        e0 = en;
        B::next_couplings(L, e + 2 * DIR, c);
        want<(M + 1) % (B::RX / 2)>(L, e + 2 * DIR);
        en = crow(ec, (e >> 1) + 2 * DIR);
        weights(Cw, e + 2 * DIR);
    }
};

__device__ __forceinline__ void wave_sum_to(double acc, double *out)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if (threadIdx.x == 0) *out = acc;
}

// Interpolation and nu sweeps, with NORM also the tile's sum of squares of the
// accurate residual into part[tid] (results as post_tile).
template <typename T, int KIND, int NU, int DIR, bool NORM>
struct WavePost : WaveInterp<T, KIND, NU, DIR> {
    using A = WaveInterp<T, KIND, NU, DIR>;
    using B = typename A::B;
    static constexpr int RX = B::RX;
    double acc;

    __device__ __forceinline__ void run(const Lev<T> &L, T *__restrict__ uout, const Wts<T> &Cw,
                                        const T *__restrict__ ec, const TileGeo &G, int tid,
                                        double *__restrict__ part, WaveLds<T, KIND, NU> &lds)
    {
        B::place(L, G, tid, lds);
        A::coarse(Cw);
        const int y0 = this->y0, y1 = this->y1;
        // the last step writes the last owned row (downward y0, which is odd),
        // with the norm it also has the row beyond it
        const int es = DIR > 0 ? (y0 - 2 * NU + 1) & ~1 : (y1 - 1 + 2 * NU) & ~1;
        const int elast = DIR > 0 ? (y1 - (NORM ? 1 : 2) + 2 * NU) & ~1 : y0 + 1 - 2 * NU;
        typename B::Couplings c[2];
        A::begin(L, Cw, ec, es, c);
        acc = 0.0;
        for (int e = es; DIR * (elast - e) >= 0; e += DIR * RX) turn<0>(L, uout, Cw, ec, e, elast, c);
        if (NORM) wave_sum_to(acc, part + tid);
    }

private:
    template <int M>
    __device__ __forceinline__ void turn(const Lev<T> &L, T *__restrict__ uout, const Wts<T> &Cw,
                                         const T *__restrict__ ec, int e, int elast, typename B::Couplings (&c)[2])
    {
        if constexpr (M < RX / 2) {
            if (DIR * (e - elast) > 0) return;
            wave_lds_order();
            B::template put_couplings<B::template at<M>(0)>(c[0]);
            B::template put_couplings<B::template at<M>(1)>(c[1]);
            wave_lds_order();
            A::template enter<M>(L, Cw, ec, e, c);
            B::template sweeps<M, 0, NU>();
            B::template write<M>(uout, e);
            if constexpr (NORM) {
                B::template norm<M, 1 - 2 * NU>(e + DIR * (1 - 2 * NU), acc);
                B::template norm<M, -2 * NU>(e - DIR * 2 * NU, acc);
            }
            turn<M + 1>(L, uout, Cw, ec, e + 2 * DIR, elast, c);
        }
    }
};

template <typename T, int KIND, int NU, bool NORM>
__global__ __launch_bounds__(64, 1) void k_post_wave(Lev<T> L, T *__restrict__ uout, Wts<T> C,
                                                     const T *__restrict__ ec, TileGeo G, double *__restrict__ part,
                                                     const int *stop)
{
    int tid, k;
    if (!tile_work(G, tid, k)) return;
    if (stopped(stop ? stop + k * G.kstop : stop)) return;
    L.u += k * G.ksf; L.b += k * G.ksf; uout += k * G.ksf;
    ec += k * G.ksc;
    if (NORM) part += k * G.kpart;
    __shared__ WaveLds<T, KIND, NU> S;
    if (wave_up(G, tid)) {
        WavePost<T, KIND, NU, 1, NORM> P;
        P.run(L, uout, C, ec, G, tid, part, S);
    } else {
        WavePost<T, KIND, NU, -1, NORM> P;
        P.run(L, uout, C, ec, G, tid, part, S);
    }
}

// The fine post pass of an FP32 refinement step together with the next step's
// FP64 residual: interpolation and nu sweeps in FP32, (x_hi, x_lo) += s u on
// the rows that come out (IrArgs), and r = B - A (x_hi + x_lo), as k_resid_dd
// forms it, on the rows whose neighbours have come out too, with the tile's
// sum of r^2 in part[tid] and max |r| in part[ntiles + tid].  The FP32
// operator is the FP64 one rounded, so the pass reads only the FP64 one: 89
// bytes per fine point (stencil 24, b and u 8, weights and e_c 9, the pair 32,
// B 8, r 8) where the post pass and the residual take 61 + 64.  Every halo point
// updates its own copy of the pair, so the new pair goes to buffers of its own
// (oh, ol).  Bound by memory: 8191^2, one sweep, 1286 us, 4.6 TB/s, where the
// two passes took 1009 + 948.
template <int NU>
struct WavePostResLds {
    static constexpr int RX = 2 * NU + 6;
    WaveLds<float, false, NU> ring;
    double W[RX * WAVE_COLS + 2];
};

struct PairOut {
    const double *B;
    double *oh, *ol, *r, *part;
};

template <int NU, int DIR>
struct WavePostRes : WaveInterp<float, false, NU, DIR> {
    using A = WaveInterp<float, false, NU, DIR>;
    using B = typename A::B;
    using V = typename A::V;
    using D2 = Pair<double>::vec;
    static constexpr int RX = B::RX;
    double O2[RX][2], S2[RX][2];
    double xh[4][2], xl[4][2];     // the new pair: the two rows a step finalises, the two of the step before
    D2 ph[2], pl[2], pb[2];        // the pair and B of the next step's rows
    D2 w2[2];
    double *sW2, sc, acc, mx;

    __device__ __forceinline__ void run(const Lev<float> &L, const Lev<double> &F, const Wts<float> &Cw,
                                        const float *__restrict__ ec, const IrArgs &ir, const PairOut &out,
                                        const TileGeo &G, int tid, WavePostResLds<NU> &lds)
    {
        B::place(L, G, tid, lds.ring);
        A::coarse(Cw);
        sW2 = lds.W + 2 * threadIdx.x;
        sc = *ir.scale;
        const int y0 = this->y0, y1 = this->y1;
        const int es = DIR > 0 ? (y0 - 2 * NU + 1) & ~1 : (y1 - 1 + 2 * NU) & ~1;
        const int elast = DIR > 0 ? (y1 - 1 + 2 * NU) & ~1 : y0 + 1 - 2 * NU;
        this->e0 = A::crow(ec, (es - DIR * (2 * NU + 2)) >> 1);
        fill64<-2 * NU - 2>(L, F, Cw, ec, es);
        want64<0>(L, F, es);
        pair_rows(ir, out, es);
        this->en = A::crow(ec, (es >> 1) + DIR);
        A::weights(Cw, es);
#pragma unroll
        for (int t = 0; t < 4; ++t) xh[t][0] = xh[t][1] = xl[t][0] = xl[t][1] = 0.0;
        acc = mx = 0.0;
        for (int e = es; DIR * (elast - e) >= 0; e += DIR * RX) turn<0>(L, F, Cw, ec, ir, out, e, elast);
        wave_sum_to(acc, out.part + tid);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_down(mx, o, 64));
        if (threadIdx.x == 0) out.part[G.ntiles + tid] = mx;
    }

private:
    template <int SL>
    __device__ __forceinline__ void request64(const Lev<float> &L, const Lev<double> &F, int row)
    {
        const V vb = B::load(L.b, row), vu = B::load(L.u, row);
        this->b[SL][0] = vb.x; this->b[SL][1] = vb.y;
        this->u[SL][0] = vu.x; this->u[SL][1] = vu.y;
        const D2 vo = B::load(F.O, row), vs = B::load(F.S, row);
        O2[SL][0] = vo.x; O2[SL][1] = vo.y;
        S2[SL][0] = vs.x; S2[SL][1] = vs.y;
    }
    template <int M>
    __device__ __forceinline__ void want64(const Lev<float> &L, const Lev<double> &F, int e)
    {
        request64<B::template at<M>(0)>(L, F, e);
        request64<B::template at<M>(1)>(L, F, e + DIR);
        w2[0] = B::load(F.W, e);
        w2[1] = B::load(F.W, e + DIR);
    }
    // the FP32 operator of a row that has arrived, and its W into both rings
    template <int SL>
    __device__ __forceinline__ void arrived64(int row, D2 w)
    {
        *reinterpret_cast<D2 *>(sW2 + SL * WAVE_COLS) = w;
        typename B::Couplings c;
        c.w = V{(float)w.x, (float)w.y};
        B::template put_couplings<SL>(c);
        this->O[SL][0] = (float)O2[SL][0];
        this->O[SL][1] = (float)O2[SL][1];
        this->S[SL][0] = (float)S2[SL][0];
        this->S[SL][1] = (float)S2[SL][1];
        B::template arrived<SL>(row);
    }
    template <int D>
    __device__ __forceinline__ void fill64(const Lev<float> &L, const Lev<double> &F, const Wts<float> &Cw,
                                           const float *ec, int es)
    {
        if constexpr (D < 0) {
            constexpr int S0 = B::template at<0>(D), S1 = B::template at<0>(D + 1);
            const int row = es + DIR * D;
            request64<S0>(L, F, row);
            request64<S1>(L, F, row + DIR);
            const float e1 = A::crow(ec, (row >> 1) + DIR);
            A::weights(Cw, row);
            arrived64<S0>(row, B::load(F.W, row));
            arrived64<S1>(row + DIR, B::load(F.W, row + DIR));
            A::template correct<S0, S1>(row, this->e0, e1);
            this->e0 = e1;
            fill64<D + 2>(L, F, Cw, ec, es);
        }
    }
    // the pair of the rows step e finalises and B of the rows whose residual it takes
    __device__ __forceinline__ void pair_rows(const IrArgs &ir, const PairOut &out, int e)
    {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row = e - DIR * (2 * NU - 2 + t);
            ph[t] = B::load((const double *)ir.XH, row);
            pl[t] = B::load((const double *)ir.XL, row);
            pb[t] = B::load(out.B, row - DIR);
        }
    }
    // r at column C of window row D (its slot S0, SD below and SU above): the
    // pair of rows below, here, above in p, q, s of xh, xl
    template <int C, int SD, int S0, int SU, int P, int Q, int R>
    __device__ __forceinline__ double resid64(double bq) const
    {
        const double a[5] = {S2[S0][C], sW2[S0 * WAVE_COLS + C], sW2[S0 * WAVE_COLS + C + 1], S2[SU][C], O2[S0][C]};
        const double x[5] = {xh[P][C], C ? xh[Q][0] : from_west(xh[Q][1]), C ? from_east(xh[Q][0]) : xh[Q][1],
                             xh[R][C], xh[Q][C]};
        const double z[5] = {xl[P][C], C ? xl[Q][0] : from_west(xl[Q][1]), C ? from_east(xl[Q][0]) : xl[Q][1],
                             xl[R][C], xl[Q][C]};
        double s = bq, c = 0.0, ns, se;
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            const double pr = a[t] * x[t];
            const double pe = fma(a[t], x[t], -pr);
            two_sum(s, -pr, ns, se);
            s = ns;
            c = c + (se - pe);
        }
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            two_sum(s, -(a[t] * z[t]), ns, se);
            s = ns;
            c = c + se;
        }
        return s + c;
    }
    // the residual of row e + DIR D; P, Q, R: its neighbours behind, itself and
    // ahead among the four kept rows
    template <int M, int D, int P, int Q, int R>
    __device__ __forceinline__ void residual_row(const PairOut &out, int row, D2 bq)
    {
        constexpr int SD = B::template at<M>(D - DIR), S0 = B::template at<M>(D), SU = B::template at<M>(D + DIR);
        constexpr int lo = DIR > 0 ? P : R, hi = DIR > 0 ? R : P;
        const double r0 = resid64<0, SD, S0, SU, lo, Q, hi>(bq.x), r1 = resid64<1, SD, S0, SU, lo, Q, hi>(bq.y);
        if (this->own && row >= this->y0 && row < this->y1) {
            B::store(out.r, row, r0, r1);
            const double q0 = this->i0 > 0 ? r0 : 0.0;      // (column 0 is the ring)
            acc += q0 * q0;
            acc += r1 * r1;
            mx = fmax(mx, fmax(fabs(q0), fabs(r1)));
        }
    }
    template <int M>
    __device__ __forceinline__ void turn(const Lev<float> &L, const Lev<double> &F, const Wts<float> &Cw,
                                         const float *__restrict__ ec, const IrArgs &ir, const PairOut &out, int e,
                                         int elast)
    {
        if constexpr (M < RX / 2) {
            if (DIR * (e - elast) > 0) return;
            constexpr int S0 = B::template at<M>(0), S1 = B::template at<M>(1);
            wave_lds_order();
            arrived64<S0>(e, w2[0]);
            arrived64<S1>(e + DIR, w2[1]);
            wave_lds_order();
            A::template correct<S0, S1>(e, this->e0, this->en);
            this->e0 = this->en;
            D2 ch[2] = {ph[0], ph[1]}, cl[2] = {pl[0], pl[1]}, cb[2] = {pb[0], pb[1]};
            want64<(M + 1) % (RX / 2)>(L, F, e + 2 * DIR);
            pair_rows(ir, out, e + 2 * DIR);
            this->en = A::crow(ec, (e >> 1) + 2 * DIR);
            A::weights(Cw, e + 2 * DIR);
            B::template sweeps<M, 0, NU>();
            // the two rows that are final: (xh, xl) += s u, kept as rows 0, 1
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int row = e - DIR * (2 * NU - 2 + t);
                const float *v = this->u[B::template at<M>(2 - 2 * NU - t)];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const double d = sc * (double)v[c];
                    double hs, he;
                    two_sum(c ? ch[t].y : ch[t].x, d, hs, he);
                    he = he + (c ? cl[t].y : cl[t].x);
                    const double hi = hs + he;
                    xl[t][c] = he - (hi - hs);
                    xh[t][c] = hi;
                }
                if (this->own && row >= this->y0 && row < this->y1) {
                    B::store(out.oh, row, xh[t][0], xh[t][1]);
                    B::store(out.ol, row, xl[t][0], xl[t][1]);
                }
            }
            // residuals of the odd row and of the even row behind it
            residual_row<M, 1 - 2 * NU, 2, 1, 0>(out, e + DIR * (1 - 2 * NU), cb[0]);
            residual_row<M, -2 * NU, 3, 2, 1>(out, e - DIR * 2 * NU, cb[1]);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                xh[2][c] = xh[0][c]; xl[2][c] = xl[0][c];
                xh[3][c] = xh[1][c]; xl[3][c] = xl[1][c];
            }
            turn<M + 1>(L, F, Cw, ec, ir, out, e + 2 * DIR, elast);
        }
    }
};

template <int NU>
__global__ __launch_bounds__(64, 1) void k_post_res_wave(Lev<float> L, Lev<double> F, Wts<float> C,
                                                         const float *__restrict__ ec, TileGeo G, const int *stop,
                                                         IrArgs ir, PairOut out)
{
    int tid, k;
    if (!tile_work(G, tid, k)) return;
    if (stopped(stop)) return;
    __shared__ WavePostResLds<NU> S;
    if (wave_up(G, tid)) {
        WavePostRes<NU, 1> P;
        P.run(L, F, C, ec, ir, out, G, tid, S);
    } else {
        WavePostRes<NU, -1> P;
        P.run(L, F, C, ec, ir, out, G, tid, S);
    }
}

// --------------------------------- post pass and the next cycle's pre pass
// The fine level's post pass of cycle k and its pre pass of cycle k + 1 as one
// pass (FP64, five-point level, one right-hand side, one post sweep, NB pre
// sweeps), so the fine level's arrays are read and written once per cycle
// (78 bytes per point where the two passes take 118): rows enter as u' + P e_c,
// sweep 0 gives the cycle's result u_k (written, and its accurate residual's
// squares summed: rows e, e - 1, e - 2, e - 3 all hold u_k between sweep 0 and
// sweep 1 of a step), sweeps 1 .. NB give u'' (written), whose residual is
// restricted.  The weights the interpolation loads stay in an LDS ring until
// the restriction of their coarse row, four and five steps later (read again
// from memory they cost 9 bytes per fine point, the caches no longer having
// them).  u_c = 0 goes to a separate coarse buffer (ucz): other tiles still read
// e_c.
template <int NB>
struct WavePostPreLds {
    static constexpr int NS = NB + 1, TURNS = NS + 3;
    WaveLds<double, false, NS> ring;
    double w[TURNS * 8 * 64];   // turn, plane, lane
};

template <int NB, int DIR>
struct WavePostPre : WaveInterp<double, false, NB + 1, DIR> {
    using T = double;
    static constexpr int NS = NB + 1;
    using A = WaveInterp<double, false, NS, DIR>;
    using B = typename A::B;
    static constexpr int RX = B::RX, TURNS = RX / 2;
    static_assert(TURNS == NS + 3, "a coarse row's weights are used up to NS + 2 turns after they arrive");
    T pr0[2], pr1[2], acc;
    T *sw;                      // this lane's weights of turn 0
    int I;
    bool rest;

    __device__ __forceinline__ void run(const Lev<T> &L, T *__restrict__ ukout, T *__restrict__ uout,
                                        const Wts<T> &Cw, const T *__restrict__ ec, const Lev<T> &Cl,
                                        T *__restrict__ ucz, const TileGeo &G, int tid, double *__restrict__ part,
                                        WavePostPreLds<NB> &lds)
    {
        B::place(L, G, tid, lds.ring);
        sw = lds.w + threadIdx.x;
        A::coarse(Cw);
        I = this->i0 >> 1;
        rest = this->own && I >= 1 && I <= this->nc;
        const int y0 = this->y0, y1 = this->y1;
        const int es = DIR > 0 ? (y0 - 2 * NS) & ~1 : (y1 + 2 * NS) & ~1;
        const int elast = DIR > 0 ? 2 * ((y1 - 1) >> 1) + 2 * NS + 2 : 2 * ((y0 + 1) >> 1) - 2 * NS - 2;
        typename B::Couplings c[2];
        A::begin(L, Cw, ec, es, c);
        pr0[0] = pr0[1] = pr1[0] = pr1[1] = 0.0;
        acc = 0.0;
        for (int e = es; DIR * (elast - e) >= 0; e += DIR * RX)
            turn<0>(L, ukout, uout, Cw, ec, Cl, ucz, e, elast, c);
        wave_sum_to(acc, part + tid);
    }

private:
    // weight PL that arrived K turns before turn M, of the lane `west` lanes west
    template <int M, int K, int PL, int WEST>
    __device__ __forceinline__ T kept() const
    {
        return sw[(((M - K) % TURNS + TURNS) % TURNS * 8 + PL) * 64 - WEST];
    }
    template <int M>
    __device__ __forceinline__ void turn(const Lev<T> &L, T *__restrict__ ukout, T *__restrict__ uout,
                                         const Wts<T> &Cw, const T *__restrict__ ec, const Lev<T> &Cl,
                                         T *__restrict__ ucz, int e, int elast, typename B::Couplings (&c)[2])
    {
        if constexpr (M < TURNS) {
            if (DIR * (e - elast) > 0) return;
            wave_lds_order();
            B::template put_couplings<B::template at<M>(0)>(c[0]);
            B::template put_couplings<B::template at<M>(1)>(c[1]);
#pragma unroll
            for (int q = 0; q < 8; ++q) sw[(M * 8 + q) * 64] = this->w[q];
            wave_lds_order();
            A::template enter<M>(L, Cw, ec, e, c);
            B::template sweeps<M, 0, 1>();
            B::template write<M, 0>(ukout, e);
            B::template norm<M, -1>(e - DIR, acc);
            B::template norm<M, -2>(e - 2 * DIR, acc);
            B::template sweeps<M, 1, NS>();
            B::template write<M, NS - 1>(uout, e);
            T r0[2], r1[2];
            r0[0] = B::template resid<M, -2 * NS, 0>();
            r0[1] = B::template resid<M, -2 * NS, 1>();
            r1[0] = B::template resid<M, -2 * NS - 1, 0>();
            r1[1] = B::template resid<M, -2 * NS - 1, 1>();
            const int f = e - DIR * (2 * NS + 2), J = f >> 1;
            const T *rd = DIR > 0 ? pr1 : r1, *ru = DIR > 0 ? r1 : pr1;
            const T dw = from_west(rd[1]), mw = from_west(pr0[1]), uw = from_west(ru[1]);
            // planes of `weights`: row J's edges and the corner rows J, J + 1
            // (the even row f arrived NS + 1 turns ago; upward its corner row
            // J + 1 came with it, J a turn before, downward J and J + 1)
            constexpr int KE = NS + 1, KL = DIR > 0 ? NS + 2 : NS + 1, KU = DIR > 0 ? NS + 1 : NS + 2;
            T s = kept<M, KL, 7, 1>() * dw;                 // LNE(I, J)
            s = s + kept<M, KL, 3, 0>() * rd[0];            // LA(I, J)
            s = s + kept<M, KL, 6, 0>() * rd[1];            // LNW(I + 1, J)
            s = s + kept<M, KE, 1, 1>() * mw;               // LR(I, J)
            s = s + pr0[0];
            s = s + kept<M, KE, 0, 0>() * pr0[1];           // LL(I + 1, J)
            s = s + kept<M, KU, 5, 1>() * uw;               // LSE(I, J + 1)
            s = s + kept<M, KU, 2, 0>() * ru[0];            // LB(I, J + 1)
            s = s + kept<M, KU, 4, 0>() * ru[1];            // LSW(I + 1, J + 1)
            if (rest && J >= 1 && J <= this->nc && f >= this->y0 && f < this->y1) {
                const size_t p = (size_t)J * this->ldc + I;
                Cl.b[p] = s;
                ucz[p] = 0.0;
            }
            pr0[0] = r0[0]; pr0[1] = r0[1];
            pr1[0] = r1[0]; pr1[1] = r1[1];
            turn<M + 1>(L, ukout, uout, Cw, ec, Cl, ucz, e + 2 * DIR, elast, c);
        }
    }
};

template <int NB>
__global__ __launch_bounds__(64, 1) void k_postpre_wave(Lev<double> L, double *__restrict__ ukout,
                                                        double *__restrict__ uout, Wts<double> C,
                                                        const double *__restrict__ ec, Lev<double> Cl,
                                                        double *__restrict__ ucz, TileGeo G,
                                                        double *__restrict__ part, const int *stop)
{
    int tid, k;
    if (!tile_work(G, tid, k)) return;
    if (stopped(stop)) return;
    __shared__ WavePostPreLds<NB> S;
    if (wave_up(G, tid)) {
        WavePostPre<NB, 1> P;
        P.run(L, ukout, uout, C, ec, Cl, ucz, G, tid, part, S);
    } else {
        WavePostPre<NB, -1> P;
        P.run(L, ukout, uout, C, ec, Cl, ucz, G, tid, part, S);
    }
}

}  // namespace bmg
