// Fused streaming passes: several operations of a V-cycle level in one read
// of the level.  A wavefront walks its window down the rows once; the rows go
// through a pipeline of red-black sweep stages (each stage lags the previous
// one by two rows), and the rows leaving the last stage are stored and,
// optionally, turned into residual rows that are full-weighted onto the
// coarse right-hand side.  Per node every stage evaluates exactly the
// expressions of the one-sweep kernel on the same operands, so a fused pass
// is bitwise the sequence of separate launches.
//
// Valid columns shrink by two per sweep and by two more for residual + full
// weighting, so windows overlap by the tiling's halo H on each side
// (H = 2 * sweeps, + 2 with the restriction, rounded up to a multiple of the
// columns per lane); valid rows shrink the same way, so a chunk reads
// 2 * sweeps (+ 1 or 2) rows beyond its own above and below.
//
// One ring for a row's whole life.  Row r sits in slot r mod K of one
// register array from the load that brings it in, through every stage's two
// colour updates, which change it in place, to its last use; the loop is
// unrolled over K steps, so every slot is a fixed register and nothing is
// ever moved: a stage pipeline with registers of its own, fed from a ring of
// loads, spent a third of its vector instructions on moves.  In place is
// exact: at step j stage s updates colour 0 of row j - 2s from rows one above
// and below, then colour 1 of the row before; stage s + 1 first touches a row
// after stage s's last use of it.  All control is wave-uniform and scalar: the
// wave index is read from lane 0, rows outside the level are clamped in
// their address (what they bring only reaches halo values), the loads are
// unconditional (the compiler then counts exactly how many may stay in
// flight), and the tests whether a row is interior exist only in the copy of
// the loop that chunks at the level's edge take.  One row of the FP64
// post-smoothing pass takes 46 vector and 41 scalar instructions where it took
// 115 and 80, of the FP32 four-sweep pass (four columns a lane) 160 and 71
// where it took 456 and 154.  Whole solves (graph replay): 1025^2 mixed 966 ->
// 820 us, 4097^2 FP64 2.43 -> 2.15 ms, 8193^2 FP64 6.65 -> 6.28 ms, mixed
// 5.91 -> 5.46 ms; 200 SOR sweeps on 3000 x 2201 3.41 -> 2.96 ms.  The finest
// FP64 passes are bound by HBM, the four-sweep pass by vector issue, the
// passes of levels below ~1000^2 by the few wavefronts' issue and launches.
#pragma once

#include "stencil_tiles.hpp"

namespace lap {

// Pointers of the field arrays are global memory (also where they come out of
// a table in memory, from which the compiler could not tell).
template <typename T> using GlobalPtr = __attribute__((address_space(1))) T*;

// A lane's V columns of a row at (uniform) address `row`, lane offset in bytes.
template <typename T, int V>
__device__ __forceinline__ void ld_lane(T (&x)[V], const T* row, unsigned lane_off) {
    using VT = typename VecT<T, V>::type;
    const VT v = *(GlobalPtr<const VT>)(reinterpret_cast<const char*>(row) + lane_off);
    if constexpr (V == 1) {
        x[0] = v;
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) x[e] = v[e];
    }
}
template <typename T, int V, bool NT>
__device__ __forceinline__ void st_lane(T* row, const T (&x)[V], unsigned lane_off) {
    using VT = typename VecT<T, V>::type;
    VT v;
    if constexpr (V == 1) {
        v = x[0];
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = x[e];
    }
    const GlobalPtr<VT> p = (GlobalPtr<VT>)(reinterpret_cast<char*>(row) + lane_off);
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

template <int FL>
constexpr int fused_sweeps() {
    return (FL & SW_FOUR) ? 4 : (FL & SW_TWO) ? 2 : 1;
}

// Rows in the ring (even: a turn keeps the row parity).  Those beyond the
// stages' own are in flight: six for two FP64 sweeps with the restriction,
// seven without, two less where a right-hand side streams along or FP64 rows
// do besides FP32 ones (their registers cost a wavefront of occupancy);
// four columns a lane and four sweeps with norms and a right-hand side (225
// registers; 268 with 14 rows, one wavefront a SIMD) keep two in flight.
template <typename T, int V, int FL>
constexpr int fused_ring() {
    if (fused_sweeps<FL>() == 4) return (FL & SW_NORM) && (FL & SW_F) ? 12 : 14;
    if (fused_sweeps<FL>() == 1 || V == 4) return 8;
    return (FL & SW_DEF) || (sizeof(T) == 8 && (FL & SW_F)) ? 10 : 12;
}

template <typename T, int V, int FL>
struct FusedRegs {
    static constexpr int NS = fused_sweeps<FL>(), K = fused_ring<T, V, FL>();
    static constexpr bool RS = (FL & SW_RESTRICT) != 0;
    // rows in flight behind the entering one: the row loaded at the end of a
    // step takes the slot of the row that saw its last use in it
    static constexpr int PF = RS ? K - 2 * NS - 2 : K - 2 * NS - 1;
    static constexpr int KC = K / 2;                       // coarse rows (one per two steps)
    static constexpr int KD = K / 2;                       // SW_DEF: FP64 rows
    static constexpr int VC = (V >= 2 ? V / 2 : 1) + 1;    // coarse columns a lane's columns need
    static_assert(K % 2 == 0 && PF >= 2, "ring too short");
    T u[K][V], f[(FL & SW_F) ? K : 1][V];
    T c[(FL & SW_PROLONG) ? KC : 1][VC];
    T rodd[V], wodd, eodd, reven[V];                       // residual rows behind the last one
    T mid[(FL & SW_NORM) && NS == 4 ? V : 1];              // a row of the iterate after two of four sweeps
    double psi[(FL & SW_DEF) ? KD : 1][V], g[(FL & SW_DEF) ? KD : 1][V];
    double s2, mx;
};

// What a lane needs of its window.
template <typename T, int V>
struct FusedLane {
    unsigned off;        // byte offset of its (clamped) columns of T in a row
    unsigned off64;      // the same for FP64 rows (SW_DEF)
    unsigned coff[(V >= 2 ? V / 2 : 1) + 1];   // byte offsets of its (clamped) coarse columns
    unsigned boff;       // byte offset of its first coarse output column
    bool st;             // it stores its columns (it holds an output column)
    bool cst[V];         // element e is an even output column (full weighting)
    bool cout[V];        // element e is an output column
    bool cint[V];        // element e is an interior column
    bool iodd;           // V == 1: the column is odd
    T w[2][V];           // relaxation by row parity (OmegaMask)
};

// SW_DEF with norms per block of kRowBlock rows: the lanes' sums of up to
// kRowPartBlocks blocks of each wavefront's chunk.
__device__ __forceinline__ double* rowpart_slot(int block) {
    __shared__ double parts[kWavesPerBlock][kRowPartBlocks][2][64];
    return &parts[wave_in_block()][block][0][threadIdx.x & 63];
}

template <int K>
__device__ __forceinline__ constexpr int ring_slot(int ph, int off) {
    return (ph + off + 8 * K) % K;
}

// x += P(lo, hi) for a fine row between coarse rows lo and hi (odd) or on lo.
template <typename T, int V, bool ODD>
__device__ __forceinline__ void add_correction(T (&x)[V], const T (&lo)[(V >= 2 ? V / 2 : 1) + 1],
                                               const T (&hi)[(V >= 2 ? V / 2 : 1) + 1], bool iodd) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int q = V >= 2 ? e >> 1 : 0;
        const T p_even = ODD ? (lo[q] + hi[q]) * T(0.5) : lo[q];
        const T p_odd = ODD ? ((lo[q] + lo[q + 1]) + (hi[q] + hi[q + 1])) * T(0.25) : (lo[q] + lo[q + 1]) * T(0.5);
        if constexpr (V >= 2)
            x[e] = x[e] + ((e & 1) ? p_odd : p_even);
        else
            x[e] = x[e] + (iodd ? p_odd : p_even);
    }
}

// One colour update of a row (elements of the colour only) from the rows
// below (S) and above (N) and its own other colour.
template <typename T, int V, int JP, bool HASF>
__device__ __forceinline__ void colour_row(T (&c)[V], const T (&S)[V], const T (&N)[V], const T (&f)[V],
                                           const T (&w)[V], T cx, T cy, T inv_d) {
    const T W0 = lane_prev(c[V - 1]), E0 = lane_next(c[0]);
#pragma unroll
    for (int e = 0; e < V; ++e) {
        if (colour_skip<V, JP>(e)) continue;
        const T W = e > 0 ? c[e - 1] : W0;
        const T E = e < V - 1 ? c[e + 1] : E0;
        const T s = fma(cy, S[e] + N[e], cx * (W + E));
        const T t = (HASF ? s - f[e] : s) * inv_d;
        c[e] = fma(w[e], t - c[e], c[e]);
    }
}

// Adds the residual of a row (c, between rows S and N) to the lane's norms.
template <typename T, int V, int FL>
__device__ __forceinline__ void norm_row(const SweepArgs<T>& A, FusedRegs<T, V, FL>& R, const FusedLane<T, V>& l,
                                         const T (&S)[V], const T (&c)[V], const T (&N)[V], const T (&f)[V]) {
    const T W0 = lane_prev(c[V - 1]), E0 = lane_next(c[0]);
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const T W = e > 0 ? c[e - 1] : W0;
        const T E = e < V - 1 ? c[e + 1] : E0;
        const T L = fma(-A.d, c[e], fma(A.cy, S[e] + N[e], A.cx * (W + E)));
        const double r = l.cout[e] ? (double)((FL & SW_F) ? f[e] - L : T(0) - L) : 0.0;
        R.s2 = fma(r, r, R.s2);
        R.mx = fmax(R.mx, fabs(r));
    }
}

// Step of phase PH at row j: input row j + 1 enters, stage s updates rows
// j - 2s and j - 2s - 1, row q = j + 1 - 2 NS is final.
template <typename T, int V, int FL, bool EDGE, bool NT, int PH>
__device__ __forceinline__ void fused_step(const SweepArgs<T>& A, FusedRegs<T, V, FL>& R, const FusedLane<T, V>& l,
                                           int j, int j0, int j1, int Lend) {
    using Regs = FusedRegs<T, V, FL>;
    constexpr int NS = Regs::NS, K = Regs::K, PF = Regs::PF, KC = Regs::KC, KD = Regs::KD, VC = Regs::VC;
    constexpr bool RS = Regs::RS, HASF = (FL & SW_F) != 0;
    constexpr int JP = ((RS ? 1 : 0) + PH) & 1;             // parity of j
    constexpr int FK = HASF ? K : 1;
    const T cx = A.cx, cy = A.cy, inv_d = A.inv_d;
    // rows are addressed clamped to the level and to the chunk's last input row
    const auto row_off = [&](int r, int last) -> ptrdiff_t { return (ptrdiff_t)max(0, min(r, last)) * A.Ps; };

    T(&in)[V] = R.u[ring_slot<K>(PH, 1)];
    if constexpr ((FL & SW_ZERO) != 0) zero<T, V>(in);
    if constexpr ((FL & SW_PROLONG) != 0) {
        // coarse row above or at input row j + 1, as a count from the chunk's first
        constexpr int JR = RS ? PH / 2 : (PH + 1) / 2;
        add_correction<T, V, JP == 0>(in, R.c[JR % KC], R.c[(JR + 1) % KC], l.iodd);
        if constexpr (JP == 1) {
            // the coarse row before JR was last used in the step before
            const int J = ((j + 1) >> 1) - 1 + KC;
            const T* base = A.ec + (ptrdiff_t)max(0, min(J, min((Lend >> 1) + 1, A.nc - 1))) * A.Pcs;
#pragma unroll
            for (int k = 0; k < VC; ++k) {
                T x[1];
                ld_lane<T, 1>(x, base, l.coff[k]);
                R.c[(JR + KC - 1) % KC][k] = x[0];
            }
        }
    }
    if constexpr ((FL & SW_NORM) != 0 && NS < 4) {
        // residual of the input at row j + 1, before row j changes
        if (j + 1 >= j0 && j + 1 <= j1)
            norm_row<T, V, FL>(A, R, l, R.u[ring_slot<K>(PH, 0)], in, R.u[ring_slot<K>(PH, 2)],
                               R.f[HASF ? ring_slot<FK>(PH, 1) : 0]);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int r = j - 2 * s;
        if constexpr ((FL & SW_NORM) != 0 && NS == 4) {
            // between the second and the third sweep: residual at row j - 4 of the
            // iterate after two (row j - 5's first colour changed a step ago)
            if (s == 2) {
                const T(&c)[V] = R.u[ring_slot<K>(PH, -4)];
                if (r >= j0 && r <= j1)
                    norm_row<T, V, FL>(A, R, l, R.mid, c, R.u[ring_slot<K>(PH, -3)],
                                       R.f[HASF ? ring_slot<FK>(PH, -4) : 0]);
                copy<T, V>(R.mid, c);
            }
        }
        if (!EDGE || (r >= 1 && r <= A.n - 2))
            colour_row<T, V, JP, HASF>(R.u[ring_slot<K>(PH, -2 * s)], R.u[ring_slot<K>(PH, -2 * s - 1)],
                                       R.u[ring_slot<K>(PH, -2 * s + 1)],
                                       R.f[HASF ? ring_slot<FK>(PH, -2 * s) : 0], l.w[JP], cx, cy, inv_d);
        if (!EDGE || (r >= 2 && r <= A.n - 1))
            colour_row<T, V, JP, HASF>(R.u[ring_slot<K>(PH, -2 * s - 1)], R.u[ring_slot<K>(PH, -2 * s - 2)],
                                       R.u[ring_slot<K>(PH, -2 * s)],
                                       R.f[HASF ? ring_slot<FK>(PH, -2 * s - 1) : 0], l.w[JP], cx, cy, inv_d);
    }
    const int q = j + 1 - 2 * NS;
    T(&o)[V] = R.u[ring_slot<K>(PH, 1 - 2 * NS)];
    if constexpr ((FL & SW_DEF) != 0) {
        // o is row q of the final correction: psi_out = psi_in + e there (the
        // perimeter stays, also beside a correction that overflowed: its own
        // value in o, weighted by zero, is then no number), and the FP64
        // residual of the updated iterate at row q - 1
        constexpr int DQ = 1 - 2 * NS;
        double(&pn)[V] = R.psi[ring_slot<KD>(PH, DQ)];
#pragma unroll
        for (int e = 0; e < V; ++e) pn[e] = pn[e] + (double)(l.cint[e] ? o[e] : T(0));
        if (q >= j0 && q <= j1 && l.st) st_lane<double, V, NT>(A.psi_out + (ptrdiff_t)q * A.Ps, pn, l.off64);
        if (q - 1 >= j0 && q - 1 <= j1) {
            const double(&pc)[V] = R.psi[ring_slot<KD>(PH, DQ - 1)];
            const double(&pm)[V] = R.psi[ring_slot<KD>(PH, DQ - 2)];
            const double(&fm)[V] = R.g[ring_slot<KD>(PH, DQ - 1)];
            const double W0 = lane_prev(pc[V - 1]), E0 = lane_next(pc[0]);
            T r32[V];
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const double W = e > 0 ? pc[e - 1] : W0;
                const double E = e < V - 1 ? pc[e + 1] : E0;
                const double L = fma(-A.dd, pc[e], fma(A.dcy, pm[e] + pn[e], A.dcx * (W + E)));
                const double rr = l.cout[e] ? fm[e] - L : 0.0;
                r32[e] = (T)rr;
                R.s2 = fma(rr, rr, R.s2);
                R.mx = fmax(R.mx, fabs(rr));
            }
            if (A.rowpart && ((q - 1) % kRowBlock == 0 || q - 1 == j1)) {
                // end of a block of kRowBlock rows: its sums, in row order
                // whatever chunk holds it, wait in LDS (reduced after the walk)
                double* part = rowpart_slot((q - 1 - j0) / kRowBlock);
                part[0] = R.s2;
                part[64] = R.mx;
                R.s2 = 0.0;
                R.mx = 0.0;
            }
            if (l.st) st_lane<T, V, NT>(A.rhs_out + (ptrdiff_t)(q - 1) * A.Ps, r32, l.off);
        }
        // psi row q - 2 saw its last use (of the source, row q - 1)
        const ptrdiff_t ro = row_off(q + KD - 2, min(j1 + 1, A.n - 1));
        ld_lane<double, V>(R.psi[ring_slot<KD>(PH, DQ - 2)], A.psi_in + ro, l.off64);
        if (A.f64 != nullptr)
            ld_lane<double, V>(R.g[ring_slot<KD>(PH, DQ - 2)], A.f64 + ro, l.off64);
    } else {
        if (q >= j0 && q <= j1 && l.st) st_lane<T, V, NT>(A.uout + (ptrdiff_t)q * A.Ps, o, l.off);
    }
    if constexpr (RS) {
        // residual of the result at row q - 1 (SW_RDIFF: in difference form),
        // then full weighting at the even row q - 2.  Only interior coarse
        // nodes are stored, whose nine fine nodes are interior.
        const T(&c)[V] = R.u[ring_slot<K>(PH, -2 * NS)];
        const T(&S)[V] = R.u[ring_slot<K>(PH, -2 * NS - 1)];
        const T(&f)[V] = R.f[HASF ? ring_slot<FK>(PH, -2 * NS) : 0];
        T r0[V];
        const T W0 = lane_prev(c[V - 1]), E0 = lane_next(c[0]);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const T W = e > 0 ? c[e - 1] : W0;
            const T E = e < V - 1 ? c[e + 1] : E0;
            T L;
            if constexpr ((FL & SW_RDIFF) != 0)
                L = cx * ((W - c[e]) + (E - c[e])) + cy * ((S[e] - c[e]) + (o[e] - c[e]));
            else
                L = fma(-A.d, c[e], fma(cy, S[e] + o[e], cx * (W + E)));
            r0[e] = HASF ? f[e] - L : T(0) - L;
        }
        // q - 2 is even exactly on steps with j odd
        if constexpr (JP == 1) {
            const T w0 = lane_prev(r0[V - 1]), e0 = V >= 2 ? T(0) : lane_next(r0[0]);
            const T w1 = lane_prev(R.reven[V - 1]), e1 = V >= 2 ? T(0) : lane_next(R.reven[0]);
            if (q - 2 >= j0 && q - 2 <= j1) {
                T* brow = A.bc + (ptrdiff_t)((q - 2) >> 1) * A.Pcs;
                T v[V];
#pragma unroll
                for (int e = 0; e < V; e += 2) {
                    const T C = R.reven[e];
                    const T W = e > 0 ? R.reven[e - 1] : w1;
                    const T E = e < V - 1 ? R.reven[e + 1] : e1;
                    const T Sr = R.rodd[e], N = r0[e];
                    const T SW = e > 0 ? R.rodd[e - 1] : R.wodd;
                    const T SE = e < V - 1 ? R.rodd[e + 1] : R.eodd;
                    const T NW = e > 0 ? r0[e - 1] : w0;
                    const T NE = e < V - 1 ? r0[e + 1] : e0;
                    v[e] = (fma(T(4), C, T(2) * ((W + E) + (Sr + N))) + ((SW + SE) + (NW + NE))) * T(0.0625);
                }
                if (V == 4 && l.cst[0] && l.cst[V == 4 ? 2 : 0]) {
                    const T pair[2] = {v[0], v[V == 4 ? 2 : 0]};
                    using VT = typename VecT<T, 2>::type;
                    *(GlobalPtr<VT>)(reinterpret_cast<char*>(brow) + l.boff) = VT{pair[0], pair[1]};
                } else {
#pragma unroll
                    for (int e = 0; e < V; e += 2)
                        if (l.cst[e])
                            *((GlobalPtr<T>)(reinterpret_cast<char*>(brow) + l.boff) + e / 2) = v[e];
                }
            }
            copy<T, V>(R.rodd, r0);
            R.wodd = w0;
            R.eodd = e0;
        } else {
            copy<T, V>(R.reven, r0);
        }
    }
    // the slot of the row that saw its last use takes the next row
    {
        const ptrdiff_t ro = row_off(j + 1 + PF, min(Lend, A.n - 1));
        if constexpr ((FL & SW_ZERO) == 0) ld_lane<T, V>(R.u[ring_slot<K>(PH, 1 + PF)], A.uin + ro, l.off);
        if constexpr (HASF) ld_lane<T, V>(R.f[ring_slot<FK>(PH, 1 + PF)], A.f + ro, l.off);
    }
}

// Steps PH, PH + 1, ... of one turn of the ring from row j: all of them, or
// (TAIL) those up to the last input row.
template <typename T, int V, int FL, bool EDGE, bool NT, bool TAIL, int PH>
__device__ __forceinline__ void fused_turn(const SweepArgs<T>& A, FusedRegs<T, V, FL>& R, const FusedLane<T, V>& l,
                                           int j, int j0, int j1, int Lend) {
    if constexpr (PH < FusedRegs<T, V, FL>::K) {
        if (TAIL && j + PH > Lend - 1) return;
        fused_step<T, V, FL, EDGE, NT, PH>(A, R, l, j + PH, j0, j1, Lend);
        fused_turn<T, V, FL, EDGE, NT, TAIL, PH + 1>(A, R, l, j, j0, j1, Lend);
    }
}

// Norms of the input alone (SW_PROBE): the same rows, in the same order.
template <typename T, int V, int FL>
__device__ __forceinline__ void probe_rows(const SweepArgs<T>& A, FusedRegs<T, V, FL>& R, const FusedLane<T, V>& l,
                                           int j0, int j1) {
    constexpr int K = 6;
    constexpr bool HASF = (FL & SW_F) != 0;
    T u[K][V], f[HASF ? K : 1][V];
    const auto off = [&](int r) -> ptrdiff_t { return (ptrdiff_t)min(r, j1 + 1) * A.Ps; };
#pragma unroll
    for (int k = 0; k < K; ++k) {
        ld_lane<T, V>(u[k], A.uin + off(j0 - 1 + k), l.off);
        if constexpr (HASF) ld_lane<T, V>(f[k], A.f + off(j0 - 1 + k), l.off);
    }
    for (int jb = j0; jb <= j1; jb += K) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = jb + k;   // row j - 1 in slot k
            if (j <= j1) {
                const T(&c)[V] = u[(k + 1) % K];
                const T W0 = lane_prev(c[V - 1]), E0 = lane_next(c[0]);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const T W = e > 0 ? c[e - 1] : W0;
                    const T E = e < V - 1 ? c[e + 1] : E0;
                    const T L = fma(-A.d, c[e], fma(A.cy, u[k][e] + u[(k + 2) % K][e], A.cx * (W + E)));
                    const double r = l.cout[e] ? (double)(HASF ? f[HASF ? (k + 1) % K : 0][e] - L : T(0) - L) : 0.0;
                    R.s2 = fma(r, r, R.s2);
                    R.mx = fmax(R.mx, fabs(r));
                }
            }
            ld_lane<T, V>(u[k], A.uin + off(j - 1 + K), l.off);
            if constexpr (HASF) ld_lane<T, V>(f[HASF ? k : 0], A.f + off(j - 1 + K), l.off);
        }
    }
}

// Odd row chunks walk upwards, through a vertically flipped view of the
// level (base at the last row, negative row strides; the coarse arrays
// likewise).  Neighbouring chunks then reach their common boundary at the
// same time, both at the start or both at the end of their walks, so the
// halo rows one of them re-reads are still in L2.  With an odd number of
// rows the flip keeps every node's colour (n - 1 is even), fine row 2J
// stays over coarse row J, and each expression only sees its north and
// south operands swapped in a commutative sum: the values are unchanged.
// tile, and everything in A0, are wave-uniform.  NT: nontemporal row stores.
template <typename T, int V, int FL, bool NT = false>
__device__ __forceinline__ void fused_tile(const SweepArgs<T>& A0, int tile, int lane) {
    using Regs = FusedRegs<T, V, FL>;
    constexpr int NS = Regs::NS, K = Regs::K, PF = Regs::PF, KC = Regs::KC, KD = Regs::KD, VC = Regs::VC;
    constexpr bool RS = Regs::RS, HASF = (FL & SW_F) != 0;
    SweepArgs<T> A = A0;
    const int win = tile % A.tl.nwin, chunk = tile / A.tl.nwin;
    const Cols<V> c(win, lane, A.m, A.P, A.tl.H);
    int j0 = 1 + chunk * A.tl.ty;
    int j1 = min(j0 + A.tl.ty - 1, A.n - 2);
    A.Ps = A.P;
    A.Pcs = A.Pc;
    if ((chunk & 1) && (A.n & 1) && !((FL & SW_DEF) && A.rowpart)) {
        const ptrdiff_t last = (ptrdiff_t)(A.n - 1) * A.P, clast = (ptrdiff_t)(A.nc - 1) * A.Pc;
        if (A.uin) A.uin += last;
        if (A.uout) A.uout += last;
        if (A.f) A.f += last;
        if constexpr ((FL & SW_DEF) != 0) {
            A.psi_in += last;
            A.psi_out += last;
            if (A.f64) A.f64 += last;
            A.rhs_out += last;
        }
        if (A.ec) A.ec += clast;
        if (A.bc) A.bc += clast;
        A.Ps = -A.P;
        A.Pcs = -A.Pc;
        const int t0 = A.n - 1 - j1;
        j1 = A.n - 1 - j0;
        j0 = t0;
    }
    if constexpr ((FL & SW_DEF) != 0) A.rp_off = win * row_blocks(A.n);

    FusedLane<T, V> l;
    {
        // columns outside the row's storage read inside it (halo values only)
        const int ic = max(0, min(c.i0, A.P - V));
        l.off = (unsigned)ic * sizeof(T);
        l.off64 = (unsigned)ic * sizeof(double);
        l.boff = (unsigned)(ic >> 1) * sizeof(T);
        l.iodd = (c.i0 & 1) != 0;
        l.st = false;
        const OmegaMask<T, V> wm(c, c.i0 & 1, A.omega);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            l.st = l.st || c.cout[e];
            l.cout[e] = c.cout[e];
            l.cint[e] = c.cint[e];
            l.cst[e] = c.cout[e] && ((c.i0 + e) & 1) == 0;
            l.w[0][e] = wm.w[0][e];
            l.w[1][e] = wm.w[1][e];
        }
        if constexpr ((FL & SW_PROLONG) != 0) {
#pragma unroll
            for (int k = 0; k < VC; ++k) l.coff[k] = (unsigned)max(0, min((c.i0 >> 1) + k, A.Pc - 1)) * sizeof(T);
        }
    }

    Regs R;
    R.s2 = 0.0;
    R.mx = 0.0;
    if constexpr ((FL & SW_PROBE) != 0) {
        probe_rows<T, V, FL>(A, R, l, j0, j1);
    } else {
        // input rows [L0, Lend]: the last stage must be exact on the chunk's rows
        // and, with the restriction, two rows around its first and last even row;
        // L0 is moved up one row if needed so the first step has parity JP0
        // (SW_DEF: the residual needs the final rows j0 - 1 .. j1 + 1)
        constexpr int JP0 = RS ? 1 : 0;
        constexpr int DX = (FL & SW_DEF) ? 1 : 0;
        const int e0 = j0 + (j0 & 1), e1 = j1 - (j1 & 1);
        int L0 = (RS ? e0 - 2 : j0 - DX) - 2 * NS;
        if (((L0 + 1) & 1) != JP0) --L0;
        const int Lend = (RS ? e1 + 2 : j1 + DX) + 2 * NS;
        const int lastrow = min(Lend, A.n - 1);
        const auto row_off = [&](int r) -> ptrdiff_t { return (ptrdiff_t)max(0, min(r, lastrow)) * A.Ps; };
        const int jb = L0 + 1;                             // step of phase 0: row jb + off in slot (0, off)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            zero<T, V>(R.u[k]);
            if constexpr (HASF) zero<T, V>(R.f[k]);
        }
        T cx0[VC];                                         // the coarse row before the ring's first
        if constexpr ((FL & SW_PROLONG) != 0) {
            const int J0 = (jb + 1) >> 1, Jl = min((Lend >> 1) + 1, A.nc - 1);
            const auto ldc = [&](T (&x)[VC], int J) {
                const T* base = A.ec + (ptrdiff_t)max(0, min(J, Jl)) * A.Pcs;
#pragma unroll
                for (int k = 0; k < VC; ++k) {
                    T y[1];
                    ld_lane<T, 1>(y, base, l.coff[k]);
                    x[k] = y[0];
                }
            };
            ldc(cx0, J0 - 1);
#pragma unroll
            for (int k = 0; k < KC; ++k) ldc(R.c[k], J0 + k);
        }
#pragma unroll
        for (int k = -1; k <= PF; ++k) {
            const ptrdiff_t ro = row_off(jb + k);
            if constexpr ((FL & SW_ZERO) == 0) ld_lane<T, V>(R.u[ring_slot<K>(0, k)], A.uin + ro, l.off);
            if constexpr (HASF) ld_lane<T, V>(R.f[ring_slot<K>(0, k)], A.f + ro, l.off);
        }
        if constexpr ((FL & SW_DEF) != 0) {
            // the first step's final row is jb + 1 - 2 NS; the KD - 2 rows from it on
            constexpr int DQ = 1 - 2 * NS;
#pragma unroll
            for (int k = 0; k < KD; ++k) {
                zero<double, V>(R.psi[k]);
                zero<double, V>(R.g[k]);
            }
#pragma unroll
            for (int k = 0; k < KD - 2; ++k) {
                const ptrdiff_t ro = (ptrdiff_t)max(0, min(jb + DQ + k, min(j1 + 1, A.n - 1))) * A.Ps;
                ld_lane<double, V>(R.psi[ring_slot<KD>(0, DQ + k)], A.psi_in + ro, l.off64);
                if (A.f64 != nullptr) ld_lane<double, V>(R.g[ring_slot<KD>(0, DQ + k)], A.f64 + ro, l.off64);
            }
        }
        if constexpr ((FL & SW_PROLONG) != 0) {
            // rows L0 and L0 + 1 enter here; the first one's coarse row is cx0
            add_correction<T, V, JP0 == 0>(R.u[ring_slot<K>(0, -1)], cx0, R.c[0], l.iodd);
            if constexpr (JP0 == 0)
                add_correction<T, V, false>(R.u[ring_slot<K>(0, 0)], R.c[0], R.c[1], l.iodd);
            else
                add_correction<T, V, true>(R.u[ring_slot<K>(0, 0)], cx0, R.c[0], l.iodd);
        }
        if constexpr (RS) {
            zero<T, V>(R.rodd);
            zero<T, V>(R.reven);
            R.wodd = R.eodd = T(0);
        }
        if constexpr ((FL & SW_NORM) != 0 && NS == 4) zero<T, V>(R.mid);
        // whole turns of the ring without an exit (one from inside a turn would
        // have the compiler wait for every load at the head of the loop), then
        // the rest, whose copy of the steps serves both kinds of chunks
        int j = jb;
        if (L0 >= 1 && Lend <= A.n - 2)
            for (; j + K - 1 <= Lend - 1; j += K) fused_turn<T, V, FL, false, NT, false, 0>(A, R, l, j, j0, j1, Lend);
        else
            for (; j + K - 1 <= Lend - 1; j += K) fused_turn<T, V, FL, true, NT, false, 0>(A, R, l, j, j0, j1, Lend);
        fused_turn<T, V, FL, true, NT, true, 0>(A, R, l, j, j0, j1, Lend);
    }
    if constexpr ((FL & (SW_NORM | SW_DEF)) != 0) {
        if ((FL & SW_DEF) && A.rowpart) {
            for (int k = 0; j0 + k * kRowBlock <= j1; ++k) {
                const double* part = rowpart_slot(k);
                const double s = wave_sum(part[0]), mx = wave_max(part[64]);
                if (lane == 0) {
                    const int b = A.rp_off + (j0 - 1) / kRowBlock + k;
                    A.partials[2 * b] = s;
                    A.partials[2 * b + 1] = mx;
                }
            }
            return;
        }
        const double s = wave_sum(R.s2);
        const double mx = wave_max(R.mx);
        if (lane == 0) {
            A.partials[2 * tile] = s;
            A.partials[2 * tile + 1] = mx;
        }
    }
}

}  // namespace lap
