// The small-level tail of a V-cycle in one workgroup, every level in LDS.
//
// A level's nodes are held as 2 x 2 patches: patch (I, J) owns the fine nodes
//   a (2I, 2J)   b (2I+1, 2J)   c (2I, 2J+1)   d (2I+1, 2J+1)
// (a and d have colour 0, b and c colour 1), one patch per thread (up to NPT
// on the top level), its values and right-hand side in registers.  LDS holds
// the level as four planes, one per position in the patch, so a thread reads
// four neighbours and writes two values per colour, all of them with
// consecutive lanes on consecutive words; the residuals of a patch are formed
// from its registers and eight neighbours, and the full weighting reads five
// of them from three residual planes.  Node by node in LDS, as it was before,
// a colour cost eleven accesses per two nodes at a two-way bank conflict, the
// full weighting 54 per coarse node, and an integer division per node and
// pass.  Bound by the one CU's instruction issue on the top level (a colour is
// 16 FP and 6 LDS instructions per patch, sixteen wavefronts on four SIMDs)
// and below it by latency: ten dependent phases a level of an LDS round trip,
// a few FP operations and a barrier; levels of at most 64 patches run in the
// first wavefront alone, without barriers.  Per launch (rocprofv3), 65 x 65
// top FP64 32.6 -> 17.7 us; FP32 81 x 57 top 13.9 us where 81 x 57 as launches
// and the 41 x 29 subtree took 22.3 + 11.7.
//
// Every node value is produced by the same expression, on the same operands,
// as in the streaming kernels, so the result is bitwise that of the
// multi-launch schedule.  The patches of an m x n level (m, n odd) number
// (m - 1) / 2 by (n - 1) / 2; the last column and row are boundary, known to
// be zero.
#pragma once

#include "stencil_tiles.hpp"

namespace lap {

template <bool WAVE>
__device__ __forceinline__ void sub_sync() {
    if constexpr (WAVE) {
        // one wavefront: its LDS accesses are in order, only the compiler must keep them so
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// A level's geometry as the patches see it.  ST: the planes' stride where it
// is fixed (the top level: the plane offsets are then immediates of the LDS
// instructions), 0: one more than its patches.  Each plane's last entry is
// zero: the neighbour of the patches at the level's edge.
template <typename T, int ST>
struct SubGeo {
    int W, H, np, stride;  // patches across, down, in all; plane stride
    T cx, cy, d, inv_d;
    T* u;                  // four planes
    template <typename L_>   // a SubLevel<T>, wherever it is stored
    __device__ __forceinline__ SubGeo(T* s, const L_& L, bool bnd = false)
        : W((L.m - 1) >> 1), H((L.n - 1) >> 1), np(W * H), stride(ST > 0 ? ST : np + 1 + (bnd ? W + H : 0)),
          cx(L.cx), cy(L.cy), d(L.d), inv_d(L.inv_d), u(s + L.ou) {}
    __device__ __forceinline__ T* plane(int k) const { return u + k * (ST > 0 ? ST : stride); }
    __device__ __forceinline__ int edge() const { return (ST > 0 ? ST : stride) - 1; }
};

// A thread's patches of one level.
template <typename T, int NPT, int ST>
struct Patches {
    using Geo = SubGeo<T, ST>;
    T a[NPT], b[NPT], c[NPT], d[NPT];        // iterate
    T fa[NPT], fb[NPT], fc[NPT], fd[NPT];    // right-hand side (zero where the node is boundary)
    T wa[NPT], wb[NPT], wc[NPT];             // relaxation, 0 where the node is boundary (d never is)
    int p[NPT], I[NPT], J[NPT];
    int kl[NPT], kr[NPT], kd[NPT], ku[NPT];  // plane entries left, right, below, above
    bool on[NPT];

    __device__ __forceinline__ bool xl(int q) const { return I[q] > 0; }
    __device__ __forceinline__ bool yl(int q) const { return J[q] > 0; }

    __device__ __forceinline__ void place(const Geo& G, T om, int nthreads, bool bnd = false) {
        const float inv = 1.0f / (float)G.W;
        const int z = G.edge();
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            p[q] = (int)threadIdx.x + q * nthreads;
            on[q] = p[q] < G.np;
            J[q] = seg_div(p[q], inv);
            I[q] = p[q] - J[q] * G.W;
            kl[q] = on[q] && I[q] > 0 ? p[q] - 1 : z;
            kr[q] = on[q] && I[q] < G.W - 1 ? p[q] + 1 : on[q] && bnd ? G.np + J[q] : z;
            kd[q] = on[q] && J[q] > 0 ? p[q] - G.W : z;
            ku[q] = on[q] && J[q] < G.H - 1 ? p[q] + G.W : on[q] && bnd ? G.np + G.H + I[q] : z;
            wa[q] = xl(q) && yl(q) ? om : T(0);
            wb[q] = yl(q) ? om : T(0);
            wc[q] = xl(q) ? om : T(0);
            a[q] = b[q] = c[q] = d[q] = T(0);
            fa[q] = fb[q] = fc[q] = fd[q] = T(0);
        }
    }
    __device__ __forceinline__ void zero_edge(const Geo& G) const {
        if (threadIdx.x < 4) G.plane(threadIdx.x)[G.edge()] = T(0);
    }
    __device__ __forceinline__ void set_rhs(int q, T va, T vb, T vc, T vd) {
        fa[q] = xl(q) && yl(q) ? va : T(0);
        fb[q] = yl(q) ? vb : T(0);
        fc[q] = xl(q) ? vc : T(0);
        fd[q] = vd;
    }

    // a red-black sweep; `zero`: the iterate is zero and the planes hold nothing yet
    template <bool WAVE>
    __device__ __forceinline__ void sweep(const Geo& G, T om, bool zero) {
        T *PA = G.plane(0), *PB = G.plane(1), *PC = G.plane(2), *PD = G.plane(3);
        if (zero) {
            const T lu = fma(G.cy, T(0), G.cx * T(0));
#pragma unroll
            for (int q = 0; q < NPT; ++q) {
                if (!on[q]) continue;
                const T xa = (lu - fa[q]) * G.inv_d, xd = (lu - fd[q]) * G.inv_d;
                a[q] = fma(wa[q], xa, T(0));
                d[q] = fma(om, xd, T(0));
                PA[p[q]] = a[q];
                PD[p[q]] = d[q];
            }
        } else {
// all neighbours first: a patch's stores would hold back the next
            // one's loads (a thread without a patch reads the zero entries)
            T bw[NPT], cs[NPT], ce[NPT], bn[NPT];
#pragma unroll
            for (int q = 0; q < NPT; ++q) {
                bw[q] = PB[kl[q]];
                cs[q] = PC[kd[q]];
                ce[q] = PC[kr[q]];
                bn[q] = PB[ku[q]];
            }
#pragma unroll
            for (int q = 0; q < NPT; ++q) {
                const T xa = (fma(G.cy, cs[q] + c[q], G.cx * (bw[q] + b[q])) - fa[q]) * G.inv_d;
                const T xd = (fma(G.cy, b[q] + bn[q], G.cx * (c[q] + ce[q])) - fd[q]) * G.inv_d;
                a[q] = fma(wa[q], xa - a[q], a[q]);
                d[q] = fma(om, xd - d[q], d[q]);
                if (!on[q]) continue;
                PA[p[q]] = a[q];
                PD[p[q]] = d[q];
            }
        }
        sub_sync<WAVE>();
        T ae[NPT], an[NPT], ds[NPT], dw[NPT];
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            ae[q] = PA[kr[q]];
            an[q] = PA[ku[q]];
            ds[q] = PD[kd[q]];
            dw[q] = PD[kl[q]];
        }
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const T xb = (fma(G.cy, ds[q] + d[q], G.cx * (a[q] + ae[q])) - fb[q]) * G.inv_d;
            const T xc = (fma(G.cy, a[q] + an[q], G.cx * (dw[q] + d[q])) - fc[q]) * G.inv_d;
            b[q] = fma(wb[q], xb - b[q], b[q]);
            c[q] = fma(wc[q], xc - c[q], c[q]);
            if (!on[q]) continue;
            PB[p[q]] = b[q];
            PC[p[q]] = c[q];
        }
        sub_sync<WAVE>();
    }

    // residuals into the planes R (b, c, d), then full weighting at the
    // interior even nodes onto the next level's right-hand side: its patch
    // planes, or (coarsest) a plain array of width mc
    template <bool WAVE>
    __device__ __forceinline__ void restrict_to(const Geo& G, T* R, T* bc, int mc, bool coarsest, bool zero) {
        const T *PA = G.plane(0), *PB = G.plane(1), *PC = G.plane(2), *PD = G.plane(3);
        T *RB = R, *RC = R + G.np, *RD = R + 2 * G.np;
        T ra[NPT], rb[NPT], rc[NPT], rd[NPT];
        const auto res = [&](T f, T u, T W, T E, T S, T N) { return f - fma(-G.d, u, fma(G.cy, S + N, G.cx * (W + E))); };
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            ra[q] = fa[q];
            rb[q] = fb[q];
            rc[q] = fc[q];
            rd[q] = fd[q];
            if (!zero) {
                const T bw = PB[kl[q]], cs = PC[kd[q]], ce = PC[kr[q]], bn = PB[ku[q]];
                const T ae = PA[kr[q]], an = PA[ku[q]], ds = PD[kd[q]], dw = PD[kl[q]];
                ra[q] = res(fa[q], a[q], bw, b[q], cs, c[q]);
                rb[q] = res(fb[q], b[q], a[q], ae, ds, d[q]);
                rc[q] = res(fc[q], c[q], dw, d[q], a[q], an);
                rd[q] = res(fd[q], d[q], c[q], ce, b[q], bn);
            }
        }
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (!on[q]) continue;
            RB[p[q]] = rb[q];
            RC[p[q]] = rc[q];
            RD[p[q]] = rd[q];
        }
        sub_sync<WAVE>();
        const int Wc = (mc - 1) >> 1, npc = Wc * (G.H >> 1);
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (!on[q] || !xl(q) || !yl(q)) continue;
            const int k = p[q];
            const T W = RB[k - 1], S = RC[k - G.W], SW = RD[k - G.W - 1], SE = RD[k - G.W], NW = RD[k - 1];
            const T v = (fma(T(4), ra[q], T(2) * ((W + rb[q]) + (S + rc[q]))) + ((SW + SE) + (NW + rd[q]))) * T(0.0625);
            const int at = coarsest ? J[q] * mc + I[q]
                                    : ((J[q] & 1) * 2 + (I[q] & 1)) * npc + (J[q] >> 1) * Wc + (I[q] >> 1);
            bc[at] = v;
        }
        sub_sync<WAVE>();
    }

    // every node's residual into four planes R (boundary nodes': not used)
    __device__ __forceinline__ void residuals(const Geo& G, T* R) {
        const T *PA = G.plane(0), *PB = G.plane(1), *PC = G.plane(2), *PD = G.plane(3);
        const auto res = [&](T f, T u, T W, T E, T S, T N) { return f - fma(-G.d, u, fma(G.cy, S + N, G.cx * (W + E))); };
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const T bw = PB[kl[q]], cs = PC[kd[q]], ce = PC[kr[q]], bn = PB[ku[q]];
            const T ae = PA[kr[q]], an = PA[ku[q]], ds = PD[kd[q]], dw = PD[kl[q]];
            if (!on[q]) continue;
            R[p[q]] = res(fa[q], a[q], bw, b[q], cs, c[q]);
            R[p[q] + G.np] = res(fb[q], b[q], a[q], ae, ds, d[q]);
            R[p[q] + 2 * G.np] = res(fc[q], c[q], dw, d[q], a[q], an);
            R[p[q] + 3 * G.np] = res(fd[q], d[q], c[q], ce, b[q], bn);
        }
    }

    // this level's right-hand side / iterate from the planes
    __device__ __forceinline__ void load_rhs(const Geo& G, const T* f) {
#pragma unroll
        for (int q = 0; q < NPT; ++q)
            if (on[q]) set_rhs(q, f[p[q]], f[p[q] + G.np], f[p[q] + 2 * G.np], f[p[q] + 3 * G.np]);
    }
    __device__ __forceinline__ void load_u(const Geo& G) {
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (!on[q]) continue;
            a[q] = G.plane(0)[p[q]];
            b[q] = G.plane(1)[p[q]];
            c[q] = G.plane(2)[p[q]];
            d[q] = G.plane(3)[p[q]];
        }
    }

    // u += P(u_C) on the interior (bilinear interpolation), into the planes
    template <bool WAVE>
    __device__ __forceinline__ void prolong_add(const Geo& G, const T* uc, int mc, bool coarsest) {
        const int Wc = (mc - 1) >> 1, stc = Wc * (G.H >> 1) + 1;   // the next level's plane stride
        const auto coarse = [&](int I, int J) {   // coarse node (I, J), zero on the boundary
            if (I < 1 || J < 1 || I >= G.W || J >= G.H) return T(0);
            return uc[coarsest ? J * mc + I : ((J & 1) * 2 + (I & 1)) * stc + (J >> 1) * Wc + (I >> 1)];
        };
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (!on[q]) continue;
            const T e00 = coarse(I[q], J[q]), e10 = coarse(I[q] + 1, J[q]);
            const T e01 = coarse(I[q], J[q] + 1), e11 = coarse(I[q] + 1, J[q] + 1);
            if (xl(q) && yl(q)) a[q] = a[q] + e00;
            if (yl(q)) b[q] = b[q] + (e00 + e10) * T(0.5);
            if (xl(q)) c[q] = c[q] + (e00 + e01) * T(0.5);
            d[q] = d[q] + ((e00 + e10) + (e01 + e11)) * T(0.25);
            G.plane(0)[p[q]] = a[q];
            G.plane(1)[p[q]] = b[q];
            G.plane(2)[p[q]] = c[q];
            G.plane(3)[p[q]] = d[q];
        }
        sub_sync<WAVE>();
    }
};

// Coarsest solve with the dense inverse by the calling threads (all of the
// workgroup, or one wavefront): x = minv rhs.  minv: in LDS or global memory.
template <typename T, bool WAVE, typename Args>
__device__ __forceinline__ void sub_coarse(const Args& S, T* s, double* rhs, const double* minv,
                                           int nthreads) {
    const auto& C = S.lv[S.nlev - 1];
    const int mi = C.m - 2, N = mi * (C.n - 2);
    const T* b = s + C.ob;
    for (int k = threadIdx.x; k < N; k += nthreads) rhs[k] = (double)b[(1 + k / mi) * C.m + 1 + k % mi];
    sub_sync<WAVE>();
    for (int k = threadIdx.x; k < N; k += nthreads) {
        double x = 0.0;
#pragma unroll 8
        for (int l = 0; l < N; ++l) x = fma(minv[(size_t)l * N + k], rhs[l], x);
        s[C.ou + (1 + k / mi) * C.m + 1 + k % mi] = (T)x;
    }
    sub_sync<WAVE>();
}

// Levels k .. nlev-1 of the cycle below a level whose full weighting has set
// level k's right-hand side: down, coarsest solve, up.  One patch per thread.
// WAVE: every level has at most 64 patches and only the first wavefront is here.
template <typename T, bool WAVE, typename Args>
__device__ __forceinline__ void sub_levels(const Args& S, T* s, double* rhs, const double* minv, int k,
                                           int nthreads) {
    const int last = S.nlev - 1;
    int l = k;
    for (; l < last; ++l) {
        const SubGeo<T, 0> G(s, S.lv[l]);
        if constexpr (!WAVE)
            if (G.np <= 64) break;
        Patches<T, 1, 0> X;
        X.place(G, S.omega, nthreads);
        X.zero_edge(G);   // read after the first colour's barrier at the earliest
        X.load_rhs(G, s + S.lv[l].ob);
        bool zero = true;
        for (int q = 0; q < S.nu1; ++q) {
            X.template sweep<WAVE>(G, S.omega, zero);
            zero = false;
        }
        X.template restrict_to<WAVE>(G, s + S.orr, s + S.lv[l + 1].ob, S.lv[l + 1].m, l + 1 == last, zero);
    }
    if constexpr (WAVE) {
        sub_coarse<T, true>(S, s, rhs, minv, 64);
    } else {
        if (l < last) {
            if (threadIdx.x < 64) sub_levels<T, true>(S, s, rhs, minv, l, 64);
            __syncthreads();
        } else if (S.bw == 0) {
            sub_coarse<T, false>(S, s, rhs, minv, nthreads);
        } else {
            const auto& C = S.lv[last];
            CoarseArgs<T> A{};
            A.b = s + C.ob;
            A.out = s + C.ou;
            A.minv = S.minv;
            A.work = S.work;
            A.bw = S.bw;
            A.ifast = S.ifast;
            A.m = C.m;
            A.n = C.n;
            A.P = C.m;
            A.cx = S.ccx;
            A.cy = S.ccy;
            coarse_block<T>(A, rhs);
            __syncthreads();
        }
    }
    for (--l; l >= k; --l) {
        const SubGeo<T, 0> G(s, S.lv[l]);
        Patches<T, 1, 0> X;
        X.place(G, S.omega, nthreads);
        X.load_rhs(G, s + S.lv[l].ob);
        if (S.nu1 > 0) X.load_u(G);
        X.template prolong_add<WAVE>(G, s + S.lv[l + 1].ou, S.lv[l + 1].m, l + 1 == last);
        for (int q = 0; q < S.nu2; ++q) X.template sweep<WAVE>(G, S.omega, false);
    }
}

// The coarsest inverse into LDS (with the first loads in flight) when the
// launch has room for it: N at most kSubInvMax unknowns.
template <typename Args>
__device__ __forceinline__ const double* sub_stage_inverse(const Args& S, double* rhs) {
    if (S.inv_lds == 0) return S.minv;
    const auto& C = S.lv[S.nlev - 1];
    const int N = (C.m - 2) * (C.n - 2);
    for (int k = threadIdx.x; k < N * N; k += blockDim.x) rhs[N + k] = S.minv[k];
    return rhs + N;
}

// The sub-V-cycle from the top level (zero start) for a workgroup of any
// number of wavefronts with at most NPT patches of the top level per thread.
// Args: SubtreeArgs<T>, in the kernel's arguments or in constant memory.
template <typename T, int NPT, typename Args>
__device__ __forceinline__ void subtree_block(const Args& S, T* s, double* rhs) {
    using V2 = typename VecT<T, 2>::type;
    constexpr int ST = sub_top_stride(NPT);
    const SubGeo<T, ST> G(s, S.lv[0]);
    const int nt = blockDim.x;
    Patches<T, NPT, ST> X;
    X.place(G, S.omega, nt);
    X.zero_edge(G);
    if (S.b != nullptr) {
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (!X.on[q]) continue;
            const T* f = S.b + (size_t)(2 * X.J[q]) * S.P + 2 * X.I[q];
            const V2 r0 = *reinterpret_cast<const V2*>(f), r1 = *reinterpret_cast<const V2*>(f + S.P);
            X.set_rhs(q, r0.x, r0.y, r1.x, r1.y);
        }
    }
    const double* minv = sub_stage_inverse(S, rhs);
    bool zero = true;
    for (int q = 0; q < S.nu1; ++q) {
        X.template sweep<false>(G, S.omega, zero);
        zero = false;
    }
    const bool two = S.nlev == 2;
    X.template restrict_to<false>(G, s + S.orr, s + S.lv[1].ob, S.lv[1].m, two, zero);
    sub_levels<T, false>(S, s, rhs, minv, 1, nt);
    X.template prolong_add<false>(G, s + S.lv[1].ou, S.lv[1].m, two);
    for (int q = 0; q < S.nu2; ++q) X.template sweep<false>(G, S.omega, false);
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        if (!X.on[q]) continue;
        T* o = S.out + (size_t)(2 * X.J[q]) * S.P + 2 * X.I[q];
        *reinterpret_cast<V2*>(o) = V2{X.a[q], X.b[q]};
        *reinterpret_cast<V2*>(o + S.P) = V2{X.c[q], X.d[q]};
        // the boundary column and row beyond the last patches
        const bool right = X.I[q] == G.W - 1;
        if (right) o[2] = o[S.P + 2] = T(0);
        if (X.J[q] == G.H - 1) {
            o[2 * (size_t)S.P] = o[2 * (size_t)S.P + 1] = T(0);
            if (right) o[2 * (size_t)S.P + 2] = T(0);
        }
    }
}

// ---------------------------------------------------- whole small solves
// An FP64 multigrid solve of a grid whose hierarchy fits LDS, in one launch of
// one workgroup: the residual norms and the stopping test, then the V-cycle,
// until the test ends the solve.  Launched pass by pass such a solve is all
// dispatches, round trips to memory and the host's polls (25 x 17 chamber, 7
// cycles: 464 us a call against 219 us, 68 of them the launch).  The norms are those of the
// launched solve bit for bit: the canonical tiles' lanes sum the same nodes in
// the same order (rows of odd chunks from above where the first pass flips
// them), and the partials are reduced by the same butterfly.
template <int NPT>
__device__ __forceinline__ void mg_solve_block(const MgSolveArgs& A, double* s, double* rhs) {
    using T = double;
    using V2 = typename VecT<T, 2>::type;
    const SubtreeArgs<T>& S = A.sub;
    const SubGeo<T, 0> G(s, S.lv[0], true);
    const int m = S.lv[0].m, n = S.lv[0].n, nt = blockDim.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t P = (size_t)S.P;
    __shared__ double parts[2 * kMgSolveTiles];
    __shared__ Ctrl ctrl;
    Patches<T, NPT, 0> X;
    X.place(G, S.omega, nt, true);
    T *PA = G.plane(0), *PB = G.plane(1), *PC = G.plane(2), *PD = G.plane(3);
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        if (!X.on[q]) continue;
        const size_t at = (size_t)(2 * X.J[q]) * P + 2 * X.I[q];
        const V2 u0 = *reinterpret_cast<const V2*>(S.out + at), u1 = *reinterpret_cast<const V2*>(S.out + at + P);
        X.a[q] = u0.x;
        X.b[q] = u0.y;
        X.c[q] = u1.x;
        X.d[q] = u1.y;
        if (S.b != nullptr) {
            const V2 f0 = *reinterpret_cast<const V2*>(S.b + at), f1 = *reinterpret_cast<const V2*>(S.b + at + P);
            X.set_rhs(q, f0.x, f0.y, f1.x, f1.y);
        }
        const int k = X.p[q];
        PA[k] = u0.x;
        PB[k] = u0.y;
        PC[k] = u1.x;
        PD[k] = u1.y;
    }
    for (int J = threadIdx.x; J < G.H; J += nt) {
        const int k = G.np + J;
        PA[k] = S.out[(size_t)(2 * J) * P + m - 1];
        PC[k] = S.out[(size_t)(2 * J + 1) * P + m - 1];
        PB[k] = PD[k] = 0.0;
    }
    for (int I = threadIdx.x; I < G.W; I += nt) {
        const int k = G.np + G.H + I;
        PA[k] = S.out[(size_t)(n - 1) * P + 2 * I];
        PB[k] = S.out[(size_t)(n - 1) * P + 2 * I + 1];
        PC[k] = PD[k] = 0.0;
    }
    X.zero_edge(G);
    if (threadIdx.x == 0) {
        if (A.fresh) {
            ctrl = Ctrl{};
            ctrl.tol = A.tol;
            ctrl.stop = A.stop;
            ctrl.max_iter = A.max_iter;
            ctrl.step = 1;
        } else {
            ctrl = *A.ctrl;
        }
    }
    const double* minv = sub_stage_inverse(S, rhs);
    __syncthreads();
    const bool two = S.nlev == 2;
    // at most A.cycles cycles a launch; the next one opens with the test that is due
    for (int k = 0;; ++k) {
        if (k == A.cycles) break;
        // every node's residual into four planes (the last one in the next
        // level's room, idle between cycles and larger), then the canonical
        // tiles' sums: a lane adds its two columns row by row
        X.residuals(G, s + S.orr);
        __syncthreads();
        for (int t = wave; t < A.tl.ntiles; t += nt >> 6) {
            const int win = t % A.tl.nwin, chunk = t / A.tl.nwin;
            const Cols<kNormPassV> c(win, lane, m, S.P, A.tl.H);
            const int j0 = 1 + chunk * A.tl.ty, j1 = min(j0 + A.tl.ty - 1, n - 2);
            const int step = A.flip && (chunk & 1) ? -1 : 1;
            const double* r = s + S.orr + min(max(c.i0 >> 1, 0), G.W - 1);   // column pair c.i0, c.i0 + 1
            double s2 = 0.0, mx = 0.0;
#pragma unroll 4
            for (int k = 0, j = step > 0 ? j0 : j1; k <= j1 - j0; ++k, j += step) {
                const double* rj = r + 2 * (j & 1) * G.np + (j >> 1) * G.W;
#pragma unroll
                for (int e = 0; e < kNormPassV; ++e) {
                    const double v = c.cout[e] ? rj[e * G.np] : 0.0;
                    s2 = fma(v, v, s2);
                    mx = fmax(mx, fabs(v));
                }
            }
            s2 = wave_sum(s2);
            mx = wave_max(mx);
            if (lane == 0) {
                parts[2 * t] = s2;
                parts[2 * t + 1] = mx;
            }
        }
        __syncthreads();
        if (wave == 0) {
            // k_finalize's first wavefront; its others have nothing to add
            const bool have = lane < A.tl.ntiles;
            const double sum = wave_sum(have ? 0.0 + parts[2 * lane] : 0.0);
            const double mx = wave_max(have ? fmax(0.0, parts[2 * lane + 1]) : 0.0);
            if (lane == 0) decide_test(0.0 + sum, fmax(0.0, mx), &ctrl, 0);
        }
        __syncthreads();
        if (ctrl.done) break;
        for (int q = 0; q < S.nu1; ++q) X.template sweep<false>(G, S.omega, false);
        X.template restrict_to<false>(G, s + S.orr, s + S.lv[1].ob, S.lv[1].m, two, false);
        sub_levels<T, false>(S, s, rhs, minv, 1, nt);
        X.template prolong_add<false>(G, s + S.lv[1].ou, S.lv[1].m, two);
        for (int q = 0; q < S.nu2; ++q) X.template sweep<false>(G, S.omega, false);
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        if (!X.on[q]) continue;
        T* o = S.out + (size_t)(2 * X.J[q]) * P + 2 * X.I[q];
        *reinterpret_cast<V2*>(o) = V2{X.a[q], X.b[q]};
        *reinterpret_cast<V2*>(o + P) = V2{X.c[q], X.d[q]};
    }
    if (threadIdx.x == 0) *A.ctrl = *A.host = ctrl;
}

}  // namespace lap
