// The paper's own sequential methods on the GPU, with the paper's update
// order: Jacobi (Eq. (5)), lexicographic Gauss-Seidel / SOR (Eqs. (6)-(7)),
// SLOR by rows with the relaxation after the line solve (SLORA, Eqs. (8)-(9))
// or inside it (SLORB, Eq. (10)), and ADI as all rows in ascending order
// followed by all columns in ascending order (ADI section).
//
// One workgroup holds the whole grid in LDS and runs the whole solve: every
// iteration, its stopping test and the next iteration stay on the chip, so a
// small problem such as the 25 x 17 chamber costs a few microseconds per
// iteration instead of several launches.  The sequential methods are one
// serial chain of operations with no bandwidth to speak of, so they run in
// ONE wavefront (LDS accesses of a wavefront are in order and its barriers
// are free; sixteen wavefronts spent most of their time meeting at barriers),
// and what is not on the chain is taken off it.  A residual as the monitored
// quantity is no chain: further wavefronts wait through the sweep and form it
// with the first (paper_residual).
//
// Order.  Lexicographic SOR updates node (i, j) after (i-1, j) and (i, j-1)
// and before (i+1, j) and (i, j+1).  All nodes of one anti-diagonal i + j = d
// depend only on diagonals d - 1 (already new) and d + 1 (still old), so the
// wavefront updates a diagonal at once and moves to the next:
// every node sees exactly the operands of the row-by-row loop.  The line
// methods solve one line after another (each line's Thomas recurrence is
// sequential; its right-hand side and its relaxation are computed by all
// threads).
//
// Arithmetic.  Every expression is the plain one of the methods, unfused
// (the file is built with -ffp-contract=off):
//   t = ((cx (W + E) + cy (S + N)) - f) * inv_d,   psi <- psi + w (t - psi),
// and the line systems by the Thomas recurrences, every quotient that of an
// IEEE division (see paper_line).
//
// Measured (25 x 17 chamber to max update 1e-9, whole call): ADI in the
// paper's order, w = 1.3, 6.66 ms with 1024 threads and the divisions on the
// chain, 3.12 ms now.  Bound by the latency of the chain's dependent FP64
// operations: four per unknown forwards, two backwards.
#include <algorithm>
#include <cmath>

#include "lap_kernels.hpp"
#include "../../include/lap.h"

namespace lap {

constexpr int kPaperRed = 16;   // reduction slots: wavefronts of 1024 lanes

__device__ __forceinline__ double block_max(double v, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double r = red[0];
    for (int k = 1; k < nw; ++k) r = fmax(r, red[k]);
    __syncthreads();
    return r;
}

// Order between the lanes of the one wavefront that sweeps: its LDS accesses
// are in order, only the compiler must keep them so.  NT: the largest workgroup.
template <int NT>
__device__ __forceinline__ void paper_sync() {
    if constexpr (NT == 64) {
        __syncthreads();
        return;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A line system of K unknowns (row line: along i; column line: along j) and
// where its elements are in LDS; the coupling e of the end values.
struct PaperLine {
    int K, at0, stride, across, line, dir;
    double cc, e;
    __device__ PaperLine(const PaperArgs& A, int line_, int dir_) : line(line_), dir(dir_) {
        K = dir == 0 ? A.m - 2 : A.n - 2;
        at0 = dir == 0 ? line * A.m + 1 : A.m + line;
        stride = dir == 0 ? 1 : A.m;
        across = dir == 0 ? A.m : 1;
        const double lc = dir == 0 ? A.cx : A.cy;
        cc = dir == 0 ? A.cy : A.cx;
        e = A.form == 0 ? lc : A.omega * lc;
    }
};

// The line's right-hand sides.
__device__ __forceinline__ void paper_rhs(const PaperArgs& A, const PaperLine& g, const double* u, double* rhs) {
    for (int k = threadIdx.x; k < g.K; k += 64) {
        const int p = g.at0 + k * g.stride;
        const int j = g.dir == 0 ? g.line : k + 1, i = g.dir == 0 ? k + 1 : g.line;
        const double fv = A.f != nullptr ? A.f[(size_t)j * A.P + i] : 0.0;
        const double base = g.cc * (u[p - g.across] + u[p + g.across]) - fv;
        double r = A.form == 0 ? base : (1.0 - A.omega) * A.d * u[p] + A.omega * base;
        if (k == 0) r = r + g.e * u[p - g.stride];   // end values enter with the line coupling
        if (k == g.K - 1) r = r + g.e * u[p + g.stride];
        rhs[k] = r;
    }
}

// The line's new values from its solution x, relaxed (form 0).  Returns the
// lane's largest |new - base| of the line, base the node's value in u0 or
// (KEEP) before this line, which u0, if not null, then takes.
template <bool KEEP>
__device__ __forceinline__ double paper_relax(const PaperArgs& A, const PaperLine& g, double* u, double* u0,
                                              const double* x) {
    double mx = 0.0;
    for (int k = threadIdx.x; k < g.K; k += 64) {
        const int p = g.at0 + k * g.stride;
        const double old = u[p];
        const double v = A.form == 0 ? old + A.omega * (x[k] - old) : x[k];
        u[p] = v;
        if constexpr (KEEP) {
            if (u0 != nullptr) u0[p] = old;
            mx = fmax(mx, fabs(v - old));
        } else {
            mx = fmax(mx, fabs(v - u0[p]));
        }
    }
    return mx;
}

// Line scratch (LDS): rhs, then the solution, K values; xq, the pairs
// (x_k, rp_k) of the forward recurrence.  Per direction: cp[k] = c'_k =
// a / pivot_k (a the off-diagonal, pivot_0 = d, pivot_k = d - a c'_{k-1}) and
// y[k], the reciprocal of pivot_k as an unevaluated sum y.x + y.y (1 / pivot_k
// rounded, the rest rounded).  The factors do not depend on the line, so they
// are computed once per solve.  Arrays hold kPaperPad values more than the
// longest line: the chains run in whole groups of eight.
constexpr int kPaperPad = 8;
struct PaperFactor {
    double a;
    double* cp;
    double2* y;
};
__device__ void paper_factor(const PaperFactor& F, double d, int K) {
    double cp = 0.0;
    for (int k = 0; k < K; ++k) {
        const double piv = k == 0 ? d : d - F.a * cp;
        cp = F.a / piv;
        F.cp[k] = cp;
        const double y = 1.0 / piv;
        F.y[k] = double2{y, fma(-piv, y, 1.0) * y};
    }
}

// One line solved in place on u by the Thomas recurrences, by one wavefront.
//
// The forward recurrence rp_k = (rhs_k - a rp_{k-1}) / pivot_k is the chain
// the whole solve waits on, and a division is most of it.  On the chain the
// quotient x / pivot is x y.x + x y.y with one rounding at the end: the sum
// carries 105 bits of the reciprocal, so it is the correctly rounded quotient
// unless x / pivot lies that close to a rounding boundary.  Every quotient is
// then compared, all of a line's at once (a lane each), with the IEEE
// division of the same operands; should one differ (also where the operands
// overflow, vanish or are not numbers), the line's recurrence is run again
// with divisions.  The values are those of the plain recurrence either way.
// The operands of the next eight steps are read while eight are computed.
template <bool KEEP, int NT>
__device__ double paper_line(const PaperArgs& A, double* u, double* u0, int line, int dir, const PaperFactor& F,
                             double* rhs, double2* xq) {
    const PaperLine g(A, line, dir);
    const int K = g.K;
    const double d = A.d, a = F.a;
    paper_rhs(A, g, u, rhs);
    paper_sync<NT>();
    constexpr int B = 8;
    if (threadIdx.x == 0) {
        double q = 0.0;
        double r0[B], r1[B];
        double2 y0[B], y1[B];
        const auto load = [&](double (&r)[B], double2 (&y)[B], int k) {
#pragma unroll
            for (int e = 0; e < B; ++e) {
                r[e] = rhs[k + e];
                y[e] = F.y[k + e];
            }
        };
        const auto chain = [&](const double (&r)[B], const double2 (&y)[B], int k) {
#pragma unroll
            for (int e = 0; e < B; ++e) {
                const double x = e == 0 && k == 0 ? r[e] : r[e] - a * q;
                q = fma(x, y[e].x, x * y[e].y);
                xq[k + e] = double2{x, q};
            }
        };
        load(r0, y0, 0);
        for (int k = 0; k < K; k += 2 * B) {
            if (k + B < K) load(r1, y1, k + B);
            chain(r0, y0, k);
            if (k + B >= K) break;
            if (k + 2 * B < K) load(r0, y0, k + 2 * B);
            chain(r1, y1, k + B);
        }
    }
    paper_sync<NT>();
    bool same = true;
    for (int k = threadIdx.x; k < K; k += 64) {
        const double piv = k == 0 ? d : d - a * F.cp[k - 1];
        same = same && __double_as_longlong(xq[k].x / piv) == __double_as_longlong(xq[k].y);
    }
    if (__any(!same)) {
        paper_sync<NT>();
        if (threadIdx.x == 0) {
            double q = 0.0;
            for (int k = 0; k < K; ++k) {
                const double piv = k == 0 ? d : d - a * F.cp[k - 1];
                q = k == 0 ? rhs[0] / piv : (rhs[k] - a * q) / piv;
                xq[k].y = q;
            }
        }
    }
    paper_sync<NT>();
    if (threadIdx.x == 0) {
        // x_k = rp_k - c'_k x_{k+1}, in groups of eight from the top; the first
        // group holds the steps beyond the line's end
        double x = 0.0;
        double r0[B], c0[B], r1[B], c1[B];
        const auto load = [&](double (&r)[B], double (&c)[B], int k) {
#pragma unroll
            for (int e = 0; e < B; ++e) {
                r[e] = xq[k + e].y;
                c[e] = F.cp[k + e];
            }
        };
        const auto chain = [&](const double (&r)[B], const double (&c)[B], int k) {
#pragma unroll
            for (int e = B - 1; e >= 0; --e) {
                x = r[e] - c[e] * x;
                rhs[k + e] = x;
            }
        };
        int k = (K - 1) / B * B;
        load(r0, c0, k);
        if (k >= B) load(r1, c1, k - B);
#pragma unroll
        for (int e = B - 1; e >= 0; --e)
            if (k + e < K) {
                x = k + e == K - 1 ? r0[e] : r0[e] - c0[e] * x;
                rhs[k + e] = x;
            }
        for (k -= B; k >= 0; k -= 2 * B) {
            if (k >= B) load(r0, c0, k - B);
            chain(r1, c1, k);
            if (k < B) break;
            if (k >= 2 * B) load(r1, c1, k - 2 * B);
            chain(r0, c0, k - B);
        }
    }
    paper_sync<NT>();
    const double mx = paper_relax<KEEP>(A, g, u, u0, rhs);
    paper_sync<NT>();
    return mx;
}

// The same for a grid that leaves no room for the factors: the plain
// recurrence with its divisions.  rhs, cp, rp: K values each.
template <bool KEEP, int NT>
__device__ double paper_line_plain(const PaperArgs& A, double* u, double* u0, int line, int dir, double a,
                                   double* rhs, double* cp, double* rp) {
    const PaperLine g(A, line, dir);
    paper_rhs(A, g, u, rhs);
    paper_sync<NT>();
    if (threadIdx.x == 0) {
        const double b = A.d;
        cp[0] = a / b;
        rp[0] = rhs[0] / b;
        for (int k = 1; k < g.K; ++k) {
            const double piv = b - a * cp[k - 1];
            cp[k] = a / piv;
            rp[k] = (rhs[k] - a * rp[k - 1]) / piv;
        }
        rhs[g.K - 1] = rp[g.K - 1];
        for (int k = g.K - 2; k >= 0; --k) rhs[k] = rp[k] - cp[k] * rhs[k + 1];
    }
    paper_sync<NT>();
    const double mx = paper_relax<KEEP>(A, g, u, u0, rhs);
    paper_sync<NT>();
    return mx;
}

// Residual norms of u over the workgroup: max |r| (SUM: sum r^2).  The sum is
// that of 1024 lanes, lane t adding nodes t, t + 1024, ... in order, then a
// butterfly per 64 lanes and the results in order, whatever number of
// threads forms it: the monitored values do not depend on the launch.  By the
// sweep's wavefront alone it is N / 64 turns of one wave: 30 iterations of
// lexicographic SOR on 97 x 97 took 2.92 ms, with 16 wavefronts 2.07 (2.01
// with the largest update, which comes with the sweep, as the rule).
constexpr int kPaperLanes = 1024;
template <bool SUM>
__device__ double paper_residual(const PaperArgs& A, const double* u, double* red) {
    const int m = A.m, mi = m - 2, N = mi * (A.n - 2), nt = blockDim.x;
    const float inv = 1.0f / (float)mi;
    const auto res = [&](int q) {
        const int jj = seg_div(q, inv), i = 1 + q - jj * mi, j = 1 + jj;
        const int p = j * m + i;
        const double Lu = (A.cx * (u[p - 1] + u[p + 1]) + A.cy * (u[p - m] + u[p + m])) - A.d * u[p];
        return (A.f != nullptr ? A.f[(size_t)j * A.P + i] : 0.0) - Lu;
    };
    if constexpr (!SUM) {
        double mx = 0.0;
        for (int q = threadIdx.x; q < N; q += nt) mx = fmax(mx, fabs(res(q)));
        return block_max(mx, red);
    }
    for (int v = 0; v < N && v < kPaperLanes; v += nt) {
        double s2 = 0.0;
        for (int q = v + (int)threadIdx.x; q < N; q += kPaperLanes) {
            const double r = res(q);
            s2 = s2 + r * r;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s2 += __shfl_xor(s2, o);
        if ((threadIdx.x & 63) == 0) red[(v + (int)threadIdx.x) >> 6] = s2;
    }
    __syncthreads();
    double s = red[0];
    for (int k = 1; k < min((N + 63) >> 6, kPaperRed); ++k) s = s + red[k];
    __syncthreads();
    return s;
}

// The monitored quantity of the stopping rule after an iteration: the
// largest update max|psi - psi_start| (Eq. (16); mx, the thread's largest,
// taken where the nodes were updated), max|r| or ||r||_2 / ||r_0||_2.
__device__ double paper_monitor(const PaperArgs& A, const double* u, double mx, double r0, double* red) {
    if (A.stop == LAP_STOP_DELTA) return block_max(mx, red);
    if (A.stop == LAP_STOP_REL_L2) {
        const double s = paper_residual<true>(A, u, red);
        return r0 > 0.0 ? sqrt(s) / r0 : 0.0;
    }
    return paper_residual<false>(A, u, red);
}

// LDS (doubles): reduction slots (16), for the line methods their scratch and
// factors (tables: 9 (max(m, n) + kPaperPad), rounded up to pairs; else 3
// max(m, n) of scratch alone), u (n x m, row stride m) and a second field
// (Jacobi: the other iterate; ADI: the values at the start of the iteration).
__host__ __device__ constexpr int paper_pad(int m, int n) { return ((m > n ? m : n) + kPaperPad + 1) / 2 * 2; }
__host__ __device__ constexpr int paper_scratch(int m, int n, bool lines, bool tables) {
    return lines ? (tables ? 9 * paper_pad(m, n) : 3 * (m > n ? m : n)) : 0;
}

// NT: the largest workgroup.  The sequential methods sweep in its first
// wavefront, the others meet it at the monitor.
template <int NT, bool LINES>
__global__ __launch_bounds__(NT) void k_paper(PaperArgs A, int tables) {
    extern __shared__ double2 lds2[];
    double* lds = reinterpret_cast<double*>(lds2);
    const int m = A.m, n = A.n, N = (m - 2) * (n - 2), nt = blockDim.x;
    double* red = lds;
    double* sc = lds + kPaperRed;
    double* u = sc + paper_scratch(m, n, LINES, tables != 0);
    double* u0 = u + (size_t)m * n;
    for (int q = threadIdx.x; q < m * n; q += nt) {
        const int i = q % m, j = q / m;
        u0[q] = u[q] = A.u[(size_t)j * A.P + i];
    }
    __syncthreads();
    double r0 = 0.0;
    if (A.stop == LAP_STOP_REL_L2) r0 = sqrt(paper_residual<true>(A, u, red));
    const double cx = A.cx, cy = A.cy, inv_d = A.inv_d, w = A.omega;
    // the line systems: a x_{k-1} + d x_k + a x_{k+1} = r_k, a = -c (-w c inside)
    const int L = paper_pad(m, n), Lp = m > n ? m : n;
    double2* xq = reinterpret_cast<double2*>(sc);
    PaperFactor Fx, Fy;
    Fx.a = A.form == 0 ? -cx : -w * cx;
    Fy.a = A.form == 0 ? -cy : -w * cy;
    Fx.y = xq + L;
    Fy.y = xq + 2 * L;
    double* rhs = sc + 6 * L;
    Fx.cp = rhs + L;
    Fy.cp = rhs + 2 * L;
    if (LINES && tables) {
        // the two directions' chains of divisions side by side (a lane each)
        const bool y = threadIdx.x == 1;
        PaperFactor F;
        F.a = y ? Fy.a : Fx.a;
        F.cp = y ? Fy.cp : Fx.cp;
        F.y = y ? Fy.y : Fx.y;
        if (threadIdx.x < 2) paper_factor(F, A.d, y ? n - 2 : m - 2);
        __syncthreads();
    }
    int it = 0, status = 0, done = 0;
    double q = 0.0;
    while (it < A.max_iter) {
        double mx = 0.0;
        if constexpr (LINES) {
            // SLOR: rows j = 1..n-2; ADI: the rows, then columns i = 1..m-2
            const bool adi = A.method == LAP_ADI_LEX;
            if (NT == 64 || threadIdx.x < 64) {
                for (int j = 1; j <= n - 2; ++j) {
                    double* const keep = adi ? u0 : nullptr;
                    mx = fmax(mx, tables ? paper_line<true, NT>(A, u, keep, j, 0, Fx, rhs, xq)
                                         : paper_line_plain<true, NT>(A, u, keep, j, 0, Fx.a, sc, sc + Lp, sc + 2 * Lp));
                }
                if (adi) {
                    mx = 0.0;
                    for (int i = 1; i <= m - 2; ++i)
                        mx = fmax(mx, tables ? paper_line<false, NT>(A, u, u0, i, 1, Fy, rhs, xq)
                                             : paper_line_plain<false, NT>(A, u, u0, i, 1, Fy.a, sc, sc + Lp, sc + 2 * Lp));
                }
            }
        } else if (A.method == LAP_JACOBI) {
            // every node from the values at the start of the iteration
            double* t = u0; u0 = u; u = t;
            for (int k = threadIdx.x; k < N; k += nt) {
                const int i = 1 + k % (m - 2), j = 1 + k / (m - 2);
                const int p = j * m + i;
                const double fv = A.f != nullptr ? A.f[(size_t)j * A.P + i] : 0.0;
                const double v = ((cx * (u0[p - 1] + u0[p + 1]) + cy * (u0[p - m] + u0[p + m])) - fv) * inv_d;
                u[p] = v;
                mx = fmax(mx, fabs(v - u0[p]));
            }
        } else if (threadIdx.x < 64) {
            // lexicographic SOR: anti-diagonals d = i + j in increasing order; node (i, d - i)
            // lies at d m - i (m - 1), a scalar and a constant of the lane
            const int lane = threadIdx.x, um = 1 - m, fm = 1 - A.P;
            for (int dg = 2; dg <= (m - 2) + (n - 2); ++dg) {
                const int ilo = dg - (n - 2) > 1 ? dg - (n - 2) : 1;
                const int ihi = dg - 1 < m - 2 ? dg - 1 : m - 2;
                int p = (dg - ilo) * m + ilo + lane * um, fp = (dg - ilo) * A.P + ilo + lane * fm;
                for (int i = ilo + lane; i <= ihi; i += 64, p += 64 * um, fp += 64 * fm) {
                    const double fv = A.f != nullptr ? A.f[fp] : 0.0;
                    const double old = u[p];
                    const double t = ((cx * (u[p - 1] + u[p + 1]) + cy * (u[p - m] + u[p + m])) - fv) * inv_d;
                    const double v = old + w * (t - old);
                    u[p] = v;
                    mx = fmax(mx, fabs(v - old));
                }
                paper_sync<NT>();
            }
        }
        if constexpr (!LINES || NT > 64) __syncthreads();   // (a lone wavefront's lines end with one)
        ++it;
        q = paper_monitor(A, u, mx, r0, red);
        if (!isfinite(q) || q > 1e30) {
            status = LAP_EDIVERGED;
            done = 1;
            break;
        }
        if (q < A.tol) {
            done = 1;
            break;
        }
    }
    for (int p = threadIdx.x; p < m * n; p += nt) {
        const int i = p % m, j = p / m;
        A.u[(size_t)j * A.P + i] = u[p];
    }
    if (threadIdx.x == 0) {
        A.ctrl->iters = it;
        A.ctrl->done = done;
        A.ctrl->status = status;
        A.ctrl->rel = q;          // the last monitored quantity
        A.ctrl->r0 = r0;
        A.ctrl->checks = it;
    }
}

size_t paper_lds_bytes(int m, int n) {
    const int L = m > n ? m : n;
    return (2 * (size_t)m * n + 3 * (size_t)L + 16) * sizeof(double);
}

hipError_t paper_set_lds_limit(int bytes) {
    for (const void* f : {(const void*)k_paper<64, true>, (const void*)k_paper<256, true>, (const void*)k_paper<64, false>,
                          (const void*)k_paper<1024, false>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_paper(const PaperArgs& a, int lds_max, hipStream_t s) {
    const bool lines = a.method == LAP_SLOR_LEX || a.method == LAP_ADI_LEX;
    const auto need = [&](bool tables) {
        return (2 * (size_t)a.m * a.n + kPaperRed + paper_scratch(a.m, a.n, lines, tables)) * sizeof(double);
    };
    const bool tables = need(true) <= (size_t)lds_max;
    const size_t bytes = need(tables);
    const int N = (a.m - 2) * (a.n - 2);
    const bool residual = a.stop != LAP_STOP_DELTA;
    if (lines) {
        // four wavefronts for the monitor: with more, the chain's registers would be cut
        if (residual && N > 64)
            k_paper<256, true><<<1, 256, bytes, s>>>(a, tables ? 1 : 0);
        else
            k_paper<64, true><<<1, 64, bytes, s>>>(a, tables ? 1 : 0);
        return hipGetLastError();
    }
    // Jacobi, and a residual after SOR by diagonals: one to four nodes a thread, four wavefronts to a
    // barrier, or sixteen (33 x 33 to max|r|, 100 Jacobi iterations: 185 us with 256 threads, 223
    // with 1024); the sum of a relative residual, whose lanes' order is given, a node a lane (the
    // chamber, 100 iterations: 135 us with 384 threads, 182 with 256); SOR to its largest update: a
    // wavefront
    int threads = a.method == LAP_JACOBI || (residual && N > 64) ? (N <= 1024 ? 256 : 1024) : 64;
    if (a.stop == LAP_STOP_REL_L2) threads = std::min(kPaperLanes, (N + 63) / 64 * 64);
    if (threads == 64)
        k_paper<64, false><<<1, 64, bytes, s>>>(a, 0);
    else
        k_paper<1024, false><<<1, threads, bytes, s>>>(a, 0);
    return hipGetLastError();
}

}  // namespace lap
