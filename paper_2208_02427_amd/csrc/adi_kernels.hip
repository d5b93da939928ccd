// gfx950 kernels of line ADI: batched Thomas solves of all rows (or all
// columns) of one parity (zebra order), SLOR/ADI sections of the paper,
// Eqs. (8)-(10).
//
// Line system of row j (unknowns i = 1..m-2), relaxation after (SLORA):
//     -cx t_{i-1} + d t_i - cx t_{i+1} = cy (u_{i,j-1} + u_{i,j+1}) - f_ij
//     (+ cx u_{0,j} on the first, + cx u_{m-1,j} on the last unknown),
//     then u <- u + w (t - u);
// relaxation inside (SLORB):
//     -w cx t_{i-1} + d t_i - w cx t_{i+1} = (1-w) d u_ij + w (cy (...) - f_ij)
//     (+ w cx times the end values), then u <- t.
// Columns mirror it with x and y exchanged.  The coefficients are constant
// along a line, so the factorisation c'_k, pivot_k is computed once on the
// host; the kernels do the forward elimination and back substitution.
// Expression order and divisions follow the plain definition exactly (no
// fused multiply-add: the file is built with -ffp-contract=off).
//
// Two solvers.  The segmented one (lines of up to 4095 unknowns) splits every
// line into short blocks solved in parallel and couples them through a small
// reduced system (see lap_kernels.hpp); it reads and writes every value once.  The sequential
// one serves longer lines: columns, one thread per column line, marching j
// (consecutive threads own consecutive lines, so every row access of a
// wavefront is one contiguous span); rows, one 64-lane wavefront owns 64 row
// lines and moves through 64-column chunks, each chunk loaded / stored row by
// row through an LDS tile in which each lane walks its own line.  The
// sequential solver follows the plain recurrence (divisions, no fused
// multiply-add); the segmented one multiplies by tabulated reciprocals and
// fuses, so the two agree to rounding.
//
// The segmented solver is bound by latency: a wavefront's round trips, and the
// few thousand instructions of its serial elimination.  Hence no branch on
// lengths inside a block (addresses are clamped and values selected): with one a
// row, the column kernel waited for each of its 16 rows before it asked
// for the next, and every table value was an LDS round trip in the chain.
// Whole solves, branches a row against none: zebra multigrid of 641 x 385 3.12 ->
// 2.52 ms (columns 9.8 -> 6.4 us a launch, rows 7.2 -> 6.1), 20 ADI iterations of
// 2049 x 1500 1.38 -> 1.24 ms.
#include <cmath>
#include <cstring>
#include <type_traits>

#include "lap_kernels.hpp"
#include "stencil_tiles.hpp"

namespace lap {

// ------------------------------------------------------------------ columns
// Column line number t of the parity in A (no-op past the last line).
static __device__ void adi_col_line(const LineArgs& A, int t) {
    const int i = (A.parity ? 1 : 2) + 2 * t;
    if (i > A.m - 2) return;
    const int K = A.n - 2;
    const size_t P = (size_t)A.P;
    // in the column frame the coupling along the line is cy and across it cx
    const double cl = A.cy, cc = A.cx, d = A.d, w = A.omega, a = A.a_off;
    double rp = 0.0;
    for (int k = 0; k < K; ++k) {
        const int j = k + 1;
        const double* row = A.u + (size_t)j * P;
        const double base = cc * (row[i - 1] + row[i + 1]) - (A.f != nullptr ? A.f[(size_t)j * P + i] : 0.0);
        double r;
        if (A.form == 0) {
            r = base;
            if (k == 0) r = r + cl * A.u[i];
            if (k == K - 1) r = r + cl * A.u[(size_t)(A.n - 1) * P + i];
        } else {
            r = (1.0 - w) * d * row[i] + w * base;
            if (k == 0) r = r + w * cl * A.u[i];
            if (k == K - 1) r = r + w * cl * A.u[(size_t)(A.n - 1) * P + i];
        }
        rp = (k == 0) ? r / A.piv[0] : (r - a * rp) / A.piv[k];
        A.scratch[(size_t)j * P + t] = rp;
    }
    double x = 0.0;
    for (int k = K - 1; k >= 0; --k) {
        const int j = k + 1;
        const double q = A.scratch[(size_t)j * P + t];
        x = (k == K - 1) ? q : q - A.cprime[k] * x;
        double* p = A.u + (size_t)j * P + i;
        const double old = *p;
        *p = (A.form == 0) ? old + w * (x - old) : x;
    }
}

__global__ __launch_bounds__(kBlock) void k_adi_cols(LineArgs A) {
    if (A.ctrl != nullptr && A.ctrl->done) return;
    adi_col_line(A, blockIdx.x * blockDim.x + threadIdx.x);
}

hipError_t launch_adi_cols_seg(const LineArgs& a, int lines, hipStream_t s);

hipError_t launch_adi_cols(const LineArgs& a, hipStream_t s) {
    const int first = a.parity ? 1 : 2;
    const int lines = a.m - 2 >= first ? (a.m - 2 - first) / 2 + 1 : 0;
    if (lines <= 0) return hipSuccess;
    if (a.seg != nullptr && seg_fits(1, a.n - 2)) return launch_adi_cols_seg(a, lines, s);
    const int nb = (lines + kBlock - 1) / kBlock;
    k_adi_cols<<<nb, kBlock, 0, s>>>(a);
    return hipGetLastError();
}

// --------------------------------------------------------------------- rows

// Row lines 64*blk .. 64*blk+63 of the parity in A, one lane per line
// (block of 64 threads; tile / told are LDS scratch of 64 x 65 doubles).
static __device__ void adi_rows_block(const LineArgs& A, int blk, double (*tile)[kRowTile + 1],
                               double (*told)[kRowTile + 1]) {
    const int lane = threadIdx.x;
    const int first = A.parity ? 1 : 2;
    const int nlines = A.n - 2 >= first ? (A.n - 2 - first) / 2 + 1 : 0;
    const int line0 = blk * kRowTile;
    const int mylines = min(kRowTile, nlines - line0);
    const int K = A.m - 2;
    const size_t P = (size_t)A.P;
    const double cl = A.cx, cc = A.cy, d = A.d, w = A.omega, a = A.a_off;
    const int myj = first + 2 * (line0 + lane);          // this lane's row (valid if lane < mylines)
    const int nchunks = (K + kRowTile - 1) / kRowTile;
    // scratch row of line l: the line's own row j (distinct lines never share it)
    double rp = 0.0;
    for (int ch = 0; ch < nchunks; ++ch) {
        const int ic = 1 + ch * kRowTile;                 // first unknown of the chunk
        const int i = ic + lane;                          // column loaded by this lane
        for (int rr = 0; rr < mylines; ++rr) {
            const int j = first + 2 * (line0 + rr);
            if (i <= A.m - 2) {
                const double* row = A.u + (size_t)j * P;
                const double base = cc * (A.u[(size_t)(j - 1) * P + i] + A.u[(size_t)(j + 1) * P + i]) -
                                    (A.f != nullptr ? A.f[(size_t)j * P + i] : 0.0);
                tile[rr][lane] = (A.form == 0) ? base : (1.0 - w) * d * row[i] + w * base;
            }
        }
        __syncthreads();
        if (lane < mylines) {
            const int kend = min(kRowTile, K - ch * kRowTile);
            for (int kk = 0; kk < kend; ++kk) {
                const int k = ch * kRowTile + kk;
                double r = tile[lane][kk];
                if (k == 0) r = r + (A.form == 0 ? cl : w * cl) * A.u[(size_t)myj * P];
                if (k == K - 1) r = r + (A.form == 0 ? cl : w * cl) * A.u[(size_t)myj * P + A.m - 1];
                rp = (k == 0) ? r / A.piv[0] : (r - a * rp) / A.piv[k];
                tile[lane][kk] = rp;
            }
        }
        __syncthreads();
        for (int rr = 0; rr < mylines; ++rr) {
            const int j = first + 2 * (line0 + rr);
            if (i <= A.m - 2) A.scratch[(size_t)j * P + i] = tile[rr][lane];
        }
        __syncthreads();
    }
    double x = 0.0;
    for (int ch = nchunks - 1; ch >= 0; --ch) {
        const int ic = 1 + ch * kRowTile;
        const int i = ic + lane;
        for (int rr = 0; rr < mylines; ++rr) {
            const int j = first + 2 * (line0 + rr);
            if (i <= A.m - 2) {
                tile[rr][lane] = A.scratch[(size_t)j * P + i];
                told[rr][lane] = A.u[(size_t)j * P + i];
            }
        }
        __syncthreads();
        if (lane < mylines) {
            const int kend = min(kRowTile, K - ch * kRowTile);
            for (int kk = kend - 1; kk >= 0; --kk) {
                const int k = ch * kRowTile + kk;
                const double q = tile[lane][kk];
                x = (k == K - 1) ? q : q - A.cprime[k] * x;
                const double old = told[lane][kk];
                tile[lane][kk] = (A.form == 0) ? old + w * (x - old) : x;
            }
        }
        __syncthreads();
        for (int rr = 0; rr < mylines; ++rr) {
            const int j = first + 2 * (line0 + rr);
            if (i <= A.m - 2) A.u[(size_t)j * P + i] = tile[rr][lane];
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(64) void k_adi_rows(LineArgs A) {
    if (A.ctrl != nullptr && A.ctrl->done) return;
    __shared__ double tile[kRowTile][kRowTile + 1];
    __shared__ double told[kRowTile][kRowTile + 1];
    adi_rows_block(A, blockIdx.x, tile, told);
}

hipError_t launch_adi_rows_seg(const LineArgs& a, int lines, hipStream_t s);

hipError_t launch_adi_rows(const LineArgs& a, hipStream_t s) {
    const int first = a.parity ? 1 : 2;
    const int lines = a.n - 2 >= first ? (a.n - 2 - first) / 2 + 1 : 0;
    if (lines <= 0) return hipSuccess;
    if (a.seg != nullptr && seg_fits(0, a.m - 2)) return launch_adi_rows_seg(a, lines, s);
    const int nb = (lines + kRowTile - 1) / kRowTile;
    k_adi_rows<<<nb, kRowTile, 0, s>>>(a);
    return hipGetLastError();
}

// --------------------------------------------------------- segmented solver
// Templated on the element type T of the field: FP64 for the ADI method,
// FP32 as well for zebra line smoothing inside the mixed-precision V-cycle.
// Every operation of a T solve is done in T with T coefficients and a T
// table (the FP32 table is the extended-precision one rounded once).
static_assert(kSegL + 1 == 16, "block index arithmetic assumes 16 unknowns per block and separator");
constexpr int kSegBS = kSegL + 2;   // LDS slots of a row block: kSegL unknowns, separator, separator value

template <typename T>
void adi_seg_table_t(double Dd, double Ed, int K, T* tab) {
    std::memset(tab, 0, sizeof(T) * kSegTab);
    if (K <= 0) return;
    typedef long double R;
    const int L = kSegL;
    const int S = seg_count(K);
    const int Ll = K - (S - 1) * (L + 1);
    const R D = Dd, E = Ed;
    R piv[kSegL], cq[kSegL];
    piv[0] = D;
    for (int k = 1; k < L; ++k) piv[k] = D - E * E / piv[k - 1];
    for (int k = 0; k < L; ++k) cq[k] = E / piv[k];
    // response of a block of length len to a unit value left of it:
    // solve tridiag(-E, D, -E) g = E e_1
    auto resp = [&](int len, R* g) {
        R z = 0;
        for (int k = 0; k < len; ++k) {
            z = ((k == 0 ? E : (R)0) + E * z) / piv[k];
            g[k] = z;
        }
        for (int k = len - 2; k >= 0; --k) g[k] = g[k] + cq[k] * g[k + 1];
    };
    R g[kSegL] = {}, gl[kSegL] = {};
    resp(L, g);
    resp(Ll, gl);
    for (int k = 0; k < L; ++k) {
        tab[SEG_IPIV + k] = (T)(1 / piv[k]);
        tab[SEG_CQ + k] = (T)cq[k];
        tab[SEG_G + k] = (T)g[k];
        tab[SEG_GL + k] = (T)gl[k];
    }
    tab[SEG_E] = (T)Ed;
    // one block only, or more separators than the table holds (such lines
    // take the sequential solver)
    if (S < 2 || S > kSegMaxS) return;
    // reduced system over the separators: tridiag(-E_R, D_R, -E_R), the last
    // separator couples to the last block (or, if that is empty, to nothing)
    const R ER = E * g[L - 1];
    const R DR = D - 2 * E * g[0];
    const R DRend = D - E * g[0] - (Ll > 0 ? E * gl[0] : (R)0);
    const int NR = S - 1;
    R pv = 0;
    for (int p = 0; p < NR; ++p) {
        const R dg = (p == NR - 1) ? DRend : DR;
        pv = (p == 0) ? dg : dg - ER * ER / pv;
        tab[SEG_IPIVR + p] = (T)(1 / pv);
        tab[SEG_CQR + p] = (T)(ER / pv);
    }
    tab[SEG_E + 1] = (T)ER;
    // reach of the reduced system's scans: a separator h blocks away enters
    // with a factor of at most amax^h, amax = max E_R / pivot_p; from the
    // distance on where amax^h / (1 - amax) is below 2^-60 (FP32: 2^-31) of
    // the line's largest value, a seventh bit below its rounding, further
    // scan steps only add what rounding drops.  Against the line's largest
    // value, that is: a value many orders below it keeps this error, not one
    // of its own size, and a NaN or infinity on a line spreads as far as the
    // reach in one solve, not over the whole line.
    R amax = 0;
    for (int p = 0; p < NR; ++p) amax = std::max(amax, std::fabs((R)tab[SEG_CQR + p]));
    const R drop = std::ldexp((R)1, sizeof(T) == 8 ? -60 : -31);
    int reach = 1;
    for (R a = amax; reach < NR && !(a < drop * (1 - amax)); reach *= 2) a = a * a;
    tab[SEG_E + 2] = (T)reach;
}

void adi_seg_table(double D, double E, int K, double* tab) { adi_seg_table_t<double>(D, E, K, tab); }
void adi_seg_table(double D, double E, int K, float* tab) { adi_seg_table_t<float>(D, E, K, tab); }

// Right-hand side of one unknown from its own old value, the sum of its two
// neighbours across the line and f (end values are added by the caller).
template <typename T>
__device__ __forceinline__ T seg_rhs(const LineArgsT<T>& A, T cc, T own, T nb, T fv) {
    const T base = cc * nb - fv;
    return A.form == 0 ? base : (T(1) - (T)A.omega) * (T)A.d * own + (T)A.omega * base;
}

// Forward elimination of one block given its right-hand sides r[0..len)
// (len <= kSegL, zeros behind); leaves the block's zero-end solution in r,
// returns its last value in *last.  Tb: the table's block part, in LDS.
// Without branches on len: a branch a row kept the table's reads from being
// issued ahead, an LDS round trip for each.  What the rows behind len hold
// reaches nothing: their coefficient and value enter the substitution as zeros.
template <typename T>
__device__ __forceinline__ void seg_block(const T* Tb, T E, int len, T (&r)[kSegL], T* last) {
    T ip[kSegL], cq[kSegL];
#pragma unroll
    for (int k = 0; k < kSegL; ++k) {
        ip[k] = Tb[SEG_IPIV + k];
        cq[k] = Tb[SEG_CQ + k];
    }
    T z = 0;
#pragma unroll
    for (int k = 0; k < kSegL; ++k) {
        z = fma(E, z, r[k]) * ip[k];
        r[k] = z;
    }
    T x = 0, e = 0;
#pragma unroll
    for (int k = kSegL - 1; k >= 0; --k) {
        x = fma(k < len - 1 ? cq[k] : T(0), x, k < len ? r[k] : T(0));
        r[k] = x;
        e = k == len - 1 ? x : e;
    }
    *last = e;
}

// The block's solution from its zero-end solution y and the values xl, xr
// of the separators beside it (full: a separator follows it).
template <typename T>
__device__ __forceinline__ void seg_apply(const T* Tb, bool full, T xl, T xr, T (&y)[kSegL]) {
    T g[kSegL], h[kSegL];
#pragma unroll
    for (int k = 0; k < kSegL; ++k) {
        g[k] = Tb[(full ? SEG_G : SEG_GL) + k];
        h[k] = Tb[SEG_G + kSegL - 1 - k];
    }
#pragma unroll
    for (int k = 0; k < kSegL; ++k) {
        const T t = fma(xl, g[k], y[k]);
        y[k] = full ? fma(xr, h[k], t) : t;
    }
}

// Reduced system of one line, its unknown p held by one thread (act; NR
// and the loop trip counts are uniform over the workgroup, every thread
// reaches every barrier).  The forward elimination z_p = (rho_p + E_R
// z_{p-1}) / pivot_p and the back substitution x_p = z_p + (E_R / pivot_p)
// x_{p+1} are first-order linear recurrences: each is evaluated as a
// Hillis-Steele scan of affine maps through two LDS buffer pairs (a0, b0),
// (a1, b1) addressed by slot(p).  The scan stops at the table's reach: the
// line matrix is diagonally dominant, so E_R / pivot is tiny (7e-10 at
// dx = dy) and one step, not log2 NR = 7 at 94 blocks, is all that FP64 can
// see.  ip, cq: 1 / pivot_p and E_R / pivot_p.  Returns x_p.
template <typename T, typename Slot>
__device__ __forceinline__ T seg_scan(T ER, T ip, T cq, int reach, int NR, int p, bool act, T rho, Slot slot,
                                      T* a0, T* b0, T* a1, T* b1) {
    T a = 0, b = 0;
    if (act) {
        a = p > 0 ? ER * ip : T(0);
        b = rho * ip;
        a0[slot(p)] = a;
        b0[slot(p)] = b;
    }
    __syncthreads();
    T *ra = a0, *rb = b0, *wa = a1, *wb = b1;
    for (int h = 1; h < reach; h <<= 1) {
        if (act) {
            if (p >= h) {
                const int q = slot(p - h);
                b = fma(a, rb[q], b);
                a = a * ra[q];
            }
            wa[slot(p)] = a;
            wb[slot(p)] = b;
        }
        __syncthreads();
        T* t = ra; ra = wa; wa = t;
        t = rb; rb = wb; wb = t;
    }
    // b = z_p; now x_p = c_p x_{p+1} + z_p, scanned from the end (the
    // buffers last read may still be in use: write the other pair)
    T c = (act && p < NR - 1) ? cq : T(0);
    if (act) {
        wa[slot(p)] = c;
        wb[slot(p)] = b;
    }
    __syncthreads();
    { T* t = ra; ra = wa; wa = t; t = rb; rb = wb; wb = t; }
    for (int h = 1; h < reach; h <<= 1) {
        if (act) {
            if (p + h < NR) {
                const int q = slot(p + h);
                b = fma(c, rb[q], b);
                c = c * ra[q];
            }
            if (2 * h < reach) {
                wa[slot(p)] = c;
                wb[slot(p)] = b;
            }
        }
        if (2 * h < reach) __syncthreads();
        T* t = ra; ra = wa; wa = t;
        t = rb; rb = wb; wb = t;
    }
    return b;
}

// The table's block part (SEG_IPIV .. SEG_GL) goes to LDS: read first, before
// the field's loads, and stored behind them, so that neither waits for it.
constexpr int kSegHead = 4 * kSegL;
template <typename T>
__device__ __forceinline__ T seg_table_load(const T* Tb) {
    return Tb[min((int)threadIdx.x, kSegHead - 1)];
}
template <typename T>
__device__ __forceinline__ void seg_table_store(T v, T* tab) {
    if (threadIdx.x < kSegHead) tab[threadIdx.x] = v;
}

// Two consecutive values of a row (aligned to one value only).
template <typename T> struct SegPair;
template <> struct SegPair<double> { typedef double type __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct SegPair<float> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };

// Whether the solve is over; read behind the issued loads (in place, only
// the stores at the end depend on it), so its latency is not waited for first.
__device__ __forceinline__ bool seg_done(const Ctrl* ctrl) {
    asm volatile("" ::: "memory");   // the loads above stay above
    return ctrl != nullptr && ctrl->done;
}

// Row lines of the parity in A, tile `tile` (W = NT / S lines), one
// workgroup of NT threads.  The lines are read in pairs of unknowns (coalesced,
// 16 bytes a lane in FP64), eight pairs a thread, their right-hand sides
// staged in LDS and their old values kept in registers; thread (line c, block
// s), s fastest, solves its block from LDS; the solution goes back through
// LDS and is written in the same pairs with the relaxation.  Bound by
// latency: one round trip for all of a thread's loads, then the block's
// serial elimination.  lds: NT * kSegBS + kSegHead values.
template <typename T, int NT>
static __device__ void adi_rows_seg(const LineArgsT<T>& A, const Ctrl* ctrl, int tile, T* lds) {
    typedef typename SegPair<T>::type T2;
    const int K = A.m - 2;
    const int S = seg_count(K);
    const int W = NT / S;
    const int first = A.parity ? 1 : 2;
    const int nlines = A.n - 2 >= first ? (A.n - 2 - first) / 2 + 1 : 0;
    const int line0 = tile * W;
    const int nl = min(W, nlines - line0);
    if (nl <= 0) return;
    const size_t P = (size_t)A.P;
    const T* Tg = A.seg;
    T* Tb = lds + NT * kSegBS;
    const T cc = (T)A.cy;
    const int LW = S * kSegBS;
    const int tid = threadIdx.x;
    // pair q of the tile: unknowns k, k + 1 (k = 2 (q % NP)) of line q / NP;
    // K < 16 S, so W lines have at most 8 NT pairs
    const int NP = (K + 1) >> 1;
    const int total = nl * NP;
    const float invN = 1.0f / (float)NP;
    constexpr int kU = 8, kG = sizeof(T) == 8 ? 4 : 8;   // pairs per thread; in flight at once
    T2 own[kU];
    const int c = seg_div(tid, 1.0f / (float)S);
    const int s = tid - c * S;
    const bool act = c < nl;
    const bool sep = act && s < S - 1;
    const T E = Tg[SEG_E];
    T ip = 0, cq = 0;
    const T ER = Tg[SEG_E + 1];
    const int reach = __builtin_amdgcn_readfirstlane((int)Tg[SEG_E + 2]);
    if (sep) {
        ip = Tg[SEG_IPIVR + s];
        cq = Tg[SEG_CQR + s];
    }
    const T tv = seg_table_load<T>(Tg);
#pragma unroll
    for (int g = 0; g < kU; g += kG) {
        T2 up[kG], dn[kG], fv[kG];
        T end[kG];
        int slot[kG];
        bool two[kG];
#pragma unroll
        for (int v = 0; v < kG; ++v) {
            const int q = tid + (g + v) * NT;
            slot[v] = -1;
            two[v] = false;
            up[v] = dn[v] = fv[v] = own[g + v] = T2{0, 0};
            end[v] = 0;
            if (q < total) {
                const int l = seg_div(q, invN);
                const int k = 2 * (q - l * NP);
                const size_t row = (size_t)(first + 2 * (line0 + l)) * P;
                const size_t o = row + k + 1;      // k + 1 <= K: the pair ends at node m - 1 at most
                own[g + v] = *reinterpret_cast<const T2*>(A.u + o);
                up[v] = *reinterpret_cast<const T2*>(A.u + o - P);
                dn[v] = *reinterpret_cast<const T2*>(A.u + o + P);
                if (A.f != nullptr) fv[v] = *reinterpret_cast<const T2*>(A.f + o);
                if (k == 0) end[v] = A.u[row];
                if (k + 2 == K) end[v] = A.u[row + A.m - 1];
                slot[v] = l * LW + (k >> 4) * kSegBS + (k & 15);
                two[v] = k + 1 < K;
                // K = 1 or 2: a pair holding both ends (its left end is added below)
            }
        }
        if (g == 0) {
            if (seg_done(ctrl)) return;            // uniform over the workgroup
            seg_table_store<T>(tv, Tb);
        }
#pragma unroll
        for (int v = 0; v < kG; ++v) {
            if (slot[v] < 0) continue;
            const int q = tid + (g + v) * NT;
            const int l = seg_div(q, invN);
            const int k = 2 * (q - l * NP);
            const T2 o2 = own[g + v];
            T r0 = seg_rhs<T>(A, cc, o2.x, up[v].x + dn[v].x, fv[v].x);
            T r1 = seg_rhs<T>(A, cc, o2.y, up[v].y + dn[v].y, fv[v].y);
            if (k == 0) r0 = r0 + E * (k + 2 == K ? A.u[(size_t)(first + 2 * (line0 + l)) * P] : end[v]);
            if (k + 1 == K) r0 = r0 + E * o2.y;                 // the line's last unknown; o2.y is its end value
            if (k + 2 == K) r1 = r1 + E * end[v];
            lds[slot[v]] = r0;
            if (two[v]) lds[slot[v] + 1] = r1;
        }
    }
    __syncthreads();
    const int len = s < S - 1 ? kSegL : K - (S - 1) * (kSegL + 1);
    T* blk = lds + c * LW + s * kSegBS;
    T y[kSegL];
    if (act) {
#pragma unroll
        for (int k = 0; k < kSegL; ++k) y[k] = k < len ? blk[k] : T(0);
        T e;
        seg_block<T>(Tb, E, len, y, &e);
        blk[0] = len > 0 ? y[0] : T(0);
        blk[1] = e;
    }
    __syncthreads();
    if (S > 1) {
        // slots 2..5 of each block are free now (its unknowns live in y)
        const T rho = sep ? fma(E, blk[1] + blk[kSegBS], blk[kSegL]) : T(0);
        T* lb = lds + c * LW;
        const auto at = [](int p) { return p * kSegBS; };
        const T x = seg_scan<T>(ER, ip, cq, reach, S - 1, s, sep, rho, at, lb + 2, lb + 3, lb + 4, lb + 5);
        if (sep) blk[kSegL + 1] = x;
        __syncthreads();
    }
    if (act) {
        // (slots behind len are the block's own and read by no one)
        const T xl = s > 0 ? blk[kSegL + 1 - kSegBS] : T(0);
        const T xr = sep ? blk[kSegL + 1] : T(0);
        seg_apply<T>(Tb, sep, xl, xr, y);
#pragma unroll
        for (int k = 0; k < kSegL; ++k) blk[k] = y[k];
        if (sep) blk[kSegL] = xr;
    }
    __syncthreads();
    const T w = (T)A.omega;
#pragma unroll
    for (int v = 0; v < kU; ++v) {
        const int q = tid + v * NT;
        if (q >= total) continue;
        const int l = seg_div(q, invN);
        const int k = 2 * (q - l * NP);
        T* at = A.u + (size_t)(first + 2 * (line0 + l)) * P + k + 1;
        const int sl = l * LW + (k >> 4) * kSegBS + (k & 15);
        T2 t{lds[sl], lds[sl + 1]};
        if (A.form == 0) {
            t.x = own[v].x + w * (t.x - own[v].x);
            t.y = own[v].y + w * (t.y - own[v].y);
        }
        if (k + 1 < K)
            *reinterpret_cast<T2*>(at) = t;
        else
            *at = t.x;
    }
}

// Column lines of the parity in A, tile `tile` (W lines, seg_lines), one
// workgroup of NT threads; thread (line c, block s), c fastest, so a
// wavefront's accesses to one row are contiguous.  A node and one of its
// neighbours across the line come in one aligned pair load, the other
// neighbour from the next pair (the same cache line).  Each thread keeps its
// block's old values and solution in registers.  sh: 5 * NT + kSegHead
// values (first block values, then separator values; scan buffers).
template <typename T, int NT>
static __device__ void adi_cols_seg(const LineArgsT<T>& A, const Ctrl* ctrl, int tile, T* sh) {
    typedef typename VecT<T, 2>::type T2;
    const int K = A.n - 2;
    const int S = seg_count(K);
    const int W = seg_lines_of(1, K, NT);
    const int first = A.parity ? 1 : 2;
    const int nlines = A.m - 2 >= first ? (A.m - 2 - first) / 2 + 1 : 0;
    const int line0 = tile * W;
    const int nl = min(W, nlines - line0);
    if (nl <= 0) return;
    const size_t P = (size_t)A.P;
    const T* Tg = A.seg;
    T* Tb = sh + 5 * NT;
    const T E = Tg[SEG_E], ER = Tg[SEG_E + 1];
    const int reach = __builtin_amdgcn_readfirstlane((int)Tg[SEG_E + 2]);
    const T cc = (T)A.cx;
    const int tid = threadIdx.x;
    const int s = tid >> (31 - __builtin_clz(W));      // W: a power of two
    const int c = tid - s * W;
    const bool act = c < nl && s < S;
    const bool sep = act && s < S - 1;
    const int len = s < S - 1 ? kSegL : K - (S - 1) * (kSegL + 1);
    const int i = first + 2 * (line0 + c);
    const int k0 = s * (kSegL + 1);
    const bool odd = (i & 1) != 0;                     // uniform over the launch
    T* yF = sh;
    const int me = s * W + c;
    T y[kSegL], old[kSegL];
    T osep = 0, rsep = 0, e = 0, ip = 0, cq = 0;
    const T tv = seg_table_load<T>(Tg);
    if (sep) {
        ip = Tg[SEG_IPIVR + s];
        cq = Tg[SEG_CQR + s];
    }
    if (act) {
        const T* up = A.u + (size_t)(k0 + 1) * P + (i & ~1);   // the node's aligned pair
        const int third = odd ? 2 : -1;
        const T* fp = A.f != nullptr ? A.f + (size_t)(k0 + 1) * P + i : nullptr;
        T head = 0, tail = 0;
        if (s == 0) head = A.u[i];
        if (s == S - 1 || k0 + kSegL == K - 1) tail = A.u[(size_t)(A.n - 1) * P + i];
        // rows behind the line's last one are read clamped to it, so that the
        // loads have no branches between them and kG rows' are in flight
        constexpr int kG = NT >= 1024 ? 4 : 8;
        const int klast = K - 1 - k0;                      // >= 0 wherever a row is used
        const auto rows = [&](auto has_f, int g0) {
            constexpr bool HF = decltype(has_f)::value;
            T2 q[kG];
            T t[kG], fv[kG];
#pragma unroll
            for (int v = 0; v < kG; ++v) {
                const ptrdiff_t o = (ptrdiff_t)min(g0 + v, klast) * (ptrdiff_t)P;
                q[v] = *reinterpret_cast<const T2*>(up + o);
                t[v] = up[o + third];
                fv[v] = HF ? fp[o] : T(0);
            }
#pragma unroll
            for (int v = 0; v < kG; ++v) {
                const int k = g0 + v;
                const T own = odd ? q[v].y : q[v].x;
                // the same sum of the west and east neighbours
                const T nb = odd ? q[v].x + t[v] : t[v] + q[v].y;
                const T r = seg_rhs<T>(A, cc, own, nb, fv[v]);
                if (k < kSegL) {
                    old[k] = own;
                    y[k] = k < len ? r : T(0);
                } else {
                    osep = own;
                    rsep = r;
                }
            }
        };
#pragma unroll
        for (int g0 = 0; g0 < kSegL + 1; g0 += kG) {
            if (fp != nullptr)
                rows(std::true_type{}, g0);
            else
                rows(std::false_type{}, g0);
        }
        if (s == 0) y[0] = y[0] + E * head;
        if (len > 0 && k0 + len == K) {
#pragma unroll
            for (int k = 0; k < kSegL; ++k) y[k] = k == len - 1 ? y[k] + E * tail : y[k];
        }
        if (s < S - 1 && k0 + kSegL == K - 1) rsep = rsep + E * tail;
    }
    if (seg_done(ctrl)) return;                        // uniform over the workgroup
    seg_table_store<T>(tv, Tb);
    __syncthreads();
    if (act) {
        seg_block<T>(Tb, E, len, y, &e);
        yF[me] = len > 0 ? y[0] : T(0);
    }
    __syncthreads();
    if (S > 1) {
        const T rho = sep ? fma(E, e + yF[me + W], rsep) : T(0);
        const auto at = [W, c](int p) { return p * W + c; };
        const T x = seg_scan<T>(ER, ip, cq, reach, S - 1, s, sep, rho, at, sh + NT, sh + 2 * NT, sh + 3 * NT,
                                sh + 4 * NT);
        // yF is free: every thread passed the scan's first barrier after reading it
        if (sep) yF[me] = x;
        __syncthreads();
    }
    if (act) {
        const T w = (T)A.omega;
        const T xl = s > 0 ? yF[me - W] : T(0);
        T* up = A.u + (size_t)(k0 + 1) * P + i;
        const T xr = sep ? yF[me] : T(0);
        seg_apply<T>(Tb, sep, xl, xr, y);
#pragma unroll
        for (int k = 0; k < kSegL; ++k) {
            const T t = (A.form == 0) ? old[k] + w * (y[k] - old[k]) : y[k];
            if (k < len) up[(size_t)k * P] = t;
        }
        if (sep) up[(size_t)kSegL * P] = (A.form == 0) ? osep + w * (xr - osep) : xr;
    }
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_adi_rows_seg(LineArgsT<T> A, int ntiles) {
    __shared__ T lds[NT * kSegBS + kSegHead];
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    if (t < ntiles) adi_rows_seg<T, NT>(A, A.ctrl, t, lds);
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_adi_cols_seg(LineArgsT<T> A, int ntiles) {
    __shared__ T sh[5 * NT + kSegHead];
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    if (t < ntiles) adi_cols_seg<T, NT>(A, A.ctrl, t, sh);
}

// ------------------------------------------------------- merged batch launches

template <typename T>
__device__ __forceinline__ LineArgsT<T> line_args(const BatchItem& it) {
    LineArgsT<T> a{};
    a.u = (T*)it.out;
    a.f = (const T*)it.f;
    a.scratch = it.scratch;
    a.cprime = it.cprime;
    a.piv = it.piv;
    a.ctrl = nullptr;
    a.m = it.m;
    a.n = it.n;
    a.P = it.P;
    a.cx = it.cx;
    a.cy = it.cy;
    a.d = it.d;
    a.omega = it.omega;
    a.a_off = it.a_off;
    a.form = it.flags;
    a.parity = it.parity;
    a.seg = (const T*)it.seg;
    return a;
}

// Row lines of all grids: one 64-lane block per 64-line block of a grid,
// the grid loops over all (grid, line block) tiles.
__global__ __launch_bounds__(64) void k_batch_adi_rows(const BatchItem* items, const int* tmap, int total) {
    __shared__ double tile[kRowTile][kRowTile + 1];
    __shared__ double told[kRowTile][kRowTile + 1];
    for (int t = blockIdx.x; t < total; t += gridDim.x) {
        const BatchItem& it = items[tmap[t]];
        if (it.ctrl->done) continue;
        adi_rows_block(line_args<double>(it), t - it.tile0, tile, told);
    }
}

// Column lines of all grids: one thread per line, 256 lines per tile.
__global__ __launch_bounds__(kBlock) void k_batch_adi_cols(const BatchItem* items, const int* tmap, int total) {
    for (int t = blockIdx.x; t < total; t += gridDim.x) {
        const BatchItem& it = items[tmap[t]];
        if (it.ctrl->done) continue;
        adi_col_line(line_args<double>(it), (t - it.tile0) * kBlock + threadIdx.x);
    }
}

// Segmented solver over all grids: tiles of seg_lines lines of one grid,
// dealt XCD-contiguously (neighbouring tiles share boundary lines).
template <typename T, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) void k_batch_adi_rows_seg(const BatchItem* items, const int* tmap, int total) {
    __shared__ T lds[NT * kSegBS + kSegHead];
    for (int t = xcd_remap(blockIdx.x, gridDim.x); t < total; t += gridDim.x) {
        const BatchItem& it = items[tmap[t]];
        adi_rows_seg<T, NT>(line_args<T>(it), it.ctrl, t - it.tile0, lds);
        __syncthreads();
    }
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_batch_adi_cols_seg(const BatchItem* items, const int* tmap, int total) {
    __shared__ T sh[5 * NT + kSegHead];
    for (int t = xcd_remap(blockIdx.x, gridDim.x); t < total; t += gridDim.x) {
        const BatchItem& it = items[tmap[t]];
        adi_cols_seg<T, NT>(line_args<T>(it), it.ctrl, t - it.tile0, sh);
        __syncthreads();
    }
}

template <typename T>
hipError_t launch_adi_rows_seg(const LineArgsT<T>& a, int lines, hipStream_t s) {
    const int W = seg_lines(0, a.m - 2);
    const int nt = (lines + W - 1) / W;
    switch (seg_code(0, a.m - 2)) {
        case 0: k_adi_rows_seg<T, 64><<<xcd_pad(nt), 64, 0, s>>>(a, nt); break;
        case 1: k_adi_rows_seg<T, 128><<<xcd_pad(nt), 128, 0, s>>>(a, nt); break;
        default: k_adi_rows_seg<T, 256><<<xcd_pad(nt), 256, 0, s>>>(a, nt); break;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adi_cols_seg(const LineArgsT<T>& a, int lines, hipStream_t s) {
    const int W = seg_lines(1, a.n - 2);
    const int nt = (lines + W - 1) / W;
    switch (seg_code(1, a.n - 2)) {
        case 0: k_adi_cols_seg<T, 64><<<xcd_pad(nt), 64, 0, s>>>(a, nt); break;
        case 1: k_adi_cols_seg<T, 256><<<xcd_pad(nt), 256, 0, s>>>(a, nt); break;
        case 2: k_adi_cols_seg<T, 512><<<xcd_pad(nt), 512, 0, s>>>(a, nt); break;
        default: k_adi_cols_seg<T, 1024><<<xcd_pad(nt), 1024, 0, s>>>(a, nt); break;
    }
    return hipGetLastError();
}

hipError_t launch_adi_rows_seg(const LineArgs& a, int lines, hipStream_t s) {
    return launch_adi_rows_seg<double>(a, lines, s);
}
hipError_t launch_adi_cols_seg(const LineArgs& a, int lines, hipStream_t s) {
    return launch_adi_cols_seg<double>(a, lines, s);
}

// Zebra line smoothing half (segmented solver only): lines of one parity of
// one direction, in place on a.u, FP64 or FP32.
template <typename T>
hipError_t launch_zebra_lines(const LineArgsT<T>& a, int dir, hipStream_t s) {
    const int first = a.parity ? 1 : 2;
    const int across = dir == 0 ? a.n - 2 : a.m - 2;
    const int K = dir == 0 ? a.m - 2 : a.n - 2;
    const int lines = across >= first ? (across - first) / 2 + 1 : 0;
    if (lines <= 0) return hipSuccess;
    if (a.seg == nullptr || !seg_fits(dir, K)) return hipErrorInvalidValue;
    return dir == 0 ? launch_adi_rows_seg<T>(a, lines, s) : launch_adi_cols_seg<T>(a, lines, s);
}
template hipError_t launch_zebra_lines<double>(const LineArgsT<double>&, int, hipStream_t);
template hipError_t launch_zebra_lines<float>(const LineArgsT<float>&, int, hipStream_t);

// ------------------------------------------- small-level tail of a zebra cycle
// All levels from one that fits LDS with its hierarchy down to the coarsest
// and back, in one workgroup.  As launches a level takes eight line halves, a
// restriction and a correction, 4 to 7 us each whatever its size (bound by
// the launch and one dependent chain of loads, barriers and eliminations);
// here they are the same device code on LDS, without the launch and the memory
// round trips.  256 threads: the first level's lines of one parity are about
// that many blocks, and four wavefronts make cheap barriers.  Every value is
// produced by the expressions of the separate kernels, so the result is theirs
// bit for bit.  LDS: the line solvers' scratch, then every level's iterate and
// right-hand side, then the coarsest solve's.
constexpr int kZebraScratch = kZebraTail * kSegBS + kSegHead;
static_assert(kZebraScratch % 2 == 0 && kZebraScratch >= 5 * kZebraTail + kSegHead, "line scratch");

template <typename T>
__global__ __launch_bounds__(kZebraTail) void k_zebra_tail(ZebraTailArgs<T> S) {
    if (S.ctrl != nullptr && S.ctrl->done) return;
    extern __shared__ double tail_lds[];
    constexpr int NT = kZebraTail;
    T* const lds = reinterpret_cast<T*>(tail_lds);
    const int tid = threadIdx.x;
    {
        const ZebraTailLevel<T>& L = S.lv[0];
        const float inv = 1.0f / (float)L.P;
        for (int q = tid; q < L.n * L.P; q += NT) {
            const int j = seg_div(q, inv), i = q - j * L.P;
            lds[L.ou + q] = T(0);
            lds[L.of + q] = i < L.m ? S.b[(size_t)j * S.P + i] : T(0);
        }
    }
    __syncthreads();
    // x += P(e) on the interior of level l
    const auto correct = [&](int l) {
        const ZebraTailLevel<T>&F = S.lv[l], &C = S.lv[l + 1];
        const float inv = 1.0f / (float)(F.m - 2);
        for (int q = tid; q < (F.m - 2) * (F.n - 2); q += NT) {
            const int jj = seg_div(q, inv);
            const int j = jj + 1, i = q - jj * (F.m - 2) + 1;
            const T* e = lds + C.ou + (j >> 1) * C.P + (i >> 1);
            const T lo0 = e[0], lo1 = e[i & 1], hi0 = e[(j & 1) * C.P], hi1 = e[(j & 1) * C.P + (i & 1)];
            T p;
            if (j & 1)
                p = (i & 1) ? ((lo0 + lo1) + (hi0 + hi1)) * T(0.25) : (lo0 + hi0) * T(0.5);
            else
                p = (i & 1) ? (lo0 + lo1) * T(0.5) : lo0;
            T* x = lds + F.ou + j * F.P + i;
            *x = *x + p;
        }
        __syncthreads();
    };
    int l = 0;
    bool up = false;
    for (;;) {
        const ZebraTailLevel<T>& L = S.lv[l];
        LineArgsT<T> A{};
        A.u = lds + L.ou;
        A.f = lds + L.of;
        A.m = L.m;
        A.n = L.n;
        A.P = L.P;
        A.cx = L.cx;
        A.cy = L.cy;
        A.d = L.d;
        A.omega = S.omega;
        const int halves = 4 * (up ? S.nu2 : S.nu1);
#pragma unroll 1
        for (int h = 0; h < halves; ++h) {
            A.parity = 1 - (h & 1);
            const int first = A.parity ? 1 : 2;
            if ((h & 2) == 0) {
                A.seg = L.seg[0];
                const int W = seg_lines_of(0, L.m - 2, NT);
                for (int t = 0; first + 2 * t * W <= L.n - 2; ++t) {
                    adi_rows_seg<T, NT>(A, nullptr, t, lds);
                    __syncthreads();
                }
            } else {
                A.seg = L.seg[1];
                const int W = seg_lines_of(1, L.n - 2, NT);
                for (int t = 0; first + 2 * t * W <= L.m - 2; ++t) {
                    adi_cols_seg<T, NT>(A, nullptr, t, lds);
                    __syncthreads();
                }
            }
        }
        if (up) {
            if (l == 0) break;
            --l;
            correct(l);
            continue;
        }
        // residual and its full weighting: the coarse right-hand side, and a zero start
        const ZebraTailLevel<T>& C = S.lv[l + 1];
        const T cx = (T)L.cx, cy = (T)L.cy, d = (T)L.d;
        const float inv = 1.0f / (float)C.P;
        for (int q = tid; q < C.n * C.P; q += NT) {
            const int J = seg_div(q, inv), I = q - J * C.P;
            T v = 0;
            if (I >= 1 && I <= C.m - 2 && J >= 1 && J <= C.n - 2) {
                const T* x = lds + L.ou + 2 * J * L.P + 2 * I;
                const T* f = lds + L.of + 2 * J * L.P + 2 * I;
                const auto res = [&](int a, int b) -> T {
                    const T* c = x + b * L.P + a;
                    return f[b * L.P + a] - fma(-d, c[0], fma(cy, c[-L.P] + c[L.P], cx * (c[-1] + c[1])));
                };
                v = (fma(T(4), res(0, 0), T(2) * ((res(-1, 0) + res(1, 0)) + (res(0, -1) + res(0, 1)))) +
                     ((res(-1, -1) + res(1, -1)) + (res(-1, 1) + res(1, 1)))) * T(0.0625);
            }
            lds[C.of + q] = v;
            lds[C.ou + q] = T(0);
        }
        __syncthreads();
        ++l;
        if (l == S.nlev - 1) {
            CoarseArgs<T> B{};
            B.b = lds + C.of;
            B.out = lds + C.ou;
            B.minv = S.minv;
            B.work = S.work;
            B.bw = S.bw;
            B.ifast = S.ifast;
            B.m = C.m;
            B.n = C.n;
            B.P = C.P;
            B.cx = C.cx;
            B.cy = C.cy;
            coarse_block<T>(B, tail_lds + S.rhs);
            __syncthreads();
            up = true;
            --l;
            correct(l);
        }
    }
    const ZebraTailLevel<T>& L = S.lv[0];
    const float inv = 1.0f / (float)L.m;
    for (int q = tid; q < L.n * L.m; q += NT) {
        const int j = seg_div(q, inv), i = q - j * L.m;
        S.out[(size_t)j * S.P + i] = lds[L.ou + j * L.P + i];
    }
}

template <typename T>
hipError_t launch_zebra_tail(const ZebraTailArgs<T>& a, hipStream_t s) {
    if (a.nlev < 2 || a.nlev > kMaxSub) return hipErrorInvalidValue;
    for (int k = 0; k + 1 < a.nlev; ++k)
        if (!seg_fits(0, a.lv[k].m - 2) || !seg_fits(1, a.lv[k].n - 2) ||
            seg_lines_of(0, a.lv[k].m - 2, kZebraTail) < 1 || seg_lines_of(1, a.lv[k].n - 2, kZebraTail) < 1)
            return hipErrorInvalidValue;
    k_zebra_tail<T><<<1, kZebraTail, a.lds_bytes, s>>>(a);
    return hipGetLastError();
}
template hipError_t launch_zebra_tail<double>(const ZebraTailArgs<double>&, hipStream_t);
template hipError_t launch_zebra_tail<float>(const ZebraTailArgs<float>&, hipStream_t);

hipError_t zebra_tail_set_lds_limit(int bytes) {
    const hipError_t e =
        hipFuncSetAttribute((const void*)k_zebra_tail<double>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    return e != hipSuccess ? e
                           : hipFuncSetAttribute((const void*)k_zebra_tail<float>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <typename T>
static void launch_batch_seg(int kind, int code, const BatchItem* items, const int* tmap, int total, int blocks,
                             hipStream_t s) {
    if (kind == BK_ADI_ROWS) {
        switch (code) {
            case 0: k_batch_adi_rows_seg<T, 64><<<blocks, 64, 0, s>>>(items, tmap, total); return;
            case 1: k_batch_adi_rows_seg<T, 128><<<blocks, 128, 0, s>>>(items, tmap, total); return;
            default: k_batch_adi_rows_seg<T, 256><<<blocks, 256, 0, s>>>(items, tmap, total); return;
        }
    }
    switch (code) {
        case 0: k_batch_adi_cols_seg<T, 64><<<blocks, 64, 0, s>>>(items, tmap, total); return;
        case 1: k_batch_adi_cols_seg<T, 256><<<blocks, 256, 0, s>>>(items, tmap, total); return;
        case 2: k_batch_adi_cols_seg<T, 512><<<blocks, 512, 0, s>>>(items, tmap, total); return;
        default: k_batch_adi_cols_seg<T, 1024><<<blocks, 1024, 0, s>>>(items, tmap, total); return;
    }
}

hipError_t launch_batch_adi(int kind, int flags, int dt, const BatchItem* items, const int* tmap, int total,
                            int blocks, hipStream_t s) {
    if (total <= 0) return hipSuccess;
    if (flags & ADI_SEG) {
        blocks = xcd_pad(blocks);
        const int code = (flags >> ADI_CODE_SHIFT) & 3;
        if (dt == 0)
            launch_batch_seg<double>(kind, code, items, tmap, total, blocks, s);
        else
            launch_batch_seg<float>(kind, code, items, tmap, total, blocks, s);
        return hipGetLastError();
    }
    if (dt != 0) return hipErrorInvalidValue;   // the sequential solver is FP64 only
    if (kind == BK_ADI_ROWS)
        k_batch_adi_rows<<<blocks, kRowTile, 0, s>>>(items, tmap, total);
    else
        k_batch_adi_cols<<<blocks, kBlock, 0, s>>>(items, tmap, total);
    return hipGetLastError();
}

}  // namespace lap
