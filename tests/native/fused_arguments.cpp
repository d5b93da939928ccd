// Calls the fused passes' launcher with each array missing in turn; prints
// the cases it lets through.  Every call must be refused before a launch.
#include <cstdio>

#include "lap_kernels.hpp"

using namespace lap;

template <typename T>
static int refused(const char* name, int flags, void (*drop)(SweepArgs<T>&)) {
    SweepArgs<T> a{};
    T* const some = reinterpret_cast<T*>(4096);   // never read: the launch is refused
    double* const some64 = reinterpret_cast<double*>(4096);
    a.uin = a.f = a.ec = some;
    a.uout = a.bc = a.rhs_out = some;
    a.partials = some64;
    a.psi_in = some64;
    a.psi_out = some64;
    a.m = a.n = 65;
    a.P = 128;
    a.mc = a.nc = 33;
    a.Pc = 64;
    a.tl = make_tiling(65, 65, 2, 16, 0, 10);
    drop(a);
    const hipError_t e = launch_fused<T>(a, flags, nullptr);
    if (e != hipErrorInvalidValue) std::printf("%s: %d\n", name, (int)e);
    return e != hipErrorInvalidValue;
}

int main() {
    using D = SweepArgs<double>;
    using F = SweepArgs<float>;
    int bad = 0;
    bad += refused<double>("input", SW_TWO, [](D& a) { a.uin = nullptr; });
    bad += refused<double>("input of a correction", SW_TWO | SW_PROLONG | SW_F, [](D& a) { a.uin = nullptr; });
    bad += refused<double>("input of four sweeps", SW_FOUR, [](D& a) { a.uin = nullptr; });
    bad += refused<double>("input of a probe", SW_PROBE | SW_RESTRICT | SW_TWO | SW_NORM, [](D& a) { a.uin = nullptr; });
    bad += refused<double>("output", SW_TWO | SW_F, [](D& a) { a.uout = nullptr; });
    bad += refused<double>("source", SW_TWO | SW_F, [](D& a) { a.f = nullptr; });
    bad += refused<double>("correction", SW_TWO | SW_PROLONG, [](D& a) { a.ec = nullptr; });
    bad += refused<double>("coarse right-hand side", SW_RESTRICT | SW_TWO, [](D& a) { a.bc = nullptr; });
    bad += refused<double>("partials", SW_TWO | SW_NORM, [](D& a) { a.partials = nullptr; });
    const int def = SW_DEF | SW_PROLONG | SW_TWO | SW_F;
    bad += refused<float>("float input", SW_RESTRICT | SW_F, [](F& a) { a.uin = nullptr; });
    bad += refused<float>("iterate", def, [](F& a) { a.psi_in = nullptr; });
    bad += refused<float>("update", def, [](F& a) { a.psi_out = nullptr; });
    bad += refused<float>("new right-hand side", def, [](F& a) { a.rhs_out = nullptr; });
    bad += refused<float>("defect partials", def, [](F& a) { a.partials = nullptr; });
    return bad;
}
