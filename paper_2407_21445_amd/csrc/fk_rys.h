// Rys quadrature roots and weights from the generated piecewise-polynomial
// tables (see gen_rys_table.py for how the tables are made).
//
// The n-point rule reproduces the Boys-function moments
// sum_r w_r u_r^k = F_k(T), k < 2n, of the paper's auxiliary integrals
// (eq. boys-fn-def), which is what lets a product of three 1-D factors per root
// stand in for the m-indexed auxiliary integrals of the vertical recurrences.
#pragma once

#include <math.h>

#include <vector>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define FK_HD __host__ __device__ __forceinline__
#else
#define FK_HD inline
#endif

#include "rys_table.inc"

namespace fk {

// offset of the n-point rule in the half-range Gauss-Hermite arrays
constexpr int gh_offset(int n) { return n * (n - 1) / 2; }

struct GHConst {
    double y2[28], w[28];
};

// 1/sqrt(x) for x > 0: on the host the library functions; on the device the
// hardware estimate y (some 25 bits) and one step of third order: with
// e = 1 - x y^2, 1/sqrt(x) = y (1 - e)^(-1/2) = y (1 + e/2 + 3 e^2/8 + O(e^3)),
// five operations and a chain of four where two Newton steps take seven or
// eight and a chain of six.  What is left out is below 2^-70; the result is
// within one unit in the last place, as after two Newton steps.
FK_HD double rys_rsqrt(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
#else
    return 1.0 / sqrt(x);
#endif
}

// Doubles between consecutive intervals of the n-point segment as staged for
// the kernels: the (RYS_DEG + 1) 2n coefficients padded to 2 mod 16, so that
// lanes reading the same coefficient of different intervals start 16 bytes
// apart modulo 128 bytes and spread over the LDS banks (a multiple of 8 or 16
// doubles would put every interval on the same few banks).
constexpr int rys_stride(int n)
{
    const int d = (RYS_DEG + 1) * 2 * n;
    return d + ((2 - d % 16) + 16) % 16;
}

// T from which the n-point rule is the half-range Gauss-Hermite rule: the
// asymptotic moments Gamma(k+1/2)/(2 T^(k+1/2)) it reproduces differ from
// F_k(T), k < 2n, by e^-T T^(k-1/2)/Gamma(k+1/2) relative, below 3e-15 from
// here on (checked by the generator against 80-digit Boys values).
constexpr double rys_tswitch(int n)
{
    return n == 1 ? RYS_TSWITCH_1 : n == 2 ? RYS_TSWITCH_2 : n == 3 ? RYS_TSWITCH_3 : n == 4 ? RYS_TSWITCH_4
         : n == 5 ? RYS_TSWITCH_5 : n == 6 ? RYS_TSWITCH_6 : RYS_TSWITCH_7;
}

// Intervals of the n-point table: a uniform grid up to the switch for small n,
// the four-region grid up to RYS_TMAX for the others.
constexpr int rys_nint(int n) { return rys_table_nint[n]; }
static_assert(rys_table_nint[1] == (int)(RYS_TSWITCH_1 * RYS_UNI_INVH) &&
              rys_table_nint[RYS_UNI_NMAX] == (int)(RYS_TSWITCH_4 * RYS_UNI_INVH) &&
              rys_table_nint[RYS_UNI_NMAX + 1] == RYS_NINT, "table layout");

// The values of one interval's coefficients as the kernels use them: read before
// the first is used.  The compiler otherwise reads two, waits for them, uses them
// and reads the next two, one LDS latency after the other down the recurrence.
// rys_read2 reads a root's u and w, which lie side by side, in one go (C20H42
// 6.63 -> 6.53 ms, exchange of 21 waters 19.9 -> 19.45 against one after the
// other).
template <int M>
FK_HD void rys_read(const double *__restrict c, int step, double *__restrict v)
{
#pragma unroll
    for (int k = 0; k < M; ++k) v[k] = c[k * step];
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(M == 10, "operands of the statement below");
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]),
                      "+v"(v[8]), "+v"(v[9]));
#endif
}

template <int M>
FK_HD void rys_read2(const double *__restrict c, int step, double *__restrict u, double *__restrict w)
{
#pragma unroll
    for (int k = 0; k < M; ++k) {
        u[k] = c[k * step];
        w[k] = c[k * step + 1];
    }
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(M == 10, "operands of the statement below");
    asm volatile("" : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]), "+v"(u[4]), "+v"(u[5]), "+v"(u[6]), "+v"(u[7]),
                      "+v"(u[8]), "+v"(u[9]), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]),
                      "+v"(w[6]), "+v"(w[7]), "+v"(w[8]), "+v"(w[9]));
#endif
}

// Evaluate the n-point rule at T.  `tab` points at the n-point segment of the
// table ([interval][coefficient][function], intervals rys_stride(n) apart);
// gy2/gw at the n-point Gauss-Hermite data (y_i^2 and h_i) for the region
// tables (the uniform-grid case takes them as constants).  NEED_U = false
// evaluates the weights only (enough when L = 0).
//
// Uniform grid (small n), BRANCHLESS: both rules are evaluated -- a lane
// beyond the switch reads the last interval, which every such lane shares (one
// LDS broadcast) -- and the lane's rule selected, so that the code of a primitive
// quartet is one basic block the compiler can interleave with the next one's
// (at the cost of both results being live at once).  Otherwise the two rules
// are separate branches, so a wave whose lanes all lie beyond the switch
// skips the table and only lanes below it read the LDS.
template <int N, bool NEED_U, bool BRANCHLESS = false>
FK_HD void rys_roots_from(double T, const double *__restrict tab, const double *__restrict gy2,
                          const double *__restrict gw, double *u, double *w)
{
    constexpr int NF = 2 * N;
    static_assert(rys_tswitch(N) <= RYS_TMAX, "the table must cover T below the switch");
    static_assert(RYS_NREG == 4 && RYS_REG1_T0 == 16.0 && RYS_REG1_INVH == 1.0 && RYS_REG3_BASE == 56,
                  "closed-form region selection assumes the generated four-region layout");
    if constexpr (N <= RYS_UNI_NMAX && BRANCHLESS) {
        // every lane beyond the switch reads the end of the last interval
        const bool in_tab = T < rys_tswitch(N);
        constexpr double ylast = rys_table_nint[N] * (1.0 - 0x1p-53);
        const double y = fmin(T * RYS_UNI_INVH, ylast);
        const int iv = (int)y;
        const double x = fma(2.0, y - (double)iv, -1.0);
        const double *c = tab + iv * rys_stride(N);
        const double sT = rys_rsqrt(T);  // not used below the switch, where it may be anything (T = 0)
        const double rT = sT * sT;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double cw[RYS_DEG + 1], cu[RYS_DEG + 1];
            if constexpr (NEED_U) rys_read2<RYS_DEG + 1>(c + 2 * i, NF, cu, cw);
            else rys_read<RYS_DEG + 1>(c + 2 * i + 1, NF, cw);
            double vw = cw[RYS_DEG];
#pragma unroll
            for (int k = RYS_DEG - 1; k >= 0; --k) vw = vw * x + cw[k];
            w[i] = in_tab ? vw : rys_gh_w[gh_offset(N) + i] * sT;
            if constexpr (NEED_U) {
                double vu = cu[RYS_DEG];
#pragma unroll
                for (int k = RYS_DEG - 1; k >= 0; --k) vu = vu * x + cu[k];
                u[i] = in_tab ? vu : rys_gh_y2[gh_offset(N) + i] * rT;
            }
        }
    } else if (T < rys_tswitch(N)) {
        int iv;
        double x;
        if constexpr (N <= RYS_UNI_NMAX) {
            const double y = T * RYS_UNI_INVH;
            iv = (int)y;
            x = fma(2.0, y - (double)iv, -1.0);
        } else {
            // region k = floor(T/16) (k <= 3) has interval width 2^(k-1) and
            // starts at interval 64 - 2^(6-k)
            int k = (int)(T * (1.0 / 16.0));
            k = k < 3 ? k : 3;
            const double ih = (double)(2 >> k) + (k == 3 ? 0.25 : 0.0) + (k == 2 ? 0.5 : 0.0);
            const double y = (T - 16.0 * k) * ih;
            const int j = (int)y;
            iv = 64 - (64 >> k) + j;
            x = 2.0 * (y - j) - 1.0;
        }
        const double *c = tab + iv * rys_stride(N);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double cw[RYS_DEG + 1], cu[RYS_DEG + 1];
            if constexpr (NEED_U) rys_read2<RYS_DEG + 1>(c + 2 * i, NF, cu, cw);
            else rys_read<RYS_DEG + 1>(c + 2 * i + 1, NF, cw);
            double vw = cw[RYS_DEG];
#pragma unroll
            for (int k = RYS_DEG - 1; k >= 0; --k) vw = vw * x + cw[k];
            w[i] = vw;
            if constexpr (NEED_U) {
                double vu = cu[RYS_DEG];
#pragma unroll
                for (int k = RYS_DEG - 1; k >= 0; --k) vu = vu * x + cu[k];
                u[i] = vu;
            }
        }
    } else {
        const double sT = rys_rsqrt(T);
        const double rT = sT * sT;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (NEED_U) u[i] = rys_gh_y2[gh_offset(N) + i] * rT;
            w[i] = rys_gh_w[gh_offset(N) + i] * sT;
        }
    }
}

}  // namespace fk

// Size of one staged n-point table segment and of the segment plus its
// Gauss-Hermite data (y_i^2 then h_i), which is how kernels stage it in LDS.
constexpr int rys_seg_size(int n) { return fk::rys_nint(n) * fk::rys_stride(n); }
constexpr int rys_lds_size(int n) { return rys_seg_size(n) + 2 * n; }

// `tab` holds rys_lds_size(N) doubles: the segment followed by y_i^2 and h_i.
template <int N, bool NEED_U, bool BRANCHLESS = false>
FK_HD void rys_roots(double T, const double *__restrict tab, double *u, double *w)
{
    fk::rys_roots_from<N, NEED_U, BRANCHLESS>(T, tab, tab + rys_seg_size(N), tab + rys_seg_size(N) + N, u, w);
}

// One root at a time, for the classes whose root loop is not unrolled: rys_at
// finds the interval (or the asymptotic factors) of T once, rys_root_at
// evaluates root r of it.  `tab` as for rys_roots.
template <int N>
struct RysAt {
    const double *c, *gh;  // the interval's coefficients; y_i^2, then h_i
    double x, sT, rT;
    bool in_tab, any_tab;  // this lane below the switch; any lane of the wave
};
template <int N>
FK_HD RysAt<N> rys_at(double T, const double *__restrict tab)
{
    RysAt<N> a;
    a.in_tab = T < fk::rys_tswitch(N);
#if defined(__HIP_DEVICE_COMPILE__)
    a.any_tab = __ballot(a.in_tab) != 0ull;
#else
    a.any_tab = a.in_tab;
#endif
    const double Tc = a.in_tab ? T : 0.0;
    int iv;
    if constexpr (N <= RYS_UNI_NMAX) {
        const double y = Tc * RYS_UNI_INVH;
        iv = (int)y;
        a.x = fma(2.0, y - (double)iv, -1.0);
    } else {
        int k = (int)(Tc * (1.0 / 16.0));
        k = k < 3 ? k : 3;
        const double ih = (double)(2 >> k) + (k == 3 ? 0.25 : 0.0) + (k == 2 ? 0.5 : 0.0);
        const double y = (Tc - 16.0 * k) * ih;
        const int j = (int)y;
        iv = 64 - (64 >> k) + j;
        a.x = 2.0 * (y - j) - 1.0;
    }
    a.c = tab + iv * fk::rys_stride(N);
    a.gh = tab + rys_seg_size(N);
    a.sT = fk::rys_rsqrt(a.in_tab ? 1.0 : T);
    a.rT = a.sT * a.sT;
    return a;
}
template <int N>
FK_HD void rys_root_at(const RysAt<N> &a, int r, double &u, double &w)
{
    constexpr int NF = 2 * N;
    u = a.gh[r] * a.rT;
    w = a.gh[N + r] * a.sT;
    if (a.any_tab) {
        const double *c = a.c + 2 * r;
        double cu[RYS_DEG + 1], cw[RYS_DEG + 1];
        fk::rys_read2<RYS_DEG + 1>(c, NF, cu, cw);
        double vu = cu[RYS_DEG], vw = cw[RYS_DEG];
#pragma unroll
        for (int k = RYS_DEG - 1; k >= 0; --k) {
            vu = vu * a.x + cu[k];
            vw = vw * a.x + cw[k];
        }
        u = a.in_tab ? vu : u;
        w = a.in_tab ? vw : w;
    }
}

constexpr int rys_staged_offset(int n)
{
    int o = 0;
    for (int m = 1; m < n; ++m) o += rys_lds_size(m);
    return o;
}
constexpr int rys_staged_total() { return rys_staged_offset(RYS_NMAX + 1); }

// Host copy of every n-point segment followed by its Gauss-Hermite data, the
// layout uploaded to the device and staged into LDS by the kernels.
inline const double *rys_staged_host()
{
    static const std::vector<double> v = [] {
        std::vector<double> t;
        t.reserve(rys_staged_total());
        for (int n = 1; n <= RYS_NMAX; ++n) {
            const int d = (RYS_DEG + 1) * 2 * n;
            for (int iv = 0; iv < fk::rys_nint(n); ++iv) {
                const double *src = rys_table_data + rys_table_offset[n - 1] + (size_t)iv * d;
                t.insert(t.end(), src, src + d);
                t.insert(t.end(), fk::rys_stride(n) - d, 0.0);
            }
            for (int i = 0; i < n; ++i) t.push_back(rys_gh_y2[fk::gh_offset(n) + i]);
            for (int i = 0; i < n; ++i) t.push_back(rys_gh_w[fk::gh_offset(n) + i]);
        }
        return t;
    }();
    return v.data();
}
