// Device building blocks shared by the forward and adjoint kernels: the
// Rosenbrock tableau, wave helpers, the per-cell LDS layout, thermodynamics,
// reaction rates with their analytical derivatives, the right-hand side and
// Jacobian passes (both families'), the dense LU and solves, one Rosenbrock
// attempt and the step-size controller.
//
// Work decomposition: one 64-lane wavefront integrates one cell (one
// independent homogeneous reactor, paper Sec. 1).  Inside the wave
//   - state, stage and error vectors are lane-distributed: lane i holds
//     component i of (Y_0..Y_{N-1}, T), so vector algebra is one VALU op;
//   - thermodynamics runs with lanes over species, rates and their analytical
//     derivatives with lanes over reactions (Sec. 2.5: sparse analytical
//     Jacobian), scattering into LDS with LDS floating-point atomics;
//   - the iteration matrix I/(h gamma) - J is formed in VGPRs, row i in lane
//     i, and factorised without pivoting in a fixed order, in blocks of 16
//     pivots whose rows are broadcast inside the multiply-adds; the factors
//     leave for LDS block by block (column-major, an odd stride) for the
//     triangular solves;
//   - the Rosenbrock stepper and its error/step-size controller run uniformly
//     per wave (no divergence: every lane follows its cell's control flow).
// Everything is FP64.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "devmech.hpp"

namespace scdev {


// ---------------------------------------------------------------------------
// Rosenbrock tableau (transformed form; derivation in tableau.py, ros4()):
// 4 stages, order 4, L-stable, embedded order 3; stage 4 is evaluated at the
// stage-3 point, so a step costs 3 function evaluations (one of them in the
// Jacobian pass), 1 factorisation and 4 solves.
// ---------------------------------------------------------------------------
constexpr int NS = 4;
constexpr double GAM = 0.572816062482135;
static __constant__ double TA[NS][NS] = {{0.0, 0.0, 0.0, 0.0},
                                  {1.0474566606950075, 0.0, 0.0, 0.0},
                                  {1.5266834054578882, 0.49110997987229194, 0.0, 0.0},
                                  {1.5266834054578882, 0.49110997987229194, 0.0, 0.0}};
static __constant__ double TC[NS][NS] = {{0.0, 0.0, 0.0, 0.0},
                                  {-2.8287104387961546, 0.0, 0.0, 0.0},
                                  {-1.1423273772481277, 0.9544101947030211, 0.0, 0.0},
                                  {-3.972521690537523, -0.6901523982223108, -1.548869644699513, 0.0}};
static __constant__ double TM[NS] = {2.326763557172835, -0.7953731300411474, 1.6632540048577067, 1.0474566606950075};
static __constant__ double TE[NS] = {0.4092508278871161, -1.0795845833425672, 0.9649495643943683,
                              1.0474566606950078};  // m - mhat
// function value of a stage: 0 = f(y) from the Jacobian pass, -1 = evaluate,
// k > 0 = reuse the value evaluated at stage k (same point)
static __constant__ int TREUSE[NS] = {0, -1, -1, 2};
// step-size exponent 1/(embedded order + 1) = 1/4 (ctl_end takes the fourth root)

constexpr int WAVE = 64;
// LDS loads issued ahead per group in the unrolled row/solve loops; bounds
// the scheduler's hoisting (register pressure) while keeping latency hidden
constexpr int LD_GROUP = 8;
#define SC_FENCE_EVERY(i) \
    if (((i) + 1) % LD_GROUP == 0) __builtin_amdgcn_sched_barrier(0)

// ---------------------------------------------------------------------------
// wave helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ double rdlane(double v, int lane)
{
    int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// One step of a butterfly sum in registers: v plus the value a DPP control
// brings from the same row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}

// Sum over aligned groups of G lanes (16, 32 or 64), left in every lane of
// the group: a butterfly over lane distances G/2, ..., 1, so the additions
// and their order are those of xor shuffles.  The distances 32 and 16 are
// half-wave and row swaps (a swap of v with itself leaves the low half in one
// result and the high half in the other), 8 and 4 are rotations of a row
// (after the step at distance 8 the row repeats with period 8, so a rotation
// by 4 reads the lane at distance 4), 2 and 1 permute quads.  A shuffle is an
// LDS permute whose round trip the next step waits for; a 64-lane sum took
// about 900 cycles of the wave's chain with shuffles, 13 sums a step.
template <int G>
__device__ __forceinline__ double group_sum(double v)
{
    static_assert(G == 16 || G == 32 || G == 64, "aligned group of lanes");
    if constexpr (G == 64) {
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    if constexpr (G >= 32) {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    v = add_dpp<0x128>(v);  // row_ror:8
    v = add_dpp<0x124>(v);  // row_ror:4
    v = add_dpp<0x4e>(v);   // quad_perm [2,3,0,1]
    return add_dpp<0xb1>(v);  // quad_perm [1,0,3,2]
}

__device__ __forceinline__ double wave_sum(double v) { return group_sum<WAVE>(v); }

// v from lane K of each cell's group, K known at compile time: a row
// broadcast of the DPP unit for 16 lanes; for 32, readlane of both groups and
// a select.
template <int G, int K>
__device__ __forceinline__ double bcast(double v)
{
    static_assert(G == 16 || G == 32, "groups of several cells per wave");
    if constexpr (G == 16) {
        const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + K, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + K, 0xf, 0xf, true);
        return __hiloint2double(hi, lo);
    } else {
        const double a = rdlane(v, K), b = rdlane(v, 32 + K);
        return threadIdx.x & 32 ? b : a;
    }
}

// z -= a z_K, z_K from lane K of the row of 16 lanes: one instruction (the
// broadcast reads a register two wait states after it was written)
template <int K>
__device__ __forceinline__ void fmac_row(double &z, double a)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %0, -%1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+&v"(z) : "v"(a), "n"(K));
}
// the same for four vectors
template <int K>
__device__ __forceinline__ void fmac_row4(double &x, double &y, double &z, double &w, double a)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %0, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %1, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %2, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %3, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+&v"(x), "+&v"(y), "+&v"(z), "+&v"(w)
        : "v"(a), "n"(K));
}
// z -= a z_K on the lanes of the rows in ROWS
template <int K, int ROWS>
__device__ __forceinline__ void fmac_in(double &z, double a)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %0, -%1 row_newbcast:%2 row_mask:%3 bank_mask:0xf"
        : "+&v"(z)
        : "v"(a), "n"(K), "n"(ROWS));
}
// z -= a x_K, x_K from lane K of the row
template <int K>
__device__ __forceinline__ void fmac_from(double &z, double x, double a)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
        : "+&v"(z)
        : "v"(x), "v"(a), "n"(K));
}
// x, y, z, w -= a times lane K of p, q, r, s
template <int K>
__device__ __forceinline__ void fmac_from4(double &x, double &y, double &z, double &w, double p, double q, double r,
                                           double s, double a)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, -%8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %5, -%8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %6, -%8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %7, -%8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(x), "+&v"(y), "+&v"(z), "+&v"(w)
        : "v"(p), "v"(q), "v"(r), "v"(s), "v"(a), "n"(K));
}
// z -= sum a[i] x_{K + i}, i = 0..3, on the lanes of the rows in ROWS
template <int K, int ROWS>
__device__ __forceinline__ void fmac_by4(double &z, double x, const double *a)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, -%2 row_newbcast:%6 row_mask:%10 bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, -%3 row_newbcast:%7 row_mask:%10 bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, -%4 row_newbcast:%8 row_mask:%10 bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, -%5 row_newbcast:%9 row_mask:%10 bank_mask:0xf"
        : "+&v"(z)
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(K), "n"(K + 1), "n"(K + 2), "n"(K + 3), "n"(ROWS));
}
// the lanes of row B of 16 in every row
template <int B>
__device__ __forceinline__ double spread_row(double v)
{
    auto half = [](int x) __attribute__((always_inline)) {
        const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        const int y = B & 1 ? a[1] : a[0];
        const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
        return (int)(B & 2 ? b[1] : b[0]);
    };
    return __hiloint2double(half(__double2hiint(v)), half(__double2loint(v)));
}

// f(0), ..., f(N - 1) with compile-time arguments
template <int N, class F, int... I>
__device__ __forceinline__ void unrolled_(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F &&f)
{
    unrolled_<N>(f, std::make_integer_sequence<int, N>{});
}


__device__ __forceinline__ void wave_sync() { __syncthreads(); }

// Order between the LDS accesses of the wave's lanes.  A wave's LDS
// instructions take effect in order: the compiler must not move them across,
// but nothing has to be waited for (a workgroup barrier's fence also waits for
// the loads sent ahead).  Between the waves of a workgroup it orders only this:
// what a wave wrote or added before a store is there for whoever reads that
// store's value, since the LDS takes the instructions of one wave one after the
// other (a crew's turn counter is handed on so); everything else goes through
// barriers.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Who works on a cell: here the one wave; the sparse kernels also know crews.
struct Solo {
    static constexpr int w = 1, rank = 0;
    __device__ __forceinline__ void sync() const { lds_sync(); }
    __device__ __forceinline__ void barrier() const {}
    __device__ __forceinline__ void start(const DevRx &) const {}
    __device__ __forceinline__ int first(const DevRx &sp) const { return sp.passes - 1; }
    __device__ __forceinline__ int next(const DevRx &, int q) const { return q - 1; }
    __device__ __forceinline__ void await(int) const {}
    __device__ __forceinline__ void pass_on(int) const {}
};


// ---------------------------------------------------------------------------
// Dual numbers (value, directional derivative): the chemistry below is
// written once for a scalar type S; S = double is the integrator, S = Dual
// carries an exact directional derivative through the same arithmetic (used
// by the adjoint for the derivative of the Jacobian along a direction).
// ---------------------------------------------------------------------------
// (the double overloads stay visible next to the Dual ones below)
using ::exp;
using ::log;
using ::log10;

struct Dual {
    double v, d;
    Dual() = default;
    __host__ __device__ constexpr Dual(double x) : v(x), d(0.0) {}
    __host__ __device__ constexpr Dual(double x, double t) : v(x), d(t) {}
};
__device__ __forceinline__ Dual operator+(Dual a, Dual b) { return {a.v + b.v, a.d + b.d}; }
__device__ __forceinline__ Dual operator-(Dual a, Dual b) { return {a.v - b.v, a.d - b.d}; }
__device__ __forceinline__ Dual operator-(Dual a) { return {-a.v, -a.d}; }
__device__ __forceinline__ Dual operator*(Dual a, Dual b) { return {a.v * b.v, fma(a.d, b.v, a.v * b.d)}; }
__device__ __forceinline__ Dual operator/(Dual a, Dual b)
{
    const double q = a.v / b.v;
    return {q, (a.d - q * b.d) / b.v};
}
__device__ __forceinline__ Dual operator+(Dual a, double b) { return {a.v + b, a.d}; }
__device__ __forceinline__ Dual operator+(double a, Dual b) { return {a + b.v, b.d}; }
__device__ __forceinline__ Dual operator-(Dual a, double b) { return {a.v - b, a.d}; }
__device__ __forceinline__ Dual operator-(double a, Dual b) { return {a - b.v, -b.d}; }
__device__ __forceinline__ Dual operator*(Dual a, double b) { return {a.v * b, a.d * b}; }
__device__ __forceinline__ Dual operator*(double a, Dual b) { return {a * b.v, a * b.d}; }
__device__ __forceinline__ Dual operator/(Dual a, double b) { return {a.v / b, a.d / b}; }
__device__ __forceinline__ Dual operator/(double a, Dual b)
{
    const double q = a / b.v;
    return {q, -q * b.d / b.v};
}
__device__ __forceinline__ Dual &operator+=(Dual &a, Dual b) { return a = a + b; }
__device__ __forceinline__ Dual &operator-=(Dual &a, Dual b) { return a = a - b; }
__device__ __forceinline__ Dual &operator*=(Dual &a, Dual b) { return a = a * b; }
__device__ __forceinline__ Dual exp(Dual a)
{
    const double e = exp(a.v);
    return {e, e * a.d};
}
__device__ __forceinline__ Dual log(Dual a) { return {log(a.v), a.d / a.v}; }
__device__ __forceinline__ Dual log10(Dual a) { return {log10(a.v), a.d / (a.v * 2.302585092994046)}; }
__device__ __forceinline__ Dual rdlane(Dual v, int lane) { return {rdlane(v.v, lane), rdlane(v.d, lane)}; }
__device__ __forceinline__ Dual wave_sum(Dual v) { return {wave_sum(v.v), wave_sum(v.d)}; }

// the part a pass reports: the value (S = double) or the derivative (Dual)
__device__ __forceinline__ double part(double x) { return x; }
__device__ __forceinline__ double part(Dual x) { return x.d; }
__device__ __forceinline__ double value(double x) { return x; }
__device__ __forceinline__ double value(Dual x) { return x.v; }

// LDS access of a scalar: a Dual's derivative lives toff doubles from its value
template <class S>
__device__ __forceinline__ S lds_get(const double *lds, int i, int toff);
template <>
__device__ __forceinline__ double lds_get<double>(const double *lds, int i, int)
{
    return lds[i];
}
template <>
__device__ __forceinline__ Dual lds_get<Dual>(const double *lds, int i, int toff)
{
    return {lds[i], lds[i + toff]};
}
__device__ __forceinline__ void lds_put(double *lds, int i, double x, int) { lds[i] = x; }
__device__ __forceinline__ void lds_put(double *lds, int i, Dual x, int toff)
{
    lds[i] = x.v;
    lds[i + toff] = x.d;
}
__device__ __forceinline__ void lds_add(double *lds, int i, double x, int) { atomicAdd(&lds[i], x); }
__device__ __forceinline__ void lds_add(double *lds, int i, Dual x, int toff)
{
    atomicAdd(&lds[i], x.v);
    atomicAdd(&lds[i + toff], x.d);
}

// The reactor model as a compile-time constant.  Every device routine is
// inlined into its kernel, so a kernel that calls this on its DevMech
// argument gets the branches on m.cv folded away.
template <bool CV>
__device__ __forceinline__ DevMech fix_reactor(DevMech m)
{
    m.cv = CV ? 1 : 0;
    return m;
}

// ---------------------------------------------------------------------------
// LDS layout of one cell (doubles)
// ---------------------------------------------------------------------------
template <int NP>
struct Lds {
    // row stride of the Jacobian terms: lanes reading their own rows hit
    // addresses a stride apart; an odd stride spreads them over the banks
    static constexpr int PS = NP + 1;
    static constexpr int P = 0;          // NP x PS Jacobian terms, later the LU factors (stride PS)
    // the term region is also where the adjoint's dual passes keep the
    // derivatives of the pairs and of its own V vector (each at a fixed
    // offset -RX from the value), which ends 8 NP + NS WAVE doubles in
    static constexpr int NV = NP;           // places of the passes' vectors: species, then the temperature's
    static constexpr int RXV = 5 * NV;      // their pairs and Euler terms
    static constexpr int DUAL = RXV + 3 * NP + NS * WAVE;
    static constexpr int PREG = NP * PS > DUAL ? NP * PS : DUAL;
    static constexpr int RX = PREG;         // the passes' vectors
    static_assert(PREG % 2 == 0 && NV % 2 == 0, "the passes' pairs are read in one");
    static constexpr int IW = RX + RXV;  // 1/W_c (0 for c >= N)
    static constexpr int U = IW + NP;    // NS stage vectors, WAVE apart
    static constexpr int SIZE = U + NS * WAVE;
};

// Per-cell uniform quantities at the point where a right-hand side was taken.
// p is the pressure; cp the heat capacity of the reactor's energy balance
// (c_p at constant pressure, c_v at constant volume).
template <class S = double>
struct Mix {
    S T, invT, lnT;
    double p;
    S rho, Wbar, cp;
};

template <class S = double>
struct Thermo {
    S cpR, hRT, sR, dcpR;
};

// NASA-7 of species k (single temperature range)
template <class S>
__device__ __forceinline__ Thermo<S> nasa7(const DevMech &m, int k, S T, S lnT, S invT)
{
    const int N = m.N;
    const double *a = m.nasa();
    const double a0 = a[k], a1 = a[N + k], a2 = a[2 * N + k], a3 = a[3 * N + k], a4 = a[4 * N + k],
                 a5 = a[5 * N + k], a6 = a[6 * N + k];
    Thermo<S> t;
    t.cpR = a0 + T * (a1 + T * (a2 + T * (a3 + T * a4)));
    t.hRT = a0 + T * (a1 * 0.5 + T * (a2 * (1.0 / 3.0) + T * (a3 * 0.25 + T * a4 * 0.2))) + a5 * invT;
    t.sR = a0 * lnT + T * (a1 + T * (a2 * 0.5 + T * (a3 * (1.0 / 3.0) + T * a4 * 0.25))) + a6;
    t.dcpR = a1 + T * (2.0 * a2 + T * (3.0 * a3 + T * 4.0 * a4));
    return t;
}

// Mixture state from the lane-distributed y (lane k < N: Y_k, lane N: T);
// writes C, g/RT, h/RT to LDS and clears the accumulators.  With S = Dual
// the derivatives go toff doubles beyond the values.  p is the pressure, or
// in a constant-volume reactor the density.
// the point itself; yw: the lane's Y/W
template <class S>
__device__ __forceinline__ Mix<S> mixture_point(const DevMech &m, S y, double p, Thermo<S> &th, int lane, S &yw)
{
    const int N = m.N;
    Mix<S> x;
    x.T = rdlane(y, N);
    x.invT = 1.0 / x.T;
    x.lnT = log(x.T);
    x.p = p;
    yw = 0.0;
    S cpw = 0.0;
    th = Thermo<S>{0.0, 0.0, 0.0, 0.0};
    if (lane < N) {
        th = nasa7<S>(m, lane, x.T, x.lnT, x.invT);
        yw = y * m.invW()[lane];
        cpw = th.cpR * yw;
    }
    x.Wbar = 1.0 / wave_sum(yw);
    x.cp = m.Rgas * wave_sum(cpw);
    if (m.cv) {
        x.rho = p;
        x.p = value(p * m.Rgas * x.T / x.Wbar);
        x.cp = x.cp - m.Rgas / x.Wbar;
    } else {
        x.rho = p * x.Wbar * x.invT / m.Rgas;
    }
    return x;
}
// Horner evaluation of the degree-d polynomial with coefficients c[0..d] at t
__device__ __forceinline__ double poly_t(const double *c, int d, double t)
{
    double p = c[d];
#pragma unroll 1
    for (int q = d - 1; q >= 0; --q) p = fma(p, t, c[q]);
    return p;
}

// Address of species c's pair in the pair array at place `at` (SPL_CG, SPL_HW)
template <int NV>
__device__ __forceinline__ double *pair(double *lds, int at, int c)
{
    return lds + at * NV + 2 * c;
}

// One pass's record of this lane's reaction (SparseRx): three 16-byte words.
struct Rec {
    uint4 a, b, c;
    __device__ __forceinline__ double lnA() const { return __hiloint2double(a.y, a.x); }
    __device__ __forceinline__ double bT() const { return __hiloint2double(a.w, a.z); }
    __device__ __forceinline__ double EaR() const { return __hiloint2double(b.y, b.x); }
    __device__ __forceinline__ uint32_t slot(int i) const  // byte offset of a side species' pair
    {
        const uint32_t w = i < 2 ? b.z : i < 4 ? b.w : c.x;
        return i % 2 ? w >> 16 : w & 0xffff;
    }
    __device__ __forceinline__ uint32_t bits() const { return c.y; }
    __device__ __forceinline__ int nu(int i) const { return (c.y >> (2 * i)) & 3; }
    __device__ __forceinline__ int dnu() const { return (int)((c.y >> 12) & 31) - 16; }
    __device__ __forceinline__ int order(int side) const { return (c.y >> (17 + 4 * side)) & 15; }
    __device__ __forceinline__ int kind() const { return (c.y >> 25) & 3; }
    __device__ __forceinline__ uint32_t enh(int e) const { return ((c.z >> (8 * e)) & 0xff) << 4; }
    __device__ __forceinline__ int orig() const { return c.w; }
};
template <int G>
__device__ __forceinline__ Rec load_rx(const DevRx &sp, int pass, int lane)
{
    const uint4 *q = (const uint4 *)sp.rec + (size_t)pass * sc::RXW_WORDS * G + lane;
    return Rec{q[0], q[G], q[2 * G]};
}

// One reaction's rate of progress and, with JAC, its derivatives: d[0..5] with
// respect to the side species' concentrations (what an unused slot holds goes
// to the trash), dqM with respect to [M] (dq/dC of an enhanced species is dqM
// times its alpha - 1), dT at fixed C, euler (the Euler remainder, or dqM in a
// constant-volume reactor) and the reaction enthalpy / RT.  The Euler remainder
// q - sum C dq/dC is taken from the reaction's orders (C d(C^nu)/dC = nu C^nu).
// With S = Dual the derivatives of the pairs lie toff doubles from the values.
template <class S = double>
struct RxTerms {
    S q, d[6], dqM;
    double ea[sc::MAXENH];
    S dT, euler, dH;
};
template <class S>
__device__ __forceinline__ S make(double v, double d)
{
    if constexpr (std::is_same_v<S, double>)
        return v;
    else
        return S(v, d);
}
template <bool JAC, int NV, class S = double>
__device__ __forceinline__ RxTerms<S> reaction_sp(const DevMech &m, const DevRx &sp, int ideg, double *lds, const Rec &r,
                                               uint32_t flags, int j, const Mix<S> &x, double dl, const double *itb,
                                               double itt, int toff = 0)
{
    RxTerms<S> o;
    S c[6], p[6], dp[6];
    double nu[6];
    S dG = 0.0, dH = 0.0;
    // a falloff pass's other tables, loaded ahead of the work (they come from L2)
    TroeRec tr;
    if ((flags & sc::RXF_TROE) && j < sp.n_troe) tr = sp.troe[j];
    if (flags & sc::RXF_TB) {
#pragma unroll
        for (int e = 0; e < sc::MAXENH; ++e) o.ea[e] = j < sp.n_tb ? sp.eam1[4 * j + e] : 0.0;
    }
    const S lnkinf = r.lnA() + dl + r.bT() * x.lnT - r.EaR() * x.invT;
    const S kinf = exp(lnkinf);
    const char *cg = (const char *)(lds + SPL_CG * NV), *hw = (const char *)(lds + SPL_HW * NV);
    S g[6], h[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const double2 v = *(const double2 *)(cg + r.slot(i));
        double2 t = make_double2(0.0, 0.0);
        if (!std::is_same_v<S, double>) t = *(const double2 *)(cg + r.slot(i) + 8 * toff);
        c[i] = make<S>(v.x, t.x);
        g[i] = make<S>(v.y, t.y);
        if (JAC)
            h[i] = make<S>(*(const double *)(hw + r.slot(i)),
                           std::is_same_v<S, double> ? 0.0 : *(const double *)(hw + r.slot(i) + 8 * toff));
        p[i] = c[i];
        dp[i] = 1.0;
        nu[i] = 1.0;
    }
    if (flags & sc::RXF_NU) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int v = r.nu(i);
            nu[i] = v;
            const S c2 = c[i] * c[i];
            p[i] = v == 2 ? c2 : v == 3 ? c2 * c[i] : c[i];
            dp[i] = v == 2 ? 2.0 * c[i] : v == 3 ? 3.0 * c2 : S(1.0);
        }
    }
    if (itb) {
        // the lanes behind the last reaction read a block of zeros: their rate
        // constants are zero, and times 1/K_c beyond the largest double NaN
        const double *itc = itb + (size_t)min(j, m.R) * 2 * (ideg + 1);
        dG = -poly_t(itc, ideg, itt);
        if (JAC) dH = poly_t(itc + ideg + 1, ideg, itt);
    } else {
        // an unused slot of a pass with larger coefficients has nu = 0 and
        // its place's g = h = 0 in any other
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            dG += nu[3 + i] * g[3 + i] - nu[i] * g[i];
            if (JAC) dH += nu[3 + i] * h[3 + i] - nu[i] * h[i];
        }
    }
    const double dnu = r.dnu();
    const S lnKc = -dG + dnu * (m.lnp0R - x.lnT);
    const S M0 = x.p * x.invT / m.Rgas;
    S M = M0, Me = 0.0;
    if (flags & sc::RXF_TB) {
        if (j < sp.n_tb) {
#pragma unroll
            for (int e = 0; e < sc::MAXENH; ++e) Me += o.ea[e] * make<S>(*(const double *)(cg + r.enh(e)),
                                                  std::is_same_v<S, double> ? 0.0 : *(const double *)(cg + r.enh(e) + 8 * toff));
        }
        M += Me;
    }
    const int kind = r.kind();
    S kf = kinf, phi = 0.0, dlnF_T = 0.0, dlnk0 = 0.0;
    if ((flags & sc::RXF_TROE) && kind == sc::RX_TROE) {
        const S lnk0 = tr.lnA0 + dl + tr.b0 * x.lnT - tr.Ea0R * x.invT;
        const S Pr = exp(lnk0 - lnkinf) * M;
        const double a = tr.a, iT3 = tr.iT3, iT1 = tr.iT1, T2 = tr.T2;
        const S e3 = exp(-x.T * iT3), e1 = exp(-x.T * iT1), e2 = exp(-T2 * x.invT);
        const S Fc = (1.0 - a) * e3 + a * e1 + e2;
        const S L = log10(Fc);
        const S cc = -0.4 - 0.67 * L, nn = 0.75 - 1.27 * L;
        const S X = log10(Pr) + cc;
        const S D = nn - 0.14 * X;
        const S f = X / D;
        const S opf = 1.0 + f * f;
        const S lF = L / opf;
        kf = kinf * (Pr / (1.0 + Pr)) * exp(2.302585092994046 * lF);
        if (JAC) {
            const S gg = -L * 2.0 * f / (opf * opf);
            phi = 1.0 / (1.0 + Pr) + gg * (nn / (D * D));  // dln kf / dln Pr
            const S dlF_dL = 1.0 / opf + gg * ((-0.67 * nn + 1.27 * X) / (D * D));
            const S dFc = -(1.0 - a) * iT3 * e3 - a * iT1 * e1 + T2 * x.invT * x.invT * e2;
            dlnF_T = dlF_dL * dFc / Fc;  // dln F/dT at fixed Pr
            dlnk0 = (tr.b0 + tr.Ea0R * x.invT) * x.invT;
        }
    }
    const S kr = kf * exp(-lnKc);
    const S Rf = kf * (p[0] * p[1] * p[2]), Rr = kr * (p[3] * p[4] * p[5]);
    const S q0 = Rf - Rr;
    const bool third = (flags & sc::RXF_TB) && kind == sc::RX_THIRD;
    const S fsc = third ? M : S(1.0);
    o.q = fsc * q0;
    if (!JAC) return o;
    const S F = fsc * kf, B = -fsc * kr;
    o.d[0] = F * (p[1] * p[2]) * dp[0];
    o.d[1] = F * (p[0] * p[2]) * dp[1];
    o.d[2] = F * (p[0] * p[1]) * dp[2];
    o.d[3] = B * (p[4] * p[5]) * dp[3];
    o.d[4] = B * (p[3] * p[5]) * dp[4];
    o.d[5] = B * (p[3] * p[4]) * dp[5];
    const S dlnkinf = (r.bT() + r.EaR() * x.invT) * x.invT;
    const S dlnKc = (dH - dnu) * x.invT;
    S dlnkf = dlnkinf;
    o.dqM = 0.0;
    const S dMdT = m.cv ? S(0.0) : -M0 * x.invT;
    if (flags & sc::RXF_TB) {
        if (kind == sc::RX_THIRD) {
            o.dqM = q0;
        } else if (kind == sc::RX_TROE) {
            o.dqM = q0 * phi / M;
            dlnkf = dlnkinf + phi * (dlnk0 - dlnkinf + dMdT / M) + dlnF_T;
        }
    }
    o.dT = fsc * (q0 * dlnkf + Rr * dlnKc);
    if (third) o.dT += q0 * dMdT;
    // q - sum_s C_s dq/dC_s: (1 - order) of each direction, less the
    // enhanced species' share of [M]
    o.euler = m.cv ? o.dqM
                   : fsc * ((1.0 - r.order(0)) * Rf - (1.0 - r.order(1)) * Rr) - o.dqM * Me;
    o.dH = dH;
    return o;
}

// The reactions' production rates added up in the pairs: the passes of one wave
// (or of its share of a crew's), nxt the first one's record.  A lane adds for
// the slots its reaction uses only: at full occupancy the LDS additions bind,
// about 14 cycles for 64 lanes and more where they meet in one address (with
// every lane adding, the unused slots into trash entries, 65,536 evaluations
// took 341 us instead of 262, 4,096 Jacobians 139 instead of 120, 16,384 cells
// of 9 species 47 ms instead of 40).
template <int G, int NV, bool TABLES, class CR>
__device__ __forceinline__ void rhs_passes(const CR &crew, const DevMech &m, const DevRx &sp, int ideg, double *lds,
                                           const Mix<> &x, const double *dlnA, int lane, const double *itb, double itt,
                                           Rec nxt)
{
    char *wd = (char *)(lds + SPL_HW * NV + 1);
#pragma unroll 1
    for (int q = crew.first(sp), qn; q >= 0; q = qn) {
        qn = crew.next(sp, q);
        const Rec r = nxt;
        nxt = load_rx<G>(sp, max(qn, 0), lane);
        const uint32_t flags = __builtin_amdgcn_readfirstlane(r.bits());
        const double dl = dlnA ? dlnA[r.orig()] : 0.0;
        const RxTerms<> o = reaction_sp<false, NV>(m, sp, ideg, lds, r, flags, q * G + lane, x, dl,
                                                 TABLES ? itb : nullptr, itt);
        crew.await(q);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            if (i == 2 && !(flags & sc::RXF_THIRD_REAC)) continue;
            if (i == 5 && !(flags & sc::RXF_THIRD_PROD)) continue;
            double v = i < 3 ? -o.q : o.q;
            if (flags & sc::RXF_NU) v *= r.nu(i);
            if (r.nu(i) > 0) atomicAdd((double *)(wd + r.slot(i)), v);
        }
        crew.pass_on(q);
    }
}

// The Jacobian pass's sums: the production rates and Euler terms, SGN nu dq/dC
// and SGN nu dq/dT in the species rows of the entries E, the enthalpy-weighted
// derivatives in the temperature row.  OFF: the entries are byte offsets,
// otherwise numbers.  What every reaction adds to, the (T, T) entry and a
// constant-volume reactor's border term, stays in a register per lane (64 LDS
// additions to one address run one by one), a crew's in ts[0] and ts[NV]
// between its waves.
template <int G, int NV, bool OFF, int SGN, bool TABLES, class CR>
__device__ __forceinline__ void jac_passes(const CR &crew, const DevMech &m, const DevRx &sp, int ideg, double *lds,
                                           double *E, const Mix<> &x, double RT, const double *dlnA, int lane,
                                           const double *itb, double itt, Rec nxt, double *ts, double &tt, double &tm)
{
    constexpr double sgn = SGN;
    const int N = m.N;
    char *wd = (char *)(lds + SPL_HW * NV + 1), *ua = (char *)(lds + SPL_UA * NV);
    auto add = [&](uint32_t o, double v) __attribute__((always_inline)) {
        atomicAdd((double *)((char *)E + (OFF ? o : 8 * o)), v);
    };
#pragma unroll 1
    for (int q = crew.first(sp), qn; q >= 0; q = qn) {
        qn = crew.next(sp, q);
        const Rec r = nxt;
        const uint4 *ip = (const uint4 *)sp.ix + (size_t)q * sc::RXW_IX * G + lane;
        uint32_t ix[4 * sc::RXW_IX];
#pragma unroll
        for (int c = 0; c < sc::RXW_IX; ++c) {
            const uint4 w = ip[c * G];
            ix[4 * c] = w.x, ix[4 * c + 1] = w.y, ix[4 * c + 2] = w.z, ix[4 * c + 3] = w.w;
        }
        nxt = load_rx<G>(sp, max(qn, 0), lane);
        const uint32_t flags = __builtin_amdgcn_readfirstlane(r.bits());
        const double dl = dlnA ? dlnA[r.orig()] : 0.0;
        const int j = q * G + lane;
        const RxTerms<> o = reaction_sp<true, NV>(m, sp, ideg, lds, r, flags, j, x, dl,
                                                TABLES ? itb : nullptr, itt);
        auto at = [&](int e) __attribute__((always_inline)) { return e % 2 ? ix[e / 2] >> 16 : ix[e / 2] & 0xffff; };
        // temperature-row weight: the reaction enthalpy (constant pressure) or
        // internal energy (constant volume), per unit of progress
        const double dHJ = m.cv ? (o.dH - r.dnu()) * RT : o.dH * RT;
        uint32_t ie[4 * sc::RXW_IXE];
        auto enhanced = [&]() __attribute__((always_inline)) {
            const uint4 *ep = (const uint4 *)sp.ixe + (size_t)q * sc::RXW_IXE * G + lane;
#pragma unroll
            for (int c = 0; c < sc::RXW_IXE; ++c) {
                const uint4 w = ep[c * G];
                ie[4 * c] = w.x, ie[4 * c + 1] = w.y, ie[4 * c + 2] = w.z, ie[4 * c + 3] = w.w;
            }
        };
        // a crew's wave loads them before its turn
        if (!std::is_same_v<CR, Solo> && (flags & sc::RXF_TB) && j < sp.n_tb) enhanced();
        crew.await(q);
        auto row = [&](auto I, auto NU) __attribute__((always_inline)) {
            constexpr int i = I;
            if (r.nu(i) == 0) return;
            double w = i < 3 ? -1.0 : 1.0;
            if (decltype(NU)::value) w *= r.nu(i);
            // without coefficients the weight is a constant and the products fold to signs
            atomicAdd((double *)(wd + r.slot(i)), w * o.q);
            atomicAdd((double *)(ua + r.slot(i) / 2), w * o.euler);
            add(at(7 * i), sgn * w * o.d[0]);
            add(at(7 * i + 1), sgn * w * o.d[1]);
            if (r.nu(2) > 0) add(at(7 * i + 2), sgn * w * o.d[2]);
            add(at(7 * i + 3), sgn * w * o.d[3]);
            add(at(7 * i + 4), sgn * w * o.d[4]);
            if (r.nu(5) > 0) add(at(7 * i + 5), sgn * w * o.d[5]);
            add(at(7 * i + 6), sgn * w * o.dT);
        };
        auto rows = [&](auto NU) __attribute__((always_inline)) {
            row(std::integral_constant<int, 0>{}, NU);
            row(std::integral_constant<int, 1>{}, NU);
            if (flags & sc::RXF_THIRD_REAC) row(std::integral_constant<int, 2>{}, NU);
            row(std::integral_constant<int, 3>{}, NU);
            row(std::integral_constant<int, 4>{}, NU);
            if (flags & sc::RXF_THIRD_PROD) row(std::integral_constant<int, 5>{}, NU);
        };
        if (flags & sc::RXF_NU)
            rows(std::true_type{});
        else
            rows(std::false_type{});
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            if ((s == 2 || s == 5) && r.nu(s) == 0) continue;
            add(at(42 + s), dHJ * o.d[s]);
        }
        if (crew.w > 1) tt = ts[0], tm = ts[NV];
        tt = fma(dHJ, o.dT, tt);
        if (m.cv) tm = fma(dHJ, o.euler, tm);
        if (crew.w > 1) ts[0] = tt, ts[NV] = tm;
        if ((flags & sc::RXF_TB) && j < sp.n_tb) {
            if (std::is_same_v<CR, Solo>) enhanced();
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const double w = i == 6 ? dHJ * o.dqM : (i < 3 ? -sgn * o.dqM : sgn * o.dqM) * r.nu(i < 6 ? i : 0);
#pragma unroll
                for (int e = 0; e < sc::MAXENH; ++e) {
                    const int k = 4 * i + e;
                    if (r.enh(e) == 16u * N || (i < 6 && r.nu(i) == 0)) continue;
                    add(k % 2 ? ie[k / 2] >> 16 : ie[k / 2] & 0xffff, w * o.ea[e]);
                }
            }
        }
        crew.pass_on(q);
    }
}

// mixture() for the reaction passes: C and g/RT, h/RT and the production rate
// in pairs; what an unused slot of a reaction reads lies in the temperature's
// place N.  The lanes behind it hold the same (the last place, where there are
// more lanes than places).
template <int NP, class S = double>
__device__ __forceinline__ Mix<S> mixture_pairs(const DevMech &m, double *lds, S y, double p, Thermo<S> &th, int lane,
                                                int toff = 0)
{
    constexpr int NV = Lds<NP>::NV;
    // species c's pairs (a Dual's derivatives toff doubles away) and Euler term
    auto put = [&](int c, S conc, S g, S h) __attribute__((always_inline)) {
        const int cg = Lds<NP>::RX + SPL_CG * NV + 2 * c, hw = Lds<NP>::RX + SPL_HW * NV + 2 * c;
        lds_put(lds, cg, conc, toff);
        lds_put(lds, cg + 1, g, toff);
        lds_put(lds, hw, h, toff);
        lds_put(lds, hw + 1, S(0.0), toff);
        lds[Lds<NP>::RX + SPL_UA * NV + c] = 0.0;
    };
    S yw;
    const Mix<S> x = mixture_point(m, y, p, th, lane, yw);
    put(NP < WAVE ? min(lane, NV - 1) : lane, lane < m.N ? x.rho * yw : S(1.0), th.hRT - th.sR, th.hRT);
    return x;
}

// Right-hand side f(y), lane-distributed (0 in padding lanes).
template <int NP>
__device__ __forceinline__ double rhs(const DevMech &m, double *lds, double y, double p, const double *dlnA, int lane)
{
    const int N = m.N;
    constexpr int NV = Lds<NP>::NV;
    double *v = lds + Lds<NP>::RX;
    Thermo<> th;
    const Rec first = load_rx<WAVE>(m.pass, m.pass.passes - 1, lane);
    const Mix<> x = mixture_pairs<NP>(m, lds, y, p, th, lane);
    lds_sync();
    rhs_passes<WAVE, NV, false>(Solo{}, m, m.pass, 0, v, x, dlnA, lane, nullptr, 0.0, first);
    lds_sync();
    double f = 0.0, hw = 0.0;
    if (lane < N) {
        const double wd = pair<NV>(v, SPL_HW, lane)[1];
        f = m.W()[lane] * wd / x.rho;
        hw = (m.cv ? th.hRT - 1.0 : th.hRT) * wd;  // h_k/RT, or u_k/RT at constant volume
    }
    const double H = m.Rgas * x.T * wave_sum(hw);
    if (lane == N) f = -H / (x.rho * x.cp);
    lds_sync();
    return f;
}

// Per-lane coefficients turning row `lane` of the finalised LDS terms into a
// Jacobian row:  J[c] = IW[c] (alpha P[c] + beta) + [c == N] (alphaT P[c] + betaT).
struct RowCoef {
    double alpha, beta, alphaT, betaT;
};

// Jacobian pass: f(y) plus the analytical terms, finalised in LDS.
template <int NP>
__device__ __forceinline__ double rhs_jac(const DevMech &m, double *lds, double y, double p, const double *dlnA, int lane,
                          RowCoef &rc)
{
    const int N = m.N;
    constexpr int NV = Lds<NP>::NV;
    double *P = lds + Lds<NP>::P, *v = lds + Lds<NP>::RX;
    Thermo<> th;
    const Rec first = load_rx<WAVE>(m.pass, m.pass.passes - 1, lane);
    const Mix<> x = mixture_pairs<NP>(m, lds, y, p, th, lane);
#pragma unroll 4
    for (int e = 2 * lane; e < NP * Lds<NP>::PS; e += 2 * WAVE) *(double2 *)(P + e) = make_double2(0.0, 0.0);
    lds_sync();
    const double RT = m.Rgas * x.T;
    double tt = 0.0, tm = 0.0;
    jac_passes<WAVE, NV, true, 1, false>(Solo{}, m, m.pass, 0, v, P, x, RT, dlnA, lane, nullptr, 0.0, first, nullptr,
                                         tt, tm);
    lds_sync();
    // m.cv: the energy balance is on u_k = h_k - R T, the heat capacity c_v
    const double one = m.cv ? 1.0 : 0.0;
    // No branches from here to the factorisation: the compiler puts the copies
    // of the registers it keeps over it at the last point where branches join,
    // and there before the join, where the lanes of one side miss them.
    const bool own = lane < N;
    const int k = min(lane, N - 1);
    const double Wk = own ? m.W()[k] : 0.0, iw = own ? m.invW()[k] : 0.0;
    const double wd = own ? pair<NV>(v, SPL_HW, k)[1] : 0.0, ua = own ? v[SPL_UA * NV + k] : 0.0;
    double f = Wk * wd / x.rho;
    const double uk = Wk * ua / x.rho;
    const double hw = (th.hRT - one) * wd;
    const double eu = th.hRT * uk * iw;           // (h_k/(R T W_k)) u_k
    const double cpf = (th.cpR - one) * f * iw;   // cp_k/(R W_k) f_k (cv_k at constant volume)
    const double dcp = th.dcpR * y * iw;          // dcp_k/dT/(R W_k) Y_k
    const double H = RT * wave_sum(hw);
    const double Eu = m.cv ? 0.0 : RT * wave_sum(eu);  // sum_k (h_k/W_k) u_k
    const double Scpf = m.Rgas * wave_sum(cpf);
    const double Sdcp = m.Rgas * wave_sum(dcp);
    const double fT = -H / (x.rho * x.cp);
    f = lane == N ? fT : f;
    // fold the column-dependent parts of the temperature row into P[N][*].
    // Constant pressure:
    //   J_Tm = -(1/cp) (1/W_m) (P_Tm + Wbar Eu + fT cp_m),
    //   J_TT = -(1/cp) (P_TT/rho + Eu/T + sum cp_k f_k/W_k + fT sum dcp_k Y_k/W_k);
    // constant volume (C_k = rho Y_k/W_k, no density border; the rank-one
    // part of d[M]/dC accumulated in tb for this row, UA[k] for row k):
    //   J_Tm = -(1/cv) (1/W_m) (P_Tm + tb + fT cv_m),
    //   J_TT = -(1/cv) (P_TT/rho + sum cv_k f_k/W_k + fT sum dcp_k Y_k/W_k)
    const int PS = Lds<NP>::PS;
    const double TT = wave_sum(tt), tb = m.cv ? wave_sum(tm) : x.Wbar * Eu;
    double *row = P + (lane <= N ? N * PS + lane : lane % 16 * PS + NP);  // the others': the column behind
    *row = own ? *row + (tb + fT * m.Rgas * (th.cpR - one)) : TT / x.rho + Eu * x.invT + Scpf + fT * Sdcp;
    lds[Lds<NP>::IW + (NP < WAVE ? min(lane, NP - 1) : lane)] = iw;  // zero from the temperature's place on
    lds_sync();
    const double invcp = 1.0 / x.cp;
    // species rows, constant pressure: J_km = (W_k/W_m) P_km + u_k Wbar/W_m,
    // J_kT = (W_k/rho) P_kT + u_k/T; constant volume: J_km = (W_k/W_m)
    // (P_km + UA_k), J_kT = (W_k/rho) P_kT.  W_k, u_k and UA_k are zero in the
    // other lanes.
    rc.alpha = lane == N ? -invcp : Wk;
    rc.beta = m.cv ? Wk * ua : uk * x.Wbar;
    rc.alphaT = lane == N ? -invcp : Wk / x.rho;
    rc.betaT = m.cv ? 0.0 : uk * x.invT;
    return f;
}

// Row `lane` of J from the finalised LDS terms into registers.
template <int NP>
__device__ __forceinline__ void jac_row(const DevMech &m, const double *lds, const RowCoef &rc, int lane,
                                        double (&a)[NP])
{
    const int N = m.N;
    const double *P = lds + Lds<NP>::P + (lane < NP ? lane : 0) * Lds<NP>::PS;
    const double *IW = lds + Lds<NP>::IW;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
        const double pv = P[c];
        const double t = c == N ? fma(rc.alphaT, pv, rc.betaT) : 0.0;
        a[c] = fma(IW[c], fma(rc.alpha, pv, rc.beta), t);
        SC_FENCE_EVERY(c);
    }
}

// M = I/hg - J into registers (padding rows get the identity).
template <int NP>
__device__ __forceinline__ void form_matrix(const DevMech &m, const double *lds, const RowCoef &rc, int lane,
                                            double inv_hg, double (&a)[NP])
{
    jac_row<NP>(m, lds, rc, lane, a);
    const int n = m.N + 1;
    const double diag = lane < n ? inv_hg : 1.0;
#pragma unroll
    for (int c = 0; c < NP; ++c) a[c] = c == lane ? diag - a[c] : -a[c];
}

// LU without pivoting, natural order, of the rows in registers (row i in lane
// i), parked in F column-major (F[c PS + i] = row i, column c): below the
// diagonal L with a unit diagonal, above it U scaled to one, and in the
// lanes' return value 1/U_ii.  A broadcast of one lane to the 16 of its row
// costs nothing inside a multiply-add (DPP), where one to the whole wave takes
// two readlanes at twice a multiply-add's time each; so the pivots go in
// blocks of 16, whose rows S are copied to all four rows of lanes, and every
// row of lanes eliminates in its copy and in its own rows from that.  The
// block's columns leave for F and the others move to the front, so that one
// piece of code does every block and stays in the instruction cache.  (As one
// unrolled elimination with a readlane pair per entry, 64 KB of code, 53
// species took 134k cycles of a lone wave, most of them waiting for
// instructions; 45k now.)
template <int NP>
__device__ __forceinline__ double lu_factor(double (&a)[NP], double *F, int lane)
{
    constexpr int PS = Lds<NP>::PS, NR = (NP + 15) / 16 * 16;  // columns, up to whole blocks
    int c = lane & 15, row = lane >> 4;
    double r[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) r[j] = j < NP ? a[j < NP ? j : 0] : 0.0;
    double dinv = 0.0;
#pragma unroll 1
    for (int b = 0; b < NR / 16; ++b) {
        asm volatile("" : "+v"(c), "+v"(row));  // the masks are cheaper made again than kept and spilled
        const int k0 = 16 * b;
        const bool in = row == b, after = row > b;
        const int from = 4 * (k0 + c);
        auto spread = [&](double v) __attribute__((always_inline)) {
            return __hiloint2double(__builtin_amdgcn_ds_bpermute(from, __double2hiint(v)),
                                    __builtin_amdgcn_ds_bpermute(from, __double2loint(v)));
        };
        double S[16], db = 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j) S[j] = spread(r[j]);
        unrolled<16>([&](auto K) __attribute__((always_inline)) {
            constexpr int k = K;
            if (NP % 16 == 0 || k < NP % 16 || k0 + k < NP) {
                const double inv = 1.0 / bcast<16, k>(S[k]);
                const double l = c > k ? S[k] * inv : 0.0, lr = after ? r[k] * inv : 0.0;
                db = c == k ? inv : db;
                S[k] = c > k ? l : S[k];
                r[k] = after ? lr : r[k];
                if constexpr (k < 15) fmac_row<k>(S[k + 1], l);
                constexpr int j0 = k + 2;
#pragma unroll
                for (int j = j0; j + 3 < 16; j += 4) fmac_row4<k>(S[j], S[j + 1], S[j + 2], S[j + 3], l);
#pragma unroll
                for (int j = j0 + (j0 < 16 ? (16 - j0) / 4 * 4 : 0); j < 16; ++j) fmac_row<k>(S[j], l);
#pragma unroll
                for (int j = k + 1; j + 3 < 16; j += 4)
                    fmac_from4<k>(r[j], r[j + 1], r[j + 2], r[j + 3], S[j], S[j + 1], S[j + 2], S[j + 3], lr);
#pragma unroll
                for (int j = k + 1 + (15 - k) / 4 * 4; j < 16; ++j) fmac_from<k>(r[j], S[j], lr);
            }
        });
        dinv = in ? db : dinv;
        double *Fb = F + k0 * PS + min(lane, NP);  // lanes without a row: the row behind
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (NP % 16 == 0 || k < NP % 16 || k0 + k < NP) Fb[k * PS] = in ? S[k] * (k > c ? db : 1.0) : r[k];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            S[k] = c > k ? S[k] : 0.0;
            r[k] = after ? r[k] : 0.0;
        }
#pragma unroll
        for (int j = 16; j < NR; j += 4)
            if (k0 + j < NP) {
                double s0 = spread(r[j]), s1 = spread(r[j + 1]), s2 = spread(r[j + 2]), s3 = spread(r[j + 3]);
                unrolled<15>([&](auto K) __attribute__((always_inline)) { fmac_row4<K>(s0, s1, s2, s3, S[K]); });
                unrolled<16>([&](auto K) __attribute__((always_inline)) {
                    fmac_from4<K>(r[j], r[j + 1], r[j + 2], r[j + 3], s0, s1, s2, s3, r[K]);
                });
                r[j] = in ? s0 * db : r[j];
                r[j + 1] = in ? s1 * db : r[j + 1];
                r[j + 2] = in ? s2 * db : r[j + 2];
                r[j + 3] = in ? s3 * db : r[j + 3];
            }
#pragma unroll
        for (int j = 16; j < NR; ++j) r[j - 16] = r[j];
    }
    return dinv;
}

// Solve with the factors in F, b lane-distributed: (L D U) x = b, or with
// `transposed` the transpose, U^T D L^T.  Lane j's coefficient of unknown k is
// the entry at (j, k), transposed (k, j); PS is odd, so both reads fall on
// different banks.  The chain through a block's 16 unknowns runs inside the
// row of lanes that holds them, one broadcasting multiply-add each; the
// block's solution is then spread to all rows of lanes and those behind it
// apply it, off the chain.
template <int NP, bool transposed = false>
__device__ __forceinline__ double lu_solve(const double *F, double dinv, double b, int lane)
{
    constexpr int PS = Lds<NP>::PS, NB = (NP + 15) / 16;
    const double *Fl = F + (lane < NP ? lane : 0) * (transposed ? PS : 1);
    asm volatile("" : "+v"(lane));  // the masks below are cheaper made again than kept and spilled
    auto load = [&](int q, bool lower, double (&a)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int k = 16 * q + i;
            const double v = k < NP ? Fl[k * (transposed ? 1 : PS)] : 0.0;
            a[i] = (lower ? lane > k : lane < k) ? v : 0.0;
        }
    };
    double a[16], nx[16];
    load(0, true, a);
    unrolled<NB>([&](auto Q) __attribute__((always_inline)) {
        constexpr int q = Q;
        if constexpr (q + 1 < NB) load(q + 1, true, nx);
        unrolled<15>([&](auto K) __attribute__((always_inline)) {
            if constexpr (16 * q + K < NP) fmac_in<K, 1 << q>(b, a[K]);
        });
        if constexpr (q + 1 < NB) {
            const double x = spread_row<q>(b);
            constexpr int behind = 0xf & ~((2 << q) - 1);
            unrolled<4>([&](auto K) __attribute__((always_inline)) { fmac_by4<4 * K, behind>(b, x, &a[4 * K]); });
#pragma unroll
            for (int i = 0; i < 16; ++i) a[i] = nx[i];
        }
    });
    b *= dinv;
    load(NB - 1, false, a);
    unrolled<NB>([&](auto Q) __attribute__((always_inline)) {
        constexpr int q = NB - 1 - Q;
        if constexpr (q > 0) load(q - 1, false, nx);
        unrolled<15>([&](auto K) __attribute__((always_inline)) {
            if constexpr (16 * q + 15 - K < NP) fmac_in<15 - K, 1 << q>(b, a[15 - K]);
        });
        if constexpr (q > 0) {
            const double x = spread_row<q>(b);
            constexpr int behind = (1 << q) - 1;
            unrolled<4>([&](auto K) __attribute__((always_inline)) { fmac_by4<4 * K, behind>(b, x, &a[4 * K]); });
#pragma unroll
            for (int i = 0; i < 16; ++i) a[i] = nx[i];
        }
    });
    return lane < NP ? b : 0.0;
}

// Form, factorise and park M = I/hg - J in F (the LDS term region itself,
// or per-cell global scratch); returns 1/U_ii of this lane.
template <int NP>
__device__ __forceinline__ double factor_matrix(const DevMech &m, double *lds, const RowCoef &rc, int lane,
                                                double inv_hg, double *F)
{
    double a[NP];
    form_matrix<NP>(m, lds, rc, lane, inv_hg, a);
    wave_sync();  // every lane has read its row of the terms
    const double dinv = lu_factor<NP>(a, F, lane);
    wave_sync();
    return dinv;
}

// One Rosenbrock attempt of size hc from y: Jacobian pass, factorisation
// (parked in F), the four stages (stage vectors u_i left in LDS) and the
// embedded error.  Returns the new state; *err gets the scaled RMS error.
// Forward integration and adjoint replay both call this, so a replayed
// step reproduces the recorded one bit for bit.
template <int NP>
__device__ __forceinline__ double ros_attempt(const DevMech &m, const Opts &o, double *lds, double *F, double y, double p,
                              const double *dlnA, int lane, double hc, double *err, double *dinv_out = nullptr)
{
    const int n = m.N + 1;
    double *U = lds + Lds<NP>::U;
    RowCoef rc;
    const double f0 = rhs_jac<NP>(m, lds, y, p, dlnA, lane, rc);
    const double dinv = factor_matrix<NP>(m, lds, rc, lane, 1.0 / (GAM * hc), F);
    if (dinv_out) *dinv_out = dinv;
    const double ih = 1.0 / hc;
    double flast = f0;
#pragma unroll 1
    for (int i = 0; i < NS; ++i) {
        double fi;
        const int reuse = TREUSE[i];
        if (reuse == 0) {
            fi = f0;
        } else if (reuse > 0) {
            fi = flast;  // the stage it names is the last one evaluated
        } else {
            double ys = y;
            for (int j = 0; j < i; ++j) ys += TA[i][j] * U[j * WAVE + lane];
            fi = rhs<NP>(m, lds, ys, p, dlnA, lane);
            flast = fi;
        }
        for (int j = 0; j < i; ++j) fi += (TC[i][j] * ih) * U[j * WAVE + lane];
        if (lane >= n) fi = 0.0;
        U[i * WAVE + lane] = lu_solve<NP>(F, dinv, fi, lane);
    }
    double ynew = y, ev = 0.0;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const double ui = U[i * WAVE + lane];
        ynew += TM[i] * ui;
        ev += TE[i] * ui;
    }
    double e2 = 0.0;
    if (lane < n) {
        const double sc = o.atol + o.rtol * fmax(fabs(y), fabs(ynew));
        const double r = ev / sc;
        e2 = r * r;
    }
    *err = sqrt(wave_sum(e2) / n);
    return ynew;
}

// One step of the extrapolation baseline: the linearly implicit Euler method
//   (I - h J(y0)) (y_{i+1} - y_i) = h f(y_i),  h = H / n_j,
// on the step numbers n_j = j (j = 1..EXK), each column's end state T_{j,1}
// extrapolated to h -> 0 by Aitken-Neville for an expansion in powers of h,
//   T_{j,l+1} = T_{j,l} + (T_{j,l} - T_{j-1,l}) (j - l) / l.
// T_{EXK,EXK} is the new state (order EXK); T_{EXK,EXK} - T_{EXK,EXK-1} the
// error estimate (order EXK - 1 local error, so the controller's
// err^(-1/4) matches EXK = 4).  The LDS term region holds one matrix, so
// each column recomputes J(y0) before factorising I/h - J (the same
// Jacobian: the pass is deterministic).  Row j of the tableau overwrites
// row j - 1 in the stage-vector area U.
constexpr int EXK = 4;
template <int NP>
__device__ __forceinline__ double extrap_attempt(const DevMech &m, const Opts &o, double *lds, double y, double p,
                                 const double *dlnA, int lane, double H, double *err)
{
    const int n = m.N + 1;
    double *U = lds + Lds<NP>::U;
    double *F = lds + Lds<NP>::P;
    double tkk = y, tk1 = y;
#pragma unroll 1
    for (int j = 1; j <= EXK; ++j) {
        RowCoef rc;
        const double f0 = rhs_jac<NP>(m, lds, y, p, dlnA, lane, rc);
        const double h = H / j;
        const double dinv = factor_matrix<NP>(m, lds, rc, lane, 1.0 / h, F);
        double yi = y, fi = f0;
#pragma unroll 1
        for (int i = 0; i < j; ++i) {
            if (i > 0) fi = rhs<NP>(m, lds, yi, p, dlnA, lane);
            if (lane >= n) fi = 0.0;
            yi += lu_solve<NP>(F, dinv, fi, lane);
        }
        // row j of the tableau from row j - 1 (U[l-1] holds T_{j-1,l})
        double t = yi;
#pragma unroll 1
        for (int l = 1; l < j; ++l) {
            const double told = U[(l - 1) * WAVE + lane];
            const double next = t + (t - told) * ((double)(j - l) / (double)l);
            U[(l - 1) * WAVE + lane] = t;
            t = next;
        }
        U[(j - 1) * WAVE + lane] = t;
        if (j == EXK) {
            tkk = t;
            tk1 = U[(EXK - 2) * WAVE + lane];
        }
    }
    double e2 = 0.0;
    if (lane < n) {
        const double sc = o.atol + o.rtol * fmax(fabs(y), fabs(tkk));
        const double r = (tkk - tk1) / sc;
        e2 = r * r;
    }
    *err = sqrt(wave_sum(e2) / n);
    return lane < n ? tkk : 0.0;
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
__device__ __forceinline__ double load_state(const DevMech &m, const double *T, const double *Y, int64_t ld,
                                             int64_t c, int lane)
{
    if (lane < m.N) return Y[(int64_t)lane * ld + c];
    if (lane == m.N) return T[c];
    return 0.0;
}

// ---------------------------------------------------------------------------
// step-size controller
// ---------------------------------------------------------------------------
// Controller state of one cell.
struct Ctl {
    double t, h, hnext;
    int nacc, nrej, nonfinite;
    bool last_rej;
};

__device__ __forceinline__ Ctl ctl_init(double h, double dt) { return Ctl{0.0, h, dt, 0, 0, 0, false}; }

// Size of the next attempt.  Returns SC_CELL_OK (hc and last set) or the
// status that ends the cell.
__device__ __forceinline__ int ctl_begin(const Ctl &s, const Opts &o, double dt, double &hc, bool &last)
{
    if (s.nacc + s.nrej >= o.max_steps) return SC_CELL_MAX_STEPS;
    if (s.h < 1e-20 * dt) return SC_CELL_H_UNDERFLOW;
    last = false;
    hc = o.hmax_frac > 0.0 ? fmin(s.h, o.hmax_frac * dt) : s.h;
    if (s.t + hc >= dt) {
        hc = dt - s.t;
        last = true;
    }
    return SC_CELL_OK;
}

// Decision on an attempt of size hc with scaled error err: 1 accepted,
// 0 rejected, or minus the status that ends the cell.  Adaptive mode: new
// step 0.9 err^(-1/4) clamped to [0.2, 6] (no growth right after a
// rejection); five non-finite estimates in a row give up.  Fixed mode: every
// finite attempt is accepted and h stays.
__device__ __forceinline__ int ctl_end(Ctl &s, const Opts &o, double err, double hc, bool last, double dt)
{
    if (o.fixed) {
        if (!isfinite(err)) return -SC_CELL_NONFINITE;
        ++s.nacc;
        s.t = last ? dt : s.t + hc;
        s.hnext = s.h;
        return 1;
    }
    if (!isfinite(err)) {
        ++s.nrej;
        s.h = hc * 0.2;
        s.last_rej = true;
        if (++s.nonfinite >= 5) return -SC_CELL_NONFINITE;
        return 0;
    }
    s.nonfinite = 0;
    // err^(-1/4) as two correctly rounded square roots: no library pow,
    // whose simplification depends on the surrounding code, so every
    // kernel that runs the controller takes the same steps
    double fac = 0.9 / sqrt(sqrt(fmax(err, 1e-300)));
    fac = fmin(6.0, fmax(0.2, fac));
    if (err <= 1.0) {
        ++s.nacc;
        s.t = last ? dt : s.t + hc;
        if (s.last_rej) fac = fmin(fac, 1.0);
        s.last_rej = false;
        s.h = hc * fac;
        s.hnext = s.h;
        return 1;
    }
    ++s.nrej;
    s.last_rej = true;
    s.h = hc * fmin(fac, 1.0);
    return 0;
}

// Integrate one cell's state y over [0, dt] (dt > 0) from the initial step
// h: error-controlled (or fixed) steps of the method METH (SC_METHOD_*).
// Returns the cell status; the controller state (step counts, proposed
// next step) is left in s.
template <int NP, int METH = SC_METHOD_ROS4>
__device__ __forceinline__ int advance(const DevMech &m, const Opts &o, double *lds, double &y, double p, double dt,
                       const double *dlnA, int lane, Ctl &s)
{
#pragma unroll 1
    while (true) {
        double hc;
        bool last;
        const int st = ctl_begin(s, o, dt, hc, last);
        if (st != SC_CELL_OK) return st;
        double err;
        double ynew;
        if constexpr (METH == SC_METHOD_EXTRAP)
            ynew = extrap_attempt<NP>(m, o, lds, y, p, dlnA, lane, hc, &err);
        else
            ynew = ros_attempt<NP>(m, o, lds, lds + Lds<NP>::P, y, p, dlnA, lane, hc, &err);
        const int r = ctl_end(s, o, err, hc, last, dt);
        if (r < 0) return -r;
        if (r == 1) {
            y = ynew;
            if (last) return SC_CELL_OK;
        }
    }
}

// Validate a cell's inputs (uniform decision over the wave).
__device__ __forceinline__ bool bad_input(const DevMech &m, double y, double p, double dt, int lane)
{
    const int n = m.N + 1;
    const bool bad_lane = lane < n && !isfinite(y);
    const double T = rdlane(y, m.N);
    return __any(bad_lane) || !(T > 0.0) || !isfinite(T) || !(p > 0.0) || !isfinite(p) || !(dt >= 0.0) ||
           !isfinite(dt);
}

// Initial step: dt, or the caller's h when positive and finite (capped at dt).
__device__ __forceinline__ double initial_step(const double *h_io, int64_t c, double dt)
{
    double h = dt;
    if (h_io) {
        const double h0 = h_io[c];
        if (h0 > 0.0 && isfinite(h0)) h = fmin(h0, dt);
    }
    return h;
}
}  // namespace scdev
