// Kernels with the sparse linear algebra (gfx950): one 64-lane wavefront per
// cell, as in the dense kernels, but the iteration matrix lives in LDS as the
// L+U entries of the bordered system the mechanism compiler built
// (sparse.cpp).  State vectors hold VPL components per lane (component
// c = lane + 64 v, species in elimination order), so mechanisms of up to 126
// species fit one wave; small ones run two or four cells per wave.
//
// The bordered system (order N + 2, unknowns z_k = x_k / W_k, x_T, sigma):
//   row k:     z_k/hg - sum_m P_km z_m - us_k sigma - (P_kT/rho + ct us_k) x_T = b_k / W_k
//   row T:     sum_m A_Tm z_m + A_TT x_T = b_T
//   row sigma: vs sum_m z_m - sigma = 0
// with P_km = sum_j nu_kj dq_j/dC_m (the sparse analytical terms, scattered
// reaction by reaction), us_k = UA_k/rho, vs = Wbar, ct = 1/T at constant
// pressure (the density border) and us_k = UA_k, vs = 1, ct = 0 at constant
// volume (the total-concentration border); UA_k = sum_j nu_kj e_j with e_j
// the reaction's Euler remainder (constant pressure) or dq_j/d[M] (constant
// volume).  Eliminating sigma gives back M = I/hg - J exactly (paper
// Sec. 2.5: sparse analytical Jacobian, sparse algebra management).
//
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "core.hpp"

namespace scdev {


// ---------------------------------------------------------------------------
// lane geometry: G lanes per cell.  G = 64: one cell per wave, VPL slots per
// lane.  G = 32 or 16: two or four cells per wave (mechanisms whose N + 2
// positions fit G), each cell in its own aligned group of lanes with one
// slot per lane.  Below, `lane` is the lane within the cell's group; sums
// and broadcasts stay inside the group.
// ---------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ double gsum(double v)
{
    return group_sum<G>(v);
}

template <int G>
__device__ __forceinline__ double gbcast(double v, int k)
{
    if constexpr (G == WAVE)
        return rdlane(v, k);
    else
        return __shfl(v, k, G);
}

template <int G>
__device__ __forceinline__ bool gany(bool b)
{
    if constexpr (G == WAVE)
        return __any(b);
    else
        return gsum<G>(b ? 1.0 : 0.0) > 0.0;
}

// ---------------------------------------------------------------------------
// helpers over VPL components per lane
// ---------------------------------------------------------------------------
template <int VPL, int G = WAVE>
__device__ __forceinline__ double vsum(const double (&a)[VPL])
{
    double s = a[0];
#pragma unroll
    for (int v = 1; v < VPL; ++v) s += a[v];
    return gsum<G>(s);
}

// the temperature component c = N sits in slot N / 64, lane N % 64 (with
// two slots per lane, N = 63 still has it in the first)
template <int VPL, int G = WAVE>
__device__ __forceinline__ double comp_T(const DevMech &m, const double (&y)[VPL])
{
    if (VPL == 1 || m.N < 64) return gbcast<G>(y[0], m.N & 63);
    return gbcast<G>(y[VPL - 1], m.N & 63);
}

template <int VPL, int G = WAVE>
__device__ __forceinline__ void load_state_v(const DevMech &m, const DevSparse &sp, const double *T, const double *Y, int64_t ld,
                                             int64_t cell, int lane, double (&y)[VPL])
{
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        y[v] = c < m.N ? Y[(int64_t)sp.perm[c] * ld + cell] : c == m.N ? T[cell] : 0.0;
    }
}

template <int VPL, int G = WAVE>
__device__ __forceinline__ void store_state_v(const DevMech &m, const DevSparse &sp, double *T, double *Y, int64_t ld, int64_t cell,
                                              int lane, const double (&y)[VPL])
{
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        if (c < m.N) Y[(int64_t)sp.perm[c] * ld + cell] = y[v];
        if (c == m.N) T[cell] = y[v];
    }
}

// ---------------------------------------------------------------------------
// thermodynamics, right-hand side and Jacobian terms
// ---------------------------------------------------------------------------
// Mixture state from y; writes C, g/RT, h/RT and clears the accumulators.
template <int VPL, int G = WAVE>
__device__ __forceinline__ Mix<> mixture_v(const DevMech &m, const DevSparse &sp, double *lds,
                                           const double (&y)[VPL], double p, Thermo<> (&th)[VPL], int lane)
{
    const int N = m.N;
    Mix<> x;
    x.T = comp_T<VPL, G>(m, y);
    x.invT = 1.0 / x.T;
    x.lnT = log(x.T);
    x.p = p;
    double yw[VPL], cpw[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        th[v] = Thermo<>{0.0, 0.0, 0.0, 0.0};
        yw[v] = cpw[v] = 0.0;
        if (c < N) {
            th[v] = nasa7<double>(m, c, x.T, x.lnT, x.invT);
            yw[v] = y[v] * m.invW()[c];
            cpw[v] = th[v].cpR * yw[v];
        }
    }
    x.Wbar = 1.0 / vsum<VPL, G>(yw);
    x.cp = m.Rgas * vsum<VPL, G>(cpw);
    if (m.cv) {
        x.rho = p;
        x.p = p * m.Rgas * x.T / x.Wbar;
        x.cp = x.cp - m.Rgas / x.Wbar;
    } else {
        x.rho = p * x.Wbar * x.invT / m.Rgas;
    }
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        if (c < N) {
            lds[sp.C + c] = x.rho * yw[v];
            lds[sp.G + c] = th[v].hRT - th[v].sR;
            lds[sp.H + c] = th[v].hRT;
            lds[sp.WD + c] = 0.0;
        }
        if (c <= N) lds[sp.UA + c] = 0.0;
    }
    return x;
}

// A kernel instantiated without the tables sees a null table pointer as a
// compile-time constant, so the tables' code paths fold away.
template <bool TB>
__device__ __forceinline__ DevSparse fix_tables(DevSparse sp)
{
    if constexpr (!TB) sp.itab = nullptr;
    return sp;
}

// With interpolated thermodynamics: the cell's interval of the table (its
// reactions' coefficient blocks) and the local coordinate t in [-1, 1];
// null for exact thermodynamics or a T outside the table's range.
__device__ __forceinline__ const double *thermo_block(const DevSparse &sp, int R, double lnT, double &t)
{
    t = 0.0;
    if (!sp.itab) return nullptr;
    const double uu = (lnT - sp.iu0) * sp.iinvdu;
    if (!(uu >= 0.0) || !(uu < (double)sp.inint)) return nullptr;
    const int iv = (int)uu;
    t = 2.0 * (uu - iv) - 1.0;
    return sp.itab + (size_t)iv * R * 2 * (sp.ideg + 1);
}

// f(y): dY_k/dt and dT/dt, VPL components per lane (0 beyond N).
template <int VPL, int G = WAVE>
__device__ __forceinline__ void rhs_v(const DevMech &m, const DevSparse &sp, double *lds, const double (&y)[VPL], double p,
                      const double *dlnA, int lane, double (&f)[VPL])
{
    const int N = m.N, R = m.R;
    Thermo<> th[VPL];
    const Mix<> x = mixture_v<VPL, G>(m, sp, lds, y, p, th, lane);
    double itt;
    const double *itb = thermo_block(sp, R, x.lnT, itt);
    __syncthreads();
    // the reaction loop, compiled once with the tables and once without (the
    // exact path's code does not carry the tables' branches)
    auto pass = [&](auto tables) __attribute__((always_inline)) {
#pragma unroll 1
        for (int j = lane; j < R; j += G) {
            const RxRec rr = load_rec(m, j);
            const double dl = dlnA ? dlnA[rr.orig] : 0.0;
            RxOut<> o;
            if constexpr (decltype(tables)::value)
                o = reaction<false>(m, lds, rr, x, dl, sp.C, sp.G, sp.H, 0, itb + (size_t)j * 2 * (sp.ideg + 1), itt,
                                    sp.ideg);
            else
                o = reaction<false>(m, lds, rr, x, dl, sp.C, sp.G, sp.H);
#pragma unroll
            for (int i = 0; i < sc::MAXSIDE; ++i) {
                if (i < rr.nr) atomicAdd(&lds[sp.WD + rr.rsp[i]], -(double)rr.rnu[i] * o.q);
                if (i < rr.np) atomicAdd(&lds[sp.WD + rr.psp[i]], (double)rr.pnu[i] * o.q);
            }
        }
    };
    if (itb)
        pass(std::true_type{});
    else
        pass(std::false_type{});
    __syncthreads();
    double hw[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        f[v] = hw[v] = 0.0;
        if (c < N) {
            const double wd = lds[sp.WD + c];
            f[v] = m.W()[c] * wd / x.rho;
            hw[v] = (m.cv ? th[v].hRT - 1.0 : th[v].hRT) * wd;
        }
    }
    const double fT = -m.Rgas * x.T * vsum<VPL, G>(hw) / (x.rho * x.cp);
#pragma unroll
    for (int v = 0; v < VPL; ++v)
        if (lane + G * v == N) f[v] = fT;
    __syncthreads();
}

// Jacobian pass: f(y), and the bordered matrix of I/hg - J formed in the L+U
// entries (fill entries zero).  The reaction loop scatters -nu dq/dC and
// -nu dq/dT into the species rows and the reaction-enthalpy-weighted
// derivatives into the temperature row; the border entries are finished per
// state component after one barrier.
template <int VPL, int G = WAVE>
__device__ __forceinline__ void jac_v(const DevMech &m, const DevSparse &sp, double *lds, const double (&y)[VPL], double p,
                      const double *dlnA, int lane, double inv_hg, double (&f)[VPL])
{
    const int N = m.N, R = m.R;
    double *E = lds + sp.E;
    Thermo<> th[VPL];
    const Mix<> x = mixture_v<VPL, G>(m, sp, lds, y, p, th, lane);
#pragma unroll 4
    for (int e = lane; e <= sp.nnz; e += G) E[e] = 0.0;  // and the zero slot E[nnz]
    __syncthreads();
    const double RT = m.Rgas * x.T;
    double itt;
    const double *itb = thermo_block(sp, R, x.lnT, itt);
    auto pass = [&](auto tables) __attribute__((always_inline)) {
#pragma unroll 1
    for (int j = lane; j < R; j += G) {
        const RxRec rr = load_rec(m, j);
        const double dl = dlnA ? dlnA[rr.orig] : 0.0;
        RxOut<> o;
        if constexpr (decltype(tables)::value)
            o = reaction<true>(m, lds, rr, x, dl, sp.C, sp.G, sp.H, 0, itb + (size_t)j * 2 * (sp.ideg + 1), itt,
                               sp.ideg);
        else
            o = reaction<true>(m, lds, rr, x, dl, sp.C, sp.G, sp.H);
        // the reaction's entry indices are loaded once its rate terms are
        // done, so they do not hold registers through the rate arithmetic
        __builtin_amdgcn_sched_barrier(0);
        uint16_t ix[sc::RXI_SIZE];
        __builtin_memcpy(ix, sp.rxi + (size_t)j * sc::RXI_SIZE, sizeof ix);
        // temperature-row weight: the reaction enthalpy (constant pressure) or
        // internal energy (constant volume), per unit of progress
        const double dHJ = m.cv ? (o.dH - rr.dnu) * RT : o.dH * RT;
        bool use[sc::NDEP];
#pragma unroll
        for (int i = 0; i < sc::MAXSIDE; ++i) {
            use[i] = i < rr.nr;
            use[3 + i] = i < rr.np;
        }
#pragma unroll
        for (int e = 0; e < sc::MAXENH; ++e) use[6 + e] = e < rr.neff;
#pragma unroll
        for (int r = 0; r < 2 * sc::MAXSIDE; ++r) {
            const bool isr = r < sc::MAXSIDE;
            const int ri = isr ? r : r - sc::MAXSIDE;
            if (ri >= (isr ? rr.nr : rr.np)) continue;
            const int row = isr ? rr.rsp[ri] : rr.psp[ri];
            const double nu = isr ? -(double)rr.rnu[ri] : (double)rr.pnu[ri];
            atomicAdd(&lds[sp.WD + row], nu * o.q);
            atomicAdd(&lds[sp.UA + row], nu * o.euler);
#pragma unroll
            for (int s = 0; s < sc::NDEP; ++s)
                if (use[s]) atomicAdd(&E[ix[r * sc::RXI_ROW + s]], -nu * o.d[s]);
            atomicAdd(&E[ix[r * sc::RXI_ROW + sc::NDEP]], -nu * o.dT);
        }
#pragma unroll
        for (int s = 0; s < sc::NDEP; ++s)
            if (use[s]) atomicAdd(&E[ix[sc::RXI_TROW + s]], dHJ * o.d[s]);
        atomicAdd(&E[ix[sc::RXI_TROW + sc::NDEP]], dHJ * o.dT);
        if (m.cv) atomicAdd(&lds[sp.UA + N], dHJ * o.euler);
    }
    };
    if (itb)
        pass(std::true_type{});
    else
        pass(std::false_type{});
    __syncthreads();
    const double one = m.cv ? 1.0 : 0.0;
    double hw[VPL], eu[VPL], cpf[VPL], dcp[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        f[v] = hw[v] = eu[v] = cpf[v] = dcp[v] = 0.0;
        if (c < N) {
            const double Wk = m.W()[c], iw = m.invW()[c];
            const double wd = lds[sp.WD + c], ua = lds[sp.UA + c];
            f[v] = Wk * wd / x.rho;
            hw[v] = (th[v].hRT - one) * wd;
            eu[v] = th[v].hRT * ua / x.rho;      // (h_k/(R T W_k)) u_k, u_k = W_k UA_k / rho
            cpf[v] = (th[v].cpR - one) * f[v] * iw;
            dcp[v] = th[v].dcpR * y[v] * iw;
        }
    }
    const double H = RT * vsum<VPL, G>(hw);
    const double Eu = m.cv ? 0.0 : RT * vsum<VPL, G>(eu);
    const double Scpf = m.Rgas * vsum<VPL, G>(cpf);
    const double Sdcp = m.Rgas * vsum<VPL, G>(dcp);
    const double fT = -H / (x.rho * x.cp);
    const double vs = m.cv ? 1.0 : x.Wbar;
    const double ct = m.cv ? 0.0 : x.invT;
    const double tb = m.cv ? lds[sp.UA + N] : x.Wbar * Eu;
    const double icp = 1.0 / x.cp;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        const uint16_t *cm = sp.comp + 8 * c;
        if (c < N) {
            const double us = m.cv ? lds[sp.UA + c] : lds[sp.UA + c] / x.rho;
            E[cm[0]] += inv_hg;
            E[cm[1]] = E[cm[1]] / x.rho - ct * us;
            E[cm[2]] = -us;
            E[cm[3]] = (E[cm[3]] + tb + fT * m.Rgas * (th[v].cpR - one)) * icp;
            E[cm[4]] = vs;
        } else if (c == N) {
            f[v] = fT;
            const double eT = m.cv ? 0.0 : Eu * x.invT;
            E[cm[0]] = inv_hg + (E[cm[0]] / x.rho + eT + Scpf + fT * Sdcp) * icp;
            E[cm[1]] = -1.0;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// linear algebra
// ---------------------------------------------------------------------------
// The entry an operand table names: a byte offset (n <= 64) or a number.
template <int VPL>
__device__ __forceinline__ double entry(const double *E, uint32_t o)
{
    return VPL == 1 ? *(const double *)((const char *)E + o) : E[o];
}

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
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %0, -%1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(z) : "v"(a), "n"(K));
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

// The factors between the factorisation and the solves.  Several cells per
// wave: each lane's row in registers, L and U apart with zeros elsewhere (16
// lanes; the column sweep is then one multiply-add with a row broadcast) or in
// one array (32 lanes: two arrays would not leave registers for the reaction
// pass).  One cell per wave: in the entries in LDS.
template <int VPL, int G>
struct Factors {};
template <>
struct Factors<1, 16> {
    double l[16], u[16], dinv;
};
template <>
struct Factors<1, 32> {
    double a[32], dinv;
};

// z -= a zk on the lanes above (below) K; the mask goes straight to the
// execution mask, one scalar instruction, where a select costs three vector
// ones.  `all` is the mask to go back to.  The scalar operand comes from
// readlane: two wait states until a vector instruction may read it.
template <int K>
__device__ __forceinline__ void fma_above(double &z, double a, double zk, uint64_t all)
{
    asm volatile("s_lshl_b64 exec, -2, %3\n\ts_nop 1\n\tv_fma_f64 %0, -%1, %2, %0\n\ts_mov_b64 exec, %4"
                 : "+v"(z)
                 : "v"(a), "s"(zk), "n"(K), "s"(all)
                 : "scc");
}
template <int K>
__device__ __forceinline__ void fma_below(double &z, double a, double zk, uint64_t all)
{
    asm volatile("s_bfm_b64 exec, %3, 0\n\ts_nop 1\n\tv_fma_f64 %0, -%1, %2, %0\n\ts_mov_b64 exec, %4"
                 : "+v"(z)
                 : "v"(a), "s"(zk), "n"(K), "s"(all));
}
// the same with the lane in a scalar register
__device__ __forceinline__ void fma_above(double &z, double a, double zk, int k, uint64_t all)
{
    asm volatile("s_lshl_b64 exec, -2, %3\n\ts_nop 1\n\tv_fma_f64 %0, -%1, %2, %0\n\ts_mov_b64 exec, %4"
                 : "+v"(z)
                 : "v"(a), "s"(zk), "s"(k), "s"(all)
                 : "scc");
}
__device__ __forceinline__ void fma_below(double &z, double a, double zk, int k, uint64_t all)
{
    asm volatile("s_bfm_b64 exec, %3, 0\n\ts_nop 1\n\tv_fma_f64 %0, -%1, %2, %0\n\ts_mov_b64 exec, %4"
                 : "+v"(z)
                 : "v"(a), "s"(zk), "s"(k), "s"(all));
}
__device__ __forceinline__ uint64_t exec_mask()
{
    uint64_t m;
    asm volatile("s_mov_b64 %0, exec" : "=s"(m));
    return m;
}

// ---- several cells per wave: the factorisation in registers, row per lane --
// n <= G rows, so the rows of a whole system fit one group's registers (2 G
// of them); every pivot row is broadcast inside the group.  Padding rows and
// columns hold zeros; pivots at or beyond n are skipped.
template <int G>
__device__ __forceinline__ void lu_group(const DevSparse &sp, const double *E, int lane, Factors<1, G> &f)
{
    const int n = sp.n;
    double a[G];
    const uint32_t *ix = (const uint32_t *)(sp.row + G * lane);
#pragma unroll
    for (int c = 0; c < G; c += 2) {
        const uint32_t w = ix[c / 2];
        a[c] = entry<1>(E, w & 0xffff);
        a[c + 1] = entry<1>(E, w >> 16);
    }
    f.dinv = 0.0;
    unrolled<G>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = K;
        if (k < n) {
            const double akk = bcast<G, k>(a[k]);
            if (lane == k) f.dinv = 1.0 / akk;
            const double l = lane > k ? a[k] / akk : 0.0;
            if (lane > k) a[k] = l;
#pragma unroll
            for (int j = k + 1; j < G; ++j) {
                if constexpr (G == 16)
                    fmac_row<k>(a[j], l);
                else
                    a[j] = fma(-l, bcast<G, k>(a[j]), a[j]);
            }
        }
    });
    // U to a unit diagonal
#pragma unroll
    for (int c = 0; c < G; ++c) {
        if constexpr (G == 16) {
            f.l[c] = lane > c ? a[c] : 0.0;
            f.u[c] = lane < c ? a[c] * f.dinv : 0.0;
        } else {
            f.a[c] = lane < c ? a[c] * f.dinv : a[c];
        }
    }
}

template <int G>
__device__ __forceinline__ void sweeps_group(const DevSparse &sp, const Factors<1, G> &f, int lane, double &z)
{
    const int n = sp.n;
    unrolled<G - 1>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = K;
        if (k % 4 != 0 || k < n) {
            if constexpr (G == 16)
                fmac_row<k>(z, f.l[k]);
            else
                z = fma(lane > k ? -f.a[k] : 0.0, bcast<G, k>(z), z);
        }
    });
    z *= f.dinv;
    unrolled<G - 1>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = G - 1 - K;
        if (k < n) {
            if constexpr (G == 16)
                fmac_row<k>(z, f.u[k]);
            else
                z = fma(lane < k ? -f.a[k] : 0.0, bcast<G, k>(z), z);
        }
    });
}

// ---- one cell per wave: levels, dense Schur update, register tail -----------
__device__ __forceinline__ int lo16(uint64_t x) { return (int)(x & 0xffff); }
__device__ __forceinline__ int mid16(uint64_t x) { return (int)((x >> 16) & 0xffff); }
__device__ __forceinline__ int hi16(uint64_t x) { return (int)((x >> 32) & 0xffff); }

// The first four groups of 64 items of a phase, loaded one level ahead, so
// their memory latency overlaps the level before; groups past the phase's end
// are skipped by a uniform branch.
template <class I>
struct Items {
    I it[4];
    int q0, q1;
};
template <class I>
__device__ __forceinline__ Items<I> items(const I *list, int q0, int q1, int lane)
{
    Items<I> p;
    p.q0 = q0;
    p.q1 = q1;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int q = q0 + u * WAVE + lane;
        p.it[u] = q < q1 ? list[q] : (I)0;
    }
    return p;
}

// l_ik = a_ik / a_kk (e_ik | e_kk << 16)
__device__ __forceinline__ void lu_scale_items(double *E, const Items<uint32_t> &p, int lane)
{
    double a[4], d[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (p.q0 + u * WAVE >= p.q1) break;
        a[u] = E[p.it[u] & 0xffff];
        d[u] = E[p.it[u] >> 16];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (p.q0 + u * WAVE >= p.q1) break;
        if (p.q0 + u * WAVE + lane < p.q1) E[p.it[u] & 0xffff] = a[u] / d[u];
    }
}

// a_ij -= l_ik u_kj (e_ij | e_ik << 16 | e_kj << 32); items of one phase may
// share a target: LDS additions
__device__ __forceinline__ void lu_update_items(double *E, const Items<uint64_t> &p, int lane)
{
    double a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (p.q0 + u * WAVE >= p.q1) break;
        a[u] = E[mid16(p.it[u])];
        b[u] = E[hi16(p.it[u])];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (p.q0 + u * WAVE >= p.q1) break;
        if (p.q0 + u * WAVE + lane < p.q1) atomicAdd(&E[lo16(p.it[u])], -a[u] * b[u]);
    }
}

// The pivots before the dense block, level by level: their L entries, then
// their updates of entries outside the block (the block's own updates are
// left to the dense product).
__device__ __forceinline__ void lu_levels(const DevSparse &sp, double *E, int lane)
{
    if (sp.nl == 0) return;
    Items<uint32_t> pb = items(sp.hb, 0, sp.hb_lvl[1], lane);
    Items<uint64_t> pc = items(sp.hc, 0, sp.hc_lvl[1], lane);
#pragma unroll 1
    for (int l = 0; l < sp.nl; ++l) {
        const int b1 = sp.hb_lvl[l + 1], c1 = sp.hc_lvl[l + 1];
        lu_scale_items(E, pb, lane);
#pragma unroll 1
        for (int q = pb.q0 + 4 * WAVE; q < b1; q += 4 * WAVE) lu_scale_items(E, items(sp.hb, q, b1, lane), lane);
        pb = items(sp.hb, b1, sp.hb_lvl[l + 2], lane);
        __syncthreads();
        const int c0 = pc.q0;
        if (c1 > c0) {
            lu_update_items(E, pc, lane);
#pragma unroll 1
            for (int q = c0 + 4 * WAVE; q < c1; q += 4 * WAVE) lu_update_items(E, items(sp.hc, q, c1, lane), lane);
            __syncthreads();
        }
        pc = items(sp.hc, c1, sp.hc_lvl[l + 2], lane);
    }
}

typedef double d4 __attribute__((ext_vector_type(4)));

// acc -= A B on one 16 x 16 tile with four pivots: lane l gives A[l % 16][l / 16]
// and B[l / 16][l % 16] and holds rows 4 r + l / 16 of column l % 16 (the
// last argument negates A)
__device__ __forceinline__ d4 tile_sub(double a, double b, d4 acc)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 1);
}

// Schur update of the dense block [t0, n) of up to 32 positions, A22 -= L21
// U12, on the matrix cores: 2 x 2 tiles, pivots in steps of four, operands
// gathered from the L+U entries through the tables (absent entries read the
// zero slot).  Entry (i, j) of the block is the column's end minus n - i.
// What this replaces: 6,160 scheduled multiply-adds (53 species) read their
// indices from L2 in 33 dependent rounds and met in LDS additions.
__device__ __forceinline__ void lu_schur(const DevSparse &sp, double *E, int lane, const uint2 (&g0)[8])
{
    const int n = sp.n, t0 = sp.dense0, steps = (t0 + 3) / 4;
    if (steps == 0) return;
    const int c = lane & 15, r0 = lane >> 4;
    int base[2];
    d4 acc[2][2];
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
        const int j = min(t0 + 16 * tj + c, n - 1);
        base[tj] = sp.cstart[j + 1] - n + t0 + r0;  // entry (t0 + r0, j)
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[ti][tj][r] = E[base[tj] + 16 * ti + 4 * r];
    }
    const uint2 *g = (const uint2 *)sp.ga + lane;
#pragma unroll 1
    for (int s0 = 0; s0 < steps; s0 += 8) {
        uint2 gi[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s0 == 0)
                gi[s] = g0[s];
            else if (s0 + s < steps)
                gi[s] = g[(s0 + s) * WAVE];
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s0 + s >= steps) break;
            const double a0 = entry<1>(E, gi[s].x & 0xffff), a1 = entry<1>(E, gi[s].x >> 16);
            const double b0 = entry<1>(E, gi[s].y & 0xffff), b1 = entry<1>(E, gi[s].y >> 16);
            acc[0][0] = tile_sub(a0, b0, acc[0][0]);
            acc[0][1] = tile_sub(a0, b1, acc[0][1]);
            acc[1][0] = tile_sub(a1, b0, acc[1][0]);
            acc[1][1] = tile_sub(a1, b1, acc[1][1]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + 16 * tj + c < n && t0 + 16 * ti + 4 * r + r0 < n) E[base[tj] + 16 * ti + 4 * r] = acc[ti][tj][r];
    __syncthreads();
}

// The same for a block of any width: A22 -= L21 U12 over the block [t0, n)
// with the pivots [k0, k1), operands A(tile, step) and B(tile, step) through
// functors; 16 steps of four pivots at a time, one column of tiles at a time.
template <class FA, class FB>
__device__ __forceinline__ void lu_schur_wide(const DevSparse &sp, double *E, int lane, int t0, int steps, FA fa,
                                              FB fb)
{
    const int n = sp.n, tiles = (n - t0 + 15) / 16;
    const int c = lane & 15, r0 = lane >> 4;
#pragma unroll 1
    for (int s0 = 0; s0 < steps; s0 += 16) {
#pragma unroll 1
        for (int tj = 0; tj < tiles; ++tj) {
            const int j = t0 + 16 * tj + c;
            const int base = sp.cstart[min(j, n - 1) + 1] - n + t0 + r0;
            double b[16];
            fb(tj, s0, b);
#pragma unroll 1
            for (int ti = 0; ti < tiles; ++ti) {
                double a[16];
                fa(ti, s0, a);
                double *e = E + base + 16 * ti;
                const int i = t0 + 16 * ti + r0;
                d4 acc;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = i + 4 * r < n ? e[4 * r] : 0.0;
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    if (s0 + s >= steps) break;
                    acc = tile_sub(a[s], b[s], acc);
                }
                if (j < n) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (i + 4 * r < n) e[4 * r] = acc[r];
                }
            }
        }
        __syncthreads();
    }
}

// Row broadcasts of one pivot row are read four columns at a time, so that
// the wait a vector instruction needs after a readlane is spent reading the
// next ones.
template <int W, int K>
__device__ __forceinline__ void apply_pivot(double (&a)[W], double l)
{
    constexpr int J0 = K + 1;
#pragma unroll
    for (int j = J0; j < W; j += 4) {
        double u[4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (j + d < W) u[d] = rdlane(a[j + d], K);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (j + d < W) a[j + d] = fma(-l, u[d], a[j + d]);
    }
}

// The dense trailing block [t0, n) (w = n - t0 <= W positions, full L+U
// pattern) in registers: lane r holds row t0 + r, columns t0..n-1.  The
// rows of the block are the last w entries of each of its columns (entries
// are numbered column by column), so no index table is read.  Right-looking
// elimination: per pivot k, the pivot row is broadcast entry by entry and
// every row below applies it; rows at or above the pivot multiply by zero.
// Padding (rows and columns from w to W) holds zeros and takes part
// unconditionally: the loops have fixed trip counts, the array stays in
// registers.  L is stored scaled (l_ik = a_ik / a_kk), U and the diagonal
// as computed.
template <int W>
__device__ __forceinline__ void lu_tail(const DevSparse &sp, double *E, int t0, int lane)
{
    const int n = sp.n, w = n - t0;
    const bool row = lane < w;
    const int back = n - t0 - lane;  // entry (t0 + lane, c) = cstart[c + 1] - back
    const int cend = row ? sp.cstart[t0 + lane + 1] : 0;  // lane j: end of column t0 + j
    double a[W];
    // loads at a clamped index and selects (no lane mask per column is kept
    // alive until the stores)
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const int e = __builtin_amdgcn_readlane(cend, j) - back;
        const bool ok = j < w && row;
        const double x = E[ok ? e : 0];
        a[j] = ok ? x : 0.0;
    }
    unrolled<W - 1>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = K;
        const double akk = rdlane(a[k], k);
        const bool sub = row && lane > k;  // a row below the pivot
        const double l = sub ? a[k] / akk : 0.0;
        a[k] = sub ? l : a[k];
        apply_pivot<W, k>(a, l);
    });
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const int e = __builtin_amdgcn_readlane(cend, j) - back;
        if (j < w && row) E[e] = a[j];
    }
}

// A panel of P <= 16 pivots [t, t + P) of a dense trailing block wider than
// the 64 rows of the register tail: the panel's columns for all rows of the
// block in registers (two rows per lane), then the panel's rows of U column
// per lane, then the rest of the block on the matrix cores.
__device__ __forceinline__ void lu_panel(const DevSparse &sp, double *E, int t, int P, int lane)
{
    constexpr int W = 16;
    const int n = sp.n, w = n - t;
    double a[2][W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const int cend = sp.cstart[min(t + k, n - 1) + 1];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int i = lane + 64 * s;
            a[s][k] = k < P && i < w ? E[cend - w + i] : 0.0;
        }
    }
    unrolled<W>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = K;
        if (k < P) {
            const double akk = rdlane(a[0][k], k);
            const double l0 = lane > k ? a[0][k] / akk : 0.0, l1 = a[1][k] / akk;
            if (lane > k) a[0][k] = l0;
            a[1][k] = l1;
#pragma unroll
            for (int j = k + 1; j < W; ++j) {
                const double u = rdlane(a[0][j], k);
                a[0][j] = fma(-l0, u, a[0][j]);
                a[1][j] = fma(-l1, u, a[1][j]);
            }
        }
    });
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const int cend = sp.cstart[min(t + k, n - 1) + 1];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int i = lane + 64 * s;
            if (k < P && i < w) E[cend - w + i] = a[s][k];
        }
    }
    // rows t .. t + P - 1 of the columns beyond the panel: U12 = L11^-1 A12,
    // L11 broadcast from the lanes that hold it
#pragma unroll 1
    for (int j0 = t + P; j0 < n; j0 += WAVE) {
        const int j = j0 + lane;
        double *e = E + sp.cstart[min(j, n - 1) + 1] - w;  // entry (t, j)
        double u[W];
#pragma unroll
        for (int k = 0; k < W; ++k) u[k] = k < P && j < n ? e[k] : 0.0;
        unrolled<W>([&](auto K) __attribute__((always_inline)) {
            constexpr int k = K;
            if (k < P) {
#pragma unroll
                for (int m = k + 1; m < W; ++m) u[m] = fma(-rdlane(a[0][k], m), u[k], u[m]);
            }
        });
#pragma unroll
        for (int k = 0; k < W; ++k)
            if (k < P && j < n) e[k] = u[k];
    }
    __syncthreads();
    const int t1 = t + P;
    const int c = lane & 15, kk = lane >> 4;
    lu_schur_wide(
        sp, E, lane, t1, (P + 3) / 4,
        [&](int ti, int, double (&v)[16]) {
            const int i = t1 + 16 * ti + c;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 4 * s + kk;
                v[s] = k < P && i < n ? E[sp.cstart[t + k + 1] - n + i] : 0.0;
            }
        },
        [&](int tj, int, double (&v)[16]) {
            const int j = t1 + 16 * tj + c;
            const double *e = E + sp.cstart[min(j, n - 1) + 1] - w;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 4 * s + kk;
                v[s] = k < P && j < n ? e[k] : 0.0;
            }
        });
}

// Numeric LU of the formed matrix in E, then dinv = 1/u_kk and the rows of U
// scaled to a unit diagonal.
template <int VPL, int G>
__device__ void lu_v(const DevSparse &sp, double *lds, int lane, Factors<VPL, G> &fac)
{
    double *E = lds + sp.E;
    if constexpr (G < WAVE) {
        lu_group<G>(sp, E, lane, fac);
        __syncthreads();
        return;
    } else {
        double *DINV = lds + sp.DINV;
        if constexpr (VPL == 1) {
            // the Schur operands' indices, on their way during the levels
            uint2 g0[8];
            const uint2 *g = (const uint2 *)sp.ga + lane;
#pragma unroll
            for (int s = 0; s < 8; ++s) g0[s] = 4 * s < sp.dense0 ? g[s * WAVE] : make_uint2(0, 0);
            lu_levels(sp, E, lane);
            lu_schur(sp, E, lane, g0);
            lu_tail<sc::SPARSE_TAIL_MAX>(sp, E, sp.dense0, lane);
        } else {
            lu_levels(sp, E, lane);
            const int t0 = sp.dense0, steps = (t0 + 3) / 4, pad = (steps + 15) / 16 * 16;
            auto load = [&](const uint16_t *tab, int tile, int s0, double (&v)[16]) {
                const uint32_t *q = (const uint32_t *)(tab + ((size_t)tile * WAVE + lane) * pad + s0);
#pragma unroll
                for (int s = 0; s < 16; s += 2) {
                    const uint32_t w = q[s / 2];
                    v[s] = E[w & 0xffff];
                    v[s + 1] = E[w >> 16];
                }
            };
            lu_schur_wide(
                sp, E, lane, t0, steps, [&](int ti, int s0, double (&v)[16]) { load(sp.ga, ti, s0, v); },
                [&](int tj, int s0, double (&v)[16]) { load(sp.gb, tj, s0, v); });
            int t = t0;
#pragma unroll 1
            while (sp.n - t > sc::SPARSE_TAIL_MAX_WIDE) {
                const int P = min(16, sp.n - t - sc::SPARSE_TAIL_MAX_WIDE);
                lu_panel(sp, E, t, P, lane);
                t += P;
            }
            lu_tail<sc::SPARSE_TAIL_MAX_WIDE>(sp, E, t, lane);
        }
        // the scaling's items, loaded while the diagonal is inverted
        constexpr int UI = VPL == 1 ? 8 : 16;
        uint32_t it[UI];
#pragma unroll
        for (int u = 0; u < UI; ++u) it[u] = u * WAVE + lane < sp.n_u ? sp.lu_u[u * WAVE + lane] : 0u;
        __syncthreads();
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const int k = lane + WAVE * v;
            if (k < sp.n) DINV[k] = 1.0 / E[sp.diag[k]];
        }
        __syncthreads();
#pragma unroll 1
        for (int q = 0; q < sp.n_u; q += UI * WAVE) {
            if (q > 0) {
#pragma unroll
                for (int u = 0; u < UI; ++u)
                    it[u] = q + u * WAVE + lane < sp.n_u ? sp.lu_u[q + u * WAVE + lane] : 0u;
            }
            double x[UI];
#pragma unroll
            for (int u = 0; u < UI; ++u) x[u] = E[it[u] & 0xffff] * DINV[it[u] >> 16];
#pragma unroll
            for (int u = 0; u < UI; ++u)
                if (q + u * WAVE + lane < sp.n_u) E[it[u] & 0xffff] = x[u];
        }
        __syncthreads();
    }
}

// Solve M x = b with the factors (b, x: VPL components per lane; a lane holds
// the same position as component and as row).  The vector is swept in
// registers, one column of L (then of the unit-diagonal U) at a time: the
// pivot value is broadcast with readlane and the lanes behind it apply their
// entry of the column.
//
// The chain of 2 n broadcasts and multiply-adds bounds a solve, so nothing
// else is on it: each lane's entries come eight columns at a time from LDS
// through a table of its row, ahead of their use, and the lanes are masked by
// the execution mask.  With each entry's place computed from the column's
// mask at its turn a column took 189 cycles of a lone wave (53 species).
__device__ __forceinline__ void sweeps(const DevSparse &sp, const double *E, const double *DINV, int lane,
                                       double (&z)[1])
{
    const int n = sp.n;
    const uint64_t all = exec_mask();
    uint4 ix[8];  // byte offsets of the row's entries, 64 columns
    const uint4 *t = (const uint4 *)(sp.row + 64 * lane);
#pragma unroll
    for (int b = 0; b < 8; ++b) ix[b] = t[b];
    const double dinv = lane < n ? DINV[lane] : 0.0;
    auto load = [&](const uint4 &w, double (&v)[8]) {
        v[0] = entry<1>(E, w.x & 0xffff);
        v[1] = entry<1>(E, w.x >> 16);
        v[2] = entry<1>(E, w.y & 0xffff);
        v[3] = entry<1>(E, w.y >> 16);
        v[4] = entry<1>(E, w.z & 0xffff);
        v[5] = entry<1>(E, w.z >> 16);
        v[6] = entry<1>(E, w.w & 0xffff);
        v[7] = entry<1>(E, w.w >> 16);
    };
    double cur[8], nxt[8];
    load(ix[0], cur);
    unrolled<8>([&](auto B) __attribute__((always_inline)) {
        constexpr int b = B;
        if (8 * b < n) {
            if constexpr (b < 7) load(ix[b + 1], nxt);
            unrolled<8>([&](auto D) __attribute__((always_inline)) {
                constexpr int k = 8 * b + D;
                if constexpr (k < 63) fma_above<k>(z[0], cur[D], rdlane(z[0], k), all);
            });
#pragma unroll
            for (int d = 0; d < 8; ++d) cur[d] = nxt[d];
        }
    });
    z[0] *= dinv;
    unrolled<8>([&](auto B) __attribute__((always_inline)) {
        constexpr int b = 7 - B;
        if (8 * b < n) {
            // the block a column at n - 1 lies in is the first one read
            if (8 * b + 8 >= n) load(ix[b], cur);
            if constexpr (b > 0) load(ix[b - 1], nxt);
            unrolled<8>([&](auto D) __attribute__((always_inline)) {
                constexpr int k = 8 * b + 7 - D;
                if constexpr (k > 0) fma_below<k>(z[0], cur[7 - D], rdlane(z[0], k), all);
            });
#pragma unroll
            for (int d = 0; d < 8; ++d) cur[d] = nxt[d];
        }
    });
}

// Two rows per lane: columns in blocks of eight, their table entries loaded
// two blocks and their values one block ahead.
__device__ __forceinline__ void sweeps(const DevSparse &sp, const double *E, const double *DINV, int lane,
                                       double (&z)[2])
{
    const int n = sp.n, nb = (n + 7) / 8;
    const uint64_t all = exec_mask();
    const uint4 *t0 = (const uint4 *)(sp.row + 128 * lane), *t1 = t0 + 64 * 16;
    struct Blk {
        double a[2][8];
    };
    struct Ix {
        uint4 w[2];
    };
    auto index = [&](int b) { return Ix{{t0[b], t1[b]}}; };
    auto load = [&](const Ix &x) {
        Blk v;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t w[4] = {x.w[s].x, x.w[s].y, x.w[s].z, x.w[s].w};
#pragma unroll
            for (int d = 0; d < 8; ++d) v.a[s][d] = E[d % 2 ? w[d / 2] >> 16 : w[d / 2] & 0xffff];
        }
        return v;
    };
    const double d0 = DINV[lane], d1 = lane + 64 < n ? DINV[lane + 64] : 0.0;
    // blocks 0 .. nb - 1 forward, then nb - 1 .. 0 backward, one pipeline
    auto blk = [&](int q) { return min(q < nb ? q : 2 * nb - 1 - q, nb - 1); };
    Ix ix = index(blk(1));
    Blk nxt = load(index(0));
#pragma unroll 1
    for (int q = 0; q < 2 * nb; ++q) {
        const Blk cur = nxt;
        nxt = load(ix);
        ix = index(max(blk(q + 2), 0));
        const int k0 = __builtin_amdgcn_readfirstlane(8 * blk(q));
        if (q == nb) {
            z[0] *= d0;
            z[1] *= d1;
        }
        if (q < nb) {
            if (k0 < 64) {
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const double zk = rdlane(z[0], k0 + d);
                    z[1] = fma(-cur.a[1][d], zk, z[1]);
                    fma_above(z[0], cur.a[0][d], zk, k0 + d, all);
                }
            } else {
#pragma unroll
                for (int d = 0; d < 8; ++d)
                    fma_above(z[1], cur.a[1][d], rdlane(z[1], k0 + d - 64), k0 + d - 64, all);
            }
        } else if (k0 >= 64) {
#pragma unroll
            for (int d = 7; d >= 0; --d) {
                const double zk = rdlane(z[1], k0 + d - 64);
                z[0] = fma(-cur.a[0][d], zk, z[0]);
                fma_below(z[1], cur.a[1][d], zk, k0 + d - 64, all);
            }
        } else {
#pragma unroll
            for (int d = 7; d >= 0; --d) fma_below(z[0], cur.a[0][d], rdlane(z[0], k0 + d), k0 + d, all);
        }
    }
}

template <int VPL, int G>
__device__ void solve_v(const DevMech &m, const DevSparse &sp, double *lds, const Factors<VPL, G> &fac,
                        const double (&b)[VPL], int lane, double (&x)[VPL])
{
    const int N = m.N;
    // scaled unknowns z_k = x_k / W_k; the sigma row's right-hand side is zero
    double z[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        z[v] = c < N ? b[v] * m.invW()[c] : c == N ? b[v] : 0.0;
    }
    if constexpr (G < WAVE)
        sweeps_group<G>(sp, fac, lane, z[0]);
    else
        sweeps(sp, lds + sp.E, lds + sp.DINV, lane, z);
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        x[v] = c < N ? z[v] * m.W()[c] : c == N ? z[v] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// one Rosenbrock attempt and the integration of a cell
// ---------------------------------------------------------------------------
template <int VPL, int G = WAVE>
__device__ void ros_attempt_v(const DevMech &m, const DevSparse &sp, const Opts &o, double *lds,
                              const double (&y)[VPL], double p, const double *dlnA, int lane, double hc, double *err,
                              double (&ynew)[VPL])
{
    const int n = m.N + 1;
    double *U = lds + sp.U;
    const int NV = sp.NV;
    double f0[VPL], flast[VPL];
    jac_v<VPL, G>(m, sp, lds, y, p, dlnA, lane, 1.0 / (GAM * hc), f0);
    Factors<VPL, G> fac;
    lu_v<VPL, G>(sp, lds, lane, fac);
    const double ih = 1.0 / hc;
#pragma unroll
    for (int v = 0; v < VPL; ++v) flast[v] = f0[v];
#pragma unroll 1
    for (int i = 0; i < NS; ++i) {
        double fi[VPL];
        const int reuse = TREUSE[i];
        if (reuse == 0) {
#pragma unroll
            for (int v = 0; v < VPL; ++v) fi[v] = f0[v];
        } else if (reuse > 0) {
#pragma unroll
            for (int v = 0; v < VPL; ++v) fi[v] = flast[v];
        } else {
            double ys[VPL];
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                ys[v] = y[v];
                for (int j = 0; j < i; ++j) ys[v] += TA[i][j] * U[j * NV + lane + G * v];
            }
            rhs_v<VPL, G>(m, sp, lds, ys, p, dlnA, lane, fi);
#pragma unroll
            for (int v = 0; v < VPL; ++v) flast[v] = fi[v];
        }
        double ui[VPL];
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            for (int j = 0; j < i; ++j) fi[v] += (TC[i][j] * ih) * U[j * NV + lane + G * v];
            if (lane + G * v >= n) fi[v] = 0.0;
        }
        solve_v<VPL, G>(m, sp, lds, fac, fi, lane, ui);
#pragma unroll
        for (int v = 0; v < VPL; ++v) U[i * NV + lane + G * v] = ui[v];
    }
    double e2[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        double yn = y[v], ev = 0.0;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const double ui = U[i * NV + lane + G * v];
            yn += TM[i] * ui;
            ev += TE[i] * ui;
        }
        ynew[v] = yn;
        e2[v] = 0.0;
        if (lane + G * v < n) {
            const double sc = o.atol + o.rtol * fmax(fabs(y[v]), fabs(yn));
            const double r = ev / sc;
            e2[v] = r * r;
        }
    }
    *err = sqrt(vsum<VPL, G>(e2) / n);
}

template <int VPL, int G = WAVE>
__device__ int advance_v(const DevMech &m, const DevSparse &sp, const Opts &o, double *lds, double (&y)[VPL],
                         double p, double dt, const double *dlnA, int lane, Ctl &s)
{
#pragma unroll 1
    while (true) {
        double hc;
        bool last;
        const int st = ctl_begin(s, o, dt, hc, last);
        if (st != SC_CELL_OK) return st;
        double err, ynew[VPL];
        ros_attempt_v<VPL, G>(m, sp, o, lds, y, p, dlnA, lane, hc, &err, ynew);
        const int r = ctl_end(s, o, err, hc, last, dt);
        if (r < 0) return -r;
        if (r == 1) {
#pragma unroll
            for (int v = 0; v < VPL; ++v) y[v] = ynew[v];
            if (last) return SC_CELL_OK;
        }
    }
}

template <int VPL, int G = WAVE>
__device__ __forceinline__ bool bad_input_v(const DevMech &m, const double (&y)[VPL], double p, double dt, int lane)
{
    bool bad = false;
#pragma unroll
    for (int v = 0; v < VPL; ++v) bad = bad || (lane + G * v <= m.N && !isfinite(y[v]));
    const double T = comp_T<VPL, G>(m, y);
    return gany<G>(bad) || !(T > 0.0) || !isfinite(T) || !(p > 0.0) || !isfinite(p) || !(dt >= 0.0) ||
           !isfinite(dt);
}

template <int VPL, int G = WAVE>
__device__ __forceinline__ void integrate_cell_v(const DevMech &m, const DevSparse &sp, const Opts &o, double *lds, int64_t c,
                                 int lane, const double *T0, const double *P, const double *Y0, int64_t ld,
                                 const double *DT, const double *dlnA, double *h_io, double *T1, double *Y1,
                                 int32_t *status, int32_t *nacc_out, int32_t *nrej_out, const int32_t *ref)
{
    // a cell mapped onto another cell's result is left to the mapping pass
    if (ref && ref[c] != c) return;
    double y[VPL];
    load_state_v<VPL, G>(m, sp, T0, Y0, ld, c, lane, y);
    const double p = P[c], dt = DT[c];
    int st = SC_CELL_OK;
    Ctl s = ctl_init(initial_step(h_io, c, dt), dt);
    if (bad_input_v<VPL, G>(m, y, p, dt, lane)) {
        st = SC_CELL_BAD_INPUT;
    } else if (dt > 0.0) {
        st = advance_v<VPL, G>(m, sp, o, lds, y, p, dt, dlnA, lane, s);
    }
    store_state_v<VPL, G>(m, sp, T1, Y1, ld, c, lane, y);
    if (lane == 0) {
        status[c] = st;
        if (nacc_out) nacc_out[c] = s.nacc;
        if (nrej_out) nrej_out[c] = s.nrej;
        if (h_io && st == SC_CELL_OK && dt > 0.0) h_io[c] = s.hnext;
    }
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// One-wave mechanisms (VPL = 1) run two waves per SIMD: their LDS allows it
// (under 20 KB per cell up to 53 species) and the second wave hides the
// first's LDS, memory and broadcast latencies.  The register cap this
// implies spills about a hundred registers to scratch, outside the inner
// loops; measured on the 53-species batch it is still 1.6x faster than one
// wave per SIMD.
#define SP_OCC __attribute__((amdgpu_waves_per_eu(VPL == 1 ? 2 : 1, VPL == 1 ? 2 : 1)))
// CPW cells per wave: each cell takes G = 64 / CPW lanes and its own LDS
// region (sp.size doubles); lane = threadIdx.x % G, group = threadIdx.x / G.
#define SP_GEOMETRY                                   \
    constexpr int G = WAVE / CPW;                     \
    const int lane = (int)threadIdx.x % G;            \
    const int grp = (int)threadIdx.x / G;             \
    double *ldsg = lds + (size_t)grp * sp.size;

template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) SP_OCC k_integrate_sp(DevMech mk, DevSparse spk, Opts o, int64_t n,
                                                       const double *T0, const double *P, const double *Y0,
                                                       int64_t ld, const double *DT, const double *dlnA,
                                                       double *h_io, double *T1, double *Y1, int32_t *status,
                                                       int32_t *nacc, int32_t *nrej, const int32_t *ref)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    SP_GEOMETRY
    const int64_t c = (int64_t)blockIdx.x * CPW + grp;
    if (c >= n) return;
    integrate_cell_v<VPL, G>(m, sp, o, ldsg, c, lane, T0, P, Y0, ld, DT, dlnA, h_io, T1, Y1, status, nacc, nrej,
                             ref);
}

// Each pull takes tile * CPW queue positions; the wave's groups take them
// CPW at a time (a group whose position is past the end idles).
template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) SP_OCC k_integrate_sp_persistent(DevMech mk, DevSparse spk, Opts o, int64_t n,
                                                                  const double *T0, const double *P,
                                                                  const double *Y0, int64_t ld, const double *DT,
                                                                  const double *dlnA, double *h_io, double *T1,
                                                                  double *Y1, int32_t *status, int32_t *nacc,
                                                                  int32_t *nrej, unsigned long long *queue,
                                                                  const int32_t *perm, int tile, const int32_t *ref)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    SP_GEOMETRY
#pragma unroll 1
    while (true) {
        unsigned long long base = 0;
        if (threadIdx.x == 0) base = atomicAdd(queue, (unsigned long long)tile * CPW);
        base = __shfl(base, 0, WAVE);
        if (base >= (unsigned long long)n) break;
        const int64_t end = min((int64_t)base + (int64_t)tile * CPW, n);
#pragma unroll 1
        for (int64_t i = (int64_t)base; i < end; i += CPW) {
            const int64_t q = i + grp;
            if (q < end) {
                const int64_t c = perm ? (int64_t)perm[q] : q;
                integrate_cell_v<VPL, G>(m, sp, o, ldsg, c, lane, T0, P, Y0, ld, DT, dlnA, h_io, T1, Y1, status,
                                         nacc, nrej, ref);
            }
        }
    }
}

template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) SP_OCC k_integrate_sp_static(DevMech mk, DevSparse spk, Opts o, int64_t n,
                                                              const double *T0, const double *P, const double *Y0,
                                                              int64_t ld, const double *DT, const double *dlnA,
                                                              double *h_io, double *T1, double *Y1,
                                                              int32_t *status, int32_t *nacc, int32_t *nrej,
                                                              int64_t group, const int32_t *ref)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    SP_GEOMETRY
    const int64_t c0 = (int64_t)blockIdx.x * group;
    const int64_t c1 = min(c0 + group, n);
#pragma unroll 1
    for (int64_t c = c0 + grp; c < c1; c += CPW)
        integrate_cell_v<VPL, G>(m, sp, o, ldsg, c, lane, T0, P, Y0, ld, DT, dlnA, h_io, T1, Y1, status, nacc,
                                 nrej, ref);
}

template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) k_rhs_sp(DevMech mk, DevSparse spk, int64_t n, const double *T,
                                                 const double *P, const double *Y, int64_t ld, const double *dlnA,
                                                 double *fT, double *fY)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    SP_GEOMETRY
    const int64_t c = (int64_t)blockIdx.x * CPW + grp;
    if (c >= n) return;
    double y[VPL], f[VPL];
    load_state_v<VPL, G>(m, sp, T, Y, ld, c, lane, y);
    rhs_v<VPL, G>(m, sp, ldsg, y, P[c], dlnA, lane, f);
    store_state_v<VPL, G>(m, sp, fT, fY, ld, c, lane, f);
}

// The Jacobian J (dense output, [c][i][j] over (Y, T)) recovered from the
// bordered matrix formed with 1/hg = 0 (the -J of the scaled system with the
// sigma border): eliminating sigma, M'_ij = A_ij + A_i,sigma A_sigma,j, and
// undoing the scaling, J_ij = -(W_i / W_j) M'_ij (species i, j), J_iT =
// -W_i A_iT, J_Tj = -A_Tj / W_j, J_TT = -A_TT.
template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) k_jac_sp(DevMech mk, DevSparse spk, int64_t n, const double *T,
                                                 const double *P, const double *Y, int64_t ld, const double *dlnA,
                                                 double *J)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    SP_GEOMETRY
    const int64_t c = (int64_t)blockIdx.x * CPW + grp;
    if (c >= n) return;
    double y[VPL], f[VPL];
    load_state_v<VPL, G>(m, sp, T, Y, ld, c, lane, y);
    jac_v<VPL, G>(m, sp, ldsg, y, P[c], dlnA, lane, 0.0, f);
    const double *E = ldsg + sp.E;
    const int N = m.N, nn = N + 1, ns = sp.n;
    const int pS = ns - 1;
    auto A = [&](int pi, int pj) {
        const uint16_t e = sp.emap[pi * ns + pj];
        return e == sc::NOENT ? 0.0 : E[e];
    };
#pragma unroll 1
    for (int q = lane; q < nn * nn; q += G) {
        const int i = q / nn, j = q % nn;
        const int pi = sp.pos[i], pj = sp.pos[j];
        double val;
        if (i < N && j < N) val = -(m.W()[pi] * m.invW()[pj]) * (A(pi, pj) + A(pi, pS) * A(pS, pj));
        else if (i < N) val = -m.W()[pi] * A(pi, pj);
        else if (j < N) val = -A(pi, pj) * m.invW()[pj];
        else val = -A(pi, pj);
        J[(c * nn + i) * nn + j] = val;
    }
}

template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) k_linsolve_sp(DevMech mk, DevSparse spk, int64_t n, const double *T,
                                                      const double *P, const double *Y, int64_t ld,
                                                      const double *dlnA, const double *hg, const double *b,
                                                      double *x)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    SP_GEOMETRY
    const int64_t c = (int64_t)blockIdx.x * CPW + grp;
    if (c >= n) return;
    double y[VPL], f[VPL], bb[VPL], xx[VPL];
    load_state_v<VPL, G>(m, sp, T, Y, ld, c, lane, y);
    jac_v<VPL, G>(m, sp, ldsg, y, P[c], dlnA, lane, 1.0 / hg[c], f);
    Factors<VPL, G> fac;
    lu_v<VPL, G>(sp, ldsg, lane, fac);
    const int nn = m.N + 1;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int i = lane + G * v;
        bb[v] = i < nn ? b[c * nn + sp.perm[i]] : 0.0;
    }
    solve_v<VPL, G>(m, sp, ldsg, fac, bb, lane, xx);
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int i = lane + G * v;
        if (i < nn) x[c * nn + sp.perm[i]] = xx[v];
    }
}

// ---------------------------------------------------------------------------
// launchers (host)
// ---------------------------------------------------------------------------
#define SP_KERNEL(k) k<VPLV, CVV, CPWV, TBV>
#define SP_CASE(vplv, cpwv, ...)                                                                 \
    if (vpl == (vplv) && cpw == (cpwv)) {                                                        \
        constexpr int VPLV = vplv, CPWV = cpwv;                                                  \
        if (m.cv && sp.itab) { constexpr bool CVV = true, TBV = true; __VA_ARGS__; }            \
        else if (m.cv) { constexpr bool CVV = true, TBV = false; __VA_ARGS__; }                 \
        else if (sp.itab) { constexpr bool CVV = false, TBV = true; __VA_ARGS__; }              \
        else { constexpr bool CVV = false, TBV = false; __VA_ARGS__; }                          \
        return hipGetLastError();                                                                \
    }
#define SP_DISPATCH(...)                   \
    SP_CASE(1, 1, __VA_ARGS__)             \
    SP_CASE(1, 2, __VA_ARGS__)             \
    SP_CASE(1, 4, __VA_ARGS__)             \
    SP_CASE(2, 1, __VA_ARGS__)             \
    return hipErrorInvalidValue;

// LDS of one workgroup: one region of sp.size doubles per cell of the wave
static size_t sp_lds(const DevSparse &sp, int cpw) { return sizeof(double) * (size_t)sp.size * cpw; }
static unsigned sp_blocks(int64_t n, int cpw) { return (unsigned)((n + cpw - 1) / cpw); }

hipError_t launch_rhs_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                         const double *p, const double *Y, int64_t ld, const double *dlnA, double *fT, double *fY,
                         hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_rhs_sp), dim3(sp_blocks(n, cpw)), dim3(WAVE), sp_lds(sp, cpw), s, m,
                                   sp, n, T, p, Y, ld, dlnA, fT, fY))
}

hipError_t launch_jac_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                         const double *p, const double *Y, int64_t ld, const double *dlnA, double *J, hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_jac_sp), dim3(sp_blocks(n, cpw)), dim3(WAVE), sp_lds(sp, cpw), s, m,
                                   sp, n, T, p, Y, ld, dlnA, J))
}

hipError_t launch_linsolve_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                              const double *p, const double *Y, int64_t ld, const double *dlnA, const double *hg,
                              const double *b, double *x, hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_linsolve_sp), dim3(sp_blocks(n, cpw)), dim3(WAVE), sp_lds(sp, cpw),
                                   s, m, sp, n, T, p, Y, ld, dlnA, hg, b, x))
}

hipError_t launch_integrate_sp(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o, int64_t n,
                               const double *T0, const double *p, const double *Y0, int64_t ld, const double *dt,
                               const double *dlnA, double *h_io, double *T1, double *Y1, int32_t *st, int32_t *na,
                               int32_t *nr, const int32_t *ref, hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_integrate_sp), dim3(sp_blocks(n, cpw)), dim3(WAVE), sp_lds(sp, cpw),
                                   s, m, sp, o, n, T0, p, Y0, ld, dt, dlnA, h_io, T1, Y1, st, na, nr, ref))
}

hipError_t launch_integrate_sp_persistent(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o,
                                          int64_t n, const double *T0, const double *p, const double *Y0,
                                          int64_t ld, const double *dt, const double *dlnA, double *h_io,
                                          double *T1, double *Y1, int32_t *st, int32_t *na, int32_t *nr,
                                          unsigned long long *queue, const int32_t *perm, int tile, int grid,
                                          const int32_t *ref, hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_integrate_sp_persistent), dim3((unsigned)grid), dim3(WAVE),
                                   sp_lds(sp, cpw), s, m, sp, o, n, T0, p, Y0, ld, dt, dlnA, h_io, T1, Y1, st, na,
                                   nr, queue, perm, tile, ref))
}

hipError_t launch_integrate_sp_static(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o, int64_t n,
                                      const double *T0, const double *p, const double *Y0, int64_t ld,
                                      const double *dt, const double *dlnA, double *h_io, double *T1, double *Y1,
                                      int32_t *st, int32_t *na, int32_t *nr, int grid, const int32_t *ref,
                                      hipStream_t s)
{
    const int cpw = sp.cpw;
    const int64_t group = (n + grid - 1) / grid;
    const unsigned g = (unsigned)((n + group - 1) / group);
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_integrate_sp_static), dim3(g), dim3(WAVE), sp_lds(sp, cpw), s, m,
                                   sp, o, n, T0, p, Y0, ld, dt, dlnA, h_io, T1, Y1, st, na, nr, group, ref))
}

int persistent_capacity_sp(int vpl, const DevSparse &sp, int device)
{
    int per_cu = 0, cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    hipError_t e = hipErrorInvalidValue;
    const int cpw = sp.cpw;
    auto occ = [&](auto kern) { return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, WAVE, sp_lds(sp, cpw)); };
    if (vpl == 1 && cpw == 1) e = occ(k_integrate_sp_persistent<1, false, 1, false>);
    else if (vpl == 1 && cpw == 2) e = occ(k_integrate_sp_persistent<1, false, 2, false>);
    else if (vpl == 1 && cpw == 4) e = occ(k_integrate_sp_persistent<1, false, 4, false>);
    else if (vpl == 2 && cpw == 1) e = occ(k_integrate_sp_persistent<2, false, 1, false>);
    return e == hipSuccess ? per_cu * cus : 0;
}

}  // namespace scdev
