// Kernels with the sparse linear algebra (gfx950): one 64-lane wavefront per
// cell, as in the dense kernels, but the iteration matrix lives in LDS as the
// L+U entries of the bordered system the mechanism compiler built
// (sparse.cpp).  State vectors hold VPL components per lane (component
// c = lane + 64 v, species in elimination order), so mechanisms of up to 126
// species fit one wave (127 without the solves); small ones run two or four
// cells per wave.
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

#include <algorithm>
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

// Who works on a cell: one wave, or a crew of the workgroup's waves on one
// LDS region.  Every wave of a crew holds the cell's state and takes its every
// decision from the same numbers.  What splits are the passes over the
// reactions and the tiles of the factorization; the passes' sums are added in
// the order of the passes, so the results are those of one wave, bit for bit.
__device__ __forceinline__ int64_t uniform(int64_t v)
{
    return (int64_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ double uniform(double v) { return __longlong_as_double(uniform((int64_t)__double_as_longlong(v))); }

struct Crew {
    int w, rank;  // w a power of two
    int *turn;    // the pass whose sums are to be added next
    uint64_t own; // the wave's passes, where there are at most 64
    __device__ __forceinline__ void barrier() const
    {
        if (w > 1) __syncthreads();
    }
    __device__ __forceinline__ void sync() const
    {
        if (w > 1)
            __syncthreads();
        else
            lds_sync();
    }
    // before the passes; a barrier follows
    __device__ __forceinline__ void start(const DevRx &sp) const
    {
        if (rank == 0 && threadIdx.x % WAVE == 0) *turn = sp.passes - 1;
    }
    // The passes are taken from the last to the first, so that the long ones
    // (the falloff reactions', about eight times the others' time) add at the
    // end and nobody waits for them.  Those go round from the last wave on; of
    // the others, the waves with one long pass less take eight more.
    __device__ __forceinline__ bool mine(const DevRx &sp, int q) const
    {
        const int heavy = (sp.n_tb + WAVE - 1) / WAVE, i = sp.passes - 1 - q;
        if (q < heavy) return w - 1 - (q & (w - 1)) == rank;
        const int few = w - (heavy & (w - 1)), even = few == w ? sp.passes : (sp.passes - heavy - 8 * few) & -w;
        return (i < even ? i & (w - 1) : (i - max(even, 0)) % few) == rank;
    }
    __device__ __forceinline__ int first(const DevRx &sp) const { return next(sp, sp.passes); }
    // the wave's pass after q
    __device__ __forceinline__ int next(const DevRx &sp, int q) const
    {
        if (w > 1 && sp.passes <= 64) {
            const uint64_t left = q < 64 ? own & ((1ull << q) - 1) : own;
            return left ? 63 - __builtin_clzll(left) : -1;
        }
        --q;
        if (w > 1)
            while (q >= 0 && !mine(sp, q)) --q;
        return q;
    }
    __device__ __forceinline__ void join(const DevRx &sp, int waves, int wave)
    {
        w = waves, rank = wave, own = 0;
        for (int q = 0; q < min(sp.passes, 64); ++q) own |= (uint64_t)mine(sp, q) << q;
    }
    __device__ __forceinline__ void await(int q) const
    {
        if (w > 1) {
            while (__builtin_amdgcn_readfirstlane(
                       __hip_atomic_load(turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != q) {}
            lds_sync();
        }
    }
    // (a wave's LDS operations take effect in order)
    __device__ __forceinline__ void pass_on(int q) const
    {
        if (w > 1) {
            lds_sync();
            if (threadIdx.x % WAVE == 0)
                __hip_atomic_store(turn, q - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
};

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
// Mixture state from y; writes C, g/RT, h/RT (and what an unused slot of a
// reaction reads, in the temperature's place) and clears the accumulators.
template <int VPL, int G, class CR>
__device__ __forceinline__ Mix<> mixture_v(const CR &crew, const DevMech &m, const DevSparse &sp, double *lds, const double (&y)[VPL],
                                           double p, Thermo<> (&th)[VPL], int lane)
{
    constexpr int NV = G * VPL;
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
    crew.start(sp);
    if (crew.rank != 0) return x;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;  // lanes beyond the species hold zeros: unused slots need only a concentration
        double *cg = pair<NV>(lds, SPL_CG, c), *hw = pair<NV>(lds, SPL_HW, c);
        cg[0] = c < N ? x.rho * yw[v] : 1.0;
        cg[1] = th[v].hRT - th[v].sR;
        hw[0] = th[v].hRT;
        hw[1] = 0.0;
        lds[SPL_UA * NV + c] = 0.0;
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
    return sp.itab + (size_t)iv * (R + 1) * 2 * (sp.ideg + 1);
}

// f(y): dY_k/dt and dT/dt, VPL components per lane (0 beyond N).  Per pass
// the record loads of the next are in flight.
template <int VPL, int G, class CR>
__device__ __forceinline__ void rhs_v(const CR &crew, const DevMech &m, const DevSparse &sp, double *lds, const double (&y)[VPL], double p,
                      const double *dlnA, int lane, double (&f)[VPL])
{
    constexpr int NV = G * VPL;
    const int N = m.N;
    Thermo<> th[VPL];
    Rec nxt = load_rx<G>(sp, max(crew.first(sp), 0), lane);
    const Mix<> x = mixture_v<VPL, G>(crew, m, sp, lds, y, p, th, lane);
    double itt;
    const double *itb = thermo_block(sp, m.R, x.lnT, itt);
    crew.sync();
    // compiled once with the tables and once without (the exact path's code
    // does not carry the tables' branches)
    if (itb)
        rhs_passes<G, NV, true>(crew, m, sp, sp.ideg, lds, x, dlnA, lane, itb, itt, nxt);
    else
        rhs_passes<G, NV, false>(crew, m, sp, 0, lds, x, dlnA, lane, nullptr, 0.0, nxt);
    crew.sync();
    double hw[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        f[v] = hw[v] = 0.0;
        if (c < N) {
            const double wdk = pair<NV>(lds, SPL_HW, c)[1];
            f[v] = m.W()[c] * wdk / x.rho;
            hw[v] = (m.cv ? th[v].hRT - 1.0 : th[v].hRT) * wdk;
        }
    }
    const double fT = -m.Rgas * x.T * vsum<VPL, G>(hw) / (x.rho * x.cp);
#pragma unroll
    for (int v = 0; v < VPL; ++v)
        if (lane + G * v == N) f[v] = fT;
    crew.sync();
}

// Jacobian pass: f(y), and the bordered matrix of I/hg - J formed in the L+U
// entries (fill entries zero).  The reaction loop scatters -nu dq/dC and
// -nu dq/dT into the species rows and the reaction-enthalpy-weighted
// derivatives into the temperature row; the border entries are finished per
// state component after one barrier.
template <int VPL, int G, class CR>
__device__ __forceinline__ void jac_v(const CR &crew, const DevMech &m, const DevSparse &sp, double *lds, const double (&y)[VPL], double p,
                      const double *dlnA, int lane, double inv_hg, double (&f)[VPL])
{
    constexpr int NV = G * VPL;
    const int N = m.N;
    double *E = lds + SPL_E * NV;
    Thermo<> th[VPL];
    Rec nxt = load_rx<G>(sp, max(crew.first(sp), 0), lane);
    crew.barrier();  // what it clears has been read
    const Mix<> x = mixture_v<VPL, G>(crew, m, sp, lds, y, p, th, lane);
    double *const ts = lds + SPL_U * NV + lane;  // a crew's tt and tm
    if (crew.rank == 0 && crew.w > 1) ts[0] = ts[NV] = 0.0;
    // and the zero slot (the same number of turns for every lane)
#pragma unroll 4
    for (int e = 2 * G * crew.rank; e <= sp.nnz; e += 2 * G * crew.w)
        *(double2 *)(E + min(e + 2 * lane, sp.nnz & ~1)) = make_double2(0.0, 0.0);
    crew.sync();
    const double RT = m.Rgas * x.T;
    double itt;
    const double *itb = thermo_block(sp, m.R, x.lnT, itt);
    double tt = 0.0, tm = 0.0;
    if (itb)
        jac_passes<G, NV, VPL == 1, -1, true>(crew, m, sp, sp.ideg, lds, E, x, RT, dlnA, lane, itb, itt, nxt, ts, tt, tm);
    else
        jac_passes<G, NV, VPL == 1, -1, false>(crew, m, sp, 0, lds, E, x, RT, dlnA, lane, nullptr, 0.0, nxt, ts, tt, tm);
    crew.sync();
    if (crew.w > 1) tt = ts[0], tm = ts[NV];
    const double one = m.cv ? 1.0 : 0.0;
    double hw[VPL], eu[VPL], cpf[VPL], dcp[VPL], uak[VPL];
    uint4 cm[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        cm[v] = ((const uint4 *)sp.comp)[c];
        // no branches from here to the factorisation (see rhs_jac)
        const bool own = c < N;
        const int k = min(c, N - 1);
        const double Wk = own ? m.W()[k] : 0.0, iw = own ? m.invW()[k] : 0.0;
        const double wdk = own ? pair<NV>(lds, SPL_HW, c)[1] : 0.0;
        uak[v] = own ? lds[SPL_UA * NV + c] : 0.0;
        f[v] = Wk * wdk / x.rho;
        hw[v] = (th[v].hRT - one) * wdk;
        eu[v] = th[v].hRT * uak[v] / x.rho;      // (h_k/(R T W_k)) u_k, u_k = W_k UA_k / rho
        cpf[v] = (th[v].cpR - one) * f[v] * iw;
        dcp[v] = th[v].dcpR * y[v] * iw;
    }
    const double H = RT * vsum<VPL, G>(hw);
    const double Eu = m.cv ? 0.0 : RT * vsum<VPL, G>(eu);
    const double Scpf = m.Rgas * vsum<VPL, G>(cpf);
    const double Sdcp = m.Rgas * vsum<VPL, G>(dcp);
    const double TT = gsum<G>(tt);
    const double fT = -H / (x.rho * x.cp);
    const double vs = m.cv ? 1.0 : x.Wbar;
    const double ct = m.cv ? 0.0 : x.invT;
    const double tb = m.cv ? gsum<G>(tm) : x.Wbar * Eu;
    const double icp = 1.0 / x.cp;
    const double MTT = inv_hg + (TT / x.rho + (m.cv ? 0.0 : Eu * x.invT) + Scpf + fT * Sdcp) * icp;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        const int e0 = cm[v].x & 0xffff, e1 = cm[v].x >> 16, e2 = cm[v].y & 0xffff, e3 = cm[v].y >> 16, e4 = cm[v].z & 0xffff;
        f[v] = c == N ? fT : f[v];
        if constexpr (!std::is_same_v<CR, Solo>)
            if (crew.rank != 0) continue;
        // the temperature's lane has (T, T) and the corner of the borders; what
        // it and the lanes behind it do not have are trash entries
        const bool own = c < N;
        const double us = m.cv ? uak[v] : uak[v] / x.rho;
        const double a0 = E[e0], a1 = E[e1], a3 = E[e3];
        E[e0] = own ? a0 + inv_hg : MTT;
        E[e1] = own ? a1 / x.rho - ct * us : -1.0;
        E[e2] = -us;
        E[e3] = (a3 + tb + fT * m.Rgas * (th[v].cpR - one)) * icp;
        E[e4] = vs;
    }
    crew.sync();
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

// ---- one cell per wave: blocks of 16 pivots --------------------------------
typedef double d4 __attribute__((ext_vector_type(4)));

// acc -= A B on one 16 x 16 tile with four pivots: lane l gives A[l % 16][l / 16]
// and B[l / 16][l % 16] and holds rows 4 r + l / 16 of column l % 16 (the
// last argument negates A)
__device__ __forceinline__ d4 tile_sub(double a, double b, d4 acc)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 1);
}

__device__ __forceinline__ uint32_t half_of(const uint4 &w, int h)
{
    const uint32_t x = h < 2 ? w.x : h < 4 ? w.y : h < 6 ? w.z : w.w;
    return h % 2 ? x >> 16 : x & 0xffff;
}
template <int VPL>
__device__ __forceinline__ void put(double *E, uint32_t o, double v)
{
    if (VPL == 1)
        *(double *)((char *)E + o) = v;
    else
        E[o] = v;
}

// Numeric LU of the formed matrix in E, blocks of 16 pivots in position order:
// L scaled, U scaled to a unit diagonal, 1/u_kk in DINV.  A broadcast of one
// lane to the 16 of its row costs nothing inside a multiply-add (DPP), where
// one to the whole wave takes two readlanes at twice a multiply-add's time
// each; so everything of a block is laid out in rows of 16 lanes:
//   - the diagonal block, a row per lane, the same in all four rows of lanes;
//   - the block's rows of U, a row per lane, the columns dealt to the four
//     rows of lanes, eliminated together with the diagonal block;
//   - the block's columns of L, a column per lane, the rows dealt likewise,
//     as L D by the unit upper part of the diagonal block;
//   - the rest, A -= (L D) (D^-1 U), on the matrix cores.
// Entries outside the pattern are read from the zero slot and stay zero in
// exact zeros, so they are written back there and no lane is masked.  (The
// elimination by levels of independent pivots it replaces took 48k cycles of
// a lone wave on 53 species, waiting for 8 levels of indices from L2 and for
// the broadcasts of a 30-wide register tail.)
template <int VPL, class CR>
__device__ __forceinline__ void lu_blocks(const CR &crew, const DevSparse &sp, double *E, double *DINV, int lane)
{
    constexpr int Q = 4 * VPL - 1;  // most blocks after one
    const int n = sp.n, nb = (n + 15) / 16;
    // this wave's blocks beside the diagonal one, and its tiles (VPL = 1)
    uint32_t own = 0, mine = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if ((q & (crew.w - 1)) == crew.rank) own |= 1u << q;
        if (VPL == 1)
#pragma unroll
            for (int q2 = 0; q2 < Q; ++q2)
                if (((q + 2 * q2) & (crew.w - 1)) == crew.rank) mine |= 1u << (q + Q * q2);
    }
    const int c = lane & 15;
    const uint4 *t = (const uint4 *)sp.blk + lane;
    // a block's first words, loaded one block ahead
    uint4 wd[4], wu[Q];
    auto words = [&](int r) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < 4; ++w) wd[w] = t[w * WAVE];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (q < r && (own >> q & 1)) wu[q] = t[(4 + q) * WAVE];
    };
    words(nb - 1);
#pragma unroll 1
    for (int b = 0; b < nb; ++b) {
        const int k0 = 16 * b, r = nb - 1 - b;
        const uint32_t act = own & ((1u << r) - 1);
        const uint4 id0 = wd[0], id1 = wd[1], it0 = wd[2], it1 = wd[3];
        uint4 ul[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) ul[q] = wu[q];
        const uint4 *ta = t + (4 + r) * WAVE;  // the rest of this block's words
        const uint2 *ct = (const uint2 *)(t - lane + (4 + 2 * r) * WAVE) + lane;
        t += (4 + 2 * r) * WAVE + r * r * (WAVE / 2);
        double D[16], u[Q][4], x[Q][4];
#pragma unroll
        for (int k = 0; k < 16; ++k) D[k] = entry<VPL>(E, half_of(k < 8 ? id0 : id1, k % 8));
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (act >> q & 1) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    u[q][h] = entry<VPL>(E, half_of(ul[q], h));
                    x[q][h] = entry<VPL>(E, half_of(ul[q], 4 + h));
                }
            }
        if (r > 0) words(r - 1);
        double dinv = 0.0;
        unrolled<16>([&](auto K) __attribute__((always_inline)) {
            constexpr int k = K;
            if (k0 + k < n) {
                const double inv = 1.0 / bcast<16, k>(D[k]);
                const double l = c > k ? D[k] * inv : 0.0;
                dinv = c == k ? inv : dinv;
                D[k] = c > k ? l : D[k];
                if constexpr (k < 15) {
                    fmac_row<k>(D[k + 1], l);
                    constexpr int j0 = k + 2;
#pragma unroll
                    for (int j = j0; j + 3 < 16; j += 4) fmac_row4<k>(D[j], D[j + 1], D[j + 2], D[j + 3], l);
#pragma unroll
                    for (int j = j0 + (16 - j0) / 4 * 4; j < 16; ++j) fmac_row<k>(D[j], l);
#pragma unroll
                    for (int q = 0; q < Q; ++q)
                        if (act >> q & 1) fmac_row4<k>(u[q][0], u[q][1], u[q][2], u[q][3], l);
                }
            }
        });
        crew.barrier();  // the block has been read
        if (crew.rank == 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                D[k] *= k > c ? dinv : 1.0;
                put<VPL>(E, half_of(k < 8 ? id0 : id1, k % 8), D[k]);
            }
            if (lane < 16 && k0 + c < n) DINV[k0 + c] = dinv;
        }
        if (r == 0) break;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (act >> q & 1) {
#pragma unroll
                for (int h = 0; h < 4; ++h) put<VPL>(E, half_of(ul[q], h), u[q][h] * dinv);
            }
        crew.sync();
        uint4 ab[VPL == 1 ? Q : 1];
        uint2 ci[VPL == 1 ? Q : 1][VPL == 1 ? Q : 1];
        if constexpr (VPL == 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q < r) {
                    ab[q] = ta[q * WAVE];
#pragma unroll
                    for (int q1 = 0; q1 < Q; ++q1)
                        if (q1 < r && (mine >> (q1 + Q * q) & 1)) ci[q1][q] = ct[(q1 * r + q) * WAVE];
                }
        }
#pragma unroll
        for (int k = 0; k < 15; ++k) D[k] = entry<VPL>(E, half_of(k < 8 ? it0 : it1, k % 8));
        unrolled<15>([&](auto K) __attribute__((always_inline)) {
            constexpr int k = K;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (act >> q & 1) fmac_row4<k>(x[q][0], x[q][1], x[q][2], x[q][3], D[k]);
        });
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (act >> q & 1) {
#pragma unroll
                for (int h = 0; h < 4; ++h) put<VPL>(E, half_of(ul[q], 4 + h), x[q][h]);
            }
        crew.sync();
        auto tile = [&](const uint4 &wa, const uint2 &ci, const double (&B)[4]) __attribute__((always_inline)) {
            const uint32_t co[4] = {ci.x & 0xffff, ci.x >> 16, ci.y & 0xffff, ci.y >> 16};
            d4 acc;
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = entry<VPL>(E, co[i]);
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = tile_sub(entry<VPL>(E, half_of(wa, s)), B[s], acc);
#pragma unroll
            for (int i = 0; i < 4; ++i) put<VPL>(E, co[i], acc[i]);
        };
        if constexpr (VPL == 1) {
#pragma unroll
            for (int q2 = 0; q2 < Q; ++q2) {
                if (q2 < r) {
                    double B[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) B[s] = entry<VPL>(E, half_of(ab[q2], 4 + s));
#pragma unroll
                    for (int q1 = 0; q1 < Q; ++q1)
                        if (q1 < r && (mine >> (q1 + Q * q2) & 1)) tile(ab[q1], ci[q1][q2], B);
                }
            }
        } else {
            // up to 49 tiles: one loop, a tile's indices loaded during the one before
            const int first = min(crew.rank, r * r - 1);
            uint4 wa = ta[first % r * WAVE], wb = ta[first / r * WAVE];
            uint2 cn = ct[(first % r * r + first / r) * WAVE];
            double B[4];
            int q0 = -1;
#pragma unroll 1
            for (int q = crew.rank; q < r * r; q += crew.w) {
                const int q2 = q / r, nx = min(q + crew.w, r * r - 1);
                if (q2 != q0) {
                    q0 = q2;
#pragma unroll
                    for (int s = 0; s < 4; ++s) B[s] = entry<VPL>(E, half_of(wb, 4 + s));
                }
                const uint4 w = wa;
                const uint2 c2 = cn;
                wa = ta[nx % r * WAVE];
                wb = ta[nx / r * WAVE];
                cn = ct[((nx % r) * r + nx / r) * WAVE];
                tile(w, c2, B);
            }
        }
        crew.sync();
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (act >> q & 1) {
#pragma unroll
                for (int h = 0; h < 4; ++h) put<VPL>(E, half_of(ul[q], 4 + h), x[q][h] * dinv);
            }
    }
    crew.sync();
}

template <int VPL, int G, class CR>
__device__ __forceinline__ void lu_v(const CR &crew, const DevSparse &sp, double *lds, int lane, Factors<VPL, G> &fac)
{
    constexpr int NV = G * VPL;
    double *E = lds + SPL_E * NV;
    if constexpr (G < WAVE) {
        lu_group<G>(sp, E, lane, fac);
        lds_sync();
    } else {
        lu_blocks<VPL>(crew, sp, E, lds + SPL_DINV * NV, lane);
    }
}

// Solve M x = b with the factors (b, x: VPL components per lane; a lane holds
// the same position as component and as row), in blocks of 16 columns: the
// chain through a block's 16 pivots runs inside the row of lanes that holds
// them, one broadcasting multiply-add a pivot; the block's solution is then
// spread to all four rows of lanes and the rows behind apply it, four
// multiply-adds at a time off the chain.  Each lane's entries come a block
// ahead from LDS through a table of its row (the zero slot where it has none
// on that side).  (A column took 189 cycles of a lone wave with each entry's
// place computed from the column's mask at its turn, 56 with the table and a
// broadcast to the whole wave by two readlanes.)
template <int VPL>
__device__ __forceinline__ void sweeps(const DevSparse &sp, const double *E, const double *DINV, int lane,
                                       double (&z)[VPL])
{
    constexpr int NB = 4 * VPL;
    const int n = sp.n;
    // tables: [slot][lane][64 VPL columns], two words per block
    const uint4 *tl = (const uint4 *)sp.low + 8 * VPL * lane, *tu = (const uint4 *)sp.up + 8 * VPL * lane;
    uint4 il[NB][VPL][2], iu[NB][VPL][2];
    auto index = [&](const uint4 *t, int b, uint4 (&w)[VPL][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            w[s][0] = t[s * WAVE * 8 * VPL + 2 * b];
            w[s][1] = t[s * WAVE * 8 * VPL + 2 * b + 1];
        }
    };
    auto load = [&](const uint4 (&w)[VPL][2], double (&a)[VPL][16]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < VPL; ++s)
#pragma unroll
            for (int k = 0; k < 16; ++k) a[s][k] = entry<VPL>(E, half_of(w[s][k / 8], k % 8));
    };
    // the tables' words all at once: one trip to L2
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (16 * b < n) index(tl, b, il[b]);
#pragma unroll
    for (int b = NB - 1; b >= 0; --b)
        if (16 * b < n) index(tu, b, iu[b]);
    double dinv[VPL];
#pragma unroll
    for (int s = 0; s < VPL; ++s) dinv[s] = lane + WAVE * s < n ? DINV[lane + WAVE * s] : 0.0;
    double a[VPL][16], nx[VPL][16];
    load(il[0], a);
    unrolled<NB>([&](auto B) __attribute__((always_inline)) {
        constexpr int b = B, s = b / 4, g = b % 4;
        if (16 * b < n) {
            if constexpr (b + 1 < NB) if (16 * b + 16 < n) load(il[b + 1], nx);
            unrolled<15>([&](auto K) __attribute__((always_inline)) { fmac_in<K, 1 << g>(z[s], a[s][K]); });
            if constexpr (b + 1 < NB) {
                const double xb = spread_row<g>(z[s]);
                constexpr int behind = 0xf & ~((2 << g) - 1);
                unrolled<4>([&](auto K) __attribute__((always_inline)) {
                    if constexpr (behind != 0) fmac_by4<4 * K, behind>(z[s], xb, &a[s][4 * K]);
                    if constexpr (s + 1 < VPL) fmac_by4<4 * K, 0xf>(z[VPL - 1], xb, &a[VPL - 1][4 * K]);
                });
            }
#pragma unroll
            for (int v = 0; v < VPL; ++v)
#pragma unroll
                for (int k = 0; k < 16; ++k) a[v][k] = nx[v][k];
        }
    });
#pragma unroll
    for (int s = 0; s < VPL; ++s) z[s] *= dinv[s];
    unrolled<NB>([&](auto B) __attribute__((always_inline)) {
        constexpr int b = NB - 1 - B, s = b / 4, g = b % 4;
        if (16 * b < n) {
            if (16 * b + 16 >= n) load(iu[b], a);  // the first block taken
            if constexpr (b > 0) load(iu[b - 1], nx);
            unrolled<15>([&](auto K) __attribute__((always_inline)) { fmac_in<15 - K, 1 << g>(z[s], a[s][15 - K]); });
            if constexpr (b > 0) {
                const double xb = spread_row<g>(z[s]);
                constexpr int behind = (1 << g) - 1;
                unrolled<4>([&](auto K) __attribute__((always_inline)) {
                    if constexpr (behind != 0) fmac_by4<4 * K, behind>(z[s], xb, &a[s][4 * K]);
                    if constexpr (s > 0) fmac_by4<4 * K, 0xf>(z[0], xb, &a[0][4 * K]);
                });
            }
#pragma unroll
            for (int v = 0; v < VPL; ++v)
#pragma unroll
                for (int k = 0; k < 16; ++k) a[v][k] = nx[v][k];
        }
    });
}

template <int VPL, int G>
__device__ __forceinline__ void solve_v(const DevMech &m, const DevSparse &sp, double *lds, const Factors<VPL, G> &fac,
                        const double (&b)[VPL], int lane, double (&x)[VPL])
{
    const int N = m.N;
    // scaled unknowns z_k = x_k / W_k; the sigma row's right-hand side is zero
    double z[VPL], W[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        const double iw = c < N ? m.invW()[c] : c == N ? 1.0 : 0.0;
        W[v] = c < N ? m.W()[c] : c == N ? 1.0 : 0.0;  // loaded ahead of the sweeps
        z[v] = b[v] * iw;
    }
    if constexpr (G < WAVE)
        sweeps_group<G>(sp, fac, lane, z[0]);
    else
        sweeps<VPL>(sp, lds + SPL_E * G * VPL, lds + SPL_DINV * G * VPL, lane, z);
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int c = lane + G * v;
        x[v] = c <= N ? z[v] * W[v] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// one Rosenbrock attempt and the integration of a cell
// ---------------------------------------------------------------------------
template <int VPL, int G, class CR>
__device__ __forceinline__ void ros_attempt_v(const CR &crew, const DevMech &m, const DevSparse &sp, const Opts &o, double *lds,
                              const double (&y)[VPL], double p, const double *dlnA, int lane, double hc, double *err,
                              double (&ynew)[VPL])
{
    const int n = m.N + 1;
    constexpr int NV = G * VPL;
    double *U = lds + SPL_U * NV;
    double f0[VPL], flast[VPL];
    jac_v<VPL, G>(crew, m, sp, lds, y, p, dlnA, lane, 1.0 / (GAM * hc), f0);
    Factors<VPL, G> fac;
    lu_v<VPL, G>(crew, sp, lds, lane, fac);
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
            rhs_v<VPL, G>(crew, m, sp, lds, ys, p, dlnA, lane, fi);
#pragma unroll
            for (int v = 0; v < VPL; ++v) flast[v] = fi[v];
        }
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            for (int j = 0; j < i; ++j) fi[v] += (TC[i][j] * ih) * U[j * NV + lane + G * v];
            if (lane + G * v >= n) fi[v] = 0.0;
        }
        if (crew.rank == 0) {  // one wave of a crew: four of them wait for the LDS
            double ui[VPL];
            solve_v<VPL, G>(m, sp, lds, fac, fi, lane, ui);
#pragma unroll
            for (int v = 0; v < VPL; ++v) U[i * NV + lane + G * v] = ui[v];
        }
        crew.barrier();
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
__device__ __forceinline__ int advance_v(const DevMech &m, const DevSparse &sp, const Opts &o, double *lds, double (&y)[VPL],
                         double p, double dt, const double *dlnA, int lane, Ctl &s)
{
#pragma unroll 1
    while (true) {
        double hc;
        bool last;
        const int st = ctl_begin(s, o, dt, hc, last);
        if (st != SC_CELL_OK) return st;
        double err, ynew[VPL];
        ros_attempt_v<VPL, G>(Solo{}, m, sp, o, lds, y, p, dlnA, lane, hc, &err, ynew);
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
// implies spills 13 to 39 registers to scratch with one cell per wave, 33 to 61
// with four and 63 to 100 with two (whose rows in registers are the longest),
// outside the inner loops.  With two slots per lane (398 to 418 registers) one
// wave takes a SIMD and nothing is spilled.
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

// The persistent launch of one cell per wave's 64 lanes: workgroups of one, two
// or four waves (crew_choice).  With one slot per lane each wave has its own LDS
// region and works by itself while the queue lasts; a wave that finds it empty
// waits, and when one wave of the workgroup is left with a cell, all of them
// finish it as a crew.  With two slots the workgroup has one region and is a crew
// of its waves from the beginning.  Every wait ends: a wave with a cell always gets on, by itself
// or as the crew, and the one that runs out last counts itself in as well.
// (A step of 53 species takes a lone wave 62 us, a crew of four 54: the pivots'
// chains and the solves do not split.  4,096 cells of 110 species, where the
// LDS leaves half a CU's SIMDs without a wave otherwise: 48.0 -> 41.3 ms; eight
// substeps of 300 cells of 53 species 42.0 -> 39.1 ms.)
struct CrewShare {
    int idle, owner, turn, pad;
    int64_t next, i, end;
    Ctl s;
};
constexpr int CREW_SHARE = 16;  // doubles ahead of the regions
static_assert(sizeof(CrewShare) <= CREW_SHARE * sizeof(double));
static_assert(CREW_SHARE % 2 == 0, "the regions' pairs are read in one");
constexpr int crew_most(int vpl) { return vpl == 1 ? 4 : 2; }

template <int VPL, bool CV, bool TB>
__global__ void __launch_bounds__(crew_most(VPL) * WAVE) SP_OCC
k_integrate_sp_crew(DevMech mk, DevSparse spk, Opts o, int64_t n, const double *T0, const double *P, const double *Y0,
                    int64_t ld, const double *DT, const double *dlnA, double *h_io, double *T1, double *Y1,
                    int32_t *status, int32_t *nacc, int32_t *nrej, unsigned long long *queue, const int32_t *perm,
                    int tile, const int32_t *ref)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    constexpr int NV = WAVE * VPL;
    CrewShare *sh = (CrewShare *)lds;
    const int lane = (int)threadIdx.x % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE), waves = (int)blockDim.x / WAVE;
    if (threadIdx.x == 0) sh->idle = 0, sh->owner = -1;
    __syncthreads();
    // the first tiles go round the workgroups, the queue has those behind
    Crew crew{1, 0, &sh->turn, 0};
    if (VPL > 1) crew.join(sp, waves, wave);
    double *L = lds + CREW_SHARE + (VPL == 1 ? (size_t)wave * sp.size : 0);
    int64_t i = ((int64_t)(VPL == 1 ? wave : 0) * gridDim.x + blockIdx.x) * tile, end = min(i + tile, n);
    bool busy = false;
    double y[VPL], p = 0.0, dt = 0.0;
    Ctl s = ctl_init(0.0, 0.0);
#pragma unroll 1
    while (true) {
        int st = -1;  // the cell's status, once it ends
        int64_t c = 0;
        if (!busy) {
            if (i >= end && (VPL > 1 || crew.w == 1)) {
                int64_t next = n;
                if (VPL > 1) {
                    __syncthreads();
                    if (queue && threadIdx.x == 0) sh->next = (int64_t)atomicAdd(queue, (unsigned long long)tile);
                    __syncthreads();
                    if (queue) next = sh->next;
                } else if (queue && lane == 0) {
                    next = (int64_t)atomicAdd(queue, (unsigned long long)tile);
                }
                i = uniform(next);
                end = min(i + tile, n);
            }
            if (i < end) {
                c = perm ? (int64_t)perm[i] : i;
                if (ref && ref[c] != c) {  // left to the mapping pass
                    ++i;
                    continue;
                }
                load_state_v<VPL, WAVE>(m, sp, T0, Y0, ld, c, lane, y);
                p = P[c], dt = DT[c];
                s = ctl_init(initial_step(h_io, c, dt), dt);
                busy = true;
                if (bad_input_v<VPL, WAVE>(m, y, p, dt, lane))
                    st = SC_CELL_BAD_INPUT;
                else if (!(dt > 0.0))
                    st = SC_CELL_OK;
            } else if (sc::crew_leaves(VPL, crew.w, waves)) {
                break;
            }
        }
        if (VPL == 1 && crew.w < waves && st < 0) {
            int idle, owner = -1;
            if (!busy) {
                if (lane == 0) __hip_atomic_fetch_add(&sh->idle, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
                while (true) {
                    // the count first: it is full only when no owner can come any more
                    idle = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(&sh->idle, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
                    owner = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(&sh->owner, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
                    if (owner >= 0 || idle == waves) break;
                    __builtin_amdgcn_s_sleep(16);
                }
                if (owner < 0) break;
            } else {
                idle = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&sh->idle, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (idle == waves - 1) {
                    owner = wave;
#pragma unroll
                    for (int v = 0; v < VPL; ++v) L[SPL_U * NV + lane + WAVE * v] = y[v];
                    if (lane == 0) {
                        sh->i = i, sh->end = end, sh->s = s;
                        __hip_atomic_store(&sh->owner, wave, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
            if (owner >= 0) {
                __syncthreads();
                L = lds + CREW_SHARE + (size_t)owner * sp.size;
                i = uniform(sh->i), end = uniform(sh->end);
                s.t = uniform(sh->s.t), s.h = uniform(sh->s.h), s.hnext = uniform(sh->s.hnext);
                s.nacc = __builtin_amdgcn_readfirstlane(sh->s.nacc);
                s.nrej = __builtin_amdgcn_readfirstlane(sh->s.nrej);
                s.nonfinite = __builtin_amdgcn_readfirstlane(sh->s.nonfinite);
                s.last_rej = __builtin_amdgcn_readfirstlane(sh->s.last_rej);
#pragma unroll
                for (int v = 0; v < VPL; ++v) y[v] = L[SPL_U * NV + lane + WAVE * v];
                c = perm ? (int64_t)perm[i] : i;
                p = P[c], dt = DT[c];
                crew.join(sp, waves, wave);
                busy = true;
                __syncthreads();
            }
        }
        if (st < 0) {
            double hc;
            bool last;
            st = ctl_begin(s, o, dt, hc, last);
            if (st == SC_CELL_OK) {
                st = -1;
                double err, ynew[VPL];
                ros_attempt_v<VPL, WAVE>(crew, m, sp, o, L, y, p, dlnA, lane, hc, &err, ynew);
                const int r = ctl_end(s, o, uniform(err), hc, last, dt);
                if (r < 0) st = -r;
                if (r == 1) {
#pragma unroll
                    for (int v = 0; v < VPL; ++v) y[v] = ynew[v];
                    if (last) st = SC_CELL_OK;
                }
            }
        }
        if (st >= 0) {
            if (crew.rank == 0) {
                c = perm ? (int64_t)perm[i] : i;
                store_state_v<VPL, WAVE>(m, sp, T1, Y1, ld, c, lane, y);
                if (lane == 0) {
                    status[c] = st;
                    if (nacc) nacc[c] = s.nacc;
                    if (nrej) nrej[c] = s.nrej;
                    if (h_io && st == SC_CELL_OK && dt > 0.0) h_io[c] = s.hnext;
                }
            }
            busy = false;
            ++i;
        }
    }
}

// Doubles of one cell's LDS in the right-hand side kernel: the pairs and the
// Euler accumulator, without the L+U entries (2.5 KB a cell instead of 19 at
// 53 species, so registers bound the waves in flight: 16 a CU instead of 8).
template <int VPL, int G>
constexpr int rhs_region()
{
    static_assert(5 * G * VPL % 2 == 0, "the pairs are read in one");
    return 5 * G * VPL + (G == 32 ? 16 : 0);
}

// Consecutive workgroups go to the eight dies in turn; the eight cells of a
// 64-byte line of the state go to one, which reads the line once.
__device__ __forceinline__ int64_t line_cell(int64_t b, int64_t n)
{
    return b / 64 * 64 + 64 <= n ? b / 64 * 64 + b % 8 * 8 + b / 8 % 8 : b;
}

template <int VPL, bool CV, int CPW, bool TB>
__global__ void __launch_bounds__(WAVE) k_rhs_sp(DevMech mk, DevSparse spk, int64_t n, const double *T,
                                                 const double *P, const double *Y, int64_t ld, const double *dlnA,
                                                 double *fT, double *fY)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    constexpr int G = WAVE / CPW;
    const int lane = (int)threadIdx.x % G, grp = (int)threadIdx.x / G;
    double *ldsg = lds + grp * rhs_region<VPL, G>();
    const int64_t c = line_cell(blockIdx.x, gridDim.x) * CPW + grp;
    if (c >= n) return;
    double y[VPL], f[VPL];
    load_state_v<VPL, G>(m, sp, T, Y, ld, c, lane, y);
    rhs_v<VPL, G>(Solo{}, m, sp, ldsg, y, P[c], dlnA, lane, f);
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
    jac_v<VPL, G>(Solo{}, m, sp, ldsg, y, P[c], dlnA, lane, 0.0, f);
    // a row at a time, columns across the lanes (species order); what depends
    // on the column only is taken once
    const double *E = ldsg + SPL_E * G * VPL;
    const int N = m.N, nn = N + 1;
    double cj[VPL], sj[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int j = lane + G * v;
        cj[v] = j < N ? m.invW()[sp.pos[j]] : 1.0;
        sj[v] = j < N ? E[sp.comp[8 * sp.pos[j] + 4]] : 0.0;
    }
#pragma unroll 1
    for (int i0 = 0; i0 < nn; i0 += 6) {
        uint16_t e[6][VPL];
        double a[6], w[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            const int i = min(i0 + d, N), pi = sp.pos[i];
            a[d] = i < N ? E[sp.comp[8 * pi + 2]] : 0.0;
            w[d] = i < N ? m.W()[pi] : 1.0;
#pragma unroll
            for (int v = 0; v < VPL; ++v) e[d][v] = sp.jmap[i * nn + min(lane + G * v, N)];
        }
#pragma unroll
        for (int d = 0; d < 6; ++d)
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                const int j = lane + G * v;
                if (i0 + d < nn && j < nn)
                    J[(c * nn + i0 + d) * nn + j] = -(w[d] * cj[v]) * (E[e[d][v]] + a[d] * sj[v]);
            }
    }
}

// W waves a cell (with two slots per lane two where they are a crew)
template <int VPL, bool CV, int CPW, bool TB, int W>
__global__ void __launch_bounds__(W * WAVE) k_linsolve_sp(DevMech mk, DevSparse spk, int64_t n, const double *T,
                                                      const double *P, const double *Y, int64_t ld,
                                                      const double *dlnA, const double *hg, const double *b,
                                                      double *x)
{
    extern __shared__ double lds[];
    const DevMech m = fix_reactor<CV>(mk);
    const DevSparse sp = fix_tables<TB>(spk);
    constexpr int G = WAVE / CPW;
    const int lane = (int)threadIdx.x % G, grp = W == 1 ? (int)threadIdx.x / G : 0;
    const int64_t c = (int64_t)blockIdx.x * CPW + grp;
    if (c >= n) return;
    double *ldsg = lds + (W == 1 ? (size_t)grp * sp.size : CREW_SHARE);
    std::conditional_t<W == 1, Solo, Crew> crew;
    if constexpr (W > 1) {
        crew.turn = &((CrewShare *)lds)->turn;
        crew.join(sp, W, __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE));
    }
    double y[VPL], f[VPL], bb[VPL], xx[VPL];
    load_state_v<VPL, G>(m, sp, T, Y, ld, c, lane, y);
    jac_v<VPL, G>(crew, m, sp, ldsg, y, P[c], dlnA, lane, 1.0 / hg[c], f);
    Factors<VPL, G> fac;
    lu_v<VPL, G>(crew, sp, ldsg, lane, fac);
    const int nn = m.N + 1;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int i = lane + G * v;
        bb[v] = i < nn ? b[c * nn + sp.perm[i]] : 0.0;
    }
    if (crew.rank != 0) return;
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
// and of a crew workgroup: a region per wave, one in all with two slots per lane
static size_t crew_lds(int vpl, const DevSparse &sp, int waves)
{
    return sizeof(double) * (CREW_SHARE + (size_t)sp.size * (vpl == 1 ? waves : 1));
}
static unsigned sp_blocks(int64_t n, int cpw) { return (unsigned)((n + cpw - 1) / cpw); }

hipError_t launch_rhs_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                         const double *p, const double *Y, int64_t ld, const double *dlnA, double *fT, double *fY,
                         hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(hipLaunchKernelGGL(SP_KERNEL(k_rhs_sp), dim3(sp_blocks(n, cpw)), dim3(WAVE),
                                   (sizeof(double) * rhs_region<VPLV, WAVE / CPWV>() * cpw), s, m, sp, n, T, p, Y, ld,
                                   dlnA, fT, fY))
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
                              const double *b, double *x, int waves, hipStream_t s)
{
    const int cpw = sp.cpw;
    auto launch = [&](auto kern, size_t bytes) {
        hipLaunchKernelGGL(kern, dim3(sp_blocks(n, cpw)), dim3(waves * WAVE), bytes, s, m, sp, n, T, p, Y, ld, dlnA,
                           hg, b, x);
    };
    SP_DISPATCH(if (VPLV == 2 && waves == 2) launch(k_linsolve_sp<VPLV, CVV, CPWV, TBV, VPLV>, crew_lds(vpl, sp, 2));
                else launch(k_linsolve_sp<VPLV, CVV, CPWV, TBV, 1>, sp_lds(sp, cpw)))
}

hipError_t launch_integrate_sp(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o, int64_t n,
                               const double *T0, const double *p, const double *Y0, int64_t ld, const double *dt,
                               const double *dlnA, double *h_io, double *T1, double *Y1, int32_t *st, int32_t *na,
                               int32_t *nr, const int32_t *ref, int waves, hipStream_t s)
{
    const int cpw = sp.cpw;
    // a crew per cell, or where they would be more than a launch's 2^32
    // threads, four waves each, per tile of cells
    const int tile = (int)((n >> 22) + 1);
    if (waves > 0)
        return launch_integrate_sp_persistent(vpl, m, sp, o, n, T0, p, Y0, ld, dt, dlnA, h_io, T1, Y1, st, na, nr,
                                              nullptr, nullptr, tile, (int)((n + tile - 1) / tile), waves, ref, s);
    SP_DISPATCH(if constexpr (VPLV == 1) hipLaunchKernelGGL(
        SP_KERNEL(k_integrate_sp), dim3(sp_blocks(n, cpw)), dim3(WAVE), sp_lds(sp, cpw), s, m, sp, o, n, T0, p, Y0,
        ld, dt, dlnA, h_io, T1, Y1, st, na, nr, ref))
}

hipError_t launch_integrate_sp_persistent(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o,
                                          int64_t n, const double *T0, const double *p, const double *Y0,
                                          int64_t ld, const double *dt, const double *dlnA, double *h_io,
                                          double *T1, double *Y1, int32_t *st, int32_t *na, int32_t *nr,
                                          unsigned long long *queue, const int32_t *perm, int tile, int grid,
                                          int waves, const int32_t *ref, hipStream_t s)
{
    const int cpw = sp.cpw;
    SP_DISPATCH(if constexpr (CPWV == 1) hipLaunchKernelGGL(
                    (k_integrate_sp_crew<VPLV, CVV, TBV>), dim3((unsigned)grid), dim3(waves * WAVE),
                    crew_lds(vpl, sp, waves), s, m, sp, o, n, T0, p, Y0, ld, dt, dlnA, h_io, T1, Y1, st, na, nr,
                    queue, perm, tile, ref);
                else hipLaunchKernelGGL(SP_KERNEL(k_integrate_sp_persistent), dim3((unsigned)grid), dim3(WAVE),
                                        sp_lds(sp, cpw), s, m, sp, o, n, T0, p, Y0, ld, dt, dlnA, h_io, T1, Y1, st,
                                        na, nr, queue, perm, tile, ref))
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

int64_t queue_start_sp(int vpl, const DevSparse &sp, int grid, int tile, int waves)
{
    if (sp.cpw > 1) return 0;
    return (int64_t)grid * tile * (vpl == 1 ? waves : 1);
}

SpCapacity capacity_sp(int vpl, const DevSparse &sp, int device)
{
    SpCapacity r{};
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return r;
    const int cpw = sp.cpw;
    auto occ = [&](auto kern, int threads, size_t bytes) {
        int per_cu = 0;
        if (sc::lds_held(bytes) == 0 ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, bytes) != hipSuccess)
            return 0;
        return std::min(per_cu, sc::lds_held(bytes)) * cus;
    };
    auto set = [&](auto pers, auto stat) {
        if (cpw > 1) r.groups[0] = occ(pers, WAVE, sp_lds(sp, cpw));
        else
            for (int k = 0; 1 << k <= crew_most(vpl); ++k) r.groups[k] = occ(pers, WAVE << k, crew_lds(vpl, sp, 1 << k));
        r.fixed = occ(stat, WAVE, sp_lds(sp, cpw));
    };
    if (vpl == 1 && cpw == 1) set(k_integrate_sp_crew<1, false, false>, k_integrate_sp_static<1, false, 1, false>);
    else if (vpl == 1 && cpw == 2) set(k_integrate_sp_persistent<1, false, 2, false>, k_integrate_sp_static<1, false, 2, false>);
    else if (vpl == 1 && cpw == 4) set(k_integrate_sp_persistent<1, false, 4, false>, k_integrate_sp_static<1, false, 4, false>);
    else if (vpl == 2 && cpw == 1) {
        set(k_integrate_sp_crew<2, false, false>, k_integrate_sp_static<2, false, 1, false>);
        r.solve[0] = occ(k_linsolve_sp<2, false, 1, false, 1>, WAVE, sp_lds(sp, 1));
        r.solve[1] = occ(k_linsolve_sp<2, false, 1, false, 2>, 2 * WAVE, crew_lds(vpl, sp, 2));
    }
    return r;
}

}  // namespace scdev
