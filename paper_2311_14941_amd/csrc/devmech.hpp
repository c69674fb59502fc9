// Device view of a compiled mechanism and the launch interface of the
// kernels (shared by kernels.hip and capi.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mech.hpp"
#include "stiffchem.h"

namespace scdev {

// A falloff reaction's low-pressure rate and blending parameters
struct TroeRec {
    double lnA0, b0, Ea0R, a, iT3, iT1, T2, pad;
};

// The reactions as the kernels' passes read them (SparseRx's tables).
struct DevRx {
    int passes, n_tb, n_troe;  // reaction passes; third-body and falloff reactions (the first ones)
    const uint32_t *rec;
    const uint16_t *ix, *ixe;
    const double *eam1;
    const TroeRec *troe;
};

// A compiled mechanism on the device: species table sp = W[N] invW[N]
// nasa[7][N] (species index fastest).  Few base pointers keep the kernels'
// scalar-register footprint small.
struct DevMech {
    int N, R;
    int cv;  // 1: constant-volume reactor (the per-cell p input is the density)
    double Rgas, lnp0R;  // lnp0R = ln(p0 / Rgas)
    const double *sp;
    DevRx pass;  // the dense kernels' packed passes

    __host__ __device__ const double *W() const { return sp; }
    __host__ __device__ const double *invW() const { return sp + N; }
    __host__ __device__ const double *nasa() const { return sp + 2 * N; }  // [c*N + k]
};

using sc::SPL_CG, sc::SPL_HW, sc::SPL_UA, sc::SPL_U, sc::SPL_DINV, sc::SPL_E;

// The sparse kernels' view of a mechanism's compiled sparse algebra (device
// pointers).  Their DevMech has the species in elimination order, so a
// lane holds the same position as component and as matrix row.
struct DevSparse : DevRx {
    int n, nnz;
    int size;  // LDS doubles of one cell's region
    int cpw;  // cells per wave (1, 2 or 4): each cell takes 64 / cpw lanes
    const uint16_t *comp;  // [position][8]: e_kk, e_kT, e_kS, e_Tk, e_Sk; at N: e_TT, e_SS; else trash entries
    const int32_t *perm;   // position -> species (N: temperature)
    const int32_t *pos;    // species -> position
    const uint16_t *jmap;    // (N + 1)^2: (row, column) component in species order -> entry (or the zero slot)
    const uint16_t *row, *low, *up, *blk;  // SparseDev's operand tables
    // interpolated thermodynamics (null: exact): per interval of ln T and
    // reaction (execution order) the 2 (ideg + 1) coefficients of -dG/RT and
    // dH/RT in t = 2 (ln T - u_i) iinvdu - 1, then as many zeros
    const double *itab;
    int ideg, inint;
    double iu0, iinvdu;
};

struct Opts {
    double rtol, atol;
    double hmax_frac;  // > 0: steps capped at hmax_frac * dt
    int max_steps;
    int fixed;  // 1: fixed steps of the caller's h, no error control
};

hipError_t launch_rhs(int np, const DevMech &m, int64_t n, const double *T, const double *p, const double *Y,
                      int64_t ld, const double *dlnA, double *fT, double *fY, hipStream_t s);
hipError_t launch_jac(int np, const DevMech &m, int64_t n, const double *T, const double *p, const double *Y,
                      int64_t ld, const double *dlnA, double *J, hipStream_t s);
hipError_t launch_linsolve(int np, const DevMech &m, int64_t n, const double *T, const double *p,
                           const double *Y, int64_t ld, const double *dlnA, const double *hg, const double *b,
                           double *x, hipStream_t s);
hipError_t launch_integrate(int np, const DevMech &m, const Opts &o, int method, int64_t n,
                            const double *T0, const double *p, const double *Y0, int64_t ld, const double *dt,
                            const double *dlnA, double *h_io, double *T1, double *Y1, int32_t *st, int32_t *na,
                            int32_t *nr, const int32_t *ref, hipStream_t s);
hipError_t launch_integrate_persistent(int np, const DevMech &m, const Opts &o, int method, int64_t n,
                                       const double *T0, const double *p, const double *Y0, int64_t ld,
                                       const double *dt, const double *dlnA, double *h_io, double *T1, double *Y1,
                                       int32_t *st, int32_t *na, int32_t *nr, unsigned long long *queue,
                                       const int32_t *perm, int tile, int grid, const int32_t *ref, hipStream_t s);
hipError_t launch_integrate_static(int np, const DevMech &m, const Opts &o, int method, int64_t n,
                                   const double *T0, const double *p, const double *Y0, int64_t ld, const double *dt,
                                   const double *dlnA, double *h_io, double *T1, double *Y1, int32_t *st,
                                   int32_t *na, int32_t *nr, int grid, const int32_t *ref, hipStream_t s);
hipError_t order_cells(int order, int64_t n, const double *dt, const int32_t *na, const int32_t *nr,
                       void **ws, size_t *ws_bytes, int32_t **perm, hipStream_t s);
hipError_t order_ws_need(int order, int64_t n, size_t *need, hipStream_t s);
hipError_t order_cells_in(int order, int64_t n, const double *dt, const int32_t *na, const int32_t *nr, void *ws,
                          size_t ws_bytes, int32_t **perm, hipStream_t s);
// device address, size and cell limit of the allocation-free entry point's
// fixed scratch on `device` (which must be current)
hipError_t noalloc_scratch(int device, void **ptr, size_t *bytes, int64_t *max_cells);
hipError_t launch_set_u64(unsigned long long *p, unsigned long long v, hipStream_t s);
int persistent_capacity(int np, int device);

// sparse linear algebra kernels (sparse.hip); vpl = state components per lane
hipError_t launch_rhs_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                         const double *p, const double *Y, int64_t ld, const double *dlnA, double *fT, double *fY,
                         hipStream_t s);
hipError_t launch_jac_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                         const double *p, const double *Y, int64_t ld, const double *dlnA, double *J,
                         hipStream_t s);
hipError_t launch_linsolve_sp(int vpl, const DevMech &m, const DevSparse &sp, int64_t n, const double *T,
                              const double *p, const double *Y, int64_t ld, const double *dlnA, const double *hg,
                              const double *b, double *x, int waves, hipStream_t s);
hipError_t launch_integrate_sp(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o, int64_t n,
                               const double *T0, const double *p, const double *Y0, int64_t ld, const double *dt,
                               const double *dlnA, double *h_io, double *T1, double *Y1, int32_t *st, int32_t *na,
                               int32_t *nr, const int32_t *ref, int waves, hipStream_t s);
hipError_t launch_integrate_sp_persistent(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o,
                                          int64_t n, const double *T0, const double *p, const double *Y0,
                                          int64_t ld, const double *dt, const double *dlnA, double *h_io,
                                          double *T1, double *Y1, int32_t *st, int32_t *na, int32_t *nr,
                                          unsigned long long *queue, const int32_t *perm, int tile, int grid,
                                          int waves, const int32_t *ref, hipStream_t s);
hipError_t launch_integrate_sp_static(int vpl, const DevMech &m, const DevSparse &sp, const Opts &o, int64_t n,
                                      const double *T0, const double *p, const double *Y0, int64_t ld,
                                      const double *dt, const double *dlnA, double *h_io, double *T1, double *Y1,
                                      int32_t *st, int32_t *na, int32_t *nr, int grid, const int32_t *ref,
                                      hipStream_t s);
// where the queue of a persistent launch starts: behind the workgroups' first tiles
int64_t queue_start_sp(int vpl, const DevSparse &sp, int grid, int tile, int waves);
// Resident workgroups (0 where there are none): of 1, 2 and 4 waves of the
// persistent kernel (of one wave only with several cells per wave) and, with two
// slots per lane, of the linear solve's; and of the static kernel.
struct SpCapacity {
    int groups[sc::CREW_SIZES], solve[sc::CREW_SIZES], fixed;
};
SpCapacity capacity_sp(int vpl, const DevSparse &sp, int device);

// zonal reference-cell mapping (mapping.hip): the zone table is cleared,
// every mappable cell claims its zone (lowest index wins) and gets its
// reference in ref (ref[c] = c for cells that are integrated); after the
// integration, apply writes the mapped cells from their references
struct MapParams {
    const double *w;     // N per-species weights of Bilger's coupling function
    double beta_ox, dbeta, z_tol;  // dbeta = beta_fuel - beta_ox
    double dT, dlnp;     // band widths (dlnp = 0: no pressure bands)
    int nT, np;          // band counts; the table holds nT * np zones
    int32_t *table;      // nT * np zone claims
};
hipError_t launch_map_classify(const MapParams &mp, int N, int64_t n, const double *T, const double *p,
                               const double *Y, int64_t ld, const double *dt, int32_t *ref, hipStream_t s);
hipError_t launch_map_apply(int N, int64_t n, const int32_t *ref, const double *T0, const double *Y0, int64_t ld,
                            const double *dt, double *T1, double *Y1, int32_t *st, int32_t *na, int32_t *nr,
                            hipStream_t s);

// adjoint (adjoint.hip)
hipError_t launch_vjp(int np, const DevMech &m, int64_t cells, int64_t n, const double *T, const double *p, const double *Y,
                      int64_t ld, const double *dlnA, const double *wT, const double *wY, double *gT, double *gY,
                      double *gcell, hipStream_t s);
hipError_t launch_adjoint(int np, const DevMech &m, const Opts &o, int64_t n, const double *T0, const double *p,
                          const double *Y0, int64_t ld, const double *dt, const double *dlnA, const double *h_in,
                          const double *gT1, const double *gY1, double *gT0, double *gY0, double *gcell,
                          int32_t *st, int32_t *na, double *T1, double *Y1, double *scratch, int64_t slot_doubles,
                          int hcap, unsigned long long *queue, const int32_t *perm, int grid, hipStream_t s);
hipError_t launch_sum_cells(const double *g, int64_t n, int R, double *out, hipStream_t s);
int adjoint_capacity(int np, int R, int device);

// operator-split driver support (transport.hip)
hipError_t launch_transport2d(int nx, int ny, int ncomp, const double *in, int64_t ld, const double *u,
                              const double *dt, double dx, double D, const double *inflow, double *out,
                              hipStream_t s);
int adjoint_slot_checkpoints();
size_t lds_bytes_for(int np);

}  // namespace scdev
