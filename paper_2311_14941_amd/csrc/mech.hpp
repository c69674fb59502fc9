// Host-side mechanism model and compiler.
//
// The paper's chemistry library keeps "internal sparse algebra management of
// mechanism-related quantities" and a sparse analytical Jacobian (Sec. 2.5).
// Here that is a compile step run once per mechanism: parse and validate the
// text, convert the rate parameters to SI and log form, lay the reactions out
// as structure-of-arrays tables with fixed per-reaction slots (reactant,
// product and enhanced third-body species), derive the sparsity pattern of the
// analytical Jacobian terms, and count the work of every kernel phase.
#pragma once

#include <algorithm>
#include <cstdint>
#include <stdexcept>
#include <string>
#include <vector>

namespace sc {

constexpr int MAXSIDE = 3;                  // distinct species per reaction side
constexpr int MAXENH = 4;                   // enhanced third-body species per reaction
constexpr int NDEP = 2 * MAXSIDE + MAXENH;  // dependency slots per reaction
constexpr int MAX_STATE = 64;               // N + 1 supported by the dense one-wave kernels
constexpr int MAX_STATE_SPARSE = 128;       // N + 1 supported by the sparse kernels (two components per lane)
constexpr int MAX_SOLVE = 128;              // N + 2 their factorisation and solves hold (two rows per lane)
// widest dense trailing block the level schedule leaves out (sc_mech_sparse_array)
constexpr int SPARSE_TAIL_MAX = 32;
constexpr int SPARSE_TAIL_MAX_WIDE = 64;
constexpr int sparse_tail_max(int n) { return n <= 64 ? SPARSE_TAIL_MAX : SPARSE_TAIL_MAX_WIDE; }
// per-reaction entry indices of the sparse kernels: for each row slot (3
// reactants, 3 products) the entries of its dependency slots and of the
// temperature column, then the temperature row's entries of the dependency
// slots (unused slots hold NOENT)
constexpr int RXI_ROW = NDEP + 1;
constexpr int RXI_TROW = 2 * MAXSIDE * RXI_ROW;
constexpr int RXI_SIZE = RXI_TROW + NDEP + 2;  // 80 (a 160-byte record)
constexpr uint16_t NOENT = 0xffff;

// The sparse linear algebra of one mechanism (paper Sec. 2.5: the sparse
// analytical Jacobian and the sparse algebra management of the mechanism).
// The iteration matrix M = I/(h gamma) - J is solved through a bordered
// system of order n = N + 2 in the scaled unknowns z_k = x_k / W_k, x_T and
// sigma = (sum_m v_m x_m), in which the species block holds only the terms
// P_km = sum_j nu_kj dq_j/dC_m (fixed sparsity from the reaction list, with
// the third-body concentration rewritten so only enhanced species appear),
// and the dense couplings are two border rows and columns (temperature and
// the density term of constant pressure, or the total concentration of
// constant volume).  The species block is put in minimum-degree order, the
// borders last, so no fill enters the species block from them.  The
// symbolic LU (right-looking, no pivoting) fixes the L+U pattern.  The kernels
// read operand tables made from it (SparseDev, SparseRx); the schedule in levels
// of independent operations and the row masks and sweep tables below count the
// work and serve sc_mech_sparse_array, for inspection and tests: no kernel reads
// them.
struct SparseLU {
    int n = 0, nnz = 0;
    std::vector<int> perm;        // position -> variable (species 0..N-1, N = T, N + 1 = sigma)
    std::vector<int> pos;         // variable -> position
    std::vector<int> erow, ecol;  // entry -> (row position, column position), column-major order
    std::vector<int> emap;        // n * n: (row position, column position) -> entry or -1
    std::vector<int> cstart;      // n + 1: first entry of each column
    std::vector<uint64_t> cmask;  // per column two words (three where n > 128), bit i set where row i holds an entry
    // per column k of a system of at most 64 positions, 4 words each: the
    // rows below the diagonal holding an entry (mask low, high word) and the
    // first of those entries (forward sweep); the same for the rows above
    // the diagonal (backward sweep)
    std::vector<uint32_t> sweep_f, sweep_b;
    // n <= 64: per column k and row i (64 rows per column), the entry of
    // (i, k) below (sweep_fi) or above (sweep_bi) the diagonal, else nnz
    std::vector<uint16_t> sweep_fi, sweep_bi;
    std::vector<uint8_t> apat;    // n * n: structural pattern of the bordered matrix (before fill)
    // LU, level by level: scale the L entries of the level's pivots
    // (b items: e_ik | e_kk << 16), then the Schur updates (c items:
    // e_ij | e_ik << 16 | e_kj << 32) whose targets may repeat within a level
    std::vector<int> lu_b_lvl, lu_c_lvl;  // level offsets into b / c items (size levels + 1)
    std::vector<uint32_t> lu_b;
    std::vector<uint64_t> lu_c;
    std::vector<uint32_t> lu_u;           // strict U entries with their pivot: e_kj | k << 16 (row scaling)
    // the dense trailing block [tail0, n) (full L+U pattern, at most
    // sparse_tail_max(n) positions): its pivots are not in the level schedule
    // but eliminated densely after it
    int tail0 = 0;
    std::vector<uint32_t> diag;           // diagonal entry of each position
    // triangular solves (unit L, then the row-scaled unit U): items
    // i | p << 16 | e << 32 meaning x_i -= value(e) x_p, level by level
    std::vector<int> fw_lvl, bw_lvl;
    std::vector<uint64_t> fw, bw;
    // transposed solves (U'^T, then L^T)
    std::vector<int> tfw_lvl, tbw_lvl;
    std::vector<uint64_t> tfw, tbw;
    std::vector<uint16_t> rxi;            // [R][RXI_SIZE] entry indices per reaction, original order
    // entries each state component writes when the matrix is formed: per
    // species k: diagonal, T column, sigma column, T row, sigma row; for T:
    // (T,T), (sigma,sigma), (T,sigma), (sigma,T) (the last two may be absent)
    std::vector<int> e_kk, e_kT, e_kS, e_Tk, e_Sk;
    int e_TT = -1, e_SS = -1, e_TS = -1, e_ST = -1;
    int64_t nnz_a = 0, updates = 0;       // bordered matrix before fill; Schur updates
    int64_t flops_lu = 0, flops_solve = 0;
};

// Entry indices of the sparse kernels' operand tables are 16-bit byte
// offsets into a cell's L+U entries for systems of up to 64 positions (at
// most 64 * 64 entries), entry numbers beyond.
constexpr int sparse_off(int n, int e) { return n <= 64 ? 8 * e : e; }

constexpr int SPARSE_TRASH = 16;  // entries that unused slots of a reaction's record add to

// LDS of one cell in the sparse kernels, in doubles: fixed places first, so
// they are immediate offsets of the LDS instructions, then the L+U entries, the
// zero slot and the trash slots.  C and g/RT, and h/RT and the production
// rate, are pairs: one address and one wide read serve both.
constexpr int SPL_CG = 0, SPL_HW = 2, SPL_UA = 4, SPL_U = 5, SPL_DINV = 9, SPL_E = 10;  // times NV
static_assert(SPL_HW % 2 == 0 && SPL_E % 2 == 0, "pairs and cleared entries are 16-byte accesses");
// Size of that region for `lanes` lanes a cell.  Regions follow each other in a
// workgroup's LDS, so it is even: every pair stays 16-byte aligned.  Several
// cells per wave: half a bank row (16 doubles modulo 32) apart, so that the
// groups' like accesses fall on different banks.
constexpr int sparse_region(int n, int nnz, int lanes)
{
    const int size = SPL_E * lanes * (n <= 64 ? 1 : 2) + nnz + 1 + SPARSE_TRASH;
    return lanes < 64 ? size + (16 - size % 32 + 32) % 32 : size + size % 2;
}

// Waves of a workgroup of the sparse kernels, 1, 2 or 4, for n cells:
// groups[k] workgroups of 2^k waves are resident on the device, at most `limit`
// of them are launched.  With one slot per lane each wave has a cell (and a
// region of LDS) until the last ones are shared, with two the workgroup has one.
// The choice is by the cells in flight at a time, then by the waves: a crew
// gains less on a cell (four waves 1.2 times a step of one-slot mechanisms, two
// 1.1 to 1.3 times of two-slot ones) than a CU loses with its cells.  Regions of
// 20 to 27 KB (57 to 62 species) leave room for one workgroup of four waves, three
// of two or seven of one; regions of 27 to 52 KB (63 to about 89 species) for two
// crews of two or three to four single waves.  4,096 cells, waves by the rule
// against the most that fit: 57 species 63.0 and 77.8 ms, 65 species 105.0 and
// 161.0, 80 species 177 and 198, linear solves of 65 species 0.36 and 0.53 (ms).
constexpr int CREW_SIZES = 3;
// Workgroups of `bytes` each that a CU's LDS holds: 160 KB, given out in pieces
// of 1,280 bytes (three times 54,000 bytes, of 90 species, would fit by the sum,
// but do not: taken for three, 4,096 cells took 280 ms, with crews of two 226)
constexpr int lds_held(size_t bytes) { return (int)(128 / ((bytes + 1279) / 1280)); }
inline int crew_choice(int vpl, const int (&groups)[CREW_SIZES], int64_t limit, int64_t n)
{
    int waves = 1;
    int64_t most = 0;
    for (int k = 0; k < CREW_SIZES; ++k) {
        const int64_t in_flight = std::min(n, std::min<int64_t>(groups[k], limit) << (vpl == 1 ? k : 0));
        if (in_flight > 0 && in_flight >= most) most = in_flight, waves = 1 << k;
    }
    return waves;
}
// A wave of a workgroup of `waves` that finds the queue empty and has no cell,
// w waves working as one (1 until the last cell is handed over): it leaves
// where nobody can hand it a cell any more.  With two slots per lane the
// workgroup works as one from the beginning; with one it waits for the last
// cell first, if there is another wave to bring it.
constexpr bool crew_leaves(int vpl, int w, int waves) { return vpl > 1 || w == waves; }

// What the device reads of a mechanism's sparse algebra (built per plan from
// SparseLU; `lanes` lanes hold one cell's positions, two slots each when
// n > 64).  Absent entries, and rows and columns beyond n, name the zero slot
// (entry nnz).
struct SparseDev {
    // solve operands, per slot, lane and column the entry of the lane's row:
    // the whole row (several cells per wave), or the strictly lower and the
    // strictly upper part (one cell per wave)
    std::vector<uint16_t> row, low, up;
    // factorisation operands (one cell per wave) by block b of 16 pivots, in
    // 16-byte words [word][lane], with c = lane % 16, g = lane / 16 and
    // r = the blocks after b:
    //   2 words   (b c, b k), k = 0..15: the diagonal block, a row per lane
    //   2 words   (b k, b c) where c > k: its upper part, a column per lane
    //   r words   block q: (b c, q 4m + g), m = 0..3, then (q 4m + g, b c)
    //   r words   block q: (q c, b 4s + g), s = 0..3, then (b 4s + g, q c)
    //   r r half words [q1][q2][lane]: (q1 4i + g, q2 c), i = 0..3
    // one block's words after the other's
    std::vector<uint16_t> blk;
    // per component (position order) eight: its entries kk, kT, kS, Tk, Sk, the
    // temperature's TT and SS; trash entries where it has none and behind
    std::vector<uint16_t> comp;
};

enum RxKind { RX_PLAIN = 0, RX_THIRD = 1, RX_TROE = 2 };

struct ParseError : std::runtime_error {
    using std::runtime_error::runtime_error;
};
struct Unsupported : std::runtime_error {
    using std::runtime_error::runtime_error;
};

struct Reaction {
    int kind = RX_PLAIN;
    double log10A = 0, b = 0, Ea = 0;  // cgs log10 A, J/mol
    std::vector<std::pair<int, int>> reac, prod;
    std::vector<std::pair<int, double>> eff;  // (species, efficiency)
    double troe[7] = {0, 0, 0, 0, 0, 0, 0};  // log10 A0, b0, Ea0, a, T3, T1, T2
};

// Device tables in host memory, structure-of-arrays, reaction index fastest.
struct Tables {
    int N = 0, R = 0, n_troe = 0;
    double Rgas = 0, p0 = 0;
    std::vector<double> W, invW, nasa;  // nasa[c*N + k]
    std::vector<int32_t> kind, nr, np, dnu, neff, tix;
    std::vector<int32_t> rsp, rnu, psp, pnu;  // [slot*R + j]
    std::vector<int32_t> esp;                 // [slot*R + j]
    std::vector<double> eam1;                 // alpha - 1, [slot*R + j]
    std::vector<double> lnA, b, EaR;          // SI, log form
    std::vector<double> troe;                 // [field*n_troe + t]: lnA0, b0, Ea0R, a, 1/T3, 1/T1, T2
};

struct Counts {
    int nnz_jac = 0, nnz_lu = 0;
    int exp_per_rhs = 0;
    int64_t flops_rhs = 0, flops_jac = 0, flops_lu = 0, flops_solve = 0, flops_step = 0;
    int64_t flops_attempt = 0, flops_accept = 0;
    int64_t flops_jac_terms = 0;  // the Jacobian pass beyond its right-hand side (reaction derivative terms)
};

struct Mech {
    std::string name;
    int N = 0, R = 0, E = 0;
    double Rgas = 8.314462618, p0 = 101325.0;
    std::vector<std::string> names, elements;
    std::vector<double> W;
    std::vector<int> comp;    // [k*E + e]
    std::vector<double> nasa; // [k*7 + i]
    std::vector<Reaction> rx;
    int n_third = 0, n_troe = 0;
    int n_padded = 0;
    Tables tab;
    Counts cnt;         // the dense kernels' work
    Counts cnt_sparse;  // the sparse kernels' work (LU and solves from the schedule)
    std::vector<uint8_t> pattern;  // N^2 structural pattern of the species terms P_km (with the diagonal)
    SparseLU sp;

    int species(const std::string &s) const;
};

// Parse + validate + compile.  Throws ParseError or Unsupported.
Mech load_mechanism(const std::string &text);

// Interpolation tables of each reaction's -dG/RT and dH/RT in u = ln T
// (thermo_fit.cpp): per interval, reaction and function the d + 1
// coefficients of the polynomial in t in [-1, 1].
constexpr int THERMO_FIT_MAX_DEGREE = 8;
constexpr int THERMO_FIT_MAX_INTERVALS = 4096;
constexpr size_t THERMO_FIT_TABLE_BYTES = 4u << 20;  // the optimal degree's table limit
struct ThermoFit {
    int degree = 0, nint = 0;
    double Tmin = 0, Tmax = 0, u0 = 0, du = 0, max_err = 0;
    std::vector<double> coef;  // [interval][reaction (mechanism order)][2][degree + 1]
};
// degree 0: the lowest degree whose table meets tol within THERMO_FIT_TABLE_BYTES
ThermoFit fit_thermo(const Mech &m, double Tmin, double Tmax, double tol, int degree);

// The sparse compile (sparse.cpp): ordering, symbolic LU, schedules, entry
// indices and counts of a parsed, validated mechanism.
void compile_sparse(Mech &m);

// The device tables of a compiled mechanism for `lanes` lanes per cell.
SparseDev sparse_device(const Mech &m, int lanes);

// The reactions as the sparse kernels read them: `lanes` reactions per pass,
// one per lane, padded with null reactions; every table in 16-byte words,
// word w of a pass at [pass][w][lane], so a load is one contiguous burst.
// Falloff reactions come first, then third-body ones, then the rest, each by
// coefficients and side sizes, so that what only some reactions need is in
// as few passes as can be.  Unused slots name the temperature's place as a
// species (index N: concentration 1, g = h = 0) and trash entries, so the arithmetic has no
// per-lane branches; what a whole pass does not need is skipped by the flags,
// which every record of the pass carries, and a lane adds only for the slots
// in use (coefficient above zero).
constexpr int RXW_WORDS = 3;  // lnA, b, Ea/R; side species (byte offsets, 16 per species); bits; enhanced species; index
constexpr int RXW_IX = 6;     // entries: six rows of six slots and T, then the T row
constexpr int RXW_IXE = 4;    // entries of the enhanced species: six rows of four, then the T row
enum { RXF_THIRD_REAC = 1u << 27, RXF_THIRD_PROD = 1u << 28, RXF_NU = 1u << 29, RXF_TB = 1u << 30, RXF_TROE = 1u << 31 };
struct SparseRx {
    int passes = 0, n_tb = 0, n_troe = 0;
    std::vector<int> order;  // execution position -> reaction
    std::vector<uint32_t> rec;
    std::vector<uint16_t> ix, ixe;
    std::vector<double> eam1, troe;  // per third-body reaction 4 alpha - 1; per falloff reaction 8 (lnA0, b0, Ea0/R, a, 1/T3, 1/T1, T2)
};
SparseRx sparse_reactions(const Mech &m, int lanes);
// and for the dense kernels: species in their own order, entries in the matrix
// of n_padded rows of n_padded + 1 (byte offsets; N + 1 <= MAX_STATE)
SparseRx dense_reactions(const Mech &m);

}  // namespace sc
