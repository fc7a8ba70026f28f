// Krylov-subspace diagonalization on the device (not part of the C ABI): the three-term
// recurrence of many unit right-hand sides' Krylov bases and the local Green's function of
// their reduced Hamiltonians (Sec. 3.2, eq. Ham_in_KS).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace scocg {

struct HubbardOp;

// Right-hand sides per thread of the recurrence: vectors are stored as [K / LZ_RB][n][LZ_RB]
// (the LZ_RB right-hand sides of a group interleaved row by row), so one column and value
// load of the stored matrix serves LZ_RB right-hand sides and their gathers are 32 B.
constexpr int LZ_RB = 4;
// rows per workgroup of the recurrence, one partial sum each
constexpr int LZ_TILE = 256;
// an invariant subspace ends the recurrence: b_{m+1} <= LZ_STOP_REL (|a_m| + b_m)
constexpr double LZ_STOP_REL = 1e-12;

struct LzRhs {
    double bprev;  // b_n of the step in progress (0 before the first)
    double rb;     // 1 / b_n (K_n is the vector of step n - 1 times it; 1 before the first)
    double rb2;    // 1 / b_{n-1}
    double a;      // a_n of the step in progress
    int64_t j;     // row of the unit start vector
    int32_t m;     // steps completed (dimension of the subspace so far)
    int32_t done;  // recurrence finished (nu steps, or an invariant subspace)
};

struct LzDev {
    const HubbardOp *hub;      // matrix-free operator (device), or null for the stored matrix
    const int64_t *slice_ptr;  // stored matrix, 64-row slices (see DevCSR)
    const int32_t *slice_w;
    const int32_t *ell_col;
    const double *ell_val;
    int64_t n;
    int64_t K;     // right-hand sides (padded to groups of rb with finished entries)
    int64_t nblk;  // 256-row tiles, one partial sum each
    int32_t nu;
    int32_t rb;    // right-hand sides interleaved per group: LZ_RB, or 1 (one plain vector)
    int32_t groups;  // K / rb (set by launch_lanczos_step)
    double *W[3];  // unnormalized vectors w of step n at n mod 3: [K / rb][n][rb].  The basis vectors are
                   // not stored: K_n = w_{n-1} / b_n wherever it is read
    double *part;  // [2][K][nblk] partial sums of K_n . w and of ||w||^2
    double *ab;    // [K][2][nu]: a_1..a_m, then b_2..b_{m+1}
    LzRhs *st;     // [2][K]: by parity of the step where the steps' sums are folded, else and at the
                   // end the first one
    const double *x0;    // rb 1: the start vector [n], unit norm; null for the unit vectors e_j (rb LZ_RB)
    double *acc;         // rb 1: null, or [n]: accumulates sum_n coef[n] K_n (the Ritz vector)
    const double *coef;  // [nu] with acc
    double *edge;        // [hub_Du][256] products of the tiles two down-spin blocks share (see
                         // k_lz_hub), or null: the operator's rows one by one
    int64_t hub_Dd, hub_Du;
    double gscale;       // G is scaled by this: 1 for unit start vectors, |b|^2 for a start vector b
};

// The sums of a step are folded into the kernels that need them (krylov.hip: k_lz_matvec, k_lz_axpy)
// up to this many tiles, which one wave sums with four loads per lane.
constexpr int64_t LZ_FOLD_TILES = 256;
constexpr int LZ_HUB_THREADS = 1024;  // of a workgroup of the tiled product

// Operators the tiled product takes (krylov.hip: k_lz_hub): a 256-row tile may touch two down-spin blocks
// at most, a block with its tiles' ends fits four rows per thread, and the sector is beyond the folded
// sums.  Below, its five launches a step lose to the general product's two, most of all where few
// up-spin configurations leave most of the chip idle: 200 steps of 14 sites with 1 + 7 electrons (14
// blocks of 3432) 5.2 ms against 2.9, 11 sites with 1 + 5 (11 of 462) 3.8 against 2.6, 12 sites with
// 2 + 6 (66 of 924) 4.4 against 3.0; above, 13 sites with 2 + 6 (78 of 1716) 4.7 against 5.0 in four
// launches, 14 sites with 3 + 7 (364 of 3432) 8.6 against 13.4.  And a launch
// has fewer than 2^32 threads along x, which 4.5 million blocks (1.3e9 rows at 300 down-spin
// configurations) exceed; the general product has one thread per row.
inline bool lz_hub_fits(int64_t n, int64_t Dd)
{
    if (Dd < 256 || Dd > 4 * 1024 - 255 || (n + LZ_TILE - 1) / LZ_TILE <= LZ_FOLD_TILES) return false;
    return (n / Dd + 7) / 8 * 8 * LZ_HUB_THREADS < (1LL << 32);
}

// Single real vector of n rows on the stored matrix or the matrix-free operator; one partial
// per 256-row tile, summed in fixed order by one workgroup into the device scalars scal[].
struct SvDev {
    const HubbardOp *hub;  // matrix-free operator (device), or null
    const int64_t *slice_ptr;
    const int32_t *slice_w;
    const int32_t *ell_col;
    const double *ell_val;
    int64_t n, nblk;
    double *part;  // [2][nblk]
    double *scal;  // [8] device scalars
};

// one step n (0-based) of the recurrence for every unfinished right-hand side
hipError_t launch_lanczos_step(const LzDev &s, int n, hipStream_t st);
// lowest two eigenvalues of each reduced Hamiltonian (eig [K][2]) and the eigenvector of the
// lowest (u [K][nu], zero past m); scratch [K][nu]
hipError_t launch_lanczos_lowest(const LzDev &s, double *eig, double *u, double *scratch, hipStream_t st);
// y = H x; scal[0] = x . y; then scal[1] = ||y - scal[0] x||^2
hipError_t sv_rayleigh(const SvDev &s, const double *x, double *y, hipStream_t st);
// x <- x / ||x||, with the sign that makes x . ref >= 0 when ref is given; scal[2], scal[3]
hipError_t sv_normalize(const SvDev &s, double *x, const double *ref, hipStream_t st);
// real part to complex and back (n entries)
hipError_t sv_to_complex(const double *x, double2 *z, int64_t n, hipStream_t st);
hipError_t sv_real_part(const double2 *z, double *x, int64_t n, hipStream_t st);
// Fermion operator between Hubbard sectors: y[target(r)] = sign(r) x[r] for every source state
// r with the mode (site, spin) occupied (annihilation) or empty (creation); y is zeroed first.
// up_src/dn_src: the source sector's species patterns; binom: [L+1][L+1] binomial table;
// dn_tgt_count: the target sector's down-spin basis size.
hipError_t launch_fermion_op(const uint32_t *up_src, const uint32_t *dn_src, int64_t Du, int64_t Dd,
                             const int64_t *binom, int L, int n_up, int site, int spin, int create,
                             int64_t Dd_tgt, int64_t D_tgt, const double2 *x, double2 *y, hipStream_t st);
// G[k][r] = [(z_k - T_r)^{-1}]_11 for M shifts z (device) and K right-hand sides
hipError_t launch_lanczos_greens(const LzDev &s, const double2 *z, int64_t M, int64_t K_out, double2 *G,
                                 hipStream_t st);

}  // namespace scocg
