// Krylov-subspace diagonalization (Sec. 3.2, eq. Ham_in_KS) for many unit right-hand sides:
// the three-term recurrence builds each orthonormal basis {K_n} of K_nu(H, |j>), in which H
// is the tridiagonal T with diagonal a_n = <K_n|H|K_n> and off-diagonal b_{n+1} = <K_{n+1}|H|K_n>;
// the local Green's function is then G_jj(z) = [(z - T)^{-1}]_11, evaluated as the continued
// fraction of T.  Per step, for every unfinished right-hand side:
//   w = H K_n - b_n K_{n-1};  a_n = K_n . w;  w <- w - a_n K_n;  b_{n+1} = ||w||;
//   K_{n+1} = w / b_{n+1}  (applied on the fly by the next steps as w * (1 / b_{n+1})).
// Start vectors are unit vectors, so every basis vector is real.  Sums are fixed-order
// (per 256-row tile, then the tiles in index order), so results do not depend on scheduling.
#include <algorithm>

#include "device_common.h"
#include "hubbard_rows.h"
#include "krylov.h"

namespace scocg {

typedef double d4v __attribute__((ext_vector_type(4)));
static_assert(LZ_TILE == WG, "one 256-row tile per workgroup");

// One row of a group of RB interleaved vectors: four doubles (one 32-byte access), or one.
template <int RB> struct LzRow;
template <> struct LzRow<4> {
    typedef d4v T;
};
struct LzOne {
    double v;
    __device__ double &operator[](int) { return v; }
    __device__ double operator[](int) const { return v; }
};
template <> struct LzRow<1> {
    typedef LzOne T;
};

// Tree sums of RB values over the WG threads: wave b returns the sum of value b in its lane 0.
template <int RB>
__device__ inline double block_sum_rb(const double (&v)[RB], double (*sh)[WG])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int b = 0; b < RB; ++b) sh[b][t] = v[b];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    if (wave >= RB) return 0.0;
    const double *x = sh[wave] + lane;
    return lane_tree((x[0] + x[128]) + (x[64] + x[192]));
}

// The sum that sum_tiles gives of at most LZ_FOLD_TILES partials, by one wave (result in lane 0).
__device__ inline double sum_few_tiles(const double *part, int nblk, int lane)
{
    double v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = part[min(lane + 64 * c, nblk - 1)];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = lane + 64 * c < nblk ? 0.0 + v[c] : 0.0;
    return lane_tree((v[0] + v[2]) + (v[1] + v[3]));
}

// Group and tile of a workgroup.  Workgroups go to the 8 XCDs in turn: a row of the grid
// (8 LZ_SET nblk workgroups) takes 8 LZ_SET groups, LZ_SET to an XCD, tile by tile, so an XCD's L2 holds their
// vectors for the gathers and each tile of the matrix is read into it once for LZ_SET groups (256 right-
// hand sides on 16,384 rows, 3.5 MB of matrix: one group after the other 47.5 us, 2 by 2 45.1, 4 by 4
// 44.4).  In the last row fewer groups are left: they are dealt out over all XCDs.
constexpr int LZ_SET = 4;
__device__ inline void lz_place(const LzDev &s, unsigned x, int64_t &g, int64_t &tile)
{
    const int64_t g0 = (int64_t)blockIdx.y * (8 * LZ_SET);
    if (g0 + 8 * LZ_SET <= s.groups) {
        g = g0 + x % (8 * LZ_SET);
        tile = x / (8 * LZ_SET);
    } else {
        const unsigned q = x / (unsigned)s.nblk;
        g = g0 + q;
        tile = x - q * (unsigned)s.nblk;
    }
}

// the state after b_{n+1} = b ended step n
__device__ inline LzRhs lz_next(LzRhs st, double b, int n, int nu)
{
    st.m = n + 1;
    if (n == nu - 1 || b <= LZ_STOP_REL * (fabs(st.a) + st.bprev)) {
        st.done = 1;
    } else {
        st.rb2 = st.rb;
        st.bprev = b;
        st.rb = 1.0 / b;
    }
    return st;
}

// Fixed-order sum of a right-hand side's tile partials by one workgroup (result in thread 0):
// thread t adds partials t, t + WG, ... in order, then the threads' sums as a tree.
__device__ inline double sum_tiles(const double *part, int64_t nblk, double *sh)
{
    double acc = 0;
    int64_t b = threadIdx.x;
    // TILE_LOADS partials in flight per thread (46,010 tiles of the 14-site ring: with 8 in flight
    // the sum took 19 us, 23 round trips; now 9), the last ones, where a loop would wait for each, as
    // well: those past the end are not added.  Up to 256 tiles the plain loop's single load does.
    constexpr int TILE_LOADS = 32;
    for (; b + (TILE_LOADS - 1) * WG < nblk; b += TILE_LOADS * WG) {
        double v[TILE_LOADS];
#pragma unroll
        for (int u = 0; u < TILE_LOADS; ++u) v[u] = part[b + u * WG];
#pragma unroll
        for (int u = 0; u < TILE_LOADS; ++u) acc += v[u];
    }
    for (; nblk > WG && b < nblk; b += 8 * WG) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = b + u * WG < nblk ? part[b + u * WG] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + u * WG < nblk) acc += v[u];
    }
    for (; b < nblk; b += WG) acc += part[b];
    const int t = threadIdx.x;
    sh[t] = acc;
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if (t < h) sh[t] += sh[t + h];
        __syncthreads();
    }
    return sh[0];
}

// w = H K_n - b_n K_{n-1} and the partials of K_n . w, with K_n = w_{n-1} / b_n taken from the vectors of
// the steps before (or the start vector).  UNIT0: step 0
// from unit vectors.  FOLD: the end of step n - 1 (see k_lz_beta) is worked out
// here by every workgroup of the group, wave b for right-hand side b; the first tile's keeps it.
// Bound by memory: three vectors' traffic (w_{n-1}, w_{n-2}, w) besides the matrix, which serves four
// right-hand sides.  256 right-hand sides, 16,384 rows, 18 entries a row: 45 us
// when each gather waited for its own column load; 45 with the loads of three slots together and two
// vectors less to move but 74 registers, 41.7 with 60 (eight waves per SIMD; 2 or 4 slots 42.9 and 45).
template <int RB, bool FOLD, bool UNIT0>
__global__ void __launch_bounds__(WG, 8) k_lz_matvec(LzDev s, int n)
{
    typedef typename LzRow<RB>::T VR;
    __shared__ double sh[RB][WG];
    __shared__ LzRhs sst[RB];
    int64_t g, tile;
    lz_place(s, blockIdx.x, g, tile);
    if (g >= s.groups) return;
    const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (FOLD && n > 0) {
        if (wave < RB) {
            const int64_t j = g * RB + wave;
            LzRhs st = s.st[(int64_t)((n + 1) & 1) * s.K + j];
            double b = 0;
            if (!st.done) {
                b = sqrt(sum_few_tiles(s.part + (s.K + j) * s.nblk, (int)s.nblk, lane));
                if (lane == 0 && tile == 0) s.ab[j * 2 * s.nu + s.nu + n - 1] = b;
                st = lz_next(st, b, n - 1, s.nu);
            }
            if (lane == 0) {
                sst[wave] = st;
                if (tile == 0) s.st[(int64_t)(n & 1) * s.K + j] = st;
            }
        }
    } else if (lane == 0 && wave < RB) {
        sst[wave] = s.st[g * RB + wave];
    }
    __syncthreads();
    double bprev[RB], rb[RB], rb2[RB];
    bool any = false;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const double b0 = first_lane(sst[b].bprev), b1 = first_lane(sst[b].rb), b2 = first_lane(sst[b].rb2);
        const bool run = __builtin_amdgcn_readfirstlane(sst[b].done) == 0;
        bprev[b] = run ? b0 : 0.0;
        rb[b] = run ? b1 : 0.0;
        rb2[b] = run ? b2 : 0.0;
        any = any || run;
    }
    if (!any) return;  // uniform over the workgroup
    const int64_t base = g * s.n;
    // w_{n-1} and w_{n-2}; the start vector stands for w_{-1} with a factor of 1
    const VR *Wp = (const VR *)(RB == 1 && n == 0 ? s.x0 : s.W[(n + 2) % 3]) + base;
    const VR *Wq = (const VR *)(RB == 1 && n == 1 ? s.x0 : s.W[(n + 1) % 3]) + base;
    VR *Wn = (VR *)(s.W[n % 3]) + base;
    const int64_t row = tile * WG + threadIdx.x;
    double dot[RB] = {};
    if (row < s.n) {
        double acc[RB] = {};
        auto entry = [&](int64_t c, double (&x)[RB]) {
            if constexpr (UNIT0) {
#pragma unroll
                for (int b = 0; b < RB; ++b) x[b] = (c == sst[b].j) ? 1.0 : 0.0;
            } else {
                const VR wc = Wp[c];
#pragma unroll
                for (int b = 0; b < RB; ++b) x[b] = wc[b] * rb[b];
            }
        };
        if (s.hub) {
            // the operator's terms in the stored row's column order: the same sums
            hubbard_row_terms(s.hub, row, [&](int64_t c, double v) {
                double x[RB];
                entry(c, x);
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b] = fma(v, x[b], acc[b]);
            });
        } else {
            const int64_t slice = tile * (WG / 64) + wave;
            const int64_t off = s.slice_ptr[slice];
            const int w = s.slice_w[slice];
            const int32_t *colp = s.ell_col + off + lane;
            const double *valp = s.ell_val + off + lane;
            // slots in the stored order, LZ_CHUNK at a time: the next chunk's columns and values are
            // on their way during a chunk's gathers, and the gathers are issued together
            constexpr int LZ_CHUNK = 3;
            int32_t c[LZ_CHUNK];
            double v[LZ_CHUNK];
            auto fetch = [&](int k) {
#pragma unroll
                for (int u = 0; u < LZ_CHUNK; ++u) {
                    const int64_t at = (int64_t)min(k + u, w - 1) * 64;
                    c[u] = colp[at];
                    v[u] = valp[at];
                }
            };
            if (w > 0) fetch(0);
            for (int k = 0; k < w; k += LZ_CHUNK) {
                double x[LZ_CHUNK][RB], vc[LZ_CHUNK];
                const int m = min(w - k, LZ_CHUNK);
#pragma unroll
                for (int u = 0; u < LZ_CHUNK; ++u) {
                    vc[u] = v[u];
                    entry(c[u], x[u]);
                }
                fetch(k + LZ_CHUNK);
#pragma unroll
                for (int u = 0; u < LZ_CHUNK; ++u) {
                    if (u < m) {
#pragma unroll
                        for (int b = 0; b < RB; ++b) acc[b] = fma(vc[u], x[u][b], acc[b]);
                    }
                }
            }
        }
        VR vo, wo;
        if constexpr (UNIT0) {
#pragma unroll
            for (int b = 0; b < RB; ++b) vo[b] = (row == sst[b].j) ? 1.0 : 0.0;
        } else {
            const VR wr = Wp[row];
#pragma unroll
            for (int b = 0; b < RB; ++b) vo[b] = wr[b] * rb[b];
        }
        if (n == 0) {
#pragma unroll
            for (int b = 0; b < RB; ++b) wo[b] = acc[b];
        } else {
            VR vr;
            if (RB > 1 && n == 1) {
#pragma unroll
                for (int b = 0; b < RB; ++b) vr[b] = (row == sst[b].j) ? 1.0 : 0.0;
            } else {
                const VR wq = Wq[row];
#pragma unroll
                for (int b = 0; b < RB; ++b) vr[b] = wq[b] * rb2[b];
            }
#pragma unroll
            for (int b = 0; b < RB; ++b) wo[b] = fma(-bprev[b], vr[b], acc[b]);
        }
        Wn[row] = wo;
        if (RB == 1 && s.acc) s.acc[row] = fma(s.coef[n], vo[0], s.acc[row]);
#pragma unroll
        for (int b = 0; b < RB; ++b) dot[b] = vo[b] * wo[b];
    }
    const double sum = block_sum_rb<RB>(dot, sh);
    if (lane == 0 && wave < RB && sst[wave].done == 0) s.part[(g * RB + wave) * s.nblk + tile] = sum;
}

// The same step for one plain vector on a matrix-free operator whose down-spin blocks fit in LDS: one
// workgroup per up-spin configuration iu stages x = K_n of its block in LDS, where the down-spin hops
// read it; the up-spin hops of iu are the same for the whole block and read contiguous stretches.
// Rows, their terms' order and the 256-row tiles' sums are those of k_lz_matvec (same bits): a
// thread's rows are counted from the start of the block's first tile (RPT rows, NT apart), so a tile
// inside the block is summed here, and of a tile that two blocks share each block leaves its products
// in `edge` for k_lz_edge.
// Bound by the gathers of the up-spin neighbours (one read of the vector per hop from L2 and the
// Infinity Cache).  14-site ring, 7 + 7, 11.8 million rows: 448 us with one row per thread and one term
// at a time, 192 us here (the hops one per lane, taken with readlane, and the tiles' sums in the same
// kernel: 284 us before those two; 224 while the basis vectors were also written out).
template <int RPT>
__global__ void __launch_bounds__(LZ_HUB_THREADS, 8) k_lz_hub(LzDev s, int n)
{
    constexpr int NT = LZ_HUB_THREADS;
    constexpr int HC = RPT == 4 ? 3 : 8 / RPT;             // up-spin hops gathered at once
    constexpr int SC = 8;                                  // down-spin hops read at once
    __shared__ double xl[NT * RPT + 1];  // xl[Dd] = 0 for the fillers
    __shared__ double dots[NT * RPT];
    const LzRhs st = s.st[0];
    if (st.done) return;
    const int64_t iu = hub_block(blockIdx.x, s.hub_Du);
    if (iu >= s.hub_Du) return;
    HubbardOp h = *s.hub;
    h.up_ptr = first_lane(h.up_ptr);
    h.up_hop = first_lane(h.up_hop);
    h.dn_conf = first_lane(h.dn_conf);
    h.dn_slot = first_lane(h.dn_slot);
    h.t = first_lane(h.t);
    h.U = first_lane(h.U);
    h.V = first_lane(h.V);
    h.L = __builtin_amdgcn_readfirstlane(h.L);
    const int nl = __builtin_amdgcn_readfirstlane(h.dn_low), nhi = __builtin_amdgcn_readfirstlane(h.dn_high);
    // a term's value: -t, or +t where bit 31 is set (the sign alone changes); its column's address in
    // LDS drops the bit
    const double mt = -h.t;
    auto dn_val = [&](uint32_t e) -> double {
        const unsigned long long m = (unsigned long long)__double_as_longlong(mt);
        return __longlong_as_double((long long)(m ^ ((unsigned long long)(e & 0x80000000u) << 32)));
    };
    const int Dd = (int)s.hub_Dd;
    const int64_t r0 = iu * Dd;
    const int off = (int)(r0 & (LZ_TILE - 1));  // rows of the first tile before the block
    // w_{n-1} and w_{n-2}; the start vector stands for w_{-1} with a factor of 1
    const double bprev = first_lane(st.bprev), rb = first_lane(st.rb), rb2 = first_lane(st.rb2);
    const double *Wp = n == 0 ? s.x0 : s.W[(n + 2) % 3];
    const double *Wq = (n <= 1 ? s.x0 : s.W[(n + 1) % 3]) + r0;
    double *Wn = s.W[n % 3] + r0;
    // x at `at` rows from row c0 on (wave-uniform c0)
    auto x_of = [&](int64_t c0, unsigned at) -> double { return (Wp + c0)[at] * rb; };
    unsigned id[RPT];
    bool ok[RPT];
    double acc[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int k = (int)threadIdx.x + i * NT - off;
        ok[i] = k >= 0 && k < Dd;
        id[i] = (unsigned)min(max(k, 0), Dd - 1);
        acc[i] = 0.0;
        if (ok[i]) xl[id[i]] = x_of(r0, id[i]);
    }
    // the block's up-spin hops (at most 30), one per lane; those to lower configurations come first
    const int32_t u0 = __builtin_amdgcn_readfirstlane(gptr(h.up_ptr)[iu]);
    const int nh = __builtin_amdgcn_readfirstlane(gptr(h.up_ptr)[iu + 1]) - u0;
    const int hl = (int)(threadIdx.x & 63);
    const uint32_t my_hop = hl < nh ? gptr(h.up_hop)[u0 + hl] : ~0u;
    auto hop = [&](int k) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)my_hop, k); };
    const int usplit = __popcll(__ballot(hl < nh && (int64_t)(my_hop & 0x7fffffffu) < iu));
    const uint32_t cu = (uint32_t)__builtin_amdgcn_readfirstlane((int)gptr(h.up_conf)[iu]);
    auto hop_val = [&](uint32_t e) { return (e >> 31) ? h.t : -h.t; };
    auto up_range = [&](int k0, int k1) {
        for (int k = k0; k < k1; k += HC) {
            double v[HC], x[HC][RPT];
#pragma unroll
            for (int c = 0; c < HC; ++c) {
                if (k + c < k1) {
                    const uint32_t e = hop(k + c);
                    v[c] = hop_val(e);
#pragma unroll
                    for (int i = 0; i < RPT; ++i) x[c][i] = x_of((int64_t)(e & 0x7fffffffu) * Dd, id[i]);
                }
            }
#pragma unroll
            for (int c = 0; c < HC; ++c) {
                if (k + c < k1) {
#pragma unroll
                    for (int i = 0; i < RPT; ++i) acc[i] = fma(v[c], x[c][i], acc[i]);
                }
            }
        }
    };
    if (threadIdx.x == 0) xl[Dd] = 0.0;
    up_range(0, usplit);
    __syncthreads();
    const auto *slot = gptr(h.dn_slot);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const uint32_t cd = gptr(h.dn_conf)[id[i]];
        const int on = __popc(cu & cd);
        const int inter = __popc(cu & ring_next(cu, h.L)) + __popc(cd & ring_next(cd, h.L)) +
                          __popc(cu & ring_next(cd, h.L)) + __popc(cd & ring_next(cu, h.L));
        const double diag = h.U * (double)on + h.V * (double)inter;
        auto dn_range = [&](int m, int m1) {
            for (; m < m1; m += SC) {
                uint32_t e[SC];
#pragma unroll
                for (int c = 0; c < SC; ++c)
                    if (m + c < m1) e[c] = (slot + (m + c) * Dd)[id[i]];
#pragma unroll
                for (int c = 0; c < SC; ++c) {
                    if (m + c >= m1) break;
                    acc[i] = fma(dn_val(e[c]), *(const double *)((const char *)xl + (e[c] << 3)), acc[i]);
                }
            }
        };
        dn_range(0, nl);
        acc[i] = fma(diag, xl[id[i]], acc[i]);
        dn_range(nl, nl + nhi);
        if constexpr (RPT > 1) {
            // one row after the other, not all their loads at once (registers)
            asm volatile("" : "+v"(acc[i])::"memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    up_range(usplit, nh);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        double dot = 0.0;
        if (ok[i]) {
            const double vo = xl[id[i]];
            const double wo = n == 0 ? acc[i] : fma(-bprev, Wq[id[i]] * rb2, acc[i]);
            Wn[id[i]] = wo;
            if (s.acc) {
                double *a = s.acc + r0 + id[i];
                *a = fma(s.coef[n], vo, *a);
            }
            dot = vo * wo;
        }
        dots[threadIdx.x + i * NT] = dot;
    }
    __syncthreads();
    // the block's tiles, one per wave: 0 .. nt - 1 from row r0 - off on
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = (off + Dd + LZ_TILE - 1) / LZ_TILE;
    const bool last = iu == s.hub_Du - 1;
    for (int t = wave; t < nt; t += NT / 64) {
        const double *dt = dots + LZ_TILE * t + lane;
        const double d0 = dt[0], d1 = dt[64], d2 = dt[128], d3 = dt[192];
        const bool head = t == 0 && off > 0, tail = !last && LZ_TILE * (t + 1) > off + Dd;
        if (head || tail) {
            // shared with the block before (after) this one: rows of this block only
            double *e = s.edge + (head ? iu - 1 : iu) * LZ_TILE;
            const double d[4] = {d0, d1, d2, d3};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int k = LZ_TILE * t + lane + 64 * c - off;
                if (k >= 0 && k < Dd) e[lane + 64 * c] = d[c];
            }
        } else {
            const double v = lane_tree((d0 + d2) + (d1 + d3));
            if (lane == 0) s.part[r0 / LZ_TILE + t] = v;
        }
    }
}

// the sums of the tiles that the blocks iu and iu + 1 share, one per wave
__global__ void __launch_bounds__(WG) k_lz_edge(LzDev s)
{
    if (s.st[0].done) return;
    const int lane = threadIdx.x & 63;
    const int64_t iu = (int64_t)blockIdx.x * (WG / 64) + (threadIdx.x >> 6);
    const int64_t end = (iu + 1) * s.hub_Dd;
    if (iu >= s.hub_Du - 1 || (end & (LZ_TILE - 1)) == 0) return;
    const double *e = s.edge + iu * LZ_TILE + lane;
    const double v = lane_tree((e[0] + e[128]) + (e[64] + e[192]));
    if (lane == 0) s.part[end / LZ_TILE] = v;
}

// a_n from the partials of K_n . w
__global__ void __launch_bounds__(WG) k_lz_alpha(LzDev s, int n)
{
    __shared__ double sh[WG];
    const int64_t j = blockIdx.x;
    if (s.st[j].done) return;
    const double a = sum_tiles(s.part + j * s.nblk, s.nblk, sh);
    if (threadIdx.x == 0) {
        s.st[j].a = a;
        s.ab[j * 2 * s.nu + n] = a;
    }
}

// w <- w - a_n K_n and the partials of ||w||^2.  FOLD: a_n (see k_lz_alpha) from the tiles' sums by every
// workgroup.  Bound by memory, two vectors read and one written: 17.5 us for 100 MB at the sizes above
// (5.7 TB/s).
template <int RB, bool FOLD>
__global__ void __launch_bounds__(WG) k_lz_axpy(LzDev s, int n)
{
    typedef typename LzRow<RB>::T VR;
    __shared__ double sh[RB][WG];
    __shared__ LzRhs sst[RB];
    int64_t g, tile;
    lz_place(s, blockIdx.x, g, tile);
    if (g >= s.groups) return;
    const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave < RB) {
        const int64_t j = g * RB + wave;
        LzRhs *st = s.st + (FOLD ? (int64_t)(n & 1) * s.K : 0) + j;
        if (lane == 0) sst[wave] = *st;
        if (FOLD) {
            const double an = sum_few_tiles(s.part + j * s.nblk, (int)s.nblk, lane);
            if (lane == 0 && !sst[wave].done) {
                sst[wave].a = an;
                if (tile == 0) {
                    st->a = an;
                    s.ab[j * 2 * s.nu + n] = an;
                }
            }
        }
    }
    __syncthreads();
    double a[RB], rb[RB];
    bool any = false;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const double a0 = first_lane(sst[b].a), b1 = first_lane(sst[b].rb);
        const bool run = __builtin_amdgcn_readfirstlane(sst[b].done) == 0;
        a[b] = run ? a0 : 0.0;
        rb[b] = run ? b1 : 0.0;
        any = any || run;
    }
    if (!any) return;
    const int64_t base = g * s.n;
    const VR *Wp = (const VR *)(RB == 1 && n == 0 ? s.x0 : s.W[(n + 2) % 3]) + base;
    VR *Wn = (VR *)(s.W[n % 3]) + base;
    const int64_t row = tile * WG + threadIdx.x;
    double nn[RB] = {};
    if (row < s.n) {
        VR v;
        if (RB > 1 && n == 0) {
#pragma unroll
            for (int b = 0; b < RB; ++b) v[b] = (row == sst[b].j) ? 1.0 : 0.0;
        } else {
            const VR wp = Wp[row];
#pragma unroll
            for (int b = 0; b < RB; ++b) v[b] = wp[b] * rb[b];
        }
        VR w = Wn[row];
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            w[b] = fma(-a[b], v[b], w[b]);
            nn[b] = w[b] * w[b];
        }
        Wn[row] = w;
    }
    const double sum = block_sum_rb<RB>(nn, sh);
    if (lane == 0 && wave < RB && sst[wave].done == 0) s.part[(s.K + g * RB + wave) * s.nblk + tile] = sum;
}

// b_{n+1} = ||w||, the end test, and the state for the next step (read from half `from` of st)
__global__ void __launch_bounds__(WG) k_lz_beta(LzDev s, int n, int from)
{
    __shared__ double sh[WG];
    const int64_t j = blockIdx.x;
    const LzRhs st = s.st[from * s.K + j];
    if (!st.done) {
        const double b = sqrt(sum_tiles(s.part + (s.K + j) * s.nblk, s.nblk, sh));
        if (threadIdx.x == 0) {
            s.ab[j * 2 * s.nu + s.nu + n] = b;
            s.st[j] = lz_next(st, b, n, s.nu);
        }
    } else if (from && threadIdx.x == 0) {
        s.st[j] = st;
    }
}

// G[k][r] = [(z_k - T_r)^{-1}]_11 by the continued fraction of T_r, innermost level first
__global__ void __launch_bounds__(WG) k_lz_greens(LzDev s, const double2 *__restrict__ z, int64_t M, int64_t K,
                                                  double2 *__restrict__ G)
{
    const int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (i >= M * K) return;
    const int64_t k = i / K, r = i % K;
    const int m = s.st[r].m;
    const double *a = s.ab + r * 2 * s.nu;
    const double *b = a + s.nu;
    const double2 zk = z[k];
    double2 g = cdiv(cmk(1, 0), cmk(zk.x - a[m - 1], zk.y));
    for (int t = m - 2; t >= 0; --t) {
        const double bb = b[t] * b[t];
        g = cdiv(cmk(1, 0), cmk(zk.x - a[t] - bb * g.x, zk.y - bb * g.y));
    }
    G[k * K + r] = make_double2(s.gscale * g.x, s.gscale * g.y);
}

// Lowest two eigenvalues of the reduced Hamiltonian by bisection on Sturm counts (the number
// of negative pivots of T - x), and the eigenvector of the lowest by inverse iteration with a
// tridiagonal solve.  One thread per right-hand side.
__device__ inline int sturm_count(const double *a, const double *b, int m, double x)
{
    int cnt = 0;
    double d = 1.0;
    for (int t = 0; t < m; ++t) {
        const double off = t > 0 ? b[t - 1] * b[t - 1] : 0.0;
        d = a[t] - x - (t > 0 ? off / d : 0.0);
        if (d == 0.0) d = -1e-300;
        cnt += d < 0.0;
    }
    return cnt;
}

__device__ inline double kth_eigenvalue(const double *a, const double *b, int m, int k, double lo, double hi)
{
    // smallest x with at least k eigenvalues below it
    for (int it = 0; it < 200 && hi - lo > 1e-15 * fmax(1.0, fmax(fabs(lo), fabs(hi))); ++it) {
        const double mid = 0.5 * (lo + hi);
        if (sturm_count(a, b, m, mid) >= k) hi = mid;
        else lo = mid;
    }
    return 0.5 * (lo + hi);
}

__global__ void __launch_bounds__(64) k_lz_lowest(LzDev s, double *eig, double *u, double *scratch)
{
    if (threadIdx.x != 0) return;
    const int64_t j = blockIdx.x;
    const int m = s.st[j].m;
    const double *a = s.ab + j * 2 * s.nu;
    const double *b = a + s.nu;
    double lo = 0, hi = 0;
    for (int t = 0; t < m; ++t) {
        const double r = (t > 0 ? fabs(b[t - 1]) : 0.0) + (t + 1 < m ? fabs(b[t]) : 0.0);
        lo = t == 0 ? a[t] - r : fmin(lo, a[t] - r);
        hi = t == 0 ? a[t] + r : fmax(hi, a[t] + r);
    }
    lo -= 1e-12 * fmax(1.0, fabs(lo));
    hi += 1e-12 * fmax(1.0, fabs(hi));
    const double e0 = kth_eigenvalue(a, b, m, 1, lo, hi);
    const double e1 = m > 1 ? kth_eigenvalue(a, b, m, 2, lo, hi) : e0;
    eig[2 * j] = e0;
    eig[2 * j + 1] = e1;
    // (T - e0) v = w by the tridiagonal elimination, twice from w = 1
    double *v = u + j * s.nu;
    double *cp = scratch + j * s.nu;
    // a pivot that vanishes (the shift is an eigenvalue) is replaced by 1e-14 of the scale:
    // the solve then amplifies the eigenvector by about 1e14, which the normalization removes
    const double tiny = 1e-14 * fmax(1.0, fabs(e0));
    auto guard = [&](double d) { return fabs(d) < tiny ? (d < 0 ? -tiny : tiny) : d; };
    for (int t = 0; t < s.nu; ++t) v[t] = t < m ? 1.0 : 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        double den = guard(a[0] - e0);
        cp[0] = m > 1 ? b[0] / den : 0.0;
        v[0] = v[0] / den;
        for (int t = 1; t < m; ++t) {
            den = guard(a[t] - e0 - b[t - 1] * cp[t - 1]);
            cp[t] = t + 1 < m ? b[t] / den : 0.0;
            v[t] = (v[t] - b[t - 1] * v[t - 1]) / den;
        }
        for (int t = m - 2; t >= 0; --t) v[t] -= cp[t] * v[t + 1];
        double vmax = 0;
        for (int t = 0; t < m; ++t) vmax = fmax(vmax, fabs(v[t]));
        double nn = 0;
        for (int t = 0; t < m; ++t) {
            v[t] /= vmax;
            nn += v[t] * v[t];
        }
        const double inv = 1.0 / sqrt(nn);
        for (int t = 0; t < m; ++t) v[t] *= inv;
    }
}

// ---- single vector on the stored matrix ----
__global__ void __launch_bounds__(WG) k_sv_matvec(SvDev s, const double *__restrict__ x, double *__restrict__ y)
{
    __shared__ double sh[WG];
    const int64_t row = (int64_t)blockIdx.x * WG + threadIdx.x;
    double d = 0;
    if (row < s.n) {
        double acc = 0;
        if (s.hub) {
            hubbard_row_terms(s.hub, row, [&](int64_t c, double v) { acc = fma(v, x[c], acc); });
        } else {
            const int64_t slice = row >> 6;
            const int lane = (int)(row & 63);
            const int64_t off = s.slice_ptr[slice];
            const int w = s.slice_w[slice];
            for (int k = 0; k < w; ++k) {
                const int64_t e = off + (int64_t)k * 64 + lane;
                acc = fma(s.ell_val[e], x[s.ell_col[e]], acc);
            }
        }
        y[row] = acc;
        d = x[row] * acc;
    }
    sh[threadIdx.x] = d;
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) s.part[blockIdx.x] = sh[0];
}

// partials of ||y - E x||^2 (E = scal[0]) into part, or of ||x||^2 and x . ref into part, part + nblk
__global__ void __launch_bounds__(WG) k_sv_resid(SvDev s, const double *__restrict__ x, const double *__restrict__ y)
{
    __shared__ double sh[WG];
    const int64_t row = (int64_t)blockIdx.x * WG + threadIdx.x;
    double d = 0;
    if (row < s.n) {
        const double r = fma(-s.scal[0], x[row], y[row]);
        d = r * r;
    }
    sh[threadIdx.x] = d;
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) s.part[blockIdx.x] = sh[0];
}

__global__ void __launch_bounds__(WG) k_sv_norm_dot(SvDev s, const double *__restrict__ x, const double *__restrict__ ref)
{
    __shared__ double sh[2][WG];
    const int64_t row = (int64_t)blockIdx.x * WG + threadIdx.x;
    double nn = 0, dd = 0;
    if (row < s.n) {
        nn = x[row] * x[row];
        dd = ref ? x[row] * ref[row] : 0.0;
    }
    sh[0][threadIdx.x] = nn;
    sh[1][threadIdx.x] = dd;
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + h];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        s.part[blockIdx.x] = sh[0][0];
        s.part[s.nblk + blockIdx.x] = sh[1][0];
    }
}

// scal[slot] = sum of the nblk partials at part + off (fixed order)
__global__ void __launch_bounds__(WG) k_sv_sum(SvDev s, int64_t off, int slot)
{
    __shared__ double sh[WG];
    const double v = sum_tiles(s.part + off, s.nblk, sh);
    if (threadIdx.x == 0) s.scal[slot] = v;
}

__global__ void __launch_bounds__(WG) k_sv_scale(SvDev s, double *__restrict__ x)
{
    const int64_t row = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (row >= s.n) return;
    const double f = (s.scal[3] < 0 ? -1.0 : 1.0) / sqrt(s.scal[2]);
    x[row] *= f;
}

__global__ void k_to_complex(const double *__restrict__ x, double2 *__restrict__ z, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) z[i] = cmk(x[i], 0.0);
}

__global__ void k_real_part(const double2 *__restrict__ z, double *__restrict__ x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = z[i].x;
}

// ---- fermion operator between Hubbard sectors ----
// Rank of an L-bit pattern among the patterns with the same number of set bits, in
// increasing integer order: sum over its set bits p_0 < p_1 < ... of C(p_t, t + 1).
__device__ inline int64_t pattern_rank(uint32_t s, const int64_t *binom, int L)
{
    int64_t r = 0;
    int t = 0;
    for (int p = 0; p < L; ++p)
        if ((s >> p) & 1u) {
            ++t;
            r += binom[p * (L + 1) + t];
        }
    return r;
}

__global__ void k_zero2(double2 *y, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = cmk(0, 0);
}

__global__ void k_fermion_op(const uint32_t *__restrict__ up, const uint32_t *__restrict__ dn, int64_t Du, int64_t Dd,
                             const int64_t *__restrict__ binom, int L, int n_up, int site, int spin, int create,
                             int64_t Dd_tgt, const double2 *__restrict__ x, double2 *__restrict__ y)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= Du * Dd) return;
    const int64_t iu = r / Dd, idn = r % Dd;
    const uint32_t su = up[iu], sd = dn[idn];
    const uint32_t bit = 1u << site;
    const uint32_t s = spin == 0 ? su : sd;
    const bool occupied = (s & bit) != 0;
    if (occupied == (create != 0)) return;
    // Jordan-Wigner order: all up-spin modes (sites ascending), then all down-spin modes
    const int before = __popc(s & (bit - 1u)) + (spin == 0 ? 0 : n_up);
    const double sg = (before & 1) ? -1.0 : 1.0;
    int64_t k;
    if (spin == 0) k = pattern_rank(su ^ bit, binom, L) * Dd_tgt + idn;
    else k = iu * Dd_tgt + pattern_rank(sd ^ bit, binom, L);
    y[k] = make_double2(sg * x[r].x, sg * x[r].y);
}

hipError_t launch_lanczos_step(const LzDev &s0, int n, hipStream_t st)
{
    LzDev s = s0;
    if (s.rb != 1 && s.rb != LZ_RB) return hipErrorInvalidValue;
    const int64_t groups = s.K / s.rb;
    if (s.nblk > 0x7fffffffLL || groups > 65535 || s.K > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if (s.nblk * groups > 0x7fffffffLL || (s.rb == 1) != (s.x0 != nullptr) || (s.rb == 1 && s.K != 1))
        return hipErrorInvalidValue;
    s.groups = (int32_t)groups;
    const dim3 gv((unsigned)(s.nblk * std::min<int64_t>(groups, 8 * LZ_SET)), (unsigned)((groups + 8 * LZ_SET - 1) / (8 * LZ_SET)));
    // up to LZ_FOLD_TILES tiles the sums are worked out by the kernels that need them: two launches a
    // step instead of four (256 right-hand sides on 16,384 rows: the
    // two sums' launches were 10 of 72 us a step; 95 on 1,176 rows: 22.6 -> 15 us a step)
    if (s.nblk <= LZ_FOLD_TILES) {
        if (s.rb == 1) {
            hipLaunchKernelGGL((k_lz_matvec<1, true, false>), gv, dim3(WG), 0, st, s, n);
            hipLaunchKernelGGL((k_lz_axpy<1, true>), gv, dim3(WG), 0, st, s, n);
        } else {
            if (n == 0) hipLaunchKernelGGL((k_lz_matvec<LZ_RB, true, true>), gv, dim3(WG), 0, st, s, n);
            else hipLaunchKernelGGL((k_lz_matvec<LZ_RB, true, false>), gv, dim3(WG), 0, st, s, n);
            hipLaunchKernelGGL((k_lz_axpy<LZ_RB, true>), gv, dim3(WG), 0, st, s, n);
        }
        if (n == s.nu - 1) hipLaunchKernelGGL(k_lz_beta, dim3((unsigned)s.K), dim3(WG), 0, st, s, n, n & 1);
        return hipGetLastError();
    }
    if (s.edge) {
        if (!s.hub || s.rb != 1 || !lz_hub_fits(s.n, s.hub_Dd) || s.hub_Dd * s.hub_Du != s.n)
            return hipErrorInvalidValue;
        const dim3 gh((unsigned)(8 * hub_stretch(s.hub_Du)));
        const int64_t span = s.hub_Dd + LZ_TILE - 1;  // rows from a block's first tile on, at most
        if (span <= 1024) hipLaunchKernelGGL(k_lz_hub<1>, gh, dim3(LZ_HUB_THREADS), 0, st, s, n);
        else if (span <= 2048) hipLaunchKernelGGL(k_lz_hub<2>, gh, dim3(LZ_HUB_THREADS), 0, st, s, n);
        else hipLaunchKernelGGL(k_lz_hub<4>, gh, dim3(LZ_HUB_THREADS), 0, st, s, n);
        hipLaunchKernelGGL(k_lz_edge, dim3((unsigned)((s.hub_Du + 3) / 4)), dim3(WG), 0, st, s);
    } else if (s.rb == 1) hipLaunchKernelGGL((k_lz_matvec<1, false, false>), gv, dim3(WG), 0, st, s, n);
    else if (n == 0) hipLaunchKernelGGL((k_lz_matvec<LZ_RB, false, true>), gv, dim3(WG), 0, st, s, n);
    else hipLaunchKernelGGL((k_lz_matvec<LZ_RB, false, false>), gv, dim3(WG), 0, st, s, n);
    hipLaunchKernelGGL(k_lz_alpha, dim3((unsigned)s.K), dim3(WG), 0, st, s, n);
    if (s.rb == 1) hipLaunchKernelGGL((k_lz_axpy<1, false>), gv, dim3(WG), 0, st, s, n);
    else hipLaunchKernelGGL((k_lz_axpy<LZ_RB, false>), gv, dim3(WG), 0, st, s, n);
    hipLaunchKernelGGL(k_lz_beta, dim3((unsigned)s.K), dim3(WG), 0, st, s, n, 0);
    return hipGetLastError();
}

hipError_t launch_lanczos_greens(const LzDev &s, const double2 *z, int64_t M, int64_t K_out, double2 *G,
                                 hipStream_t st)
{
    const int64_t total = M * K_out;
    if (total == 0) return hipSuccess;
    if ((total + WG - 1) / WG > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_lz_greens, dim3((unsigned)((total + WG - 1) / WG)), dim3(WG), 0, st, s, z, M, K_out, G);
    return hipGetLastError();
}

hipError_t launch_lanczos_lowest(const LzDev &s, double *eig, double *u, double *scratch, hipStream_t st)
{
    hipLaunchKernelGGL(k_lz_lowest, dim3((unsigned)s.K), dim3(64), 0, st, s, eig, u, scratch);
    return hipGetLastError();
}

hipError_t sv_rayleigh(const SvDev &s, const double *x, double *y, hipStream_t st)
{
    const dim3 g((unsigned)s.nblk);
    hipLaunchKernelGGL(k_sv_matvec, g, dim3(WG), 0, st, s, x, y);
    hipLaunchKernelGGL(k_sv_sum, dim3(1), dim3(WG), 0, st, s, (int64_t)0, 0);
    hipLaunchKernelGGL(k_sv_resid, g, dim3(WG), 0, st, s, x, (const double *)y);
    hipLaunchKernelGGL(k_sv_sum, dim3(1), dim3(WG), 0, st, s, (int64_t)0, 1);
    return hipGetLastError();
}

hipError_t sv_normalize(const SvDev &s, double *x, const double *ref, hipStream_t st)
{
    const dim3 g((unsigned)s.nblk);
    hipLaunchKernelGGL(k_sv_norm_dot, g, dim3(WG), 0, st, s, (const double *)x, ref);
    hipLaunchKernelGGL(k_sv_sum, dim3(1), dim3(WG), 0, st, s, (int64_t)0, 2);
    hipLaunchKernelGGL(k_sv_sum, dim3(1), dim3(WG), 0, st, s, s.nblk, 3);
    hipLaunchKernelGGL(k_sv_scale, g, dim3(WG), 0, st, s, x);
    return hipGetLastError();
}

hipError_t sv_to_complex(const double *x, double2 *z, int64_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_to_complex, dim3((unsigned)((n + WG - 1) / WG)), dim3(WG), 0, st, x, z, n);
    return hipGetLastError();
}

hipError_t sv_real_part(const double2 *z, double *x, int64_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_real_part, dim3((unsigned)((n + WG - 1) / WG)), dim3(WG), 0, st, z, x, n);
    return hipGetLastError();
}

hipError_t launch_fermion_op(const uint32_t *up_src, const uint32_t *dn_src, int64_t Du, int64_t Dd,
                             const int64_t *binom, int L, int n_up, int site, int spin, int create,
                             int64_t Dd_tgt, int64_t D_tgt, const double2 *x, double2 *y, hipStream_t st)
{
    const int64_t D = Du * Dd;
    if ((D + WG - 1) / WG > 0x7fffffffLL || (D_tgt + WG - 1) / WG > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_zero2, dim3((unsigned)((D_tgt + WG - 1) / WG)), dim3(WG), 0, st, y, D_tgt);
    hipLaunchKernelGGL(k_fermion_op, dim3((unsigned)((D + WG - 1) / WG)), dim3(WG), 0, st, up_src, dn_src, Du, Dd, binom, L,
                       n_up, site, spin, create, Dd_tgt, x, y);
    return hipGetLastError();
}

}  // namespace scocg
