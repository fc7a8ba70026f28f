// The seed iterations of a whole block in one launch, for right-hand sides whose direction p
// fits in the LDS of one workgroup.
#include "device_common.h"

#include <utility>

namespace scocg {

// f(0), f(1) ... f(N - 1) with the index a constant in each call: register arrays indexed by it
// never become memory.
template <typename F, int... I>
__device__ inline void unroll_seq(F &f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ inline void unroll(F &&f)
{
    unroll_seq(f, std::make_integer_sequence<int, N>{});
}

// ---------------------------------------------------------------------------------------
// One workgroup per right-hand side runs the block's TB iterations of the five seed kernels
// (k_pupd, k_spmv, k_alpha, k_rupd, k_beta in kernels.hip): p lives in LDS, where the product
// with H gathers it; r and q stay in registers; only the residuals the deferred update needs
// (one vector per iteration) go to memory.  The launches and the kernel boundaries between the
// phases become workgroup barriers that wait on LDS only.
//
// What bounds it: up to 1024 rows the chain of one iteration (gathers, two sums over the rows,
// two complex divisions, three to seven barriers); above, where the matrix does not fit in
// registers, that chain and the latency of its slots, one chunk of which is in flight per wave: with
// 4096 rows of 7 entries (8.5 us an iteration) the waves wait for 56 % of their cycles, the LDS is
// busy for 23 %, the vector units issue for 47 %, and the matrix comes at 40 GB/s; each further
// slot costs 0.148 ns (81 GB/s), so wide rows are left to the launches (seed_block_pays).
// Measured per iteration, five launches against this: 200 rows of up to 17 entries 20 -> 1.7 us,
// 512 rows (cubic 8^3) 20 -> 2.3 us, 4096 rows (cubic 16^3) 16.2 -> 8.5 us for one right-hand side
// and 36 -> 12 us for 300.
//
// Same bits as the five kernels.  Every sum is theirs: a 256-row tile adds entry t + 128 to entry
// t, then t + 64, then 32 ... 1, and the tile partials are added as a tree in the same way.  With
// WPT waves per tile a lane holds the rows l + 64 h + 64 WPT i of its tile (h: the wave within
// the tile), so the two wide levels are additions inside a lane or between the tile's waves and
// the six narrow ones lane moves.  Products and quotients use the rounding of the five
// kernels (cmul_f, cdiv_f, csq_f).
//
// NPAD: rows the instance has room for (256 ... 8192).  W: matrix slots per row a lane keeps in
// registers for the whole block (rows of up to W entries; columns as 16-bit pairs), or 0: the
// slots are read each iteration, the next ones in flight while the last are added.  (Two instances
// spill: <8192, 0> 60 vector registers, 236 bytes of scratch a lane, and <2048, 0> four; the
// first is ahead of the launches all the same, 4.6 against 5.4 ms, see seed_block_holds.)
// ---------------------------------------------------------------------------------------
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Element i of a vector of at most 2^16 rows at a wave-uniform address: the offset stays in 32 bits.
template <typename T>
__device__ inline T *elem(T *p, unsigned i)
{
    return (T *)((char *)const_cast<double2 *>(p) + i * 16u);
}

__device__ inline void set_zero(double &a) { a = 0.0; }
__device__ inline void set_zero(double2 &a) { a = make_double2(0.0, 0.0); }

template <int NPAD, int W>
struct SeedBlock {
    // threads; 512 (256 registers each) where the matrix slots do not fit the 128 of 1024 threads
    static constexpr int NT = NPAD <= 512 ? NPAD : (NPAD == 1024 && W > 12 ? 512 : 1024);
    static constexpr int WAVES = NT / 64;
    static constexpr int RL = NPAD / NT;                        // rows per lane
    static constexpr int WPT = RL >= 4 ? 1 : 4 / RL;            // waves per 256-row tile
    static constexpr int RT = 4 / WPT;                          // rows of one tile per lane
    static constexpr int TPW = RL / RT;                         // tiles per wave
    static constexpr int TILES = NPAD / 256;
    static_assert(NPAD >= 256 && RL * NT == NPAD && TPW * RT == RL && (W == 0 || RL <= 2), "");
};

// A lane's rows of one tile, added as the tile's wide levels do: entry t + 128, then t + 64.
template <typename B, typename T>
struct TileSum {
    T a[B::TPW], b;
    __device__ inline void row(int i, T v)
    {
        const int q = i / B::RT;
        if (i % B::RT == 0) a[q] = v;
        else if (B::RT == 2 || i % B::RT == 2) a[q] = vadd(a[q], v);
        else if (i % B::RT == 1) b = v;
        else a[q] = vadd(a[q], vadd(b, v));
    }
};

// First half of the sum over the rows: the tiles' partials into part (one barrier before they
// may be read).  Where a tile is spread over several waves, tile_share first hands the waves'
// rows on through xb (a barrier between the two).  With a single tile every wave forms its
// partial itself (sum_rows) and part is not used.
template <typename B, typename T>
__device__ inline void tile_share(const TileSum<B, T> &v, T *xb, int wave, int lane)
{
    if (B::WPT > 1) xb[64 * wave + lane] = v.a[0];
}
template <typename B, typename T>
__device__ inline T tile_total(const TileSum<B, T> &v, const T *xb, int wave, int lane)
{
    const int w0 = wave & ~(B::WPT - 1);
    T t = vadd(xb[64 * w0 + lane], xb[64 * (w0 + B::WPT / 2) + lane]);
    if constexpr (B::WPT == 4) t = vadd(t, vadd(xb[64 * (w0 + 1) + lane], xb[64 * (w0 + 3) + lane]));
    return lane_tree(t);
}
template <typename B, bool ALWAYS = false, typename T>
__device__ inline void tile_partials(const TileSum<B, T> &v, const T *xb, T *part, int wave, int lane)
{
    if constexpr (B::WPT == 1) {
#pragma unroll
        for (int q = 0; q < B::TPW; ++q) {
            const T t = lane_tree(v.a[q]);
            if (lane == 0) part[wave + q * B::WAVES] = t;
        }
    } else if ((B::TILES > 1 || ALWAYS) && (wave & (B::WPT - 1)) == 0) {
        const T t = tile_total(v, xb, wave, lane);
        if (lane == 0) part[wave / B::WPT] = t;
    }
}
// Second half: every wave adds the np partials (the tree's levels from np on only add zeros).
template <int TILES, typename T>
__device__ inline T sum_parts(const T *part, int np, int lane)
{
    T x;
    set_zero(x);
    if (lane < np) x = vadd(x, part[lane]);
    return first_lane(lane_tree<TILES>(x));
}
template <typename B, typename T>
__device__ inline T sum_rows(const TileSum<B, T> &v, const T *xb, const T *part, int np, int wave, int lane)
{
    if constexpr (B::TILES == 1) {
        T x;
        set_zero(x);
        return first_lane(vadd(x, tile_total(v, xb, wave, lane)));
    } else {
        return sum_parts<B::TILES>(part, np, lane);
    }
}

template <int NPAD, int W>
__global__ void __launch_bounds__((SeedBlock<NPAD, W>::NT)) k_seed_block(SolveDev s)
{
    using B = SeedBlock<NPAD, W>;
    constexpr int RL = B::RL;
    constexpr int CH = RL >= 4 ? 4 : 8;  // slots read and gathered at once (W = 0)
    constexpr int XB = B::WPT > 1 ? B::NT : 1;
    __shared__ double2 pl[NPAD + 1];  // pl[NPAD] = 0: what the slots past a row's width multiply
    __shared__ double2 xb_a[XB], xb_b[XB];
    __shared__ double xb_n[XB];
    __shared__ double2 part_a[B::TILES], part_b[B::TILES], part_w[B::TILES];
    __shared__ double part_n[B::TILES];
    // With more than one wave per SIMD the totals and the divisions are one wave's work (the others
    // would only repeat them in the same issue slots): alpha, beta and the state go through LDS.
    constexpr bool LEAD = B::WAVES > 4;
    __shared__ double2 sc_alpha, sc_beta;
    __shared__ int sc_status;
    const int64_t j = blockIdx.x;
    SeedState st = s.seed[j];
    if (!seed_running(st, s.TB)) return;
    const RhsDesc d = s.desc[j];
    const int n = (int)d.n;
    const int np = (n + 255) / 256;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // lane row i: tile (wave / WPT) + (i / RT) WAVES / WPT, in it slice (wave % WPT) + (i % RT) WPT
    auto slice_of = [&](int i) -> int {
        return 4 * (wave / B::WPT + (i / B::RT) * (B::WAVES / B::WPT)) + (wave & (B::WPT - 1)) + (i % B::RT) * B::WPT;
    };
    auto row_of = [&](int i) -> unsigned { return (unsigned)(slice_of(i) * 64 + lane); };
    int nl = n;
    auto ok = [&](int i) -> bool { return row_of(i) < (unsigned)nl; };
    const auto *colg = gptr(d.ell_col);
    const auto *valg = gptr(d.ell_val);
    int off[RL], wid[RL];
    // the residual stays in registers (one row per lane) or, up to 4096 rows, in LDS; beyond, p
    // fills the LDS and it is read back from the ring (each lane the rows it wrote)
    constexpr bool RREG = RL == 1, RLDS = RL > 1 && NPAD <= 4096;
    __shared__ double2 rl[RLDS ? NPAD : 1];
    double2 r = make_double2(0.0, 0.0), q[RL];
    const double2 *rg = ring_slot(s, (st.base + st.step) % s.R, d);
    double2 *pg = s.p + p_index(s, j, d, 0);
    const int ps = s.spmv_rb;  // p of row c is pg[ps c]
    double2 po = make_double2(0.0, 0.0);  // one row per lane: its own p, kept beside the LDS copy
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        const int sl = slice_of(i);
        off[i] = 0;
        wid[i] = 0;
        if (sl < (int)d.nslices) {
            off[i] = __builtin_amdgcn_readfirstlane((int)gptr(d.slice_ptr)[sl]);
            wid[i] = __builtin_amdgcn_readfirstlane(gptr(d.slice_w)[sl]);
        }
        const unsigned row = row_of(i);
        if constexpr (RREG) r = ok(i) ? rg[row] : make_double2(0.0, 0.0);
        if constexpr (RLDS) rl[row] = ok(i) ? rg[row] : make_double2(0.0, 0.0);
        po = ok(i) ? pg[(int64_t)ps * row] : make_double2(0.0, 0.0);
        pl[row] = po;
    }
    // `count` slots from entry e of the slices on (at most CH): columns and values.  A slot past
    // the last reads the last one again, so no branch stands between the loads.
    auto fetch = [&](int e, int count, int *c, double *v) {
        if (count <= 0) return;
        unroll<CH>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            const int at = e + 64 * (u < count ? u : count - 1);
            c[u] = (colg + at)[(unsigned)lane];
            v[u] = (valg + at)[(unsigned)lane];
        });
    };
    // W > 0: the whole rows in registers (two rows per lane: a column pair per register)
    constexpr int NS = W > 0 ? W : CH;
    double vr[W > 0 ? RL : 1][NS];
    unsigned cp[W > 0 ? RL : 1][RL == 1 ? NS : (NS + 1) / 2];
    int c0[CH];
    if constexpr (W > 0) {
        unroll<RL>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            unroll<NS>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                // past the slice's width: -0 times p = +0 is -0, and adding -0 leaves every sum as it is
                unsigned c = NPAD;
                vr[i][u] = -0.0;
                if (u < wid[i]) {
                    c = (unsigned)(colg + (off[i] + 64 * u))[(unsigned)lane];
                    vr[i][u] = (valg + (off[i] + 64 * u))[(unsigned)lane];
                }
                if constexpr (RL == 1) cp[i][u] = c;
                else if (u & 1) cp[i][u / 2] |= c << 16;
                else cp[i][u / 2] = c;
            });
        });
    } else {
        fetch(off[0], wid[0], c0, vr[0]);
    }
    // several rows per lane: one or two at a time (all at once they would need more registers)
    auto few_rows = [&](int i) {
        if (RL >= 4 && (i & 1)) __builtin_amdgcn_sched_barrier(0);
    };
    if (threadIdx.x == 0) pl[NPAD] = make_double2(0.0, 0.0);
    while (st.status == SEED_RUNNING && st.step < s.TB) {
        const int t = st.step;
        asm volatile("" : "+s"(nl));  // (likewise the tests of the rows)
        const double2 *ro = ring_slot(s, (st.base + t) % s.R, d);
        double2 *rn = ring_slot(s, (st.base + t + 1) % s.R, d);
        auto res = [&](int i) -> double2 {
            if constexpr (RREG) return r;
            else if constexpr (RLDS) return rl[row_of(i)];
            else return *elem(ro, ok(i) ? row_of(i) : (unsigned)nl - 1u);
        };
        // p <- r + beta p (each lane its own rows; rows past the last stay out of every sum and of
        // the ring, and no column names them)
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const double2 v = cfma(st.beta_prev, RL == 1 ? po : pl[row_of(i)], res(i));
            if (RL == 1) po = v;
            pl[row_of(i)] = v;
            few_rows(i);
        }
        if (s.wproj) {
            TileSum<B, double2> wr;
            // vector projection: s_n = w . r_n
#pragma unroll
            for (int i = 0; i < RL; ++i)
                wr.row(i, ok(i) ? cmul_f(*elem(s.wproj + d.voff, row_of(i)), res(i)) : make_double2(0.0, 0.0));
            if constexpr (B::WPT > 1) {
                tile_share(wr, xb_a, wave, lane);
                lds_barrier();
            }
            tile_partials<B, true>(wr, xb_a, part_w, wave, lane);
        }
        lds_barrier();
        if (s.wproj) {
            const double2 sn = sum_parts<B::TILES>(part_w, np, lane);
            if (threadIdx.x == 0) s.shist[j * s.TB + t] = sn;
        }
        // q = z p - H p and the partials of p.q
        TileSum<B, double2> pq;
        unroll<RL>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            double ax = 0.0, ay = 0.0;
            // opaque, or the tests of all slots are kept in scalar registers over the whole block
            int w = wid[i];
            asm volatile("" : "+s"(w));
            if constexpr (W > 0) {
                double2 pc[NS];
                unroll<NS>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    if constexpr (RL == 1) {
                        pc[u] = pl[cp[i][u]];
                    } else {
                        unsigned w2 = cp[i][u / 2];
                        // (opaque: unpacked once for the whole block they would fill the registers)
                        asm volatile("" : "+v"(w2));
                        pc[u] = pl[u & 1 ? w2 >> 16 : w2 & 0xffffu];
                    }
                });
                unroll<NS>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    ax = fma(vr[i][u], pc[u].x, ax);
                    ay = fma(vr[i][u], pc[u].y, ay);
                });
            } else {
                // the next slots (of this row, the next one, or the first row's for the iteration
                // after) are in flight while these are gathered and added
                constexpr int ni = i < RL - 1 ? i + 1 : 0;
                for (int k = 0;; k += CH) {
                    const bool more = w > k + CH;
                    int c1[CH];
                    double v1[CH];
                    fetch(more ? off[i] + 64 * (k + CH) : off[ni], more ? w - k - CH : wid[ni], c1, v1);
                    if (w > k) {
                        double2 pc[CH];
                        unroll<CH>([&](auto uc) {
                            constexpr int u = decltype(uc)::value;
                            pc[u] = pl[c0[u]];
                        });
                        unroll<CH>([&](auto uc) {
                            constexpr int u = decltype(uc)::value;
                            if (k + u < w) {
                                ax = fma(vr[0][u], pc[u].x, ax);
                                ay = fma(vr[0][u], pc[u].y, ay);
                            }
                        });
                    }
                    unroll<CH>([&](auto uc) {
                        constexpr int u = decltype(uc)::value;
                        c0[u] = c1[u];
                        vr[0][u] = v1[u];
                    });
                    if (!more) break;
                }
            }
            const double2 pr = RL == 1 ? po : pl[row_of(i)];
            q[i] = cfma(st.zs, pr, make_double2(-ax, -ay));
            pq.row(i, keep_if(ok(i), cmul_f(pr, q[i])));
            few_rows(i);
        });
        if constexpr (B::WPT > 1) {
            tile_share(pq, xb_a, wave, lane);
            lds_barrier();
        }
        tile_partials(pq, xb_a, part_a, wave, lane);
        if constexpr (B::TILES > 1) lds_barrier();
        double2 a;
        if (!LEAD || wave == 0) {
            const double2 tot = sum_rows(pq, xb_a, part_a, np, wave, lane);
            if (cis0(tot) || cis0(st.rho)) st.status = SEED_BREAKDOWN;
            a = cdiv_f(st.rho, tot);
            if (LEAD && lane == 0) {
                sc_alpha = a;
                sc_status = st.status;
            }
        }
        if constexpr (LEAD) {
            lds_barrier();
            a = sc_alpha;
            st.status = __builtin_amdgcn_readfirstlane(sc_status);
        }
        if (st.status == SEED_BREAKDOWN) break;
        // r <- r - alpha q into the ring, and the partials of r.r and |r|^2
        TileSum<B, double2> rr;
        TileSum<B, double> nn;
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const double2 v = cfma(make_double2(-a.x, -a.y), q[i], res(i));
            if constexpr (RREG) r = v;
            if constexpr (RLDS) rl[row_of(i)] = v;
            if (ok(i)) *elem(rn, row_of(i)) = v;
            rr.row(i, keep_if(ok(i), csq_f(v)));
            nn.row(i, ok(i) ? cabs2_f(v) : 0.0);
            few_rows(i);
        }
        if constexpr (B::WPT > 1) {
            tile_share(rr, xb_b, wave, lane);
            tile_share(nn, xb_n, wave, lane);
            lds_barrier();
        }
        tile_partials(rr, xb_b, part_b, wave, lane);
        tile_partials(nn, xb_n, part_n, wave, lane);
        if constexpr (B::TILES > 1) lds_barrier();
        if (!LEAD || wave == 0) {
            const double2 rho = sum_rows(rr, xb_b, part_b, np, wave, lane);
            const double rnorm = sqrt(sum_rows(nn, xb_n, part_n, np, wave, lane));
            const double2 beta = cdiv_f(rho, st.rho);
            st.alpha_prev = a;
            st.beta_prev = beta;
            st.rho = rho;
            st.rnorm = rnorm;
            st.iter += 1;
            if (st.iter >= st.limit) st.status = SEED_LIMIT;
            else if (!s.fixed && s.switching && rnorm / st.nb < s.tol) st.status = SEED_PAUSED;
            if (threadIdx.x == 0) {
                s.ahist[j * s.TB + t] = a;
                s.bhist[j * s.TB + t] = beta;
                s.rnhist[j * s.TB + t] = rnorm;
                if (LEAD) {
                    sc_beta = beta;
                    sc_status = st.status;
                }
            }
        }
        if constexpr (LEAD) {
            lds_barrier();
            st.beta_prev = sc_beta;
            st.status = __builtin_amdgcn_readfirstlane(sc_status);
        }
        st.step = t + 1;
    }
    // p for the next block (each lane its own rows, which no other lane writes)
#pragma unroll
    for (int i = 0; i < RL; ++i)
        if (ok(i)) pg[(int64_t)ps * row_of(i)] = RL == 1 ? po : pl[row_of(i)];
    if (threadIdx.x == 0) {
        SeedState *w = s.seed + j;
        w->alpha_prev = st.alpha_prev;
        w->beta_prev = st.beta_prev;
        w->rho = st.rho;
        w->rnorm = st.rnorm;
        w->iter = st.iter;
        w->step = st.step;
        w->status = st.status;
    }
}

template <int NPAD, int W>
static void launch_w(const SolveDev &s, hipStream_t st)
{
    hipLaunchKernelGGL((k_seed_block<NPAD, W>), dim3((unsigned)s.K), dim3(SeedBlock<NPAD, W>::NT), 0, st, s);
}

// Widths of the rows kept in registers: 7 and 17 are those of the cubic and the four-orbital
// diamond lattice, the others take what lies between (unused slots cost a gather each).
template <int NPAD>
static void launch_npad(const SolveDev &s, hipStream_t st)
{
    if constexpr (NPAD <= 2048) {
        if (s.max_w <= 7) return launch_w<NPAD, 7>(s, st);
    }
    if constexpr (NPAD <= 1024) {
        if (s.max_w <= 12) return launch_w<NPAD, 12>(s, st);
        if (s.max_w <= 17) return launch_w<NPAD, 17>(s, st);
    }
    launch_w<NPAD, 0>(s, st);
}

hipError_t launch_seed_block(const SolveDev &s, hipStream_t st)
{
    if (s.has_hub || s.n > SEED_BLOCK_ROWS_MANY) return hipErrorInvalidConfiguration;
    if (s.n <= 256) launch_npad<256>(s, st);
    else if (s.n <= 512) launch_npad<512>(s, st);
    else if (s.n <= 1024) launch_npad<1024>(s, st);
    else if (s.n <= 2048) launch_npad<2048>(s, st);
    else if (s.n <= 4096) launch_npad<4096>(s, st);
    else launch_npad<8192>(s, st);
    return hipGetLastError();
}

}  // namespace scocg
