// line.hip -- the phi-line block preconditioner: its solve, and the PCG
// iteration with it.
#include "kernels.hpp"
#include "stencil_ops.hpp"

#include <algorithm>
#include <cmath>

namespace pot3d {

// ---------------------------------------------------------------------------
// phi-line block preconditioner: z = M^-1 r, where M keeps, for every (i, j)
// row, the diagonal of A and its two periodic azimuthal weights, and drops
// every coupling between rows (a stronger preconditioner than the point
// Jacobi of Sec. 2.3: near the poles the azimuthal weights, which carry
// 1 / sin(theta), dominate the diagonal).
//
// On a uniform phi grid the block of row (i, j) is the circulant
//     d I - w (S + S^-1),   w = pq / dphi,   d = dphi s + 2 w
// (S: the periodic shift by one cell), which factors as
//     (w / mu) (I - mu S) (I - mu S^-1),   mu + 1/mu = d / w,  0 < mu < 1.
// So z = (mu / w) v with two first-order periodic recurrences
//     u_k = r_k + mu u_{k-1},     v_k = u_k + mu v_{k+1}        (k mod np).
// With d / (2 w) = 1 + e, mu = 1 / (1 + e + sqrt(e (2 + e))), free of
// cancellation for small e (pole rows) and large e alike.
//
// One wavefront solves one row.  Lane l owns the run of cells
// [l NB, l NB + n_l), n_l = min(NB, max(0, np - l NB)): the row moves through
// LDS from the coalesced layout (cell 64 q + lane) to these runs and back.
// Each recurrence runs within a lane's run from a zero start, then an
// inclusive scan across the 64 lanes joins the runs: a run is the affine map
// c -> mu^n_l c + E_l (E_l its end value from a zero start), and maps compose
// as (M1, E1) then (M2, E2) = (M1 M2, E1 M2 + E2).  The carry into run l then
// enters its cell t with mu^(t + 1) (forward; mu^(n_l - t) backward).  The
// periodic wrap is closed afterwards: the value that comes round the row is
// the non-periodic end value divided by 1 - mu^np, and it enters every cell
// with its own power of mu (the scan's products give mu^(l NB) and
// mu^(np - (l + 1) NB)).  Every value is FP64; each row reads r once and
// writes z once (16 bytes per unknown in FP64 storage).  Per-workgroup
// partial sums of r.z and r.r follow in fixed order.
//
// The iteration with this preconditioner (line_iteration_kernel) is the one-sweep iteration of the point Jacobi (kernels.hip), in two kernels,
// since a tile that recomputed its neighbours' p_j would have to solve their
// rows again.  Per iteration they move 8 + 24 bytes per unknown (FP64), and x's
// 24 in every other iteration less the p_{j-1} that is there already.
// ---------------------------------------------------------------------------
// m^e for an integer e >= 0 by binary powering.
__device__ __forceinline__ double powi(double m, int e)
{
    double r = 1.0;
    while (e > 0) {
        if (e & 1) r *= m;
        m *= m;
        e >>= 1;
    }
    return r;
}

// Inclusive scans of affine maps c -> M c + E across the 64 lanes, without
// LDS: DPP shifts by 1, 2, 4, 8 inside each 16-lane row, then the rows are
// chained through their composites read out of one lane each.  UP: lane l
// ends with the composite of lanes 0..l applied in order, (M1, E1) then
// (M2, E2) = (M1 M2, E1 M2 + E2).  Down: the composite of lanes l..63 with
// the lanes to the right applied first, (M, F) of l then the rest R =
// (M Mr, F + M Fr).
template <bool UP>
__device__ __forceinline__ void affine_scan(double &M, double &E, int lane)
{
    // Branch-free: a DPP read of a lane that is switched off returns 0, so the
    // shifts must run with every lane on.  A source outside the row reads
    // (0, 0), which the step turns into the identity (1, 0) by adding 1 to M.
    const int rl = lane & 15, row = lane >> 4;
    auto step = [&](double Mo, double Eo, bool ok) {
        E = __builtin_fma(Eo, M, E);
        M = (Mo + (ok ? 0.0 : 1.0)) * M;
    };
    if (UP) {
        { const double Mo = row_shift<0x111>(M), Eo = row_shift<0x111>(E); step(Mo, Eo, rl >= 1); }
        { const double Mo = row_shift<0x112>(M), Eo = row_shift<0x112>(E); step(Mo, Eo, rl >= 2); }
        { const double Mo = row_shift<0x114>(M), Eo = row_shift<0x114>(E); step(Mo, Eo, rl >= 4); }
        { const double Mo = row_shift<0x118>(M), Eo = row_shift<0x118>(E); step(Mo, Eo, rl >= 8); }
        // rows: prefix composites of rows 0, 0-1, 0-2 from lanes 15, 31, 47
        const double m0 = lane_value(M, 15), e0 = lane_value(E, 15);
        const double m1 = lane_value(M, 31), e1 = lane_value(E, 31);
        const double m2 = lane_value(M, 47), e2 = lane_value(E, 47);
        const double p1m = m0 * m1, p1e = __builtin_fma(e0, m1, e1);     // rows 0-1
        const double p2m = p1m * m2, p2e = __builtin_fma(p1e, m2, e2);   // rows 0-2
        const double pm = row == 0 ? 1.0 : row == 1 ? m0 : row == 2 ? p1m : p2m;
        const double pe = row == 0 ? 0.0 : row == 1 ? e0 : row == 2 ? p1e : p2e;
        E = __builtin_fma(pe, M, E);
        M = pm * M;
    } else {
        { const double Mo = row_shift<0x101>(M), Eo = row_shift<0x101>(E); step(Mo, Eo, rl + 1 < 16); }
        { const double Mo = row_shift<0x102>(M), Eo = row_shift<0x102>(E); step(Mo, Eo, rl + 2 < 16); }
        { const double Mo = row_shift<0x104>(M), Eo = row_shift<0x104>(E); step(Mo, Eo, rl + 4 < 16); }
        { const double Mo = row_shift<0x108>(M), Eo = row_shift<0x108>(E); step(Mo, Eo, rl + 8 < 16); }
        // rows: suffix composites of rows 3, 2-3, 1-3 from lanes 48, 32, 16
        const double m3 = lane_value(M, 48), e3 = lane_value(E, 48);
        const double m2 = lane_value(M, 32), e2 = lane_value(E, 32);
        const double m1 = lane_value(M, 16), e1 = lane_value(E, 16);
        const double s2m = m2 * m3, s2e = __builtin_fma(m2, e3, e2);     // rows 2-3
        const double s1m = m1 * s2m, s1e = __builtin_fma(m1, s2e, e1);   // rows 1-3
        const double sm = row == 3 ? 1.0 : row == 2 ? m3 : row == 1 ? s2m : s1m;
        const double se = row == 3 ? 0.0 : row == 2 ? e3 : row == 1 ? s2e : s1e;
        E = __builtin_fma(se, M, E);
        M = sm * M;
    }
}

// The value at position n - 1 of a register array (0 for n = 0), by a
// chain of selects (the index is per lane).
template <int NB>
__device__ __forceinline__ double t_end(const double (&u)[NB], int n)
{
    double v = 0.0;
#pragma unroll
    for (int t = 0; t < NB; ++t) v = (t == n - 1) ? u[t] : v;
    return v;
}

// The forward recurrence over a row, u_k = r_k + mu u_{k-1} (k mod np), u = 0
// past the run's cells.  m_run: mu^n_l; inv_wrap: 1 / (1 - mu^np).
template <int NB>
__device__ __forceinline__ void line_forward(const double (&rv)[NB], double (&u)[NB], double mu, double m_run,
                                             double inv_wrap, int lane, int n_l, int last_lane)
{
    double acc = 0.0;   // the run from a zero start
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        acc = __builtin_fma(mu, acc, rv[t]);
        u[t] = acc;
    }
    double M = m_run, E = t_end(u, n_l);
    affine_scan<true>(M, E, lane);
    // carry into this run (u at cell l NB - 1, non-periodic) and mu^(l NB)
    // (lane 0 reads 0 for both; branch-free, as in affine_scan)
    const double C = shr1(E);
    const double B = shr1(M) + (lane == 0 ? 1.0 : 0.0);
    const double ulast = lane_value(E, last_lane);              // u_{np-1}, non-periodic
    const double cin = __builtin_fma(B, ulast * inv_wrap, C);   // carry plus the wrap
    double pw = mu;
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        u[t] = t < n_l ? __builtin_fma(pw, cin, u[t]) : 0.0;
        pw *= mu;
    }
}

// The backward recurrence, v_k = u_k + mu v_{k+1}, in place, short of the
// carry into the run, which is returned: cell t of it lacks mu^(n_l - t) of it.
template <int NB>
__device__ __forceinline__ double line_backward(double (&u)[NB], double mu, double m_run, double inv_wrap, int lane)
{
    double acc = 0.0;   // the run from a zero end
#pragma unroll
    for (int t = NB - 1; t >= 0; --t) {
        acc = __builtin_fma(mu, acc, u[t]);
        u[t] = acc;
    }
    double M = m_run, F = u[0];
    affine_scan<false>(M, F, lane);
    // v at cell (l + 1) NB (non-periodic) and mu^(np - (l + 1) NB)
    // (lane 63 reads 0 for both; branch-free)
    const double D = shl1(F);
    const double T = shl1(M) + (lane == kWave - 1 ? 1.0 : 0.0);
    const double v0 = lane_value(F, 0);                      // v_0, non-periodic
    return __builtin_fma(T, v0 * inv_wrap, D);               // carry plus the wrap
}

// NB = cells per lane's run, ceil(np / 64) (np in (64 (NB - 1), 64 NB]).  V is
// the storage type of r and z (FP64, or FP32 for the inner iterations of the
// refined mode); the recurrences always run in FP64.  LDS: one row per
// wavefront, cell k at k + k / NB (one slot of padding per run, so that the
// lanes' strided run accesses spread over the banks).
template <int NB, typename V>
__global__ void __launch_bounds__(kThreads)
line_solve_kernel(GridArgs g, const V *__restrict__ rin, V *__restrict__ zout, double *__restrict__ partial)
{
    constexpr int kRowSlots = NB * kWave + kWave;
    __shared__ double rowbuf[kWaves][kRowSlots];
    __shared__ double red[kWaves][2];
    const GPtr<const V> gr = to_global(rin);
    const GPtr<V> gz = to_global(zout);
    const CPtr<const RowCoef> crows = to_const(g.rows);
    const int np = g.np;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double *const row = rowbuf[w];
    const int n_l = min(NB, max(0, np - lane * NB));   // cells of this lane's run
    const int run0 = lane * (NB + 1);                  // LDS slot of the run's first cell
    const int last_lane = (np - 1) / NB;               // the lane that holds cell np - 1
    const double dph = to_global(g.dphi)[0];           // uniform phi: every width is 2 pi / np
    const double ih = to_global(g.ih)[0];
    const long long nrows = (long long)g.nr * g.nt;
    double acc_rz = 0.0, acc_rr = 0.0;

    // r of a row, coalesced (cell 64 q + lane), into registers (storage type)
    auto load_r = [&](long long rw, V (&rq)[NB]) {
        const long long base = rw * g.pitch;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int k = q * kWave + lane;
            rq[q] = k < np ? stream_load(gr + CHK(base + k, g.npad)) : V(0);
        }
    };
    // FP32 storage: the next row's r is loaded under this row's work (the
    // registers it takes leave the occupancy unchanged there; in FP64 they
    // would cost a wavefront per SIMD at 601 cells)
    constexpr bool kPrefetch = sizeof(V) == 4;
    const long long rstride = (long long)gridDim.x * kWaves;
    V rq[NB];
    long long rw = (long long)blockIdx.x * kWaves + w;
    if (kPrefetch && rw < nrows) load_r(rw, rq);
    for (; rw < nrows; rw += rstride) {
        const RowCoef rc = load_row(crows, CHK(rw, nrows));
        const long long base = rw * g.pitch;
        if (!kPrefetch) load_r(rw, rq);
        // r into LDS, then each lane's run into registers
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int k = q * kWave + lane;
            if (k < np) row[CHK(k + k / NB, kRowSlots)] = (double)rq[q];
        }
        if (kPrefetch && rw + rstride < nrows) load_r(rw + rstride, rq);
        wave_sync();
        double rv[NB], u[NB];
#pragma unroll
        for (int t = 0; t < NB; ++t) rv[t] = t < n_l ? row[CHK(run0 + t, kRowSlots)] : 0.0;
        wave_sync();

        const double wgt = rc.pq * ih;                       // azimuthal weight w
        const double e = dph * rc.s / (2.0 * wgt);           // d / (2 w) - 1 > 0
        const double mu = 1.0 / (1.0 + e + sqrt(e * (2.0 + e)));
        const double inv_wrap = 1.0 / (1.0 - powi(mu, np)); // 1 / (1 - mu^np)
        const double m_run = powi(mu, n_l);                  // mu^n_l (1 for an empty run)

        line_forward(rv, u, mu, m_run, inv_wrap, lane, n_l, last_lane);
        const double din = line_backward(u, mu, m_run, inv_wrap, lane);
        const double scale = mu / wgt;
        double pw = mu;
#pragma unroll
        for (int t = NB - 1; t >= 0; --t) {
            if (t < n_l) {
                const double z = scale * __builtin_fma(pw, din, u[t]);
                u[t] = z;
                acc_rz = __builtin_fma(rv[t], z, acc_rz);
                acc_rr = __builtin_fma(rv[t], rv[t], acc_rr);
                pw *= mu;
            }
        }
        // z back through LDS to the coalesced layout
#pragma unroll
        for (int t = 0; t < NB; ++t)
            if (t < n_l) row[CHK(run0 + t, kRowSlots)] = u[t];
        wave_sync();
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int k = q * kWave + lane;
            if (k < np) stream_store(gz + CHK(base + k, g.npad), (V)row[CHK(k + k / NB, kRowSlots)]);
        }
        wave_sync();
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        acc_rz += __shfl_xor(acc_rz, off, kWave);
        acc_rr += __shfl_xor(acc_rr, off, kWave);
    }
    if (lane == 0) {
        red[w][0] = acc_rz;
        red[w][1] = acc_rr;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) t += red[q][threadIdx.x];
        to_global(partial)[CHK((long long)threadIdx.x * gridDim.x + blockIdx.x, 2LL * gridDim.x)] = t;
    }
}

// ---------------------------------------------------------------------------
// The iteration.  With the vectors and scalars of sweep j (SweepVecs, kFinLine):
//   step        z_{j-1} = p_{j-1} - beta_{j-1} p_{j-2},  w = A p_{j-1},
//               z_j = z_{j-1} - alpha_{j-1} M^-1 w,  r_j = M z_j,
//               p_j = z_j + beta_j p_{j-1} (stored), x as in the sweeps;
//               sums r_j.z_j, r_j.r_j and -beta_j p_j.w, which is
//               -beta_j p_{j-1}.A p_j (A is symmetric)
//   curvature   w_j = A p_j; sums p_j.w_j and w_j.M^-1 w_j.
// z_j.w_j is p_j.w_j - beta_j p_{j-1}.w_j.  w.M^-1 w takes the forward
// recurrence only: M^-1 = (mu / w) B^T B with B = (I - mu S)^-1, so it is
// (mu / w) |B w|^2.
//
// A wavefront walks a chunk of g.ci radial layers of one polar row with p of
// layers i - 1, i and i + 1 in registers; it reads the two rows beside from
// memory and needs no other wavefront.  At 151 x 301 x 601 the step without x /
// with x and the curvature take 138 / 207 and 80 us (FP64; FP32 102 / 128 and
// 56), where direction update, r/x update and line pass took 393 together
// (24, 36 and 16 bytes per unknown; now 24 / 40 and 8).  FP64 rows are bound
// by memory, without x at 4.8 TB/s, the curvature by its arithmetic (about 700
// instructions per row).  A wavefront per row in any order, with all four
// rows around it from the caches, took 175 / 240 and 101 us: the caches
// delivered five rows for one at about 10 TB/s.  Rows lent through LDS to the
// workgroup's other wavefronts saved loads but waited for each other: 196 / 242
// and 82 us.
// ---------------------------------------------------------------------------

// What a row's recurrences need besides the row.  A lane works them out for
// one of its wavefront's next 64 layers (a square root, three divisions and
// three powers: a quarter of a solve if every lane did so for every row).
struct LineScalars {
    double mu, inv_wrap, scale, m_full, m_tail;   // scale = mu / w; mu^NB and mu^(cells of the last run)
};

// Cells per lane whose loads a wavefront has in flight together: of the rows
// beside, and of x.
constexpr int kBeside = 10;
template <typename V> constexpr int kXGroup = sizeof(V) == 8 ? 3 : 10;

template <int NB, typename V>
struct LineLds {
    double row[kWaves][NB * kWave + kWave];       // a row on its way to the runs and back; before that p of layer i
    V dph[NB * kWave], ih[NB * kWave + 1];        // widths and azimuthal factors; ih[k] at ih[k + 1]
    double red[kWaves][3];
};

// Wavefronts per SIMD that the registers are held to: as many as a row length
// allows without spilling much.  FP32 steps of 22 to 26 cells per lane spill 20
// to 54 at two and are faster for it (60 x 300 x 1537 refined: 352 us per
// iteration at one, 289 at two).
constexpr int line_waves(int nb, int bytes, bool step)
{
    return nb <= 5 ? 4 : (nb <= 10 ? 3 : (nb <= (bytes == 8 ? 16 : (step ? 26 : 32)) ? 2 : 1));
}

template <int NB, typename V, bool STEP>
__global__ void __launch_bounds__(kThreads, line_waves(NB, sizeof(V), STEP))
line_iteration_kernel(GridArgs g, SweepVecs<V> v)
{
    const CPtr<const DevScalars> csc = to_const(v.sc);
    if (csc->done) return;   // uniform over the workgroup
    __shared__ LineLds<NB, V> lds;
    const int sweep = csc->sweep;
    const V *const pvec = ring_at(v, sweep, STEP ? 1 : 0);
    const GPtr<const V> p = to_global(pvec), gp2 = to_global((const V *)ring_at(v, sweep, 2));
    const GPtr<V> gpn = to_global(ring_at(v, sweep, 0)), gx = to_global(v.x);
    const double alpha = csc->alpha, beta = csc->beta;
    // z_{j-1} = zp p_{j-1} - beta_{j-1} p_{j-2} (zp = 0 in sweep 0, whose p_{-2} is z_0)
    const double bprev = csc->beta_prev, zp = sweep == 0 ? 0.0 : 1.0;
    const bool xskip = v.xmode == 1;
    const V alpha_p = v.xmode == 2 ? (V)csc->alpha_prev : V(0);
    if (STEP && blockIdx.x == 0 && threadIdx.x == 0) {   // the increment x lacks if this is the last sweep
        v.sc->x_lag = xskip ? alpha : 0.0;
        v.sc->x_lag_p = xskip ? (unsigned long long)pvec : 0ull;
    }

    constexpr int kX = kXGroup<V>;
    const int nr = g.nr, nt = g.nt, np = g.np;
    int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double *const row = lds.row[w];
    int n_l = min(NB, max(0, np - lane * NB));         // cells of this lane's run
    const int last_lane = (np - 1) / NB;               // the lane that holds cell np - 1
    const GPtr<const double> gd = to_global(g.dphi), gi = to_global(g.ih);
    const CPtr<const RowCoef> crows = to_const(g.rows);
    const double dph0 = gd[0], ih0 = gi[0];            // uniform phi: M is built on the first cell's width
    for (int k = threadIdx.x; k < NB * kWave; k += kThreads) {
        lds.dph[k] = k < np ? (V)gd[CHK(k, np)] : V(0);
        lds.ih[k + 1] = k < np ? (V)gi[CHK(k, np)] : V(0);
    }
    if (threadIdx.x == 0) lds.ih[0] = (V)gi[np - 1];
    __syncthreads();

    // A cell of this lane; only the last of the NB lies past the row's end in some lanes.
    auto cell = [&](int q) { return q * kWave + lane; };
    auto in = [&](int q) { return q < NB - 1 || cell(q) < np; };
    auto addr = [&](int q) { return q < NB - 1 ? cell(q) : min(cell(q), np - 1); };
    // The cell of the row at `base`: the row's address is uniform, so an
    // access takes it in scalar registers and 32 bits per lane.
    auto at = [&](auto vec, long long base, int q) {
#ifdef POT3D_CHECKED
        return vec + CHK(base + addr(q), g.npad);
#else
        return at_byte(vec + base, (unsigned)addr(q) * (unsigned)sizeof(V));
#endif
    };
    // Keeps the loads that follow behind the work before.
    auto fence = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // The workgroup's items (chunk, group of polar rows; the group fastest): a
    // contiguous share of them per XCD, whose workgroups then walk
    // neighbouring rows side by side.
    const unsigned items = (unsigned)(g.nchunk * g.ntj), nb = gridDim.x, xcd = blockIdx.x % kXcds;
    const unsigned pre = xcd * (nb / kXcds) + min(xcd, nb % kXcds);    // workgroups of the XCDs before
    const unsigned own = nb / kXcds + (xcd < nb % kXcds ? 1u : 0u);    // of this one
    const unsigned it0 = (unsigned)((unsigned long long)items * pre / nb) + blockIdx.x / kXcds;
    const unsigned it1 = (unsigned)((unsigned long long)items * (pre + own) / nb);

    double acc[3] = {0.0, 0.0, 0.0};
    for (unsigned item = it0; item < it1; item += own) {
        const int ic = item / g.ntj;
        const int j = (item - ic * g.ntj) * kWaves + w;
        const bool on = j < nt;
        const int jc = min(j, nt - 1);   // a wavefront past the last row repeats it and keeps nothing
        const int i0 = ic * g.ci, i1 = min(i0 + g.ci, nr);
        auto base_of = [&](int i, int jj) {
            return (long long)min(max(i, 0), nr - 1) * g.plane + (long long)jj * g.pitch;
        };
        LineScalars ls_l{};
        V pm[NB], pc[NB], pn[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            pm[q] = *at(p, base_of(i0 - 1, jc), q);
            pc[q] = *at(p, base_of(i0, jc), q);
            pn[q] = *at(p, base_of(i0 + 1, jc), q);
        }
        for (int i = i0; i < i1; ++i) {
            // What derives from these is worked out again per layer: held over
            // the loop, the addresses and masks spill.
            asm volatile("" : "+v"(lane), "+v"(n_l));
            const RowCoef rc = load_row(crows, CHK((long long)i * nt + jc, (long long)nr * nt));
            const int n = (i - i0) & (kWave - 1);
            if (n == 0) {   // this lane's layer of the next 64
                const GPtr<const RowCoef> rl = to_global(g.rows) + CHK((long long)min(i + lane, nr - 1) * nt + jc, (long long)nr * nt);
                const double wgt = rl->pq * ih0;                    // azimuthal weight w
                const double e = dph0 * rl->s / (2.0 * wgt);        // d / (2 w) - 1 > 0
                const double mu = 1.0 / (1.0 + e + sqrt(e * (2.0 + e)));
                ls_l.mu = mu;
                ls_l.inv_wrap = 1.0 / (1.0 - powi(mu, np));
                ls_l.scale = mu / wgt;
                ls_l.m_full = powi(mu, NB);
                ls_l.m_tail = powi(mu, np - last_lane * NB);
            }
            const double mu = lane_value(ls_l.mu, n), inv_wrap = lane_value(ls_l.inv_wrap, n);
            const double scale = lane_value(ls_l.scale, n), m_full = lane_value(ls_l.m_full, n);
            const double m_tail = lane_value(ls_l.m_tail, n);
            const double m_run = n_l == NB ? m_full : (n_l == 0 ? 1.0 : m_tail);

            // w = A p: the rows beside from memory, the cells beside through LDS
            const long long bjm = base_of(i, max(jc - 1, 0)), bjp = base_of(i, min(jc + 1, nt - 1));
            V wv[NB];
            double sig = 0.0;
            wave_sync();   // y of the last layer is read
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                reinterpret_cast<V *>(row)[cell(q)] = pc[q];
                wv[q] = vfma<V>(-(V)rc.rm, pm[q], (V)rc.s * pc[q]);
            }
            wave_sync();
            const V *const own_p = reinterpret_cast<const V *>(row);
#pragma unroll
            for (int q0 = 0; q0 < NB; q0 += kBeside) {
                V n[kBeside][2];
#pragma unroll
                for (int t = 0; t < kBeside; ++t) {
                    if (q0 + t >= NB) continue;
                    n[t][0] = *at(p, bjm, q0 + t);
                    n[t][1] = *at(p, bjp, q0 + t);
                }
#pragma unroll
                for (int t = 0; t < kBeside; ++t) {
                    const int q = q0 + t;
                    if (q >= NB) continue;
                    const int k = addr(q);
                    const int kl = q == 0 ? (k == 0 ? np - 1 : k - 1) : k - 1;
                    const int kr = q < NB - 1 ? k + 1 : (k == np - 1 ? 0 : k + 1);
                    V u = lds.ih[k] * (pc[q] - own_p[kl]);
                    u = vfma<V>(lds.ih[k + 1], pc[q] - own_p[kr], u);
                    V a = vfma<V>(-(V)rc.rp, pn[q], wv[q]);
                    a = vfma<V>(-(V)rc.tm, n[t][0], a);
                    a = vfma<V>(-(V)rc.tp, n[t][1], a);
                    a = vfma<V>(lds.dph[k], a, (V)rc.pq * u);
                    wv[q] = in(q) ? a : V(0);
                    if (!STEP) sig = __builtin_fma((double)pc[q], (double)wv[q], sig);
                }
                fence();
            }
            if (!STEP && on) acc[0] += sig;
            wave_sync();   // p of layer i is read: the row may carry w

            // coalesced layout -> runs (0 past the row's end in both)
#pragma unroll
            for (int q = 0; q < NB; ++q)
                row[CHK(cell(q) + cell(q) / NB, NB * kWave + kWave)] = (double)wv[q];
            wave_sync();
            double u[NB];
            {
                double rv[NB];
#pragma unroll
                for (int t = 0; t < NB; ++t) rv[t] = row[lane * (NB + 1) + t];
                wave_sync();
                line_forward(rv, u, mu, m_run, inv_wrap, lane, n_l, last_lane);
            }
            if constexpr (!STEP) {
                double t = 0.0;
#pragma unroll
                for (int q = 0; q < NB; ++q) t = __builtin_fma(u[q], u[q], t);
                if (on) acc[1] = __builtin_fma(scale, t, acc[1]);
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    pm[q] = pc[q];
                    pc[q] = pn[q];
                    if (i + 1 < i1) pn[q] = *at(p, base_of(i + 2, jc), q);
                }
            } else {
                const double din = line_backward(u, mu, m_run, inv_wrap, lane);
                double pw = mu;
#pragma unroll
                for (int t = NB - 1; t >= 0; --t) {
                    u[t] = __builtin_fma(pw, din, u[t]);
                    pw = t < n_l ? pw * mu : pw;
                }
                const long long base = base_of(i, jc);
                V p2[NB];
#pragma unroll
                for (int q = 0; q < NB; ++q) p2[q] = stream_load(at(gp2, base, q));
#pragma unroll
                for (int t = 0; t < NB; ++t)
                    row[CHK(lane * (NB + 1) + t, NB * kWave + kWave)] = u[t];
                wave_sync();
                const double as = alpha * scale;
                double z[NB];
#pragma unroll
                for (int q0 = 0; q0 < NB; q0 += kX) {
                    V xv[kX];
#pragma unroll
                    for (int t = 0; t < kX; ++t) {
                        if (q0 + t >= NB) continue;
                        if (!xskip) xv[t] = stream_load(at(gx, base, q0 + t));
                    }
#pragma unroll
                    for (int t = 0; t < kX; ++t) {
                        const int q = q0 + t;
                        if (q >= NB) continue;
                        const double y = row[addr(q) + addr(q) / NB];
                        const double zq = __builtin_fma(-as, y, __builtin_fma(-bprev, (double)p2[q], zp * (double)pc[q]));
                        z[q] = in(q) ? zq : 0.0;
                        const V pj = (V)__builtin_fma(beta, (double)pc[q], zq);
                        if (on && in(q)) {
                            stream_store(at(gpn, base, q), pj);
                            if (!xskip)
                                stream_store(at(gx, base, q), vfma<V>((V)alpha, pc[q], vfma<V>(alpha_p, p2[q], xv[t])));
                            acc[2] = __builtin_fma((double)pj, (double)wv[q], acc[2]);
                        }
                        pm[q] = pc[q];
                        pc[q] = pn[q];
                    }
                    fence();
                }
                // the next layer's p under the last sums
#pragma unroll
                for (int q = 0; q < NB; ++q)
                    if (i + 1 < i1) pn[q] = *at(p, base_of(i + 2, jc), q);
                const double wgt = rc.pq * ih0, d = __builtin_fma(dph0, rc.s, 2.0 * wgt);
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    const double zl = q > 0 ? lane_value(z[q - 1], kWave - 1) : lane_value(z[NB - 1], (np - 1) & (kWave - 1));
                    const double zr = q < NB - 1 ? lane_value(z[q + 1], 0) : lane_value(z[0], 0);
                    const double zm = shr1(z[q]), zq = shl1(z[q]);
                    const bool right = q < NB - 1 ? lane == kWave - 1 : cell(q) >= np - 1;
                    const double rq = __builtin_fma(d, z[q], -wgt * ((lane == 0 ? zl : zm) + (right ? zr : zq)));
                    if (on && in(q)) {
                        acc[0] = __builtin_fma(rq, z[q], acc[0]);
                        acc[1] = __builtin_fma(rq, rq, acc[1]);
                    }
                }
            }
        }
    }
    if (STEP) acc[2] *= -beta;
    constexpr int kSums = STEP ? 3 : 2;
    const int comp[3] = {STEP ? 0 : 2, STEP ? 1 : 4, 3};
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1)
#pragma unroll
        for (int c = 0; c < kSums; ++c) acc[c] += __shfl_xor(acc[c], off, kWave);
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < kSums; ++c) lds.red[w][c] = acc[c];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < kSums; ++c) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) t += lds.red[q][c];
            to_global(v.partial)[CHK((long long)comp[c] * gridDim.x + blockIdx.x, 5LL * gridDim.x)] = t;
        }
}

template <int NB, typename V>
static hipError_t launch_line_nb(int nb, const GridArgs &g, const V *r, V *z, double *partial, int nblocks,
                                 hipStream_t s)
{
    if constexpr (NB > 1) {
        if (nb < NB) return launch_line_nb<NB - 1, V>(nb, g, r, z, partial, nblocks, s);
    }
    line_solve_kernel<NB, V><<<nblocks, kThreads, 0, s>>>(g, r, z, partial);
    return hipGetLastError();
}

template <typename V>
hipError_t launch_line(const GridArgs &g, const V *r, V *z, double *partial, int nblocks, hipStream_t s)
{
    const int nb = (g.np + kWave - 1) / kWave;
    if (nb < 1 || nb > kMaxLineCells / kWave) return hipErrorInvalidValue;
    return launch_line_nb<kMaxLineCells / kWave, V>(nb, g, r, z, partial, nblocks, s);
}
template hipError_t launch_line<double>(const GridArgs &, const double *, double *, double *, int, hipStream_t);
template hipError_t launch_line<float>(const GridArgs &, const float *, float *, double *, int, hipStream_t);

template <int NB, typename V>
static hipError_t launch_iteration_nb(int nb, const GridArgs &g, const SweepVecs<V> &v, hipStream_t s)
{
    if constexpr (NB > 1) {
        if (nb < NB) return launch_iteration_nb<NB - 1, V>(nb, g, v, s);
    }
    line_iteration_kernel<NB, V, true><<<g.nblocks, kThreads, 0, s>>>(g, v);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    line_iteration_kernel<NB, V, false><<<g.nblocks, kThreads, 0, s>>>(g, v);
    return hipGetLastError();
}

template <typename V>
hipError_t launch_line_iteration(const GridArgs &g, const SweepVecs<V> &v, hipStream_t s)
{
    const int nb = (g.np + kWave - 1) / kWave;
    if (nb < 1 || nb > kMaxLineCells / kWave || g.ntj * kWaves < g.nt || (long long)g.nchunk * g.ci < g.nr)
        return hipErrorInvalidValue;
    return launch_iteration_nb<kMaxLineCells / kWave, V>(nb, g, v, s);
}
template hipError_t launch_line_iteration<double>(const GridArgs &, const SweepVecs<double> &, hipStream_t);
template hipError_t launch_line_iteration<float>(const GridArgs &, const SweepVecs<float> &, hipStream_t);

template <int NB, typename V>
static int line_blocks_per_cu_nb(int nb, bool iteration)
{
    if constexpr (NB > 1) {
        if (nb < NB) return line_blocks_per_cu_nb<NB - 1, V>(nb, iteration);
    }
    const void *f = iteration ? reinterpret_cast<const void *>(&line_iteration_kernel<NB, V, true>)
                              : reinterpret_cast<const void *>(&line_solve_kernel<NB, V>);
    int n = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, kThreads, 0) == hipSuccess ? n : 0;
}

template <typename V>
int line_blocks_per_cu(int np, bool iteration)
{
    const int nb = (np + kWave - 1) / kWave;
    if (nb < 1 || nb > kMaxLineCells / kWave) return 0;
    return line_blocks_per_cu_nb<kMaxLineCells / kWave, V>(nb, iteration);
}
template int line_blocks_per_cu<double>(int, bool);
template int line_blocks_per_cu<float>(int, bool);

unsigned line_oob_line() { return read_oob_line(); }

}  // namespace pot3d
