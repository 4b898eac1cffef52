// onchip.hip -- the point-Jacobi PCG of small grids, run by one resident
// kernel whose vectors stay in registers and LDS.
//
// A small grid's sweep is bound by latency, not by bytes: each workgroup
// walks its radial layers one after the other, a finisher runs between the
// sweeps, and the chip is mostly idle (64 x 128 x 256: 39 us per iteration for
// vectors that 256 MB of cache could deliver in 8).  Here one workgroup per compute
// unit owns a box of M layers x 8 polar rows x 64 azimuthal cells (at most)
// for a whole solve: wavefront w holds the column of polar row j0 + w, lane l
// the cell k0 + l of its M layers, with z = D^-1 r, x and v = D^-1 A p in
// registers, and the direction p in LDS, where the polar and azimuthal
// neighbours read it.  Device memory sees the vectors only when a launch
// begins and ends.  512 threads, so that a lane may hold 256 registers: the
// vectors of M = 16 FP64 layers take 96 of them.  Boxes of up to 64 bytes per
// lane and vector keep p and D^-1 in registers too; the taller ones work out
// D^-1 again in every step (holding it spilled x, 26 us per step).
//
// The operator is applied by its factors: with dphi_k, 1/(phi differences) and
// the factors of the polar row folded into five constants per lane,
//   (A p) = face' [a_i (p - p_{i-1}) + a_{i+1} (p - p_{i+1})]
//         + dr_i [c' (p - p_{j-1}) + c'' (p - p_{j+1}) + u' (p - p_{k-1}) + u'' (p - p_{k+1})]
// needs three scalars per layer (the top face's Phi = 0 is a_nr with p = 0
// beyond it), where the row table of the sweeps has six per layer and row; a
// fourth, a_i + a_{i+1}, gives the diagonal in two operations.
// Lanes and layers of a box that lie outside the grid have zero factors, so
// the stencil has no branches: they hold zeros throughout.
//
// The iteration is the one-sweep one (see kernels.hip): in step j
//   z_j = z_{j-1} - alpha_{j-1} v_{j-1},  x_j = x_{j-1} + alpha_{j-1} p_{j-1},
//   p_j = z_j + beta_j p_{j-1},  w_j = A p_j,  v_j = D^-1 w_j
// and, with r = D z, the sums r.z, r.r, p.w, z.w, w.v, from which every
// workgroup forms alpha_j, the predicted r.z and beta_{j+1} for itself.  So a
// step needs one exchange between the workgroups, in which the sums and the
// boundary cells of v travel together: a workgroup keeps z and p of the one-cell ring around
// its box too, and with the ring's v it advances them by the same operations
// as their owner, bit for bit.
//
// The exchange.  A workgroup's boundary v goes to its faces in device memory
// (two sets of them, in turn), packed: as cells of a vector they lay at powers
// of two from each other and took 2.7 us to store at M = 16.  When those
// stores have completed, it posts its five sums as ten 64-bit words, each of
// 32 bits of data and the step's 32-bit number, so that a word that carries
// the awaited number is whole and no flag or counter is needed.  Every
// workgroup polls all workgroups' words, sums them in a fixed order, and then
// reads its ring of v from its neighbours' faces.  All of it is relaxed
// agent-scope atomics, which go past the L2 caches of the XCDs; a fence would
// write those back.  A workgroup can post step j + 2 only after it has seen
// every post of step j + 1, each made after its workgroup had read the words
// and the ring of step j, so two sets in turn suffice.  Two other exchanges
// were slower: sums over groups of 16 workgroups first, so that fewer words
// are polled (1.3 us more per step at 256 workgroups, for the second round
// trip), and sums posted before the stores have completed with a flag for the
// neighbours after them (1 to 2 us).
//
// The closed wall (CLOSED).  The constants are in A's null space there.  b has
// none of their part, but rounding puts some eps |r_0| of it into the residual,
// where no direction reaches it.  Once the rest of the residual is smaller, r.z
// no longer falls, while p.w does, and alpha and p grow without bound: 1.3
// times the iterations to 1e-13 further on, Phi was lost.  (The sweeps'
// operator, a diagonal times p less the neighbours, leaves rounding errors of a
// constant p in p.w, which end that at a residual of 1e-12 to 1e-6.)  So a
// sixth sum, of r, gives the constant that z_j holds, and z_{j+1} is formed
// without it: 45 x 91 x 179 7.4 us per step with it, 7.2 without.
//
// All workgroups of a launch must be on the chip at once.  There are at most
// as many as compute units and each fits one, and the host runs one such
// launch at a time per device; should they still not come together (another
// process's work holds compute units), a wait ends after a time limit and sets a
// flag that the others read while they poll, so that one limit ends them all.
// The launch then reports that it gave up, and the host starts the solve again
// from its inputs, in sweeps (x and the exchange's buffers hold partial work).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "context.hpp"
#include "stencil_ops.hpp"

namespace pot3d {

namespace {

constexpr int kOcWaves = 8;                   // polar rows of a box
constexpr int kOcThreads = kOcWaves * kWave;
constexpr int kOcSums = 5;      // and a sixth with the closed wall
static_assert(kOnchipStop == kWave, "a lane looks at its own word");

// Relaxed agent-scope accesses of the exchange.
template <typename P, typename T>
__device__ __forceinline__ void put_shared(P p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename P>
__device__ __forceinline__ auto get_shared(P p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the 64 lanes in a fixed order, on every lane.
__device__ __forceinline__ double wave_sum(double v)
{
    v += row_shift<0x111>(v);
    v += row_shift<0x112>(v);
    v += row_shift<0x114>(v);
    v += row_shift<0x118>(v);   // lane 15 of each 16-lane row holds the row's sum
    return (lane_value(v, 15) + lane_value(v, 31)) + (lane_value(v, 47) + lane_value(v, 63));
}

template <int M, typename V, int SUMS>
struct OcLds {
    V p[M][kOcWaves + 2][kWave + 2];          // p_j of the box and its ring
    V edge[kOcWaves][2 * M];                  // v of the box's left and right cells
    double acc[SUMS][kOcThreads];             // per-thread sums
    double tot[SUMS];                         // sums over the grid
    double alpha, beta, rho, sigma;           // of this step, for the next
    double rr, relres;
    int k, status, converged, curved, gave_up;
};

// After step j, what the sweeps' finisher does: the convergence test (one
// wavefront), and alpha and beta (another one at the same time).
template <typename L>
__device__ __forceinline__ void test_residual(L &l, int j, double tol, double bnorm, int maxit, int lane)
{
    if (j == 0) return;
    const double rr = l.tot[1], rel = sqrt(rr) / bnorm;
    if (lane != 0) return;
    l.k = j;
    l.rr = rr;
    l.relres = rel;
    l.converged = 1;
    if (!isfinite(rel)) l.status = POT3D_EBREAKDOWN;
    else if (rel <= tol) l.status = POT3D_OK;
    else if (j >= maxit) l.status = POT3D_ENOCONV;
    else l.converged = 0;
}
template <typename L>
__device__ __forceinline__ void next_scalars(L &l, int lane)
{
    const double rho = l.tot[0], sigma = l.tot[2];
    const double alpha = rho / sigma;
    const double rho_next = fma(alpha * alpha, l.tot[4], fma(-2.0 * alpha, l.tot[3], rho));
    const double beta = (rho_next > 0.0 && isfinite(rho_next)) ? rho_next / rho : 0.0;
    if (lane != 0) return;
    l.curved = sigma > 0.0 && isfinite(sigma) ? 1 : 0;
    l.rho = rho;
    l.sigma = sigma;
    l.alpha = alpha;
    l.beta = beta;
}

// Up to `chunk` steps.  seq0: the number before this launch's first step.
template <int M, typename V, bool CLOSED>
__global__ void __launch_bounds__(kOcThreads)
onchip_kernel(OnchipArgs<V> a, int chunk, unsigned seq0, int fresh, long long wait_ticks)
{
    constexpr int kSums = CLOSED ? kOcSums + 1 : kOcSums;
    __shared__ OcLds<M, V, kSums> lds;
    constexpr int NJ = (2 * M + kOcWaves - 1) / kOcWaves;   // polar ring rows per wavefront
    static_assert(2 * M * kOcWaves <= kOcThreads, "azimuthal ring: one cell per thread");
    const CPtr<const DevScalars> csc = to_const(a.sc);
    if (csc->done) return;   // the same for every workgroup

    const int nr = a.nr, nt = a.nt, np = a.np, pitch = a.pitch, nwg = a.nti * a.ntj * a.ntk;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int b = blockIdx.x;
    const int kt = b % a.ntk, jt = (b / a.ntk) % a.ntj, it = b / (a.ntk * a.ntj);
    const int i0 = it * a.ti, j0 = jt * a.tj, k0 = kt * a.tk;
    const int tin = min(a.ti, nr - i0), tjn = min(a.tj, nt - j0), tkn = min(a.tk, np - k0);
    const bool own = w < tjn && lane < tkn;
    const int j = min(j0 + w, nt - 1);
    const unsigned k = min(k0 + lane, np - 1);
    // This lane's cell in layer i0 + m and polar row j + dj of a vector: a scalar
    // base and a 32-bit byte offset.  The lane's part of the offset is made
    // opaque in every step: the compiler would otherwise work out all offsets
    // once and keep them in registers.
    const int planeb = nt * pitch * (int)sizeof(V), rowb = pitch * (int)sizeof(V);
    unsigned lane_off = (unsigned)((i0 * nt + j) * pitch + (int)k) * (unsigned)sizeof(V);
#ifdef POT3D_CHECKED
    auto in_range = [&](unsigned boff) { return (unsigned)CHK(boff / sizeof(V), a.npad) * (unsigned)sizeof(V); };
#else
    auto in_range = [](unsigned boff) { return boff; };
#endif
    auto cell = [&](auto *v, int m, int dj = 0) { return at_byte(to_global(v), in_range(lane_off + (unsigned)(m * planeb + dj * rowb))); };
    const GPtr<const double> gdphi = to_global(a.dphi), gih = to_global(a.ih);
    // the operator's factors of a column (see the top), and the diagonal in a
    // layer, by the same operations wherever the cell is held
    struct Column {
        V face, ct, cp, um, uk, dsum;
    };
    auto column = [&](int jj, unsigned kk) -> Column {
        const CPtr<const OnchipRow> row = to_const(a.polar) + jj;
        const double dph = gdphi[kk];
        Column c{(V)(row->face * dph), (V)(row->cm * dph), (V)(row->cp * dph),
                 (V)(row->q * gih[kk == 0 ? np - 1 : kk - 1]), (V)(row->q * gih[kk]), V(0)};
        c.dsum = (c.ct + c.cp) + (c.um + c.uk);
        return c;
    };
    CPtr<const OnchipLayer> layers = to_const(a.layers);
    auto z_at = [&](V rv, int i, int jj, unsigned kk) -> V {   // z from what a.r holds
        if (!fresh) return rv;
        const Column c = column(jj, kk);
        return rv * recip(vfma<V>((V)layers[i].dr, c.dsum, c.face * (V)layers[i].sum));
    };
    Column c = column(j, k);
    const V dface = own ? c.face : V(1), dsum = own ? c.dsum : V(1);   // a positive diagonal on every lane
    if (!own) c.face = c.ct = c.cp = c.um = c.uk = V(0);

    // this lane's p in LDS: layer m of its own cell at lp[own_p + m * kLpLayer] (opaque like lane_off)
    V *const lp = &lds.p[0][0][0];
    constexpr int kLpRow = kWave + 2, kLpLayer = (kOcWaves + 2) * kLpRow;
    int own_p = (w + 1) * kLpRow + lane + 1;

    // the box: z, x, p, v = D^-1 A p of this lane's M cells
    constexpr bool kPreg = sizeof(V) * M <= 64;   // p and 1/diag in registers too
    V z[M], x[kPreg ? M : 1], p[kPreg ? M : 1], v[M], inv[kPreg ? M : 1];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const bool on = own && m < tin;
        z[m] = on ? z_at(*cell(a.r, m), i0 + m, j, k) : V(0);
        if constexpr (kPreg) x[m] = on ? *cell(a.x, m) : V(0);
        if constexpr (kPreg) p[m] = on ? *cell(a.p, m) : V(0);
        v[m] = on && !fresh ? *cell(a.v, m) : V(0);
        if constexpr (kPreg) inv[m] = recip(vfma<V>((V)layers[i0 + m].dr, dsum, dface * (V)layers[i0 + m].sum));
        __builtin_amdgcn_sched_barrier(0);
    }
    // the ring: cells below and above the box in this lane's column ...
    const bool lo_on = own && i0 > 0, hi_on = own && i0 + tin < nr;
    V z_lo = lo_on ? z_at(*cell(a.r, -1), i0 - 1, j, k) : V(0), p_lo = lo_on ? *cell(a.p, -1) : V(0);
    V z_hi = hi_on ? z_at(*cell(a.r, tin), i0 + tin, j, k) : V(0), p_hi = hi_on ? *cell(a.p, tin) : V(0);
    // ... polar ring rows in turn over the wavefronts: M rows before the box's
    // first polar row, M after its last (wavefront w: rows w, w + 8, ..)
    auto j_side = [&](int n) { return M >= kOcWaves ? n >= NJ / 2 : w >= M; };
    auto j_layer = [&](int n) { return M >= kOcWaves ? w + kOcWaves * (n % (NJ > 1 ? NJ / 2 : 1)) : w % M; };
    auto j_row = [&](int n) { return j_side(n) ? j0 + tjn : j0 - 1; };
    auto j_on = [&](int n) {
        return w + n * kOcWaves < 2 * M && j_layer(n) < tin && j_row(n) >= 0 && j_row(n) < nt && lane < tkn;
    };
    auto c_j = [&](auto *v, int n) { return cell(v, j_layer(n), j_row(n) - j); };
    auto l_j = [&](int n) { return own_p + j_layer(n) * kLpLayer + ((j_side(n) ? tjn : -1) - w) * kLpRow; };
    V z_j[NJ];
#pragma unroll
    for (int n = 0; n < NJ; ++n)
        z_j[n] = j_on(n) ? z_at(*c_j(a.r, n), i0 + j_layer(n), j_row(n), k) : V(0);
    // ... and the azimuthal ring cells (wrapping in phi), at most one per thread
    const int kside = tid >= M * kOcWaves, ke = kside ? tid - M * kOcWaves : tid;
    const int km = ke % M, kcol = min(ke / M, kOcWaves - 1);
    const unsigned kk = kside ? (k0 + tkn >= np ? 0 : k0 + tkn) : (k0 == 0 ? np - 1 : k0 - 1);
    const bool k_on = tid < 2 * M * kOcWaves && km < tin && kcol < tjn;
    const unsigned o_k = (unsigned)CHK((min(i0 + km, nr - 1) * nt + min(j0 + kcol, nt - 1)) * pitch + kk, a.npad) * (unsigned)sizeof(V);
    const unsigned l_k = (unsigned)((km * (kOcWaves + 2) + kcol + 1) * (kWave + 2) + (kside ? tkn + 1 : 0));
    V z_k = k_on ? z_at(*at_byte(to_global(a.r), o_k), min(i0 + km, nr - 1), min(j0 + kcol, nt - 1), kk) : V(0);

    for (int c = tid; c < M * (kOcWaves + 2) * (kWave + 2); c += kOcThreads) lp[c] = V(0);
    if (tid == 0) {
        lds.rr = csc->rr;
        lds.relres = csc->relres;
        lds.k = csc->k;
        lds.status = csc->status;
        lds.converged = 0;
        lds.gave_up = 0;
    }
    __syncthreads();
    if constexpr (!kPreg) {
        if (own)
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (m < tin) lp[own_p + m * kLpLayer] = *cell(a.p, m);
    }
#pragma unroll
    for (int n = 0; n < NJ; ++n)
        if (j_on(n)) lp[l_j(n)] = *c_j(a.p, n);
    if (k_on) lp[l_k] = *at_byte(to_global(a.p), o_k);

    // scalars of the recurrence, uniform (committed once a step is known not to end the solve)
    double s_alpha = csc->alpha, s_beta = csc->beta, s_rho = csc->rho, s_sigma = csc->sigma;
    V alpha = (V)s_alpha, beta = (V)s_beta;
    V shift = V(0);   // closed wall: the constant that z_j holds (see the top)
    auto advanced = [&](V zz, V vv, V by) -> V { return vfma<V>(-alpha, vv, CLOSED ? zz - by : zz); };   // z_{j+1}
    const double tol = csc->tol, bnorm = csc->bnorm;
    const int maxit = csc->maxit;
    int sweep = csc->sweep;
    bool stop = false;
    unsigned seq = seq0;
    layers += i0;

    // v of the ring: none before the first step, from a.v when a launch goes on,
    // then from the neighbours' faces of step seq
    V v_lo = V(0), v_hi = V(0), v_j[NJ], v_k = V(0);
#pragma unroll
    for (int n = 0; n < NJ; ++n) v_j[n] = V(0);
    if (!fresh) {
        if (lo_on) v_lo = *cell(a.v, -1);
        if (hi_on) v_hi = *cell(a.v, tin);
#pragma unroll
        for (int n = 0; n < NJ; ++n)
            if (j_on(n)) v_j[n] = *c_j(a.v, n);
        if (k_on) v_k = *at_byte(to_global(a.v), o_k);
    }
    // faces of workgroup g in step s: [2][8][64] below and above, [2][M][64]
    // south and north, [2][8][M] left and right
    constexpr int kFaceJ = 2 * kOcWaves * kWave, kFaceK = kFaceJ + 2 * M * kWave;
    auto faces = [&](unsigned s, int g) { return to_global(a.faces) + CHK((s & 1) * nwg + g, 2 * nwg) * onchip_faces(M); };
    // base + c1 + c2 ..: a place among the n from base (summed up otherwise, the
    // addresses took more registers and M = 16 0.6 us more per step)
    auto within = [](int n, auto base, auto... c) {
#ifdef POT3D_CHECKED
        return base + CHK((c + ...), n);
#else
        (void)n;
        return (base + ... + c);
#endif
    };
    constexpr int kFaces = onchip_faces(M), kWords = 2 * kOnchipMaxWg;
    // The stop words lie behind the sums, which so need one address less per lane
    // (10 x 20 x 40 3.34 us per step against 3.64, 45 x 91 x 179 7.1 against 7.2
    // and with the closed wall 7.4 against 7.7); boxes of 16 layers have them in
    // front (64 x 128 x 256 11.6 us against 11.7, FP32 8.6 against 8.9).
    constexpr int kFirstStop = M == 16 ? 0 : kWords, kFirstSum = M == 16 ? kOnchipStop : 0;
    const int step_i = a.ntk * a.ntj;
    const int g_k = kside ? (kt + 1 < a.ntk ? b + 1 : b + 1 - a.ntk) : (kt > 0 ? b - 1 : b + a.ntk - 1);
    auto fetch_ring = [&]() {
        asm volatile("" : "+v"(lane_off), "+v"(own_p));
        if (lo_on) v_lo = get_shared(within(kFaces, faces(seq, b - step_i), (kOcWaves + w) * kWave, lane));
        if (hi_on) v_hi = get_shared(within(kFaces, faces(seq, b + step_i), w * kWave, lane));
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
            const int far = j_side(n) ? 0 : M;   // the north neighbour's first row, or the south one's last
            if (j_on(n)) v_j[n] = get_shared(within(kFaces, faces(seq, j_side(n) ? b + a.ntk : b - a.ntk), kFaceJ, (far + j_layer(n)) * kWave, lane));
        }
        if (k_on) v_k = get_shared(within(kFaces, faces(seq, g_k), kFaceK, ((kside ? 0 : kOcWaves) + kcol) * M, km));
    };

    for (int step = 0; step < chunk; ++step) {
        // z and p of the box, then of the ring with the v fetched at the last step's end
        // (x of the tallest FP64 boxes is this lane's alone in memory, where it
        // stays in the XCD's L2: eight layers at a time)
        constexpr int MB = kPreg ? M : 8;
        if (own) {
#pragma unroll
            for (int mb = 0; mb < M; mb += MB) {
                V xm[MB];
#pragma unroll
                for (int u = 0; u < MB; ++u) xm[u] = kPreg ? x[kPreg ? mb + u : 0] : *cell(a.x, min(mb + u, tin - 1));
#pragma unroll
                for (int u = 0; u < MB; ++u) {
                    const int m = mb + u;
                    const V p0 = kPreg ? p[kPreg ? m : 0] : lp[own_p + m * kLpLayer];
                    xm[u] = vfma<V>(alpha, p0, xm[u]);
                    z[m] = advanced(z[m], v[m], m < tin ? shift : V(0));   // zeros above the grid
                    const V pn = vfma<V>(beta, p0, z[m]);
                    if constexpr (kPreg) {
                        p[m] = pn;
                        x[m] = xm[u];
                    } else {
                        if (m < tin) *cell(a.x, m) = xm[u];
                    }
                    lp[own_p + m * kLpLayer] = pn;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        z_lo = advanced(z_lo, v_lo, shift);
        p_lo = vfma<V>(beta, p_lo, z_lo);
        z_hi = advanced(z_hi, v_hi, shift);
        p_hi = vfma<V>(beta, p_hi, z_hi);
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
            z_j[n] = advanced(z_j[n], v_j[n], shift);
            if (j_on(n)) lp[l_j(n)] = vfma<V>(beta, lp[l_j(n)], z_j[n]);
        }
        z_k = advanced(z_k, v_k, shift);
        if (k_on) lp[l_k] = vfma<V>(beta, lp[l_k], z_k);
        __syncthreads();

        // w = A p on the box, v's boundary to the faces, and the sums
        ++seq;
        // the layers' scalars are read again in every step: held across the
        // steps they would not fit the scalar registers
        asm volatile("" : "+s"(layers), "+v"(lane_off), "+v"(own_p));
        double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0, acc4 = 0.0, acc5 = 0.0;
        V pim = p_lo, pc = kPreg ? p[0] : lp[own_p];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const V pip = m + 1 == M ? p_hi : kPreg ? p[kPreg && m + 1 < M ? m + 1 : 0] : lp[own_p + (m + 1) * kLpLayer];
            const int c0 = own_p + m * kLpLayer;
            const V pjm = lp[c0 - kLpRow], pjp = lp[c0 + kLpRow], pkm = lp[c0 - 1], pkp = lp[c0 + 1];
            const V dr = (V)layers[m].dr;
            V t = (V)layers[m].lo * (pc - pim);
            t = vfma<V>((V)layers[m].hi, pc - pip, t);
            V u = c.ct * (pc - pjm);
            u = vfma<V>(c.cp, pc - pjp, u);
            u = vfma<V>(c.um, pc - pkm, u);
            u = vfma<V>(c.uk, pc - pkp, u);
            const V ap = vfma<V>(dr, u, c.face * t);
            const V d = vfma<V>(dr, dsum, dface * (V)layers[m].sum), r = d * z[m];
            v[m] = ap * (kPreg ? inv[kPreg ? m : 0] : recip(d));
            acc0 = __builtin_fma((double)r, (double)z[m], acc0);
            acc1 = __builtin_fma((double)r, (double)r, acc1);
            acc2 = __builtin_fma((double)pc, (double)ap, acc2);
            acc3 = __builtin_fma((double)z[m], (double)ap, acc3);
            acc4 = __builtin_fma((double)v[m], (double)ap, acc4);
            if constexpr (CLOSED) acc5 += (double)r;
            pim = pc;
            pc = pip;
            if (m & 1) __builtin_amdgcn_sched_barrier(0);   // loads no further ahead: registers
        }
        const GPtr<V> face = faces(seq, b);
        if (own) {
            put_shared(within(kFaces, face, w * kWave, lane), v[0]);
            if (tin == M) put_shared(within(kFaces, face, (kOcWaves + w) * kWave, lane), v[M - 1]);   // else nothing lies above
#pragma unroll
            for (int side = 0; side < 2; ++side)
                if (w == (side ? tjn - 1 : 0)) {
#pragma unroll
                    for (int m = 0; m < M; ++m) put_shared(within(kFaces, face, kFaceJ, (side * M + m) * kWave, lane), v[m]);
                }
            // left and right: gathered in LDS, so that they go out as whole lines
#pragma unroll
            for (int side = 0; side < 2; ++side)
                if (lane == (side ? tkn - 1 : 0)) {
#pragma unroll
                    for (int m = 0; m < M; ++m) lds.edge[w][side * M + m] = v[m];
                }
        }
        wave_sync();
        if (w < tjn && lane < 2 * M) {
            const int side = lane >= M;
            put_shared(within(kFaces, face, kFaceK, (side * kOcWaves + w) * M, lane - side * M), lds.edge[w][lane]);
        }
        lds.acc[0][tid] = acc0;
        lds.acc[1][tid] = acc1;
        lds.acc[2][tid] = acc2;
        lds.acc[3][tid] = acc3;
        lds.acc[4][tid] = acc4;
        if constexpr (CLOSED) lds.acc[kSums - 1][tid] = acc5;
        // this wavefront's boundary stores are complete before the workgroup posts
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();

        if (w < kSums) {   // wavefront c posts, awaits and sums component c
            double part = 0.0;
#pragma unroll
            for (int u = 0; u < kOcWaves; ++u) part += lds.acc[w][u * kWave + lane];
            part = wave_sum(part);
            // records of 16 bytes, two words each: lane pairs store and read them whole
            unsigned long long *words = a.words + ((seq & 1) * kSums + w) * kOnchipSums + kFirstSum;
            const unsigned long long tag = (unsigned long long)seq << 32;
            if (lane < 2) put_shared(within(kWords, words, 2 * b, lane), tag | (unsigned)(lane ? __double2hiint(part) : __double2loint(part)));
            bool late = false;
            auto await = [&](auto loads) -> double {   // loads: reads of 64 words that cover the records
                constexpr int NW = decltype(loads)::value;
                unsigned long long got[NW];
                const long long t0 = wall_clock64();
                for (int n = 1;; ++n) {
                    bool ok = true;
#pragma unroll
                    for (int u = 0; u < NW; ++u) {
                        got[u] = tag;
                        if (u * kWave + lane < 2 * nwg) got[u] = get_shared(within(kWords, words, u * kWave, lane));
                    }
#pragma unroll
                    for (int u = 0; u < NW; ++u) ok = ok && (unsigned)(got[u] >> 32) == seq;
                    if (__all(ok)) break;
                    if ((n & 15) == 0 || wait_ticks == 0) {   // bounded: see the top
                        const bool stopped = __any(get_shared(words + (kFirstStop - kFirstSum) + lane) != 0);
                        late = stopped | (wall_clock64() - t0 >= wait_ticks);
                    }
                    if (late) break;
                }
                double s = 0.0;
#pragma unroll
                for (int u = 0; u < NW; ++u) {
                    const int mine = (int)(unsigned)got[u], other = __builtin_amdgcn_mov_dpp(mine, 0xB1, 0xF, 0xF, true);
                    s += (lane & 1) ? 0.0 : __hiloint2double(other, mine);   // the lane to the right holds the high half
                }
                return wave_sum(s);
            };
            const double s = nwg <= kWave ? await(std::integral_constant<int, 2>()) : await(std::integral_constant<int, 8>());
            if (lane == 0) {
                lds.tot[w] = s;
                if (late) lds.gave_up = 1;
            }
        }
        __syncthreads();
        if (lds.gave_up) {   // the same for the whole workgroup
            if (tid == 0) put_shared(&a.sc->gave_up, 1);
            if (tid < 2 * kSums) put_shared(a.words + tid * kOnchipSums + kFirstStop, 1ull);
            return;
        }
        fetch_ring();   // in flight under the scalars
        if (w == 0) next_scalars(lds, lane);
        if (w == 1) test_residual(lds, sweep, tol, bnorm, maxit, lane);
        ++sweep;
        __syncthreads();
        stop = lds.converged != 0;
        if (!stop) {
            s_rho = wave_uniform(lds.rho);
            s_sigma = wave_uniform(lds.sigma);
            if (lds.curved) {
                s_alpha = wave_uniform(lds.alpha);
                s_beta = wave_uniform(lds.beta);
                alpha = (V)s_alpha;
                beta = (V)s_beta;
                if constexpr (CLOSED) shift = (V)(wave_uniform(lds.tot[kSums - 1]) * a.inv_dsum);
            } else {
                stop = true;
                if (tid == 0) lds.status = POT3D_EBREAKDOWN;
            }
        }
        if (stop) break;
    }

    // The vectors back to memory.  A solve that goes on needs all of them; one
    // that has stopped x, and beta_k p_{k-1} = p_k - z_k for a refined segment
    // that continues this direction.
    if (own) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if (m >= tin) continue;
            if constexpr (kPreg) *cell(a.x, m) = x[m];
            const V pm = kPreg ? p[kPreg ? m : 0] : lp[own_p + m * kLpLayer];
            if (stop) {
                *cell(a.p, m) = pm - z[m];
            } else {
                *cell(a.r, m) = CLOSED ? z[m] - shift : z[m];
                *cell(a.p, m) = pm;
                *cell(a.v, m) = v[m];
            }
        }
    }
    if (b == 0 && tid == 0) {
        DevScalars *sc = a.sc;
        sc->rho = s_rho;
        sc->sigma = s_sigma;
        sc->rr = lds.rr;
        sc->relres = lds.relres;
        sc->alpha = s_alpha;
        sc->beta = s_beta;
        sc->k = lds.k;
        sc->sweep = sweep;
        sc->x_lag = 0.0;
        sc->x_lag_p = 0ull;
        if (stop) {
            sc->status = lds.status;
            sc->done = 1;
        }
    }
}

// The kernel of a plan; NULL: none for these boxes.
template <typename V, bool CLOSED>
auto onchip_form(int m) -> void (*)(OnchipArgs<V>, int, unsigned, int, long long)
{
    switch (m) {
    case 1: return onchip_kernel<1, V, CLOSED>;
    case 2: return onchip_kernel<2, V, CLOSED>;
    case 4: return onchip_kernel<4, V, CLOSED>;
    case 8: return onchip_kernel<8, V, CLOSED>;
    case 16: return onchip_kernel<16, V, CLOSED>;
    default: return nullptr;
    }
}
template <typename V>
auto onchip_form(int m, bool closed)
{
    return closed ? onchip_form<V, true>(m) : onchip_form<V, false>(m);
}

}  // namespace

template <typename V>
hipError_t launch_onchip(const OnchipArgs<V> &a, int m, bool closed, int chunk, unsigned seq0, int fresh,
                         long long wait_ticks, hipStream_t s)
{
    const int nwg = a.nti * a.ntj * a.ntk;
    const auto kernel = onchip_form<V>(m, closed);
    if (!kernel || nwg < 1 || nwg > kOnchipMaxWg || a.ti != m || a.tj > kOcWaves || a.tk > kWave)
        return hipErrorInvalidValue;
    kernel<<<nwg, kOcThreads, 0, s>>>(a, chunk, seq0, fresh, wait_ticks);
    return hipGetLastError();
}
template hipError_t launch_onchip<double>(const OnchipArgs<double> &, int, bool, int, unsigned, int, long long,
                                          hipStream_t);
template hipError_t launch_onchip<float>(const OnchipArgs<float> &, int, bool, int, unsigned, int, long long,
                                         hipStream_t);

unsigned onchip_oob_line() { return read_oob_line(); }

namespace host {

// Boxes of the fewest layers, up to 8, that take at most 64 workgroups;
// otherwise of the fewest that take at most one per compute unit.  A step is
// one lane's chain of layers plus an exchange that grows with the workgroups:
// 32 x 64 x 128 took 5.4 us per step with 64 workgroups of 8 layers or 128 of 4,
// 6.0 with 256 of 2 and 9.0 with 32 of 16; 16 x 60 x 120 4.7 with 64 of 4, 5.0
// with 32 of 8 and 5.1 with 128 of 2; 45 x 91 x 179 7.2 with 216 of 8 and 10.2
// with 108 of 16.  (Its sweeps take 32 and 42 us.)
OnchipPlan plan_onchip(const pot3d_ctx *c)
{
    OnchipPlan o;
    if (env_int("POT3D_ONCHIP", 1) == 0) return o;
    // a launch shape asked of the sweeps is for the sweeps
    for (const char *name : {"POT3D_SWEEP_ROWS", "POT3D_SWEEP_TJ", "POT3D_SWEEP_TK", "POT3D_SWEEP_CI", "POT3D_SWEEP_X",
                             "POT3D_TARGET_BLOCKS_S", "POT3D_REVERSE_S"})
        if (std::getenv(name)) return o;
    o.closed = c->upper_bc == POT3D_UPPER_CLOSED_WALL;
    const int slots = std::min(kOnchipMaxWg, c->num_cu);
    o.ntj = (c->nt + kOcWaves - 1) / kOcWaves;
    o.ntk = (c->np + kWave - 1) / kWave;
    const long long cols = (long long)o.ntj * o.ntk;
    const int only = env_int("POT3D_ONCHIP_M", 0);
    auto smallest = [&](int most, long long wgs) {
        for (int m : {1, 2, 4, 8, 16})
            if (m <= most && (only == 0 || m == only) && cols * ((c->nr + m - 1) / m) <= wgs) return m;
        return 0;
    };
    o.m = smallest(8, std::min(64, slots));
    if (!o.m) o.m = smallest(kOnchipMaxLayers, slots);
    if (o.m) {
        const void *f = c->precision == POT3D_FP32_REFINED ? reinterpret_cast<const void *>(onchip_form<float>(o.m, o.closed))
                                                           : reinterpret_cast<const void *>(onchip_form<double>(o.m, o.closed));
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kOcThreads, 0) != hipSuccess || per_cu < 1) o.m = 0;
    }
    if (!o.m) return o;
    // only the top box may hold fewer layers than the kernel's M: nothing lies beyond those
    o.ti = o.m;
    o.nti = (c->nr + o.ti - 1) / o.ti;
    o.tj = (c->nt + o.ntj - 1) / o.ntj;
    o.ntj = (c->nt + o.tj - 1) / o.tj;
    o.tk = (c->np + o.ntk - 1) / o.ntk;
    o.ntk = (c->np + o.tk - 1) / o.tk;
    o.face_bytes = 2 * (size_t)(o.nti * o.ntj * o.ntk) * onchip_faces(o.m) *
                   (c->precision == POT3D_FP32_REFINED ? sizeof(float) : sizeof(double));
    onchip_place(o, c->nr, c->nt, nullptr);   // bytes
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, c->device) != hipSuccess || khz <= 0) khz = 100000;
    // an exchange takes microseconds; two seconds without one means that the workgroups are not all running
    const int wait_us = std::max(0, env_int("POT3D_ONCHIP_WAIT_US", 2000000));
    o.wait_ticks = (long long)(khz * 1e-3 * wait_us);
    // 64 waits: where launches never come together, trying costs less than 2 % of the time
    const int retry_ms = env_int("POT3D_ONCHIP_RETRY_MS", -1);
    o.retry_s = retry_ms >= 0 ? 1e-3 * retry_ms : 64e-6 * wait_us;
    return o;
}

void onchip_place(OnchipPlan &o, int nr, int nt, void *base)
{
    auto padded = [](size_t n) { return (n + 255) & ~size_t(255); };
    const size_t layers = padded(kOnchipWords * sizeof(*o.words));
    const size_t polar = layers + padded(((size_t)nr + kOnchipMaxLayers) * sizeof(OnchipLayer));
    const size_t faces = polar + padded((size_t)nt * sizeof(OnchipRow));
    o.bytes = faces + o.face_bytes;
    if (!base) return;
    char *const b = static_cast<char *>(base);
    o.words = reinterpret_cast<unsigned long long *>(b);
    o.layers = reinterpret_cast<OnchipLayer *>(b + layers);
    o.polar = reinterpret_cast<OnchipRow *>(b + polar);
    o.faces = b + faces;
}

void onchip_tables(OnchipPlan &o, int nr, int nt, int np, const double *rf, const double *tf, const double *ih,
                   int upper_bc, OnchipLayer *layers, OnchipRow *polar)
{
    auto mid = [](const double *f, int q) { return 0.5 * (f[q] + f[q + 1]); };
    for (int i = nr; i < nr + kOnchipMaxLayers; ++i) layers[i] = OnchipLayer{0.0, 0.0, 0.0, 1.0};
    for (int i = 0; i < nr; ++i) {
        const double top = upper_bc == POT3D_UPPER_SOURCE_SURFACE ? rf[nr] * rf[nr] / (rf[nr] - mid(rf, nr - 1)) : 0.0;
        layers[i].lo = i == 0 ? 0.0 : rf[i] * rf[i] / (mid(rf, i) - mid(rf, i - 1));
        layers[i].hi = i == nr - 1 ? top : rf[i + 1] * rf[i + 1] / (mid(rf, i + 1) - mid(rf, i));
        layers[i].dr = rf[i + 1] - rf[i];
        layers[i].sum = layers[i].lo + layers[i].hi;
    }
    for (int j = 0; j < nt; ++j) {
        const double sj = std::sin(mid(tf, j)), dt = tf[j + 1] - tf[j];
        polar[j].face = sj * dt;
        polar[j].cm = j > 0 ? std::sin(tf[j]) / (mid(tf, j) - mid(tf, j - 1)) : 0.0;
        polar[j].cp = j < nt - 1 ? std::sin(tf[j + 1]) / (mid(tf, j + 1) - mid(tf, j)) : 0.0;
        polar[j].q = dt / sj;
    }
    // the diagonal summed over the cells, by its factors (the phi widths add up to 2 pi)
    double width = 0.0, coupling = 0.0, face = 0.0, polar_c = 0.0, azimuthal = 0.0, inverse = 0.0;
    for (int i = 0; i < nr; ++i) width += layers[i].dr, coupling += layers[i].sum;
    for (int j = 0; j < nt; ++j) face += polar[j].face, polar_c += polar[j].cm + polar[j].cp, azimuthal += polar[j].q;
    for (int k = 0; k < np; ++k) inverse += ih[k];
    o.inv_dsum = 1.0 / (kTwoPi * (face * coupling + width * polar_c) + 2.0 * width * azimuthal * inverse);
}

std::mutex &onchip_lock(int device)
{
    static std::mutex locks[64];
    return locks[device & 63];
}

// By device: when resident launches may be tried again (steady clock, seconds).
static std::atomic<double> &onchip_closed_until(int device)
{
    static std::atomic<double> until[64];
    return until[device & 63];
}

static double steady_seconds()
{
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

bool onchip_open(int device) { return steady_seconds() >= onchip_closed_until(device).load(); }

void onchip_gave_up(int device, const OnchipPlan &plan)
{
    std::atomic<double> &until = onchip_closed_until(device);
    const double t = steady_seconds() + plan.retry_s;
    for (double was = until.load(); was < t && !until.compare_exchange_weak(was, t);) {}
}

template <typename V>
static int queue_with(pot3d_ctx *c, V *r, V *x, V *p, V *v, V *faces, DevScalars *sc, int chunk, bool fresh, hipStream_t s)
{
    OnchipPlan &o = c->oc;
    OnchipArgs<V> a{c->nr, c->nt, c->np, c->pitch, o.ti, o.tj, o.tk, o.nti, o.ntj, o.ntk, o.layers, o.polar,
                    c->dphi, c->ih, r, x, p, v, faces, sc, o.words, c->npad, o.inv_dsum};
    HIP_TRY(c, launch_onchip<V>(a, o.m, o.closed, chunk, o.seq, fresh ? 1 : 0, o.wait_ticks, s));
    o.seq += (unsigned)chunk;
    return POT3D_OK;
}

int queue_onchip(pot3d_ctx *c, int chunk, bool fresh, hipStream_t s)
{
    if (c->precision == POT3D_FP32_REFINED)
        return queue_with<float>(c, c->r32, c->e32, c->p32[0], c->p32[1], static_cast<float *>(c->oc.faces), c->sc32, chunk, fresh, s);
    return queue_with<double>(c, c->r, c->x, c->p[0], c->p[1], static_cast<double *>(c->oc.faces), c->sc, chunk, fresh, s);
}

int run_onchip(pot3d_ctx *c, hipStream_t s, int *launches, DevScalars *final_out)
{
    constexpr int kChunk = 2048;   // steps per launch: about 10 ms
    DevScalars *sc = c->precision == POT3D_FP32_REFINED ? c->sc32 : c->sc;
    HIP_TRY(c, hipStreamSynchronize(s));   // so the lock is not held for earlier work on s
    for (bool fresh = true;; fresh = false) {
        {
            std::lock_guard<std::mutex> one(onchip_lock(c->device));
            const int rc = queue_onchip(c, kChunk, fresh, s);
            if (rc != POT3D_OK) return rc;
            HIP_TRY(c, hipMemcpyAsync(&c->h_sc[0], sc, sizeof(DevScalars), hipMemcpyDeviceToHost, s));
            HIP_TRY(c, hipStreamSynchronize(s));
        }
        ++*launches;
        if (c->h_sc[0].gave_up) {
            onchip_gave_up(c->device, c->oc);
            return kOnchipGaveUp;
        }
        if (c->h_sc[0].done) break;
    }
    *final_out = c->h_sc[0];
    return POT3D_OK;
}

}  // namespace host
}  // namespace pot3d
