// onchip.hpp -- the resident solve of small grids (onchip.hip).
#pragma once

#include "solver.hpp"

#include <mutex>

struct pot3d_ctx;

namespace pot3d {

constexpr int kOnchipMaxWg = 256;   // workgroups of a resident launch

constexpr int kOnchipMaxLayers = 16;   // layers of a box

// The operator's factors: of a layer (radial couplings at its lower and upper
// face over the face's angular area, width) and of a polar row (sin dtheta, the polar
// couplings below and above over dr dphi, dtheta / sin).
struct alignas(32) OnchipLayer {
    double lo, hi, dr, sum;   // sum = lo + hi
};
struct OnchipRow {
    double face, cm, cp, q;
};

// How a grid is split over the workgroups: boxes of ti x tj x tk cells at most
// (ti = m layers, tj <= 8 polar rows, tk <= 64 cells).  m = 0: the grid does
// not run on chip.
struct OnchipPlan {
    int m = 0;
    int ti = 0, tj = 0, tk = 0, nti = 0, ntj = 0, ntk = 0;
    unsigned seq = 0;                 // number of the last exchange step
    bool closed = false;              // closed upper wall: A has the constants in its null space
    double inv_dsum = 0.0;            // 1 / the sum of A's diagonal (onchip_tables)
    long long wait_ticks = 0;         // longest wait of an exchange (device wall clock)
    double retry_s = 0.0;             // how long the device stays with sweeps after a give-up
    unsigned long long *words = nullptr;   // device: posted sums, [2][6][kOnchipSums]
    void *faces = nullptr;                 // device: the workgroups' boundary cells (FP64, or FP32 in refined contexts)
    size_t face_bytes = 0;
    size_t bytes = 0;                      // of the four arrays together (onchip_place)
    OnchipLayer *layers = nullptr;         // device, nr + kOnchipMaxLayers (beyond nr: no couplings, diagonal 1)
    OnchipRow *polar = nullptr;            // device, nt
};
// Boundary cells of a box of m layers, with some cells between the boxes' sets.
constexpr int onchip_faces(int m) { return 2 * (8 * 64 + m * 64 + m * 8) + 16; }
// Posted sums of one step and component: two words per workgroup, and beside
// them kOnchipStop words of which any is set once an exchange has waited too long.
constexpr int kOnchipStop = 64;
constexpr int kOnchipSums = kOnchipStop + 2 * kOnchipMaxWg;
constexpr size_t kOnchipWords = 2 * 6 * (size_t)kOnchipSums;

template <typename V>
struct OnchipArgs {
    int nr, nt, np, pitch;
    int ti, tj, tk, nti, ntj, ntk;
    const OnchipLayer *layers;
    const OnchipRow *polar;
    const double *dphi, *ih;
    V *r;       // r_0 in (the residual); z at the end of a launch that goes on
    V *x;       // x in and out
    V *p;       // p_{-1} in; at the end p, or beta_k p_{k-1} once the solve has stopped
    V *v;       // D^-1 A p, from a launch to the next
    V *faces;   // [2][workgroups][onchip_faces(m)]: boundary v of the exchange steps, in turn
    DevScalars *sc;
    unsigned long long *words;
    long long npad;
    double inv_dsum;   // closed wall: OnchipPlan's
};

// One launch of up to `chunk` iterations.  seq0: plan.seq; fresh: no launch of
// this solve has run yet.
template <typename V>
hipError_t launch_onchip(const OnchipArgs<V> &a, int m, bool closed, int chunk, unsigned seq0, int fresh,
                         long long wait_ticks, hipStream_t s);
unsigned onchip_oob_line();   // take_oob's line of onchip.hip, 0 if none

namespace host {

// The plan for a context's grid and precision (m = 0 if it does not fit).
OnchipPlan plan_onchip(const pot3d_ctx *c);
// Host tables of the operator's factors (nr + kOnchipMaxLayers layers, nt polar
// rows), and from them and 1/(phi differences) ih the plan's inv_dsum.
void onchip_tables(OnchipPlan &o, int nr, int nt, int np, const double *rf, const double *tf, const double *ih,
                   int upper_bc, OnchipLayer *layers, OnchipRow *polar);
// The plan's arrays in `bytes` of device memory at base, words first.
void onchip_place(OnchipPlan &o, int nr, int nt, void *base);
// Resident launches of one device run one at a time: held from before a launch
// until it has completed.
std::mutex &onchip_lock(int device);
// Whether a device takes resident launches: not for plan.retry_s after one gave
// up, since what kept it from coming together (another process's kernels, a
// stream that may not use every compute unit) is likely still there, and every
// try costs the whole wait.
bool onchip_open(int device);
void onchip_gave_up(int device, const OnchipPlan &plan);
// One launch on s with the context's vectors (FP64, or the FP32 inner ones);
// the caller holds the lock and copies the scalars back.
int queue_onchip(pot3d_ctx *c, int chunk, bool fresh, hipStream_t s);
// The iterations of a started solve until its done flag.  kOnchipGaveUp: the
// launch could not come together; nothing usable is left, solve again without.
constexpr int kOnchipGaveUp = 1;
int run_onchip(pot3d_ctx *c, hipStream_t s, int *launches, DevScalars *final_out);

}  // namespace host
}  // namespace pot3d
