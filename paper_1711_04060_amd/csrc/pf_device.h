// pf_device.h -- device state and helpers shared by the stencil kernels
// (pf_kernels.h) and the on-chip Krylov kernel (pf_chip.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pfk {

// node flag bits (one byte per node)
enum : uint8_t { F_DIR_PHI = 1, F_DIR_PSI = 2, F_SOLVENT = 4, F_SOLUTE = 8 };

// Device-side BiCGSTAB state (FP64 even when the vectors are FP32).  Values
// produced inside an iteration are kept per iteration parity q = i & 1: a
// kernel of iteration i reads the slots of iteration i-1 (or of its own
// iteration written by an earlier kernel) and its leading workgroup writes
// slot q, so no workgroup reads a slot that its own kernel writes.
struct Scalars {
    double rho[2];     // shadow . r at the start of iteration i
    double alpha[2];   // alpha_i
    double omega[2];   // omega_i
    double rr;         // ||r||^2 of the recurrence, last completed iteration
    double tol2;       // (rel_tol * ||b_lift||)^2
    double rt2;        // ||r_shadow||^2 at the last (re)start
    double red[4];     // sums of the last standalone reduction (residual, relaxation)
    int iter[2];       // iterations completed when iteration i starts
    int iter_done;     // iterations completed (host view)
    int maxit;
    int stop;          // ST_RUN while iterating, else the terminal state
    int stop_a;        // state decided by the last step A, published by the step B after it
    int fresh;         // 1 from a (re)start until step B of the first iteration
    int neg_shift;     // set when a free row of the operator has sigma < 0
    int shift_class;   // set when sigma is one value per palette class on the free rows
    int gave_up;       // set by a tile of an on-chip run that stopped waiting for the others
};
enum { ST_RUN = 0, ST_CONV = 1, ST_RESTART = 3, ST_NONFINITE = 4, ST_MAXIT = 5 };

// stencil operation selector
enum { OP_SPMV = 0, OP_SPMV_JAC = 1, OP_RESID = 2, OP_BA = 3, OP_BB = 4 };

// how the BiCGSTAB steps get the diagonal shift sigma of the own node: none,
// read from a per-node array, or (palette form) from a table by the node's
// palette class, where sigma is one value per class on the free rows (the
// linearised systems, whose shift is uniform in the solvent and zero in the
// solute)
enum { SIG_NONE = 0, SIG_NODE = 1, SIG_CLASS = 2 };

// Palette form of the coefficient field: fields with at most PAL_MAX
// distinct values (the piecewise-constant dielectric of Eq. (7): eps_m in the
// solute region, eps_s in the solvent) are stored as one byte per node, the
// value's palette index with the Dirichlet mark in bit 7, and the face
// coefficient of each pair of palette values is precomputed (a table staged
// in LDS).
constexpr int PAL_MAX = 16;
constexpr int FTAB = PAL_MAX * PAL_MAX;

// ------------------------------------------------------------- helpers

// Workgroups are dispatched round-robin over the 8 XCDs (block b runs on XCD
// b % 8).  Remap so that each XCD receives a contiguous range of logical
// tiles: neighbouring strips then share that XCD's L2 for their halos.
__device__ __forceinline__ int xcd_remap(int b, int G)
{
    const int X = 8;
    const int per = G / X, rem = G % X;
    const int xcd = b % X, idx = b / X;
    return (xcd < rem) ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// 1/d for d > 0: the hardware reciprocal estimate refined by two Newton steps
// (FP64; within an ulp or so of the correctly rounded quotient) or the
// hardware FP32 reciprocal (1 ulp).
__device__ __forceinline__ double rcp_pos(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    double e = __builtin_fma(-d, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-d, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float rcp_pos(float d) { return __builtin_amdgcn_rcpf(d); }

// Face coefficient: harmonic mean of the two nodal values, divided by h^2.
template <typename T>
__device__ __forceinline__ T face(T a, T b, T ih2)
{
    return (T(2) * a * b * ih2) * rcp_pos(a + b);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
    return v;
}

// Partials: PSTRIDE doubles per workgroup (up to PSTRIDE quantities).
constexpr int PSTRIDE = 8;

// The BiCGSTAB stencil steps issue every store unconditionally: a store whose
// node is outside the tile (or a step past its last plane) goes to a sink
// slot of the thread instead.  Stores count in the same wait counter as
// loads, and a store under a branch would make the compiler assume the
// shorter path and wait for loads still meant to be in flight.
constexpr int SINK_ELEMS = 2048;   // >= threads * nodes per thread

// Reduce NQ per-thread values over the workgroup; thread 0 gets the result.
template <int NQ, int NT, bool MAX = false>
__device__ __forceinline__ void block_reduce(double (&v)[NQ])
{
    __shared__ double red[NT / 64][NQ];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double s = MAX ? wave_max(v[q]) : wave_sum(v[q]);
        if (lane == 0) red[w][q] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            double s = red[0][q];
            for (int i = 1; i < NT / 64; ++i) s = MAX ? fmax(s, red[i][q]) : s + red[i][q];
            v[q] = s;
        }
    }
}

// Store the workgroup partials (thread 0 holds the reduced values).
template <int NQ>
__device__ __forceinline__ void store_partials(const double (&v)[NQ], double *partials, int slot)
{
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) partials[slot * PSTRIDE + q] = v[q];
    }
}

// Fixed-order sum (or max) of the G partials, run by a finalize workgroup.
template <int NQ, int NT, bool MAX = false>
__device__ __forceinline__ void final_reduce(double (&v)[NQ], const double *partials, int G)
{
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = 0.0;
    for (int i = threadIdx.x; i < G; i += NT) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double p = partials[i * PSTRIDE + q];
            v[q] = MAX ? fmax(v[q], p) : v[q] + p;
        }
    }
    __syncthreads();
    block_reduce<NQ, NT, MAX>(v);
}

__device__ __forceinline__ bool finite(double x) { return __builtin_isfinite(x); }

// Sum of NQ quantities over G partials in one fixed order whatever the
// workgroup size (lanes 0..255 each add the partials lane, lane + 256, ...
// in increasing order, then a fixed tree), so every workgroup of a consumer
// kernel and the one-workgroup finalize kernel obtain identical bits.  The
// loads are split from the sum so that a kernel can issue them together with
// its first data loads: the first PJ*256 partials are loaded without a loop
// (indices past G load slot 0 and are not added).
constexpr int PJ = 4;

template <int NQ>
struct PartLoad {
    double l[PJ][NQ];
};

template <int NQ>
__device__ __forceinline__ void load_partials(PartLoad<NQ> &pl, const double *partials, int G)
{
    const int lane = threadIdx.x & 255;
#pragma unroll
    for (int j = 0; j < PJ; ++j) {
        const int i = lane + 256 * j;
        const int ic = i < G ? i : 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) pl.l[j][q] = partials[ic * PSTRIDE + q];
    }
}

// Every thread receives the result.
template <int NQ>
__device__ __forceinline__ void sum_loaded_partials(double (&tot)[NQ], const PartLoad<NQ> &pl,
                                                    const double *partials, int G)
{
    __shared__ double sred[4][NQ];
    __shared__ double sout[NQ];
    double v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = 0.0;
    if (threadIdx.x < 256) {
        const int lane = threadIdx.x;
#pragma unroll
        for (int j = 0; j < PJ; ++j) {
            if (lane + 256 * j < G) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) v[q] += pl.l[j][q];
            }
        }
        for (int i = lane + 256 * PJ; i < G; i += 256) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[q] += partials[i * PSTRIDE + q];
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const double sw = wave_sum(v[q]);
        if (lane == 0 && w < 4) sred[w][q] = sw;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) sout[q] = ((sred[0][q] + sred[1][q]) + sred[2][q]) + sred[3][q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) tot[q] = sout[q];
}

template <int NQ>
__device__ __forceinline__ void sum_partials(double (&tot)[NQ], const double *partials, int G)
{
    PartLoad<NQ> pl;
    load_partials<NQ>(pl, partials, G);
    sum_loaded_partials<NQ>(tot, pl, partials, G);
}

// Start of step A of iteration i (parity q).  Step A also finishes iteration
// i-1: its x, r update (Table 3 steps 16, 17) needs omega_{i-1} = t.s / t.t
// (step 15), and the p update needs beta_i (step 8), i.e. rho_i = shadow . r_i
// (step 4).  Since r_i = s - omega t, rho_i = shadow . s - omega shadow . t
// from step B's sums, so no pass over r_i has to finish first; ||r_i||^2 for
// the stop test is summed from r_i itself in this step and tested by step B.
// tot: t.s, t.t, s.s, shadow . s, shadow . t of iteration i-1.
struct FinB {
    double alpha, omega, beta, rho, rr;
    int iter, stop;
    bool update;   // apply the x, r update of iteration i-1
};

__device__ __forceinline__ FinB fin_b(const Scalars *sc, const double (&tot)[5], int q)
{
    const int qp = q ^ 1;
    const double ts = tot[0], tt = tot[1], ss = tot[2], rs = tot[3], rtt = tot[4];
    FinB f{};
    f.alpha = sc->alpha[qp];
    f.iter = sc->iter[qp] + 1;
    f.stop = ST_RUN;
    f.update = true;
    if (!finite(ts) || !finite(tt) || !finite(ss) || !finite(rs) || !finite(rtt)) {
        f.stop = ST_NONFINITE;
        f.update = false;
        return f;
    }
    if (ss <= sc->tol2) {
        // ||s|| already meets the tolerance: x += alpha M^-1 p, r = s
        f.omega = 0.0;
        f.rho = rs;
        f.rr = ss;
        f.stop = ST_CONV;
        return f;
    }
    if (tt == 0.0) {
        f.stop = ST_RESTART;
        f.update = false;
        return f;
    }
    f.omega = ts / tt;
    f.rho = rs - f.omega * rtt;
    f.rr = fmax(0.0, ss - 2.0 * f.omega * ts + f.omega * f.omega * tt);
    if (f.rr > sc->tol2) {   // otherwise step B decides on the summed ||r_i||^2
        if (f.iter >= sc->maxit) {
            f.stop = ST_MAXIT;
            return f;
        }
        if (f.omega == 0.0 || fabs(f.rho) < 1e-300 || f.rho * f.rho < 1e-28 * sc->rt2 * f.rr) {
            f.stop = ST_RESTART;   // shadow residual nearly orthogonal to r
            return f;
        }
    }
    if (f.omega != 0.0 && sc->rho[qp] != 0.0) f.beta = (f.rho / sc->rho[qp]) * (f.alpha / f.omega);
    return f;
}

// Written by the leading workgroup.  The stop state goes to stop_a, not stop:
// the other workgroups of this step A test stop on entry and must still apply
// the x, r update when the state ends the run.
__device__ __forceinline__ void fin_b_store(Scalars *sc, const FinB &f, int q)
{
    sc->stop_a = f.stop;
    if (!f.update) return;
    sc->omega[q ^ 1] = f.omega;
    sc->rho[q] = f.rho;
    sc->iter[q] = f.iter;
    sc->iter_done = f.iter;
    sc->rr = f.rr;
}

}  // namespace pfk
