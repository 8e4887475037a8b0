// Device kernels of the entropy-stable DGSEM shallow-water solver for gfx950.
//
// Work decomposition: a workgroup holds E elements of (N+1)^2 nodes, one
// thread per node (E ~ 256 / (N+1)^2, so a workgroup is four 64-wide waves);
// nodal state and the contravariant metric directions are staged in LDS, the
// state arrays are read and written in the coalesced SoA order
// [K][(N+1)^2], and the face work of the E elements is spread over the same
// threads (one face node per thread and pass).  Workgroup -> element-tile
// mapping is XCD-aware so that each of the eight XCDs sweeps one contiguous
// block of tiles and neighbour traces mostly hit its own L2.
//
// Kernels: per RK stage stage_kernel (split-form volume term, interface flux,
// source, artificial viscosity, stage update, positivity limiter and the
// modal indicator of the result, fused); per step dt_kernel (adaptive steps);
// indicator_kernel for a state no stage produced.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "esdg_tables.hpp"

namespace esdg {

// ------------------------------------------------------------------------
// Shapes
// ------------------------------------------------------------------------
// Workgroup shape per degree.  Where whole elements fill a 64-wide wave
// with (almost) no idle lanes (N = 2, 3, 7) a workgroup is one wave: its
// barriers are cheap and waves run independently.  Otherwise four waves
// hold E = floor(256/(N+1)^2) elements packed across the waves.
template <int N>
struct Shape {
    static constexpr int nf = N + 1;
    static constexpr int np = nf * nf;
    static constexpr bool one_wave = (np <= 64) && (64 - (64 / np) * np) * 16 <= 64;
    static constexpr int T = one_wave ? 64 : 256;                  // threads per workgroup
    static constexpr int E = (T / np) > 0 ? (T / np) : 1;          // elements per workgroup
    static constexpr int NFACE = E * 4 * nf;                       // face-node slots per workgroup
    static_assert(E * np <= T, "elements must fit the workgroup");
};

// Workgroup sizes of the stage kernel: the default one is Shape's, but 256
// threads at N = 2, where a wave's seven elements have 84 face slots and every
// wave of a one-wave tile takes a second round of them for 20 lanes (with 28
// elements' 336 slots, two waves of four do: 128 -> 123 us at 601^2; 192
// threads 128, 128 threads 125; both slots of a lane prefetched 127); the
// alternative one is one wave at N = 2, 256 threads at N = 3 and 7, else 128.
template <int N>
struct StageThreads {
    static constexpr int dflt = N == 2 ? 256 : Shape<N>::T;
    static constexpr int alt = N == 2 ? 64 : (Shape<N>::T == 64 ? 256 : 128);
};

template <int N, int TT>
struct TileShape {
    static constexpr int nf = N + 1;
    static constexpr int np = nf * nf;
    static constexpr int T = TT;
    static constexpr int E = (T / np) > 0 ? (T / np) : 1;
    static constexpr int NFACE = E * 4 * nf;
    static_assert(E * np <= T, "elements must fit the workgroup");
};

// Compiled variants of the stage kernel, chosen at run time by the
// autotuner (esdg_autotune); every variant does the same arithmetic per
// element in the same order (results are bitwise the same):
//   0  the default tile, its register budget and partner unroll;
//   1  the alternative workgroup size (StageThreads), no register budget;
//   2  the default tile with one wave per SIMD less in its register budget
//      (more registers where the budget binds: FP64 at N = 2, 3 and 8 takes
//      88-94 with either);
//   3  the default tile with the other partner unroll (by two, or fully where
//      the default is by two: N = 7 in FP64, N = 6 and 8 in FP32);
//   4  the default tile with bank-conflict-free staging rows: padded by one
//      node (the paper's LDS padding, appendix C), or at N = 7 XOR-swizzled
//      columns (no more LDS; StageCfg::SWZ); unrolled by two (a full unroll
//      of the padded rows spills 50-270 registers).
// Default register budget in the FP64 update modes: six waves per SIMD at
// N = 5, 6 and 7 (at N = 5, 255^2, 86 us with five and 82 with six), five
// otherwise (six spill on wet/dry tiles: N = 3, 200^2 bowl 26.0 -> 28.2 us; on
// all at N = 2 and 8: 129 -> 135, 57 -> 66); in the FP32 update modes eight (seven for
// variant 2, none for variant 1): left free, the compiler gave some FP32
// variants 100-120 registers; no constraint in the right-hand-side mode.
// Against an unroll by two the full one runs 2-3% faster at N = 6 and within
// 1% at the other degrees.
constexpr int kStageVariants = 5;

template <int N, int V>
struct StageCfg {
    static_assert(V >= 0 && V < kStageVariants, "stage variant");
    static constexpr int T = V == 1 ? StageThreads<N>::alt : StageThreads<N>::dflt;
    static constexpr int base_waves = V == 1 ? 1 : ((N >= 5 && N <= 7) ? 6 : 5);
    static constexpr int waves = V == 2 ? base_waves - 1 : base_waves;
    // partner-loop unroll, double and single precision: at N = 7 the doubles'
    // by two (a smooth flow even; with wet/dry tiles at 128^2 40.4 -> 39.6 us,
    // fewer registers being spilled on them), the floats' at N = 6 and 8, where
    // eight waves per SIMD spill 13 and 10 registers of the full unroll (512^2:
    // 294 -> 272 and 489 -> 454 us; with seven waves the full one is as good);
    // variant 3 takes the other one of two and full
    static constexpr bool by_two = N == 7, by_two32 = N == 6 || N == 8;
    static constexpr int VU = (V == 4 || by_two != (V == 3)) ? 2 : N + 1;
    static constexpr int VU32 = (V == 4 || (V == 3 ? !by_two32 : V == 0 && by_two32)) ? 2 : N + 1;
    // Variant 4 avoids the LDS bank conflicts of the eta-direction partner
    // reads (a wave reads column mm of every row, rows 16(N+1) bytes apart in
    // FP64: at N = 7 eight rows on two bank groups).  At N = 7 the columns of
    // row i are XOR-swizzled (node (i, j) in column j ^ (i >> 1)), which puts
    // the eight rows' reads on distinct banks in both directions with no more
    // LDS; at the other degrees, whose N + 1 is no power of two, each row is
    // padded by one node.
    static constexpr bool SWZ = V == 4 && N == 7;
    static constexpr int PAD = (V == 4 && !SWZ) ? 1 : 0;
};

// Column of node (i, j) in its LDS staging row (see StageCfg::SWZ).
template <int N, int V>
__device__ __forceinline__ int stage_col(int i, int j)
{
    if constexpr (StageCfg<N, V>::SWZ) return j ^ (i >> 1);
    else return j;
}

template <int N, typename R, int MODE, int V>
struct StageWaves {
    static constexpr int value =
        MODE == 0 ? 1 : (sizeof(R) == 8 ? StageCfg<N, V>::waves : (V == 1 ? 1 : (V == 2 ? 7 : 8)));
};

// Workgroup barrier for exchanges through LDS only: orders LDS accesses
// without waiting for outstanding global loads and stores (which
// __syncthreads() would).  A one-wave workgroup needs no barrier.
template <int T>
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    if constexpr (T > 64) __builtin_amdgcn_s_barrier();
    else __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The kernel's one argument, a struct A, read where it lies (the kernarg
// segment) instead of through the parameter: a parameter's fields are all
// loaded at the kernel's entry and held, which with some forty pointers and
// the operator tables spills scalar registers.  Each call of kernarg starts
// afresh: fields read through its result are loaded behind the call, and
// need not live from one phase of the kernel to the next.
template <typename A>
__device__ __forceinline__ const A &kernarg()
{
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const A *)p;
}

// x, as a value the compiler cannot know: what is computed from it behind
// this point is computed there, not kept in registers from further up.
__device__ __forceinline__ int fresh(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

constexpr int kXcds = 8;
constexpr int kDtSlots = 64;

// Device status flags of a context: negative element mean, limited
// elements, no admissible step, J <= 0 at mesh upload, non-finite output.
constexpr int kFlagNegMean = 0, kFlagLimited = 1, kFlagDtPos = 2, kFlagBadJ = 3, kFlagNonFinite = 4;
// a step that exceeded twice the CFL / viscous bound of the state it produced
constexpr int kFlagStepBound = 5;
constexpr int kNumFlags = 8;

// Tile of workgroup b when B = round_up(ntiles, 8) workgroups are launched:
// hardware places workgroup b on XCD b % 8, so XCD x gets tiles
// [x*per, (x+1)*per).  Tiles >= ntiles return -1.  (A tile holds at least one
// of the at most INT32_MAX elements.)
__device__ inline int64_t xcd_tile(int64_t ntiles)
{
    const uint32_t b = blockIdx.x, n = (uint32_t)ntiles;
    const uint32_t per = (n + kXcds - 1) / kXcds;
    const uint32_t tile = (b % kXcds) * per + b / kXcds;
    return tile < n ? (int64_t)tile : -1;
}

// Face node k of local side s -> local (i, j).
template <int N>
__device__ __forceinline__ void side_node(int s, int k, int &i, int &j)
{
    i = (s == 0 || s == 2) ? k : (s == 1 ? N : 0);
    j = (s == 1 || s == 3) ? k : (s == 2 ? N : 0);
}

// ------------------------------------------------------------------------
// Arguments
// ------------------------------------------------------------------------
// Operator tables of one degree, in device memory.
template <typename R>
struct Tab {
    R D[kMaxNF * kMaxNF];     // derivative matrix (this and the next two in rows of N + 1)
    R Dz[kMaxNF * kMaxNF];    // the same with a zero diagonal (flux differencing)
    R Vinv[kMaxNF * kMaxNF];  // Vandermonde inverse
    R w[kMaxNF];              // LGL weights
    R iw0;                    // 1 / w_0 (end weight)
};

// The entries that kernels read as scalars, passed by value.
template <typename R>
struct Uni {
    R w[kMaxNF];              // LGL weights
    R ve[kMaxNF], vo[kMaxNF]; // rows of Vinv: the even and the odd one of modes N and N - 1
    R iw0;                    // 1 / w_0
};

template <typename R>
inline Uni<R> uniform_entries(const Tab<R> &t, int N)
{
    Uni<R> u;
    const int e = N & 1 ? N - 1 : N, o = N & 1 ? N : N - 1;
    for (int k = 0; k < kMaxNF; ++k) {
        u.w[k] = k <= N ? t.w[k] : R(0);
        u.ve[k] = k <= N ? t.Vinv[e * (N + 1) + k] : R(0);
        u.vo[k] = k <= N ? t.Vinv[o * (N + 1) + k] : R(0);
    }
    u.iw0 = t.iw0;
    return u;
}

template <typename R>
struct Mesh {
    int64_t K;
    const R *Ax, *Cx;   // J grad(xi)  = ( y_eta, -x_eta)  [K][np]
    const R *Ae, *Ce;   // J grad(eta) = (-y_xi,   x_xi)   [K][np]
    const R *bx, *by;   // split-form bathymetry derivatives (eq. SourceDisc)
    const double *xr, *yr;  // float64 coordinates less the element's first node [K][np] (float64 contexts)
    const R *mref;      // float32 contexts: [K][4] (Ax, Cx, Ae, Ce) of each element's middle node
    const R *bface;     // bathymetry on the faces [K][4][nf]
    const int32_t *nbr; // [K][4] neighbour element
    const int8_t *code; // [K][4] neighbour side | flip << 2 | wall << 3 (a wall names the element itself)
    int walls;          // some side is a wall (else the wall bit is never looked at)
};

// Single precision stores the metric terms of each node less those of its
// element's middle node (Mesh::mref): differences between an element's
// nodes, which the jump-form volume sums take, are then rounded at the size
// of the terms' variation across the element rather than of the terms.  On a
// fine mesh the terms vary little across an element, and their rounding at
// full size breaks the discrete metric identities by far more than the
// arithmetic's own rounding.  The terms themselves are the sums.
template <typename R>
constexpr bool kMetricRel = sizeof(R) == 4;

// Metric terms J grad(xi) = (Ax, Cx), J grad(eta) = (Ae, Ce) at node q of
// element e.
template <typename R>
__device__ __forceinline__ void metric_at(const Mesh<R> &m, int64_t q, int64_t e, R &Ax, R &Cx, R &Ae, R &Ce)
{
    Ax = m.Ax[q]; Cx = m.Cx[q]; Ae = m.Ae[q]; Ce = m.Ce[q];
    if constexpr (kMetricRel<R>) {
        const R *r = m.mref + 4 * e;
        Ax += r[0]; Cx += r[1]; Ae += r[2]; Ce += r[3];
    }
}

template <typename R>
struct Phys {
    R g, h_tol, eps0, sigma_min, sigma_max, cfl, cfl_visc;
    R i2g;                 // 1 / (2 g)
    R ratio_min, ratio_max; // 10^sigma_min, 10^sigma_max
    R visc_c, br1;          // viscous bound: visc_c / (br1 eps max|grad|^2)
    R smooth_tau;           // threshold of smooth_line (0: no line is taken to be smooth)
    int ec, limiter_on;
};

// Neighbour node of face node (s, k) of element e.  At a solid wall the face
// map names the element's own side (the node itself): the interface flux then
// mirrors the velocity (is_wall), the viscous terms see no jump.
template <int N, typename R>
__device__ __forceinline__ int64_t nbr_node(const Mesh<R> &m, int64_t e, int s, int k,
                                           int64_t &en, int &ns, int &kk)
{
    constexpr int nf = N + 1, np = nf * nf;
    en = m.nbr[e * 4 + s];
    const int c = m.code[e * 4 + s];
    ns = c & 3;
    kk = ((c >> 2) & 1) ? N - k : k;
    int i, j;
    side_node<N>(ns, kk, i, j);
    return en * np + i * nf + j;
}

template <typename R>
__device__ __forceinline__ bool is_wall(const Mesh<R> &m, int64_t e, int s)
{
    return m.walls && ((m.code[e * 4 + s] >> 3) & 1);
}

// Reflecting-wall outside state: the velocity with its normal component
// reversed about the unit normal (nx, ny); height and bathymetry unchanged.
template <typename R>
__device__ __forceinline__ void wall_mirror(R nx, R ny, R &u, R &v)
{
    const R dn = u * nx + v * ny;
    u -= R(2) * dn * nx;
    v -= R(2) * dn * ny;
}

// 1/x from the hardware reciprocal estimate refined by two Newton-Raphson
// steps r <- r + r (1 - x r) (quadratic convergence; normal positive x)
__device__ __forceinline__ double rcp_nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ float rcp_nr(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// sqrt(x) for x >= 0 from the hardware's reciprocal square root: one coupled
// Newton step for sqrt(x) and 1/(2 sqrt(x)), then two residual corrections of
// the root (published as Goldschmidt's iteration).  The library's sqrt scales
// its argument around the same steps for the sake of subnormal x; here x is a
// squared wave speed or length.
__device__ __forceinline__ double sqrt_nr(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y, k = 0.5 * y;
    const double r = fma(-k, s, 0.5);
    s = fma(s, r, s);
    k = fma(k, r, k);
    s = fma(fma(-s, s, x), k, s);
    s = fma(fma(-s, s, x), k, s);
    return x > 0.0 ? s : 0.0;
}
__device__ __forceinline__ float sqrt_nr(float x) { return sqrtf(x); }

// s = sqrt(x) and i = 1/sqrt(x) for a positive normal x, the reciprocal with
// the last Newton step of rcp_nr.
__device__ __forceinline__ void sqrt_rcp(double x, double &s, double &i)
{
    const double y = __builtin_amdgcn_rsq(x);
    double k = 0.5 * y;
    s = x * y;
    const double r = fma(-k, s, 0.5);
    s = fma(s, r, s);
    k = fma(k, r, k);
    s = fma(fma(-s, s, x), k, s);
    s = fma(fma(-s, s, x), k, s);
    k += k;
    i = fma(k, fma(-s, k, 1.0), k);
}
__device__ __forceinline__ void sqrt_rcp(float x, float &s, float &i)
{
    const float y = __builtin_amdgcn_rsqf(x);
    s = x * y;
    s = fmaf(fmaf(-s, s, x), 0.5f * y, s);
    i = fmaf(y, fmaf(-s, y, 1.0f), y);
}

template <typename R>
__device__ __forceinline__ R rcp_wet(R h, R h_tol)
{
    return h > h_tol ? rcp_nr(h) : R(0);
}

// The single-precision stage kernel forms the volume and interface terms from
// jumps to the own node (interface_flux_delta and the volume loop): the
// two-point sums of flux-sized terms whose result is a derivative lose the
// flux-to-derivative ratio (about N^2 / element size) in relative accuracy,
// which double precision absorbs and single precision does not.
template <typename R>
constexpr bool kJumpForm = sizeof(R) == 4;

// The stage kernel computes its lanes' places in the tile a second time after
// the volume sums (fresh) instead of keeping them where registers are short:
// in double precision (stage of a smooth flow, N = 3: 46.0 -> 40.8 us, N = 4:
// 56.0 -> 49.5, N = 6: 57.2 -> 55.7, others even), in single precision at N =
// 5 (36.7 -> 32.8 us; others 1-3% slower).
template <int N, typename R>
constexpr bool kFreshLanes = sizeof(R) == 8 || N == 5;

// At N <= 4 the double-precision stage kernel reads each node's two
// coordinates (relative to its element's first node) instead of its four
// metric terms and forms the metric terms itself, with the sums of
// geometry_kernel in the same order (so bit for bit the stored values): 16
// fewer bytes per node and stage for 4(N+1) multiply-adds and two more
// workgroup barriers.  Measured on the stage kernel: 3-7% faster at N = 2..4,
// 2% slower at N = 5 and 6% at N = 7, where the longer sums and the registers
// it holds across the face prefetch cost more than the bytes.  In single precision the four metric
// terms take as many bytes as the two float64 coordinates.
template <int N, typename R>
constexpr bool kMetricInKernel = sizeof(R) == 8 && N <= 4;

// Rotated numerical interface flux along the unit normal (nx, ny), '-' =
// own trace, '+' = neighbour (appendix B): EC part plus, for the entropy
// stable flux, -1/2 R |Lambda| R^T [[q~]] expanded in closed form.
// Velocities are the primitive ones (zero at dry nodes).
template <typename R>
__device__ __forceinline__ void interface_flux(R hm, R um, R vm, R bm, R hp, R up, R vp, R bp, R nx, R ny,
                                               const Phys<R> &P, R &F0, R &F1, R &F2)
{
    const R g = P.g;
    const R utm = nx * um + ny * vm, vtm = nx * vm - ny * um;
    const R utp = nx * up + ny * vp, vtp = nx * vp - ny * up;
    const R cm = sqrt_nr(g * fmax(hm, R(0)));
    const R cp = sqrt_nr(g * fmax(hp, R(0)));
    const R ah = R(0.5) * (hm + hp), au = R(0.5) * (utm + utp), av = R(0.5) * (vtm + vtp);
    const R ah2 = R(0.5) * (hm * hm + hp * hp), ac = R(0.5) * (cm + cp);
    R f0 = ah * au;
    R f1 = ah * au * au + R(0.5) * g * ah2;
    R f2 = ah * au * av;
    if (!P.ec) {
        const R dq1 = g * ((hp + bp) - (hm + bm)) -
                      R(0.5) * ((utp * utp + vtp * vtp) - (utm * utm + vtm * vtm));
        const R dq2 = utp - utm, dq3 = vtp - vtm;
        const R lp = fabs(au + ac) * P.i2g, l2 = fabs(ah * au), lm = fabs(au - ac) * P.i2g;
        const R r1 = lp * (dq1 + (au + ac) * dq2 + av * dq3);
        const R r2 = l2 * dq3;
        const R r3 = lm * (dq1 + (au - ac) * dq2 + av * dq3);
        f0 -= R(0.5) * (r1 + r3);
        f1 -= R(0.5) * ((au + ac) * r1 + (au - ac) * r3);
        f2 -= R(0.5) * (av * (r1 + r3) + r2);
    }
    F0 = f0;
    F1 = nx * f1 - ny * f2;
    F2 = ny * f1 + nx * f2;
}

// The same interface flux less the own trace's physical flux along n,
// f*(-, +) - f(-).n, written in the jumps dh = h+ - h-, du, dv only (the
// single-precision stage kernel).  With a mean m = a- + d/2:
//   {h}{u_n} - h- u_n-           = (h- du_n + dh {u_n}) / 2
//   {h}{u_n}^2 - h- u_n-^2       = {u_n} df0 + du_n h- u_n- / 2
//   g/2 ({h^2} - h-^2)           = g dh {h} / 2
//   {h}{u_n}{v_t} - h- u_n- v_t- = {v_t} df0 + dv_t h- u_n- / 2
// and, in the dissipation, [[g(h+b) - |u|^2/2]] with |u+|^2 - |u-|^2 =
// du (u+ + u-) + dv (v+ + v-).  The own flux is the row-sum part of the
// volume term's two-point sums at a face node, where it cancels against this
// subtracted part; formed from the jumps, neither part is rounded at the
// size of the flux itself, only at the size of its variation.
template <typename R>
__device__ __forceinline__ void interface_flux_delta(R hm, R um, R vm, R bm, R hp, R up, R vp, R bp, R nx,
                                                     R ny, const Phys<R> &P, R &F0, R &F1, R &F2)
{
    const R g = P.g;
    const R dh = hp - hm, du = up - um, dv = vp - vm;
    const R utm = nx * um + ny * vm, vtm = nx * vm - ny * um;
    const R dut = nx * du + ny * dv, dvt = nx * dv - ny * du;
    const R ah = R(0.5) * (hm + hp), au = utm + R(0.5) * dut, av = vtm + R(0.5) * dvt;
    const R fo = hm * utm;
    R f0 = R(0.5) * (hm * dut + dh * au);
    R f1 = au * f0 + R(0.5) * (dut * fo + g * dh * ah);
    R f2 = av * f0 + R(0.5) * dvt * fo;
    if (!P.ec) {
        const R cm = sqrt_nr(g * fmax(hm, R(0)));
        const R cp = sqrt_nr(g * fmax(hp, R(0)));
        const R ac = R(0.5) * (cm + cp);
        const R dq1 = g * (dh + (bp - bm)) - R(0.5) * (du * (up + um) + dv * (vp + vm));
        const R dq2 = dut, dq3 = dvt;
        const R lp = fabs(au + ac) * P.i2g, l2 = fabs(ah * au), lm = fabs(au - ac) * P.i2g;
        const R r1 = lp * (dq1 + (au + ac) * dq2 + av * dq3);
        const R r2 = l2 * dq3;
        const R r3 = lm * (dq1 + (au - ac) * dq2 + av * dq3);
        f0 -= R(0.5) * (r1 + r3);
        f1 -= R(0.5) * ((au + ac) * r1 + (au - ac) * r3);
        f2 -= R(0.5) * (av * (r1 + r3) + r2);
    }
    F0 = f0;
    F1 = nx * f1 - ny * f2;
    F2 = ny * f1 + nx * f2;
}

// ------------------------------------------------------------------------
// Geometry: metric terms by the derivative matrix (eq. NablaRelation)
// ------------------------------------------------------------------------
template <int N, typename R>
__global__ void geometry_kernel(int64_t K, const double *__restrict__ x, const double *__restrict__ y,
                                R *Ax, R *Cx, R *Ae, R *Ce, R *mref, double *xr, double *yr, int *bad,
                                Tab<double> tab)
{
    constexpr int nf = N + 1, np = nf * nf;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= K * np) return;
    const int64_t e = q / np;
    const int p = (int)(q - e * np), i = p / nf, j = p - i * nf;
    const double *xe = x + e * np, *ye = y + e * np;
    // differentiate coordinates relative to the element's first node: the
    // metric terms are translation invariant and the sums stay at the
    // element's size (no cancellation against the absolute position)
    const double x0 = xe[0], y0 = ye[0];
    double xxi = 0, xeta = 0, yxi = 0, yeta = 0;
#pragma unroll
    for (int m = 0; m < nf; ++m) {
        xxi += tab.D[i * nf + m] * (xe[m * nf + j] - x0);
        yxi += tab.D[i * nf + m] * (ye[m * nf + j] - y0);
        xeta += tab.D[j * nf + m] * (xe[i * nf + m] - x0);
        yeta += tab.D[j * nf + m] * (ye[i * nf + m] - y0);
    }
    const double J = xxi * yeta - xeta * yxi;
    if (!(J > 0.0)) atomicOr(bad, 1);
    // the differenced coordinates themselves, for the float64 stage kernel,
    // which forms the same sums from them (the same values bit for bit)
    if (xr) {
        xr[q] = xe[p] - x0;
        yr[q] = ye[p] - y0;
    }
    if constexpr (kMetricRel<R>) {
        // the middle node's terms by the same sums, rounded, and each node's
        // terms less them (kMetricRel)
        constexpr int c = N / 2;
        double cxxi = 0, cxeta = 0, cyxi = 0, cyeta = 0;
#pragma unroll
        for (int m = 0; m < nf; ++m) {
            cxxi += tab.D[c * nf + m] * (xe[m * nf + c] - x0);
            cyxi += tab.D[c * nf + m] * (ye[m * nf + c] - y0);
            cxeta += tab.D[c * nf + m] * (xe[c * nf + m] - x0);
            cyeta += tab.D[c * nf + m] * (ye[c * nf + m] - y0);
        }
        const R r0 = (R)cyeta, r1 = (R)(-cxeta), r2 = (R)(-cyxi), r3 = (R)cxxi;
        if (p == 0) {
            mref[4 * e + 0] = r0;
            mref[4 * e + 1] = r1;
            mref[4 * e + 2] = r2;
            mref[4 * e + 3] = r3;
        }
        Ax[q] = (R)(yeta - (double)r0);
        Cx[q] = (R)(-xeta - (double)r1);
        Ae[q] = (R)(-yxi - (double)r2);
        Ce[q] = (R)(xxi - (double)r3);
    } else {
        Ax[q] = (R)yeta;
        Cx[q] = (R)(-xeta);
        Ae[q] = (R)(-yxi);
        Ce[q] = (R)xxi;
    }
}

// Split-form bathymetry derivatives (eq. SourceDisc, read with D), face traces
// and nodal copy of the caller's bathymetry b, whose element perm[e] is
// internal element e; metric terms in float64 from the coordinates.  A tile's
// coordinates, b and the products of its metric terms with b are staged in
// LDS: with every thread forming the metric terms of both its lines again
// from global memory (4(N+1)^2 cached loads a line), behind a pass that
// brought b into internal order and before one that copied it, the three took
// 66 us at 128^2, N = 5; now 12.4 (N = 7, 512^2: 2370 -> 208).
template <int N, typename R>
__global__ __launch_bounds__(Shape<N>::T) void bathymetry_kernel(int64_t K, const double *__restrict__ x,
                                                                 const double *__restrict__ y,
                                                                 const double *__restrict__ b,
                                                                 const int32_t *__restrict__ perm, R *bx, R *by,
                                                                 R *bface, R *bnode, int64_t ntiles,
                                                                 Tab<double> tab)
{
    using S = Shape<N>;
    constexpr int nf = S::nf, np = S::np, E = S::E, T = S::T;
    __shared__ double s_x[T], s_y[T], s_b[T], s_p[4][T], s_D[nf * nf];
    const int64_t tile = xcd_tile(ntiles);
    if (tile < 0) return;
    const int t = threadIdx.x;
    const bool lane = t < E * np;
    const int el = lane ? t / np : E - 1, p = lane ? t - el * np : 0, i = p / nf, j = p - i * nf;
    const int64_t e = tile * E + el;
    const bool act = lane && e < K;
    const int64_t q = act ? e * np + p : 0;
    for (int c = t; c < nf * nf; c += T) s_D[c] = tab.D[c];
    const int64_t q0 = act ? e * np : 0;
    const double bn = act ? b[(int64_t)perm[e] * np + p] : 0.0;
    s_x[t] = x[q] - x[q0];
    s_y[t] = y[q] - y[q0];
    lds_sync<T>();
    const int base = el * np;
    double xxi = 0, xeta = 0, yxi = 0, yeta = 0;
    for (int m = 0; m < nf; ++m) {
        const double di = s_D[i * nf + m], dj = s_D[j * nf + m];
        xxi += di * s_x[base + m * nf + j];
        yxi += di * s_y[base + m * nf + j];
        xeta += dj * s_x[base + i * nf + m];
        yeta += dj * s_y[base + i * nf + m];
    }
    s_b[t] = bn;
    s_p[0][t] = yeta * bn;
    s_p[1][t] = xeta * bn;
    s_p[2][t] = yxi * bn;
    s_p[3][t] = xxi * bn;
    lds_sync<T>();
    double Db_xi = 0, Dyb_xi = 0, Dxb_xi = 0, Db_eta = 0, Dyb_eta = 0, Dxb_eta = 0;
    for (int m = 0; m < nf; ++m) {
        const double dxi = s_D[i * nf + m], deta = s_D[j * nf + m];
        const int qi = base + m * nf + j, qe = base + i * nf + m;
        Db_xi += dxi * s_b[qi];
        Dyb_xi += dxi * s_p[0][qi];   // y_eta b
        Dxb_xi += dxi * s_p[1][qi];   // x_eta b
        Db_eta += deta * s_b[qe];
        Dyb_eta += deta * s_p[2][qe]; // y_xi b
        Dxb_eta += deta * s_p[3][qe]; // x_xi b
    }
    if (!act) return;
    bx[q] = (R)(yeta * Db_xi + Dyb_xi - yxi * Db_eta - Dyb_eta);
    by[q] = (R)(-xeta * Db_xi - Dxb_xi + xxi * Db_eta + Dxb_eta);
    bnode[q] = (R)bn;
    // face traces: the thread of a face node writes every side the node is on
    if (j == 0) bface[(e * 4 + 0) * nf + i] = (R)bn;
    if (i == N) bface[(e * 4 + 1) * nf + j] = (R)bn;
    if (j == N) bface[(e * 4 + 2) * nf + i] = (R)bn;
    if (i == 0) bface[(e * 4 + 3) * nf + j] = (R)bn;
}

// ------------------------------------------------------------------------
// Cross-lane reductions inside one wave with DPP moves (GFX9 encodings:
// quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E, row_mirror = 0x140,
// row_half_mirror = 0x141, row_bcast:15 = 0x142, row_bcast:31 = 0x143).
// Lanes of rows outside ROWMASK receive an unspecified value.  Called in
// uniform control flow with every lane of the wave active.
// ------------------------------------------------------------------------
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_mov(double v)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)x, CTRL, ROWMASK, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, ROWMASK, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, ROWMASK, 0xF, false));
}

__device__ __forceinline__ double read_lane63(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ float read_lane63(float v)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

template <bool MIN, int CTRL, int ROWMASK, typename R>
__device__ __forceinline__ R dpp_step(R v)
{
    const R o = dpp_mov<CTRL, ROWMASK>(v);
    return MIN ? fmin(o, v) : v + o;
}

// Sum (MIN: minimum) over the 16 lanes of each row, in every lane of the row
// (the four patterns read valid lanes only).
template <bool MIN, typename R>
__device__ __forceinline__ R row16_reduce(R v)
{
    v = dpp_step<MIN, 0xB1, 0xF>(v);
    v = dpp_step<MIN, 0x4E, 0xF>(v);
    v = dpp_step<MIN, 0x141, 0xF>(v);
    return dpp_step<MIN, 0x140, 0xF>(v);
}

// Sum (MIN: minimum) over the 64 lanes of the wave, in every lane: the row
// totals are carried into lane 63 (rows 1, 3 add row 0, 2; rows 2, 3 add
// lane 31), whose value is broadcast; the other lanes' partials are not used.
template <bool MIN, typename R>
__device__ __forceinline__ R wave64_reduce(R v)
{
    v = row16_reduce<MIN>(v);
    v = dpp_step<MIN, 0x142, 0xA>(v);
    v = dpp_step<MIN, 0x143, 0xC>(v);
    return read_lane63(v);
}

// True in every thread if pred holds in some thread of the workgroup.
template <int T>
__device__ __forceinline__ bool block_any(bool pred)
{
    if constexpr (T == 64) return __ballot(pred) != 0ull;   // one wave
    else return __syncthreads_or(pred) != 0;
}

// The same through flag, T/64 ints of LDS used for nothing else: one barrier
// that does not wait for global stores, as __syncthreads_or() would.
template <int T>
__device__ __forceinline__ bool block_any_lds(bool pred, int *flag, int t)
{
    const bool mine = __ballot(pred) != 0ull;
    if constexpr (T == 64) return mine;
    if ((t & 63) == 0) flag[t >> 6] = mine;
    lds_sync<T>();
    int any = 0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) any |= flag[w];
    return any != 0;
}

// ------------------------------------------------------------------------
// Workgroup-level per-element reductions over the nodes of each element.
// red: LDS scratch of T*NQ reals; returns the element total in every thread.
// ------------------------------------------------------------------------
template <int N, typename R, int NQ>
struct ElemReduce {
    static constexpr int nf = N + 1, np = nf * nf, E = Shape<N>::E, T = Shape<N>::T;
    // v[0..NQ-1] summed, except v[NQ-1] which is reduced by min when MINLAST
    template <bool MINLAST>
    __device__ __forceinline__ static void run(R (&v)[NQ], R *red, int t, int el, int p)
    {
#pragma unroll
        for (int c = 0; c < NQ; ++c) red[c * T + t] = v[c];
        lds_sync<T>();
        R part[NQ];
        const bool row = (t < E * np) && (p < nf);   // thread (el, p<nf) reduces column p
        if (row) {
#pragma unroll
            for (int c = 0; c < NQ; ++c) {
                R s = red[c * T + el * np + p];
#pragma unroll
                for (int r = 1; r < nf; ++r) {
                    const R val = red[c * T + el * np + r * nf + p];
                    if (MINLAST && c == NQ - 1) s = val < s ? val : s;
                    else s += val;
                }
                part[c] = s;
            }
        }
        lds_sync<T>();
        if (row) {
#pragma unroll
            for (int c = 0; c < NQ; ++c) red[c * T + el * np + p] = part[c];
        }
        lds_sync<T>();
        if (t < E * np) {
#pragma unroll
            for (int c = 0; c < NQ; ++c) {
                R s = red[c * T + el * np];
#pragma unroll
                for (int r = 1; r < nf; ++r) {
                    const R val = red[c * T + el * np + r];
                    if (MINLAST && c == NQ - 1) s = val < s ? val : s;
                    else s += val;
                }
                v[c] = s;
            }
        }
        lds_sync<T>();
    }
};

// Element totals: NQ values per thread summed over the nodes of each element
// (the last reduced by min when MINLAST); only thread p == 0 of each element
// receives the totals.  Two barriers; red: NQ*T reals of LDS.  The caller
// synchronises before reusing red.
template <int N, typename R, int NQ, bool MINLAST, int T = Shape<N>::T>
__device__ __forceinline__ void elem_totals(R (&v)[NQ], R *red, int t, int el, int p, bool lane)
{
    constexpr int nf = N + 1, np = nf * nf;
#pragma unroll
    for (int c = 0; c < NQ; ++c) red[c * T + t] = v[c];
    lds_sync<T>();
    if (lane && p < nf) {
        // column p of element el; its total goes to the column's first slot,
        // which only this thread reads
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            R s = red[c * T + el * np + p];
#pragma unroll
            for (int r = 1; r < nf; ++r) {
                const R val = red[c * T + el * np + r * nf + p];
                if (MINLAST && c == NQ - 1) s = val < s ? val : s;
                else s += val;
            }
            red[c * T + el * np + p] = s;
        }
    }
    lds_sync<T>();
    if (lane && p == 0) {
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            R s = red[c * T + el * np];
#pragma unroll
            for (int r = 1; r < nf; ++r) {
                const R val = red[c * T + el * np + r];
                if (MINLAST && c == NQ - 1) s = val < s ? val : s;
                else s += val;
            }
            v[c] = s;
        }
    }
}

// Element totals as elem_totals (valid at least in thread p == 0): with lane
// exchanges where an element is one whole wave (np = 64) or one 16-lane row
// of a one-wave workgroup (np = 16), through LDS otherwise.
template <int N, typename R, int NQ, bool MINLAST, int T = Shape<N>::T>
__device__ __forceinline__ void elem_totals_any(R (&v)[NQ], R *red, int t, int el, int p, bool lane)
{
    constexpr int np = (N + 1) * (N + 1);
    if constexpr (np == 64 && T % 64 == 0) {
        // one element per wave
#pragma unroll
        for (int c = 0; c < NQ; ++c)
            v[c] = (MINLAST && c == NQ - 1) ? wave64_reduce<true>(v[c]) : wave64_reduce<false>(v[c]);
    } else if constexpr (np == 16 && T % 64 == 0) {
        // one element per 16-lane row
#pragma unroll
        for (int c = 0; c < NQ; ++c)
            v[c] = (MINLAST && c == NQ - 1) ? row16_reduce<true>(v[c]) : row16_reduce<false>(v[c]);
    } else {
        elem_totals<N, R, NQ, MINLAST, T>(v, red, t, el, p, lane);
    }
}

// ------------------------------------------------------------------------
// Artificial viscosity (appendix A, Theorem 1)
// ------------------------------------------------------------------------
// Viscosity from the indicator's element totals: modal energy of all modes,
// of the top shell, of the modes up to N-1 and of shell N-1; zero for a dry
// element (no node above h_tol).
template <typename R>
__device__ __forceinline__ R viscosity_from_totals(R all, R top, R allM, R topM, bool wet, const Phys<R> &P)
{
    if (!wet) return R(0);
    // smooth elements (both fractions clearly below 10^sigma_min) leave
    // before the divisions; the margin keeps the decision that of the
    // quotients below
    const R pre = R(0.999999) * P.ratio_min;
    if (!(top > pre * all) && !(topM > pre * allM)) return R(0);
    const R r1 = all > R(0) ? top / all : R(0);
    const R r2 = allM > R(0) ? topM / allM : R(0);
    const R rm = r1 > r2 ? r1 : r2;
    // sigma = log10(rm) against the thresholds, compared as rm against
    // 10^sigma (the ramp is continuous at both ends); log10 and sin only on
    // the ramp
    if (!(rm > P.ratio_min)) return R(0);
    if (rm >= P.ratio_max) return P.eps0;
    const R sg = log10(rm);
    const R smin = P.sigma_min, smax = P.sigma_max;
    if (sg >= smax) return P.eps0;
    if (!(sg > smin)) return R(0);
    return R(0.5) * P.eps0 *
           (R(1) + sin(R(3.14159265358979323846) * (sg - R(0.5) * (smax + smin)) / (smax - smin)));
}

// Is nodal line l (l < 2(N+1): the lines of the two directions) of an
// element whose heights sit at sh[i*(N+1) + j] certainly smooth?  An element
// with 2(N+1) smooth lines has no viscosity, so that the modal transform of
// element_viscosity is only needed where some line is not smooth.
//
// With c_j the coefficient of mode N of xi-line j and d_i that of eta-line i,
// the top shell's energy is at most the sum over both sets of lines of their
// squared L2 norms along the other direction, hence at most sum_j w_j c_j^2 +
// sum_i w_i d_i^2 (the LGL rule overestimates squares of degree N).  The
// energy of all modes is at least (N / (2N+1))^2 sum_ij w_i w_j h_ij^2 (it
// overestimates by at most 2 + 1/N per direction), and sum_r w_r h_r^2 on a
// line is at least half the square of m = sum_r w_r h_r.  So c^2 <= tau m^2
// on every line, with 2 tau = 0.99 x (N / (2N+1))^2 / 2 x 10^sigma_min x (1 -
// 10^sigma_min), keeps the top shell's share below 10^sigma_min, and the same
// for mode N - 1 keeps shell N - 1's share of the modes up to N - 1 below it:
// the exact test of viscosity_from_totals would give zero too.  tau = 0
// (thresholds near rounding, see phys()) leaves every element to that test.
//
// Per line N+1 LDS reads and about 4(N+1) + 6 operations (eight per mirrored
// pair of nodes) on 2(N+1) lanes, against 4(N+1) reads, 2(N+1) multiply-adds
// and three reductions on every lane for the transform, with which the
// epilogue was bound by LDS and its barriers.  The stage kernel of a smooth
// flow took 5% less for it at N = 7, 512^2 (float32, 384^2: 10%), 15% at N = 5,
// 255^2, 9% at N = 2, 601^2 (571, 214, 107 and 152 us before).  Tiles at
// wet/dry fronts pay for both tests: even on a 200^2, N = 3 mesh of which a
// twentieth is such.
template <int N, typename R>
__device__ __forceinline__ bool smooth_line(const R *sh, int l, const Uni<R> &tab, R tau)
{
    constexpr int nf = N + 1;
    const int o = l < nf ? l : (l - nf) * nf, st = l < nf ? nf : 1;
    // the nodes and modes are symmetric: even modes from the sums of mirrored
    // nodes, odd ones from their differences
    constexpr int half = nf / 2;
    constexpr bool odd = (N & 1) != 0;
    R m = 0, ce = 0, co = 0;   // mean, even and odd mode of N and N - 1
    const R mid = odd ? sh[o] : sh[o + half * st];
    // (the even mode's sum over jumps from one node: no rounding at the size
    // of h itself, which single precision would see)
#pragma unroll
    for (int r = 0; r < half; ++r) {
        const R a = sh[o + r * st], b = sh[o + (N - r) * st];
        m += tab.w[r] * (a + b);
        ce += tab.ve[r] * ((a - mid) + (b - mid));
        co += tab.vo[r] * (a - b);
    }
    if constexpr (!odd) m += tab.w[half] * mid;
    const R lim = tau * m * m;
    return ce * ce <= lim && co * co <= lim;
}

// Lane t's line of a tile of E elements, node (i, j) of element el at
// sh[el*np + i*(N+1) + j]: true if the element needs element_viscosity.
template <int N, typename R, int E>
__device__ __forceinline__ bool rough_line(const R *sh, int t, const Uni<R> &tab, const Phys<R> &P)
{
    constexpr int nf = N + 1, np = nf * nf;
    if (!(P.smooth_tau > R(0))) return true;
    if (t >= E * 2 * nf) return false;
    const int el = t / (2 * nf);
    return !smooth_line<N, R>(sh + el * np, t - el * 2 * nf, tab, P.smooth_tau);
}

// Element viscosity of the elements whose nodal water heights are staged in
// sh[el*np + p]: modal coefficients Q^ = V^{-1} h V^{-T}, the energy
// fractions of the top two mode shells, sigma = log10 of the larger, and the
// sine ramp between sigma_min and sigma_max; zero for dry elements.  The
// result is valid in thread p == 0 of each element.  red: 6*T reals of LDS
// (the last T hold the intermediate V^{-1} h); vinv: V^{-1} row-major with
// row stride N+1, staged in LDS by the caller (stage_vinv).  Three barriers.
template <int N, typename R, int T = Shape<N>::T>
__device__ R element_viscosity(const R *sh, R *red, const R *vinv, const Phys<R> &P, int t, int el, int p,
                               bool lane, R h)
{
    constexpr int nf = N + 1, np = nf * nf;
    const int i = p / nf, j = p - i * nf;
    // single precision transforms h - c (c the element's first nodal height):
    // the higher modes of a smooth element are small against h itself, and
    // in h their FP32 rounding would move the energy ratios, hence eps on
    // the ramp.  A constant has the one mode (0, 0), of coefficient 2c (the
    // orthonormal Legendre L_0 = 1/sqrt(2) in both directions), restored below.
    const R c0 = (kJumpForm<R> && lane) ? sh[el * np] : R(0);
    R Tq = 0;
    if (lane) {
#pragma unroll
        for (int r = 0; r < nf; ++r) Tq += vinv[i * nf + r] * (sh[el * np + r * nf + j] - c0);
    }
    red[5 * T + t] = Tq;
    lds_sync<T>();
    R Qh = 0;
    if (lane) {
#pragma unroll
        for (int c = 0; c < nf; ++c) Qh += red[5 * T + el * np + i * nf + c] * vinv[j * nf + c];
    }
    if constexpr (kJumpForm<R>)
        if (p == 0) Qh += R(2) * c0;
    const R q2 = Qh * Qh;
    const int mx = i > j ? i : j;
    // the energy of all modes is the top shell's plus that of the modes up to N-1
    if constexpr ((np == 64 || np == 16) && T % 64 == 0) {
        // the element's lanes lie in one wave: its wetness by a ballot
        // instead of a max reduction of h
        const uint64_t wm = __ballot(lane && h > P.h_tol);
        const uint64_t mine = np == 64 ? ~0ull : (0xFFFFull << ((t & 63) - p));
        R vals[3] = {mx == N ? q2 : R(0), mx <= N - 1 ? q2 : R(0), mx == N - 1 ? q2 : R(0)};
        elem_totals_any<N, R, 3, false, T>(vals, red, t, el, p, lane);
        return viscosity_from_totals<R>(vals[0] + vals[1], vals[0], vals[1], vals[2], (wm & mine) != 0ull, P);
    } else {
        R vals[4] = {mx == N ? q2 : R(0), mx <= N - 1 ? q2 : R(0), mx == N - 1 ? q2 : R(0),
                     lane ? -h : R(3.0e38)};
        elem_totals_any<N, R, 4, true, T>(vals, red, t, el, p, lane);
        return viscosity_from_totals<R>(vals[0] + vals[1], vals[0], vals[1], vals[2], -vals[3] > P.h_tol, P);
    }
}

// Copy V^{-1} (row stride N+1) into LDS; ordered by the caller's next barrier.
template <int N, typename R, int T>
__device__ __forceinline__ void stage_vinv(R *dst, const Tab<R> &tab, int t)
{
    constexpr int nf = N + 1;
    for (int q = t; q < nf * nf; q += T) dst[q] = tab.Vinv[q];
}

// ------------------------------------------------------------------------
// Stage kernel
// ------------------------------------------------------------------------
enum StageMode { kModeRhs = 0, kModeLsrk = 1, kModeSsp = 2 };

// CFL bound of one node: cfl (2/(N+1)) J / (|(A_xi . u)| + c |A_xi| + |(A_eta . u)| + c |A_eta|),
// with the contravariant directions A_xi = (Ax, Cx), A_eta = (Ae, Ce).
template <int N, typename R>
__device__ __forceinline__ R cfl_bound(R h, R hu, R hv, R Ax, R Cx, R Ae, R Ce, R J, const Phys<R> &P)
{
    const R ih = rcp_wet(h, P.h_tol);
    const R u = hu * ih, v = hv * ih;
    const R cs = sqrt_nr(P.g * fmax(h, R(0)));
    const R lx = fabs(Ax * u + Cx * v) + cs * sqrt_nr(Ax * Ax + Cx * Cx);
    const R le = fabs(Ae * u + Ce * v) + cs * sqrt_nr(Ae * Ae + Ce * Ce);
    return lx + le > R(0) ? P.cfl * (R(2) / R(N + 1)) * J / (lx + le) : R(3.0e38);
}

// Viscous bound of an element with viscosity eps > 0.
template <typename R>
__device__ __forceinline__ R visc_bound(R eps, R gmax, const Phys<R> &P)
{
    return P.visc_c / (P.br1 * eps * gmax);
}

template <typename R> struct Vec2;
template <> struct Vec2<double> { using type = double2; };
template <> struct Vec2<float> { using type = float2; };

template <typename R>
struct StageArgs {
    Mesh<R> m;
    Phys<R> P;
    Uni<R> tab;                  // uniform entries (read as scalars)
    const Tab<R> *tg;            // the same tables in device memory: per-lane entries
    const R *h, *hu, *hv;        // stage input W
    const R *h0, *hu0, *hv0;     // SSP: W^n
    R *oh, *ohu, *ohv;           // output: R (rhs mode) or the new state
    const int32_t *perm;         // rhs mode: the caller's element of each (nullptr: internal order)
    R *dh, *dhu, *dhv;           // LSRK register dU (in place)
    int store_du;                // 0 on the last LSRK stage: the next step's first stage does not read dU
    // artificial viscosity (nullptr eps: off)
    const R *eps;                // [K] viscosity of the input state
    const R *vfl;                // [K][4][nf][2] face_parts of its elements with viscosity
    R *eps_out, *vfl_out;        // the same of the output state (update modes)
    R *dtc_out, *dtv_out;        // last stage of a step: per-element CFL / viscous bounds of the output
    R *frec_out;                 // with them (limiter on): face records [K][4][nf][3] (h, u, v) of the output
    const int32_t *inst;         // [K] instance of each element (ensembles), nullptr: one instance
    const R *gmax;               // [K] max |grad xi|^2 + |grad eta|^2 (viscous bound)
    const double *dt;            // per instance k: the current step at dt[8k]
    R ca, cb;                    // LSRK a_k, b_k; SSP alpha_k, beta_k
    int *flags;                  // status flags (kFlag*)
    int *iflags;                 // [instance] step flags that ensembles with step retries read (1: negative mean)
    const int *imask;            // with inst: only elements of instances k with imask[k] != 0 (a retry of
                                 // some instances), else nullptr
    int64_t ntiles;
    int variant;                 // compiled variant 0..kStageVariants-1 (launch side)
};

// ---- artificial viscosity (Theorem 1, eq. BR1) ----
// The viscous flux h eps grad u of an element needs the derivatives of its
// own velocities and, on its sides, the jumps U* - u = (u_nbr - u) / 2.  Its
// neighbours need n . (h eps grad u) on the shared sides.  The part without
// the jumps is known where the element's state is: whoever computes a viscosity
// eps > 0 (the stage kernel's epilogue, the indicator pass) leaves it per face
// node (face_parts), and the next stage kernel adds the jumps to it
// (nbr_viscous_flux) and forms the element's own divergence from its staged
// velocities.  So a stage is one launch: with the viscous fluxes and their
// divergence in two passes of their own, over a list of elements, most often
// empty, each stage spent two more launches of 4.6-5 us.

// Derivatives along both lines through node (i, j) of a pair of staged
// values: the D rows from the zero-diagonal table dz, whose missing diagonal
// is -+N(N+1)/4 at the ends and zero between; at(i, j) returns the pair.
// Single precision sums over the jumps from the node's own values (D's rows
// sum to zero), so that neither the rounding of the table's row sums nor that
// of products at the size of the values themselves enters (kJumpForm).
template <int N, typename R, typename At>
__device__ __forceinline__ void line_derivatives(const R *dz, int i, int j, const At &at, typename Vec2<R>::type own,
                                                 R &dx1, R &dx2, R &de1, R &de2)
{
    constexpr int nf = N + 1;
    constexpr R end = R(0.25) * R(N * (N + 1));
    const R o1 = kJumpForm<R> ? own.x : R(0), o2 = kJumpForm<R> ? own.y : R(0);
    dx1 = dx2 = de1 = de2 = R(0);
#pragma unroll 2
    for (int m = 0; m < nf; ++m) {
        R di = dz[i * nf + m], dj = dz[j * nf + m];
        if constexpr (!kJumpForm<R>) {
            if (m == i) di = i == N ? end : (i == 0 ? -end : R(0));
            if (m == j) dj = j == N ? end : (j == 0 ? -end : R(0));
        }
        const auto a = at(m, j), b = at(i, m);
        dx1 += di * (a.x - o1);
        dx2 += di * (a.y - o2);
        de1 += dj * (b.x - o1);
        de2 += dj * (b.y - o2);
    }
}

// n . (h eps grad u), n . (h eps grad v) without the side jumps at node
// (i, j) of element e, n the outward scaled normal, for each side that the
// node lies on, to vfl [K][4][nf][2].  he: h eps at the node.
template <int N, typename R, typename At>
__device__ __forceinline__ void face_parts(R *vfl, const R *dz, int64_t e, int i, int j, const At &at,
                                           typename Vec2<R>::type own, R he, R Ax, R Cx, R Ae, R Ce)
{
    constexpr int nf = N + 1;
    R dxu, dxv, deu, dev;
    line_derivatives<N, R>(dz, i, j, at, own, dxu, dxv, deu, dev);
    const R sc = he / (Ce * Ax - Cx * Ae);
    const R aa = sc * (Ax * Ax + Cx * Cx), ae = sc * (Ax * Ae + Cx * Ce), ee = sc * (Ae * Ae + Ce * Ce);
    const R xu = aa * dxu + ae * deu, xv = aa * dxv + ae * dev;   // normal (Ax, Cx)
    const R yu = ae * dxu + ee * deu, yv = ae * dxv + ee * dev;   // normal (Ae, Ce)
    auto rec = [&](int s, int k, R a, R b) {
        R *const r = vfl + ((e * 4 + s) * nf + k) * 2;
        r[0] = a;
        r[1] = b;
    };
    if (j == 0) rec(0, i, -yu, -yv);
    if (i == N) rec(1, j, xu, xv);
    if (j == N) rec(2, i, yu, yv);
    if (i == 0) rec(3, j, -xu, -xv);
}

// Half the jump of (u, v) across side s at node k of element e, whose own
// velocities there are (u0, v0): U* - u, V* - v (zero at a wall, which names
// the node itself).
template <int N, typename R>
__device__ __forceinline__ void side_jump(const StageArgs<R> &a, int64_t e, int s, int k, R u0, R v0, R &ju, R &jv)
{
    int64_t en;
    int ns, kk;
    const int64_t qn = nbr_node<N>(a.m, e, s, k, en, ns, kk);
    const R in = rcp_wet(a.h[qn], a.P.h_tol);
    ju = R(0.5) * (a.hu[qn] * in - u0);
    jv = R(0.5) * (a.hv[qn] * in - v0);
}

// n . (h eps grad u), n . (h eps grad v) of element e (eps > 0) at node k of
// its side s, n its outward scaled normal, with the velocities (uo, vo) across
// the side.
template <int N, typename R>
__device__ __forceinline__ void nbr_viscous_flux(const StageArgs<R> &a, int64_t e, int s, int k, R uo, R vo, R &fu,
                                                 R &fv)
{
    constexpr int nf = N + 1, np = nf * nf;
    int i, j;
    side_node<N>(s, k, i, j);
    const R *const r = a.vfl + ((e * 4 + s) * nf + k) * 2;
    fu = r[0];
    fv = r[1];
    // a corner also lies on a side t of the other direction (any other node:
    // the same loads on side s, left out below, so that no branch holds them up)
    const int t = (s & 1) ? (j == N ? 2 : (j == 0 ? 0 : -1)) : (i == N ? 1 : (i == 0 ? 3 : -1));
    int64_t ec;
    int nc, kc;
    const int64_t qc = nbr_node<N>(a.m, e, t >= 0 ? t : s, t >= 0 ? ((s & 1) ? i : j) : k, ec, nc, kc);
    const R hc = a.h[qc], huc = a.hu[qc], hvc = a.hv[qc];
    const int64_t q = e * np + i * nf + j;
    R Ax, Cx, Ae, Ce;
    metric_at(a.m, q, e, Ax, Cx, Ae, Ce);
    const R h = a.h[q], ih = rcp_wet(h, a.P.h_tol), u = a.hu[q] * ih, v = a.hv[q] * ih;
    const R sc = a.tab.iw0 * h * a.eps[e] / (Ce * Ax - Cx * Ae);
    const R aa = sc * (Ax * Ax + Cx * Cx), ae = sc * (Ax * Ae + Cx * Ce), ee = sc * (Ae * Ae + Ce * Ce);
    // the jump across a side enters the derivative along its normal with the
    // side's sign, and n . the metric once more: squared on the side itself
    const R d = (s & 1) ? aa : ee;
    fu += d * R(0.5) * (uo - u);
    fv += d * R(0.5) * (vo - v);
    if (t >= 0) {
        const R ic = rcp_wet(hc, a.P.h_tol);
        const bool pos = ((s == 1 || s == 2) == (t == 1 || t == 2));
        fu += (pos ? ae : -ae) * (R(0.5) * (huc * ic - u));
        fv += (pos ? ae : -ae) * (R(0.5) * (hvc * ic - v));
    }
}

// Indicator sweep over all elements (initial data, or after the state was
// replaced): element viscosity and the viscous face fluxes' own part.
template <int N, typename R>
struct IndicatorArgs {
    Phys<R> P;
    Uni<R> tab;                  // uniform entries (read as scalars)
    const Tab<R> *tg;            // the same tables in device memory: per-lane entries
    int64_t K;
    Mesh<R> m;
    const R *h, *hu, *hv;
    R *eps;             // [K]
    R *vfl;             // [K][4][nf][2]
    int64_t ntiles;
};

template <int N, typename R>
__global__ __launch_bounds__(Shape<N>::T) void indicator_kernel(IndicatorArgs<N, R> a)
{
    using S = Shape<N>;
    constexpr int np = S::np, E = S::E, T = S::T;
    __shared__ __align__(16) R s_red[6 * T];
    __shared__ R s_h[T], s_vinv[(N + 1) * (N + 1)];
    __shared__ int s_any[2][T / 64];
    const int64_t tile = xcd_tile(a.ntiles);
    if (tile < 0) return;
    const int t = threadIdx.x;
    stage_vinv<N, R, T>(s_vinv, *a.tg, t);
    const bool lane = t < E * np;
    const int el = lane ? t / np : E - 1, p = lane ? t - el * np : 0;
    const int64_t e = tile * E + el;
    const bool act = lane && (e < a.K);
    const R h = act ? a.h[e * np + p] : R(0);
    s_h[t] = h;
    lds_sync<T>();
    R eps = R(0);
    if (block_any_lds<T>(rough_line<N, R, E>(s_h, t, a.tab, a.P), s_any[0], t))
        eps = element_viscosity<N, R>(s_h, s_red, s_vinv, a.P, t, el, p, lane, h);
    if (act && p == 0) a.eps[e] = eps;
    // (as in the stage kernel's epilogue)
    if (!block_any_lds<T>(act && p == 0 && eps > R(0), s_any[1], t)) return;
    using V2 = typename Vec2<R>::type;
    V2 *const s_w = (V2 *)s_red;
    const int64_t q = e * np + p;
    const R ih = rcp_wet(h, a.P.h_tol);
    const V2 w = act ? V2{a.hu[q] * ih, a.hv[q] * ih} : V2{R(0), R(0)};
    lds_sync<T>();
    if (lane && p == 0) s_h[el * np] = eps;
    s_w[t] = w;
    for (int c = t; c < np; c += T) s_vinv[c] = a.tg->Dz[c];
    lds_sync<T>();
    const int i = p / (N + 1), j = p - i * (N + 1);
    const R ev = s_h[el * np];
    if (act && ev > R(0) && (i == 0 || i == N || j == 0 || j == N)) {
        R Ax, Cx, Ae, Ce;
        metric_at(a.m, q, e, Ax, Cx, Ae, Ce);
        face_parts<N, R>(a.vfl, s_vinv, e, i, j, [&](int r, int c) { return s_w[el * np + r * (N + 1) + c]; }, w,
                         h * ev, Ax, Cx, Ae, Ce);
    }
}

// Face slot data loaded ahead of the LDS staging (slots t, t + T, ... of lane t).
// Kept small (it is live across the LDS staging): the neighbour element and
// one packed word.
template <typename R>
struct FacePrefetch {
    int32_t en = 0;          // neighbour element
    int code = 0;            // neighbour side | face node << 2 | (visc_nbr) << 8 | wall << 9
    R h = 0, hu = 0, hv = 0, bo = 0, bn = 0;
    __device__ int ns() const { return code & 3; }
    __device__ int kk() const { return (code >> 2) & 63; }
    // with AV: the neighbour (not a wall) has viscosity
    __device__ bool visc_nbr() const { return (code >> 8) & 1; }
    __device__ bool wall() const { return (code >> 9) & 1; }
};

// Slot f of the tile whose first element is e0.
template <int N, typename R, int E, int NF>
__device__ __forceinline__ void prefetch_face(const StageArgs<R> &a, int f, int64_t e0, FacePrefetch<R> &pf)
{
    constexpr int nf = N + 1, np = nf * nf;
    if (f >= NF) return;
    const int side = f / nf, fel = side / 4, k = f - side * nf;
    if (e0 + fel >= a.m.K) return;
    const int32_t en = (a.m.nbr + 4 * e0)[side];
    const int c = (a.m.code + 4 * e0)[side];
    pf.bo = (a.m.bface + e0 * 4 * nf)[f];
    const int ns = c & 3, kk = (c & 4) ? N - k : k;
    int i, j;
    side_node<N>(ns, kk, i, j);
    if ((uint32_t)(en - (int32_t)e0) >= (uint32_t)E) {
        const uint64_t qn = (uint64_t)(uint32_t)en * np + (uint32_t)(i * nf + j);
        pf.h = a.h[qn];
        pf.hu = a.hu[qn];
        pf.hv = a.hv[qn];
    }
    pf.bn = a.m.bface[(uint64_t)(uint32_t)en * (4 * nf) + (uint32_t)(ns * nf + kk)];
    const bool vn = a.eps && !(c & 8) && a.eps[en] > R(0);
    pf.en = en;
    pf.code = ns | (kk << 2) | ((int)vn << 8) | ((c & 8) << 6);
}

template <int N, typename R, int MODE, int V>
__global__ __launch_bounds__((StageCfg<N, V>::T), (StageWaves<N, R, MODE, V>::value)) void stage_kernel(StageArgs<R> a)
{
    using S = TileShape<N, StageCfg<N, V>::T>;
    constexpr int nf = S::nf, np = S::np, E = S::E, T = S::T, NF = S::NFACE;
    static_assert((T & (T - 1)) == 0, "workgroup size must be a power of two");
    using V2 = typename Vec2<R>::type;
    // one contiguous staging region: reused as reduction scratch at the end.
    // Pairs read together are stored together (one 16-byte LDS read in FP64).
    // Node (i, j) of tile element el sits at el*PS + i*RS + stage_col(i, j)
    // (RS = N + 1 + PAD); lanes past the tile's nodes write to spare slots
    // after them.
    constexpr int RS = nf + StageCfg<N, V>::PAD, PS = nf * RS, LEN = E * PS + (T - E * np);
    static_assert(LEN >= T, "staging rows");
    __shared__ __align__(16) R s_st[9 * LEN];
    V2 *const s_q = (V2 *)s_st;                 // (hu, hv)
    V2 *const s_w = (V2 *)(s_st + 2 * LEN);     // (u, v)
    V2 *const s_a = (V2 *)(s_st + 4 * LEN);     // J grad(xi)  = (Ax, Cx)
    V2 *const s_b = (V2 *)(s_st + 6 * LEN);     // J grad(eta) = (Ae, Ce)
    R *const s_h = s_st + 8 * LEN;
    __shared__ R s_fl[3][NF];
    __shared__ R s_lim[4 * E];
    __shared__ int s_any[4][T / 64];    // block_any_lds
    __shared__ R s_dz[nf * nf];         // D with a zero diagonal (volume term)
    __shared__ R s_mref[kMetricRel<R> ? 4 * E : 1];  // the tile elements' Mesh::mref (single precision)

    const int64_t tile = xcd_tile(a.ntiles);
    if (tile < 0) return;
    const int t = threadIdx.x;
    // lanes past the last element's nodes shadow node 0 of the last slot
    // (all LDS indices stay in range; they never store)
    const bool lane = t < E * np;
    const int el = lane ? t / np : E - 1, p = lane ? t - el * np : 0, i = p / nf, j = p - i * nf;
    const int64_t e0 = tile * E, e = e0 + el;
    const bool act = lane && (e < a.m.K) && (!a.imask || a.imask[a.inst[e]] != 0);
    // a retry of some instances: tiles with none of their elements leave
    // every output as it is
    if (a.imask && !block_any<T>(act)) return;
    // Node el*np + p of the tile is lane t's: every field is read and written
    // at its tile's start (a scalar) plus the one lane offset, which lanes
    // without a node of their own set to the tile's first node (their values
    // are never stored or summed).  One 64-bit address per field and lane,
    // masked loads and a table load behind the face slots' cost 2% at N = 7,
    // 512^2 (548 us), 8% at 128^2, 5% at N = 5, 255^2, 4% at N = 2, 601^2, and
    // in single precision 5% at N = 7, 384^2.
    const int64_t q0 = e0 * np;
    const uint32_t tq = act ? (uint32_t)t : 0u;
    const Phys<R> &P = a.P;
    const bool av = a.eps != nullptr;

    // the table first: its staging then waits for nothing behind it
    static_assert(nf * nf <= T, "one table entry per lane");
    const R dz_t = a.tg->Dz[t < nf * nf ? t : 0];
    const R h = (a.h + q0)[tq], hu = (a.hu + q0)[tq], hv = (a.hv + q0)[tq];
    R Ax = 0, Cx = 0, Ae = 0, Ce = 0;
    double xr = 0, yr = 0;
    if constexpr (kMetricInKernel<N, R>) {
        xr = (a.m.xr + q0)[tq]; yr = (a.m.yr + q0)[tq];
    } else {
        Ax = (a.m.Ax + q0)[tq]; Cx = (a.m.Cx + q0)[tq];
        Ae = (a.m.Ae + q0)[tq]; Ce = (a.m.Ce + q0)[tq];
    }
    // single precision: the stored terms are relative to the element's
    // middle node (kMetricRel); staged and held as they are until the volume
    // sums, the element's reference in LDS (s_mref)
    if constexpr (kMetricRel<R>) {
        if (act && p == 0) {
            const R *r = a.m.mref + 4 * e;
            s_mref[4 * el + 0] = r[0]; s_mref[4 * el + 1] = r[1];
            s_mref[4 * el + 2] = r[2]; s_mref[4 * el + 3] = r[3];
        }
    }
    // The face slots' neighbour traces and face bathymetry are loaded here,
    // with the element's own data, so that their latency is not paid a second
    // time after the LDS staging.  With more slots than lanes (N = 2) only
    // the first slot is prefetched; the lanes with a further slot load it
    // when they evaluate it.
    constexpr int NS = (NF + T - 1) / T;
    FacePrefetch<R> pf0;
    prefetch_face<N, R, E, NF>(a, t, e0, pf0);
    // has this lane's element viscosity (a lane mask; the value itself is
    // read again where it is used)
    const bool visc = av && act && (a.eps + e0)[el] > R(0);
    const R ih = rcp_wet(h, P.h_tol);
    const R u = hu * ih, v = hv * ih;
    const int st = lane ? el * PS + i * RS + stage_col<N, V>(i, j) : E * PS + (t - E * np);
    s_h[st] = h;
    s_q[st] = V2{hu, hv};
    s_w[st] = V2{u, v};
    if constexpr (kMetricInKernel<N, R>) {
        // metric terms from the staged coordinates: J grad(xi) = (y_eta, -x_eta),
        // J grad(eta) = (-y_xi, x_xi), each a derivative-matrix sum along a line
        // (eq. NablaRelation); D (with its diagonal) sits in the face-flux
        // slots until the face loop needs them
        static_assert(3 * NF >= nf * nf, "D in the face-flux slots");
        R *const s_D = &s_fl[0][0];
        s_a[st] = V2{xr, yr};
        for (int c = t; c < nf * nf; c += T) s_D[c] = a.tg->D[c];
        lds_sync<T>();
        const int base = el * PS;
        R xxi = 0, yxi = 0, xeta = 0, yeta = 0;
#pragma unroll 2
        for (int m = 0; m < nf; ++m) {
            const R di = s_D[i * nf + m], dj = s_D[j * nf + m];
            const V2 ci = s_a[base + m * RS + stage_col<N, V>(m, j)], cj = s_a[base + i * RS + stage_col<N, V>(i, m)];
            xxi += di * ci.x;
            yxi += di * ci.y;
            xeta += dj * cj.x;
            yeta += dj * cj.y;
        }
        Ax = yeta; Cx = -xeta; Ae = -yxi; Ce = xxi;
        lds_sync<T>();   // every lane's coordinate reads done before the metric replaces them
    }
    s_a[st] = V2{Ax, Cx};
    s_b[st] = V2{Ae, Ce};
    // the per-lane table entries of the volume term from LDS rather than
    // through the vector memory path (3-6% faster)
    if (t < nf * nf) s_dz[t] = dz_t;
    lds_sync<T>();

    // ---- interface: (1/w_0) J^surf F*(own, nbr, n_out) per face node, and
    // next to an element with viscosity the neighbour's half of the mean
    // viscous flux, (1/(2 w_0)) n . Fv_nbr with the neighbour's normal in L ----
    auto face_slot = [&](const int f, const FacePrefetch<R> &pfr) {
        const int side = f / nf, fel = side / 4, s = side & 3, k = f - side * nf;
        R c0 = 0, c1 = 0, c2 = 0;
        if (e0 + fel < a.m.K) {
            int fi, fj;
            side_node<N>(s, k, fi, fj);
            const int lp = fel * PS + fi * RS + stage_col<N, V>(fi, fj);
            // outward scaled normal: +-J grad(xi) on xi = +-1, +-J grad(eta) on eta = +-1
            V2 dir = (s & 1) ? s_a[lp] : s_b[lp];
            if constexpr (kMetricRel<R>) {
                dir.x += s_mref[4 * fel + ((s & 1) ? 0 : 2)];
                dir.y += s_mref[4 * fel + ((s & 1) ? 1 : 3)];
            }
            const R sg = (s == 0 || s == 3) ? R(-1) : R(1);
            const R snx = sg * dir.x, sny = sg * dir.y;
            R js, ijs;
            sqrt_rcp(snx * snx + sny * sny, js, ijs);
            // neighbour trace: from LDS when the neighbour is in this workgroup
            const uint32_t enl = (uint32_t)(pfr.en - (int32_t)e0);
            R hn, un, vn;
            if (enl < (uint32_t)E) {
                int ni, nj;
                side_node<N>(pfr.ns(), pfr.kk(), ni, nj);
                const int qs = (int)enl * PS + ni * RS + stage_col<N, V>(ni, nj);
                hn = s_h[qs];
                const V2 w = s_w[qs];
                un = w.x;
                vn = w.y;
            } else {
                hn = pfr.h;
                const R in = rcp_wet(hn, P.h_tol);
                un = pfr.hu * in;
                vn = pfr.hv * in;
            }
            const R bo = pfr.bo, bn = pfr.bn;
            if (pfr.wall()) wall_mirror(snx * ijs, sny * ijs, un, vn);
            R F0, F1, F2;
            const V2 wl = s_w[lp];
            if constexpr (kJumpForm<R>)
                interface_flux_delta<R>(s_h[lp], wl.x, wl.y, bo, hn, un, vn, bn, snx * ijs, sny * ijs, P,
                                        F0, F1, F2);
            else
                interface_flux<R>(s_h[lp], wl.x, wl.y, bo, hn, un, vn, bn, snx * ijs, sny * ijs, P, F0,
                                  F1, F2);
            const R sc = js * a.tab.iw0;
            c0 = sc * F0; c1 = sc * F1; c2 = sc * F2;
            // interface bathymetry penalty of eq. SourceDisc for a bottom
            // that jumps at the face, (1/w_0) (g/2) {h} [[b]] J^surf n in L
            // (zero for a continuous bottom and at walls, where bn = bo)
            const R pen = R(0.25) * P.g * a.tab.iw0 * (s_h[lp] + hn) * (bn - bo);
            c1 += pen * snx; c2 += pen * sny;
            if (__builtin_expect(av && pfr.visc_nbr(), 0)) {
                const StageArgs<R> &va = kernarg<StageArgs<R>>();
                R fu, fv;
                const V2 wo = s_w[lp];
                nbr_viscous_flux<N, R>(va, pfr.en, pfr.ns(), pfr.kk(), wo.x, wo.y, fu, fv);
                const R hw = R(0.5) * va.tab.iw0;
                c1 += hw * fu;
                c2 += hw * fv;
            }
        }
        s_fl[0][f] = c0; s_fl[1][f] = c1; s_fl[2][f] = c2;
    };
    if (t < NF) face_slot(t, pf0);
    if constexpr (NS > 1) {
        for (int f = t + T; f < NF; f += T) {
            FacePrefetch<R> pfl;
            prefetch_face<N, R, E, NF>(a, f, e0, pfl);
            face_slot(f, pfl);
        }
    }

    // ---- volume: sum_m 2 D_im F~(i,m) + sum_m 2 D_jm G~(j,m) (D~ has a zero
    // diagonal).  Per pair with contravariant direction (A, C):
    //   F1' = s_hu sA + s_hv sC,  F2' = s_u F1' + 2g h h_m sA,  F3' = s_v F1' + 2g h h_m sC
    // and 2 D F~ = D (F1'/2, F2'/4, F3'/4).  With s_u = u + u_m the sums split
    // into the own factors times partner sums, accumulated over both
    // directions at once:
    //   sum D F2' = u sum D F1' + sum D F1' u_m + 2g h sum D h_m sA   (F3' alike)
    R A1 = 0, A2 = 0, A3 = 0, C2 = 0, C3 = 0;
    if constexpr (kJumpForm<R>) {
        // single precision: the same sums taken over the partners' jumps
        // from the own node, dX = X_m - X.  With F1'(own) = 4 (hu A + hv C),
        // F2'(own) the own momentum part and e = dhu sA + dhv sC,
        //   F1'_m - F1'(own) = 2 (hu dA + hv dC) + e,  F1'_m = 2 (hu sA + hv sC) + e
        //   F2'_m - F2'(own) = 2u (F1'_m - F1'(own)) + du F1'_m + 2g h (h dA + dh sA)
        // (F3' alike), so sum_m D (F' - F'(own)) holds no term of the size of
        // the flux itself; the row-sum parts D~ 1 F'(own) left out are the
        // own-flux parts the face slots subtract (interface_flux_delta).  The
        // sums of D dA and D dC over both directions are the discrete metric
        // identities (D_xi y_eta = D_eta y_xi, the terms being D's own
        // derivatives of the coordinates): zero, left out, and with them the
        // rounding of the stored terms that they would add.  sA is pA, the same
        // for the whole line, plus the partner's small am.x: the sums of d dhu,
        // d dhv and d dh meet pA and pC after the loop (Hu, Hv, H), so that A1,
        // C2 and C3 are not rounded at full size per partner.  22 operations a
        // partner, against 27 with the jumps of A and C and their sums; this
        // kernel is bound by vector instructions.  The right-hand side's mass
        // error went from 7.4e-7 to 6.3e-7 of its maximum at N = 7, 512^2 (N =
        // 8: 8.2e-7 to 5.1e-7).  With e and dh sA summed as they are it is 18
        // operations and a stage 2% shorter, but errors of 1.1e-6 for both.
        const int base = el * PS;
        constexpr int VU = StageCfg<N, V>::VU32;
        // (the staged and own terms are relative to the element's middle
        // node: the sums of two absolute ones from the own plus twice the
        // reference)
        const R *const mr = s_mref + 4 * el;
        const R hu2 = R(2) * hu, hv2 = R(2) * hv;
        auto pair = [&](R d, V2 am, V2 qm, V2 wm, R hm, R pA, R pC, R F0, R &H, R &Hu, R &Hv) {
            const R dhu = qm.x - hu, dhv = qm.y - hv;
            const R q = dhu * am.x + dhv * am.y;
            const R dF = d * (q + (dhu * pA + (dhv * pC + (hu2 * am.x + (hv2 * am.y + F0)))));
            const R dh = d * (hm - h);
            Hu += d * dhu;
            Hv += d * dhv;
            A1 += d * q;
            A2 += dF * (wm.x - u);
            A3 += dF * (wm.y - v);
            H += dh;
            C2 += dh * am.x;
            C3 += dh * am.y;
        };
        {
            const R pA = Ax + R(2) * mr[0], pC = Cx + R(2) * mr[1];
            const R F0 = hu2 * pA + hv2 * pC;
            R H = 0, Hu = 0, Hv = 0;
#pragma unroll VU
            for (int mm = 0; mm < nf; ++mm) {
                const int qq = base + mm * RS + stage_col<N, V>(mm, j);
                pair(s_dz[i * nf + mm], s_a[qq], s_q[qq], s_w[qq], s_h[qq], pA, pC, F0, H, Hu, Hv);
            }
            C2 += H * pA;
            A1 += Hu * pA + Hv * pC;
            C3 += H * pC;
        }
        {
            const R pA = Ae + R(2) * mr[2], pC = Ce + R(2) * mr[3];
            const R F0 = hu2 * pA + hv2 * pC;
            R H = 0, Hu = 0, Hv = 0;
#pragma unroll VU
            for (int mm = 0; mm < nf; ++mm) {
                const int qq = base + i * RS + stage_col<N, V>(i, mm);
                pair(s_dz[j * nf + mm], s_b[qq], s_q[qq], s_w[qq], s_h[qq], pA, pC, F0, H, Hu, Hv);
            }
            C2 += H * pA;
            A1 += Hu * pA + Hv * pC;
            C3 += H * pC;
        }
    } else {
        const int base = el * PS;
        // partner-loop unroll of the variant (StageCfg)
        constexpr int VU = StageCfg<N, V>::VU;
#pragma unroll VU
        for (int mm = 0; mm < nf; ++mm) {
            // the self pair has coefficient 0 (no branch: D~ has a zero diagonal)
            const int qq = base + mm * RS + stage_col<N, V>(mm, j);
            const R d = s_dz[i * nf + mm];
            const V2 am = s_a[qq], qm = s_q[qq], wm = s_w[qq];
            const R sA = Ax + am.x, sC = Cx + am.y;
            const R df = d * ((hu + qm.x) * sA + (hv + qm.y) * sC);
            const R dh = d * s_h[qq];
            A1 += df;
            A2 += df * wm.x;
            A3 += df * wm.y;
            C2 += dh * sA;
            C3 += dh * sC;
        }
#pragma unroll VU
        for (int mm = 0; mm < nf; ++mm) {
            const int qq = base + i * RS + stage_col<N, V>(i, mm);
            const R d = s_dz[j * nf + mm];
            const V2 bm = s_b[qq], qm = s_q[qq], wm = s_w[qq];
            const R sA = Ae + bm.x, sC = Ce + bm.y;
            const R df = d * ((hu + qm.x) * sA + (hv + qm.y) * sC);
            const R dh = d * s_h[qq];
            A1 += df;
            A2 += df * wm.x;
            A3 += df * wm.y;
            C2 += dh * sA;
            C3 += dh * sC;
        }
    }
    {
    // the lane's place in the tile once more (see fresh): kept across the
    // volume sums, the indices spilled at N = 4 and 6
    const int t = kFreshLanes<N, R> ? fresh(threadIdx.x) : (int)threadIdx.x;
    const int el = lane ? t / np : E - 1, p = lane ? t - el * np : 0, i = p / nf, j = p - i * nf;
    const int st = lane ? el * PS + i * RS + stage_col<N, V>(i, j) : E * PS + (t - E * np);
    const int64_t e = e0 + el;
    const uint32_t tq = act ? (uint32_t)t : 0u;
    const R h2g = R(2) * P.g * h;
    // (the jump form's mass sum enters the momentum sums twice: 2u dF1)
    const R uA = kJumpForm<R> ? R(2) * u : u, vA = kJumpForm<R> ? R(2) * v : v;
    R L1 = R(0.5) * A1, L2 = R(0.25) * (uA * A1 + A2 + h2g * C2), L3 = R(0.25) * (vA * A1 + A3 + h2g * C3);
    lds_sync<T>();   // face slots complete; staging region free from here on
    {
        const int fb = el * 4 * nf;
        // (a node lies on at most one side of each direction)
        if (j == 0 || j == N) {
            const int f = fb + (j == 0 ? 0 : 2) * nf + i;
            L1 += s_fl[0][f]; L2 += s_fl[1][f]; L3 += s_fl[2][f];
        }
        if (i == 0 || i == N) {
            const int f = fb + (i == 0 ? 3 : 1) * nf + j;
            L1 += s_fl[0][f]; L2 += s_fl[1][f]; L3 += s_fl[2][f];
        }
    }
    if constexpr (kMetricRel<R>) {
        // the own terms absolute from here on
        const R *const mr = s_mref + 4 * el;
        Ax += mr[0]; Cx += mr[1]; Ae += mr[2]; Ce += mr[3];
    }
    const R J = Ce * Ax - Cx * Ae;

    // ---- R = (1/J)(-L + S + L^v), S = -(g/2) h (b_x, b_y) ----
    // (the arguments afresh from here on, see kernarg: held from the entry, they
    // spilled 24-44 scalar registers; read so from the entry, their latency
    // cost a 128^2 mesh at N = 7 3%)
    const StageArgs<R> &late = kernarg<StageArgs<R>>();
    const Phys<R> &PL = late.P;
    const R bxv = (late.m.bx + q0)[tq], byv = (late.m.by + q0)[tq];
    // ---- viscous divergence of the elements with viscosity (eq.
    // ViscTermsDisc, interface fluxes {F^v}): from the staged velocities, the
    // contravariant fluxes staged in place of the metric directions.  An
    // element without viscosity has no viscous flux of its own; the
    // neighbours' halves came with the face slots ----
    R Lv2 = 0, Lv3 = 0;
    // (the update's operands too are read ahead of the branch, behind which
    // their latency would be paid once more)
    R w0 = 0, w1 = 0, w2 = 0;   // LSRK: the register dU; SSP: W^n
    if constexpr (MODE == kModeLsrk) {
        // the first stage has a_1 = 0: the register is not read
        if (late.ca != R(0)) { w0 = (late.dh + q0)[tq]; w1 = (late.dhu + q0)[tq]; w2 = (late.dhv + q0)[tq]; }
    } else if constexpr (MODE == kModeSsp) {
        w0 = (late.h0 + q0)[tq]; w1 = (late.hu0 + q0)[tq]; w2 = (late.hv0 + q0)[tq];
    }
    if (av && __builtin_expect(block_any_lds<T>(visc, s_any[2], t), 0)) {
        const int base = el * PS;
        V2 fa = V2{R(0), R(0)}, fb = fa;
        if (visc) {
            const R eps_e = (late.eps + e0)[el];
            // (the jumps' loads, two behind each other, go out ahead of the sums)
            const R sx = i == N ? late.tab.iw0 : -late.tab.iw0, se = j == N ? late.tab.iw0 : -late.tab.iw0;
            R jxu = 0, jxv = 0, jeu = 0, jev = 0;
            if (i == 0 || i == N) side_jump<N>(late, e, i == N ? 1 : 3, j, u, v, jxu, jxv);
            if (j == 0 || j == N) side_jump<N>(late, e, j == N ? 2 : 0, i, u, v, jeu, jev);
            R dxu, dxv, deu, dev;
            line_derivatives<N, R>(s_dz, i, j, [&](int r, int c) { return s_w[base + r * RS + stage_col<N, V>(r, c)]; },
                                   V2{u, v}, dxu, dxv, deu, dev);
            dxu += sx * jxu;
            dxv += sx * jxv;
            deu += se * jeu;
            dev += se * jev;
            // contravariant fluxes J grad(xi) . (h eps grad), J grad(eta) . (...)
            const R sc = h * eps_e / J;
            const R aa = sc * (Ax * Ax + Cx * Cx), ae = sc * (Ax * Ae + Cx * Ce), ee = sc * (Ae * Ae + Ce * Ce);
            fa = V2{aa * dxu + ae * deu, aa * dxv + ae * dev};
            fb = V2{ae * dxu + ee * deu, ae * dxv + ee * dev};
        }
        s_a[st] = fa;
        s_b[st] = fb;
        lds_sync<T>();
        if (visc) {
            R ax, ay, bx, by;
            R x1, x2, y1, y2;
            line_derivatives<N, R>(s_dz, i, j, [&](int r, int c) { return s_a[base + r * RS + stage_col<N, V>(r, c)]; },
                                   fa, ax, ay, x1, x2);
            line_derivatives<N, R>(s_dz, i, j, [&](int r, int c) { return s_b[base + r * RS + stage_col<N, V>(r, c)]; },
                                   fb, y1, y2, bx, by);
            Lv2 = ax + bx;
            Lv3 = ay + by;
            // the own half at the faces, -(1/(2 w_0)) n . Fv (none at a wall)
            const R hw = R(0.5) * late.tab.iw0;
            auto face = [&](int s, V2 f, R sg) {
                if (is_wall(late.m, e, s)) return;
                Lv2 -= sg * f.x;
                Lv3 -= sg * f.y;
            };
            if (j == 0) face(0, fb, -hw);
            if (i == N) face(1, fa, hw);
            if (j == N) face(2, fb, hw);
            if (i == 0) face(3, fa, -hw);
        }
        lds_sync<T>();
    }
    const R iJ = act ? rcp_nr(J) : R(0);
    const R hg = R(0.5) * PL.g * h;
    const R R1 = -L1 * iJ;
    const R R2 = (-L2 - hg * bxv + Lv2) * iJ;
    const R R3 = (-L3 - hg * byv + Lv3) * iJ;

    if constexpr (MODE == kModeRhs) {
        if (act) {
            // in the caller's element order where perm gives it
            const int64_t o = late.perm ? (int64_t)late.perm[e] * np + p : q0 + tq;
            late.oh[o] = R1; late.ohu[o] = R2; late.ohv[o] = R3;
        }
        return;
    } else {
        const R dt = (R)late.dt[late.inst ? 8 * (int64_t)late.inst[act ? e : e0] : 0];
        R nh, nhu, nhv;
        R d0 = 0, d1 = 0, d2 = 0;
        if constexpr (MODE == kModeLsrk) {
            d0 = late.ca * w0 + dt * R1;
            d1 = late.ca * w1 + dt * R2;
            d2 = late.ca * w2 + dt * R3;
            nh = h + late.cb * d0; nhu = hu + late.cb * d1; nhv = hv + late.cb * d2;
        } else {
            nh = late.ca * w0 + late.cb * (h + dt * R1);
            nhu = late.ca * w1 + late.cb * (hu + dt * R2);
            nhv = late.ca * w2 + late.cb * (hv + dt * R3);
        }
        // positivity limiter (eq. PosPres) toward the J-weighted means; an
        // element without a negative node keeps theta = 1, so the means are
        // only formed when some element of the workgroup has one
        if (PL.limiter_on && __builtin_expect(block_any_lds<T>(act && nh < R(0), s_any[0], t), 0)) {
            const R wq = act ? J * late.tg->w[i] * late.tg->w[j] : R(0);
            R vals[5] = {wq, wq * nh, wq * nhu, wq * nhv, act ? nh : R(3.0e38)};
            elem_totals_any<N, R, 5, true, T>(vals, s_st, t, el, p, lane);
            if (lane && p == 0) {
                const R area = vals[0];
                const R mh = vals[1] / area, mhu = vals[2] / area, mhv = vals[3] / area, mn = vals[4];
                R th = R(1);
                if (act && mn < R(0)) {
                    if (mh < R(0)) {
                        th = R(0);
                        atomicOr(&late.flags[kFlagNegMean], 1);
                        atomicOr(&late.iflags[late.inst ? late.inst[e] : 0], 1);
                    } else {
                        th = mh / (mh - mn);
                        th = th < R(1) ? th : R(1);
                    }
                    atomicAdd(&late.flags[kFlagLimited], 1);
                }
                s_lim[4 * el + 0] = th; s_lim[4 * el + 1] = mh;
                s_lim[4 * el + 2] = mhu; s_lim[4 * el + 3] = mhv;
            }
            lds_sync<T>();
            const R th = s_lim[4 * el];
            if (act && th != R(1)) {
                const R mh = s_lim[4 * el + 1], mhu = s_lim[4 * el + 2], mhv = s_lim[4 * el + 3];
                nh = th * (nh - mh) + mh;
                nhu = th * (nhu - mhu) + mhu;
                nhv = th * (nhv - mhv) + mhv;
            }
        }
        if (PL.limiter_on && nh < PL.h_tol) { nhu = R(0); nhv = R(0); }
        // a non-finite value in any of the three (an infinity or NaN makes
        // their sum non-finite) is reported once per esdg_step
        if (act && !__builtin_isfinite(nh + nhu + nhv)) atomicOr(&late.flags[kFlagNonFinite], 1);
        if (act) {
            (late.oh + q0)[tq] = nh; (late.ohu + q0)[tq] = nhu; (late.ohv + q0)[tq] = nhv;
            if constexpr (MODE == kModeLsrk) {
                if (late.store_du) { (late.dh + q0)[tq] = d0; (late.dhu + q0)[tq] = d1; (late.dhv + q0)[tq] = d2; }
            }
        }
        R en = R(0);
        if (av) {
            // viscosity of the new state for the next stage (appendix A)
            s_st[8 * T + t] = nh;
            lds_sync<T>();
            if (__builtin_expect(block_any_lds<T>(rough_line<N, R, E>(s_st + 8 * T, t, late.tab, PL), s_any[1], t), 0)) {
                static_assert(2 * T >= nf * nf, "V^{-1} between the reduction scratch and the heights");
                R *const s_vinv = s_st + 6 * T;
                if (t < nf * nf) s_vinv[t] = late.tg->Vinv[t];
                lds_sync<T>();
                en = element_viscosity<N, R, T>(s_st + 8 * T, s_st, s_vinv, PL, t, el, p, lane, nh);
            }
            if (act && p == 0) late.eps_out[e] = en;
            // the viscous face fluxes' own part for the next stage
            if (__builtin_expect(block_any_lds<T>(act && p == 0 && en > R(0), s_any[3], t), 0)) {
                V2 *const s_nw = (V2 *)s_st;   // velocities of the new state
                const R ihn = rcp_wet(nh, PL.h_tol);
                const V2 nw = V2{nhu * ihn, nhv * ihn};
                lds_sync<T>();
                if (lane && p == 0) s_lim[el] = en;
                s_nw[t] = nw;
                lds_sync<T>();
                const R ev = s_lim[el];
                if (act && ev > R(0) && (i == 0 || i == N || j == 0 || j == N))
                    face_parts<N, R>(late.vfl_out, s_dz, e, i, j,
                                     [&](int r, int c) { return s_nw[el * np + r * nf + c]; }, nw, nh * ev, Ax, Cx,
                                     Ae, Ce);
                lds_sync<T>();
            }
        }
        if (late.dtc_out) {
            // face records of the new state for the Lemma 2 bounds of the
            // next step: per face node the height and both velocities, the
            // values the time-step pass would read from the state (corner
            // nodes write both sides)
            if (late.frec_out && act) {
                const R ihn = rcp_wet(nh, PL.h_tol);
                const R un = nhu * ihn, vn = nhv * ihn;
                auto rec = [&](int s, int k) {
                    R *const r = late.frec_out + ((e * 4 + s) * nf + k) * 3;
                    r[0] = nh;
                    r[1] = un;
                    r[2] = vn;
                };
                if (j == 0) rec(0, i);
                if (i == N) rec(1, j);
                if (j == N) rec(2, i);
                if (i == 0) rec(3, j);
            }
            // CFL and viscous bounds of the new state for the next step
            R vals[1] = {act ? cfl_bound<N, R>(nh, nhu, nhv, Ax, Cx, Ae, Ce, J, PL) : R(3.0e38)};
            lds_sync<T>();   // scratch free
            elem_totals_any<N, R, 1, true, T>(vals, s_st, t, el, p, lane);
            if (act && p == 0) {
                late.dtc_out[e] = vals[0];
                if (late.dtv_out) late.dtv_out[e] = en > R(0) ? visc_bound<R>(en, late.gmax[e], PL) : R(3.0e38);
            }
        }
    }
    }
}

// ------------------------------------------------------------------------
// Standalone limiter (initial data / esdg_limit)
// ------------------------------------------------------------------------
template <int N, typename R>
__global__ __launch_bounds__(Shape<N>::T) void limit_kernel(Mesh<R> m, Phys<R> P, Uni<R> tab, R *h_,
                                                            R *hu_, R *hv_, int *flags, int64_t ntiles)
{
    using S = Shape<N>;
    constexpr int nf = S::nf, np = S::np, E = S::E, T = S::T;
    __shared__ R s_red[5 * T];
    const int64_t tile = xcd_tile(ntiles);
    if (tile < 0) return;
    const int t = threadIdx.x;
    const bool lane = t < E * np;
    const int el = lane ? t / np : E - 1, p = lane ? t - el * np : 0, i = p / nf, j = p - i * nf;
    const int64_t e = tile * E + el;
    const bool act = lane && (e < m.K);
    const int64_t q = e * np + p;
    R nh = 0, nhu = 0, nhv = 0, J = 0;
    if (act) {
        nh = h_[q]; nhu = hu_[q]; nhv = hv_[q];
        R Ax, Cx, Ae, Ce;
        metric_at(m, q, e, Ax, Cx, Ae, Ce);
        J = Ce * Ax - Cx * Ae;
    }
    const R wq = act ? J * tab.w[i] * tab.w[j] : R(0);
    R vals[5] = {wq, wq * nh, wq * nhu, wq * nhv, act ? nh : R(3.0e38)};
    ElemReduce<N, R, 5>::template run<true>(vals, s_red, t, el, p);
    const R area = vals[0];
    const R mh = vals[1] / area, mhu = vals[2] / area, mhv = vals[3] / area, mn = vals[4];
    if (!act) return;
    if (mn < R(0)) {
        R th;
        if (mh < R(0)) {
            th = R(0);
            if (p == 0) atomicOr(&flags[kFlagNegMean], 1);
        } else {
            th = mh / (mh - mn);
            th = th < R(1) ? th : R(1);
        }
        if (p == 0) atomicAdd(&flags[kFlagLimited], 1);
        nh = th * (nh - mh) + mh;
        nhu = th * (nhu - mhu) + mhu;
        nhv = th * (nhv - mhv) + mhv;
    }
    if (nh < P.h_tol) { nhu = R(0); nhv = R(0); }
    h_[q] = nh; hu_[q] = nhu; hv_[q] = nhv;
}

// ------------------------------------------------------------------------
// Time step bounds: CFL, viscous (AV), Lemma 2.  Minima go to 64 slots per
// bound by atomicMin on the bit patterns of non-negative doubles (which order
// like unsigned integers); the workgroup that adds the last minima of an
// instance reduces and resets its slots and sets its step (dt_finish), so
// that a step's bounds are one launch.
//
// The last stage of every step leaves the per-element CFL and viscous bounds
// of its output state in dtc/dtv (stage epilogue); the time-step pass then
// only reduces those and evaluates Lemma 2 at the face nodes.  For a state
// no stage produced (initial data, after a limiter call or a retry) the pass
// evaluates every bound itself.  All loops are flat over nodes, face nodes
// and elements, with a fixed grid: each XCD takes one contiguous range of
// each index space so that neighbour traces hit its L2.  Each workgroup
// issues one atomic per bound and one or two tickets.
// ------------------------------------------------------------------------
constexpr int kDtThreads = 256;
constexpr unsigned kDtMaxBlocks = 2048;
constexpr int kDtUnroll = 4;        // face nodes a thread evaluates at once
constexpr int64_t kDtOne = 4;       // rounds that one workgroup takes alone before more share them
// Ticket counters of an instance: each workgroup counts in one of the first
// kDtTickets, the last of each in the one behind them (a single counter would
// serialise up to 2048 atomics on one address), every counter in a cache line
// of its own: atomics on one line are taken one after the other wherever they
// point, and with all counters in two lines the bounds of a new state at 128^2,
// N = 5 without viscosity and limiter took 42.4 us a call (now 35.7).
constexpr int kDtTickets = 32;
constexpr int kDtTicketStride = 128 / sizeof(unsigned);

// One chunk of the ensemble time-step pass: elements [lo, hi) of instance
// inst, its index among that instance's n chunks.
struct DtChunk {
    int64_t lo, hi;
    int32_t inst, index, n, pad;
};

// What the host reads of a step, its statistics or the diagnostics (pinned host
// memory that the GPU writes).
struct alignas(128) HostStatus {
    int flags[kNumFlags];
    double time;
    double sums[8];
    int64_t viscous;
};

// Report the flags and the time and clear the flags (all but that of the mesh).
__device__ inline void report_status(HostStatus *host, int *flags, const double *time)
{
    for (int f = 0; f < kNumFlags; ++f) {
        host->flags[f] = __hip_atomic_load(&flags[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (f != kFlagBadJ) flags[f] = 0;
    }
    host->time = *time;
}

// A step exceeds the bounds of the state it produced when it is above this
// many times the smaller of the CFL and viscous ones (the factors cfl and
// cfl_visc are inside the bounds).
constexpr double kStepBoundFactor = 2.0;

// What the pass does with the minima: set each instance's step (and add it to
// its time when advance), or check the step that produced the state against
// them (a-posteriori check, reading of the remark that the step is adjusted
// when a smaller one is found to be needed, section 6): raise kFlagStepBound
// and bit 2 of the instance's flag, and leave the step as it is.
enum DtMode { kDtSet = 0, kDtAdvance = 1, kDtCheck = 2 };

template <typename R>
struct DtArgs {
    Mesh<R> m;
    Phys<R> P;
    const R *h, *hu, *hv;
    const R *eps;              // full pass with AV: element viscosity of the state
    const R *dtc, *dtv;        // per-element CFL / viscous bounds from the stage epilogue (nullptr: full pass)
    const R *gmax;             // [K] max over the element's nodes of |grad xi|^2 + |grad eta|^2
    const R *fgeo;             // [K][4][nf][3] outward unit normal and w_0 J / J^surf per face node
    const R *frec;             // with dtc: [K][4][nf][3] face records (h, u, v) of the state
    unsigned long long *slots; // [instance][3][kDtSlots]
    const DtChunk *chunk;      // ensembles: [nchunks] element chunks, none across instances
    int64_t nchunks;
    unsigned *tickets;         // [instance][kDtTickets + 1][kDtTicketStride], zero between launches
    double *dt;                // per instance k: dt[8k..8k+3] step and its bounds, dt[8k+4] time
    int mode;                  // DtMode
    int *flags, *iflags;
    HostStatus *host;          // check: the flags go here (nullptr: they stay)
};

__device__ __forceinline__ void slot_min(unsigned long long *slot, double v)
{
    if (v >= 0.0 && v < __builtin_huge_val()) {
        // (the old value is waited for: the minimum has then reached the
        // device's point of coherence, see dt_finish)
        const unsigned long long old = atomicMin(slot, (unsigned long long)__double_as_longlong(v));
        asm volatile("" ::"v"(old));
    }
}

template <typename R>
__device__ __forceinline__ R wave_min(R v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const R o = __shfl_xor(v, off, 64);
        v = o < v ? o : v;
    }
    return v;
}

// Per-element max of |grad xi|^2 + |grad eta|^2 (mesh constant; used by the
// viscous bound).  One thread per element.
template <int N, typename R>
__global__ void gmax_kernel(Mesh<R> m, R *gmax)
{
    constexpr int np = (N + 1) * (N + 1);
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m.K) return;
    R gm = R(0);
    for (int p = 0; p < np; ++p) {
        const int64_t q = e * np + p;
        R Ax, Cx, Ae, Ce;
        metric_at(m, q, e, Ax, Cx, Ae, Ce);
        const R J = Ce * Ax - Cx * Ae;
        const R gg = (Ax * Ax + Cx * Cx + Ae * Ae + Ce * Ce) / (J * J);
        gm = gg > gm ? gg : gm;
    }
    gmax[e] = gm;
}

// Face geometry for Lemma 2 (mesh constant): per face node the outward unit
// normal and w_0 J / J^surf.  One thread per face node.
template <int N, typename R>
__global__ void face_geometry_kernel(Mesh<R> m, R w0, R *fgeo)
{
    constexpr int nf = N + 1, np = nf * nf;
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= m.K * 4 * nf) return;
    const int64_t e = f / (4 * nf);
    const int r = (int)(f - e * 4 * nf), s = r / nf, k = r - s * nf;
    int i, j;
    side_node<N>(s, k, i, j);
    const int64_t q = e * np + i * nf + j;
    R Ax, Cx, Ae, Ce;
    metric_at(m, q, e, Ax, Cx, Ae, Ce);
    R snx, sny;
    if (s == 1) { snx = Ax; sny = Cx; }
    else if (s == 3) { snx = -Ax; sny = -Cx; }
    else if (s == 2) { snx = Ae; sny = Ce; }
    else { snx = -Ae; sny = -Ce; }
    const R js = sqrt(snx * snx + sny * sny);
    const R J = Ce * Ax - Cx * Ae;
    fgeo[f * 3 + 0] = snx / js;
    fgeo[f * 3 + 1] = sny / js;
    fgeo[f * 3 + 2] = w0 * (J / js);
}

// Index range [b, e) and stride of this workgroup over n items: XCD x of 8
// takes the x-th contiguous eighth.
struct XcdRange {
    int64_t b, e, stride;
    __device__ XcdRange(int64_t n, int T)
    {
        if (gridDim.x == 1) {   // (dt_kernel on a small mesh)
            b = threadIdx.x;
            e = n;
            stride = T;
            return;
        }
        const int64_t per = (n + kXcds - 1) / kXcds;
        const int64_t lo = (int64_t)(blockIdx.x % kXcds) * per;
        const int64_t hi = lo + per < n ? lo + per : n;
        b = lo + (int64_t)(blockIdx.x / kXcds) * T + threadIdx.x;
        e = hi;
        stride = (int64_t)(gridDim.x / kXcds) * T;
    }
};

// The two bounds of eq. CFLConstraints for own trace (hm, utm) and
// neighbour (hp, utp), normal velocities along the outward unit normal.
template <typename R>
__device__ __forceinline__ R lemma2_formula(R hm, R hp, R utm, R utp, R w0a, const Phys<R> &P)
{
    const R cm = sqrt(P.g * (hm > R(0) ? hm : R(0))), cp = sqrt(P.g * (hp > R(0) ? hp : R(0)));
    const R au = R(0.5) * (utm + utp), ac = R(0.5) * (cm + cp);
    const R A = fabs(au + ac) + fabs(au - ac), B = fabs(au + ac) - fabs(au - ac);
    R posb = R(3.0e38);
    const R den1 = A + R(2) * au;
    if (den1 > R(0)) { const R bnd = w0a / den1; posb = bnd < posb ? bnd : posb; }
    const R den2 = ac * B * (utp - utm);
    if (hm > R(0) && den2 < R(0)) { const R bnd = fabs(w0a * P.g * hm / den2); posb = bnd < posb ? bnd : posb; }
    return posb;
}

// Lemma 2 bounds at face node f (own trace '-', neighbour '+').
template <int N, typename R>
__device__ __forceinline__ R lemma2_bound(const DtArgs<R> &a, int64_t f)
{
    constexpr int nf = N + 1, np = nf * nf;
    const Phys<R> &P = a.P;
    const int64_t fe = f / (4 * nf);
    const int rr = (int)(f - fe * 4 * nf), s = rr / nf, k = rr - s * nf;
    int fi, fj, ns, kk;
    int64_t en;
    side_node<N>(s, k, fi, fj);
    const int64_t qo = fe * np + fi * nf + fj;
    const int64_t qn = nbr_node<N>(a.m, fe, s, k, en, ns, kk);
    const R nx = a.fgeo[f * 3 + 0], ny = a.fgeo[f * 3 + 1], w0a = a.fgeo[f * 3 + 2];
    const R hm = a.h[qo], hp = a.h[qn];
    const R im = rcp_wet(hm, P.h_tol), ip = rcp_wet(hp, P.h_tol);
    const R utm = nx * (a.hu[qo] * im) + ny * (a.hv[qo] * im);
    const R utp = is_wall(a.m, fe, s) ? -utm : nx * (a.hu[qn] * ip) + ny * (a.hv[qn] * ip);
    return lemma2_formula<R>(hm, hp, utm, utp, w0a, P);
}

// Lemma 2 bounds at face node f from the face records the last stage left:
// the same heights and velocities lemma2_bound reads from the state, so the
// same bounds bit for bit, without reading whole elements.
template <int N, typename R>
__device__ __forceinline__ R lemma2_bound_rec(const DtArgs<R> &a, int64_t f)
{
    constexpr int nf = N + 1;
    const int64_t fe = f / (4 * nf);
    const int rr = (int)(f - fe * 4 * nf), s = rr / nf, k = rr - s * nf;
    const int64_t en = a.m.nbr[fe * 4 + s];
    const int c = a.m.code[fe * 4 + s];
    const int ns = c & 3, kk = ((c >> 2) & 1) ? N - k : k;
    const R *const rm = a.frec + f * 3, *const rp = a.frec + ((en * 4 + ns) * nf + kk) * 3;
    const R nx = a.fgeo[f * 3 + 0], ny = a.fgeo[f * 3 + 1], w0a = a.fgeo[f * 3 + 2];
    const R hm = rm[0], hp = rp[0];
    const R utm = nx * rm[1] + ny * rm[2];
    const R utp = is_wall(a.m, fe, s) ? -utm : nx * rp[1] + ny * rp[2];
    return lemma2_formula<R>(hm, hp, utm, utp, w0a, a.P);
}

// Minimum of the Lemma 2 bounds over the face nodes b, b + stride, ... < e.
// Each iteration takes U of them at once, with clamped indices and no branch,
// so that the loads of all U (face map, then both traces) are in flight
// together; the minimum does not depend on the order.
template <int N, typename R, bool REC, int U>
__device__ __forceinline__ R lemma2_min(const DtArgs<R> &a, int64_t b, int64_t e, int64_t stride)
{
    R posb = R(3.0e38);
    for (; b < e; b += U * stride) {
        R v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t f = b + u * stride;
            const int64_t fc = f < e ? f : e - 1;
            if constexpr (REC) v[u] = lemma2_bound_rec<N, R>(a, fc);
            else v[u] = lemma2_bound<N, R>(a, fc);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = b + u * stride < e;
            posb = (in && v[u] < posb) ? v[u] : posb;
        }
    }
    return posb;
}

// After a step: from the face records its last stage left (with dtc).
template <int N, typename R, int U>
__device__ __forceinline__ R lemma2_min(const DtArgs<R> &a, int64_t b, int64_t e, int64_t stride)
{
    return a.frec ? lemma2_min<N, R, true, U>(a, b, e, stride) : lemma2_min<N, R, false, U>(a, b, e, stride);
}

// CFL bound at node q from the stored state and metric.
template <int N, typename R>
__device__ __forceinline__ R cfl_node(const DtArgs<R> &a, int64_t q)
{
    R Ax, Cx, Ae, Ce;
    metric_at(a.m, q, q / ((N + 1) * (N + 1)), Ax, Cx, Ae, Ce);
    return cfl_bound<N, R>(a.h[q], a.hu[q], a.hv[q], Ax, Cx, Ae, Ce, Ce * Ax - Cx * Ae, a.P);
}

// Workgroup minima of the three bounds into slots[3][kDtSlots] (slot sl), or,
// with own, to own[3] in LDS (+inf where there is none).
template <typename R>
__device__ __forceinline__ void dt_block_min(R cflb, R viscb, R posb, unsigned long long *slots, int sl,
                                             double *own = nullptr)
{
    constexpr int T = kDtThreads;
    __shared__ R s_w[3][T / 64];
    cflb = wave_min(cflb);
    viscb = wave_min(viscb);
    posb = wave_min(posb);
    const int t = threadIdx.x, wv = t >> 6;
    if ((t & 63) == 0) {
        s_w[0][wv] = cflb;
        s_w[1][wv] = viscb;
        s_w[2][wv] = posb;
    }
    lds_sync<T>();
    if (t < 3) {
        R v = s_w[t][0];
#pragma unroll
        for (int w = 1; w < T / 64; ++w) v = s_w[t][w] < v ? s_w[t][w] : v;
        if (own) own[t] = v >= R(0) && v < R(1.0e38) ? (double)v : __builtin_huge_val();
        else if (v < R(1.0e38)) slot_min(&slots[t * kDtSlots + sl], (double)v);
    }
    lds_sync<T>();
}

// Minimum over the wave of an instance's slots of one bound, which go back to
// +inf.  Loads and stores are atomic (past this XCD's L2).
__device__ __forceinline__ double take_slots(unsigned long long *slots, int lane)
{
    static_assert(kDtSlots == 64, "one slot per lane");
    const unsigned long long v = __hip_atomic_load(&slots[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slots[lane], 0x7FF0000000000000ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return wave_min(__longlong_as_double((long long)v));
}

// What a.mode asks with instance k's minima (one thread).
template <typename R>
__device__ __forceinline__ void dt_conclude(const DtArgs<R> &a, int k, double cfl, double visc, double pos)
{
    double *const dt = a.dt + 8 * (int64_t)k;
    if (a.mode == kDtCheck) {
        if (dt[0] > kStepBoundFactor * fmin(cfl, visc)) {
            atomicOr(&a.flags[kFlagStepBound], 1);
            atomicOr(&a.iflags[k], 2);
        }
        if (a.host) report_status(a.host, a.flags, dt + 4);
        return;
    }
    double step = fmin(cfl, visc);
    if (a.P.limiter_on) step = fmin(step, pos);
    if (!(step > 0.0) || !(step < __builtin_huge_val())) {
        atomicOr(&a.flags[kFlagDtPos], 1);
        step = 0.0;
    }
    dt[0] = step;
    dt[1] = cfl;
    dt[2] = visc;
    dt[3] = pos;
    if (a.mode == kDtAdvance) dt[4] += step;
}

// Called by every workgroup when its minima of instance k are in the slots:
// the last of the n workgroups (or chunks), of which this is number idx, does
// what a.mode asks with the minima.  A ticket a piece and no waiting: every
// workgroup ends whatever the others do.  Slots and tickets are only touched
// by device-scope atomics, and a workgroup draws its ticket when its own
// minima's atomics have returned: whoever draws the last one finds them all.
// (With fences instead, each a write-back of the XCD's L2, the pass took twice
// its time on a large mesh.  As a launch of its own behind the pass this took
// another 4.7 us a step.)
template <typename R>
__device__ __forceinline__ void dt_finish(const DtArgs<R> &a, int k, unsigned idx, unsigned n)
{
    __shared__ int s_last;
    __shared__ double s_min[3];
    const int t = threadIdx.x;
    // (behind dt_block_min's last barrier its three lanes' atomics have returned)
    if (t == 0) {
        unsigned *const tk = a.tickets + (int64_t)k * (kDtTickets + 1) * kDtTicketStride;
        // (few workgroups: one counter)
        const unsigned sub = idx % kDtTickets, in_sub = (n - sub + kDtTickets - 1) / kDtTickets;
        const bool two = n > (unsigned)kDtTickets;
        bool up = !two;
        unsigned *const mine = tk + sub * kDtTicketStride, *const all = tk + kDtTickets * kDtTicketStride;
        if (two && atomicAdd(mine, 1u) == in_sub - 1) {
            atomicExch(mine, 0u);
            up = true;
        }
        int last = 0;
        if (up && atomicAdd(all, 1u) == (two ? (unsigned)kDtTickets : n) - 1) {
            atomicExch(all, 0u);
            last = 1;
        }
        s_last = last;
    }
    __syncthreads();
    if (s_last) {
        unsigned long long *const sl = a.slots + (int64_t)k * 3 * kDtSlots;
        const int w = t >> 6;
        if (w < 3) {
            const double v = take_slots(sl + w * kDtSlots, t & 63);
            if ((t & 63) == 0) s_min[w] = v;
        }
        __syncthreads();
        if (t == 0) {
            dt_conclude<R>(a, k, s_min[0], s_min[1], s_min[2]);
        }
    }
    __syncthreads();   // the next chunk's minima and tickets
}

template <int N, typename R>
__global__ __launch_bounds__(kDtThreads) void dt_kernel(DtArgs<R> a)
{
    constexpr int nf = N + 1, np = nf * nf, T = kDtThreads;
    const int64_t K = a.m.K;
    R cflb = R(3.0e38), viscb = R(3.0e38), posb = R(3.0e38);
    if (a.dtc) {
        // per-element bounds left by the stage epilogue
        for (XcdRange r(K, T); r.b < r.e; r.b += r.stride) {
            const R c = a.dtc[r.b];
            cflb = c < cflb ? c : cflb;
            if (a.dtv) {
                const R v = a.dtv[r.b];
                viscb = v < viscb ? v : viscb;
            }
        }
    } else {
        for (XcdRange r(K * np, T); r.b < r.e; r.b += r.stride) {
            const R c = cfl_node<N, R>(a, r.b);
            cflb = c < cflb ? c : cflb;
        }
        if (a.eps) {
            for (XcdRange r(K, T); r.b < r.e; r.b += r.stride) {
                const R eps = a.eps[r.b];
                if (eps > R(0)) {
                    const R v = visc_bound<R>(eps, a.gmax[r.b], a.P);
                    viscb = v < viscb ? v : viscb;
                }
            }
        }
    }
    if (a.P.limiter_on && a.mode != kDtCheck) {
        const XcdRange r(K * 4 * nf, T);
        posb = lemma2_min<N, R, kDtUnroll>(a, r.b, r.e, r.stride);
    }
    if (gridDim.x == 1) {
        __shared__ double s_own[3];
        dt_block_min<R>(cflb, viscb, posb, nullptr, 0, s_own);
        if (threadIdx.x == 0) dt_conclude<R>(a, 0, s_own[0], s_own[1], s_own[2]);
        return;
    }
    dt_block_min<R>(cflb, viscb, posb, a.slots, blockIdx.x % kDtSlots);
    dt_finish<R>(a, 0, blockIdx.x, gridDim.x);
}

// The same per instance of an ensemble: each workgroup takes whole chunks
// of elements (a chunk lies inside one instance) and adds its minima to that
// instance's slots.
template <int N, typename R>
__global__ __launch_bounds__(kDtThreads) void dt_batch_kernel(DtArgs<R> a)
{
    constexpr int nf = N + 1, np = nf * nf, T = kDtThreads;
    const int t = threadIdx.x;
    for (int64_t c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
        const DtChunk ch = a.chunk[c];
        const int64_t lo = ch.lo, hi = ch.hi;
        R cflb = R(3.0e38), viscb = R(3.0e38), posb = R(3.0e38);
        if (a.dtc) {
            for (int64_t e = lo + t; e < hi; e += T) {
                const R v = a.dtc[e];
                cflb = v < cflb ? v : cflb;
                if (a.dtv) {
                    const R w = a.dtv[e];
                    viscb = w < viscb ? w : viscb;
                }
            }
        } else {
            for (int64_t q = lo * np + t; q < hi * np; q += T) {
                const R v = cfl_node<N, R>(a, q);
                cflb = v < cflb ? v : cflb;
            }
            if (a.eps) {
                for (int64_t e = lo + t; e < hi; e += T) {
                    const R eps = a.eps[e];
                    if (eps > R(0)) {
                        const R v = visc_bound<R>(eps, a.gmax[e], a.P);
                        viscb = v < viscb ? v : viscb;
                    }
                }
            }
        }
        if (a.P.limiter_on && a.mode != kDtCheck)
            posb = lemma2_min<N, R, 1>(a, lo * 4 * nf + t, hi * 4 * nf, T);
        dt_block_min<R>(cflb, viscb, posb, a.slots + (int64_t)ch.inst * 3 * kDtSlots, ch.index % kDtSlots);
        dt_finish<R>(a, ch.inst, (unsigned)ch.index, (unsigned)ch.n);
    }
}

// ------------------------------------------------------------------------
// Diagnostics: per-workgroup partial sums of J w w (h, hu, hv, e, q.R),
// min h, max h, #dry nodes.
// ------------------------------------------------------------------------
template <int N, typename R>
__global__ __launch_bounds__(Shape<N>::T) void diag_kernel(Mesh<R> m, Phys<R> P, Uni<R> tab, const R *h_,
                                                           const R *hu_, const R *hv_, const R *b_,
                                                           const R *r0, const R *r1, const R *r2,
                                                           double *part)
{
    using S = Shape<N>;
    constexpr int nf = S::nf, np = S::np, T = S::T;
    __shared__ double s[8][T];
    const int t = threadIdx.x;
    const int64_t q = (int64_t)blockIdx.x * T + t;
    double v[8] = {0, 0, 0, 0, 0, 1e300, -1e300, 0};
    if (q < m.K * np) {
        const int p = (int)(q % np), i = p / nf, j = p - i * nf;
        R Ax, Cx, Ae, Ce;
        metric_at(m, q, q / np, Ax, Cx, Ae, Ce);
        const double J = (double)Ce * Ax - (double)Cx * Ae;
        const double wq = J * tab.w[i] * tab.w[j];
        const double h = h_[q], hu = hu_[q], hv = hv_[q], b = b_[q];
        const double ih = h > P.h_tol ? 1.0 / h : 0.0;
        const double u = hu * ih, vv = hv * ih, g = P.g;
        v[0] = wq * h;
        v[1] = wq * hu;
        v[2] = wq * hv;
        v[3] = wq * (0.5 * h * (u * u + vv * vv) + 0.5 * g * h * h + g * h * b);
        v[4] = wq * ((g * (h + b) - 0.5 * (u * u + vv * vv)) * r0[q] + u * r1[q] + vv * r2[q]);
        v[5] = h;
        v[6] = h;
        v[7] = h > P.h_tol ? 0.0 : 1.0;
    }
    for (int c = 0; c < 8; ++c) s[c][t] = v[c];
    lds_sync<T>();
    for (int st = T / 2; st > 0; st >>= 1) {
        if (t < st) {
            for (int c = 0; c < 5; ++c) s[c][t] += s[c][t + st];
            s[5][t] = fmin(s[5][t], s[5][t + st]);
            s[6][t] = fmax(s[6][t], s[6][t + st]);
            s[7][t] += s[7][t + st];
        }
        lds_sync<T>();
    }
    if (t < 8) part[blockIdx.x * 8 + t] = s[t][0];
}

}  // namespace esdg
