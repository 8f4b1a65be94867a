// gfx950 kernels of the reverse-mode derivatives of the FP64 tracer step.
//
// The paper has no adjoint; these are the derivatives of the discrete map the
// step kernel computes (eq. rk4_update with the spatial interpolation of
// Sec. 3.4 and the temporal interpolation of eq. temporal_interp), for
// finite-time Lyapunov exponents (dx_T/dx_0) and for gradients of a scalar
// loss with respect to the gridded velocity.  Inside a cell the cell index
// is constant, so d(xi)/dx = n/L; across a cell edge bilinear interpolation
// is only continuous, and its derivative is the one-sided one of the cell
// that holds the point.
//
// One thread carries one particle's adjoint vector(s) backwards through a run
// of steps: for each it recomputes the four stage points from the step's start
// position (read from the segment tape), with the Jacobian of the interpolated
// velocity from the same nodes, then applies the chain rule through the RK4
// combine, the stage states and the interpolation.  Grid gradients are
// scatter-added: by default with FP64 atomics (summation order, hence the
// last bits, depends on scheduling); in the deterministic mode as exact
// fixed-point integers (value = hi 2^-32 + lo 2^-64, each contribution
// rounded once to a multiple of 2^-64), whose sums do not depend on the
// order of the additions.
#include "field_dev.h"

namespace lpt {

struct Loc64 {
    int i, j;          // periodic cell
    double xi, eta;    // in-cell coordinates
};

__device__ __forceinline__ Loc64 locate64(const StepParams &P, double x, double y)
{
    const double sx = x * P.invh, sy = y * P.invh;
    const double fx = floor(sx), fy = floor(sy);
    Loc64 l;
    l.xi = sub_rn(sx, fx);
    l.eta = sub_rn(sy, fy);
    l.i = cell_of_floor(fx, P.n, P.mask);
    l.j = cell_of_floor(fy, P.n, P.mask);
    return l;
}

// Derivatives of the Catmull-Rom and B-spline kernels in s.
__device__ __forceinline__ void dweights_cr(double s, double w[4])
{
    w[0] = -0.5 + s * (2.0 - 1.5 * s);
    w[1] = s * (-5.0 + 4.5 * s);
    w[2] = 0.5 + s * (4.0 - 4.5 * s);
    w[3] = s * (-1.0 + 1.5 * s);
}

__device__ __forceinline__ void dweights_bs(double s, double w[4])
{
    const double r = 1.0 - s;
    w[0] = -0.5 * r * r;
    w[1] = s * (1.5 * s - 2.0);
    w[2] = 0.5 + s * (1.0 - 1.5 * s);
    w[3] = 0.5 * s * s;
}

// Stencil of the point: K x K nodes starting at (i0, j0) (K = 2 bilinear,
// 4 bicubic), with 1D weights and their derivatives per axis.  K is a
// compile-time size, so the arrays stay in registers.
template <int K>
struct Sten64 {
    int i0, j0;
    double wx[K], wy[K], dx[K], dy[K];
};

// Whether the point's stencil is bilinear (the scheme, or the paper's
// bilinear fallback near the grid edge).
__device__ __forceinline__ bool bilinear_at(const StepParams &P, int scheme, const Loc64 &l)
{
    return scheme == kBilinear || edge_cell(P.compat_edge, l.i, l.j, P.n);
}

template <int K>
__device__ __forceinline__ Sten64<K> stencil64(int scheme, const Loc64 &l)
{
    Sten64<K> s;
    if constexpr (K == 2) {
        s.i0 = l.i;
        s.j0 = l.j;
        s.wx[0] = 1.0 - l.xi;
        s.wx[1] = l.xi;
        s.wy[0] = 1.0 - l.eta;
        s.wy[1] = l.eta;
        s.dx[0] = -1.0;
        s.dx[1] = 1.0;
        s.dy[0] = -1.0;
        s.dy[1] = 1.0;
    } else {
        s.i0 = l.i - 1;
        s.j0 = l.j - 1;
        if (scheme == kCatmullRom) {
            weights_cr(l.xi, s.wx);
            weights_cr(l.eta, s.wy);
            dweights_cr(l.xi, s.dx);
            dweights_cr(l.eta, s.dy);
        } else {
            weights_bs(l.xi, s.wx);
            weights_bs(l.eta, s.wy);
            dweights_bs(l.xi, s.dx);
            dweights_bs(l.eta, s.dy);
        }
    }
    return s;
}

// Time-blended interpolated velocity (u, v) at a stencil, in the operations of
// the step kernel (bil64 and cub64), and its spatial Jacobian J = [du/dx,
// du/dy, dv/dx, dv/dy], from one read of its K x K nodes through N (the LDS
// tile or the ghost-bordered records, so the stencil never wraps).
template <int K, typename Nodes>
__device__ __forceinline__ void eval_nodes(const Nodes &N, const StepParams &P,
                                           const Sten64<K> &s, const Loc64 &loc, double wa,
                                           double wb, int smode, double &u, double &v, double J[4])
{
    double ux = 0.0, uy = 0.0, vx = 0.0, vy = 0.0, su = 0.0, sv = 0.0;
    with_smode(smode, [&](auto mode) {
        constexpr int SM = decltype(mode)::value;
        double nu[K][2], nv[K][2];   // K == 2: both rows
#pragma unroll
        for (int b = 0; b < K; ++b) {
            double rux = 0.0, rvx = 0.0, ru = 0.0, rv = 0.0;
            typename Nodes::template Raw<SM> raw[K];
#pragma unroll
            for (int a = 0; a < K; ++a) raw[a] = N.template load<SM>(a, b);
#pragma unroll
            for (int a = 0; a < K; ++a) {
                double mu, mv;
                raw[a].blend(wa, wb, mu, mv);
                rux += s.dx[a] * mu;
                rvx += s.dx[a] * mv;
                ru += s.wx[a] * mu;
                rv += s.wx[a] * mv;
                if constexpr (K == 2) {
                    nu[a][b] = mu;
                    nv[a][b] = mv;
                }
            }
            ux += s.wy[b] * rux;
            vx += s.wy[b] * rvx;
            uy += s.dy[b] * ru;
            vy += s.dy[b] * rv;
            su += s.wy[b] * ru;
            sv += s.wy[b] * rv;
        }
        if constexpr (K == 2) {
            double w00, w10, w01, w11;
            bilinear_weights(loc.xi, loc.eta, w00, w10, w01, w11);
            su = w00 * nu[0][0] + w10 * nu[1][0] + w01 * nu[0][1] + w11 * nu[1][1];
            sv = w00 * nv[0][0] + w10 * nv[1][0] + w01 * nv[0][1] + w11 * nv[1][1];
        }
    });
    u = su;
    v = sv;
    J[0] = ux * P.invh;
    J[1] = uy * P.invh;
    J[2] = vx * P.invh;
    J[3] = vy * P.invh;
}

// The same from the block's LDS tile when the stencil lies inside it, else
// from global memory.
template <int K>
__device__ __forceinline__ void eval_stencil(const Rec64 *__restrict__ rec0, const double2 *tile,
                                             const Tile &T, const StepParams &P,
                                             const Sten64<K> &s, const Loc64 &loc, double wa,
                                             double wb, int smode, double &u, double &v,
                                             double J[4])
{
    int t;
    if (tile_index(T, s.i0, s.j0, K, P.n, P.mask, t))
        eval_nodes<K>(TileNodes64{(LdsPair64)tile + t, T.w, T.w * T.h}, P, s, loc, wa, wb, smode, u, v, J);
    else
        eval_nodes<K>(RecNodes64{rec0 + (__mul24(s.j0, P.pitch) + s.i0), P.pitch}, P, s, loc, wa,
                      wb, smode, u, v, J);
}

// Exact fixed-point form of a contribution c (|c| < 2^31): c ~ hi 2^-32 +
// lo 2^-64 with hi = floor(c 2^32) and 0 <= lo < 2^32 the next 32 bits
// (truncated).  The scaling by 2^32 and the fractional part are exact in
// binary64, so the pair depends on c alone; sums of pairs are integer sums
// (hi in two's complement, lo unsigned), exact and order-independent.
__device__ __forceinline__ void to_fixed(double c, unsigned long long &hi, unsigned long long &lo)
{
    const double f = c * 0x1p32;
    const double h = floor(f);
    hi = (unsigned long long)(long long)h;
    lo = (unsigned long long)((f - h) * 0x1p32);
}

// Additions to LDS and to global memory.  Each is spelt with a pointer of its own
// kind: a generic one would make them flat.
typedef __attribute__((address_space(3))) double *LdsF64;
typedef __attribute__((address_space(3))) unsigned long long *LdsU64;

__device__ __forceinline__ void add_to(LdsF64 p, double c)
{
    (void)__hip_atomic_fetch_add(p, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void add_to(LdsU64 p, unsigned long long c)
{
    (void)__hip_atomic_fetch_add(p, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void add_to(double *p, double c)
{
    typedef __attribute__((address_space(1))) double *G;
    (void)__hip_atomic_fetch_add((G)p, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void add_to(unsigned long long *p, unsigned long long c)
{
    typedef __attribute__((address_space(1))) unsigned long long *G;
    (void)__hip_atomic_fetch_add((G)p, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename Ptr>
__device__ __forceinline__ void add_fixed(Ptr pair, double c)
{
    unsigned long long hi, lo;
    to_fixed(c, hi, lo);
    add_to(pair, hi);
    add_to(pair + 1, lo);
}

// Accumulator of dL/d(grid) for one block.  gU in global memory is laid out
// [slot][u, v][n * n]: doubles, or (DET) pairs of 64-bit fixed-point words.
// The block's box B of nodes in LDS holds
//   - by default, planes of the stencil weights times the adjoint stage
//     vector per RK4 time level (g = 0: the first stage, 1: the two middle
//     stages, which share a time, 2: the last), u then v: the two slots'
//     temporal weights are applied once per node when the box is flushed;
//   - DET: fixed-point pairs of the four (slot, component) planes.
template <bool DET>
struct GridGrad {
    void *gU;
    void *acc;   // LDS planes, used when B.on
    Tile B;
};

// The grid gradient of one stage's stencil, K x K nodes: node weight w times
// the stage's adjoint vector (lx, ly), times the temporal weight of each slot.
template <int K, bool DET>
__device__ __forceinline__ void scatter64(const GridGrad<DET> &G, const StepParams &P,
                                          const Sten64<K> &s, int grp, double wa, double wb,
                                          double lx, double ly)
{
    const int n = P.n;
    const int64_t nn = (int64_t)n * n;
    const int area = G.B.w * G.B.h;
    const double wt[2] = {wa, wb};
#pragma unroll
    for (int b = 0; b < K; ++b) {
        const int j = wrap_cell(s.j0 + b, n, P.mask);
        int ry = j - G.B.y0;
        ry += ry < 0 ? n : 0;
#pragma unroll
        for (int a = 0; a < K; ++a) {
            const int i = wrap_cell(s.i0 + a, n, P.mask);
            int rx = i - G.B.x0;
            rx += rx < 0 ? n : 0;
            const double w = s.wx[a] * s.wy[b];
            const bool local = G.B.on && rx < G.B.w && ry < G.B.h;
            const int k = ry * G.B.w + rx;
            if (local && !DET) {
                const LdsF64 acc = (LdsF64)static_cast<double *>(G.acc);
                add_to(acc + ((2 * grp) * area + k), w * lx);
                add_to(acc + ((2 * grp + 1) * area + k), w * ly);
                continue;
            }
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                const double c = wt[sl] * w;
                if (c == 0.0) continue;
                if constexpr (DET) {
                    if (local) {
                        const LdsU64 q = (LdsU64)static_cast<unsigned long long *>(G.acc) +
                                         2 * ((2 * sl) * area + k);
                        add_fixed(q, c * lx);
                        add_fixed(q + 2 * area, c * ly);
                    } else {
                        unsigned long long *q = static_cast<unsigned long long *>(G.gU) +
                                                2 * ((2 * sl) * nn + (int64_t)j * n + i);
                        add_fixed(q, c * lx);
                        add_fixed(q + 2 * nn, c * ly);
                    }
                } else {
                    double *g = static_cast<double *>(G.gU) + (int64_t)j * n + i;
                    add_to(g + (2 * sl) * nn, c * lx);
                    add_to(g + (2 * sl + 1) * nn, c * ly);
                }
            }
        }
    }
}

// The block's box to gU: one atomic per nonzero entry, the two slots' temporal
// weights applied once per node.
template <bool DET>
__device__ __forceinline__ void flush_box(const GridGrad<DET> &G, const StepParams &P,
                                          const StageWeights &W)
{
    const int n = P.n, area = G.B.w * G.B.h;
    const int64_t nn = (int64_t)n * n;
    for (int k = threadIdx.x; k < area; k += blockDim.x) {
        const int ty = k / G.B.w, tx = k - ty * G.B.w;
        int gx = G.B.x0 + tx, gy = G.B.y0 + ty;
        gx -= gx >= n ? n : 0;
        gy -= gy >= n ? n : 0;
        const int64_t g = (int64_t)gy * n + gx;
        if constexpr (DET) {
            const LdsU64 acc = (LdsU64)static_cast<unsigned long long *>(G.acc);
            unsigned long long *out = static_cast<unsigned long long *>(G.gU);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned long long hi = acc[2 * (q * area + k)];
                const unsigned long long lo = acc[2 * (q * area + k) + 1];
                if (hi | lo) {
                    add_to(out + 2 * (q * nn + g), hi);
                    add_to(out + 2 * (q * nn + g) + 1, lo);
                }
            }
        } else {
            const LdsF64 acc = (LdsF64)static_cast<double *>(G.acc);
            double *out = static_cast<double *>(G.gU);
            // time levels 0, 1, 2 were taken at the weights of stages 0, 1, 3
            const double wa[3] = {W.wa[0], W.wa[1], W.wa[3]};
            const double wb[3] = {W.wb[0], W.wb[1], W.wb[3]};
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int g3 = 0; g3 < 3; ++g3) {
                    const double v = acc[(2 * g3 + c) * area + k];
                    s0 += wa[g3] * v;
                    s1 += wb[g3] * v;
                }
                if (s0 != 0.0) add_to(out + c * nn + g, s0);
                if (s1 != 0.0) add_to(out + (2 + c) * nn + g, s1);
            }
        }
    }
}

__device__ __forceinline__ void add_jt(const double J[4], const double l[2], double out[2])
{
    out[0] = J[0] * l[0] + J[2] * l[1];
    out[1] = J[1] * l[0] + J[3] * l[1];
}

// Positions of R.nsteps steps from `in`: tape[(k + 1) np + p] = wrap(position
// after step k), with the step kernel's tile for each step; store_first: the
// start positions go to tape[p] too.
template <bool CUBIC>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(CUBIC ? 4 : 6)))
void recompute64_kernel(StepParams P, StepRun R, const Rec64 *__restrict__ rec, const double2 *in,
                        double2 *tape, int64_t np, int store_first)
{
    const int lb = blockIdx.x;
    const SpeciesDev &sp = P.sp[species_of(P, lb)];
    const int64_t base = (int64_t)(lb - sp.block_begin) * blockDim.x;
    const int64_t local = base + threadIdx.x;
    const bool active = local < sp.count;
    const int64_t p = sp.offset + local;
    const Rec64 *rec0 = rec + P.pitch + 1;
    Rec64 *lds = reinterpret_cast<Rec64 *>(lpt_dyn_lds);
    const double2 *planes = reinterpret_cast<const double2 *>(lpt_dyn_lds);
    double2 x = active ? in[p] : make_double2(0.0, 0.0);
    if (active && store_first) tape[p] = x;
    const double2 a0 = in[sp.offset + base];
    int ax = cell_of_floor(floor(a0.x * P.invh), P.n, P.mask);
    int ay = cell_of_floor(floor(a0.y * P.invh), P.n, P.mask);
    for (int k = 0; k < R.nsteps; ++k) {
        Tile T = no_tile();
        if (P.tile_cap > 0) {
            T = tile64(P, sp, lds, rec0, x, active, ax, ay, base);
            ax = wrap_cell(T.x0 + T.w / 2, P.n, P.mask);
            ay = wrap_cell(T.y0 + T.h / 2, P.n, P.mask);
        }
        if (!active) continue;
        double ddx, ddy;
        if (!CUBIC || sp.scheme == kBilinear)
            rk4_tracer64<false>(rec0, planes, T, P, R.w[k], sp.scheme, x, ddx, ddy);
        else
            rk4_tracer64<true>(rec0, planes, T, P, R.w[k], sp.scheme, x, ddx, ddy);
        x = make_double2(wrap_pos(x.x + ddx, P.L), wrap_pos(x.y + ddy, P.L));
        tape[(k + 1) * np + p] = x;
    }
}

extern __shared__ __align__(32) unsigned char adj_dyn_lds[];

// Box of the stencils of a block's stage points, for the gradient accumulators:
// it holds every node they touch, unless that is more than `cap` nodes.  Then
// it is cut down about its centre to a window that fits, or, beyond kBoxWaste
// times the capacity, left out (B.on = 0): what falls outside goes to global
// memory.  Windows of a sixteenth of the box still pay (2^22 unsorted lattice
// tracers on 1024^2, 31 KiB: left out beyond twice the capacity 8125 us a reverse
// step, beyond eight times 6428, never 6339); for one that holds hardly a stencil
// the clearing and the flush are lost time (4096 unsorted particles on 1024^2: 20
// us without a box, 22 with).
constexpr int kBoxWaste = 16;

__device__ __forceinline__ Tile gradient_box(BoxAcc b, int ax, int ay, const StepParams &P, int lo,
                                             int hi, int cap)
{
    const int n = P.n;
    Tile B = block_box_reduce(b, ax, ay, n, P.mask, lo, hi);
    B.w = min(B.w, n);
    B.h = min(B.h, n);
    B.on = B.w * B.h <= kBoxWaste * cap;   // at most 2^30 either side
    if (B.on && B.w * B.h > cap) {
        const float f = sqrtf((float)cap / (float)(B.w * B.h));
        const int w = max(1, (int)((float)B.w * f));
        const int h = min(B.h, cap / w);
        B.x0 = wrap_cell(B.x0 + (B.w - w) / 2, n, P.mask);
        B.y0 = wrap_cell(B.y0 + (B.h - h) / 2, n, P.mask);
        B.w = w;
        B.h = h;
    }
    return B;
}

// R.nsteps reverse steps, newest first; tape[k np + p] is the position at the
// start of step k.  lam holds NL adjoint vectors per particle (lam[p * NL +
// r]), which stay in registers in between; gU (GRID) receives the grid
// gradient of the first one.  Each step has its field tile, and, once its
// stages are evaluated, the same LDS takes the block's contributions to the
// grid gradient (gradient_box), which then go to gU with one atomic per nonzero
// entry.  DET: gU holds fixed-point pairs (see to_fixed), and so does the box.
//
// Bound by its atomics and by latency at three waves per SIMD (167 registers with
// the grid gradient, 150-167 without; at four, with 124 bytes a lane spilled, 11%
// slower) or, bicubic with the grid gradient, two (170).  2^22 lattice tracers on
// 2048^2, bilinear: 417 -> 358 us a step with each stage's loads together, ->
// 280 with the exact box (the box of the cells widened by the displacement
// bound held 60% more nodes), the tile beside it and one read of the nodes for
// velocity and Jacobian; 2^18 Catmull-Rom tracers on 1024^2, whose boxes
// outgrew the fixed LDS: 1300 -> 130 us.
template <int NL, bool GRID, bool CUBIC, bool DET>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(CUBIC ? 2 : 3)))
void adjoint64_kernel(StepParams P, StepRun R, const Rec64 *__restrict__ rec,
                      const double2 *__restrict__ tape, int64_t np, double2 *__restrict__ lam,
                      void *gU, int lds_bytes)
{
    const int lb = blockIdx.x;
    const SpeciesDev &sp = P.sp[species_of(P, lb)];
    const int64_t base = (int64_t)(lb - sp.block_begin) * blockDim.x;
    const int64_t local = base + threadIdx.x;
    const bool active = local < sp.count;
    const int64_t p = sp.offset + local;
    const Rec64 *rec0 = rec + P.pitch + 1;
    const int scheme = sp.scheme;
    const double dt = P.dt, hdt = 0.5 * P.dt, dt6 = P.dt / 6.0, dt3 = P.dt / 3.0;
    const double2 *planes = reinterpret_cast<const double2 *>(adj_dyn_lds);
    int lo, hi;
    stencil_reach(scheme, lo, hi);

    double lx[NL][2];
#pragma unroll
    for (int r = 0; r < NL; ++r) {
        const double2 l = active ? lam[p * NL + r] : make_double2(0.0, 0.0);
        lx[r][0] = l.x;
        lx[r][1] = l.y;
    }
    for (int k = R.nsteps - 1; k >= 0; --k) {
        const StageWeights &W = R.w[k];
        const double2 *row = tape + (int64_t)k * np;
        const double2 x = active ? row[p] : make_double2(0.0, 0.0);
        const double2 a0 = row[sp.offset + base];
        const int ax = cell_of_floor(floor(a0.x * P.invh), P.n, P.mask);
        const int ay = cell_of_floor(floor(a0.y * P.invh), P.n, P.mask);
        Tile T = no_tile();
        if (P.tile_cap > 0)
            T = tile64(P, sp, reinterpret_cast<Rec64 *>(adj_dyn_lds), rec0, x, active, ax, ay,
                       base);

        // forward recomputation of the stage points, exactly as the step
        // kernel, with the Jacobian at each
        double px[4], py[4], J[4][4], lk[NL][4][2];
        BoxAcc box = box_init();
        if (active) {
            double ku = 0.0, kv = 0.0;
            const double ahead[4] = {0.0, hdt, hdt, dt};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                px[q] = q == 0 ? x.x : x.x + ahead[q] * ku;
                py[q] = q == 0 ? x.y : x.y + ahead[q] * kv;
                const Loc64 loc = locate64(P, px[q], py[q]);
                if (!CUBIC || bilinear_at(P, scheme, loc))
                    eval_stencil<2>(rec0, planes, T, P, stencil64<2>(scheme, loc), loc, W.wa[q],
                                    W.wb[q], W.smode[q], ku, kv, J[q]);
                else if constexpr (CUBIC)
                    eval_stencil<4>(rec0, planes, T, P, stencil64<4>(scheme, loc), loc, W.wa[q],
                                    W.wb[q], W.smode[q], ku, kv, J[q]);
                if constexpr (GRID) {
                    const BoxAcc c = box_of(loc.i, loc.j, ax, ay, P.n);
                    box = q == 0 ? c : BoxAcc{pmax16(box.up, c.up), pmax16(box.dn, c.dn)};
                }
            }
            // Back through x' = x + dt/6 (k1 + 2 k2 + 2 k3 + k4), k_q = U(x_q),
            // x_q = x + c_q dt k_(q-1) (c = 1/2, 1/2, 1): per adjoint vector r,
            // lx[r] collects dL/dx and lk[r][q] the adjoint of k_q.
#pragma unroll
            for (int r = 0; r < NL; ++r) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    lk[r][0][c] = dt6 * lx[r][c];
                    lk[r][1][c] = dt3 * lx[r][c];
                    lk[r][2][c] = dt3 * lx[r][c];
                    lk[r][3][c] = dt6 * lx[r][c];
                }
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    double ls[2];
                    add_jt(J[q], lk[r][q], ls);
                    lx[r][0] += ls[0];
                    lx[r][1] += ls[1];
                    if (q > 0) {
                        lk[r][q - 1][0] += ahead[q] * ls[0];
                        lk[r][q - 1][1] += ahead[q] * ls[1];
                    }
                }
            }
        }
        if constexpr (GRID) {
            // LDS per box node: three time levels x (u, v) doubles, or (DET)
            // four (slot, component) planes of fixed-point pairs
            constexpr int kNodeBytes = DET ? 64 : 48;
            // every thread has read its tile when the box is known
            GridGrad<DET> G{gU, adj_dyn_lds,
                            gradient_box(box, ax, ay, P, lo, hi, lds_bytes / kNodeBytes)};
            const int area = G.B.w * G.B.h;
            if (G.B.on) {
                const LdsU64 acc = (LdsU64)static_cast<unsigned long long *>(G.acc);
                for (int w = threadIdx.x; w < (kNodeBytes / 8) * area; w += blockDim.x)
                    acc[w] = 0ull;   // 0.0 too
            }
            // the accumulators are clear; and, box or no box, every thread has
            // read the box's reduction before the next one overwrites it
            __syncthreads();
            if (active) {
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    const Loc64 loc = locate64(P, px[q], py[q]);
                    const int grp = q == 0 ? 0 : (q == 3 ? 2 : 1);   // time level of the stage
                    if (!CUBIC || bilinear_at(P, scheme, loc))
                        scatter64<2, DET>(G, P, stencil64<2>(scheme, loc), grp, W.wa[q], W.wb[q],
                                          lk[0][q][0], lk[0][q][1]);
                    else if constexpr (CUBIC)
                        scatter64<4, DET>(G, P, stencil64<4>(scheme, loc), grp, W.wa[q], W.wb[q],
                                          lk[0][q][0], lk[0][q][1]);
                }
            }
            if (G.B.on) {
                __syncthreads();
                flush_box<DET>(G, P, W);
                // the next step's first barrier (in its box) keeps the
                // accumulators until every thread has flushed
            }
        }
    }
    if (active)
#pragma unroll
        for (int r = 0; r < NL; ++r) lam[p * NL + r] = make_double2(lx[r][0], lx[r][1]);
}

// lam[p * NL + r] from the caller's per-id seeds: NL == 1: (gx[id], gy[id]);
// NL == 2: the unit vectors (d x_T, d y_T).
__global__ void seed_adjoint_kernel(const uint32_t *__restrict__ id, int64_t np, int nl,
                                    const double *__restrict__ gx, const double *__restrict__ gy,
                                    double2 *lam)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    if (nl == 1) {
        const uint32_t g = id[p];
        lam[p] = make_double2(gx[g], gy[g]);
    } else {
        lam[2 * p] = make_double2(1.0, 0.0);
        lam[2 * p + 1] = make_double2(0.0, 1.0);
    }
}

// Finite-time Lyapunov exponent of one Jacobian F = [[a, b], [c, d]]:
// (1/T) ln sqrt(lambda_max(F^T F)), with the largest eigenvalue of the
// symmetric Cauchy-Green tensor [[p, r], [r, q]] (p = a^2 + c^2,
// q = b^2 + d^2, r = ab + cd) in closed form,
// lambda_max = (p + q)/2 + sqrt(((p - q)/2)^2 + r^2).
__device__ __forceinline__ double ftle_of(double a, double b, double c, double d, double T)
{
    const double p = a * a + c * c, q = b * b + d * d, r = a * b + c * d;
    const double h = 0.5 * (p - q);
    const double lam = 0.5 * (p + q) + sqrt(h * h + r * r);
    return 0.5 * log(lam) / T;
}

// Results back in original (id) order: NL == 1: gx0, gy0; NL == 2: the
// Jacobian F[id] = [[dx/dx0, dx/dy0], [dy/dx0, dy/dy0]] and/or its FTLE over
// the time T (any output may be null).
__global__ void gather_adjoint_kernel(const uint32_t *__restrict__ id, int64_t np, int nl,
                                      const double2 *__restrict__ lam, double *gx, double *gy,
                                      double *F, double *sigma, double T)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const uint32_t g = id[p];
    if (nl == 1) {
        const double2 l = lam[p];
        if (gx) gx[g] = l.x;
        if (gy) gy[g] = l.y;
    } else {
        const double2 r0 = lam[2 * p], r1 = lam[2 * p + 1];
        if (F) {
            F[4 * (int64_t)g + 0] = r0.x;
            F[4 * (int64_t)g + 1] = r0.y;
            F[4 * (int64_t)g + 2] = r1.x;
            F[4 * (int64_t)g + 3] = r1.y;
        }
        if (sigma) sigma[g] = ftle_of(r0.x, r0.y, r1.x, r1.y, T);
    }
}

hipError_t launch_recompute64(const StepParams &P, const StepRun &R, const Rec64 *rec,
                              const double2 *in, double2 *tape, int64_t np, bool store_first,
                              bool cubic, int block, hipStream_t st)
{
    // the step kernel's tile: two planes of 16-byte entries, whole 64-entry chunks
    const size_t lds = P.tile_cap > 0 ? (size_t)(2 * P.tile_cap + kWave) * 16 : 0;
    if (cubic)
        hipLaunchKernelGGL(recompute64_kernel<true>, dim3(P.total_blocks), dim3(block), lds, st, P,
                           R, rec, in, tape, np, (int)store_first);
    else
        hipLaunchKernelGGL(recompute64_kernel<false>, dim3(P.total_blocks), dim3(block), lds, st,
                           P, R, rec, in, tape, np, (int)store_first);
    return hipGetLastError();
}

// LDS of the adjoint kernel: 31 KiB, so that five 256-thread blocks fit in a
// CU's 160 KiB: 960 nodes of field tile, then 661 nodes of gradient box (496 of
// fixed-point pairs).  Where the particles of a block are spread over more cells
// than that, the box takes what it needs, down to one block per CU.  Unsorted
// particles spread over an unknown number: bound by the atomics that miss the box,
// their blocks take the whole CU (2^22 lattice tracers on 2048^2 at 0.3 cells a
// step: 31 KiB 2291 us a reverse step, 79 KiB 1347, 159 KiB 1019), except
// one-wave blocks, which go four to a CU (2^14 lattice tracers on 64^2: 31 KiB
// 25 us, 39 KiB 22; 4096 on 64^2: 39 KiB 20, 159 KiB 36).
constexpr int kAdjLdsBytes = 31 * 1024;

static int gradient_lds(const StepParams &P, int block, bool cubic, bool sorted, bool det)
{
    if (!sorted) return (block == kWave ? 39 : 159) * 1024;
    double cells = 0.0;                 // of a block, at its species' density
    for (int s = 0; s < P.nspecies; ++s)
        cells = fmax(cells, (double)block * P.n * P.n / (double)P.sp[s].count);
    const double side = sqrt(cells) + (cubic ? 8.0 : 6.0);
    const double need = side * side * (det ? 64.0 : 48.0);
    for (int per_cu = 5; per_cu >= 1; --per_cu) {
        const int lds = (160 / per_cu - 1) * 1024;
        if (need <= lds) return lds < kAdjLdsBytes ? kAdjLdsBytes : lds;
    }
    return kAdjLdsBytes;
}

template <int NL, bool GRID, bool CUBIC, bool DET>
static hipError_t launch_adjoint64_t(const StepParams &P, const StepRun &R, const Rec64 *rec,
                                     const double2 *tape, int64_t np, double2 *lam, void *gU,
                                     int block, bool sorted, hipStream_t st)
{
    const int lds = GRID ? gradient_lds(P, block, CUBIC, sorted, DET) : kAdjLdsBytes;
    StepParams Q = P;
    // the tile's last fill chunk may run one chunk over
    const int cap = (lds / 16 - kWave) / 2;
    if (Q.tile_cap > cap) Q.tile_cap = cap;
    hipLaunchKernelGGL((adjoint64_kernel<NL, GRID, CUBIC, DET>), dim3(P.total_blocks), dim3(block),
                       GRID || P.tile_cap > 0 ? lds : 0, st, Q, R, rec, tape, np, lam, gU, lds);
    return hipGetLastError();
}

template <bool CUBIC>
static hipError_t launch_adjoint64_c(const StepParams &P, const StepRun &R, const Rec64 *rec,
                                     const double2 *tape, int64_t np, double2 *lam, int nl,
                                     void *gU, bool det, int block, bool sorted, hipStream_t st)
{
    if (nl != 1)
        return launch_adjoint64_t<2, false, CUBIC, false>(P, R, rec, tape, np, lam, nullptr, block,
                                                          sorted, st);
    if (!gU)
        return launch_adjoint64_t<1, false, CUBIC, false>(P, R, rec, tape, np, lam, nullptr, block,
                                                          sorted, st);
    return det ? launch_adjoint64_t<1, true, CUBIC, true>(P, R, rec, tape, np, lam, gU, block,
                                                          sorted, st)
               : launch_adjoint64_t<1, true, CUBIC, false>(P, R, rec, tape, np, lam, gU, block,
                                                           sorted, st);
}

hipError_t launch_adjoint64(const StepParams &P, const StepRun &R, const Rec64 *rec,
                            const double2 *tape, int64_t np, double2 *lam, int nl, void *gU,
                            bool det, bool cubic, int block, bool sorted, hipStream_t st)
{
    return cubic ? launch_adjoint64_c<true>(P, R, rec, tape, np, lam, nl, gU, det, block, sorted,
                                            st)
                 : launch_adjoint64_c<false>(P, R, rec, tape, np, lam, nl, gU, det, block, sorted,
                                             st);
}

// Fixed-point pairs (hi 2^-32 + lo 2^-64) to binary64, in place order.
__global__ void fixed_to_double_kernel(const unsigned long long *__restrict__ pairs, int64_t count,
                                       double *out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const long long hi = (long long)pairs[2 * k];
    const unsigned long long lo = pairs[2 * k + 1];
    out[k] = (double)hi * 0x1p-32 + (double)lo * 0x1p-64;
}

hipError_t launch_fixed_to_double(const void *pairs, int64_t count, double *out, hipStream_t st)
{
    const int b = 256;
    hipLaunchKernelGGL(fixed_to_double_kernel, dim3((unsigned)((count + b - 1) / b)), dim3(b), 0,
                       st, static_cast<const unsigned long long *>(pairs), count, out);
    return hipGetLastError();
}

__global__ void zero_words_kernel(unsigned long long *p, int64_t count)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < count) p[k] = 0ull;
}

hipError_t launch_zero_words(void *p, int64_t words, hipStream_t st)
{
    const int b = 256;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((words + b - 1) / b)), dim3(b), 0, st,
                       static_cast<unsigned long long *>(p), words);
    return hipGetLastError();
}

// Adjoint vectors from one segment's slot order to the previous segment's:
// the sort at the segment's start filled slot i from slot perm[i], so
// out[perm[i]] = in[i] (NL vectors per slot).
__global__ void unpermute_adjoint_kernel(const uint32_t *__restrict__ perm, int64_t np, int nl,
                                         const double2 *__restrict__ in, double2 *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    const int64_t j = perm[i];
    for (int r = 0; r < nl; ++r) out[j * nl + r] = in[i * nl + r];
}

hipError_t launch_unpermute_adjoint(const uint32_t *perm, int64_t np, int nl, const double2 *in,
                                    double2 *out, hipStream_t st)
{
    const int b = 256;
    hipLaunchKernelGGL(unpermute_adjoint_kernel, dim3((unsigned)((np + b - 1) / b)), dim3(b), 0,
                       st, perm, np, nl, in, out);
    return hipGetLastError();
}

hipError_t launch_seed_adjoint(const uint32_t *id, int64_t np, int nl, const double *gx,
                               const double *gy, double2 *lam, hipStream_t st)
{
    const int b = 256;
    hipLaunchKernelGGL(seed_adjoint_kernel, dim3((unsigned)((np + b - 1) / b)), dim3(b), 0, st, id,
                       np, nl, gx, gy, lam);
    return hipGetLastError();
}

hipError_t launch_gather_adjoint(const uint32_t *id, int64_t np, int nl, const double2 *lam,
                                 double *gx, double *gy, double *F, double *sigma, double T,
                                 hipStream_t st)
{
    const int b = 256;
    hipLaunchKernelGGL(gather_adjoint_kernel, dim3((unsigned)((np + b - 1) / b)), dim3(b), 0, st,
                       id, np, nl, lam, gx, gy, F, sigma, T);
    return hipGetLastError();
}

}  // namespace lpt
