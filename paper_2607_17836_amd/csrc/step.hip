// gfx950 kernels of the particle step: snapshot packing, RK4 + interpolation
// (FP64 and FP32-split), initial state, velocity probe, readout and the
// statistics finalisation.
//
// One thread advances one particle (two with rows = 2; four lanes one in the
// small-population bicubic kernels) by a launch's RK4 steps, one or a run of
// them (Alg. coupled_EL, particle loop; eqs. rk4_update / rk4_inertial).  Each of
// the four stages gathers the 4 (bilinear) or 16 (bicubic) node records around
// the stage position; a node record carries both retained time levels, so one
// gather serves the temporal interpolation (eq. temporal_interp) too, and a stage
// whose temporal weight is (1, 0) or (0, 1) loads only the half it needs.  Records
// carry a periodic ghost border, so a stencil never wraps: its nodes are fixed
// offsets from one base address.  State is structure-of-arrays with interleaved (x, y) pairs,
// so the per-step state stream is fully coalesced; the gathers rely on
// cell-ordered particles (sort.hip) and an XCD-aware block order for L2 reuse.
#include "field_dev.h"

#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

namespace lpt {

// The device clock after `steps` steps, added as that many launches add them
// (by one thread of the launch: the caller picks the block).
__device__ __forceinline__ void advance_clock(const StepParams &P, int steps, DevClock *clock)
{
    if (threadIdx.x == 0) {
        double t = clock->t;
        for (int k = 0; k < steps; ++k) t += P.dt;
        clock->t = t;
        clock->step += steps;
    }
}

// One logical block of the FP64 run kernel: R.nsteps steps of the block's
// particles, which stay in registers, with a new tile for each.  Slot p of D
// takes the particle of slot p of S (D = S: in place), or, on the steps that
// follow a re-sort, of slot perm[p], id included.  The box of a step is taken
// about the centre of the box before (any cell near the particles will do).
template <bool CUBIC, bool INERTIAL, bool STATS>
__device__ __forceinline__ void run64_block(const StepParams &P, const StepRun &R,
                                            const State64 &S, const State64 &D,
                                            const uint32_t *perm, const Rec64 *__restrict__ rec,
                                            double *__restrict__ partials, DevClock *clock, int lb)
{
    Rec64 *lds = reinterpret_cast<Rec64 *>(lpt_dyn_lds);
    const double2 *planes = reinterpret_cast<const double2 *>(lpt_dyn_lds);   // tile, two planes
    const SpeciesDev &sp = P.sp[species_of(P, lb)];
    const int64_t base = (int64_t)(lb - sp.block_begin) * blockDim.x;
    const int64_t local = base + threadIdx.x;
    const bool active = local < sp.count;
    const int64_t p = sp.offset + local;
    const Rec64 *rec0 = rec + P.pitch + 1;
    const bool inert = INERTIAL && sp.inertial;

    int64_t q = p;
    double2 x = make_double2(0.0, 0.0), d = x, vn = x;
    if (active) {
        if (perm) q = perm[p];
        x = S.pos[q];
        d = S.disp[q];
        if (inert) vn = S.vel[q];
    }
    int ax = 0, ay = 0;
    if (P.tile_cap > 0) {
        const int64_t a0 = sp.offset + base;
        const double2 a = S.pos[perm ? (int64_t)perm[a0] : a0];
        ax = cell_of_floor(floor(a.x * P.invh), P.n, P.mask);
        ay = cell_of_floor(floor(a.y * P.invh), P.n, P.mask);
    }
    for (int k = 0; k < R.nsteps; ++k) {
        const StageWeights &W = R.w[k];
        Tile T = no_tile();
        if (P.tile_cap > 0) {
            T = tile64(P, sp, lds, rec0, x, active, ax, ay, base);
            ax = wrap_cell(T.x0 + T.w / 2, P.n, P.mask);
            ay = wrap_cell(T.y0 + T.h / 2, P.n, P.mask);
        }
        if (active) {
            double ddx, ddy;
            if (inert)
                rk4_inertial64<CUBIC>(rec0, planes, T, P, W, sp.scheme, sp.inv_st, x, vn, ddx, ddy);
            else
                rk4_tracer64<CUBIC>(rec0, planes, T, P, W, sp.scheme, x, ddx, ddy);
            x = make_double2(wrap_pos(x.x + ddx, P.L), wrap_pos(x.y + ddy, P.L));
            d.x += ddx;
            d.y += ddy;
        }
    }
    if (active) {
        // wrapped coordinates for evaluation/output, unwrapped displacement
        // for statistics
        D.pos[p] = x;
        D.disp[p] = d;
        if (inert) D.vel[p] = vn;
        if (perm) D.id[p] = S.id[q];
    }
    if (STATS)
        wave_stats(active ? d.x * d.x : 0.0, active ? d.y * d.y : 0.0, active,
                   partials + (int64_t)kStatTerms *
                                  ((int64_t)lb * (blockDim.x / kWave) + threadIdx.x / kWave));
    if (lb == 0) advance_clock(P, R.nsteps, clock);
}

// One logical block of the FP64 step, in place.
template <bool CUBIC, bool INERTIAL, bool STATS>
__device__ __forceinline__ void step64_block(const StepParams &P, const State64 &S,
                                             const Rec64 *__restrict__ rec,
                                             double *__restrict__ partials, DevClock *clock,
                                             int lb)
{
    Rec64 *lds = reinterpret_cast<Rec64 *>(lpt_dyn_lds);
    const double2 *planes = reinterpret_cast<const double2 *>(lpt_dyn_lds);   // tile, two planes
    const SpeciesDev &sp = P.sp[species_of(P, lb)];
    const int64_t base = (int64_t)(lb - sp.block_begin) * blockDim.x;
    const int64_t local = base + threadIdx.x;
    const bool active = local < sp.count;
    const int64_t p = sp.offset + local;
    const Rec64 *rec0 = rec + P.pitch + 1;
    double r2x = 0.0, r2y = 0.0;

    const double2 x = active ? S.pos[p] : make_double2(0.0, 0.0);
    Tile T = no_tile();
    if (P.tile_cap > 0) {
        const double2 a = S.pos[sp.offset + base];
        T = tile64(P, sp, lds, rec0, x, active, cell_of_floor(floor(a.x * P.invh), P.n, P.mask),
                   cell_of_floor(floor(a.y * P.invh), P.n, P.mask), base);
    }
    if (active) {
        double2 d = S.disp[p];
        double ddx, ddy;
        if (INERTIAL && sp.inertial) {
            double2 vn = S.vel[p];
            rk4_inertial64<CUBIC>(rec0, planes, T, P, P.w, sp.scheme, sp.inv_st, x, vn, ddx, ddy);
            S.vel[p] = vn;
        } else {
            rk4_tracer64<CUBIC>(rec0, planes, T, P, P.w, sp.scheme, x, ddx, ddy);
        }
        S.pos[p] = make_double2(wrap_pos(x.x + ddx, P.L), wrap_pos(x.y + ddy, P.L));
        d.x += ddx;
        d.y += ddy;
        S.disp[p] = d;
        r2x = d.x * d.x;
        r2y = d.y * d.y;
    }
    if (STATS)
        wave_stats(r2x, r2y, active,
                   partials + (int64_t)kStatTerms *
                                  ((int64_t)lb * (blockDim.x / kWave) + threadIdx.x / kWave));
    if (lb == 0) advance_clock(P, 1, clock);
}

// Bound by the latency of the stages' gathers, so by the waves that stay
// resident: registers are bounded to six waves per SIMD for bilinear tracers
// (80 registers, on record steps 24 bytes a lane of scratch; an 800-record tile
// leaves room for six blocks) and to four otherwise (124-128; the bicubic
// inertial bodies spill 16-28 bytes; unbounded 133 and three waves).  With each
// stage's loads in flight together (see NodeRaw64): 1024^2 Catmull-Rom, 2^20 tracers + 2^20
// inertial particles 136 -> 106 us a step; 2048^2, 2^20 bilinear tracers 58.9
// -> 51.4 us; 4096^2, 2^24 bilinear tracers 421 -> 394 us with the shipped
// 800-record tile, 479 -> 447 us with the default.
template <bool CUBIC, bool INERTIAL, bool STATS>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(CUBIC || INERTIAL ? 4 : 6)))
void step64_kernel(StepParams P, State64 S, const Rec64 *__restrict__ rec,
                   double *__restrict__ partials, DevClock *clock)
{
    BlockWalk w = block_walk(P, 0, P.total_blocks);
    for (int lb = 0; block_next(w, lb);)
        step64_block<CUBIC, INERTIAL, STATS>(P, S, rec, partials, clock, lb);
}

// Runs of steps in one launch, and the step that follows a re-sort, in the same
// bounds (bilinear tracers 79 registers and 20-36 bytes a lane of scratch, the
// others 115-128 and up to 32).
template <bool CUBIC, bool INERTIAL, bool STATS>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(CUBIC || INERTIAL ? 4 : 6)))
void run64_kernel(StepParams P, StepRun R, State64 S, State64 D, const uint32_t *perm,
                  const Rec64 *__restrict__ rec, double *__restrict__ partials, DevClock *clock)
{
    BlockWalk w = block_walk(P, 0, P.total_blocks);
    for (int lb = 0; block_next(w, lb);)
        run64_block<CUBIC, INERTIAL, STATS>(P, R, S, D, perm, rec, partials, clock, lb);
}

// ===========================================================================
// FP32 split path.  Positions are (cell, offset) with the offset in cell
// units; the packed field is in cells per unit time, so every stage works in
// cell units: q = offset + c*dt*k, cell = stored cell + floor(q), in-cell
// coordinate = fract(q).
// ===========================================================================
// wa a + wb b of the two levels (eq. temporal_interp), with the fused product
// spelt out: left to the compiler, which of the two is fused depends on the
// code around it, and a trajectory on the kernel that computes it.
__device__ __forceinline__ float blend32(float wa, float a, float wb, float b)
{
    return fmaf(wa, a, wb * b);
}

template <int SM>
__device__ __forceinline__ float2 half32(const float4 *r)
{
    return reinterpret_cast<const float2 *>(r)[SM];
}

__device__ __forceinline__ void bil32(const float4 *p, int pitch, float xi, float eta, int smode,
                                      float wa, float wb, float &u, float &v)
{
    float w00, w10, w01, w11;
    bilinear_weights(xi, eta, w00, w10, w01, w11);
    if (smode == kSlot0) {
        const float2 a = half32<0>(p), b = half32<0>(p + 1);
        const float2 c = half32<0>(p + pitch), d = half32<0>(p + pitch + 1);
        u = w00 * a.x + w10 * b.x + w01 * c.x + w11 * d.x;
        v = w00 * a.y + w10 * b.y + w01 * c.y + w11 * d.y;
    } else if (smode == kSlot1) {
        const float2 a = half32<1>(p), b = half32<1>(p + 1);
        const float2 c = half32<1>(p + pitch), d = half32<1>(p + pitch + 1);
        u = w00 * a.x + w10 * b.x + w01 * c.x + w11 * d.x;
        v = w00 * a.y + w10 * b.y + w01 * c.y + w11 * d.y;
    } else {
        const float4 a = p[0], b = p[1], c = p[pitch], d = p[pitch + 1];
        const float ua = w00 * a.x + w10 * b.x + w01 * c.x + w11 * d.x;
        const float va = w00 * a.y + w10 * b.y + w01 * c.y + w11 * d.y;
        const float ub = w00 * a.z + w10 * b.z + w01 * c.z + w11 * d.z;
        const float vb = w00 * a.w + w10 * b.w + w01 * c.w + w11 * d.w;
        u = blend32(wa, ua, wb, ub);
        v = blend32(wa, va, wb, vb);
    }
}

__device__ __forceinline__ void cub32(const float4 *p, int pitch, const float wx[4],
                                      const float wy[4], int smode, float wa, float wb, float &u,
                                      float &v)
{
    if (smode != kBlend) {
        const int h = smode;   // which half of the record
        float au = 0.f, av = 0.f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const float2 *q = reinterpret_cast<const float2 *>(p) + h;
            float ru = 0.f, rv = 0.f;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const float2 r = q[2 * a];
                ru += wx[a] * r.x;
                rv += wx[a] * r.y;
            }
            au += wy[b] * ru;
            av += wy[b] * rv;
            p += pitch;
        }
        u = au;
        v = av;
    } else {
        float au = 0.f, av = 0.f, bu = 0.f, bv = 0.f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float ru = 0.f, rv = 0.f, su = 0.f, sv = 0.f;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const float4 r = p[a];
                ru += wx[a] * r.x;
                rv += wx[a] * r.y;
                su += wx[a] * r.z;
                sv += wx[a] * r.w;
            }
            au += wy[b] * ru;
            av += wy[b] * rv;
            bu += wy[b] * su;
            bv += wy[b] * sv;
            p += pitch;
        }
        u = blend32(wa, au, wb, bu);
        v = blend32(wa, av, wb, bv);
    }
}

template <bool CUBIC>
__device__ __forceinline__ void vel32(const float4 *__restrict__ rec0, const float4 *tile,
                                      const Tile &T, const StepParams &P, int scheme, int cx,
                                      int cy, float qx, float qy, float wa, float wb, int smode,
                                      float &u, float &v)
{
    const float fx = floorf(qx), fy = floorf(qy);
    const float xi = __builtin_amdgcn_fractf(qx), eta = __builtin_amdgcn_fractf(qy);
    const int n = P.n, mask = P.mask;
    const int i = cell_plus(cx, fx, n, mask), j = cell_plus(cy, fy, n, mask);
    int t;
    if (!CUBIC || scheme == kBilinear || edge_cell(P.compat_edge, i, j, n)) {
        if (tile_index(T, i, j, 2, n, mask, t))
            bil32(tile + t, T.w, xi, eta, smode, wa, wb, u, v);
        else
            bil32(rec0 + (__mul24(j, P.pitch) + i), P.pitch, xi, eta, smode, wa, wb, u, v);
        return;
    }
    if constexpr (CUBIC) {
        float wx[4], wy[4];
        if (scheme == kCatmullRom) {
            weights_cr(xi, wx);
            weights_cr(eta, wy);
        } else {
            weights_bs(xi, wx);
            weights_bs(eta, wy);
        }
        if (tile_index(T, i - 1, j - 1, 4, n, mask, t))
            cub32(tile + t, T.w, wx, wy, smode, wa, wb, u, v);
        else
            cub32(rec0 + (__mul24(j - 1, P.pitch) + (i - 1)), P.pitch, wx, wy, smode, wa, wb, u, v);
    }
}

// New (cell, offset) after a displacement of dq cells from offset o; the
// offset stays in [0, 1) (fract never returns 1).
__device__ __forceinline__ int advance_split(int &c, float &o, float dq, const StepParams &P)
{
    const float q = o + dq;
    const float f = __builtin_amdgcn_fmed3f(floorf(q), -kCellClampF, kCellClampF);
    float r = __builtin_amdgcn_fractf(q);
    if (!(r >= 0.0f)) r = 0.0f;   // NaN guard keeps the state in range
    const int m = (int)f;         // the cell move (0 for NaN)
    c = wrap_cell(c + m, P.n, P.mask);
    o = r;
    return m;
}

// Unwrapped cell plus a move, wrapping modulo 2^32 (moves are clamped, so
// only an absurd state, never a real trajectory, gets there).
__device__ __forceinline__ int ucell_plus(int u, int m)
{
    return (int)((uint32_t)u + (uint32_t)m);
}

// Split form of a binary64 position: the cell floor(x n / L) in [0, n) and the
// binary32 offset in [0, 1) (the initial state of a particle).
__device__ __forceinline__ void split_of(double x, const StepParams &P, int &c, float &o)
{
    const double s = x * P.invh;
    const double f = floor(s);
    float r = (float)(s - f);
    int ci = cell_of_floor(f, P.n, P.mask);
    if (r >= 1.0f) {
        r = 0.0f;
        ci = wrap_cell(ci + 1, P.n, P.mask);
    }
    if (!(r >= 0.0f)) r = 0.0f;
    c = ci;
    o = r;
}

// Counter-indexed SplitMix64 (Steele, Lea & Flood, OOPSLA 2014): output k of
// the stream seeded with s is mix(s + (k + 1) * golden gamma).
__device__ __forceinline__ uint64_t splitmix_at(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

// Uniform initial position of particle k of a species drawn with `seed`:
// outputs 2k and 2k + 1 of the stream, top 53 bits as a fraction of L.  The
// one definition both the initialisation and the record steps use, so a
// position drawn again is the stored one, bit for bit.
__device__ __forceinline__ double2 draw_x0(uint64_t seed, uint64_t k, double L)
{
    const double ux = (double)(splitmix_at(seed, 2 * k) >> 11) * 0x1p-53;
    const double uy = (double)(splitmix_at(seed, 2 * k + 1) >> 11) * 0x1p-53;
    return make_double2(wrap_pos(L * ux, L), wrap_pos(L * uy, L));
}

// Initial position of particle g (global id) of species sp: drawn again
// where the species was initialised uniformly (a few integer operations
// instead of a gather in particle order, which is random after re-sorts),
// else read.
__device__ __forceinline__ double2 initial_pos(const SpeciesDev &sp, const double2 *x0, uint32_t g,
                                               const StepParams &P)
{
    if (sp.x0_drawn) return draw_x0(sp.x0_seed, (uint64_t)((int64_t)g - sp.offset), P.L);
    return x0[g];
}

// Displacement since initialisation (physical units) of a particle at
// unwrapped cell u, offset o, that started at x0.
__device__ __forceinline__ double2 split_disp(int2 u, float2 o, double2 x0, const StepParams &P)
{
    int cx, cy;
    float ox, oy;
    split_of(x0.x, P, cx, ox);
    split_of(x0.y, P, cy, oy);
    return make_double2(((double)(int)((uint32_t)u.x - (uint32_t)cx) + ((double)o.x - (double)ox)) * P.h,
                        ((double)(int)((uint32_t)u.y - (uint32_t)cy) + ((double)o.y - (double)oy)) * P.h);
}

// ---------------------------------------------------------------------------
// The FP32-split step, specialised per block on (scheme, particle kind).
// Stage positions are kept relative to the particle's stored cell: the stage
// cell is (cx + floor(qx), cy + floor(qy)) and, inside the LDS tile, its tile
// coordinate is (rx + floor(qx), ry + floor(qy)) with (rx, ry) the stored
// cell's tile coordinate, computed once per particle.  Only a stencil that
// leaves the tile needs the periodic wrap and a global gather.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wrapn(int c, const StepParams &P)
{
    return wrap_cell(c, P.n, P.mask);
}

// Node accessors of the FP32 step.  Global memory holds one {u0, v0, u1, v1}
// record per node (ghost-bordered rows of `pitch` records); the LDS tile
// holds two planes of (u, v), one per time level, so that a stage reading a
// single level gathers 8 dense bytes per node.  Both are addressed from the
// stencil's origin node (a, b: column and row offsets from it).
struct GlobalNodes {
    const float4 *p;
    int pitch;
    __device__ __forceinline__ float2 level(int a, int b, int h) const
    {
        return reinterpret_cast<const float2 *>(p + (b * pitch + a))[h];
    }
    __device__ __forceinline__ float4 both(int a, int b) const { return p[b * pitch + a]; }
};

// (The tile is addressed through an LDS pointer, not a generic one: where the
// compiler merges the two accessors' code it must not fall back to flat loads.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) f32x4 *LdsRec32;

struct TileNodes {
    LdsRec32 p;   // origin node
    int pitch;    // tile width
    __device__ __forceinline__ float2 level(int a, int b, int h) const
    {
        typedef const __attribute__((address_space(3))) f32x2 *LdsHalf32;
        const f32x2 v = ((LdsHalf32)(p + (b * pitch + a)))[h];
        return make_float2(v.x, v.y);
    }
    __device__ __forceinline__ float4 both(int a, int b) const
    {
        const f32x4 v = p[b * pitch + a];
        return make_float4(v.x, v.y, v.z, v.w);
    }
};

// Velocity of one stencil (eqs. bilinear_interp, cr_interp, bspline_interp)
// with the temporal interpolation of eq. temporal_interp: ONE reads only
// level h (weight (1, 0) or (0, 1)); otherwise both levels blend with
// (wa, wb).  LANES = 4: a bicubic stencil split by rows over a group of four
// lanes with the same arguments (the same sums in the same order).
template <int SCH, int LANES, typename Nodes>
__device__ __forceinline__ void eval32(const Nodes &N, float xi, float eta, bool one, int h,
                                       float wa, float wb, float &u, float &v)
{
    if constexpr (SCH == kBilinear) {
        float w00, w10, w01, w11;
        bilinear_weights(xi, eta, w00, w10, w01, w11);
        if (one) {
            const float2 a = N.level(0, 0, h), b = N.level(1, 0, h);
            const float2 c = N.level(0, 1, h), d = N.level(1, 1, h);
            u = w00 * a.x + w10 * b.x + w01 * c.x + w11 * d.x;
            v = w00 * a.y + w10 * b.y + w01 * c.y + w11 * d.y;
        } else {
            const float4 a = N.both(0, 0), b = N.both(1, 0), c = N.both(0, 1), d = N.both(1, 1);
            const float ua = w00 * a.x + w10 * b.x + w01 * c.x + w11 * d.x;
            const float va = w00 * a.y + w10 * b.y + w01 * c.y + w11 * d.y;
            const float ub = w00 * a.z + w10 * b.z + w01 * c.z + w11 * d.z;
            const float vb = w00 * a.w + w10 * b.w + w01 * c.w + w11 * d.w;
            u = blend32(wa, ua, wb, ub);
            v = blend32(wa, va, wb, vb);
        }
    } else {
        float wx[4], wy[4];
        if constexpr (SCH == kCatmullRom) {
            weights_cr(xi, wx);
            weights_cr(eta, wy);
        } else {
            weights_bs(xi, wx);
            weights_bs(eta, wy);
        }
        if constexpr (LANES == 4) {
            const int b = (int)threadIdx.x & 3;
            float ru = 0.f, rv = 0.f, su = 0.f, sv = 0.f;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                float4 r;
                if (one) {
                    const float2 q = N.level(a, b, h);
                    r = make_float4(q.x, q.y, 0.f, 0.f);
                } else {
                    r = N.both(a, b);
                }
                ru += wx[a] * r.x;
                rv += wx[a] * r.y;
                su += wx[a] * r.z;
                sv += wx[a] * r.w;
            }
            u = quad_rows(wy, ru);
            v = quad_rows(wy, rv);
            if (!one) {
                u = blend32(wa, u, wb, quad_rows(wy, su));
                v = blend32(wa, v, wb, quad_rows(wy, sv));
            }
        } else if (one) {
            // the loads of a whole stencil, or of half of one with both levels,
            // before their first use: 32 registers in flight
            float2 r[4][4];
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) r[b][a] = N.level(a, b, h);
            float au = 0.f, av = 0.f;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                float ru = 0.f, rv = 0.f;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    ru += wx[a] * r[b][a].x;
                    rv += wx[a] * r[b][a].y;
                }
                au += wy[b] * ru;
                av += wy[b] * rv;
            }
            u = au;
            v = av;
        } else {
            float au = 0.f, av = 0.f, bu = 0.f, bv = 0.f;
#pragma unroll
            for (int b0 = 0; b0 < 4; b0 += 2) {
                float4 r[2][4];
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int a = 0; a < 4; ++a) r[b][a] = N.both(a, b0 + b);
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    float ru = 0.f, rv = 0.f, su = 0.f, sv = 0.f;
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        ru += wx[a] * r[b][a].x;
                        rv += wx[a] * r[b][a].y;
                        su += wx[a] * r[b][a].z;
                        sv += wx[a] * r[b][a].w;
                    }
                    au += wy[b0 + b] * ru;
                    av += wy[b0 + b] * rv;
                    bu += wy[b0 + b] * su;
                    bv += wy[b0 + b] * sv;
                }
            }
            u = blend32(wa, au, wb, bu);
            v = blend32(wa, av, wb, bv);
        }
    }
}

__device__ __forceinline__ TileNodes tile_nodes(const float4 *lds, const Tile &T, int tx, int ty)
{
    return TileNodes{(LdsRec32)lds + (__mul24(ty, T.w) + tx), T.w};
}

__device__ __forceinline__ GlobalNodes global_nodes(const float4 *rec0, const StepParams &P,
                                                    int i, int j)
{
    return GlobalNodes{rec0 + (__mul24(j, P.pitch) + i), P.pitch};
}

// Fluid velocity (cells per unit time) of one RK4 stage at stored cell
// (cx, cy) + q.  (rx, ry): tile coordinate of the stored cell.
template <int SCH, int LANES>
__device__ __forceinline__ void stage32(const float4 *__restrict__ rec0, const float4 *lds,
                                        const Tile &T, const StepParams &P, int cx, int cy,
                                        int rx, int ry, float qx, float qy, bool one, int h,
                                        float wa, float wb, float &u, float &v)
{
    constexpr int c1 = SCH == kBilinear ? 0 : 1;
    constexpr int span = SCH == kBilinear ? 2 : 4;
    qx = __builtin_amdgcn_fmed3f(qx, -kCellClampF, kCellClampF);
    qy = __builtin_amdgcn_fmed3f(qy, -kCellClampF, kCellClampF);
    const float flx = floorf(qx), fly = floorf(qy);
    const int fx = (int)flx, fy = (int)fly;
    const float xi = qx - flx, eta = qy - fly;
    if constexpr (SCH != kBilinear) {
        if (P.compat_edge) {   // the paper's bilinear fallback near the grid edge
            const int i = wrapn(cx + fx, P), j = wrapn(cy + fy, P);
            if (edge_cell(1, i, j, P.n)) {
                eval32<kBilinear, 1>(global_nodes(rec0, P, i, j), xi, eta, one, h, wa, wb, u, v);
                return;
            }
        }
    }
    const int tx = rx + fx - c1, ty = ry + fy - c1;
    if (T.on && (unsigned)tx <= (unsigned)(T.w - span) && (unsigned)ty <= (unsigned)(T.h - span)) {
        eval32<SCH, LANES>(tile_nodes(lds, T, tx, ty), xi, eta, one, h, wa, wb, u, v);
    } else {
        const int i = wrapn(cx + fx, P) - c1, j = wrapn(cy + fy, P) - c1;
        eval32<SCH, LANES>(global_nodes(rec0, P, i, j), xi, eta, one, h, wa, wb, u, v);
    }
}

// The first stage sits at the stored position itself: stored cell, in-cell
// coordinates = the stored offset in [0, 1) (so floor(q) = 0 and the general
// stage computes the same values).  The stored cell lies inside the block's
// box and the box adds the stencil reach, so the stencil is inside the tile
// unless the box was cut down to the tile's capacity.
template <int SCH, bool ONE, int LANES>
__device__ __forceinline__ void stage32_first(const float4 *__restrict__ rec0, const float4 *lds,
                                              const Tile &T, const StepParams &P, int cx, int cy,
                                              int rx, int ry, float2 o, int h, float wa, float wb,
                                              float &u, float &v)
{
    constexpr int c1 = SCH == kBilinear ? 0 : 1;
    if (SCH != kBilinear && P.compat_edge) {
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x, o.y, ONE, h, wa, wb, u, v);
        return;
    }
    constexpr int span = SCH == kBilinear ? 2 : 4;
    if (T.on && (unsigned)(rx - c1) <= (unsigned)(T.w - span) &&
        (unsigned)(ry - c1) <= (unsigned)(T.h - span))
        eval32<SCH, LANES>(tile_nodes(lds, T, rx - c1, ry - c1), o.x, o.y, ONE, h, wa, wb, u, v);
    else
        eval32<SCH, LANES>(global_nodes(rec0, P, cx - c1, cy - c1), o.x, o.y, ONE, h, wa, wb, u, v);
}

// The move (dqx, dqy), in cells, of one RK4 step of one particle at stored
// cell (cx, cy) and offset o (eqs. rk4_update / rk4_inertial, Stokes drag of
// eq. drag_rk4); an inertial particle's velocity vn is advanced too.  ONE:
// the first and the last stage read a single time level.
template <int SCH, bool INERT, bool ONE, int LANES>
__device__ __forceinline__ void rk4_split(const StepParams &P, const StageWeights &W,
                                          const float4 *__restrict__ rec0, const float4 *lds,
                                          const Tile &T, const SpeciesDev &sp, int cx, int cy,
                                          int rx, int ry, float2 o, float2 &vn, float &dqx,
                                          float &dqy)
{
    const float dt = P.dtf, hdt = P.hdtf, dt6 = P.dt6f;
    if constexpr (INERT) {
        const float is = (float)sp.inv_st;
        float u, v;
        const float V1x = vn.x, V1y = vn.y;
        stage32_first<SCH, ONE, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o, W.h0, W.waf[0],
                                       W.wbf[0], u, v);
        const float A1x = (u - V1x) * is, A1y = (v - V1y) * is;
        const float V2x = vn.x + hdt * A1x, V2y = vn.y + hdt * A1y;
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x + hdt * V1x, o.y + hdt * V1y,
                            false, 0, W.waf[1], W.wbf[1], u, v);
        const float A2x = (u - V2x) * is, A2y = (v - V2y) * is;
        const float V3x = vn.x + hdt * A2x, V3y = vn.y + hdt * A2y;
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x + hdt * V2x, o.y + hdt * V2y,
                            false, 0, W.waf[2], W.wbf[2], u, v);
        const float A3x = (u - V3x) * is, A3y = (v - V3y) * is;
        const float V4x = vn.x + dt * A3x, V4y = vn.y + dt * A3y;
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x + dt * V3x, o.y + dt * V3y, ONE,
                            W.h3, W.waf[3], W.wbf[3], u, v);
        const float A4x = (u - V4x) * is, A4y = (v - V4y) * is;
        dqx = dt6 * (V1x + 2.0f * V2x + 2.0f * V3x + V4x);
        dqy = dt6 * (V1y + 2.0f * V2y + 2.0f * V3y + V4y);
        vn = make_float2(vn.x + dt6 * (A1x + 2.0f * A2x + 2.0f * A3x + A4x),
                         vn.y + dt6 * (A1y + 2.0f * A2y + 2.0f * A3y + A4y));
    } else {
        float k1x, k1y, k2x, k2y, k3x, k3y, k4x, k4y;
        stage32_first<SCH, ONE, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o, W.h0, W.waf[0],
                                       W.wbf[0], k1x, k1y);
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x + hdt * k1x, o.y + hdt * k1y,
                            false, 0, W.waf[1], W.wbf[1], k2x, k2y);
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x + hdt * k2x, o.y + hdt * k2y,
                            false, 0, W.waf[2], W.wbf[2], k3x, k3y);
        stage32<SCH, LANES>(rec0, lds, T, P, cx, cy, rx, ry, o.x + dt * k3x, o.y + dt * k3y, ONE,
                            W.h3, W.waf[3], W.wbf[3], k4x, k4y);
        dqx = dt6 * (k1x + 2.0f * k2x + 2.0f * k3x + k4x);
        dqy = dt6 * (k1y + 2.0f * k2y + 2.0f * k3y + k4y);
    }
}

// The split position after a move (dqx, dqy): (cx, cy) is the stored cell,
// (uc, o) the unwrapped cell and the offset.
__device__ __forceinline__ void advance_cell(const StepParams &P, int cx, int cy, float dqx,
                                             float dqy, int2 &uc, float2 &o)
{
    float ox = o.x, oy = o.y;
    const int mx = advance_split(cx, ox, dqx, P);
    const int my = advance_split(cy, oy, dqy, P);
    uc = make_int2(ucell_plus(uc.x, mx), ucell_plus(uc.y, my));
    o = make_float2(ox, oy);
}

// rk4_split of the block's species.  SCHS: the scheme of every species of the
// launch (one launch per scheme), or kAnyScheme in a fused launch.  KINDS: 0
// tracers only (St == 0 included), 1 tracers and/or inertial species.
template <int SCHS, int KINDS>
__device__ __forceinline__ void rk4_species(const StepParams &P, const StageWeights &W,
                                            const float4 *__restrict__ rec0, const float4 *lds,
                                            const Tile &T, const SpeciesDev &sp, int cx, int cy,
                                            float2 o, float2 &vn, float &dqx, float &dqy)
{
    if constexpr (SCHS == kAnyScheme) {   // fused launch: the block's species decides
        if (sp.scheme == kBilinear)
            rk4_species<kBilinear, KINDS>(P, W, rec0, lds, T, sp, cx, cy, o, vn, dqx, dqy);
        else if (sp.scheme == kCatmullRom)
            rk4_species<kCatmullRom, KINDS>(P, W, rec0, lds, T, sp, cx, cy, o, vn, dqx, dqy);
        else
            rk4_species<kBSpline, KINDS>(P, W, rec0, lds, T, sp, cx, cy, o, vn, dqx, dqy);
    } else {
        int rx = 0, ry = 0;
        if (T.on) {   // cx - T.x0 lies in (-n, n)
            rx = cx - T.x0;
            ry = cy - T.y0;
            rx += rx < 0 ? P.n : 0;
            ry += ry < 0 ? P.n : 0;
        }
        if (W.ends_one) {
            if (KINDS != 0 && sp.inertial)
                rk4_split<SCHS, KINDS != 0, true, 1>(P, W, rec0, lds, T, sp, cx, cy, rx, ry, o, vn,
                                                     dqx, dqy);
            else
                rk4_split<SCHS, false, true, 1>(P, W, rec0, lds, T, sp, cx, cy, rx, ry, o, vn, dqx,
                                                dqy);
        } else {
            if (KINDS != 0 && sp.inertial)
                rk4_split<SCHS, KINDS != 0, false, 1>(P, W, rec0, lds, T, sp, cx, cy, rx, ry, o,
                                                      vn, dqx, dqy);
            else
                rk4_split<SCHS, false, false, 1>(P, W, rec0, lds, T, sp, cx, cy, rx, ry, o, vn,
                                                 dqx, dqy);
        }
    }
}

// One logical block of a launch: R.nsteps steps of the block's particles, which
// stay in registers, with a new tile for each step.  A logical block holds
// ROWS rows of blockDim.x slots: thread t takes slot t of every row, so that
// the block's set-up (its box, tile and launch bookkeeping) is shared by ROWS
// particles per thread.  Slot p of D takes the particle of slot p of S (D = S:
// in place), or, on the steps that follow a re-sort, of slot perm[p], id
// included.  The box of a step is taken about the centre of the box before
// (any cell near the particles will do).  RUN = false: one step in place (perm
// null, the weights in P.w), without the run's bookkeeping.
template <int SCHS, int KINDS, bool STATS, int ROWS, bool RUN>
__device__ __forceinline__ void step32_block(const StepParams &P, const StepRun &R,
                                             const State32 &S, const State32 &D,
                                             const uint32_t *perm_, const float4 *__restrict__ rec,
                                             double *__restrict__ partials, DevClock *clock,
                                             int lb)
{
    const uint32_t *perm = RUN ? perm_ : nullptr;
    const int nsteps = RUN ? R.nsteps : 1;
    float4 *lds = reinterpret_cast<float4 *>(lpt_dyn_lds);
    const SpeciesDev &sp = P.sp[P.nspecies > 1 ? species_of(P, lb) : 0];
    const int threads = (int)blockDim.x;
    const int64_t slots = (int64_t)threads * ROWS;
    const int64_t base = (int64_t)(lb - sp.block_begin) * slots;
    const int64_t first = base + threadIdx.x;   // row r: first + r * threads
    const float4 *rec0 = rec + P.pitch + 1;
    const bool inert = KINDS != 0 && sp.inertial;

    int2 uc[ROWS];
    float2 o[ROWS], vn[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        uc[r] = make_int2(0, 0);
        o[r] = vn[r] = make_float2(0.f, 0.f);
        const int64_t local = first + (int64_t)r * threads;
        if (local < sp.count) {
            const int64_t p = sp.offset + local, q = perm ? (int64_t)perm[p] : p;
            uc[r] = ld_stream(S.uc + q);
            o[r] = ld_stream(S.off + q);
            if (inert) vn[r] = ld_stream(S.vel + q);
        }
    }
    int ax = 0, ay = 0, lo = 0, hi = 0, nact = 0;
    if (P.tile_cap > 0) {
        stencil_reach(sp.scheme, lo, hi);
        const int H = step_halo(P, sp.scheme, P.dtf);
        lo += H;
        hi += H;
        const int64_t left = sp.count - base;
        nact = (int)(left < slots ? left : slots);
        const int64_t a0 = sp.offset + base;
        const int2 a = S.uc[perm ? (int64_t)perm[a0] : a0];
        ax = wrapn(a.x, P);
        ay = wrapn(a.y, P);
    }
    for (int k = 0; k < nsteps; ++k) {
        const StageWeights &W = RUN ? R.w[k] : P.w;
        Tile T = no_tile();
        if (P.tile_cap > 0) {
            BoxAcc b = box_init();
            bool any = false;
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
                if (first + (int64_t)r * threads < sp.count) {
                    const BoxAcc c = box_of(wrapn(uc[r].x, P), wrapn(uc[r].y, P), ax, ay, P.n);
                    b = any ? BoxAcc{pmax16(b.up, c.up), pmax16(b.dn, c.dn)} : c;
                    any = true;
                }
            T = stage_tile_acc<float4>(lds, rec0, P, b, ax, ay, lo, hi, nact);
            ax = wrapn(T.x0 + T.w / 2, P);
            ay = wrapn(T.y0 + T.h / 2, P);
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (first + (int64_t)r * threads < sp.count) {
                const int cx = wrapn(uc[r].x, P), cy = wrapn(uc[r].y, P);
                float dqx, dqy;
                rk4_species<SCHS, KINDS>(P, W, rec0, lds, T, sp, cx, cy, o[r], vn[r], dqx, dqy);
                advance_cell(P, cx, cy, dqx, dqy, uc[r], o[r]);
            }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int64_t local = first + (int64_t)r * threads;
        const bool active = local < sp.count;
        double r2x = 0.0, r2y = 0.0;
        if (active) {
            const int64_t p = sp.offset + local;
            st_stream(D.uc + p, uc[r]);
            st_stream(D.off + p, o[r]);
            if (inert) st_stream(D.vel + p, vn[r]);
            if (perm || STATS) {
                const uint32_t g = S.id[perm ? (int64_t)perm[p] : p];
                if (perm) D.id[p] = g;
                if (STATS) {   // the displacement since initialisation, from the new state
                    const double2 d = split_disp(uc[r], o[r], initial_pos(sp, S.x0, g, P), P);
                    r2x = d.x * d.x;
                    r2y = d.y * d.y;
                }
            }
        }
        // one partial per 64 slots, in slot order: wave w of row r covers the
        // slots lb * slots + r * threads + 64 w + [0, 64)
        if (STATS)
            wave_stats(r2x, r2y, active,
                       partials + (int64_t)kStatTerms *
                                      (((int64_t)lb * slots + (int64_t)r * threads) / kWave +
                                       threadIdx.x / kWave));
    }
    if (lb == 0) advance_clock(P, nsteps, clock);
}

// One launch advances every particle of its logical blocks by one step in place
// (block_walk: one workgroup per logical block in XCD-aware order, a
// persistent walk, or a fused launch's block-order table).
// Bilinear blocks hold eight 256-thread blocks per CU (the LDS tile's
// budget), i.e. eight waves per SIMD, so their registers are bounded to fit
// that (49-63); the bicubic bodies, and the fused kernel that holds every body
// (SCHS = kAnyScheme), need more and are bounded to six (73-80; inertial ones
// spill up to 40 bytes a lane, in the run kernels below up to 48).
template <int SCHS, int KINDS, bool STATS, int ROWS>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(SCHS == kBilinear ? 8 : 6, SCHS == kBilinear ? 8 : 6)))
void step32_kernel(StepParams P, State32 S, const float4 *__restrict__ rec,
                   double *__restrict__ partials, DevClock *clock)
{
    const StepRun none{};
    BlockWalk w = block_walk(P, P.block_base, P.launch_blocks);
    for (int lb = 0; block_next(w, lb);)
        step32_block<SCHS, KINDS, STATS, ROWS, false>(P, none, S, S, nullptr, rec, partials, clock,
                                                      lb);
}

// Runs of steps in one launch, and the step that follows a re-sort.
template <int SCHS, int KINDS, bool STATS, int ROWS>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(SCHS == kBilinear ? 8 : 6, SCHS == kBilinear ? 8 : 6)))
void run32_kernel(StepParams P, StepRun R, State32 S, State32 D, const uint32_t *perm,
                  const float4 *__restrict__ rec, double *__restrict__ partials, DevClock *clock)
{
    BlockWalk w = block_walk(P, P.block_base, P.launch_blocks);
    for (int lb = 0; block_next(w, lb);)
        step32_block<SCHS, KINDS, STATS, ROWS, true>(P, R, S, D, perm, rec, partials, clock, lb);
}

// ===========================================================================
// Runs of steps for populations too small to fill the chip, or too sparse to
// share a tile.  Such a launch lasts as long as one wave's chain of dependent
// gathers, plus the launch itself, whatever the number of particles, so the
// particles keep their state in registers for up to kMaxRun steps (to the next record,
// re-sort or checkpoint), every wave has a CU to itself where there are
// enough (workgroups of 64 slots), and a bicubic stencil is split by rows
// over four lanes, which quarters the loads of the chain.  No LDS tile: the
// few particles of a workgroup share no nodes worth staging.  Each unit of 64
// slots is one statistics partial, as in the other step kernels, and every
// sum is taken in their order, so the results are the same bits.  4096
// particles, 64^2, 100 steps with 10 records: 911 -> 365 us a call; which
// populations count as small is decided where these are launched.
// ===========================================================================
template <int LANES>
struct SmallSlot {
    int64_t p, q;   // the slot, and where its particle is read from
    bool active;
    int64_t wave;   // statistics partial
};

// Unit u of 64 slots of species sp's logical block u / (block / 64).
template <int LANES>
__device__ __forceinline__ SmallSlot<LANES> small_slot(const SpeciesDev &sp, int unit,
                                                       int units_per_block, const uint32_t *perm)
{
    SmallSlot<LANES> s;
    const int64_t local = (int64_t)(unit - sp.block_begin * units_per_block) * kWave +
                          (int)threadIdx.x / LANES;
    s.active = local < sp.count;
    s.p = sp.offset + local;
    s.q = s.active && perm ? (int64_t)perm[s.p] : s.p;
    s.wave = unit;
    return s;
}

// The unit's statistics partial, by its first wave (one slot a lane).
template <int LANES>
__device__ __forceinline__ void small_stats(const SmallSlot<LANES> &s, double r2x, double r2y,
                                            double *partials)
{
    double *out = partials + (int64_t)kStatTerms * s.wave;
    if constexpr (LANES == 1) {
        wave_stats(r2x, r2y, s.active, out);
    } else {
        __shared__ double r2[2][kWave];
        __shared__ int on[kWave];
        if (threadIdx.x % LANES == 0) {
            const int k = (int)threadIdx.x / LANES;
            r2[0][k] = r2x;
            r2[1][k] = r2y;
            on[k] = s.active;
        }
        __syncthreads();
        if (threadIdx.x < kWave)
            wave_stats(r2[0][threadIdx.x], r2[1][threadIdx.x], on[threadIdx.x] != 0, out);
    }
}

template <bool CUBIC, bool INERTIAL, bool STATS>
__global__ __launch_bounds__(CUBIC ? 4 * kWave : kWave) void small64_kernel(
    StepParams P, StepRun R, State64 S, State64 D, const uint32_t *perm,
    const Rec64 *__restrict__ rec, double *__restrict__ partials, DevClock *clock,
    int units_per_block)
{
    constexpr int LANES = CUBIC ? 4 : 1;
    const int unit = xcd_logical_block(blockIdx.x, gridDim.x);
    const SpeciesDev &sp = P.sp[species_of(P, unit / units_per_block)];
    const SmallSlot<LANES> s = small_slot<LANES>(sp, unit, units_per_block, perm);
    const Rec64 *rec0 = rec + P.pitch + 1;
    double r2x = 0.0, r2y = 0.0;
    if (s.active) {
        double2 x = S.pos[s.q], d = S.disp[s.q], vn = make_double2(0.0, 0.0);
        const bool inert = INERTIAL && sp.inertial;
        if (inert) vn = S.vel[s.q];
        for (int k = 0; k < R.nsteps; ++k) {
            const StageWeights &W = R.w[k];
            double ddx, ddy;
            if (inert)
                rk4_inertial64<CUBIC, LANES>(rec0, nullptr, no_tile(), P, W, sp.scheme, sp.inv_st,
                                             x, vn, ddx, ddy);
            else
                rk4_tracer64<CUBIC, LANES>(rec0, nullptr, no_tile(), P, W, sp.scheme, x, ddx, ddy);
            x = make_double2(wrap_pos(x.x + ddx, P.L), wrap_pos(x.y + ddy, P.L));
            d.x += ddx;
            d.y += ddy;
        }
        if (threadIdx.x % LANES == 0) {
            D.pos[s.p] = x;
            D.disp[s.p] = d;
            if (inert) D.vel[s.p] = vn;
            if (perm) D.id[s.p] = S.id[s.q];
        }
        r2x = d.x * d.x;
        r2y = d.y * d.y;
    }
    if (STATS) small_stats<LANES>(s, r2x, r2y, partials);
    if (blockIdx.x == 0) advance_clock(P, R.nsteps, clock);
}

// The steps of one split particle of one scheme.
template <int SCH, bool INERT, int LANES>
__device__ __forceinline__ void small32_steps(const StepParams &P, const StepRun &R,
                                              const float4 *__restrict__ rec0,
                                              const SpeciesDev &sp, int2 &uc, float2 &o,
                                              float2 &vn)
{
    for (int k = 0; k < R.nsteps; ++k) {
        const StageWeights &W = R.w[k];
        const int cx = wrapn(uc.x, P), cy = wrapn(uc.y, P);
        float dqx, dqy;
        if (W.ends_one)
            rk4_split<SCH, INERT, true, LANES>(P, W, rec0, nullptr, no_tile(), sp, cx, cy, 0, 0, o,
                                               vn, dqx, dqy);
        else
            rk4_split<SCH, INERT, false, LANES>(P, W, rec0, nullptr, no_tile(), sp, cx, cy, 0, 0,
                                                o, vn, dqx, dqy);
        advance_cell(P, cx, cy, dqx, dqy, uc, o);
    }
}

template <bool CUBIC, bool INERTIAL, bool STATS>
__global__ __launch_bounds__(CUBIC ? 4 * kWave : kWave) void small32_kernel(
    StepParams P, StepRun R, State32 S, State32 D, const uint32_t *perm,
    const float4 *__restrict__ rec, double *__restrict__ partials, DevClock *clock,
    int units_per_block)
{
    constexpr int LANES = CUBIC ? 4 : 1;
    const int unit = xcd_logical_block(blockIdx.x, gridDim.x);
    const SpeciesDev &sp = P.sp[species_of(P, unit / units_per_block)];
    const SmallSlot<LANES> s = small_slot<LANES>(sp, unit, units_per_block, perm);
    const float4 *rec0 = rec + P.pitch + 1;
    double r2x = 0.0, r2y = 0.0;
    if (s.active) {
        int2 uc = S.uc[s.q];
        float2 o = S.off[s.q], vn = make_float2(0.f, 0.f);
        const bool inert = INERTIAL && sp.inertial;
        if (inert) vn = S.vel[s.q];
        auto steps = [&](auto kind) {
            constexpr bool K = decltype(kind)::value;
            if (!CUBIC || sp.scheme == kBilinear)
                small32_steps<kBilinear, K, LANES>(P, R, rec0, sp, uc, o, vn);
            else if (sp.scheme == kCatmullRom)
                small32_steps<kCatmullRom, K, LANES>(P, R, rec0, sp, uc, o, vn);
            else
                small32_steps<kBSpline, K, LANES>(P, R, rec0, sp, uc, o, vn);
        };
        if (INERTIAL && inert)
            steps(std::integral_constant<bool, INERTIAL>{});
        else
            steps(std::integral_constant<bool, false>{});
        if (threadIdx.x % LANES == 0) {
            D.uc[s.p] = uc;
            D.off[s.p] = o;
            if (inert) D.vel[s.p] = vn;
            if (perm) D.id[s.p] = S.id[s.q];
        }
        if (STATS) {   // the displacement since initialisation, from the new state
            const double2 d = split_disp(uc, o, initial_pos(sp, S.x0, S.id[s.q], P), P);
            r2x = d.x * d.x;
            r2y = d.y * d.y;
        }
    }
    if (STATS) small_stats<LANES>(s, r2x, r2y, partials);
    if (blockIdx.x == 0) advance_clock(P, R.nsteps, clock);
}

// Grid of a launch: one workgroup per logical block (per table entry in a
// fused launch), or -- when the step parameters ask for a persistent launch
// -- as many workgroups as the device keeps resident (occupancy of this
// kernel at this block size and LDS size, times the CU count, capped at
// P.max_wg if set; a multiple of the XCD count in a fused launch), if that
// is fewer.
template <typename K>
static int launch_grid(K kernel, const StepParams &P, int block, size_t lds, int grid,
                       StepParams &Q)
{
    Q = P;
    Q.persistent = 0;
    if (P.order) grid = 8 * P.order_len;
    if (!P.persistent) return grid;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, lds) != hipSuccess ||
        per_cu < 1) {
        (void)hipGetLastError();
        return grid;
    }
    int64_t resident = (int64_t)per_cu * cus;
    if (P.max_wg > 0 && resident > P.max_wg) resident = P.max_wg;
    if (P.order) resident = resident < 8 ? 8 : resident / 8 * 8;
    if (resident >= grid) return grid;
    Q.persistent = 1;
    return (int)resident;
}

// Automatic LDS tile capacity of an FP32 step kernel at a block size: the
// CU's LDS split between as many blocks as the kernel's registers let stay
// resident (less each block's static LDS), in whole 64-entry fill chunks,
// lowered while it would still cost a resident block.  planes: 16-byte
// entries per node record (one for FP32; two, plus one chunk of fill
// overrun, for FP64).  The occupancy queries run once per (kernel, block
// size, device).
template <typename K>
static int32_t auto_tile_cap(K kernel, int block, int planes, int32_t fallback)
{
    static std::mutex mu;
    static std::map<std::tuple<const void *, int, int>, int32_t> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return fallback;
    }
    const auto key = std::make_tuple(reinterpret_cast<const void *>(kernel), block, dev);
    std::lock_guard<std::mutex> lock(mu);
    const auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    auto lds_of = [planes](int32_t cap) {
        return planes == 1 ? (size_t)cap * 16 : (size_t)(2 * cap + kWave) * 16;
    };
    int lds_cu = 0, blocks = 0;
    hipFuncAttributes fa{};
    int32_t cap = fallback;
    if (hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) ==
            hipSuccess &&
        hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(kernel)) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, block, 0) == hipSuccess &&
        blocks > 0 && lds_cu > 0) {
        const int64_t per_block = (int64_t)lds_cu / blocks - (int64_t)fa.sharedSizeBytes;
        const int64_t entries = per_block / 16 - (planes == 1 ? 0 : kWave);
        int64_t c = entries / planes / kWave * kWave;
        const int64_t most = (int64_t)(61440 / (16 * planes)) / kWave * kWave;
        c = c > most ? most : c;
        int resident = 0;
        while (c >= kWave &&
               (hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, kernel, block,
                                                             lds_of((int32_t)c)) != hipSuccess ||
                resident < blocks))
            c -= kWave;
        if (c >= kWave) cap = (int32_t)c;
    }
    (void)hipGetLastError();
    cache.emplace(key, cap);
    return cap;
}

template <bool C, bool I, bool S>
static hipError_t launch64_t(const StepParams &P, const StepRun &R, const State64 &St, const State64 &Dst,
                             const uint32_t *perm, const Rec64 *rec, double *partials,
                             DevClock *clock, int block, int grid, hipStream_t st)
{
    // The FP64 tile keeps its fixed capacity in automatic mode too: sized to
    // the register-bound occupancy it would leave too many boxes uncovered.
    const StepParams &P1 = P;
    // two planes of 16-byte entries; the fill writes whole 64-entry chunks of each
    const size_t lds = P1.tile_cap > 0 ? (size_t)(2 * P1.tile_cap + kWave) * 16 : 0;
    StepParams Q;
    if (perm || R.nsteps > 1) {
        const int g = launch_grid(run64_kernel<C, I, S>, P1, block, lds, grid, Q);
        hipLaunchKernelGGL((run64_kernel<C, I, S>), dim3(g), dim3(block), lds, st, Q, R, St, Dst,
                           perm, rec, partials, clock);
    } else {
        const int g = launch_grid(step64_kernel<C, I, S>, P1, block, lds, grid, Q);
        hipLaunchKernelGGL((step64_kernel<C, I, S>), dim3(g), dim3(block), lds, st, Q, St, rec,
                           partials, clock);
    }
    return hipGetLastError();
}

template <int SCHS, int KINDS, bool ST, int ROWS>
static hipError_t launch32_r(const StepParams &P, const StepRun &R, const State32 &S, const State32 &D,
                             const uint32_t *perm, const float4 *rec, double *partials,
                             DevClock *clock, int block, int grid, hipStream_t st)
{
    // a logical block of `block` slots runs on block / ROWS threads
    const int threads = block / ROWS;
    StepParams P1 = P;
    const bool run = perm || R.nsteps > 1;
    if (P.tile_auto && P.tile_cap > 0)
        P1.tile_cap = run ? auto_tile_cap(run32_kernel<SCHS, KINDS, ST, ROWS>, threads, 1,
                                          P.tile_cap)
                          : auto_tile_cap(step32_kernel<SCHS, KINDS, ST, ROWS>, threads, 1,
                                          P.tile_cap);
    // whole 64-entry chunks: the tile fill writes LDS a wave's chunk at a time
    const size_t lds =
        P1.tile_cap > 0 ? (size_t)((P1.tile_cap + kWave - 1) / kWave * kWave) * sizeof(float4) : 0;
    StepParams Q;
    if (run) {
        const int g = launch_grid(run32_kernel<SCHS, KINDS, ST, ROWS>, P1, threads, lds, grid, Q);
        hipLaunchKernelGGL((run32_kernel<SCHS, KINDS, ST, ROWS>), dim3(g), dim3(threads), lds, st,
                           Q, R, S, D, perm, rec, partials, clock);
    } else {
        const int g = launch_grid(step32_kernel<SCHS, KINDS, ST, ROWS>, P1, threads, lds, grid, Q);
        hipLaunchKernelGGL((step32_kernel<SCHS, KINDS, ST, ROWS>), dim3(g), dim3(threads), lds, st,
                           Q, S, rec, partials, clock);
    }
    return hipGetLastError();
}

template <int SCHS, int KINDS, bool ST>
static hipError_t launch32_t(const StepParams &P, const StepRun &R, const State32 &S, const State32 &D,
                             const uint32_t *perm, const float4 *rec, double *partials,
                             DevClock *clock, int block, int grid, hipStream_t st)
{
    // two rows per thread exist for the bilinear tracer bodies only (the
    // bodies where the block's set-up is the largest share of the work);
    // every other body runs one row, whatever P.rows asks
    if constexpr (SCHS == kBilinear && KINDS == 0)
        if (P.rows == 2)
            return launch32_r<SCHS, KINDS, ST, 2>(P, R, S, D, perm, rec, partials, clock, block, grid,
                                                  st);
    return launch32_r<SCHS, KINDS, ST, 1>(P, R, S, D, perm, rec, partials, clock, block, grid, st);
}

template <int SCHS>
static hipError_t launch32_s(const StepParams &P, const StepRun &R, const State32 &S, const State32 &D,
                             const uint32_t *perm, const float4 *rec, double *partials,
                             DevClock *clock, bool stats, bool inertial, int block, int grid,
                             hipStream_t st)
{
    if (inertial)
        return stats ? launch32_t<SCHS, 1, true>(P, R, S, D, perm, rec, partials, clock, block, grid,
                                                 st)
                     : launch32_t<SCHS, 1, false>(P, R, S, D, perm, rec, partials, clock, block,
                                                  grid, st);
    return stats ? launch32_t<SCHS, 0, true>(P, R, S, D, perm, rec, partials, clock, block, grid, st)
                 : launch32_t<SCHS, 0, false>(P, R, S, D, perm, rec, partials, clock, block, grid,
                                              st);
}

#define LPT_DISPATCH(fn, ...)                                                        \
    do {                                                                             \
        const int sel = (cubic ? 4 : 0) | (inertial ? 2 : 0) | (stats ? 1 : 0);      \
        switch (sel) {                                                               \
        case 0: return fn<false, false, false>(__VA_ARGS__);                          \
        case 1: return fn<false, false, true>(__VA_ARGS__);                           \
        case 2: return fn<false, true, false>(__VA_ARGS__);                           \
        case 3: return fn<false, true, true>(__VA_ARGS__);                            \
        case 4: return fn<true, false, false>(__VA_ARGS__);                           \
        case 5: return fn<true, false, true>(__VA_ARGS__);                            \
        case 6: return fn<true, true, false>(__VA_ARGS__);                            \
        default: return fn<true, true, true>(__VA_ARGS__);                            \
        }                                                                            \
    } while (0)

hipError_t launch_step64(const StepParams &P, const StepRun &R, const State64 &S,
                         const State64 &D, const uint32_t *perm, const Rec64 *rec,
                         double *partials, DevClock *clock, bool stats, bool cubic,
                         bool inertial, int block, int grid, hipStream_t st)
{
    LPT_DISPATCH(launch64_t, P, R, S, D, perm, rec, partials, clock, block, grid, st);
}

hipError_t launch_step32(const StepParams &P, const StepRun &R, const State32 &S, const State32 &D,
                         const uint32_t *perm, const float4 *rec, double *partials,
                         DevClock *clock, bool stats, int schemes, bool inertial, int block,
                         int grid, hipStream_t st)
{
    switch (schemes) {
    case kBilinear:
        return launch32_s<kBilinear>(P, R, S, D, perm, rec, partials, clock, stats, inertial, block,
                                     grid, st);
    case kCatmullRom:
        return launch32_s<kCatmullRom>(P, R, S, D, perm, rec, partials, clock, stats, inertial,
                                       block, grid, st);
    case kBSpline:
        return launch32_s<kBSpline>(P, R, S, D, perm, rec, partials, clock, stats, inertial, block,
                                    grid, st);
    case kAnyScheme:
        return launch32_s<kAnyScheme>(P, R, S, D, perm, rec, partials, clock, stats, inertial,
                                      block, grid, st);
    default:
        return hipErrorInvalidValue;
    }
}
template <bool C, bool I, bool ST>
static hipError_t small64_t(const StepParams &P, const StepRun &R, const State64 &S,
                            const State64 &D, const uint32_t *perm, const Rec64 *rec,
                            double *partials, DevClock *clock, int block, hipStream_t st)
{
    const int upb = block / kWave;
    hipLaunchKernelGGL((small64_kernel<C, I, ST>), dim3(P.total_blocks * upb),
                       dim3(C ? 4 * kWave : kWave), 0, st, P, R, S, D, perm, rec, partials, clock,
                       upb);
    return hipGetLastError();
}

template <bool C, bool I, bool ST>
static hipError_t small32_t(const StepParams &P, const StepRun &R, const State32 &S,
                            const State32 &D, const uint32_t *perm, const float4 *rec,
                            double *partials, DevClock *clock, int block, hipStream_t st)
{
    const int upb = block / kWave;
    hipLaunchKernelGGL((small32_kernel<C, I, ST>), dim3(P.total_blocks * upb),
                       dim3(C ? 4 * kWave : kWave), 0, st, P, R, S, D, perm, rec, partials, clock,
                       upb);
    return hipGetLastError();
}

hipError_t launch_small64(const StepParams &P, const StepRun &R, const State64 &S,
                          const State64 &D, const uint32_t *perm, const Rec64 *rec,
                          double *partials, DevClock *clock, bool stats, bool cubic,
                          bool inertial, int block, hipStream_t st)
{
    LPT_DISPATCH(small64_t, P, R, S, D, perm, rec, partials, clock, block, st);
}

hipError_t launch_small32(const StepParams &P, const StepRun &R, const State32 &S,
                          const State32 &D, const uint32_t *perm, const float4 *rec,
                          double *partials, DevClock *clock, bool stats, bool cubic,
                          bool inertial, int block, hipStream_t st)
{
    LPT_DISPATCH(small32_t, P, R, S, D, perm, rec, partials, clock, block, st);
}

// ===========================================================================
// Statistics: fixed-order merge of the per-wave partials into one record per
// species (Sec. 3.2 and 5.5 quantities).  A wave's partial becomes (count,
// sum dx^2, sum dy^2, mean of r2, M2) with M2 = sum d^2 - (sum d)^2 / count
// the sum of squared deviations of r2 = dx^2 + dy^2 about the wave's mean (d
// is r2 shifted by a sample of the wave; see wave_stats).  Two partials
// merge by the pairwise update of Chan, Golub & LeVeque (1979):
// n = na + nb, delta = mean_b - mean_a, mean = mean_a + delta nb / n,
// M2 = M2a + M2b + delta^2 na nb / n.  Stage 1 merges runs of kFinChunk waves
// of one species per workgroup (sequentially per thread, then a butterfly
// over each wave, then the block's waves in order); stage 2 merges the runs
// of every species at once, one wave per species.  (A single launch whose
// last workgroup merges the runs needs agent-scope fences, whose L2
// write-backs cost more than the second launch.)  Every merge pairs the
// same operands in the same order whatever the scheduling, so the record
// does not depend on it.
// ===========================================================================
constexpr int kFinThreads = 256;
constexpr int kFinPerThread = 4;
constexpr int kFinChunk = kFinThreads * kFinPerThread;   // waves per stage-1 workgroup

struct Moments {
    double n, sx, sy, mean, m2;
};

__device__ __forceinline__ Moments merge_moments(const Moments &a, const Moments &b)
{
    if (b.n == 0.0) return a;
    if (a.n == 0.0) return b;
    const double n = a.n + b.n;
    const double f = b.n / n;
    const double d = b.mean - a.mean;
    return Moments{n, a.sx + b.sx, a.sy + b.sy, a.mean + d * f, a.m2 + b.m2 + d * d * (a.n * f)};
}

__device__ __forceinline__ double shfl_xor_f64(double v, int m)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)b, m);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(b >> 32), m);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Butterfly merge over a wave: at each level a lane pair merges (lower lane,
// higher lane), so both hold the same result; every lane ends with the merge
// of all 64 in a fixed tree order.
__device__ __forceinline__ Moments wave_merge(Moments m)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
#pragma unroll
    for (int k = 1; k < kWave; k <<= 1) {
        const Moments o{shfl_xor_f64(m.n, k), shfl_xor_f64(m.sx, k), shfl_xor_f64(m.sy, k),
                        shfl_xor_f64(m.mean, k), shfl_xor_f64(m.m2, k)};
        m = (lane & k) ? merge_moments(o, m) : merge_moments(m, o);
    }
    return m;
}

struct FinParams {
    int32_t nspecies;
    int32_t chunk_begin[kMaxSpecies + 1];   // first stage-1 chunk of each species
    int64_t wave_begin[kMaxSpecies];        // first wave partial of each species
    int64_t nwaves[kMaxSpecies];
    int64_t count[kMaxSpecies];
};

// Record of species s from the merged moments (lane 0 of the calling wave).
__device__ __forceinline__ void write_record(const FinParams &F, int s, const Moments &m, double t,
                                             double t0, int64_t idx, double *records, int64_t cap)
{
    if (idx >= cap) return;
    const double nn = (double)F.count[s];
    const double mx = m.sx / nn, my = m.sy / nn;
    const double var = F.count[s] > 1 ? m.m2 / (nn - 1.0) : 0.0;
    const double el = t - t0;
    double *r = records + ((int64_t)s * cap + idx) * 8;
    r[0] = t;
    r[1] = mx;
    r[2] = my;
    r[3] = mx + my;
    r[4] = el > 0.0 ? mx / (2.0 * el) : 0.0;
    r[5] = el > 0.0 ? my / (2.0 * el) : 0.0;
    r[6] = sqrt(var / nn);
    reinterpret_cast<int64_t *>(r)[7] = F.count[s];
}

// The run of kFinChunk waves of species s that starts at wave w0, merged by a
// group of kFinThreads threads (thread tid of it; the group's kFinThreads /
// kWave waves meet in sm); the group's first thread receives the run's
// moments.  Every thread of the block must call it.
__device__ __forceinline__ Moments merge_run(const FinParams &F, int s, int64_t w0, int tid,
                                             const double *__restrict__ partials,
                                             double (*sm)[5])
{
    Moments m{0.0, 0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < kFinPerThread; ++k) {
        const int64_t lw = w0 + (int64_t)tid * kFinPerThread + k;   // wave within the species
        if (lw >= F.nwaves[s]) break;
        const int64_t left = F.count[s] - lw * kWave;
        const int cnt = (int)(left < kWave ? (left > 0 ? left : 0) : kWave);
        if (cnt == 0) break;
        const double *q = partials + (int64_t)kStatTerms * (F.wave_begin[s] + lw);
        const double n = (double)cnt;
        const double m2 = fmax(q[3] - q[2] * (q[2] / n), 0.0);
        m = merge_moments(m, Moments{n, q[0], q[1], (q[0] + q[1]) / n, m2});
    }
    m = wave_merge(m);
    const int wv = tid / kWave;
    if ((tid & (kWave - 1)) == 0) {
        sm[wv][0] = m.n;
        sm[wv][1] = m.sx;
        sm[wv][2] = m.sy;
        sm[wv][3] = m.mean;
        sm[wv][4] = m.m2;
    }
    __syncthreads();
    Moments r{sm[0][0], sm[0][1], sm[0][2], sm[0][3], sm[0][4]};
    if (tid == 0)
        for (int k = 1; k < kFinThreads / kWave; ++k)
            r = merge_moments(r, Moments{sm[k][0], sm[k][1], sm[k][2], sm[k][3], sm[k][4]});
    return r;
}

__global__ __launch_bounds__(kFinThreads) void fin_chunks_kernel(FinParams F,
                                                                 const double *__restrict__ partials,
                                                                 double *__restrict__ chunks)
{
    __shared__ double sm[kFinThreads / kWave][5];
    const int c = blockIdx.x;
    int s = 0;
    while (s + 1 < F.nspecies && c >= F.chunk_begin[s + 1]) ++s;
    const Moments r = merge_run(F, s, (int64_t)(c - F.chunk_begin[s]) * kFinChunk,
                                (int)threadIdx.x, partials, sm);
    if (threadIdx.x == 0) {
        double *o = chunks + 5 * (int64_t)c;
        o[0] = r.n;
        o[1] = r.sx;
        o[2] = r.sy;
        o[3] = r.mean;
        o[4] = r.m2;
    }
}

// The record of species that are one run of waves each (up to 65536 particles):
// the run's moments are the species', so one workgroup merges and writes them
// all, a group of kFinThreads threads per species, in one launch (4.3 + 2.7 us
// as two).
constexpr int kFinGroups = 4;

__global__ __launch_bounds__(kFinThreads * kFinGroups) void fin_small_kernel(
    FinParams F, const double *__restrict__ partials, DevClock *clock, double *records,
    int64_t cap, double t0)
{
    __shared__ double sm[kFinGroups][kFinThreads / kWave][5];
    const int group = (int)threadIdx.x / kFinThreads, tid = (int)threadIdx.x % kFinThreads;
    const int groups = (int)blockDim.x / kFinThreads;
    const double t = clock->t;
    const int64_t idx = clock->nrec;
    for (int s0 = 0; s0 < F.nspecies; s0 += groups) {
        const int s = s0 + group < F.nspecies ? s0 + group : F.nspecies - 1;
        const Moments m = merge_run(F, s, 0, tid, partials, sm[group]);
        if (tid == 0 && s0 + group < F.nspecies) write_record(F, s, m, t, t0, idx, records, cap);
        __syncthreads();   // sm is written again; every thread has read the record index
    }
    if (threadIdx.x == 0) clock->nrec = idx + 1;
}

// One wave per species (blockDim.x = 64 x nspecies): lane l merges the runs
// l, l + 64, ... of its species in order, then the wave's butterfly; lane 0
// writes the record.
__global__ __launch_bounds__(kWave * kMaxSpecies) void fin_records_kernel(
    FinParams F, const double *__restrict__ chunks, DevClock *clock, double *records,
    int64_t cap, double t0)
{
    const double t = clock->t;
    const int64_t idx = clock->nrec;
    const int s = (int)threadIdx.x / kWave, lane = (int)(threadIdx.x & (kWave - 1));
    Moments m{0.0, 0.0, 0.0, 0.0, 0.0};
    for (int c = F.chunk_begin[s] + lane; c < F.chunk_begin[s + 1]; c += kWave) {
        const double *q = chunks + 5 * (int64_t)c;
        m = merge_moments(m, Moments{q[0], q[1], q[2], q[3], q[4]});
    }
    m = wave_merge(m);
    if (lane == 0) write_record(F, s, m, t, t0, idx, records, cap);
    __syncthreads();   // every wave has read the record index
    if (threadIdx.x == 0) clock->nrec = idx + 1;
}

int64_t stat_partials_doubles(const StepParams &P, int block)
{
    const int64_t waves = (int64_t)P.total_blocks * (block / kWave);
    return (int64_t)kStatTerms * waves + 5 * (waves / kFinChunk + P.nspecies + 1);
}

hipError_t launch_finalize(const StepParams &P, double *partials, DevClock *clock,
                           double *records, int64_t rec_cap, double t0, int block,
                           hipStream_t st)
{
    const int wpb = block / kWave;
    FinParams F{};
    F.nspecies = P.nspecies;
    int chunks = 0;
    for (int s = 0; s < P.nspecies; ++s) {
        const SpeciesDev &d = P.sp[s];
        F.chunk_begin[s] = chunks;
        F.wave_begin[s] = (int64_t)d.block_begin * wpb;
        F.nwaves[s] = (int64_t)(d.block_end - d.block_begin) * wpb;
        F.count[s] = d.count;
        chunks += (int)((F.nwaves[s] + kFinChunk - 1) / kFinChunk);
    }
    F.chunk_begin[P.nspecies] = chunks;
    bool one_run = true;
    for (int s = 0; s < P.nspecies; ++s) one_run = one_run && F.nwaves[s] <= kFinChunk;
    if (one_run) {
        const int groups = P.nspecies < kFinGroups ? P.nspecies : kFinGroups;
        hipLaunchKernelGGL(fin_small_kernel, dim3(1), dim3(kFinThreads * groups), 0, st, F,
                           partials, clock, records, rec_cap, t0);
        return hipGetLastError();
    }
    double *chunk_buf = partials + (int64_t)kStatTerms * P.total_blocks * wpb;
    if (chunks > 0)
        hipLaunchKernelGGL(fin_chunks_kernel, dim3(chunks), dim3(kFinThreads), 0, st, F, partials,
                           chunk_buf);
    hipLaunchKernelGGL(fin_records_kernel, dim3(1), dim3(kWave * P.nspecies), 0, st, F, chunk_buf,
                       clock, records, rec_cap, t0);
    return hipGetLastError();
}

// ===========================================================================
// Snapshot ingest: planar u, v of one time level into its half of the padded
// node records (ghost nodes are periodic images).
// ===========================================================================
__device__ __forceinline__ int ghost_source(int a, int n)
{
    int i = a - kGhostLo;
    if (i < 0) i += n;
    if (i >= n) i -= n;
    return i;
}

// Block-wide maximum of m folded into *out with an unsigned max on the
// binary32 bit pattern (non-negative floats order like their bits).  The
// atomic is skipped when *out already holds at least m: *out only grows, so
// a stale read can only cause an unneeded atomic, never a missed one (with a
// thousand blocks on one address the atomics are what costs).  Every thread
// of the block must call it.
__device__ __forceinline__ void block_max_to(float m, unsigned *out)
{
    __shared__ float red[kMaxBlock / kWave];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < (int)(blockDim.x / kWave); ++k) m = fmaxf(m, red[k]);
        const unsigned bits = __float_as_uint(m);
        if (bits > __atomic_load_n(out, __ATOMIC_RELAXED)) atomicMax(out, bits);
    }
}

// Grid centred differences of psi (eq. particle_velocity_reconstruction with
// the interpolation moved onto the grid): periodic neighbours.
__device__ __forceinline__ int nxt(int i, int n) { return i + 1 == n ? 0 : i + 1; }
__device__ __forceinline__ int prv(int i, int n) { return i == 0 ? n - 1 : i - 1; }

// One ingest pass: each node record's half for this level (ghost records
// are periodic images), and the level's largest |u| or |v| times vscale
// (cells per unit time), which the step kernel's LDS tile halo uses, folded
// into *umax.  PSI: the level is a stream function f = psi, and the node's
// velocity is its grid centred difference, u = (psi(j+1) - psi(j-1)) / 2h,
// v = -(psi(i+1) - psi(i-1)) / 2h, formed here (g is unused); else f = u,
// g = v.  Blocks walk columns a of the padded grid and stride over its rows,
// so the grid stays at about a thousand blocks (one atomic each); each
// thread issues the loads of kRows rows before it stores any of them.
template <bool FP64, bool PSI>
__global__ __launch_bounds__(256) void pack_kernel(void *rec, int slot, const double *__restrict__ f,
                                                   const double *__restrict__ g, int n,
                                                   double scale, double vscale, double inv2h,
                                                   unsigned *umax)
{
    constexpr int kRows = 4;
    const int pitch = n + kGhostLo + kGhostHi;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int G = gridDim.y;
    float m = 0.0f;
    if (a < pitch) {
        const int i = ghost_source(a, n);
        for (int b0 = blockIdx.y; b0 < pitch; b0 += kRows * G) {
            double uu[kRows], vv[kRows];
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const int b = b0 + k * G;
                uu[k] = vv[k] = 0.0;
                if (b < pitch) {
                    const int j = ghost_source(b, n);
                    if constexpr (PSI) {
                        uu[k] = (f[(int64_t)nxt(j, n) * n + i] - f[(int64_t)prv(j, n) * n + i]) * inv2h;
                        vv[k] = -(f[(int64_t)j * n + nxt(i, n)] - f[(int64_t)j * n + prv(i, n)]) * inv2h;
                    } else {
                        uu[k] = f[(int64_t)j * n + i];
                        vv[k] = g[(int64_t)j * n + i];
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const int b = b0 + k * G;
                if (b >= pitch) break;
                const int64_t r = (int64_t)b * pitch + a;
                if constexpr (FP64)
                    reinterpret_cast<double2 *>(static_cast<Rec64 *>(rec) + r)[slot] =
                        make_double2(uu[k], vv[k]);
                else
                    reinterpret_cast<float2 *>(static_cast<float4 *>(rec) + r)[slot] =
                        make_float2((float)(uu[k] * scale), (float)(vv[k] * scale));
                m = fmaxf(m, (float)(fmax(fabs(uu[k]), fabs(vv[k])) * vscale));
            }
        }
    }
    block_max_to(m, umax);
}

template <bool PSI>
static void launch_pack_t(void *rec, bool fp64, int slot, const double *f, const double *g, int n,
                          double scale, double vscale, double inv2h, float *umax, hipStream_t st)
{
    const int pitch = n + kGhostLo + kGhostHi, b = 256;
    const dim3 grid((pitch + b - 1) / b, pitch < 128 ? pitch : 128);
    unsigned *out = reinterpret_cast<unsigned *>(umax);
    if (fp64)
        hipLaunchKernelGGL((pack_kernel<true, PSI>), grid, dim3(b), 0, st, rec, slot, f, g, n, scale,
                           vscale, inv2h, out);
    else
        hipLaunchKernelGGL((pack_kernel<false, PSI>), grid, dim3(b), 0, st, rec, slot, f, g, n,
                           scale, vscale, inv2h, out);
}

hipError_t launch_pack(void *rec, bool fp64, int slot, const double *u, const double *v, int n,
                       double scale, double vscale, float *umax, hipStream_t st)
{
    launch_pack_t<false>(rec, fp64, slot, u, v, n, scale, vscale, 0.0, umax, st);
    return hipGetLastError();
}

hipError_t launch_pack_psi(void *rec, bool fp64, int slot, const double *psi, int n, double h,
                           double scale, double vscale, float *umax, hipStream_t st)
{
    launch_pack_t<true>(rec, fp64, slot, psi, nullptr, n, scale, vscale, 1.0 / (2.0 * h), umax,
                        st);
    return hipGetLastError();
}

// ===========================================================================
// Initial state.  Positions come from x0 (original order); the velocity of an
// inertial species is taken from the field or from v0.
// ===========================================================================
__device__ __forceinline__ int smode_of(double wa, double wb)
{
    return wb == 0.0 && wa == 1.0 ? kSlot0 : (wa == 0.0 && wb == 1.0 ? kSlot1 : kBlend);
}

__global__ void init64_kernel(StepParams P, State64 S, const double2 *__restrict__ x0,
                              const double2 *__restrict__ v0, const Rec64 *__restrict__ rec,
                              int species, int64_t begin, int64_t count, double wa, double wb,
                              int vel_from_field)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int64_t p = begin + k;
    const SpeciesDev &sp = P.sp[species];
    const double2 x = x0[p];
    S.pos[p] = make_double2(wrap_pos(x.x, P.L), wrap_pos(x.y, P.L));
    S.disp[p] = make_double2(0.0, 0.0);
    S.id[p] = (uint32_t)p;
    if (sp.inertial) {
        if (vel_from_field) {
            double u, v;
            vel64<true>(rec + P.pitch + 1, nullptr, no_tile(), P, sp.scheme, x.x, x.y, wa, wb, smode_of(wa, wb), u, v);
            S.vel[p] = make_double2(u, v);
        } else {
            S.vel[p] = v0[p];
        }
    }
}

__global__ void init32_kernel(StepParams P, State32 S, const double2 *__restrict__ x0,
                              const double2 *__restrict__ v0, const float4 *__restrict__ rec,
                              int species, int64_t begin, int64_t count, double wa, double wb,
                              int vel_from_field)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int64_t p = begin + k;
    const SpeciesDev &sp = P.sp[species];
    const double2 x = x0[p];
    int cx, cy;
    float ox, oy;
    split_of(x.x, P, cx, ox);
    split_of(x.y, P, cy, oy);
    S.uc[p] = make_int2(cx, cy);
    S.off[p] = make_float2(ox, oy);
    S.id[p] = (uint32_t)p;
    if (sp.inertial) {
        if (vel_from_field) {
            float u, v;
            vel32<true>(rec + P.pitch + 1, nullptr, no_tile(), P, sp.scheme, cx, cy, ox, oy, (float)wa, (float)wb,
                        smode_of(wa, wb), u, v);
            S.vel[p] = make_float2(u, v);
        } else {
            S.vel[p] = make_float2((float)(v0[p].x * P.invh), (float)(v0[p].y * P.invh));
        }
    }
}

hipError_t launch_init64(const StepParams &P, const State64 &S, const double2 *x0,
                         const double2 *v0, const Rec64 *rec, int species, int64_t begin,
                         int64_t count, double wa, double wb, int vel_from_field,
                         hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const int b = 256;
    hipLaunchKernelGGL(init64_kernel, dim3((unsigned)((count + b - 1) / b)), dim3(b), 0, st, P,
                       S, x0, v0, rec, species, begin, count, wa, wb, vel_from_field);
    return hipGetLastError();
}

hipError_t launch_init32(const StepParams &P, const State32 &S, const double2 *x0,
                         const double2 *v0, const float4 *rec, int species, int64_t begin,
                         int64_t count, double wa, double wb, int vel_from_field,
                         hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const int b = 256;
    hipLaunchKernelGGL(init32_kernel, dim3((unsigned)((count + b - 1) / b)), dim3(b), 0, st, P,
                       S, x0, v0, rec, species, begin, count, wa, wb, vel_from_field);
    return hipGetLastError();
}

__global__ void interleave_kernel(double2 *dst, const double *__restrict__ a,
                                  const double *__restrict__ b, int64_t n)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = make_double2(a[k], b[k]);
}

hipError_t launch_interleave(double2 *dst, const double *a, const double *b, int64_t n,
                             hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int bs = 256;
    hipLaunchKernelGGL(interleave_kernel, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, st,
                       dst, a, b, n);
    return hipGetLastError();
}

__global__ void splitmix_kernel(double2 *x0, int64_t count, uint64_t seed, double L)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    x0[k] = draw_x0(seed, (uint64_t)k, L);
}

hipError_t launch_splitmix(double2 *x0, int64_t count, uint64_t seed, double L, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const int b = 256;
    hipLaunchKernelGGL(splitmix_kernel, dim3((unsigned)((count + b - 1) / b)), dim3(b), 0, st,
                       x0, count, seed, L);
    return hipGetLastError();
}

// ===========================================================================
// Velocity probe at arbitrary points (verification entry point).
// ===========================================================================
__global__ void interp64_kernel(StepParams P, const Rec64 *__restrict__ rec, int scheme,
                                int64_t npts, const double *__restrict__ x,
                                const double *__restrict__ y, double wa, double wb, double *u,
                                double *v)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= npts) return;
    double uu, vv;
    vel64<true>(rec + P.pitch + 1, nullptr, no_tile(), P, scheme, x[k], y[k], wa, wb, smode_of(wa, wb), uu, vv);
    u[k] = uu;
    v[k] = vv;
}

__global__ void interp32_kernel(StepParams P, const float4 *__restrict__ rec, int scheme,
                                int64_t npts, const double *__restrict__ x,
                                const double *__restrict__ y, double wa, double wb, double *u,
                                double *v)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= npts) return;
    int cx, cy;
    float ox, oy;
    split_of(x[k], P, cx, ox);
    split_of(y[k], P, cy, oy);
    float uu, vv;
    vel32<true>(rec + P.pitch + 1, nullptr, no_tile(), P, scheme, cx, cy, ox, oy, (float)wa, (float)wb,
                smode_of(wa, wb), uu, vv);
    u[k] = (double)uu * P.h;
    v[k] = (double)vv * P.h;
}

hipError_t launch_interp64(const StepParams &P, const Rec64 *rec, int scheme, int64_t npts,
                           const double *x, const double *y, double wa, double wb, double *u,
                           double *v, hipStream_t st)
{
    if (npts <= 0) return hipSuccess;
    const int b = 256;
    hipLaunchKernelGGL(interp64_kernel, dim3((unsigned)((npts + b - 1) / b)), dim3(b), 0, st, P,
                       rec, scheme, npts, x, y, wa, wb, u, v);
    return hipGetLastError();
}

hipError_t launch_interp32(const StepParams &P, const float4 *rec, int scheme, int64_t npts,
                           const double *x, const double *y, double wa, double wb, double *u,
                           double *v, hipStream_t st)
{
    if (npts <= 0) return hipSuccess;
    const int b = 256;
    hipLaunchKernelGGL(interp32_kernel, dim3((unsigned)((npts + b - 1) / b)), dim3(b), 0, st, P,
                       rec, scheme, npts, x, y, wa, wb, u, v);
    return hipGetLastError();
}

// ===========================================================================
// Readout in original particle order.
// ===========================================================================
__global__ void readout64_kernel(State64 S, const double2 *__restrict__ x0, int64_t offset,
                                 int64_t count, double *xw, double *yw, double *xu, double *yu,
                                 double *vx, double *vy)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int64_t p = offset + k;
    const uint32_t g = S.id[p];
    const int64_t q = (int64_t)g - offset;
    if (q < 0 || q >= count) return;
    const double2 x = S.pos[p];
    if (xw) xw[q] = x.x;
    if (yw) yw[q] = x.y;
    if (xu || yu) {
        const double2 d = S.disp[p];
        const double2 a = x0[g];
        if (xu) xu[q] = a.x + d.x;
        if (yu) yu[q] = a.y + d.y;
    }
    if (vx || vy) {
        const double2 w = S.vel[p];
        if (vx) vx[q] = w.x;
        if (vy) vy[q] = w.y;
    }
}

__global__ void readout32_kernel(StepParams P, State32 S, int64_t offset, int64_t count,
                                 double *xw, double *yw, double *xu, double *yu, double *vx,
                                 double *vy)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int64_t p = offset + k;
    const uint32_t g = S.id[p];
    const int64_t q = (int64_t)g - offset;
    if (q < 0 || q >= count) return;
    const int2 u = S.uc[p];
    const float2 o = S.off[p];
    if (xw) xw[q] = ((double)wrap_cell(u.x, P.n, P.mask) + (double)o.x) * P.h;
    if (yw) yw[q] = ((double)wrap_cell(u.y, P.n, P.mask) + (double)o.y) * P.h;
    if (xu || yu) {
        const double2 a = S.x0[g];
        const double2 d = split_disp(u, o, a, P);
        if (xu) xu[q] = a.x + d.x;
        if (yu) yu[q] = a.y + d.y;
    }
    if (vx || vy) {
        const float2 w = S.vel[p];
        if (vx) vx[q] = (double)w.x * P.h;
        if (vy) vy[q] = (double)w.y * P.h;
    }
}

// Readout out of cell order, in two passes.  Written straight from slot order,
// every output is a scatter of 8-byte words in id order (random after a
// re-sort), and each word costs a memory sector of its own per array, as does
// the gather of the initial position.  Here the first pass scatters each
// particle's whole 16- or 32-byte record (the two halves of the spare buffer's
// position pair taken as one array of records), one sector per particle; the
// second streams records, initial positions and outputs in id order.  Bound by
// the scatter's sectors.  Four positions of 2^24 sorted particles: FP32-split
// 2542 -> 401 us, FP64 2641 -> 874 us (a copy of the 0.8 and 1.3 GB that are
// read and written would take 130 and 210 us); velocities 545 -> 264 us.
struct alignas(32) Pair64 { double2 pos, disp; };
struct alignas(16) Pair32 { int2 uc; float2 off; };

template <typename Rec, typename A, typename B>
__global__ __launch_bounds__(256) void by_id_kernel(const A *__restrict__ a, const B *__restrict__ b,
                                                    const uint32_t *__restrict__ id,
                                                    int64_t offset, int64_t count, Rec *out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int64_t p = offset + k;
    const int64_t q = (int64_t)ld_stream(id + p) - offset;
    if (q < 0 || q >= count) return;
    out[q] = Rec{ld_stream(a + p), ld_stream(b + p)};
}

template <typename V>
__global__ __launch_bounds__(256) void vel_by_id_kernel(const V *__restrict__ v,
                                                        const uint32_t *__restrict__ id,
                                                        int64_t offset, int64_t count, V *out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int64_t p = offset + k;
    const int64_t q = (int64_t)ld_stream(id + p) - offset;
    if (q < 0 || q >= count) return;
    out[q] = ld_stream(v + p);
}

__device__ __forceinline__ void st_out(double *p, double v) { __builtin_nontemporal_store(v, p); }

__global__ __launch_bounds__(256) void readout_pairs64_kernel(const Pair64 *__restrict__ rec,
                                                              const double2 *__restrict__ x0,
                                                              int64_t count, double *xw,
                                                              double *yw, double *xu, double *yu)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= count) return;
    const Pair64 r = rec[q];
    if (xw) st_out(xw + q, r.pos.x);
    if (yw) st_out(yw + q, r.pos.y);
    if (xu || yu) {
        const double2 a = ld_stream(x0 + q);
        if (xu) st_out(xu + q, a.x + r.disp.x);
        if (yu) st_out(yu + q, a.y + r.disp.y);
    }
}

__global__ __launch_bounds__(256) void readout_pairs32_kernel(StepParams P,
                                                              const Pair32 *__restrict__ rec,
                                                              const double2 *__restrict__ x0,
                                                              int64_t count, double *xw,
                                                              double *yw, double *xu, double *yu)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= count) return;
    const Pair32 r = rec[q];
    if (xw) st_out(xw + q, ((double)wrap_cell(r.uc.x, P.n, P.mask) + (double)r.off.x) * P.h);
    if (yw) st_out(yw + q, ((double)wrap_cell(r.uc.y, P.n, P.mask) + (double)r.off.y) * P.h);
    if (xu || yu) {
        const double2 a = ld_stream(x0 + q);
        const double2 d = split_disp(r.uc, r.off, a, P);
        if (xu) st_out(xu + q, a.x + d.x);
        if (yu) st_out(yu + q, a.y + d.y);
    }
}

__global__ __launch_bounds__(256) void readout_vel_kernel(const double2 *v64, const float2 *v32,
                                                          double h, int64_t count, double *vx,
                                                          double *vy)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= count) return;
    double2 w;
    if (v64) {
        w = v64[q];
    } else {
        const float2 f = v32[q];
        w = make_double2((double)f.x * h, (double)f.y * h);
    }
    if (vx) st_out(vx + q, w.x);
    if (vy) st_out(vy + q, w.y);
}

// From this many particles on, a reordered species takes the two passes: below
// it the outputs stay in the caches, which merge the scattered words, and the
// second launch costs more than it saves.  One pass against two, FP64: positions
// of 2^17 particles 7.6 / 8.7 us, of 2^18 16.3 / 12.7 us in a loop but no gain
// behind a step (300 007 particles: 683 / 694 us with eight steps), of 2^20
// 68 / 47 us; velocities of 2^18 particles 7.4 / 8.4 us, of 2^20 30.2 / 28.7 us.
constexpr int64_t kTwoPassPositions = 1 << 19, kTwoPassVelocities = 1 << 20;

hipError_t launch_readout64(const State64 &S, const State64 &spare, const double2 *x0,
                            int64_t offset, int64_t count, bool reordered, double *xw, double *yw,
                            double *xu, double *yu, double *vx, double *vy, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const int b = 256;
    const dim3 g((unsigned)((count + b - 1) / b));
    const bool vel = vx || vy;
    if (!reordered || count < (vel ? kTwoPassVelocities : kTwoPassPositions)) {
        hipLaunchKernelGGL(readout64_kernel, g, dim3(b), 0, st, S, x0, offset, count, xw, yw, xu,
                           yu, vx, vy);
        return hipGetLastError();
    }
    if (xw || yw || xu || yu) {
        Pair64 *rec = reinterpret_cast<Pair64 *>(spare.pos);   // pos and disp, back to back
        hipLaunchKernelGGL((by_id_kernel<Pair64, double2, double2>), g, dim3(b), 0, st, S.pos,
                           S.disp, S.id, offset, count, rec);
        hipLaunchKernelGGL(readout_pairs64_kernel, g, dim3(b), 0, st, rec, x0 + offset, count, xw,
                           yw, xu, yu);
    }
    if (vel) {
        hipLaunchKernelGGL(vel_by_id_kernel<double2>, g, dim3(b), 0, st, S.vel, S.id, offset,
                           count, spare.vel);
        hipLaunchKernelGGL(readout_vel_kernel, g, dim3(b), 0, st, spare.vel,
                           (const float2 *)nullptr, 0.0, count, vx, vy);
    }
    return hipGetLastError();
}

hipError_t launch_readout32(const StepParams &P, const State32 &S, const State32 &spare,
                            int64_t offset, int64_t count, bool reordered, double *xw, double *yw,
                            double *xu, double *yu, double *vx, double *vy, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const int b = 256;
    const dim3 g((unsigned)((count + b - 1) / b));
    const bool vel = vx || vy;
    if (!reordered || count < (vel ? kTwoPassVelocities : kTwoPassPositions)) {
        hipLaunchKernelGGL(readout32_kernel, g, dim3(b), 0, st, P, S, offset, count, xw, yw, xu,
                           yu, vx, vy);
        return hipGetLastError();
    }
    if (xw || yw || xu || yu) {
        Pair32 *rec = reinterpret_cast<Pair32 *>(spare.uc);   // uc and off, back to back
        hipLaunchKernelGGL((by_id_kernel<Pair32, int2, float2>), g, dim3(b), 0, st, S.uc, S.off,
                           S.id, offset, count, rec);
        hipLaunchKernelGGL(readout_pairs32_kernel, g, dim3(b), 0, st, P, rec, S.x0 + offset, count,
                           xw, yw, xu, yu);
    }
    if (vel) {
        hipLaunchKernelGGL(vel_by_id_kernel<float2>, g, dim3(b), 0, st, S.vel, S.id, offset, count,
                           spare.vel);
        hipLaunchKernelGGL(readout_vel_kernel, g, dim3(b), 0, st, (const double2 *)nullptr,
                           spare.vel, P.h, count, vx, vy);
    }
    return hipGetLastError();
}

}  // namespace lpt
