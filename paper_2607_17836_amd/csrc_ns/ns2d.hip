// Eulerian field producer: pseudospectral vorticity-streamfunction solver of
// Sec. 3.1 on gfx950 (C ABI in ns2d.h).
//
// One step, with the grid fields (u, v, dw/dx, dw/dy) of the current level
// already resident:
//   1. product kernel: N = u dw/dx + v dw/dy on the grid (one pass over HBM);
//   2. hipFFT D2Z of N;
//   3. spectral kernel, one thread per half-plane mode: the 2/3 band, the
//      right-hand side -N - nu k^2 w (eq. spectral_vorticity_evolution), the
//      AB2 update (eq. ab2_fluid) with the previous right-hand side kept in
//      HBM, then the Poisson solve (eq. poisson_spectral) and the four
//      spectral fields i k_y psi, -i k_x psi (eq. spectral_velocity),
//      i k_x w, i k_y w (eq. spectral_vorticity_derivatives), pre-scaled by
//      1/n^2 so that the inverse transforms come out normalised;
//   4. one batched hipFFT Z2D of the four fields.
// Every pointwise operation lives in the two kernels, so each step reads and
// writes each spectral array once.
//
// For every power of two n from 64 to 4096 (the default) the built-in
// transforms (fft_lds.h) replace the library's (which stay available as an
// explicit cross-check, and for other n) and fuse with the pointwise work,
// over a transposed spectral layout (entry (row jy, column ix) of a
// half-plane spectrum at ix * n + jy, so that every column is contiguous)
// that holds only the columns inside the 2/3 band.  A step starts from the
// x-transformed advection term of the current level:
//   a. column_fwd_kernel: per band column, its transform along y, the band
//      and the AB2 update; column_emit_kernel: per band column and field,
//      the field's values and its inverse transform along y (up to n = 512
//      one kernel does both, column_step_kernel);
//   b. rows_kernel: per pair of grid rows, the four fields' inverse transforms
//      along x (two real rows packed into one complex transform, Hermitian
//      extension), their product u dw/dx + v dw/dy, and its forward transform
//      along x, unpacked into two half spectra: the next step's start.  The
//      grid holds the velocity only, written by a call's last step.
// The vorticity's gradient and the advection term never reach HBM on the grid.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <cmath>
#include <cstdio>
#include <new>
#include <string>
#include <vector>

#include "fft_lds.h"
#include "ns2d.h"

namespace {

constexpr int kBlock = 256;

struct Spec {
    int n, nh;        // grid side, half-plane width n/2 + 1
    double kscale;    // 2 pi / L
    double nu, dt;
    double inv_nn;    // 1 / n^2
    size_t plane;     // n * nh complex entries per spectral field
};

// Signed mode index of row j of a length-n transform (rows n/2 .. n-1 hold
// the negative modes).
__device__ __forceinline__ int signed_mode(int j, int n) { return j < n / 2 ? j : j - n; }

// 2/3 rule: a mode is kept when 3|m| < n on both axes.
__device__ __forceinline__ bool in_band(int mx, int my, int n)
{
    return 3 * abs(mx) < n && 3 * abs(my) < n;
}

// The four spectral fields of vorticity w at wavenumber (kx, ky), scaled by
// 1/n^2, into the four planes of `out`.
__device__ __forceinline__ void emit_fields(double2 *__restrict__ out, size_t idx, size_t plane,
                                            double kx, double ky, double2 w, double s)
{
    const double k2 = kx * kx + ky * ky;
    double2 p = make_double2(0.0, 0.0);
    if (k2 > 0.0) p = make_double2(w.x / k2, w.y / k2);
    // i a z = (-a z.y, a z.x)
    out[idx] = make_double2(-ky * p.y * s, ky * p.x * s);                  // u  =  i k_y psi
    out[idx + plane] = make_double2(kx * p.y * s, -kx * p.x * s);          // v  = -i k_x psi
    out[idx + 2 * plane] = make_double2(-kx * w.y * s, kx * w.x * s);      // dw/dx
    out[idx + 3 * plane] = make_double2(-ky * w.y * s, ky * w.x * s);      // dw/dy
}

__global__ __launch_bounds__(kBlock) void product_kernel(const double2 *__restrict__ u,
                                                         const double2 *__restrict__ v,
                                                         const double2 *__restrict__ wx,
                                                         const double2 *__restrict__ wy,
                                                         double2 *__restrict__ out, size_t count2)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count2; i += stride) {
        const double2 a = u[i], b = v[i], c = wx[i], d = wy[i];
        out[i] = make_double2(a.x * c.x + b.x * d.x, a.y * c.y + b.y * d.y);
    }
}

// After the forward transform of the initial vorticity: keep the band and
// emit the fields of that state.
__global__ __launch_bounds__(kBlock) void init_kernel(double2 *__restrict__ w_hat,
                                                      double2 *__restrict__ fields, Spec S)
{
    const int ix = blockIdx.x * kBlock + threadIdx.x, jy = blockIdx.y;
    if (ix >= S.nh) return;
    const size_t idx = (size_t)jy * S.nh + ix;
    const int my = signed_mode(jy, S.n);
    double2 w = w_hat[idx];
    if (!in_band(ix, my, S.n)) w = make_double2(0.0, 0.0);
    w_hat[idx] = w;
    emit_fields(fields, idx, S.plane, S.kscale * ix, S.kscale * my, w, S.inv_nn);
}

// One AB2 step in spectral space.  Plane 0 of `fields` holds the forward
// transform of the advection term on entry; all four planes are overwritten
// with the new level's fields (each thread reads its entry before writing).
template <bool FIRST>
__global__ __launch_bounds__(kBlock) void ab2_kernel(double2 *__restrict__ w_hat,
                                                     double2 *__restrict__ r_prev,
                                                     double2 *__restrict__ fields, Spec S)
{
    const int ix = blockIdx.x * kBlock + threadIdx.x, jy = blockIdx.y;
    if (ix >= S.nh) return;
    const size_t idx = (size_t)jy * S.nh + ix;
    const int my = signed_mode(jy, S.n);
    const double kx = S.kscale * ix, ky = S.kscale * my;
    const double k2 = kx * kx + ky * ky;
    const double2 w = w_hat[idx];
    double2 N = fields[idx];
    if (!in_band(ix, my, S.n)) N = make_double2(0.0, 0.0);
    const double visc = S.nu * k2;
    const double2 r = make_double2(-N.x - visc * w.x, -N.y - visc * w.y);
    const double2 r_old = FIRST ? r : r_prev[idx];
    const double2 wn = make_double2(w.x + S.dt * (1.5 * r.x - 0.5 * r_old.x),
                                    w.y + S.dt * (1.5 * r.y - 0.5 * r_old.y));
    w_hat[idx] = wn;
    r_prev[idx] = r;
    emit_fields(fields, idx, S.plane, kx, ky, wn, S.inv_nn);
}

// omega_hat / n^2 (which = 0) or psi_hat / n^2 (which = 1) into one plane.
__global__ __launch_bounds__(kBlock) void scaled_kernel(const double2 *__restrict__ w_hat,
                                                        double2 *__restrict__ out, Spec S,
                                                        int which)
{
    const int ix = blockIdx.x * kBlock + threadIdx.x, jy = blockIdx.y;
    if (ix >= S.nh) return;
    const size_t idx = (size_t)jy * S.nh + ix;
    const int my = signed_mode(jy, S.n);
    const double kx = S.kscale * ix, ky = S.kscale * my;
    const double k2 = kx * kx + ky * ky;
    double2 w = w_hat[idx];
    if (which == 1) w = k2 > 0.0 ? make_double2(w.x / k2, w.y / k2) : make_double2(0.0, 0.0);
    out[idx] = make_double2(w.x * S.inv_nn, w.y * S.inv_nn);
}

// ---- built-in transform path (n = 64, 128, ..., 4096) ---------------------

// Contiguous logical block ranges per XCD (workgroups go to the eight XCDs
// round-robin): XCD x = b mod 8 takes logical blocks [x G/8, (x+1) G/8) up to
// the remainder, so consecutive logical blocks share an L2.
__device__ __forceinline__ int xcd_block(int b, int G)
{
    const int x = b % 8, k = b / 8, q = G / 8, r = G % 8;
    return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

// Columns ix = 0 .. band_cols(N) - 1 are the ones with 3 ix < N.  Every other
// column of the band-limited state, of the four fields and of the read-back
// fields is zero, so the built-in path neither transforms nor stores it:
// the row passes skip it and the inverse row pass supplies the zeros.
constexpr int band_cols(int N) { return (N - 1) / 3 + 1; }

// Columns of the band a thread of a row pass takes: k = t + c N / 8.
template <int N>
constexpr int cols_per_thread() { return (band_cols(N) + N / 8 - 1) / (N / 8); }

// Two grid rows a, b transformed along x as z = a + i b (v[q] is point t + q N
// / 8), unpacked into their half spectra A(k) = (Z(k) + conj Z(-k)) / 2,
// B(k) = (Z(k) - conj Z(-k)) / (2i) at rows jy0 and jy0 + 1 of specT.
template <int N, bool BLOCK = true>
__device__ __forceinline__ void rows_forward(double2 v[8], int t, double2 *buf,
                                             double2 *__restrict__ specT, int jy0,
                                             const double2 *__restrict__ W)
{
    constexpr int T = N / 8, KB = band_cols(N);
    ns_fft::fft<N, false, BLOCK>(v, t, buf, W);
    ns_fft::sync<BLOCK>();
#pragma unroll
    for (int q = 0; q < 8; ++q) buf[ns_fft::pad(t) + q * ns_fft::padded(T)] = v[q];
    ns_fft::sync<BLOCK>();
#pragma unroll
    for (int c = 0; c < cols_per_thread<N>(); ++c) {
        const int k = t + c * T;
        if (k >= KB) break;
        // entry -k is N - k, and entry 0 for k = 0
        const double2 z = buf[ns_fft::pad(t) + c * ns_fft::padded(T)];
        const double2 zc = k == 0 ? z : buf[ns_fft::pad(N - t) - c * ns_fft::padded(T)];
        double2 *dst = specT + (size_t)k * N + jy0;
        dst[0] = make_double2(0.5 * (z.x + zc.x), 0.5 * (z.y - zc.y));
        dst[1] = make_double2(0.5 * (z.y + zc.y), -0.5 * (z.x - zc.x));
    }
}

// Rows jy0 and jy0 + 1 of one field (a plane of the transposed spectra, already
// transformed along y) back to the grid: Z(k) = A(k) + i B(k) and Z(N-k) =
// conj A(k) + i conj B(k) for the band columns (the imaginary parts at k = 0
// dropped as in any complex-to-real transform), zero elsewhere; z = IFFT(Z)
// has a = Re z, b = Im z, v[q] at point t + q N / 8.
template <int N, bool BLOCK = true>
__device__ __forceinline__ void rows_inverse(double2 v[8], int t, double2 *buf,
                                             const double2 *__restrict__ field, int jy0,
                                             const double2 *__restrict__ W)
{
    constexpr int T = N / 8, KB = band_cols(N), C = cols_per_thread<N>();
    field += ns_fft::opaque_zero();
    double2 A[C], B[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int k = t + c * T;
        A[c] = B[c] = make_double2(0.0, 0.0);
        if (k < KB) {
            const double2 *sp = field + (size_t)k * N + jy0;
            A[c] = sp[0];
            B[c] = sp[1];
        }
    }
    ns_fft::sync<BLOCK>();   // the buffer's last readers are done
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int k = t + c * T;
        if (k >= KB) break;
        if (k == 0) A[c].y = B[c].y = 0.0;
        buf[ns_fft::pad(t) + c * ns_fft::padded(T)] =
            make_double2(A[c].x - B[c].y, A[c].y + B[c].x);
        if (k > 0)
            buf[ns_fft::pad(N - t) - c * ns_fft::padded(T)] =
                make_double2(A[c].x + B[c].y, B[c].x - A[c].y);
    }
    ns_fft::sync<BLOCK>();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = t + q * T;
        v[q] = i >= KB && i <= N - KB ? make_double2(0.0, 0.0)
                                      : buf[ns_fft::pad(t) + q * ns_fft::padded(T)];
    }
    ns_fft::fft<N, true, BLOCK>(v, t, buf, W);
    ns_fft::settle(v);
}

template <int N>
__device__ __forceinline__ void store_rows(const double2 v[8], int t, double *__restrict__ grid,
                                           int jy0)
{
    constexpr int T = N / 8;
    double *ra = grid + (size_t)jy0 * N + t;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        ra[q * T] = v[q].x;
        ra[q * T + N] = v[q].y;
    }
}

// The x-transform of one grid field g.  Blocks take pairs of rows in XCD order
// (the four pairs that share each 128-byte line of a transposed column run on
// one XCD and share its L2), as in the row passes below.
template <int N>
__global__ __launch_bounds__(N / 8) void fwd_rows_kernel(const double *__restrict__ g,
                                                        double2 *__restrict__ specT,
                                                        const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_rows[];
    constexpr int T = N / 8;
    const int jy0 = 2 * xcd_block(blockIdx.x, N / 2);
    const double *ra = g + (size_t)jy0 * N;
    double2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
        v[q] = make_double2(ra[threadIdx.x + q * T], ra[threadIdx.x + q * T + N]);
    rows_forward<N>(v, threadIdx.x, lds_rows, specT, jy0, W);
}

// One field back to the grid (read-back of omega or psi).
template <int N>
__global__ __launch_bounds__(N / 8) void inv_rows_kernel(const double2 *__restrict__ field,
                                                        double *__restrict__ grid,
                                                        const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_rows[];
    const int jy0 = 2 * xcd_block(blockIdx.x, N / 2);
    double2 v[8];
    rows_inverse<N>(v, threadIdx.x, lds_rows, field, jy0, W);
    store_rows<N>(v, threadIdx.x, grid, jy0);
}

// One pair of rows from the four fields' column transforms to the x-transform
// of the advection term u dw/dx + v dw/dy.  STORE: the velocity goes to the
// grid too (u, then v).  Bound by the latency of its five transforms in a row,
// so by the waves resident: registers are held to four per SIMD (124; see
// opaque_zero and settle), which at N = 2048 makes all 1024 blocks resident at
// once.
template <int N, bool STORE>
__global__ __launch_bounds__(N / 8) __attribute__((amdgpu_waves_per_eu(4, 4)))
void rows_kernel(const double2 *__restrict__ fields, size_t plane, double *__restrict__ grid,
                 double2 *__restrict__ specT, const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_rows[];
    constexpr size_t cells = (size_t)N * N;
    const int jy0 = 2 * xcd_block(blockIdx.x, N / 2), t = threadIdx.x;
    double2 a[8], b[8], p[8];
    rows_inverse<N>(a, t, lds_rows, fields, jy0, W);               // u
    if (STORE) store_rows<N>(a, t, grid, jy0);
    rows_inverse<N>(b, t, lds_rows, fields + 2 * plane, jy0, W);   // dw/dx
#pragma unroll
    for (int q = 0; q < 8; ++q) p[q] = make_double2(a[q].x * b[q].x, a[q].y * b[q].y);
    ns_fft::settle(p);
    rows_inverse<N>(a, t, lds_rows, fields + plane, jy0, W);       // v
    if (STORE) store_rows<N>(a, t, grid + cells, jy0);
    rows_inverse<N>(b, t, lds_rows, fields + 3 * plane, jy0, W);   // dw/dy
#pragma unroll
    for (int q = 0; q < 8; ++q)
        p[q] = make_double2(fma(a[q].x, b[q].x, p[q].x), fma(a[q].y, b[q].y, p[q].y));
    rows_forward<N>(p, t, lds_rows, specT, jy0, W);
}

// rows_kernel for small grids, whose few blocks leave the chip idle: the four
// fields' transforms side by side, by four groups of N / 8 threads each inside
// one wave, then the product and its transform by the first group.  Two
// transforms in a row instead of five, without barriers.
template <int N, bool STORE>
__global__ __launch_bounds__(N / 2) void rows_small_kernel(const double2 *__restrict__ fields,
                                                          size_t plane, double *__restrict__ grid,
                                                          double2 *__restrict__ specT,
                                                          const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_rows[];   // a buffer per field
    constexpr int T = N / 8, E = ns_fft::lds_entries<N>();
    const int jy0 = 2 * xcd_block(blockIdx.x, N / 2);
    const int f = threadIdx.x / T, t = threadIdx.x % T;
    double2 *buf = lds_rows + f * E;
    double2 v[8];
    rows_inverse<N, false>(v, t, buf, fields + f * plane, jy0, W);
    if (STORE && f < 2) store_rows<N>(v, t, grid + f * ((size_t)N * N), jy0);
    ns_fft::sync<false>();
#pragma unroll
    for (int q = 0; q < 8; ++q) buf[ns_fft::pad(t) + q * ns_fft::padded(T)] = v[q];
    __syncthreads();
    if (f > 0) return;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const double2 *b = buf + ns_fft::pad(t) + q * ns_fft::padded(T);
        const double2 y = b[E], wx = b[2 * E], wy = b[3 * E];
        v[q] = make_double2(fma(y.x, wy.x, v[q].x * wx.x), fma(y.y, wy.y, v[q].y * wx.y));
    }
    rows_forward<N, false>(v, t, buf, specT, jy0, W);
}

enum ColumnMode { kColInit = 0, kColFirst = 1, kColStep = 2 };

// The new state of one mode from the transform Nh of the advection term: the
// band, the right-hand side and AB2 (MODE init: Nh is the vorticity).
template <int N, int MODE>
__device__ __forceinline__ void advance_mode(double2 Nh, int ix, int jy, const Spec &S,
                                             const double2 *w_hat, const double2 *r_prev,
                                             size_t idx, double2 &w_new, double2 &r)
{
    const int my = signed_mode(jy, N);
    if (!in_band(ix, my, N)) Nh = make_double2(0.0, 0.0);
    if constexpr (MODE == kColInit) {
        w_new = Nh;
        r = make_double2(0.0, 0.0);
    } else {
        const double kx = S.kscale * ix, ky = S.kscale * my;
        const double visc = S.nu * (kx * kx + ky * ky);
        const double2 w = w_hat[idx];
        r = make_double2(-Nh.x - visc * w.x, -Nh.y - visc * w.y);
        const double2 r_old = MODE == kColFirst ? r : r_prev[idx];
        w_new = make_double2(w.x + S.dt * (1.5 * r.x - 0.5 * r_old.x),
                             w.y + S.dt * (1.5 * r.y - 0.5 * r_old.y));
    }
}

// Value of one field at one mode of vorticity w, scaled by 1/n^2: u = i k_y
// psi, v = -i k_x psi, dw/dx = i k_x w, dw/dy = i k_y w, or omega or psi.
enum Field { kU = 0, kV = 1, kWx = 2, kWy = 3, kOmega = 4, kPsi = 5 };

__device__ __forceinline__ double2 field_mode(int f, double2 w, double kx, double ky, double s)
{
    if (f == kU || f == kV || f == kPsi) {
        const double k2 = kx * kx + ky * ky;
        double2 p = make_double2(0.0, 0.0);
        if (k2 > 0.0) p = make_double2(w.x / k2, w.y / k2);
        if (f == kU) return make_double2(-ky * p.y * s, ky * p.x * s);
        if (f == kV) return make_double2(kx * p.y * s, -kx * p.x * s);
        return make_double2(p.x * s, p.y * s);
    }
    if (f == kWx) return make_double2(-kx * w.y * s, kx * w.x * s);
    if (f == kWy) return make_double2(-ky * w.y * s, ky * w.x * s);
    return make_double2(w.x * s, w.y * s);
}

// Column ix < band_cols(N) of the transposed spectra, one block per column:
// the x-transformed rows at specT transformed along y, the band taken, and
// the state stored (init) or advanced by AB2 (step).
template <int N, int MODE>
__global__ __launch_bounds__(N / 8) void column_fwd_kernel(double2 *__restrict__ w_hat,
                                                          double2 *__restrict__ r_prev,
                                                          const double2 *__restrict__ specT,
                                                          Spec S, const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_col[];
    constexpr int T = N / 8;
    const int ix = blockIdx.x, t = threadIdx.x;
    const size_t col = (size_t)ix * N;
    double2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = specT[col + t + q * T];
    ns_fft::fft<N, false>(v, t, lds_col, W);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const size_t idx = col + t + q * T;
        double2 w, r;
        advance_mode<N, MODE>(v[q], ix, t + q * T, S, w_hat, r_prev, idx, w, r);
        w_hat[idx] = w;
        if (MODE != kColInit) r_prev[idx] = r;
    }
}

// One field of one band column, transformed back along y: the four fields
// (nf = 4, plane f each) or one (nf = 1).  Logical block l = column * nf +
// field, so a column's fields run on one XCD and re-read its state from that
// L2.
template <int N>
__global__ __launch_bounds__(N / 8) void column_emit_kernel(const double2 *__restrict__ w_hat,
                                                           double2 *__restrict__ fields, int f0,
                                                           int nf, Spec S,
                                                           const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_col[];
    constexpr int T = N / 8;
    const int l = xcd_block(blockIdx.x, band_cols(N) * nf);
    const int ix = l / nf, f = l % nf, t = threadIdx.x;
    const size_t col = (size_t)ix * N;
    double2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = w_hat[col + t + q * T];
#pragma unroll
    for (int q = 0; q < 8; ++q)
        v[q] = field_mode(f0 + f, v[q], S.kscale * ix, S.kscale * signed_mode(t + q * T, N),
                          S.inv_nn);
    ns_fft::fft<N, true>(v, t, lds_col, W);
    double2 *dst = fields + (size_t)f * S.plane + col;
#pragma unroll
    for (int q = 0; q < 8; ++q) dst[t + q * T] = v[q];
}

// column_fwd_kernel and column_emit_kernel of a step in one, for small grids:
// four groups of N / 8 threads each advance the column's state and take one
// field back along y.  The state stays where it is (a captured step can be
// replayed): the first group stores it once all have read it.  One launch and
// one trip through memory less for three more transforms of a column.
template <int N, int MODE>
__global__ __launch_bounds__(N / 2) void column_step_kernel(double2 *w_hat, double2 *r_prev,
                                                           const double2 *__restrict__ specT,
                                                           double2 *__restrict__ fields, Spec S,
                                                           const double2 *__restrict__ W)
{
    extern __shared__ double2 lds_col[];   // a buffer per field
    constexpr int T = N / 8;
    const int ix = blockIdx.x, f = threadIdx.x / T, t = threadIdx.x % T;
    const size_t col = (size_t)ix * N;
    double2 *buf = lds_col + f * ns_fft::lds_entries<N>();
    double2 v[8], w[8], r[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = specT[col + t + q * T];
    ns_fft::fft<N, false, false>(v, t, buf, W);
#pragma unroll
    for (int q = 0; q < 8; ++q)
        advance_mode<N, MODE>(v[q], ix, t + q * T, S, w_hat, r_prev, col + t + q * T, w[q], r[q]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int jy = t + q * T;
        if (f == 0) {
            w_hat[col + jy] = w[q];
            r_prev[col + jy] = r[q];
        }
        v[q] = field_mode(f, w[q], S.kscale * ix, S.kscale * signed_mode(jy, N), S.inv_nn);
    }
    ns_fft::fft<N, true, false>(v, t, buf, W);
    double2 *dst = fields + (size_t)f * S.plane + col;
#pragma unroll
    for (int q = 0; q < 8; ++q) dst[t + q * T] = v[q];
}

// Grids up to kSmallGrid take rows_small_kernel and column_step_kernel (whose
// groups of N / 8 threads have to stay inside a wave).  Us a step with the
// general kernels and with these: n = 64 12.6 / 9.4, 256 15.4 /
// 11.0, 512 24 / 15.4.
constexpr int kSmallGrid = 512;

template <int N>
void launch_rows(bool store, const double2 *fields, size_t plane, double *grid, double2 *adv,
                 const double2 *W, hipStream_t st)
{
    const size_t lds = (size_t)ns_fft::lds_entries<N>() * sizeof(double2);
    if constexpr (N <= kSmallGrid) {
        if (store)
            rows_small_kernel<N, true><<<N / 2, N / 2, 4 * lds, st>>>(fields, plane, grid, adv, W);
        else
            rows_small_kernel<N, false><<<N / 2, N / 2, 4 * lds, st>>>(fields, plane, grid, adv, W);
    } else {
        if (store)
            rows_kernel<N, true><<<N / 2, N / 8, lds, st>>>(fields, plane, grid, adv, W);
        else
            rows_kernel<N, false><<<N / 2, N / 8, lds, st>>>(fields, plane, grid, adv, W);
    }
}

}  // namespace

struct ns2d_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int n = 0, nh = 0;
    double L = 0, nu = 0, dt = 0;
    double2 *spectra = nullptr;   // one allocation: the spectral planes that follow
    double2 *w_hat = nullptr, *r_prev = nullptr, *fields = nullptr;   // fields: 4 planes
    double *grid = nullptr;   // 4 grid fields: u, v, dw/dx, dw/dy (built-in path: u, v and,
                              // in place of the others, the x-transformed advection term)
    double *tmp = nullptr;    // grid scratch: advection term, read-back transforms
    hipfftHandle r2c = 0, c2r4 = 0, c2r1 = 0;
    bool r2c_ok = false, c2r4_ok = false, c2r1_ok = false;
    bool builtin = false;        // built-in transforms, transposed spectral layout
    double2 *twiddle = nullptr;  // the passes' twiddles (built-in path, see fft_lds.h)
    bool have_state = false, first = true;
    int64_t steps = 0;
    std::string err;
};

namespace {

ns2d_status fail(ns2d_ctx *c, ns2d_status s, const std::string &msg)
{
    if (c) c->err = msg;
    return s;
}

#define NS_HIP(c, expr)                                                                  \
    do {                                                                                 \
        hipError_t e_ = (expr);                                                          \
        if (e_ != hipSuccess)                                                            \
            return fail((c), NS2D_E_HIP, std::string(#expr ": ") + hipGetErrorString(e_)); \
    } while (0)

#define NS_FFT(c, expr)                                                                  \
    do {                                                                                 \
        hipfftResult r_ = (expr);                                                        \
        if (r_ != HIPFFT_SUCCESS)                                                        \
            return fail((c), NS2D_E_FFT, std::string(#expr " failed, hipfftResult ") +     \
                                             std::to_string((int)r_));                   \
    } while (0)

Spec make_spec(const ns2d_ctx *c)
{
    Spec S;
    S.n = c->n;
    S.nh = c->nh;
    S.kscale = 2.0 * M_PI / c->L;
    S.nu = c->nu;
    S.dt = c->dt;
    S.inv_nn = 1.0 / ((double)c->n * (double)c->n);
    S.plane = (size_t)c->n * c->nh;
    return S;
}

dim3 spectral_grid(const ns2d_ctx *c) { return dim3((c->nh + kBlock - 1) / kBlock, c->n); }

void release(ns2d_ctx *c)
{
    if (c->r2c_ok) hipfftDestroy(c->r2c);
    if (c->c2r4_ok) hipfftDestroy(c->c2r4);
    if (c->c2r1_ok) hipfftDestroy(c->c2r1);
    if (c->spectra) (void)hipFree(c->spectra);
    if (c->grid) (void)hipFree(c->grid);
    if (c->tmp) (void)hipFree(c->tmp);
    if (c->twiddle) (void)hipFree(c->twiddle);
}

// kOpStep: a step whose velocity nobody reads (not the last of a call)
enum BuiltinOp { kOpInit, kOpStep, kOpLastStep, kOpReadW, kOpReadPsi };

template <int N>
ns2d_status run_builtin_n(ns2d_ctx *c, BuiltinOp op)
{
    constexpr int T = N / 8;
    const size_t lds = (size_t)ns_fft::lds_entries<N>() * sizeof(double2);
    const dim3 rows(N / 2), cols(band_cols(N)), cols4(4 * band_cols(N));
    const Spec S = make_spec(c);
    hipStream_t st = c->stream;
    const double2 *Wt = c->twiddle;
    double2 *adv = reinterpret_cast<double2 *>(c->grid + 2 * (size_t)N * N);
    switch (op) {
    case kOpInit:
        fwd_rows_kernel<N><<<rows, T, lds, st>>>(c->tmp, adv, Wt);
        column_fwd_kernel<N, kColInit><<<cols, T, lds, st>>>(c->w_hat, c->r_prev, adv, S, Wt);
        column_emit_kernel<N><<<cols4, T, lds, st>>>(c->w_hat, c->fields, kU, 4, S, Wt);
        launch_rows<N>(true, c->fields, S.plane, c->grid, adv, Wt, st);
        break;
    case kOpStep:
    case kOpLastStep:
        if constexpr (N <= kSmallGrid) {
            if (c->first)
                column_step_kernel<N, kColFirst><<<cols, 4 * T, 4 * lds, st>>>(
                    c->w_hat, c->r_prev, adv, c->fields, S, Wt);
            else
                column_step_kernel<N, kColStep><<<cols, 4 * T, 4 * lds, st>>>(
                    c->w_hat, c->r_prev, adv, c->fields, S, Wt);
        } else {
            if (c->first)
                column_fwd_kernel<N, kColFirst><<<cols, T, lds, st>>>(c->w_hat, c->r_prev, adv, S, Wt);
            else
                column_fwd_kernel<N, kColStep><<<cols, T, lds, st>>>(c->w_hat, c->r_prev, adv, S, Wt);
            column_emit_kernel<N><<<cols4, T, lds, st>>>(c->w_hat, c->fields, kU, 4, S, Wt);
        }
        launch_rows<N>(op == kOpLastStep, c->fields, S.plane, c->grid, adv, Wt, st);
        break;
    case kOpReadW:
    case kOpReadPsi:
        column_emit_kernel<N><<<cols, T, lds, st>>>(c->w_hat, c->fields,
                                                    op == kOpReadW ? kOmega : kPsi, 1, S, Wt);
        inv_rows_kernel<N><<<rows, T, lds, st>>>(c->fields, c->tmp, Wt);
        break;
    }
    NS_HIP(c, hipGetLastError());
    return NS2D_OK;
}

ns2d_status run_builtin(ns2d_ctx *c, BuiltinOp op)
{
    switch (c->n) {
    case 64: return run_builtin_n<64>(c, op);
    case 128: return run_builtin_n<128>(c, op);
    case 256: return run_builtin_n<256>(c, op);
    case 512: return run_builtin_n<512>(c, op);
    case 1024: return run_builtin_n<1024>(c, op);
    case 2048: return run_builtin_n<2048>(c, op);
    case 4096: return run_builtin_n<4096>(c, op);
    default: return fail(c, NS2D_E_STATE, "no built-in transform for this n");
    }
}

// The four spectral planes to the four grid fields.
ns2d_status to_grid4(ns2d_ctx *c)
{
    NS_FFT(c, hipfftExecZ2D(c->c2r4, reinterpret_cast<hipfftDoubleComplex *>(c->fields), c->grid));
    return NS2D_OK;
}

ns2d_status copy_out(ns2d_ctx *c, double *dst, const double *src, int32_t on_device)
{
    const size_t bytes = (size_t)c->n * c->n * sizeof(double);
    NS_HIP(c, hipMemcpyAsync(dst, src, bytes, on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                             c->stream));
    return NS2D_OK;
}

}  // namespace

extern "C" {

ns2d_status ns2d_create(const ns2d_config *cfg, ns2d_ctx **out)
{
    if (!cfg || !out) return NS2D_E_ARG;
    *out = nullptr;
    const int n = cfg->n;
    const double L = cfg->length == 0.0 ? 2.0 * M_PI : cfg->length;
    if (n < 8 || n > 16384 || (n & 1)) return NS2D_E_ARG;
    if (!(L > 0.0) || !std::isfinite(L)) return NS2D_E_ARG;
    if (!(cfg->nu >= 0.0) || !std::isfinite(cfg->nu)) return NS2D_E_ARG;
    if (!(cfg->dt > 0.0) || !std::isfinite(cfg->dt)) return NS2D_E_ARG;
    if (cfg->transforms < 0 || cfg->transforms > 2) return NS2D_E_ARG;
    // the built-in transforms (transforms 0 or 2) exist for powers of two
    // from 64 to 4096; hipFFT only on request (transforms 1)
    const bool own = cfg->transforms != 1;
    if (own && (n < 64 || n > 4096 || (n & (n - 1)))) return NS2D_E_ARG;
    ns2d_ctx *c = new (std::nothrow) ns2d_ctx;
    if (!c) return NS2D_E_NOMEM;
    c->n = n;
    c->nh = n / 2 + 1;
    c->L = L;
    c->nu = cfg->nu;
    c->dt = cfg->dt;
    c->stream = reinterpret_cast<hipStream_t>(cfg->hip_stream);
    auto bail = [&](ns2d_status s) {
        release(c);
        delete c;
        return s;
    };
    if (hipGetDevice(&c->device) != hipSuccess) return bail(NS2D_E_HIP);
    const size_t plane = (size_t)n * c->nh, cells = (size_t)n * n;
    if (hipMalloc(&c->spectra, 6 * plane * sizeof(double2)) != hipSuccess ||
        hipMalloc(&c->grid, 4 * cells * sizeof(double)) != hipSuccess ||
        hipMalloc(&c->tmp, cells * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        return bail(NS2D_E_NOMEM);
    }
    c->fields = c->spectra;
    c->w_hat = c->spectra + 4 * plane;
    c->r_prev = c->spectra + 5 * plane;
    // measured faster than hipFFT at the sizes compared (2048^2: 98 vs 337
    // us a step; 1024^2: 39 vs 101; 512^2: 16 vs 43)
    c->builtin = own;
    if (c->builtin) {
        // twiddles from the long-double cosine and sine, rounded once
        std::vector<double2> w((size_t)ns_fft::table_entries(n));
        size_t e = 0;
        for (int ns = 8; ns < n; ns *= 8) {
            const int R = n / ns >= 8 ? 8 : n / ns;
            for (int r = 1; r < R; ++r)
                for (int k = 0; k < ns; ++k) {
                    const long long m = (long long)r * k * (n / (ns * R));
                    const long double a = 2.0L * 3.14159265358979323846264338327950288L * m / n;
                    w[e++] = make_double2((double)cosl(a), (double)-sinl(a));
                }
        }
        if (hipMalloc(&c->twiddle, w.size() * sizeof(double2)) != hipSuccess) {
            (void)hipGetLastError();
            return bail(NS2D_E_NOMEM);
        }
        if (hipMemcpy(c->twiddle, w.data(), w.size() * sizeof(double2), hipMemcpyHostToDevice) !=
            hipSuccess)
            return bail(NS2D_E_HIP);
        *out = c;
        return NS2D_OK;
    }
    int dims[2] = {n, n};
    if (hipfftPlan2d(&c->r2c, n, n, HIPFFT_D2Z) != HIPFFT_SUCCESS) return bail(NS2D_E_FFT);
    c->r2c_ok = true;
    if (hipfftPlanMany(&c->c2r4, 2, dims, nullptr, 1, 0, nullptr, 1, 0, HIPFFT_Z2D, 4) != HIPFFT_SUCCESS)
        return bail(NS2D_E_FFT);
    c->c2r4_ok = true;
    if (hipfftPlan2d(&c->c2r1, n, n, HIPFFT_Z2D) != HIPFFT_SUCCESS) return bail(NS2D_E_FFT);
    c->c2r1_ok = true;
    if (hipfftSetStream(c->r2c, c->stream) != HIPFFT_SUCCESS ||
        hipfftSetStream(c->c2r4, c->stream) != HIPFFT_SUCCESS ||
        hipfftSetStream(c->c2r1, c->stream) != HIPFFT_SUCCESS)
        return bail(NS2D_E_FFT);
    *out = c;
    return NS2D_OK;
}

void ns2d_destroy(ns2d_ctx *ctx)
{
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    (void)hipStreamSynchronize(ctx->stream);
    release(ctx);
    delete ctx;
}

const char *ns2d_last_error(const ns2d_ctx *ctx) { return ctx ? ctx->err.c_str() : "null context"; }

ns2d_status ns2d_synchronize(ns2d_ctx *c)
{
    if (!c) return NS2D_E_ARG;
    NS_HIP(c, hipSetDevice(c->device));
    NS_HIP(c, hipStreamSynchronize(c->stream));
    return NS2D_OK;
}

ns2d_status ns2d_set_vorticity(ns2d_ctx *c, const double *omega, int32_t on_device)
{
    if (!c) return NS2D_E_ARG;
    if (!omega) return fail(c, NS2D_E_ARG, "omega is NULL");
    if (on_device != 0 && on_device != 1) return fail(c, NS2D_E_ARG, "on_device is 0 or 1");
    NS_HIP(c, hipSetDevice(c->device));
    const size_t bytes = (size_t)c->n * c->n * sizeof(double);
    NS_HIP(c, hipMemcpyAsync(c->tmp, omega, bytes, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                             c->stream));
    if (c->builtin) {
        const ns2d_status st = run_builtin(c, kOpInit);
        if (st != NS2D_OK) return st;
    } else {
        NS_FFT(c, hipfftExecD2Z(c->r2c, c->tmp, reinterpret_cast<hipfftDoubleComplex *>(c->w_hat)));
        const Spec S = make_spec(c);
        init_kernel<<<spectral_grid(c), kBlock, 0, c->stream>>>(c->w_hat, c->fields, S);
        NS_HIP(c, hipGetLastError());
        const ns2d_status st = to_grid4(c);
        if (st != NS2D_OK) return st;
    }
    if (!on_device) NS_HIP(c, hipStreamSynchronize(c->stream));   // host buffer read before return
    c->have_state = true;
    c->first = true;
    c->steps = 0;
    return NS2D_OK;
}

ns2d_status ns2d_step(ns2d_ctx *c, int32_t count)
{
    if (!c) return NS2D_E_ARG;
    if (count < 0) return fail(c, NS2D_E_ARG, "count must be >= 0");
    if (!c->have_state) return fail(c, NS2D_E_STATE, "ns2d_set_vorticity has not been called");
    NS_HIP(c, hipSetDevice(c->device));
    const Spec S = make_spec(c);
    const size_t cells = (size_t)c->n * c->n, count2 = cells / 2;
    const double2 *g = reinterpret_cast<const double2 *>(c->grid);
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device);
    const size_t want = (count2 + kBlock - 1) / kBlock;
    const unsigned pgrid = (unsigned)(want < (size_t)cus * 16 ? want : (size_t)cus * 16);
    if (c->builtin) {
        for (int32_t s = 0; s < count; ++s) {
            const ns2d_status st = run_builtin(c, s + 1 < count ? kOpStep : kOpLastStep);
            if (st != NS2D_OK) return st;
            c->first = false;
            ++c->steps;
        }
        return NS2D_OK;
    }
    for (int32_t s = 0; s < count; ++s) {
        product_kernel<<<pgrid, kBlock, 0, c->stream>>>(g, g + count2, g + 2 * count2, g + 3 * count2,
                                                        reinterpret_cast<double2 *>(c->tmp), count2);
        NS_HIP(c, hipGetLastError());
        NS_FFT(c, hipfftExecD2Z(c->r2c, c->tmp, reinterpret_cast<hipfftDoubleComplex *>(c->fields)));
        if (c->first)
            ab2_kernel<true><<<spectral_grid(c), kBlock, 0, c->stream>>>(c->w_hat, c->r_prev, c->fields, S);
        else
            ab2_kernel<false><<<spectral_grid(c), kBlock, 0, c->stream>>>(c->w_hat, c->r_prev, c->fields, S);
        NS_HIP(c, hipGetLastError());
        const ns2d_status st = to_grid4(c);
        if (st != NS2D_OK) return st;
        c->first = false;
        ++c->steps;
    }
    return NS2D_OK;
}

ns2d_status ns2d_velocity(ns2d_ctx *c, const double **u, const double **v)
{
    if (!c) return NS2D_E_ARG;
    if (!u || !v) return fail(c, NS2D_E_ARG, "u and v must not be NULL");
    if (!c->have_state) return fail(c, NS2D_E_STATE, "ns2d_set_vorticity has not been called");
    const size_t cells = (size_t)c->n * c->n;
    *u = c->grid;
    *v = c->grid + cells;
    return NS2D_OK;
}

ns2d_status ns2d_get_fields(ns2d_ctx *c, double *u, double *v, double *omega, double *psi,
                            int32_t on_device)
{
    if (!c) return NS2D_E_ARG;
    if (on_device != 0 && on_device != 1) return fail(c, NS2D_E_ARG, "on_device is 0 or 1");
    if (!c->have_state) return fail(c, NS2D_E_STATE, "ns2d_set_vorticity has not been called");
    NS_HIP(c, hipSetDevice(c->device));
    const size_t cells = (size_t)c->n * c->n;
    ns2d_status st;
    if (u && (st = copy_out(c, u, c->grid, on_device)) != NS2D_OK) return st;
    if (v && (st = copy_out(c, v, c->grid + cells, on_device)) != NS2D_OK) return st;
    const Spec S = make_spec(c);
    double *outs[2] = {omega, psi};
    for (int which = 0; which < 2; ++which) {
        if (!outs[which]) continue;
        // plane 0 of the spectral fields is free between steps (the next step
        // rewrites it before it is read)
        if (c->builtin) {
            if ((st = run_builtin(c, which == 0 ? kOpReadW : kOpReadPsi)) != NS2D_OK) return st;
        } else {
            scaled_kernel<<<spectral_grid(c), kBlock, 0, c->stream>>>(c->w_hat, c->fields, S, which);
            NS_HIP(c, hipGetLastError());
            NS_FFT(c, hipfftExecZ2D(c->c2r1, reinterpret_cast<hipfftDoubleComplex *>(c->fields), c->tmp));
        }
        if ((st = copy_out(c, outs[which], c->tmp, on_device)) != NS2D_OK) return st;
    }
    if (!on_device) NS_HIP(c, hipStreamSynchronize(c->stream));
    return NS2D_OK;
}

ns2d_status ns2d_get_transforms(const ns2d_ctx *c, int32_t *builtin)
{
    if (!c || !builtin) return NS2D_E_ARG;
    *builtin = c->builtin ? 1 : 0;
    return NS2D_OK;
}

ns2d_status ns2d_get_steps(const ns2d_ctx *c, int64_t *steps)
{
    if (!c || !steps) return NS2D_E_ARG;
    *steps = c->steps;
    return NS2D_OK;
}

}  // extern "C"
