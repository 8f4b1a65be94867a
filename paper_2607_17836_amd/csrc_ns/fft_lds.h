// Complex FFT of N = 64, 128, ..., 4096 FP64 points by one workgroup of N / 8
// threads, eight points a thread, exchanged through LDS between passes.
//
// Stockham autosort formulation (Govindaraju et al., "High performance
// discrete Fourier transforms on graphics processors", SC 2008): pass p of
// radix R reads butterfly j's R inputs at stride N / R, twists input r by
// exp(-+2 pi i r k / (Ns R)) with k = j mod Ns (Ns = product of the earlier
// radices), applies the R-point DFT and writes the outputs at stride Ns
// starting from (j - k) R + k; after the last pass the result is in natural
// order.  Radix-8 passes and a last 2 or 4 where log2 N is not a multiple of
// 3 (64 = 8 8, 128 = 8 8 2, 256 = 8 8 4, 512 = 8 8 8, 1024 = 8 8 8 2,
// 2048 = 8 8 8 4, 4096 = 8 8 8 8).  Forward: exp(-2 pi i jk / N); inverse:
// exp(+2 pi i jk / N), unnormalised.
//
// With T = N / 8 threads, thread t's inputs of every pass are the points t + q
// T, q = 0 .. 7, and so are its outputs of the last one: a transform starts and
// ends in registers, and only the exchanges between passes touch LDS (three at
// N = 512 and above; with the points staged in LDS before and after it was
// five).  Entry i sits at i + i / 8 there, so that the first exchange's stride
// of eight 16-byte entries spreads over the banks.  Twiddles come from a table
// per pass, laid out [r - 1][k], so that a wave's reads are contiguous.
#pragma once

#include <hip/hip_runtime.h>

namespace ns_fft {

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// z * (-i) for the forward transform, z * (+i) for the inverse.
template <bool INV>
__device__ __forceinline__ double2 rot90(double2 z)
{
    return INV ? make_double2(-z.y, z.x) : make_double2(z.y, -z.x);
}

template <bool INV>
__device__ __forceinline__ void dft2(double2 *v)
{
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

// 4-point DFT in natural order.
template <bool INV>
__device__ __forceinline__ void dft4(double2 *v)
{
    const double2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const double2 t2 = cadd(v[1], v[3]), t3 = rot90<INV>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
}

// 8-point DFT in natural order: 4-point DFTs of the even and odd inputs,
// combined with the eighth roots of unity.
template <bool INV>
__device__ __forceinline__ void dft8(double2 *v)
{
    constexpr double c = 0.70710678118654752440;   // sqrt(1/2)
    double2 e[4] = {v[0], v[2], v[4], v[6]};
    double2 o[4] = {v[1], v[3], v[5], v[7]};
    dft4<INV>(e);
    dft4<INV>(o);
    // w^s = exp(-+2 pi i s / 8)
    const double2 o1 = INV ? make_double2(c * (o[1].x - o[1].y), c * (o[1].x + o[1].y))
                           : make_double2(c * (o[1].x + o[1].y), c * (o[1].y - o[1].x));
    const double2 o2 = rot90<INV>(o[2]);
    const double2 o3 = INV ? make_double2(-c * (o[3].x + o[3].y), c * (o[3].x - o[3].y))
                           : make_double2(c * (o[3].y - o[3].x), -c * (o[3].x + o[3].y));
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
}

template <int R, bool INV>
__device__ __forceinline__ void dft(double2 *v)
{
    if constexpr (R == 8) dft8<INV>(v);
    else if constexpr (R == 4) dft4<INV>(v);
    else dft2<INV>(v);
}

// LDS entries of one transform's exchange buffer, and the place of entry i.
template <int N>
constexpr int lds_entries() { return N + N / 8; }
__device__ __forceinline__ int pad(int i) { return i + (i >> 3); }
// Distance of the places of entries i and i + n, for n a multiple of 8.
constexpr int padded(int n) { return n + n / 8; }

// Radix of the pass that follows NS points (8 unless fewer are left).
template <int N, int NS>
constexpr int radix() { return N / NS >= 8 ? 8 : N / NS; }

// Twiddle table of N: for NS = 8, 64, 512 (below N) the (R - 1) NS values
// exp(-2 pi i r k / (NS R)), r = 1 .. R - 1, k < NS, at table_offset(NS).
constexpr int table_offset(int ns) { return ns == 8 ? 0 : ns == 64 ? 7 * 8 : 7 * 72; }
inline int table_entries(int n)
{
    int e = 0;
    for (int ns = 8; ns < n; ns *= 8) e += ((n / ns >= 8 ? 8 : n / ns) - 1) * ns;
    return e;
}

// The butterflies of one pass on a thread's eight points: v[b + r B] is input
// (and output) r of butterfly j = t + b T.
template <int N, int NS, bool INV>
__device__ __forceinline__ void butterflies(double2 v[8], int t, const double2 *__restrict__ W)
{
    constexpr int R = radix<N, NS>(), B = 8 / R, T = N / 8;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        double2 x[R];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = v[b + r * B];
        if constexpr (NS > 1) {
            const int k = (t + b * T) & (NS - 1);
            const double2 *w0 = W + table_offset(NS) + k;
#pragma unroll
            for (int r = 1; r < R; ++r) {
                double2 w = w0[(r - 1) * NS];
                if (INV) w.y = -w.y;
                x[r] = cmul(x[r], w);
            }
        }
        dft<R, INV>(x);
#pragma unroll
        for (int r = 0; r < R; ++r) v[b + r * B] = x[r];
    }
}

// Who takes a transform: the whole block, or (BLOCK = false) a group of N / 8 <=
// 64 threads inside one wave, whose LDS accesses are in order by themselves, so
// that the blocks' barriers fall away.
template <bool BLOCK>
__device__ __forceinline__ void sync()
{
    if constexpr (BLOCK) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// The pass's outputs to LDS and the next pass's inputs back, synchronised
// before the buffer is written and before it is read.
template <int N, int NS, bool BLOCK>
__device__ __forceinline__ void exchange(double2 v[8], int t, double2 *buf)
{
    constexpr int R = radix<N, NS>(), B = 8 / R, T = N / 8;
    sync<BLOCK>();
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int j = t + b * T, k = j & (NS - 1), base = (j - k) * R + k;
#pragma unroll
        for (int r = 0; r < R; ++r)
            buf[pad(base) + r * (NS == 1 ? 1 : padded(NS))] = v[b + r * B];
    }
    sync<BLOCK>();
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = buf[pad(t) + q * padded(T)];
}

// Zero, but not to the compiler.  Added to the index of what a transform loads,
// it keeps a block that takes several transforms in a row from loading all
// their inputs at once and from holding the twiddles of every pass in
// registers from one to the next (250 registers and two waves per SIMD).
__device__ __forceinline__ int opaque_zero()
{
    int z = 0;
    asm volatile("" : "+s"(z) : : "memory");
    return z;
}

// The values of v are formed here, not where they are used: a block that takes
// several transforms in a row would otherwise carry the last pass's inputs and
// twiddles of each into the next.
__device__ __forceinline__ void settle(double2 v[8])
{
#pragma unroll
    for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(v[q].x), "+v"(v[q].y));
}

// N-point transform by N / 8 threads (see sync; t: the thread's number among
// them): v[q] is point t + q N / 8 on entry and on return.  buf
// (lds_entries<N>()) is written after a synchronisation, and may still be read
// by other threads on return.
template <int N, bool INV, bool BLOCK = true>
__device__ __forceinline__ void fft(double2 v[8], int t, double2 *buf,
                                    const double2 *__restrict__ W)
{
    static_assert(N >= 64 && N <= 4096 && (N & (N - 1)) == 0, "built-in transform sizes");
    static_assert(BLOCK || N <= 512, "a group stays inside a wave");
    W += opaque_zero();
    butterflies<N, 1, INV>(v, t, W);
    exchange<N, 1, BLOCK>(v, t, buf);
    butterflies<N, 8, INV>(v, t, W);
    if constexpr (N > 64) {
        exchange<N, 8, BLOCK>(v, t, buf);
        butterflies<N, 64, INV>(v, t, W);
    }
    if constexpr (N > 512) {
        exchange<N, 64, BLOCK>(v, t, buf);
        butterflies<N, 512, INV>(v, t, W);
    }
}

}  // namespace ns_fft
