// Field generation, float64 lattice sums and the batched 3D real-to-complex FFT
// with the +i sign (X_k = sum_R x_R e^{+2 pi i k.R / n}), for gfx950.
//
//  k_sums        float64 sums S^{pqr}_{m,mu} = sum_R delta u1^p u2^q u3^r (nuclear) or
//                sum_R delta M_c (magnetic): the k = 0 coefficient of every field,
//                used for the Bragg points and to centre the float32 fields.
//  k_plane_regs  generates the real fields of one lattice plane R1 (the Taylor
//                monomials delta u1^p u2^q u3^r of Sec. III.C, the occupancy of Sec.
//                III.B or the spin components of Sec. III.D), minus their mean, and
//                transforms them along axes 3 (real-to-complex, two real rows packed
//                in one complex line) and 2, entirely in LDS.
//  k_axis1_regs  transforms along axis 1 in place.
// Both take edges n = A B with A, B <= 16, or A a prime up to 61 on axis 1 and up to 47 in
// the planes (both edges of a plane then): A (then B) points per thread in registers.
// Edges 8, 16 and 32 have kernels with the length fixed at compile time
// (k_fft_planes_reg, k_fft_axis1_reg).  The remaining edges (a larger prime factor, or no
// such split, as 250 = 25 x 10) take k_fft_planes and k_fft_axis1: Stockham auto-sort
// passes in LDS of radix 2, 3, 4, 5 and a direct DFT, one output per thread, for any other
// prime (planned first, where it needs no twiddles); twiddles come from a
// float64-generated table.
#include <algorithm>
#include <type_traits>

#include "dsx_internal.h"

namespace dsx {

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmuli(float2 a) { return make_float2(-a.y, a.x); }   // i a
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }

// Quotient a / b for 0 <= a < 2^22 and 0 < b < 2^22, with rb ~= 1/b (float): the
// float estimate is off by at most one and is corrected with one remainder check.
__device__ __forceinline__ int qdiv(int a, int b, float rb)
{
    int q = (int)((float)a * rb);
    const int r = a - q * b;
    q += (r >= b) ? 1 : 0;
    q -= (r < 0) ? 1 : 0;
    return q;
}

// One Stockham pass of radix R over nf x nlines lines of length n held in LDS.
// Element e of line l of batch b sits at base[b * fstride + l * lstride + e * estride].
// Ns is the product of the radices of the earlier passes.
__device__ void stockham_pass(const float2* __restrict__ src, float2* __restrict__ dst,
                              int nlines, int lstride, int estride, int nf, int fstride,
                              int n, int R, int Ns, const float2* __restrict__ tw)
{
    const int nb = n / R;
    const int twstep = n / (Ns * R);
    const int total = nf * nlines * nb;
    const float rnb = 1.f / (float)nb, rnl = 1.f / (float)nlines, rns = 1.f / (float)Ns;
    if (R > 5) {
        // odd prime R: one output per work item, so a pass keeps every thread busy.
        // y_k = x'_0 + sum_{r=1}^{(R-1)/2} [(x'_r + x'_{R-r}) cos(2 pi r k / R)
        //                                   + i (x'_r - x'_{R-r}) sin(2 pi r k / R)],
        // x'_r = x_r e^{2 pi i r te / n} (te = 0 in the first pass).  r te <= R te < n
        // and r k mod R is stepped, so no index needs a division.
        const int step = n / R, h = (R - 1) / 2;
        const float rR = 1.f / (float)R;
        for (int it = threadIdx.x; it < total * R; it += blockDim.x) {
            const int B = qdiv(it, R, rR);
            const int k = it - B * R;
            const int L = qdiv(B, nb, rnb);
            const int j = B - L * nb;
            const int fb = qdiv(L, nlines, rnl), l = L - fb * nlines;
            const float2* x = src + fb * fstride + l * lstride + j * estride;
            const int jm = j - qdiv(j, Ns, rns) * Ns;
            const int o = (j - jm) * R + jm;
            const int te = jm * twstep;
            const int xs = nb * estride;
            float2 y = x[0];
            int b = 0;
            for (int r = 1; r <= h; ++r) {
                b += k;
                b -= (b >= R) ? R : 0;
                float2 xr = x[r * xs], xq = x[(R - r) * xs];
                if (Ns > 1) {
                    xr = cmul(xr, tw[r * te]);
                    xq = cmul(xq, tw[(R - r) * te]);
                }
                const float2 w = tw[b * step];
                const float2 sm = cadd(xr, xq), df = csub(xr, xq);
                y.x += sm.x * w.x - df.y * w.y;
                y.y += sm.y * w.x + df.x * w.y;
            }
            dst[fb * fstride + l * lstride + (o + k * Ns) * estride] = y;
        }
        return;
    }
    for (int it = threadIdx.x; it < total; it += blockDim.x) {
        const int L = qdiv(it, nb, rnb);
        const int j = it - L * nb;
        const int fb = qdiv(L, nlines, rnl), l = L - fb * nlines;
        const float2* s = src + fb * fstride + l * lstride;
        float2* d = dst + fb * fstride + l * lstride;
        const int jm = j - qdiv(j, Ns, rns) * Ns;
        const int o = (j - jm) * R + jm;          // (j / Ns) * Ns * R + j mod Ns
        const int te = jm * twstep;               // twiddle exponent step, r * te < n
        if (R == 4) {
            float2 v0 = s[j * estride];
            float2 v1 = cmul(s[(j + nb) * estride], tw[te]);
            float2 v2 = cmul(s[(j + 2 * nb) * estride], tw[2 * te]);
            float2 v3 = cmul(s[(j + 3 * nb) * estride], tw[3 * te]);
            float2 a0 = cadd(v0, v2), a1 = csub(v0, v2), a2 = cadd(v1, v3), a3 = cmuli(csub(v1, v3));
            d[o * estride] = cadd(a0, a2);
            d[(o + Ns) * estride] = cadd(a1, a3);
            d[(o + 2 * Ns) * estride] = csub(a0, a2);
            d[(o + 3 * Ns) * estride] = csub(a1, a3);
        } else if (R == 2) {
            float2 v0 = s[j * estride];
            float2 v1 = cmul(s[(j + nb) * estride], tw[te]);
            d[o * estride] = cadd(v0, v1);
            d[(o + Ns) * estride] = csub(v0, v1);
        } else if (R == 3) {
            const float h = 0.86602540378443864676f;   // sin(2 pi / 3)
            float2 v0 = s[j * estride];
            float2 v1 = cmul(s[(j + nb) * estride], tw[te]);
            float2 v2 = cmul(s[(j + 2 * nb) * estride], tw[2 * te]);
            float2 sm = cadd(v1, v2);
            float2 t = make_float2(v0.x - 0.5f * sm.x, v0.y - 0.5f * sm.y);
            float2 u = cscale(cmuli(csub(v1, v2)), h);
            d[o * estride] = cadd(v0, sm);
            d[(o + Ns) * estride] = cadd(t, u);
            d[(o + 2 * Ns) * estride] = csub(t, u);
        } else {   // R == 5
            const float c1 = 0.30901699437494742410f, c2 = -0.80901699437494742410f;
            const float s1 = 0.95105651629515357212f, s2 = 0.58778525229247312917f;
            float2 v0 = s[j * estride];
            float2 v1 = cmul(s[(j + nb) * estride], tw[te]);
            float2 v2 = cmul(s[(j + 2 * nb) * estride], tw[2 * te]);
            float2 v3 = cmul(s[(j + 3 * nb) * estride], tw[3 * te]);
            float2 v4 = cmul(s[(j + 4 * nb) * estride], tw[4 * te]);
            float2 b1 = cadd(v1, v4), b2 = cadd(v2, v3), d1 = csub(v1, v4), d2 = csub(v2, v3);
            float2 ra = make_float2(v0.x + c1 * b1.x + c2 * b2.x, v0.y + c1 * b1.y + c2 * b2.y);
            float2 rb = make_float2(v0.x + c2 * b1.x + c1 * b2.x, v0.y + c2 * b1.y + c1 * b2.y);
            float2 ia = cmuli(make_float2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y));
            float2 ib = cmuli(make_float2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y));
            d[o * estride] = make_float2(v0.x + b1.x + b2.x, v0.y + b1.y + b2.y);
            d[(o + Ns) * estride] = cadd(ra, ia);
            d[(o + 4 * Ns) * estride] = csub(ra, ia);
            d[(o + 2 * Ns) * estride] = cadd(rb, ib);
            d[(o + 3 * Ns) * estride] = csub(rb, ib);
        }
    }
}

// Full 1D transforms of all lines; ping-pongs between a and b and returns the
// buffer holding the result.  Caller synchronises before (inputs visible).
__device__ float2* lds_fft(float2* a, float2* b, int nlines, int lstride, int estride,
                           const AxisPlan& P, const float2* tw, int nf = 1, int fstride = 0)
{
    int Ns = 1;
    for (int s = 0; s < P.nrad; ++s) {
        stockham_pass(a, b, nlines, lstride, estride, nf, fstride, P.n, P.rad[s], Ns, tw);
        __syncthreads();
        Ns *= P.rad[s];
        float2* t = a; a = b; b = t;
    }
    return a;
}

// ---------------------------------------------------------------------------- sums
// Each thread walks P.chunk / 256 lattice cells and accumulates the monomials in
// groups of kSumsGroup float64 accumulators.  A group is reduced across the wave
// by recursive halving (each exchange moves half of the remaining values, so 32
// values need 32 exchanges instead of 32 x 6), then across the four waves through
// LDS.  The order of every addition is fixed: the sums are reproducible.
constexpr int kSumsGroup = 32;
constexpr int kSumsMaxPer = 8;    // cells per thread at most (the host's chunk is <= 8 x 256 cells)

template <int N>
struct MonoTable {
    int p[n_monomials(N)], q[n_monomials(N)], r[n_monomials(N)];
};

// (p, q, r) of every monomial index, in mono_index order
template <int N>
__host__ __device__ constexpr MonoTable<N> mono_table()
{
    MonoTable<N> m{};
    for (int dg = 0; dg <= N; ++dg)
        for (int p = dg; p >= 0; --p)
            for (int q = dg - p; q >= 0; --q) {
                const int t = mono_index(p, q, dg - p - q);
                m.p[t] = p; m.q[t] = q; m.r[t] = dg - p - q;
            }
    return m;
}

// One halving step: lanes with bit MASK set keep the upper HALF values, the others
// the lower HALF, each adding the partner's copy of the values it keeps.
template <int HALF, int MASK>
__device__ __forceinline__ void halve(double (&acc)[kSumsGroup], int lane)
{
    const bool hi = (lane & MASK) != 0;
#pragma unroll
    for (int k = 0; k < HALF; ++k) {
        const double send = hi ? acc[k] : acc[k + HALF];
        const double keep = hi ? acc[k + HALF] : acc[k];
        acc[k] = keep + __shfl_xor(send, MASK, 64);
    }
}

// Sum over the 64 lanes of acc[t] for every t; lane l (even) returns the total of
// acc[l >> 1].
__device__ __forceinline__ double wave_transpose_sum(double (&acc)[kSumsGroup], int lane)
{
    static_assert(kSumsGroup == 32, "five halving steps");
    halve<16, 32>(acc, lane);
    halve<8, 16>(acc, lane);
    halve<4, 8>(acc, lane);
    halve<2, 4>(acc, lane);
    halve<1, 2>(acc, lane);
    return acc[0] + __shfl_xor(acc[0], 1, 64);
}

template <int N, class PT>
__device__ __forceinline__ void sums_nuclear_body(PT P, const int bx)
{
    constexpr int T = n_monomials(N);
    constexpr MonoTable<N> mt = mono_table<N>();
    __shared__ double red[4][kSumsGroup];
    const int chunk = bx % P.nchunk;
    const int ms = bx / P.nchunk;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = chunk * P.chunk + threadIdx.x;
    const int c1 = min(P.ncell, (chunk + 1) * P.chunk);
    // this thread's cells (c0, c0 + 256, ...), loaded once for every monomial group;
    // the count is the same for the whole block
    const int ncl = (c1 - chunk * P.chunk + 255) / 256;
    float dv[kSumsMaxPer], uv[kSumsMaxPer][3];
#pragma unroll
    for (int i = 0; i < kSumsMaxPer; ++i) {
        const int c = c0 + 256 * i;
        const bool in = i < ncl && c < c1;
        const size_t at = (size_t)ms * P.ncell + (in ? c : 0);
        dv[i] = in ? (P.occ ? gptr(P.occ)[at] : 1.f) : 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) uv[i][a] = (in && N > 0 && P.vec) ? gptr(P.vec)[3 * at + a] : 0.f;
    }
    // orders above kMaxOrderFast keep the group loop rolled (up to 31 groups of 32)
    constexpr int kGroupUnroll = N <= kMaxOrderFast ? 8 : 1;
#pragma unroll kGroupUnroll
    for (int g0 = 0; g0 < T; g0 += kSumsGroup) {
        double acc[kSumsGroup];
#pragma unroll
        for (int t = 0; t < kSumsGroup; ++t) acc[t] = 0.0;
#pragma unroll
        for (int i = 0; i < kSumsMaxPer; ++i) {
            if (i >= ncl) break;
            const double d = (double)dv[i];
            double pw[3][N + 1];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                pw[a][0] = 1.0;
                const double u = (double)uv[i][a];
#pragma unroll
                for (int k = 1; k <= N; ++k) pw[a][k] = pw[a][k - 1] * u;
            }
#pragma unroll
            for (int t = 0; t < kSumsGroup; ++t)
                if (g0 + t < T)
                    acc[t] += d * pw[0][mt.p[g0 + t]] * pw[1][mt.q[g0 + t]] * pw[2][mt.r[g0 + t]];
        }
        const double v = wave_transpose_sum(acc, lane);
        if ((lane & 1) == 0) red[wave][lane >> 1] = v;
        __syncthreads();
        if (threadIdx.x < kSumsGroup && g0 + (int)threadIdx.x < T) {
            const int t = threadIdx.x;
            P.partial[((size_t)ms * P.nchunk + chunk) * T + g0 + t] =
                (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
        }
        __syncthreads();
    }
}

template <int N>
__global__ __launch_bounds__(256) void k_sums_nuclear(SumsParams P) { sums_nuclear_body<N, SumsParams>(P, blockIdx.x); }
template <int N>
__global__ __launch_bounds__(256) void k_sums_nuclear_merged(const SumsParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) sums_nuclear_body<N, const SumsParams&>(tab[d], bx);
}

template <class PT>
__device__ __forceinline__ void sums_magnetic_body(PT P, const int bx)
{
    __shared__ double red[4][3];
    const int chunk = bx % P.nchunk;
    const int ms = bx / P.nchunk;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double acc[3] = {0.0, 0.0, 0.0};
    const int c0 = chunk * P.chunk;
    const int c1 = min(P.ncell, c0 + P.chunk);
    for (int c = c0 + threadIdx.x; c < c1; c += blockDim.x) {
        const size_t at = (size_t)ms * P.ncell + c;
        const double d = P.occ ? (double)gptr(P.occ)[at] : 1.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) acc[a] += d * (double)gptr(P.vec)[3 * at + a];
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        double v = acc[t];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) red[wave][t] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) v += red[w][threadIdx.x];
        P.partial[((size_t)ms * P.nchunk + chunk) * 3 + threadIdx.x] = v;
    }
}

__global__ __launch_bounds__(256) void k_sums_magnetic(SumsParams P) { sums_magnetic_body<SumsParams>(P, blockIdx.x); }
__global__ __launch_bounds__(256) void k_sums_magnetic_merged(const SumsParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) sums_magnetic_body<const SumsParams&>(tab[d], bx);
}

// One wave per output sum: lanes read the chunk partials, then a fixed-order
// shuffle reduction (reproducible).
template <class PT>
__device__ __forceinline__ void sums_reduce_body(PT P, const int bx)
{
    const int idx = bx * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (idx >= P.M * P.S * P.T) return;
    const int ms = idx / P.T, t = idx - ms * P.T;
    double v = 0.0;
    for (int c = lane; c < P.nchunk; c += 64) v += P.partial[((size_t)ms * P.nchunk + c) * P.T + t];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) gptr(P.sums)[idx] = v;
}

__global__ __launch_bounds__(256) void k_sums_reduce(SumsParams P) { sums_reduce_body<SumsParams>(P, blockIdx.x); }
__global__ __launch_bounds__(256) void k_sums_reduce_merged(const SumsParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) sums_reduce_body<const SumsParams&>(tab[d], bx);
}

template <int N>
static hipError_t launch_sums_t(const SumsParams& p, hipStream_t st)
{
    return dispatch(k_sums_nuclear<N>, k_sums_nuclear_merged<N>, p.M * p.S * p.nchunk, 256, 0, st, p);
}

hipError_t launch_sums(const SumsParams& p, int order, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (p.kind == 1) {
        e = dispatch(k_sums_magnetic, k_sums_magnetic_merged, p.M * p.S * p.nchunk, 256, 0, st, p);
    } else {
        switch (order) {
            case 0: e = launch_sums_t<0>(p, st); break;
            case 1: e = launch_sums_t<1>(p, st); break;
            case 2: e = launch_sums_t<2>(p, st); break;
            case 3: e = launch_sums_t<3>(p, st); break;
            case 4: e = launch_sums_t<4>(p, st); break;
            case 5: e = launch_sums_t<5>(p, st); break;
            case 6: e = launch_sums_t<6>(p, st); break;
            case 7: e = launch_sums_t<7>(p, st); break;
            case 8: e = launch_sums_t<8>(p, st); break;
            case 9: e = launch_sums_t<9>(p, st); break;
            case 10: e = launch_sums_t<10>(p, st); break;
            case 11: e = launch_sums_t<11>(p, st); break;
            case 12: e = launch_sums_t<12>(p, st); break;
            case 13: e = launch_sums_t<13>(p, st); break;
            case 14: e = launch_sums_t<14>(p, st); break;
            case 15: e = launch_sums_t<15>(p, st); break;
            case 16: e = launch_sums_t<16>(p, st); break;
            default: return hipErrorInvalidValue;
        }
    }
    if (e != hipSuccess) return e;
    const int tot = p.M * p.S * p.T;
    return dispatch(k_sums_reduce, k_sums_reduce_merged, (tot + 3) / 4, 256, 0, st, p);
}

// ---------------------------------------------------------------------------- plane FFT
// Generates the nfb fields fa.. of rows 2 j0 .. 2 (j0 + nj) - 1 of the npl lattice planes
// R1 .. R1 + npl - 1 of site mu, configuration m (centred by their float64 mean), packs two
// real rows per complex line, transforms the lines along axis 3 in LDS and separates the
// two half spectra.  Item b = pl nfb + fb is field fa + fb of plane R1 + pl.  Returns the
// LDS buffer holding row r (local) of item b at [b * BE + r * nh + k3]; A and B are
// ping-pong buffers of npl nfb x BE elements.
__device__ __forceinline__ float2* planes_rows(const PlaneParams& P, float2* A, float2* B, const float2* tw3, int m, int mu,
                               int R1, int npl, int j0, int nj, int fa, int nfb, int BE)
{
    const int n2 = P.n2, n3 = P.n3, nh = P.nh;
    const int ncell = P.n1 * n2 * n3;
    const size_t plane0 = ((size_t)(m * P.S + mu)) * ncell + (size_t)R1 * n2 * n3;
    const auto* occ0 = P.occ ? gptr(P.occ) + plane0 : nullptr;
    const auto* vec0 = P.vec ? gptr(P.vec) + 3 * plane0 : nullptr;
    const float rpn3 = 1.f / (float)(nj * n3), rn3 = 1.f / (float)n3, rnh = 1.f / (float)nh;
    const float rpnh = 1.f / (float)(nj * nh), rnfb = 1.f / (float)nfb;
    const int nb = npl * nfb;
    for (int idx = threadIdx.x; idx < nb * nj * n3; idx += blockDim.x) {
        const int b = qdiv(idx, nj * n3, rpn3);
        const int rem = idx - b * nj * n3;
        const int jj = qdiv(rem, n3, rn3), R3 = rem - jj * n3;
        const int pl = qdiv(b, nfb, rnfb), fb = b - pl * nfb;
        const auto* occ = occ0 ? occ0 + (size_t)pl * n2 * n3 : nullptr;
        const auto* vec = vec0 ? vec0 + (size_t)3 * pl * n2 * n3 : nullptr;
        const int f = fa + fb;
        const int ep = P.mono[3 * f], eq = P.mono[3 * f + 1], er = P.mono[3 * f + 2];
        const int t = P.kind == 1 ? f : mono_index(ep, eq, er);    // index of the field's lattice sum
        const float mean = (float)(gptr(P.sums)[(size_t)(m * P.S + mu) * P.T + t] / (double)ncell);
        float xv[2] = {0.f, 0.f};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int R2 = 2 * (j0 + jj) + h;
            if (R2 < n2) {
                const int c = R2 * n3 + R3;
                float v;
                if (P.kind == 1) {
                    v = vec[3 * c + t];
                } else {
                    v = 1.f;
                    if (ep | eq | er) {
                        const float u0 = vec[3 * c], u1 = vec[3 * c + 1], u2 = vec[3 * c + 2];
                        for (int k = 0; k < ep; ++k) v *= u0;
                        for (int k = 0; k < eq; ++k) v *= u1;
                        for (int k = 0; k < er; ++k) v *= u2;
                    }
                }
                if (occ) v *= occ[c];
                xv[h] = v - mean;
            }
        }
        A[b * BE + jj * n3 + R3] = make_float2(xv[0], xv[1]);
    }
    __syncthreads();
    float2* Z = lds_fft(A, B, nj, n3, 1, P.p3, tw3, nb, BE);
    float2* C = (Z == A) ? B : A;
    // unpack the packed real transforms: X_a = (Z_k + conj Z_-k)/2, X_b = -i (Z_k - conj Z_-k)/2
    for (int idx = threadIdx.x; idx < nb * nj * nh; idx += blockDim.x) {
        const int b = qdiv(idx, nj * nh, rpnh);
        const int rem = idx - b * nj * nh;
        const int jj = qdiv(rem, nh, rnh), k = rem - jj * nh;
        const float2 zk = Z[b * BE + jj * n3 + k];
        const int km = (k == 0) ? 0 : n3 - k;
        const float2 zm = Z[b * BE + jj * n3 + km];
        const float2 xa = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
        const float2 xb = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
        C[b * BE + (2 * jj) * nh + k] = xa;
        if (2 * (j0 + jj) + 1 < n2) C[b * BE + (2 * jj + 1) * nh + k] = xb;
    }
    __syncthreads();
    return C;
}

template <class PT>
__device__ __forceinline__ void fft_planes_body(PT P, const int bx)
{
    extern __shared__ float2 smem[];
    float2* tw2 = smem;
    float2* tw3 = tw2 + P.n2;
    float2* A = tw3 + P.n3;
    float2* B = A + P.npl * P.fchunk * P.buf_elems;

    int b = bx;
    const int fc = b % P.nfchunk; b /= P.nfchunk;
    const int nrb = (P.n1 + P.npl - 1) / P.npl;      // plane blocks per (site, configuration)
    const int R1 = (b % nrb) * P.npl; b /= nrb;
    const int mu = b % P.S;
    const int m = b / P.S;
    const int n2 = P.n2, nh = P.nh;
    const int SF = P.S * P.F;

    for (int i = threadIdx.x; i < n2; i += blockDim.x) tw2[i] = ldg2(P.tw2, i);
    for (int i = threadIdx.x; i < P.n3; i += blockDim.x) tw3[i] = ldg2(P.tw3, i);
    const int fa = fc * P.fchunk;
    const int nfb = min(P.F, fa + P.fchunk) - fa;     // fields of this block, batched
    const int npl = min(P.npl, P.n1 - R1);            // and planes
    const int BE = P.buf_elems;
    __syncthreads();   // twiddles visible
    float2* C = planes_rows(P, A, B, tw3, m, mu, R1, npl, 0, (n2 + 1) / 2, fa, nfb, BE);
    float2* D = (C == A) ? B : A;
    float2* Y = lds_fft(C, D, nh, 1, nh, P.p2, tw2, npl * nfb, BE);
    // write: for each plane and k2, the block's fields are contiguous runs of nh complex
    const float rnh = 1.f / (float)nh, rfnh = 1.f / (float)(nfb * nh), rpl = 1.f / (float)(n2 * nfb * nh);
    float2* out = P.X + ((size_t)(m * P.n1 + R1) * n2) * SF * nh + (size_t)(mu * P.F + fa) * nh;
    for (int idx = threadIdx.x; idx < npl * n2 * nfb * nh; idx += blockDim.x) {
        const int pl = qdiv(idx, n2 * nfb * nh, rpl);
        const int r2 = idx - pl * n2 * nfb * nh;
        const int k2 = qdiv(r2, nfb * nh, rfnh);
        const int rem = r2 - k2 * nfb * nh;
        const int fb = qdiv(rem, nh, rnh), k3 = rem - fb * nh;
        stg2(out, ((size_t)pl * n2 + k2) * SF * nh + rem, Y[(pl * nfb + fb) * BE + k2 * nh + k3]);
    }
}

__global__ __launch_bounds__(256) void k_fft_planes(PlaneParams P) { fft_planes_body<PlaneParams>(P, blockIdx.x); }
__global__ __launch_bounds__(256) void k_fft_planes_merged(const PlaneParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) fft_planes_body<const PlaneParams&>(tab[d], bx);
}

// Planes that do not fit the LDS: rows 2 j0 .. of a plane (P.row_pairs pairs per block)
// generated and transformed along axis 3 only, written with the row index R2 in place
// of k2; the axis-2 transform then runs in place like the axis-1 one.
template <class PT>
__device__ __forceinline__ void fft_rows_body(PT P, const int bx)
{
    extern __shared__ float2 smem[];
    float2* tw3 = smem;
    float2* A = tw3 + P.n3;
    float2* B = A + P.fchunk * P.buf_elems;
    int b = bx;
    const int fc = b % P.nfchunk; b /= P.nfchunk;
    const int rc = b % P.nrchunk; b /= P.nrchunk;
    const int R1 = b % P.n1; b /= P.n1;
    const int mu = b % P.S;
    const int m = b / P.S;
    const int n2 = P.n2, nh = P.nh;
    const int SF = P.S * P.F;
    for (int i = threadIdx.x; i < P.n3; i += blockDim.x) tw3[i] = ldg2(P.tw3, i);
    const int fa = fc * P.fchunk;
    const int nfb = min(P.F, fa + P.fchunk) - fa;
    const int j0 = rc * P.row_pairs;
    const int nj = min((n2 + 1) / 2, j0 + P.row_pairs) - j0;
    const int BE = P.buf_elems;
    __syncthreads();
    const float2* C = planes_rows(P, A, B, tw3, m, mu, R1, 1, j0, nj, fa, nfb, BE);
    const int nrow = min(n2, 2 * (j0 + nj)) - 2 * j0;
    const float rnh = 1.f / (float)nh, rfnh = 1.f / (float)(nfb * nh);
    float2* out = P.X + ((size_t)(m * P.n1 + R1) * n2 + 2 * j0) * SF * nh + (size_t)(mu * P.F + fa) * nh;
    for (int idx = threadIdx.x; idx < nrow * nfb * nh; idx += blockDim.x) {
        const int r = qdiv(idx, nfb * nh, rfnh);
        const int rem = idx - r * nfb * nh;
        const int fb = qdiv(rem, nh, rnh), k3 = rem - fb * nh;
        stg2(out, (size_t)r * SF * nh + rem, C[fb * BE + r * nh + k3]);
    }
}

__global__ __launch_bounds__(256) void k_fft_rows(PlaneParams P) { fft_rows_body<PlaneParams>(P, blockIdx.x); }
__global__ __launch_bounds__(256) void k_fft_rows_merged(const PlaneParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) fft_rows_body<const PlaneParams&>(tab[d], bx);
}

// ---------------------------------------------------------------------------- register lines
// Lengths n = A B with A, B <= kMaxRegRadix (powers of two up to 256, 10, 12, 18, 20, 24, 40,
// 96, ...) or A a prime up to kMaxRegPrime: each thread transforms A (then B) points in registers, so a line takes one or two
// passes where the Stockham form takes one per radix, and its indices, twiddles and barriers
// are paid once per A or B points.  The transform of A points is unrolled at compile time
// (fours first, then the smallest prime; primes above 5 through the cosine and sine sums of
// their pairs), its twiddles are constants rounded from float64.
// On the 64^3 supercell (140 fields) the plane pass took 266 us in Stockham passes and 106 us
// here (151 MB written; the vector unit is busy about 70 % of it: the transforms of 8 points,
// their twiddles and the generation), axis 1 192 and 51 us (302 MB read and written); on
// 18 x 20 x 27 (1008 fields) 70 and 37 us, 35 and 19 us; on 40^3 (96 fields) 50 and 27 us, 32
// and 13 us.
//   n = A B:  y_j[k]   = sum_i x[j + B i] e^{2 pi i i k / A}          (j < B, k < A)
//             X[k + A l] = sum_j (e^{2 pi i j k / n} y_j[k]) e^{2 pi i j l / B}   (l < B)
template <int N>
struct TwTable {
    float c[N], s[N];
};

// cos and sin of 2 pi t / N in float64 (argument reduced to the first octant, then the Taylor
// series: the terms past x^18 are below 1e-18 there)
__host__ __device__ constexpr double octant_cos(double x)
{
    double v = 1.0, t = 1.0;
    for (int k = 1; k <= 9; ++k) { t *= -x * x / ((2 * k - 1) * (2 * k)); v += t; }
    return v;
}
__host__ __device__ constexpr double octant_sin(double x)
{
    double v = x, t = x;
    for (int k = 1; k <= 9; ++k) { t *= -x * x / ((2 * k) * (2 * k + 1)); v += t; }
    return v;
}
template <int N>
__host__ __device__ constexpr TwTable<N> tw_table()
{
    TwTable<N> tb{};
    for (int t = 0; t < N; ++t) {
        // 2 pi t / N = q pi / 2 + r pi / (4 N) with |r| <= N (q the nearest quadrant)
        const int q = (8 * t + N) / (2 * N);
        const int r = 8 * t - 2 * N * q;
        const double x = 3.14159265358979323846 * (double)r / (4.0 * N);
        const double c = octant_cos(x), s = octant_sin(x);
        const int m = q & 3;
        tb.c[t] = (float)(m == 0 ? c : m == 1 ? -s : m == 2 ? -c : s);
        tb.s[t] = (float)(m == 0 ? s : m == 1 ? c : m == 2 ? -s : -c);
    }
    return tb;
}

// a e^{2 pi i T / N}, T a constant after unrolling
template <int N>
__device__ __forceinline__ float2 rot(float2 a, int T)
{
    constexpr TwTable<N> tb = tw_table<N>();
    if (T == 0) return a;
    if (4 * T == N) return cmuli(a);
    if (2 * T == N) return make_float2(-a.x, -a.y);
    return make_float2(a.x * tb.c[T] - a.y * tb.s[T], a.x * tb.s[T] + a.y * tb.c[T]);
}

__host__ __device__ constexpr int first_factor(int n)
{
    if (n % 4 == 0) return 4;
    for (int f = 2; f < n; ++f)
        if (n % f == 0) return f;
    return n;
}

// z <- its transform of length N, natural order in and out
template <int N>
__device__ __forceinline__ void fft_small(float2 (&z)[N])
{
    constexpr int P = first_factor(N);
    if constexpr (N == 1) {
    } else if constexpr (N == 2) {
        const float2 a = z[0], b = z[1];
        z[0] = cadd(a, b);
        z[1] = csub(a, b);
    } else if constexpr (N == 4) {
        const float2 a0 = cadd(z[0], z[2]), a1 = csub(z[0], z[2]), a2 = cadd(z[1], z[3]), a3 = cmuli(csub(z[1], z[3]));
        z[0] = cadd(a0, a2);
        z[1] = cadd(a1, a3);
        z[2] = csub(a0, a2);
        z[3] = csub(a1, a3);
    } else if constexpr (P == N) {
        // odd prime: X_k = x_0 + sum_r [(x_r + x_{N-r}) cos(2 pi r k / N) + i (x_r - x_{N-r}) sin(2 pi r k / N)],
        // and X_{N-k} the same with the sines' sign turned
        constexpr TwTable<N> tb = tw_table<N>();
        constexpr int H = (N - 1) / 2;
        float2 sm[H], df[H];
        float2 x0 = z[0];
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            sm[r - 1] = cadd(z[r], z[N - r]);
            df[r - 1] = csub(z[r], z[N - r]);
        }
#pragma unroll
        for (int k = 1; k <= H; ++k) {
            float2 e = x0, o = make_float2(0.f, 0.f);
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const float c = tb.c[(r * k) % N], s = tb.s[(r * k) % N];
                e.x = fmaf(c, sm[r - 1].x, e.x);
                e.y = fmaf(c, sm[r - 1].y, e.y);
                o.x = fmaf(-s, df[r - 1].y, o.x);
                o.y = fmaf(s, df[r - 1].x, o.y);
            }
            z[k] = cadd(e, o);
            z[N - k] = csub(e, o);
        }
#pragma unroll
        for (int r = 0; r < H; ++r) x0 = cadd(x0, sm[r]);
        z[0] = x0;
    } else {
        constexpr int Q = N / P;
        float2 y[P][Q];
#pragma unroll
        for (int a = 0; a < P; ++a) {
#pragma unroll
            for (int b = 0; b < Q; ++b) y[a][b] = z[a + P * b];
            fft_small<Q>(y[a]);
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            float2 t[P];
#pragma unroll
            for (int a = 0; a < P; ++a) t[a] = rot<N>(y[a][k], a * k);
            fft_small<P>(t);
#pragma unroll
            for (int c = 0; c < P; ++c) z[k + Q * c] = t[c];
        }
    }
}

// The transform of length N of z, each value handed to put(k, X_k) (z is overwritten).  Primes
// above kMaxRegRadix: the sums and differences of the pairs take z's place and every output is
// put as soon as it is formed, so a thread holds the line once (2 N registers), not twice.
template <int N, class Put>
__device__ __forceinline__ void fft_line(float2 (&z)[N], Put put)
{
    if constexpr (N <= kMaxRegRadix) {
        fft_small<N>(z);
#pragma unroll
        for (int k = 0; k < N; ++k) put(k, z[k]);
    } else {
        constexpr TwTable<N> tb = tw_table<N>();
        constexpr int H = (N - 1) / 2;
        float2 x0 = z[0];
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            const float2 a = z[r], b = z[N - r];
            z[r] = cadd(a, b);
            z[N - r] = csub(a, b);
            x0 = cadd(x0, z[r]);
        }
        put(0, x0);
#pragma unroll
        for (int k = 1; k <= H; ++k) {
            float2 e = z[0], o = make_float2(0.f, 0.f);
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const float c = tb.c[(r * k) % N], s = tb.s[(r * k) % N];
                e.x = fmaf(c, z[r].x, e.x);
                e.y = fmaf(c, z[r].y, e.y);
                o.x = fmaf(-s, z[N - r].y, o.x);
                o.y = fmaf(s, z[N - r].x, o.y);
            }
            put(k, cadd(e, o));
            put(N - k, csub(e, o));
            __builtin_amdgcn_sched_barrier(0);       // one pair of outputs at a time in registers
        }
    }
}

// Long lines: addresses for eight loads at a time, not for the whole line.
template <int N>
__device__ __forceinline__ void load_fence(int i)
{
    if (N > kMaxRegRadix && (i & 7) == 7) __builtin_amdgcn_sched_barrier(0);
}

// x as it is, its derivation hidden from the compiler: base + i * stride then stays one add per
// element instead of a product rebuilt for each
__device__ __forceinline__ int opaque(int x)
{
    asm("" : "+v"(x));
    return x;
}

__device__ __forceinline__ float2* opaque(float2* p)
{
    asm("" : "+v"(p));
    return p;
}

// f(std::integral_constant<int, n>) for the run-time (block-uniform) n in 1..kMaxRegRadix, and,
// with BIG > 0, the primes above it up to BIG (kernels of their own: their lines take more registers)
template <int BIG = 0, class F>
__device__ __forceinline__ void with_radix(int n, F f)
{
    if constexpr (BIG >= 61) {
        switch (n) {
            case 53: f(std::integral_constant<int, 53>{}); return;
            case 59: f(std::integral_constant<int, 59>{}); return;
            case 61: f(std::integral_constant<int, 61>{}); return;
            default: break;
        }
    }
    if constexpr (BIG >= 47) {
        switch (n) {
            case 17: f(std::integral_constant<int, 17>{}); return;
            case 19: f(std::integral_constant<int, 19>{}); return;
            case 23: f(std::integral_constant<int, 23>{}); return;
            case 29: f(std::integral_constant<int, 29>{}); return;
            case 31: f(std::integral_constant<int, 31>{}); return;
            case 37: f(std::integral_constant<int, 37>{}); return;
            case 41: f(std::integral_constant<int, 41>{}); return;
            case 43: f(std::integral_constant<int, 43>{}); return;
            case 47: f(std::integral_constant<int, 47>{}); return;
            default: break;
        }
    }
    switch (n) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
        case 8: f(std::integral_constant<int, 8>{}); break;
        case 9: f(std::integral_constant<int, 9>{}); break;
        case 10: f(std::integral_constant<int, 10>{}); break;
        case 11: f(std::integral_constant<int, 11>{}); break;
        case 12: f(std::integral_constant<int, 12>{}); break;
        case 13: f(std::integral_constant<int, 13>{}); break;
        case 14: f(std::integral_constant<int, 14>{}); break;
        case 15: f(std::integral_constant<int, 15>{}); break;
        default: f(std::integral_constant<int, 16>{}); break;
    }
}

// Generates the block's fields of npl planes (or of the row pairs j0 .. j0 + nj - 1 of one
// plane), centred by their float64 mean, packs two real rows per complex line and transforms
// the lines along axis 3.  Line l = b nj + jj (b = pl nfb + fb) holds Z_k, k < n3, at
// Q[l lp + k]; its two half spectra are separated by whoever reads it (unpack_row).  A is
// the other buffer.  Lanes run over the lines (lp odd): no bank conflicts at any n3.
template <bool BIG>
__device__ __forceinline__ void plane_lines(const PlaneParams& P, float2* A, float2* Q, const float2* tw3, const float* meanf, const int* expo, int m, int mu,
                            int R1, int npl, int j0, int nj, int fa, int nfb)
{
    const int n2 = P.n2, n3 = P.n3, lp = P.lp, T = P.threads;
    const int ncell = P.n1 * n2 * n3;
    const int nb = npl * nfb, nl = nb * nj;
    // generation: a thread takes the cells of one column of a row pair (both parts of a packed
    // value) and loads their variables once for all the block's fields, up to four pairs at a
    // time so that their loads share one latency.  The loop over the fields is uniform:
    // exponents are scalars, a field that continues the p-run of the previous one costs one
    // product.
    const int pairs = npl * nj * n3;
    const size_t at0 = (size_t)(m * P.S + mu) * ncell + ((size_t)R1 * n2 + 2 * j0) * n3;
    const auto* occ = reinterpret_cast<const __attribute__((address_space(1))) char*>(P.occ ? gptr(P.occ) + at0 : nullptr);
    const auto* vec = reinterpret_cast<const __attribute__((address_space(1))) char*>(P.vec ? gptr(P.vec) + 3 * at0 : nullptr);
    const float rn3 = 1.f / (float)n3, rnj = 1.f / (float)nj;
    const int last = n2 - 2 * j0;                  // rows of the plane from 2 j0 on
    // the thread's pairs c0, c0 + T, ...: their column R3 and row pair r (over all planes) are stepped
    const int dr = __builtin_amdgcn_readfirstlane(qdiv(T, n3, rn3)), dR3 = T - dr * n3;
    int r = qdiv(threadIdx.x, n3, rn3), R3 = (int)threadIdx.x - r * n3;
    auto generate = [&](auto un) {
        constexpr int UN = decltype(un)::value;
#pragma unroll 1
        for (int c0 = threadIdx.x; c0 < pairs; c0 += UN * T) {
            float d[UN][2], v[UN][2];
            float3 u[UN][2];
            int at[UN];
            bool odd[UN];                          // the pair's second row exists
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                const bool in = c0 + i * T < pairs;
                const int rc = in ? r : 0, pl = npl == 1 ? 0 : qdiv(rc, nj, rnj), jj = rc - __umul24(pl, nj);
                at[i] = __umul24(__umul24(pl, nfb * nj) + jj, lp) + R3;
                odd[i] = 2 * jj + 1 < last;
                const uint32_t cell = __umul24(__umul24(pl, n2) + 2 * jj, n3) + R3;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t c = cell + (h && odd[i] ? (uint32_t)n3 : 0u);
                    d[i][h] = occ ? *reinterpret_cast<const __attribute__((address_space(1))) float*>(occ + 4u * c) : 1.f;
                    u[i][h] = make_float3(0.f, 0.f, 0.f);
                    if (vec) {
                        const auto* w = reinterpret_cast<const __attribute__((address_space(1))) float*>(vec + 12u * c);
                        u[i][h] = make_float3(w[0], w[1], w[2]);
                    }
                    v[i][h] = 1.f;
                }
                r += dr;
                R3 += dR3;
                if (R3 >= n3) { R3 -= n3; ++r; }
            }
            int pe = -1, qe = -1, re = -1;
            for (int fb = 0; fb < nfb; ++fb) {
                const int f = fa + fb;
                const float mf = meanf[fb];
                if (P.kind == 1) {
#pragma unroll
                    for (int i = 0; i < UN; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h) v[i][h] = f == 0 ? u[i][h].x : f == 1 ? u[i][h].y : u[i][h].z;
                } else {
                    const int ex = __builtin_amdgcn_readfirstlane(expo[fb]);
                    const int ep = ex & 0xff, eq = (ex >> 8) & 0xff, er = ex >> 16;
                    const bool next = ep == pe + 1 && eq == qe && er == re;
                    if (!next)
#pragma unroll
                        for (int i = 0; i < UN; ++i) v[i][0] = v[i][1] = 1.f;
                    for (int e = next ? ep - 1 : 0; e < ep; ++e)
#pragma unroll
                        for (int i = 0; i < UN; ++i) { v[i][0] *= u[i][0].x; v[i][1] *= u[i][1].x; }
                    for (int e = next ? eq : 0; e < eq; ++e)
#pragma unroll
                        for (int i = 0; i < UN; ++i) { v[i][0] *= u[i][0].y; v[i][1] *= u[i][1].y; }
                    for (int e = next ? er : 0; e < er; ++e)
#pragma unroll
                        for (int i = 0; i < UN; ++i) { v[i][0] *= u[i][0].z; v[i][1] *= u[i][1].z; }
                    pe = ep; qe = eq; re = er;
                }
                float2* const dst = A + fb * nj * lp;
#pragma unroll
                for (int i = 0; i < UN; ++i)
                    if (c0 + i * T < pairs)
                        dst[at[i]] = make_float2(0.5f * (v[i][0] * d[i][0] - mf), odd[i] ? 0.5f * (v[i][1] * d[i][1] - mf) : 0.f);
            }
        }
    };
    if (pairs <= T) generate(std::integral_constant<int, 1>{});
    else if (pairs <= 2 * T) generate(std::integral_constant<int, 2>{});
    else generate(std::integral_constant<int, 4>{});
    __syncthreads();
    const int A3 = P.a3, B3 = P.b3;
    const float rnl = 1.f / (float)nl;
    with_radix<BIG ? kMaxPlanePrime : 0>(A3, [&](auto len) {
        constexpr int R = decltype(len)::value;
#pragma unroll 1
        for (int it = threadIdx.x; it < nl * B3; it += T) {
            const int j = qdiv(it, nl, rnl), l = it - j * nl;
            const int line = opaque(l * lp), a0 = line + j;
            float2 z[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                z[i] = A[a0 + i * B3];
                load_fence<R>(i);
            }
            if constexpr (R > kMaxRegRadix) {
                fft_line<R>(z, [&](int k, float2 v) {
                    if (B3 > 1) A[a0 + k * B3] = cmul(v, tw3[j * k]);
                    else Q[line + k] = v;
                });
                continue;
            } else {
                fft_small<R>(z);
            }
            if (B3 > 1) {
                // (in place: y_j[k] takes the place of x[j + B k])
#pragma unroll
                for (int k = 1; k < R; ++k) z[k] = cmul(z[k], tw3[j * k]);
#pragma unroll
                for (int k = 0; k < R; ++k) A[a0 + k * B3] = z[k];
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) Q[line + k] = z[k];
            }
        }
    });
    __syncthreads();
    if (B3 > 1) {
        with_radix(B3, [&](auto len) {
            constexpr int R = decltype(len)::value;
#pragma unroll 1
            for (int it = threadIdx.x; it < nl * A3; it += T) {
                const int k = qdiv(it, nl, rnl), l = it - k * nl;
                const int line = l * lp, a0 = opaque(line + k * B3), q0 = opaque(line + k);
                float2 z[R];
#pragma unroll
                for (int j = 0; j < R; ++j) z[j] = A[a0 + j];
                fft_small<R>(z);
#pragma unroll
                for (int i = 0; i < R; ++i) Q[q0 + i * A3] = z[i];
            }
        });
        __syncthreads();
    }
}

// Row `h` (0, 1) of the pair whose packed transform is Z, at k: X_a = Z_k + conj Z_-k or
// X_b = -i (Z_k - conj Z_-k); the packed values are halved when they are generated
__device__ __forceinline__ float2 unpack_row(const float2* Z, int k, int n3, int h)
{
    const float2 zk = Z[k], zm = Z[k ? n3 - k : 0];
    return h ? make_float2(zk.y + zm.y, zm.x - zk.x) : make_float2(zk.x + zm.x, zk.y - zm.y);
}

// Blocks of one (configuration, site, plane group) differ in their fields and read the same
// cells: they are dealt to one XCD (blocks go round-robin to the 8 XCDs), whose L2 then holds
// the cells and merges the runs they write.  ng groups, nc field chunks each; the groups past
// the last multiple of 8 keep the plain order.
__device__ __forceinline__ void group_chunk(int bx, int ng, int nc, int& g, int& c)
{
    const int ng8 = ng & ~7;
    if (bx < ng8 * nc) {
        const int q = bx >> 3;
        g = (q / nc) * 8 + (bx & 7);
        c = q % nc;
    } else {
        const int r = bx - ng8 * nc;
        g = ng8 + r / nc;
        c = r % nc;
    }
}

// Plane transforms of any A B edges: generation, axis 3, axis 2, written to the spectra.  Boxes with
// every edge <= kMaxRegRadix (P.a1) are transformed whole: after axis 2 the planes, in LDS, are
// transformed along axis 1 before the one write, one launch and no pass over the spectra where
// planes and axis 1 took two: a 12^3 model alone 3 us less per call (a launch), 1024 of them 51 us
// where planes and axis 1 took 28 + 19, 100 x 32 fields of 10^3 20 us where they took 28.
template <bool BIG, class PT>
__device__ __forceinline__ void plane_regs_body(PT P, const int bx)
{
    extern __shared__ float2 smem[];
    __shared__ float meanf[kPlaneMaxFields];
    __shared__ int expo[kPlaneMaxFields];           // the fields' exponents p | q << 8 | r << 16
    const int n2 = P.n2, n3 = P.n3, nh = P.nh, lp = P.lp, T = P.threads;
    const bool rows = P.row_pairs > 0;
    const int nrb = rows ? P.n1 * P.nrchunk : (P.n1 + P.npl - 1) / P.npl;   // groups per (configuration, site)
    int gi, ci;
    group_chunk(bx, P.M * P.S * nrb, P.nfchunk, gi, ci);
    // (quotients by run-time divisors come out of the vector unit: back to scalars, so that the
    // addresses built from them are scalar too)
    const int g = __builtin_amdgcn_readfirstlane(gi), fc = __builtin_amdgcn_readfirstlane(ci);
    const int ms = __builtin_amdgcn_readfirstlane(g / nrb), rb = g - ms * nrb;
    const int m = __builtin_amdgcn_readfirstlane(ms / P.S), mu = ms - m * P.S;
    const int R1 = rows ? __builtin_amdgcn_readfirstlane(rb / P.nrchunk) : rb * P.npl;
    const int npl = rows ? 1 : min(P.npl, P.n1 - R1);
    const int j0 = rows ? (rb - R1 * P.nrchunk) * P.row_pairs : 0;
    const int nj = (rows ? min((n2 + 1) / 2, j0 + P.row_pairs) : (n2 + 1) / 2) - j0;
    const int fa = fc * P.fchunk;
    const int nfb = min(P.F, fa + P.fchunk) - fa;
    float2* tw3 = smem;
    float2* tw2 = tw3 + n3;
    float2* A = tw2 + (rows ? 0 : n2);
    float2* Q = A + P.npl * P.fchunk * P.buf_elems;
    for (int i = threadIdx.x; i < n3; i += T) tw3[i] = ldg2(P.tw3, i);
    if (!rows)
        for (int i = threadIdx.x; i < n2; i += T) tw2[i] = ldg2(P.tw2, i);
    const bool box = !BIG && P.a1 > 0;
    if ((int)threadIdx.x < nfb) {
        const int f = fa + threadIdx.x;
        const int ep = P.mono[3 * f], eq = P.mono[3 * f + 1], er = P.mono[3 * f + 2];
        const int t = P.kind == 1 ? f : mono_index(ep, eq, er);
        expo[threadIdx.x] = ep | (eq << 8) | (er << 16);
        meanf[threadIdx.x] = (float)(gptr(P.sums)[(size_t)(m * P.S + mu) * P.T + t] / (double)(P.n1 * n2 * n3));
    }
    __syncthreads();
    plane_lines<BIG>(P, A, Q, tw3, meanf, expo, m, mu, R1, npl, j0, nj, fa, nfb);
    // one (k1, k2) column of the spectra (scalar: steps between columns are scalar offsets)
    const int col = __builtin_amdgcn_readfirstlane(P.S * P.F * nh);
    const int run = nfb * nh;                       // contiguous in the spectra for each (k1, k2)
    const float rrun = 1.f / (float)run, rnh = 1.f / (float)nh;
    float2* out = P.X + ((size_t)(m * P.n1 + R1) * n2 + 2 * j0) * col + (size_t)(mu * P.F + fa) * nh;
    if (rows) {
        // axis 3 only: the axis-2 transform follows in place
        const int nr = min(n2, 2 * (j0 + nj)) - 2 * j0;
        for (int it = threadIdx.x; it < nr * run; it += T) {
            const int r = qdiv(it, run, rrun), e = it - r * run;
            const int fb = qdiv(e, nh, rnh), k3 = e - fb * nh;
            stg2(out, (size_t)r * col + e, unpack_row(Q + (fb * nj + (r >> 1)) * lp, k3, n3, r & 1));
        }
        return;
    }
    const int A2 = P.a2, B2 = P.b2;
    const int colA = __builtin_amdgcn_readfirstlane(A2 * col), B2nh = B2 * nh;
    const float rB2 = 1.f / (float)B2, rA2 = 1.f / (float)A2;
    with_radix<BIG ? kMaxPlanePrime : 0>(A2, [&](auto len) {
        constexpr int R = decltype(len)::value;
#pragma unroll 1
        for (int it = threadIdx.x; it < npl * B2 * run; it += T) {
            const int q = qdiv(it, run, rrun), e = it - q * run;
            const int pl = B2 == 1 ? q : qdiv(q, B2, rB2), j = q - pl * B2;
            const int fb = qdiv(e, nh, rnh), k3 = e - fb * nh;
            const int bi = pl * nfb + fb;
            const float2* const Z = Q + bi * nj * lp;
            float2 z[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int row = j + B2 * i;
                z[i] = unpack_row(Z + __umul24(row >> 1, lp), k3, n3, row & 1);
                load_fence<R>(i);
            }
            if constexpr (R > kMaxRegRadix) {
                const int a0 = opaque((bi * n2 + j) * nh + k3);
                float2* const o = opaque(out + (size_t)pl * n2 * col + e);
                fft_line<R>(z, [&](int k, float2 v) {
                    if (B2 > 1) A[a0 + k * B2nh] = cmul(v, tw2[j * k]);
                    else stg2(o + k * (size_t)col, 0, v);
                });
                continue;
            } else {
                fft_small<R>(z);
            }
            if (box) {
                const int a0 = opaque(bi * n2 * nh + k3);
#pragma unroll
                for (int k = 0; k < R; ++k) A[a0 + k * nh] = z[k];
            } else if (B2 > 1) {
                const int a0 = opaque((bi * n2 + j) * nh + k3);
#pragma unroll
                for (int k = 1; k < R; ++k) z[k] = cmul(z[k], tw2[j * k]);
#pragma unroll
                for (int k = 0; k < R; ++k) A[a0 + k * B2nh] = z[k];
            } else {
                float2* const o = opaque(out + (size_t)pl * n2 * col + e);
#pragma unroll
                for (int k = 0; k < R; ++k) stg2(o + k * (size_t)col, 0, z[k]);
            }
        }
    });
    if constexpr (!BIG) {
        if (box) {
            // axis 1: a column (field, k2, k3) over the planes
            __syncthreads();
            const size_t plane = (size_t)n2 * col;
            const int step = nfb * n2 * nh;
            with_radix(P.a1, [&](auto len) {
                constexpr int R = decltype(len)::value;
#pragma unroll 1
                for (int it = threadIdx.x; it < n2 * run; it += T) {
                    const int k2 = qdiv(it, run, rrun), e = it - k2 * run;
                    const int fb = qdiv(e, nh, rnh), k3 = e - fb * nh;
                    const int a0 = opaque((fb * n2 + k2) * nh + k3);
                    float2 z[R];
#pragma unroll
                    for (int i = 0; i < R; ++i) z[i] = A[a0 + i * step];
                    fft_small<R>(z);
                    float2* const o = opaque(out + (size_t)k2 * col + e);
#pragma unroll
                    for (int k = 0; k < R; ++k) stg2(o + k * plane, 0, z[k]);
                }
            });
            return;
        }
    }
    if (B2 == 1) return;
    __syncthreads();
    with_radix(B2, [&](auto len) {
        constexpr int R = decltype(len)::value;
#pragma unroll 1
        for (int it = threadIdx.x; it < npl * A2 * run; it += T) {
            const int q = qdiv(it, run, rrun), e = it - q * run;
            const int pl = qdiv(q, A2, rA2), k = q - pl * A2;
            const int fb = qdiv(e, nh, rnh), k3 = e - fb * nh;
            const int a0 = opaque(((pl * nfb + fb) * n2 + k * B2) * nh + k3);
            float2 z[R];
#pragma unroll
            for (int j = 0; j < R; ++j) z[j] = A[a0 + j * nh];
            fft_small<R>(z);
            float2* const o = opaque(out + (size_t)(pl * n2 + k) * col + e);
#pragma unroll
            for (int l = 0; l < R; ++l) stg2(o + l * (size_t)colA, 0, z[l]);
        }
    });
}

// (at most 96 VGPRs: the transforms of up to 16 points fit, and two 512-thread blocks or more share a CU)
template <bool BIG>
__global__ __launch_bounds__(512, BIG ? 3 : 5) void k_plane_regs(PlaneParams P) { plane_regs_body<BIG, PlaneParams>(P, blockIdx.x); }
template <bool BIG>
__global__ __launch_bounds__(512, BIG ? 3 : 5) void k_plane_regs_merged(const PlaneParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) plane_regs_body<BIG, const PlaneParams&>(tab[d], bx);
}

// Axis 1 in place for n1 = A B: a thread loads A values of a column straight into registers
// (the lanes' columns are contiguous), transforms them, and exchanges them through LDS for its
// B values of the second pass: one read and one write of the spectra, one barrier.
template <bool BIG, class PT>
__device__ __forceinline__ void axis1_regs_body(PT P, const int bx)
{
    extern __shared__ float2 smem[];
    const int A1 = P.a, B1 = P.b, tc = P.tc, n1 = P.n1;
    const int b = __builtin_amdgcn_readfirstlane(bx / P.ncolblk), cb = bx - b * P.ncolblk;
    const int m = __builtin_amdgcn_readfirstlane(b / P.n2), k2 = b - m * P.n2;
    const int c0 = cb * tc, nc = min(tc, P.cols - c0);
    const size_t rowstride = (size_t)P.n2 * P.cols;
    const size_t rowB = rowstride * B1, rowA = rowstride * A1;
    float2* const base = P.X + ((size_t)m * n1 * P.n2 + k2) * P.cols + c0;
    float2* const tw = smem;
    float2* const W = tw + n1;                       // [n1][tc]
    const float rtc = 1.f / (float)tc;
    if (B1 > 1) {
        for (int i = threadIdx.x; i < n1; i += blockDim.x) tw[i] = ldg2(P.tw1, i);
        __syncthreads();
    }
    with_radix<BIG ? kMaxRegPrime : 0>(A1, [&](auto len) {
        constexpr int R = decltype(len)::value;
        for (int it = threadIdx.x; it < tc * B1; it += blockDim.x) {
            const int j = qdiv(it, tc, rtc), c = it - j * tc;
            if (c >= nc) continue;
            float2* const src = opaque(base + (size_t)j * rowstride + c);
            float2 z[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                z[i] = ldg2(src + i * rowB, 0);
                load_fence<R>(i);
            }
            if constexpr (R > kMaxRegRadix) {
                const int w0 = opaque(it);
                fft_line<R>(z, [&](int k, float2 v) {
                    if (B1 > 1) W[w0 + k * B1 * tc] = cmul(v, tw[j * k]);
                    else stg2(src + k * rowstride, 0, v);
                });
                continue;
            } else {
                fft_small<R>(z);
            }
            if (B1 > 1) {
                const int w0 = opaque(it);              // j tc + c
#pragma unroll
                for (int k = 1; k < R; ++k) z[k] = cmul(z[k], tw[j * k]);
#pragma unroll
                for (int k = 0; k < R; ++k) W[w0 + k * B1 * tc] = z[k];
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) stg2(src, (size_t)k * rowstride, z[k]);
            }
        }
    });
    if (B1 == 1) return;
    __syncthreads();
    with_radix(B1, [&](auto len) {
        constexpr int R = decltype(len)::value;
        for (int it = threadIdx.x; it < tc * A1; it += blockDim.x) {
            const int k = qdiv(it, tc, rtc), c = it - k * tc;
            if (c >= nc) continue;
            const int w0 = opaque(k * B1 * tc + c);
            float2 z[R];
#pragma unroll
            for (int j = 0; j < R; ++j) z[j] = W[w0 + j * tc];
            fft_small<R>(z);
            float2* const dst = opaque(base + (size_t)k * rowstride + c);
#pragma unroll
            for (int l = 0; l < R; ++l) stg2(dst + l * rowA, 0, z[l]);
        }
    });
}

template <bool BIG>
__global__ __launch_bounds__(256) void k_axis1_regs(Axis1Params P) { axis1_regs_body<BIG, Axis1Params>(P, blockIdx.x); }
template <bool BIG>
__global__ __launch_bounds__(256) void k_axis1_regs_merged(const Axis1Params* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) axis1_regs_body<BIG, const Axis1Params&>(tab[d], bx);
}

// ---------------------------------------------------------------------------- register FFTs
// Power-of-two lengths L <= 32 are transformed by one thread in registers
// (radix-2 decimation in time, input in bit-reversed order), so a line needs no
// LDS passes and no barriers.
__host__ __device__ constexpr int bit_reverse(int i, int L)
{
    int r = 0;
    for (int b = 1; b < L; b <<= 1) { r = (r << 1) | (i & 1); i >>= 1; }
    return r;
}

template <int L>
__device__ __forceinline__ void fft_reg(float2 (&z)[L], const float2* __restrict__ tw)   // tw[t] = e^{+2 pi i t / L}
{
#pragma unroll
    for (int st = 0; (1 << st) < L; ++st) {
        const int half = 1 << st;
        const int step = L / (2 * half);
#pragma unroll
        for (int k = 0; k < L; k += 2 * half) {
#pragma unroll
            for (int j = 0; j < half; ++j) {
                const float2 a = z[k + j];
                float2 b = z[k + j + half];
                if (j * step == L / 4) b = cmuli(b);          // e^{+i pi / 2} = i
                else if (j != 0) b = cmul(b, tw[j * step]);
                z[k + j] = cadd(a, b);
                z[k + j + half] = csub(a, b);
            }
        }
    }
}

// Axis 1 in place: one thread per column (k2, c), the L1 values of the column in
// registers.  Columns are contiguous in memory, so every load and store of a wave
// is one contiguous run.
template <int L1, class PT>
__device__ __forceinline__ void fft_axis1_reg_body(PT P, const int bx)
{
    __shared__ float2 tw[L1];
    for (int i = threadIdx.x; i < L1; i += blockDim.x) tw[i] = ldg2(P.tw1, i);
    __syncthreads();
    const unsigned per_m = (unsigned)P.n2 * (unsigned)P.cols;
    const unsigned g = bx * blockDim.x + threadIdx.x;
    if (g >= per_m * (unsigned)P.M) return;
    const unsigned m = g / per_m, rem = g - m * per_m;
    float2* base = P.X + (size_t)m * L1 * per_m + rem;
    float2 z[L1];
#pragma unroll
    for (int i = 0; i < L1; ++i) z[i] = ldg2(base, (size_t)bit_reverse(i, L1) * per_m);
    fft_reg<L1>(z, tw);
#pragma unroll
    for (int k = 0; k < L1; ++k) stg2(base, (size_t)k * per_m, z[k]);
}

template <int L1>
__global__ __launch_bounds__(256) void k_fft_axis1_reg(Axis1Params P) { fft_axis1_reg_body<L1, Axis1Params>(P, blockIdx.x); }
template <int L1>
__global__ __launch_bounds__(256) void k_fft_axis1_reg_merged(const Axis1Params* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) fft_axis1_reg_body<L1, const Axis1Params&>(tab[d], bx);
}

// One lattice plane R1 of one site, a chunk of kRegFC fields, for power-of-two
// n2 = L2, n3 = L3 <= 32:
//  1. every thread generates the chunk's fields of a few cells (the powers of a
//     p-run are stepped by one factor u_1 each), centred by the FP64 mean, into LDS;
//  2. one thread per (field, row pair) packs two real rows into one complex line and
//     transforms it along axis 3 in registers, then separates the two half spectra;
//  3. one thread per (field, k3) transforms the column along axis 2 in registers and
//     writes it to the spectra (k3 fastest across the wave: contiguous runs).
constexpr int kRegFC = 8, kRegThreads = 128;

template <int L2, int L3, class PT>
__device__ __forceinline__ void fft_planes_reg_body(PT P, const int bx)
{
    constexpr int NH = L3 / 2 + 1;
    constexpr int RP = L3 + 1;                         // real row pitch (floats)
    constexpr int FS = ((L2 * RP + 31) / 32) * 32 + 1; // real field stride: lanes of two fields hit other banks
    constexpr int CP = L2 + 1;                         // complex column pitch
    constexpr int CS = NH * CP;                        // complex field stride
    constexpr int UN = (kRegFC * FS > 2 * kRegFC * CS) ? kRegFC * FS : 2 * kRegFC * CS;   // floats
    __shared__ float2 tw2[L2], tw3[L3];
    __shared__ float buf[UN];
    __shared__ float meanf[kRegFC];

    int b = bx;
    const int fc = b % P.nfchunk; b /= P.nfchunk;
    const int R1 = b % P.n1; b /= P.n1;
    const int mu = b % P.S;
    const int m = b / P.S;
    const int ncell = P.n1 * L2 * L3;
    const int fa = fc * kRegFC;
    const int nfb = min(P.F, fa + kRegFC) - fa;
    for (int i = threadIdx.x; i < L2; i += blockDim.x) tw2[i] = ldg2(P.tw2, i);
    for (int i = threadIdx.x; i < L3; i += blockDim.x) tw3[i] = ldg2(P.tw3, i);
    if (threadIdx.x < nfb) {
        const int f = fa + threadIdx.x;
        const int ep = P.mono[3 * f], eq = P.mono[3 * f + 1], er = P.mono[3 * f + 2];
        const int t = P.kind == 1 ? f : mono_index(ep, eq, er);
        meanf[threadIdx.x] = (float)(gptr(P.sums)[(size_t)(m * P.S + mu) * P.T + t] / (double)ncell);
    }
    __syncthreads();

    // 1. generation.  The thread's cells are loaded together (one memory latency);
    //    the loop over the chunk's fields is uniform, so exponents are scalars and a
    //    field continuing the p-run of the previous one costs one product per cell.
    const size_t plane0 = ((size_t)(m * P.S + mu)) * ncell + (size_t)R1 * L2 * L3;
    static_assert(kRegThreads % L3 == 0, "a thread's cells share r3");
    constexpr int CPT = (L2 * L3 + kRegThreads - 1) / kRegThreads;   // cells per thread
    constexpr int RSTEP = kRegThreads / L3;            // rows between a thread's cells
    const bool gen = threadIdx.x < L2 * L3;           // false only on planes under kRegThreads cells
    float cd[CPT], cu0[CPT], cu1[CPT], cu2[CPT], v[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const size_t c = plane0 + threadIdx.x + k * kRegThreads;
        cd[k] = (gen && P.occ) ? gptr(P.occ)[c] : 1.f;
        cu0[k] = cu1[k] = cu2[k] = 0.f;
        if (gen && P.vec) {
            const auto* u = gptr(P.vec) + 3 * c;
            cu0[k] = u[0]; cu1[k] = u[1]; cu2[k] = u[2];
        }
        v[k] = 1.f;
    }
    float* const dst0 = buf + (threadIdx.x / L3) * RP + threadIdx.x % L3;
    int pe = -1, qe = -1, re = -1;                     // exponents of the previous field
    for (int fb = 0; fb < (gen ? nfb : 0); ++fb) {
        const int f = fa + fb;
        const float mf = meanf[fb];
        float* const dst = dst0 + fb * FS;
        if (P.kind == 1) {
#pragma unroll
            for (int k = 0; k < CPT; ++k)
                dst[k * RSTEP * RP] = (f == 0 ? cu0[k] : f == 1 ? cu1[k] : cu2[k]) * cd[k] - mf;
            continue;
        }
        const int ep = P.mono[3 * f], eq = P.mono[3 * f + 1], er = P.mono[3 * f + 2];
        if (ep == pe + 1 && eq == qe && er == re) {
#pragma unroll
            for (int k = 0; k < CPT; ++k) v[k] *= cu0[k];
        } else {
#pragma unroll
            for (int k = 0; k < CPT; ++k) v[k] = 1.f;
            for (int e = 0; e < ep; ++e)
#pragma unroll
                for (int k = 0; k < CPT; ++k) v[k] *= cu0[k];
            for (int e = 0; e < eq; ++e)
#pragma unroll
                for (int k = 0; k < CPT; ++k) v[k] *= cu1[k];
            for (int e = 0; e < er; ++e)
#pragma unroll
                for (int k = 0; k < CPT; ++k) v[k] *= cu2[k];
        }
        pe = ep; qe = eq; re = er;
#pragma unroll
        for (int k = 0; k < CPT; ++k) dst[k * RSTEP * RP] = v[k] * cd[k] - mf;
    }
    __syncthreads();

    // 2. axis 3: two real rows per complex line, then the two half spectra
    constexpr int NP = L2 / 2;
    const int t = threadIdx.x;
    const int fb3 = t / NP, j = t - fb3 * NP;
    const bool act3 = t < kRegFC * NP && fb3 < nfb;
    float2 z[L3];
    if (act3) {
        const float* r0 = buf + fb3 * FS + (2 * j) * RP;
#pragma unroll
        for (int i = 0; i < L3; ++i) z[i] = make_float2(r0[bit_reverse(i, L3)], r0[RP + bit_reverse(i, L3)]);
        fft_reg<L3>(z, tw3);
    }
    __syncthreads();                      // the real rows are no longer needed
    float2* cb = reinterpret_cast<float2*>(buf);
    if (act3) {
        float2* col = cb + fb3 * CS + 2 * j;
#pragma unroll
        for (int k = 0; k < NH; ++k) {
            const float2 zk = z[k], zm = z[(L3 - k) % L3];
            col[k * CP] = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
            col[k * CP + 1] = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
        }
    }
    __syncthreads();

    // 3. axis 2, written to the spectra
    const int SF = P.S * P.F;
    float2* out = P.X + ((size_t)(m * P.n1 + R1) * L2) * SF * NH + (size_t)(mu * P.F + fa) * NH;
    for (int it = threadIdx.x; it < nfb * NH; it += blockDim.x) {
        const int fb = it / NH, k = it - fb * NH;
        const float2* col = cb + fb * CS + k * CP;
        float2 y[L2];
#pragma unroll
        for (int i = 0; i < L2; ++i) y[i] = col[bit_reverse(i, L2)];
        fft_reg<L2>(y, tw2);
#pragma unroll
        for (int k2 = 0; k2 < L2; ++k2) stg2(out, (size_t)k2 * SF * NH + it, y[k2]);
    }
}

template <int L2, int L3>
__global__ __launch_bounds__(kRegThreads) void k_fft_planes_reg(PlaneParams P) { fft_planes_reg_body<L2, L3, PlaneParams>(P, blockIdx.x); }
template <int L2, int L3>
__global__ __launch_bounds__(kRegThreads) void k_fft_planes_reg_merged(const PlaneParams* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) fft_planes_reg_body<L2, L3, const PlaneParams&>(tab[d], bx);
}

template <int L2, int L3>
static hipError_t launch_planes_reg(const PlaneParams& p, hipStream_t st)
{
    PlaneParams q = p;
    q.fchunk = kRegFC;
    q.nfchunk = (p.F + kRegFC - 1) / kRegFC;
    return dispatch(k_fft_planes_reg<L2, L3>, k_fft_planes_reg_merged<L2, L3>, q.M * q.S * q.n1 * q.nfchunk,
                    kRegThreads, 0, st, q);
}

template <int L2>
static hipError_t launch_planes_reg2(const PlaneParams& p, hipStream_t st)
{
    switch (p.n3) {
        case 8: return launch_planes_reg<L2, 8>(p, st);
        case 16: return launch_planes_reg<L2, 16>(p, st);
        case 32: return launch_planes_reg<L2, 32>(p, st);
        default: return hipErrorInvalidValue;
    }
}

size_t planes_lds_bytes(const PlaneParams& p)
{
    if (p.a3 > 0)
        return sizeof(float2) * (size_t)((p.row_pairs > 0 ? 0 : p.n2) + p.n3 +
                                         p.npl * p.fchunk * (p.buf_elems + (p.row_pairs > 0 ? p.row_pairs : (p.n2 + 1) / 2) * p.lp));
    return sizeof(float2) * (size_t)((p.row_pairs > 0 ? 0 : p.n2) + p.n3 + 2 * (p.npl > 1 ? p.npl : 1) * p.fchunk * p.buf_elems);
}

hipError_t launch_fft_planes(const PlaneParams& p, hipStream_t st)
{
    if (p.a3 == 0 && fft_reg_supported(p.n2) && fft_reg_supported(p.n3)) {
        switch (p.n2) {
            case 8: return launch_planes_reg2<8>(p, st);
            case 16: return launch_planes_reg2<16>(p, st);
            default: return launch_planes_reg2<32>(p, st);
        }
    }
    const size_t lds = planes_lds_bytes(p);
    if (p.a1 > 0 && (p.a1 != p.n1 || p.npl != p.n1 || p.b2 != 1 || p.b3 != 1 || p.n1 > kMaxRegRadix)) return hipErrorInvalidValue;
    if (p.a3 > 0) {
        if (p.a3 > kMaxPlanePrime || p.a2 > kMaxPlanePrime) return hipErrorInvalidValue;
        const int groups = p.row_pairs > 0 ? p.n1 * p.nrchunk : (p.n1 + p.npl - 1) / p.npl;
        if (p.npl < 1 || p.fchunk < 1 || p.fchunk > kPlaneMaxFields || p.threads < 64 || p.threads > 512 || p.a3 * p.b3 != p.n3 ||
            p.lp < p.n3 || (p.row_pairs <= 0 && p.a2 * p.b2 != p.n2))
            return hipErrorInvalidValue;
        const bool big = p.a3 > kMaxRegRadix || (p.row_pairs <= 0 && p.a2 > kMaxRegRadix);
        const auto one = big ? k_plane_regs<true> : k_plane_regs<false>;
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute((const void*)one, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        return dispatch(one, big ? k_plane_regs_merged<true> : k_plane_regs_merged<false>, p.M * p.S * groups * p.nfchunk,
                        p.threads, lds, st, p);
    }
    if (p.row_pairs > 0) {
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute((const void*)k_fft_rows,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        return dispatch(k_fft_rows, k_fft_rows_merged, p.M * p.S * p.n1 * p.nrchunk * p.nfchunk, 256, lds, st, p);
    }
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)k_fft_planes,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (p.npl < 1) return hipErrorInvalidValue;
    return dispatch(k_fft_planes, k_fft_planes_merged, p.M * p.S * ((p.n1 + p.npl - 1) / p.npl) * p.nfchunk, 256, lds,
                    st, p);
}

// ---------------------------------------------------------------------------- axis-1 FFT
template <class PT>
__device__ __forceinline__ void fft_axis1_body(PT P, const int bx)
{
    extern __shared__ float2 smem[];
    float2* tw = smem;
    float2* A = tw + P.n1;
    float2* B = A + P.n1 * P.tc;
    int b = bx;
    const int cb = b % P.ncolblk; b /= P.ncolblk;
    const int k2 = b % P.n2;
    const int m = b / P.n2;
    const int tc = P.tc, n1 = P.n1;
    const int c0 = cb * tc;
    const size_t rowstride = (size_t)P.n2 * P.cols;
    float2* base = P.X + ((size_t)m * n1 * P.n2 + k2) * P.cols + c0;
    for (int i = threadIdx.x; i < n1; i += blockDim.x) tw[i] = ldg2(P.tw1, i);
    for (int b0 = threadIdx.x; b0 < n1 * tc; b0 += 8 * blockDim.x) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = b0 + u * blockDim.x;
            const int R1 = idx / tc, c = idx - R1 * tc;
            v[u] = (idx < n1 * tc && c0 + c < P.cols) ? ldg2(base, R1 * rowstride + c) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = b0 + u * blockDim.x;
            if (idx < n1 * tc) A[idx] = v[u];
        }
    }
    __syncthreads();
    float2* Y = lds_fft(A, B, tc, 1, tc, P.p1, tw);
    for (int idx = threadIdx.x; idx < n1 * tc; idx += blockDim.x) {
        const int k1 = idx / tc, c = idx - k1 * tc;
        if (c0 + c < P.cols) stg2(base, k1 * rowstride + c, Y[idx]);
    }
}

__global__ __launch_bounds__(256) void k_fft_axis1(Axis1Params P) { fft_axis1_body<Axis1Params>(P, blockIdx.x); }
__global__ __launch_bounds__(256) void k_fft_axis1_merged(const Axis1Params* __restrict__ tab, const Slot* __restrict__ slots)
{
    int d, bx;
    if (slot_of(slots, d, bx)) fft_axis1_body<const Axis1Params&>(tab[d], bx);
}

size_t axis1_lds_bytes(const Axis1Params& p)
{
    if (p.a > 0) return p.b > 1 ? sizeof(float2) * (size_t)(p.n1 + p.n1 * p.tc) : 0;
    return sizeof(float2) * (size_t)(p.n1 + 2 * p.n1 * p.tc);
}

hipError_t launch_fft_axis1(const Axis1Params& p, hipStream_t st)
{
    if (fft_reg_supported(p.n1)) {
        const unsigned total = (unsigned)p.M * p.n2 * p.cols;
        const unsigned grid = (total + 255) / 256;
        if (p.n1 == 8) return dispatch(k_fft_axis1_reg<8>, k_fft_axis1_reg_merged<8>, grid, 256, 0, st, p);
        if (p.n1 == 16) return dispatch(k_fft_axis1_reg<16>, k_fft_axis1_reg_merged<16>, grid, 256, 0, st, p);
        return dispatch(k_fft_axis1_reg<32>, k_fft_axis1_reg_merged<32>, grid, 256, 0, st, p);
    }
    const size_t lds = axis1_lds_bytes(p);
    if (p.a > 0) {
        if (p.a * p.b != p.n1) return hipErrorInvalidValue;
        const bool big = p.a > kMaxRegRadix;
        const auto one = big ? k_axis1_regs<true> : k_axis1_regs<false>;
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute((const void*)one, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        const int items = p.tc * (p.b > 1 ? std::max(p.a, p.b) : 1);
        const unsigned threads = std::min(256, (items + 63) / 64 * 64);
        return dispatch(one, big ? k_axis1_regs_merged<true> : k_axis1_regs_merged<false>, p.M * p.n2 * p.ncolblk, threads,
                        lds, st, p);
    }
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)k_fft_axis1,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return dispatch(k_fft_axis1, k_fft_axis1_merged, p.M * p.n2 * p.ncolblk, 256, lds, st, p);
}

}  // namespace dsx
