// Nonstationary Wiener deblurring (appendix D of the paper).
//
// The Hessian is taken as locally translation invariant, hence diagonal in
// the Fourier basis of each local block.  Per block, with F its Fourier
// transform, the regularised inverse eigenvalues are
//   Lambda^-1 = conj(F m_blur) F m_ref / (|F m_blur|^2 + eps)
// and the block's estimate is F^-1 [Lambda^-1 F m_in] (eq. sol); eps is
// eps_rel times the block's largest |F m_blur|^2.  Blocks of `block` nodes
// per axis start every block/2 nodes from -block/2 and are tapered with
// sin^2(pi (u + 1/2) / block) per axis, so every node lies in 2^ndim blocks
// whose tapers add up to one; the estimates are merged with these valences,
// dm = sum_w dm_w / sum_w t_w.
//
// Steps: each image is scaled by its largest magnitude (the filter is
// invariant to the scale of m_ref and m_blur and linear in m_in, and migrated
// images can be small enough for |F m|^2 to leave the FP32 range), a gather
// kernel builds the tapered blocks of the three images (one batch of complex
// arrays), hipFFT transforms them, one workgroup per block forms the filtered
// spectrum, hipFFT transforms back, and a gather kernel merges the 2^ndim
// blocks over each node and restores the scale.
//
// 2D blocks of 16, 32 or 64 nodes take another route: a workgroup carries a
// block from the images to its estimate in LDS (k_w_block), for all images of
// a call at once, and only the estimates go through memory.
#include "common.h"
#include "kernels.h"
#include "wave.h"
#include <hipfft/hipfft.h>

#include <cmath>
#include <vector>

namespace lsrtm {

struct WArgs {
    int n[3];          // image sizes (z, x, y); n[2] = 1 in 2D
    int ndim;
    int B;             // block size per axis
    int K[3];          // blocks per axis
    long long nwin;    // K[0] K[1] K[2]
    long long bs;      // B^ndim
    long long N;       // n[0] n[1] n[2]
    const float* taper;
    const float* scale;  // largest |value| of ref, blur, in
};

constexpr int NPART = 256;

// Images that the LDS route takes per launch, and has room for from its first
// call on (a later call of more images allocates nothing): 16 B per block node,
// where the spectra of one image take 24 in the other route.
constexpr int WIMG = 4;
constexpr int WPART = 64;            // partial maxima per image of that route

struct WienerWork {
    int ndim = 0, n[3] = {0, 0, 0}, block = 0;
    float* est = nullptr;            // [WIMG][nwin][bs] block estimates (LDS route)
    float* part = nullptr;           // [WIMG][3][WPART] partial maxima
    double2* root = nullptr;         // [block] exp(-2 pi i k / block)
    long long nwin = 0, bs = 0;
    hipfftComplex* buf = nullptr;    // [3][nwin][bs]: ref, blur, in spectra
    float* taper = nullptr;          // [block]
    float* scale = nullptr;          // [NPART * 3] partial maxima, then the 3 scales
    hipfftHandle fwd = 0, inv = 0;
    bool plans = false;
};

namespace {

__device__ __forceinline__ void window_origin(const WArgs& a, long long w, int (&o)[3]) {
    const int h = a.B / 2;
    const int wz = (int)(w % a.K[0]);
    const long long r = w / a.K[0];
    const int wx = (int)(r % a.K[1]);
    const int wy = (int)(r / a.K[1]);
    o[0] = wz * h - h;
    o[1] = wx * h - h;
    o[2] = a.ndim == 3 ? wy * h - h : 0;
}

// Largest |value| of the three images: NPART partial maxima per image, then
// one workgroup reduces them into scale[0..2].
__global__ void k_w_maxabs(const float* __restrict__ ref, const float* __restrict__ blur,
                           const float* __restrict__ in, long long n, float* __restrict__ part) {
    __shared__ float red[NTHREADS];
    const float* img = blockIdx.y == 0 ? ref : (blockIdx.y == 1 ? blur : in);
    float m = 0.f;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        m = fmaxf(m, fabsf(img[i]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = NTHREADS / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.y * NPART + blockIdx.x] = red[0];
}

__global__ void k_w_scale(float* __restrict__ part) {
    __shared__ float red[NTHREADS];
    for (int k = 0; k < 3; ++k) {
        red[threadIdx.x] = threadIdx.x < NPART ? part[k * NPART + threadIdx.x] : 0.f;
        __syncthreads();
        for (int s = NTHREADS / 2; s > 0; s >>= 1) {
            if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
            __syncthreads();
        }
        if (threadIdx.x == 0) part[3 * NPART + k] = red[0];
        __syncthreads();
    }
}

__global__ void k_w_extract(WArgs a, const float* __restrict__ ref, const float* __restrict__ blur,
                            const float* __restrict__ in, hipfftComplex* __restrict__ buf) {
    const long long per = a.nwin * a.bs;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < 3 * per;
         e += (long long)gridDim.x * blockDim.x) {
        const int k = (int)(e / per);
        const long long r = e % per;
        const long long w = r / a.bs;
        const long long u = r % a.bs;
        int o[3];
        window_origin(a, w, o);
        const int uz = (int)(u % a.B);
        const int ux = (int)((u / a.B) % a.B);
        const int uy = a.ndim == 3 ? (int)(u / ((long long)a.B * a.B)) : 0;
        const int gz = o[0] + uz, gx = o[1] + ux, gy = o[2] + uy;
        float v = 0.f;
        if ((unsigned)gz < (unsigned)a.n[0] && (unsigned)gx < (unsigned)a.n[1] && (unsigned)gy < (unsigned)a.n[2]) {
            const long long g = gz + (long long)a.n[0] * (gx + (long long)a.n[1] * gy);
            const float* img = k == 0 ? ref : (k == 1 ? blur : in);
            float t = a.taper[uz] * a.taper[ux];
            if (a.ndim == 3) t *= a.taper[uy];
            const float sc = a.scale[k];
            v = sc > 0.f ? t * (img[g] / sc) : 0.f;
        }
        buf[e] = make_hipFloatComplex(v, 0.f);
    }
}

// One workgroup per block: the filtered spectrum Lambda^-1 F m_in / bs (the
// inverse transform is unnormalised) written over F m_ref.  The block's
// F m_blur is first divided by its largest component magnitude beta (blocks
// at the edge of the illumination can hold values whose squares leave the
// FP32 range), which leaves Lambda^-1 beta unchanged:
//   Lambda^-1 = conj(b') F m_ref / (|b'|^2 + eps_rel max |b'|^2) / beta,  b' = F m_blur / beta.
__device__ __forceinline__ float block_max(float v, float* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = NTHREADS / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    const float r = red[0];
    __syncthreads();
    return r;
}

__global__ void k_w_filter(WArgs a, double eps_rel, hipfftComplex* __restrict__ buf) {
    __shared__ float red[NTHREADS];
    const long long w = blockIdx.x;
    hipfftComplex* A = buf + w * a.bs;
    const hipfftComplex* Bh = buf + (a.nwin + w) * a.bs;
    const hipfftComplex* C = buf + (2 * a.nwin + w) * a.bs;
    float m = 0.f;
    for (long long u = threadIdx.x; u < a.bs; u += NTHREADS) {
        const hipfftComplex b = Bh[u];
        m = fmaxf(m, fmaxf(fabsf(b.x), fabsf(b.y)));
    }
    const float beta = block_max(m, red);
    if (!(beta > 0.f)) {
        for (long long u = threadIdx.x; u < a.bs; u += NTHREADS) A[u] = make_hipFloatComplex(0.f, 0.f);
        return;
    }
    const float ib = 1.f / beta;
    float p = 0.f;
    for (long long u = threadIdx.x; u < a.bs; u += NTHREADS) {
        const hipfftComplex b = Bh[u];
        const float bx = b.x * ib, by = b.y * ib;
        p = fmaxf(p, bx * bx + by * by);
    }
    const float eps = (float)(eps_rel * (double)block_max(p, red));
    const float inv_bs = 1.f / (float)a.bs;
    for (long long u = threadIdx.x; u < a.bs; u += NTHREADS) {
        const hipfftComplex b = Bh[u], r = A[u], c = C[u];
        const float bx = b.x * ib, by = b.y * ib;
        const float den = (bx * bx + by * by) + eps;
        // conj(b') r / den / beta
        const float gx = ((bx * r.x + by * r.y) / den) * ib;
        const float gy = ((bx * r.y - by * r.x) / den) * ib;
        // (g c) / bs
        A[u] = make_hipFloatComplex((gx * c.x - gy * c.y) * inv_bs, (gx * c.y + gy * c.x) * inv_bs);
    }
}

__global__ void k_w_merge(WArgs a, const hipfftComplex* __restrict__ bufA, float* __restrict__ out) {
    const int h = a.B / 2;
    for (long long g = blockIdx.x * (long long)blockDim.x + threadIdx.x; g < a.N;
         g += (long long)gridDim.x * blockDim.x) {
        const int c[3] = {(int)(g % a.n[0]), (int)((g / a.n[0]) % a.n[1]),
                          (int)(g / ((long long)a.n[0] * a.n[1]))};
        float num = 0.f, den = 0.f;
        const int ncomb = a.ndim == 3 ? 8 : 4;
        for (int m = 0; m < ncomb; ++m) {
            long long w = 0, u = 0, wstride = 1, ustride = 1;
            float t = 1.f;
            bool ok = true;
            for (int ax = 0; ax < a.ndim; ++ax) {
                // blocks k = c/h and c/h + 1 start at (k - 1) h and cover c
                const int k = c[ax] / h + ((m >> ax) & 1);
                const int loc = c[ax] - (k * h - h);
                ok = ok && k < a.K[ax] && loc >= 0 && loc < a.B;
                w += k * wstride;
                u += loc * ustride;
                wstride *= a.K[ax];
                ustride *= a.B;
                t *= ok ? a.taper[loc] : 0.f;
            }
            if (!ok) continue;
            num += bufA[w * a.bs + u].x;
            den += t;
        }
        // undo the scaling: the filter is linear in m_in and scales as
        // |m_ref| / |m_blur|
        const float sr = a.scale[0], sb = a.scale[1], si = a.scale[2];
        const float back = sb > 0.f ? (sr / sb) * si : 0.f;
        out[g] = den > 0.f ? (num / den) * back : 0.f;
    }
}

// ---------------------------------------------------------------------------
// 2D blocks of B = 16, 32 or 64: one workgroup per block and image
//
// What bounds the general route at common sizes is its launches (seven per
// image, 3 to 10 us each) and the spectra's way through memory (24 B per node
// and transform for data of 4).  Here a block's three real images are
// transformed in LDS, two columns of one image to a complex transform (never
// two images, whose magnitudes can be far apart), filtered and transformed
// back.  Two images of 240 x 737 take 28 us with blocks of 64 and 38 us with
// blocks of 16 (the general route: 168 and 115).
//
// A transform of B = 8 T points runs in T lanes of one wave, 8 points each:
// point n = t + T r, a radix-8 butterfly over r, twiddles w_B^(t k1), an
// exchange through the group's LDS, a radix-T butterfly over t; the lane ends
// with the frequencies (t + T i) + 8 k2.
// The butterflies run in 64 bits, LDS holds 32: the call takes 28 us instead of 26
// with 32-bit butterflies, and its error against 64 bits is 1.6e-7 instead
// of 2.5e-7 (the general route: 2.3e-7; relative L2, blocks of 64).
// ---------------------------------------------------------------------------
template <int B>
struct WShape {
    static constexpr int T = B / 8;                  // lanes of a transform
    static constexpr int H = B / 2 + 1;              // rows of a half spectrum
    static constexpr int LS = B + B / 8;             // stride of a row: the exchange pads every 8
    static constexpr int NT = B == 64 ? 512 : B == 32 ? 256 : 64;
    static constexpr int NG = NT / T;                // transforms at once
};

__device__ __forceinline__ double2 to64(float2 a) { return {(double)a.x, (double)a.y}; }
__device__ __forceinline__ float2 to32(double2 a) { return {(float)a.x, (float)a.y}; }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return {a.x - b.x, a.y - b.y}; }
// times -i (forward) or i (inverse)
template <bool INV>
__device__ __forceinline__ double2 crot(double2 a) {
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}
template <bool INV>
__device__ __forceinline__ double2 cmul(double2 a, double2 w) {   // w conjugated for the inverse
    const double wy = INV ? -w.y : w.y;
    return {fma(a.x, w.x, -a.y * wy), fma(a.x, wy, a.y * w.x)};
}

// Butterflies in place, natural order in and out.
template <bool INV>
__device__ __forceinline__ void fly2(double2* v) {
    const double2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
}
template <bool INV>
__device__ __forceinline__ void fly4(double2* v) {
    const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = crot<INV>(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
}
template <bool INV>
__device__ __forceinline__ void fly8(double2* v) {
    constexpr double r = 0.70710678118654752440;
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    fly4<INV>(e);
    fly4<INV>(o);
    const double2 o1 = cmul<INV>(o[1], make_double2(r, -r)), o2 = crot<INV>(o[2]), o3 = cmul<INV>(o[3], make_double2(-r, -r));
    v[0] = cadd(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[4] = csub(e[0], o[0]);
    v[5] = csub(e[1], o1);
    v[6] = csub(e[2], o2);
    v[7] = csub(e[3], o3);
}

// v[r] = point t + T r in, v[i T + k2] = frequency (t + T i) + 8 k2 out; x is
// the group's LDS row.
template <int B, bool INV>
__device__ __forceinline__ void transform(double2 (&v)[8], float2* x, int t, const double2 (&tw)[8]) {
    constexpr int T = WShape<B>::T;
    fly8<INV>(v);
    wave_order();
#pragma unroll
    for (int k = 0; k < 8; ++k) x[t * 9 + k] = to32(k == 0 ? v[0] : cmul<INV>(v[k], tw[k]));
    wave_order();
#pragma unroll
    for (int i = 0; i < 8 / T; ++i) {
#pragma unroll
        for (int u = 0; u < T; ++u) v[i * T + u] = to64(x[u * 9 + t + T * i]);
        if constexpr (T == 8) fly8<INV>(v + i * T);
        else if constexpr (T == 4) fly4<INV>(v + i * T);
        else fly2<INV>(v + i * T);
    }
    wave_order();
}

// Largest of v over the workgroup.
template <int NT>
__device__ __forceinline__ float group_max(float v, float* red) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v = fmaxf(v, __shfl_xor(v, s));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) v = fmaxf(v, red[i]);
    return v;
}

// Largest |value| of image m of an image triple.
__device__ __forceinline__ float wscale(const float* __restrict__ part, int m) {
    float v = part[m * WPART + (threadIdx.x & 63)];
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v = fmaxf(v, __shfl_xor(v, s));
    return v;
}

__global__ void k_w_part(const float* __restrict__ ref, const float* __restrict__ blur, const float* __restrict__ in,
                         long long n, float* __restrict__ part) {
    __shared__ float red[NTHREADS / 64];
    const int k = blockIdx.y, img = blockIdx.z;
    const float* const f = (k == 0 ? ref : k == 1 ? blur : in) + img * n;
    float m = 0.f;
    for (long long i = blockIdx.x * (long long)NTHREADS + threadIdx.x; i < n; i += (long long)WPART * NTHREADS)
        m = fmaxf(m, fabsf(f[i]));
    m = group_max<NTHREADS>(m, red);
    if (threadIdx.x == 0) part[(img * 3 + k) * WPART + blockIdx.x] = m;
}

// IN: m_in is an image of its own (otherwise it is m_ref).
template <int B, bool IN>
__global__ void __launch_bounds__(WShape<B>::NT)
k_w_block(WArgs a, double eps_rel, const float* __restrict__ ref, const float* __restrict__ blur,
          const float* __restrict__ in, const double2* __restrict__ root, const float* __restrict__ part,
          float* __restrict__ est) {
    using W = WShape<B>;
    constexpr int T = W::T, H = W::H, LS = W::LS, NT = W::NT, NG = W::NG, M = IN ? 3 : 2;
    __shared__ __align__(16) float2 spec[M][H][LS];   // half spectra, rows of constant k_z
    __shared__ float2 work[NG][LS];
    __shared__ float red[NT / 64], taper[B];
    const int t = threadIdx.x % T, gr = threadIdx.x / T;
    const int oz = (int)(blockIdx.x % a.K[0]) * (B / 2) - B / 2, ox = (int)(blockIdx.x / a.K[0]) * (B / 2) - B / 2;
    part += blockIdx.y * 3 * WPART;
    est += ((long long)blockIdx.y * a.nwin + blockIdx.x) * (B * B);
    float scale[M];
#pragma unroll
    for (int m = 0; m < M; ++m) scale[m] = wscale(part, m);
    for (int i = threadIdx.x; i < B; i += NT) taper[i] = a.taper[i];
    double2 tw[8], v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) tw[k] = root[t * k];
    __syncthreads();
    // along z: columns 2 j and 2 j + 1 of an image as one complex transform
    for (int f = gr; f < M * (B / 2); f += NG) {
        const int m = f / (B / 2), j = f % (B / 2), gx = ox + 2 * j;
        const float sc = m == 0 ? scale[0] : m == 1 ? scale[1] : scale[M - 1];
        const float* const img = (m == 0 ? ref : m == 1 ? blur : in) + blockIdx.y * a.N;
        const float* const c0 = img + (long long)gx * a.n[0];
        const bool x0 = (unsigned)gx < (unsigned)a.n[1], x1 = (unsigned)(gx + 1) < (unsigned)a.n[1];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int uz = t + T * r, gz = oz + uz;
            const bool z = (unsigned)gz < (unsigned)a.n[0] && sc > 0.f;
            v[r].x = z && x0 ? taper[uz] * taper[2 * j] * (c0[gz] / sc) : 0.f;
            v[r].y = z && x1 ? taper[uz] * taper[2 * j + 1] * (c0[gz + a.n[0]] / sc) : 0.f;
        }
        float2* const x = work[gr];
        transform<B, false>(v, x, t, tw);
#pragma unroll
        for (int i = 0; i < 8 / T; ++i)
#pragma unroll
            for (int k2 = 0; k2 < T; ++k2) x[(t + T * i) + 8 * k2] = to32(v[i * T + k2]);
        wave_order();
        for (int k = t; k < H; k += T) {
            const float2 p = x[k], q = x[(B - k) % B];   // Z(k), Z(-k)
            *reinterpret_cast<float4*>(&spec[m][k][2 * j]) =
                make_float4(0.5f * (p.x + q.x), 0.5f * (p.y - q.y), 0.5f * (p.y + q.y), 0.5f * (q.x - p.x));
        }
        wave_order();
    }
    __syncthreads();
    // along x, in place
    for (int f = gr; f < M * H; f += NG) {
        float2* const x = spec[f / H][f % H];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = to64(x[t + T * r]);
        transform<B, false>(v, x, t, tw);
#pragma unroll
        for (int i = 0; i < 8 / T; ++i)
#pragma unroll
            for (int k2 = 0; k2 < T; ++k2) x[(t + T * i) + 8 * k2] = to32(v[i * T + k2]);
    }
    __syncthreads();
    // the filter, as in k_w_filter; a half spectrum has every magnitude.  A NaN in
    // the block leaves no number in the spectra of these sizes there, and the
    // estimate is zero; here two columns share a transform, which leaves a few, so
    // it is looked for
    float mx = 0.f;
    for (int u = threadIdx.x; u < H * B; u += NT) {
        const float2 b = spec[1][u / B][u % B];
        mx = fmaxf(mx, b.x != b.x || b.y != b.y ? INFINITY : fmaxf(fabsf(b.x), fabsf(b.y)));
    }
    const float beta = group_max<NT>(mx, red);
    if (!(beta > 0.f && beta < INFINITY)) {
        for (int u = threadIdx.x; u < B * B; u += NT) est[u] = 0.f;
        return;
    }
    const float ib = 1.f / beta;
    float pw = 0.f;
    for (int u = threadIdx.x; u < H * B; u += NT) {
        const float2 b = spec[1][u / B][u % B];
        const float bx = b.x * ib, by = b.y * ib;
        pw = fmaxf(pw, bx * bx + by * by);
    }
    const float eps = (float)(eps_rel * (double)group_max<NT>(pw, red));
    const float inv_bs = 1.f / (float)(B * B);
    for (int u = threadIdx.x; u < H * B; u += NT) {
        const float2 b = spec[1][u / B][u % B], r = spec[0][u / B][u % B], c = spec[IN ? M - 1 : 0][u / B][u % B];
        const float bx = b.x * ib, by = b.y * ib;
        const float den = (bx * bx + by * by) + eps;
        const float gx = ((bx * r.x + by * r.y) / den) * ib;
        const float gy = ((bx * r.y - by * r.x) / den) * ib;
        spec[0][u / B][u % B] = {(gx * c.x - gy * c.y) * inv_bs, (gx * c.y + gy * c.x) * inv_bs};
    }
    __syncthreads();
    for (int f = gr; f < H; f += NG) {
        float2* const x = spec[0][f];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = to64(x[t + T * r]);
        transform<B, true>(v, x, t, tw);
#pragma unroll
        for (int i = 0; i < 8 / T; ++i)
#pragma unroll
            for (int k2 = 0; k2 < T; ++k2) x[(t + T * i) + 8 * k2] = to32(v[i * T + k2]);
    }
    __syncthreads();
    for (int j = gr; j < B / 2; j += NG) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int k = t + T * r;
            const float4 s = *reinterpret_cast<const float4*>(&spec[0][k < H ? k : B - k][2 * j]);
            // the rows 0 and B / 2 are their own conjugates: their values are real
            const double sg = k == 0 || k == B / 2 ? 0.0 : k < H ? 1.0 : -1.0;
            v[r] = {s.x - sg * s.w, sg * s.y + s.z};
        }
        transform<B, true>(v, work[gr], t, tw);
#pragma unroll
        for (int i = 0; i < 8 / T; ++i)
#pragma unroll
            for (int k2 = 0; k2 < T; ++k2) {
                const int uz = (t + T * i) + 8 * k2;
                est[2 * j * B + uz] = (float)v[i * T + k2].x;
                est[(2 * j + 1) * B + uz] = (float)v[i * T + k2].y;
            }
    }
}

// One column of one image per workgroup: k_w_merge's sums, in its order.
__global__ void k_w_merge2(WArgs a, int own_in, const float* __restrict__ part, const float* __restrict__ est,
                           float* __restrict__ out) {
    const int gx = blockIdx.x, h = a.B / 2;
    part += blockIdx.y * 3 * WPART;
    est += (long long)blockIdx.y * a.nwin * a.bs;
    out += blockIdx.y * a.N + (long long)gx * a.n[0];
    const float sr = wscale(part, 0), sb = wscale(part, 1), si = own_in ? wscale(part, 2) : sr;
    const float back = sb > 0.f ? (sr / sb) * si : 0.f;
    const int kx = gx / h, lx = gx - (kx - 1) * h;
    for (int gz = threadIdx.x; gz < a.n[0]; gz += NTHREADS) {
        const int kz = gz / h, lz = gz - (kz - 1) * h;
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int wz = kz + (m & 1), wx = kx + (m >> 1), uz = lz - (m & 1) * h, ux = lx - (m >> 1) * h;
            if (wz >= a.K[0] || wx >= a.K[1]) continue;
            num += est[((long long)wx * a.K[0] + wz) * a.bs + ux * a.B + uz];
            den += a.taper[uz] * a.taper[ux];
        }
        out[gz] = den > 0.f ? (num / den) * back : 0.f;
    }
}

template <int B>
void launch_block(const WArgs& a, double eps_rel, const float* ref, const float* blur, const float* in, int nimg,
                  const WienerWork* W, hipStream_t st) {
    const dim3 grid((unsigned)a.nwin, nimg);
    if (in == ref) k_w_block<B, false><<<grid, WShape<B>::NT, 0, st>>>(a, eps_rel, ref, blur, in, W->root, W->part, W->est);
    else k_w_block<B, true><<<grid, WShape<B>::NT, 0, st>>>(a, eps_rel, ref, blur, in, W->root, W->part, W->est);
}

int grid_of(long long n) {
    long long b = (n + NTHREADS - 1) / NTHREADS;
    return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

}  // namespace

void wiener_free(WienerWork* w) {
    if (!w) return;
    if (w->plans) {
        (void)hipfftDestroy(w->fwd);
        (void)hipfftDestroy(w->inv);
    }
    if (w->buf) (void)hipFree(w->buf);
    if (w->est) (void)hipFree(w->est);
    if (w->part) (void)hipFree(w->part);
    if (w->root) (void)hipFree(w->root);
    if (w->taper) (void)hipFree(w->taper);
    if (w->scale) (void)hipFree(w->scale);
    delete w;
}

const char* wiener_apply(WienerWork** work, int ndim, const int n[3], int block, double eps_rel,
                         const float* ref, const float* blur, const float* in, int nimg, float* out,
                         hipStream_t st) {
    if (block < 2 || (block & 1)) return "block must be even and >= 2";
    if (!(eps_rel >= 0.0)) return "eps_rel must be >= 0";
    WienerWork* W = *work;
    // lanes of a wave per transform, whole waves per workgroup: 16, 32, 64
    const bool in_lds = ndim == 2 && (block == 16 || block == 32 || block == 64);
    const bool same = W && W->ndim == ndim && W->block == block && W->n[0] == n[0] && W->n[1] == n[1] &&
                      W->n[2] == n[2];
    if (!same) {
        wiener_free(W);
        W = new WienerWork();
        *work = W;
        W->ndim = ndim;
        for (int a = 0; a < 3; ++a) W->n[a] = n[a];
        const int h = block / 2;
        W->nwin = 1;
        W->bs = 1;
        for (int a = 0; a < ndim; ++a) {
            W->nwin *= (n[a] - 1) / h + 2;
            W->bs *= block;
        }
        if (hipMalloc(&W->taper, block * sizeof(float)) != hipSuccess) return "out of memory";
        std::vector<float> t(block);
        for (int u = 0; u < block; ++u) {
            const double s = std::sin(M_PI * (u + 0.5) / block);
            t[u] = (float)(s * s);
        }
        if (hipMemcpy(W->taper, t.data(), block * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
            return "taper upload failed";
        if (in_lds) {
            if (hipMalloc(&W->part, WIMG * 3 * WPART * sizeof(float)) != hipSuccess) return "out of memory";
            if (hipMalloc(&W->root, block * sizeof(double2)) != hipSuccess) return "out of memory";
            if (hipMalloc(&W->est, WIMG * W->nwin * W->bs * sizeof(float)) != hipSuccess) return "out of memory";
            std::vector<double2> r(block);
            for (int k = 0; k < block; ++k)
                r[k] = {std::cos(2.0 * M_PI * k / block), -std::sin(2.0 * M_PI * k / block)};
            if (hipMemcpy(W->root, r.data(), block * sizeof(double2), hipMemcpyHostToDevice) != hipSuccess)
                return "twiddle upload failed";
        } else {
            if (hipMalloc(&W->buf, 3 * W->nwin * W->bs * sizeof(hipfftComplex)) != hipSuccess) return "out of memory";
            if (hipMalloc(&W->scale, (3 * NPART + 3) * sizeof(float)) != hipSuccess) return "out of memory";
            int dims[3] = {block, block, block};
            if (hipfftPlanMany(&W->fwd, ndim, dims, nullptr, 1, (int)W->bs, nullptr, 1, (int)W->bs, HIPFFT_C2C,
                               (int)(3 * W->nwin)) != HIPFFT_SUCCESS)
                return "hipfftPlanMany (forward) failed";
            if (hipfftPlanMany(&W->inv, ndim, dims, nullptr, 1, (int)W->bs, nullptr, 1, (int)W->bs, HIPFFT_C2C,
                               (int)W->nwin) != HIPFFT_SUCCESS) {
                (void)hipfftDestroy(W->fwd);
                return "hipfftPlanMany (inverse) failed";
            }
            W->plans = true;
        }
        W->block = block;            // complete: a later call may take it
    }
    WArgs a;
    for (int ax = 0; ax < 3; ++ax) {
        a.n[ax] = n[ax];
        a.K[ax] = ax < ndim ? (n[ax] - 1) / (block / 2) + 2 : 1;
    }
    a.ndim = ndim;
    a.B = block;
    a.nwin = W->nwin;
    a.bs = W->bs;
    a.N = (long long)n[0] * n[1] * n[2];
    a.taper = W->taper;
    if (in_lds) {
        for (int k = 0; k < nimg; k += WIMG) {
            const int m = nimg - k < WIMG ? nimg - k : WIMG;
            const float *r = ref + k * a.N, *b = blur + k * a.N, *x = in + k * a.N;
            k_w_part<<<dim3(WPART, in == ref ? 2 : 3, m), NTHREADS, 0, st>>>(r, b, x, a.N, W->part);
            if (block == 64) launch_block<64>(a, eps_rel, r, b, x, m, W, st);
            else if (block == 32) launch_block<32>(a, eps_rel, r, b, x, m, W, st);
            else launch_block<16>(a, eps_rel, r, b, x, m, W, st);
            k_w_merge2<<<dim3(n[1], m), NTHREADS, 0, st>>>(a, in != ref, W->part, W->est, out + k * a.N);
            if (hipGetLastError() != hipSuccess) return "block kernels failed";
        }
        return nullptr;
    }
    a.scale = W->scale + 3 * NPART;
    if (hipfftSetStream(W->fwd, st) != HIPFFT_SUCCESS || hipfftSetStream(W->inv, st) != HIPFFT_SUCCESS)
        return "hipfftSetStream failed";
    for (int k = 0; k < nimg; ++k) {
        const long long off = k * a.N;
        k_w_maxabs<<<dim3(NPART, 3), NTHREADS, 0, st>>>(ref + off, blur + off, in + off, a.N, W->scale);
        k_w_scale<<<1, NTHREADS, 0, st>>>(W->scale);
        if (hipGetLastError() != hipSuccess) return "scale kernels failed";
        k_w_extract<<<grid_of(3 * a.nwin * a.bs), NTHREADS, 0, st>>>(a, ref + off, blur + off, in + off, W->buf);
        if (hipGetLastError() != hipSuccess) return "extract kernel failed";
        if (hipfftExecC2C(W->fwd, W->buf, W->buf, HIPFFT_FORWARD) != HIPFFT_SUCCESS) return "forward FFT failed";
        k_w_filter<<<(int)a.nwin, NTHREADS, 0, st>>>(a, eps_rel, W->buf);
        if (hipGetLastError() != hipSuccess) return "filter kernel failed";
        if (hipfftExecC2C(W->inv, W->buf, W->buf, HIPFFT_BACKWARD) != HIPFFT_SUCCESS) return "inverse FFT failed";
        k_w_merge<<<grid_of(a.N), NTHREADS, 0, st>>>(a, W->buf, out + off);
        if (hipGetLastError() != hipSuccess) return "merge kernel failed";
    }
    return nullptr;
}

}  // namespace lsrtm
