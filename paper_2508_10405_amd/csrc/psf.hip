// Interpolated point-spread-function Hessian (appendix C of the paper) for
// image-domain LSRTM (section 3, eq. migdeconobj).
//
// PSF images P[q][p] (response in parameter p to the scatterer lattice of
// parameter q, computed by one Born and one migration pass) sample columns of
// H = L^T L.  Column j of block (p, q) is the window |o_a| <= W of the PSF
// images around the lattice corners c of j, shifted to j and weighted with
// the multilinear weights of j between its corners (eq. trilinear; bilinear
// in 2D):  H_pq[j + o, j] = sum_c w_c(j) P[q][p][c + o], where j + o and c + o
// lie in the grid.  Per axis, the corners and the weight of every coordinate
// come from a small table (c0, c1, w) built on the host.
//
// Both products are gathers over the window of one output point (one thread
// per point, FP32 accumulation in a fixed order):
//   y = H x   : y_p[i] = sum_o sum_q x_q[i - o] sum_c w_c(i - o) P[q][p][c(i - o) + o]
//   y = H^T x : y_q[j] = sum_o sum_p x_p[j + o] sum_c w_c(j) P[q][p][c(j) + o]
// mono = 1 keeps the lnIp block (vectors of one parameter).
//
// 2D products (k_psf_t, k_psf_f) take the sums in another order, corner by
// corner: the window of a corner is the same for every point it serves, so a
// tap costs one fused multiply-add per block with a factor that the whole wave
// shares (scalar loads of the windows, packed by k_psf_pack with zeros outside
// the grid) instead of four table look-ups and four gathered images:
//   H^T: y_q[j] = sum over the 4 corners c of j of w_c(j) (sum_o sum_p P[q][p][c + o] x_p[j + o])
//   H  : y_p[i] = sum over the corners c near i of sum_o sum_q P[q][p][c + o] (w_c x_q)[i - o]
// What bounds them is the multiply-adds: 361 taps x 4 corners x 4 blocks per
// point for H^T at spacing 20; H visits 9 corners, with the taps that a piece
// of outputs cannot use left out.  The gathers stay for 3D, for windows whose
// patch of x does not fit in LDS and for spacings below 5, whose windows of 1 or
// 9 taps leave nothing to share (calls of H and H^T with both parameters, gathers
// and corners: 500 x 1000 at spacing 4 97 and 98 us against 117 and 133, 40 x 52 46
// against 46; at spacing 5 and its 25 taps the corners win on every grid timed,
// 20 x 30 to 500 x 1000).  Measured
// on 240 x 737, both parameters, H and H^T: spacing 20 1258 and 1231 -> 146 and
// 122 us, 12 438 and 427 -> 75 and 49, 6 109 and 105 -> 43 and 26.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "wave.h"

namespace lsrtm {

namespace {

// Corners and weight of coordinate j along axis a.
struct Cell {
    int c0, c1;
    float w;
};

__device__ __forceinline__ Cell cell_of(const PsfArgs& a, int ax, int j) {
    const int* t = a.tab + 3 * a.off[ax];
    Cell c;
    c.c0 = t[3 * j];
    c.c1 = t[3 * j + 1];
    c.w = __int_as_float(t[3 * j + 2]);
    return c;
}

// Sum over the 2^ndim corners of w_c * P[q][p][c + o] for the blocks in use;
// out[p][q] (mono: out[0][0] is the lnIp block).
__device__ __forceinline__ void corner_sum(const PsfArgs& a, const Cell (&cl)[3], int oz, int ox, int oy,
                                           float (&out)[2][2]) {
    const int nb = a.mono ? 1 : 2;
    for (int p = 0; p < 2; ++p)
        for (int q = 0; q < 2; ++q) out[p][q] = 0.f;
    const int ncorner = a.ndim == 3 ? 8 : 4;
    for (int m = 0; m < ncorner; ++m) {
        const int bz = m & 1, bx = (m >> 1) & 1, by = (m >> 2) & 1;
        const float wz = bz ? cl[0].w : 1.f - cl[0].w;
        const float wx = bx ? cl[1].w : 1.f - cl[1].w;
        const float wy = a.ndim == 3 ? (by ? cl[2].w : 1.f - cl[2].w) : 1.f;
        const float wgt = (wz * wx) * wy;
        if (wgt == 0.f) continue;
        const int sz = (bz ? cl[0].c1 : cl[0].c0) + oz;
        const int sx = (bx ? cl[1].c1 : cl[1].c0) + ox;
        const int sy = a.ndim == 3 ? (by ? cl[2].c1 : cl[2].c0) + oy : 0;
        if ((unsigned)sz >= (unsigned)a.n[0] || (unsigned)sx >= (unsigned)a.n[1] ||
            (unsigned)sy >= (unsigned)a.n[2])
            continue;
        const long long s = sz + (long long)a.n[0] * (sx + (long long)a.n[1] * sy);
        for (int p = 0; p < nb; ++p)
            for (int q = 0; q < nb; ++q) {
                // blocks stored [q][p][N]; mono reads the (1, 1) block
                const int qq = a.mono ? 1 : q, pp = a.mono ? 1 : p;
                out[p][q] = fmaf(wgt, a.psf[((long long)qq * 2 + pp) * a.N + s], out[p][q]);
            }
    }
}

// One output point of H x or H^T x by gathers: acc[v], v < 1 (mono) or 2.
__device__ __forceinline__ void gather_point(const PsfArgs& a, const float* __restrict__ x, int transpose, int iz, int ix,
                                             int iy, float (&acc)[2]) {
    const int nb = a.mono ? 1 : 2;
    const int Wy = a.ndim == 3 ? a.W : 0;
    Cell cl[3];
    if (transpose) {
        cl[0] = cell_of(a, 0, iz);
        cl[1] = cell_of(a, 1, ix);
        cl[2] = a.ndim == 3 ? cell_of(a, 2, iy) : Cell{0, 0, 0.f};
    }
    for (int oy = -Wy; oy <= Wy; ++oy)
        for (int ox = -a.W; ox <= a.W; ++ox)
            for (int oz = -a.W; oz <= a.W; ++oz) {
                // forward: source point j = i - o; transpose: partner i + o
                const int sgn = transpose ? 1 : -1;
                const int jz = iz + sgn * oz, jx = ix + sgn * ox, jy = iy + sgn * oy;
                if ((unsigned)jz >= (unsigned)a.n[0] || (unsigned)jx >= (unsigned)a.n[1] ||
                    (unsigned)jy >= (unsigned)a.n[2])
                    continue;
                if (!transpose) {
                    cl[0] = cell_of(a, 0, jz);
                    cl[1] = cell_of(a, 1, jx);
                    cl[2] = a.ndim == 3 ? cell_of(a, 2, jy) : Cell{0, 0, 0.f};
                }
                float hs[2][2];
                corner_sum(a, cl, oz, ox, oy, hs);
                const long long jl = jz + (long long)a.n[0] * (jx + (long long)a.n[1] * jy);
                for (int u = 0; u < nb; ++u) {
                    const float xv = x[u * a.N + jl];
                    for (int v = 0; v < nb; ++v) {
                        // forward: y_p += H_pq x_q (u = q, v = p);
                        // transpose: y_q += H_pq x_p (u = p, v = q)
                        const float hv = transpose ? hs[u][v] : hs[v][u];
                        acc[v] = fmaf(hv, xv, acc[v]);
                    }
                }
            }
}

__global__ void k_psf_apply(PsfArgs a, const float* __restrict__ x, float* __restrict__ y, int transpose) {
    const int nb = a.mono ? 1 : 2;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < a.N;
         i += (long long)gridDim.x * blockDim.x) {
        const long long r = i / a.n[0];
        float acc[2] = {0.f, 0.f};
        gather_point(a, x, transpose, (int)(i % a.n[0]), (int)(r % a.n[1]), (int)(r / a.n[1]), acc);
        for (int v = 0; v < nb; ++v) y[v * a.N + i] = acc[v];
    }
}

constexpr int PSF_WAVES = 3;

// Corner windows packed as [corner][ox][oz][block], corner = kx Kz + kz, the
// blocks (q, p) of one tap together, zero where c + o lies outside the grid.
// A sample that is no finite number is noted under the number of this packing.
__global__ void k_psf_pack(Psf2Args a) {
    const int D = 2 * a.W + 1, nb = a.mono ? 1 : 4;
    bool finite = true;
    const long long n = (long long)a.K[0] * a.K[1] * D * D * nb;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const int m = a.mono ? 3 : (int)(e % nb);            // block q * 2 + p
        long long r = e / nb;
        const int oz = (int)(r % D);
        r /= D;
        const int ox = (int)(r % D), k = (int)(r / D);
        const int z = (k % a.K[0]) * a.s + oz, x = (k / a.K[0]) * a.s + ox;   // c - W = k s
        const float f = z < a.n[0] && x < a.n[1] ? a.psf[m * a.N + (z + (long long)a.n[0] * x)] : 0.f;
        a.pack[e] = f;
        finite = finite && isfinite(f);
    }
    if (!finite) atomicMax(a.bad, a.packing);
}

// The corner sums multiply samples by weights and by staged values that are
// zero where the definition leaves the term out, which is the same only for
// finite samples.  With any other among the samples, a block serves its piece
// (lz x lx points from (z0, x0)) by gathers.
__device__ __forceinline__ void gather_piece(const Psf2Args& a, const float* __restrict__ x, float* __restrict__ y,
                                             int transpose, int z0, int lz, int x0, int lx) {
    PsfArgs g;
    g.ndim = 2;
    g.W = a.W;
    g.mono = a.mono;
    g.N = a.N;
    g.tab = a.tab;
    g.psf = a.psf;
    for (int ax = 0; ax < 3; ++ax) {
        g.n[ax] = ax < 2 ? a.n[ax] : 1;
        g.off[ax] = ax < 2 ? a.off[ax] : 0;
    }
    for (int e = threadIdx.x; e < lz * lx; e += blockDim.x) {
        const int z = z0 + e % lz, c = x0 + e / lz;
        float acc[2] = {0.f, 0.f};
        gather_point(g, x, transpose, z, c, 0, acc);
        for (int v = 0; v < (a.mono ? 1 : 2); ++v) y[v * a.N + z + (long long)a.n[0] * c] = acc[v];
    }
}

// Weight of corner k of an axis at coordinate j (0 outside its support).
__device__ __forceinline__ float hat(const int* t, int j, int c) {
    const int c0 = t[3 * j], c1 = t[3 * j + 1];
    const float w = __int_as_float(t[3 * j + 2]);
    return c0 == c ? 1.f - w : c1 == c ? w : 0.f;
}

// y = H^T x: a block serves a piece of one cell of the lattice (all its points
// have the same corners), two rows of z per thread.  The columns of the window
// are dealt to SPLIT groups of threads, whose sums are added through LDS.
template <int NB, int SPLIT>
__global__ void __launch_bounds__(SPLIT * NTHREADS) k_psf_t(Psf2Args a, const float* __restrict__ pack,
                                                    const float* __restrict__ x, float* __restrict__ y) {
    extern __shared__ float xs[];
    const int W = a.W, D = 2 * W + 1;
    const int4 sz = a.tz[blockIdx.x % a.ntz], sx = a.tx[blockIdx.x / a.ntz];   // (start, length, corner, corner)
    const int lz = sz.y, lx = sx.y, pz = lz + 2 * W + 1, px = lx + 2 * W;
    const int bad = *a.bad;
    for (int e = threadIdx.x; e < pz * px; e += SPLIT * NTHREADS) {
        const int jz = sz.x - W + e % pz, jx = sx.x - W + e / pz;
        const bool in = (unsigned)jz < (unsigned)a.n[0] && (unsigned)jx < (unsigned)a.n[1];
#pragma unroll
        for (int p = 0; p < NB; ++p) xs[p * pz * px + e] = in ? x[p * a.N + jz + (long long)a.n[0] * jx] : 0.f;
    }
    __syncthreads();
    const long long win = (long long)D * D * NB * NB;
    const float* P[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) P[c] = pack + ((long long)(c & 2 ? sx.w : sx.z) * a.K[0] + (c & 1 ? sz.w : sz.z)) * win;
    const int np = (lz + 1) / 2;
    const int group = SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NTHREADS) : 0;
    float* const sum = xs + NB * pz * px + threadIdx.x % NTHREADS;   // [SPLIT - 1][NB][2][NTHREADS]
    for (int t0 = 0; t0 < np * lx; t0 += NTHREADS) {
        const int t = t0 + threadIdx.x % NTHREADS;
        const bool on = t < np * lx;
        const int z = on ? 2 * (t % np) : 0, col = on ? t / np : 0;
        float acc[4][NB][2] = {};
        for (int ox = D * group / SPLIT; ox < D * (group + 1) / SPLIT; ++ox) {
            const float* row = xs + (col + ox) * pz + z;
            float xv[NB][2];
#pragma unroll
            for (int p = 0; p < NB; ++p) xv[p][1] = row[p * pz * px];
            const int o0 = ox * D * NB * NB;
#pragma unroll 4
            for (int oz = 0; oz < D; ++oz) {
#pragma unroll
                for (int p = 0; p < NB; ++p) {
                    xv[p][0] = xv[p][1];
                    xv[p][1] = row[p * pz * px + oz + 1];
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int q = 0; q < NB; ++q)
#pragma unroll
                        for (int p = 0; p < NB; ++p) {
                            const float f = P[c][o0 + (oz * NB + q) * NB + p];
                            acc[c][q][0] = fmaf(f, xv[p][0], acc[c][q][0]);
                            acc[c][q][1] = fmaf(f, xv[p][1], acc[c][q][1]);
                        }
            }
        }
        const int jx = sx.x + col;
        const float wx1 = sx.w != sx.z ? __int_as_float(a.tab[3 * (a.off[1] + jx) + 2]) : 0.f;
        float v[NB][2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int jz = min(sz.x + z + r, a.n[0] - 1);
            const float wz1 = sz.w != sz.z ? __int_as_float(a.tab[3 * (a.off[0] + jz) + 2]) : 0.f;
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                v[q][r] = 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    v[q][r] = fmaf((c & 2 ? wx1 : 1.f - wx1) * (c & 1 ? wz1 : 1.f - wz1), acc[c][q][r], v[q][r]);
                if (group > 0) sum[((group - 1) * NB + q) * 2 * NTHREADS + r * NTHREADS] = v[q][r];
            }
        }
        if (SPLIT > 1) __syncthreads();
        if (group == 0 && on)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int q = 0; q < NB; ++q) {
#pragma unroll
                    for (int g = 1; g < SPLIT; ++g)
                        v[q][r] = v[q][r] + sum[((g - 1) * NB + q) * 2 * NTHREADS + r * NTHREADS];
                    if (z + r < lz) y[q * a.N + sz.x + z + r + (long long)a.n[0] * jx] = v[q][r];
                }
        if (SPLIT > 1) __syncthreads();
    }
    if (bad >= a.packing) {
        __syncthreads();                                     // over the outputs just stored
        gather_piece(a, x, y, 1, sz.x, lz, sx.x, lx);
    }
}

// y = H x: a block serves a piece of outputs, two rows of z per thread, and
// visits the corners whose support its windows reach; its waves take the
// corners' columns in turn and add their sums through LDS.
template <int NB>
__global__ void __launch_bounds__(64 * PSF_WAVES) k_psf_f(Psf2Args a, const float* __restrict__ pack,
                                              const float* __restrict__ x, float* __restrict__ y) {
    extern __shared__ float lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float* const xs = lds + wave * (int)(a.lds_f / sizeof(float)) * NB;
    constexpr int CH = 2;                                    // passes over the piece (at most 128 pairs)
    const int W = a.W, D = 2 * W + 1;
    const int4 sz = a.fz[blockIdx.x % a.nfz], sx = a.fx[blockIdx.x / a.nfz];   // (start, length, corners first .. last)
    const int lz = sz.y, lx = sx.y, np = (lz + 1) / 2;
    const int *tz = a.tab + 3 * a.off[0], *tx = a.tab + 3 * a.off[1];
    const int bad = *a.bad;
    float acc[CH][NB][2] = {};
    // points a corner serves on an axis
    auto lo = [&](int k) { return k == 0 ? 0 : W + (k - 1) * a.s + 1; };
    auto hi = [&](int k, int ax) { return k == a.K[ax] - 1 ? a.n[ax] - 1 : W + (k + 1) * a.s - 1; };
    for (int kx = sx.z + wave; kx <= sx.w; kx += PSF_WAVES) {
        const int xa = max(-W, sx.x - hi(kx, 1)), xb = min(W, sx.x + lx - 1 - lo(kx));
        for (int kz = sz.z; kz <= sz.w; ++kz) {
            const int za = max(-W, sz.x - hi(kz, 0)), zb = min(W, sz.x + lz - 1 - lo(kz));
            if (xa > xb || za > zb) continue;
            wave_order();                                    // the taps of the corner before have been read
            // w_c x on the points that these taps reach
            const int pz = lz + zb - za + 1, px = lx + xb - xa;
            for (int e = lane; e < pz * px; e += 64) {
                const int jz = sz.x - zb + e % pz, jx = sx.x - xb + e / pz;
                const bool in = (unsigned)jz < (unsigned)a.n[0] && (unsigned)jx < (unsigned)a.n[1];
                const float w = in ? hat(tz, jz, W + kz * a.s) * hat(tx, jx, W + kx * a.s) : 0.f;
#pragma unroll
                for (int q = 0; q < NB; ++q)
                    xs[q * pz * px + e] = w != 0.f ? w * x[q * a.N + jz + (long long)a.n[0] * jx] : 0.f;
            }
            wave_order();                                    // the wave's own patch: no other wave reads it
            const float* P = pack + ((long long)kx * a.K[0] + kz) * D * D * NB * NB;
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) {
                const int t = lane + 64 * ch;
                if (64 * ch >= np * lx) break;
                const int tt = min(t, np * lx - 1), z = 2 * (tt % np), col = tt / np;
                for (int ox = xa; ox <= xb; ++ox) {
                    const float* row = xs + (col + xb - ox) * pz + z + zb;
                    const int o0 = (ox + W) * D + W;
                    float xv[NB][2];
#pragma unroll
                    for (int q = 0; q < NB; ++q) xv[q][0] = row[q * pz * px - za + 1];
#pragma unroll 4
                    for (int oz = za; oz <= zb; ++oz) {
#pragma unroll
                        for (int q = 0; q < NB; ++q) {
                            xv[q][1] = xv[q][0];
                            xv[q][0] = row[q * pz * px - oz];
                        }
#pragma unroll
                        for (int q = 0; q < NB; ++q)
#pragma unroll
                            for (int p = 0; p < NB; ++p) {
                                const float f = P[((o0 + oz) * NB + q) * NB + p];
                                acc[ch][p][0] = fmaf(f, xv[q][0], acc[ch][p][0]);
                                acc[ch][p][1] = fmaf(f, xv[q][1], acc[ch][p][1]);
                            }
                    }
                }
            }
        }
    }
    __syncthreads();
    if (wave > 0)
#pragma unroll
        for (int e = 0; e < CH * NB * 2; ++e)
            lds[((wave - 1) * CH * NB * 2 + e) * 64 + lane] = acc[e / (2 * NB)][e / 2 % NB][e % 2];
    __syncthreads();
    if (bad >= a.packing) {
        gather_piece(a, x, y, 0, sz.x, lz, sx.x, lx);
        return;
    }
    if (wave > 0) return;
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
        const int t = lane + 64 * ch;
        if (t >= np * lx) continue;
        const int z = 2 * (t % np), col = t / np;
#pragma unroll
        for (int p = 0; p < NB; ++p)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                float v = acc[ch][p][r];
#pragma unroll
                for (int g = 1; g < PSF_WAVES; ++g) v = v + lds[((g - 1) * CH * NB * 2 + (ch * NB + p) * 2 + r) * 64 + lane];
                if (z + r < lz) y[p * a.N + sz.x + z + r + (long long)a.n[0] * (sx.x + col)] = v;
            }
    }
}

}  // namespace

hipError_t launch_psf_pack(const Psf2Args& a, hipStream_t st) {
    const long long n = (long long)a.K[0] * a.K[1] * (2 * a.W + 1) * (2 * a.W + 1) * (a.mono ? 1 : 4);
    k_psf_pack<<<(int)std::min<long long>(65536, (n + NTHREADS - 1) / NTHREADS), NTHREADS, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_psf2_apply(const Psf2Args& a, const float* x, float* y, int transpose, hipStream_t st) {
    if (transpose) {
        const dim3 g((unsigned)(a.ntz * a.ntx));
        // wide windows leave few blocks, each with a long chain of scalar
        // loads: two groups of threads from a spacing of 22 on (20: 122 us in
        // one group, 129 in two; 24: 187 and 149; 30: 236 and 167)
        const size_t sums = 2 * NTHREADS * sizeof(float);
        if (a.s >= 22) {
            if (a.mono) k_psf_t<1, 2><<<g, 2 * NTHREADS, a.lds_t + sums, st>>>(a, a.pack, x, y);
            else k_psf_t<2, 2><<<g, 2 * NTHREADS, 2 * (a.lds_t + sums), st>>>(a, a.pack, x, y);
        } else {
            if (a.mono) k_psf_t<1, 1><<<g, NTHREADS, a.lds_t, st>>>(a, a.pack, x, y);
            else k_psf_t<2, 1><<<g, NTHREADS, 2 * a.lds_t, st>>>(a, a.pack, x, y);
        }
    } else {
        const dim3 g((unsigned)(a.nfz * a.nfx));
        // the patches, or the sums that take their place
        const size_t l = PSF_WAVES * std::max(a.lds_f, 4 * 64 * sizeof(float));
        if (a.mono) k_psf_f<1><<<g, 64 * PSF_WAVES, l, st>>>(a, a.pack, x, y);
        else k_psf_f<2><<<g, 64 * PSF_WAVES, 2 * l, st>>>(a, a.pack, x, y);
    }
    return hipGetLastError();
}

hipError_t launch_psf_apply(const PsfArgs& a, const float* x, float* y, int transpose, hipStream_t st) {
    long long nb = (a.N + NTHREADS - 1) / NTHREADS;
    if (nb > 65536) nb = 65536;
    if (nb < 1) nb = 1;
    k_psf_apply<<<(int)nb, NTHREADS, 0, st>>>(a, x, y, transpose);
    return hipGetLastError();
}

// Unit spikes of parameter q on the scatterer lattice (all other entries of
// the [2][N] model vector zero).
__global__ void k_psf_spikes(PsfArgs a, int q, float* __restrict__ dm) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < 2 * a.N;
         i += (long long)gridDim.x * blockDim.x) {
        const int par = (int)(i / a.N);
        const long long g = i % a.N;
        const int iz = (int)(g % a.n[0]);
        const long long r = g / a.n[0];
        const int ix = (int)(r % a.n[1]);
        const int iy = (int)(r / a.n[1]);
        auto on = [&](int ax, int j) {
            // a lattice node is its own first corner with weight 0
            const Cell c = cell_of(a, ax, j);
            return (c.c0 == j && c.w == 0.f) || (c.c1 == j && c.w == 1.f);
        };
        const bool spike = par == q && on(0, iz) && on(1, ix) && (a.ndim == 2 || on(2, iy));
        dm[i] = spike ? 1.f : 0.f;
    }
}

hipError_t launch_psf_spikes(const PsfArgs& a, int q, float* dm, hipStream_t st) {
    long long nb = (2 * a.N + NTHREADS - 1) / NTHREADS;
    if (nb > 65536) nb = 65536;
    k_psf_spikes<<<(int)nb, NTHREADS, 0, st>>>(a, q, dm);
    return hipGetLastError();
}

}  // namespace lsrtm
