// Device code shared by the resident 2D kernels (resident_fwd.h, resident_adj.h).
//
// Layout of a slab: wave w of a workgroup owns columns w CX .. w CX + CX - 1
// of its slab; lane l owns rows l BZ .. l BZ + BZ - 1 of each, so a wave spans
// the whole z extent.  z-neighbours outside the lane come from the next lanes
// (DPP shifts, zero beyond the wave as the operators define it); x-neighbours
// from an LDS copy of the slab with the halo columns, [column][row k][lane].
#pragma once
#include "resident.h"

namespace lsrtm {

using u64 = unsigned long long;
using gu64 = __attribute__((address_space(1))) u64;

// The value that lane - 1 / lane + 1 holds; 0 in the first / last lane.
__device__ __forceinline__ float lane_below(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_above(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}

// The staggered differences of the streaming kernels (d_half, d_node) on a
// window w[i]: both are sum_m c_m (w[i + 4 + m] - w[i + 3 - m]), the window of
// the half-node derivative starting three nodes below, of the node one four.
__device__ __forceinline__ float d_win(const float* w, const float* ck) {
    float r = ck[0] * (w[4] - w[3]);
    r = fmaf(ck[1], w[5] - w[2], r);
    r = fmaf(ck[2], w[6] - w[1], r);
    r = fmaf(ck[3], w[7] - w[0], r);
    return r;
}

// e[4 + o] = the column's value o rows above the lane's first row, o = -4 .. BZ + 3.
template <int BZ>
__device__ __forceinline__ void col_ext(const float (&f)[BZ], float (&e)[BZ + 8]) {
#pragma unroll
    for (int k = 0; k < BZ; ++k) e[4 + k] = f[k];
#pragma unroll
    for (int o = 1; o <= 4; ++o) e[4 - o] = lane_below(e[4 - o + BZ]);
#pragma unroll
    for (int j = 0; j < 4; ++j) e[4 + BZ + j] = lane_above(e[4 + j]);
}

// The z-derivative of a column: rows o above / below the lane's own come from
// the lanes next to it.  HALF = 1: at half nodes (three below, four above),
// 0: at nodes (four below, three above); the differences of d_win.  Each
// shifted value is used right after it is formed, so that the shift becomes
// an operand modifier of the subtraction.
template <int BZ, int HALF>
__device__ __forceinline__ void d_col(const float (&f)[BZ], const float* ck, float (&r)[BZ]) {
    float d[BZ][4];              // d[k][m] = value at k + HALF + m minus value at k + HALF - 1 - m
    if constexpr (BZ >= 4) {
#pragma unroll
        for (int k = 0; k < BZ; ++k)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int u = k + HALF + m, l = k + HALF - 1 - m;
                if (u < BZ && l >= 0) d[k][m] = f[u] - f[l];
            }
#pragma unroll
        for (int o = 1; o <= 4; ++o) {
            const float s = lane_below(f[BZ - o]);      // value at -o
#pragma unroll
            for (int k = 0; k < BZ; ++k)
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (k + HALF - 1 - m == -o && k + HALF + m < BZ) d[k][m] = f[k + HALF + m] - s;
        }
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const float s = lane_above(f[o]);           // value at BZ + o
#pragma unroll
            for (int k = 0; k < BZ; ++k)
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (k + HALF + m == BZ + o && k + HALF - 1 - m >= 0) d[k][m] = s - f[k + HALF - 1 - m];
        }
#pragma unroll
        for (int k = 0; k < BZ; ++k)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int u = k + HALF + m, l = k + HALF - 1 - m;
                if (u >= BZ && l < 0) d[k][m] = lane_above(f[u - BZ]) - lane_below(f[l + BZ]);
            }
#pragma unroll
        for (int k = 0; k < BZ; ++k) {
            float v = ck[0] * d[k][0];
            v = fmaf(ck[1], d[k][1], v);
            v = fmaf(ck[2], d[k][2], v);
            r[k] = fmaf(ck[3], d[k][3], v);
        }
    } else {
        float e[BZ + 8];
        col_ext<BZ>(f, e);
#pragma unroll
        for (int k = 0; k < BZ; ++k) r[k] = d_win(e + k + HALF, ck);
    }
}

// Keeps the computation of x where it is written: values that are needed in a
// later phase only would otherwise be computed there, and their operands (the
// windows of a whole phase) held in registers until then.
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }

__device__ __forceinline__ float uniform(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
// A descriptor's pointer, kept in scalar registers.  Read from the descriptor
// inside the time loop it is a vector load (the kernel stores to memory), and the
// wait for it is also one for every word just published: a background step of 7 shots
// of 280 x 777 took 4.5 us with the source's amplitude read so, 4.1 without.
template <typename G>
__device__ __forceinline__ G* uniform(G* p) {
    const u64 b = (u64)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return (G*)(((u64)hi << 32) | lo);
}

// Where a workgroup stands in its shot's grid, and what a thread owns.
template <typename G>
struct ByteOf {
    using T = gchar;
};
template <>
struct ByteOf<const gfloat> {
    using T = const gchar;
};
template <typename G>
using Byte = typename ByteOf<G>::T;

template <int BZ, int CX, bool XP>
struct Place {
    static constexpr int CW = RES_WAVES * CX;        // slab width
    static constexpr int LC = CW + 2 * HW;           // columns of an LDS copy: HW halo columns on either side
    static constexpr int ROW = BZ * 64;              // elements per column
    int lane, w, j0, x, nz, nx, nv;                  // j0: first own column in the slab, nv: valid rows
    unsigned ldz;
    long long segn;                                  // elements of one replay-buffer array of a step
    bool zp;                                         // the lane holds rows of a z strip
    int zslot;
    __device__ __forceinline__ Place(const DSlot& S, const ResBlock& B, int npml) {
        lane = threadIdx.x & 63;
        w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        j0 = w * CX;
        x = B.x0 + j0;
        nz = S.n[0];
        nx = S.n[1];
        ldz = (unsigned)S.ldz;
        segn = res_segn(S.npts, nx, BZ);
        nv = nz - lane * BZ;
        // lanes with rows < npml, then lanes with rows >= nz - npml - 1
        const int low = (npml + BZ - 1) / BZ, top = max(0, nz - npml - 1) / BZ;
        zp = npml > 0 && nv > 0 && (lane < low || lane >= top);
        zslot = !zp ? RES_ZSLOTS - 1 : lane < low ? lane : lane - max(top, low) + low;
    }
    // a slab without strip columns lies inside the grid
    __device__ __forceinline__ bool col(int c) const { return !XP || x + c < nx; }
    __device__ __forceinline__ bool ok(int c, int k) const { return col(c) && k < nv; }
    // Addresses: a base that is uniform over the wave and one lane offset.
    // Standard layout of a shot's arrays:
    template <typename G>
    __device__ __forceinline__ G& at(G* f, int c, int k) const {
        return *reinterpret_cast<G*>(reinterpret_cast<Byte<G>*>(f + ((long long)(x + c) * ldz + k)) + (unsigned)(lane * (4 * BZ)));
    }
    // Replay buffer of a step: [column][row k][lane], so that a wave's accesses
    // are whole lines and lie a constant apart.  Rows past the grid hold whatever
    // the differences make of the rows above them; their readers have zeros there
    // to multiply them by (Q, U_a, dt b_a), and store none of their own.
    template <typename G>
    __device__ __forceinline__ G& seg(G* f, int c, int k) const {
        return *reinterpret_cast<G*>(reinterpret_cast<Byte<G>*>(f + (long long)x * ROW) + (unsigned)(lane * 4) + (c * BZ + k) * 256);
    }
    __device__ __forceinline__ float seg_load(const gfloat* f, int c, int k) const {
        if (XP && !col(c)) return 0.f;
        return __builtin_nontemporal_load(&seg(f, c, k));
    }
    // whole lines, the rows past the grid included: stores of the 224 bytes of
    // 56 lanes ran at two thirds of the rate
    __device__ __forceinline__ void seg_store(gfloat* f, int c, int k, float v) const {
        if (col(c)) __builtin_nontemporal_store(v, &seg(f, c, k));
    }
    __device__ __forceinline__ int lds(int c, int k) const { return (j0 + c) * ROW + k * 64 + lane; }
    // after the time loop: nothing of the addresses is kept in registers
    // through it
    __device__ __forceinline__ void forget() {
        asm volatile("" : "+v"(lane), "+v"(nv));
        asm volatile("" : "+s"(x), "+s"(ldz));
    }
    // a shot's value at the nearest node inside the grid: loads that no branch
    // separates
    template <typename G>
    __device__ __forceinline__ float near(G* f, int c, int k) const {
        const int z = min(lane * BZ + k, nz - 1), g = XP ? min(x + c, nx - 1) : x + c;
        return *reinterpret_cast<G*>(reinterpret_cast<Byte<G>*>(f + (long long)g * ldz) + (unsigned)(z * 4));
    }
    __device__ __forceinline__ void get(const gfloat* f, float (&v)[CX][BZ]) const {
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) v[c][k] = near(f, c, k);
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) v[c][k] = ok(c, k) ? v[c][k] : 0.f;
    }
    // the upper neighbours along an axis (0: z, 1: x), zero outside the grid
    __device__ __forceinline__ void next(const gfloat* f, int axis, float (&v)[CX][BZ]) const {
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                const int z = min(lane * BZ + k + (axis == 0 ? 1 : 0), nz - 1), g = min(x + c + (axis == 1 ? 1 : 0), nx - 1);
                v[c][k] = *reinterpret_cast<const gfloat*>(reinterpret_cast<const gchar*>(f + (long long)g * ldz) + (unsigned)(z * 4));
            }
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) v[c][k] = ok(c, k) ? v[c][k] : 0.f;
    }
    __device__ __forceinline__ void put(gfloat* f, const float (&v)[CX][BZ]) const {
#pragma unroll
        for (int c = 0; c < CX; ++c) {
#pragma unroll
            for (int k = 0; k < BZ; ++k)
                if (ok(c, k)) at(f, c, k) = v[c][k];
        }
    }
    __device__ __forceinline__ void get_x(const gfloat* f, float (&v)[CX][BZ], int npml) const {
#pragma unroll
        for (int c = 0; c < CX; ++c) {
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                const float m = near(f, c, k);
                v[c][k] = ok(c, k) && in_pml(x + c, nx, npml) ? m : 0.f;
            }
        }
    }
    __device__ __forceinline__ void put_x(gfloat* f, const float (&v)[CX][BZ], int npml) const {
#pragma unroll
        for (int c = 0; c < CX; ++c) {
#pragma unroll
            for (int k = 0; k < BZ; ++k)
                if (ok(c, k) && in_pml(x + c, nx, npml)) at(f, c, k) = v[c][k];
        }
    }
};

// Every workgroup of the launch is resident, or none of them starts: a
// workgroup counts itself in and waits for the others; the first one to wait
// too long (another process or stream holds part of the GPU) turns the count
// negative, after which every workgroup leaves.  Past this point every wait
// is for a workgroup that is running.
__device__ __forceinline__ bool res_admit(const ResArgs& a, int* shared) {
    if (threadIdx.x == 0) {
        int ok = 0;
        if (__hip_atomic_load(a.abort_, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
            const int total = (int)gridDim.x;
            int v = __hip_atomic_fetch_add(a.ctl, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
            const long long t0 = wall_clock64();
            while (v >= 0 && v < total) {
                if (wall_clock64() - t0 > RES_ADMIT_TICKS &&
                    __hip_atomic_compare_exchange_strong(a.ctl, &v, -(1 << 30), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)) {
                    v = -1;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
                v = __hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            ok = v >= 0;
            if (!ok) __hip_atomic_store(a.abort_, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        *shared = ok;
    }
    __syncthreads();
    const bool ok = *shared != 0;
    __syncthreads();
    return ok;
}

// Exchange of boundary columns.  A lane's rows of a column are published as
// 64-bit words that each carry a tag in their top 10 bits, stored and loaded
// whole at device scope, so a reader needs no flag and no fence: it loads the
// words until every tag matches.  Steps alternate between two buffers: a slab
// can be at most one exchange ahead of its neighbour, because it needs the
// neighbour's columns to go on, so a word holds this step's values, those of
// two steps ago, or an earlier launch's, and the launch's number with the
// parity of (step / 2) tells them apart.
//
// What the exchange costs is its bytes, at device scope past the XCD's L2, and
// the loads' latency (0.75 us when the words are there).  With a word per value
// (40 B for 5 rows, now 24) and a Born step's two fields fetched one after the
// other by the same waves, steps of 7 shots of 280 x 777 took 8.7 us (Born) and
// 5.6 us (replay), now 7.4 and 4.2.
template <int BZ, int NF>
struct Exchange {
    static constexpr int W = res_words(BZ), R = BZ - W;   // R values lie across the words' upper halves
    static constexpr unsigned LOW = (1u << 22) - 1;       // value bits of an upper half
    u64* ex;                     // of this launch
    long long per;               // words per workgroup
    int me, nb;
    unsigned id;
    int* abort_;
    bool in;                     // the lane holds rows of the grid (the others neither publish nor wait)
    bool dead = false;
    __device__ __forceinline__ Exchange(const ResArgs& a, int b, int nb_, bool in_)
        : ex(a.ex), per(res_ex_words(BZ, NF)), me(b), nb(nb_), id(a.id), abort_(a.abort_), in(in_) {}
    // tag of the launch's i-th step
    __device__ __forceinline__ unsigned tag(int i) const { return (id << 1 | ((unsigned)i >> 1 & 1)) << 22; }
    // A column's words: a base that is uniform over the wave, and the lane.
    // (opaque, so that no 64-bit lane address is kept through the time loop)
    __device__ __forceinline__ gu64* words(int b, int phase, int par, int side, int f, int col) const {
        gu64* p = (gu64*)(ex + b * per + ((((((phase * 2 + par) * 2 + side) * NF + f) * RES_EXCOLS) + col) * W) * 64);
        asm volatile("" : "+s"(p));
        return p;
    }
    static __device__ __forceinline__ gu64* lane_word(gu64* base, int k) {
        return (gu64*)((gchar*)(base + k * 64) + ((threadIdx.x & 63u) << 3));
    }
    __device__ __forceinline__ void publish(int phase, int par, int side, int f, int col, const float (&v)[BZ],
                                            unsigned tag) const {
        gu64* const p = words(me, phase, par, side, f, col);
        if (!in) return;
        const unsigned e0 = R > 0 ? __float_as_uint(v[R > 0 ? W : 0]) : 0, e1 = R > 1 ? __float_as_uint(v[R > 1 ? W + 1 : 0]) : 0;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            unsigned bits;           // a copy: the value itself is not tied to the word's register pair
            asm volatile("v_mov_b32 %0, %1" : "=v"(bits) : "v"(v[k]));
            const unsigned up = k == 0 ? e0 : k == 1 ? __builtin_amdgcn_alignbit(e1, e0, 22) : k == 2 ? e1 >> 12 : 0;
            __hip_atomic_store(lane_word(p, k), ((u64)((up & LOW) | tag) << 32) | bits, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // Columns col .. col + N - 1 of a neighbour's published side, fields f ..
    // f + F - 1, into LDS (field g, column i, row k at dst[g * stride + i * BZ *
    // 64 + k * 64]); all words are loaded before any is waited for.
    template <int N, int F = 1>
    __device__ __forceinline__ void fetch(int from, int phase, int par, int side, int f, int col, float* dst,
                                          int stride, unsigned tag) {
        u64 v[F][N * W];
        long long t0 = 0;
        for (int it = 1;; ++it) {
            unsigned differ = 0;
#pragma unroll
            for (int g = 0; g < F; ++g) {
                gu64* const p = words(from, phase, par, side, f + g, col);
#pragma unroll
                for (int k = 0; k < N * W; ++k)
                    v[g][k] = __hip_atomic_load(lane_word(p, k), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int g = 0; g < F; ++g)
#pragma unroll
                for (int k = 0; k < N * W; ++k) differ |= (unsigned)(v[g][k] >> 32) ^ tag;
            if (__all(differ <= LOW || !in) || dead) break;
            if ((it & 255) == 0) {
                const long long now = wall_clock64();
                if (t0 == 0) t0 = now;
                if (now - t0 > RES_WAIT_TICKS ||
                    __hip_atomic_load(abort_, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                    // give up: run on without waiting, so that every wave ends
                    __hip_atomic_store(abort_, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    dead = true;
                    break;
                }
            }
        }
        if (in)
#pragma unroll
            for (int g = 0; g < F; ++g)
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    float* const d = dst + g * stride + i * BZ * 64;
                    auto up = [&](int k) { return (unsigned)(v[g][i * W + k] >> 32); };
#pragma unroll
                    for (int k = 0; k < W; ++k) d[k * 64] = __uint_as_float((unsigned)v[g][i * W + k]);
                    if constexpr (R > 0) d[W * 64] = __uint_as_float((up(0) & LOW) | up(1) << 22);
                    if constexpr (R > 1) d[(W + 1) * 64] = __uint_as_float((up(1) >> 10 & 0xfff) | up(2) << 12);
                }
    }
    // The halo columns of an LDS copy (HL of them to the left), two or three to a
    // wave: the left ones by waves 0 and 1, the right ones by waves 6 and 7,
    // every field of the exchange at once; or, where registers do not allow that,
    // the second field by the waves next to them (a wave that fetched one field
    // after the other would wait for two round trips).
    template <int HL, int CW, bool SPLIT>
    __device__ __forceinline__ void halo(int w, int phase, int par, float* lds, int stride, unsigned tag) {
        constexpr int HR = RES_HALO - HL, ROW = BZ * 64, F = SPLIT ? 1 : NF;
        float* l = lds + (threadIdx.x & 63);
        int f = 0;
        if (SPLIT && w >= 2 && w < 6) {
            w = w < 4 ? w - 2 : w + 2;
            f = 1;
            l += stride;
        }
        if (nb & 1) {
            if (w == 0) fetch<2, F>(me - 1, phase, par, 1, f, 0, l + (HW - HL) * ROW, stride, tag);
            if (w == 1) fetch<HL - 2, F>(me - 1, phase, par, 1, f, 2, l + (HW - HL + 2) * ROW, stride, tag);
        }
        if (nb & 2) {
            if (w == 6) fetch<2, F>(me + 1, phase, par, 0, f, 0, l + (HW + CW) * ROW, stride, tag);
            if (w == 7) fetch<HR - 2, F>(me + 1, phase, par, 0, f, 2, l + (HW + CW + 2) * ROW, stride, tag);
        }
    }
};

// The waves that publish and fetch columns (the outer two on either side) run
// at a higher priority than the inner wave on their SIMD: they publish early,
// and the words travel while the inner waves compute.
__device__ __forceinline__ void res_priority(int w) {
    if (w < 2 || w >= RES_WAVES - 2) __builtin_amdgcn_s_setprio(2);
}

// a b, and 0 where a is 0, whatever b is.
__device__ __forceinline__ float mul0(float a, float b) {
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// CPML memories of the z strips: in registers where they are to spare, or in
// LDS slots of the lanes that hold strip rows (the other lanes share one slot of
// zeros).  Every lane does the arithmetic, with zero coefficients outside the
// strips, where mul0 keeps an Inf or NaN of the fields out of the shared slot (the
// lane whose store is the last there would hand its own to all the others): a branch around it put the wave's outstanding memory accesses in front
// of it (a replay step of 7 shots of 280 x 777 took 8.6 us with the branch, 5.6
// without).
template <int BZ, int CX, bool REG>
struct ZMem {
    float r[REG ? CX : 1][REG ? BZ : 1];
    float* l;                    // the lane's slots
    __device__ __forceinline__ float get(int c, int k) const { return REG ? r[REG ? c : 0][REG ? k : 0] : l[(c * BZ + k) * RES_ZSLOTS]; }
    __device__ __forceinline__ void set(int c, int k, float v) {
        if (REG) r[REG ? c : 0][REG ? k : 0] = v;
        else l[(c * BZ + k) * RES_ZSLOTS] = v;
    }
    // a coefficient times what goes into a memory
    static __device__ __forceinline__ float times(float a, float v) { return REG ? a * v : mul0(a, v); }
    // g += psi with psi = b psi + a g (a lane's rows outside the strips have
    // a = 0, psi = 0)
    __device__ __forceinline__ void step(const float (&a)[BZ], const float (&b)[BZ], int c, float (&g)[BZ]) {
#pragma unroll
        for (int k = 0; k < BZ; ++k) {
            const float ps = fmaf(b[k], get(c, k), times(a[k], g[k]));
            set(c, k, ps);
            g[k] = g[k] + ps;
        }
    }
    template <typename P>
    __device__ __forceinline__ void load(const P& pl, const gfloat* f, int npml) {
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                // zero outside the strips (global memory holds anything there)
                const float m = pl.near(f, c, k);
                set(c, k, pl.ok(c, k) && in_pml(pl.lane * BZ + k, pl.nz, npml) ? m : 0.f);
            }
    }
    template <typename P>
    __device__ __forceinline__ void store(const P& pl, gfloat* f, int npml) const {
        if (!pl.zp) return;
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k)
                if (pl.ok(c, k) && in_pml(pl.lane * BZ + k, pl.nz, npml)) pl.at(f, c, k) = get(c, k);
    }
};

// One coefficient table's rows of the lane.
template <int BZ>
__device__ __forceinline__ void zrow(const float* t, float (&v)[BZ]) {
#pragma unroll
    for (int k = 0; k < BZ; ++k) v[k] = t[k * 64];
}

// A receiver of the workgroup, kept in LDS.
struct LdsRec {
    long long out;
    int idx, stride;
};
// Where the data of a thread's receiver node are, if it has one receiver.
struct LdsNode {
    long long out;
    int stride, pad;
};

// The z axis' coefficient tables (half-node a, b; node a, b) as [4][BZ][64].
// ADJ: b = 0 outside the strips, where the adjoint has no memory (its memories
// take in the field itself, not a times it).
template <int BZ, bool ADJ = false>
__device__ __forceinline__ void load_ztab(const DSlot& S, float* zt) {
    const int nz = S.n[0];
    for (int e = threadIdx.x; e < 4 * BZ * 64; e += RES_NT) {
        const int t = e / (BZ * 64), k = (e / 64) % BZ, z = (e & 63) * BZ + k;
        float v = z < nz ? elem(S.cpml[0], (unsigned)(t * nz + z)) : 0.f;
        if (ADJ && (t & 1) && z < nz && elem(S.cpml[0], (unsigned)((t - 1) * nz + z)) == 0.f) v = 0.f;
        zt[e] = v;
    }
}

}  // namespace lsrtm
