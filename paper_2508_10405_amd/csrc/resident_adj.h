// Resident 2D adjoint steps with imaging (see resident_dev.h for the layout).
// The arithmetic of every node is that of the streaming kernels (k2_a, k2_b),
// operation by operation, so the results are the same bits.
#pragma once
#include "resident_dev.h"

namespace lsrtm {

template <int BZ, int CX, bool XP>
__device__ __forceinline__ void adj_body(const ResArgs& a, const ResBlock& B, float* lds) {
    using P = Place<BZ, CX, XP>;
    constexpr bool TIGHT = BZ * CX > 10;             // keep the scheduler from running out of registers
    constexpr int CW = P::CW, LC = P::LC, ROW = P::ROW, HE = HW - 1, HG = HW;
    const DSlot& S = a.slots[B.slot];
    P pl(S, B, a.npml);
    constexpr int zs = RES_ZSLOTS;
    const int lane = pl.lane, w = pl.w;
    // LDS: copies of e~_x, of g~_x and of the lnrho product along x (one
    // column to the left), z-strip tables and memories, data sums at the
    // receiver nodes
    float* const le = lds;
    float* const lg = le + LC * ROW;
    float* const lx = lg + LC * ROW;                 // column j at (j + 1) * ROW
    float* const zt = lx + (CW + 1) * ROW;
    float* const zm = zt + 4 * ROW + (w * CX * BZ) * zs + pl.zslot;
    constexpr bool ZREG = res_zreg(R_ADJ, BZ, CX);
    constexpr int zmem = ZREG ? 0 : RES_WAVES * CX * BZ * zs;
    ZMem<BZ, CX, ZREG> chi, phi;                     // chi_z, phi~_z
    chi.l = zm;
    phi.l = zm + zmem;
    float* const inj = zt + 4 * ROW + 2 * zmem;
    const float *zah = zt + lane, *zbh = zah + ROW, *zan = zbh + ROW, *zbn = zan + ROW;
    for (int e = threadIdx.x; e < (2 * LC + CW + 1 + 4) * ROW + 2 * zmem; e += RES_NT) lds[e] = 0.f;
    __syncthreads();
    load_ztab<BZ, true>(S, zt);
    __syncthreads();

    float Q[CX][BZ], uz[CX][BZ], ux[CX][BZ], gk[CX][BZ], gr[CX][BZ];
    float kd[CX][BZ], bz[CX][BZ], bx[CX][BZ];
    float mc[XP ? CX : 1][BZ], mf[XP ? CX : 1][BZ];  // chi_x, phi~_x
    pl.get(S.q, Q);
    pl.get(S.w[0], uz);
    pl.get(S.w[1], ux);
    pl.get(S.gk, gk);
    pl.get(S.gr, gr);
    pl.get(S.kdt, kd);
    chi.load(pl, S.xi[0], a.npml);
    phi.load(pl, S.eta[0], a.npml);
    if constexpr (XP) {
        pl.get_x(S.xi[1], mc, a.npml);
        pl.get_x(S.eta[1], mf, a.npml);
    }
    // dt b_a = sb at the node times sb at its upper neighbour (the last node of
    // an axis takes its own value)
    {
        float s[CX][BZ], n[CX][BZ];
        pl.get(S.sb, s);
        pl.next(S.sb, 0, n);
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) bz[c][k] = s[c][k] * n[c][k];
        pl.next(S.sb, 1, n);
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) bx[c][k] = s[c][k] * n[c][k];
    }
    float axh[XP ? CX : 1], bxh[XP ? CX : 1], axn[XP ? CX : 1], bxn[XP ? CX : 1];
    if constexpr (XP)
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            const unsigned g = pl.col(c) ? pl.x + c : 0;
            const float on = pl.col(c) ? 1.f : 0.f;
            axh[c] = uniform(on * elem(S.cpml[1], g));
            axn[c] = uniform(on * elem(S.cpml[1], 2 * pl.nx + g));
            // no memory outside the strips
            bxh[c] = axh[c] != 0.f ? uniform(elem(S.cpml[1], pl.nx + g)) : 0.f;
            bxn[c] = axn[c] != 0.f ? uniform(elem(S.cpml[1], 3 * pl.nx + g)) : 0.f;
        }
    const gfloat* const seg0 = uniform(S.seg);
    Exchange<BZ, 1> X(a, 0, B.nb, pl.nv > 0);
    X.me = xcd_remap(blockIdx.x, gridDim.x);
    // receiver nodes: bit c BZ + k of mask, data sums at inj[first ...] in that
    // order (one register: mask, and first above bit 18)
    static_assert(CX * BZ <= 18, "a thread's nodes in 18 bits");
    unsigned mask = 0, wmask = 0;
    const int q0 = a.y ? a.nptr[X.me] : 0, q1 = a.y ? a.nptr[X.me + 1] : 0;
    int* const own = reinterpret_cast<int*>(inj);    // owner thread << 8 | node of the thread
    for (int j = q0 + (int)threadIdx.x; j < q1; j += RES_NT) own[j - q0] = a.node[j].x;
    __syncthreads();
    for (int j = 0; j < q1 - q0; ++j) {
        const int o = own[j];
        if ((o >> 8) == (int)threadIdx.x) {
            if (!mask) mask = (unsigned)j << 18;
            mask |= 1u << (o & 255);
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < CX * BZ; ++b) wmask |= __any((mask >> b) & 1) ? 1u << b : 0u;
    unsigned* const masks = reinterpret_cast<unsigned*>(inj + 6 * a.maxnodes) + threadIdx.x;
    *masks = mask;
    if (threadIdx.x == 0) masks[RES_NT] = 0;             // a zero, as an integer or a float

    auto share_e = [&](int par, unsigned tag) {      // e~_x = Q + aci (phi~ + Q)
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            const int j = pl.j0 + c;
            float e[BZ];
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                e[k] = Q[c][k];
                if constexpr (XP)
                    e[k] = e[k] + axn[c] * (mf[c][k] + e[k]);
                le[HW * ROW + pl.lds(c, k)] = e[k];
            }
            if ((B.nb & 1) && j < RES_HALO - HE) X.publish(0, par, 0, 0, j, e, tag);
            if ((B.nb & 2) && j >= CW - HE) X.publish(0, par, 1, 0, j - (CW - HE), e, tag);
        }
    };
    // the last row of the grid: its row index in the lane, and the lane's share
    const int zlast = (pl.nz - 1) % BZ;
    const float flast = lane == (pl.nz - 1) / BZ ? 0.5f : 0.f;
    unsigned tag = X.tag(0);
    share_e(0, tag);
    // q and the gradients of a step, from the replay buffer: each loaded half
    // a step before it is used, right after a fetch, so that the next fetch
    // does not wait behind it
    float sz[CX][BZ], sx[CX][BZ], sq[CX][BZ];
    auto load_seg = [&](int n) {
        const gfloat* const f = seg0 + (long long)(a.sstep0 + n - a.n0) * 3 * pl.segn;
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                sq[c][k] = pl.seg_load(f + 2 * pl.segn, c, k);
                sx[c][k] = pl.seg_load(f + pl.segn, c, k);
            }
    };
    auto load_z = [&](int n) {
        const gfloat* const f = seg0 + (long long)(a.sstep0 + n - a.n0) * 3 * pl.segn;
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) sz[c][k] = pl.seg_load(f, c, k);
    };
    load_seg(a.n1 - 1);
    load_z(a.n1 - 1);
    // the sum of a node's receivers at step n, in list order; the data of a
    // node with one receiver (the usual case) are loaded a step ahead
    auto node_sum = [&](const int4& u, int n) {
        float s = 0.f;
        for (int r = u.y; r < u.z; ++r) {
            const Rec R = a.rec[r];
            s = s + a.y[R.out + (long long)n * R.stride];
        }
        return s;
    };
    const bool mine = (int)threadIdx.x < q1 - q0;
    LdsNode* const node = reinterpret_cast<LdsNode*>(inj + 2 * a.maxnodes) + threadIdx.x;
    bool single = false;
    float pend = 0.f;
    if (mine) {
        const int4 u = a.node[q0 + (int)threadIdx.x];
        single = u.z - u.y == 1;
        if (single) {
            const Rec R = a.rec[u.y];
            *node = {R.out, R.stride, 0};
            if (a.n1 > 1) pend = a.y[R.out + (long long)(a.n1 - 2) * R.stride];
        }
    }

    res_priority(w);
    for (int n = a.n1 - 1; n >= a.n0; --n) {
        const int par = (a.n1 - 1 - n) & 1;
        const bool skip = a.first && n == a.n1 - 1;
        // ---- phase A, z
        float tn[BZ], th[BZ], tb[BZ];
        zrow<BZ>(zan, tn);
        zrow<BZ>(zah, th);
        zrow<BZ>(zbh, tb);
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float e[BZ], dd[BZ];
#pragma unroll
            for (int k = 0; k < BZ; ++k) e[k] = Q[c][k];
            {
#pragma unroll
                for (int k = 0; k < BZ; ++k) {
                    e[k] = e[k] + tn[k] * (phi.get(c, k) + e[k]);
                    if (!skip) chi.set(c, k, chi.times(tb[k], chi.get(c, k) + uz[c][k]));
                }
            }
            d_col<BZ, 1>(e, a.C.c[0], dd);
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                uz[c][k] = uz[c][k] + bz[c][k] * dd[k];
                pin(uz[c][k]);
            }
        }
        // the replay buffer's values come last in a phase: the wait for them
        // is one for the words published before it too
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                gk[c][k] = gk[c][k] + sq[c][k] * Q[c][k];
                pin(gk[c][k]);
            }
        X.template halo<HE, CW, false>(w, 0, par, le, 0, tag);
        __syncthreads();
        // data of step n - 1 at the receiver nodes: here the words published
        // before the barrier no longer hold up the wait for them
        if (w * 64 < q1 - q0 && n > 0) {
            float* const to = inj + (n & 1) * a.maxnodes;
            if (single) to[threadIdx.x] = 0.f + pend;
            else if (mine) to[threadIdx.x] = node_sum(a.node[q0 + (int)threadIdx.x], n - 1);
            for (int j = RES_NT + (int)threadIdx.x; j < q1 - q0; j += RES_NT) to[j] = node_sum(a.node[q0 + j], n - 1);
            if (single && n > 1) pend = a.y[node->out + (long long)(n - 2) * node->stride];
        }
        if (n < a.n1 - 1) load_z(n);
        // ---- phase A, x
#pragma unroll
        for (int k = 0; k < BZ; ++k) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float win[CX + RES_HALO];
#pragma unroll
            for (int i = 0; i < CX + RES_HALO; ++i)
                win[i] = !XP && i >= HE && i < HE + CX ? Q[i - HE][k] : le[pl.lds(i + HW - HE, k)];
#pragma unroll
            for (int c = 0; c < CX; ++c) {
                if constexpr (XP)
                    if (!skip) mc[c][k] = bxh[c] * (mc[c][k] + ux[c][k]);
                ux[c][k] = ux[c][k] + bx[c][k] * d_win(win + c, a.C.c[1]);
                pin(ux[c][k]);
            }
        }
        // g~_x = U_x + ach (chi + U_x) and the product -(G_x p + psi_x) U_x
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            const int j = pl.j0 + c;
            float g[BZ], x[BZ];
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                g[k] = ux[c][k];
                if constexpr (XP)
                    g[k] = g[k] + axh[c] * (mc[c][k] + g[k]);
                x[k] = -sx[c][k] * ux[c][k];
                lg[HW * ROW + pl.lds(c, k)] = g[k];
                lx[ROW + pl.lds(c, k)] = x[k];
            }
            if ((B.nb & 1) && j < RES_HALO - HG) X.publish(1, par, 0, 0, j, g, tag);
            if ((B.nb & 2) && j >= CW - HG) X.publish(1, par, 1, 0, j - (CW - HG), g, tag);
            if ((B.nb & 2) && j == CW - 1) X.publish(1, par, 1, 0, HG, x, tag);
        }
        // ---- phase B, z
        zrow<BZ>(zbn, tb);
        float dz[CX][BZ];
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float g[BZ];
#pragma unroll
            for (int k = 0; k < BZ; ++k) g[k] = uz[c][k];
            {
#pragma unroll
                for (int k = 0; k < BZ; ++k) {
                    g[k] = g[k] + th[k] * (chi.get(c, k) + g[k]);
                    phi.set(c, k, phi.times(tb[k], phi.get(c, k) + Q[c][k]));
                }
            }
            d_col<BZ, 0>(g, a.C.c[0], dz[c]);
#pragma unroll
            for (int k = 0; k < BZ; ++k) pin(dz[c][k]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            float x[BZ];
#pragma unroll
            for (int k = 0; k < BZ; ++k) x[k] = -sz[c][k] * uz[c][k];
            const float xb = lane_below(x[BZ - 1]);
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                sz[c][k] = 0.5f * (x[k] + (k ? x[k ? k - 1 : 0] : xb));
                // the last node of an axis takes the other half of its own
                // product too (rounded by itself: half an odd subnormal is inexact)
                if (k == zlast) sz[c][k] = sz[c][k] + flast * x[k];
                pin(sz[c][k]);
            }
        }
        X.template halo<HG, CW, false>(w, 1, par, lg, 0, tag);
        if (w == 2 && (B.nb & 1)) X.template fetch<1>(X.me - 1, 1, par, 1, 0, HG, lx + lane, 0, tag);
        __syncthreads();
        if (n > a.n0) load_seg(n - 1);
        // ---- phase B, x
#pragma unroll
        for (int k = 0; k < BZ; ++k) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float win[CX + RES_HALO], x[CX + 1];
#pragma unroll
            for (int i = 0; i < CX + RES_HALO; ++i)
                win[i] = !XP && i >= HG && i < HG + CX ? ux[i - HG][k] : lg[pl.lds(i, k)];
#pragma unroll
            for (int i = 0; i < CX + 1; ++i) x[i] = lx[pl.lds(i, k)];
#pragma unroll
            for (int c = 0; c < CX; ++c) {
                float tx = 0.5f * (x[c + 1] + x[c]);
                if (XP && pl.x + c + 1 == pl.nx) tx = tx + 0.5f * x[c + 1];
                gr[c][k] = gr[c][k] + (sz[c][k] + tx);
                if constexpr (XP)
                    mf[c][k] = bxn[c] * (mf[c][k] + Q[c][k]);
                Q[c][k] = Q[c][k] + kd[c][k] * (dz[c][k] + d_win(win + c, a.C.c[1]));
                pin(gr[c][k]);
                pin(Q[c][k]);
            }
        }
        if (wmask && n > 0) {
            // a row of nodes at a time, the nodes that are none taking the zero
            const unsigned mask = *masks;
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                unsigned row = 0;
#pragma unroll
                for (int c = 0; c < CX; ++c) row |= 1u << (c * BZ + k);
                if (!(wmask & row)) continue;
                float v[CX];
#pragma unroll
                for (int c = 0; c < CX; ++c) {
                    const int b = c * BZ + k, at = (n & 1) * a.maxnodes + (int)(mask >> 18) + __popc(mask & ((1u << b) - 1));
                    v[c] = inj[(mask >> b) & 1 ? at : 6 * a.maxnodes + RES_NT];
                }
#pragma unroll
                for (int c = 0; c < CX; ++c) Q[c][k] = Q[c][k] - kd[c][k] * v[c];
            }
        }
        tag = X.tag(a.n1 - n);
        share_e(par ^ 1, tag);
    }
    pl.forget();
    pl.put(S.q, Q);
    pl.put(S.w[0], uz);
    pl.put(S.w[1], ux);
    pl.put(S.gk, gk);
    pl.put(S.gr, gr);
    chi.store(pl, S.xi[0], a.npml);
    phi.store(pl, S.eta[0], a.npml);
    if constexpr (XP) {
        pl.put_x(S.xi[1], mc, a.npml);
        pl.put_x(S.eta[1], mf, a.npml);
    }
}

template <int BZ, int CX>
__global__ void __attribute__((amdgpu_flat_work_group_size(RES_NT, RES_NT), amdgpu_waves_per_eu(2, 2)))
k2r_adj(ResArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ int flag;
    if (!res_admit(a, &flag)) return;
    const ResBlock B = a.blocks[xcd_remap(blockIdx.x, gridDim.x)];
    if (B.nb & 4) adj_body<BZ, res_cx_edge(CX), true>(a, B, lds);
    else adj_body<BZ, CX, false>(a, B, lds);
}

}  // namespace lsrtm
