// Resident 2D forward steps: background, replay and Born (see resident_dev.h
// for the layout).  The arithmetic of every node is that of the streaming
// kernels (k2_v, k2_p), operation by operation, so the results are the same
// bits.
#pragma once
#include "resident_dev.h"

namespace lsrtm {

template <int BZ, int CX, int KIND, bool XP>
__device__ __forceinline__ void fwd_body(const ResArgs& a, const ResBlock& B, float* lds) {
    using P = Place<BZ, CX, XP>;
    constexpr bool BG = KIND != R_BORN_RC, SC = KIND == R_BORN || KIND == R_BORN_RC, RC = KIND == R_BORN_RC;
    constexpr bool SEGW = KIND == R_SEG;
    constexpr int NF = (BG ? 1 : 0) + (SC ? 1 : 0), IS = BG ? 1 : 0;   // IS: index of the scattered field
    constexpr bool ALIAS = res_alias(KIND, BZ, CX);  // one LDS copy serves p and v_x in turn
    constexpr bool ZREG = res_zreg(KIND, BZ, CX);
    constexpr bool TIGHT = KIND >= R_BORN && BZ * CX > (KIND == R_BORN ? 6 : 10);   // keep the scheduler from running out of registers
    constexpr int CW = P::CW, LC = P::LC, ROW = P::ROW, HP = HW - 1, HV = HW;
    const DSlot& S = a.slots[B.slot];
    P pl(S, B, a.npml);
    constexpr int zs = RES_ZSLOTS;
    const int lane = pl.lane, w = pl.w;
    // LDS: copies of p (and the scattered pressure), of v_x, z-strip tables and memories
    float* const lp = lds;
    float* const lv = ALIAS ? lds : lds + NF * LC * ROW;
    float* const zt = lds + (ALIAS ? 1 : 2) * NF * LC * ROW;
    float* const zm = zt + 4 * ROW + (w * CX * BZ) * zs + pl.zslot;
    constexpr int zmem = ZREG ? 0 : RES_WAVES * CX * BZ * zs;   // one memory of the workgroup
    ZMem<BZ, CX, ZREG> mz[2 * NF];                       // psi_z, phi_z (background), xi_z, eta_z
#pragma unroll
    for (int m = 0; m < 2 * NF; ++m) mz[m].l = zm + m * zmem;
    const float *zah = zt + lane, *zbh = zah + ROW, *zan = zbh + ROW, *zbn = zan + ROW;
    for (int e = threadIdx.x; e < (ALIAS ? 1 : 2) * NF * LC * ROW + 4 * ROW + 2 * NF * zmem; e += RES_NT) lds[e] = 0.f;
    __syncthreads();
    load_ztab<BZ>(S, zt);
    __syncthreads();

    float p[BG ? CX : 1][BZ], vz[BG ? CX : 1][BZ], vx[BG ? CX : 1][BZ];
    float q[SC ? CX : 1][BZ], wz[SC ? CX : 1][BZ], wx[SC ? CX : 1][BZ];
    float kd[CX][BZ], bz[CX][BZ], bx[CX][BZ];
    float lk[SC ? CX : 1][BZ], rz[SC ? CX : 1][BZ], rx[SC ? CX : 1][BZ];
    float mv[XP && BG ? CX : 1][BZ], mp[XP && BG ? CX : 1][BZ];   // psi_x, phi_x
    float nv_[XP && SC ? CX : 1][BZ], np[XP && SC ? CX : 1][BZ];  // xi_x, eta_x
    if constexpr (BG) {
        pl.get(S.p, p);
        pl.get(S.v[0], vz);
        pl.get(S.v[1], vx);
        mz[0].load(pl, S.psi[0], a.npml);
        mz[1].load(pl, S.phi[0], a.npml);
        if constexpr (XP) {
            pl.get_x(S.psi[1], mv, a.npml);
            pl.get_x(S.phi[1], mp, a.npml);
        }
    }
    if constexpr (SC) {
        pl.get(S.q, q);
        pl.get(S.w[0], wz);
        pl.get(S.w[1], wx);
        pl.get(S.dlnk, lk);
        mz[2 * IS].load(pl, S.xi[0], a.npml);
        mz[2 * IS + 1].load(pl, S.eta[0], a.npml);
        if constexpr (XP) {
            pl.get_x(S.xi[1], nv_, a.npml);
            pl.get_x(S.eta[1], np, a.npml);
        }
    }
    pl.get(S.kdt, kd);
    // dt b_a = sb at the node times sb at its upper neighbour (the last node of
    // an axis takes its own value); the same neighbours in the averages of
    // dlnrho
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
        if constexpr (SC) {
            pl.get(S.dlnr, s);
            pl.next(S.dlnr, 0, n);
#pragma unroll
            for (int c = 0; c < CX; ++c)
#pragma unroll
                for (int k = 0; k < BZ; ++k) rz[c][k] = 0.5f * (s[c][k] + n[c][k]);
            pl.next(S.dlnr, 1, n);
#pragma unroll
            for (int c = 0; c < CX; ++c)
#pragma unroll
                for (int k = 0; k < BZ; ++k) rx[c][k] = 0.5f * (s[c][k] + n[c][k]);
        }
    }
    float axh[XP ? CX : 1], bxh[XP ? CX : 1], axn[XP ? CX : 1], bxn[XP ? CX : 1];
    if constexpr (XP)
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            const unsigned g = pl.col(c) ? pl.x + c : 0;
            const float on = pl.col(c) ? 1.f : 0.f;
            axh[c] = uniform(on * elem(S.cpml[1], g));
            bxh[c] = uniform(on * elem(S.cpml[1], pl.nx + g));
            axn[c] = uniform(on * elem(S.cpml[1], 2 * pl.nx + g));
            bxn[c] = uniform(on * elem(S.cpml[1], 3 * pl.nx + g));
        }
    gfloat* const seg0 = uniform(S.seg);
    // the source node, if this thread owns it; its amplitude is loaded a step ahead
    int isrc = -1;
    if (BG && S.src >= 0) {
        const int sz = S.src % (int)pl.ldz, sxc = S.src / (int)pl.ldz - pl.x, k = sz - lane * BZ;
        if (sxc >= 0 && sxc < CX && k >= 0 && k < BZ) isrc = sxc * BZ + k;
    }
    const bool wsrc = __any(isrc >= 0);
    const auto src_amp = uniform(S.src_amp);
    float amp = wsrc ? elem(src_amp, a.n0) : 0.f;

    Exchange<BZ, NF> X(a, (int)blockIdx.x, B.nb, pl.nv > 0);
    X.me = xcd_remap(blockIdx.x, gridDim.x);
    // put the own columns of a field where the neighbours find them
    auto share = [&](int phase, int par, int HL, int f, float* l, const float (&v)[CX][BZ], unsigned tag) {
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            const int j = pl.j0 + c;
#pragma unroll
            for (int k = 0; k < BZ; ++k) l[HW * ROW + pl.lds(c, k)] = v[c][k];
            if ((B.nb & 1) && j < RES_HALO - HL) X.publish(phase, par, 0, f, j, v[c], tag);
            if ((B.nb & 2) && j >= CW - HL) X.publish(phase, par, 1, f, j - (CW - HL), v[c], tag);
        }
    };
    const int r0 = a.rptr && a.d ? a.rptr[X.me] : 0, r1 = a.rptr && a.d ? a.rptr[X.me + 1] : 0;
    LdsRec* const rec = reinterpret_cast<LdsRec*>(zt + 4 * ROW + 2 * NF * zmem);
    for (int j = threadIdx.x; j < r1 - r0; j += RES_NT) {
        const Rec R = a.rec[r0 + j];
        rec[j] = {R.out, R.idx, R.stride};
    }
    auto record = [&](int n) {
        const float* l = lp + (SC ? IS : 0) * LC * ROW;
        for (int j = threadIdx.x; j < r1 - r0; j += RES_NT) {
            const LdsRec R = rec[j];
            a.d[R.out + (long long)n * R.stride] = l[R.idx];
        }
    };
    unsigned tag = X.tag(0);
    if constexpr (BG) share(0, 0, HP, 0, lp, p, tag);
    if constexpr (SC) share(0, 0, HP, IS, lp + IS * LC * ROW, q, tag);

    // background of the step, from the replay cache: the gradients a phase ahead
    float cgz[RC ? CX : 1][BZ], cgx[RC ? CX : 1][BZ];
    auto load_seg = [&](int n, int arr, auto& v) {
        const gfloat* const f = seg0 + ((long long)(a.sstep0 + n - a.n0) * 3 + arr) * pl.segn;
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int k = 0; k < BZ; ++k) v[c][k] = pl.seg_load(f, c, k);
    };
    if constexpr (RC) {
        load_seg(a.n0, 0, cgz);
        load_seg(a.n0, 1, cgx);
    }

    res_priority(w);
    for (int n = a.n0; n < a.n1; ++n) {
        const int par = (n - a.n0) & 1;
        gfloat* const seg = seg0 + (long long)(a.sstep0 + n - a.n0) * 3 * pl.segn;
        float cq[RC ? CX : 1][BZ];
        // ---- velocity phase, z: own columns and lanes
        float ta[BZ], tb[BZ];
        zrow<BZ>(zah, ta);
        zrow<BZ>(zbh, tb);
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float g[BZ], dv[BZ];
            if constexpr (BG) {
                d_col<BZ, 1>(p[c], a.C.c[0], g);
                mz[0].step(ta, tb, c, g);
#pragma unroll
                for (int k = 0; k < BZ; ++k) {
                    dv[k] = -bz[c][k] * g[k];
                    vz[c][k] = vz[c][k] + dv[k];
                    pin(vz[c][k]);
                    if (SEGW) pl.seg_store(seg, c, k, g[k]);
                }
            } else {
#pragma unroll
                for (int k = 0; k < BZ; ++k) dv[k] = -bz[c][k] * cgz[c][k];
            }
            if constexpr (SC) {
                d_col<BZ, 1>(q[c], a.C.c[0], g);
                mz[2 * IS].step(ta, tb, c, g);
#pragma unroll
                for (int k = 0; k < BZ; ++k) {
                    wz[c][k] = (wz[c][k] - bz[c][k] * g[k]) - rz[c][k] * dv[k];
                    pin(wz[c][k]);
                }
            }
        }
        X.template halo<HP, CW, KIND == R_BORN && TIGHT>(w, 0, par, lp, LC * ROW, tag);
        __syncthreads();
        // loads from the replay cache start right after a fetch, so that the
        // next fetch does not wait behind them
        if constexpr (RC) load_seg(n, 2, cq);
        if (n > a.n0) record(n - 1);
        // ---- velocity phase, x
#pragma unroll
        for (int k = 0; k < BZ; ++k) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float dv[CX];
            if constexpr (BG) {
                float win[CX + RES_HALO];
#pragma unroll
                for (int i = 0; i < CX + RES_HALO; ++i)
                    win[i] = i >= HP && i < HP + CX ? p[i - HP][k] : lp[pl.lds(i + HW - HP, k)];
#pragma unroll
                for (int c = 0; c < CX; ++c) {
                    float g = d_win(win + c, a.C.c[1]);
                    if constexpr (XP) {
                        mv[c][k] = fmaf(bxh[c], mv[c][k], axh[c] * g);
                        g = g + mv[c][k];
                    }
                    dv[c] = -bx[c][k] * g;
                    vx[c][k] = vx[c][k] + dv[c];
                    pin(vx[c][k]);
                    if (SEGW) pl.seg_store(seg + pl.segn, c, k, g);
                }
            } else {
#pragma unroll
                for (int c = 0; c < CX; ++c) dv[c] = -bx[c][k] * cgx[c][k];
            }
            if constexpr (SC) {
                const float* l = lp + IS * LC * ROW;
                float win[CX + RES_HALO];
#pragma unroll
                for (int i = 0; i < CX + RES_HALO; ++i)
                    win[i] = i >= HP && i < HP + CX ? q[i - HP][k] : l[pl.lds(i + HW - HP, k)];
#pragma unroll
                for (int c = 0; c < CX; ++c) {
                    float g = d_win(win + c, a.C.c[1]);
                    if constexpr (XP) {
                        nv_[c][k] = fmaf(bxh[c], nv_[c][k], axh[c] * g);
                        g = g + nv_[c][k];
                    }
                    wx[c][k] = (wx[c][k] - bx[c][k] * g) - rx[c][k] * dv[c];
                    pin(wx[c][k]);
                }
            }
        }
        if (ALIAS) __syncthreads();
        if constexpr (BG) share(1, par, HV, 0, lv, vx, tag);
        if constexpr (SC) share(1, par, HV, IS, lv + IS * LC * ROW, wx, tag);
        // ---- pressure phase, z
        float ez[BG ? CX : 1][BZ], fz[SC ? CX : 1][BZ];
        zrow<BZ>(zan, ta);
        zrow<BZ>(zbn, tb);
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            if constexpr (BG) {
                d_col<BZ, 0>(vz[c], a.C.c[0], ez[c]);
                mz[1].step(ta, tb, c, ez[c]);
#pragma unroll
                for (int k = 0; k < BZ; ++k) pin(ez[c][k]);
            }
            if constexpr (SC) {
                d_col<BZ, 0>(wz[c], a.C.c[0], fz[c]);
                mz[2 * IS + 1].step(ta, tb, c, fz[c]);
#pragma unroll
                for (int k = 0; k < BZ; ++k) pin(fz[c][k]);
            }
        }
        X.template halo<HV, CW, KIND == R_BORN && TIGHT>(w, 1, par, lv, LC * ROW, tag);
        __syncthreads();
        if constexpr (RC)
            if (n + 1 < a.n1) {
                load_seg(n + 1, 0, cgz);
                load_seg(n + 1, 1, cgx);
            }
        // ---- pressure phase, x
#pragma unroll
        for (int k = 0; k < BZ; ++k) {
            if (TIGHT) __builtin_amdgcn_sched_barrier(0);
            float dq[CX];
            if constexpr (BG) {
                float win[CX + RES_HALO];
#pragma unroll
                for (int i = 0; i < CX + RES_HALO; ++i)
                    win[i] = i >= HV && i < HV + CX ? vx[i - HV][k] : lv[pl.lds(i, k)];
#pragma unroll
                for (int c = 0; c < CX; ++c) {
                    float g = d_win(win + c, a.C.c[1]);
                    if constexpr (XP) {
                        mp[c][k] = fmaf(bxn[c], mp[c][k], axn[c] * g);
                        g = g + mp[c][k];
                    }
                    dq[c] = ez[c][k] + g;
                    p[c][k] = p[c][k] - kd[c][k] * dq[c];
                    pin(p[c][k]);
                    if (SEGW) pl.seg_store(seg + 2 * pl.segn, c, k, dq[c]);
                }
            } else {
#pragma unroll
                for (int c = 0; c < CX; ++c) dq[c] = cq[c][k];
            }
            if constexpr (SC) {
                const float* l = lv + IS * LC * ROW;
                float win[CX + RES_HALO];
#pragma unroll
                for (int i = 0; i < CX + RES_HALO; ++i)
                    win[i] = i >= HV && i < HV + CX ? wx[i - HV][k] : l[pl.lds(i, k)];
#pragma unroll
                for (int c = 0; c < CX; ++c) {
                    float g = d_win(win + c, a.C.c[1]);
                    if constexpr (XP) {
                        np[c][k] = fmaf(bxn[c], np[c][k], axn[c] * g);
                        g = g + np[c][k];
                    }
                    const float sq = fz[c][k] + g;
                    q[c][k] = (q[c][k] - kd[c][k] * sq) + lk[c][k] * (-kd[c][k] * dq[c]);
                    pin(q[c][k]);
                }
            }
        }
        if (wsrc) {
#pragma unroll
            for (int c = 0; c < (BG ? CX : 0); ++c)
#pragma unroll
                for (int k = 0; k < BZ; ++k)
                    if (isrc == c * BZ + k) p[c][k] = p[c][k] + amp;
            if (n + 1 < a.n1) amp = elem(src_amp, n + 1);
        }
        if (ALIAS) __syncthreads();
        tag = X.tag(n - a.n0 + 1);
        if constexpr (BG) share(0, par ^ 1, HP, 0, lp, p, tag);
        if constexpr (SC) share(0, par ^ 1, HP, IS, lp + IS * LC * ROW, q, tag);
    }
    __syncthreads();
    record(a.n1 - 1);
    if constexpr (SEGW) return;      // the next segment starts from its checkpoint
    pl.forget();
    if constexpr (BG) {
        pl.put(S.p, p);
        pl.put(S.v[0], vz);
        pl.put(S.v[1], vx);
        mz[0].store(pl, S.psi[0], a.npml);
        mz[1].store(pl, S.phi[0], a.npml);
        if constexpr (XP) {
            pl.put_x(S.psi[1], mv, a.npml);
            pl.put_x(S.phi[1], mp, a.npml);
        }
    }
    if constexpr (SC) {
        pl.put(S.q, q);
        pl.put(S.w[0], wz);
        pl.put(S.w[1], wx);
        mz[2 * IS].store(pl, S.xi[0], a.npml);
        mz[2 * IS + 1].store(pl, S.eta[0], a.npml);
        if constexpr (XP) {
            pl.put_x(S.xi[1], nv_, a.npml);
            pl.put_x(S.eta[1], np, a.npml);
        }
    }
}

template <int BZ, int CX, int KIND>
__global__ void __attribute__((amdgpu_flat_work_group_size(RES_NT, RES_NT), amdgpu_waves_per_eu(2, 2)))
k2r_fwd(ResArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ int flag;
    if (!res_admit(a, &flag)) return;
    const ResBlock B = a.blocks[xcd_remap(blockIdx.x, gridDim.x)];
    if (B.nb & 4) fwd_body<BZ, res_cx_edge(CX), KIND, true>(a, B, lds);
    else fwd_body<BZ, CX, KIND, false>(a, B, lds);
}

}  // namespace lsrtm
