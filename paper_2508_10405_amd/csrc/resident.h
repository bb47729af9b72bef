// Resident 2D time stepping: what the kernels (kern2r_*.hip) and the runtime
// share.
//
// A shot's padded grid is cut into vertical slabs, one workgroup each, and the
// workgroups of a shot (a team) advance it through many time steps in one
// launch, its fields and model in registers.  Per step only the columns that
// a neighbouring slab's stencil reads leave the workgroup.
//
// Why: the streaming kernels read and write every field on every step (88, 56
// and 72 B per node for a Born, replay and adjoint step) and are bound by that
// traffic; a shot's fields and model (12 floats per node in a Born step) fit in
// the registers of a few dozen CUs, after which a Born step moves nothing and a
// replay or adjoint step its 12 B per node of replay buffer.  What bounds a
// step then is instruction issue (two waves per SIMD), the latency of two
// exchanges of boundary columns, and for the replay and adjoint steps the
// buffer's traffic.  Measured on 120 shots of 280 x 777 padded nodes, a Born
// pass of 600 steps went from 219 to 80 ms, a migration pass of 500 steps from
// 298 to 113 ms; on one shot of 140 x 240, 1000 steps, from 8.7 to 3.9 ms and
// from 17.6 to 6.5 ms, where it is the launches that no longer count.
#pragma once
#include "common.h"

namespace lsrtm {

constexpr int RES_WAVES = 8;
constexpr int RES_NT = 64 * RES_WAVES;
constexpr int RES_HALO = 2 * HW - 1;         // columns of other slabs that a derivative reads
constexpr int RES_ZSLOTS = 32;               // LDS slots: lanes that hold rows of the z strips, and one for the others
constexpr int RES_EXCOLS = 5;                // columns published per side (the adjoint's product takes one more)

enum ResKind {
    R_BG = 0,      // background
    R_SEG = 1,     // background, stores G_a p + psi_a and q (replay)
    R_BORN = 2,    // background + scattered
    R_BORN_RC = 3, // scattered, on a background read from the replay cache
    R_ADJ = 4,     // adjoint + images, reads the replay buffer
    R_KINDS = 5
};

// One workgroup of a launch.  nb: bit 0 / 1 = a slab of the same shot lies to
// the left / right (the previous / next workgroup), bit 2 = the slab has
// columns in the absorbing strips (narrow body).
struct ResBlock {
    int slot;
    int x0;                      // first column
    int nb;
    int pad;
};

struct ResArgs {
    const DSlot* slots;
    const ResBlock* blocks;      // [gridDim.x]
    Coef C;
    int n0, n1;                  // steps of the launch (the adjoint walks them backwards)
    int sstep0;                  // replay-buffer step of n0
    int first;                   // adjoint: n1 - 1 is the first reverse step (no pending chi update)
    int npml;
    const int* rptr;             // receivers of a workgroup (CSR over the launch's blocks), or null
    const Rec* rec;              // idx: LDS element of the node (record) or its first receiver (inject)
    float* d;                    // record here
    const float* y;              // inject from here
    const int* nptr;             // adjoint: receiver nodes of a workgroup (CSR), and per node
    const int4* node;            // (owner thread << 8 | c BZ + k, first receiver, one past the last, 0)
    int maxnodes;                // most receiver nodes of a workgroup
    unsigned long long* ex;      // exchange words [block][phase][parity][side][field][col][res_words][64]
    unsigned id;                 // 1 .. RES_IDS - 1: of this launch, since the words were cleared
    int* ctl;                    // arrival count of this launch (0 before it)
    int* abort_;                 // set when a launch gives up
};

// Time limits of a wait, in ticks of the 100 MHz wall clock: all workgroups of
// the launch resident; a neighbour's columns after that.
constexpr long long RES_ADMIT_TICKS = 100000000LL / 2;
constexpr long long RES_WAIT_TICKS = 100000000LL * 5;

// Elements of one replay-buffer array of a step: nx columns of bz rows of 64
// lanes, and no less than the streaming kernels' array, which may take its
// place.
__host__ __device__ constexpr long long res_segn(long long npts, int nx, int bz) {
    return npts > (long long)nx * bz * 64 ? npts : (long long)nx * bz * 64;
}

// A column of a lane travels as res_words(bz) words of 64 bits: bz floats and
// in the top 10 bits of each word a tag, which is the launch and every second
// step's parity.
constexpr int res_words(int bz) { return bz / 2 + 1; }
constexpr int RES_IDS = 512;
// Exchange words of one workgroup.
constexpr long long res_ex_words(int bz, int nf) { return 2LL * 2 * 2 * nf * RES_EXCOLS * res_words(bz) * 64; }
// Columns per wave of a strip slab whose launch's interior slabs have cx: the
// strips' x memories take the registers of a column.
constexpr int res_cx_edge(int cx) { return cx > 1 ? cx - 1 : cx; }
// The z strips' memories in registers: where a thread's nodes leave them.
constexpr bool res_zreg(int kind, int bz, int cx) { return kind <= R_SEG || bz * cx <= (kind == R_BORN ? 6 : 10); }
// LDS floats of the copies of p and v_x (each with its halo), and of the z
// strips' tables and memories.
constexpr size_t res_copy_floats(int bz, int cx) { return (size_t)(RES_WAVES * cx + 2 * HW) * bz * 64; }
constexpr size_t res_strip_floats(int kind, int bz, int cx) {
    const size_t nf = kind == R_BORN ? 2 : 1;
    return 4 * (size_t)bz * 64 + (res_zreg(kind, bz, cx) ? 0 : 2 * nf * RES_WAVES * cx * bz * RES_ZSLOTS);
}
// The Born step keeps one copy that serves p and v_x in turn (two more
// barriers) where two do not fit.
constexpr size_t RES_LDS = 160 * 1024 - 64;
constexpr bool res_alias(int kind, int bz, int cx) {
    return kind == R_BORN && 4 * (4 * res_copy_floats(bz, cx) + res_strip_floats(kind, bz, cx)) > RES_LDS - 4096;
}
// Dynamic LDS bytes of a workgroup whose interior slabs have cx columns per
// wave; most: receivers (adjoint: receiver nodes) of the workgroup that has most.
constexpr size_t res_lds_of(int kind, int bz, int cx, int most) {
    const size_t copy = res_copy_floats(bz, cx), nf = kind == R_BORN ? 2 : 1;
    const size_t copies = kind == R_ADJ ? 2 * copy + (size_t)(RES_WAVES * cx + 1) * bz * 64
                                        : (res_alias(kind, bz, cx) ? 1 : 2) * nf * copy;
    return 4 * (copies + res_strip_floats(kind, bz, cx) + (kind == R_ADJ ? 6 : 4) * (size_t)most + (kind == R_ADJ ? RES_NT + 1 : 0));
}
constexpr size_t res_lds_bytes(int kind, int bz, int cx, int most) {
    const size_t a = res_lds_of(kind, bz, cx, most), b = res_lds_of(kind, bz, res_cx_edge(cx), most);
    return a > b ? a : b;
}
// Instantiated shapes: rows per lane (64 bz >= padded nz) and columns per wave.
constexpr int RES_BZ_MIN = 2, RES_BZ_MAX = 6, RES_CX_MAX = 3;
template <int BZ>
hipError_t launch_resident_bz(int kind, int cx, int nblocks, size_t lds, hipStream_t st, const ResArgs& a,
                              hipEvent_t e0, hipEvent_t e1);
template <> hipError_t launch_resident_bz<2>(int, int, int, size_t, hipStream_t, const ResArgs&, hipEvent_t, hipEvent_t);
template <> hipError_t launch_resident_bz<3>(int, int, int, size_t, hipStream_t, const ResArgs&, hipEvent_t, hipEvent_t);
template <> hipError_t launch_resident_bz<4>(int, int, int, size_t, hipStream_t, const ResArgs&, hipEvent_t, hipEvent_t);
template <> hipError_t launch_resident_bz<5>(int, int, int, size_t, hipStream_t, const ResArgs&, hipEvent_t, hipEvent_t);
template <> hipError_t launch_resident_bz<6>(int, int, int, size_t, hipStream_t, const ResArgs&, hipEvent_t, hipEvent_t);

}  // namespace lsrtm
