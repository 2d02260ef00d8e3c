// patch_kernels.hpp -- gfx950 device code of the patch form: several time steps per launch on
// rectangular patches of a small mesh, one cell per lane, for single cases and for batches.
//
// What it is for.  The march of kernels.hpp walks a wave up a block of rows: on a mesh of a few
// hundred cells a side there are too few strips and row blocks to fill the chip, and a launch
// lasts as long as the chain of rows that one wave advances in turn (about 1 us a row).  Here
// every lane owns one cell, its nine values stay in registers for all the steps of a launch,
// and a step costs one row's arithmetic however tall the mesh is.
//
// Layout.  A workgroup of W waves owns a patch of up to W * (64 / tw) rows of tw columns: a wave
// holds 64 / tw rows side by side in its lanes, so x-neighbours are DPP lane moves as in the
// march (the lanes at the ends of a row are halo and may receive anything), and rows meet
// through LDS: phi of every cell (9 values) and the values on every cell's north face (the 6
// directions that cross it), with one barrier behind each.  A patch carries `halo` extra cells
// on each side, so `halo` steps can follow each other without other patches; each step spoils
// one more ring of them.  Beyond a non-periodic side there is no halo but one ghost row or
// column, refilled at every step by the march's ghost rule.
//
// Every face and cell is evaluated with the march's functions and metrics in the march's order,
// and 16-bit storage is rounded after every step: the bits are those of one-step launches.
#pragma once
#include "kernels.hpp"

namespace lbfv {

constexpr int PATCH_WAVES = 8;    // most waves of a workgroup: 512 lanes, two waves per SIMD
// Values per lane in LDS: phi (9) and the north face (6), side by side, so that they are reached
// by constant offsets from one address; an odd count, so that lanes in a row meet no bank conflict.
constexpr int PATCH_LDS = 15;

// Patches of one mesh: an axis of n cells split into np runs of qn or qn + 1 cells, the rn
// longer ones first.
struct PatchGrid {
    int32_t tw;         // lanes per row of a patch, halo and ghost columns included (at most 64)
    int32_t fit;        // rows per wave, 64 / tw
    int32_t halo;       // halo width = most steps per launch (less than a periodic axis)
    int32_t npx, npy;   // patches per axis
    int32_t qx, rx, qy, ry;
};

template <typename T, typename S, int SCHEME, bool BND, bool REF>
struct Patch : March<T, S, SCHEME, BND, 2, REF> {
    using M = March<T, S, SCHEME, BND, 2, REF>;
    using M::P;
    using M::lane;
    uint32_t off;               // byte offset of this lane's cell within a direction plane
    bool out;                   // the lane's result is stored
    int slot, up, down;         // LDS slots of its cell and of the cells above and below
    T lamN, bnN, isy, cdy;      // metrics of its north face and row
    // What the patch's sides ask for (`sides`, the same for the workgroup) and this lane's part in
    // it (`part`), one bit each: as separate flags they fill the scalar registers and push the
    // equilibrium's constants into vector registers (188 for FP64 DUGKS, two waves per SIMD).
    // The side's values stay in registers too: read from the parameters inside the step loop,
    // each is a scalar load that a lone wave waits for (twice the time of a step).
    uint32_t sides, part;
    enum : uint32_t { EXT_W = 1, MIR_W = 2, WALL_W = 4, EXT_E = 8, MIR_E = 16, WALL_E = 32,   // sides
                      SOUTH = 64, MIR_S = 128, WALL_S = 256, NORTH = 512, MIR_N = 1024, WALL_N = 2048 };
    enum : uint32_t { GHOST_W = 1, FACE_W = 2, GHOST_E = 4,   // column -1, column 0, column nx
                      FIXED = 8,        // a ghost cell that holds a constant state (inflow), kept in LDS
                      ROW_G = 16,       // a south ghost cell that follows from its rows
                      NEXT_S = 32, NEXT_N = 64,   // the cell next to such a ghost cell
                      MIRROR = 128,     // ... which is mirrored (symmetry), not extrapolated
                      LAST = 256, FIRST = 512,    // its north face is the north / south side's
                      BOUNCE = 1024, REFLECT = 2048 };   // ... and a wall / a symmetry plane there
    T ex, ey;                   // its ghost factors, beyond an x side and beyond a y side
    T bx[2], by[2];             // wall terms of its x-face and its y-face

    __device__ __forceinline__ Patch(const StepParams<T> &p, const S *s, S *d) : M(p, s, d, 0) {}

    // Patch (px, py): this lane's cell, its neighbours and its coefficients.
    __device__ __forceinline__ void place(const PatchGrid &G, int px, int py, int wave, int waves, T *lds) {
        const int nx = P.nx, ny = P.ny;
        const int ox0 = px * G.qx + min(px, G.rx), ox1 = ox0 + G.qx + (px < G.rx ? 1 : 0);
        const int oy0 = py * G.qy + min(py, G.ry), oy1 = oy0 + G.qy + (py < G.ry ? 1 : 0);
        const int c0 = this->per_x ? ox0 - G.halo : max(ox0 - G.halo, -1);
        const int r0 = this->per_y ? oy0 - G.halo : max(oy0 - G.halo, -1);
        // lanes past the last whole row of the wave repeat its last lane (and store nothing)
        const int l = min(lane, G.fit * G.tw - 1);
        const int seg = l / G.tw, c = l - seg * G.tw;
        const int col = c0 + c, row = r0 + wave * G.fit + seg;
        out = lane == l && col >= ox0 && col < ox1 && row >= oy0 && row < oy1;
        slot = wave * 64 + lane;
        up = lane == l ? slot_above(G, waves, wave, seg, c) : slot;
        down = lane == l ? slot_below(G, wave, seg, c) : slot;

        // a periodic axis wraps once; what is still outside belongs to lanes past the halo
        int cc = col, rr = row;
        if (this->per_x) cc += cc < 0 ? nx : (cc >= nx ? -nx : 0);
        if (this->per_y) rr += rr < 0 ? ny : (rr >= ny ? -ny : 0);
        cc = min(max(cc, 0), nx - 1);
        rr = min(max(rr, 0), ny - 1);
        off = (uint32_t)(((int64_t)rr * P.pitch + col_slot(cc, P.strip)) * (int64_t)sizeof(S));

        // the march's coefficients of this column (a periodic column takes its wrapped copy's)
        const T *lam = P.xm, *id = P.xm + (nx + 1), *is = P.xm + 2 * (nx + 1), *cd = is + nx;
        const int fW = this->per_x ? cc : min(max(col, 0), nx);
        const int fE = this->per_x ? cc + 1 : min(max(col + 1, 0), nx);
        const T lE = lam[fE], iE = id[fE], lW = lam[fW], iW = id[fW];
        this->cE0 = lE;
        this->cEp = fma(-P.hc, iE, lE);
        this->cEm = fma(P.hc, iE, lE);
        this->sLE = P.hc * ((T)1 - lE);
        this->cW0 = lW;
        this->cWp = fma(-P.hc, iW, lW);
        this->cWm = fma(P.hc, iW, lW);
        this->sRW = P.hc * lW;
        this->dxs = P.hc * is[cc];
        this->cdx = cd[cc];
        // and of its row: the north face is face row + 1 (a ghost row's is face 0)
        const int gN = this->per_y ? rr + 1 : min(max(row + 1, 0), ny);
        lamN = P.ym[gN];
        bnN = P.hc * P.ym[ny + 1 + gN];
        isy = P.ym[2 * (ny + 1) + rr];
        cdy = P.ym[3 * ny + 2 + rr];
        if (BND) {
            // a patch whose halo reaches beyond a side holds the side's ghost cells (kind -1: none)
            const int kW = !this->per_x && ox0 < G.halo ? P.bc[SIDE_W] : -1;
            const int kE = !this->per_x && ox1 + G.halo > nx ? P.bc[SIDE_E] : -1;
            const int kS = !this->per_y && oy0 < G.halo ? P.bc[SIDE_S] : -1;
            const int kN = !this->per_y && oy1 + G.halo > ny ? P.bc[SIDE_N] : -1;
            const int fromS = kS >= 0 ? P.wfrom[SIDE_S] : -1, fromN = kN >= 0 ? P.wfrom[SIDE_N] : -1;
            auto ext = [](int k) { return k == BC_WALL || k == BC_OUTFLOW; };
            sides = (ext(kW) ? EXT_W : 0) | (kW == BC_SYMMETRY ? MIR_W : 0) | (kW == BC_WALL ? WALL_W : 0) |
                    (ext(kE) ? EXT_E : 0) | (kE == BC_SYMMETRY ? MIR_E : 0) | (kE == BC_WALL ? WALL_E : 0) |
                    (kS >= 0 ? SOUTH : 0) | (kS == BC_SYMMETRY ? MIR_S : 0) | (kS == BC_WALL || fromS >= 0 ? WALL_S : 0) |
                    (kN >= 0 ? NORTH : 0) | (kN == BC_SYMMETRY ? MIR_N : 0) | (kN == BC_WALL || fromN >= 0 ? WALL_N : 0);
            const bool segS = fromS >= 0 && col >= fromS, segN = fromN >= 0 && col >= fromN;
            const bool southern = row <= 0, seg_y = southern ? segS : segN;
            const int sx = col <= 0 ? SIDE_W : SIDE_E, sy = southern ? SIDE_S : SIDE_N, ky = southern ? kS : kN;
            const bool beyond_x = (kW >= 0 && col == -1) || (kE >= 0 && col == nx);
            const bool beyond_y = (kS >= 0 && row == -1) || (kN >= 0 && row == ny);
            // (the y side's rule holds in the corners)
            const bool fixed = beyond_y ? ky == BC_INFLOW && !seg_y : beyond_x && (col == -1 ? kW : kE) == BC_INFLOW;
            const bool rule = ky >= 0 && (seg_y || ky != BC_INFLOW);   // ghost rows that follow from their rows
            const bool first = kS >= 0 && row == -1, last = kN >= 0 && row == ny - 1;
            part = (col == -1 ? GHOST_W : 0) | (col == 0 ? FACE_W : 0) | (col == nx ? GHOST_E : 0) | (fixed ? FIXED : 0) |
                   (first && rule && lane == l ? ROW_G : 0) | (rule && row == 0 && kS >= 0 ? NEXT_S : 0) |
                   (last && kN >= 0 && (segN || kN != BC_INFLOW) ? NEXT_N : 0) | (last ? LAST : 0) | (first ? FIRST : 0);
            // a one-row mesh has no rule of its own here: ny >= 2, so row 0 is not row ny - 1
            if (ky == BC_SYMMETRY && !seg_y) part |= MIRROR;
            if ((first || last) && (ky == BC_WALL || seg_y)) part |= BOUNCE;
            if ((first || last) && ky == BC_SYMMETRY && !seg_y) part |= REFLECT;
            if (part & ROW_G) down = slot_above(G, waves, up >> 6, ((up & 63) - c) / G.tw, c);   // its second row: row 1
            if (fixed) {
                const int side = beyond_y ? sy : sx;
#pragma unroll
                for (int a = 0; a < 9; ++a) lds[slot * PATCH_LDS + a] = P.gin[side][a];
            }
            ex = P.gext[sx];
            ey = seg_y ? P.ext[sy] : P.gext[sy];
            bx[0] = P.bcv[sx][0];
            bx[1] = P.bcv[sx][1];
            by[0] = seg_y ? P.wsv[sy][0] : P.bcv[sy][0];
            by[1] = seg_y ? P.wsv[sy][1] : P.bcv[sy][1];
        }
    }
    __device__ __forceinline__ int slot_above(const PatchGrid &G, int waves, int wave, int seg, int c) const {
        return seg + 1 < G.fit ? wave * 64 + (seg + 1) * G.tw + c
                               : (wave + 1 < waves ? (wave + 1) * 64 + c : wave * 64 + seg * G.tw + c);
    }
    __device__ __forceinline__ int slot_below(const PatchGrid &G, int wave, int seg, int c) const {
        return seg > 0 ? wave * 64 + (seg - 1) * G.tw + c
                       : (wave > 0 ? (wave - 1) * 64 + (G.fit - 1) * G.tw + c : wave * 64 + c);
    }

    // A value whose use stays where it is written: the compiler otherwise forms the wall terms of
    // all directions before the loop and holds 16 registers for them.
    static __device__ __forceinline__ T here(T v) {
        asm volatile("" : "+v"(v));
        return v;
    }

    // the march's yface with this lane's own metrics
    __device__ __forceinline__ void north_face(const T (&lo)[9], const T (&hi)[9], T (&fb)[9]) const {
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const T dn = hi[a] - lo[a];
            const T q = fma(lamN, dn, lo[a]);
            T v = q;
            if (EY[a] != 0) v = fma(EY[a] > 0 ? -bnN : bnN, dn, v);
            if (EX[a] != 0) v = fma(EX[a] > 0 ? -this->dxs : this->dxs, shl1(q) - shr1(q), v);
            fb[a] = v;
        }
    }

    // The ghost columns of a row (x sides first, as in the march; inflow states stay in LDS): the
    // march's ghost rule, one branch per kind of side.
    __device__ __forceinline__ void ghost_columns(T (&phi)[9]) const {
        const bool w = part & GHOST_W, e = part & GHOST_E;
        if (sides & MIR_W) {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const T m = shl1(phi[MIRX[a]]);
                phi[a] = w ? m : phi[a];
            }
        }
        if (sides & EXT_W) {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const T g1 = shl1(phi[a]), g2 = shl1(g1);
                const T v = fma(g1 - g2, ex, g1);
                phi[a] = w ? v : phi[a];
            }
        }
        if (sides & MIR_E) {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const T m = shr1(phi[MIRX[a]]);
                phi[a] = e ? m : phi[a];
            }
        }
        if (sides & EXT_E) {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const T g1 = shr1(phi[a]), g2 = shr1(g1);
                const T v = fma(g1 - g2, ex, g1);
                phi[a] = e ? v : phi[a];
            }
        }
    }

    // the ghost rule beyond a y side from the adjacent row r1 and the next one r2
    __device__ __forceinline__ void ghost_of(const T (&r1)[9], const T (&r2)[9], T (&out)[9]) const {
        const bool mirror = part & MIRROR;
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const T v = fma(r1[a] - r2[a], ey, r1[a]);
            out[a] = mirror ? r1[MIRY[a]] : v;
        }
    }

    // `steps` (at most G.halo) time steps of patch (px, py); lds holds PATCH_LDS values per lane
    __device__ __forceinline__ void run(const PatchGrid &G, int px, int py, int steps, T *lds) {
        const int waves = (int)(blockDim.x >> 6);
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        place(G, px, py, wave, waves, lds);
        T *const mine = lds + slot * PATCH_LDS;
        const T *const above = lds + up * PATCH_LDS, *const below = lds + down * PATCH_LDS;
        const int bytes = (int)(P.plane * (int64_t)sizeof(S));
        T x[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const __amdgpu_buffer_rsrc_t b =
                __builtin_amdgcn_make_buffer_rsrc((void *)(this->src + a * P.plane), (short)0, bytes, kBufWord3);
            x[a] = Storage<S>::load(BufIO<S>::load(b, off), a);
        }
        for (int s = 0; s < steps; ++s) {
            T phi[9], psi[9];
            this->cell_t(x, phi, psi);
            if constexpr (BND) ghost_columns(phi);
            if (!BND || !(part & FIXED)) {
#pragma unroll
                for (int a = 0; a < 9; ++a) mine[a] = phi[a];
            }
            __syncthreads();
            T hi[9], lo[9];
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                hi[a] = above[a];
                lo[a] = BND || EY[a] != 0 ? below[a] : (T)0;
            }
            if (BND && (part & FIXED)) {
#pragma unroll
                for (int a = 0; a < 9; ++a) phi[a] = mine[a];
            }
            if (BND && (sides & SOUTH)) {
                if (part & ROW_G) ghost_of(hi, lo, phi);   // (lo holds row 1 there)
                if (part & NEXT_S) ghost_of(phi, hi, lo);
            }
            if (BND && (sides & NORTH)) {
                if (part & NEXT_N) ghost_of(phi, lo, hi);
            }
            T dy[9];
#pragma unroll
            for (int a = 0; a < 9; ++a) dy[a] = EY[a] != 0 ? hi[a] - lo[a] : (T)0;
            // the north face first: its values are what the row above waits for
            T fN[9];
            north_face(phi, hi, fN);
            // (a south ghost cell's north face is the south face of row 0)
            if (BND && (sides & WALL_N)) this->template bounce<0, 1>(fN, here(by[0]), here(by[1]), (part & (LAST | BOUNCE)) == (LAST | BOUNCE));
            if (BND && (sides & MIR_N)) this->template specular<0, 1>(fN, (part & (LAST | REFLECT)) == (LAST | REFLECT));
            if (BND && (sides & WALL_S)) this->template bounce<0, -1>(fN, here(by[0]), here(by[1]), (part & (FIRST | BOUNCE)) == (FIRST | BOUNCE));
            if (BND && (sides & MIR_S)) this->template specular<0, -1>(fN, (part & (FIRST | REFLECT)) == (FIRST | REFLECT));
            this->template face_mix<1>(fN);
            int q = 0;
#pragma unroll
            for (int a = 0; a < 9; ++a)
                if (EY[a] != 0) mine[9 + q++] = fN[a];
            // x-faces while the row below writes
            T fW[9];
            this->xface(phi, dy, isy, fW);
            if (BND && (sides & WALL_W)) this->template bounce<-1, 0>(fW, here(bx[0]), here(bx[1]), part & FACE_W);
            if (BND && (sides & MIR_W)) this->template specular<-1, 0>(fW, part & FACE_W);
            if (BND && (sides & WALL_E)) this->template bounce<1, 0>(fW, here(bx[0]), here(bx[1]), part & GHOST_E);
            if (BND && (sides & MIR_E)) this->template specular<1, 0>(fW, part & GHOST_E);
            this->template face_mix<0>(fW);
            __syncthreads();
            q = 0;
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                T u = (SCHEME == SCHEME_DUGKS) ? psi[a] : phi[a];
                if (EX[a] != 0) {
                    const T fE = shl1(fW[a]);
                    u = fma(EX[a] > 0 ? -this->cdx : this->cdx, fE - fW[a], u);
                }
                if (EY[a] != 0) {
                    const T fS = below[9 + q++];
                    u = fma(EY[a] > 0 ? -cdy : cdy, fN[a] - fS, u);
                }
                // what a one-step launch would store and read back
                x[a] = sizeof(S) == 2 ? Storage<S>::load(Storage<S>::store(u, a), a) : u;
            }
        }
        if (out) {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const __amdgpu_buffer_rsrc_t b =
                    __builtin_amdgcn_make_buffer_rsrc((void *)(this->dst + a * P.plane), (short)0, bytes, kBufWord3);
                BufIO<S>::store(Storage<S>::store(x[a], a), b, off);
            }
        }
    }
};

// One launch = `steps` time steps of one case, one workgroup per patch.  Doubly periodic meshes
// take the parameters by value, meshes with a non-periodic side through a device copy, as the
// step kernels do.
template <typename T, typename S, int SCHEME, bool REF>
__global__ __launch_bounds__(64 * PATCH_WAVES) void patch_kernel(StepParams<T> P, int parity, int steps, PatchGrid G) {
    extern __shared__ char patch_lds[];
    const int b = xcd_block();
    const int py = b / G.npx, px = b - py * G.npx;
    Patch<T, S, SCHEME, false, REF> m(P, (const S *)P.buf[parity], (S *)P.buf[parity ^ 1]);
    m.run(G, px, py, steps, (T *)patch_lds);
}
template <typename T, typename S, int SCHEME, bool REF>
__global__ __launch_bounds__(64 * PATCH_WAVES) void patch_ptr_kernel(const StepParams<T> *__restrict__ Pp, int parity,
                                                                     int steps, PatchGrid G) {
    extern __shared__ char patch_lds[];
    const StepParams<T> &P = *Pp;
    const int b = xcd_block();
    const int py = b / G.npx, px = b - py * G.npx;
    Patch<T, S, SCHEME, true, REF> m(P, (const S *)P.buf[parity], (S *)P.buf[parity ^ 1]);
    m.run(G, px, py, steps, (T *)patch_lds);
}

// The batched form: one workgroup per patch of any case; each case has its own mesh and patches,
// all patches the same waves and at most the same steps.
struct PatchItem {
    int32_t c, px, py;
};
template <typename T, typename S, int SCHEME, bool BND>
__global__ __launch_bounds__(64 * PATCH_WAVES) void batch_patch_kernel(const StepParams<T> *__restrict__ cases,
                                                                       const PatchGrid *__restrict__ grids,
                                                                       const PatchItem *__restrict__ items, int parity,
                                                                       int steps) {
    extern __shared__ char patch_lds[];
    const PatchItem it = items[xcd_block()];
    const StepParams<T> &P = cases[it.c];
    const PatchGrid G = grids[it.c];
    Patch<T, S, SCHEME, BND, false> m(P, (const S *)P.buf[parity], (S *)P.buf[parity ^ 1]);
    m.run(G, it.px, it.py, steps, (T *)patch_lds);
}

}  // namespace lbfv
