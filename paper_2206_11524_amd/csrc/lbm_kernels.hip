// HIP kernels (gfx950) of the HMCSC lattice Boltzmann update.
//
// Layout in HBM: populations are grouped by plane.  For one component the 19
// direction arrays of plane z lie next to each other, P[((s*nz + z)*19 + i)*
// plane + n], n = y*nx + x the in-plane index ("split" layout, FP64 and
// single-component runs).  Two-component runs in FP32 and the 16-bit formats
// keep the two components of one (cell, direction) in one word (64 or 32
// bits), P[(((z*19 + i)*plane + n) << 1) + s] ("pair" layout), so one load
// brings both.
// Streaming is "pull": a buffer holds the populations that left each cell at
// the previous step, so the pre-collision state of Eq. (LGS) at cell x is
// f_i(x) = P_i(x - c_i) (periodic).  Every stored value is shifted,
// h = f - w_i*rho0_s (scaled by 2^k for the 16-bit formats); the whole
// collision is written in the shifted variables (the shift cancels in the
// partial bounce-back blend because w_ibar = w_i), which keeps small deviations
// representable in reduced precision.
//
// The step kernels are fused 2.5-D sweeps: a block owns a column of w x h
// cells and marches along z.  For every plane it pulls the populations of its
// cells once (kept for the collision of a later iteration), forms the
// densities, and stages them in LDS together with a one-cell ring of densities
// recomputed from the ring cells' populations, plus the n_s field.  The
// cohesion force (Eq. SC_F_inter) and adhesion force (Eq. SC_F_ads) then read
// their 18 neighbours from LDS, so HBM sees each population read once and
// written once per step (ring and z-halo re-reads hit L2/MALL).  Every plane
// is addressed through its own buffer descriptor (base = start of the plane
// block, 64-bit, built on the scalar unit), so no 32-bit offset spans more
// than one plane and domains of any size that fits the device are addressed.
#include "lbm_device.h"

#include <algorithm>

namespace hm {

// One thread per (cell, component): a block of NC*kCells threads owns a column of
// w x h cells; threads [s*kCells, (s+1)*kCells) handle component s.  The two
// components of a cell meet only through LDS (densities and first moments),
// which halves the registers per thread and doubles the waves per CU.
//
// LDS holds four density / n_s plane slots (plane p in slot p mod 4) and three
// first-moment slots (p mod 3), so one barrier per plane suffices: a wave that
// runs ahead into staging plane z+2 writes slots that no wave still colliding
// plane z reads, and every wave has left the collision of plane z-1 before the
// barrier that precedes the collision of plane z.
//
// A tile is any w x h cells of at most kCells with rows of up to 64 and at most
// kRows rows, fitted to the domain like the pair sweep's (the row bound keeps the
// staged planes within the 160 KB of LDS; lanes take the cells row by row).
template <typename ST, int NC, int CNS, int CELLS = split_cells(sizeof(typename ST::T) == 8, NC)>
struct TileShared {
    using T = typename ST::T;
    static constexpr int kCells = CELLS;
    static constexpr int kRows =
        CELLS < split_cells(sizeof(T) == 8, NC) ? kThinRows : split_rows(sizeof(T) == 8, NC, CNS);
    static constexpr int kStaged = 66 * (kCells / 64 + 2);  // cells of a tile with its ring, at most
    static constexpr int LW = 66;
    static constexpr int LP = LW * (kRows + 2);
    static constexpr int NTC = kCells;
    static constexpr int NT = NC * NTC;
    // the populations of the plane staged last wait here (private to each
    // thread) until it is collided, which frees the registers that keep the
    // next plane's loads in flight
    T hs[kQ][NT];
    T rho[4][NC][LP];
    float ns[4][CNS][LP];
    T j[NC == 2 ? 3 : 1][NC][3][NC == 2 ? NTC : 1];
};

// The sweep of one tile column (logical tile index L of the domain described
// by a).  Shared by the single-domain and the batched kernels.
template <typename ST, int NC, int CNS, int FS, bool ONE, int AUX, int CELLS>
__device__ __forceinline__ void step_tile(const Args<typename ST::T>& a, const typename ST::E* __restrict__ A,
                                          typename ST::E* __restrict__ B, const float* __restrict__ ns, int L,
                                          uint32_t t, TileShared<ST, NC, CNS, CELLS>& sh)
{
    using T = typename ST::T;
    using E = typename ST::E;
    using Shared = TileShared<ST, NC, CNS, CELLS>;
    constexpr int LW = Shared::LW, LP = Shared::LP;
    constexpr int NTC = Shared::NTC;  // threads per component
    constexpr int NT = Shared::NT;
    constexpr int NSMAX = (Shared::kStaged + NT - 1) / NT;  // n_s cells staged per thread and plane
    auto& s_rho = sh.rho;
    auto& s_ns = sh.ns;
    auto& s_j = sh.j;

    const int tx = L % a.ntx;
    const int ty = (L / a.ntx) % a.nty;
    const int tz = L / (a.ntx * a.nty);
    const int x0 = tx * a.tw, y0 = ty * a.th;
    const int zs = tz * a.zchunk;
    const int ze = min(zs + a.zchunk, a.nz);
    const int TXe = min(a.tw, a.nx - x0);
    const int TYe = min(a.th, a.ny - y0);
    const int plane = a.nx * a.ny;

    // component of this thread; NTC is a multiple of 64, so it is the same
    // for every lane of a wave: saying so keeps the buffer descriptors and
    // everything derived from s in scalar registers (otherwise each load
    // becomes a loop over the distinct descriptor values of the wave)
    const int s = NC == 1 ? 0 : __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / NTC);
    static_assert(NTC % 64 == 0, "a wave must not straddle two components");
    const int tl = static_cast<int>(threadIdx.x) - s * NTC;
    // a lane beyond the last cell duplicates it
    const int tj = min(tl, TXe * TYe - 1);  // cell of the tile, first-moment slot
    const int ly = TXe == 64 ? tj >> 6 : tj / TXe;
    const int x = x0 + (tj - ly * TXe);
    const int y = y0 + ly;
    const int me = (ly + 1) * LW + (x - x0 + 1);  // LDS cell
    const PlaneOffs qme = plane_offs<sizeof(E)>(x, y, a.nx, a.ny);
    const uint32_t own = static_cast<uint32_t>(y * a.nx + x) * static_cast<uint32_t>(sizeof(E));

    // ring cell of this thread (if any): top row, bottom row, left, right column
    const int ring_n = 2 * (TXe + 2) + 2 * TYe;
    const bool ring = NC == 2 && tl < ring_n;  // only the cohesion stencil reads ring densities
    int rlx, rly;
    {
        const int r = min(tl, ring_n - 1);
        if (r < TXe + 2) { rlx = r - 1; rly = -1; }
        else if (r < 2 * (TXe + 2)) { rlx = r - (TXe + 2) - 1; rly = TYe; }
        else if (r < 2 * (TXe + 2) + TYe) { rlx = -1; rly = r - 2 * (TXe + 2); }
        else { rlx = TXe; rly = r - 2 * (TXe + 2) - TYe; }
    }
    const int rx = ((x0 + rlx) % a.nx + a.nx) % a.nx;
    const int ry = ((y0 + rly) % a.ny + a.ny) % a.ny;
    const int rme = (rly + 1) * LW + (rlx + 1);
    const PlaneOffs qring = plane_offs<sizeof(E)>(rx, ry, a.nx, a.ny);

    // n_s cells staged by this thread: LDS index and in-plane offset
    const int nsw = TXe + 2, nsh = TYe + 2;
    int ns_lds[NSMAX], ns_off[NSMAX];
#pragma unroll
    for (int k = 0; k < NSMAX; ++k) {
        const int c = static_cast<int>(threadIdx.x) + k * NT;
        if (c < nsw * nsh) {
            const int llx = c % nsw - 1, lly = c / nsw - 1;
            const int gx = ((x0 + llx) % a.nx + a.nx) % a.nx;
            const int gy = ((y0 + lly) % a.ny + a.ny) % a.ny;
            ns_lds[k] = (lly + 1) * LW + llx + 1;
            ns_off[k] = gy * a.nx + gx;
        } else {
            ns_lds[k] = -1;
            ns_off[k] = 0;
        }
    }

    auto wrapz = [&](int p) { return p < 0 ? p + a.nz : (p >= a.nz ? p - a.nz : p); };
    const uint32_t t_key = fmix32(t ^ kGolden);  // stochastic rounding: time part of the counter

    // The 19 direction arrays of one plane of this component form a block;
    // each plane block is addressed through its own buffer descriptor (64-bit
    // base on the scalar unit, 32-bit offsets within the block).
    const size_t cstride = static_cast<size_t>(a.nz) * kQ * static_cast<size_t>(plane);
    const E* Ac = A + static_cast<size_t>(s) * cstride;
    E* Bc = B + static_cast<size_t>(s) * cstride;
    const uint32_t dir_bytes = static_cast<uint32_t>(plane) * static_cast<uint32_t>(sizeof(E));
    const uint32_t blk_bytes = static_cast<uint32_t>(kQ) * dir_bytes;
    auto blk = [&](const E* base, int p) {
        return make_rsrc(base + static_cast<size_t>(p) * kQ * static_cast<size_t>(plane), blk_bytes);
    };

    // A select per value rather than a per-lane branch: in divergent control
    // flow a branch makes the compiler merge the two versions of all 19
    // values through copies, doubling the registers they hold.  The selects
    // are skipped as a whole when no lane of the wave is in a reservoir (the
    // common case; a branch taken by the whole wave).
    auto reservoir_override = [&](int cx, int cy, int cz, T h[kQ]) {
        T dr;
        const bool in = reservoir_dr(a, s, cx, cy, cz, dr);
        if (__builtin_amdgcn_ballot_w64(in) != 0) {
#pragma unroll
            for (int i = 0; i < kQ; ++i) h[i] = in ? wgt<T>(i) * dr : h[i];
        }
    };

    // Collision of plane z of this thread's component from h (pre-collision,
    // shifted) and the LDS slots of planes z-1, z, z+1.
    const TileGeom<LW, LP> geo;
    auto collide = [&](int z, int sm, int s0, int sp, int js, const T h[kQ]) {
        T jc[NC][3];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (NC == 1) {
                jc[c][0] = first_moment<T, 0>(h);
                jc[c][1] = first_moment<T, 1>(h);
                jc[c][2] = first_moment<T, 2>(h);
            } else {
#pragma unroll
                for (int d = 0; d < 3; ++d) jc[c][d] = s_j[js][c][d][tj];
            }
        }
        const rsrc_t rz = blk(Bc, z);
        const uint32_t cell =
            static_cast<uint32_t>(z) * static_cast<uint32_t>(plane) + static_cast<uint32_t>(y * a.nx + x);
        split_collide<ST, NC, CNS, FS>(
            geo, a, s, t_key, cell, me, &s_rho[sm][0][0], &s_rho[s0][0][0], &s_rho[sp][0][0], &s_ns[sm][0][0],
            &s_ns[s0][0][0], &s_ns[sp][0][0], jc, h,
            [&](int i, E v) { raw_store<AUX>(v, rz, own, static_cast<uint32_t>(i) * dir_bytes); });
    };

    // plane p (zs-1 <= p <= ze) uses density slot (p - zs + 1) mod 4 and
    // first-moment slot (p - zs) mod 3
    auto rslot = [&](int p) { return (p - zs + 1) & 3; };
    auto jslot = [&](int p) { return (p - zs) % 3; };

    // Three planes at a time: plane z is collided from registers, plane
    // z+1 waits in LDS (hs), and the own loads of plane z+2 are in flight
    // over the barrier and the collision of plane z.
    //
    // The compiler counts outstanding memory operations per control-flow
    // path, and after a branch that may have skipped some it has to wait
    // as if they had been issued last; a load or store under a per-lane
    // condition would therefore make every later wait drain the loads
    // kept in flight.  So nothing here touches memory conditionally:
    // lanes beyond a ragged tile edge duplicate an active lane (same
    // cell, same LDS slots, identical values written twice), lanes
    // without a ring cell load the tile's last ring cell (a cell of the
    // domain; the values are not used), and lanes without an n_s cell
    // duplicate cell 0 of the staging list.
    T* hs = &sh.hs[0][0] + threadIdx.x;
    const PlaneOffs& qr = qring;
    // list cell 0 is the corner (x0 - 1, y0 - 1), LDS index 0
    const int ns_off0 = (((y0 - 1) % a.ny + a.ny) % a.ny) * a.nx + ((x0 - 1) % a.nx + a.nx) % a.nx;
    int nl[NSMAX], no[NSMAX];
#pragma unroll
    for (int k = 0; k < NSMAX; ++k) {
        nl[k] = ns_lds[k] >= 0 ? ns_lds[k] : 0;
        no[k] = ns_lds[k] >= 0 ? ns_off[k] : ns_off0;
    }
    auto issue = [&](int p, const PlaneOffs& q, E e[kQ]) {
        const rsrc_t r3[3] = {blk(Ac, wrapz(p + 1)), blk(Ac, p), blk(Ac, wrapz(p - 1))};
        pull_raw<ST>(r3, dir_bytes, q, e);
    };
    if constexpr (ONE) {
        // One cell deep (the instance launched for nz = 1): planes z - 1,
        // z and z + 1 are all plane 0, so it is staged once and collided
        // against itself (one memory round trip per step instead of the
        // sweep's three; the three slots the sweep would fill hold the
        // same values).  A kernel of its own: as a branch in the 3-D
        // kernels it changed their register allocation.
        const int slot = rslot(0), js = jslot(0);
        E r1[kQ];
        E r2[NC == 2 ? kQ : 1];
        issue(0, qme, r1);
        if constexpr (NC == 2) issue(0, qr, r2);
        float nsv[NSMAX][CNS];
#pragma unroll
        for (int k = 0; k < NSMAX; ++k)
#pragma unroll
            for (int c = 0; c < CNS; ++c) nsv[k][c] = ns[static_cast<size_t>(c) * a.N + no[k]];
        T h[kQ];
#pragma unroll
        for (int i = 0; i < kQ; ++i) h[i] = ST::dec(r1[i], a.inv_scale);
        reservoir_override(x, y, 0, h);
        s_rho[slot][s][me] = a.rho0[s] + sum19(h);
        if constexpr (NC == 2) {
            s_j[js][s][0][tj] = first_moment<T, 0>(h);
            s_j[js][s][1][tj] = first_moment<T, 1>(h);
            s_j[js][s][2][tj] = first_moment<T, 2>(h);
            if (ring) {
                T hr[kQ];
#pragma unroll
                for (int i = 0; i < kQ; ++i) hr[i] = ST::dec(r2[i], a.inv_scale);
                reservoir_override(rx, ry, 0, hr);
                s_rho[slot][s][rme] = a.rho0[s] + sum19(hr);
            }
        }
#pragma unroll
        for (int k = 0; k < NSMAX; ++k)
#pragma unroll
            for (int c = 0; c < CNS; ++c) s_ns[slot][c][nl[k]] = nsv[k][c];
        __syncthreads();
        collide(0, slot, slot, slot, js, h);
        return;
    }
    if constexpr (sizeof(E) == 8 || (sizeof(E) == 4 && FS == kForcingGuo)) {
        E rr[kQ];  // own populations of the next plane to stage, raw
        E er[kQ];  // ring populations of the plane being staged, raw
        // Stage plane p, whose own loads are in rr: ring loads and n_s are
        // issued first; the own values give the density and first moments
        // and go to hs, whose previous content (the plane before) moves to
        // hz; then the own loads of plane pn are issued, and only after them
        // the ring values are consumed, so a wait for the ring does not wait
        // for plane pn.
        auto stage_pipe = [&](int p, int slot, int js, int pn, T hz[kQ]) {
            if constexpr (NC == 2) issue(p, qr, er);
            const float* nsp = ns + static_cast<size_t>(p) * plane;
            float nsv[NSMAX][CNS];
#pragma unroll
            for (int k = 0; k < NSMAX; ++k)
#pragma unroll
                for (int c = 0; c < CNS; ++c) nsv[k][c] = nsp[static_cast<size_t>(c) * a.N + no[k]];
            __builtin_amdgcn_sched_barrier(0);
            {
                T h[kQ];
#pragma unroll
                for (int i = 0; i < kQ; ++i) h[i] = ST::dec(rr[i], a.inv_scale);
                reservoir_override(x, y, p, h);
                s_rho[slot][s][me] = a.rho0[s] + sum19(h);
                if (NC == 2 && js >= 0) {
                    s_j[js][s][0][tj] = first_moment<T, 0>(h);
                    s_j[js][s][1][tj] = first_moment<T, 1>(h);
                    s_j[js][s][2][tj] = first_moment<T, 2>(h);
                }
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    hz[i] = hs[i * NT];
                    hs[i * NT] = h[i];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            issue(pn, qme, rr);
            __builtin_amdgcn_sched_barrier(0);
            if (ring) {
                T hr[kQ];
#pragma unroll
                for (int i = 0; i < kQ; ++i) hr[i] = ST::dec(er[i], a.inv_scale);
                reservoir_override(rx, ry, p, hr);
                s_rho[slot][s][rme] = a.rho0[s] + sum19(hr);
            }
#pragma unroll
            for (int k = 0; k < NSMAX; ++k)
#pragma unroll
                for (int c = 0; c < CNS; ++c) s_ns[slot][c][nl[k]] = nsv[k][c];
        };

        T hz[kQ];
        // prologue: plane zs-1 (densities only), plane zs (to hs)
        issue(wrapz(zs - 1), qme, rr);
        stage_pipe(wrapz(zs - 1), rslot(zs - 1), -1, zs, hz);
        stage_pipe(zs, rslot(zs), jslot(zs), wrapz(zs + 1), hz);
        for (int z = zs; z < ze; ++z) {
            // after the last plane the next loads repeat the one just staged (L2 hits)
            const int pn = z + 2 <= ze ? wrapz(z + 2) : wrapz(z + 1);
            stage_pipe(wrapz(z + 1), rslot(z + 1), jslot(z + 1), pn, hz);
            __syncthreads();
            collide(z, rslot(z - 1), rslot(z), rslot(z + 1), jslot(z), hz);
        }
    } else {
        // One component in FP32 or a 16-bit format (two components run
        // the pair kernel): no ring, and in 16-bit two planes of own loads
        // in flight (a wave has at most 63 memory operations outstanding,
        // and the 16-bit loads carry half the bytes each; for FP32 the
        // deeper prefetch did not pay).
        static_assert(NC == 1, "two components in FP32 or 16-bit run the pair kernel");
        constexpr bool DEEP = sizeof(E) == 2;
        constexpr int AHEAD = DEEP ? 2 : 1;  // planes between issue and consumption
        E rA[kQ];
        E rB[DEEP ? kQ : 1];
        // Stage plane p, whose own loads are in rc: the n_s loads are
        // issued first; the own values give the density and go to hs,
        // whose previous content (the plane before) moves to hz; then the
        // own loads of plane pn are issued into rc.
        auto stage_pipe = [&](int p, int slot, int pn, T hz[kQ], E rc[kQ]) {
            const float* nsp = ns + static_cast<size_t>(p) * plane;
            float nsv[NSMAX][CNS];
#pragma unroll
            for (int k = 0; k < NSMAX; ++k)
#pragma unroll
                for (int c = 0; c < CNS; ++c) nsv[k][c] = nsp[static_cast<size_t>(c) * a.N + no[k]];
            __builtin_amdgcn_sched_barrier(0);
            {
                T h[kQ];
#pragma unroll
                for (int i = 0; i < kQ; ++i) h[i] = ST::dec(rc[i], a.inv_scale);
                reservoir_override(x, y, p, h);
                s_rho[slot][s][me] = a.rho0[s] + sum19(h);
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    hz[i] = hs[i * NT];
                    hs[i * NT] = h[i];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            issue(pn, qme, rc);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < NSMAX; ++k)
#pragma unroll
                for (int c = 0; c < CNS; ++c) s_ns[slot][c][nl[k]] = nsv[k][c];
        };
        // the plane whose loads a stage of plane p issues: p + AHEAD, or
        // after the last plane one already staged again (L2 hits)
        auto ahead = [&](int p) { return wrapz(p + AHEAD <= ze ? p + AHEAD : ze); };
        // register sets: planes zs-1, zs+1, ... in r_odd, planes zs, zs+2, ...
        // in r_even (one and the same set unless two planes are in flight)
        E (&r_odd)[kQ] = rA;
        E (&r_even)[kQ] = *reinterpret_cast<E(*)[kQ]>(DEEP ? static_cast<E*>(rB) : static_cast<E*>(rA));

        T hz[kQ];
        // prologue: planes zs-1 (densities only) and zs (to hs)
        issue(wrapz(zs - 1), qme, r_odd);
        if constexpr (DEEP) issue(zs, qme, r_even);
        stage_pipe(wrapz(zs - 1), rslot(zs - 1), ahead(zs - 1), hz, r_odd);
        stage_pipe(zs, rslot(zs), ahead(zs), hz, r_even);
        // unrolled by two so the register sets keep fixed names
        for (int z = zs; z < ze; z += 2) {
            stage_pipe(wrapz(z + 1), rslot(z + 1), ahead(z + 1), hz, r_odd);
            __syncthreads();
            collide(z, rslot(z - 1), rslot(z), rslot(z + 1), jslot(z), hz);
            if (z + 1 >= ze) break;
            stage_pipe(wrapz(z + 2), rslot(z + 2), ahead(z + 2), hz, r_even);
            __syncthreads();
            collide(z + 1, rslot(z), rslot(z + 1), rslot(z + 2), jslot(z + 1), hz);
        }
    }
}

// ---------------------------------------------------------------------------
// Pair kernel: two components in FP32 or a 16-bit format, one thread per cell.
//
// In the pair layout one word (32 bits for the 16-bit formats, 64 for FP32)
// holds both components' value of one (cell, direction), so a thread pulls
// its cell's 38 populations with 19 loads and stores them with 19 stores.
// Per memory operation that moves twice the bytes of a lone value, which
// doubles the bytes a wave keeps in flight under the same limit on
// outstanding operations and halves the memory instructions per cell.  The two
// components of a cell meet in registers, so the first moments need no LDS
// exchange; the densities still go to LDS for the force stencils.
//
// The waves of a block have fixed roles.  The first CELLS threads own one
// cell each: they pull, collide and store it, with the next plane's loads in
// flight.  The last NR threads (whole waves) stage the one-cell ring of
// densities around the tile and the n_s planes: they hold no collision state,
// so the cell waves keep their registers for the prefetch.
//
// LDS: four density / n_s plane slots (plane p in slot p mod 4, one barrier
// per plane) and the raw words of the last planes staged, private to each
// cell thread.  16-bit: two planes, and the collision reads its plane's words
// from LDS, so no register holds them while two planes of loads are in
// flight.  FP32: one plane (its words take twice the room), the plane being
// collided in registers, one plane of loads in flight.
//
// A tile is any w x h cells of at most 512, rows of up to 64: the host fits it
// to the domain (choose_launch), and the lanes take its cells row by row
// without gaps, so a width that is no multiple of 64 leaves few lanes idle.  A
// plane costs a block 3.5 us of its CU's issue slots and waits in 16 bits, with
// or without idle lanes, against 3.7 us of HBM time for 512 cells with every CU
// at work: on ragged domains idle lanes were the bound (131^3 in FP16, 66 % of
// the lanes: 136 us a step with 64 x 8 tiles, 108 with 44 x 11).  The LDS row
// stride stays 66, so that every stencil offset is an instruction's immediate
// (a run-time stride cost FP32 eight registers and spilled); the words come
// first in LDS because their 78 KB reach past the 64 KB of such offsets.
constexpr int kPairCells = 512;    // cells of a tile (one thread each), at most
constexpr int kPairW = 64;         // cells of a tile row, at most
constexpr int kPairH = 16;         // rows of a tile, at most
constexpr int kPairRing = 192;     // ring / n_s threads per block (three waves)
static_assert(2 * (kPairW + 2) + 2 * kPairH <= kPairRing, "one ring cell per ring thread");

template <typename ST, int CNS, int CELLS = kPairCells>
struct PairShared {
    using W = typename PairWordOf<ST>::W;
    static constexpr int LW = kPairW + 2;
    static constexpr int LP = LW * ((CELLS < kPairCells ? kThinRows : kPairH) + 2);
    static constexpr int NT = CELLS;
    static constexpr int kStaged = LW * (CELLS / kPairW + 2);  // cells of a tile with its ring, at most
    static constexpr int NB = sizeof(W) == 4 ? 2 : 1;  // planes of words held in LDS
    W hs[NB][kQ][NT];
    float rho[4][2][LP];
    float ns[4][CNS][LP];
};

// Planes a cell wave keeps in flight ahead of the one it stages (1 or 2).
#ifndef LBM_PAIR_AHEAD
#define LBM_PAIR_AHEAD 2
#endif

template <typename ST, int CNS, int FS, bool ONE, int RND, int AUX, int CELLS>
__device__ __forceinline__ void step_tile_pair(const Args<float>& a,
                                               const typename PairWordOf<ST>::W* __restrict__ A,
                                               typename PairWordOf<ST>::W* __restrict__ B,
                                               const float* __restrict__ ns, int L, uint32_t t,
                                               PairShared<ST, CNS, CELLS>& sh)
{
    using T = float;
    using W = typename PairWordOf<ST>::W;
    using Shared = PairShared<ST, CNS, CELLS>;
    constexpr int LW = Shared::LW, LP = Shared::LP;
    constexpr int NT = CELLS;
    constexpr int NR = kPairRing;
    constexpr int NSR = (Shared::kStaged + NR - 1) / NR;  // n_s cells staged per ring thread and plane
    static_assert(NT % 64 == 0, "the roles must fill whole waves");
    auto& s_rho = sh.rho;
    auto& s_ns = sh.ns;

    const int tx = L % a.ntx;
    const int ty = (L / a.ntx) % a.nty;
    const int tz = L / (a.ntx * a.nty);
    const int x0 = tx * a.tw, y0 = ty * a.th;
    const int zs = tz * a.zchunk;
    const int ze = min(zs + a.zchunk, a.nz);
    const int TXe = min(a.tw, a.nx - x0);
    const int TYe = min(a.th, a.ny - y0);
    const TileGeom<LW, LP> geo;
    const int plane = a.plane;
    const int tl = static_cast<int>(threadIdx.x);

    auto wrapz = [&](int p) { return p < 0 ? p + a.nz : (p >= a.nz ? p - a.nz : p); };
    // one buffer descriptor per plane block of 19 direction arrays of words
    const uint32_t dir_bytes = static_cast<uint32_t>(plane) * static_cast<uint32_t>(sizeof(W));
    const uint32_t blk_bytes = static_cast<uint32_t>(kQ) * dir_bytes;
    auto blk = [&](const W* base, int p) {
        return make_rsrc(base + static_cast<size_t>(p) * kQ * static_cast<size_t>(plane), blk_bytes);
    };
    auto issue = [&](int p, const PlaneOffs& q, W e[kQ]) {
        const rsrc_t r3[3] = {blk(A, wrapz(p + 1)), blk(A, p), blk(A, wrapz(p - 1))};  // c_z = -1, 0, +1
#pragma unroll
        for (int i = 0; i < kQ; ++i)
            e[i] = word_load<W>(r3[CZ[i] + 1], q.o[CY[i] + 1][CX[i] + 1], static_cast<uint32_t>(i) * dir_bytes);
    };
    auto moments = [&](uint32_t rbits, const W e[kQ], T& r0, T& r1, T* j) { pair_moments<ST>(a, rbits, e, r0, r1, j); };
    auto densities = [&](uint32_t rbits, const W e[kQ], T& r0, T& r1) {
        moments(rbits, e, r0, r1, static_cast<T*>(nullptr));
    };
    auto rslot = [&](int p) { return (p - zs + 1) & 3; };

    if (tl >= NT) {
        // ---- ring / n_s waves ----
        const int r = tl - NT;
        const int ring_n = 2 * (TXe + 2) + 2 * TYe;
        const bool ring = r < ring_n;
        int rlx, rly;
        {
            const int q = min(r, ring_n - 1);  // threads past the ring repeat its last cell
            if (q < TXe + 2) { rlx = q - 1; rly = -1; }
            else if (q < 2 * (TXe + 2)) { rlx = q - (TXe + 2) - 1; rly = TYe; }
            else if (q < 2 * (TXe + 2) + TYe) { rlx = -1; rly = q - 2 * (TXe + 2); }
            else { rlx = TXe; rly = q - 2 * (TXe + 2) - TYe; }
        }
        const int rx = ((x0 + rlx) % a.nx + a.nx) % a.nx;
        const int ry = ((y0 + rly) % a.ny + a.ny) % a.ny;
        const int rme = (rly + 1) * LW + (rlx + 1);
        const PlaneOffs qring = plane_offs<sizeof(W)>(rx, ry, a.nx, a.ny);
        const uint32_t rxy = reservoir_xy_bits(a, rx, ry);
        // n_s cells of this thread (LDS index, in-plane index); past the list
        // a thread repeats its first cell, the corner (x0 - 1, y0 - 1)
        const int nsw = TXe + 2, nsh = TYe + 2;
        const int ns_off0 = (((y0 - 1) % a.ny + a.ny) % a.ny) * a.nx + ((x0 - 1) % a.nx + a.nx) % a.nx;
        int nl[NSR], no[NSR];
#pragma unroll
        for (int k = 0; k < NSR; ++k) {
            const int c = r + k * NR;
            if (c < nsw * nsh) {
                const int llx = c % nsw - 1, lly = c / nsw - 1;
                const int gx = ((x0 + llx) % a.nx + a.nx) % a.nx;
                const int gy = ((y0 + lly) % a.ny + a.ny) % a.ny;
                nl[k] = (lly + 1) * LW + llx + 1;
                no[k] = gy * a.nx + gx;
            } else {
                nl[k] = 0;
                no[k] = ns_off0;
            }
        }
        W er[kQ];
        float nsv[NSR][CNS];
        auto issue_ring = [&](int p) {
            issue(p, qring, er);
            const float* nsp = ns + static_cast<size_t>(p) * static_cast<size_t>(plane);
#pragma unroll
            for (int k = 0; k < NSR; ++k)
#pragma unroll
                for (int c = 0; c < CNS; ++c) nsv[k][c] = nsp[static_cast<size_t>(c) * a.N + no[k]];
        };
        // consume the loads of plane p into LDS slot `slot`
        auto consume_ring = [&](int p, int slot) {
            T r0, r1;
            densities(rxy | reservoir_z_bits(a, p), er, r0, r1);
            if (ring) {
                s_rho[slot][0][rme] = r0;
                s_rho[slot][1][rme] = r1;
            }
#pragma unroll
            for (int k = 0; k < NSR; ++k)
#pragma unroll
                for (int c = 0; c < CNS; ++c) s_ns[slot][c][nl[k]] = nsv[k][c];
        };
        // ... then issue those of plane pn (unconditionally, so the waits stay
        // exact)
        auto stage_ring = [&](int p, int slot, int pn) {
            consume_ring(p, slot);
            __builtin_amdgcn_sched_barrier(0);
            issue_ring(pn);
        };
        if constexpr (ONE) {
            issue_ring(0);
            consume_ring(0, rslot(0));
            __syncthreads();
            return;
        } else {
            auto next = [&](int p) { return wrapz(p + 1 <= ze ? p + 1 : ze); };
            issue_ring(wrapz(zs - 1));
            stage_ring(wrapz(zs - 1), rslot(zs - 1), zs);
            stage_ring(zs, rslot(zs), next(zs));
            for (int z = zs; z < ze; ++z) {
                stage_ring(wrapz(z + 1), rslot(z + 1), next(z + 1));
                __syncthreads();
            }
            return;
        }
    }

    // ---- cell waves ----
    // lanes take the tile's cells row by row, without gaps; a lane beyond the
    // last cell duplicates it (same cell, same LDS slots, identical values
    // written twice)
    const int cq = min(tl, TXe * TYe - 1);
    const int ly = TXe == 64 ? cq >> 6 : cq / TXe;
    const int x = x0 + (cq - ly * TXe);
    const int y = y0 + ly;
    const int me = (y - y0 + 1) * LW + (x - x0 + 1);
    const PlaneOffs qme = plane_offs<sizeof(W)>(x, y, a.nx, a.ny);
    const uint32_t own = static_cast<uint32_t>(y * a.nx + x) * static_cast<uint32_t>(sizeof(W));
    const uint32_t t_key = fmix32(t ^ kGolden);  // stochastic rounding: time part of the counter
    const uint32_t cxy = reservoir_xy_bits(a, x, y);

    // Collision of plane z from the words wd of the own cell and the LDS slots
    // of planes z-1, z, z+1.
    auto collide = [&](int z, int sm, int s0, int sp, const T (&jm)[6], auto&& wd) {
        const rsrc_t rz = blk(B, z);
        const uint32_t cell =
            static_cast<uint32_t>(z) * static_cast<uint32_t>(plane) + static_cast<uint32_t>(y * a.nx + x);
        pair_collide<ST, CNS, FS, RND>(
            geo, a, cxy | reservoir_z_bits(a, z), t_key, cell, me, &s_rho[sm][0][0], &s_rho[s0][0][0], &s_rho[sp][0][0],
            &s_ns[sm][0][0], &s_ns[s0][0][0], &s_ns[sp][0][0], jm, wd,
            [&](int i, W v) { raw_store<AUX>(v, rz, own, static_cast<uint32_t>(i) * dir_bytes); });
    };

    if constexpr (ONE) {
        // One cell deep: planes z - 1, z and z + 1 are all plane 0, staged
        // once and collided against itself.
        const int slot = rslot(0);
        W r1[kQ];
        issue(0, qme, r1);
        T d0, d1, jm[6];
        moments(cxy | reservoir_z_bits(a, 0), r1, d0, d1, jm);
        s_rho[slot][0][me] = d0;
        s_rho[slot][1][me] = d1;
        __syncthreads();
        collide(0, slot, slot, slot, jm, [&](int i) { return r1[i]; });
        return;
    } else if constexpr (sizeof(W) == 8) {
        // FP32 words: LDS holds one plane of them.  Plane z is collided from
        // registers (hz), plane z+1 waits in LDS (hs), and the loads of plane
        // z+2 are in flight over the barrier and the collision.  The ring
        // waves issue the ring loads of a plane at the same stage as these
        // own loads, while the neighbouring tiles' copies are still in L2.
        W* hsl = &sh.hs[0][0][0] + tl;
        W rc[kQ];
        W hz[kQ];
        T jA[6], jB[6];
        // Stage plane p, whose loads are in rc: densities to LDS, first
        // moments to jm, the words of the plane before from hs to hz and
        // plane p's into hs; then the loads of plane pn are issued.
        auto stage_pipe = [&](int p, int pu, int pn, T (&jm)[6]) {
            T d0, d1;
            moments(cxy | reservoir_z_bits(a, p), rc, d0, d1, jm);
            const int slot = rslot(pu);
            s_rho[slot][0][me] = d0;
            s_rho[slot][1][me] = d1;
#pragma unroll
            for (int i = 0; i < kQ; ++i) {
                hz[i] = hsl[i * NT];
                hsl[i * NT] = rc[i];
            }
            __builtin_amdgcn_sched_barrier(0);
            issue(pn, qme, rc);
        };
        auto wd = [&](int i) { return hz[i]; };
        // the plane whose loads a stage of plane p issues: p + 1, or after the
        // last plane the one just staged again (cache hits)
        auto next = [&](int p) { return wrapz(p + 1 <= ze ? p + 1 : ze); };
        issue(wrapz(zs - 1), qme, rc);
        stage_pipe(wrapz(zs - 1), zs - 1, zs, jB);
        stage_pipe(zs, zs, next(zs), jA);
        // unrolled by two so the moment sets keep fixed names
        for (int z = zs; z < ze; z += 2) {
            stage_pipe(wrapz(z + 1), z + 1, next(z + 1), jB);
            __syncthreads();
            collide(z, rslot(z - 1), rslot(z), rslot(z + 1), jA, wd);
            if (z + 1 >= ze) break;
            stage_pipe(wrapz(z + 2), z + 2, next(z + 2), jA);
            __syncthreads();
            collide(z + 1, rslot(z), rslot(z + 1), rslot(z + 2), jB, wd);
        }
    } else {
        // Three planes at a time: the words of planes z and z+1 wait in LDS
        // (hs, double-buffered), plane z is collided, and the loads of plane
        // z+1+AHEAD are in flight over the barrier and the collision.  No
        // memory access in the sweep is conditional (a skipped access would
        // make the compiler's waits drain the loads kept in flight).
        constexpr int AHEAD = LBM_PAIR_AHEAD;
        constexpr bool DEEP = AHEAD == 2;
        auto hbuf = [&](int p) { return &sh.hs[(p - zs + 2) & 1][0][0] + tl; };
        uint32_t rA[kQ];
        uint32_t rB[DEEP ? kQ : 1];
        // Stage plane p, whose loads are in rc: its densities go to LDS and
        // its words to hs; then the loads of plane pn are issued into rc.
        // the first moments of a staged plane wait in registers for its
        // collision (two sets, for the planes z and z+1)
        T jA[6], jB[6];
        auto stage_pipe = [&](int p, int pu, int pn, uint32_t rc[kQ], T (&jm)[6]) {
            T d0, d1;
            moments(cxy | reservoir_z_bits(a, p), rc, d0, d1, jm);
            const int slot = rslot(pu);
            s_rho[slot][0][me] = d0;
            s_rho[slot][1][me] = d1;
            uint32_t* hw = hbuf(pu);
#pragma unroll
            for (int i = 0; i < kQ; ++i) hw[i * NT] = rc[i];
            __builtin_amdgcn_sched_barrier(0);
            issue(pn, qme, rc);
        };
        auto collide_z = [&](int z, const T (&jm)[6]) {
            const uint32_t* hr = hbuf(z);
            collide(z, rslot(z - 1), rslot(z), rslot(z + 1), jm, [&](int i) { return hr[i * NT]; });
        };
        // the plane whose loads a stage of plane p issues: p + AHEAD, or after
        // the last plane one already staged again (cache hits)
        auto ahead = [&](int p) { return wrapz(p + AHEAD <= ze ? p + AHEAD : ze); };
        uint32_t (&r_odd)[kQ] = rA;
        uint32_t (&r_even)[kQ] = *reinterpret_cast<uint32_t(*)[kQ]>(DEEP ? static_cast<uint32_t*>(rB) : static_cast<uint32_t*>(rA));
        // prologue: planes zs-1 (densities only) and zs
        issue(wrapz(zs - 1), qme, r_odd);
        if constexpr (DEEP) issue(zs, qme, r_even);
        stage_pipe(wrapz(zs - 1), zs - 1, ahead(zs - 1), r_odd, jB);
        stage_pipe(zs, zs, ahead(zs), r_even, jA);
        // unrolled by two so the register sets keep fixed names
        for (int z = zs; z < ze; z += 2) {
            stage_pipe(wrapz(z + 1), z + 1, ahead(z + 1), r_odd, jB);
            __syncthreads();
            collide_z(z, jA);
            if (z + 1 >= ze) break;
            stage_pipe(wrapz(z + 2), z + 2, ahead(z + 2), r_even, jA);
            __syncthreads();
            collide_z(z + 1, jB);
        }
    }
}

template <typename ST, int NC, int FS = kForcingShanChen>
constexpr int kBlockCells = kPair<ST, NC, FS> ? kPairCells : split_cells(sizeof(typename ST::T) == 8, NC);

template <typename ST, int NC, int FS = kForcingShanChen, int CELLS = kBlockCells<ST, NC, FS>>
constexpr int kThreads = kPair<ST, NC, FS> ? CELLS + kPairRing : NC * CELLS;

// CELLS: cells of a block, kBlockCells or, in thin domains, kThinCells.
template <typename ST, int NC, int CNS, int FS, bool ONE, int RND, int AUX, int CELLS>
__global__ __launch_bounds__((kThreads<ST, NC, FS, CELLS>)) void k_step(Args<typename ST::T> a,
                                                                        const typename ST::E* __restrict__ A,
                                                                        typename ST::E* __restrict__ B,
                                                                        const float* __restrict__ ns)
{
    // One block fits a CU, two with one component in FP32 arithmetic (77 KB of
    // LDS) and, but for two n_s fields with the GS-WBS, with the smaller blocks of
    // thin domains: a round of the 256 CUs is 256 or 512 blocks.  Runs per round
    // instead of one run of the whole grid: 181^3 in FP64, 690 blocks, 948 us against
    // 1050.
    constexpr bool TWO = CELLS < kBlockCells<ST, NC, FS> || (NC == 1 && sizeof(typename ST::T) == 4);
    const int L = xcd_tile(blockIdx.x, gridDim.x, TWO ? 512 : 256);
    if constexpr (kPair<ST, NC, FS>) {
        using W = typename PairWordOf<ST>::W;
        __shared__ PairShared<ST, CNS, CELLS> sh;
        step_tile_pair<ST, CNS, FS, ONE, RND, AUX, CELLS>(a, reinterpret_cast<const W*>(A), reinterpret_cast<W*>(B), ns,
                                                          L, a.t, sh);
    } else {
        __shared__ TileShared<ST, NC, CNS, CELLS> sh;
        step_tile<ST, NC, CNS, FS, ONE, AUX, CELLS>(a, A, B, ns, L, a.t, sh);
    }
}

// ---------------------------------------------------------------------------
// Batched step: the tiles of many domains in one launch.  The device table
// holds a header and one entry per domain (geometry, parameters, ping-pong
// buffers, steps to take in this tick, first tile index).  Blocks stride over
// the concatenated tile list, so the grid size does not depend on the mix and
// a captured graph of K launches (k = 0..K-1) stays valid when domains come
// and go: only the table changes.
template <typename T>
struct BatchEntry {
    Args<T> a;
    const void* buf[2];
    const float* ns;
    int parity;      // buffer holding the state at k = 0
    int steps;       // launches k < steps advance this domain
    int tile_begin;  // first tile of this domain in the concatenated list
    int ntiles;
};

struct BatchHeader {
    int ndom;
    int total_tiles;
    int pad[2];
};

constexpr size_t kBatchEntryOffset = 64;

template <typename ST, int NC, int CNS, int AUX>
__global__ __launch_bounds__((kThreads<ST, NC>)) void k_step_batch(const char* __restrict__ table, int k)
{
    using T = typename ST::T;
    using E = typename ST::E;
    const BatchHeader* hdr = reinterpret_cast<const BatchHeader*>(table);
    const BatchEntry<T>* ent = reinterpret_cast<const BatchEntry<T>*>(table + kBatchEntryOffset);
    const int total = hdr->total_tiles;
    const int nd = hdr->ndom;
    // XCD-aware order, as in k_step: blocks are dispatched round-robin over
    // the 8 XCDs, so give each XCD a contiguous run of every stride of tiles
    // (neighbouring tiles re-read each other's edge cells through its L2)
    const int nb = gridDim.x;
    const int b0 = (nb & 7) == 0 ? (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    using Shared = std::conditional_t<kPair<ST, NC>, PairShared<ST, CNS>, TileShared<ST, NC, CNS>>;
    __shared__ Shared sh;
    for (int w = b0; w < total; w += nb) {
        int lo = 0, hi = nd - 1;  // last domain with tile_begin <= w
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (ent[mid].tile_begin <= w) lo = mid;
            else hi = mid - 1;
        }
        const BatchEntry<T>& e = ent[lo];
        if (k >= e.steps) continue;
        const int cur = (e.parity + k) & 1;
        __syncthreads();  // the previous tile's LDS is no longer read
        if constexpr (kPair<ST, NC>) {
            // the rounding of each domain picks a tile sweep compiled for it
            // (FP32 rounds to nearest only)
            using W = typename PairWordOf<ST>::W;
            const W* src = static_cast<const W*>(e.buf[cur]);
            W* dst = static_cast<W*>(const_cast<void*>(e.buf[1 - cur]));
            const uint32_t tk = e.a.t + static_cast<uint32_t>(k);
            if (sizeof(E) == 2 && e.a.sr)
                step_tile_pair<ST, CNS, kForcingShanChen, false, sizeof(E) == 2 ? kRoundStochastic : kRoundNearest,
                               AUX, kPairCells>(e.a, src, dst, e.ns, w - e.tile_begin, tk, sh);
            else
                step_tile_pair<ST, CNS, kForcingShanChen, false, kRoundNearest, AUX, kPairCells>(
                    e.a, src, dst, e.ns, w - e.tile_begin, tk, sh);
        } else
            step_tile<ST, NC, CNS, kForcingShanChen, false, AUX, kBlockCells<ST, NC>>(
                e.a, static_cast<const E*>(e.buf[cur]), static_cast<E*>(const_cast<void*>(e.buf[1 - cur])), e.ns,
                w - e.tile_begin, e.a.t + static_cast<uint32_t>(k), sh);
    }
}

// ---------------------------------------------------------------------------
// Auxiliary kernels (initialisation, checkpoints, FP64 diagnostics).  They run
// once per call, not per step: plain grid-stride loops over the cells.

#define CELL_LOOP(n, N)                                                                                      \
    for (int64_t n = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; n < (N);                  \
         n += static_cast<int64_t>(gridDim.x) * blockDim.x)

struct Cell {
    int x, y, z, ip;  // coordinates and in-plane index
};

template <typename T>
__device__ __forceinline__ Cell cell_of(const Args<T>& a, int64_t n)
{
    Cell c;
    c.z = static_cast<int>(n / a.plane);
    c.ip = static_cast<int>(n - static_cast<int64_t>(c.z) * a.plane);
    c.x = c.ip % a.nx;
    c.y = c.ip / a.nx;
    return c;
}

template <typename T>
__device__ __forceinline__ int64_t cell_at(const Args<T>& a, int x, int y, int z)
{
    return static_cast<int64_t>(z) * a.plane + y * a.nx + x;
}

// direction i as (cx, cy, cz, w_i) for a runtime i
template <typename T>
__device__ __forceinline__ void dir_of(int i, int& dx, int& dy, int& dz, T& w)
{
    dx = dy = dz = 0;
    w = T(0);
#pragma unroll
    for (int k = 0; k < kQ; ++k)
        if (k == i) {
            dx = CX[k];
            dy = CY[k];
            dz = CZ[k];
            w = wgt<T>(k);
        }
}

template <typename ST>
__global__ void k_init(Args<typename ST::T> a, int ncomp, const double* __restrict__ rho_init,
                       typename ST::E* __restrict__ A)
{
    using T = typename ST::T;
    CELL_LOOP(n, a.N)
    {
        const Cell c = cell_of(a, n);
        // A_i(y) must hold f_i(y + c_i, 0) (pull storage)
        for (int s = 0; s < ncomp; ++s) {
#pragma unroll
            for (int i = 0; i < kQ; ++i) {
                const int xd = (c.x + CX[i] + a.nx) % a.nx, yd = (c.y + CY[i] + a.ny) % a.ny,
                          zd = (c.z + CZ[i] + a.nz) % a.nz;
                const int res = reservoir_of(a, xd, yd, zd);
                const double rho = res >= 0 ? static_cast<double>(a.res_dr[res][s]) + static_cast<double>(a.rho0[s])
                                            : rho_init[static_cast<size_t>(s) * a.N + cell_at(a, xd, yd, zd)];
                const double h = wgt<double>(i) * (rho - static_cast<double>(a.rho0[s]));
                A[pidx(a, s, i, c.z, c.ip)] = ST::enc(static_cast<T>(h), a.scale);
            }
        }
    }
}

template <typename ST>
__global__ void k_canonical(Args<typename ST::T> a, const typename ST::E* __restrict__ A, int s, int i,
                            double* __restrict__ out)
{
    int dx, dy, dz;
    double w;
    dir_of(i, dx, dy, dz, w);
    CELL_LOOP(n, a.N)
    {
        const Cell c = cell_of(a, n);
        const int res = reservoir_of(a, c.x, c.y, c.z);
        double v;
        if (res >= 0) {
            v = w * (static_cast<double>(a.res_dr[res][s]) + static_cast<double>(a.rho0[s]));
        } else {
            const int xs = (c.x - dx + a.nx) % a.nx, ys = (c.y - dy + a.ny) % a.ny, zs = (c.z - dz + a.nz) % a.nz;
            v = static_cast<double>(ST::dec(A[pidx(a, s, i, zs, ys * a.nx + xs)], a.inv_scale)) +
                w * static_cast<double>(a.rho0[s]);
        }
        out[n] = v;
    }
}

template <typename ST>
__global__ void k_set_canonical(Args<typename ST::T> a, const double* __restrict__ in, int s, int i,
                                typename ST::E* __restrict__ A)
{
    using T = typename ST::T;
    int dx, dy, dz;
    double w;
    dir_of(i, dx, dy, dz, w);
    CELL_LOOP(n, a.N)
    {
        const Cell c = cell_of(a, n);
        // A_i(y) = f_i(y + c_i)
        const int xd = (c.x + dx + a.nx) % a.nx, yd = (c.y + dy + a.ny) % a.ny, zd = (c.z + dz + a.nz) % a.nz;
        const double h = in[cell_at(a, xd, yd, zd)] - w * static_cast<double>(a.rho0[s]);
        A[pidx(a, s, i, c.z, c.ip)] = ST::enc(static_cast<T>(h), a.scale);
    }
}

constexpr int kRedThreads = 256;

// Sum of v over the block, the same on every run: a butterfly over each
// wave's 64 lanes (cross-lane moves, no LDS round trips or barriers), then
// the waves' sums in wave order; thread k < K writes out[k].
template <int K>
__device__ __forceinline__ void block_sum(double (&v)[K], double* __restrict__ out)
{
    __shared__ double ws[kRedThreads / 64][K];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
    const int wv = static_cast<int>(threadIdx.x) >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) ws[wv][k] = v[k];
    __syncthreads();
    if (threadIdx.x < K) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kRedThreads / 64; ++w) s += ws[w][threadIdx.x];
        out[threadIdx.x] = s;
    }
}

// Diagnostics, first pass (the only one that reads the populations): per cell
// the FP64 densities rho_s (Eq. rho_BGK) and first moments j_s (Eq. mom_BGK) of
// the pre-collision state; writes rho [ncomp][N] and, when m_out is given, the
// local part of rho u_macro of Eq. (HMCSC_u_macro), sum_s (1 - n_s)(j_s +
// F_ext,s / 2) with F_ext,s of Eq. (SC_F_ext), into m_out [3][N].  Block
// totals {M_0, M_1, sum of that local part} go to partials[block][5].
template <typename ST>
__global__ __launch_bounds__(kRedThreads) void k_dens(Args<typename ST::T> a, int ncomp, int c_ns,
                                                      const typename ST::E* __restrict__ A,
                                                      const float* __restrict__ ns, double* __restrict__ rho,
                                                      double* __restrict__ m_out, double* __restrict__ partials)
{
    double acc[5] = {0, 0, 0, 0, 0};
    CELL_LOOP(n, a.N)
    {
        const Cell c = cell_of(a, n);
        const int res = reservoir_of(a, c.x, c.y, c.z);
        const int xs[3] = {wrap_inc(c.x, a.nx), c.x, wrap_dec(c.x, a.nx)};  // x - c, c = -1, 0, 1
        const int ys[3] = {wrap_inc(c.y, a.ny), c.y, wrap_dec(c.y, a.ny)};
        const int zs[3] = {wrap_inc(c.z, a.nz), c.z, wrap_dec(c.z, a.nz)};
        double rs[2] = {0, 0}, j[2][3] = {{0, 0, 0}, {0, 0, 0}}, rtot = 0;
        for (int s = 0; s < ncomp; ++s) {
            double d = 0;
            if (res >= 0) {
                d = static_cast<double>(a.res_dr[res][s]);
            } else {
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    const double h = static_cast<double>(
                        ST::dec(A[pidx(a, s, i, zs[CZ[i] + 1], ys[CY[i] + 1] * a.nx + xs[CX[i] + 1])], a.inv_scale));
                    d += h;
                    j[s][0] += CX[i] * h;
                    j[s][1] += CY[i] * h;
                    j[s][2] += CZ[i] * h;
                }
            }
            rs[s] = static_cast<double>(a.rho0[s]) + d;
            rho[static_cast<size_t>(s) * a.N + n] = rs[s];
            rtot += rs[s];
        }
        double m[3] = {0, 0, 0};
        for (int s = 0; s < ncomp; ++s) {
            const double wfl = 1.0 - static_cast<double>(ns[static_cast<size_t>(c_ns == 2 ? s : 0) * a.N + n]);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double fext = rtot > 0 ? rs[s] / rtot * static_cast<double>(a.F[d]) : 0.0;
                m[d] += wfl * (j[s][d] + fext / 2.0);
            }
        }
        if (m_out)
#pragma unroll
            for (int d = 0; d < 3; ++d) m_out[static_cast<size_t>(d) * a.N + n] = m[d];
        acc[0] += rs[0];
        acc[1] += rs[1];
#pragma unroll
        for (int d = 0; d < 3; ++d) acc[2 + d] += m[d];
    }
    block_sum<5>(acc, partials + static_cast<size_t>(blockIdx.x) * 5);
}

// Diagnostics, second pass (densities and n_s only): the half cohesion and
// adhesion forces of Eqs. (SC_F_inter), (SC_F_ads) weighted by (1 - n_s), the
// rest of rho u_macro.  When u is given it holds the first pass's local part
// and receives u_macro of Eq. (HMCSC_u_macro); p receives Eq. (SC_pressure).
// Block totals {0, 0, sum of the force part} go to partials[block][5].
template <typename T>
__global__ __launch_bounds__(kRedThreads) void k_force(Args<T> a, int ncomp, int c_ns, double G_s, double Gads0,
                                                       double Gads1, double gG_p, const float* __restrict__ ns,
                                                       const double* __restrict__ rho, double* __restrict__ u,
                                                       double* __restrict__ p_out, double* __restrict__ partials)
{
    double acc[5] = {0, 0, 0, 0, 0};
    const double Gads[2] = {Gads0, Gads1};
    CELL_LOOP(n, a.N)
    {
        const Cell c = cell_of(a, n);
        // neighbours x + c_i (note: opposite of the pull)
        const int cols[3] = {wrap_dec(c.x, a.nx), c.x, wrap_inc(c.x, a.nx)};
        const int rows[3] = {wrap_dec(c.y, a.ny), c.y, wrap_inc(c.y, a.ny)};
        const int plns[3] = {wrap_dec(c.z, a.nz), c.z, wrap_inc(c.z, a.nz)};
        double rs[2] = {0, 0}, rtot = 0;
        for (int s = 0; s < ncomp; ++s) {
            rs[s] = rho[static_cast<size_t>(s) * a.N + n];
            rtot += rs[s];
        }
        double m[3] = {0, 0, 0};
        for (int s = 0; s < ncomp; ++s) {
            double gi[3] = {0, 0, 0}, ga[3] = {0, 0, 0};
            const size_t cn = static_cast<size_t>(c_ns == 2 ? s : 0);
#pragma unroll
            for (int i = 1; i < kQ; ++i) {
                const int64_t nb = cell_at(a, cols[CX[i] + 1], rows[CY[i] + 1], plns[CZ[i] + 1]);
                const double wi = wgt<double>(i);
                if (ncomp == 2) {
                    const double r = rho[static_cast<size_t>(1 - s) * a.N + nb];
                    gi[0] += wi * r * CX[i]; gi[1] += wi * r * CY[i]; gi[2] += wi * r * CZ[i];
                }
                const double v = static_cast<double>(ns[cn * a.N + nb]);
                ga[0] += wi * v * CX[i]; ga[1] += wi * v * CY[i]; ga[2] += wi * v * CZ[i];
            }
            const double wfl = 1.0 - static_cast<double>(ns[cn * a.N + n]);
#pragma unroll
            for (int d = 0; d < 3; ++d) m[d] += wfl * ((-rs[s] * G_s * gi[d] - rs[s] * Gads[s] * ga[d]) / 2.0);
        }
        if (u)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double& ud = u[static_cast<size_t>(d) * a.N + n];
                ud = rtot > 0 ? (ud + m[d]) / rtot : 0.0;
            }
        if (p_out) p_out[n] = (rtot + (ncomp == 2 ? gG_p * rs[0] * rs[1] : 0.0)) / 3.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) acc[2 + d] += m[d];
    }
    block_sum<5>(acc, partials + static_cast<size_t>(blockIdx.x) * 5);
}

// FP64 density of component s at cell (x, y, z) of the pre-collision state:
// the pulled populations summed in direction order, or the reservoir's
// prescribed density.
template <typename ST>
__device__ __forceinline__ double density_at(const Args<typename ST::T>& a, const typename ST::E* __restrict__ A,
                                             int s, int x, int y, int z)
{
    const int res = reservoir_of(a, x, y, z);
    double d = 0;
    if (res >= 0) {
        d = static_cast<double>(a.res_dr[res][s]);
    } else {
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const int xs = (x - CX[i] + a.nx) % a.nx, ys = (y - CY[i] + a.ny) % a.ny, zs = (z - CZ[i] + a.nz) % a.nz;
            d += static_cast<double>(ST::dec(A[pidx(a, s, i, zs, ys * a.nx + xs)], a.inv_scale));
        }
    }
    return static_cast<double>(a.rho0[s]) + d;
}

// The FP64 totals of k_dens and k_force in one pass with no per-cell field:
// each cell recomputes the densities of its 18 neighbours from their pulled
// populations (19 times the reads of one pass, cache hits for the most part).
// Block totals {M_0, M_1, J_x, J_y, J_z} go to partials[block][5].
template <typename ST>
__global__ __launch_bounds__(kRedThreads) void k_totals_one_pass(Args<typename ST::T> a, int ncomp, int c_ns,
                                                                 double G_s, double Gads0, double Gads1,
                                                                 const typename ST::E* __restrict__ A,
                                                                 const float* __restrict__ ns,
                                                                 double* __restrict__ partials)
{
    double acc[5] = {0, 0, 0, 0, 0};
    const double Gads[2] = {Gads0, Gads1};
    CELL_LOOP(n, a.N)
    {
        const Cell c = cell_of(a, n);
        const int res = reservoir_of(a, c.x, c.y, c.z);
        const int xs[3] = {wrap_inc(c.x, a.nx), c.x, wrap_dec(c.x, a.nx)};  // x - c, c = -1, 0, 1
        const int ys[3] = {wrap_inc(c.y, a.ny), c.y, wrap_dec(c.y, a.ny)};
        const int zs[3] = {wrap_inc(c.z, a.nz), c.z, wrap_dec(c.z, a.nz)};
        double rs[2] = {0, 0}, j[2][3] = {{0, 0, 0}, {0, 0, 0}}, rtot = 0;
        for (int s = 0; s < ncomp; ++s) {
            if (res < 0) {
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    const double h = static_cast<double>(
                        ST::dec(A[pidx(a, s, i, zs[CZ[i] + 1], ys[CY[i] + 1] * a.nx + xs[CX[i] + 1])], a.inv_scale));
                    j[s][0] += CX[i] * h;
                    j[s][1] += CY[i] * h;
                    j[s][2] += CZ[i] * h;
                }
            }
            rs[s] = density_at<ST>(a, A, s, c.x, c.y, c.z);
            rtot += rs[s];
        }
        double m[3] = {0, 0, 0};
        for (int s = 0; s < ncomp; ++s) {
            double gi[3] = {0, 0, 0}, ga[3] = {0, 0, 0};
            const size_t cn = static_cast<size_t>(c_ns == 2 ? s : 0);
#pragma unroll
            for (int i = 1; i < kQ; ++i) {
                // neighbour x + c_i
                const int nx_ = (c.x + CX[i] + a.nx) % a.nx, ny_ = (c.y + CY[i] + a.ny) % a.ny,
                          nz_ = (c.z + CZ[i] + a.nz) % a.nz;
                const double wi = wgt<double>(i);
                if (ncomp == 2) {
                    const double r = density_at<ST>(a, A, 1 - s, nx_, ny_, nz_);
                    gi[0] += wi * r * CX[i]; gi[1] += wi * r * CY[i]; gi[2] += wi * r * CZ[i];
                }
                const double v = static_cast<double>(ns[cn * a.N + cell_at(a, nx_, ny_, nz_)]);
                ga[0] += wi * v * CX[i]; ga[1] += wi * v * CY[i]; ga[2] += wi * v * CZ[i];
            }
            const double wfl = 1.0 - static_cast<double>(ns[cn * a.N + n]);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double fext = rtot > 0 ? rs[s] / rtot * static_cast<double>(a.F[d]) : 0.0;
                const double ft = -rs[s] * G_s * gi[d] - rs[s] * Gads[s] * ga[d] + fext;
                m[d] += wfl * (j[s][d] + ft / 2.0);
            }
        }
        acc[0] += rs[0];
        acc[1] += rs[1];
#pragma unroll
        for (int d = 0; d < 3; ++d) acc[2 + d] += m[d];
    }
    block_sum<5>(acc, partials + static_cast<size_t>(blockIdx.x) * 5);
}

// Electrolyte-filling diagnostics (Sec. 4) from the FP64 fields: per-block
// sums of p and cell counts over the inlet and outlet slabs (Eq. CapPressure),
// and of (1 - n_s) [rho_comp >= threshold] and (1 - n_s) over the pore slab
// (Eq. Saturation).
__global__ __launch_bounds__(kRedThreads) void k_fill(int nx, int ny, int nz, int64_t N, FillQuery q, int ns_field,
                                                      const double* __restrict__ rho, const double* __restrict__ p,
                                                      const float* __restrict__ ns, double* __restrict__ partials)
{
    double acc[6] = {0, 0, 0, 0, 0, 0};
    const int64_t plane = static_cast<int64_t>(nx) * ny;
    CELL_LOOP(n, N)
    {
        const int z = static_cast<int>(n / plane);
        const int ip = static_cast<int>(n - z * plane);
        const int x = ip % nx, y = ip / nx;
        const int c = q.axis == 0 ? x : (q.axis == 1 ? y : z);
        if (c >= q.inlet_lo && c < q.inlet_hi) {
            acc[0] += p[n];
            acc[1] += 1.0;
        }
        if (c >= q.outlet_lo && c < q.outlet_hi) {
            acc[2] += p[n];
            acc[3] += 1.0;
        }
        if (c >= q.pore_lo && c < q.pore_hi) {
            const double wfl = 1.0 - static_cast<double>(ns[static_cast<size_t>(ns_field) * N + n]);
            acc[4] += rho[static_cast<size_t>(q.comp) * N + n] >= q.threshold ? wfl : 0.0;
            acc[5] += wfl;
        }
    }
    (void)nz;
    block_sum<6>(acc, partials + static_cast<size_t>(blockIdx.x) * 6);
}

// Permeability (Eq. Permeability) from the FP64 fields: per-block sums of
// rho_s u_macro[axis] for each component (the component's share of the
// mixture momentum, used for relative permeabilities) and of rho u_macro[axis].
__global__ __launch_bounds__(kRedThreads) void k_flux(int64_t N, int ncomp, int axis, const double* __restrict__ rho,
                                                      const double* __restrict__ u, double* __restrict__ partials)
{
    double acc[3] = {0, 0, 0};
    CELL_LOOP(n, N)
    {
        const double ua = u[static_cast<size_t>(axis) * N + n];
        const double r0 = rho[n];
        const double r1 = ncomp == 2 ? rho[static_cast<size_t>(N) + n] : 0.0;
        acc[0] += r0 * ua;
        acc[1] += r1 * ua;
        acc[2] += (r0 + r1) * ua;
    }
    block_sum<3>(acc, partials + static_cast<size_t>(blockIdx.x) * 3);
}

// Static-droplet measurement (Sec. 3.3) from an FP64 field f: per-block sums
// of f and cell counts over the ball |x - c| <= sqrt(r_in2) and over the
// cells with |x - c| >= sqrt(r_out2), distances taken to the nearest periodic
// image of the centre c (2-D when nz = 1).
__global__ __launch_bounds__(kRedThreads) void k_ball(int nx, int ny, int nz, int64_t N, double cx, double cy,
                                                      double cz, double r_in2, double r_out2,
                                                      const double* __restrict__ f, double* __restrict__ partials)
{
    double acc[4] = {0, 0, 0, 0};
    const int64_t plane = static_cast<int64_t>(nx) * ny;
    CELL_LOOP(n, N)
    {
        const int z = static_cast<int>(n / plane);
        const int ip = static_cast<int>(n - z * plane);
        const int x = ip % nx, y = ip / nx;
        double dx = x - cx, dy = y - cy, dz = z - cz;
        dx -= nx * rint(dx / nx);
        dy -= ny * rint(dy / ny);
        dz -= nz * rint(dz / nz);
        const double d2 = dx * dx + dy * dy + dz * dz;
        if (d2 <= r_in2) {
            acc[0] += f[n];
            acc[1] += 1.0;
        }
        if (d2 >= r_out2) {
            acc[2] += f[n];
            acc[3] += 1.0;
        }
    }
    block_sum<4>(acc, partials + static_cast<size_t>(blockIdx.x) * 4);
}

// Fixed-order sum of nblocks partials of K doubles each (one block): the
// result does not depend on timing.
template <int K>
__global__ __launch_bounds__(kRedThreads) void k_reduce(const double* __restrict__ partials, int nblocks,
                                                        double* __restrict__ out)
{
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kRedThreads)
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += partials[static_cast<size_t>(b) * K + k];
    block_sum<K>(acc, out);
}

// ---------------------------------------------------------------------------
// Launchers.

bool pair_layout(int storage, int ncomp, int forcing)
{
    return ((storage == kF32 && forcing != kForcingGuo) || storage == kF16 || storage == kBF16) && ncomp == 2;
}

void tile_limits(const Problem& p, int* cells, int* rows)
{
    const bool pair = pair_layout(p.storage, p.ncomp, p.forcing);
    *cells = pair ? kPairCells : split_cells(p.storage == kF64, p.ncomp);
    *rows = pair ? kPairH : split_rows(p.storage == kF64, p.ncomp, p.c_ns);
}

bool tile_supported(const Problem& p, int tx, int ty)
{
    int cells, rows;
    tile_limits(p, &cells, &rows);
    return tx >= 1 && ty >= 1 && tx <= 64 && ty <= rows && tx * ty <= cells;
}

int block_cells(const Problem& p, int tx, int ty)
{
    int cells, rows;
    tile_limits(p, &cells, &rows);
    return p.ny <= kThinRows && ty <= kThinRows && tx * ty <= kThinCells ? std::min(cells, kThinCells) : cells;
}

int storage_bytes(int storage)
{
    switch (storage) {
    case kF64: return 8;
    case kF32: return 4;
    case kF16: return 2;
    case kBF16: return 2;
    default: return 0;
    }
}

template <typename ST, int NC, int CNS, int FS, bool ONE>
static hipError_t step_t(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                         hipStream_t st)
{
    using T = typename ST::T;
    using E = typename ST::E;
    Args<T> a = make_args<T>(p);
    a.zchunk = l.zchunk;
    a.tw = l.tile_x;
    a.th = l.tile_y;
    a.ntx = (p.nx + l.tile_x - 1) / l.tile_x;
    a.nty = (p.ny + l.tile_y - 1) / l.tile_y;
    a.nzc = (p.nz + l.zchunk - 1) / l.zchunk;
    a.t = static_cast<uint32_t>(t);
    const int nblocks = a.ntx * a.nty * a.nzc;
    // one instance per block size and store policy (two components in FP64 and one
    // plane keep non-temporal stores), and of the pair kernel per rounding mode;
    // the split kernels branch on it (their two store sequences are alike)
    constexpr int CELLS = kBlockCells<ST, NC, FS>;
    auto go = [&](auto rnd, auto aux, auto cells) {
        constexpr int NB = decltype(cells)::value;
        hipLaunchKernelGGL((k_step<ST, NC, CNS, FS, ONE, decltype(rnd)::value, decltype(aux)::value, NB>),
                           dim3(nblocks), dim3(kThreads<ST, NC, FS, NB>), 0, st, a, static_cast<const E*>(A),
                           static_cast<E*>(B), ns);
    };
    using Nt = std::integral_constant<int, kNT>;
    using Cached = std::integral_constant<int, ONE || (sizeof(E) == 8 && NC == 2) ? kNT : 0>;
    using Full = std::integral_constant<int, CELLS>;
    using Thin = std::integral_constant<int, std::min(CELLS, kThinCells)>;
    auto block = [&](auto rnd, auto aux) { l.cells < CELLS ? go(rnd, aux, Thin{}) : go(rnd, aux, Full{}); };
    auto policy = [&](auto rnd) { l.nt_stores ? block(rnd, Nt{}) : block(rnd, Cached{}); };
    if constexpr (kPair<ST, NC, FS>) {
        // FP32 rounds to nearest
        if (sizeof(E) == 2 && p.stochastic)
            policy(std::integral_constant<int, sizeof(E) == 2 ? kRoundStochastic : kRoundNearest>{});
        else policy(std::integral_constant<int, kRoundNearest>{});
    } else {
        policy(std::integral_constant<int, kRoundEither>{});
    }
    return hipGetLastError();
}

template <typename ST, int NC, int CNS>
static hipError_t step_fs(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                          hipStream_t st)
{
    constexpr int SC = kForcingShanChen, GUO = kForcingGuo;
    if (!tile_supported(p, l.tile_x, l.tile_y) || l.cells != block_cells(p, l.tile_x, l.tile_y))
        return hipErrorInvalidValue;
    const bool one = p.nz == 1;
    if (p.forcing == GUO)
        return one ? step_t<ST, NC, CNS, GUO, true>(p, l, t, A, B, ns, st)
                   : step_t<ST, NC, CNS, GUO, false>(p, l, t, A, B, ns, st);
    return one ? step_t<ST, NC, CNS, SC, true>(p, l, t, A, B, ns, st)
               : step_t<ST, NC, CNS, SC, false>(p, l, t, A, B, ns, st);
}

template <typename ST>
static hipError_t step_st(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                          hipStream_t st)
{
    if (p.ncomp == 1) return step_fs<ST, 1, 1>(p, l, t, A, B, ns, st);
    if (p.c_ns == 1) return step_fs<ST, 2, 1>(p, l, t, A, B, ns, st);
    return step_fs<ST, 2, 2>(p, l, t, A, B, ns, st);
}

hipError_t launch_step(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                       hipStream_t st)
{
    if (l.bx > 0) return launch_step_box(p, l, t, A, B, ns, st);
    switch (p.storage) {
    case kF64: return step_st<F64>(p, l, t, A, B, ns, st);
    case kF32: return step_st<F32>(p, l, t, A, B, ns, st);
    case kF16: return step_st<F16>(p, l, t, A, B, ns, st);
    case kBF16: return step_st<BF16>(p, l, t, A, B, ns, st);
    default: return hipErrorInvalidValue;
    }
}

// Grid of a cell loop: enough blocks to fill the device a few times over.
static unsigned cell_blocks(int64_t N)
{
    return static_cast<unsigned>(std::min<int64_t>((N + 255) / 256, int64_t(1) << 20));
}

template <typename F>
static hipError_t by_storage(int storage, F&& f)
{
    switch (storage) {
    case kF64: return f(F64{});
    case kF32: return f(F32{});
    case kF16: return f(F16{});
    case kBF16: return f(BF16{});
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_init(const Problem& p, const double* rho_init, void* A, hipStream_t st)
{
    return by_storage(p.storage, [&](auto tag) {
        using ST = decltype(tag);
        Args<typename ST::T> a = make_args<typename ST::T>(p);
        hipLaunchKernelGGL((k_init<ST>), dim3(cell_blocks(p.N)), dim3(256), 0, st, a, p.ncomp, rho_init,
                           static_cast<typename ST::E*>(A));
        return hipGetLastError();
    });
}

hipError_t launch_canonical(const Problem& p, const void* A, int s, int i, double* out, hipStream_t st)
{
    return by_storage(p.storage, [&](auto tag) {
        using ST = decltype(tag);
        Args<typename ST::T> a = make_args<typename ST::T>(p);
        hipLaunchKernelGGL((k_canonical<ST>), dim3(cell_blocks(p.N)), dim3(256), 0, st, a,
                           static_cast<const typename ST::E*>(A), s, i, out);
        return hipGetLastError();
    });
}

hipError_t launch_set_canonical(const Problem& p, const double* in, int s, int i, void* A, hipStream_t st)
{
    return by_storage(p.storage, [&](auto tag) {
        using ST = decltype(tag);
        Args<typename ST::T> a = make_args<typename ST::T>(p);
        hipLaunchKernelGGL((k_set_canonical<ST>), dim3(cell_blocks(p.N)), dim3(256), 0, st, a, in, s, i,
                           static_cast<typename ST::E*>(A));
        return hipGetLastError();
    });
}

int moments_max_blocks() { return 1024; }

static int diag_blocks(int64_t N)
{
    return static_cast<int>(std::min<int64_t>(moments_max_blocks(), (N + kRedThreads - 1) / kRedThreads));
}

hipError_t launch_diagnostics(const Problem& p, const void* A, const float* ns, bool forces, double* rho, double* u,
                              double* pr, double* partials, double* out, hipStream_t st)
{
    const int nb = diag_blocks(p.N);
    hipError_t e = by_storage(p.storage, [&](auto tag) {
        using ST = decltype(tag);
        Args<typename ST::T> a = make_args<typename ST::T>(p);
        hipLaunchKernelGGL((k_dens<ST>), dim3(nb), dim3(kRedThreads), 0, st, a, p.ncomp, p.c_ns,
                           static_cast<const typename ST::E*>(A), ns, rho, u, partials);
        if (forces)
            hipLaunchKernelGGL((k_force<typename ST::T>), dim3(nb), dim3(kRedThreads), 0, st, a, p.ncomp, p.c_ns, p.G_s,
                               p.Gads_s[0], p.Gads_s[1], p.g_scale * p.G_inter, ns, rho, u, pr,
                               partials + static_cast<size_t>(nb) * 5);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce<5>, dim3(1), dim3(kRedThreads), 0, st, partials, forces ? 2 * nb : nb, out);
    return hipGetLastError();
}

hipError_t launch_totals_one_pass(const Problem& p, const void* A, const float* ns, double* partials, int max_blocks,
                                  double* out, hipStream_t st)
{
    const int nb = static_cast<int>(std::min<int64_t>(max_blocks, (p.N + kRedThreads - 1) / kRedThreads));
    hipError_t e = by_storage(p.storage, [&](auto tag) {
        using ST = decltype(tag);
        Args<typename ST::T> a = make_args<typename ST::T>(p);
        hipLaunchKernelGGL((k_totals_one_pass<ST>), dim3(nb), dim3(kRedThreads), 0, st, a, p.ncomp, p.c_ns, p.G_s,
                           p.Gads_s[0], p.Gads_s[1], static_cast<const typename ST::E*>(A), ns, partials);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce<5>, dim3(1), dim3(kRedThreads), 0, st, partials, nb, out);
    return hipGetLastError();
}

hipError_t launch_fill(const Problem& p, const FillQuery& q, const double* rho, const double* pr, const float* ns,
                       double* partials, double* out, hipStream_t st)
{
    const int nb = diag_blocks(p.N);
    const int ns_field = p.c_ns == 2 ? q.comp : 0;
    hipLaunchKernelGGL(k_fill, dim3(nb), dim3(kRedThreads), 0, st, p.nx, p.ny, p.nz, p.N, q, ns_field, rho, pr, ns,
                       partials);
    hipLaunchKernelGGL(k_reduce<6>, dim3(1), dim3(kRedThreads), 0, st, partials, nb, out);
    return hipGetLastError();
}

hipError_t launch_ball(const Problem& p, const double c[3], double r_in, double r_out, const double* f,
                       double* partials, double* out, hipStream_t st)
{
    const int nb = diag_blocks(p.N);
    hipLaunchKernelGGL(k_ball, dim3(nb), dim3(kRedThreads), 0, st, p.nx, p.ny, p.nz, p.N, c[0], c[1], c[2],
                       r_in * r_in, r_out * r_out, f, partials);
    hipLaunchKernelGGL(k_reduce<4>, dim3(1), dim3(kRedThreads), 0, st, partials, nb, out);
    return hipGetLastError();
}

hipError_t launch_flux(const Problem& p, int axis, const double* rho, const double* u, double* partials, double* out,
                       hipStream_t st)
{
    const int nb = diag_blocks(p.N);
    hipLaunchKernelGGL(k_flux, dim3(nb), dim3(kRedThreads), 0, st, p.N, p.ncomp, axis, rho, u, partials);
    hipLaunchKernelGGL(k_reduce<3>, dim3(1), dim3(kRedThreads), 0, st, partials, nb, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Convergence monitor of the server: for every domain of a table, the FP64
// sums over its cells of the local part of rho u_macro (Eq. HMCSC_u_macro
// without the neighbour forces), sum_s (1 - n_s)(j_s + F_ext,s / 2), and of
// the mass.  One launch covers all domains (each owns a run of blocks); a
// second launch reduces each domain's blocks in a fixed order.
template <typename T>
struct MonitorEntry {
    Args<T> a;
    const void* state;
    const float* ns;
    int ncomp, c_ns;
    int block_begin, nblocks;
};

struct MonitorHeader {
    int ndom;
    int total_blocks;
    int pad[2];
};

template <typename ST>
__global__ __launch_bounds__(kRedThreads) void k_monitor(const char* __restrict__ table, double* __restrict__ partials)
{
    using T = typename ST::T;
    const MonitorHeader* hdr = reinterpret_cast<const MonitorHeader*>(table);
    const MonitorEntry<T>* ent = reinterpret_cast<const MonitorEntry<T>*>(table + kBatchEntryOffset);
    const int b = blockIdx.x;
    int lo = 0, hi = hdr->ndom - 1;  // last domain with block_begin <= b
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ent[mid].block_begin <= b) lo = mid;
        else hi = mid - 1;
    }
    const MonitorEntry<T>& e = ent[lo];
    const Args<T>& a = e.a;
    const typename ST::E* A = static_cast<const typename ST::E*>(e.state);
    double acc[4] = {0, 0, 0, 0};
    const int64_t stride = static_cast<int64_t>(e.nblocks) * blockDim.x;
    for (int64_t n = static_cast<int64_t>(b - e.block_begin) * blockDim.x + threadIdx.x; n < a.N; n += stride) {
        const Cell c = cell_of(a, n);
        const int res = reservoir_of(a, c.x, c.y, c.z);
        const int xs[3] = {wrap_inc(c.x, a.nx), c.x, wrap_dec(c.x, a.nx)};
        const int ys[3] = {wrap_inc(c.y, a.ny), c.y, wrap_dec(c.y, a.ny)};
        const int zs[3] = {wrap_inc(c.z, a.nz), c.z, wrap_dec(c.z, a.nz)};
        double rs[2] = {0, 0}, j[2][3] = {{0, 0, 0}, {0, 0, 0}}, rtot = 0;
        for (int s = 0; s < e.ncomp; ++s) {
            double d = 0;
            if (res >= 0) {
                d = static_cast<double>(a.res_dr[res][s]);
            } else {
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    const double h = static_cast<double>(
                        ST::dec(A[pidx(a, s, i, zs[CZ[i] + 1], ys[CY[i] + 1] * a.nx + xs[CX[i] + 1])], a.inv_scale));
                    d += h;
                    j[s][0] += CX[i] * h;
                    j[s][1] += CY[i] * h;
                    j[s][2] += CZ[i] * h;
                }
            }
            rs[s] = static_cast<double>(a.rho0[s]) + d;
            rtot += rs[s];
        }
        for (int s = 0; s < e.ncomp; ++s) {
            const double wfl = 1.0 - static_cast<double>(e.ns[static_cast<size_t>(e.c_ns == 2 ? s : 0) * a.N + n]);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double fext = rtot > 0 ? rs[s] / rtot * static_cast<double>(a.F[d]) : 0.0;
                acc[d] += wfl * (j[s][d] + fext / 2.0);
            }
        }
        acc[3] += rtot;
    }
    block_sum<4>(acc, partials + static_cast<size_t>(b) * 4);
}

template <typename ST>
__global__ __launch_bounds__(kRedThreads) void k_monitor_reduce(const char* __restrict__ table,
                                                                const double* __restrict__ partials,
                                                                double* __restrict__ out)
{
    using T = typename ST::T;
    const MonitorEntry<T>* ent = reinterpret_cast<const MonitorEntry<T>*>(table + kBatchEntryOffset);
    const MonitorEntry<T>& e = ent[blockIdx.x];
    double acc[4] = {0, 0, 0, 0};
    for (int b = threadIdx.x; b < e.nblocks; b += kRedThreads)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += partials[static_cast<size_t>(e.block_begin + b) * 4 + k];
    block_sum<4>(acc, out + static_cast<size_t>(blockIdx.x) * 4);
}

template <typename T>
static size_t monitor_bytes_t(int max_domains)
{
    return kBatchEntryOffset + sizeof(MonitorEntry<T>) * static_cast<size_t>(max_domains > 0 ? max_domains : 1);
}

size_t monitor_table_bytes(int storage, int max_domains)
{
    return storage == kF64 ? monitor_bytes_t<double>(max_domains) : monitor_bytes_t<float>(max_domains);
}

int monitor_max_blocks(int max_domains) { return kMonitorBlocksPerDomain * (max_domains > 0 ? max_domains : 1); }

template <typename T>
static int monitor_encode_t(const MonitorDomain* d, int n, void* host)
{
    MonitorHeader* h = static_cast<MonitorHeader*>(host);
    MonitorEntry<T>* e = reinterpret_cast<MonitorEntry<T>*>(static_cast<char*>(host) + kBatchEntryOffset);
    int blocks = 0;
    for (int i = 0; i < n; ++i) {
        e[i].a = make_args<T>(d[i].prob);
        e[i].state = d[i].state;
        e[i].ns = d[i].ns;
        e[i].ncomp = d[i].prob.ncomp;
        e[i].c_ns = d[i].prob.c_ns;
        e[i].block_begin = blocks;
        e[i].nblocks = static_cast<int>(
            std::max<int64_t>(1, std::min<int64_t>(kMonitorBlocksPerDomain, (d[i].prob.N + 4095) / 4096)));
        blocks += e[i].nblocks;
    }
    h->ndom = n;
    h->total_blocks = blocks;
    h->pad[0] = h->pad[1] = 0;
    return blocks;
}

int monitor_encode(int storage, const MonitorDomain* d, int n, void* host)
{
    return storage == kF64 ? monitor_encode_t<double>(d, n, host) : monitor_encode_t<float>(d, n, host);
}

hipError_t launch_monitor(int storage, const void* table, int ndom, int total_blocks, double* partials, double* out,
                          hipStream_t st)
{
    if (ndom < 1) return hipSuccess;
    return by_storage(storage, [&](auto tag) {
        using ST = decltype(tag);
        hipLaunchKernelGGL((k_monitor<ST>), dim3(total_blocks), dim3(kRedThreads), 0, st,
                           static_cast<const char*>(table), partials);
        hipLaunchKernelGGL((k_monitor_reduce<ST>), dim3(ndom), dim3(kRedThreads), 0, st,
                           static_cast<const char*>(table), partials, out);
        return hipGetLastError();
    });
}

// ---------------------------------------------------------------------------
// Batched launches.

template <typename T>
static size_t batch_bytes_t(int max_domains)
{
    return kBatchEntryOffset + sizeof(BatchEntry<T>) * static_cast<size_t>(max_domains > 0 ? max_domains : 1);
}

size_t batch_table_bytes(int storage, int max_domains)
{
    return storage == kF64 ? batch_bytes_t<double>(max_domains) : batch_bytes_t<float>(max_domains);
}

template <typename T>
static int batch_encode_t(const BatchDomain* d, int n, void* host)
{
    BatchHeader* h = static_cast<BatchHeader*>(host);
    BatchEntry<T>* e = reinterpret_cast<BatchEntry<T>*>(static_cast<char*>(host) + kBatchEntryOffset);
    int tiles = 0;
    for (int i = 0; i < n; ++i) {
        Args<T> a = make_args<T>(d[i].prob);
        a.zchunk = d[i].zchunk;
        a.tw = d[i].tile_x;
        a.th = d[i].tile_y;
        a.ntx = (d[i].prob.nx + a.tw - 1) / a.tw;
        a.nty = (d[i].prob.ny + a.th - 1) / a.th;
        a.nzc = (d[i].prob.nz + a.zchunk - 1) / a.zchunk;
        a.t = static_cast<uint32_t>(d[i].t);
        e[i].a = a;
        e[i].buf[0] = d[i].buf[0];
        e[i].buf[1] = d[i].buf[1];
        e[i].ns = d[i].ns;
        e[i].parity = d[i].parity;
        e[i].steps = d[i].steps;
        e[i].tile_begin = tiles;
        e[i].ntiles = a.ntx * a.nty * a.nzc;
        tiles += e[i].ntiles;
    }
    h->ndom = n;
    h->total_tiles = tiles;
    h->pad[0] = h->pad[1] = 0;
    return tiles;
}

int batch_encode(int storage, const BatchDomain* d, int n, void* host)
{
    return storage == kF64 ? batch_encode_t<double>(d, n, host) : batch_encode_t<float>(d, n, host);
}

// Kernel of a store policy (FP64 has one).
template <typename ST, int NC, int CNS>
static auto batch_kernel(bool nt)
{
    constexpr int CACHED = sizeof(typename ST::E) == 8 ? kNT : 0;
    return nt ? k_step_batch<ST, NC, CNS, kNT> : k_step_batch<ST, NC, CNS, CACHED>;
}

template <typename ST, int NC, int CNS>
static hipError_t batch_t(const void* table, int k, int grid, bool nt, hipStream_t st)
{
    hipLaunchKernelGGL((batch_kernel<ST, NC, CNS>(nt)), dim3(grid), dim3(kThreads<ST, NC>), 0, st,
                       static_cast<const char*>(table), k);
    return hipGetLastError();
}

template <typename ST, int NC, int CNS>
static int batch_occ_t()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel<ST, NC, CNS>(true), kThreads<ST, NC>, 0) !=
        hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

// One function for every (format, components, n_s fields) of the batched
// kernel: f receives the compiled instance's launcher and occupancy.
template <typename F>
static hipError_t batch_dispatch(int storage, int ncomp, int c_ns, F&& f)
{
    return by_storage(storage, [&](auto tag) {
        using ST = decltype(tag);
        if (ncomp == 1) return f(batch_t<ST, 1, 1>, batch_occ_t<ST, 1, 1>);
        if (c_ns == 1) return f(batch_t<ST, 2, 1>, batch_occ_t<ST, 2, 1>);
        return f(batch_t<ST, 2, 2>, batch_occ_t<ST, 2, 2>);
    });
}

bool batch_tile_supported(int storage, int ncomp, int tx, int ty)
{
    if (pair_layout(storage, ncomp)) return tx == 64 && ty == 8;
    return (tx == 64 && ty == 8) || (tx == 32 && ty == 8);
}

int batch_blocks_per_cu(int storage, int ncomp, int c_ns)
{
    int n = 1;
    (void)batch_dispatch(storage, ncomp, c_ns, [&](auto, auto occ) {
        n = occ();
        return hipSuccess;
    });
    return n;
}

hipError_t launch_step_batch(int storage, int ncomp, int c_ns, const void* table, int k, int grid, bool nt,
                             hipStream_t st)
{
    return batch_dispatch(storage, ncomp, c_ns, [&](auto launch, auto) { return launch(table, k, grid, nt, st); });
}

}  // namespace hm
