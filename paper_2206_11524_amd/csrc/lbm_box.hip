// Step kernel for small domains: one box of cells per block.
//
// The 2.5-D sweeps of lbm_kernels.hip march a block along z, one memory round
// trip per plane; on a domain whose planes give only a few blocks that chain of
// round trips is the whole step (32^3 in FP64: six planes, 25.7 us a step).  Here a
// block owns a box of bx x by x bz cells and takes it in ONE round trip: waves
// of their own pull the cells of the box and of the one-cell halo around it at
// once (the halo only for the densities and n_s), exchange densities through
// LDS, and after a single barrier the box's waves collide and store.  The halo
// re-reads one to two times the box, from the caches that a small domain's state
// sits in; what bounds the step then is one launch, one round trip and, from
// about 10^5 cells, the caches' bandwidth.  Us a step, sweep / box: 500 x 2 x 1
// FP64 7.1 / 5.0, 300 x 50 x 1 FP32 7.0 / 4.7, 32^3 FP64 25.7 / 8.1, 48 x 48 x 64
// FP16 21.7 / 11.1, 64 x 64 x 128 FP32 with one component 18.5 / 15.7.
#include "lbm_device.h"

#include <algorithm>

namespace hm {

constexpr int kBoxCells = 1152;   // staged cells of a box with its halo, at most
constexpr int kBoxCells1 = 2048;  // the same with one component (only n_s is staged around the box)
constexpr int kBoxMaxThreads = 1024;

// Box dimensions of a launch and the thread groups of a block: own_pad and
// halo_pad are the largest own and halo cell counts, in whole waves.
struct BoxDims {
    int bx, by, bz;
    int nbx, nby;
    int own_pad, halo_pad;
};

template <typename ST, int NC, int CNS, bool PAIR>
struct BoxShared {
    using T = typename ST::T;
    static constexpr int LP = NC == 1 ? kBoxCells1 : kBoxCells;
    T rho[NC][LP];
    float ns[CNS][LP];
    T j[PAIR || NC == 1 ? 1 : 2][3][PAIR || NC == 1 ? 1 : kBoxMaxThreads / 2];
};

template <typename ST, int NC, int CNS, int FS, int RND, int AUX>
__global__ __launch_bounds__(kBoxMaxThreads) void k_step_box(Args<typename ST::T> a, BoxDims b,
                                                             const typename ST::E* __restrict__ A,
                                                             typename ST::E* __restrict__ B,
                                                             const float* __restrict__ ns)
{
    using T = typename ST::T;
    constexpr bool PAIR = kPair<ST, NC, FS>;
    using W = std::conditional_t<PAIR, typename PairWordOf<ST>::W, typename ST::E>;
    constexpr int GROUPS = PAIR ? 1 : NC;  // threads per cell
    __shared__ BoxShared<ST, NC, CNS, PAIR> sh;

    const int L = xcd_tile(blockIdx.x, gridDim.x);
    const int ix = L % b.nbx, iyz = L / b.nbx;
    const int iy = iyz % b.nby, iz = iyz / b.nby;
    const int x0 = ix * b.bx, y0 = iy * b.by, z0 = iz * b.bz;
    const int ex = min(b.bx, a.nx - x0), ey = min(b.by, a.ny - y0), ez = min(b.bz, a.nz - z0);
    // a one-plane domain is its own neighbour in z: no halo planes, plane
    // stride 0
    const bool one = a.nz == 1;
    const BoxGeom<BoxShared<ST, NC, CNS, PAIR>::LP> geo{ex + 2};
    const int lxy = one ? 0 : geo.lw * (ey + 2);

    // role of this wave: own cells of component s, or halo cells of s
    const int wbase = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) & ~63);
    const bool halo = wbase >= GROUPS * b.own_pad;
    const int rel = halo ? wbase - GROUPS * b.own_pad : wbase;
    const int pad = halo ? b.halo_pad : b.own_pad;
    const int s = GROUPS == 1 ? 0 : (rel >= pad ? 1 : 0);
    const int c = rel - s * pad + (static_cast<int>(threadIdx.x) & 63);
    const int face = geo.lw * (ey + 2), ringn = 2 * geo.lw + 2 * ey;
    const int ncell = halo ? (one ? 0 : 2 * face) + ez * ringn : ex * ey * ez;
    const bool act = c < ncell;
    const bool mine = act && !halo;

    int lx, ly, lz;
    if (!halo) {
        const int q = min(c, ncell - 1);
        const int r = q / ex;
        lx = q - r * ex;
        lz = r / ey;
        ly = r - lz * ey;
    } else {
        // z faces (whole staged planes), then the ring of each plane of the box
        int q = min(c, ncell - 1);
        if (!one && q < 2 * face) {
            lz = q < face ? -1 : ez;
            q = q < face ? q : q - face;
            ly = q / geo.lw;
            lx = q - ly * geo.lw - 1;
            ly -= 1;
        } else {
            q -= one ? 0 : 2 * face;
            lz = q / ringn;
            q -= lz * ringn;
            if (q < 2 * geo.lw) {
                ly = q < geo.lw ? -1 : ey;
                lx = (q < geo.lw ? q : q - geo.lw) - 1;
            } else {
                q -= 2 * geo.lw;
                lx = q < ey ? -1 : ex;
                ly = q < ey ? q : q - ey;
            }
        }
    }
    auto wrap = [](int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    const int x = wrap(x0 + lx, a.nx), y = wrap(y0 + ly, a.ny), z = wrap(z0 + lz, a.nz);
    const int me = (lz + 1) * lxy + (ly + 1) * geo.lw + lx + 1;

    // the whole buffer through one descriptor (the host takes this kernel
    // only below 2 GiB a component)
    const uint32_t dir_bytes = static_cast<uint32_t>(a.plane) * static_cast<uint32_t>(sizeof(W));
    const uint32_t pl_bytes = static_cast<uint32_t>(kQ) * dir_bytes;
    const uint32_t all_bytes = static_cast<uint32_t>(a.nz) * pl_bytes;
    const size_t cstride = static_cast<size_t>(a.nz) * kQ * static_cast<size_t>(a.plane);
    const rsrc_t ra = make_rsrc(reinterpret_cast<const W*>(A) + s * cstride, all_bytes);
    const PlaneOffs q = plane_offs<sizeof(W)>(x, y, a.nx, a.ny);
    const uint32_t zo[3] = {static_cast<uint32_t>(wrap(z + 1, a.nz)) * pl_bytes, static_cast<uint32_t>(z) * pl_bytes,
                            static_cast<uint32_t>(wrap(z - 1, a.nz)) * pl_bytes};  // z - c, c = -1, 0, 1

    W e[kQ];
    float nsv[CNS];
    if (act) {
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const uint32_t vo = zo[CZ[i] + 1] + q.o[CY[i] + 1][CX[i] + 1];
            if constexpr (PAIR) e[i] = word_load<W>(ra, vo, static_cast<uint32_t>(i) * dir_bytes);
            else e[i] = ST::bld(ra, vo, static_cast<uint32_t>(i) * dir_bytes);
        }
        const int64_t n = static_cast<int64_t>(z) * a.plane + y * a.nx + x;
#pragma unroll
        for (int k = 0; k < CNS; ++k) nsv[k] = ns[static_cast<size_t>(k) * a.N + n];
    }
    if constexpr (NC == 1) {
        // one component has no cohesion: no halo cells are pulled (halo_pad is
        // 0), and the own threads stage n_s of the box and its halo
        const int staged = face * (one ? 1 : ez + 2);
        for (int k = static_cast<int>(threadIdx.x); k < staged; k += static_cast<int>(blockDim.x)) {
            const int pl = k / face, in = k - pl * face, ry = in / geo.lw, rx = in - ry * geo.lw;
            const int gx = wrap(x0 + rx - 1, a.nx), gy = wrap(y0 + ry - 1, a.ny);
            const int gz = one ? 0 : wrap(z0 + pl - 1, a.nz);
            sh.ns[0][k] = ns[static_cast<int64_t>(gz) * a.plane + gy * a.nx + gx];
        }
    }

    const uint32_t ip = static_cast<uint32_t>(y * a.nx + x);
    const uint32_t cell = static_cast<uint32_t>(z) * static_cast<uint32_t>(a.plane) + ip;
    const uint32_t t_key = fmix32(a.t ^ kGolden);
    const uint32_t own = static_cast<uint32_t>(z) * pl_bytes + ip * static_cast<uint32_t>(sizeof(W));
    const T* rho0 = &sh.rho[0][0];
    const float* ns0 = &sh.ns[0][0];

    if constexpr (PAIR) {
        const uint32_t rbits = reservoir_xy_bits(a, x, y) | reservoir_z_bits(a, z);
        T d0, d1, jm[6];
        if (act) {
            pair_moments<ST>(a, rbits, e, d0, d1, jm);
            sh.rho[0][me] = d0;
            sh.rho[1][me] = d1;
#pragma unroll
            for (int k = 0; k < CNS; ++k) sh.ns[k][me] = nsv[k];
        }
        __syncthreads();
        if (!mine) return;
        const rsrc_t rb = make_rsrc(reinterpret_cast<W*>(B), all_bytes);
        pair_collide<ST, CNS, FS, RND>(
            geo, a, rbits, t_key, cell, me, rho0 - lxy, rho0, rho0 + lxy, ns0 - lxy, ns0, ns0 + lxy, jm,
            [&](int i) { return e[i]; },
            [&](int i, W v) { raw_store<AUX>(v, rb, own, static_cast<uint32_t>(i) * dir_bytes); });
    } else {
        T h[kQ];
        if (act) {
            T dr;
            const bool in = reservoir_dr(a, s, x, y, z, dr);
#pragma unroll
            for (int i = 0; i < kQ; ++i) {
                const T v = ST::dec(e[i], a.inv_scale);
                h[i] = in ? wgt<T>(i) * dr : v;
            }
            sh.rho[s][me] = a.rho0[s] + sum19(h);
            if constexpr (NC == 2) {
                if (!halo) {
                    sh.j[s][0][c] = first_moment<T, 0>(h);
                    sh.j[s][1][c] = first_moment<T, 1>(h);
                    sh.j[s][2][c] = first_moment<T, 2>(h);
                }
                if (s == 0)
#pragma unroll
                    for (int k = 0; k < CNS; ++k) sh.ns[k][me] = nsv[k];
            }
        }
        __syncthreads();
        if (!mine) return;
        T jc[NC][3];
        if constexpr (NC == 1) {
            jc[0][0] = first_moment<T, 0>(h);
            jc[0][1] = first_moment<T, 1>(h);
            jc[0][2] = first_moment<T, 2>(h);
        } else {
#pragma unroll
            for (int k = 0; k < NC; ++k)
#pragma unroll
                for (int d = 0; d < 3; ++d) jc[k][d] = sh.j[k][d][c];
        }
        const rsrc_t rb = make_rsrc(reinterpret_cast<W*>(B) + s * cstride, all_bytes);
        split_collide<ST, NC, CNS, FS>(
            geo, a, s, t_key, cell, me, rho0 - lxy, rho0, rho0 + lxy, ns0 - lxy, ns0, ns0 + lxy, jc, h,
            [&](int i, W v) { raw_store<AUX>(v, rb, own, static_cast<uint32_t>(i) * dir_bytes); });
    }
}

// ---------------------------------------------------------------------------
// Launcher.

// Halo cells that a box pulls: the z faces with their edges, and a ring per
// plane; none with one component.
static int box_halo(const Problem& p, int bx, int by, int bz)
{
    if (p.ncomp == 1) return 0;
    return (p.nz == 1 ? 0 : 2 * (bx + 2) * (by + 2)) + bz * (2 * (bx + 2) + 2 * by);
}

// Threads per cell: the split layout takes each component of a cell by a
// thread of its own, the pair layout both by one.
static int box_groups(const Problem& p)
{
    return p.ncomp == 2 && !pair_layout(p.storage, p.ncomp, p.forcing) ? 2 : 1;
}

static int whole_waves(int64_t n) { return static_cast<int>((n + 63) / 64); }

bool box_fits(const Problem& p, int bx, int by, int bz)
{
    if (bx < 1 || by < 1 || bz < 1 || bx > p.nx || by > p.ny || bz > p.nz) return false;
    if (static_cast<int64_t>(bx + 2) * (by + 2) * (p.nz == 1 ? 1 : bz + 2) > (p.ncomp == 1 ? kBoxCells1 : kBoxCells))
        return false;
    const int groups = box_groups(p);
    const int waves = groups * (whole_waves(bx * by * bz) + whole_waves(box_halo(p, bx, by, bz)));
    // one 32-bit buffer offset spans a component's populations
    const int64_t bytes = p.N * kQ * storage_bytes(p.storage) * (groups == 1 ? p.ncomp : 1);
    return waves * 64 <= kBoxMaxThreads && bytes < (int64_t(1) << 31);
}

// The box kernel takes a domain up to this many cells; beyond, the sweep, which
// re-reads a ring per plane instead of a whole halo, comes to move less from the
// caches.  The bounds are below the sizes where the two meet: they were set while
// the box stored past the caches at every size (it then lost at 64^3 in FP32 and 50^3
// in FP64), and small domains gain most.  us a step, box / sweep, at the bound and
// beyond: two components in 16 bits 16.4 / 21.9 at 64^3, 29 / 30 at 80^3, 47 / 43 at 96^3;
// in FP32 18.6 / 23.1 at 57^3, 23.3 / 25.9 at 64^3, 32 / 31 at 72^3; in FP64 (a thread per
// component) 23.6 / 29.5 at 47 x 47 x 43, 28.8 / 30.2 at 50^3, 37 / 32 at 56^3, and in FP32
// with the GS-WBS 17.1 / 27.5 at 45^3, 22.1 / 27.8 at 56^3.  One component pulls no halo
// and meets the sweep at twice the bound, sooner or later with the shape: in FP32
// 15.7 / 18.5 at 64 x 64 x 128, 29.1 / 34.0 at 128 x 64 x 128, but 28.4 / 26.8 at 96^3 and
// 33.4 / 31.1 at 100^3; in FP16 13.9 / 16.1, 24.3 / 26.0, 25.6 / 25.1 and 27.1 / 28.0; in
// FP64 30.4 / 37.9 at 80^3, 62.8 / 70.1 at 128 x 64 x 128, 56.7 / 57.1 at 96^3.  One plane
// deep 9.2 / 13.7 (FP32) and 18.2 / 25.3 (FP64) at 360 x 360, 15.5 / 18.5 (FP32) at 500 x
// 500.
static int64_t box_max_cells(const Problem& p)
{
    if (p.nz == 1) return int64_t(1) << 17;
    if (p.ncomp == 1) return int64_t(1) << 19;
    if (box_groups(p) == 2) return int64_t(3) << 15;
    return p.storage == kF32 ? int64_t(3) << 16 : int64_t(1) << 18;
}

// Box of a small domain: the least work of the most loaded CU, in waves of own
// and halo cells, weighted by 1 + 16 / bx because short rows cover more cache
// lines per load (50^3 in FP16: 25 x 5 x 2 boxes 8.5 us, 8 x 4 x 8 and the like
// 14 to 20).  Sizes that split the domain evenly are tried.  Over 36 domains and
// formats, with some 20 boxes each timed, the choice is 3 % off the best on
// average and 19 % at most.
bool choose_box(const Problem& p, int cus, int* bx, int* by, int* bz)
{
    if (p.N > box_max_cells(p)) return false;
    const int64_t ncu = std::max(cus, 1);
    double best = -1.0;
    auto part = [](int n, int k) { return (n + k - 1) / k; };
    // the sizes that k even parts of n have, largest first, and the next one
    auto first = [&](int n, int most) { return part(n, part(n, std::min(n, most))); };
    auto next = [&](int n, int v) { return v > 1 ? part(n, part(n, v - 1)) : 0; };
    const int least_x = std::min(p.nx, 8);  // shorter rows never win
    for (int x = first(p.nx, 128); x >= least_x; x = next(p.nx, x))
        for (int y = first(p.ny, 32); y; y = next(p.ny, y))
            for (int z = first(p.nz, 32); z; z = next(p.nz, z)) {
                if (!box_fits(p, x, y, z)) continue;
                const int64_t blocks = static_cast<int64_t>(part(p.nx, x)) * part(p.ny, y) * part(p.nz, z);
                const int waves = box_groups(p) * (whole_waves(x * y * z) + whole_waves(box_halo(p, x, y, z)));
                // one component stages n_s of the whole box with its own threads
                const double stage = p.ncomp == 1 ? 0.1 / 64 * (x + 2) * (y + 2) * (p.nz == 1 ? 1 : z + 2) : 0.0;
                const double cost = static_cast<double>((blocks + ncu - 1) / ncu) * (waves + stage) * (1.0 + 16.0 / x);
                if (best < 0.0 || cost < best) {
                    best = cost;
                    *bx = x;
                    *by = y;
                    *bz = z;
                }
            }
    return best >= 0.0;
}

// While both buffers stay in the L2 caches (4 MB in each of 8 XCDs), stores past
// them cost nothing or save up to a tenth: the lines that they would fill are
// those that the next step reads.  Beyond, the rows of most boxes start and end
// inside lines, which two boxes write in parts, and cached stores merge them; rows of
// whole lines keep non-temporal ones (64 x 64 x 128 with one component in FP32 15.9
// cached, 15.7 past the caches).  Cached
// against non-temporal, us a step: 41^3 in FP32 (10 MB a buffer) 9.3 / 8.7, 57^3 in
// FP16 (14 MB) 15.2 / 17.3, 53 x 148 x 28 in FP16 (17 MB) 16.5 / 20.4, 42^3 in FP64
// (23 MB) 17.9 / 20.6; one component crosses later: 247 x 111 x 8 in FP32 (17 MB)
// 11.6 / 10.1, 101 x 118 x 21 (19 MB) 11.2 / 11.1, 268 x 22 x 51 (23 MB) 12.0 / 13.3,
// 261 x 95 x 19 (36 MB) 17.1 / 22.5, in FP64 (72 MB) 31.9 / 38.4.
bool box_nt_stores(const Problem& p, int bx)
{
    const int64_t state = p.N * kQ * storage_bytes(p.storage) * p.ncomp;
    const int word = storage_bytes(p.storage) * (pair_layout(p.storage, p.ncomp, p.forcing) ? 2 : 1);
    return state < (p.ncomp == 2 ? 14000000 : 22000000) || (p.nx * word % 128 == 0 && bx * word % 128 == 0);
}

template <typename ST, int NC, int CNS, int FS>
static hipError_t box_t(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                        hipStream_t st)
{
    using T = typename ST::T;
    using E = typename ST::E;
    Args<T> a = make_args<T>(p);
    a.t = static_cast<uint32_t>(t);
    constexpr bool PAIR = kPair<ST, NC, FS>;
    BoxDims b{};
    b.bx = l.bx; b.by = l.by; b.bz = l.bz;
    b.nbx = (p.nx + b.bx - 1) / b.bx;
    b.nby = (p.ny + b.by - 1) / b.by;
    const int nbz = (p.nz + b.bz - 1) / b.bz;
    b.own_pad = 64 * whole_waves(b.bx * b.by * b.bz);
    b.halo_pad = 64 * whole_waves(box_halo(p, b.bx, b.by, b.bz));
    const int threads = (PAIR ? 1 : NC) * (b.own_pad + b.halo_pad);
    const dim3 grid(static_cast<unsigned>(b.nbx) * b.nby * nbz);
    auto go = [&](auto rnd, auto aux) {
        hipLaunchKernelGGL((k_step_box<ST, NC, CNS, FS, decltype(rnd)::value, decltype(aux)::value>), grid,
                           dim3(threads), 0, st, a, b, static_cast<const E*>(A), static_cast<E*>(B), ns);
    };
    auto policy = [&](auto rnd) {
        l.nt_stores ? go(rnd, std::integral_constant<int, kNT>{}) : go(rnd, std::integral_constant<int, 0>{});
    };
    constexpr int SR = sizeof(E) == 2 && PAIR ? kRoundStochastic : kRoundNearest;
    if (p.stochastic) policy(std::integral_constant<int, SR>{});
    else policy(std::integral_constant<int, kRoundNearest>{});
    return hipGetLastError();
}

template <typename ST, int NC, int CNS>
static hipError_t box_fs(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                         hipStream_t st)
{
    if (p.forcing == kForcingGuo) return box_t<ST, NC, CNS, kForcingGuo>(p, l, t, A, B, ns, st);
    return box_t<ST, NC, CNS, kForcingShanChen>(p, l, t, A, B, ns, st);
}

template <typename ST>
static hipError_t box_st(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                         hipStream_t st)
{
    if (p.ncomp == 1) return box_fs<ST, 1, 1>(p, l, t, A, B, ns, st);
    if (p.c_ns == 1) return box_fs<ST, 2, 1>(p, l, t, A, B, ns, st);
    return box_fs<ST, 2, 2>(p, l, t, A, B, ns, st);
}

hipError_t launch_step_box(const Problem& p, const Launch& l, int64_t t, const void* A, void* B, const float* ns,
                           hipStream_t st)
{
    if (!box_fits(p, l.bx, l.by, l.bz)) return hipErrorInvalidValue;
    switch (p.storage) {
    case kF64: return box_st<F64>(p, l, t, A, B, ns, st);
    case kF32: return box_st<F32>(p, l, t, A, B, ns, st);
    case kF16: return box_st<F16>(p, l, t, A, B, ns, st);
    case kBF16: return box_st<BF16>(p, l, t, A, B, ns, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hm
