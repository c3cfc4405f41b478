// Host runtime of the HMCSC library: the C ABI of include/lbm.h on top of the
// HIP kernels.  One context = one periodic D3Q19 domain on one device, its two
// population buffers (A -> B, swapped every step), the n_s field, and a scratch
// area for FP64 diagnostics and checkpoint staging.
#include "lbm.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "lbm_internal.h"

namespace hm_rt {

int validate(const lbm_domain* d, const lbm_params* p)
{
    if (!d || !p) return LBM_EINVAL;
    if (d->nx < 1 || d->ny < 1 || d->nz < 1) return LBM_EINVAL;
    // each plane block of 19 direction arrays is addressed through one
    // buffer descriptor with 32-bit offsets
    const int64_t plane = static_cast<int64_t>(d->nx) * d->ny;
    if (plane * hm::kQ * 8 >= (int64_t(1) << 32)) return LBM_EINVAL;
    if (static_cast<int64_t>(d->nz) * plane >= (int64_t(1) << 40)) return LBM_EINVAL;
    if (p->ncomp < 1 || p->ncomp > 2) return LBM_EINVAL;
    if (p->c_ns < 1 || p->c_ns > 2 || p->c_ns > p->ncomp) return LBM_EINVAL;
    for (int s = 0; s < p->ncomp; ++s) {
        if (!(p->tau[s] > 0.5) || !std::isfinite(p->tau[s])) return LBM_EINVAL;
        if (!std::isfinite(p->G_ads[s]) || !std::isfinite(p->rho_shift[s])) return LBM_EINVAL;
    }
    if (!std::isfinite(p->G_inter) || !std::isfinite(p->g_scale)) return LBM_EINVAL;
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(p->F_ext[a])) return LBM_EINVAL;
    if (p->storage < LBM_F64 || p->storage > LBM_BF16S) return LBM_EINVAL;
    if (p->store_scale_log2 < -30 || p->store_scale_log2 > 30) return LBM_EINVAL;
    if ((p->storage == LBM_F64 || p->storage == LBM_F32) && p->store_scale_log2 != 0) return LBM_EINVAL;
    if (p->n_res < 0 || p->n_res > LBM_MAX_RES) return LBM_EINVAL;
    const int dims[3] = {d->nx, d->ny, d->nz};
    for (int r = 0; r < p->n_res; ++r) {
        const lbm_reservoir& R = p->res[r];
        if (R.axis < 0 || R.axis > 2 || R.lo < 0 || R.hi < R.lo || R.hi > dims[R.axis]) return LBM_EINVAL;
        for (int s = 0; s < p->ncomp; ++s)
            if (!std::isfinite(R.rho[s])) return LBM_EINVAL;
    }
    if (p->check_every < 0) return LBM_EINVAL;
    if (p->rounding != LBM_ROUND_NEAREST && p->rounding != LBM_ROUND_STOCHASTIC) return LBM_EINVAL;
    if (p->forcing != LBM_FORCING_SHAN_CHEN && p->forcing != LBM_FORCING_GUO) return LBM_EINVAL;
    return LBM_OK;
}

hm::Problem make_problem(const lbm_domain* d, const lbm_params* p)
{
    hm::Problem q{};
    q.nx = d->nx; q.ny = d->ny; q.nz = d->nz;
    q.N = static_cast<int64_t>(d->nx) * d->ny * d->nz;
    q.ncomp = p->ncomp; q.c_ns = p->c_ns; q.storage = p->storage;
    for (int s = 0; s < 2; ++s) {
        q.tau[s] = s < p->ncomp ? p->tau[s] : 1.0;
        q.Gads_s[s] = s < p->ncomp ? p->G_ads[s] * p->g_scale : 0.0;
        q.rho0[s] = s < p->ncomp ? p->rho_shift[s] : 0.0;
    }
    q.G_s = p->G_inter * p->g_scale;
    q.g_scale = p->g_scale;
    q.G_inter = p->G_inter;
    for (int a = 0; a < 3; ++a) q.F[a] = p->F_ext[a];
    q.scale = std::ldexp(1.0, p->store_scale_log2);
    q.stochastic = (p->storage == LBM_F16S || p->storage == LBM_BF16S) && p->rounding == LBM_ROUND_STOCHASTIC;
    q.forcing = p->forcing == LBM_FORCING_GUO ? hm::kForcingGuo : hm::kForcingShanChen;
    q.n_res = p->n_res;
    for (int r = 0; r < hm::kMaxRes; ++r) {
        if (r < p->n_res) {
            q.res_axis[r] = p->res[r].axis; q.res_lo[r] = p->res[r].lo; q.res_hi[r] = p->res[r].hi;
            q.res_rho[r][0] = p->res[r].rho[0];
            q.res_rho[r][1] = p->ncomp == 2 ? p->res[r].rho[1] : 0.0;
        } else {
            q.res_axis[r] = 0; q.res_lo[r] = 0; q.res_hi[r] = 0;
            q.res_rho[r][0] = q.res_rho[r][1] = 0.0;
        }
    }
    return q;
}

int env_int(const char* name, int dflt)
{
    const char* v = std::getenv(name);
    if (!v || !*v) return dflt;
    return std::atoi(v);
}

hm::Launch choose_launch(const hm::Problem& p, int cus, bool batched)
{
    hm::Launch l{};
    // small domains: the box kernel, unless a tile or chunk of the sweep is
    // asked for (LBM_BOX = "bx,by,bz" sets the box, "0" keeps to the sweep)
    const char* box = std::getenv("LBM_BOX");
    if (box && *box) {
        int d[3] = {0, 0, 0};
        if (std::sscanf(box, "%d,%d,%d", d, d + 1, d + 2) == 3 && hm::box_fits(p, d[0], d[1], d[2])) {
            l.bx = d[0]; l.by = d[1]; l.bz = d[2];
        }
    } else if (!batched && !env_int("LBM_TILE_X", 0) && !env_int("LBM_TILE_Y", 0) && !env_int("LBM_ZCHUNK", 0) &&
               !hm::choose_box(p, cus, &l.bx, &l.by, &l.bz)) {
        l.bx = 0;
    }
    const bool pair = hm::pair_layout(p.storage, p.ncomp, p.forcing);
    int cells, rows;
    hm::tile_limits(p, &cells, &rows);
    const int env_x = env_int("LBM_TILE_X", 0), env_y = env_int("LBM_TILE_Y", 0), env_z = env_int("LBM_ZCHUNK", 0);
    l.tile_x = env_x ? env_x : 64;
    l.tile_y = env_y ? env_y : std::min(cells / 64, p.ny);
    const bool given = (env_x || env_y) && hm::tile_supported(p, l.tile_x, l.tile_y);
    if (!given) {
        l.tile_x = 64;
        l.tile_y = std::min(cells / 64, p.ny);
    }
    l.cells = hm::block_cells(p, l.tile_x, l.tile_y);
    const int64_t ncu = std::max(cus, 1);
    const int64_t word = hm::storage_bytes(p.storage) * (pair ? 2 : 1);
    auto part = [](int n, int k) { return (n + k - 1) / k; };
    // One block fits a CU (registers and LDS), so blocks run in rounds of one
    // per CU, and a block takes about (chunk + fill) plane times: the halo planes,
    // the pipeline fill and drain and the block's start cost as much as about
    // eight planes (fitted to timings of 192^3 to 384^3 domains), as five in the
    // 16-bit pair sweep, which keeps two planes of loads in flight: 254 x 268 x 30
    // takes 64 x 7 tiles of 10 planes, 107 us a step, 129 with 64 x 5 of 30.  Take
    // the tile and chunking with the least rounds x (chunk + fill) x plane time,
    // the fewest chunks among equals.  Two blocks fit a CU with one component in
    // FP32 arithmetic and in thin domains, but share its time: over 123 domains
    // with one component the choices are 1.8 % off the best with one block counted
    // per CU, 10 % with two.
    // Chunks shorter than 16 planes spend too much on their halo, unless the domain
    // would then give fewer than two such tiles per CU: a small domain would leave
    // most CUs idle, and its halo re-reads are L2 hits.
    //
    // The sweeps take any tile within tile_limits.  A plane time falls with the
    // lanes that have a cell, by 30 % at most where the domain streams from
    // memory and by 15 % where the caches hold both buffers (the planes then wait
    // on latency: 64 x 64 x 129 with 6 of 8 rows and 6 planes per block takes 45 us in
    // FP32 and 33 in FP16, whole 64 x 8 tiles of 5 planes 41 and 29; 63^3 in FP64
    // with 63 x 2 and 8 planes 54, with 63 x 4 and 4 planes 38).  It rises with
    // shorter rows (8 / w, 10 / w in the 16-bit pair sweep) and with tiles that split cache lines: by 30 % beyond the
    // caches where the rows of the domain are whole ones (160 x 242 x 96 with one
    // component in FP32, 54-wide tiles 172 us, 32-wide 108), otherwise by 8 % in
    // domains many times the caches' size (with two components in FP64, which store
    // past the caches, by 3 and 12 %).  Lines count 64 bytes in FP64, where a
    // non-temporal store of eight values fills such a sector (200 x 200 x 100 with one
    // component: 50-wide tiles 319 us, 40-wide 247), 128 in the other formats.  Over
    // 324 domains of 1.4 thousand to 14 million cells in six formats, up to 16 tiles
    // and chunks each, the choice is 1.2 % off the best on average.
    // Even parts of the domain are tried beside 64 x 8: 131^3 in FP16 takes 44 x 11
    // tiles (109 us a step, 125 with 64 x 8), 100^3 50 x 10 (48 / 56); 192^3 and 224^3
    // keep 64 x 8 (264 against 266 us with 64 x 7, 416 against 516 with 56 x 9 in FP16);
    // one component 150^3 50 x 9 (FP32 115 / 148, FP16 80 / 91); the GS-WBS in FP32 150 x
    // 150 x 100 50 x 9 (205 / 236).
    //
    // In a batched launch every block strides over many tiles: there the tile of
    // the least columns x plane time is taken, with 60 % of the time following
    // the lanes in FP32, where enough tiles fill the memory, and a higher price of
    // short rows (eight 96^3 domains in FP32: 501 us a step with 64 x 8 tiles, 486
    // with 48 x 10, 518 with 32 x 16; twelve 67^3 431 and 310 with 34 x 14; in FP16 276
    // and 188), and no tile that splits the lines of rows
    // that are whole ones (64 domains of edges 32 to 128, all but 48 whole lines,
    // in FP16: 38.9 million cells at 25.3 GLUPS with such tiles and cached stores,
    // 26.8 with whole lines and non-temporal stores).
    //
    // Two components in FP64 take 256 cells: 200 x 200 x 100 64 x 4 tiles 600 us, 50 x 5
    // 638; 131^3 44 x 5 363, 64 x 4 407.
    const int64_t state = p.N * hm::kQ * hm::storage_bytes(p.storage) * p.ncomp;
    const bool f64 = p.storage == hm::kF64;
    const bool cached = state < (int64_t(1) << 27);  // both buffers within the 256 MB of the last cache
    const double follow = cached ? 0.15 : 0.3;
    const bool half = pair && p.storage != hm::kF32;
    const int fill = half ? 5 : 8;
    const double narrow_row = half ? 10.0 : 8.0;
    const bool wide = f64 && p.ncomp == 2;
    const double split = wide ? (p.N > 1500000 ? 1.12 : 1.03) : (p.N > 6000000 ? 1.08 : 1.005);
    const int64_t line = f64 ? 64 : 128;
    auto each_tile = [&](auto&& consider) {
        const int k0 = part(p.nx, 64);
        for (int k = k0 - 1; k <= k0 + 3; ++k) {
            const int w = k < k0 ? 64 : part(p.nx, k);
            if (w > p.nx || (k > k0 && w < 24)) continue;
            int h = part(p.ny, part(p.ny, std::min(std::min(rows, cells / w), p.ny)));
            for (;;) {
                consider(w, h);
                if (h == 1 || h * w < cells / 2) break;
                h = part(p.ny, part(p.ny, h - 1));
            }
        }
    };
    auto columns = [&](int w, int h) { return static_cast<int64_t>(part(p.nx, w)) * part(p.ny, h); };
    auto lanes_of = [&](int64_t cols, int block) {
        return static_cast<double>(p.nx) * p.ny / (static_cast<double>(cols) * block);
    };
    // the tile in batched launches (one plane: whole rows)
    l.batch_x = 64;
    l.batch_y = std::min(cells / 64, p.ny);
    double batch_best = -1.0;
    if (p.nz > 1)
        each_tile([&](int w, int h) {
            const int64_t cols = columns(w, h);
            const double lanes = lanes_of(cols, cells);
            const double share = p.storage == hm::kF32 || p.storage == hm::kF64 ? 0.6 : 0.3;
            const bool aligned = p.nx * word % 128 == 0 && w * word % 128 == 0;
            const double narrow = 1.0 + (hm::storage_bytes(p.storage) == 2 ? 20.0 : 16.0) / w;
            const double column =
                static_cast<double>(cols) * (1.0 - share + share * lanes) * narrow * (aligned ? 1.0 : 1.08);
            const bool splits = p.nx * word % 128 == 0 && w * word % 128 != 0;
            if (!splits && (batch_best < 0.0 || column < batch_best)) {
                batch_best = column;
                l.batch_x = w;
                l.batch_y = h;
            }
        });
    if (batched) return l;
    // the tile and chunk of the sweep
    double best = -1.0;
    auto consider = [&](int w, int h) {
        const int64_t cols = columns(w, h);
        const double lanes = lanes_of(cols, l.cells);
        const double lines = (h * w == l.cells && w % 32 == 0 ? 1.0 : split) *
                             (!cached && p.nx * word % line == 0 && w * word % line != 0 ? 1.3 : 1.0);
        const double plane = (1.0 - follow + follow * lanes) * (1.0 + narrow_row / w) * lines;
        const int64_t tiles16 = cols * ((p.nz + 15) / 16);
        const int min_chunk = tiles16 >= 2 * ncu ? 16 : 4;
        // the distinct chunk lengths of even parts of nz, longest first
        for (int z = env_z ? std::min(std::max(env_z, 1), p.nz) : p.nz;;) {
            const int64_t blocks = cols * part(p.nz, z);
            const double cost = static_cast<double>(((blocks + ncu - 1) / ncu) * (z + fill)) * plane;
            if (best < 0.0 || cost < best) {
                best = cost;
                l.tile_x = w;
                l.tile_y = h;
                l.zchunk = z;
            }
            if (env_z || z == 1) break;
            z = part(p.nz, part(p.nz, z - 1));
            if (z < min_chunk) break;
        }
    };
    if (given || p.nz == 1) consider(l.tile_x, l.tile_y);
    else each_tile(consider);
    // Non-temporal stores keep the written state out of the caches' way, but
    // where a tile's rows start or end inside a 128-byte line the two tiles that
    // share it each write part of it, and only a cached line is merged before it
    // goes out: 131^3 in FP32 179 us a step with cached stores against 206, 100^3 in
    // FP16 49 against 56; with whole lines non-temporal stores are the faster ones
    // (256^3 in FP32 970 against 997).
    // Two components in FP64 keep them (150^3 548 against 577, 160^3 528 against 550);
    // one component follows its 64-byte lines: 150^3 226 cached against 267, 131 x 110 x
    // 209 202 against 250, 317 x 125 x 210 528 against 605, but 160^3 4 % slower.
    if (l.bx > 0) l.nt_stores = hm::box_nt_stores(p, l.bx);
    else l.nt_stores = wide || (l.tile_x * word % line == 0 && p.nx * word % line == 0);
    return l;
}

}  // namespace hm_rt

using namespace hm_rt;

#define HIP_TRY(expr)                                  \
    do {                                               \
        if ((expr) != hipSuccess) return LBM_EDEVICE;  \
    } while (0)

// Queue the FP64 diagnostics (the per-cell fields and the totals in scratch); a
// caller that only launches on from the fields need not wait for the totals.
static int launch_fields(lbm_ctx* c, bool fields, bool forces)
{
    double* rho = reinterpret_cast<double*>(c->scratch + c->sl.rho);
    double* u = reinterpret_cast<double*>(c->scratch + c->sl.u);
    double* p = reinterpret_cast<double*>(c->scratch + c->sl.p);
    double* part = reinterpret_cast<double*>(c->scratch + c->sl.partials);
    double* tots = reinterpret_cast<double*>(c->scratch + c->sl.totals);
    HIP_TRY(hm::launch_diagnostics(c->prob, c->buf[c->cur], c->ns, forces || fields, rho, fields ? u : nullptr,
                                   fields ? p : nullptr, part, tots, c->stream));
    return LBM_OK;
}

int hm_rt::compute_totals(lbm_ctx* c, bool fields, bool forces, lbm_totals* tot)
{
    const int rc = launch_fields(c, fields, forces);
    if (rc) return rc;
    const double* tots = reinterpret_cast<const double*>(c->scratch + c->sl.totals);
    double h[5];
    HIP_TRY(hipMemcpyAsync(h, tots, sizeof(h), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (tot) {
        tot->mass[0] = h[0];
        tot->mass[1] = c->prm.ncomp == 2 ? h[1] : 0.0;
        for (int a = 0; a < 3; ++a) tot->momentum[a] = h[2 + a];
        tot->time = c->t;
        int fin = 1;
        for (double v : h) fin &= std::isfinite(v) ? 1 : 0;
        tot->finite = fin;
        tot->pad = 0;
    }
    return LBM_OK;
}

extern "C" {

const char* lbm_strerror(int code)
{
    switch (code) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument";
    case LBM_ENOMEM: return "out of memory";
    case LBM_EDEVICE: return "HIP device error";
    case LBM_EUNSTABLE: return "non-finite state (unstable simulation)";
    case LBM_ENOTFOUND: return "unknown ticket";
    case LBM_EAGAIN: return "not ready";
    default: return "unknown error";
    }
}

int lbm_required_bytes(const lbm_domain* d, const lbm_params* p, lbm_sizes* out)
{
    const int rc = validate(d, p);
    if (rc) return rc;
    if (!out) return LBM_EINVAL;
    const int64_t N = static_cast<int64_t>(d->nx) * d->ny * d->nz;
    out->pop_bytes = align_up(static_cast<size_t>(hm::storage_bytes(p->storage)) * hm::kQ * p->ncomp * N);
    out->ns_bytes = align_up(sizeof(float) * static_cast<size_t>(p->c_ns) * N);
    out->scratch_bytes = scratch_layout(N, p->ncomp).bytes;
    return LBM_OK;
}

static void free_owned(lbm_ctx* c)
{
    if (!c->owned) return;
    if (c->buf[0]) (void)hipFree(c->buf[0]);
    if (c->buf[1]) (void)hipFree(c->buf[1]);
    if (c->ns) (void)hipFree(c->ns);
    if (c->scratch) (void)hipFree(c->scratch);
    c->buf[0] = c->buf[1] = nullptr;
    c->ns = nullptr;
    c->scratch = nullptr;
}

void lbm_destroy(lbm_ctx* c)
{
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    free_owned(c);
    if (c->ev0) (void)hipEventDestroy(c->ev0);
    if (c->ev1) (void)hipEventDestroy(c->ev1);
    delete c;
}

int lbm_create(const lbm_domain* dom, const float* n_s, const double* rho_init, const lbm_params* prm,
               const lbm_device_buffers* bufs, void* stream, lbm_ctx** out)
{
    if (!out) return LBM_EINVAL;
    *out = nullptr;
    int rc = validate(dom, prm);
    if (rc) return rc;
    if (!n_s || !rho_init) return LBM_EINVAL;
    const int64_t N = static_cast<int64_t>(dom->nx) * dom->ny * dom->nz;
    for (int64_t k = 0; k < static_cast<int64_t>(prm->c_ns) * N; ++k)
        if (!(n_s[k] >= 0.0f && n_s[k] <= 1.0f)) return LBM_EINVAL;
    for (int64_t k = 0; k < static_cast<int64_t>(prm->ncomp) * N; ++k)
        if (!std::isfinite(rho_init[k])) return LBM_EINVAL;
    if (bufs && (!bufs->f_a || !bufs->f_b || !bufs->n_s || !bufs->scratch)) return LBM_EINVAL;
    if (bufs) {
        const void* ps[4] = {bufs->f_a, bufs->f_b, bufs->n_s, bufs->scratch};
        for (const void* q : ps)
            if (reinterpret_cast<uintptr_t>(q) % kAlign) return LBM_EINVAL;
    }

    lbm_ctx* c = new (std::nothrow) lbm_ctx();
    if (!c) return LBM_ENOMEM;
    c->dom = *dom;
    c->prm = *prm;
    c->prob = make_problem(dom, prm);

    lbm_required_bytes(dom, prm, &c->sizes);
    c->sl = scratch_layout(N, prm->ncomp);
    c->stream = static_cast<hipStream_t>(stream);
    c->cur = 0;
    c->t = 0;
    if (hipGetDevice(&c->device) != hipSuccess) { delete c; return LBM_EDEVICE; }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
        delete c;
        return LBM_EDEVICE;
    }
    c->launch = choose_launch(c->prob, cus, false);
    if (hipEventCreate(&c->ev0) != hipSuccess || hipEventCreate(&c->ev1) != hipSuccess) {
        lbm_destroy(c);
        return LBM_EDEVICE;
    }
    if (bufs) {
        c->owned = false;
        c->buf[0] = bufs->f_a;
        c->buf[1] = bufs->f_b;
        c->ns = static_cast<float*>(bufs->n_s);
        c->scratch = static_cast<char*>(bufs->scratch);
    } else {
        c->owned = true;
        if (hipMalloc(&c->buf[0], c->sizes.pop_bytes) != hipSuccess ||
            hipMalloc(&c->buf[1], c->sizes.pop_bytes) != hipSuccess ||
            hipMalloc(reinterpret_cast<void**>(&c->ns), c->sizes.ns_bytes) != hipSuccess ||
            hipMalloc(reinterpret_cast<void**>(&c->scratch), c->sizes.scratch_bytes) != hipSuccess) {
            (void)hipGetLastError();
            lbm_destroy(c);
            return LBM_ENOMEM;
        }
    }
    // n_s and the initial densities; the densities are staged in the rho slot of scratch
    double* rho_dev = reinterpret_cast<double*>(c->scratch + c->sl.rho);
    if (hipMemcpyAsync(c->ns, n_s, sizeof(float) * prm->c_ns * N, hipMemcpyHostToDevice, c->stream) != hipSuccess ||
        hipMemcpyAsync(rho_dev, rho_init, sizeof(double) * prm->ncomp * N, hipMemcpyHostToDevice, c->stream) !=
            hipSuccess ||
        hm::launch_init(c->prob, rho_dev, c->buf[0], c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess) {
        lbm_destroy(c);
        return LBM_EDEVICE;
    }
    *out = c;
    return LBM_OK;
}

}  // extern "C"

// A context over caller buffers that already hold (or will receive) its
// state: no device work, no synchronisation (the server initialises the
// state itself, on its admission stream).
int hm_rt::ctx_bind(const lbm_domain* dom, const lbm_params* prm, const lbm_device_buffers* bufs, hipStream_t stream,
                    lbm_ctx** out)
{
    *out = nullptr;
    int rc = validate(dom, prm);
    if (rc) return rc;
    if (!bufs || !bufs->f_a || !bufs->f_b || !bufs->n_s || !bufs->scratch) return LBM_EINVAL;
    lbm_ctx* c = new (std::nothrow) lbm_ctx();
    if (!c) return LBM_ENOMEM;
    c->dom = *dom;
    c->prm = *prm;
    c->prob = make_problem(dom, prm);
    lbm_required_bytes(dom, prm, &c->sizes);
    c->sl = scratch_layout(c->prob.N, prm->ncomp);
    c->stream = stream;
    c->cur = 0;
    c->t = 0;
    c->owned = false;
    c->buf[0] = bufs->f_a;
    c->buf[1] = bufs->f_b;
    c->ns = static_cast<float*>(bufs->n_s);
    c->scratch = static_cast<char*>(bufs->scratch);
    int cus = 0;
    if (hipGetDevice(&c->device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess ||
        hipEventCreate(&c->ev0) != hipSuccess || hipEventCreate(&c->ev1) != hipSuccess) {
        lbm_destroy(c);
        return LBM_EDEVICE;
    }
    c->launch = choose_launch(c->prob, cus, true);
    *out = c;
    return LBM_OK;
}

extern "C" {

int lbm_step(lbm_ctx* c, int64_t nsteps)
{
    if (!c || nsteps < 0) return LBM_EINVAL;
    if (nsteps == 0) return LBM_OK;
    HIP_TRY(hipEventRecord(c->ev0, c->stream));
    for (int64_t k = 0; k < nsteps; ++k) {
        HIP_TRY(hm::launch_step(c->prob, c->launch, c->t, c->buf[c->cur], c->buf[1 - c->cur], c->ns, c->stream));
        c->cur = 1 - c->cur;
        c->t += 1;
        if (c->prm.check_every > 0 && c->t % c->prm.check_every == 0) {
            lbm_totals tt;
            const int rc = compute_totals(c, false, false, &tt);
            if (rc) return rc;
            if (!tt.finite) return LBM_EUNSTABLE;
        }
    }
    HIP_TRY(hipEventRecord(c->ev1, c->stream));
    c->timed_steps = nsteps;
    return LBM_OK;
}

double lbm_last_step_ms(const lbm_ctx* c)
{
    if (!c || c->timed_steps <= 0) return 0.0;
    if (hipEventSynchronize(c->ev1) != hipSuccess) return 0.0;
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, c->ev0, c->ev1) != hipSuccess) return 0.0;
    return static_cast<double>(ms) / static_cast<double>(c->timed_steps);
}

int lbm_moments(lbm_ctx* c, double* rho, double* u, double* p, lbm_totals* tot)
{
    if (!c) return LBM_EINVAL;
    const bool fields = rho || u || p;
    const int rc = compute_totals(c, fields, true, tot);
    if (rc) return rc;
    const int64_t N = c->prob.N;
    if (rho)
        HIP_TRY(hipMemcpy(rho, c->scratch + c->sl.rho, sizeof(double) * c->prm.ncomp * N, hipMemcpyDeviceToHost));
    if (u) HIP_TRY(hipMemcpy(u, c->scratch + c->sl.u, sizeof(double) * 3 * N, hipMemcpyDeviceToHost));
    if (p) HIP_TRY(hipMemcpy(p, c->scratch + c->sl.p, sizeof(double) * N, hipMemcpyDeviceToHost));
    return LBM_OK;
}

int lbm_totals_get(lbm_ctx* c, lbm_totals* tot)
{
    if (!c || !tot) return LBM_EINVAL;
    return compute_totals(c, false, true, tot);
}

int lbm_get_populations(lbm_ctx* c, double* f)
{
    if (!c || !f) return LBM_EINVAL;
    const int64_t N = c->prob.N;
    double* stage = reinterpret_cast<double*>(c->scratch + c->sl.u);  // N doubles (u slot holds 3N)
    for (int s = 0; s < c->prm.ncomp; ++s)
        for (int i = 0; i < hm::kQ; ++i) {
            HIP_TRY(hm::launch_canonical(c->prob, c->buf[c->cur], s, i, stage, c->stream));
            HIP_TRY(hipMemcpyAsync(f + static_cast<size_t>(s * hm::kQ + i) * N, stage, sizeof(double) * N,
                                   hipMemcpyDeviceToHost, c->stream));
            HIP_TRY(hipStreamSynchronize(c->stream));
        }
    return LBM_OK;
}

int lbm_set_populations(lbm_ctx* c, const double* f)
{
    if (!c || !f) return LBM_EINVAL;
    const int64_t N = c->prob.N;
    for (int64_t k = 0; k < static_cast<int64_t>(c->prm.ncomp) * hm::kQ * N; ++k)
        if (!std::isfinite(f[k])) return LBM_EINVAL;
    double* stage = reinterpret_cast<double*>(c->scratch + c->sl.u);
    for (int s = 0; s < c->prm.ncomp; ++s)
        for (int i = 0; i < hm::kQ; ++i) {
            HIP_TRY(hipMemcpyAsync(stage, f + static_cast<size_t>(s * hm::kQ + i) * N, sizeof(double) * N,
                                   hipMemcpyHostToDevice, c->stream));
            HIP_TRY(hm::launch_set_canonical(c->prob, stage, s, i, c->buf[c->cur], c->stream));
            HIP_TRY(hipStreamSynchronize(c->stream));
        }
    return LBM_OK;
}

int lbm_set_reservoir(lbm_ctx* c, int32_t r, const double rho[2])
{
    if (!c || !rho || r < 0 || r >= c->prm.n_res) return LBM_EINVAL;
    for (int s = 0; s < c->prm.ncomp; ++s)
        if (!std::isfinite(rho[s])) return LBM_EINVAL;
    for (int s = 0; s < c->prm.ncomp; ++s) {
        c->prm.res[r].rho[s] = rho[s];
        c->prob.res_rho[r][s] = rho[s];
    }
    return LBM_OK;
}

int lbm_fill_state_get(lbm_ctx* c, const lbm_fill_query* q, lbm_fill_state* out)
{
    if (!c || !q || !out) return LBM_EINVAL;
    if (q->axis < 0 || q->axis > 2 || q->comp < 0 || q->comp >= c->prm.ncomp) return LBM_EINVAL;
    const int len = q->axis == 0 ? c->dom.nx : (q->axis == 1 ? c->dom.ny : c->dom.nz);
    auto slab_ok = [&](int lo, int hi, bool nonempty) { return lo >= 0 && hi <= len && (nonempty ? lo < hi : lo <= hi); };
    if (!slab_ok(q->inlet_lo, q->inlet_hi, true) || !slab_ok(q->outlet_lo, q->outlet_hi, true) ||
        !slab_ok(q->pore_lo, q->pore_hi, false) || !std::isfinite(q->threshold))
        return LBM_EINVAL;
    const int rc = launch_fields(c, true, true);  // FP64 densities and pressure into the scratch
    if (rc) return rc;
    hm::FillQuery f{q->axis, q->inlet_lo, q->inlet_hi, q->outlet_lo, q->outlet_hi, q->pore_lo, q->pore_hi, q->comp,
                    q->threshold};
    double* part = reinterpret_cast<double*>(c->scratch + c->sl.partials);
    double* tots = reinterpret_cast<double*>(c->scratch + c->sl.totals);
    HIP_TRY(hm::launch_fill(c->prob, f, reinterpret_cast<const double*>(c->scratch + c->sl.rho),
                            reinterpret_cast<const double*>(c->scratch + c->sl.p), c->ns, part, tots, c->stream));
    double h[6];
    HIP_TRY(hipMemcpyAsync(h, tots, sizeof(h), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    out->p_inlet = h[0] / h[1];
    out->p_outlet = h[2] / h[3];
    out->dp = out->p_inlet - out->p_outlet;
    out->saturation = h[5] > 0.0 ? h[4] / h[5] : 0.0;
    out->pore_volume = h[5];
    out->time = c->t;
    return LBM_OK;
}

int lbm_permeability_get(lbm_ctx* c, int32_t axis, lbm_permeability* out)
{
    if (!c || !out || axis < 0 || axis > 2) return LBM_EINVAL;
    const double F = c->prm.F_ext[axis];
    if (F == 0.0 || (c->prm.ncomp == 2 && c->prm.tau[0] != c->prm.tau[1])) return LBM_EINVAL;
    const int rc = launch_fields(c, true, true);  // FP64 densities and u_macro into the scratch
    if (rc) return rc;
    double* part = reinterpret_cast<double*>(c->scratch + c->sl.partials);
    double* tots = reinterpret_cast<double*>(c->scratch + c->sl.totals);
    HIP_TRY(hm::launch_flux(c->prob, axis, reinterpret_cast<const double*>(c->scratch + c->sl.rho),
                            reinterpret_cast<const double*>(c->scratch + c->sl.u), part, tots, c->stream));
    double h[3];
    HIP_TRY(hipMemcpyAsync(h, tots, sizeof(h), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    const double N = static_cast<double>(c->prob.N);
    const double nu = (c->prm.tau[0] - 0.5) / 3.0;
    out->nu = nu;
    out->momentum = h[2] / N;
    out->k = nu * out->momentum / F;
    out->k_comp[0] = nu * (h[0] / N) / F;
    out->k_comp[1] = c->prm.ncomp == 2 ? nu * (h[1] / N) / F : 0.0;
    out->time = c->t;
    return LBM_OK;
}

int lbm_droplet_get(lbm_ctx* c, const lbm_droplet_query* q, lbm_droplet_state* out)
{
    if (!c || !q || !out || q->comp < 0 || q->comp >= c->prm.ncomp) return LBM_EINVAL;
    for (double v : q->center)
        if (!std::isfinite(v)) return LBM_EINVAL;
    if (!(q->r_core > 0.0) || !(q->r_far > q->r_core) || !(q->margin >= 0.0) || !std::isfinite(q->r_far) ||
        !std::isfinite(q->margin))
        return LBM_EINVAL;
    lbm_totals tot{};
    const int rc = compute_totals(c, true, true, &tot);  // FP64 densities and pressure into the scratch
    if (rc) return rc;
    const int64_t N = c->prob.N;
    const double* rho = reinterpret_cast<const double*>(c->scratch + c->sl.rho) + static_cast<size_t>(q->comp) * N;
    const double* pr = reinterpret_cast<const double*>(c->scratch + c->sl.p);
    double* part = reinterpret_cast<double*>(c->scratch + c->sl.partials);
    double* tots = reinterpret_cast<double*>(c->scratch + c->sl.totals);
    double h[4];
    auto ball = [&](const double* f, double r_in, double r_out) -> int {
        HIP_TRY(hm::launch_ball(c->prob, q->center, r_in, r_out, f, part, tots, c->stream));
        HIP_TRY(hipMemcpyAsync(h, tots, sizeof(h), hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        return (h[1] > 0.0 && h[3] > 0.0) ? LBM_OK : LBM_EINVAL;
    };
    int r = ball(rho, q->r_core, q->r_far);
    if (r) return r;
    const double rho_in = h[0] / h[1], rho_out = h[2] / h[3];
    if (!(std::fabs(rho_in - rho_out) > 0.0)) return LBM_EINVAL;
    const double V = (tot.mass[q->comp] - rho_out * static_cast<double>(N)) / (rho_in - rho_out);
    if (!(V > 0.0)) return LBM_EINVAL;
    const bool two_d = c->dom.nz == 1;
    const double pi = 3.14159265358979323846;
    const double R = two_d ? std::sqrt(V / pi) : std::cbrt(3.0 * V / (4.0 * pi));
    r = ball(pr, R / 2.0, R + q->margin);
    if (r) return r;
    out->R = R;
    out->rho_in = rho_in;
    out->rho_out = rho_out;
    out->p_in = h[0] / h[1];
    out->p_out = h[2] / h[3];
    out->dp = out->p_in - out->p_out;
    out->gamma = two_d ? out->dp * R : out->dp * R / 2.0;
    out->time = c->t;
    return LBM_OK;
}

int64_t lbm_time(const lbm_ctx* c) { return c ? c->t : -1; }

int lbm_set_time(lbm_ctx* c, int64_t t)
{
    if (!c || t < 0) return LBM_EINVAL;
    c->t = t;
    return LBM_OK;
}

int lbm_sync(lbm_ctx* c)
{
    if (!c) return LBM_EINVAL;
    HIP_TRY(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

}  // extern "C"
