// Device code shared by the HIP kernels: the velocity set, storage formats,
// kernel parameters, reservoirs, staged-plane stencils and the collision of one
// cell.  Every kernel evaluates these same expressions, so a cell's result does
// not depend on which kernel or launch shape updated it.
#pragma once

#include <stdint.h>

#include <type_traits>

#include "lbm_kernels.h"

namespace hm {

// ---------------------------------------------------------------------------
// D3Q19 velocity set, ordered as printed in Appendix A: directions i and i+9
// (i = 1..9) are opposite.  Weights 1/3, 1/18 (|c| = 1), 1/36 (|c| = sqrt 2).
__device__ constexpr int CX[kQ] = {0, -1, 0, 0, -1, -1, -1, -1, 0, 0, 1, 0, 0, 1, 1, 1, 1, 0, 0};
__device__ constexpr int CY[kQ] = {0, 0, -1, 0, -1, 1, 0, 0, -1, -1, 0, 1, 0, 1, -1, 0, 0, 1, 1};
__device__ constexpr int CZ[kQ] = {0, 0, 0, -1, 0, 0, -1, 1, -1, 1, 0, 0, 1, 0, 0, 1, -1, 1, -1};

__host__ __device__ constexpr int opp(int i) { return i == 0 ? 0 : (i <= 9 ? i + 9 : i - 9); }

template <typename T>
__host__ __device__ constexpr T wgt(int i)
{
    return i == 0 ? T(1) / T(3)
                  : ((CX[i] * CX[i] + CY[i] * CY[i] + CZ[i] * CZ[i]) == 1 ? T(1) / T(18) : T(1) / T(36));
}

// ---------------------------------------------------------------------------
// Storage formats.  decode() returns the shifted value h in the arithmetic
// type T, encode() rounds h back (round to nearest even for 16-bit).
// Buffer resources: raw (stride 0) descriptors whose range check turns any
// access beyond num_records into a zero load / dropped store.  Stores of the
// step are non-temporal (cache-policy bit NT): the next step reads them only
// after the whole domain has streamed through the caches.
using rsrc_t = __amdgpu_buffer_rsrc_t;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf162_t __attribute__((ext_vector_type(2)));
constexpr int kNT = 2;  // cache policy: non-temporal

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                             static_cast<int>(bytes), 0x00020000);
}

struct F64 {
    using E = double;
    using T = double;
    static __device__ __forceinline__ T dec(E v, T) { return v; }
    static __device__ __forceinline__ E enc(T v, T) { return v; }
    static __device__ __forceinline__ E enc_sr(T v, T, uint32_t) { return v; }  // rounds to nearest
    static __device__ __forceinline__ E bld(rsrc_t r, uint32_t vo, uint32_t so)
    {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
    }
};
struct F32 {
    using E = float;
    using T = float;
    static __device__ __forceinline__ T dec(E v, T) { return v; }
    static __device__ __forceinline__ E enc(T v, T) { return v; }
    static __device__ __forceinline__ E enc_sr(T v, T, uint32_t) { return v; }  // rounds to nearest
    static __device__ __forceinline__ E bld(rsrc_t r, uint32_t vo, uint32_t so)
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
    }
};
struct Half16 {
    static __device__ __forceinline__ uint16_t bld(rsrc_t r, uint32_t vo, uint32_t so)
    {
        return __builtin_amdgcn_raw_buffer_load_b16(r, vo, so, 0);
    }
};
struct F16 : Half16 {
    using E = uint16_t;
    using T = float;
    static __device__ __forceinline__ T dec(E v, T inv_scale)
    {
        return static_cast<float>(__builtin_bit_cast(_Float16, v)) * inv_scale;
    }
    static __device__ __forceinline__ E enc(T v, T scale)
    {
        return __builtin_bit_cast(uint16_t, static_cast<_Float16>(v * scale));
    }
    // Stochastic rounding with the random word r (v_cvt_sr_f16_f32): the
    // instruction reads its random operand as a binary fraction from the top
    // bit down and rounds the magnitude up with probability equal to the
    // value's fraction of the binary16 spacing, subnormals included (checked
    // on the device: up only for bit 31 at half a spacing, frequencies equal
    // to the fraction, exact values unchanged, inf and NaN kept).  The top 16
    // bits of r are random (see lcg24), so the probability is resolved to
    // 2^-16.
    static __device__ __forceinline__ E enc_sr(T v, T scale, uint32_t r)
    {
        half2_t h = {0, 0};
        h = __builtin_amdgcn_cvt_sr_f16_f32(h, v * scale, r, false);
        return __builtin_bit_cast(uint16_t, h[0]);
    }
};
struct BF16 : Half16 {
    using E = uint16_t;
    using T = float;
    static __device__ __forceinline__ T dec(E v, T inv_scale)
    {
        return __uint_as_float(static_cast<uint32_t>(v) << 16) * inv_scale;
    }
    // round to nearest, ties to even (gfx950's v_cvt_pk_bf16_f32)
    static __device__ __forceinline__ E enc(T v, T scale)
    {
        return __builtin_bit_cast(uint16_t, static_cast<__bf16>(v * scale));
    }
    // Stochastic rounding with the random word r (v_cvt_sr_bf16_f32, the same
    // convention as the binary16 instruction).
    static __device__ __forceinline__ E enc_sr(T v, T scale, uint32_t r)
    {
        bf162_t h = {0, 0};
        h = __builtin_amdgcn_cvt_sr_bf16_f32(h, v * scale, r, false);
        return __builtin_bit_cast(uint16_t, h[0]);
    }
};

// MurmurHash3's 32-bit finaliser (Appleby): a bijective avalanche mixer; the
// random bits of the stochastic rounding are fmix32 of a counter built from
// cell, component, direction and time step.
__device__ __forceinline__ uint32_t fmix32(uint32_t h)
{
    h ^= h >> 16;
    h *= 0x85ebca6bu;
    h ^= h >> 13;
    h *= 0xc2b2ae35u;
    h ^= h >> 16;
    return h;
}
constexpr uint32_t kGolden = 0x9e3779b9u;

// The following random words of one (cell, component), after fmix32 has
// seeded them: a linear congruential step modulo 2^24 (multiplier = 1 mod 4,
// odd increment: full period by Hull and Dobell's conditions) on the low 24
// bits of the previous word, kept as the 32-bit value a*x + c, whose top 16
// bits the rounding reads.  One 24-bit multiply-add (v_mad_u32_u24) per
// stored value.
constexpr uint32_t kLcgA = 0x6d2b79u, kLcgC = 0x2b5a3fu;
static_assert(kLcgA % 4 == 1 && kLcgC % 2 == 1 && kLcgA < (1u << 24), "full-period LCG modulo 2^24");
__device__ __forceinline__ uint32_t lcg24(uint32_t x) { return (x & 0xffffffu) * kLcgA + kLcgC; }

// Two 16-bit values of one (cell, direction) in one 32-bit word of the pair
// layout: component 0 in the low half, component 1 in the high half.  The
// pair kernel works on the stored scale (h * 2^k): the power-of-two factor
// is folded into the few per-cell coefficients instead of every value, which
// changes no bit (scaling by 2^k commutes with rounding).
template <typename ST>
struct PairCodec {
    static __device__ __forceinline__ float lo(uint32_t v) { return ST::dec(static_cast<uint16_t>(v & 0xffffu), 1.0f); }
    static __device__ __forceinline__ float hi(uint32_t v) { return ST::dec(static_cast<uint16_t>(v >> 16), 1.0f); }
    // x_H + y_H and x_H - y_H for the halves H (0 low, 1 high) of two words,
    // each rounded once to FP32.  Binary16: one v_fma_mix_f32 (x * 1 + y with
    // both sources converted from binary16 inside the instruction) instead of
    // two conversions and an add; the result is the same, as the conversions
    // are exact.  bfloat16 decodes with one shift or mask per value anyway.
    template <int H>
    static __device__ __forceinline__ float sum(uint32_t x, uint32_t y)
    {
        if constexpr (std::is_same_v<ST, F16>) {
            float r;
            if constexpr (H == 0)
                asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "v"(y));
            else
                asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "v"(y));
            return r;
        } else {
            return H == 0 ? lo(x) + lo(y) : hi(x) + hi(y);
        }
    }
    template <int H>
    static __device__ __forceinline__ float diff(uint32_t x, uint32_t y)
    {
        if constexpr (std::is_same_v<ST, F16>) {
            float r;
            if constexpr (H == 0)
                asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "v"(y));
            else
                asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "v"(y));
            return r;
        } else {
            return H == 0 ? lo(x) - lo(y) : hi(x) - hi(y);
        }
    }
    static __device__ __forceinline__ uint32_t enc(float a, float b)
    {
        if constexpr (std::is_same_v<ST, BF16>) {
            const bf162_t h = {static_cast<__bf16>(a), static_cast<__bf16>(b)};
            return __builtin_bit_cast(uint32_t, h);
        } else {
            const half2_t h = {static_cast<_Float16>(a), static_cast<_Float16>(b)};
            return __builtin_bit_cast(uint32_t, h);
        }
    }
    // stochastic rounding (see F16::enc_sr) of a into the low and b into the
    // high half of one word, with the random words ra and rb
    static __device__ __forceinline__ uint32_t enc_sr(float a, float b, uint32_t ra, uint32_t rb)
    {
        if constexpr (std::is_same_v<ST, BF16>) {
            bf162_t h = {0, 0};
            h = __builtin_amdgcn_cvt_sr_bf16_f32(h, a, ra, false);
            h = __builtin_amdgcn_cvt_sr_bf16_f32(h, b, rb, true);
            return __builtin_bit_cast(uint32_t, h);
        } else {
            half2_t h = {0, 0};
            h = __builtin_amdgcn_cvt_sr_f16_f32(h, a, ra, false);
            h = __builtin_amdgcn_cvt_sr_f16_f32(h, b, rb, true);
            return __builtin_bit_cast(uint32_t, h);
        }
    }
};

// FP32 pair words: component 0 in the low, component 1 in the high 32 bits
// (stored as they are, rounded to nearest by the collision's arithmetic).
template <>
struct PairCodec<F32> {
    static __device__ __forceinline__ float lo(u32x2 v) { return __uint_as_float(v.x); }
    static __device__ __forceinline__ float hi(u32x2 v) { return __uint_as_float(v.y); }
    template <int H>
    static __device__ __forceinline__ float sum(u32x2 x, u32x2 y)
    {
        return H == 0 ? lo(x) + lo(y) : hi(x) + hi(y);
    }
    template <int H>
    static __device__ __forceinline__ float diff(u32x2 x, u32x2 y)
    {
        return H == 0 ? lo(x) - lo(y) : hi(x) - hi(y);
    }
    static __device__ __forceinline__ u32x2 enc(float a, float b)
    {
        u32x2 w;
        w.x = __float_as_uint(a);
        w.y = __float_as_uint(b);
        return w;
    }
};

// Word of the pair layout: both components of one (cell, direction), 32 bits
// for the 16-bit formats, 64 bits for FP32.
template <typename ST>
struct PairWordOf {
    using W = uint32_t;
};
template <>
struct PairWordOf<F32> {
    using W = u32x2;
};

template <typename W>
__device__ __forceinline__ W word_load(rsrc_t r, uint32_t vo, uint32_t so)
{
    if constexpr (sizeof(W) == 8) return __builtin_bit_cast(W, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
    else return __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0);
}

// store of one stored value or word of 2, 4 or 8 bytes with cache policy AUX
template <int AUX, typename V>
__device__ __forceinline__ void raw_store(V v, rsrc_t r, uint32_t vo, uint32_t so)
{
    if constexpr (sizeof(V) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, vo, so, AUX);
    else if constexpr (sizeof(V) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, vo, so, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b16(v, r, vo, so, AUX);
}

// Bounds of the split sweep's tiles: cells (a thread per cell and component) and
// rows.  FP64 with two components takes half the cells to stay within the
// register file without spills.
constexpr int split_cells(bool f64, int ncomp) { return f64 && ncomp == 2 ? 256 : 512; }
constexpr int split_rows(bool f64, int ncomp, int c_ns)
{
    return ncomp == 1 ? 16 : (f64 ? 5 : (c_ns == 1 ? 10 : 8));
}

// Blocks of both sweeps in domains of at most kThinRows rows: with rows of up to
// 64 cells a tile there has at most kThinCells, so a larger block would idle, and
// mostly two of these fit a CU.  us a step, 512 cells / 256: 40000 x 4 x 1 in FP16 17 / 11,
// 400 x 4 x 400 in FP16 52 / 41 and with the GS-WBS in FP32 74 / 61, 300 x 3 x 300 in
// FP16 29 / 23; with five to seven rows 512 are the faster ones (30000 x 7 x 1 in
// FP32 8 / 11).
constexpr int kThinRows = 4, kThinCells = 256;

// Kernel parameters in the arithmetic type.
template <typename T>
struct Args {
    int nx, ny, nz;
    int plane;   // nx * ny
    int64_t N;   // cells
    int pair;    // populations in the pair layout
    int zchunk, ntx, nty, nzc;
    int tw, th;  // tile of the sweep
    T inv_tau[2], tau[2];
    T G_s, Gads_s[2];
    T F[3];
    T rho0[2];
    T scale, inv_scale;
    T guo[2];    // 1 - 1/(2 tau): weight of the Guo forcing term (GS-WBS)
    int sr;      // stochastic rounding of stored values
    uint32_t t;  // time step of the state read by the launch (single-domain launches)
    int n_res;
    int res_axis[kMaxRes], res_lo[kMaxRes], res_hi[kMaxRes];
    T res_dr[kMaxRes][2];  // rho_res - rho0, shifted density of the reservoir
};

template <typename T>
static Args<T> make_args(const Problem& p)
{
    Args<T> a{};
    a.nx = p.nx; a.ny = p.ny; a.nz = p.nz;
    a.plane = p.nx * p.ny;
    a.N = p.N;
    a.pair = pair_layout(p.storage, p.ncomp, p.forcing) ? 1 : 0;
    for (int s = 0; s < 2; ++s) {
        a.tau[s] = static_cast<T>(p.tau[s]);
        a.inv_tau[s] = static_cast<T>(1.0 / p.tau[s]);
        a.guo[s] = static_cast<T>(1.0 - 0.5 / p.tau[s]);
        a.Gads_s[s] = static_cast<T>(p.Gads_s[s]);
        a.rho0[s] = static_cast<T>(p.rho0[s]);
    }
    a.G_s = static_cast<T>(p.G_s);
    for (int d = 0; d < 3; ++d) a.F[d] = static_cast<T>(p.F[d]);
    a.scale = static_cast<T>(p.scale);
    a.inv_scale = static_cast<T>(1.0 / p.scale);
    a.sr = p.stochastic;
    a.t = 0;
    a.n_res = p.n_res;
    for (int r = 0; r < kMaxRes; ++r) {
        a.res_axis[r] = p.res_axis[r];
        a.res_lo[r] = p.res_lo[r];
        a.res_hi[r] = p.res_hi[r];
        for (int s = 0; s < 2; ++s) a.res_dr[r][s] = static_cast<T>(p.res_rho[r][s] - p.rho0[s]);
    }
    return a;
}

// Element index of population (component s, direction i) of in-plane cell n of
// plane z, in either layout (auxiliary kernels; the step kernels address whole
// plane blocks through buffer descriptors).
template <typename T>
__device__ __forceinline__ size_t pidx(const Args<T>& a, int s, int i, int z, int64_t n)
{
    if (a.pair) return (((static_cast<size_t>(z) * kQ + i) * static_cast<size_t>(a.plane) + n) << 1) + s;
    return ((static_cast<size_t>(s) * a.nz + z) * kQ + i) * static_cast<size_t>(a.plane) + n;
}

template <typename T>
__device__ __forceinline__ int reservoir_of(const Args<T>& a, int x, int y, int z)
{
    int r_found = -1;
    for (int r = 0; r < kMaxRes; ++r) {
        if (r >= a.n_res) break;
        const int c = a.res_axis[r] == 0 ? x : (a.res_axis[r] == 1 ? y : z);
        if (r_found < 0 && c >= a.res_lo[r] && c < a.res_hi[r]) r_found = r;
    }
    return r_found;
}

// The same search for the step kernel, returning the shifted density of
// component s in that reservoir.  The loop runs over the slots with
// compile-time indices and s is the same for the whole wave, so every
// parameter is read with scalar loads (a per-lane indexed load would be a
// vector memory load, and waiting for it would wait for every load issued
// before it).
template <typename T>
__device__ __forceinline__ bool reservoir_dr(const Args<T>& a, int s, int x, int y, int z, T& dr)
{
    bool in = false;
    dr = T(0);
#pragma unroll
    for (int r = 0; r < kMaxRes; ++r) {
        if (r < a.n_res) {
            const int c = a.res_axis[r] == 0 ? x : (a.res_axis[r] == 1 ? y : z);
            const bool hit = !in && c >= a.res_lo[r] && c < a.res_hi[r];
            dr = hit ? (s == 0 ? a.res_dr[r][0] : a.res_dr[r][1]) : dr;
            in = in || hit;
        }
    }
    return in;
}

// Reservoir membership as bit masks (pair kernel): bit r is set when the cell
// lies in slot r.  Slots along x or y depend on the cell's column only, so a
// thread computes their bits once; slots along z depend on the plane only, the
// same for the whole block.  The lowest set bit is the slot that applies
// (slots are searched in order, as in reservoir_dr).
template <typename T>
__device__ __forceinline__ uint32_t reservoir_xy_bits(const Args<T>& a, int x, int y)
{
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < kMaxRes; ++r) {
        const int c = a.res_axis[r] == 0 ? x : y;
        if (r < a.n_res && a.res_axis[r] != 2 && c >= a.res_lo[r] && c < a.res_hi[r]) m |= 1u << r;
    }
    return m;
}

template <typename T>
__device__ __forceinline__ uint32_t reservoir_z_bits(const Args<T>& a, int z)
{
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < kMaxRes; ++r)
        if (r < a.n_res && a.res_axis[r] == 2 && z >= a.res_lo[r] && z < a.res_hi[r]) m |= 1u << r;
    return m;
}

// shifted densities of the slot of the lowest bit of m (m != 0)
template <typename T>
__device__ __forceinline__ void reservoir_pick(const Args<T>& a, uint32_t m, T& dr0, T& dr1)
{
    dr0 = a.res_dr[kMaxRes - 1][0];
    dr1 = a.res_dr[kMaxRes - 1][1];
#pragma unroll
    for (int r = kMaxRes - 2; r >= 0; --r) {
        const bool hit = (m >> r) & 1u;
        dr0 = hit ? a.res_dr[r][0] : dr0;
        dr1 = hit ? a.res_dr[r][1] : dr1;
    }
}

// XCD-aware tile order: blocks are dispatched round-robin over the 8 XCDs, each
// with an L2 of its own, so every XCD gets a contiguous run of the nb tiles
// (neighbouring tiles re-read each other's edge cells).  Runs differ by one
// tile where nb is no multiple of 8.
__device__ __forceinline__ int xcd_tile(int b, int nb)
{
    const int k = b & 7, q = nb >> 3, r = nb & 7;
    return k * q + min(k, r) + (b >> 3);
}

// The same for sweeps whose blocks run in rounds of `resident`: the runs are
// those of each round, so that one round covers one stretch of the domain.
__device__ __forceinline__ int xcd_tile(int b, int nb, int resident)
{
    const int base = b / resident * resident;
    return base + xcd_tile(b - base, min(resident, nb - base));
}

__device__ __forceinline__ int wrap_dec(int v, int n) { return v == 0 ? n - 1 : v - 1; }
__device__ __forceinline__ int wrap_inc(int v, int n) { return v == n - 1 ? 0 : v + 1; }

// In-plane byte offsets of the nine (x - cx, y - cy) sources of a cell, for
// elements of EB bytes.
struct PlaneOffs {
    uint32_t o[3][3];  // [cy + 1][cx + 1]
};

template <int EB>
__device__ __forceinline__ PlaneOffs plane_offs(int x, int y, int nx, int ny)
{
    const int xs[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};  // x - c, c = -1, 0, 1
    const int ys[3] = {y == ny - 1 ? 0 : y + 1, y, y == 0 ? ny - 1 : y - 1};
    PlaneOffs q;
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) q.o[b][a] = static_cast<uint32_t>(ys[b] * nx + xs[a]) * static_cast<uint32_t>(EB);
    return q;
}

// Pull loads of one cell (raw stored values): direction i comes from the
// source plane z - c_iz, whose block descriptor is r3[c_iz + 1], at the
// in-plane offset of (x - c_ix, y - c_iy) plus i direction strides.
template <typename ST>
__device__ __forceinline__ void pull_raw(const rsrc_t r3[3], uint32_t dir_bytes, const PlaneOffs& q,
                                         typename ST::E e[kQ])
{
#pragma unroll
    for (int i = 0; i < kQ; ++i)
        e[i] = ST::bld(r3[CZ[i] + 1], q.o[CY[i] + 1][CX[i] + 1], static_cast<uint32_t>(i) * dir_bytes);
}

template <typename T>
__device__ __forceinline__ T sum19(const T h[kQ])
{
    T acc = h[0];
#pragma unroll
    for (int i = 1; i <= 9; ++i) acc += h[i] + h[i + 9];
    return acc;
}

// sum_i sign(c_ia) v_i over the directions with c_ia != 0, paired i / i+9
template <typename T, int AX>
__device__ __forceinline__ T first_moment(const T h[kQ])
{
    T acc = T(0);
#pragma unroll
    for (int i = 1; i <= 9; ++i) {
        const int c = AX == 0 ? CX[i] : (AX == 1 ? CY[i] : CZ[i]);
        if (c) acc += c > 0 ? h[i] - h[i + 9] : h[i + 9] - h[i];
    }
    return acc;
}

// Geometry of the staged LDS planes: row stride lw, and stride lp between the
// planes of the two components (or n_s fields).  Compile-time for the sweeps'
// fixed tiles, a run-time row stride for the boxes of the small-domain kernel.
template <int LW, int LP>
struct TileGeom {
    static constexpr int lw = LW, lp = LP;
};
template <int LP>
struct BoxGeom {
    int lw;
    static constexpr int lp = LP;
};

// Neighbour stencil sum_i w_i phi(x + c_i) c_i read from an LDS plane triple.
template <typename T, typename V, typename G>
__device__ __forceinline__ void stencil(const G& geo, const V* pm, const V* p0, const V* pp, int me, T g[3])
{
    // group by weight: axis neighbours (1/18) and diagonals (1/36)
    T ax[3] = {0, 0, 0}, dg[3] = {0, 0, 0};
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
        const V* pl = CZ[i] == 0 ? p0 : (CZ[i] > 0 ? pp : pm);
        const T v = static_cast<T>(pl[me + CY[i] * geo.lw + CX[i]]);
        const bool axis = (CX[i] * CX[i] + CY[i] * CY[i] + CZ[i] * CZ[i]) == 1;
        T* acc = axis ? ax : dg;
        if (CX[i]) acc[0] += CX[i] > 0 ? v : -v;
        if (CY[i]) acc[1] += CY[i] > 0 ? v : -v;
        if (CZ[i]) acc[2] += CZ[i] > 0 ? v : -v;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) g[d] = ax[d] * (T(1) / T(18)) + dg[d] * (T(1) / T(36));
}

// 1/x: correctly rounded in FP64; in FP32 the hardware reciprocal (within
// one unit in the last place), one instruction instead of a division
template <typename T>
__device__ __forceinline__ T recip(T x)
{
    if constexpr (sizeof(T) == 4) return __builtin_amdgcn_rcpf(x);
    else return T(1) / x;
}

// Per-cell physics shared by the step kernels: every kernel evaluates the
// same expressions, so the result of a cell does not depend on which kernel
// or launch shape updated it.

// Equilibrium velocity of component s at one cell, Eq. (SC_u_eq): the common
// velocity sum_c (j_c / tau_c) / sum_c (rho_c / tau_c) plus tau_s F_tot,s /
// rho_s, with F_tot,s the sum of Eqs. (SC_F_inter), (SC_F_ads) and
// (SC_F_ext); no force shift for an absent component.  rho_m/0/p point at the
// LDS density planes z-1, z, z+1 ([NC][LP]), ns_m/0/p at the n_s planes
// ([CNS][LP]); me is the cell's LDS index and jc[c] the first moment of
// component c at the cell.  Also returns the own density and n_s.
template <typename T, int NC, int CNS, typename G>
__device__ __forceinline__ void cell_velocity(const G& geo, const Args<T>& a, int s, int me, const T* rho_m,
                                              const T* rho_0, const T* rho_p, const float* ns_m, const float* ns_0,
                                              const float* ns_p, const T (&jc)[NC][3], T ueq[3], T& rho_own, T& n)
{
    T rho = 0, den = 0, num[3] = {0, 0, 0};
    rho_own = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const T rc = rho_0[c * geo.lp + me];
        if (c == s) rho_own = rc;
        rho += rc;
        den += rc * a.inv_tau[c];
#pragma unroll
        for (int d = 0; d < 3; ++d) num[d] += jc[c][d] * a.inv_tau[c];
    }
    const T inv_den = den > T(0) ? recip(den) : T(0);
    const T inv_rho = rho > T(0) ? recip(rho) : T(0);
    const int cn = CNS == 2 ? s : 0;
    T ga[3];
    stencil<T, float>(geo, ns_m + cn * geo.lp, ns_0 + cn * geo.lp, ns_p + cn * geo.lp, me, ga);
    T gi[3] = {0, 0, 0};
    if constexpr (NC == 2)
        stencil<T, T>(geo, rho_m + (1 - s) * geo.lp, rho_0 + (1 - s) * geo.lp, rho_p + (1 - s) * geo.lp, me, gi);
    const bool present = rho_own > T(0);
    const T tau_s = a.tau[s], Gads = a.Gads_s[s];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const T acc = -a.G_s * gi[d] - Gads * ga[d] + a.F[d] * inv_rho;
        ueq[d] = num[d] * inv_den + (present ? tau_s * acc : T(0));
    }
    n = static_cast<T>(ns_0[cn * geo.lp + me]);
}

// The GS-WBS of Eq. (GS-WBS) takes its equilibrium at u_macro of
// Eq. (HMCSC_u_macro), common to the components: sum_c (1 - n_c)(j_c +
// F_tot,c / 2) / rho.  That needs the total force of every component at the
// cell (both cohesion stencils); returns u_macro, the own total force, the own
// density and n_s.
template <typename T, int NC, int CNS, typename G>
__device__ __forceinline__ void cell_velocity_guo(const G& geo, const Args<T>& a, int s, int me, const T* rho_m,
                                                  const T* rho_0, const T* rho_p, const float* ns_m,
                                                  const float* ns_0, const float* ns_p, const T (&jc)[NC][3],
                                                  T um[3], T fo[3], T& rho_own, T& n_own)
{
    T rc[NC], rho = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        rc[c] = rho_0[c * geo.lp + me];
        rho += rc[c];
    }
    const T inv_rho = rho > T(0) ? recip(rho) : T(0);
    T m[3] = {0, 0, 0};
    T ga[3];
    if constexpr (CNS == 1) stencil<T, float>(geo, ns_m, ns_0, ns_p, me, ga);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int cn = CNS == 2 ? c : 0;
        if constexpr (CNS == 2)
            stencil<T, float>(geo, ns_m + cn * geo.lp, ns_0 + cn * geo.lp, ns_p + cn * geo.lp, me, ga);
        T gi[3] = {0, 0, 0};
        if constexpr (NC == 2)
            stencil<T, T>(geo, rho_m + (1 - c) * geo.lp, rho_0 + (1 - c) * geo.lp, rho_p + (1 - c) * geo.lp, me, gi);
        const T nc = static_cast<T>(ns_0[cn * geo.lp + me]);
        T F[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            F[d] = rc[c] * (-a.G_s * gi[d] - a.Gads_s[c] * ga[d] + a.F[d] * inv_rho);
            m[d] += (T(1) - nc) * (jc[c][d] + T(0.5) * F[d]);
        }
        if (c == s) {
#pragma unroll
            for (int d = 0; d < 3; ++d) fo[d] = F[d];
            rho_own = rc[c];
            n_own = nc;
        }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) um[d] = m[d] * inv_rho;
}

// Force-shifted BGK collision blended with partial bounce-back, Eq. (LGS), in
// the shifted variables: post_i = (1-n)(h_i - (h_i - h^eq_i)/tau_s) + n h_ibar
// with h^eq from Eq. (Maxwell) at u_eq (the w_i rho0 shift cancels because
// w_ibar = w_i).  relax_coef gathers the per-cell factors, relax_dir gives the
// results of one direction pair (i, i+9), relax_rest that of direction 0.
template <typename T>
struct RelaxCoef {
    T ca, n;                  // weights of h_i and h_ibar
    T K0[3], K1[3], K2[3];    // weight of h^eq_i: K0 + K1 c.u + K2 (c.u)^2 per weight class
    T u[3];
};

template <typename T>
__device__ __forceinline__ RelaxCoef<T> relax_coef(const Args<T>& a, int s, T rho_own, const T ueq[3], T n)
{
    RelaxCoef<T> k;
    const T uu = ueq[0] * ueq[0] + ueq[1] * ueq[1] + ueq[2] * ueq[2];
    const T omn = T(1) - n;
    const T cb = omn * a.inv_tau[s];  // weight of h^eq
    k.ca = omn - cb;                  // weight of h
    k.n = n;
    const T base0 = (rho_own - a.rho0[s]) - T(1.5) * rho_own * uu;
    const T r3 = T(3) * rho_own, r45 = T(4.5) * rho_own;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const T wk = cb * (c == 0 ? T(1) / T(3) : (c == 1 ? T(1) / T(18) : T(1) / T(36)));
        k.K0[c] = wk * base0;
        k.K1[c] = wk * r3;
        k.K2[c] = wk * r45;
        k.u[c] = ueq[c];
    }
    return k;
}

template <typename T>
__device__ __forceinline__ T relax_rest(const RelaxCoef<T>& k, T h0)
{
    return k.ca * h0 + k.n * h0 + k.K0[0];
}

// i in 1..9: hi = h_i, ho = h_{i+9}
template <typename T>
__device__ __forceinline__ void relax_dir(const RelaxCoef<T>& k, int i, T hi, T ho, T& post_i, T& post_o)
{
    const int c = (CX[i] * CX[i] + CY[i] * CY[i] + CZ[i] * CZ[i]) == 1 ? 1 : 2;
    T cu = T(0);
    if (CX[i]) cu += CX[i] > 0 ? k.u[0] : -k.u[0];
    if (CY[i]) cu += CY[i] > 0 ? k.u[1] : -k.u[1];
    if (CZ[i]) cu += CZ[i] > 0 ? k.u[2] : -k.u[2];
    const T t = k.K2[c] * (cu * cu) + k.K0[c];
    const T e = k.K1[c] * cu;
    post_i = k.ca * hi + (k.n * ho + (t + e));
    post_o = k.ca * ho + (k.n * hi + (t - e));
}

// The forcing term of Guo, Zheng and Shi (2002), weighted by (1 - n_s) as in
// Eq. (GS-WBS): F_i = A w_i [3 (c_i - u).F + 9 (c_i.u)(c_i.F)] with
// A = (1 - n)(1 - 1/(2 tau)).  For a pair (i, ibar) the part even in c_i,
// A w (9 cu cF - 3 u.F), adds to both, the odd part A w 3 cF with opposite
// signs, as in relax_dir.
template <typename T>
struct GuoCoef {
    T gw[3];   // A w per weight class
    T f[3];    // F_tot of the component
    T uF;
};

template <typename T>
__device__ __forceinline__ GuoCoef<T> guo_coef(const Args<T>& a, int s, T n, const T F[3], const T u[3])
{
    GuoCoef<T> g;
    const T A = (T(1) - n) * a.guo[s];
#pragma unroll
    for (int c = 0; c < 3; ++c) g.gw[c] = A * (c == 0 ? T(1) / T(3) : (c == 1 ? T(1) / T(18) : T(1) / T(36)));
#pragma unroll
    for (int d = 0; d < 3; ++d) g.f[d] = F[d];
    g.uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2];
    return g;
}

template <typename T>
__device__ __forceinline__ T relax_rest_guo(const RelaxCoef<T>& k, const GuoCoef<T>& g, T h0)
{
    return k.ca * h0 + k.n * h0 + (k.K0[0] + g.gw[0] * (T(-3) * g.uF));
}

template <typename T>
__device__ __forceinline__ void relax_dir_guo(const RelaxCoef<T>& k, const GuoCoef<T>& g, int i, T hi, T ho,
                                              T& post_i, T& post_o)
{
    const int c = (CX[i] * CX[i] + CY[i] * CY[i] + CZ[i] * CZ[i]) == 1 ? 1 : 2;
    T cu = T(0), cF = T(0);
    if (CX[i]) { cu += CX[i] > 0 ? k.u[0] : -k.u[0]; cF += CX[i] > 0 ? g.f[0] : -g.f[0]; }
    if (CY[i]) { cu += CY[i] > 0 ? k.u[1] : -k.u[1]; cF += CY[i] > 0 ? g.f[1] : -g.f[1]; }
    if (CZ[i]) { cu += CZ[i] > 0 ? k.u[2] : -k.u[2]; cF += CZ[i] > 0 ? g.f[2] : -g.f[2]; }
    const T t = k.K2[c] * (cu * cu) + k.K0[c] + g.gw[c] * (T(9) * (cu * cF) - T(3) * g.uF);
    const T e = k.K1[c] * cu + g.gw[c] * (T(3) * cF);
    post_i = k.ca * hi + (k.n * ho + (t + e));
    post_o = k.ca * ho + (k.n * hi + (t - e));
}

// Both components of one cell (pair kernel): the equilibrium velocities of
// Eq. (SC_u_eq) for s = 0 and 1, with the same expressions, in the same order,
// as cell_velocity evaluates for each component, so a cell's result does not
// depend on which kernel updated it.  The adhesion stencil of a single n_s
// field is shared by the two components.
template <int CNS, typename G>
__device__ __forceinline__ void cell_velocity_pair(const G& geo, const Args<float>& a, int me, const float* rho_m,
                                                   const float* rho_0, const float* rho_p, const float* ns_m,
                                                   const float* ns_0, const float* ns_p, const float (&jc)[2][3],
                                                   float ueq[2][3], float rho_own[2], float n[2])
{
    using T = float;
    T rho = 0, den = 0, num[3] = {0, 0, 0};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const T rc = rho_0[c * geo.lp + me];
        rho_own[c] = rc;
        rho += rc;
        den += rc * a.inv_tau[c];
#pragma unroll
        for (int d = 0; d < 3; ++d) num[d] += jc[c][d] * a.inv_tau[c];
    }
    const T inv_den = den > T(0) ? recip(den) : T(0);
    const T inv_rho = rho > T(0) ? recip(rho) : T(0);
    // one stencil at a time (a scheduling fence after each): all 54 or 72
    // neighbour reads in flight at once would need as many registers
    T ga[CNS][3];
#pragma unroll
    for (int cn = 0; cn < CNS; ++cn) {
        stencil<T, float>(geo, ns_m + cn * geo.lp, ns_0 + cn * geo.lp, ns_p + cn * geo.lp, me, ga[cn]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int cn = CNS == 2 ? s : 0;
        T gi[3];
        stencil<T, T>(geo, rho_m + (1 - s) * geo.lp, rho_0 + (1 - s) * geo.lp, rho_p + (1 - s) * geo.lp, me, gi);
        __builtin_amdgcn_sched_barrier(0);
        const bool present = rho_own[s] > T(0);
        const T tau_s = a.tau[s], Gads = a.Gads_s[s];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const T acc = -a.G_s * gi[d] - Gads * ga[cn][d] + a.F[d] * inv_rho;
            ueq[s][d] = num[d] * inv_den + (present ? tau_s * acc : T(0));
        }
        n[s] = static_cast<T>(ns_0[cn * geo.lp + me]);
    }
}

// The GS-WBS for both components of one cell: u_macro of Eq. (HMCSC_u_macro)
// and each component's total force, as cell_velocity_guo computes them.
template <int CNS, typename G>
__device__ __forceinline__ void cell_velocity_guo_pair(const G& geo, const Args<float>& a, int me, const float* rho_m,
                                                       const float* rho_0, const float* rho_p, const float* ns_m,
                                                       const float* ns_0, const float* ns_p,
                                                       const float (&jc)[2][3], float um[3], float fo[2][3],
                                                       float rho_own[2], float n_own[2])
{
    using T = float;
    T rc[2], rho = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        rc[c] = rho_0[c * geo.lp + me];
        rho += rc[c];
    }
    const T inv_rho = rho > T(0) ? recip(rho) : T(0);
    T m[3] = {0, 0, 0};
    T ga[3];
    if constexpr (CNS == 1) stencil<T, float>(geo, ns_m, ns_0, ns_p, me, ga);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int cn = CNS == 2 ? c : 0;
        if constexpr (CNS == 2)
            stencil<T, float>(geo, ns_m + cn * geo.lp, ns_0 + cn * geo.lp, ns_p + cn * geo.lp, me, ga);
        T gi[3];
        stencil<T, T>(geo, rho_m + (1 - c) * geo.lp, rho_0 + (1 - c) * geo.lp, rho_p + (1 - c) * geo.lp, me, gi);
        const T nc = static_cast<T>(ns_0[cn * geo.lp + me]);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            fo[c][d] = rc[c] * (-a.G_s * gi[d] - a.Gads_s[c] * ga[d] + a.F[d] * inv_rho);
            m[d] += (T(1) - nc) * (jc[c][d] + T(0.5) * fo[c][d]);
        }
        rho_own[c] = rc[c];
        n_own[c] = nc;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) um[d] = m[d] * inv_rho;
}

// Densities rho_0, rho_1 of a cell of the pair layout from its raw words, and
// its first moments (Eq. mom_BGK) when j is given; a reservoir cell (rbits its
// reservoir bits) has the Dirichlet density instead, summed in the same order
// over the rest populations w_i dr (computed only when a lane of the wave is
// in a reservoir), and first moments 0 (w_i = w_ibar).  The words are decoded
// into the running sums, never held as 38 floats.
template <typename ST>
__device__ __forceinline__ void pair_moments(const Args<float>& a, uint32_t rbits,
                                             const typename PairWordOf<ST>::W e[kQ], float& r0, float& r1, float* j)
{
    using T = float;
    using PC = PairCodec<ST>;
    T s0 = PC::lo(e[0]), s1 = PC::hi(e[0]);
    T j0[3] = {T(0), T(0), T(0)}, j1[3] = {T(0), T(0), T(0)};
#pragma unroll
    for (int i = 1; i <= 9; ++i) {
        // sums and differences of opposite populations, each rounded once
        // (b - a is exactly -(a - b), so the sign goes into the update)
        const T p0 = PC::template sum<0>(e[i], e[i + 9]), p1 = PC::template sum<1>(e[i], e[i + 9]);
        s0 += p0;
        s1 += p1;
        if (j) {
            const T d0 = PC::template diff<0>(e[i], e[i + 9]), d1 = PC::template diff<1>(e[i], e[i + 9]);
            if (CX[i]) { j0[0] = CX[i] > 0 ? j0[0] + d0 : j0[0] - d0; j1[0] = CX[i] > 0 ? j1[0] + d1 : j1[0] - d1; }
            if (CY[i]) { j0[1] = CY[i] > 0 ? j0[1] + d0 : j0[1] - d0; j1[1] = CY[i] > 0 ? j1[1] + d1 : j1[1] - d1; }
            if (CZ[i]) { j0[2] = CZ[i] > 0 ? j0[2] + d0 : j0[2] - d0; j1[2] = CZ[i] > 0 ? j1[2] + d1 : j1[2] - d1; }
        }
    }
    s0 *= a.inv_scale;
    s1 *= a.inv_scale;
    if (j) {
        const bool in = rbits != 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            j[d] = in ? T(0) : j0[d] * a.inv_scale;
            j[3 + d] = in ? T(0) : j1[d] * a.inv_scale;
        }
    }
    const bool in = rbits != 0;
    if (__builtin_amdgcn_ballot_w64(in) != 0) {
        T dr0, dr1;
        reservoir_pick(a, rbits, dr0, dr1);
        T w0 = wgt<T>(0) * dr0, w1 = wgt<T>(0) * dr1;
#pragma unroll
        for (int i = 1; i <= 9; ++i) {
            w0 += wgt<T>(i) * dr0 + wgt<T>(i + 9) * dr0;
            w1 += wgt<T>(i) * dr1 + wgt<T>(i + 9) * dr1;
        }
        s0 = in ? w0 : s0;
        s1 = in ? w1 : s1;
    }
    r0 = a.rho0[0] + s0;
    r1 = a.rho0[1] + s1;
}

// Rounding of the stored words: kRoundNearest and kRoundStochastic fix it at
// compile time; kRoundEither follows the domain's flag without a branch
// (both roundings computed and one selected), so that the stores of a
// collision form one straight sequence (after a branch between two store
// sequences the compiler's wait counts lose track of how many stores were
// issued, and its waits for the next plane's loads then wait for the
// stores as well).
constexpr int kRoundNearest = 0, kRoundStochastic = 1, kRoundEither = 2;

// Collision of one cell of the pair layout, both components: rbits its
// reservoir bits, cell its index n (keys the stochastic rounding with t_key),
// rho_m/0/p and ns_m/0/p the staged planes z-1, z, z+1 with the cell at me, jm
// its first moments.  wd(i) gives the raw word of direction i; the words are
// decoded where they are used (twice: first moments, then the relaxation)
// rather than held as 38 floats.  store(i, w) takes the 19 results, in the
// order 0, 1, 10, 2, 11, ...
template <typename ST, int CNS, int FS, int RND, typename G, typename WD, typename STORE>
__device__ __forceinline__ void pair_collide(const G& geo, const Args<float>& a, uint32_t rbits, uint32_t t_key,
                                             uint32_t cell, int me, const float* rho_m, const float* rho_0,
                                             const float* rho_p, const float* ns_m, const float* ns_0,
                                             const float* ns_p, const float (&jm)[6], WD&& wd, STORE&& store)
{
    using T = float;
    using W = typename PairWordOf<ST>::W;
    using PC = PairCodec<ST>;
    const bool in = rbits != 0;
    T dr0, dr1;
    reservoir_pick(a, rbits, dr0, dr1);
    // populations on the stored scale: h_i * 2^k
    const T ds0 = dr0 * a.scale, ds1 = dr1 * a.scale;
    // (the word is read unconditionally: a conditional operator around
    // the read would become a branch per value)
    auto h0 = [&](int i) {
        const T v = PC::lo(wd(i));
        return in ? wgt<T>(i) * ds0 : v;
    };
    auto h1 = [&](int i) {
        const T v = PC::hi(wd(i));
        return in ? wgt<T>(i) * ds1 : v;
    };
    const T jc[2][3] = {{jm[0], jm[1], jm[2]}, {jm[3], jm[4], jm[5]}};
    T ueq[2][3], rho_own[2], n[2], fo[2][3];
    if constexpr (FS == kForcingGuo) {
        T um[3];
        cell_velocity_guo_pair<CNS>(geo, a, me, rho_m, rho_0, rho_p, ns_m, ns_0, ns_p, jc, um, fo, rho_own, n);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int d = 0; d < 3; ++d) ueq[c][d] = um[d];
    } else {
        cell_velocity_pair<CNS>(geo, a, me, rho_m, rho_0, rho_p, ns_m, ns_0, ns_p, jc, ueq, rho_own, n);
    }
    RelaxCoef<T> k0 = relax_coef<T>(a, 0, rho_own[0], ueq[0], n[0]);
    RelaxCoef<T> k1 = relax_coef<T>(a, 1, rho_own[1], ueq[1], n[1]);
    GuoCoef<T> g0{}, g1{};
    if constexpr (FS == kForcingGuo) {
        g0 = guo_coef<T>(a, 0, n[0], fo[0], ueq[0]);
        g1 = guo_coef<T>(a, 1, n[1], fo[1], ueq[1]);
    }
    // the terms not proportional to h go to the stored scale
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        k0.K0[c] *= a.scale; k0.K1[c] *= a.scale; k0.K2[c] *= a.scale;
        k1.K0[c] *= a.scale; k1.K1[c] *= a.scale; k1.K2[c] *= a.scale;
        g0.gw[c] *= a.scale; g1.gw[c] *= a.scale;
    }
    auto rest = [&](const RelaxCoef<T>& k, const GuoCoef<T>& g, T h) {
        if constexpr (FS == kForcingGuo) return relax_rest_guo(k, g, h);
        else return relax_rest(k, h);
    };
    auto pairdir = [&](const RelaxCoef<T>& k, const GuoCoef<T>& g, int i, T hi_, T ho_, T& pi, T& po) {
        if constexpr (FS == kForcingGuo) relax_dir_guo(k, g, i, hi_, ho_, pi, po);
        else relax_dir(k, i, hi_, ho_, pi, po);
    };
    // the random streams of the split kernels: per (cell, component)
    // fmix32 of the counter, then one lcg24 step per stored value
    uint32_t r0 = 0, r1 = 0;
    if constexpr (RND != kRoundNearest) {
        r0 = fmix32(t_key ^ (2u * cell));
        r1 = fmix32(t_key ^ (2u * cell + 1u));
    }
    const uint32_t sr_mask = RND == kRoundEither ? 0u - static_cast<uint32_t>(a.sr != 0) : 0u;
    auto word = [&](T v0, T v1, uint32_t ra, uint32_t rb) -> W {
        if constexpr (RND == kRoundStochastic) return PC::enc_sr(v0, v1, ra, rb);
        else if constexpr (RND == kRoundNearest) return PC::enc(v0, v1);
        else return (PC::enc_sr(v0, v1, ra, rb) & sr_mask) | (PC::enc(v0, v1) & ~sr_mask);
    };
    store(0, word(rest(k0, g0, h0(0)), rest(k1, g1, h1(0)), r0, r1));
#pragma unroll
    for (int i = 1; i <= 9; ++i) {
        T pi0, po0, pi1, po1;
        pairdir(k0, g0, i, h0(i), h0(i + 9), pi0, po0);
        pairdir(k1, g1, i, h1(i), h1(i + 9), pi1, po1);
        uint32_t ri0 = 0, ri1 = 0;
        if constexpr (RND != kRoundNearest) {
            ri0 = lcg24(r0);
            ri1 = lcg24(r1);
            r0 = lcg24(ri0);
            r1 = lcg24(ri1);
        }
        store(i, word(pi0, pi1, ri0, ri1));
        store(i + 9, word(po0, po1, r0, r1));
    }
}

// Collision of one component of one cell (split layout), from its
// pre-collision populations h and the staged planes, as pair_collide; jc holds
// the first moments of every component at the cell.
template <typename ST, int NC, int CNS, int FS, typename G, typename STORE>
__device__ __forceinline__ void split_collide(const G& geo, const Args<typename ST::T>& a, int s, uint32_t t_key,
                                              uint32_t cell, int me, const typename ST::T* rho_m,
                                              const typename ST::T* rho_0, const typename ST::T* rho_p,
                                              const float* ns_m, const float* ns_0, const float* ns_p,
                                              const typename ST::T (&jc)[NC][3], const typename ST::T* h,
                                              STORE&& store)
{
    using T = typename ST::T;
    T ueq[3], rho_own, n, fo[3];
    if constexpr (FS == kForcingGuo)
        cell_velocity_guo<T, NC, CNS>(geo, a, s, me, rho_m, rho_0, rho_p, ns_m, ns_0, ns_p, jc, ueq, fo, rho_own, n);
    else
        cell_velocity<T, NC, CNS>(geo, a, s, me, rho_m, rho_0, rho_p, ns_m, ns_0, ns_p, jc, ueq, rho_own, n);
    const RelaxCoef<T> k = relax_coef<T>(a, s, rho_own, ueq, n);
    GuoCoef<T> g{};
    if constexpr (FS == kForcingGuo) g = guo_coef<T>(a, s, n, fo, ueq);
    auto rest = [&]() {
        if constexpr (FS == kForcingGuo) return relax_rest_guo(k, g, h[0]);
        else return relax_rest(k, h[0]);
    };
    auto pair = [&](int i, T& pi, T& po) {
        if constexpr (FS == kForcingGuo) relax_dir_guo(k, g, i, h[i], h[i + 9], pi, po);
        else relax_dir(k, i, h[i], h[i + 9], pi, po);
    };
    if (a.sr) {
        // one random word per stored value: fmix32 of (cell, component,
        // time step) for the rest population, then lcg24 steps in the
        // order of the stores
        uint32_t r = fmix32(t_key ^ (2u * cell + static_cast<uint32_t>(s)));
        store(0, ST::enc_sr(rest(), a.scale, r));
#pragma unroll
        for (int i = 1; i <= 9; ++i) {
            T pi, po;
            pair(i, pi, po);
            r = lcg24(r);
            store(i, ST::enc_sr(pi, a.scale, r));
            r = lcg24(r);
            store(i + 9, ST::enc_sr(po, a.scale, r));
        }
    } else {
        store(0, ST::enc(rest(), a.scale));
#pragma unroll
        for (int i = 1; i <= 9; ++i) {
            T pi, po;
            pair(i, pi, po);
            store(i, ST::enc(pi, a.scale));
            store(i + 9, ST::enc(po, a.scale));
        }
    }
}

// Two components in FP32 or a 16-bit format use the pair layout and kernel,
// except FP32 with the GS-WBS: its collision, with both components' Guo
// terms, needs more registers than the FP32 pair sweep leaves (it spilled and
// ran 4.6 % slower than in the split layout).
template <typename ST, int NC, int FS = kForcingShanChen>
constexpr bool kPair =
    (sizeof(typename ST::E) == 2 || (std::is_same_v<ST, F32> && FS != kForcingGuo)) && NC == 2;

}  // namespace hm
