// lgf_device.hpp -- device-side building blocks of the gfx950 gauge-fixing
// kernels: complex 3x3 algebra in registers, the storage formats and their
// parity-split structure-of-arrays layout, lattice geometry, Philox4x32-10.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace lgf {

// ----------------------------------------------------------------------------
// Complex numbers and 3x3 complex matrices held in registers.
// ----------------------------------------------------------------------------

template <typename T> struct cpx { T re, im; };

template <typename T> __device__ __forceinline__ cpx<T> operator+(cpx<T> a, cpx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T> __device__ __forceinline__ cpx<T> operator-(cpx<T> a, cpx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T> __device__ __forceinline__ cpx<T> operator*(cpx<T> a, cpx<T> b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T> __device__ __forceinline__ cpx<T> conj(cpx<T> a) { return {a.re, -a.im}; }
// a * conj(b)
template <typename T> __device__ __forceinline__ cpx<T> mul_conj(cpx<T> a, cpx<T> b)
{
    return {a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im};
}
template <typename T> __device__ __forceinline__ T norm2(cpx<T> a) { return a.re * a.re + a.im * a.im; }

template <typename T> struct mat3 { cpx<T> e[3][3]; };

template <typename T> __device__ __forceinline__ void set_identity(mat3<T> &a)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) a.e[i][j] = {T(i == j ? 1 : 0), T(0)};
}

template <typename T> __device__ __forceinline__ void set_zero(mat3<T> &a)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) a.e[i][j] = {T(0), T(0)};
}

// acc += u + v^dag
template <typename T>
__device__ __forceinline__ void add_fwd_bwd(mat3<T> &acc, const mat3<T> &u, const mat3<T> &v)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            acc.e[i][j].re += u.e[i][j].re + v.e[j][i].re;
            acc.e[i][j].im += u.e[i][j].im - v.e[j][i].im;
        }
}

// row 2 = conj(row0 x row1): the last row of a unitary matrix with det 1
template <typename T> __device__ __forceinline__ void rebuild_row2(mat3<T> &u)
{
    u.e[2][0] = conj(u.e[0][1] * u.e[1][2] - u.e[0][2] * u.e[1][1]);
    u.e[2][1] = conj(u.e[0][2] * u.e[1][0] - u.e[0][0] * u.e[1][2]);
    u.e[2][2] = conj(u.e[0][0] * u.e[1][1] - u.e[0][1] * u.e[1][0]);
}

// r = g * u, rows [0, R) only
template <int R, typename T>
__device__ __forceinline__ void left_mul(mat3<T> &r, const mat3<T> &g, const mat3<T> &u)
{
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            r.e[i][j] = g.e[i][0] * u.e[0][j] + g.e[i][1] * u.e[1][j] + g.e[i][2] * u.e[2][j];
}

// r = u * g^dag, rows [0, R) only
template <int R, typename T>
__device__ __forceinline__ void right_mul_dag(mat3<T> &r, const mat3<T> &u, const mat3<T> &g)
{
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            r.e[i][j] = mul_conj(u.e[i][0], g.e[j][0]) + mul_conj(u.e[i][1], g.e[j][1]) +
                        mul_conj(u.e[i][2], g.e[j][2]);
}

// 1 / sqrt(x) for the SU(2) normalisation, which amplifies rounding errors on
// ill-conditioned sites: FP32 keeps the correctly rounded square root and
// division.  FP64 takes the hardware's estimate y (relative error < 6e-8) and
// one third-order step: with e = 1 - x y^2, 1/sqrt(x) = y (1 - e)^(-1/2)
// = y (1 + e/2 + 3/8 e^2 + O(e^3)), 6 instructions instead of the 26 of a square
// root and a division.  Over 5e8 values in [2^-40, 2^24) its largest error is 1.25
// and its mean 0.40 units of 2^-53, against 1.50 and 0.50 of 1.0 / sqrt(x).
// Outside the range where the step's products stay normal: 1.0 / sqrt(x).
template <typename T> __device__ __forceinline__ T inv_sqrt(T x);
template <> __device__ __forceinline__ float inv_sqrt<float>(float x) { return 1.0f / sqrtf(x); }
template <> __device__ __forceinline__ double inv_sqrt<double>(double x)
{
    if (__builtin_expect(!(x >= 0x1p-960 && x <= 0x1p960), 0)) return 1.0 / sqrt(x);
    const double y = __builtin_amdgcn_rsq(x);
    const double t = x * y;
    const double e = __builtin_fma(-t, y, 1.0);
    const double p = __builtin_fma(0.375, e, 0.5);
    return __builtin_fma(y * e, p, y);
}

// Project a 3x3 matrix onto SU(3) in FP64: normalise row 0, orthogonalise
// and normalise row 1, row 2 = conj(row0 x row1).
__device__ __forceinline__ void reunitarize(mat3<double> &u)
{
    double n0 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) n0 += norm2(u.e[0][k]);
    const double i0 = 1.0 / sqrt(n0);
#pragma unroll
    for (int k = 0; k < 3; ++k) { u.e[0][k].re *= i0; u.e[0][k].im *= i0; }
    cpx<double> d = {0.0, 0.0};  // <row0, row1> = sum_k conj(row0_k) row1_k
#pragma unroll
    for (int k = 0; k < 3; ++k) d = d + conj(u.e[0][k]) * u.e[1][k];
#pragma unroll
    for (int k = 0; k < 3; ++k) u.e[1][k] = u.e[1][k] - d * u.e[0][k];
    double n1 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) n1 += norm2(u.e[1][k]);
    const double i1 = 1.0 / sqrt(n1);
#pragma unroll
    for (int k = 0; k < 3; ++k) { u.e[1][k].re *= i1; u.e[1][k].im *= i1; }
    rebuild_row2(u);
}

template <typename A, typename B>
__device__ __forceinline__ void convert(mat3<B> &dst, const mat3<A> &src)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) dst.e[i][j] = {B(src.e[i][j].re), B(src.e[i][j].im)};
}

// The value of another lane of the same four (quad): lane i of a quad gets the
// value of its lane P_i.  A DPP move inside the vector unit, where a shuffle
// goes through LDS (18 or 36 of them sum one matrix over the lanes of a site).
template <int P0, int P1, int P2, int P3> __device__ __forceinline__ float quad_perm(float v)
{
    constexpr int ctrl = P0 | (P1 << 2) | (P2 << 4) | (P3 << 6);
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xF, 0xF, true));
}
template <int P0, int P1, int P2, int P3> __device__ __forceinline__ double quad_perm(double v)
{
    constexpr int ctrl = P0 | (P1 << 2) | (P2 << 4) | (P3 << 6);
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xF, 0xF, true));
}

// m summed over the LPS (1, 2 or 4) lanes of a site, pairs first
template <int LPS, typename T> __device__ __forceinline__ void lane_sum(mat3<T> &m)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if constexpr (LPS >= 2) {
                m.e[i][j].re += quad_perm<1, 0, 3, 2>(m.e[i][j].re);
                m.e[i][j].im += quad_perm<1, 0, 3, 2>(m.e[i][j].im);
            }
            if constexpr (LPS >= 4) {
                m.e[i][j].re += quad_perm<2, 3, 0, 1>(m.e[i][j].re);
                m.e[i][j].im += quad_perm<2, 3, 0, 1>(m.e[i][j].im);
            }
        }
}

// the value of the even / odd lane of a pair, in both
template <typename T> __device__ __forceinline__ T pair_even(T v) { return quad_perm<0, 0, 2, 2>(v); }
template <typename T> __device__ __forceinline__ T pair_odd(T v) { return quad_perm<1, 1, 3, 3>(v); }

// ----------------------------------------------------------------------------
// Storage formats.  A field is split by parity; within a parity, direction
// and vector slot, the Vh = V/2 sites form one contiguous stream of 8- or
// 16-byte vectors ("planes"), so a wavefront's 64 consecutive sites load
// 512 B - 1 KB contiguous per instruction:
//     vector index = ((parity*4 + mu)*NV + slot)*Vh + h
// A link is stored row-major, (row, column, re/im), rows 0..R-1.
// ----------------------------------------------------------------------------

// kF64_12S: the fixed-link sweep in FP64 with g stored as FP64-12 and the
// read-only links in the split storage below (never a link field's format).
enum : int { kF64_18 = 0, kF32_18 = 1, kF32_12 = 2, kF64_12 = 3, kF64_12S = 4 };

typedef double v2d __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <int F> struct Fmt;
template <> struct Fmt<kF64_18> { using T = double; using V = v2d; static constexpr int R = 3, NV = 9, CPV = 1; };
template <> struct Fmt<kF64_12> { using T = double; using V = v2d; static constexpr int R = 2, NV = 6, CPV = 1; };
template <> struct Fmt<kF32_18> { using T = float;  using V = v2f; static constexpr int R = 3, NV = 9, CPV = 1; };
template <> struct Fmt<kF32_12> { using T = float;  using V = v4f; static constexpr int R = 2, NV = 3, CPV = 2; };
template <> struct Fmt<kF64_12S> : Fmt<kF64_12> {};  // the site field g

// A device pointer that was read from memory (a descriptor's) is generic to the
// compiler, which then emits flat loads: their waits cover LDS and memory
// together, so no two stay in flight across one.  Buffers of the library are
// all global memory; this states it.
template <typename T> __device__ __forceinline__ T *as_global(T *p)
{
    // (through an integer: a plain cast there and back is folded away)
    return (T *)reinterpret_cast<__attribute__((address_space(1))) T *>(reinterpret_cast<uintptr_t>(p));
}

// the same value, of which the compiler knows nothing any more (no instruction)
__device__ __forceinline__ void forget(uint32_t &v) { asm volatile("" : "+v"(v)); }

// what of a link sweep goes past the caches: nothing, loads and stores, stores
constexpr int kCached = 0, kStream = 1, kStreamStores = 2;

// vector load / store, optionally marked non-temporal (streamed past the
// caches: every link is read and written once per half-sweep)
template <bool NT, typename V> __device__ __forceinline__ V vload(const V *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT, typename V> __device__ __forceinline__ void vstore(V *p, V v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// base pointer of the (parity, mu) block
template <int F>
__device__ __forceinline__ typename Fmt<F>::V *block_ptr(void *field, uint32_t Vh, int parity, int mu)
{
    return reinterpret_cast<typename Fmt<F>::V *>(field) +
           (size_t)((parity * 4 + mu) * Fmt<F>::NV) * Vh;
}

// the NV vectors of one link, row-major, into a matrix (rows 0..R-1)
template <int F>
__device__ __forceinline__ void unpack_link(mat3<typename Fmt<F>::T> &u, const typename Fmt<F>::V *v)
{
    using S = Fmt<F>;
    if constexpr (S::CPV == 1) {
#pragma unroll
        for (int k = 0; k < S::NV; ++k) u.e[k / 3][k % 3] = {v[k].x, v[k].y};
    } else {
#pragma unroll
        for (int k = 0; k < S::NV; ++k) {
            u.e[(2 * k) / 3][(2 * k) % 3] = {v[k].x, v[k].y};
            u.e[(2 * k + 1) / 3][(2 * k + 1) % 3] = {v[k].z, v[k].w};
        }
    }
}

// ROW2 = false leaves row 2 of a 12-real link unset (for callers that only
// read rows 0 and 1)
template <int F, bool NT = false, bool ROW2 = true>
__device__ __forceinline__ void load_link(mat3<typename Fmt<F>::T> &u, const typename Fmt<F>::V *blk,
                                          uint32_t Vh, uint32_t h)
{
    using S = Fmt<F>;
    typename S::V v[S::NV];
#pragma unroll
    for (int k = 0; k < S::NV; ++k) v[k] = vload<NT>(blk + (size_t)k * Vh + h);
    unpack_link<F>(u, v);
    if constexpr (S::R == 2 && ROW2) rebuild_row2(u);
}

// Split FP64 storage of read-only links: rows 0 and 1 of each link rounded
// to FP32, laid out as the FP32-12 field, followed by a second field of the
// same shape holding each element's remainder x - hi as a 16-bit integer q in
// units of 2^-40 (three 4 x int16 vectors per link).  The element read back,
// hi + q 2^-40, is exact in FP64 and within 2^-40 of x for |x| <= 1 (every
// entry of an SU(3) matrix): 72 B per link instead of 96 B in FP64-12.
typedef short v4s __attribute__((ext_vector_type(4)));
constexpr double kSplitUnit = 0x1p-40;

__device__ __forceinline__ v4s *split_res_ptr(void *field, uint32_t Vh, int parity, int mu)
{
    return reinterpret_cast<v4s *>(reinterpret_cast<v4f *>(field) + (size_t)24 * Vh) +
           (size_t)((parity * 4 + mu) * 3) * Vh;
}

__device__ __forceinline__ void split_encode(double x, float &hi, short &q)
{
    hi = (float)x;  // round to nearest, ties to even
    const double r = rint((x - (double)hi) * 0x1p40);  // x - hi is exact
    q = (short)fmin(fmax(r, -32767.0), 32767.0);
}

template <bool NT>
__device__ __forceinline__ void load_link_split(mat3<double> &u, void *field, uint32_t Vh, int parity, int mu,
                                                uint32_t h)
{
    const v4f *hb = block_ptr<kF32_12>(field, Vh, parity, mu);
    const v4s *qb = split_res_ptr(field, Vh, parity, mu);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const v4f a = vload<NT>(hb + (size_t)k * Vh + h);
        const v4s q = vload<NT>(qb + (size_t)k * Vh + h);
        u.e[(2 * k) / 3][(2 * k) % 3] = {(double)a.x + (double)q.x * kSplitUnit,
                                         (double)a.y + (double)q.y * kSplitUnit};
        u.e[(2 * k + 1) / 3][(2 * k + 1) % 3] = {(double)a.z + (double)q.z * kSplitUnit,
                                                 (double)a.w + (double)q.w * kSplitUnit};
    }
}

// Per-site link records: a read-only copy of a 12-real link field for the
// sweeps that keep the links fixed.  For each parity, the sites are grouped
// in tiles of kRecTile consecutive half indices; a tile holds, for each of
// its sites, the 8 links one site update reads -- U_mu(x) in slot mu and
// U_mu(x - mu) in slot 4 + mu -- vector by vector across the tile's sites:
//     vector index = ((parity * rec_tiles(Vh) + h / T) * 8 + slot) * NV * T
//                    + k * T + h % T,    T = kRecTile, k < NV
// so the 8 links of a wavefront's 32 sites are one contiguous block (every
// link is stored twice, once with each end; a last partial tile is padded).
// kF64_12S records hold the split storage: per (parity, tile, slot) the 3
// FP32 vectors of the tile's links as above (NV = 3), then their 3 remainder
// vectors (v4s) in the same order, 72 B per link.
constexpr uint32_t kRecTile = 32;
__host__ __device__ inline uint32_t rec_tiles(uint32_t Vh) { return (Vh + kRecTile - 1) / kRecTile; }

// The tile of site h and its place in it.  UNIFORM: every active lane of the
// wave holds a site of one tile (2 or 4 lanes per site and waves that start at
// a multiple of 32 or 16 sites), so the tile's address is formed once per wave
// in scalar registers: 64-bit addresses per lane cost the FP64 update 8 more
// vector registers and its third wave per SIMD.
struct RecPos {
    uint32_t tile, pos;
};

template <bool UNIFORM> __device__ __forceinline__ RecPos rec_pos(uint32_t h)
{
    const uint32_t t = h / kRecTile;
    return {UNIFORM ? (uint32_t)__builtin_amdgcn_readfirstlane((int)t) : t, h % kRecTile};
}

// first FP32 vector and first remainder vector of link `slot` of a site in
// kF64_12S records
__device__ __forceinline__ const v4f *rec_split_hi(const void *rec, uint32_t Vh, int parity, int slot, RecPos p)
{
    const char *b = reinterpret_cast<const char *>(rec) + ((size_t)parity * rec_tiles(Vh) + p.tile) * (8 * kRecTile * 72);
    return reinterpret_cast<const v4f *>(b + (uint32_t)slot * (kRecTile * 72)) + p.pos;
}
__device__ __forceinline__ const v4s *rec_split_lo(const void *rec, uint32_t Vh, int parity, int slot, RecPos p)
{
    const char *b = reinterpret_cast<const char *>(rec) + ((size_t)parity * rec_tiles(Vh) + p.tile) * (8 * kRecTile * 72);
    return reinterpret_cast<const v4s *>(b + (uint32_t)slot * (kRecTile * 72) + kRecTile * 48) + p.pos;
}

template <int F>
__device__ __forceinline__ const typename Fmt<F>::V *rec_ptr(const void *rec, uint32_t Vh, int parity, int slot,
                                                             RecPos p)
{
    const typename Fmt<F>::V *b = reinterpret_cast<const typename Fmt<F>::V *>(rec) +
                                  ((size_t)parity * rec_tiles(Vh) + p.tile) * (8 * Fmt<F>::NV * kRecTile);
    return b + ((uint32_t)slot * (Fmt<F>::NV * kRecTile) + p.pos);
}

// link `slot` of a site's record, rows 0 and 1 (streamed past the caches)
template <int F>
__device__ __forceinline__ void load_link_rec(mat3<typename Fmt<F>::T> &u, const void *rec, uint32_t Vh, int parity,
                                              int slot, RecPos p)
{
    static_assert(Fmt<F>::R == 2, "records hold 12-real links");
    if constexpr (F == kF64_12S) {
        const v4f *hb = rec_split_hi(rec, Vh, parity, slot, p);
        const v4s *qb = rec_split_lo(rec, Vh, parity, slot, p);
        v4f a[3];
        v4s q[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            a[k] = vload<true>(hb + (size_t)k * kRecTile);
            q[k] = vload<true>(qb + (size_t)k * kRecTile);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            u.e[(2 * k) / 3][(2 * k) % 3] = {(double)a[k].x + (double)q[k].x * kSplitUnit,
                                             (double)a[k].y + (double)q[k].y * kSplitUnit};
            u.e[(2 * k + 1) / 3][(2 * k + 1) % 3] = {(double)a[k].z + (double)q[k].z * kSplitUnit,
                                                     (double)a[k].w + (double)q[k].w * kSplitUnit};
        }
    } else {
        const typename Fmt<F>::V *b = rec_ptr<F>(rec, Vh, parity, slot, p);
        typename Fmt<F>::V v[Fmt<F>::NV];
#pragma unroll
        for (int k = 0; k < Fmt<F>::NV; ++k) v[k] = vload<true>(b + (size_t)k * kRecTile);
        unpack_link<F>(u, v);
    }
}

template <int F, bool NT = false>
__device__ __forceinline__ void store_link(typename Fmt<F>::V *blk, uint32_t Vh, uint32_t h,
                                           const mat3<typename Fmt<F>::T> &u)
{
    using S = Fmt<F>;
#pragma unroll
    for (int k = 0; k < S::NV; ++k) {
        typename S::V v;
        if constexpr (S::CPV == 1) {
            v.x = u.e[k / 3][k % 3].re;
            v.y = u.e[k / 3][k % 3].im;
        } else {
            v.x = u.e[(2 * k) / 3][(2 * k) % 3].re;
            v.y = u.e[(2 * k) / 3][(2 * k) % 3].im;
            v.z = u.e[(2 * k + 1) / 3][(2 * k + 1) % 3].re;
            v.w = u.e[(2 * k + 1) / 3][(2 * k + 1) % 3].im;
        }
        vstore<NT>(blk + (size_t)k * Vh + h, v);
    }
}

// ----------------------------------------------------------------------------
// Lattice geometry.  Half index h of a site of parity p is floor(s/2) with
// s the lexicographic index (Lx even, so each x-row holds Lx/2 sites of each
// parity); the parity-(1-p) neighbours of x in the t, z, y directions sit at
// h -/+ the half strides, the x neighbours at the same row position or one off.
// ----------------------------------------------------------------------------

// Exact division of n < 2^31 by a divisor fixed on the host:
// n / d = floor(2n m / 2^32) >> l with l = ceil(log2 d), m = floor(2^(31+l) / d) + 1
// (Granlund and Montgomery, PLDI'94; the factor 2 keeps d = 1 inside 32 bits).
struct FastDiv {
    uint32_t m, l;
};

inline FastDiv make_fast_div(uint32_t d)
{
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    return {(uint32_t)((1ull << (31 + l)) / d + 1), l};
}

__host__ __device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv &f)
{
    return (uint32_t)((uint64_t)(2u * n) * f.m >> 32) >> f.l;
}

// Which of n items (workgroups' shares, ordered like the sites) workgroup b
// takes: the dispatch deals workgroups to the 8 XCDs in turn, and each XCD
// takes runs of consecutive items, so that what neighbouring items share stays
// in its L2.
struct XcdRuns {
    uint32_t run;
    FastDiv d;
};

__host__ __device__ __forceinline__ uint32_t xcd_item(uint32_t b, const XcdRuns &r)
{
    const uint32_t s = b >> 3, j = fast_div(s, r.d);
    return (j * 8u + (b & 7u)) * r.run + (s - j * r.run);
}

struct Geom {
    uint32_t L[4];   // Lt, Lz, Ly, Lx
    uint32_t hx;     // Lx / 2
    uint32_t Vh;     // V / 2
    uint32_t hs[3];  // half strides of t, z, y: Lz*Ly*hx, Ly*hx, hx
    FastDiv dx, dy, dz;  // division by hx, Ly, Lz
};

// workgroup b's place when n workgroups are walked backwards, on the XCD that has
// it forwards where n allows
__host__ __device__ __forceinline__ uint32_t backwards(uint32_t b, uint32_t n)
{
    return (n & 7u) ? n - 1u - b : n - 8u - (b & ~7u) + (b & 7u);
}

// The order of a link sweep's workgroups: contiguous ranges per XCD (the grid a
// multiple of 8); from the end of the lattice (the odd half-sweep, which then
// starts on what the even one read last).
constexpr int kXcdRanges = 1, kBackward = 2;
__host__ __device__ __forceinline__ uint32_t launch_place(uint32_t b, uint32_t n, int order)
{
    if (order & kBackward) b = backwards(b, n);
    return (order & kXcdRanges) ? (b & 7u) * (n >> 3) + (b >> 3) : b;
}

// Runs for n items over the lattice g whose sites take site_bytes each (0 for
// items that share nothing across t), and the grid they need (items at n and beyond are to be left out by the kernel).  One
// run per XCD while the 8 t-slices that are then read at a time stay in the
// last-level cache until the next one reads them again (256 MB, of which they may
// take 200); else the 8 XCDs share a t-slice.  64^4, shared slices against one
// run per XCD: F and theta 1896 against 2161 us (FP64-18), 650 against 700
// (FP32-12); plaquette 3968 against 4294 and 1600 against 1700.
inline XcdRuns xcd_runs(uint32_t n, const Geom &g, size_t site_bytes, uint32_t *grid)
{
    uint32_t run = (n + 7u) / 8u;
    if (16ull * g.hs[0] * site_bytes > 200000000ull) {
        const uint32_t share = ((n + g.L[0] - 1u) / g.L[0] + 7u) / 8u;
        run = share < run ? share : run;
    }
    const uint32_t per = 8u * run;
    *grid = (n + per - 1u) / per * per;
    return {run, make_fast_div(run)};
}

struct Site {
    uint32_t t, z, y, x;
    uint32_t row;  // (t*Lz + z)*Ly + y
    uint32_t xh;   // position in the row's half: x / 2
};

__device__ __forceinline__ Site decode(const Geom &g, int parity, uint32_t h)
{
    Site c;
    c.row = fast_div(h, g.dx);
    c.xh = h - c.row * g.hx;
    const uint32_t tz = fast_div(c.row, g.dy);
    c.y = c.row - tz * g.L[2];
    c.t = fast_div(tz, g.dz);
    c.z = tz - c.t * g.L[1];
    c.x = 2 * c.xh + ((parity + c.t + c.z + c.y) & 1u);
    return c;
}

// Coordinate, extent and half stride of a site along mu (mu = 3: positions in
// the row's half).  Selects, not an indexed read of g: mu depends on the lane
// in the kernels with several lanes per site, and an index would put a memory
// access in front of every neighbour's address.
struct Axis {
    uint32_t c, e, s;
};

__device__ __forceinline__ Axis axis_of(const Geom &g, const Site &c, int mu)
{
    Axis a;
    a.c = (mu == 0) ? c.t : (mu == 1) ? c.z : (mu == 2) ? c.y : c.xh;
    a.e = (mu == 0) ? g.L[0] : (mu == 1) ? g.L[1] : (mu == 2) ? g.L[2] : g.hx;
    a.s = (mu == 0) ? g.hs[0] : (mu == 1) ? g.hs[1] : (mu == 2) ? g.hs[2] : 1u;
    return a;
}

// half index (in the other parity) of the site x - mu (along x, the site at
// an odd x has its left neighbour at its own position of the other half)
__device__ __forceinline__ uint32_t back_half(const Geom &g, const Site &c, uint32_t h, int mu)
{
    const Axis a = axis_of(g, c, mu);
    const uint32_t n = (a.c == 0) ? h + (a.e - 1) * a.s : h - a.s;
    return (mu == 3 && (c.x & 1u)) ? h : n;
}

// half index (in the other parity) of the site x + mu
__device__ __forceinline__ uint32_t fwd_half(const Geom &g, const Site &c, uint32_t h, int mu)
{
    const Axis a = axis_of(g, c, mu);
    const uint32_t n = (a.c + 1 == a.e) ? h - (a.e - 1) * a.s : h + a.s;
    return (mu == 3 && !(c.x & 1u)) ? h : n;
}

__device__ __forceinline__ uint32_t lex_index(const Geom &g, const Site &c) { return c.row * g.L[3] + c.x; }

// ----------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of
// (x0, x1, x2, x3) -> (hi(M1 x2) ^ x1 ^ k0, lo(M1 x2), hi(M0 x0) ^ x3 ^ k1,
// lo(M0 x0)) with the key bumped by the Weyl increments between rounds.
// ----------------------------------------------------------------------------

__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
    constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = M0 * c.x, hi0 = __umulhi(M0, c.x);
        const uint32_t lo1 = M1 * c.z, hi1 = __umulhi(M1, c.z);
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        k0 += W0;
        k1 += W1;
    }
    return c;
}

}  // namespace lgf
