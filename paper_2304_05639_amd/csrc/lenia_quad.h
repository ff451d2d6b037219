// Quads (four cells adjacent in a row, one lane) on gfx950: 16-byte plane
// accesses, five-point disks with the neighbouring lanes' cells, and the lattice
// helpers of the kernels that walk a kernel's support in quads.
#pragma once

#include <type_traits>

#include "lenia_device.h"
#include "lenia_internal.h"

namespace lenia {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 pld4(plane_t r, uint32_t off)
{
    return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ void pst4(plane_t r, uint32_t off, f4 v)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, (int)off, 0, 0);
}
// non-temporal
__device__ __forceinline__ f4 pld4_stream(plane_t r, uint32_t off)
{
    return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 2));
}
// non-temporal, as pst_stream
__device__ __forceinline__ void pst4_stream(plane_t r, uint32_t off, f4 v)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, (int)off, 0, 2);
}

// Gene stores of a world whose rows are whole cache lines (W a multiple of 32)
// go past the caches, else through them: there two tiles write parts of one
// line, which L2 joins (four steps of 1021 x 771: 470 against 498 us, 700^2 258
// against 279; at 1024^2 the other way round, 558 against 528, and 8200 against
// 7500 at 4096^2).  Rows of whole half lines (W a multiple of 16) go past them on
// worlds whose 96 planes of a step exceed them by a quarter (from blobs, one step
// of 1000 x 976 92 us, 104 through them, 1658 x 1232 176 and 213, two dense ones
// 516 and 533; but 900 x 816 65 and 53, 272 x 400, three steps, 67 and 62).
__device__ __forceinline__ bool rows_of_lines(int H, int W)
{
    constexpr uint32_t kCells = (320u << 20) / (96 * 4);
    return (W & 31) == 0 || ((W & 15) == 0 && (uint32_t)H * (uint32_t)W > kCells);
}
__device__ __forceinline__ void pst4_rows(bool lines, plane_t r, uint32_t off, f4 v)
{
    if (lines)
        pst4_stream(r, off, v);
    else
        pst4(r, off, v);
}

// f(integral_constant<int, B>), ..., f(integral_constant<int, E - 1>)
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(static_cast<F&&>(f));
    }
}

// Largest b with a^2 + b^2 < R^2.
constexpr int half_width(int R, int a)
{
    int w = 0;
    while ((w + 1) * (w + 1) + a * a < R * R) ++w;
    return w;
}

// Index of the orbit of (a, b) in ShellBasis<R>::tab.
template <int R>
constexpr int orbit_index(int a, int b)
{
    const int hi = a > b ? a : b, lo = a > b ? b : a;
    for (int o = 0; o < ShellBasis<R>::NO; ++o)
        if (ShellBasis<R>::tab.a[o] == hi && ShellBasis<R>::tab.b[o] == lo) return o;
    return -1;
}

// A quad's five-point disks of one gene plane: the quad, the quads above and
// below, and for the first and last quad of a tile row the cell beside it (the
// others take theirs from the neighbouring lane).
struct QuadDisk {
    f4 u, c, d;
    float e;
};

// Data-parallel primitive controls: the value of the lane before or after
// within a row of 16 lanes.  A lane whose source is outside its row, or not
// active, keeps the old value.
constexpr int kLaneBefore = 0x111, kLaneAfter = 0x101;   // row_shr:1, row_shl:1

// src of the lane before (or after); e in the lanes that begin (or end) a tile
// row of QR quads.  The neighbouring lane must be active.
template <int QR, int CTRL>
__device__ __forceinline__ float beside(float src, float e, bool edge)
{
    static_assert(QR == 8 || QR == 16, "a row of 16 lanes holds whole tile rows");
    const float v = __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, e), __builtin_bit_cast(int, src), CTRL, 0xf, 0xf, false));
    return (QR == 16) ? v : (edge ? e : v);
}

// Diffusion of the quad (diffuse_disk for each cell, the sums in its order);
// n[e] = count of values above the cutoff (0: no quotient, d[e] is not used).
template <int QR>
__device__ __forceinline__ void diffuse_quad(const QuadDisk& v, bool first, bool last, float cs, float ncs,
                                             float (&d)[4], float (&n)[4])
{
    const float row[6] = {beside<QR, kLaneBefore>(v.c[3], v.e, first), v.c[0], v.c[1], v.c[2], v.c[3],
                          beside<QR, kLaneAfter>(v.c[0], v.e, last)};
    float k[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) k[i] = clip01(fmaf(row[i], cs, ncs));
    const float k12 = k[1] + k[2], k34 = k[3] + k[4];
    const float h[4] = {k[0] + k12, k12 + k[3], k[2] + k34, k34 + k[5]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        n[e] = h[e] + (clip01(fmaf(v.u[e], cs, ncs)) + clip01(fmaf(v.d[e], cs, ncs)));
        const float num = (((v.u[e] + row[e]) + row[e + 1]) + row[e + 2]) + v.d[e];
        d[e] = clip01(num * __builtin_amdgcn_rcpf(n[e]));
    }
}

// Byte offsets of a quad and of its disks' other cells: the rows above and below
// and, in the lanes at the ends of a tile row, the cell beside it (elsewhere past
// the plane, no access).
struct Around {
    uint32_t u, c, d, e;
};
template <int TX>
__device__ __forceinline__ Around around(int gy, int gx, int lq, int H, int W)
{
    const int ym = (gy == 0) ? H - 1 : gy - 1, yp = (gy == H - 1) ? 0 : gy + 1;
    const uint32_t row = (uint32_t)gy * (uint32_t)W;
    const bool first = (lq == 0), last = (lq == TX / 4 - 1);
    int xe = first ? gx - 1 : gx + 4;
    xe += (xe < 0) ? W : 0;
    xe -= (xe >= W) ? W : 0;
    return Around{4u * ((uint32_t)ym * (uint32_t)W + (uint32_t)gx), 4u * (row + (uint32_t)gx),
                  4u * ((uint32_t)yp * (uint32_t)W + (uint32_t)gx),
                  (first || last) ? 4u * (row + (uint32_t)xe) : 0xFFFFFFF0u};
}

// Whether plane 0 of the disks of the tile at (y0, x0) is at or below the cutoff
// everywhere (alpha then fails in all its cells); if so the channel's A' =
// clip01(A) is written.  Every wave tests all the tile's cells.
template <int TY, int TX>
__device__ __forceinline__ bool still_empty(const WorldArgs& wd, int ch, int y0, int x0)
{
    const uint32_t pb = 4u * (uint32_t)wd.H * (uint32_t)wd.W;
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));   // nothing here is kept for the live tile's code
    const int lq = lane % (TX / 4);
    const Around n = around<TX>(y0 + lane / (TX / 4), x0 + 4 * lq, lq, wd.H, wd.W);
    const plane_t p0 = plane(wd.P, pb);
    const f4 u = pld4(p0, n.u), c = pld4(p0, n.c), d = pld4(p0, n.d);
    const float b = pld(p0, n.e);
    const f4 a = pld4(plane(wd.A + (size_t)ch * wd.H * wd.W, pb), n.c);
    bool live = n.e != 0xFFFFFFF0u && b > wd.eps;
#pragma unroll
    for (int e = 0; e < 4; ++e) live = live || u[e] > wd.eps || c[e] > wd.eps || d[e] > wd.eps;
    if (__any(live)) return false;
    pst4(plane(wd.A_out + (size_t)ch * wd.H * wd.W, pb), n.c, f4{clip01(a[0]), clip01(a[1]), clip01(a[2]), clip01(a[3])});
    return true;
}

// Nibble i of a table packed into one integer.
__device__ __forceinline__ int nibble(uint32_t t, int i) { return (int)((t >> (4 * i)) & 15u); }

// The kernels writing channel c, in summation order, and their positions
// source * KPS + slot, packed.
template <class T>
constexpr uint32_t pack_kernels(int c)
{
    uint32_t t = 0;
    for (int j = 0; j < T::KPD; ++j) t |= (uint32_t)T::kdst[c][j] << (4 * j);
    return t;
}
// The kernels reading channel s, packed.
template <class T>
constexpr uint32_t pack_sources(int s)
{
    uint32_t t = 0;
    for (int j = 0; j < T::KPS; ++j) t |= (uint32_t)T::kidx[s][j] << (4 * j);
    return t;
}
template <class T>
constexpr int position_of(int k)
{
    for (int p = 0; p < T::NK; ++p)
        if (T::kidx[p / T::KPS][p % T::KPS] == k) return p;
    return -1;
}
template <class T>
constexpr uint32_t pack_positions(int c)
{
    uint32_t t = 0;
    for (int j = 0; j < T::KPD; ++j) t |= (uint32_t)position_of<T>(T::kdst[c][j]) << (4 * j);
    return t;
}

// The walk of one plane staged at c (the quad's cells at floats 12 .. 15 of row
// c): rows a = 0 .. R - 1 as V_a[x] = row(a)[x] + row(-a)[x], then
// t = V_a[x + b] + V_a[x - b] per column distance b, handed to use(a, b, t) where
// wanted(a, b).
template <int R, int PITCH, class WANTED, class USE>
__device__ __forceinline__ void walk_quad(const float* c, WANTED wanted, USE use)
{
    static_for<0, R>([&](auto ac) {
        constexpr int a = decltype(ac)::value, w = half_width(R, a);
        constexpr unsigned need = [] {   // 16-byte groups of the row in use
            unsigned m = 0;
            for (int b = (a == 0) ? 1 : 0; b <= w; ++b)
                if (WANTED::test(a, b))
                    for (int e = 0; e < 4; ++e) m |= (1u << ((12 + e + b) / 4)) | (1u << ((12 + e - b) / 4));
            return m;
        }();
        if constexpr (need != 0) {
            // one row at a time: left alone, the compiler reads all rows first
            // and spills them
            __builtin_amdgcn_sched_barrier(0);
            float v[28];
#pragma unroll
            for (int q = 0; q < 7; ++q) {
                if (need & (1u << q)) {
                    f4 x = *reinterpret_cast<const f4*>(c + a * PITCH + 4 * q);
                    if constexpr (a > 0) x += *reinterpret_cast<const f4*>(c - a * PITCH + 4 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
                }
            }
            static_for<(a == 0) ? 1 : 0, w + 1>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                if constexpr (WANTED::test(a, b)) {
                    float t[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = (b == 0) ? v[12 + e] : v[12 + e + b] + v[12 + e - b];
                    use(ac, bc, t);
                }
            });
        }
        (void)wanted;
    });
}

// Every offset of the support.
struct Everywhere {
    static constexpr bool test(int, int) { return true; }
};

}  // namespace lenia
