// Step with ring-decomposed localized kernels (Section 2.4, see lenia_step.hip) in
// quads, for worlds of at least one 4 x 64 tile.
//
// One cell per lane held the 63 ring sums of its three channels (157 registers,
// three waves per SIMD) and read 675 gene values one by one: 0.42 ns per cell, 438
// us at 1024^2, where the genes' own traffic takes 245.  Here a workgroup of three
// waves serves a 4 x 64 tile, wave s the kernels reading channel s: a lane holds
// the 21 ring sums of one channel for the four cells of its quad, and a gene
// plane's disks are three 16-byte reads and, at the ends of a tile row, a scalar:
// 353 us (three waves per SIMD; 433 with two), 700 x 333 143 -> 102.
// The waves meet once, to join alpha and to sum the growth of each target channel
// (handed over through LDS, added in the order of the one-cell form).
#include "lenia_device.h"
#include "lenia_internal.h"
#include "lenia_plan.h"
#include "lenia_quad.h"
#include "lenia_ring.h"

namespace lenia {

template <int R>
struct RingTile {
    static constexpr int TY = 4, TX = 64, HALO = R - 1, PAD = 12;
    static constexpr int PY = TY + 2 * HALO, PITCH = TX + 2 * PAD, QX = PITCH / 4;
    static constexpr int NQ = PY * QX, IT = (NQ + 63) / 64;
};

template <class T, int R>
__global__ __launch_bounds__(192, 3) void ring_quad_kernel(WorldArgs wd)
{
    using L = RingTile<R>;
    constexpr int NK = T::NK, KPS = T::KPS, NPG = 9 * NK, NRE = kRings<R>.nre, NR = RingTables<R>::NR;
    constexpr int CELLS = L::TY * L::TX;
    static_assert(KPS * CELLS <= L::PY * L::PITCH, "the growths fit the channel's region");
    __shared__ __attribute__((aligned(16))) float sA[T::C][L::PY * L::PITCH];
    __shared__ int masks[T::C][64];
    __shared__ int flags[T::C];
    const int H = wd.H, W = wd.W;
    const size_t HW = (size_t)H * W;
    const uint32_t pb = 4u * (uint32_t)HW;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    // (0 without a list: past the end of a plane of 0 bytes)
    const int zero_byte = (int)__builtin_amdgcn_raw_buffer_load_b8(
        plane((const float*)wd.p_zero, wd.p_zero != nullptr ? (uint32_t)wd.n_tiles : 0u), tile, 0, 0);
    int tyi, txi;
    band_tile(tile, wd.tiles_x, wd.n_tiles, tyi, txi);
    // tiles at the far edges end there; cells that two tiles share are computed by
    // both, alike
    const int y0 = min(tyi * L::TY, H - L::TY), x0 = min(txi * L::TX, W - L::TX);
    const int ch = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), g = threadIdx.x & 63;
    const int ly = g >> 4, lq = g & 15, gy = y0 + ly, gx = x0 + 4 * lq;
    const uint32_t ob = 4u * ((uint32_t)gy * (uint32_t)W + (uint32_t)gx);
    float* own = sA[ch];

    // a tile that the output buffer holds as 0, as in quad_tile (1024^2, 12 steps
    // from blobs: 3.15 ms, 3.21 with every tile staged)
    const bool was_zero = __builtin_amdgcn_readfirstlane(zero_byte) != 0;
    if (was_zero && still_empty<L::TY, L::TX>(wd, ch, y0, x0)) return;

    // 1. stage the channel (rows y0 - HALO .., columns x0 - 12 .., wrapped; a group
    // of four columns across the seam is read cell by cell)
    float most = 0.f;
    {
        const plane_t pa = plane(wd.A + (size_t)ch * HW, pb);
        f4 v[L::IT];
#pragma unroll
        for (int it = 0; it < L::IT; ++it) {
            const int i = g + 64 * it, yy = i / L::QX, xx = i - yy * L::QX;
            int sy = y0 + yy - L::HALO, sx = x0 + 4 * xx - L::PAD;
            wrap2(sy, sx, H, W, true);
            const uint32_t row = (uint32_t)sy * (uint32_t)W;
            v[it] = f4{0.f, 0.f, 0.f, 0.f};
            if (i < L::NQ) {
                if (sx + 3 < W) {
                    v[it] = pld4(pa, 4u * (row + (uint32_t)sx));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[it][e] = pld(pa, 4u * (row + (uint32_t)(sx + e >= W ? sx + e - W : sx + e)));
                }
            }
        }
#pragma unroll
        for (int it = 0; it < L::IT; ++it) {
            const int i = g + 64 * it;
            if (i < L::NQ) *reinterpret_cast<f4*>(own + 4 * i) = v[it];
            most = fmaxf(fmaxf(most, fmaxf(v[it][0], v[it][1])), fmaxf(v[it][2], v[it][3]));
        }
    }
    // tiles where alpha = 0 everywhere: an empty channel or a dead gene plane 0
    {
        constexpr int G1X = L::TX + 2, NG1 = (L::TY + 2) * G1X;
        const plane_t p0 = plane(wd.P, pb);
        bool live = false;
#pragma unroll
        for (int i0 = 0; i0 < NG1; i0 += 192) {
            const int i = i0 + (int)threadIdx.x;
            if (i < NG1) {
                const int yy = i / G1X;
                int sy = y0 + yy - 1, sx = x0 + (i - yy * G1X) - 1;
                wrap2(sy, sx, H, W, true);
                live = live || (pld(p0, 4u * ((uint32_t)sy * (uint32_t)W + (uint32_t)sx)) > wd.eps);
            }
        }
        const int bits = (__any(most > wd.skip_thr) ? (1 << ch) : 0) | (__any(live) ? 8 : 0);
        if (g == 0) flags[ch] = bits;
    }
    __syncthreads();
    const float* c = own + (ly + L::HALO) * L::PITCH + 4 * lq;   // the quad is at c[12 .. 15]
    const f4 a = *reinterpret_cast<const f4*>(c + L::PAD);
    const plane_t paout = plane(wd.A_out + (size_t)ch * HW, pb);
    const f4 zero4 = {0.f, 0.f, 0.f, 0.f};
    {
        const bool dead = (flags[0] | flags[1] | flags[2]) != 15;
        // (every thread has read the byte before the barrier above)
        if (wd.p_zero != nullptr && threadIdx.x == 0) wd.p_zero[tile] = dead ? 1 : 0;
        if (dead) {
            pst4(paout, ob, f4{clip01(a[0]), clip01(a[1]), clip01(a[2]), clip01(a[3])});
            if (!was_zero) {
#pragma unroll
                for (int i = 0; i < NPG / T::C; ++i)
                    pst4_stream(plane(wd.P_out + (size_t)(ch * (NPG / T::C) + i) * HW, pb), ob, zero4);
            }
            return;
        }
    }

    // 2. ring sums of the channel
    float S[NRE][4];
#pragma unroll
    for (int sl = 0; sl < NRE; ++sl)
#pragma unroll
        for (int e = 0; e < 4; ++e) S[sl][e] = (sl == kRings<R>.slot[0]) ? a[e] : 0.f;   // the centre
    walk_quad<R, L::PITCH>(c, Everywhere{}, [&](auto ac, auto bc, const float (&t)[4]) {
        constexpr int A = decltype(ac)::value, B = decltype(bc)::value;
        constexpr int sl = kRings<R>.slot[ring_of_d2(R, NR, A * A + B * B)];
#pragma unroll
        for (int e = 0; e < 4; ++e) S[sl][e] += t[e];
    });
    // formed here: otherwise the compiler moves sums to their first use and keeps
    // the taps until then
#pragma unroll
    for (int sl = 0; sl < NRE; ++sl)
#pragma unroll
        for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(S[sl][e]));

    // 3. the kernels reading the channel: their 9 gene planes (r1, w1, b1, r2, w2,
    // b2, m, s, h), the next plane's reads in flight under this one's arithmetic
    // (two planes ahead is slower: 405 against 378 us at 1024^2); genes are stored
    // while alpha holds for what has been read
    const uint32_t kpack = (ch == 0) ? pack_sources<T>(0) : (ch == 1) ? pack_sources<T>(1) : pack_sources<T>(2);
    const bool first = (lq == 0), last = (lq == 15);
    const int ym = (gy == 0) ? H - 1 : gy - 1, yp = (gy == H - 1) ? 0 : gy + 1;
    const uint32_t ou = 4u * ((uint32_t)ym * (uint32_t)W + (uint32_t)gx);
    const uint32_t od = 4u * ((uint32_t)yp * (uint32_t)W + (uint32_t)gx);
    int xe = first ? gx - 1 : gx + 4;
    xe += (xe < 0) ? W : 0;
    xe -= (xe >= W) ? W : 0;
    const uint32_t oe = (first || last) ? ob - 4u * (uint32_t)gx + 4u * (uint32_t)xe : 0xFFFFFFF0u;
    QuadDisk v[3];
    auto load = [&](QuadDisk& q, int j, int t) {
        const plane_t pl = plane(wd.P + (size_t)(t * NK + nibble(kpack, j)) * HW, pb);
        q.u = pld4(pl, ou);
        q.c = pld4(pl, ob);
        q.d = pld4(pl, od);
        q.e = pld(pl, oe);
    };
    const float cs = wd.cnt_scale, ncs = wd.cnt_bias, eps = wd.eps;
    float dm[4];   // running minimum of what alpha tests (0: failed)
#pragma unroll
    for (int e = 0; e < 4; ++e) dm[e] = 3.0e38f;
    load(v[0], 0, 0);
#pragma unroll 1
    for (int j = 0; j < KPS; ++j) {
        // a wave whose cells have all lost alpha stops reading
        if (!__any(dm[0] > eps || dm[1] > eps || dm[2] > eps || dm[3] > eps)) break;
        const int k = nibble(kpack, j);
        float gene[6][4];
        auto plane_of = [&](auto tc, float (&d)[4]) {
            constexpr int t = decltype(tc)::value;
            if constexpr (t + 1 < 9) load(v[(t + 1) % 3], j, t + 1);
            else if (j + 1 < KPS) load(v[0], j + 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            float n[4];
            diffuse_quad<16>(v[t % 3], first, last, cs, ncs, d, n);
            f4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dm[e] = fminf(fminf(dm[e], d[e]), n[e]);
                x[e] = (dm[e] > eps) ? d[e] : 0.f;
            }
            pst4_stream(plane(wd.P_out + (size_t)(t * NK + k) * HW, pb), ob, x);
            __builtin_amdgcn_sched_barrier(0);
        };
        static_for<0, 6>([&](auto tc) { plane_of(tc, gene[decltype(tc)::value]); });
        // ring weights of the two bumps: b exp2(c (x - r)^2), c = -log2(e) / (2 w^2)
        float num[4], den[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            gene[1][e] = -0.72134752044448170f * __builtin_amdgcn_rcpf(gene[1][e] * gene[1][e]);
            gene[4][e] = -0.72134752044448170f * __builtin_amdgcn_rcpf(gene[4][e] * gene[4][e]);
            num[e] = den[e] = 0.f;
        }
#pragma unroll
        for (int sl = 0; sl < NRE; ++sl) {
            constexpr float inv_nr = 1.0f / (float)NR;
            const float x = (float)kRings<R>.ring_of_slot[sl] * inv_nr;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d1 = x - gene[0][e], d2 = x - gene[3][e];
                const float kw = gene[2][e] * __builtin_amdgcn_exp2f(gene[1][e] * (d1 * d1)) +
                                 gene[5][e] * __builtin_amdgcn_exp2f(gene[4][e] * (d2 * d2));
                num[e] = fmaf(kw, S[sl][e], num[e]);
                den[e] = fmaf(kw, (float)kRings<R>.size_of_slot[sl], den[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] = (den[e] > 0.f) ? num[e] / den[e] : 0.f;   // u
        static_for<6, 9>([&](auto tc) { plane_of(tc, gene[decltype(tc)::value - 6]); });
        f4 gk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dm[e] = (num[e] > eps) ? dm[e] : 0.f;
            gk[e] = growth(num[e], gene[0][e], gene[1][e], gene[2][e]);
        }
        *reinterpret_cast<f4*>(own + j * CELLS + 4 * g) = gk;   // the channel's taps are no longer needed
    }
    int m = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) m |= (dm[e] > eps) ? (1 << e) : 0;
    masks[ch][g] = m;
    __syncthreads();
    const int alpha = masks[0][g] & masks[1][g] & masks[2][g];

    // 4. update of channel ch
    const uint32_t ppack = (ch == 0) ? pack_positions<T>(0) : (ch == 1) ? pack_positions<T>(1) : pack_positions<T>(2);
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < T::KPD; ++j) {
        const int pos = nibble(ppack, j), s = (pos * 13) >> 6;   // pos / 5 for pos < 15
        const f4 gk = *reinterpret_cast<const f4*>(sA[s] + (pos - s * KPS) * CELLS + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += (alpha & (1 << e)) ? gk[e] : 0.f;
    }
    f4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = clip01((alpha & (1 << e)) ? fmaf(wd.dt, sum[e], a[e]) : a[e]);
    pst4(paout, ob, out);
    if (alpha != 15) {
        // genes masked to 0: whole quads, or single cells
#pragma unroll 1
        for (int t = 0; t < 9 * KPS; ++t) {
            const plane_t pl = plane(wd.P_out + (size_t)((t % 9) * NK + nibble(kpack, t / 9)) * HW, pb);
            if (alpha == 0) {
                pst4_stream(pl, ob, zero4);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!(alpha & (1 << e))) pst_stream(pl, ob + 4u * e, 0.f);
            }
        }
    }
}

static hipError_t launch_ring_quad(const WorldArgs& w, int, hipStream_t s)
{
    hipLaunchKernelGGL((ring_quad_kernel<Table3x15, 12>), dim3(w.n_tiles), dim3(192), 0, s, w);
    return hipGetLastError();
}

step_launch_fn find_ring_quad_launcher(int table, int R)
{
    return (table == TABLE_3x15 && R == 12) ? &launch_ring_quad : nullptr;
}

}  // namespace lenia
