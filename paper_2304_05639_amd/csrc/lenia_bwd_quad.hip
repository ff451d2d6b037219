// Adjoint of a gene-updating step of the 15-kernel table (see lenia_bwd.hip for
// the formulas), for worlds of at least one 4 x 64 tile.  Three kernels:
//   1. cells: the growth's and clips' cotangents, numbar (the cotangent of each
//      diffusion's numerator), ubar, and per source channel the six combinations
//        W_p = sum_j shc[j][p] ubar_j        (p: a (B, shell) pair)
//   2. convolution: gA_s = direct term + sum_p core_p (x) W_p, and the products
//        M_{k,i} = <ubar_k, core_{B_k,i} (x) A_src>  per tile
//   3. diffusion transpose gP = sum over the disk of numbar, and the shell-height
//      gradient from the M of all tiles.
//
// Why shells.  sum_j K~_j (x) ubar_j with K~_j = sum_i beta_{j,i} / z_j core_i is
// linear in the six cores, and the cores of one B split the disk, so each tap
// takes three planes (one per B) instead of five, with compile-time weights; the
// shell-height gradient needs the forward's six shell sums of A (3 multiply-adds
// per orbit) instead of fifteen.  A constant added to A cancels in it, so A is
// staged relative to the middle of the tile's range, which keeps the terms that
// cancel small.
//
// Why four waves.  A workgroup serves one tile and source channel: wave 0 the
// shell sums of A, wave B = 1, 2, 3 the planes of B, each lane a quad.  Each wave
// stages its planes one after another into its own buffer (no barrier until the
// sums are joined), reading the next while it walks one.  One cell and all six
// planes per lane read 437 x 24 bytes of LDS per cell and channel, and the gather
// took 352 us of the 421 us adjoint at 600 x 1000; a quad's row of the disk is
// seven 16-byte reads per plane for four cells.
//
// W, ubar and the direct term pass through gP_t, which kernel 3 overwrites.
#include "lenia_bwd.h"
#include "lenia_plan.h"
#include "lenia_quad.h"

namespace lenia {

constexpr int kWPlane = 0, kUPlane = 18, kDirectPlane = 33;   // in gP_t: W, ubar, direct term

// ---------------------------------------------------------------------------
// 1. cells: three waves per 64 cells, wave c the kernels writing channel c
// ---------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(192) void bwd_cell_quad_kernel(BwdArgs b)
{
    constexpr int NK = T::NK, KPD = T::KPD, KPS = T::KPS;
    __shared__ float ub[NK][64];
    const int H = b.H, W = b.W;
    const uint32_t HW = (uint32_t)H * (uint32_t)W;
    const int c = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const bool in = blockIdx.x * 64u + lane < HW;
    const uint32_t idx = in ? blockIdx.x * 64u + lane : HW - 1;
    const int gy = (int)(idx / (uint32_t)W), gx = (int)(idx - (uint32_t)gy * W);
    const float eps = b.eps, dt = b.dt;
    const bool alpha = b.alpha[idx] != 0;
    const float a = (b.A + (size_t)c * HW)[idx];
    const float g1 = (b.gA1 + (size_t)c * HW)[idx];
    float zb = (a >= 0.f && a <= 1.f) ? g1 : 0.f;   // where alpha = 0: no growth, z = A
    float ubar[KPD];
#pragma unroll
    for (int j = 0; j < KPD; ++j) ubar[j] = 0.f;
    auto kernel_of = [&](int j) { return (c == 0) ? T::kdst[0][j] : (c == 1) ? T::kdst[1][j] : T::kdst[2][j]; };
    if (alpha) {
        // every read is issued before the arithmetic that needs it
        const Nbr nb = neighbours(gy, gx, H, W);
        float pv[3][KPD][5], u[KPD], gp1[3][KPD];
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int j = 0; j < KPD; ++j) {
                const float* pl = b.P + (size_t)(p * NK + kernel_of(j)) * HW;
                pv[p][j][0] = pl[nb.ou];
                pv[p][j][1] = pl[nb.ol];
                pv[p][j][2] = pl[nb.oc];
                pv[p][j][3] = pl[nb.orr];
                pv[p][j][4] = pl[nb.od];
            }
#pragma unroll
        for (int j = 0; j < KPD; ++j) u[j] = (b.U + (size_t)kernel_of(j) * HW)[idx];
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int j = 0; j < KPD; ++j) gp1[p][j] = b.gP1 ? (b.gP1 + (size_t)(p * NK + kernel_of(j)) * HW)[idx] : 0.f;
        float pd[3][KPD], rn[3][KPD];
        bool clip_ok[3][KPD];
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int j = 0; j < KPD; ++j) {
                const Diffused df = diffuse_vals(pv[p][j], eps);
                const float inv = (df.n > 0) ? __builtin_amdgcn_rcpf((float)df.n) : 0.f;
                const float qq = df.num * inv;
                pd[p][j] = df.v;
                clip_ok[p][j] = (df.n > 0) && (qq >= 0.f) && (qq <= 1.f);
                rn[p][j] = inv;
            }
        // forward growth and pre-clip update, in the step's order
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < KPD; ++j) sum = growth_acc(sum, u[j], pd[0][j], pd[1][j], pd[2][j]);
        const float z = fmaf(dt, sum, a);
        zb = (z >= 0.f && z <= 1.f) ? g1 : 0.f;
        const float gb = dt * zb;
#pragma unroll
        for (int j = 0; j < KPD; ++j) {
            const float m = pd[0][j], s = pd[1][j], h = pd[2][j];
            const float d = u[j] - m;
            const float e = growth_bell(d, s);
            const float is2 = __builtin_amdgcn_rcpf(s * s);
            const float common = 2.f * h * e * d * is2;   // dg/dm = -dg/du
            ubar[j] = -gb * common;
            const float dd[3] = {gb * common, gb * common * d * __builtin_amdgcn_rcpf(s), gb * (2.f * e - 1.f)};
            if (in) {
                (b.gP + (size_t)(kUPlane + kernel_of(j)) * HW)[idx] = ubar[j];
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    b.numbar[(size_t)(p * NK + kernel_of(j)) * HW + idx] = clip_ok[p][j] ? (gp1[p][j] + dd[p]) * rn[p][j] : 0.f;
            }
        }
    }
    if (in) (b.gP + (size_t)(kDirectPlane + c) * HW)[idx] = zb;
#pragma unroll
    for (int j = 0; j < KPD; ++j) ub[kernel_of(j)][lane] = ubar[j];
    __syncthreads();
    // W of source channel c (0 where alpha = 0)
    float w[6];
#pragma unroll
    for (int p = 0; p < 6; ++p) w[p] = 0.f;
    typedef float f8v __attribute__((ext_vector_type(8)));
    typedef const __attribute__((address_space(4))) f8v cf8v;
#pragma unroll
    for (int j = 0; j < KPS; ++j) {
        const int k = (c == 0) ? T::kidx[0][j] : (c == 1) ? T::kidx[1][j] : T::kidx[2][j];
        const f8v cv = *(cf8v*)((cfloat*)b.shc + (c * KPS + j) * 8);
        const float x = ub[k][lane];
#pragma unroll
        for (int p = 0; p < 6; ++p) w[p] = fmaf(cv[p], x, w[p]);
    }
    if (in) {
#pragma unroll
        for (int p = 0; p < 6; ++p) (b.gP + (size_t)(kWPlane + c * 6 + p) * HW)[idx] = w[p];
    }
}

// ---------------------------------------------------------------------------
// 2. convolution
// ---------------------------------------------------------------------------
template <int R>
struct BwdTile {
    static constexpr int TY = 4, TX = 64, HALO = R - 1, PAD = 12;
    static constexpr int PY = TY + 2 * HALO, PITCH = TX + 2 * PAD, QX = PITCH / 4;
    static constexpr int NQ = PY * QX, IT = (NQ + 63) / 64;
};

// Offsets with a nonzero core in shell pair P of B shells.
template <int R, int B, int P>
struct InShell {
    static constexpr bool test(int a, int b)
    {
        const int o = orbit_index<R>(a, b);
        return ShellBasis<R>::tab.pair[o][B - 1] == P && ShellBasis<R>::tab.core[o][B - 1] != 0.f;
    }
};
// Sum over the wave, in lane 63 (a fixed order: within rows of 16 lanes, then
// across them).
template <int CTRL, int ROWS>
__device__ __forceinline__ float add_dpp(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, true));
}
__device__ __forceinline__ float wave_sum_last(float v)
{
    v = add_dpp<0x111, 0xf>(v);   // row_shr:1, 2, 4, 8
    v = add_dpp<0x112, 0xf>(v);
    v = add_dpp<0x114, 0xf>(v);
    v = add_dpp<0x118, 0xf>(v);
    v = add_dpp<0x142, 0xa>(v);   // row_bcast:15
    v = add_dpp<0x143, 0xc>(v);   // row_bcast:31
    return v;
}
__device__ __forceinline__ float wave_max_all(float v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m));
    return v;
}

template <class T, int R>
__global__ __launch_bounds__(256, 4) void bwd_conv_kernel(BwdArgs b)
{
    using L = BwdTile<R>;
    constexpr int KPS = T::KPS;
    __shared__ __attribute__((aligned(16))) float st[4][L::PY * L::PITCH];
    const int H = b.H, W = b.W;
    const size_t HW = (size_t)H * W;
    const uint32_t pb = 4u * (uint32_t)HW;
    const int s = blockIdx.y;
    int tyi, txi;
    band_tile(xcd_tile(blockIdx.x, b.n_tiles), b.tiles_x, b.n_tiles, tyi, txi);
    const int y0 = min(tyi * L::TY, H - L::TY), x0 = min(txi * L::TX, W - L::TX);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), g = threadIdx.x & 63;
    const int ly = g >> 4, lq = g & 15;
    const int gy = y0 + ly, gx = x0 + 4 * lq;
    const uint32_t ob = 4u * ((uint32_t)gy * (uint32_t)W + (uint32_t)gx);
    float* own = st[wave];
    const float* c = own + (ly + L::HALO) * L::PITCH + 4 * lq;

    // a plane's tile and halo (rows y0 - HALO .., columns x0 - 12 ..), wrapped on
    // the torus; a group of four columns across the seam is read cell by cell
    uint32_t off[L::IT];
    unsigned seam = 0;   // bit it: the group crosses the seam
#pragma unroll
    for (int it = 0; it < L::IT; ++it) {
        const int i = g + 64 * it, yy = i / L::QX, xx = i - yy * L::QX;
        int sy = y0 + yy - L::HALO, sx = x0 + 4 * xx - L::PAD;
        wrap2(sy, sx, H, W, true);
        off[it] = (i < L::NQ) ? 4u * ((uint32_t)sy * (uint32_t)W + (uint32_t)sx) : 0xFFFFFFF0u;
        if (i < L::NQ && sx + 3 >= W) seam |= 1u << it;
    }
    auto read = [&](f4 (&v)[L::IT], plane_t pl) {
#pragma unroll
        for (int it = 0; it < L::IT; ++it) {
            if (seam & (1u << it)) {
                const uint32_t row = off[it] / 4u / (uint32_t)W * (uint32_t)W, sx = off[it] / 4u - row;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[it][e] = pld(pl, 4u * (row + (sx + e >= (uint32_t)W ? sx + e - W : sx + e)));
            } else {
                v[it] = pld4(pl, off[it]);
            }
        }
    };
    auto put = [&](const f4 (&v)[L::IT], float less) {
        bool some = false;
#pragma unroll
        for (int it = 0; it < L::IT; ++it) {
            const int i = g + 64 * it;
            const f4 x = v[it] - f4{less, less, less, less};
            if (i < L::NQ) *reinterpret_cast<f4*>(own + 4 * i) = x;
            some = some || x[0] != 0.f || x[1] != 0.f || x[2] != 0.f || x[3] != 0.f;
        }
        __builtin_amdgcn_wave_barrier();
        return some;
    };

    if (wave == 0) {
        // M_{k,i} of the cells that no earlier tile holds
        uint32_t al = 0;
        __builtin_memcpy(&al, b.alpha + (ob >> 2), 4);
        bool mine[4];
        bool any = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mine[e] = ((al >> (8 * e)) & 0xffu) != 0 && gy >= tyi * L::TY && gx + e >= txi * L::TX;
            any = any || mine[e];
        }
        float m[KPS * 3];
#pragma unroll
        for (int i = 0; i < KPS * 3; ++i) m[i] = 0.f;
        if (__any(any)) {
            f4 v[L::IT];
            read(v, plane(b.A + (size_t)s * HW, pb));
            float lo = 3.0e38f, hi = -3.0e38f;
#pragma unroll
            for (int it = 0; it < L::IT; ++it)
                if (g + 64 * it < L::NQ) {
                    lo = fminf(fminf(lo, fminf(v[it][0], v[it][1])), fminf(v[it][2], v[it][3]));
                    hi = fmaxf(fmaxf(hi, fmaxf(v[it][0], v[it][1])), fmaxf(v[it][2], v[it][3]));
                }
            put(v, 0.5f * (wave_max_all(hi) - wave_max_all(-lo)));
            f4 ub[KPS];
#pragma unroll
            for (int j = 0; j < KPS; ++j) {
                const int k = (s == 0) ? T::kidx[0][j] : (s == 1) ? T::kidx[1][j] : T::kidx[2][j];
                ub[j] = pld4(plane(b.gP + (size_t)(kUPlane + k) * HW, pb), ob);
            }
            float acc[6][4];
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[p][e] = 0.f;
            walk_quad<R, L::PITCH>(c, Everywhere{}, [&](auto ac, auto bc, const float (&t)[4]) {
                constexpr int o = orbit_index<R>(decltype(ac)::value, decltype(bc)::value);
                static_for<0, 3>([&](auto Bc) {
                    constexpr int B = decltype(Bc)::value;
                    constexpr float k = ShellBasis<R>::tab.core[o][B];
                    constexpr int p = ShellBasis<R>::tab.pair[o][B];
                    if constexpr (k != 0.f) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[p][e] = fmaf(k, t[e], acc[p][e]);
                    }
                });
            });
            // formed here: otherwise the compiler moves each sum to the branch of
            // the kernel that uses it and keeps every tap until then
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(acc[p][e]));
#pragma unroll
            for (int j = 0; j < KPS; ++j) {
                const int k = (s == 0) ? T::kidx[0][j] : (s == 1) ? T::kidx[1][j] : T::kidx[2][j];
                const int B = b.n_shells[k];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = mine[e] ? ub[j][e] : 0.f;
                    const float s0 = (B == 1) ? acc[0][e] : (B == 2) ? acc[1][e] : acc[3][e];
                    const float s1 = (B == 2) ? acc[2][e] : acc[4][e];
                    m[3 * j] = fmaf(x, s0, m[3 * j]);
                    m[3 * j + 1] = fmaf(x, s1, m[3 * j + 1]);
                    m[3 * j + 2] = fmaf(x, acc[5][e], m[3 * j + 2]);
                }
            }
        }
        const int tile = tyi * b.tiles_x + txi;
#pragma unroll
        for (int j = 0; j < KPS; ++j) {
            const int k = (s == 0) ? T::kidx[0][j] : (s == 1) ? T::kidx[1][j] : T::kidx[2][j];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const float x = wave_sum_last(m[3 * j + i]);
                if (g == 63) b.part[(size_t)(3 * k + i) * b.n_tiles + tile] = x;
            }
        }
    } else {
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
        auto shells = [&](auto Bc) {
            constexpr int B = decltype(Bc)::value;
            auto src = [&](int i) { return plane(b.gP + (size_t)(kWPlane + s * 6 + shell_pair(B, i)) * HW, pb); };
            f4 v[L::IT];
            read(v, src(0));
            static_for<0, B>([&](auto ic) {
                constexpr int i = decltype(ic)::value, P = shell_pair(B, i);
                const bool some = put(v, 0.f);
                if constexpr (i + 1 < B) read(v, src(i + 1));
                if (__any(some))   // W is 0 where alpha is
                    walk_quad<R, L::PITCH>(c, InShell<R, B, P>{}, [&](auto ac, auto bc, const float (&t)[4]) {
                        constexpr float k =
                            ShellBasis<R>::tab.core[orbit_index<R>(decltype(ac)::value, decltype(bc)::value)][B - 1];
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[e] = fmaf(k, t[e], sum[e]);
                    });
                __builtin_amdgcn_wave_barrier();
            });
        };
        if (wave == 1) shells(std::integral_constant<int, 1>{});
        else if (wave == 2) shells(std::integral_constant<int, 2>{});
        else shells(std::integral_constant<int, 3>{});
        *reinterpret_cast<f4*>(own + 4 * g) = f4{sum[0], sum[1], sum[2], sum[3]};
    }
    __syncthreads();
    if (wave == 1) {
        const f4 d = pld4(plane(b.gP + (size_t)(kDirectPlane + s) * HW, pb), ob);
        const f4 g1 = *reinterpret_cast<const f4*>(st[1] + 4 * g), g2 = *reinterpret_cast<const f4*>(st[2] + 4 * g),
                 g3 = *reinterpret_cast<const f4*>(st[3] + 4 * g);
        pst4(plane(b.gA + (size_t)s * HW, pb), ob, d + ((g1 + g2) + g3));
    }
}

// ---------------------------------------------------------------------------
// 3. diffusion transpose (blocks below n_tiles: three waves, 15 gene planes each)
// and the shell-height gradient (one further block per kernel)
// ---------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(192) void bwd_diffuse_kernel(BwdArgs b, float* gbeta)
{
    constexpr int NK = T::NK;
    __shared__ double red[3][3];
    if ((int)blockIdx.x >= b.n_tiles) {
        const int k = (int)blockIdx.x - b.n_tiles;
        double m[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 3; ++i)
            for (int t = threadIdx.x; t < b.n_tiles; t += 192) m[i] += (double)b.part[(size_t)(3 * k + i) * b.n_tiles + t];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) m[i] += __shfl_xor(m[i], d);
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][i] = m[i];
        }
        __syncthreads();
        if ((int)threadIdx.x < b.n_shells[k]) {
            double x = 0.0;
#pragma unroll
            for (int j = 0; j < 3; ++j)
                x += b.bcomb[9 * k + 3 * threadIdx.x + j] * ((red[0][j] + red[1][j]) + red[2][j]);
            gbeta[3 * k + threadIdx.x] += (float)x;
        }
        return;
    }
    const int H = b.H, W = b.W;
    const size_t HW = (size_t)H * W;
    const uint32_t pb = 4u * (uint32_t)HW;
    int tyi, txi;
    band_tile(xcd_tile(blockIdx.x, b.n_tiles), b.tiles_x, b.n_tiles, tyi, txi);
    const int y0 = min(tyi * 4, H - 4), x0 = min(txi * 64, W - 64);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), g = threadIdx.x & 63;
    const int gy = y0 + (g >> 4), gx = x0 + 4 * (g & 15);
    const bool first = (g & 15) == 0, last = (g & 15) == 15;
    const uint32_t oc = (uint32_t)gy * (uint32_t)W + (uint32_t)gx;
    const uint32_t ou = (uint32_t)(gy == 0 ? H - 1 : gy - 1) * (uint32_t)W + (uint32_t)gx;
    const uint32_t od = (uint32_t)(gy == H - 1 ? 0 : gy + 1) * (uint32_t)W + (uint32_t)gx;
    int xe = first ? gx - 1 : gx + 4;
    xe += (xe < 0) ? W : 0;
    xe -= (xe >= W) ? W : 0;
    const uint32_t oe = oc - (uint32_t)gx + (uint32_t)xe;
    // numbar holds values only where alpha does
    uint32_t au, ac, ad;
    __builtin_memcpy(&au, b.alpha + ou, 4);
    __builtin_memcpy(&ac, b.alpha + oc, 4);
    __builtin_memcpy(&ad, b.alpha + od, 4);
    const bool ae = (first || last) && b.alpha[oe] != 0;
    // lanes whose disks hold any, and the lanes beside them (a lane takes the
    // neighbouring cells from active lanes only)
    const int some = (int)((ac | au | ad) != 0) | (int)ae;
    const bool act = (some | __builtin_amdgcn_update_dpp(0, some, kLaneBefore, 0xf, 0xf, false) |
                      __builtin_amdgcn_update_dpp(0, some, kLaneAfter, 0xf, 0xf, false)) != 0;
    constexpr int NPW = 3 * NK / 3, AHEAD = 3;
    QuadDisk v[AHEAD + 1];
    auto load = [&](int t) {
        const plane_t pl = plane(b.numbar + (size_t)(wave * NPW + t) * HW, pb);
        QuadDisk& q = v[t % (AHEAD + 1)];
        q.u = pld4(pl, 4u * ou);
        q.c = pld4(pl, 4u * oc);
        q.d = pld4(pl, 4u * od);
        q.e = pld(pl, ae ? 4u * oe : 0xFFFFFFF0u);
    };
    if (act) {
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) load(t);
#pragma unroll
        for (int t = 0; t < NPW; ++t) {
            if (t + AHEAD < NPW) load(t + AHEAD);
            __builtin_amdgcn_sched_barrier(0);
            const QuadDisk& q = v[t % (AHEAD + 1)];
            f4 u, x, d;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t byte = 0xffu << (8 * e);
                u[e] = (au & byte) ? q.u[e] : 0.f;
                x[e] = (ac & byte) ? q.c[e] : 0.f;
                d[e] = (ad & byte) ? q.d[e] : 0.f;
            }
            const float row[6] = {beside<16, kLaneBefore>(x[3], q.e, first), x[0], x[1], x[2], x[3],
                                  beside<16, kLaneAfter>(x[0], q.e, last)};
            f4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (((u[e] + row[e]) + row[e + 1]) + row[e + 2]) + d[e];
            pst4_stream(plane(b.gP + (size_t)(wave * NPW + t) * HW, pb), 4u * oc, o);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int t = 0; t < NPW; ++t)
            pst4_stream(plane(b.gP + (size_t)(wave * NPW + t) * HW, pb), 4u * oc, f4{0.f, 0.f, 0.f, 0.f});
    }
}

template <class T, int R>
static hipError_t launch(const BwdArgs& a, float* gbeta, hipStream_t s)
{
    const unsigned cells = (unsigned)a.H * (unsigned)a.W;
    hipLaunchKernelGGL((bwd_cell_quad_kernel<T>), dim3((cells + 63) / 64), dim3(192), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bwd_conv_kernel<T, R>), dim3(a.n_tiles, T::C), dim3(256), 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bwd_diffuse_kernel<T>), dim3(a.n_tiles + T::NK), dim3(192), 0, s, a, gbeta);
    return hipGetLastError();
}

hipError_t launch_bwd_quad(int R, const BwdArgs& a, float* gbeta, hipStream_t s)
{
    return R == 12 ? launch<Table3x15, 12>(a, gbeta, s) : launch<Table3x15, 13>(a, gbeta, s);
}

}  // namespace lenia
