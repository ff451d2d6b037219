// Step of the single-kernel table with global genes (one channel, alpha = 1), for
// worlds of at least one 4 x 64 tile.
//
// What bounds it: latency.  A 64^2 world is 16 tiles; one cell per lane read its
// 516 taps and the kernel's weights one after another, 10.3 us a step of which an
// empty launch takes 2.4.  Here a lane takes a quad (a row of the disk is seven
// 16-byte LDS reads for four cells) and the four waves of a workgroup share the
// tile's quads by rows of the disk (row distance a goes to wave a mod 4, which
// balances them within a sixth), so a wave walks a quarter of the taps; the four
// partial sums are joined in a fixed order, one cell per lane.
#include "lenia_device.h"
#include "lenia_internal.h"
#include "lenia_quad.h"

namespace lenia {

template <int WAVE>
struct RowsOf {
    static constexpr bool test(int a, int) { return a % 4 == WAVE; }
};

template <int R>
struct GlobalTile {
    static constexpr int TY = 4, TX = 64, HALO = R - 1, PAD = 12;
    static constexpr int PY = TY + 2 * HALO, PITCH = TX + 2 * PAD, QX = PITCH / 4;
    static_assert(R <= 13, "12 columns on either side");
};

template <int R>
__device__ __forceinline__ void global_tile(const WorldArgs& wd, int tile, int mode)
{
    using L = GlobalTile<R>;
    __shared__ __attribute__((aligned(16))) float sA[L::PY * L::PITCH];
    __shared__ __attribute__((aligned(16))) float part[4][L::TY * L::TX];
    const int H = wd.H, W = wd.W;
    const uint32_t pb = 4u * (uint32_t)H * (uint32_t)W;
    int tyi, txi;
    band_tile(tile, wd.tiles_x, wd.n_tiles, tyi, txi);
    // tiles at the far edges end there (shared cells are computed alike)
    const int y0 = min(tyi * L::TY, H - L::TY), x0 = min(txi * L::TX, W - L::TX);
    {
        constexpr int NQ = L::PY * L::QX, IT = (NQ + 255) / 256;
        const plane_t pa = plane(wd.A, pb);
        f4 v[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int i = threadIdx.x + 256 * it, yy = i / L::QX, xx = i - yy * L::QX;
            int sy = y0 + yy - L::HALO, sx = x0 + 4 * xx - L::PAD;
            wrap2(sy, sx, H, W, true);
            const uint32_t row = (uint32_t)sy * (uint32_t)W;
            if (i < NQ) {
                if (sx + 3 < W) {
                    v[it] = pld4(pa, 4u * (row + (uint32_t)sx));
                } else {   // a group across the seam
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[it][e] = pld(pa, 4u * (row + (uint32_t)(sx + e >= W ? sx + e - W : sx + e)));
                }
            }
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int i = threadIdx.x + 256 * it;
            if (i < NQ) *reinterpret_cast<f4*>(sA + 4 * i) = v[it];
        }
    }
    __syncthreads();
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), g = threadIdx.x & 63;
        const float* c = sA + ((g >> 4) + L::HALO) * L::PITCH + 4 * (g & 15);
        cfloat* wt = (cfloat*)wd.wt;   // K~ by orbit
        float u[4] = {0.f, 0.f, 0.f, 0.f};
        auto weigh = [&](auto ac, auto bc, const float (&t)[4]) {
            constexpr int o = orbit_index<R>(decltype(ac)::value, decltype(bc)::value);
            const float k = wt[o];
#pragma unroll
            for (int e = 0; e < 4; ++e) u[e] = fmaf(k, t[e], u[e]);
        };
        if (wave == 0) walk_quad<R, L::PITCH>(c, RowsOf<0>{}, weigh);
        else if (wave == 1) walk_quad<R, L::PITCH>(c, RowsOf<1>{}, weigh);
        else if (wave == 2) walk_quad<R, L::PITCH>(c, RowsOf<2>{}, weigh);
        else walk_quad<R, L::PITCH>(c, RowsOf<3>{}, weigh);
        *reinterpret_cast<f4*>(part[wave] + 4 * g) = f4{u[0], u[1], u[2], u[3]};
    }
    __syncthreads();
    const int ly = threadIdx.x >> 6, lx = threadIdx.x & 63;
    const uint32_t o = (uint32_t)(y0 + ly) * (uint32_t)W + (uint32_t)(x0 + lx);
    const float u = (part[0][threadIdx.x] + part[1][threadIdx.x]) + (part[2][threadIdx.x] + part[3][threadIdx.x]);
    if (wd.U_save) pst(plane(wd.U_save, pb), 4u * o, u);
    if (mode == MODE_POTENTIALS) return;
    if (wd.alpha_save) wd.alpha_save[o] = 1;
    const float a = sA[(ly + L::HALO) * L::PITCH + lx + L::PAD];
    const float sum = growth_acc(0.f, u, wd.gm[0], wd.gs[0], wd.gh[0]);
    pst(plane(wd.A_out, pb), 4u * o, clip01(fmaf(wd.dt, sum, a)));
}

template <int R>
__global__ __launch_bounds__(256) void global_step_kernel(WorldArgs wd, int mode)
{
    global_tile<R>(wd, xcd_tile(blockIdx.x, gridDim.x), mode);
}

template <int R>
__global__ __launch_bounds__(256) void global_batch_kernel(BatchList bl, int mode)
{
    typedef const __attribute__((address_space(4))) int cint;
    if ((int)blockIdx.x >= bl.n_items) return;
    const cint* item = (const cint*)(bl.items + xcd_tile(blockIdx.x, bl.n_items));
    const int world = item[0], tile = item[1];
    constexpr int NW = sizeof(WorldArgs) / sizeof(int);
    const cint* src = (const cint*)(bl.worlds + world);
    int words[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) words[i] = src[i];
    const WorldArgs wd = __builtin_bit_cast(WorldArgs, words);
    global_tile<R>(wd, tile, mode);
}

template <int R>
static hipError_t launch_global_step(const WorldArgs& w, int mode, hipStream_t s)
{
    hipLaunchKernelGGL((global_step_kernel<R>), dim3(w.n_tiles), dim3(256), 0, s, w, mode);
    return hipGetLastError();
}

template <int R>
static hipError_t launch_global_batch(const BatchList& b, int mode, hipStream_t s)
{
    if (b.n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL((global_batch_kernel<R>), dim3(b.n_items), dim3(256), 0, s, b, mode);
    return hipGetLastError();
}

step_launch_fn find_global_step_launcher(int R)
{
    return R == 12 ? &launch_global_step<12> : R == 13 ? &launch_global_step<13> : nullptr;
}

batch_launch_fn find_global_batch_launcher(int R)
{
    return R == 12 ? &launch_global_batch<12> : R == 13 ? &launch_global_batch<13> : nullptr;
}

}  // namespace lenia
