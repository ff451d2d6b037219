// Fused Lenia step for gfx950, four cells per lane (the 15-kernel table on
// worlds at least one tile large).
//
// A workgroup takes a TY x TX tile with three threads per quad, a quad being
// four cells adjacent in a row: thread (s, quad) forms the potentials of the
// five kernels reading channel s, then, as (c, quad), the genes, growth and
// update of the five kernels writing channel c.  Whole waves belong to one
// channel, so everything that depends on the channel is wave-uniform.
//
// What bounds it and why this split.  One cell per lane reads every tap of
// the 436-cell disk from LDS: at 4096^2 the potentials alone took 1.57 ms and
// the step 1.97, its memory traffic hidden under them.  With four cells per
// lane a row of the disk is seven 16-byte reads of one channel for all four,
// 141 reads where the four cells took 1748, and the gene disks of a plane are
// three 16-byte reads and, in the lanes at the ends of a tile row, one scalar
// instead of twenty scalars.  The potentials take 0.83 ms (VALU issue) and the
// dense step 1.84: it is bound by memory traffic (8.0 GB at 4.4 TB/s, where a
// plain copy of the 45 planes in the same plane-by-plane pattern reaches 4.6 to
// 5.3).  Three threads per quad leave each lane the registers of one channel
// only (160 VGPRs, three waves per SIMD; a budget of four waves, which forms
// more of the walk's sums twice, takes 1.96 ms) and give small worlds three
// times the waves: 256^2 takes 16.6 us a step instead of 20, 512^2 36 instead of
// 48, 1021 x 771 117 instead of 159.  The 4 x 64 tile: a row of 16 quads reads
// LDS without bank conflicts, and a world's odd right edge cuts the fewest
// cache lines; 8 x 32 (one line per row) takes 2.0 ms.
//
// Tiles at the right and bottom edges are moved up to end at the edge; the
// cells two tiles share are computed by both, alike, and written twice with
// the same values.  Smaller worlds run step_kernel (lenia_step.hip), whose
// sums follow the same order (ShellWalk), so the two agree bitwise.
#include "lenia_device.h"
#include "lenia_internal.h"
#include "lenia_plan.h"
#include "lenia_quad.h"

namespace lenia {

// Staged tile of one channel, transposed: PX columns (the tile's and HALO on
// either side) of PITCH floats, row y0 - 12 + i of a column at float i (so that
// four cells of a column begin on a 16-byte boundary).  The pitches leave the
// 16-byte reads of 16 neighbouring columns without bank conflicts.  After the
// walk the channel's region holds the potentials of its five kernels, TY x TX
// floats each, row by row.
template <class T, int R, int TY, int TX>
struct QuadTile {
    static_assert(R <= 13 && (TY == 4 || TY == 8), "12 rows on either side, pitches");
    static constexpr int HALO = R - 1, PAD = 12;
    static constexpr int PX = TX + 2 * HALO, PITCH = (TY == 4) ? 28 : 36;
    static constexpr int G = TY * TX / 4;              // quads, and columns of four cells
    static constexpr int NT = T::C * G;
    static constexpr int REGION = (PX * PITCH > T::KPS * TY * TX) ? PX * PITCH : T::KPS * TY * TX;
    static_assert(G == 64, "one wave per channel");
};

// Potentials of the five kernels reading the channel staged at c, for four
// cells of one column (floats 12 .. 15 of the column c): u[j][e] for slot j and
// row e.  The same sums in the same order as conv_cells_shells (lenia_step.hip),
// so the results are bitwise its results: with H_d[y] = A[y][x + d] + A[y][x - d]
// and Q(r, d) = H_d[y + r] + H_d[y - r], the axis orbits are (A[y + a] + A[y - a])
// + H_a[y], the diagonal ones Q(a, a), the general ones Q(a, b) + Q(b, a), b < a.
// The column pair at distance a is read once for Q(b, a) of every b < a; it
// also gives Q(r, a) for the later orbits (r, a), of which the nearest kHold
// are held in registers until the walk is at column distance r.  The farther
// ones are formed again from LDS when they are needed: holding all of them
// takes 116 registers and leaves two waves per SIMD instead of three.
template <int R>
constexpr int kHold = (R == 12) ? 7 : 6;

template <class T, int R, int PITCH, bool FEW>
__device__ __forceinline__ void quad_potentials(const float* c, cfloat* __restrict__ shc, float (&u)[T::KPS][4])
{
    constexpr int HOLD = kHold<R>;
    float acc[6][4];
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[p][e] = 0.f;
    // acc[(B, shell)] += core * t for B = 1, 2, 3
    auto weigh = [&](auto ac, auto bc, const float (&t)[4]) {
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
    };
    // an offset of 0 that the compiler cannot look through, renewed per step:
    // otherwise it merges the reads of one column in different steps and keeps
    // (and spills) them in between
    int fresh = 0;
    auto renew = [&]() {
        if constexpr (!FEW) __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(fresh));
    };
    // floats i0 .. i1 of H_d (the 16-byte groups that hold them)
    auto pair_rows = [&](float (&h)[28], auto dc, auto i0c, auto i1c) {
        constexpr int d = decltype(dc)::value, q0 = decltype(i0c)::value / 4, q1 = decltype(i1c)::value / 4;
#pragma unroll
        for (int q = q0; q <= q1; ++q) {
            const f4 x = *reinterpret_cast<const f4*>(c + fresh + d * PITCH + 4 * q) +
                         *reinterpret_cast<const f4*>(c + fresh - d * PITCH + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) h[4 * q + e] = x[e];
        }
    };
    // Q(r, d) from H_d alone
    auto far_sum = [&](float (&t)[4], auto rc, auto dc) {
        constexpr int r = decltype(rc)::value;
        float h[28];
        pair_rows(h, dc, std::integral_constant<int, 12 - r>{}, std::integral_constant<int, 15 - r>{});
        if constexpr ((12 + r) / 4 > (15 - r) / 4)
            pair_rows(h, dc, std::integral_constant<int, 12 + r>{}, std::integral_constant<int, 15 + r>{});
        else
            pair_rows(h, dc, std::integral_constant<int, 4 * ((15 - r) / 4) + 4>{}, std::integral_constant<int, 15 + r>{});
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = h[12 + e + r] + h[12 + e - r];
    };
    // axis orbits
    {
        float v[28];
        constexpr int q0 = (12 - (R - 1)) / 4, q1 = (15 + (R - 1)) / 4;
#pragma unroll
        for (int q = q0; q <= q1; ++q) {
            const f4 x = *reinterpret_cast<const f4*>(c + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
        }
        static_for<1, R>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            float h[28], t[4];
            pair_rows(h, ac, std::integral_constant<int, 12>{}, std::integral_constant<int, 15>{});
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = (v[12 + e + a] + v[12 + e - a]) + h[12 + e];
            weigh(ac, std::integral_constant<int, 0>{}, t);
        });
    }
    // diagonal orbits
    static_for<1, R>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        if constexpr (2 * a * a < R * R) {
            if constexpr (!FEW && a % 4 == 1) renew();
            float t[4];
            far_sum(t, ac, ac);
            weigh(ac, ac, t);
        }
    });
    // general orbits, by a, then b
    float held[R][HOLD + 1][4];   // held[r][r - d] = Q(r, d)
    static_for<1, R>([&](auto ac) {
        constexpr int a = decltype(ac)::value, w = half_width(R, a);
        constexpr int nb = (w < a - 1) ? w : a - 1;                    // b = 1 .. nb
        constexpr int nh = (w < a + HOLD) ? w : a + HOLD;            // r = a + 1 .. nh
        constexpr int m = (nh > a) ? nh : nb;                          // rows of H_a in use
        renew();
        float h[28];
        pair_rows(h, ac, std::integral_constant<int, 12 - m>{}, std::integral_constant<int, 15 + m>{});
        static_for<1, nb + 1>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            float t[4];
            if constexpr (a - b <= HOLD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = held[a][a - b][e];
            } else {
                far_sum(t, ac, bc);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] += h[12 + e + b] + h[12 + e - b];
            weigh(ac, bc, t);
        });
        static_for<a + 1, nh + 1>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
#pragma unroll
            for (int e = 0; e < 4; ++e) held[r][r - a][e] = h[12 + e + r] + h[12 + e - r];
        });
    });
    typedef float f8v __attribute__((ext_vector_type(8)));
    typedef const __attribute__((address_space(4))) f8v cf8v;
#pragma unroll
    for (int j = 0; j < T::KPS; ++j) {
        const f8v cv = *(cf8v*)(shc + j * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x = cv[0] * acc[0][e];
#pragma unroll
            for (int p = 1; p < 6; ++p) x = fmaf(cv[p], acc[p][e], x);
            u[j][e] = x;
        }
    }
}

// GIVEN: the potentials are read from U (the second kernel of a step whose
// potentials the MFMA transforms formed), and it and the genes are written past the
// caches if STREAM.
template <class T, int R, int TY, int TX, bool FEW, bool GIVEN = false, bool STREAM = false>
__device__ __forceinline__ void quad_tile(const WorldArgs& wd, int tile, int mode, float* sA, int* masks, int* flags,
                                          uint64_t* above_eps, const float* U = nullptr)
{
    using L = QuadTile<T, R, TY, TX>;
    constexpr int REGION = GIVEN ? T::KPS * TY * TX : L::REGION;
    constexpr int NK = T::NK, KPS = T::KPS, G = L::G, NT = L::NT, NPG = 3 * NK;
    constexpr int CELLS = TY * TX;
    constexpr bool EARLY = !FEW && !GIVEN;
    static_assert(T::C == 3 && T::KPD == T::KPS, "three channels");
    const int H = wd.H, W = wd.W;
    const size_t HW = (size_t)H * W;
    const uint32_t pb = 4u * (uint32_t)HW;
    const bool may_skip = !GIVEN && (mode == MODE_LOCAL_UPDATE) && (wd.U_save == nullptr);
    const bool want_flags = (wd.flags_out != nullptr);
    const bool listed = may_skip && wd.p_zero != nullptr;
    // (0 without a list: past the end of a plane of 0 bytes)
    const int zero_byte = EARLY ? (int)__builtin_amdgcn_raw_buffer_load_b8(
                                      plane((const float*)wd.p_zero, listed ? (uint32_t)wd.n_tiles : 0u), tile, 0, 0)
                                : 0;
    int tyi, txi;
    band_tile(tile, wd.tiles_x, wd.n_tiles, tyi, txi);
    const int y0 = min(tyi * TY, H - TY), x0 = min(txi * TX, W - TX);
    const int ch = __builtin_amdgcn_readfirstlane((int)threadIdx.x / G);   // wave-uniform
    const int g0 = (int)threadIdx.x - ch * G;
    const int ly0 = g0 / (TX / 4), lq0 = g0 % (TX / 4);
    const int gy = y0 + ly0, gx = x0 + 4 * lq0;
    const bool lines = GIVEN ? STREAM : rows_of_lines(H, W);
    float* own = sA + ch * REGION;

    // A tile whose genes the output buffer already holds as 0 was empty two steps
    // ago and mostly still is: where plane 0 confirms it, nothing is staged.  The
    // window of a 4 x 64 tile is 2236 values a channel, and staging it for every
    // tile took most of a sparse world's step: 60 steps of 4096^2, blobs of 24 x 24
    // on 9% of the cells, 41.8 ms, 33.9 so (2048^2, 20 steps, 3.92 and 3.40 ms).
    // Worlds of at most a workgroup per compute unit do not gain by it and would
    // wait for the byte (256^2, 8 steps: 143 us, 139 without).
    bool was_zero = false;
    if constexpr (EARLY) {
        was_zero = __builtin_amdgcn_readfirstlane(zero_byte) != 0;
        if (was_zero && !want_flags && still_empty<TY, TX>(wd, ch, y0, x0)) return;
    }
    // 1. stage the channel: the tile and HALO cells around it, wrapped on the
    // torus.  Lanes take neighbouring columns, four rows (one 16-byte write) at a
    // time.  The tile's first 64 columns have one row per load, so a row's
    // offset is scalar; the remaining ones are dealt to the lanes by (rows,
    // column).  Rows of a column beyond the halo are not read (their loads fall
    // past the plane and give 0).
    float most = 0.f;
    if constexpr (!GIVEN) {
        constexpr int I0 = L::PAD - L::HALO, I1 = L::PAD + TY + L::HALO;   // rows of a column in use: [I0, I1)
        constexpr int NQ = (I1 + 3) / 4, REST = L::PX - 64, IR = (NQ * REST + 63) / 64;
        constexpr uint32_t NONE = 0xFFFFFFF0u;
        const plane_t pa = plane(wd.A + (size_t)ch * HW, pb);
        const auto column = [&](int xx) {   // byte offset of staged column xx
            int sx = x0 + xx - L::HALO;
            sx += (sx < 0) ? W : 0;
            sx -= (sx >= W) ? W : 0;
            return 4u * (uint32_t)sx;
        };
        const auto row = [&](int i) {       // byte offset of staged row i
            int sy = y0 + i - L::PAD;
            sy += (sy < 0) ? H : 0;
            sy -= (sy >= H) ? H : 0;
            return 4u * (uint32_t)sy * (uint32_t)W;
        };
        f4 v[NQ], r[IR > 0 ? IR : 1];
        const uint32_t oc = (REST >= 0 || g0 < L::PX) ? column(g0) : NONE;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[q][e] = (4 * q + e >= I0 && 4 * q + e < I1)
                              ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(pa, (int)oc, (int)row(4 * q + e), 0))
                              : 0.f;
        if constexpr (REST > 0) {
#pragma unroll
            for (int it = 0; it < IR; ++it) {
                const int i = g0 + 64 * it, q = i / REST, xx = 64 + i - q * REST;
                const uint32_t o = column(xx);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = 4 * q + e;
                    r[it][e] = pld(pa, (i < NQ * REST && k >= I0 && k < I1) ? o + row(k) : NONE);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (REST >= 0 || g0 < L::PX) *reinterpret_cast<f4*>(own + g0 * L::PITCH + 4 * q) = v[q];
            most = fmaxf(fmaxf(most, fmaxf(v[q][0], v[q][1])), fmaxf(v[q][2], v[q][3]));
        }
        if constexpr (REST > 0) {
#pragma unroll
            for (int it = 0; it < IR; ++it) {
                const int i = g0 + 64 * it, q = i / REST, xx = 64 + i - q * REST;
                if (i < NQ * REST) *reinterpret_cast<f4*>(own + xx * L::PITCH + 4 * q) = r[it];
                most = fmaxf(fmaxf(most, fmaxf(r[it][0], r[it][1])), fmaxf(r[it][2], r[it][3]));
            }
        }
    }
    const bool above = most > (want_flags ? wd.org_thr : wd.skip_thr);
    // Tiles where alpha = 0 everywhere, as in step_kernel: a channel whose
    // window stays at or below the threshold, or a dead gene plane 0.
    if (may_skip) {
        bool live = false;
        if (!want_flags) {
            constexpr int G1X = TX + 2, NG1 = (TY + 2) * G1X;
            const plane_t p0 = plane(wd.P, pb);
#pragma unroll
            for (int i0 = 0; i0 < NG1; i0 += NT) {
                const int i = i0 + (int)threadIdx.x;
                if (i < NG1) {
                    const int yy = i / G1X;
                    int sy = y0 + yy - 1, sx = x0 + (i - yy * G1X) - 1;
                    wrap2(sy, sx, H, W, true);
                    live = live || (pld(p0, 4u * ((uint32_t)sy * (uint32_t)W + (uint32_t)sx)) > wd.eps);
                }
            }
        }
        const int bits = (__any(above) ? (1 << ch) : 0) | (__any(live) ? 8 : 0);
        if ((threadIdx.x & 63) == 0) flags[threadIdx.x >> 6] = bits;
    }
    if constexpr (!GIVEN) __syncthreads();
    const uint32_t ob0 = 4u * ((uint32_t)gy * (uint32_t)W + (uint32_t)gx);
    f4 a;
    if constexpr (GIVEN) a = pld4(plane(wd.A + (size_t)ch * HW, pb), ob0);
#pragma unroll
    for (int e = 0; e < 4 && !GIVEN; ++e) a[e] = own[(4 * lq0 + e + L::HALO) * L::PITCH + L::PAD + ly0];
    const plane_t paout = plane(wd.A_out + (size_t)ch * HW, pb);
    const bool upd = (mode == MODE_LOCAL_UPDATE);
    if (may_skip) {
        int bits = 0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) bits |= flags[i];
        const bool dead = want_flags ? (bits & 7) == 0 : (bits & 15) != 15;
        if (listed) {
            if constexpr (!EARLY) {
                if (dead) {
                    was_zero = wd.p_zero[tile] != 0;
                    __syncthreads();   // every thread has read the byte
                }
            }
            if (threadIdx.x == 0) wd.p_zero[tile] = dead ? 1 : 0;
        }
        if (dead) {
            // A' = clip01(A), P' = 0 (left alone where the output holds 0 already)
            const f4 z = {0.f, 0.f, 0.f, 0.f};
            pst4(paout, ob0, f4{clip01(a[0]), clip01(a[1]), clip01(a[2]), clip01(a[3])});
            if (!was_zero) {
#pragma unroll
                for (int i = 0; i < NPG / T::C; ++i)
                    pst4_rows(lines, plane(wd.P_out + (size_t)(ch * (NPG / T::C) + i) * HW, pb), ob0, z);
            }
            if (ch == 0) {
                const uint32_t none = 0;
                if (wd.alpha_save) __builtin_memcpy(wd.alpha_save + (ob0 >> 2), &none, 4);
                if (wd.flags_out) __builtin_memcpy(wd.flags_out + (ob0 >> 2), &none, 4);
            }
            return;
        }
    }

    // 2. potentials of the kernels reading channel ch, four cells of column cx
    // from row cy (of the quad, where they are given)
    if constexpr (GIVEN) {
        const uint32_t spack = (ch == 0) ? pack_sources<T>(0) : (ch == 1) ? pack_sources<T>(1) : pack_sources<T>(2);
        f4 u[KPS];
#pragma unroll
        for (int j = 0; j < KPS; ++j) {
            const plane_t pu = plane(U + (size_t)nibble(spack, j) * HW, pb);
            u[j] = lines ? pld4_stream(pu, ob0) : pld4(pu, ob0);
        }
        bool ok[4] = {true, true, true, true};
#pragma unroll
        for (int j = 0; j < KPS; ++j) {
            *reinterpret_cast<f4*>(own + j * CELLS + 4 * g0) = u[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) ok[e] = ok[e] && (u[j][e] > wd.eps);
        }
        // bit g of word e: every potential of the quad's cell e above the cutoff
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t m = __ballot(ok[e]);
            if (g0 == 0) above_eps[ch * 4 + e] = m;
        }
    } else {
        const int cx = g0 % TX, cy = 4 * (g0 / TX);
        float u[KPS][4];
        quad_potentials<T, R, L::PITCH, FEW>(own + (cx + L::HALO) * L::PITCH + cy, (cfloat*)wd.shc + ch * KPS * 8, u);
        if (wd.U_save) {
            const uint32_t o = 4u * ((uint32_t)(y0 + cy) * (uint32_t)W + (uint32_t)(x0 + cx));
#pragma unroll
            for (int j = 0; j < KPS; ++j) {
                const int k = (ch == 0) ? T::kidx[0][j] : (ch == 1) ? T::kidx[1][j] : T::kidx[2][j];
                const plane_t pu = plane(wd.U_save + (size_t)k * HW, pb);
#pragma unroll
                for (int e = 0; e < 4; ++e) pst(pu, o + 4u * (uint32_t)e * (uint32_t)W, u[j][e]);
            }
        }
        if (mode == MODE_POTENTIALS) return;
        // hand them over through the channel's region, whose taps only this wave
        // reads and no longer needs
#pragma unroll
        for (int j = 0; j < KPS; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) own[j * CELLS + (cy + e) * TX + cx] = u[j][e];
        // bit g of word e: every potential of cell (cy + e, cx) above the cutoff
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bool ok = true;
#pragma unroll
            for (int j = 0; j < KPS; ++j) ok = ok && (u[j][e] > wd.eps);
            const uint64_t m = __ballot(ok);
            if (g0 == 0) above_eps[ch * 4 + e] = m;
        }
    }
    __syncthreads();

    // 3. genes, growth and update of the kernels writing channel ch
    // The gene planes of the kernels writing channel ch, kernel by kernel (m, s,
    // h), AHEAD planes' reads in flight ahead of the one being reduced.
    const uint32_t kpack = (ch == 0) ? pack_kernels<T>(0) : (ch == 1) ? pack_kernels<T>(1) : pack_kernels<T>(2);
    const uint32_t ppack = (ch == 0) ? pack_positions<T>(0) : (ch == 1) ? pack_positions<T>(1) : pack_positions<T>(2);
    constexpr int NPL = 3 * KPS, AHEAD = FEW ? 4 : 2, NB = AHEAD + 1;
    // the quad's place is formed again: kept over the walk it takes registers that
    // the walk holds its reads ahead in (4096^2, 6 dense steps: 11.5 ms, 11.05 so)
    int tid = (int)threadIdx.x;
    if constexpr (EARLY) asm volatile("" : "+v"(tid));
    const int g = tid - ch * G, ly = g / (TX / 4), lq = g % (TX / 4);
    const bool first = (lq == 0), last = (lq == TX / 4 - 1);
    const Around at = around<TX>(y0 + ly, x0 + 4 * lq, lq, H, W);
    const uint32_t ob = at.c;
    QuadDisk v[NB];
    auto load = [&](int t) {
        const plane_t pl = plane(wd.P + (size_t)((t % 3) * NK + nibble(kpack, t / 3)) * HW, pb);
        QuadDisk& q = v[t % NB];
        q.u = pld4(pl, at.u);
        q.c = pld4(pl, ob);
        q.d = pld4(pl, at.d);
        q.e = pld(pl, at.e);
    };
    auto u_of = [&](int pos) {
        const int s = (pos * 13) >> 6;   // pos / 5 for pos < 15
        return *reinterpret_cast<const f4*>(sA + s * REGION + (pos - s * KPS) * CELLS + 4 * g);
    };
    static_assert(KPS == 5, "pos / 5");
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    int alpha = 15;
    if (upd) {
        // alpha needs every potential above the cutoff; a quad where none of
        // the four has it reads no genes, unless a quad beside it does (which
        // takes its end cells from this lane)
        int ualpha = 0;
        if constexpr (GIVEN) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                ualpha |= (int)(((above_eps[e] & above_eps[4 + e] & above_eps[8 + e]) >> g) & 1) << e;
        } else {
            const uint64_t um = above_eps[ly & 3] & above_eps[4 + (ly & 3)] & above_eps[8 + (ly & 3)];
            ualpha = (int)(um >> ((ly >> 2) * TX + 4 * lq)) & 15;
        }
        const bool reads = (ualpha | __builtin_amdgcn_update_dpp(0, ualpha, kLaneBefore, 0xf, 0xf, false) |
                            __builtin_amdgcn_update_dpp(0, ualpha, kLaneAfter, 0xf, 0xf, false)) != 0;
        float dm[4];   // running minimum of the diffused genes (0: alpha fails)
#pragma unroll
        for (int e = 0; e < 4; ++e) dm[e] = (ualpha & (1 << e)) ? 3.0e38f : 0.f;
        if (reads) {
            // A kernel's genes are stored while alpha holds for what has been
            // read; cells whose alpha fails later are cleared at the end.
            const float cs = wd.cnt_scale, ncs = wd.cnt_bias, eps = wd.eps;
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) load(t);
            float gene[3][4];
#pragma unroll
            for (int t = 0; t < NPL; ++t) {
                if (t + AHEAD < NPL) load(t + AHEAD);
                __builtin_amdgcn_sched_barrier(0);
                float n[4];
                diffuse_quad<TX / 4>(v[t % NB], first, last, cs, ncs, gene[t % 3], n);
#pragma unroll
                for (int e = 0; e < 4; ++e) dm[e] = fminf(fminf(dm[e], gene[t % 3][e]), n[e]);
                if (t % 3 == 2) {
                    const int j = t / 3, k = nibble(kpack, j);
                    const f4 u = u_of(nibble(ppack, j));
#pragma unroll
                    for (int p = 0; p < 3; ++p) {
                        f4 x;
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = (dm[e] > eps) ? gene[p][e] : 0.f;
                        pst4_rows(lines, plane(wd.P_out + (size_t)(p * NK + k) * HW, pb), ob, x);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum[e] = growth_acc(sum[e], u[e], gene[0][e], gene[1][e], gene[2][e]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        int m = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) m |= (dm[e] > wd.eps) ? (1 << e) : 0;
        masks[threadIdx.x] = m;
        __syncthreads();
        alpha = masks[g] & masks[G + g] & masks[2 * G + g];
        if (alpha != 15) {
            // genes masked to 0: whole quads, or single cells (those whose
            // potentials failed were stored as 0 above).  Unrolled, a lane's other
            // cells past the plane (dropped): as a loop that branches on each cell
            // it kept small worlds waiting (96^2 with blobs 18.4 us a step, 17.8 so;
            // 256^2 16.9 and 16.4).
            const bool whole = !reads || (alpha == 0 && ualpha != 0);
            const int late = whole ? 0 : ualpha & ~alpha;
            const auto gene_plane = [&](int t) {
                return plane(wd.P_out + (size_t)((t % 3) * NK + nibble(kpack, t / 3)) * HW, pb);
            };
            if (whole) {
#pragma unroll
                for (int t = 0; t < 3 * KPS; ++t) pst4_rows(lines, gene_plane(t), ob, f4{0.f, 0.f, 0.f, 0.f});
            }
            if (late != 0) {
                constexpr uint32_t NONE = 0xFFFFFFF0u;
                uint32_t oc[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) oc[e] = (late & (1 << e)) ? ob + 4u * e : NONE;
#pragma unroll
                for (int t = 0; t < 3 * KPS; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (GIVEN && !STREAM)
                            pst(gene_plane(t), oc[e], 0.f);
                        else
                            pst_stream(gene_plane(t), oc[e], 0.f);
                    }
            }
        }
        if (ch == 0 && wd.flags_out) {
            float su[4] = {0.f, 0.f, 0.f, 0.f};
            static_for<0, NK>([&](auto kc) {
                const f4 u = u_of(position_of<T>(decltype(kc)::value));
#pragma unroll
                for (int e = 0; e < 4; ++e) su[e] += u[e];
            });
            uint32_t f = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                f |= (uint32_t)(((alpha >> e) & 1) | ((su[e] > wd.eps) ? 2 : 0)) << (8 * e);
            __builtin_memcpy(wd.flags_out + (ob >> 2), &f, 4);
        }
    } else if (mode == MODE_LOCAL_READONLY) {
#pragma unroll
        for (int j = 0; j < KPS; ++j) {
            const int k = nibble(kpack, j);
            const f4 u = u_of(nibble(ppack, j));
            const f4 m = pld4(plane(wd.P + (size_t)k * HW, pb), ob);
            const f4 s = pld4(plane(wd.P + (size_t)(NK + k) * HW, pb), ob);
            const f4 h = pld4(plane(wd.P + (size_t)(2 * NK + k) * HW, pb), ob);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = growth_acc(sum[e], u[e], m[e], s[e], h[e]);
        }
    } else {
        static_for<0, NK>([&](auto pc) {
            constexpr int pos = decltype(pc)::value, k = T::kidx[pos / KPS][pos % KPS];
            if (T::dst[k] == ch) {
                const f4 u = u_of(pos);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] = growth_acc(sum[e], u[e], wd.gm[k], wd.gs[k], wd.gh[k]);
            }
        });
    }
    if (ch == 0 && wd.alpha_save) {
        const uint32_t f = (uint32_t)(alpha & 1) | (uint32_t)(alpha & 2) << 7 | (uint32_t)(alpha & 4) << 14 |
                           (uint32_t)(alpha & 8) << 21;
        __builtin_memcpy(wd.alpha_save + (ob >> 2), &f, 4);
    }
    f4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = clip01(fmaf(wd.dt, (alpha & (1 << e)) ? sum[e] : 0.f, a[e]));
    pst4(paout, ob, out);
}

template <class T, int R, int TY, int TX>
struct QuadShared {
    using L = QuadTile<T, R, TY, TX>;
    __attribute__((aligned(16))) float sA[T::C * L::REGION];
    int masks[L::NT];
    int flags[L::NT / 64];
    uint64_t above_eps[T::C * 4];
};

template <class T, int R, int TY, int TX, bool FEW>
__global__ __launch_bounds__((QuadTile<T, R, TY, TX>::NT), (FEW ? 2 : 3)) void quad_step_kernel(WorldArgs wd, int mode)
{
    __shared__ QuadShared<T, R, TY, TX> sh;
    quad_tile<T, R, TY, TX, FEW>(wd, xcd_tile(blockIdx.x, gridDim.x), mode, sh.sA, sh.masks, sh.flags, sh.above_eps);
}

template <class T, int R, int TY, int TX>
__global__ __launch_bounds__((QuadTile<T, R, TY, TX>::NT), 3) void quad_batch_kernel(BatchList bl, int mode)
{
    __shared__ QuadShared<T, R, TY, TX> sh;
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
    quad_tile<T, R, TY, TX, false>(wd, tile, mode, sh.sA, sh.masks, sh.flags, sh.above_eps);
}

// The rest of a step whose potentials are given, bound by memory traffic (111
// planes; 90 us at 1024^2, 5.2 TB/s, where one cell per lane took 123).  The
// potentials are not needed again.
template <class T, bool STREAM>
__global__ __launch_bounds__(192, 4) void quad_given_kernel(WorldArgs wd, const float* U, int mode)
{
    constexpr int TY = 4, TX = 64;
    __shared__ __attribute__((aligned(16))) float sU[T::NK * TY * TX];
    __shared__ int masks[192];
    __shared__ uint64_t above_eps[T::C * 4];
    quad_tile<T, 12, TY, TX, false, true, STREAM>(wd, xcd_tile(blockIdx.x, gridDim.x), mode, sU, masks, nullptr, above_eps, U);
}

bool step_exceeds_caches(const WorldArgs& w) { return 111.0 * 4.0 * w.H * w.W > (double)(256 << 20); }

// Past the caches where the step exceeds them and rows are whole lines (1024^2, the
// step with its transforms: 208 us, 216 through them), else through them: the next
// step finds there what this one wrote (four steps of 512^2 302 -> 281 us, of 384^2
// 273 -> 257, from blobs 271 -> 253; with a kernel of its own each, as either kind
// of store alone takes 76 registers, a choice between them 125).
hipError_t launch_quad_given(const WorldArgs& w, const float* U, int mode, hipStream_t s)
{
    WorldArgs a = w;
    a.tiles_x = (w.W + 63) / 64;
    a.n_tiles = (w.H + 3) / 4 * a.tiles_x;
    if (step_exceeds_caches(w) && w.W % 32 == 0)
        hipLaunchKernelGGL((quad_given_kernel<Table3x15, true>), dim3(a.n_tiles), dim3(192), 0, s, a, U, mode);
    else
        hipLaunchKernelGGL((quad_given_kernel<Table3x15, false>), dim3(a.n_tiles), dim3(192), 0, s, a, U, mode);
    return hipGetLastError();
}

// At most one workgroup per compute unit: a SIMD then runs one wave, and nothing but
// the wave's own reads ahead hides their latency.  FEW keeps four gene planes in
// flight instead of two and lets the walk's reads move across its steps (167 VGPRs,
// within the three waves' budget all the same).
constexpr int kFewTiles = 256;

template <class T, int R, int TY, int TX>
hipError_t launch_quad_step(const WorldArgs& w, int mode, hipStream_t s)
{
    constexpr int NT = QuadTile<T, R, TY, TX>::NT;
    if (w.n_tiles <= kFewTiles)
        hipLaunchKernelGGL((quad_step_kernel<T, R, TY, TX, true>), dim3(w.n_tiles), dim3(NT), 0, s, w, mode);
    else
        hipLaunchKernelGGL((quad_step_kernel<T, R, TY, TX, false>), dim3(w.n_tiles), dim3(NT), 0, s, w, mode);
    return hipGetLastError();
}

template <class T, int R, int TY, int TX>
hipError_t launch_quad_batch(const BatchList& b, int mode, hipStream_t s)
{
    if (b.n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL((quad_batch_kernel<T, R, TY, TX>), dim3(b.n_items), dim3(QuadTile<T, R, TY, TX>::NT), 0, s, b, mode);
    return hipGetLastError();
}

struct QuadEntry {
    int R, ty, tx;
    step_launch_fn step;
    batch_launch_fn batch;
};

#define LENIA_QUAD_ENTRY(RR, TYY, TXX)                                                                      \
    {RR, TYY, TXX, &launch_quad_step<Table3x15, RR, TYY, TXX>, &launch_quad_batch<Table3x15, RR, TYY, TXX>}

static const QuadEntry kQuadEntries[] = {
    LENIA_QUAD_ENTRY(12, 4, 64),
    LENIA_QUAD_ENTRY(12, 8, 32),
    LENIA_QUAD_ENTRY(13, 4, 64),
    LENIA_QUAD_ENTRY(13, 8, 32),
};

static const QuadEntry* find_quad(int table, int R, int ty, int tx)
{
    for (const QuadEntry& e : kQuadEntries)
        if (table == TABLE_3x15 && e.R == R && e.ty == ty && e.tx == tx) return &e;
    return nullptr;
}

bool quad_fits(int R, int ty, int tx, int H, int W) { return H >= ty && H >= R && W >= tx; }

step_launch_fn find_quad_step_launcher(int table, int R, int ty, int tx)
{
    const QuadEntry* e = find_quad(table, R, ty, tx);
    return e ? e->step : nullptr;
}

batch_launch_fn find_quad_batch_launcher(int table, int R, int ty, int tx)
{
    const QuadEntry* e = find_quad(table, R, ty, tx);
    return e ? e->batch : nullptr;
}

}  // namespace lenia
