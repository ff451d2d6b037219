// Ring decomposition of the disk |d| < R into 2R rings (Section 2.4): compile-time
// tables of its orbits and rings (internal).
#pragma once

namespace lenia {

struct RingOrbit {
    int a, b, ring;   // representative offset (a, b), 0 <= b <= a
};

// floor(NR sqrt(d2) / R) in integers
constexpr int ring_of_d2(int R, int NR, int d2)
{
    int j = 0;
    while ((j + 1) * (j + 1) * R * R <= NR * NR * d2) ++j;
    return j;
}

template <int R>
struct RingTables {
    static constexpr int NR = 2 * R;
    static constexpr int NO = [] {
        int n = 0;
        for (int a = 0; a < R; ++a)
            for (int b = 0; b <= a; ++b)
                if (a * a + b * b < R * R) ++n;
        return n;
    }();
    RingOrbit orb[NO];    // in ring order (centre first)
    int slot[NR];         // ring -> index among the non-empty rings, or -1
    int ring_of_slot[NR];
    int size_of_slot[NR];
    int nre;              // number of non-empty rings
};

template <int R>
constexpr RingTables<R> make_ring_tables()
{
    RingTables<R> t{};
    constexpr int NR = RingTables<R>::NR;
    int size[NR] = {};
    for (int dy = -R; dy <= R; ++dy)
        for (int dx = -R; dx <= R; ++dx)
            if (dy * dy + dx * dx < R * R) ++size[ring_of_d2(R, NR, dy * dy + dx * dx)];
    t.nre = 0;
    for (int j = 0; j < NR; ++j) {
        t.slot[j] = -1;
        if (size[j] > 0) {
            t.slot[j] = t.nre;
            t.ring_of_slot[t.nre] = j;
            t.size_of_slot[t.nre] = size[j];
            ++t.nre;
        }
    }
    int n = 0;
    for (int j = 0; j < NR; ++j)
        for (int a = 0; a < R; ++a)
            for (int b = 0; b <= a; ++b)
                if (a * a + b * b < R * R && ring_of_d2(R, NR, a * a + b * b) == j) t.orb[n++] = {a, b, j};
    return t;
}

template <int R>
inline constexpr RingTables<R> kRings = make_ring_tables<R>();

}  // namespace lenia
