// Host check of the tables that the march's search reads beside the planes
// (tet_build.cpp), run under the sanitizers, against brute force:
// * the float32 planes with their error bound: where they decide a point (the
//   kernels' pre-test, the same operations), the float64 planes with the tie
//   bits decide alike -- points in the part's box, on faces, and as far beyond
//   it as steps much longer than the part reach; parts far from the origin,
//   flat ones and slivers of 1e-10 of the part;
// * the cells' heads: of a cell with tetrahedra its list, of an empty one its
//   distance to the nearest cell with tetrahedra.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "tet_build.h"

using namespace dpvr;

static int g_fail = 0;
#define EXPECT(c)                                                           \
    do {                                                                    \
        if (!(c)) {                                                         \
            ++g_fail;                                                       \
            if (g_fail < 20) std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #c); \
        }                                                                   \
    } while (0)

static uint64_t g_state = 0x2545f4914f6cdd1dULL;
static double uniform() {                       // splitmix64
    uint64_t z = (g_state += 0x9e3779b97f4a7c15ULL);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    z ^= z >> 31;
    return (double)(z >> 11) * 0x1p-53;
}

static bool holds(const TetTables& t, int e, const double p[3]) {
    for (int i = 0; i < 4; ++i) {
        const double* q = &t.planes[16 * (size_t)e + 4 * i];
        const double d = ((q[0] * p[0] + q[1] * p[1]) + q[2] * p[2]) - q[3];
        if (d < 0.0 || (d == 0.0 && !((t.owned[e] >> i) & 1u))) return false;
    }
    return true;
}

// The pre-test: -1 held, 1 rejected, 0 undecided.
static int pretest(const TetTables& t, int e, const double p[3]) {
    float x[3], l[4], sum = 0.0f;
    for (int c = 0; c < 3; ++c) x[c] = (float)(p[c] - t.glo[c]);
    l[3] = 1.0f;
    for (int i = 0; i < 3; ++i) {
        const float* n = &t.planes32[12 * (size_t)e + 4 * i];
        l[i] = fmaf(n[0], x[0], fmaf(n[1], x[1], fmaf(n[2], x[2], -n[3])));
        l[3] -= l[i];
        sum = fmaf(std::fabs(n[0]), t.err32[0], fmaf(std::fabs(n[1]), t.err32[1], fmaf(std::fabs(n[2]), t.err32[2], sum)));
    }
    const float least = std::fmin(std::fmin(l[0], l[1]), std::fmin(l[2], l[3]));
    return least + sum < 0.0f ? 1 : least - sum > 0.0f ? -1 : 0;
}

static long g_decided = 0, g_held = 0;
static void check_point(const TetTables& t, int e, const double p[3]) {
    const int r = pretest(t, e, p);
    if (r == 0) return;
    ++g_decided;
    g_held += r < 0;
    EXPECT((r < 0) == holds(t, e, p));
}

static const int kPerms[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};

// The Kuhn mesh of n[0] x n[1] x n[2] cells, interior vertices jittered,
// scaled by s, turned and moved to o; the cells of the x layers that keep()
// wants.
template <typename Keep>
static void mesh(const int n[3], double jitter, const double s[3], double turn, const double o[3], Keep keep,
                 std::vector<double>& v, std::vector<int32_t>& t) {
    auto vid = [&](const int c[3]) { return (c[0] * (n[1] + 1) + c[1]) * (n[2] + 1) + c[2]; };
    v.clear();
    t.clear();
    const double a = turn, b = 0.7 * turn;
    const double m[3][3] = {{cos(a), -sin(a) * cos(b), sin(a) * sin(b)}, {sin(a), cos(a) * cos(b), -cos(a) * sin(b)},
                            {0.0, sin(b), cos(b)}};
    for (int i = 0; i <= n[0]; ++i)
        for (int j = 0; j <= n[1]; ++j)
            for (int k = 0; k <= n[2]; ++k) {
                const int c[3] = {i, j, k};
                double q[3];
                for (int d = 0; d < 3; ++d) {
                    const bool in = c[d] > 0 && c[d] < n[d];
                    q[d] = s[d] * (c[d] + (in ? jitter * (2.0 * uniform() - 1.0) : 0.0));
                }
                for (int d = 0; d < 3; ++d) v.push_back(o[d] + ((m[d][0] * q[0] + m[d][1] * q[1]) + m[d][2] * q[2]));
            }
    for (int i = 0; i < n[0]; ++i)
        for (int j = 0; j < n[1]; ++j)
            for (int k = 0; k < n[2]; ++k)
                for (const auto& pm : kPerms) {
                    if (!keep(i)) continue;
                    int c[3] = {i, j, k};
                    t.push_back(vid(c));
                    for (int d = 0; d < 3; ++d) {
                        ++c[pm[d]];
                        t.push_back(vid(c));
                    }
                }
}

static void check_heads(const TetTables& t) {
    const int gx = t.gdim[0], gy = t.gdim[1], gz = t.gdim[2];
    const long cells = (long)gx * gy * gz;
    EXPECT((long)t.cell_head.size() == 4 * (cells + 1));
    EXPECT(t.cell_head[4 * cells] == -1);
    std::vector<int> full;
    for (long c = 0; c < cells; ++c)
        if (t.cell_start[c + 1] > t.cell_start[c]) full.push_back((int)c);
    for (long c = 0; c < cells; ++c) {
        const int32_t* h = &t.cell_head[4 * c];
        const int first = t.cell_start[c], n = t.cell_start[c + 1] - first;
        if (n > 0) {
            EXPECT(h[0] == t.cell_tets[first] && h[1] == (n > 1 ? t.cell_tets[first + 1] : -1));
            EXPECT(h[2] == first + std::min(n, 2) && h[3] == first + n);
            continue;
        }
        int best = kFarMax;
        for (int f : full) {
            const int dx = std::abs(f % gx - (int)(c % gx)), dy = std::abs(f / gx % gy - (int)(c / gx % gy)),
                      dz = std::abs(f / gx / gy - (int)(c / gx / gy));
            best = std::min(best, std::max(dx, std::max(dy, dz)));
        }
        EXPECT(h[0] == -best);
    }
}

int main() {
    struct Case {
        int n[3];
        double jitter, s[3], o[3];
        int hole;                    // x layers [2, 2 + hole) are another part's
    };
    const Case cases[] = {
        {{3, 4, 2}, 0.2, {1, 1, 1}, {0, 0, 0}, 0},
        {{3, 4, 2}, 0.3, {1, 1, 1}, {3e5, -2e5, 7e4}, 0},
        {{5, 5, 5}, 0.1, {1e-3, 1, 40}, {-2, 0, 900}, 0},
        {{4, 4, 2}, 0.2, {1, 1, 1e-6}, {0, 0, 0}, 0},
        {{2, 2, 1}, 0.0, {1, 1, 1e-8}, {10, 0, 0}, 0},
        {{2, 1, 1}, 0.0, {1, 1, 1e-10}, {0, 0, 0}, 0},
        {{40, 2, 2}, 0.2, {1, 1, 1}, {0, 0, 0}, 36},
        {{24, 3, 3}, 0.2, {0.5, 2, 1}, {0, 0, 0}, 20},
    };
    for (const Case& c : cases)
        for (int turn = 0; turn < 4; ++turn) {
            std::vector<double> v;
            std::vector<int32_t> t;
            mesh(c.n, c.jitter, c.s, 0.9 * turn, c.o, [&](int i) { return i < 2 || i >= 2 + c.hole; }, v, t);
            TetTables tab;
            std::string err;
            EXPECT(build_tet_tables(v.data(), (int32_t)v.size() / 3, t.data(), (int32_t)t.size() / 4, tab, err));
            check_heads(tab);
            double X = 0.0;
            for (int d = 0; d < 3; ++d) X = std::max(X, tab.gdim[d] / tab.ginv[d]);
            for (int e = 0; e < tab.n_tets; e += std::max(1, tab.n_tets / 60)) {
                auto vertex = [&](int j, int d) { return v[3 * (size_t)t[4 * (size_t)e + j] + d]; };
                for (int q = 0; q < 120; ++q) {
                    double w[4], sum = 0.0, p[3] = {0, 0, 0};
                    for (int j = 0; j < 4; ++j) sum += w[j] = q % 5 == j ? 0.0 : uniform();
                    for (int j = 0; j < 4; ++j)
                        for (int d = 0; d < 3; ++d) p[d] += w[j] / sum * vertex(j, d);
                    check_point(tab, e, p);                       // in the tetrahedron or on a face
                    // off it: along a random edge (in a sliver's plane) or anywhere,
                    // from 1e-6 to 1e4 of the part
                    const double far = X * std::pow(10.0, 10.0 * uniform() - 6.0);
                    const int j = (int)(4.0 * uniform()), i = (j + 1 + (int)(3.0 * uniform())) & 3;
                    double dir[3], len = 0.0;
                    for (int d = 0; d < 3; ++d) {
                        dir[d] = q & 1 ? vertex(j, d) - vertex(i, d) : 2.0 * uniform() - 1.0;
                        len += dir[d] * dir[d];
                    }
                    for (int d = 0; d < 3; ++d) p[d] += far * dir[d] / std::sqrt(len);
                    check_point(tab, e, p);
                }
            }
        }
    EXPECT(g_decided > 100000 && g_held > 10000);
    // a part without tetrahedra
    TetTables tab;
    std::string err;
    EXPECT(build_tet_tables(nullptr, 0, nullptr, 0, tab, err));
    EXPECT(tab.cell_head.size() == 8 && tab.cell_head[0] == -kFarMax && tab.cell_head[4] == -1);
    std::printf("%s: %d failed expectations (%ld points decided, %ld held)\n", g_fail ? "FAIL" : "OK", g_fail,
                g_decided, g_held);
    return g_fail ? 1 : 0;
}
