// The FP32 tiles' decisions on the host's tables: every way a pair can be
// called certain (its column's slot, one edge, a few edges, its cell) is
// formed here from the tables with a squared distance that is off by up to
// its error bound, and has to give the slot of the exact distance's band.
// Edges of all kinds, first edges at 0 and below the FP32 band among them;
// columns at the rows' mean.  Prints the number of decisions.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <vector>

#include "edges.h"
#include "internal.h"

using namespace tpcf;

static uint32_t bits(float f) {
    uint32_t b;
    memcpy(&b, &f, 4);
    return b;
}

struct Tables {
    int ne = 0, q_exp = 0;
    Band32 band;
    CellTable cells;
    std::vector<float> slots, edges;
};

static Tables tables(int metric, const std::vector<double> &e, double extent, int max_cells) {
    Tables t;
    EdgeTables et;
    std::string why;
    const int nbins = (int)e.size() - 1;
    if (!(metric ? compile_edges_3d(e.data(), nbins, &et, &why) : compile_edges(e.data(), nbins, &et, &why))) {
        printf("edges: %s\n", why.c_str());
        exit(1);
    }
    t.ne = nbins + 1;
    t.band = metric ? make_band32_3d(et, extent) : make_band32(et, extent);
    uint32_t top = metric ? qtop_key_3d(extent) : qtop_key(extent);
    t.q_exp = tile_scale_exp(metric, extent);
    scale_band32(2 * t.q_exp, &t.band, &top);
    t.cells = make_cells_tiles(et, t.band, top, max_cells);
    // the FP64 path has a table of the same edges
    const CellTable c = make_cells64(et, max_cells, metric ? fmax(4.0 * extent * extent * 1.001, 1e-300) : 2.0);
    if (c.lo > c.hi || (int)c.cells.size() != c.hi - c.lo + 1) {
        printf("FP64 cells %d to %d: %zu\n", c.lo, c.hi, c.cells.size());
        exit(1);
    }
    make_tile_tables(t.band, &t.slots, &t.edges);
    return t;
}

// Slot of a squared distance of the FP32 copies, -1 inside a band.
static int slot_of(const Tables &t, double q) {
    int lo = 0, hi = 0;
    for (int k = 0; k < t.ne; ++k) {
        lo += q >= (double)t.band.qhi[k];
        hi += !(q < (double)t.band.qlo[k]);
    }
    return lo == hi ? lo : -1;
}

struct Entry {
    int slot;           // the lower one of an open cell, 0 with several edges
    bool open, multi;
};

static Entry entry(const Tables &t, float q) {
    int32_t b = (int32_t)bits(q) >> t.cells.shift;
    b = b < t.cells.lo ? t.cells.lo : b > t.cells.hi ? t.cells.hi : b;
    const uint16_t v = t.cells.cells[(size_t)(b - t.cells.lo)];
    if (v == kMulti)
        return {0, true, true};
    return {v & 0x7FFF, (v & kMedium) != 0, false};
}

static const float u = 5.9604644775390625e-08f;
static long long decisions = 0;

static bool wrong(const char *way, const Tables &t, float nb, double q, float qh, float e, int slot) {
    ++decisions;
    const int want = slot_of(t, q);
    if (slot == want)
        return false;
    printf("%s: column at %g, q = %.9g (%.9g within %g): slot %d, band %d of %d edges\n", way, nb, q, qh, e, slot, want,
           t.ne);
    return true;
}

// One pair at squared distance q, known as qh within e, of a column at nb.
static bool pair(const Tables &t, float nb, double q, float qh, float e) {
    const int ne = t.ne, at = entry(t, nb).slot;
    const float *sl = &t.slots[2 * (size_t)at];
    {   // the column's slot
        const float es = fmaf(8.0f * u, fabsf(sl[0]), e);
        const float x = qh - (sl[0] + es), wd = fmaxf(fmaf(-2.0f, es, sl[1]), 0.0f);
        if (bits(x) < bits(wd) && wrong("slot", t, nb, q, qh, e, at))
            return false;
    }
    {   // the nearest edge
        const uint32_t k = nearest_edge((uint32_t)at, nb, sl[0], sl[1], (uint32_t)ne);
        if (k >= (uint32_t)ne) {
            printf("column at %g, slot %d: edge %u of %d\n", nb, at, k, ne);
            return false;
        }
        const float *ed = &t.edges[4 * (size_t)k];
        const float eh = fmaf(8.0f * u, ed[0], e), room = fminf(ed[2], fmaf(-2.0f, eh, ed[3]));
        const float x = qh - (ed[0] + eh);
        const int32_t lim = (int32_t)bits(fmaf(-2.0f, eh, -ed[1]));
        if (fabsf(x) < room && (int32_t)bits(x) > lim &&
            wrong("edge", t, nb, q, qh, e, (int)k + (bits(x) >> 31 ? 0 : 1)))
            return false;
    }
    if (!(qh * kTileFar > e) && e > 0.0f)
        return true;
    {   // the edges between two cells
        const Entry lo = entry(t, qh - e), hi = entry(t, qh + e);
        if (!lo.multi && !hi.multi) {
            int s = lo.slot;
            const int last = hi.slot + (hi.open ? 1 : 0);
            if (last > ne || lo.slot > last) {
                printf("cells of %g -+ %g: slots %d to %d of %d edges\n", qh, e, lo.slot, last, ne);
                return false;
            }
            bool open = false;
            for (int k = lo.slot; k < last; ++k) {
                const float x = qh - (t.band.qhi[k] + e);
                const int32_t lim = (int32_t)bits(fmaf(-2.0f, e, t.band.qlo[k] - t.band.qhi[k]));
                open = open || (int32_t)bits(x) <= lim;
                s += bits(x) >> 31 ? 0 : 1;
            }
            if (!open && wrong("edges", t, nb, q, qh, e, s))
                return false;
        }
    }
    {   // the pair's own cell
        const Entry c = entry(t, qh);
        if (!c.open) {
            if (wrong("cell", t, nb, q, qh, e, c.slot))
                return false;
        } else if (!c.multi) {
            const float lo = t.band.qlo[c.slot], hi = t.band.qhi[c.slot];
            if (qh - e >= hi ? wrong("cell", t, nb, q, qh, e, c.slot + 1)
                             : qh + e < lo && wrong("cell", t, nb, q, qh, e, c.slot))
                return false;
        }
    }
    return true;
}

static bool check(int metric, const std::vector<double> &edges, double extent, int max_cells, std::mt19937_64 &g) {
    const Tables t = tables(metric, edges, extent, max_cells);
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    const double S = ldexp(1.0, t.q_exp), most = 4.0 * S * S * (metric ? extent * extent : 1.0);
    // squared distances of columns and pairs: none, at and around every edge, all magnitudes, up to the largest
    std::vector<double> at{0.0, most};
    for (int k = 0; k < t.ne; ++k)
        for (double v : {(double)t.band.qlo[k], (double)t.band.qhi[k]})
            if (v > 0.0 && v < most)
                for (double f : {1.0, 1.0 - 1e-7, 1.0 + 1e-7, 0.999, 1.001, 0.8, 1.25})
                    at.push_back((double)(float)fmin(v * f, most));
    std::shuffle(at.begin() + 2, at.end(), g);      // (many edges: some of them)
    at.resize(std::min<size_t>(at.size(), 120));
    for (int i = 0; i < 40; ++i)
        at.push_back((double)(float)(most * exp(-40.0 * uni(g) * uni(g))));
    for (double nb : at)
        for (double q : at) {
            // |b| from the rows' mean, a row at |a| with |b| - |a| <= sqrt(q) <= |b| + |a| and the farthest row no
            // nearer: the derived error of q^ for that row, in the bound that the launch uses
            const double b = sqrt(nb), a = fabs(sqrt(q) - b) + 2.0 * fmin(b, sqrt(q)) * uni(g) * uni(g);
            const double rho2 = a * a * (1.0 + 3.0 * uni(g) * uni(g));
            const double off = u * (8.0 * (a + b) * (a + b) + 3.0 * nb + 48.0 * a * b + 20.0 * a * a + 2.0 * a + b + 8.0);
            const float e = u * (kTileErrN * (float)nb + (kTileErrA * (float)rho2 + kTileErr0));
            for (double f : {-1.0, 0.0, 1.0, 2.0 * uni(g) - 1.0})
                if (!pair(t, (float)nb, q, (float)(q + f * off), e))
                    return false;
            if (!pair(t, (float)nb, q, (float)q, 0.0f))      // from FP32 differences
                return false;
        }
    return true;
}

int main() {
    std::mt19937_64 g(97);
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    const double eps = ldexp(1.0, -51);
    struct Case {
        int metric;
        double extent;
        std::vector<double> edges;
    };
    std::vector<Case> cases = {
        // first edges whose band reaches 0, last edges on both sides of the points
        {1, 1.0, {1e-9, 2.0}},
        {1, 1.0, {1e-9, 0.5}},
        {1, 1.0, {0.0, 1e-9, 2.0}},
        {1, sqrt(3.0), {1e-9, 0.5, 1.5}},
        {1, sqrt(3.0), {1e-9, 0.5, 2.0}},
        {1, 1e6, {1e-3, 0.1, 50.0, 2e5}},
        // several edges in the bottom cell
        {1, 1.0, {0.0, 1e-9, 2e-9, 4e-9, 0.3, 1.1}},
        {1, 1.0, {1e-10, 1e-9, 1e-8, 1.0}},
        // ordinary ones, one bin, edges out of reach
        {1, 1000.0, {0.0, 20.0, 60.0, 110.0}},
        {1, 1000.0, {0.5, 150.0}},
        {1, 10.0, {1.0, 1e30, 1e140}},
        {1, 1e-30, {1e-33, 1e-31, 5e-31}},
        {1, 1.9e15, {1e8, 1e12, 1e15}},
        // the first edge beyond every pair, and no extent at all
        {1, 1.0, {10.0, 20.0}},
        {1, 1.0, {2.5, 1e30}},
        {1, 1.0, {0.0, 20.0, 1e140}},
        {1, 0.0, {0.0, 1.0}},
        {1, 0.0, {1e-9, 1.0}},
        {0, eps, {0.0, 180.0}},
        {0, eps, {1e-6, 90.0}},
        {0, eps, {1e-9, 1e-7, 1e-6, 1e-5, 120.0}},
        {0, ldexp(1.0, -20), {0.0, 0.01, 0.1, 179.99, 180.0}},
    };
    for (int n : {12, 40, 200, 256})
        for (int lin = 0; lin < 2; ++lin) {
            Case c{0, eps, {}}, d{1, 1000.0, {}};
            for (int k = 0; k <= n; ++k) {
                const double f = (double)k / n;
                c.edges.push_back(lin ? 1e-3 + 100.0 * f : 0.0005 * pow(60000.0, f));
                d.edges.push_back(lin ? 500.0 * f : 0.2 * pow(1000.0, f));
            }
            cases.push_back(c);
            cases.push_back(d);
        }
    for (int i = 0; i < 40; ++i) {      // a few edges of all sizes
        Case c{1, 1.0, {}};
        double e = i % 3 ? pow(10.0, -10.0 * uni(g)) : 0.0;
        for (int k = 0; k <= 1 + i % 5; ++k) {
            c.edges.push_back(e);
            e = e > 0.0 ? e * pow(10.0, 0.01 + 4.0 * uni(g)) : pow(10.0, -10.0 * uni(g));
        }
        cases.push_back(c);
    }
    for (const Case &c : cases)
        for (int cells : {2048, 12288})
            if (!check(c.metric, c.edges, c.extent, cells, g)) {
                printf("metric %d, extent %g, %zu edges from %g\n", c.metric, c.extent, c.edges.size(), c.edges[0]);
                return 1;
            }
    printf("%lld\n", decisions);
    return 0;
}
