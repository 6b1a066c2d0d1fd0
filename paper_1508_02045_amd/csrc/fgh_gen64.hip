// fgh_gen64.hip -- the run-time-length passes in double precision and their tile choice.
#include "fgh_gen_launch.hpp"

#include <algorithm>

namespace fgh {

FGH_GEN_INSTANTIATE(double)

namespace {

// Dense products of a tile of `lines` lines of length q p, and the wavefronts that share them.
struct Dense {
    int items, ni, waves;
    double eff;  // the share of product columns that are in use
};
Dense dense_of(const Axis& ax, int lines)
{
    Dense r;
    const int h = (ax.p - 1) / 2;
    const int nrt = (h + 16) / 16, ncol = ax.q * lines, nct = (ncol + 15) / 16;
    r.items = nrt * nct;
    r.ni = (r.items + 7) / 8;
    r.waves = std::min(8, std::max(4, (r.items + r.ni - 1) / r.ni));
    r.eff = (double)ncol / (16.0 * nct);
    return r;
}

// One candidate tile: `lines` lines in LDS, `blocks` workgroups in the launch.  The score weighs what
// bounds a pass: enough workgroups for the 256 compute units (two each), LDS that lets several
// share one, dense columns in use, and the cache lines of a tile's row segment (seg bytes).
//
// scarce: no width of the pass gives each unit two workgroups.  A dense step is then scored against
// one workgroup per unit, and its LDS counts only where it keeps workgroups waiting: one column per
// workgroup left a third of the 16-wide dense columns empty and shared units unevenly.  FP64 middle
// pass, before and after: 1023 x 767 41.6 -> 32.0 us (1 -> 2 columns), 999 x 999 44.3 -> 35.6 us.
// Where two workgroups per unit can be had the rule stays as it was: 93^3 slows from 19.4 to 24.4 us
// with the other one; so it does for lengths that are one dense step (q = 1), where the other goes
// either way (667 x 211 166 -> 170 us, 1021 x 1021 352 -> 337 us).
void consider(GenTile* best, double* score, const Axis& ax, int n, int lines, size_t lds, long long blocks, size_t seg,
              bool scarce = false)
{
    if (lds + kLdsStatic > kLdsPerUnit) return;
    GenTile t{true, n, 0, 0, lds};
    scarce = scarce && ax.p > kGenRadix && ax.q > 1;
    double s = std::min(1.0, (double)blocks / (scarce ? 256.0 : 512.0));
    if (ax.p <= kGenRadix) {
        if (ax.q * lines > 256) return;  // one step-A subsequence per thread
        t.threads = std::min(256, std::max(64, (std::max(ax.q, ax.p) * lines + 63) / 64 * 64));
    } else {
        const Dense d = dense_of(ax, lines);
        if (d.ni > kGenMaxItems) return;
        t.ni = d.ni;
        t.threads = 64 * d.waves;
        s *= d.eff;
    }
    if (!scarce || blocks > 256 * (long long)(kLdsPerUnit / lds))
        s *= lds <= 40 * 1024 ? 1.0 : lds <= 54 * 1024 ? 0.95 : lds <= 80 * 1024 ? 0.85 : 0.6;
    s *= seg >= 128 ? 1.0 : seg >= 64 ? 0.9 : seg >= 32 ? 0.75 : 0.6;
    s *= 1.0 - 0.3 / lines;  // the twiddle table each workgroup loads
    if (s > *score) {
        *score = s;
        *best = t;
    }
}

}  // namespace

GenTile gen_row_tile(const Axis& ax, int d, long long rows, size_t cs, int cap)
{
    GenTile best{};
    double score = 0.0;
    const size_t tab = 2 * kMaxPhases * 6 * (cs / 2);
    for (int r : {32, 24, 20, 16, 14, 12, 10, 8, 6, 4, 2, 1}) {  // even: rows pair into complex rows alike
        if ((r > rows && r > 2) || r > cap) continue;
        const int npen = (r * d + 1) / 2;
        consider(&best, &score, ax, r, npen, (size_t)(ax.L + (size_t)npen * ax.L) * cs + tab, (rows + r - 1) / r, 128);
    }
    return best;
}

GenTile gen_axis_tile(const Axis& ax, int inner, long long outer, size_t cs)
{
    GenTile best{};
    double score = 0.0;
    for (int P = 16; P >= 1; P--) {
        if (P > inner) continue;
        const long long nt = (inner + P - 1) / P;
        GenTile b = best;
        double s = score;
        consider(&b, &s, ax, P, P, (size_t)(ax.L + (size_t)P * ax.L) * cs, nt * outer, P * cs);
        // a ragged last tile leaves lanes idle
        const double fill = (double)inner / (double)(nt * P);
        if (b.ok && s * fill > score) {
            best = b;
            score = s * fill;
        }
    }
    return best;
}

GenTile gen_mid_tile(const Axis& ax, int cols, size_t cs)
{
    GenTile best{};
    double score = 0.0;
    for (int P : {16, 12, 8, 7, 6, 5, 4, 3, 2, 1}) {
        if (P > cols) continue;
        consider(&best, &score, ax, P, 2 * P, (size_t)(ax.L + 2 * (size_t)P * ax.L) * cs, (cols + P - 1) / P, P * cs,
                 cols < 512);
    }
    return best;
}

}  // namespace fgh
