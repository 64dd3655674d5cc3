// Plan of the fp32 raw-row kernel (conv_rows.hip): how a layer is cut into workgroups and chunks, and where things lie in LDS.  Host code only.
#pragma once

#include "internal.h"

#include <algorithm>
#include <cmath>

namespace dp {

constexpr int cr_qmax(int k) { return k == 5 ? 2 : 4; }
constexpr int CR_PIECES = 4;                    // 16-byte pieces a thread moves per chunk

struct RowsPlan {
    int nm, nn, tiles_m, tiles_n, q, rows, chunks, rpr, xp, cha, chx, bufs, waves_a, ex_per_wg;
    int tail;                       // dword of LDS where the table of runs starts, then 16 partial norms; chunks and epilogue lie before it
    unsigned lds;
    double us;                      // estimated time of a call alone
    bool ok;
};

inline int odd_quads(int floats) { const int v = (floats + 3) / 4; return (v | 1) * 4; }     // consecutive channels start in different banks

// us of a per-example call alone.  A launch lasts as long as the compute unit with most blocks, which takes them in rounds of as many
// workgroups as it has room for.  Chunk by chunk a round needs the longer of two things (a little more where they are close): what
// the SIMD with most waves issues for all its workgroups -- MFMAs and vector instructions take turns on a SIMD, and the waves of every
// workgroup start on the same one, so K q waves count as ceil(K q / 4) on it --, or one workgroup's own chain of barrier, loads, staging and
// MFMAs.  Constants (cycles; per kernel size and stride) fitted to 4223 launches of 181 layers with forced plans: the plan it prefers is 3.5 %
// slower than the best one on average.
inline double rows_us(int k, int s, const RowsPlan &p, double blocks, int unit, int groups, long long pieces, bool ragged, int resident)
{
    struct Fit { double mfma, vector, group, slot, ragged, chunk, chain, finish, block, launch, lone; };
    static const Fit fits[2][2] = {{{0.56, 0.33, 175.0, 304.0, 135.0, 2415.0, 0.0, 7000.0, 357.0, 3.7, 595.0}, {0.7, 0.0, 47.0, 278.0, 73.0, 2472.0, 411.0, 13240.0, 254.0, 3.1, 198.0}},
                                   {{1.19, 0.0, 0.0, 194.0, 75.0, 1893.0, 0.0, 24200.0, 0.0, 2.6, 1617.0}, {1.11, 0.0, 0.0, 213.0, 78.0, 2432.0, 0.0, 21070.0, 206.0, 1.9, 289.0}}};
    const Fit &c = fits[k / 2 - 1][s - 1];
    const int turns = (groups + p.q - 1) / p.q;
    const double group = p.nm * p.nn * k * 6 * 18.8 * c.mfma + (24 * p.nn * s + 4 * p.nm * p.nn * k) * 2.65 * c.vector + c.group;
    const double staging = (double)pieces / (64 * k * p.q) * (c.slot + (ragged ? c.ragged : 0.0)), chunks = (double)p.chunks * unit;
    const auto round = [&](double r) {
        if (r <= 0.0) return 0.0;
        const double all = r * ((k * p.q + 3) / 4) * (turns * group + staging), own = c.chunk + turns * (group + c.chain) + staging + (p.bufs == 1 ? c.lone : 0.0);
        return chunks * std::cbrt(all * all * all + own * own * own) + (c.finish + c.block * p.nm * p.nn * k * (p.q + 1)) * (0.6 + 0.4 * r);
    };
    const double most = std::ceil(blocks / 256.0), r = std::min<double>(most, resident), full = std::floor(most / r);
    return c.launch + (full * round(r) + round(most - full * r)) / 2400.0;
}

// Blocks of 16 channels that a workgroup takes of `c` channels (5 x 5: one of input channels, five accumulators a block).
inline int rows_nm(const Geo &g) { return g.cout > 16 ? 2 : 1; }
inline int rows_nn(const Geo &g) { return g.kh == 3 && g.cin > 16 ? 2 : 1; }

inline RowsPlan rows_plan(const Geo &g, bool shared)
{
    RowsPlan best = {}, p = {};
    const int K = g.kh, S = g.stride;
    p.nm = rows_nm(g);
    p.nn = rows_nn(g);
    const int CO = 16 * p.nm, CI = 16 * p.nn;
    p.rpr = (g.ow + 7) / 8;
    p.xp = 12 * S * (p.rpr + 1);                // a run reads sixteen numbers
    p.tiles_m = (g.cout + CO - 1) / CO;
    p.tiles_n = (g.cin + CI - 1) / CI;
    const int lc = g.cout < CO ? g.cout : CO, ln = g.cin < CI ? g.cin : CI;      // channels that are staged
    const double own = (double)(g.n / g.unit) * p.tiles_m * p.tiles_n;
    // Inside a batch call of several layers the plan with the best rate of a full chip, eight blocks on every compute unit, whatever
    // this layer brings: the other layers' workgroups run on the units beside its own.  ResNet-20, 256 examples on eight streams: 758 us
    // as alone, 641 so; 4 x 32: 473, 393.
    const double blocks = shared ? 8.0 * 256.0 : own;
    // several examples in a row where there are far more (example, block) pairs than workgroups that run at a time
    const int e = (int)(own / 4096.0);
    p.ex_per_wg = g.unit * (e < 1 ? 1 : e > 8 ? 8 : e);
    for (p.q = 1; p.q <= cr_qmax(K); ++p.q)
        for (p.rows = 1; p.rows <= g.oh && p.rows <= 64; ++p.rows) {
            const int lines = (p.rows - 1) * S + K;
            if (lines > 127) break;
            const long long pieces_a = (long long)lc * p.rows * ((g.ow + 3) / 4), pieces_x = (long long)ln * lines * ((g.w + 3) / 4), pieces = pieces_a + pieces_x;
            // waves in proportion to the pieces
            const int waves = K * p.q;
            p.waves_a = std::min<long long>(std::max<long long>((pieces_a * waves + pieces / 2) / pieces, 1), waves - 1);
            if (pieces_a > CR_PIECES * 64ll * p.waves_a) ++p.waves_a;
            if (p.waves_a == waves || pieces_a > CR_PIECES * 64ll * p.waves_a || pieces_x > CR_PIECES * 64ll * (waves - p.waves_a)) {
                if (pieces > CR_PIECES * 64ll * waves) break;
                continue;
            }
            const int groups = (p.rows * p.rpr + 3) / 4;
            p.cha = odd_quads(groups * 48);
            p.chx = odd_quads(lines * p.xp);
            const long long chunk = (long long)CO * p.cha + (long long)CI * p.chx;
            if (chunk > 0xffff) break;
            p.chunks = (g.oh + p.rows - 1) / p.rows;
            for (p.bufs = 1; p.bufs <= 2; ++p.bufs) {
                // the epilogue's block or bias sums may need more than the chunks whose place they take
                p.tail = (int)std::max<long long>({p.bufs * chunk, p.q * 16ll * (CI * K * K + 2), CR_PIECES * 64ll * p.waves_a});
                // LDS in a few even shares of what a compute unit has: layers of different sizes share a launch
                const unsigned need = (unsigned)(p.tail + groups * 4 + 16) * 4;
                if (need > 156 * 1024) break;
                p.lds = 156 * 1024;
                for (int share : {2, 3, 4, 6, 8})
                    if (need <= (unsigned)(156 / share * 1024)) p.lds = 156 / share * 1024;
                const int resident = std::max(1, std::min({(int)(156 * 1024 / p.lds), 12 / (K * p.q), 8}));
                p.us = rows_us(K, S, p, blocks, g.unit, groups, pieces, g.w % 4 || g.ow % 4, resident);
                p.ok = true;
                if (!best.ok || p.us < best.us) best = p;
            }
        }
    return best;
}

}  // namespace dp
