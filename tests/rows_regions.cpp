// Walks sizes of the fp32 raw-row kernel and checks that the regions of LDS that its workgroups use at the same time are disjoint: the chunks,
// then in their place the rows of a block that is computed again in fp32, the shares of a 16-row block and the bias sums, must end before the
// table of runs and the partial norms.
#include "rows_plan.h"

#include <cstdio>

using namespace dp;

int main()
{
    long long plans = 0, larger = 0, several = 0, bad = 0;
    const int channels[] = {1, 3, 16, 17, 32, 40, 64, 128, 256}, heights[] = {1, 2, 3, 4, 5, 7, 8, 14, 28, 56}, widths[] = {1, 2, 3, 4, 7, 8, 9, 16, 17, 28, 56};
    for (int k : {3, 5})
        for (int stride : {1, 2})
            for (int cin : channels)
                for (int cout : channels)
                    for (int h : heights)
                        for (int w : widths)
                            for (int n : {8, 256, 2048, 32768})
                                for (int unit : {1, 4})
                                    for (bool shared : {false, true}) {
                                        Geo g = {};
                                        g.n = n; g.unit = unit; g.cin = cin; g.cout = cout; g.h = h; g.w = w;
                                        g.kh = g.kw = k; g.stride = stride; g.pad = (k - 1) / 2;
                                        g.oh = (h - 1) / stride + 1; g.ow = (w - 1) / stride + 1;
                                        const RowsPlan p = rows_plan(g, shared);
                                        if (!p.ok) continue;
                                        const int groups = (p.rows * p.rpr + 3) / 4;
                                        const long long chunks = (long long)p.bufs * 16 * (p.nm * p.cha + p.nn * p.chx);
                                        const long long block = 16ll * p.q * (16 * p.nn * k * k + 2), bias = 256ll * p.waves_a;
                                        const long long again = 16ll * p.nm * (g.ow | 1) + 16ll * p.nn * ((k * w) | 1);
                                        ++plans;
                                        larger += block > chunks || bias > chunks;
                                        several += (block > chunks || bias > chunks) && p.ex_per_wg > unit;
                                        if (chunks <= p.tail && again <= p.tail && block <= p.tail && bias <= p.tail && 4ll * (p.tail + 4 * groups + 16) <= p.lds && k * p.q <= 16) continue;
                                        if (!bad++)
                                            printf("%dx%d stride %d, %d -> %d on %d x %d, %d examples in units of %d: chunks %lld, again %lld, block %lld, bias %lld, table at %d, LDS %u bytes\n",
                                                   k, k, stride, cin, cout, h, w, n, unit, chunks, again, block, bias, p.tail, p.lds);
                                    }
    printf("%lld plans, %lld with an epilogue larger than the chunks, %lld of these for several examples, %lld overlap\n", plans, larger, several, bad);
    return bad || !several;
}
