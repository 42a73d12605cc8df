// Workgroups of a ring plan with its links in LDS (ring_lds_workgroups), on the
// host: every rank, channel and wave count, from one piece to many.
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <initializer_list>

#include "ar_internal.h"

static int failures = 0;
static void expect(bool ok, const char *what, int n, int c, int w, uint64_t pieces, uint64_t got)
{
    if (ok) return;
    if (++failures < 20)
        printf("%s: N=%d C=%d W=%d pieces=%llu -> %llu\n", what, n, c, w, (unsigned long long)pieces,
               (unsigned long long)got);
}

int main()
{
    const uint64_t piece = 1024;
    for (int n = 2; n <= AR_MAX_RANKS; ++n)
        for (int c = 1; c <= AR_MAX_CHANNELS; c += c < 20 ? 1 : 7)
            for (int w = 1; w <= AR_MAX_WAVES; ++w)
                for (int coll = 0; coll < 3; ++coll)
                    for (uint64_t pieces : {1ull, 2ull, 63ull, 300ull, 5000ull, 1ull << 20}) {
                        ar_plan_info g;
                        memset(&g, 0, sizeof g);
                        g.nranks = n;
                        g.nchannels = c;
                        g.nwaves = w;
                        g.coll = coll;
                        const uint64_t seg = (pieces - 1) * piece + 16;  // the last piece nearly empty
                        const uint64_t got = ar::ring_lds_workgroups(g, seg, piece);
                        const uint64_t in = seg * n * (coll == AR_COLL_ALLGATHER ? 1 : n);
                        const uint64_t once = n == 2 ? 1024 : n < 5 ? 512 : 256;
                        const uint64_t most = in > (128ull << 20) ? once : 2 * once;
                        const uint64_t named = (uint64_t)c * n * ((w + 1) / 2), waves = 4ull * c * w;
                        const uint64_t asked = named > waves ? named : waves;
                        expect(got >= 1 && got <= pieces, "no more than pieces", n, c, w, pieces, got);
                        expect(got <= most && got <= asked, "no more than asked or room", n, c, w, pieces, got);
                        expect(got <= 256 || got == pieces || got % 256 == 0, "even rounds", n, c, w, pieces, got);
                        if (asked <= 256 && asked <= pieces) expect(got == asked, "as asked", n, c, w, pieces, got);
                        // few ranks have at least half the waves an eight-rank plan has, and room for them
                        if (n < 8 && waves <= 256 && waves <= pieces) expect(got >= waves, "waves", n, c, w, pieces, got);
                    }
    printf("ring count: %s\n", failures ? "FAILED" : "ok");
    return failures != 0;
}
