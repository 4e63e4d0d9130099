// Host-side checks of rules that the kernels' launches and index ranges rest
// on.  Runs without a GPU: no kernel is launched.
#include "kernels.hpp"
#include "plane.hpp"
#include "tile.hpp"
#include "march.hpp"

#include <cstdio>
#include <cstring>

using namespace cps;

static int bad = 0;
#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);     \
            ++bad;                                                  \
        }                                                           \
    } while (0)

// The buffer a batched level reads its coarse correction from, by the path of
// the coarse level; a finest level too large to march lies above one that does.
static void coarse_correction()
{
    float x, r, xt, mt;
    LDesc<float> d;
    std::memset(&d, 0, sizeof d);
    d.x = &x;
    d.r = &r;
    CHECK(level_result(d) == &x);
    d.mt = &mt;
    CHECK(level_result(d) == &r);
    d.mt = nullptr;
    d.tile = 1;
    d.xt = &xt;
    CHECK(level_result(d) == &xt);
    CHECK(!march_fits(make_geo(1024, 512, 512)) && march_fits(make_geo(512, 256, 256)));
}

// The LDS slots that the wavefronts of an elimination block read, for every
// length of the chunked form and every block it is launched in: the single
// solve's, a batch's (always kTriWaves wavefronts) and a one-launch row's.
static void elimination_block(const TriLaunch& t, int waves)
{
    CHECK(waves <= kTriWaves && t.gpb >= 1);
    int held = 0;
    for (int wv = 0; wv < waves; ++wv) {
        const TriLine l = tri_line(t, wv);
        CHECK(0 <= l.lo && l.lo <= wv && wv < l.hi && l.hi <= waves);
        CHECK(l.hi - l.lo == (l.live ? t.nw : 1));
        held += l.live;
    }
    CHECK(held == t.nw * t.gpb); // every line is whole
}

static void elimination_slots()
{
    for (int nr = 1; nr <= kTriChunk * kTriWaves; ++nr)
        for (int nh = 2; nh <= kPlaneLds; nh *= 2) {
            const Geo g = make_geo(nr, 6, 2 * nh);
            CHECK(tri_chunked(g));
            const TriLaunch one = tri_launch(g, 0), all = tri_launch(g, 0, kTriWaves);
            elimination_block(one, one.threads / 64);
            elimination_block(all, kTriWaves);
            if (!plane_row_fits(g)) continue;
            for (int waves : {plane_row_threads(g) / 64, kTriWaves}) {
                TriLaunch t = one;
                t.gpb = waves / t.nw; // as d_plane_row
                elimination_block(t, waves);
            }
        }
}

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "coarse_correction")) coarse_correction();
    else if (!std::strcmp(what, "elimination_slots")) elimination_slots();
    else return 2;
    return bad ? 1 : 0;
}
