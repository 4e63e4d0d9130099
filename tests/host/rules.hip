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

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "coarse_correction")) coarse_correction();
    else return 2;
    return bad ? 1 : 0;
}
