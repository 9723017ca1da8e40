// Plans that a thread keeps: after any other layer, a layer's plan is that of a thread that
// planned nothing before.  The layers differ from a base in one value each (or in the few that
// must go together), and every ordered pair of them is asked for in turn.
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "bsp_common.h"

using namespace bsp;

namespace {

struct Layer {
    bsp_scheme s;
    bsp_conv_shape c;
    bool conv;
    bsp_dtype dt;
    int batch;
};
struct Result {
    bsp_status st;
    Plan p, alt;
};

Result plan(const Layer &l) {
    Result r;
    memset((void *)&r, 0, sizeof(r));
    r.st = make_plan(&l.s, l.conv ? &l.c : nullptr, l.dt, l.batch, &r.p, &r.alt);
    if (r.st != BSP_OK) memset((void *)&r.p, 0, sizeof(r.p));
    if (r.st != BSP_OK || !r.p.alt) memset((void *)&r.alt, 0, sizeof(r.alt));
    return r;
}
Result fresh(const Layer &l) {
    Result r;
    std::thread t([&] { r = plan(l); });
    t.join();
    return r;
}
bool same(const Result &a, const Result &b) {
    return a.st == b.st && memcmp(&a.p, &b.p, sizeof(Plan)) == 0 && memcmp(&a.alt, &b.alt, sizeof(Plan)) == 0;
}

}  // namespace

int main() {
    Layer base;
    memset((void *)&base, 0, sizeof(base));
    base.s.rows = 96; base.s.cols = 64 * 9; base.s.bh = 32; base.s.bw = 32; base.s.regularity = BSP_PUNCHED;
    base.s.rate = 2; base.s.khw = 9;
    base.c = {1, 64, 14, 14, 3, 3, 1, 1, 1, 1};
    base.conv = true; base.dt = BSP_BF16;
    std::vector<Layer> all = {base};
    auto with = [&](auto change) {
        Layer l = base;
        change(l);
        all.push_back(l);
    };
    with([](Layer &l) { l.s.rows = 80; });
    with([](Layer &l) { l.s.cols = 640; });   // an error: not the columns of the filters
    with([](Layer &l) { l.s.bh = 16; });
    with([](Layer &l) { l.s.bw = 16; });
    with([](Layer &l) { l.s.regularity = BSP_COL; });
    with([](Layer &l) { l.s.rate = 4; });
    with([](Layer &l) { l.s.khw = 3; });      // an error
    with([](Layer &l) { l.dt = BSP_F32; });
    with([](Layer &l) { l.conv = false; });
    with([](Layer &l) { l.conv = false; l.batch = -1; });   // list structure only
    with([](Layer &l) { l.c.cin = 32; });     // an error
    with([](Layer &l) { l.c.h = 13; });
    with([](Layer &l) { l.c.w = 13; });
    with([](Layer &l) { l.c.h = 4; l.c.w = 4; });           // packed for two kernels
    with([](Layer &l) { l.c.kh = 9; l.c.kw = 1; });
    with([](Layer &l) { l.c.kh = 1; l.c.kw = 9; });
    with([](Layer &l) { l.c.stride_h = 2; });
    with([](Layer &l) { l.c.stride_w = 2; });
    with([](Layer &l) { l.c.pad_h = 2; });
    with([](Layer &l) { l.c.pad_w = 2; });
    std::vector<Result> first;
    for (const Layer &l : all) first.push_back(fresh(l));
    int bad = 0;
    for (size_t i = 1; i < all.size(); ++i)
        if (same(first[i], first[0])) { printf("layer %zu plans as the base\n", i); ++bad; }
    for (size_t i = 0; i < all.size(); ++i)
        for (size_t j = 0; j < all.size(); ++j) {
            plan(all[i]);
            if (!same(plan(all[j]), first[j])) { printf("layer %zu after %zu\n", j, i); ++bad; }
        }
    // more layers than are kept, twice
    for (int r = 0; r < 2; ++r)
        for (int h = 3; h < 300; ++h) {
            Layer l = base;
            l.c.h = h;
            plan(l);
            if (h % 7 == 0 && !same(plan(l), fresh(l))) { printf("height %d\n", h); ++bad; }
        }
    // the batch does not enter
    Layer b = base;
    b.c.n = 64;
    if (!same(plan(b), first[0])) { printf("batch\n"); ++bad; }
    printf("%d faults\n", bad);
    return bad;
}
