// Exercises the launch rules of the row quantizers (csrc/nvfp4_quantize_plan.h, host-only) under the address and
// undefined-behaviour sanitizers.  Prints "ok" on success.
#include "../../paper_2605_18739_amd/csrc/nvfp4_quantize_plan.h"

#include <cstdio>
#include <cstdlib>

using namespace nvfp4;

static void require(bool ok, const char *what, long long n)
{
    if (ok) return;
    std::printf("%s (%lld)\n", what, n);
    std::abort();
}

// Where nothing is reduced at a workgroup's head (a given scale) a lane takes one block, up to the largest grid; with partial
// maxima at most four (the plain rule two, as many as it holds in flight, from 1.5 M blocks on), and no fewer than 1024 workgroups while there are
// blocks for them.
static void check_grid(int64_t nblk)
{
    const int64_t one_a_lane = std::min<int64_t>((nblk + 255) / 256, 16384);
    for (bool search : {false, true}) {
        require(encode_rows_grid(nblk, true, search) == one_a_lane, "given scale: one block a lane", nblk);
        const int64_t g = encode_rows_grid(nblk, false, search), most = !search && nblk >= 1500000 ? 2 : 4;
        require(g >= 1 && g <= one_a_lane, "a workgroup without a block", nblk);
        require(g >= std::min<int64_t>(one_a_lane, 1024), "fewer workgroups than four to a compute unit", nblk);
        require(g == 16384 || g * 256 * most >= nblk, "too many blocks a lane below the largest grid", nblk);
    }
}

// The search and the smoothed keys take two passes; the plain rule one launch below 12 k and from 0.95 M blocks on, and from 0.8 M on
// where the two passes would share the library's scratch array.
static void check_one_launch()
{
    for (int64_t n : {1, 11999, 12000, 799999, 800000, 887040, 949999, 950000, 3800000}) {
        for (bool scratch : {false, true}) {
            require(!one_launch_pays(n, true, false, scratch) && !one_launch_pays(n, true, true, scratch), "search in one launch", n);
            require(one_launch_pays(n, false, false, scratch) == (n < 12000 || n >= (scratch ? 800000 : 950000)), "plain rule", n);
        }
    }
}

int main()
{
    for (int64_t b = 1; b <= (1ll << 40); b <<= 1)
        for (int64_t e : {-1, 0, 1, 255, 257})
            if (b + e > 0) check_grid(b + e);
    for (int64_t b : {256 * 1024, 4 * 256 * 1024, 1500000, 256 * 16384, 2 * 256 * 16384, 4 * 256 * 16384})
        for (int64_t e = -2; e <= 2; ++e) check_grid(b + e);
    check_one_launch();
    std::printf("ok\n");
    return 0;
}
