// Exercises the index division and the launch rules of the row quantizers (csrc/nvfp4_quantize_plan.h, no HIP) under the
// address and undefined-behaviour sanitizers.  Prints "ok" on success.
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

// The division that the kernels run: numbers beside multiples of the width, where a wrong factor shows first, and at both ends
// of the range; from 2^31 indexes on, and for widths that have no factor, the plain division.
static void check_divisor(int64_t d, uint64_t &seed)
{
    const int64_t top = 1ll << 31;
    const Divisor by(d, top), beyond(d, top + 1);
    require(beyond.m == 0, "a factor beyond its range", d);
    require((by.m != 0) == (d < top), "no factor inside its range", d);
    for (int i = 0; i < 64; ++i) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        const int64_t q = i == 0 ? 0 : i == 1 ? (top - 1) / d : (int64_t)((seed >> 16) % (uint64_t)((top - 1) / d + 1));
        for (int64_t n : {q * d - 1, q * d, q * d + 1, q * d + d - 1, top - 1}) {
            if (n >= 0 && n < top) require(divide(n, d, by) == n / d, "quotient", n);
            const int64_t large = n + (1ll << 33);
            if (n >= 0) require(divide(large, d, beyond) == large / d, "quotient of a large index", large);
        }
    }
}

int main()
{
    uint64_t seed = 31;
    for (int64_t d = 1; d < 3000; ++d) check_divisor(d, seed);
    for (int k = 9; k <= 31; ++k)
        for (int64_t e : {-1, 0, 1}) check_divisor((1ll << k) + e, seed);
    for (int i = 0; i < 3000; ++i) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        check_divisor(1 + (int64_t)((seed >> 20) % ((1ull << 31) - 1)), seed);
    }
    for (int64_t b = 1; b <= (1ll << 40); b <<= 1)
        for (int64_t e : {-1, 0, 1, 255, 257})
            if (b + e > 0) check_grid(b + e);
    for (int64_t b : {256 * 1024, 4 * 256 * 1024, 1500000, 256 * 16384, 2 * 256 * 16384, 4 * 256 * 16384})
        for (int64_t e = -2; e <= 2; ++e) check_grid(b + e);
    check_one_launch();
    std::printf("ok\n");
    return 0;
}
