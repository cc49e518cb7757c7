// gemm_cost.hpp -- measured cost of the projection products per tile (host).
//
// What decides between tiles of a mid-sized or small product is how the grid
// falls on the 256 CUs and how long a workgroup's step takes when it has the CU
// to itself (its barrier and loads then lie open) or shares it.  So a tile's
// time is modelled as
//   start + steps * g,   g = one, two (the busiest CU has 1 or 2 workgroups) or
//                            more * (workgroups per CU, mean of the average and
//                            the busiest),
// and never less than 2 us plus the operands and the result at 4.5 TB/s.  The
// four constants (us) were fitted per tile and product to event times of every
// tile on 210 shapes, 64 .. 8192 tokens, ranks of 8 .. 64 and odd multiples of
// 8 among them (630 products, MI355X, back to back).  The tile picked by them
// (default_tile in api.cpp) is 2.7% slower than the best of the 21 in the
// geometric mean and within 7% on 9 of 10 products; the preference orders alone
// were 24% slower, within 70% on 9 of 10.
// (The loads have since been spread over a step's products, proj_gemm.hip: on 240
// other shapes, 720 products, the pick is 4.8% from the best; constants fitted
// again on 130 of them gained 0.5 .. 1.2% there, inside what two timings of such a
// sweep differ by, so they stay.  Nor were the steps of tiles 11, 12 and 17 .. 20,
// forward and weight gradient, scaled by what a swizzle without bank conflicts for
// 256-column tiles gave, 0.98 .. 0.85.)
#pragma once

#include "gemm_tiles.hpp"

namespace fbl {

struct GemmCost {
    float start, one, two, more;
};

// [tile][0: forward, 1: data gradient, 2: weight gradient]
constexpr GemmCost kGemmCost[][3] = {
    {{4.4f, 0.350f, 0.557f, 0.325f}, {4.3f, 0.342f, 0.645f, 0.366f}, {5.5f, 0.318f, 0.511f, 0.339f}},  // 0
    {{3.6f, 0.243f, 0.373f, 0.227f}, {3.5f, 0.240f, 0.410f, 0.274f}, {4.0f, 0.239f, 0.370f, 0.212f}},  // 1
    {{3.6f, 0.256f, 0.362f, 0.192f}, {3.5f, 0.239f, 0.411f, 0.246f}, {4.1f, 0.236f, 0.354f, 0.200f}},  // 2
    {{2.9f, 0.174f, 0.252f, 0.127f}, {2.7f, 0.161f, 0.238f, 0.160f}, {3.1f, 0.154f, 0.257f, 0.138f}},  // 3
    {{4.1f, 0.618f, 0.971f, 0.584f}, {4.0f, 0.610f, 1.032f, 0.580f}, {4.5f, 0.569f, 0.999f, 0.670f}},  // 4
    {{3.7f, 0.405f, 0.611f, 0.390f}, {3.7f, 0.412f, 0.610f, 0.410f}, {3.7f, 0.406f, 0.690f, 0.459f}},  // 5
    {{3.7f, 0.397f, 0.615f, 0.356f}, {3.7f, 0.397f, 0.604f, 0.357f}, {3.9f, 0.400f, 0.675f, 0.425f}},  // 6
    {{3.0f, 0.264f, 0.387f, 0.223f}, {3.1f, 0.262f, 0.367f, 0.240f}, {2.9f, 0.246f, 0.449f, 0.286f}},  // 7
    {{5.8f, 0.536f, 1.217f, 0.693f}, {5.5f, 0.498f, 1.251f, 0.708f}, {6.2f, 0.505f, 1.215f, 0.856f}},  // 8
    {{3.3f, 0.410f, 1.006f, 0.562f}, {3.4f, 0.397f, 0.886f, 0.542f}, {3.1f, 0.396f, 1.163f, 0.756f}},  // 9
    {{5.5f, 0.591f, 1.422f, 0.821f}, {5.4f, 0.571f, 1.397f, 0.898f}, {5.4f, 0.634f, 1.650f, 1.064f}},  // 10
    {{8.2f, 0.869f, 2.012f, 1.161f}, {8.3f, 0.862f, 2.029f, 1.387f}, {9.1f, 0.869f, 2.389f, 1.786f}},  // 11
    {{8.2f, 0.891f, 2.046f, 1.195f}, {8.1f, 0.886f, 2.106f, 1.404f}, {9.2f, 0.825f, 2.333f, 1.669f}},  // 12
    {{3.1f, 0.282f, 0.463f, 0.301f}, {2.9f, 0.278f, 0.415f, 0.300f}, {2.8f, 0.292f, 0.513f, 0.378f}},  // 13
    {{2.9f, 0.307f, 0.620f, 0.404f}, {2.9f, 0.282f, 0.509f, 0.373f}, {2.7f, 0.326f, 0.625f, 0.478f}},  // 14
    {{3.0f, 0.271f, 0.426f, 0.244f}, {3.0f, 0.276f, 0.422f, 0.253f}, {2.8f, 0.284f, 0.538f, 0.332f}},  // 15
    {{2.8f, 0.209f, 0.412f, 0.261f}, {3.0f, 0.189f, 0.288f, 0.218f}, {2.5f, 0.243f, 0.568f, 0.326f}},  // 16
    {{9.5f, 0.872f, 1.950f, 1.194f}, {10.0f, 0.848f, 2.179f, 0.991f}, {10.8f, 1.088f, 2.506f, 1.572f}},  // 17
    {{9.2f, 1.647f, 3.673f, 2.215f}, {9.7f, 1.677f, 4.303f, 1.956f}, {10.5f, 1.931f, 4.774f, 2.961f}},  // 18
    {{8.7f, 1.422f, 3.271f, 2.125f}, {9.0f, 1.428f, 3.692f, 1.678f}, {9.9f, 1.775f, 4.358f, 2.736f}},  // 19
    {{8.8f, 1.515f, 3.397f, 2.204f}, {9.0f, 1.514f, 3.877f, 1.762f}, {9.9f, 1.841f, 4.439f, 2.752f}},  // 20
};
static_assert(sizeof(kGemmCost) / sizeof(kGemmCost[0]) == kGemmTileCount, "every tile");

// Modelled time (us) of a product with rows x cols outputs and contraction kc.
inline double gemm_cost(int tile, int product, long long rows, long long cols, long long kc) {
    const GemmTile& t = kGemmTiles[tile];
    const GemmCost& c = kGemmCost[tile][product];
    const auto tiles = [](long long n, int tile) { return (n + tile - 1) >> __builtin_ctz(tile); };  // powers of two
    const long long wgs = tiles(rows, t.bm) * tiles(cols, t.bn);
    const long long busiest = (wgs + 255) / 256;
    const double g = busiest == 1 ? c.one : busiest == 2 ? c.two : c.more * 0.5 * ((double)busiest + (double)wgs / 256);
    const double time = c.start + (double)tiles(kc, t.bk) * g;
    const double bytes = 2.0 * ((double)rows * kc + (double)kc * cols + (double)rows * cols);
    const double least = 2.0 + bytes / 4.5e6;
    return time > least ? time : least;
}

}  // namespace fbl
