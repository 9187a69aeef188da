// Host check of the launch rules (launch.hpp): at sizes where two ways of running a call were timed, the rule takes
// the faster one.  Cases where the two differ by less than 4 % are left out.
#include <cstdio>

#include "gemm_shape.hpp"

using namespace lacache;

static int failures = 0;

static void check(bool rule, double if_true, double if_false, const char* what, int a, int b, int c) {
    if (rule == (if_true < if_false)) return;
    std::printf("%s (%d, %d, %d): %.2f us if taken, %.2f us if not, rule says %d\n", what, a, b, c, if_true, if_false,
                (int)rule);
    ++failures;
}

// Lookups in one launch or two, us a call: queries, padded key columns, columns of all prefix models.
static void one_launch() {
    struct {
        int B, N, d_pad, resp;
        double one, two;
    } t[] = {{1, 10000, 384, 384, 9.57, 10.77},     {8, 10000, 384, 384, 10.52, 11.48},
             {16, 10000, 128, 128, 9.22, 10.13},    {12, 1000, 384, 384, 10.58, 11.33},
             {24, 10000, 384, 384, 13.89, 13.09},   {32, 10000, 384, 384, 16.55, 14.45},
             {24, 10000, 1024, 1024, 21.90, 19.79}, {32, 10000, 1024, 1024, 24.47, 20.09},
             {32, 200000, 768, 768, 60.23, 56.34},  {1, 20000, 768, 3200, 16.61, 17.57},
             {16, 20000, 768, 3200, 24.41, 21.12},  {16, 20000, 768, 3584, 28.45, 24.28},
             {16, 20000, 768, 1152, 20.11, 18.31},  {32, 20000, 768, 1536, 30.13, 22.05},
             {16, 20000, 768, 6144, 33.92, 26.13},  {1, 200000, 1536, 1536, 117.98, 106.75},
             {32, 200000, 1536, 1536, 135.66, 108.29}};
    for (auto& x : t) check(lookup_in_one_launch(x.B, x.N, x.d_pad, x.resp), x.one, x.two, "one launch: queries, columns, columns of models",
              x.B, x.d_pad, x.resp);
}

// Acceptance with sixteen or four waves on a row, in a replayed graph: rows, logits a row, dtype (0 float32).
static void accept() {
    struct {
        int rows, V, dtype;
        double sixteen, four;
    } t[] = {{256, 4000, 0, 5.87, 5.62},    {256, 12000, 0, 6.25, 7.14},  {1, 12000, 1, 5.03, 5.69},
             {100, 12000, 1, 5.46, 6.12},   {1, 16000, 1, 5.46, 6.97},    {256, 16000, 0, 6.88, 9.18},
             {256, 32000, 1, 10.01, 14.86}, {100, 50257, 0, 9.31, 12.31}, {256, 100003, 0, 23.54, 25.69},
             {1024, 8192, 0, 10.18, 8.62},  {512, 1000, 0, 5.66, 5.24},   {512, 8192, 1, 7.03, 6.41},
             {1000, 32000, 0, 27.56, 26.30}, {2048, 128256, 1, 95.03, 88.11}, {1000, 8192, 1, 10.16, 8.04},
             {512, 100003, 1, 22.09, 38.89}, {1024, 151936, 1, 55.79, 68.80}, {1024, 32000, 0, 28.14, 26.77}};
    for (auto& x : t)
        check(accept_many_waves(x.rows, x.V, x.dtype), x.sixteen, x.four, "sixteen waves: rows, logits, dtype", x.rows,
              x.V, x.dtype);
}

// Signatures by a wave per group and byte or by the bulk kernel: rows, bits, columns.
static void simhash() {
    struct {
        int n, bits, d;
        double wave, bulk;
    } t[] = {{8193, 64, 2048, 25.06, 38.49},   {8193, 128, 768, 22.29, 25.66},   {8193, 256, 2048, 46.30, 62.66},
             {16384, 64, 1024, 21.40, 26.33},  {32768, 64, 2048, 41.10, 46.59},  {49152, 64, 768, 30.22, 27.60},
             {49152, 32, 2048, 46.79, 48.72},  {12288, 128, 1024, 24.64, 29.11}, {24576, 128, 1024, 34.76, 30.92},
             {24576, 128, 2048, 53.75, 47.69}, {12288, 192, 768, 28.82, 30.11},  {24576, 192, 384, 27.98, 24.66},
             {12288, 256, 1536, 45.16, 52.03}, {24576, 256, 768, 45.75, 36.41},  {65536, 256, 2048, 228.55, 78.56},
             {65536, 128, 768, 53.78, 35.54}};
    for (auto& x : t)
        check(simhash_by_wave(x.n, x.bits), x.wave, x.bulk, "signatures by wave: rows, bits, columns", x.n, x.bits, x.d);
}

// Tile heights of the GEMM for one query tile (100 queries): rows, columns, the least of four times with 320-, 384-, 448-
// and 512-row tiles.  The chosen height's time is within 4 % of the best.
static void tile_heights() {
    struct {
        int n, d;
        double us[4];
    } t[] = {{150000, 1536, {98.7, 105.3, 116.5, 125.1}},  {190000, 1536, {133.1, 119.4, 125.5, 130.3}},
             {210000, 1536, {139.6, 150.0, 133.6, 149.1}}, {220000, 1536, {141.3, 151.3, 140.5, 136.6}},
             {250000, 1536, {170.4, 157.7, 174.4, 151.8}}, {180000, 1792, {154.0, 131.9, 146.3, 152.4}},
             {150000, 2048, {123.8, 137.0, 153.1, 164.0}},
             {200000, 2048, {169.0, 193.0, 174.2, 168.3}}, {220000, 2048, {176.5, 195.1, 181.2, 173.5}},
             {250000, 2048, {215.9, 198.9, 227.2, 192.7}}};
    for (auto& x : t) {
        const GemmShape g = gemm_shape(x.n, 100, x.d, 256);
        double best = x.us[0];
        for (double u : x.us) best = u < best ? u : best;
        const double us = x.us[g.kb - kGemmMinKB];
        if (us <= 1.04 * best) continue;
        std::printf("%d x %d keys in %d-row tiles: %.1f us, best %.1f us\n", x.n, x.d, 64 * g.kb, us, best);
        ++failures;
    }
}

int main() {
    one_launch();
    accept();
    simhash();
    tile_heights();
    if (failures) return 1;
    std::printf("ok dispatch rules\n");
    return 0;
}
