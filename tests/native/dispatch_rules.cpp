// Host check of the launch rules (launch.hpp): at sizes where two ways of running a call were timed, the rule takes
// the faster one.  Cases where the two differ by less than 4 % are left out.
#include <cstdio>

#include "launch.hpp"

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

int main() {
    one_launch();
    if (failures) return 1;
    std::printf("ok dispatch rules\n");
    return 0;
}
