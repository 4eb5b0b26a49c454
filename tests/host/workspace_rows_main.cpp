// The rows of partial sums that decode_base_rows and mx_plain_rows report for T tokens, against every batch of up to T: none
// has more, one has as many.  Host rules only; no GPU call that needs a device.
#include <cstdio>
#include <vector>

#include "../../paper_2410_09687_amd/csrc/kernels.h"

int main()
{
    const int widths[][2] = {{64, 8},      {72, 136},    {256, 256},   {1000, 2048},  {1024, 1416},  {2048, 256},   {2048, 2048}, {2048, 5632},
                             {2048, 8192}, {2048, 11264}, {4096, 4096}, {4096, 11008}, {5632, 2048},  {5632, 8192},  {5640, 256},  {5640, 1000},
                             {2056, 136},  {8192, 128},   {8192, 32000}, {2048, 65536}, {11008, 4096}, {16384, 1024}, {128, 16384}};
    const int64_t max_t = 40000;
    long long bad = 0;
    for (const auto &w : widths) {
        const int d_in = w[0], d_out = w[1];
        int64_t most = 0, mx_most = 0;
        for (int64_t t = 1; t <= max_t; ++t) {
            const int64_t own = t * moin::decode_base_splits(t, d_in, d_out), said = moin::decode_base_rows(t, d_in, d_out);
            if (own > most) most = own;
            if (said != most && ++bad <= 10)
                std::printf("%d -> %d, %lld tokens: %lld rows reported, %lld asked for\n", d_in, d_out, (long long)t, (long long)said, (long long)most);
            if (d_in % 128) continue;
            int parts = 0, per = 0;
            moin::mx_plain_shape(t, d_in, d_out, &parts, &per);
            if (t * parts > mx_most) mx_most = t * parts;
            const int64_t mx_said = moin::mx_plain_rows(t, d_in, d_out);
            if (mx_said != mx_most && ++bad <= 10)
                std::printf("quantised %d -> %d, %lld tokens: %lld rows reported, %lld asked for\n", d_in, d_out, (long long)t, (long long)mx_said,
                            (long long)mx_most);
        }
    }
    if (bad) return 1;
    std::printf("workspace rows agree\n");
    return 0;
}
