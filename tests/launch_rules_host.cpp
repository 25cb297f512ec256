// The launch rules of csrc/tune.h on the host: which row lengths get launches of their
// own, and the waves of a column launch.
#include <cstdio>
#include <vector>

#include "../paper_2201_03509_amd/csrc/tune.h"

static int failed = 0;
static void expect(bool ok, int line) {
    if (!ok) {
        printf("line %d\n", line);
        failed = 1;
    }
}
#define EXPECT(x) expect(x, __LINE__)

int main() {
    using c3tune::col_waves;
    using c3tune::kOwnPoints;
    using c3tune::own_rows;
    typedef std::vector<char> V;
    const int64_t P = kOwnPoints;
    EXPECT(own_rows({}) == V{});
    EXPECT(own_rows({0}) == V{1});  // alone: always
    EXPECT(own_rows({1}) == V{1});
    EXPECT((own_rows({P / 2, P / 2 - 1}) == V{0, 0}));  // together less than a tail is worth
    EXPECT((own_rows({P / 2, P / 2}) == V{1, 1}));
    EXPECT((own_rows({P - 1, 1}) == V{1, 1}));
    EXPECT((own_rows({P, 1}) == V{1, 1}));        // the second is left alone
    EXPECT((own_rows({P, 1, 1}) == V{1, 0, 0}));  // the others share
    EXPECT((own_rows({P - 1, P - 1, 1}) == V{0, 0, 0}));
    EXPECT((own_rows({P - 1, P - 1, 2}) == V{1, 1, 1}));
    EXPECT((own_rows({P, P, P, P}) == V{1, 1, 1, 1}));
    // what the tuner times: three lengths of two segments share, one length does not, nor
    // does one with many segments beside others
    const auto few = c3tune::own_lengths({{100000, 2}, {112500, 2}, {115200, 2}});
    for (const auto &kv : few) EXPECT(!kv.second);
    EXPECT(c3tune::own_lengths({{100000, 2}}).at(100000));
    const auto big = c3tune::own_lengths({{100000, (int)(P / 50000)}, {112500, 2}, {115200, 2}});
    EXPECT(big.at(100000) && !big.at(112500) && !big.at(115200));
    for (int64_t n : {1, 2048, 3073, 4096, 6145, 8192}) EXPECT(col_waves(n) == 2);
    for (int64_t n : {2049, 3072}) EXPECT(col_waves(n) == 3);
    EXPECT(col_waves(4097) == 2 && col_waves(6144) == 2);  // a tie: six wave-rounds either way
    EXPECT(col_waves(8193) == 3 && col_waves(9216) == 3);
    if (!failed) puts("launch rules ok");
    return failed;
}
