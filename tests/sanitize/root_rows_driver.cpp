// Host check of the index arithmetic behind the rows that a compressed root level does not store: every list of up to five
// coordinates, in order or not, repeated or outside the mode, against places and gaps worked out directly.
#include <cstdio>
#include <vector>

#include "../../paper_2102_05187_amd/csrc/kernels.hpp"
#include "../../paper_2102_05187_amd/csrc/mttkrp_plan.hpp"

int main() {
    long lists = 0;
    for (int nrows = 1; nrows <= 7; ++nrows)
        for (int n = 1; n <= 5; ++n) {
            long all = 1;
            for (int i = 0; i < n; ++i) all *= nrows + 2;
            for (long code = 0; code < all; ++code, ++lists) {
                std::vector<int32_t> idx(n);
                long c = code;
                bool increases = true;
                for (int i = 0; i < n; ++i, c /= nrows + 2) {
                    idx[i] = (int32_t)(c % (nrows + 2)) - 1;
                    if (idx[i] < 0 || idx[i] >= nrows || (i > 0 && idx[i] <= idx[i - 1])) increases = false;
                }
                int expect = 0;
                for (int r = 0; r < nrows; ++r) {
                    const int64_t p = comet::unstored_place(idx.data(), n, nrows, r);
                    if (p < -1 || (p >= 0 && p >= nrows - n)) { printf("place %ld of row %d outside\n", (long)p, r); return 1; }
                    if (!increases) continue;
                    bool stored = false;
                    for (int x : idx) stored |= x == r;
                    if (p != (stored ? -1 : expect)) { printf("row %d at %ld\n", r, (long)p); return 1; }
                    if (!stored) ++expect;
                }
                if (increases && expect != nrows - n) { printf("%d of %d rows listed\n", expect, nrows - n); return 1; }
                for (int s = 0; s <= n; ++s) {
                    const int64_t from = s ? idx[s - 1] : -1, to = s < n ? idx[s] : nrows;
                    const int g = comet::mt_gap(from, to);
                    if (g < 0 || (to > from ? g != to - from - 1 : g != 0)) { printf("gap %d\n", g); return 1; }
                    const unsigned rec = comet::mt_sum(300, 16, comet::kMtSlice, g);      // the fields beside it stay as they are
                    if ((rec & 0xffffu) != comet::mt_sum(300, 16, comet::kMtSlice, 0) || (int)(rec >> 16) != g) { printf("record %x\n", rec); return 1; }
                }
            }
        }
    if (comet::mt_gap(-1, int64_t(1) << 31) != 65535 || comet::mt_gap(int64_t(1) << 31, 0) != 0) { printf("long gap\n"); return 1; }
    printf("lists %ld ok\n", lists);
    return 0;
}
