// xcd_item's order of a launch's items, for every count up to 400 and every
// number of H items: each item exactly once, each XCD's H items before its S
// items. Prints the number of counts for which that fails.
#include <cstdio>
#include <vector>

#include "../paper_1611_00606_amd/csrc/hs_internal.h"

int main() {
    int bad = 0;
    for (int n = 1; n <= 400; ++n)
        for (int first = 0; first <= n + 9; ++first) {
            std::vector<int> seen(n, 0);
            bool ok = true;
            for (int x = 0; x < 8; ++x) {
                int last = -1;
                for (int b = x; b < hs::xcd_blocks(n); b += 8) {
                    const int i = hs::xcd_item(b, n, first);
                    if (i < 0) continue;
                    ok = ok && i < n && i > last && ++seen[i] == 1;
                    last = i;
                }
            }
            for (int c : seen) ok = ok && c == 1;
            bad += !ok;
        }
    std::printf("%d\n", bad);
    return 0;
}
