// The index rules of the front kernels over every position of small fronts:
// rows that a panel launch's waves load lie in the front.  Prints "ok".
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "../../paper_2606_04725_amd/csrc/front_rules.h"

using namespace nmpc;

static void need(bool ok, const char* what, int a, int b, int c, int d) {
    if (ok) return;
    std::printf("%s: %d %d %d %d\n", what, a, b, c, d);
    std::exit(1);
}

static void panel_rows() {
    const int panel = 64;
    for (int w : {1, 2, 5, 15, 16, 17, 48, 63, 64, 65, 79, 80, 128, 130})
        for (int below : {0, 1, 15, 16, 17, 63, 64, 65, 200})
            for (int kb = 0; kb < w; kb += panel) {
                const int m = w + below, pw = w - kb < panel ? w - kb : panel;
                const int rest = m - kb - pw, blocks = rest > 0 ? (rest + kRowBlock - 1) / kRowBlock : 1;
                for (int b = 0; b < blocks; ++b)
                    for (int wave = 0; wave <= kPanelRowWaves; ++wave)
                        for (int li = 0; li < 16; ++li) {
                            const int r = panel_first_row(kb, pw, b, wave) + li;
                            need((r < m ? r : m - 1) >= 0, "row before the front", w, m, wave, r);
                            if (wave >= 1) need(r == kb + pw + b * kRowBlock + 16 * (wave - 1) + li, "row", w, m, wave, r);
                        }
            }
}

int main() {
    panel_rows();
    std::printf("ok\n");
    return 0;
}
