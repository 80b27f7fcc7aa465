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

// Every row of a front that one workgroup factors has a lane, whatever the
// shared memory of the device, with any of the kernel's workgroups.
static void one_workgroup() {
    for (size_t kb : {64, 100, 160, 164, 168, 176, 192, 256, 320, 1024})
        for (int rows = 1; rows <= 600; ++rows) {
            const size_t lds = kb * 1024;
            if (kb == 160)   // gfx950: shared memory alone decides
                need(one_workgroup_front(rows, lds) == (rows <= 200), "class", rows, 0, 0, 0);
            for (int w : {1, 8, 16, 17, 100, 142, 143, 255, 256, 257, 600}) {
                if (w > rows) continue;
                if (one_workgroup_solve(rows, w, lds)) need(w <= kSolveThreads && front_solve_bytes(rows, w) <= lds, "solve", rows, w, 0, 0);
                if (kb == 160) need(one_workgroup_solve(rows, w, lds) == (front_solve_bytes(rows, w) <= lds), "solve class", rows, w, 0, 0);
            }
            if (!one_workgroup_front(rows, lds)) continue;
            need(front_bytes(rows) <= lds, "bytes", rows, 0, 0, 0);
            const int m = rows + 1;   // with the right-hand side
            for (int threads : kFactorThreads)
                for (int first = 0; first < rows; first += 16)
                    for (int r = first + 16; r < m; ++r) {
                        int held = 0;
                        for (int wave = 0; wave < threads / kCholWave; ++wave)
                            held += r >= panel_wave_begin(first, wave) && r < panel_wave_end(first, wave);
                        need(held == 1, "row without a lane", rows, threads, first, r);
                    }
        }
}

int main() {
    one_workgroup();
    panel_rows();
    std::printf("ok\n");
    return 0;
}
