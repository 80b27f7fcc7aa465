// The report word and the wait for it: every field on its own, numbers past the
// 16-bit wrap, and a stream that drains or fails without the report.  Prints "ok".
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "../../paper_2606_04725_amd/csrc/report.h"

using namespace nmpc;

static void need(bool ok, const char* what, long a) {
    if (ok) return;
    std::printf("%s: %ld\n", what, a);
    std::exit(1);
}

static void fields() {
    for (unsigned number : {0u, 1u, 65535u, 65536u, 65537u, 4294967295u})
        for (unsigned running : {0u, 1u, 24u, (1u << 24) - 1})
            for (unsigned waiting : {0u, 1u, 24u, (1u << 22) - 1})
                for (bool ended : {false, true}) {
                    const unsigned long long w = report_word(number, running, waiting, ended);
                    need(report_number(w) == (uint16_t)number, "number", number);
                    need(report_running(w) == (int)running, "running", running);
                    need(report_waiting(w) == (int)waiting, "waiting", waiting);
                    need(report_ended(w) == ended, "ended", ended);
                }
}

// A host that counts with 16 bits and a device that counts with 32 agree over
// the wrap, and the report before the awaited one is never taken for it.
static void wrap() {
    uint16_t host = 65530;
    for (unsigned dev = 65530; dev < 65550; ++dev, ++host) {
        unsigned long long word = 0;
        int asked = 0;
        const ReportState r = await_report(
            host, [&] { return report_word(asked < 3 ? dev - 1 : dev, asked < 3 ? 7 : 3, 0, false); },
            [&] { return ++asked % 2 ? StreamState::kNotAsked : StreamState::kBusy; }, word);
        need(r == ReportState::kArrived && asked == 3 && report_running(word) == 3, "wrap", dev);
    }
}

static void streams() {
    for (unsigned stale : {0u, 6u, 8u, 65535u}) {
        unsigned long long word = 0;
        // drained, the word never changes: the counts in it are not this report's
        need(await_report(7, [&] { return report_word(stale, 0, 0, true); }, [] { return StreamState::kDrained; }, word) ==
                 ReportState::kMissing, "drained with another number", stale);
        // drained, the report came after the first look
        int looks = 0;
        need(await_report(7, [&] { return ++looks < 2 ? report_word(stale, 0, 0, true) : report_word(7, 5, 1, false); },
                          [] { return StreamState::kDrained; }, word) == ReportState::kArrived &&
                 report_running(word) == 5 && report_waiting(word) == 1, "drained with the report", stale);
        need(await_report(7, [&] { return report_word(stale, 0, 0, true); }, [] { return StreamState::kFailed; }, word) ==
                 ReportState::kFailed, "failed", stale);
        // an arrived report counts whatever the stream would answer
        need(await_report(7, [] { return report_word(7, 0, 0, false); }, [] { return StreamState::kFailed; }, word) ==
                 ReportState::kArrived, "arrived", stale);
    }
}

// A call ends in an error with reports enqueued that it has not counted (or
// counted and not enqueued); the next call waits for its own.
static void resumed() {
    for (int uncounted = -3; uncounted <= 3; ++uncounted)
        for (unsigned made : {3u, 65534u, 65535u, 65536u, 131071u}) {
            ReportCount c;
            c.last[0] = (uint16_t)(made - uncounted);
            c.last[1] = (uint16_t)(made + 1);
            const unsigned long long words[2] = {report_word(made, 0, 0, true), report_word(made + 9, 0, 0, false)};
            c.resume(words);
            for (int k = 0; k < 2; ++k) {
                unsigned next = made + (k ? 9 : 0), looks = 0;
                unsigned long long word = 0;
                need(await_report(++c.last[k], [&] { return report_word(looks++ < 2 ? next : next + 1, 1, 0, false); },
                                  [] { return StreamState::kBusy; }, word) == ReportState::kArrived && looks == 3,
                     "after an error", made);
            }
        }
}

int main() {
    fields();
    wrap();
    resumed();
    streams();
    std::printf("ok\n");
    return 0;
}
