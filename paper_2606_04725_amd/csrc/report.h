// The word in which the device reports to a host that polls it: number of the
// report (16 bits, from the top), 1 if an instance ended in this evaluation,
// instances waiting for corrections (22 bits), instances running (24 bits).
// Without device code, so that a host program can check it.
#pragma once

#include <cstdint>

namespace nmpc {

constexpr int kRepWaiting = 24, kRepEnded = 46, kRepSeq = 48;

constexpr unsigned long long report_word(unsigned number, unsigned running, unsigned waiting, bool ended) {
    return ((unsigned long long)(number & 0xffffu) << kRepSeq) | ((unsigned long long)ended << kRepEnded) |
           ((unsigned long long)waiting << kRepWaiting) | running;
}
constexpr uint16_t report_number(unsigned long long w) { return (uint16_t)(w >> kRepSeq); }
constexpr int report_running(unsigned long long w) { return (int)(w & ((1u << kRepWaiting) - 1)); }
constexpr int report_waiting(unsigned long long w) {
    return (int)((w >> kRepWaiting) & ((1u << (kRepEnded - kRepWaiting)) - 1));
}
constexpr bool report_ended(unsigned long long w) { return (w >> kRepEnded) & 1; }

// The host's count of the reports enqueued (0: the passes', 1: the conjugate
// gradients').  A call that ends in an error may leave some enqueued uncounted:
// the next call, once the work is at its end, takes the numbers of the words.
struct ReportCount {
    uint16_t last[2] = {0, 0};
    bool open = false;   // a call that waits for reports is running, or ended in an error
    void resume(const unsigned long long* words) {
        for (int k = 0; k < 2; ++k) last[k] = report_number(words[k]);
    }
};

// The report number as soon as load() returns it.  stream() tells, now and then,
// how the work that makes the report stands: a report that work at its end has
// not made never comes, whatever the word still holds.
enum class StreamState { kNotAsked, kBusy, kDrained, kFailed };
enum class ReportState { kArrived, kMissing, kFailed };
template <class Load, class Stream>
ReportState await_report(uint16_t number, Load&& load, Stream&& stream, unsigned long long& word) {
    while (true) {
        word = load();
        if (report_number(word) == number) return ReportState::kArrived;
        switch (stream()) {
            case StreamState::kFailed:
                return ReportState::kFailed;
            case StreamState::kDrained:   // the report may have come between the two
                word = load();
                return report_number(word) == number ? ReportState::kArrived : ReportState::kMissing;
            default:
                break;
        }
    }
}

}  // namespace nmpc
