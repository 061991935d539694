// A few host threads for one loop.
#ifndef QMI_TEAM_H
#define QMI_TEAM_H

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <thread>

namespace qmi {

constexpr int kTeamMax = 8;

// Runs work(k) for k in [0, n) on up to kTeamMax threads, the caller among them; work must not
// throw.  Threads that cannot be started are done without.
template <typename F>
void run_team(int64_t n, const F& work) {
    std::atomic<int64_t> next{0};
    auto body = [&] {
        for (int64_t k; (k = next.fetch_add(1, std::memory_order_relaxed)) < n;) work(k);
    };
    std::thread team[kTeamMax];
    int started = 0;
    const int hw = (int)std::thread::hardware_concurrency();
    const int64_t want = std::min<int64_t>({n, (int64_t)kTeamMax, (int64_t)(hw > 0 ? hw : 1)});
    try {
        for (; started + 1 < want; ++started) team[started] = std::thread(body);
    } catch (...) {  // no thread, or no memory for one; those started are joined below
    }
    body();
    for (int k = 0; k < started; ++k) team[k].join();
}

}  // namespace qmi

#endif  // QMI_TEAM_H
