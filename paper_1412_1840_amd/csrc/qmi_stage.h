// Host copies through page-locked memory.
//
// A copy from or to pageable memory goes through the runtime's own staging buffer, one array and
// one thread at a time: 16 us per small array, and 2 to 3 GB/s for a large result, most of it the
// first touch of the caller's fresh pages.  Here a call's inputs are gathered into one page-locked
// block and one device buffer, and large copies are cut into chunks that several threads move
// while the copy engine moves others.  Measured: cut, detrending and whitening of 2048 curves
// (99 MB over the bus) 13.0 -> 4.1 ms, the results of 256 periodograms of 20 000 frequencies with
// their search 2.9 ms less, one of 5000 frequencies with its potentials 181 -> 141 us, one of 9 from
// device arrays 130 -> 100 us.  The page-locked memory that every context begins with costs 10 to 20
// us of its creation and 15 to 25 of its end; a first call is 25 us shorter with it.
#ifndef QMI_STAGE_H
#define QMI_STAGE_H

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>
#include <functional>
#include <vector>

#include "qmi_team.h"

namespace qmi {

constexpr size_t kStageMin = size_t(256) << 10;  // held by every context (a one-curve search)
constexpr size_t kStageMax = size_t(32) << 20;   // most page-locked memory of a context
// Bytes a thread moves at a time: 60 MB in and 39 MB out take 5.2, 4.4, 4.1, 4.4 and 4.5 ms in
// chunks of 0.5, 1, 2, 4 and 8 MB, with 4 to 14 threads.
constexpr size_t kStageChunk = size_t(2) << 20;
constexpr int kStageChunks = (int)(kStageMax / kStageChunk);
// Threads pay from about this many bytes on (starting and joining a team takes 0.1 ms, as long as
// one thread takes to move 0.5 MB into fresh pages).
constexpr size_t kTeamBytes = size_t(2) << 20;

// A context's page-locked block, used by one call at a time.  A call that ends with an error may
// leave copies of it in flight: the next one waits for them first.
struct Stage {
    char* p = nullptr;
    size_t bytes = 0;
    hipEvent_t ev[kStageChunks] = {};
    bool have_ev = false;
    bool busy = false;  // copies of the block may be in flight

    // Room for min(want, kStageMax) bytes; false: use pageable copies.
    bool grow(size_t want, hipStream_t st) {
        want = std::min(want, kStageMax);
        if (bytes >= want) return bytes > 0;
        if (p) {
            if (hipStreamSynchronize(st) != hipSuccess) return false;
            (void)hipHostFree(p);
        }
        want = std::min((std::max(want, 2 * bytes) + 4095) / 4096 * 4096, kStageMax);
        p = nullptr;
        bytes = 0;
        if (hipHostMalloc(reinterpret_cast<void**>(&p), want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            p = nullptr;
            return false;
        }
        bytes = want;
        return true;
    }
    bool events() {
        while (!have_ev) {
            int k = 0;
            for (; k < kStageChunks && (ev[k] || hipEventCreateWithFlags(
                                                     &ev[k], hipEventDisableTiming) == hipSuccess);
                 ++k) {
            }
            if (k < kStageChunks) {
                (void)hipGetLastError();
                return false;
            }
            have_ev = true;
        }
        return true;
    }
    void release() {
        if (p) (void)hipHostFree(p);
        for (hipEvent_t& e : ev)
            if (e) (void)hipEventDestroy(e);
        p = nullptr;
        bytes = 0;
        have_ev = false;
    }
};

// The host arrays of a call and their places in one device buffer.
struct Upload {
    struct Seg {
        const void* src;
        size_t bytes, at;
    };
    std::vector<Seg> segs;
    size_t total = 0;
    size_t place(size_t bytes) {  // room without contents
        const size_t at = (total + 255) / 256 * 256;
        total = at + std::max<size_t>(bytes, 1);
        return at;
    }
    size_t add(const void* src, size_t bytes) {
        const size_t at = place(bytes);
        if (bytes) segs.push_back({src, bytes, at});
        return at;
    }
    // Copies [lo, hi) of the buffer's contents to `to`.
    void gather(char* to, size_t lo, size_t hi) const {
        for (const Seg& s : segs) {
            const size_t a = std::max(lo, s.at), b = std::min(hi, s.at + s.bytes);
            if (a < b) std::memcpy(to + (a - lo), (const char*)s.src + (a - s.at), b - a);
        }
    }
};

// Queues the copy of an upload to dst; the sources may go when it returns.  may_grow: page-locked
// memory may be allocated.
inline hipError_t upload(Stage& sg, const Upload& up, char* dst, int device, hipStream_t st,
                         bool may_grow) {
    hipError_t e = sg.busy ? hipStreamSynchronize(st) : hipSuccess;
    if (e != hipSuccess) return e;
    sg.busy = true;
    if (!(may_grow ? sg.grow(up.total, st) : sg.bytes >= up.total)) {
        for (const Upload::Seg& s : up.segs) {
            e = hipMemcpyAsync(dst + s.at, s.src, s.bytes, hipMemcpyHostToDevice, st);
            if (e != hipSuccess) break;
        }
        // A copy of pageable memory may still read it after the call that queued it.
        const hipError_t w = hipStreamSynchronize(st);
        return e != hipSuccess ? e : w;
    }
    for (size_t lo = 0; lo < up.total; lo += sg.bytes) {
        if (lo > 0 && (e = hipStreamSynchronize(st)) != hipSuccess) return e;
        const size_t len = std::min(sg.bytes, up.total - lo);
        if (len < kTeamBytes) {
            up.gather(sg.p, lo, lo + len);
            e = hipMemcpyAsync(dst + lo, sg.p, len, hipMemcpyHostToDevice, st);
            if (e != hipSuccess) return e;
            continue;
        }
        std::atomic<int> bad{(int)hipSuccess};
        run_team((int64_t)((len + kStageChunk - 1) / kStageChunk), [&](int64_t k) {
            const size_t a = (size_t)k * kStageChunk, b = std::min(len, a + kStageChunk);
            up.gather(sg.p + a, lo + a, lo + b);
            hipError_t r = hipSetDevice(device);
            if (r == hipSuccess)
                r = hipMemcpyAsync(dst + lo + a, sg.p + a, b - a, hipMemcpyHostToDevice, st);
            if (r != hipSuccess) bad.store((int)r);
        });
        if (bad.load() != (int)hipSuccess) return (hipError_t)bad.load();
    }
    return e;
}

// Results on their way to the host: put(src, offset, bytes) takes a piece of one of them (from
// several threads at once, pieces in any order).
struct Download {
    struct Seg {
        const char* src;
        size_t bytes;
        std::function<void(const char*, size_t, size_t)> put;
        char* direct;  // where a pageable copy can go at once
    };
    std::vector<Seg> segs;
    size_t total = 0;
    void add(void* dst, const void* src, size_t bytes) {
        char* to = (char*)dst;
        if (bytes)
            segs.push_back({(const char*)src, bytes,
                            [to](const char* from, size_t at, size_t len) {
                                std::memcpy(to + at, from, len);
                            },
                            to});
        total += bytes;
    }
    void add(std::function<void(const char*, size_t, size_t)> put, const void* src, size_t bytes) {
        if (bytes) segs.push_back({(const char*)src, bytes, std::move(put), nullptr});
        total += bytes;
    }
};

// Copies the results and waits for them, and for all work queued before.
inline hipError_t download(Stage& sg, const Download& dn, hipStream_t st, bool may_grow) {
    struct Piece {
        int seg;
        size_t at, len, in;
    };
    hipError_t e = hipSuccess;
    sg.busy = true;
    const bool staged = (may_grow ? sg.grow(dn.total, st) : sg.bytes >= dn.total);
    const bool team = staged && dn.total >= kTeamBytes && sg.events();
    if (!staged) {
        std::vector<char> tmp;
        for (const Download::Seg& s : dn.segs) {
            if (!s.direct) tmp.resize(s.bytes);
            e = hipMemcpyAsync(s.direct ? s.direct : tmp.data(), s.src, s.bytes,
                               hipMemcpyDeviceToHost, st);
            if (e == hipSuccess && !s.direct) e = hipStreamSynchronize(st);
            if (e != hipSuccess) break;
            if (!s.direct) s.put(tmp.data(), 0, s.bytes);
        }
        const hipError_t w = hipStreamSynchronize(st);  // also the copies before one that failed
        if (e == hipSuccess) e = w;
        sg.busy = e != hipSuccess;
        return e;
    }
    int seg = 0;
    size_t at = 0;
    std::vector<Piece> now;
    do {
        // A round: pieces of the results until the block is full.
        now.clear();
        size_t in = 0;
        while (seg < (int)dn.segs.size() && in < sg.bytes &&
               (!team || now.size() < (size_t)kStageChunks)) {
            const size_t len = std::min({team ? kStageChunk : sg.bytes, dn.segs[seg].bytes - at,
                                         sg.bytes - in});
            e = hipMemcpyAsync(sg.p + in, dn.segs[seg].src + at, len, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess && team) e = hipEventRecord(sg.ev[now.size()], st);
            if (e != hipSuccess) break;
            now.push_back({seg, at, len, in});
            in += len;
            at += len;
            if (at == dn.segs[seg].bytes) {
                at = 0;
                ++seg;
            }
        }
        if (!team || e != hipSuccess) {
            const hipError_t w = hipStreamSynchronize(st);
            if (e == hipSuccess) e = w;
            if (e != hipSuccess) return e;
            for (const Piece& p : now) dn.segs[p.seg].put(sg.p + p.in, p.at, p.len);
        } else {
            std::atomic<int> bad{(int)hipSuccess};
            run_team((int64_t)now.size(), [&](int64_t k) {
                const hipError_t r = hipEventSynchronize(sg.ev[k]);
                const Piece& p = now[k];
                if (r != hipSuccess) bad.store((int)r);
                else dn.segs[p.seg].put(sg.p + p.in, p.at, p.len);
            });
            if (bad.load() != (int)hipSuccess) return (hipError_t)bad.load();
        }
    } while (seg < (int)dn.segs.size());
    if (team) e = hipStreamSynchronize(st);
    sg.busy = e != hipSuccess;
    return e;
}

}  // namespace qmi

#endif  // QMI_STAGE_H
