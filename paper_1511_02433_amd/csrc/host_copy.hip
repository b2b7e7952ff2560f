// Host-side helpers of the library: a loop split over a few host threads, the copies
// between caller (pageable) host memory and the device through pinned staging slots,
// and the pool that a handle's device memory comes from.
#include <algorithm>
#include <cstring>
#include <exception>
#include <iterator>
#include <new>
#include <thread>
#include <vector>

#include "ccdpp_internal.hpp"

namespace ccdk {

int host_workers() {
    const unsigned hc = std::thread::hardware_concurrency();
    return (int)std::max(1u, std::min(hc == 0 ? 1u : hc, 8u));
}

void parallel_ranges(int64_t n, int workers, const std::function<void(int, int64_t, int64_t)>& f) {
    workers = (int)std::max<int64_t>(1, std::min<int64_t>(workers, n));
    const int64_t per = (n + workers - 1) / workers;
    std::vector<std::thread> pool;
    pool.reserve(workers - 1);
    int w = 0;
    for (; w + 1 < workers; ++w) {
        const int64_t lo = std::min(n, w * per), hi = std::min(n, lo + per);
        try {
            pool.emplace_back(f, w, lo, hi);
        } catch (const std::exception&) {
            break;  // no more threads, or no memory for one: the calling thread does the rest
        }
    }
    f(w, std::min(n, w * per), n);
    for (auto& t : pool) t.join();
}

// ---- staging ------------------------------------------------------------------------

// The pinned slots, on first use (one allocation).
bool Stager::ready() {
    if (tried_) return pinned_ != nullptr;
    tried_ = true;
    workers_ = std::min(host_workers(), kCopyWorkers);
    void* p = nullptr;
    if (hipHostMalloc(&p, (size_t)workers_ * 2 * kChunk, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    pinned_ = static_cast<char*>(p);
    for (int w = 0; w < workers_; ++w)
        for (int i = 0; i < 2; ++i) {
            slot_[w][i].p = pinned_ + (size_t)(2 * w + i) * kChunk;
            if (hipEventCreateWithFlags(&slot_[w][i].ev, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                slot_[w][i].ev = nullptr;
                release();
                tried_ = true;
                return false;
            }
        }
    return true;
}

bool Stager::staged(size_t bytes) {
    if (bytes < kStageMin) return false;
    const size_t known = std::min(bytes, expected_);
    expected_ -= known;
    seen_ += bytes - known;
    return seen_ >= kPinFrom && ready();
}

hipError_t Stager::idle(Slot& sl) {
    if (!sl.busy) return hipSuccess;
    sl.busy = false;
    return hipEventSynchronize(sl.ev);
}

hipError_t Stager::finish() {
    hipError_t e = hipSuccess;
    for (auto& ws : slot_)
        for (Slot& sl : ws) {
            const hipError_t r = idle(sl);
            if (e == hipSuccess) e = r;
        }
    return e;
}

void Stager::release() {
    (void)finish();
    for (auto& ws : slot_)
        for (Slot& sl : ws) {
            if (sl.ev) (void)hipEventDestroy(sl.ev);
            sl = Slot{};
        }
    if (pinned_) (void)hipHostFree(pinned_);
    pinned_ = nullptr;
    tried_ = false;
}

template <class F>
hipError_t Stager::run(size_t bytes, int device, hipStream_t s, F&& f) {
    const int64_t chunks = (int64_t)((bytes + kChunk - 1) / kChunk);
    // hipStreamPerThread names another stream in each thread: the calling thread does it all.
    const int used = s == hipStreamPerThread ? 1 : (int)std::min<int64_t>(workers_, chunks);
    hipError_t err[kCopyWorkers] = {};  // hipSuccess
    auto work = [&](int, int64_t lo, int64_t hi) {
        int before = 0;  // the current device is a thread's own
        const bool moved = hipGetDevice(&before) == hipSuccess && before != device &&
                           hipSetDevice(device) == hipSuccess;
        for (int64_t w = lo; w < hi; ++w) err[w] = f((int)w, used, chunks);
        if (moved) (void)hipSetDevice(before);
    };
    try {
        parallel_ranges(used, used, work);
    } catch (const std::bad_alloc&) {  // thrown before any worker runs
        return hipErrorOutOfMemory;
    }
    for (hipError_t e : err)
        if (e != hipSuccess) return e;
    return hipSuccess;
}

hipError_t Stager::to_device(void* dst, const void* src, size_t bytes, int device, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (bytes < kStageMin) return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
    if (!staged(bytes)) {  // the source may go when this returns
        hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
        return e == hipSuccess ? hipStreamSynchronize(s) : e;
    }
    return run(bytes, device, s, [&](int w, int used, int64_t chunks) -> hipError_t {
        int i = 0;
        for (int64_t c = w; c < chunks; c += used, i ^= 1) {
            Slot& sl = slot_[w][i];
            hipError_t e = idle(sl);  // its last copy has read it
            if (e != hipSuccess) return e;
            const size_t off = (size_t)c * kChunk, len = std::min(kChunk, bytes - off);
            std::memcpy(sl.p, static_cast<const char*>(src) + off, len);
            e = hipMemcpyAsync(static_cast<char*>(dst) + off, sl.p, len, hipMemcpyHostToDevice, s);
            if (e == hipSuccess) e = hipEventRecord(sl.ev, s);
            if (e != hipSuccess) return e;
            sl.busy = true;
        }
        return hipSuccess;
    });
}

hipError_t Stager::to_host(void* dst, const void* src, size_t bytes, int device, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (!staged(bytes)) {
        hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
        return e == hipSuccess ? hipStreamSynchronize(s) : e;
    }
    return run(bytes, device, s, [&](int w, int used, int64_t chunks) -> hipError_t {
        auto request = [&](int64_t c, Slot& sl) -> hipError_t {
            hipError_t e = idle(sl);
            if (e != hipSuccess) return e;
            const size_t off = (size_t)c * kChunk, len = std::min(kChunk, bytes - off);
            e = hipMemcpyAsync(sl.p, static_cast<const char*>(src) + off, len, hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipEventRecord(sl.ev, s);
            if (e == hipSuccess) sl.busy = true;
            return e;
        };
        hipError_t e = request(w, slot_[w][0]);
        int i = 0;
        for (int64_t c = w; e == hipSuccess && c < chunks; c += used, i ^= 1) {
            if (c + used < chunks) e = request(c + used, slot_[w][i ^ 1]);
            if (e == hipSuccess) e = idle(slot_[w][i]);  // this chunk has arrived
            if (e != hipSuccess) break;
            const size_t off = (size_t)c * kChunk, len = std::min(kChunk, bytes - off);
            std::memcpy(static_cast<char*>(dst) + off, slot_[w][i].p, len);
        }
        return e;
    });
}

// ---- device memory --------------------------------------------------------------------

hipError_t DevicePool::take(void** p, size_t bytes) {
    *p = nullptr;
    if (alloc_injected()) return hipErrorOutOfMemory;
    const size_t len = std::max<size_t>((bytes + 255) / 256 * 256, 256);
    for (int attempt = 0;; ++attempt) {
        for (size_t i = 0; i < slabs_.size(); ++i) {
            Slab& sl = slabs_[i];
            for (auto it = sl.free.begin(); it != sl.free.end(); ++it) {
                if (it->second < len) continue;
                const size_t off = it->first, rest = it->second - len;
                try {
                    blocks_.emplace(sl.base + off, Block{i, off, len});
                } catch (const std::bad_alloc&) {  // host memory; nothing has changed
                    return hipErrorOutOfMemory;
                }
                auto node = sl.free.extract(it);  // (its node is used again: no allocation)
                if (rest) {
                    node.key() = off + len;
                    node.mapped() = rest;
                    sl.free.insert(std::move(node));
                }
                *p = sl.base + off;
                return hipSuccess;
            }
        }
        if (attempt) return hipErrorOutOfMemory;  // (not reached: the new one has room)
        // A new allocation: what is expected, else a quarter of what is held (up to 32 MiB);
        // 1 MiB at a time for little memory: below 2 MiB the runtime cuts them from blocks of
        // its own in some microseconds, from there on they cost the call some 300 (the
        // first element-wise run of 405,005 ratings: 490 us with 3 MiB, 126 now).
        const size_t mib = size_t(1) << 20;
        size_t size = next_ >= 8 * mib ? next_ : held_ >= 32 * mib ? std::min(32 * mib, held_ / 4) : mib;
        size = std::max(size, len);
        next_ = 0;
        void* base = nullptr;
        hipError_t e = hipMalloc(&base, size);
        if (e != hipSuccess && size > len) {
            (void)hipGetLastError();
            size = len;
            e = hipMalloc(&base, size);
        }
        if (e != hipSuccess) {
            // What this pool and its peer hold without use goes back to the device first.
            (void)hipGetLastError();
            trim(0);
            if (peer_) peer_->trim(0);
            e = hipMalloc(&base, size);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        try {
            size_t at = 0;
            while (at < slabs_.size() && slabs_[at].base) ++at;
            if (at == slabs_.size()) slabs_.emplace_back();
            slabs_[at].free.emplace(0, size);
            slabs_[at].base = static_cast<char*>(base);
            slabs_[at].size = size;
        } catch (const std::bad_alloc&) {
            (void)hipFree(base);
            return hipErrorOutOfMemory;
        }
        held_ += size;
    }
}

void DevicePool::give(void* p) {
    const auto it = blocks_.find(p);
    if (it == blocks_.end()) return;
    const Block b = it->second;
    blocks_.erase(it);
    std::map<size_t, size_t>& fr = slabs_[b.slab].free;
    size_t off = b.off, len = b.len;
    auto next = fr.lower_bound(off);
    if (next != fr.end() && off + len == next->first) {
        len += next->second;
        next = fr.erase(next);
    }
    if (next != fr.begin()) {
        const auto prev = std::prev(next);
        if (prev->first + prev->second == off) {
            prev->second += len;
            return;
        }
    }
    try {
        fr.emplace(off, len);
    } catch (const std::bad_alloc&) {
        // Stays taken until release().
    }
}

void DevicePool::trim(size_t keep) {
    for (Slab& sl : slabs_) {
        if (held_ <= keep) return;
        if (!sl.base || sl.free.size() != 1 || sl.free.begin()->second != sl.size) continue;
        (void)hipFree(sl.base);
        held_ -= sl.size;
        sl = Slab{};
    }
}

void DevicePool::release() {
    for (Slab& sl : slabs_)
        if (sl.base) (void)hipFree(sl.base);
    slabs_.clear();
    blocks_.clear();
    held_ = 0;
    next_ = 0;
}

}  // namespace ccdk
