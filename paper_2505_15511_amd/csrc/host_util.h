// Host-side helpers shared by the stand-alone entry points (index, quality measures, initialisation).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "nomad.h"

// Device memory that calls and contexts have given back, kept for the next one that asks for about as much.  hipMalloc and
// hipFree of work space cost a call on small inputs more than its kernels (and 1.5 ms a call for the half gigabyte of a
// million points: page tables).  Bounded: at most kKeepBytes in all, nothing larger than half of that, and what 1,024 requests
// in a row have not taken is freed; when the device runs out of memory everything kept is freed before the request fails, and
// nomad_release_memory frees it for others (torch's allocator cannot ask for it).
// A block comes back only after the work that used it has been waited for, so any thread and stream may take it next.
class DevicePool {
public:
    // held: the block's size, which may be half as large again (and 64 KB) as what was asked for
    hipError_t take(void** p, size_t bytes, size_t* held = nullptr) {
        *p = nullptr;
        const size_t want = (std::max<size_t>(bytes, 1) + kGrain - 1) / kGrain * kGrain;
        int device = 0;
        hipError_t e = hipGetDevice(&device);
        if (e != hipSuccess) return e;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            ++requests_;
            size_t best = kept_.size();
            for (size_t i = 0; i < kept_.size(); ++i)
                if (kept_[i].device == device && kept_[i].bytes >= want && kept_[i].bytes <= want + want / 2 + (64u << 10) &&
                    (best == kept_.size() || kept_[i].bytes < kept_[best].bytes))
                    best = i;
            if (best < kept_.size()) {
                *p = kept_[best].p;
                sizes_[*p] = {kept_[best].bytes, device};
                if (held) *held = kept_[best].bytes;
                bytes_ -= kept_[best].bytes;
                kept_.erase(kept_.begin() + (long)best);
                return hipSuccess;
            }
        }
        e = hipMalloc(p, want);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            trim(0);
            e = hipMalloc(p, want);
        }
        if (e != hipSuccess) { *p = nullptr; return e; }
        if (held) *held = want;
        std::lock_guard<std::mutex> lock(mutex_);
        sizes_[*p] = {want, device};
        return hipSuccess;
    }
    // p from take; no work that uses it is pending
    void give(void* p) {
        if (!p) return;
        std::vector<Block> old;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            const auto it = sizes_.find(p);
            const Size s = it->second;
            sizes_.erase(it);
            Block b{p, s.bytes, s.device, requests_};
            if (b.bytes > kKeepBytes / 2) old.push_back(b);
            else { kept_.push_back(b); bytes_ += b.bytes; }
            drop(old, kKeepBytes, 1024);
        }
        for (const Block& b : old) (void)hipFree(b.p);
    }
    void trim(size_t keep) {
        std::vector<Block> old;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            drop(old, keep, ~0ull >> 1);
        }
        for (const Block& b : old) (void)hipFree(b.p);
    }
    static DevicePool& get() {
        static DevicePool* pool = new DevicePool();   // lives as long as the process: the runtime may be gone before static destructors run
        return *pool;
    }

private:
    static constexpr size_t kGrain = 512, kKeepBytes = (size_t)2 << 30;
    struct Block { void* p; size_t bytes; int device; uint64_t since; };
    struct Size { size_t bytes; int device; };
    // oldest first (they are in the order of their return): what is over `keep` bytes, and what `age` requests passed by
    void drop(std::vector<Block>& out, size_t keep, uint64_t age) {
        size_t i = 0;
        while (i < kept_.size() && (bytes_ > keep || requests_ - kept_[i].since > age)) { bytes_ -= kept_[i].bytes; out.push_back(kept_[i]); ++i; }
        kept_.erase(kept_.begin(), kept_.begin() + (long)i);
    }
    std::mutex mutex_;
    std::vector<Block> kept_;
    std::unordered_map<void*, Size> sizes_;   // of the blocks in use
    size_t bytes_ = 0;
    uint64_t requests_ = 0;
};

namespace {

struct Buffers {   // device allocations of one call, given back on every path once its stream has been waited for
    hipStream_t stream = nullptr;
    std::vector<void*> ptrs;
    explicit Buffers(hipStream_t st) : stream(st) {}
    ~Buffers() {
        if (ptrs.empty()) return;
        (void)hipStreamSynchronize(stream);   // (a call that has run to its end has waited already)
        for (void* p : ptrs) DevicePool::get().give(p);
    }
    template <typename T>
    hipError_t alloc(T** p, size_t count) {
        void* q = nullptr;
        hipError_t e = DevicePool::get().take(&q, std::max<size_t>(count, 1) * sizeof(T));
        *p = (T*)q;
        if (e == hipSuccess) ptrs.push_back(q);
        return e;
    }
};

// A word that a call reads back while the device goes on: pinned memory and an event, both kept for the next call (making
// them costs more than a copy).  At most kKeep of them are kept.
class HostWord {
public:
    ~HostWord() {
        if (!s_.word) return;
        if (pending_) (void)hipEventSynchronize(s_.event);
        {
            std::lock_guard<std::mutex> lock(mutex());
            if (kept().size() < kKeep) { kept().push_back(s_); return; }
        }
        release(s_);
    }
    hipError_t take() {
        int device = 0;
        hipError_t e = hipGetDevice(&device);
        if (e != hipSuccess) return e;
        {
            std::lock_guard<std::mutex> lock(mutex());
            for (size_t i = kept().size(); i-- > 0;)
                if (kept()[i].device == device) {
                    s_ = kept()[i];
                    kept().erase(kept().begin() + (long)i);
                    return hipSuccess;
                }
        }
        Slot s{nullptr, nullptr, device};
        if ((e = hipEventCreateWithFlags(&s.event, hipEventDisableTiming)) != hipSuccess) return e;
        if ((e = hipHostMalloc((void**)&s.word, sizeof(unsigned long long), hipHostMallocDefault)) != hipSuccess) { (void)hipEventDestroy(s.event); return e; }
        s_ = s;
        return hipSuccess;
    }
    // the word is written by a kernel that has been enqueued
    hipError_t record(hipStream_t st) {
        const hipError_t e = hipEventRecord(s_.event, st);
        if (e == hipSuccess) pending_ = true;
        return e;
    }
    hipError_t wait() { pending_ = false; return hipEventSynchronize(s_.event); }
    unsigned long long value() const { return *s_.word; }
    // for a kernel to write and the host to read once it has waited for the stream: no copy on the way
    unsigned long long* word() const { return s_.word; }

private:
    static constexpr size_t kKeep = 8;
    struct Slot { unsigned long long* word; hipEvent_t event; int device; };
    static void release(const Slot& s) { (void)hipHostFree(s.word); (void)hipEventDestroy(s.event); }
    static std::mutex& mutex() { static std::mutex* m = new std::mutex(); return *m; }   // (both outlive the runtime's own statics)
    static std::vector<Slot>& kept() { static std::vector<Slot>* k = new std::vector<Slot>(); return *k; }
    Slot s_{nullptr, nullptr, 0};
    bool pending_ = false;
};

struct HostArrays {   // small host arrays that travel to the device in one copy, which has been waited for when they go
    std::vector<uint8_t> bytes;
    uint8_t* device = nullptr;
    hipStream_t stream = nullptr;
    ~HostArrays() { if (device) (void)hipStreamSynchronize(stream); }   // (a call that has run to its end has waited already)
    template <typename T>
    size_t add(const std::vector<T>& v) {   // -> offset
        const size_t at = (bytes.size() + 15) / 16 * 16;
        bytes.resize(at + std::max<size_t>(v.size(), 1) * sizeof(T));
        if (!v.empty()) memcpy(bytes.data() + at, v.data(), v.size() * sizeof(T));
        return at;
    }
    hipError_t upload(Buffers& buf, hipStream_t st) {
        stream = st;
        hipError_t e = buf.alloc(&device, bytes.size());
        return e != hipSuccess ? e : hipMemcpyAsync(device, bytes.data(), bytes.size(), hipMemcpyHostToDevice, st);
    }
    template <typename T>
    T* at(size_t offset) const { return (T*)(device + offset); }
};

#define KTRY(call)                                                          \
    do {                                                                    \
        hipError_t e_ = (call);                                             \
        if (e_ != hipSuccess) return e_ == hipErrorOutOfMemory ? NOMAD_E_OOM : NOMAD_E_HIP; \
    } while (0)

inline uint32_t blocks_of(int64_t items, int per) { return (uint32_t)((items + per - 1) / per); }

}  // namespace
