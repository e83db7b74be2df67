// host_copy.h -- checks, conversions and first touches of large host field arrays, split
// over a few threads, and the buffers that several callers' copies go through.
//
// A solve's fields cross the host's memory once on the way in and once out; on one core
// that is bound by page faults and scalar code (a burst of twelve served solves, 288 MB
// each way: 48 ms to submit and 45 to fetch on one core, 22 and 12.5 so, against 3 ms on
// the device).  Up to eight threads, each with at least 2 MB, share it.
#pragma once
#include <sys/mman.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <thread>
#include <vector>

namespace eifp {

// f(begin, end) over [0, n) of items of `bytes` bytes; the calling thread takes a share, and
// all of what threads that cannot be started would have taken.
template <class F>
void host_ranges(long long n, long long bytes, F f) {
    constexpr int kMaxThreads = 8;
    constexpr long long kMinBytes = 2LL << 20;
    const long long want = std::min<long long>(kMaxThreads, n * bytes / kMinBytes);
    const int nt = (int)std::max<long long>(1, std::min<long long>(want, std::thread::hardware_concurrency()));
    const long long per = (n + nt - 1) / nt;
    std::vector<std::thread> ts;
    int t = 1;
    try {
        ts.reserve(nt);
        for (; t < nt; ++t) ts.emplace_back(f, std::min(n, t * per), std::min(n, (t + 1) * per));
    } catch (...) {
    }
    f(0LL, std::min(n, per));
    if (t < nt) f(std::min(n, t * per), n);
    for (std::thread& x : ts) x.join();
}

// The first index of [begin, end) whose value is NaN or infinite (end: none); with COPY, also
// copies the values to dst, rounded to TO.  Branch-free blocks: x * 0 is NaN for such x
// alone.  COPY is a template argument so that the loop is free of branches as well (98304
// values: 35.8 us with a test of dst inside, 17.0 without; plain isfinite calls 37.5).
template <bool COPY, typename TO>
long long check_block(const double* src, TO* dst, long long begin, long long end) {
    for (long long b = begin; b < end; b += 4096) {
        const long long e = std::min(end, b + 4096);
        double a[8] = {};
        long long q = b;
        for (; q + 8 <= e; q += 8)
            for (int i = 0; i < 8; ++i) {
                a[i] += src[q + i] * 0.0;
                if constexpr (COPY) dst[q + i] = (TO)src[q + i];
            }
        for (; q < e; ++q) {
            a[0] += src[q] * 0.0;
            if constexpr (COPY) dst[q] = (TO)src[q];
        }
        double s = 0;
        for (double x : a) s += x;
        if (!(s == 0.0))
            for (q = b; q < e; ++q)
                if (!std::isfinite(src[q])) return q;
    }
    return end;
}
template <typename TO>
long long check_finite(const double* src, TO* dst, long long n) {
    std::mutex mu;
    long long first = n;
    host_ranges(n, 8, [&](long long b, long long e) {
        const long long q = dst ? check_block<true>(src, dst, b, e) : check_block<false>(src, dst, b, e);
        if (q < e) {
            std::lock_guard<std::mutex> lk(mu);
            first = std::min(first, q);
        }
    });
    return first;
}

// At most N buffers, each allocated by the first call that finds none free and kept until
// release().  take() waits for no other user: with all N out, or none to be had, it returns
// null and the caller does without.
template <int N>
class BufferPool {
    std::mutex mu_;
    void* free_[N] = {};
    int nfree_ = 0, made_ = 0;

public:
    template <class Alloc>
    void* take(Alloc alloc) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (nfree_ > 0) return free_[--nfree_];
            if (made_ == N) return nullptr;
            ++made_;
        }
        void* p = alloc();
        if (!p) {
            std::lock_guard<std::mutex> lk(mu_);
            --made_;
        }
        return p;
    }
    void give(void* p) {
        std::lock_guard<std::mutex> lk(mu_);
        free_[nfree_++] = p;
    }
    // every buffer is back; the pool is empty again
    template <class Free>
    void release(Free f) {
        while (nfree_ > 0) f(free_[--nfree_]);
        made_ = 0;
    }
};

// Whether the array's pages look mapped: 16 of them, spread over it (a mincore call each).
inline bool looks_resident(const char* p, long long bytes) {
    constexpr long long kSamples = 16, kPage = 4096;
    for (long long i = 0; i < kSamples; ++i) {
        unsigned char in = 0;
        const std::uintptr_t at = (std::uintptr_t)(p + (bytes - 1) * i / (kSamples - 1)) & ~(std::uintptr_t)(kPage - 1);
        if (mincore((void*)at, kPage, &in) != 0 || !(in & 1)) return false;
    }
    return true;
}

// Fault the pages of a large output array in before a copy fills it (256^3 fields: 78 -> 56
// ms; of no use below 32 MB).  An array that has them, as one that a program reads its fields
// into again and again, is left alone: touching it cost 1.4 ms at 256^3 and 0.3 at 128^3.
inline void touch_pages(void* p, long long bytes) {
    if (bytes < (32LL << 20) || looks_resident((const char*)p, bytes)) return;
    char* c = (char*)p;
    host_ranges(bytes / 4096, 4096, [c](long long b, long long e) {
        for (long long q = b; q < e; ++q) {
            volatile char* x = c + q * 4096;
            *x = *x;
        }
    });
}

}  // namespace eifp
