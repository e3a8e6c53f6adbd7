// Device to host transfers of a context: its few words of sweep state (energies,
// counters, flags) and its amplitudes, through pinned memory of its own.
//
// A copy to pageable memory costs 11 to 15 us however small it is, and the host
// waits for each; a large one runs at 17 GB/s.  Here a kernel stores to mapped
// pinned memory: the words at once, amplitudes through four slots of 512 KiB, the
// host's copy out of one beside the stores into the others.  The amplitudes of
// N=66, n^2<=36 (8.3 MB) take 480 -> 284 us (395 with the slots filled by the copy
// engine; slots of 256 KiB or 1 MiB 340 to 350), of N=66, n^2<=20 (2.7 MB) 155 ->
// 103.  A host read of the state words between chunks of sweeps, with the copies
// that went before: 65 -> 25 us; a solve of N=14, n^2<=4 937 -> 599 us.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <mutex>

namespace ccd {

static __global__ void __launch_bounds__(256) k_words_out(double* dst, const double* src, int n) {
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) dst[e] = src[e];
}

struct HostIO {
    static constexpr size_t kSlot = 512 * 1024;
    static constexpr int kSlots = 4;
    char* words = nullptr;    // host copy of the state words
    char* words_d = nullptr;  // its device address (pinned), or null: plain memory
    size_t words_cap = 0;
    char* stage = nullptr;  // kSlots pinned slots, or null: none to be had
    char* stage_d = nullptr;
    hipEvent_t ev[kSlots] = {};
    int device = -1;  // of the memory that is read
    std::mutex mu;    // of the slots and of `words` until they are copied out

    HostIO() = default;
    HostIO(const HostIO&) = delete;
    HostIO& operator=(const HostIO&) = delete;
    ~HostIO() {
        if (words_d) (void)hipHostFree(words);
        else std::free(words);
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        if (stage) (void)hipHostFree(stage);
    }

    // without pinned memory or events the plain copies stay; false: no memory at all.
    // mem: the device memory that will be read
    bool init(size_t nwords, const void* mem) {
        hipPointerAttribute_t at;
        if (hipPointerGetAttributes(&at, mem) == hipSuccess) device = at.device;
        words_cap = 8 * std::max<size_t>(nwords, 1);
        void* p = nullptr;
        if (hipHostMalloc(&p, words_cap, hipHostMallocMapped | hipHostMallocPortable) == hipSuccess) {
            void* q = nullptr;
            if (hipHostGetDevicePointer(&q, p, 0) == hipSuccess) {
                words = (char*)p;
                words_d = (char*)q;
            } else {
                (void)hipHostFree(p);
            }
        }
        if (!words) words = (char*)std::malloc(words_cap);
        bool ok = true;
        for (hipEvent_t& e : ev) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
        p = nullptr;
        if (ok && hipHostMalloc(&p, kSlot * kSlots, hipHostMallocMapped | hipHostMallocPortable) == hipSuccess) {
            void* q = nullptr;
            if (hipHostGetDevicePointer(&q, p, 0) == hipSuccess) {
                stage = (char*)p;
                stage_d = (char*)q;
            } else {
                (void)hipHostFree(p);
            }
        }
        (void)hipGetLastError();
        return words != nullptr;
    }

    // A caller may read a context while another GPU is current.  The null stream is
    // then that GPU's, and a kernel there cannot reach this memory; a copy can.
    bool here() const {
        int d = -1;
        return hipGetDevice(&d) == hipSuccess && d == device;
    }

    // the first n words at src into `words` (and to out), after all work on s
    hipError_t read_words(const void* src, size_t n, hipStream_t s, void* out = nullptr) {
        std::lock_guard<std::mutex> lock(mu);
        if (words_d && here()) {
            k_words_out<<<dim3((unsigned)std::min<size_t>((n + 1023) / 1024, 64)), 256, 0, s>>>(
                (double*)words_d, (const double*)src, (int)n);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        } else {
            hipError_t e = hipMemcpyAsync(words, src, 8 * n, hipMemcpyDeviceToHost, s);
            if (e != hipSuccess) return e;
        }
        const hipError_t e = hipStreamSynchronize(s);
        if (e == hipSuccess && out) std::memcpy(out, words, 8 * n);
        return e;
    }

    // bytes (a multiple of 8) from device memory to dst, after all work on s
    hipError_t download(void* dst, const void* src, size_t bytes, hipStream_t s) {
        std::lock_guard<std::mutex> lock(mu);
        if (!stage || !here()) {
            hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
            return e == hipSuccess ? hipStreamSynchronize(s) : e;
        }
        const size_t n = (bytes + kSlot - 1) / kSlot;
        auto len = [&](size_t k) { return std::min(kSlot, bytes - k * kSlot); };
        hipError_t e = hipSuccess;
        auto issue = [&](size_t k) {
            const size_t w = len(k) / 8;
            k_words_out<<<dim3((unsigned)std::min<size_t>((w + 255) / 256, 256)), 256, 0, s>>>(
                (double*)(stage_d + (k % kSlots) * kSlot), (const double*)((const char*)src + k * kSlot), (int)w);
            e = hipGetLastError();
            if (e == hipSuccess) e = hipEventRecord(ev[k % kSlots], s);
        };
        for (size_t k = 0; k < std::min<size_t>(n, kSlots) && e == hipSuccess; k++) issue(k);
        for (size_t k = 0; k < n && e == hipSuccess; k++) {
            e = hipEventSynchronize(ev[k % kSlots]);
            if (e != hipSuccess) break;
            std::memcpy((char*)dst + k * kSlot, stage + (k % kSlots) * kSlot, len(k));
            if (k + kSlots < n) issue(k + kSlots);
        }
        if (e != hipSuccess) (void)hipStreamSynchronize(s);  // nothing may still write to the slots
        return e;
    }
};

}  // namespace ccd
