// Device to host transfers of a context: its few words of sweep state (energies,
// counters, flags) and its amplitudes, through pinned memory of its own.
//
// A copy to pageable memory costs 10 to 25 us however small it is, some of 32 to 200
// KB three times that (it depends on the pages), and the host waits for each; a large
// one runs at 17 GB/s.  Here a kernel stores to mapped pinned memory: the words and
// amplitudes up to 512 KiB at once (6 KB 21 -> 11 us, 64 KB 11 to 36 -> 16, 512 KB 29
// -> 32), larger ones through four slots of that size, the host's copy out of one
// beside the stores into the others (1 MB 67 -> 57 us, 8 MB 500 -> 350; filled by the
// copy engine 395, slots of 256 KiB or 1 MiB 340 to 350 where these took 284).  A host
// read of the state words between chunks of sweeps, with the copies that went before:
// 65 -> 25 us; a solve of N=14, n^2<=4 937 -> 599 us.
//
// The pinned memory is one allocation no larger than the context's problems can use
// (the first 2 MiB of a process cost 0.3 ms to pin, 16 KB 0.02).
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
    size_t stage_off = 0, stage_cap = 0;  // the staging area after the words, or 0: plain copies
    hipEvent_t ev[kSlots] = {};
    int device = -1;  // of the memory that is read
    std::mutex mu;    // of the staging area and of `words` until they are copied out

    HostIO() = default;
    HostIO(const HostIO&) = delete;
    HostIO& operator=(const HostIO&) = delete;
    ~HostIO() {
        if (words_d) (void)hipHostFree(words);
        else std::free(words);
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }

    // the staging area that a download of so many bytes uses
    static size_t stage_of(size_t bytes) { return std::min(bytes, kSlot * kSlots); }

    // without pinned memory or events the plain copies stay; false: no memory at all.
    // stage: the largest stage_of() of the downloads to come; mem: the device memory
    // that will be read
    bool init(size_t nwords, size_t stage, const void* mem) {
        hipPointerAttribute_t at;
        if (hipPointerGetAttributes(&at, mem) == hipSuccess) device = at.device;
        const size_t nw = 8 * std::max<size_t>(nwords, 1);
        if (stage > kSlot)
            for (hipEvent_t& e : ev)
                if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) stage = 0;
        stage_off = (nw + 255) & ~(size_t)255;
        void *p = nullptr, *q = nullptr;
        if (hipHostMalloc(&p, stage_off + stage, hipHostMallocMapped | hipHostMallocPortable) == hipSuccess) {
            if (hipHostGetDevicePointer(&q, p, 0) == hipSuccess) {
                words = (char*)p;
                words_d = (char*)q;
                stage_cap = stage;
            } else {
                (void)hipHostFree(p);
            }
        }
        if (!words) words = (char*)std::malloc(nw);
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
        if (bytes == 0) return hipStreamSynchronize(s);  // (a problem may have no amplitudes)
        std::lock_guard<std::mutex> lock(mu);
        if (stage_of(bytes) > stage_cap || !here()) {
            hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
            return e == hipSuccess ? hipStreamSynchronize(s) : e;
        }
        char *stage = words + stage_off, *stage_d = words_d + stage_off;
        auto store = [&](size_t at, size_t off, size_t len) {
            const size_t w = len / 8;
            k_words_out<<<dim3((unsigned)std::min<size_t>((w + 255) / 256, 256)), 256, 0, s>>>(
                (double*)(stage_d + at), (const double*)((const char*)src + off), (int)w);
            return hipGetLastError();
        };
        if (bytes <= kSlot) {
            hipError_t e = store(0, 0, bytes);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e == hipSuccess) std::memcpy(dst, stage, bytes);
            return e;
        }
        const size_t n = (bytes + kSlot - 1) / kSlot;
        auto len = [&](size_t k) { return std::min(kSlot, bytes - k * kSlot); };
        hipError_t e = hipSuccess;
        auto issue = [&](size_t k) {
            e = store((k % kSlots) * kSlot, k * kSlot, len(k));
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
