// The host's side of a render's counts (host code only).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <string.h>

#include <chrono>
#include <thread>

#include "host_note.hpp"

namespace recogs {

// The host's side of HostNote: one pinned line per thread, allocated on the thread's first
// eager render and given back when the thread ends. A call waits for its own sequence
// number before it goes on, so the line serves any stream and device in turn.
// hipHostMalloc and hipHostFree are refused while any thread captures a stream in the
// global mode, unless the calling thread's own mode is relaxed. None of the calls here
// touches a captured stream, so they are made in that mode. A thread that still gets no line
// reads its counts back instead and asks again in its next render.
class KeyNote {
public:
    ~KeyNote() {
        if (!words_) return;
        const Relaxed mode;
        if (hipHostFree(words_) != hipSuccess) (void)hipGetLastError();
    }
    // words null when there is no pinned line, or the stream is being captured (nothing runs
    // then: the caller's read-back reports it)
    HostNote next(hipStream_t stream) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
            (void)hipGetLastError();
            return HostNote{nullptr, 0u};
        }
        if (cap != hipStreamCaptureStatusNone) return HostNote{nullptr, 0u};
        if (!words_) {
            const Relaxed mode;
            void *p = nullptr;
            if (hipHostMalloc(&p, 8 * sizeof(uint64_t),
                              hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess)
                words_ = (uint64_t *)memset(p, 0, 8 * sizeof(uint64_t));
            else
                (void)hipGetLastError();
        }
        if (++seq_ == 0) seq_ = 1;
        return HostNote{words_, seq_};
    }
    // The words, once the kernel that was given `note` has left them. Ends without them when
    // the stream reports an error or has run dry (asked each millisecond: a query may put
    // a marker behind the work in flight).
    hipError_t wait(const HostNote &note, hipStream_t stream, uint32_t (&out)[8]) const {
        using clock = std::chrono::steady_clock;
        const auto ms = std::chrono::milliseconds(1);
        auto ask = clock::now() + ms;
        for (uint32_t spins = 1;; ++spins) {
            if (arrived(note, out)) return hipSuccess;
            if ((spins & 255u) || clock::now() < ask) continue;
            const hipError_t e = query(stream);
            if (e != hipSuccess && e != hipErrorNotReady) return e;
            if (e == hipSuccess) return arrived(note, out) ? hipSuccess : hipErrorUnknown;
            (void)hipGetLastError();
            std::this_thread::yield();
            ask = clock::now() + ms;
        }
    }

private:
    struct Relaxed {   // the thread's capture mode, relaxed while this lives
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        Relaxed() { swap(); }
        ~Relaxed() { swap(); }
        void swap() {
            if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) (void)hipGetLastError();
        }
    };
    static hipError_t query(hipStream_t stream) {
        const Relaxed mode;
        return hipStreamQuery(stream);
    }
    static bool arrived(const HostNote &note, uint32_t (&out)[8]) {
        for (int k = 0; k < 8; ++k) {
            const uint64_t w = __atomic_load_n(note.words + k, __ATOMIC_ACQUIRE);
            if ((uint32_t)(w >> 32) != note.seq) return false;
            out[k] = (uint32_t)w;
        }
        return true;
    }
    uint64_t *words_ = nullptr;
    uint32_t seq_ = 0;
};

}  // namespace recogs
