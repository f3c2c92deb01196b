// Pieces shared by the closure and batch drivers.
#pragma once

#include <immintrin.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "cfpq_internal.h"

namespace cfpq {

// CFPQ_LOG in the environment names a file ("-": stderr) that receives JSON
// lines: one per loop of the host-driven closure, one per replay of captured
// loops, and one per closure call with its totals.  Each line is written
// with one call and flushed, so calls on several threads do not interleave
// within a line.
struct JsonLog {
    FILE* f = nullptr;
    bool own = false;
    JsonLog() {
        const char* v = std::getenv("CFPQ_LOG");
        if (!v || !*v) return;
        if (std::strcmp(v, "-") == 0) {
            f = stderr;
        } else {
            f = std::fopen(v, "a");
            own = f != nullptr;
        }
    }
    ~JsonLog() {
        if (own) std::fclose(f);
    }
    JsonLog(const JsonLog&) = delete;
    JsonLog& operator=(const JsonLog&) = delete;
    void line(const std::string& text) {
        if (!f) return;
        std::fputs((text + "\n").c_str(), f);
        std::fflush(f);
    }
};

inline const char* path_name(int32_t path) {
    switch (path) {
        case CFPQ_PATH_BITS: return "bits";
        case CFPQ_PATH_MFMA: return "mfma";
        case CFPQ_PATH_FP4: return "fp4";
        case CFPQ_PATH_ROWS: return "rows";
        case CFPQ_PATH_COLS: return "cols";
        default: return "auto";
    }
}

// Waits until the report for loop t has been written (or the stream failed).
template <typename Report>
hipError_t await_report(const Report* rep, int32_t t, hipStream_t s) {
    for (uint32_t spin = 1;; ++spin) {
        if (__atomic_load_n(&rep->loop, __ATOMIC_ACQUIRE) >= t) return hipSuccess;
        _mm_pause();
        if ((spin & 0xFFFF) == 0) {  // a few ms of spinning: is the stream still at work?
            const hipError_t e = hipStreamQuery(s);
            if (e == hipErrorNotReady) continue;
            if (e != hipSuccess) return e;
            return __atomic_load_n(&rep->loop, __ATOMIC_ACQUIRE) >= t ? hipSuccess : hipErrorUnknown;
        }
    }
}

// Waits for the stream when destroyed while armed: whatever ends a call early,
// no queued report outlives its use of the pinned buffer.
struct Drain {
    hipStream_t s;
    bool armed = true;
    ~Drain() {
        if (armed) (void)hipStreamSynchronize(s);
    }
};

// AUTO: the autotuned kernel of the size bucket, else the fp4 MFMA while fp32 sums
// are exact.  *tile is only changed for an autotuned choice.
int32_t choose_path(const Layout& L, int32_t requested, int32_t* tile = nullptr);

// Cost model of one product at this size for the dense kernel `path`
// (tuned_ms: its autotuned time, or 0).
HybridModel make_model(const Layout& L, int32_t path, float tuned_ms);

}  // namespace cfpq
