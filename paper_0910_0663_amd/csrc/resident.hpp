// The resident solver (resident.hip): a whole run of port-to-port sweeps and its
// residual checks in one cooperative launch, for circuits whose port operators fit
// the chip's registers.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

namespace vtm {

// Where the next residual check goes.  With adaptive checks, once two checks
// show the residual falling, the per-sweep rate predicts the sweeps left to the
// target; the next check comes after half of them (a multiple of m, at most
// 64 m), so checks thin out far from the target and return to every m sweeps
// near it.
struct Cadence {
    int64_t m = 1;
    bool adaptive = false;
    double reach = 0.5;     // fraction of the predicted sweeps to the target before the next check
    int64_t cap = 64;       // at most this many m between checks
    int64_t s_prev = -1, s_last = -1;
    double r_prev = 0.0, r_last = 0.0;
    __host__ __device__ void record(int64_t s, double r) {
        s_prev = s_last;
        r_prev = r_last;
        s_last = s;
        r_last = r;
    }
    __host__ __device__ int64_t next(double target) const {
        if (!adaptive || s_prev < 0 || !(r_last < r_prev) || !(r_last > 0.0) || !(target > 0.0) ||
            !(r_last > target))
            return m;
        const double rate = log(r_last / r_prev) / double(s_last - s_prev);  // < 0
        const double left = log(target / r_last) / rate;                       // > 0
        const int64_t k = int64_t(reach * left / double(m)) * m;
        const int64_t lo = k < m ? m : k;
        return lo > cap * m ? cap * m : lo;
    }
};

// With graphs, check intervals are m times a power of two (a few graphs cover them all).
__host__ __device__ inline int64_t graph_length(int64_t m, int64_t k) {
    int64_t len = m;
    while (2 * len <= k) len *= 2;
    return len;
}

// why a resident run ended (kAborted: never finished, a bounded wait ran out)
enum ResidentStop { kAborted = 0, kDone = 1, kBad = 2, kSweepLimit = 3, kStalled = 4, kMore = 5 };

constexpr int kResidentHist = 1024;             // checks of one launch
constexpr int64_t kResidentSweeps = 1 << 20;    // a launch ends at the first check after this many
// the largest check_every: chunks (at most 64 of it) are exchanged as 32-bit words
constexpr int64_t kResidentEvery = 1 << 20;

// How a run is controlled: on entry, and back as it ended (without bb and first).
struct ResidentControl {
    Cadence cad;
    double tol = 0.0;         // target of the relative residual
    double divergence = 0.0;  // above this (or not finite) the run ends as kBad
    double bb = 0.0;          // the residual's denominator, squared (unless ResidentArgs::bb is set)
    int64_t sweeps = 0, max_sweeps = 0;
    int64_t first = 1;        // sweeps before the first check
    int32_t inner = 0;        // inner solve of a refinement: ends at the target or when two checks in a
                              // row bring no 20% below the best; no history
    int32_t since = 0;
    int32_t pow2 = 0;         // intervals between checks are m times a power of two (graph_length)
    double best = 0.0;
};

// What a run leaves, in pinned host memory.
struct ResidentState {
    ResidentControl ctl;
    int32_t stop;             // ResidentStop; the host sets kAborted before the launch
    int32_t timeout;          // some workgroup's wait ran out
    int32_t checks;
    int32_t hist_len;
    double rel;
    double hist[kResidentHist];
    int64_t hist_sweeps[kResidentHist];
};

// What a run reads; T: FP64 or FP32 operators, waves and h.
template <typename T>
struct ResidentArgs {
    ResidentControl ctl;
    const double* bb;            // null, or where an earlier launch on the stream leaves ctl.bb
    int S;
    int64_t nports;
    const T* op;                 // packed triangles (packed) or column-group k x k blocks
    const int64_t* ofs;
    int packed;
    const int32_t *pn_off, *pn_pfirst, *port_off, *port_twin;
    const T *c, *beta, *gamma, *h;
    const T* w;                  // packed: line admittance per port, null: W for every one
    T W;
    const double *c64, *beta64, *gamma64, *gd, *g;
    T* a[2];                     // wave buffers; the first sweep reads a[cur]
    int cur;
    unsigned long long* slots;   // resident_slot_words words, zero before the first launch
    unsigned long long* sums;    // 2 words per workgroup, then the decision and the abort word, zero too
    unsigned epoch;              // tags of earlier launches on these words are at most this
    unsigned long long wait_ticks;  // bound of every wait (100 MHz)
    ResidentState* state;
};

template <typename T>
inline size_t resident_slot_words(int64_t nports) {
    return size_t(nports) * 2 * (sizeof(T) / 4);
}

// Sweeping workgroups of a run, 0 when it cannot run resident: some sub-circuit has more
// than 128 ports (dense operators: more than 512, or 320 port nodes; FP32, packed ones: more
// than 64), or the current device cannot hold every workgroup at once.
template <typename T>
int resident_blocks(int S, int max_npn, int max_ports, bool packed);

// One run.  hipErrorCooperativeLaunchTooLarge (or another launch error) leaves
// everything as it was.
template <typename T>
hipError_t launch_resident(const ResidentArgs<T>& args, int max_npn, int max_ports, hipStream_t st);

}  // namespace vtm
