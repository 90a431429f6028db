// Resident port-to-port sweeps.
//
// A small circuit's sweep as a launch of its own costs 4-8 us, nearly all of it
// the launch and the first round trips to memory, and each residual check another
// 25-30 us of launches and host round trip.  Here one cooperative launch holds
// every sub-circuit's port operator in registers and runs all the sweeps and
// checks of a solve: workgroups exchange waves directly, each waiting only for the
// ports of its own neighbours, so there is no grid-wide barrier between sweeps (the
// iteration is the same: sweep k + 1 of a sub-circuit reads the waves sweep k of its
// neighbours sent).  Bound by the exchange's latency; alone it takes 1.3 us a sweep up to
// 400 workgroups, 1.6 at 1,024, 3.1 at 4,096 (there the polls' traffic).  Measured, solve
// before and after: 64x64 in 16x16 blocks to 1e-10 (296 sweeps) 1.3-1.5 -> 0.50 ms;
// 331x290 in random cuts (272 sweeps) 1.7 -> 0.69 ms; 768x640 in 8x8 blocks (7,680
// sub-circuits, 832 sweeps) 6.9 -> 2.5 ms, 3.0 us a sweep.
//
// A circuit runs resident whenever it fits.  At the largest that do, solves, a launch per
// sweep and resident, FP64 and FP32: 8,100 sub-circuits of 32 ports 4.2 -> 1.7 and 3.8 -> 2.0
// ms, 1,260 of 64 2.2 -> 1.0 and 2.2 -> 1.1; FP64 506 of 96 2.1 -> 0.8, 506 of 128 3.1 -> 1.4,
// 448 dense ones of 96 6.1 -> 2.8; a compute unit each, 255 of 384 ports 12.4 -> 4.8 and
// 8.7 -> 4.2.
//
// Exchange.  A wave travels as 8-byte words, each 32 bits of data and the 32-bit
// number of its sweep (FP64: two words), written and read as relaxed agent-scope
// atomics: a reader that finds the number it waits for has the data, with no fence
// and no separate flag.  Two words sets alternate.  A writer reaches a set again
// only two sweeps later, after it has received the wave its twin sent between, and
// the twin sent that after its workgroup had read the earlier set.
//
// Checks.  Every workgroup sends its sum of squares of the port residual the same
// way; one more workgroup adds them in a fixed order, decides (the rules of the host
// driver) and publishes the sweeps until the next check, or 0.
//
// Every wait is bounded: one that runs out raises the abort word, which all waits
// look at, the kernel ends, and the host runs the solve with a launch per sweep.
#include "resident.hpp"

#include "kernels.hpp"
#include "layout.hpp"

#include <algorithm>

namespace vtm {

namespace {

typedef unsigned long long u64;

__device__ inline u64 word_load(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void word_store(u64* p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ inline void send(u64* slot, double v, unsigned tag) {
    const u64 b = u64(__double_as_longlong(v)), t = u64(tag) << 32;
    word_store(slot, (b & 0xffffffffull) | t);
    word_store(slot + 1, (b >> 32) | t);
}
__device__ inline void send(u64* slot, float v, unsigned tag) {
    word_store(slot, u64(__float_as_uint(v)) | (u64(tag) << 32));
}
__device__ inline bool receive(const u64* slot, unsigned tag, double& v) {
    const u64 lo = word_load(slot), hi = word_load(slot + 1);
    if (unsigned(lo >> 32) != tag || unsigned(hi >> 32) != tag) return false;
    v = __longlong_as_double((long long)((lo & 0xffffffffull) | (hi << 32)));
    return true;
}
__device__ inline bool receive(const u64* slot, unsigned tag, float& v) {
    const u64 w = word_load(slot);
    if (unsigned(w >> 32) != tag) return false;
    v = __uint_as_float(unsigned(w));
    return true;
}

// The waves' words through buffer instructions: an FP64 wave's two words are one
// 16-byte access (each word carries its own tag, so only 8-byte halves need to be
// whole), which halves the requests of a poll.  Agent scope (sc1), as an atomic's;
// the empty asm before a load keeps the compiler from reusing an earlier one.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
constexpr int kAgent = 16;
__device__ inline void send(__amdgpu_buffer_rsrc_t r, unsigned slot, double v, unsigned tag) {
    const u64 b = u64(__double_as_longlong(v));
    const u32x4 w = {unsigned(b), tag, unsigned(b >> 32), tag};
    __builtin_amdgcn_raw_buffer_store_b128(w, r, int(slot * 16u), 0, kAgent);
}
__device__ inline void send(__amdgpu_buffer_rsrc_t r, unsigned slot, float v, unsigned tag) {
    const u32x2 w = {__float_as_uint(v), tag};
    __builtin_amdgcn_raw_buffer_store_b64(w, r, int(slot * 8u), 0, kAgent);
}
__device__ inline bool receive(__amdgpu_buffer_rsrc_t r, unsigned slot, unsigned tag, double& v) {
    asm volatile("" ::: "memory");
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, int(slot * 16u), 0, kAgent);
    v = __longlong_as_double((long long)(u64(w.x) | (u64(w.z) << 32)));
    return w.y == tag && w.w == tag;
}
__device__ inline bool receive(__amdgpu_buffer_rsrc_t r, unsigned slot, unsigned tag, float& v) {
    asm volatile("" ::: "memory");
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, int(slot * 8u), 0, kAgent);
    v = __uint_as_float(w.x);
    return w.y == tag;
}

// Repeats `ready` for the lanes that `want` it until it holds for all of them; false
// when the bound ran out here or elsewhere.  Wave-uniform (all lanes of a wavefront
// call it together).  The clock and the abort word are looked at once in 256 tries;
// a bound of 0 gives up after the first.
template <typename F>
__device__ inline bool wait_for(bool want, F ready, u64* abort_word, unsigned tag, u64 ticks) {
    u64 t0 = 0;
    for (unsigned n = 1;; ++n) {
        if (want) want = !ready();  // a lane that has its data asks no more
        if (!__any(want)) return true;
        if ((n & 255u) == 0 || ticks == 0) {
            if (unsigned(word_load(abort_word)) == tag) return false;
            const u64 now = __builtin_amdgcn_s_memrealtime();
            if (t0 == 0) t0 = now;
            if (now - t0 >= ticks) {
                word_store(abort_word, tag);
                return false;
            }
        }
    }
}

// Bound of a wait that lasts as long as the run of n sweeps before it: 50 us more a sweep,
// seven times what the slowest takes.
__device__ inline u64 run_ticks(u64 ticks, unsigned n) { return ticks ? ticks + u64(n) * 5000 : 0; }

// Shapes by the largest port count QB (per_simd: wavefronts a SIMD should hold, which
// bounds the registers; more sub-circuits then fit the chip) of a sub-circuit.  Row p of the operator
// (lane) is port p's node against every port's node: z_n(p) = sum_p' S(n_p, n_p') c_p' a_p'.
// As compiled, FP64 of up to 32, 64 and 128 ports spills 6 to 9 registers and FP32 in sixteens
// one, all written once before the sweeps.
// Up to 32 ports, a wavefront takes two sub-circuits, all 32 columns of a row in a
// lane (64 registers in FP64), and a workgroup one wavefront or eight (kManySubs).  Above, a workgroup takes one: RG groups of 64 rows
// by CG groups of COLS columns, the partial sums meeting in LDS; 16-32 columns a lane
// keep the chain of multiply-adds short and the registers low.
//
// FP32 (packed operators, up to 64 ports; dense ones: k_resident_wide_f) forms z in the order of the packed sweep of a
// launch per sweep (ports.hip), bit for bit: row r is port node r, and lane r holds for
// each diagonal d both S(r, r + d) and S(r - d, r); t = c a summed per node is staged
// between zeros.  An FP32 inner solve stops where rounding is a visible part of its
// residual, so another order would now and then end it at another check.
template <int QB>
struct Shape;
template <>
struct Shape<32> {
    static constexpr int RG = 1, CG = 1, COLS = 32;
    template <typename T>
    static constexpr int per_simd() { return 4; }
};
template <>
struct Shape<64> {
    static constexpr int RG = 1, CG = 4, COLS = 16;
    template <typename T>
    static constexpr int per_simd() { return 5; }
};
template <>
struct Shape<96> {
    static constexpr int RG = 2, CG = 4, COLS = 24;
    template <typename T>
    static constexpr int per_simd() { return 4; }
};
template <>
struct Shape<128> {
    static constexpr int RG = 2, CG = 4, COLS = 32;
    template <typename T>
    static constexpr int per_simd() { return 4; }
};

// threads of a workgroup of SUBS sub-circuits (more than one: 32 lanes each)
template <int QB, int SUBS>
constexpr int kThreads = SUBS > 1 ? 32 * SUBS : 64 * Shape<QB>::RG * Shape<QB>::CG;

// pair m of diagonals of a packed triangle (ports.hip)
__device__ inline int packed_at(int k, int i, int j) {
    const int lo = min(i, j), d = max(i, j) - lo, m = d >> 1;
    return 2 * m * (k - m + 1) + 2 * lo + (d & 1);
}

// The last workgroup controls the run: it collects the n other workgroups' sums at
// every check, decides, and publishes.  (In a workgroup of its own the decision's
// logarithms hold no registers beside an operator.)
template <typename T>
__device__ __forceinline__ void control(const ResidentArgs<T>& A, unsigned n) {
    __shared__ double red[8];
    __shared__ int bad;
    __shared__ unsigned next_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    u64* const decision = A.sums + 2 * size_t(n);
    u64* const abort_word = decision + 1;
    ResidentState* const st = A.state;
    ResidentControl ctl = A.ctl;
    if (A.bb) ctl.bb = *A.bb;
    int checks = 0, hist = 0;
    unsigned tag = A.epoch, run = unsigned(ctl.first);
    if (tid == 0) bad = 0;
    while (true) {
        tag += run;
        // every workgroup's sum: each thread its strided share in order, then a tree
        double sum = 0.0;
        for (unsigned b0 = 0; b0 < n; b0 += blockDim.x) {
            double v = 0.0;
            const unsigned b = b0 + tid;
            const u64* const slot = A.sums + 2 * size_t(b < n ? b : 0);
            if (!wait_for(b < n, [&] { return receive(slot, tag, v); }, abort_word, A.epoch + 1,
                          run_ticks(A.wait_ticks, run))) {
                bad = st->timeout = 1;
                break;
            }
            sum += b < n ? v : 0.0;
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
        if (lane == 0) red[wave] = sum;
        __syncthreads();
        if (bad) return;
        if (tid == 0) {
            sum = red[0];
            for (int v = 1; v < waves; ++v) sum += red[v];
            const double rel = ctl.bb > 0.0 ? sqrt(sum / ctl.bb) : sqrt(sum);
            ctl.sweeps += run;
            ++checks;
            int stop = kAborted;
            const bool finite = isfinite(rel);
            if (!ctl.inner) {
                st->hist[hist] = rel;
                st->hist_sweeps[hist] = ctl.sweeps;
                ++hist;
                if (!finite || rel > ctl.divergence)
                    stop = kBad;
                else if (rel <= ctl.tol)
                    stop = kDone;
                else if (ctl.sweeps >= ctl.max_sweeps)
                    stop = kSweepLimit;
            } else {
                const bool improved = rel < 0.8 * ctl.best;
                if (rel < ctl.best) ctl.best = rel;
                ctl.since = improved ? 0 : ctl.since + 1;
                if (!finite)
                    stop = kBad;
                else if (rel <= ctl.tol)
                    stop = kDone;
                else if (ctl.since >= 2)
                    stop = kStalled;
                else if (ctl.sweeps >= ctl.max_sweeps)
                    stop = kSweepLimit;
            }
            unsigned nx = 0;
            if (stop == kAborted) {
                ctl.cad.record(ctl.sweeps, rel);
                if (hist == kResidentHist || ctl.sweeps - A.ctl.sweeps >= kResidentSweeps) {
                    stop = kMore;
                } else {
                    int64_t n2 = ctl.cad.next(ctl.inner && ctl.tol > 1.0 ? 1.0 : ctl.tol);
                    if (ctl.pow2) n2 = graph_length(ctl.cad.m, n2);
                    if (n2 > ctl.max_sweeps - ctl.sweeps) n2 = ctl.max_sweeps - ctl.sweeps;
                    nx = unsigned(n2);
                }
            }
            if (nx == 0) {
                st->ctl = ctl;
                st->checks = checks;
                st->hist_len = hist;
                st->rel = rel;
                st->stop = stop;
            }
            word_store(decision, u64(nx) | (u64(tag) << 32));
            next_s = nx;
        }
        __syncthreads();
        run = next_s;
        if (run == 0) return;
        __syncthreads();  // next_s is read before the next check writes it
    }
}

// One check of a sweeping workgroup: its sum of squares of the port residual is sent,
// and next_s, the sweeps since the check before, becomes those until the next one.  A thread of the first `waves`
// wavefronts that is an owner holds port p, the entry base + row of first, cnt, xs and
// vs.  False: a wait ran out.
//
// The residual from port quantities: with o and an the waves that left and
// arrived in this sweep, x_i = (o - gamma a) / beta on this side of a wire and
// x_j = (an - gamma o_prev) / beta on the other (both ends share the wire's
// coefficients; the twin's incoming wave was this port's previous one).
template <typename T>
__device__ __forceinline__ bool residual_check(const ResidentArgs<T>& A, unsigned nb, bool owner, int p, int base,
                                               int row, T o, T a, T an, T o_prev, double* xs, double* vs, double* red,
                                               int waves, const int32_t* first, const int32_t* cnt, int& bad,
                                               unsigned& next_s, unsigned tag, unsigned abort_tag) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    u64* const decision = A.sums + 2 * size_t(nb);
    double be64 = 1.0, ga64 = 0.0;
    if (owner) {
        be64 = A.beta64[p];
        ga64 = A.gamma64[p];
        xs[base + row] = (double(o) - ga64 * double(a)) / be64;
    }
    __syncthreads();
    if (bad) return false;
    if (owner) {
        const double xj = (double(an) - ga64 * double(o_prev)) / be64;
        vs[base + row] = A.gd[p] * xs[base + first[base + row]] + A.g[p] * xj - A.c64[p] * double(a);
    }
    __syncthreads();
    double rr = 0.0;
    if (owner && first[base + row] == row) {
        double r = 0.0;
        for (int i = 0; i < cnt[base + row]; ++i) r += vs[base + row + i];
        rr = r * r;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) rr += __shfl_xor(rr, d);
    if (lane == 0) red[wave] = rr;
    __syncthreads();
    if (tid == 0) {
        rr = red[0];
        for (int v = 1; v < waves; ++v) rr += red[v];
        send(A.sums + 2 * size_t(blockIdx.x), rr, tag);
    }
    if (wave == 0) {
        unsigned nx = 0;
        const bool ok = wait_for(
            true,
            [&] {
                const u64 v = word_load(decision);
                nx = unsigned(v);
                return unsigned(v >> 32) == tag;
            },
            decision + 1, abort_tag, run_ticks(A.wait_ticks, next_s));  // (next_s: the sweeps before this check)
        if (!ok) bad = A.state->timeout = 1;
        next_s = nx;
    }
    __syncthreads();
    return !bad;
}

// staged t of one sub-circuit: rows of zeros before and after it
template <int QB>
constexpr int kSpan = 3 * (QB <= 32 ? 32 : 64);

template <typename T, int QB, int SUBS>
__global__ void __launch_bounds__((kThreads<QB, SUBS>), Shape<QB>::template per_simd<T>())
    k_resident(ResidentArgs<T> A) {
    const unsigned nb = gridDim.x - 1;         // workgroups that sweep
    if (blockIdx.x == nb) {
        control<T>(A, nb);
        return;
    }
    using Sh = Shape<QB>;
    constexpr int RG = Sh::RG, CG = Sh::CG, COLS = Sh::COLS;
    constexpr bool MANY = SUBS > 1;            // 32 lanes a sub-circuit
    constexpr int ROWS = MANY ? 32 : 64 * RG;  // rows (ports) of a sub-circuit
    constexpr int ALL = ROWS * SUBS;           // of the workgroup's
    constexpr int LOCAL = SUBS > 2 ? ALL : 0;  // waves between its sub-circuits go through LDS
    constexpr int STAGE = CG * COLS + 2;       // staged c a of a sub-circuit (the pad keeps two sub-circuits'
                                               // broadcast reads in different banks)
    constexpr int W = sizeof(T) / 4;           // words of a wave
    constexpr bool ORDERED = sizeof(T) == 4;   // the packed sweep's order (see above)
    constexpr int CHUNKS = ORDERED && CG > 1 ? 8 : CG;
    __shared__ alignas(16) T ca[SUBS][STAGE];
    __shared__ T zp[CHUNKS][ALL];
    __shared__ T lex[2][LOCAL ? LOCAL : 1];
    __shared__ T ts[ORDERED ? SUBS : 1][ORDERED ? kSpan<QB> : 1];
    __shared__ double xs[ALL], vs[ALL], red[8];
    __shared__ int32_t node[ALL], first[ALL], cnt[ALL];
    __shared__ int bad;
    __shared__ unsigned next_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int unit = xcd_block(blockIdx.x, nb);
    const int sub = MANY ? tid >> 5 : 0;
    const int rg = MANY ? 0 : wave % RG, cg = MANY ? 0 : wave / RG;
    const int row = MANY ? (lane & 31) : rg * 64 + lane;
    const int s = min(unit * SUBS + sub, A.S - 1);
    const bool real = unit * SUBS + sub < A.S;
    const int p0 = A.port_off[s], q = real ? A.port_off[s + 1] - p0 : 0;
    const int k0 = A.pn_off[s], k = A.pn_off[s + 1] - k0;
    const int base = sub * 32;                 // this sub-circuit's entries of node, first, cnt, xs, vs
    const bool owner = cg == 0 && row < q;     // this thread exchanges port p0 + row
    u64* const abort_word = A.sums + 2 * size_t(nb) + 1;
    const __amdgpu_buffer_rsrc_t slots =
        __builtin_amdgcn_make_buffer_rsrc(A.slots, 0, int(unsigned(A.nports) * unsigned(W) * 16u), 0x00020000);
    ResidentState* const st = A.state;

    // ports of each node: node, first and count per port
    if (tid == 0) bad = 0, next_s = unsigned(A.ctl.first);
    if (cg == 0) {
        for (int j = row; j < (real ? k : 0); j += ROWS) {
            const int f0 = A.pn_pfirst[k0 + j] - p0, f1 = A.pn_pfirst[k0 + j + 1] - p0;
            for (int p = f0; p < f1; ++p) {
                node[base + p] = j;
                first[base + p] = f0;
                cnt[base + p] = f1 - f0;
            }
        }
        for (int j = row; j < STAGE; j += ROWS) ca[sub][j] = T(0);
    }
    __syncthreads();
    if constexpr (ORDERED)
        for (int j = row; cg == 0 && j < kSpan<QB>; j += ROWS) ts[sub][j] = T(0);
    // this lane's diagonals when ORDERED: chunks of 8, cg and cg + 4 of them with several wavefronts
    auto diagonal = [&](int j) { return CG == 1 ? j : 8 * (j < 8 ? cg : cg + 4) + (j & 7); };
    // the operator's row, columns cg COLS .. of this lane
    T op[COLS], lo[ORDERED ? COLS : 1];
    if constexpr (ORDERED) {
        const T* blk = A.op + A.ofs[s];
#pragma unroll
        for (int j = 0; j < COLS; ++j) {
            const int d = diagonal(j);
            op[j] = real && row + d < k ? blk[packed_at(k, row, row + d)] : T(0);
            lo[j] = real && d > 0 && row < k && row >= d ? blk[packed_at(k, row - d, row)] : T(0);
        }
    } else {
        const T* blk = A.op + A.ofs[s];
        const int i = row < q ? node[base + row] : 0;
#pragma unroll
        for (int j = 0; j < COLS; ++j) {
            const int col = cg * COLS + j;
            T v = T(0);
            if (row < q && col < q) {
                const int jn = node[base + col];
                v = A.packed ? blk[packed_at(k, i, jn)] : blk[inv_offset<T>(k, i, jn)];
            }
            op[j] = v;
        }
    }
    // ports of this lane's node (ORDERED)
    int f0 = 0, f1 = 0;
    if (ORDERED && real && row < k) {
        f0 = A.pn_pfirst[k0 + row] - p0;
        f1 = A.pn_pfirst[k0 + row + 1] - p0;
    }
    T a = T(0), o = T(0), o_prev = T(0), h = T(0), c = T(0), be = T(0), ga = T(0), an = T(0);
    int tw = 0;
    const int p = p0 + row;
    // the workgroup's ports: a twin among them gets its wave through LDS
    const int pw = LOCAL ? A.port_off[unit * SUBS] : 0, pe = LOCAL ? A.port_off[min(unit * SUBS + SUBS, A.S)] : 0;
    bool near = false;
    if (owner) {
        tw = A.port_twin[p];
        near = LOCAL && tw >= pw && tw < pe;
        a = A.a[A.cur][p];
        o_prev = A.a[A.cur][tw];
        h = A.h[p];
        c = A.c[p];
        if (A.packed) {
            // beta and gamma from the rounded c, as the packed sweep forms them: the lines then
            // stay exactly passive in FP32 too
            be = T(2) * (A.w ? A.w[p] : A.W) * c;
            ga = T(1) - T(2) * c;
        } else {
            be = A.beta[p];
            ga = A.gamma[p];
        }
    }
    unsigned left = unsigned(A.ctl.first);
    unsigned tag = A.epoch;
    const unsigned abort_tag = A.epoch + 1;    // this launch's: no other launch on these words has it

    while (true) {
        // one sweep
        ++tag;
        const unsigned set = (tag & 1) ? unsigned(A.nports) : 0u;
        if (owner) ca[sub][row] = c * a;
        __syncthreads();
        if (bad) return;
        T z = T(0);
        if constexpr (ORDERED) {
#pragma clang fp contract(off)
            constexpr int MID = kSpan<QB> / 3;
            if (cg == 0 && real && row < k) {
                T t = T(0);
                for (int i = f0; i < f1; ++i) t += ca[sub][i];
                ts[sub][MID + row] = t;
            }
            __syncthreads();
            const T* tr = &ts[sub][MID + row];
            if constexpr (CG == 1) {
#pragma unroll
                for (int j = 0; j < COLS; ++j) {
                    z = __builtin_fmaf(op[j], tr[j], z);
                    const T up = lo[j] * tr[-j];
                    z += j > 0 ? up : T(0);
                }
                zp[0][tid] = z;
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    T zc = T(0);
#pragma unroll
                    for (int j = 8 * i; j < 8 * i + 8; ++j) {
                        const int d = diagonal(j);
                        zc = __builtin_fmaf(op[j], tr[d], zc);
                        const T up = lo[j] * tr[-d];
                        zc += d > 0 ? up : T(0);
                    }
                    zp[cg + 4 * i][row] = zc;
                }
            }
            __syncthreads();
            if (owner) {
                const int n = base + node[base + row];
                if constexpr (CG == 1) {
                    z = zp[0][n];
                } else {
                    z = T(0);
#pragma unroll
                    for (int v = 0; v < CHUNKS; ++v) z += zp[v][n];
                }
                o = packed_wave_out<T>(be, c, z, a, h);
            }
        } else {
        T z0 = T(0), z1 = T(0), z2 = T(0), z3 = T(0);
#pragma unroll
        for (int j = 0; j < COLS; j += 4) {
            const T* cc = &ca[sub][cg * COLS + j];
            z0 += op[j] * cc[0];
            z1 += op[j + 1] * cc[1];
            z2 += op[j + 2] * cc[2];
            z3 += op[j + 3] * cc[3];
            // bounds the staged values read ahead (their registers would displace op's)
            if (j % 8 == 4 && j + 4 < COLS) asm volatile("" : "+v"(z0), "+v"(z1), "+v"(z2), "+v"(z3) : : "memory");
        }
        z = (z0 + z1) + (z2 + z3);
        if constexpr (CG > 1) {
            zp[cg][rg * 64 + lane] = z;
            __syncthreads();
            if (cg == 0) {
                z = zp[0][row];
#pragma unroll
                for (int v = 1; v < CG; ++v) z += zp[v][row];
            }
        }
        if (owner) o = be * z + ga * a + h;
        }
        if (cg == 0) {
            if (owner) {
                if (near)
                    lex[tag & 1][LOCAL ? tw - pw : 0] = o;
                else
                    send(slots, set + unsigned(tw), o, tag);
            }
            // (the set is written again after the next sweep's barrier, which every reader of it reaches)
            if constexpr (LOCAL > 0) __syncthreads();
            if (!wait_for(owner && !near, [&] { return receive(slots, set + unsigned(p), tag, an); }, abort_word,
                          abort_tag, A.wait_ticks))
                bad = st->timeout = 1;
            if (near) an = lex[tag & 1][LOCAL ? p - pw : 0];
        }
        if (--left == 0) {
            if (!residual_check(A, nb, owner, p, base, row, o, a, an, o_prev, xs, vs, red, MANY ? SUBS / 2 : RG, first,
                                cnt, bad, next_s,
                                tag, abort_tag))
                return;
            left = next_s;
            if (left == 0) {
                if (owner) {
                    // the last sweep read buffer cur when the run had an odd number of sweeps
                    const int in = (A.cur + int((tag - A.epoch - 1) & 1)) & 1;
                    A.a[in][p] = a;
                    A.a[in ^ 1][p] = an;
                }
                return;
            }
        }
        o_prev = o;
        a = an;
    }
}

// Larger sub-circuits, FP64: up to 64 RG port nodes and 512 ports, a compute unit each.
// Rows are port nodes; wavefront w takes the column pairs w, w + 8, ..., whose entries
// of every row lane it keeps: the first REG of them in registers, the next LDS ones in
// LDS, and the last STREAM (RG = 5 only) are read every sweep, forwards and backwards in
// turn so that the XCD's L2, which stays warm inside a launch, holds most of them.  As a
// launch a sweep reads every operator from the memory-side cache.  Solves, a launch per
// sweep and resident: 210 sub-circuits of 296 port nodes (44x40x52) 10.8 -> 4.7 ms, 7.2 us
// a sweep for 18; 105 of them 7.2 -> 3.6; 216 of 218 (42x42x42 in blocks of 7) 9.9 -> 2.8;
// 64 of 196 (400x400 in blocks of 50) 1.95 -> 1.28.  RG = 5 spills 11 registers with
// eight pairs in registers, written once and read in the sweeps; with nine pairs 37.
template <int RG>
struct Wide {
    static constexpr int PAIRS = 4 * RG;  // 32 RG column pairs over eight wavefronts
    static constexpr int REG = RG >= 5 ? 8 : RG == 4 ? 12 : PAIRS;
    static constexpr int LDS = RG >= 5 ? 3 : PAIRS - REG;
    static constexpr int STREAM = PAIRS - REG - LDS;
};
constexpr int kWidePorts = 512, kWideRows = 5;

template <int RG>
__global__ void __launch_bounds__(512, 2) k_resident_wide(ResidentArgs<double> A) {
    const unsigned nb = gridDim.x - 1;
    if (blockIdx.x == nb) {
        control<double>(A, nb);
        return;
    }
    using Wd = Wide<RG>;
    constexpr int PAIRS = Wd::PAIRS, REG = Wd::REG, LP = Wd::LDS, ST = Wd::STREAM, ROWS = 64 * RG;
    constexpr int AHEAD = ST > 0 ? 2 : 1;
    __shared__ double2 keep[LP > 0 ? LP * RG * 512 : 1];
    __shared__ double part[8 * ROWS < 2 * kWidePorts ? 2 * kWidePorts : 8 * ROWS];
    __shared__ alignas(16) double tv[16 * PAIRS];
    __shared__ double ca[kWidePorts], red[8];
    __shared__ int32_t node[kWidePorts], first[kWidePorts], cnt[kWidePorts];
    __shared__ int bad;
    __shared__ unsigned next_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = xcd_block(blockIdx.x, nb);
    const int p0 = A.port_off[s], q = A.port_off[s + 1] - p0;
    const int k0 = A.pn_off[s], k = A.pn_off[s + 1] - k0;
    const int pairs = (k + 1) >> 1;
    const bool owner = tid < q;
    int p = p0 + tid;
    u64* const abort_word = A.sums + 2 * size_t(nb) + 1;
    const __amdgpu_buffer_rsrc_t slots =
        __builtin_amdgcn_make_buffer_rsrc(A.slots, 0, int(unsigned(A.nports) * 32u), 0x00020000);
    // the operator, range-checked: rows past the last one read what follows, or zeros
    const __amdgpu_buffer_rsrc_t ops =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(A.op) + A.ofs[s], 0, k * k * 8, 0x00020000);

    if (tid == 0) bad = 0, next_s = unsigned(A.ctl.first);
    for (int j = tid; j < 16 * PAIRS; j += 512) tv[j] = 0.0;
    // this thread's port node, and the ports of each node
    int f0 = 0, f1 = 0;
    if (tid < k) {
        f0 = A.pn_pfirst[k0 + tid] - p0;
        f1 = A.pn_pfirst[k0 + tid + 1] - p0;
        for (int i = f0; i < f1; ++i) {
            node[i] = tid;
            first[i] = f0;
            cnt[i] = f1 - f0;
        }
    }
    // entries of this lane's rows in column pair g (wave-uniform): zeros past the operator;
    // a last single column comes with what follows it, which meets a zero of tv
    auto entries = [&](int g, double2 (&v)[RG]) {
        const bool whole = 2 * g + 1 < k;
        const unsigned vo = 2 * g < k ? unsigned(lane * (whole ? 16 : 8)) + unsigned(g * k * 16) : 0x80000000u;
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
            v[rg] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(
                                                    ops, int(vo + unsigned(rg * (whole ? 1024 : 512))), 0, 0));
    };
    double2 op[REG][RG];
#pragma unroll
    for (int i = 0; i < REG; ++i) entries(wave + 8 * i, op[i]);
    if constexpr (LP > 0)
        for (int i = 0; i < LP; ++i) {
            double2 v[RG];
            entries(wave + 8 * (REG + i), v);
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) keep[(i * RG + rg) * 512 + tid] = v[rg];
        }
    // the streamed pairs of this wavefront, and those of them that are there
    const int count = ST > 0 ? max(0, min(ST, (pairs - wave - 8 * (REG + LP) + 7) >> 3)) : 0;
    double2 sv[AHEAD][RG];
    auto stream = [&](int e, bool back, double2 (&buf)[RG]) {
        if (e < count) entries(wave + 8 * (REG + LP + (back ? count - 1 - e : e)), buf);  // wave-uniform
    };
    // (the port's coefficients are read anew every sweep: their registers would displace op's)
    double a = 0.0, o = 0.0, o_prev = 0.0, an = 0.0;
    int tw = 0;
    if (owner) {
        tw = A.port_twin[p];
        a = A.a[A.cur][p];
        o_prev = A.a[A.cur][tw];
    }
    unsigned left = unsigned(A.ctl.first);
    unsigned tag = A.epoch;
    const unsigned abort_tag = A.epoch + 1;
    // whether the streamed pairs go backwards in a sweep: by its number in the solve, not by
    // its tag, whose parity earlier solves leave either way (the order shows in the sums' bits)
    auto backwards = [&](unsigned t) { return ((t ^ A.epoch ^ unsigned(A.ctl.sweeps)) & 1u) != 0; };
    if constexpr (ST > 0) {
#pragma unroll
        for (int e = 0; e < AHEAD; ++e) stream(e, backwards(tag + 1), sv[e]);
    }

    while (true) {
        ++tag;
        const unsigned set = (tag & 1) ? unsigned(A.nports) : 0u;
        asm volatile("" : "+v"(p));  // or the addresses of all its coefficients are kept, too
        if (owner) ca[tid] = A.c[p] * a;
        __syncthreads();
        if (bad) return;
        if (tid < k) {
            double t = 0.0;
            for (int i = f0; i < f1; ++i) t += ca[i];
            tv[tid] = t;
        }
        __syncthreads();
        double acc[RG];
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) acc[rg] = 0.0;
        auto pair = [&](int g) { return *reinterpret_cast<const double2*>(tv + 2 * g); };
#pragma unroll
        for (int i = 0; i < REG; ++i) {
            const double2 t = pair(wave + 8 * i);
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) acc[rg] = fma(op[i][rg].y, t.y, fma(op[i][rg].x, t.x, acc[rg]));
            // bounds the staged values read ahead (their registers would displace op's)
            if (i % 2 == 1) asm volatile("" : "+v"(acc[0]) : : "memory");
        }
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            const double2 t = pair(wave + 8 * (REG + i));
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) {
                const double2 v = keep[(i * RG + rg) * 512 + tid];
                acc[rg] = fma(v.y, t.y, fma(v.x, t.x, acc[rg]));
            }
            asm volatile("" : "+v"(acc[0]) : : "memory");
        }
        if constexpr (ST > 0) {
            const bool back = backwards(tag);
            for (int e0 = 0; e0 < count; e0 += AHEAD) {
#pragma unroll
                for (int e = 0; e < AHEAD; ++e) {
                    if (e0 + e >= count) continue;  // wave-uniform
                    const double2 t = pair(wave + 8 * (REG + LP + (back ? count - 1 - e0 - e : e0 + e)));
#pragma unroll
                    for (int rg = 0; rg < RG; ++rg) acc[rg] = fma(sv[e][rg].y, t.y, fma(sv[e][rg].x, t.x, acc[rg]));
                    stream(e0 + e + AHEAD, back, sv[e]);
                }
            }
        }
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) part[wave * ROWS + rg * 64 + lane] = acc[rg];
        double be = 0.0, rest = 0.0;
        if (owner) {
            be = A.beta[p];
            rest = A.gamma[p] * a + A.h[p];
        }
        __syncthreads();
        if (owner) {
            const int n = node[tid];
            double z = 0.0;
#pragma unroll
            for (int w = 0; w < 8; ++w) z += part[w * ROWS + n];
            o = be * z + rest;
            send(slots, set + unsigned(tw), o, tag);
        }
        // the next sweep's first streamed pairs are on their way while the waves are
        if constexpr (ST > 0) {
#pragma unroll
            for (int e = 0; e < AHEAD; ++e) stream(e, backwards(tag + 1), sv[e]);
        }
        if (!wait_for(owner, [&] { return receive(slots, set + unsigned(p), tag, an); }, abort_word, abort_tag,
                      A.wait_ticks))
            bad = A.state->timeout = 1;
        if (--left == 0) {
            __syncthreads();  // part's sums are read before the check takes its place
            if (!residual_check(A, nb, owner, p, 0, tid, o, a, an, o_prev, part, part + kWidePorts, red, 8, first, cnt,
                                bad, next_s, tag, abort_tag))
                return;
            left = next_s;
            if (left == 0) {
                if (owner) {
                    // the last sweep read buffer cur when the run had an odd number of sweeps
                    const int in = (A.cur + int((tag - A.epoch - 1) & 1)) & 1;
                    A.a[in][p] = a;
                    A.a[in ^ 1][p] = an;
                }
                return;
            }
        }
        o_prev = o;
        a = an;
    }
}

// The same in FP32, in the order of the port-node sweep of a launch per sweep (k_sweep_ppn,
// ports.hip), bit for bit: a row's entries come in groups of four columns, and each of the
// four has a running sum over the groups.  Wavefront w takes the sum w % 4 of every second
// row group from w / 4 on: REG groups in registers, the rest in LDS, the k % 4 last columns
// with the first sum.  Refined solves, a launch per sweep and resident: 168 sub-circuits of
// 296 port nodes (29x44x53) 7.7 -> 4.2 ms, 125 of 152 (30x30x30 in blocks of 6) 4.9 -> 2.1,
// 169 of 128 (400x400 in blocks of 33) 1.9 -> 1.0.
template <int RG>
struct WideF {
    static constexpr int GROUPS = 16 * RG, ROWS = (RG + 1) / 2;  // ROWS: row groups of a wavefront
    static constexpr int REG = RG >= 5 ? 54 : GROUPS, LDS = GROUPS - REG;
};

template <int RG>
__global__ void __launch_bounds__(512, 2) k_resident_wide_f(ResidentArgs<float> A) {
    const unsigned nb = gridDim.x - 1;
    if (blockIdx.x == nb) {
        control<float>(A, nb);
        return;
    }
    using Wd = WideF<RG>;
    constexpr int GROUPS = Wd::GROUPS, REG = Wd::REG, LG = Wd::LDS, NR = Wd::ROWS, ROWS = 64 * RG;
    __shared__ float keep[LG > 0 ? LG * RG * 256 : 1];
    __shared__ float part[4 * ROWS];
    __shared__ double xs[kWidePorts], red[8];
    __shared__ alignas(16) float tv[4 * GROUPS];
    __shared__ float av[kWidePorts];
    __shared__ int32_t node[kWidePorts], first[kWidePorts], cnt[kWidePorts];
    __shared__ int bad;
    __shared__ unsigned next_s;
    __shared__ double vs[kWidePorts];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cls = wave & 3, half = wave >> 2;
    const int s = xcd_block(blockIdx.x, nb);
    const int p0 = A.port_off[s], q = A.port_off[s + 1] - p0;
    const int k0 = A.pn_off[s], k = A.pn_off[s + 1] - k0;
    const int ng = k >> 2, full = 4 * ng;
    const bool owner = tid < q;
    int p = p0 + tid;
    u64* const abort_word = A.sums + 2 * size_t(nb) + 1;
    const __amdgpu_buffer_rsrc_t slots =
        __builtin_amdgcn_make_buffer_rsrc(A.slots, 0, int(unsigned(A.nports) * 16u), 0x00020000);
    const __amdgpu_buffer_rsrc_t ops =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A.op) + A.ofs[s], 0, k * k * 4, 0x00020000);

    if (tid == 0) bad = 0, next_s = unsigned(A.ctl.first);
    for (int j = tid; j < 4 * GROUPS; j += 512) tv[j] = 0.0f;
    int f0 = 0, f1 = 0;
    if (tid < k) {
        f0 = A.pn_pfirst[k0 + tid] - p0;
        f1 = A.pn_pfirst[k0 + tid + 1] - p0;
        for (int i = f0; i < f1; ++i) {
            node[i] = tid;
            first[i] = f0;
            cnt[i] = f1 - f0;
        }
    }
    auto load = [&](unsigned at) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ops, int(at), 0, 0));
    };
    // this wavefront's entry of group g in row group rg: zeros past the groups
    auto entry = [&](int g, int rg) {
        return load(g < ng ? unsigned((g * k + rg * 64 + lane) * 4 + cls) * 4u : 0x80000000u);
    };
    float op[REG][NR], last[3][NR];
#pragma unroll
    for (int i = 0; i < REG; ++i)
#pragma unroll
        for (int r = 0; r < NR; ++r) op[i][r] = entry(i, half + 2 * r);
    if constexpr (LG > 0)
        for (int i = 0; i < LG; ++i)
            for (int r = 0; r < NR; ++r)
                if (half + 2 * r < RG) keep[((i * RG + half + 2 * r) * 4 + cls) * 64 + lane] = entry(REG + i, half + 2 * r);
#pragma unroll
    for (int e = 0; e < 3; ++e)
#pragma unroll
        for (int r = 0; r < NR; ++r)
            last[e][r] = load(full + e < k ? unsigned((full + e) * k + (half + 2 * r) * 64 + lane) * 4u : 0x80000000u);
    // (the port's coefficients are read anew every sweep: their registers would displace op's)
    float a = 0.0f, o = 0.0f, o_prev = 0.0f, an = 0.0f;
    int tw = 0;
    if (owner) {
        tw = A.port_twin[p];
        a = A.a[A.cur][p];
        o_prev = A.a[A.cur][tw];
    }
    unsigned left = unsigned(A.ctl.first);
    unsigned tag = A.epoch;
    const unsigned abort_tag = A.epoch + 1;

    while (true) {
        ++tag;
        const unsigned set = (tag & 1) ? unsigned(A.nports) : 0u;
        asm volatile("" : "+v"(p));  // or the addresses of all its coefficients are kept, too
        if (owner) av[tid] = a;
        __syncthreads();
        if (bad) return;
        if (tid < k) {
            float t = 0.0f;
            for (int i = f0; i < f1; ++i) t = __builtin_fmaf(A.c[p0 + i], av[i], t);
            tv[tid] = t;
        }
        __syncthreads();
        float acc[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int i = 0; i < REG; ++i) {
            const float t = tv[4 * i + cls];
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = __builtin_fmaf(op[i][r], t, acc[r]);
            // bounds the staged values read ahead (their registers would displace op's)
            if (i % 8 == 7) asm volatile("" : "+v"(acc[0]) : : "memory");
        }
        if constexpr (LG > 0) {
#pragma unroll 4
            for (int i = 0; i < LG; ++i) {
                const float t = tv[4 * (REG + i) + cls];
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (half + 2 * r < RG)
                        acc[r] = __builtin_fmaf(keep[((i * RG + half + 2 * r) * 4 + cls) * 64 + lane], t, acc[r]);
            }
        }
        if (cls == 0) {  // wave-uniform
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (full + e < k) {
                    const float t = tv[full + e];
#pragma unroll
                    for (int r = 0; r < NR; ++r) acc[r] = __builtin_fmaf(last[e][r], t, acc[r]);
                }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r)
            if (half + 2 * r < RG) part[cls * ROWS + (half + 2 * r) * 64 + lane] = acc[r];
        float be = 0.0f, ga = 0.0f, h = 0.0f;
        if (owner) {
            be = A.beta[p];
            ga = A.gamma[p];
            h = A.h[p];
        }
        __syncthreads();
        if (owner) {
            const int n = node[tid];
            float z = part[n];
#pragma unroll
            for (int j = 1; j < 4; ++j) z += part[j * ROWS + n];
            o = dense_wave_out<float>(be, z, ga, a, h);
            send(slots, set + unsigned(tw), o, tag);
        }
        if (!wait_for(owner, [&] { return receive(slots, set + unsigned(p), tag, an); }, abort_word, abort_tag,
                      A.wait_ticks))
            bad = A.state->timeout = 1;
        if (--left == 0) {
            if (!residual_check(A, nb, owner, p, 0, tid, o, a, an, o_prev, xs, vs, red, 8, first, cnt, bad, next_s, tag,
                                abort_tag))
                return;
            left = next_s;
            if (left == 0) {
                if (owner) {
                    // the last sweep read buffer cur when the run had an odd number of sweeps
                    const int in = (A.cur + int((tag - A.epoch - 1) & 1)) & 1;
                    A.a[in][p] = a;
                    A.a[in ^ 1][p] = an;
                }
                return;
            }
        }
        o_prev = o;
        a = an;
    }
}

// workgroups of `kernel` (threads each) that the current device holds at once, at most
// `blocks` and the controlling one: blocks or 0
int fitting(const void* kernel, int threads, int64_t blocks) {
    int dev = 0, cus = 0, coop = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return blocks < int64_t(per) * cus ? int(blocks) : 0;
}

template <typename T>
const void* wide_kernel(int max_npn) {
    if constexpr (sizeof(T) == 4) {
        switch ((max_npn + 63) / 64) {
            case 0:
            case 1:
            case 2: return reinterpret_cast<const void*>(&k_resident_wide_f<2>);
            case 3: return reinterpret_cast<const void*>(&k_resident_wide_f<3>);
            case 4: return reinterpret_cast<const void*>(&k_resident_wide_f<4>);
            default: return reinterpret_cast<const void*>(&k_resident_wide_f<5>);
        }
    }
    switch ((max_npn + 63) / 64) {
        case 0:
        case 1:
        case 2: return reinterpret_cast<const void*>(&k_resident_wide<2>);
        case 3: return reinterpret_cast<const void*>(&k_resident_wide<3>);
        case 4: return reinterpret_cast<const void*>(&k_resident_wide<4>);
        default: return reinterpret_cast<const void*>(&k_resident_wide<5>);
    }
}

template <typename T, int QB, int SUBS = 1>
int blocks_of(int S) {
    return fitting(reinterpret_cast<const void*>(&k_resident<T, QB, SUBS>), kThreads<QB, SUBS>,
                   (int64_t(S) + SUBS - 1) / SUBS);
}

template <typename T, int QB, int SUBS = 1>
hipError_t launch_q(const ResidentArgs<T>& args, hipStream_t st) {
    ResidentArgs<T> a = args;
    void* params[] = {&a};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&k_resident<T, QB, SUBS>),
                                      dim3((unsigned(args.S) + SUBS - 1) / SUBS + 1), dim3(kThreads<QB, SUBS>), params,
                                      0, st);
}

// Up to 32 ports: sub-circuits of a workgroup.  Sixteen send nearly half of their waves
// through LDS (neighbours in the block order), which relieves the exchange of many; few
// are better off without the workgroup's barriers, each of their wavefronts on a compute
// unit of its own (solves with 2 / 8 / 16: 7,680 sub-circuits 4.53 / 2.69 / 2.51 ms, 1,444
// 0.99 / 0.91 / 0.95, 1,156 1.15 / 1.13 / 1.18, 437 in FP32 1.04 / 1.16 / 1.25, 64
// 0.73 / 0.76 / 0.79).
constexpr int kManySubs = 1280;

}  // namespace

// Whether sub-circuits take a compute unit each: dense operators beyond the shapes above
template <typename T>
bool wide(int max_npn, int max_ports, bool packed) {
    return !packed && (sizeof(T) == 4 || max_ports > 128) && max_ports <= kWidePorts && max_npn <= 64 * kWideRows;
}

template <typename T>
int resident_blocks(int S, int max_npn, int max_ports, bool packed) {
    if (S < 1) return 0;
    if (wide<T>(max_npn, max_ports, packed)) return fitting(wide_kernel<T>(max_npn), 512, S);
    if constexpr (sizeof(T) == 4) {
        if (!packed || max_ports > 64) return 0;
        return max_ports > 32 ? blocks_of<T, 64>(S) : S > kManySubs ? blocks_of<T, 32, 16>(S) : blocks_of<T, 32, 2>(S);
    } else {
        if (max_ports > 128) return 0;
        return max_ports <= 32   ? (S > kManySubs ? blocks_of<T, 32, 16>(S) : blocks_of<T, 32, 2>(S))
               : max_ports <= 64 ? blocks_of<T, 64>(S)
               : max_ports <= 96 ? blocks_of<T, 96>(S)
                                 : blocks_of<T, 128>(S);
    }
}

template <typename T>
hipError_t launch_resident(const ResidentArgs<T>& args, int max_npn, int max_ports, hipStream_t st) {
    if (args.S < 1) return hipErrorInvalidValue;
    if (wide<T>(max_npn, max_ports, args.packed)) {
        ResidentArgs<T> a = args;
        void* params[] = {&a};
        return hipLaunchCooperativeKernel(wide_kernel<T>(max_npn), dim3(unsigned(args.S) + 1), dim3(512), params, 0,
                                          st);
    }
    if constexpr (sizeof(T) == 4) {
        if (!args.packed || max_ports > 64) return hipErrorInvalidValue;
        return max_ports > 32         ? launch_q<T, 64>(args, st)
               : args.S > kManySubs ? launch_q<T, 32, 16>(args, st)
                                    : launch_q<T, 32, 2>(args, st);
    } else {
        if (max_ports > 128) return hipErrorInvalidValue;
        return max_ports <= 32   ? (args.S > kManySubs ? launch_q<T, 32, 16>(args, st) : launch_q<T, 32, 2>(args, st))
               : max_ports <= 64 ? launch_q<T, 64>(args, st)
               : max_ports <= 96 ? launch_q<T, 96>(args, st)
                                 : launch_q<T, 128>(args, st);
    }
}

template int resident_blocks<double>(int, int, int, bool);
template int resident_blocks<float>(int, int, int, bool);
template hipError_t launch_resident<double>(const ResidentArgs<double>&, int, int, hipStream_t);
template hipError_t launch_resident<float>(const ResidentArgs<float>&, int, int, hipStream_t);

}  // namespace vtm
