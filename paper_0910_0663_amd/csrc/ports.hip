// Port-to-port form of the sweep (the interface-only iteration of the
// Appendix, eqs. 23-26, written for the eliminated twins).
//
// With the incident waves a_s at the q ports of sub-circuit s and
// x = K^-1 (b + sum_p c_p a_p e_i(p)), the outgoing waves are
//     o_p = beta_p x_i(p) + gamma_p a_p = h_p + sum_p' M_pp' a_p'
// with M = diag(beta) K^-1[i(P), i(P)] diag(c) + diag(gamma) and
// h = beta (K^-1 b)[i(P)].  A sweep then streams the q x q operator M instead
// of the n x n inverse; x itself is rebuilt by a full sweep where needed.
#include "kernels.hpp"
#include "layout.hpp"

#include <algorithm>

#include <type_traits>

namespace vtm {

namespace {

constexpr int kBlock = 256;

// M_s in the column-group layout (n = q), from the stored inverse K_s
template <typename TO>
__global__ void __launch_bounds__(kBlock)
    k_port_matrix(const int32_t* __restrict__ sub_off, const int64_t* __restrict__ kofs,
                  const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_node,
                  const double* __restrict__ pc, const double* __restrict__ pbeta, const double* __restrict__ pgamma,
                  const TO* __restrict__ K, const int64_t* __restrict__ pofs, TO* __restrict__ M, Coupling<double> B) {
    const int s = blockIdx.x;
    const int ns = sub_off[s + 1] - sub_off[s];
    const int p0 = port_off[s], q = port_off[s + 1] - p0;
    const TO* Ks = K + kofs[s];
    TO* Ms = M + pofs[s];
    const int64_t cnt = int64_t(q) * q;
    for (int64_t d = int64_t(blockIdx.y) * blockDim.x + threadIdx.x; d < cnt; d += int64_t(blockDim.x) * gridDim.y) {
        int r, c;
        inv_rc<TO>(q, d, r, c);
        const int pr = p0 + r, pcol = p0 + c;
        const int j = port_node[pcol];
        double v;
        if (B.row) {  // (B K^-1[i(P), i(P)])_{r c}: B's row r over the ports of this sub-circuit
            v = 0.0;
            for (int k = B.row[pr]; k < B.row[pr + 1]; ++k)
                v += B.val[k] * double(Ks[inv_offset<TO>(ns, port_node[B.col[k]], j)]);
            v *= pc[pcol];
        } else {
            v = pbeta[pr] * double(Ks[inv_offset<TO>(ns, port_node[pr], j)]) * pc[pcol];
        }
        if (r == c) v += pgamma[pr];
        Ms[d] = TO(v);
    }
}

// h_p = beta_p x_i(p) for x = K^-1 b, per right-hand side (x and h are
// [rows][nrhs], right-hand side fastest)
template <typename TV>
__global__ void __launch_bounds__(kBlock)
    k_port_h(int nrhs, const int32_t* __restrict__ sub_off, const int32_t* __restrict__ port_off,
             const int32_t* __restrict__ port_node, const TV* __restrict__ pbeta, const TV* __restrict__ x,
             TV* __restrict__ h, Coupling<TV> B) {
    const int s = blockIdx.x;
    const int off = sub_off[s], p0 = port_off[s];
    const int cnt = (port_off[s + 1] - p0) * nrhs;
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
        const int p = p0 + t / nrhs, r = t % nrhs;
        TV v;
        if (B.row) {
            v = TV(0);
            for (int k = B.row[p]; k < B.row[p + 1]; ++k)
                v += B.val[k] * x[int64_t(off + port_node[B.col[k]]) * nrhs + r];
        } else {
            v = pbeta[p] * x[int64_t(off + port_node[p]) * nrhs + r];
        }
        h[int64_t(p) * nrhs + r] = v;
    }
}

// coupled lines: the outgoing waves from the x of a full sweep
template <typename TV>
__global__ void __launch_bounds__(kBlock)
    k_wave_coupled(int n_ports, int nrhs, Coupling<TV> B, const int32_t* __restrict__ port_row,
                   const TV* __restrict__ pgamma, const int32_t* __restrict__ port_twin, const TV* __restrict__ x,
                   const TV* __restrict__ a_cur, TV* __restrict__ a_next) {
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n_ports) * nrhs) return;
    const int p = int(t / nrhs), r = int(t - int64_t(p) * nrhs);
    TV v = pgamma[p] * a_cur[t];
    for (int k = B.row[p]; k < B.row[p + 1]; ++k) v += B.val[k] * x[int64_t(port_row[B.col[k]]) * nrhs + r];
    a_next[int64_t(port_twin[p]) * nrhs + r] = v;
}

typedef double pp_d2 __attribute__((ext_vector_type(2)));
typedef unsigned long long u64p;
typedef float pp_f4 __attribute__((ext_vector_type(4)));

// 16 bytes of operator entries (NT: non-temporal).  Plain loads go through HIP's vector
// types: through the compiler's own the same loops held 58 to 60 registers for 46 to 48
// and swept up to 2.4% slower (150 sub-circuits of 296 port nodes in FP32: 10.9 -> 11.15 us).
template <typename T, bool NT = false>
__device__ inline void load16p(const T* p, T (&v)[Group<T>::G]) {
    if constexpr (sizeof(T) == 8) {
        if constexpr (NT) {
            const pp_d2 w = __builtin_nontemporal_load(reinterpret_cast<const pp_d2*>(p));
            v[0] = w.x, v[1] = w.y;
        } else {
            const double2 w = *reinterpret_cast<const double2*>(p);
            v[0] = w.x, v[1] = w.y;
        }
    } else if constexpr (NT) {
        const pp_f4 w = __builtin_nontemporal_load(reinterpret_cast<const pp_f4*>(p));
        v[0] = w.x, v[1] = w.y, v[2] = w.z, v[3] = w.w;
    } else {
        const float4 w = *reinterpret_cast<const float4*>(p);
        v[0] = w.x;
        v[1] = w.y;
        v[2] = w.z;
        v[3] = w.w;
    }
}

// One port-to-port sweep, one workgroup per sub-circuit and block of up to R
// right-hand sides (a_next[twin(p)] = h_p + (M a)_p).  SPLIT = 2 (q <= 32, one
// wavefront, R = 1): lane l takes row l % 32 and half the column groups, and the
// halves are added with a cross-lane shuffle.  SPLIT = 1: one row per thread.
template <typename TO, typename TV, int SPLIT, int R>
__global__ void __launch_bounds__(256)
    k_sweep_pp(int ny, int nrhs, const TO* __restrict__ M, const int64_t* __restrict__ pofs,
               const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
               const TV* __restrict__ h, const TV* __restrict__ a_cur, TV* __restrict__ a_next) {
    constexpr int G = Group<TO>::G;
    extern __shared__ char smem[];
    TV* av = reinterpret_cast<TV*>(smem);  // [q][R]
    const int u = xcd_block(blockIdx.x, gridDim.x);
    const int s = R == 1 ? u : u / ny, r0 = R == 1 ? 0 : (u - s * ny) * R;
    const int w = R == 1 ? 1 : min(R, nrhs - r0);
    const int p0 = port_off[s], q = port_off[s + 1] - p0;
    const int lane = threadIdx.x;
    const TO* Ms = M + pofs[s];
    const int ng = q / G, full = ng * G;
    const int bs = blockDim.x;
    for (int t = lane; t < q * R; t += bs)
        av[t] = t % R < w ? a_cur[int64_t(p0 + t / R) * nrhs + r0 + t % R] : TV(0);
    __syncthreads();
    if constexpr (SPLIT == 2) {
        const int row = lane & 31, half = lane >> 5;
        const int g_lo = half ? (ng + 1) / 2 : 0, g_hi = half ? ng : (ng + 1) / 2;
        TV acc[G];
#pragma unroll
        for (int j = 0; j < G; ++j) acc[j] = TV(0);
        if (row < q) {
#pragma unroll 4
            for (int g = g_lo; g < g_hi; ++g) {
                TO v[G];
                load16p<TO>(Ms + (int64_t(g) * q + row) * G, v);
#pragma unroll
                for (int j = 0; j < G; ++j) acc[j] += TV(v[j]) * av[g * G + j];
            }
            if (half == 0)
                for (int c = full; c < q; ++c) acc[0] += TV(Ms[int64_t(full) * q + int64_t(c - full) * q + row]) * av[c];
        }
        TV v = acc[0];
#pragma unroll
        for (int j = 1; j < G; ++j) v += acc[j];
        v += __shfl_down(v, 32, 64);
        if (half == 0 && row < q) a_next[port_twin[p0 + row]] = h[p0 + row] + v;
    } else {
        for (int row = lane; row < q; row += bs) {
            TV acc[R][G];
#pragma unroll
            for (int k = 0; k < R; ++k)
#pragma unroll
                for (int j = 0; j < G; ++j) acc[k][j] = TV(0);
#pragma unroll 4
            for (int g = 0; g < ng; ++g) {
                TO v[G];
                load16p<TO>(Ms + (int64_t(g) * q + row) * G, v);
#pragma unroll
                for (int j = 0; j < G; ++j)
#pragma unroll
                    for (int k = 0; k < R; ++k) acc[k][j] += TV(v[j]) * av[(g * G + j) * R + k];
            }
            for (int c = full; c < q; ++c) {
                const TV v = TV(Ms[int64_t(full) * q + int64_t(c - full) * q + row]);
#pragma unroll
                for (int k = 0; k < R; ++k) acc[k][0] += v * av[c * R + k];
            }
            const int64_t tw = int64_t(port_twin[p0 + row]) * nrhs + r0, po = int64_t(p0 + row) * nrhs + r0;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                TV v = acc[k][0];
#pragma unroll
                for (int j = 1; j < G; ++j) v += acc[k][j];
                if (k < w) a_next[tw + k] = h[po + k] + v;
            }
        }
    }
}

// The same with few sub-circuits of many ports (tears at interfacial nodes): a
// workgroup of KS wavefronts takes 64 rows of one sub-circuit, each wavefront
// every KS-th chunk of its column groups, and the partial sums meet in LDS in
// wavefront order.  Bound by latency: with one wavefront per 64 rows each lane had a
// chain of q / G rounds of loads and the chip was idle (six sub-circuits of up to
// 200 ports, 1.4 MB of operators: 7.5 us a sweep, now 5.0, of which ~2.4 are the
// launch).
template <typename TO, typename TV, int R, int KS>
__global__ void __launch_bounds__(64 * KS)
    k_sweep_pp_split(int ny, int nrhs, const TO* __restrict__ M, const int64_t* __restrict__ pofs,
                     const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
                     const TV* __restrict__ h, const TV* __restrict__ a_cur, TV* __restrict__ a_next, int max_q) {
    constexpr int G = Group<TO>::G, CH = 4;  // column groups per chunk, loaded together
    extern __shared__ char smem[];
    TV* av = reinterpret_cast<TV*>(smem);  // [max_q][R]
    TV* part = av + max_q * R;             // [KS][64][R]
    const int s = R == 1 ? int(blockIdx.x) : int(blockIdx.x) / ny;
    const int r0 = R == 1 ? 0 : (int(blockIdx.x) - s * ny) * R;
    const int w = R == 1 ? 1 : min(R, nrhs - r0);
    const int p0 = port_off[s], q = port_off[s + 1] - p0;
    const int row0 = int(blockIdx.y) * 64;
    if (row0 >= q) return;  // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = row0 + lane, rowc = min(row, q - 1);
    const TO* Ms = M + pofs[s];
    const int ng = q / G, full = ng * G;
    // this wavefront's first chunk is in flight while the waves are staged
    TO v[CH][G];
    auto load = [&](int g0) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (g0 + i < ng) {  // wave-uniform
                load16p<TO>(Ms + (int64_t(g0 + i) * q + rowc) * G, v[i]);
            } else {
#pragma unroll
                for (int j = 0; j < G; ++j) v[i][j] = TO(0);
            }
        }
    };
    load(wave * CH);
    for (int t = tid; t < q * R; t += 64 * KS)
        av[t] = t % R < w ? a_cur[int64_t(p0 + t / R) * nrhs + r0 + t % R] : TV(0);
    __syncthreads();
    TV acc[R];
#pragma unroll
    for (int k = 0; k < R; ++k) acc[k] = TV(0);
    for (int g0 = wave * CH; g0 < ng; g0 += KS * CH) {
        TO u[CH][G];
#pragma unroll
        for (int i = 0; i < CH; ++i)
#pragma unroll
            for (int j = 0; j < G; ++j) u[i][j] = v[i][j];
        load(g0 + KS * CH);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int g = min(g0 + i, ng - 1);  // past the end: zeros times a staged wave
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int k = 0; k < R; ++k)
                    acc[k] += g0 + i < ng ? TV(u[i][j]) * av[(g * G + j) * R + k] : TV(0);
        }
    }
    if (wave == KS - 1)
        for (int c = full; c < q; ++c) {
            const TV m = TV(Ms[int64_t(full) * q + int64_t(c - full) * q + rowc]);
#pragma unroll
            for (int k = 0; k < R; ++k) acc[k] += m * av[c * R + k];
        }
#pragma unroll
    for (int k = 0; k < R; ++k) part[(wave * 64 + lane) * R + k] = acc[k];
    __syncthreads();
    for (int t = tid; t < 64 * R; t += 64 * KS) {
        const int i = t / R, k = t % R;
        if (row0 + i >= q || k >= w) continue;
        TV z = TV(0);
#pragma unroll
        for (int v2 = 0; v2 < KS; ++v2) z += part[v2 * 64 * R + t];
        const int p = p0 + row0 + i;
        a_next[int64_t(port_twin[p]) * nrhs + r0 + k] = h[int64_t(p) * nrhs + r0 + k] + z;
    }
}

// Port-node form for any A (the packed kernel below needs A symmetric): with
// z = K^-1[N, N] t over the k port nodes N of a sub-circuit and
// t_n = sum_{p at n} c_p a_p, the outgoing wave of port p is
// o_p = beta_p z_n(p) + gamma_p a_p + h_p.  K^-1[N, N] (k x k, fewer than the
// q x q entries of M when nodes carry several ports) is stored in the column-
// group layout (n = k) at Sn + nofs[s].
template <typename TO>
__global__ void __launch_bounds__(kBlock)
    k_port_node_dense(const int32_t* __restrict__ sub_off, const int64_t* __restrict__ kofs,
                      const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_node,
                      const TO* __restrict__ K, const int64_t* __restrict__ nofs, TO* __restrict__ Sn,
                      int transpose) {
    const int s = blockIdx.x;
    const int ns = sub_off[s + 1] - sub_off[s];
    const int k0 = pn_off[s], k = pn_off[s + 1] - k0;
    const TO* Ks = K + kofs[s];
    TO* out = Sn + nofs[s];
    for (int t = threadIdx.x; t < k * k; t += blockDim.x) {
        const int r = t / k, c = t - r * k;
        const int i = pn_node[k0 + (transpose ? c : r)], j = pn_node[k0 + (transpose ? r : c)];
        out[inv_offset<TO>(k, r, c)] = Ks[inv_offset<TO>(ns, i, j)];
    }
}

// One workgroup per sub-circuit, one port node (row of K^-1[N, N]) per thread.  NT: of
// every 16 sub-circuits the first `keep` read their operators as usual and the others
// non-temporally (launch_sweep_ppn).  Bound by HBM: 4,096 sub-circuits of 296 port nodes
// in FP32 (1.44 GB) 255 us a sweep, 5.6 TB/s, with every operator read as usual in one
// order; 247 with every other sweep backwards; 220, 6.5 TB/s, with 3 of 16 kept.
// Non-temporal loads take no room in the 256 MB memory-side cache, so a kept share
// that fits it is found there by every sweep; read as usual, a stream several times
// its size leaves nothing of itself behind.
template <typename TO, typename TV, bool NT>
__global__ void __launch_bounds__(512)
    k_sweep_ppn(const TO* __restrict__ Sn, const int64_t* __restrict__ nofs, const int32_t* __restrict__ pn_off,
                const int32_t* __restrict__ pn_pfirst, const int32_t* __restrict__ port_off,
                const int32_t* __restrict__ port_twin, const TV* __restrict__ pc, const TV* __restrict__ pbeta,
                const TV* __restrict__ pgamma, const TV* __restrict__ h, const TV* __restrict__ a_cur,
                TV* __restrict__ a_next, int max_npn, int reverse, int keep) {
    constexpr int G = Group<TO>::G;
    extern __shared__ char smem[];
    TV* tv = reinterpret_cast<TV*>(smem);
    TV* zv = tv + max_npn;
    int32_t* pnode = reinterpret_cast<int32_t*>(zv + max_npn);
    const int s = reverse ? xcd_block_reversed(blockIdx.x, gridDim.x) : xcd_block(blockIdx.x, gridDim.x);
    const int k0 = pn_off[s], k = pn_off[s + 1] - k0;
    const int p0 = port_off[s], p1 = port_off[s + 1];
    const int tid = threadIdx.x, bs = blockDim.x;
    const TO* Ss = Sn + nofs[s];
    // t per port node, in port order
    for (int j = tid; j < k; j += bs) {
        const int f0 = pn_pfirst[k0 + j], f1 = pn_pfirst[k0 + j + 1];
        TV acc = TV(0);
        for (int p = f0; p < f1; ++p) {
            acc = fused(pc[p], a_cur[p], acc);
            pnode[p - p0] = j;
        }
        tv[j] = acc;
    }
    __syncthreads();
    // z = K^-1[N, N] t
    const int ng = k / G, full = ng * G;
    auto product = [&](auto nt) {
        for (int row = tid; row < k; row += bs) {
            TV acc[G];
#pragma unroll
            for (int j = 0; j < G; ++j) acc[j] = TV(0);
#pragma unroll 4
            for (int g = 0; g < ng; ++g) {
                TO v[G];
                load16p<TO, decltype(nt)::value>(Ss + (int64_t(g) * k + row) * G, v);
#pragma unroll
                for (int j = 0; j < G; ++j) acc[j] = fused(TV(v[j]), tv[g * G + j], acc[j]);
            }
            for (int c = full; c < k; ++c)
                acc[0] = fused(TV(Ss[int64_t(full) * k + int64_t(c - full) * k + row]), tv[c], acc[0]);
            TV v = acc[0];
#pragma unroll
            for (int j = 1; j < G; ++j) v += acc[j];
            zv[row] = v;
        }
    };
    if constexpr (NT) {
        if ((s & 15) < keep)
            product(std::false_type{});
        else
            product(std::true_type{});
    } else {
        product(std::false_type{});
    }
    __syncthreads();
    for (int p = p0 + tid; p < p1; p += bs)
        a_next[port_twin[p]] = dense_wave_out<TV>(pbeta[p], zv[pnode[p - p0]], pgamma[p], a_cur[p], h[p]);
}

// The same in FP64, 64 rows per workgroup: their columns spread over KS wavefronts, whose
// partial sums meet in LDS.  Every row block of a sub-circuit forms all of t again.  One
// workgroup per sub-circuit leaves a chip of 256 compute units with five wavefronts on
// each of 210 of them (44 x 40 x 52 nodes in blocks of 8, 296 port nodes: 19.2 us a
// sweep; here 18.1, 7.3 TB/s of 132 MB in the memory-side cache), or four loads in flight
// a wavefront to a workgroup that waits for its slowest (96 x 90 x 92, 1 GB: a solve 107.7
// -> 94.0 ms).  Six column pairs in flight keep the kernel under 64 registers, so four
// workgroups share a compute unit; four and eight: 11.0 and 11.1 ms where six make 10.8.
constexpr int kPpnSplit = 8, kPpnPairs = 6;  // wavefronts, column pairs in flight in each
template <int KS, int CH, bool NT>
__global__ void __launch_bounds__(64 * KS)
    k_sweep_ppn_split(int ry, const double* __restrict__ Sn, const int64_t* __restrict__ nofs,
                      const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_pfirst,
                      const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
                      const double* __restrict__ pc, const double* __restrict__ pbeta,
                      const double* __restrict__ pgamma, const double* __restrict__ h,
                      const double* __restrict__ a_cur, double* __restrict__ a_next, int max_npn, int reverse,
                      int keep) {
    extern __shared__ char smem[];
    double* tv = reinterpret_cast<double*>(smem);
    double* part = tv + max_npn;
    int32_t* pnode = reinterpret_cast<int32_t*>(part + 64 * KS);
    const int unit = reverse ? xcd_block_reversed(blockIdx.x, gridDim.x) : xcd_block(blockIdx.x, gridDim.x);
    const int s = unit / ry, row0 = (unit - s * ry) * 64;
    const int k0 = pn_off[s], k = pn_off[s + 1] - k0;
    if (row0 >= k) return;
    const int p0 = port_off[s];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = row0 + lane, rowc = min(row, k - 1);
    const double* Ss = Sn + nofs[s];
    const int ng = k / 2;  // whole column pairs; this wavefront takes wave, wave + KS, ...
    double v[CH][2];
    auto product = [&](auto nt) {
        auto load = [&](int g, double (&u)[2]) {
            if (g < ng) load16p<double, decltype(nt)::value>(Ss + (int64_t(g) * k + rowc) * 2, u);
        };
#pragma unroll
        for (int i = 0; i < CH; ++i) load(wave + KS * i, v[i]);
        // this block's ports, one per thread
        const int b0 = pn_pfirst[k0 + row0], b1 = pn_pfirst[k0 + min(row0 + 64, k)];
        const int pb = b0 + tid;
        double beta = 0.0, rest = 0.0;
        int twin = 0;
        if (pb < b1) {
            beta = pbeta[pb];
            rest = pgamma[pb] * a_cur[pb] + h[pb];
            twin = port_twin[pb];
        }
        // t per port node, in port order
        for (int j = tid; j < k; j += 64 * KS) {
            const int f0 = pn_pfirst[k0 + j], f1 = pn_pfirst[k0 + j + 1];
            double acc = 0.0;
            for (int p = f0; p < f1; ++p) {
                acc += pc[p] * a_cur[p];
                pnode[p - p0] = j - row0;
            }
            tv[j] = acc;
        }
        __syncthreads();
        double acc0 = 0.0, acc1 = 0.0;
        for (int g0 = wave; g0 < ng; g0 += KS * CH) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int g = g0 + KS * i;
                if (g < ng) {
                    acc0 += v[i][0] * tv[2 * g];
                    acc1 += v[i][1] * tv[2 * g + 1];
                }
                load(g + KS * CH, v[i]);
            }
        }
        if ((k & 1) && wave == KS - 1) acc0 += Ss[int64_t(2 * ng) * k + rowc] * tv[k - 1];
        part[wave * 64 + lane] = acc0 + acc1;
        __syncthreads();
        auto z = [&](int p) {
            const int r = pnode[p - p0];
            double v2 = 0.0;
#pragma unroll
            for (int w = 0; w < KS; ++w) v2 += part[w * 64 + r];
            return v2;
        };
        if (pb < b1) a_next[twin] = beta * z(pb) + rest;
        for (int p = pb + 64 * KS; p < b1; p += 64 * KS)
            a_next[port_twin[p]] = pbeta[p] * z(p) + (pgamma[p] * a_cur[p] + h[p]);
    };
    if constexpr (NT) {
        if ((s & 15) < keep)
            product(std::false_type{});
        else
            product(std::true_type{});
    } else {
        product(std::false_type{});
    }
}

}  // namespace

template <typename TO>
hipError_t launch_port_node_dense(int S, const int32_t* sub_off, const int64_t* kofs, const int32_t* pn_off,
                                  const int32_t* pn_node, const TO* K, const int64_t* nofs, TO* Sn, bool transpose,
                                  hipStream_t st) {
    hipLaunchKernelGGL(k_port_node_dense<TO>, dim3(S), dim3(kBlock), 0, st, sub_off, kofs, pn_off, pn_node, K, nofs,
                       Sn, transpose ? 1 : 0);
    return hipGetLastError();
}

template <typename TO, typename TV>
hipError_t launch_sweep_ppn(int S, int max_npn, int max_ports, int64_t op_bytes, const TO* Sn, const int64_t* nofs,
                            const int32_t* pn_off, const int32_t* pn_pfirst, const int32_t* port_off,
                            const int32_t* port_twin, const TV* pc, const TV* pbeta, const TV* pgamma, const TV* h,
                            const TV* a_cur, TV* a_next, int reverse, hipStream_t st) {
    const size_t lds = 2 * size_t(max_npn) * sizeof(TV) + size_t(max_ports) * 4;
    if (lds > 65536) return hipErrorInvalidValue;
    // Every other sweep walks backwards and finds in the caches what the sweep before read
    // last (FP32, one order / alternating: 3,720 sub-circuits of random cuts, 75 MB, 11.5 / 11.1
    // us a sweep, 5,852 of them 17.6 / 16.0, 288 MB in blocks of 8 55.0 / 54.2, 387 MB 87.1 /
    // 80.8; 28 more circuits of 56 to 225 MB, even and ragged, FP32 and FP64, the same within
    // 1%, as two runs of one kernel differ).
    // Up to twice the cache, plain loads reuse more of it
    // (358 MB: 30.9 ms a solve, 31.4 with the share that fits kept, 29.8 with none kept; 192
    // MB: 17.2, and 21-23 with any non-temporal); above, the share that fits is kept (700 MB:
    // 65.0 -> 58.7 ms, 59.5 with none kept; 1.44 GB: 144 -> 128, 133).
    constexpr int64_t kCache = int64_t(256) << 20;
    const int keep = op_bytes <= 2 * kCache ? 16 : std::max(1, int((16 * kCache + op_bytes / 2) / op_bytes));
    // FP64: rows and columns of a sub-circuit spread out, where a column's wavefronts have
    // enough of it or the sub-circuits alone do not fill the chip (solves, one workgroup per
    // sub-circuit / spread: 105 of 296 port nodes 11.0 / 7.2 ms, 512 of 98 8.6 / 6.7, 1,728 of
    // 98 21.4 / 23.9, 1,764 of 92 5.1 / 5.5, 961 of 124 5.37 / 5.18, 1,000 of 152 20.2 / 19.1,
    // 576 of 296 30.5 / 27.8, 729 of 296 48.9 / 40.5).  Of more than 320 port nodes, nearly as
    // many as the compute units keep a workgroup each where the operators fit the cache: their
    // six or more wavefronts on every unit stream from it at 7.3 TB/s, and spread out they make
    // more than one round (180 of 337 27.0 / 27.6 us a sweep, 210 uneven ones 26.8 / 28.4, 256
    // 30.9 / 32.8; 150 23.9 / 22.8, of 296 17.6 / 14.6, 240 of 488, 435 MB, 65.1 / 58.9).  So do
    // those of 193 to 320 between one and two a unit, which all run at once: within 6% either
    // way (300 of 296 28.2 / 27.4, 360 33.4 / 32.4, 420 37.8 / 37.8, 420 uneven ones 33.6 /
    // 34.8); of more nodes the spread form wins there, too (300 of 337 56.9 / 46.9, 490 91.8 /
    // 81.9, 300 of 488 108 / 78).
    // FP32 keeps the order of its sums: its inner solves stop near the rounding floor.
    if constexpr (sizeof(TO) == 8) {
        const int64_t ry = (max_npn + 63) / 64;
        const size_t need = (size_t(max_npn) + 64 * kPpnSplit) * 8 + size_t(max_ports) * 4;
        const int cus = compute_units();
        const bool one_round = (max_npn > 192 && max_npn <= 320 && S > cus && S < 2 * cus) ||
                               (max_npn > 320 && 3 * S > 2 * cus && S <= cus && op_bytes <= kCache);
        if ((max_npn > 112 || (max_npn > 64 && S <= 2 * cus)) && !one_round && S * ry <= INT32_MAX && need <= 65536) {
            auto kern = keep == 16 ? k_sweep_ppn_split<kPpnSplit, kPpnPairs, false>
                                   : k_sweep_ppn_split<kPpnSplit, kPpnPairs, true>;
            hipLaunchKernelGGL(kern, dim3(unsigned(S * ry)), dim3(64 * kPpnSplit), need, st, int(ry), Sn, nofs, pn_off,
                               pn_pfirst, port_off, port_twin, pc, pbeta, pgamma, h, a_cur, a_next, max_npn, reverse,
                               keep);
            return hipGetLastError();
        }
    }
    // one pass over the rows where possible
    const int bs = std::min(512, std::max(64, ((max_npn + 63) / 64) * 64));
    auto kern = keep == 16 ? k_sweep_ppn<TO, TV, false> : k_sweep_ppn<TO, TV, true>;
    hipLaunchKernelGGL(kern, dim3(S), dim3(bs), lds, st, Sn, nofs, pn_off, pn_pfirst, port_off, port_twin, pc, pbeta,
                       pgamma, h, a_cur, a_next, max_npn, reverse, keep);
    return hipGetLastError();
}

template hipError_t launch_port_node_dense<double>(int, const int32_t*, const int64_t*, const int32_t*,
                                                   const int32_t*, const double*, const int64_t*, double*, bool,
                                                   hipStream_t);
template hipError_t launch_port_node_dense<float>(int, const int32_t*, const int64_t*, const int32_t*,
                                                  const int32_t*, const float*, const int64_t*, float*, bool,
                                                  hipStream_t);
template hipError_t launch_sweep_ppn<double, double>(int, int, int, int64_t, const double*, const int64_t*, const int32_t*,
                                                     const int32_t*, const int32_t*, const int32_t*, const double*,
                                                     const double*, const double*, const double*, const double*,
                                                     double*, int, hipStream_t);
template hipError_t launch_sweep_ppn<float, float>(int, int, int, int64_t, const float*, const int64_t*, const int32_t*,
                                                   const int32_t*, const int32_t*, const int32_t*, const float*,
                                                   const float*, const float*, const float*, const float*, float*,
                                                   int, hipStream_t);

template <typename TO>
hipError_t launch_port_matrix(int S, const int32_t* sub_off, const int64_t* kofs, const int32_t* port_off,
                              const int32_t* port_node, const double* pc, const double* pbeta, const double* pgamma,
                              const TO* K, const int64_t* pofs, TO* M, hipStream_t st, Coupling<double> B) {
    // few sub-circuits: several workgroups each
    const int parts = S < 2048 ? (2048 + S - 1) / S : 1;
    hipLaunchKernelGGL(k_port_matrix<TO>, dim3(S, parts), dim3(kBlock), 0, st, sub_off, kofs, port_off, port_node,
                       pc, pbeta, pgamma, K, pofs, M, B);
    return hipGetLastError();
}

template <typename TV>
hipError_t launch_port_h(int S, int nrhs, const int32_t* sub_off, const int32_t* port_off, const int32_t* port_node,
                         const TV* pbeta, const TV* x, TV* h, hipStream_t st, Coupling<TV> B) {
    hipLaunchKernelGGL(k_port_h<TV>, dim3(S), dim3(nrhs > 1 ? 256 : 64), 0, st, nrhs, sub_off, port_off, port_node,
                       pbeta, x, h, B);
    return hipGetLastError();
}

template <typename TV>
hipError_t launch_wave_coupled(int n_ports, int nrhs, Coupling<TV> B, const int32_t* port_row, const TV* pgamma,
                               const int32_t* port_twin, const TV* x, const TV* a_cur, TV* a_next, hipStream_t st) {
    const int64_t total = int64_t(n_ports) * nrhs;
    if (total == 0) return hipSuccess;
    if (!B.row) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_wave_coupled<TV>, dim3(unsigned((total + kBlock - 1) / kBlock)), dim3(kBlock), 0, st,
                       n_ports, nrhs, B, port_row, pgamma, port_twin, x, a_cur, a_next);
    return hipGetLastError();
}
template hipError_t launch_wave_coupled<double>(int, int, Coupling<double>, const int32_t*, const double*,
                                                const int32_t*, const double*, const double*, double*, hipStream_t);
template hipError_t launch_wave_coupled<float>(int, int, Coupling<float>, const int32_t*, const float*,
                                               const int32_t*, const float*, const float*, float*, hipStream_t);

template <typename TO, typename TV, int R>
hipError_t launch_pp_r(int S, int max_q, int nrhs, const TO* M, const int64_t* pofs, const int32_t* port_off,
                       const int32_t* port_twin, const TV* h, const TV* a_cur, TV* a_next, hipStream_t st) {
    const int ny = (nrhs + R - 1) / R;
    const unsigned nb = unsigned(S) * unsigned(ny);
    const size_t lds = size_t(max_q > 0 ? max_q : 1) * R * sizeof(TV);
    if constexpr (R == 1)
        if (max_q <= 32) {
            hipLaunchKernelGGL((k_sweep_pp<TO, TV, 2, 1>), dim3(nb), dim3(64), lds, st, ny, nrhs, M, pofs, port_off,
                               port_twin, h, a_cur, a_next);
            return hipGetLastError();
        }
    // few sub-circuits with many ports: the rows of each spread over several workgroups
    // and its columns over their wavefronts
    if (S < 1024 && max_q > 64) {
        constexpr int KS = 8;
        const size_t lds2 = lds + size_t(KS) * 64 * R * sizeof(TV);
        if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(&k_sweep_pp_split<TO, TV, R, KS>), lds2);
            e != hipSuccess)
            return e;
        hipLaunchKernelGGL((k_sweep_pp_split<TO, TV, R, KS>), dim3(nb, unsigned((max_q + 63) / 64)), dim3(64 * KS),
                           lds2, st, ny, nrhs, M, pofs, port_off, port_twin, h, a_cur, a_next, max_q);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_sweep_pp<TO, TV, 1, R>), dim3(nb), dim3(max_q <= 64 ? 64 : 256), lds, st, ny, nrhs, M, pofs,
                       port_off, port_twin, h, a_cur, a_next);
    return hipGetLastError();
}

template <typename TO, typename TV>
hipError_t launch_sweep_pp(int S, int max_q, int nrhs, const TO* M, const int64_t* pofs, const int32_t* port_off,
                           const int32_t* port_twin, const TV* h, const TV* a_cur, TV* a_next, hipStream_t st) {
    if (S == 0) return hipSuccess;
    // the waves of a block of right-hand sides in 64 KiB of LDS
    auto fits = [&](int r) { return size_t(max_q > 0 ? max_q : 1) * r * sizeof(TV) <= 65536; };
    if (!fits(1)) return hipErrorInvalidValue;
    if (nrhs == 1 || !fits(2))
        return nrhs == 1 ? launch_pp_r<TO, TV, 1>(S, max_q, nrhs, M, pofs, port_off, port_twin, h, a_cur, a_next, st)
                         : hipErrorInvalidValue;
    if (nrhs == 2 || !fits(4))
        return launch_pp_r<TO, TV, 2>(S, max_q, nrhs, M, pofs, port_off, port_twin, h, a_cur, a_next, st);
    if (nrhs <= 4 || !fits(8))
        return launch_pp_r<TO, TV, 4>(S, max_q, nrhs, M, pofs, port_off, port_twin, h, a_cur, a_next, st);
    return launch_pp_r<TO, TV, 8>(S, max_q, nrhs, M, pofs, port_off, port_twin, h, a_cur, a_next, st);
}

template hipError_t launch_port_matrix<double>(int, const int32_t*, const int64_t*, const int32_t*, const int32_t*,
                                               const double*, const double*, const double*, const double*,
                                               const int64_t*, double*, hipStream_t, Coupling<double>);
template hipError_t launch_port_matrix<float>(int, const int32_t*, const int64_t*, const int32_t*, const int32_t*,
                                              const double*, const double*, const double*, const float*,
                                              const int64_t*, float*, hipStream_t, Coupling<double>);
template hipError_t launch_port_h<double>(int, int, const int32_t*, const int32_t*, const int32_t*, const double*,
                                          const double*, double*, hipStream_t, Coupling<double>);
template hipError_t launch_port_h<float>(int, int, const int32_t*, const int32_t*, const int32_t*, const float*,
                                         const float*, float*, hipStream_t, Coupling<float>);
template hipError_t launch_sweep_pp<double, double>(int, int, int, const double*, const int64_t*, const int32_t*,
                                                    const int32_t*, const double*, const double*, double*,
                                                    hipStream_t);
template hipError_t launch_sweep_pp<float, float>(int, int, int, const float*, const int64_t*, const int32_t*,
                                                  const int32_t*, const float*, const float*, float*, hipStream_t);

}  // namespace vtm

// ---------------------------------------------------------------------------
// Symmetric A: the port-node form.  K^-1 restricted to the port nodes,
// S = K^-1[N, N], is symmetric, and with beta = 2 W c and gamma = 1 - 2 c the
// outgoing waves are
//     o_p = 2 W_p c_p z_n(p) + (1 - 2 c_p) a_p + h_p,   z = S t,  t_n = sum_{p at n} c_p a_p,
// so a sweep streams only the upper triangle of S besides the per-port wave,
// c, h and twin.  The triangle of a sub-circuit with k port nodes is stored as
// pairs of diagonals: pair m holds, for rows r = 0 .. k - 2m - 1, the two
// entries S(r, r + 2m) and S(r, r + 2m + 1) side by side (the second is zero
// in the pair's last row), and starts at 2m (k - m + 1).  Lane r reads both
// entries of every pair with one coalesced 16-byte (FP64) load and receives
// S(r - d, r) from lane r - d.
// ---------------------------------------------------------------------------
namespace vtm {
namespace {

// diagonals per chunk of the packed sweep, each lane's loads of one chunk in
// flight together (even: whole pairs)
constexpr int kPpsChunk = 8;
// chunks issued before the first barrier when two sub-circuits share a wavefront
// (the rest stream that far ahead)
constexpr int kPpsPre = 2;
// the same in FP64 (pps_pair64): 1 to 4 chunks ahead make 22.6, 22.0, 21.2, 21.2 ms of
// a 2048 x 2048 solve, and 5.58, 5.60, 5.36, 5.50 ms of one of 1000 x 1000
constexpr int kPpsPre64 = 3;
// wavefronts per sub-circuit when a sub-circuit has 33..64 port nodes (k_sweep_pps_split)
constexpr int kPpsSplit = 8;

// pair m of diagonals (2m, 2m + 1), rows r = 0 .. k - 2m - 1 each holding both entries
__host__ __device__ inline int pair_start(int k, int m) { return 2 * m * (k - m + 1); }

template <typename TO>
__global__ void __launch_bounds__(256)
    k_port_node_matrix(const int32_t* __restrict__ sub_off, const int64_t* __restrict__ kofs,
                       const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_node,
                       const TO* __restrict__ K, const int64_t* __restrict__ sofs, TO* __restrict__ Sp) {
    const int s = blockIdx.x;
    const int ns = sub_off[s + 1] - sub_off[s];
    const int k0 = pn_off[s], k = pn_off[s + 1] - k0;
    const TO* Ks = K + kofs[s];
    TO* out = Sp + sofs[s];
    for (int t = threadIdx.x; t < k * k; t += blockDim.x) {
        const int r = t / k, c = t - r * k;
        if (r <= c)
            out[pair_start(k, (c - r) >> 1) + 2 * r + ((c - r) & 1)] =
                Ks[inv_offset<TO>(ns, pn_node[k0 + r], pn_node[k0 + c])];
    }
}

// One wavefront per sub-circuit (HALF: two, 32 lanes each).  Lane r owns port
// node r and port r of its sub-circuit.  The offsets come from scalar loads of
// a wave-uniform base; every other global load of the sweep is issued before
// the first barrier, PRE chunks of CH diagonals among them, and the rest
// stream PRE chunks ahead of use.  Inside a chunk there are no branches: a
// lane past the end of a pair loads a valid entry (the block's first two) and
// multiplies it by a zero of the padded t (each sub-circuit's t takes a
// 64-entry region, zero beyond its k port nodes), so the compiler can keep
// loads in flight across it; the only branch, a wave-uniform exit once the
// chunks pass the larger k of the wavefront, is scalar.
template <typename TO, typename TV, bool HALF>
__device__ inline void pps_unit(int unit, int S, const TO* __restrict__ Sp, const int64_t* __restrict__ sofs,
                                const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_pfirst,
                                const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
                                const TV* __restrict__ pc, const TV* __restrict__ pW, TV W,
                                const TV* __restrict__ h, const TV* __restrict__ a_cur, TV* __restrict__ a_next,
                                TV* ca, TV* tv, TV* zv, int32_t* pnode) {
    constexpr int L = HALF ? 32 : 64;
    constexpr int CH = kPpsChunk;
    constexpr int NCH = L / CH;
    constexpr int PRE = HALF ? kPpsPre : 1;
    static_assert(L % CH == 0 && PRE >= 1 && PRE <= NCH, "diagonal chunks must tile the lanes");
    const int tid = threadIdx.x, r = tid % L, hb = tid - r, half = tid / L;
    const int tb = half * 64;  // this sub-circuit's t region
    // wave-uniform offsets of the (one or two) sub-circuits, indices clamped to S
    const int sb = unit * (64 / L);
    const int sa = min(sb, S), sm = min(sb + 1, S), sz = min(sb + 2, S);
    const int nA = pn_off[sa], nB = pn_off[sm], nC = HALF ? pn_off[sz] : 0;
    const int pA = port_off[sa], pB = port_off[sm], pC = HALF ? port_off[sz] : 0;
    const int64_t eA = sofs[sa], eB = HALF ? sofs[sm] : 0;
    const bool valid = sb + half < S;
    const int n0 = half ? nB : nA, k = valid ? (half ? nC - nB : nB - nA) : 0;
    const int p0 = half ? pB : pA, q = valid ? (half ? pC - pB : pB - pA) : 0;
    const TO* blk = Sp + (valid ? (half ? eB : eA) : 0);
    const bool has_port = r < q;
    TV c = TV(0), a = TV(0), hp = TV(0), w = W;
    int tw = 0;
    if (has_port) {
        const int p = p0 + r;
        c = pc[p];
        a = a_cur[p];
        hp = h[p];
        tw = port_twin[p];
        if (pW) w = pW[p];
        ca[hb + r] = c * a;
    }
    int f0 = 0, f1 = 0;
    if (r < k) f0 = pn_pfirst[n0 + r] - p0;
    {
        const int nx = __shfl(f0, tid + 1);  // lane r + 1's first port (the last lane: q)
        f1 = r + 1 < k ? nx : q;
    }
    TO buf[L];  // diagonal d of this lane's row (compile-time indices only)
    // CH / 2 pairs per chunk, one 16-byte (FP64) load each: S(r, r + 2m), S(r, r + 2m + 1)
    static_assert(CH % 2 == 0, "chunks hold whole pairs");
    using V2 = typename std::conditional<sizeof(TO) == 8, double2, float2>::type;
    auto load = [&](int ci) {
#pragma unroll
        for (int j = 0; j < CH / 2; ++j) {
            const int m = ci * (CH / 2) + j;
            const V2 v2 = *reinterpret_cast<const V2*>(blk + ((r + 2 * m < k) ? pair_start(k, m) + 2 * r : 0));
            buf[2 * m] = v2.x;
            buf[2 * m + 1] = v2.y;
        }
    };
#pragma unroll
    for (int ci = 0; ci < PRE; ++ci) load(ci);
    tv[tid] = TV(0);
    tv[tid + 64] = TV(0);
    __syncthreads();
    // t_n = sum of c_p a_p over the ports at n, in port order
    if (r < k) {
        TV acc = TV(0);
        for (int i = f0; i < f1; ++i) {
            acc += ca[hb + i];
            pnode[hb + i] = r;
        }
        tv[tb + r] = acc;
    }
    __syncthreads();
    // z_r = sum_d S(r, r + d) t_{r+d} + sum_{d>0} S(r - d, r) t_{r-d}; the second
    // product is formed by lane r - d (which holds S(r - d, r)) and shuffled up.
    // d < L keeps tb + r + d inside tv.
    const TV tr = tv[tb + r];
    TV acc = TV(0);
    int kmax = k;
    if (HALF) kmax = max(k, __shfl_xor(k, 32));
    kmax = __builtin_amdgcn_readfirstlane(kmax);  // wave-uniform: the chunk loop branches on scalars
#pragma unroll
    for (int ci = 0; ci < NCH; ++ci) {
        if (ci * CH >= kmax) break;
        if (ci + PRE < NCH) load(ci + PRE);
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int d = ci * CH + j;
            const TV sv = TV(buf[d]);
            acc += sv * tv[tb + r + d];
            const TV up = __shfl(sv * tr, tid - d);
            acc += (d > 0 && r >= d) ? up : TV(0);
        }
    }
    if (r < k) zv[hb + r] = acc;
    __syncthreads();
    if (has_port) a_next[tw] = packed_wave_out<TV>(TV(2) * w * c, c, zv[hb + pnode[hb + r]], a, hp);
}

// v of the lane below (0 in lane 0): one shift of the wavefront
__device__ inline double shift_up(double v) {
    const u64p b = __builtin_bit_cast(u64p, v);
    const int lo = __builtin_amdgcn_update_dpp(0, int(unsigned(b)), 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, int(unsigned(b >> 32)), 0x138, 0xf, 0xf, true);
    return __builtin_bit_cast(double, u64p(unsigned(lo)) | (u64p(unsigned(hi)) << 32));
}

// The same in FP64, the lower triangle's products gathered by single-lane shifts: with
// the diagonals taken from the last to the first, low = shift_up(low + S(r, r + d) t_r)
// ends as sum_{d>0} S(r - d, r) t_{r-d}.  A shift is two register moves; a product
// shuffled d lanes up goes through LDS twice, and those instructions bound the sweep of
// operators that the memory-side cache holds (1000 x 1000 in 8x8 blocks, 70 MB: a solve
// 6.62 -> 5.36 ms; 1500 x 1500, 158 MB: 12.1 -> 11.1).  Past that it is the stream of the
// operators (2048 x 2048, 295 MB: 21.9 -> 21.2, 3000 x 3000: 53.3 -> 52.3), for which the
// loads run one chunk further ahead.  They are range-checked buffer loads: a lane past the
// end of a pair reads zeros, so that nothing of one sub-circuit is shifted into the other.
// FP32 keeps the shuffles, and with them the order of its sums: its inner solves stop near
// the rounding floor, where another order moves the sweep at which they stop.
// NCH: chunks of diagonals held, all that the largest sub-circuit has.  With four a wavefront
// takes 94 registers; operators of up to 8 port nodes need one, and their sweeps as many
// wavefronts as fit (111,556 sub-circuits of 8, 1000 x 1000 in 3x3 blocks: shuffled 25.6 us a
// sweep, four chunks 26.3, one 19.7; 250,000 of 4: 52.3, 54.7, 39.1).
template <int NCH>
__device__ inline void pps_pair64(int unit, int S, const double* __restrict__ Sp, const int64_t* __restrict__ sofs,
                                  const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_pfirst,
                                  const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
                                  const double* __restrict__ pc, const double* __restrict__ pW, double W,
                                  const double* __restrict__ h, const double* __restrict__ a_cur,
                                  double* __restrict__ a_next, double* ca, double* tv, double* zv, int32_t* pnode) {
    constexpr int L = 32, CH = kPpsChunk, PRE = kPpsPre64 < NCH ? kPpsPre64 : NCH;
    static_assert(L % CH == 0 && NCH * CH <= L && CH % 2 == 0 && PRE >= 1 && PRE <= NCH, "whole pairs in chunks that tile the lanes");
    const int tid = threadIdx.x, r = tid % L, hb = tid - r, half = tid / L;
    const int tb = half * 64;  // this sub-circuit's t region
    // wave-uniform offsets of the two sub-circuits, indices clamped to S
    const int sb = unit * 2;
    const int sa = min(sb, S), sm = min(sb + 1, S), sz = min(sb + 2, S);
    const int nA = pn_off[sa], nB = pn_off[sm], nC = pn_off[sz];
    const int pA = port_off[sa], pB = port_off[sm], pC = port_off[sz];
    const int64_t eA = sofs[sa], eB = sofs[sm], eC = sofs[sz];
    const int n0 = half ? nB : nA, k = half ? nC - nB : nB - nA;
    const int p0 = half ? pB : pA, q = half ? pC - pB : pB - pA;
    const int kmax = max(nB - nA, nC - nB), top = (kmax + CH - 1) / CH;
    // the two blocks are neighbours in memory: one resource over both
    const __amdgpu_buffer_rsrc_t ops =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(Sp) + eA, 0, int(unsigned(eC - eA) * 8u), 0x00020000);
    const unsigned blk = half ? unsigned(eB - eA) * 8u : 0u;
    const bool has_port = r < q;
    double c = 0.0, a = 0.0, hp = 0.0, w = W;
    int tw = 0;
    if (has_port) {
        const int p = p0 + r;
        c = pc[p];
        a = a_cur[p];
        hp = h[p];
        tw = port_twin[p];
        if (pW) w = pW[p];
        ca[hb + r] = c * a;
    }
    int f0 = 0, f1 = 0;
    if (r < k) f0 = pn_pfirst[n0 + r] - p0;
    {
        const int nx = __shfl(f0, tid + 1);  // lane r + 1's first port (the last lane: q)
        f1 = r + 1 < k ? nx : q;
    }
    double buf[NCH * CH];  // diagonal d of this lane's row (compile-time indices only)
    auto load = [&](int ci) {
#pragma unroll
        for (int j = 0; j < CH / 2; ++j) {
            const int m = ci * (CH / 2) + j;
            const unsigned off = r + 2 * m < k ? blk + 8u * unsigned(pair_start(k, m) + 2 * r) : 0x80000000u;
            const pp_d2 v2 = __builtin_bit_cast(pp_d2, __builtin_amdgcn_raw_buffer_load_b128(ops, int(off), 0, 0));
            buf[2 * m] = v2.x;
            buf[2 * m + 1] = v2.y;
        }
    };
#pragma unroll
    for (int ci = NCH - 1; ci >= 0; --ci)
        if (ci < top && ci >= top - PRE) load(ci);
    tv[tid] = 0.0;
    tv[tid + 64] = 0.0;
    __syncthreads();
    // t_n = sum of c_p a_p over the ports at n, in port order
    if (r < k) {
        double acc = 0.0;
        for (int i = f0; i < f1; ++i) {
            acc += ca[hb + i];
            pnode[hb + i] = r;
        }
        tv[tb + r] = acc;
    }
    __syncthreads();
    // a t that is not finite makes every z of its sub-circuit so, and is kept out of the
    // shifts: its products with the zeros past a pair's end would reach the other one
    const double t = tv[tb + r];
    const bool finite = __builtin_isfinite(t);
    const bool lost = ((~__ballot(finite)) >> hb & 0xffffffffull) != 0;
    const double tr = finite ? t : 0.0;
    double acc = lost ? __builtin_nan("") : 0.0, low = 0.0;
#pragma unroll
    for (int ci = NCH - 1; ci >= 0; --ci) {
        if (ci >= top) continue;  // scalar
        if (ci >= PRE) load(ci - PRE);
#pragma unroll
        for (int j = CH - 1; j >= 0; --j) {
            const int d = ci * CH + j;
            acc += buf[d] * tv[tb + r + d];
            if (d > 0) low = shift_up(low + buf[d] * tr);
        }
    }
    if (r < k) zv[hb + r] = acc + low;
    __syncthreads();
    if (has_port) a_next[tw] = packed_wave_out<double>(2.0 * w * c, c, zv[hb + pnode[hb + r]], a, hp);
}

// One workgroup (one wavefront) per unit: a pair of sub-circuits when HALF (then FP64
// takes pps_pair64, of NCH chunks).
template <typename TO, typename TV, bool HALF, int NCH>
__global__ void __launch_bounds__(64)
    k_sweep_pps(int S, const TO* __restrict__ Sp, const int64_t* __restrict__ sofs,
                const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_pfirst,
                const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
                const TV* __restrict__ pc, const TV* __restrict__ pW, TV W, const TV* __restrict__ h,
                const TV* __restrict__ a_cur, TV* __restrict__ a_next, int reverse) {
    __shared__ TV ca[64], tv[128], zv[64];
    __shared__ int32_t pnode[64];
    // every other sweep walks each XCD's units backwards, so that the operators it
    // reads first are the ones the previous sweep read last (still in the
    // memory-side cache), while each XCD keeps the same units (and its L2)
    const int unit = reverse ? xcd_block_reversed(blockIdx.x, gridDim.x) : xcd_block(blockIdx.x, gridDim.x);
    if constexpr (HALF && sizeof(TO) == 8)
        pps_pair64<NCH>(unit, S, Sp, sofs, pn_off, pn_pfirst, port_off, port_twin, pc, pW, W, h, a_cur, a_next, ca, tv,
                        zv, pnode);
    else
        pps_unit<TO, TV, HALF>(unit, S, Sp, sofs, pn_off, pn_pfirst, port_off, port_twin, pc, pW, W, h, a_cur, a_next,
                               ca, tv, zv, pnode);
}

// One sub-circuit of up to 64 port nodes per workgroup of WV wavefronts: lane r of
// every wavefront keeps row r, and wavefront v takes the diagonal chunks
// v, v + WV, ...  All of a wavefront's operator loads are issued at once, before
// the first barrier (WV times fewer per lane than with one wavefront, so the
// sweep of few, large sub-circuits waits on fewer round trips); the partial
// sums z_r of the wavefronts meet in LDS.
template <typename TO, typename TV, int WV>
__global__ void __launch_bounds__(64 * WV)
    k_sweep_pps_split(const TO* __restrict__ Sp, const int64_t* __restrict__ sofs,
                      const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_pfirst,
                      const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin,
                      const TV* __restrict__ pc, const TV* __restrict__ pW, TV W, const TV* __restrict__ h,
                      const TV* __restrict__ a_cur, TV* __restrict__ a_next, int reverse) {
    constexpr int CH = kPpsChunk, NCH = 64 / CH, LCH = NCH / WV;
    static_assert(WV >= 2 && NCH % WV == 0 && CH % 2 == 0, "chunks must split evenly over the wavefronts");
    __shared__ TV ca[64], tv[128], zp[WV][64];
    __shared__ int32_t pnode[64];
    const int s = reverse ? xcd_block_reversed(blockIdx.x, gridDim.x) : xcd_block(blockIdx.x, gridDim.x);
    const int tid = threadIdx.x, r = tid & 63, wv = tid >> 6;
    const int n0 = pn_off[s], k = pn_off[s + 1] - n0;
    const int p0 = port_off[s], q = port_off[s + 1] - p0;
    const TO* blk = Sp + sofs[s];
    // this wavefront's diagonals d = ci CH + j, ci = li WV + wv (pairs: one 16-byte
    // FP64 load gives S(r, r + 2m) and S(r, r + 2m + 1))
    using V2 = typename std::conditional<sizeof(TO) == 8, double2, float2>::type;
    TO buf[LCH * CH];
#pragma unroll
    for (int li = 0; li < LCH; ++li) {
        const int ci = li * WV + wv;
        if (ci * CH < k) {
#pragma unroll
            for (int j = 0; j < CH / 2; ++j) {
                const int m = ci * (CH / 2) + j;
                const V2 v2 = *reinterpret_cast<const V2*>(blk + ((r + 2 * m < k) ? pair_start(k, m) + 2 * r : 0));
                buf[li * CH + 2 * j] = v2.x;
                buf[li * CH + 2 * j + 1] = v2.y;
            }
        }
    }
    // wavefront 0: the ports (lane r = port p0 + r) and each node's port range
    TV c = TV(0), a = TV(0), hp = TV(0), w = W;
    int tw = 0, f0 = 0, f1 = 0;
    const bool has_port = wv == 0 && r < q;
    if (has_port) {
        const int p = p0 + r;
        c = pc[p];
        a = a_cur[p];
        hp = h[p];
        tw = port_twin[p];
        if (pW) w = pW[p];
        ca[r] = c * a;
    }
    if (wv == 0 && r < k) {
        f0 = pn_pfirst[n0 + r] - p0;
        f1 = pn_pfirst[n0 + r + 1] - p0;
    }
    if (tid < 128) tv[tid] = TV(0);
    __syncthreads();
    // t_n = sum of c_p a_p over the ports at node n, in port order
    if (wv == 0 && r < k) {
        TV acc = TV(0);
        for (int i = f0; i < f1; ++i) {
            acc += ca[i];
            pnode[i] = r;
        }
        tv[r] = acc;
    }
    __syncthreads();
    // partial z_r over this wavefront's diagonals: S(r, r + d) t_{r+d}, and for
    // d > 0 S(r - d, r) t_{r-d}, formed by lane r - d and shuffled up
    const TV tr = tv[r];
    TV acc = TV(0);
#pragma unroll
    for (int li = 0; li < LCH; ++li) {
        const int ci = li * WV + wv;
        if (ci * CH < k) {
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int d = ci * CH + j;
                const TV sv = TV(buf[li * CH + j]);
                acc += sv * tv[r + d];
                const TV up = __shfl(sv * tr, r - d);
                acc += (d > 0 && r >= d) ? up : TV(0);
            }
        }
    }
    zp[wv][r] = acc;
    __syncthreads();
    if (has_port) {
        const int n = pnode[r];
        TV z = TV(0);
#pragma unroll
        for (int v = 0; v < WV; ++v) z += zp[v][n];
        a_next[tw] = packed_wave_out<TV>(TV(2) * w * c, c, z, a, hp);
    }
}

}  // namespace

template <typename TO>
hipError_t launch_port_node_matrix(int S, const int32_t* sub_off, const int64_t* kofs, const int32_t* pn_off,
                                   const int32_t* pn_node, const TO* K, const int64_t* sofs, TO* Sp,
                                   hipStream_t st) {
    hipLaunchKernelGGL(k_port_node_matrix<TO>, dim3(S), dim3(256), 0, st, sub_off, kofs, pn_off, pn_node, K, sofs,
                       Sp);
    return hipGetLastError();
}

template <typename TO, typename TV, bool HALF, int NCH>
hipError_t launch_pps(int S, const TO* Sp, const int64_t* sofs, const int32_t* pn_off, const int32_t* pn_pfirst,
                      const int32_t* port_off, const int32_t* port_twin, const TV* pc, const TV* pW, TV W,
                      const TV* h, const TV* a_cur, TV* a_next, int reverse, hipStream_t st) {
    const int units = HALF ? (S + 1) / 2 : S;
    hipLaunchKernelGGL((k_sweep_pps<TO, TV, HALF, NCH>), dim3(units), dim3(64), 0, st, S, Sp, sofs, pn_off, pn_pfirst,
                       port_off, port_twin, pc, pW, W, h, a_cur, a_next, reverse);
    return hipGetLastError();
}

template <typename TO, typename TV>
hipError_t launch_sweep_pps(int S, int max_npn, int max_ports, const TO* Sp, const int64_t* sofs,
                            const int32_t* pn_off, const int32_t* pn_pfirst, const int32_t* port_off,
                            const int32_t* port_twin, const TV* pc, const TV* pW, TV W, const TV* h,
                            const TV* a_cur, TV* a_next, int reverse, hipStream_t st) {
    if (max_npn > 64 || max_ports > 64) return hipErrorInvalidValue;
    if (S == 0) return hipSuccess;
    if constexpr (sizeof(TO) == 8)
        if (max_npn <= kPpsChunk && max_ports <= 32)
            return launch_pps<TO, TV, true, 1>(S, Sp, sofs, pn_off, pn_pfirst, port_off, port_twin, pc, pW, W, h, a_cur,
                                               a_next, reverse, st);
    if (max_npn <= 32 && max_ports <= 32)
        return launch_pps<TO, TV, true, 32 / kPpsChunk>(S, Sp, sofs, pn_off, pn_pfirst, port_off, port_twin, pc, pW, W, h, a_cur,
                                        a_next, reverse, st);
    hipLaunchKernelGGL((k_sweep_pps_split<TO, TV, kPpsSplit>), dim3(S), dim3(64 * kPpsSplit), 0, st, Sp, sofs, pn_off,
                       pn_pfirst, port_off, port_twin, pc, pW, W, h, a_cur, a_next, reverse);
    return hipGetLastError();
}

template hipError_t launch_port_node_matrix<double>(int, const int32_t*, const int64_t*, const int32_t*,
                                                    const int32_t*, const double*, const int64_t*, double*,
                                                    hipStream_t);
template hipError_t launch_port_node_matrix<float>(int, const int32_t*, const int64_t*, const int32_t*,
                                                   const int32_t*, const float*, const int64_t*, float*,
                                                   hipStream_t);
template hipError_t launch_sweep_pps<double, double>(int, int, int, const double*, const int64_t*,
                                                     const int32_t*, const int32_t*, const int32_t*, const int32_t*,
                                                     const double*, const double*, double, const double*,
                                                     const double*, double*, int, hipStream_t);
template hipError_t launch_sweep_pps<float, float>(int, int, int, const float*, const int64_t*, const int32_t*,
                                                   const int32_t*, const int32_t*, const int32_t*, const float*,
                                                   const float*, float, const float*, const float*, float*, int,
                                                   hipStream_t);

}  // namespace vtm

// ---------------------------------------------------------------------------
// Several right-hand sides: the port-node form on the matrix cores.
// ---------------------------------------------------------------------------
namespace vtm {
namespace {

typedef double ppt_d4 __attribute__((ext_vector_type(4)));
typedef float ppt_f4 __attribute__((ext_vector_type(4)));

template <typename T>
struct NodeMma;
template <>
struct NodeMma<double> {
    using Frag = double2;
    using Acc = ppt_d4;
    static __device__ Acc step(const Frag& a, int j, double b, Acc acc) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(j ? a.y : a.x, b, acc, 0, 0, 0);
    }
    static __device__ int out_row(int l, int v) { return (l >> 4) + 4 * v; }
};
template <>
struct NodeMma<float> {
    using Frag = float4;
    using Acc = ppt_f4;
    static __device__ Acc step(const Frag& a, int j, float b, Acc acc) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(j == 0 ? a.x : j == 1 ? a.y : j == 2 ? a.z : a.w, b, acc, 0, 0, 0);
    }
    static __device__ int out_row(int l, int v) { return 4 * (l >> 4) + v; }
};

template <typename T>
__global__ void __launch_bounds__(256)
    k_port_node_tiles(const int32_t* __restrict__ sub_off, const int64_t* __restrict__ kofs,
                      const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_node, const T* __restrict__ K,
                      const int64_t* __restrict__ ntofs, T* __restrict__ Nt, int transpose) {
    const int s = blockIdx.x;
    const int ns = sub_off[s + 1] - sub_off[s];
    const int k0 = pn_off[s], k = pn_off[s + 1] - k0;
    constexpr int KT = 64 / int(sizeof(T)), E = KT / 4;
    const int np = node_tile_pad(k), kt_n = np / KT, units = np / 16 * kt_n * 64;
    const T* Ks = K + kofs[s];
    T* out = Nt + ntofs[s];
    // a thread the 16 bytes of one lane in one tile (node_tile_rc)
    for (int u = blockIdx.y * blockDim.x + threadIdx.x; u < units; u += blockDim.x * gridDim.y) {
        const int tile = u >> 6, lane = u & 63, mt = tile / kt_n, kt = tile - mt * kt_n;
        const int r = mt * 16 + (lane & 15), c0 = kt * KT + (lane >> 4);
        const int nr = r < k ? pn_node[k0 + r] : 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const int c = c0 + 4 * j;
            T v = T(0);
            if (r < k && c < k) {
                const int nc = pn_node[k0 + c];
                v = Ks[transpose ? inv_offset<T>(ns, nc, nr) : inv_offset<T>(ns, nr, nc)];
            }
            out[int64_t(u) * E + j] = v;
        }
    }
}

// A tiles in flight per wavefront
constexpr int kPptAhead = 4;

// One workgroup per sub-circuit and block of w <= 16 right-hand sides.  NI > 0: a
// thread keeps its (at most NI) items -- a port and a right-hand side -- in
// registers from its first loads to its stores; 0: it reads them again.  All loads
// that depend on nothing but the sub-circuit's offsets are issued first: the
// waves, coefficients, h and twins of the thread's (port, right-hand side) items,
// and the wavefront's first A tiles.  c a goes to LDS per port, is summed per port
// node in port order into T (the B operand, [node][w]); each wavefront then forms
// row tiles of Z, which replaces c a in LDS, and every item's thread its wave.
// The matrix cores take 16 columns at a time; lanes of columns past w read column
// w - 1 again and their results are dropped.  They are used for few columns too
// because a vector form reads a staged value from LDS per multiply-add, and that
// alone would take as long.  At the measured sizes it is bound by instructions and by
// latency (226 vector instructions a wavefront, 3 of its 7 us waiting on memory), not
// by bytes: 3,276 sub-circuits of 8x8, six right-hand sides, FP64: 9.3 us a sweep (10.9
// with a run-time division per item and gamma, a and h held apart), the full inverses
// it replaces 29.1; 768 of 16x16, four, FP32: 5.8 against 35.  A form that reads the
// packed triangles instead (40% of the operator's bytes) and picks its operands out of
// LDS took 11.5 us.
template <typename T, int NI>
__global__ void __launch_bounds__(512)
    k_sweep_ppt(int ny, int rc, unsigned irc, int nrhs, const T* __restrict__ Nt, const int64_t* __restrict__ ntofs,
                const int32_t* __restrict__ pn_off, const int32_t* __restrict__ pn_pfirst,
                const int32_t* __restrict__ port_off, const int32_t* __restrict__ port_twin, const T* __restrict__ pc,
                const T* __restrict__ pbeta, const T* __restrict__ pgamma, const T* __restrict__ h,
                const T* __restrict__ a_cur, T* __restrict__ a_next, int max_np, int max_rows, int reverse) {
    using M = NodeMma<T>;
    constexpr int KT = 64 / int(sizeof(T)), E = KT / 4;
    extern __shared__ char smem[];
    const int u = reverse ? xcd_block_reversed(blockIdx.x, gridDim.x) : xcd_block(blockIdx.x, gridDim.x);
    const int s = u / ny, r0 = (u - s * ny) * rc;
    const int w = min(rc, nrhs - r0);
    // t / w (t < 2^28, w <= 16) as one multiplication
    const unsigned iw = w == rc ? irc : 0xffffffffu / unsigned(w) + 1u;
    auto over = [&](int t) { return w == 1 ? t : int(__umulhi(unsigned(t), iw)); };
    T* tv = reinterpret_cast<T*>(smem);            // [max_np][rc]
    T* ca = tv + max_np * rc;                      // [max_rows][rc]: c a per port, then Z per port node
    int32_t* pnode = reinterpret_cast<int32_t*>(ca + max_rows * rc);  // [q] (pf after it)
    const int p0 = port_off[s], q = port_off[s + 1] - p0;
    const int k0 = pn_off[s], k = pn_off[s + 1] - k0;
    int32_t* pf = pnode + q;                       // [k + 1]
    const int np = node_tile_pad(k), kt_n = np / KT, mt_n = np / 16;
    const int tid = threadIdx.x, bs = blockDim.x, lane = tid & 63, wave = tid >> 6, waves = bs >> 6;
    const typename M::Frag* A0 = reinterpret_cast<const typename M::Frag*>(Nt + ntofs[s]) + lane;
    // this wavefront's A tiles in order: row tiles wave, wave + waves, ..., each kt_n long;
    // the next kPptAhead are always in flight, across row tiles too
    typename M::Frag af[kPptAhead];
    int lmt = wave, lkt = 0;
    auto next_tile = [&](typename M::Frag& f) {
        if (lmt < mt_n) f = A0[(int64_t(lmt) * kt_n + lkt) * 64];
        if (++lkt == kt_n) {
            lkt = 0;
            lmt += waves;
        }
    };
#pragma unroll
    for (int d = 0; d < kPptAhead; ++d) next_tile(af[d]);
    const int items = q * w;
    constexpr int NR = NI > 0 ? NI : 1;
    T vb[NR], vr[NR];  // beta, gamma a + h
    int tw[NR];
    if constexpr (NI > 0) {
        T va[NR], vh[NR], vg[NR], vc[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int t = tid + i * bs;
            va[i] = vh[i] = vb[i] = vg[i] = vc[i] = T(0);
            tw[i] = 0;
            if (t < items) {
                const int pl = over(t), p = p0 + pl;
                const int64_t o = int64_t(p) * nrhs + r0 + (t - pl * w);
                va[i] = a_cur[o];
                vc[i] = pc[p];
                vh[i] = h[o];
                vb[i] = pbeta[p];
                vg[i] = pgamma[p];
                tw[i] = port_twin[p];
            }
        }
        for (int j = tid; j <= k; j += bs) pf[j] = pn_pfirst[k0 + j] - p0;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int t = tid + i * bs;
            if (t < items) ca[t] = vc[i] * va[i];
            vr[i] = vg[i] * va[i] + vh[i];
        }
    } else {
        for (int j = tid; j <= k; j += bs) pf[j] = pn_pfirst[k0 + j] - p0;
        for (int t = tid; t < items; t += bs) {
            const int pl = over(t), p = p0 + pl;
            ca[t] = pc[p] * a_cur[int64_t(p) * nrhs + r0 + (t - pl * w)];
        }
    }
    __syncthreads();
    for (int t = tid; t < np * w; t += bs) {
        const int j = over(t), r = t - j * w;
        T acc = T(0);
        if (j < k) {
            const int f1 = pf[j + 1];
            for (int p = pf[j]; p < f1; ++p) {
                acc += ca[p * w + r];
                if (r == 0) pnode[p] = j;
            }
        }
        tv[t] = acc;
    }
    __syncthreads();
    const int nc = min(lane & 15, w - 1);
    for (int mt = wave; mt < mt_n; mt += waves) {
        typename M::Acc acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = T(0);
        // kt_n is a multiple of 2 (FP64) or 1 (FP32); the ring turns by U tiles
        constexpr int U = sizeof(T) == 8 ? 2 : 1;
        for (int kt = 0; kt < kt_n; kt += U) {
#pragma unroll
            for (int d = 0; d < U; ++d) {
                const typename M::Frag a = af[d];
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    const T b = tv[((kt + d) * KT + 4 * j + (lane >> 4)) * w + nc];
                    acc = M::step(a, j, b, acc);
                }
            }
#pragma unroll
            for (int d = 0; d + U < kPptAhead; ++d) af[d] = af[d + U];
#pragma unroll
            for (int d = kPptAhead - U; d < kPptAhead; ++d) next_tile(af[d]);
        }
        if ((lane & 15) < w) {
#pragma unroll
            for (int v = 0; v < 4; ++v) ca[(mt * 16 + M::out_row(lane, v)) * w + nc] = acc[v];
        }
    }
    __syncthreads();
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int t = tid + i * bs;
            if (t < items) {
                const int p = over(t), r = t - p * w;
                a_next[int64_t(tw[i]) * nrhs + r0 + r] = vb[i] * ca[pnode[p] * w + r] + vr[i];
            }
        }
    } else {
        for (int t = tid; t < items; t += bs) {
            const int p = over(t), r = t - p * w;
            const int64_t o = int64_t(p0 + p) * nrhs + r0 + r;
            a_next[int64_t(port_twin[p0 + p]) * nrhs + r0 + r] =
                pbeta[p0 + p] * ca[pnode[p] * w + r] + (pgamma[p0 + p] * a_cur[o] + h[o]);
        }
    }
}

}  // namespace

template <typename T>
hipError_t launch_port_node_tiles(int S, const int32_t* sub_off, const int64_t* kofs, const int32_t* pn_off,
                                  const int32_t* pn_node, const T* K, const int64_t* ntofs, T* Nt, bool transpose,
                                  hipStream_t st) {
    if (S == 0) return hipSuccess;
    // few sub-circuits: up to 32 workgroups each
    const int y = std::max(1, std::min(32, 4 * compute_units() / S));
    hipLaunchKernelGGL(k_port_node_tiles<T>, dim3(S, y), dim3(256), 0, st, sub_off, kofs, pn_off, pn_node, K, ntofs, Nt,
                       transpose ? 1 : 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_sweep_ppt(int S, int max_npn, int max_ports, int nrhs, size_t lds_limit, const T* Nt,
                            const int64_t* ntofs, const int32_t* pn_off, const int32_t* pn_pfirst,
                            const int32_t* port_off, const int32_t* port_twin, const T* pc, const T* pbeta,
                            const T* pgamma, const T* h, const T* a_cur, T* a_next, int reverse, hipStream_t st) {
    if (S == 0) return hipSuccess;
    const int np = node_tile_pad(max_npn), rows = std::max(np, max_ports);
    // at most 16 right-hand sides a workgroup (an MFMA's columns), fewer where their
    // staging would leave a CU less than two workgroups
    int rc = std::min(16, nrhs);
    while (rc > 1 && ppt_lds_bytes<T>(np, max_ports, rc) > std::min<size_t>(lds_limit, 80 * 1024)) rc = (rc + 1) / 2;
    const size_t lds = ppt_lds_bytes<T>(np, max_ports, rc);
    if (lds > lds_limit) return hipErrorInvalidValue;
    const int ny = (nrhs + rc - 1) / rc;
    // a wavefront per row tile, up to 8
    const int bs = 64 * std::min(8, std::max(1, np / 16));
    const int64_t items = int64_t(max_ports) * rc;
    auto kern = items <= 2 * bs ? k_sweep_ppt<T, 2> : items <= 4 * bs ? k_sweep_ppt<T, 4> : k_sweep_ppt<T, 0>;
    if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(unsigned(S) * unsigned(ny)), dim3(bs), lds, st, ny, rc,
                       rc > 1 ? 0xffffffffu / unsigned(rc) + 1u : 0u, nrhs, Nt, ntofs, pn_off,
                       pn_pfirst, port_off, port_twin, pc, pbeta, pgamma, h, a_cur, a_next, np, rows, reverse);
    return hipGetLastError();
}

#define VTM_PPT(T)                                                                                                   \
    template hipError_t launch_port_node_tiles<T>(int, const int32_t*, const int64_t*, const int32_t*,              \
                                                  const int32_t*, const T*, const int64_t*, T*, bool, hipStream_t); \
    template hipError_t launch_sweep_ppt<T>(int, int, int, int, size_t, const T*, const int64_t*, const int32_t*,   \
                                            const int32_t*, const int32_t*, const int32_t*, const T*, const T*,     \
                                            const T*, const T*, const T*, T*, int, hipStream_t);
VTM_PPT(double)
VTM_PPT(float)
#undef VTM_PPT

}  // namespace vtm
