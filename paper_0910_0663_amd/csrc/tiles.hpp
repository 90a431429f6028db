// MFMA operand-tile layout of the per-sub-circuit inverses (batched sweep).
//
// An n x n inverse is cut into A-operand tiles of 16 rows: BF16 tiles are 16 x 32
// (v_mfma_f32_16x16x32_bf16), FP64 tiles are 16 x 8 (two v_mfma_f64_16x16x4f64
// steps).  It is zero-padded to whole tiles, tile_rows(n) x tile_cols(n), no
// further: padded to multiples of 32 both ways, uneven sub-circuits (8 to 24 nodes a
// side) carried 1.5 times the products of their ports.  Tile (mt, kt) is stored
// at ((mt * (tile_cols / K) + kt) * 64 + lane) * E + j, lane-major, E = 16 bytes of
// elements per lane, so one 16-byte load per lane fetches a whole operand:
//   BF16: lane l holds A[16 mt + l%16][32 kt + 8 (l/16) + j], j < 8
//   FP64: lane l holds A[16 mt + l%16][8 kt + l/16] (j = 0) and
//         A[16 mt + l%16][8 kt + 4 + l/16] (j = 1)
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace vtm {

// the bound of a sub-circuit's padded size in either element type (LDS limits)
__host__ __device__ inline int tile_pad(int n) { return (n + 31) & ~31; }
__host__ __device__ inline int tile_rows(int n) { return (n + 15) & ~15; }

template <typename T>
struct MfmaTypes;
template <>
struct MfmaTypes<__bf16> {
    using TV = float;           // vectors and waves of the BF16 path
    using TB = __bf16;          // its right-hand side (the staged operand is BF16)
    static constexpr int K = 32;
    static constexpr int E = 8;
};
template <>
struct MfmaTypes<double> {
    using TV = double;
    using TB = double;
    static constexpr int K = 8;
    static constexpr int E = 2;
};

template <typename T>
__host__ __device__ inline int tile_cols(int n) {
    constexpr int K = MfmaTypes<T>::K;
    return (n + K - 1) / K * K;
}
// elements of a tiled n x n block
template <typename T>
__host__ __device__ inline int64_t tile_elems(int n) {
    return int64_t(tile_rows(n)) * tile_cols<T>(n);
}

// LDS bytes for the staged right-hand-side block (np = tile_cols rows, rc columns)
template <typename T>
__host__ __device__ inline size_t tile_lds_bytes(int np, int rc) {
    if constexpr (sizeof(T) == 2)
        return size_t(rc) * (np + 8) * sizeof(T);   // [n][k], row stride np + 8
    else
        return size_t(np) * rc * sizeof(T);         // [k][n]
}

// Batched port-to-port sweep: the BF16 path also stages h (FP32, row stride rc + 16,
// so that the epilogue's four 16-lane row groups fall in disjoint LDS banks) when
// the operator leaves room for it; the FP64 path stages the waves unpadded.

// row stride of the staged incident waves of the batched port-to-port sweep
template <typename T>
__host__ __device__ inline int pp_stage_stride(int qp, int rc) {
    if constexpr (sizeof(T) == 2)
        return qp + 8;                         // [n][k]
    else
        return rc;                             // [k][n]
}

// LDS bytes of the batched port-to-port sweep: staged waves, then (BF16, when
// with_h) h
template <typename T>
__host__ __device__ inline size_t pp_lds_bytes(int qp, int rc, bool with_h = true) {
    if constexpr (sizeof(T) == 2)
        return size_t(rc) * (qp + 8) * sizeof(T) +
               (with_h ? size_t(qp) * (rc + 16) * sizeof(float) : 0);
    else
        return size_t(qp) * rc * sizeof(T);
}

// (r, c) of the d-th stored element of a block of np padded columns
template <typename T>
__host__ __device__ inline void tile_rc(int np, int64_t d, int& r, int& c) {
    constexpr int K = MfmaTypes<T>::K, E = MfmaTypes<T>::E;
    const int j = int(d % E);
    const int lane = int((d / E) % 64);
    const int64_t tile = d / (64 * E);
    const int kt_n = np / K;
    const int mt = int(tile / kt_n), kt = int(tile % kt_n);
    const int m = lane % 16, q = lane / 16;
    r = mt * 16 + m;
    if constexpr (sizeof(T) == 2)
        c = kt * 32 + 8 * q + j;
    else
        c = kt * 8 + 4 * j + q;
}

// Port-node operators of the several-right-hand-side sweep (FP64 and FP32): k x k
// entries zero-padded to np = roundup(k, 16), cut into tiles of 16 rows by
// K = 64 / sizeof(T) columns, lane-major with 16 bytes per lane, E = K / 4 entries:
// lane l holds A[16 mt + l % 16][K kt + 4 j + l / 16], j < E, the A operands of E
// steps of a 16 x 16 x 4 MFMA.  Tile (mt, kt) starts at (mt (np / K) + kt) 64 E.
__host__ __device__ inline int node_tile_pad(int k) { return (k + 15) & ~15; }

template <typename T>
__host__ __device__ inline void node_tile_rc(int np, int64_t d, int& r, int& c) {
    constexpr int K = 64 / int(sizeof(T)), E = K / 4;
    const int j = int(d % E), lane = int((d / E) % 64);
    const int64_t tile = d / (64 * E);
    const int kt_n = np / K;
    r = int(tile / kt_n) * 16 + lane % 16;
    c = int(tile % kt_n) * K + 4 * j + lane / 16;
}

// LDS bytes of that sweep with rc right-hand sides per workgroup: T (np rows), the
// staged c a (q rows, then Z), each port's node and each node's first port
template <typename T>
__host__ __device__ inline size_t ppt_lds_bytes(int np, int q, int rc) {
    return size_t(np + (q > np ? q : np)) * rc * sizeof(T) + size_t(q + np + 1) * 4;
}

}  // namespace vtm
