// Dense k-qubit gate (k = 3, 4, 5) on the matrix cores: a batched GEMM.
//
// For every group of 2^k amplitudes that differ only in the gate's qubits
// (Sec. 2.2), y = U x.  Written in real arithmetic on interleaved (re, im)
// vectors, y_r = M_r x_r with the 2^(k+1) x 2^(k+1) real matrix
//   M_r[2r][2c] = Re U[r][c],  M_r[2r][2c+1] = -Im U[r][c],
//   M_r[2r+1][2c] = Im U[r][c], M_r[2r+1][2c+1] = Re U[r][c],
// so a wave computes Y = M_r X for 16 groups at once (X: 2^(k+1) x 16) with
// 16x16x4 MFMA steps: complex64 states on FP32 MFMA, complex128 on FP64 MFMA.
//
// Operand layout of the 16x16x4 MFMA (one block): lane l = j + 16 q holds
// A[j][q] and B[q][j] of each k-step.  Accumulator v of lane l holds
// D[4q + v][j] for the FP32 instruction and D[4v + q][j] for the FP64 one
// (output groups of 4 rows vs 1 row per lane block).  Every lane keeps its
// slice of M_r in registers for the whole launch.
//
// M_r's columns are taken in the order that lets a lane load a whole
// amplitude: k-steps 2i and 2i + 1 take the real and the imaginary parts of
// amplitudes 4i .. 4i + 3, one to each lane block.  Its rows are taken so
// that a lane's four accumulators are two whole amplitudes (FP32: as they
// come; FP64: v = 0, 1 and v = 2, 3), so neither side exchanges lanes.
//
// Bound: the state's read and write (at k = 5 in complex64 the products take
// 0.46 of the 0.8 ms that a copy of 2^28 amplitudes takes, and run under it).
// With a load of one part a lane (half the bytes an instruction, twice the
// instructions) k = 5 in complex64 took 1.045 ms at 28 qubits, now 0.910 ms
// (4.7 TB/s).  The grid of 8192 workgroups at the compiler's three waves a
// SIMD is the measured best: four waves, a workgroup a batch and no prefetch
// all lose 11 to 30%.
#include "device.hpp"

namespace qs {

namespace {

constexpr int kMfmaThreads = 256;

template <typename R> struct Mfma;
template <> struct Mfma<float> {
    static constexpr bool kRowsPerLaneContiguous = true;   // D[4q + v][j]
    typedef float acc_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};
template <> struct Mfma<double> {
    static constexpr bool kRowsPerLaneContiguous = false;  // D[4v + q][j]
    typedef double acc_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};

template <typename R, int K>
__global__ __launch_bounds__(kMfmaThreads) void k_dense_mfma(c2_t<R> *__restrict__ a, const R *__restrict__ mr,
                                                             uint64_t nbatches, GateDesc g)
{
    using V = c2_t<R>;
    using acc_t = typename Mfma<R>::acc_t;
    constexpr int D = 2 << K;   // real dimension
    constexpr int T = D / 16;   // 16-row output tiles
    constexpr int S = D / 4;    // k-steps of 4
    const uint32_t lane = threadIdx.x & 63, j = lane & 15, q = lane >> 4;

    R areg[T][S];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        // real row of M_r behind row j of tile t
        const uint32_t row = Mfma<R>::kRowsPerLaneContiguous
                                 ? 16 * t + j
                                 : 16 * t + 8 * (j >> 3) + 2 * (j & 3) + ((j >> 2) & 1);
#pragma unroll
        for (int s = 0; s < S; ++s) areg[t][s] = mr[row * D + 2 * (4 * (s / 2) + q) + (s & 1)];
    }

    // amplitude offset of matrix index c (bit t of c <-> qubit q[t])
    auto off = [&](int c) {
        uint64_t o = 0;
#pragma unroll
        for (int t = 0; t < K; ++t)
            if ((c >> t) & 1) o |= 1ull << g.q[t];
        return o;
    };
    // amplitudes 4i + q as they are loaded: a wave-uniform offset plus the
    // lane's bits for q (gate qubits 0 and 1)
    const uint64_t lane_in = off((int)q);
    // output amplitudes of this lane, two per tile
    uint64_t out_off[T][2];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (Mfma<R>::kRowsPerLaneContiguous) {
            out_off[t][0] = off(8 * t + 2 * (int)q);
            out_off[t][1] = off(8 * t + 2 * (int)q + 1);
        } else {
            out_off[t][0] = off(8 * t + (int)q);
            out_off[t][1] = off(8 * t + 4 + (int)q);
        }
    }

    constexpr int L = S / 2;  // amplitudes a lane loads
    auto load_b = [&](uint64_t bb, V *bv) {
        const V *p = a + (insert_zeros<K>(bb * 16 + j, g.sorted) | lane_in);
#pragma unroll
        for (int i = 0; i < L; ++i) bv[i] = p[off(4 * i)];
    };
    const uint64_t wave = ((uint64_t)blockIdx.x * kMfmaThreads + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * kMfmaThreads) >> 6;
    V bv[L], bn[L];
    if (wave < nbatches) load_b(wave, bv);
    for (uint64_t b = wave; b < nbatches; b += nwaves) {
        // the next batch's operands are loaded while this batch's products run
        if (b + nwaves < nbatches) load_b(b + nwaves, bn);
        const uint64_t base = insert_zeros<K>(b * 16 + j, g.sorted);
        acc_t acc[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            acc[t] = acc_t{R(0), R(0), R(0), R(0)};
#pragma unroll
            for (int i = 0; i < L; ++i) {
                acc[t] = Mfma<R>::mma(areg[t][2 * i], bv[i].x, acc[t]);
                acc[t] = Mfma<R>::mma(areg[t][2 * i + 1], bv[i].y, acc[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                V y;
                y.x = acc[t][2 * h];
                y.y = acc[t][2 * h + 1];
                a[base | out_off[t][h]] = y;
            }
#pragma unroll
        for (int i = 0; i < L; ++i) bv[i] = bn[i];
    }
}

}  // namespace

template <typename R>
hipError_t launch_dense_mfma(void *state, int n, const GateDesc &g, const void *mat, hipStream_t s)
{
    const int k = (int)g.k;
    if (k < 3 || k > 5 || n < k + 4) return hipErrorInvalidValue;
    const uint64_t nbatches = 1ull << (n - k - 4);
    const uint64_t waves_per_block = kMfmaThreads / 64;
    uint64_t blocks = (nbatches + waves_per_block - 1) / waves_per_block;
    if (blocks > 8192) blocks = 8192;
    auto *a = (c2_t<R> *)state;
    auto *m = (const R *)mat;
    if (k == 3) k_dense_mfma<R, 3><<<(uint32_t)blocks, kMfmaThreads, 0, s>>>(a, m, nbatches, g);
    else if (k == 4) k_dense_mfma<R, 4><<<(uint32_t)blocks, kMfmaThreads, 0, s>>>(a, m, nbatches, g);
    else k_dense_mfma<R, 5><<<(uint32_t)blocks, kMfmaThreads, 0, s>>>(a, m, nbatches, g);
    return hipGetLastError();
}

template hipError_t launch_dense_mfma<float>(void *, int, const GateDesc &, const void *, hipStream_t);
template hipError_t launch_dense_mfma<double>(void *, int, const GateDesc &, const void *, hipStream_t);

}  // namespace qs
