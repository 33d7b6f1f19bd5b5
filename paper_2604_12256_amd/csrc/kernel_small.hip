// Small-state kernel: one workgroup runs a gate list on a state that fits in
// LDS (2^n amplitudes, n <= 13 for complex128 and n <= 14 for complex64 in
// 128 KiB).  Used for the merge booster's sub-states (Sec. 4.4:
// entanglement-free gate blocks simulated on small sub-state vectors) and for
// small circuits whose plan has no cache-blocked stage (one workgroup per
// circuit).  The starting state is read, or created as |0...0>, or formed as
// the tensor product of two finished sub-states (Alg. 7's merge), so a
// booster level is one launch: its initialisations and merges need none of
// their own.
//
// Bound: latency.  A sub-state of 2^4 to 2^8 amplitudes gives each lane one
// amplitude, and a gate is a few dependent LDS reads and a barrier.  With the
// gate records and matrices in global memory every gate also waited for two
// dependent misses (24 to 30 us for the 10 to 20 gates of a level); they are
// copied to LDS in blocks first, one wait for up to 64 gates.
#include <algorithm>

#include "device.hpp"

namespace qs {

namespace {

constexpr int kSmallThreads = 512;
constexpr uint32_t kSmallStateBytes = 128u * 1024u;
constexpr uint32_t kSmallLdsBytes = kSmallStateBytes + kSmallGateWords * 4 * kSmallBlockGates + kSmallBlockBytes;

__device__ __forceinline__ uint32_t gate_qubit(const uint32_t *rec, uint32_t t)
{
    return (rec[1 + (t >> 2)] >> (8 * (t & 3))) & 0xffu;
}

// One gate (record in LDS, table m in LDS or global memory) on the state s.
// Gates on one or two qubits update whole groups of 2^k amplitudes in place,
// one thread per group.  Wider dense gates are output-stationary: each thread
// owns the amplitudes i = tid + u * blockDim and computes them from the LDS
// state, all before any is written back, so that register use does not grow
// with 2^k.
template <typename R, typename MP>
__device__ __forceinline__ void apply_small(c2_t<R> *s, uint32_t len, const uint32_t *rec, MP m)
{
    using V = c2_t<R>;
    constexpr int kPer = (kSmallStateBytes / sizeof(V)) / kSmallThreads;  // 16 (c128) / 32 (c64)
    const uint32_t k = rec[0] & 0xffu;
    if (rec[0] >> 8) {  // diagonal
        for (uint32_t i = threadIdx.x; i < len; i += blockDim.x) {
            uint32_t y = 0;
            for (uint32_t t = 0; t < k; ++t) y |= ((i >> gate_qubit(rec, t)) & 1u) << t;
            s[i] = cmul(s[i], ldc<R>(m, y));
        }
        __syncthreads();
        return;
    }
    if (k == 1) {
        const uint32_t q = gate_qubit(rec, 0), bit = 1u << q;
        const V m00 = ldc<R>(m, 0), m01 = ldc<R>(m, 1), m10 = ldc<R>(m, 2), m11 = ldc<R>(m, 3);
        for (uint32_t g = threadIdx.x; g < (len >> 1); g += blockDim.x) {
            const uint32_t i = ((g >> q) << (q + 1)) | (g & (bit - 1));
            const V a = s[i], b = s[i | bit];
            V x = cmul(m00, a), y = cmul(m10, a);
            cmac(x, m01, b);
            cmac(y, m11, b);
            s[i] = x;
            s[i | bit] = y;
        }
        __syncthreads();
        return;
    }
    if (k == 2) {
        const uint32_t q0 = gate_qubit(rec, 0), q1 = gate_qubit(rec, 1);
        const uint32_t lo = min(q0, q1), hi = max(q0, q1);
        for (uint32_t g = threadIdx.x; g < (len >> 2); g += blockDim.x) {
            uint32_t i = ((g >> lo) << (lo + 1)) | (g & ((1u << lo) - 1));
            i = ((i >> hi) << (hi + 1)) | (i & ((1u << hi) - 1));
            const uint32_t at[4] = {i, i | (1u << q0), i | (1u << q1), i | (1u << q0) | (1u << q1)};
            V v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = s[at[c]];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                V acc = cmul(ldc<R>(m, 4 * r), v[0]);
#pragma unroll
                for (int c = 1; c < 4; ++c) cmac(acc, ldc<R>(m, 4 * r + c), v[c]);
                s[at[r]] = acc;
            }
        }
        __syncthreads();
        return;
    }
    uint32_t gmask = 0;
    for (uint32_t t = 0; t < k; ++t) gmask |= 1u << gate_qubit(rec, t);
    const uint32_t d = 1u << k;
    V out[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t i = threadIdx.x + (uint32_t)u * blockDim.x;
        if (i < len) {
            uint32_t r = 0;
            for (uint32_t t = 0; t < k; ++t) r |= ((i >> gate_qubit(rec, t)) & 1u) << t;
            const uint32_t base = i & ~gmask;
            V acc;
            acc.x = R(0);
            acc.y = R(0);
            for (uint32_t c = 0; c < d; ++c) {
                uint32_t o = base;
                for (uint32_t t = 0; t < k; ++t)
                    if ((c >> t) & 1u) o |= 1u << gate_qubit(rec, t);
                cmac(acc, ldc<R>(m, r * d + c), s[o]);
            }
            out[u] = acc;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t i = threadIdx.x + (uint32_t)u * blockDim.x;
        if (i < len) s[i] = out[u];
    }
    __syncthreads();
}

// state_bytes: LDS bytes reserved for the state of the launch's widest item;
// the records and the tables of the current block of gates follow it.
template <typename R>
__device__ __forceinline__ void run_small(const SmallItem &it, uint32_t state_bytes)
{
    using V = c2_t<R>;
    extern __shared__ char smem_raw[];
    V *s = reinterpret_cast<V *>(smem_raw);
    uint32_t *recs = reinterpret_cast<uint32_t *>(smem_raw + state_bytes);
    R *ltab = reinterpret_cast<R *>(smem_raw + state_bytes + kSmallGateWords * 4 * kSmallBlockGates);
    const uint32_t len = 1u << it.n;
    V *gstate = reinterpret_cast<V *>(it.state);
    const R *tables = reinterpret_cast<const R *>(it.tables);
    const V *klo = reinterpret_cast<const V *>(it.klo), *khi = reinterpret_cast<const V *>(it.khi);
    for (uint32_t i = threadIdx.x; i < len; i += blockDim.x) {
        V v;
        if (it.start == kSmallZero) {
            v.x = i == 0 ? R(1) : R(0);
            v.y = R(0);
        } else if (it.start == kSmallKron) {
            v = cmul(klo[i & ((1u << it.knlo) - 1)], khi[i >> it.knlo]);
        } else {
            v = gstate[i];
        }
        s[i] = v;
    }
    for (uint32_t g0 = 0; g0 < it.ngates;) {
        const SmallGate &head = it.gates[g0];
        const uint32_t ng = head.block_gates, first = head.table, entries = head.block_entries;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(it.gates + g0);
        for (uint32_t i = threadIdx.x; i < ng * kSmallGateWords; i += blockDim.x) recs[i] = src[i];
        const R *tsrc = tables + 2 * (uint64_t)first;
        for (uint32_t i = threadIdx.x; i < 2 * entries; i += blockDim.x) ltab[i] = tsrc[i];
        __syncthreads();
        for (uint32_t g = 0; g < ng; ++g) {
            const uint32_t *rec = recs + g * kSmallGateWords;
            if (entries) apply_small<R>(s, len, rec, (const R *)(ltab + 2 * (rec[7] - first)));
            else apply_small<R>(s, len, rec, tables + 2 * (uint64_t)rec[7]);
        }
        g0 += ng;
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < len; i += blockDim.x) gstate[i] = s[i];
}

template <typename R>
__global__ __launch_bounds__(kSmallThreads) void k_small(const SmallItem *__restrict__ items, uint32_t state_bytes)
{
    run_small<R>(items[blockIdx.x], state_bytes);
}

// Items addressed by pointer (kernel argument), one workgroup each, so that
// items of different contexts share a launch without a device list.
template <typename R>
__global__ __launch_bounds__(kSmallThreads) void k_small_ptrs(SmallPtrs P, uint32_t state_bytes)
{
    run_small<R>(*P.item[blockIdx.x], state_bytes);
}

}  // namespace

int small_max_qubits(bool c128) { return c128 ? 13 : 14; }

namespace {

// Launch shape of items of up to max_n qubits: one amplitude a lane up to 512
// of them (a single wave waits for no other at a barrier), the state's LDS
// bytes, and the block of gates behind it.
hipError_t small_shape(uint32_t amp_bytes, uint32_t max_n, uint32_t *threads, uint32_t *state_bytes, uint32_t *lds)
{
    if (max_n > 14 || (amp_bytes << max_n) > kSmallStateBytes) return hipErrorInvalidValue;
    *threads = std::min<uint32_t>(kSmallThreads, std::max<uint32_t>(64, 1u << max_n));
    *state_bytes = std::max(16u, amp_bytes << max_n);
    *lds = *state_bytes + (kSmallLdsBytes - kSmallStateBytes);
    return hipSuccess;
}

template <typename K> hipError_t small_lds_attr(K kernel, bool *done)
{
    if (*done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)kSmallLdsBytes);
    *done = e == hipSuccess;
    return e;
}

}  // namespace

template <typename R>
hipError_t launch_small_batch(const SmallItem *items_dev, uint32_t count, uint32_t max_n, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    uint32_t threads, bytes, lds;
    hipError_t e = small_shape((uint32_t)sizeof(c2_t<R>), max_n, &threads, &bytes, &lds);
    static bool attr_set = false;
    if (e == hipSuccess) e = small_lds_attr(k_small<R>, &attr_set);
    if (e != hipSuccess) return e;
    k_small<R><<<count, threads, lds, s>>>(items_dev, bytes);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_small_ptrs(const SmallPtrs &P, uint32_t count, uint32_t max_n, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    if (count > (uint32_t)kSmallBatchMax) return hipErrorInvalidValue;
    uint32_t threads, bytes, lds;
    hipError_t e = small_shape((uint32_t)sizeof(c2_t<R>), max_n, &threads, &bytes, &lds);
    static bool attr_set = false;
    if (e == hipSuccess) e = small_lds_attr(k_small_ptrs<R>, &attr_set);
    if (e != hipSuccess) return e;
    k_small_ptrs<R><<<count, threads, lds, s>>>(P, bytes);
    return hipGetLastError();
}

template hipError_t launch_small_batch<double>(const SmallItem *, uint32_t, uint32_t, hipStream_t);
template hipError_t launch_small_batch<float>(const SmallItem *, uint32_t, uint32_t, hipStream_t);
template hipError_t launch_small_ptrs<double>(const SmallPtrs &, uint32_t, uint32_t, hipStream_t);
template hipError_t launch_small_ptrs<float>(const SmallPtrs &, uint32_t, uint32_t, hipStream_t);

}  // namespace qs
