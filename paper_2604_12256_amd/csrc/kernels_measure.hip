// Measurement on the state vector: the projective model in which the
// operator M_i^j keeps the amplitudes whose qubit j is i (the paper's
// measurement background, Sec. 2).  Three operations:
//
// * collapse of one qubit to an outcome, renormalised (one pass);
// * shot sampling by the inverse of the cumulative distribution in logical
//   index order, for caller-supplied uniforms (a marginal over the top
//   logical qubits picks the block, then one workgroup per needed block
//   scans it);
// * expectation values of Z strings, <psi| Z_S |psi> = sum_x |a_x|^2 (-1)^|x & S|.
//
// Every sum is FP64 in a fixed order, so results are deterministic.
#include <algorithm>

#include "device.hpp"

namespace qs {

namespace {

constexpr int kBlock = 256;

template <typename R>
__global__ __launch_bounds__(kBlock) void k_collapse(c2_t<R> *__restrict__ a, uint64_t len, uint64_t bit,
                                                     uint64_t want, R scale)
{
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t x = (uint64_t)blockIdx.x * kBlock + threadIdx.x; x < len; x += stride) {
        c2_t<R> v;
        if ((x & bit) == want) {
            v = a[x];
            v.x *= scale;
            v.y *= scale;
        } else {
            v.x = (R)0;
            v.y = (R)0;
        }
        a[x] = v;
    }
}

// One workgroup per needed block of 2^nlow consecutive logical indices.
// Thread t owns the segment [t 2^seg, (t+1) 2^seg) of the block; segment
// sums and their prefix are formed in a fixed order, then every shot of the
// block finds its segment by bisection and its index by a sequential scan.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_sample(const c2_t<R> *__restrict__ a, SampleArgs S,
                                                   const uint64_t *__restrict__ tabs,
                                                   const uint64_t *__restrict__ bases,
                                                   const uint64_t *__restrict__ ids,
                                                   const uint32_t *__restrict__ start,
                                                   const double *__restrict__ resid, uint64_t *__restrict__ out)
{
    __shared__ uint64_t tl[512], th[512];
    __shared__ double P[kBlock];
    for (int i = threadIdx.x; i < 512; i += kBlock) {
        tl[i] = tabs[i];
        th[i] = tabs[512 + i];
    }
    __syncthreads();
    const uint32_t bi = blockIdx.x;
    const uint64_t base = bases[bi];
    const uint32_t t = threadIdx.x;
    const uint64_t L = 1ull << S.seg_log2;
    auto prob = [&](uint64_t w) {
        const c2_t<R> v = a[base | tl[w & 511] | th[w >> 9]];
        const double re = (double)v.x, im = (double)v.y;
        return re * re + im * im;
    };
    double s = 0.0;
    if (t < S.nthr)
        for (uint64_t k = 0; k < L; ++k) s += prob(((uint64_t)t << S.seg_log2) + k);
    P[t] = s;
    __syncthreads();
    if (t == 0) {
        double acc = 0.0;
        for (int i = 0; i < S.nthr; ++i) {
            acc += P[i];
            P[i] = acc;
        }
    }
    __syncthreads();
    const int nthr = S.nthr;
    for (uint32_t j = start[bi] + t; j < start[bi + 1]; j += kBlock) {
        double r = resid[j];
        int seg;
        if (!(r < P[nthr - 1])) {
            // rounding put the target past this block's own total: take the
            // last segment with mass, and in it the last amplitude with mass
            seg = nthr - 1;
            while (seg > 0 && !(P[seg] > P[seg - 1])) --seg;
            r = P[seg];
        } else {
            int lo = 0, hi = nthr - 1;  // smallest i with P[i] > r
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (P[mid] > r) hi = mid;
                else lo = mid + 1;
            }
            seg = lo;
        }
        double acc = seg ? P[seg - 1] : 0.0;
        const uint64_t w0 = (uint64_t)seg << S.seg_log2;
        uint64_t pick = w0, last_pos = w0;
        bool found = false;
        for (uint64_t k = 0; k < L; ++k) {
            const double p = prob(w0 + k);
            if (p > 0.0) last_pos = w0 + k;
            acc += p;
            if (acc > r) {
                pick = w0 + k;
                found = true;
                break;
            }
        }
        if (!found) pick = last_pos;
        out[j] = (ids[bi] << S.nlow) | pick;
    }
}

template <typename V> __device__ __forceinline__ double mass_of(V v)
{
    const double re = (double)v.x, im = (double)v.y;
    return re * re + im * im;
}

// <psi| Z_S |psi> for many masks S at once.  The sums over x of
// |a_x|^2 (-1)^popcount(x & S) are entries of the Walsh-Hadamard transform of
// the probabilities.  A workgroup transforms tiles of 2^12 consecutive ones
// (12 additions an amplitude, whatever the number of masks); a mask then
// takes one entry of each tile, the one its low 12 bits name, with the sign
// its other bits give the tile.
//
// Bound: one read of the state.  Adding every amplitude to every mask's sum
// (two FP64 operations a mask) was VALU-bound from 8 masks on and took a pass
// for 16 of them.  Measured: 24 masks on 2^28 complex64 amplitudes 0.37 ms
// (1.88 ms before), 300 masks on 2^25 complex128 ones 0.14 ms (3.1 ms).
//
// The tile lies in registers 16 to a thread: bits 8..11 of the index as
// loaded, then 4..7, then 0..3, with an exchange through LDS before each of
// the last two (one slot of padding in 16 keeps the three access patterns off
// each other's banks).
constexpr uint32_t kZBlocks = 1024;
constexpr int kZTileBits = 12;
static_assert((1 << kZTileBits) == kBlock * 16, "16 amplitudes a thread");
constexpr int kZPerThread = (kZMasksPerLaunch + kBlock - 1) / kBlock;

__device__ __forceinline__ uint32_t z_slot(uint32_t x) { return x + (x >> 4); }

__device__ __forceinline__ void walsh16(double *v)
{
#pragma unroll
    for (int h = 1; h < 16; h <<= 1)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (!(j & h)) {
                const double a = v[j], b = v[j | h];
                v[j] = a + b;
                v[j | h] = a - b;
            }
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_expect_z_partial(const c2_t<R> *__restrict__ a, uint64_t len, ZArgs Z,
                                                             double *__restrict__ part)
{
    __shared__ double sh[(1 << kZTileBits) + (1 << (kZTileBits - 4))];
    const uint32_t t = threadIdx.x;
    double acc[kZPerThread];
    uint64_t m[kZPerThread];
#pragma unroll
    for (int k = 0; k < kZPerThread; ++k) {
        const int i = (int)t + k * kBlock;
        acc[k] = 0.0;
        m[k] = i < Z.nm ? Z.m[i] : 0;
    }
    const uint64_t ntiles = (len + (1u << kZTileBits) - 1) >> kZTileBits;
    c2_t<R> w[16];
    auto load = [&](uint64_t x0) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const uint64_t x = x0 + t + (uint32_t)(j * kBlock);
            if (x < len) w[j] = a[x];  // states below 2^12 amplitudes fill part of one tile
            else w[j].x = w[j].y = (R)0;
        }
    };
    load((uint64_t)blockIdx.x << kZTileBits);
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {  // uniform across the workgroup
        const uint64_t x0 = tile << kZTileBits;
        double v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = mass_of(w[j]);
        // the next tile's loads run while this one is transformed
        if (tile + gridDim.x < ntiles) load((tile + gridDim.x) << kZTileBits);
        walsh16(v);
        __syncthreads();  // the last tile's entries have been read
#pragma unroll
        for (int j = 0; j < 16; ++j) sh[z_slot(t + (uint32_t)(j * kBlock))] = v[j];
        __syncthreads();
        const uint32_t mid = (t & 15u) | ((t >> 4) << 8);
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = sh[z_slot(mid + (uint32_t)(j * 16))];
        walsh16(v);
#pragma unroll
        for (int j = 0; j < 16; ++j) sh[z_slot(mid + (uint32_t)(j * 16))] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = sh[z_slot(t * 16 + (uint32_t)j)];
        walsh16(v);
#pragma unroll
        for (int j = 0; j < 16; ++j) sh[z_slot(t * 16 + (uint32_t)j)] = v[j];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kZPerThread; ++k)
            if ((int)t + k * kBlock < Z.nm) {
                const double e = sh[z_slot((uint32_t)m[k] & ((1u << kZTileBits) - 1))];
                acc[k] += (__popcll(x0 & m[k]) & 1) ? -e : e;
            }
    }
#pragma unroll
    for (int k = 0; k < kZPerThread; ++k)
        if ((int)t + k * kBlock < Z.nm) part[(uint64_t)blockIdx.x * Z.nm + t + (uint32_t)(k * kBlock)] = acc[k];
}

// One workgroup per mask: fixed strided sums over the partials, then a
// fixed tree.
__global__ __launch_bounds__(kBlock) void k_expect_z_final(const double *__restrict__ part, uint32_t nblocks,
                                                           int nm, double *__restrict__ out)
{
    __shared__ double sh[kBlock];
    const int k = blockIdx.x;
    double acc = 0.0;
    for (uint32_t b = threadIdx.x; b < nblocks; b += kBlock) acc += part[(uint64_t)b * nm + k];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kBlock / 2; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[k] = sh[0];
}

uint32_t grid_for(uint64_t len)
{
    uint64_t b = (len + kBlock - 1) / kBlock;
    if (b > (1ull << 20)) b = 1ull << 20;
    return (uint32_t)(b ? b : 1);
}

}  // namespace

template <typename R>
hipError_t launch_collapse(void *state, int n, int phys_qubit, int outcome, double scale, hipStream_t s)
{
    if (phys_qubit < 0 || phys_qubit >= n || (outcome != 0 && outcome != 1)) return hipErrorInvalidValue;
    const uint64_t len = 1ull << n, bit = 1ull << phys_qubit;
    k_collapse<R><<<grid_for(len), kBlock, 0, s>>>((c2_t<R> *)state, len, bit, outcome ? bit : 0ull, (R)scale);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_sample(const void *state, const SampleArgs &S, uint32_t nblocks, const uint64_t *tabs,
                         const uint64_t *bases, const uint64_t *ids, const uint32_t *start, const double *resid,
                         uint64_t *out, hipStream_t s)
{
    if (nblocks == 0) return hipSuccess;
    if (S.nlow < 0 || S.nlow > 18 || S.nthr < 1 || S.nthr > kBlock || S.seg_log2 < 0 ||
        ((uint64_t)S.nthr << S.seg_log2) != (1ull << S.nlow))
        return hipErrorInvalidValue;
    k_sample<R><<<nblocks, kBlock, 0, s>>>((const c2_t<R> *)state, S, tabs, bases, ids, start, resid, out);
    return hipGetLastError();
}

size_t expect_z_scratch_bytes(uint32_t n_masks)
{
    return (size_t)kZBlocks * std::min<uint32_t>(n_masks, kZMasksPerLaunch) * sizeof(double);
}

template <typename R>
hipError_t launch_expect_z(const void *state, int n, const ZArgs &Z, double *out, double *scratch, hipStream_t s)
{
    if (Z.nm < 1 || Z.nm > kZMasksPerLaunch) return hipErrorInvalidValue;
    const uint64_t len = 1ull << n;
    // four workgroups a CU (LDS) keep 256 KiB of loads in flight on each
    const uint32_t nb = (uint32_t)std::min<uint64_t>(kZBlocks, (len + (1u << kZTileBits) - 1) >> kZTileBits);
    k_expect_z_partial<R><<<nb, kBlock, 0, s>>>((const c2_t<R> *)state, len, Z, scratch);
    k_expect_z_final<<<Z.nm, kBlock, 0, s>>>(scratch, nb, Z.nm, out);
    return hipGetLastError();
}

#define QS_INSTANTIATE_MEASURE(R)                                                                          \
    template hipError_t launch_collapse<R>(void *, int, int, int, double, hipStream_t);                  \
    template hipError_t launch_sample<R>(const void *, const SampleArgs &, uint32_t, const uint64_t *,    \
                                         const uint64_t *, const uint64_t *, const uint32_t *,            \
                                         const double *, uint64_t *, hipStream_t);                       \
    template hipError_t launch_expect_z<R>(const void *, int, const ZArgs &, double *, double *, hipStream_t);
QS_INSTANTIATE_MEASURE(double)
QS_INSTANTIATE_MEASURE(float)

}  // namespace qs
