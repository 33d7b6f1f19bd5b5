// Measurement on the state vector: the projective model in which the
// operator M_i^j keeps the amplitudes whose qubit j is i (the paper's
// measurement background, Sec. 2).  Three operations:
//
// * collapse of one qubit to an outcome, renormalised (one pass);
// * shot sampling by the inverse of the cumulative distribution in logical
//   index order, for caller-supplied uniforms (a marginal over the top
//   logical qubits and its prefix sums pick the bin, then one wave per shot
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

// Shot sampling by the inverse of the cumulative distribution in logical
// index order, in three levels: groups of 2^kScanBits bins, bins of 2^nlow
// consecutive logical indices (a marginal over the top qubits), and the
// amplitudes of one bin.  k_sample_prefix forms the inclusive prefix sums of
// the bins inside each group, k_sample_groups those of the group totals, and
// k_sample gives every shot to one wave, which bisects both and scans its
// bin's amplitudes 64 at a time.  Nothing passes through the host between the
// uniforms and the indices.
//
// Bound: the bins' read of the state.  With 2^16 bins the second level
// read every touched bin whole (0.93 ms for 20,000 shots on a 27-qubit state
// stored bit-reversed, one cache line an amplitude), after a sort of the
// shots by bin on the host; bins of 64 amplitudes (up to 28 qubits) leave one
// load a shot: 0.65 ms in place of 4.0 ms for the whole call.
constexpr int kScanBits = kSampleScanBits;

// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ double wave_prefix(double v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
    }
    return v;
}

// Logical bin of a physical index.
__device__ __forceinline__ uint64_t bin_of(uint64_t x, const SampleArgs &S)
{
    if (S.ordered) return x >> S.nlow;
    uint64_t b = 0;
    for (int q = S.nlow; q < S.n; ++q) b |= ((x >> S.layout[q]) & 1ull) << (q - S.nlow);
    return b;
}

template <typename V> __device__ __forceinline__ double mass_of(V v)
{
    const double re = (double)v.x, im = (double)v.y;
    return re * re + im * im;
}

// Bin masses where the low logical qubits are the low physical ones: a bin is
// a run of 2^nlow amplitudes, 2^(nlow - 6) rows of 64.  A wave takes 16 rows
// (or the rows of one bin) with all their loads in flight; the sums over the
// lanes merge two rows a step, so 16 rows cost 17 exchanges instead of 96.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_bins_runs(const c2_t<R> *__restrict__ a, SampleArgs S,
                                                      double *__restrict__ bins)
{
    const uint32_t lane = threadIdx.x & 63;
    const int rbits = S.nlow - 6, tail = rbits < 4 ? rbits : 4;
    const uint32_t blocks = rbits > 4 ? 1u << (rbits - 4) : 1u;
    const uint64_t row0 = ((uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * (16ull * blocks);
    if (row0 >= (1ull << (S.n - 6))) return;
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = 0.0;
    for (uint32_t k = 0; k < blocks; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] += mass_of(nt_load(a + (((row0 + 16 * k + (uint32_t)i) << 6) | lane)));
    // lane bits 5..2 end as row bits 3..0
#pragma unroll
    for (int half = 8; half >= 1; half >>= 1) {
        const bool up = lane & (uint32_t)(4 * half);
#pragma unroll
        for (int i = 0; i < half; ++i) {
            const double mine = up ? v[i + half] : v[i], other = up ? v[i] : v[i + half];
            v[i] = mine + __shfl_xor(other, 4 * half, 64);
        }
    }
    double m = v[0];
    m += __shfl_xor(m, 2, 64);
    m += __shfl_xor(m, 1, 64);
    for (int b = 0; b < tail; ++b) m += __shfl_xor(m, 4 << b, 64);
    const uint32_t row = lane >> 2;
    if ((lane & 3u) == 0 && (row & ((1u << tail) - 1)) == 0) bins[bin_of((row0 + row) << 6, S)] = m;
}

// Bin masses in any layout: a wave reads rows of 64 amplitudes (the low six
// physical bits); the lanes' selected bits are part of the bin, the others
// are summed over by a butterfly.  High bits not in the bin index are walked
// by a masked add.  The rows of a wave's successive bins differ in the bits
// `run` (of the high selected bits), which hold the lowest bin bits, so that a
// lane's writes fill a line: 27 qubits in reversed order, complex128, 424 us
// (5.1 TB/s), 468 with neighbouring rows in the wave and each bin in a line of
// its own.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_bins(const c2_t<R> *__restrict__ a, SampleArgs S, uint64_t sel_high,
                                                 uint64_t run, uint64_t rest_high, uint32_t sel_lane,
                                                 uint32_t each, double *__restrict__ bins)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t nrows = 1ull << __popcll(sel_high), nz = 1ull << __popcll(rest_high);
    const uint64_t y0 = ((uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * each;
    if (y0 >= nrows) return;
    const uint64_t zstep = rest_high & (~rest_high + 1);
    const uint64_t outer = sel_high & ~run;
    const int nrun = __popcll(run);
    const bool mine = S.n >= 6 || lane < (1u << S.n);
    auto next_z = [&](uint64_t z) { return ((z | ~rest_high) + zstep) & rest_high; };
    for (uint64_t i = y0; i < y0 + each; ++i) {
        const uint64_t y = deposit(i & ((1ull << nrun) - 1), run) | deposit(i >> nrun, outer);
        double acc = 0.0;
        uint64_t z = 0;
        if (nz >= 8) {
            for (uint64_t j = 0; j < nz; j += 8) {
                c2_t<R> v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u, z = next_z(z)) v[u] = nt_load(a + (y | z | lane));
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += mass_of(v[u]);
            }
        } else if (mine) {
            for (uint64_t j = 0; j < nz; ++j, z = next_z(z)) acc += mass_of(a[y | z | lane]);
        }
#pragma unroll
        for (int b = 0; b < 6; ++b)
            if (!((sel_lane >> b) & 1u)) acc += __shfl_xor(acc, 1 << b, 64);
        if ((lane & ~sel_lane) == 0) bins[bin_of(y | lane, S)] = acc;
    }
}

// pre[i] = sum of the bins of i's group of 2^kScanBits up to and including i:
// 16 consecutive ones to a thread, then the threads' totals in order.  Every
// sum is the one before it plus one term, so a bin without mass repeats its
// predecessor's value exactly and no target falls on it.
__global__ __launch_bounds__(kBlock) void k_sample_prefix(const double *__restrict__ bins, uint64_t nbins,
                                                          double *__restrict__ pre)
{
    constexpr int kEach = (1 << kScanBits) / kBlock;
    __shared__ double sh[(1 << kScanBits) + kBlock], base[kBlock];
    const uint32_t t = threadIdx.x;
    const uint64_t i0 = (uint64_t)blockIdx.x << kScanBits;
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const uint32_t i = t + (uint32_t)(k * kBlock);
        sh[i + i / kEach] = i0 + i < nbins ? bins[i0 + i] : 0.0;
    }
    __syncthreads();
    double v[kEach], run = 0.0;
#pragma unroll
    for (int k = 0; k < kEach; ++k) v[k] = run += sh[t * (kEach + 1) + (uint32_t)k];
    base[t] = run;
    __syncthreads();
    if (t == 0) {
        double acc = 0.0;
#pragma unroll 16
        for (int w = 0; w < kBlock; ++w) {
            const double tot = base[w];
            base[w] = acc;
            acc += tot;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kEach; ++k) sh[t * (kEach + 1) + (uint32_t)k] = base[t] + v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const uint32_t i = t + (uint32_t)(k * kBlock);
        if (i0 + i < nbins) pre[i0 + i] = sh[i + i / kEach];
    }
}

// cum[g] = total of groups 0..g, added in order; one workgroup.
__global__ __launch_bounds__(kBlock) void k_sample_groups(const double *__restrict__ pre, uint64_t nbins, int ngroups,
                                                          double *__restrict__ cum)
{
    __shared__ double sh[kSampleGroupsMax];
    for (int g = threadIdx.x; g < ngroups; g += kBlock) {
        const uint64_t end = ((uint64_t)g + 1) << kScanBits;
        sh[g] = pre[(end < nbins ? end : nbins) - 1];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double acc = 0.0;
#pragma unroll 16
        for (int g = 0; g < ngroups; ++g) sh[g] = acc += sh[g];
    }
    __syncthreads();
    for (int g = threadIdx.x; g < ngroups; g += kBlock) cum[g] = sh[g];
}

// First i in [0, n) with c[i] > r; where rounding put r past the last, the
// last i that adds mass.
__device__ __forceinline__ uint64_t first_above(const double *__restrict__ c, uint64_t n, double r, bool *past)
{
    *past = !(c[n - 1] > r);
    if (*past) r = c[n - 1];
    uint64_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (*past ? c[mid] >= r : c[mid] > r) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_sample(const c2_t<R> *__restrict__ a, SampleArgs S,
                                                   const double *__restrict__ pre, const double *__restrict__ cum,
                                                   const double *__restrict__ u, uint64_t nshots,
                                                   uint64_t *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t nbins = 1ull << (S.n - S.nlow);
    const int ngroups = (int)((nbins + (1ull << kScanBits) - 1) >> kScanBits);
    const uint64_t nwaves = (uint64_t)gridDim.x * (kBlock / 64);
    uint64_t lane_phys = 0;
    for (int q = 0; q < 6 && q < S.nlow; ++q) lane_phys |= (uint64_t)((lane >> q) & 1u) << S.layout[q];
    const bool mine = S.nlow >= 6 || lane < (1u << S.nlow);
    for (uint64_t j = (uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); j < nshots; j += nwaves) {
        bool past, over;
        double r = u[j] * cum[ngroups - 1];
        const uint64_t g = first_above(cum, (uint64_t)ngroups, r, &over);
        r -= g ? cum[g - 1] : 0.0;
        const double *p = pre + (g << kScanBits);
        const uint64_t in_group = nbins - (g << kScanBits) < (1ull << kScanBits) ? nbins : 1ull << kScanBits;
        if (over) r = p[in_group - 1];
        const uint64_t b = first_above(p, in_group, r, &past);
        over |= past;
        r -= b ? p[b - 1] : 0.0;
        const uint64_t bin = (g << kScanBits) + b;
        uint64_t base = lane_phys;
        for (int q = S.nlow; q < S.n; ++q) base |= ((bin >> (q - S.nlow)) & 1ull) << S.layout[q];
        // the bin's amplitudes in logical order, 64 at a time; `last` is the
        // last one with mass, taken when rounding puts the target past all
        double run = 0.0;
        uint64_t pick = 0, last = 0;
        bool found = false;
        const uint32_t strips = S.nlow > 6 ? 1u << (S.nlow - 6) : 1u;
        for (uint32_t s = 0; s < strips && !found; ++s) {
            uint64_t x = base;
            for (int q = 6; q < S.nlow; ++q) x |= (uint64_t)((s >> (q - 6)) & 1u) << S.layout[q];
            double w = 0.0;
            if (mine) w = mass_of(a[x]);
            const double c = run + wave_prefix(w);
            const uint64_t mass = __ballot(w > 0.0), above = over ? 0 : __ballot(w > 0.0 && c > r);
            if (mass) last = ((uint64_t)s << 6) + (uint32_t)(63 - __clzll(mass));
            if (above) {
                pick = ((uint64_t)s << 6) + (uint32_t)__builtin_ctzll(above);
                found = true;
            }
            run = __shfl(c, 63, 64);
        }
        if (lane == 0) out[j] = (bin << S.nlow) | (found ? pick : last);
    }
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
            if (x < len) w[j] = nt_load(a + x);  // states below 2^12 amplitudes fill part of one tile
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
hipError_t launch_sample(const void *state, SampleArgs S, double *bins, double *pre, double *cum, const double *u,
                         uint64_t nshots, uint64_t *out, hipStream_t s)
{
    if (nshots == 0) return hipSuccess;
    if (S.n < 1 || S.n > 40 || S.nlow < 0 || S.nlow > S.n || S.n - S.nlow > kSampleBinBits) return hipErrorInvalidValue;
    const uint64_t all = (1ull << S.n) - 1;
    uint64_t low = 0, seen = 0;
    S.ordered = 1;
    for (int q = 0; q < S.n; ++q) {
        if (S.layout[q] < 0 || S.layout[q] >= S.n) return hipErrorInvalidValue;
        seen |= 1ull << S.layout[q];
        if (q < S.nlow) low |= 1ull << S.layout[q];
        else S.ordered &= S.layout[q] == q;
    }
    if (seen != all) return hipErrorInvalidValue;
    const auto *a = (const c2_t<R> *)state;
    constexpr uint64_t kWaves = kBlock / 64;
    if (S.nlow >= 6 && S.n >= 10 && S.n - S.nlow >= 4 && low == (1ull << S.nlow) - 1) {
        const uint64_t waves = (1ull << (S.n - 6)) / (16ull << std::max(0, S.nlow - 10));
        k_bins_runs<R><<<(uint32_t)((waves + kWaves - 1) / kWaves), kBlock, 0, s>>>(a, S, bins);
    } else {
        const uint64_t sel = all & ~low;
        const uint64_t rows = 1ull << __builtin_popcountll(sel & ~63ull);
        // a wave takes the rows of eight bins that follow each other, so that
        // its lanes' writes fill lines
        uint64_t run = 0;
        for (int q = S.nlow; q < S.n && q < S.nlow + 3; ++q)
            if (S.layout[q] >= 6) run |= 1ull << S.layout[q];
        const uint64_t nrun = 1ull << __builtin_popcountll(run);
        const uint32_t each = (uint32_t)std::max<uint64_t>(nrun, std::min<uint64_t>(64, rows >> 14));
        const uint64_t waves = rows / each;
        k_bins<R><<<(uint32_t)((waves + kWaves - 1) / kWaves), kBlock, 0, s>>>(a, S, sel & ~63ull, run, low & ~63ull,
                                                                               (uint32_t)(sel & 63u), each, bins);
    }
    const uint64_t nbins = 1ull << (S.n - S.nlow);
    const uint32_t ngroups = (uint32_t)sample_groups(S.n - S.nlow);
    k_sample_prefix<<<ngroups, kBlock, 0, s>>>(bins, nbins, pre);
    k_sample_groups<<<1, kBlock, 0, s>>>(pre, nbins, (int)ngroups, cum);
    const uint64_t wgs = std::min<uint64_t>((nshots + kWaves - 1) / kWaves, 1u << 16);
    k_sample<R><<<(uint32_t)wgs, kBlock, 0, s>>>(a, S, pre, cum, u, nshots, out);
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
    template hipError_t launch_sample<R>(const void *, SampleArgs, double *, double *, double *,          \
                                         const double *, uint64_t, uint64_t *, hipStream_t);              \
    template hipError_t launch_expect_z<R>(const void *, int, const ZArgs &, double *, double *, hipStream_t);
QS_INSTANTIATE_MEASURE(double)
QS_INSTANTIATE_MEASURE(float)

}  // namespace qs
