// Device-side helpers and the launch interface between the executor and the
// kernels.  gfx950 (CDNA4) only: 64-lane wavefronts.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

namespace qs {

// Read-only data every lane of a wave reads at the same address (gate
// matrices, stage programs) is addressed through the constant address space,
// so the compiler issues scalar loads for it.
#define QS_CONST __attribute__((address_space(4)))
template <typename T> __device__ __forceinline__ const QS_CONST T *as_const(const T *p)
{
    return (const QS_CONST T *)(p);
}

// Complex entry i of an interleaved (re, im) real array, in any address space.
template <typename R, typename P>
__device__ __forceinline__ auto ldc(P m, uint64_t i)
{
    using V = typename std::conditional<sizeof(R) == 8, double2, float2>::type;
    V v;
    v.x = m[2 * i];
    v.y = m[2 * i + 1];
    return v;
}

// Interleaved complex amplitude: double2 (complex128) or float2 (complex64).
template <typename R> struct C2;
template <> struct C2<double> { using T = double2; };
template <> struct C2<float> { using T = float2; };
template <typename R> using c2_t = typename C2<R>::T;

// Amplitudes that a kernel reads or writes once, in whole lines an instruction
// (double2, float2): not kept in the caches.  Rotation stages: a batch of 128
// circuits of 10 to 13 qubits 345 -> 265 us, 48 of 16 qubits 261 -> 255 us, 30
// qubits 1% less, 22 the same; general stages of 25 qubits 435 -> 409 us a
// pass; Z strings of 30 qubits 3.02 -> 2.57 ms (complex64 1.51 -> 1.36),
// marginals of high qubits 2.95 -> 2.75 (1.53 -> 1.36).  Not where instructions
// fill parts of lines: the matrix-core kernel takes 938 us for 909 (5 qubits,
// 28-qubit complex64 state) and 1137 for 885 (4 qubits) with it.
template <typename V> __device__ __forceinline__ V nt_load(const V *p)
{
    using E = decltype(V::x);
    typedef E vec_t __attribute__((ext_vector_type(2)));
    const vec_t t = __builtin_nontemporal_load(reinterpret_cast<const vec_t *>(p));
    V v;
    v.x = t[0];
    v.y = t[1];
    return v;
}
template <typename V> __device__ __forceinline__ void nt_store(V *p, V v)
{
    using E = decltype(V::x);
    typedef E vec_t __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(vec_t{v.x, v.y}, reinterpret_cast<vec_t *>(p));
}

template <typename V>
__device__ __forceinline__ V cmul(V a, V b)
{
    V r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}

// acc += m * a
template <typename V>
__device__ __forceinline__ void cmac(V &acc, V m, V a)
{
    acc.x = fma(m.x, a.x, acc.x);
    acc.x = fma(-m.y, a.y, acc.x);
    acc.y = fma(m.x, a.y, acc.y);
    acc.y = fma(m.y, a.x, acc.y);
}

// Quadratic-phase operator of the stage kernels: amplitude x is multiplied by
// e^{i phi(x)}, phi(x) = c + sum a_q x_q + sum b_qp x_q x_p over the buffer's
// qubits, formed in FP64 (also for complex64 states, whose amplitudes take
// one FP32 rounding per operator).  Its block of complex FP64
// unit factors (in the program words) holds, for the chunk's share, rows
// selected by the low and the high half of the chunk index: lane l < C forms
// B_l = e^{i beta_l} (the coefficient the chunk bits give local bit l) as the
// product of its two row entries, and a wave product over the other lanes
// forms the chunk bits' own factor E.  A thread starts from its table entry
// (constant and thread-bit terms) times E, takes in B of each set thread bit,
// and walks its 2^RB amplitudes in Gray-code order with a running product:
// flipping register bit b multiplies by G_b = e^{i(a_b + thread and chunk
// terms of b)} (or its conjugate) and by the pair factors with the register
// bits already set.  w: the operator's record.
template <typename R, int RB>
__device__ __forceinline__ void quad_op(c2_t<R> *amp, const uint32_t *w, const uint32_t *Pg, uint64_t chunk,
                                        uint32_t tid, int C, uint32_t rmask, uint32_t t0, uint32_t t1, uint32_t t2)
{
    using V = c2_t<double>;
    constexpr int NR = 1 << RB;
    const int h = (int)(w[5] & 0xffu), nhi = (int)((w[5] >> 8) & 0xffu);
    const int ncl = C + nhi + 1, nch = C + 1;
    const int lane = (int)(tid & 63u);
    const uint64_t glo = chunk & ((1ull << h) - 1), ghi = chunk >> h;
    const V *blk = reinterpret_cast<const V *>(Pg + w[3]);
    const V *tlo = blk + w[4] + glo * (uint64_t)ncl;
    const V *thi = blk + w[6] + ghi * (uint64_t)nch;
    const V one{1.0, 0.0};
    const V vlo = lane < ncl ? tlo[lane] : one;
    const V vhi = lane < nch ? thi[lane] : one;
    const V B = cmul(vlo, vhi);
    V p = one;
    if (lane >= C && lane < C + nhi && ((ghi >> (lane - C)) & 1ull)) p = vlo;
    if (lane == C + nhi) p = vlo;
    if (lane == C) p = cmul(p, vhi);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) p = cmul(p, V{__shfl_xor(p.x, off), __shfl_xor(p.y, off)});

    const int nt = C - RB;
    const V *row = blk + (size_t)tid * (1 + RB);
    const V *qm = blk + w[7];
    V F = cmul(row[0], p);
    for (int i = 0; i < nt; ++i) {
        const uint32_t t = i < 4 ? t0 : i < 8 ? t1 : t2;
        const int j = (int)((t >> (8 * (i & 3))) & 0xffu);
        const V f2 = cmul(F, V{__shfl(B.x, j), __shfl(B.y, j)});
        if ((tid >> i) & 1u) F = f2;
    }
    V G[RB];
    uint32_t rm = rmask;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int j = __builtin_ctz(rm);
        rm &= rm - 1u;
        G[b] = cmul(row[1 + b], V{__shfl(B.x, j), __shfl(B.y, j)});
    }
    V Q = F;
    amp[0] = cmul(amp[0], c2_t<R>{(R)Q.x, (R)Q.y});
#pragma unroll
    for (int k = 1; k < NR; ++k) {
        const int g = k ^ (k >> 1), b = __builtin_ctz(k), prev = g ^ (1 << b);
        const bool set = (g >> b) & 1;
        V f = set ? G[b] : V{G[b].x, -G[b].y};
#pragma unroll
        for (int b2 = 0; b2 < RB; ++b2) {
            if (b2 == b || !((prev >> b2) & 1)) continue;
            const int lo = b < b2 ? b : b2, hi = b < b2 ? b2 : b;
            const V q = qm[lo * (2 * RB - lo - 1) / 2 + (hi - lo - 1)];
            f = cmul(f, set ? q : V{q.x, -q.y});
        }
        Q = cmul(Q, f);
        amp[g] = cmul(amp[g], c2_t<R>{(R)Q.x, (R)Q.y});
    }
}

// Scatter the low bits of x to the set bit positions of mask (bit-deposit).
__device__ __forceinline__ uint64_t deposit(uint64_t x, uint64_t mask)
{
    uint64_t r = 0;
    while (mask) {
        const uint64_t low = mask & (~mask + 1);
        if (x & 1) r |= low;
        x >>= 1;
        mask &= mask - 1;
    }
    return r;
}

// Insert a zero bit at each of the ascending positions pos[0..k-1].
template <int K>
__device__ __forceinline__ uint64_t insert_zeros(uint64_t g, const int *pos)
{
#pragma unroll
    for (int t = 0; t < K; ++t) {
        const uint64_t lo = g & ((1ull << pos[t]) - 1);
        g = ((g >> pos[t]) << (pos[t] + 1)) | lo;
    }
    return g;
}

struct GateDesc {            // a full-pass gate
    uint32_t diag;           // 1: table is a 2^k diagonal (k <= 24); else a dense 2^k x 2^k matrix (k <= 6)
    uint32_t k;
    int32_t q[24];           // matrix bit t <-> qubit q[t]
    int32_t sorted[6];       // dense: q ascending
    uint64_t table;          // offset (complex entries) in the table arena
    uint32_t nctl;           // diagonal: control qubits, not in q (every entry off their values is 1)
    int32_t ctl[6];          // ascending
    uint64_t ctl_bits;       // their values, at their positions
};

// A gate of a small-state program.  The kernel copies records and tables to
// LDS in blocks of consecutive gates whose tables are consecutive in the
// arena; a block's first record says how many gates it holds and how many
// table entries to copy (0: the tables stay in global memory).
struct SmallGate {
    uint32_t kind;           // k | diagonal << 8 (2^k diagonal, k <= 24; else a dense matrix, k <= 6)
    uint32_t q[6];           // bytes: matrix bit t <-> qubit q[t]
    uint32_t table;          // offset (complex entries) in the table arena
    uint32_t block_gates, block_entries, pad[2];
};
constexpr uint32_t kSmallGateWords = 12, kSmallBlockGates = 64, kSmallBlockBytes = 16u * 1024u;
static_assert(sizeof(SmallGate) == 4 * kSmallGateWords, "record size");

enum : uint32_t { kSmallLoad = 0, kSmallZero = 1, kSmallKron = 2 };
struct SmallItem {           // one gate list on one small state
    void *state;             // buffer holding 2^n amplitudes
    const SmallGate *gates;  // device program
    const void *tables;      // device table arena (same dtype as the state)
    const void *klo, *khi;   // start == kSmallKron: amplitude x = klo[x mod 2^knlo] * khi[x >> knlo]
    uint32_t n, ngates;
    uint32_t start;          // kSmallLoad: read the buffer; kSmallZero: |0...0>; kSmallKron
    uint32_t knlo;
};

constexpr int kSmallBatchMax = 448;  // 3.5 KiB of kernel arguments
struct SmallPtrs {           // kernel-argument list of items for one batched launch
    const SmallItem *item[kSmallBatchMax];
};

// ---- launchers (return hipError_t of the launch) ---------------------------
template <typename R> hipError_t launch_init(void *state, int n, hipStream_t s);
template <typename R> hipError_t launch_dense(void *state, int n, const GateDesc &g, const void *mat, hipStream_t s);
template <typename R> hipError_t launch_dense_mfma(void *state, int n, const GateDesc &g, const void *mat, hipStream_t s);
template <typename R> hipError_t launch_diag(void *state, int n, const GateDesc &g, const void *table, hipStream_t s);
template <typename R> hipError_t launch_kron(void *dst, const void *lo, int nlo, const void *hi, int nhi, hipStream_t s);
// in-place exchange of physical bits lo[k] <-> hi[k] (lo < 6 <= hi)
template <typename R> hipError_t launch_swap_bits(void *state, int n, const int *lo, const int *hi, int npairs,
                                                  hipStream_t s);
template <typename RA, typename RB> hipError_t launch_inner_perm(const void *a, const void *b, int n, const int *map,
                                                                 double *out, double *scratch, hipStream_t s);
template <typename R> hipError_t launch_gather(const void *state, const uint64_t *idx, uint64_t m, double *out, hipStream_t s);
// marginal over the physical qubits q[0..nq): out[2^nq] doubles (device), scratch as sized by marginal_scratch_bytes
template <typename R> hipError_t launch_marginal(const void *state, int n, const int *q, int nq, double *out,
                                                 double *scratch, hipStream_t s);
size_t marginal_scratch_bytes(int n, const int *q, int nq);  // q ascending, as passed to launch_marginal
// out[y] = in[b(y)], bit t of y at bit where[t] of b (device arrays of 2^nq doubles)
hipError_t launch_permute_bins(const double *in, double *out, int nq, const int *where, hipStream_t s);
template <typename RA, typename RB> hipError_t launch_inner(const void *a, const void *b, int n, double *out,
                                                            double *scratch, hipStream_t s);
size_t inner_scratch_bytes(int n);
template <typename R> hipError_t launch_small_batch(const SmallItem *items_dev, uint32_t count, uint32_t max_n,
                                                    hipStream_t s);
template <typename R> hipError_t launch_small_ptrs(const SmallPtrs &P, uint32_t count, uint32_t max_n,
                                                   hipStream_t s);
int small_max_qubits(bool c128);

// Stage kernel: program built by the executor (see kernel_stage.hip).
// LDS slot swizzle of the stage kernel's transpose buffer (linear over XOR):
// 16-byte slots (complex128) fold local-index bits 4..15 into bits 0..3,
// 8-byte slots (complex64) fold bits 5..14 into bits 0..4, so that local bit
// l lands on slot bit l mod 4 (resp. l mod 5).  The host writes the
// swizzled byte offsets of each register set into the stage program.
__host__ __device__ inline uint32_t stage_swizzle(uint32_t i, bool c64)
{
    return c64 ? i ^ (((i >> 5) ^ (i >> 10)) & 31u) : i ^ (((i >> 4) ^ (i >> 8) ^ (i >> 12)) & 15u);
}
constexpr int kStageHeaderWords = 160;   // program header incl. neutral offsets at [128, 128 + 2^RB)
constexpr int kStagePhaseWords = 16;     // phase header before its register offsets

struct StageLaunch {
    void *state;
    const uint32_t *prog;    // device program words
    const void *tables;      // device table arena
    int n, C, nphases;
    uint64_t nchunks;
    uint64_t xbits = 0;      // bits OR-ed into the wave-uniform base for selectors only (the
                             // outer qubits of a host-memory offload window, at bits >= n)
    // tensor product formed on load: when kron_lo is set, the chunk is read as
    // kron_lo[x mod 2^kron_nlo] * kron_hi[x >> kron_nlo] instead of state[x]
    const void *kron_lo = nullptr, *kron_hi = nullptr;
    int kron_nlo = 0;
    // the program holds quadratic-phase operators: launched on the kernel
    // variant that has them (the others keep the register allocation of the
    // kernel without)
    bool quad = false;
};
template <typename R> hipError_t launch_stage(const StageLaunch &L, hipStream_t s);

// One stage of each of several independent states in one launch (kernel
// argument, so no device allocation): job j owns workgroups
// first_block[j] .. first_block[j + 1] - 1, one chunk each.  Every job's
// program uses the launch's chunk size C and has nchunks = its block count.
constexpr uint32_t kStageJobsMax = 64;
struct StageJob {
    void *state;
    const uint32_t *prog;
    const void *tables;
    const void *kron_lo, *kron_hi;  // as in StageLaunch (kron_lo NULL: read the state)
    int32_t kron_nlo, pad;
};
struct StageJobs {
    uint32_t n;
    uint32_t first_block[kStageJobsMax + 1];
    StageJob job[kStageJobsMax];
};
template <typename R> hipError_t launch_stage_multi(const StageJobs &J, int C, bool quad, hipStream_t s);

// Rotation stages (kernel_rot.hip): 8- or 4-byte slots, local-index bits
// 5..14 folded into bits 0..4, so that local bit l lands on slot bit l mod 5.
__host__ __device__ inline uint32_t rot_swizzle(uint32_t i) { return i ^ (((i >> 5) ^ (i >> 10)) & 31u); }
constexpr int kRotOpWords = 32;
template <typename R> hipError_t launch_rot(const StageLaunch &L, hipStream_t s);
template <typename R> hipError_t launch_rot_multi(const StageJobs &J, int C, bool quad, hipStream_t s);

hipError_t launch_copy(void *dst, const void *src, uint64_t bytes, hipStream_t s);
// host-memory offload: window v (outer qubits fixed) between the mapped host
// state and a device window; rows of row_bytes, 2^S windows interleaved
hipError_t launch_window_copy(void *dst, const void *src, uint64_t window_bytes, uint64_t row_bytes, int S,
                              uint64_t v, bool to_host, hipStream_t s);

// ---- measurement (kernels_measure.hip) ----
// Inverse-CDF sampling over bins of 2^nlow consecutive logical indices (at
// most 2^kSampleBinBits bins); layout: logical -> physical qubit.  bins, pre:
// room for the bins' masses and their prefix sums; cum: kSampleGroupsMax doubles, whose entry
// sample_groups(n - nlow) - 1 is the total mass.
constexpr int kSampleBinBits = 22, kSampleScanBits = 12;
constexpr int kSampleGroupsMax = 1 << (kSampleBinBits - kSampleScanBits);
inline int sample_groups(int bin_bits) { return bin_bits > kSampleScanBits ? 1 << (bin_bits - kSampleScanBits) : 1; }
struct SampleArgs {
    int32_t n, nlow;
    int32_t ordered;        // the bin qubits lie in logical order (set by the launcher)
    int32_t layout[40];
};
constexpr int kZMasksPerLaunch = 448;  // 3.5 KiB of kernel arguments
struct ZArgs {
    uint64_t m[kZMasksPerLaunch];   // physical qubit masks of the Z strings
    int32_t nm, pad;
};
template <typename R> hipError_t launch_collapse(void *state, int n, int phys_qubit, int outcome, double scale,
                                                 hipStream_t s);
template <typename R> hipError_t launch_sample(const void *state, SampleArgs S, double *bins, double *pre, double *cum,
                                               const double *u, uint64_t nshots, uint64_t *out,
                                               hipStream_t s);
size_t expect_z_scratch_bytes(uint32_t n_masks);
template <typename R> hipError_t launch_expect_z(const void *state, int n, const ZArgs &Z, double *out,
                                                 double *scratch, hipStream_t s);

}  // namespace qs
