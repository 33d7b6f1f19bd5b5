// Cache-blocked stage kernel for stages whose gates are one-qubit gates and
// diagonals (rotation stages; the general kernel is kernel_stage.hip, whose
// chunk, register phases and thread maps these share).
//
// A one-qubit gate is a real rotation between two diagonals,
//   U = DL [[1, 0], [q, 1]] [[1, p], [0, 1]] DR     (|p| <= 1),
// with X to the left where its off-diagonal is the larger part.  The kernel
// applies the two shears, 2 FMA an amplitude where a 2x2 complex product
// takes 8.  The host multiplies DL, the next gate's DR and the circuit's own
// diagonals into one table of 2^RB factors per level of rotations (DR, DL and
// the gates between commute), and X costs nothing: it renames registers until
// the next exchange, whose slot addresses take the renaming in.
//
// So a phase is a few levels of two fixed pieces of code, rotations on any
// register bits and one product of every register with a factor read through
// scalar loads, instead of a choice among operators on every subset of
// register bits.  That choice cost the general kernel its registers (240, two
// waves a SIMD, 128 of them two copies of the amplitudes); this one needs 121
// (89 in complex64), and exchanges real and imaginary parts one after the
// other through half the LDS, so four workgroups of a 2^12 chunk share a CU
// where two did.
//
// Bound: the chunk-strided read and write of the state (7.6 ms for 2^30
// complex128 amplitudes with no gates at all and cached accesses; 6.9 to 7.3
// ms, 4.8 TB/s, for the few rotations of a QAOA stage, bypassing the caches).
// A pass of the 30-qubit layered circuit takes 8.3 to 8.9 ms on average (13.7
// on the general kernel), its 15 passes 125 to 133 ms (206); complex64: 5.3 to
// 5.5 ms (8.2), 79 to 83 ms (140).  What is above the bound: 4.6 ms of VALU
// and 5.0 ms of LDS time that four workgroups a CU do not quite hide.
//
// The variant with quadratic phases (QD) holds their running products in FP64
// besides the amplitudes: three waves a SIMD.  A layer of couplings between
// all qubits is one such operator in one of the layer's stages.  QAOA of 25
// qubits and 5 layers, run: 4.12 -> 2.57 ms (11 passes; on the general kernel
// the couplings fill tables in every stage), 26 qubits and 3 layers in
// complex64 2.50 -> 1.86 ms.
//
// Program words (built on the host; read with wave-uniform loads):
//   header  as in kernel_stage.hip, [24] bytes of the header, phases and ops,
//           [25, 26] byte offset of the first table  [27] bytes of the tables
//   phase   [0] nops  [2] register local mask  [3] number of wave bits
//           [4..6] local bit of thread-id bit i (bytes)  [8, 9] physical bit of wave bit i (bytes)
//           [10] LDS byte offset (XOR) of the registers renamed at the end of the phase
//           [16 + j] LDS byte offset of register j
//           [16 + 2^RB + 32 o ...] op o (128 bytes)
//   op      [0] bit 0 level, bit 1 diagonal selected by lanes, bit 2 quadratic phase | ...
//     level: rotated register bits << 8 | number of fields << 16; [1, 2] table byte offset,
//       [3 + f] selector field f: first physical position | width << 16; [16...] p, q of each
//       register bit, in the state's precision; the table holds 2^RB factors per selector value
//     by lanes: halves << 8 | selector count << 24; bit 2 b + v of halves
//       multiplies the registers whose bit b is v, bit 2 RB all of them; [1, 2] table byte
//       offset, [3...5] selector sources (bytes): 0x80 | b is lane bit b, any other the
//       physical position of a chunk or wave bit
//     quadratic phase (first in its phase; kernel variant): [3...7] as in kernel_stage.hip
#include "device.hpp"

namespace qs {

namespace {

constexpr int kRotMaxThreads = 512;
constexpr uint32_t kRotLdsBytes = 64u * 1024u;
constexpr uint64_t kRotWarmChunks = 1024;

typedef __attribute__((address_space(3))) char lds_byte_t;

// In place, so that the compiler keeps one copy of the amplitudes: d += s * v
// with s in scalar registers, and (x, y) *= f.
__device__ __forceinline__ void fmac_s(double &d, double s, double v)
{
    asm("v_fmac_f64 %0, %1, %2" : "+v"(d) : "s"(s), "v"(v));
}
__device__ __forceinline__ void fmac_s(float &d, float s, float v)
{
    asm("v_fmac_f32 %0, %1, %2" : "+v"(d) : "s"(s), "v"(v));
}
#define QS_CMUL(T, bits, kind, name)                                                                              \
    __device__ __forceinline__ void name(T &x, T &y, T fx, T fy)                                                  \
    {                                                                                                             \
        T t, u;                                                                                                   \
        asm("v_mul_" bits "_e64 %2, -%5, %1\n\tv_mul_" bits "_e64 %3, %5, %0\n\t"                                 \
            "v_fma_" bits " %0, %4, %0, %2\n\tv_fma_" bits " %1, %4, %1, %3"                                      \
            : "+v"(x), "+v"(y), "=&v"(t), "=&v"(u)                                                                \
            : kind(fx), kind(fy));                                                                                \
    }
QS_CMUL(double, "f64", "s", cmul_s)
QS_CMUL(double, "f64", "v", cmul_v)
QS_CMUL(float, "f32", "s", cmul_s)
QS_CMUL(float, "f32", "v", cmul_v)
#undef QS_CMUL

// One part (real or imaginary) of the chunk between two mappings.  The thread
// and register parts of a local index have disjoint bits, so a slot is a
// per-thread term XOR a wave-uniform one.
template <typename R, int NR, typename Get>
__device__ __forceinline__ void exchange_part(Get part, uint32_t wb, const QS_CONST uint32_t *old_off, uint32_t rb,
                                              const QS_CONST uint32_t *new_off)
{
    typedef __attribute__((address_space(3))) R lds_r_t;
    // complex64 has 2 x 32 slots: their addresses are formed again for each
    // part, not kept from one to the next
    if constexpr (sizeof(R) == 4) asm volatile("" : "+v"(wb), "+v"(rb));
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; ++j) *reinterpret_cast<lds_r_t *>((uintptr_t)(wb ^ old_off[j])) = part(j);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; ++j) part(j) = *reinterpret_cast<const lds_r_t *>((uintptr_t)(rb ^ new_off[j]));
}

// Reads a word that nobody uses.
__device__ __forceinline__ void touch(const char *p)
{
    const uint32_t w = *reinterpret_cast<const uint32_t *>(p);
    asm volatile("" ::"v"(w));
}

struct RotRec {
    uint32_t w[16];
};

// The first half of an op record.  (One is read past a phase's last op: every
// program ends with a spare record.)
__device__ __forceinline__ RotRec load_head(const QS_CONST uint32_t *p)
{
    RotRec r;
#pragma unroll
    for (int i = 0; i < 16; ++i) r.w[i] = p[i];
    return r;
}

template <typename R, int RB, bool QD>
__device__ __forceinline__ void rot_chunks(c2_t<R> *__restrict__ state, const uint32_t *__restrict__ Pg,
                                           const c2_t<R> *__restrict__ tables, uint64_t first, uint64_t nchunks,
                                           uint64_t step, uint64_t xbits, const c2_t<R> *__restrict__ klo,
                                           const c2_t<R> *__restrict__ khi, int knlo)
{
    using V = c2_t<R>;
    constexpr int NR = 1 << RB;
    const QS_CONST uint32_t *P = as_const(Pg);
    const QS_CONST char *ctables = reinterpret_cast<const QS_CONST char *>(as_const(reinterpret_cast<const R *>(tables)));
    const char *vtables = reinterpret_cast<const char *>(tables);
    extern __shared__ char smem_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(lds_byte_t *)smem_raw;
    const int C = (int)P[0], nph = (int)P[2];
    const uint64_t Lmask = (uint64_t)P[4] | ((uint64_t)P[5] << 32);
    const uint64_t Gmask = (uint64_t)P[6] | ((uint64_t)P[7] << 32);
    const uint32_t tid = threadIdx.x;
    uint32_t wave;
    asm volatile("v_readfirstlane_b32 %0, %1" : "=s"(wave) : "v"(tid));
    wave >>= 6;
    const uint32_t neutral_r = ((1u << C) - 1) & ~((1u << (C - RB)) - 1);
    uint32_t neutral_t[3] = {0, 0, 0};
    for (int i = 0; i < C - RB; ++i) neutral_t[i / 4] |= (uint32_t)i << (8 * (i % 4));
    const uint64_t tphys = deposit(tid, Lmask);
    auto reg_off = [&](int j) {
        uint64_t o = 0;
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if ((j >> b) & 1) o |= 1ull << P[8 + C - RB + b];
        return o;
    };

    // With one chunk a workgroup every record and table would be waited for in
    // turn, from memory: their lines are brought into the L2 at once.  (48
    // circuits of 16 qubits, a program each: 251 -> 209 us; one of 13 qubits in
    // complex64, 40 layers, run 0.143 -> 0.097 ms; 22 qubits 0.565 -> 0.533 ms.)
    // By the workgroups that run first, four a CU: later ones find the lines
    // there, and a program with many tables has more of them than its chunks
    // have amplitudes.  (First run of one-qubit gates and couplings mixed, 26
    // and 27 qubits: 1.41 and 2.64 ms with all workgroups, 1.38 and 2.60 with
    // these, 1.39 and 2.61 with none; 24 qubits, layered: 0.621, 0.612, 0.651.)
    if (nchunks - first <= step && first < kRotWarmChunks) {
        const uint32_t pbytes = P[24], tbytes = P[27];
        const char *pp = reinterpret_cast<const char *>(Pg);
        const char *tp = vtables + ((uint64_t)P[25] | ((uint64_t)P[26] << 32));
        const uint32_t line = 128, row = line << (C - RB);
        for (uint32_t i = tid * line; i < pbytes; i += row) touch(pp + i);
        for (uint32_t i = tid * line; i < tbytes; i += row) touch(tp + i);
    }

    V amp[NR];
    const uint64_t cstep = deposit(step, Gmask);
    uint64_t cbase = deposit(first, Gmask);
    for (uint64_t chunk = first; chunk < nchunks; chunk += step, cbase = ((cbase | ~Gmask) + cstep) & Gmask) {
        if (klo) {
            // the tensor product klo (x) khi, formed on load
            const uint64_t lomask = (1ull << knlo) - 1, base = cbase | tphys, rbits = reg_off(NR - 1);
            if (!(rbits & lomask)) {  // register bits all in the high factor
                const V lo = klo[base & lomask];
#pragma unroll
                for (int j = 0; j < NR; ++j) amp[j] = cmul(lo, khi[(base | reg_off(j)) >> knlo]);
            } else if (!(rbits >> knlo)) {  // all in the low factor
                const V hi = khi[base >> knlo];
#pragma unroll
                for (int j = 0; j < NR; ++j) amp[j] = cmul(klo[(base | reg_off(j)) & lomask], hi);
            } else {
#pragma unroll
                for (int j = 0; j < NR; ++j) {
                    const uint64_t x = base | reg_off(j);
                    amp[j] = cmul(klo[x & lomask], khi[x >> knlo]);
                }
            }
        } else {
            const V *pt = state + (cbase | tphys);
#pragma unroll
            for (int j = 0; j < NR; ++j) amp[j] = nt_load(pt + reg_off(j));
        }
        uint32_t cur_lb = tid, cur_r = neutral_r, cur_flip = 0;
        uint32_t cur_t0 = neutral_t[0], cur_t1 = neutral_t[1], cur_t2 = neutral_t[2];
        const QS_CONST uint32_t *cur_off = P + 128;
        for (int p = 0; p <= nph; ++p) {
            // after the last phase, back to the load mapping
            const bool last = p == nph;
            const QS_CONST uint32_t *ph = P + P[32 + (last ? 0 : p)];
            const uint32_t rmask = last ? neutral_r : ph[2];
            const uint32_t t0 = last ? neutral_t[0] : ph[4], t1 = last ? neutral_t[1] : ph[5],
                           t2 = last ? neutral_t[2] : ph[6];
            if (rmask != cur_r || t0 != cur_t0 || t1 != cur_t1 || t2 != cur_t2 || cur_flip) {
                const QS_CONST uint32_t *off = last ? P + 128 : ph + 16;
                uint32_t lb = 0;
                const uint32_t t[3] = {t0, t1, t2};
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (i < C - RB) lb |= ((tid >> i) & 1u) << ((t[i / 4] >> (8 * (i % 4))) & 0xffu);
                uint32_t wb = (lds | (rot_swizzle(cur_lb) * (uint32_t)sizeof(R))) ^ cur_flip;
                uint32_t rb = lds | (rot_swizzle(lb) * (uint32_t)sizeof(R));
                asm volatile("" : "+v"(wb));
                asm volatile("" : "+v"(rb));
                exchange_part<R, NR>([&](int j) -> R & { return amp[j].x; }, wb, cur_off, rb, off);
                exchange_part<R, NR>([&](int j) -> R & { return amp[j].y; }, wb, cur_off, rb, off);
                cur_lb = lb;
                cur_r = rmask;
                cur_t0 = t0;
                cur_t1 = t1;
                cur_t2 = t2;
                cur_off = off;
            }
            if (last) break;
            cur_flip = ph[10];
            uint64_t ub = cbase | xbits;
            const uint32_t nwave = ph[3];
            for (uint32_t i = 0; i < nwave; ++i)
                ub |= (uint64_t)((wave >> i) & 1u) << ((ph[8 + (i >> 2)] >> ((i & 3u) * 8)) & 0xffu);
            const uint32_t nops = ph[0];
            const QS_CONST uint32_t *rec = ph + kStagePhaseWords + NR;
            RotRec h = load_head(rec);
            for (uint32_t o = 0; o < nops; ++o) {
                // no alternatives, only pieces that are skipped: the compiler
                // then keeps the amplitudes in one set of registers
                const uint32_t w0 = h.w[0];
                const uint64_t toff = (uint64_t)h.w[1] | ((uint64_t)h.w[2] << 32);
                if (w0 & 1u) {
                    uint32_t sel = 0, u = 0;
                    const uint32_t nf = (w0 >> 16) & 15u;
#pragma unroll
                    for (uint32_t f = 0; f < 8; ++f)
                        if (f < nf) {
                            const uint32_t d = h.w[3 + f], w = d >> 16;
                            sel |= ((uint32_t)(ub >> (d & 63u)) & ((1u << w) - 1u)) << u;
                            u += w;
                        }
                    const QS_CONST R *m = reinterpret_cast<const QS_CONST R *>(
                        ctables + toff + (uint64_t)sel * (uint32_t)(NR * sizeof(V)));
                    const QS_CONST R *pq = reinterpret_cast<const QS_CONST R *>(rec + 16);
                    // p, q and the first half of the factors in scalar registers
                    // before the rotations, which then wait for no load
                    R s[2 * RB], f[NR];
#pragma unroll
                    for (int i = 0; i < 2 * RB; ++i) s[i] = pq[i];
#pragma unroll
                    for (int i = 0; i < NR; ++i) f[i] = m[i];
#pragma unroll
                    for (int i = 0; i < 2 * RB; ++i) asm volatile("" : "+s"(s[i]));
#pragma unroll
                    for (int i = 0; i < NR; ++i) asm volatile("" : "+s"(f[i]));
#pragma unroll
                    for (int b = 0; b < RB; ++b) {
                        if (!((w0 >> (8 + b)) & 1u)) continue;
#pragma unroll
                        for (int j = 0; j < NR; ++j) {
                            if ((j >> b) & 1) continue;
                            const int k = j | (1 << b);
                            fmac_s(amp[j].x, s[2 * b], amp[k].x);
                            fmac_s(amp[j].y, s[2 * b], amp[k].y);
                            fmac_s(amp[k].x, s[2 * b + 1], amp[j].x);
                            fmac_s(amp[k].y, s[2 * b + 1], amp[j].y);
                        }
                    }
                    R g[NR];
#pragma unroll
                    for (int i = 0; i < NR; ++i) g[i] = m[NR + i];
#pragma unroll
                    for (int j = 0; j < NR / 2; ++j) cmul_s(amp[j].x, amp[j].y, f[2 * j], f[2 * j + 1]);
#pragma unroll
                    for (int j = 0; j < NR / 2; ++j)
                        cmul_s(amp[NR / 2 + j].x, amp[NR / 2 + j].y, g[2 * j], g[2 * j + 1]);
                }
                if constexpr (QD)
                    if (w0 & 4u) quad_op<R, RB>(amp, h.w, Pg, chunk, tid, C, rmask, t0, t1, t2);
                if (w0 & 2u) {
                    uint32_t sel = 0;
                    const uint32_t nsel = w0 >> 24;
                    for (uint32_t u = 0; u < nsel; ++u) {
                        const uint32_t s = (rec[3 + (u >> 2)] >> ((u & 3u) * 8)) & 0xffu;
                        sel |= ((s & 0x80u) ? (tid >> (s & 63u)) & 1u : (uint32_t)(ub >> (s & 63u)) & 1u) << u;
                    }
                    const V f = *reinterpret_cast<const V *>(vtables + toff + (uint64_t)sel * (uint32_t)sizeof(V));
                    // mask bit 2 b + v: the registers whose bit b is v; bit 2 RB: all
#pragma unroll
                    for (int hf = 0; hf <= 2 * RB; ++hf) {
                        if (!((w0 >> (8 + hf)) & 1u)) continue;
#pragma unroll
                        for (int j = 0; j < NR; ++j)
                            if (hf == 2 * RB || ((j >> (hf >> 1)) & 1) == (hf & 1))
                                cmul_v(amp[j].x, amp[j].y, f.x, f.y);
                    }
                }
                rec += kRotOpWords;
                h = load_head(rec);
            }
        }
        {
            // the store's addresses are formed again, not kept through the ops
            uint64_t tp = tphys;
            asm volatile("" : "+v"(tp));
            V *pt = state + (cbase | tp);
#pragma unroll
            for (int j = 0; j < NR; ++j) nt_store(pt + reg_off(j), amp[j]);
        }
        __syncthreads();  // LDS reuse by the next chunk
    }
}

template <typename R, int RB, bool QD>
__global__ __launch_bounds__(kRotMaxThreads) __attribute__((amdgpu_waves_per_eu(QD ? 3 : 4))) void
k_rot(c2_t<R> *__restrict__ state, const uint32_t *__restrict__ Pg, const c2_t<R> *__restrict__ tables,
      uint64_t nchunks, uint64_t xbits, const c2_t<R> *__restrict__ klo, const c2_t<R> *__restrict__ khi, int knlo)
{
    rot_chunks<R, RB, QD>(state, Pg, tables, blockIdx.x, nchunks, gridDim.x, xbits, klo, khi, knlo);
}

// Stages of several independent states, as k_stage_multi, of any chunk sizes:
// the workgroups have the threads and the LDS of the largest, the waves beyond
// a smaller one's end at once.  A chunk is a chain of phases that takes 40 to
// 65 us however few there are, so states of 10, 11 and 12 qubits in a launch
// for each size took the sum of those (128 circuits of 10 to 13 qubits:
// 257 us, 211 together).
template <typename R, int RB, bool QD>
__global__ __launch_bounds__(kRotMaxThreads) __attribute__((amdgpu_waves_per_eu(QD ? 3 : 4))) void
k_rot_multi(const StageJobs J)
{
    const uint32_t b = blockIdx.x;
    uint32_t lo = 0, hi = J.n;  // first_block[lo] <= b < first_block[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (J.first_block[mid] <= b) lo = mid;
        else hi = mid;
    }
    const StageJob &job = J.job[lo];
    const uint64_t chunk = b - J.first_block[lo];
    if (threadIdx.x >= (1u << (as_const(job.prog)[0] - RB))) return;  // whole waves
    rot_chunks<R, RB, QD>((c2_t<R> *)job.state, job.prog, (const c2_t<R> *)job.tables, chunk, chunk + 1, 1, 0,
                      (const c2_t<R> *)job.kron_lo, (const c2_t<R> *)job.kron_hi, job.kron_nlo);
}

template <typename R, int RB, bool QD> hipError_t rot_shape(int C, uint32_t *threads, uint32_t *lds)
{
    static bool done = false;
    if (C < RB + 6 || C > 16) return hipErrorInvalidValue;
    *threads = 1u << (C - RB);
    *lds = (uint32_t)sizeof(R) << C;
    if (*threads > (uint32_t)kRotMaxThreads || *lds > kRotLdsBytes) return hipErrorInvalidValue;
    if (done) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void *)k_rot<R, RB, QD>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kRotLdsBytes);
    // the batched kernel with quadratic phases exists for complex128 only (in
    // complex64 it would need scratch memory)
    if constexpr (!QD || sizeof(R) == 8)
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)k_rot_multi<R, RB, QD>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kRotLdsBytes);
    done = e == hipSuccess;
    return e;
}

}  // namespace

template <typename R>
hipError_t launch_rot(const StageLaunch &L, hipStream_t s)
{
    constexpr int RB = sizeof(R) == 8 ? 4 : 5;
    uint32_t threads, lds;
    const hipError_t e =
        L.quad ? rot_shape<R, RB, true>(L.C, &threads, &lds) : rot_shape<R, RB, false>(L.C, &threads, &lds);
    if (e != hipSuccess) return e;
    if (L.kron_lo && (L.kron_nlo < 1 || L.kron_nlo >= L.n || !L.kron_hi)) return hipErrorInvalidValue;
    // as many workgroups as the general kernel: each walks several chunks of a
    // large state, so its set-up is paid once for them
    const uint32_t grid = (uint32_t)(L.nchunks < (1ull << 15) ? L.nchunks : (1ull << 15));
    const auto kernel = L.quad ? k_rot<R, RB, true> : k_rot<R, RB, false>;
    kernel<<<grid, threads, lds, s>>>((c2_t<R> *)L.state, L.prog, (const c2_t<R> *)L.tables, L.nchunks, L.xbits,
                                      (const c2_t<R> *)L.kron_lo, (const c2_t<R> *)L.kron_hi, L.kron_nlo);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_rot_multi(const StageJobs &J, int C, bool quad, hipStream_t s)
{
    constexpr int RB = sizeof(R) == 8 ? 4 : 5;
    if (J.n == 0 || J.n > kStageJobsMax || J.first_block[0] != 0) return hipErrorInvalidValue;
    for (uint32_t j = 0; j < J.n; ++j)
        if (J.first_block[j + 1] <= J.first_block[j] || J.job[j].state == nullptr || J.job[j].prog == nullptr)
            return hipErrorInvalidValue;
    uint32_t threads, lds;
    if constexpr (sizeof(R) == 8) {
        if (quad) {
            const hipError_t e = rot_shape<R, RB, true>(C, &threads, &lds);
            if (e != hipSuccess) return e;
            k_rot_multi<R, RB, true><<<J.first_block[J.n], threads, lds, s>>>(J);
            return hipGetLastError();
        }
    } else if (quad) {
        return hipErrorInvalidValue;
    }
    const hipError_t e = rot_shape<R, RB, false>(C, &threads, &lds);
    if (e != hipSuccess) return e;
    k_rot_multi<R, RB, false><<<J.first_block[J.n], threads, lds, s>>>(J);
    return hipGetLastError();
}

template hipError_t launch_rot<double>(const StageLaunch &, hipStream_t);
template hipError_t launch_rot<float>(const StageLaunch &, hipStream_t);
template hipError_t launch_rot_multi<double>(const StageJobs &, int, bool, hipStream_t);
template hipError_t launch_rot_multi<float>(const StageJobs &, int, bool, hipStream_t);

}  // namespace qs
