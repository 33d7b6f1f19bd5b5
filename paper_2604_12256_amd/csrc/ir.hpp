// Internal representation shared by the host optimiser, the executor and the
// C ABI.  Host-only C++17; no HIP types here.
#pragma once

#include <algorithm>
#include <array>
#include <complex>
#include <cstdint>
#include <cstring>
#include <memory>
#include <string>
#include <type_traits>
#include <vector>

#include "qsim355.h"

namespace qs {

using cplx = std::complex<double>;

constexpr int kMaxGateQubits = 6;

// a * b.  (std::complex's own product checks for infinities in a call of its
// own; operators here are finite.)
template <typename T> inline std::complex<T> mul(const std::complex<T> &a, const std::complex<T> &b)
{
    return std::complex<T>(a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real());
}
// Factors that every amplitude of a state meets are formed wide and rounded
// once: their errors do not average out over the state.
typedef std::complex<long double> wide;

// Vector of plain values with room for N of them inside the object: the
// optimiser holds thousands of one- and two-qubit gates, whose qubit lists and
// matrices then cost no allocation of their own.
template <typename T, size_t N> class SmallVec {
    static_assert(std::is_trivially_copyable<T>::value, "plain values");

  public:
    SmallVec() = default;
    SmallVec(const SmallVec &o) { assign(o.begin(), o.end()); }
    SmallVec(const std::vector<T> &o) { assign(o.begin(), o.end()); }
    SmallVec(SmallVec &&o) noexcept { take(o); }
    SmallVec &operator=(const SmallVec &o)
    {
        if (this != &o) assign(o.begin(), o.end());
        return *this;
    }
    SmallVec &operator=(SmallVec &&o) noexcept
    {
        if (this != &o) {
            if (heap()) delete[] p_;
            take(o);
        }
        return *this;
    }
    ~SmallVec()
    {
        if (heap()) delete[] p_;
    }
    operator std::vector<T>() const { return std::vector<T>(begin(), end()); }
    size_t size() const { return n_; }
    bool empty() const { return n_ == 0; }
    T *begin() { return data(); }
    T *end() { return data() + n_; }
    const T *begin() const { return data(); }
    const T *end() const { return data() + n_; }
    T *data() { return heap() ? p_ : reinterpret_cast<T *>(in_); }
    const T *data() const { return heap() ? p_ : reinterpret_cast<const T *>(in_); }
    T &operator[](size_t i) { return data()[i]; }
    const T &operator[](size_t i) const { return data()[i]; }
    void push_back(T v)
    {
        if (n_ == cap_) grow(2 * n_);
        data()[n_++] = v;
    }
    void resize(size_t n) { resize(n, T()); }
    void resize(size_t n, T v)
    {
        if (n > cap_) grow(n);
        for (size_t i = n_; i < n; ++i) data()[i] = v;
        n_ = n;
    }
    void assign(size_t n, T v)
    {
        n_ = 0;
        resize(n, v);
    }
    template <typename I, typename = typename std::iterator_traits<I>::iterator_category> void assign(I b, I e)
    {
        const size_t n = (size_t)(e - b);
        n_ = 0;
        if (n > cap_) grow(n);
        std::copy(b, e, data());
        n_ = n;
    }
    void assign(std::initializer_list<T> l) { assign(l.begin(), l.end()); }
    void clear() { n_ = 0; }
    void swap(SmallVec &o) { std::swap(*this, o); }

  private:
    bool heap() const { return cap_ > N; }
    void grow(size_t n)
    {
        T *q = new T[n];
        std::copy(begin(), end(), q);
        if (heap()) delete[] p_;
        p_ = q;
        cap_ = n;
    }
    void take(SmallVec &o)
    {
        n_ = o.n_;
        cap_ = o.cap_;
        if (o.heap()) p_ = o.p_;
        else std::memcpy(in_, o.in_, sizeof(T) * n_);
        o.n_ = 0;
        o.cap_ = N;
    }

    size_t n_ = 0, cap_ = N;
    union {
        T *p_;
        alignas(T) unsigned char in_[sizeof(T) * N];
    };
};

// A linear operator on an ordered qubit list: bit t of the row/column index
// is qubit q[t] of the buffer it acts on.  `diag` operators store only the
// 2^k diagonal; dense ones store the 2^k x 2^k matrix row-major.
struct Operator {
    SmallVec<int, 6> q;
    bool diag = false;
    SmallVec<cplx, 4> m;
    // a diagonal kept as the product of these (qubits: positions in q) until
    // its own table is needed (m is then empty)
    std::shared_ptr<const std::vector<Operator>> parts;

    int k() const { return (int)q.size(); }
    uint64_t mask() const {
        uint64_t s = 0;
        for (int x : q) s |= 1ull << x;
        return s;
    }
    cplx at(uint64_t r, uint64_t c) const {
        if (diag) return r == c ? m[r] : cplx(0.0, 0.0);
        return m[(r << q.size()) + c];
    }
};

// Qubits on which the operator is not block diagonal (the qubits a stage must
// hold locally); on the others it only selects a block, like a control.
uint64_t need_mask(const Operator &op);
// True when every off-diagonal entry is exactly zero.
bool is_diagonal(const Operator &op);
// Table of a product of diagonal operators (every qubit of each in `to`) on
// the list `to`, times f[t][v] for the first qubits t of the list in the value
// v.  Formed wide, rounded once.
std::vector<cplx> diag_product(const std::vector<int> &to, const std::vector<const Operator *> &ds,
                               const std::vector<std::array<wide, 2>> &f = {});
// Gives an operator kept as parts its own table.
void materialize(Operator &op);
// The members of an operator kept as parts, on its qubits.
std::vector<Operator> parts_of(const Operator &op);
// A unitary 2x2 matrix u (row-major) as X^flip diag(l) [[1, 0], [q, 1]]
// [[1, p], [0, 1]] diag(1, r1) with real p, q, |p| <= 1 (l takes up what their
// rounding leaves).
struct Shears {
    bool flip;
    double p, q;
    wide l[2], r1;
};
Shears shears_of(const wide *u);
// Diagonals (with a table) whose entries are phases to rounding.
bool unit_phases(const Operator &op);
// One-qubit dense gates that shears_of reproduces to rounding.
bool is_rotation(const Operator &op);
// The blocks of a product of operators (the first applied first) that acts on
// the qubits `reg` and is block diagonal on `sel`: for every value of sel (bit
// t <-> sel[t]) a 2^|reg| x 2^|reg| matrix, row-major, bit t <-> reg[t].
std::vector<cplx> block_product(const std::vector<int> &reg, const std::vector<int> &sel,
                                const std::vector<const Operator *> &ops);
// Left-multiplies `acc` (on list acc.q) in place by `g`, whose qubits must all
// be in acc.q.
void apply_left(Operator &acc, const Operator &g);
// Validated input gate with its textbook matrix.
Operator gate_operator(const sim_gate &g, int n_qubits, std::string *err);

// ---------------------------------------------------------------------------
// Plan

// One op executed by the stage kernel on the registers of a phase.
struct KOp {
    // DENSE, DIAG, QUAD: the general kernel's; ROT, TABLE, LANE: the rotation
    // kernel's
    enum Type : uint32_t { DENSE = 1, DIAG = 2, QUAD = 3, ROT = 4, TABLE = 5, LANE = 6 } type;
    uint32_t reg_mask = 0;            // DENSE: register bits acted on
    std::vector<int> sel;             // physical qubits selecting the block (DENSE)
    std::vector<int> dq;              // DIAG: physical qubits of the table index (bit t <-> dq[t])
    std::vector<cplx> table;          // DENSE: 2^|sel| blocks of (2^k)^2; DIAG: 2^|dq| entries
    // the gates it is the product of, in order, multiplied into `table` once
    // the plan is final (planning compares lowerings before that)
    std::vector<const Operator *> members;
    // QUAD: a diagonal whose phase is a quadratic form of the index bits,
    // phi(x) = qc + sum_q qa[q] x_q + sum_{q<p} qb[q * n + p] x_q x_p over the
    // buffer's n physical qubits (the product of members on one or two
    // qubits: every such diagonal of unit modulus has this form exactly)
    long double qc = 0;
    std::vector<long double> qa, qb;
    // QUAD while planning: the diagonal tables it replaces, and their cost
    // (microseconds per 2^30 amplitudes), in case the stage keeps tables
    std::vector<KOp> alt;
    double alt_us = 0;
    // ROT: a product of one-qubit gates on each register bit of reg_mask
    // (rot[b], the first applied first) without the diagonals around it; pq:
    // the two shears of each register bit.  Registers renamed (by X on the
    // bits of a mask) before and after it.
    // TABLE: a diagonal on all register bits and the wave-uniform qubits sel,
    // table[sel][register index].  LANE: one on the registers whose bit `bit`
    // is `half` (bit < 0: all), selected by sel, which may be lane bits.
    // Tables name registers as the circuit does; `flip` says how they are
    // renamed where the operator runs.
    std::vector<std::vector<const Operator *>> rot;
    std::vector<double> pq;
    uint32_t flip = 0, flip_out = 0;
    int bit = -1, half = 1;
};

struct Phase {
    std::vector<int> reg;             // local bit index of register bit b
    std::vector<int> tmap;            // local bit index of thread-id bit i (lanes = i < 6)
    std::vector<KOp> ops;
    uint32_t flip = 0;                // registers renamed at the end (rotation stages)
};

struct PlanOp {
    sim_op_kind kind;
    int buffer = 0;                   // 0 = full state
    int buffer_qubits = 0;
    int src_lo = 0, src_hi = 0;       // KRON
    Operator op;                      // DENSE / DIAG (physical qubits of the buffer)
    std::vector<int> perm;            // PERM: destination bit of source bit p
    // STAGE
    std::vector<int> local;           // physical local qubits, ascending; local bit i <-> local[i]
    // the stage's operators in execution order (semantic): gates of a
    // whole-buffer run, or pointers into Plan::keep for a stage with phases
    std::vector<Operator> gates;
    std::vector<const Operator *> taken;
    size_t n_gates() const { return taken.empty() ? gates.size() : taken.size(); }
    const Operator &gate(size_t i) const { return taken.empty() ? gates[i] : *taken[i]; }
    std::vector<Phase> phases;        // kernel program
    bool rot = false;                 // ... of the rotation kernel
    double flops = 0;                 // floating-point operations of the op
    double bytes = 0;                 // algorithmic HBM bytes of the op
    double est_s = 0;                 // STAGE: modelled device seconds of its operators
    // WINDOW (host-memory offload pass): the next pass_ops ops run on each
    // window of the state whose outer qubits [outer_lo, outer_lo + outer_n)
    // are fixed; their qubits are window bits (physical bit p below outer_lo
    // stays p, one above the range becomes p - outer_n, and the outer bits
    // sit at W, W + 1, ... where only selectors may read them)
    int outer_lo = 0, outer_n = 0, pass_ops = 0;
    bool init_window = false;         // the windows start as |0...0> instead of being read
};

struct PlanStats {
    uint64_t full_passes = 0, write_passes = 0, n_stages = 0, n_dense = 0, n_diag = 0,
             n_kron = 0, n_perm = 0, n_subruns = 0, n_ops = 0;
    double bytes = 0, flops = 0, plan_ms = 0, est_ms = 0;
    uint64_t dd_visits = 0, booster_gates = 0, booster_groups = 0;
    uint64_t offload_passes = 0;
    double pcie_bytes = 0;
};

struct Options {
    uint32_t opt = 0, C = 0, F = 5, D = 10, B = 4, force_fuse_k = 0;
    int reg_bits = 4;                 // register bits per thread in a stage
    int fixed_low = 6;                // physical bits every stage keeps local (coalescing; set per dtype)
    int window_qubits = 0;            // host-memory offload: qubits of a device window (0 = off)
};

struct Plan {
    int n = 0;
    sim_dtype dtype = SIM_C128;
    Options opt;
    std::vector<int> buffer_qubits;   // [0] = n; booster sub-states after
    std::vector<PlanOp> ops;
    std::vector<int> layout;          // logical qubit -> physical bit at the end
    PlanStats stats;
    // gate lists on physical qubits that stages and their operators point into
    std::vector<std::shared_ptr<std::vector<Operator>>> keep;
};

// Fills the defaults of the options for a dtype.
Options resolve_options(const sim_options *o, sim_dtype dtype, int n);
// Builds the plan (all host passes).  Throws std::runtime_error on failure.
void build_plan(Plan &plan, const std::vector<Operator> &gates);

// Host-memory offload: physical bit of window bit w of a pass whose outer
// range is [lo, lo + n) in a state of `nq` qubits (window bits at and above
// nq - n name the outer bits, in order).
inline int window_to_physical(int w, int lo, int n, int nq)
{
    const int W = nq - n;
    if (w >= W) return lo + (w - W);
    return w < lo ? w : w + n;
}
inline int physical_to_window(int p, int lo, int n, int nq)
{
    const int W = nq - n;
    if (p < lo) return p;
    if (p < lo + n) return W + (p - lo);
    return p - n;
}
// Window qubits for a device work area of `dev_bytes` holding two windows
// (at most nq - 1); 0 if not even one qubit fits.
int offload_window_qubits(uint64_t dev_bytes, uint64_t amp_bytes, int nq);

// Passes, exposed for the plan builder and its tests.
std::vector<Operator> diagonal_detector(int n, int D, const std::vector<Operator> &in, uint64_t *visits);
void divider(int n, int div_size, std::vector<int> &que);

}  // namespace qs
