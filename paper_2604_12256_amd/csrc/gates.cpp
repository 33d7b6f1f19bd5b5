// Gate library and operator algebra of the host optimiser (FP64).
//
// The paper names the gates it uses (Z, CP, RZZ in Sec. 3 and 4.5; RX, H, RY in
// Sec. 4.5; CNOT and RZ in Sec. 5.1) but prints no matrices; the textbook ones
// are used.  Matrix layout follows Sec. 2.2: bit t of the row/column index is
// qubit q[t].
#include <algorithm>
#include <cmath>
#include <stdexcept>

#include "ir.hpp"

namespace qs {

namespace {

int arity(uint32_t kind, uint32_t nq)
{
    switch (kind) {
    case SIM_G_MATRIX: case SIM_G_DIAG: return (int)nq;
    case SIM_G_CZ: case SIM_G_CNOT: case SIM_G_CPHASE: case SIM_G_RZZ: case SIM_G_SWAP: return 2;
    default: return 1;
    }
}

}  // namespace

Operator gate_operator(const sim_gate &g, int n, std::string *err)
{
    Operator op;
    if (g.kind >= SIM_G_NKINDS) { *err = "unknown gate kind"; return op; }
    const int k = arity(g.kind, g.nq);
    if (k < 1 || k > kMaxGateQubits || (int)g.nq != k) { *err = "bad qubit count for gate kind"; return op; }
    for (int t = 0; t < k; ++t) {
        if ((int)g.q[t] >= n) { *err = "qubit index out of range"; return op; }
        for (int u = 0; u < t; ++u)
            if (g.q[u] == g.q[t]) { *err = "duplicate qubit in gate"; return op; }
        op.q.push_back((int)g.q[t]);
    }
    const int d = 1 << k;
    const double th = g.theta, c = std::cos(th / 2), s = std::sin(th / 2), r2 = std::sqrt(0.5);
    const cplx I(0.0, 1.0);
    auto dense = [&](std::initializer_list<cplx> v) { op.diag = false; op.m.assign(v); };
    auto diagv = [&](std::initializer_list<cplx> v) { op.diag = true; op.m.assign(v); };
    switch (g.kind) {
    case SIM_G_MATRIX: {
        if (!g.data) { *err = "MATRIX gate without data"; return op; }
        op.diag = false;
        op.m.resize((size_t)d * d);
        for (int i = 0; i < d * d; ++i) op.m[i] = cplx(g.data[2 * i], g.data[2 * i + 1]);
        // unitarity: |M^H M - I| <= 1e-10 entrywise
        for (int a = 0; a < d; ++a)
            for (int b = 0; b < d; ++b) {
                cplx acc = 0;
                for (int r = 0; r < d; ++r) acc += mul(std::conj(op.m[r * d + a]), op.m[r * d + b]);
                if (std::abs(acc - (a == b ? 1.0 : 0.0)) > 1e-10) { *err = "MATRIX gate is not unitary"; return op; }
            }
        if (is_diagonal(op)) {
            SmallVec<cplx, 4> dv;
            for (int i = 0; i < d; ++i) dv.push_back(op.m[(size_t)i * d + i]);
            op.m = dv;
            op.diag = true;
        }
        break;
    }
    case SIM_G_DIAG:
        if (!g.data) { *err = "DIAG gate without data"; return op; }
        op.diag = true;
        op.m.resize(d);
        for (int i = 0; i < d; ++i) {
            op.m[i] = cplx(g.data[2 * i], g.data[2 * i + 1]);
            if (std::abs(std::abs(op.m[i]) - 1.0) > 1e-10) { *err = "DIAG entry is not of unit modulus"; return op; }
        }
        break;
    case SIM_G_H: dense({r2, r2, r2, -r2}); break;
    case SIM_G_X: dense({0, 1, 1, 0}); break;
    case SIM_G_Y: dense({0, -I, I, 0}); break;
    case SIM_G_Z: diagv({1, -1}); break;
    case SIM_G_S: diagv({1, I}); break;
    case SIM_G_T: diagv({1, cplx(r2, r2)}); break;
    case SIM_G_SX: dense({cplx(0.5, 0.5), cplx(0.5, -0.5), cplx(0.5, -0.5), cplx(0.5, 0.5)}); break;
    case SIM_G_RX: dense({c, -I * s, -I * s, c}); break;
    case SIM_G_RY: dense({c, -s, s, c}); break;
    case SIM_G_RZ: diagv({cplx(c, -s), cplx(c, s)}); break;
    case SIM_G_CZ: diagv({1, 1, 1, -1}); break;
    case SIM_G_CPHASE: diagv({1, 1, 1, cplx(std::cos(th), std::sin(th))}); break;
    case SIM_G_RZZ: diagv({cplx(c, -s), cplx(c, s), cplx(c, s), cplx(c, -s)}); break;
    case SIM_G_CNOT:  // index = b(control) + 2 b(target)
        dense({1, 0, 0, 0,  0, 0, 0, 1,  0, 0, 1, 0,  0, 1, 0, 0});
        break;
    case SIM_G_SWAP:
        dense({1, 0, 0, 0,  0, 0, 1, 0,  0, 1, 0, 0,  0, 0, 0, 1});
        break;
    default: *err = "unknown gate kind"; return op;
    }
    return op;
}

bool is_diagonal(const Operator &op)
{
    if (op.diag) return true;
    const uint64_t d = 1ull << op.q.size();
    for (uint64_t r = 0; r < d; ++r)
        for (uint64_t c = 0; c < d; ++c)
            if (r != c && op.m[r * d + c] != cplx(0.0, 0.0)) return false;
    return true;
}

uint64_t need_mask(const Operator &op)
{
    if (op.diag) return 0;
    const int k = op.k();
    const uint64_t d = 1ull << k;
    uint64_t need = 0;
    for (int t = 0; t < k; ++t) {
        bool blockdiag = true;
        for (uint64_t r = 0; r < d && blockdiag; ++r)
            for (uint64_t c = 0; c < d; ++c)
                if ((((r ^ c) >> t) & 1) && op.m[r * d + c] != cplx(0.0, 0.0)) { blockdiag = false; break; }
        if (!blockdiag) need |= 1ull << op.q[t];
    }
    return need;
}

void apply_left(Operator &acc, const Operator &g)
{
    const int K = acc.k(), k = g.k();
    std::vector<int> pos(k);
    for (int t = 0; t < k; ++t) {
        pos[t] = -1;
        for (int u = 0; u < K; ++u)
            if (acc.q[u] == g.q[t]) pos[t] = u;
        if (pos[t] < 0) throw std::runtime_error("apply_left: qubit not in accumulator");
    }
    const uint64_t D = 1ull << K, d = 1ull << k;
    if (acc.diag && g.diag) {
        for (uint64_t x = 0; x < D; ++x) {
            uint64_t r = 0;
            for (int t = 0; t < k; ++t) r |= ((x >> pos[t]) & 1ull) << t;
            acc.m[x] = mul(acc.m[x], g.m[r]);
        }
        return;
    }
    if (acc.diag) {  // promote to dense
        SmallVec<cplx, 4> full;
        full.assign(D * D, cplx(0.0, 0.0));
        for (uint64_t x = 0; x < D; ++x) full[x * D + x] = acc.m[x];
        acc.m.swap(full);
        acc.diag = false;
    }
    uint64_t gmask = 0;
    std::vector<uint64_t> off(d);
    for (uint64_t r = 0; r < d; ++r) {
        uint64_t o = 0;
        for (int t = 0; t < k; ++t)
            if ((r >> t) & 1) o |= 1ull << pos[t];
        off[r] = o;
    }
    for (int t = 0; t < k; ++t) gmask |= 1ull << pos[t];
    std::vector<cplx> u(d * d), v(d), w(d);
    for (uint64_t r = 0; r < d; ++r)
        for (uint64_t c = 0; c < d; ++c) u[r * d + c] = g.at(r, c);
    // every column of acc is a state of K qubits; apply g to it
    cplx *m = acc.m.data();
    for (uint64_t col = 0; col < D; ++col)
        for (uint64_t base = 0; base < D; ++base) {
            if (base & gmask) continue;
            for (uint64_t c = 0; c < d; ++c) v[c] = m[(base | off[c]) * D + col];
            for (uint64_t r = 0; r < d; ++r) {
                cplx s = 0;
                for (uint64_t c = 0; c < d; ++c) s += mul(u[r * d + c], v[c]);
                w[r] = s;
            }
            for (uint64_t r = 0; r < d; ++r) m[(base | off[r]) * D + col] = w[r];
        }
}

namespace {

int position(const std::vector<int> &list, int q)
{
    for (size_t u = 0; u < list.size(); ++u)
        if (list[u] == q) return (int)u;
    return -1;
}

// ds with each operator kept as parts replaced by them, on its own qubits;
// `own` holds the copies.
std::vector<const Operator *> expand_parts(const std::vector<const Operator *> &ds, std::vector<Operator> &own)
{
    size_t n = 0;
    for (const Operator *d : ds) n += d->parts ? d->parts->size() : 0;
    own.reserve(n);
    std::vector<const Operator *> out;
    out.reserve(ds.size() + n);
    for (const Operator *d : ds) {
        if (!d->parts) {
            out.push_back(d);
            continue;
        }
        for (const Operator &part : *d->parts) {
            own.push_back(part);
            for (int &q : own.back().q) q = d->q[q];
            out.push_back(&own.back());
        }
    }
    return out;
}

// A product of diagonals as c * prod_q a_q^x_q * prod_qp b_qp^(x_q x_p) * the
// terms on more than two bits of x: f where all bits of `vars` are set.
struct Term {
    uint32_t vars;
    wide f;
};

// Its table on K bits, built bit by bit: the upper half is the lower half times
// the factor of bit t, which is a form of the same kind on the bits that t is
// coupled with: two products an entry at most, however many diagonals.
// (Layers of three-qubit diagonals and H on 22 qubits, complex128, load: 1.43
// ms with each diagonal multiplied into the finished table, 0.51 ms.)
void form_table(int K, const wide &c, const wide *a, const wide *b, const std::vector<Term> &high, wide *out)
{
    const wide one(1);
    std::vector<wide> row;
    out[0] = c;
    for (int t = 0; t < K; ++t) {
        const size_t half = (size_t)1 << t;
        uint32_t coupled = 0;
        for (int i = 0; i < t; ++i)
            if (b[(size_t)t * K + i] != one) coupled |= 1u << i;
        bool terms = false;
        for (const Term &h : high)
            if (h.vars >> t == 1) {
                coupled |= h.vars ^ (1u << t);
                terms = true;
            }
        if (!coupled) {
            if (a[t] == one) std::copy(out, out + half, out + half);
            else
                for (size_t x = 0; x < half; ++x) out[x | half] = mul(out[x], a[t]);
            continue;
        }
        // row: the factor by the coupled bits, packed
        const int n = __builtin_popcount(coupled);
        if (row.size() < ((size_t)1 << n)) row.resize((size_t)1 << n);
        if (!terms) {
            row[0] = a[t];
            size_t m = 1;
            for (uint32_t left = coupled; left; left &= left - 1, m *= 2) {
                const wide f = b[(size_t)t * K + __builtin_ctz(left)];
                for (size_t x = 0; x < m; ++x) row[x | m] = mul(row[x], f);
            }
        } else {
            std::vector<wide> a2(n), b2((size_t)n * n, one);
            std::vector<Term> high2;
            int at[32];
            for (uint32_t left = coupled, j = 0; left; left &= left - 1, ++j) {
                at[__builtin_ctz(left)] = (int)j;
                a2[j] = b[(size_t)t * K + __builtin_ctz(left)];
            }
            for (const Term &h : high) {
                if (h.vars >> t != 1) continue;
                uint32_t vars = 0;
                for (uint32_t left = h.vars ^ (1u << t); left; left &= left - 1) vars |= 1u << at[__builtin_ctz(left)];
                if (__builtin_popcount(vars) > 2) {
                    high2.push_back({vars, h.f});
                } else {
                    wide &v = b2[(size_t)(31 - __builtin_clz(vars)) * n + __builtin_ctz(vars)];
                    v = mul(v, h.f);
                }
            }
            form_table(n, a[t], a2.data(), b2.data(), high2, row.data());
        }
        if ((size_t)1 << n == half) {
            for (size_t x = 0; x < half; ++x) out[x | half] = mul(out[x], row[x]);
        } else {
            for (size_t x = 0, r = 0; x < half; ++x) {
                out[x | half] = mul(out[x], row[r]);
                // r: the bits of x + 1 on `coupled`, packed (the step flips the bits up to x's lowest 0)
                r ^= ((size_t)1 << __builtin_popcountll(coupled & (x ^ (x + 1)))) - 1;
            }
        }
    }
}

}  // namespace

std::vector<cplx> diag_product(const std::vector<int> &to, const std::vector<const Operator *> &members,
                               const std::vector<std::array<wide, 2>> &bits)
{
    const int K = (int)to.size();
    if (K > 30) throw std::runtime_error("diag_product: too many qubits");
    std::vector<Operator> own;
    const std::vector<const Operator *> ds = expand_parts(members, own);
    // The form's factors are quotients of the gates' entries, which are of unit
    // modulus.  They and the table are wide: they meet every entry of half a
    // table alike, and in FP64 a 12-qubit QAOA of 5 levels came out 8 times
    // further off (1.4e-14) than by products of the gates' own entries.
    const wide one(1);
    wide c(1);
    std::vector<wide> a(K, one), b((size_t)K * K, one), f;
    for (size_t t = 0; t < bits.size(); ++t) {
        c = mul(c, bits[t][0]);
        a[t] = mul(bits[t][1], std::conj(bits[t][0]) / std::norm(bits[t][0]));
    }
    std::vector<Term> high;
    for (const Operator *d : ds) {
        if (!d->diag) throw std::runtime_error("diag_product: member not diagonal");
        const int k = d->k();
        int pos[32];
        for (int t = 0; t < k; ++t)
            if ((pos[t] = position(to, d->q[t])) < 0) throw std::runtime_error("diag_product: qubit not in target list");
        f.assign(d->m.begin(), d->m.end());
        for (int t = 0; t < k; ++t)
            for (size_t y = 0; y < f.size(); ++y)
                if (!((y >> t) & 1)) {
                    if (f[y] == one) continue;
                    f[y | ((size_t)1 << t)] = mul(f[y | ((size_t)1 << t)], std::conj(f[y]) / std::norm(f[y]));
                }
        for (size_t y = 0; y < f.size(); ++y) {
            if (f[y] == one) continue;
            uint32_t vars = 0;
            for (int t = 0; t < k; ++t) vars |= (uint32_t)((y >> t) & 1) << pos[t];
            const int w = __builtin_popcount(vars);
            if (w > 2) {
                high.push_back({vars, f[y]});
                continue;
            }
            wide &v = w == 0 ? c : w == 1 ? a[__builtin_ctz(vars)]
                                          : b[(size_t)(31 - __builtin_clz(vars)) * K + __builtin_ctz(vars)];
            v = mul(v, f[y]);
        }
    }
    std::vector<wide> out((size_t)1 << K);
    form_table(K, c, a.data(), b.data(), high, out.data());
    return std::vector<cplx>(out.begin(), out.end());
}

std::vector<Operator> parts_of(const Operator &op)
{
    std::vector<Operator> out;
    if (!op.parts) return out;
    out.reserve(op.parts->size());
    for (const Operator &part : *op.parts) {
        out.push_back(part);
        for (int &q : out.back().q) q = op.q[q];
    }
    return out;
}

Shears shears_of(const wide *u)
{
    Shears s;
    s.flip = std::norm(u[0]) < std::norm(u[1]);
    const wide *top = s.flip ? u + 2 : u, *bot = s.flip ? u : u + 2;
    // rows (l0, l0 p r1) and (l1 q, l1 (1 + p q) r1); l1 r1 = det / l0
    s.l[0] = top[0];
    const wide x = mul(top[1], std::conj(top[0])) / std::norm(top[0]);
    const long double p = std::sqrt(std::norm(x));
    s.r1 = p > 0 ? x / p : wide(1);
    const wide l1 = mul(bot[1] - mul(bot[0], x), std::conj(s.r1));
    s.p = (double)p;
    s.q = (double)(mul(bot[0], std::conj(l1)).real() / std::norm(l1));
    s.l[1] = mul(bot[1], std::conj(s.r1)) / (1 + (long double)s.p * s.q);
    return s;
}

bool unit_phases(const Operator &op)
{
    return std::all_of(op.m.begin(), op.m.end(), [](const cplx &x) { return std::abs(std::norm(x) - 1.0) < 4e-15; });
}

bool is_rotation(const Operator &op)
{
    if (op.diag || op.k() != 1) return false;
    // rows orthogonal, so that shears_of finds a real q, and of norm 1, so
    // that the rows of products are orthogonal too (a MATRIX gate may be off
    // by 1e-10)
    return std::norm(mul(op.m[0], std::conj(op.m[2])) + mul(op.m[1], std::conj(op.m[3]))) < 1e-30 &&
           std::abs(std::norm(op.m[0]) + std::norm(op.m[1]) - 1.0) < 4e-15 &&
           std::abs(std::norm(op.m[2]) + std::norm(op.m[3]) - 1.0) < 4e-15;
}

void materialize(Operator &op)
{
    if (!op.parts) return;
    std::vector<int> to(op.q.size());
    std::vector<const Operator *> ds;
    for (size_t i = 0; i < to.size(); ++i) to[i] = (int)i;
    for (const Operator &part : *op.parts) ds.push_back(&part);
    op.m = diag_product(to, ds);
    op.parts.reset();
}

std::vector<cplx> block_product(const std::vector<int> &reg, const std::vector<int> &sel,
                                const std::vector<const Operator *> &members)
{
    const int kr = (int)reg.size(), ks = (int)sel.size();
    std::vector<Operator> own;
    const std::vector<const Operator *> ops = expand_parts(members, own);
    const uint32_t d = 1u << kr;
    std::vector<cplx> out((size_t)d * d << ks, cplx(0.0, 0.0));
    for (uint32_t v = 0; v < (1u << ks); ++v)
        for (uint32_t i = 0; i < d; ++i) out[((size_t)v * d + i) * d + i] = 1.0;
    std::vector<cplx> sub((size_t)d * d), in(d);
    std::vector<uint32_t> off(d);
    for (const Operator *g : ops) {
        const int k = g->k();
        int rp[8], rt[8], nr = 0, sp[8], st[8], ns = 0;  // (position in reg / sel, matrix bit)
        if (k > 8 && !g->diag) throw std::runtime_error("block_product: gate too wide");
        // wide diagonals act entry by entry below; narrow gates by sub-matrices
        uint32_t gmask = 0;
        std::vector<int> where(k);
        for (int t = 0; t < k; ++t) {
            const int r = position(reg, g->q[t]), s = r < 0 ? position(sel, g->q[t]) : -1;
            if (r < 0 && s < 0) throw std::runtime_error("block_product: qubit in neither list");
            where[t] = r >= 0 ? r : kr + s;
            if (r >= 0) gmask |= 1u << r;
            if (!g->diag) {
                if (r >= 0) {
                    rp[nr] = r;
                    rt[nr++] = t;
                } else {
                    sp[ns] = s;
                    st[ns++] = t;
                }
            }
        }
        for (uint32_t v = 0; v < (1u << ks); ++v) {
            cplx *acc = out.data() + (size_t)v * d * d;
            if (g->diag) {
                for (uint32_t i = 0; i < d; ++i) {
                    const uint64_t x = i | ((uint64_t)v << kr);
                    uint64_t y = 0;
                    for (int t = 0; t < k; ++t) y |= ((x >> where[t]) & 1ull) << t;
                    const cplx f = g->m[y];
                    for (uint32_t col = 0; col < d; ++col) acc[i * d + col] = mul(f, acc[i * d + col]);
                }
                continue;
            }
            const uint32_t dn = 1u << nr;
            uint64_t fix = 0;
            for (int u = 0; u < ns; ++u) fix |= (uint64_t)((v >> sp[u]) & 1u) << st[u];
            for (uint32_t r = 0; r < dn; ++r) {
                off[r] = 0;
                uint64_t row = fix;
                for (int u = 0; u < nr; ++u)
                    if ((r >> u) & 1) {
                        off[r] |= 1u << rp[u];
                        row |= 1ull << rt[u];
                    }
                for (uint32_t c = 0; c < dn; ++c) {
                    uint64_t col = fix;
                    for (int u = 0; u < nr; ++u)
                        if ((c >> u) & 1) col |= 1ull << rt[u];
                    sub[r * dn + c] = g->m[(row << k) + col];
                }
            }
            for (uint32_t base = 0; base < d; ++base) {
                if (base & gmask) continue;
                for (uint32_t col = 0; col < d; ++col) {
                    for (uint32_t c = 0; c < dn; ++c) in[c] = acc[(base | off[c]) * d + col];
                    for (uint32_t r = 0; r < dn; ++r) {
                        cplx s(0.0, 0.0);
                        for (uint32_t c = 0; c < dn; ++c) s += mul(sub[r * dn + c], in[c]);
                        acc[(base | off[r]) * d + col] = s;
                    }
                }
            }
        }
    }
    return out;
}

}  // namespace qs
