// Host-only check of the run kernel's plans, built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_run_plans.py: every circuit of a
// binary file (records as in planner_driver.cpp) is planned and its steps are
// carried out on a state of complex<double> as the kernel does, forward and
// back, and compared with the circuit's gates applied one by one.
#include <cmath>
#include <complex>
#include <cstdio>
#include <vector>

#include "runs.hpp"

using namespace qlayer;
using C = std::complex<double>;

namespace {

double angle(int slot) { return 0.3 + 0.77 * slot - 0.0013 * slot * slot; }

struct M2 {
    C a[4];  // m00 m01 m10 m11
};
M2 mul(const M2& x, const M2& y) {
    return {{x.a[0] * y.a[0] + x.a[1] * y.a[2], x.a[0] * y.a[1] + x.a[1] * y.a[3],
             x.a[2] * y.a[0] + x.a[3] * y.a[2], x.a[2] * y.a[1] + x.a[3] * y.a[3]}};
}
M2 gate(int kind, double th, int which) {
    const C i(0, 1);
    const double c = std::cos(th / 2), s = std::sin(th / 2), r = std::sqrt(0.5);
    switch (kind) {
        case K_H: return {{r, r, r, -r}};
        case K_RX: return {{c, -i * s, -i * s, c}};
        case K_RY: return {{c, -s, s, c}};
        case K_RZ: return {{C(c, -s), 0, 0, C(c, s)}};
        default:
            if (which == 1) return {{0, 1, 1, 0}};
            if (which == 2) return {{0, -i, i, 0}};
            if (which == 3) return {{1, 0, 0, -1}};
            return {{1, 0, 0, 1}};
    }
}

int fail(int n_case, const char* what) {
    std::printf("case %d: %s\n", n_case, what);
    return 1;
}

int check(int n_case, const Circuit& c, const RunPlan& p, long& exchanges, long& runs) {
    const int n = c.n, N = 1 << n, T = 1 << p.log_t, R = 1 << p.log_r;
    std::vector<C> want(N, 0), st(N, 0);
    want[0] = 1;
    if (c.embed != E_NONE)
        for (int j = 0; j < N; j++) want[j] = C(std::sin(1.0 + j), std::cos(3.0 * j));
    std::vector<C> start = want;
    for (const Gate& g : c.gates) {
        if (g.kind == K_CNOT || g.kind == K_CZ) {
            for (int j = 0; j < N; j++) {
                if (g.kind == K_CZ && (j >> g.q0 & j >> g.q1 & 1)) want[j] = -want[j];
                if (g.kind == K_CNOT && (j >> g.q0 & 1) && !(j >> g.q1 & 1)) std::swap(want[j], want[j | 1 << g.q1]);
            }
            continue;
        }
        const M2 m = gate(g.kind, g.slot >= 0 ? angle(g.slot) : 0, g.slot >= 0 ? g.slot % 4 : 0);
        for (int j = 0; j < N; j++)
            if (!(j >> g.q0 & 1)) {
                const C u = want[j], v = want[j | 1 << g.q0];
                want[j] = m.a[0] * u + m.a[1] * v;
                want[j | 1 << g.q0] = m.a[2] * u + m.a[3] * v;
            }
    }
    // the matrix table
    std::vector<C> mat(p.n_mat, C(NAN, NAN));
    std::vector<char> cs_used(p.n_cs, 0);
    for (const DevRunEntry& e : p.entries)
        for (int v = 0; v < (e.controlled ? 2 : 1); v++) {
            M2 m{{1, 0, 0, 1}};
            for (int k = 0; k < e.count; k++) {
                const DevRunMember& x = p.members.at(e.first + k);
                const int at = x.cs + v;
                if (at >= p.n_cs || cs_used[at]++) return fail(n_case, "angle pair index");
                double th = x.slot >= 0 ? angle(x.slot) : 0;
                if (e.controlled) th += v ? -angle(x.slot2) : angle(x.slot2);
                m = mul(gate(x.kind, th, x.slot >= 0 ? x.slot % 4 : 0), m);
            }
            const C rows[4] = {m.a[0], m.a[1], m.a[3], m.a[2]};
            for (int i = 0; i < 4; i++) mat.at(e.mat + 4 * v + i) = rows[i];
        }
    // storage index: (thread << log_r | register)
    auto amp_of = [&](int t, const std::vector<int32_t>& q) {
        int j = 0;
        for (int b = 0; b < n; b++) j |= (t >> b & 1) << q[b];
        return j;
    };
    if (c.embed != E_NONE) {
        for (int t = 0; t < N; t++) st[t] = start[amp_of(t, p.first_qubit)];
    } else {
        for (int t = 0; t < N; t++) {
            C a = 1;
            for (int b = 0; b < n; b++) {
                const bool one = t >> b & 1;
                if (!(p.prefix >> b & 1)) a *= one ? 0.0 : 1.0;
                else a *= mat.at(4 * b + (one ? 3 : 0));
            }
            st[t] = a;
        }
    }
    const std::vector<C> init = st;
    auto sign = [&](uint32_t at, int th, int r) {
        return p.words.at(at + th / 4) >> (8 * (th % 4) + r) & 1u;
    };
    std::vector<int> unbank(N, -1);  // LDS slot -> register-major storage index
    for (int v = 0; v < N; v++) unbank.at(runs_bank((uint32_t)v)) = v;
    for (int v : unbank)
        if (v < 0) return fail(n_case, "bank permutation");
    auto slot = [&](uint32_t at, int th, int r) {
        uint32_t w = p.words.at(at + (th & 63)) ^ p.words.at(at + 64 + (th >> 6));
        for (int m = 0; m < p.log_r; m++)
            if (r >> m & 1) w ^= p.words.at(at + 64 + p.n_waves + m);
        return (int)w;
    };
    auto step = [&](const DevRunStep& s, bool back) {
        if (s.op == RS_SIGN || s.op == RS_EXCHANGE) {
            const uint32_t sg = s.op == RS_SIGN ? s.mat : s.ctl;
            std::vector<C> o(N, C(NAN, NAN));
            for (int th = 0; th < T; th++)
                for (int r = 0; r < R; r++) {
                    const int t = th << p.log_r | r;
                    int u = t;
                    if (s.op == RS_EXCHANGE) {
                        const int w = unbank.at((size_t)slot(s.mat, th, r));
                        u = (w & (T - 1)) << p.log_r | w >> p.log_t;
                    }
                    const double f = sg != RUNS_NONE && sign(sg, th, r) ? -1 : 1;
                    if (back) o[t] = f * st.at(u);
                    else o.at(u) = f * st[t];
                }
            st = o;
            exchanges += s.op == RS_EXCHANGE;
            return;
        }
        auto apply = [&](int pos, uint32_t at, int ctl) {
            for (int t = 0; t < N; t++)
                if (!(t >> pos & 1)) {
                    const uint32_t e = at + (ctl >= 0 ? ((uint32_t)(t >> p.log_r) >> ctl & 1u) * 4 : 0u);
                    C m00 = mat.at(e), m01 = mat.at(e + 1), m11 = mat.at(e + 2), m10 = mat.at(e + 3);
                    if (s.op == RS_LAYER_REAL)  // the kernel reads the real parts only
                        for (C* m : {&m00, &m01, &m11, &m10}) *m = m->real();
                    if (back) {
                        m00 = std::conj(m00);
                        m11 = std::conj(m11);
                        const C x = std::conj(m01);
                        m01 = std::conj(m10);
                        m10 = x;
                    }
                    const C u = st[t], v = st[t | 1 << pos];
                    st[t] = m00 * u + m01 * v;
                    st[t | 1 << pos] = m10 * u + m11 * v;
                }
            runs++;
        };
        if (s.op == RS_LAYER || s.op == RS_LAYER_REAL) {
            for (int pos = 0; pos < p.n_pos; pos++)
                if (s.ctl >> pos & 1) apply(pos, s.mat + 4 * pos, -1);
        } else {
            apply((int)s.op - RS_CRUN, s.mat, (int)s.ctl);
        }
    };
    if (p.steps.empty() || p.steps.back().op != RS_END) return fail(n_case, "no end");
    const int S = (int)p.steps.size() - 1;
    // matrices are numbered in the order of the steps, and a run knows its step's
    int next = p.n_pos;
    for (int i = 0; i < S; i++) {
        const DevRunStep& s = p.steps[i];
        if (s.op >= RS_EXCHANGE) continue;
        const int first = (int)s.mat / 4, end = first + (s.op < RS_LAYER_REAL ? 2 : p.n_pos);
        if (first != next) return fail(n_case, "order of the matrices");
        next = end;
        for (const DevRunEntry& e : p.entries)
            if ((int)e.mat / 4 >= first && (int)e.mat / 4 < end && (e.layer_first != first || e.layer_end != end))
                return fail(n_case, "matrices of a run's step");
    }
    if (4 * next != p.n_mat) return fail(n_case, "number of matrices");
    for (int i = 0; i < S; i++) {
        const DevRunStep& s = p.steps[i];
        if (s.op < RS_LAYER_REAL && ((int)s.op >= p.n_pos || (int)s.ctl >= p.log_t)) return fail(n_case, "controlled run's positions");
        if ((s.op == RS_LAYER || s.op == RS_LAYER_REAL) && s.ctl >> p.n_pos) return fail(n_case, "run on a wavefront bit");
        step(s, false);
    }
    for (int t = 0; t < N; t++)
        if (std::abs(st[t] - want[amp_of(t, p.last_qubit)]) > 1e-11 * (c.embed ? N : 1))
            return fail(n_case, "forward state differs");
    for (int i = S - 1; i >= 0; i--) step(p.steps[i], true);
    for (int t = 0; t < N; t++)
        if (!(std::abs(st[t] - init[t]) < 1e-11 * (c.embed ? N : 1))) return fail(n_case, "backward state differs");
    return 0;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    FILE* f = std::fopen(argv[1], "rb");
    if (!f) return 2;
    int n_cases = 0;
    long exchanges = 0, runs = 0;
    for (;;) {
        int32_t hdr[8];
        if (std::fread(hdr, sizeof(int32_t), 8, f) != 8) break;
        std::vector<int32_t> g((size_t)hdr[1] * 5);
        std::vector<double> pp((size_t)hdr[6] * 3);
        if (hdr[1] && std::fread(g.data(), sizeof(int32_t), g.size(), f) != g.size()) return 3;
        if (hdr[6] && std::fread(pp.data(), sizeof(double), pp.size(), f) != pp.size()) return 3;
        Extras ext;
        ext.embed = hdr[4];
        ext.embed_first = hdr[5];
        ext.pauli_p = hdr[6] ? pp.data() : nullptr;
        Circuit c;
        const std::string err = build_circuit(hdr[0], g.data(), hdr[1], hdr[2], hdr[3], ext, Options{}, c);
        if (!err.empty()) {
            std::printf("case %d: %s\n", n_cases, err.c_str());
            return 4;
        }
        const long x0 = exchanges, r0 = runs;
        RunPlan p;
        for (int dt = 1; dt >= 0; dt--) {
            if (dt == 1 && runs_log_regs(c.n, 0) == runs_log_regs(c.n, 1)) continue;
            build_run_plan(c, runs_log_regs(c.n, dt), p);
            if (!p.ok) return fail(n_cases, "no plan");
            if (check(n_cases, c, p, exchanges, runs)) return 5;
        }
        if (argc > 2)
            std::printf("case %d: n %d gates %d: %ld exchanges, %ld runs, %d prefix, %zu words, %zu steps\n", n_cases, hdr[0], hdr[1],
                        (exchanges - x0) / 2, (runs - r0) / 2, __builtin_popcount(p.prefix), p.words.size(), p.steps.size());
        n_cases++;
    }
    std::printf("cases %d exchanges %ld runs %ld\n", n_cases, exchanges, runs);
    return 0;
}
