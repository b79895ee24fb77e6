// runs.cpp -- the planner of the run kernel (see runs.hpp).
#include "runs.hpp"

#include <algorithm>

namespace qlayer {

namespace {

struct Item {
    enum Type { ONE, CNOT, CZ, CR } type;
    int q0, q1;  // CNOT, CR: control, target
    DevRunMember m;
};

// The circuit's gates with every controlled rotation as one item again.
std::vector<Item> items_of(const Circuit& c) {
    std::vector<Item> out;
    auto member = [&](const Gate& g, int slot2) {
        const double scale = g.slot >= 0 ? c.slots[g.slot].scale : 1.0;
        const int src = g.slot >= 0 ? c.slots[g.slot].src : (int)S_NONE;
        return DevRunMember{g.slot, slot2, g.kind, 0, src, g.index, scale};
    };
    for (size_t i = 0; i < c.gates.size(); i++) {
        const Gate& g = c.gates[i];
        if (i + 3 < c.gates.size() && c.gates[i + 3].user == g.user) {  // R(t/2) E R(-t/2) E
            const Gate& e = c.gates[i + 1];
            out.push_back({Item::CR, e.q0, e.q1, member(g, c.gates[i + 2].slot)});
            i += 3;
        } else if (g.kind == K_CNOT || g.kind == K_CZ) {
            out.push_back({g.kind == K_CNOT ? Item::CNOT : Item::CZ, g.q0, g.q1, {}});
        } else {
            out.push_back({Item::ONE, g.q0, -1, member(g, -1)});
        }
    }
    return out;
}

struct Planner {
    const Circuit& c;
    RunPlan& p;
    std::vector<Item> items;
    size_t now = 0;                                  // item being placed
    std::vector<int> at;                             // qubit -> position
    std::vector<std::vector<DevRunMember>> pend;     // open run of each qubit
    struct Open {
        int c = -1, t = -1;
        std::vector<DevRunMember> m;
    };
    std::vector<Open> open;                          // open controlled runs
    std::vector<Item> ent;                           // CNOTs and CZs not yet applied
    uint32_t ent_q = 0, touched = 0;                 // qubits of `ent`; qubits any step or entangler has touched
    int layer = -1;                                  // open layer: the last step, while only runs are added
    std::vector<std::vector<int>> uses;              // per qubit: items at which a run of it is due

    Planner(const Circuit& c_, RunPlan& p_) : c(c_), p(p_) {}

    int lanes_end() const { return std::min(p.n, p.log_r + 6); }
    bool on_wave(int q) const { return at[q] >= p.log_r + 6; }

    // Items at which a run of q has to be applied: the two-qubit gates on q
    // that follow a one-qubit gate on q (its run is due there), and the
    // controlled rotations with target q.
    void find_uses() {
        uses.assign(p.n, {});
        std::vector<char> has(p.n, 0);
        for (size_t i = 0; i < items.size(); i++) {
            const Item& it = items[i];
            if (it.type == Item::ONE) {
                has[it.q0] = 1;
                continue;
            }
            for (int q : {it.q0, it.q1}) {
                if (has[q] || (it.type == Item::CR && q == it.q1)) uses[q].push_back((int)i);
                has[q] = 0;
            }
        }
        for (int q = 0; q < p.n; q++)
            if (has[q]) uses[q].push_back((int)items.size() + q);
    }
    int next_use(int q) const {
        auto it = std::lower_bound(uses[q].begin(), uses[q].end(), (int)now);
        return it == uses[q].end() ? (1 << 30) : *it;
    }
    // whether q is the control of a controlled rotation soon (registers are
    // not for those)
    int next_control(int q) const {
        for (size_t i = now; i < items.size(); i++)
            if (items[i].type == Item::CR && items[i].q0 == q) return (int)i;
        return 1 << 30;
    }

    // Positions for every qubit: the qubits whose runs are due last on
    // wavefront bits (never those of `near`), registers for qubits that are no
    // control soon (never those of `no_reg`), the qubits due first on the
    // lane bits whose partners cost least (0-3).
    std::vector<int> layout(uint32_t near, uint32_t no_reg) const {
        const int w = std::max(0, p.n - p.log_r - 6);
        std::vector<int> q(p.n), pos(p.n, -1);
        for (int i = 0; i < p.n; i++) q[i] = i;
        std::vector<int> use(p.n), ctl(p.n);
        for (int i = 0; i < p.n; i++) {
            use[i] = (near >> i & 1u) ? -1 : next_use(i);
            ctl[i] = (no_reg >> i & 1u) ? -1 : next_control(i);
        }
        std::stable_sort(q.begin(), q.end(), [&](int a, int b) { return use[a] > use[b]; });
        for (int i = 0; i < w; i++) pos[q[i]] = p.log_r + 6 + i;
        std::vector<int> rest(q.begin() + w, q.end());  // due last first
        std::vector<int> byctl = rest;
        std::stable_sort(byctl.begin(), byctl.end(), [&](int a, int b) { return ctl[a] > ctl[b]; });
        for (int i = 0; i < p.log_r; i++) pos[byctl[i]] = i;
        int next = lanes_end() - 1;
        for (int x : rest)
            if (pos[x] < 0) pos[x] = next--;
        return pos;
    }

    // LDS bank columns of the lanes under the exchange from layout `at` to
    // `to`: how many of the lane bits 0..2 (16-byte amplitudes, 8 bank groups)
    // and 0..3 (8-byte ones, 16) fall on independent bank bits. The other side
    // of an exchange, contiguous in the thread index, has no conflicts.
    int bank_rank(const std::vector<int>& to) const {
        int score = 0;
        for (int nb : {3, 4}) {
            uint32_t basis[4] = {0, 0, 0, 0};
            int rank = 0;
            for (int b = 0; b < std::min(nb, p.log_t); b++) {
                uint32_t v = runs_bank(slot_of(map(1u << qubit_at(p.log_r + b)), to)) & ((1u << nb) - 1u);
                for (int k = nb - 1; k >= 0 && v; k--)
                    if (v >> k & 1u) {
                        if (basis[k]) {
                            v ^= basis[k];
                        } else {
                            basis[k] = v;
                            rank++;
                            v = 0;
                        }
                    }
            }
            score += rank;
        }
        return score;
    }
    int qubit_at(int pos) const { return (int)(std::find(at.begin(), at.end(), pos) - at.begin()); }
    uint32_t map(uint32_t j) const {  // the pending CNOTs on an amplitude index
        for (const Item& it : ent)
            if (it.type == Item::CNOT) j ^= (j >> it.q0 & 1u) << it.q1;
        return j;
    }
    // LDS slot of amplitude j in layout `to`: register-major
    uint32_t slot_of(uint32_t j, const std::vector<int>& to) const {
        uint32_t t = 0;
        for (int q = 0; q < p.n; q++) t |= (j >> q & 1u) << to[q];
        return (t & ((1u << p.log_r) - 1u)) << p.log_t | t >> p.log_r;
    }
    // `to` with its lane positions permuted for the fewest bank conflicts of
    // the move there (a fixed sequence of trial swaps)
    std::vector<int> spread(std::vector<int> to) const {
        const int lo = p.log_r, hi = lanes_end(), full = std::min(3, p.log_t) + std::min(4, p.log_t);
        int best = bank_rank(to);
        for (int round = 0; round < 2 && best < full; round++)
            for (int i = lo; i < hi && best < full; i++)
                for (int j = i + 1; j < hi && best < full; j++) {
                    std::vector<int> t = to;
                    for (int& x : t) x = x == i ? j : x == j ? i : x;
                    const int r = bank_rank(t);
                    if (r > best) {
                        best = r;
                        to = t;
                    }
                }
        return to;
    }

    // Apply the pending entanglers and move to layout `to` (null: stay, if
    // nothing has to move).
    void settle(const std::vector<int>* want) {
        layer = -1;
        const std::vector<int> to = want ? spread(*want) : at;
        bool cnots = false;
        for (const Item& it : ent) cnots |= it.type == Item::CNOT;
        const int T = 1 << p.log_t, R = 1 << p.log_r;
        const bool signs = !ent.empty() && std::any_of(ent.begin(), ent.end(), [](const Item& i) { return i.type == Item::CZ; });
        const bool move = cnots || to != at;
        auto amp_of = [&](uint32_t t, const std::vector<int>& pos) {
            uint32_t j = 0;
            for (int q = 0; q < p.n; q++) j |= (t >> pos[q] & 1u) << q;
            return j;
        };
        auto bank_slot = [&](uint32_t j) { return runs_bank(slot_of(j, to)); };
        auto image = [&](uint32_t j, uint32_t& neg) {
            neg = 0;
            for (const Item& it : ent) {
                if (it.type == Item::CNOT) j ^= (j >> it.q0 & 1u) << it.q1;
                else neg ^= j >> it.q0 & j >> it.q1 & 1u;
            }
            return j;
        };
        if (signs || move) {
            DevRunStep s{move ? RS_EXCHANGE : RS_SIGN, 0, RUNS_NONE, RUNS_NONE};
            uint32_t sign_at = RUNS_NONE, neg;
            if (signs) {
                sign_at = (uint32_t)p.words.size();
                p.words.resize(sign_at + (size_t)(T + 3) / 4, 0);
                for (int t = 0; t < T; t++)
                    for (int i = 0; i < R; i++) {
                        image(amp_of((uint32_t)(t << p.log_r | i), at), neg);
                        p.words[sign_at + t / 4] |= neg << (8 * (t % 4) + i);
                    }
            }
            if (move) {
                s.ctl = sign_at;
                s.mat = (uint32_t)p.words.size();
                // linear over GF(2): the parts of the lane, the wavefront and the register bits
                for (int l = 0; l < 64; l++)
                    p.words.push_back(l < T ? bank_slot(map(amp_of((uint32_t)l << p.log_r, at))) : 0u);
                for (int w = 0; w < p.n_waves; w++)
                    p.words.push_back(bank_slot(map(amp_of((uint32_t)w << (p.log_r + 6), at))));
                for (int m = 0; m < p.log_r; m++)
                    p.words.push_back(bank_slot(map(amp_of(1u << m, at))));
                p.n_exchanges++;
            } else {
                s.mat = sign_at;
            }
            p.steps.push_back(s);
        }
        ent.clear();
        ent_q = 0;
        at = to;
    }

    void emit(int q, int ctl, std::vector<DevRunMember>& m) {
        DevRunEntry e{};
        e.first = (int)p.members.size();
        e.count = (int)m.size();
        e.controlled = ctl >= 0;
        e.cs = p.n_cs;
        bool rot = false, real = true;
        for (DevRunMember x : m) {
            x.cs = p.n_cs;
            p.n_cs += ctl >= 0 ? 2 : 1;
            real &= x.kind == K_RY || x.kind == K_H;
            rot |= x.kind == K_RX || x.kind == K_RY || x.kind == K_RZ;
            p.members.push_back(x);
        }
        const uint32_t qs = 1u << q | (ctl >= 0 ? 1u << ctl : 0u), bit = 1u << at[q];
        if (ctl >= 0) {
            layer = -1;
            e.mat = (uint32_t)p.n_mat;
            p.n_mat += 8;
            e.grad = (uint32_t)p.n_grads++;
            p.controlled = true;
            e.layer_first = (int)e.mat / 4;
            e.layer_end = e.layer_first + 2;
            p.steps.push_back({RS_CRUN + (uint32_t)at[q], e.mat, (uint32_t)(at[ctl] - p.log_r), e.grad});
        } else if (c.embed == E_NONE && !(touched & qs) && p.n_exchanges == 0) {
            p.prefix |= bit;
            e.mat = 4u * (uint32_t)at[q];
            e.grad = (uint32_t)at[q];
        } else {
            if (layer < 0 || (p.steps[layer].ctl & bit)) {
                layer = (int)p.steps.size();
                p.steps.push_back({RS_LAYER_REAL, (uint32_t)p.n_mat, 0, (uint32_t)p.n_grads});
                p.n_mat += 4 * p.n_pos;
                p.n_grads += p.n_pos;
            }
            DevRunStep& s = p.steps[layer];
            s.ctl |= bit;
            e.mat = s.mat + 4u * (uint32_t)at[q];
            e.layer_first = (int)s.mat / 4;
            e.layer_end = e.layer_first + p.n_pos;
            e.grad = s.grad + (uint32_t)at[q];
        }
        if (!rot) e.grad = RUNS_NONE;
        if (ctl < 0 && !real)  // a complex matrix makes its layer a complex one
            for (DevRunStep& s : p.steps)
                if (s.op == RS_LAYER_REAL && s.mat <= e.mat && e.mat < s.mat + 4u * (uint32_t)p.n_pos) s.op = RS_LAYER;
        touched |= qs;
        p.entries.push_back(e);
        m.clear();
    }

    void flush(int q) {
        if (pend[q].empty()) return;
        if ((ent_q >> q & 1u) || on_wave(q)) {
            // a change of layout only when something has to move
            bool cnots = false;
            for (const Item& it : ent) cnots |= it.type == Item::CNOT;
            const std::vector<int> to = layout(1u << q, 0);
            settle(on_wave(q) || cnots ? &to : nullptr);
        }
        emit(q, -1, pend[q]);
    }

    void close(size_t i) {
        Open o = std::move(open[i]);
        open.erase(open.begin() + (long)i);
        const uint32_t qs = 1u << o.c | 1u << o.t;
        const bool bad = on_wave(o.t) || at[o.c] < p.log_r;
        if ((ent_q & qs) || bad) {
            bool cnots = false;
            for (const Item& it : ent) cnots |= it.type == Item::CNOT;
            const std::vector<int> to = layout(1u << o.t, 1u << o.c);
            settle(bad || cnots ? &to : nullptr);
        }
        emit(o.t, o.c, o.m);
    }
    void close_on(int q) {
        for (size_t i = 0; i < open.size();)
            if (open[i].c == q || open[i].t == q) close(i);
            else i++;
    }

    // whether every gate of q's open run commutes with a CNOT's control or a
    // CZ (K_RZ), or with a CNOT's target (K_RX)
    bool only(int q, int kind) const {
        for (const DevRunMember& m : pend[q])
            if (m.kind != kind) return false;
        return true;
    }

    void entangle(const Item& it) {
        ent.push_back(it);
        ent_q |= 1u << it.q0 | 1u << it.q1;
        touched |= 1u << it.q0 | 1u << it.q1;
    }

    void run() {
        items = items_of(c);
        find_uses();
        pend.resize(p.n);
        p.n_pos = lanes_end();
        p.n_mat = 4 * p.n_pos;  // the prefix layer's
        p.n_grads = p.n_pos;
        at = layout(0, 0);
        p.first_qubit.assign(p.n, 0);
        for (int q = 0; q < p.n; q++) p.first_qubit[at[q]] = q;
        for (now = 0; now < items.size(); now++) {
            const Item& it = items[now];
            if (it.type == Item::ONE) {
                close_on(it.q0);
                pend[it.q0].push_back(it.m);
            } else if (it.type == Item::CR) {
                size_t i = 0;
                while (i < open.size() && !(open[i].c == it.q0 && open[i].t == it.q1)) i++;
                if (i == open.size()) {
                    close_on(it.q0);
                    close_on(it.q1);
                    if (!only(it.q0, K_RZ)) flush(it.q0);
                    flush(it.q1);
                    open.push_back({it.q0, it.q1, {}});
                    i = open.size() - 1;
                }
                open[i].m.push_back(it.m);
            } else {
                close_on(it.q0);
                close_on(it.q1);
                if (!only(it.q0, K_RZ)) flush(it.q0);
                if (!only(it.q1, it.type == Item::CNOT ? K_RX : K_RZ)) flush(it.q1);
                entangle(it);
            }
        }
        while (!open.empty()) close(0);
        for (int q = 0; q < p.n; q++)
            if (!on_wave(q)) flush(q);
        for (int q = 0; q < p.n; q++) flush(q);
        if (!ent.empty()) settle(nullptr);
        p.last_qubit.assign(p.n, 0);
        for (int q = 0; q < p.n; q++) p.last_qubit[at[q]] = q;
        p.steps.push_back({RS_END, 0, 0, 0});
    }
};

}  // namespace

void build_run_plan(const Circuit& c, int log_r, RunPlan& out) {
    out = RunPlan{};
    if (c.n > RUNS_MAX_QUBITS || c.gates.size() > (1u << 14)) return;
    out.n = c.n;
    out.log_r = log_r;
    out.log_t = c.n - out.log_r;
    out.n_waves = out.log_t > 6 ? 1 << (out.log_t - 6) : 1;
    Planner(c, out).run();
    out.ok = out.words.size() <= RUNS_MAX_WORDS && out.n_mat < (1 << 16);
}

}  // namespace qlayer
