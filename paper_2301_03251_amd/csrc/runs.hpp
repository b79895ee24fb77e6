// runs.hpp -- plans of the run kernel (host C++, no HIP): small states, one
// workgroup per sample, one 2x2 matrix per run of one-qubit gates.
//
// The state of a sample is held in a workgroup's registers. An amplitude's
// storage index t has n bits: bits [0, log_r) select the register, the next
// six the lane (a storage lane bit is a bit of runs_lane(lane), see kernel),
// the rest the wavefront. A layout is a bit position for every qubit. The
// circuit becomes a list of steps:
//
//   * a layer of runs: a run is the product of consecutive one-qubit gates of a
//     qubit (rotations, H, Paulis) as one 2x2 matrix, applied where the qubit's
//     bit is a register or lane bit; a layer holds at most one per position;
//   * a controlled run: consecutive controlled rotations of one control and
//     target as a pair of matrices, chosen by the control's bit;
//   * an exchange through LDS: any sequence of CNOTs and any change of layout
//     is one linear map over GF(2) of the storage index;
//   * a sign step: any set of CZs between two other steps is one sign per
//     amplitude, from a table.
//
// Runs at the start of the circuit act on |0...0>, where they make a product
// state that the kernel writes directly ("prefix" runs).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "plan.hpp"

namespace qlayer {

enum RunOp : uint32_t {
    RS_CRUN = 0,      // + position of the target's bit: a controlled run
    RS_LAYER_REAL = 14,  // the same with real matrices only (RY and H): half the arithmetic
    RS_LAYER = 15,    // runs on several positions
    RS_EXCHANGE = 16, // through LDS (signs first)
    RS_SIGN = 17,     // signs only
    RS_END = 18,
};

constexpr uint32_t RUNS_NONE = 0xffffffffu;
// Most qubits of a plan: 2^12 amplitudes as 8 registers of 512 threads.
constexpr int RUNS_MAX_QUBITS = 12;
// Most words of the tables (they are held in LDS).
constexpr size_t RUNS_MAX_WORDS = 12288;

struct DevRunStep {
    uint32_t op;
    uint32_t mat;   // controlled run: first complex element of its matrices in the LDS table; layer: of position
                    // 0's (4 per position); exchange: first word of its address table; sign: of its sign table
    uint32_t ctl;   // controlled run: storage thread bit of the control; layer: positions with a run (mask);
                    // exchange: first word of its sign table (RUNS_NONE: no signs)
    uint32_t grad;  // controlled run: index of its three gradient sums; layer: of position 0's (one per position)
};

// One run: members [first, first + count), its matrices at element `mat` of
// the table (4 complex elements: m00, m01, m11, m10; 8 with a control: the
// matrices for control bit 0 and 1), its gradient sums and its members' first
// (cos, sin) pair (one pair per member, two with a control).
struct DevRunEntry {
    int32_t first, count;
    int32_t controlled;
    uint32_t mat, grad;
    int32_t cs;
    int32_t layer_first, layer_end;  // matrices (of 4 elements) of its step
};

// One gate of a run, in circuit order. kind K_H, K_RX, K_RY, K_RZ or K_PAULI;
// slot of its angle (H: -1), whose source, index and scale are repeated here
// (one load less in the chain to the angle). A controlled rotation has the two
// half-angle slots of its rewriting (scales +1/2 and -1/2): its angle is slot
// + slot2 for control bit 0 and slot - slot2 for control bit 1. `cs` is the
// index of its (cos, sin) pairs.
struct DevRunMember {
    int32_t slot, slot2;  // read as a pair
    int32_t kind, cs;
    int32_t src, index;
    double scale;
};

static_assert(offsetof(DevRunMember, slot) % 8 == 0 && offsetof(DevRunMember, slot2) == offsetof(DevRunMember, slot) + 4 &&
                  sizeof(DevRunMember) % 8 == 0,
              "a member's slots are read as one aligned pair");

// A step as the kernel reads it: op | mat << 8, and for a run or layer ctl |
// grad << 9, for an exchange its sign table + 1 (0: no signs).
struct RunRecord {
    uint32_t x, y;
};
constexpr RunRecord run_record(const DevRunStep& s) {
    return {s.op | s.mat << 8, s.op < RS_EXCHANGE ? s.ctl | s.grad << 9 : s.op == RS_EXCHANGE ? s.ctl + 1u : 0u};
}

struct RunPlan {
    bool ok = false;
    int n = 0, log_r = 0, log_t = 0;       // 2^log_t threads hold amplitudes (a launch has at least 64)
    int n_waves = 1;
    int n_pos = 0;                         // positions a run can have: registers and lanes
    std::vector<DevRunStep> steps;         // RS_END last
    uint32_t prefix = 0;                   // positions with a prefix run: a layer of its own, matrices and sums at 0
    std::vector<DevRunEntry> entries;
    std::vector<DevRunMember> members;
    // Tables. Exchange: 64 + n_waves + log_r words; amplitude (lane, wavefront,
    // register) goes to the LDS slot that is the XOR of its lane's word, its
    // wavefront's and those of its set register bits (slots are register-major:
    // register << log_t | thread, then spread over the LDS banks by runs_bank).
    // Signs: one byte per thread, bit i: register i is negated.
    std::vector<uint32_t> words;
    std::vector<int32_t> first_qubit, last_qubit;  // [n] qubit at each position, first and last layout
    int n_mat = 0;                         // complex elements of the matrix table
    int n_cs = 0;                          // (cos, sin) pairs
    int n_grads = 0;                       // gradient sums (three each)
    int n_exchanges = 0;
    bool controlled = false;               // has runs under a control
};

// Bank-spreading permutation of the exchange slots, linear over GF(2): folds
// the higher bits into the lowest four.
constexpr uint32_t runs_bank(uint32_t s) { return s ^ (((s >> 4) ^ (s >> 8)) & 15u); }

// Register bits of a plan: one wavefront while 4 registers hold the state (n
// <= 8), 4 registers up to 11 qubits, 8 where workgroups get large: 12 qubits
// (1024 threads left room for one workgroup per CU: 1000 samples forward,
// complex64, 90 against 74 us) and 11 in complex128 (64 against 57 us; in
// complex64 4 registers step 45 against 49 us at 37 samples).
constexpr int runs_log_regs(int n, int dtype) {
    return n <= 6 ? 0 : n == 7 ? 1 : n <= 10 || (n == 11 && dtype == 0) ? 2 : 3;
}

// Plan a circuit of at most RUNS_MAX_QUBITS qubits for 2^log_r registers (ok =
// false: too long).
void build_run_plan(const Circuit& c, int log_r, RunPlan& out);

}  // namespace qlayer
