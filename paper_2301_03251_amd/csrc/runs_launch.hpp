// runs_launch.hpp -- host-side launcher of the run kernel (runs.hip).
#pragma once

#include "launch.hpp"
#include "runs.hpp"

namespace qlayer {

// LDS of a run-kernel workgroup, as byte offsets after the exchange buffers.
struct RunLds {
    uint32_t alt;    // bytes from one exchange buffer to the next (0: only one, used with two barriers)
    uint32_t lam;    // bytes from psi's part of an exchange buffer to lambda's
    uint32_t mat, cs, kind, scale, words, norm, red, go, sum, gs;
    uint32_t total;
};

// One workgroup per circuit of the call.
struct RunArgs {
    const uint2* steps;            // [n_steps + 1] packed (run_record)
    const DevRunEntry* entries;    // [n_entries]
    const DevRunMember* members;   // [n_members]
    const uint32_t* words;         // [n_words] address and sign tables
    const SlotSrc* slots;
    const int32_t* x_ptr;          // [F+1] CSR: rotation slots bound to input f
    const int32_t* x_slot;
    const int32_t* w_ptr;          // [P+1] CSR: rotation slots bound to weight p
    const int32_t* w_slot;
    const void* inputs;            // [.][F] Real
    const void* weights;           // [P] Real
    const void* grad_out;          // [B][n] Real
    void* expz;                    // [B][n] Real or null
    void* psi_out;                 // [B][2^n] complex or null
    void* grad_inputs;             // [B][F] Real or null
    void* grad_weights;            // [P] Real: the weight gradients of a single sample, or null
    double* gpart;                 // [n_slots][B]: the weight slots' terms, or null
    int64_t B, v0;
    int32_t vper, bwd;
    int32_t n, log_t, F, P, n_slots;
    int32_t n_steps, n_entries, n_members, n_words, n_mats;
    int32_t embed, first;          // initial state (E_*) and its first feature
    uint64_t first_qubit, last_qubit;  // qubit of every position, four bits each: first and last layout
    uint32_t prefix;                   // positions with a prefix run (matrices and sums of layer 0)
    RunLds lds;
};

// LDS of a plan's launches.
RunLds runs_lds(int dtype, const RunPlan& p, int n_slots, bool bwd);
hipError_t launch_runs(int dtype, int log_r, const RunArgs& a, int threads, hipStream_t s);
hipError_t configure_runs_kernels(size_t max_lds);

}  // namespace qlayer
