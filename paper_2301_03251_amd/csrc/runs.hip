// runs.hip -- the run kernel k_runs (gfx950): small states, one workgroup per
// sample, the whole forward + adjoint of a sample in one launch.
//
// What bounds it: a small batch leaves each SIMD one or two wavefronts, so a
// step costs its instructions' latency, and the number of steps is what
// counts. A step is a whole run of one-qubit gates (one 2x2 matrix, formed per
// sample in fp64 by the workgroup itself), a whole group of CNOTs (one linear
// permutation through LDS) or a whole group of CZs (one sign per amplitude);
// see runs.hpp. A run on a lane bit gets its partner amplitudes by one DPP
// move, so most runs need no layout change at all. The gradients of all
// rotations of a run come from the three sums Im <lambda| P |psi>, P = X, Y, Z
// on its qubit, taken once after the run: un-applying its gates one by one
// rotates the three sums like the axes of the Bloch sphere (in fp64).
#include "kcommon.hpp"
#include "runs_launch.hpp"

namespace qlayer {
namespace {

// Storage lane bits: bit b of runs_lane(lane) is flipped alone by the lane move
// xor 1, 2, 7, 8, 16, 32 for b = 0..5 (7 = the half-row mirror, a single DPP
// move where xor 4 would take two).
__device__ __forceinline__ int runs_lane(int lane) { return lane ^ ((lane & 4) ? 3 : 0); }

template <int B>
__device__ __forceinline__ uint32_t partner_u32(uint32_t v, int lane) {
    if constexpr (B < 4) {
        constexpr int CTRL = B == 0 ? 0xB1 : B == 1 ? 0x4E : B == 2 ? 0x141 : 0x128;  // ..., row_ror:8
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
    } else {
        const auto r = B == 4 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                              : __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return ((lane >> B) & 1) ? r[0] : r[1];
    }
}
template <int B>
__device__ __forceinline__ float partner(float v, int lane) {
    return __builtin_bit_cast(float, partner_u32<B>(__builtin_bit_cast(uint32_t, v), lane));
}
template <int B>
__device__ __forceinline__ double partner(double v, int lane) {
    uint2 u = __builtin_bit_cast(uint2, v);
    u.x = partner_u32<B>(u.x, lane);
    u.y = partner_u32<B>(u.y, lane);
    return __builtin_bit_cast(double, u);
}

// Trade register bit 0 for lane bit B (4 or 5): one permlane swap per word of
// a register pair.
template <int B>
__device__ __forceinline__ void swap_words(uint32_t& lo, uint32_t& hi) {
    const auto r = B == 4 ? __builtin_amdgcn_permlane16_swap(lo, hi, false, false)
                          : __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
    lo = r[0];
    hi = r[1];
}
template <int B>
__device__ __forceinline__ void swap_real(float& lo, float& hi) {
    uint32_t l = __builtin_bit_cast(uint32_t, lo), h = __builtin_bit_cast(uint32_t, hi);
    swap_words<B>(l, h);
    lo = __builtin_bit_cast(float, l);
    hi = __builtin_bit_cast(float, h);
}
template <int B>
__device__ __forceinline__ void swap_real(double& lo, double& hi) {
    uint2 l = __builtin_bit_cast(uint2, lo), h = __builtin_bit_cast(uint2, hi);
    swap_words<B>(l.x, h.x);
    swap_words<B>(l.y, h.y);
    lo = __builtin_bit_cast(double, l);
    hi = __builtin_bit_cast(double, h);
}
template <int R, int B, typename T2>
__device__ __forceinline__ void swap_reg0(T2* a) {
#pragma unroll
    for (int i = 0; i < R; i += 2) {
        swap_real<B>(a[i].x, a[i + 1].x);
        swap_real<B>(a[i].y, a[i + 1].y);
    }
}

// a u + b v (REAL: a and b are real)
template <bool REAL, typename T2>
__device__ __forceinline__ T2 mix(T2 a, T2 u, T2 b, T2 v) {
    T2 r;
    if constexpr (REAL) {
        r.x = fma(b.x, v.x, a.x * u.x);
        r.y = fma(b.x, v.y, a.x * u.y);
        return r;
    }
    r.x = fma(-b.y, v.y, fma(b.x, v.x, fma(-a.y, u.y, a.x * u.x)));
    r.y = fma(b.y, v.x, fma(b.x, v.y, fma(a.y, u.x, a.x * u.y)));
    return r;
}
template <typename T2>
__device__ __forceinline__ T2 conj(T2 a) {
    a.y = -a.y;
    return a;
}

// The two matrix rows a lane uses: `own` = (m_bb, m_b(1-b)) of its bit b of the
// run's qubit, `oth` = (m_(1-b)(1-b), m_(1-b)b).
template <typename T2>
struct Rows {
    T2 own0, own1, oth0, oth1;
};

template <typename T2>
__device__ __forceinline__ Rows<T2> load_rows(const T2* m, int bit) {
    const T2 *p = m + 2 * bit, *q = m + 2 - 2 * bit;
    return {p[0], p[1], q[0], q[1]};
}

// Gradient sums of one run on register bit M (pairs (i, i | 1 << M)).
template <int R, int M, bool REAL, typename T2, typename Real>
__device__ __forceinline__ void grads_reg(const T2* p, const T2* l, Real& sx, Real& sy, Real& sz) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (i >> M & 1) continue;
        const T2 p0 = p[i], p1 = p[i | 1 << M], l0 = l[i], l1 = l[i | 1 << M];
        if constexpr (!REAL) sx = fma(l0.x, p1.y, fma(-l0.y, p1.x, fma(l1.x, p0.y, fma(-l1.y, p0.x, sx))));
        sy = fma(l1.x, p0.x, fma(l1.y, p0.y, fma(-l0.x, p1.x, fma(-l0.y, p1.y, sy))));
        if constexpr (!REAL) sz = fma(l0.x, p0.y, fma(-l0.y, p0.x, fma(-l1.x, p1.y, fma(l1.y, p1.x, sz))));
    }
}

template <int R, int M, bool INV, bool REAL, typename T2>
__device__ __forceinline__ void apply_reg(T2* s, const Rows<T2>& m) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (i >> M & 1) continue;
        const T2 u = s[i], v = s[i | 1 << M];
        if (INV) {
            s[i] = mix<REAL>(conj(m.own0), u, conj(m.oth1), v);
            s[i | 1 << M] = mix<REAL>(conj(m.oth0), v, conj(m.own1), u);
        } else {
            s[i] = mix<REAL>(m.own0, u, m.own1, v);
            s[i | 1 << M] = mix<REAL>(m.oth0, v, m.oth1, u);
        }
    }
}

// What a run does: the matrix on psi; this thread's share of the gradient
// sums, then the inverse on psi and lambda; or the sums alone.
enum { RUN_FWD = 0, RUN_BWD = 1, RUN_SUMS = 2 };

// One run. POS: the position of its qubit. REAL: its matrix is real (RY and H
// only); un-applying RY and H never mixes the Y sum with the others, so it is
// the only one needed.
template <int LOG_R, int POS, int MODE, bool REAL, typename T2, typename Real>
__device__ __forceinline__ void run_step(T2* ps, T2* lm, const Rows<T2>& m, int lane, Real& sx, Real& sy, Real& sz) {
    constexpr bool INV = MODE != RUN_FWD;
    constexpr int R = 1 << LOG_R;
    if constexpr (POS < LOG_R) {
        if constexpr (INV) {
            grads_reg<R, POS, REAL, T2, Real>(ps, lm, sx, sy, sz);
            if constexpr (MODE == RUN_SUMS) return;
            apply_reg<R, POS, true, REAL>(lm, m);
        }
        apply_reg<R, POS, INV, REAL>(ps, m);
    } else {
        constexpr int B = POS - LOG_R;
        if constexpr (INV) {
            T2 pp[R];
#pragma unroll
            for (int i = 0; i < R; ++i) pp[i] = mk<T2>(partner<B>(ps[i].x, lane), partner<B>(ps[i].y, lane));
            Real ty = 0, tz = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if constexpr (!REAL) sx = fma(lm[i].x, pp[i].y, fma(-lm[i].y, pp[i].x, sx));
                ty = fma(lm[i].x, pp[i].x, fma(lm[i].y, pp[i].y, ty));
                if constexpr (!REAL) tz = fma(lm[i].x, ps[i].y, fma(-lm[i].y, ps[i].x, tz));
            }
            const bool one = (runs_lane(lane) >> B) & 1;
            sy = one ? ty : -ty;
            sz = one ? -tz : tz;
            if constexpr (MODE == RUN_SUMS) return;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const T2 lp = mk<T2>(partner<B>(lm[i].x, lane), partner<B>(lm[i].y, lane));
                lm[i] = mix<REAL>(conj(m.own0), lm[i], conj(m.oth1), lp);
                ps[i] = mix<REAL>(conj(m.own0), ps[i], conj(m.oth1), pp[i]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const T2 pp = mk<T2>(partner<B>(ps[i].x, lane), partner<B>(ps[i].y, lane));
                ps[i] = mix<REAL>(m.own0, ps[i], m.own1, pp);
            }
        }
    }
}

// Lane bits 4 and 5 with more than one register: the run is made on register
// bit 0 between two permlane swaps (4 instructions per amplitude pair against
// 12 for fetching both partners).
template <int LOG_R, int POS, int MODE, bool REAL, typename T2, typename Real>
__device__ __forceinline__ void run_any(T2* ps, T2* lm, const Rows<T2>& m, int lane, Real& sx, Real& sy, Real& sz) {
    constexpr int R = 1 << LOG_R, B = POS - LOG_R;
    if constexpr (LOG_R > 0 && (B == 4 || B == 5)) {
        swap_reg0<R, B>(ps);
        if constexpr (MODE != RUN_FWD) swap_reg0<R, B>(lm);
        run_step<LOG_R, 0, MODE, REAL, T2, Real>(ps, lm, m, lane, sx, sy, sz);
        swap_reg0<R, B>(ps);
        if constexpr (MODE != RUN_FWD) swap_reg0<R, B>(lm);
    } else {
        run_step<LOG_R, POS, MODE, REAL, T2, Real>(ps, lm, m, lane, sx, sy, sz);
    }
}

// The bit whose rows a thread takes for a run at position pos: its lane bit,
// or 0 where the run is made on a register bit.
template <int LOG_R>
__device__ __forceinline__ int row_bit(int pos, int sid) {
    const int b = pos - LOG_R;
    if (b < 0 || (LOG_R > 0 && b >= 4)) return 0;
    return (sid >> b) & 1;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return dpp_f32<CTRL>(v); }
template <int CTRL>
__device__ __forceinline__ double dpp(double v) { return dpp_f64<CTRL>(v); }

// The wavefront's gradient sums of one run into its words of the table. The
// three sums share the first two levels of the reduction: a permlane swap of
// two of them leaves one's halves in the lower lanes and the other's in the
// upper, so one add folds both. Rows 0, 1, 2 end with X, Z, Y. The last two
// levels are fp64: 16 lanes are added in fp32.
template <bool REAL, typename Real>
__device__ __forceinline__ void store_sums(Real* o, Real sx, Real sy, Real sz, int lane) {
    if constexpr (REAL) {
        const double y = wave_total(sy);
        if (lane == 0) {
            o[0] = (Real)0;
            o[1] = (Real)y;
            o[2] = (Real)0;
        }
    } else {
        swap_real<5>(sx, sy);
        Real u = sx + sy, v = sz;  // lower half: X, upper half: Y
        swap_real<5>(sz, v);
        v += sz;
        swap_real<4>(u, v);
        u += v;
        u += dpp<0xB1>(u);
        u += dpp<0x4E>(u);
        double t = (double)u;  // the last levels in fp64
        t += dpp_f64<0x141>(t);
        t += dpp_f64<0x140>(t);
        if ((lane & 15) == 0 && lane < 48) o[lane == 0 ? 0 : lane == 16 ? 2 : 1] = (Real)t;
    }
}

// A layer: the runs of the positions in `mask`, in order of position (on
// distinct qubits, so any order is right). `base`: position 0's matrix, `o`:
// this wavefront's sums of position 0, `stride` to the next position's. The
// rows of the next position are fetched during a run.
template <int LOG_R, int MODE, int POS, bool REAL, typename T2, typename Real>
__device__ __forceinline__ void layer(T2* ps, T2* lm, const T2* base, uint32_t mask, const Rows<T2>& cur, Real* o,
                                      int stride, int sid, int lane) {
    if constexpr (POS < LOG_R + 6) {
        Rows<T2> nxt = cur;
        if constexpr (POS + 1 < LOG_R + 6 && MODE != RUN_SUMS)
            nxt = load_rows(base + 4 * (POS + 1), row_bit<LOG_R>(POS + 1, sid));
        if (mask >> POS & 1u) {
            Real sx = 0, sy = 0, sz = 0;
            run_any<LOG_R, POS, MODE, REAL, T2, Real>(ps, lm, cur, lane, sx, sy, sz);
            if constexpr (MODE != RUN_FWD) store_sums<REAL>(o + POS * stride, sx, sy, sz, lane);
        }
        layer<LOG_R, MODE, POS + 1, REAL, T2, Real>(ps, lm, base, mask, nxt, o, stride, sid, lane);
    }
}

template <int R, typename T2>
__device__ __forceinline__ void flip_signs(T2* a, uint32_t m) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const bool on = (m >> i) & 1u;
        a[i].x = on ? -a[i].x : a[i].x;
        a[i].y = on ? -a[i].y : a[i].y;
    }
}

// |m|^2 - 1 of a run's rounded matrix with first column (u, v). Such a matrix
// is a rotation times its norm (its entries round in pairs), so the states of a
// plan differ from normed ones by one factor, the same for every amplitude, and
// taking it out of the sums at the end leaves the rounding of the angles: 8
// layers of RY at 10 qubits, relative errors of <Z>, input and weight gradients
// 4.3e-7, 5.3e-7, 6.4e-7 -> 2.1e-7, 2.6e-7, 3.1e-7. Complex64 only (a reference
// in fp64 rounds its own rotations alike). A controlled run scales the halves of
// the state apart and is left as it is.
__device__ __forceinline__ double deviation(float2 u, float2 v) {
    const double a = u.x, b = u.y, c = v.x, d = v.y;
    return fma(a, a, fma(b, b, fma(c, c, fma(d, d, -1.0))));
}

// Gate record of a step held by a lane (see run_record).
struct Step {
    uint32_t op, mat, y;
};

// The kernel's arguments, read again: what only the ends of the kernel use would
// else hold scalar registers through the steps (59 spilled, shift of 10 qubits
// and 256 samples 1.88 ms).
typedef const __attribute__((address_space(4))) RunArgs* LateArgs;
__device__ __forceinline__ LateArgs late_args() {
    LateArgs p = (LateArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// One workgroup per sample, 2^log_t threads (at least one wavefront; lanes
// past 2^n hold zeros and mix with nothing). Every table the steps read is in
// LDS or in the lanes: lane i holds the packed record of step 64 c + i, read
// by readlane. (With the records read by scalar loads a step waited about 800
// cycles for its record and then its rows, whatever it computed.)
template <typename Real, int LOG_R, int MAXT>
__global__ void __launch_bounds__(MAXT) k_runs(const RunArgs a, const uint2* __restrict__ steps,
                                               const DevRunEntry* __restrict__ entries,
                                               const DevRunMember* __restrict__ members,
                                               const SlotSrc* __restrict__ slots,
                                               const uint32_t* __restrict__ words_g) {
    using T2 = typename Cx<Real>::T;
    constexpr int R = 1 << LOG_R;
    constexpr bool NORMS = sizeof(Real) == 4;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x, NW = nt >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sid = (tid & ~63) | runs_lane(lane);  // storage thread index
    const int64_t b = blockIdx.x;
    const int n = a.n, log_t = a.log_t, dim = 1 << n;
    T2* mat = (T2*)(smem + a.lds.mat);                   // [n_mat]
    // prefix runs (positions' matrices at the head of the table): the factors of
    // bit 0 and 1 of position p at fac[FS p], fac[FS p + 1]
    double2* fac = (double2*)mat;
    constexpr int FS = (int)(4 * sizeof(T2) / sizeof(double2));
    double2* cs = (double2*)(smem + a.lds.cs);           // [n_cs]
    double* scale = (double*)(smem + a.lds.scale);       // [n_mats] (fp32): see deviation()
    uint8_t* kinds = smem + a.lds.kind;                  // [n_members]
    uint32_t* words = (uint32_t*)(smem + a.lds.words);   // [n_words]
    Real* go = (Real*)(smem + a.lds.go);                 // [n] upstream gradient by position
    Real* sums = (Real*)(smem + a.lds.sum);              // [n_grads][NW][3]
    const bool active = sid < (1 << log_t);
    auto qubit_at = [&](uint64_t qubits, int p) { return (int)((qubits >> (4 * p)) & 15u); };

    // ---- the sample's matrices: angles first, one member per thread, then
    // one run per thread
    uint2 rec = steps[min(lane, a.n_steps)];  // the first steps' records
    DevRunEntry my{};                                      // this thread's first run
    if (tid < a.n_entries) my = entries[tid];
    for (int i = tid; i < a.n_words; i += nt) words[i] = words_g[i];
    if (NORMS && a.bwd)
        for (int i = tid; i < a.n_mats; i += nt) scale[i] = 0.0;
    if (a.bwd && tid < n) go[tid] = ((const Real*)a.grad_out)[b * n + qubit_at(a.last_qubit, tid)];
    const int64_t bs = a.vper > 0 ? (a.v0 + b) / a.vper : b;
    for (int i = tid; i < a.n_members; i += nt) {
        const DevRunMember m = members[i];
        kinds[i] = (uint8_t)m.kind;
        if (m.slot < 0) continue;
        if (m.src == S_PAULI) {
            cs[m.cs] = make_double2((double)pauli_of<Real>(a.inputs, a.F, slots[m.slot], b, a.v0, a.vper), 0.0);
            continue;
        }
        const double v = m.scale * (m.src == S_WEIGHT ? (double)((const Real*)a.weights)[m.index]
                                                      : (double)((const Real*)a.inputs)[bs * a.F + m.index]);
        double th = v + shift_of(b, a.v0, a.vper, m.slot);
        double sn, c;
        if (m.slot2 >= 0) {  // a controlled rotation: its angle for control bit 0, then for 1
            const double t2 = -v + shift_of(b, a.v0, a.vper, m.slot2);
            sincos(0.5 * (th - t2), &sn, &c);
            cs[m.cs + 1] = make_double2(c, sn);
            th += t2;
        }
        sincos(0.5 * th, &sn, &c);
        cs[m.cs] = make_double2(c, sn);
    }
    __syncthreads();
    double norms = 0.0;  // deviations of this thread's runs
    for (int i = tid; i < a.n_entries; i += nt) {
        const DevRunEntry e = i == tid ? my : entries[i];
        for (int v = 0; v < 1 + e.controlled; ++v) {
            // the first column (a, c); the determinant is -1 after an odd
            // number of H and Paulis, so the second is (-det c*, det a*)
            double2 a1 = make_double2(1.0, 0.0), c1 = make_double2(0.0, 0.0);
            bool odd = false;
            for (int k = 0; k < e.count; ++k) {
                const int kind = kinds[e.first + k];
                const double2 t = cs[e.cs + (k << e.controlled) + v], u = a1, w = c1;
                left_row(kind, t, u, w, a1, c1);
                odd ^= kind == K_H || (kind == K_PAULI && t.x != 0.0);
            }
            if (e.mat < 4 * (uint32_t)min(n, LOG_R + 6)) {  // a prefix run: its first column, in fp64
                fac[FS * (e.mat >> 2)] = a1;
                fac[FS * (e.mat >> 2) + 1] = c1;
                continue;
            }
            T2* o = mat + e.mat + 4 * v;
            o[0] = to_real<T2, Real>(a1);
            o[1] = to_real<T2, Real>(odd ? make_double2(c1.x, -c1.y) : make_double2(-c1.x, c1.y));
            o[2] = to_real<T2, Real>(odd ? make_double2(-a1.x, a1.y) : make_double2(a1.x, -a1.y));
            o[3] = to_real<T2, Real>(c1);
            if constexpr (NORMS)
                if (!e.controlled) {
                    const double d = deviation(o[0], o[3]);
                    norms += d;
                    if (a.bwd) scale[e.mat >> 2] = d;
                }
        }
    }
    if constexpr (NORMS) {
        norms = wave_total(norms);
        if (lane == 0) ((double*)(smem + a.lds.norm))[wave] = norms;
    }
    __syncthreads();
    if (NORMS && a.bwd && wave == 0) {  // the sums over the matrices up to each (read after the next barrier)
        double before = 0.0;
        for (int i0 = 0; i0 < a.n_mats; i0 += 64) {
            const int i = i0 + lane;
            const double t = before + lane_scan(i < a.n_mats ? scale[i] : 0.0);
            if (i < a.n_mats) scale[i] = t;
            before = lane_value(t, 63);
        }
    }

    // ---- initial state. Amplitude index of (thread, register i): bits of the
    // storage index moved to their qubits.
    auto amp_index = [&](uint64_t qubits, int i) {
        const uint32_t t = (uint32_t)(sid << LOG_R | i);
        int j = 0;
        for (int p = 0; p < n; ++p) j |= (int)((t >> p) & 1u) << ((qubits >> (4 * p)) & 15u);
        return j;
    };
    T2 ps[R], lm[R];
    // the product of the prefix runs' first columns (bits past n are 0 in
    // every active thread); the thread's factor in fp64
    auto product_state = [&](T2* dst, uint32_t prefix) {
        auto factor = [&](int p, int bit) {
            const double2 f = fac[FS * p + bit];
            return (prefix >> p) & 1u ? f : make_double2(bit ? 0.0 : 1.0, 0.0);
        };
        auto two = [&](int l) { return cxmul(factor(LOG_R + l, (sid >> l) & 1), factor(LOG_R + l + 1, (sid >> (l + 1)) & 1)); };
        double2 c = cxmul(cxmul(two(0), two(2)), two(4));
        if (!active || wave > 0) c = make_double2(0.0, 0.0);  // (no prefix run on a wavefront bit)
        dst[0] = to_real<T2, Real>(c);
#pragma unroll
        for (int m = 0; m < LOG_R; ++m) {
            const T2 f0 = to_real<T2, Real>(factor(m, 0)), f1 = to_real<T2, Real>(factor(m, 1));
#pragma unroll
            for (int i = 0; i < (1 << m); ++i) {
                dst[i | 1 << m] = cxmul(dst[i], f1);
                dst[i] = cxmul(dst[i], f0);
            }
        }
    };
    const Real* x = a.embed ? (const Real*)a.inputs + bs * a.F + a.first : nullptr;
    double norm = 0.0;
    if (a.embed == E_AMPLITUDE) {
        double *red0 = (double*)(smem + a.lds.red), acc = 0.0;
        for (int j = tid; j < dim; j += nt) acc = fma((double)x[j], (double)x[j], acc);
        acc = wave_total(acc);
        if (lane == 0) red0[wave] = acc;
        __syncthreads();
        for (int w = 0; w < NW; ++w) norm += red0[w];
        norm = sqrt(norm);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const Real v = active ? x[amp_index(a.first_qubit, i)] : (Real)0;
            ps[i] = mk<T2>(norm > 0 ? (Real)((double)v / norm) : (Real)0, (Real)0);
        }
    } else if (a.embed == E_BASIS) {
        int idx = 0;
        for (int q = 0; q < n; ++q)
            if ((double)x[q] >= 0.5) idx |= 1 << q;
#pragma unroll
        for (int i = 0; i < R; ++i)
            ps[i] = mk<T2>((Real)(active && amp_index(a.first_qubit, i) == idx), (Real)0);
    } else {
        product_state(ps, a.prefix);
    }

    // ---- steps
    auto step_of = [&](int i) {
        const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)rec.x, i);
        return Step{w & 0xffu, w >> 8, (uint32_t)__builtin_amdgcn_readlane((int)rec.y, i)};
    };
    const int sum_stride = 3 * NW;
    Real* my_sums = sums + 3 * wave;
    uint32_t nat[R];  // this thread's own slots, in the order of the threads
#pragma unroll
    for (int i = 0; i < R; ++i) nat[i] = runs_bank((uint32_t)(i << log_t | sid));
    const uint8_t* bytes = (const uint8_t*)words;
    auto signs_of = [&](uint32_t at) { return active ? (uint32_t)bytes[4 * at + sid] : 0u; };
    // exchange buffers: with two (lds.alt != 0), consecutive exchanges
    // alternate and one barrier each is enough: a wavefront that writes a
    // buffer again has passed the barrier between, which every wavefront
    // reaches after reading this buffer
    uint32_t xb = 0;
    auto slot_of = [&](uint32_t at, uint32_t* to) {
        const uint32_t base = words[at + (sid & 63)] ^ words[at + 64 + wave];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            to[i] = base;
#pragma unroll
            for (int m = 0; m < LOG_R; ++m)
                if (i >> m & 1) to[i] ^= words[at + 64 + NW + m];
        }
    };
// a controlled run: the matrices of this thread's control bit
#define QL_CRUN_CASE(P, MODE)                                                                     \
    case RS_CRUN + P:                                                                             \
        if constexpr (P < LOG_R + 6) {                                                            \
            const T2* m = mat + cur.mat + (((sid >> (cur.y & 31u)) & 1) << 2);                    \
            Real sx = 0, sy = 0, sz = 0;                                                          \
            run_any<LOG_R, P, MODE, false, T2, Real>(ps, lm, load_rows(m, row_bit<LOG_R>(P, sid)), lane, \
                                              sx, sy, sz);                                        \
            if constexpr (MODE != RUN_FWD) {                                                      \
                if (!((sid >> (cur.y & 31u)) & 1)) sx = sy = sz = 0; /* the control's 1 half */   \
                store_sums<false>(my_sums + (cur.y >> 9) * sum_stride, sx, sy, sz, lane);                \
            }                                                                                     \
        }                                                                                         \
        break;
#define QL_CRUN_CASES(MODE)                                                                       \
    QL_CRUN_CASE(0, MODE) QL_CRUN_CASE(1, MODE) QL_CRUN_CASE(2, MODE) QL_CRUN_CASE(3, MODE)        \
    QL_CRUN_CASE(4, MODE) QL_CRUN_CASE(5, MODE) QL_CRUN_CASE(6, MODE) QL_CRUN_CASE(7, MODE) QL_CRUN_CASE(8, MODE)
    for (int c0 = 0; c0 < a.n_steps; c0 += 64) {
        if (c0 > 0) rec = steps[min(c0 + lane, a.n_steps)];
        const int cnt = min(64, a.n_steps - c0);
        for (int s = 0; s < cnt; ++s) {
            const Step cur = step_of(s);
            switch (cur.op) {
                QL_CRUN_CASES(RUN_FWD)
                case RS_LAYER_REAL: {
                    const T2* base = mat + cur.mat;
                    layer<LOG_R, RUN_FWD, 0, true, T2, Real>(ps, lm, base, cur.y & 0x1ffu,
                                                             load_rows(base, row_bit<LOG_R>(0, sid)), (Real*)nullptr, 0,
                                                             sid, lane);
                } break;
                case RS_LAYER: {
                    const T2* base = mat + cur.mat;
                    layer<LOG_R, RUN_FWD, 0, false, T2, Real>(ps, lm, base, cur.y & 0x1ffu,
                                                              load_rows(base, row_bit<LOG_R>(0, sid)), (Real*)nullptr, 0,
                                                              sid, lane);
                } break;
                case RS_SIGN:
                    flip_signs<R>(ps, signs_of(cur.mat));
                    break;
                case RS_EXCHANGE: {
                    if (cur.y) flip_signs<R>(ps, signs_of(cur.y - 1));
                    T2* buf = (T2*)(smem + xb);
                    uint32_t to[R];
                    slot_of(cur.mat, to);
                    if (active) {
#pragma unroll
                        for (int i = 0; i < R; ++i) buf[to[i]] = ps[i];
                    }
                    __syncthreads();
                    if (active) {
#pragma unroll
                        for (int i = 0; i < R; ++i) ps[i] = buf[nat[i]];
                    }
                    if (a.lds.alt) xb ^= a.lds.alt;
                    else __syncthreads();
                } break;
                default:
                    break;
            }
        }
    }

    // ---- <Z> and the final state, in the last layout
    const LateArgs f = late_args();
    const uint64_t last = f->last_qubit;
    // sums of a wavefront: four of 16 lanes each in fp32, added in fp64 below
    constexpr int ROWS = sizeof(Real) == 4 ? 4 : 1;
    Real* red = (Real*)(smem + f->lds.red);  // [n][NW][ROWS]
    auto put_sum = [&](int p, Real v) {
        if constexpr (ROWS == 4) {
            v = row_sum(v);
            if ((lane & 15) == 0) red[(p * NW + wave) * 4 + (lane >> 4)] = v;
        } else {
            const double t = wave_total(v);
            if (lane == 0) red[p * NW + wave] = t;
        }
    };
    if (f->psi_out && active) {
#pragma unroll
        for (int i = 0; i < R; ++i) ((T2*)f->psi_out)[b * dim + amp_index(last, i)] = ps[i];
    }
    if (f->expz) {
        Real pt = 0, dm[LOG_R + 1];
#pragma unroll
        for (int m = 0; m < LOG_R; ++m) dm[m] = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const Real p = ps[i].x * ps[i].x + ps[i].y * ps[i].y;
            pt += p;
#pragma unroll
            for (int m = 0; m < LOG_R; ++m) dm[m] += (i >> m & 1) ? -p : p;
        }
#pragma unroll
        for (int m = 0; m < LOG_R; ++m) put_sum(m, dm[m]);
#pragma unroll
        for (int l = 0; l < 6; ++l)
            if (LOG_R + l < n) put_sum(LOG_R + l, (sid >> l & 1) ? -pt : pt);
        for (int p = LOG_R + 6; p < n; ++p) put_sum(p, (wave >> (p - LOG_R - 6) & 1) ? -pt : pt);
        __syncthreads();
        if (tid < n) {
            double t = 0.0, u = 1.0;
            for (int w = 0; w < NW * ROWS; ++w) t += (double)red[tid * NW * ROWS + w];
            if constexpr (NORMS)
                for (int w = 0; w < NW; ++w) u += ((const double*)(smem + f->lds.norm))[w];
            ((Real*)f->expz)[b * n + qubit_at(last, tid)] = (Real)(NORMS ? t / u : t);
        }
    }
    if (!f->bwd) return;

    // ---- lambda = (sum_q g_q Z_q) psi
    {
        Real base = 0;
#pragma unroll
        for (int p = LOG_R; p < RUNS_MAX_QUBITS; ++p)
            if (p < n) base += (sid >> (p - LOG_R) & 1) ? -go[p] : go[p];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            Real d = base;
#pragma unroll
            for (int m = 0; m < LOG_R; ++m) d += (i >> m & 1) ? -go[m] : go[m];
            lm[i] = mk<T2>(d * ps[i].x, d * ps[i].y);
        }
    }

    // ---- backward steps: gradient sums, then the inverse on psi and lambda;
    // the prefix runs at the end: sums only
    for (int c1 = a.n_steps; c1 > 0;) {  // chunks of up to 64 steps, [c0, c1)
        const int c0 = max(0, c1 - 64);
        rec = steps[min(c0 + lane, a.n_steps)];
        for (int s = c1 - 1 - c0; s >= 0; --s) {
            const Step cur = step_of(s);
            switch (cur.op) {
                QL_CRUN_CASES(RUN_BWD)
                case RS_LAYER_REAL: {
                    const T2* base = mat + cur.mat;
                    layer<LOG_R, RUN_BWD, 0, true, T2, Real>(ps, lm, base, cur.y & 0x1ffu,
                                                             load_rows(base, row_bit<LOG_R>(0, sid)),
                                                             my_sums + (cur.y >> 9) * sum_stride, sum_stride, sid, lane);
                } break;
                case RS_LAYER: {
                    const T2* base = mat + cur.mat;
                    layer<LOG_R, RUN_BWD, 0, false, T2, Real>(ps, lm, base, cur.y & 0x1ffu,
                                                              load_rows(base, row_bit<LOG_R>(0, sid)),
                                                              my_sums + (cur.y >> 9) * sum_stride, sum_stride, sid, lane);
                } break;
                case RS_SIGN: {
                    const uint32_t m = signs_of(cur.mat);
                    flip_signs<R>(ps, m);
                    flip_signs<R>(lm, m);
                } break;
                case RS_EXCHANGE: {
                    T2 *buf = (T2*)(smem + xb), *lbuf = (T2*)(smem + xb + a.lds.lam);
                    uint32_t from[R];
                    slot_of(cur.mat, from);
                    if (active) {
#pragma unroll
                        for (int i = 0; i < R; ++i) {
                            buf[nat[i]] = ps[i];
                            lbuf[nat[i]] = lm[i];
                        }
                    }
                    __syncthreads();
                    if (active) {
#pragma unroll
                        for (int i = 0; i < R; ++i) {
                            ps[i] = buf[from[i]];
                            lm[i] = lbuf[from[i]];
                        }
                    }
                    if (a.lds.alt) xb ^= a.lds.alt;
                    else __syncthreads();
                    if (cur.y) {
                        const uint32_t m = signs_of(cur.y - 1);
                        flip_signs<R>(ps, m);
                        flip_signs<R>(lm, m);
                    }
                } break;
                default:
                    break;
            }
        }
        c1 = c0;
    }
    const LateArgs t = late_args();
    if (t->prefix) product_state(ps, t->prefix);  // exact, not un-computed
    layer<LOG_R, RUN_SUMS, 0, false, T2, Real>(ps, lm, mat, t->prefix, Rows<T2>{}, my_sums, sum_stride, sid, lane);
#undef QL_CRUN_CASE
#undef QL_CRUN_CASES
    __syncthreads();

    // ---- the gradient of every rotation, one run per thread
    const uint8_t* kinds_t = smem + t->lds.kind;
    const double2* cs_t = (const double2*)(smem + t->lds.cs);
    double* gs = (double*)(smem + t->lds.gs);
    double* red_t = (double*)(smem + t->lds.red);
    const double* scale_t = (const double*)(smem + t->lds.scale);
    const double all = NORMS ? scale_t[t->n_mats - 1] : 0.0;
    for (int i = tid; i < t->n_entries; i += nt) {
        const DevRunEntry e = i == tid ? my : entries[i];
        if (e.grad == RUNS_NONE) continue;
        double S[3] = {0.0, 0.0, 0.0};
        for (int w = 0; w < NW; ++w)
            for (int c = 0; c < 3; ++c) S[c] += (double)sums[((size_t)e.grad * NW + w) * 3 + c];
        // psi and lambda have the scale of every run, and of those undone before these sums once more
        if constexpr (NORMS) {
            const int at = (int)(e.mat >> 2);
            double off = all;
            if (at >= min(n, LOG_R + 6)) off += (all - scale_t[e.layer_end - 1]) + (scale_t[at - 1] - scale_t[e.layer_first - 1]);
            const double f = 1.0 / (1.0 + off);
            for (int c = 0; c < 3; ++c) S[c] *= f;
        }
        // the sums seen before each gate: g^dagger P g mixes them like a rotation of the three axes
        for (int k = e.count - 1; k >= 0; --k) {
            const int kind = kinds_t[e.first + k];
            const double2 h = cs_t[e.cs + (k << e.controlled) + e.controlled];
            if (kind == K_H) {
                const double u = S[0];
                S[0] = S[2];
                S[1] = -S[1];
                S[2] = u;
            } else if (kind == K_PAULI) {
                const int w = (int)h.x;
                if (w == 2 || w == 3) S[0] = -S[0];
                if (w == 1 || w == 3) S[1] = -S[1];
                if (w == 1 || w == 2) S[2] = -S[2];
            } else {
                const double c = h.x * h.x - h.y * h.y, sn = 2.0 * h.x * h.y;
                const double own = kind == K_RX ? S[0] : kind == K_RY ? S[1] : S[2];
                const int2 sl = *(const int2*)&members[e.first + k].slot;
                gs[sl.x] = own;
                if (sl.y >= 0) gs[sl.y] = -own;  // the half-angle pair: scales +1/2 and -1/2
                sums_before(kind, c, sn, S);
            }
        }
    }
    __syncthreads();
    for (int s = tid; s < t->n_slots; s += nt)
        if (t->gpart && slots[s].src == S_WEIGHT) t->gpart[(size_t)s * t->B + b] = gs[s];
    if (t->grad_weights)
        for (int p = tid; p < t->P; p += nt) {
            double acc = 0.0;
            for (int i = t->w_ptr[p]; i < t->w_ptr[p + 1]; ++i) acc += slots[t->w_slot[i]].scale * gs[t->w_slot[i]];
            ((Real*)t->grad_weights)[p] = (Real)acc;
        }
    if (!t->grad_inputs) return;

    // ---- input gradients: the rotations bound to each feature, and the
    // amplitude embedding's (2 / |x|) (Re lambda_0 - psi_0 L), L = sum psi_0 Re lambda_0
    Real* lx = (Real*)smem;  // Re lambda_0 by amplitude index
    double L = 0.0;
    if (t->embed == E_AMPLITUDE) {
        // (the last exchange's reads are over: two barriers since)
        if (active) {
#pragma unroll
            for (int i = 0; i < R; ++i) lx[amp_index(t->first_qubit, i)] = lm[i].x;
        }
        __syncthreads();
        double acc = 0.0;
        for (int j = tid; j < dim; j += nt) acc = fma((double)x[j], (double)lx[j], acc);
        acc = wave_total(acc);
        if (lane == 0) red_t[wave] = acc;
        __syncthreads();
        for (int w = 0; w < NW; ++w) L += red_t[w];
        L = norm > 0 ? L / norm : 0.0;
    }
    for (int f = tid; f < t->F; f += nt) {
        double acc = 0.0;
        for (int i = t->x_ptr[f]; i < t->x_ptr[f + 1]; ++i) {
            const int s = t->x_slot[i];
            acc += slots[s].scale * gs[s];
        }
        const int j = f - t->first;
        if (t->embed == E_AMPLITUDE && j >= 0 && j < dim && norm > 0)
            acc += 2.0 / norm * ((double)lx[j] - (double)x[j] / norm * L) / (1.0 + all);
        ((Real*)t->grad_inputs)[b * t->F + f] = (Real)acc;
    }
}

}  // namespace

RunLds runs_lds(int dtype, const RunPlan& p, int n_slots, bool bwd) {
    const size_t real = dtype == 0 ? 4 : 8, amp = 2 * real;
    RunLds l{};
    l.lam = (uint32_t)(amp << p.n);
    const size_t one = (amp << p.n) * (bwd ? 2 : 1);
    // a second exchange buffer saves a barrier per exchange of several
    // wavefronts; small ones only, so that workgroups still share a CU
    const bool two = p.n_waves > 1 && p.n_exchanges > 0 && one <= 16384;
    l.alt = two ? (uint32_t)one : 0u;
    size_t off = two ? 2 * one : one;
    auto put = [&](size_t bytes) {
        const size_t at = (off + 15) & ~(size_t)15;
        off = at + bytes;
        return (uint32_t)at;
    };
    l.mat = put((size_t)(p.n_mat + 4 * 9) * amp);  // a layer fetches the rows of all 9 positions
    l.cs = put((size_t)p.n_cs * 16);
    l.kind = put(p.members.size());
    l.scale = put(dtype == 0 && bwd ? (size_t)(p.n_mat / 4) * 8 : 0);
    l.words = put(p.words.size() * 4);
    l.norm = put(dtype == 0 ? (size_t)p.n_waves * 8 : 0);
    l.red = put((size_t)p.n * p.n_waves * (dtype == 0 ? 16 : 8));
    l.go = put(bwd ? (size_t)p.n * real : 0);
    l.sum = put(bwd ? (size_t)p.n_grads * p.n_waves * 3 * real : 0);
    l.gs = put(bwd ? (size_t)n_slots * 8 : 0);
    l.total = (uint32_t)off;
    return l;
}

template <typename Real>
static hipError_t launch_runs_t(int log_r, const RunArgs& a, int threads, hipStream_t s) {
    const dim3 grid((unsigned)a.B), block((unsigned)threads);
#define QL_LR(LR, MT)                                                                                            \
    hipLaunchKernelGGL((k_runs<Real, LR, MT>), grid, block, a.lds.total, s, a, a.steps, a.entries, a.members, a.slots, a.words)
    if (threads == 64) {
        if (log_r == 0) QL_LR(0, 64);
        else if (log_r == 1) QL_LR(1, 64);
        else QL_LR(2, 64);
    } else if (log_r == 3 && threads <= 512) {  // 11 (complex128) and 12 qubits
        QL_LR(3, 512);
    } else if (log_r == 2 && threads <= 256) {
        QL_LR(2, 256);
    } else {
        if constexpr (sizeof(Real) == 4)
            if (log_r == 2 && threads <= 512) {  // 11 qubits
                QL_LR(2, 512);
                return hipGetLastError();
            }
        return hipErrorInvalidValue;
    }
#undef QL_LR
    return hipGetLastError();
}

hipError_t launch_runs(int dtype, int log_r, const RunArgs& a, int threads, hipStream_t s) {
    return dtype == 0 ? launch_runs_t<float>(log_r, a, threads, s) : launch_runs_t<double>(log_r, a, threads, s);
}

hipError_t configure_runs_kernels(size_t max_lds) {
    hipError_t e = hipSuccess;
#define QL_AT(REAL, LR, MT)                                                                              \
    if (e == hipSuccess)                                                                                 \
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_runs<REAL, LR, MT>),                     \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds);
#define QL_ATS(REAL) QL_AT(REAL, 0, 64) QL_AT(REAL, 1, 64) QL_AT(REAL, 2, 64) QL_AT(REAL, 2, 256) QL_AT(REAL, 3, 512)
    QL_ATS(float) QL_AT(float, 2, 512)
    QL_ATS(double)
#undef QL_ATS
#undef QL_AT
    return e;
}

}  // namespace qlayer
