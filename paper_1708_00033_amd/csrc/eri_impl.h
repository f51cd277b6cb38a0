// Direct J/K digestion kernels: one launch per canonical quartet class.
//
// Work decomposition (the paper's algorithm 3 re-expressed for one GPU):
// pairs of a class are sorted by Schwarz bound Q, so for a bra pair r the
// kets that survive screening Q_r Q_s >= tau are a prefix of the ket list
// (for bra and ket of the same class, additionally s <= r keeps each
// unordered quartet once).  A workgroup task is one bra pair and up to
// consecutive kets of its prefix (at most task_quartets); lanes take one
// quartet each.
//
// Digestion (section 4.1, eq. 2) accumulates W with
//   W_ab += 2 cj g D_cd,  W_cd += 2 cj g D_ab,
//   W_ac -= ck g D_bd,    W_bd -= ck g D_ac,  W_ad -= ck g D_bc,  W_bc -= ck g D_ad,
// g = s (ab|cd), s the number of distinct permutations of the unique quartet,
// and the two-electron Fock part is (W + W^T)/8 = cj J - ck K.
//
// MODE 0 (LDS-staged): like algorithm 3's private F_I / F_J buffers, the two
// bra rows a and b of W live in LDS for the whole task: the bra block W_ab
// is summed in registers, W_ac/W_ad/W_bc/W_bd go to LDS with ds_add_f64, and
// only the ket block W_cd goes straight to HBM with global atomics.  At the
// end of the task the LDS rows are flushed with one atomic per touched
// element.  MODE 1 (global): every update is a global atomic, into one
// shared W or (private digestion, ClassArgs::wrep) into the copy of W of the
// XCD the wave runs on; the copies are summed after the class launches.
#pragma once
#include <type_traits>

#include "hfx_internal.h"

#define HFX_WG 256
// digestion: integral blocks up to this size read all their D' elements first
#define HFX_LOADS_FIRST_MAX_NI 18
// One lane's FP64 block of at least this many integrals ((dp|pp): 162; larger
// ones are shared between lanes) is evaluated and digested in two halves of shell
// a's components: its 144 sums over primitives and 162 integrals do not fit in
// 512 registers, those of a half nearly do.  What spills is written and read once
// per primitive quartet, so that halves gain with many of those to a quartet (44-atom
// sheet, 17: 19.3 -> 11.6 ms) and pay for the recursions run twice with few (64
// waters: 1.94 and 1.96 ms, resident grids 2.01 and 1.96).  Chosen per task by its
// primitives, both forms in one kernel, the sheet took 12.4 to 12.7 ms and waters
// 1.8 to 1.9.  Thirds the same; (dp|ds) and (dd|ps), 108 integrals that fit, 3.6 ->
// 3.9 and 1.7 -> 2.5.
#define HFX_HALVES_MIN_NI 162

// K update of W[grow][gcol]: MODE 0 into the task's LDS bra row at column
// lcol (gcol less the column base of its window), MODE 1 straight into W.
template <int MODE>
__device__ __forceinline__ void row_add(double* lds_row, double* W, int grow, int gcol, int N, int lcol, double v) {
    if constexpr (MODE == 0) {
        atomicAdd(lds_row + lcol, v);
    } else {
        atomicAdd(W + (size_t)grow * N + gcol, v);
    }
}

// dcd: the ket's gathered D'_cd; W receives the J updates and WK the K updates of MODE 1 (one matrix for a
// Fock build, separate J and K accumulators for a multi-density build).
// DST (LDS digestion): bit 0, the bra's D' rows of shell a come from their
// LDS copy DI (same columns as FI); bit 1, those of shell b from DJ.
template <int NA, int NB, int NC, int ND, int MODE, int DST = 0>
__device__ __forceinline__ void digest(const double* I, double g, const ClassArgs& a, const PairInfo& bra,
                                       int fc, int fd, int spos, const double* dab, double* jab, double* FI,
                                       double* FJ, const double* __restrict__ D, double* W, int N,
                                       int RS, int cb, int db, const double* dcd, double* WK, double* wket,
                                       const double* DI = nullptr, const double* DJ = nullptr) {
    const int fa = bra.bfa, fb = bra.bfb;
    const double cj2 = 2.0 * a.cj * g, ckg = -a.ck * g;
    // the D' elements of the exchange updates
    auto load_bd = [&](double* v) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int s = 0; s < ND; ++s)
                v[n * ND + s] = (DST & 2) ? DJ[n * RS + fd + s - db] : D[(size_t)(fb + n) * N + fd + s];
    };
    auto load_ac = [&](double* v) {
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int l = 0; l < NC; ++l)
                v[m * NC + l] = (DST & 1) ? DI[m * RS + fc + l - cb] : D[(size_t)(fa + m) * N + fc + l];
    };
    auto load_bc = [&](double* v) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int l = 0; l < NC; ++l)
                v[n * NC + l] = (DST & 2) ? DJ[n * RS + fc + l - cb] : D[(size_t)(fb + n) * N + fc + l];
    };
    auto load_ad = [&](double* v) {
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int s = 0; s < ND; ++s)
                v[m * ND + s] = (DST & 1) ? DI[m * RS + fd + s - db] : D[(size_t)(fa + m) * N + fd + s];
    };
    // Small blocks: all of them before the first update.  The compiler keeps
    // the order of loads and atomics, so that each update would wait for its
    // own loads (four round trips to LDS or L2 per quartet); larger blocks
    // have no registers for it.
    constexpr bool FIRST = NA * NB * NC * ND <= HFX_LOADS_FIRST_MAX_NI;
    double dbd[NB * ND], dac[NA * NC], dbc[NB * NC], dad[NA * ND];
    if constexpr (FIRST) {
        load_bd(dbd);
        load_ac(dac);
        load_bc(dbc);
        load_ad(dad);
    }
    // J, bra block: per-lane running sums over the task (reduced at the end)
    {
#pragma unroll
        for (int mn = 0; mn < NA * NB; ++mn) {
            double v = 0.0;
#pragma unroll
            for (int ls = 0; ls < NC * ND; ++ls) v += I[mn * NC * ND + ls] * dcd[ls];
            jab[mn] += g * v;
        }
    }
    // J, ket block.  MODE 0: into the ket list's own accumulator, indexed by
    // ket position so that a wave's atomics fall in a few 64-byte lines
    // (scattered into W once per build); MODE 1: straight into W.
#pragma unroll
    for (int l = 0; l < NC; ++l)
#pragma unroll
        for (int s = 0; s < ND; ++s) {
            double v = 0.0;
#pragma unroll
            for (int mn = 0; mn < NA * NB; ++mn) v += I[mn * NC * ND + l * ND + s] * dab[mn];
            if constexpr (MODE == 0)
                atomicAdd(wket + (size_t)(l * ND + s) * a.nket_list + spos, cj2 * v);
            else
                atomicAdd(W + (size_t)(fc + l) * N + fd + s, cj2 * v);
        }
    // K: W_ac -= ck g sum_{nu sigma} I D_bd
    {
        if constexpr (!FIRST) load_bd(dbd);
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int l = 0; l < NC; ++l) {
                double v = 0.0;
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int s = 0; s < ND; ++s) v += I[((m * NB + n) * NC + l) * ND + s] * dbd[n * ND + s];
                row_add<MODE>(FI + m * RS, WK, fa + m, fc + l, N, fc + l - cb, ckg * v);
            }
    }
    // K: W_bd -= ck g sum_{mu lambda} I D_ac
    {
        if constexpr (!FIRST) load_ac(dac);
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int s = 0; s < ND; ++s) {
                double v = 0.0;
#pragma unroll
                for (int m = 0; m < NA; ++m)
#pragma unroll
                    for (int l = 0; l < NC; ++l) v += I[((m * NB + n) * NC + l) * ND + s] * dac[m * NC + l];
                row_add<MODE>(FJ + n * RS, WK, fb + n, fd + s, N, fd + s - db, ckg * v);
            }
    }
    // K: W_ad -= ck g sum_{nu lambda} I D_bc
    {
        if constexpr (!FIRST) load_bc(dbc);
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int s = 0; s < ND; ++s) {
                double v = 0.0;
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int l = 0; l < NC; ++l) v += I[((m * NB + n) * NC + l) * ND + s] * dbc[n * NC + l];
                row_add<MODE>(FI + m * RS, WK, fa + m, fd + s, N, fd + s - db, ckg * v);
            }
    }
    // K: W_bc -= ck g sum_{mu sigma} I D_ad
    {
        if constexpr (!FIRST) load_ad(dad);
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int l = 0; l < NC; ++l) {
                double v = 0.0;
#pragma unroll
                for (int m = 0; m < NA; ++m)
#pragma unroll
                    for (int s = 0; s < ND; ++s) v += I[((m * NB + n) * NC + l) * ND + s] * dad[m * ND + s];
                row_add<MODE>(FJ + n * RS, WK, fb + n, fc + l, N, fc + l - cb, ckg * v);
            }
    }
}

// The updates of digest() for the register-tiled kernels: D_cd comes in
// registers (read once per ket) and the ket block's J contribution is summed
// into jcd over the bras of a block (one atomic per ket and component after
// the block) instead of one atomic per quartet.
template <int NA, int NB, int NC, int ND, int MODE>
__device__ __forceinline__ void digest_kr(const double* I, double g, double ck, const PairInfo& bra, int fc, int fd,
                                          const double* dcd, const double* dab, double* jab, double* jcd,
                                          double* FI, double* FJ, const double* __restrict__ D,
                                          double* __restrict__ W, int N, int RS, int cb, int db) {
    const int fa = bra.bfa, fb = bra.bfb;
    const double ckg = -ck * g;
#pragma unroll
    for (int mn = 0; mn < NA * NB; ++mn) {
        double v = 0.0;
#pragma unroll
        for (int ls = 0; ls < NC * ND; ++ls) v += I[mn * NC * ND + ls] * dcd[ls];
        jab[mn] += g * v;
    }
#pragma unroll
    for (int ls = 0; ls < NC * ND; ++ls) {
        double v = 0.0;
#pragma unroll
        for (int mn = 0; mn < NA * NB; ++mn) v += I[mn * NC * ND + ls] * dab[mn];
        jcd[ls] += g * v;
    }
    {   // K: W_ac -= ck g sum I D_bd
        double dbd[NB * ND];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int s = 0; s < ND; ++s) dbd[n * ND + s] = D[(size_t)(fb + n) * N + fd + s];
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int l = 0; l < NC; ++l) {
                double v = 0.0;
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int s = 0; s < ND; ++s) v += I[((m * NB + n) * NC + l) * ND + s] * dbd[n * ND + s];
                row_add<MODE>(FI + m * RS, W, fa + m, fc + l, N, fc + l - cb, ckg * v);
            }
    }
    {   // K: W_bd -= ck g sum I D_ac
        double dac[NA * NC];
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int l = 0; l < NC; ++l) dac[m * NC + l] = D[(size_t)(fa + m) * N + fc + l];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int s = 0; s < ND; ++s) {
                double v = 0.0;
#pragma unroll
                for (int m = 0; m < NA; ++m)
#pragma unroll
                    for (int l = 0; l < NC; ++l) v += I[((m * NB + n) * NC + l) * ND + s] * dac[m * NC + l];
                row_add<MODE>(FJ + n * RS, W, fb + n, fd + s, N, fd + s - db, ckg * v);
            }
    }
    {   // K: W_ad -= ck g sum I D_bc
        double dbc[NB * NC];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int l = 0; l < NC; ++l) dbc[n * NC + l] = D[(size_t)(fb + n) * N + fc + l];
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int s = 0; s < ND; ++s) {
                double v = 0.0;
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int l = 0; l < NC; ++l) v += I[((m * NB + n) * NC + l) * ND + s] * dbc[n * NC + l];
                row_add<MODE>(FI + m * RS, W, fa + m, fd + s, N, fd + s - db, ckg * v);
            }
    }
    {   // K: W_bc -= ck g sum I D_ad
        double dad[NA * ND];
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int s = 0; s < ND; ++s) dad[m * ND + s] = D[(size_t)(fa + m) * N + fd + s];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int l = 0; l < NC; ++l) {
                double v = 0.0;
#pragma unroll
                for (int m = 0; m < NA; ++m)
#pragma unroll
                    for (int s = 0; s < ND; ++s) v += I[((m * NB + n) * NC + l) * ND + s] * dad[m * ND + s];
                row_add<MODE>(FJ + n * RS, W, fb + n, fc + l, N, fc + l - cb, ckg * v);
            }
    }
}

// A wave's evaluated-quartet counts (per-lane running counts) into the
// class's counter slot of this workgroup.  All lanes of the wave call it.
__device__ __forceinline__ void flush_counts(const ClassArgs& a, unsigned c64, unsigned c32) {
    const unsigned long long s64 = (unsigned long long)wave_sum((double)c64);
    const unsigned long long s32 = (unsigned long long)wave_sum((double)c32);
    if ((threadIdx.x & 63) == 0 && a.counters) {
        const int slot = (int)(blockIdx.x % HFX_CNT_SLOTS);
        if (s64) atomicAdd(a.counters + slot * HFX_CNT_STRIDE, s64);
        if (s32) atomicAdd(a.counters + (HFX_CNT_SLOTS + slot) * HFX_CNT_STRIDE, s32);
    }
}

// One class, one digestion mode, one precision scheme (FP32 = 0: FP64
// evaluation; FP32 = 1, a mixed build: every task's kets below split[task]
// in FP64, the rest, a suffix of its Q-sorted range, in FP32 widened to FP64
// before digestion, both in the same launch and into the same LDS rows).
//
// LDS of a class kernel: the class's FP64 Boys rows (the FP32 evaluation
// rounds their coefficients), the J sums of the current task's bra block, then
// (MODE 0) its bra rows F_I, F_J.
template <class E>
struct LdsLayout {
    static constexpr int L = E::LA + E::LB + E::LC + E::LD;
    static constexpr int JSUM = boys_rows(L) * BOYS_ROW;   // offsets in doubles
    static constexpr int ROWS = JSUM + hfx_jsum_doubles(hfx_ncart(E::LA) * hfx_ncart(E::LB));
};

// Uniform per workgroup: padding tasks (XCD striping) and other shards' bras do nothing.
__device__ __forceinline__ bool task_active(const ClassArgs& a, const int4 task) {
    return task.x >= 0 && (a.nshards <= 1 || task.x % a.nshards == a.shard);
}

template <class E>
__device__ __forceinline__ void load_boys_lds(const ClassArgs& a, double* t64) {
    using LL = LdsLayout<E>;
    const double2* __restrict__ g = reinterpret_cast<const double2*>(a.boys64 + boys_block(LL::L));
    double2* t = reinterpret_cast<double2*>(t64);
    for (int i = threadIdx.x; i < LL::JSUM / 2; i += E::WGS) t[i] = g[i];
    __syncthreads();
}

// LDS ordering point of the lanes that run one task: the workgroup, or (WAVE)
// the single wave, whose LDS operations are processed in order.
template <bool WAVE>
__device__ __forceinline__ void task_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// One task (one bra, a range of its kets): what the kernels need of it.
struct BraTask {
    PairInfo bra;
    int s0, split, send;   // kets [s0, split) in FP64, [split, send) in FP32
    int w;                 // its windows and list
    int N;                 // leading dimension of the molecule's blocks, which start at element mo
    // LDS bra rows of length RS: whole rows, or (column windows) the task's
    // window of shell c at [0, RS/2) and of shell d at [RS/2, RS) (one region
    // when both windows coincide); column col sits at col - cb (c) / col - db (d)
    int RS, cb, db, half;
    size_t mo, wo;         // wo: offset in W (private digestion: in this XCD's own copy, algorithm
                           // 2's private Fock matrix, one per XCD instead of one per thread)
    bool on;               // false: no task, padding (XCD striping) or another shard's bra
};

// ti uniform; -1: none.
template <int FP32>
__device__ __forceinline__ BraTask load_task(const ClassArgs& a, const int ti) {
    BraTask t;
    t.on = false;
    t.RS = 0;
    if (ti < 0) return t;
    const int4 task = uniform_task(a.tasks, ti);
    if (!task_active(a, task)) return t;
    t.on = true;
    t.bra = uniform_pair(a.bra, task.x);
    t.s0 = task.y;
    t.send = task.z;
    t.w = task.w;
    t.split = FP32 ? min(max(((const HFX_CONST_AS int*)a.split)[ti], t.s0), t.send) : t.send;
    t.N = t.RS = t.half = t.bra.ld;
    t.cb = t.db = 0;
    t.mo = (size_t)((const HFX_CONST_AS long long*)a.moff)[t.bra.mol];
    t.wo = t.mo + (a.wrep ? (size_t)hfx_xcc_id() * a.wrep : 0);
    if (a.win) {
        t.RS = a.rs;
        t.half = t.RS / 2;
        const int wc = hfx_task_wc(task.w), wd = hfx_task_wd(task.w);
        t.cb = wc * a.win;
        t.db = wd == wc ? t.cb : wd * a.win - t.half;
    }
    return t;
}

// Adds the rows at F (NA of shell a, NB of shell b) to w (the molecule's block
// of W or WK) and clears them, on NT lanes: a lane takes a column of every row
// at once (no divisions by the row length, all reads in flight together).
template <int NA, int NB, int NT>
__device__ __forceinline__ void flush_rows(double* F, int tid, int RS, int half, int cb, int db, int N, int bfa, int bfb,
                                           double* __restrict__ w) {
    for (int c = tid; c < RS; c += NT) {
        const int col = c + (c < half ? cb : db);
        double v[NA + NB];
#pragma unroll
        for (int r = 0; r < NA + NB; ++r) v[r] = F[r * RS + c];
#pragma unroll
        for (int r = 0; r < NA + NB; ++r)
            if (v[r] != 0.0) {
                F[r * RS + c] = 0.0;
                if (col < N) atomicAdd(w + (size_t)(r < NA ? bfa + r : bfb + r - NA) * N + col, v[r]);
            }
    }
}

// The kernels of one task on the lanes of the workgroup or (WAVE) of one wave,
// whose bra rows are the wave's own LDS region.  DST: the bra's D' rows staged
// in LDS for the LDS digestion (bit 0 shell a's, bit 1 shell b's), a kernel
// variant of the classes with small blocks.  LDS of a region: F_I, F_J, zero
// between tasks, then at a fixed place (rows of a batch differ in length) the
// staged rows.
template <class E, int MODE, int FP32, bool WAVE, int DST>
struct BraRun {
    static constexpr int NA = hfx_ncart(E::LA), NB = hfx_ncart(E::LB), NC = hfx_ncart(E::LC), ND = hfx_ncart(E::LD);
    static constexpr int NAB = NA * NB, NI = NA * NB * NC * ND;
    static constexpr int NT = WAVE ? 64 : E::WGS;   // lanes of the task
    static constexpr int PARTS = NI >= HFX_HALVES_MIN_NI ? 2 : 1, NAP = NA / PARTS;   // shell a's rows at a time
    static constexpr int nda = (DST & 1) ? NA : 0, ndb = (DST & 2) ? NB : 0;
    static_assert(DST == 0 || (MODE == 0 && NI <= HFX_STAGE_D_MAX_NI), "no staged D' rows");
    const ClassArgs& args;
    const double* t64;
    int tid;
    double *JS, *F, *DR;     // the bra block's J sums (zero between tasks); F_I and F_J; staged rows
    double dab[NAB];
    unsigned n64 = 0, n32 = 0;

    __device__ __forceinline__ BraRun(const ClassArgs& launch, double* lds)
        : args(launch), t64(lds), tid(WAVE ? (int)(threadIdx.x & 63) : (int)threadIdx.x) {
        JS = lds + LdsLayout<E>::JSUM;
        F = lds + LdsLayout<E>::ROWS + (WAVE ? (int)(threadIdx.x >> 6) * (NA + NB + nda + ndb) * args.rs : 0);
        DR = F + (NA + NB) * args.rs;
    }
    __device__ __forceinline__ void clear_rows() {
        if (!WAVE && tid < NAB) JS[tid] = 0.0;
        if constexpr (MODE == 0)
            for (int i = tid; i < (NA + NB) * args.rs; i += NT) F[i] = 0.0;
    }
    // D'_ab and the staged rows of a task, over the same columns as F_I / F_J
    // (zero past the molecule's last column).
    __device__ __forceinline__ void stage(const BraTask& t) {
        const double* __restrict__ Dm = args.D + t.mo;
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n) dab[m * NB + n] = Dm[(size_t)(t.bra.bfa + m) * t.N + t.bra.bfb + n];
        if constexpr (DST != 0) {
            for (int c = tid; c < t.RS; c += NT) {
                const int col = c + (c < t.half ? t.cb : t.db);
#pragma unroll
                for (int r = 0; r < nda + ndb; ++r)
                    DR[r * t.RS + c] =
                        col < t.N ? Dm[(size_t)(r < nda ? t.bra.bfa + r : t.bra.bfb + r - nda) * t.N + col] : 0.0;
            }
        }
    }
    __device__ __forceinline__ void flush(const BraTask& t) {
        if constexpr (MODE == 0)
            flush_rows<NA, NB, NT>(F, tid, t.RS, t.half, t.cb, t.db, t.N, t.bra.bfa, t.bra.bfb, args.W + t.wo);
        if (!WAVE && tid < NAB) {
            atomicAdd(args.W + t.wo + (size_t)(t.bra.bfa + tid / NB) * t.N + t.bra.bfb + tid % NB, JS[tid]);
            JS[tid] = 0.0;
        }
    }
    // The task's kets: evaluation, digestion into the LDS rows (MODE 0) and
    // W, then the bra block's J.
    __device__ __forceinline__ void kets(const BraTask& t) {
        const ClassArgs a = of_list(args, t.w);
        const PairInfo& bra = t.bra;
        const double* __restrict__ Dm = a.D + t.mo;
        double* __restrict__ Wm = a.W + t.wo;
        const int N = t.N, RS = t.RS, cb = t.cb, db = t.db;
        double *FI = F, *FJ = F + NA * RS, *DI = DR, *DJ = DR + nda * RS;
        double jab[NAB];
#pragma unroll
        for (int mn = 0; mn < NAB; ++mn) jab[mn] = 0.0;
        const double sbra = bra.a != bra.b ? 2.0 : 1.0;
        const int kps = a.nket_list, kfs = a.nket_list * a.knprim;
        // The task's kets in slots of 64 consecutive kets, dealt to the task's
        // waves in turn (wave w takes slots w, w + nw, ...): the FP64 part
        // [s0, split) fills the first slots and the FP32 part [split, send) the
        // rest, so every slot is uniform in precision and the two parts cost at
        // most one partial slot more than one part (a per-lane choice, or one
        // loop per part over the whole workgroup, costs a full workgroup
        // iteration per task, which short tasks cannot hide).  With one part this
        // is the plain interleaving s = s0 + tid + i NT.
        const int nw = NT / 64, wv = tid >> 6, ln = tid & 63;
        const int slots64 = (t.split - t.s0 + 63) >> 6;
        const int slots = slots64 + ((t.send - t.split + 63) >> 6);
        for (int j = wv; j < slots; j += nw) {
            const bool lo = j < slots64;   // wave-uniform
            const int s = lo ? t.s0 + (j << 6) + ln : t.split + ((j - slots64) << 6) + ln;
            if (s >= (lo ? t.split : t.send)) continue;   // the part's last, partial slot
            // the ket's record and D'_cd (gathered in ket-list order before the
            // build, coalesced across lanes); small blocks load them ahead of the
            // primitive loops
            int4 kb;
            double dcd[NC * ND];
            auto load_ket = [&]() {
                kb = a.kbf[s];   // ket's first basis functions and shells
#pragma unroll
                for (int i = 0; i < NC * ND; ++i) dcd[i] = a.dket[(size_t)i * a.nket_list + s];
            };
            if constexpr (NI <= HFX_LOADS_FIRST_MAX_NI) load_ket();
            const double* kab = a.ket[s].AB;
            double g;
            auto factor = [&]() {
                if constexpr (NI > HFX_LOADS_FIRST_MAX_NI) load_ket();
                g = sbra * (kb.z != kb.w ? 2.0 : 1.0) * ((kb.z == bra.a && kb.w == bra.b) ? 1.0 : 2.0);
            };
            // FP64: half p of PARTS of the block's rows evaluated and digested (all
            // indexes are constants, so what only the other half needs is not computed)
            auto part = [&](auto p) {
                constexpr int m0 = decltype(p)::value * NAP;
                double I[NI];
                E::template run<double>((const double*)(a.prim + bra.prim_off), bra.nprim, a.kprim + s, kfs, kps,
                                        a.knprim, bra.AB, kab, t64, I);
                if constexpr (m0 == 0) factor();
                PairInfo rows = bra;
                rows.bfa += m0;
                digest<NAP, NB, NC, ND, MODE, DST>(I + m0 * (NI / NA), g, a, rows, kb.x, kb.y, s, dab + m0 * NB,
                                                   jab + m0 * NB, FI + m0 * RS, FJ, Dm, Wm, N, RS, cb, db, dcd, Wm,
                                                   a.wket, DI + m0 * RS, DJ);
            };
            if (!FP32 || lo) {
                part(std::integral_constant<int, 0>());
                if constexpr (PARTS > 1) part(std::integral_constant<int, 1>());
                ++n64;
            } else if constexpr (FP32) {
                // FP32 primitive copies, the FP64 Boys rows rounded; the block digested in FP64
                float If[NI];
                double I[NI];
                E::template run<float>(a.prim32 + (size_t)bra.prim_off * HFX_PRIM_FIELDS, bra.nprim,
                                       a.kprim32 + s, kfs, kps, a.knprim, bra.AB, kab, t64, If);
#pragma unroll
                for (int i = 0; i < NI; ++i) I[i] = (double)If[i];
                factor();
                digest<NA, NB, NC, ND, MODE, DST>(I, g, a, bra, kb.x, kb.y, s, dab, jab, FI, FJ, Dm, Wm, N, RS, cb, db,
                                                  dcd, Wm, a.wket, DI, DJ);
                ++n32;
            }
        }
        // bra J block: summed over each wave, then over the workgroup in LDS, so
        // that a task adds once to W (column bfb may lie outside its windows)
#pragma unroll
        for (int mn = 0; mn < NAB; ++mn) {
            const double v = wave_sum(jab[mn]);
            if ((threadIdx.x & 63) == 0)
                atomicAdd(WAVE ? Wm + (size_t)(bra.bfa + mn / NB) * N + bra.bfb + mn % NB : JS + mn, 2.0 * a.cj * v);
        }
    }
};

// A reader of the eight XCD queues (one lane): the queue of XCD x0, then the
// others in turn, so that no XCD idles while another still has work.  ahead()
// draws an entry without waiting for it, take() turns it into a task index, or
// -1 when every queue is drained.
struct QueueReader {
    const ClassArgs& a;
    int x0, q = 0, drawn = 0;
    __device__ __forceinline__ explicit QueueReader(const ClassArgs& args) : a(args), x0(blockIdx.x & 7) {}
    __device__ __forceinline__ void ahead() {
        if (q < 8) drawn = (int)atomicAdd(a.work + ((x0 + q) & 7), 1ull);
    }
    __device__ __forceinline__ int take() {
        while (q < 8) {
            if (drawn < a.qlen) return 8 * drawn + ((x0 + q) & 7);
            ++q;
            ahead();
        }
        return -1;
    }
};

// Register-tiled task: a block of nb <= NBL consecutive bras of the class's
// Q-sorted list (one molecule) against one range of kets whose primitive
// count KP is a compile-time constant.  Each lane takes kets of the range; a
// ket's primitives, D'_cd and record are read once into registers and
// serve every bra of the block, whose screened prefixes differ: bra r takes
// ket s iff Q_r Q_s >= tau (and, for bra and ket of one pair class, the ket's
// class position <= r), the same test that sizes the plan's prefixes.  The
// ket block's J sum over the block goes out in one atomic per component; each
// bra has its own LDS rows F_I, F_J (MODE 0).  FP64 only.
template <class E, int MODE, int KP, int NBL>
__device__ __forceinline__ void class_task_kr(const ClassArgs& args, const int ti, const double* t64, unsigned& cnt64) {
    constexpr int NA = hfx_ncart(E::LA), NB = hfx_ncart(E::LB), NC = hfx_ncart(E::LC), ND = hfx_ncart(E::LD);
    constexpr int NAB = NA * NB, NCD = NC * ND, NI = NAB * NCD;
    constexpr int NT = E::WGS;
    const int tid = (int)threadIdx.x;
    extern __shared__ __align__(16) double lds[];
    const int4 task = uniform_task(args.tasks, __builtin_amdgcn_readfirstlane(ti));
    if (task.x < 0) return;
    const ClassArgs a = of_list(args, task.w);
    const int r0 = task.x & 0x0fffffff;
    const int nb = (task.x >> 28) + 1;
    const int s0 = task.y, send = task.z;
    PairInfo bra[NBL];
    bool on[NBL];
#pragma unroll
    for (int i = 0; i < NBL; ++i) {
        on[i] = i < nb && (a.nshards <= 1 || (r0 + i) % a.nshards == a.shard);
        bra[i] = uniform_pair(a.bra, r0 + (i < nb ? i : 0));
    }
    bool any = false;
#pragma unroll
    for (int i = 0; i < NBL; ++i) any |= on[i];
    if (!any) return;   // uniform: another shard's block
    // the block's molecule (shared by its bras): blocks of D', W, leading dimension
    const int N = bra[0].ld;
    const double* __restrict__ Dm = a.D + a.moff[bra[0].mol];
    double* __restrict__ Wm = a.W + a.moff[bra[0].mol] + (a.wrep ? (size_t)hfx_xcc_id() * a.wrep : 0);
    int RS = N, cb = 0, db = 0, half = N;
    if (a.win) {
        RS = a.rs;
        half = RS / 2;
        const int wc = hfx_task_wc(task.w), wd = hfx_task_wd(task.w);
        cb = wc * a.win;
        db = wd == wc ? cb : wd * a.win - half;
    }
    constexpr int ROWS = (NA + NB);
    double* F0 = lds + LdsLayout<E>::ROWS;   // bra i's rows at F0 + i ROWS a.rs
    if constexpr (MODE == 0) {
        for (int i = tid; i < nb * ROWS * a.rs; i += NT) F0[i] = 0.0;
        __syncthreads();
    }
    double dab[NBL][NAB], jab[NBL][NAB], sbra[NBL];
#pragma unroll
    for (int i = 0; i < NBL; ++i) {
        sbra[i] = bra[i].a != bra[i].b ? 2.0 : 1.0;
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                dab[i][m * NB + n] = Dm[(size_t)(bra[i].bfa + m) * N + bra[i].bfb + n];
                jab[i][m * NB + n] = 0.0;
            }
    }
    const int nl = a.nket_list;
    unsigned n64 = 0;
    for (int s = s0 + tid; s < send; s += NT) {
        const int4 kb = a.kbf[s];
        const int fc = kb.x, fd = kb.y;
        double kv[KP][9];
#pragma unroll
        for (int k = 0; k < KP; ++k)
#pragma unroll
            for (int f = 0; f < 9; ++f) kv[k][f] = a.kprim[(size_t)(f * KP + k) * nl + s];
        double dcd[NCD], jcd[NCD];
#pragma unroll
        for (int ls = 0; ls < NCD; ++ls) {
            dcd[ls] = a.dket[(size_t)ls * nl + s];
            jcd[ls] = 0.0;
        }
        const double qs = a.ketq[s];
        const int ks = a.same ? a.kpos[s] : 0;
        const double* kab = a.ket[s].AB;   // read only by classes with a p or d ket
        const double gk = kb.z != kb.w ? 2.0 : 1.0;
        bool hit = false;
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
            if (!on[i]) continue;
            if (!(qs * bra[i].Q >= a.tau) || ks > r0 + i) continue;
            const double g = sbra[i] * gk * ((kb.z == bra[i].a && kb.w == bra[i].b) ? 1.0 : 2.0);
            double I[NI];
            E::template run_kr<double, KP>(a.prim + bra[i].prim_off, bra[i].nprim, kv, bra[i].AB, kab,
                                                        t64, I);
            ++n64;
            hit = true;
            double* FI = F0 + i * ROWS * a.rs;
            digest_kr<NA, NB, NC, ND, MODE>(I, g, a.ck, bra[i], fc, fd, dcd, dab[i], jab[i], jcd, FI, FI + NA * RS,
                                            Dm, Wm, N, RS, cb, db);
        }
        if (hit) {
            const double cj2 = 2.0 * a.cj;
#pragma unroll
            for (int l = 0; l < NC; ++l)
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    if constexpr (MODE == 0)
                        atomicAdd(a.wket + (size_t)(l * ND + d) * nl + s, cj2 * jcd[l * ND + d]);
                    else
                        atomicAdd(Wm + (size_t)(fc + l) * N + fd + d, cj2 * jcd[l * ND + d]);
                }
        }
    }
    const int lane = tid & 63;
#pragma unroll
    for (int i = 0; i < NBL; ++i) {
        if (!on[i]) continue;
#pragma unroll
        for (int mn = 0; mn < NAB; ++mn) {
            const double v = wave_sum(jab[i][mn]);
            if (lane == 0) atomicAdd(Wm + (size_t)(bra[i].bfa + mn / NB) * N + bra[i].bfb + mn % NB, 2.0 * a.cj * v);
        }
    }
    cnt64 += n64;
    if constexpr (MODE == 0) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NBL; ++k)
            if (k < nb)
                flush_rows<NA, NB, NT>(F0 + k * ROWS * a.rs, tid, RS, half, cb, db, N, bra[k].bfa, bra[k].bfb, Wm);
    }
}

// Persistent register-tiled launch (same queues as k_class_persist).
template <class E, int MODE, int KP, int NBL>
__global__ __launch_bounds__(E::WGS) void k_class_kr(const ClassArgs a) {
    extern __shared__ __align__(16) double lds[];
    __shared__ int next_entry;
    double* t64 = lds;
    load_boys_lds<E>(a, t64);
    unsigned cnt64 = 0;
    const int x0 = blockIdx.x & 7;
    for (int q = 0; q < 8;) {
        const int x = (x0 + q) & 7;
        if (threadIdx.x == 0) next_entry = (int)atomicAdd(a.work + x, 1ull);
        __syncthreads();
        const int k = next_entry;
        __syncthreads();
        if (k >= a.qlen) {
            ++q;
            continue;
        }
        class_task_kr<E, MODE, KP, NBL>(a, 8 * k + x, t64, cnt64);
    }
    flush_counts(a, cnt64, 0);
}

// Several densities in one pass over the integrals (FP64): every quartet of
// the task is evaluated once and digested for each density d < a.ndens
// (D'_d, its gathered D'_cd, its J and K accumulators and its ket-block J
// accumulator at offsets d dstride / d kstride), the J updates into a.W (the
// ket block's via a.wket in MODE 0) and the K updates into a.WK.  MODE 0
// stages each density's bra rows of K in LDS (a.ndens row sets; the host
// groups the densities so that they fit), MODE 1 uses global atomics.  The
// bra block's J sums are reduced over each wave per ket iteration (all lanes
// of a wave iterate together).  Tasks may be blocks of bras (register-tiled
// plans): each bra keeps the kets of its own screened prefix, the test the
// planner used.
template <class E, int MODE>
__device__ __forceinline__ void class_task_multi(const ClassArgs& args, const int ti, const double* t64,
                                                 unsigned& cnt64) {
    constexpr int NA = hfx_ncart(E::LA), NB = hfx_ncart(E::LB), NC = hfx_ncart(E::LC), ND = hfx_ncart(E::LD);
    constexpr int NAB = NA * NB, NI = NAB * NC * ND;
    constexpr int NT = E::WGS;
    extern __shared__ __align__(16) double lds[];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int4 task = uniform_task(args.tasks, __builtin_amdgcn_readfirstlane(ti));
    if (task.x < 0) return;
    const ClassArgs a = of_list(args, task.w);
    const int r0 = task.x & 0x0fffffff, nb = (task.x >> 28) + 1;
    const int s0 = task.y, nq = task.z - task.y;
    unsigned n64 = 0;
    for (int i = 0; i < nb; ++i) {
        const int r = r0 + i;
        if (a.nshards > 1 && r % a.nshards != a.shard) continue;   // uniform
        const PairInfo bra = uniform_pair(a.bra, r);
        const int N = bra.ld;
        const size_t moff = (size_t)a.moff[bra.mol];
        const double sbra = bra.a != bra.b ? 2.0 : 1.0;
        // LDS rows of density d at F0 + d (NA + NB) a.rs, windows as in class_task
        int RS = N, cb = 0, db = 0, half = N;
        if (a.win) {
            RS = a.rs;
            half = RS / 2;
            const int wc = hfx_task_wc(task.w), wd = hfx_task_wd(task.w);
            cb = wc * a.win;
            db = wd == wc ? cb : wd * a.win - half;
        }
        double* F0 = lds + LdsLayout<E>::ROWS;
        const int rowset = (NA + NB) * a.rs;
        if constexpr (MODE == 0) {
            for (int x = tid; x < a.ndens * rowset; x += NT) F0[x] = 0.0;
            __syncthreads();
        }
        for (int base = 0; base < nq; base += NT) {
            const int it = base + tid;
            bool valid = it < nq;
            const int s = s0 + (valid ? it : 0);
            if (valid) valid = a.ketq[s] * bra.Q >= a.tau && !(a.same && a.kpos[s] > r);
            const int4 kb = a.kbf[s];
            const double g = sbra * (kb.z != kb.w ? 2.0 : 1.0) * ((kb.z == bra.a && kb.w == bra.b) ? 1.0 : 2.0);
            double I[NI];
            if (valid) {
                E::template run<double>((const double*)(a.prim + bra.prim_off), bra.nprim, a.kprim + s,
                                                     a.nket_list * a.knprim, a.nket_list, a.knprim, bra.AB, a.ket[s].AB,
                                                     t64, I);
                ++n64;
            }
            for (int d = 0; d < a.ndens; ++d) {
                const double* __restrict__ Dd = a.D + (size_t)d * a.dstride + moff;
                double* WJ = a.W + (size_t)d * a.dstride + moff;
                double* WKd = a.WK + (size_t)d * a.dstride + moff;
                const double* dket = a.dket + (size_t)d * a.kstride;
                double* wket = a.wket + (size_t)d * a.kstride;
                double* FI = F0 + d * rowset;
                double dab[NAB], jt[NAB];
#pragma unroll
                for (int mn = 0; mn < NAB; ++mn) {
                    dab[mn] = Dd[(size_t)(bra.bfa + mn / NB) * N + bra.bfb + mn % NB];
                    jt[mn] = 0.0;
                }
                if (valid) {
                    double dcd[NC * ND];
#pragma unroll
                    for (int i = 0; i < NC * ND; ++i) dcd[i] = dket[(size_t)i * a.nket_list + s];
                    digest<NA, NB, NC, ND, MODE>(I, g, a, bra, kb.x, kb.y, s, dab, jt, FI, FI + NA * RS, Dd, WJ, N, RS,
                                                 cb, db, dcd, WKd, wket);
                }
#pragma unroll
                for (int mn = 0; mn < NAB; ++mn) {
                    const double v = wave_sum(jt[mn]);
                    if (lane == 0 && v != 0.0)
                        atomicAdd(WJ + (size_t)(bra.bfa + mn / NB) * N + bra.bfb + mn % NB, 2.0 * a.cj * v);
                }
            }
        }
        if constexpr (MODE == 0) {   // each density's K rows into its K accumulator
            __syncthreads();
            for (int d = 0; d < a.ndens; ++d)
                flush_rows<NA, NB, NT>(F0 + d * rowset, tid, RS, half, cb, db, N, bra.bfa, bra.bfb,
                                       a.WK + (size_t)d * a.dstride + moff);
            __syncthreads();
        }
    }
    cnt64 += n64;
}

template <class E, int MODE>
__global__ __launch_bounds__(E::WGS) void k_class_multi(const ClassArgs a) {
    extern __shared__ __align__(16) double lds[];
    __shared__ int next_entry;
    load_boys_lds<E>(a, lds);
    unsigned cnt64 = 0;
    const int x0 = blockIdx.x & 7;
    for (int q = 0; q < 8;) {
        const int x = (x0 + q) & 7;
        if (threadIdx.x == 0) next_entry = (int)atomicAdd(a.work + x, 1ull);
        __syncthreads();
        const int k = next_entry;
        __syncthreads();
        if (k >= a.qlen) {
            ++q;
            continue;
        }
        class_task_multi<E, MODE>(a, 8 * k + x, lds, cnt64);
    }
    flush_counts(a, cnt64, 0);
}

// Static launch: workgroup i runs task task_off + i (a plan's tasks may span
// several launches: a grid is limited to 2^32 work-items).
template <class E, int MODE, int FP32, int DST = 0>
__global__ __launch_bounds__(E::WGS) void k_class(const ClassArgs a) {
    extern __shared__ __align__(16) double lds[];
    __shared__ unsigned long long wg_count[2];   // the workgroup's counts: one global add each
    const BraTask t = load_task<FP32>(a, a.task_off + (int)blockIdx.x);
    if (!t.on) return;
    if (threadIdx.x == 0) wg_count[0] = wg_count[1] = 0;
    BraRun<E, MODE, FP32, false, DST> r(a, lds);
    r.stage(t);
    r.clear_rows();
    load_boys_lds<E>(a, lds);   // ends with a barrier
    r.kets(t);
    const unsigned long long s64 = (unsigned long long)wave_sum((double)r.n64);
    const unsigned long long s32 = (unsigned long long)wave_sum((double)r.n32);
    if ((threadIdx.x & 63) == 0) {
        if (s64) atomicAdd(&wg_count[0], s64);
        if (s32) atomicAdd(&wg_count[1], s32);
    }
    __syncthreads();
    r.flush(t);
    if (threadIdx.x == 0 && a.counters) {
        const int slot = (int)(blockIdx.x % HFX_CNT_SLOTS);
        if (wg_count[0]) atomicAdd(a.counters + slot * HFX_CNT_STRIDE, wg_count[0]);
        if (wg_count[1]) atomicAdd(a.counters + (HFX_CNT_SLOTS + slot) * HFX_CNT_STRIDE, wg_count[1]);
    }
}

// Persistent launch: a resident grid; a workgroup on XCD x (workgroup index
// mod 8, the hardware's round-robin placement) takes entries of XCD x's
// queue through an atomic counter, then drains the other queues in turn (the
// dynamic load balancing of ddi_dlbnext in algorithms 1-3).  A separate kernel
// so that the static form keeps its register allocation.
//
// Between two tasks the workgroup's lanes wait on one chain: the drawn entry,
// its records (task, bra, molecule), the staged rows, the flush of the last
// task's rows.  So the entry is drawn while the last task's kets run, the flush
// clears the rows for the next task, and rows are walked by columns, every row
// of a column in flight at once, instead of by a flat index that is divided by
// the row length: 64 waters, all classes, 95.0 -> 92.6 ms; 112 waters 618 ->
// 563 ms (its tasks are short: four windows a bra); (ss|ss) of a 44-atom
// sheet, whose tasks are long, 2.7 -> 2.9 ms, its classes together unchanged.
// Reading the next task's records and rows before the last flush was slower
// (20 more registers).
template <class E, int MODE, int FP32, int DST = 0>
__global__ __launch_bounds__(E::WGS) void k_class_persist(const ClassArgs a) {
    extern __shared__ __align__(16) double lds[];
    __shared__ int next_task;
    BraRun<E, MODE, FP32, false, DST> r(a, lds);
    QueueReader queue(a);
    if (threadIdx.x == 0) queue.ahead();
    r.clear_rows();
    load_boys_lds<E>(a, lds);   // once per resident workgroup
    for (;;) {
        if (threadIdx.x == 0) next_task = queue.take();
        __syncthreads();   // also: the last task's rows are flushed and cleared
        const int ti = __builtin_amdgcn_readfirstlane(next_task);
        if (ti < 0) break;
        const BraTask t = load_task<FP32>(a, ti);
        if (t.on) r.stage(t);
        __syncthreads();
        if (threadIdx.x == 0) queue.ahead();
        if (!t.on) continue;
        r.kets(t);
        __syncthreads();
        r.flush(t);
    }
    flush_counts(a, r.n64, r.n32);
}

// Persistent launch with one task per wave: each wave of a resident
// workgroup takes its own queue entries (same queues and order as
// k_class_persist) and digests into its own LDS bra rows, so short tasks
// (small molecules of a batch) occupy 64 lanes instead of a workgroup.  The
// Boys rows are shared by the workgroup's waves.
template <class E, int MODE, int FP32, int DST = 0>
__global__ __launch_bounds__(E::WGS) void k_class_wave(const ClassArgs a) {
    extern __shared__ __align__(16) double lds[];
    BraRun<E, MODE, FP32, true, DST> r(a, lds);
    QueueReader queue(a);
    const bool first = (threadIdx.x & 63) == 0;
    if (first) queue.ahead();
    r.clear_rows();
    load_boys_lds<E>(a, lds);
    for (;;) {
        const int ti = __builtin_amdgcn_readfirstlane(first ? queue.take() : 0);
        if (ti < 0) break;
        if (first) queue.ahead();
        const BraTask t = load_task<FP32>(a, ti);
        if (!t.on) continue;
        r.stage(t);
        task_sync<true>();
        r.kets(t);
        task_sync<true>();
        r.flush(t);
        task_sync<true>();
    }
    flush_counts(a, r.n64, r.n32);
}

// Schwarz bound of every pair of one pair class: Q = sqrt(max (mn|mn)) with
// the component normalisation s_m s_n applied (always FP64).
// 1/sqrt((2lx-1)!!(2ly-1)!!(2lz-1)!!) of Cartesian component c of shell l.
__device__ __forceinline__ double comp_scale(int l, int c) {
    return (l == 2 && (c == 0 || c == 3 || c == 5)) ? 0.57735026918962576451 : 1.0;
}

template <class E>
__global__ __launch_bounds__(HFX_WG) void k_schwarz(const PairInfo* __restrict__ pairs, int npairs,
                                                     const PrimPair* __restrict__ prim,
                                                     const double* __restrict__ boys, double* __restrict__ Q) {
    constexpr int NA = hfx_ncart(E::LA), NB = hfx_ncart(E::LB);
    const int i = blockIdx.x * HFX_WG + threadIdx.x;
    if (i >= npairs) return;
    const PairInfo pr = pairs[i];
    double I[NA * NB * NA * NB];
    // ket read from the array-of-structures layout: field stride 1, primitive stride 10 doubles
    E::template run<double>((const double*)(prim + pr.prim_off), pr.nprim, (const double*)(prim + pr.prim_off), 1,
                            (int)(sizeof(PrimPair) / sizeof(double)), pr.nprim, pr.AB, pr.AB,
                            boys + boys_block(E::LA + E::LB + E::LC + E::LD), I);
    double mx = 0.0;
#pragma unroll
    for (int m = 0; m < NA; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const double s = comp_scale(E::LA, m) * comp_scale(E::LB, n);
            const double v = I[(m * NB + n) * NA * NB + m * NB + n] * s * s;
            mx = v > mx ? v : mx;
        }
    Q[i] = sqrt(mx);
}


// Kernel variants of one class: launch form x digestion mode x precision.
template <class E>
struct ClassKernelsOne {
    static constexpr int NI = hfx_ncart(E::LA) * hfx_ncart(E::LB) * hfx_ncart(E::LC) * hfx_ncart(E::LD);
    static constexpr bool kStage = NI <= HFX_STAGE_D_MAX_NI;
    // LDS digestion with staged D' rows (DST 1: shell a's, 3: both shells'):
    // form 0 static, 1 persistent, 2 one task per wave
    template <int DST>
    static const void* staged(int form, int mixed) {
        static const void* t[6] = {(const void*)k_class<E, 0, 0, DST>,         (const void*)k_class<E, 0, 1, DST>,
                                   (const void*)k_class_persist<E, 0, 0, DST>, (const void*)k_class_persist<E, 0, 1, DST>,
                                   (const void*)k_class_wave<E, 0, 0, DST>,    (const void*)k_class_wave<E, 0, 1, DST>};
        return t[2 * form + mixed];
    }
    // variant = 4 persistent + 2 mode + mixed (FP64 prefix and FP32 suffix of
    // every task); bit 4: one task per wave (persistent); bits 5-6: staged
    // D' rows (1: shell a's, 2: both shells'; LDS digestion only)
    static const void* get(int variant) {
        if (const int ds = (variant >> 5) & 3) {
            if constexpr (kStage) {
                if (variant & 2) return nullptr;
                const int form = (variant & 16) ? 2 : (variant & 4) ? 1 : 0;
                return ds == 1 ? staged<1>(form, variant & 1) : staged<3>(form, variant & 1);
            } else {
                return nullptr;
            }
        }
        if (variant & 16) {
            static const void* w[4] = {(const void*)k_class_wave<E, 0, 0>, (const void*)k_class_wave<E, 0, 1>,
                                       (const void*)k_class_wave<E, 1, 0>, (const void*)k_class_wave<E, 1, 1>};
            return w[variant & 3];
        }
        static const void* t[8] = {(const void*)k_class<E, 0, 0>,         (const void*)k_class<E, 0, 1>,
                                   (const void*)k_class<E, 1, 0>,         (const void*)k_class<E, 1, 1>,
                                   (const void*)k_class_persist<E, 0, 0>, (const void*)k_class_persist<E, 0, 1>,
                                   (const void*)k_class_persist<E, 1, 0>, (const void*)k_class_persist<E, 1, 1>};
        return t[variant];
    }
};

// variant bit 3: the class's alternative workgroup size (EA; the same kernels
// when EA has E's size); bit 4: one task per wave.
template <class E, class EA>
struct ClassKernels {
    static const void* get(int variant) {
        if constexpr (EA::WGS != E::WGS) {
            if (variant & 8) return ClassKernelsOne<EA>::get(variant & 119);
        }
        return ClassKernelsOne<E>::get(variant & 119);
    }
};

// Register-tiled kernels of one class: variant = mode + 2 kpi + 6 (NBL - 1),
// ket primitive count 1, 3 or 9 (kpi 0, 1, 2), blocks of 1 or 2 bras.
template <class E>
struct ClassKernelsKr {
    static const void* get(int v) {
        static const void* t[12] = {
            (const void*)k_class_kr<E, 0, 1, 1>, (const void*)k_class_kr<E, 1, 1, 1>,
            (const void*)k_class_kr<E, 0, 3, 1>, (const void*)k_class_kr<E, 1, 3, 1>,
            (const void*)k_class_kr<E, 0, 9, 1>, (const void*)k_class_kr<E, 1, 9, 1>,
            (const void*)k_class_kr<E, 0, 1, 2>, (const void*)k_class_kr<E, 1, 1, 2>,
            (const void*)k_class_kr<E, 0, 3, 2>, (const void*)k_class_kr<E, 1, 3, 2>,
            (const void*)k_class_kr<E, 0, 9, 2>, (const void*)k_class_kr<E, 1, 9, 2>};
        return (v >= 0 && v < 12) ? t[v] : nullptr;
    }
};

// Register-tiled kernels use the class's alternative (smaller) workgroup
// size: the ket primitives in registers need more than the 128 VGPRs a
// 1024-lane workgroup leaves each lane.
#define HFX_CLASS_KR(cid) \
    extern "C" const void* hfx_class_kernel_kr_##cid(int v) { return ClassKernelsKr<Eval##cid##A>::get(v); }
#define HFX_CLASS_NO_KR(cid) \
    extern "C" const void* hfx_class_kernel_kr_##cid(int) { return nullptr; }

// Per-class translation unit: evaluator wrapper, the kernel variants, the
// Schwarz kernel and C lookups.
#define HFX_CLASS_TU(cid, fname, la_, lb_, lc_, ld_, wgs_, wgs_alt_)                                               \
    struct Eval##cid {                                                                                 \
        static constexpr int LA = la_, LB = lb_, LC = lc_, LD = ld_, WGS = wgs_;                       \
        template <typename R, typename SP = double>                                                    \
        __device__ __forceinline__ static void run(const SP* bp, int nbp, const SP* kq0, int kfs,      \
                                                   int kps, int nkp, const double* ab,                 \
                                                   const double* cd, const double* tab, R* out) {      \
            fname<R, SP>(bp, nbp, kq0, kfs, kps, nkp, R(ab[0]), R(ab[1]), R(ab[2]), R(cd[0]),          \
                         R(cd[1]), R(cd[2]), tab, out);                                                \
        }                                                                                              \
        template <typename R, int KP>                                                                  \
        __device__ __forceinline__ static void run_kr(const PrimPair* bp, int nbp,                     \
                                                      const R (&kv)[KP][9], const double* ab,          \
                                                      const double* cd, const double* tab, R* out) {   \
            fname##_kr<R, KP>(bp, nbp, kv, R(ab[0]), R(ab[1]), R(ab[2]), R(cd[0]), R(cd[1]),           \
                              R(cd[2]), tab, out);                                                     \
        }                                                                                              \
    };                                                                                                 \
    struct Eval##cid##A : Eval##cid {                                                                   \
        static constexpr int WGS = wgs_alt_;                                                           \
    };                                                                                                 \
    extern "C" const void* hfx_class_kernel_##cid(int variant) {                                       \
        return ClassKernels<Eval##cid, Eval##cid##A>::get(variant);                                    \
    }                                                                                                  \
    extern "C" const void* hfx_class_kernel_multi_##cid(int mode) {                                   \
        return mode ? (const void*)k_class_multi<Eval##cid, 1> : (const void*)k_class_multi<Eval##cid, 0>; \
    }                                                                                                  \
    extern "C" const void* hfx_schwarz_kernel_##cid(void) { return (const void*)k_schwarz<Eval##cid>; }
