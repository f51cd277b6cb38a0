// Internal data layout and device helpers of the HIP Fock-build library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// ---- shell-pair data in HBM ---------------------------------------------------
// One primitive pair (alpha on the pair's first shell A, beta on B) in the
// pair's canonical orientation (l_A >= l_B):
//   p = alpha + beta, inv2p = 1/(2p), P = (alpha A + beta B)/p, PA = P - A,
//   K = c_A c_B exp(-alpha beta/p |AB|^2) sqrt(2 pi^{5/2}) / p
// so that the quartet prefactor 2 pi^{5/2}/(p q sqrt(p+q)) K_ab K_cd is
// K_bra K_ket / sqrt(p+q).  80 bytes, read per lane from L2.
struct PrimPair {
    double p, inv2p;
    double P[3];
    double PA[3];
    double K;
    double pad;
};
#define HFX_PRIM_FIELDS 10   // elements of one PrimPair (an FP32 copy has the same layout in floats)
// LDS digestion with the bra's D' rows staged in LDS: classes with at most
// this many integrals per quartet (two more kernel variants per launch form)
#define HFX_STAGE_D_MAX_NI 64

// One shell pair in canonical orientation: shells a (higher l) and b, their
// first basis functions, its primitive pairs, its Schwarz bound and A - B.
struct PairInfo {
    int a, b;          // shells (global index)
    int bfa, bfb;      // first basis functions, local to the molecule
    int prim_off, nprim;
    double Q;
    double AB[3];
    int mol;           // molecule of a batch
    int ld;            // its basis size (leading dimension of its blocks)
};

// Workgroups of one launch at most: 2^20 x 1024 lanes stay below the grid limit of
// 2^32 work-items; a multiple of 8 keeps workgroup i on XCD i mod 8 in step with
// the task queues.
constexpr int HFX_MAX_GROUPS = 1 << 20;

// An element of a ket list's blocks: its place in the ragged matrices (< 0:
// padding between lists) and the product of its component factors.
struct KetElem {
    long long idx;
    double s;
};

// What the start of a build writes (misc_kernels.hip, k_start_build).
struct StartBufs {
    double *Dp, *W, *dket, *wket;
    unsigned long long* dmax_bits;   // null: max |D| not needed (FP64 builds)
    unsigned long long* counters;
    int ncounters;
    unsigned long long* work;
    int nwork;
};

// One ket list (pairs of one class with one primitive count) in the context's
// arrays, which hold the lists one after the other.
struct KetListDev {
    long long soa;     // its first element of the ket primitives
    long long koff;    // and of the ket blocks (dket, wket)
    int s0;            // its first ket
    int n, kp;         // kets, primitive pairs per ket
    int pad;
};

// A task's last word: column windows wc and wd, and the ket list.  Contractions
// of 1 to HFX_MAX_NPRIM = 16 primitives have 97 primitive-pair counts, so a context
// has at most 97 x 6 pair classes x 3 sets = 1746 lists; 2^10 windows, none narrower
// than 300 columns, are 3e5 functions, whose matrices take 720 GB each.
constexpr int HFX_MAX_NPRIM = 16;
constexpr int HFX_TASK_WIN_BITS = 10, HFX_TASK_MAX_LISTS = 1 << (32 - 2 * HFX_TASK_WIN_BITS);
constexpr int hfx_task_code(int wc, int wd, int list) {
    return (int)((unsigned)wc | (unsigned)wd << HFX_TASK_WIN_BITS | (unsigned)list << 2 * HFX_TASK_WIN_BITS);
}
constexpr int hfx_task_wc(int w) { return w & ((1 << HFX_TASK_WIN_BITS) - 1); }
constexpr int hfx_task_wd(int w) { return w >> HFX_TASK_WIN_BITS & ((1 << HFX_TASK_WIN_BITS) - 1); }
constexpr int hfx_task_list(int w) { return (int)((unsigned)w >> 2 * HFX_TASK_WIN_BITS); }

// Arguments of one class kernel launch, whose tasks may be of several ket
// lists of the class.  The kets of a task all have the same number of primitive
// pairs (knprim), so the primitive loop trip count is uniform across a wave.
// Ket primitive data are a structure of arrays: field f (the PrimPair member
// order p, inv2p, P[3], PA[3], K) of primitive k of ket s of a list at
// kprim[(f * knprim + k) * nket_list + s].  The host passes the arrays of all
// lists; of_list() gives a task's view.
struct ClassArgs {
    const PairInfo* __restrict__ bra;   // bra pairs of the class, Q descending
    const PairInfo* __restrict__ ket;   // ket pairs (one primitive count), Q descending
    const int4* __restrict__ kbf;       // per ket: first basis functions and shells (bfa, bfb, a, b)
    const double* __restrict__ dket;    // per build: D'_cd of every ket, [component][ket position]
    const PrimPair* __restrict__ prim;  // all primitive pairs (bra access)
    const double* __restrict__ kprim;   // ket primitives, structure of arrays
    const float* __restrict__ prim32;   // FP32 copies of both (mixed builds: the FP32 evaluation reads
    const float* __restrict__ kprim32;  // them without conversions)
    const KetListDev* __restrict__ lists;
    int nket_list, knprim;              // of a task's list
    const int* __restrict__ split;      // mixed builds, per task: kets below this list position use FP64,
                                        // the rest FP32 (one launch evaluates both parts)
    const int4* __restrict__ tasks;     // (bra index, first ket, end ket, hfx_task_code); bra -1:
                                        // empty.  Task 8k + x is entry k of XCD x's queue.  Register-tiled
                                        // plans: bra index | (bras in the block - 1) << 28
    const double* __restrict__ ketq;    // register-tiled plans: Q of every ket (list order)
    const int* __restrict__ kpos;       // and its position in its pair class's Q-sorted list
    double tau;                         // Schwarz threshold
    int same;                           // bra and ket of the same pair class (ket position <= bra index)
    long long wrep;                     // private digestion: elements between the per-XCD replicas of W
                                        // (W is replica 0); 0: one shared W
    // multi-density builds (k_class_multi): ndens densities D' (and their J
    // accumulators W, K accumulators WK) dstride elements apart, their
    // gathered D'_cd (dket) and ket-block J accumulators (wket) kstride
    // elements apart
    int ndens;
    long long dstride, kstride;
    double* WK;
    int win, rs;                        // column window (0: whole rows) and LDS bra-row length (doubles)
    int dstage;                         // staged D' rows (0, 1: shell a's, 3: both): selects the kernel variant
    int task_off;                       // static launch: workgroup i runs task task_off + i
    unsigned long long* __restrict__ work;  // persistent launch: 8 per-XCD queue counters (zeroed before the
                                            // launch); null: one task per workgroup
    int qlen;                           // entries per XCD queue (tasks = 8 qlen)
    const long long* __restrict__ moff; // per molecule: element offset of its blocks in D', W
    const double* __restrict__ boys64;
    const double* __restrict__ rys;     // cooperative classes: the quadrature table of their point count
    const double* __restrict__ D;       // component-scaled density D'
    double* __restrict__ W;             // accumulator, F_2e = s (W + W^T) s / 8
    double* __restrict__ wket;          // LDS mode: ket-block J sums, [component][ket position]
    unsigned long long* __restrict__ counters;  // the class's quartet counters (HFX_CNT_CLASS words)
    int shard, nshards;                 // only bras with r % nshards == shard (1 shard: all)
    double cj, ck;                      // W_ab += cj*2 g D_cd ; W_ac -= ck g D_bd
};

// Constant address space: loads through such a pointer at a wave-uniform
// address become scalar (SMEM) loads.
#define HFX_CONST_AS __attribute__((address_space(4)))

// A task and a bra pair, both the same in every lane: read into scalar registers.
__device__ __forceinline__ int4 uniform_task(const int4* tasks, int ti) {
    const HFX_CONST_AS int* t = (const HFX_CONST_AS int*)(tasks + ti);
    return make_int4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ PairInfo uniform_pair(const PairInfo* pairs, int r) {
    const HFX_CONST_AS PairInfo* p = (const HFX_CONST_AS PairInfo*)pairs + r;
    PairInfo v;
    v.a = p->a;
    v.b = p->b;
    v.bfa = p->bfa;
    v.bfb = p->bfb;
    v.prim_off = p->prim_off;
    v.nprim = p->nprim;
    v.Q = p->Q;
    v.AB[0] = p->AB[0];
    v.AB[1] = p->AB[1];
    v.AB[2] = p->AB[2];
    v.mol = p->mol;
    v.ld = p->ld;
    return v;
}

// The arguments as the tasks of a list see them (w: the task's last word, the
// same in every lane: the list's record goes to scalar registers).
__device__ __forceinline__ ClassArgs of_list(const ClassArgs& a, int w) {
    const HFX_CONST_AS KetListDev* L =
        (const HFX_CONST_AS KetListDev*)a.lists + __builtin_amdgcn_readfirstlane(hfx_task_list(w));
    const int s0 = L->s0;
    const long long koff = L->koff, soa = L->soa;
    ClassArgs v = a;
    v.ket += s0;
    v.kbf += s0;
    v.ketq += s0;
    v.kpos += s0;
    v.dket += koff;
    v.wket += koff;
    v.kprim += soa;
    v.kprim32 += soa;
    v.nket_list = L->n;
    v.knprim = L->kp;
    return v;
}

// Evaluated-quartet counters of a build: per class, FP64 then FP32, each
// spread over HFX_CNT_SLOTS words one 128-byte line apart (a workgroup adds
// into slot blockIdx mod HFX_CNT_SLOTS), summed on the host.  Kernels add once
// per wave at the end of a persistent launch, once per workgroup in the
// static form: one hot word per class taking an atomic per wave and task cost
// more than some classes' integrals.
#define HFX_CNT_SLOTS 8
#define HFX_CNT_STRIDE 16
#define HFX_CNT_CLASS (2 * HFX_CNT_SLOTS * HFX_CNT_STRIDE)
#define HFX_CNT_WORDS (21 * HFX_CNT_CLASS)   // then one word: the non-finite flag

// Index (0..7) of the accelerator complex die (XCD) the wave runs on, read
// from the hardware register.  It only selects which private copy of the
// accumulator a wave adds into: device-wide atomics keep any choice correct.
__device__ __forceinline__ int hfx_xcc_id() {
    unsigned x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    return (int)(x & 7u);
}

// Sums over the two halves of the wave (BIT 5) or over the two rows of 16 lanes
// of each half (BIT 4) of two values: lanes with that bit 0 get the sum of
// even, the others that of odd.  Every lane of the wave calls it.
template <int BIT>
__device__ __forceinline__ double lane_pair_sum(double even, double odd) {
    const unsigned long long e = (unsigned long long)__double_as_longlong(even), o = (unsigned long long)__double_as_longlong(odd);
    unsigned r[4];
    if constexpr (BIT == 5) {
        const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)e, (unsigned)o, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(e >> 32), (unsigned)(o >> 32), false, false);
        r[0] = lo[0]; r[1] = lo[1]; r[2] = hi[0]; r[3] = hi[1];
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)e, (unsigned)o, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(e >> 32), (unsigned)(o >> 32), false, false);
        r[0] = lo[0]; r[1] = lo[1]; r[2] = hi[0]; r[3] = hi[1];
    }
    return __longlong_as_double((long long)(((unsigned long long)r[2] << 32) | r[0])) +
           __longlong_as_double((long long)(((unsigned long long)r[3] << 32) | r[1]));
}
// Sum over the wave, in every lane: lane exchanges within rows of 16 by DPP,
// across rows and halves by permlane swaps (no LDS round trips).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
    const unsigned a = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const unsigned b = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return v + __longlong_as_double((long long)(((unsigned long long)b << 32) | a));
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xb1>(v);    // quad_perm 1 0 3 2
    v = dpp_add<0x4e>(v);    // quad_perm 2 3 0 1
    v = dpp_add<0x141>(v);   // row_half_mirror
    v = dpp_add<0x140>(v);   // row_mirror
    v = lane_pair_sum<4>(v, v);
    return lane_pair_sum<5>(v, v);
}

// ---- Boys function tables ---------------------------------------------------
// For every order l < BOYS_NL one block of BOYS_NT rows of 80 bytes:
//   row k: F_{l+j}(T_k) / j!, j = 0..8, then e^{-T_k},  T_k = k * BOYS_DT,
// so that F_l(T) = sum_j c_j d^j, d = T_k - T, about the nearest grid point
// (dF_m/dT = -F_{m+1}): 8 terms in FP64 (|d| <= 0.05: remainder < 1e-16 F), 5
// in FP32 (< 3e-9 F).  The class kernels copy the rows that their order needs
// into LDS.  The 80-byte stride lets the 16-byte reads of lanes at different
// rows start in 8 distinct groups of 4 of the 32 LDS banks (64 bytes: in 2).
#define BOYS_DT 0.1
#define BOYS_INV_DT 10.0
#define BOYS_NT 522
#define BOYS_NL 6
#define BOYS_ROW 10
#define BOYS_EXP 9        // e^{-T_k}
#define BOYS_ORDER64 8    // Taylor terms
#define BOYS_ORDER32 5
#define BOYS_TAB_ENTRIES (BOYS_NL * BOYS_NT * BOYS_ROW)
void hfx_boys_table(double* tab);   // host, BOYS_TAB_ENTRIES entries

// Where the asymptotic form F_m = (2m-1)!! / (2T)^m sqrt(pi/T)/2 takes over for
// total angular momentum L: its relative error, e^{-T} T^{L-1/2} /
// Gamma(L+1/2) for F_L and less for the lower orders, is below 1e-16 there.
__host__ __device__ constexpr int boys_tmax(int L) {
    return L <= 1 ? 40 : L == 2 ? 44 : L == 3 ? 46 : L == 4 ? 48 : 52;
}
__host__ __device__ constexpr int boys_rows(int L) { return boys_tmax(L) * 10 + 2; }
// The block that a class of total angular momentum L reads: its own order;
// L = 1 takes F_0 and F_1 = -dF_0/dT from the order-0 row.
__host__ __device__ constexpr int boys_block(int L) { return (L == 1 ? 0 : L) * BOYS_NT * BOYS_ROW; }
__host__ __device__ constexpr int boys_lds_bytes(int L) { return boys_rows(L) * BOYS_ROW * 8; }

// ---- Rys quadrature tables ----------------------------------------------------
// For n = RYS_NMIN..RYS_NMAX points, over T in [0, RYS_NT): per unit interval
// k and point r one row of RYS_NC coefficients of the root x_r = t_r^2 in
// powers of z = 2 (T - k) - 1, then RYS_NC of the weight w_r (12 coefficients:
// moments to 2e-15 relative, the rounding of the sums; 11 give 5e-15, 10 give
// 2e-13); after the intervals the n pairs (h_r, v_r) of the asymptotic
// x_r = h_r / T, w_r = v_r / sqrt(T).
#define RYS_NMIN 4
#define RYS_NMAX 5
#define RYS_NT 60
#define RYS_NC 12
#define RYS_ROW (2 * RYS_NC)
__host__ __device__ constexpr int rys_block(int n) {   // first entry of the n-point block
    int o = 0;
    for (int k = RYS_NMIN; k < n; ++k) o += RYS_NT * k * RYS_ROW + 2 * RYS_NMAX;
    return o;
}
#define RYS_TAB_ENTRIES (rys_block(RYS_NMAX + 1))
void hfx_rys_table(double* tab);   // host, RYS_TAB_ENTRIES entries

// 1/sqrt(x) for x > 0: the hardware estimate, refined in FP64 by one
// third-order step y (1 + e/2 + 3 e^2/8), e = 1 - x y^2 (five operations; two
// Newton steps take seven), in FP32 by one Newton step.
__device__ __forceinline__ double hfx_rsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ float hfx_rsqrt(float x) {
    float y = __builtin_amdgcn_rsqf(x);
    return y * (1.5f - 0.5f * x * y * y);
}

__host__ __device__ constexpr double boys_inv_fact(int n) {
    double f = 1.0;
    for (int i = 2; i <= n; ++i) f *= i;
    return 1.0 / f;
}

template <typename R> struct BoysOrder;
template <> struct BoysOrder<double> { static constexpr int value = BOYS_ORDER64; };
template <> struct BoysOrder<float> { static constexpr int value = BOYS_ORDER32; };

// Nearest grid point: its row and d = T_k - T.  FP64: rounding by adding 1.5
// 2^52, whose low word is then k (two additions instead of two conversions,
// which run at a quarter of their rate); 24-bit product for the address.
__device__ __forceinline__ const double* boys_row(const double* tab, double T, double& d) {
    const double magic = 6755399441055744.0, t = fma(T, BOYS_INV_DT, magic);
    d = fma(t - magic, BOYS_DT, -T);
    return reinterpret_cast<const double*>(reinterpret_cast<const char*>(tab) +
                                           __umul24((unsigned)__double2loint(t), BOYS_ROW * 8u));
}
__device__ __forceinline__ const double* boys_row(const double* tab, float T, float& d) {
    const int k = (int)(T * float(BOYS_INV_DT) + 0.5f);
    d = float(k) * float(BOYS_DT) - T;
    return reinterpret_cast<const double*>(reinterpret_cast<const char*>(tab) + __umul24((unsigned)k, BOYS_ROW * 8u));
}

// First N coefficients of a row in the evaluation's precision.
template <int N, typename R>
__device__ __forceinline__ void boys_coefs(const double* __restrict__ row, R (&c)[N]) {
    const double2* r2 = reinterpret_cast<const double2*>(row);
#pragma unroll
    for (int i = 0; i < (N + 1) / 2; ++i) {
        const double2 v = r2[i];
        c[2 * i] = R(v.x);
        if (2 * i + 1 < N) c[2 * i + 1] = R(v.y);
    }
}

// F_0(X / s) / sqrt(s) of a class with L = 0, X = p q |PQ|^2 and s = p + q: one
// reciprocal square root serves both regimes (far: sqrt(pi)/2 / sqrt(X)).
template <typename R>
__device__ __forceinline__ R boys_zero(R s, R X, const double* __restrict__ tab) {
    constexpr int NO = BoysOrder<R>::value;
    const bool far = X >= R(boys_tmax(0)) * s;
    const R y = hfx_rsqrt(far ? X : s);
    R f = R(0.886226925452758013649083741671);   // sqrt(pi)/2
    if (!far) {
        R d, c[NO];
        boys_coefs<NO>(boys_row(tab, X * (y * y), d), c);
        f = c[NO - 1];
#pragma unroll
        for (int j = NO - 2; j >= 0; --j) f = c[j] + f * d;
    }
    return f * y;
}

// F[0..L] at T, L >= 1; tab: the rows of boys_block(L).  Near: L = 1, F_0 and
// F_1 as the value and the derivative of one polynomial of one term more; L >=
// 2, F_L by Taylor expansion, e^{-T} = e^{-T_k} e^d (a 9- or 5-term series)
// and the downward recursion F_m = (2T F_{m+1} + e^{-T}) / (2m+1).  Far: the
// asymptotic form, no exponential.  Lanes of a wave usually straddle the two.
// Against 64-bit-exact values over 0 <= T <= 150 the largest relative error of
// an order up to 5 is 2.1e-15 (2.9e-15 with the exponential function and
// upward recursion in this place).  A primitive quartet of the low classes is
// bound by about 50 vector instructions and 4 LDS row reads; this form with
// hfx_rsqrt took the 64-water launches of (ss|ss) from 20.2 to 18.0 ms,
// (ps|ss) from 19.9 to 18.4, (ds|ss) from 12.7 to 11.4 and (ds|ps) from 8.8 to
// 8.5, a 44-carbon bilayer's (ps|ps) from 10.4 to 7.4 and (ps|ss) from 9.0 to
// 7.7 ms.
template <typename R, int L>
__device__ __forceinline__ void boys_eval(R T, R* F, const double* __restrict__ tab) {
    static_assert(L >= 1 && L < BOYS_NL, "orders of the table");
    constexpr int NO = BoysOrder<R>::value;
    if (T < R(boys_tmax(L))) {
        R d;
        const double* row = boys_row(tab, T, d);
        if constexpr (L == 1) {
            R c[NO + 1];
            boys_coefs<NO + 1>(row, c);
            R f = c[NO], g = c[NO];
#pragma unroll
            for (int j = NO - 1; j >= 1; --j) {
                f = c[j] + f * d;
                g = f + g * d;
            }
            F[0] = c[0] + f * d;
            F[1] = g;
        } else {
            R c[NO];
            boys_coefs<NO>(row, c);
            R f = c[NO - 1];
#pragma unroll
            for (int j = NO - 2; j >= 0; --j) f = c[j] + f * d;
            constexpr int NE = sizeof(R) == 8 ? 9 : 5;
            R e = R(boys_inv_fact(NE - 1));   // (e^d - 1) / d
#pragma unroll
            for (int j = NE - 2; j >= 1; --j) e = R(boys_inv_fact(j)) + e * d;
            const R ek = R(row[BOYS_EXP]);
            e = ek + ek * (e * d);
            F[L] = f;
            const R t2 = R(2) * T;
#pragma unroll
            for (int m = L - 1; m >= 0; --m) F[m] = (t2 * F[m + 1] + e) * R(1.0 / (2 * m + 1));
        }
    } else {
        const R rt = hfx_rsqrt(T), h = R(0.5) * rt * rt;   // 1 / (2T)
        F[0] = R(0.886226925452758013649083741671) * rt;
#pragma unroll
        for (int m = 0; m < L; ++m) F[m + 1] = R(2 * m + 1) * h * F[m];
    }
}

constexpr int hfx_ncart(int l) { return (l + 1) * (l + 2) / 2; }
// LDS doubles of the J sums of a bra block of n components (an even number)
constexpr int hfx_jsum_doubles(int n) { return (n + 1) / 2 * 2; }
