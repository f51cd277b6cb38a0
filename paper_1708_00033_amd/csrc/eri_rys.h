// Cooperative Rys-quadrature kernels of the large quartet classes.
//
// The integrals of a class with a d shell on the bra and 200 to 1300
// integrals per quartet do not fit in one lane: evaluated per lane (vertical
// and horizontal recurrences) they spilled 2-7 KB per lane to scratch at one
// wave per SIMD and ran below 2 % of the FP64 rate.  Here the lanes of a
// workgroup share the quartets of a batch of NK kets.  Every integral is
//   (ab|cd) = sum_r Ix_r(a_x, b_x, c_x, d_x) Iy_r(..) Iz_r(..)
// over the n = L/2 + 1 points of the Rys quadrature (Dupuis, Rys and King,
// J. Chem. Phys. 65, 111 (1976); Rys, Dupuis and King, J. Comput. Chem. 4,
// 154 (1983)), so the one-dimensional integrals of a primitive quartet, a few
// hundred numbers, are all that the lanes exchange:
//   phase 1, one lane per (ket, axis, root): quadrature point, the
//     two-index recurrence I(e, f), the bra transfer to I(a, b; f), into LDS;
//   phase 2, one lane per (ket, component pair (a_m b_n)): the products over
//     the axes summed over the roots and, in registers, over the primitives,
//     for l_c <= |f| <= l_c + l_d, then the ket transfer to (a_m b_n|cd) and
//     the six updates of eq. 2.
// A lane holds at most 31 accumulators and 36 integrals, so nothing spills
// and the code of a class is 10-20 KB instead of 70-330 KB.
//
// The K updates go to the bra's rows of W staged in LDS (MODE 0), or (MODE 1)
// into an LDS block per ket, (NA + NB) x (NC + ND), added to W with one
// global atomic per element and batch: 36 lanes of a quartet share those
// elements.  The ket block's J sums take the same way in both modes.  LDS
// atomics on shared addresses were the largest cost of a first version (36
// per lane, four to seven lanes of a wave on one address: 10,000 of 16,000
// cycles of a (dd|dp) batch).  So the lanes of a wave are arranged such that
// the sums over neighbouring components run across lane halves and rows
// (v_permlane32_swap, v_permlane16_swap: two values are summed and split over
// the two halves by one exchange and one addition), and each lane is left
// with a quarter or a half of the values and addresses of its own.
#pragma once
#include <type_traits>

#include "hfx_internal.h"

template <int LC, int LD>
struct RysKet {   // ket functions f of the contracted [ab|f0), by degree
    static constexpr int FM = LC + LD;
    static __host__ __device__ constexpr int cart_index(int y, int z) { return (y + z) * (y + z + 1) / 2 + z; }
    static __host__ __device__ constexpr int level(int l) {   // first index of degree l
        int o = 0;
        for (int k = LC; k < l; ++k) o += hfx_ncart(k);
        return o;
    }
    static constexpr int NF = level(FM + 1);
    static __host__ __device__ constexpr int index(int x, int y, int z) { return level(x + y + z) + cart_index(y, z); }
};

template <class E>
struct RysDims {
    static constexpr int LA = E::LA, LB = E::LB, LC = E::LC, LD = E::LD;
    static constexpr int NA = hfx_ncart(LA), NB = hfx_ncart(LB), NC = hfx_ncart(LC), ND = hfx_ncart(LD);
    static constexpr int NAB = NA * NB, NCD = NC * ND;
    static constexpr int NR = (LA + LB + LC + LD) / 2 + 1;
    static constexpr int EM = LA + LB, FM = LC + LD, F1 = FM + 1;
    static constexpr int AB1 = (LA + 1) * (LB + 1);
    static constexpr int NK = E::NK;                        // kets per batch: 8 or 16
    // lane of phase 2: ket (low bits), lane bits 4 and 5 and unit: with six
    // functions on shell b, unit = 2 x 2 components, bit 4 the low bit of n,
    // bit 5 that of m; with three (or one), bit 5 the low bit of m and bit 4
    // the low bit of the index of (m / 2, n)
    static constexpr bool SQUARE = NB == 6;
    static constexpr int UNITS = SQUARE ? (NA / 2) * (NB / 2) : ((NA / 2) * NB + 1) / 2;
    static constexpr int UPW = 16 / NK;                     // units per wave
    static constexpr int WAVES = (UNITS + UPW - 1) / UPW;
    static_assert(NA == 6 && (NK == 8 || NK == 16) && E::WGS == 64 * WAVES, "workgroup size");
    // one ket's one-dimensional integrals [axis + 3 root][a b][f]; the stride
    // between kets is odd or 4 mod 8 doubles, so that lanes of neighbouring kets
    // start in different LDS banks
    static constexpr int S1 = AB1 * F1;
    static constexpr int RAW = 3 * NR * S1;
    static constexpr int KET = F1 % 2 ? RAW | 1 : RAW + ((12 - RAW % 8) % 8);
    static constexpr int KC = NC + ND, KROWS = NA + NB;
    // The 48 registers of a table row fetched a step ahead pay where they do
    // not spill: (dp|dp) 10.5 ms with against 12.0 ms without (a 44-carbon
    // bilayer), (dd|dp) 3.6 against 3.8; the 576-lane workgroups (168
    // registers a lane) and (dd|dd) run faster without: (dd|ds) 3.6 ms against
    // 4.6 (64 waters), (dd|pp) 0.85 against 1.12, (dd|dd) 0.28 against 0.39.
    static constexpr bool PREFETCH = E::WGS <= 512 && RysKet<LC, LD>::NF <= 16;
    // LDS in doubles, without the rows of W: integrals, per density the ket
    // block's J sums and the bra block's, and (MODE 1) the K block per ket
    static __host__ __device__ constexpr int per_density(int mode) {
        return NK * NCD + NAB + (mode ? NK * KROWS * KC : 0);
    }
    static __host__ __device__ constexpr int lds(int mode, int ndens) {
        return ((NK * KET + ndens * per_density(mode)) + 1) & ~1;
    }
    static_assert(NK * 3 * NR <= E::WGS, "one phase-1 item per lane");
};

// Phase 2: a lane's ket slot, its components (m, n) of the bra pair and the
// offsets of their one-dimensional integrals in the ket's block.
struct RysLane {
    int j, mn, m, n, ox, oy, oz;
    bool on;
};

template <class E>
__device__ __forceinline__ RysLane rys_lane() {
    using X = RysDims<E>;
    RysLane l;
    const int lane = (int)threadIdx.x & 63, b4 = (lane >> 4) & 1, b5 = lane >> 5;
    const int unit = ((int)threadIdx.x >> 6) * X::UPW + (lane & 15) / X::NK;
    l.j = lane & (X::NK - 1);
    if constexpr (X::SQUARE) {
        l.on = unit < X::UNITS;
        l.m = 2 * (unit / (X::NB / 2)) + b5;
        l.n = 2 * (unit % (X::NB / 2)) + b4;
    } else {
        const int u = 2 * unit + b4;
        l.on = u < (X::NA / 2) * X::NB;
        l.m = 2 * (u / X::NB) + b5;
        l.n = u % X::NB;
    }
    if (!l.on) l.m = l.n = 0;
    l.mn = l.m * X::NB + l.n;
    // component index = yz (yz + 1) / 2 + z, yz = y + z <= 2
    const int myz = l.m < 1 ? 0 : l.m < 3 ? 1 : 2, mz = l.m - myz * (myz + 1) / 2;
    const int nyz = l.n < 1 ? 0 : l.n < 3 ? 1 : 2, nz = l.n - nyz * (nyz + 1) / 2;
    constexpr int LB1 = X::LB + 1;
    l.ox = ((X::LA - myz) * LB1 + (X::LB - nyz)) * X::F1;
    l.oy = X::S1 + ((myz - mz) * LB1 + (nyz - nz)) * X::F1;
    l.oz = 2 * X::S1 + (mz * LB1 + nz) * X::F1;
    return l;
}

// The table entries of quadrature point r of NR at T (loads only): the
// interval's coefficients of the root, then of the weight, or above RYS_NT
// the asymptotic pair.
template <int NR, typename R>
__device__ __forceinline__ void rys_point_load(R T, int r, const double* __restrict__ tab, double2 (&c)[RYS_NC]) {
    const bool near = T < R(RYS_NT);
    const int k = near ? (int)T : RYS_NT;
    const double2* __restrict__ row =
        reinterpret_cast<const double2*>(tab + (near ? ((size_t)k * NR + r) * RYS_ROW : (size_t)RYS_NT * NR * RYS_ROW + 2 * r));
    c[0] = row[0];
    if (near) {
#pragma unroll
        for (int i = 1; i < RYS_NC; ++i) c[i] = row[i];
    }
}

// Root x = t^2 and weight from those entries.
template <typename R>
__device__ __forceinline__ void rys_point(R T, const double2 (&c)[RYS_NC], R& x, R& w) {
    if (T < R(RYS_NT)) {
        const R z = R(2) * (T - R((int)T)) - R(1);
        x = R(c[RYS_NC / 2 - 1].y);
        w = R(c[RYS_NC - 1].y);
#pragma unroll
        for (int i = RYS_NC - 2; i >= 0; --i) {
            x = R(i & 1 ? c[i / 2].y : c[i / 2].x) + x * z;
            w = R(i & 1 ? c[(RYS_NC + i) / 2].y : c[(RYS_NC + i) / 2].x) + w * z;
        }
    } else {
        const R rt = hfx_rsqrt(T);
        x = R(c[0].x) * rt * rt;
        w = R(c[0].y) * rt;
    }
}

// (a_m b_n|cd) from [ab|f0): (c, d + 1_i| = (c + 1_i, d| + CD_i (c, d|.
template <int LC, int LD, typename R>
__device__ __forceinline__ void rys_ket_transfer(const R* f, const R* cd, R* out) {
    using K = RysKet<LC, LD>;
    if constexpr (LD == 0) {
#pragma unroll
        for (int i = 0; i < K::NF; ++i) out[i] = f[i];
    } else {
        int o = 0;
#pragma unroll
        for (int cx = LC; cx >= 0; --cx)
#pragma unroll
            for (int cy = LC - cx; cy >= 0; --cy) {
                const int cz = LC - cx - cy;
                // (c + u, 1_i| for a displacement u of the first shell
                auto one = [&](int x, int y, int z, int i) {
                    return f[K::index(x + (i == 0), y + (i == 1), z + (i == 2))] + cd[i] * f[K::index(x, y, z)];
                };
                if constexpr (LD == 1) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) out[o++] = one(cx, cy, cz, i);
                } else {
                    static_assert(LD == 2, "s, p and d shells");
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int j = i; j < 3; ++j)   // d components xx xy xz yy yz zz
                            out[o++] = one(cx + (i == 0), cy + (i == 1), cz + (i == 2), j) + cd[i] * one(cx, cy, cz, j);
                }
            }
    }
}

// lane_pair_sum over N values: lane bit BIT = 0 is left with the sums of the
// values of even index, 1 with those of odd index.
template <int BIT, int N>
__device__ __forceinline__ void rys_split_sums(const double* v, double* out) {
#pragma unroll
    for (int i = 0; i < (N + 1) / 2; ++i) out[i] = lane_pair_sum<BIT>(v[2 * i], 2 * i + 1 < N ? v[2 * i + 1] : 0.0);
}

// A lane's ket primitive in phase 1 and, for one bra primitive, what is ready
// before the table entries arrive.
template <typename R>
struct RysPrim {
    R q, i2q, Q0, Q1, Q2, QC, K;
};
template <typename R>
struct RysFront {
    R p, i2p, q, i2q, ipq, T, PA, PQ, QC, pre;
    double2 c[RYS_NC];
};

// Phase 1 and 2 of a workgroup's sequence of (batch, ket primitive, bra
// primitive) steps.  kprim: field f of primitive k of ket j at
// [f kfs + k kps + j].
//
// At the sizes where the rows of W leave room for one workgroup per CU the
// steps are bound by latency (about 4,000 cycles, a third of it in each of
// phase 1, the next step's preparation and phase 2), so each step's loads are
// issued ahead: the ket primitives two steps, the quadrature table's entries
// (PREFETCH) one step before their use, over phase 2 of the steps between.
template <class E, typename R, typename SP>
struct RysSteps {
    using X = RysDims<E>;
    using K = RysKet<X::LC, X::LD>;
    using Real = R;
    static constexpr int NR = X::NR, EM = X::EM, FM = X::FM, F1 = X::F1;
    const double* __restrict__ tab;
    const SP* __restrict__ bprim;
    const SP* __restrict__ kprim;
    int nbp, nkp, kps, kfs, nket;    // nket: kets of the sequence
    R ab;                            // AB of this lane's axis
    R* __restrict__ g1;
    const R* __restrict__ g2;
    int j1, ax, root;
    bool lane1;
    // next step to fetch ket primitives for, and next to prepare
    int pb, pk, fb, fk, fi;          // batch start and ket primitive; batch start, ket and bra primitive
    RysPrim<R> prim;
    RysFront<R> front;
    R bp, bi2p, bP0, bP1, bP2, bPA, bK;   // the bra primitive of the next step (bPA: of this lane's axis)

    __device__ __forceinline__ RysSteps(const double* tab_, const SP* bprim_, int nbp_, const SP* kprim_, int nkp_,
                                        int kps_, int kfs_, int nket_, double ab0, double ab1, double ab2, R* G, int j2)
        : tab(tab_), bprim(bprim_), kprim(kprim_), nbp(nbp_), nkp(nkp_), kps(kps_), kfs(kfs_), nket(nket_) {
        const int tid = (int)threadIdx.x;
        j1 = tid % X::NK;
        const int xr = tid / X::NK;   // axis + 3 root
        lane1 = xr < 3 * NR;
        ax = xr % 3;
        root = xr / 3;
        ab = R(ax == 0 ? ab0 : ax == 1 ? ab1 : ab2);
        g1 = G + j1 * X::KET + xr * X::S1;
        g2 = G + j2 * X::KET;
        pb = pk = fb = fk = fi = 0;
        prim = RysPrim<R>{R(1), R(0), R(0), R(0), R(0), R(0), R(0)};
        load_bra();
        fetch();
        prepare();
    }
    __device__ __forceinline__ void load_bra() {
        const HFX_CONST_AS SP* B = (const HFX_CONST_AS SP*)(bprim + fi * HFX_PRIM_FIELDS);
        bp = R(B[0]);
        bi2p = R(B[1]);
        bP0 = R(B[2]);
        bP1 = R(B[3]);
        bP2 = R(B[4]);
        bPA = R(bprim[fi * HFX_PRIM_FIELDS + 5 + ax]);
        bK = R(B[8]);
    }
    __device__ __forceinline__ bool on(int base) const { return lane1 && base + j1 < nket; }

    // Loads of the next ket primitives.
    __device__ __forceinline__ void fetch() {
        if (on(pb)) {
            const SP* kq = kprim + (size_t)pk * kps + pb + j1;
            prim.q = R(kq[0]);
            prim.i2q = R(kq[kfs]);
            prim.Q0 = R(kq[2 * (size_t)kfs]);
            prim.Q1 = R(kq[3 * (size_t)kfs]);
            prim.Q2 = R(kq[4 * (size_t)kfs]);
            prim.QC = R(kq[(5 + ax) * (size_t)kfs]);
            prim.K = R(kq[8 * (size_t)kfs]);
        }
        if (++pk == nkp) {
            pk = 0;
            pb += X::NK;
        }
    }
    // The next step up to the loads of its table entries.  The loads of the
    // following ket primitives go out before those: waiting for them must not
    // wait for the table.
    __device__ __forceinline__ void prepare() {
        const bool now = on(fb);
        if (now) {
            const R p = bp, q = prim.q;
            const R PQ0 = bP0 - prim.Q0, PQ1 = bP1 - prim.Q1, PQ2 = bP2 - prim.Q2;
            const R rs = hfx_rsqrt(p + q), ipq = rs * rs;
            front.p = p;
            front.i2p = bi2p;
            front.q = q;
            front.i2q = prim.i2q;
            front.ipq = ipq;
            front.T = p * q * ipq * (PQ0 * PQ0 + PQ1 * PQ1 + PQ2 * PQ2);
            front.PA = bPA;
            front.PQ = ax == 0 ? PQ0 : ax == 1 ? PQ1 : PQ2;
            front.QC = prim.QC;
            front.pre = bK * prim.K * rs;
        }
        if (++fi == nbp) {
            fi = 0;
            if (++fk == nkp) {
                fk = 0;
                fb += X::NK;
            }
            if (fb < nket) fetch();
        }
        if (nbp > 1) load_bra();   // one primitive: loaded once
        if (X::PREFETCH && now) rys_point_load<NR>(front.T, root, tab, front.c);
    }
    // One step of the batch at base: phase 1 of the prepared step, the next
    // step's preparation, phase 2 into acc.  Ends after a barrier.
    __device__ __forceinline__ void step(int base, const RysLane& ln, bool on2, R* acc) {
        if (on(base)) {
            R u, w;
            if constexpr (!X::PREFETCH) rys_point_load<NR>(front.T, root, tab, front.c);
            rys_point(front.T, front.c, u, w);
            const R up = u * front.ipq;   // u / (p + q)
            const R b00 = R(0.5) * up, b10 = front.i2p * (R(1) - front.q * up), b01 = front.i2q * (R(1) - front.p * up);
            const R c0 = front.PA - front.q * up * front.PQ, d0 = front.QC + front.p * up * front.PQ;
            R I[EM + 1][F1];
            I[0][0] = ax == 2 ? w * front.pre : R(1);
#pragma unroll
            for (int e = 0; e < EM; ++e) I[e + 1][0] = c0 * I[e][0] + (e ? R(e) * b10 * I[e - 1][0] : R(0));
#pragma unroll
            for (int f = 0; f < FM; ++f)
#pragma unroll
                for (int e = 0; e <= EM; ++e) {
                    R v = d0 * I[e][f];
                    if (f) v += R(f) * b01 * I[e][f - 1];
                    if (e) v += R(e) * b00 * I[e - 1][f];
                    I[e][f + 1] = v;
                }
            // bra transfer per axis: (a, b + 1) = (a + 1, b) + AB (a, b)
#pragma unroll
            for (int f = 0; f < F1; ++f)
#pragma unroll
                for (int i = 0; i <= X::LA; ++i) {
                    g1[(i * (X::LB + 1)) * F1 + f] = I[i][f];
                    const R h0 = I[i + 1][f] + ab * I[i][f];
                    g1[(i * (X::LB + 1) + 1) * F1 + f] = h0;
                    if constexpr (X::LB == 2) {
                        const R h1 = I[i + 2][f] + ab * I[i + 1][f];
                        g1[(i * (X::LB + 1) + 2) * F1 + f] = h1 + ab * h0;
                    }
                }
        }
        __syncthreads();
        if (fb < nket) prepare();
        if (on2) {
#pragma unroll 2
            for (int r = 0; r < NR; ++r) {
                const R* __restrict__ gr = g2 + r * (3 * X::S1);
                R x[F1], y[F1], z[F1];
#pragma unroll
                for (int f = 0; f < F1; ++f) {
                    x[f] = gr[ln.ox + f];
                    y[f] = gr[ln.oy + f];
                    z[f] = gr[ln.oz + f];
                }
#pragma unroll
                for (int fx = 0; fx <= FM; ++fx)
#pragma unroll
                    for (int fy = 0; fy <= FM - fx; ++fy) {
                        const R xy = x[fx] * y[fy];
#pragma unroll
                        for (int fz = 0; fz <= FM - fx - fy; ++fz)
                            if (fx + fy + fz >= X::LC) acc[K::index(fx, fy, fz)] += xy * z[fz];
                    }
            }
        }
        __syncthreads();
    }
    // All steps of the batch at base, then this lane's (a_m b_n|cd) block
    // (valid where its ket exists); kab: its ket's C - D.
    __device__ __forceinline__ void batch(int base, const RysLane& ln, bool on2, const double* kab, R* out) {
        const R cd[3] = {R(kab[0]), R(kab[1]), R(kab[2])};
        R acc[K::NF];
#pragma unroll
        for (int i = 0; i < K::NF; ++i) acc[i] = R(0);
#pragma unroll 1
        for (int n = nkp * nbp; n > 0; --n) step(base, ln, on2, acc);
        rys_ket_transfer<X::LC, X::LD>(acc, cd, out);
    }
};

// One task (one bra, a range of its kets) on the workgroup.  Counts the
// evaluated quartets of the workgroup on lane 0.
template <class E, int MODE, int FP32, bool MULTI>
__device__ __forceinline__ void class_task_rys(const ClassArgs& args, const int ti, unsigned& cnt64, unsigned& cnt32) {
    using X = RysDims<E>;
    constexpr int NA = X::NA, NB = X::NB, NC = X::NC, ND = X::ND, NCD = X::NCD, NK = X::NK, NT = E::WGS;
    extern __shared__ __align__(16) double lds[];
    const int4 task = uniform_task(args.tasks, __builtin_amdgcn_readfirstlane(ti));
    const int r = task.x;
    if (!task_active(args, task)) return;
    const ClassArgs a = of_list(args, task.w);
    const int s0 = task.y, send = task.z;
    const int split = FP32 ? min(max(a.split[ti], s0), send) : send;
    const PairInfo bra = uniform_pair(a.bra, r);
    const int N = bra.ld, tid = (int)threadIdx.x;
    const size_t mo = (size_t)a.moff[bra.mol] + (a.wrep ? (size_t)hfx_xcc_id() * a.wrep : 0);
    const int ndens = MULTI ? a.ndens : 1;
    // LDS: integrals, then per density the small sums, then the rows
    double* S0 = lds + NK * X::KET;
    double* F0 = lds + X::lds(MODE, ndens);
    constexpr int PD = X::per_density(MODE);
    const int rowset = (NA + NB) * a.rs;
    int RS = N, cb = 0, db = 0, half = N;   // column windows as in class_task
    if (a.win) {
        RS = a.rs;
        half = RS / 2;
        const int wc = hfx_task_wc(task.w), wd = hfx_task_wd(task.w);
        cb = wc * a.win;
        db = wd == wc ? cb : wd * a.win - half;
    }
    for (int i = tid; i < ndens * PD; i += NT) S0[i] = 0.0;
    if constexpr (MODE == 0)
        for (int i = tid; i < ndens * rowset; i += NT) F0[i] = 0.0;
    const RysLane ln = rys_lane<E>();
    const int j2 = ln.j, mn = ln.mn, m = ln.m, n = ln.n;
    const double sbra = bra.a != bra.b ? 2.0 : 1.0;
    double jab = 0.0;
    const double dab1 = MULTI ? 0.0 : a.D[(size_t)a.moff[bra.mol] + (size_t)(bra.bfa + m) * N + bra.bfb + n];
    __syncthreads();
    // the six updates of one batch (v: this lane's integrals, kb: its ket's record)
    auto digest = [&](int base, int cnt, bool on2, const int4 kb, const double* v) {
        const int s = base + (on2 ? j2 : 0);
        // lanes without a ket add zeros, to their own slot of the batch
        const double g = !on2 ? 0.0
                              : sbra * (kb.z != kb.w ? 2.0 : 1.0) * ((kb.z == bra.a && kb.w == bra.b) ? 1.0 : 2.0);
        const double ckg = -a.ck * g;
        const int fc = kb.x, fd = kb.y;
        constexpr int NV = NC + ND;
        const int b4 = (tid >> 4) & 1, b5 = (tid >> 5) & 1;
        for (int d = 0; d < ndens; ++d) {
            const double* __restrict__ Dm = a.D + (size_t)a.moff[bra.mol] + (MULTI ? (size_t)d * a.dstride : 0);
            const double* __restrict__ Da = Dm + (size_t)(bra.bfa + m) * N;
            const double* __restrict__ Db = Dm + (size_t)(bra.bfb + n) * N;
            const double* __restrict__ dk = a.dket + (MULTI ? (size_t)d * a.kstride : 0) + s;
            const double gd = 2.0 * a.cj * g * (MULTI ? Da[bra.bfb + n] : dab1);
            // every load before the first atomic: the compiler keeps their order
            double dcd[NCD], dac[NC], dbc[NC], dad[ND], dbd[ND];
#pragma unroll
            for (int i = 0; i < NCD; ++i) dcd[i] = dk[(size_t)i * a.nket_list];
#pragma unroll
            for (int l = 0; l < NC; ++l) {
                dac[l] = Da[fc + l];
                dbc[l] = Db[fc + l];
            }
#pragma unroll
            for (int q = 0; q < ND; ++q) {
                dad[q] = Da[fd + q];
                dbd[q] = Db[fd + q];
            }
            // K: W_ac -= ck g I D_bd and W_ad -= ck g I D_bc (summed over the
            // two n of the unit), W_bc -= ck g I D_ad and W_bd -= ck g I D_ac
            // (over its two m)
            double wa[NV], wb[NV];
#pragma unroll
            for (int l = 0; l < NC; ++l) {
                wa[l] = wb[l] = 0.0;
#pragma unroll
                for (int q = 0; q < ND; ++q) {
                    wa[l] += v[l * ND + q] * dbd[q];
                    wb[l] += v[l * ND + q] * dad[q];
                }
            }
#pragma unroll
            for (int q = 0; q < ND; ++q) {
                wa[NC + q] = wb[NC + q] = 0.0;
#pragma unroll
                for (int l = 0; l < NC; ++l) {
                    wa[NC + q] += v[l * ND + q] * dbc[l];
                    wb[NC + q] += v[l * ND + q] * dac[l];
                }
            }
            double *ra, *rb;   // rows of W of a_m and b_n; columns of c and d at oc, od
            int oc, od;
            if constexpr (MODE == 0) {
                ra = F0 + d * rowset + m * RS;
                rb = F0 + d * rowset + (NA + n) * RS;
                oc = fc - cb;
                od = fd - db;
            } else {
                double* k0 = S0 + d * PD + NK * NCD + X::NAB + j2 * (X::KROWS * X::KC);
                ra = k0 + m * X::KC;
                rb = k0 + (NA + n) * X::KC;
                oc = 0;
                od = NC;
            }
            double sum[(NV + 1) / 2];
            if constexpr (X::SQUARE) {
                rys_split_sums<4, NV>(wa, sum);
#pragma unroll
                for (int i = 0; i < (NV + 1) / 2; ++i) {
                    const int k = 2 * i + b4;
                    if (on2 && k < NV) atomicAdd(ra + (k < NC ? oc + k : od + k - NC), ckg * sum[i]);
                }
            } else {
                if (on2) {
#pragma unroll
                    for (int k = 0; k < NV; ++k) atomicAdd(ra + (k < NC ? oc + k : od + k - NC), ckg * wa[k]);
                }
            }
            rys_split_sums<5, NV>(wb, sum);
#pragma unroll
            for (int i = 0; i < (NV + 1) / 2; ++i) {
                const int k = 2 * i + b5;
                if (on2 && k < NV) atomicAdd(rb + (k < NC ? oc + k : od + k - NC), ckg * sum[i]);
            }
            // J: the bra block per lane, the ket block summed over the unit
            double t = 0.0, jv[NCD], h[(NCD + 1) / 2], q4[((NCD + 1) / 2 + 1) / 2];
#pragma unroll
            for (int i = 0; i < NCD; ++i) {
                t += v[i] * dcd[i];
                jv[i] = gd * v[i];
            }
            if constexpr (MULTI) {
                if (on2) atomicAdd(S0 + d * PD + NK * NCD + mn, g * t);
            } else {
                jab += g * t;
            }
            rys_split_sums<5, NCD>(jv, h);
            rys_split_sums<4, (NCD + 1) / 2>(h, q4);
            double* jk = S0 + d * PD + j2 * NCD;
#pragma unroll
            for (int i = 0; i < ((NCD + 1) / 2 + 1) / 2; ++i) {
                const int k = 4 * i + 2 * b4 + b5;
                if (k < NCD) atomicAdd(jk + k, q4[i]);
            }
        }
        __syncthreads();
        // the batch's ket-block sums (and MODE 1: K blocks) into memory,
        // cleared for the next batch (whose updates come after further barriers)
        // (from the last wave down: phase 1 of the next batch runs on the first
        // waves and would wait for their atomics)
        for (int i = NT - 1 - tid; i < ndens * NK * NCD; i += NT) {
            const int d = MULTI ? i / (NK * NCD) : 0, x = i - d * (NK * NCD), j = x / NCD, q = x % NCD;
            double* jk = S0 + d * PD + x;
            if (j < cnt) {
                const double t = *jk;
                *jk = 0.0;
                if constexpr (MODE == 0) {
                    atomicAdd(a.wket + (MULTI ? (size_t)d * a.kstride : 0) + (size_t)q * a.nket_list + base + j, t);
                } else {
                    const int4 kb = a.kbf[base + j];
                    atomicAdd(a.W + mo + (MULTI ? (size_t)d * a.dstride : 0) + (size_t)(kb.x + q / ND) * N + kb.y + q % ND,
                              t);
                }
            }
        }
        if constexpr (MODE == 1) {
            constexpr int KB = X::KROWS * X::KC;
            double* WK = MULTI ? a.WK : a.W;
            for (int i = tid; i < ndens * NK * KB; i += NT) {
                const int d = MULTI ? i / (NK * KB) : 0, x = i - d * (NK * KB), j = x / KB, row = (x % KB) / X::KC,
                          col = x % X::KC;
                if (j < cnt) {
                    double* kx = S0 + d * PD + NK * NCD + X::NAB + x;
                    const double t = *kx;
                    *kx = 0.0;
                    const int4 kb = a.kbf[base + j];
                    const int gr = row < NA ? bra.bfa + row : bra.bfb + row - NA;
                    const int gc = col < NC ? kb.x + col : kb.y + col - NC;
                    atomicAdd(WK + mo + (MULTI ? (size_t)d * a.dstride : 0) + (size_t)gr * N + gc, t);
                }
            }
        }
    };
    // the kets below split in FP64, then the others in FP32, each part in
    // batches of NK; part runs one of the two
    auto part = [&](int first, int end, auto& steps, unsigned& count) {
        for (int base = first; base < end; base += NK) {
            const int cnt = min(NK, end - base);
            const bool on2 = ln.on && j2 < cnt;
            const double* kab = a.ket[base + (on2 ? j2 : 0)].AB;
            const int4 kb = a.kbf[base + (on2 ? j2 : 0)];
            typename std::remove_reference<decltype(steps)>::type::Real v0[NCD];
            steps.batch(base - first, ln, on2, kab, v0);
            double v[NCD];
#pragma unroll
            for (int i = 0; i < NCD; ++i) v[i] = (double)v0[i];
            if (tid == 0) count += cnt;
            digest(base, cnt, on2, kb, v);
        }
    };
    if (s0 < split) {
        RysSteps<E, double, double> steps(a.rys, (const double*)(a.prim + bra.prim_off), bra.nprim, a.kprim + s0, a.knprim,
                                          a.nket_list, a.nket_list * a.knprim, split - s0, bra.AB[0], bra.AB[1],
                                          bra.AB[2], lds, j2);
        part(s0, split, steps, cnt64);
    }
    if constexpr (FP32)
        if (split < send) {
            RysSteps<E, float, float> steps(a.rys, a.prim32 + (size_t)bra.prim_off * HFX_PRIM_FIELDS, bra.nprim,
                                            a.kprim32 + split, a.knprim, a.nket_list, a.nket_list * a.knprim, send - split,
                                            bra.AB[0], bra.AB[1], bra.AB[2], (float*)lds, j2);
            part(split, send, steps, cnt32);
        }
    // the bra block's J sums, then the rows of W
    if constexpr (!MULTI)
        if (ln.on && j2 < send - s0) atomicAdd(S0 + NK * NCD + mn, jab);
    __syncthreads();
    for (int i = tid; i < ndens * X::NAB; i += NT) {
        const int d = i / X::NAB, q = i % X::NAB;
        atomicAdd(a.W + mo + (MULTI ? (size_t)d * a.dstride : 0) + (size_t)(bra.bfa + q / NB) * N + bra.bfb + q % NB,
                  2.0 * a.cj * S0[d * PD + NK * NCD + q]);
    }
    if constexpr (MODE == 0) {
        double* WK = MULTI ? a.WK : a.W;
        for (int i = tid >> 6; i < ndens * X::KROWS; i += NT >> 6) {   // a wave per row
            const int d = MULTI ? i / X::KROWS : 0, row = i - d * X::KROWS;
            const double* f = F0 + d * rowset + row * RS;
            double* w = WK + mo + (MULTI ? (size_t)d * a.dstride : 0) +
                        (size_t)(row < NA ? bra.bfa + row : bra.bfb + row - NA) * N;
            for (int c = tid & 63; c < RS; c += 64) {
                const double t = f[c];
                const int col = c + (c < half ? cb : db);
                if (t != 0.0 && col < N) atomicAdd(w + col, t);
            }
        }
    }
}

// Workgroup i runs task task_off + i, or (args.work set) a resident grid
// drains the eight XCD queues as k_class_persist does.  FP32 = 1: each task's
// kets from split[task] on are evaluated in FP32.
template <class E, int MODE, int FP32, bool MULTI>
__global__ __launch_bounds__(E::WGS) void k_class_rys(const ClassArgs a) {
    __shared__ int next_entry;
    unsigned cnt64 = 0, cnt32 = 0;
    if (!a.work) {
        class_task_rys<E, MODE, FP32, MULTI>(a, a.task_off + (int)blockIdx.x, cnt64, cnt32);
    } else {
        const int x0 = blockIdx.x & 7;
        for (int q = 0; q < 8;) {
            const int x = (x0 + q) & 7;
            if (threadIdx.x == 0) next_entry = (int)atomicAdd(a.work + x, 1ull);
            __syncthreads();   // also: the last task's LDS is free
            const int k = next_entry;
            __syncthreads();
            if (k >= a.qlen) {
                ++q;
                continue;
            }
            class_task_rys<E, MODE, FP32, MULTI>(a, 8 * k + x, cnt64, cnt32);
        }
    }
    flush_counts(a, cnt64, cnt32);
}

// Schwarz bounds Q = sqrt(max (mn|mn)) of a pair class, one workgroup per pair
// (a batch of one ket).
template <class E>
__global__ __launch_bounds__(E::WGS) void k_schwarz_rys(const PairInfo* __restrict__ pairs,
                                                    const PrimPair* __restrict__ prim,
                                                    const double* __restrict__ tab, double* __restrict__ Q) {
    using X = RysDims<E>;
    static_assert(X::NAB == X::NCD, "bra and ket of one pair class");
    __shared__ __align__(16) double G[X::NK * X::KET];
    __shared__ double best[X::WAVES];
    const PairInfo pr = pairs[blockIdx.x];
    RysLane ln = rys_lane<E>();
    const bool on = ln.on && ln.j == 0;
    const double* pp = (const double*)(prim + pr.prim_off);
    double v[X::NCD];
    RysSteps<E, double, double> steps(tab, pp, pr.nprim, pp, pr.nprim, HFX_PRIM_FIELDS, 1, 1, pr.AB[0], pr.AB[1],
                                      pr.AB[2], G, ln.j);
    steps.batch(0, ln, on, pairs[blockIdx.x].AB, v);
    double d = 0.0;
#pragma unroll
    for (int i = 0; i < X::NCD; ++i) d = i == ln.mn ? v[i] : d;
    const double s = comp_scale(E::LA, ln.m) * comp_scale(E::LB, ln.n);
    d = on ? d * s * s : 0.0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) d = fmax(d, __shfl_xor(d, off, 64));
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < X::WAVES; ++w) d = fmax(d, best[w]);
        Q[blockIdx.x] = sqrt(d);
    }
}

// Kernels of a class: variant = mode + 2 mixed + 4 multi; lds: bytes of LDS
// without the rows of W, and kets per batch.
#define HFX_CLASS_TU_RYS(cid, la_, lb_, lc_, ld_, wgs_, nk_, fp64_only_)                                       \
    struct Eval##cid {                                                                                    \
        static constexpr int LA = la_, LB = lb_, LC = lc_, LD = ld_, WGS = wgs_, NK = nk_;                \
    };                                                                                                    \
    extern "C" const void* hfx_class_kernel_##cid(int) { return nullptr; }                                \
    extern "C" const void* hfx_class_kernel_kr_##cid(int) { return nullptr; }                             \
    extern "C" const void* hfx_class_kernel_multi_##cid(int) { return nullptr; }                          \
    extern "C" const void* hfx_class_kernel_rys_##cid(int v) {                                            \
        if (v < 0 || v > 5) return nullptr;                                                               \
        if constexpr (fp64_only_) {                                                                       \
            if (v == 2 || v == 3) return nullptr;                                                         \
        } else {                                                                                          \
            if (v == 2) return (const void*)k_class_rys<Eval##cid, 0, 1, false>;                          \
            if (v == 3) return (const void*)k_class_rys<Eval##cid, 1, 1, false>;                          \
        }                                                                                                 \
        if (v >= 4)                                                                                       \
            return v == 4 ? (const void*)k_class_rys<Eval##cid, 0, 0, true>                               \
                          : (const void*)k_class_rys<Eval##cid, 1, 0, true>;                              \
        return v ? (const void*)k_class_rys<Eval##cid, 1, 0, false> : (const void*)k_class_rys<Eval##cid, 0, 0, false>; \
    }                                                                                                     \
    extern "C" int hfx_class_rys_lds_##cid(int mode, int ndens) {                                         \
        return 8 * RysDims<Eval##cid>::lds(mode, ndens);                                                  \
    }                                                                                                     \
    extern "C" int hfx_class_rys_kets_##cid(void) { return RysDims<Eval##cid>::NK; }

// The Schwarz kernel of a class with bra and ket of one pair class.
#define HFX_SCHWARZ_RYS(cid)                                                                              \
    extern "C" const void* hfx_schwarz_kernel_##cid(void) { return (const void*)k_schwarz_rys<Eval##cid>; }
#define HFX_NO_SCHWARZ(cid) \
    extern "C" const void* hfx_schwarz_kernel_##cid(void) { return nullptr; }
