// One-electron integrals S and H = T + V (Obara-Saika).  Overlap from the 1-D
// recursion
//   S_{i+1,j} = X_PA S_ij + (i S_{i-1,j} + j S_{i,j-1})/(2p), same for j with X_PB;
// kinetic from -1/2 d^2/dx^2 acting on the ket Gaussian:
//   T_ij = -1/2 [ j(j-1) S_{i,j-2} - 2 beta (2j+1) S_ij + 4 beta^2 S_{i,j+2} ];
// nuclear attraction from the vertical recursion on centre A,
//   [a+1_i]^(m) = PA_i [a]^(m) - PC_i [a]^(m+1) + a_i/(2p) ([a-1_i]^(m) - [a-1_i]^(m+1)),
//   [0]^(m) = 2 pi / p exp(-alpha beta/p |AB|^2) F_m(p |PC|^2),
// summed over primitives and nuclei, then the transfer
//   (a|b+1_i) = (a+1_i|b) + AB_i (a|b).
//
// One wave per shell pair.  The work is primitive pairs x nuclei Boys functions
// and recursions, independent of each other: lanes take (primitive pair,
// nucleus) items, their sums are added over the wave once, and the transfer
// runs on the sums.  The angular momenta are template parameters (shell A the
// higher one), so that every array of the recursions is in registers.  One
// thread per shell pair, looping over primitives and nuclei on arrays in
// scratch, took 8.4 ms for 29 waters (290 shells, 87 nuclei); the six launches 0.14 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "hfx_ctx.h"

namespace {

// Cartesian component c of order l in lexicographic order, and its index.
struct Cart {
    int e[3];
};
constexpr Cart cart_of(int l, int c) {
    int k = 0;
    for (int x = l; x >= 0; --x)
        for (int y = l - x; y >= 0; --y, ++k)
            if (k == c) return {{x, y, l - x - y}};
    return {{0, 0, 0}};
}
constexpr int cart_off(int l) { return l * (l + 1) * (l + 2) / 6; }   // components of lower orders
constexpr int cart_pos(const Cart& c) {
    const int yz = c.e[1] + c.e[2];
    return cart_off(c.e[0] + yz) + yz * (yz + 1) / 2 + c.e[2];
}

// Vertical recursion of one component (order >= 1): direction, the terms one
// and two below in it (two: -1 if absent) and the count in front of the latter.
struct Vrr {
    int dir, one, two, n;
};
struct VrrTable {
    Vrr v[35];
    constexpr VrrTable() : v{} {
        for (int l = 1; l <= 4; ++l)
            for (int c = 0; c < hfx_ncart(l); ++c) {
                Cart e = cart_of(l, c);
                Vrr r{e.e[0] > 0 ? 0 : (e.e[1] > 0 ? 1 : 2), 0, -1, 0};
                e.e[r.dir] -= 1;
                r.one = cart_pos(e);
                if (e.e[r.dir] > 0) {
                    r.n = e.e[r.dir];
                    e.e[r.dir] -= 1;
                    r.two = cart_pos(e);
                }
                v[cart_off(l) + c] = r;
            }
    }
};

struct PairPrim {   // one primitive pair in LDS
    double p, i2p, x, y, z, pre;   // exponent, 1/(2p), P - A, -2 pi / p c_a c_b exp(-mu AB^2)
};

// One class (LA >= LB) of one molecule: pairs of its nla shells of LA with its
// nlb of LB (LA = LB: i >= j), by the order's shell lists.
template <int LA, int LB>
__global__ __launch_bounds__(64) void k_one_electron(const OneElMol* __restrict__ mols, const int* __restrict__ order,
                                                     const ShellHost* __restrict__ sh, const double* __restrict__ exps,
                                                     const double* __restrict__ coefs,
                                                     const double* __restrict__ atoms /*x,y,z,Z*/,
                                                     const double* __restrict__ cscale, const double* __restrict__ boys,
                                                     double* __restrict__ S, double* __restrict__ H) {
    constexpr int NA = hfx_ncart(LA), NB = hfx_ncart(LB), L = LA + LB;
    constexpr int E0 = cart_off(LA), NE = cart_off(L + 1);   // transfer reads components [E0, NE)
    constexpr VrrTable VT{};
    __shared__ PairPrim pp[64];
    const OneElMol M = mols[blockIdx.y];
    const int lane = threadIdx.x;
    const int nla = M.n[LA], nlb = M.n[LB];
    const long long npair = LA == LB ? (long long)nla * (nla + 1) / 2 : (long long)nla * nlb;
    for (long long pid = blockIdx.x; pid < npair; pid += gridDim.x) {
        int i, j;
        if constexpr (LA == LB) {
            i = (int)((sqrt(8.0 * (double)pid + 1.0) - 1.0) * 0.5);
            while ((long long)i * (i + 1) / 2 > pid) --i;
            while ((long long)(i + 1) * (i + 2) / 2 <= pid) ++i;
            j = (int)(pid - (long long)i * (i + 1) / 2);
        } else {
            i = (int)(pid / nlb);
            j = (int)(pid % nlb);
        }
        const ShellHost A = sh[order[M.first[LA] + i]], B = sh[order[M.first[LB] + j]];
        const double AB[3] = {A.x - B.x, A.y - B.y, A.z - B.z};
        const double ab2 = AB[0] * AB[0] + AB[1] * AB[1] + AB[2] * AB[2];
        double s_acc[NA * NB], t_acc[NA * NB], v_acc[NE - E0];
#pragma unroll
        for (int k = 0; k < NA * NB; ++k) s_acc[k] = t_acc[k] = 0.0;
#pragma unroll
        for (int k = 0; k < NE - E0; ++k) v_acc[k] = 0.0;
        const int np = A.nprim * B.nprim;
        const int q1 = 64 / M.natom, r1 = 64 % M.natom;   // a lane's step in (primitive pair, nucleus)
        for (int base = 0; base < np; base += 64) {       // 64 primitive pairs at a time
            const int n = min(64, np - base);
            if (lane < n) {
                const int ia = (base + lane) / B.nprim, ib = (base + lane) % B.nprim;
                const double al = exps[A.prim_off + ia], be = exps[B.prim_off + ib];
                const double p = al + be, i2p = 0.5 / p, mu = al * be / p;
                // P - A and P - B from A - B: as differences of coordinates they lose the
                // digits that tight functions far from the origin need
                const double fa = -be / p, fb = al / p;
                const double k3 = coefs[A.prim_off + ia] * coefs[B.prim_off + ib] * exp(-mu * ab2);
                pp[lane] = PairPrim{p, i2p, fa * AB[0], fa * AB[1], fa * AB[2], -2.0 * M_PI / p * k3};
                // 1-D overlaps and kinetic integrals
                double S1[3][LA + 1][LB + 3], T1[3][LA + 1][LB + 1];
                const double s00 = sqrt(M_PI / p);
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    const double PA = fa * AB[x], PB = fb * AB[x];
#pragma unroll
                    for (int a = 0; a <= LA; ++a) {
                        S1[x][a][0] = a == 0 ? s00
                                             : PA * S1[x][a > 0 ? a - 1 : 0][0] +
                                                   (a > 1 ? (a - 1) * i2p * S1[x][a > 1 ? a - 2 : 0][0] : 0.0);
#pragma unroll
                        for (int b = 1; b <= LB + 2; ++b)
                            S1[x][a][b] = PB * S1[x][a][b - 1] +
                                          i2p * ((a > 0 ? a * S1[x][a > 0 ? a - 1 : 0][b - 1] : 0.0) +
                                                 (b > 1 ? (b - 1) * S1[x][a][b > 1 ? b - 2 : 0] : 0.0));
#pragma unroll
                        for (int b = 0; b <= LB; ++b)
                            T1[x][a][b] = -0.5 * ((b >= 2 ? b * (b - 1) * S1[x][a][b >= 2 ? b - 2 : 0] : 0.0) -
                                                  2.0 * be * (2 * b + 1) * S1[x][a][b] +
                                                  4.0 * be * be * S1[x][a][b + 2]);
                    }
                }
#pragma unroll
                for (int m = 0; m < NA; ++m)
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        const Cart ea = cart_of(LA, m), eb = cart_of(LB, k);
                        const double sx = S1[0][ea.e[0]][eb.e[0]], sy = S1[1][ea.e[1]][eb.e[1]],
                                     sz = S1[2][ea.e[2]][eb.e[2]];
                        const double tx = T1[0][ea.e[0]][eb.e[0]], ty = T1[1][ea.e[1]][eb.e[1]],
                                     tz = T1[2][ea.e[2]][eb.e[2]];
                        s_acc[m * NB + k] += k3 * (sx * sy * sz);
                        t_acc[m * NB + k] += k3 * (tx * sy * sz + sx * ty * sz + sx * sy * tz);
                    }
            }
            __syncthreads();   // the workgroup is one wave
            int q = lane / M.natom, r = lane % M.natom;
            while (q < n) {
                const PairPrim pr = pp[q];
                const double* at = atoms + 4 * (size_t)(M.aoff + r);
                const double PA[3] = {pr.x, pr.y, pr.z};
                const double PC[3] = {PA[0] + (A.x - at[0]), PA[1] + (A.y - at[1]), PA[2] + (A.z - at[2])};
                // a centre without charge adds zero, wherever it lies
                const double T = at[3] != 0.0 ? pr.p * (PC[0] * PC[0] + PC[1] * PC[1] + PC[2] * PC[2]) : 0.0;
                double F[L + 1];
                if constexpr (L == 0) F[0] = boys_zero(1.0, T, boys + boys_block(0));
                else boys_eval<double, L>(T, F, boys + boys_block(L));
                double th[NE][L + 1];
                const double pre = pr.pre * at[3];
#pragma unroll
                for (int m = 0; m <= L; ++m) th[0][m] = pre * F[m];
#pragma unroll
                for (int l = 1; l <= L; ++l)
#pragma unroll
                    for (int c = 0; c < hfx_ncart(l); ++c) {
                        const Vrr v = VT.v[cart_off(l) + c];
#pragma unroll
                        for (int m = 0; m <= L - l; ++m) {
                            double t = PA[v.dir] * th[v.one][m] - PC[v.dir] * th[v.one][m + 1];
                            if (v.two >= 0) t += v.n * pr.i2p * (th[v.two][m] - th[v.two][m + 1]);
                            th[cart_off(l) + c][m] = t;
                        }
                    }
#pragma unroll
                for (int k = E0; k < NE; ++k) v_acc[k - E0] += th[k][0];
                q += q1;
                r += r1;
                if (r >= M.natom) {
                    r -= M.natom;
                    ++q;
                }
            }
            __syncthreads();
        }
        // sums over the wave; lane m NB + k keeps element (m, k)
#pragma unroll
        for (int k = 0; k < NE - E0; ++k) v_acc[k] = wave_sum(v_acc[k]);
        double so = 0.0, ho = 0.0;
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                // (x - B)^j = sum_k C(j, k) (x - A)^(j - k) (A - B)^k on each axis
                const Cart ea = cart_of(LA, m), eb = cart_of(LB, k);
                double v = 0.0;
#pragma unroll
                for (int kx = 0; kx <= eb.e[0]; ++kx)
#pragma unroll
                    for (int ky = 0; ky <= eb.e[1]; ++ky)
#pragma unroll
                        for (int kz = 0; kz <= eb.e[2]; ++kz) {
                            const Cart e{{ea.e[0] + eb.e[0] - kx, ea.e[1] + eb.e[1] - ky, ea.e[2] + eb.e[2] - kz}};
                            double f = v_acc[cart_pos(e) - E0];
                            if (kx == 1) f *= eb.e[0] * AB[0];
                            if (kx == 2) f *= AB[0] * AB[0];
                            if (ky == 1) f *= eb.e[1] * AB[1];
                            if (ky == 2) f *= AB[1] * AB[1];
                            if (kz == 1) f *= eb.e[2] * AB[2];
                            if (kz == 2) f *= AB[2] * AB[2];
                            v += f;
                        }
                const double s = wave_sum(s_acc[m * NB + k]), t = wave_sum(t_acc[m * NB + k]);
                if (lane == m * NB + k) {
                    so = s;
                    ho = t + v;
                }
            }
        // a shell with itself: one of the two lanes of an element, so that the matrices are symmetric
        if (lane < NA * NB && (LA != LB || i != j || lane / NB >= lane % NB)) {
            const int r = A.bf + lane / NB, c = B.bf + lane % NB;
            const double sc = cscale[M.boff + r] * cscale[M.boff + c];
            const size_t rc = M.moff + (size_t)r * M.nbf + c, cr = M.moff + (size_t)c * M.nbf + r;
            S[rc] = S[cr] = sc * so;
            H[rc] = H[cr] = sc * ho;
        }
    }
}

template <int LA, int LB>
hipError_t launch(int nmol, long long npair, const OneElMol* mols, const int* order, const ShellHost* sh,
                  const double* exps, const double* coefs, const double* atoms, const double* cscale,
                  const double* boys, double* S, double* H, hipStream_t st) {
    // below 2^32 lanes: workgroups stride over the pairs, molecules go in groups
    const unsigned gx = (unsigned)std::min(npair, 1ll << 16);
    for (int m0 = 0; m0 < nmol && npair > 0; m0 += 512)
        hipLaunchKernelGGL((k_one_electron<LA, LB>), dim3(gx, std::min(nmol - m0, 512)), dim3(64), 0, st, mols + m0,
                           order, sh, exps, coefs, atoms, cscale, boys, S, H);
    return hipGetLastError();
}

}  // namespace

hipError_t hfx_one_electron(int nmol, const OneElMol* hmols, const OneElMol* mols, const int* order,
                            const ShellHost* sh, const double* exps, const double* coefs, const double* atoms,
                            const double* cscale, const double* boys, double* S, double* H, hipStream_t st) {
    hipError_t e = hipSuccess;
    auto run = [&](auto fn, int la, int lb) {
        long long most = 0;   // pairs of the molecule with the most
        for (int m = 0; m < nmol; ++m) {
            const long long a = hmols[m].n[la], b = hmols[m].n[lb];
            most = std::max(most, la == lb ? a * (a + 1) / 2 : a * b);
        }
        if (e == hipSuccess)
            e = fn(nmol, most, mols, order, sh, exps, coefs, atoms, cscale, boys, S, H, st);
    };
    run(launch<0, 0>, 0, 0);
    run(launch<1, 0>, 1, 0);
    run(launch<1, 1>, 1, 1);
    run(launch<2, 0>, 2, 0);
    run(launch<2, 1>, 2, 1);
    run(launch<2, 2>, 2, 2);
    return e;
}
