// Learned initial guess: pair descriptors and frames, the network's BF16
// MFMA forward and backward passes with FP32 accumulation, Adam, and the
// rotation of density blocks between pair frames and the molecule.
//
// The SCF of section 3 needs a starting density; the library's default is a
// superposition of atomic densities (SAD).  This extension predicts, for each
// atom pair within 6 A, the converged-minus-SAD density block in a local frame
// of the pair, from a 164-number descriptor of the pair's surroundings:
//   [one-hot element of A, of B, 32 radial Gaussians of R_AB with a cosine
//    cutoff, A's environment (log(1 + the radial functions summed over
//    neighbours), one 32-block per element), B's environment].
// Network: 164 -> 256 -> 256 -> 256 (SiLU) -> one linear head per pair type
// (O-O 225, O-H 30, H-H 4 outputs = the 15 x 15, 15 x 2, 2 x 2 blocks).
// Layers run on the matrix units (v_mfma_f32_16x16x32_bf16): BF16 operands, FP32
// accumulation; a workgroup takes 32 rows through the whole network, with
// pre-activations and gradients in FP32 registers, Adam updates FP32 master
// weights.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "hfx_ctx.h"

namespace {

constexpr int NFEAT = 164, NRAD = 32, HID = 256, XLD = 192;   // XLD: padded feature row (bf16)
constexpr int NTYPE = 3;
constexpr int HEAD_OUT[NTYPE] = {225, 30, 4};
constexpr int MAXB = 16;                 // basis functions per atom handled by the block kernels
constexpr double BOHR_PER_A = 1.0 / 0.529177210903;
constexpr double RCUT_A = 6.0;
constexpr double TIE_BOHR = 1e-6;
constexpr double NONCOLLINEAR_SIN = 0.1;
constexpr float INPUT_CLIP = 4.0f;       // standardised inputs are clipped to +-INPUT_CLIP

typedef unsigned short bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---- parameter layout (FP32, packed): W1 b1 W2 b2 W3 b3, per head W c,
//      feature mean, feature scale, three target scales -----------------------------------

struct ParamLayout {
    long long off[15], size[15], total;
    ParamLayout() {
        const long long s[15] = {(long long)HID * NFEAT, HID, (long long)HID * HID, HID, (long long)HID * HID, HID,
                                 (long long)HEAD_OUT[0] * HID, HEAD_OUT[0], (long long)HEAD_OUT[1] * HID, HEAD_OUT[1],
                                 (long long)HEAD_OUT[2] * HID, HEAD_OUT[2], NFEAT, NFEAT, NTYPE};
        long long o = 0;
        for (int i = 0; i < 15; ++i) {
            off[i] = o;
            size[i] = s[i];
            o += s[i];
        }
        total = o;
    }
};
const ParamLayout PL;
enum { P_W1, P_B1, P_W2, P_B2, P_W3, P_B3, P_H0, P_C0, P_H1, P_C1, P_H2, P_C2, P_FMEAN, P_FSCALE, P_TSCALE };
constexpr int NTRAIN = 12;

// ---- small helpers -------------------------------------------------------------------

__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }   // nearest even
__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu_f(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

constexpr int WG = 256;
inline unsigned blocks_for(long long n) { return (unsigned)std::max<long long>(1, (n + WG - 1) / WG); }

// ---- descriptors and frames ------------------------------------------------------------

__device__ void radial(double r_a, double* g) {
    const double dmu = 5.5 / (NRAD - 1), eta = 1.0 / (2.0 * dmu * dmu);
    const double fc = r_a < RCUT_A ? 0.5 * (cos(M_PI * r_a / RCUT_A) + 1.0) : 0.0;
    for (int k = 0; k < NRAD; ++k) {
        const double mu = 0.5 + dmu * k, d = r_a - mu;
        g[k] = exp(-eta * d * d) * fc;
    }
}

__device__ __forceinline__ double dist(const double* xyz, int a, int b) {
    const double dx = xyz[3 * b] - xyz[3 * a], dy = xyz[3 * b + 1] - xyz[3 * a + 1], dz = xyz[3 * b + 2] - xyz[3 * a + 2];
    return sqrt(dx * dx + dy * dy + dz * dz);
}

// env[a][e*32 + k] = log(1 + sum over atoms c != a of element e of G_k(R_ac));
// one thread per (atom, e, k)
__global__ void k_env(int natom, const double* __restrict__ xyz, const int* __restrict__ elem, double* __restrict__ env) {
    const long long i = (long long)blockIdx.x * WG + threadIdx.x;
    if (i >= (long long)natom * 2 * NRAD) return;
    const int a = (int)(i / (2 * NRAD)), q = (int)(i % (2 * NRAD)), e = q / NRAD, k = q % NRAD;
    const double dmu = 5.5 / (NRAD - 1), eta = 1.0 / (2.0 * dmu * dmu), mu = 0.5 + dmu * k;
    double acc = 0.0;
    for (int c = 0; c < natom; ++c) {
        if (c == a || elem[c] != e) continue;
        const double r = dist(xyz, a, c) / BOHR_PER_A;
        if (r >= RCUT_A) continue;
        const double d = r - mu;
        acc += exp(-eta * d * d) * 0.5 * (cos(M_PI * r / RCUT_A) + 1.0);
    }
    env[i] = log1p(acc);
}

// ordering key of candidate atoms: distance in bins of TIE_BOHR, then index
__device__ __forceinline__ bool key_less(double da, int a, double db, int b) {
    const double fa = floor(da / TIE_BOHR), fb = floor(db / TIE_BOHR);
    return fa < fb || (fa == fb && a < b);
}

// One thread per pair: 164 features and the frame (rows x, y, z).
__global__ void k_pair_setup(int natom, const double* __restrict__ xyz, const int* __restrict__ elem,
                             const double* __restrict__ env, int npair, const int4* __restrict__ pairs,
                             float* __restrict__ feat, double* __restrict__ frames) {
    const int p = blockIdx.x * WG + threadIdx.x;
    if (p >= npair) return;
    const int a = pairs[p].x;
    int b = pairs[p].y;
    float* f = feat + (size_t)p * NFEAT;
    for (int k = 0; k < NFEAT; ++k) f[k] = 0.0f;
    f[elem[a]] = 1.0f;
    f[2 + elem[b]] = 1.0f;
    double g[NRAD];
    radial(dist(xyz, a, b) / BOHR_PER_A, g);
    for (int k = 0; k < NRAD; ++k) f[4 + k] = (float)g[k];
    for (int k = 0; k < 2 * NRAD; ++k) {
        f[4 + NRAD + k] = (float)env[(size_t)a * 2 * NRAD + k];
        f[4 + 3 * NRAD + k] = (float)env[(size_t)b * 2 * NRAD + k];
    }
    // frame
    double* R = frames + (size_t)p * 9;
    if (a == b) {   // self block: z toward the nearest atom
        int best = -1;
        double bd = 0.0;
        for (int c = 0; c < natom; ++c) {
            if (c == a) continue;
            const double d = dist(xyz, a, c);
            if (best < 0 || key_less(d, c, bd, best)) { best = c; bd = d; }
        }
        if (best < 0) {
            for (int i = 0; i < 9; ++i) R[i] = (i % 4 == 0) ? 1.0 : 0.0;
            return;
        }
        b = best;
    }
    double z[3] = {xyz[3 * b] - xyz[3 * a], xyz[3 * b + 1] - xyz[3 * a + 1], xyz[3 * b + 2] - xyz[3 * a + 2]};
    double n = sqrt(z[0] * z[0] + z[1] * z[1] + z[2] * z[2]);
    for (int i = 0; i < 3; ++i) z[i] /= n;
    int best = -1;
    double bd = 0.0;
    for (int c = 0; c < natom; ++c) {
        if (c == a || c == b) continue;
        const double v[3] = {xyz[3 * c] - xyz[3 * a], xyz[3 * c + 1] - xyz[3 * a + 1], xyz[3 * c + 2] - xyz[3 * a + 2]};
        const double d = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
        const double cx = (v[1] * z[2] - v[2] * z[1]) / d, cy = (v[2] * z[0] - v[0] * z[2]) / d,
                     cz = (v[0] * z[1] - v[1] * z[0]) / d;
        if (sqrt(cx * cx + cy * cy + cz * cz) <= NONCOLLINEAR_SIN) continue;
        if (best < 0 || key_less(d, c, bd, best)) { best = c; bd = d; }
    }
    double x[3];
    if (best >= 0) {
        const double v[3] = {xyz[3 * best] - xyz[3 * a], xyz[3 * best + 1] - xyz[3 * a + 1],
                             xyz[3 * best + 2] - xyz[3 * a + 2]};
        const double vz = v[0] * z[0] + v[1] * z[1] + v[2] * z[2];
        for (int i = 0; i < 3; ++i) x[i] = v[i] - vz * z[i];
    } else {   // global axis least aligned with z
        int k = 0;
        for (int i = 1; i < 3; ++i)
            if (fabs(z[i]) < fabs(z[k])) k = i;
        for (int i = 0; i < 3; ++i) x[i] = (i == k ? 1.0 : 0.0) - z[k] * z[i];
    }
    n = sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
    for (int i = 0; i < 3; ++i) x[i] /= n;
    const double y[3] = {z[1] * x[2] - z[2] * x[1], z[2] * x[0] - z[0] * x[2], z[0] * x[1] - z[1] * x[0]};
    for (int i = 0; i < 3; ++i) {
        R[i] = x[i];
        R[3 + i] = y[i];
        R[6 + i] = z[i];
    }
}

// ---- block rotation --------------------------------------------------------------------

struct AtomBasis {
    const int* first;   // first basis function of the atom (molecule-local)
    const int* nb;      // functions on the atom
    const int* shoff;   // shell list offset
    const int* nsh;     // shells on the atom
    const int* shl;     // shell angular momenta
};

// T (n x n, row-major, LDS) with phi(R r) = T phi(r) for the atom's shells:
// s -> 1, p -> R, unit-normalised Cartesian d -> N M(R) N^-1.
__device__ void build_T(const AtomBasis& ab, int atom, const double* R, bool transpose_R, double* T, int n) {
    for (int i = threadIdx.x; i < n * n; i += blockDim.x) T[i] = 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
        double Q[9];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) Q[3 * i + j] = transpose_R ? R[3 * j + i] : R[3 * i + j];
        const int dc[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
        const double s3 = 0.57735026918962576451;
        const double dn[6] = {s3, 1.0, 1.0, s3, 1.0, s3};
        int o = 0;
        for (int s = 0; s < ab.nsh[atom]; ++s) {
            const int l = ab.shl[ab.shoff[atom] + s];
            if (l == 0) {
                T[o * n + o] = 1.0;
                o += 1;
            } else if (l == 1) {
                for (int i = 0; i < 3; ++i)
                    for (int j = 0; j < 3; ++j) T[(o + i) * n + o + j] = Q[3 * i + j];
                o += 3;
            } else {
                for (int p = 0; p < 6; ++p)
                    for (int q = 0; q < 6; ++q) {
                        const int a = dc[p][0], b = dc[p][1], i = dc[q][0], j = dc[q][1];
                        double m = Q[3 * a + i] * Q[3 * b + j];
                        if (i != j) m += Q[3 * a + j] * Q[3 * b + i];
                        T[(o + p) * n + o + q] = dn[p] * m / dn[q];
                    }
                o += 6;
            }
        }
    }
    __syncthreads();
}

// P = TA^T X TB for one pair (n_a x n_b), all in LDS; tmp n_a x n_b.
__device__ void sandwich(const double* TA, int na, const double* X, const double* TB, int nb, double* tmp, double* P) {
    for (int i = threadIdx.x; i < na * nb; i += blockDim.x) {
        const int r = i / nb, c = i % nb;
        double s = 0.0;
        for (int k = 0; k < nb; ++k) s += X[r * nb + k] * TB[k * nb + c];
        tmp[i] = s;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < na * nb; i += blockDim.x) {
        const int r = i / nb, c = i % nb;
        double s = 0.0;
        for (int k = 0; k < na; ++k) s += TA[k * na + r] * tmp[k * nb + c];
        P[i] = s;
    }
    __syncthreads();
}

// Local blocks of (D - Dbase): P = T_A(R^T)^T (D - Dbase)_AB T_B(R^T), packed FP32.
__global__ __launch_bounds__(64) void k_to_local(int npair, const int4* __restrict__ pairs,
                                                 const double* __restrict__ frames, AtomBasis ab,
                                                 const long long* __restrict__ out_off, const double* __restrict__ D,
                                                 const double* __restrict__ Db, int n, float* __restrict__ out) {
    __shared__ double TA[MAXB * MAXB], TB[MAXB * MAXB], X[MAXB * MAXB], tmp[MAXB * MAXB], P[MAXB * MAXB];
    const int p = blockIdx.x;
    const int a = pairs[p].x, b = pairs[p].y;
    const int na = ab.nb[a], nb = ab.nb[b];
    const double* R = frames + (size_t)p * 9;
    build_T(ab, a, R, true, TA, na);
    build_T(ab, b, R, true, TB, nb);
    const int fa = ab.first[a], fb = ab.first[b];
    for (int i = threadIdx.x; i < na * nb; i += blockDim.x) {
        const size_t g = (size_t)(fa + i / nb) * n + fb + i % nb;
        X[i] = D[g] - (Db ? Db[g] : 0.0);
    }
    __syncthreads();
    sandwich(TA, na, X, TB, nb, tmp, P);
    for (int i = threadIdx.x; i < na * nb; i += blockDim.x) out[out_off[p] + i] = (float)P[i];
}

// D = Dbase + sum over pairs of T_A(R)^T P T_B(R) at (A, B) and its transpose
// at (B, A) (a self block symmetrised).  Each block belongs to one pair.
__global__ __launch_bounds__(64) void k_assemble_blocks(int npair, const int4* __restrict__ pairs,
                                                        const double* __restrict__ frames, AtomBasis ab,
                                                        const long long* __restrict__ in_off,
                                                        const float* __restrict__ blocks, int n,
                                                        double* __restrict__ D) {
    __shared__ double TA[MAXB * MAXB], TB[MAXB * MAXB], X[MAXB * MAXB], tmp[MAXB * MAXB], P[MAXB * MAXB];
    const int p = blockIdx.x;
    const int a = pairs[p].x, b = pairs[p].y;
    const int na = ab.nb[a], nb = ab.nb[b];
    const double* R = frames + (size_t)p * 9;
    build_T(ab, a, R, false, TA, na);
    build_T(ab, b, R, false, TB, nb);
    const float* in = blocks + in_off[p];
    for (int i = threadIdx.x; i < na * nb; i += blockDim.x) {
        const int r = i / nb, c = i % nb;
        X[i] = a == b ? 0.5 * ((double)in[r * nb + c] + (double)in[c * nb + r]) : (double)in[i];
    }
    __syncthreads();
    sandwich(TA, na, X, TB, nb, tmp, P);
    const int fa = ab.first[a], fb = ab.first[b];
    for (int i = threadIdx.x; i < na * nb; i += blockDim.x) {
        const int r = i / nb, c = i % nb;
        D[(size_t)(fa + r) * n + fb + c] += P[i];
        if (a != b) D[(size_t)(fb + c) * n + fa + r] += P[i];
    }
}

__global__ void k_copy(const double* __restrict__ s, size_t n, double* __restrict__ d) {
    for (size_t i = (size_t)blockIdx.x * WG + threadIdx.x; i < n; i += (size_t)gridDim.x * WG) d[i] = s[i];
}

// out[0] += sum D_ij S_ij, out[1] += number of non-finite D_ij
__global__ void k_trace_check(const double* __restrict__ D, const double* __restrict__ S, size_t n, double* out) {
    double acc = 0.0, bad = 0.0;
    for (size_t i = (size_t)blockIdx.x * WG + threadIdx.x; i < n; i += (size_t)gridDim.x * WG) {
        const double d = D[i];
        if (isfinite(d)) acc += d * S[i]; else bad += 1.0;
    }
    for (int off = 32; off >= 1; off >>= 1) {
        acc += __shfl_xor(acc, off, 64);
        bad += __shfl_xor(bad, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(out, acc);
        atomicAdd(out + 1, bad);
    }
}

// ---- the network -----------------------------------------------------------------------

// Rows are walked in blocks of 32 consecutive pairs of one type (the last block
// of a type is padded).  An operand of v_mfma_f32_16x16x32_bf16 is 16 x 32: lane
// l holds row l & 15, k = 8 (l >> 4) .. + 7, so a "fragment" of 512 BF16 in lane
// order is one contiguous 16-byte load per lane.  Everything a kernel reads from
// memory lies in fragments: the weights W[n][k] as [n / 16][k / 32] (and their
// transposes for the backward pass), and the activations and gradients, for the
// weight gradients whose contracted index is the row, as [row block][column / 16].
constexpr int RB = 32, FRAG = 512;        // rows of a block, BF16 of a fragment
constexpr int NET_WG = 512;               // eight waves, 32 output columns each
constexpr int ALD = HID + 8;              // LDS row of activations
constexpr int FB = HID / 16, XFB = XLD / 16, YFB = 16;   // fragments of a row block: hidden, input, head output
constexpr int NCB = 3 * HID + HEAD_OUT[0] + HEAD_OUT[1] + HEAD_OUT[2];   // biases
__host__ __device__ constexpr int head_kpad(int t) { return t == 0 ? 256 : 32; }   // head outputs, padded

// offsets (BF16) of the packed weights: forward layers, heads, and transposes
constexpr int PW1 = 0, PW2 = PW1 + HID * XLD, PW3 = PW2 + HID * HID, PW2T = PW3 + HID * HID, PW3T = PW2T + HID * HID;
constexpr int PH0 = PW3T + HID * HID, PH1 = PH0 + 256 * HID, PH2 = PH1 + 32 * HID;   // heads
constexpr int PH0T = PH2 + 32 * HID, PH1T = PH0T + HID * 256, PH2T = PH1T + HID * 32, PWTOT = PH2T + HID * 32;

struct NetParams {   // packed FP32 parameters and their offsets
    const float* p;
    long long w1, b1, w2, b2, w3, b3, h[NTYPE], c[NTYPE], fmean, fscale;
};

// element i of a fragment-ordered matrix with ks fragments along k: its (n, k)
__device__ __forceinline__ void frag_nk(int i, int ks, int& n, int& k) {
    const int f = i / FRAG, e = i % FRAG, l = e >> 3;
    n = (f / ks) * 16 + (l & 15);
    k = (f % ks) * 32 + (l >> 4) * 8 + (e & 7);
}

// All weights as BF16 fragments, zero in the padding.
__global__ void k_pack(const NetParams w, bf16_t* __restrict__ out) {
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i >= PWTOT) return;
    int n, k;
    float v = 0.0f;
    if (i < PW2) {
        frag_nk(i - PW1, XLD / 32, n, k);
        if (k < NFEAT) v = w.p[w.w1 + n * NFEAT + k];
    } else if (i < PH0) {
        const int q = (i - PW2) / (HID * HID);   // W2, W3, W2^T, W3^T
        frag_nk((i - PW2) % (HID * HID), HID / 32, n, k);
        v = w.p[((q & 1) ? w.w3 : w.w2) + (q < 2 ? n * HID + k : k * HID + n)];
    } else if (i < PH0T) {
        const int t = i < PH1 ? 0 : i < PH2 ? 1 : 2;
        frag_nk(i - (t == 0 ? PH0 : t == 1 ? PH1 : PH2), HID / 32, n, k);
        if (n < (t == 0 ? HEAD_OUT[0] : t == 1 ? HEAD_OUT[1] : HEAD_OUT[2])) v = w.p[w.h[t] + n * HID + k];
    } else {
        const int t = i < PH1T ? 0 : i < PH2T ? 1 : 2;
        frag_nk(i - (t == 0 ? PH0T : t == 1 ? PH1T : PH2T), head_kpad(t) / 32, n, k);
        if (k < (t == 0 ? HEAD_OUT[0] : t == 1 ? HEAD_OUT[1] : HEAD_OUT[2])) v = w.p[w.h[t] + k * HID + n];
    }
    out[i] = f2bf(v);
}

struct NetArgs {
    NetParams w;
    const bf16_t* pk;              // packed weights
    const float* X;                // rows of NFEAT, by type
    const float* T;                // gradient: targets, packed by type
    float* out;                    // forward: predictions, packed by type
    int count[NTYPE], blk0[NTYPE + 1];   // rows; first row block (blk0[NTYPE]: all)
    long long row0[NTYPE], yoff[NTYPE];
    float tscale[NTYPE], inv_tscale[NTYPE], gs;
    // gradient: fragments of the inputs, H1 H2 H3, dZ1 dZ2 dZ3 and dY, and per
    // row block the column sums of dZ1 dZ2 dZ3 and dY and the squared error
    bf16_t *fx, *fh[3], *fg[3], *fy;
    float* csum;
    double* esum;
};

typedef f32x4 Acc[2][2];   // a wave's 32 rows x 32 columns

// acc = A B: A from LDS (32 rows), B the wave's two column blocks of fragments,
// four steps of k ahead (the first four loaded before the barrier that completes A).
template <int KS>
struct WaveB {
    static constexpr int AHEAD = KS < 4 ? KS : 4;
    const uint4* f;
    uint4 w[2][AHEAD];
    __device__ __forceinline__ void load(const bf16_t* __restrict__ frags, int jb0) {
        f = reinterpret_cast<const uint4*>(frags + (size_t)jb0 * KS * FRAG) + (threadIdx.x & 63);
#pragma unroll
        for (int ks = 0; ks < AHEAD; ++ks)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) w[bj][ks] = f[(bj * KS + ks) * (FRAG / 8)];
    }
    __device__ __forceinline__ void mul(const bf16_t* A, Acc& acc) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int bi = 0; bi < 2; ++bi) {
                const uint4 ua =
                    *reinterpret_cast<const uint4*>(A + (bi * 16 + (lane & 15)) * ALD + ks * 32 + (lane >> 4) * 8);
#pragma unroll
                for (int bj = 0; bj < 2; ++bj)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ua),
                                                                         __builtin_bit_cast(bf16x8, w[bj][ks % AHEAD]),
                                                                         acc[bi][bj], 0, 0, 0);
            }
            if (ks + AHEAD < KS)
#pragma unroll
                for (int bj = 0; bj < 2; ++bj) w[bj][ks % AHEAD] = f[(bj * KS + ks + AHEAD) * (FRAG / 8)];
        }
    }
};

// A wave's 32 x 32 block as BF16: rows into LDS for the next product, and (fr)
// the transposed fragments, where a lane's four rows are eight bytes; padded
// rows are zero in the fragments.
template <bool ROWS, bool FRAGS>
__device__ __forceinline__ void put_block(const Acc& v, int col0, int nr, bf16_t* rows, bf16_t* __restrict__ fr) {
    const int lane = threadIdx.x & 63, q = lane >> 4;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            bf16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = bi * 16 + q * 4 + r;
                h[r] = f2bf(v[bi][bj][r]);
                if (ROWS) rows[row * ALD + col0 + bj * 16 + (lane & 15)] = h[r];
                if (row >= nr) h[r] = 0;
            }
            if (FRAGS)
                *reinterpret_cast<uint2*>(fr + (size_t)(col0 / 16 + bj) * FRAG +
                                          ((bi * 2 + (q >> 1)) * 16 + (lane & 15)) * 8 + (q & 1) * 4) =
                    make_uint2(h[0] | (unsigned)h[1] << 16, h[2] | (unsigned)h[3] << 16);
        }
}

// Column sums of a wave's block over its valid rows.
__device__ __forceinline__ void put_sums(const Acc& v, int nr, float* __restrict__ out, int ncol) {
    const int lane = threadIdx.x & 63, q = lane >> 4;
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
        float s = 0.0f;
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (bi * 16 + q * 4 + r < nr) s += v[bi][bj][r];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (q == 0 && bj * 16 + lane < ncol) out[bj * 16 + lane] = s;
    }
}

// The network on one block of 32 rows: GRAD = 0 the predictions, GRAD = 1 the
// squared error and everything of the gradient that belongs to rows (dY, dZ3,
// dZ2, dZ1), with the fragments and sums that the weight gradients need.
// Activations stay in LDS and pre-activations in registers (FP32), so that
// memory holds what the weight gradients read and nothing else.  32 rows: 8192
// rows are 256 workgroups, one per CU, and every weight fragment (0.9 MB over
// both directions, from L2) serves two row blocks of the matrix unit.  A layer's
// first weights are loaded before the barrier that ends the last one.  Products
// run over k in ascending order with FP32 accumulation.  What bounds it is the
// vector unit (exponentials and divisions of SiLU and its derivative) in two
// waves per SIMD; with 128 registers two workgroups share a CU: 8192 rows 47 us
// against 55 us without spills (258 workgroups, two rounds), 500 rows 29 us
// against 26.  The chain of separate launches (products of 64 x 64 tiles that
// gathered two bytes a lane, elementwise and column-sum kernels between) took
// 5.4 ms for the whole gradient at 8192 rows, 2 x 1.3 ms of it in a pair of
// weight gradients; this kernel, k_wgrad and k_grad_sum take 47 + 15 + 8 us.
template <bool GRAD>
__global__ __launch_bounds__(NET_WG, 4) void k_net(const NetArgs a) {
    __shared__ __align__(16) bf16_t buf[2][RB * ALD];
    __shared__ double red[NET_WG / 64];
    const int blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = lane >> 4;
    const int t = blk < a.blk0[1] ? 0 : blk < a.blk0[2] ? 1 : 2;   // uniform
    const int lr0 = (blk - a.blk0[t]) * RB, nr = min(RB, a.count[t] - lr0);
    const int nout = t == 0 ? HEAD_OUT[0] : t == 1 ? HEAD_OUT[1] : HEAD_OUT[2];
    const int col0 = wv * 32, j0 = col0 + (lane & 15);
    const float* p = a.w.p;
    Acc z[3], v;
    {
        WaveB<XLD / 32> w;
        w.load(a.pk + PW1, wv * 2);
        // standardised, clipped inputs
        const float* X = a.X + (a.row0[t] + lr0) * NFEAT;
#pragma unroll
        for (int i0 = 0; i0 < RB * XLD; i0 += NET_WG) {
            const int i = i0 + tid, r = i / XLD, c = i % XLD;
            buf[0][r * ALD + c] =
                r < nr && c < NFEAT
                    ? f2bf(fminf(fmaxf((X[r * NFEAT + c] - p[a.w.fmean + c]) / p[a.w.fscale + c], -INPUT_CLIP),
                                 INPUT_CLIP))
                    : (bf16_t)0;
        }
        __syncthreads();
        if constexpr (GRAD)
            for (int i = tid; i < XFB * 64; i += NET_WG) {
                const int l = i & 63, c = (i >> 6) * 16 + (l & 15);
                bf16_t h[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) h[e] = buf[0][((l >> 4) * 8 + e) * ALD + c];
                reinterpret_cast<uint4*>(a.fx + (size_t)blk * XFB * FRAG)[i] =
                    make_uint4(h[0] | (unsigned)h[1] << 16, h[2] | (unsigned)h[3] << 16, h[4] | (unsigned)h[5] << 16,
                               h[6] | (unsigned)h[7] << 16);
            }
        w.mul(buf[0], z[0]);
    }
    // z += bias, v = silu(z)
    auto activate = [&](Acc& zz, long long bias) {
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            const float b = p[bias + j0 + bj * 16];
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    zz[bi][bj][r] += b;
                    v[bi][bj][r] = silu_f(zz[bi][bj][r]);
                }
        }
    };
    const size_t fo = (size_t)blk * FB * FRAG;
    activate(z[0], a.w.b1);
    put_block<true, GRAD>(v, col0, nr, buf[1], a.fh[0] + fo);
    {
        WaveB<HID / 32> w;
        w.load(a.pk + PW2, wv * 2);
        __syncthreads();
        w.mul(buf[1], z[1]);
    }
    activate(z[1], a.w.b2);
    put_block<true, GRAD>(v, col0, nr, buf[0], a.fh[1] + fo);
    {
        WaveB<HID / 32> w;
        w.load(a.pk + PW3, wv * 2);
        __syncthreads();
        w.mul(buf[0], z[2]);
    }
    activate(z[2], a.w.b3);
    put_block<true, GRAD>(v, col0, nr, buf[1], a.fh[2] + fo);
    // the type's head (waves past its columns idle)
    double e = 0.0;
    const bool head = col0 < head_kpad(t);
    {
        WaveB<HID / 32> w;
        if (head) w.load(a.pk + (t == 0 ? PH0 : t == 1 ? PH1 : PH2), wv * 2);
        __syncthreads();
        if (head) {
            w.mul(buf[1], v);
            const long long y0 = a.yoff[t] + (long long)lr0 * nout;
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) {
                const int j = j0 + bj * 16;
                const float b = j < nout ? p[a.w.c[t] + j] : 0.0f;
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = bi * 16 + q * 4 + r;
                        const bool on = j < nout && row < nr;
                        const float y = v[bi][bj][r] + b;
                        if constexpr (GRAD) {   // d = Y - T / tscale; dY = gs d
                            const float d = on ? y - a.T[y0 + (long long)row * nout + j] * a.inv_tscale[t] : 0.0f;
                            e += (double)d * d;
                            v[bi][bj][r] = a.gs * d;
                        } else if (on) {
                            a.out[y0 + (long long)row * nout + j] = y * a.tscale[t];
                        }
                    }
            }
        }
    }
    if constexpr (GRAD) {
        float* cs = a.csum + (size_t)blk * NCB;
        if (head) {
            put_block<true, true>(v, col0, nr, buf[0], a.fy + (size_t)blk * YFB * FRAG);
            const int c0 = 3 * HID + (t > 0 ? HEAD_OUT[0] : 0) + (t > 1 ? HEAD_OUT[1] : 0);
            put_sums(v, nr, cs + c0 + col0, nout - col0);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) e += __shfl_xor(e, off, 64);
        if (lane == 0) red[wv] = e;
        // v = dH of a layer -> dZ = dH silu'(z), its fragments and sums
        auto backward = [&](const Acc& zz, int layer) {
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[bi][bj][r] *= dsilu_f(zz[bi][bj][r]);
            put_sums(v, nr, cs + layer * HID + col0, 32);
        };
        if (t == 0) {
            WaveB<8> w;
            w.load(a.pk + PH0T, wv * 2);
            __syncthreads();
            w.mul(buf[0], v);
        } else {
            WaveB<1> w;
            w.load(a.pk + (t == 1 ? PH1T : PH2T), wv * 2);
            __syncthreads();
            w.mul(buf[0], v);
        }
        if (tid == 0) {
            double s = 0.0;
            for (int k = 0; k < NET_WG / 64; ++k) s += red[k];
            a.esum[blk] = s;
        }
        backward(z[2], 2);
        put_block<true, true>(v, col0, nr, buf[1], a.fg[2] + fo);
        {
            WaveB<HID / 32> w;
            w.load(a.pk + PW3T, wv * 2);
            __syncthreads();
            w.mul(buf[1], v);
        }
        backward(z[1], 1);
        put_block<true, true>(v, col0, nr, buf[0], a.fg[1] + fo);
        {
            WaveB<HID / 32> w;
            w.load(a.pk + PW2T, wv * 2);
            __syncthreads();
            w.mul(buf[0], v);
        }
        backward(z[0], 0);
        put_block<false, true>(v, col0, nr, nullptr, a.fg[0] + fo);
    }
}

// Weight gradients, dW = G^T H: 64 x 64 tiles of the six matrices, the
// contracted rows split over chunks of row blocks (blockIdx.x), within a chunk
// over the workgroup's four waves.  A tile's chain over 8192 rows on one
// workgroup left 16 workgroups at work for over a millisecond a layer; eight
// chunks are 544 workgroups, 15 us, and 0.96 MB of partial sums each.  All
// fragments are whole, so loads need no bounds.
constexpr int GTILES = 3 * 16 - 4 + 16 + 4 + 4;   // W3, W2 (16 each), W1 (12), H0 (16), H1, H2 (4 each)

struct WGradArgs {
    const bf16_t *fx, *fh[3], *fg[3], *fy;
    int blk0[NTYPE + 1], chunk;          // row blocks per chunk
    long long off[6];                    // of the matrices' gradients: W3 W2 W1 H0 H1 H2
    float* part;                         // per chunk, packed as the parameters
    long long stride;                    // of a chunk in part
};

__global__ __launch_bounds__(256) void k_wgrad(const WGradArgs a) {
    __shared__ float red[4][32][64];
    const int tile = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int m, idx, nj = 4, t = -1;          // matrix, tile in it, tiles per row
    if (tile < 32) {
        m = tile >> 4;
        idx = tile & 15;
    } else if (tile < 44) {
        m = 2;
        idx = tile - 32;
        nj = 3;
    } else {
        t = tile < 60 ? 0 : tile < 64 ? 1 : 2;
        m = 3 + t;
        idx = tile - (t == 0 ? 44 : t == 1 ? 60 : 64);
    }
    const int it = idx / nj, jt = idx % nj;
    const int rows = t < 0 ? HID : t == 0 ? HEAD_OUT[0] : t == 1 ? HEAD_OUT[1] : HEAD_OUT[2];
    const int cols = m == 2 ? NFEAT : HID;
    const int afb = t < 0 ? FB : YFB, bfb = m == 2 ? XFB : FB;
    const bf16_t* A = t < 0 ? a.fg[2 - m] : a.fy;
    const bf16_t* B = m == 2 ? a.fx : m == 0 ? a.fh[1] : m == 1 ? a.fh[0] : a.fh[2];
    const int lo = max((int)blockIdx.x * a.chunk, t < 0 ? 0 : a.blk0[t]);
    const int hi = min(((int)blockIdx.x + 1) * a.chunk, t < 0 ? a.blk0[NTYPE] : a.blk0[t + 1]);
    if (lo >= hi) return;                // a head's chunk without rows of its type: not summed either
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ni = min(4, (rows + 15) / 16 - it * 4);   // fragments of the tile that hold rows of the matrix
    for (int k = lo + wv; k < hi; k += 4) {
        const uint4* pa = reinterpret_cast<const uint4*>(A + ((size_t)k * afb + it * 4) * FRAG) + lane;
        const uint4* pb = reinterpret_cast<const uint4*>(B + ((size_t)k * bfb + jt * 4) * FRAG) + lane;
        uint4 ua[4], ub[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ua[i] = i < ni ? pa[i * 64] : make_uint4(0, 0, 0, 0);
            ub[i] = pb[i * 64];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, ua[i]), __builtin_bit_cast(bf16x8, ub[j]), acc[i][j], 0, 0, 0);
    }
    float* out = a.part + blockIdx.x * a.stride + a.off[m];
    const int col = jt * 64 + lane;
#pragma unroll
    for (int h = 0; h < 2; ++h) {        // the waves' sums, 32 rows at a time
        if (h) __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    red[wv][i * 16 + (lane >> 4) * 4 + r][j * 16 + (lane & 15)] = acc[2 * h + i][j][r];
        __syncthreads();
        for (int r = wv; r < 32; r += 4) {
            const int row = it * 64 + h * 32 + r;
            if (row < rows && col < cols)
                out[(size_t)row * cols + col] = red[0][r][lane] + red[1][r][lane] + red[2][r][lane] + red[3][r][lane];
        }
    }
}

// Sums over chunks (weights) and over row blocks (biases, squared error) into
// the packed gradient: blocks [0, nwb) take the weights, then one block per 16
// biases, then one for the error.
struct GradSumArgs {
    long long off[NTRAIN + 1];           // parameter offsets
    const float* part;
    long long stride;
    int blk0[NTYPE + 1], chunk, nwb;
    const float* csum;
    const double* esum;
    float* gr;
    double* loss;
};

__global__ __launch_bounds__(WG) void k_grad_sum(const GradSumArgs a) {
    __shared__ double red[WG];
    const int b = blockIdx.x, nblk = a.blk0[NTYPE];
    if (b < a.nwb) {
        const long long i = (long long)b * WG + threadIdx.x;
        if (i >= a.off[NTRAIN]) return;
        int s = 0;
        while (i >= a.off[s + 1]) ++s;
        if (s & 1) return;               // a bias
        const int t = s / 2 - 3;         // head, or < 0
        const int lo = t < 0 ? 0 : a.blk0[t] / a.chunk;
        const int hi = t < 0 ? (nblk + a.chunk - 1) / a.chunk
                             : a.blk0[t + 1] > a.blk0[t] ? (a.blk0[t + 1] - 1) / a.chunk + 1 : lo;
        float v = 0.0f;
        for (int c = lo; c < hi; ++c) v += a.part[c * a.stride + i];
        a.gr[i] = v;
        return;
    }
    const int nbb = (NCB + 15) / 16;
    if (b < a.nwb + nbb) {
        const int cx = threadIdx.x & 15, ry = threadIdx.x >> 4, j = (b - a.nwb) * 16 + cx;
        float v = 0.0f;
        long long o = 0;
        if (j < NCB) {
            int lo = 0, hi = nblk;
            if (j < 3 * HID) {
                o = a.off[P_B1 + 2 * (j / HID)] + j % HID;
            } else {
                const int h = j - 3 * HID, t = h < HEAD_OUT[0] ? 0 : h < HEAD_OUT[0] + HEAD_OUT[1] ? 1 : 2;
                lo = a.blk0[t];
                hi = a.blk0[t + 1];
                o = a.off[P_C0 + 2 * t] + h - (t > 0 ? HEAD_OUT[0] : 0) - (t > 1 ? HEAD_OUT[1] : 0);
            }
#pragma unroll 4
            for (int k = lo + ry; k < hi; k += 16) v += a.csum[(size_t)k * NCB + j];
        }
        red[threadIdx.x] = v;
        __syncthreads();
        if (ry == 0 && j < NCB) {
            for (int k = 1; k < 16; ++k) v += (float)red[cx + 16 * k];
            a.gr[o] = v;
        }
        return;
    }
    double e = 0.0;
    for (int k = threadIdx.x; k < nblk; k += WG) e += a.esum[k];
    red[threadIdx.x] = e;
    __syncthreads();
    for (int h = WG / 2; h >= 1; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *a.loss = red[0];
}

__global__ void k_fill_f(float* __restrict__ p, long long n, float v) {
    const long long i = (long long)blockIdx.x * WG + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long long n, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
    const long long i = (long long)blockIdx.x * WG + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

}  // namespace

// ---- context side: pairs, frames, features ----------------------------------------------

struct GuessPairsDev {
    int counts[NTYPE] = {0, 0, 0};
    int npair = 0;
    long long npacked = 0;
    int4* d_pairs = nullptr;
    double* d_frames = nullptr;
    float* d_feat = nullptr;
    long long* d_off = nullptr;
    double* d_xyz = nullptr;
    int* d_elem = nullptr;
    double* d_env = nullptr;
    int *d_first = nullptr, *d_nb = nullptr, *d_shoff = nullptr, *d_nsh = nullptr, *d_shl = nullptr;
    float* d_T = nullptr;
    double* d_red = nullptr;
    std::vector<int> hpairs;
    AtomBasis ab() const { return AtomBasis{d_first, d_nb, d_shoff, d_nsh, d_shl}; }
};

template <typename T>
static void gfree(T*& p) {
    if (p) (void)hipFree((void*)p);
    p = nullptr;
}
template <typename T>
static hipError_t galloc(T** p, size_t n) {
    *p = nullptr;
    return hipMalloc((void**)p, std::max<size_t>(n, 1) * sizeof(T));
}

void hfx_guess_release(hfx_ctx* c) {
    GuessPairsDev* G = c->guess;
    if (!G) return;
    gfree(G->d_pairs);
    gfree(G->d_frames);
    gfree(G->d_feat);
    gfree(G->d_off);
    gfree(G->d_xyz);
    gfree(G->d_elem);
    gfree(G->d_env);
    gfree(G->d_first);
    gfree(G->d_nb);
    gfree(G->d_shoff);
    gfree(G->d_nsh);
    gfree(G->d_shl);
    gfree(G->d_T);
    gfree(G->d_red);
    delete G;
    c->guess = nullptr;
}

#define GCK(call)                                                        \
    do {                                                                 \
        hfx_status _s = hfx_hip_check(c, (call), #call);                 \
        if (_s != HFX_OK) return _s;                                     \
    } while (0)

static int element_index(int z) { return z == 8 ? 0 : (z == 1 ? 1 : -1); }

extern "C" hfx_status hfx_guess_setup(hfx_ctx* c, int* counts) {
    if (!c) return HFX_ERR_INVALID_ARG;
    if (!c->loaded) return hfx_fail(c, HFX_ERR_STATE, "guess: nothing loaded");
    if (c->nmol != 1) return hfx_fail(c, HFX_ERR_STATE, "guess: single molecules only");
    GCK(hipSetDevice(c->opt.device));
    hfx_guess_release(c);
    const int na = c->natom;
    std::vector<int> elem(na), first(na, -1), nb(na, 0), nsh(na, 0), shoff(na, 0), shl;
    for (int a = 0; a < na; ++a) {
        elem[a] = element_index(c->Z[a]);
        if (elem[a] < 0) return hfx_fail(c, HFX_ERR_INVALID_ARG, "guess: elements O and H only");
    }
    std::vector<std::vector<int>> als(na);
    for (int s = 0; s < c->nshell; ++s) {
        const int a = c->shell_atom[s];
        if (first[a] < 0) first[a] = c->shells[s].bf;
        als[a].push_back(c->shells[s].l);
        nb[a] += (c->shells[s].l + 1) * (c->shells[s].l + 2) / 2;
    }
    for (int a = 0; a < na; ++a) {
        const int want = elem[a] == 0 ? 15 : 2;
        if (nb[a] != want)
            return hfx_fail(c, HFX_ERR_INVALID_ARG, "guess: the network needs 15 functions on O and 2 on H");
        shoff[a] = (int)shl.size();
        nsh[a] = (int)als[a].size();
        for (int l : als[a]) shl.push_back(l);
    }
    // pairs within the cutoff, A <= B in (element, index) order; sorted by type
    std::vector<int4> pairs;
    for (int a = 0; a < na; ++a)
        for (int b = 0; b < na; ++b) {
            if (std::make_pair(elem[a], a) > std::make_pair(elem[b], b)) continue;
            const double* pa = &c->axyz[3 * a];
            const double* pb = &c->axyz[3 * b];
            const double dx = pb[0] - pa[0], dy = pb[1] - pa[1], dz = pb[2] - pa[2];
            if (std::sqrt(dx * dx + dy * dy + dz * dz) / BOHR_PER_A >= RCUT_A) continue;
            pairs.push_back(int4{a, b, elem[a] + elem[b], 0});
        }
    std::stable_sort(pairs.begin(), pairs.end(), [](const int4& u, const int4& v) {
        return u.z != v.z ? u.z < v.z : (u.x != v.x ? u.x < v.x : u.y < v.y);
    });
    auto* G = new GuessPairsDev();
    c->guess = G;
    G->npair = (int)pairs.size();
    std::vector<long long> off(pairs.size());
    long long o = 0;
    for (size_t p = 0; p < pairs.size(); ++p) {
        G->counts[pairs[p].z]++;
        off[p] = o;
        o += (long long)nb[pairs[p].x] * nb[pairs[p].y];
    }
    G->npacked = o;
    for (auto& p : pairs) {
        G->hpairs.push_back(p.x);
        G->hpairs.push_back(p.y);
    }
    GCK(galloc(&G->d_pairs, pairs.size()));
    GCK(galloc(&G->d_frames, pairs.size() * 9));
    GCK(galloc(&G->d_feat, pairs.size() * NFEAT));
    GCK(galloc(&G->d_off, pairs.size()));
    GCK(galloc(&G->d_xyz, (size_t)na * 3));
    GCK(galloc(&G->d_elem, na));
    GCK(galloc(&G->d_env, (size_t)na * 2 * NRAD));
    GCK(galloc(&G->d_first, na));
    GCK(galloc(&G->d_nb, na));
    GCK(galloc(&G->d_shoff, na));
    GCK(galloc(&G->d_nsh, na));
    GCK(galloc(&G->d_shl, shl.size()));
    GCK(galloc(&G->d_T, (size_t)o));
    GCK(galloc(&G->d_red, 2));
    GCK(hipMemcpy(G->d_pairs, pairs.data(), pairs.size() * sizeof(int4), hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_off, off.data(), off.size() * 8, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_xyz, c->axyz.data(), (size_t)na * 3 * 8, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_elem, elem.data(), na * 4, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_first, first.data(), na * 4, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_nb, nb.data(), na * 4, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_shoff, shoff.data(), na * 4, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_nsh, nsh.data(), na * 4, hipMemcpyHostToDevice));
    GCK(hipMemcpy(G->d_shl, shl.data(), shl.size() * 4, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_env, dim3(blocks_for((long long)na * 2 * NRAD)), dim3(WG), 0, nullptr, na, G->d_xyz,
                       G->d_elem, G->d_env);
    GCK(hipGetLastError());
    if (G->npair > 0) {
        hipLaunchKernelGGL(k_pair_setup, dim3(blocks_for(G->npair)), dim3(WG), 0, nullptr, na, G->d_xyz, G->d_elem,
                           G->d_env, G->npair, G->d_pairs, G->d_feat, G->d_frames);
        GCK(hipGetLastError());
    }
    GCK(hipDeviceSynchronize());
    if (counts)
        for (int t = 0; t < NTYPE; ++t) counts[t] = G->counts[t];
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_features(hfx_ctx* c, float* X, int* pairs, double* frames) {
    if (!c) return HFX_ERR_INVALID_ARG;
    if (!c->guess) return hfx_fail(c, HFX_ERR_STATE, "guess: call hfx_guess_setup first");
    GuessPairsDev* G = c->guess;
    GCK(hipSetDevice(c->opt.device));
    if (X) GCK(hipMemcpy(X, G->d_feat, (size_t)G->npair * NFEAT * 4, hipMemcpyDeviceToHost));
    if (frames) GCK(hipMemcpy(frames, G->d_frames, (size_t)G->npair * 9 * 8, hipMemcpyDeviceToHost));
    if (pairs) std::memcpy(pairs, G->hpairs.data(), G->hpairs.size() * sizeof(int));
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_features_dev(hfx_ctx* c, const float** dX) {
    if (!c || !dX) return HFX_ERR_INVALID_ARG;
    if (!c->guess) return hfx_fail(c, HFX_ERR_STATE, "guess: call hfx_guess_setup first");
    *dX = c->guess->d_feat;
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_targets_dev(hfx_ctx* c, const double* dD, const double* dDbase, float* dT,
                                            void* stream) {
    if (!c || !dD || !dT) return c ? hfx_fail(c, HFX_ERR_INVALID_ARG, "null pointer") : HFX_ERR_INVALID_ARG;
    if (!c->guess) return hfx_fail(c, HFX_ERR_STATE, "guess: call hfx_guess_setup first");
    GuessPairsDev* G = c->guess;
    GCK(hipSetDevice(c->opt.device));
    if (G->npair == 0) return HFX_OK;
    hipLaunchKernelGGL(k_to_local, dim3(G->npair), dim3(64), 0, (hipStream_t)stream, G->npair, G->d_pairs,
                       G->d_frames, G->ab(), G->d_off, dD, dDbase, c->nbf, dT);
    GCK(hipGetLastError());
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_assemble_dev(hfx_ctx* c, const float* dT, const double* dDbase, double* dD,
                                             void* stream) {
    if (!c || !dT || !dD) return c ? hfx_fail(c, HFX_ERR_INVALID_ARG, "null pointer") : HFX_ERR_INVALID_ARG;
    if (!c->guess) return hfx_fail(c, HFX_ERR_STATE, "guess: call hfx_guess_setup first");
    GuessPairsDev* G = c->guess;
    GCK(hipSetDevice(c->opt.device));
    const size_t nn = (size_t)c->nbf * c->nbf;
    if (dDbase && dDbase != dD)
        hipLaunchKernelGGL(k_copy, dim3(blocks_for((long long)std::min<size_t>(nn, 1u << 22))), dim3(WG), 0,
                           (hipStream_t)stream, dDbase, nn, dD);
    if (G->npair > 0)
        hipLaunchKernelGGL(k_assemble_blocks, dim3(G->npair), dim3(64), 0, (hipStream_t)stream, G->npair,
                           G->d_pairs, G->d_frames, G->ab(), G->d_off, dT, c->nbf, dD);
    GCK(hipGetLastError());
    return HFX_OK;
}

// ---- the network object ----------------------------------------------------------------

struct hfx_guess {
    int device = 0;
    std::string err;
    std::vector<float> hp;
    float *p = nullptr, *gr = nullptr, *m = nullptr, *v = nullptr;
    bf16_t* pk = nullptr;      // packed weights: packed where p changes, so that passes only read them
    // gradient scratch for cap row blocks and pcap chunks
    long long cap = 0, pcap = 0;
    bf16_t *fx = nullptr, *fh[3] = {}, *fg[3] = {}, *fy = nullptr;
    float *csum = nullptr, *part = nullptr;
    double *esum = nullptr, *d_loss = nullptr;
    long long step = 0;
};

static hfx_status gfail(hfx_guess* g, hfx_status s, const std::string& msg) {
    if (g) g->err = msg;
    return s;
}
#define NCK(call)                                                                                   \
    do {                                                                                            \
        hipError_t _e = (call);                                                                     \
        if (_e != hipSuccess)                                                                       \
            return gfail(g, _e == hipErrorOutOfMemory ? HFX_ERR_OOM : HFX_ERR_DEVICE,               \
                         std::string(#call) + ": " + hipGetErrorString(_e));                        \
    } while (0)

static void free_acts(hfx_guess* g) {
    gfree(g->fx);
    for (auto& f : g->fh) gfree(f);
    for (auto& f : g->fg) gfree(f);
    gfree(g->fy);
    gfree(g->csum);
    gfree(g->esum);
    gfree(g->part);
    g->cap = g->pcap = 0;
}

extern "C" void hfx_guess_destroy(hfx_guess* g) {
    if (!g) return;
    (void)hipSetDevice(g->device);
    free_acts(g);
    gfree(g->p);
    gfree(g->gr);
    gfree(g->m);
    gfree(g->v);
    gfree(g->pk);
    gfree(g->d_loss);
    delete g;
}

extern "C" long long hfx_guess_param_count(void) { return PL.total; }

static NetParams net_params(const hfx_guess* g) {
    return NetParams{g->p,
                     PL.off[P_W1], PL.off[P_B1], PL.off[P_W2], PL.off[P_B2], PL.off[P_W3], PL.off[P_B3],
                     {PL.off[P_H0], PL.off[P_H1], PL.off[P_H2]},
                     {PL.off[P_C0], PL.off[P_C1], PL.off[P_C2]},
                     PL.off[P_FMEAN], PL.off[P_FSCALE]};
}

static hipError_t pack_weights(const hfx_guess* g, hipStream_t st) {
    hipLaunchKernelGGL(k_pack, dim3(blocks_for(PWTOT)), dim3(WG), 0, st, net_params(g), g->pk);
    return hipGetLastError();
}

extern "C" hfx_status hfx_guess_create(int device, hfx_guess** out) {
    if (!out) return HFX_ERR_INVALID_ARG;
    *out = nullptr;
    auto* g = new hfx_guess();
    g->device = device;
    auto fail = [&](hfx_status s) {
        hfx_guess_destroy(g);
        return s;
    };
    if (hipSetDevice(device) != hipSuccess) return fail(HFX_ERR_DEVICE);
    const long long n = PL.total;
    if (galloc(&g->p, n) || galloc(&g->gr, n) || galloc(&g->m, n) || galloc(&g->v, n) ||
        galloc(&g->pk, (size_t)PWTOT) || galloc(&g->d_loss, 1))
        return fail(HFX_ERR_OOM);
    g->hp.assign(n, 0.0f);
    for (int k = 0; k < NFEAT; ++k) g->hp[PL.off[P_FSCALE] + k] = 1.0f;
    for (int t = 0; t < NTYPE; ++t) g->hp[PL.off[P_TSCALE] + t] = 1.0f;
    if (hipMemcpy(g->p, g->hp.data(), n * 4, hipMemcpyHostToDevice) != hipSuccess) return fail(HFX_ERR_DEVICE);
    hipLaunchKernelGGL(k_fill_f, dim3(blocks_for(n)), dim3(WG), 0, nullptr, g->m, n, 0.0f);
    hipLaunchKernelGGL(k_fill_f, dim3(blocks_for(n)), dim3(WG), 0, nullptr, g->v, n, 0.0f);
    hipLaunchKernelGGL(k_fill_f, dim3(blocks_for(n)), dim3(WG), 0, nullptr, g->gr, n, 0.0f);
    if (pack_weights(g, nullptr) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return fail(HFX_ERR_DEVICE);
    *out = g;
    return HFX_OK;
}

extern "C" const char* hfx_guess_last_error(const hfx_guess* g) { return g ? g->err.c_str() : "null network"; }

extern "C" hfx_status hfx_guess_set_params(hfx_guess* g, const float* params) {
    if (!g || !params) return HFX_ERR_INVALID_ARG;
    for (long long i = 0; i < PL.total; ++i)
        if (!std::isfinite(params[i])) return gfail(g, HFX_ERR_NUMERICAL, "guess: non-finite parameter");
    for (int k = 0; k < NFEAT; ++k)
        if (!(params[PL.off[P_FSCALE] + k] > 0.0f)) return gfail(g, HFX_ERR_INVALID_ARG, "guess: feature scale <= 0");
    for (int t = 0; t < NTYPE; ++t)
        if (!(params[PL.off[P_TSCALE] + t] > 0.0f)) return gfail(g, HFX_ERR_INVALID_ARG, "guess: target scale <= 0");
    NCK(hipSetDevice(g->device));
    g->hp.assign(params, params + PL.total);
    NCK(hipMemcpy(g->p, params, PL.total * 4, hipMemcpyHostToDevice));
    NCK(pack_weights(g, nullptr));
    NCK(hipStreamSynchronize(nullptr));   // passes may follow on any stream
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_get_params(hfx_guess* g, float* params) {
    if (!g || !params) return HFX_ERR_INVALID_ARG;
    NCK(hipSetDevice(g->device));
    NCK(hipMemcpy(params, g->p, PL.total * 4, hipMemcpyDeviceToHost));
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_get_grads(hfx_guess* g, float* grads) {
    if (!g || !grads) return HFX_ERR_INVALID_ARG;
    NCK(hipSetDevice(g->device));
    NCK(hipMemcpy(grads, g->gr, PL.total * 4, hipMemcpyDeviceToHost));
    return HFX_OK;
}

// Gradient scratch for nblk row blocks in nchunk chunks.
static hfx_status ensure_cap(hfx_guess* g, long long nblk, long long nchunk) {
    if (nblk <= g->cap && nchunk <= g->pcap) return HFX_OK;
    const long long cap = std::max({nblk, g->cap, 32ll}), pcap = std::max(nchunk, g->pcap);
    free_acts(g);
    NCK(galloc(&g->fx, cap * XFB * FRAG));
    for (auto& f : g->fh) NCK(galloc(&f, cap * FB * FRAG));
    for (auto& f : g->fg) NCK(galloc(&f, cap * FB * FRAG));
    NCK(galloc(&g->fy, cap * YFB * FRAG));
    NCK(galloc(&g->csum, cap * NCB));
    NCK(galloc(&g->esum, cap));
    NCK(galloc(&g->part, pcap * PL.off[NTRAIN]));
    g->cap = cap;
    g->pcap = pcap;
    return HFX_OK;
}

// The network's arguments for a batch: rows of type t follow those of type
// t - 1 in X, its outputs in the packed blocks.
static hfx_status net_args(hfx_guess* g, const float* dX, const int* counts, NetArgs& a, long long& ny) {
    for (int t = 0; t < NTYPE; ++t)
        if (counts[t] < 0) return gfail(g, HFX_ERR_INVALID_ARG, "guess: negative row count");
    a = NetArgs{};
    a.w = net_params(g);
    a.pk = g->pk;
    a.X = dX;
    long long M = 0;
    ny = 0;
    for (int t = 0; t < NTYPE; ++t) {
        a.count[t] = counts[t];
        a.row0[t] = M;
        a.yoff[t] = ny;
        a.blk0[t + 1] = a.blk0[t] + (counts[t] + RB - 1) / RB;
        a.tscale[t] = g->hp[PL.off[P_TSCALE] + t];
        a.inv_tscale[t] = 1.0f / a.tscale[t];
        M += counts[t];
        ny += (long long)counts[t] * HEAD_OUT[t];
    }
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_forward_dev(hfx_guess* g, const float* dX, const int* counts, float* dT,
                                            void* stream) {
    if (!g || !counts || !dT || !dX) return HFX_ERR_INVALID_ARG;
    NCK(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    NetArgs a;
    long long ny;
    hfx_status s = net_args(g, dX, counts, a, ny);
    if (s != HFX_OK) return s;
    a.out = dT;
    if (a.blk0[NTYPE] > 0)
        hipLaunchKernelGGL(k_net<false>, dim3(a.blk0[NTYPE]), dim3(NET_WG), 0, st, a);
    NCK(hipGetLastError());
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_grad_dev(hfx_guess* g, const float* dX, const int* counts, const float* dT,
                                         void* stream, double* loss) {
    if (!g || !counts || !dT || !dX) return HFX_ERR_INVALID_ARG;
    NCK(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    NetArgs a;
    long long ny;
    hfx_status s = net_args(g, dX, counts, a, ny);
    if (s != HFX_OK) return s;
    const int nblk = a.blk0[NTYPE];
    // Chunks in eights: the workgroups of a chunk, eight apart in launch order,
    // then share an XCD, whose 4 MB L2 holds the chunk's fragments (124 KB a row
    // block; up to 32 blocks, 4 MB, to 1024 blocks in all).  At most 32 chunks: the
    // partial sums stay below 31 MB for any batch.
    const int want = nblk <= 16 ? 1 : 8 * std::min(4, (nblk + 255) / 256);
    const int chunk = std::max(1, (nblk + want - 1) / want), nchunk = nblk <= 16 ? 1 : want;
    s = ensure_cap(g, nblk, nchunk);
    if (s != HFX_OK) return s;
    if (ny == 0) return gfail(g, HFX_ERR_INVALID_ARG, "guess: empty batch");
    WGradArgs wg{};
    GradSumArgs gs{};
    a.T = dT;
    a.gs = 2.0f / (float)ny;
    a.fx = g->fx;
    a.fy = g->fy;
    a.csum = g->csum;
    a.esum = g->esum;
    wg.fx = g->fx;
    wg.fy = g->fy;
    for (int k = 0; k < 3; ++k) {
        wg.fh[k] = a.fh[k] = g->fh[k];
        wg.fg[k] = a.fg[k] = g->fg[k];
    }
    const int mats[6] = {P_W3, P_W2, P_W1, P_H0, P_H1, P_H2};
    for (int k = 0; k < 6; ++k) wg.off[k] = PL.off[mats[k]];
    for (int t = 0; t <= NTYPE; ++t) wg.blk0[t] = gs.blk0[t] = a.blk0[t];
    for (int k = 0; k <= NTRAIN; ++k) gs.off[k] = PL.off[k];
    wg.chunk = gs.chunk = chunk;
    wg.stride = gs.stride = PL.off[NTRAIN];
    wg.part = g->part;
    gs.part = g->part;
    gs.nwb = (int)blocks_for(PL.off[NTRAIN]);
    gs.csum = g->csum;
    gs.esum = g->esum;
    gs.gr = g->gr;
    gs.loss = g->d_loss;
    hipLaunchKernelGGL(k_net<true>, dim3(nblk), dim3(NET_WG), 0, st, a);
    hipLaunchKernelGGL(k_wgrad, dim3(nchunk, GTILES), dim3(256), 0, st, wg);
    hipLaunchKernelGGL(k_grad_sum, dim3(gs.nwb + (NCB + 15) / 16 + 1), dim3(WG), 0, st, gs);
    NCK(hipGetLastError());
    if (loss) {
        double l = 0.0;
        NCK(hipMemcpyAsync(&l, g->d_loss, 8, hipMemcpyDeviceToHost, st));
        NCK(hipStreamSynchronize(st));
        *loss = l / (double)ny;
    }
    return HFX_OK;
}

extern "C" hfx_status hfx_guess_adam(hfx_guess* g, double lr, void* stream) {
    if (!g || !(lr > 0)) return g ? gfail(g, HFX_ERR_INVALID_ARG, "guess: lr must be positive") : HFX_ERR_INVALID_ARG;
    NCK(hipSetDevice(g->device));
    g->step += 1;
    const double b1 = 0.9, b2 = 0.999;
    const float c1 = (float)(1.0 / (1.0 - std::pow(b1, (double)g->step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow(b2, (double)g->step)));
    const long long n = PL.off[NTRAIN];   // weights and biases only
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(WG), 0, (hipStream_t)stream, g->p, g->gr, g->m, g->v, n,
                       (float)lr, (float)b1, (float)b2, 1e-8f, c1, c2);
    NCK(hipGetLastError());
    NCK(pack_weights(g, (hipStream_t)stream));
    return HFX_OK;
}

// D (device, in/out): the SAD density on entry; on success D + sum of the
// predicted blocks.  The prediction is rejected (D restored, *used = 0) when
// it is not finite or |tr(D S) - nocc| > 0.05 nocc.
extern "C" hfx_status hfx_guess_apply(hfx_ctx* c, hfx_guess* g, double* dD, void* stream, int* used) {
    if (!c || !g || !dD) return c ? hfx_fail(c, HFX_ERR_INVALID_ARG, "null pointer") : HFX_ERR_INVALID_ARG;
    if (used) *used = 0;
    hfx_status s = HFX_OK;
    if (!c->guess) {
        s = hfx_guess_setup(c, nullptr);
        if (s != HFX_OK) return s;
    }
    GuessPairsDev* G = c->guess;
    hipStream_t st = (hipStream_t)stream;
    GCK(hipSetDevice(c->opt.device));
    const size_t nn = (size_t)c->nbf * c->nbf;
    double* base = nullptr;
    GCK(galloc(&base, nn));
    hipLaunchKernelGGL(k_copy, dim3(blocks_for((long long)std::min<size_t>(nn, 1u << 22))), dim3(WG), 0, st, dD, nn,
                       base);
    s = hfx_guess_forward_dev(g, G->d_feat, G->counts, G->d_T, stream);
    if (s != HFX_OK) {
        gfree(base);
        return hfx_fail(c, s, std::string("guess network: ") + g->err);
    }
    s = hfx_guess_assemble_dev(c, G->d_T, nullptr, dD, stream);
    if (s != HFX_OK) {
        gfree(base);
        return s;
    }
    double red[2] = {0.0, 0.0};
    hipError_t e = hipMemsetAsync(G->d_red, 0, 16, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_trace_check, dim3(blocks_for((long long)std::min<size_t>(nn, 1u << 20))), dim3(WG), 0,
                           st, dD, c->d_S, nn, G->d_red);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(red, G->d_red, 16, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        gfree(base);
        return hfx_hip_check(c, e, "guess trace check");
    }
    const bool ok = red[1] == 0.0 && std::isfinite(red[0]) && std::fabs(red[0] - c->nocc) <= 0.05 * c->nocc;
    if (!ok)
        hipLaunchKernelGGL(k_copy, dim3(blocks_for((long long)std::min<size_t>(nn, 1u << 22))), dim3(WG), 0, st, base,
                           nn, dD);
    e = hipStreamSynchronize(st);
    gfree(base);
    GCK(e);
    if (used) *used = ok ? 1 : 0;
    return HFX_OK;
}
