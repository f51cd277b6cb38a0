// Support kernels around the class kernels: density preparation, the
// per-bra FP64/FP32 split, Fock assembly and the small SCF helpers.  All are HBM-bound elementwise passes or tiny.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hfx_internal.h"

#define MISC_WG 256

// ---- per build --------------------------------------------------------------

// Matrices are stored per molecule (ragged): molecule m's nbf_m x nbf_m
// block starts at element moff[m]; its basis functions are global indices
// mboff[m] .. mboff[m] + nbf_m - 1 (component factors cs[]).  Elementwise
// kernels run on a (gx, nmol) grid, row y = molecule.

// The start of a build in one launch.  A small molecule's build is bound by its
// launches: fills, density and a fill, a gather and a scatter per ket list, 23
// beside the class kernels of a water dimer, are now this, one scatter and the
// assembly: 183 -> 134 us (five waters as a replayed graph 566 -> 455 us).
// The first gx columns of the grid, row y = molecule: D' = s_m s_n D (component
// normalisation moved onto the density), W = 0, and, where dmax_bits is given
// (zeroed before), dmax = max |D| (the bit pattern of a non-negative double is
// order preserving).  The other columns: per element of the ket lists' blocks
// D'_cd in list order, from D itself, so that the class kernels read it
// coalesced by ket position, and the zeroed J accumulator.  Workgroup 0 clears
// the counters and the queues.
__global__ void k_start_build(const double* __restrict__ D, const double* __restrict__ cs,
                              const long long* __restrict__ moff, const int* __restrict__ mdim,
                              const int* __restrict__ mboff, int gx, const KetElem* __restrict__ ke, size_t nke,
                              const StartBufs b) {
    if ((int)blockIdx.x >= gx) {
        const size_t kx = gridDim.x - gx, step = kx * gridDim.y * MISC_WG;
        for (size_t i = ((size_t)blockIdx.y * kx + blockIdx.x - gx) * MISC_WG + threadIdx.x; i < nke; i += step) {
            const KetElem e = ke[i];
            if (e.idx < 0) continue;   // between two lists
            b.dket[i] = e.s * D[e.idx];
            b.wket[i] = 0.0;
        }
        return;
    }
    const int mol = blockIdx.y;
    const int n = mdim[mol];
    const size_t nn = (size_t)n * n, base = (size_t)moff[mol];
    const double* __restrict__ c = cs + mboff[mol];
    double mx = 0.0;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < nn; i += (size_t)gx * MISC_WG) {
        const double d = D[base + i];
        b.Dp[base + i] = c[i / n] * c[i % n] * d;
        b.W[base + i] = 0.0;
        const double ad = fabs(d);
        mx = (ad > mx || ad != ad) ? ad : mx;   // NaN propagates
    }
    if (b.dmax_bits) {
        // one word for the whole build, on which atomics run one after the other: one
        // per workgroup, and none where the word is as large already (it only grows).
        // With one per wave a batch of 256 clusters, on a grid for its largest
        // molecule, spent 4.4 ms here, more than FP32 evaluation saved.
        __shared__ double wave_max[MISC_WG / 64];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const double o = __shfl_xor(mx, off, 64);
            mx = (o > mx || o != o) ? o : mx;
        }
        if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = mx;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < MISC_WG / 64; ++w) mx = (wave_max[w] > mx || wave_max[w] != wave_max[w]) ? wave_max[w] : mx;
            const unsigned long long u =
                mx != mx ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(mx);
            if (u > __hip_atomic_load(b.dmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(b.dmax_bits, u);
        }
    }
    if (blockIdx.x == 0 && mol == 0) {
        for (int i = threadIdx.x; i < b.ncounters; i += MISC_WG) b.counters[i] = 0ull;
        for (int i = threadIdx.x; i < b.nwork; i += MISC_WG) b.work[i] = 0ull;
    }
}

__global__ void k_fill(double* __restrict__ p, size_t n, double v) {
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < n; i += (size_t)gridDim.x * MISC_WG) p[i] = v;
}

__global__ void k_fill_u64(unsigned long long* __restrict__ p, int n) {
    const int i = blockIdx.x * MISC_WG + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// FP64/FP32 split per task (bra r, kets [s0, s1) of one group): the kets s
// with Q_r Q_s max|D| >= fp32_tau come first (Q descending within a group);
// split[t] is the list position of the first FP32 ket (s1 if none).
__global__ void k_split(const PairInfo* __restrict__ bra, const KetListDev* __restrict__ lists,
                        const double* __restrict__ all_ketq, const int4* __restrict__ tasks, int ntask, double fp32_tau,
                        const unsigned long long* __restrict__ dmax_bits, int* __restrict__ split) {
    const int t = blockIdx.x * MISC_WG + threadIdx.x;
    if (t >= ntask) return;
    const int4 tk = tasks[t];
    if (tk.x < 0) {
        split[t] = 0;
        return;
    }
    const double* ketq = all_ketq + lists[hfx_task_list(tk.w)].s0;
    const double qr = bra[tk.x].Q * __longlong_as_double((long long)*dmax_bits);
    int lo = tk.y, hi = tk.z;   // Q descending within a task's kets: the FP32 ones are a suffix
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ketq[mid] * qr >= fp32_tau) lo = mid + 1; else hi = mid;
    }
    split[t] = lo;
}

// F = H + s_m s_n (W + W^T) / 8 per molecule block (H may be null: two-electron
// part only); raises *bad if a non-finite value appears.
__global__ void k_assemble(const double* __restrict__ H, const double* __restrict__ W, const double* __restrict__ cs,
                           const long long* __restrict__ moff, const int* __restrict__ mdim,
                           const int* __restrict__ mboff, double* __restrict__ F, int* __restrict__ bad) {
    const int mol = blockIdx.y;
    const int n = mdim[mol];
    const size_t nn = (size_t)n * n, base = (size_t)moff[mol];
    const double* __restrict__ c = cs + mboff[mol];
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < nn; i += (size_t)gridDim.x * MISC_WG) {
        const size_t r = i / n, col = i % n;
        const double g = 0.125 * c[r] * c[col] * (W[base + i] + W[base + col * n + r]);
        const double f = (H ? H[base + i] : 0.0) + g;
        F[base + i] = f;
        if (!isfinite(f) && bad) *bad = 1;
    }
}

// W += sum of the nrep private copies of W (replica x at x * n): the
// reduction of algorithm 2's private Fock matrices, here one per XCD.
__global__ void k_reduce_replicas(const double* __restrict__ rep, int nrep, size_t n, double* __restrict__ W) {
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < n; i += (size_t)gridDim.x * MISC_WG) {
        double v = 0.0;
        for (int x = 0; x < nrep; ++x) v += rep[(size_t)x * n + i];
        W[i] += v;
    }
}

// FP32 copy of the primitive pairs.
__global__ void k_prim32(const double* __restrict__ prim, size_t n, float* __restrict__ out) {
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < n; i += (size_t)gridDim.x * MISC_WG)
        out[i] = (float)prim[i];
}

// The primitives of one list (kp a ket) as a structure of arrays, field f of
// primitive k of ket s at (f kp + k) n + s, and their FP32 copy.  Formed here
// and not on the host: loading 29 waters spent 2.5 ms on building and copying
// these arrays, now 1.1 ms with everything else of the ket lists.
__global__ void k_ket_soa(const PairInfo* __restrict__ kets, int n, int kp, const double* __restrict__ prim,
                          double* __restrict__ soa, float* __restrict__ soa32) {
    const long long tot = (long long)n * kp;
    for (long long i = (long long)blockIdx.x * MISC_WG + threadIdx.x; i < tot; i += (long long)gridDim.x * MISC_WG) {
        const int s = (int)(i % n), k = (int)(i / n);
        const double* p = prim + (size_t)(kets[s].prim_off + k) * HFX_PRIM_FIELDS;
#pragma unroll
        for (int f = 0; f < 9; ++f) {
            const size_t o = ((size_t)f * kp + k) * n + s;
            soa[o] = p[f];
            soa32[o] = (float)p[f];
        }
    }
}

// The elements of one list's ket blocks, component comp of pair s at comp n + s:
// their places in the matrices and the products of their component factors.
__global__ void k_ket_elems(const PairInfo* __restrict__ kets, int n, int nc, int nd, const long long* __restrict__ moff,
                            const int* __restrict__ mboff, const double* __restrict__ cs, KetElem* __restrict__ out) {
    const long long i = (long long)blockIdx.x * MISC_WG + threadIdx.x;
    if (i >= (long long)n * nc * nd) return;
    const int s = (int)(i % n), comp = (int)(i / n);
    const PairInfo p = kets[s];
    const int r = p.bfa + comp / nd, c = p.bfb + comp % nd;
    const double* m = cs + mboff[p.mol];
    out[i] = KetElem{moff[p.mol] + (long long)r * p.ld + c, m[r] * m[c]};
}

// W += the ket lists' J sums: each pair owns its W block, so plain
// read-modify-write (no atomics) after the class kernels.
__global__ void k_scatter_kets(const KetElem* __restrict__ ke, size_t nke, const double* __restrict__ wket,
                               double* __restrict__ W) {
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < nke; i += (size_t)gridDim.x * MISC_WG) {
        const long long idx = ke[i].idx;
        if (idx < 0) continue;
        const double v = wket[i];
        if (v != 0.0) W[idx] += v;
    }
}

// ---- SCF helpers ------------------------------------------------------------------

// out = A - A^T (column- or row-major alike)
__global__ void k_antisym(const double* __restrict__ A, int n, double* __restrict__ out) {
    const size_t nn = (size_t)n * n;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < nn; i += (size_t)gridDim.x * MISC_WG) {
        const size_t r = i / n, c = i % n;
        out[i] = A[i] - A[c * n + r];
    }
}

// partial sums of sum_i a_i * b_i (b may be null: sum a_i^2) and of (a_i - b_i)^2 (mode 1)
__global__ void k_dot(const double* __restrict__ a, const double* __restrict__ b, size_t n, int mode,
                      double* __restrict__ out) {
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < n; i += (size_t)gridDim.x * MISC_WG) {
        if (mode == 0) acc += a[i] * b[i];
        else { const double d = a[i] - b[i]; acc += d * d; }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    __shared__ double red[MISC_WG / 64];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < MISC_WG / 64; ++w) s += red[w];
        out[blockIdx.x] = s;
    }
}

// E-term: sum_ij D_ij (H_ij + F_ij)
__global__ void k_energy(const double* __restrict__ D, const double* __restrict__ H, const double* __restrict__ F,
                         size_t n, double* __restrict__ out) {
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < n; i += (size_t)gridDim.x * MISC_WG)
        acc += D[i] * (H[i] + F[i]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    __shared__ double red[MISC_WG / 64];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < MISC_WG / 64; ++w) s += red[w];
        out[blockIdx.x] = s;
    }
}

// out = sum_k c_k M_k (k < m), matrices of size n
__global__ void k_lincomb(const double* const* __restrict__ M, const double* __restrict__ c, int m, size_t n,
                          double* __restrict__ out) {
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < n; i += (size_t)gridDim.x * MISC_WG) {
        double s = 0.0;
        for (int k = 0; k < m; ++k) s += c[k] * M[k][i];
        out[i] = s;
    }
}

// X (column-major n x nk) from eigenpairs of S: symmetric S^{-1/2} when
// nothing is dropped, canonical U_k w_k^{-1/2} otherwise.
__global__ void k_scale_cols(const double* __restrict__ U, const double* __restrict__ w, const int* __restrict__ keep,
                             int n, int nk, double* __restrict__ out) {
    const size_t tot = (size_t)n * nk;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < tot; i += (size_t)gridDim.x * MISC_WG) {
        const int col = (int)(i / n), row = (int)(i % n);
        const int src = keep[col];
        out[i] = U[(size_t)src * n + row] / sqrt(w[src]);
    }
}

// Batched eigensolves over molecules of different sizes: slot m (NP x NP) of
// dst holds molecule m's block (n_m x n_m) in its top-left corner, `pad` on
// the rest of the diagonal and zeros elsewhere, so that the slot's
// eigenpairs are the block's plus (pad, unit vectors), sorted after them.
__global__ void k_pad_blocks(const double* __restrict__ src, const long long* __restrict__ moff,
                             const int* __restrict__ dim, int NP, double pad, double* __restrict__ dst) {
    const int mol = blockIdx.y;
    const int n = dim[mol];
    const size_t tot = (size_t)NP * NP;
    double* __restrict__ d = dst + (size_t)mol * tot;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < tot; i += (size_t)gridDim.x * MISC_WG) {
        const int r = (int)(i / NP), col = (int)(i % NP);
        d[i] = (r < n && col < n) ? src[moff[mol] + (size_t)r * n + col] : (r == col ? pad : 0.0);
    }
}

// Outside the top-left k_m x k_m block of every slot: pad on the diagonal, zeros elsewhere.
__global__ void k_pad_rest(const int* __restrict__ dim, int NP, double pad, double* __restrict__ dst) {
    const int mol = blockIdx.y;
    const int k = dim[mol];
    const size_t tot = (size_t)NP * NP;
    double* __restrict__ d = dst + (size_t)mol * tot;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < tot; i += (size_t)gridDim.x * MISC_WG) {
        const int r = (int)(i / NP), col = (int)(i % NP);
        if (r >= k || col >= k) d[i] = (r == col) ? pad : 0.0;
    }
}

// C (column-major n x nmo) -> weighted density D = sum_k occ_k C_k C_k^T
__global__ void k_weight_cols(const double* __restrict__ C, const double* __restrict__ occ, int n, int nk,
                              double* __restrict__ out) {
    const size_t tot = (size_t)n * nk;
    for (size_t i = (size_t)blockIdx.x * MISC_WG + threadIdx.x; i < tot; i += (size_t)gridDim.x * MISC_WG)
        out[i] = C[i] * occ[i / n];
}

// ---- C wrappers ---------------------------------------------------------------------

static int grid_for(size_t n) {
    size_t g = (n + MISC_WG - 1) / MISC_WG;
    if (g > 4096) g = 4096;
    return (int)(g ? g : 1);
}

extern "C" {
// Columns of a (columns, nmol) grid at most: below 2^32 work-items (the kernels stride).
static size_t most_columns(int nmol) { return ((1ull << 32) - 1) / ((size_t)MISC_WG * nmol); }
static dim3 ragged_grid(int max_ld, int nmol) {
    const size_t g = ((size_t)max_ld * max_ld + MISC_WG - 1) / MISC_WG;
    return dim3((unsigned)std::max<size_t>(1, std::min({g, (size_t)4096, most_columns(nmol)})), (unsigned)nmol);
}
hipError_t hfx_start_build(const double* D, const double* cs, int nmol, const long long* moff, const int* mdim,
                           const int* mboff, int max_ld, const KetElem* ke, size_t nke, const StartBufs* b,
                           hipStream_t st) {
    dim3 g = ragged_grid(max_ld, nmol);
    const size_t most = std::max<size_t>(2, most_columns(nmol));
    const size_t per = (size_t)MISC_WG * nmol, kx = std::min({(nke + per - 1) / per, (size_t)4096, most / 2});
    const int gx = (int)std::min<size_t>(g.x, most - kx);
    g.x = (unsigned)(gx + kx);
    hipLaunchKernelGGL(k_start_build, g, dim3(MISC_WG), 0, st, D, cs, moff, mdim, mboff, gx, ke, nke, *b);
    return hipGetLastError();
}
hipError_t hfx_fill(double* p, size_t n, double v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n)), dim3(MISC_WG), 0, st, p, n, v);
    return hipGetLastError();
}
hipError_t hfx_reduce_replicas(const double* rep, int nrep, size_t n, double* W, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_replicas, dim3(grid_for(n)), dim3(MISC_WG), 0, st, rep, nrep, n, W);
    return hipGetLastError();
}
hipError_t hfx_fill_u64(unsigned long long* p, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3((n + MISC_WG - 1) / MISC_WG), dim3(MISC_WG), 0, st, p, n);
    return hipGetLastError();
}
hipError_t hfx_split(const PairInfo* bra, const KetListDev* lists, const double* ketq, const int4* tasks, int ntask,
                     double fp32_tau, const unsigned long long* dmax_bits, int* split, hipStream_t st) {
    if (ntask <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_split, dim3((ntask + MISC_WG - 1) / MISC_WG), dim3(MISC_WG), 0, st, bra, lists, ketq,
                       tasks, ntask, fp32_tau, dmax_bits, split);
    return hipGetLastError();
}
hipError_t hfx_prim32(const PrimPair* prim, size_t n, float* out, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_prim32, dim3(grid_for(n * HFX_PRIM_FIELDS)), dim3(MISC_WG), 0, st, (const double*)prim,
                       n * HFX_PRIM_FIELDS, out);
    return hipGetLastError();
}
hipError_t hfx_ket_soa(const PairInfo* kets, int n, int kp, const PrimPair* prim, double* soa, float* soa32,
                       hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ket_soa, dim3(grid_for((size_t)n * kp)), dim3(MISC_WG), 0, st, kets, n, kp,
                       (const double*)prim, soa, soa32);
    return hipGetLastError();
}
hipError_t hfx_ket_elems(const PairInfo* kets, int n, int nc, int nd, const long long* moff, const int* mboff,
                         const double* cs, KetElem* out, hipStream_t st) {
    const long long tot = (long long)n * nc * nd;
    if (tot <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ket_elems, dim3((unsigned)((tot + MISC_WG - 1) / MISC_WG)), dim3(MISC_WG), 0, st, kets, n, nc,
                       nd, moff, mboff, cs, out);
    return hipGetLastError();
}
hipError_t hfx_scatter_kets(const KetElem* ke, size_t nke, const double* wket, double* W, hipStream_t st) {
    if (nke == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter_kets, dim3(grid_for(nke)), dim3(MISC_WG), 0, st, ke, nke, wket, W);
    return hipGetLastError();
}
hipError_t hfx_assemble(const double* H, const double* W, const double* cs, int nmol, const long long* moff,
                        const int* mdim, const int* mboff, int max_ld, double* F, int* bad, hipStream_t st) {
    hipLaunchKernelGGL(k_assemble, ragged_grid(max_ld, nmol), dim3(MISC_WG), 0, st, H, W, cs, moff, mdim, mboff, F, bad);
    return hipGetLastError();
}
hipError_t hfx_antisym(const double* A, int n, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_antisym, dim3(grid_for((size_t)n * n)), dim3(MISC_WG), 0, st, A, n, out);
    return hipGetLastError();
}
// returns the number of partial sums written to out (<= 4096)
int hfx_dot_partial(const double* a, const double* b, size_t n, int mode, double* out, hipStream_t st) {
    const int g = grid_for(n);
    hipLaunchKernelGGL(k_dot, dim3(g), dim3(MISC_WG), 0, st, a, b, n, mode, out);
    return g;
}
int hfx_energy_partial(const double* D, const double* H, const double* F, size_t n, double* out, hipStream_t st) {
    const int g = grid_for(n);
    hipLaunchKernelGGL(k_energy, dim3(g), dim3(MISC_WG), 0, st, D, H, F, n, out);
    return g;
}
hipError_t hfx_lincomb(const double* const* M, const double* c, int m, size_t n, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_lincomb, dim3(grid_for(n)), dim3(MISC_WG), 0, st, M, c, m, n, out);
    return hipGetLastError();
}
hipError_t hfx_scale_cols(const double* U, const double* w, const int* keep, int n, int nk, double* out,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_scale_cols, dim3(grid_for((size_t)n * nk)), dim3(MISC_WG), 0, st, U, w, keep, n, nk, out);
    return hipGetLastError();
}
hipError_t hfx_pad_blocks(const double* src, const long long* moff, const int* dim, int nmol, int NP, double pad,
                          double* dst, hipStream_t st) {
    const unsigned gx = (unsigned)std::min<size_t>(((size_t)NP * NP + MISC_WG - 1) / MISC_WG, 1024);
    hipLaunchKernelGGL(k_pad_blocks, dim3(gx, nmol), dim3(MISC_WG), 0, st, src, moff, dim, NP, pad, dst);
    return hipGetLastError();
}
hipError_t hfx_pad_rest(const int* dim, int nmol, int NP, double pad, double* dst, hipStream_t st) {
    const unsigned gx = (unsigned)std::min<size_t>(((size_t)NP * NP + MISC_WG - 1) / MISC_WG, 1024);
    hipLaunchKernelGGL(k_pad_rest, dim3(gx, nmol), dim3(MISC_WG), 0, st, dim, NP, pad, dst);
    return hipGetLastError();
}
hipError_t hfx_weight_cols(const double* C, const double* occ, int n, int nk, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_weight_cols, dim3(grid_for((size_t)n * nk)), dim3(MISC_WG), 0, st, C, occ, n, nk, out);
    return hipGetLastError();
}
}
