// Acquisition of the BOAC outer loop on the device, FP64: posterior mean, standard deviation and
// expected improvement (Eqs. 7-10, minimisation) of a fitted GP at M query points.
//
// With k*_m = k(q_m, u_.) (Eq. 8), the GP weights alpha = K^-1 z and X = L^-1 (K = L L^T):
//   mu_m = m0 + s k*_m . alpha,   var_m = s^2 (amp - |X k*_m|^2),
//   gamma = (J_best - mu - xi) / sigma,  EI = sigma (gamma Phi(gamma) + phi(gamma)).
// |X k*_m|^2 for all m is a triangular matrix product Z = X K*^T (n x M) reduced over its rows:
// Up to kGpFuseMax observations one kernel does all of it per 16 queries (k_gp_fused, after k_gp_pack has
// put X into the matrix cores' operand order); above that, where K* of 16 queries does not fit in LDS:
//   k_gp_kstar  K* [M][npad] (zero past n)
//   k_gp_zsq    per (64-row block of X, 64-query block): the Z block over j <= i on the FP64 matrix
//               cores, squared and summed over its rows -> part [n/64][M] (fixed order, no atomics)
//   k_gp_ei     one wave per query: k* . alpha, sum of the row-block partials, EI
// Both paths add in the same order and give the same bits.
#include <algorithm>

#include "launch.h"

namespace boac {

constexpr int kGpT = 64;   // rows of X and queries per block
constexpr int kGpJ = 16;   // columns per staging step

__global__ __launch_bounds__(256) void k_gp_kstar(GpEiArgs A) {
    const size_t total = (size_t)A.M * A.npad;
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < total; t += (size_t)gridDim.x * blockDim.x) {
        const int m = (int)(t / A.npad), j = (int)(t - (size_t)m * A.npad);
        double k = 0.0;
        if (j < A.n) {
            double d2 = 0.0;
            for (int c = 0; c < A.d; ++c) {
                const double e = A.q[(size_t)m * A.d + c] - A.u[(size_t)j * A.d + c];
                d2 = fma(e, e, d2);
            }
            k = A.amp * exp(-d2 * A.inv2l2);
        }
        A.ks[t] = k;
    }
}

typedef double v4d __attribute__((ext_vector_type(4)));

// Z block on the FP64 matrix cores: D[16 x 16] += A[16 x 4] B[4 x 16] per v_mfma_f64_16x16x4f64, with
// lane l holding A[l % 16][l / 16], B[l / 16][l % 16] and D[l / 16 + 4 v][l % 16] (v = 0..3).
// Wave w of the 4 takes queries m0 + 16 w .. + 15 and all 64 rows (4 row tiles of 16): A = X rows,
// B = K*^T, so D[i][m] = sum_j X[i][j] K*[m][j]. X and K* pass through LDS 16 columns at a time.
__global__ __launch_bounds__(256) void k_gp_zsq(GpEiArgs A) {
    __shared__ double Xs[kGpJ][kGpT + 1];  // X[i0 + r][j0 + c] at [c][r]
    __shared__ double Ks[kGpJ][kGpT + 1];  // K*[m0 + r][j0 + c] at [c][r]
    __shared__ double red[4][kGpT];
    const int i0 = blockIdx.x * kGpT, m0 = blockIdx.y * kGpT;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    v4d acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
    // X is lower triangular: row block [i0, i0 + 64) needs columns j < min(i0 + 64, n)
    const int jend = min(i0 + kGpT, A.n);
    for (int j0 = 0; j0 < jend; j0 += kGpJ) {
        for (int e = threadIdx.x; e < kGpT * kGpJ; e += blockDim.x) {
            const int r = e / kGpJ, c = e - r * kGpJ;
            const int i = i0 + r, m = m0 + r, j = j0 + c;
            Xs[c][r] = (i < A.n && j < A.n) ? A.linv[(size_t)i * A.n + j] : 0.0;
            Ks[c][r] = (m < A.M && j < A.npad) ? A.ks[(size_t)m * A.npad + j] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kGpJ; kk += 4) {
            const double b = Ks[kk + lk][16 * w + lr];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(Xs[kk + lk][16 * t + lr], b, acc[t], 0, 0, 0);
        }
        __syncthreads();
    }
    // this lane: query m0 + 16 w + lr, rows 16 t + lk + 4 v; sum of squares over its 16 rows
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) s = fma(acc[t][v], acc[t][v], s);
    red[lk][16 * w + lr] = s;
    __syncthreads();
    if (threadIdx.x < kGpT) {
        const double q = ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
        const int m = m0 + threadIdx.x;
        if (m < A.M) A.part[(size_t)blockIdx.x * A.M + m] = q;
    }
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Mean, deviation and EI of query m from a = k* . alpha and q = |X k*|^2.
__device__ __forceinline__ void gp_emit(const GpEiArgs &A, int m, double a, double q) {
    const double mu = A.m0 + A.s * a;
    const double var = A.amp - q;
    const double sd = A.s * sqrt(var > 0.0 ? var : 0.0);
    const double imp = A.best - mu - A.xi;
    double ei;
    if (sd > 0.0) {
        const double g = imp / sd;
        const double cdf = 0.5 * erfc(-g * 0.70710678118654752440);
        const double pdf = 0.39894228040143267794 * exp(-0.5 * g * g);
        // g Phi(g) + phi(g) > 0, but for g far below 0 its two terms cancel and rounding can leave a
        // tiny negative: EI, the mean of a non-negative improvement, is clamped at 0
        ei = sd * fma(g, cdf, pdf);
        if (!(ei > 0.0)) ei = 0.0;
    } else {
        ei = imp > 0.0 ? imp : 0.0;
    }
    if (A.mu) A.mu[m] = mu;
    if (A.sd) A.sd[m] = sd;
    A.ei[m] = ei;
}

__global__ __launch_bounds__(256) void k_gp_ei(GpEiArgs A) {
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= A.M) return;  // uniform per wave
    double a = 0.0;
    for (int j = lane; j < A.n; j += 64) a = fma(A.ks[(size_t)m * A.npad + j], A.alpha[j], a);
    a = wave_sum(a);
    double q = 0.0;
    for (int t = lane; t < A.nti; t += 64) q += A.part[(size_t)t * A.M + m];
    q = wave_sum(q);
    if (lane == 0) gp_emit(A, m, a, q);
}

// ------------------------------------------------------------------ fused acquisition
// X in operand order: the 16-row tile rt, 16-column chunk ch holds, for its 4 matrix steps s = 2 p + h
// (columns 16 ch + 4 s + l / 16 of row 16 rt + l % 16 in lane l), the doubles [p][lane][h]: a wave loads two
// steps of a tile with one 16-byte load per lane, 1 KB contiguous. Zero past n.
__global__ __launch_bounds__(256) void k_gp_pack(const double *__restrict__ linv, int n, int npad,
                                                 double *__restrict__ xp) {
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (t >= (size_t)npad * npad) return;
    const int h = t & 1, l = (t >> 1) & 63, p = (t >> 7) & 1;
    const int tile = (int)(t >> 8), nch = npad / 16;
    const int i = 16 * (tile / nch) + (l & 15), j = 16 * (tile % nch) + 4 * (2 * p + h) + (l >> 4);
    xp[t] = (i < n && j < n) ? linv[(size_t)i * n + j] : 0.0;
}

constexpr int kFuseQ = 16;          // queries per workgroup (one matrix tile)
constexpr int kFuseP = kFuseQ + 1;  // LDS row of K*: the odd pitch spreads a column's rows over the banks

// One workgroup (4 waves) per 16 queries: K* of the queries into LDS ([j][query]), Z = X K*^T by 64-row
// blocks on the FP64 matrix cores (X from L2 in operand order, 16 columns ahead in registers; a wave takes
// whole blocks, dealt back and forth so that the triangle's long rows spread evenly), the blocks' row
// sums of squares, then k* . alpha and EI. K* never goes to memory and X passes through no LDS. The sums run
// in k_gp_kstar's, k_gp_zsq's and k_gp_ei's order, so the values are theirs bit for bit. Bound by the
// matrix cores: a 16 x 16 x 4 FP64 step takes 64 cycles of a SIMD (246 us for 512 observations and 65536
// queries, which take 415 us; the three kernels took 1343). A local round of 4096 queries at 384
// observations takes 28 us (130 us as three EI kernels and three small ones).
// LOCAL: the queries are a round's points of the local search, formed here (GpLocalArgs): the centre moves
// to the first best point of its previous round, the points are set around it, the chains step.
// D: the number of dimensions where it is known (8, the head model's), so that an observation's coordinates
// are loaded together instead of one memory round trip each; 0: any.
template <bool LOCAL, int D>
__global__ __launch_bounds__(256, 2) void k_gp_fused(GpEiArgs A, GpLocalArgs L) {
    extern __shared__ double sm[];
    double *Ks = sm;                            // [npad][kFuseP]
    double *part = Ks + A.npad * kFuseP;        // [nti][kFuseQ]
    double *Qs = part + A.nti * kFuseQ;         // [kFuseQ][d]
    double *fin = Qs + kFuseQ * A.d;            // [2][kFuseQ]
    double *al = fin + 2 * kFuseQ;              // [npad] alpha
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m0 = blockIdx.x * kFuseQ, d = D ? D : A.d;
    if constexpr (LOCAL) {
        // 16 lanes per query
        const int hl = tid & 15, qi = tid >> 4, m = m0 + qi;
        if (m < A.M) {
            const int c = m / L.per;
            const double ce = L.Ce_src[c];
            double bv = -INFINITY;
            int bi = 0;
            if (L.e_prev) {
                const double *ep = L.e_prev + (size_t)c * L.per;
                for (int k0 = hl; k0 < L.per; k0 += 64) {
                    double v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = ep[min(k0 + 16 * i, L.per - 1)];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k0 + 16 * i < L.per && v[i] > bv) {
                            bv = v[i];
                            bi = k0 + 16 * i;
                        }
                }
#pragma unroll
                for (int off = 8; off > 0; off >>= 1) {
                    const double ov = __shfl_xor(bv, off);
                    const int oi = __shfl_xor(bi, off);
                    if (ov > bv || (ov == bv && oi < bi)) {
                        bv = ov;
                        bi = oi;
                    }
                }
            }
            const bool better = L.e_prev && bv > ce;
            const bool owner = L.C_dst && m == c * L.per;
            for (int k = hl; k < d; k += 16) {
                const double z = L.z[(size_t)m * d + k];
                const double base = better ? L.U_prev[((size_t)c * L.per + bi) * d + k] : L.C_src[(size_t)c * d + k];
                const double wz = 2.0 * z - 1.0;
                const double v = base + L.r * wz;
                const double lo = v > 0.0 ? v : 0.0;  // clip to [0, 1] as max then min, comparisons only
                const double u = lo < 1.0 ? lo : 1.0;
                Qs[qi * d + k] = u;
                L.U[(size_t)m * d + k] = u;
                L.z[(size_t)m * d + k] = (4.0 * z) * (1.0 - z);
                if (owner) L.C_dst[(size_t)c * d + k] = base;
            }
            if (owner && hl == 0) L.Ce_dst[c] = better ? bv : ce;
        } else {
            for (int k = hl; k < d; k += 16) Qs[qi * d + k] = 0.0;
        }
        // chains past the last centre's step too
        if (blockIdx.x == gridDim.x - 1)
            for (int t = A.M * d + tid; t < L.P * d; t += blockDim.x) {
                const double z = L.z[t];
                L.z[t] = (4.0 * z) * (1.0 - z);
            }
    } else {
        for (int t = tid; t < kFuseQ * d; t += blockDim.x) {
            const size_t o = (size_t)m0 * d + t;
            Qs[t] = o < (size_t)A.M * d ? A.q[o] : 0.0;
        }
    }
    __syncthreads();
    for (int j = tid; j < A.npad; j += blockDim.x) al[j] = j < A.n ? A.alpha[j] : 0.0;
    // K*: 4 queries of one observation per thread and step, the next observation's coordinates in flight
    constexpr int DU = D ? D : 1;
    double un[DU];
    auto fetch_u = [&](int j) {
        if constexpr (D > 0) {
            const double *uj = A.u + (size_t)min(j, A.n - 1) * D;
#pragma unroll
            for (int c = 0; c < D; ++c) un[c] = uj[c];
        }
    };
    fetch_u(tid >> 2);
    for (int e = tid; e < 4 * A.npad; e += blockDim.x) {
        const int j = e >> 2, q0 = 4 * (e & 3);
        double d2[4] = {0.0, 0.0, 0.0, 0.0};
        auto add = [&](int c, double u) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double t = Qs[(q0 + i) * d + c] - u;
                d2[i] = fma(t, t, d2[i]);
            }
        };
        if constexpr (D > 0) {
            double u[DU];
#pragma unroll
            for (int c = 0; c < D; ++c) u[c] = un[c];
            fetch_u((e + (int)blockDim.x) >> 2);
#pragma unroll
            for (int c = 0; c < D; ++c) add(c, u[c]);
        } else {
            const double *uj = A.u + (size_t)min(j, A.n - 1) * d;
            for (int c = 0; c < d; ++c) add(c, uj[c]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) Ks[j * kFuseP + q0 + i] = j < A.n ? A.amp * exp(-d2[i] * A.inv2l2) : 0.0;
    }
    __syncthreads();
    const int lr = lane & 15, lk = lane >> 4;
    const int nchunks = A.npad / 16;
    for (int r = 0; r < A.nti; ++r) {
        if (((r & 4) ? 3 - (r & 3) : (r & 3)) != w) continue;
        const int b = A.nti - 1 - r;
        const int nch = (min(64 * b + 64, A.n) + 15) / 16;
        const double2 *x[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            x[t] = reinterpret_cast<const double2 *>(A.xp) + (size_t)(4 * b + t) * nchunks * 128 + lane;
        v4d acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
        // two chunk buffers in turn: one is loaded while the other's 16 matrix steps run (the barrier keeps the
        // loads ahead of them); past the last chunk the loads repeat it, so that none sits in a branch
        double2 xa[4][2], xb[4][2];
        auto fetch = [&](double2(&v)[4][2], int ch) {
            const size_t o = (size_t)min(ch, nch - 1) * 128;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int p = 0; p < 2; ++p) v[t][p] = x[t][o + 64 * p];
            __builtin_amdgcn_sched_barrier(0);
        };
        auto multiply = [&](const double2(&v)[4][2], int ch) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double bq = Ks[(16 * ch + 4 * s + lk) * kFuseP + lr];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((s & 1) ? v[t][s >> 1].y : v[t][s >> 1].x, bq, acc[t],
                                                                  0, 0, 0);
            }
        };
        fetch(xa, 0);
        for (int ch = 0; ch < nch; ch += 2) {
            fetch(xb, ch + 1);
            multiply(xa, ch);
            if (ch + 1 < nch) {
                fetch(xa, ch + 2);
                multiply(xb, ch + 1);
            }
        }
        double s = 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) s = fma(acc[t][v], acc[t][v], s);
        const double s0 = __shfl(s, lr), s1 = __shfl(s, lr + 16), s2 = __shfl(s, lr + 32), s3 = __shfl(s, lr + 48);
        if (lane < 16) part[b * kFuseQ + lane] = ((s0 + s1) + s2) + s3;
    }
    __syncthreads();
    // the wave's 4 queries w, w + 4, ... side by side
    double a[4] = {0.0, 0.0, 0.0, 0.0}, q[4] = {0.0, 0.0, 0.0, 0.0};
    for (int j = lane; j < A.n; j += 64) {
        const double v = al[j];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = fma(Ks[j * kFuseP + w + 4 * i], v, a[i]);
    }
    for (int t = lane; t < A.nti; t += 64)
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] += part[t * kFuseQ + w + 4 * i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] += __shfl_xor(a[i], off);
            q[i] += __shfl_xor(q[i], off);
        }
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fin[w + 4 * i] = a[i];
            fin[kFuseQ + w + 4 * i] = q[i];
        }
    __syncthreads();
    if (tid < kFuseQ && m0 + tid < A.M) gp_emit(A, m0 + tid, fin[tid], fin[kFuseQ + tid]);
}

// ------------------------------------------------------------------ acquisition search, local stage
// (Bayesian Optimization, step 5: chaotic search). Per round: the query points of every centre's chains,
// U = clip(C_c + r (2 z - 1), 0, 1) in FP64 with the host search's operation order (no contraction), so
// the device search takes the same points as one run on the host; after the EI kernels, each centre
// moves to the first of its chains' best points when that beats its value; then z <- 4 z (1 - z).
__global__ __launch_bounds__(256) void k_chaos_points(const double *__restrict__ z, const double *__restrict__ C,
                                                      double r, int per, int d, int count, double *__restrict__ U) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;  // element of U [nc * per][d]; z rows match U rows
    if (t >= count) return;
    const int row = t / d, k = t - row * d;
    const double w = 2.0 * z[t] - 1.0;
    const double v = C[(row / per) * d + k] + r * w;
    const double m = v > 0.0 ? v : 0.0;  // clip to [0, 1] as max then min, comparisons only
    U[t] = m < 1.0 ? m : 1.0;
}

// The centres after a round: from (C_src, Ce_src) to (C, Ce), which may be the same buffers.
__global__ __launch_bounds__(256) void k_chaos_centres(const double *__restrict__ U, const double *__restrict__ e,
                                                       int per, int nc, int d, const double *C_src,
                                                       const double *Ce_src, double *C, double *Ce) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    const double *ec = e + (size_t)c * per;
    int j = 0;
    double best = ec[0];
    for (int k = 1; k < per; ++k)
        if (ec[k] > best) {
            best = ec[k];
            j = k;
        }
    const double ce = Ce_src[c];
    const bool better = best > ce;
    Ce[c] = better ? best : ce;
    for (int k = 0; k < d; ++k)
        C[(size_t)c * d + k] = better ? U[((size_t)c * per + j) * d + k] : C_src[(size_t)c * d + k];
}

__global__ __launch_bounds__(256) void k_chaos_step(double *__restrict__ z, int count) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const double v = z[t];
    z[t] = (4.0 * v) * (1.0 - v);
}

// The global stage's points: rounds [count] copies of the chains at z0, each a step on from the one before;
// z receives the chains after the last.
__global__ __launch_bounds__(256) void k_chaos_rounds(const double *__restrict__ z0, int count, int rounds,
                                                      double *__restrict__ pts, double *__restrict__ z) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    double v = z0[t];
    for (int r = 0; r < rounds; ++r) {
        pts[(size_t)r * count + t] = v;
        v = (4.0 * v) * (1.0 - v);
    }
    z[t] = v;
}

// ------------------------------------------------------------------ pools and greedy choice
// The order of the search's selections: larger value first, lower index on ties (as a stable sort in
// decreasing value). Values are taken to be finite.
__device__ __forceinline__ bool ranks_before(double va, int ia, double vb, int ib) {
    return va > vb || (va == vb && ia < ib);
}
// Unsigned key of the same order as the values (-0 as 0)
__device__ __forceinline__ unsigned long long rank_key(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v + 0.0);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// Exclusive prefix sum of v over the block's 1024 threads (thread order); total: the sum. scratch: 16 ints.
__device__ __forceinline__ int block_scan_1024(int v, int *scratch, int &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(inc, off);
        if (lane >= off) inc += o;
    }
    __syncthreads();
    if (lane == 63) scratch[wave] = inc;
    __syncthreads();
    int base = 0;
    total = 0;
    for (int i = 0; i < 16; ++i) {
        if (i < wave) base += scratch[i];
        total += scratch[i];
    }
    return base + inc - v;
}

// One workgroup per round: the `keep` highest-ranked of the round's M values, written in index order
// (values and their points) to the round's pool slot of min(M, keep) entries. M <= kPoolMax.
// A radix select, 8 bits of the key a pass, finds the keep-th rank; it ends as soon as the keys that share
// the prefix are all wanted. Each thread holds kPoolMax / 1024 consecutive values, so two prefix sums (the
// wanted ties, then all chosen) give index order. 16-23 us for 16-32 rounds of 4096 (125 us as a sort).
__global__ __launch_bounds__(1024) void k_pool_top(const double *__restrict__ pts, const double *__restrict__ vals,
                                                   int M, int d, int keep, double *__restrict__ pool_pts,
                                                   double *__restrict__ pool_vals) {
    constexpr int V = kPoolMax / 1024;
    __shared__ int hist[256];
    __shared__ int scratch[16];
    __shared__ int found[2];
    const int r = blockIdx.x, tid = threadIdx.x;
    const int kept = M < keep ? M : keep;
    const double *v = vals + (size_t)r * M;
    const double *p = pts + (size_t)r * M * d;
    double *ov = pool_vals + (size_t)r * kept;
    double *op = pool_pts + (size_t)r * kept * d;
    if (M <= keep) {
        for (int t = tid; t < M * d; t += blockDim.x) op[t] = p[t];
        for (int t = tid; t < M; t += blockDim.x) ov[t] = v[t];
        return;
    }
    const int per = (M + 1023) / 1024, first = tid * per;
    unsigned long long key[V];
    double val[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const bool in = i < per && first + i < M;
        val[i] = in ? v[first + i] : 0.0;
        key[i] = in ? rank_key(val[i]) : 0;  // 0 ranks below every finite value
    }
    // rank `need` (1-based) among the keys whose bits above `shift` equal prefix
    unsigned long long prefix = 0;
    int need = keep, shift = 64;
    while (shift > 0) {
        shift -= 8;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (i < per && first + i < M && (shift == 56 || (key[i] >> (shift + 8)) == prefix))
                atomicAdd(&hist[(int)((key[i] >> shift) & 255)], 1);
        __syncthreads();
        if (tid < 64) {
            // 4 bins a lane, the highest bins in lane 0: the bin that holds the rank
            int h[4], sum = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = hist[255 - (4 * tid + i)];
                sum += h[i];
            }
            int inc = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(inc, off);
                if (tid >= off) inc += o;
            }
            int above = inc - sum;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (above < need && need <= above + h[i]) {
                    found[0] = 255 - (4 * tid + i);
                    found[1] = above;
                }
                above += h[i];
            }
        }
        __syncthreads();
        const int bin = found[0];
        prefix = (prefix << 8) | (unsigned)bin;
        need -= found[1];
        if (hist[bin] == need) break;  // every key with this prefix is wanted
        __syncthreads();               // hist and found are read
    }
    int ties = 0;
#pragma unroll
    for (int i = 0; i < V; ++i)
        if (i < per && first + i < M && (key[i] >> shift) == prefix) ++ties;
    int total;
    int tie = block_scan_1024(ties, scratch, total);
    int chosen = 0;
    bool take[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const unsigned long long h = key[i] >> shift;
        take[i] = i < per && first + i < M && (h > prefix || (h == prefix && tie < need));
        if (i < per && first + i < M && h == prefix) ++tie;
        chosen += take[i] ? 1 : 0;
    }
    int pos = block_scan_1024(chosen, scratch, total);
#pragma unroll
    for (int i = 0; i < V; ++i)
        if (take[i]) {
            ov[pos] = val[i];
            const double *src = p + (size_t)(first + i) * d;
            double *dst = op + (size_t)pos * d;
            for (int k = 0; k < d; ++k) dst[k] = src[k];
            ++pos;
        }
}

// Squared distance of two d-vectors, in coordinate order. D: d where it is known (the loads then go out
// together), else 0.
template <int D>
__device__ __forceinline__ double dist2(const double *a, const double *b, int d) {
    double s = 0.0;
    if constexpr (D > 0) {
        double e[D];
#pragma unroll
        for (int k = 0; k < D; ++k) e[k] = a[k] - b[k];
#pragma unroll
        for (int k = 0; k < D; ++k) s += e[k] * e[k];
    } else {
        for (int k = 0; k < d; ++k) {
            const double e = a[k] - b[k];
            s += e * e;
        }
    }
    return s;
}

// alive[i] = 0 where entry i is nearer than sqrt(ex2) to a row of `taken`, else 1: four lanes per entry, a
// quarter of the rows each, over the whole GPU (24 us for 12288 entries and 384 rows; one workgroup, inside the
// greedy choice, took 8 ms).
template <int D>
__global__ __launch_bounds__(256) void k_screen(const double *__restrict__ pts, int N, int d,
                                                const double *__restrict__ taken, int T, double ex2,
                                                unsigned char *__restrict__ alive) {
    const int i = blockIdx.x * 64 + (threadIdx.x >> 2), part = threadIdx.x & 3;
    int near = 0;
    if (i < N)
        for (int t = part; t < T; t += 4) near |= dist2<D>(pts + (size_t)i * d, taken + (size_t)t * d, d) < ex2;
    near |= __shfl_xor(near, 1);
    near |= __shfl_xor(near, 2);
    if (i < N && part == 0) alive[i] = near ? 0 : 1;
}

// One workgroup: up to q pool entries in rank order, each at least sqrt(ex2) from the entries chosen before
// it (a greedy choice: the best remaining entry is chosen and every entry nearer than the exclusion to it is
// dropped), out of those alive (null: all). idx[0..count) receive the choices in order; *vmax the largest pool
// value. N <= 1024 E. Thread t holds the values of entries t, t + 1024, ... in registers with its own best
// one, renewed only when that one is dropped; the entries' first coordinates (two up to 16384 entries, one
// above: the LDS) are kept as floats, and a distance is formed only where they are near enough for it to
// matter (a margin covers their rounding). One barrier per choice. 64 choices out of 12288 entries take
// 345 us and out of 4096 entries 127 us (665 us with every entry's coordinates read for each choice).
template <int E, int D>
__global__ __launch_bounds__(1024) void k_greedy(const double *__restrict__ pts, const double *__restrict__ vals,
                                                 int N, int d, const unsigned char *__restrict__ live, int q,
                                                 double ex2, int *__restrict__ idx, int *__restrict__ count,
                                                 double *__restrict__ vmax) {
    constexpr int NF = E <= 16 ? 2 : 1;
    extern __shared__ float first[];  // [N][NF] first coordinates
    __shared__ double wv[2][16];
    __shared__ int wi[2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the root in doubles (ex2 may be below the floats), with a floor for coordinates that are
    const float reach = (float)sqrt(ex2) * 1.00001f + 1e-30f;
    double val[E];  // -infinity: dropped, or past the end
    unsigned alive = 0xffffffffu;
    double mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = tid + 1024 * e, ic = min(i, N - 1);
        const double v = vals[ic];
        const bool in = i < N;
        if (in)
#pragma unroll
            for (int k = 0; k < NF; ++k) first[i * NF + k] = (float)pts[(size_t)i * d + min(k, d - 1)];
        mx = in ? fmax(mx, v) : mx;
        val[e] = in && (!live || live[ic]) ? v : -INFINITY;
    }
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if (lane == 0) wv[1][wave] = mx;
    __syncthreads();
    if (tid == 0) {
        double m = wv[1][0];
        for (int w = 1; w < 16; ++w) m = fmax(m, wv[1][w]);
        *vmax = m;
    }
    int n = 0;
    bool renew = true;
    double own = -INFINITY;
    int own_i = 0x7fffffff;
    for (int it = 0; it < q; ++it) {
        if (renew) {
            own = -INFINITY;
            own_i = 0x7fffffff;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (val[e] > own) {  // ties keep the lower index
                    own = val[e];
                    own_i = tid + 1024 * e;
                }
            renew = false;
        }
        double bv = own;
        int bi = own_i;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double ov = __shfl_xor(bv, off);
            const int oi = __shfl_xor(bi, off);
            if (ranks_before(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
        }
        const int s = it & 1;
        if (lane == 0) {
            wv[s][wave] = bv;
            wi[s][wave] = bi;
        }
        __syncthreads();  // the other slot is written only after the next barrier's predecessors read this one
        bv = wv[s][lane & 15];
        bi = wi[s][lane & 15];
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) {
            const double ov = __shfl_xor(bv, off);
            const int oi = __shfl_xor(bi, off);
            if (ranks_before(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
        }
        if (bi == 0x7fffffff) break;
        if (tid == 0) idx[n] = bi;
        ++n;
        const double *pp = pts + (size_t)bi * d;
        float p[NF];
#pragma unroll
        for (int k = 0; k < NF; ++k) p[k] = first[bi * NF + k];
        unsigned close = 0;
#pragma unroll 4
        for (int e = 0; e < E; ++e) {
            bool far = false;
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                const float f = first[min(tid + 1024 * e, N - 1) * NF + k];
                far |= fabsf(f - p[k]) > reach + 1e-6f * (fabsf(f) + fabsf(p[k]));
            }
            if (!far) close |= 1u << e;
        }
        close &= alive;
        unsigned drop = 0;
        while (close) {
            const int e = __ffs(close) - 1;
            close &= close - 1;
            const int i = tid + 1024 * e;
            if (i < N && (i == bi || dist2<D>(pts + (size_t)i * d, pp, d) < ex2)) {
                drop |= 1u << e;
                renew |= i == own_i;
            }
        }
        alive &= ~drop;
        if (drop) {
#pragma unroll
            for (int e = 0; e < E; ++e) val[e] = (drop >> e & 1u) ? -INFINITY : val[e];
        }
    }
    if (tid == 0) *count = n;
}

// dst rows r = src rows idx[r] (r < *count, at most rows), and the matching values if vdst.
__global__ __launch_bounds__(256) void k_take_rows(const double *__restrict__ src, const double *__restrict__ vsrc,
                                                   const int *__restrict__ idx, const int *__restrict__ count,
                                                   int rows, int d, double *__restrict__ dst, double *__restrict__ vdst) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= rows * d) return;
    const int r = t / d, k = t - r * d;
    if (r >= *count) return;
    dst[t] = src[(size_t)idx[r] * d + k];
    if (vdst && k == 0) vdst[r] = vsrc[idx[r]];
}

hipError_t launch_pool_top(const double *pts, const double *vals, int rounds, int M, int d, int keep, double *pool_pts,
                           double *pool_vals, hipStream_t st) {
    if (M > kPoolMax || keep < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pool_top, dim3((unsigned)rounds), dim3(1024), 0, st, pts, vals, M, d, keep, pool_pts,
                       pool_vals);
    return hipGetLastError();
}

hipError_t launch_screen(const double *pts, int N, int d, const double *taken, int T, double ex2,
                         unsigned char *alive, hipStream_t st) {
    const dim3 grid((unsigned)((N + 63) / 64));
    if (d == 8)
        hipLaunchKernelGGL(k_screen<8>, grid, dim3(256), 0, st, pts, N, d, taken, T, ex2, alive);
    else
        hipLaunchKernelGGL(k_screen<0>, grid, dim3(256), 0, st, pts, N, d, taken, T, ex2, alive);
    return hipGetLastError();
}

template <int E>
static void greedy_go(const double *pts, const double *vals, int N, int d, const unsigned char *alive, int q, double ex2,
                      int *idx, int *count, double *vmax, hipStream_t st) {
    const size_t lds = sizeof(float) * (size_t)N * (E <= 16 ? 2 : 1);
    if (d == 8)
        hipLaunchKernelGGL((k_greedy<E, 8>), dim3(1), dim3(1024), lds, st, pts, vals, N, d, alive, q, ex2, idx, count,
                           vmax);
    else
        hipLaunchKernelGGL((k_greedy<E, 0>), dim3(1), dim3(1024), lds, st, pts, vals, N, d, alive, q, ex2, idx, count,
                           vmax);
}

hipError_t launch_greedy(const double *pts, const double *vals, int N, int d, const unsigned char *alive, int q,
                         double ex2, int *idx, int *count, double *vmax, hipStream_t st) {
    if (N < 1 || N > kGreedyMax) return hipErrorInvalidValue;
    if (N <= 4 * 1024)
        greedy_go<4>(pts, vals, N, d, alive, q, ex2, idx, count, vmax, st);
    else if (N <= 16 * 1024)
        greedy_go<16>(pts, vals, N, d, alive, q, ex2, idx, count, vmax, st);
    else
        greedy_go<32>(pts, vals, N, d, alive, q, ex2, idx, count, vmax, st);
    return hipGetLastError();
}

hipError_t launch_take_rows(const double *src, const double *vsrc, const int *idx, const int *count, int rows, int d,
                            double *dst, double *vdst, hipStream_t st) {
    const int n = rows * d;
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(k_take_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, vsrc, idx, count, rows,
                       d, dst, vdst);
    return hipGetLastError();
}

hipError_t launch_chaos_rounds(const double *z0, int count, int rounds, double *pts, double *z, hipStream_t st) {
    hipLaunchKernelGGL(k_chaos_rounds, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, z0, count, rounds, pts,
                       z);
    return hipGetLastError();
}

hipError_t launch_chaos_points(const double *z, const double *C, double r, int per, int nc, int d, double *U,
                               hipStream_t st) {
    const int count = per * nc * d;
    hipLaunchKernelGGL(k_chaos_points, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, z, C, r, per, d,
                       count, U);
    return hipGetLastError();
}

hipError_t launch_chaos_centres(const double *U, const double *e, int per, int nc, int d, const double *C_src,
                                const double *Ce_src, double *C, double *Ce, hipStream_t st) {
    hipLaunchKernelGGL(k_chaos_centres, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st, U, e, per, nc, d, C_src,
                       Ce_src, C, Ce);
    return hipGetLastError();
}

hipError_t launch_chaos_step(double *z, int count, hipStream_t st) {
    hipLaunchKernelGGL(k_chaos_step, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, z, count);
    return hipGetLastError();
}

static size_t fused_lds(const GpEiArgs &a) {
    return sizeof(double) * ((size_t)a.npad * kFuseP + (size_t)a.nti * kFuseQ + (size_t)kFuseQ * a.d + 2 * kFuseQ +
                             a.npad);
}

hipError_t launch_gp_pack(const GpEiArgs &a, double *xp, hipStream_t st) {
    const size_t count = (size_t)a.npad * a.npad;
    hipLaunchKernelGGL(k_gp_pack, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, a.linv, a.n, a.npad, xp);
    return hipGetLastError();
}

template <bool LOCAL>
static hipError_t fused_go(const GpEiArgs &a, const GpLocalArgs &l, hipStream_t st) {
    const dim3 grid((unsigned)((a.M + kFuseQ - 1) / kFuseQ));
    if (a.d == 8)
        hipLaunchKernelGGL((k_gp_fused<LOCAL, 8>), grid, dim3(256), fused_lds(a), st, a, l);
    else
        hipLaunchKernelGGL((k_gp_fused<LOCAL, 0>), grid, dim3(256), fused_lds(a), st, a, l);
    return hipGetLastError();
}

hipError_t launch_gp_local(const GpEiArgs &a, const GpLocalArgs &l, hipStream_t st) {
    if (!a.xp) return hipErrorInvalidValue;
    return fused_go<true>(a, l, st);
}

hipError_t launch_gp_ei(const GpEiArgs &a, hipStream_t st) {
    if (a.xp) return fused_go<false>(a, GpLocalArgs{}, st);
    size_t blocks = ((size_t)a.M * a.npad + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_gp_kstar, dim3((unsigned)blocks), dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gp_zsq, dim3((unsigned)a.nti, (unsigned)((a.M + kGpT - 1) / kGpT)), dim3(256), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gp_ei, dim3((unsigned)((a.M + 3) / 4)), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace boac
