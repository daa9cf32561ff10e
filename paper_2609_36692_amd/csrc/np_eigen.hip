// Dense symmetric eigensolver on the GPU, for the interaction matrix
// Gamma = Psi Psi^T of one active orientation (n = its order, up to a few
// thousand):
//   * Householder reduction to tridiagonal form (working matrix stored in
//     fp32, all arithmetic and the vectors in fp64): one launch per column
//     down to a trailing block of 256, which one workgroup reduces with the
//     block in registers;
//   * eigenvalues of the tridiagonal matrix by multisection on Sturm counts
//     (a wave per eigenvalue, any subset of indices);
//   * eigenvectors of the selected eigenvalues by inverse iteration with a
//     partially pivoted tridiagonal LU, Gram-Schmidt inside clusters of
//     close eigenvalues, and back-transformation through the reflectors in
//     blocks of 32 (compact WY form).
// Used by the exact variant of NormPre-L (App. B, exact eigenspace
// extraction: the leading eigenvectors of Gamma span the selected modes), by
// the Rayleigh-Ritz problems of the sketch (one workgroup each up to l = 80),
// and by the spectral diagnostics of the normalized and unnormalized Grams
// (App. A, spectral dynamics).  Matrices of one launch share n (grid y).
#include "np_internal.h"
#include "np_lanes.h"

#include <algorithm>
#include <cfloat>
#include <type_traits>

namespace np {
namespace {

constexpr int kVecThreads = 256;      // Gram-Schmidt

// Sum over the wave in a fixed order by DPP (row shifts, then the two row
// broadcasts): the total arrives in lane 63 and is read back as a scalar.
// Six steps of two moves and an add, against six pairs of LDS permutes for
// __shfl_xor.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_take(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Lane l's value, as a scalar.
__device__ __forceinline__ double lane_value(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double wave_sum_d(double v) {
    v += dpp_take<0x111, 0xf>(v);   // row_shr:1
    v += dpp_take<0x112, 0xf>(v);   // row_shr:2
    v += dpp_take<0x114, 0xf>(v);   // row_shr:4
    v += dpp_take<0x118, 0xf>(v);   // row_shr:8
    v += dpp_take<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_take<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return lane_value(v, 63);
}

// Exchange-and-add of two values: afterwards lanes with bit 5 (bit 4) clear
// hold a summed over that bit, the others b.
__device__ __forceinline__ double swap32_add(double a, double b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double swap16_add(double a, double b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
// The same over the lower lane bits by DPP (row_ror:8 flips bit 3;
// row_half_mirror bits 2, 1 and 0, of which the lower two are summed over
// afterwards; quad_perm bits 1 and 0).  A lane sends the value its partner keeps.
template <int CTRL>
__device__ __forceinline__ double swap_dpp_add(double a, double b, bool upper) {
    const double keep = upper ? b : a, send = upper ? a : b;
    return keep + dpp_take<CTRL, 0xf>(send);
}
__device__ __forceinline__ double sum_quad(double v) {
    v += dpp_take<0x4e, 0xf>(v);    // quad_perm [2,3,0,1]
    v += dpp_take<0xb1, 0xf>(v);    // quad_perm [1,0,3,2]
    return v;
}

// Workgroup barrier that orders LDS only: __syncthreads() also waits for the
// wave's outstanding global loads and stores.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kDppBit3 = 0x128, kDppBit2 = 0x141, kDppBit1 = 0x4e, kDppBit0 = 0xb1;

// N values per lane summed over the 32 lanes of each half wave (W = 32) or over
// the wave (W = 64): every exchange halves the values a lane carries.  Returns
// the sum of value `slot` to the lanes where lane_sum says so; of the lanes that
// share one, `first` is set in one, and never in a lane left with padding.
template <int BIT, int N>
__device__ __forceinline__ double halve_values(const double (&v)[N], int lane) {
    constexpr int H = (N + 1) / 2;
    const bool up = lane & BIT;
    if constexpr (BIT == 0) {
        return v[0];
    } else if constexpr (N == 1) {
        double r[1];
        if constexpr (BIT == 32) r[0] = swap32_add(v[0], v[0]);
        else if constexpr (BIT == 16) r[0] = swap16_add(v[0], v[0]);
        else r[0] = v[0] + dpp_take<BIT == 8 ? kDppBit3 : BIT == 4 ? kDppBit2 : BIT == 2 ? kDppBit1 : kDppBit0, 0xf>(v[0]);
        return halve_values<BIT / 2, 1>(r, lane);
    } else {
        double r[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const double a = v[i], b = i + H < N ? v[i + H < N ? i + H : i] : 0.0;
            if constexpr (BIT == 32) r[i] = swap32_add(a, b);
            else if constexpr (BIT == 16) r[i] = swap16_add(a, b);
            else r[i] = swap_dpp_add<BIT == 8 ? kDppBit3 : BIT == 4 ? kDppBit2 : BIT == 2 ? kDppBit1 : kDppBit0>(a, b, up);
        }
        return halve_values<BIT / 2, H>(r, lane);
    }
}
template <int W, int N>
__device__ __forceinline__ double sum_values(const double (&v)[N], int lane, int& slot, bool& first) {
    static_assert(N <= W && lane_sum_complete(W, N), "every value stored by one lane");
    const LaneSum o = lane_sum(W, N, lane & (W - 1));
    slot = o.slot;
    first = o.first;
    return halve_values<W / 2, N>(v, lane);
}

// Sum over the block in a fixed order (every thread returns the same value).
template <int NT>
__device__ double block_sum_d(double v, double* red) {
    v = wave_sum_d(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) t += red[i];
    return t;
}

// Gamma fp32 (GEMM output, ld ldg) -> symmetrized n x n (ld n).
__global__ void gamma_sym_kernel(const float* g, int64_t ldg, int64_t strideg, int n, float* A,
                                 int64_t strideA) {
    const int z = blockIdx.y;
    const float* gz = g + (int64_t)z * strideg;
    float* Az = A + (int64_t)z * strideA;
    const int64_t nn = (int64_t)n * n;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < nn; idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx / n, k = idx - i * n;
        Az[idx] = (float)(0.5 * ((double)gz[i * ldg + k] + (double)gz[k * ldg + i]));
    }
}

// fp64 reciprocal and reciprocal square root: the hardware estimates refined
// by two Newton steps, a shorter chain than the IEEE division and root.
__device__ __forceinline__ double recip(double q) {
    double r = __builtin_amdgcn_rcp(q);
    r = fma(r, fma(-q, r, 1.0), r);
    return fma(r, fma(-q, r, 1.0), r);
}
__device__ __forceinline__ double rsqrt_d(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// Reflector of a column with leading entry alpha and squared norm sig of the
// entries below it: H = I - t v v^T, v = (1, col * scal), H col = beta e_1.
struct Reflector {
    double beta, t, scal;
};
__device__ __forceinline__ Reflector reflector(double alpha, double sig) {
    Reflector r{alpha, 0.0, 0.0};
    if (sig > 0.0) {
        const double q = fma(alpha, alpha, sig), rn = rsqrt_d(q);
        // Squares too small to carry a full reciprocal root (entries below
        // 1e-150): no reflection, a change far below the matrix's rounding.
        if (q > 1e-300) {
            r.beta = -copysign(q * rn, alpha);
            r.t = fma(fabs(alpha), rn, 1.0);        // (beta - alpha) / beta
            r.scal = recip(alpha - r.beta);
        }
    }
    return r;
}

// Column j of the reduction in one launch.  vec holds per matrix
// [v (2 ping-pong slots) | p (2 slots)], n doubles each: slot j & 1 of v and p
// belongs to step j.
// Every block forms the same reflector v_j from row j of A (rows are only
// updated through step j - 2, so step j - 1's rank-2 term v w^T + w v^T,
// w = p - (tau/2)(p^T v) v, is subtracted on the fly), then updates its own
// rows i > j with step j - 1's term and forms p_j[i] = tau_j A(i, :) v_j from
// the updated row.  The forming is O(n) and repeated per block, which costs
// less than a launch of its own (a one-block kernel for it and a second
// launch took 6.4 of the 21 us per column of an order-2048 matrix).
// A thread owns the columns c0 + tid + NT u of every row of its block, so the
// vectors stay in its registers for all of them, and the first RB rows are
// requested before the reflector is formed.  Row i always belongs to block
// i mod nb, nb a multiple of 8: with the round-robin dispatch over the 8 XCDs
// a row meets the same L2 in every launch (16 MB, order 2048, fit the eight
// L2s).  Bound by the latency of one launch (load, two block sums, row pass,
// store) down to about order 1000 and by the read and write of the trailing
// rows above it: order 2048, 9.2 us per column while 1024 or more are left, 7.1
// and 5.3 us for the next 512 and 256 (14.4 ms in all, 38.5 ms before).
// Block 0 keeps v_j, and writes v_{j-1} into row j - 1 of A for the
// back-transformation (no block reads that row any more).
template <int NT, int U, int RB>
__global__ void __launch_bounds__(NT) tri_step_kernel(float* A, int64_t strideA, int n, int j, int c0, double* vec,
                                                      int64_t stride_vec, double* dd, double* ee, double* tau,
                                                      int64_t stride_n) {
    constexpr int NW = NT / 64;
    __shared__ double red1[NW], red2[NW], redp[2][NW][RB];
    const int z = blockIdx.y, nb = gridDim.x, x = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool first = j == 0;
    float* Az = A + (int64_t)z * strideA;
    double* V = vec + (int64_t)z * stride_vec;
    const double* __restrict__ vprev = V + (int64_t)((j + 1) & 1) * n;
    double* vcur = V + (int64_t)(j & 1) * n;
    const double* __restrict__ pprev = V + (int64_t)(2 + ((j + 1) & 1)) * n;
    double* pcur = V + (int64_t)(2 + (j & 1)) * n;
    const float* row = Az + (int64_t)j * n;
    const int i0 = j + 1 + (x + nb - (j + 1) % nb) % nb;   // first row > j of this block
    float tile[RB][U];
    double arow[U], vp[U], w[U], v[U];
    auto load_tile = [&](int i) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int ir = i + r * nb;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = c0 + tid + NT * u;
                tile[r][u] = ir < n && k > j && k < n ? Az[(int64_t)ir * n + k] : 0.f;
            }
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = c0 + tid + NT * u;
        const bool in = k >= j && k < n;
        arow[u] = in ? (double)row[k] : 0.0;
        vp[u] = in && !first ? vprev[k] : 0.0;
        w[u] = in && !first ? pprev[k] : 0.0;       // p_{j-1} for now
    }
    double djj = row[j], alpha = row[j + 1];
    const double pj = first ? 0.0 : pprev[j], pj1 = first ? 0.0 : pprev[j + 1], vj1 = first ? 0.0 : vprev[j + 1];
    const double tp = first ? 0.0 : tau[(int64_t)z * stride_n + j - 1];
    load_tile(i0);
    // v_{j-1} and p_{j-1} of the pass's rows, row r in lane r.
    double vl = 0.0, pl = 0.0;
    auto load_scalars = [&](int i) {
        const int ir = i + (lane % RB) * nb;
        vl = !first && ir < n ? vprev[ir] : 0.0;
        pl = !first && ir < n ? pprev[ir] : 0.0;
    };
    load_scalars(i0);
    double K = 0.0;
    if (!first) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) s += w[u] * vp[u];
        s = wave_sum_d(s);
        if (lane == 0) red1[wave] = s;
        lds_barrier();
        s = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) s += red1[q];
        K = 0.5 * tp * s;
        const double wj = pj - K;                   // v_{j-1}[j] = 1
#pragma unroll
        for (int u = 0; u < U; ++u) {
            w[u] -= K * vp[u];
            arow[u] -= vp[u] * wj + w[u];
        }
        djj -= 2.0 * wj;
        alpha -= vj1 * wj + (pj1 - K * vj1);
    }
    double sig = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (c0 + tid + NT * u >= j + 2) sig += arow[u] * arow[u];
    sig = wave_sum_d(sig);
    if (lane == 0) red2[wave] = sig;
    lds_barrier();
    sig = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) sig += red2[q];
    const Reflector h = reflector(alpha, sig);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = c0 + tid + NT * u;
        v[u] = k <= j ? 0.0 : (k == j + 1 ? 1.0 : arow[u] * h.scal);
    }
    if (x == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = c0 + tid + NT * u;
            if (k < n) {
                vcur[k] = v[u];
                if (!first && k >= j) Az[(int64_t)(j - 1) * n + k] = (float)vp[u];
            }
        }
        if (tid == 0) {
            dd[(int64_t)z * stride_n + j] = djj;
            ee[(int64_t)z * stride_n + j] = h.beta;
            tau[(int64_t)z * stride_n + j] = h.t;
        }
    }
    int par = 0;
    for (int i = i0; i < n; i += RB * nb, par ^= 1) {
        double dot[RB];
        const double wl = pl - K * vl;
#pragma unroll
        for (int r = 0; r < RB; ++r) dot[r] = 0.0;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int ir = i + r * nb;
            if (ir >= n) break;
            const double vi = lane_value(vl, r), wi = lane_value(wl, r);
            float* Ar = Az + (int64_t)ir * n;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = c0 + tid + NT * u;
                const double a = (double)tile[r][u] - (vi * w[u] + wi * vp[u]);
                if (!first && k > j && k < n) Ar[k] = (float)a;
                dot[r] += a * v[u];
            }
        }
        if (i + RB * nb < n) {
            load_tile(i + RB * nb);
            load_scalars(i + RB * nb);
        }
        int rs;
        bool first_lane;
        const double d = sum_values<64>(dot, lane, rs, first_lane);
        if (first_lane) redp[par][wave][rs] = d;
        lds_barrier();
        if (tid < RB) {
            double s = 0.0;
#pragma unroll
            for (int q2 = 0; q2 < NW; ++q2) s += redp[par][q2][tid];
            const int ir = i + tid * nb;
            if (ir < n) pcur[ir] = h.t * s;
        }
    }
}

// Householder tridiagonalization of the trailing m x m block (m = n - j0 <=
// kTriRegMax) of one matrix per workgroup, the block in registers: thread
// (wave w, lane) holds the rows 16 s + 2 w + (lane >> 5), s < 16, and the columns
// 32 c + (lane & 31), c < 8, in fp32 (all arithmetic fp64).  Per column: the
// wave that owns row jj (= column jj) forms the reflector from its own
// registers; p = tau M v as up to sixteen dots per thread, summed over the 32
// column lanes by halving exchanges; w = p - (tau/2)(p^T v) v; then the rank-2 update
// in registers.  Two barriers per column (v and p alternate between two LDS
// buffers).  The column loop is unrolled over the 16-row slots, so finished
// rows and columns drop out at compile time.  2.4 us per column, fp64 issue and
// the chain of the reflector about equal (with the block in LDS, up to 192
// columns, the same reduction took 8.4 us per column).
// With j0 > 0 the per-column launches have done columns 0 .. j0 - 1 and left
// the rank-2 update of column j0 - 1 pending (its reflector and p = tau A v in
// `vec`): the block is loaded with that update applied.
constexpr int kTriRegMax = 256;
constexpr int kTriWaves = 8, kTriThreads = 64 * kTriWaves, kTriSlots = kTriRegMax / (2 * kTriWaves);

template <int C>
struct TriRegShared {
    double v[2][32 * C], p[2][32 * C], t[2];
};

// The columns of the row slots S, S + 1, ... of an m x m block held by NW waves:
// slot s of thread (wave, half wave) is row 2 NW s + 2 wave + half, its column c
// of 32 the column 32 c + (lane & 31).  dd, ee, tau and Ag (where the
// reflectors go, row stride n) start at the block's first column.
template <int NW, int R, int C, int S>
__device__ __forceinline__ void tri_reg_cols(float (&M)[R][C], TriRegShared<C>& sh, int& par, int m, float* Ag, int n,
                                             double* dd, double* ee, double* tau) {
    constexpr int RS = 2 * NW, C0 = RS * S / 32;     // rows per slot, first live column block
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, cl = lane & 31;
    for (int jr = 0; jr < RS; ++jr, par ^= 1) {
        const int jj = RS * S + jr;
        if (jj >= m) break;
        if (wave == jr >> 1) {
            // Row jj (= column jj) sits in one half of this wave.
            const bool mine = half == (jr & 1);
            double x[C], sig = 0.0;
#pragma unroll
            for (int c = C0; c < C; ++c) {
                x[c] = M[S][c];
                if (32 * c + cl >= jj + 2) sig += x[c] * x[c];
            }
            sig = wave_sum_d(mine ? sig : 0.0);
            const int l0 = (jr & 1) << 5;
            const double dj = lane_value(x[C0], l0 | (jj & 31));
            const double alpha = (jj & 31) < 31 ? lane_value(x[C0], l0 | ((jj + 1) & 31))
                                 : C0 + 1 < C   ? lane_value(x[C0 + 1 < C ? C0 + 1 : C0], l0)
                                                : 0.0;
            const Reflector h = reflector(alpha, sig);
#pragma unroll
            for (int c = C0; c < C; ++c) {
                const int k = 32 * c + cl;
                const double vk = k <= jj ? 0.0 : (k == jj + 1 ? 1.0 : x[c] * h.scal);
                if (mine) {
                    sh.v[par][k] = vk;
                    if (k > jj && k < m) Ag[(int64_t)jj * n + k] = (float)vk;
                }
            }
            if (lane == 0) {
                sh.t[par] = h.t;
                dd[jj] = dj;
                ee[jj] = h.beta;
                tau[jj] = h.t;
            }
        }
        lds_barrier();
        const double t = sh.t[par];
        if (t == 0.0) continue;   // H = I (uniform across the block)
        {
            double vc[C], dot[R - S];
#pragma unroll
            for (int c = C0; c < C; ++c) vc[c] = sh.v[par][32 * c + cl];
#pragma unroll
            for (int s = S; s < R; ++s) {
                dot[s - S] = 0.0;
#pragma unroll
                for (int c = C0; c < C; ++c) dot[s - S] += (double)M[s][c] * vc[c];
                __builtin_amdgcn_sched_barrier(0);      // register pressure
            }
            int slot;
            bool first;
            const double d = sum_values<32>(dot, lane, slot, first);
            const int i = RS * (S + slot) + 2 * wave + half;
            if (first && i < 32 * C) sh.p[par][i] = i > jj ? t * d : 0.0;
        }
        // The fp64 copies of M are made anew below: kept across the barrier
        // (the compiler's choice) they would not fit the registers.
#pragma unroll
        for (int s = S; s < R; ++s)
#pragma unroll
            for (int c = C0; c < C; ++c) asm volatile("" : "+v"(M[s][c]));
        lds_barrier();
        double vc[C], wc[C], pv = 0.0;
#pragma unroll
        for (int c = C0; c < C; ++c) {
            const int k = 32 * c + cl;
            vc[c] = sh.v[par][k];
            // Only the live slots' rows were written this time; v is zero elsewhere.
            wc[c] = k >= RS * S && k < RS * R ? sh.p[par][k] : 0.0;
            pv += wc[c] * vc[c];
        }
        const double K = 0.5 * t * wave_sum_d(half ? 0.0 : pv);
#pragma unroll
        for (int c = C0; c < C; ++c) wc[c] -= K * vc[c];
#pragma unroll
        for (int s = S; s < R; ++s) {
            const int i = RS * s + 2 * wave + half;
            const double vi = sh.v[par][i], wi = sh.p[par][i] - K * vi;
#pragma unroll
            for (int c = C0; c < C; ++c) M[s][c] = (float)((double)M[s][c] - vi * wc[c] - wi * vc[c]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (S + 1 < R) tri_reg_cols<NW, R, C, S + 1>(M, sh, par, m, Ag, n, dd, ee, tau);
}

__global__ void __launch_bounds__(kTriThreads) tri_reg_kernel(float* A, int64_t strideA, int n, int j0,
                                                              const double* vec, int64_t stride_vec, double* dd,
                                                              double* ee, double* tau, int64_t stride_n) {
    __shared__ TriRegShared<8> sh;
    __shared__ double red[kTriThreads / 64];
    const int z = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, cl = lane & 31;
    const int m = n - j0;
    float* Ag = A + (int64_t)z * strideA;
    float M[kTriSlots][8];
#pragma unroll
    for (int s = 0; s < kTriSlots; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int i = 2 * kTriWaves * s + 2 * wave + half, k = 32 * c + cl;
            M[s][c] = i < m && k < m ? Ag[(int64_t)(j0 + i) * n + j0 + k] : 0.f;
        }
    if (j0 > 0) {
        const double* V = vec + (int64_t)z * stride_vec;
        const double* vp = V + (int64_t)((j0 - 1) & 1) * n;
        const double* P = V + (int64_t)(2 + ((j0 - 1) & 1)) * n;
        const double tp = tau[(int64_t)z * stride_n + j0 - 1];
        double vt = 0.0, pt = 0.0;
        if (tid < m) {
            vt = vp[j0 + tid];
            pt = P[j0 + tid];
            Ag[(int64_t)(j0 - 1) * n + j0 + tid] = (float)vt;
        }
        const double K = 0.5 * tp * block_sum_d<kTriThreads>(vt * pt, red);
        if (tid < kTriRegMax) {
            sh.v[0][tid] = vt;
            sh.p[0][tid] = pt - K * vt;
        }
        __syncthreads();
        double vc[8], wc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            vc[c] = sh.v[0][32 * c + cl];
            wc[c] = sh.p[0][32 * c + cl];
        }
#pragma unroll
        for (int s = 0; s < kTriSlots; ++s) {
            const int i = 2 * kTriWaves * s + 2 * wave + half;
            const double vi = sh.v[0][i], wi = sh.p[0][i];
#pragma unroll
            for (int c = 0; c < 8; ++c) M[s][c] = (float)((double)M[s][c] - vi * wc[c] - wi * vc[c]);
        }
        __syncthreads();
    }
    int par = 0;
    float* Ab = Ag + (int64_t)j0 * n + j0;
    double* db = dd + (int64_t)z * stride_n + j0;
    double* eb = ee + (int64_t)z * stride_n + j0;
    double* ub = tau + (int64_t)z * stride_n + j0;
    tri_reg_cols<kTriWaves, kTriSlots, 8, 0>(M, sh, par, m, Ab, n, db, eb, ub);
}

// Eigenvalues by multisection, one wave per eigenvalue ((first + t)-th largest
// for wave t): each round the 64 lanes count the eigenvalues below 64 interior
// points of the bracket, which shrinks 65x.  The count is the number of sign
// changes of the leading principal minors of T - x I,
//   p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1},
// whose dependent chain is one FMA per step (the LDL^T pivots' form needs a
// reciprocal); the pair is rescaled by a power of two every kSturmRun steps.
// T is scaled by a power of two to norm at most 1, and every e^2 is raised to at
// least 2^-200 (a perturbation of at most 2^-99, far below the rounding of T),
// so neither overflow nor a vanishing pair can occur between rescalings.  The
// scaled (d, e^2) pairs are staged in LDS once per block.  Stops at a width of
// 2 eps max(|lo|, |hi|) + 2^-70 (of the scaled T).  All 2048
// eigenvalues of order 2048 take 0.75 ms (16 lanes per eigenvalue and pivots
// with a reciprocal: 1.89 ms).
constexpr int kBisectWaves = 4;
constexpr int kSturmRun = 8;

// Sign changes at the P points x of the scaled matrix de = (d_i, e_{i-1}^2),
// padded to np8.  The signs of a run are collected one bit per step.
template <int P>
__device__ __forceinline__ void sturm_changes(const double2* de, int np8, const double (&x)[P], int (&changes)[P]) {
    double p[P], pp[P];
    unsigned sg[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        p[k] = 1.0;
        pp[k] = 0.0;
        sg[k] = 0;
        changes[k] = 0;
    }
    static_assert(kSturmRun < 32, "sign bits of a run and its start");
    for (int i = 0; i < np8; i += kSturmRun) {
        double2 v[kSturmRun];
#pragma unroll
        for (int q = 0; q < kSturmRun; ++q) v[q] = de[i + q];
#pragma unroll
        for (int q = 0; q < kSturmRun; ++q)
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double pn = fma(v[q].x - x[k], p[k], -v[q].y * pp[k]);
                sg[k] = __builtin_amdgcn_alignbit(sg[k], (unsigned)__double2hiint(pn), 31);    // sg << 1 | sign
                pp[k] = p[k];
                p[k] = pn;
            }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            changes[k] += __popc((sg[k] ^ sg[k] >> 1) & ((1u << kSturmRun) - 1));
            const int sc = -__builtin_amdgcn_frexp_exp(fmax(fabs(p[k]), fabs(pp[k])));
            p[k] = ldexp(p[k], sc);
            pp[k] = ldexp(pp[k], sc);
        }
    }
}
// Entry i of de for the matrix scaled by 2^-ex.  Past the end: d = 4 > x and no
// coupling, which adds no sign change.
__device__ __forceinline__ double2 sturm_entry(const double* d, const double* e, int n, int i, int ex) {
    const double es = i > 0 && i < n ? ldexp(e[i - 1], -ex) : 0.0;
    return make_double2(i < n ? ldexp(d[i], -ex) : 4.0, i < n ? fmax(es * es, 0x1p-200) : 0.0);
}
// The (idx + 1)-th smallest eigenvalue by the L lanes of a group (`sub` in it,
// first lane `base`), P points each (lane s takes the points s + 1 + L k),
// starting from the scaled bracket [lo, hi].
template <int L, int P>
__device__ __forceinline__ double multisect(const double2* de, int np8, int idx, double lo, double hi, int sub,
                                            int base) {
    constexpr int N = L * P;
    for (int it = 0; it < 100; ++it) {
        const double w = hi - lo;
        if (w <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi)) + 0x1p-70) break;
        auto pt = [&](int k) { return lo + (w * (double)k) * (1.0 / (N + 1)); };
        double x[P];
        int c[P];
#pragma unroll
        for (int k = 0; k < P; ++k) x[k] = pt(sub + 1 + L * k);
        sturm_changes<P>(de, np8, x, c);
        // First point whose count exceeds idx (N: none does).
        int s = N;
#pragma unroll
        for (int k = P - 1; k >= 0; --k) {
            const unsigned long long mask = __ballot(c[k] > idx) >> base & (L == 64 ? ~0ull : (1ull << (L & 63)) - 1);
            if (mask) s = L * k + __builtin_ctzll(mask);
        }
        const double nlo = s > 0 ? pt(s) : lo;
        const double nhi = s < N ? pt(s + 1) : hi;
        if (!(nlo > lo) && !(nhi < hi)) break;
        lo = nlo;
        hi = nhi;
    }
    return 0.5 * (lo + hi);
}

__global__ void __launch_bounds__(64 * kBisectWaves) tri_bisect_kernel(const double* dd, const double* ee,
                                                                       int64_t stride_n, int n, int first, int nvals,
                                                                       double* out, int64_t stride_out) {
    extern __shared__ double2 de[];     // (d_i, e_{i-1}^2), scaled; padded to a multiple of kSturmRun
    __shared__ double rlo[kBisectWaves], rhi[kBisectWaves];
    const int z = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double* d = dd + (int64_t)z * stride_n;
    const double* e = ee + (int64_t)z * stride_n;
    // Gershgorin interval.
    double lo = DBL_MAX, hi = -DBL_MAX;
    for (int i = tid; i < n; i += 64 * kBisectWaves) {
        const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0);
        lo = fmin(lo, d[i] - r);
        hi = fmax(hi, d[i] + r);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, 64));
        hi = fmax(hi, __shfl_xor(hi, o, 64));
    }
    if (lane == 0) {
        rlo[wave] = lo;
        rhi[wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kBisectWaves; ++q) {
        lo = fmin(lo, rlo[q]);
        hi = fmax(hi, rhi[q]);
    }
    const double span = fmax(fabs(lo), fabs(hi));
    const int t = blockIdx.x * kBisectWaves + wave;
    if (!(span > 0.0)) {                // T = 0 (fmin and fmax drop NaN: an all-NaN T ends at 0 below)
        if (t < nvals && lane == 0) out[(int64_t)z * stride_out + t] = span;
        return;
    }
    int ex;
    (void)frexp(span, &ex);             // span = f 2^ex, f in [1/2, 1)
    const int np8 = (n + kSturmRun - 1) / kSturmRun * kSturmRun;
    for (int i = tid; i < np8; i += 64 * kBisectWaves) de[i] = sturm_entry(d, e, n, i, ex);
    __syncthreads();
    if (t >= nvals) return;
    lo = ldexp(lo, -ex) - 2.0 * DBL_EPSILON;
    hi = ldexp(hi, -ex) + 2.0 * DBL_EPSILON;
    // smallest x with count(x) > idx, idx counted from the bottom
    const double x = multisect<64, 1>(de, np8, n - 1 - (first + t), lo, hi, lane, 0);
    if (lane == 0) out[(int64_t)z * stride_out + t] = ldexp(x, ex);
}

// Inverse iteration with the factors in LDS: the partially pivoted LU of
// T - lambda I and its solves for one eigenvalue per lane.  Row i of the factors
// (f: multiplier, r: 1 / pivot, m: first superdiagonal, sw: rows swapped; the
// second superdiagonal is e_{i+1} where they were) is entry i st of each array,
// the working vector entry i ys of y; de = (d_i, e_i).
constexpr int kInvRun = 8;
struct InvLds {
    const double2* de;
    double *f, *r, *m;
    unsigned char* sw;
    double* y;
    int st, ys;
};

// Factorization and the first solve's forward sweep in one pass; the start
// vector is the fixed pseudo-random sequence of eigenvalue k when init, else y.
// Returns the running entry after the sweep.
__device__ __forceinline__ double inv_factor(const InvLds& a, int n, double lk, double floor_piv, int k, bool init) {
    auto floored = [&](double g) { return fabs(g) < floor_piv ? (g < 0.0 ? -floor_piv : floor_piv) : g; };
    uint32_t h = 0x9e3779b9u * (uint32_t)(k + 1);
    auto draw = [&]() {     // in [-1, 1], distinct per k
        h ^= h << 13; h ^= h >> 17; h ^= h << 5;
        return ((double)(h >> 8) * (1.0 / 8388608.0)) - 1.0;
    };
    // g, u: the current diagonal and superdiagonal entries of row i (row i + 1
    // of the matrix is still untouched when step i starts); c: the running
    // entry of the P L solve.
    double g = a.de[0].x - lk, u = a.de[0].y, c = init ? draw() : a.y[0];
    auto step = [&](int i, double l, double dn, double un, double nx) {
        const int o = i * a.st;
        const double gn = dn - lk;
        const bool keep = fabs(g) >= fabs(l);
        const double r = recip(floored(keep ? g : l));
        const double f = (keep ? l : g) * r, m = keep ? u : gn;
        a.f[o] = f;
        a.r[o] = r;
        a.m[o] = m;
        a.sw[o] = !keep;
        g = (keep ? gn : u) - f * m;
        u = keep ? un : -f * un;
        const double top = keep ? c : nx;
        a.y[i * a.ys] = top;
        c = (keep ? nx : c) - f * top;
    };
    int i0 = 0;
    for (; i0 + kInvRun < n; i0 += kInvRun) {
        double2 w[kInvRun + 1];
        double nx[kInvRun];
#pragma unroll
        for (int q = 0; q <= kInvRun; ++q) w[q] = a.de[i0 + q];
#pragma unroll
        for (int q = 0; q < kInvRun; ++q) nx[q] = init ? draw() : a.y[(i0 + q + 1) * a.ys];
#pragma unroll
        for (int q = 0; q < kInvRun; ++q) step(i0 + q, w[q].y, w[q + 1].x, w[q + 1].y, nx[q]);
    }
    for (; i0 + 1 < n; ++i0)
        step(i0, a.de[i0].y, a.de[i0 + 1].x, a.de[i0 + 1].y, init ? draw() : a.y[(i0 + 1) * a.ys]);
    a.r[(n - 1) * a.st] = recip(floored(g));
    return c;
}

// Forward sweep (P L) of y scaled by `scale`; returns the running entry.
__device__ __forceinline__ double inv_forward(const InvLds& a, int n, double scale) {
    double c = a.y[0] * scale;
    auto step = [&](int i, double nx, double f, bool swap) {
        const double top = swap ? nx : c;
        a.y[i * a.ys] = top;
        c = (swap ? c : nx) - f * top;
    };
    int i0 = 0;
    for (; i0 + kInvRun < n; i0 += kInvRun) {
        double nx[kInvRun], fl[kInvRun];
        int pf[kInvRun];
#pragma unroll
        for (int q = 0; q < kInvRun; ++q) {
            nx[q] = a.y[(i0 + q + 1) * a.ys] * scale;
            fl[q] = a.f[(i0 + q) * a.st];
            pf[q] = a.sw[(i0 + q) * a.st];
        }
#pragma unroll
        for (int q = 0; q < kInvRun; ++q) step(i0 + q, nx[q], fl[q], pf[q]);
    }
    for (; i0 + 1 < n; ++i0) step(i0, a.y[(i0 + 1) * a.ys] * scale, a.f[i0 * a.st], a.sw[i0 * a.st]);
    return c;
}

// Backward sweep from the running entry c; returns 1 / max |y_i| (1 for y = 0).
__device__ __forceinline__ double inv_backward(const InvLds& a, int n, double c) {
    double y1 = c * a.r[(n - 1) * a.st], y2 = 0.0, mx = fabs(y1);
    a.y[(n - 1) * a.ys] = y1;
    auto step = [&](int i, double yv, double m, double e1, double r) {
        const double y0 = (yv - e1 * y2 - m * y1) * r;
        a.y[i * a.ys] = y0;
        mx = fmax(mx, fabs(y0));
        y2 = y1;
        y1 = y0;
    };
    int i0 = n - 2;
    for (; i0 >= kInvRun - 1; i0 -= kInvRun) {
        double yv[kInvRun], m[kInvRun], e1[kInvRun], r[kInvRun];
#pragma unroll
        for (int q = 0; q < kInvRun; ++q) {
            const int i = i0 - q, o = i * a.st;
            yv[q] = a.y[i * a.ys];
            m[q] = a.m[o];
            r[q] = a.r[o];
            const double ev = a.de[i + 1].y;
            e1[q] = a.sw[o] ? ev : 0.0;
        }
#pragma unroll
        for (int q = 0; q < kInvRun; ++q) step(i0 - q, yv[q], m[q], e1[q], r[q]);
    }
    for (; i0 >= 0; --i0)
        step(i0, a.y[i0 * a.ys], a.m[i0 * a.st], a.sw[i0 * a.st] ? a.de[i0 + 1].y : 0.0, a.r[i0 * a.st]);
    return mx > 0.0 ? recip(mx) : 1.0;
}

// Pivot floor eps ||T||; the bound keeps its reciprocal finite for T = 0.
__device__ __forceinline__ double inv_floor(double tnorm) { return fmax(tnorm * DBL_EPSILON, 0x1p-900); }

// Inverse iteration for orders up to kInvLdsMax: one wave per block, `vpb`
// eigenvalues of one matrix in its first lanes.  The factorization is repeated
// by each launch (it costs about one solve) instead of being kept in memory.  A
// step's chain is a few fp64 operations and its operands come from LDS a run
// of steps ahead, where the global-memory form waits on L2 at every eight
// steps: 32 vectors of four matrices of order 768 take 0.47 ms for both
// launches, 256 vectors of order 264 0.18 ms (0.72 ms).  The order limit is the
// 160 KB of LDS.
constexpr int kInvLdsMax = 2800;
inline int64_t inv_lds_bytes(int n, int vpb) { return (int64_t)n * (16 + 33 * (int64_t)vpb); }

__global__ void __launch_bounds__(64) tri_inverse_lds_kernel(const double* dd, const double* ee, int64_t stride_n,
                                                             int n, const double* lam, int64_t stride_lam, int nvals,
                                                             double* y, int solves, int init, int vpb) {
    extern __shared__ double sh[];
    const int z = blockIdx.y, lane = threadIdx.x, k0 = blockIdx.x * vpb;
    const int nk = min(vpb, nvals - k0);            // eigenvalues of this block
    double2* de = reinterpret_cast<double2*>(sh);   // (d_i, e_i)
    double* base = sh + 2 * n;
    const int64_t nv = (int64_t)n * vpb;
    double* yw = base + 3 * nv;
    const InvLds a{de, base + lane, base + nv + lane, base + 2 * nv + lane,
                   reinterpret_cast<unsigned char*>(base + 4 * nv) + lane, yw + lane, vpb, vpb};
    const double* d0 = dd + (int64_t)z * stride_n;
    const double* e0 = ee + (int64_t)z * stride_n;
    double* yz = y + ((int64_t)z * nvals + k0) * (int64_t)n;
    double tn = 0.0;
    for (int i = lane; i < n; i += 64) {
        const double di = d0[i], ei = i + 1 < n ? e0[i] : 0.0, em = i > 0 ? e0[i - 1] : 0.0;
        de[i] = make_double2(di, ei);
        tn = fmax(tn, fabs(di) + fabs(ei) + fabs(em));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) tn = fmax(tn, __shfl_xor(tn, o, 64));
    if (!init)
        for (int k = 0; k < nk; ++k)
            for (int i = lane; i < n; i += 64) yw[(int64_t)i * vpb + k] = yz[(int64_t)k * n + i];
    __syncthreads();
    double scale = 1.0;
    if (lane < nk) {
        double c = inv_factor(a, n, lam[(int64_t)z * stride_lam + k0 + lane], inv_floor(tn), k0 + lane, init);
        for (int sv = 0; sv < solves; ++sv) {
            if (sv > 0) c = inv_forward(a, n, scale);
            scale = inv_backward(a, n, c);
        }
    }
    __syncthreads();
    for (int k = 0; k < nk; ++k) {
        const double sk = lane_value(scale, k);
        for (int i = lane; i < n; i += 64) yz[(int64_t)k * n + i] = yw[(int64_t)i * vpb + k] * sk;
    }
}

// Inverse iteration for orders above kInvLdsMax, one thread per eigenvalue k of
// matrix z: partially
// pivoted LU of T - lambda_k I, then `solves` solves of y (start: a fixed
// pseudo-random vector when init is set, else y as left by the previous
// launch), each followed by scaling to max |y_i| = 1.  The factors
// [dl | 1/d | du | du2 | pivot flag] and the working vector live in `lu`,
// interleaved across the eigenvalues of a matrix (entry i of vector k at
// [i nvals + k]) so each load and store of a wave is contiguous; the values
// a step carries to the next stay in registers.  y (one contiguous row per
// vector) is read at the start when init is clear and written at the end.
__global__ void __launch_bounds__(64) tri_inverse_kernel(const double* dd, const double* ee, int64_t stride_n, int n,
                                                         const double* lam, int64_t stride_lam, int nvals, double* lu,
                                                         double* y, int solves, int init) {
    const int z = blockIdx.y, k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nvals) return;
    const double* __restrict__ d0 = dd + (int64_t)z * stride_n;
    const double* __restrict__ e0 = ee + (int64_t)z * stride_n;
    const int64_t nv = nvals, an = (int64_t)n * nv;
    double* base = lu + (int64_t)z * 6 * an + k;
    double* __restrict__ dl = base;
    double* __restrict__ ig = base + an;
    double* __restrict__ du = base + 2 * an;
    double* __restrict__ du2 = base + 3 * an;
    double* __restrict__ pv = base + 4 * an;
    double* __restrict__ yw = base + 5 * an;
    double* __restrict__ yk = y + ((int64_t)z * nvals + k) * (int64_t)n;
    const double lk = lam[(int64_t)z * stride_lam + k];
    if (init) {
        // Scale of T for the pivot floor.
        double tn = 0.0;
        for (int i = 0; i < n; ++i)
            tn = fmax(tn, fabs(d0[i]) + (i > 0 ? fabs(e0[i - 1]) : 0.0) + (i + 1 < n ? fabs(e0[i]) : 0.0));
        const double floor_piv = fmax(tn, DBL_MIN) * DBL_EPSILON;
        auto floored = [&](double g) { return fabs(g) < floor_piv ? (g < 0.0 ? -floor_piv : floor_piv) : g; };
        // g, u: the current diagonal and superdiagonal entries of row i (row
        // i + 1 of the matrix is still untouched when step i starts).
        double g = d0[0] - lk, u = n > 1 ? e0[0] : 0.0;
#pragma unroll 4
        for (int i = 0; i + 1 < n; ++i) {
            const double l = e0[i], gn = d0[i + 1] - lk, un = i + 2 < n ? e0[i + 1] : 0.0;
            const int64_t o = (int64_t)i * nv;
            if (fabs(g) >= fabs(l)) {
                const double f = g != 0.0 ? l / g : 0.0;
                dl[o] = f;
                ig[o] = 1.0 / floored(g);
                du[o] = u;
                du2[o] = 0.0;
                pv[o] = 0.0;
                g = gn - f * u;
                u = un;
            } else {
                const double f = g / l;
                dl[o] = f;
                ig[o] = 1.0 / floored(l);
                du[o] = gn;
                du2[o] = un;
                pv[o] = 1.0;
                g = u - f * gn;
                u = -f * un;
            }
        }
        ig[(int64_t)(n - 1) * nv] = 1.0 / floored(g);
        // Start vector: a fixed pseudo-random sequence in [-1, 1], distinct per k.
        uint32_t h = 0x9e3779b9u * (uint32_t)(k + 1);
        for (int i = 0; i < n; ++i) {
            h ^= h << 13; h ^= h >> 17; h ^= h << 5;
            yw[(int64_t)i * nv] = ((double)(h >> 8) * (1.0 / 8388608.0)) - 1.0;
        }
    } else {
#pragma unroll 8
        for (int i = 0; i < n; ++i) yw[(int64_t)i * nv] = yk[i];
    }
    // Both sweeps load eight steps' operands before the first of their stores
    // (the loads of the working vector would otherwise wait on the stores).
    constexpr int B = 8;
    double scale = 1.0;
    for (int sv = 0; sv < solves; ++sv) {
        // Forward: P L, the running entry c = y[i] in a register.
        double c = yw[0] * scale;
        for (int i0 = 0; i0 + 1 < n; i0 += B) {
            double nx[B], fl[B], pf[B];
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const int64_t o = (int64_t)(i0 + j) * nv;
                const bool in = i0 + j + 1 < n;
                nx[j] = in ? yw[o + nv] * scale : 0.0;
                fl[j] = in ? dl[o] : 0.0;
                pf[j] = in ? pv[o] : 0.0;
            }
#pragma unroll
            for (int j = 0; j < B; ++j) {
                if (i0 + j + 1 >= n) break;
                const int64_t o = (int64_t)(i0 + j) * nv;
                if (pf[j] == 0.0) {
                    yw[o] = c;
                    c = nx[j] - fl[j] * c;
                } else {
                    yw[o] = nx[j];
                    c = c - fl[j] * nx[j];
                }
            }
        }
        // Backward: U with two superdiagonals, y[i + 1] and y[i + 2] carried.
        double y1 = c * ig[(int64_t)(n - 1) * nv], y2 = 0.0, mx = fabs(y1);
        yw[(int64_t)(n - 1) * nv] = y1;
        for (int i0 = n - 2; i0 >= 0; i0 -= B) {
            double yv[B], uu[B], u2[B], gi[B];
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const int i = i0 - j;
                const int64_t o = (int64_t)(i < 0 ? 0 : i) * nv;
                yv[j] = i >= 0 ? yw[o] : 0.0;
                uu[j] = i >= 0 ? du[o] : 0.0;
                u2[j] = i >= 0 && i + 2 < n ? du2[o] : 0.0;
                gi[j] = i >= 0 ? ig[o] : 0.0;
            }
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const int i = i0 - j;
                if (i < 0) break;
                const double y0 = (yv[j] - uu[j] * y1 - u2[j] * y2) * gi[j];
                yw[(int64_t)i * nv] = y0;
                mx = fmax(mx, fabs(y0));
                y2 = y1;
                y1 = y0;
            }
        }
        scale = mx > 0.0 ? 1.0 / mx : 1.0;
    }
#pragma unroll 8
    for (int i = 0; i < n; ++i) yk[i] = yw[(int64_t)i * nv] * scale;
}

// Modified Gram-Schmidt inside clusters (eigenvalues, descending, closer
// than ortol = 1e-9 * max |lambda| to their neighbour), then unit norm.  With
// shifts accurate to a few ulps, two solves leave a neighbour at gap g with a
// weight of about (eps ||T|| / g)^2, so only near-degenerate eigenvalues (the
// same shift from bisection) need the explicit orthogonalization.  Block k
// owns the cluster that starts at eigenvalue k (other blocks return), so
// clusters, mostly single vectors, run in parallel.
__global__ void __launch_bounds__(kVecThreads) vec_cluster_mgs_kernel(const double* lam, int64_t stride_lam, int n,
                                                                     int nvals, double* y) {
    __shared__ double red[kVecThreads / 64];
    const int z = blockIdx.y, k0 = blockIdx.x, tid = threadIdx.x;
    const double* lz = lam + (int64_t)z * stride_lam;
    const double ortol = 1e-9 * fmax(fabs(lz[0]), fabs(lz[nvals - 1]));
    if (k0 > 0 && !(lz[k0 - 1] - lz[k0] > ortol)) return;
    int k1 = k0 + 1;
    while (k1 < nvals && !(lz[k1 - 1] - lz[k1] > ortol)) ++k1;
    double* yz = y + (int64_t)z * nvals * n;
    for (int k = k0; k < k1; ++k) {
        double* yk = yz + (int64_t)k * n;
        for (int q = k0; q < k; ++q) {
            const double* yq = yz + (int64_t)q * n;
            double s = 0.0;
            for (int i = tid; i < n; i += kVecThreads) s += yk[i] * yq[i];
            s = block_sum_d<kVecThreads>(s, red);
            for (int i = tid; i < n; i += kVecThreads) yk[i] -= s * yq[i];
            __syncthreads();
        }
        double s = 0.0;
        for (int i = tid; i < n; i += kVecThreads) s += yk[i] * yk[i];
        s = block_sum_d<kVecThreads>(s, red);
        const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
        for (int i = tid; i < n; i += kVecThreads) yk[i] *= inv;
        __syncthreads();
    }
}

// Compact WY form of the reflectors in panels of kWy: H_{j0} ... H_{j0+31} =
// I - V T V^T with T upper triangular, T(k, k) = tau_k and
// T(0..k-1, k) = -tau_k T(0..k-1, 0..k-1) V(:, 0..k-1)^T v_k.  One block per panel
// and matrix: V^T V from LDS slabs of 64 columns, then T, one row per lane.
// Reflector j is row j of A from column j + 1 on (v_j[j + 1] = 1).
constexpr int kWy = 32;

__global__ void __launch_bounds__(256) wy_t_kernel(const float* A, int64_t strideA, int n, const double* tau,
                                                   int64_t stride_n, double* wy, int64_t stride_wy) {
    __shared__ float vs[kWy][65];
    __shared__ double G[kWy][kWy + 1];
    const int z = blockIdx.y, j0 = blockIdx.x * kWy, tid = threadIdx.x;
    const float* Az = A + (int64_t)z * strideA;
    const int gk = (tid >> 4) * 2, gl = (tid & 15) * 2;   // 2 x 2 entries of V^T V
    double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
    for (int i0 = (j0 + 1) & ~63; i0 < n; i0 += 64) {
#pragma unroll
        for (int t = 0; t < kWy * 64 / 256; ++t) {
            const int q = tid + 256 * t, r = q >> 6, i = i0 + (q & 63), j = j0 + r;
            const float a = Az[(int64_t)min(j, n - 1) * n + min(i, n - 1)];
            vs[r][q & 63] = j < n && i > j && i < n ? a : 0.f;
        }
        __syncthreads();
#pragma unroll 8
        for (int c = 0; c < 64; ++c) {
            const double a0 = vs[gk][c], a1 = vs[gk + 1][c], b0 = vs[gl][c], b1 = vs[gl + 1][c];
            acc[0][0] += a0 * b0;
            acc[0][1] += a0 * b1;
            acc[1][0] += a1 * b0;
            acc[1][1] += a1 * b1;
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) G[gk + a][gl + b] = acc[a][b];
    __syncthreads();
    if (tid < kWy) {
        double t[kWy];
        double* o = wy + (int64_t)z * stride_wy + (int64_t)blockIdx.x * kWy * kWy + tid * kWy;
#pragma unroll
        for (int k = 0; k < kWy; ++k) {
            const double tk = j0 + k < n ? tau[(int64_t)z * stride_n + j0 + k] : 0.0;
            double s = 0.0;
#pragma unroll
            for (int l = 0; l < k; ++l) s += t[l] * G[l][k];
            t[k] = k < tid ? 0.0 : (k == tid ? tk : -tk * s);
            o[k] = t[k];
        }
    }
}

// u = H_0 H_1 ... H_{n-1} y_k in place in y, one block per vector, u in LDS: per
// panel from the last, s = V^T u (a wave per four reflectors), c = T s,
// u -= V c.  0.38 us per reflector at order 768 (one reflector at a time, two
// barriers each: 2.4 us).
constexpr int kBackThreads = 512;

__global__ void __launch_bounds__(kBackThreads) wy_apply_kernel(const float* A, int64_t strideA, int n,
                                                                const double* wy, int64_t stride_wy, double* y,
                                                                int nvals) {
    extern __shared__ double ul[];      // n
    __shared__ double sv[kWy], cv[kWy];
    const int z = blockIdx.y, k = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int R = kWy / (kBackThreads / 64);
    double* u = y + ((int64_t)z * nvals + k) * (int64_t)n;
    const float* Az = A + (int64_t)z * strideA;
    const double* Tz = wy + (int64_t)z * stride_wy;
    for (int i = tid; i < n; i += kBackThreads) ul[i] = u[i];
    __syncthreads();
    const int tr = tid >> 3, tc = tid & 7;      // c = T s: eight lanes per row
    for (int p = (n - 1) / kWy; p >= 0; --p) {
        const int j0 = p * kWy;
        double tq[kWy / 8];
        if (tid < 8 * kWy)
#pragma unroll
            for (int q = 0; q < kWy / 8; ++q) tq[q] = Tz[(int64_t)p * kWy * kWy + tr * kWy + tc + 8 * q];
        // Reflector rows of this wave (clamped: row n - 1 stands in past the
        // end, its T entries are zero).  The masks concern the first 32
        // entries only; the loads are unconditional, so they overlap.
        const float* vr[R];
        double s[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            vr[r] = Az + (int64_t)min(j0 + R * wave + r, n - 1) * n;
            s[r] = 0.0;
        }
#pragma unroll 4
        for (int i = j0 + 1 + lane; i < n; i += 64) {
            const double ui = ul[i];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float a = vr[r][i];
                s[r] += (double)(i > j0 + R * wave + r ? a : 0.f) * ui;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double v = wave_sum_d(s[r]);
            if (lane == 0) sv[R * wave + r] = v;
        }
        __syncthreads();
        if (tid < 8 * kWy) {
            double c = 0.0;
#pragma unroll
            for (int q = 0; q < kWy / 8; ++q) c += tq[q] * sv[tc + 8 * q];
            c += dpp_take<0x141, 0xf>(c);
            c = sum_quad(c);
            if (tc == 0) cv[tr] = c;
        }
        __syncthreads();
        for (int i = j0 + 1 + tid; i < n; i += kBackThreads) {
            const float* col = Az + (int64_t)j0 * n + i;
            double acc = 0.0;
#pragma unroll 16
            for (int r = 0; r < kWy; ++r) {
                const float a = col[(int64_t)min(r, n - 1 - j0) * n];
                acc += (double)(j0 + r < i ? a : 0.f) * cv[r];
            }
            ul[i] -= acc;
        }
        __syncthreads();
    }
    for (int i = tid; i < n; i += kBackThreads) u[i] = ul[i];
}

// The eigenvectors y (nvals x n per matrix, contiguous) as fp32 rows (ld,
// zero padded to ld; rows nvals .. rows_out - 1 zero).
__global__ void __launch_bounds__(256) vec_rows_kernel(const double* y, int nvals, int n, float* out, int64_t ld_out,
                                                       int64_t stride_out) {
    const int z = blockIdx.y, k = blockIdx.x;
    float* o = out + (int64_t)z * stride_out + (int64_t)k * ld_out;
    const double* u = y + ((int64_t)z * nvals + k) * (int64_t)n;
    for (int64_t i = threadIdx.x; i < ld_out; i += 256) o[i] = k < nvals && i < n ? (float)u[i] : 0.f;
}

// The same as two fp16 parts, hi = fp16(y) and lo = fp16(2^11 (y - hi)):
// together 22 bits, so hi Psi + 2^-11 lo Psi carries y to fp32 accuracy.
__global__ void __launch_bounds__(256) vec_split_kernel(const double* y, int nvals, int n, half_t* hi, half_t* lo,
                                                        int64_t ld_out, int64_t stride_out) {
    const int z = blockIdx.y, k = blockIdx.x;
    const int64_t o = (int64_t)z * stride_out + (int64_t)k * ld_out;
    const double* u = y + ((int64_t)z * nvals + k) * (int64_t)n;
    for (int64_t i = threadIdx.x; i < ld_out; i += 256) {
        const double v = k < nvals && i < n ? u[i] : 0.0;
        const half_t h = (half_t)(float)v;
        hi[o + i] = h;
        lo[o + i] = (half_t)(float)((v - (double)(float)h) * 2048.0);
    }
}
// a += 2^-11 b, float4-wise over `rows` x len per matrix (one stride).
__global__ void __launch_bounds__(256) join_split_kernel(float4* a, const float4* b, int64_t n4, int64_t stride4) {
    const int64_t o = (int64_t)blockIdx.y * stride4;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
        float4 x = a[o + i];
        const float4 v = b[o + i];
        x.x += v.x * 0x1p-11f;
        x.y += v.y * 0x1p-11f;
        x.z += v.z * 0x1p-11f;
        x.w += v.w * 0x1p-11f;
        a[o + i] = x;
    }
}

// Summed fp64 Gram partials (upper 16 x 16 tiles, chunks x l_pad x l_pad)
// -> symmetric n x n fp32 matrix.
__global__ void gram_to_mat_kernel(const double* partial, int chunks, int ell_pad, int n, float* A) {
    const int z = blockIdx.y;
    const double* part = partial + (int64_t)z * chunks * ell_pad * ell_pad;
    float* Az = A + (int64_t)z * n * n;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n * n; idx += gridDim.x * blockDim.x) {
        const int c = idx / n, d = idx - (idx / n) * n;
        Az[idx] = (float)gram_at(part, ell_pad, c, d, chunks);
    }
}

// Selection of the top eigenpairs (lam descending, z rows) above one, Ritz
// values and |C|; K = Z_C diag(lambda^-1/2 - 1) Z_C^T (l_pad x l_pad, zero
// outside n x n), 256 entries per block.
__global__ void __launch_bounds__(256) select_k_kernel(const double* lam, int top, const float* zbuf, int n,
                                                       int ell_pad, float* kmat, float* ritz, int ritz_stride,
                                                       int* nsel) {
    const int z = blockIdx.y;
    const double* lz = lam + (int64_t)z * top;
    const float* Z = zbuf + (int64_t)z * top * n;
    int ns = 0;
    while (ns < top && lz[ns] > 1.0) ++ns;      // descending: the selected ones lead
    if (blockIdx.x == 0) {
        for (int t = threadIdx.x; t < top; t += 256) ritz[(int64_t)z * ritz_stride + t] = (float)lz[t];
        if (threadIdx.x == 0) nsel[z] = ns;
    }
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= ell_pad * ell_pad) return;
    const int c = q / ell_pad, d = q - (q / ell_pad) * ell_pad;
    double sacc = 0.0;
    if (c < n && d < n)
        for (int t = 0; t < ns; ++t) sacc += (double)Z[t * n + c] * (1.0 / sqrt(lz[t]) - 1.0) * (double)Z[t * n + d];
    kmat[(int64_t)z * ell_pad * ell_pad + q] = (float)sacc;
}

// Ritz pairs, selection and K of one l x l problem per workgroup, l <= kRitzMax:
// the dense solver's steps (reduction in registers, multisection, inverse
// iteration with one lane per vector, Gram-Schmidt inside clusters,
// back-transformation) with everything between them in LDS, in one launch.  All
// of them are chains of l steps whose LDS instructions all waves share (an
// access of few lanes takes the pipe as long as one of 64), so the workgroup
// has four waves: with sixteen the same steps took three times as long.
//   LDS: y (top x n doubles, odd pitch), the LU factors of `batch` vectors, and
//   the tridiagonal matrix; the reflectors go to K's memory until K is formed.
// 138 us per launch at l = 40 (48 matrices), 304 at l = 72 (112), 70 at l = 24, a
// third of it the reduction at 1.0-1.25 us per column; the round-robin fp32
// Jacobi it replaces took 194, 692 and 99 us (six sweeps of l rounds).
constexpr int kRitzMax = 80;
constexpr int kRitzWaves = 4, kRitzThreads = 64 * kRitzWaves;
constexpr size_t kRitzLds = 156 * 1024;

inline size_t ritz_fixed_lds(int n, int top) {
    const int np8 = (n + kSturmRun - 1) / kSturmRun * kSturmRun;
    return (size_t)8 * ((size_t)top * (n | 1) + 3 * n + 1 + 2 * np8 + 2 * n + 2 * top);
}
inline size_t ritz_vec_lds(int n) { return (size_t)n * 25; }

template <int R, int C>
__global__ void __launch_bounds__(kRitzThreads) ritz_kernel(EigArgs a, int batch) {
    extern __shared__ double dyn[];
    __shared__ TriRegShared<C> sh;
    __shared__ double gl[kRitzWaves], gh[kRitzWaves], gt[kRitzWaves];
    constexpr int NW = kRitzWaves;
    const int z = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, cl = lane & 31;
    const int n = a.ell, lp = a.ell_pad, top = min(a.rank, n), ny = n | 1;
    const int np8 = (n + kSturmRun - 1) / kSturmRun * kSturmRun;
    double* y = dyn;                                // [t][i], pitch ny
    double* d = y + (size_t)top * ny;
    double* e = d + n;
    double* tau = e + n;
    double2* ds = reinterpret_cast<double2*>(tau + n + ((top * ny + 3 * n) & 1));     // scaled (d, e^2)
    double2* de = ds + np8;                         // (d_i, e_i)
    double* lam = reinterpret_cast<double*>(de + n);
    double* fc = lam + top;
    double* lu = fc + top;                          // f, r, m of a batch
    unsigned char* sw = reinterpret_cast<unsigned char*>(lu + 3 * (size_t)n * batch);
    float* K = a.kmat + (int64_t)z * lp * lp;
    float* V = K;                                   // n x n, until K is formed
    const double* part = a.partial + (int64_t)z * a.chunks * lp * lp;
    float M[R][C];
#pragma unroll
    for (int s = 0; s < R; ++s)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int i = 2 * NW * s + 2 * wave + half, k = 32 * c + cl;
            const double v = gram_at(part, lp, min(i, n - 1), min(k, n - 1), a.chunks);
            M[s][c] = i < n && k < n ? (float)v : 0.f;
        }
    int par = 0;
    tri_reg_cols<NW, R, C, 0>(M, sh, par, n, V, n, d, e, tau);
    __syncthreads();
    // Gershgorin interval and the norm for the pivot floor.
    double lo = DBL_MAX, hi = -DBL_MAX, tn = 0.0;
    for (int i = tid; i < n; i += kRitzThreads) {
        const double em = i > 0 ? fabs(e[i - 1]) : 0.0, ei = i + 1 < n ? fabs(e[i]) : 0.0;
        lo = fmin(lo, d[i] - em - ei);
        hi = fmax(hi, d[i] + em + ei);
        tn = fmax(tn, fabs(d[i]) + em + ei);
        de[i] = make_double2(d[i], i + 1 < n ? e[i] : 0.0);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, 64));
        hi = fmax(hi, __shfl_xor(hi, o, 64));
        tn = fmax(tn, __shfl_xor(tn, o, 64));
    }
    if (lane == 0) {
        gl[wave] = lo;
        gh[wave] = hi;
        gt[wave] = tn;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        lo = fmin(lo, gl[q]);
        hi = fmax(hi, gh[q]);
        tn = fmax(tn, gt[q]);
    }
    const double span = fmax(fabs(lo), fabs(hi));
    int ex = 0;
    if (span > 0.0) (void)frexp(span, &ex);
    for (int i = tid; i < np8; i += kRitzThreads) ds[i] = sturm_entry(d, e, n, i, ex);
    __syncthreads();
    {
        const double slo = ldexp(lo, -ex) - 2.0 * DBL_EPSILON, shi = ldexp(hi, -ex) + 2.0 * DBL_EPSILON;
        // As many lanes per eigenvalue as one pass over all of them allows.
        auto all = [&](auto lanes) {
            constexpr int L = decltype(lanes)::value, G = 64 / L;
            for (int t0 = G * wave; t0 < top; t0 += G * NW) {
                const int t = t0 + lane / L;
                // Groups past the last eigenvalue repeat it (the ballots need all lanes).
                const double x = span > 0.0 ? multisect<L, 2>(ds, np8, n - 1 - min(t, top - 1), slo, shi, lane % L,
                                                              lane / L * L)
                                            : 0.0;
                if (lane % L == 0 && t < top) lam[t] = ldexp(x, ex);
            }
        };
        if (top <= 4 * NW) all(std::integral_constant<int, 16>{});
        else if (top <= 8 * NW) all(std::integral_constant<int, 8>{});
        else all(std::integral_constant<int, 4>{});
    }
    __syncthreads();
    // After two solves the clusters are orthogonalized and one more solve
    // follows.
    constexpr int E = (32 * C + 63) / 64;           // entries of a vector per lane
    auto orthonormal = [&]() {
        const double ortol = 1e-9 * fmax(fabs(lam[0]), fabs(lam[top - 1]));
        for (int k0 = wave; k0 < top; k0 += NW) {
            if (k0 > 0 && !(lam[k0 - 1] - lam[k0] > ortol)) continue;   // inside a cluster
            int k1 = k0 + 1;
            while (k1 < top && !(lam[k1 - 1] - lam[k1] > ortol)) ++k1;
            for (int k = k0; k < k1; ++k) {
                double v[E];
#pragma unroll
                for (int c = 0; c < E; ++c) v[c] = lane + 64 * c < n ? y[k * ny + lane + 64 * c] : 0.0;
                for (int q = k0; q < k; ++q) {
                    double s = 0.0;
#pragma unroll
                    for (int c = 0; c < E; ++c) s += lane + 64 * c < n ? v[c] * y[q * ny + lane + 64 * c] : 0.0;
                    s = wave_sum_d(s);
#pragma unroll
                    for (int c = 0; c < E; ++c)
                        if (lane + 64 * c < n) v[c] -= s * y[q * ny + lane + 64 * c];
                }
                double s = 0.0;
#pragma unroll
                for (int c = 0; c < E; ++c) s += v[c] * v[c];
                s = wave_sum_d(s);
                const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
                for (int c = 0; c < E; ++c)
                    if (lane + 64 * c < n) y[k * ny + lane + 64 * c] = v[c] * inv;
            }
        }
    };
    const double floor_piv = inv_floor(tn);
    const int per_wave = (batch + NW - 1) / NW;     // lanes of each wave that hold a vector
    for (int pass = 0; pass < 2; ++pass) {
        for (int b0 = 0; b0 < top; b0 += batch) {
            const int v = per_wave * wave + lane, t = b0 + v;
            if (lane < per_wave && v < batch && t < top) {
                const size_t nb = (size_t)n * batch;
                const InvLds w{de, lu + v, lu + nb + v, lu + 2 * nb + v, sw + v, y + (size_t)t * ny, batch, 1};
                // A single batch keeps its factors for the second pass.
                const double c = pass == 0 || top > batch ? inv_factor(w, n, lam[t], floor_piv, t, pass == 0)
                                                          : inv_forward(w, n, 1.0);
                double sc = inv_backward(w, n, c);
                if (pass == 0) sc = inv_backward(w, n, inv_forward(w, n, sc));
                for (int i = 0; i < n; ++i) w.y[i] *= sc;
            }
        }
        __syncthreads();
        orthonormal();
        __syncthreads();
    }
    // u = H_0 ... H_{n-2} y, a wave per eight vectors.
    for (int t0 = 8 * wave; t0 < top; t0 += 8 * NW) {
        double u[8][E], vn[E];
        auto load_v = [&](int j) {
#pragma unroll
            for (int c = 0; c < E; ++c) {
                const int i = lane + 64 * c;
                const float x = V[max(j, 0) * n + min(i, n - 1)];
                vn[c] = i > j && i < n ? (double)x : 0.0;
            }
        };
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int c = 0; c < E; ++c) u[q][c] = lane + 64 * c < n ? y[min(t0 + q, top - 1) * ny + lane + 64 * c] : 0.0;
        load_v(n - 2);
        for (int j = n - 2; j >= 0; --j) {
            double v[E], s[8];
#pragma unroll
            for (int c = 0; c < E; ++c) v[c] = vn[c];
            load_v(j - 1);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                s[q] = 0.0;
#pragma unroll
                for (int c = 0; c < E; ++c) s[q] += v[c] * u[q][c];
            }
            int slot;
            bool first;
            const double sum = tau[j] * sum_values<64>(s, lane, slot, first);
            // The sum of vector q sits in the lanes with bits 5, 4, 3 = q.
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double f = lane_value(sum, 8 * q);
#pragma unroll
                for (int c = 0; c < E; ++c) u[q][c] -= f * v[c];
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int c = 0; c < E; ++c)
                if (t0 + q < top && lane + 64 * c < n) y[(t0 + q) * ny + lane + 64 * c] = u[q][c];
    }
    // Selection (lam is descending, so the selected ones lead) and K = Z_C
    // diag(lambda^-1/2 - 1) Z_C^T in 4 x 4 blocks.
    int ns = 0;
    while (ns < top && lam[ns] > 1.0) ++ns;
    for (int t = tid; t < top; t += kRitzThreads) {
        fc[t] = t < ns ? 1.0 / sqrt(lam[t]) - 1.0 : 0.0;
        a.ritz[(int64_t)z * a.ritz_stride + t] = (float)lam[t];
    }
    if (tid == 0) a.nsel[z] = ns;
    __syncthreads();
    const int nb = lp / 4;
    for (int b = tid; b < nb * nb; b += kRitzThreads) {
        const int c0 = b / nb * 4, d0 = (b - b / nb * nb) * 4;
        double acc[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
        if (c0 < n && d0 < n)
            for (int t = 0; t < ns; ++t) {
                const double f = fc[t];
                double zc[4], zd[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    zc[u] = y[t * ny + min(c0 + u, n - 1)] * f;
                    zd[u] = y[t * ny + min(d0 + u, n - 1)];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[u][v] = fma(zc[u], zd[v], acc[u][v]);
            }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float4 o;
            o.x = c0 + u < n && d0 < n ? (float)acc[u][0] : 0.f;
            o.y = c0 + u < n && d0 + 1 < n ? (float)acc[u][1] : 0.f;
            o.z = c0 + u < n && d0 + 2 < n ? (float)acc[u][2] : 0.f;
            o.w = c0 + u < n && d0 + 3 < n ? (float)acc[u][3] : 0.f;
            *(float4*)(K + (int64_t)(c0 + u) * lp + d0) = o;
        }
    }
}

}  // namespace

hipError_t launch_gamma_sym(const float* g, int64_t ldg, int64_t strideg, int n, float* A, int batch,
                            hipStream_t s) {
    const int64_t nn = (int64_t)n * n;
    const unsigned blocks = (unsigned)std::min<int64_t>(4096, (nn + 255) / 256);
    hipLaunchKernelGGL(gamma_sym_kernel, dim3(blocks, batch), dim3(256), 0, s, g, ldg, strideg, n, A, nn);
    return hipGetLastError();
}

hipError_t launch_tridiagonalize(const TriWork& w, int n, int batch, hipStream_t s) {
    if (n < 1) return hipErrorInvalidValue;
    // Columns 0 .. j0 - 1 one launch each, then the trailing block of at most
    // kTriRegMax in one launch.
    const int j0 = std::max(0, n - kTriRegMax);
    for (int j = 0; j < j0; ++j) {
        // Columns from c0 (a multiple of 64, for aligned rows) on; threads and
        // columns per thread by what is left, RB rows per pass.
        const int c0 = j & ~63, cols = n - c0, rows = n - j - 1;
        auto step = [&](auto kern, int nt, int rb) {
            // One pass of rows per block while the blocks fit the chip at once
            // (2048 threads per CU), more passes beyond; a multiple of 8.
            const int fit = std::max(8, 256 * (2048 / nt) / batch & ~7);
            const int nb = std::min(((rows + rb - 1) / rb + 7) & ~7, fit);
            hipLaunchKernelGGL(kern, dim3(nb, batch), dim3(nt), 0, s, w.A, (int64_t)n * n, n, j, c0, w.vec,
                               4 * (int64_t)n, w.d, w.e, w.tau, (int64_t)n);
        };
        if (cols <= 512) step(tri_step_kernel<256, 2, 8>, 256, 8);
        else if (cols <= 1024) step(tri_step_kernel<256, 4, 8>, 256, 8);
        else if (cols <= 2048) step(tri_step_kernel<512, 4, 8>, 512, 8);
        else if (cols <= 4096) step(tri_step_kernel<512, 8, 4>, 512, 4);
        else if (cols <= 8192) step(tri_step_kernel<1024, 8, 2>, 1024, 2);
        else return hipErrorInvalidValue;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(tri_reg_kernel, dim3(batch), dim3(kTriThreads), 0, s, w.A, (int64_t)n * n, n, j0, w.vec,
                       4 * (int64_t)n, w.d, w.e, w.tau, (int64_t)n);
    return hipGetLastError();
}

hipError_t launch_tri_eigvals(const TriWork& w, int n, int first, int nvals, double* out, int64_t stride_out,
                              int batch, hipStream_t s) {
    if (nvals < 1) return hipSuccess;
    const size_t lds = (size_t)((n + kSturmRun - 1) / kSturmRun * kSturmRun) * sizeof(double2);
    hipLaunchKernelGGL(tri_bisect_kernel, dim3((nvals + kBisectWaves - 1) / kBisectWaves, batch),
                       dim3(64 * kBisectWaves), lds, s, w.d, w.e, (int64_t)n, n, first, nvals, out, stride_out);
    return hipGetLastError();
}

// Orders above this keep the inverse iteration's factors in global memory
// (TriWork::lu).
bool tri_needs_lu(int n) { return n > kInvLdsMax; }

hipError_t launch_tri_eigvecs(const TriWork& w, int n, const double* lam, int nvals, int batch, hipStream_t s) {
    if (nvals < 1) return hipErrorInvalidValue;
    auto inverse = [&](int solves, int init) {
        if (tri_needs_lu(n)) {
            hipLaunchKernelGGL(tri_inverse_kernel, dim3((nvals + 63) / 64, batch), dim3(64), 0, s, w.d, w.e,
                               (int64_t)n, n, lam, (int64_t)nvals, nvals, w.lu, w.y, solves, init);
        } else {
            // Few eigenvalues per block: the blocks' chains run side by side
            // on the CUs.  Up to four while there are more than 256 blocks.
            int vpb = 1;
            while (vpb < 4 && (int64_t)((nvals + vpb - 1) / vpb) * batch > 256 &&
                   inv_lds_bytes(n, 2 * vpb) <= 80 * 1024)
                vpb *= 2;
            hipLaunchKernelGGL(tri_inverse_lds_kernel, dim3((nvals + vpb - 1) / vpb, batch), dim3(64),
                               (size_t)inv_lds_bytes(n, vpb), s, w.d, w.e, (int64_t)n, n, lam, (int64_t)nvals, nvals,
                               w.y, solves, init, vpb);
        }
        return hipGetLastError();
    };
    auto orthonormal = [&]() {
        hipLaunchKernelGGL(vec_cluster_mgs_kernel, dim3(nvals, batch), dim3(kVecThreads), 0, s, lam, (int64_t)nvals,
                           n, nvals, w.y);
        return hipGetLastError();
    };
    hipError_t e = inverse(2, 1);
    if (e == hipSuccess) e = orthonormal();
    if (e == hipSuccess) e = inverse(1, 0);
    if (e == hipSuccess) e = orthonormal();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(wy_t_kernel, dim3((n + kWy - 1) / kWy, batch), dim3(256), 0, s, w.A, (int64_t)n * n, n, w.tau,
                       (int64_t)n, w.wy, w.stride_wy);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(wy_apply_kernel, dim3(nvals, batch), dim3(kBackThreads), (size_t)n * sizeof(double), s, w.A,
                       (int64_t)n * n, n, w.wy, w.stride_wy, w.y, nvals);
    return hipGetLastError();
}

hipError_t launch_vec_rows(const double* y, int nvals, int n, float* out, int64_t ld_out, int rows_out,
                           int64_t stride_out, int batch, hipStream_t s) {
    if (nvals > rows_out || n > ld_out) return hipErrorInvalidValue;
    hipLaunchKernelGGL(vec_rows_kernel, dim3(rows_out, batch), dim3(256), 0, s, y, nvals, n, out, ld_out, stride_out);
    return hipGetLastError();
}

hipError_t launch_vec_split(const double* y, int nvals, int n, half_t* hi, half_t* lo, int64_t ld_out, int rows_out,
                            int64_t stride_out, int batch, hipStream_t s) {
    if (nvals > rows_out || n > ld_out) return hipErrorInvalidValue;
    hipLaunchKernelGGL(vec_split_kernel, dim3(rows_out, batch), dim3(256), 0, s, y, nvals, n, hi, lo, ld_out,
                       stride_out);
    return hipGetLastError();
}

hipError_t launch_join_split(float* a, const float* b, int64_t count, int64_t stride, int batch, hipStream_t s) {
    if (count % 4 || stride % 4) return hipErrorInvalidValue;
    const int64_t n4 = count / 4;
    hipLaunchKernelGGL(join_split_kernel, dim3((unsigned)std::min<int64_t>(1024, (n4 + 255) / 256), batch), dim3(256),
                       0, s, reinterpret_cast<float4*>(a), reinterpret_cast<const float4*>(b), n4, stride / 4);
    return hipGetLastError();
}

}  // namespace np

namespace np {

hipError_t launch_eig_select_dense(const EigArgs& a, const TriWork& w, double* lam, float* zbuf, int batch,
                                   hipStream_t s) {
    const int n = a.ell, lp = a.ell_pad, top = std::min(a.rank, n);
    if (a.chunks < 1 || a.chunks > kGramChunks || n < 1 || n > lp) return hipErrorInvalidValue;
    const unsigned gb = (unsigned)std::min<int64_t>(1024, ((int64_t)n * n + 255) / 256);
    hipLaunchKernelGGL(gram_to_mat_kernel, dim3(gb, batch), dim3(256), 0, s, a.partial, a.chunks, lp, n, w.A);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_tridiagonalize(w, n, batch, s);
    if (e != hipSuccess) return e;
    e = launch_tri_eigvals(w, n, 0, top, lam, top, batch, s);
    if (e != hipSuccess) return e;
    e = launch_tri_eigvecs(w, n, lam, top, batch, s);
    if (e != hipSuccess) return e;
    e = launch_vec_rows(w.y, top, n, zbuf, n, top, (int64_t)top * n, batch, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(select_k_kernel, dim3((unsigned)(((int64_t)lp * lp + 255) / 256), batch), dim3(256), 0, s,
                       lam, top, zbuf, n, lp, a.kmat, a.ritz, a.ritz_stride, a.nsel);
    return hipGetLastError();
}

// Largest width of the one-workgroup Ritz kernel.
int ritz_small_max() { return kRitzMax; }

hipError_t launch_eig_select(const EigArgs& a, int batch_mats, hipStream_t s) {
    const int n = a.ell, top = std::min(a.rank, n);
    if (n < 1 || n > kRitzMax || n > a.ell_pad || a.ell_pad % 4 || top < 1 || a.chunks < 1 || a.chunks > kGramChunks ||
        a.chunks % 4)
        return hipErrorInvalidValue;
    // All vectors at once where their factors fit, else equal batches.
    const size_t fixed = ritz_fixed_lds(n, top);
    const int most = std::min(64 * kRitzWaves, (int)((kRitzLds - fixed) / ritz_vec_lds(n)));
    const int batches = (top + most - 1) / most, batch = (top + batches - 1) / batches;
    const size_t lds = fixed + batch * ritz_vec_lds(n);
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(batch_mats), dim3(kRitzThreads), lds, s, a, batch);
    };
    if (n <= 16) run(ritz_kernel<2, 1>);
    else if (n <= 32) run(ritz_kernel<4, 1>);
    else if (n <= 48) run(ritz_kernel<6, 2>);
    else if (n <= 64) run(ritz_kernel<8, 2>);
    else run(ritz_kernel<10, 3>);
    return hipGetLastError();
}

}  // namespace np
