// Small and latency-bound kernels of the NormPre-L randomized interaction
// sketch (Alg. 2, App. B) for gfx950:
//   * the Gaussian test matrix Omega (Philox4x32-10 of Salmon et al., SC'11,
//     with the Box-Muller transform),
//   * the deterministic reduction of K-split partial products,
//   * fp64 Gram matrices of l-major skinny matrices (for the orthogonal
//     basis Q = qr(Y) and for the Rayleigh-Ritz matrix Gamma_Q = B B^T),
//   * Cholesky-QR: Cholesky of the Gram with dropping of numerically
//     dependent columns, and the triangular inverse,
//   * small products M^T V with an l x l matrix M.
#include "np_internal.h"

#include <algorithm>
#include <type_traits>

namespace np {
namespace {

// ------------------------------------------------------------- Philox ---
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
        const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
        const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
    }
    return c;
}

__device__ __forceinline__ uint4 omega_bits(uint64_t seed, int64_t step, uint32_t id, int64_t blk) {
    const uint4 ctr = make_uint4((uint32_t)blk, id, (uint32_t)((uint64_t)step & 0xffffffffu),
                                 (uint32_t)((uint64_t)step >> 32));
    return philox4x32_10(ctr, (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32));
}
// Box-Muller: the cosine and the sine normal of one pair of words.
__device__ __forceinline__ void omega_pair(uint32_t a, uint32_t b, float& zc, float& zs) {
    const float u1 = (float)((a >> 8) + 1u) * 0x1p-24f;
    const float u2 = (float)(b >> 8) * 0x1p-24f;
    const float rad = sqrtf(-2.f * logf(u1));
    float s, c;
    sincospif(2.f * u2, &s, &c);
    zc = rad * c;
    zs = rad * s;
}
// The four normal variates of block blk of the stream keyed by (seed, step, id).
__device__ __forceinline__ void omega_block(uint64_t seed, int64_t step, uint32_t id, int64_t blk, float (&v)[4]) {
    const uint4 x = omega_bits(seed, step, id, blk);
    omega_pair(x.x, x.y, v[0], v[1]);
    omega_pair(x.z, x.w, v[2], v[3]);
}

// Normal variate number e of the stream keyed by (seed, step, id).
__device__ __forceinline__ float omega_value(uint64_t seed, int64_t step, uint32_t id, int64_t e) {
    const uint4 x = omega_bits(seed, step, id, e >> 2);
    const int lane = (int)(e & 3);
    float zc, zs;
    omega_pair(lane < 2 ? x.x : x.z, lane < 2 ? x.y : x.w, zc, zs);
    return (lane & 1) ? zs : zc;
}

__global__ void __launch_bounds__(256) omega_f16_kernel(OmegaArgs a) {
    const int z = blockIdx.y;
    int g = 0;
    while (g + 1 < a.n && z >= a.zbeg[g + 1]) ++g;
    const int64_t ld = a.ld[g], b = a.b[g], total4 = (int64_t)a.ell_pad * ld / 4;
    half_t* out = a.out[g] + (int64_t)(z - a.zbeg[g]) * a.stride[g];
    const uint32_t id = (uint32_t)a.ids[z];
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total4; q += (int64_t)gridDim.x * 256) {
        const int c = (int)(4 * q / ld);
        const int64_t i = 4 * q - (int64_t)c * ld;
        half_t v[4] = {(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};
        if (c < a.ell) {
            // Four consecutive entries are one generator block when b % 4 == 0.
            if ((b & 3) == 0) {
                if (i < b) {
                    float x[4];
                    omega_block(a.seed, a.step, id, ((int64_t)c * b + i) >> 2, x);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (half_t)x[e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < b) v[e] = (half_t)omega_value(a.seed, a.step, id, (int64_t)c * b + i + e);
            }
        }
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        *(f16x4*)(out + 4 * q) = f16x4{v[0], v[1], v[2], v[3]};
    }
}

__global__ void omega_f32_kernel(uint64_t seed, int64_t step, uint32_t id, int64_t b, int ell, float* out) {
    const int64_t total = b * ell;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        // out is b x l row-major: out[i*l + j] = Omega_ij, e = j*b + i.
        const int64_t i = idx / ell, j = idx - i * ell;
        out[idx] = omega_value(seed, step, id, j * b + i);
    }
}

// ------------------------------------------------------ split reduction ---
// Partial sums of one split-K product: out = sum over splits in split order
// (fp32), to fp32 and/or fp16 (times scale16).
__device__ __forceinline__ void reduce_splits_one(const float4* p, int splits, int64_t split4, int64_t i,
                                                  float* out32, half_t* out16, float scale16) {
    float4 s = p[i];
    for (int k = 1; k < splits; ++k) {
        const float4 q = p[i + k * split4];
        s.x += q.x; s.y += q.y; s.z += q.z; s.w += q.w;
    }
    if (out32) reinterpret_cast<float4*>(out32)[i] = s;
    if (out16) {
        half_t h[4] = {(half_t)(s.x * scale16), (half_t)(s.y * scale16), (half_t)(s.z * scale16),
                       (half_t)(s.w * scale16)};
        reinterpret_cast<uint2*>(out16)[i] = *reinterpret_cast<const uint2*>(h);
    }
}

__global__ void reduce_splits_kernel(const float* part, int splits, int64_t stride_split, int64_t stride_mat,
                                     int64_t n4, float* out32, half_t* out16, float scale16, int64_t stride_out) {
    const int z = blockIdx.y;
    const float4* p = reinterpret_cast<const float4*>(part + (int64_t)z * stride_mat);
    float* o32 = out32 ? out32 + (int64_t)z * stride_out : nullptr;
    half_t* o16 = out16 ? out16 + (int64_t)z * stride_out : nullptr;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x)
        reduce_splits_one(p, splits, stride_split / 4, i, o32, o16, scale16);
}

// The split sums of several sketch products, matrix z of the launch in the
// group whose range holds it.
__global__ void reduce_splits_grouped_kernel(ReduceGroups g) {
    const int z = blockIdx.y;
    int gi = 0;
    while (gi + 1 < g.n && z >= g.zbeg[gi + 1]) ++gi;
    const int lz = z - g.zbeg[gi];
    const float4* p = reinterpret_cast<const float4*>(g.part[gi] + (int64_t)lz * g.stride_mat[gi]);
    float* o32 = g.out32[gi] ? g.out32[gi] + (int64_t)lz * g.stride_out[gi] : nullptr;
    half_t* o16 = g.out16[gi] ? g.out16[gi] + (int64_t)lz * g.stride_out[gi] : nullptr;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < g.n4[gi];
         i += (int64_t)gridDim.x * blockDim.x)
        reduce_splits_one(p, g.splits[gi], g.stride_split[gi] / 4, i, o32, o16, g.scale16[gi]);
}

// ------------------------------------------------------------ fp64 Gram ---
// Item of launch matrix z in a grouped launch (few items: a linear scan).
template <class T>
__device__ __forceinline__ int item_of(const T& t, int z) {
    int g = 0;
    while (g + 1 < t.n && z >= t.zbeg[g + 1]) ++g;
    return g;
}

// fp64 Gram by v_mfma_f64_16x16x4: lane (i, q) = (lane % 16, lane / 16) supplies
// row i, k = q of the A operand and column i, k = q of the B operand, and receives
// rows q + 4 r, column i of the product (registers r).  Both operands are rows
// of the same V in the same form, so a 16-column run of V is one float4 per
// lane and operand, converted to fp64 and used as four k-steps (element e of
// the float4 as step e: any order of k serves), with no LDS.  A block takes
// three of the upper 16 x 16 tiles (their count is a multiple of three for most
// l) in each of its eight waves, every wave a part of the length, summed
// through LDS in the order of the parts; the grid adds `chunks` slots of parts
// and the groups of tiles.  Short blocks, since the lengths of one launch differ
// up to eleven times (one block of all tiles with longer parts left CUs with
// two long blocks each).  Bound by the fp64 matrix rate and the blocks' start and
// reduction.  112 matrices of l = 72 and 512 to 5632 columns: 195 -> 86 us per
// launch; 48 of l = 40: 26 -> 19 us; one of l = 264 and 16384 columns: 64 -> 29
// us; one of l = 24: 10 -> 4.6 us (before: fp64 FMAs on 64 x 64 tiles in LDS).
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kGramWaves = 8, kGramTiles = 3;

__global__ void __launch_bounds__(64 * kGramWaves) gram64_kernel(Gram64Items t, int ell_pad, double* partial) {
    __shared__ double red[kGramWaves][kGramTiles * 4][64];
    const int z = blockIdx.z, slot = blockIdx.y;
    const int g = item_of(t, z);
    const int64_t ld = t.ld[g], len = t.len[g];
    const int ell = t.ell, nb = (ell + 15) / 16, nt = nb * (nb + 1) / 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, q = lane >> 4;
    const int t0 = blockIdx.x * kGramTiles;
    // Tile (r, c) of each of this wave's tiles, in row-major upper order.
    int tr[kGramTiles], tc[kGramTiles];
    {
        int w = min(t0, nt - 1), r = 0;
        while (w >= nb - r) { w -= nb - r; ++r; }
        int c = r + w;
#pragma unroll
        for (int u = 0; u < kGramTiles; ++u) {
            tr[u] = r;
            tc[u] = c;
            if (t0 + u + 1 < nt && ++c == nb) { ++r; c = r; }
        }
    }
    const int parts = t.chunks * kGramWaves;
    const int64_t part_len = (len / 16 + parts - 1) / parts * 16;
    const int64_t j0 = (int64_t)(slot * kGramWaves + wave) * part_len, j1 = min(len, j0 + part_len);
    const float* v = t.v[g] + (int64_t)(z - t.zbeg[g]) * t.stride[g];
    const float* pa[kGramTiles];
    const float* pb[kGramTiles];
    float ma[kGramTiles], mb[kGramTiles];   // 0 for rows past l
#pragma unroll
    for (int u = 0; u < kGramTiles; ++u) {
        const int ra = 16 * tr[u] + row, rb = 16 * tc[u] + row;
        pa[u] = v + (int64_t)min(ra, ell - 1) * ld + 4 * q;
        pb[u] = v + (int64_t)min(rb, ell - 1) * ld + 4 * q;
        ma[u] = ra < ell ? 1.f : 0.f;
        mb[u] = rb < ell ? 1.f : 0.f;
    }
    f64x4 acc[kGramTiles];
#pragma unroll
    for (int u = 0; u < kGramTiles; ++u) acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
    float4 a[kGramTiles], b[kGramTiles];
    auto load = [&](int64_t j) {
#pragma unroll
        for (int u = 0; u < kGramTiles; ++u) {
            a[u] = *(const float4*)(pa[u] + j);
            b[u] = *(const float4*)(pb[u] + j);
        }
    };
    if (j0 < j1) load(j0);
    for (int64_t j = j0; j < j1; j += 16) {
        float4 ca[kGramTiles], cb[kGramTiles];
#pragma unroll
        for (int u = 0; u < kGramTiles; ++u) {
            ca[u] = a[u];
            cb[u] = b[u];
        }
        if (j + 16 < j1) load(j + 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < kGramTiles; ++u) {
                const float xa = e == 0 ? ca[u].x : e == 1 ? ca[u].y : e == 2 ? ca[u].z : ca[u].w;
                const float xb = e == 0 ? cb[u].x : e == 1 ? cb[u].y : e == 2 ? cb[u].z : cb[u].w;
                acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(ma[u] != 0.f ? xa : 0.f),
                                                              (double)(mb[u] != 0.f ? xb : 0.f), acc[u], 0, 0, 0);
            }
    }
#pragma unroll
    for (int u = 0; u < kGramTiles; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][4 * u + r][lane] = acc[u][r];
    __syncthreads();
    double* out = partial + ((int64_t)z * t.chunks + slot) * ell_pad * ell_pad;
#pragma unroll
    for (int u = 0; u < kGramTiles; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if ((4 * u + r) % kGramWaves != wave || t0 + u >= nt) continue;
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < kGramWaves; ++k) sum += red[k][4 * u + r][lane];
            out[(int64_t)(16 * tr[u] + q + 4 * r) * ell_pad + 16 * tc[u] + row] = sum;
        }
}

// -------------------------------------------------------- Cholesky + inverse
// One block per matrix.  G = R^T R with R upper triangular; a pivot below
// kDropTol * G_kk (relative to the column's own squared norm) marks the
// column as numerically dependent: its row of R and of R^{-1} is zero, so the
// matching column of Q = Y R^{-1} is zero and it never reaches the selection.
constexpr double kDropTol = 1e-12;
constexpr int kCholRegMax = 192;    // largest l of the register kernel
// fp64 1/sqrt(x) and 1/x for x > 0: the hardware estimates refined by two
// Newton steps, accurate to fp64 rounding with a much shorter dependent chain
// than the IEEE square-root and division sequences (which sit on the
// per-pivot critical path of the factorizations below).
__device__ __forceinline__ double rsqrt_f64(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    y = y * fma(-h * y, y, 1.5);
    return y * fma(-h * y, y, 1.5);
}
__device__ __forceinline__ double rcp_f64(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

// Cholesky and inverse of one l x l matrix per workgroup, l <= kCholG T, all in
// registers: elimination of the rows of [G | I] turns G into (scaled) R and I
// into (scaled) R^{-T}, so the inverse costs no pass of its own.  Thread
// (ti, tj) holds the entries (ti + kCholG a, tj + kCholG b): of the G part the
// tiles a <= b, of the inverse part a >= b.  Two pivots per step: both pivot
// rows go through LDS (two buffers, one barrier per step) and every thread
// eliminates the second by the first for the columns it needs, so the chain
// of a step is one exchange, two reciprocals and a few FMAs.  256 threads: with
// 1024 and a quarter of the entries each, the LDS reads of the pivot row by 16
// waves took twice as long.  Per launch: 48 matrices of l = 40 17 us (45 us with
// the matrix in LDS, one pivot per barrier, and the inverse one column per
// thread); 112 of l = 72 34 us and 22 us for the chunk sums (137 us); one of
// l = 264 in its two-level form 0.2 ms in all (0.73 ms in row panels).
constexpr int kCholG = 16;
constexpr int kGramSum = 4;
constexpr int kCholThreads = kCholG * kCholG;
template <int T>
struct CholRegs {
    double g[T][T], e[T][T];
};
struct CholShared {
    // pivot rows k, k + 1 as [G | inverse], the original diagonal, kept pivots,
    // transposing tile
    double row[2][2][2 * kCholRegMax], diag0[kCholRegMax + 1], pivot[kCholRegMax + 1];
    double tile[2][kCholG][kCholG + 1];
};

template <int T, int A0>
__device__ __forceinline__ void chol_columns(CholRegs<T>& r, CholShared& sh, int& par, int ell) {
    const int tid = threadIdx.x, ti = tid / kCholG, tj = tid % kCholG;
    for (int kk = 0; kk < kCholG; kk += 2, par ^= 1) {
        const int k = kCholG * A0 + kk;
        if (k >= ell) return;
        const double *g0 = sh.row[par][0], *g1 = sh.row[par][1];
        const double *e0 = g0 + kCholRegMax, *e1 = g1 + kCholRegMax;
        const double piv0 = g0[k], a01 = g0[k + 1], a11 = g1[k + 1], d0 = sh.diag0[k], d1 = sh.diag0[k + 1];
        double rg0[T], rg1[T], re0[T], re1[T], rf0[T], rf1[T];
#pragma unroll
        for (int b = A0; b < T; ++b) {
            rg0[b] = g0[tj + kCholG * b];
            rg1[b] = g1[tj + kCholG * b];
            rf0[b] = g0[ti + kCholG * b];
            rf1[b] = g1[ti + kCholG * b];
        }
#pragma unroll
        for (int b = 0; b <= A0; ++b) {
            re0[b] = e0[tj + kCholG * b];
            re1[b] = e1[tj + kCholG * b];
        }
        const bool keep0 = d0 > 0.0 && piv0 > kDropTol * d0;
        const double ip0 = keep0 ? rcp_f64(piv0) : 0.0, f01 = a01 * ip0, piv1 = fma(-f01, a01, a11);
        const bool keep1 = d1 > 0.0 && piv1 > kDropTol * d1;
        const double ip1 = keep1 ? rcp_f64(piv1) : 0.0;
        if (tid == 0) {
            sh.pivot[k] = keep0 ? piv0 : 0.0;
            sh.pivot[k + 1] = keep1 ? piv1 : 0.0;
        }
#pragma unroll
        for (int b = A0; b < T; ++b) {
            rg1[b] = fma(-f01, rg0[b], rg1[b]);
            rf1[b] = fma(-f01, rf0[b], rf1[b]);
        }
#pragma unroll
        for (int b = 0; b <= A0; ++b) re1[b] = fma(-f01, re0[b], re1[b]);
#pragma unroll
        for (int a = A0; a < T; ++a) {
            const double f0 = a > A0 || ti > kk ? rf0[a] * ip0 : 0.0;
            const double f1 = a > A0 || ti > kk + 1 ? rf1[a] * ip1 : 0.0;
#pragma unroll
            for (int b = a; b < T; ++b) r.g[a][b] = fma(-f1, rg1[b], fma(-f0, rg0[b], r.g[a][b]));
#pragma unroll
            for (int b = 0; b <= A0; ++b) r.e[a][b] = fma(-f1, re1[b], fma(-f0, re0[b], r.e[a][b]));
        }
        // The next two pivot rows into the other buffer.
        const int nk = (kk + 2) % kCholG;
        if (ti == nk || ti == nk + 1) {
            double* ng = sh.row[par ^ 1][ti - nk];
            double* ne = ng + kCholRegMax;
            auto put = [&](auto at) {
                constexpr int A1 = decltype(at)::value;
                if constexpr (A1 < T) {
#pragma unroll
                    for (int b = A1; b < T; ++b) ng[tj + kCholG * b] = r.g[A1][b];
#pragma unroll
                    for (int b = 0; b <= A1; ++b) ne[tj + kCholG * b] = r.e[A1][b];
                }
            };
            if (nk > 0) put(std::integral_constant<int, A0>{});
            else put(std::integral_constant<int, A0 + 1>{});
        }
        __syncthreads();
    }
    if constexpr (A0 + 1 < T) chol_columns<T, A0 + 1>(r, sh, par, ell);
}

// The block of order ell at row and column `off` of the l x l matrix: SUM takes
// it (off = 0, the whole matrix) from the chunk partials and also clears the
// rest of rinv, else it is read from src (ld ell_pad); the diagonal that the
// dropping test compares with is always the Gram's own.  x64, when given,
// receives R^{-1} (upper triangle) in fp64.  Entries past ell but inside
// ell_pad are loaded and discarded, so the loads need no branches.  SUM takes
// kGramSum slots.
template <int T, bool SUM>
__global__ void __launch_bounds__(kCholThreads) chol_reg_kernel(const double* src, int64_t stride, int ell,
                                                                int ell_pad, const double* partial, int chunks,
                                                                int off, double* x64, int64_t stride_x, float* rinv) {
    __shared__ CholShared sh;
    const int z = blockIdx.x, tid = threadIdx.x, ti = tid / kCholG, tj = tid % kCholG;
    const double* part = partial + (int64_t)z * chunks * ell_pad * ell_pad;
    const double* p = SUM ? part : src + (int64_t)z * stride;
    CholRegs<T> r;
    for (int q = tid; q < 2 * 2 * 2 * kCholRegMax; q += kCholThreads) (&sh.row[0][0][0])[q] = 0.0;
    if (tid <= kCholRegMax) sh.diag0[tid] = !SUM && tid < ell ? gram_at(part, ell_pad, off + tid, off + tid, chunks) : 0.0;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < T; ++a) {
#pragma unroll
        for (int b = a; b < T; ++b) {
            const int i = ti + kCholG * a, j = tj + kCholG * b;
            const int c = min(min(i, j), ell - 1), d = min(max(i, j), ell - 1);
            double v = 0.0;
            const double* q = p + (int64_t)c * ell_pad + d;
            if constexpr (SUM) {
                double w[kGramSum];
#pragma unroll
                for (int u = 0; u < kGramSum; ++u) w[u] = q[(int64_t)u * ell_pad * ell_pad];
#pragma unroll
                for (int u = 0; u < kGramSum; ++u) v += w[u];
            } else {
                v = q[0];
            }
            r.g[a][b] = j < ell && i < ell ? v : 0.0;
            if (SUM && a == b && i == j && j < ell) sh.diag0[j] = v;
        }
    }
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) r.e[a][b] = a == b && ti == tj ? 1.0 : 0.0;
    __syncthreads();
    if (ti < 2) {
#pragma unroll
        for (int b = 0; b < T; ++b) sh.row[0][ti][tj + kCholG * b] = r.g[0][b];
        sh.row[0][ti][kCholRegMax + tj] = r.e[0][0];
    }
    __syncthreads();
    int par = 0;
    chol_columns<T, 0>(r, sh, par, ell);
    // R^{-1}(j, i) = e(i, j) / sqrt(pivot i), transposed through LDS by tiles.
    float* out = rinv + (int64_t)z * ell_pad * ell_pad;
    double* xo = x64 ? x64 + (int64_t)z * stride_x : nullptr;
    __syncthreads();
    int flip = 0;
#pragma unroll
    for (int a = 0; a < T; ++a) {
        if (kCholG * a >= ell) break;
        const int i = ti + kCholG * a;
        const double pv = i < ell ? sh.pivot[i] : 0.0, s = pv > 0.0 ? rsqrt_f64(pv) : 0.0;
#pragma unroll
        for (int b = 0; b <= a; ++b, flip ^= 1) {
            sh.tile[flip][tj][ti] = r.e[a][b] * s;
            __syncthreads();
            const int jo = kCholG * b + ti, io = kCholG * a + tj;      // row, column of R^{-1}
            if (jo <= io && io < ell) {
                const double v = sh.tile[flip][ti][tj];
                out[(int64_t)jo * ell_pad + io] = (float)v;
                if (xo) xo[(int64_t)jo * ell_pad + io] = v;
            }
        }
    }
    if (SUM)
        for (int q = tid; q < ell_pad * ell_pad; q += kCholThreads) {
            const int i = q / ell_pad, j = q - (q / ell_pad) * ell_pad;
            if (!(i <= j && j < ell)) out[q] = 0.f;
        }
}

// Dense G (upper triangle, ld ell_pad) from the chunk partials in many blocks;
// zeros in the lower triangle of x (R^{-1} in fp64) and in the entries of rinv
// outside the upper triangle.
__global__ void __launch_bounds__(256) chol_sum_kernel(const double* partial, int chunks, int ell, int ell_pad, double* g,
                                                       double* x, int64_t stride, float* rinv) {
    const int z = blockIdx.y, q = blockIdx.x * 256 + threadIdx.x;
    if (q >= ell_pad * ell_pad) return;
    const int i = q / ell_pad, j = q - (q / ell_pad) * ell_pad;
    const double* p = partial + (int64_t)z * chunks * ell_pad * ell_pad;
    if (i <= j && j < ell) {
        g[(int64_t)z * stride + q] = gram_at(p, ell_pad, i, j, chunks);
    } else {
        x[(int64_t)z * stride + q] = 0.0;
        rinv[(int64_t)z * ell_pad * ell_pad + q] = 0.f;
    }
}

// C = C0 +- A B in fp64 for the blocks of a two-level factorization: A(i, k) =
// a[i ai + k ak], B(k, j) = b[k bk + j bj], C at c[i ldc + j] (and / or fp32 c32).
// 32 x 32 output tiles, 2 x 2 per thread.
struct SmallDgemm {
    const double* a; int64_t ai, ak, stride_a;
    const double* b; int64_t bk, bj, stride_b;
    const double* c0; int64_t ldc0, stride_c0;  // null: 0
    double sign;
    double* c; int64_t ldc, stride_c;           // may be null
    float* c32; int64_t ldc32, stride_c32;      // may be null
    int m, n, k;
};
__global__ void __launch_bounds__(256) small_dgemm_kernel(SmallDgemm p) {
    __shared__ double as[32][33], bs[32][33];   // [k][i], [k][j]
    const int z = blockIdx.z, i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    const double* a = p.a + (int64_t)z * p.stride_a;
    const double* b = p.b + (int64_t)z * p.stride_b;
    double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
    double ra[4], rb[4];        // the next slab, in flight during this one's FMAs
    auto load = [&](int k0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int q = tid + 256 * t, hi = q >> 5, lo = q & 31;
            // The unit-stride index along the lanes; clamped, then masked.
            const int ka = k0 + (p.ai == 1 ? hi : lo), ia = i0 + (p.ai == 1 ? lo : hi);
            const int kb = k0 + (p.bj == 1 ? hi : lo), jb = j0 + (p.bj == 1 ? lo : hi);
            const double va = a[min(ia, p.m - 1) * p.ai + min(ka, p.k - 1) * p.ak];
            const double vb = b[min(kb, p.k - 1) * p.bk + min(jb, p.n - 1) * p.bj];
            ra[t] = ia < p.m && ka < p.k ? va : 0.0;
            rb[t] = jb < p.n && kb < p.k ? vb : 0.0;
        }
    };
    load(0);
    for (int k0 = 0; k0 < p.k; k0 += 32) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int q = tid + 256 * t, hi = q >> 5, lo = q & 31;
            as[p.ai == 1 ? hi : lo][p.ai == 1 ? lo : hi] = ra[t];
            bs[p.bj == 1 ? hi : lo][p.bj == 1 ? lo : hi] = rb[t];
        }
        __syncthreads();
        if (k0 + 32 < p.k) load(k0 + 32);
#pragma unroll 8
        for (int k = 0; k < 32; ++k) {
            const double x0 = as[k][ty], x1 = as[k][ty + 16], y0 = bs[k][tx], y1 = bs[k][tx + 16];
            acc[0][0] = fma(x0, y0, acc[0][0]);
            acc[0][1] = fma(x0, y1, acc[0][1]);
            acc[1][0] = fma(x1, y0, acc[1][0]);
            acc[1][1] = fma(x1, y1, acc[1][1]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int i = i0 + ty + 16 * u, j = j0 + tx + 16 * v;
            if (i >= p.m || j >= p.n) continue;
            double x = p.sign * acc[u][v];
            if (p.c0) x += p.c0[(int64_t)z * p.stride_c0 + i * p.ldc0 + j];
            if (p.c) p.c[(int64_t)z * p.stride_c + i * p.ldc + j] = x;
            if (p.c32) p.c32[(int64_t)z * p.stride_c32 + i * p.ldc32 + j] = (float)x;
        }
}

// ------------------------------------------------------------- M^T V ----
// out(c, j) = sum_d M(d, c) V(d, j), d < l, c < l_pad, j < len.  Block: a
// 64 (c) x 128 (j) output tile, 256 threads of 4 c x 8 j each (j in two runs
// of four, 64 apart, so a row of the tile is 16 threads x 16 B contiguous).
// The l dimension runs in chunks of 16 staged through LDS, the next chunk's
// global loads in flight during the current chunk's FMAs.  Every d sums in
// increasing order, one fp32 FMA per term.  len and the row strides of V and
// the outputs are multiples of 128 (the 256-padded matrix sides), l_pad of 64.
constexpr int kSmBM = 64, kSmBN = 128, kSmBK = 16;

__global__ void __launch_bounds__(256) small_mul_kernel(SmallMulArgs args) {
    const int z = blockIdx.z;
    const int g = item_of(args, z), lz = z - args.zbeg[g];
    const SmallMulItem& a = args.it[g];
    const int64_t j0 = (int64_t)blockIdx.x * kSmBN;
    if (j0 >= a.len_pad) return;
    const int c0 = blockIdx.y * kSmBM;
    const int ell = args.ell, ell_pad = args.ell_pad;
    const int tid = threadIdx.x, tc = tid >> 4, tj = tid & 15;
    const float* M = a.mat + (int64_t)lz * ell_pad * ell_pad;
    const float* V = a.v + (int64_t)lz * a.stride_v;
    __shared__ float4 sm[kSmBK][kSmBM / 4];
    __shared__ float4 sv[kSmBK][kSmBN / 4];
    // Global -> register staging: one float4 of M, two of V per thread.
    const int mr = tid >> 4, mc = tid & 15;           // M: row, float4 column
    const int vr = tid >> 5, vc = tid & 31;           // V: rows vr, vr + 8
    float4 rm, rv0, rv1;
    auto load = [&](int d0) {
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        const int dm = d0 + mr, dv0 = d0 + vr, dv1 = d0 + vr + 8;
        rm = dm < ell ? *(const float4*)(M + (int64_t)dm * ell_pad + c0 + 4 * mc) : zero;
        rv0 = dv0 < ell ? *(const float4*)(V + (int64_t)dv0 * a.ld_v + j0 + 4 * vc) : zero;
        rv1 = dv1 < ell ? *(const float4*)(V + (int64_t)dv1 * a.ld_v + j0 + 4 * vc) : zero;
    };
    auto stage = [&]() {
        sm[mr][mc] = rm;
        sv[vr][vc] = rv0;
        sv[vr + 8][vc] = rv1;
    };
    float acc[4][8];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[u][e] = 0.f;
    load(0);
    stage();
    __syncthreads();
    for (int d0 = 0; d0 < ell; d0 += kSmBK) {
        const bool more = d0 + kSmBK < ell;
        if (more) load(d0 + kSmBK);
#pragma unroll 4
        for (int dd = 0; dd < kSmBK; ++dd) {
            const float4 m4 = sm[dd][tc];
            const float4 va = sv[dd][tj], vb = sv[dd][16 + tj];
            const float mv[4] = {m4.x, m4.y, m4.z, m4.w};
            const float vv[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[u][e] = fmaf(mv[u], vv[e], acc[u][e]);
        }
        if (more) {
            __syncthreads();
            stage();
            __syncthreads();
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = c0 + 4 * tc + u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t j = j0 + 64 * h + 4 * tj;
            const float* q = acc[u] + 4 * h;
            if (a.out32)
                *(float4*)(a.out32 + (int64_t)lz * a.stride_out32 + (int64_t)c * a.ld_v + j) =
                    make_float4(q[0], q[1], q[2], q[3]);
            if (a.out16) {
                half_t* o = a.out16 + (int64_t)lz * a.stride_out16 + (int64_t)c * a.ld_v + j;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (half_t)q[e];
            }
        }
    }
    if (a.out16t) {
        // len-major: row j holds l_pad consecutive c; four of them per store.
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t j = j0 + 64 * h + 4 * tj + e;
                half_t* o = a.out16t + (int64_t)lz * a.stride_out16t + j * ell_pad + c0 + 4 * tc;
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = (half_t)acc[u][4 * h + e];
            }
    }
}

}  // namespace

hipError_t launch_omega_f16(const OmegaArgs& a, hipStream_t s) {
    if (a.n < 1 || a.n > kMaxItems || a.zbeg[0] != 0 || a.zbeg[a.n] > kOmegaIds) return hipErrorInvalidValue;
    int64_t most = 0;
    for (int g = 0; g < a.n; ++g) {
        if (a.zbeg[g + 1] <= a.zbeg[g] || a.ld[g] % 4 || a.stride[g] % 4) return hipErrorInvalidValue;
        most = std::max(most, (int64_t)a.ell_pad * a.ld[g] / 4);
    }
    const unsigned blocks = (unsigned)std::min<int64_t>((most + 255) / 256, 1024);
    hipLaunchKernelGGL(omega_f16_kernel, dim3(blocks, a.zbeg[a.n]), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_omega_f32(uint64_t seed, int64_t step, int id, int64_t b, int ell, float* out, hipStream_t s) {
    const int64_t total = b * ell;
    const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(omega_f32_kernel, dim3(blocks), dim3(256), 0, s, seed, step, (uint32_t)id, b, ell, out);
    return hipGetLastError();
}

hipError_t launch_reduce_splits(const float* part, int splits, int64_t stride_split, int64_t stride_mat, int rows,
                                int64_t len, float* out32, half_t* out16, float scale16, int64_t stride_out,
                                int batch, hipStream_t s) {
    if (len % 4 || stride_split % 4) return hipErrorInvalidValue;
    const int64_t n4 = (int64_t)rows * len / 4;
    const unsigned blocks = (unsigned)std::min<int64_t>((n4 + 255) / 256, 2048);
    hipLaunchKernelGGL(reduce_splits_kernel, dim3(blocks, batch), dim3(256), 0, s, part, splits, stride_split,
                       stride_mat, n4, out32, out16, scale16, stride_out);
    return hipGetLastError();
}

hipError_t launch_reduce_splits_grouped(const ReduceGroups& g, hipStream_t s) {
    if (g.n < 1 || g.n > kMaxItems || g.zbeg[0] != 0) return hipErrorInvalidValue;
    int64_t n4 = 0;
    for (int i = 0; i < g.n; ++i) {
        if (g.zbeg[i + 1] <= g.zbeg[i] || g.splits[i] < 1 || g.stride_split[i] % 4 || g.n4[i] < 1)
            return hipErrorInvalidValue;
        n4 = std::max(n4, g.n4[i]);
    }
    const unsigned blocks = (unsigned)std::min<int64_t>((n4 + 255) / 256, 2048);
    hipLaunchKernelGGL(reduce_splits_grouped_kernel, dim3(blocks, g.zbeg[g.n]), dim3(256), 0, s, g);
    return hipGetLastError();
}

// Slots of the partial sums: 4 (32 parts of the length), or 16 for few long
// matrices, whose parts' chains would leave the chip idle.
static int gram_groups(int ell) {
    const int nb = (ell + 15) / 16;
    return (nb * (nb + 1) / 2 + kGramTiles - 1) / kGramTiles;
}
int gram64_slots(int ell, int count, int64_t max_len) {
    return (int64_t)count * gram_groups(ell) * 4 * kGramWaves < 1024 && max_len > 4096 ? kGramChunks : 4;
}

int64_t gram64_slots_all(int ell, int count, int64_t max_len) {
    const int64_t few = std::min<int64_t>(count, 1023 / (gram_groups(ell) * 4 * kGramWaves));
    return std::max((int64_t)count * gram64_slots(ell, count, max_len),
                    few > 0 ? few * gram64_slots(ell, (int)few, max_len) : 0);
}

hipError_t launch_gram64(const Gram64Items& t, int ell_pad, double* partial, hipStream_t s) {
    if (ell_pad % 64 || t.ell < 1 || t.ell > ell_pad || t.n < 1 || t.n > kMaxItems || t.zbeg[0] != 0 ||
        t.chunks < 1 || t.chunks > kGramChunks)
        return hipErrorInvalidValue;
    for (int g = 0; g < t.n; ++g)
        if (t.len[g] % 16 || t.ld[g] % 4 || t.stride[g] % 4 || t.zbeg[g + 1] <= t.zbeg[g]) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gram64_kernel, dim3(gram_groups(t.ell), t.chunks, t.zbeg[t.n]), dim3(64 * kGramWaves), 0, s, t,
                       ell_pad, partial);
    return hipGetLastError();
}

hipError_t launch_chol_inv(const double* partial, int chunks, int ell, int ell_pad, double* scratch, float* rinv,
                           int batch, hipStream_t s) {
    if (ell < 1 || ell > 384 || ell_pad < ell || ell_pad > 384 || chunks < 1 || chunks > kGramChunks)
        return hipErrorInvalidValue;
    const int64_t lp2 = (int64_t)ell_pad * ell_pad, ld = ell_pad;
    // Up to 96 the workgroup sums few slots itself, its loads all in flight;
    // otherwise many blocks do in a launch of their own.
    if (ell <= 96 && chunks == kGramSum) {
        auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(batch), dim3(kCholThreads), 0, s, (const double*)nullptr, (int64_t)0, ell,
                               ell_pad, partial, chunks, 0, (double*)nullptr, (int64_t)0, rinv);
        };
        switch ((ell + kCholG - 1) / kCholG) {
            case 1: run(chol_reg_kernel<1, true>); break;
            case 2: run(chol_reg_kernel<2, true>); break;
            case 3: run(chol_reg_kernel<3, true>); break;
            case 4: run(chol_reg_kernel<4, true>); break;
            case 5: run(chol_reg_kernel<5, true>); break;
            default: run(chol_reg_kernel<6, true>); break;
        }
        return hipGetLastError();
    }
    // scratch per matrix: G, then X = R^{-1} (ell_pad^2 doubles each).
    const int64_t st = 2 * lp2;
    double *G = scratch, *X = scratch + lp2;
    hipLaunchKernelGGL(chol_sum_kernel, dim3((unsigned)((lp2 + 255) / 256), batch), dim3(256), 0, s, partial, chunks,
                       ell, ell_pad, G, X, st, rinv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto factor = [&](int off, int n, const double* src, bool x64) {
        auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(batch), dim3(kCholThreads), 0, s, src, st, n, ell_pad, partial, chunks,
                               off, x64 ? X + off * (ld + 1) : nullptr, st, rinv + off * (ld + 1));
        };
        switch ((n + 2 * kCholG - 1) / (2 * kCholG)) {
            case 1: run(chol_reg_kernel<2, false>); break;
            case 2: run(chol_reg_kernel<4, false>); break;
            case 3: run(chol_reg_kernel<6, false>); break;
            case 4: run(chol_reg_kernel<8, false>); break;
            case 5: run(chol_reg_kernel<10, false>); break;
            default: run(chol_reg_kernel<12, false>); break;
        }
        return hipGetLastError();
    };
    if (ell <= kCholRegMax) return factor(0, ell, G, false);
    // Two levels: [G11 G12; . G22], about half the rows each (a pivot of a
    // smaller block costs less).
    //   R12 = R11^{-T} G12 (kept transposed under G11), S = G22 - R12^T R12,
    //   X12 = -X11 (R12 X22).
    const int l1 = (int)round_up((ell + 1) / 2, kCholG), l2 = ell - l1;
    double* G12 = G + l1;                           // then R12 X22
    double* R12t = G + (int64_t)l1 * ld;            // l2 x l1
    double* G22 = G + (int64_t)l1 * (ld + 1);       // then S
    double* X22 = X + (int64_t)l1 * (ld + 1);
    auto gemm = [&](const double* ga, int64_t ai, int64_t ak, const double* gb, int64_t bk, int64_t bj,
                    const double* c0, double sign, double* c, float* c32, int m, int n, int k) {
        const SmallDgemm p{ga, ai, ak, st, gb, bk, bj, st, c0, ld, st, sign, c, ld, st, c32, ld, lp2, m, n, k};
        hipLaunchKernelGGL(small_dgemm_kernel, dim3((n + 31) / 32, (m + 31) / 32, batch), dim3(256), 0, s, p);
        return hipGetLastError();
    };
    e = factor(0, l1, G, true);
    if (e == hipSuccess) e = gemm(G12, 1, ld, X, ld, 1, nullptr, 1.0, R12t, nullptr, l2, l1, l1);
    if (e == hipSuccess) e = gemm(R12t, ld, 1, R12t, 1, ld, G22, -1.0, G22, nullptr, l2, l2, l1);
    if (e == hipSuccess) e = factor(l1, l2, G22, true);
    if (e == hipSuccess) e = gemm(R12t, 1, ld, X22, ld, 1, nullptr, 1.0, G12, nullptr, l1, l2, l2);
    if (e == hipSuccess) e = gemm(X, ld, 1, G12, ld, 1, nullptr, -1.0, nullptr, rinv + l1, l1, l2, l1);
    return e;
}

hipError_t launch_small_mul(const SmallMulArgs& a, hipStream_t s) {
    if (a.n < 1 || a.n > kMaxItems || a.zbeg[0] != 0) return hipErrorInvalidValue;
    if (a.ell < 1 || a.ell > a.ell_pad || a.ell_pad % kSmBM) return hipErrorInvalidValue;
    int64_t len_pad = 0;
    for (int g = 0; g < a.n; ++g) {
        const SmallMulItem& m = a.it[g];
        if (a.zbeg[g + 1] <= a.zbeg[g] || m.len_pad % kSmBN || m.ld_v % kSmBN || m.ld_v < m.len_pad)
            return hipErrorInvalidValue;
        len_pad = std::max(len_pad, m.len_pad);
    }
    dim3 grid((unsigned)(len_pad / kSmBN), (unsigned)(a.ell_pad / kSmBM), a.zbeg[a.n]);
    hipLaunchKernelGGL(small_mul_kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace np
