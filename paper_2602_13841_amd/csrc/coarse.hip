// Direct solver of the coarsest multigrid level: the inverse of the dense FP64
// coarse matrix, formed once per Newton state over the whole device, and its
// application in one launch per V-cycle.
//
// Inversion: blocked Gauss-Jordan elimination with partial pivoting, in place.
// For the panel J of nb columns, with D the (pivoted) diagonal block, B the
// rows J and C the columns J of the rest:
//     A_JJ <- D^{-1},  A_J. <- D^{-1} B,  A_.J <- W = -C D^{-1},  A <- A + W B,
// so every panel is three launches: the pivot search on the panel (one
// workgroup, rows in registers), the row interchanges with W and B (whole
// device), and one rank-nb update of the whole matrix on MFMA.  With the row
// permutation P the result is (P A)^{-1}; its application gathers the
// right-hand side through P.  The error against the exact solution is that of
// the LU substitution (measured on 2D/3D coarse matrices of 126 to 2276
// unknowns, condition 5e3 to 3e6: 0.3 to 1.9 times it).
//
// Against the LU it replaced (panel in global memory, 25 us per column at
// m = 2274; one workgroup per substitution): the factorization was bound by
// the latency of its panel columns, the substitution by one CU's.
#include "vanka.h"

#include "stmg_internal.h"

#include <type_traits>
#include <utility>

namespace stmg {

namespace {

typedef double doublex4_t __attribute__((ext_vector_type(4)));

// f(0), f(1), ... with compile-time arguments (register arrays indexed by them
// stay in registers however long the unrolled code gets)
template <int... I, typename F> __device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// wavefront maximum by DPP (rows of 16 lanes, then across the rows), as a
// uniform value
__device__ __forceinline__ double wave_max(double v)
{
    auto step = [](double x, auto dpp) {
        const long long b = __double_as_longlong(x);
        const int lo = dpp((int)(b & 0xffffffff)), hi = dpp((int)(b >> 32));
        return fmax(x, __longlong_as_double(((long long)hi << 32) | (unsigned)lo));
    };
    v = step(v, [](int x) { return __builtin_amdgcn_update_dpp(x, x, 0x111, 0xf, 0xf, false); });   // row_shr 1
    v = step(v, [](int x) { return __builtin_amdgcn_update_dpp(x, x, 0x112, 0xf, 0xf, false); });   // row_shr 2
    v = step(v, [](int x) { return __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false); });   // row_shr 4
    v = step(v, [](int x) { return __builtin_amdgcn_update_dpp(x, x, 0x118, 0xf, 0xf, false); });   // row_shr 8
    // lanes 15, 31, 47, 63 hold the maxima of their rows
    const long long b = __double_as_longlong(v);
    double r = -1.0;
#pragma unroll
    for (int l = 15; l < 64; l += 16) {
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
        const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
        r = fmax(r, __longlong_as_double(((long long)hi << 32) | (unsigned)lo));
    }
    return r;
}

// ---------------------------------------------------------------------------
// Pivots and D^{-1} of one panel: columns [j0, j0 + nb), candidate rows
// [j0, m), each thread RPT rows of NB columns in registers (RPT NTH >= m - j0).
// Rows stay where they are; a thread tracks the logical position of its rows
// under the interchanges.  Two barriers per column (candidates of the
// wavefronts; the pivot row).  Latency bound: 0.3-0.5 us per column.
// Writes rowsrc[i] = row that the interchanges bring to position i >= j0, the
// accumulated permutation perm, and D^{-1} (NB x NB, zero padded); A is only
// read.
// ---------------------------------------------------------------------------
template <int NB, int RPT, int NTH>
__global__ void __launch_bounds__(NTH) inv_panel_kernel(const double *__restrict__ A, int m, int ld, int j0, int nb,
                                                        double *__restrict__ dinv, int *__restrict__ rowsrc,
                                                        int *__restrict__ perm)
{
    constexpr int NW = NTH / 64;
    __shared__ double wval[NW];
    __shared__ int wlog[NW];
    __shared__ double prow[NB];
    __shared__ double Dt[NB][NB];   // transposed: Dt[column][row]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int mr = m - j0;
    double a[RPT][NB];
    int lg[RPT];
    unsigned open = 0;   // rows that are not pivotal yet
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = tid + i * NTH;
        lg[i] = r;
        if (r < mr) open |= 1u << i;
        const double *src = A + (long long)(j0 + min(r, mr - 1)) * ld + j0;
#pragma unroll
        for (int k = 0; k < NB; ++k) a[i][k] = src[min(k, nb - 1)];
    }
    auto column = [&](auto cc) {
        constexpr int c = decltype(cc)::value;
        if (c >= nb) return;
        double best = -1.0;
        int bl = 0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const double v = fabs(a[i][c]);
            if (((open >> i) & 1u) && v > best) {
                best = v;
                bl = lg[i];
            }
        }
        const double wm = wave_max(best);
        const unsigned long long hit = __ballot(best == wm);
        if (lane == __builtin_ctzll(hit | (1ull << 63))) {
            wval[wv] = wm;
            wlog[wv] = bl;
        }
        __syncthreads();
        // a column without a comparable entry (all NaN) keeps its own row
        double bv = -1.0;
        int p = c;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const double v = wval[w];
            if (v > bv) {
                bv = v;
                p = wlog[w];
            }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (((open >> i) & 1u) && lg[i] == p) {
#pragma unroll
                for (int k = c; k < NB; ++k) prow[k] = a[i][k];
            }
        __syncthreads();
        const double d = prow[c];
        const double inv = d != 0.0 ? 1.0 / d : 0.0;
        double l[RPT];
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const bool op = (open >> i) & 1u, piv = op && lg[i] == p;
            if (op && !piv) a[i][c] *= inv;
            l[i] = op && !piv ? a[i][c] : 0.0;   // pivotal rows stay
            if (op && !piv && lg[i] == c) lg[i] = p;
            if (piv) {
                lg[i] = c;
                open &= ~(1u << i);
            }
        }
#pragma unroll
        for (int k = c + 1; k < NB; ++k) {
            const double u = prow[k];
#pragma unroll
            for (int i = 0; i < RPT; ++i) a[i][k] -= l[i] * u;
        }
    };
    static_for(std::make_integer_sequence<int, NB>{}, column);
    int before[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = tid + i * NTH;
        if (r < mr) {
            before[i] = j0 == 0 ? r : perm[j0 + r];
            rowsrc[j0 + lg[i]] = j0 + r;
            if (lg[i] < nb) {
#pragma unroll
                for (int k = 0; k < NB; ++k) Dt[k][lg[i]] = a[i][k];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPT; ++i)
        if (tid + i * NTH < mr) perm[j0 + lg[i]] = before[i];
    // D^{-1} = U^{-1} L^{-1}, one column per lane
    if (tid < NB) {
        double y[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) y[c] = c == tid ? 1.0 : 0.0;
        // (identity beyond nb)
        static_for(std::make_integer_sequence<int, NB>{}, [&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if (k < nb) {
#pragma unroll
                for (int c = k + 1; c < NB; ++c) y[c] -= Dt[k][c] * y[k];
            }
        });
        static_for(std::make_integer_sequence<int, NB>{}, [&](auto kk) {
            constexpr int k = NB - 1 - decltype(kk)::value;
            if (k < nb) {
                y[k] /= Dt[k][k];
#pragma unroll
                for (int c = 0; c < k; ++c) y[c] -= Dt[k][c] * y[k];
            }
        });
#pragma unroll
        for (int c = 0; c < NB; ++c) dinv[c * NB + tid] = c < nb && tid < nb ? y[c] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Interchanges, W and B of one panel.  Blocks [0, wblk): 64 rows of W each,
// W_i = -A_{src(i) J} D^{-1} (rows of J: D^{-1}); the others: one column
// outside J per thread, rows J of the permuted matrix to B and the rows that
// the pivots came from refilled with the rows they replaced.
// ---------------------------------------------------------------------------
template <int NB>
__global__ void __launch_bounds__(256) inv_swap_kernel(double *__restrict__ A, int m, int ld, int j0, int nb,
                                                       const double *__restrict__ dinv,
                                                       const int *__restrict__ rowsrc, double *__restrict__ W,
                                                       double *__restrict__ B, int wblk)
{
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < wblk) {
        __shared__ double D[NB][NB];
        __shared__ double C[64][NB + 1];
        const int i0 = blockIdx.x * 64;
        for (int e = tid; e < NB * NB; e += 256) D[e / NB][e % NB] = dinv[e];
        for (int e = tid; e < 64 * NB; e += 256) {
            const int i = e / NB, k = e % NB, row = i0 + i;
            double v = 0.0;
            if (row < m && k < nb) v = A[(long long)(row < j0 ? row : rowsrc[row]) * ld + j0 + k];
            C[i][k] = v;
        }
        __syncthreads();
        constexpr int KT = NB / 4;   // outputs per thread
        const int i = tid >> 2, q = (tid & 3) * KT, row = i0 + i;
        if (row >= m) return;
        double s[KT];
        if (row >= j0 && row < j0 + nb) {
#pragma unroll
            for (int k = 0; k < KT; ++k) s[k] = D[row - j0][q + k];
        } else {
#pragma unroll
            for (int k = 0; k < KT; ++k) s[k] = 0.0;
#pragma unroll 4
            for (int j = 0; j < NB; ++j) {
                const double c = C[i][j];
#pragma unroll
                for (int k = 0; k < KT; ++k) s[k] -= c * D[j][q + k];
            }
        }
#pragma unroll
        for (int k = 0; k < KT; ++k) W[(long long)row * NB + q + k] = s[k];
        return;
    }
    const int col = (blockIdx.x - wblk) * 256 + tid;
    if (col >= m || (col >= j0 && col < j0 + nb)) return;
    double b[NB], v[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        b[k] = v[k] = 0.0;
        if (k < nb) {
            const int s = rowsrc[j0 + k];
            b[k] = A[(long long)s * ld + col];
            if (s >= j0 + nb) v[k] = A[(long long)rowsrc[s] * ld + col];
        }
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        B[(long long)k * ld + col] = b[k];
        if (k < nb) {
            const int s = rowsrc[j0 + k];
            if (s >= j0 + nb) A[(long long)s * ld + col] = v[k];
        }
    }
}

// ---------------------------------------------------------------------------
// A <- A + W B (rows J: W B alone; columns J: W), one 32 x 32 tile per
// wavefront on v_mfma_f64_16x16x4f64 (A lane l -> (row l%16, k l/16), B lane
// l -> (k l/16, col l%16), D register i -> (row l/16 + 4i, col l%16)).  Bound
// by the read and write of A; W (m x nb) and B stay in L2.
// ---------------------------------------------------------------------------
template <int NB>
__global__ void __launch_bounds__(256) inv_update_kernel(double *__restrict__ A, int m, int ld, int j0, int nb,
                                                         const double *__restrict__ W, const double *__restrict__ B)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int nt = (m + 31) / 32, t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= nt * nt) return;
    const int R = (t / nt) * 32, C = (t % nt) * 32;
    doublex4_t acc[2][2];
#pragma unroll
    for (int si = 0; si < 2; ++si)
#pragma unroll
        for (int sj = 0; sj < 2; ++sj)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = R + 16 * si + g + 4 * i;
                const bool keep = row < m && !(row >= j0 && row < j0 + nb);
                acc[si][sj][i] = keep ? A[(long long)row * ld + C + 16 * sj + l16] : 0.0;
            }
    double a[NB / 4][2], b[NB / 4][2];
#pragma unroll
    for (int k = 0; k < NB / 4; ++k)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            a[k][s] = W[(long long)(R + 16 * s + l16) * NB + 4 * k + g];
            b[k][s] = B[(long long)(4 * k + g) * ld + C + 16 * s + l16];
        }
#pragma unroll
    for (int k = 0; k < NB / 4; ++k)
#pragma unroll
        for (int si = 0; si < 2; ++si)
#pragma unroll
            for (int sj = 0; sj < 2; ++sj)
                acc[si][sj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k][si], b[k][sj], acc[si][sj], 0, 0, 0);
#pragma unroll
    for (int si = 0; si < 2; ++si)
#pragma unroll
        for (int sj = 0; sj < 2; ++sj)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = R + 16 * si + g + 4 * i, col = C + 16 * sj + l16;
                if (row < m) {
                    const bool inj = col >= j0 && col < j0 + nb;
                    A[(long long)row * ld + col] = inj ? W[(long long)row * NB + col - j0] : acc[si][sj][i];
                }
            }
}

// d = (inverse) r on the first n rows: the right-hand side gathered through
// the row permutation into LDS (border rows have a zero right-hand side), one
// wavefront per row of the inverse (two rows for large systems), summed in a
// fixed order.  Bound by the read of the inverse.
template <typename T, int ROWS>
__global__ void __launch_bounds__(256) inv_apply_kernel(const double *__restrict__ A, int m, int ld, int n,
                                                        const int *__restrict__ perm, const T *__restrict__ r,
                                                        T *__restrict__ d)
{
    extern __shared__ unsigned char lds_raw[];
    double *b = reinterpret_cast<double *>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    for (int j = tid; j < m; j += 256) {
        const int p = perm[j];
        b[j] = p < n ? (double)r[p] : 0.0;
    }
    __syncthreads();
    const int row0 = (blockIdx.x * 4 + (tid >> 6)) * ROWS;
    double s[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) s[i] = 0.0;
#pragma unroll 4
    for (int j = lane; j < m; j += 64) {
        const double x = b[j];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) s[i] += A[(long long)min(row0 + i, m - 1) * ld + j] * x;
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        for (int off = 32; off > 0; off >>= 1) s[i] += __shfl_xor(s[i], off, 64);
        if (lane == 0 && row0 + i < n) d[row0 + i] = (T)s[i];
    }
}

// coarse matrix from the columns J e_i (row i of Y) and the border of
// constant pressures: transposed through LDS, 32 x 32 tiles
__global__ void __launch_bounds__(256) inv_matrix_kernel(const double *__restrict__ Y, int n, int nb, long long pbase,
                                                         long long Np1, int npm, double *__restrict__ A, int ld)
{
    __shared__ double t[32][33];
    const int m = n + nb, r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int i = ty; i < 32; i += 8) {
        const int col = c0 + i, row = r0 + tx;   // Y holds column col in its row
        t[i][tx] = row < n && col < n ? Y[(long long)col * n + row] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int i = ty; i < 32; i += 8) {
        const int row = r0 + i, col = c0 + tx;
        if (row >= m) continue;
        double v = t[tx][i];
        const int a = (row >= n) != (col >= n && col < m) ? max(row, col) - n : -1;
        if (a >= 0 && col < m) {
            const long long q = min(row, col) - pbase;
            v = q >= a * Np1 && q < (a + 1) * Np1 && (q - a * Np1) % npm == 0 ? 1.0 : 0.0;
        }
        A[(long long)row * ld + col] = v;
    }
}

} // namespace

hipError_t launch_inv_matrix(const double *Y, int n, int nb, long long pbase, long long Np1, int npm, double *A,
                             int ld, hipStream_t s)
{
    const unsigned nt = (unsigned)((n + nb + 31) / 32);
    hipLaunchKernelGGL(inv_matrix_kernel, dim3(nt, nt), dim3(256), 0, s, Y, n, nb, pbase, Np1, npm, A, ld);
    return hipGetLastError();
}

hipError_t launch_dense_inverse(const DenseInverse &w, hipStream_t s)
{
    const int m = w.m, ld = w.ld;
    if (m <= 0) return hipSuccess;
    if (m > DINV_MAX_M) return hipErrorInvalidValue;
    const int wblk = (m + 63) / 64, cblk = (m + 255) / 256, nt = (m + 31) / 32, ublk = (nt * nt + 3) / 4;
    for (int j0 = 0; j0 < m;) {
        // the widest panel whose candidate rows fit the registers of one
        // workgroup (RPT NB doubles per thread: 192 registers at 8 wavefronts,
        // 96 at 16), and the fewest wavefronts that hold them
        const int mr = m - j0;
        int nb = 0;
#define STMG_PANEL(NB, RPT, NTH)                                                                                       \
    {                                                                                                                  \
        nb = min(NB, mr);                                                                                              \
        hipLaunchKernelGGL((inv_panel_kernel<NB, RPT, NTH>), dim3(1), dim3(NTH), 0, s, (const double *)w.A, m, ld, j0, \
                           nb, w.dinv, w.rowsrc, w.perm);                                                              \
    }
#define STMG_REST(NB)                                                                                                  \
    {                                                                                                                  \
        hipLaunchKernelGGL(inv_swap_kernel<NB>, dim3(wblk + cblk), dim3(256), 0, s, w.A, m, ld, j0, nb,                \
                           (const double *)w.dinv, (const int *)w.rowsrc, w.W, w.B, wblk);                             \
        hipLaunchKernelGGL(inv_update_kernel<NB>, dim3(ublk), dim3(256), 0, s, w.A, m, ld, j0, nb,                     \
                           (const double *)w.W, (const double *)w.B);                                                  \
    }
        if (mr <= 1536) {
            if (mr <= 256) STMG_PANEL(32, 1, 256)
            else if (mr <= 512) STMG_PANEL(32, 1, 512)
            else if (mr <= 1024) STMG_PANEL(32, 2, 512)
            else STMG_PANEL(32, 3, 512)
            STMG_REST(32)
        } else if (mr <= 3072) {
            STMG_PANEL(16, 3, 1024)
            STMG_REST(16)
        } else {
            STMG_PANEL(8, 6, 1024)
            STMG_REST(8)
        }
#undef STMG_PANEL
#undef STMG_REST
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        j0 += nb;
    }
    return hipSuccess;
}

template <typename T>
hipError_t launch_inverse_apply(const DenseInverse &w, const T *r, T *d, int n, hipStream_t s)
{
    const size_t lds = (size_t)w.m * sizeof(double);
    if (w.m <= 1024)
        hipLaunchKernelGGL((inv_apply_kernel<T, 1>), dim3((n + 3) / 4), dim3(256), lds, s, (const double *)w.A, w.m,
                           w.ld, n, (const int *)w.perm, r, d);
    else
        hipLaunchKernelGGL((inv_apply_kernel<T, 2>), dim3((n + 7) / 8), dim3(256), lds, s, (const double *)w.A, w.m,
                           w.ld, n, (const int *)w.perm, r, d);
    return hipGetLastError();
}

template hipError_t launch_inverse_apply<double>(const DenseInverse &, const double *, double *, int, hipStream_t);
template hipError_t launch_inverse_apply<float>(const DenseInverse &, const float *, float *, int, hipStream_t);

} // namespace stmg
