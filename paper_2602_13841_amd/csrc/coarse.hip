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
#include "coarse.h"

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
    v = step(v, [](int x) { return __builtin_amdgcn_update_dpp(x, x, 0x142, 0xa, 0xf, false); });   // row_bcast 15
    v = step(v, [](int x) { return __builtin_amdgcn_update_dpp(x, x, 0x143, 0xc, 0xf, false); });   // row_bcast 31
    const long long b = __double_as_longlong(v);   // lane 63: all lanes
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), 63);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// ---------------------------------------------------------------------------
// Pivots and D^{-1} of one panel: columns [j0, j0 + nb),
// candidate rows [j0, m), each thread RPT rows of NB columns in registers (RPT
// NTH >= m - j0).  Rows stay where they are; a thread tracks the logical
// position of its rows under the interchanges.  A latency chain: two barriers
// per column (candidates of the wavefronts; the pivot row).  The column loops
// are not unrolled: each step shifts the row by one column as it updates it
// (the current column is always a[.][0]), eight columns per loop with the
// width shrinking in between.
//
// The panel comes from its transposed copy Pt [column][row], so that the loads
// of consecutive rows are contiguous (from A, one 256-byte row segment per
// lane, they took 13 us of a 55 us panel); the multipliers of all rows go to
// Lt [column][row].  Writes rowsrc[i] = row that the interchanges bring to
// position i >= j0, the accumulated permutation perm, and D^{-1} (NB x NB, zero
// beyond nb).
// ---------------------------------------------------------------------------
template <int NB, int RPT, int NTH>
__global__ void __launch_bounds__(NTH) inv_panel_kernel(const double *__restrict__ Pt, double *__restrict__ Lt, int m,
                                                        int ld, int j0, int nb, double *__restrict__ dinv,
                                                        int *__restrict__ rowsrc, int *__restrict__ perm)
{
    constexpr int NW = NTH / 64;
    __shared__ double wval[NW];
    __shared__ int wlog[NW];
    __shared__ alignas(16) double urow[NB][NB];   // urow[c][j] = U of D, row c, column c + j
    __shared__ int pivrow[NB];
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
        const double *src = Pt + j0 + min(r, mr - 1);
#pragma unroll
        for (int k = 0; k < NB; ++k) a[i][k] = src[(long long)min(k, nb - 1) * ld];
    }
    auto columns = [&](auto width, int c0) {
        constexpr int WD = decltype(width)::value;   // columns that are left
        const int c1 = min(c0 + 8, nb);
#pragma unroll 1
        for (int c = c0; c < c1; ++c) {
            double best = -1.0;
            int bl = 0;
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const double v = fabs(a[i][0]);
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
            double bv[NW];
            int bp[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                bv[w] = wval[w];
                bp[w] = wlog[w];
            }
#pragma unroll
            for (int h = NW / 2; h > 0; h /= 2)
#pragma unroll
                for (int w = 0; w < h; ++w)
                    if (bv[w + h] > bv[w]) {
                        bv[w] = bv[w + h];
                        bp[w] = bp[w + h];
                    }
            // a column without a comparable entry (all NaN) keeps its own row
            const int p = bv[0] < 0.0 ? c : bp[0];
#pragma unroll
            for (int i = 0; i < RPT; ++i)
                if (((open >> i) & 1u) && lg[i] == p) {
                    pivrow[c] = j0 + tid + i * NTH;
#pragma unroll
                    for (int k = 0; k < WD; ++k) urow[c][k] = a[i][k];
                }
            __syncthreads();
            const double d = urow[c][0];
            const double inv = d != 0.0 ? 1.0 / d : 0.0;
            double l[RPT];
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const bool op = (open >> i) & 1u, piv = op && lg[i] == p;
                l[i] = op && !piv ? a[i][0] * inv : 0.0;
                if (op && !piv) Lt[(long long)c * ld + j0 + tid + i * NTH] = l[i];
                if (op && !piv && lg[i] == c) lg[i] = p;
                if (piv) {
                    lg[i] = c;
                    open &= ~(1u << i);
                }
            }
#pragma unroll
            for (int k = 1; k < WD; ++k) {
                const double u = urow[c][k];
#pragma unroll
                for (int i = 0; i < RPT; ++i) a[i][k - 1] = a[i][k] - l[i] * u;
            }
        }
    };
    static_for(std::make_integer_sequence<int, NB / 8>{}, [&](auto s) {
        constexpr int c0 = 8 * decltype(s)::value;
        if (c0 < nb) columns(std::integral_constant<int, NB - c0>{}, c0);
    });
    int before[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = tid + i * NTH;
        if (r < mr) {
            before[i] = j0 == 0 ? r : perm[j0 + r];
            rowsrc[j0 + lg[i]] = j0 + r;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPT; ++i)
        if (tid + i * NTH < mr) perm[j0 + lg[i]] = before[i];
    // D^{-1} = U^{-1} L^{-1}: lane i holds row i, each wavefront CPW columns;
    // both substitutions are y -= coef_k y_k with y_k broadcast from lane k (U
    // divided by its diagonal, which scales the rows at the end)
    constexpr int CPW = NB / NW;
    const int i = min(lane, NB - 1), ir = min(i, nb - 1);
    double coef[NB], y[CPW];
#pragma unroll
    for (int k = 0; k < NB; ++k) coef[k] = k < i && i < nb ? Lt[(long long)k * ld + pivrow[ir]] : 0.0;
#pragma unroll
    for (int q = 0; q < CPW; ++q) y[q] = i == wv * CPW + q ? 1.0 : 0.0;
    auto bcast = [](double x, int l) {
        const long long b = __double_as_longlong(x);
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
        const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
        return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    };
#pragma unroll
    for (int k = 0; k < NB - 1; ++k)
#pragma unroll
        for (int q = 0; q < CPW; ++q) y[q] -= coef[k] * bcast(y[q], k);
    const double rd = i < nb ? 1.0 / urow[ir][0] : 1.0;
#pragma unroll
    for (int k = 0; k < NB; ++k) coef[k] = k > i && k < nb ? urow[i][k - i] * bcast(rd, k) : 0.0;
#pragma unroll
    for (int k = NB - 1; k > 0; --k)
#pragma unroll
        for (int q = 0; q < CPW; ++q) y[q] -= coef[k] * bcast(y[q], k);
    if (lane < NB) {
#pragma unroll
        for (int q = 0; q < CPW; ++q) {
            const int j = wv * CPW + q;
            dinv[lane * NB + j] = lane < nb && j < nb ? y[q] * rd : 0.0;
        }
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
// A <- A + W B (rows J: W B alone; columns J: W), with a transposed copy of the
// next panel's columns [jn, jn + nbn) to Pt; one 32 x 32 tile per wavefront on v_mfma_f64_16x16x4f64 (A lane l -> (row l%16, k l/16), B lane
// l -> (k l/16, col l%16), D register i -> (row l/16 + 4i, col l%16)).  Bound
// by the read and write of A; W (m x nb) and B stay in L2.
// ---------------------------------------------------------------------------
template <int NB>
__global__ void __launch_bounds__(256) inv_update_kernel(double *__restrict__ A, int m, int ld, int j0, int nb,
                                                         const double *__restrict__ W, const double *__restrict__ B,
                                                         double *__restrict__ Pt, int jn, int nbn)
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
                    if (col >= jn && col < jn + nbn) Pt[(long long)(col - jn) * ld + row] = acc[si][sj][i];
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
                                                         long long Np1, int npm, double *__restrict__ A, int ld,
                                                         double *__restrict__ Pt)
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
        if (col < 32) Pt[(long long)col * ld + row] = v;   // the first panel, transposed
    }
}

// the widest panel whose candidate rows fit the registers of one workgroup
// (RPT NB = 96 doubles per thread at 8 wavefronts)
int panel_width(int rows) { return min(rows, rows <= 1536 ? 32 : rows <= 3072 ? 16 : 8); }

} // namespace

hipError_t launch_inv_matrix(const double *Y, int n, int nb, long long pbase, long long Np1, int npm,
                             const DenseInverse &w, hipStream_t s)
{
    const unsigned nt = (unsigned)((n + nb + 31) / 32);
    hipLaunchKernelGGL(inv_matrix_kernel, dim3(nt, nt), dim3(256), 0, s, Y, n, nb, pbase, Np1, npm, w.A, w.ld, w.Pt);
    return hipGetLastError();
}

hipError_t launch_dense_inverse(const DenseInverse &w, hipStream_t s)
{
    const int m = w.m, ld = w.ld;
    if (m <= 0) return hipSuccess;
    if (m > DINV_MAX_M) return hipErrorInvalidValue;
    const int wblk = (m + 63) / 64, cblk = (m + 255) / 256, nt = (m + 31) / 32, ublk = (nt * nt + 3) / 4;
    for (int j0 = 0; j0 < m;) {
        const int mr = m - j0, nb = panel_width(mr), jn = j0 + nb, nbn = jn < m ? panel_width(m - jn) : 0;
#define STMG_PANEL(NB, RPT, NTH)                                                                                       \
    hipLaunchKernelGGL((inv_panel_kernel<NB, RPT, NTH>), dim3(1), dim3(NTH), 0, s, (const double *)w.Pt, w.B, m, ld, \
                       j0, nb, w.dinv, w.rowsrc, w.perm)
#define STMG_REST(NB)                                                                                                  \
    {                                                                                                                  \
        hipLaunchKernelGGL(inv_swap_kernel<NB>, dim3(wblk + cblk), dim3(256), 0, s, w.A, m, ld, j0, nb,                \
                           (const double *)w.dinv, (const int *)w.rowsrc, w.W, w.B, wblk);                             \
        hipLaunchKernelGGL(inv_update_kernel<NB>, dim3(ublk), dim3(256), 0, s, w.A, m, ld, j0, nb,                     \
                           (const double *)w.W, (const double *)w.B, w.Pt, jn, nbn);                                   \
    }
        // the fewest wavefronts that hold the candidate rows: every wavefront
        // reads the whole pivot row from LDS in each column
        if (mr <= 1536) {
            if (mr <= 256) STMG_PANEL(32, 1, 256);
            else if (mr <= 512) STMG_PANEL(32, 2, 256);
            else if (mr <= 768) STMG_PANEL(32, 3, 256);
            else if (mr <= 1024) STMG_PANEL(32, 2, 512);
            else STMG_PANEL(32, 3, 512);
            STMG_REST(32)
        } else if (mr <= 3072) {
            STMG_PANEL(16, 6, 512);
            STMG_REST(16)
        } else {
            STMG_PANEL(8, 12, 512);
            STMG_REST(8)
        }
#undef STMG_PANEL
#undef STMG_REST
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        j0 = jn;
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
