// LU factorizations of the time-decoupled patch systems and the sweeps that
// use them.
//
// One workgroup factors one matrix (real or complex planar, FP32 or FP64,
// row-major), left-looking in block columns of 32: the block column is held in
// MFMA accumulators (32 x 32 row tiles over the wavefronts), receives the
// updates of all finished block columns, is factored in panels of 16 columns
// and written once.  A right-looking factorization moves the trailing matrix
// through HBM once per block (13.3 MB per 395 x 395 complex FP32 matrix of 1.25
// MB measured for the two-level kernel this replaced); here each block column
// is read and written once and L once per later block column (6.4 MB).
// 13824 matrices of 395 complex FP32: 93.7 -> 43.7 ms (52 TFLOP/s of the 148
// that a large FP32 product reaches); 1728 of 202: 3.7 -> 1.7 ms; 13824 of 85:
// 7.0 -> 2.1 ms; 512 complex FP64 of 202: 2.0 -> 1.2 ms.  What bounds it at 395,
// two workgroups per CU (cycles of a workgroup, per matrix): the MFMA updates
// 1.27 M (they keep the matrix cores busy 38 % of the time), the panel columns
// 1.1 M (a latency chain of 1100 cycles in pivot search and publishing per
// column), U products 0.3 M, panel staging and inverses 0.6 M.
//
// Rows never move: cur[p] is the stored row at position p of the permuted
// matrix, and everything addresses rows through it (loads and stores of whole
// row segments, so the indirection costs nothing).  Position tiles are
// therefore exact: tile K < J of block column J holds the pivot rows of block
// K, and the update with block K touches the tiles behind it only.
//
// Format left in A (position p at row perm[p]): L below the diagonal blocks, U
// above them, and in each 32 x 32 diagonal block the strict lower part of
// L_JJ^{-1} and the upper triangle of U_JJ^{-1}; the factorization applies
// L_JJ^{-1} by MFMA and the sweeps replace both substitutions of a diagonal
// block by products.
#include "vanka.h"

#include "stmg_internal.h"

#include <type_traits>
#include <utility>

// every multiply-add below is written out: the results do not depend on which
// products the compiler would fuse in which instantiation
#pragma clang fp contract(off)

namespace stmg {

namespace {

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float abs_(float x) { return __builtin_fabsf(x); }
__device__ __forceinline__ double abs_(double x) { return __builtin_fabs(x); }
template <typename T> __device__ __forceinline__ bool finite_(T x) { return abs_(x) < T(__builtin_inf()); }

typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef double doublex4_t __attribute__((ext_vector_type(4)));
// 16-byte row segments at element alignment
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef double doublex2_u __attribute__((ext_vector_type(2), aligned(8)));

template <typename T> struct Vec;
template <> struct Vec<float> {
    using acc = floatx4_t;
    using seg = floatx4_u;
    static constexpr int W = 4;      // elements of a 16-byte segment
    static constexpr int LDU = 36;   // row stride of a U block in LDS: the four k groups on disjoint banks
    static __device__ __forceinline__ acc mfma(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // row of accumulator register i of lane group g
    static __device__ __forceinline__ int row(int g, int i) { return 4 * g + i; }
};
template <> struct Vec<double> {
    using acc = doublex4_t;
    using seg = doublex2_u;
    static constexpr int W = 2;
    static constexpr int LDU = 40;
    static __device__ __forceinline__ acc mfma(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int i) { return g + 4 * i; }
};

template <int... I, typename F> __device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// x moved by a DPP control (both halves of a double)
template <int CTRL, int RM> __device__ __forceinline__ float dpp(float x)
{
    const int b = __float_as_int(x);
    return __int_as_float(__builtin_amdgcn_update_dpp(b, b, CTRL, RM, 0xf, false));
}
template <int CTRL, int RM> __device__ __forceinline__ double dpp(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = (int)(b & 0xffffffff), hi = (int)(b >> 32);
    const int l = __builtin_amdgcn_update_dpp(lo, lo, CTRL, RM, 0xf, false);
    const int h = __builtin_amdgcn_update_dpp(hi, hi, CTRL, RM, 0xf, false);
    return __longlong_as_double(((long long)h << 32) | (unsigned)l);
}
__device__ __forceinline__ double lane_value(double x, int l)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Pivot keys: order the candidates of a column like their moduli, a NaN below
// every number and a row that is no candidate below a NaN, so that a NaN is
// the pivot only of a column without a number (and is not a zero pivot).  FP32: the bits of the modulus (>= +0) as an integer, which has the order of
// the values and makes each step of the maxima one instruction.
template <typename T> struct Pivot;
template <> struct Pivot<float> {
    using key = int;
    static constexpr key NONE = -2;
    static __device__ __forceinline__ key of(float modulus) { return modulus >= 0.0f ? __float_as_int(modulus) : -1; }
};
template <> struct Pivot<double> {
    using key = double;
    static constexpr key NONE = -2.0;
    static __device__ __forceinline__ key of(double modulus) { return modulus >= 0.0 ? modulus : -1.0; }
};
template <int CTRL, int RM> __device__ __forceinline__ int dpp(int x)
{
    return __builtin_amdgcn_update_dpp(x, x, CTRL, RM, 0xf, false);
}
__device__ __forceinline__ int lane_value(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ int max_of(int a, int b) { return max(a, b); }
__device__ __forceinline__ double max_of(double a, double b) { return fmax(a, b); }
// wavefront maximum, uniform (row_shr 1, 2, 4, 8, then row_bcast 15 and 31)
__device__ __forceinline__ int wave_max(int v)
{
    constexpr int lowest = -0x7fffffff - 1;
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, dpp<0x111, 0xf>(v));
    v = fmax(v, dpp<0x112, 0xf>(v));
    v = fmax(v, dpp<0x114, 0xf>(v));
    v = fmax(v, dpp<0x118, 0xf>(v));
    v = fmax(v, dpp<0x142, 0xa>(v));
    v = fmax(v, dpp<0x143, 0xc>(v));
    return lane_value(v, 63);
}

// ---------------------------------------------------------------------------
// small dense pieces, one wavefront each, 16 x 16 blocks in LDS (row stride
// LS entries of P words)
// ---------------------------------------------------------------------------
constexpr int TD_BW = 32;   // block columns
constexpr int TD_PW = 16;   // panel columns
constexpr int TD_LS = 17;   // row stride of panels and small blocks (entries)

// C (+)= A B on one 16 x 16 tile, K = 16, A and B as LDS blocks: lane (r, g)
// supplies A[r][k] and B[k][r] for k = 4W h + W g + s
template <typename T, bool CX>
__device__ __forceinline__ void mm16(const T *A, const T *B, typename Vec<T>::acc &cr, typename Vec<T>::acc &ci)
{
    constexpr int P = CX ? 2 : 1, W = Vec<T>::W;
    const int l = threadIdx.x & 63, r = l & 15, g = l >> 4;
#pragma unroll
    for (int h = 0; h < 16 / (4 * W); ++h)
#pragma unroll
        for (int s = 0; s < W; ++s) {
            const int k = 4 * W * h + W * g + s;
            const T *a = A + (r * TD_LS + k) * P, *b = B + (k * TD_LS + r) * P;
            cr = Vec<T>::mfma(a[0], b[0], cr);
            if constexpr (CX) {
                cr = Vec<T>::mfma(-a[1], b[1], cr);
                ci = Vec<T>::mfma(a[0], b[1], ci);
                ci = Vec<T>::mfma(a[1], b[0], ci);
            }
        }
}

// inverse of a 16 x 16 triangular block (unit lower, or upper): lane (i, g)
// holds row i of columns 4g .. 4g+3; one step per eliminated row, its values
// broadcast inside the 16-lane rows.  coef(i, k): entry (i, k) of the block,
// zero outside the strict triangle; rd: reciprocal of the lane's own diagonal
// entry (1 for the lower block)
template <typename T, bool CX, bool UPPER, typename F>
__device__ __forceinline__ void tri_inverse16(F coef, T rdr, T rdi, T (&yr)[4], T (&yi)[4])
{
    const int l = threadIdx.x & 63, i = l & 15, g = l >> 4;
    T cr[16], ci[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) coef(i, k, cr[k], ci[k]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        yr[q] = i == 4 * g + q ? T(1) : T(0);
        yi[q] = T(0);
    }
    static_for(std::make_integer_sequence<int, 15>{}, [&](auto kk) {
        constexpr int k = UPPER ? 15 - decltype(kk)::value : decltype(kk)::value;
        constexpr int BC = 0x150 + k;   // row_newbcast
        T ar = cr[k], ai = ci[k];
        if constexpr (UPPER) {
            // column k divided by its diagonal entry: the rows are scaled last
            const T dr = dpp<BC, 0xf>(rdr);
            if constexpr (CX) {
                const T di = dpp<BC, 0xf>(rdi), t = fma_(ar, dr, -(ai * di));
                ai = fma_(ar, di, ai * dr);
                ar = t;
            } else {
                ar *= dr;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T br = dpp<BC, 0xf>(yr[q]);
            if constexpr (CX) {
                const T bi = dpp<BC, 0xf>(yi[q]);
                yr[q] = fma_(ai, bi, fma_(-ar, br, yr[q]));
                yi[q] = fma_(-ai, br, fma_(-ar, bi, yi[q]));
            } else {
                yr[q] = fma_(-ar, br, yr[q]);
            }
        }
    });
    if constexpr (UPPER) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (CX) {
                const T t = fma_(yr[q], rdr, -(yi[q] * rdi));
                yi[q] = fma_(yr[q], rdi, yi[q] * rdr);
                yr[q] = t;
            } else {
                yr[q] *= rdr;
            }
        }
    }
}

template <typename T, bool CX> __device__ __forceinline__ void reciprocal(T dr, T di, T &ir, T &ii)
{
    if constexpr (CX) {
        const T den = fma_(dr, dr, di * di);
        const T inv = T(1) / den;
        ir = dr * inv;
        ii = -di * inv;
        // a pivot so small that 1 / den overflows (FP32: below 5.4e-20) still
        // has a finite reciprocal; zero: no elimination
        if (!(inv < T(__builtin_inf()))) {
            ir = den != T(0) ? dr / den : T(0);
            ii = den != T(0) ? -di / den : T(0);
        }
    } else {
        const T inv = T(1) / dr;
        ir = dr != T(0) ? inv : T(0);
        ii = T(0);
    }
}

// LDS bytes of one factorization: panel, U blocks (and L of a diagonal block:
// STD), positions and ranks
template <typename T, bool CX, int PW, bool STD> constexpr size_t left_lu_lds_bytes(int m)
{
    constexpr int P = CX ? 2 : 1;
    const size_t pan = (size_t)m * (PW + 1) * P, ub = (size_t)P * TD_BW * Vec<T>::LDU;
    return (pan + 2 * ub + (STD ? TD_BW * (TD_BW + 1) : 0)) * sizeof(T) +
           (size_t)(2 * ((m + 31) & ~31) + TD_BW) * sizeof(int);
}

// ---------------------------------------------------------------------------
// the factorization of one matrix by the workgroup: NW wavefronts, SLOTS row
// tiles per wavefront (32 NW SLOTS >= m), RPT panel rows per thread (64 NW RPT
// >= m), panels of PW columns.  STD = false: the format of the time-decoupled
// systems (ip: the permutation); STD = true (real only): LAPACK's, L and U of
// the row-permuted matrix (ip: the interchanges), at the price of one more
// pass that permutes the rows, and with each U block by substitution.
// ---------------------------------------------------------------------------
template <typename T, bool CX, int NW, int SLOTS, int RPT, int PW, bool STD>
__device__ __forceinline__ void lu_left(T *__restrict__ Ar, int m, int ld, int *__restrict__ ip, int *info,
                                        unsigned char *lds_raw)
{
    static_assert(!STD || (!CX && NW <= 8), "the LAPACK format is real");
    using V = Vec<T>;
    using acc_t = typename V::acc;
    using seg_t = typename V::seg;
    constexpr int P = CX ? 2 : 1, W = V::W, LDU = V::LDU, NTH = 64 * NW;
    constexpr int NH = TD_BW / (4 * W);   // 16-byte segments per lane along K = 32
    constexpr int LS = PW + 1;            // row stride of the panel
    T *pan = reinterpret_cast<T *>(lds_raw);                  // [rows from the block on][LS][P]
    T *ub1 = pan + (size_t)m * LS * P;                         // [P][32][LDU]
    T *ub2 = ub1 + P * TD_BW * LDU;                            // [P][32][LDU] (negated U)
    // 16 x 16 blocks of the panel phase, in the U blocks: A12 (then L21), a
    // product and V2 in the first, U12, I1, V1 and I2 in the second
    constexpr int SB = 16 * TD_LS * P;
    static_assert(4 * SB <= P * TD_BW * LDU, "four small blocks fit a U block");
    T *sV2 = ub1 + 2 * SB, *sI1 = ub2 + SB, *sV1 = ub2 + 2 * SB, *sI2 = ub2 + 3 * SB;
    T *lkk = ub2 + P * TD_BW * LDU;                            // [32][33] columns of L_KK (STD)
    int *cur = reinterpret_cast<int *>(lkk + (STD ? TD_BW * (TD_BW + 1) : 0));   // stored row at each position
    int *rk = cur + ((m + 31) & ~31);                          // rank of a panel row among the block's pivots, or -1
    int *pl = rk + ((m + 31) & ~31);                           // panel row of each pivot of the block
    // pivot candidates of the wavefronts, by column parity: key, panel row |
    // position << 16, and the row from its current column on
    using PV = Pivot<T>;
    using key_t = typename PV::key;
    __shared__ alignas(16) key_t wval[2][NW];
    __shared__ alignas(16) int wkey[2][NW];
    __shared__ alignas(16) T pub[2][NW][16 * P];

    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    T *Ai = Ar + (CX ? (long long)m * ld : 0);
    // entries of A by byte offset (32-bit offsets from a uniform base)
    const unsigned ldb = ld * sizeof(T);
    auto at = [](T *base, unsigned o) { return reinterpret_cast<T *>(reinterpret_cast<char *>(base) + o); };
    const int nt = (m + 31) / 32;
    for (int p = tid; p < m; p += NTH) cur[p] = p;
    __syncthreads();

    for (int J = 0; J < nt; ++J) {
        const int j0 = 32 * J, nbj = min(32, m - j0), mr = m - j0;
        // opaque to the compiler, so that it does not keep every address that
        // depends on the lane alive (spilled) across the block columns
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        const int l16 = lane & 15, g = lane >> 4;
        const unsigned jb = j0 * sizeof(T);
        // ---- the block column, rows in position order ------------------------------
        acc_t ar[SLOTS][2][2], ai[CX ? SLOTS : 1][2][2];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            // (tiles past the end reload the last row: no branch between the loads)
            const int t = wv + NW * s;
#pragma unroll
            for (int si = 0; si < 2; ++si)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned o = cur[min(32 * t + 16 * si + V::row(g, i), m - 1)] * ldb + jb;
#pragma unroll
                    for (int sj = 0; sj < 2; ++sj) {
                        const unsigned c = min(16 * sj + l16, nbj - 1) * sizeof(T);
                        ar[s][si][sj][i] = *at(Ar, o + c);
                        if constexpr (CX) ai[s][si][sj][i] = *at(Ai, o + c);
                    }
                }
        }
        // ---- updates of the finished block columns ------------------------------------
        // row offsets of the L operands of this wavefront's tiles (many tiles:
        // looked up for each segment, the accumulators leave no registers)
        constexpr bool RO = SLOTS <= 4;
        unsigned ro[RO ? SLOTS : 1][2];
        auto row_offset = [&](int s, int si) -> unsigned {
            return cur[min(32 * (wv + NW * s) + 16 * si + l16, m - 1)] * ldb + 16 * g;
        };
        if constexpr (RO) {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int si = 0; si < 2; ++si) ro[s][si] = row_offset(s, si);
        }
        // U = L_KK^{-1} (tile K), its four 16 x 16 tiles spread over the
        // wavefronts (tile q: rows 16 (q / 2), columns 16 (q % 2)); the rows
        // of L_KK^{-1} are loaded one block ahead
        // (STD: L_KK itself, transposed into LDS, and one substitution per
        // wavefront, lane = row)
        constexpr int UT = NW >= 4 ? 1 : 4 / NW, LE = TD_BW * TD_BW / NTH;
        seg_t fr[STD ? 1 : UT][NH], fi[CX ? UT : 1][NH];
        T le[STD ? LE : 1];
        auto load_inverse = [&](int K) {
            if constexpr (STD) {
#pragma unroll
                for (int u = 0; u < LE; ++u) {
                    const int e = tid + u * NTH;
                    le[u] = *at(Ar, cur[32 * K + (e >> 5)] * ldb + (32 * K + (e & 31)) * sizeof(T));
                }
            } else {
#pragma unroll
                for (int u = 0; u < UT; ++u) {
                    const int si0 = ((wv + NW * u) >> 1) & 1;
                    const unsigned o = cur[32 * K + 16 * si0 + l16] * ldb + 32 * K * sizeof(T) + 16 * g;
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        fr[u][h] = *(const seg_t *)at(Ar, o + 64 * h);
                        if constexpr (CX) fi[u][h] = *(const seg_t *)at(Ai, o + 64 * h);
                    }
                }
            }
        };
        if (J > 0 && (STD || wv < 4)) load_inverse(0);
#pragma unroll 1
        for (int K = 0; K < J; ++K) {
            // tile K: the pivot rows of block K
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (wv + NW * s == K) {
#pragma unroll
                    for (int si = 0; si < 2; ++si)
#pragma unroll
                        for (int sj = 0; sj < 2; ++sj)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int o = (16 * si + V::row(g, i)) * LDU + 16 * sj + l16;
                                ub1[o] = ar[s][si][sj][i];
                                if constexpr (CX) ub1[TD_BW * LDU + o] = ai[s][si][sj][i];
                            }
                }
            if constexpr (STD) {
#pragma unroll
                for (int u = 0; u < LE; ++u) {
                    const int e = tid + u * NTH, i = e >> 5, k = e & 31;
                    lkk[k * (TD_BW + 1) + i] = k < i ? le[u] : T(0);
                }
            }
            __syncthreads();
            if constexpr (STD) {
                // lane (i, g): rows i and 16 + i of CL columns, the solved
                // rows broadcast inside the 16-lane rows
                constexpr int CL = TD_BW / NW / 4 > 0 ? TD_BW / NW / 4 : 1;
                const int cw = wv * (TD_BW / NW) + g * CL;
                T y0[CL], y1[CL];
#pragma unroll
                for (int q = 0; q < CL; ++q) {
                    y0[q] = ub1[l16 * LDU + cw + q];
                    y1[q] = ub1[(16 + l16) * LDU + cw + q];
                }
                static_for(std::make_integer_sequence<int, 16>{}, [&](auto kk) {
                    constexpr int k = decltype(kk)::value;
                    const T c0 = lkk[k * (TD_BW + 1) + l16], c1 = lkk[k * (TD_BW + 1) + 16 + l16];
#pragma unroll
                    for (int q = 0; q < CL; ++q) {
                        const T v = dpp<0x150 + k, 0xf>(y0[q]);
                        y0[q] = fma_(-c0, v, y0[q]);
                        y1[q] = fma_(-c1, v, y1[q]);
                    }
                });
                static_for(std::make_integer_sequence<int, 15>{}, [&](auto kk) {
                    constexpr int k = decltype(kk)::value;
                    const T c1 = lkk[(16 + k) * (TD_BW + 1) + 16 + l16];
#pragma unroll
                    for (int q = 0; q < CL; ++q) y1[q] = fma_(-c1, dpp<0x150 + k, 0xf>(y1[q]), y1[q]);
                });
#pragma unroll
                for (int q = 0; q < CL; ++q) {
                    ub2[l16 * LDU + cw + q] = -y0[q];
                    ub2[(16 + l16) * LDU + cw + q] = -y1[q];
                }
                bool fin = true;
#pragma unroll
                for (int q = 0; q < CL; ++q) fin = fin && finite_(y0[q]) && finite_(y1[q]);
                if (__any(!fin)) {
                    // an infinity or NaN must not reach the rows above it (zero
                    // times its value): plain substitution, one column per lane
                    if (l16 < CL)
#pragma unroll 1
                        for (int i = 0; i < 32; ++i) {
                            T v = -ub1[i * LDU + cw + l16];
#pragma unroll 1
                            for (int k = 0; k < i; ++k)
                                v = fma_(-lkk[k * (TD_BW + 1) + i], ub2[k * LDU + cw + l16], v);
                            ub2[i * LDU + cw + l16] = v;
                        }
                }
                if (K + 1 < J) load_inverse(K + 1);
            } else if (wv < 4) {
#pragma unroll
                for (int u = 0; u < UT; ++u) {
                    const int si0 = ((wv + NW * u) >> 1) & 1, sj0 = (wv + NW * u) & 1;
                    acc_t dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
                    const int row = 16 * si0 + l16;
#pragma unroll
                    for (int h = 0; h < NH; ++h)
#pragma unroll
                        for (int s = 0; s < W; ++s) {
                            const int k = 4 * W * h + W * g + s, o = k * LDU + 16 * sj0 + l16;
                            const T lr = k < row ? fr[u][h][s] : (k == row ? T(1) : T(0));
                            const T br = ub1[o];
                            dr = V::mfma(lr, br, dr);
                            if constexpr (CX) {
                                const T li = k < row ? fi[u][h][s] : T(0), bi = ub1[TD_BW * LDU + o];
                                dr = V::mfma(-li, bi, dr);
                                di = V::mfma(lr, bi, di);
                                di = V::mfma(li, br, di);
                            }
                        }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int r = 16 * si0 + V::row(g, i), c = 16 * sj0 + l16, o = r * LDU + c;
                        ub2[o] = -dr[i];
                        if constexpr (CX) ub2[TD_BW * LDU + o] = -di[i];
                        if (c < nbj) {
                            const unsigned a = cur[32 * K + r] * ldb + jb + c * sizeof(T);
                            *at(Ar, a) = dr[i];
                            if constexpr (CX) *at(Ai, a) = di[i];
                        }
                    }
                }
                if (K + 1 < J) load_inverse(K + 1);
            }
            __syncthreads();
            if constexpr (STD) {
#pragma unroll
                for (int u = 0; u < LE; ++u) {
                    const int e = tid + u * NTH, r = e >> 5, c = e & 31;
                    if (c < nbj) *at(Ar, cur[32 * K + r] * ldb + jb + c * sizeof(T)) = -ub2[r * LDU + c];
                }
            }
            // tiles behind K: C -= L U, one 16-byte segment of L per lane and
            // row tile at a time, the next one loaded before the products of
            // the current (512 real FP64 matrices of 1185, whose loads were
            // waited for: 40 -> 33 ms; 4096 complex FP32 of 395: 14.5 -> 14.0)
            seg_t nr[2], ni[2];
            auto load_l = [&](int s, int h) {
#pragma unroll
                for (int si = 0; si < 2; ++si) {
                    const unsigned o = (RO ? ro[RO ? s : 0][si] : row_offset(s, si)) + 32 * K * sizeof(T) + 64 * h;
                    nr[si] = *(const seg_t *)at(Ar, o);
                    if constexpr (CX) ni[si] = *(const seg_t *)at(Ai, o);
                }
            };
            bool loaded = false;
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const int t = wv + NW * s;
                if (t > K && t < nt) {
                    if (!loaded) load_l(s, 0);
                    loaded = true;
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        seg_t lr[2], li[2];
#pragma unroll
                        for (int si = 0; si < 2; ++si) {
                            lr[si] = nr[si];
                            if constexpr (CX) li[si] = ni[si];
                        }
                        // (past the last tile: a row that exists, not used)
                        if (h + 1 < NH) load_l(s, h + 1);
                        else if (s + 1 < SLOTS) load_l(s + 1, 0);
                        T br[W][2], bi[W][2];
#pragma unroll
                        for (int u = 0; u < W; ++u)
#pragma unroll
                            for (int sj = 0; sj < 2; ++sj) {
                                const int o = (4 * W * h + W * g + u) * LDU + 16 * sj + l16;
                                br[u][sj] = ub2[o];
                                bi[u][sj] = CX ? ub2[CX ? TD_BW * LDU + o : 0] : T(0);
                            }
#pragma unroll
                        for (int u = 0; u < W; ++u)
#pragma unroll
                            for (int si = 0; si < 2; ++si)
#pragma unroll
                                for (int sj = 0; sj < 2; ++sj) {
                                    ar[s][si][sj] = V::mfma(lr[si][u], br[u][sj], ar[s][si][sj]);
                                    if constexpr (CX) {
                                        ar[s][si][sj] = V::mfma(-li[si][u], bi[u][sj], ar[s][si][sj]);
                                        ai[s][si][sj] = V::mfma(lr[si][u], bi[u][sj], ai[s][si][sj]);
                                        ai[s][si][sj] = V::mfma(li[si][u], br[u][sj], ai[s][si][sj]);
                                    }
                                }
                    }
                }
            }
        }
        // ---- the block's panels -------------------------------------------------------
        // this thread's panel rows: whole sets of 64 RPT rows per wavefront, so
        // that wavefronts run out of rows one after the other and then only
        // keep the barriers (with the winner found by lanes below: 1024 real
        // matrices of 202 0.95 -> 0.81 ms, 64 FP32 of 1185 7.2 -> 6.5 ms)
        auto row_of = [&](int i) { return (wv * RPT + i) * 64 + lane; };
        const bool idle = row_of(0) - lane >= mr;
        int lg[RPT];         // position of this thread's rows, relative to the block
        unsigned open = 0;   // rows that are not pivotal yet
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = row_of(i);
            lg[i] = r;
            if (r < mr) {
                open |= 1u << i;
                rk[r] = -1;
            }
        }
        static_for(std::make_integer_sequence<int, TD_BW / PW>{}, [&](auto hc) {
            constexpr int h = decltype(hc)::value, c0 = PW * h;
            constexpr int sjh = c0 / 16, cs = c0 % 16;   // the panel's accumulator tile and its first column there
            const int nb = min(PW, nbj - c0);
            if (nb <= 0) return;
            __syncthreads();   // the panel region is free
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const int t = wv + NW * s;
                if (t >= J && t < nt) {
#pragma unroll
                    for (int si = 0; si < 2; ++si)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = 32 * (t - J) + 16 * si + V::row(g, i);
                            if (r < mr && (PW == 16 || (l16 >= cs && l16 < cs + PW))) {
                                T *q = pan + (r * LS + l16 - cs) * P;
                                q[0] = ar[s][si][sjh][i];
                                if constexpr (CX) q[1] = ai[s][si][sjh][i];
                            }
                        }
                }
            }
            __syncthreads();
            {
                T xr[RPT][PW], xi[CX ? RPT : 1][PW];
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const T *q = pan + min(row_of(i), mr - 1) * LS * P;
#pragma unroll
                    for (int k = 0; k < PW; ++k) {
                        xr[i][k] = q[k * P];
                        if constexpr (CX) xi[i][k] = q[k * P + 1];
                    }
                }
                // columns c .. of a row are x[.][0 ..]: every step shifts by one as it updates.
                // One barrier per column; no branches but the publishing ones.
                T *urow = ub1;   // [PW][PW] pivot rows from their own column on
                auto columns = [&](auto width, int cb) {
                    constexpr int WD = decltype(width)::value;
                    const int ce = min(cb + 4, nb);
                    if (idle) {
                        if (lane < 2) {
                            wval[lane][wv] = PV::NONE;
                            wkey[lane][wv] = 0;
                        }
                        for (int c = cb; c < ce; ++c) __syncthreads();
                        return;
                    }
#pragma unroll 1
                    for (int c = cb; c < ce; ++c) {
                        const int par = c & 1;
                        key_t best = PV::NONE;
                        int bi_ = 0, bl = 0x7fffffff;
#pragma unroll
                        for (int i = 0; i < RPT; ++i) {
                            const key_t v = PV::of(
                                CX ? fma_(xr[i][0], xr[i][0], xi[CX ? i : 0][0] * xi[CX ? i : 0][0]) : abs_(xr[i][0]));
                            const bool better = ((open >> i) & 1u) && (v > best || (STD && v == best && lg[i] < bl));
                            best = better ? v : best;
                            bl = better ? lg[i] : bl;
                            bi_ = better ? i : bi_;
                        }
                        const key_t wm = wave_max(best);
                        unsigned long long hit = __ballot(best == wm);
                        if (STD && __popcll(hit) > 1) {
                            // LAPACK: ties go to the smallest position
                            int low = best == wm ? bl : 0x7fffffff;
                            for (int off = 32; off > 0; off >>= 1) low = min(low, __shfl_xor(low, off, 64));
                            hit = __ballot(best == wm && bl == low);
                        }
                        const bool cand = lane == __builtin_ctzll(hit);
                        // the wavefront's candidate publishes its row
                        auto publish = [&](T *q, int i) {
#pragma unroll
                            for (int k = 0; k < WD; ++k) {
                                q[k * P] = xr[i][k];
                                if constexpr (CX) q[k * P + 1] = xi[i][k];
                            }
                        };
#pragma unroll
                        for (int i = 0; i < RPT; ++i)
                            if (cand && i == bi_) {
                                publish(pub[par][wv], i);
                                wval[par][wv] = wm;
                                wkey[par][wv] = min(row_of(i), mr - 1) | lg[i] << 16;
                            }
                        __syncthreads();
                        // the winner: candidate w in lane w (mod NW)
                        const key_t cv = wval[par][lane & (NW - 1)];
                        const int ck = wkey[par][lane & (NW - 1)] | (lane & (NW - 1)) << 12;
                        key_t top = cv;
                        if constexpr (NW > 1) top = max_of(top, dpp<0xB1, 0xf>(top));    // quad_perm 1,0,3,2
                        if constexpr (NW > 2) top = max_of(top, dpp<0x4E, 0xf>(top));    // quad_perm 2,3,0,1
                        if constexpr (NW > 4) top = max_of(top, dpp<0x141, 0xf>(top));   // row_half_mirror
                        unsigned long long win = __ballot(cv == top) & ((1ull << NW) - 1);
                        if (STD && __popcll(win) > 1) {
                            const int pos = cv == top ? ck >> 16 : 0x7fffffff;
                            int low = pos;
                            for (int off = NW / 2; off > 0; off >>= 1) low = min(low, __shfl_xor(low, off, 64));
                            win = __ballot(pos == low) & ((1ull << NW) - 1);
                        }
                        const int key = __builtin_amdgcn_readlane(ck, __builtin_ctzll(win | (1ull << 63)));
                        const int R = key & 0xfff, p = key >> 16;
                        const T *u = pub[par][(key >> 12) & 0xf];
                        T ur[WD], ui[WD];
#pragma unroll
                        for (int k = 0; k < WD; ++k) {
                            ur[k] = u[k * P];
                            ui[k] = CX ? u[CX ? k * P + 1 : 0] : T(0);
                        }
                        // (the whole row in flight before its first use)
                        __builtin_amdgcn_sched_barrier(0);
                        if (tid == 0) {
                            pl[c0 + c] = R;
                            rk[R] = c0 + c;
                            if constexpr (STD) ip[j0 + c0 + c] = j0 + p;
                            if (info && lane_value(top, 0) == key_t(0)) atomicAdd(info, 1);
                        }
                        T ir, ii;
                        reciprocal<T, CX>(ur[0], ui[0], ir, ii);
                        T lr[RPT], li[RPT];
#pragma unroll
                        for (int i = 0; i < RPT; ++i) {
                            const int r = row_of(i);
                            const bool op = (open >> i) & 1u, me = op && r == R, upd = op && !me;
                            T tr, ti;
                            if constexpr (CX) {
                                tr = fma_(xr[i][0], ir, -(xi[i][0] * ii));
                                ti = fma_(xr[i][0], ii, xi[i][0] * ir);
                            } else {
                                tr = xr[i][0] * ir;
                                ti = T(0);
                            }
                            lr[i] = upd ? tr : T(0);
                            li[i] = upd ? ti : T(0);
                            // (other rows write their padding entry)
                            T *q = pan + (min(r, m - 1) * LS + (upd ? c : PW)) * P;
                            q[0] = lr[i];
                            if constexpr (CX) q[1] = li[i];
                            if (me) publish(urow + c * PW * P, i);
                            lg[i] = me ? c0 + c : (op && lg[i] == c0 + c ? p : lg[i]);
                            open = me ? open & ~(1u << i) : open;
                        }
                        // (entries beyond the panel are never used; row sets of the
                        // wavefront past the end are skipped)
#pragma unroll
                        for (int i = 0; i < RPT; ++i) {
                            if (row_of(i) - lane >= mr) continue;
#pragma unroll
                            for (int k = 1; k < WD; ++k) {
                                T vr = fma_(-lr[i], ur[k], xr[i][k]);
                                if constexpr (CX) {
                                    vr = fma_(li[i], ui[k], vr);
                                    xi[i][k - 1] = fma_(-li[i], ur[k], fma_(-lr[i], ui[k], xi[i][k]));
                                }
                                xr[i][k - 1] = vr;
                            }
                        }
                    }
                };
                static_for(std::make_integer_sequence<int, PW / 4>{}, [&](auto q) {
                    constexpr int cb = 4 * decltype(q)::value;
                    if (cb < nb) columns(std::integral_constant<int, PW - cb>{}, cb);
                });
                __syncthreads();
                for (int e = tid; e < PW * PW; e += NTH) {
                    const int c = e / PW, k = e % PW;
                    if (c < nb && c + k < PW) {
                        T *q = pan + (pl[c0 + c] * LS + c + k) * P;
                        q[0] = urow[(c * PW + k) * P];
                        if constexpr (CX) q[1] = urow[(c * PW + k) * P + 1];
                    }
                }
            }
            __syncthreads();
            // the panel to A (rows that became pivots in the first panel hold U here already)
#pragma unroll 4
            for (int r = tid / PW; r < mr; r += NTH / PW) {
                const int c = tid % PW;
                if (c < nb && !(h > 0 && rk[r] >= 0 && rk[r] < c0)) {
                    const unsigned o = cur[j0 + r] * ldb + jb + (c0 + c) * sizeof(T);
                    *at(Ar, o) = pan[(r * LS + c) * P];
                    if constexpr (CX) *at(Ai, o) = pan[(r * LS + c) * P + 1];
                }
            }
            // inverses of the panel's triangles (identity beyond nb)
            // (STD: only L's, and only for the rest of the block)
            if (wv < (STD ? 1 : 2) && (!STD || c0 + PW < nbj)) {
                T yr[4], yi[4];
                const T *prow = pan + pl[c0 + min(l16, nb - 1)] * LS * P;
                auto entry = [&](int i, int k, bool in, T &cr, T &ci) {
                    const int kc = min(k, PW - 1);
                    const T vr = prow[kc * P], vi = CX ? prow[kc * P + 1] : T(0);
                    cr = in && i < nb && k < nb ? vr : T(0);
                    ci = in && i < nb && k < nb ? vi : T(0);
                };
                T *dst;
                if (wv == 0) {
                    tri_inverse16<T, CX, false>([&](int i, int k, T &cr, T &ci) { entry(i, k, k < i, cr, ci); }, T(1),
                                                T(0), yr, yi);
                    dst = STD || h == 0 ? sI1 : sI2;
                } else {
                    T dr, di, rr = T(1), ri = T(0);
                    entry(l16, l16, true, dr, di);
                    if (l16 < nb) {
                        if constexpr (CX) {
                            const T den = fma_(dr, dr, di * di);
                            rr = dr / den;
                            ri = -di / den;
                        } else {
                            rr = T(1) / dr;
                        }
                    }
                    tri_inverse16<T, CX, true>([&](int i, int k, T &cr, T &ci) { entry(i, k, k > i, cr, ci); }, rr, ri,
                                               yr, yi);
                    dst = h == 0 ? sV1 : sV2;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    T *d = dst + (l16 * TD_LS + 4 * g + q) * P;
                    d[0] = yr[q];
                    if constexpr (CX) d[1] = yi[q];
                }
            }
            if (c0 + PW < nbj) {
                // the rest of the block, one tile of 16 columns at a time (those
                // of finished panels in it get garbage): U12 = L11^{-1} A12, then
                // C -= L21 U12
                T *u0 = ub1, *u12 = ub2;   // 16 x 16 blocks of row stride TD_LS
#pragma unroll
                for (int sj = 0; sj < 2; ++sj) {
                    if (16 * sj + 16 <= c0 + PW) continue;
                    if constexpr (PW < 16) {
                        __syncthreads();   // the previous tile's U blocks are read
                        for (int e = tid; e < 16 * (16 - PW); e += NTH) u0[(PW + e / 16) * TD_LS + e % 16] = T(0);
                    }
#pragma unroll
                    for (int s = 0; s < SLOTS; ++s) {
                        const int t = wv + NW * s;
                        if (t >= J && t < nt) {
#pragma unroll
                            for (int si = 0; si < 2; ++si)
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const int r = 32 * (t - J) + 16 * si + V::row(g, i);
                                    const int q = r < mr ? rk[r] - c0 : -1;
                                    if (q >= 0) {
                                        u0[(q * TD_LS + l16) * P] = ar[s][si][sj][i];
                                        if constexpr (CX) u0[(q * TD_LS + l16) * P + 1] = ai[s][si][sj][i];
                                    }
                                }
                        }
                    }
                    __syncthreads();
                    if (wv == 0) {
                        acc_t dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
                        mm16<T, CX>(sI1, u0, dr, di);
                        if constexpr (STD) {
                            bool fin = true;
#pragma unroll
                            for (int i = 0; i < 4; ++i) fin = fin && finite_(dr[i]);
                            if (__any(!fin)) {
                                // an infinity or NaN must not reach the rows above
                                // it: by substitution, one column per lane
#pragma unroll 1
                                for (int i = 0; i < PW; ++i) {
                                    const T *li = pan + pl[c0 + i] * LS;
                                    T v = u0[i * TD_LS + l16];
#pragma unroll 1
                                    for (int k = 0; k < i; ++k) v = fma_(-li[k], u12[k * TD_LS + l16], v);
                                    u12[i * TD_LS + l16] = v;
                                }
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    dr[i] = V::row(g, i) < PW ? u12[V::row(g, i) * TD_LS + l16] : T(0);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = V::row(g, i), c = 16 * sj + l16;
                            u12[(r * TD_LS + l16) * P] = dr[i];
                            if constexpr (CX) u12[(r * TD_LS + l16) * P + 1] = di[i];
                            if (r < PW && c >= c0 + PW && c < nbj) {
                                const unsigned o = cur[j0 + pl[c0 + r]] * ldb + jb + c * sizeof(T);
                                *at(Ar, o) = dr[i];
                                if constexpr (CX) *at(Ai, o) = di[i];
                            }
                        }
                    }
                    __syncthreads();
                    constexpr int HP = PW / (4 * W);
                    T br[HP][W], bi[HP][W];
#pragma unroll
                    for (int hh = 0; hh < HP; ++hh)
#pragma unroll
                        for (int s = 0; s < W; ++s) {
                            const T *q = u12 + ((4 * W * hh + W * g + s) * TD_LS + l16) * P;
                            br[hh][s] = -q[0];
                            bi[hh][s] = CX ? -q[CX ? 1 : 0] : T(0);
                        }
#pragma unroll
                    for (int s = 0; s < SLOTS; ++s) {
                        const int t = wv + NW * s;
                        if (t >= J && t < nt) {
#pragma unroll
                            for (int si = 0; si < 2; ++si) {
                                const T *q = pan + min(32 * (t - J) + 16 * si + l16, mr - 1) * LS * P;
#pragma unroll
                                for (int hh = 0; hh < HP; ++hh)
#pragma unroll
                                    for (int u = 0; u < W; ++u) {
                                        const int k = 4 * W * hh + W * g + u;
                                        const T lr = q[k * P];
                                        ar[s][si][sj] = V::mfma(lr, br[hh][u], ar[s][si][sj]);
                                        if constexpr (CX) {
                                            const T li = q[k * P + 1];
                                            ar[s][si][sj] = V::mfma(-li, bi[hh][u], ar[s][si][sj]);
                                            ai[s][si][sj] = V::mfma(lr, bi[hh][u], ai[s][si][sj]);
                                            ai[s][si][sj] = V::mfma(li, br[hh][u], ai[s][si][sj]);
                                        }
                                    }
                            }
                        }
                    }
                }
            }
        });
        __syncthreads();
        // ---- the diagonal block: L_JJ^{-1} = [I1; -I2 L21 I1, I2], U_JJ^{-1} =
        //      [V1, -V1 U12 V2; V2] -------------------------------------------------------
        if (!STD && wv < 2) {
            // scratch blocks: L21, product of the lower part, product of the upper part
            T *l21 = ub1, *p1 = ub1 + SB, *p2 = pan;
            acc_t dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
            if (nbj > 16) {
                if (wv == 0) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r = 4 * q + g;   // panel row of pivot 16 + r, columns l16
                        T vr = T(0), vi = T(0);
                        if (16 + r < nbj) {
                            const unsigned o = cur[j0 + pl[16 + r]] * ldb + jb + l16 * sizeof(T);
                            vr = *at(Ar, o);
                            if constexpr (CX) vi = *at(Ai, o);
                        }
                        l21[(r * TD_LS + l16) * P] = vr;
                        if constexpr (CX) l21[(r * TD_LS + l16) * P + 1] = vi;
                    }
                    mm16<T, CX>(l21, sI1, dr, di);
                } else {
                    mm16<T, CX>(ub2, sV2, dr, di);
                }
                T *pp = wv == 0 ? p1 : p2;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pp[(V::row(g, i) * TD_LS + l16) * P] = -dr[i];
                    if constexpr (CX) pp[(V::row(g, i) * TD_LS + l16) * P + 1] = -di[i];
                }
                dr = acc_t{0, 0, 0, 0};
                di = acc_t{0, 0, 0, 0};
                if (wv == 0) mm16<T, CX>(sI2, p1, dr, di);
                else mm16<T, CX>(sV1, p2, dr, di);
            }
            // wavefront 0: strict lower part, wavefront 1: upper triangle
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const T *src = wv == 0 ? (b ? sI2 : sI1) : (b ? sV2 : sV1);
                for (int q = 0; q < 4; ++q) {
                    const int r = 4 * q + g, c = l16;
                    const bool in = wv == 0 ? c < r : c >= r;
                    if (in && 16 * b + r < nbj && 16 * b + c < nbj) {
                        const unsigned o = cur[j0 + pl[16 * b + r]] * ldb + jb + (16 * b + c) * sizeof(T);
                        *at(Ar, o) = src[(r * TD_LS + c) * P];
                        if constexpr (CX) *at(Ai, o) = src[(r * TD_LS + c) * P + 1];
                    }
                }
            }
            if (nbj > 16) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = V::row(g, i) + (wv == 0 ? 16 : 0), c = l16 + (wv == 0 ? 0 : 16);
                    if (r < nbj && c < nbj) {
                        const unsigned o = cur[j0 + pl[r]] * ldb + jb + c * sizeof(T);
                        *at(Ar, o) = dr[i];
                        if constexpr (CX) *at(Ai, o) = di[i];
                    }
                }
            }
        }
        // ---- positions after the block's interchanges --------------------------------------
        int row[RPT];
#pragma unroll
        for (int i = 0; i < RPT; ++i) row[i] = cur[j0 + min(row_of(i), mr - 1)];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (row_of(i) < mr) cur[j0 + lg[i]] = row[i];
        __syncthreads();
    }
    if constexpr (!STD) {
        for (int p = tid; p < m; p += NTH) ip[p] = cur[p];
    } else {
        // rows to their positions, 32 columns at a time through registers
#pragma unroll 1
        for (int J = 0; J < nt; ++J) {
            int lane = tid & 63;
            asm volatile("" : "+v"(lane));
            const int c = 32 * J + (lane & 31);
            const unsigned cb = min(c, m - 1) * sizeof(T);
            T v[SLOTS][16];
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    v[s][i] = *at(Ar, cur[min(32 * (wv + NW * s) + 2 * i + (lane >> 5), m - 1)] * ldb + cb);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int p = 32 * (wv + NW * s) + 2 * i + (lane >> 5);
                    if (p < m && c < m) *at(Ar, p * ldb + cb) = v[s][i];
                }
            __syncthreads();
        }
    }
}

template <typename T, bool CX, int NW, int SLOTS, int RPT>
__global__ void __launch_bounds__(64 * NW, 2) lu_td_kernel(T *__restrict__ A, int *__restrict__ perm, int m, int ld,
                                                        long long a_stride, int *info)
{
    extern __shared__ unsigned char lds_raw[];
    lu_left<T, CX, NW, SLOTS, RPT, TD_PW, false>(A + (long long)blockIdx.x * a_stride, m, ld,
                                                 perm + (long long)blockIdx.x * m, info, lds_raw);
}

// a batch of real matrices of mixed sizes in LAPACK's format, one workgroup per
// matrix (block b: entry b of the metadata).  LARGE: above 512 rows.
constexpr int STD_SMALL_M = 512;
template <typename T, bool LARGE>
__global__ void __launch_bounds__(LARGE ? 512 : 256, 2) lu_std_kernel(T *__restrict__ A, int *__restrict__ piv, LuBatch B,
                                                                   int *info)
{
    extern __shared__ unsigned char lds_raw[];
    const int m = __builtin_amdgcn_readfirstlane(B.m_of[blockIdx.x]);
    T *a = A + B.a_off[blockIdx.x];
    int *ip = piv + B.p_off[blockIdx.x];
    if constexpr (LARGE) {
        constexpr int PW = sizeof(T) == 8 ? 8 : 16;
        if constexpr (sizeof(T) == 4) {
            if (m > 1280) {
                lu_left<T, false, 8, 8, 4, PW, true>(a, m, m, ip, info, lds_raw);
                return;
            }
        }
        lu_left<T, false, 8, 5, 3, PW, true>(a, m, m, ip, info, lds_raw);
    } else {
        if (m <= 256) lu_left<T, false, 4, 2, 1, 16, true>(a, m, m, ip, info, lds_raw);
        else lu_left<T, false, 4, 4, 2, 16, true>(a, m, m, ip, info, lds_raw);
    }
}

// ---------------------------------------------------------------------------
// sweeps: one patch per workgroup
// ---------------------------------------------------------------------------
constexpr int TDS_THREADS = 256;   // 32 rows x 8 lanes

// four consecutive factor entries of a row
template <typename TP, typename TF> struct Quad {
    TP v[4];
    __device__ __forceinline__ void load(const TF *p)
    {
        if constexpr (std::is_same<TF, unsigned short>::value) {
            typedef unsigned short u16x4 __attribute__((ext_vector_type(4), aligned(2)));
            const u16x4 q = *(const u16x4 *)p;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = __uint_as_float((unsigned)q[i] << 16);
        } else {
            typedef TF seg __attribute__((ext_vector_type(16 / sizeof(TF)), aligned(sizeof(TF))));
            constexpr int W = 16 / sizeof(TF);
#pragma unroll
            for (int h = 0; h < 4 / W; ++h) {
                const seg q = *(const seg *)(p + W * h);
#pragma unroll
                for (int i = 0; i < W; ++i) v[W * h + i] = q[i];
            }
        }
    }
    // columns c .. c+3 of a row of MS entries; entries past its end repeat the
    // last one (their unknowns are zero)
    __device__ __forceinline__ void load_edge(const TF *row, int c, int MS)
    {
        if (c + 4 <= MS) {
            load(row + c);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const TF q = row[min(c + i, MS - 1)];
                if constexpr (std::is_same<TF, unsigned short>::value) v[i] = __uint_as_float((unsigned)q << 16);
                else v[i] = q;
            }
        }
    }
};

// sum over the 8 lanes of a row group, in every lane (fixed order)
template <typename T> __device__ __forceinline__ T sum8(T x)
{
    x += dpp<0xB1, 0xf>(x);    // quad_perm 1,0,3,2
    x += dpp<0x4E, 0xf>(x);    // quad_perm 2,3,0,1
    x += dpp<0x141, 0xf>(x);   // row_half_mirror
    return x;
}

// Substitutions with the factors of lu_td_kernel, b (br, bi, NB blocks of 32,
// zero padded) in LDS, overwritten.  Bound by the read of the factors where
// there are enough of them (r = 3, 13824 cells: 4.2 -> 3.3 ms, 5.3 TB/s; a
// device copy reaches 5.2), by the chain of block rows below (r = 1, 4096
// cells: 145 -> 62 us; before, each diagonal block was substituted by one
// wavefront, 32 dependent steps).  Per block of 32 rows: the products with
// the solved blocks (8 lanes per row, 16 bytes per lane and block: every row
// segment is a whole 128-byte line in FP32), then the inverse diagonal block.
// The factors depend on nothing, so a batch of UB column blocks is in flight
// per thread and, up to three blocks (SMALL), the whole matrix before the
// first product.
template <typename TP, typename TF, bool CX, int MS, int LDM>
__device__ __forceinline__ void td_substitute(const TF *__restrict__ Lr, const TF *__restrict__ Li, const int *perm,
                                              TP *br, TP *bi, TP *tr, TP *ti)
{
    constexpr int NB = (MS + 31) / 32, UB = sizeof(TP) == 8 ? 2 : 4;
    const int tid = threadIdx.x, rr = tid >> 3, q4 = (tid & 7) * 4;
    using Q = Quad<TP, TF>;
    // s -= (or +=) row segment . x
    auto dot = [&](const Q &ar, const Q &ai, const TP *xr, const TP *xi, TP &sr, TP &si) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (CX) {
                sr = fma_(-ai.v[e], xi[e], fma_(ar.v[e], xr[e], sr));
                si = fma_(ai.v[e], xr[e], fma_(ar.v[e], xi[e], si));
            } else {
                sr = fma_(ar.v[e], xr[e], sr);
            }
        }
    };
    // the diagonal block: x_I = D^{-1} t (strictly lower with unit diagonal, or
    // upper), t = b_I - sums
    auto finish = [&](int I, bool lower, Q dr, Q di, TP sr, TP si) {
        sr = sum8(sr);
        if constexpr (CX) si = sum8(si);
        const int row = 32 * I + rr;
        if (q4 == 0) {
            // (rows past the end stay zero: the edge columns multiply them)
            tr[rr] = row < MS ? br[row] - sr : TP(0);
            if constexpr (CX) ti[rr] = row < MS ? bi[row] - si : TP(0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool in = lower ? q4 + e < rr : q4 + e >= rr;
            dr.v[e] = in ? dr.v[e] : TP(0);
            di.v[e] = in ? di.v[e] : TP(0);
        }
        __syncthreads();
        TP yr = 0, yi = 0;
        dot(dr, di, tr + q4, ti + q4, yr, yi);
        yr = sum8(yr);
        if constexpr (CX) yi = sum8(yi);
        if (q4 == 0 && row < MS) {
            br[row] = lower ? yr + tr[rr] : yr;
            if constexpr (CX) bi[row] = lower ? yi + ti[rr] : yi;
        }
        __syncthreads();
    };
    if constexpr (NB <= 3 && NB * NB * (CX ? 2 : 1) * sizeof(TP) <= 72) {
        Q fr[NB][NB], fi[CX ? NB : 1][CX ? NB : 1];
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            const int o = perm[min(32 * I + rr, MS - 1)] * LDM;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                fr[I][j].load_edge(Lr + o, 32 * j + q4, MS);
                if constexpr (CX) fi[I][j].load_edge(Li + o, 32 * j + q4, MS);
            }
        }
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            TP sr = 0, si = 0;
#pragma unroll
            for (int j = 0; j < I; ++j)
                dot(fr[I][j], fi[CX ? I : 0][CX ? j : 0], br + 32 * j + q4, bi + 32 * j + q4, sr, si);
            finish(I, true, fr[I][I], fi[CX ? I : 0][CX ? I : 0], sr, si);
        }
#pragma unroll
        for (int I = NB - 1; I >= 0; --I) {
            TP sr = 0, si = 0;
#pragma unroll
            for (int j = I + 1; j < NB; ++j)
                dot(fr[I][j], fi[CX ? I : 0][CX ? j : 0], br + 32 * j + q4, bi + 32 * j + q4, sr, si);
            finish(I, false, fr[I][I], fi[CX ? I : 0][CX ? I : 0], sr, si);
        }
    } else {
        // products with the column blocks [j0, j1) of one block row
        auto products = [&](int o, int j0, int j1, TP &sr, TP &si) {
#pragma unroll 1
            for (int jb = j0; jb < j1; jb += UB) {
                Q ar[UB], ai[CX ? UB : 1];
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    // (blocks past the range reload the last one against zero)
                    const int j = min(jb + u, j1 - 1);
                    ar[u].load_edge(Lr + o, 32 * j + q4, MS);
                    if constexpr (CX) ai[u].load_edge(Li + o, 32 * j + q4, MS);
                }
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    if (jb + u < j1)
                        dot(ar[u], ai[CX ? u : 0], br + 32 * (jb + u) + q4, bi + 32 * (jb + u) + q4, sr, si);
            }
        };
#pragma unroll 1
        for (int I = 0; I < NB; ++I) {
            const int o = perm[min(32 * I + rr, MS - 1)] * LDM;
            Q dr, di;
            dr.load_edge(Lr + o, 32 * I + q4, MS);
            if constexpr (CX) di.load_edge(Li + o, 32 * I + q4, MS);
            else di = dr;
            TP sr = 0, si = 0;
            products(o, 0, I, sr, si);
            finish(I, true, dr, di, sr, si);
        }
#pragma unroll 1
        for (int I = NB - 1; I >= 0; --I) {
            const int o = perm[min(32 * I + rr, MS - 1)] * LDM;
            Q dr, di;
            dr.load_edge(Lr + o, 32 * I + q4, MS);
            if constexpr (CX) di.load_edge(Li + o, 32 * I + q4, MS);
            else di = dr;
            TP sr = 0, si = 0;
            products(o, I + 1, NB, sr, si);
            finish(I, false, dr, di, sr, si);
        }
    }
}

template <int DIM, int R> struct TdSize {
    static constexpr int N1 = R + 2;
    static constexpr int NL = DIM == 2 ? N1 * N1 : N1 * N1 * N1;
    static constexpr int NPM = DIM == 2 ? (R + 1) * (R + 2) / 2 : (R + 1) * (R + 2) * (R + 3) / 6;
    static constexpr int NV = DIM * NL, MS = NV + NPM, MSP = (MS + 31) & ~31;
};

// one time-decoupled patch solve per cell: gather the patch defect of all
// time nodes, per eigen-system transform (with the row permutation of the
// factors), substitute, transform back; velocity to the cell buffer E, pressure
// updated in place (pressure unknowns belong to one cell)
template <int DIM, int R, typename T, typename TP, typename TF>
__global__ void __launch_bounds__(TDS_THREADS, sizeof(TP) == 8 ? 2 : 4) solve_td_kernel(SolveTdArgs<T, TP, TF> A)
{
    using Z = TdSize<DIM, R>;
    constexpr int N1 = Z::N1, NL = Z::NL, NPM = Z::NPM, NV = Z::NV, MS = Z::MS, MSP = Z::MSP;
    constexpr int LDM = td_ld(MS);
    constexpr long long MAT = (long long)MS * LDM;
    extern __shared__ unsigned char lds_raw[];
    const int nt = A.nt;
    TP *br = reinterpret_cast<TP *>(lds_raw), *bi = br + MSP, *tr = bi + MSP, *ti = tr + 32;
    TP *rl = ti + 32;                           // [nt][MSP] patch defect
    TP *out = rl + nt * MSP;                    // [nt][MSP] patch correction
    int *perm = reinterpret_cast<int *>(out + nt * MSP);   // [MSP]
    const int cell = xcd_cell(blockIdx.x, gridDim.x), tid = threadIdx.x;
    const int c0 = cell % A.n0, c1 = (cell / A.n0) % A.n1, c2 = DIM == 3 ? cell / (A.n0 * A.n1) : 0;
    const long long N0 = (long long)(R + 1) * A.n0 + 1, N1g = (long long)(R + 1) * A.n1 + 1;
    const long long pbase = (long long)nt * A.Nv1;
    for (int j = tid; j < MS; j += TDS_THREADS) {
        perm[j] = A.perm[0][(long long)cell * MS + j];
        long long g, st;
        if (j < NV) {
            const int l = j % NL, c = j / NL;
            const int i0 = l % N1, i1 = (l / N1) % N1, i2 = DIM == 3 ? l / (N1 * N1) : 0;
            g = c * A.Nn +
                (((long long)(R + 1) * c0 + i0) + N0 * (((long long)(R + 1) * c1 + i1) + N1g * ((long long)(R + 1) * c2 + i2)));
            st = A.Nv1;
        } else {
            g = pbase + (long long)cell * NPM + (j - NV);
            st = A.Np1;
        }
        for (int a = 0; a < nt; ++a) {
            rl[a * MSP + j] = (TP)A.defect[g + a * st];
            out[a * MSP + j] = TP(0);
        }
    }
    __syncthreads();
    for (int s = 0; s < A.nsys; ++s) {
        const bool cx = A.cplx[s] != 0;
        if (s > 0) {
            for (int i = tid; i < MS; i += TDS_THREADS) perm[i] = A.perm[s][(long long)cell * MS + i];
            __syncthreads();
        }
        for (int i = tid; i < MSP; i += TDS_THREADS) {
            TP sr = 0, si = 0;
            if (i < MS) {
                const int src = perm[i];
                for (int a = 0; a < nt; ++a) {
                    sr = fma_(A.Tre[s * 4 + a], rl[a * MSP + src], sr);
                    si = fma_(A.Tim[s * 4 + a], rl[a * MSP + src], si);
                }
            }
            br[i] = sr;
            bi[i] = si;
        }
        __syncthreads();
        const TF *LU = A.sys[s] + (long long)cell * (cx ? 2 : 1) * MAT;
        if (cx) td_substitute<TP, TF, true, MS, LDM>(LU, LU + MAT, perm, br, bi, tr, ti);
        else td_substitute<TP, TF, false, MS, LDM>(LU, LU, perm, br, bi, tr, ti);
        for (int j = tid; j < MS; j += TDS_THREADS)
            for (int a = 0; a < nt; ++a) {
                TP v = A.Fre[a * 4 + s] * br[j];
                if (cx) v = fma_(-A.Fim[a * 4 + s], bi[j], v);
                out[a * MSP + j] += v;
            }
        __syncthreads();
    }
    T *Ec = A.E + (long long)cell * nt * NV;
    for (int j = tid; j < MS; j += TDS_THREADS)
        for (int a = 0; a < nt; ++a) {
            if (j < NV) Ec[a * NV + j] = (T)out[a * MSP + j];
            else {
                T &d = A.d[pbase + a * A.Np1 + (long long)cell * NPM + (j - NV)];
                d = fma_(A.omega, (T)out[a * MSP + j], d);
            }
        }
}

} // namespace

// Workgroup shapes, by the row tiles that the accumulators hold (32 rows and
// 32 columns each: 16 registers per lane and plane in FP32, 32 in FP64, of 256):
// two workgroups of 4 wavefronts per CU share it best (FP32 complex m = 395,
// 4096 matrices: 13.9 ms, 17.0 ms with one of 8 wavefronts); up to 128 rows 2
// wavefronts (cheaper barriers: 8192 of m = 85 in 1.2 instead of 1.6 ms); FP64
// complex tiles need 8 wavefronts from 129 rows on.
template <typename T>
hipError_t launch_lu_td(T *A, int *perm, int m, int ld, bool cplx, int batch, int *info, hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    const long long st = (long long)(cplx ? 2 : 1) * m * ld;
#define LTD(CX, NW, SLOTS, RPT)                                                                                        \
    {                                                                                                                  \
        static_assert(SLOTS <= 2 * RPT, "panel rows cover the tiles");                                                 \
        const size_t bytes = left_lu_lds_bytes<T, CX, TD_PW, false>(m);                                                                \
        hipError_t e = lds_attr((const void *)lu_td_kernel<T, CX, NW, SLOTS, RPT>, bytes);                             \
        if (e != hipSuccess) return e;                                                                                 \
        hipLaunchKernelGGL((lu_td_kernel<T, CX, NW, SLOTS, RPT>), dim3(batch), dim3(64 * NW), bytes, s, A, perm, m,    \
                           ld, st, info);                                                                              \
        return hipGetLastError();                                                                                      \
    }
    constexpr bool wide = sizeof(T) == 8;
    if (m < 17 || m > 512) return hipErrorInvalidValue;
    if (cplx) {
        if constexpr (wide) {
            if (m <= 128) LTD(true, 4, 1, 1)
            if (m <= 256) LTD(true, 8, 1, 1)
            LTD(true, 8, 2, 1)
        } else {
            if (m <= 128) LTD(true, 2, 2, 1)
            if (m <= 256) LTD(true, 4, 2, 1)
            LTD(true, 4, 4, 2)
        }
    }
    if (m <= 128) LTD(false, 2, 2, 1)
    if (m <= 256) LTD(false, 4, 2, 1)
    LTD(false, 4, 4, 2)
#undef LTD
}

template <typename T, typename TP, typename TF>
hipError_t launch_solve_td(int dim, int r, const SolveTdArgs<T, TP, TF> &a, int ncell, hipStream_t s)
{
#define SC(D, RR)                                                                                                      \
    if (dim == D && r == RR) {                                                                                         \
        constexpr size_t msp = TdSize<D, RR>::MSP;                                                                     \
        const size_t bytes = ((2 + 2 * (size_t)a.nt) * msp + 64) * sizeof(TP) + msp * sizeof(int);                     \
        hipError_t e = lds_attr((const void *)solve_td_kernel<D, RR, T, TP, TF>, bytes);                               \
        if (e != hipSuccess) return e;                                                                                 \
        hipLaunchKernelGGL((solve_td_kernel<D, RR, T, TP, TF>), dim3(ncell), dim3(TDS_THREADS), bytes, s, a);         \
        return hipGetLastError();                                                                                      \
    }
    SC(2, 1) SC(2, 2) SC(2, 3) SC(3, 1) SC(3, 2) SC(3, 3)
#undef SC
    return hipErrorInvalidValue;
}

// Large matrices first (the batch is sorted by decreasing size): one launch of
// 8 wavefronts per matrix and one or two matrices per CU above 512 rows, one
// of 4 wavefronts and two to four matrices per CU for the rest.
template <typename T>
hipError_t launch_lu_std(T *A, int *piv, const LuBatch &b, const int *m_host, int batch, int *info, hipStream_t s)
{
    int nl = 0;
    while (nl < batch && m_host[nl] > STD_SMALL_M) ++nl;
#define LSTD(LARGE, NTH, PW, M, N, MB)                                                                                 \
    {                                                                                                                  \
        const size_t bytes = left_lu_lds_bytes<T, false, PW, true>(M);                                                 \
        hipError_t e = lds_attr((const void *)lu_std_kernel<T, LARGE>, bytes);                                         \
        if (e != hipSuccess) return e;                                                                                 \
        hipLaunchKernelGGL((lu_std_kernel<T, LARGE>), dim3(N), dim3(NTH), bytes, s, A, piv, MB, info);                 \
        e = hipGetLastError();                                                                                         \
        if (e != hipSuccess) return e;                                                                                 \
    }
    if (nl > 0 && m_host[0] > lu_std_max_m(sizeof(T) == 8)) return hipErrorInvalidValue;
    if (nl > 0) LSTD(true, 512, (sizeof(T) == 8 ? 8 : 16), m_host[0], nl, b)
    if (nl < batch) {
        LuBatch r = b;
        r.m_of += nl;
        r.a_off += nl;
        r.p_off += nl;
        LSTD(false, 256, 16, m_host[nl], batch - nl, r)
    }
#undef LSTD
    return hipSuccess;
}

template hipError_t launch_lu_std<double>(double *, int *, const LuBatch &, const int *, int, int *, hipStream_t);
template hipError_t launch_lu_std<float>(float *, int *, const LuBatch &, const int *, int, int *, hipStream_t);
template hipError_t launch_lu_td<double>(double *, int *, int, int, bool, int, int *, hipStream_t);
template hipError_t launch_lu_td<float>(float *, int *, int, int, bool, int, int *, hipStream_t);
template hipError_t launch_solve_td(int, int, const SolveTdArgs<double, double, double> &, int, hipStream_t);
template hipError_t launch_solve_td(int, int, const SolveTdArgs<float, float, float> &, int, hipStream_t);
template hipError_t launch_solve_td(int, int, const SolveTdArgs<float, float, unsigned short> &, int, hipStream_t);

} // namespace stmg
