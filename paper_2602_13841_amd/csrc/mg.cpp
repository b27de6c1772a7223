// hp space-time multigrid (Sec. "Preconditioning of GMRES by hp space-time
// multigrid"), FGMRES (eq. inexact) and the inexact Newton method with
// Eisenstat-Walker forcing and nonmonotone Armijo backtracking (Alg.
// "Inexact Newton-Krylov", Alg. "Armijo").  Host code driving device
// kernels; the Givens rotations run on the device (one FP64 workgroup), and
// the stopping tests and the line search use scalars read back once per
// iteration.
//
// Readings where the paper leaves details open:
// * hierarchy: p-coarsening first, (k, r) -> (k, max(1, r//2)) by default,
//   (k//2 if k >= 2 else k, max(1, r//2)) with time_coarsening = 1, then
//   h-coarsening while every n is even and >= 4;
// * level operators: rediscretized at the finer state evaluated at the
//   coarser nodes and Radau nodes; the coarsest level is solved directly in
//   FP64, bordered by the constant pressure of each time node when Gamma_D
//   is the whole boundary;
// * smoother relaxation: each unknown's correction divided by the number of
//   patches holding it, omega = 1 (default), or the plain sum with a scalar
//   omega = 1.4 / 2^d;
// * FGMRES: Arnoldi in the M_n inner product, classical Gram-Schmidt with
//   one reorthogonalization, zero initial guess, no restart;
// * Newton: Eisenstat-Walker update of Alg. "Inexact Newton-Krylov";
//   g0 = (M r).(J dU); the nonmonotone window keeps the last accepted merit
//   values across Newton steps of a slab; interpolated backtracking uses the
//   quadratic model after the first failure and the cubic model through the
//   last two failures, clamped to [0.1 alpha, 0.5 alpha]; the rebuild
//   thresholds theta_N, theta_L, kappa_abs, (s, theta) are options.
#include "mg.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>

namespace stmg {

// progress log on stderr when the environment variable STMG_VERBOSE is set
static bool verbose()
{
    static int v = -1;
    if (v < 0) {
        const char *e = std::getenv("STMG_VERBOSE");
        v = (e && *e && *e != '0') ? 1 : 0;
    }
    return v == 1;
}

static double now_s()
{
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

namespace {

template <typename T> T *state_of(MgLevel &M) { return std::is_same<T, double>::value ? M.st64.as<T>() : M.st32.as<T>(); }

std::vector<double> coarse_vertices(const std::vector<double> &v, int dim, const int n[3])
{
    if (v.empty()) return {};
    std::vector<double> out;
    int nz = dim == 3 ? n[2] : 0;
    for (int i2 = 0; i2 <= nz; i2 += 2)
        for (int i1 = 0; i1 <= n[1]; i1 += 2)
            for (int i0 = 0; i0 <= n[0]; i0 += 2) {
                long long idx = i0 + (long long)(n[0] + 1) * (i1 + (long long)(n[1] + 1) * i2);
                for (int a = 0; a < dim; ++a) out.push_back(v[idx * dim + a]);
            }
    return out;
}

} // namespace

void Krylov::ensure(long long N_, int maxit_)
{
    if (N_ == N && maxit_ <= maxit) return;
    if (maxit > 0) throw HipError("Krylov workspace was sized for fewer iterations", STMG_EINVAL);
    N = N_;
    maxit = maxit_;
    V.alloc(sizeof(double) * N * (maxit + 1));
    MV.alloc(sizeof(double) * N * (maxit + 1));
    Z.alloc(sizeof(double) * N * maxit);
    w.alloc(sizeof(double) * N);
    u.alloc(sizeof(double) * N);
    h.alloc(sizeof(double) * 3 * (maxit + 2));
    partial.alloc(sizeof(double) * multidot_partial_words(maxit + 1));
    y.alloc(sizeof(double) * (maxit + 1));
    H.alloc(sizeof(double) * (maxit + 1) * maxit);
    cs.alloc(sizeof(double) * maxit);
    sn.alloc(sizeof(double) * maxit);
    g.alloc(sizeof(double) * (maxit + 1));
    report.alloc(sizeof(double) * 2);
    for (DevBuf *b : {&r, &Mr, &dU, &Ut, &rt, &tmp}) b->alloc(sizeof(double) * N);
    dot.alloc(8 * 8);
}

void mg_build(stmg_ctx *ctx)
{
    auto mg = std::make_unique<Mg>();
    const stmg_options &o = ctx->opt;
    Level &L0 = *ctx->levels[0];
    mg->prec = o.prec_mg == STMG_F64 ? STMG_F64 : STMG_F32;
    mg->weighting = o.vanka_weighting ? 1 : 0;
    mg->td = o.vanka_time_decoupled != 0;
    mg->omega = o.vanka_omega > 0 ? o.vanka_omega : (mg->weighting ? 1.0 : 1.4 / double(1 << L0.dim));
    mg->nu1 = std::max(0, o.nu1);
    mg->nu2 = std::max(0, o.nu2);
    mg->use_graph = o.use_graphs != 0;
    mg->diag = o.vanka_diagonal != 0 && mg->td;
    mg->diag_block = o.vanka_diagonal == 2;
    mg->factor_bf16 = o.vanka_factor_bf16 != 0 && mg->prec == STMG_F32 && mg->td && !mg->diag;
    int dev = 0, lds = 65536;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess)
        mg->max_lds = (size_t)lds;
    mg->max_lds = mg->max_lds > 8192 ? mg->max_lds - 8192 : mg->max_lds;   // static LDS of the LU kernel
    int k = L0.k, r = L0.r, n[3] = {L0.n[0], L0.n[1], L0.n[2]};
    const int maxl = o.max_levels;
    std::vector<char> kinds;
    std::vector<double> verts = L0.vert_host;
    auto count = [&]() { return (int)ctx->levels.size(); };
    const bool tcoarse = o.time_coarsening != 0;
    while ((r > 1 || (tcoarse && k > 1)) && (maxl == 0 || count() < maxl)) {
        r = std::max(1, r / 2);
        if (tcoarse) k = k >= 2 ? k / 2 : k;
        auto L = std::make_unique<Level>();
        L->init(ctx->prob, k, r, n[0], n[1], n[2], r == L0.r ? L0.nq : default_nq(r), verts);
        L->timers = &ctx->timers;
        ctx->levels.push_back(std::move(L));
        kinds.push_back('p');
    }
    auto hok = [&]() {
        for (int a = 0; a < L0.dim; ++a)
            if (n[a] % 2 != 0 || n[a] < 4) return false;
        return true;
    };
    while (hok() && (maxl == 0 || count() < maxl)) {
        verts = coarse_vertices(verts, L0.dim, n);
        for (int a = 0; a < L0.dim; ++a) n[a] /= 2;
        auto L = std::make_unique<Level>();
        L->init(ctx->prob, k, r, n[0], n[1], n[2], r == L0.r ? L0.nq : default_nq(r), verts);
        L->timers = &ctx->timers;
        ctx->levels.push_back(std::move(L));
        kinds.push_back('h');
    }
    const int nl = (int)ctx->levels.size();
    mg->lv.resize(nl);
    for (int l = 0; l < nl; ++l) {
        MgLevel &M = mg->lv[l];
        M.L = ctx->levels[l].get();
        size_t N = (size_t)M.L->N;
        M.st64.alloc(N * 8);
        if (!arena_counting()) STMG_HIP(vec_fill<double>((long long)N, 0.0, M.st64.as<double>(), ctx->stream));
        if (mg->prec == STMG_F32) {
            M.st32.alloc(N * 4);
            if (!arena_counting()) STMG_HIP(vec_fill<float>((long long)N, 0.0f, M.st32.as<float>(), ctx->stream));
        }
        size_t w = mg->prec == STMG_F64 ? 8 : 4;
        M.r.alloc(N * w);
        M.d.alloc(N * w);
        M.t.alloc(N * w);
        M.E.alloc((size_t)M.L->ncell * M.L->nt * M.L->dim * M.L->nl * w);
    }
    for (int l = 0; l + 1 < nl; ++l) {
        auto T = std::make_unique<Transfer>();
        T->build(*ctx->levels[l], *ctx->levels[l + 1], kinds[l]);
        mg->tr.push_back(std::move(T));
    }
    mg->border = L0.dmask == (unsigned)((1 << (2 * L0.dim)) - 1);
    ctx->mg = std::move(mg);
    mg_allocate(ctx);
}

// Every buffer the context will use, allocated once here with its final size
// (nothing is allocated later, so the bytes consumed at creation are the
// context's whole footprint): operator work buffers, smoother buffers of every
// smoothed level, the coarse-level matrices, the Krylov and Newton vectors,
// the staging of the captured V-cycle and the slab data.
void mg_allocate(stmg_ctx *ctx)
{
    Mg &mg = *ctx->mg;
    const stmg_options &o = ctx->opt;
    const int nl = (int)mg.lv.size();
    const size_t w = mg.prec == STMG_F64 ? 8 : 4;
    for (int l = 0; l < nl; ++l) {
        Level &L = *mg.lv[l].L;
        // FP64 everywhere (Newton, level states, the coarse matrix assembly with
        // one column per unknown on the coarsest level), FP32 for an FP32
        // multigrid and for FP32 applications of the slab operator
        const bool coarsest = l == nl - 1;
        L.alloc_work(coarsest ? (int)std::max<long long>(1, L.N) : 1,
                     (mg.prec == STMG_F32 || l == 0) ? 1 : 0);
    }
    for (int l = 0; l + 1 < nl; ++l) {
        MgLevel &M = mg.lv[l];
        Level &L = *M.L;
        M.vstar.alloc((size_t)L.Nv1 * w);
        M.elem.alloc((size_t)L.ncell * elem_record_words(L.dim, L.r) * w);
        M.m = L.nt * (L.dim * L.nl + L.npm);
        M.ms = L.dim * L.nl + L.npm;
        M.info.alloc(4);
        if (mg.td) {
            // one spatial system per eigen-system of the time coupling; which
            // systems are complex depends only on k
            M.tdg = time_diagonalization(L.tc);
            const long long ms = M.ms, ld = td_ld(M.ms), mat = ms * ld;
            long long off = 0;
            for (int sy = 0; sy < M.tdg.nsys; ++sy) {
                M.sys_off[sy] = off;
                M.piv_off[sy] = (long long)sy * L.ncell * ms;
                off += (long long)L.ncell * (M.tdg.cplx[sy] ? 2 : 1) * mat;
            }
            M.nfac = off;
            M.patches.alloc((size_t)off * w);
            const size_t ib = (size_t)M.tdg.nsys * L.ncell * ms * 4;
            M.perm.alloc(ib);
            if (mg.diag) {
                const int nv = mg.diag_block ? L.nl * L.dim * L.dim : L.dim * L.nl, npm = L.npm, ns = M.tdg.nsys;
                M.dv_dinv.alloc((size_t)ns * L.ncell * 2 * nv * w);
                M.dv_schur.alloc((size_t)ns * L.ncell * 2 * npm * npm * w);
                M.dv_piv.alloc((size_t)ns * L.ncell * npm * sizeof(int));
            } else if (mg.factor_bf16) {
                M.fac16.alloc((size_t)off * 2);
            }
        } else {
            M.patches.alloc((size_t)L.ncell * M.m * M.m * w);
            M.piv.alloc((size_t)L.ncell * M.m * 4);
        }
    }
    // coarsest level: dense Jacobian (bordered by the constant pressures of
    // each time node when every face is Dirichlet) and its inverse (LU beyond DINV_MAX_M)
    {
        Level &Lc = *mg.lv[nl - 1].L;
        const int n = (int)Lc.N, m = n + (mg.border ? Lc.nt : 0);
        mg.cX.alloc((size_t)n * n * 8);
        mg.cY.alloc((size_t)n * n * 8);
        mg.cn = n;
        mg.cm = m;
        mg.inverse = m <= DINV_MAX_M;
        if (mg.inverse) {
            const size_t ld = (size_t)dinv_ld(m);
            mg.cA.alloc((size_t)m * ld * 8);
            mg.cW.alloc(ld * 32 * 8);
            mg.cB.alloc(32 * ld * 8);
            mg.cP.alloc(32 * ld * 8);
            mg.cdinv.alloc(32 * 32 * 8);
            mg.crow.alloc((size_t)m * 4);
            mg.cperm.alloc((size_t)m * 4);
        } else {
            mg.cA.alloc((size_t)m * m * 8);
            mg.cpiv.alloc((size_t)m * 4);
            mg.cinfo.alloc(4);
            mg.cr64.alloc((size_t)m * 8);
            mg.cx64.alloc((size_t)m * 8);
        }
    }
    const long long N = mg.lv[0].L->N;
    ctx->kry.ensure(N, std::max(1, o.fgmres_maxit));
    if (mg.use_graph) {
        mg.graph.in.alloc((size_t)N * 8);
        mg.graph.out.alloc((size_t)N * 8);
    }
    ctx->rhs.alloc((size_t)N * 8);
    ctx->vprev.alloc((size_t)mg.lv[0].L->Nv1 * 8);
}

void mg_set_state(stmg_ctx *ctx, const double *u)
{
    Mg &mg = *ctx->mg;
    hipStream_t s = ctx->stream;
    mg.graph.reset(s);
    const int nl = (int)mg.lv.size();
    STMG_HIP(hipMemcpyAsync(mg.lv[0].st64.p, u, mg.lv[0].L->N * 8, hipMemcpyDeviceToDevice, s));
    for (int l = 1; l < nl; ++l)
        mg.tr[l - 1]->interpolate_state<double>(*mg.lv[l - 1].L, *mg.lv[l].L, mg.lv[l - 1].st64.as<double>(),
                                                mg.lv[l].st64.as<double>(), s);
    if (mg.prec == STMG_F32)
        for (int l = 0; l < nl; ++l)
            STMG_HIP((vec_cast<double, float>(mg.lv[l].L->N, mg.lv[l].st64.as<double>(), mg.lv[l].st32.as<float>(), s)));
    // coarsest level: dense Jacobian from J e_i, bordered, inverted in FP64
    // (beyond DINV_MAX_M unknowns: LU)
    MgLevel &C = mg.lv[nl - 1];
    Level &Lc = *C.L;
    const int n = (int)Lc.N, nb = mg.border ? Lc.nt : 0, m = n + nb;
    if (mg.cn != n || mg.cm != m) throw HipError("coarse-level buffers not prepared", STMG_ESTATE);
    {
        TimerScope ts(&ctx->timers, "coarse_factor", s);
        STMG_HIP(launch_identity(mg.cX.as<double>(), n, s));
        Lc.apply<double>(Mode::Jac, C.st64.as<double>(), mg.cX.as<double>(), mg.cY.as<double>(), nullptr, nullptr, n, s);
        if (mg.inverse) {
            const DenseInverse w = mg.dense_inverse();
            STMG_HIP(launch_inv_matrix(mg.cY.as<double>(), n, nb, (long long)Lc.nt * Lc.Nv1, Lc.Np1, Lc.npm, w, s));
            STMG_HIP(launch_dense_inverse(w, s));
        } else {
            STMG_HIP(launch_coarse_matrix(mg.cY.as<double>(), n, nb, Lc.nt, (long long)Lc.nt * Lc.Nv1, Lc.Np1, Lc.npm,
                                          Lc.ncell, mg.cA.as<double>(), s));
            STMG_HIP(hipMemsetAsync(mg.cinfo.p, 0, 4, s));
            STMG_HIP(launch_lu_dense(mg.cA.as<double>(), mg.cpiv.as<int>(), m, mg.cinfo.as<int>(), s));
        }
    }
    mg.state_set = true;
}

template <typename T> static void rebuild_level(stmg_ctx *ctx, MgLevel &M, size_t max_lds)
{
    Level &L = *M.L;
    hipStream_t s = ctx->stream;
    M.vstar.require((size_t)L.Nv1 * sizeof(T), "vstar");
    STMG_HIP(launch_midpoint<T>(state_of<T>(M), L.Nv1, L.nt, L.tc.phimid, M.vstar.as<T>(), s));
    const long long rw = elem_record_words(L.dim, L.r);
    M.elem.require((size_t)L.ncell * rw * sizeof(T), "elem");
    ElemArgs<T> ea{};
    ea.n0 = L.n[0];
    ea.n1 = L.n[1];
    ea.n2 = L.n[2];
    ea.Nn = L.Nn;
    ea.vstar = M.vstar.as<T>();
    ea.tab = std::is_same<T, double>::value ? (const T *)L.tab64.p : (const T *)L.tab32.p;
    ea.vert = L.mapped ? L.vert.as<double>() : nullptr;
    ea.mapped = L.mapped ? 1 : 0;
    ea.dmask = L.dmask;
    ea.nu = (T)L.nu;
    ea.g1 = (T)L.g1;
    ea.g2 = (T)L.g2;
    ea.out = M.elem.as<T>();
    ea.rec_words = rw;
    ea.bcells = L.bcells.as<int>();
    ea.nbcell = L.nbcell;
    {
        TimerScope ts(&ctx->timers, "vanka_elem", s);
        STMG_HIP(launch_elem<T>(L.dim, L.r, L.nq, ea, (int)L.ncell, s));
    }
    M.m = L.nt * (L.dim * L.nl + L.npm);
    M.ms = L.dim * L.nl + L.npm;
    if (ctx->mg->td) {
        // one spatial matrix per eigen-system of the time coupling
        M.tdg = time_diagonalization(L.tc);
        const long long ms = M.ms, ld = td_ld(M.ms), mat = ms * ld;   // rows padded to 32 elements
        long long off = 0;
        for (int sy = 0; sy < M.tdg.nsys; ++sy) {
            M.sys_off[sy] = off;
            M.piv_off[sy] = (long long)sy * L.ncell * ms;
            off += (long long)L.ncell * (M.tdg.cplx[sy] ? 2 : 1) * mat;
        }
        M.nfac = off;
        M.patches.require((size_t)off * sizeof(T), "patches");
        PatchTdArgs<T, T> pa{};
        pa.n0 = L.n[0];
        pa.n1 = L.n[1];
        pa.n2 = L.n[2];
        pa.elem = M.elem.as<T>();
        pa.rec_words = rw;
        pa.nsys = M.tdg.nsys;
        for (int sy = 0; sy < M.tdg.nsys; ++sy) {
            pa.cplx[sy] = M.tdg.cplx[sy];
            pa.lre[sy] = M.tdg.lre[sy];
            pa.lim[sy] = M.tdg.lim[sy];
            pa.sys[sy] = M.patches.as<T>() + M.sys_off[sy];
        }
        {
            TimerScope ts(&ctx->timers, "vanka_patch", s);
            STMG_HIP((launch_patch_td<T, T>(L.dim, L.r, pa, (int)L.ncell, s)));
        }
        STMG_HIP(hipMemsetAsync(M.info.p, 0, 4, s));
        if (ctx->mg->diag) {
            // diagonal Vanka: D^{-1} and the LU of the pressure Schur
            // complement per system; the systems stay unfactored
            const int nv = ctx->mg->diag_block ? L.nl * L.dim * L.dim : L.dim * L.nl, npm = L.npm, ns = M.tdg.nsys;
            M.dv_dinv.require((size_t)ns * L.ncell * 2 * nv * sizeof(T), "dv_dinv");
            M.dv_schur.require((size_t)ns * L.ncell * 2 * npm * npm * sizeof(T), "dv_schur");
            M.dv_piv.require((size_t)ns * L.ncell * npm * sizeof(int), "dv_piv");
            DvArgs<T> da{};
            da.nsys = ns;
            for (int sy = 0; sy < ns; ++sy) {
                da.cplx[sy] = M.tdg.cplx[sy];
                da.sys[sy] = M.patches.as<T>() + M.sys_off[sy];
                da.dinv[sy] = M.dv_dinv.as<T>() + (size_t)sy * L.ncell * 2 * nv;
                da.schur[sy] = M.dv_schur.as<T>() + (size_t)sy * L.ncell * 2 * npm * npm;
                da.spiv[sy] = M.dv_piv.as<int>() + (size_t)sy * L.ncell * npm;
            }
            da.info = M.info.as<int>();
            da.block = ctx->mg->diag_block ? 1 : 0;
            TimerScope ts(&ctx->timers, "vanka_lu", s);
            STMG_HIP(launch_dv_setup<T>(L.dim, L.r, da, (int)L.ncell, s));
            M.have_patches = true;
            return;
        }
        {
            TimerScope ts(&ctx->timers, "vanka_lu", s);
            for (int sy = 0; sy < M.tdg.nsys; ++sy)
                STMG_HIP(launch_lu_td<T>(M.patches.as<T>() + M.sys_off[sy], M.perm.as<int>() + M.piv_off[sy], M.ms, (int)ld,
                                         M.tdg.cplx[sy] != 0, (int)L.ncell, M.info.as<int>(), s));
            if constexpr (std::is_same<T, float>::value) {
                if (ctx->mg->factor_bf16) {
                    // the sweeps read a BF16 copy of the factors (half the bytes)
                    M.fac16.require((size_t)off * 2, "fac16");
                    STMG_HIP(launch_pack_bf16(M.patches.as<float>(), M.fac16.as<unsigned short>(), off, s));
                }
            }
        }
        M.have_patches = true;
        return;
    }
    M.patches.require((size_t)L.ncell * M.m * M.m * sizeof(T), "patches");
    M.piv.require((size_t)L.ncell * M.m * 4, "piv");
    PatchArgs<T, T> pa{};
    pa.cell0 = -1;
    pa.n0 = L.n[0];
    pa.n1 = L.n[1];
    pa.n2 = L.n[2];
    pa.nt = L.nt;
    pa.elem = M.elem.as<T>();
    pa.rec_words = rw;
    for (int i = 0; i < L.nt * L.nt; ++i) pa.K[i] = L.tc.K[i];
    for (int i = 0; i < L.nt; ++i) pa.w[i] = L.tc.w[i];
    pa.patches = M.patches.as<T>();
    {
        TimerScope ts(&ctx->timers, "vanka_patch", s);
        STMG_HIP((launch_patch<T, T>(L.dim, L.r, pa, (int)L.ncell, s)));
    }
    STMG_HIP(hipMemsetAsync(M.info.p, 0, 4, s));
    {
        TimerScope ts(&ctx->timers, "vanka_lu", s);
        STMG_HIP(launch_lu<T>(M.patches.as<T>(), M.piv.as<int>(), M.m, (int)L.ncell, M.info.as<int>(), max_lds, s));
    }
    M.have_patches = true;
}

void mg_rebuild(stmg_ctx *ctx)
{
    Mg &mg = *ctx->mg;
    mg.graph.reset(ctx->stream);
    TimerScope ts(&ctx->timers, "vanka_rebuild", ctx->stream);
    for (size_t l = 0; l + 1 < mg.lv.size(); ++l) {
        double t0 = verbose() ? now_s() : 0.0;
        if (mg.prec == STMG_F64) rebuild_level<double>(ctx, mg.lv[l], mg.max_lds);
        else rebuild_level<float>(ctx, mg.lv[l], mg.max_lds);
        if (verbose()) {
            STMG_HIP(hipStreamSynchronize(ctx->stream));
            std::fprintf(stderr, "[stmg] rebuild level %zu: %lld patches of %d, %.3f s\n", l, mg.lv[l].L->ncell,
                         mg.lv[l].m, now_s() - t0);
            std::fflush(stderr);
        }
    }
}

template <typename T> void mg_smooth(stmg_ctx *ctx, int l, const T *r, T *d, bool d_zero)
{
    Mg &mg = *ctx->mg;
    MgLevel &M = mg.lv[l];
    Level &L = *M.L;
    hipStream_t s = ctx->stream;
    T *t = M.t.as<T>();
    const T *defect = r;   // r - J d with d = 0
    if (!d_zero) {
        L.apply<T>(Mode::Jac, state_of<T>(M), d, t, nullptr, nullptr, 1, s);
        STMG_HIP(vec_axpby<T>(L.N, T(1), r, T(-1), t, s));
        defect = t;
    }
    TimerScope ts(&ctx->timers, "vanka_apply", s);
    bool applied = false;
    if (mg.td && mg.diag) {
        const int nv = mg.diag_block ? L.nl * L.dim * L.dim : L.dim * L.nl, npm = L.npm;   // stored D^{-1} entries
        DvArgs<T> da{};
        da.n0 = L.n[0];
        da.n1 = L.n[1];
        da.n2 = L.n[2];
        da.nt = L.nt;
        da.Nn = L.Nn;
        da.Nv1 = L.Nv1;
        da.Np1 = L.Np1;
        da.defect = defect;
        da.nsys = M.tdg.nsys;
        for (int sy = 0; sy < M.tdg.nsys; ++sy) {
            da.cplx[sy] = M.tdg.cplx[sy];
            da.sys[sy] = M.patches.as<T>() + M.sys_off[sy];
            da.dinv[sy] = M.dv_dinv.as<T>() + (size_t)sy * L.ncell * 2 * nv;
            da.schur[sy] = M.dv_schur.as<T>() + (size_t)sy * L.ncell * 2 * npm * npm;
            da.spiv[sy] = M.dv_piv.as<int>() + (size_t)sy * L.ncell * npm;
            for (int a = 0; a < L.nt; ++a) {
                da.Tre[sy * 4 + a] = (T)M.tdg.Tre[sy * MAX_NT + a];
                da.Tim[sy * 4 + a] = (T)M.tdg.Tim[sy * MAX_NT + a];
                da.Fre[a * 4 + sy] = (T)M.tdg.Fre[a * MAX_NT + sy];
                da.Fim[a * 4 + sy] = (T)M.tdg.Fim[a * MAX_NT + sy];
            }
        }
        da.E = M.E.as<T>();
        da.d = d;
        da.omega = (T)mg.omega;
        da.block = mg.diag_block ? 1 : 0;
        STMG_HIP(launch_solve_dv<T>(L.dim, L.r, da, (int)L.ncell, s));
        applied = true;
    }
    if constexpr (std::is_same<T, float>::value) {
        if (!applied && mg.td && mg.factor_bf16) {
            SolveTdArgs<float, float, unsigned short> sb{};
            sb.n0 = L.n[0];
            sb.n1 = L.n[1];
            sb.n2 = L.n[2];
            sb.nt = L.nt;
            sb.Nn = L.Nn;
            sb.Nv1 = L.Nv1;
            sb.Np1 = L.Np1;
            sb.defect = defect;
            sb.nsys = M.tdg.nsys;
            for (int sy = 0; sy < M.tdg.nsys; ++sy) {
                sb.cplx[sy] = M.tdg.cplx[sy];
                sb.sys[sy] = M.fac16.as<unsigned short>() + M.sys_off[sy];
                sb.perm[sy] = M.perm.as<int>() + M.piv_off[sy];
                for (int a = 0; a < L.nt; ++a) {
                    sb.Tre[sy * 4 + a] = (float)M.tdg.Tre[sy * MAX_NT + a];
                    sb.Tim[sy * 4 + a] = (float)M.tdg.Tim[sy * MAX_NT + a];
                    sb.Fre[a * 4 + sy] = (float)M.tdg.Fre[a * MAX_NT + sy];
                    sb.Fim[a * 4 + sy] = (float)M.tdg.Fim[a * MAX_NT + sy];
                }
            }
            sb.E = M.E.as<float>();
            sb.d = d;
            sb.omega = (float)mg.omega;
            STMG_HIP((launch_solve_td<float, float, unsigned short>(L.dim, L.r, sb, (int)L.ncell, s)));
            applied = true;
        }
    }
    if (applied) {
        // patch corrections already in M.E
    } else if (mg.td) {
        SolveTdArgs<T, T> sa{};
        sa.n0 = L.n[0];
        sa.n1 = L.n[1];
        sa.n2 = L.n[2];
        sa.nt = L.nt;
        sa.Nn = L.Nn;
        sa.Nv1 = L.Nv1;
        sa.Np1 = L.Np1;
        sa.defect = defect;
        sa.nsys = M.tdg.nsys;
        for (int sy = 0; sy < M.tdg.nsys; ++sy) {
            sa.cplx[sy] = M.tdg.cplx[sy];
            sa.sys[sy] = M.patches.as<T>() + M.sys_off[sy];
            sa.perm[sy] = M.perm.as<int>() + M.piv_off[sy];
            for (int a = 0; a < L.nt; ++a) {
                sa.Tre[sy * 4 + a] = (T)M.tdg.Tre[sy * MAX_NT + a];
                sa.Tim[sy * 4 + a] = (T)M.tdg.Tim[sy * MAX_NT + a];
                sa.Fre[a * 4 + sy] = (T)M.tdg.Fre[a * MAX_NT + sy];
                sa.Fim[a * 4 + sy] = (T)M.tdg.Fim[a * MAX_NT + sy];
            }
        }
        sa.E = M.E.as<T>();
        sa.d = d;
        sa.omega = (T)mg.omega;
        STMG_HIP((launch_solve_td<T, T, T>(L.dim, L.r, sa, (int)L.ncell, s)));
    } else {
        SolveArgs<T, T> sa{};
        sa.n0 = L.n[0];
        sa.n1 = L.n[1];
        sa.n2 = L.n[2];
        sa.nt = L.nt;
        sa.Nn = L.Nn;
        sa.Nv1 = L.Nv1;
        sa.Np1 = L.Np1;
        sa.defect = defect;
        sa.patches = M.patches.as<T>();
        sa.piv = M.piv.as<int>();
        sa.E = M.E.as<T>();
        sa.d = d;
        sa.omega = (T)mg.omega;
        STMG_HIP((launch_solve<T, T>(L.dim, L.r, sa, (int)L.ncell, M.m, s)));
    }
    GatherArgs<T> g = L.gather_args<T>();
    g.E = M.E.as<T>();
    g.rhs = nullptr;
    g.y = d;
    g.ystride = L.N;
    g.alpha = (T)mg.omega;
    g.accumulate = 1;
    g.inv_mult = mg.weighting;
    STMG_HIP(launch_gather<T>(g, 1, s));
}

template <typename T> void mg_vcycle(stmg_ctx *ctx, int l, const T *r, T *d)
{
    Mg &mg = *ctx->mg;
    const int nl = (int)mg.lv.size();
    hipStream_t s = ctx->stream;
    MgLevel &M = mg.lv[l];
    Level &L = *M.L;
    if (l == nl - 1) {
        TimerScope ts(&ctx->timers, "coarse_solve", s);
        if (mg.inverse) {
            STMG_HIP(launch_inverse_apply<T>(mg.dense_inverse(), r, d, mg.cn, s));
            return;
        }
        STMG_HIP((vec_cast<T, double>(L.N, r, mg.cr64.as<double>(), s)));
        STMG_HIP(launch_dense_solve(mg.cA.as<double>(), mg.cpiv.as<int>(), mg.cm, mg.cr64.as<double>(),
                                    mg.cx64.as<double>(), mg.cn, s));
        STMG_HIP((vec_cast<double, T>(L.N, mg.cx64.as<double>(), d, s)));
        return;
    }
    STMG_HIP(vec_fill<T>(L.N, T(0), d, s));
    for (int i = 0; i < mg.nu1; ++i) mg_smooth<T>(ctx, l, r, d, i == 0);
    T *t = M.t.as<T>();
    L.apply<T>(Mode::Jac, state_of<T>(M), d, t, nullptr, nullptr, 1, s);
    STMG_HIP(vec_axpby<T>(L.N, T(1), r, T(-1), t, s));
    MgLevel &C = mg.lv[l + 1];
    mg.tr[l]->restrict_<T>(L, *C.L, t, C.r.as<T>(), s);
    mg_vcycle<T>(ctx, l + 1, C.r.as<T>(), C.d.as<T>());
    mg.tr[l]->prolongate<T>(L, *C.L, C.d.as<T>(), d, T(1), s);
    for (int i = 0; i < mg.nu2; ++i) mg_smooth<T>(ctx, l, r, d);
}

template void mg_smooth<double>(stmg_ctx *, int, const double *, double *, bool);
template void mg_smooth<float>(stmg_ctx *, int, const float *, float *, bool);
template void mg_vcycle<double>(stmg_ctx *, int, const double *, double *);
template void mg_vcycle<float>(stmg_ctx *, int, const float *, float *);

static void precondition_eager(stmg_ctx *ctx, const double *v, double *z)
{
    Mg &mg = *ctx->mg;
    MgLevel &M = mg.lv[0];
    hipStream_t s = ctx->stream;
    if (mg.prec == STMG_F64) {
        mg_vcycle<double>(ctx, 0, v, z);
        return;
    }
    STMG_HIP((vec_cast<double, float>(M.L->N, v, M.r.as<float>(), s)));
    mg_vcycle<float>(ctx, 0, M.r.as<float>(), M.d.as<float>());
    STMG_HIP((vec_cast<float, double>(M.L->N, M.d.as<float>(), z, s)));
}

// capture the preconditioner application on the staging vectors; false if the
// runtime refuses (the caller then stays eager)
static bool capture_vcycle(stmg_ctx *ctx)
{
    Mg &mg = *ctx->mg;
    VcycleGraph &G = mg.graph;
    hipStream_t s = ctx->stream;
    const long long N = mg.lv[0].L->N;
    G.in.require((size_t)N * 8, "graph staging");
    G.out.require((size_t)N * 8, "graph staging");
    if (!G.warm) {
        // one eager cycle first: lazy allocations and kernel attributes happen
        // outside the capture
        STMG_HIP(vec_fill<double>(N, 0.0, G.in.as<double>(), s));
        precondition_eager(ctx, G.in.as<double>(), G.out.as<double>());
        G.warm = true;
    }
    if (!G.cs) STMG_HIP(hipStreamCreateWithFlags(&G.cs, hipStreamNonBlocking));
    std::lock_guard<std::recursive_mutex> lk(device_api_mutex());
    // record on the private stream: every launch below reads ctx->stream
    const bool timers_on = ctx->timers.on;
    ctx->timers.on = false;
    ctx->stream = G.cs;
    hipGraph_t g = nullptr;
    bool ok = hipStreamBeginCapture(G.cs, hipStreamCaptureModeRelaxed) == hipSuccess;
    if (ok) {
        try {
            precondition_eager(ctx, G.in.as<double>(), G.out.as<double>());
        } catch (const HipError &) {
            ok = false;
        }
        const hipError_t e = hipStreamEndCapture(G.cs, &g);
        ok = ok && e == hipSuccess && g != nullptr;
    }
    ctx->stream = s;
    ctx->timers.on = timers_on;
    if (ok) ok = hipGraphInstantiate(&G.x, g, nullptr, nullptr, 0) == hipSuccess;
    if (!ok) {
        if (g) (void)hipGraphDestroy(g);
        G.x = nullptr;
        (void)hipGetLastError();
        return false;
    }
    G.g = g;
    G.valid = true;
    return true;
}

void mg_precondition(stmg_ctx *ctx, const double *v, double *z)
{
    Mg &mg = *ctx->mg;
    VcycleGraph &G = mg.graph;
    hipStream_t s = ctx->stream;
    if (!mg.use_graph || G.failed) {
        precondition_eager(ctx, v, z);
        return;
    }
    if (!G.valid && !capture_vcycle(ctx)) {
        G.failed = true;
        precondition_eager(ctx, v, z);
        return;
    }
    const size_t bytes = (size_t)mg.lv[0].L->N * 8;
    STMG_HIP(hipMemcpyAsync(G.in.p, v, bytes, hipMemcpyDeviceToDevice, s));
    {
        TimerScope ts(&ctx->timers, "vcycle_graph", s);
        STMG_HIP(hipGraphLaunch(G.x, s));
    }
    STMG_HIP(hipMemcpyAsync(z, G.out.p, bytes, hipMemcpyDeviceToDevice, s));
}

} // namespace stmg
