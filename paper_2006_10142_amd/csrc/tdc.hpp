// tdc.hpp -- one step of eq. (CN1) with a coefficient that changes in time:
// c^{n+1} multiplies the Laplacian of u^{n+1}, c^{n-1} that of u^{n-1}.  With
// delta = u^{n+1} - 2u^n + u^{n-1}, beta = dt^2/2 and r = beta kappa / h^2,
//     (I - beta K^{n+1} Lap) delta = dt^2 f + 2 r^{n+1} S(u^n) + (r^{n-1} - r^{n+1}) S(u^{n-1}),
// S(v) = v_W + v_E + v_S + v_N - 4 v_C, and the ADI step factors the operator as
// (I - beta K^{n+1} Lxx)(I - beta K^{n+1} Lyy): the x-lines, then the y-lines and
// the update, with exact line solves on the coefficient r^{n+1}.  For a coefficient
// constant in time it is the plain step.  Two launches where a row fits 256 threads and
// a column one workgroup (k_tdc_x and the whole-column y-solve: 1024^2 FP32 23 us a
// step, 203 by the separate kernels), else the separate kernels.  Included at the end of
// adiwave.hip.

namespace adw {

// rho = 2 rn S(uc) + (rp - rn) S(up)
template <typename T>
__global__ void __launch_bounds__(256) k_rhs_tdc(const T* __restrict__ uc, const T* __restrict__ up,
                                                 const T* __restrict__ rn, const T* __restrict__ rp,
                                                 T* __restrict__ rho, int nx, int ny)
{
    const long long n = (long long)nx * ny;
    for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) {
        const int j = (int)(p / nx), i = (int)(p - (long long)j * nx);
        auto S = [&](const T* u) {
            const T w_ = i > 0 ? u[p - 1] : T(0), e_ = i < nx - 1 ? u[p + 1] : T(0);
            const T s_ = j > 0 ? u[p - nx] : T(0), n_ = j < ny - 1 ? u[p + nx] : T(0);
            return ((w_ + e_) + (s_ + n_)) - T(4) * u[p];
        };
        const T r1 = rn[p];
        rho[p] = fma_rn(rp[p] - r1, S(up), T(2) * r1 * S(uc));
    }
}

// The x-lines of a time-dependent step in one launch (line groups of up to 256 threads):
// r^{n+1} = sn * kn and r^{n-1} = sp * kp formed where they are used, the right-hand side
// above with the point sources, the row's entry pivots from r^{n+1} (one scan of pivot
// maps, xsweep.hpp), and the line solve.  r^{n+1} and the entry pivots are written as the
// handle's (rout NULL: the coefficient is unchanged).  The maps are formed and composed in
// FP64, as in k_xpivots: composed in FP32 the step at 1024^2 takes 22.2 us instead of 23.2,
// but at r = 2 the pivots are further from 64 bits than a sequential FP32 sweep's (rms
// 5.7e-8 on 4-node segments and 5.52e-8 on 8, against 5.5e-8 and 5.47e-8; in FP64 4.9e-8
// and 5.2e-8).  Bound by latency at 1024^2; as launches of their own the same work took
// 27 us a step there.
template <typename T>
struct TdcArgs {
    XArgs<T> x;          // u = u^n, qin and w written; sources
    const T* up;         // u^{n-1}
    const T* kn;
    const T* kp;
    T sn, sp;
    T* rout;
    T* qout;
};

template <typename T, int TR>
struct TdcShared {
    XShared<T, TR, false> x;
    PivotMap<double> tot[2][TR / 64];
};

template <typename T, int TR>
__global__ void __launch_bounds__(256) k_tdc_x(TdcArgs<T> B)
{
    constexpr int E = kSeg, G = 256 / TR;
    constexpr int ES = (int)sizeof(T);
    __shared__ TdcShared<T, TR> shg[G];
    const XArgs<T>& A = B.x;
    const int blk = A.xcd() ? xcd_band(blockIdx.x) : (int)blockIdx.x;
    const int RS = A.rows_per_strip, nx = A.nx, ny = A.ny, nseg = A.nseg();
    if (blk * G * RS >= ny) return;
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x / TR);
    const int t = threadIdx.x - g * TR, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    TdcShared<T, TR>& sh = shg[g];
    const int j0 = (blk * G + g) * RS;
    const int i0 = E * t;
    const bool act = t < nseg;
    const int L = act ? min(E, nx - i0) : 0;
    const int voff = i0 * ES, row_bytes = nx * ES;
    auto row_of = [&](const T* base, int j) {
        const bool in = j >= 0 && j < ny;
        return buf(base + (size_t)(in ? j : 0) * nx, in ? row_bytes : 0);
    };
    // S(v) of row j's nodes
    auto stencil = [&](const T* v, int j, T (&s)[E]) {
        T c[E], n[E], o[E];
        const rsrc_t rc = row_of(v, j);
        bload8<T>(rc, voff, c);
        bload8<T>(row_of(v, j - 1), voff, o);
        bload8<T>(row_of(v, j + 1), voff, n);
        const T w = bload1<T>(rc, voff - ES);     // before the row's start the offset wraps past its end
        const T e = bload1<T>(rc, voff + E * ES);
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const T vw = k == 0 ? w : c[k - 1], ve = k == E - 1 ? e : c[k + 1];
            s[k] = ((vw + ve) + (o[k] + n[k])) - T(4) * c[k];
        }
    };
    for (int it = 0; it < RS; ++it) {
        const int j = j0 + it;
        const bool live = j < ny;
        T rc[E], rp[E], su[E], sp[E];
        bload8<T>(row_of(B.kn, live ? j : -1), voff, rc);
        bload8<T>(row_of(B.kp, live ? j : -1), voff, rp);
        stencil(A.u, live ? j : -2, su);
        stencil(B.up, live ? j : -2, sp);
        T rho[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            rc[e] = B.sn * rc[e];
            rho[e] = fma_rn(B.sp * rp[e] - rc[e], sp[e], T(2) * rc[e] * su[e]);
        }
        if (it == 0) stage_sources<T, TR, false>(A, j0, RS, t, sh.x);   // (seen after entry_pivot's barrier)
        PivotMap<double> m{0.0, 1.0, 0.0};
        if (act) m = pivot_map<double>(rc);
        const T q = (T)entry_pivot(m, sh.tot[it & 1], lane, wv);
        const int ns = sh.x.src_n;
        for (int k = 0; live && k < (ns >= 0 ? ns : A.nsrc); ++k) {
            int i = -1;
            T add = T(0);
            if (ns >= 0) {
                if ((sh.x.src_pos[k] >> 16) == it) { i = (sh.x.src_pos[k] & 0xffff) - i0; add = sh.x.src_add[k]; }
            } else {
                const int id = A.src_idx[k];
                if (id >= 0 && id / nx == j) { i = id - j * nx - i0; add = A.tau2 * A.src_amp[k]; }
            }
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e == i) rho[e] += add;
        }
        T wout[E];
        xline_row<T, TR>(rho, rc, q, L, act, lane, wv, it & 1, sh.x.totf, sh.x.totb, []() {}, wout);
        bstore8<T>(row_of(A.w, live ? j : -1), voff, wout);
        if (B.rout) {
            bstore8<T>(row_of(B.rout, live ? j : -1), voff, rc);
            if (live && act) B.qout[(size_t)j * nseg + t] = q;
        }
    }
}

}  // namespace adw

namespace {

template <typename T>
void launch_tdc_x(int tr, int grid, const TdcArgs<T>& a, hipStream_t st)
{
    switch (tr) {
        case 64: hipLaunchKernelGGL((k_tdc_x<T, 64>), dim3(grid), dim3(256), 0, st, a); break;
        case 128: hipLaunchKernelGGL((k_tdc_x<T, 128>), dim3(grid), dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL((k_tdc_x<T, 256>), dim3(grid), dim3(256), 0, st, a); break;
    }
}

// Rows of up to 2048 nodes and columns that the whole-column y-solve takes: one launch
// for the x-lines (k_tdc_x), one for the y-lines with their pivots and the receivers.
template <typename T>
adi_status step_tdc_rows(adi_wave_s* w, void** u_prev, void** u_curr, const void* kappa_prev, const void* kappa_next,
                         const adi_source* f, const adi_receivers* rec)
{
    const double s = w->dt * w->dt / (2.0 * w->h * w->h);
    if (kappa_next) {
        ++w->gen;
        adjoint_invalidate(w);
        coef_unmeasured(w);      // the one-pass step stays off until the next set_kappa
    }
    TdcArgs<T> a{};
    a.x = make_x<T>(w, *u_curr, f, 0, T(1));
    a.x.rows_per_strip = w->xp.rs;
    a.up = static_cast<const T*>(*u_prev);
    a.kn = static_cast<const T*>(kappa_next ? kappa_next : w->r);
    a.sn = kappa_next ? (T)s : T(1);
    a.kp = static_cast<const T*>(kappa_prev ? kappa_prev : w->r);
    a.sp = kappa_prev ? (T)s : T(1);
    a.rout = kappa_next ? static_cast<T*>(w->r) : nullptr;
    a.qout = static_cast<T*>(w->qin);
    launch_tdc_x<T>(w->xp.tr, xsweep_grid(w->ny, w->xp.rs, x_groups_per_wg(w->xp.tr)), a, w->stream);
    ADI_LAUNCHED("x_sweep (time-dependent coefficient)");
    YColArgs<T> ya = make_ycol<T>(w, make_y<T>(w, *u_curr, *u_prev, *u_prev, T(2), T(-1)));
    if (rec && rec->count > 0) {
        ya.nrec = rec->count;
        ya.rec_idx = rec->idx;
        ya.rec_out = static_cast<T*>(rec->traces);
    }
    if (!launch_ycol<T, true>(w->yct, ya, w->stream)) return fail(ADI_EUNSUPPORTED, "no column kernel for this plan");
    ADI_LAUNCHED("y_solve_update");
    if (kappa_next && !w->ycs)           // the exact step's y-lines are chunked: their planes of the new r
        if (adi_status e = static_planes<T>(w)) return e;
    std::swap(*u_prev, *u_curr);
    return ADI_OK;
}

template <typename T>
adi_status do_step_tdc(adi_wave_s* w, void** u_prev, void** u_curr, const void* kappa_prev,
                       const void* kappa_next, const adi_source* f, const adi_receivers* rec)
{
    // (line groups of 1024 threads have no registers for the two stencils; columns too
    // long for one workgroup need the chunked y-solve's planes of the new coefficient)
    if (w->xp.tr <= 256 && w->yct) return step_tdc_rows<T>(w, u_prev, u_curr, kappa_prev, kappa_next, f, rec);
    const long long n = (long long)w->nx * w->ny;
    const size_t bytes = (size_t)n * sizeof(T);
    if (!w->r_prev || !w->rho_buf) {
        if (!w->r_prev && hipMalloc(&w->r_prev, bytes) != hipSuccess) {
            (void)hipGetLastError();
            w->r_prev = nullptr;
            return fail(ADI_ENOMEM, "hipMalloc of the previous coefficient failed");
        }
        if (!w->rho_buf && hipMalloc(&w->rho_buf, bytes) != hipSuccess) {
            (void)hipGetLastError();
            w->rho_buf = nullptr;
            return fail(ADI_ENOMEM, "hipMalloc of the right-hand side failed");
        }
        w->bytes += 2 * bytes;
    }
    const double s = w->dt * w->dt / (2.0 * w->h * w->h);
    // r^{n-1}: from kappa_prev, or the handle's current coefficient
    if (kappa_prev) {
        hipLaunchKernelGGL((k_coef<T>), dim3(cr_grid(n)), dim3(256), 0, w->stream, static_cast<const T*>(kappa_prev),
                           T(0), 0, (T)s, static_cast<T*>(w->r_prev), n);
        ADI_LAUNCHED("coef (previous level)");
    } else {
        ADI_HIP(hipMemcpyAsync(w->r_prev, w->r, bytes, hipMemcpyDeviceToDevice, w->stream));
    }
    // r^{n+1} with its x-line pivots and y-chunk planes becomes the handle's coefficient
    if (kappa_next) {
        if (adi_status st = set_coef<T>(w, kappa_next, 0.0, 0, false)) return st;
        coef_unmeasured(w);      // the one-pass step stays off until the next set_kappa
    }
    hipLaunchKernelGGL((k_rhs_tdc<T>), dim3(cr_grid(n)), dim3(256), 0, w->stream, static_cast<const T*>(*u_curr),
                       static_cast<const T*>(*u_prev), static_cast<const T*>(w->r),
                       static_cast<const T*>(w->r_prev), static_cast<T*>(w->rho_buf), w->nx, w->ny);
    ADI_LAUNCHED("rhs (time-dependent coefficient)");
    if (f && f->count > 0) {
        hipLaunchKernelGGL((k_cr_sources<T>), dim3(1), dim3(64), 0, w->stream, static_cast<T*>(w->rho_buf), f->idx,
                           static_cast<const T*>(f->amp), f->count, (T)(w->dt * w->dt), n);
        ADI_LAUNCHED("sources");
    }
    if (adi_status st = queue_xsolve<T>(w, w->rho_buf, w->w)) return st;
    if (adi_status st = queue_y<T>(w, make_y<T>(w, *u_curr, *u_prev, *u_prev, T(2), T(-1)), false, nullptr)) return st;
    if (rec && rec->count > 0) {
        hipLaunchKernelGGL((k_record<T>), dim3((rec->count + 255) / 256), dim3(256), 0, w->stream,
                           static_cast<const T*>(*u_prev), rec->idx, static_cast<T*>(rec->traces), rec->count, n);
        ADI_LAUNCHED("record");
    }
    std::swap(*u_prev, *u_curr);
    return ADI_OK;
}

}  // namespace

extern "C" {

adi_status adi_wave_step_tdc(adi_wave_t w, void** u_prev, void** u_curr, const void* kappa_prev,
                             const void* kappa_next, const adi_source* f, const adi_receivers* rec)
{
    if (adi_status s = check_handle(w)) return s;
    if (!u_prev || !u_curr || !*u_prev || !*u_curr) return fail(ADI_EINVAL, "null level pointer");
    if (*u_prev == *u_curr) return fail(ADI_EINVAL, "u_prev and u_curr must be distinct buffers");
    if (adi_status s = check_src(f)) return s;
    if (adi_status s = check_rec(rec)) return s;
    return w->dtype == ADI_F32 ? do_step_tdc<float>(w, u_prev, u_curr, kappa_prev, kappa_next, f, rec)
                               : do_step_tdc<double>(w, u_prev, u_curr, kappa_prev, kappa_next, f, rec);
}

}  // extern "C"
