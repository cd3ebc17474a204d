// ycol.hpp -- whole y-lines in one launch: the right-hand side's columns solved
// exactly and the update u^{n+1} = 2u^n - u^{n-1} + d written, with every column of a
// block of CB columns held in the registers of one workgroup.  Included by adiwave.hip
// after fusedr.hpp.
//
// The chunked y-solve (kernels.hpp) takes three launches and reads w and r twice; on
// grids of up to 2048 rows its launches are bound by their own latency (1501 x 997
// FP32: 4.2 + 4.8 + 6.2 us).  Here thread (column, p) holds rows [p S, p S + S): it
// eliminates them from the column's full-line entry pivot (k_ycol_pivots, built once
// per coefficient), which leaves the affine maps of the x-lines (xsweep.hpp),
//     g_out = G + Q g_in,   x_first = H + E g_in + Q x_below,
// and one wavefront per column scans the maps of its at most 64 segments (lane p =
// segment p; the maps pass through LDS).  u^n and u^{n-1} are requested before the
// scans where the registers allow it (PRE).  Lanes run along the columns first, so a
// wavefront reads CB neighbouring values of 64 / CB rows.
// Latency-bound on small grids, by bytes (w and r once: 20 B a node FP32) on wide ones.
// The exact step, x-sweep included, before (chunked) and after: 128^2 FP64 14.5 -> 9.1
// us, 1024^2 FP64 25.3 -> 20.1, 1024^2 FP32 17.9 -> 14.8, 1501 x 997 FP32 22 -> 17.6
// (this kernel 11 us), 8192 x 1024 FP32 66.6 -> 54.1.

namespace adw {

constexpr int kYcP = 64;          // segments per column (lanes of the scanning wavefront)

// (96 bytes for FP64: the hidden launch arguments behind it stay in the second 64-byte line)
template <typename T>
struct YColArgs {
    const T* w;          // x-sweep result
    const T* r;
    T* qy;               // entry pivot of every segment (DYN: written here)
    const T* u;          // update: out = alpha*u + beta*v + d
    const T* v;          // may be null when beta == 0
    T* out;
    T alpha, beta;
    int nx, ny;
    int rhs_times_r;     // right-hand side is r * w (adjoint solves)
    int nrec;            // DYN: receivers of the level written
    const int* rec_idx;
    T* rec_out;
};

template <typename T, int CB, bool DYN>
struct YColShared {
    union {
        T m[4][kYcP][CB + 1];                    // G (then g_in), Q, H (then x_below), E
        double v[DYN ? 3 : 1][kYcP][CB + 1];     // DYN: the pivot maps al (then al of the run so far), be, ga
    };
};
template <int CB>
struct YPivShared {
    double m[3][kYcP][CB + 1];       // al (then the entry pivot), be, ga
};

// pivot entering every S-row segment of every column: qy[p * nx + i]
template <typename T, int S, int CB>
__global__ void __launch_bounds__(kYcP * CB) k_ycol_pivots(const T* __restrict__ r, T* __restrict__ qy, int nx, int ny)
{
    __shared__ YPivShared<CB> sh;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), nw = blockDim.x >> 6;
    const int col = t % CB, p = t / CB, P = blockDim.x / CB;
    const int i = blockIdx.x * CB + col;
    // (all requested before the sweep)
    T rv[S];
#pragma unroll
    for (int k = 0; k < S; ++k) rv[k] = i < nx && p * S + k < ny ? r[(size_t)(p * S + k) * nx + i] : T(0);
    double q = 0.0, pi = 1.0, ga = 0.0;
#pragma unroll
    for (int k = 0; k < S; ++k) {
        (void)pivot_step<double>((double)rv[k], q);
        const double x = pi * q;
        ga = fma_rn(pi, x, ga);
        pi = x;
    }
    sh.m[0][p][col] = q;
    sh.m[1][p][col] = pi * pi;
    sh.m[2][p][col] = ga;
    __syncthreads();
    for (int c = wv; c < CB; c += nw) {
        PivotMap<double> m{0.0, 1.0, 0.0};
        if (lane < P) m = {sh.m[0][lane][c], sh.m[1][lane][c], sh.m[2][lane][c]};
        m = pivot_scan(m, lane);
        if (lane + 1 < P) sh.m[0][lane + 1][c] = m.al;   // al: the run's last pivot from 0
        if (lane == 0) sh.m[0][0][c] = 0.0;
    }
    __syncthreads();
    if (i < nx && p * S < ny) qy[(size_t)p * nx + i] = (T)sh.m[0][p][col];
}

// DYN: r is new (the time-dependent step): the entry pivots are formed here and kept in
// A.qy, and the receivers of the new level are recorded.
template <typename T, int S, int CB, bool DYN = false>
__global__ void __launch_bounds__(kYcP * CB) k_ycol(YColArgs<T> A)
{
    constexpr int ES = (int)sizeof(T);
    constexpr bool PRE = S * ES <= 64;
    __shared__ YColShared<T, CB, DYN> sh;
    const int blk = xcd_band(blockIdx.x);                 // neighbouring columns on one XCD
    if (blk * CB >= A.nx) return;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), nw = blockDim.x >> 6;
    const int col = t % CB, p = t / CB, P = blockDim.x / CB;
    const int nx = A.nx, ny = A.ny;
    const int i = blk * CB + col;
    const int plane = nx * ny * ES;                       // at most kFuOOB bytes
    const int rowb = nx * ES;
    const rsrc_t rw = buf(A.w, plane), rr = buf(A.r, plane);
    const rsrc_t ru = buf(A.u, A.u ? plane : 0), rv = buf(A.v, A.v ? plane : 0);
    // rows past the grid lie past the plane's end, columns past it start there: both read 0
    const int off = i < nx ? (p * S * nx + i) * ES : kFuOOB;
    T g[S], q[S];
#pragma unroll
    for (int k = 0; k < S; ++k) {
        q[k] = fr_load1<T, 0>(rr, off + k * rowb, 0);
        g[k] = fr_load1<T, 0>(rw, off + k * rowb, 0);
    }
    const rsrc_t rq = buf(A.qy, (ny + S - 1) / S * rowb);
    const int qoff = i < nx ? (p * nx + i) * ES : kFuOOB;
    T qq = T(0);
    if constexpr (!DYN) qq = fr_load1<T, 0>(rq, qoff, 0);
    T uu[PRE ? S : 1], vv[PRE ? S : 1];
    if constexpr (PRE) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
            uu[k] = fr_load1<T, 0>(ru, off + k * rowb, 0);
            vv[k] = fr_load1<T, 0>(rv, off + k * rowb, 0);
        }
    }
    if constexpr (DYN) {
        const PivotMap<double> own = pivot_map<double>(q);  // (in FP64: the pivots of k_ycol_pivots)
        sh.v[0][p][col] = own.al;
        sh.v[1][p][col] = own.be;
        sh.v[2][p][col] = own.ga;
        __syncthreads();
        for (int c = wv; c < CB; c += nw) {
            PivotMap<double> m{0.0, 1.0, 0.0};
            if (lane < P) m = {sh.v[0][lane][c], sh.v[1][lane][c], sh.v[2][lane][c]};
            m = pivot_scan(m, lane);
            if (lane < P) sh.v[0][lane][c] = m.al;          // the run's last pivot from 0
        }
        __syncthreads();
        if (p > 0) qq = (T)sh.v[0][p - 1][col];
        fr_store1<T, 0>(qq, rq, qoff, 0);
        __syncthreads();                                    // the maps' place is written again
    }
    const bool sc = A.rhs_times_r != 0;
    {
        T Gv = T(0), Qv = T(1), h = T(0), ee = T(0);
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const T rk = q[k];
            const T rhs = sc ? rk * g[k] : g[k];
            const T m = pivot_step<T>(rk, qq);
            const T Pv = Qv;
            Gv = fma_rn(m, rhs, qq * Gv);
            Qv = qq * Qv;
            h = fma_rn(Pv, Gv, h);
            ee = fma_rn(Pv, Qv, ee);
            g[k] = Gv;
            q[k] = qq;
        }
        sh.m[0][p][col] = Gv;
        sh.m[1][p][col] = Qv;
        sh.m[2][p][col] = h;
        sh.m[3][p][col] = ee;
    }
    __syncthreads();
    for (int c = wv; c < CB; c += nw) {
        T a = T(0), b = T(1), h = T(0), ee = T(0);
        if (lane < P) { a = sh.m[0][lane][c]; b = sh.m[1][lane][c]; h = sh.m[2][lane][c]; ee = sh.m[3][lane][c]; }
        T bb = b;
        wave_scan_fwd(a, b);
        const T gin = dpp<kWaveShr1>(T(0), a);
        T ba = fma_rn(ee, gin, h);
        fr_scan_bwd2<T>(ba, bb, lane);
        const T xb = dpp<kWaveShl1>(T(0), ba);
        if (lane < P) { sh.m[0][lane][c] = gin; sh.m[2][lane][c] = xb; }
    }
    __syncthreads();
    const T gin = sh.m[0][p][col];
    T x = sh.m[2][p][col];
    {
        T Qv = T(1);
#pragma unroll
        for (int k = 0; k < S; ++k) {
            Qv = q[k] * Qv;
            g[k] = fma_rn(Qv, gin, g[k]);
        }
    }
    const rsrc_t ro = buf(A.out, plane);
    constexpr int GR = PRE ? S : ES == 4 ? 4 : 8;                       // rows requested together
#pragma unroll
    for (int k1 = S - 1; k1 >= 0; k1 -= GR) {
        if constexpr (!PRE) {
            T un[GR], vn[GR];
#pragma unroll
            for (int k = 0; k < GR; ++k) {
                un[k] = fr_load1<T, 0>(ru, off + (k1 - k) * rowb, 0);
                vn[k] = fr_load1<T, 0>(rv, off + (k1 - k) * rowb, 0);
            }
#pragma unroll
            for (int k = 0; k < GR; ++k) {
                x = fma_rn(q[k1 - k], x, g[k1 - k]);
                fr_store1<T, 0>(fma_rn(A.beta, vn[k], A.alpha * un[k]) + x, ro, off + (k1 - k) * rowb, 0);
            }
        } else {
#pragma unroll
            for (int k = S - 1; k >= 0; --k) {
                x = fma_rn(q[k], x, g[k]);
                fr_store1<T, 0>(fma_rn(A.beta, vv[k], A.alpha * uu[k]) + x, ro, off + k * rowb, 0);
            }
        }
    }
    if constexpr (DYN) {
        if (A.nrec > 0) {
            __syncthreads();                                // the block's columns are written
            for (int k = t; k < A.nrec; k += blockDim.x) {
                const int id = A.rec_idx[k];
                const bool in = id >= 0 && id < nx * ny;
                const int c = in ? id % nx - blk * CB : -1;
                if (c >= 0 && c < CB) A.rec_out[k] = A.out[id];
                else if (!in && blk == 0) A.rec_out[k] = T(NAN);
            }
        }
    }
}

}  // namespace adw
