// adjrev.hpp -- one reverse step of the FP32 adjoint in one launch, on tiles: the
// transposed y-lines z = A_y^{-1} (r lambda^{k+1}), the transposed x-lines t = A_x^{-1} z
// and the update of dJ/dkappa and lambda (the expressions of k_adjoint_update), for
// handles that take the one-pass step.  Included by adjoint.hpp.
//
// Both line solves run on windows, cut as the one-pass step's (fused.hpp): every z used
// is 9 rows or more and every t used 9 columns or more from a cut, so they differ from
// the full-line solves by at most 2 qs^9 max|z| and 2 qs^9 max|t|, which the one-pass
// bound keeps below half an ulp.
//
// A tile is Wt output columns (a multiple of 8, at most kArWmax) by kArHt = 22 output
// rows; LDS holds 40 rows of the column window [c0 - 16, c0 + Wt + 16).
//   load     r lambda^{k+1} and r of the rows [r0 - 9, r0 + 31), 16 bytes a lane.
//   y-lines  two windows of 28 rows a column, one thread each, in registers; their 12
//            central rows, together the 24 rows [r0 - 1, r0 + 23), replace r lambda.
//   x-lines  two rows per wavefront, four nodes a lane, from the full-line entry pivots
//            (fused4.hpp's scheme); z and r stay in registers, t goes to LDS.
//   update   the wavefront's own rows: t of the rows above and below from LDS, the
//            x-neighbours from the neighbouring lanes, and u^{k-1}, u^k, u^{k+1} of four
//            rows, requested before the x-lines.
// Bound by latency on grids of about a tile per compute unit: 11.7 us at 1024^2 (42 MB,
// 6.8 us at the copy kernel's rate), against 8.7 + 14.4 us for the two launches before
// (y-lines on windows of 48 rows; x-lines of whole rows with the update, whose two halo
// rows a row were solved again).

namespace adw {

constexpr int kArHb = 12;                       // z rows of a y-window
constexpr int kArNb = kArHb + 2 * kFuKy;        // rows of a y-window (28)
constexpr int kArNr = 2 * kArHb;                // x-rows of a tile (24)
constexpr int kArHt = kArNr - 2;                // output rows of a tile (22)
constexpr int kArRows = kArNr + 2 * kFuKy;      // rows in LDS (40)
constexpr int kArKx = 2 * kFuKx;                // window columns beyond the tile (9 needed, whole segments)
constexpr int kArWmax = 64 * kF4Seg - 2 * kArKx;   // widest tile (224)
constexpr int kArWaves = kArNr / 2;             // wavefronts: two x-rows each (12)
static_assert(64 * kArWaves >= 2 * (kArWmax + 2 * kArKx), "a thread for each y-window");

struct ARShared {
    alignas(16) float z[kArRows * 64 * kF4Seg];   // r lambda, then z, then t
    alignas(16) float r[kArRows * 64 * kF4Seg];
    int src_pos[kStripSrc];   // sources of the output tile: x-row * 2^16 + window column
    int src_k[kStripSrc];     //   and the source's index
    int src_n;                // -1: more than kStripSrc
};

__global__ void __launch_bounds__(64 * kArWaves) k_adjoint_step(AdjArgs<float> A, const float* __restrict__ qin, int nseg,
                                                              int wt, int tiles_x, int tiles)
{
    constexpr int E = kF4Seg;
    __shared__ ARShared sh;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nx = A.nx, ny = A.ny;
    if (A.gout && blockIdx.x == 0)               // sources outside the grid: zero gradient
        for (int k = t; k < A.nsrc; k += blockDim.x)
            if (A.sidx[k] < 0 || A.sidx[k] >= A.npts) A.gout[k] = 0.f;
    const int tile = xcd_band(blockIdx.x);
    if (tile >= tiles) return;
    const int c0 = (tile % tiles_x) * wt, r0 = (tile / tiles_x) * kArHt;
    const int nl = (wt + 2 * kArKx) / E;         // lanes of the window
    const int ws = nl * E;
    const int row_bytes = nx * 4;
    const bool inwin = lane < nl;
    const int col0 = c0 - kArKx + lane * E;      // columns off the grid: offsets past every range
    const int voff = inwin && col0 >= 0 ? col0 * 4 : kFuOOB;
    auto rows = [&](const float* base, int j) {
        const bool ok = j >= 0 && j < ny;
        return buf(base + (size_t)(ok ? j : 0) * nx, ok ? row_bytes : 0);
    };
    // the lanes of the output columns, and their byte offset in a row
    const bool outl = lane >= kArKx / E && lane < nl - kArKx / E && col0 < nx;
    const int ooff = outl ? voff : kFuOOB;
    auto load4at = [&](rsrc_t rs, int off, float (&v)[E]) {
        const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    };
    auto load4 = [&](rsrc_t rs, float (&v)[E]) { load4at(rs, voff, v); };
    auto load4o = [&](rsrc_t rs, float (&v)[E]) { load4at(rs, ooff, v); };

    // ------------------------------------------------------------------ load
#pragma unroll
    for (int k = 0; k < (kArRows + kArWaves - 1) / kArWaves; ++k) {
        const int lr = wv + k * kArWaves;
        if (lr < kArRows) {
            const int j = r0 - 1 - kFuKy + lr;
            float l[E], r[E];
            load4(rows(A.lam1, j), l);
            load4(rows(A.r, j), r);
            if (inwin) {
                const int o4 = lr * nl + lane;
                reinterpret_cast<float4*>(sh.z)[o4] = make_float4(r[0] * l[0], r[1] * l[1], r[2] * l[2], r[3] * l[3]);
                reinterpret_cast<float4*>(sh.r)[o4] = make_float4(r[0], r[1], r[2], r[3]);
            }
        }
    }
    if (t < 64) {                                // sources of the output tile, in source order
        int n = 0;
        for (int base = 0; base < A.nsrc; base += 64) {
            const int k = base + t;
            const int id = (A.sidx && k < A.nsrc) ? A.sidx[k] : -1;
            const int row = (id >= 0 && id < A.npts) ? id / nx : -1;
            const int col = row >= 0 ? id - row * nx : 0;
            const bool hit = row >= r0 && row < r0 + kArHt && col >= c0 && col < c0 + wt;
            const unsigned long long mask = __ballot(hit);
            const int before = __popcll(mask & ((1ull << t) - 1ull));
            if (hit && n + before < kStripSrc) {
                sh.src_pos[n + before] = ((row - r0 + 1) << 16) | (col - (c0 - kArKx));
                sh.src_k[n + before] = k;
            }
            n += __popcll(mask);
        }
        if (t == 0) sh.src_n = n <= kStripSrc ? n : -1;
    }
    __syncthreads();

    // --------------------------------------------------------------- y-lines
    {
        const bool ythr = t < 2 * ws;
        const int win = ythr ? t / ws : 0;
        const int ci = ythr ? t - win * ws : 0;
        float gk[kArNb], qk[kArNb];
        if (ythr) {
            float q = 0.f, g = 0.f;
            int o = win * kArHb * ws + ci;
#pragma unroll
            for (int k = 0; k < kArNb; ++k, o += ws) {
                const float m = pivot_step<float>(sh.r[o], q);
                g = fma_rn(m, sh.z[o], q * g);
                gk[k] = g;
                qk[k] = q;
            }
        }
        __syncthreads();
        if (ythr) {
            float d = 0.f;
            float* zc = sh.z + win * kArHb * ws + ci;
#pragma unroll
            for (int k = kArNb - 1; k >= kFuKy; --k) {
                d = fma_rn(qk[k], d, gk[k]);
                if (k < kFuKy + kArHb) zc[k * ws] = d;
            }
        }
    }

    // the update's levels, rows j0 - 1 .. j0 + 2 of u^{k-1}, u^k, u^{k+1}; the rows' entry
    // pivots, lambda^{k+1}, lambda^{k+2} and gradient
    const int j0 = r0 - 1 + 2 * wv;              // this wavefront's rows j0, j0 + 1 (x-rows 2 wv, 2 wv + 1)
    float un[4][E], dn[4][E], l1[2][E], l2[2][E], gr[2][E], qe0[2];
    {
        float um[4][E], up[4][E];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            load4(rows(A.uk, j0 - 1 + k), un[k]);
            load4(rows(A.up, j0 - 1 + k), up[k]);
            load4(rows(A.um, j0 - 1 + k), um[k]);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int j = j0 + k;
            const bool ok = j >= 0 && j < ny;
            const int seg = col0 >= 0 ? col0 / kSeg : -1;
            qe0[k] = bload1<float>(buf(qin + (size_t)(ok ? j : 0) * nseg, ok ? nseg * 4 : 0),
                                   inwin && seg >= 0 ? seg * 4 : kFuOOB);
            load4o(rows(A.lam1, j), l1[k]);
            load4o(rows(A.lam2, j), l2[k]);
            load4o(rows(A.grad, j), gr[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < E; ++e) dn[k][e] = (up[k][e] - 2.f * un[k][e]) + um[k][e];
    }
    __syncthreads();

    // --------------------------------------------------------------- x-lines
    float zr[2][E], rr[2][E], tr[2][E];
    const int lr0 = kFuKy + 2 * wv;
    {
        float Ge[2][E], qe[2][E], Qe[2][E];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int o4 = (lr0 + k) * nl + (inwin ? lane : 0);
            const float4 zv = reinterpret_cast<const float4*>(sh.z)[o4];
            const float4 rv = reinterpret_cast<const float4*>(sh.r)[o4];
            zr[k][0] = zv.x; zr[k][1] = zv.y; zr[k][2] = zv.z; zr[k][3] = zv.w;
            rr[k][0] = rv.x; rr[k][1] = rv.y; rr[k][2] = rv.z; rr[k][3] = rv.w;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (!inwin) { zr[k][e] = 0.f; rr[k][e] = 0.f; }
            // odd lanes carry their segment's entry pivot over the even lane before them
            float q = qe0[k], qo = q;
#pragma unroll
            for (int e = 0; e < E; ++e) (void)pivot_step<float>(dpp<kRowShr + 1>(0.f, rr[k][e]), qo);
            if (lane & 1) q = qo;
            float Gv = 0.f, Qv = 1.f;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float m = pivot_step<float>(rr[k][e], q);
                Gv = fma_rn(m, zr[k][e], q * Gv);
                Qv = q * Qv;
                Ge[k][e] = Gv;
                qe[k][e] = q;
                Qe[k][e] = Qv;
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float gin = enter_left<16 / E>(Ge[k][E - 1], Qe[k][E - 1]);
            float first = 0.f;                   // the lane's first value with nothing from below
#pragma unroll
            for (int e = E - 1; e >= 0; --e) {
                Ge[k][e] = fma_rn(Qe[k][e], gin, Ge[k][e]);
                first = fma_rn(qe[k][e], first, Ge[k][e]);
            }
            float x = enter_right<16 / E>(inwin ? first : 0.f, Qe[k][E - 1]);
#pragma unroll
            for (int e = E - 1; e >= 0; --e) {
                x = fma_rn(qe[k][e], x, Ge[k][e]);
                tr[k][e] = x;
            }
            if (inwin)
                reinterpret_cast<float4*>(sh.z)[(lr0 + k) * nl + lane] = make_float4(tr[k][0], tr[k][1], tr[k][2], tr[k][3]);
        }
    }
    __syncthreads();

    // ---------------------------------------------------------------- update
    const int ns = sh.src_n;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int xr = 2 * wv + k, j = j0 + k;
        const bool out = xr >= 1 && xr <= kArHt && j < ny;      // uniform over the wavefront
        float tm[E], tp[E];
        {
            // t of the row above and below: the wavefront's own other row, or LDS
            const int ol = k == 0 ? lr0 - 1 : lr0 + 2;
            const float4 v = reinterpret_cast<const float4*>(sh.z)[ol * nl + (inwin ? lane : 0)];
            const float o[E] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < E; ++e) {
                tm[e] = k == 0 ? o[e] : tr[0][e];
                tp[e] = k == 0 ? tr[1][e] : o[e];
            }
        }
        float syd[E], wq[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            syd[e] = (dn[k][e] + dn[k + 2][e]) - 2.f * dn[k + 1][e];
            wq[e] = dn[k + 1][e] - rr[k][e] * syd[e];
        }
        const float twl = dpp<kWaveShr1>(0.f, tr[k][E - 1]), ter = dpp<kWaveShl1>(0.f, tr[k][0]);
        const float uwl = dpp<kWaveShr1>(0.f, un[k + 1][E - 1]), uer = dpp<kWaveShl1>(0.f, un[k + 1][0]);
        const float wwl = dpp<kWaveShr1>(0.f, wq[E - 1]), wer = dpp<kWaveShl1>(0.f, wq[0]);
        if (!out) continue;
        const bool row_rec = A.rvals && A.rrow[j] != 0;
        float go[E], lo[E], inv[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float tw = e == 0 ? twl : tr[k][e - 1], te = e == E - 1 ? ter : tr[k][e + 1];
            const float uw = e == 0 ? uwl : un[k + 1][e - 1], ue = e == E - 1 ? uer : un[k + 1][e + 1];
            const float ww = e == 0 ? wwl : wq[e - 1], we = e == E - 1 ? wer : wq[e + 1];
            const float s5t = ((tw + te) + (tm[e] + tp[e])) - 4.f * tr[k][e];
            const float s5u = ((uw + ue) + (un[k][e] + un[k + 2][e])) - 4.f * un[k + 1][e];
            const float sxw = (ww + we) - 2.f * wq[e];
            inv[e] = nr_rcp(rr[k][e]);
            const float mu = tr[k][e] * inv[e], nu = zr[k][e] * inv[e];
            go[e] = gr[k][e] + (mu * (A.c1 * s5u + A.c2 * sxw) + nu * (A.c2 * syd[e]));
            lo[e] = (2.f * l1[k][e] - l2[k][e]) + 2.f * s5t;
            if (row_rec && outl) {
                const int n0 = A.rmap[(size_t)j * nx + col0 + e];
                for (int n = n0 < A.nrec ? n0 : -1; n >= 0; n = A.rnext[n]) lo[e] += A.rvals[n];
            }
        }
        const f32x4 gv = {go[0], go[1], go[2], go[3]}, lv = {lo[0], lo[1], lo[2], lo[3]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, gv), rows(A.grad, j), ooff, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, lv), rows(A.lam2, j), ooff, 0, 0);
        // dJ/d(source value) = tau^2 t / r at the source nodes of the row
        if (A.gout) {
            for (int s = 0; s < (ns >= 0 ? ns : A.nsrc); ++s) {
                int wc = -1, kk = s;
                if (ns >= 0) {
                    if ((sh.src_pos[s] >> 16) == xr) { wc = sh.src_pos[s] & 0xffff; kk = sh.src_k[s]; }
                } else {
                    const int id = A.sidx[s];
                    if (id >= 0 && id < A.npts && id / nx == j) wc = id - j * nx - (c0 - kArKx);
                }
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (outl && lane * E + e == wc) A.gout[kk] = A.tau2 * (tr[k][e] * inv[e]);
            }
        }
    }
}

// tiles of the grid: the fewest columns of tiles of at most kArWmax, balanced
inline void adjoint_tiles(int nx, int ny, int& wt, int& tx, int& tiles)
{
    tx = (nx + kArWmax - 1) / kArWmax;
    wt = ((nx + tx - 1) / tx + 7) / 8 * 8;
    tx = (nx + wt - 1) / wt;
    tiles = tx * ((ny + kArHt - 1) / kArHt);
}

}  // namespace adw
