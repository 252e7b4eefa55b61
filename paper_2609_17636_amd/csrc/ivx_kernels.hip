// gfx950 kernels of one Classic3D objective/gradient evaluation.
//
// Forward direction (Sect. 2.1), per (pointing k, channel c) block:
//   k_image_rows  bilinear SIN reprojection of the sky (Eq. sin_projection) x beam x flux
//                 scale x deapodization, zero-padded to the fine grid, and the row FFT of
//                 two real rows packed in one complex transform (half spectrum kept);
//   k_col_fwd     column FFT of the n_sub non-zero rows, written to an extended grid that
//                 carries the periodic wrap in rows and the Hermitian mirror in columns,
//                 so a footprint never needs a modulo;
//   k_gridmx /    per fine-grid tile: interpolate every visibility from the grid window
//   k_grid        (degridding), form the residual and its weighted square (Sect. 2.2,
//                 J_k), and spread w * r back into the window's accumulation (matrix-core
//                 products in registers, or per-wave LDS accumulators; no global atomics);
//                 the window is written to a private slot.
// Adjoint direction (gradient, Sect. 3.4):
//   k_ext_sum     sum the slots covering each cell of the extended grid (the fold);
//   k_col_inv     alias sum and symmetrisation H -> (H + conj H(-t))/2 as it loads, which
//                 makes the real part of the adjoint a half-spectrum inverse FFT; inverse
//                 column FFT, keeping the n_sub rows of the sub-image;
//   k_row_inv     inverse row FFT of two rows at once, crop, deapodization x beam x flux;
//   k_sky         transpose of the bilinear reprojection (gather over a pixel-major CSR,
//                 fixed order), plus the Laplacian regulariser (Eq. 3) and the single-dish
//                 gradient (Sect. 2.4); k_sd_rows / k_sd_cols give the single-dish model.
// The NUFFT is the exponential-of-semicircle scheme of Barnett et al. (2019): kernel
// phi(z) = exp(beta (sqrt(1 - (2z/W)^2) - 1)), deapodization by its Fourier transform.
#include "ivx_internal.hpp"
#include "ivx_fft.hpp"

#include <math.h>

#include <algorithm>

#include <type_traits>

namespace ivx {

// --------------------------------------------------------------- forward row pass
template <int LOGN>
__global__ __launch_bounds__(NT) void k_image_rows(Geom g, const real *__restrict__ sky,
                                                   const real *__restrict__ beams,
                                                   const real *__restrict__ interp,
                                                   const real *__restrict__ fscale,
                                                   const real *__restrict__ dq,
                                                   const cpx *__restrict__ tw, cpx *__restrict__ R) {
    constexpr int N = 1 << LOGN;
    using F = Fft<LOGN, 1, (LOGN >= 11)>;
    __shared__ cpx buf[N + 1]; // + a sink cell for the stores of positions past the end
    __shared__ cpx tws[tw_len<LOGN>()];
    TwStage<LOGN> twr;
    twr.fetch(tw);
    const int tid = threadIdx.x;
    const int item = blockIdx.y;
    const int k = item / g.C, c = item - (item / g.C) * g.C;
    const int a0 = 2 * blockIdx.x;
    const int nk = g.nk;
    const real *x = sky + (int64_t)c * g.N * g.N;
    const real *A = beams + (int64_t)k * nk * nk;
    const real *G = interp + (int64_t)k * nk * nk * 2;
    const real s = fscale[c];
    for (int i = tid; i < N; i += NT) buf[i] = cpx{0, 0};
    __syncthreads();
    const real q0 = s * dq[a0], q1 = s * dq[a0 + 1];
    // IR_U columns per thread: their beam values and sample positions are requested together,
    // then every sky tap of both rows (positions past the end read column 0 and store to the
    // sink cell): two round trips instead of two per row and column
    constexpr int IR_U = 2;
    for (int b0 = tid; b0 < nk; b0 += IR_U * NT) {
        real dv[IR_U], a_0[IR_U], a_1[IR_U], y0[IR_U], x0[IR_U], y1[IR_U], x1[IR_U];
#pragma unroll
        for (int u = 0; u < IR_U; ++u) {
            const int b = b0 + u * NT < nk ? b0 + u * NT : 0;
            const int64_t e0 = (int64_t)a0 * nk + b, e1 = e0 + nk;
            dv[u] = dq[b];
            a_0[u] = A[e0];
            a_1[u] = A[e1];
            y0[u] = G[2 * e0];
            x0[u] = G[2 * e0 + 1];
            y1[u] = G[2 * e1];
            x1[u] = G[2 * e1 + 1];
        }
        BilinearTaps t0[IR_U], t1[IR_U];
        real p0[IR_U][4], p1[IR_U][4];
#pragma unroll
        for (int u = 0; u < IR_U; ++u) {
            t0[u] = bilinear_taps(g.N, y0[u], x0[u]);
            t1[u] = bilinear_taps(g.N, y1[u], x1[u]);
        }
#pragma unroll
        for (int u = 0; u < IR_U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                p0[u][j] = x[t0[u].o[j]];
                p1[u][j] = x[t1[u].o[j]];
            }
#pragma unroll
        for (int u = 0; u < IR_U; ++u) {
            const int b = b0 + u * NT;
            const real f0 = q0 * dv[u] * a_0[u] * t0[u].combine(p0[u][0], p0[u][1], p0[u][2], p0[u][3]);
            const real f1 = q1 * dv[u] * a_1[u] * t1[u].combine(p1[u][0], p1[u][1], p1[u][2], p1[u][3]);
            buf[b < nk ? F::at((b - nk / 2) & (N - 1)) : N] = cpx{f0, f1};
        }
    }
    twr.store(tws);
    __syncthreads();
    F::forward(buf, tws);
    cpx *R0 = R + (int64_t)item * g.r_stride + (int64_t)a0 * g.rw;
    cpx *R1 = R0 + g.rw;
    for (int kk = tid; kk <= N / 2; kk += NT) {
        const cpx z = buf[F::at(kk)], zm = buf[F::at((N - kk) & (N - 1))];
        // X = (Z + conj Zm)/2 (row a0), Y = (Z - conj Zm)/(2i) (row a0+1)
        R0[kk] = cpx{real(0.5) * (z.re + zm.re), real(0.5) * (z.im - zm.im)};
        R1[kk] = cpx{real(0.5) * (z.im + zm.im), real(0.5) * (zm.re - z.re)};
    }
}

// -------------------------------------------------------------- forward column pass
template <int LOGN, int CB>
__global__ __launch_bounds__(NT) void k_col_fwd(Geom g, const cpx *__restrict__ R,
                                                const cpx *__restrict__ tw, cpx *__restrict__ ext) {
    constexpr int N = 1 << LOGN;
    using F = ColFft<LOGN, CB>;
    constexpr int MAXE = 8 * CB;
    __shared__ cpx buf[F::LEN + 1]; // + a sink cell for the stores of positions past the end
    __shared__ cpx tws[tw_len<LOGN>()];
    TwStage<LOGN> twr;
    twr.fetch(tw);
    __shared__ int ent_col[MAXE];
    __shared__ int ent_src[MAXE];
    __shared__ int n_ent;
    const int tid = threadIdx.x;
    int item, c0;
    if (!col_block<CB>(g, item, c0)) return;
    const int nk = g.nk;
    for (int i = tid; i < F::LEN; i += NT) buf[i] = cpx{0, 0};
    if (tid == 0) {
        // extended columns fed by this block's source columns: direct copies at
        // src + O + m N, Hermitian mirrors (conjugate, row-reversed) at N - src + O + m N
        int n = 0;
        for (int cc = 0; cc < CB; ++cc) {
            const int src = c0 + cc;
            if (src >= g.rw) break;
            for (int m = -2; m <= 2; ++m) {
                const int ec = src + g.O + m * N;
                if (ec >= 0 && ec < g.ew && n < MAXE) { ent_col[n] = ec; ent_src[n] = cc; ++n; }
            }
            if (src != 0 && src != N / 2) {
                for (int m = -2; m <= 2; ++m) {
                    const int ec = N - src + g.O + m * N;
                    if (ec >= 0 && ec < g.ew && n < MAXE) { ent_col[n] = ec; ent_src[n] = cc | 0x10000; ++n; }
                }
            }
        }
        n_ent = n;
    }
    __syncthreads();
    const cpx *Ri = R + (int64_t)item * g.r_stride;
    // COL_LOADS rows of the source per thread are requested before the first is stored, so
    // that a block keeps that many loads per lane in flight instead of one.  Loads and stores
    // are unconditional (positions past the end read element 0 and store to the sink cell):
    // with either behind a branch the compiler waits for each load before issuing the next.
    for (int e0 = tid; e0 < nk * CB; e0 += COL_LOADS * NT) {
        cpx v[COL_LOADS];
#pragma unroll
        for (int u = 0; u < COL_LOADS; ++u) {
            const int e = e0 + u * NT, a = e / CB, cc = e - (e / CB) * CB;
            const bool ok = e < nk * CB && c0 + cc < g.rw;
            v[u] = Ri[ok ? (int64_t)a * g.rw + c0 + cc : 0];
        }
#pragma unroll
        for (int u = 0; u < COL_LOADS; ++u) {
            const int e = e0 + u * NT, a = e / CB, cc = e - (e / CB) * CB;
            const bool ok = e < nk * CB && c0 + cc < g.rw;
            buf[ok ? F::at((a - nk / 2) & (N - 1), cc) : F::LEN] = v[u];
        }
    }
    twr.store(tws);
    __syncthreads();
    F::forward(buf, tws);
    cpx *E = ext + (int64_t)item * g.ext_stride;
    const int ne = n_ent;
    for (int e = tid; e < ne * g.eh; e += NT) {
        const int en = e / g.eh, er = e - (e / g.eh) * g.eh;
        const int src = ent_src[en];
        const int cc = src & 0xFFFF;
        const int t1 = (er - g.O) & (N - 1);
        cpx v;
        if (src & 0x10000) {
            v = buf[F::at((N - t1) & (N - 1), cc)];
            v.im = -v.im;
        } else {
            v = buf[F::at(t1, cc)];
        }
        E[(int64_t)ent_col[en] * g.eh + er] = v; // column-major
    }
}

// ------------------------------------------------------------------- gridding kernel
// phi(z) = exp(beta (sqrt(1 - (2z/W)^2) - 1)).  In the float build the exponential is
// taken as exp2 of a prescaled argument (v_exp_f32, v_sqrt_f32): an argument error d
// changes phi by phi * d, and phi * |argument| never exceeds 1/e, so the absolute error
// stays at the rounding level of the peak weight.  v_sqrt_f32 rounds down on average, which beta makes a
// common factor of all weights (-1.5e-7 an axis at W = 6, and -3e-7 in the matrix-core gridder's
// scaling); half the remainder q - s^2, its Newton correction where s is near 1, leaves -1e-8.
// beta2 = beta (double build) or beta * log2(e) (float build).
__device__ __forceinline__ real es_kernel(real z, real inv_half_w, real beta2) {
    const real t = z * inv_half_w;
    const real q = real(1) - t * t;
#ifdef IVX_REAL_DOUBLE
    return exp(beta2 * (sqrt(q > real(0) ? q : real(0)) - real(1)));
#else
    const float p = q > 0.f ? q : 0.f, s = __builtin_amdgcn_sqrtf(p);
    return __builtin_amdgcn_exp2f(beta2 * __builtin_fmaf(0.5f, __builtin_fmaf(-s, s, p), s - 1.f));
#endif
}

__device__ __forceinline__ void decode(const VisCoord &v, int &ix, int &iy, real &fx, real &fy) {
#ifdef IVX_REAL_DOUBLE
    ix = (int)v.ix;
    iy = (int)v.iy;
    fx = v.fx;
    fy = v.fy;
#else
    ix = (int)(v.xq >> 24);
    iy = (int)(v.yq >> 24);
    fx = (real)(v.xq & 0xFFFFFFu) * real(5.9604644775390625e-08); // 2^-24
    fy = (real)(v.yq & 0xFFFFFFu) * real(5.9604644775390625e-08);
#endif
}

struct GridArgs {
    Geom g;
    const WorkItem *work;
    const VisCoord *crd;
    const cpx *vis;
    const real *wgt;
    const int32_t *perm;
    const int64_t *boff;
    const cpx *ext;
    cpx *slots;
    double *jpart;
    const cpx *caller_in;
    cpx *caller_out;
    int nwave;
    int n_work;
    int unweighted; // adjoint mode: spread the given visibilities without the natural weights
    // w-plane modes
    const WZ *wz;
    cpx *wacc;
    const cpx *wq;
    int wplane;
    int wW;
    real wbeta2; // w kernel shape, scaled like beta2 below
    const int32_t *wcnt; // record counts below each half plane per work item, or NULL
    int wncnt;
    uint8_t *wsact;      // adjoint plane pass: slot written (1) or skipped (0), or NULL
    float esc, esb;      // matrix-core gridder: phi(z) = 2^(esc sqrt(W^2 / 4 - z^2) - esb)
    float minus1;        // -1
};

// Signed distance, in planes, of a record's w from plane p.
__device__ __forceinline__ real wz_dist(WZ z, int p) {
#ifdef IVX_REAL_DOUBLE
    return z - (double)p;
#else
    return (real)((int)(z >> 24) - p) + (real)(z & 0xFFFFFFu) * real(5.9604644775390625e-08);
#endif
}

// First record of a work item's (sorted) list whose plane coordinate reaches the given
// number of half planes: lower bound of zeta >= h2 / 2.
__device__ __forceinline__ int wz_lower(const WZ *__restrict__ z, int n, int h2) {
#ifdef IVX_REAL_DOUBLE
    const double key = 0.5 * (double)h2;
#else
    const int64_t k = (int64_t)h2 << 23;
    if (k <= 0) return 0;
    if (k > (int64_t)0xFFFFFFFFll) return n;
    const uint32_t key = (uint32_t)k;
#endif
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (z[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Work items per row of the gridding launch: the dispatch packet counts work-items of one
// grid dimension in 32 bits, so long work lists (spectral cubes) wrap into blockIdx.y.
constexpr unsigned GRID_ROW = 1u << 22;

// ---- cross-lane moves inside a 16-lane DPP row (VALU, no LDS traffic)
// (mov_dpp with bound_ctrl: lanes without a source read 0, and no old value has to be
// materialised first)
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ double dpp(double v) {
    const int2 p = __builtin_bit_cast(int2, v);
    int2 r;
    r.x = __builtin_amdgcn_mov_dpp(p.x, CTRL, 0xF, 0xF, true);
    r.y = __builtin_amdgcn_mov_dpp(p.y, CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, r);
}
template <int L> __device__ __forceinline__ real row_bcast(real v) { return dpp<0x150 + L>(v); }


__device__ __forceinline__ real row_shr8(real v) { return dpp<0x118>(v); }

// Lane layout of a G-lane group (one visibility at a time):
//   G = 8  (W <= 8): lane j owns footprint column j, all W rows (two groups per DPP row);
//   G = 16, W <= 8 : lane t owns column t & 7 and every other row starting at t >> 3;
//   G = 16, W > 8  : lane t < W owns column t, all W rows.
template <int W, int G> struct Layout {
    static_assert(G == 16 || W <= 8, "8-lane groups need W <= 8");
    static constexpr int S = (G == 16 && W <= 8) ? 2 : 1; // row stride of a lane
    static constexpr int NR = (W + S - 1) / S;            // rows per lane (upper bound)
};

// Row weights of the group in every lane: wsel[k] is the weight of the lane's k-th row.
template <int W, int G, int I> struct RowWeights {
    __device__ __forceinline__ static void run(real mine, bool upper, real *wsel) {
        if constexpr (G == 8) {
            const real lo = row_bcast<I>(mine), hi = row_bcast<8 + I>(mine);
            wsel[I] = upper ? hi : lo;
        } else if constexpr (Layout<W, G>::S == 2) {
            // rows 2k (lanes h = 0) and 2k + 1 (h = 1) come from lanes 8 + 2k and 8 + 2k + 1
            if constexpr (I % 2 == 0) {
                const real e0 = row_bcast<8 + I>(mine);
                const real e1 = (I + 1 < W) ? row_bcast<8 + ((I + 1 < W) ? I + 1 : I)>(mine) : real(0);
                wsel[I / 2] = upper ? e1 : e0;
            }
        } else {
            wsel[I] = row_bcast<I>(mine);
        }
        RowWeights<W, G, I + 1>::run(mine, upper, wsel);
    }
};
template <int W, int G> struct RowWeights<W, G, W> {
    __device__ __forceinline__ static void run(real, bool, real *) {}
};

// sum over the lanes of the group, returned in every lane of the group
template <int G> __device__ __forceinline__ real group_sum(real v) {
    v += dpp<0xB1>(v);  // quad xor 1
    v += dpp<0x4E>(v);  // quad xor 2
    v += dpp<0x141>(v); // half-row mirror: the other quad of the 8
    if constexpr (G == 16) v += dpp<0x140>(v); // row mirror: the other half
    return v;
}

// One block per work item (a fine-grid tile, or a chunk of one).  The block's waves split
// into groups of G lanes; group g walks its own contiguous segment of the tile's
// visibility list.  Inside a group the kernel weights are evaluated once (one or two per
// lane) and moved across lanes with DPP row operations, and the degridded value is a DPP
// group sum, so no cross-lane traffic touches the LDS.  Every group spreads into its own
// LDS accumulator window with plain read-modify-write (the lanes of a group own distinct
// cells and no other group writes there): no atomics.  The windows are summed in a fixed
// order at the end, so results do not depend on scheduling.
// LDS: F window (unless MODE_ADJ) + one accumulator window per group (unless MODE_FWD),
// each column-major with column stride ldw: the rows a lane owns in one footprint column
// are then a few cells apart, so their offsets are immediates of the LDS instructions.
template <int W, int MODE, int G, int VPI>
__global__ __launch_bounds__(NT) void k_grid(GridArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[NT / 64];
    constexpr int S = Layout<W, G>::S, NR = Layout<W, G>::NR;
    constexpr int GPW = 64 / G; // groups per wave
    const Geom &g = a.g;
    const int win = g.win, ldw = g.ldw;
    const int wsz = win * ldw;
    const int nwave = a.nwave;
    const int ngroups = nwave * GPW;
    cpx *Fw = reinterpret_cast<cpx *>(smem_raw);
    constexpr bool WPL = MODE == MODE_WFWD || MODE == MODE_WADJ; // one w plane of the full model
    constexpr bool NOGRID = MODE == MODE_ADJ || MODE == MODE_WADJ; // the grid window is not read
    constexpr bool SPREAD = MODE == MODE_OBJ || MODE == MODE_ADJ || MODE == MODE_WADJ;
    constexpr bool DATA = MODE == MODE_OBJ || MODE == MODE_VAL; // residual against the data
    cpx *Hw = Fw + (NOGRID ? 0 : wsz);
    const int64_t wid = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (wid >= a.n_work) return; // tail of the last row: the whole block leaves together
    const WorkItem wi = a.work[wid];
    const int tid = threadIdx.x;
    // e = cc * win + r without an integer division: (e + 1/2) / win is never within float
    // rounding of an integer for e < 2^16
    const float inv_win = 1.0f / (float)win;
    // a w plane only takes the records whose w kernel reaches it, zeta in [p - W_w / 2,
    // p + W_w / 2): a contiguous range of the work item's list (sorted by zeta).  Most work
    // items meet a plane with no such record: the degrid pass then has nothing to do and the
    // spread pass writes a zero window (the values are block-uniform, so the whole block
    // leaves together).
    int base = 0, cnt = wi.count;
    if constexpr (WPL) {
        const int h0 = 2 * a.wplane - a.wW, h1 = 2 * a.wplane + a.wW;
        if (a.wcnt) {
            // two independent loads from the work item's table instead of two chains of
            // dependent loads
            const int32_t *c = a.wcnt + wid * (int64_t)a.wncnt;
            base = h0 <= 0 ? 0 : (h0 >= a.wncnt ? wi.count : c[h0]);
            cnt = (h1 <= 0 ? 0 : (h1 >= a.wncnt ? wi.count : c[h1])) - base;
        } else {
            const WZ *z = a.wz + wi.begin;
            base = wz_lower(z, wi.count, h0);
            cnt = wz_lower(z, wi.count, h1) - base;
        }
        if (MODE == MODE_WADJ && a.wsact && tid == 0) a.wsact[wi.slot] = cnt > 0 ? 1 : 0;
        if (cnt == 0) {
            if (MODE == MODE_WADJ && !a.wsact) {
                cpx *Sl = a.slots + (int64_t)wi.slot * g.win_stride;
                for (int e = tid; e < win * win; e += blockDim.x) Sl[e] = cpx{0, 0};
            }
            return;
        }
    }
    if (!NOGRID) {
        const cpx *F = a.ext + (int64_t)wi.item * g.ext_stride + (int64_t)(wi.tx * g.T) * g.eh + wi.ty * g.T;
        for (int e = tid; e < win * win; e += blockDim.x) {
            const int cc = (int)(((float)e + 0.5f) * inv_win), r = e - cc * win;
            Fw[cc * ldw + r] = F[cc * g.eh + r];
        }
    }
    if (SPREAD) {
        for (int e = tid; e < ngroups * wsz; e += blockDim.x) Hw[e] = cpx{0, 0};
    }
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6;
    const int t = lane & (G - 1);
    const int j = (S == 2) ? (t & 7) : t;   // footprint column owned
    const int h = (S == 2) ? (t >> 3) : 0;  // first footprint row owned
    const bool upper = (lane & 8) != 0;      // second half of the DPP row
    const bool colok = j < W;
    const int gid = wave * GPW + lane / G;
    cpx *Hg = Hw + gid * wsz;
    const real inv_hw = real(2) / real(W);
#ifdef IVX_REAL_DOUBLE
    const real beta2 = g.beta;
#else
    const real beta2 = (float)g.esc * (0.5f * (float)g.W); // exact (es_shape)
#endif
    const real zoff = real(0.5) * real(W) - real(1);
    real jacc = real(0);

    // this group's segment of the tile's list (of the plane's range), walked VPI visibilities
    // at a time
    const int seg = (cnt + ngroups - 1) / ngroups;
    const int v0 = base + gid * seg;
    const int v1 = min(base + cnt, v0 + seg);
    const int nit = (seg + VPI - 1) / VPI;
    const VisCoord *crd = a.crd + wi.begin;
    const cpx *vis = a.vis + wi.begin;
    const real *wgt = a.wgt + wi.begin;
    const int32_t *perm = a.perm + wi.begin;
    cpx *caller_out = nullptr;
    const cpx *caller_in = nullptr;
    if (MODE == MODE_FWD) caller_out = a.caller_out + a.boff[wi.item];
    if (MODE == MODE_ADJ) caller_in = a.caller_in + a.boff[wi.item];
    // per-lane record index as an unsigned 32-bit byte offset from the block's (uniform)
    // bases, so the loads take the scalar-base + 32-bit vector-offset form
    auto rec = [&](int vv) -> unsigned { return (unsigned)(vv < v1 ? vv : 0); };
    auto at = [](const auto *base, unsigned i) {
        using T = std::remove_cv_t<std::remove_pointer_t<decltype(base)>>;
        return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + i * (unsigned)sizeof(T));
    };

    // record of one visibility (the fields this mode reads)
    struct Rec {
        VisCoord c;
        cpx y;
        real w;
        int32_t p;
    };
    auto load = [&](Rec (&r)[VPI], int it) {
#pragma unroll
        for (int u = 0; u < VPI; ++u) {
            const unsigned vn = rec(v0 + it * VPI + u);
            r[u].c = at(crd, vn);
            r[u].y = cpx{0, 0};
            r[u].w = real(0);
            r[u].p = 0;
            if (DATA) { r[u].y = at(vis, vn); r[u].w = at(wgt, vn); }
            if (MODE == MODE_ADJ) { r[u].w = a.unweighted ? real(1) : at(wgt, vn); r[u].p = at(perm, vn); }
            if (MODE == MODE_FWD) { r[u].p = at(perm, vn); }
            if constexpr (WPL) {
                // w carries the record's w-kernel weight for this plane, y its coefficient
                r[u].w = es_kernel(wz_dist(at(a.wz + wi.begin, vn), a.wplane), real(2) / real(a.wW), a.wbeta2);
                if (MODE == MODE_WADJ) r[u].y = at(a.wq + wi.begin, vn);
            }
        }
    };

    // one iteration: VPI visibilities of this group's segment
    auto step = [&](const Rec (&cur)[VPI], int it) {
        bool valid[VPI];
#pragma unroll
        for (int u = 0; u < VPI; ++u) valid[u] = v0 + it * VPI + u < v1;
        int off[VPI];
        real wxj[VPI], wsel[VPI][NR];
#pragma unroll
        for (int u = 0; u < VPI; ++u) {
            int ix, iy;
            real fx, fy;
            decode(cur[u].c, ix, iy, fx, fy);
            // kernel weights: x weight of the owned column, y weights of the owned rows
            if constexpr (G == 16 && S == 2) {
                // lanes 0-7 evaluate the column weights, lanes 8-15 the row weights; DPP row
                // moves hand every lane its column's weight and its rows' weights
                const bool isx = t < 8;
                const int k = t & 7;
                real mine = real(0);
                if (k < W) mine = es_kernel(zoff + (isx ? fx : fy) - real(k), inv_hw, beta2);
                const real sh = row_shr8(mine);
                wxj[u] = isx ? mine : sh;
                RowWeights<W, G, 0>::run(mine, upper, wsel[u]);
            } else if constexpr (G == 8) {
                real mx = real(0), my = real(0);
                if (colok) {
                    mx = es_kernel(zoff + fx - real(j), inv_hw, beta2);
                    my = es_kernel(zoff + fy - real(j), inv_hw, beta2);
                }
                wxj[u] = mx;
                RowWeights<W, G, 0>::run(my, upper, wsel[u]);
            } else {
                real mx = real(0), my = real(0);
                if (colok) {
                    mx = es_kernel(zoff + fx - real(j), inv_hw, beta2);
                    my = es_kernel(zoff + fy - real(j), inv_hw, beta2);
                }
                wxj[u] = mx;
                RowWeights<W, G, 0>::run(my, upper, wsel[u]);
            }
            if (!valid[u]) wxj[u] = real(0);
            off[u] = (int)__umul24((unsigned)(ix + j), (unsigned)ldw) + iy + h;
        }
        real ar[VPI], ai[VPI];
#pragma unroll
        for (int u = 0; u < VPI; ++u) {
            ar[u] = real(0);
            ai[u] = real(0);
        }
        if (!NOGRID) {
            if (colok) {
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    if (S == 1 || h + S * k < W) {
#pragma unroll
                        for (int u = 0; u < VPI; ++u) {
                            const cpx f = Fw[off[u] + S * k];
                            ar[u] += wsel[u][k] * f.re;
                            ai[u] += wsel[u][k] * f.im;
                        }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < VPI; ++u) {
                ar[u] = group_sum<G>(ar[u] * wxj[u]);
                ai[u] = group_sum<G>(ai[u] * wxj[u]);
            }
        }
        if (MODE == MODE_FWD) {
#pragma unroll
            for (int u = 0; u < VPI; ++u) {
                if (valid[u] && t == 0) {
                    if (cur[u].p < 0) caller_out[~cur[u].p] = cpx{ar[u], -ai[u]};
                    else caller_out[cur[u].p] = cpx{ar[u], ai[u]};
                }
            }
            return;
        }
        if (MODE == MODE_WFWD) {
            // planes run as successive launches and a record belongs to one group of one work
            // item: a plain read-modify-write, in plane order
#pragma unroll
            for (int u = 0; u < VPI; ++u) {
                if (valid[u] && t == 0) {
                    cpx *o = a.wacc + wi.begin + (v0 + it * VPI + u);
                    cpx ov = *o;
                    ov.re += cur[u].w * ar[u];
                    ov.im += cur[u].w * ai[u];
                    *o = ov;
                }
            }
            return;
        }
        real cre[VPI], cim[VPI];
#pragma unroll
        for (int u = 0; u < VPI; ++u) {
            if (DATA) {
                const real rr = ar[u] - cur[u].y.re, ri = ai[u] - cur[u].y.im;
                if (valid[u] && t == 0) jacc += cur[u].w * (rr * rr + ri * ri); // halved at the end
                const real ww = cur[u].w * wxj[u];
                cre[u] = ww * rr;
                cim[u] = ww * ri;
            } else if (MODE == MODE_WADJ) {
                cre[u] = cur[u].w * cur[u].y.re * wxj[u];
                cim[u] = cur[u].w * cur[u].y.im * wxj[u];
            } else {
                cpx y = caller_in[cur[u].p < 0 ? ~cur[u].p : cur[u].p];
                if (cur[u].p < 0) y.im = -y.im;
                cre[u] = cur[u].w * y.re * wxj[u];
                cim[u] = cur[u].w * y.im * wxj[u];
            }
        }
        // spread: the visibilities of one iteration go in program order, so a cell shared
        // by two of them (owned by different lanes) sees both updates
        if (SPREAD && colok) {
#pragma unroll
            for (int u = 0; u < VPI; ++u) {
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    if (S == 1 || h + S * k < W) {
                        cpx *hp = Hg + off[u] + S * k;
                        cpx hv = *hp;
                        hv.re += cre[u] * wsel[u][k];
                        hv.im += cim[u] * wsel[u][k];
                        *hp = hv;
                    }
                }
            }
        }
    };

    // three record sets rotate: the records of iteration it + 2 are requested as iteration
    // it starts, two iterations of latency cover (no register copies between stages)
    Rec r0[VPI], r1[VPI], r2[VPI];
    load(r0, 0);
    load(r1, 1);
    for (int it = 0; it < nit; it += 3) {
        if (it + 2 < nit) load(r2, it + 2);
        step(r0, it);
        if (it + 1 >= nit) break;
        if (it + 3 < nit) load(r0, it + 3);
        step(r1, it + 1);
        if (it + 2 >= nit) break;
        if (it + 4 < nit) load(r1, it + 4);
        step(r2, it + 2);
    }
    if (MODE == MODE_FWD || MODE == MODE_WFWD) return;
    if (SPREAD) {
        __syncthreads();
        cpx *Sl = a.slots + (int64_t)wi.slot * g.win_stride; // column-major window
        for (int e = tid; e < win * win; e += blockDim.x) {
            const int cc = (int)(((float)e + 0.5f) * inv_win), r = e - cc * win;
            real sr = real(0), si = real(0);
            for (int q = 0; q < ngroups; ++q) {
                const cpx hh = Hw[q * wsz + cc * ldw + r];
                sr += hh.re;
                si += hh.im;
            }
            Sl[e] = cpx{sr, si};
        }
    }
    if (DATA) {
        double d = 0.5 * (double)jacc;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) d += __shfl_xor(d, m, 64);
        if (lane == 0) red[wave] = d;
        __syncthreads();
        if (tid == 0) {
            double sacc = 0.0;
            for (int w = 0; w < nwave; ++w) sacc += red[w];
            a.jpart[wid] = sacc;
        }
    }
}

int grid_groups_per_wave(int W, int lanes) { return (lanes == 8 && W <= 8) ? 8 : 4; }

#ifndef IVX_REAL_DOUBLE
// ---------------------------------------------------- gridding on the matrix cores
// The same degrid / residual / spread as k_grid, written as per-tile matrix products (float
// build, windows of at most 16 x 16 cells).  One wave per work item; per batch of 32
// visibilities, with PX[m][b] and PY[m][a] the kernel weights of visibility m at the window's
// columns b and rows a (zero outside its footprint),
//   degrid   Q[a][m] = sum_b F[a][b] PX[m][b]                  (K = b, re and im rows stacked)
//            V_m     = sum_a PY[m][a] Q[a][m]                  (8 rows per lane, one lane swap)
//   spread   H[a][b] += sum_m PY[m][a] (w_m r_m) PX[m][b]      (K = m)
// The window F and the accumulation H stay in registers for the whole work item; H is
// written to the work item's slot at the end.
//
// Arithmetic.  Every factor is split into two half-precision parts, x = h + l with h the
// nearest half and l the nearest half to x - h, and a product is the three matrix products
// h h' + h l' + l h' accumulated in FP32 (v_mfma_f32_32x32x16_f16, v_mfma_f32_16x16x32_f16).
// A half has 11 bits, so |l| is at most 2^-11 |x|, the pair is x to 2^-24 of the power of two above |x| (one FP32
// unit, for a quarter of the values), and the dropped l l' reaches 2^-22 of h h': at worst a product is 2^-21
// off, eight times an FP32 one.  On average the matrix instructions' fewer roundings of the sum make up for it: dot
// products of 32 and of 256 normal deviates are 8.2e-8 and 2.0e-7 off, 1.1e-7 and 2.8e-7 on v_mfma_f32_16x16x4_f32.
// Whole calls (L2 error against 64 bits, geometric mean of 21 problems; in brackets this kernel on FP32 products with the
// same weights): gradient 2.52e-7 (2.48), model 3.31e-7 (3.18), adjoint 2.28e-7 (2.24); the kernel on FP32 products
// that it replaced, whose weights carried the rounding of the square root and of the exponent's constant, 6.2, 5.0
// and 4.6e-7.  With l l' they are 2.49, 3.28 and 2.26e-7, for 5% of the time.
// Halves reach down to 2^-24, so the window and w r are scaled by powers of two (exactly): the window by
// its largest value, w r by a scale of the work item that is lowered, with H, when a batch
// exceeds it; weights are at most 1 and keep 2^-24 of the peak.  A record 2^17 and more below its item's largest has
// fewer bits; what it loses is 2^-39 of the largest, whose own FP32 rounding is 2^-24 of it.  (Adjoints of data that spread
// over 2^20 and 2^40, or with one or 1% of the samples 10^6 and 10^7 times the rest, are off as they are on FP32 products.)
//
// What bounds it: instruction issue.  A wave64 vector instruction takes 4 cycles of its SIMD, an
// exponential or square root 8, and a matrix instruction holds the SIMD's issue for 16 whatever
// its size, so the eight-times cheaper half-precision products leave the vector work (the weights,
// their splits, the row sum) as the cost.  Each weight is therefore evaluated once, by lane
// (m = l % 32, axis l / 32), stored to a row of LDS between zeros that are never overwritten, and
// read back at the window's fixed positions as a row shifted by the footprint's start: no
// per-batch clearing and no test of the footprint's bounds.  The K = m operands of the spread are
// rows [m][position] read through the transposing LDS load.  157 vector instructions (14 of them exponentials and
// roots) and 9 matrix instructions a batch at W = 7, and some 290 an item: 883 cycles of a SIMD a batch with its share
// of the item's (seven batches an item on the 128-channel cube).  Measured against FP32 matrix products in batches
// of 16 (gridding alone): 845 -> 481 us on 34.4 M visibilities of 36 pointings in 192,839 items, 122.0 -> 81.7 ms on
// 128 channels of them (5.1e9 in 24.7 M), 29 -> 19.7 us on one 512^2 pointing of 630,000.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int MX_B = 32;             // visibilities per batch
constexpr int MX_FBITS = 14;         // the window's largest value lies in [2^14, 2^15)
constexpr int MX_RBITS = 14;         // a new scale puts the largest |w r| in [2^14, 2^15) ...
constexpr float MX_RMAX = 65000.f;   // ... and is kept while they stay below this (weights are <= 1)

// LDS hand-off between the lanes of the (single-wave) block: a wave's LDS operations are
// performed in order, so only the compiler has to be kept from moving accesses across;
// unlike a block barrier this does not wait for the wave's outstanding global loads.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Largest x of the wave, in every lane (x >= 0; a NaN is passed over).
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp<0xB1>(x));
    x = fmaxf(x, dpp<0x4E>(x));
    x = fmaxf(x, dpp<0x141>(x));
    x = fmaxf(x, dpp<0x140>(x));
    const unsigned u = __float_as_uint(x);
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned v = __float_as_uint(fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1])));
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// Sum over the wave, in every lane.
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp<0xB1>(x);
    x += dpp<0x4E>(x);
    x += dpp<0x141>(x);
    x += dpp<0x140>(x);
    const uint2 u = __builtin_bit_cast(uint2, x);
    const auto p0 = __builtin_amdgcn_permlane16_swap(u.x, u.x, false, false);
    const auto p1 = __builtin_amdgcn_permlane16_swap(u.y, u.y, false, false);
    x = __builtin_bit_cast(double, uint2{p0[0], p1[0]}) + __builtin_bit_cast(double, uint2{p0[1], p1[1]});
    const uint2 v = __builtin_bit_cast(uint2, x);
    const auto q0 = __builtin_amdgcn_permlane32_swap(v.x, v.x, false, false);
    const auto q1 = __builtin_amdgcn_permlane32_swap(v.y, v.y, false, false);
    return __builtin_bit_cast(double, uint2{q0[0], q1[0]}) + __builtin_bit_cast(double, uint2{q0[1], q1[1]});
}

// Exponent s (|s| <= 126) such that 2^s x lies in [2^(bits), 2^(bits + 1)) as far as s reaches;
// 0, infinity and NaN give some s in range.
__device__ __forceinline__ int scale_bits(float x, int bits) {
    const int e = bits + 127 - (int)((__float_as_uint(x) >> 23) & 0xFF);
    return e > 126 ? 126 : (e < -126 ? -126 : e);
}

__device__ __forceinline__ float exp2_int(int e) { return __uint_as_float((unsigned)(e + 127) << 23); } // |e| <= 126

// Eight values as halves hi + lo: x = hi + lo to 2^-24 of the power of two above |x| (and to
// 2^-25 absolutely).  m1 is -1 in a register the compiler cannot see through: x - hi is then one
// mixed-precision multiply-add on the half instead of a conversion back and a subtraction.
__device__ __forceinline__ void split_halves(const float (&x)[8], float m1, f16x8 &hi, f16x8 &lo) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x2 v = {x[2 * i], x[2 * i + 1]};
        const f16x2 h = __builtin_convertvector(v, f16x2);
        const f32x2 d = {__builtin_fmaf((float)h[0], m1, v[0]), __builtin_fmaf((float)h[1], m1, v[1])};
        const f16x2 r = __builtin_convertvector(d, f16x2);
        hi[2 * i] = h[0];
        hi[2 * i + 1] = h[1];
        lo[2 * i] = r[0];
        lo[2 * i + 1] = r[1];
    }
}

// Operand of a K = m product from a table of rows [m][16 positions] of halves: lane (c = l % 16,
// g = l / 16) receives position c of the rows 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3 (K in an
// order that both operands share).  A table is stored as two halves of 8 positions, so that the
// lanes' 16-byte writes are consecutive.  at: this lane's chunk, row 4 g + c / 4, positions
// 4 (c % 4) .. + 3.
__device__ __forceinline__ f16x8 column_operand(const _Float16 *at) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    union {
        s16x4 p[2];
        f16x8 v;
    } r;
    r.p[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)at);
    r.p[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at + 128));
    return r.v;
}

// KW > 0 fixes the kernel width at compile time; KW = 0 reads it from the geometry.
// The LDS (7.7 KB, one table of the spread at a time) admits five waves per SIMD; all three tables at once left four
// (4% slower), and weight rows by visibility instead of by position cost 18% in bank conflicts.
template <int MODE, int KW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_gridmx(GridArgs a) {
    constexpr bool WPL = MODE == MODE_WFWD || MODE == MODE_WADJ; // one w plane of the full model
    constexpr bool NOGRID = MODE == MODE_ADJ || MODE == MODE_WADJ; // the grid window is not read
    constexpr bool SPREAD = MODE == MODE_OBJ || MODE == MODE_ADJ || MODE == MODE_WADJ;
    constexpr bool DATA = MODE == MODE_OBJ || MODE == MODE_VAL; // residual against the data
    // Weights, one row of 32 visibilities per position: the x weights in rows XR .. XR + 7, the y
    // weights in rows YR .. YR + 7, zeros around them.  A footprint starting at window cell i reads
    // position p at row XR - i + p, i <= 16 - W, p <= 15.  Lane m stays in bank m whatever i is.
    constexpr int ZR = KW > 0 ? 16 - KW : 12, XR = ZR, YR = XR + 8 + (ZR > 8 ? ZR : 8), NROW = YR + 16;
    __shared__ __align__(16) float PW[NROW * MX_B];
    // a table of the spread, hi and lo: PX, then the real and the imaginary part of w r PY in turn
    constexpr int TH = MX_B * 8 + 32, TB = 2 * TH; // halves of half a table (+ a bank offset), of one table
    __shared__ __align__(16) _Float16 TS[SPREAD ? 2 * TB : 8];
    const int64_t wid = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (wid >= a.n_work) return;
    const WorkItem wi = a.work[wid];
    if (wi.count <= 0) return; // (the work list holds no empty items)
    const Geom &g = a.g;
    const int l = threadIdx.x, m = l & 31, hf = l >> 5;
    const int c16 = l & 15, g4 = l >> 4;
    const int W = KW > 0 ? KW : g.W, win = g.win;
    const float m1 = a.minus1;
    // the records of this work item that the pass takes: all, or the plane's range
    int base = 0, n = wi.count;
    if constexpr (WPL) {
        const int h0 = 2 * a.wplane - a.wW, h1 = 2 * a.wplane + a.wW;
        if (a.wcnt) {
            const int32_t *c = a.wcnt + wid * (int64_t)a.wncnt;
            base = h0 <= 0 ? 0 : (h0 >= a.wncnt ? wi.count : c[h0]);
            n = (h1 <= 0 ? 0 : (h1 >= a.wncnt ? wi.count : c[h1])) - base;
        } else {
            const WZ *z = a.wz + wi.begin;
            base = wz_lower(z, wi.count, h0);
            n = wz_lower(z, wi.count, h1) - base;
        }
        if (MODE == MODE_WADJ && a.wsact && l == 0) a.wsact[wi.slot] = n > 0 ? 1 : 0;
        if (n == 0) { // (uniform over the wave) no record near the plane: no window, or a zero one
            if (MODE == MODE_WADJ && !a.wsact) {
                cpx *Sl = a.slots + (int64_t)wi.slot * g.win_stride;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 4 * g4 + v;
                    if (r < win && c16 < win) Sl[c16 * win + r] = cpx{0.f, 0.f};
                }
            }
            return;
        }
    }
    const VisCoord *crd = a.crd + wi.begin + base;
    const float *vis = reinterpret_cast<const float *>(a.vis + wi.begin);
    const real *wgt = a.wgt + wi.begin;
    const int32_t *perm = a.perm + wi.begin;
    const WZ *wzp = WPL ? a.wz + wi.begin + base : nullptr;
    float *wacc = MODE == MODE_WFWD ? reinterpret_cast<float *>(a.wacc + wi.begin + base) : nullptr;
    const float *wq = MODE == MODE_WADJ ? reinterpret_cast<const float *>(a.wq + wi.begin + base) : nullptr;
    const float inv_hww = WPL ? 2.f / (float)a.wW : 0.f;
    float *caller_out = MODE == MODE_FWD ? reinterpret_cast<float *>(a.caller_out + a.boff[wi.item]) : nullptr;
    const float *caller_in = MODE == MODE_ADJ ? reinterpret_cast<const float *>(a.caller_in + a.boff[wi.item]) : nullptr;
    // Records of a batch; two sets rotate so that the next batch's records are in flight while
    // the current batch is processed.  Lane (m, hf) takes the real (hf = 0) or imaginary
    // component of visibility m.  Every lane loads, at indices clamped to the last record (a batch
    // past the end reloads it and ignores it): with no per-lane branches around the loads the
    // wait before a batch covers only that batch's own loads.
    struct MxRec {
        VisCoord c;
        float y, w;
        int p;
    };
    // (uniform base + 32-bit byte offset, the form the load instructions take)
    auto at = [](const auto *base, unsigned bytes) {
        using T = std::remove_cv_t<std::remove_pointer_t<decltype(base)>>;
        return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + bytes);
    };
    auto fetch = [&](MxRec &r, int v0) {
        const unsigned o4 = 4u * (unsigned)min(v0 + m, n - 1), o8 = 2 * o4, oc = o8 + 4u * hf;
        r.c = at(crd, o8);
        if (DATA) { r.y = at(vis, oc); r.w = at(wgt, o4); }
        if (MODE == MODE_ADJ) { r.w = a.unweighted ? 1.f : at(wgt, o4); r.p = at(perm, o4); }
        if (MODE == MODE_FWD) r.p = at(perm, o4);
        if constexpr (WPL) {
            // w carries the record's w-kernel weight at this plane, y its coefficient
            r.w = es_kernel(wz_dist(at(wzp, o4), a.wplane), inv_hww, a.wbeta2);
            if (MODE == MODE_WADJ) r.y = at(wq, oc);
        }
    };
    MxRec ra{}, rb{};
    fetch(ra, 0);
    // window as the operand [32 rows: re rows 0..15, im rows 0..15][columns 8 hf .. 8 hf + 7].  Cells
    // past the window repeat its last row or column: their weights are zero.
    f16x8 fh{}, fl{};
    float vscale = 0.f;
    if (!NOGRID) {
        const float *F = reinterpret_cast<const float *>(a.ext + (int64_t)wi.item * g.ext_stride +
                                                         (int64_t)(wi.tx * g.T) * g.eh + wi.ty * g.T);
        float f[8], fm = 0.f;
        const unsigned row = 8u * min(c16, win - 1) + 4u * (m >> 4), col = 8u * g.eh;
        if (win == 16) {
            const unsigned o = row + 8u * hf * col;
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = at(F + 2 * j * g.eh, o);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = at(F, row + min(8 * hf + j, win - 1) * col);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) fm = fmaxf(fm, fabsf(f[j]));
        const int sb = scale_bits(wave_max(fm), MX_FBITS);
        const float sc = exp2_int(sb);
        vscale = exp2_int(-sb);
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] *= sc;
        split_halves(f, m1, fh, fl);
    }
#pragma unroll
    for (int i = 0; i < NROW * MX_B; i += 256)
        if (i + 256 <= NROW * MX_B || i + 4 * l < NROW * MX_B) *reinterpret_cast<f32x4 *>(PW + i + 4 * l) = f32x4{0.f, 0.f, 0.f, 0.f};
    const float hw2 = 0.25f * (float)(W * W), zoff = 0.5f * (float)W - 1.f;
    const float esc = a.esc, esb = a.esb, escw = a.esc / (float)W;
    f32x4 hre = {0.f, 0.f, 0.f, 0.f}, him = {0.f, 0.f, 0.f, 0.f};
    float jacc = 0.f;
    int rbits = 126;              // w r is scaled by 2^rbits
    float rscale = exp2_int(126);
    float *prow = PW + (hf ? YR : XR) * MX_B + m;
    const float *pxr = PW + (XR + 8 * hf) * MX_B + m, *pyr = PW + (YR + 4 * hf) * MX_B + m;
    const int tw = hf * TH + m * 8, tr = ((c16 >> 1) & 1) * TH + (4 * g4 + (c16 >> 2)) * 8 + 4 * (c16 & 1);
    auto batch = [&](const MxRec &r, int v0) {
        const bool ok = v0 + m < n;
        // the W weights of axis hf of visibility m (phi at distance z: see es_kernel)
        {
            const uint32_t q = hf ? r.c.yq : r.c.xq;
            const float zf = zoff + (float)(q & 0xFFFFFFu) * 5.9604644775390625e-08f;
#pragma unroll
            for (int k = 0; k < (KW > 0 ? KW : 8); ++k) {
                const float z = zf - (float)k; // exact, and |z| <= W / 2
                const float t = __builtin_fmaf(-z, z, hw2);
                const float s = __builtin_amdgcn_sqrtf(t);
                float w = __builtin_amdgcn_exp2f(__builtin_fmaf(__builtin_fmaf(-s, s, t), escw, __builtin_fmaf(esc, s, -esb)));
                if (KW == 0 && k >= W) w = 0.f; // (t may be negative)
                prow[k * MX_B] = w;
            }
        }
        wave_sync();
        // weights at the window's columns 8 hf + j, and at its rows 4 hf + j (j < 4) and
        // 4 hf + 4 + j (j >= 4): the rows this lane holds of Q
        float x[8], y[8];
        const float *px = pxr - (int)(r.c.xq >> 24) * MX_B, *py = pyr - (int)(r.c.yq >> 24) * MX_B;
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = px[j * MX_B];
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = py[(j < 4 ? j : j + 4) * MX_B];
        wave_sync(); // (the rows are rewritten by the next batch)
        f16x8 xh, xl, bh, bl;
        split_halves(x, m1, xh, xl);
        if (SPREAD) { // PX as the K = m operand
            *reinterpret_cast<f16x8 *>(TS + tw) = xh;
            *reinterpret_cast<f16x8 *>(TS + TB + tw) = xl;
            wave_sync();
            bh = column_operand(TS + tr);
            bl = column_operand(TS + TB + tr);
            wave_sync();
        }
        float wr;
        if (!NOGRID) {
            f32x16 d = {};
            d = __builtin_amdgcn_mfma_f32_32x32x16_f16(fl, xh, d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh, xl, d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh, xh, d, 0, 0, 0);
            float vr = 0.f, vi = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                vr += y[j] * d[j];
                vi += y[j] * d[8 + j];
            }
            // both halves' sums: the real part of V_m in lane (m, 0), the imaginary in (m, 1)
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(vr), __float_as_uint(vi), false, false);
            const float v = (__uint_as_float(p[0]) + __uint_as_float(p[1])) * vscale;
            if (MODE == MODE_FWD) {
                if (ok) caller_out[2 * (int64_t)(r.p < 0 ? ~r.p : r.p) + hf] = r.p < 0 && hf ? -v : v;
                return;
            }
            if (MODE == MODE_WFWD) {
                // planes run as successive launches and a record belongs to one work item: a
                // plain read-modify-write, in plane order
                if (ok) wacc[2 * (v0 + m) + hf] += r.w * v;
                return;
            }
            const float res = v - r.y;
            wr = ok ? r.w * res : 0.f;
            if (ok) jacc += r.w * (res * res); // halved at the end
            if (!SPREAD) return;
        } else if (MODE == MODE_ADJ) {
            const float yv = caller_in[2 * (int64_t)(r.p < 0 ? ~r.p : r.p) + hf];
            wr = ok ? r.w * (r.p < 0 && hf ? -yv : yv) : 0.f;
        } else {
            wr = ok ? r.w * r.y : 0.f;
        }
        if (__any(fabsf(wr) * rscale > MX_RMAX)) { // (uniform) lower the scale, and H with it
            const int nb = scale_bits(wave_max(fabsf(wr)), MX_RBITS), down = nb - rbits;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                hre[v] = ldexpf(hre[v], down);
                him[v] = ldexpf(him[v], down);
            }
            rbits = nb;
            rscale = exp2_int(nb);
        }
        wr *= rscale;
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(wr), __float_as_uint(wr), false, false);
        const float wre = __uint_as_float(s[0]), wim = __uint_as_float(s[1]);
#pragma unroll
        for (int comp = 0; comp < 2; ++comp) {
            float z[8];
            f16x8 zh, zl;
#pragma unroll
            for (int j = 0; j < 8; ++j) z[j] = (comp ? wim : wre) * y[j];
            split_halves(z, m1, zh, zl);
            *reinterpret_cast<f16x8 *>(TS + tw) = zh;
            *reinterpret_cast<f16x8 *>(TS + TB + tw) = zl;
            wave_sync();
            const f16x8 ah = column_operand(TS + tr), al = column_operand(TS + TB + tr);
            f32x4 &acc = comp ? him : hre;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bh, acc, 0, 0, 0);
            wave_sync(); // the table is rewritten
        }
    };
    wave_sync();
    for (int v0 = 0; v0 < n; v0 += 2 * MX_B) {
        fetch(rb, v0 + MX_B);
        batch(ra, v0);
        if (v0 + MX_B >= n) break;
        fetch(ra, v0 + 2 * MX_B);
        batch(rb, v0 + MX_B);
    }
    if (MODE == MODE_FWD || MODE == MODE_WFWD) return;
    if (SPREAD) {
        cpx *Sl = a.slots + (int64_t)wi.slot * g.win_stride; // column-major window
        // table position 8 h + j holds window row 4 h + j (j < 4) or 4 h + 4 + j
        const int r0 = 8 * (g4 & 1) + 4 * (g4 >> 1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = r0 + v;
            if (r < win && c16 < win)
                Sl[c16 * win + r] = cpx{ldexpf(hre[v], -rbits), ldexpf(him[v], -rbits)};
        }
    }
    if (DATA) {
        const double d = wave_sum(0.5 * (double)jacc);
        if (l == 0) a.jpart[wid] = d;
    }
}
#endif

// ----------------------------------------------------------------------- fold
// Two passes.  (1) k_ext_sum: the adjoint extended grid E = sum of every work item's
// window placed at its tile, computed owner-wise: the T x T cells starting at (vy T, vx T), those
// of the (virtual) tile (vy, vx), are reached only by the windows of tiles
// (vy - dy, vx - dx), dy, dx in {0, 1} (a window spans T + W - 1 <= 2T cells), and the window
// reads are contiguous along rows.  E overwrites the forward extended grid, which the gridding pass has consumed.
// (2) in the adjoint column pass, every half-plane cell sums the extended-grid cells that
// alias to it (periodic rows and columns) and is symmetrised, Hs = (H(t) + conj H(-t)) / 2,
// as it is loaded for the inverse column FFT.
constexpr int FOLD_LOADS = 8; // slot loads per thread in flight in k_ext_sum
constexpr int FOLD_COLS = 4;  // columns a thread sums together where every tile has one slot
constexpr int64_t FOLD_WAVES = 4096;

// A wave owns 64 consecutive rows of the columns of one virtual tile column (`cols` of them): the four
// tiles of a row's cells, their slots and flags are looked up once for all columns, and the stores
// are whole lines.  Where no tile of the wave has a second slot, FOLD_COLS columns are requested together.
// One thread per cell, tile by tile, spent its time on those lookups: 182 us a plane of the wide mosaic (36
// x 1036 x 520 cells), now 130; 100 for its bytes at the rate of a copy.
__global__ __launch_bounds__(NT) void k_ext_sum(Geom g, int cols, const int32_t *__restrict__ tslot,
                                                const cpx *__restrict__ slots, const uint8_t *__restrict__ sact,
                                                cpx *__restrict__ E) {
    const int item = blockIdx.y;
    const int T = g.T, win = g.win;
    const int chunks = (g.eh + 63) / 64, parts = (T + cols - 1) / cols;
    const int w = blockIdx.x * (NT / 64) + (threadIdx.x >> 6); // (chunk, part, tile column), chunk fastest
    const int vx = w / (chunks * parts), wp = w - vx * (chunks * parts), part = wp / chunks;
    if (vx > g.ntx) return; // (a whole wave)
    const int er = (wp - part * chunks) * 64 + (threadIdx.x & 63);
    const int vy = (int)(((float)er + 0.5f) / (float)T), r = er - vy * T;
    const int32_t *ts = tslot + (int64_t)item * (g.nty * g.ntx + 1);
    int lo[4], cnt[4];
    bool live[4], single = true; // live: the first slot is there and was written this pass
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ty = vy - (q >> 1), tx = vx - (q & 1);
        lo[q] = cnt[q] = 0;
        if (er < g.eh && r + (q >> 1) * T < win && ty >= 0 && tx >= 0 && ty < g.nty && tx < g.ntx) {
            lo[q] = ts[ty * g.ntx + tx];
            cnt[q] = ts[ty * g.ntx + tx + 1] - lo[q];
        }
        live[q] = cnt[q] > 0 && (!sact || sact[lo[q]]);
        single = single && cnt[q] <= 1;
    }
    const int c0 = part * cols, c1 = min(min(T, c0 + cols), g.ew - vx * T);
    cpx *Ec = E + (int64_t)item * g.ext_stride + (int64_t)(vx * T) * g.eh + er;
    if (__all(single)) {
        const cpx *at[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) at[q] = slots + (int64_t)lo[q] * g.win_stride + (q & 1) * T * win + r + (q >> 1) * T;
        for (int c = c0; c < c1; c += FOLD_COLS) {
            cpx h[FOLD_COLS][4];
#pragma unroll
            for (int u = 0; u < FOLD_COLS; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h[u][q] = cpx{0, 0};
                    if (live[q] && c + u < c1 && c + u + (q & 1) * T < win) h[u][q] = at[q][(c + u) * win];
                }
#pragma unroll
            for (int u = 0; u < FOLD_COLS; ++u) {
                real sr = real(0), si = real(0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    sr += h[u][q].re;
                    si += h[u][q].im;
                }
                if (c + u < c1 && er < g.eh) Ec[(int64_t)(c + u) * g.eh] = cpx{sr, si};
            }
        }
        return;
    }
    if (er >= g.eh) return;
    for (int c = c0; c < c1; ++c) {
        // the (quadrant, slot) terms of the cell in one list, quadrant-major: FOLD_LOADS of
        // them are loaded at a time and then added in list order (the order of a plain
        // quadrant-by-quadrant, slot-by-slot sum)
        int off[4], p[5];
        p[0] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int lc = c + (q & 1) * T;
            off[q] = lc * win + r + (q >> 1) * T;
            p[q + 1] = p[q] + (lc < win ? cnt[q] : 0);
        }
        real sr = real(0), si = real(0);
        for (int i0 = 0; i0 < p[4]; i0 += FOLD_LOADS) {
            cpx h[FOLD_LOADS];
            int sl[FOLD_LOADS], oo[FOLD_LOADS];
            bool on[FOLD_LOADS];
#pragma unroll
            for (int u = 0; u < FOLD_LOADS; ++u) {
                const int i = i0 + u;
                const int q = (i >= p[1]) + (i >= p[2]) + (i >= p[3]);
                const int pq = q == 0 ? p[0] : q == 1 ? p[1] : q == 2 ? p[2] : p[3];
                const int first = q == 0 ? lo[0] : q == 1 ? lo[1] : q == 2 ? lo[2] : lo[3];
                oo[u] = q == 0 ? off[0] : q == 1 ? off[1] : q == 2 ? off[2] : off[3];
                sl[u] = first + i - pq;
                on[u] = i < p[4];
            }
            // the flags and the windows of the batch are requested together (one memory latency
            // per batch, not two); a window that was not written this pass may hold anything and
            // is dropped by the select, never added
            uint8_t f[FOLD_LOADS];
#pragma unroll
            for (int u = 0; u < FOLD_LOADS; ++u) {
                f[u] = 1;
                if (on[u]) {
                    if (sact) f[u] = sact[sl[u]];
                    h[u] = slots[(int64_t)sl[u] * g.win_stride + oo[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < FOLD_LOADS; ++u) {
                if (on[u] && f[u]) {
                    sr += h[u].re;
                    si += h[u].im;
                }
            }
        }
        Ec[(int64_t)c * g.eh] = cpx{sr, si};
    }
}

__device__ __forceinline__ cpx alias_sum(const Geom &g, const cpx *__restrict__ Ei, int t1, int t2) {
    const int msk = g.nf - 1;
    real sr = real(0), si = real(0);
    for (int ec = (t2 + g.O) & msk; ec < g.ew; ec += g.nf)
        for (int er = (t1 + g.O) & msk; er < g.eh; er += g.nf) {
            const cpx h = Ei[(int64_t)ec * g.eh + er];
            sr += h.re;
            si += h.im;
        }
    return cpx{sr, si};
}

// alias_sum for grids whose extended rows stop below 2 n_f and columns below n_f: the cell's
// column exists at most once and its row at most twice.  alias_pair loads the (up to) two
// values; pair_sum adds them in alias_sum's order (starting from zero, so a lone -0 reads
// as +0 there as well).
__device__ __forceinline__ void alias_pair(const Geom &g, const cpx *__restrict__ Ei, int t1, int t2, cpx &a,
                                           cpx &b) {
    const int msk = g.nf - 1;
    const int ec = (t2 + g.O) & msk, er = (t1 + g.O) & msk;
    if (ec < g.ew) {
        const cpx *col = Ei + (int64_t)ec * g.eh;
        if (er < g.eh) a = col[er];
        if (er + g.nf < g.eh) b = col[er + g.nf];
    }
}

__device__ __forceinline__ cpx pair_sum(const Geom &g, int t1, int t2, cpx a, cpx b) {
    const int msk = g.nf - 1;
    const int ec = (t2 + g.O) & msk, er = (t1 + g.O) & msk;
    real sr = real(0), si = real(0);
    if (ec < g.ew) {
        if (er < g.eh) { sr += a.re; si += a.im; }
        if (er + g.nf < g.eh) { sr += b.re; si += b.im; }
    }
    return cpx{sr, si};
}

// ------------------------------------------------------------ adjoint column pass
template <int LOGN, int CB>
__global__ __launch_bounds__(NT) void k_col_inv(Geom g, const cpx *__restrict__ E,
                                                const cpx *__restrict__ tw, cpx *__restrict__ R) {
    constexpr int N = 1 << LOGN;
    using F = ColFft<LOGN, CB>;
    __shared__ cpx buf[F::LEN];
    __shared__ cpx tws[tw_len<LOGN>()];
    TwStage<LOGN> twr;
    twr.fetch(tw);
    const int tid = threadIdx.x;
    int item, c0;
    if (!col_block<CB>(g, item, c0)) return;
    const cpx *Ei = E + (int64_t)item * g.ext_stride;
    if (g.eh <= 2 * g.nf && g.ew <= g.nf) {
        // every cell has at most two aliases (rows t and t + n_f of one column): the loads of
        // COL_LOADS cells are issued together, then summed in the order of alias_sum
        for (int e0 = tid; e0 < N * CB; e0 += COL_LOADS * NT) {
            cpx h0[COL_LOADS], h1[COL_LOADS], m0[COL_LOADS], m1[COL_LOADS];
#pragma unroll
            for (int u = 0; u < COL_LOADS; ++u) {
                const int e = e0 + u * NT, cc = e >> LOGN, t1 = e & (N - 1), t2 = c0 + cc;
                h0[u] = h1[u] = m0[u] = m1[u] = cpx{0, 0};
                if (e < N * CB && t2 < g.rw) {
                    alias_pair(g, Ei, t1, t2, h0[u], h1[u]);
                    alias_pair(g, Ei, (N - t1) & (N - 1), (N - t2) & (N - 1), m0[u], m1[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < COL_LOADS; ++u) {
                const int e = e0 + u * NT, cc = e >> LOGN, t1 = e & (N - 1), t2 = c0 + cc;
                if (e >= N * CB) break;
                cpx v = cpx{0, 0};
                if (t2 < g.rw) {
                    const cpx h = pair_sum(g, t1, t2, h0[u], h1[u]);
                    const cpx m = pair_sum(g, (N - t1) & (N - 1), (N - t2) & (N - 1), m0[u], m1[u]);
                    v = cpx{real(0.5) * (h.re + m.re), real(0.5) * (h.im - m.im)};
                }
                buf[F::at(t1, cc)] = v;
            }
        }
    } else {
        for (int e = tid; e < N * CB; e += NT) {
            const int cc = e >> LOGN, t1 = e & (N - 1);
            const int t2 = c0 + cc;
            cpx v = cpx{0, 0};
            if (t2 < g.rw) {
                const cpx h = alias_sum(g, Ei, t1, t2);
                const cpx m = alias_sum(g, Ei, (N - t1) & (N - 1), (N - t2) & (N - 1));
                v = cpx{real(0.5) * (h.re + m.re), real(0.5) * (h.im - m.im)};
            }
            buf[F::at(t1, cc)] = v;
        }
    }
    twr.store(tws);
    __syncthreads();
    F::inverse(buf, tws);
    cpx *Ri = R + (int64_t)item * g.r_stride;
    const int nk = g.nk;
    for (int e = tid; e < nk * CB; e += NT) {
        const int a = e / CB, cc = e - (e / CB) * CB;
        if (c0 + cc < g.rw) Ri[(int64_t)a * g.rw + c0 + cc] = buf[F::at((a - nk / 2) & (N - 1), cc)];
    }
}

// ------------------------------------------- adjoint column pass straight from the slots
// k_ext_sum followed by k_col_inv without the extended grid in between: the block of a column
// group forms every extended cell its columns need from the slots that cover it (quadrant by
// quadrant, slot by slot, as k_ext_sum adds them), adds the second row alias and the
// Hermitian mirror in the order of k_col_inv, and runs the inverse column FFT.  The slot
// columns of a cell's tile are read by the one block that owns the cell's column, as whole
// 8-byte-per-row runs, instead of being written to and read back from the extended grid.
// Valid when every cell has at most two row aliases and one column alias (eh <= 2 n_f,
// ew <= n_f); the launcher falls back to the two-kernel path otherwise.

// Slot range and in-window offset of quadrant q of extended cell (er, ec): the window of tile
// (er / T - (q >> 1), ec / T - (q & 1)) covers the cell when the offset stays in the window.
__device__ __forceinline__ void cell_quadrant(const Geom &g, const int32_t *__restrict__ ts, int er, int ec, int q,
                                              int &lo, int &cnt, int &off) {
    const int vy = er / g.T, vx = ec / g.T;
    const int r = er - vy * g.T, c = ec - vx * g.T;
    const int ty = vy - (q >> 1), tx = vx - (q & 1);
    const int lr = r + (q >> 1) * g.T, lc = c + (q & 1) * g.T;
    lo = 0;
    cnt = 0;
    off = lc * g.win + lr;
    if (ty >= 0 && tx >= 0 && ty < g.nty && tx < g.ntx && lr < g.win && lc < g.win) {
        lo = ts[ty * g.ntx + tx];
        cnt = ts[ty * g.ntx + tx + 1] - lo;
    }
}

// Extended cell (er, ec) summed from the slots, in k_ext_sum's order (cells outside the
// extended grid are 0).
__device__ __forceinline__ cpx ext_cell(const Geom &g, const int32_t *__restrict__ ts, const cpx *__restrict__ slots,
                                        int er, int ec) {
    real sr = real(0), si = real(0);
    if (er >= g.eh || ec >= g.ew) return cpx{sr, si};
    for (int q = 0; q < 4; ++q) {
        int lo, cnt, off;
        cell_quadrant(g, ts, er, ec, q, lo, cnt, off);
        for (int k = 0; k < cnt; ++k) {
            const cpx h = slots[(int64_t)(lo + k) * g.win_stride + off];
            sr += h.re;
            si += h.im;
        }
    }
    return cpx{sr, si};
}

// alias_pair + pair_sum of k_col_inv with the cells formed from the slots.
__device__ __forceinline__ cpx alias_from_slots(const Geom &g, const int32_t *__restrict__ ts,
                                                const cpx *__restrict__ slots, int t1, int t2) {
    const int msk = g.nf - 1;
    const int ec = (t2 + g.O) & msk, er = (t1 + g.O) & msk;
    real sr = real(0), si = real(0);
    if (ec < g.ew) {
        if (er < g.eh) {
            const cpx a = ext_cell(g, ts, slots, er, ec);
            sr += a.re;
            si += a.im;
        }
        if (er + g.nf < g.eh) {
            const cpx b = ext_cell(g, ts, slots, er + g.nf, ec);
            sr += b.re;
            si += b.im;
        }
    }
    return cpx{sr, si};
}

// Cells per thread whose slot loads are in flight together, and columns per block of the fused
// pass: two and two measured fastest on the spectral cube (four cells per thread, or wider
// blocks, cost registers or LDS and with them the loads in flight per compute unit).
#ifndef IVX_FOLD_CELLS
#define IVX_FOLD_CELLS 2
#endif
#ifndef IVX_FOLD_CB
#define IVX_FOLD_CB 2
#endif
constexpr int FOLD_CELLS = IVX_FOLD_CELLS;

template <int LOGN, int CB>
__global__ __launch_bounds__(NT) void k_col_inv_slots(Geom g, const int32_t *__restrict__ tslot,
                                                      const cpx *__restrict__ slots, const cpx *__restrict__ tw,
                                                      cpx *__restrict__ R) {
    constexpr int N = 1 << LOGN;
    using F = Fft<LOGN, CB, false>;
    // tile rows of the grid: (n_f + O) / T + 1 with T >= 4 and O <= 8
    constexpr int MAXROWS = (N + 8) / 4 + 2;
    __shared__ cpx buf[F::LEN];
    __shared__ cpx tws[tw_len<LOGN>()];
    // slot-list prefix of tile columns vxa - 1 .. vxa + 2 in every tile row: the tiles whose
    // windows reach this block's columns (CB <= T consecutive columns lie in at most two
    // tile columns)
    __shared__ int rng[MAXROWS + 1][4]; // + a sink row for the stores of entries past the end
    TwStage<LOGN> twr;
    twr.fetch(tw);
    const int tid = threadIdx.x;
    int item, c0;
    if (!col_block<CB>(g, item, c0)) return;
    const int32_t *ts = tslot + (int64_t)item * (g.nty * g.ntx + 1);
    const int msk = N - 1;
    const int vxa = (c0 + g.O) / g.T;
    // the prefix entries, RNG_U per thread requested together (loads clamped to entry 0,
    // stores past the end into the sink row; a guarded load would wait for the previous one)
    constexpr int RNG_U = 2;
    for (int e0 = tid; e0 < g.nty * 4; e0 += RNG_U * NT) {
        int32_t pv[RNG_U];
#pragma unroll
        for (int u = 0; u < RNG_U; ++u) {
            const int e = e0 + u * NT, ty = e >> 2, tx = vxa - 1 + (e & 3);
            const bool ok = e < g.nty * 4 && tx >= 0 && tx <= g.ntx;
            pv[u] = ts[ok ? ty * g.ntx + tx : 0];
        }
#pragma unroll
        for (int u = 0; u < RNG_U; ++u) {
            const int e = e0 + u * NT, ty = e >> 2, tx = vxa - 1 + (e & 3);
            const bool ok = e < g.nty * 4 && tx >= 0 && tx <= g.ntx;
            rng[e < g.nty * 4 ? ty : MAXROWS][e & 3] = ok ? pv[u] : 0;
        }
    }
    // the item's first slot (a valid address for the loads of empty quadrants), if it has any
    const int32_t s_first = ts[0];
    const bool any_slot = ts[g.nty * g.ntx] > s_first;
    __syncthreads();
    const float inv_t = 1.0f / (float)g.T;
    for (int e0 = tid; e0 < N * CB; e0 += FOLD_CELLS * NT) {
        // the quadrant lists of FOLD_CELLS cells (first row alias) from the LDS table, then
        // the first slot of every quadrant of every cell requested together, then the sums in
        // k_ext_sum's order
        int lo[FOLD_CELLS][4], cnt[FOLD_CELLS][4], off[FOLD_CELLS][4];
        cpx first[FOLD_CELLS][4];
#pragma unroll
        for (int u = 0; u < FOLD_CELLS; ++u) {
            const int e = e0 + u * NT, cc = e >> LOGN, t1 = e & msk, t2 = c0 + cc;
            const int er = (t1 + g.O) & msk, ec = (t2 + g.O) & msk;
            const bool live = e < N * CB && t2 < g.rw && er < g.eh && ec < g.ew;
            const int vy = (int)(((float)er + 0.5f) * inv_t), vx = (int)(((float)ec + 0.5f) * inv_t);
            const int r = er - vy * g.T, c = ec - vx * g.T;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ty = vy - (q >> 1), tx = vx - (q & 1);
                const int lr = r + (q >> 1) * g.T, lc = c + (q & 1) * g.T;
                const int j = tx - (vxa - 1);
                lo[u][q] = 0;
                cnt[u][q] = 0;
                off[u][q] = lc * g.win + lr;
                if (live && ty >= 0 && tx >= 0 && ty < g.nty && tx < g.ntx && lr < g.win && lc < g.win) {
                    lo[u][q] = rng[ty][j];
                    cnt[u][q] = rng[ty][j + 1] - lo[u][q];
                }
            }
        }
        // every load unconditional (an empty quadrant reads the item's first slot and scales it
        // by 0; a select would be turned back into a branch around the load): a load behind a
        // branch waits for its own round trip before the next is issued
        if (any_slot) {
#pragma unroll
            for (int u = 0; u < FOLD_CELLS; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool on = cnt[u][q] > 0;
                    const int64_t at = on ? (int64_t)lo[u][q] * g.win_stride + off[u][q] : (int64_t)s_first * g.win_stride;
                    const cpx h = slots[at];
                    const real keep = on ? real(1) : real(0);
                    first[u][q] = cpx{h.re * keep, h.im * keep};
                }
        } else {
#pragma unroll
            for (int u = 0; u < FOLD_CELLS; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) first[u][q] = cpx{0, 0};
        }
#pragma unroll
        for (int u = 0; u < FOLD_CELLS; ++u) {
            const int e = e0 + u * NT, cc = e >> LOGN, t1 = e & msk, t2 = c0 + cc;
            if (e >= N * CB) break;
            cpx v = cpx{0, 0};
            if (t2 < g.rw) {
                // extended cell of the first row alias
                real ar = real(0), ai = real(0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (cnt[u][q] > 0) {
                        ar += first[u][q].re;
                        ai += first[u][q].im;
                        for (int k = 1; k < cnt[u][q]; ++k) {
                            const cpx h = slots[(int64_t)(lo[u][q] + k) * g.win_stride + off[u][q]];
                            ar += h.re;
                            ai += h.im;
                        }
                    }
                }
                // pair_sum: the first alias (present when inside the grid), then the second
                const int er = (t1 + g.O) & msk, ec = (t2 + g.O) & msk;
                real hr = real(0), hi = real(0);
                if (ec < g.ew) {
                    if (er < g.eh) {
                        hr += ar;
                        hi += ai;
                    }
                    if (er + g.nf < g.eh) {
                        const cpx b = ext_cell(g, ts, slots, er + g.nf, ec);
                        hr += b.re;
                        hi += b.im;
                    }
                }
                // the Hermitian mirror: extended columns outside this block's tile columns, only
                // near t2 = 0 and t2 = n_f / 2
                const cpx m = alias_from_slots(g, ts, slots, (N - t1) & msk, (N - t2) & msk);
                v = cpx{real(0.5) * (hr + m.re), real(0.5) * (hi - m.im)};
            }
            buf[F::at(t1, cc)] = v;
        }
    }
    twr.store(tws);
    __syncthreads();
    F::inverse(buf, tws);
    cpx *Ri = R + (int64_t)item * g.r_stride;
    const int nk = g.nk;
    for (int e = tid; e < nk * CB; e += NT) {
        const int a = e / CB, cc = e - (e / CB) * CB;
        if (c0 + cc < g.rw) Ri[(int64_t)a * g.rw + c0 + cc] = buf[F::at((a - nk / 2) & (N - 1), cc)];
    }
}

// --------------------------------------------------------------- adjoint row pass
template <int LOGN>
__global__ __launch_bounds__(NT) void k_row_inv(Geom g, const cpx *__restrict__ R,
                                                const real *__restrict__ beams,
                                                const real *__restrict__ fscale,
                                                const real *__restrict__ dq,
                                                const cpx *__restrict__ tw, real *__restrict__ gp) {
    constexpr int N = 1 << LOGN;
    using F = RowFft<LOGN>;
    __shared__ cpx buf[N];
    __shared__ cpx tws[tw_len<LOGN>()];
    TwStage<LOGN> twr;
    twr.fetch(tw);
    const int tid = threadIdx.x;
    const int item = blockIdx.y;
    const int k = item / g.C, c = item - (item / g.C) * g.C;
    const int a0 = 2 * blockIdx.x;
    const int nk = g.nk;
    const cpx *X = R + (int64_t)item * g.r_stride + (int64_t)a0 * g.rw;
    const cpx *Y = X + g.rw;
    for (int k0 = tid; k0 < N; k0 += COL_LOADS * NT) {
        cpx xv[COL_LOADS], yv[COL_LOADS];
#pragma unroll
        for (int u = 0; u < COL_LOADS; ++u) {
            const int kk = k0 + u * NT;
            if (kk < N) {
                const int src = kk <= N / 2 ? kk : N - kk;
                xv[u] = X[src];
                yv[u] = Y[src];
            }
        }
#pragma unroll
        for (int u = 0; u < COL_LOADS; ++u) {
            const int kk = k0 + u * NT;
            if (kk >= N) break;
            cpx x = xv[u], y = yv[u];
            if (kk <= N / 2) {
                if (kk == 0 || kk == N / 2) { x.im = real(0); y.im = real(0); }
            } else {
                x.im = -x.im;
                y.im = -y.im;
            }
            buf[F::at(kk)] = cpx{x.re - y.im, x.im + y.re}; // x + i y
        }
    }
    twr.store(tws);
    __syncthreads();
    F::inverse(buf, tws);
    const real *A = beams + (int64_t)k * nk * nk;
    real *out = gp + (int64_t)item * nk * nk;
    const real s = fscale[c];
    const real q0 = s * dq[a0], q1 = s * dq[a0 + 1];
    for (int b = tid; b < nk; b += NT) {
        const cpx z = buf[F::at((b - nk / 2) & (N - 1))];
        const int64_t e0 = (int64_t)a0 * nk + b;
        out[e0] = q0 * dq[b] * A[e0] * z.re;
        out[e0 + nk] = q1 * dq[b] * A[e0 + nk] * z.im;
    }
}

// ------------------------------------------------------------------- single dish
__device__ __forceinline__ int floordiv(int a, int b) { return (a >= 0) ? a / b : -((-a + b - 1) / b); }
__device__ __forceinline__ int ceildiv(int a, int b) { return -floordiv(-a, b); }

// The beam sums split their taps over SD_ROW_P lanes (rows) and SD_COL_P (columns), SD_LOADS in flight
// each: one thread per output was a chain of some 130 loads on 4 and 57 blocks, 28.6 and 16.5 us at 30^2
// samples of a 480^2 sky and 35 and 19 at 64^2 of 1024^2, now 3.4, 3.7 and 5.2, 6.1.
// Maps of every pixel that fill the chip with one lane an output (SD_FULL of them) keep that: neighbouring lanes read
// neighbouring pixels then (512^2 of them 13 us, 15.2 split).  Launches are bounded and blocks run over the rest of
// the outputs: the work items of a launch do not limit the size of a map.  (Columns on a sixteenth of these blocks took
// 26.8 us at 512^2 instead of 22.)
constexpr int SD_ROW_P = 8, SD_COL_P = 16, SD_LOADS = 8;
constexpr int64_t SD_FULL = 1 << 18, SD_ROW_BLOCKS = 1 << 16, SD_COL_BLOCKS = 1 << 14;

// sum over t = lo + part, lo + part + P, ... <= hi of gB[t + rb] v[t vs]
template <int P> __device__ __forceinline__ real sd_taps(const real *__restrict__ gB, int rb, const real *__restrict__ v,
                                                         int64_t vs, int lo, int hi, int part) {
    real s = real(0);
    for (int t0 = lo + part; t0 <= hi; t0 += P * SD_LOADS) {
        real w[SD_LOADS], x[SD_LOADS];
#pragma unroll
        for (int u = 0; u < SD_LOADS; ++u) {
            const int t = min(t0 + u * P, hi);
            w[u] = gB[t + rb];
            x[u] = v[t * vs];
        }
#pragma unroll
        for (int u = 0; u < SD_LOADS; ++u) s = t0 + u * P <= hi ? s + w[u] * x[u] : s;
    }
    return s;
}

// U[c][i][q] = sum_j g(o + q S - j) x[c][i][j]   (beam along columns, sampled columns)
template <int P>
__global__ __launch_bounds__(NT) void k_sd_rows(Geom g, const real *__restrict__ sky,
                                                const real *__restrict__ gB, int rb, int sd_n,
                                                int stride, int offset, real *__restrict__ U) {
    const int64_t tot = (int64_t)g.C * g.N * sd_n;
    for (int64_t idx = (int64_t)blockIdx.x * (NT / P) + threadIdx.x / P; idx < tot; idx += (int64_t)gridDim.x * (NT / P)) {
        const int q = (int)(idx % sd_n);
        const int64_t ci = idx / sd_n; // c * N + i
        const int cen = offset + q * stride;
        const int lo = cen - rb < 0 ? -cen : -rb;
        const int hi = cen + rb >= g.N ? g.N - 1 - cen : rb;
        real s = sd_taps<P>(gB, rb, sky + ci * g.N + cen, 1, lo, hi, threadIdx.x % P);
#pragma unroll
        for (int m = P / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64); // (a group of lanes has one idx)
        if (threadIdx.x % P == 0) U[idx] = s;
    }
}

// T~[c][p][q] = sum_i g(o + p S - i) U[c][i][q];  E = (T~ - T)/sigma^2;  K partials
// (neighbouring lanes take neighbouring q, 16 of them a block)
__global__ __launch_bounds__(NT) void k_sd_cols(Geom g, const real *__restrict__ U,
                                                const real *__restrict__ gB, int rb, int sd_n,
                                                int stride, int offset, const real *__restrict__ sdmap,
                                                real inv_var, real *__restrict__ E, double *__restrict__ kpart) {
    constexpr int PER = NT / SD_COL_P;
    __shared__ real sums[NT];
    const int64_t tot = (int64_t)g.C * sd_n * sd_n;
    double kk = 0.0;
    for (int64_t first = (int64_t)blockIdx.x * PER; first < tot; first += (int64_t)gridDim.x * PER) { // (uniform)
        const int64_t idx = first + threadIdx.x % PER;
        real s = real(0);
        if (idx < tot) {
            const int q = (int)(idx % sd_n);
            const int p = (int)((idx / sd_n) % sd_n);
            const int c = (int)(idx / ((int64_t)sd_n * sd_n));
            const int cen = offset + p * stride;
            const int lo = cen - rb < 0 ? -cen : -rb;
            const int hi = cen + rb >= g.N ? g.N - 1 - cen : rb;
            s = sd_taps<SD_COL_P>(gB, rb, U + ((int64_t)c * g.N + cen) * sd_n + q, sd_n, lo, hi, threadIdx.x / PER);
        }
        sums[threadIdx.x] = s;
        __syncthreads();
        if (threadIdx.x < PER && idx < tot) {
            real v = real(0);
#pragma unroll
            for (int part = 0; part < SD_COL_P; ++part) v += sums[part * PER + threadIdx.x];
            const real res = v - sdmap[idx];
            E[idx] = res * inv_var;
            kk += 0.5 * (double)res * (double)res * (double)inv_var;
        }
        __syncthreads(); // (the sums are rewritten)
    }
    if (threadIdx.x >= 64) return;
    for (int m = PER / 2; m >= 1; m >>= 1) kk += __shfl_xor(kk, m, 64);
    if (threadIdx.x == 0) kpart[blockIdx.x] = kk;
}

// V[c][p][j] = sum_q g(o + q S - j) E[c][p][q]: the column half of B^T S^T E, so that the
// sky pass needs only the row sum over the few p whose beam reaches row i
__global__ __launch_bounds__(NT) void k_sd_back(Geom g, const real *__restrict__ E, const real *__restrict__ gB,
                                                int rb, int sd_n, int stride, int offset, real *__restrict__ V) {
    const int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t tot = (int64_t)g.C * sd_n * g.N;
    if (idx >= tot) return;
    const int j = (int)(idx % g.N);
    const int64_t cp = idx / g.N; // c * sd_n + p
    const int q0 = max(0, ceildiv(j - rb - offset, stride)), q1 = min(sd_n - 1, floordiv(j + rb - offset, stride));
    const real *Ep = E + cp * sd_n;
    real s = real(0);
    for (int q = q0; q <= q1; ++q) s += gB[offset + q * stride - j + rb] * Ep[q];
    V[idx] = s;
}

// --------------------------------------------------------------------- sky level
static_assert(SKY_T * SKY_T == NT, "one thread per pixel of a sky block");

struct SkyArgs {
    Geom g;
    const real *sky;
    const real *gp;
    const int32_t *cptr;
    const CsrEnt *cent;
    real lambda_r, lambda_s;
    const real *E;
    const real *gB;
    int rb, sd_n, stride, offset;
    real *grad;
    double *rpart;
    int mode;   // SkyMode
    real scale; // gradient multiplier
    real lambda_nu;
    double *npart;
};

constexpr int SKY_LOADS = 8; // CSR entries per lane in flight in k_sky

__global__ __launch_bounds__(NT) void k_sky(SkyArgs a) {
    __shared__ real xs[SKY_T + 4][SKY_T + 5];
    __shared__ real dxs[SKY_T + 2][SKY_T + 3];
    __shared__ double red[NT / 64];
    const Geom &g = a.g;
    const int N = g.N;
    // XCD-aware block order (as col_block) on cubes: each XCD takes a contiguous band of
    // (channel, tile row, tile column) triples, so neighbouring tiles, whose CSR entries
    // gather from the same lines of g', share an L2.  With few channels a band is a strip
    // of one image whose pointing overlap (and so CSR length) varies, which unbalances the
    // XCDs: the launch order is kept there.
    const int nb = (N + SKY_T - 1) / SKY_T;
    const int64_t total = (int64_t)nb * nb * g.C, per = (total + 7) / 8;
    const int64_t bw = g.C >= 8 ? (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3) : (int64_t)blockIdx.x;
    if (bw >= total) return;
    const int bx = (int)(bw % nb), by = (int)((bw / nb) % nb);
    const int c = (int)(bw / ((int64_t)nb * nb));
    const int i0 = by * SKY_T, j0 = bx * SKY_T;
    const int tid = threadIdx.x;
    const int ti = tid / SKY_T, tj = tid - (tid / SKY_T) * SKY_T;
    const real *x = a.sky + (int64_t)c * N * N;
    const bool adjoint_only = a.mode == SKY_ADJOINT, value_only = a.mode == SKY_VALUE;
    const bool reg = (a.lambda_r != real(0)) && !adjoint_only;
    const bool sd = (a.lambda_s != real(0)) && (a.sd_n > 0) && !adjoint_only && !value_only;
    const bool spec = (a.lambda_nu != real(0)) && !adjoint_only && g.C > 1;
    double nloc = 0.0;
    double rloc = 0.0;
    if (reg) {
        for (int e = tid; e < (SKY_T + 4) * (SKY_T + 4); e += NT) {
            const int r = e / (SKY_T + 4), cc = e - (e / (SKY_T + 4)) * (SKY_T + 4);
            const int gi = i0 - 2 + r, gj = j0 - 2 + cc;
            xs[r][cc] = (gi >= 0 && gi < N && gj >= 0 && gj < N) ? x[(int64_t)gi * N + gj] : real(0);
        }
        __syncthreads();
        for (int e = tid; e < (SKY_T + 2) * (SKY_T + 2); e += NT) {
            const int r = e / (SKY_T + 2), cc = e - (e / (SKY_T + 2)) * (SKY_T + 2);
            const int gi = i0 - 1 + r, gj = j0 - 1 + cc;
            real d = real(0);
            if (gi >= 0 && gi < N && gj >= 0 && gj < N)
                d = real(4) * xs[r + 1][cc + 1] - xs[r][cc + 1] - xs[r + 2][cc + 1] - xs[r + 1][cc] - xs[r + 1][cc + 2];
            dxs[r][cc] = d;
        }
        __syncthreads();
    }
    const int i = i0 + ti, j = j0 + tj;
    // spectral term: this pixel in the neighbouring channels
    real xc = real(0), xm = real(0), xp = real(0);
    if (spec && i < N && j < N) {
        const int64_t pix = (int64_t)i * N + j, cs = (int64_t)N * N;
        xc = x[pix];
        if (c > 0) xm = x[pix - cs];
        if (c + 1 < g.C) {
            xp = x[pix + cs];
            const real d = xp - xc;
            nloc = 0.5 * (double)d * (double)d;
        }
    }
    if (value_only) {
        if (reg && i < N && j < N) {
            const real d = dxs[ti + 1][tj + 1];
            rloc = 0.5 * (double)d * (double)d;
        }
    } else if (i < N && j < N) {
        real gsum = real(0);
        const int64_t p = (int64_t)i * N + j;
        const int64_t coff = (int64_t)c * g.nk * g.nk;
        (void)p;
        // this wave's slice: entries lane-contiguous, padded with zero weights
        const int slice = (by * nb + bx) * (NT / 64) + (tid >> 6);
        const int e0 = a.cptr[slice], len = (a.cptr[slice + 1] - e0) >> 6;
        const CsrEnt *en = a.cent + e0 + (tid & 63);
        // SKY_LOADS entries, then their SKY_LOADS gathers, are requested before the first is
        // used; the products are added in entry order
        for (int t0 = 0; t0 < len; t0 += SKY_LOADS) {
            CsrEnt q[SKY_LOADS];
            real v[SKY_LOADS];
#pragma unroll
            for (int u = 0; u < SKY_LOADS; ++u)
                if (t0 + u < len) q[u] = en[(t0 + u) * 64];
#pragma unroll
            for (int u = 0; u < SKY_LOADS; ++u)
                if (t0 + u < len) v[u] = a.gp[(int64_t)q[u].off + coff];
#pragma unroll
            for (int u = 0; u < SKY_LOADS; ++u)
                if (t0 + u < len) gsum += q[u].w * v[u];
        }
        if (reg) {
            const real d = dxs[ti + 1][tj + 1];
            gsum += a.lambda_r * (real(4) * d - dxs[ti][tj + 1] - dxs[ti + 2][tj + 1] - dxs[ti + 1][tj] - dxs[ti + 1][tj + 2]);
            rloc = 0.5 * (double)d * (double)d;
        }
        if (sd) {
            const int S = a.stride, o = a.offset, rb = a.rb;
            const int p0 = max(0, ceildiv(i - rb - o, S)), p1 = min(a.sd_n - 1, floordiv(i + rb - o, S));
            const real *Vc = a.E + (int64_t)c * a.sd_n * N; // V of k_sd_back
            real s = real(0);
            for (int pp = p0; pp <= p1; ++pp) s += a.gB[o + pp * S - i + rb] * Vc[(int64_t)pp * N + j];
            gsum += a.lambda_s * s;
        }
        if (spec) {
            real ds = real(0);
            if (c > 0) ds += xc - xm;
            if (c + 1 < g.C) ds -= xp - xc;
            gsum += a.lambda_nu * ds;
        }
        a.grad[(int64_t)c * N * N + p] = a.scale == real(1) ? gsum : a.scale * gsum;
    }
    if (!adjoint_only) {
        for (int m = 32; m >= 1; m >>= 1) rloc += __shfl_xor(rloc, m, 64);
        if ((tid & 63) == 0) red[tid >> 6] = rloc;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < NT / 64; ++w) s += red[w];
            a.rpart[bw] = s;
        }
        if (spec) {
            __syncthreads(); // red is reused
            for (int m = 32; m >= 1; m >>= 1) nloc += __shfl_xor(nloc, m, 64);
            if ((tid & 63) == 0) red[tid >> 6] = nloc;
            __syncthreads();
            if (tid == 0) {
                double s = 0.0;
                for (int w = 0; w < NT / 64; ++w) s += red[w];
                a.npart[bw] = s;
            }
        }
    }
}

// ---------------------------------------------------------------------- reductions
// out[b] = sum of in[b * per .. (b + 1) * per) (fixed order: strided per thread, then tree)
__global__ __launch_bounds__(NT) void k_partial_sums(const double *__restrict__ in, int n, int per,
                                                     double *__restrict__ out) {
    __shared__ double red[NT / 64];
    const int b0 = blockIdx.x * per, b1 = min(n, b0 + per);
    double v = 0.0;
    int i = b0 + threadIdx.x;
    for (; i + 7 * NT < b1; i += 8 * NT) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = in[i + u * NT];
#pragma unroll
        for (int u = 0; u < 8; ++u) v += t[u];
    }
    for (; i < b1; i += NT) v += in[i];
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w) s += red[w];
        out[blockIdx.x] = s;
    }
}

constexpr int NT_FINAL = 1024;
constexpr int FINAL_PER = 1024; // work-item partials per pre-reduction block
__global__ __launch_bounds__(NT_FINAL) void k_final(const double *__restrict__ jpart, int nj,
                                                    const double *__restrict__ rpart, int nr,
                                                    const double *__restrict__ kpart, int nkp,
                                                    const double *__restrict__ npart, int nnp,
                                                    double lambda_r, double lambda_s, double lambda_nu,
                                                    double *terms, double *terms_user) {
    __shared__ double sh[4][NT_FINAL / 64];
    const int tid = threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    // each thread sums its strided entries in index order; 8 loads are issued before they
    // are added, so their latencies overlap instead of chaining
    auto strided_sum = [&](const double *__restrict__ p, int n, double &acc) {
        int i = tid;
        for (; i + 7 * NT_FINAL < n; i += 8 * NT_FINAL) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = p[i + u * NT_FINAL];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += t[u];
        }
        for (; i < n; i += NT_FINAL) acc += p[i];
    };
    strided_sum(jpart, nj, v[0]);
    strided_sum(rpart, nr, v[1]);
    strided_sum(kpart, nkp, v[2]);
    strided_sum(npart, nnp, v[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int m = 32; m >= 1; m >>= 1) v[q] += __shfl_xor(v[q], m, 64);
        if ((tid & 63) == 0) sh[q][tid >> 6] = v[q];
    }
    __syncthreads();
    if (tid == 0) {
        double Q = 0.0, R = 0.0, K = 0.0, Nu = 0.0;
        for (int w = 0; w < NT_FINAL / 64; ++w) {
            Q += sh[0][w];
            R += sh[1][w];
            K += sh[2][w];
            Nu += sh[3][w];
        }
        double qt = Q + lambda_s * K + lambda_r * R;
        if (lambda_nu != 0.0) qt += lambda_nu * Nu;
        const double t5[5] = {qt, Q, K, R, Nu};
        for (int q = 0; q < 5; ++q) terms[q] = t5[q];
        if (terms_user)
            for (int q = 0; q < 4; ++q) terms_user[q] = t5[q];
    }
}

__global__ __launch_bounds__(NT) void k_zero(uint32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) p[i] = 0u;
}

// ------------------------------------------------------------------------ feathering
// App. B: out = F^-1[B F[sd] + (1 - B) F[int]] = int + F^-1[B F[sd - int]] (B real and even),
// per channel of n x n maps: a real row FFT of the difference (two rows packed in one complex
// transform, half spectrum kept), a column FFT, the Gaussian transfer function
// B(k) = exp(-2 pi^2 sigma^2 |k|^2), the inverse column FFT, and the inverse row FFT, added to
// the interferometric map with the 1 / n^2 of the unscaled transform pair.  Work: the
// half-spectra [C][n][n/2 + 1] complex.  Twiddles are formed in LDS from FP64 sincospi.
template <int LOGN> __device__ __forceinline__ void tw_fill(cpx *tws) {
    constexpr int N = 1 << LOGN;
    for (int t = threadIdx.x; t < tw_len<LOGN>(); t += NT) {
        double sv, cv;
        sincospi(-2.0 * (double)t / (double)N, &sv, &cv);
        tws[t] = cpx{(real)cv, (real)sv};
    }
}

template <int LOGN>
__global__ __launch_bounds__(NT) void k_feather_rows(const real *__restrict__ interf, const real *__restrict__ sd,
                                                     cpx *__restrict__ work) {
    constexpr int N = 1 << LOGN, RW = N / 2 + 1;
    using F = RowFft<LOGN>;
    __shared__ cpx buf[N];
    __shared__ cpx tws[tw_len<LOGN>()];
    const int c = blockIdx.y, a0 = 2 * blockIdx.x;
    const int64_t base = ((int64_t)c * N + a0) * N;
    for (int b = threadIdx.x; b < N; b += NT)
        buf[F::at(b)] = cpx{sd[base + b] - interf[base + b], sd[base + N + b] - interf[base + N + b]};
    tw_fill<LOGN>(tws);
    __syncthreads();
    F::forward(buf, tws);
    cpx *W0 = work + ((int64_t)c * N + a0) * RW, *W1 = W0 + RW;
    for (int kk = threadIdx.x; kk < RW; kk += NT) {
        const cpx z = buf[F::at(kk)], zm = buf[F::at((N - kk) & (N - 1))];
        W0[kk] = cpx{real(0.5) * (z.re + zm.re), real(0.5) * (z.im - zm.im)};
        W1[kk] = cpx{real(0.5) * (z.im + zm.im), real(0.5) * (zm.re - z.re)};
    }
}

template <int LOGN, int CB>
__global__ __launch_bounds__(NT) void k_feather_cols(cpx *__restrict__ work, double knorm2) {
    constexpr int N = 1 << LOGN, RW = N / 2 + 1;
    using F = ColFft<LOGN, CB>;
    __shared__ cpx buf[F::LEN];
    __shared__ cpx tws[tw_len<LOGN>()];
    const int c = blockIdx.y, c0 = blockIdx.x * CB;
    cpx *Wc = work + (int64_t)c * N * RW;
    // (COL_LOADS rows in flight, columns past the end read element 0: 57 -> 42 us at 8 x 1024^2, 14 for its bytes)
    for (int e0 = threadIdx.x; e0 < N * CB; e0 += COL_LOADS * NT) {
        cpx v[COL_LOADS];
#pragma unroll
        for (int u = 0; u < COL_LOADS; ++u) {
            const int e = e0 + u * NT, q = e / CB, cc = e - q * CB;
            v[u] = Wc[e < N * CB && c0 + cc < RW ? (int64_t)q * RW + c0 + cc : 0];
        }
#pragma unroll
        for (int u = 0; u < COL_LOADS; ++u) {
            const int e = e0 + u * NT, q = e / CB, cc = e - q * CB;
            if (e < N * CB) buf[F::at(q, cc)] = c0 + cc < RW ? v[u] : cpx{0, 0};
        }
    }
    tw_fill<LOGN>(tws);
    __syncthreads();
    F::forward(buf, tws);
    // B(k) with k^2 = (p^2 + q^2) / (n delta)^2; knorm2 = 2 pi^2 sigma^2 / (n delta)^2
    for (int e = threadIdx.x; e < N * CB; e += NT) {
        const int q = e / CB, cc = e - q * CB;
        const int qs = q < N / 2 ? q : q - N, ps = c0 + cc;
        const real bk = (real)exp(-knorm2 * ((double)ps * ps + (double)qs * qs));
        cpx &z = buf[F::at(q, cc)];
        z = cpx{bk * z.re, bk * z.im};
    }
    __syncthreads();
    F::inverse(buf, tws);
    for (int e = threadIdx.x; e < N * CB; e += NT) {
        const int q = e / CB, cc = e - q * CB;
        if (c0 + cc < RW) Wc[(int64_t)q * RW + c0 + cc] = buf[F::at(q, cc)];
    }
}

template <int LOGN>
__global__ __launch_bounds__(NT) void k_feather_rows_inv(const real *__restrict__ interf, const cpx *__restrict__ work,
                                                         real *__restrict__ out) {
    constexpr int N = 1 << LOGN, RW = N / 2 + 1;
    using F = RowFft<LOGN>;
    __shared__ cpx buf[N];
    __shared__ cpx tws[tw_len<LOGN>()];
    const int c = blockIdx.y, a0 = 2 * blockIdx.x;
    const cpx *X = work + ((int64_t)c * N + a0) * RW, *Y = X + RW;
    for (int kk = threadIdx.x; kk < N; kk += NT) {
        const int src = kk <= N / 2 ? kk : N - kk;
        cpx x = X[src], y = Y[src];
        if (kk > N / 2) {
            x.im = -x.im;
            y.im = -y.im;
        }
        buf[F::at(kk)] = cpx{x.re - y.im, x.im + y.re}; // x + i y
    }
    tw_fill<LOGN>(tws);
    __syncthreads();
    F::inverse(buf, tws);
    const real sc = real(1) / ((real)N * (real)N);
    const int64_t base = ((int64_t)c * N + a0) * N;
    for (int b = threadIdx.x; b < N; b += NT) {
        out[base + b] = interf[base + b] + sc * buf[F::at(b)].re;
        out[base + N + b] = interf[base + N + b] + sc * buf[F::at(b)].im;
    }
}

// ===================================================================== launchers

#define IVX_LOGN_SWITCH(LOGN_VAR, ...)                       \
    switch (LOGN_VAR) {                                      \
    case 6: { constexpr int L = 6; __VA_ARGS__; } break;     \
    case 7: { constexpr int L = 7; __VA_ARGS__; } break;     \
    case 8: { constexpr int L = 8; __VA_ARGS__; } break;     \
    case 9: { constexpr int L = 9; __VA_ARGS__; } break;     \
    case 10: { constexpr int L = 10; __VA_ARGS__; } break;   \
    case 11: { constexpr int L = 11; __VA_ARGS__; } break;   \
    default: return hipErrorInvalidValue;                    \
    }

static int n_items(const Geom &g) { return g.C * g.P; }

hipError_t launch_image_rows(const Geom &g, const real *sky, const real *beams, const real *interp,
                             const real *fscale, const real *dq, const cpx *tw, cpx *R, hipStream_t st) {
    dim3 grid(g.nk / 2, n_items(g));
    IVX_LOGN_SWITCH(g.logn, (k_image_rows<L><<<grid, NT, 0, st>>>(g, sky, beams, interp, fscale, dq, tw, R)));
    return hipGetLastError();
}

// Columns per block: col_batch's width (wider blocks write longer row segments), but narrow
// enough that the launch has about two blocks per compute unit.
template <int LOGN> static int pick_cb(const Geom &g) {
    int cb = col_batch<LOGN>();
    while (cb > 1 && (int64_t)((g.rw + cb - 1) / cb) * n_items(g) < 512) cb >>= 1;
    return cb;
}

// Launch size of a column pass: (item, column group) pairs rounded up to a multiple of 8
// (see col_block).
static dim3 col_grid(const Geom &g, int cb) {
    const int64_t total = (int64_t)((g.rw + cb - 1) / cb) * n_items(g);
    return dim3((unsigned)(8 * ((total + 7) / 8)));
}

#define IVX_CB_SWITCH(CBV, ...)                                                   \
    switch (CBV) {                                                                \
    case 1: { constexpr int B = 1; __VA_ARGS__; } break;                          \
    case 2: { constexpr int B = 2 <= col_batch<L>() ? 2 : 1; __VA_ARGS__; } break;   \
    case 4: { constexpr int B = 4 <= col_batch<L>() ? 4 : 1; __VA_ARGS__; } break;   \
    case 8: { constexpr int B = 8 <= col_batch<L>() ? 8 : 1; __VA_ARGS__; } break;   \
    default: { constexpr int B = 16 <= col_batch<L>() ? 16 : 1; __VA_ARGS__; } break; \
    }

hipError_t launch_col_fwd(const Geom &g, const cpx *R, const cpx *tw, cpx *ext, hipStream_t st) {
    IVX_LOGN_SWITCH(g.logn, {
        const int cb = pick_cb<L>(g);
        IVX_CB_SWITCH(cb, {
            k_col_fwd<L, B><<<col_grid(g, B), NT, 0, st>>>(g, R, tw, ext);
        });
    });
    return hipGetLastError();
}

hipError_t launch_col_inv(const Geom &g, const cpx *E, const cpx *tw, cpx *R, hipStream_t st) {
    IVX_LOGN_SWITCH(g.logn, {
        const int cb = pick_cb<L>(g);
        IVX_CB_SWITCH(cb, {
            k_col_inv<L, B><<<col_grid(g, B), NT, 0, st>>>(g, E, tw, R);
        });
    });
    return hipGetLastError();
}

// The fused pass has one block per (item, column group): worth it once that fills the chip
// several times over (the two-kernel fold has more, smaller blocks for few-item plans).
constexpr int64_t FUSED_FOLD_MIN_BLOCKS = 2048;

bool fold_fusable(const Geom &g) { return g.eh <= 2 * g.nf && g.ew <= g.nf; }

bool fold_fusion_pays(const Geom &g) {
    const int64_t ngrp = (g.rw + IVX_FOLD_CB - 1) / IVX_FOLD_CB;
    return ngrp * g.C * g.P >= FUSED_FOLD_MIN_BLOCKS;
}

hipError_t launch_col_inv_slots(const Geom &g, const int32_t *tslot, const cpx *slots, const cpx *tw, cpx *R,
                                hipStream_t st) {
    if (!fold_fusable(g)) return hipErrorInvalidValue;
    IVX_LOGN_SWITCH(g.logn, {
        const int cb = std::min(pick_cb<L>(g), IVX_FOLD_CB);
        IVX_CB_SWITCH(cb, {
            k_col_inv_slots<L, B><<<col_grid(g, B), NT, 0, st>>>(g, tslot, slots, tw, R);
        });
    });
    return hipGetLastError();
}

hipError_t launch_fold(const Geom &g, const int32_t *tslot, const cpx *slots, cpx *ext, hipStream_t st,
                       const uint8_t *sact) {
    // all columns of a tile to a wave once that gives every SIMD four waves, else fewer (1,024 and 16,384 waves
    // measure the same on the wide mosaic and 2 to 7 us more on single fields of 100)
    const int64_t waves = (int64_t)((g.eh + 63) / 64) * (g.ntx + 1);
    int cols = g.T;
    while (cols > 1 && waves * n_items(g) * ((g.T + cols - 1) / cols) < FOLD_WAVES) cols = (cols + 1) / 2;
    const int64_t blocks = (waves * ((g.T + cols - 1) / cols) + NT / 64 - 1) / (NT / 64);
    k_ext_sum<<<dim3((unsigned)blocks, n_items(g)), NT, 0, st>>>(g, cols, tslot, slots, sact, ext);
    return hipGetLastError();
}

hipError_t launch_row_inv(const Geom &g, const cpx *R, const real *beams, const real *fscale,
                          const real *dq, const cpx *tw, real *gp, hipStream_t st) {
    dim3 grid(g.nk / 2, n_items(g));
    IVX_LOGN_SWITCH(g.logn, (k_row_inv<L><<<grid, NT, 0, st>>>(g, R, beams, fscale, dq, tw, gp)));
    return hipGetLastError();
}

size_t grid_lds_bytes(const Geom &g, int nwave, int lanes) {
    if (lanes == GRID_MFMA_LANES) return 0;
    return (size_t)(1 + grid_groups_per_wave(g.W, lanes) * nwave) * g.win * g.ldw * sizeof(cpx);
}

template <int W, int G, int VPI>
static hipError_t launch_grid_wg(int mode, const GridArgs &a, int n_work, hipStream_t st) {
    const size_t wsz = (size_t)a.g.win * a.g.ldw * sizeof(cpx);
    const int threads = 64 * a.nwave;
    const int ng = (64 / G) * a.nwave;
    const unsigned gx = (unsigned)n_work < GRID_ROW ? (unsigned)n_work : GRID_ROW;
    const dim3 grid(gx, (unsigned)((n_work + gx - 1) / gx));
    switch (mode) {
    case MODE_OBJ: k_grid<W, MODE_OBJ, G, VPI><<<grid, threads, (1 + ng) * wsz, st>>>(a); break;
    case MODE_FWD: k_grid<W, MODE_FWD, G, VPI><<<grid, threads, wsz, st>>>(a); break;
    case MODE_VAL: k_grid<W, MODE_VAL, G, VPI><<<grid, threads, wsz, st>>>(a); break;
    default: k_grid<W, MODE_ADJ, G, VPI><<<grid, threads, ng * wsz, st>>>(a); break;
    }
    return hipGetLastError();
}

template <int W, int G, int VPI> static hipError_t prepare_grid_wg(const Geom &g, int nwave) {
    // raise the dynamic-LDS limit of the three modes ahead of any stream capture
    const size_t wsz = (size_t)g.win * g.ldw * sizeof(cpx);
    const int ng = (64 / G) * nwave;
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void *)k_grid<W, MODE_OBJ, G, VPI>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)((1 + ng) * wsz))) != hipSuccess)
        return e;
    if ((e = hipFuncSetAttribute((const void *)k_grid<W, MODE_FWD, G, VPI>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)wsz)) != hipSuccess)
        return e;
    if ((e = hipFuncSetAttribute((const void *)k_grid<W, MODE_VAL, G, VPI>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)wsz)) != hipSuccess)
        return e;
    return hipFuncSetAttribute((const void *)k_grid<W, MODE_ADJ, G, VPI>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(ng * wsz));
}

template <int W, int G>
static hipError_t dispatch_wg(bool prepare, int vpi, int mode, const GridArgs &a, int n_work, hipStream_t st) {
    if (vpi == 2) return prepare ? prepare_grid_wg<W, G, 2>(a.g, a.nwave) : launch_grid_wg<W, G, 2>(mode, a, n_work, st);
    return prepare ? prepare_grid_wg<W, G, 1>(a.g, a.nwave) : launch_grid_wg<W, G, 1>(mode, a, n_work, st);
}

// variant = 10 * lanes + visibilities per group per iteration (81, 82, 161, 162)
template <int W>
static hipError_t dispatch_w(bool prepare, int variant, int mode, const GridArgs &a, int n_work, hipStream_t st) {
    const int lanes = variant / 10, vpi = variant % 10;
    if constexpr (W <= 8) {
        if (lanes == 8) return dispatch_wg<W, 8>(prepare, vpi, mode, a, n_work, st);
    }
    return dispatch_wg<W, 16>(prepare, vpi, mode, a, n_work, st);
}

static hipError_t dispatch(bool prepare, int variant, int mode, const GridArgs &a, int n_work, hipStream_t st) {
    switch (a.g.W) {
    case 4: return dispatch_w<4>(prepare, variant, mode, a, n_work, st);
    case 5: return dispatch_w<5>(prepare, variant, mode, a, n_work, st);
    case 6: return dispatch_w<6>(prepare, variant, mode, a, n_work, st);
    case 7: return dispatch_w<7>(prepare, variant, mode, a, n_work, st);
    case 8: return dispatch_w<8>(prepare, variant, mode, a, n_work, st);
    case 9: return dispatch_w<9>(prepare, variant, mode, a, n_work, st);
    case 10: return dispatch_w<10>(prepare, variant, mode, a, n_work, st);
    case 11: return dispatch_w<11>(prepare, variant, mode, a, n_work, st);
    case 12: return dispatch_w<12>(prepare, variant, mode, a, n_work, st);
    case 13: return dispatch_w<13>(prepare, variant, mode, a, n_work, st);
    case 14: return dispatch_w<14>(prepare, variant, mode, a, n_work, st);
    case 15: return dispatch_w<15>(prepare, variant, mode, a, n_work, st);
    case 16: return dispatch_w<16>(prepare, variant, mode, a, n_work, st);
    default: return hipErrorInvalidValue;
    }
}

#ifndef IVX_REAL_DOUBLE
template <int KW> void launch_gridmx(int mode, dim3 grid, GridArgs a, hipStream_t st) {
    a.esc = (float)a.g.esc;
    a.esb = a.esc * (0.5f * (float)a.g.W);
    a.minus1 = -1.f;
    switch (mode) {
    case MODE_OBJ: k_gridmx<MODE_OBJ, KW><<<grid, 64, 0, st>>>(a); break;
    case MODE_FWD: k_gridmx<MODE_FWD, KW><<<grid, 64, 0, st>>>(a); break;
    case MODE_VAL: k_gridmx<MODE_VAL, KW><<<grid, 64, 0, st>>>(a); break;
    case MODE_WFWD: k_gridmx<MODE_WFWD, KW><<<grid, 64, 0, st>>>(a); break;
    case MODE_WADJ: k_gridmx<MODE_WADJ, KW><<<grid, 64, 0, st>>>(a); break;
    default: k_gridmx<MODE_ADJ, KW><<<grid, 64, 0, st>>>(a); break;
    }
}
#endif

// w-plane passes: 16-lane groups, one visibility per group per iteration, any kernel width.
template <int W> static hipError_t wgrid_w(bool prepare, int mode, const GridArgs &a, int n_work, hipStream_t st) {
    const size_t wsz = (size_t)a.g.win * a.g.ldw * sizeof(cpx);
    const int ng = 4 * a.nwave;
    if (prepare) {
        hipError_t e = hipFuncSetAttribute((const void *)k_grid<W, MODE_WFWD, 16, 1>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)wsz);
        if (e != hipSuccess) return e;
        return hipFuncSetAttribute((const void *)k_grid<W, MODE_WADJ, 16, 1>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)(ng * wsz));
    }
    const unsigned gx = (unsigned)n_work < GRID_ROW ? (unsigned)n_work : GRID_ROW;
    const dim3 grid(gx, (unsigned)((n_work + gx - 1) / gx));
    if (mode == MODE_WFWD) k_grid<W, MODE_WFWD, 16, 1><<<grid, 64 * a.nwave, wsz, st>>>(a);
    else k_grid<W, MODE_WADJ, 16, 1><<<grid, 64 * a.nwave, ng * wsz, st>>>(a);
    return hipGetLastError();
}

static hipError_t wgrid_dispatch(bool prepare, int mode, const GridArgs &a, int n_work, hipStream_t st) {
    switch (a.g.W) {
    case 4: return wgrid_w<4>(prepare, mode, a, n_work, st);
    case 5: return wgrid_w<5>(prepare, mode, a, n_work, st);
    case 6: return wgrid_w<6>(prepare, mode, a, n_work, st);
    case 7: return wgrid_w<7>(prepare, mode, a, n_work, st);
    case 8: return wgrid_w<8>(prepare, mode, a, n_work, st);
    case 9: return wgrid_w<9>(prepare, mode, a, n_work, st);
    case 10: return wgrid_w<10>(prepare, mode, a, n_work, st);
    case 11: return wgrid_w<11>(prepare, mode, a, n_work, st);
    case 12: return wgrid_w<12>(prepare, mode, a, n_work, st);
    case 13: return wgrid_w<13>(prepare, mode, a, n_work, st);
    case 14: return wgrid_w<14>(prepare, mode, a, n_work, st);
    case 15: return wgrid_w<15>(prepare, mode, a, n_work, st);
    case 16: return wgrid_w<16>(prepare, mode, a, n_work, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t prepare_wgrid(const Geom &g, int nwave) {
    GridArgs a{};
    a.g = g;
    a.nwave = nwave;
    return wgrid_dispatch(true, MODE_WFWD, a, 0, nullptr);
}

hipError_t launch_wgrid(int mode, const Geom &g, const WorkItem *work, int n_work, const VisCoord *crd,
                        const cpx *ext, cpx *slots, const WPlane &wp, int nwave, int variant, hipStream_t st) {
    if (mode != MODE_WFWD && mode != MODE_WADJ) return hipErrorInvalidValue;
    if (n_work <= 0) return hipSuccess;
    if (nwave < 1 || nwave > NT / 64 || wp.W < 2 || wp.W > 16) return hipErrorInvalidValue;
    GridArgs a{};
    a.g = g;
    a.work = work;
    a.crd = crd;
    a.ext = ext;
    a.slots = slots;
    a.nwave = nwave;
    a.n_work = n_work;
    a.wz = wp.wz;
    a.wacc = wp.acc;
    a.wq = wp.q;
    a.wplane = wp.plane;
    a.wW = wp.W;
    a.wcnt = wp.cnt;
    a.wncnt = wp.ncnt;
    a.wsact = mode == MODE_WADJ ? wp.sact : nullptr;
#ifdef IVX_REAL_DOUBLE
    a.wbeta2 = wp.beta;
#else
    a.wbeta2 = (real)(wp.beta * 1.4426950408889634);
#endif
    if (variant == GRID_MFMA_VARIANT) {
#ifdef IVX_REAL_DOUBLE
        return hipErrorInvalidValue;
#else
        if (g.win > 16) return hipErrorInvalidValue;
        const unsigned gx = (unsigned)n_work < GRID_ROW ? (unsigned)n_work : GRID_ROW;
        const dim3 grid(gx, (unsigned)((n_work + gx - 1) / gx));
        switch (g.W) {
        case 7: launch_gridmx<7>(mode, grid, a, st); break;
        case 8: launch_gridmx<8>(mode, grid, a, st); break;
        default: launch_gridmx<0>(mode, grid, a, st); break;
        }
        return hipGetLastError();
#endif
    }
    return wgrid_dispatch(false, mode, a, n_work, st);
}

hipError_t prepare_grid(const Geom &g, int nwave, int variant) {
    if (variant == GRID_MFMA_VARIANT) return hipSuccess; // static LDS only
    GridArgs a{};
    a.g = g;
    a.nwave = nwave;
    return dispatch(true, variant, MODE_OBJ, a, 0, nullptr);
}


hipError_t launch_grid(int mode, const Geom &g, const WorkItem *work, int n_work, const VisCoord *crd,
                       const cpx *vis, const real *wgt, const int32_t *perm, const int64_t *boff, const cpx *ext,
                       cpx *slots, double *jpart, const cpx *caller_in, cpx *caller_out, int nwave, int variant,
                       hipStream_t st, bool unweighted) {
    if (n_work <= 0) return hipSuccess;
    if (nwave < 1 || nwave > NT / 64) return hipErrorInvalidValue;
    GridArgs a{g, work, crd, vis, wgt, perm, boff, ext, slots, jpart, caller_in, caller_out, nwave, n_work,
               unweighted ? 1 : 0};
    if (variant == GRID_MFMA_VARIANT) {
#ifdef IVX_REAL_DOUBLE
        return hipErrorInvalidValue;
#else
        if (g.win > 16) return hipErrorInvalidValue;
        const unsigned gx = (unsigned)n_work < GRID_ROW ? (unsigned)n_work : GRID_ROW;
        const dim3 grid(gx, (unsigned)((n_work + gx - 1) / gx));
        switch (g.W) {
        case 7: launch_gridmx<7>(mode, grid, a, st); break;
        case 8: launch_gridmx<8>(mode, grid, a, st); break;
        default: launch_gridmx<0>(mode, grid, a, st); break;
        }
        return hipGetLastError();
#endif
    }
    return dispatch(false, variant, mode, a, n_work, st);
}

hipError_t launch_sd_rows(const Geom &g, const real *sky, const real *gB, int rb, int sd_n, int stride,
                          int offset, real *U, hipStream_t st) {
    const int64_t tot = (int64_t)g.C * g.N * sd_n;
    const bool one = stride == 1 && tot >= SD_FULL;
    const int64_t per = one ? NT : NT / SD_ROW_P;
    const unsigned blocks = (unsigned)std::min((tot + per - 1) / per, SD_ROW_BLOCKS);
    if (one) k_sd_rows<1><<<blocks, NT, 0, st>>>(g, sky, gB, rb, sd_n, stride, offset, U);
    else k_sd_rows<SD_ROW_P><<<blocks, NT, 0, st>>>(g, sky, gB, rb, sd_n, stride, offset, U);
    return hipGetLastError();
}

int sd_col_blocks(const Geom &g, int sd_n) {
    constexpr int PER = NT / SD_COL_P;
    return (int)std::min(((int64_t)g.C * sd_n * sd_n + PER - 1) / PER, SD_COL_BLOCKS);
}

hipError_t launch_sd_cols(const Geom &g, const real *U, const real *gB, int rb, int sd_n, int stride,
                          int offset, const real *sdmap, real inv_var, real *E, double *kpart, hipStream_t st) {
    k_sd_cols<<<(unsigned)sd_col_blocks(g, sd_n), NT, 0, st>>>(g, U, gB, rb, sd_n, stride, offset, sdmap, inv_var, E, kpart);
    return hipGetLastError();
}

hipError_t launch_sd_back(const Geom &g, const real *E, const real *gB, int rb, int sd_n, int stride, int offset,
                          real *V, hipStream_t st) {
    const int64_t tot = (int64_t)g.C * sd_n * g.N;
    k_sd_back<<<(unsigned)((tot + NT - 1) / NT), NT, 0, st>>>(g, E, gB, rb, sd_n, stride, offset, V);
    return hipGetLastError();
}

int sky_blocks(const Geom &g) {
    const int nb = (g.N + SKY_T - 1) / SKY_T;
    return nb * nb * g.C;
}

hipError_t launch_sky(const Geom &g, const real *sky, const real *gp, const int32_t *cptr, const CsrEnt *cent,
                      real lambda_r, real lambda_s, const real *E, const real *gB, int rb, int sd_n, int stride,
                      int offset, real *grad, double *rpart, int mode, real scale, hipStream_t st, real lambda_nu,
                      double *npart) {
    const int nb = (g.N + SKY_T - 1) / SKY_T;
    if (lambda_nu != real(0) && !npart) return hipErrorInvalidValue;
    SkyArgs a{g,    sky,  gp,    cptr,  cent,      lambda_r, lambda_s, E, gB, rb, sd_n, stride, offset, grad, rpart,
              mode, scale, lambda_nu, npart};
    const int64_t total = (int64_t)nb * nb * g.C;
    k_sky<<<dim3((unsigned)(8 * ((total + 7) / 8))), NT, 0, st>>>(a);
    return hipGetLastError();
}

int final_scratch(int nj) { return nj > 32 * FINAL_PER ? (nj + FINAL_PER - 1) / FINAL_PER : 0; }

hipError_t launch_final(const double *jpart, int nj, double *scratch, const double *rpart, int nr,
                        const double *kpart, int nkp, const double *npart, int nnp, double lambda_r,
                        double lambda_s, double lambda_nu, double *terms, double *terms_user, hipStream_t st) {
    const int nb = final_scratch(nj);
    if (nb > 0) {
        // long per-work-item lists (large mosaics): pre-reduce in fixed blocks first
        k_partial_sums<<<nb, NT, 0, st>>>(jpart, nj, FINAL_PER, scratch);
        jpart = scratch;
        nj = nb;
    }
    k_final<<<1, NT_FINAL, 0, st>>>(jpart, nj, rpart, nr, kpart, nkp, npart, nnp, lambda_r, lambda_s, lambda_nu, terms,
                                    terms_user);
    return hipGetLastError();
}

int64_t feather_work_bytes(int n_chan, int n) { return (int64_t)n_chan * n * (n / 2 + 1) * (int64_t)sizeof(cpx); }

hipError_t launch_feather(int n_chan, int n, double delta, double theta, const real *interf, const real *sd, real *out,
                          void *work, hipStream_t st) {
    int logn = 0;
    while ((1 << logn) < n) ++logn;
    cpx *w = static_cast<cpx *>(work);
    const double sigma = theta / (2.0 * sqrt(2.0 * log(2.0)));
    const double knorm2 = 2.0 * M_PI * M_PI * sigma * sigma / ((double)n * delta * (double)n * delta);
    const int rw = n / 2 + 1;
    IVX_LOGN_SWITCH(logn, {
        constexpr int CB = col_batch<L>();
        k_feather_rows<L><<<dim3(n / 2, n_chan), NT, 0, st>>>(interf, sd, w);
        k_feather_cols<L, CB><<<dim3((rw + CB - 1) / CB, n_chan), NT, 0, st>>>(w, knorm2);
        k_feather_rows_inv<L><<<dim3(n / 2, n_chan), NT, 0, st>>>(interf, w, out);
    });
    return hipGetLastError();
}

hipError_t launch_zero(void *p, int64_t bytes, hipStream_t st) {
    if (bytes <= 0) return hipSuccess;
    if (bytes % 4) return hipErrorInvalidValue;
    const int64_t n = bytes / 4;
    int64_t blocks = (n + NT - 1) / NT;
    if (blocks > 4096) blocks = 4096;
    k_zero<<<(unsigned)blocks, NT, 0, st>>>((uint32_t *)p, n);
    return hipGetLastError();
}

} // namespace ivx
