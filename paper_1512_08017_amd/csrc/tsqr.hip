// Streaming QR fit: the least-squares problem of Sec. II solved through an
// orthogonal factorisation of V = [t_i^k] (the comparator of Sec. III, QR
// instead of the normal equations), in the tall-skinny tree form: every lane
// factors the rows it streams, and the factors are merged lane -> wave ->
// block -> fit.  The error is governed by cond(V) rather than cond(V)^2.
//
// A factor of the rows seen so far is kept without square roots (Gentleman's
// square-root-free Givens rotations): R = D^(1/2) Rb with Rb unit upper
// triangular, D = diag(d), the rotated right side th (Rb b = th solves the
// fit) and the residual sum of squares e.  Including a row (x; y) of weight w
// rotates it into the factor column by column:
//   d' = d_i + w x_i^2,  w <- w d_i / d',
//   x_k <- x_k - x_i Rb_ik,  Rb_ik <- (d_i Rb_ik + w x_i x_k) / d'   (k > i, old x_k; and y/th),
// and adds w y^2 to e at the end.  The factor holds U = D Rb (and D th) and 1/d_i in
// place of Rb, so that an entry of a rotation is two multiply-adds,
//   x_k <- x_k - (x_i / d_i) U_ik,  U_ik <- U_ik + w x_i x_k,
// and no term is larger than the sums it stands for.  Updating Rb_ik itself in as many
// operations, as Rb_ik + s x_k' with the reduced x_k', cancels where d_i is small
// against w x_i^2, that is where rows of nearly equal t meet others: x in pairs 1e-8
// apart left the coefficients 1e-9 off at cond(V) = 2, sorted x in eleven clusters
// 1e-4 wide 1e-11 (so 1e-15).  Two factors merge by including the rows of one,
// (weight d_i, row Rb_i, right side th_i), into the other.
//
// A single fit large enough for it (qr_sampled in api.hip) first tries a shorter route to the
// same R and solution, a Cholesky factorisation of a Gram matrix that is near
// the identity to begin with (k_qr_sampled, k_qr_sampled_finish): every wave
// orthogonalises the powers of t over the range sample of the points (the
// discrete orthogonal polynomials p_0..p_m of the sample, by Stieltjes'
// three-term recurrence), fits the sample in them, and the pass sums the Gram
// matrix of p_0..p_m and the right sides of the remaining residual over all the
// points.  With P = [p_k(t_i)] the factor of V is R = chol(P^T P) R_sample, and
// cond(P) is near 1 wherever the sample stands for the points, so squaring it
// costs nothing and the error is governed by cond(V) as in the rotations.  The
// finish computes that condition.  Where the sample does not stand for the points (tails
// of x that 256 samples miss), chol(P^T P) still gives the recurrence of the
// polynomials that are orthogonal over all the points, and a second pass in them, with the
// first one's solution as the fit to take the residual from, is near the identity by
// construction (k_qr_if_left; Cholesky QR done twice).  What is beyond that as
// well is left to the rotations, which need no assumption.
#include "kernels_impl.hpp"

namespace lsefit {

// 1/v for v > 0: the hardware reciprocal refined by two Newton steps
// (r <- r + r (1 - v r)), to within a unit or so in the last place; a rotation
// with such c, s stays orthogonal to the same order as its rounding
__device__ inline double recip(double v) {
    double r = __builtin_amdgcn_rcp(v);
    r = fma(r, fma(-v, r, 1.0), r);
    r = fma(r, fma(-v, r, 1.0), r);
    return r;
}

template <int N>
struct GivensQR {
    static constexpr int NR = N * (N - 1) / 2;   // strict upper part, packed by rows
    static constexpr int LEN = 2 * N + NR + 1;   // flat: d, th, Rb, e
    double d[N], iv[N];                          // iv_i = 1/d_i, 0 while d_i is
    double uy[N], u[NR > 0 ? NR : 1], e;         // D th and D Rb

    __device__ inline void zero() {
#pragma unroll
        for (int i = 0; i < N; ++i) d[i] = iv[i] = uy[i] = 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) u[k] = 0.0;
        e = 0.0;
    }
    // offset of U_(i, i+1) in u
    static constexpr int row_at(int i) { return i * N - i * (i + 1) / 2; }
    __device__ inline double rb(int i, int k) const { return u[row_at(i) + k - i - 1] * iv[i]; }
    __device__ inline double th(int i) const { return uy[i] * iv[i]; }

    // include the row (x; y) of weight w whose entries before column S are zero.
    // GUARD = false when every d_i (i >= S) is already positive: then
    // d_i' >= d_i > 0 (w x_i^2 >= 0), the zero-weight case cannot occur, and
    // the result is the same bit for bit without its selects
    template <int S, bool GUARD = true>
    __device__ inline void include(double w, double (&x)[N], double y) {
#pragma unroll
        for (int i = S; i < N; ++i) {
            const double xi = x[i];
            const double di = d[i];
            const double wxi = w * xi;
            const double dpi = fma(wxi, xi, di);
            const bool nz = !GUARD || dpi != 0.0;
            const double g = xi * iv[i];
            iv[i] = nz ? recip(dpi) : 0.0;
            w *= nz ? di * iv[i] : 1.0;
            d[i] = dpi;
#pragma unroll
            for (int k = i + 1; k < N; ++k) {
                double& uik = u[row_at(i) + k - i - 1];
                const double old = x[k];
                x[k] = fma(-g, uik, old);
                uik = fma(wxi, old, uik);
            }
            const double old = y;
            y = fma(-g, uy[i], old);
            uy[i] = fma(wxi, old, uy[i]);
            // degrees 7 and 8: the scheduler keeps to one column, else the live values of
            // several exceed the registers (a fit left to the rotations, degree 8: 127 us, else 158)
            if constexpr (N >= 8) __builtin_amdgcn_sched_barrier(0);
        }
        e = fma(w * y, y, e);
    }

    // every d_i of columns 1.. positive (d_0 counts the rows, so it is too
    // once one row is in): from then on data rows need no zero-weight guard
    __device__ inline bool settled() const {
        bool ok = true;
#pragma unroll
        for (int i = 1; i < N; ++i) ok = ok && d[i] > 0.0;
        return ok;
    }

    // a data row: x_0 = 1 and weight 1, so the first column needs no products.
    // With TABLE, 1/(d_0 + 1) is read from tab (tab[j] = recip(j + 1), the same
    // value): d_0 counts the data rows exactly, and the caller has checked that
    // it is below the table's length
    template <bool GUARD = true, bool TABLE = false>
    __device__ inline void include_data(double (&x)[N], double y, const double* tab = nullptr) {
        const double dp = d[0] + 1.0;
        const double g = iv[0];
        if constexpr (TABLE) iv[0] = tab[(int)d[0]];
        else iv[0] = recip(dp);
        const double w = d[0] * iv[0];
        d[0] = dp;
#pragma unroll
        for (int k = 1; k < N; ++k) {
            double& u0k = u[k - 1];
            const double old = x[k];
            x[k] = fma(-g, u0k, old);
            u0k += old;
        }
        const double old = y;
        y = fma(-g, uy[0], old);
        uy[0] += old;
        if constexpr (N > 1) include<1, GUARD>(w, x, y);
        else e = fma(w * y, y, e);
    }

    // merge another factor, given by a reader of its flat entries: get(j) = flat[j]
    template <class Get>
    __device__ inline void merge(Get&& get) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double x[N];
#pragma unroll
            for (int k = 0; k < N; ++k) x[k] = k == i ? 1.0 : 0.0;
#pragma unroll
            for (int k = i + 1; k < N; ++k) x[k] = get(2 * N + row_at(i) + k - i - 1);
            include_row(i, get(i), x, get(N + i));
        }
        e += get(LEN - 1);
    }
    template <int I = 0>
    __device__ inline void include_row(int i, double w, double (&x)[N], double y) {
        if constexpr (I < N) {
            if (i == I) include<I>(w, x, y);
            else include_row<I + 1>(i, w, x, y);
        }
    }

    __device__ inline double flat(int j) const {
        double v = e;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (j == i) v = d[i];
            if (j == N + i) v = th(i);
#pragma unroll
            for (int k = i + 1; k < N; ++k)
                if (j == 2 * N + row_at(i) + k - i - 1) v = rb(i, k);
        }
        return v;
    }
};

// 1/(j+1) for j < kRecipRows, by recip() once per block into LDS: a factor of
// k data rows has d_0 = k exactly, so the first-column reciprocal of its next
// row is entry k, read instead of recomputed (the float64 reciprocal issues at
// a quarter of the rate and needs two Newton steps)
constexpr int kRecipRows = 1024;

__device__ inline void fill_recip_rows(double* tab) {
    for (int j = threadIdx.x; j < kRecipRows; j += blockDim.x) tab[j] = recip((double)(j + 1));
    __syncthreads();
}

// one point of the streaming pass: the row (1, t, .., t^m; y), weight 1
template <int M>
struct AccQR {
    static constexpr int N = M + 1;
    GivensQR<N> q;
    double inv_s, nc;
    bool settled = false;   // q.settled() (d_i only grow, so once true it stays true)
    const double* tab;   // kRecipRows reciprocals 1/(j+1) in LDS (fill_recip_rows)
    __device__ inline void init(double c, double is, const double* t) {
        q.zero();
        inv_s = is;
        nc = -c * is;
        tab = t;
    }
    template <bool GUARD = true, bool TABLE = false>
    __device__ inline void point(double xv, double yv) {
        const double t = fma(xv, inv_s, nc);
        double row[N];
        row[0] = 1.0;
#pragma unroll
        for (int k = 1; k < N; ++k) row[k] = row[k - 1] * t;
        q.template include_data<GUARD, TABLE>(row, yv, tab);
    }
    template <bool GUARD, bool TABLE, typename V, int VW>
    __device__ inline void rows(const V& xv, const V& yv) {
#pragma unroll
        for (int e = 0; e < VW; ++e) point<GUARD, TABLE>((double)xv[e], (double)yv[e]);
    }
    // a lane whose factor has settled (after its first N distinct points or
    // so) takes the rows without the zero-weight selects, and
    // while its row count stays inside the table, the first column's
    // reciprocals from it
    template <typename V, int VW>
    __device__ inline void vec(const V& xv, const V& yv) {
        if (settled) {
            if (q.d[0] <= (double)(kRecipRows - VW)) rows<false, true, V, VW>(xv, yv);
            else rows<false, false, V, VW>(xv, yv);
        } else {
            rows<true, false, V, VW>(xv, yv);
            settled = q.settled();
        }
    }
    __device__ inline void scalar(double xv, double yv) { point(xv, yv); }
};

// lanes 0 .. 63 -> lane 0: at each level lane l < off merges the factor of lane
// l + off, row by row; the senders (lanes >= off) do not change during the
// level, and every lane takes part in the shuffles.  Fixed order, so the
// result is reproducible.  A loop over the levels: unrolled, the six of degree 8 were too
// much code to inline and the factor went through scratch memory (65,536 fits of 64
// points 5.2 ms, 1.2 as a loop; no lower degree is slower).
template <int N, int LANES = kWave>
__device__ inline void wave_merge(GivensQR<N>& q) {
    const int lane = lane_id() % LANES;   // LANES < 64: within each group of that many lanes
#pragma unroll 1
    for (int off = LANES / 2; off >= 1; off >>= 1) {
        const bool recv = lane < off;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double wi = __shfl_down(q.d[i], off, kWave);
            const double yi = __shfl_down(q.th(i), off, kWave);
            double x[N];
#pragma unroll
            for (int k = 0; k < N; ++k) x[k] = k == i ? 1.0 : 0.0;
#pragma unroll
            for (int k = i + 1; k < N; ++k) x[k] = __shfl_down(q.rb(i, k), off, kWave);
            if (recv) q.include_row(i, wi, x, yi);
        }
        const double eo = __shfl_down(q.e, off, kWave);
        if (recv) q.e += eo;
    }
}

// the block's waves -> one factor, written sum-major (entry j of block g of G at
// part[j G + g])
template <int N>
__device__ inline void block_merge_store(const Work& w, GivensQR<N>& q, int64_t block, int64_t blocks) {
    constexpr int LEN = GivensQR<N>::LEN;
    __shared__ double sh[4][LEN];
    wave_merge(q);
    const int wid = wave_id_in_block();
    if (lane_id() == 0 && wid > 0) {
#pragma unroll
        for (int j = 0; j < LEN; ++j) sh[wid][j] = q.flat(j);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = blockDim.x / kWave;
        for (int v = 1; v < nw; ++v) q.merge([&](int j) { return sh[v][j]; });
#pragma unroll
        for (int j = 0; j < LEN; ++j) w.part[(int64_t)j * blocks + block] = q.flat(j);
    }
}

// Every point updates the same factor, so the rounds carry no parallel work
// worth registers: one vector per round and a register budget (96 VGPRs,
// 5 waves per SIMD, up to m = 2; 128 and 4 to m = 4; 256 above) keep the
// compiler from hoisting across points, and the extra waves cover the
// dependence chain through each column's reciprocal.
constexpr int qr_waves_per_eu(int M) { return M <= 2 ? 5 : (M <= 4 ? 4 : 2); }

// the share of wave `wave` of W, in block `block` of `blocks`
template <typename In, int U, int M>
__device__ __forceinline__ void qr_single_pass(const FitDesc& d, const Work& w, const In* __restrict__ x,
                                      const In* __restrict__ y, int64_t wave, int64_t W, int64_t block, int64_t blocks,
                                      int mis, const RangeArg& ra) {
    double c, inv_s;
    single_range(d, w, x, ra, &c, &inv_s);
    __shared__ double tab[kRecipRows];
    fill_recip_rows(tab);
    AccQR<M> acc;
    acc.init(c, inv_s, tab);
    stream_strided<U>(x, y, d.n_single, mis, wave, W, acc);
    block_merge_store<M + 1>(w, acc.q, block, blocks);
}

template <typename In, int U, int M>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(qr_waves_per_eu(M))))
    k_qr_single(FitDesc d, Work w, const In* __restrict__ x, const In* __restrict__ y, int64_t W, int mis,
                RangeArg ra) {
    const KernelClock kclock_(w.clock);
    const int64_t wave = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave_id_in_block();
    qr_single_pass<In, U, M>(d, w, x, y, wave, W, blockIdx.x, gridDim.x, mis, ra);
}

// Solve Rb b = th for a merged factor of npts rows and write a_0..a_m to out
// (then b_0..b_m after them with write_b) and b to the record; returns the
// status.  Singular when fewer than m+1 points or some d_i <= 2^-80 max_k d_k
// (|R_ii| <= 2^-40 max_k |R_kk|); non-finite when any entry is.
template <int N>
__device__ inline int qr_solve_store(const GivensQR<N>& q, int64_t npts, double c, double s, double* rec_b,
                                     double* out, bool write_b) {
    int st = npts < N ? LSEFIT_ERR_SINGULAR : LSEFIT_OK;
    bool finite = isfinite(q.e);
    double dmax = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        finite = finite && isfinite(q.d[i]) && isfinite(q.uy[i]);
        dmax = fmax(dmax, q.d[i]);
    }
#pragma unroll
    for (int k = 0; k < GivensQR<N>::NR; ++k) finite = finite && isfinite(q.u[k]);
    if (!finite) st = LSEFIT_ERR_NONFINITE;
    const double tiny = ldexp(dmax, -80);
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (st == LSEFIT_OK && !(q.d[i] > tiny)) st = LSEFIT_ERR_SINGULAR;
    double b[N], a[N];
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
        double acc = q.uy[i];
#pragma unroll
        for (int k = i + 1; k < N; ++k) acc -= q.u[GivensQR<N>::row_at(i) + k - i - 1] * b[k];
        b[i] = acc * q.iv[i];
    }
    if (st == LSEFIT_OK) {
        to_x_basis<N>(b, c, s, a);
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (!isfinite(a[k]) || !isfinite(b[k])) st = LSEFIT_ERR_NONFINITE;
    }
    if (st != LSEFIT_OK) {
#pragma unroll
        for (int k = 0; k < N; ++k) a[k] = b[k] = NAN;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        out[k] = a[k];
        if (write_b) out[N + k] = b[k];
        rec_b[k] = b[k];
    }
    return st;
}

// Merge the G block factors (thread t takes blocks t, t + T, ... of the block's
// T <= 256 threads, in order; then lanes, then waves, in order), solve, and
// write [a | b], the status and, if asked, info = [c, s, e].
template <int M>
__device__ inline void qr_finish_block(const FitDesc& d, const Work& w, int64_t G, int maxm, double* __restrict__ coef,
                                       int32_t* __restrict__ status, double* __restrict__ info) {
    constexpr int N = M + 1;
    constexpr int LEN = GivensQR<N>::LEN;
    __shared__ double sh[4][LEN];
    GivensQR<N> q;
    q.zero();
    for (int64_t g = threadIdx.x; g < G; g += blockDim.x) q.merge([&](int j) { return w.part[(int64_t)j * G + g]; });
    wave_merge(q);
    const int wid = wave_id_in_block();
    if (lane_id() == 0 && wid > 0) {
#pragma unroll
        for (int j = 0; j < LEN; ++j) sh[wid][j] = q.flat(j);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const int nw = blockDim.x / kWave;
    for (int v = 1; v < nw; ++v) q.merge([&](int j) { return sh[v][j]; });
    double* r = w.rec;
    const int st = qr_solve_store<N>(q, d.n_single, r[0], r[1], r + rec_b(maxm), coef, true);
    w.pstatus[0] = st;
    status[0] = st;
    if (info) {
        info[0] = r[0];
        info[1] = r[1];
        info[2] = st == LSEFIT_OK ? q.e : NAN;
    }
}

template <int M>
__global__ void __launch_bounds__(256)
    k_qr_finish(FitDesc d, Work w, int64_t G, int maxm, double* __restrict__ coef, int32_t* __restrict__ status,
                double* __restrict__ info) {
    const KernelClock kclock_(w.clock);
    qr_finish_block<M>(d, w, G, maxm, coef, status, info);
}

// ---------------------------------------------------------------------------
// the sampled route of a single fit
// ---------------------------------------------------------------------------

// Sums of the pass: with p_0..p_m the sample's polynomials, sum p_k (m), sum
// p_k p_m (m), sum r p_k (m + 1) and sum r^2.  The rest of the Gram matrix follows from
// the recurrence, as in the Chebyshev basis: since (t - al_k) p_k = ga_k (p_(k+1) +
// p_(k-1)), taking <p_j, t p_k> both ways gives
//   G_(j+1),k = (ga_k (G_j,(k+1) + G_j,(k-1)) + (al_k - al_j) G_jk) / ga_j - G_(j-1),k,
// which fills row j + 1 from the two above it, its last entry summed.  That is 6m + 3
// float64 operations per point (t and the recurrence 2m, the residual m + 1, its sums and
// square 2, the other sums 3m; with the two conversions 35 at m = 5, 53 at m = 8)
// where all m (m + 1) / 2 products take 5m + 3 + m (m + 1) / 2 of them, and
// the rotations about (m + 1)(m + 2) + 12 m.
__host__ __device__ constexpr int gram_len(int m) { return 3 * m + 2; }

// The sample's polynomials, orthogonal over it and scaled so that their
// recurrence is p_(k+1) = ((t - al_k) / ga_k) p_k - p_(k-1) (two multiply-adds
// per point, as (t - al_k) / ga_k is affine in t), p_1 = t - al_0, and the fit of the
// sample in them, sum_k de_k p_k.  Orthogonality to p_(k-1) sets
// ga_k = ga_(k-1) |p_k|^2 / |p_(k-1)|^2.  Every wave computes them from the same
// samples (those of single_range, which its rule for (c, s) also takes), so they
// are the same bits everywhere.  A sample with too few distinct t, or a
// non-finite one, gives NaN, which the finish sees in the sums.
template <int M>
struct OrthoBasis {
    double al[M], ga[M], de[M + 1];
    double last;   // |p_M|^2 / |p_(M-1)|^2
    double c, s;

    // kept in the fit's record between the launches, in the place of sums and lambda
    static constexpr int kAl = rec_S(M), kGa = kAl + M, kLast = kGa + M, kDe = rec_lam(M);
    __device__ inline void store(double* r) const {
#pragma unroll
        for (int k = 0; k < M; ++k) {
            r[kAl + k] = al[k];
            r[kGa + k] = ga[k];
        }
        r[kLast] = last;
#pragma unroll
        for (int k = 0; k <= M; ++k) r[kDe + k] = de[k];
    }
    __device__ inline void load(const double* r) {
        c = r[0];
        s = r[1];
#pragma unroll
        for (int k = 0; k < M; ++k) {
            al[k] = r[kAl + k];
            ga[k] = r[kGa + k];
        }
        last = r[kLast];
#pragma unroll
        for (int k = 0; k <= M; ++k) de[k] = r[kDe + k];
    }

    // the samples are loaded once, x and y together, for the range and the basis
    template <typename In>
    __device__ inline void build(const In* __restrict__ x, const In* __restrict__ y, int64_t n, const RangeArg& ra) {
        constexpr int J = kSingleRangeSamples / kWave;
        double t[J], r[J], p[J], pp[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int64_t i = sample_at(lane_id() + j * kWave, n);
            t[j] = (double)x[i];
            r[j] = (double)y[i];
        }
        c = ra.c;
        s = ra.s;
        if (ra.mode == LSEFIT_RANGE_AUTO) {
            double lo = INFINITY, hi = -INFINITY;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                if (isfinite(t[j])) {
                    lo = fmin(lo, t[j]);
                    hi = fmax(hi, t[j]);
                }
            }
            snap_range(wave_min(lo), wave_max(hi), &c, &s);
        }
        const double inv_s = 1.0 / s, nc = -c * inv_s;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            t[j] = fma(t[j], inv_s, nc);
            p[j] = 1.0;
            pp[j] = 0.0;
        }
        double before = 1.0;   // 1 / |p_(k-1)|^2
#pragma unroll
        for (int k = 0; k <= M; ++k) {
            double nu = 0.0, tp = 0.0, rp = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const double sq = p[j] * p[j];
                nu += sq;
                tp = fma(t[j], sq, tp);
                rp = fma(r[j], p[j], rp);
            }
            nu = wave_sum(nu);
            rp = wave_sum(rp);
            const double inv = recip(nu);
            const double ratio = nu * before;
            before = inv;
            de[k] = rp * inv;
            if (k < M) {
                al[k] = wave_sum(tp) * inv;
                ga[k] = k > 0 ? ga[k > 0 ? k - 1 : 0] * ratio : 1.0;
                const double step = recip(ga[k]);
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    r[j] = fma(-de[k], p[j], r[j]);
                    const double pn = fma((t[j] - al[k]) * step, p[j], -pp[j]);
                    pp[j] = p[j];
                    p[j] = pn;
                }
            } else {
                last = ratio;
            }
        }
    }
};

template <int M>
struct AccGram {
    double S[M], H[M], R[M + 1], E;
    double u1[M], u0[M], nd[M + 1];   // (t - al_k) / ga_k = u1 t + u0; -de_k
    // t by itself first: its one rounding is t's own, where a coefficient of x that
    // holds 1 / ga_k would be off by c / s roundings of t (time stamps in seconds over an
    // hour: 5e-11 in the coefficients)
    double inv_s, nc;
    __device__ inline void init(const OrthoBasis<M>& b) {
#pragma unroll
        for (int k = 0; k < M; ++k) S[k] = H[k] = 0.0;
#pragma unroll
        for (int k = 0; k <= M; ++k) R[k] = 0.0;
        E = 0.0;
        inv_s = 1.0 / b.s;
        nc = -b.c * inv_s;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            u1[k] = recip(b.ga[k]);
            u0[k] = -b.al[k] * u1[k];
        }
#pragma unroll
        for (int k = 0; k <= M; ++k) nd[k] = -b.de[k];
    }
    __device__ inline void point(double xv, double yv) {
        const double t = fma(xv, inv_s, nc);
        double p[M + 1];
        p[0] = 1.0;
        p[1] = t + u0[0];   // ga_0 = 1
#pragma unroll
        for (int k = 1; k < M; ++k) p[k + 1] = fma(fma(t, u1[k], u0[k]), p[k], -p[k - 1]);
        double r = yv + nd[0];
#pragma unroll
        for (int k = 1; k <= M; ++k) r = fma(nd[k], p[k], r);
        R[0] += r;
        E = fma(r, r, E);
#pragma unroll
        for (int k = 1; k <= M; ++k) {
            S[k - 1] += p[k];
            H[k - 1] = fma(p[k], p[M], H[k - 1]);
            R[k] = fma(r, p[k], R[k]);
        }
    }
    template <typename V, int VW>
    __device__ inline void vec(const V& xv, const V& yv) {
#pragma unroll
        for (int e = 0; e < VW; ++e) point((double)xv[e], (double)yv[e]);
    }
    __device__ inline void scalar(double xv, double yv) { point(xv, yv); }
    __device__ inline void out(double (&v)[gram_len(M)]) const {
#pragma unroll
        for (int k = 0; k < M; ++k) {
            v[k] = S[k];
            v[M + k] = H[k];
        }
#pragma unroll
        for (int k = 0; k <= M; ++k) v[2 * M + k] = R[k];
        v[3 * M + 1] = E;
    }
};

// the sweep of the power sums in a basis that `basis` makes while the first loads are in flight
template <typename In, int U, int M, class Make>
__device__ inline void gram_pass(const FitDesc& d, const Work& w, const In* __restrict__ x, const In* __restrict__ y,
                                 int64_t W, int mis, OrthoBasis<M>& b, Make&& basis) {
    const int64_t wave = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave_id_in_block();
    AccGram<M> acc;
    stream_strided<U, true>(x, y, d.n_single, mis, wave, W, acc, [&] {
        basis();
        acc.init(b);
    });
    double v[gram_len(M)];
    acc.out(v);
#pragma unroll
    for (int k = 0; k < gram_len(M); ++k) v[k] = wave_sum(v[k]);
    single_block_partial<gram_len(M), gram_len(M)>(w, v);
}

// The pass, its prologue the sample basis in every wave (about 0.7 us a degree, a
// chain of wave sums, behind the first loads).
// Measured against the rotations: 1e8 float32 points, m = 3, 346 -> 133 us (6.0 TB/s,
// near the sweep's own bound); 1e7 points, m = 5, 69 -> 26 us and m = 8, 127 -> 35 us
// (float64 issue); the finish 22 -> 5.5 us at m = 5 and 44 -> 8.2 us at m = 8.
template <typename In, int U, int M>
__global__ void __launch_bounds__(256)
    k_qr_sampled(FitDesc d, Work w, const In* __restrict__ x, const In* __restrict__ y, int64_t W, int mis,
                 RangeArg ra) {
    const KernelClock kclock_(w.clock);
    OrthoBasis<M> b;
    gram_pass<In, U, M>(d, w, x, y, W, mis, b, [&] { b.build(x, y, d.n_single, ra); });
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        w.rec[0] = b.c;
        w.rec[1] = b.s;
        b.store(w.rec);
    }
}

// what is left of a fit after a pass in an orthogonal basis and its finish
enum SampledLeft { kNothingLeft = 0, kRotationsLeft = 1, kSecondPassLeft = 2 };

// One thread: fill the Gram matrix from the pass's sums and solve: L D L^T = P^T P, the
// correction of the fit that the residual was taken from, the residual sum of squares
// sum r^2 - |D^(-1/2) L^-1 P^T r|^2, and the change from p to powers of t and x.
// rs: the fit's record (range and basis).  With e_k the norms that the recurrence says,
// n / K |p_k|^2 for the sample's, the result is written when
//  - every number is finite and every pivot positive;
//  - H = E^(-1/2) P^T P E^(-1/2) has |H^(1/2)|_F^2 |H^(-1/2)|_F^2 <= 1.5 N^2 (N^2 for the
//    identity; 32 N^2 at degree 2, any at degree 1): the pivots alone do not bound its
//    condition.  Emulated on the CPU over x uniform, normal, Laplace, logistic,
//    exponential, lognormal, Student, arcsine and in clusters, degrees 1 to 8, 1,025 to
//    60,001 points: the errors of fits accepted up to there are those of the rotations (a
//    few 1e-16 at degree 4, 1e-15 to 1e-14 at 8); from degree 3 on they are larger past
//    4 N^2, tenfold past 30 N^2 (normal x, degree 8: 5e-12 against 5e-14), at degree 2
//    past 100 N^2, at degree 1 nowhere;
//  - the correction, in this norm, is at most twice the solution: else its rounding, relative
//    to the sample's noise, shows (values that are nearly all noise);
//  - the be_k = ga_k ga_(k-1) of the monic recurrence (1/4 of the squared half-range
//    for smooth densities, k s^2 for a normal one) lie within 2^8 of each other in the
//    sample's basis, so that filling the matrix scales no entry's rounding by more than 2^4 a
//    row, and within 2^16 in the second pass's, where they grow with k for x with tails;
//  - the correction takes less than 63/64 of sum r^2: then the difference is
//    good to 64 roundings;
//  - |R_kk|, R_kk^2 = D_k times the squared leading coefficient, stays above 2^-36
//    of the largest: 16 times clear of the singular rule.
// Where only the second or third fails, H up to 2^40 N^2, the factor gives the
// polynomials orthogonal over all the points, P' = L^-1 P: their recurrence is
//   al'_k = al_k + l_(k+1),k - l_k,(k-1),  be'_k = D_k / D_(k-1)   (monic p),
// and the solution in them, L^T de + D^-1 L^-1 P^T r; both go to the record for a second
// pass, whose H is the identity to 2^40 roundings or so (emulated, up to 2^49: to 1e-3).
template <int M>
__device__ __forceinline__ SampledLeft solve_sampled(const FitDesc& d, const Work& w, const double* sums,
                                                     const double* rs, bool first, double* __restrict__ coef,
                                                     int32_t* __restrict__ status, double* __restrict__ info) {
    constexpr int N = M + 1;
    OrthoBasis<M> B;
    B.load(rs);
    const double n = (double)d.n_single;
    // A: lower triangle, A[k][j] = G_jk; 1 / lead_k: leading coefficients
    double A[N][N], z[N], step[M], e[N], lead[N];
#pragma unroll
    for (int k = 0; k < M; ++k) step[k] = recip(B.ga[k]);
    A[0][0] = n;
#pragma unroll
    for (int k = 1; k <= M; ++k) A[k][0] = sums[k - 1];
#pragma unroll
    for (int j = 1; j <= M; ++j) A[M][j] = sums[M + j - 1];
#pragma unroll
    for (int j = 0; j + 1 < M; ++j) {
#pragma unroll
        for (int k = j + 1; k < M; ++k) {
            const double v = fma(B.ga[k], A[k + 1][j] + A[k - 1][j], (B.al[k] - B.al[j]) * A[k][j]) * step[j];
            A[k][j + 1] = j > 0 ? v - A[k][j > 0 ? j - 1 : 0] : v;
        }
    }
#pragma unroll
    for (int k = 0; k <= M; ++k) z[k] = sums[2 * M + k];
    const double E = sums[gram_len(M) - 1];
    e[0] = n;
    lead[0] = 1.0;
    double trace = 1.0;   // of H
#pragma unroll
    for (int k = 1; k < N; ++k) {   // |p_k|^2 / |p_(k-1)|^2 and the leading coefficient 1 / (ga_0 .. ga_(k-1))
        e[k] = e[k - 1] * (k < M ? B.ga[k < M ? k : 0] * step[k - 1] : B.last);
        lead[k] = lead[k - 1] * B.ga[k - 1];
        trace = fma(A[k][k], recip(e[k]), trace);
    }
    // A = L D L^T in place (unit L below the diagonal), z = L^-1 P^T r
    bool sound = isfinite(E);
    double dmax = 0.0, dmin = INFINITY, taken = 0.0;
    double D[N], inv[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double dk = D[k] = A[k][k];
        sound = sound && isfinite(z[k]) && dk > 0.0 && isfinite(dk);
        dmax = fmax(dmax, dk * lead[k] * lead[k]);
        dmin = fmin(dmin, dk * lead[k] * lead[k]);
        inv[k] = recip(dk);
        taken = fma(z[k] * inv[k], z[k], taken);
        double l[N];
#pragma unroll
        for (int i = k + 1; i < N; ++i) l[i] = A[i][k] * inv[k];
#pragma unroll
        for (int i = k + 1; i < N; ++i) {
#pragma unroll
            for (int j = k + 1; j <= i; ++j) A[i][j] = fma(-l[i], A[j][k], A[i][j]);
            z[i] = fma(-l[i], z[k], z[i]);
        }
#pragma unroll
        for (int i = k + 1; i < N; ++i) A[i][k] = l[i];
    }
    sound = sound && dmin > ldexp(dmax, -72);
    double be_min = INFINITY, be_max = 0.0;
#pragma unroll
    for (int k = 1; k < M; ++k) {
        be_min = fmin(be_min, B.ga[k] * B.ga[k - 1]);
        be_max = fmax(be_max, B.ga[k] * B.ga[k - 1]);
    }
    if (M > 2) sound = sound && be_max <= (first ? 0x1p8 : 0x1p16) * be_min;
    // |H^(-1/2)|_F^2 = sum over L^-1 of (L^-1)_ij^2 e_j / D_i
    double back = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double X[N];
#pragma unroll
        for (int i = j; i < N; ++i) {
            double a = i == j ? 1.0 : 0.0;
#pragma unroll
            for (int k = j; k < i; ++k) a = fma(-A[i][k], X[k], a);
            X[i] = a;
            back = fma(a * a * e[j], inv[i], back);
        }
    }
    const double cond = trace * back * (1.0 / (N * N));
    double g[N], size = 0.0;
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
        double a = z[i] * inv[i];
#pragma unroll
        for (int k = i + 1; k < N; ++k) a = fma(-A[k][i], g[k], a);
        g[i] = a;
        size = fma((B.de[i] + a) * (B.de[i] + a), e[i], size);
    }
    constexpr double limit = M == 1 ? 0x1p40 : (M == 2 ? 32.0 : 1.5);
    const bool near = cond <= limit && taken <= 4.0 * size;
    bool ok = sound && near && taken <= 0.984375 * E;
    if (first && sound && !near && cond <= 0x1p40) {
        OrthoBasis<M> next;
        double up = 1.0;   // lead' of the next basis
        bool good = true;
        double lo = INFINITY, hi = 0.0;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            next.al[k] = fma(B.ga[k], A[k + 1][k], B.al[k]);
            next.ga[k] = 1.0;
            if (k > 0) {
                next.al[k] = fma(-B.ga[k - 1], A[k][k > 0 ? k - 1 : 0], next.al[k]);
                const double be = D[k] * inv[k - 1] * B.ga[k - 1] * B.ga[k - 1];
                next.ga[k] = be * recip(next.ga[k - 1]);
                lo = fmin(lo, be);
                hi = fmax(hi, be);
            }
            good = good && isfinite(next.al[k]) && isfinite(next.ga[k]) && next.ga[k] > 0.0;
        }
        const double r = B.ga[M - 1] * recip(next.ga[M - 1]);
        next.last = D[M] * inv[M - 1] * r * r;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            double a = fma(z[k], inv[k], B.de[k]);
#pragma unroll
            for (int i = k + 1; i < N; ++i) a = fma(A[i][k], B.de[i], a);
            next.de[k] = a * (up * recip(lead[k]));
            good = good && isfinite(next.de[k]);
            if (k < M) up *= next.ga[k < M ? k : 0];
        }
        if (good && isfinite(next.last) && (M <= 2 || hi <= 0x1p16 * lo)) {
            next.store(w.rec);
            return kSecondPassLeft;
        }
    }
    // sum_k (de_k + g_k) p_k in powers of t, from the recurrence
    double b[N], p[N], pp[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        p[j] = j == 0 ? 1.0 : 0.0;
        pp[j] = 0.0;
        b[j] = 0.0;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double a = B.de[k] + g[k];
#pragma unroll
        for (int j = 0; j <= k; ++j) b[j] = fma(a, p[j], b[j]);
        if (k < M) {
            double pn[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const double up = j > 0 ? p[j - 1] : 0.0;
                pn[j] = fma(fma(-B.al[k < M ? k : 0], p[j], up), step[k < M ? k : 0], -pp[j]);
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                pp[j] = p[j];
                p[j] = pn[j];
            }
        }
    }
    double a[N];
    to_x_basis<N>(b, B.c, B.s, a);
#pragma unroll
    for (int k = 0; k < N; ++k) ok = ok && isfinite(a[k]) && isfinite(b[k]);
    if (!ok) return kRotationsLeft;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        coef[k] = a[k];
        coef[N + k] = b[k];
        w.rec[rec_b(M) + k] = b[k];
    }
    w.pstatus[0] = LSEFIT_OK;
    status[0] = LSEFIT_OK;
    if (info) {
        info[0] = B.c;
        info[1] = B.s;
        info[2] = E - taken;
    }
    return kNothingLeft;
}

// Sum the block partials and solve.  The first word of w.tile_start, unused by a
// single fit otherwise, says what is left; the second one counts blocks in the launch after.
template <int M>
__global__ void __launch_bounds__(kFinishWaves * kWave)
    k_qr_sampled_finish(FitDesc d, Work w, int64_t G, double* __restrict__ coef, int32_t* __restrict__ status,
                        double* __restrict__ info) {
    const KernelClock kclock_(w.clock);
    constexpr int rl = rec_len(M);
    __shared__ double sums[gram_len(M)];
    __shared__ double rs[rl];
    const double rv = threadIdx.x < rl ? w.rec[threadIdx.x] : 0.0;
    block_sum_partials<gram_len(M)>(w.part, G, sums);
    if (threadIdx.x < rl) rs[threadIdx.x] = rv;
    __syncthreads();
    if (threadIdx.x != 0) return;
    w.tile_start[0] = solve_sampled<M>(d, w, sums, rs, true, coef, status, info);
    w.tile_start[1] = 0;
}

// the same sums (the same bits) by a block of any number of waves, four of them at a time; the
// partials of G blocks of a grid of `stride`
template <int NK>
__device__ inline void block_sum_partials_by(const double* __restrict__ part, int64_t stride, int64_t G, int waves,
                                             double* out) {
    constexpr int C = 4;
    const int lane = lane_id();
    for (int k0 = C * wave_id_in_block(); k0 < NK; k0 += C * waves) {
        double t[C];
#pragma unroll
        for (int c = 0; c < C; ++c) t[c] = 0.0;
        for (int64_t g0 = 0; g0 < G; g0 += kFinishChunk * kWave) {
            double x[kFinishChunk][C];
#pragma unroll
            for (int i = 0; i < kFinishChunk; ++i) {
                const int64_t g = min(g0 + i * kWave + lane, G - 1);
#pragma unroll
                for (int c = 0; c < C; ++c) x[i][c] = part[(int64_t)min(k0 + c, NK - 1) * stride + g];
            }
#pragma unroll
            for (int i = 0; i < kFinishChunk; ++i) {
                const bool in = g0 + i * kWave + lane < G;
#pragma unroll
                for (int c = 0; c < C; ++c) t[c] = in ? t[c] + x[i][c] : t[c];
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const double tot = wave_sum(t[c]);
            if (lane == 0 && k0 + c < NK) out[k0 + c] = tot;
        }
    }
}

// Whether this block is the last of `blocks` to get here: it then sees what every
// one has stored.  Thread 0 releases its block's stores behind the barrier; only the last
// block acquires (an acquire by every block, which throws cached lines away, cost a
// fit with a second pass over 1e6 points 7 us more).  No block waits for another.
__device__ inline bool last_block(const Work& w, int64_t blocks) {
    __shared__ bool last;
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned long long before = __hip_atomic_fetch_add((unsigned long long*)&w.tile_start[1], 1ull,
                                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = before + 1 == (unsigned long long)blocks;
        if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return last;
}

// What the sampled route has left of a fit (else the kernel returns at once): the second
// pass in the basis of the record, or the rotations.  One launch, so that an accepted
// fit pays for one empty launch and not for several: the last block to store its part
// finishes.  A second pass that its finish does not take (it is the identity by construction; no
// data is known where it does not) is left to the rotations of that block alone.
// Of a small fit only as many blocks take part as have a vector for every lane: the others'
// parts would only be more to merge.
template <typename In, int U, int M>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(M <= 3 ? 4 : 2)))
    k_qr_if_left(FitDesc d, Work w, const In* __restrict__ x, const In* __restrict__ y, int mis, RangeArg ra,
                 double* __restrict__ coef, int32_t* __restrict__ status, double* __restrict__ info) {
    const int64_t left = w.tile_start[0];
    if (left == kNothingLeft) return;
    const int nw = blockDim.x / kWave;
    const int64_t rounds = d.n_single / (VecOf<In>::W * kWave * nw) + 1;   // of one vector a lane
    int64_t blocks = rounds < gridDim.x ? rounds : gridDim.x;
    if (blockIdx.x >= blocks) return;
    int64_t first = (int64_t)blockIdx.x * nw, waves = blocks * nw, block = blockIdx.x;
    if (left == kSecondPassLeft) {
        constexpr int rl = rec_len(M);
        __shared__ double sums[gram_len(M)];
        __shared__ double rs[rl];
        __shared__ int still;
        OrthoBasis<M> b;
        gram_pass<In, 2, M>(d, w, x, y, waves, mis, b, [&] { b.load(w.rec); });
        if (!last_block(w, blocks)) return;
        block_sum_partials_by<gram_len(M)>(w.part, gridDim.x, blocks, nw, sums);
        for (int i = threadIdx.x; i < rl; i += blockDim.x) rs[i] = w.rec[i];
        __syncthreads();
        if (threadIdx.x == 0) still = solve_sampled<M>(d, w, sums, rs, false, coef, status, info);
        __syncthreads();
        if (still == kNothingLeft) return;
        first = block = 0;
        waves = nw;
        blocks = 1;
    }
    qr_single_pass<In, U, M>(d, w, x, y, first + wave_id_in_block(), waves, block, blocks, mis, ra);
    if (left != kSecondPassLeft && !last_block(w, blocks)) return;
    __syncthreads();   // thread 0 has stored the only block's factor
    qr_finish_block<M>(d, w, blocks, M, coef, status, info);
}

// ---------------------------------------------------------------------------
// batches: each wave factors its segment of every fit it streams, merges the
// factor to lane 0 and writes it to the fit's slot w + f (qr_len(maxm)
// doubles); one thread per fit then merges the fit's slots in wave order.
//
// Bound by the rotations' float64 chain, and for short fits by the merge: 6
// levels of dependent rotations are what a whole fit of 64 points costs.  So up
// to degree 4 short fits go 8 to a wave, as in the moment pass (3 levels, and 8
// fits share them).  65,536 fits, float32, this pass: 16 points at degree 2
// 184 -> 24 us; 64 points at degree 3 239 -> 38 us; 16 to 256 points (log-uniform) at
// degrees 1 to 3 257 -> 117 us; 4,096 fits of 4,096 points 73 us (71 before); 16 to
// 65,536 points 1.6 ms both.  Above degree 4 the factor alone takes most of the
// register file, so there the walk stays one fit at a time, its descriptors read
// ahead.
// 3 waves per SIMD up to degree 4 (4 before): at 4 both loops together left
// fits of 4,096 points 2 to 7% slower, at 3 they are no slower than before.
// ---------------------------------------------------------------------------
template <typename In, int MAXC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MAXC <= 4 ? 3 : 2)))
    k_qr_batch(FitDesc d, Work w, const In* __restrict__ x, const In* __restrict__ y, int64_t W,
               int mis, int maxm) {
    const KernelClock kclock_(w.clock);
    const int64_t wave = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave_id_in_block();
    const int stride = qr_len(maxm);
    const int rl = rec_len(maxm);
    __shared__ double tab[kRecipRows];
    fill_recip_rows(tab);
    auto one_fit = [&](int64_t, int64_t lo, int64_t hi, int64_t slot, const SegMeta& mt) {
        if (mt.st != LSEFIT_OK) return;
        const double c = mt.c, inv_s = 1.0 / mt.s;
        double* __restrict__ out = w.part + slot * stride;
        auto body = [&]<int M>() {
            AccQR<M> acc;
            acc.init(c, inv_s, tab);
            stream_segment<1>(x, y, lo, hi, mis, acc);
            wave_merge(acc.q);
            if (lane_id() == 0) {
#pragma unroll
                for (int j = 0; j < GivensQR<M + 1>::LEN; ++j) out[j] = acc.q.flat(j);
            }
        };
        dispatch_degree<MAXC>(mt.deg, body);
    };
    if constexpr (MAXC <= 4) {
        // short fits, kGroups at a time and those of one degree together: 8 lanes
        // factor a fit's rows and merge in 3 levels instead of 6
        auto short_fits = [&](int64_t f, bool mine, const SegMeta& mt) {
            uint64_t left = __ballot(mine);
            while (left) {
                const int deg = __builtin_amdgcn_readlane(mt.deg, __ffsll((unsigned long long)left) - 1);
                const bool now = mine && mt.deg == deg;
                left &= ~__ballot(now);
                auto body = [&]<int M>() {
                    AccQR<M> acc;
                    acc.init(mt.c, 1.0 / mt.s, tab);
                    stream_group<1>(x, y, mt.lo, now ? (int)(mt.hi - mt.lo) : 0, acc);
                    wave_merge<M + 1, kGroup>(acc.q);
                    double* __restrict__ out = w.part + (wave + f) * stride;
                    if (now && lane_id() % kGroup == 0) {
#pragma unroll
                        for (int j = 0; j < GivensQR<M + 1>::LEN; ++j) out[j] = acc.q.flat(j);
                    }
                };
                dispatch_degree<MAXC>(deg, body);
            }
        };
        walk_grouped(d, w.tile_start, w.pstatus, w.rec, rl, wave, W, (int)sizeof(In), short_fits, one_fit);
    } else {
        walk_segments_ahead(d, w.tile_start, w.pstatus, w.rec, rl, wave, W, one_fit);
    }
}

template <int MAXC>
__global__ void __launch_bounds__(256)
    k_qr_combine(FitDesc d, Work w, int64_t W, int maxm, double* __restrict__ coef, int32_t coef_stride,
                 int32_t* __restrict__ status, double* __restrict__ sse) {
    const KernelClock kclock_(w.clock);
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= d.batch) return;
    double* out = coef + f * (int64_t)coef_stride;
    const int m = fit_deg(d, f);
    const int pst = w.pstatus[f];
    if (pst != LSEFIT_OK) {
        const int n = (m >= 1 && m <= maxm) ? m + 1 : coef_stride;
        for (int k = 0; k < n; ++k) out[k] = NAN;
        status[f] = pst;
        if (sse) sse[f] = NAN;
        return;
    }
    const int stride = qr_len(maxm);
    const int64_t NT = w.tile_start[d.batch];
    const int64_t w0 = wave_of_tile(w.tile_start[f], NT, W), w1 = wave_of_tile(w.tile_start[f + 1] - 1, NT, W);
    double* r = w.rec + f * rec_len(maxm);
    auto body = [&]<int M>() {
        GivensQR<M + 1> q;
        q.zero();
        for (int64_t wv = w0; wv <= w1; ++wv) {
            if (!wave_owns_tiles(wv, NT, W)) continue;
            const double* p = w.part + (wv + f) * stride;
            q.merge([&](int j) { return p[j]; });
        }
        const int st = qr_solve_store<M + 1>(q, fit_hi(d, f) - fit_lo(d, f), r[0], r[1], r + rec_b(maxm), out, false);
        w.pstatus[f] = st;
        status[f] = st;
        if (sse) sse[f] = st == LSEFIT_OK ? q.e : NAN;
    };
    dispatch_degree<MAXC>(m, body);
}

hipError_t launch_qr_single(const FitDesc& d, const Work& w, int dtype, const void* x, const void* y,
                            const Launch& L, int mis, const RangeArg& ra, hipStream_t st) {
    const dim3 grid(L.waves / L.wpb), block(L.wpb * kWave);
    auto body = [&]<int M>() {
        if (dtype == LSEFIT_F32)
            launch_timed((k_qr_single<float, 1, M>), grid, block, st, d, w, (const float*)x,
                               (const float*)y, L.waves, mis, ra);
        else
            launch_timed((k_qr_single<double, 1, M>), grid, block, st, d, w, (const double*)x,
                               (const double*)y, L.waves, mis, ra);
    };
    dispatch_degree<LSEFIT_MAX_DEGREE>(d.degree, body);
    return hipGetLastError();
}

hipError_t launch_qr_sampled(const FitDesc& d, const Work& w, int dtype, const void* x, const void* y,
                             const Launch& L, int mis, const RangeArg& ra, hipStream_t st) {
    const dim3 grid(L.waves / L.wpb), block(L.wpb * kWave);
    auto body = [&]<int M>() {
        if (dtype == LSEFIT_F32)
            launch_timed((k_qr_sampled<float, 2, M>), grid, block, st, d, w, (const float*)x, (const float*)y, L.waves,
                         mis, ra);
        else
            launch_timed((k_qr_sampled<double, 2, M>), grid, block, st, d, w, (const double*)x, (const double*)y,
                         L.waves, mis, ra);
    };
    dispatch_degree<LSEFIT_MAX_DEGREE>(d.degree, body);
    return hipGetLastError();
}

hipError_t launch_qr_sampled_finish(const FitDesc& d, const Work& w, int64_t G, double* coef, int32_t* status,
                                    double* info, hipStream_t st) {
    auto body = [&]<int M>() {
        launch_timed(k_qr_sampled_finish<M>, dim3(1), dim3(kFinishWaves * kWave), st, d, w, G, coef, status, info);
    };
    dispatch_degree<LSEFIT_MAX_DEGREE>(d.degree, body);
    return hipGetLastError();
}

hipError_t launch_qr_if_left(const FitDesc& d, const Work& w, int dtype, const void* x, const void* y,
                             const Launch& L, int mis, const RangeArg& ra, double* coef, int32_t* status,
                             double* info, hipStream_t st) {
    const dim3 grid(L.waves / L.wpb), block(L.wpb * kWave);
    auto body = [&]<int M>() {
        if (dtype == LSEFIT_F32)
            hipLaunchKernelGGL((k_qr_if_left<float, 1, M>), grid, block, 0, st, d, w, (const float*)x, (const float*)y,
                               mis, ra, coef, status, info);
        else
            hipLaunchKernelGGL((k_qr_if_left<double, 1, M>), grid, block, 0, st, d, w, (const double*)x,
                               (const double*)y, mis, ra, coef, status, info);
    };
    dispatch_degree<LSEFIT_MAX_DEGREE>(d.degree, body);
    return hipGetLastError();
}

hipError_t launch_qr_batch(const FitDesc& d, const Work& w, int maxm, int dtype, const void* x, const void* y,
                           const Launch& L, int mis, hipStream_t st) {
    const dim3 grid(L.waves / L.wpb), block(L.wpb * kWave);
    auto go = [&]<int MAXC>() {
        if (dtype == LSEFIT_F32)
            launch_timed((k_qr_batch<float, MAXC>), grid, block, st, d, w, (const float*)x, (const float*)y,
                               L.waves, mis, maxm);
        else
            launch_timed((k_qr_batch<double, MAXC>), grid, block, st, d, w, (const double*)x,
                               (const double*)y, L.waves, mis, maxm);
    };
    if (maxm <= 4) go.template operator()<4>();
    else go.template operator()<LSEFIT_MAX_DEGREE>();
    return hipGetLastError();
}

hipError_t launch_qr_combine(const FitDesc& d, const Work& w, int maxm, int64_t W, double* coef, int32_t coef_stride,
                             int32_t* status, double* sse, hipStream_t st) {
    const int64_t blocks = (d.batch + 255) / 256;
    if (maxm <= 4)
        launch_timed(k_qr_combine<4>, dim3(blocks), dim3(256), st, d, w, W, maxm, coef, coef_stride, status,
                           sse);
    else
        launch_timed(k_qr_combine<LSEFIT_MAX_DEGREE>, dim3(blocks), dim3(256), st, d, w, W, maxm, coef,
                           coef_stride, status, sse);
    return hipGetLastError();
}

hipError_t launch_qr_finish(const FitDesc& d, const Work& w, int64_t G, double* coef, int32_t* status, double* info,
                            hipStream_t st) {
    auto body = [&]<int M>() {
        launch_timed(k_qr_finish<M>, dim3(1), dim3(256), st, d, w, G, d.degree, coef, status, info);
    };
    dispatch_degree<LSEFIT_MAX_DEGREE>(d.degree, body);
    return hipGetLastError();
}

}  // namespace lsefit
