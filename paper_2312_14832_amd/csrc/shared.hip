// Batched restarted PDHG over one shared matrix (a parametric family: K
// fixed, c, q, l, u per instance).  The slot structure is the single-LP
// solver's, with one difference that matters for memory traffic: each sparse
// product is an SpMM over interleaved iterates, so K is read once per product
// for a whole group of W instances, and the gather of x[j][0..W) for a nonzero
// K_ij is a contiguous run of W values rather than one value per instance.
// Every per-instance quantity (step size, primal weight, restarts,
// termination) lives in the instance's own controller; within a group a
// lane's instance is fixed (thread t serves instance t % W), so per-instance
// partial sums need no atomics.
#include "device.h"

#include <algorithm>
#include <type_traits>

namespace pdlp {

// One row of the SpMM for instance b: sum over the row's entries [rs, re)
// of v[p] x[ci[p]][b], in entry order.  Eight entries at a time in three
// straight-line phases (indices and values, then the eight gathers, then the
// products), so eight gathers of the row are in flight at once; slots past
// the row's end re-read its last entry and are masked out of the sum.
template <typename T>
__device__ __forceinline__ T spmm_row(const int *__restrict__ ci, const T *__restrict__ v, const T *__restrict__ x,
                                      int rs, int re, int lgW, int b)
{
    constexpr int U = 8;
    T acc = T(0);
    for (int p = rs; p < re; p += U) {
        int c[U];
        T a[U], g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = min(p + u, re - 1);
            c[u] = ci[t];
            a[u] = v[t];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) g[u] = x[((size_t)c[u] << lgW) + b];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (p + u < re) acc += a[u] * g[u];
    }
    return acc;
}

// The value of lane N of the thread's W lanes (W = 8 or 16, a half or a whole
// row of the DPP unit); all W are active.
template <int W, int N>
__device__ __forceinline__ int lane_of(int v)
{
    static_assert(W == 8 || W == 16, "half or whole DPP rows");
    if constexpr (W == 16) return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xf, 0xf, false);   // row_newbcast
    const int lo = __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xf, 0xf, false);
    return __builtin_amdgcn_update_dpp(lo, v, 0x150 + 8 + N % 8, 0xf, 0xc, false);   // the upper half alone
}
template <int W, int N>
__device__ __forceinline__ float lane_of(float v)
{
    return __int_as_float(lane_of<W, N>(__float_as_int(v)));
}
template <int W, int N>
__device__ __forceinline__ double lane_of(double v)
{
    return __hiloint2double(lane_of<W, N>(__double2hiint(v)), lane_of<W, N>(__double2loint(v)));
}

// entries [Q, Q + 4) of the W that a row's lanes hold, then the ones after;
// the branches are the wavefront's, taken while any row has so many left
template <typename T, int W, int Q>
__device__ __forceinline__ void gather_from(int c, const T *x, int left, T *g)
{
    if constexpr (Q < W) {
        if (__ballot(left > Q)) {
            g[Q] = x[lane_of<W, Q>(c)];
            g[Q + 1] = x[lane_of<W, Q + 1>(c)];
            g[Q + 2] = x[lane_of<W, Q + 2>(c)];
            g[Q + 3] = x[lane_of<W, Q + 3>(c)];
            gather_from<T, W, Q + 4>(c, x, left, g);
        }
    }
}
template <typename T, int W, int Q>
__device__ __forceinline__ void add_from(T a, int left, const T *g, T &acc)
{
    if constexpr (Q < W) {
        if (__ballot(left > Q)) {
            const T a0 = lane_of<W, Q>(a), a1 = lane_of<W, Q + 1>(a), a2 = lane_of<W, Q + 2>(a),
                    a3 = lane_of<W, Q + 3>(a);
            if (left > Q) acc += a0 * g[Q];
            if (left > Q + 1) acc += a1 * g[Q + 1];
            if (left > Q + 2) acc += a2 * g[Q + 2];
            if (left > Q + 3) acc += a3 * g[Q + 3];
            add_from<T, W, Q + 4>(a, left, g, acc);
        }
    }
}

// spmm_row for groups of W instances, a power of two from 8, whose W lanes are
// all active: each lane loads one of D consecutive entries of the row, which
// the others get from its register.  The products were bound by the vector
// memory unit's address and data path, busy 84 to 88 percent of their time:
// with every lane loading every index and value, two of three of its
// instructions went to those.  64 members, 1e5 columns, 5e4 rows, 1e6 entries:
// in FP64 sk_dual 118 -> 87 us, sk_update 240 -> 167 us (0.69 GB it cannot do
// without and 0.51 GB of gathers).  x: the group's vector at this lane's column.
template <typename T, int W>
__device__ __forceinline__ T spmm_group(const int *__restrict__ ci, const T *__restrict__ v, const T *__restrict__ x,
                                        int rs, int re, int l)
{
    constexpr int D = W < 16 ? W : 16;
    T acc = T(0);
    int t = max(min(rs + (l & (D - 1)), re - 1), 0);   // past the row's end its last entry, not added
    int c = ci[t];
    T a = v[t];
    for (int p = rs; __ballot(p < re); p += D) {
        // the next entries' loads go out ahead of this pass's gathers
        t = max(min(t + D, re - 1), 0);
        const int cn = ci[t];
        const T an = v[t];
        T g[D];
        gather_from<T, D, 0>(c * W, x, re - p, g);
        add_from<T, D, 0>(a, re - p, g, acc);
        c = cn;
        a = an;
    }
    return acc;
}

// row [rs, re) for the thread's instance; W = 0: any group width
template <typename T, int W>
__device__ __forceinline__ T shared_row(const int *__restrict__ ci, const T *__restrict__ v, const T *__restrict__ x,
                                        int rs, int re, int lgW, int b)
{
    if constexpr (W > 0) return spmm_group<T, W>(ci, v, x + b, rs, re, b);
    else return spmm_row(ci, v, x, rs, re, lgW, b);
}

// The share of a workgroup: XCD x (workgroups x, x + 8, ...) has the groups
// that lie in [x G / 8, (x + 1) G / 8), whole or in eighths, and its P
// workgroups take the 256-element tiles of its share in turn, on from one
// group to the next.  Every workgroup stores a partial for each group of its
// XCD: those of group g come from XCDs x_lo(g) on.
struct Share {
    int x, k, P, g0, g1, W, lgW, G, over_G;
    template <typename T>
    __device__ __forceinline__ explicit Share(const SDev<T> &S)
        : x((int)(blockIdx.x % kXcds)), k((int)(blockIdx.x / kXcds)), P((int)(gridDim.x / kXcds)),
          g0((int)((unsigned)(x * S.G) / kXcds)), g1((int)((unsigned)((x + 1) * S.G - 1) / kXcds)), W(1 << S.lgW),
          lgW(S.lgW), G(S.G), over_G(S.over_G)
    {
    }
    // this thread's column in a group's vectors
    __device__ __forceinline__ int column() const { return (int)threadIdx.x & (W - 1); }
    // 8 g / G with S.over_G = 2^16 / G + 1, exact for G <= 64: a division
    // costs as much as a small launch's whole set-up
    __device__ __forceinline__ int slot(int g) const { return (x - (kXcds * g * over_G >> 16)) * P + k; }
};

// partials that each instance of group g gets from a grid of `grid` workgroups
template <typename T>
__device__ __forceinline__ int group_slots(const SDev<T> &S, int g, int grid)
{
    const int lo = kXcds * g * S.over_G >> 16, hi = (kXcds * (g + 1) + S.G - 1) * S.over_G >> 16;
    return (hi - lo) * (int)((unsigned)grid / kXcds);
}

// This thread's elements lo, lo + step, ... < hi of group g in interleaved
// vectors of `rows` rows that start at `base`; used: tiles of the earlier groups.
struct Walk {
    int base, lo, hi, step;
    // one group (of few instances), every workgroup on all of it
    __device__ __forceinline__ explicit Walk(int len)
        : base(0), lo((int)(blockIdx.x * kBlock + threadIdx.x)), hi(len), step((int)(gridDim.x * kBlock))
    {
    }
    __device__ __forceinline__ Walk(const Share &w, int g, int rows, int &used)
    {
        const int len = rows << w.lgW;
        const unsigned tiles = (unsigned)(len + kBlock - 1) / kBlock;
        const int at = kXcds * g, a = max(w.x * w.G, at) - at, b = min((w.x + 1) * w.G, at + kXcds) - at;
        const int t0 = (int)(tiles * a / kXcds), t1 = (int)(tiles * b / kXcds);
        int first = w.k;
        if (used) {
            first -= used % w.P;
            if (first < 0) first += w.P;
        }
        used += t1 - t0;
        base = g * len;
        lo = base + (t0 + first) * kBlock + (int)threadIdx.x;
        hi = base + min(t1 * kBlock, len);
        step = w.P * kBlock;
    }
    // whether the workgroup has any element
    __device__ __forceinline__ bool any() const { return lo - (int)threadIdx.x < hi; }
};

// the partials of a workgroup without elements of a group, as store_inst_partials stores them
template <int NV>
__device__ __forceinline__ void store_zero_partials(int W, int b0, int slot, int slots, double *out)
{
    const int t = (int)threadIdx.x;
    if (t >= W) return;
#pragma unroll
    for (int k = 0; k < NV; ++k) out[((size_t)(b0 + t) * slots + slot) * NV + k] = 0.0;
}

// The buffer that a group's lanes gather from: each lane's own c where it
// takes part, and the first such lane's where it does not (finished and padded
// instances compute with the others, on lines that are fetched anyway).
__device__ __forceinline__ int gather_buffer(unsigned long long part, bool mine, int c)
{
    const int first = __builtin_amdgcn_readlane(c, (int)__builtin_ctzll(part));
    return mine ? c : first;
}

// K~ x' for every instance fused with the dual step.
// The step's own operands are loaded before the row's product so their
// latency overlaps the gathers.  Workgroup 0 lowers the check gate (this
// slot's step decisions raise it).  W = 0 (here and in sk_update): at most four
// instances, in one group, which takes the plain walk and whose lanes of
// finished instances have nothing to load for others.  By eighths and with the
// groups' set-up, one instance of 3e5 columns took 44 us here, with these 35.
template <typename T, int W>
__global__ __launch_bounds__(kBlock) void sk_dual(SDev<T> S)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *S.gate = 0;
    const Dev<T> &d = S.d;
    const Share w(S);
    const int b = w.column(), g0 = W ? w.g0 : 0, g1 = W ? w.g1 : 0;
    int used = 0;
    for (int g = g0; g <= g1; ++g) {
        Walk r = W ? Walk(w, g, S.m, used) : Walk(S.m << S.lgW);
        if (W && !r.any()) {   // the same for the whole workgroup
            store_zero_partials<2>(w.W, g * w.W, w.slot(g), (int)gridDim.x, d.part_dual);
            continue;
        }
        const Ctl *ctl = S.ctl + g * w.W + b;
        double v[2] = {0.0, 0.0};
        const bool run = !ctl->done;
        const int c = ctl->cur;
        int cx = c;
        if constexpr (W > 0) {
            const unsigned long long part = __ballot(run);   // the wavefront holds every instance of the group
            if (!part) continue;   // all finished: their partials are not read
            cx = gather_buffer(part, run, c);
        } else if (!run) {
            r.hi = 0;
        }
        const T *x = pick(d.xb, cx ^ 1) + ((size_t)g * S.n << S.lgW);
        const T *y = pick(d.yb, c), *kx = pick(d.Kxb, c);
        T *yn = pick(d.yb, c ^ 1), *kxn = pick(d.Kxb, c ^ 1);
        const T sigma = (T)(ctl->eta * ctl->omega);
        for (int e = r.lo; e < r.hi; e += r.step) {
            const int i = (e - r.base) >> S.lgW;
            const T yo = y[e], ko = kx[e], qi = d.qs[e];
            const T s = shared_row<T, W>(S.kci, S.kv, x, S.krp[i], S.krp[i + 1], S.lgW, b);
            // the dual step of DualEpi
            T val = yo + sigma * (qi - T(2) * s + ko);
            if (i >= S.m1 && val < T(0)) val = T(0);
            if (W && !run) continue;
            yn[e] = val;
            kxn[e] = s;
            const double dd = (double)val - (double)yo;
            v[0] += dd * dd;
            v[1] += dd * ((double)s - (double)ko);
        }
        store_inst_partials<2>(v, w.W, g * w.W, W ? w.slot(g) : (int)blockIdx.x, (int)gridDim.x, d.part_dual);
    }
}

// one workgroup per instance
template <typename T>
__global__ __launch_bounds__(kBlock) void sk_step_decide(SDev<T> S)
{
    const int b = (int)blockIdx.x, g = b >> S.lgW;
    Ctl *ctl = S.ctl + b;
    if (ctl->done) {
        if (threadIdx.x == 0) ctl->mode = MODE_NONE;
        return;
    }
    double a[1], c2[2];
    block_sum_partials<1>(S.d.part_primal + (size_t)b * S.grid, group_slots(S, g, S.grid), a);
    block_sum_partials<2>(S.d.part_dual + 2 * (size_t)b * S.grid_m, group_slots(S, g, S.grid_m), c2);
    if (threadIdx.x == 0) {
        step_decision(ctl, a[0], c2[0], c2[1]);
        if (ctl->mode != MODE_NONE) atomicExch(S.gate, 1);
    }
}

// K~' y' for every accepted instance fused with the averages and the next
// primal trial (or, after a rejection, the new trial from the same point);
// the m-side averages follow in the same walk.
template <typename T, int W>
__global__ __launch_bounds__(kBlock) void sk_update(SDev<T> S)
{
    const Dev<T> &d = S.d;
    const Share sh(S);
    const int b = sh.column(), g0 = W ? sh.g0 : 0, g1 = W ? sh.g1 : 0;
    int used_n = 0, used_m = 0;
    for (int g = g0; g <= g1; ++g) {
        const Walk rn = W ? Walk(sh, g, S.n, used_n) : Walk(S.n << S.lgW);
        const Walk rm = W ? Walk(sh, g, S.m, used_m) : Walk(S.m << S.lgW);
        if (W && !rn.any() && !rm.any()) {
            store_zero_partials<1>(sh.W, g * sh.W, sh.slot(g), (int)gridDim.x, d.part_primal);
            continue;
        }
        const Ctl *ctl = S.ctl + g * sh.W + b;
        double v[1] = {0.0};
        const bool run = !ctl->done, accepted = run && ctl->accepted;
        if (W && !__ballot(run)) continue;   // the wavefront holds every instance of the group: all finished
        const int c = ctl->cur;
        const T tau = (T)(ctl->eta / ctl->omega);
        if (run && !accepted)
            for (int e = rn.lo; e < rn.hi; e += rn.step) primal_elem(d, c, tau, e, v[0]);
        const unsigned long long part = W ? __ballot(accepted) : accepted;
        if (part) {
            const T *x = pick(d.xb, c), *y = pick(d.yb, W ? gather_buffer(part, accepted, c) : c) + rm.base;
            T *kty = pick(d.KTyb, c), *xn = pick(d.xb, c ^ 1);
            const T w = (T)ctl->avg_w;
            const bool primal = ctl->mode == MODE_NONE;
            for (int e = rn.lo; e < rn.hi; e += rn.step) {
                const int j = (e - rn.base) >> S.lgW;
                const T xj = x[e], a = d.xa[e], bb = d.KTya[e];
                const T cj = d.cs[e], lj = d.ls[e], uj = d.us[e];
                const T s = shared_row<T, W>(S.tci, S.tv, y, S.trp[j], S.trp[j + 1], S.lgW, b);
                if (W && !accepted) continue;
                // the averages and next primal trial of UpdateEpi
                kty[e] = s;
                d.xa[e] = a + w * (xj - a);
                d.KTya[e] = bb + w * (s - bb);
                if (primal) {
                    const T nv = clampv(xj - tau * (cj - s), lj, uj);
                    xn[e] = nv;
                    const double dd = (double)nv - (double)xj;
                    v[0] += dd * dd;
                }
            }
            if (accepted)
                for (int e = rm.lo; e < rm.hi; e += rm.step) average_row(d, e, c, w);
        }
        store_inst_partials<1>(v, sh.W, g * sh.W, W ? sh.slot(g) : (int)blockIdx.x, (int)gridDim.x, d.part_primal);
    }
}

// The 18 check sums and 4 ray sums of every instance in a check, over the
// same walk as sk_update.  Gated inside the solve loop.
template <typename T>
__global__ __launch_bounds__(kBlock) void sk_check_reduce(SDev<T> S, int gated)
{
    if (gated && *S.gate == 0) return;
    const Dev<T> &d = S.d;
    const Share w(S);
    int used_n = 0, used_m = 0;
    for (int g = w.g0; g <= w.g1; ++g) {
        const Walk rn(w, g, S.n, used_n), rm(w, g, S.m, used_m);
        const Ctl *ctl = S.ctl + g * w.W + w.column();
        double s[kCheckSums], r[kRaySums];
#pragma unroll
        for (int k = 0; k < kCheckSums; ++k) s[k] = 0.0;
#pragma unroll
        for (int k = 0; k < kRaySums; ++k) r[k] = 0.0;
        if (ctl->mode != MODE_NONE && !ctl->done) {
            const int c = ctl->cur, m1 = rm.base + (S.m1 << S.lgW);
            const T *x = pick(d.xb, c), *kty = pick(d.KTyb, c), *y = pick(d.yb, c), *kx = pick(d.Kxb, c);
            for (int e = rn.lo; e < rn.hi; e += rn.step) {
                col_sums(d, e, x, kty, s);
                col_sums(d, e, (const T *)d.xa, (const T *)d.KTya, s + 9);
                ray_col_sums(d, e, x, kty, r);
            }
            for (int e = rm.lo; e < rm.hi; e += rm.step) {
                row_sums(d, e, m1, y, kx, s);
                row_sums(d, e, m1, (const T *)d.ya, (const T *)d.Kxa, s + 9);
                ray_row_sums(d, e, m1, y, kx, r);
            }
        }
        store_inst_partials<kCheckSums>(s, w.W, g * w.W, w.slot(g), (int)gridDim.x, d.part_check);
        store_inst_partials<kRaySums>(r, w.W, g * w.W, w.slot(g), (int)gridDim.x, d.part_ray);
    }
}

// one workgroup per instance
template <typename T>
__global__ __launch_bounds__(kBlock) void sk_check_decide(SDev<T> S, int gated)
{
    if (gated && *S.gate == 0) return;
    const int b = (int)blockIdx.x, np = group_slots(S, b >> S.lgW, S.grid);
    Ctl *ctl = S.ctl + b;
    if (ctl->mode == MODE_NONE || ctl->done) return;
    double Sm[kCheckSums], R[kRaySums];
    block_sum_partials<kCheckSums>(S.d.part_check + (size_t)kCheckSums * b * S.grid, np, Sm);
    block_sum_partials<kRaySums>(S.d.part_ray + (size_t)kRaySums * b * S.grid, np, R);
    if (threadIdx.x == 0) check_decision(ctl, Sm, R, S.Nq[b], S.Nc[b]);
}

// restart copies, output copy and next primal trial of every instance in a
// check; its |x'' - x|^2 partial replaces the one sk_update left for it
template <typename T>
__global__ __launch_bounds__(kBlock) void sk_check_apply(SDev<T> S, int gated)
{
    if (gated && *S.gate == 0) return;
    const Dev<T> &d = S.d;
    const Share w(S);
    int used_n = 0, used_m = 0;
    for (int g = w.g0; g <= w.g1; ++g) {
        const Walk rn(w, g, S.n, used_n), rm(w, g, S.m, used_m);
        const Ctl *ctl = S.ctl + g * w.W + w.column();
        double v[1] = {0.0};
        if (ctl->mode != MODE_NONE) {
            const int c = ctl->cur, rt = ctl->restart_to, co = ctl->copy_out, sel = ctl->out_sel;
            const int np = ctl->need_primal;
            const T tau = (T)(ctl->eta / ctl->omega);
            for (int e = rn.lo; e < rn.hi; e += rn.step) apply_col(d, e, c, rt, co, sel, np, tau, v[0]);
            for (int e = rm.lo; e < rm.hi; e += rm.step) apply_row(d, e, c, rt, co, sel);
        }
        store_inst_partials<1>(v, w.W, g * w.W, w.slot(g), (int)gridDim.x, d.part_primal, S.ctl);
    }
}

// a plain product for every instance (start, resume and the anchor's products)
template <typename T, int W, int WHICH>
__global__ __launch_bounds__(kBlock) void sk_product(SDev<T> S, const T *__restrict__ in, T *__restrict__ out)
{
    const int *rp = WHICH ? S.trp : S.krp, *ci = WHICH ? S.tci : S.kci;
    const T *v = WHICH ? S.tv : S.kv;
    const Share w(S);
    const int b = w.column();
    int used = 0;
    for (int g = w.g0; g <= w.g1; ++g) {
        const Walk r(w, g, WHICH ? S.n : S.m, used);
        const T *x = in + ((size_t)g * (WHICH ? S.m : S.n) << S.lgW);
        for (int e = r.lo; e < r.hi; e += r.step) {
            const int i = (e - r.base) >> S.lgW;
            out[e] = shared_row<T, W>(ci, v, x, rp[i], rp[i + 1], S.lgW, b);
        }
    }
}

template <typename T>
__global__ void sk_start(SDev<T> S, const double *xs, const double *ys)
{
    const Dev<T> &d = S.d;
    const int e = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (e < d.n) {
        const double v0 = xs ? xs[e] * d.Dc[e] : 0.0;
        d.xb[0][e] = clampv((T)v0, d.ls[e], d.us[e]);
    }
    if (e < d.m) {
        double v0 = ys ? ys[e] * d.Dr[e] : 0.0;
        if (((e >> S.lgW) % S.m) >= S.m1 && v0 < 0.0) v0 = 0.0;
        d.yb[0][e] = (T)v0;
    }
}

template <typename T>
__global__ void sk_extract(const T *src, int lgW, int b, double *dst, int rows)
{
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i < rows) dst[i] = (double)src[((size_t)i << lgW) + b];
}

template <typename T>
__global__ void sk_insert(const double *src, int lgW, int b, T *dst, int rows)
{
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i < rows) dst[((size_t)i << lgW) + b] = (T)src[i];
}

__global__ void sk_set_final(Ctl *ctl, int Bp, int status)
{
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i < Bp && !ctl[i].done) {
        ctl[i].mode = MODE_FINAL;
        ctl[i].final_status = status;
    }
}

// ----------------------------------------------------------------------------

namespace {
inline dim3 nblocks(int64_t len) { return dim3((unsigned)((len + kBlock - 1) / kBlock > 0 ? (len + kBlock - 1) / kBlock : 1)); }
}  // namespace

// f of the width that the products are built for (0: any; 32 in FP32 alone),
// as lp_shared_load chooses it
template <typename T, typename F>
void with_width(int lgW, F f)
{
    if constexpr (sizeof(T) == 4) {
        if (lgW == 5) return f(std::integral_constant<int, 32>{});
    }
    if (lgW == 4) return f(std::integral_constant<int, 16>{});
    if (lgW == 3) return f(std::integral_constant<int, 8>{});
    f(std::integral_constant<int, 0>{});
}

template <typename T>
hipError_t launch_shared_check(const SDev<T> &S, int gated, hipStream_t s)
{
    hipLaunchKernelGGL(sk_check_reduce<T>, dim3(S.grid), dim3(kBlock), 0, s, S, gated);
    hipLaunchKernelGGL(sk_check_decide<T>, dim3(S.Bp), dim3(kBlock), 0, s, S, gated);
    hipLaunchKernelGGL(sk_check_apply<T>, dim3(S.grid), dim3(kBlock), 0, s, S, gated);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_shared_apply(const SDev<T> &S, hipStream_t s)
{
    hipLaunchKernelGGL(sk_check_apply<T>, dim3(S.grid), dim3(kBlock), 0, s, S, 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_shared_slot(const SDev<T> &S, hipStream_t s)
{
    with_width<T>(S.lgW, [&](auto w) {
        hipLaunchKernelGGL((sk_dual<T, decltype(w)::value>), dim3(S.grid_m), dim3(kBlock), 0, s, S);
        hipLaunchKernelGGL(sk_step_decide<T>, dim3(S.Bp), dim3(kBlock), 0, s, S);
        hipLaunchKernelGGL((sk_update<T, decltype(w)::value>), dim3(S.grid), dim3(kBlock), 0, s, S);
    });
    return launch_shared_check<T>(S, 1, s);
}

template <typename T>
hipError_t launch_shared_product(const SDev<T> &S, int which, const T *in, T *out, hipStream_t s)
{
    const int64_t total = (int64_t)(which ? S.d.n : S.d.m);
    if (total <= 0) return hipSuccess;
    const dim3 g((unsigned)(kXcds * std::min<int64_t>((total + kBlock * kXcds - 1) / (kBlock * kXcds), 1024)));
    with_width<T>(S.lgW, [&](auto w) {
        constexpr int W = decltype(w)::value;
        if (which == 0) hipLaunchKernelGGL((sk_product<T, W, 0>), g, dim3(kBlock), 0, s, S, in, out);
        else hipLaunchKernelGGL((sk_product<T, W, 1>), g, dim3(kBlock), 0, s, S, in, out);
    });
    return hipGetLastError();
}

template <typename T>
hipError_t launch_shared_extract(const T *src, int lgW, int b, double *dst, int rows, hipStream_t s)
{
    const int W = 1 << lgW;
    src += (size_t)(b >> lgW) * rows << lgW;   // b's group
    if (rows > 0) hipLaunchKernelGGL(sk_extract<T>, nblocks(rows), dim3(kBlock), 0, s, src, lgW, b & (W - 1), dst, rows);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_shared_insert(const double *src, int lgW, int b, T *dst, int rows, hipStream_t s)
{
    const int W = 1 << lgW;
    dst += (size_t)(b >> lgW) * rows << lgW;
    if (rows > 0) hipLaunchKernelGGL(sk_insert<T>, nblocks(rows), dim3(kBlock), 0, s, src, lgW, b & (W - 1), dst, rows);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_shared_start(const SDev<T> &S, const double *xs, const double *ys, hipStream_t s)
{
    hipLaunchKernelGGL(sk_start<T>, nblocks(std::max(S.d.n, S.d.m)), dim3(kBlock), 0, s, S, xs, ys);
    return hipGetLastError();
}

hipError_t launch_shared_set_final(Ctl *ctl, int Bp, int status, hipStream_t s)
{
    hipLaunchKernelGGL(sk_set_final, nblocks(Bp), dim3(kBlock), 0, s, ctl, Bp, status);
    return hipGetLastError();
}

#define PDLP_SHARED_INSTANTIATE(T)                                                                                 \
    template hipError_t launch_shared_slot<T>(const SDev<T> &, hipStream_t);                                       \
    template hipError_t launch_shared_check<T>(const SDev<T> &, int, hipStream_t);                                 \
    template hipError_t launch_shared_apply<T>(const SDev<T> &, hipStream_t);                                      \
    template hipError_t launch_shared_product<T>(const SDev<T> &, int, const T *, T *, hipStream_t);               \
    template hipError_t launch_shared_start<T>(const SDev<T> &, const double *, const double *, hipStream_t);      \
    template hipError_t launch_shared_extract<T>(const T *, int, int, double *, int, hipStream_t);                 \
    template hipError_t launch_shared_insert<T>(const double *, int, int, T *, int, hipStream_t);

PDLP_SHARED_INSTANTIATE(double)
PDLP_SHARED_INSTANTIATE(float)

}  // namespace pdlp
