// Amul / Tmul and the conjugate-gradient solvers.
//
// Amul is the sparse product of the lduMatrix (the "SpMVM (Amul + Tmul)" row of
// the kernel time breakdown, Sec. 4.3).  It is HBM-bound (about 0.15 flop per
// byte), so it is a pure streaming kernel: no matrix cores, coalesced 64-wide
// streams of columns and values, the x gather served from L2, and an
// atomic-free row ownership (each row is summed by exactly one lane).
//
// PCG with the diagonal preconditioner (Appendix A) runs as two or three fused
// kernels per iteration, with every scalar (rho, alpha, beta, residual) kept in
// device memory and a device "done" flag that freezes the iteration at the
// first iterate meeting the tolerance; the host only reads the scalars every
// check_every iterations, instead of synchronising after each kernel as the
// paper's executor does (Sec. 4.3, CUDA API statistics).
#include "device.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ldu {

// ---------------------------------------------------------------- products
// NT: the result is stored nontemporally (level 0 above kStreamNtCells)
template <bool CMP, typename T, bool NT = false>
__global__ void __launch_bounds__(kBlock) k_amul(SellView<T> A, const T *__restrict__ x,
                                                 T *__restrict__ y) {
    const int lane = threadIdx.x & 63;
    for_each_slice<product_cap<CMP, T>()>(A.nslices, [&](int64_t s) {
        const int64_t p = s * kWave + lane;
        if (p < A.n) {
            const int32_t i = sv_row<CMP>(A, p);
            vst<NT>(y + i, sell_row<CMP>(A, s, lane, i, Direct<T>{x}));
        }
    });
}

void launch_amul(const SellView<double> &A, const double *x, double *y, hipStream_t st) {
    const int G = stream_grid_slices(A.nslices);
    if (A.pdeg) k_amul<true, double><<<G, kBlock, 0, st>>>(A, x, y);
    else if (A.n > kStreamNtCells) k_amul<false, double, true><<<G, kBlock, 0, st>>>(A, x, y);
    else k_amul<false, double><<<G, kBlock, 0, st>>>(A, x, y);
    HIP_CHECK(hipGetLastError());
}
void launch_amul32(const SellView<float> &A, const float *x, float *y, hipStream_t st) {
    const int G = stream_grid_slices(A.nslices);
    if (A.pdeg) k_amul<true, float><<<G, kBlock, 0, st>>>(A, x, y);
    else k_amul<false, float><<<G, kBlock, 0, st>>>(A, x, y);
    HIP_CHECK(hipGetLastError());
}

// ---------------------------------------------------------------- scalars
__global__ void k_init_scalars(DevScalars *ds, double tol, int max_iter) {
    DevScalars z{};
    z.tol = tol;
    z.max_iter = max_iter;
    *ds = z;
}
__global__ void k_set_done(DevScalars *ds, int done) { ds->done = done; }
void set_done(ldu_t *h, int done, hipStream_t st) {
    k_set_done<<<1, 1, 0, st>>>(h->dev, done);
    HIP_CHECK(hipGetLastError());
}

void set_scalars_for_solve(ldu_t *h, double tol, int max_iter, hipStream_t st) {
    k_init_scalars<<<1, 1, 0, st>>>(h->dev, tol, max_iter);
    HIP_CHECK(hipGetLastError());
}

void read_scalars(ldu_t *h, hipStream_t st) {
    HIP_CHECK(hipMemcpyAsync(h->host, h->dev, sizeof(DevScalars), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
}

// Iterations to launch before the host looks at the scalars again: as many as
// the solve still needs at the rate it has had from res0 to res in `steps`
// iterations, at least one and at most `most` (which the iterations left
// bound too); `first` while there is no rate.  Iterations launched past the
// last one store nothing, but their kernels cost a launch of 2.4 us each, and
// those of the small levels, which test the stop flag before their stores, the
// loads of their rows as well: 51, 113 and 125 us an iteration of CG + V-cycle
// on 32^3, 64^3 and 128^3 pairwise, 135, 208 and 260 us a default GAMG cycle.
int next_batch(double res0, double res, int steps, double tol, int first, int most) {
    most = std::max(1, most);
    if (steps < 1) return std::min(first, most);
    if (!(res > tol) || !(res < res0) || !(tol > 0.0)) return most;
    const double left = std::log(res / tol) / std::log(res0 / res) * steps;
    return left < most ? std::max(1, (int)std::ceil(left)) : most;
}

void ensure_hist(ldu_t *h, int64_t entries) {
    // the device history keeps the first kMaxHistory entries of a solve; the
    // epilogues write entry k only while k < hist_cap
    if (entries > kMaxHistory) entries = kMaxHistory;
    if (entries < 1) entries = 1;
    if (entries <= h->hist_cap) return;
    if (h->hist) h->arena.release(h->hist);
    h->hist = nullptr;
    h->hist_cap = 0;
    h->hist = static_cast<double *>(h->arena.alloc_own(sizeof(double) * (size_t)entries));
    h->hist_cap = (int)entries;
}

void copy_history(ldu_t *h, ldu_stats *stats, int count, hipStream_t st) {
    if (!stats) return;
    stats->history_count = 0;
    if (!stats->history || stats->history_len <= 0 || count <= 0) return;
    int m = count < stats->history_len ? count : stats->history_len;
    if (m > h->hist_cap) m = h->hist_cap;
    HIP_CHECK(hipMemcpyAsync(stats->history, h->hist, sizeof(double) * m,
                             hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    stats->history_count = m;
}

// ---------------------------------------------------------------- residual
// r = b - A x, plus ||r||^2, ||b||^2 and, when P is set, p = D^-1 r (or r)
// and rho = r.p; MAXABS adds ||r||_inf.  Epilogue modes:
//   kResPlain  : scalars only (true residual, CG (re)start)
//   kResCycle  : GAMG/refinement outer loop, honours and sets the done flag
enum { kResPlain = 0, kResCycle = 1 };

template <bool CMP, bool P, bool MAXABS>
__global__ void __launch_bounds__(kBlock)
k_residual(SellView<double> A, const double *__restrict__ b, const double *__restrict__ x,
           double *__restrict__ r, double *__restrict__ p, int precond, int gated,
           double *partials, const DevScalars *ds) {
    if (gated && ds->done) return;
    const int lane = threadIdx.x & 63;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};  // rr, bb, rho, maxabs
    for_each_slice<product_cap<CMP, double>()>(A.nslices, [&](int64_t s) {
        const int64_t pos = s * kWave + lane;
        if (pos < A.n) {
            const int32_t i = sv_row<CMP>(A, pos);
            const double bi = b[i];
            const double ri = bi - sell_row<CMP>(A, s, lane, i, Direct<double>{x});
            r[i] = ri;
            acc[0] += ri * ri;
            acc[1] += bi * bi;
            if (P) {
                const double zi = precond ? ri / A.diag[i] : ri;
                p[i] = zi;
                acc[2] += ri * zi;
            }
            if (MAXABS) acc[3] = fmax(acc[3], fabs(ri));
        }
    });
    block_partials<4, 1>(acc, partials);
}

// epilogue of the residual: scalars, history entry and, for the outer loop
// of GAMG and of the refinement (kResCycle), the convergence decision
struct EpiResidual {
    int mode, write_hist, has_p;
    double *hist;
    int hist_cap;
    __device__ bool active(const DevScalars *ds) const {
        return mode != kResCycle || !ds->done;
    }
    __device__ void operator()(const double *t, DevScalars *ds) const {
        ds->rr = t[0];
        ds->bb = t[1];
        ds->bnorm = sqrt(t[1]);
        ds->maxabs = t[3];
        if (has_p) ds->rho = t[2];
        ds->x_pending = 0;  // a (re)start owes no solution update
        // b = 0 gives 0; a non-finite b or x gives a non-finite residual
        // (a NaN norm of b must not read as b = 0)
        const double res = ds->bnorm == 0.0 ? 0.0 : sqrt(t[0]) / ds->bnorm;
        ds->res = res;
        const int it = ds->iters;
        if (write_hist && hist && it < hist_cap) hist[it] = res;
        if (mode == kResCycle) {
            if (!isfinite(res)) {
                ds->status = LDU_ERR_NAN;
                ds->done = kFailed;
            } else if (res <= ds->tol) {
                ds->done = kConverged;
            } else if (it >= ds->max_iter) {
                ds->done = kMaxIter;
            } else {
                ds->iters = it + 1;
            }
        }
    }
};

template <bool P, bool MAXABS>
static void launch_residual(ldu_t *h, const SellView<double> &A, const double *b, const double *x,
                            double *r, double *p, int precond, int mode, bool write_hist,
                            hipStream_t st) {
    const int G = stream_grid_slices(A.nslices);
    if (A.pdeg)
        k_residual<true, P, MAXABS><<<G, kBlock, 0, st>>>(A, b, x, r, p, precond,
                                                          mode == kResCycle, h->partials, h->dev);
    else
        k_residual<false, P, MAXABS><<<G, kBlock, 0, st>>>(A, b, x, r, p, precond,
                                                           mode == kResCycle, h->partials, h->dev);
    launch_finalize<4, 1>(h->partials, G, h->dev,
                          EpiResidual{mode, write_hist ? 1 : 0, P ? 1 : 0, h->hist, h->hist_cap}, st);
    HIP_CHECK(hipGetLastError());
}

void launch_residual_cycle(ldu_t *h, const SellView<double> &A, const double *b,
                           const double *x, double *r, bool maxabs, int grid,
                           hipStream_t st) {
    (void)grid;
    if (maxabs) launch_residual<false, true>(h, A, b, x, r, nullptr, 0, kResCycle, true, st);
    else launch_residual<false, false>(h, A, b, x, r, nullptr, 0, kResCycle, true, st);
}

void launch_residual_plain(ldu_t *h, const SellView<double> &A, const double *b,
                           const double *x, double *r, bool write_hist, int grid,
                           hipStream_t st) {
    (void)grid;
    launch_residual<false, false>(h, A, b, x, r, nullptr, 0, kResPlain, write_hist, st);
}

double residual_norm(ldu_t *h, const Level &L, bool tr, const double *b, const double *x,
                     double *r_out, hipStream_t st) {
    launch_residual<false, false>(h, L.A.view(tr), b, x, r_out, nullptr, 0, kResPlain, false, st);
    read_scalars(h, st);
    return h->host->res;
}

// ---------------------------------------------------------------- PCG, FP64
// q = A p and p.q -> alpha = rho / p.q
template <bool CMP, bool NT = false>
__global__ void __launch_bounds__(kBlock)
k_pcg_q(SellView<double> A, const double *__restrict__ p, double *__restrict__ q,
        double *partials, const DevScalars *ds) {
    if (ds->done) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice<product_cap<CMP, double>()>(A.nslices, [&](int64_t s) {
        const int64_t pos = s * kWave + lane;
        if (pos < A.n) {
            const int32_t i = sv_row<CMP>(A, pos);
            const double qi = sell_row<CMP>(A, s, lane, i, Direct<double>{p});
            vst<NT>(q + i, qi);
            acc[0] += p[i] * qi;
        }
    });
    block_partials<1>(acc, partials);
}

void launch_product_dot(ldu_t *h, const SellView<double> &A, const double *p, double *q,
                               int grid, const DevScalars *ds, hipStream_t st) {
    if (A.pdeg) k_pcg_q<true><<<grid, kBlock, 0, st>>>(A, p, q, h->partials, ds);
    else if (A.n > kStreamNtCells)
        k_pcg_q<false, true><<<grid, kBlock, 0, st>>>(A, p, q, h->partials, ds);
    else k_pcg_q<false><<<grid, kBlock, 0, st>>>(A, p, q, h->partials, ds);
}

// iteration count, residual history and convergence test after the r update
// of a CG whose preconditioned residual comes from a V-cycle
struct EpiConverge {
    double *hist;
    int hist_cap;
    __device__ bool active(const DevScalars *ds) const { return !ds->done; }
    __device__ void operator()(const double *t, DevScalars *ds) const {
        const int it = ds->iters + 1;
        ds->iters = it;
        ds->rr = t[0];
        const double res = sqrt(t[0]) / ds->bnorm;
        ds->res = res;
        if (hist && it < hist_cap) hist[it] = res;
        if (!isfinite(res)) {
            ds->status = LDU_ERR_NAN;
            ds->done = kFailed;
        } else if (res <= ds->tol) {
            ds->done = kConverged;
        } else if (it >= ds->max_iter) {
            ds->done = kMaxIter;
        }
    }
};

void launch_converge(ldu_t *h, const double *partials, int grid, hipStream_t st) {
    k_finalize<1, 0, EpiConverge><<<1, kBlock, 0, st>>>(partials, grid, h->dev,
                                                        EpiConverge{h->hist, h->hist_cap});
}

// An iteration of diagonal CG is two or three kernels.  Scalars travel with
// them: the direction update takes ||r||^2 and r.z (the
// convergence test and beta) from the partials of the residual update and
// passes dev[0] on to dev[1], the residual update takes p.q (alpha) from the
// product's and passes dev[1] on to dev[0].  As separate one-block reductions
// these two were 9 us of a 40 us iteration at 1M cells and two of five
// launches of an 18 us one at 32,768; diagonal CG at 32^3 4.89 -> 2.87 ms, at
// 100^3 29.5 -> 26.3 ms, at 150^3 115.2 -> 108.9 ms.  The partials of p.q are
// the first kMaxGrid values, those of ||r||^2 and r.z the next two.
//
// Up to kFusedCgCells the product forms the new direction itself, also in its
// gathers (p_j = z_j + beta p_j, the same bits as the owner stores), and the
// iteration's x += alpha p rides along: the level's vectors sit in the caches
// there, so a second gather costs less than a kernel.  Above, the direction
// update is its own kernel.
//
// what the solve of one handle passes to its step kernels
struct StepHistory {
    double *hist;
    int hist_cap;
};

// The residual update's sums (||r||^2 and r.z; PBiCG: z.rt), taken by every
// thread of the kernel that follows: iteration count, history, convergence
// test and beta, the same decisions in every thread.  Block 0's first thread
// writes the scalars to `out`, which other blocks do not read (in place only
// for a launch of one block).  Only the fields a thread needs are held in
// registers: a copy of the struct went to scratch memory and cost every wave
// several microseconds.
template <bool BICG>
__device__ __forceinline__ Step step_converge(int mode, const double *__restrict__ partials,
                                              int nblocks, const DevScalars *in, DevScalars *out,
                                              const StepHistory &h) {
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const int done0 = in->done;
    Step st{in->alpha, in->beta, done0 == 0};
    if (done0 || mode != kStepReduce) {
        if (lead && in != out) *out = *in;
        return st;
    }
    const double rho = in->rho, bnorm = in->bnorm, tol = in->tol;
    const int it = in->iters + 1, max_iter = in->max_iter;
    double t[2];
    sum_partials<2>(partials, nblocks, t);
    const double res = sqrt(t[0]) / bnorm;
    int done = kRunning, status = 0;
    if (!isfinite(res)) {
        done = kFailed;
        status = LDU_ERR_NAN;
    } else if (res <= tol) {
        done = kConverged;
    } else if (it >= max_iter) {
        done = kMaxIter;
    } else if (BICG && (!isfinite(t[1]) || fabs(t[1]) <= 1e-300)) {
        done = kFailed;
        status = LDU_ERR_BREAKDOWN;
    }
    st.go = done == kRunning;
    st.beta = t[1] / rho;
    if (lead) {
        if (in != out) *out = *in;
        out->iters = it;
        out->rr = t[0];
        out->res = res;
        if (h.hist && it < h.hist_cap) h.hist[it] = res;
        if (st.go) {
            out->beta = st.beta;
            out->rho = t[1];
            out->x_pending = 0;  // the direction update applies it now
        } else {
            out->done = done;
            if (done == kFailed) out->status = status;
        }
    }
    return st;
}

// the convergence step for the host, which reads the scalars next
template <bool BICG>
__global__ void __launch_bounds__(kBlock)
k_step_converge(const double *partials, int nblocks, DevScalars *ds, StepHistory h) {
    step_converge<BICG>(kStepReduce, partials, nblocks, ds, ds, h);
}

// p_j = z_j + beta p_j
struct NewDirection {
    const double *z, *p;
    double beta;
    bool first;
    __device__ __forceinline__ double operator()(int32_t j) const {
        return first ? z[j] : z[j] + beta * p[j];
    }
};

// x += alpha p (the last iteration's); p2 = z + beta p; q = A p2; p2.q
template <bool CMP>
__global__ void __launch_bounds__(kBlock)
k_cg_pq(SellView<double> A, const double *__restrict__ z, const double *__restrict__ p,
        double *__restrict__ p2, double *__restrict__ x, double *__restrict__ q,
        double *partials, int nblocks, int mode, const DevScalars *__restrict__ in,
        DevScalars *__restrict__ out, StepHistory hist) {
    const int lane = threadIdx.x & 63;
    const bool first = mode == kStepFirst;
    Step s{};
    double acc[1] = {0.0};
    auto finish = [&](int32_t i, double pi, double pold, double qi) {
        if (!first) x[i] = x[i] + s.alpha * pold;
        p2[i] = pi;
        q[i] = qi;
        acc[0] += pi * qi;
    };
    if constexpr (CMP) {
        s = step_converge<false>(mode, partials + kMaxGrid, nblocks, in, out, hist);
        if (!s.go) return;
        const NewDirection np{z, p, s.beta, first};
        for_each_slice(A.nslices, [&](int64_t sl) {
            const int64_t pos = sl * kWave + lane;
            if (pos < A.n) {
                const int32_t i = A.perm[pos];
                const double pi = np(i);
                double qi = A.diag[i] * pi;
                cmp_entries<kCmpBatch>(A, sl, lane, np,
                                       [&](int32_t, double v, double pv) { qi = qi + v * pv; });
                finish(i, pi, first ? 0.0 : p[i], qi);
            }
        });
    } else {
        // a wave's slice is loaded, gathers included, before the scalars of
        // the step are there: of this kernel's chain of round trips at small
        // sizes (scalars, partials; slice start, entries, gathers) the two
        // halves overlap
        constexpr int B = 8;
        const SliceWalkRange r = slice_walk_range(A.nslices, gridDim.x);
        int32_t c[B], cb[B];
        double v[B], zv[B], pv[B], di = 0.0, zi = 0.0, po = 0.0;
        int w = 0;
        auto load = [&](auto c16, int64_t sl, int k) {
            constexpr bool C16 = decltype(c16)::value;
            const PlainWalk<C16, double> pw(A, sl, lane);
            w = pw.w;
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (k + u < w) pw.load(k + u, c[u], cb[u], v[u]);
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (k + u < w) {
                    c[u] = PlainWalk<C16, double>::column(c[u], cb[u]);
                    zv[u] = z[c[u]];
                    if (!first) pv[u] = p[c[u]];
                }
        };
        auto load_any = [&](int64_t sl, int k) {
            if (A.c16) load(std::true_type{}, sl, k);
            else load(std::false_type{}, sl, k);
        };
        auto load_row = [&](int64_t sl) {
            const int64_t i = sl * kWave + lane;
            if (i >= A.n) return;
            di = A.diag[i];
            zi = z[i];
            if (!first) po = p[i];
            load_any(sl, 0);
        };
        const int64_t step = r.Gx * kWavesPerBlock;
        int64_t sl = r.lo + r.j * kWavesPerBlock + r.w;
        if (sl < r.hi) load_row(sl);
        s = step_converge<false>(mode, partials + kMaxGrid, nblocks, in, out, hist);
        if (!s.go) return;
        const double beta = s.beta;
        for (; sl < r.hi; sl += step) {
            const int64_t i = sl * kWave + lane;
            if (i < A.n) {
                const double pi = first ? zi : zi + beta * po;
                double qi = di * pi;
                for (int k = 0;;) {
#pragma unroll
                    for (int u = 0; u < B; ++u)
                        if (k + u < w) qi = qi + v[u] * (first ? zv[u] : zv[u] + beta * pv[u]);
                    k += B;
                    if (k >= w) break;
                    load_any(sl, k);
                }
                finish((int32_t)i, pi, po, qi);
            }
            if (sl + step < r.hi) load_row(sl + step);
        }
    }
    block_partials<1>(acc, partials);
}

// x += alpha p (the last iteration's); p = z + beta p with z = D^-1 r.  p keeps
// the default cache policy even where the other vectors stream nontemporally
// (NT): the product gathers it next (c4's diagonal PCG: 1.05 -> 1.02 s per
// right-hand side).
template <bool NT>
__global__ void __launch_bounds__(kBlock)
k_cg_p(int32_t n, int64_t S, const double *__restrict__ D, const double *__restrict__ r,
       double *__restrict__ x, double *__restrict__ p, int precond, const double *partials,
       int nblocks, int mode, const DevScalars *in, DevScalars *out, StepHistory hist) {
    const Step s = step_converge<false>(mode, partials + kMaxGrid, nblocks, in, out, hist);
    if (!s.go || mode == kStepFirst) return;  // the first direction is z, there already
    const double alpha = s.alpha, beta = s.beta;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t sl) {
        const int64_t i = sl * kWave + lane;
        if (i < n) {
            const double pi = p[i];
            vst<NT>(x + i, vld<NT>(x + i) + alpha * pi);
            const double ri = vld<NT>(r + i);
            const double zi = precond ? ri / vld<NT>(D + i) : ri;
            p[i] = zi + beta * pi;
        }
    });
}

// r -= alpha q; ||r||^2 and r.D^-1 r; z = D^-1 r is stored for the two-kernel
// form (z given).  The iteration's x += alpha p waits for the direction
// update, which reads p anyway, or, when the solve stops in between, for
// k_x_pending: one read of p per iteration instead of two.
template <bool NT>
__global__ void __launch_bounds__(kBlock)
k_cg_r(int32_t n, int64_t S, const double *__restrict__ D, double *__restrict__ r,
       const double *__restrict__ q, double *__restrict__ z, int precond, double *partials,
       int nblocks, const DevScalars *in, DevScalars *out) {
    const Step s = step_alpha(partials, nblocks, in, out);
    if (!s.go) return;
    const double alpha = s.alpha;
    const int lane = threadIdx.x & 63;
    double acc[2] = {0.0, 0.0};
    for_each_slice(S, [&](int64_t sl) {
        const int64_t i = sl * kWave + lane;
        if (i < n) {
            const double ri = vld<NT>(r + i) - alpha * vld<NT>(q + i);
            vst<NT>(r + i, ri);
            const double zi = precond ? ri / vld<NT>(D + i) : ri;
            if (z) z[i] = zi;
            acc[0] += ri * ri;
            acc[1] += ri * zi;
        }
    });
    block_partials<2>(acc, partials + kMaxGrid);
}

// x += alpha p when the stopped solve's last iteration still owes it: alpha
// was formed (x_pending) but the direction update that applies it did not
// run.  The same expression as in the direction updates.
__global__ void __launch_bounds__(kBlock)
k_x_pending(int32_t n, int64_t S, double *__restrict__ x, const double *__restrict__ p,
            const DevScalars *ds) {
    if (!ds->x_pending) return;
    const double alpha = ds->alpha;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) x[i] = x[i] + alpha * p[i];
    });
}

void launch_x_pending(ldu_t *h, double *x, const double *p, int32_t n, int64_t S, int grid,
                      hipStream_t st) {
    k_x_pending<<<grid, kBlock, 0, st>>>(n, S, x, p, h->dev);
    HIP_CHECK(hipGetLastError());
}

__global__ void k_fill(double *a, int64_t n, double v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        a[i] = v;
}
static void fill(double *a, int64_t n, double v, hipStream_t st) {
    int64_t g = (n + kBlock - 1) / kBlock;
    g = g > 4096 ? 4096 : (g < 1 ? 1 : g);
    k_fill<<<(unsigned)g, kBlock, 0, st>>>(a, n, v);
}
void zero_vector(double *a, int64_t n, hipStream_t st) {
    fill(a, n, 0.0, st);
    HIP_CHECK(hipStreamSynchronize(st));
}

static void fill_stats_common(ldu_stats *stats) {
    if (!stats) return;
    stats->refinements = 0;
    stats->n_levels = 0;
    stats->history_count = 0;
}

// z and the second direction of the two-kernel forms.  The pointer that says
// that a set of arrays exists is set last, here and wherever a call allocates:
// a call that runs out of memory part way leaves the set as not there.
static void ensure_direction(ldu_t *h) {
    if (h->z) return;
    h->arena.reserve(2 * (sizeof(double) * (size_t)h->L0.n + 256));
    double *z = h->arena.get<double>(h->L0.n);
    h->p2 = h->arena.get<double>(h->L0.n);
    h->z = z;
}

int pcg_fp64(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
             ldu_stats *stats, hipStream_t st, bool own_hist) {
    const Level &L = h->L0;
    SellView<double> A = L.A.view(tr);
    // six vectors: x, r, p, q, D and the two-kernel form's z
    A.stream = L.A.bytes(sizeof(double)) + 6 * (int64_t)sizeof(double) * L.n > kCacheBytes;
    const int n = L.n;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    const int precond = o.precond ? 1 : 0;
    const bool nt = n > kStreamNtCells;
    // the allocation-free entry point has no room for the two-kernel form's
    // vectors; the results are the same bit for bit
    const bool fused = own_hist && n <= kFusedCgCells;
    if (fused) ensure_direction(h);
    // products on plain slices: blocks past the cap would only add zeros; the
    // residual update: see kCgBlocks
    const int Gq = A.pdeg ? G : std::min(G, kPlainF64ProductBlocks);
    const int Gr = cg_blocks(n, G);
    double *const p0 = fused ? h->z : h->p;  // where a (re)start's direction goes
    double *const pbuf[2] = {fused ? h->p2 : h->p, h->p};  // direction after j iterations: j & 1
    if (own_hist) ensure_hist(h, (int64_t)o.max_iter + 2);
    fill_stats_common(stats);
    set_scalars_for_solve(h, o.rel_tol, o.max_iter, st);
    launch_residual<true, false>(h, A, b, x, h->r, p0, precond, kResPlain, true, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        fill(x, n, 0.0, st);
        HIP_CHECK(hipStreamSynchronize(st));
        if (stats) {
            stats->iterations = 0;
            stats->converged = 1;
            stats->initial_residual = stats->final_residual = 0.0;
        }
        copy_history(h, stats, 1, st);
        return LDU_OK;
    }
    if (!std::isfinite(hs.res)) throw Error(LDU_ERR_NAN, "non-finite initial residual");
    double res = hs.res;
    int status = LDU_OK;
    const int every = o.check_every > 0 ? o.check_every : 16;
    const StepHistory conv{h->hist, h->hist_cap};
    while (res > o.rel_tol) {
        const int iters0 = hs.iters;
        int step = 0;  // iterations launched since the (re)start
        for (;;) {
            for (int k = 0; k < every; ++k, ++step) {
                const int mode = step == 0 ? kStepFirst : k == 0 ? kStepReady : kStepReduce;
                if (fused) {
                    const double *p = pbuf[step & 1];
                    double *p2 = pbuf[(step + 1) & 1];
                    if (A.pdeg)
                        k_cg_pq<true><<<Gq, kBlock, 0, st>>>(A, h->z, p, p2, x, h->q, h->partials,
                                                             Gr, mode, h->dev, h->dev + 1, conv);
                    else
                        k_cg_pq<false><<<Gq, kBlock, 0, st>>>(A, h->z, p, p2, x, h->q, h->partials,
                                                              Gr, mode, h->dev, h->dev + 1, conv);
                } else {
                    const int Gp = mode == kStepFirst ? 1 : Gr;
                    if (nt)
                        k_cg_p<true><<<Gp, kBlock, 0, st>>>(n, S, A.diag, h->r, x, h->p, precond,
                                                            h->partials, Gr, mode, h->dev,
                                                            h->dev + 1, conv);
                    else
                        k_cg_p<false><<<Gp, kBlock, 0, st>>>(n, S, A.diag, h->r, x, h->p, precond,
                                                             h->partials, Gr, mode, h->dev,
                                                             h->dev + 1, conv);
                    launch_product_dot(h, A, h->p, h->q, Gq, h->dev + 1, st);
                }
                double *z = fused ? h->z : nullptr;
                if (nt)
                    k_cg_r<true><<<Gr, kBlock, 0, st>>>(n, S, A.diag, h->r, h->q, z, precond,
                                                       h->partials, Gq, h->dev + 1, h->dev);
                else
                    k_cg_r<false><<<Gr, kBlock, 0, st>>>(n, S, A.diag, h->r, h->q, z, precond,
                                                        h->partials, Gq, h->dev + 1, h->dev);
            }
            // the last iteration's test for the host
            k_step_converge<false><<<1, kBlock, 0, st>>>(h->partials + kMaxGrid, Gr, h->dev, conv);
            HIP_CHECK(hipGetLastError());
            read_scalars(h, st);
            if (hs.done != kRunning) break;
        }
        // the stopping iteration's x += alpha p (none when alpha itself failed)
        launch_x_pending(h, x, pbuf[(hs.iters - iters0) & 1], n, S, G, st);
        if (hs.done == kFailed) {
            status = hs.status;
            break;
        }
        // true residual; restart from it if the recursive one drifted
        launch_residual<true, false>(h, A, b, x, h->r, p0, precond, kResPlain, false, st);
        read_scalars(h, st);
        res = hs.res;
        if (!std::isfinite(res)) { status = LDU_ERR_NAN; break; }
        if (res <= o.rel_tol) { status = LDU_OK; break; }
        if (hs.iters >= o.max_iter) { status = LDU_NOT_CONVERGED; break; }
        k_set_done<<<1, 1, 0, st>>>(h->dev, kRunning);
    }
    const int iters = hs.iters;
    if (stats) {
        stats->iterations = iters;
        stats->final_residual = res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, iters + 1, st);
    return status;
}

// ---------------------------------------------------------------- PBiCG
// Preconditioned bi-conjugate gradients for non-symmetric A (the paper's
// solver for the velocity and turbulence systems, whose profile pairs Amul
// with Tmul).  Shadow residual rt = r at every (re)start; M = D or I.
//   q = A p, qt = A^T pt, sigma = pt.q;  alpha = rho / sigma
//   x += alpha p; r -= alpha q; rt -= alpha qt;  ||r||^2, rho' = (M^-1 r).rt
//   beta = rho' / rho;  p = M^-1 r + beta p;  pt = M^-1 rt + beta pt

// rt = r, pt = p (the residual kernel has set r, p = M^-1 r and rho = r.p)
__global__ void __launch_bounds__(kBlock)
k_bicg_start(int32_t n, int64_t S, const double *__restrict__ r, const double *__restrict__ p,
             double *__restrict__ rt, double *__restrict__ pt, const DevScalars *ds) {
    if (ds->done) return;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            rt[i] = r[i];
            pt[i] = p[i];
        }
    });
}

// the entries of one row for A and for A^T together (valT holds A^T at the
// same positions), so that columns and slot bases are read once: q and qt add
// v x(c) and vt xt(c) in column order
template <bool C16, bool NT, class X, class XT>
__device__ __forceinline__ void plain_pair(const SellView<double> &A, const double *valT,
                                           int64_t s, int lane, const X &x, const XT &xt,
                                           double &q, double &qt) {
    constexpr int B = 8;
    const PlainWalk<C16, double, NT> pw(A, s, lane);
    const double *tp = valT + A.sptr[s] + lane;
    for (int k = 0; k < pw.w; k += B) {
        int32_t c[B], cb[B];
        double v[B], vt[B], xv[B], xtv[B];
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < pw.w) {
                pw.load(k + u, c[u], cb[u], v[u]);
                vt[u] = vld<NT>(tp + (int64_t)(k + u) * kWave);
            }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < pw.w) {
                c[u] = PlainWalk<C16, double, NT>::column(c[u], cb[u]);
                xv[u] = x(c[u]);
                xtv[u] = xt(c[u]);
            }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < pw.w) {
                q = q + v[u] * xv[u];
                qt = qt + vt[u] * xtv[u];
            }
    }
}

// the same over compressed slices, with the cache policy of A.stream as there
// (800,000 cells of a band graph, 96 MB of matrix: streamed 94 us an iteration,
// kept 79; 1,500,000 cells stream)
template <bool NT, class X, class XT>
__device__ __forceinline__ void cmp_pair(const SellView<double> &A, const double *valT, int64_t s,
                                         int lane, const X &x, const XT &xt, double &q,
                                         double &qt) {
    constexpr int B = 12;
    const int64_t b0 = A.sptr[s];
    const int w = A.pdeg[s * kWave + lane];
    const int32_t *cp = A.col + b0 + lane;
    const double *vp = A.val + b0 + lane, *tp = valT + b0 + lane;
    SliceOffsets so;
    for (int k = 0; k < w; k += B) {
        int32_t c[B];
        double v[B], vt[B], xv[B], xtv[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const bool has = k + u < w;
            const int64_t o = so.next(has);
            if (has) {
                c[u] = vld<NT>(cp + o);
                v[u] = vld<NT>(vp + o);
                vt[u] = vld<NT>(tp + o);
            }
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < w) {
                xv[u] = x(c[u]);
                xtv[u] = xt(c[u]);
            }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < w) {
                q = q + v[u] * xv[u];
                qt = qt + vt[u] * xtv[u];
            }
    }
}

template <bool CMP, class X, class XT>
__device__ __forceinline__ void pair_entries(const SellView<double> &A, const double *valT,
                                             int64_t s, int lane, const X &x, const XT &xt,
                                             double &q, double &qt) {
    if constexpr (!CMP) {
        if (A.stream) {
            if (A.c16) plain_pair<true, true>(A, valT, s, lane, x, xt, q, qt);
            else plain_pair<false, true>(A, valT, s, lane, x, xt, q, qt);
        } else {
            if (A.c16) plain_pair<true, false>(A, valT, s, lane, x, xt, q, qt);
            else plain_pair<false, false>(A, valT, s, lane, x, xt, q, qt);
        }
    } else {
        if (A.stream) cmp_pair<true>(A, valT, s, lane, x, xt, q, qt);
        else cmp_pair<false>(A, valT, s, lane, x, xt, q, qt);
    }
}

// An iteration in two or three kernels, as diagonal CG above: scalars from
// the producers' partials, x += alpha p deferred to the direction update, and
// up to kFusedBicgCells the product forms both new directions in its gathers.
// q and qt come from one pass over the columns (two sweeps over the row read
// them twice).  Convection-diffusion boxes: 32^3 1.92 -> 1.33 ms, 100^3 8.64
// -> 7.53 ms.

// p2 = z + beta p and pt2 = zt + beta pt (formed here when FUSED, else p2 and
// pt2 are p and pt); x += alpha p (the last iteration's, FUSED only);
// q = A p2, qt = A^T pt2; pt2.q
template <bool CMP, bool FUSED>
__global__ void __launch_bounds__(kBlock)
k_bicg_pq(SellView<double> A, const double *__restrict__ valT, const double *__restrict__ z,
          const double *__restrict__ zt, const double *__restrict__ p,
          const double *__restrict__ pt, double *__restrict__ p2, double *__restrict__ pt2,
          double *__restrict__ x, double *__restrict__ q, double *__restrict__ qt,
          double *partials, int nblocks, int mode, const DevScalars *in, DevScalars *out,
          StepHistory hist) {
    Step s{};
    if constexpr (FUSED) {
        s = step_converge<true>(mode, partials + kMaxGrid, nblocks, in, out, hist);
        if (!s.go) return;
    } else {
        if (in->done) return;
    }
    const bool first = mode == kStepFirst;
    const double alpha = FUSED ? s.alpha : 0.0, beta = FUSED ? s.beta : 0.0;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice<product_cap<CMP, double>()>(A.nslices, [&](int64_t sl) {
        const int64_t pos = sl * kWave + lane;
        if (pos < A.n) {
            const int32_t i = sv_row<CMP>(A, pos);
            const double di = A.diag[i];
            double pi, pti, qi, qti;
            if constexpr (FUSED) {
                const NewDirection np{z, p, beta, first}, npt{zt, pt, beta, first};
                pi = np(i);
                pti = npt(i);
                qi = di * pi;
                qti = di * pti;
                pair_entries<CMP>(A, valT, sl, lane, np, npt, qi, qti);
                if (!first) x[i] = x[i] + alpha * p[i];
                p2[i] = pi;
                pt2[i] = pti;
            } else {
                pi = p[i];
                pti = pt[i];
                qi = di * pi;
                qti = di * pti;
                pair_entries<CMP>(A, valT, sl, lane, Direct<double>{p}, Direct<double>{pt}, qi,
                                  qti);
            }
            q[i] = qi;
            qt[i] = qti;
            acc[0] += pti * qi;
        }
    });
    block_partials<1>(acc, partials);
}

// x += alpha p (the last iteration's); p = M^-1 r + beta p; pt = M^-1 rt + beta pt
__global__ void __launch_bounds__(kBlock)
k_bicg_p(int32_t n, int64_t S, const double *__restrict__ D, const double *__restrict__ r,
         const double *__restrict__ rt, double *__restrict__ x, double *__restrict__ p,
         double *__restrict__ pt, int precond, const double *partials, int nblocks, int mode,
         const DevScalars *in, DevScalars *out, StepHistory hist) {
    const Step s = step_converge<true>(mode, partials + kMaxGrid, nblocks, in, out, hist);
    if (!s.go || mode == kStepFirst) return;  // the first directions are there already
    const double alpha = s.alpha, beta = s.beta;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t sl) {
        const int64_t i = sl * kWave + lane;
        if (i < n) {
            const double di = D[i], pi = p[i];
            const double zi = precond ? r[i] / di : r[i];
            const double zti = precond ? rt[i] / di : rt[i];
            x[i] = x[i] + alpha * pi;
            p[i] = zi + beta * pi;
            pt[i] = zti + beta * pt[i];
        }
    });
}

// r -= alpha q; rt -= alpha qt; ||r||^2 and (M^-1 r) . rt; the preconditioned
// residuals are stored for the two-kernel form (z given)
__global__ void __launch_bounds__(kBlock)
k_bicg_r(int32_t n, int64_t S, const double *__restrict__ D, double *__restrict__ r,
         double *__restrict__ rt, const double *__restrict__ q, const double *__restrict__ qt,
         double *__restrict__ z, double *__restrict__ zt, int precond, double *partials,
         int nblocks, const DevScalars *in, DevScalars *out) {
    const Step s = step_alpha(partials, nblocks, in, out);
    if (!s.go) return;
    const double alpha = s.alpha;
    const int lane = threadIdx.x & 63;
    double acc[2] = {0.0, 0.0};
    for_each_slice(S, [&](int64_t sl) {
        const int64_t i = sl * kWave + lane;
        if (i < n) {
            const double di = precond ? D[i] : 1.0;
            const double ri = r[i] - alpha * q[i];
            const double rti = rt[i] - alpha * qt[i];
            r[i] = ri;
            rt[i] = rti;
            const double zi = precond ? ri / di : ri;
            if (z) {
                z[i] = zi;
                zt[i] = precond ? rti / di : rti;
            }
            acc[0] += ri * ri;
            acc[1] += zi * rti;
        }
    });
    block_partials<2>(acc, partials + kMaxGrid);
}

int pbicg_fp64(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
               ldu_stats *stats, hipStream_t st) {
    const Level &L = h->L0;
    SellView<double> A = L.A.view(tr);
    // ten vectors, and the values of A and of A^T
    A.stream = L.A.bytes(2 * sizeof(double)) + 10 * (int64_t)sizeof(double) * L.n > kCacheBytes;
    const double *valT = tr ? L.A.val : L.A.valT;
    const int n = L.n;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    const int precond = o.precond ? 1 : 0;
    if (!h->rt) {  // shadow vectors, allocated on the handle's first PBiCG solve
        h->arena.reserve(3 * (sizeof(double) * (size_t)n + 256));
        double *rt = h->arena.get<double>(n), *pt = h->arena.get<double>(n);
        h->qt = h->arena.get<double>(n);
        h->pt = pt;
        h->rt = rt;
    }
    const bool fused = n <= kFusedBicgCells;
    if (fused) ensure_direction(h);
    if (fused && !h->zt) {
        h->arena.reserve(2 * (sizeof(double) * (size_t)n + 256));
        h->pt2 = h->arena.get<double>(n);
        h->zt = h->arena.get<double>(n);
    }
    const int Gq = A.pdeg ? G : std::min(G, kPlainF64ProductBlocks);
    const int Gr = cg_blocks(n, G);
    double *const p0 = fused ? h->z : h->p, *const pt0 = fused ? h->zt : h->pt;
    double *const pbuf[2] = {fused ? h->p2 : h->p, h->p};
    double *const ptbuf[2] = {fused ? h->pt2 : h->pt, h->pt};
    ensure_hist(h, (int64_t)o.max_iter + 2);
    fill_stats_common(stats);
    set_scalars_for_solve(h, o.rel_tol, o.max_iter, st);
    launch_residual<true, false>(h, A, b, x, h->r, p0, precond, kResPlain, true, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        fill(x, n, 0.0, st);
        HIP_CHECK(hipStreamSynchronize(st));
        if (stats) {
            stats->iterations = 0;
            stats->converged = 1;
            stats->initial_residual = stats->final_residual = 0.0;
        }
        copy_history(h, stats, 1, st);
        return LDU_OK;
    }
    if (!std::isfinite(hs.res)) throw Error(LDU_ERR_NAN, "non-finite initial residual");
    double res = hs.res;
    int status = LDU_OK;
    const int every = o.check_every > 0 ? o.check_every : 16;
    const StepHistory conv{h->hist, h->hist_cap};
    while (res > o.rel_tol) {
        k_bicg_start<<<G, kBlock, 0, st>>>(n, S, h->r, p0, h->rt, pt0, h->dev);
        const int iters0 = hs.iters;
        int step = 0;  // iterations launched since the (re)start
        for (;;) {
            for (int k = 0; k < every; ++k, ++step) {
                const int mode = step == 0 ? kStepFirst : k == 0 ? kStepReady : kStepReduce;
                if (!fused)
                    k_bicg_p<<<mode == kStepFirst ? 1 : Gr, kBlock, 0, st>>>(
                        n, S, A.diag, h->r, h->rt, x, h->p, h->pt, precond, h->partials, Gr, mode,
                        h->dev, h->dev + 1, conv);
                auto product = [&](auto kernel, const DevScalars *in, DevScalars *out) {
                    kernel<<<Gq, kBlock, 0, st>>>(A, valT, h->z, h->zt, pbuf[step & 1],
                                                  ptbuf[step & 1], pbuf[(step + 1) & 1],
                                                  ptbuf[(step + 1) & 1], x, h->q, h->qt,
                                                  h->partials, Gr, mode, in, out, conv);
                };
                if (fused) {
                    if (A.pdeg) product(k_bicg_pq<true, true>, h->dev, h->dev + 1);
                    else product(k_bicg_pq<false, true>, h->dev, h->dev + 1);
                } else {
                    if (A.pdeg) product(k_bicg_pq<true, false>, h->dev + 1, nullptr);
                    else product(k_bicg_pq<false, false>, h->dev + 1, nullptr);
                }
                k_bicg_r<<<Gr, kBlock, 0, st>>>(n, S, A.diag, h->r, h->rt, h->q, h->qt,
                                               fused ? h->z : nullptr, fused ? h->zt : nullptr,
                                               precond, h->partials, Gq, h->dev + 1, h->dev);
            }
            // the last iteration's test for the host
            k_step_converge<true><<<1, kBlock, 0, st>>>(h->partials + kMaxGrid, Gr, h->dev, conv);
            HIP_CHECK(hipGetLastError());
            read_scalars(h, st);
            if (hs.done != kRunning) break;
        }
        // the stopping iteration's x += alpha p (none when alpha itself failed)
        launch_x_pending(h, x, pbuf[(hs.iters - iters0) & 1], n, S, G, st);
        if (hs.done == kFailed) {
            status = hs.status;
            break;
        }
        // true residual; restart from it (new shadow) if the recursive one drifted
        launch_residual<true, false>(h, A, b, x, h->r, p0, precond, kResPlain, false, st);
        read_scalars(h, st);
        res = hs.res;
        if (!std::isfinite(res)) { status = LDU_ERR_NAN; break; }
        if (res <= o.rel_tol) { status = LDU_OK; break; }
        if (hs.iters >= o.max_iter) { status = LDU_NOT_CONVERGED; break; }
        k_set_done<<<1, 1, 0, st>>>(h->dev, kRunning);
    }
    const int iters = hs.iters;
    if (stats) {
        stats->iterations = iters;
        stats->final_residual = res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, iters + 1, st);
    return status;
}

// ---------------------------------------------------------------- PCG, mixed
// Outer FP64 refinement with inner FP32 CG.  Inner dot products accumulate
// in FP64; alpha and beta are formed in FP64 and rounded to FP32.

// rhat = fp32(r / s), d = 0, z = rhat / D32, p = z; ||rhat||^2 and rhat.z
__global__ void __launch_bounds__(kBlock)
k_mx_start(int32_t n, int64_t S, const double *__restrict__ r, const float *__restrict__ D,
           float *__restrict__ r32, float *__restrict__ d32, float *__restrict__ p32,
           double *partials, const DevScalars *ds) {
    if (ds->done) return;
    const double sc = ds->maxabs;
    const int lane = threadIdx.x & 63;
    double acc[2] = {0.0, 0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            const float ri = (float)(r[i] / sc);
            const float zi = ri / D[i];
            r32[i] = ri;
            d32[i] = 0.0f;
            p32[i] = zi;
            acc[0] += (double)ri * (double)ri;
            acc[1] += (double)ri * (double)zi;
        }
    });
    block_partials<2>(acc, partials);
}

// start of an inner solve: ||rhat||, rho, and the inner target
// max(inner_tol, 0.3 tol / res) for the current outer residual res
struct EpiMxStart {
    int has_rho;
    __device__ bool active(const DevScalars *ds) const { return !ds->done; }
    __device__ void operator()(const double *t, DevScalars *ds) const {
        ds->scale = ds->maxabs;
        ds->r0 = sqrt(t[0]);
        if (has_rho) ds->rho = t[1];
        ds->inner_iters = 0;
        ds->inner_done = !(ds->r0 > 0.0);
        const double target = 0.3 * ds->tol / ds->res;
        ds->inner_now = target > ds->inner_tol ? target : ds->inner_tol;
    }
};

template <bool CMP>
__global__ void __launch_bounds__(kBlock)
k_mx_q(SellView<float> A, const float *__restrict__ p, float *__restrict__ q, double *partials,
       const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice(A.nslices, [&](int64_t s) {
        const int64_t pos = s * kWave + lane;
        if (pos < A.n) {
            const int32_t i = sv_row<CMP>(A, pos);
            const float qi = sell_row<CMP>(A, s, lane, i, Direct<float>{p});
            q[i] = qi;
            acc[0] += (double)p[i] * (double)qi;
        }
    });
    block_partials<1>(acc, partials);
}

template <bool DIAGZ>
__global__ void __launch_bounds__(kBlock)
k_mx_update(int32_t n, int64_t S, const float *__restrict__ D, float *__restrict__ d,
            float *__restrict__ r, const float *__restrict__ p, const float *__restrict__ q,
            double *partials, int nblocks, const DevScalars *in, DevScalars *out) {
    const Step s = step_mx_alpha(partials, nblocks, in, out);
    if (!s.go) return;
    const float af = (float)s.alpha;
    const int lane = threadIdx.x & 63;
    double acc[2] = {0.0, 0.0};
    for_each_slice(S, [&](int64_t sl) {
        const int64_t i = sl * kWave + lane;
        if (i < n) {
            const float di = d[i] + af * p[i];
            const float ri = r[i] - af * q[i];
            d[i] = di;
            r[i] = ri;
            acc[0] += (double)ri * (double)ri;
            if (DIAGZ) {
                const float zi = ri / D[i];
                acc[1] += (double)ri * (double)zi;
            }
        }
    });
    block_partials<2>(acc, partials + kMaxGrid);
}

// the stop test of an inner CG whose preconditioned direction comes from a
// V-cycle
struct EpiMxInner {
    __device__ bool active(const DevScalars *ds) const { return !vc_skip(ds); }
    __device__ void operator()(const double *t, DevScalars *ds) const {
        const int it = ds->inner_iters + 1;
        ds->inner_iters = it;
        ds->rr = t[0];
        if (sqrt(t[0]) <= ds->inner_now * ds->r0 || it >= ds->inner_max) ds->inner_done = 1;
    }
};

// the diagonal form's step for the host, which reads the scalars next
__global__ void __launch_bounds__(kBlock)
k_mx_step(const double *partials, int nblocks, DevScalars *ds) {
    step_mx_inner(kStepReduce, partials, nblocks, ds, ds);
}

__global__ void __launch_bounds__(kBlock)
k_mx_p(int32_t n, int64_t S, const float *__restrict__ D, const float *__restrict__ r,
       float *__restrict__ p, const double *partials, int nblocks, int mode,
       const DevScalars *in, DevScalars *out) {
    const Step s = step_mx_inner(mode, partials, nblocks, in, out);
    if (!s.go || mode == kStepFirst) return;  // the first direction is there already
    const float bf = (float)s.beta;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t sl) {
        const int64_t i = sl * kWave + lane;
        if (i < n) p[i] = r[i] / D[i] + bf * p[i];
    });
}

// q = A p with the scalars in dev[1]
void launch_mx_q(ldu_t *h, const SellView<float> &A32, int G, hipStream_t st) {
    if (A32.pdeg) k_mx_q<true><<<G, kBlock, 0, st>>>(A32, h->p32, h->q32, h->partials, h->dev + 1);
    else k_mx_q<false><<<G, kBlock, 0, st>>>(A32, h->p32, h->q32, h->partials, h->dev + 1);
}

// d += alpha p; r -= alpha q; ||r||^2 and the inner convergence test (the
// preconditioned direction comes from outside); Gq: blocks of the product
void launch_mx_update_plain(ldu_t *h, int32_t n, int64_t S, int G, int Gq, hipStream_t st) {
    k_mx_update<false><<<G, kBlock, 0, st>>>(n, S, nullptr, h->d32, h->r32, h->p32, h->q32,
                                             h->partials, Gq, h->dev + 1, h->dev);
    launch_finalize<1>(h->partials + kMaxGrid, G, h->dev, EpiMxInner{}, st);
}

// x += s * fp64(d)
__global__ void __launch_bounds__(kBlock)
k_mx_refine(int32_t n, int64_t S, const float *__restrict__ d, double *__restrict__ x,
            const DevScalars *ds) {
    if (ds->done) return;
    const double sc = ds->scale;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) x[i] = x[i] + sc * (double)d[i];
    });
}

__global__ void k_mx_set_inner(DevScalars *ds, double inner_tol, int inner_max) {
    ds->inner_tol = inner_tol;
    ds->inner_max = inner_max;
}
void set_inner(ldu_t *h, double inner_tol, int inner_max, hipStream_t st) {
    k_mx_set_inner<<<1, 1, 0, st>>>(h->dev, inner_tol, inner_max);
}
void launch_mx_refine(ldu_t *h, double *x, int32_t n, int64_t S, int G, hipStream_t st) {
    k_mx_refine<<<G, kBlock, 0, st>>>(n, S, h->d32, x, h->dev);
}

int pcg_mixed(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
              ldu_stats *stats, hipStream_t st) {
    Level &L = h->L0;
    ensure_f32(L, h->arena, true, st);
    const SellView<double> A = L.A.view(tr);
    const SellView<float> A32 = L.A.view32(tr);
    const int n = L.n;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    const int Gr = cg_blocks(n, G);
    ensure_hist(h, (int64_t)o.max_refine + 2);
    fill_stats_common(stats);
    set_scalars_for_solve(h, o.rel_tol, o.max_refine, st);
    k_mx_set_inner<<<1, 1, 0, st>>>(h->dev, o.inner_rel_tol, o.inner_max_iter);
    launch_residual<false, true>(h, A, b, x, h->r, nullptr, 0, kResCycle, true, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        fill(x, n, 0.0, st);
        HIP_CHECK(hipStreamSynchronize(st));
        if (stats) {
            stats->iterations = 0;
            stats->converged = 1;
            stats->initial_residual = stats->final_residual = 0.0;
        }
        copy_history(h, stats, 1, st);
        return LDU_OK;
    }
    const int every = o.check_every > 0 ? o.check_every : 16;
    long long inner_total = 0;
    while (hs.done == kRunning) {
        k_mx_start<<<G, kBlock, 0, st>>>(n, S, h->r, A32.diag, h->r32, h->d32, h->p32,
                                         h->partials, h->dev);
        launch_finalize<2>(h->partials, G, h->dev, EpiMxStart{1}, st);
        int step = 0;  // inner iterations launched
        for (;;) {
            for (int k = 0; k < every; ++k, ++step) {
                const int mode = step == 0 ? kStepFirst : k == 0 ? kStepReady : kStepReduce;
                k_mx_p<<<mode == kStepFirst ? 1 : Gr, kBlock, 0, st>>>(
                    n, S, A32.diag, h->r32, h->p32, h->partials + kMaxGrid, Gr, mode, h->dev,
                    h->dev + 1);
                launch_mx_q(h, A32, G, st);
                k_mx_update<true><<<Gr, kBlock, 0, st>>>(n, S, A32.diag, h->d32, h->r32, h->p32,
                                                         h->q32, h->partials, G, h->dev + 1,
                                                         h->dev);
            }
            k_mx_step<<<1, kBlock, 0, st>>>(h->partials + kMaxGrid, Gr, h->dev);
            HIP_CHECK(hipGetLastError());
            read_scalars(h, st);
            if (hs.inner_done) break;
        }
        inner_total += hs.inner_iters;
        k_mx_refine<<<G, kBlock, 0, st>>>(n, S, h->d32, x, h->dev);
        launch_residual<false, true>(h, A, b, x, h->r, nullptr, 0, kResCycle, true, st);
        read_scalars(h, st);
    }
    int status = LDU_OK;
    if (hs.done == kFailed) status = hs.status;
    else if (hs.done == kMaxIter) status = LDU_NOT_CONVERGED;
    if (stats) {
        stats->iterations = (int)inner_total;
        stats->refinements = hs.iters;
        stats->final_residual = hs.res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, hs.iters + 1, st);
    return status;
}

// ---------------------------------------------------------------- adjoint gradients
__global__ void k_coeff_grad(int32_t n, int64_t nf, const int32_t *__restrict__ own,
                             const int32_t *__restrict__ nb, const double *__restrict__ lam,
                             const double *__restrict__ x, double *gd, double *gu, double *gl) {
    const int64_t m = nf > n ? nf : n;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < m;
         k += (int64_t)gridDim.x * blockDim.x) {
        if (gd && k < n) gd[k] = -(lam[k] * x[k]);
        if (k < nf) {
            const int32_t o = own[k], b = nb[k];
            if (gu) gu[k] = -(lam[o] * x[b]);
            if (gl) gl[k] = -(lam[b] * x[o]);
        }
    }
}

void launch_coeff_grad(const Level &L, const double *lam, const double *x, double *gd,
                       double *gu, double *gl, hipStream_t st) {
    const int64_t m = L.nf > L.n ? L.nf : L.n;
    int64_t g = (m + kBlock - 1) / kBlock;
    g = g > 8192 ? 8192 : (g < 1 ? 1 : g);
    k_coeff_grad<<<(unsigned)g, kBlock, 0, st>>>(L.n, L.nf, L.own, L.nb, lam, x, gd, gu, gl);
    HIP_CHECK(hipGetLastError());
}

}  // namespace ldu
