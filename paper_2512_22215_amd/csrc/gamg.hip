// GAMG: pairwise agglomeration, Galerkin coarse matrices and the V-cycle.
//
// The paper runs OpenFOAM's GAMG for the pressure equation with the
// Richardson (damped Jacobi) smoother on every level and a diagonal-PCG
// coarsest solve, its fastest combination (Sec. 4.3, smoother table;
// Appendix A), and profiles agglomerateMatrix, restrictField, prolongField,
// scale and Vcycle (Sec. 4.3, kernel time breakdown).  It keeps OpenFOAM's
// serial CPU coarsening.  Here the coarsening is a parallel handshake
// matching with a strict total order on faces:
//   weight w_f = ((|upper_f| + |lower_f|) / 2)^2 / |diag_i diag_j| (the
//   squared coupling relative to the diagonals, which stays level under
//   geometric mesh grading), ties broken by a SplitMix64 hash of the face's
//   (min, max) cell pair, then by the smaller cell index;
//   each round, every unmatched cell picks its best unmatched neighbour and
//   mutual picks pair up; rounds stop when one adds no pair or after
//   match_rounds; an unmatched cell then joins the aggregate of its best
//   matched neighbour (no cascading) or stays a singleton; aggregates are
//   numbered by their seed cell (pair minimum or singleton).
// The result depends only on the matrix, not on the order in which threads
// run, and equals the greedy matching in that face order.
//
// Galerkin coarse matrices A_c = P^T A P (piecewise-constant P) are formed in
// LDU form with coarse faces sorted by (a, b); each coarse value is summed
// over its fine faces in ascending face order, and each coarse diagonal over
// member cells in ascending order and then over the aggregate's internal
// faces in ascending order.  Summation order is fixed, so the hierarchy is
// bitwise reproducible.
#include "device.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ldu {

__device__ __forceinline__ uint64_t splitmix64_out(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t tie_key(int32_t i, int32_t j) {
    const uint64_t lo = (uint32_t)(i < j ? i : j), hi = (uint32_t)(i < j ? j : i);
    return splitmix64_out((lo << 32) | hi);
}
// squared diagonally scaled coupling strength (no square root: it rounds the
// same way on every device)
__device__ __forceinline__ double strength2(double a, double at, double di, double dj) {
    const double s = 0.5 * (fabs(a) + fabs(at));
    const double den = fabs(di) * fabs(dj);
    return den > 0.0 ? (s * s) / den : s * s;
}
__device__ __forceinline__ bool better(double w1, uint64_t h1, int32_t j1, double w2,
                                       uint64_t h2, int32_t j2) {
    if (w1 != w2) return w1 > w2;
    if (h1 != h2) return h1 > h2;
    return j1 < j2;
}

static unsigned grid_n(int64_t n) {
    int64_t g = (n + kBlock - 1) / kBlock;
    g = g > 8192 ? 8192 : (g < 1 ? 1 : g);
    return (unsigned)(g >= 64 ? (g + 7) & ~int64_t(7) : g);
}
// best neighbour of row i among those whose matched state equals want_matched
__device__ int32_t best_neighbour(const Sell &A, int32_t i, const int32_t *partner,
                                  bool want_matched) {
    const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
    const int w = row_len(A, ps);
    int32_t best = -1;
    double bw = 0.0;
    uint64_t bh = 0;
    for (int k = 0; k < w; ++k) {
        const int64_t pos = entry_at(A, ps, k);
        const int32_t c = A.col[pos];
        if (c == i) continue;  // padding
        if ((partner[c] >= 0) != want_matched) continue;
        const double wt = strength2(A.val[pos], A.valT[pos], A.diag[i], A.diag[c]);
        const uint64_t hk = tie_key(i, c);
        if (best < 0 || better(wt, hk, c, bw, bh, best)) {
            best = c;
            bw = wt;
            bh = hk;
        }
    }
    return best;
}

// added[k]: round k added a pair.  A round after one that added none has
// nothing to do and returns at once (its own flag stays 0, so all later ones
// return too).
__global__ void k_match_init(int32_t n, int32_t *partner, int *added, int rounds) {
    GRID_STRIDE(i, n) partner[i] = -1;
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < rounds; k += blockDim.x) added[k] = 0;
}
__global__ void k_match_pick(Sell A, const int32_t *partner, int32_t *pick, const int *added,
                             int round) {
    if (round > 0 && !added[round - 1]) return;
    GRID_STRIDE(i, A.n) {
        pick[i] = partner[i] < 0 ? best_neighbour(A, (int32_t)i, partner, false) : -1;
    }
}
__global__ void k_match_pair(int32_t n, const int32_t *pick, int32_t *partner, int *added,
                             int round) {
    if (round > 0 && !added[round - 1]) return;
    GRID_STRIDE(i, n) {
        const int32_t j = pick[i];
        if (j >= 0 && pick[j] == (int32_t)i) {
            partner[i] = j;
            added[round] = 1;
        }
    }
}
__global__ void k_match_leftover(Sell A, const int32_t *partner, int32_t *join, int32_t *seed) {
    GRID_STRIDE(i, A.n) {
        const int32_t p = partner[i];
        const int32_t jn = p < 0 ? best_neighbour(A, (int32_t)i, partner, true) : -1;
        join[i] = jn;
        seed[i] = ((p >= 0 && (int32_t)i < p) || (p < 0 && jn < 0)) ? 1 : 0;
    }
}
__global__ void k_match_assign(int32_t n, const int32_t *partner, const int32_t *join,
                               const int32_t *rank, int32_t *agg) {
    GRID_STRIDE(i, n) {
        const int32_t p = partner[i];
        int32_t a;
        if (p >= 0) {
            a = rank[(int32_t)i < p ? (int32_t)i : p];
        } else if (join[i] < 0) {
            a = rank[i];
        } else {
            const int32_t j = join[i], pj = partner[j];
            a = rank[j < pj ? j : pj];
        }
        agg[i] = a;
    }
}

// aggregate member lists, ascending cell order
__global__ void k_agg_count(int32_t n, const int32_t *agg, int32_t *cnt) {
    GRID_STRIDE(i, n) atomicAdd(&cnt[agg[i]], 1);
}
__global__ void k_agg_fill(int32_t n, const int32_t *agg, const int32_t *start, int32_t *cursor,
                           int32_t *cells) {
    GRID_STRIDE(i, n) {
        const int32_t a = agg[i];
        cells[start[a] + atomicAdd(&cursor[a], 1)] = (int32_t)i;
    }
}
__global__ void k_agg_sort(int32_t nc, const int32_t *start, int32_t *cells) {
    GRID_STRIDE(a, nc) {
        const int32_t lo = start[a], hi = start[a + 1];
        for (int32_t k = lo + 1; k < hi; ++k) {
            const int32_t v = cells[k];
            int32_t m = k - 1;
            while (m >= lo && cells[m] > v) { cells[m + 1] = cells[m]; --m; }
            cells[m + 1] = v;
        }
    }
}

// coarse row a: the sorted distinct aggregates b > a adjacent to a
__device__ int coarse_row(const Sell &A, const int32_t *agg, const int32_t *start,
                          const int32_t *cells, int32_t a, int32_t *list, int *overflow) {
    int m = 0;
    for (int32_t k = start[a]; k < start[a + 1]; ++k) {
        const int32_t i = cells[k];
        const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
        const int w = row_len(A, ps);
        for (int e = 0; e < w; ++e) {
            const int32_t c = A.col[entry_at(A, ps, e)];
            if (c == i) continue;
            const int32_t b = agg[c];
            if (b <= a) continue;
            int pos = m;  // insertion into the sorted unique list
            while (pos > 0 && list[pos - 1] > b) --pos;
            if (pos > 0 && list[pos - 1] == b) continue;
            if (m >= kMaxCoarseRow) { *overflow = 1; return m; }
            for (int q = m; q > pos; --q) list[q] = list[q - 1];
            list[pos] = b;
            ++m;
        }
    }
    return m;
}
// One coarse row by a group of kRowLanes lanes: the members' entries are read
// side by side into LDS (the candidates b > a), duplicates drop out by
// comparison with all earlier candidates, and each distinct b's place is the
// number of smaller distinct ones.  A thread per row kept its sorted list in
// scratch memory and walked the entries one dependent load after another:
// 217 us a launch on average over a 1.8M-cell hierarchy, 62 us now.  A row
// with more candidates than fit takes that serial path.
constexpr int kRowLanes = 16;
constexpr int kRowGroups = kBlock / kRowLanes;
constexpr int kRowCand = 256;  // candidates a group's LDS holds

struct CoarseRowLds {
    int32_t c[kRowGroups][kRowCand];
};

// f(b, place) for the distinct aggregates b > a of row a, by one lane group;
// the return value is their number (every lane of the group)
template <class F>
__device__ int coarse_row_group(const Sell &A, const int32_t *agg, const int32_t *start,
                                const int32_t *cells, int32_t a, bool have, CoarseRowLds &sm,
                                int *overflow, F &&f) {
    const int l = threadIdx.x % kRowLanes;
    int32_t *cand = sm.c[threadIdx.x / kRowLanes];
    const int shift = (threadIdx.x & 63) / kRowLanes * kRowLanes;
    const uint64_t mine = ((uint64_t(1) << kRowLanes) - 1) << shift;
    const uint64_t below = mine & ((uint64_t(1) << (threadIdx.x & 63)) - 1);
    int m = 0;
    if (have) {
        for (int32_t k = start[a]; k < start[a + 1]; ++k) {
            const int32_t i = cells[k];
            const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
            const int w = row_len(A, ps);
            for (int q0 = 0; q0 < w; q0 += kRowLanes) {  // the same bounds for the group's lanes
                int32_t b = -1;
                if (q0 + l < w) {
                    const int32_t c = A.col[entry_at(A, ps, q0 + l)];
                    if (c != i) b = agg[c];
                }
                const uint64_t in = __ballot(b > a) & mine;
                const int at = m + __popcll(in & below);
                if (b > a && at < kRowCand) cand[at] = b;
                m += __popcll(in);
            }
        }
    }
    if (m > kRowCand) {  // rare: one lane, as a sorted list
        int32_t list[kMaxCoarseRow];
        int n = 0;
        if (l == 0) {
            n = coarse_row(A, agg, start, cells, a, list, overflow);
            for (int k = 0; k < n; ++k) f(list[k], k);
        }
        return __shfl(n, shift);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // first occurrences (bit t / kRowLanes of lane t % kRowLanes)
    uint32_t first = 0;
    int n = 0;
    for (int t = l; t < m; t += kRowLanes) {
        const int32_t b = cand[t];
        bool seen = false;
        for (int u = 0; u < t; ++u) seen = seen || cand[u] == b;
        if (!seen) {
            first |= 1u << (t / kRowLanes);
            ++n;
        }
    }
    int total = n;
    for (int off = 1; off < kRowLanes; off <<= 1) total += __shfl_xor(total, off);
    if (have && total > kMaxCoarseRow) {
        if (l == 0) *overflow = 1;
        return kMaxCoarseRow;
    }
    // repeats step aside, so that a place counts distinct aggregates
    __builtin_amdgcn_wave_barrier();
    int32_t own[kRowCand / kRowLanes];
#pragma unroll
    for (int j = 0; j < kRowCand / kRowLanes; ++j)
        own[j] = j * kRowLanes + l < m ? cand[j * kRowLanes + l] : 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < kRowCand / kRowLanes; ++j)
        if (j * kRowLanes + l < m && !(first >> j & 1)) cand[j * kRowLanes + l] = INT32_MAX;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < kRowCand / kRowLanes; ++j) {
        if (first >> j & 1) {
            int place = 0;
            for (int u = 0; u < m; ++u) place += cand[u] < own[j];
            f(own[j], place);
        }
    }
    return total;
}

// the group's rows, the same number of steps for every lane of a wave
#define ROW_GROUPS(a, n)                                                                  \
    for (GridRange gr_ = grid_range(n, kRowGroups); gr_.once; gr_.once = false)            \
        for (int64_t a0_ = gr_.begin; a0_ < gr_.end; a0_ += gr_.step)                      \
            if (const int64_t a = a0_ + threadIdx.x / kRowLanes; true)

__global__ void __launch_bounds__(kBlock)
k_coarse_count(Sell A, int32_t nc, const int32_t *agg, const int32_t *start,
               const int32_t *cells, int32_t *cnt, int *overflow) {
    __shared__ CoarseRowLds sm;
    ROW_GROUPS(a, nc) {
        const int n = coarse_row_group(A, agg, start, cells, (int32_t)a, a < nc, sm, overflow,
                                       [](int32_t, int) {});
        if (a < nc && threadIdx.x % kRowLanes == 0) cnt[a] = n;
    }
}
__global__ void __launch_bounds__(kBlock)
k_coarse_fill(Sell A, int32_t nc, const int32_t *agg, const int32_t *start,
              const int32_t *cells, const int32_t *cptr, int32_t *cown, int32_t *cnb,
              int *overflow) {
    __shared__ CoarseRowLds sm;
    ROW_GROUPS(a, nc) {
        const int32_t o = a < nc ? cptr[a] : 0;
        coarse_row_group(A, agg, start, cells, (int32_t)a, a < nc, sm, overflow,
                         [&](int32_t b, int place) {
                             cown[o + place] = (int32_t)a;
                             cnb[o + place] = b;
                         });
    }
}

// coarse face values: fine faces between aggregates a < b in ascending order
__global__ void k_coarse_values(int64_t ncf, const int32_t *cown, const int32_t *cnb,
                                const int32_t *agg, const int32_t *start, const int32_t *cells,
                                const int64_t *ownStart, const int32_t *fnb,
                                const double *fup, const double *flo, double *cup,
                                double *clo) {
    GRID_STRIDE(c, ncf) {
        const int32_t a = cown[c], b = cnb[c];
        int32_t ka = start[a], kb = start[b];
        const int32_t ea = start[a + 1], eb = start[b + 1];
        double up = 0.0, lo = 0.0;
        while (ka < ea || kb < eb) {  // merge the two member lists
            int32_t i;
            bool in_a;
            if (kb >= eb || (ka < ea && cells[ka] < cells[kb])) { i = cells[ka++]; in_a = true; }
            else { i = cells[kb++]; in_a = false; }
            const int32_t other = in_a ? b : a;
            for (int64_t f = ownStart[i]; f < ownStart[i + 1]; ++f) {
                if (agg[fnb[f]] != other) continue;
                if (in_a) { up += fup[f]; lo += flo[f]; }
                else { up += flo[f]; lo += fup[f]; }
            }
        }
        cup[c] = up;
        clo[c] = lo;
    }
}

// The same visits recorded once (count, then fill), so that new fine values
// only need a pass over the lists: each sum keeps its order and its bits.
// LIST = false counts, LIST = true writes at the counted offsets.
template <bool LIST>
__global__ void k_coarse_facelist(int64_t ncf, const int32_t *cown, const int32_t *cnb,
                                  const int32_t *agg, const int32_t *start,
                                  const int32_t *cells, const int64_t *ownStart,
                                  const int32_t *fnb, int64_t *count, const int64_t *offs,
                                  int32_t *list) {
    GRID_STRIDE(c, ncf) {
        const int32_t a = cown[c], b = cnb[c];
        int32_t ka = start[a], kb = start[b];
        const int32_t ea = start[a + 1], eb = start[b + 1];
        int64_t m = LIST ? offs[c] : 0;
        while (ka < ea || kb < eb) {
            int32_t i;
            bool in_a;
            if (kb >= eb || (ka < ea && cells[ka] < cells[kb])) { i = cells[ka++]; in_a = true; }
            else { i = cells[kb++]; in_a = false; }
            const int32_t other = in_a ? b : a;
            for (int64_t f = ownStart[i]; f < ownStart[i + 1]; ++f) {
                if (agg[fnb[f]] != other) continue;
                if (LIST) list[m] = in_a ? (int32_t)f : ~(int32_t)f;
                ++m;
            }
        }
        if (!LIST) count[c] = m;
    }
}
template <bool LIST>
__global__ void k_coarse_celllist(int32_t nc, const int32_t *agg, const int32_t *start,
                                  const int32_t *cells, const int64_t *ownStart,
                                  const int32_t *fnb, int64_t *count, const int64_t *offs,
                                  int32_t *list) {
    GRID_STRIDE(a, nc) {
        int64_t m = LIST ? offs[a] : 0;
        for (int32_t k = start[a]; k < start[a + 1]; ++k) {
            const int32_t i = cells[k];
            for (int64_t f = ownStart[i]; f < ownStart[i + 1]; ++f) {
                if (agg[fnb[f]] != (int32_t)a) continue;
                if (LIST) list[m] = (int32_t)f;
                ++m;
            }
        }
        if (!LIST) count[a] = m;
    }
}

// coarse values from the recorded lists (the sums of k_coarse_values and
// k_coarse_diag, term for term); a few terms' loads are in flight at a time, a
// small level's rows being one chain of loads each.  Six levels of a 151^3
// merged hierarchy: 503 -> 409 us a refresh.
__global__ void k_coarse_values_list(int64_t ncf, const int64_t *__restrict__ cfs,
                                     const int32_t *__restrict__ cff,
                                     const double *__restrict__ fup,
                                     const double *__restrict__ flo, double *__restrict__ cup,
                                     double *__restrict__ clo) {
    GRID_STRIDE(c, ncf) {
        double up = 0.0, lo = 0.0;
        const int64_t k1 = cfs[c + 1];
        for (int64_t k = cfs[c]; k < k1; k += 4) {
            int32_t g[4];
            double u[4], l[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) g[q] = k + q < k1 ? cff[k + q] : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + q < k1) {
                    u[q] = g[q] >= 0 ? fup[g[q]] : flo[~g[q]];
                    l[q] = g[q] >= 0 ? flo[g[q]] : fup[~g[q]];
                }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + q < k1) {
                    up += u[q];
                    lo += l[q];
                }
        }
        cup[c] = up;
        clo[c] = lo;
    }
}
__global__ void k_coarse_diag_list(int32_t nc, const int32_t *__restrict__ start,
                                   const int32_t *__restrict__ cells,
                                   const int64_t *__restrict__ cis,
                                   const int32_t *__restrict__ cif,
                                   const double *__restrict__ fdiag,
                                   const double *__restrict__ fup,
                                   const double *__restrict__ flo, double *__restrict__ cdiag) {
    GRID_STRIDE(a, nc) {
        double d = 0.0;
        const int32_t k1 = start[a + 1];
        const int64_t m0 = cis[a], m1 = cis[a + 1];
        for (int32_t k = start[a]; k < k1; k += 8) {
            int32_t i[8];
            double x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) i[q] = k + q < k1 ? cells[k + q] : 0;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (k + q < k1) x[q] = fdiag[i[q]];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (k + q < k1) d += x[q];
        }
        for (int64_t k = m0; k < m1; k += 8) {
            int32_t f[8];
            double x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) f[q] = k + q < m1 ? cif[k + q] : 0;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (k + q < m1) x[q] = fup[f[q]] + flo[f[q]];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (k + q < m1) d += x[q];
        }
        cdiag[a] = d;
    }
}

__global__ void k_coarse_diag(int32_t nc, const int32_t *agg, const int32_t *start,
                              const int32_t *cells, const int64_t *ownStart, const int32_t *fnb,
                              const double *fdiag, const double *fup, const double *flo,
                              double *cdiag) {
    GRID_STRIDE(a, nc) {
        double d = 0.0;
        for (int32_t k = start[a]; k < start[a + 1]; ++k) d += fdiag[cells[k]];
        for (int32_t k = start[a]; k < start[a + 1]; ++k) {
            const int32_t i = cells[k];
            for (int64_t f = ownStart[i]; f < ownStart[i + 1]; ++f)
                if (agg[fnb[f]] == (int32_t)a) d += (fup[f] + flo[f]);
        }
        cdiag[a] = d;
    }
}

// singular level: |(A 1)_i| <= 1e-12 |diag_i| for every row
__global__ void k_singular(Sell A, int *flag) {
    GRID_STRIDE(i, A.n) {
        const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
        const int64_t s = ps >> 6, lane = ps & 63;
        const SellView<double> v = A.view(false);
        struct One { __device__ double operator()(int32_t) const { return 1.0; } };
        const double y = sell_row_any(v, s, (int)lane, (int32_t)i, One{});
        if (!(fabs(y) <= 1e-12 * fabs(A.diag[i]))) atomicAnd(flag, 0);
    }
}

// ---------------------------------------------------------------- setup
// FP32 copies of every level's values; level 0's live with the handle
static void ensure_f32_levels(ldu_t *h, hipStream_t st) {
    ensure_f32(h->L0, h->L0.src ? h->gamg_arena : h->arena, !h->L0.src, st);  // a renumbered one's: hierarchy
    h->levels[0].A = h->L0.A;
    for (size_t l = 1; l < h->levels.size(); ++l) ensure_f32(h->levels[l], h->gamg_arena, false, st);
}

static void ensure_work(ldu_t *h) {
    for (Level &L : h->levels) {
        if (L.r) continue;
        Arena::Step step(h->gamg_arena);
        double *r = h->gamg_arena.get<double>(L.n);
        L.e = h->gamg_arena.get<double>(L.n);
        L.e2 = h->gamg_arena.get<double>(L.n);
        L.t = h->gamg_arena.get<double>(L.n);
        L.r = r;  // last: the four exist
        step.done();
    }
}

static void coarse_values(ldu_t *h, Level &F, Level &C, hipStream_t st) {
    if (F.cfStart) {  // recorded visits (hierarchy levels)
        if (C.nf > 0)
            k_coarse_values_list<<<grid_n(C.nf), kBlock, 0, st>>>(C.nf, F.cfStart, F.cfFace,
                                                                   F.upper, F.lower, C.upper,
                                                                   C.lower);
        k_coarse_diag_list<<<grid_n(C.n), kBlock, 0, st>>>(C.n, F.aggStart, F.aggCells,
                                                           F.ciStart, F.ciFace, F.diag, F.upper,
                                                           F.lower, C.diag);
    } else {  // the aggressive passes' temporary matrices
        if (C.nf > 0)
            k_coarse_values<<<grid_n(C.nf), kBlock, 0, st>>>(C.nf, C.own, C.nb, F.agg,
                                                              F.aggStart, F.aggCells, F.ownStart,
                                                              F.nb, F.upper, F.lower, C.upper,
                                                              C.lower);
        k_coarse_diag<<<grid_n(C.n), kBlock, 0, st>>>(C.n, F.agg, F.aggStart, F.aggCells,
                                                      F.ownStart, F.nb, F.diag, F.upper, F.lower,
                                                      C.diag);
    }
    HIP_CHECK(hipGetLastError());
}

// record the fine faces each coarse value and diagonal sums (count, scan, fill)
static void coarse_lists(Level &F, const Level &C, Arena &ar, hipStream_t st) {
    Arena tmp(&ar);
    int64_t *cnt = tmp.get<int64_t>((size_t)C.nf + 1);
    F.cfStart = ar.get<int64_t>((size_t)C.nf + 1);
    if (C.nf > 0)
        k_coarse_facelist<false><<<grid_n(C.nf), kBlock, 0, st>>>(
            C.nf, C.own, C.nb, F.agg, F.aggStart, F.aggCells, F.ownStart, F.nb, cnt, nullptr,
            nullptr);
    exclusive_scan_i64(cnt, F.cfStart, C.nf, tmp, st);
    int64_t *cntc = tmp.get<int64_t>((size_t)C.n + 1);
    F.ciStart = ar.get<int64_t>((size_t)C.n + 1);
    k_coarse_celllist<false><<<grid_n(C.n), kBlock, 0, st>>>(
        C.n, F.agg, F.aggStart, F.aggCells, F.ownStart, F.nb, cntc, nullptr, nullptr);
    exclusive_scan_i64(cntc, F.ciStart, C.n, tmp, st);
    int64_t nff = 0, nif = 0;
    HIP_CHECK(hipMemcpyAsync(&nff, F.cfStart + C.nf, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipMemcpyAsync(&nif, F.ciStart + C.n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    F.cfFace = ar.get<int32_t>((size_t)nff + 1);
    F.ciFace = ar.get<int32_t>((size_t)nif + 1);
    if (C.nf > 0)
        k_coarse_facelist<true><<<grid_n(C.nf), kBlock, 0, st>>>(
            C.nf, C.own, C.nb, F.agg, F.aggStart, F.aggCells, F.ownStart, F.nb, nullptr,
            F.cfStart, F.cfFace);
    k_coarse_celllist<true><<<grid_n(C.n), kBlock, 0, st>>>(
        C.n, F.agg, F.aggStart, F.aggCells, F.ownStart, F.nb, nullptr, F.ciStart, F.ciFace);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
}

__global__ void k_set_int(int *p, int v) { *p = v; }

static void detect_singular(ldu_t *h, Level &L, hipStream_t st) {
    k_set_int<<<1, 1, 0, st>>>(h->flag, 1);
    k_singular<<<grid_n(L.n), kBlock, 0, st>>>(L.A, h->flag);
    HIP_CHECK(hipMemcpyAsync(h->hflag, h->flag, sizeof(int), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    L.singular = (*h->hflag != 0) && L.n > 0;
}

// member lists of F's aggregation (F.agg, F.nc): aggStart and aggCells in
// ascending cell order
static void agg_lists(Level &F, Arena &ar, hipStream_t st) {
    Arena tmp(&ar);
    const int32_t n = F.n, nc = F.nc;
    const unsigned g = grid_n(n);
    int32_t *cnt = tmp.get<int32_t>(nc);
    int32_t *cursor = tmp.get<int32_t>(nc);
    HIP_CHECK(hipMemsetAsync(cnt, 0, sizeof(int32_t) * nc, st));
    HIP_CHECK(hipMemsetAsync(cursor, 0, sizeof(int32_t) * nc, st));
    k_agg_count<<<g, kBlock, 0, st>>>(n, F.agg, cnt);
    F.aggStart = ar.get<int32_t>((size_t)nc + 1);
    scan_counts_i32(cnt, F.aggStart, nc, tmp, st);
    F.aggCells = ar.get<int32_t>(n);
    k_agg_fill<<<g, kBlock, 0, st>>>(n, F.agg, F.aggStart, cursor, F.aggCells);
    k_agg_sort<<<grid_n(nc), kBlock, 0, st>>>(nc, F.aggStart, F.aggCells);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));
}

// one pairwise matching pass over level F: F.agg (in ar) and F.nc; the member
// lists go to lists_ar
static int32_t agglomerate(ldu_t *h, Level &F, int match_rounds, Arena &ar, Arena &lists_ar,
                           hipStream_t st) {
    const int32_t n = F.n;
    Arena tmp(&ar);
    int32_t *partner = tmp.get<int32_t>(n);
    int32_t *pick = tmp.get<int32_t>(n);
    int32_t *join = tmp.get<int32_t>(n);
    int32_t *seed = tmp.get<int32_t>(n);
    int32_t *rank = tmp.get<int32_t>((size_t)n + 1);
    int *added = tmp.get<int>((size_t)match_rounds + 1);
    const unsigned g = grid_n(n);
    k_match_init<<<g, kBlock, 0, st>>>(n, partner, added, match_rounds);
    for (int round = 0; round < match_rounds; ++round) {
        k_match_pick<<<g, kBlock, 0, st>>>(F.A, partner, pick, added, round);
        k_match_pair<<<g, kBlock, 0, st>>>(n, pick, partner, added, round);
    }
    k_match_leftover<<<g, kBlock, 0, st>>>(F.A, partner, join, seed);
    scan_counts_i32(seed, rank, n, tmp, st);
    int32_t nc = 0;
    HIP_CHECK(hipMemcpyAsync(&nc, rank + n, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    F.nc = nc;
    F.agg = ar.get<int32_t>(n);
    k_match_assign<<<g, kBlock, 0, st>>>(n, partner, join, rank, F.agg);
    HIP_CHECK(hipGetLastError());
    agg_lists(F, lists_ar, st);
    return nc;
}

__global__ void k_compose(int32_t n, const int32_t *__restrict__ outer, int32_t *agg) {
    GRID_STRIDE(i, n) agg[i] = outer[agg[i]];
}

static void galerkin(ldu_t *h, Level &F, Level &C, Arena &ar, hipStream_t st);

// aggregation of level F by `passes` pairwise matching passes: pass k matches
// the aggregates of pass k-1 on their Galerkin matrix (a temporary, used only
// for its coupling strengths) and the aggregate maps compose.  One pass is
// plain pairwise agglomeration.
static int32_t agglomerate_passes(ldu_t *h, Level &F, int match_rounds, int passes, Arena &ar,
                                  hipStream_t st) {
    if (passes <= 1) return agglomerate(h, F, match_rounds, ar, ar, st);
    Arena tmp(&ar);
    const int32_t nc = agglomerate(h, F, match_rounds, ar, tmp, st);
    if (nc <= 1) {
        agg_lists(F, ar, st);
        return nc;
    }
    Level T;
    galerkin(h, F, T, tmp, st);
    build_level_sell(h, tmp, T, false, st);
    const int32_t nc2 = agglomerate_passes(h, T, match_rounds, passes - 1, tmp, st);
    k_compose<<<grid_n(F.n), kBlock, 0, st>>>(F.n, T.agg, F.agg);
    HIP_CHECK(hipGetLastError());
    F.nc = nc2;
    agg_lists(F, ar, st);
    return nc2;
}

static void galerkin(ldu_t *h, Level &F, Level &C, Arena &ar, hipStream_t st) {
    Arena tmp(&ar);
    const int32_t nc = F.nc;
    int32_t *cnt = tmp.get<int32_t>(nc);
    int32_t *cptr = tmp.get<int32_t>((size_t)nc + 1);
    int *overflow = tmp.get<int>(1);
    HIP_CHECK(hipMemsetAsync(overflow, 0, sizeof(int), st));
    k_coarse_count<<<grid_n((int64_t)nc * kRowLanes), kBlock, 0, st>>>(F.A, nc, F.agg, F.aggStart, F.aggCells, cnt,
                                                  overflow);
    scan_counts_i32(cnt, cptr, nc, tmp, st);
    int32_t ncf = 0;
    int ovf = 0;
    HIP_CHECK(hipMemcpyAsync(&ncf, cptr + nc, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipMemcpyAsync(&ovf, overflow, sizeof(int), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    if (ovf) throw Error(LDU_ERR_LIMIT, "coarse level row exceeds the supported width");
    C.n = nc;
    C.nf = ncf;
    C.own = ar.get<int32_t>(ncf);
    C.nb = ar.get<int32_t>(ncf);
    C.upper = ar.get<double>(ncf);
    C.lower = ar.get<double>(ncf);
    C.diag = ar.get<double>(nc);
    k_coarse_fill<<<grid_n((int64_t)nc * kRowLanes), kBlock, 0, st>>>(F.A, nc, F.agg, F.aggStart, F.aggCells, cptr,
                                                 C.own, C.nb, overflow);
    HIP_CHECK(hipGetLastError());
    coarse_values(h, F, C, st);
    HIP_CHECK(hipStreamSynchronize(st));
}

static void ensure_rop(ldu_t *h, const ldu_gamg_opts &o, hipStream_t st);
static void ensure_gen(ldu_t *h, const ldu_gamg_opts &o, hipStream_t st);
static void refresh_rop(ldu_t *h, hipStream_t st);

// ---------------------------------------------------------------- inner numbering
// On a mesh whose numbering scatters its neighbours every gather of a level-0
// kernel pulls a cache line of its own from the Infinity Cache (128^3
// shuffled: 190 us a sweep, 33 us renumbered by level sets), and the coarse
// levels, numbered by seed cell, inherit it.  The solves then run on copies of
// the large levels in an order that the hierarchy gives for nothing: the
// members of an aggregate follow one another, aggregates in the order of their
// own level, from the coarsest level down, so that cells close in the mesh are
// close in memory at every scale.  Setup, exports, products and everything in
// the caller's numbering keep the levels as they are: the hierarchy is the
// same cell for cell, and a solve differs in the order of its sums only.
// The two-stage Gauss-Seidel smoother, whose sweeps depend on the numbering,
// solves on the original levels.  Standalone GAMG, default settings, 128^3
// shuffled: 71.2 -> 33.1 ms (natural order: 32.8).  Renumbering the coarse
// levels of meshes that are not scattered changed nothing (200^3 125.6 and
// 125.2 ms, 128^3 mixed 29.5 and 29.6).
struct NumberingScope {
    ldu_t *h;
    NumberingScope(ldu_t *hh, int smoother)
        : h(!hh->inner.empty() && smoother == LDU_SMOOTH_JACOBI ? hh : nullptr) {
        swap();
    }
    ~NumberingScope() { swap(); }
    NumberingScope(const NumberingScope &) = delete;
    NumberingScope &operator=(const NumberingScope &) = delete;
    bool active() const { return h != nullptr; }

private:
    void swap() {
        if (!h) return;
        std::swap(h->L0, h->inner_L0);
        std::swap(h->levels, h->inner);
    }
};

// a solve's or a cycle's vectors in the inner numbering
struct InnerVectors {
    const double *in;  // b or r
    double *out;       // x or e
};
static InnerVectors inner_vectors(ldu_t *h, bool active, const double *in, double *out,
                                  bool read_out, hipStream_t st) {
    if (!active) return {in, out};
    gather_cells(in, h->inner_order, h->inner_b, h->L0.n, st);
    if (read_out) gather_cells(out, h->inner_order, h->inner_x, h->L0.n, st);
    return {h->inner_b, h->inner_x};
}
static void inner_result(ldu_t *h, bool active, double *out, hipStream_t st) {
    if (!active) return;
    scatter_cells(h->inner_x, h->inner_order, out, h->L0.n, st);
    HIP_CHECK(hipStreamSynchronize(st));
}

__global__ void k_rn_identity(int32_t n, int32_t *place) {
    GRID_STRIDE(i, n) place[i] = (int32_t)i;
}
// member counts in the coarse level's order
__global__ void k_rn_counts(int32_t nc, const int32_t *start, const int32_t *cplace,
                            int32_t *cnt) {
    GRID_STRIDE(c, nc) cnt[cplace[c]] = start[c + 1] - start[c];
}
__global__ void k_rn_place(int32_t nc, const int32_t *start, const int32_t *cells,
                           const int32_t *cplace, const int32_t *offs, int32_t *place) {
    GRID_STRIDE(c, nc) {
        const int32_t o = offs[cplace[c]];
        for (int32_t k = start[c]; k < start[c + 1]; ++k) place[cells[k]] = o + (k - start[c]);
    }
}
__global__ void k_rn_order(int32_t n, const int32_t *place, int32_t *order) {
    GRID_STRIDE(i, n) order[place[i]] = (int32_t)i;
}
__global__ void k_rn_agg(int32_t n, const int32_t *order, const int32_t *agg,
                         const int32_t *cplace, int32_t *out) {
    GRID_STRIDE(p, n) {
        const int32_t c = agg[order[p]];
        out[p] = cplace ? cplace[c] : c;
    }
}

static void renumber_levels(ldu_t *h, hipStream_t st) {
    Arena &ar = h->gamg_arena;
    Arena tmp(&ar);
    const size_t nl = h->levels.size();
    std::vector<int32_t *> place(nl);
    for (size_t l = nl; l-- > 0;) {  // from the coarsest level down
        const Level &L = h->levels[l];
        place[l] = tmp.get<int32_t>(L.n);
        if (l + 1 == nl) {
            k_rn_identity<<<grid_n(L.n), kBlock, 0, st>>>(L.n, place[l]);
            continue;
        }
        int32_t *cnt = tmp.get<int32_t>(L.nc), *offs = tmp.get<int32_t>((size_t)L.nc + 1);
        k_rn_counts<<<grid_n(L.nc), kBlock, 0, st>>>(L.nc, L.aggStart, place[l + 1], cnt);
        scan_counts_i32(cnt, offs, L.nc, tmp, st);
        k_rn_place<<<grid_n(L.nc), kBlock, 0, st>>>(L.nc, L.aggStart, L.aggCells, place[l + 1],
                                                    offs, place[l]);
    }
    HIP_CHECK(hipGetLastError());
    for (size_t l = 0; l < nl; ++l) {
        const Level &L = h->levels[l];
        Level N = L;  // small levels share everything with the original
        if (L.n > kRenumberRows) {
            const bool coarse = l + 1 < nl && h->levels[l + 1].n > kRenumberRows;
            int32_t *order = ar.get<int32_t>(L.n);
            k_rn_order<<<grid_n(L.n), kBlock, 0, st>>>(L.n, place[l], order);
            build_renumbered(L.A, L.nf, order, place[l], N, ar, st);
            N.own = N.nb = nullptr;
            N.upper = N.lower = nullptr;
            if (l + 1 < nl) {
                N.agg = ar.get<int32_t>(L.n);
                k_rn_agg<<<grid_n(L.n), kBlock, 0, st>>>(L.n, order, L.agg,
                                                         coarse ? place[l + 1] : nullptr, N.agg);
                agg_lists(N, ar, st);
            }
        }
        h->inner.push_back(N);
    }
    h->inner_L0 = h->inner[0];
    h->inner_order = h->inner[0].order;
    h->inner_b = ar.get<double>(h->L0.n);
    h->inner_x = ar.get<double>(h->L0.n);
    HIP_CHECK(hipStreamSynchronize(st));  // tmp is released after this point
}

// new values of the original levels into the inner ones, by the first solve
// that runs on those: callers that go on with products, diagonal CG or
// Gauss-Seidel cycles have no use for them (set_coeffs on a shuffled
// 100 x 90 x 80 mesh 685 us, with the copies 1000)
static void refresh_inner(ldu_t *h, int smoother, hipStream_t st) {
    if (!h->inner_stale || smoother != LDU_SMOOTH_JACOBI) return;
    for (size_t l = 0; l < h->inner.size(); ++l) {
        Level &N = h->inner[l];
        if (N.src) renumbered_values(h->levels[l].A, N, st);
        refresh_f32(N, st);
        N.singular = h->levels[l].singular;
    }
    NumberingScope scope(h, smoother);
    refresh_rop(h, st);
    h->inner_stale = false;
}

void gamg_build(ldu_t *h, const ldu_gamg_opts &o, hipStream_t st) {
    h->gamg_ready = false;
    h->levels.clear();
    h->inner.clear();
    h->inner_stale = false;
    h->gamg_arena.release_all();
    Arena &ar = h->gamg_arena;
    h->levels.push_back(h->L0);
    h->levels[0].agg = h->levels[0].aggStart = h->levels[0].aggCells = nullptr;
    h->levels[0].cfStart = h->levels[0].ciStart = nullptr;
    h->levels[0].cfFace = h->levels[0].ciFace = nullptr;
    const int maxl = std::min(std::max(o.max_levels, 1), kMaxLevels);
    while ((int)h->levels.size() < maxl) {
        const size_t l = h->levels.size() - 1;
        if (h->levels[l].n <= o.n_coarsest) break;
        const int passes = (int)l >= o.aggressive_from ? o.passes : 1;
        const int32_t nc = agglomerate_passes(h, h->levels[l], o.match_rounds, passes, ar, st);
        if (100 * (int64_t)nc > 95 * (int64_t)h->levels[l].n) {
            h->levels[l].agg = nullptr;
            break;
        }
        Level C;
        galerkin(h, h->levels[l], C, ar, st);
        coarse_lists(h->levels[l], C, ar, st);  // for value refreshes on this structure
        build_level_sell(h, ar, C, false, st);
        h->levels.push_back(C);
    }
    if (h->levels.back().n > kMaxCoarsest && h->levels.back().nf > 0) {
        h->levels.clear();
        h->gamg_arena.release_all();
        throw Error(LDU_ERR_LIMIT, "coarsest GAMG level has more than 8192 cells; raise max_levels");
    }
    detect_singular(h, h->levels.back(), st);
    if (o.smoother == LDU_SMOOTH_JACOBI && h->levels.size() > 1 && scattered_numbering(h, st)) {
        Arena::Step step(ar);
        try {
            renumber_levels(h, st);
            step.done();
        } catch (const Error &e) {  // without memory for the copies: the levels as they are
            if (e.code != LDU_ERR_NOMEM) throw;
            h->inner.clear();
        }
    }
    NumberingScope scope(h, o.smoother);  // work vectors and R of the levels that solve
    ensure_work(h);
    h->coarse_work = ar.get<double>(5 * (size_t)h->levels.back().n);
    h->dic_dt = ar.get<double>(h->levels.back().n);
    h->dic_ready = false;

    if (h->L0.A.val32) ensure_f32_levels(h, st);
    h->gamg_opts = o;
    h->gamg_ready = true;
    // a Jacobi cycle with one pre-sweep will run its down leg through R (the
    // CG + V-cycle solve turns correction scaling off): build it with the
    // hierarchy
    if (o.smoother == LDU_SMOOTH_JACOBI && o.n_pre == 1) {
        ldu_gamg_opts q = o;
        q.scale_correction = 0;
        ensure_rop(h, q, st);
    } else
        ensure_gen(h, o, st);  // with R built: by the first cycle that uses V and W, as a
                               // hierarchy for the CG never does (0.8 ms on 1.8M cells)
    h->pool.trim();
}

// new level-0 values: recompute every coarse matrix on the cached structure
void gamg_refresh_values(ldu_t *h, hipStream_t st) {
    if (!h->gamg_ready) return;
    h->levels[0].A = h->L0.A;
    for (size_t l = 0; l + 1 < h->levels.size(); ++l) {
        Level &F = h->levels[l], &C = h->levels[l + 1];
        coarse_values(h, F, C, st);
        set_level_values(C, st);
        refresh_f32(C, st);
    }
    detect_singular(h, h->levels.back(), st);
    h->dic_ready = false;
    h->inner_stale = !h->inner.empty();
    refresh_rop(h, st);
}

// DIC pivots of the coarsest level (diagonal incomplete Cholesky; the paper's
// other coarsest-level preconditioner, Sec. 4.3 smoother table):
//   Dt_i = A_ii - sum_{j<i} A_ij A_ji / Dt_j, ascending j,
// with A_ji read from the transposed values at the same position.  Serial in
// one thread: the level has a few dozen rows, and this runs once per set of
// coefficients.  ok = 0 when a pivot is not finite, changes sign against
// A_ii, or falls below 1e-12 |A_ii|; the solve then uses the diagonal.
__global__ void k_dic_factor(Sell A, double *dt, int *ok) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    int good = 1;
    for (int32_t i = 0; i < A.n; ++i) {
        const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
        const int w = row_len(A, ps);
        double d = A.diag[i];
        for (int k = 0; k < w; ++k) {
            const int64_t e = entry_at(A, ps, k);
            const int32_t c = A.col[e];
            if (c < i) d = d - (A.val[e] * A.valT[e]) / dt[c];
        }
        dt[i] = d;
        if (!isfinite(d) || !(fabs(d) > 1e-12 * fabs(A.diag[i])) || ((d > 0.0) != (A.diag[i] > 0.0)))
            good = 0;
    }
    *ok = good;
}

static void ensure_dic(ldu_t *h, hipStream_t st) {
    if (h->dic_ready) return;
    Level &L = h->levels.back();
    k_dic_factor<<<1, 1, 0, st>>>(L.A, h->dic_dt, h->flag);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipMemcpyAsync(h->hflag, h->flag, sizeof(int), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    h->dic_ok = *h->hflag != 0;
    h->dic_ready = true;
}

// ---------------------------------------------------------------- V-cycle kernels
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_first(int32_t n, int64_t S, const T *__restrict__ r, const T *__restrict__ D,
           T *__restrict__ e, T omega, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) e[i] = omega * r[i] / D[i];
    });
}

template <typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_zero(int32_t n, int64_t S, T *__restrict__ e, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) e[i] = T(0);
    });
}

// The finer level's unscaled correction e_f += P e_c, applied by the kernel
// that produces e_c: row a adds its value to the members of aggregate a.
constexpr int kCorrBatch = 8;  // aggregate members a fused correction handles at once

template <typename T>
struct FineCorr {
    T *e;
    const int32_t *start, *cells;
    __device__ __forceinline__ void operator()(int32_t a, T v) const {
        apply(start[a], start[a + 1], v);
    }
    // members k0..k1-1 of the aggregate (bounds loaded ahead by the caller),
    // kCorrBatch at a time: their indices, then their values, are loaded
    // together before any store (the members are distinct cells), so an
    // aggregate of several passes costs a few round trips, not one per member
    __device__ __forceinline__ void apply(int32_t k0, int32_t k1, T v) const {
        for (int32_t k = k0; k < k1; k += kCorrBatch) {
            int32_t j[kCorrBatch];
            T ev[kCorrBatch];
#pragma unroll
            for (int u = 0; u < kCorrBatch; ++u)
                if (k + u < k1) j[u] = cells[k + u];
#pragma unroll
            for (int u = 0; u < kCorrBatch; ++u)
                if (k + u < k1) ev[u] = e[j[u]];
#pragma unroll
            for (int u = 0; u < kCorrBatch; ++u)
                if (k + u < k1) e[j[u]] = ev[u] + v;
        }
    }
};

// e_out = e + omega (r - A e) / D; DOT also accumulates the block partials of
// rdot . e_out (the preconditioned CG's r . z, saving a pass over both); CORR
// also applies the finer level's correction with e_out
template <bool CMP, bool DOT, bool CORR, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_jacobi(SellView<T> A, const T *__restrict__ r, const T *__restrict__ e,
            T *__restrict__ eo, T omega, const T *__restrict__ rdot, double *partials,
            FineCorr<T> fc, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    // with CORR the aggregate bounds of row i are loaded before the row's
    // product, so their round trip overlaps its gathers
    auto finish = [&](int32_t i, T y, T ri, T di, T ei, int32_t k0, int32_t k1) {
        const T zi = ei + omega * (ri - y) / di;
        eo[i] = zi;
        if constexpr (DOT) acc[0] += (double)rdot[i] * (double)zi;
        if constexpr (CORR) fc.apply(k0, k1, zi);
    };
    if constexpr (CMP) {
        // the row's own values (r, D, e) are loaded before its entries, so
        // their round trip overlaps the entry loads and gathers
        for_each_cmp_slice(A, [&](int64_t, const CmpHead &hd) {
            if (hd.row >= 0) {
                const int32_t i = hd.row;
                int32_t k0 = 0, k1 = 0;
                if constexpr (CORR) {
                    k0 = fc.start[i];
                    k1 = fc.start[i + 1];
                }
                const T ri = r[i], di = A.diag[i], ei = e[i];
                T y = di * ei;  // the row's order: diagonal, then columns
                auto add = [&](int32_t, T v, T xv) { y = y + v * xv; };
                if (A.stream) cmp_entries_at<kCmpBatch, true>(A, hd.b0, hd.w, lane, Direct<T>{e}, add);
                else cmp_entries_at<kCmpBatch, false>(A, hd.b0, hd.w, lane, Direct<T>{e}, add);
                finish(i, y, ri, di, ei, k0, k1);
            }
        });
    } else {
        for_each_slice<product_cap<CMP, T>()>(A.nslices, [&](int64_t s) {
            const int64_t p = s * kWave + lane;
            if (p < A.n) {
                const int32_t i = (int32_t)p;
                int32_t k0 = 0, k1 = 0;
                if constexpr (CORR) {
                    k0 = fc.start[i];
                    k1 = fc.start[i + 1];
                }
                const T y = sell_row<CMP>(A, s, lane, i, Direct<T>{e});
                // the CG's last sweep (DOT) reads r and D nontemporally: the
                // iteration reads neither again before its next CG product
                if constexpr (DOT)
                    finish(i, y, vld<true>(r + i), vld<true>(A.diag + i), e[i], k0, k1);
                else
                    finish(i, y, r[i], A.diag[i], e[i], k0, k1);
            }
        });
    }
    if constexpr (DOT) block_partials<1>(acc, partials);
}

// t = r - A e
template <bool CMP, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_resid(SellView<T> A, const T *__restrict__ r, const T *__restrict__ e,
           T *__restrict__ t, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    for_each_slice<product_cap<CMP, T>()>(A.nslices, [&](int64_t s) {
        const int64_t p = s * kWave + lane;
        if (p < A.n) {
            const int32_t i = sv_row<CMP>(A, p);
            t[i] = r[i] - sell_row<CMP>(A, s, lane, i, Direct<T>{e});
        }
    });
}

// one inner step of the two-stage Gauss-Seidel sweep (Berger-Vergiat et al.
// 2021, the paper's second GPU smoother, Sec. 4.3):
//   g_i = (t_i - sum_{j in tri(i)} A_ij src_j) / D_i
// over the strictly lower (forward sweep) or strictly upper (backward sweep)
// part of row i; src_j = t_j / D_j on the first step (SRC_T), else the
// previous step's g.  mode 0 stores g; mode 1 sets e = g (a sweep from
// zero); mode 2 adds g to e.
template <typename T>
struct DivDiag {
    const T *t, *D;
    __device__ __forceinline__ T operator()(int32_t j) const { return t[j] / D[j]; }
};

template <bool CMP, bool UPPER, bool SRC_T, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_gs(SellView<T> A, const T *__restrict__ t, const T *__restrict__ g, T *__restrict__ out,
        int mode, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    for_each_slice<product_cap<CMP, T>()>(A.nslices, [&](int64_t s) {
        const int64_t p = s * kWave + lane;
        if (p < A.n) {
            const int32_t i = sv_row<CMP>(A, p);
            T y;
            if constexpr (SRC_T) y = sell_tri<CMP, UPPER>(A, s, lane, i, DivDiag<T>{t, A.diag});
            else y = sell_tri<CMP, UPPER>(A, s, lane, i, Direct<T>{g});
            const T gi = (t[i] - y) / A.diag[i];
            out[i] = mode == 2 ? out[i] + gi : gi;
        }
    });
}

// r_c[a] = sum of t over the members of aggregate a, ascending cell order
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_restrict(int32_t nc, const int32_t *__restrict__ start, const int32_t *__restrict__ cells,
              const T *__restrict__ t, T *__restrict__ rc, T *__restrict__ ec_first,
              const T *__restrict__ Dc, T omega, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    GRID_STRIDE(a, nc) {
        const T dc = ec_first ? Dc[a] : T(1);  // loaded ahead of the member sums
        T s = T(0);
        const int32_t k1 = start[a + 1];
        for (int32_t k = start[a]; k < k1; k += kCorrBatch) {  // loads of a batch together
            int32_t j[kCorrBatch];
            T tv[kCorrBatch];
#pragma unroll
            for (int u = 0; u < kCorrBatch; ++u)
                if (k + u < k1) j[u] = cells[k + u];
#pragma unroll
            for (int u = 0; u < kCorrBatch; ++u)
                if (k + u < k1) tv[u] = t[j[u]];
#pragma unroll
            for (int u = 0; u < kCorrBatch; ++u)
                if (k + u < k1) s += tv[u];
        }
        rc[a] = s;
        // the coarse level's first Jacobi sweep from zero, e_c = omega r_c / D_c
        if (ec_first) ec_first[a] = omega * s / dc;
    }
}

// ---------------------------------------------------------------- restriction operator
// The down leg of a cycle whose pre-smoothing is one Jacobi sweep from zero,
// e = omega D^-1 r, followed by the residual and its restriction (the
// agglomeration's summation, Sec. 4.3):
//   r_c = P^T (r - A e) = P^T (I - omega A D^-1) r = R r,
//   R_cj = sum over the members i of c, ascending, of (1 - omega) when
//          j = i and -omega a_ij / D_j for the entries a_ij of row i.
// One pass over R replaces the residual kernel (which writes t) and the
// restriction (which reads it back through the member lists); the two are
// equal up to rounding.  valT holds R for A^T (a_ji).
// A large plain-slice level (a fine mesh) keeps the two steps but folds the
// sweep into its own slices: t = (I - omega A D^-1) r is a product over the
// level's layout, 16-bit columns included, with the values -omega a_ij / D_j
// (Ah), and the member sums of t follow.  R's rows there would gather from
// members of several orientations at once (a pair along z reaches two mesh
// planes, a pair along x one), so each of their gathers touches about three
// times as many cache lines per entry as the level's own rows do.

// entries a coarse row gathers before merging: its members' row entries and
// their diagonals; *wide (when given) for a row of more than kGatherPairs
constexpr int kGatherPairs = 512;

__global__ void k_rop_count(int32_t nc, const int32_t *__restrict__ start,
                            const int32_t *__restrict__ cells, Sell A, int64_t *cnt,
                            int64_t *wide) {
    GRID_STRIDE(c, nc) {
        int64_t m = 0;
        for (int32_t k = start[c]; k < start[c + 1]; ++k) {
            const int32_t i = cells[k];
            const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
            const int w = row_len(A, ps);
            m += 1;
            if (A.pdeg) m += w;  // compressed slices hold no padding
            else
                for (int q = 0; q < w; ++q) m += A.col[entry_at(A, ps, q)] != i;
        }
        cnt[c] = m;
        if (wide && m > kGatherPairs) *wide = 1;
    }
}

// per coarse row: the member contributions in member order, each member's in
// column order, as (column, source) pairs (source: the entry's position in
// the level's slices, or -1 for a member's own diagonal), ordered by column
// with equal columns in member order.  rdeg: the number of distinct columns.
// One wave per coarse row: the members' row headers are loaded side by side,
// each member's entries by as many lanes, into LDS, and a pair's place is the
// number of pairs that sort before it (all lanes read the same pair at a
// time, a broadcast).  A thread per row with an insertion sort in global
// memory took 21 ms on the 1.8M-cell merged hierarchy; this takes 0.9 ms.
// Rows of more pairs than the LDS holds are sorted by one lane in place.

__global__ void __launch_bounds__(kBlock)
k_rop_gather(int32_t nc, const int32_t *__restrict__ start, const int32_t *__restrict__ cells,
             Sell A, const int64_t *__restrict__ tstart, int32_t *tcol, int64_t *tsrc,
             int32_t *rdeg) {
    __shared__ int32_t sc[kWavesPerBlock][kGatherPairs];
    __shared__ int64_t ss[kWavesPerBlock][kGatherPairs];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t below = (uint64_t(1) << lane) - 1;
    int32_t *pc = sc[wv];
    int64_t *psrc = ss[wv];
    const GridRange gr = grid_range(nc, kWavesPerBlock);
    for (int64_t c = gr.begin + wv; c < gr.end; c += gr.step) {
        const int64_t o = tstart[c];
        const int m = (int)(tstart[c + 1] - o);
        const bool lds = m <= kGatherPairs;
        const int32_t k0 = start[c], k1 = start[c + 1];
        int base = 0;
        for (int32_t kb = k0; kb < k1; kb += kWave) {
            const int nm = min(kWave, k1 - kb);
            int32_t mi = 0, mw = 0, mt = 0;
            int64_t mb = 0;
            if (lane < nm) {
                mi = cells[kb + lane];
                const int64_t ps = A.iperm ? (int64_t)A.iperm[mi] : (int64_t)mi;
                mw = row_len(A, ps);
                mb = A.sptr[ps >> 6] + (ps & 63);
                if (A.pdeg) mt = A.tptr[ps >> 6];
            }
            for (int u = 0; u < nm; ++u) {
                const int32_t i = __shfl(mi, u), w = __shfl(mw, u), t = __shfl(mt, u);
                const int64_t b0 = __shfl(mb, u);
                int nv = 0, nb = 0;  // entries so far, and those left of the diagonal
                for (int q0 = 0; q0 < w; q0 += kWave) {
                    const int q = q0 + lane;
                    int32_t j = i;
                    int64_t e = -1;
                    if (q < w) {
                        e = b0 + (A.pdeg ? (int64_t)A.otab[t + q] : (int64_t)q * kWave);
                        j = A.col[e];
                    }
                    const uint64_t in = __ballot(j != i);  // padding points at the row
                    const int at = base + nv + __popcll(in & below) + (j > i ? 1 : 0);
                    if (j != i) {
                        if (lds) {
                            pc[at] = j;
                            psrc[at] = e;
                        } else {
                            tcol[o + at] = j;
                            tsrc[o + at] = e;
                        }
                    }
                    nv += __popcll(in);
                    nb += __popcll(__ballot(j != i && j < i));
                }
                if (lane == 0) {
                    if (lds) {
                        pc[base + nb] = i;
                        psrc[base + nb] = -1;
                    } else {
                        tcol[o + base + nb] = i;
                        tsrc[o + base + nb] = -1;
                    }
                }
                base += nv + 1;
            }
        }
        if (!lds) {
            // the wave's own stores, then one lane's stable insertion sort
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            if (lane == 0) {
                int u = 0;
                for (int a = 0; a < m; ++a) {
                    const int32_t kc = tcol[o + a];
                    const int64_t ks = tsrc[o + a];
                    int b = a - 1;
                    while (b >= 0 && tcol[o + b] > kc) {
                        tcol[o + b + 1] = tcol[o + b];
                        tsrc[o + b + 1] = tsrc[o + b];
                        --b;
                    }
                    tcol[o + b + 1] = kc;
                    tsrc[o + b + 1] = ks;
                }
                for (int a = 0; a < m; ++a) u += a == 0 || tcol[o + a] != tcol[o + a - 1];
                rdeg[c] = u;
            }
            continue;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int distinct = 0;
        for (int t0 = 0; t0 < m; t0 += kWave) {
            const int t = t0 + lane;
            const int32_t j = t < m ? pc[t] : INT32_MAX;
            int place = 0;
            bool seen = false;
            for (int u = 0; u < m; ++u) {
                const int32_t ju = pc[u];
                const bool same = ju == j && u < t;
                place += ju < j || same;
                seen = seen || same;
            }
            if (t < m) {
                tcol[o + place] = j;
                tsrc[o + place] = psrc[t];
            }
            distinct += __popcll(__ballot(t < m && !seen));
        }
        if (lane == 0) rdeg[c] = distinct;
        __builtin_amdgcn_wave_barrier();
    }
}

// R's columns, and for each entry of R the run of its sources in the sorted
// pairs (start, count): compressed slices
__global__ void k_rop_link_sell(int32_t nc, Sell R, const int64_t *__restrict__ tstart,
                                const int32_t *__restrict__ tcol, int64_t *rs0, int32_t *rsn) {
    GRID_STRIDE(c, nc) {
        const int64_t ps = R.iperm[c], o = tstart[c], o1 = tstart[c + 1];
        int q = 0;
        for (int64_t a = o; a < o1;) {
            int64_t b = a + 1;
            while (b < o1 && tcol[b] == tcol[a]) ++b;
            const int64_t e = entry_at(R, ps, q++);
            R.col[e] = tcol[a];
            rs0[e] = a;
            rsn[e] = (int32_t)(b - a);
            a = b;
        }
    }
}

// the same for CSR
__global__ void k_rop_link_csr(int32_t nc, Csr R, const int64_t *__restrict__ tstart,
                               const int32_t *__restrict__ tcol, int64_t *rs0, int32_t *rsn) {
    GRID_STRIDE(c, nc) {
        const int64_t o = tstart[c], o1 = tstart[c + 1];
        int64_t e = R.rptr[c];
        for (int64_t a = o; a < o1;) {
            int64_t b = a + 1;
            while (b < o1 && tcol[b] == tcol[a]) ++b;
            R.col[e] = tcol[a];
            rs0[e] = a;
            rsn[e] = (int32_t)(b - a);
            ++e;
            a = b;
        }
    }
}

__global__ void k_widen(int32_t n, const int32_t *__restrict__ a, int64_t *__restrict__ b) {
    GRID_STRIDE(i, n) b[i] = a[i];
}

// values of R (and of its A^T form) from the level's coefficients: each entry
// sums its sources in member order, (1 - omega) for a diagonal and
// -omega a / D_j for an entry a of column j.  Bound by the scattered reads of
// a; four sources are in flight (430,000 fine rows, merged: 449 -> 343 us)
template <class M>
__global__ void k_rop_values(int64_t nnz, M R, const int64_t *__restrict__ rs0,
                             const int32_t *__restrict__ rsn, const int64_t *__restrict__ src,
                             const double *__restrict__ aval, const double *__restrict__ avalT,
                             const double *__restrict__ D, double omega) {
    GRID_STRIDE(e, nnz) {
        const int64_t k0 = rs0[e], k1 = k0 + rsn[e];
        const double dj = D[R.col[e]];
        double v = 0.0, vT = 0.0;
        for (int64_t k = k0; k < k1; k += 4) {
            int64_t q[4];
            double a[4], t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = k + u < k1 ? src[k + u] : -1;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = q[u] < 0 ? 0.0 : aval[q[u]];
                t[u] = q[u] < 0 ? 0.0 : avalT[q[u]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k + u < k1) {
                    v = v + (q[u] < 0 ? 1.0 - omega : (-omega * a[u]) / dj);
                    vT = vT + (q[u] < 0 ? 1.0 - omega : (-omega * t[u]) / dj);
                }
        }
        R.val[e] = v;
        R.valT[e] = vT;
    }
}

__global__ void k_rop_f32(const double *a, float *b, int64_t n) {
    STREAM_STRIDE(i, n)
        b[i] = (float)a[i];
}

// Ah = -omega A D^-1 at the positions of a plain-slice level's entries (the
// same expression as a source of R's values); padding (value 0) stays 0
__global__ void k_ahat_values(int64_t nnz, const int32_t *__restrict__ col,
                              const double *__restrict__ val, const double *__restrict__ valT,
                              const double *__restrict__ D, double omega, double *__restrict__ ah,
                              double *__restrict__ ahT) {
    GRID_STRIDE(e, nnz) {
        const double dj = D[col[e]];
        ah[e] = (-omega * val[e]) / dj;
        ahT[e] = (-omega * valT[e]) / dj;
    }
}

// t = (I - omega A D^-1) r over a plain-slice level whose values are Ah:
// row i is (1 - omega) r_i plus its entries in column order
template <bool C16, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_ahat(SellView<T> Ah, const T *__restrict__ r, T *__restrict__ t, T c0,
          const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    for_each_slice<product_cap<false, T>()>(Ah.nslices, [&](int64_t s) {
        const int64_t p = s * kWave + lane;
        if (p < Ah.n) {
            T y = c0 * r[p];
            plain_entries<C16, 8>(Ah, s, lane, Direct<T>{r},
                                  [&](int32_t, T v, T xv) { y = y + v * xv; });
            t[p] = y;
        }
    });
}

// cycles whose down leg R replaces: Jacobi, one pre-sweep, no correction
// scaling (which needs the residual itself)
static bool rop_cycle(const ldu_gamg_opts &o) {
    return o.smoother == LDU_SMOOTH_JACOBI && o.n_pre == 1 && !o.scale_correction;
}

// entries a lane of the compressed-slice R product loads before its gathers:
// R's rows are longer than the level's own (47 entries on the c3 headline's
// level 1), so it takes larger batches than kCmpBatch (FP64 solves with 24,
// 32 and 48 entries: 147.2, 146.0 and 148.0 ms; mixed ones: 116.4, 115.5
// and 114.3 ms)
template <typename T>
constexpr int kRBatch = sizeof(T) == 8 ? 32 : 48;

// r_c = R r (row c: columns ascending, from zero), and the coarse level's
// first Jacobi sweep from zero e_c = omega r_c / D_c when ec_first is given
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_rrestrict_cmp(SellView<T> R, const T *__restrict__ r, T *__restrict__ rc,
               T *__restrict__ ec_first, const T *__restrict__ Dc, T omega,
               const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    for_each_cmp_slice(R, [&](int64_t, const CmpHead &hd) {
        if (hd.row >= 0) {
            const int32_t c = hd.row;
            // the coarse diagonal is loaded before the row, so its round
            // trip overlaps the row's gathers
            const T dc = ec_first ? Dc[c] : T(1);
            T acc = T(0);
            cmp_entries_at<kRBatch<T>>(R, hd.b0, hd.w, lane, Direct<T>{r},
                                       [&](int32_t, T v, T xv) { acc = acc + v * xv; });
            rc[c] = acc;
            if (ec_first) ec_first[c] = omega * acc / dc;
        }
    });
}

// the sum over row c of R of value times x(column), shared by G lanes: lane g
// of the group sums the row's entries g, g + G, g + 2G, ... in order, then
// the group adds its G partial sums by a fixed butterfly (every lane ends
// with the same total).  The order is fixed, so results are reproducible; it
// is not the row's column order.  Every lane of the wave calls this (lanes
// without a row: c >= R.n).
template <int G, bool NT, typename T, class XA>
__device__ __forceinline__ T csr_row_sum(const CsrView<T> &R, int64_t c, int g, const XA &x) {
    constexpr int U = kCsrBatch;
    T acc = T(0);
    if (c < R.n) {
        const int64_t e1 = R.rptr[c + 1];
        for (int64_t k0 = R.rptr[c] + g; k0 < e1; k0 += (int64_t)G * U) {
            int32_t cc[U];
            T vv[U], xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t k = k0 + (int64_t)u * G;
                if (k < e1) {
                    cc[u] = vld<NT>(R.col + k);
                    vv[u] = vld<NT>(R.val + k);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + (int64_t)u * G < e1) xv[u] = x(cc[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + (int64_t)u * G < e1) acc = acc + vv[u] * xv[u];
        }
    }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) acc = acc + __shfl_xor(acc, off);
    return acc;
}

// r_c = R r, and the coarse level's first Jacobi sweep from zero
// e_c = omega r_c / D_c when ec_first is given.  G lanes share a row, so a
// wave covers 64 / G consecutive rows.  R's results never had to follow the
// row's column order (R's rows are sums the oracle forms in two steps,
// residual then restriction).
template <int G, bool NT, typename T, class XA>
__global__ void __launch_bounds__(kBlock)
k_vc_rrestrict_csr(CsrView<T> R, XA x, T *__restrict__ rc,
               T *__restrict__ ec_first, const T *__restrict__ Dc, T omega,
               const DevScalars *ds) {
    const bool skip = vc_skip(ds);  // tested before the stores, off the chain of loads
    constexpr int RPW = kWave / G;
    const int lane = threadIdx.x & 63;
    const int g = lane % G;
    const int64_t chunks = (R.n + RPW - 1) / RPW;
    for_each_slice(chunks, [&](int64_t s) {
        const int64_t c = s * RPW + lane / G;
        // the coarse diagonal is loaded before the row, so its round trip
        // overlaps the row's gathers
        const T dc = (ec_first && g == 0 && c < R.n) ? Dc[c] : T(1);
        const T acc = csr_row_sum<G, NT>(R, c, g, x);
        if (c < R.n && g == 0 && !skip) {
            rc[c] = acc;
            if (ec_first) ec_first[c] = omega * acc / dc;
        }
    });
}

// ---------------------------------------------------------------- up-leg operator
// The up leg of the same cycles on a small level: the first sweep from zero,
// the coarse correction and the first post-sweep are together one linear map
// of the level's right-hand side and the coarse result,
//   e0 = omega D^-1 r + P e_c,  e = e0 + omega D^-1 (r - A e0)
//      = S r + Q e_c = U (r, e_c),
//   S = omega D^-1 (2 I - omega A D^-1),  Q = (I - omega D^-1 A) P.
// As separate steps the coarse level scattered its result through the member
// lists and the sweep then ran a lane per row: eight dependent round trips to
// memory (slice start, row header, entries, gathers, a second batch, members,
// their values), about 8 us a level, on levels whose data takes under 1 us.
// U's rows are shared by G lanes like R's, which leaves row bounds, entries
// and gathers.  Levels of 600 to 50,000 cells (100^3 box, pairwise): 8.0-12.1
// -> 4.0-7.5 us; 102,000 cells: 12.9 -> 15.2 us, so larger levels keep the
// separate steps (kUpRows).  CG + V-cycle on that box 18.5 -> 17.0 ms.
// Columns: j < n for r_j, n + c for e_c's entry c; a row holds its S entries
// in column order (diagonal in place), then its Q entries by aggregate.
template <typename T>
struct Stacked {
    const T *r, *ec;
    int32_t n;
    __device__ __forceinline__ T operator()(int32_t j) const {
        const T *p = j < n ? r + j : ec + (j - n);
        return *p;
    }
};

template <int G, bool DOT, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_up_csr(CsrView<T> U, const T *__restrict__ r, const T *__restrict__ ec, T *__restrict__ e,
            const T *__restrict__ rdot, double *partials, const DevScalars *ds) {
    const bool skip = vc_skip(ds);  // tested before the stores, off the chain of loads
    constexpr int RPW = kWave / G;
    const int lane = threadIdx.x & 63;
    const int g = lane % G;
    const int64_t chunks = (U.n + RPW - 1) / RPW;
    double acc[1] = {0.0};
    for_each_slice(chunks, [&](int64_t s) {
        const int64_t i = s * RPW + lane / G;
        const T z = csr_row_sum<G, false>(U, i, g, Stacked<T>{r, ec, U.n});
        if (i < U.n && g == 0 && !skip) {
            e[i] = z;
            if constexpr (DOT) acc[0] += (double)rdot[i] * (double)z;
        }
    });
    if (skip) return;
    if constexpr (DOT) block_partials<1>(acc, partials);
}

// 16 lanes share a row of U or V: kUpHeld aggregates held by a lane bound the
// aggregates of a row (64), and a level with a row of more runs its up leg step
// by step, as does one for the general cycles whose coarse rows gather more pairs
// than k_rop_gather's LDS holds.  Such rows (a cell with hundreds of neighbours)
// went to one lane, which looks through what it has found for every entry: on a
// chain of 3000 cells with a cell of 120 more neighbours set-up 5.4 -> 20.9 ms
// and a cycle after new coefficients 0.5 -> 3.7 ms, growing with the square.
constexpr int kUpLanes = kRowLanes;
constexpr int kUpHeld = 4;

// the aggregates that a group of kUpLanes lanes has found in its row: the k-th
// is lane k % kUpLanes's.  add() is called by the whole group, for one entry
struct HeldAggregates {
    int32_t c[kUpHeld];
    int found = 0;
    __device__ HeldAggregates() {
#pragma unroll
        for (int h = 0; h < kUpHeld; ++h) c[h] = -1;
    }
    // old(h): this lane's h-th aggregate is cu; made(h): it is cu now
    template <class Old, class New>
    __device__ __forceinline__ void add(int32_t cu, uint64_t mine, int l, Old &&old, New &&made) {
        bool hit = false;
#pragma unroll
        for (int h = 0; h < kUpHeld; ++h)
            if (c[h] == cu) {
                old(h);
                hit = true;
            }
        if (__ballot(hit) & mine) return;
#pragma unroll
        for (int h = 0; h < kUpHeld; ++h)
            if (found == h * kUpLanes + l) {
                c[h] = cu;
                made(h);
            }
        ++found;
    }
};

// row lengths of U and V: the row's entries (with the diagonal) and the
// distinct aggregates they lie in; *wide for a row of too many
__global__ void __launch_bounds__(kBlock)
k_up_count(Sell A, const int32_t *__restrict__ agg, int64_t *cnt, int64_t *wide) {
    const int l = threadIdx.x % kUpLanes;
    const int g0 = (threadIdx.x & 63) - l;  // the group's first lane
    const uint64_t mine = ((uint64_t(1) << kUpLanes) - 1) << g0;
    ROW_GROUPS(row, A.n) {
        if (row >= A.n) continue;  // the whole group
        const int32_t i = (int32_t)row;
        const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
        const int w = row_len(A, ps);
        const int32_t own = agg[i];
        HeldAggregates held;
        held.add(own, mine, l, [](int) {}, [](int) {});
        int m = 1;
        for (int k0 = 0; k0 < w && held.found <= kUpHeld * kUpLanes; k0 += kUpLanes) {
            const int32_t j = k0 + l < w ? A.col[entry_at(A, ps, k0 + l)] : i;
            const int32_t cj = j != i ? agg[j] : own;  // padding points at the row
            m += __popcll(__ballot(j != i) & mine);
            for (int u = 0; u < kUpLanes && k0 + u < w; ++u)
                held.add(__shfl(cj, g0 + u), mine, l, [](int) {}, [](int) {});
        }
        if (l == 0) {
            cnt[i] = m + held.found;
            if (held.found > kUpHeld * kUpLanes) *wide = 1;
        }
    }
}

// U's columns and values (val: A, valT: A^T) for this omega.  16 lanes share a
// row: each forms one S entry of 16, and then every lane sees the 16 in column
// order and sums those of the aggregates that it holds (the k-th found is
// lane k % 16's).  A lane that formed its row alone kept the sums in U, one
// chain of loads and stores.  Levels of 16,000, 1,700 and 190 rows of a merged
// hierarchy: 150 + 171 + 92 -> 20 + 15 + 12 us (with the other refresh kernels a
// 151^3 time step 13.2 -> 12.6 ms, a 100^3 solve and its gradient 43.8 -> 42.1).
// V (GEN) has A's own entries in place of S's and its Q entries start at qptr.
// Formed by a thread a row, V made new coefficients and one default GAMG cycle
// dearer than they had been without it (32^3, 64^3 and 128^3: 0.69, 0.98 and
// 2.46 ms): 1.51, 2.30 and 3.72 ms, now 0.83, 1.13 and 2.41; with four cycles
// 2.17, 3.32 and 6.44 -> 1.48, 2.15 and 5.13 (without V 1.88, 2.80 and 6.17).
template <bool GEN>
__global__ void __launch_bounds__(kBlock)
k_up_fill(Sell A, Csr U, int64_t *qptr, const int32_t *__restrict__ agg, double omega) {
    const int l = threadIdx.x % kUpLanes;
    const int g0 = (threadIdx.x & 63) - l;  // the group's first lane
    const uint64_t mine = ((uint64_t(1) << kUpLanes) - 1) << g0;
    ROW_GROUPS(row, A.n) {
        if (row >= A.n) continue;  // the whole group
        const int32_t i = (int32_t)row;
        const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
        const int w = row_len(A, ps);
        const int64_t e0 = U.rptr[i], e1 = U.rptr[i + 1];
        int below = 0, m = 1;  // entries before the diagonal, and with it
        for (int k = 0; k < w; k += kUpLanes) {
            const int32_t j = k + l < w ? A.col[entry_at(A, ps, k + l)] : i;
            below += __popcll(__ballot(j < i) & mine);
            m += __popcll(__ballot(j != i) & mine);  // padding points at the row
        }
        const int64_t q0 = e0 + m;
        if (GEN && l == 0) qptr[i] = q0;
        const double wi = omega / A.diag[i];
        HeldAggregates held;
        double v[kUpHeld], vT[kUpHeld];
        for (int t0 = 0; t0 < m; t0 += kUpLanes) {
            const int t = t0 + l;
            int32_t cj = -1;
            double a = 0.0, at = 0.0;
            if (t < m) {
                const int64_t e = t == below ? -1 : entry_at(A, ps, t < below ? t : t - 1);
                const int32_t j = e < 0 ? i : A.col[e];
                const double dj = A.diag[j];
                a = e < 0 ? dj : A.val[e];
                at = e < 0 ? dj : A.valT[e];
                cj = A.n + agg[j];
                U.col[e0 + t] = j;
                U.val[e0 + t] = GEN ? a : e < 0 ? wi * (2.0 - omega) : wi * ((-omega * a) / dj);
                U.valT[e0 + t] = GEN ? at : e < 0 ? wi * (2.0 - omega) : wi * ((-omega * at) / dj);
            }
            for (int u = 0; u < kUpLanes && t0 + u < m; ++u) {
                const double au = __shfl(a, g0 + u), atu = __shfl(at, g0 + u);
                held.add(
                    __shfl(cj, g0 + u), mine, l,
                    [&](int h) {
                        v[h] = v[h] + au;
                        vT[h] = vT[h] + atu;
                    },
                    [&](int h) {
                        v[h] = 0.0 + au;
                        vT[h] = 0.0 + atu;
                    });
            }
        }
        const int32_t own = A.n + agg[i];
#pragma unroll
        for (int h = 0; h < kUpHeld; ++h) {
            const int64_t k = q0 + h * kUpLanes + l;
            if (k < e1) {
                const double p = held.c[h] == own ? 1.0 : 0.0;
                U.col[k] = held.c[h];
                U.val[k] = p - wi * v[h];
                U.valT[k] = p - wi * vT[h];
            }
        }
    }
}

// ---------------------------------------------------------------- up leg of a large plain level
// A large plain-slice level (form: scaled slices) has t = (I - omega A D^-1) r
// from its down leg.  Its up leg to the end of the first post-sweep is
//   e = S r + (I - omega D^-1 A) P e_c,   S r = omega D^-1 (r + t),
// that is  e_i = c_i + omega (r_i + t_i - (A P e_c)_i) / D_i,  c = P e_c:  a
// product with A's values that gathers from the coarse vector (AC: A's slices
// with their columns mapped to aggregates).  The correction (r, D, the map and
// e_c in, e out) and the sweep after it (A, e, r, D in) were two passes.
// 200^3 in FP64: correction and sweep 44 + 137 us, this kernel 161 (columns
// mapped in the kernel, e_c[agg[j]], chain two gathers: 204); CG + V-cycle
// 124.7 -> 122.4 ms there, 15.3 -> 14.8 ms on 100^3.  The map is read past the
// caches and D through them: the CG product that follows finds D there (132
// -> 125 us; 123.1 -> 122.3 ms).
template <bool DOT, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_up_slices(SellView<T> AC, const int32_t *__restrict__ agg, const T *__restrict__ r,
               const T *__restrict__ t, const T *__restrict__ ec, T *__restrict__ e, T omega,
               double *partials, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice<product_cap<false, T>()>(AC.nslices, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < AC.n) {
            const T ci = ec[vld<true>(agg + i)];
            const T di = AC.diag[i];
            T y = di * ci;
            row_entries<false, 8>(AC, s, lane, Direct<T>{ec},
                                  [&](int32_t, T v, T xv) { y = y + v * xv; });
            // with DOT the iteration does not read r before its CG product (which
            // finds D, read with the default policy, in the Infinity Cache)
            const T ri = vld<DOT>(r + i);
            const T zi = ci + omega * (ri + vld<true>(t + i) - y) / di;
            e[i] = zi;
            if constexpr (DOT) acc[0] += (double)ri * (double)zi;
        }
    });
    if constexpr (DOT) block_partials<1>(acc, partials);
}

template <typename T>
static int launch_up_slices(const Level &L, SellView<T> A, const T *r, const T *t, const T *ec,
                            T *e, T omega, bool dot, double *partials, const DevScalars *ds,
                            hipStream_t st) {
    A.c16 = L.ac16;
    A.cbase = L.acbase;
    A.col = L.ac32;
    int G = stream_grid_slices(A.nslices);
    // with a dot product, blocks past the products' cap would only add zeros
    if (dot && sizeof(T) == sizeof(double)) G = std::min(G, kPlainF64ProductBlocks);
    if (dot)
        k_vc_up_slices<true, T><<<G, kBlock, 0, st>>>(A, L.agg, r, t, ec, e, omega, partials, ds);
    else
        k_vc_up_slices<false, T><<<G, kBlock, 0, st>>>(A, L.agg, r, t, ec, e, omega, partials, ds);
    return G;
}

// f(std::integral_constant<int, lanes per row>)
template <class F>
static void with_group(int group, F &&f) {
    switch (group) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    default: f(std::integral_constant<int, 16>{});
    }
}

// the number of blocks launched (of partials, with rdot)
template <typename T>
static int launch_up_csr(const CsrView<T> &U, const T *r, const T *ec, T *e, const T *rdot,
                         double *partials, const DevScalars *ds, hipStream_t st) {
    const int64_t chunks = (U.n + kWave / U.group - 1) / (kWave / U.group);
    const int G = stream_grid_slices(chunks);
    with_group(U.group, [&](auto lanes) {
        constexpr int L = decltype(lanes)::value;
        if (rdot) k_vc_up_csr<L, true, T><<<G, kBlock, 0, st>>>(U, r, ec, e, rdot, partials, ds);
        else k_vc_up_csr<L, false, T><<<G, kBlock, 0, st>>>(U, r, ec, e, rdot, partials, ds);
    });
    return G;
}

// x: the vector R's columns refer to (r, or (r, e) for W)
template <typename T, class XA>
static void launch_rrestrict_csr(const CsrView<T> &R, const XA &x, T *rc, T *ec_first, const T *Dc,
                                 T omega, const DevScalars *ds, hipStream_t st) {
    const int64_t chunks = (R.n + kWave / R.group - 1) / (kWave / R.group);
    const int G = stream_grid_slices(chunks);
    const bool nt = R.nnz * (int64_t)(sizeof(int32_t) + sizeof(T)) > kCsrCachedBytes;
    with_group(R.group, [&](auto lanes) {
        constexpr int L = decltype(lanes)::value;
        if (nt)
            k_vc_rrestrict_csr<L, true, T, XA><<<G, kBlock, 0, st>>>(R, x, rc, ec_first, Dc, omega, ds);
        else
            k_vc_rrestrict_csr<L, false, T, XA><<<G, kBlock, 0, st>>>(R, x, rc, ec_first, Dc, omega, ds);
    });
}

// The correction's scaling factor s = (c.t) / (c.A c) with c = P e_c, or 1
// when c.A c is ~0.  By the Galerkin product c.A c = e_c.(P^T A P) e_c =
// e_c.A_c e_c, and c.t = e_c.P^T t = e_c.r_c, so both sums run over the coarse
// level: half its rows or fewer, and gathers of e_c itself instead of
// e_c[agg[j]].  On level 0 of a shuffled 128^3 mesh 339 -> 94 us, on its
// 215,000-cell level 25 -> 15 us.  The correction takes the sums from the
// partials itself.  Standalone GAMG, default settings: 87.3 -> 72 ms there,
// 38.4 -> 33 ms in natural order.
template <bool CMP, typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_energy(SellView<T> A, const T *__restrict__ ec, const T *__restrict__ rc, double *partials,
            const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    double acc[2] = {0.0, 0.0};
    for_each_slice<product_cap<CMP, T>()>(A.nslices, [&](int64_t s) {
        const int64_t p = s * kWave + lane;
        if (p < A.n) {
            const int32_t i = sv_row<CMP>(A, p);
            const T ac = sell_row<CMP>(A, s, lane, i, Direct<T>{ec});
            const T ci = ec[i];
            acc[0] += (double)ci * (double)rc[i];
            acc[1] += (double)ci * (double)ac;
        }
    });
    block_partials<2>(acc, partials);
}

// the factor from its two sums
__device__ __forceinline__ double correction_scale(const double (&v)[2]) {
    return (isfinite(v[1]) && fabs(v[1]) > 1e-300) ? v[0] / v[1] : 1.0;
}

// ---------------------------------------------------------------- small levels, general cycles
// Small levels of cycles without the one-pass down leg (two pre-sweeps,
// scaled corrections: the solver's defaults) with G lanes per row, as R and U:
//   sweep:    e' = e + omega (r - A e) / D
//   restrict: r_c = P^T r - (P^T A) e        (W over (r, e))
//   up:       e' = e0 + s P e_c + omega D^-1 (r - A (e0 + s P e_c))
//                = e0 + omega (r - A e0) / D + s Q e_c,  Q = (I - omega D^-1 A) P
//   energy:   e.r and e.A e of the coarse level
// A row of V holds A's entries (diagonal included) and behind them Q's.  A
// level takes five launches of about 4 us for two sweeps each way; with a lane
// per row, and residual, member sums, correction and sweep apart, it took seven
// of 4-12 us.  Standalone GAMG, default settings: 128^3 33.2 -> 27.9
// ms, 64^3 12.3 -> 8.8 ms, 16^3 3.8 -> 2.5 ms.
// one row of V by G lanes: the sums over its A entries (e) and, with UP, its Q
// entries (ec); every lane of the wave calls this
template <int G, bool UP, typename T>
__device__ __forceinline__ void v_row_sums(const CsrView<T> &V, const int64_t *__restrict__ qptr,
                                           int64_t i, int g, const T *__restrict__ e,
                                           const T *__restrict__ ec, T &sa, T &sq) {
    constexpr int U = kCsrBatch;
    sa = sq = T(0);
    if (i < V.n) {
        const int64_t e1 = UP ? V.rptr[i + 1] : qptr[i];
        for (int64_t k0 = V.rptr[i] + g; k0 < e1; k0 += (int64_t)G * U) {
            int32_t cc[U];
            T vv[U], xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t k = k0 + (int64_t)u * G;
                if (k < e1) {
                    cc[u] = V.col[k];
                    vv[u] = V.val[k];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + (int64_t)u * G < e1) {
                    if constexpr (UP) xv[u] = cc[u] < V.n ? e[cc[u]] : ec[cc[u] - V.n];
                    else xv[u] = e[cc[u]];
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + (int64_t)u * G < e1) {
                    if (!UP || cc[u] < V.n) sa = sa + vv[u] * xv[u];
                    else sq = sq + vv[u] * xv[u];
                }
        }
    }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) {
        sa = sa + __shfl_xor(sa, off);
        if constexpr (UP) sq = sq + __shfl_xor(sq, off);
    }
}

// eo = e + omega (r - A e) / D, with UP plus s Q ec (s from the nblocks
// partials of an energy kernel, 1 without any); DOT: partials of rdot . eo in
// dots
template <int G, bool UP, bool DOT, typename T>
__global__ void __launch_bounds__(kBlock)
k_gen_sweep(CsrView<T> V, const int64_t *__restrict__ qptr, const T *__restrict__ D,
            const T *__restrict__ r, const T *__restrict__ e, const T *__restrict__ ec,
            T *__restrict__ eo, T omega, const double *__restrict__ scale, int nblocks,
            const T *__restrict__ rdot, double *dots, const DevScalars *ds) {
    const bool skip = vc_skip(ds);  // tested before the stores, off the chain of loads
    T sc = T(1);
    if (UP && nblocks > 0) {
        double v[2];
        sum_partials<2>(scale, nblocks, v);
        sc = (T)correction_scale(v);
    }
    constexpr int RPW = kWave / G;
    const int lane = threadIdx.x & 63;
    const int g = lane % G;
    const int64_t chunks = (V.n + RPW - 1) / RPW;
    double acc[1] = {0.0};
    for_each_slice(chunks, [&](int64_t s) {
        const int64_t i = s * RPW + lane / G;
        const bool own = i < V.n && g == 0;
        const T ri = own ? r[i] : T(0), di = own ? D[i] : T(1), ei = own ? e[i] : T(0);
        T sa, sq;
        v_row_sums<G, UP>(V, qptr, i, g, e, ec, sa, sq);
        if (own) {
            T z = ei + omega * (ri - sa) / di;
            if constexpr (UP) z = z + sc * sq;
            if (!skip) eo[i] = z;
            if constexpr (DOT) acc[0] += (double)rdot[i] * (double)z;
        }
    });
    if (skip) return;
    if constexpr (DOT) block_partials<1>(acc, dots);
}

// partials of e.r and e.A e
template <int G, typename T>
__global__ void __launch_bounds__(kBlock)
k_gen_energy(CsrView<T> V, const int64_t *__restrict__ qptr, const T *__restrict__ e,
             const T *__restrict__ r, double *partials, const DevScalars *ds) {
    const bool skip = vc_skip(ds);
    constexpr int RPW = kWave / G;
    const int lane = threadIdx.x & 63;
    const int g = lane % G;
    const int64_t chunks = (V.n + RPW - 1) / RPW;
    double acc[2] = {0.0, 0.0};
    for_each_slice(chunks, [&](int64_t s) {
        const int64_t i = s * RPW + lane / G;
        const bool own = i < V.n && g == 0;
        const T ri = own ? r[i] : T(0), ei = own ? e[i] : T(0);
        T sa, sq;
        v_row_sums<G, false>(V, qptr, i, g, e, e, sa, sq);
        if (own) {
            acc[0] += (double)ei * (double)ri;
            acc[1] += (double)ei * (double)sa;
        }
    });
    if (skip) return;
    block_partials<2>(acc, partials);
}

// W: the members of row c (value 1, columns j), then its P^T A entries
// (columns n + j), from the gathered pairs of k_rop_gather
__global__ void k_w_count(int32_t nc, const int32_t *__restrict__ start,
                          const int32_t *__restrict__ rdeg, int64_t *cnt) {
    GRID_STRIDE(c, nc) cnt[c] = rdeg[c] + (start[c + 1] - start[c]);
}
__global__ void k_w_link(int32_t nc, int32_t n, Csr W, const int32_t *__restrict__ start,
                         const int32_t *__restrict__ cells, const int64_t *__restrict__ tstart,
                         const int32_t *__restrict__ tcol, int64_t *ws0, int32_t *wsn) {
    GRID_STRIDE(c, nc) {
        int64_t e = W.rptr[c];
        for (int32_t k = start[c]; k < start[c + 1]; ++k, ++e) {
            W.col[e] = cells[k];
            W.val[e] = W.valT[e] = 1.0;
            ws0[e] = 0;
            wsn[e] = 0;
        }
        const int64_t o1 = tstart[c + 1];
        for (int64_t a = tstart[c]; a < o1; ++e) {
            int64_t b = a + 1;
            while (b < o1 && tcol[b] == tcol[a]) ++b;
            W.col[e] = n + tcol[a];
            ws0[e] = a;
            wsn[e] = (int32_t)(b - a);
            a = b;
        }
    }
}
__global__ void k_w_values(int64_t nnz, int32_t n, Csr W, const int64_t *__restrict__ ws0,
                           const int32_t *__restrict__ wsn, const int64_t *__restrict__ src,
                           const double *__restrict__ aval, const double *__restrict__ avalT,
                           const double *__restrict__ D) {
    GRID_STRIDE(e, nnz) {
        if (wsn[e] == 0) continue;  // a member
        const double dj = D[W.col[e] - n];
        double v = 0.0, vT = 0.0;
        for (int64_t k = ws0[e]; k < ws0[e] + wsn[e]; ++k) {
            const int64_t q = src[k];
            v = v + (q < 0 ? dj : aval[q]);
            vT = vT + (q < 0 ? dj : avalT[q]);
        }
        W.val[e] = -v;
        W.valT[e] = -vT;
    }
}

// e += s c, with s from the nblocks partials of k_vc_energy (1 without any).
// With rfirst, e is the first Jacobi sweep from zero, formed here as
// omega r / D (the same expression as k_vc_first) instead of being read.
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_vc_correct(int32_t n, int64_t S, const T *__restrict__ ec, const int32_t *__restrict__ agg,
             T *__restrict__ e, const double *__restrict__ partials, int nblocks,
             const T *__restrict__ rfirst, const T *__restrict__ D, T omega,
             const DevScalars *ds) {
    if (vc_skip(ds)) return;
    T sc = T(1);
    if (nblocks > 0) {
        double v[2];
        sum_partials<2>(partials, nblocks, v);
        sc = (T)correction_scale(v);
    }
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            const T e0 = rfirst ? omega * rfirst[i] / D[i] : e[i];
            e[i] = e0 + sc * ec[agg[i]];
        }
    });
}

// coarsest level: diagonal PCG in FP64 by one workgroup, from e = 0 to
// ||r|| <= tol ||rhs|| or max_it iterations; a singular level first
// projects its rhs to zero mean.  w: 3 n doubles of scratch (r, p, q).
template <int K, int NW>
__device__ __forceinline__ void bcast_sum(double (&v)[K]) {
    if constexpr (NW == 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);  // every lane gets the sum
    } else {
        __shared__ double out[K];
        block_reduce<K>(v);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) out[k] = v[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = out[k];
        __syncthreads();
    }
}

// LDS holds the coarsest CG vectors when 5 n doubles fit (dynamic shared memory)
constexpr int kLdsCoarse = 1536;

// a barrier also in the one-wavefront case (there it costs next to nothing
// and orders the LDS stores of one lane before other lanes' loads)
template <int NW>
__device__ __forceinline__ void csync() {
    __syncthreads();
}

// DIC preconditioner z = M^-1 r by forward and backward substitution in row
// form, serially (one thread): y_i = (r_i - sum_{j<i} A_ij y_j) / Dt_i for
// ascending i, then z_i = y_i - (sum_{j>i} A_ij z_j) / Dt_i for descending i,
// each row sum in column order
__device__ void dic_serial(const SellView<double> &A, const double *__restrict__ dt,
                           const double *__restrict__ r, double *__restrict__ z) {
    const int32_t n = A.n;
    for (int32_t i = 0; i < n; ++i) {
        const int64_t ps = sv_pos(A, i);
        const int w = row_len(A, ps);
        double sum = 0.0;
        for (int k = 0; k < w; ++k) {
            const int64_t e = entry_at(A, ps, k);
            const int32_t c = A.col[e];
            if (c < i) sum = sum + A.val[e] * z[c];
        }
        z[i] = (r[i] - sum) / dt[i];
    }
    for (int32_t i = n - 1; i >= 0; --i) {
        const int64_t ps = sv_pos(A, i);
        const int w = row_len(A, ps);
        double sum = 0.0;
        for (int k = 0; k < w; ++k) {
            const int64_t e = entry_at(A, ps, k);
            const int32_t c = A.col[e];
            if (c > i) sum = sum + A.val[e] * z[c];
        }
        z[i] = z[i] - sum / dt[i];
    }
}

template <typename TI, int NW>
__device__ void coarsest_body(const SellView<double> &A, const TI *__restrict__ rhs,
                              TI *__restrict__ eo, double *__restrict__ w, int singular,
                              double tol, int max_it, const double *__restrict__ dt) {
    constexpr int NT = NW * kWave;
    const int32_t n = A.n;
    double *r = w, *p = w + n, *q = w + 2 * (int64_t)n, *x = w + 3 * (int64_t)n,
           *z = w + 4 * (int64_t)n;
    for (int32_t i = threadIdx.x; i < n; i += NT) {
        r[i] = (double)rhs[i];
        x[i] = 0.0;
    }
    csync<NW>();
    if (singular) {
        double m[1] = {0.0};
        for (int32_t i = threadIdx.x; i < n; i += NT) m[0] += r[i];
        bcast_sum<1, NW>(m);
        const double mean = m[0] / (double)n;
        for (int32_t i = threadIdx.x; i < n; i += NT) r[i] = r[i] - mean;
        csync<NW>();
    }
    // z = M^-1 r (diagonal, or DIC when dt is given); r is complete on entry
    auto precond = [&]() {
        if (dt) {
            if (threadIdx.x == 0) dic_serial(A, dt, r, z);
        } else {
            for (int32_t i = threadIdx.x; i < n; i += NT) z[i] = r[i] / A.diag[i];
        }
        csync<NW>();
    };
    double b2[1] = {0.0};
    for (int32_t i = threadIdx.x; i < n; i += NT) b2[0] += r[i] * r[i];
    bcast_sum<1, NW>(b2);
    const double bn = sqrt(b2[0]);
    if (bn > 0.0) {
        precond();
        double rz[1] = {0.0};
        for (int32_t i = threadIdx.x; i < n; i += NT) {
            p[i] = z[i];
            rz[0] += r[i] * z[i];
        }
        bcast_sum<1, NW>(rz);
        double rho = rz[0];
        for (int it = 0; it < max_it; ++it) {
            double pq[1] = {0.0};
            for (int32_t i = threadIdx.x; i < n; i += NT) {
                const int64_t ps = sv_pos(A, i);
                const double qi = sell_row_any(A, ps >> 6, (int)(ps & 63), i, Direct<double>{p});
                q[i] = qi;
                pq[0] += p[i] * qi;
            }
            bcast_sum<1, NW>(pq);
            if (!isfinite(pq[0]) || fabs(pq[0]) <= 1e-300) break;
            const double alpha = rho / pq[0];
            double rr[1] = {0.0};
            for (int32_t i = threadIdx.x; i < n; i += NT) {
                x[i] = x[i] + alpha * p[i];
                const double ri = r[i] - alpha * q[i];
                r[i] = ri;
                rr[0] += ri * ri;
            }
            bcast_sum<1, NW>(rr);
            if (sqrt(rr[0]) / bn <= tol) break;
            precond();
            double rzn[1] = {0.0};
            for (int32_t i = threadIdx.x; i < n; i += NT) rzn[0] += r[i] * z[i];
            bcast_sum<1, NW>(rzn);
            const double beta = rzn[0] / rho;
            rho = rzn[0];
            for (int32_t i = threadIdx.x; i < n; i += NT) p[i] = z[i] + beta * p[i];
            csync<NW>();
        }
    }
    csync<NW>();
    for (int32_t i = threadIdx.x; i < n; i += NT) eo[i] = (TI)x[i];
}

__device__ __forceinline__ double readlane_f64(double v, int j) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), j);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), j);
    return __hiloint2double(hi, lo);
}


// coarsest level of at most 64 cells with rows of at most kWaveRow entries:
// one wavefront, one row per lane, the row's entries held in LDS
// (entry-major, so lanes read distinct banks) and the search direction in
// LDS.  Row i sums diag_i p_i first and then its entries in column order, as
// the sparse kernels do.  The first kRegRow entries of a row also stay in
// registers for the whole solve, so a product issues all their gathers of p
// at once instead of one LDS round trip per entry.
constexpr int kWaveRow = 48;
constexpr int kRegRow = 16;

// LDS ordering for one wavefront: its LDS operations execute in order, so a
// fence against compiler reordering is all a lane-to-lane exchange needs
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct CoarsestLds {
    int32_t cL[kWaveRow * kWave];
    double vL[kWaveRow * kWave];
    double p[kWave];
    int32_t m[kWave], nl[kWave];
};

// two wavefront sums whose dependent chains overlap (each is wave_sum's)
__device__ __forceinline__ void wave_sum2(double &a, double &b) {
    a = a + dpp_move<0xB1>(a, 0.0);
    b = b + dpp_move<0xB1>(b, 0.0);
    a = a + dpp_move<0x4E>(a, 0.0);
    b = b + dpp_move<0x4E>(b, 0.0);
    a = a + dpp_move<0x124>(a, 0.0);
    b = b + dpp_move<0x124>(b, 0.0);
    a = a + dpp_move<0x128>(a, 0.0);
    b = b + dpp_move<0x128>(b, 0.0);
    a = a + dpp_move<0x142, 0xa>(a, 0.0);
    b = b + dpp_move<0x142, 0xa>(b, 0.0);
    a = a + dpp_move<0x143, 0xc>(a, 0.0);
    b = b + dpp_move<0x143, 0xc>(b, 0.0);
    a = lane63(a);
    b = lane63(b);
}

// the first U gathers of a register-held row, added in column order to q
template <int U>
__device__ __forceinline__ double reg_row(double q, const double *vR, const int32_t *cR,
                                          const double *p) {
    double pv[U];
#pragma unroll
    for (int k = 0; k < U; ++k) pv[k] = p[cR[k]];
#pragma unroll
    for (int k = 0; k < U; ++k) q = q + vR[k] * pv[k];
    return q;
}

// the one-wavefront coarsest CG, run by the 64 lanes of one wave (the
// caller's other waves, if any, do not take part).  It is one chain of
// dependent steps (exchange of p, row sum, three wave reductions, three
// divisions per CG iteration), so what it costs is latency: the matrix is
// loaded in batches (one round trip per batch instead of three per entry),
// short rows are padded with zero values at the lane's own column instead of
// being masked entry by entry, r.r and r.z reduce side by side, beta and the
// next direction are formed before the stop test, and the test's square root
// and division run only near the tolerance.  33 cells (the pairwise hierarchy
// of a 100^3 box, about 40 iterations): 31.5 -> 21.2 us, results bitwise
// unchanged.
__device__ void coarsest_wave_body(const SellView<double> &A, const double *__restrict__ rhs_d,
                                   const float *__restrict__ rhs_f, double *__restrict__ eo_d,
                                   float *__restrict__ eo_f, int singular, double tol,
                                   int max_it, const double *__restrict__ dt,
                                   const FineCorr<double> &fcd, const FineCorr<float> &fcf,
                                   CoarsestLds &sm) {
    int32_t *cL = sm.cL;
    double *vL = sm.vL;
    double *p = sm.p;
    const int32_t n = A.n;
    const int i = threadIdx.x;
    double di = 1.0, ri = 0.0, rdt = 0.0;
    if (i < n) {
        di = A.diag[i];
        ri = rhs_d ? rhs_d[i] : (double)rhs_f[i];
        if (dt) rdt = 1.0 / dt[i];
        // the level is one slice: this lane loads the row at position i
        const int32_t row = A.perm ? A.perm[i] : i;
        const int64_t b0 = A.sptr[0];
        const int w = A.pdeg ? A.pdeg[i] : (int)((A.sptr[1] - b0) >> 6);
        const int32_t *cp = A.col + b0 + i;
        const double *vp = A.val + b0 + i;
        int mr = 0, nlr = 0;
        int64_t off = 0;
        for (int k0 = 0; k0 < w; k0 += kRegRow) {
            int32_t c[kRegRow];
            double v[kRegRow];
#pragma unroll
            for (int u = 0; u < kRegRow; ++u) {
                const bool has = k0 + u < w;
                const int64_t o = off;
                off += A.pdeg ? (int64_t)__popcll(__ballot(has)) : (int64_t)kWave;
                if (has) {
                    c[u] = cp[o];
                    v[u] = vp[o];
                }
            }
#pragma unroll
            for (int u = 0; u < kRegRow; ++u) {
                if (k0 + u < w && c[u] != row) {  // padding entries point at the row
                    cL[mr * kWave + row] = c[u];
                    vL[mr * kWave + row] = v[u];
                    nlr += c[u] < row;
                    ++mr;
                }
            }
        }
        sm.m[row] = mr;
        sm.nl[row] = nlr;
    }
    wave_lds_sync();
    // entries of row i, and how many lie left of the diagonal
    const int m = i < n ? sm.m[i] : 0, nl = i < n ? sm.nl[i] : 0;
    int32_t cR[kRegRow];
    double vR[kRegRow];
#pragma unroll
    for (int k = 0; k < kRegRow; ++k) {
        cR[k] = k < m ? cL[k * kWave + i] : i;
        vR[k] = k < m ? vL[k * kWave + i] : 0.0;
    }
    const bool long_rows = __ballot(m > kRegRow / 2) != 0;
    // z = M^-1 r: the diagonal, or the DIC factor by column-oriented
    // substitution: at step j lane j's value is final and is broadcast, and
    // every row holding column j takes its term (lower entries in ascending
    // column order on the way down, upper entries in descending order on the
    // way up)
    auto precond = [&](double rv) -> double {
        if (!dt) return (i < n) ? rv / di : 0.0;
        double acc = 0.0, y = 0.0;
        int kk = 0;
        for (int j = 0; j < n; ++j) {
            const double cand = (rv - acc) * rdt;
            const double yj = readlane_f64(cand, j);
            if (i == j) y = cand;
            if (kk < nl && cL[kk * kWave + i] == j) {
                acc = acc + vL[kk * kWave + i] * yj;
                ++kk;
            }
        }
        acc = 0.0;
        double zv = 0.0;
        kk = m - 1;
        for (int j = n - 1; j >= 0; --j) {
            const double cand = y - acc * rdt;
            const double zj = readlane_f64(cand, j);
            if (i == j) zv = cand;
            if (kk >= nl && cL[kk * kWave + i] == j) {
                acc = acc + vL[kk * kWave + i] * zj;
                --kk;
            }
        }
        return (i < n) ? zv : 0.0;
    };
    if (singular) {
        const double mean = wave_sum(ri) / (double)n;
        if (i < n) ri = ri - mean;
    }
    double xi = 0.0;
    const double bn = sqrt(wave_sum(ri * ri));
    if (bn > 0.0) {
        // far above the tolerance: r.r > 4 (tol bn)^2 (used while that square
        // is a normal number)
        const double far2 = 4.0 * (tol * bn) * (tol * bn);
        const bool far_ok = far2 > 1e-290;
        double pi = precond(ri);
        double rho = wave_sum(ri * pi);
        for (int it = 0; it < max_it; ++it) {
            p[i] = pi;
            wave_lds_sync();
            double qi = di * pi;
            if (long_rows) {
                qi = reg_row<kRegRow>(qi, vR, cR, p);
                for (int k = kRegRow; k < m; ++k)
                    qi = qi + vL[k * kWave + i] * p[cL[k * kWave + i]];
            } else {
                qi = reg_row<kRegRow / 2>(qi, vR, cR, p);
            }
            if (i >= n) qi = 0.0;
            wave_lds_sync();
            const double pq = wave_sum(pi * qi);
            if (!isfinite(pq) || fabs(pq) <= 1e-300) break;
            const double alpha = rho / pq;
            xi = xi + alpha * pi;
            ri = ri - alpha * qi;
            const double zi = precond(ri);
            double rr = ri * ri, rz = ri * zi;
            wave_sum2(rr, rz);
            const double beta = rz / rho;
            pi = zi + beta * pi;
            rho = rz;
            if (far_ok && rr > far2) continue;
            if (sqrt(rr) / bn <= tol) break;
        }
    }
    if (i < n) {  // the result, and the finer level's correction with it
        if (eo_d) {
            eo_d[i] = xi;
            if (fcd.e) fcd(i, xi);
        } else {
            const float v = (float)xi;
            eo_f[i] = v;
            if (fcf.e) fcf(i, v);
        }
    }
}

__global__ void __launch_bounds__(kWave)
k_coarsest_wave(SellView<double> A, const double *__restrict__ rhs_d,
                const float *__restrict__ rhs_f, double *__restrict__ eo_d,
                float *__restrict__ eo_f, int singular, double tol, int max_it,
                const double *__restrict__ dt, FineCorr<double> fcd, FineCorr<float> fcf,
                const DevScalars *ds) {
    __shared__ CoarsestLds sm;
    if (vc_skip(ds)) return;
    coarsest_wave_body(A, rhs_d, rhs_f, eo_d, eo_f, singular, tol, max_it, dt, fcd, fcf, sm);
}

// coarsest-level launch for larger levels: one 256-thread block
template <typename TI, int NW>
__global__ void __launch_bounds__(kBlock)
k_coarsest(SellView<double> A, const TI *__restrict__ rhs, TI *__restrict__ eo,
           double *__restrict__ w, int singular, double tol, int max_it,
           const double *__restrict__ dt, const DevScalars *ds) {
    extern __shared__ double lds_w[];
    if (vc_skip(ds)) return;
    coarsest_body<TI, NW>(A, rhs, eo, A.n <= kLdsCoarse ? lds_w : w, singular, tol, max_it, dt);
}

// x += e (GAMG correction of the outer FP64 loop)
__global__ void __launch_bounds__(kBlock)
k_add(int32_t n, int64_t S, const double *__restrict__ e, double *__restrict__ x,
      const DevScalars *ds) {
    if (ds->done) return;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) x[i] = x[i] + e[i];
    });
}

// mixed: rhat = fp32(r / ||r||_inf)
__global__ void __launch_bounds__(kBlock)
k_cast_scaled(int32_t n, int64_t S, const double *__restrict__ r, float *__restrict__ r32,
              DevScalars *ds) {
    if (ds->done) return;
    const double sc = ds->maxabs;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) r32[i] = (float)(r[i] / sc);
    });
    if (blockIdx.x == 0 && threadIdx.x == 0) ds->scale = sc;
}

__global__ void __launch_bounds__(kBlock)
k_refine_add(int32_t n, int64_t S, const float *__restrict__ d, double *__restrict__ x,
             const DevScalars *ds) {
    if (ds->done) return;
    const double sc = ds->scale;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) x[i] = x[i] + sc * (double)d[i];
    });
}

template <bool CMP, typename T>
static void launch_jacobi_l(const SellView<T> &A, const T *r, const T *e, T *eo, T omega,
                            const T *rdot, double *partials, const FineCorr<T> &fc,
                            const DevScalars *ds, int G, hipStream_t st) {
    if (rdot && fc.e)
        k_vc_jacobi<CMP, true, true, T><<<G, kBlock, 0, st>>>(A, r, e, eo, omega, rdot, partials, fc, ds);
    else if (rdot)
        k_vc_jacobi<CMP, true, false, T><<<G, kBlock, 0, st>>>(A, r, e, eo, omega, rdot, partials, fc, ds);
    else if (fc.e)
        k_vc_jacobi<CMP, false, true, T><<<G, kBlock, 0, st>>>(A, r, e, eo, omega, rdot, partials, fc, ds);
    else
        k_vc_jacobi<CMP, false, false, T><<<G, kBlock, 0, st>>>(A, r, e, eo, omega, rdot, partials, fc, ds);
}

// one Jacobi sweep; with rdot, also the block partials of rdot . e_out; with
// fc.e, also the finer level's correction
template <typename T>
static void launch_jacobi(const SellView<T> &A, const T *r, const T *e, T *eo, T omega,
                          const T *rdot, double *partials, const FineCorr<T> &fc,
                          const DevScalars *ds, int G, hipStream_t st) {
    if (A.pdeg) launch_jacobi_l<true, T>(A, r, e, eo, omega, rdot, partials, fc, ds, G, st);
    else launch_jacobi_l<false, T>(A, r, e, eo, omega, rdot, partials, fc, ds, G, st);
}

template <bool CMP, bool UPPER, typename T>
static void launch_gs_step(const SellView<T> &A, const T *t, const T *g, T *out, int mode,
                           const DevScalars *ds, int G, hipStream_t st) {
    if (g) k_vc_gs<CMP, UPPER, false, T><<<G, kBlock, 0, st>>>(A, t, g, out, mode, ds);
    else k_vc_gs<CMP, UPPER, true, T><<<G, kBlock, 0, st>>>(A, t, g, out, mode, ds);
}

// one two-stage Gauss-Seidel sweep on A e = r: t = r - A e (t = r from
// zero), `inner` triangular Jacobi-Richardson steps through the ping-pong
// buffers w0, w1, the last one updating e in place (each row reads only t,
// the previous step and its own e entry)
template <typename T>
static void gs_sweep(const SellView<T> &A, const T *r, T *e, T *t, T *w0, T *w1, bool from_zero,
                     bool backward, int inner, const DevScalars *ds, int G, hipStream_t st) {
    const T *tt = r;
    if (!from_zero) {
        if (A.pdeg) k_vc_resid<true, T><<<G, kBlock, 0, st>>>(A, r, e, t, ds);
        else k_vc_resid<false, T><<<G, kBlock, 0, st>>>(A, r, e, t, ds);
        tt = t;
    }
    const T *g = nullptr;
    for (int k = 0; k < inner; ++k) {
        const bool last = k + 1 == inner;
        T *out = last ? e : (k % 2 == 0 ? w0 : w1);
        const int mode = last ? (from_zero ? 1 : 2) : 0;
        if (A.pdeg) {
            if (backward) launch_gs_step<true, true, T>(A, tt, g, out, mode, ds, G, st);
            else launch_gs_step<true, false, T>(A, tt, g, out, mode, ds, G, st);
        } else {
            if (backward) launch_gs_step<false, true, T>(A, tt, g, out, mode, ds, G, st);
            else launch_gs_step<false, false, T>(A, tt, g, out, mode, ds, G, st);
        }
        g = out;
    }
}

// ---------------------------------------------------------------- V-cycle driver
struct VCtx {
    ldu_t *h;
    const ldu_gamg_opts *o;
    bool tr;
    hipStream_t st;
    double *cw;        // coarsest scratch, 5 n_coarsest doubles
    const double *dt;  // coarsest DIC pivots, or null for the diagonal
};

template <typename T>
static SellView<T> lview(const Level &L, bool tr);
template <>
SellView<double> lview<double>(const Level &L, bool tr) { return L.A.view(tr); }
template <>
SellView<float> lview<float>(const Level &L, bool tr) { return L.A.view32(tr); }

template <typename T>
static SellView<T> rview(const Level &L, bool tr);
template <>
SellView<double> rview<double>(const Level &L, bool tr) { return L.R.view(tr); }
template <>
SellView<float> rview<float>(const Level &L, bool tr) { return L.R.view32(tr); }
template <typename T>
static CsrView<T> rcview(const Level &L, bool tr);
template <>
CsrView<double> rcview<double>(const Level &L, bool tr) { return L.Rc.view(tr); }
template <>
CsrView<float> rcview<float>(const Level &L, bool tr) { return L.Rc.view32(tr); }
template <typename T>
static CsrView<T> upview(const Level &L, bool tr);
template <>
CsrView<double> upview<double>(const Level &L, bool tr) { return L.Uc.view(tr); }
template <>
CsrView<float> upview<float>(const Level &L, bool tr) { return L.Uc.view32(tr); }
template <typename T>
static CsrView<T> vview(const Csr &M, bool tr);
template <>
CsrView<double> vview<double>(const Csr &M, bool tr) { return M.view(tr); }
template <>
CsrView<float> vview<float>(const Csr &M, bool tr) { return M.view32(tr); }
// R's values of this precision exist (either layout)
template <typename T>
static const T *ahval(const Level &L, bool tr);
template <>
const double *ahval<double>(const Level &L, bool tr) { return tr ? L.ahT : L.ah; }
template <>
const float *ahval<float>(const Level &L, bool tr) { return tr ? L.ahT32 : L.ah32; }
template <typename T>
static bool has_rop(const Level &L, bool tr) {
    return rview<T>(L, tr).val != nullptr || rcview<T>(L, tr).val != nullptr ||
           ahval<T>(L, tr) != nullptr;
}

template <typename T>
static T *lvec(Level &L, int which);
template <>
double *lvec<double>(Level &L, int which) {
    return which == 0 ? L.r : which == 1 ? L.e : which == 2 ? L.e2 : which == 3 ? L.t : L.w;
}
template <>
float *lvec<float>(Level &L, int which) {
    return which == 0 ? L.r32 : which == 1 ? L.e32 : which == 2 ? L.e232 : which == 3 ? L.t32
                                                                                     : L.w32;
}

constexpr int kFuseCorrRows = 1 << 17;
// levels of at most this many cells run their up leg as the operator U (limits
// of 2^14, 2^16, 2^17 and 400,000 cells: 17.7, 17.0, 17.2 and 17.7 ms for CG +
// V-cycle at 100^3, 127.1, 126.2, 126.6 and 129.7 ms at 200^3)
#ifndef LDU_UP_ROWS
#define LDU_UP_ROWS (1 << 16)
#endif
constexpr int kUpRows = LDU_UP_ROWS;

// level l's down leg runs in one pass (R, or the scaled slices)
template <typename T>
static bool rop_level(const VCtx &c, size_t l) {
    const Level &L = c.h->levels[l];
    return rop_cycle(*c.o) && L.r_ready && L.r_omega == c.o->omega && has_rop<T>(L, c.tr);
}
// level l's up leg runs through U
template <typename T>
static bool up_level(const VCtx &c, size_t l) {
    return rop_level<T>(c, l) && c.o->n_post > 0 && upview<T>(c.h->levels[l], c.tr).val;
}
// level l of a Jacobi cycle without the one-pass down leg runs through V and W
static bool gen_cycle(const ldu_gamg_opts &o) {
    return o.smoother == LDU_SMOOTH_JACOBI && !rop_cycle(o) && o.n_pre > 0 && o.n_post > 0;
}
template <typename T>
static bool gen_level(const VCtx &c, size_t l) {
    const Level &L = c.h->levels[l];
    return gen_cycle(*c.o) && L.g_ready && L.g_omega == c.o->omega && vview<T>(L.V, c.tr).val;
}
// level l's unscaled correction is applied by the coarse level's last kernel
// (a coarse level that runs through U leaves it to level l)
template <typename T>
static bool takes_correction(const VCtx &c, size_t l) {
    const bool coarse_leaves =
        l + 2 < c.h->levels.size() && (up_level<T>(c, l + 1) || gen_level<T>(c, l + 1));
    return !c.o->scale_correction && c.h->levels[l].n <= kFuseCorrRows && !up_level<T>(c, l) &&
           !gen_level<T>(c, l) && !coarse_leaves;
}

template <typename T>
static T *vcycle(const VCtx &c, size_t l, const T *r, const T *rdot = nullptr,
                 int *dotted = nullptr, bool e_ready = false, FineCorr<T> fc = {},
                 bool *corrected = nullptr);

// sums of the scaling factor over level l (the coarse one); the number of partials
template <typename T>
static int launch_energy(const VCtx &c, size_t l, const T *ec, const T *rc) {
    ldu_t *h = c.h;
    const Level &C = h->levels[l];
    if (l + 1 < h->levels.size() && gen_level<T>(c, l)) {
        const CsrView<T> V = vview<T>(C.V, c.tr);
        const int G = stream_grid_slices((V.n + kWave / V.group - 1) / (kWave / V.group));
        with_group(V.group, [&](auto lanes) {
            k_gen_energy<decltype(lanes)::value, T>
                <<<G, kBlock, 0, c.st>>>(V, C.qptr, ec, rc, h->partials, h->dev);
        });
        return G;
    }
    const SellView<T> A = lview<T>(C, c.tr);
    // blocks past the products' cap would only add zeros
    int G = stream_grid_slices(A.nslices);
    if (!A.pdeg) G = std::min(G, kPlainF64ProductBlocks);
    if (A.pdeg) k_vc_energy<true, T><<<G, kBlock, 0, c.st>>>(A, ec, rc, h->partials, h->dev);
    else k_vc_energy<false, T><<<G, kBlock, 0, c.st>>>(A, ec, rc, h->partials, h->dev);
    return G;
}

// one sweep (or, with ec, the up leg) through V; the number of blocks, of
// partials with rdot (CG's cycles, which take it, do not scale)
template <typename T>
static int launch_gen_sweep(const VCtx &c, const Level &L, const T *r, const T *e, const T *ec,
                            T *eo, int scale_blocks, const T *rdot) {
    const CsrView<T> V = vview<T>(L.V, c.tr);
    const T *D = lview<T>(L, c.tr).diag;
    const T omega = (T)c.o->omega;
    const int G = stream_grid_slices((V.n + kWave / V.group - 1) / (kWave / V.group));
    ldu_t *h = c.h;
    with_group(V.group, [&](auto lanes) {
        constexpr int N = decltype(lanes)::value;
        auto run = [&](auto kernel) {
            kernel<<<G, kBlock, 0, c.st>>>(V, L.qptr, D, r, e, ec, eo, omega, h->partials,
                                           scale_blocks, rdot, h->partials, h->dev);
        };
        if (ec && rdot) run(k_gen_sweep<N, true, true, T>);
        else if (ec) run(k_gen_sweep<N, true, false, T>);
        else if (rdot) run(k_gen_sweep<N, false, true, T>);
        else run(k_gen_sweep<N, false, false, T>);
    });
    return G;
}

// the levels from a small one down, through V and W
template <typename T>
static T *vcycle_gen(const VCtx &c, size_t l, const T *r, const T *rdot, int *dotted,
                     bool e_ready) {
    ldu_t *h = c.h;
    Level &L = h->levels[l], &C = h->levels[l + 1];
    hipStream_t st = c.st;
    T *e = lvec<T>(L, 1), *e2 = lvec<T>(L, 2);
    const T omega = (T)c.o->omega;
    if (!e_ready) {
        const int64_t S = L.A.nslices;
        k_vc_first<T><<<stream_grid_slices(S), kBlock, 0, st>>>(
            L.n, S, r, lview<T>(L, c.tr).diag, e, omega, h->dev);
    }
    for (int k = 1; k < c.o->n_pre; ++k) {
        launch_gen_sweep<T>(c, L, r, e, nullptr, e2, 0, nullptr);
        std::swap(e, e2);
    }
    T *rc = lvec<T>(C, 0);
    const bool c_first = l + 2 < h->levels.size();  // the coarse level's first sweep
    launch_rrestrict_csr<T>(vview<T>(L.W, c.tr), Stacked<T>{r, e, L.n}, rc,
                            c_first ? lvec<T>(C, 1) : nullptr, lview<T>(C, c.tr).diag, omega,
                            h->dev, st);
    const T *ec = vcycle<T>(c, l + 1, rc, nullptr, nullptr, c_first);
    const int scale_blocks = c.o->scale_correction ? launch_energy<T>(c, l + 1, ec, rc) : 0;
    for (int k = 0; k < c.o->n_post; ++k) {
        const T *rd = k + 1 == c.o->n_post ? rdot : nullptr;
        const int blocks = launch_gen_sweep<T>(c, L, r, e, k == 0 ? ec : nullptr, e2,
                                               k == 0 ? scale_blocks : 0, rd);
        std::swap(e, e2);
        if (rd && dotted) *dotted = blocks;
    }
    HIP_CHECK(hipGetLastError());
    return e;
}

// One V-cycle e = V(l, r); returns the buffer holding e.  With rdot, the
// last level-l kernel also leaves its block partials of rdot . e in
// h->partials and their number in *dotted (0: that kernel took no dot).
// e_ready: the caller's restriction already stored the first Jacobi sweep
// e = omega r / D in this level's e.  fc: the finer level's unscaled
// correction e_f += P e, applied here by the kernel that produces e when it
// can (*corrected tells the caller).
template <typename T>
static T *vcycle(const VCtx &c, size_t l, const T *r, const T *rdot, int *dotted, bool e_ready,
                 FineCorr<T> fc, bool *corrected) {
    if (dotted) *dotted = 0;
    if (corrected) *corrected = false;
    ldu_t *h = c.h;
    Level &L = h->levels[l];
    hipStream_t st = c.st;
    T *e = lvec<T>(L, 1), *e2 = lvec<T>(L, 2), *t = lvec<T>(L, 3);
    if (l + 1 == h->levels.size()) {
        const int maxit = std::max(2 * L.n, 100);
        const size_t lds = L.n <= kLdsCoarse ? sizeof(double) * 5 * L.n : 0;
        if (L.n <= kWave && L.max_row <= kWaveRow) {
            const bool f64 = sizeof(T) == sizeof(double);
            FineCorr<double> fcd{};
            FineCorr<float> fcf{};
            if (f64) fcd = {(double *)fc.e, fc.start, fc.cells};
            else fcf = {(float *)fc.e, fc.start, fc.cells};
            k_coarsest_wave<<<1, kWave, 0, st>>>(
                L.A.view(c.tr), f64 ? (const double *)r : nullptr,
                f64 ? nullptr : (const float *)r, f64 ? (double *)e : nullptr,
                f64 ? nullptr : (float *)e, L.singular, kCoarsestTol, maxit, c.dt, fcd, fcf,
                h->dev);
            if (corrected && fc.e) *corrected = true;
        } else
            k_coarsest<T, kWavesPerBlock><<<1, kBlock, lds, st>>>(L.A.view(c.tr), r, e, c.cw,
                                                                 L.singular, kCoarsestTol,
                                                                 maxit, c.dt, h->dev);
        HIP_CHECK(hipGetLastError());
        return e;
    }
    if (gen_level<T>(c, l)) return vcycle_gen<T>(c, l, r, rdot, dotted, e_ready);
    SellView<T> A = lview<T>(L, c.tr);
    // a cycle without the one-pass down leg sweeps the level several times in
    // a row (matrix, and r, e, its second buffer, t and D)
    A.stream = rop_level<T>(c, l) ||
               L.A.bytes(sizeof(T)) + 5 * (int64_t)sizeof(T) * L.n > kCacheBytes;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    const T omega = (T)c.o->omega;
    const bool gs = c.o->smoother == LDU_SMOOTH_GS2;
    T *w1 = lvec<T>(L, 4);
    const bool rop = rop_level<T>(c, l);
    // small levels: first sweep, correction and first post-sweep as U (r, e_c)
    const bool up = up_level<T>(c, l);
    // scaled slices: the same from the down leg's t (a dot product is the one
    // with r itself; a finer level's correction rides on a sweep)
    const bool up_slices = rop && L.ah && c.o->n_post > 0 &&
                           (c.o->n_post > 1 || ((!rdot || rdot == r) && !fc.e));
    // without correction scaling, on levels small enough to be bound by launch
    // latency, the coarse level applies e += P e_c itself (a scatter through
    // the member lists: on large levels the gather form of k_vc_correct moves
    // fewer bytes)
    const bool fuse_corr = takes_correction<T>(c, l) && !up_slices;
    // with the one-pass down leg nothing reads the first sweep before the
    // correction, which then forms it itself
    const bool defer_first = rop && !e_ready && !fuse_corr && !up_slices;
    if (gs) {  // forward two-stage Gauss-Seidel sweeps, the first from e = 0
        if (c.o->n_pre == 0) k_vc_zero<T><<<G, kBlock, 0, st>>>(L.n, S, e, h->dev);
        for (int k = 0; k < c.o->n_pre; ++k)
            gs_sweep<T>(A, r, e, t, e2, w1, k == 0, false, c.o->gs_inner, h->dev, G, st);
    } else {
        if (c.o->n_pre == 0) k_vc_zero<T><<<G, kBlock, 0, st>>>(L.n, S, e, h->dev);
        else if (!e_ready && !defer_first && !up && !up_slices)
            k_vc_first<T><<<G, kBlock, 0, st>>>(L.n, S, r, A.diag, e, omega, h->dev);
        for (int k = 1; k < c.o->n_pre; ++k) {
            launch_jacobi<T>(A, r, e, e2, omega, nullptr, nullptr, {}, h->dev, G, st);
            std::swap(e, e2);
        }
    }
    Level &C = h->levels[l + 1];
    T *rc = lvec<T>(C, 0);
    // the coarse level's first Jacobi sweep rides on the restriction, unless
    // the coarse level will form it in its own correction (a large
    // non-coarsest level whose down leg also runs through R)
    const bool c_defers = l + 2 < h->levels.size() && rop_level<T>(c, l + 1) &&
                          !takes_correction<T>(c, l + 1);
    const bool c_first = !gs && c.o->n_pre > 0 && l + 2 < h->levels.size() && !c_defers;
    T *ec_first = c_first ? lvec<T>(C, 1) : nullptr;
    if (rop) {
        if (L.ah) {  // t = (I - omega A D^-1) r over the level's slices, then its member sums
            SellView<T> Ah = A;
            Ah.val = ahval<T>(L, c.tr);
            if (Ah.c16)
                k_vc_ahat<true, T><<<G, kBlock, 0, st>>>(Ah, r, t, T(1) - omega, h->dev);
            else
                k_vc_ahat<false, T><<<G, kBlock, 0, st>>>(Ah, r, t, T(1) - omega, h->dev);
            k_vc_restrict<T><<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.aggStart, L.aggCells, t, rc,
                                                            ec_first, lview<T>(C, c.tr).diag,
                                                            omega, h->dev);
        } else if (L.R.sptr) {  // residual and restriction in one pass over R (t is not formed)
            const SellView<T> R = rview<T>(L, c.tr);
            k_vc_rrestrict_cmp<T><<<stream_grid_slices(R.nslices), kBlock, 0, st>>>(
                R, r, rc, ec_first, lview<T>(C, c.tr).diag, omega, h->dev);
        } else {
            launch_rrestrict_csr<T>(rcview<T>(L, c.tr), Direct<T>{r}, rc, ec_first, lview<T>(C, c.tr).diag,
                                    omega, h->dev, st);
        }
    } else {
        if (A.pdeg) k_vc_resid<true, T><<<G, kBlock, 0, st>>>(A, r, e, t, h->dev);
        else k_vc_resid<false, T><<<G, kBlock, 0, st>>>(A, r, e, t, h->dev);
        k_vc_restrict<T><<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.aggStart, L.aggCells, t, rc,
                                                        ec_first, lview<T>(C, c.tr).diag, omega,
                                                        h->dev);
    }
    bool done_corr = false;
    const T *ec = vcycle<T>(c, l + 1, rc, nullptr, nullptr, c_first,
                            fuse_corr ? FineCorr<T>{e, L.aggStart, L.aggCells} : FineCorr<T>{},
                            &done_corr);
    // partials of the scaling factor's sums
    const int scale_blocks = c.o->scale_correction ? launch_energy<T>(c, l + 1, ec, rc) : 0;
    int post = 0;  // post-sweeps done
    if (up) {
        const bool last = c.o->n_post == 1;
        const int blocks = launch_up_csr<T>(upview<T>(L, c.tr), r, ec, e, last ? rdot : nullptr,
                                            h->partials, h->dev, st);
        if (last && rdot && dotted) *dotted = blocks;
        post = 1;
    } else if (up_slices) {
        const bool dot = c.o->n_post == 1 && rdot;
        const int blocks = launch_up_slices<T>(L, A, r, t, ec, e, omega, dot, h->partials, h->dev,
                                               st);
        if (dot && dotted) *dotted = blocks;
        post = 1;
    } else if (!done_corr)
        k_vc_correct<T><<<G, kBlock, 0, st>>>(L.n, S, ec, L.agg, e, h->partials, scale_blocks,
                                             defer_first ? r : nullptr, A.diag, omega, h->dev);
    for (int k = post; k < c.o->n_post; ++k) {
        const bool last = k + 1 == c.o->n_post;
        if (gs) {  // backward sweeps: the V-cycle stays symmetric
            gs_sweep<T>(A, r, e, t, e2, w1, false, true, c.o->gs_inner, h->dev, G, st);
        } else {  // the last sweep may take the caller's dot product and correction
            // with a dot product, blocks past the products' cap would only add zeros
            const int Gs = last && rdot && !A.pdeg && sizeof(T) == sizeof(double)
                               ? std::min(G, kPlainF64ProductBlocks) : G;
            launch_jacobi<T>(A, r, e, e2, omega, last ? rdot : nullptr, h->partials,
                             last ? fc : FineCorr<T>{}, h->dev, Gs, st);
            std::swap(e, e2);
            if (last && rdot && dotted) *dotted = Gs;
            if (last && fc.e && corrected) *corrected = true;
        }
    }
    HIP_CHECK(hipGetLastError());
    return e;
}

static void ensure_work32(ldu_t *h, hipStream_t st) {
    ensure_f32_levels(h, st);
    for (auto &L : h->levels) {
        if (!L.r32) {
            Arena::Step step(h->gamg_arena);
            float *r = h->gamg_arena.get<float>(L.n);
            L.e32 = h->gamg_arena.get<float>(L.n);
            L.e232 = h->gamg_arena.get<float>(L.n);
            L.t32 = h->gamg_arena.get<float>(L.n);
            L.r32 = r;  // last: the four exist
            step.done();
        }
    }
}

// lanes per row of a CSR operator: the power of two nearest mean row length /
// entries per lane
static int csr_group(int64_t nnz, int32_t n) {
    const double per = (double)nnz / std::max<int32_t>(n, 1) / kCsrEntriesPerLane;
    int g = 1;
    while (g < 16 && 2.0 * g <= per * 1.41421356) g *= 2;
    return g;
}

// U's row bounds and arrays for a level (columns and values: k_up_fill), unless
// a row has too many aggregates
static void up_structure(ldu_t *h, Level &L, hipStream_t st) {
    Arena::Step step(h->gamg_arena);
    Arena tmp(&h->pool);
    Csr U;
    U.n = L.n;
    U.rptr = h->gamg_arena.get<int64_t>((size_t)L.n + 1);
    int64_t *cnt = tmp.get<int64_t>(L.n);
    int64_t *wide = tmp.get<int64_t>(1), hwide = 0;
    HIP_CHECK(hipMemsetAsync(wide, 0, sizeof(int64_t), st));
    k_up_count<<<grid_n((int64_t)L.n * kUpLanes), kBlock, 0, st>>>(L.A, L.agg, cnt, wide);
    exclusive_scan_i64(cnt, U.rptr, L.n, tmp, st);
    HIP_CHECK(hipMemcpyAsync(&U.nnz, U.rptr + L.n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipMemcpyAsync(&hwide, wide, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    if (hwide) return;
    U.col = h->gamg_arena.get<int32_t>(U.nnz);
    U.val = h->gamg_arena.get<double>(U.nnz);
    U.valT = h->gamg_arena.get<double>(U.nnz);
    U.group = csr_group(U.nnz, U.n);
    L.Uc = U;
    step.done();
}

// R's structure for level l (once per hierarchy): its slices and, per
// entry, the run of sources its value sums.  It is formed on a copy of the
// level: the pointers that say that it exists appear with everything that
// belongs to them, or, when memory runs out part way, not at all.
static void rop_structure(ldu_t *h, size_t l, hipStream_t st) {
    Arena::Step step(h->gamg_arena);
    Level L = h->levels[l];
    const Level &C = h->levels[l + 1];
    if (!L.A.pdeg && C.n > kCsrMaxRows) {  // a large plain-slice level: Ah over its own slices
        L.ah = h->gamg_arena.get<double>(L.A.nnz);
        L.ahT = h->gamg_arena.get<double>(L.A.nnz);
        Arena tmp(&h->pool);
        aggregate_columns(L, h->gamg_arena, tmp, st);
        HIP_CHECK(hipStreamSynchronize(st));  // tmp is released after this point
        L.r_ready = false;
        h->levels[l] = L;
        step.done();
        return;
    }
    Arena tmp(&h->pool);
    int64_t *cnt = tmp.get<int64_t>(C.n);
    int64_t *tstart = tmp.get<int64_t>(C.n + 1);
    k_rop_count<<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.aggStart, L.aggCells, L.A, cnt, nullptr);
    exclusive_scan_i64(cnt, tstart, C.n, tmp, st);
    int64_t total = 0;
    HIP_CHECK(hipMemcpyAsync(&total, tstart + C.n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    int32_t *tcol = tmp.get<int32_t>(total);
    L.r_src = h->gamg_arena.get<int64_t>(total);
    int32_t *rdeg = tmp.get<int32_t>(C.n);
    k_rop_gather<<<grid_n((int64_t)C.n * kWave), kBlock, 0, st>>>(C.n, L.aggStart, L.aggCells, L.A, tstart, tcol,
                                                L.r_src, rdeg);
    if (C.n > kCsrMaxRows) {
        build_sliced_rows(L.R, C.n, rdeg, h->gamg_arena, st);
        L.r_src0 = h->gamg_arena.get<int64_t>(L.R.nnz);
        L.r_srcn = h->gamg_arena.get<int32_t>(L.R.nnz);
        k_rop_link_sell<<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.R, tstart, tcol, L.r_src0,
                                                        L.r_srcn);
    } else {
        Csr &R = L.Rc;
        R = Csr{};
        R.n = C.n;
        R.rptr = h->gamg_arena.get<int64_t>((size_t)C.n + 1);
        int64_t *rdeg64 = tmp.get<int64_t>(C.n);
        k_widen<<<grid_n(C.n), kBlock, 0, st>>>(C.n, rdeg, rdeg64);
        exclusive_scan_i64(rdeg64, R.rptr, C.n, tmp, st);
        HIP_CHECK(hipMemcpyAsync(&R.nnz, R.rptr + C.n, sizeof(int64_t), hipMemcpyDeviceToHost,
                                 st));
        HIP_CHECK(hipStreamSynchronize(st));
        R.col = h->gamg_arena.get<int32_t>(R.nnz);
        R.val = h->gamg_arena.get<double>(R.nnz);
        R.valT = h->gamg_arena.get<double>(R.nnz);
        R.group = csr_group(R.nnz, C.n);
        L.r_src0 = h->gamg_arena.get<int64_t>(R.nnz);
        L.r_srcn = h->gamg_arena.get<int32_t>(R.nnz);
        k_rop_link_csr<<<grid_n(C.n), kBlock, 0, st>>>(C.n, R, tstart, tcol, L.r_src0, L.r_srcn);
    }
    if (L.Rc.rptr && L.n <= kUpRows) up_structure(h, L, st);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));  // tmp is released after this point
    L.r_ready = false;
    h->levels[l] = L;
    step.done();
}

// R's values (and their FP32 copies, when present) for the given omega
static void rop_values(Level &L, double omega, hipStream_t st) {
    if (L.ah) {
        const int64_t nnz = L.A.nnz;
        k_ahat_values<<<grid_n(nnz), kBlock, 0, st>>>(nnz, L.A.col, L.A.val, L.A.valT, L.A.diag,
                                                      omega, L.ah, L.ahT);
        if (L.ah32) {
            k_rop_f32<<<grid_n(nnz), kBlock, 0, st>>>(L.ah, L.ah32, nnz);
            k_rop_f32<<<grid_n(nnz), kBlock, 0, st>>>(L.ahT, L.ahT32, nnz);
        }
        HIP_CHECK(hipGetLastError());
        L.r_omega = omega;
        L.r_ready = true;
        return;
    }
    auto fill = [&](auto &R) {
        k_rop_values<<<grid_n(R.nnz), kBlock, 0, st>>>(R.nnz, R, L.r_src0, L.r_srcn, L.r_src,
                                                      L.A.val, L.A.valT, L.A.diag, omega);
        if (R.val32) {
            k_rop_f32<<<grid_n(R.nnz), kBlock, 0, st>>>(R.val, R.val32, R.nnz);
            k_rop_f32<<<grid_n(R.nnz), kBlock, 0, st>>>(R.valT, R.valT32, R.nnz);
        }
    };
    if (L.R.sptr) fill(L.R);
    else fill(L.Rc);
    if (L.Uc.rptr) {
        k_up_fill<false><<<grid_n((int64_t)L.n * kUpLanes), kBlock, 0, st>>>(L.A, L.Uc, nullptr,
                                                                           L.agg, omega);
        if (L.Uc.val32) {
            k_rop_f32<<<grid_n(L.Uc.nnz), kBlock, 0, st>>>(L.Uc.val, L.Uc.val32, L.Uc.nnz);
            k_rop_f32<<<grid_n(L.Uc.nnz), kBlock, 0, st>>>(L.Uc.valT, L.Uc.valT32, L.Uc.nnz);
        }
    }
    HIP_CHECK(hipGetLastError());
    L.r_omega = omega;
    L.r_ready = true;
}

// FP32 copies of an operator's values: both, or none when memory runs out
static void make_f32(ldu_t *h, int64_t nnz, float *&v, float *&vT) {
    Arena::Step step(h->gamg_arena);
    float *a = h->gamg_arena.get<float>(nnz);
    vT = h->gamg_arena.get<float>(nnz);
    v = a;
    step.done();
}

// R for every level but the coarsest, for the cycles whose down leg it
// replaces: structure once per hierarchy, values again after new
// coefficients or another omega, FP32 copies once the FP32 path is in use
static void ensure_rop(ldu_t *h, const ldu_gamg_opts &o, hipStream_t st) {
    if (!rop_cycle(o)) return;
    const bool f32 = h->L0.A.val32 != nullptr;
    for (size_t l = 0; l + 1 < h->levels.size(); ++l) {
        Level &L = h->levels[l];
        if (!L.R.sptr && !L.Rc.rptr && !L.ah) rop_structure(h, l, st);
        const bool fresh = L.r_ready && L.r_omega == o.omega;
        if (!fresh) rop_values(L, o.omega, st);
        auto f32_copies = [&](auto &R) {
            if (!f32 || R.val32) return;  // values are current: only the FP32 copies are new
            make_f32(h, R.nnz, R.val32, R.valT32);
            k_rop_f32<<<grid_n(R.nnz), kBlock, 0, st>>>(R.val, R.val32, R.nnz);
            k_rop_f32<<<grid_n(R.nnz), kBlock, 0, st>>>(R.valT, R.valT32, R.nnz);
        };
        if (L.ah) {
            if (f32 && !L.ah32) {
                make_f32(h, L.A.nnz, L.ah32, L.ahT32);
                k_rop_f32<<<grid_n(L.A.nnz), kBlock, 0, st>>>(L.ah, L.ah32, L.A.nnz);
                k_rop_f32<<<grid_n(L.A.nnz), kBlock, 0, st>>>(L.ahT, L.ahT32, L.A.nnz);
            }
        } else if (L.R.sptr) {
            f32_copies(L.R);
        } else {
            f32_copies(L.Rc);
            if (L.Uc.rptr) f32_copies(L.Uc);
        }
        HIP_CHECK(hipGetLastError());
    }
}

// the values at up to 3 kMaxLevels addresses, for one look of the host
struct Sizes {
    const int64_t *at[3 * kMaxLevels];
    int n = 0;
};
__global__ void k_sizes(Sizes s, int64_t *out) {
    for (int k = threadIdx.x; k < s.n; k += blockDim.x) out[k] = *s.at[k];
}
static std::vector<int64_t> read_sizes(const Sizes &s, Arena &tmp, hipStream_t st) {
    std::vector<int64_t> v(s.n);
    int64_t *out = tmp.get<int64_t>(s.n);
    k_sizes<<<1, kWave, 0, st>>>(s, out);
    HIP_CHECK(hipMemcpyAsync(v.data(), out, sizeof(int64_t) * s.n, hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    return v;
}

// V's and W's structure for the small levels that have none yet, all levels in
// step: the host looks at their sizes twice in all.  With three looks a level
// the default set-up took 9.2 ms on a 300 x 200 x 1 mesh and 12.6 on 40 x 37 x
// 31, now 8.1 and 11.2 (before there were V and W 8.3 and 10.7)
static void gen_structures(ldu_t *h, hipStream_t st) {
    struct Build {
        size_t l;
        Level L;  // a copy, as in rop_structure
        int64_t *cnt, *tcnt, *tstart, *wide, total;
        int32_t *tcol, *rdeg;
    };
    std::vector<Build> todo;
    for (size_t l = 0; l + 1 < h->levels.size(); ++l) {
        const Level &L = h->levels[l];
        if (L.n <= kUpRows && !L.g_wide && !L.V.rptr) todo.push_back({l, L});
    }
    if (todo.empty()) return;
    Arena &ar = h->gamg_arena;
    Arena::Step step(ar);
    Arena tmp(&h->pool);
    auto bounds = [&](Csr &M, int32_t n, const int64_t *cnt) {
        M = Csr{};
        M.n = n;
        M.rptr = ar.get<int64_t>((size_t)n + 1);
        exclusive_scan_i64(cnt, M.rptr, n, tmp, st);
        return M.rptr + n;
    };
    auto arrays = [&](Csr &M, int64_t nnz) {
        M.nnz = nnz;
        M.col = ar.get<int32_t>(nnz);
        M.val = ar.get<double>(nnz);
        M.valT = ar.get<double>(nnz);
        M.group = csr_group(nnz, M.n);
    };
    int64_t *wide = tmp.get<int64_t>(todo.size());
    HIP_CHECK(hipMemsetAsync(wide, 0, sizeof(int64_t) * todo.size(), st));
    Sizes first;
    for (Build &b : todo) {
        Level &L = b.L;
        const Level &C = h->levels[b.l + 1];
        b.wide = wide++;
        b.cnt = tmp.get<int64_t>(L.n);
        b.tcnt = tmp.get<int64_t>(C.n);
        b.tstart = tmp.get<int64_t>((size_t)C.n + 1);
        k_up_count<<<grid_n((int64_t)L.n * kUpLanes), kBlock, 0, st>>>(L.A, L.agg, b.cnt, b.wide);
        k_rop_count<<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.aggStart, L.aggCells, L.A, b.tcnt,
                                                    b.wide);
        first.at[first.n++] = bounds(L.V, L.n, b.cnt);
        exclusive_scan_i64(b.tcnt, b.tstart, C.n, tmp, st);
        first.at[first.n++] = b.tstart + C.n;
        first.at[first.n++] = b.wide;
    }
    const std::vector<int64_t> v = read_sizes(first, tmp, st);
    Sizes second;
    for (size_t k = 0; k < todo.size(); ++k) {
        Build &b = todo[k];
        Level &L = b.L;
        const Level &C = h->levels[b.l + 1];
        if (v[3 * k + 2]) {
            L = h->levels[b.l];
            L.g_wide = true;
            continue;
        }
        arrays(L.V, v[3 * k]);
        b.total = v[3 * k + 1];
        L.qptr = ar.get<int64_t>(L.n);
        b.tcol = tmp.get<int32_t>(b.total);
        b.rdeg = tmp.get<int32_t>(C.n);
        L.w_src = ar.get<int64_t>(b.total);
        k_rop_gather<<<grid_n((int64_t)C.n * kWave), kBlock, 0, st>>>(
            C.n, L.aggStart, L.aggCells, L.A, b.tstart, b.tcol, L.w_src, b.rdeg);
        k_w_count<<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.aggStart, b.rdeg, b.tcnt);
        second.at[second.n++] = bounds(L.W, C.n, b.tcnt);
    }
    if (second.n) {
        const std::vector<int64_t> w = read_sizes(second, tmp, st);
        size_t q = 0;
        for (Build &b : todo) {
            Level &L = b.L;
            const Level &C = h->levels[b.l + 1];
            if (L.g_wide) continue;
            arrays(L.W, w[q++]);
            L.w_src0 = ar.get<int64_t>(L.W.nnz);
            L.w_srcn = ar.get<int32_t>(L.W.nnz);
            k_w_link<<<grid_n(C.n), kBlock, 0, st>>>(C.n, L.n, L.W, L.aggStart, L.aggCells,
                                                    b.tstart, b.tcol, L.w_src0, L.w_srcn);
            L.g_ready = false;
        }
    }
    HIP_CHECK(hipGetLastError());
    for (const Build &b : todo) h->levels[b.l] = b.L;
    step.done();  // tmp's chunks are used again in this stream's order
}

// V and W for the small levels of the other Jacobi cycles: structure once per
// hierarchy, values again after new coefficients or another omega, FP32 copies
// once the FP32 path is in use
static void ensure_gen(ldu_t *h, const ldu_gamg_opts &o, hipStream_t st) {
    if (!gen_cycle(o)) return;
    gen_structures(h, st);
    const bool f32 = h->L0.A.val32 != nullptr;
    for (size_t l = 0; l + 1 < h->levels.size(); ++l) {
        Level &L = h->levels[l];
        if (L.n > kUpRows || L.g_wide) continue;
        const bool fresh = L.g_ready && L.g_omega == o.omega;
        if (!fresh) {
            k_up_fill<true><<<grid_n((int64_t)L.n * kUpLanes), kBlock, 0, st>>>(
                L.A, L.V, L.qptr, L.agg, o.omega);
            k_w_values<<<grid_n(L.W.nnz), kBlock, 0, st>>>(L.W.nnz, L.n, L.W, L.w_src0, L.w_srcn,
                                                          L.w_src, L.A.val, L.A.valT, L.A.diag);
            L.g_omega = o.omega;
            L.g_ready = true;
        }
        for (Csr *M : {&L.V, &L.W}) {
            const bool made = f32 && !M->val32;
            if (made) make_f32(h, M->nnz, M->val32, M->valT32);
            if (M->val32 && (made || !fresh)) {
                k_rop_f32<<<grid_n(M->nnz), kBlock, 0, st>>>(M->val, M->val32, M->nnz);
                k_rop_f32<<<grid_n(M->nnz), kBlock, 0, st>>>(M->valT, M->valT32, M->nnz);
            }
        }
        HIP_CHECK(hipGetLastError());
    }
}

// new level coefficients: R's values follow at once (same omega)
static void refresh_rop(ldu_t *h, hipStream_t st) {
    for (Level &L : h->levels) L.g_ready = false;  // V and W: by the next cycle that uses them
    for (size_t l = 0; l + 1 < h->levels.size(); ++l)
        if ((h->levels[l].R.sptr || h->levels[l].Rc.rptr || h->levels[l].ah) &&
            h->levels[l].r_ready)
            rop_values(h->levels[l], h->levels[l].r_omega, st);
}

// work vectors, operators and factors that a cycle needs beyond the hierarchy,
// made by the first cycle that asks for them: among them the second ping-pong
// vector of the two-stage smoother (three or more inner steps) and the DIC pivots
// of the coarsest level
static VCtx make_ctx(ldu_t *h, const ldu_gamg_opts &o, bool tr, hipStream_t st) {
    ensure_work(h);
    ensure_rop(h, o, st);
    ensure_gen(h, o, st);
    h->pool.trim();
    if (o.smoother == LDU_SMOOTH_GS2 && o.gs_inner >= 3) {
        for (auto &L : h->levels) {
            if (!L.w) L.w = h->gamg_arena.get<double>(L.n);
            if (!L.w32) L.w32 = h->gamg_arena.get<float>(L.n);
        }
    }
    const double *dt = nullptr;
    if (o.coarsest == LDU_COARSE_DIC) {
        ensure_dic(h, st);
        if (h->dic_ok) dt = h->dic_dt;
    }
    return VCtx{h, &o, tr, st, h->coarse_work, dt};
}

static void fill_level_stats(ldu_t *h, ldu_stats *stats) {
    if (!stats) return;
    stats->n_levels = (int)h->levels.size();
    for (int l = 0; l < 64; ++l) {
        const bool in = l < (int)h->levels.size();
        stats->level_cells[l] = in ? h->levels[l].n : 0;
        stats->level_faces[l] = in ? h->levels[l].nf : 0;
    }
}

void gamg_vcycle64(ldu_t *h, const double *r, double *e, const ldu_gamg_opts &o, bool tr,
                   hipStream_t st) {
    refresh_inner(h, o.smoother, st);
    NumberingScope scope(h, o.smoother);
    const InnerVectors v = inner_vectors(h, scope.active(), r, e, false, st);
    set_scalars_for_solve(h, 0.0, 0, st);
    VCtx c = make_ctx(h, o, tr, st);
    double *res = vcycle<double>(c, 0, v.in);
    HIP_CHECK(hipMemcpyAsync(v.out, res, sizeof(double) * h->L0.n, hipMemcpyDeviceToDevice, st));
    HIP_CHECK(hipStreamSynchronize(st));
    inner_result(h, scope.active(), e, st);
}

static int finish_status(const DevScalars &hs) {
    if (hs.done == kFailed) return hs.status;
    if (hs.done == kMaxIter) return LDU_NOT_CONVERGED;
    return LDU_OK;
}

// standalone cycles launched before the host looks at the residual again, at
// most: each look costs an idle gap of 20-30 us
constexpr int kCycleBatch = 8;
// Cycles, and iterations of the CG forms, before the first look.  A full batch
// here made short solves pay for iterations that did nothing: gamg_solve with
// max_cycles 1 on 32^3, 64^3 and 128^3 1245, 1872 and 2833 us against 298, 418
// and 1015 with a look after the first cycle (each cycle looked at, before the
// small levels ran through V and W: 415, 633 and 1320); CG + V-cycle to a
// residual of 0.5, one iteration, 1054, 1987 and 2629 us against 443, 628 and
// 1123.  Long solves pay one more look.
constexpr int kFirstCycles = 1, kFirstIterations = 4;

static int gamg_fp64_run(ldu_t *h, const double *b, double *x, const ldu_gamg_opts &o, bool tr,
              ldu_stats *stats, hipStream_t st) {
    Level &L = h->levels[0];
    SellView<double> A = L.A.view(tr);
    A.stream = L.A.bytes(sizeof(double)) + 5 * (int64_t)sizeof(double) * L.n > kCacheBytes;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    ensure_hist(h, (int64_t)o.max_cycles + 2);
    fill_level_stats(h, stats);
    if (stats) { stats->refinements = 0; stats->history_count = 0; }
    set_scalars_for_solve(h, o.rel_tol, o.max_cycles, st);
    VCtx c = make_ctx(h, o, tr, st);
    launch_residual_cycle(h, A, b, x, h->r, false, G, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        zero_vector(x, L.n, st);
        if (stats) {
            stats->iterations = 0;
            stats->converged = 1;
            stats->initial_residual = stats->final_residual = 0.0;
        }
        copy_history(h, stats, 1, st);
        return LDU_OK;
    }
    const double res0 = hs.res;
    while (hs.done == kRunning) {
        const int cycles = hs.iters - 1;  // done so far
        const int batch = next_batch(res0, hs.res, cycles, o.rel_tol, kFirstCycles,
                                     std::min(kCycleBatch, o.max_cycles - cycles));
        for (int k = 0; k < batch; ++k) {
            const double *e = vcycle<double>(c, 0, h->r);
            k_add<<<G, kBlock, 0, st>>>(L.n, S, e, x, h->dev);
            launch_residual_cycle(h, A, b, x, h->r, false, G, st);
        }
        read_scalars(h, st);
    }
    const int status = finish_status(hs);
    if (stats) {
        stats->iterations = hs.iters;
        stats->final_residual = hs.res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, hs.iters + 1, st);
    return status;
}

// ---------------------------------------------------------------- CG + V-cycle
// CG preconditioned by one V-cycle per iteration, correction scaling off so
// that the preconditioner is one fixed symmetric operator: the pairing of the
// paper's AmgX configuration (Appendix A listing: PCG with an AMG V-cycle
// preconditioner) on this GAMG hierarchy.

// p = z; rho = r.z
__global__ void __launch_bounds__(kBlock)
k_pg_start(int32_t n, int64_t S, const double *__restrict__ r, const double *__restrict__ z,
           double *__restrict__ p, double *partials, const DevScalars *ds) {
    if (ds->done) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            const double zi = z[i];
            p[i] = zi;
            acc[0] += r[i] * zi;
        }
    });
    block_partials<1>(acc, partials);
}

struct EpiRho {
    __device__ bool active(const DevScalars *ds) const { return !ds->done; }
    __device__ void operator()(const double *t, DevScalars *ds) const {
        ds->rho = t[0];
        ds->x_pending = 0;
    }
};

// r -= alpha q; ||r||^2.  The iteration's x += alpha p waits for the
// direction update, which reads p anyway (k_pg_p), or, when the solve stops
// in between, for k_x_pending: one read of p per iteration instead of two.
template <bool NT>
__global__ void __launch_bounds__(kBlock)
k_pg_update(int32_t n, int64_t S, double *__restrict__ r, const double *__restrict__ q,
            double *partials, int nblocks, const DevScalars *in, DevScalars *out) {
    const Step st = step_alpha(partials, nblocks, in, out);
    if (!st.go) return;
    const double alpha = st.alpha;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            const double ri = vld<NT>(r + i) - alpha * vld<NT>(q + i);
            vst<NT>(r + i, ri);
            acc[0] += ri * ri;
        }
    });
    block_partials<1>(acc, partials + kMaxGrid);
}


// the partials of r.z, for a V-cycle whose last kernel did not take them
__global__ void __launch_bounds__(kBlock)
k_pg_rz(int32_t n, int64_t S, const double *__restrict__ r, const double *__restrict__ z,
        double *partials, const DevScalars *ds) {
    if (ds->done) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) acc[0] += r[i] * z[i];
    });
    block_partials<1>(acc, partials);
}

// x += alpha p (the iteration's solution update, deferred from k_pg_update);
// p = z + beta p.  x and z are not read again before the next iteration's
// direction update, so they stream past the caches (nontemporal) at every
// size, while p keeps the default policy at every size: the new p, which the
// CG product gathers next, then stays in the Infinity Cache (the c3 CG
// product went from 133 to 122 us).  This kernel and the residual update take
// beta and alpha from their producers' partials (100^3: 15.95 -> 15.2 ms,
// 200^3: 125.6 -> 124.4 ms; the mixed forms' inner CG likewise).
__global__ void __launch_bounds__(kBlock)
k_pg_p(int32_t n, int64_t S, double *__restrict__ x, const double *__restrict__ z,
       double *__restrict__ p, const double *partials, int nblocks, int mode,
       const DevScalars *in, DevScalars *out) {
    const Step st = step_beta(mode, partials, nblocks, in, out);
    if (!st.go || mode == kStepFirst) return;  // the first direction is there already
    const double alpha = st.alpha, beta = st.beta;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            const double pi = p[i];
            vst<true>(x + i, vld<true>(x + i) + alpha * pi);
            p[i] = vld<true>(z + i) + beta * pi;
        }
    });
}

static int pcg_gamg_fp64_run(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
                  ldu_stats *stats, hipStream_t st) {
    ldu_gamg_opts go = h->gamg_opts;
    go.scale_correction = 0;
    Level &L = h->levels[0];
    const SellView<double> A = L.A.view(tr);
    const int n = L.n;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    // products on plain slices: blocks past the cap would only add zeros
    const int Gq = A.pdeg ? G : std::min(G, kPlainF64ProductBlocks);
    const bool nt = n > kStreamNtCells;
    ensure_hist(h, (int64_t)o.max_iter + 2);
    fill_level_stats(h, stats);
    if (stats) { stats->refinements = 0; stats->history_count = 0; }
    set_scalars_for_solve(h, o.rel_tol, o.max_iter, st);
    VCtx c = make_ctx(h, go, tr, st);
    launch_residual_plain(h, A, b, x, h->r, true, G, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        zero_vector(x, n, st);
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
    while (res > o.rel_tol) {
        const double *z = vcycle<double>(c, 0, h->r);
        k_pg_start<<<G, kBlock, 0, st>>>(n, S, h->r, z, h->p, h->partials, h->dev);
        launch_finalize<1>(h->partials, G, h->dev, EpiRho{}, st);
        k_pg_p<<<1, kBlock, 0, st>>>(n, S, x, z, h->p, h->partials, G, kStepFirst, h->dev,
                                     h->dev + 1);  // passes the scalars on
        const double res0 = res;
        const int iters0 = hs.iters;
        for (;;) {
            const int batch = next_batch(res0, hs.res, hs.iters - iters0, o.rel_tol,
                                         std::min(kFirstIterations, every),
                                         std::min(every, o.max_iter - hs.iters));
            for (int k = 0; k < batch; ++k) {
                launch_product_dot(h, A, h->p, h->q, Gq, h->dev + 1, st);
                if (nt)
                    k_pg_update<true><<<G, kBlock, 0, st>>>(n, S, h->r, h->q, h->partials, Gq,
                                                            h->dev + 1, h->dev);
                else
                    k_pg_update<false><<<G, kBlock, 0, st>>>(n, S, h->r, h->q, h->partials, Gq,
                                                             h->dev + 1, h->dev);
                launch_converge(h, h->partials + kMaxGrid, G, st);
                int blocks = 0;  // the last level-0 kernel may take r.z itself
                z = vcycle<double>(c, 0, h->r, h->r, &blocks);
                if (!blocks) k_pg_rz<<<G, kBlock, 0, st>>>(n, S, h->r, z, h->partials, h->dev);
                k_pg_p<<<G, kBlock, 0, st>>>(n, S, x, z, h->p, h->partials, blocks ? blocks : G,
                                             kStepReduce, h->dev, h->dev + 1);
            }
            HIP_CHECK(hipGetLastError());
            read_scalars(h, st);
            if (hs.done != kRunning) break;
        }
        // the stopping iteration's x += alpha p (none when alpha itself failed)
        launch_x_pending(h, x, h->p, n, S, G, st);
        if (hs.done == kFailed) {
            status = hs.status;
            break;
        }
        launch_residual_plain(h, A, b, x, h->r, false, G, st);
        read_scalars(h, st);
        res = hs.res;
        if (!std::isfinite(res)) { status = LDU_ERR_NAN; break; }
        if (res <= o.rel_tol) { status = LDU_OK; break; }
        if (hs.iters >= o.max_iter) { status = LDU_NOT_CONVERGED; break; }
        set_done(h, kRunning, st);
    }
    if (stats) {
        stats->iterations = hs.iters;
        stats->final_residual = res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, hs.iters + 1, st);
    return status;
}

// FP32 inner CG preconditioned by an FP32 V-cycle (FP64 coarsest), inside FP64
// refinement; inner dot products in FP64, alpha/beta rounded to FP32

// rhat = fp32(r / ||r||_inf), d = 0; ||rhat||^2
__global__ void __launch_bounds__(kBlock)
k_mxg_start(int32_t n, int64_t S, const double *__restrict__ r, float *__restrict__ r32,
            float *__restrict__ d32, double *partials, const DevScalars *ds) {
    if (ds->done) return;
    const double sc = ds->maxabs;
    const int lane = threadIdx.x & 63;
    double acc[2] = {0.0, 0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            const float ri = (float)(r[i] / sc);
            r32[i] = ri;
            d32[i] = 0.0f;
            acc[0] += (double)ri * (double)ri;
        }
    });
    block_partials<2>(acc, partials);
}

// p = z; rho = r.z (FP32 vectors, FP64 sum)
__global__ void __launch_bounds__(kBlock)
k_mxg_p0(int32_t n, int64_t S, const float *__restrict__ r, const float *__restrict__ z,
         float *__restrict__ p, double *partials, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) {
            p[i] = z[i];
            acc[0] += (double)r[i] * (double)z[i];
        }
    });
    block_partials<1>(acc, partials);
}

struct EpiMxRho {
    __device__ bool active(const DevScalars *ds) const { return !vc_skip(ds); }
    __device__ void operator()(const double *t, DevScalars *ds) const { ds->rho = t[0]; }
};

// the partials of r.z, for a V-cycle whose last kernel did not take them
__global__ void __launch_bounds__(kBlock)
k_mxg_rz(int32_t n, int64_t S, const float *__restrict__ r, const float *__restrict__ z,
         double *partials, const DevScalars *ds) {
    if (vc_skip(ds)) return;
    const int lane = threadIdx.x & 63;
    double acc[1] = {0.0};
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) acc[0] += (double)r[i] * (double)z[i];
    });
    block_partials<1>(acc, partials);
}

__global__ void __launch_bounds__(kBlock)
k_mxg_p(int32_t n, int64_t S, const float *__restrict__ z, float *__restrict__ p,
        const double *partials, int nblocks, int mode, const DevScalars *in, DevScalars *out) {
    const Step st = step_mx_beta(mode, partials, nblocks, in, out);
    if (!st.go || mode == kStepFirst) return;  // the first direction is there already
    const float bf = (float)st.beta;
    const int lane = threadIdx.x & 63;
    for_each_slice(S, [&](int64_t s) {
        const int64_t i = s * kWave + lane;
        if (i < n) p[i] = z[i] + bf * p[i];
    });
}

struct EpiMxgStart {
    __device__ bool active(const DevScalars *ds) const { return !ds->done; }
    __device__ void operator()(const double *t, DevScalars *ds) const {
        ds->scale = ds->maxabs;
        ds->r0 = sqrt(t[0]);
        ds->inner_iters = 0;
        ds->inner_done = !(ds->r0 > 0.0);
        const double target = 0.3 * ds->tol / ds->res;
        ds->inner_now = target > ds->inner_tol ? target : ds->inner_tol;
    }
};

static int pcg_gamg_mixed_run(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
                   ldu_stats *stats, hipStream_t st) {
    ensure_work32(h, st);
    ldu_gamg_opts go = h->gamg_opts;
    go.scale_correction = 0;
    Level &L = h->levels[0];
    const SellView<double> A = L.A.view(tr);
    const SellView<float> A32 = L.A.view32(tr);
    const int n = L.n;
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    const int Gr = cg_blocks(n, G);
    ensure_hist(h, (int64_t)o.max_refine + 2);
    fill_level_stats(h, stats);
    if (stats) stats->history_count = 0;
    set_scalars_for_solve(h, o.rel_tol, o.max_refine, st);
    set_inner(h, o.inner_rel_tol, o.inner_max_iter, st);
    VCtx c = make_ctx(h, go, tr, st);
    launch_residual_cycle(h, A, b, x, h->r, true, G, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        zero_vector(x, n, st);
        if (stats) {
            stats->iterations = 0;
            stats->refinements = 0;
            stats->converged = 1;
            stats->initial_residual = stats->final_residual = 0.0;
        }
        copy_history(h, stats, 1, st);
        return LDU_OK;
    }
    const int every = o.check_every > 0 ? o.check_every : 16;
    long long inner_total = 0;
    while (hs.done == kRunning) {
        k_mxg_start<<<G, kBlock, 0, st>>>(n, S, h->r, h->r32, h->d32, h->partials, h->dev);
        launch_finalize<2>(h->partials, G, h->dev, EpiMxgStart{}, st);
        const float *z = vcycle<float>(c, 0, h->r32);
        k_mxg_p0<<<G, kBlock, 0, st>>>(n, S, h->r32, z, h->p32, h->partials, h->dev);
        launch_finalize<1>(h->partials, G, h->dev, EpiMxRho{}, st);
        k_mxg_p<<<1, kBlock, 0, st>>>(n, S, z, h->p32, h->partials, G, kStepFirst, h->dev,
                                      h->dev + 1);  // passes the scalars on
        int batch = std::min({kFirstIterations, every, o.inner_max_iter});
        for (;;) {
            for (int k = 0; k < batch; ++k) {
                launch_mx_q(h, A32, G, st);
                launch_mx_update_plain(h, n, S, Gr, G, st);
                int blocks = 0;  // the last level-0 kernel may take r.z itself
                z = vcycle<float>(c, 0, h->r32, h->r32, &blocks);
                if (!blocks) k_mxg_rz<<<G, kBlock, 0, st>>>(n, S, h->r32, z, h->partials, h->dev);
                k_mxg_p<<<Gr, kBlock, 0, st>>>(n, S, z, h->p32, h->partials, blocks ? blocks : G,
                                               kStepReduce, h->dev, h->dev + 1);
            }
            HIP_CHECK(hipGetLastError());
            read_scalars(h, st);
            if (hs.inner_done) break;
            batch = next_batch(hs.r0, std::sqrt(hs.rr), hs.inner_iters, hs.inner_now * hs.r0,
                               every, std::min(every, o.inner_max_iter - hs.inner_iters));
        }
        inner_total += hs.inner_iters;
        launch_mx_refine(h, x, n, S, G, st);
        launch_residual_cycle(h, A, b, x, h->r, true, G, st);
        read_scalars(h, st);
    }
    const int status = finish_status(hs);
    if (stats) {
        stats->iterations = (int)inner_total;
        stats->refinements = hs.iters;
        stats->final_residual = hs.res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, hs.iters + 1, st);
    return status;
}

static int gamg_mixed_run(ldu_t *h, const double *b, double *x, const ldu_gamg_opts &o, bool tr,
               ldu_stats *stats, hipStream_t st) {
    ensure_work32(h, st);
    Level &L = h->levels[0];
    const SellView<double> A = L.A.view(tr);
    const int64_t S = L.A.nslices;
    const int G = stream_grid_slices(S);
    ensure_hist(h, (int64_t)o.max_refine + 2);
    fill_level_stats(h, stats);
    if (stats) stats->history_count = 0;
    set_scalars_for_solve(h, o.rel_tol, o.max_refine, st);
    VCtx c = make_ctx(h, o, tr, st);
    launch_residual_cycle(h, A, b, x, h->r, true, G, st);
    read_scalars(h, st);
    DevScalars &hs = *h->host;
    if (stats) stats->initial_residual = hs.res;
    if (hs.bnorm == 0.0) {
        zero_vector(x, L.n, st);
        if (stats) {
            stats->iterations = 0;
            stats->refinements = 0;
            stats->converged = 1;
            stats->initial_residual = stats->final_residual = 0.0;
        }
        copy_history(h, stats, 1, st);
        return LDU_OK;
    }
    const double res0 = hs.res;
    while (hs.done == kRunning) {
        const int cycles = hs.iters - 1;  // done so far
        const int batch = next_batch(res0, hs.res, cycles, o.rel_tol, kFirstCycles,
                                     std::min(kCycleBatch, o.max_refine - cycles));
        for (int k = 0; k < batch; ++k) {
            k_cast_scaled<<<G, kBlock, 0, st>>>(L.n, S, h->r, L.r32, h->dev);
            const float *d = vcycle<float>(c, 0, L.r32);
            k_refine_add<<<G, kBlock, 0, st>>>(L.n, S, d, x, h->dev);
            launch_residual_cycle(h, A, b, x, h->r, true, G, st);
        }
        read_scalars(h, st);
    }
    const int status = finish_status(hs);
    if (stats) {
        stats->iterations = hs.iters;
        stats->refinements = hs.iters;
        stats->final_residual = hs.res;
        stats->converged = (status == LDU_OK);
    }
    copy_history(h, stats, hs.iters + 1, st);
    return status;
}

// ---------------------------------------------------------------- entry points
// the solves in the numbering that suits them
template <class Run>
static int in_numbering(ldu_t *h, int smoother, const double *b, double *x, hipStream_t st,
                        Run &&run) {
    refresh_inner(h, smoother, st);
    NumberingScope scope(h, smoother);
    const InnerVectors v = inner_vectors(h, scope.active(), b, x, true, st);
    const int rc = run(v.in, v.out);
    inner_result(h, scope.active(), x, st);
    return rc;
}

int gamg_fp64(ldu_t *h, const double *b, double *x, const ldu_gamg_opts &o, bool tr,
              ldu_stats *stats, hipStream_t st) {
    return in_numbering(h, o.smoother, b, x, st, [&](const double *bi, double *xi) {
        return gamg_fp64_run(h, bi, xi, o, tr, stats, st);
    });
}
int gamg_mixed(ldu_t *h, const double *b, double *x, const ldu_gamg_opts &o, bool tr,
               ldu_stats *stats, hipStream_t st) {
    return in_numbering(h, o.smoother, b, x, st, [&](const double *bi, double *xi) {
        return gamg_mixed_run(h, bi, xi, o, tr, stats, st);
    });
}
int pcg_gamg_fp64(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
                  ldu_stats *stats, hipStream_t st) {
    return in_numbering(h, h->gamg_opts.smoother, b, x, st, [&](const double *bi, double *xi) {
        return pcg_gamg_fp64_run(h, bi, xi, o, tr, stats, st);
    });
}
int pcg_gamg_mixed(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
                   ldu_stats *stats, hipStream_t st) {
    return in_numbering(h, h->gamg_opts.smoother, b, x, st, [&](const double *bi, double *xi) {
        return pcg_gamg_mixed_run(h, bi, xi, o, tr, stats, st);
    });
}

}  // namespace ldu
