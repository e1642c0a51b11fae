// LDU -> sliced-ELLPACK re-layout, value maps and scans (setup kernels).
//
// The paper's external-solver path converts OpenFOAM's LDU arrays to a
// row-ordered (CSR) matrix through a permutation map computed once and reused
// when the values change (Sec. 3.4).  Here the same idea produces the
// row-segmented layout the product kernels stream: per row its "lower"
// entries (faces where the row is the neighbour, i.e. OpenFOAM's losort
// order) followed by its "upper" entries (faces it owns), column-sorted, and
// two face -> position maps (slotU, slotL) so that new coefficients are
// scattered in place without redoing the structure.
#include "device.hpp"

#include <algorithm>

namespace ldu {

// ---------------------------------------------------------------- scans
constexpr int kScanItems = 8;
constexpr int kScanChunk = kBlock * kScanItems;

template <typename T>
__device__ T block_exclusive_scan(T v, T *total) {
    __shared__ T sm[kBlock];
    sm[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        T a = (threadIdx.x >= (unsigned)off) ? sm[threadIdx.x - off] : T(0);
        __syncthreads();
        sm[threadIdx.x] += a;
        __syncthreads();
    }
    T incl = sm[threadIdx.x];
    *total = sm[kBlock - 1];
    __syncthreads();
    return incl - v;
}

template <typename T>
__global__ void __launch_bounds__(kBlock) k_scan_partial(const T *in, int64_t n, T *bsum) {
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    T s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) s += in[base + k];
    T tot;
    block_exclusive_scan<T>(s, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// exclusive scan of nb block sums by one block (in place), total -> bsum[nb]
template <typename T>
__global__ void __launch_bounds__(kBlock) k_scan_sums(T *bsum, int64_t nb) {
    const int64_t per = (nb + kBlock - 1) / kBlock;
    const int64_t lo = (int64_t)threadIdx.x * per;
    T s = 0;
    for (int64_t k = lo; k < lo + per && k < nb; ++k) s += bsum[k];
    T tot;
    T off = block_exclusive_scan<T>(s, &tot);
    for (int64_t k = lo; k < lo + per && k < nb; ++k) {
        T v = bsum[k];
        bsum[k] = off;
        off += v;
    }
    if (threadIdx.x == 0) bsum[nb] = tot;
}

template <typename T>
__global__ void __launch_bounds__(kBlock) k_scan_final(const T *in, int64_t n, const T *bsum, T *out) {
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    T v[kScanItems];
    T s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : T(0);
        s += v[k];
    }
    T tot;
    T off = block_exclusive_scan<T>(s, &tot) + bsum[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = off;
        off += v[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = bsum[gridDim.x];
}

template <typename T>
static void exclusive_scan(const T *in, T *out, int64_t n, Arena &tmp, hipStream_t st) {
    const int64_t nb = (n + kScanChunk - 1) / kScanChunk;
    if (nb == 0) {
        HIP_CHECK(hipMemsetAsync(out, 0, sizeof(T), st));
        return;
    }
    T *bsum = tmp.get<T>(nb + 1);
    k_scan_partial<T><<<(unsigned)nb, kBlock, 0, st>>>(in, n, bsum);
    k_scan_sums<T><<<1, kBlock, 0, st>>>(bsum, nb);
    k_scan_final<T><<<(unsigned)nb, kBlock, 0, st>>>(in, n, bsum, out);
    HIP_CHECK(hipGetLastError());
}

void exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, Arena &tmp,
                        hipStream_t st) {
    exclusive_scan<int64_t>(in, out, n, tmp, st);
}
void scan_counts_i32(const int32_t *cnt, int32_t *out, int64_t n, Arena &tmp,
                     hipStream_t st) {
    exclusive_scan<int32_t>(cnt, out, n, tmp, st);
}

// ---------------------------------------------------------------- checks
__global__ void k_validate(int32_t n, int64_t nf, const int32_t *own, const int32_t *nb,
                           int *flag) {
    GRID_STRIDE(f, nf) {
        const int32_t o = own[f], b = nb[f];
        bool bad = o < 0 || o >= b || b >= n;
        if (f > 0) {
            const int32_t po = own[f - 1], pb = nb[f - 1];
            bad = bad || o < po || (o == po && b <= pb);
        }
        if (bad) atomicOr(flag, 1);
    }
}

__global__ void k_check_finite(const double *a, int64_t n, int *flag) {
    STREAM_STRIDE(i, n)
        if (!isfinite(a[i])) atomicOr(flag, 2);
}

static unsigned grid_for(int64_t n) {
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g > 8192) g = 8192;
    if (g >= 64) g = (g + 7) & ~int64_t(7);
    return (unsigned)(g < 1 ? 1 : g);
}

void check_finite(ldu_t *h, const double *a, int64_t n, hipStream_t st) {
    if (n > 0) k_check_finite<<<grid_for(n), kBlock, 0, st>>>(a, n, h->flag);
}

// ---------------------------------------------------------------- structure
// ownStart[i] = first face with owner >= i (faces are sorted by owner)
__global__ void k_own_start(int32_t n, int64_t nf, const int32_t *own, int64_t *ownStart) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= n;
         i += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = nf;
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if (own[mid] < i) lo = mid + 1; else hi = mid;
        }
        ownStart[i] = lo;
    }
}

__global__ void k_count_lower(int64_t nf, const int32_t *nb, int32_t *cntL) {
    GRID_STRIDE(f, nf)
        atomicAdd(&cntL[nb[f]], 1);
}

__global__ void k_degree(int32_t n, const int64_t *ownStart, const int32_t *cntL, int32_t *deg) {
    GRID_STRIDE(i, n)
        deg[i] = cntL[i] + (int32_t)(ownStart[i + 1] - ownStart[i]);
}

// entries of slice s = 64 x (longest row stored in the slice)
__global__ void k_slice_entries(int32_t n, int64_t S, const int32_t *deg, const int32_t *perm,
                                int64_t *entries) {
    GRID_STRIDE(s, S) {
        int64_t w = 0;
        for (int l = 0; l < kWave; ++l) {
            const int64_t p = s * kWave + l;
            if (p < n) {
                const int64_t d = deg[perm ? perm[p] : p];
                w = d > w ? d : w;
            }
        }
        entries[s] = w * kWave;
    }
}

// compressed slices: inside each slice of 64 rows, order the rows by length
// (longest first, ties by row index); positions past n hold no row (-1)
__global__ void k_slice_sort(int32_t n, int64_t S, const int32_t *deg, int32_t *perm,
                             int32_t *iperm, int32_t *pdeg) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < S * kWave;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s0 = (q >> 6) << 6;
        const int l = (int)(q & 63);
        const int32_t dl = q < n ? deg[q] : -1;
        int rank = 0;
        for (int j = 0; j < kWave; ++j) {
            const int32_t dj = (s0 + j) < n ? deg[s0 + j] : -1;
            rank += (dj > dl) || (dj == dl && j < l);
        }
        perm[s0 + rank] = q < n ? (int32_t)q : -1;
        pdeg[s0 + rank] = dl > 0 ? dl : 0;
        if (q < n) iperm[q] = (int32_t)(s0 + rank);
    }
}

// entries of a compressed slice (sum of its row lengths) and the length of
// its offset table (longest row + 1)
__global__ void k_slice_sizes(int64_t S, const int32_t *pdeg, int64_t *entries, int32_t *tlen) {
    GRID_STRIDE(s, S) {
        int64_t e = 0;
        for (int l = 0; l < kWave; ++l) e += pdeg[s * kWave + l];
        entries[s] = e;
        tlen[s] = pdeg[s * kWave] + 1;
    }
}

// otab[tptr[s] + k] = entries of slice s in its columns 0..k-1
__global__ void k_slice_table(int64_t S, const int32_t *pdeg, const int32_t *tptr, int32_t *otab) {
    GRID_STRIDE(s, S) {
        const int w = pdeg[s * kWave];
        int32_t off = 0;
        for (int k = 0; k <= w; ++k) {
            otab[tptr[s] + k] = off;
            int cnt = 0;
            for (int l = 0; l < kWave; ++l) cnt += pdeg[s * kWave + l] > k;
            off += cnt;
        }
    }
}

// max of a[0..n) (values >= 0) into *out, which the caller zeroes: one
// partial per block, combined by an integer atomic max (order-independent)
__global__ void __launch_bounds__(kBlock) k_max_i32(const int32_t *a, int64_t n, int32_t *out) {
    __shared__ int32_t sm[kBlock];
    int32_t m = 0;
    GRID_STRIDE(i, n)
        m = a[i] > m ? a[i] : m;
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (threadIdx.x < (unsigned)off && sm[threadIdx.x + off] > sm[threadIdx.x])
            sm[threadIdx.x] = sm[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicMax(out, sm[0]);
}

__global__ void k_fill_i32(int32_t *a, int64_t n, int32_t v) {
    GRID_STRIDE(i, n)
        a[i] = v;
}

// storage index of entry k of row i (plain or compressed slices)
struct Slots {
    const int64_t *sptr;
    const int32_t *iperm, *tptr, *otab;
    __device__ __forceinline__ int64_t operator()(int64_t i, int64_t k) const {
        const int64_t p = iperm ? (int64_t)iperm[i] : i;
        const int64_t s = p >> 6;
        if (otab) return sptr[s] + otab[tptr[s] + k] + (p & 63);
        return sptr[s] + k * kWave + (p & 63);
    }
};

__global__ void k_fill_upper(int64_t nf, const int32_t *own, const int32_t *nb,
                             const int64_t *ownStart, const int32_t *cntL, Slots slot,
                             int32_t *col, int64_t *slotU) {
    GRID_STRIDE(f, nf) {
        const int32_t i = own[f];
        const int64_t pos = slot(i, cntL[i] + (f - ownStart[i]));
        col[pos] = nb[f];
        slotU[f] = pos;
    }
}

// lower entries land in arbitrary order within their row; k_sort_lower
// orders them by column, which makes the final layout deterministic
__global__ void k_fill_lower(int64_t nf, const int32_t *own, const int32_t *nb, Slots slot,
                             int32_t *cursor, int32_t *col, int64_t *faceAt) {
    GRID_STRIDE(f, nf) {
        const int32_t j = nb[f];
        const int k = atomicAdd(&cursor[j], 1);
        const int64_t pos = slot(j, k);
        col[pos] = own[f];
        faceAt[pos] = f;
    }
}

// rows of at most kSortRegs lower entries are ranked in registers (all loads
// of the row together), longer ones by an insertion sort in place
constexpr int kSortRegs = 8;

__global__ void k_sort_lower(int32_t n, Slots slot, const int32_t *cntL, int32_t *col,
                             int64_t *faceAt, int64_t *slotL) {
    GRID_STRIDE(j, n) {
        const int m = cntL[j];
        if (m <= kSortRegs) {
            int64_t pos[kSortRegs], f[kSortRegs];
            int32_t c[kSortRegs];
#pragma unroll
            for (int a = 0; a < kSortRegs; ++a) pos[a] = a < m ? slot(j, a) : 0;
#pragma unroll
            for (int a = 0; a < kSortRegs; ++a) {
                c[a] = a < m ? col[pos[a]] : INT32_MAX;
                f[a] = a < m ? faceAt[pos[a]] : 0;
            }
#pragma unroll
            for (int a = 0; a < kSortRegs; ++a) {
                if (a >= m) continue;
                int rank = 0;
#pragma unroll
                for (int b = 0; b < kSortRegs; ++b) rank += c[b] < c[a];  // columns are distinct
                int64_t to = pos[0];
#pragma unroll
                for (int b = 1; b < kSortRegs; ++b) to = rank == b ? pos[b] : to;
                col[to] = c[a];
                slotL[f[a]] = to;
            }
            continue;
        }
        for (int a = 1; a < m; ++a) {  // insertion sort by column
            const int64_t pa = slot(j, a);
            const int32_t c = col[pa];
            const int64_t fa = faceAt[pa];
            int b = a - 1;
            while (b >= 0 && col[slot(j, b)] > c) {
                const int64_t pb = slot(j, b), pn = slot(j, b + 1);
                col[pn] = col[pb];
                faceAt[pn] = faceAt[pb];
                --b;
            }
            const int64_t pn = slot(j, b + 1);
            col[pn] = c;
            faceAt[pn] = fa;
        }
        for (int a = 0; a < m; ++a) {
            const int64_t pa = slot(j, a);
            slotL[faceAt[pa]] = pa;
        }
    }
}

// plain slices: padding entries point at their own row with value 0
// (positions past n: row 0)
__global__ void k_fill_pad(int32_t n, int64_t S, const int64_t *sptr, const int32_t *deg,
                           int32_t *col, double *val, double *valT) {
    const int64_t rows = S * kWave;
    GRID_STRIDE(p, rows) {
        const int64_t s = p >> 6;
        const int64_t w = (sptr[s + 1] - sptr[s]) >> 6;
        const int64_t d = (p < n) ? deg[p] : 0;
        for (int64_t k = d; k < w; ++k) {
            const int64_t pos = sptr[s] + k * kWave + (p & 63);
            col[pos] = (p < n) ? (int32_t)p : 0;
            val[pos] = 0.0;
            valT[pos] = 0.0;
        }
    }
}

__global__ void k_set_values(int64_t nf, const int64_t *slotU, const int64_t *slotL,
                             const double *upper, const double *lower, double *val,
                             double *valT) {
    GRID_STRIDE(f, nf) {
        const double u = upper[f], l = lower[f];
        const int64_t pu = slotU[f], pl = slotL[f];
        val[pu] = u;
        val[pl] = l;
        valT[pu] = l;
        valT[pl] = u;
    }
}

// smallest and largest value over a wave
__device__ __forceinline__ void wave_range(int32_t &lo, int32_t &hi) {
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const int32_t a = __shfl_xor(lo, d, kWave), b = __shfl_xor(hi, d, kWave);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
}

// 16-bit columns of plain slices: the smallest column of each slot (the 64
// k-th entries of a slice) and every entry minus it.  One wave per slice, a
// lane per entry: a thread per slice walked its 64 entries serially, 64
// strided reads per wave at each step.  200^3: bases and offsets 861 ->
// 214 us, a 121 x 117 x 130 box 215 -> 51.
__global__ void __launch_bounds__(kBlock)
k_col16_bases(int64_t S, const int64_t *__restrict__ sptr, const int32_t *__restrict__ col,
              int32_t *cbase, int32_t *narrow) {
    const int lane = threadIdx.x & 63;
    bool fit = false;
    for_each_slice(S, [&](int64_t s) {
        const int64_t b0 = sptr[s], b1 = sptr[s + 1];
        for (int64_t e = b0; e < b1; e += kWave) {
            int32_t lo = col[e + lane], hi = lo;
            wave_range(lo, hi);
            const bool fits = (int64_t)hi - lo <= 65535;
            if (lane == 0) cbase[e >> 6] = fits ? lo : -1;  // -1: reads the 32-bit columns
            fit = fit || fits;
        }
    });
    if (lane == 0 && fit) *narrow = 1;  // one value from every wave
}

__global__ void __launch_bounds__(kBlock)
k_col16_fill(int64_t nnz, const int32_t *__restrict__ col, const int32_t *__restrict__ cbase,
             uint16_t *__restrict__ c16) {
    GRID_STRIDE(e, nnz) {
        const int32_t b = cbase[e >> 6];
        c16[e] = b >= 0 ? (uint16_t)(col[e] - b) : 0;
    }
}

// 16-bit columns for the slots narrow enough, on a level that has any
static void build_col16(Sell &A, int64_t nslots, Arena &ar, Arena &tmp, hipStream_t st) {
    A.c16 = nullptr;
    A.cbase = nullptr;
    // plain slices only: in compressed slices the slot bases cost more than
    // the narrower columns save (measured on the Galerkin levels)
    if (A.nnz == 0 || nslots == 0 || A.pdeg) return;
    int32_t *cbase = ar.get<int32_t>(nslots);
    int32_t *narrow = tmp.get<int32_t>(1), hnarrow = 0;
    HIP_CHECK(hipMemsetAsync(narrow, 0, sizeof(hnarrow), st));
    k_col16_bases<<<stream_grid_slices(A.nslices), kBlock, 0, st>>>(A.nslices, A.sptr, A.col, cbase,
                                                                 narrow);
    HIP_CHECK(hipMemcpyAsync(&hnarrow, narrow, sizeof(hnarrow), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    if (hnarrow == 0) return;
    uint16_t *c16 = ar.get<uint16_t>(A.nnz);
    k_col16_fill<<<grid_for(A.nnz), kBlock, 0, st>>>(A.nnz, A.col, cbase, c16);
    HIP_CHECK(hipGetLastError());
    A.c16 = c16;
    A.cbase = cbase;
}

// The aggregate map composed with plain slices' columns, agg[col], as 16-bit
// columns of the same slots (positions past the last row are not read, and do
// not widen their slot).
__global__ void __launch_bounds__(kBlock)
k_agg_columns(int64_t S, int64_t n, const int64_t *__restrict__ sptr,
              const int32_t *__restrict__ col, const int32_t *__restrict__ agg, int32_t *cbase,
              uint16_t *__restrict__ c16, int32_t *wide) {
    const int lane = threadIdx.x & 63;
    bool over = false;
    for_each_slice(S, [&](int64_t s) {
        const int64_t b0 = sptr[s], b1 = sptr[s + 1];
        const bool row = s * kWave + lane < n;
        for (int64_t e = b0; e < b1; e += kWave) {
            const int32_t c = row ? agg[col[e + lane]] : 0;
            int32_t lo = row ? c : INT32_MAX, hi = row ? c : 0;
            wave_range(lo, hi);
            const bool fits = hi - lo <= 65535;
            if (lane == 0) cbase[e >> 6] = fits ? lo : -1;
            c16[e + lane] = fits && row ? (uint16_t)(c - lo) : 0;
            over = over || !fits;
        }
    });
    if (lane == 0 && over) *wide = 1;
}

__global__ void k_agg_columns32(int64_t nnz, const int32_t *col, const int32_t *agg,
                                int32_t *out) {
    GRID_STRIDE(e, nnz)
        out[e] = agg[col[e]];
}

void aggregate_columns(Level &L, Arena &ar, Arena &tmp, hipStream_t st) {
    const Sell &A = L.A;
    L.ac32 = nullptr;
    L.ac16 = ar.get<uint16_t>(A.nnz);
    L.acbase = ar.get<int32_t>(A.nnz / kWave);
    int32_t *wide = tmp.get<int32_t>(1), hwide = 0;
    HIP_CHECK(hipMemsetAsync(wide, 0, sizeof(hwide), st));
    k_agg_columns<<<stream_grid_slices(A.nslices), kBlock, 0, st>>>(
        A.nslices, A.n, A.sptr, A.col, L.agg, L.acbase, L.ac16, wide);
    HIP_CHECK(hipMemcpyAsync(&hwide, wide, sizeof(hwide), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    if (hwide == 0) return;
    L.ac32 = ar.get<int32_t>(A.nnz);  // read by the slots that are too wide
    k_agg_columns32<<<grid_for(A.nnz), kBlock, 0, st>>>(A.nnz, A.col, L.agg, L.ac32);
    HIP_CHECK(hipGetLastError());
}

__global__ void k_to_f32(const double *a, float *b, int64_t n) {
    STREAM_STRIDE(i, n)
        b[i] = (float)a[i];
}

// slices for rows of the given lengths (nnz_rows entries in all): plain ones,
// or compressed where plain ones would pad by more than 3%
int64_t layout_rows(Sell &A, int32_t n, const int32_t *deg, int64_t nnz_rows, Arena &ar, Arena &tmp,
                    hipStream_t st) {
    const int64_t S = slices_of(n);
    int64_t *entries = tmp.get<int64_t>(S);
    A.sptr = ar.get<int64_t>(S + 1);
    k_slice_entries<<<grid_for(S), kBlock, 0, st>>>(n, S, deg, nullptr, entries);
    exclusive_scan_i64(entries, A.sptr, S, tmp, st);
    int64_t nnz = 0;
    HIP_CHECK(hipMemcpyAsync(&nnz, A.sptr + S, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    A.perm = A.iperm = A.pdeg = A.tptr = A.otab = nullptr;
    int64_t nslots = nnz / kWave;  // plain slices: one slot per 64 entries
    if (nnz * 100 > 103 * std::max<int64_t>(nnz_rows, kWave)) {
        // rows of uneven length: compressed slices, lanes ordered by length
        A.perm = ar.get<int32_t>(S * kWave);
        A.iperm = ar.get<int32_t>(n);
        A.pdeg = ar.get<int32_t>(S * kWave);
        k_slice_sort<<<grid_for(S * kWave), kBlock, 0, st>>>(n, S, deg, A.perm, A.iperm,
                                                             A.pdeg);
        int32_t *tlen = tmp.get<int32_t>(S);
        k_slice_sizes<<<grid_for(S), kBlock, 0, st>>>(S, A.pdeg, entries, tlen);
        exclusive_scan_i64(entries, A.sptr, S, tmp, st);
        A.tptr = ar.get<int32_t>(S + 1);
        scan_counts_i32(tlen, A.tptr, S, tmp, st);
        int32_t ntab = 0;
        HIP_CHECK(hipMemcpyAsync(&ntab, A.tptr + S, sizeof(int32_t), hipMemcpyDeviceToHost,
                                 st));
        HIP_CHECK(hipMemcpyAsync(&nnz, A.sptr + S, sizeof(int64_t), hipMemcpyDeviceToHost,
                                 st));
        HIP_CHECK(hipStreamSynchronize(st));
        A.otab = ar.get<int32_t>(ntab);
        nslots = ntab;
        k_slice_table<<<grid_for(S), kBlock, 0, st>>>(S, A.pdeg, A.tptr, A.otab);
    }
    A.n = n;
    A.nslices = S;
    A.nnz = nnz;
    A.col = ar.get<int32_t>(nnz);
    A.val = ar.get<double>(nnz);
    A.valT = ar.get<double>(nnz);
    return nslots;
}

void build_level_sell(ldu_t *h, Arena &ar, Level &L, bool validate, hipStream_t st) {
    const int32_t n = L.n;
    const int64_t nf = L.nf;
    const int64_t S = slices_of(n);
    Arena tmp(&ar);
    if (validate) {
        HIP_CHECK(hipMemsetAsync(h->flag, 0, sizeof(int), st));
        if (nf > 0)
            k_validate<<<grid_for(nf), kBlock, 0, st>>>(n, nf, L.own, L.nb, h->flag);
        check_finite(h, L.diag, n, st);
        check_finite(h, L.upper, nf, st);
        check_finite(h, L.lower, nf, st);
        HIP_CHECK(hipMemcpyAsync(h->hflag, h->flag, sizeof(int), hipMemcpyDeviceToHost, st));
        HIP_CHECK(hipStreamSynchronize(st));
        if (*h->hflag & 1) throw Error(LDU_ERR_ADDR, "face addressing violates 0 <= owner < neighbour < nCells, sorted by (owner, neighbour), no duplicates");
        if (*h->hflag & 2) throw Error(LDU_ERR_NAN, "non-finite coefficient");
    }
    L.ownStart = ar.get<int64_t>(n + 1);
    k_own_start<<<grid_for(n + 1), kBlock, 0, st>>>(n, nf, L.own, L.ownStart);
    int32_t *cntL = tmp.get<int32_t>(n);
    HIP_CHECK(hipMemsetAsync(cntL, 0, sizeof(int32_t) * n, st));
    if (nf > 0) k_count_lower<<<grid_for(nf), kBlock, 0, st>>>(nf, L.nb, cntL);
    int32_t *deg = tmp.get<int32_t>(n);
    k_degree<<<grid_for(n), kBlock, 0, st>>>(n, L.ownStart, cntL, deg);
    const int64_t nslots = layout_rows(L.A, n, deg, 2 * nf, ar, tmp, st);
    const int64_t nnz = L.A.nnz;
    {  // longest row, for kernels that stage a whole row
        int32_t *dmax = tmp.get<int32_t>(1);
        k_fill_i32<<<1, kBlock, 0, st>>>(dmax, 1, 0);
        k_max_i32<<<grid_for(n), kBlock, 0, st>>>(deg, n, dmax);
        HIP_CHECK(hipMemcpyAsync(&L.max_row, dmax, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        HIP_CHECK(hipStreamSynchronize(st));
    }
    L.A.diag = L.diag;
    L.slotU = ar.get<int64_t>(nf);
    L.slotL = ar.get<int64_t>(nf);
    if (nf > 0) {
        const Slots slot{L.A.sptr, L.A.iperm, L.A.tptr, L.A.otab};
        k_fill_upper<<<grid_for(nf), kBlock, 0, st>>>(nf, L.own, L.nb, L.ownStart, cntL, slot,
                                                     L.A.col, L.slotU);
        int32_t *cursor = tmp.get<int32_t>(n);
        int64_t *faceAt = tmp.get<int64_t>(nnz);
        HIP_CHECK(hipMemsetAsync(cursor, 0, sizeof(int32_t) * n, st));
        k_fill_lower<<<grid_for(nf), kBlock, 0, st>>>(nf, L.own, L.nb, slot, cursor, L.A.col,
                                                     faceAt);
        k_sort_lower<<<grid_for(n), kBlock, 0, st>>>(n, slot, cntL, L.A.col, faceAt, L.slotL);
    }
    if (!L.A.pdeg)
        k_fill_pad<<<grid_for(S * kWave), kBlock, 0, st>>>(n, S, L.A.sptr, deg, L.A.col, L.A.val,
                                                          L.A.valT);
    HIP_CHECK(hipGetLastError());
    build_col16(L.A, nslots, ar, tmp, st);
    set_level_values(L, st);
    HIP_CHECK(hipStreamSynchronize(st));  // tmp is released after this point
}

// compressed slices for n rows of the given lengths (device array): the
// lane order, slice starts and offset tables, and uninitialised col, val and
// valT arrays of the total entry count (no diagonal)
void build_sliced_rows(Sell &A, int32_t n, const int32_t *deg, Arena &ar, hipStream_t st) {
    Arena tmp(&ar);
    const int64_t S = slices_of(n);
    A = Sell{};
    A.n = n;
    A.nslices = S;
    A.perm = ar.get<int32_t>(S * kWave);
    A.iperm = ar.get<int32_t>(n);
    A.pdeg = ar.get<int32_t>(S * kWave);
    k_slice_sort<<<grid_for(S * kWave), kBlock, 0, st>>>(n, S, deg, A.perm, A.iperm, A.pdeg);
    int64_t *entries = tmp.get<int64_t>(S);
    int32_t *tlen = tmp.get<int32_t>(S);
    k_slice_sizes<<<grid_for(S), kBlock, 0, st>>>(S, A.pdeg, entries, tlen);
    A.sptr = ar.get<int64_t>(S + 1);
    exclusive_scan_i64(entries, A.sptr, S, tmp, st);
    A.tptr = ar.get<int32_t>(S + 1);
    scan_counts_i32(tlen, A.tptr, S, tmp, st);
    int32_t ntab = 0;
    int64_t nnz = 0;
    HIP_CHECK(hipMemcpyAsync(&ntab, A.tptr + S, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipMemcpyAsync(&nnz, A.sptr + S, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    A.otab = ar.get<int32_t>(ntab);
    k_slice_table<<<grid_for(S), kBlock, 0, st>>>(S, A.pdeg, A.tptr, A.otab);
    A.nnz = nnz;
    A.col = ar.get<int32_t>(nnz);
    A.val = ar.get<double>(nnz);
    A.valT = ar.get<double>(nnz);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(st));  // tmp is released after this point
}

// ---------------------------------------------------------------- renumbering
// true row lengths (without padding) in the new order
__global__ void k_rn_degree(Sell A, const int32_t *order, int32_t *deg) {
    GRID_STRIDE(p, A.n) {
        const int32_t i = order[p];
        const int64_t ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
        const int w = row_len(A, ps);
        int d = 0;
        for (int k = 0; k < w; ++k) d += A.col[entry_at(A, ps, k)] != i;
        deg[p] = d;
    }
}

// columns and sources: an entry's place in its row is the number of entries
// with a smaller new column.  A lane holds a row of at most kRnRegs stored
// entries in registers (all loads of a row together).  A longer one is shared
// by the wave, 64 entries held and compared with 64 at a time.  A lane that
// read the row again for every entry added 9 ms to the set-up for one row of 200
// entries and 40 ms for one of 400 (506,000 cells: 20 ms without renumbering);
// now 1 and 9 ms, the most of it the members of the long row's aggregate being
// sorted once more.
constexpr int kRnRegs = 24;

__global__ void __launch_bounds__(kBlock)
k_rn_fill(Sell A, const int32_t *order, const int32_t *place, Slots slot, int32_t *col,
          int32_t *src) {
    const int lane = threadIdx.x & 63;
    const GridRange gr = grid_range(A.n, kBlock);
    for (int64_t p0 = gr.begin + (threadIdx.x - lane); p0 < gr.end; p0 += gr.step) {
        const int64_t p = p0 + lane;
        int32_t i = 0;
        int64_t ps = 0;
        int w = 0;
        if (p < gr.end) {
            i = order[p];
            ps = A.iperm ? (int64_t)A.iperm[i] : (int64_t)i;
            w = row_len(A, ps);
        }
        if (w <= kRnRegs) {
            int32_t e[kRnRegs], c[kRnRegs];
#pragma unroll
            for (int k = 0; k < kRnRegs; ++k) e[k] = k < w ? (int32_t)entry_at(A, ps, k) : 0;
#pragma unroll
            for (int k = 0; k < kRnRegs; ++k) c[k] = k < w ? A.col[e[k]] : i;
#pragma unroll
            for (int k = 0; k < kRnRegs; ++k) c[k] = c[k] != i ? place[c[k]] : INT32_MAX;
#pragma unroll
            for (int k = 0; k < kRnRegs; ++k) {
                if (c[k] == INT32_MAX) continue;  // padding
                int rank = 0;
#pragma unroll
                for (int q = 0; q < kRnRegs; ++q) rank += c[q] < c[k];
                const int64_t to = slot(p, rank);
                col[to] = c[k];
                src[to] = e[k];
            }
        }
        for (uint64_t left = __ballot(w > kRnRegs); left; left &= left - 1) {
            const int from = __ffsll((unsigned long long)left) - 1;
            const int32_t ri = __shfl(i, from);
            const int64_t rps = __shfl(ps, from);
            const int rw = __shfl(w, from);
            // entry k of the row and its new column (INT32_MAX: padding or none)
            auto load = [&](int k, int32_t &e) {
                if (k >= rw) return (int32_t)INT32_MAX;
                e = (int32_t)entry_at(A, rps, k);
                const int32_t j = A.col[e];
                return j != ri ? place[j] : (int32_t)INT32_MAX;
            };
            for (int k0 = 0; k0 < rw; k0 += kWave) {
                int32_t e = 0, other = 0;
                const int32_t c = load(k0 + lane, e);
                int rank = 0;
                for (int q0 = 0; q0 < rw; q0 += kWave) {
                    const int32_t cq = q0 == k0 ? c : load(q0 + lane, other);
                    for (int u = 0; u < kWave; ++u) rank += __shfl(cq, u) < c;
                }
                if (c != INT32_MAX) {
                    const int64_t to = slot(p0 + from, rank);
                    col[to] = c;
                    src[to] = e;
                }
            }
        }
    }
}

__global__ void k_rn_values(int64_t nnz, const int32_t *__restrict__ src,
                            const double *__restrict__ val, const double *__restrict__ valT,
                            double *__restrict__ v, double *__restrict__ vT) {
    GRID_STRIDE(e, nnz) {
        const int32_t q = src[e];
        v[e] = q >= 0 ? val[q] : 0.0;
        vT[e] = q >= 0 ? valT[q] : 0.0;
    }
}

__global__ void k_gather_cells(const double *__restrict__ a, const int32_t *__restrict__ order,
                               double *__restrict__ out, int64_t n) {
    GRID_STRIDE(p, n)
        out[p] = a[order[p]];
}
__global__ void k_scatter_cells(const double *__restrict__ a, const int32_t *__restrict__ order,
                                double *__restrict__ out, int64_t n) {
    GRID_STRIDE(p, n)
        out[order[p]] = a[p];
}
void gather_cells(const double *a, const int32_t *order, double *out, int64_t n, hipStream_t st) {
    k_gather_cells<<<grid_for(n), kBlock, 0, st>>>(a, order, out, n);
    HIP_CHECK(hipGetLastError());
}
void scatter_cells(const double *a, const int32_t *order, double *out, int64_t n,
                   hipStream_t st) {
    k_scatter_cells<<<grid_for(n), kBlock, 0, st>>>(a, order, out, n);
    HIP_CHECK(hipGetLastError());
}

void renumbered_values(const Sell &A, Level &L, hipStream_t st) {
    if (L.A.nnz > 0)
        k_rn_values<<<grid_for(L.A.nnz), kBlock, 0, st>>>(L.A.nnz, L.src, A.val, A.valT, L.A.val,
                                                          L.A.valT);
    gather_cells(A.diag, L.order, L.A.diag, L.n, st);
}

void build_renumbered(const Sell &A, int64_t nf, const int32_t *order, const int32_t *place,
                      Level &L, Arena &ar, hipStream_t st) {
    Arena tmp(&ar);
    const int32_t n = A.n;
    int32_t *deg = tmp.get<int32_t>(n);
    k_rn_degree<<<grid_for(n), kBlock, 0, st>>>(A, order, deg);
    L.A = Sell{};
    const int64_t nslots = layout_rows(L.A, n, deg, 2 * nf, ar, tmp, st);
    L.diag = ar.get<double>(n);
    L.A.diag = L.diag;
    L.src = ar.get<int32_t>(L.A.nnz);
    L.order = const_cast<int32_t *>(order);
    if (L.A.nnz > 0) {
        k_fill_i32<<<grid_for(L.A.nnz), kBlock, 0, st>>>(L.src, L.A.nnz, -1);
        const Slots slot{L.A.sptr, L.A.iperm, L.A.tptr, L.A.otab};
        k_rn_fill<<<grid_for(n), kBlock, 0, st>>>(A, order, place, slot, L.A.col, L.src);
    }
    if (!L.A.pdeg)
        k_fill_pad<<<grid_for(L.A.nslices * kWave), kBlock, 0, st>>>(n, L.A.nslices, L.A.sptr, deg,
                                                                    L.A.col, L.A.val, L.A.valT);
    HIP_CHECK(hipGetLastError());
    build_col16(L.A, nslots, ar, tmp, st);
    renumbered_values(A, L, st);
    HIP_CHECK(hipStreamSynchronize(st));  // tmp is released after this point
}

// sum of |column - row| over the faces
__global__ void __launch_bounds__(kBlock)
k_face_span(int64_t nf, const int32_t *__restrict__ own, const int32_t *__restrict__ nb,
            unsigned long long *out) {
    unsigned long long s = 0;
    GRID_STRIDE(f, nf)
        s += (unsigned long long)(nb[f] - own[f]);
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(out, s);
}

// whether a face joins cells that lie more than a sixteenth of the mesh apart
// on average: a random numbering has a third, a mesh generator's or a
// Cuthill-McKee numbering a few layers, n^(2/3)
bool scattered_numbering(ldu_t *h, hipStream_t st) {
    const Level &L = h->L0;
    if (L.n < kRenumberCells || L.nf == 0) return false;
    if (L.A.nnz > INT32_MAX) return false;  // Level::src holds positions in 32 bits
    Arena tmp(&h->pool);
    unsigned long long *sum = tmp.get<unsigned long long>(1), host = 0;
    k_fill_i32<<<1, kBlock, 0, st>>>(reinterpret_cast<int32_t *>(sum), 2, 0);
    k_face_span<<<std::min(grid_for(L.nf), 2048u), kBlock, 0, st>>>(L.nf, L.own, L.nb, sum);
    HIP_CHECK(hipMemcpyAsync(&host, sum, sizeof(host), hipMemcpyDeviceToHost, st));
    HIP_CHECK(hipStreamSynchronize(st));
    return (double)host > (double)L.nf * (double)L.n / 16.0;
}

void set_level_values(Level &L, hipStream_t st) {
    if (L.nf > 0)
        k_set_values<<<grid_for(L.nf), kBlock, 0, st>>>(L.nf, L.slotU, L.slotL, L.upper,
                                                        L.lower, L.A.val, L.A.valT);
    HIP_CHECK(hipGetLastError());
}

void refresh_f32(Level &L, hipStream_t st) {
    if (!L.A.val32) return;
    k_to_f32<<<grid_for(L.A.nnz), kBlock, 0, st>>>(L.A.val, L.A.val32, L.A.nnz);
    k_to_f32<<<grid_for(L.A.nnz), kBlock, 0, st>>>(L.A.valT, L.A.valT32, L.A.nnz);
    k_to_f32<<<grid_for(L.n), kBlock, 0, st>>>(L.diag, L.A.diag32, L.n);
    HIP_CHECK(hipGetLastError());
}

// `own`: arrays of their own.  A single matrix asks for these three alone, and
// a chunk sized by what the handle holds takes longer than they do: the first
// FP32 product on 69,120 cells 350 us from a chunk, 40 us from arrays.
void ensure_f32(Level &L, Arena &ar, bool own, hipStream_t st) {
    if (L.A.val32) return;
    auto floats = [&](int64_t n) {
        return own ? static_cast<float *>(ar.alloc_own(sizeof(float) * (size_t)n))
                   : ar.get<float>(n);
    };
    float *v = floats(L.A.nnz), *vT = floats(L.A.nnz);
    L.A.diag32 = floats(L.n);
    L.A.val32 = v;
    L.A.valT32 = vT;
    refresh_f32(L, st);
}

}  // namespace ldu
