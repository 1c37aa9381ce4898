// Setup of a dpcg handle on the GPU: every factorisation the iteration applies.
//
//   validation   CSR structure of K and Z, block partition, symmetry of K
//   block-CSR    K packed into 3x3 blocks (nine value planes)
//   block-Jacobi Cholesky and explicit inverse of each block (one wave per block)
//   Z^T          transpose of Z with rows ascending in every column
//   K Z, E       per deflation vector j: K z_j on a dense window of rows (deterministic
//                gather, no atomics on values), E[j, :] = (K z_j)^T Z
//   E^-1         block Gauss-Jordan sweeps (32 x 32 pivots), SPD check on every pivot
// All sums run in a fixed order, so a setup is bitwise reproducible.
#include <algorithm>
#include <cfloat>
#include <vector>

#include "dpcg_internal.h"

namespace dpcg {

namespace {

constexpr int kTileDofs = 239;   // block-Jacobi tile window: tiles hold <= 239 + 17 = 256 DoFs

// ---------------------------------------------------------------- small helpers
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t *lds, int64_t &total) {
    // 256 threads; lds >= 4 entries.  Returns the exclusive prefix of v, total = sum.
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int64_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    __syncthreads();
    if (lane == 63) lds[wv] = x;
    __syncthreads();
    int64_t base = 0;
    for (int w = 0; w < wv; ++w) base += lds[w];
    total = lds[0] + lds[1] + lds[2] + lds[3];
    return base + x - v;
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ double bsum(double v, double *lds) {
    v = wsum(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// ---------------------------------------------------------------- scans (int64)
constexpr int kScanChunk = 2048;

__global__ __launch_bounds__(256) void k_scan_partials(const int64_t *__restrict__ a, int64_t n,
                                                       int64_t *__restrict__ part) {
    __shared__ int64_t l64[4];
    const int64_t b = (int64_t)blockIdx.x * kScanChunk;
    int64_t s = 0;
    for (int i = threadIdx.x; i < kScanChunk; i += 256)
        if (b + i < n) s += a[b + i];
    int64_t tot;
    block_exclusive_scan(s, l64, tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_scan_top(int64_t *part, int m) {
    __shared__ int64_t l64[4];
    int64_t carry = 0;
    for (int c = 0; c < m; c += 256) {
        const int i = c + threadIdx.x;
        const int64_t v = i < m ? part[i] : 0;
        int64_t tot;
        const int64_t ex = block_exclusive_scan(v, l64, tot);
        if (i < m) part[i] = carry + ex;
        carry += tot;
        __syncthreads();
    }
}

// out[i] = exclusive prefix of a (out has n+1 entries; out[n] = total).
__global__ __launch_bounds__(256) void k_scan_apply(const int64_t *__restrict__ a, int64_t n,
                                                    const int64_t *__restrict__ part, int64_t *__restrict__ out) {
    __shared__ int64_t l64[4];
    const int64_t b = (int64_t)blockIdx.x * kScanChunk;
    int64_t carry = part[blockIdx.x];
    for (int c = 0; c < kScanChunk; c += 256) {
        const int64_t i = b + c + threadIdx.x;
        const int64_t v = i < n ? a[i] : 0;
        int64_t tot;
        const int64_t ex = block_exclusive_scan(v, l64, tot);
        if (i < n) out[i] = carry + ex;
        if (i == n - 1) out[n] = carry + ex + v;
        carry += tot;
        __syncthreads();
    }
}

__global__ void k_to_i32(const int64_t *__restrict__ a, int64_t n, int32_t *__restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (int32_t)a[i];
}

// ---------------------------------------------------------------- validation
// flags[0]: first invalid row of K (or INT_MAX), flags[1]: first invalid row of Z,
// flags[2]: first invalid block, flags[3]: first asymmetric row.
// Checks of a CSR matrix: row pointer monotone and in range, columns strictly increasing
// and in range, values finite.  Pass 1 (one thread per
// row): the row pointer, and a bit at each nonempty row's first entry.  Pass 2 (one
// thread per entry): column in range, value finite, and, unless the next entry opens a
// row, a larger column in the next entry; the failing row is found by bisection of the
// row pointer.  Optionally the per-workgroup maxima of |value| (for the symmetry
// tolerance) go to mxpart.
__global__ __launch_bounds__(256) void k_csr_rows(int64_t rows, const int64_t *__restrict__ ptr, int64_t nnz,
                                                  uint32_t *bits, int *flag) {
    for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256) {
        const int64_t a = ptr[i], b = ptr[i + 1];
        const bool ok = (i != 0 || a == 0) && a >= 0 && a <= b && b <= nnz;
        if (!ok) atomicMin(flag, (int)i);
        else if (a < b) atomicOr(&bits[a >> 5], 1u << (a & 31));
    }
}

__global__ __launch_bounds__(256) void k_csr_entries(int64_t rows, int64_t cols, const int64_t *__restrict__ ptr,
                                                     const int32_t *__restrict__ idx,
                                                     const double *__restrict__ val, int64_t nnz,
                                                     const uint32_t *__restrict__ bits, int *flag,
                                                     double *__restrict__ mxpart) {
    __shared__ double lds[4];
    double mx = 0.0;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * 256) {
        const int64_t c = idx[e];
        const double v = val[e];
        bool bad = c < 0 || c >= cols || !isfinite(v);
        const int64_t n1 = e + 1;
        if (n1 < nnz && !((bits[n1 >> 5] >> (n1 & 31)) & 1u) && idx[n1] <= c) bad = true;
        mx = fmax(mx, fabs(v));
        if (bad) {
            int64_t lo = 0, hi = rows;  // last row with ptr <= e
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (ptr[mid] <= e) lo = mid;
                else hi = mid;
            }
            atomicMin(flag, (int)lo);
        }
    }
    if (!mxpart) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) mxpart[blockIdx.x] = fmax(fmax(lds[0], lds[1]), fmax(lds[2], lds[3]));
}

// flag = first invalid block; maxsize = size of the largest block
__global__ void k_check_blocks(int32_t nblocks, const int32_t *__restrict__ bp, int64_t n, int *flag, int *maxsize) {
    int big = 0;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nblocks; b += gridDim.x * blockDim.x) {
        const int64_t s = bp[b], e = bp[b + 1];
        bool ok = (b != 0 || s == 0) && (b != nblocks - 1 || e == n) && e - s >= 1 && e - s <= kMaxDense;
        if (!ok) atomicMin(flag, b);
        else big = max(big, (int)(e - s));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) big = max(big, __shfl_xor(big, off));
    if ((threadIdx.x & 63) == 0 && big > kMaxBlock) atomicMax(maxsize, big);
}

// part[0] = max over part[0..m): one workgroup, fixed order
__global__ __launch_bounds__(256) void k_max_reduce(double *part, int m) {
    __shared__ double lds[4];
    double x = 0.0;
    for (int i = threadIdx.x; i < m; i += 256) x = fmax(x, part[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off));
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) part[0] = fmax(fmax(lds[0], lds[1]), fmax(lds[2], lds[3]));
}

// |K_ij - K_ji| <= 1e-12 max|K| over the packed 3x3 blocks, one thread per block (R, C)
// with R = brow[b].  A diagonal block is compared with its own transpose; block (R, C),
// C > R, with the transpose of block (C, R), found by binary search in block row C (a
// missing block counts as 0).  Blocks below the diagonal are only counted: when their
// number equals the number of upper blocks whose mirror was found, every lower block is
// such a mirror and has been compared; otherwise k_check_sym_lower compares the
// unpaired ones with 0.  part[2 w], part[2 w + 1]: lower blocks, found mirrors of
// workgroup w.
__device__ __forceinline__ int64_t find_block(const int32_t *__restrict__ bcol, int64_t l, int64_t h, int32_t col) {
    while (l < h) {
        const int64_t mid = (l + h) >> 1;
        if (bcol[mid] < col) l = mid + 1;
        else h = mid;
    }
    return l;
}

__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t *lds4) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
    __syncthreads();
    return (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
}

__global__ __launch_bounds__(256) void k_check_sym(const int32_t *__restrict__ bptr, const int32_t *__restrict__ brow,
                                                   const int32_t *__restrict__ bcol, const double *__restrict__ bval,
                                                   int64_t nnzb, const double *__restrict__ maxpart, int nmax, int *flag,
                                                   int64_t *__restrict__ part) {
    __shared__ int64_t lds4[4];
    double mx = 0.0;
    for (int i = 0; i < nmax; ++i) mx = fmax(mx, maxpart[i]);
    const double tol = 1e-12 * mx;
    int64_t lower = 0, found_n = 0;
    // a contiguous range of blocks per workgroup, runs of neighbouring ranges per XCD:
    // the mirrors of neighbouring rows sit side by side in the same block rows, so they
    // share the XCD's L2 lines
    const int64_t per = ((nnzb + gridDim.x - 1) / gridDim.x + 255) / 256 * 256;
    const int64_t b0 = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * per, b1 = min(nnzb, b0 + per);
    for (int64_t b = b0 + threadIdx.x; b < b1; b += 256) {
        const int32_t R = brow[b], C = bcol[b];
        if (C < R) {
            ++lower;
            continue;
        }
        const int64_t bR = bptr[R], mR = bptr[R + 1] - bR;
        double v[9];
        for (int e = 0; e < 9; ++e) v[e] = bval[9 * bR + (int64_t)e * mR + (b - bR)];
        bool ok = true;
        if (C == R) {
            for (int i = 0; i < 3; ++i)
                for (int j = i + 1; j < 3; ++j) ok = ok && fabs(v[3 * i + j] - v[3 * j + i]) <= tol;
        } else {
            const int64_t bC = bptr[C], mC = bptr[C + 1] - bC;
            const int64_t l = find_block(bcol, bC, bC + mC, R);
            const bool found = l < bC + mC && bcol[l] == R;
            found_n += found;
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) {
                    const double m = found ? bval[9 * bC + (int64_t)(3 * j + i) * mC + (l - bC)] : 0.0;
                    ok = ok && fabs(v[3 * i + j] - m) <= tol;
                }
        }
        if (!ok) atomicMin(flag + 3, 3 * R);
    }
    lower = block_sum(lower, lds4);
    __syncthreads();
    found_n = block_sum(found_n, lds4);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = lower;
        part[2 * blockIdx.x + 1] = found_n;
    }
}

// need[0] = 1 when some block below the diagonal has no mirror above it
__global__ __launch_bounds__(256) void k_sym_reduce(const int64_t *__restrict__ part, int nwg, int *need) {
    __shared__ int64_t lds4[4];
    int64_t d = 0;
    for (int w = threadIdx.x; w < nwg; w += 256) d += part[2 * w] - part[2 * w + 1];
    d = block_sum(d, lds4);
    if (threadIdx.x == 0) need[0] = d != 0;
}

__global__ __launch_bounds__(256) void k_check_sym_lower(const int32_t *__restrict__ bptr,
                                                         const int32_t *__restrict__ brow,
                                                         const int32_t *__restrict__ bcol,
                                                         const double *__restrict__ bval, int64_t nnzb,
                                                         const double *__restrict__ maxpart, int nmax, int *flag,
                                                         const int *__restrict__ need) {
    if (!need[0]) return;
    double mx = 0.0;
    for (int i = 0; i < nmax; ++i) mx = fmax(mx, maxpart[i]);
    const double tol = 1e-12 * mx;
    for (int64_t b = blockIdx.x * 256ll + threadIdx.x; b < nnzb; b += (int64_t)gridDim.x * 256) {
        const int32_t R = brow[b], C = bcol[b];
        if (C >= R) continue;
        const int64_t bC = bptr[C], mC = bptr[C + 1] - bC;
        const int64_t l = find_block(bcol, bC, bC + mC, R);
        if (l < bC + mC && bcol[l] == R) continue;
        const int64_t bR = bptr[R], mR = bptr[R + 1] - bR;
        bool ok = true;
        for (int e = 0; e < 9; ++e) ok = ok && fabs(bval[9 * bR + (int64_t)e * mR + (b - bR)]) <= tol;
        if (!ok) atomicMin(flag + 3, 3 * R);
    }
}

// ---------------------------------------------------------------- block-CSR over DoF triplets
// Block columns of block row R: the union of col/3 over scalar rows 3R..3R+2.  One
// wave per block row.  When the three rows have the same set of block columns (a K
// assembled from 3x3 nodal blocks always does), a block's position is the rank of its
// block column among the row's distinct block columns, found with ballots; otherwise
// lane 0 merges the three rows.
constexpr int kMaxDistinct = 256;

__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// distinct block columns of one scalar row, ranks from ballots; returns the count
__device__ int row_distinct(int64_t a, int64_t e, const int32_t *__restrict__ idx, int32_t *dcol) {
    const int lane = threadIdx.x & 63;
    int count = 0;
    for (int64_t base = a; base < e; base += 64) {
        const int64_t p = base + lane;
        const bool in = p < e;
        const int32_t c = in ? idx[p] / 3 : -1;
        const bool first = in && (p == a || idx[p - 1] / 3 != c);
        const unsigned long long bal = __ballot(first);
        const int rank = count + __popcll(bal & ((1ull << lane) - 1ull));
        if (first && rank < kMaxDistinct) dcol[rank] = c;
        count += __popcll(bal);
    }
    return count;
}

// Block-CSR of K, one wave per block row R (its scalar rows 3R, 3R+1, 3R+2).  FILL false:
// the number of distinct block columns; FILL true: block columns, block rows and the nine
// value planes.  Rows of at most 128 entries each (nearly all) are read once, all three
// rows' loads in one round, and ranked from registers with ballots; longer rows are ranked
// chunk by chunk from memory.  Rows whose three scalar rows do not share one block-column
// set take the serial merge of lane 0.
template <bool FILL>
__global__ __launch_bounds__(256) void k_bsr(int32_t nb, const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                             const double *__restrict__ val, int64_t *__restrict__ cnt,
                                             const int32_t *__restrict__ bptr, int32_t *__restrict__ bcol,
                                             double *__restrict__ bval, int32_t *__restrict__ brow) {
    __shared__ int32_t dcol_s[4][3][kMaxDistinct];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int64_t R = blockIdx.x * 4ll + wv; R < nb; R += (int64_t)gridDim.x * 4) {
        int64_t a[3], e[3];
        for (int i = 0; i < 3; ++i) {
            a[i] = ptr[3 * R + i];
            e[i] = ptr[3 * R + i + 1];
        }
        const bool small = e[0] - a[0] <= 128 && e[1] - a[1] <= 128 && e[2] - a[2] <= 128;
        int dn[3];
        unsigned long long bal[3][2] = {{0ull, 0ull}, {0ull, 0ull}, {0ull, 0ull}};
        double cv[3][2] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
        int32_t ci[3][2];
        if (small) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int64_t p = a[i] + 64 * c + lane;
                    const bool in = p < e[i];
                    ci[i][c] = in ? idx[p] : -3;
                    if (FILL) cv[i][c] = in ? val[p] : 0.0;
                }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                int count = 0;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int32_t cur = ci[i][c];
                    // the previous entry of the row: lane - 1 of this chunk, or lane 63 of the last
                    int32_t prev = __shfl_up(cur, 1);
                    const int32_t last = __shfl(ci[i][0], 63);
                    if (lane == 0) prev = c == 0 ? -3 : last;
                    const bool in = a[i] + 64 * c + lane < e[i];
                    const bool first = in && (prev < 0 || prev / 3 != cur / 3);
                    bal[i][c] = __ballot(first);
                    const int rank = count + __popcll(bal[i][c] & below);
                    if (first && rank < kMaxDistinct) dcol_s[wv][i][rank] = cur / 3;
                    count += __popcll(bal[i][c]);
                }
                dn[i] = count;
            }
        } else {
            for (int i = 0; i < 3; ++i) dn[i] = row_distinct(a[i], e[i], idx, dcol_s[wv][i]);
        }
        wave_sync();
        bool same = dn[0] == dn[1] && dn[1] == dn[2] && dn[0] <= kMaxDistinct;
        if (same)
            for (int t = lane; t < dn[0]; t += 64)
                if (dcol_s[wv][0][t] != dcol_s[wv][1][t] || dcol_s[wv][0][t] != dcol_s[wv][2][t]) same = false;
        same = __ballot(!same) == 0ull;
        if (same) {
            if (!FILL) {
                if (lane == 0) cnt[R] = dn[0];
            } else {
                const int64_t beg = bptr[R], m = dn[0];
                for (int t = lane; t < m; t += 64) {
                    bcol[beg + t] = dcol_s[wv][0][t];
                    brow[beg + t] = (int32_t)R;
                }
                if (small) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        int count = 0;
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            // rank of the entry's block column: first entries up to and including it, minus 1
                            const int rank = count + __popcll(bal[i][c] & (below | (1ull << lane))) - 1;
                            if (a[i] + 64 * c + lane < e[i])
                                bval[9 * beg + (int64_t)(3 * i + ci[i][c] % 3) * m + rank] = cv[i][c];
                            count += __popcll(bal[i][c]);
                        }
                    }
                } else {
                    for (int i = 0; i < 3; ++i) {
                        int count = 0;
                        for (int64_t base = a[i]; base < e[i]; base += 64) {
                            const int64_t p = base + lane;
                            const bool in = p < e[i];
                            const int32_t c = in ? idx[p] : 0;
                            const bool first = in && (p == a[i] || idx[p - 1] / 3 != c / 3);
                            const unsigned long long bl = __ballot(first);
                            const int rank = count + __popcll(bl & ((2ull << lane) - 1ull)) - 1;
                            if (in) bval[9 * beg + (int64_t)(3 * i + c % 3) * m + rank] = val[p];
                            count += __popcll(bl);
                        }
                    }
                }
            }
        } else if (lane == 0) {
            int64_t h[3] = {a[0], a[1], a[2]};
            const int64_t beg = FILL ? bptr[R] : 0, m = FILL ? (int64_t)bptr[R + 1] - bptr[R] : 0;
            int64_t pos = beg, count = 0;
            while (true) {
                int32_t cur = INT32_MAX;
                for (int i = 0; i < 3; ++i)
                    if (h[i] < e[i]) cur = min(cur, idx[h[i]] / 3);
                if (cur == INT32_MAX) break;
                if (FILL) {
                    bcol[pos] = cur;
                    brow[pos] = (int32_t)R;
                }
                for (int i = 0; i < 3; ++i)
                    while (h[i] < e[i] && idx[h[i]] / 3 == cur) {
                        if (FILL) bval[9 * beg + (int64_t)(3 * i + idx[h[i]] % 3) * m + (pos - beg)] = val[h[i]];
                        ++h[i];
                    }
                ++pos;
                ++count;
            }
            if (!FILL) cnt[R] = count;
        }
        wave_sync();
    }
}

// ---------------------------------------------------------------- block-Jacobi
__global__ void k_block_sq(int32_t nblocks, const int32_t *__restrict__ bp, int64_t *__restrict__ sq) {
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nblocks; b += gridDim.x * blockDim.x) {
        const int64_t m = bp[b + 1] - bp[b];
        sq[b] = m <= kMaxBlock ? m * m : 0;  // larger blocks keep dense inverses of their own
    }
}

// Block-Jacobi inverses: Cholesky with the pivot test m * DBL_EPSILON * |original
// diagonal entry|, then the explicit inverse L^-T L^-1, in the operation order of a
// sequential column algorithm.  Blocks of up to kSmallBlock DoFs take one thread each
// (register arrays, every index a compile-time constant); larger blocks one wave each.
constexpr int kSmallBlock = 6;

// list (may be null): factorise only the nlist blocks list[0..nlist) instead of all.
__global__ __launch_bounds__(256) void k_bj_small(int32_t nblocks, const int32_t *__restrict__ bp,
                                                  const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                                  const double *__restrict__ val, const int64_t *__restrict__ moff,
                                                  double *__restrict__ minv, int32_t *__restrict__ rowoff,
                                                  int32_t *__restrict__ meta, int *bad_block,
                                                  const int32_t *__restrict__ list, int32_t nlist) {
    constexpr int M = kSmallBlock;
    const int count = list ? nlist : nblocks;
    for (int ib = blockIdx.x * blockDim.x + threadIdx.x; ib < count; ib += gridDim.x * blockDim.x) {
        const int b = list ? list[ib] : ib;
        const int32_t s = bp[b];
        const int m = bp[b + 1] - s;
        if (m > M) continue;
        double A[M][M], Li[M][M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
#pragma unroll
            for (int j = 0; j < M; ++j) A[i][j] = 0.0;
            if (i < m) {
                // first entry of the row with column >= s (columns are sorted)
                int64_t lo = ptr[s + i], hi = ptr[s + i + 1];
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (idx[mid] < s) lo = mid + 1;
                    else hi = mid;
                }
                const int64_t end = ptr[s + i + 1];
#pragma unroll
                for (int j = 0; j < M; ++j)
                    if (j < m && lo < end && idx[lo] == s + j) {
                        A[i][j] = val[lo];
                        ++lo;
                    }
            }
        }
        bool ok = true;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            if (j >= m) continue;
            double d = A[j][j];
            const double fl = m * DBL_EPSILON * fabs(d);
#pragma unroll
            for (int p = 0; p < j; ++p) d -= A[j][p] * A[j][p];
            if (!(d > fl) || !isfinite(d)) ok = false;
            const double l = sqrt(d > 0.0 ? d : 1.0);
            A[j][j] = l;
#pragma unroll
            for (int i = j + 1; i < M; ++i) {
                if (i >= m) continue;
                double sacc = A[i][j];
#pragma unroll
                for (int p = 0; p < j; ++p) sacc -= A[i][p] * A[j][p];
                A[i][j] = sacc / l;
            }
        }
        if (!ok) {
            atomicMin(bad_block, b);
            continue;
        }
#pragma unroll
        for (int j = 0; j < M; ++j)
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if (i < j || i >= m || j >= m) {
                    Li[i][j] = 0.0;
                    continue;
                }
                double sacc = (i == j) ? 1.0 : 0.0;
#pragma unroll
                for (int p = j; p < i; ++p) sacc -= A[i][p] * Li[p][j];
                Li[i][j] = sacc / A[i][i];
            }
        double *out = minv + moff[b];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if (i >= m) continue;
#pragma unroll
            for (int j = i; j < M; ++j) {
                if (j >= m) continue;
                double sacc = 0.0;
#pragma unroll
                for (int p = j; p < M; ++p)
                    if (p < m) sacc += Li[p][i] * Li[p][j];
                out[i * m + j] = sacc;
                out[j * m + i] = sacc;
            }
            rowoff[s + i] = (int32_t)(moff[b] + (int64_t)i * m);
            meta[s + i] = (m << 8) | i;
        }
    }
}

__global__ __launch_bounds__(64) void k_bj_factor(int32_t nblocks, const int32_t *__restrict__ bp,
                                                  const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                                  const double *__restrict__ val, const int64_t *__restrict__ moff,
                                                  double *__restrict__ minv, int32_t *__restrict__ rowoff,
                                                  int32_t *__restrict__ meta, int *bad_block,
                                                  const int32_t *__restrict__ list, int32_t nlist) {
    __shared__ double A[kMaxBlock * kMaxBlock];
    __shared__ double Li[kMaxBlock * kMaxBlock];
    __shared__ int fail;
    const int lane = threadIdx.x;
    const int count = list ? nlist : nblocks;
    for (int ib = blockIdx.x; ib < count; ib += gridDim.x) {
        const int b = list ? list[ib] : ib;
        const int32_t s = bp[b];
        const int m = bp[b + 1] - s;
        if (m <= kSmallBlock || m > kMaxBlock) continue;
        __syncthreads();
        for (int t = lane; t < m * m; t += 64) A[t] = 0.0;
        if (lane == 0) fail = 0;
        __syncthreads();
        if (lane < m) {
            // the row's entries in columns [s, s + m) follow its first column >= s
            int64_t lo = ptr[s + lane], hi = ptr[s + lane + 1];
            const int64_t end = hi;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (idx[mid] < s) lo = mid + 1;
                else hi = mid;
            }
#pragma unroll
            for (int q = 0; q < kMaxBlock; ++q) {
                const int64_t e = lo + q;
                if (q < m && e < end) {
                    const int32_t c = idx[e];
                    if (c < s + m) A[lane * m + (c - s)] = val[e];
                }
            }
        }
        __syncthreads();
        for (int j = 0; j < m; ++j) {
            if (lane == 0) {
                double d = A[j * m + j];
                const double fl = m * DBL_EPSILON * fabs(d);
                for (int p = 0; p < j; ++p) d -= A[j * m + p] * A[j * m + p];
                if (!(d > fl) || !isfinite(d)) fail = 1;
                else A[j * m + j] = sqrt(d);
            }
            __syncthreads();
            if (fail) break;
            const double l = A[j * m + j];
            if (lane > j && lane < m) {
                double sacc = A[lane * m + j];
                for (int p = 0; p < j; ++p) sacc -= A[lane * m + p] * A[j * m + p];
                A[lane * m + j] = sacc / l;
            }
            __syncthreads();
        }
        if (fail) {
            if (lane == 0) atomicMin(bad_block, b);
            continue;
        }
        // column j of L^-1 (lane j), rows i >= j
        if (lane < m) {
            const int j = lane;
            for (int i = 0; i < m; ++i) {
                if (i < j) {
                    Li[i * m + j] = 0.0;
                    continue;
                }
                double sacc = (i == j) ? 1.0 : 0.0;
                for (int p = j; p < i; ++p) sacc -= A[i * m + p] * Li[p * m + j];
                Li[i * m + j] = sacc / A[i * m + i];
            }
        }
        __syncthreads();
        double *out = minv + moff[b];
        if (lane < m) {
            const int i = lane;
            for (int j = i; j < m; ++j) {
                double sacc = 0.0;
                for (int p = j; p < m; ++p) sacc += Li[p * m + i] * Li[p * m + j];
                out[i * m + j] = sacc;
                out[j * m + i] = sacc;
            }
            rowoff[s + i] = (int32_t)(moff[b] + (int64_t)i * m);
            meta[s + i] = (m << 8) | i;
        }
    }
}

// tile t = blocks starting in [t * window, (t+1) * window); start = first such block,
// or t * window itself when that DoF lies inside a block of more than kMaxBlock DoFs
// (their rows need no neighbours in the tile), so a tile holds < window + kMaxBlock DoFs.
// One thread per block b <= nblocks (bp[nblocks] = n): the targets t * window in
// (bp[b-1], bp[b]] have b as their first block starting at or after the target, so b
// writes those tiles (usually none or one) and no thread searches.
__global__ void k_tiles(int32_t ntiles, int32_t nblocks, const int32_t *__restrict__ bp, int64_t n,
                        int32_t window, int32_t *__restrict__ tile_start) {
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b <= nblocks; b += gridDim.x * blockDim.x) {
        const int64_t hi = bp[b];
        const int64_t t0 = b == 0 ? 0 : (int64_t)bp[b - 1] / window + 1;
        const int64_t t1 = min<int64_t>(ntiles - 1, hi / window);
        const bool split = b > 0 && hi - bp[b - 1] > kMaxBlock;  // the target lies inside block b - 1
        for (int64_t t = t0; t <= t1; ++t) tile_start[t] = split ? (int32_t)(t * window) : (int32_t)hi;
        if (b == nblocks) tile_start[ntiles] = (int32_t)n;
    }
}

// Block columns as offsets from their block row in 16 bits (the iteration SpMV reads 2
// bytes per block instead of 4); *bad becomes 1 when an offset does not fit.
__global__ void k_bcol16(int64_t nnzb, const int32_t *__restrict__ brow, const int32_t *__restrict__ bcol,
                         int16_t *__restrict__ out, int *bad) {
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < nnzb; b += (int64_t)gridDim.x * blockDim.x) {
        const int32_t d = bcol[b] - brow[b];
        const bool fits = d >= INT16_MIN && d <= INT16_MAX;
        out[b] = fits ? (int16_t)d : (int16_t)0;
        if (!fits) *bad = 1;
    }
}

// *longest (0 on entry) becomes the largest number of blocks in a row.
__global__ __launch_bounds__(256) void k_longest_row(int32_t nb, const int32_t *__restrict__ ptr, int *longest) {
    __shared__ int ms[4];
    int m = 0;
    for (int r = blockIdx.x * 256 + threadIdx.x; r < nb; r += gridDim.x * 256) m = max(m, ptr[r + 1] - ptr[r]);
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) ms[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(longest, max(max(ms[0], ms[1]), max(ms[2], ms[3])));
}

// ---------------------------------------------------------------- Z^T
// Z^T by a stable counting sort over chunks of Z's entries in row-major order.  Pass 1
// counts each chunk's entries per column into cnt[c * nch + w]; an exclusive scan in
// (column, chunk) order gives every (column, chunk) pair its first slot; pass 2 walks a
// chunk's entries in order with one wave and places them, so every column of Z^T lists
// its rows in increasing order without atomics on global memory.  Columns go in ranges
// of kZtCols (LDS tables), one grid row per range.
constexpr int kZtCols = 8192;

__global__ void k_entry_rows(int64_t rows, const int64_t *__restrict__ ptr, int32_t *__restrict__ erow) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < rows; r += (int64_t)gridDim.x * blockDim.x)
        for (int64_t e = ptr[r]; e < ptr[r + 1]; ++e) erow[e] = (int32_t)r;
}

__global__ __launch_bounds__(256) void k_zt_count(int64_t nnz, int64_t per, int nch, int32_t k,
                                                  const int32_t *__restrict__ idx, int64_t *__restrict__ cnt) {
    extern __shared__ int32_t hist[];
    const int w = blockIdx.x;
    const int32_t c0 = blockIdx.y * kZtCols, nc = min(kZtCols, k - c0);
    for (int t = threadIdx.x; t < nc; t += 256) hist[t] = 0;
    __syncthreads();
    const int64_t e0 = (int64_t)w * per, e1 = min(nnz, e0 + per);
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
        const int32_t c = idx[e] - c0;
        if (c >= 0 && c < nc) atomicAdd(&hist[c], 1);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nc; t += 256) cnt[(int64_t)(c0 + t) * nch + w] = hist[t];
}

__global__ void k_zt_ptr(int32_t k, int nch, const int64_t *__restrict__ off, int64_t *__restrict__ ztp) {
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c <= k; c += (int64_t)gridDim.x * blockDim.x)
        ztp[c] = off[c * nch];
}

__global__ __launch_bounds__(64) void k_zt_place(int64_t nnz, int64_t per, int nch, int32_t k,
                                                 const int32_t *__restrict__ idx, const double *__restrict__ val,
                                                 const int32_t *__restrict__ erow, const int64_t *__restrict__ off,
                                                 int32_t *__restrict__ zti, double *__restrict__ ztv) {
    extern __shared__ int64_t run[];
    const int w = blockIdx.x, lane = threadIdx.x;
    const int32_t c0 = blockIdx.y * kZtCols, nc = min(kZtCols, k - c0);
    for (int t = lane; t < nc; t += 64) run[t] = off[(int64_t)(c0 + t) * nch + w];
    __syncthreads();
    const int64_t e0 = (int64_t)w * per, e1 = min(nnz, e0 + per);
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int64_t base = e0; base < e1; base += 64) {
        const int64_t e = base + lane;
        const int32_t c = e < e1 ? idx[e] - c0 : -1;
        const bool mine = c >= 0 && c < nc;
        unsigned long long todo = __ballot(mine);
        // one distinct column per step: its lanes take consecutive slots in lane order
        while (todo) {
            const int leader = __builtin_ctzll(todo);
            const int32_t cl = __shfl(c, leader);
            const unsigned long long grp = __ballot(mine && c == cl);
            const int64_t b = run[cl];
            if (mine && c == cl) {
                const int64_t q = b + __popcll(grp & lt);
                zti[q] = erow[e];
                ztv[q] = val[e];
            }
            if (lane == leader) run[cl] = b + __popcll(grp);
            todo &= ~grp;
        }
    }
}

// ---------------------------------------------------------------- K Z and E
// Row window of K z_j: [first column of K over the rows of z_j, last column].
__global__ __launch_bounds__(256) void k_kz_window(int32_t k, const int64_t *__restrict__ ztp,
                                                   const int32_t *__restrict__ zti, const int64_t *__restrict__ kp,
                                                   const int32_t *__restrict__ kc, int64_t *__restrict__ wlo,
                                                   int64_t *__restrict__ wsize) {
    __shared__ int64_t lo_s[4], hi_s[4];
    const int j = blockIdx.x;
    if (j >= k) return;
    int64_t lo = INT64_MAX, hi = -1;
    for (int64_t e = ztp[j] + threadIdx.x; e < ztp[j + 1]; e += 256) {
        const int64_t r = zti[e];
        if (kp[r + 1] > kp[r]) {
            lo = min<int64_t>(lo, kc[kp[r]]);
            hi = max<int64_t>(hi, kc[kp[r + 1] - 1]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min<int64_t>(lo, __shfl_xor(lo, off));
        hi = max<int64_t>(hi, __shfl_xor(hi, off));
    }
    if ((threadIdx.x & 63) == 0) {
        lo_s[threadIdx.x >> 6] = lo;
        hi_s[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        lo = min(min(lo_s[0], lo_s[1]), min(lo_s[2], lo_s[3]));
        hi = max(max(hi_s[0], hi_s[1]), max(hi_s[2], hi_s[3]));
        wlo[j] = hi >= lo ? lo : 0;
        wsize[j] = hi >= lo ? hi - lo + 1 : 0;
    }
}

// ---- K Z and E in batches of kBatch consecutive deflation vectors ----
// A batch owns the union window of its vectors' rows in whole DoF triplets
// [lo3, lo3 + w3).  Per scalar row t of the window (t = row - 3 lo3): zd[t][b] =
// Z[row, j0+b] and kd[t][b] = (K z_{j0+b})_row.  Per triplet T: rb[T] = vectors with a
// nonzero in triplet lo3 + T, mk[T] = vectors whose K z_j has that triplet in its block
// structure (coupled by a 3x3 block of K to a triplet of z_j).  K z_j is evaluated on
// the packed 3x3 blocks; a structure triplet contributes its three rows.  Windows are
// processed in slices of kSlice triplets, one workgroup per (slice, batch).
constexpr int kBatch = 16;
constexpr int kSlice = 1024;
constexpr int kTouchLds = 2048;  // LDS words of the touched-vector bitmap (k <= 65536)

// K z_j is zero on most of its structure: a rigid-body mode stores no energy in an element
// all of whose nodes move with it, so inside the subdomain (and for the enriched modes inside
// their supports) only the rounding of the sum is left.  (KZ)^T keeps a triplet of a run of
// vectors with the same structure (the modes of one subdomain) where one of its entries
// exceeds that rounding, 4 eps sum_j |K_ij| |z_j| of its own row i; the rest, a quarter to a
// third of the entries, is left out.
struct KzBatch {
    int64_t j0, ncol, lo3, w3, off3, slice0, nslice, bit0;
    int64_t moff;  // first triplet of the batch's window in the masks mk, rb and km
};

// clears the batch's touched bits and, when masks, its structure masks and run bits
__global__ __launch_bounds__(256) void k_kzb_init(const KzBatch *__restrict__ bt, int words, uint32_t *__restrict__ mk,
                                                  uint32_t *__restrict__ rb, uint32_t *__restrict__ touched,
                                                  uint32_t *__restrict__ ends, int masks) {
    const KzBatch B = bt[blockIdx.y];
    if (blockIdx.x >= B.nslice) return;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = min<int64_t>(B.w3, t0 + kSlice);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 256) {
        if (masks) {
            mk[B.moff + t] = 0u;
            rb[B.moff + t] = 0u;
        }
    }
    if (blockIdx.x == 0)
        for (int t = threadIdx.x; t < words; t += 256) touched[B.bit0 + t] = 0u;
    if (masks && blockIdx.x == 0 && threadIdx.x == 0) ends[blockIdx.y] = 0u;
}

// one workgroup per (vector, batch): scatter z_j and flag its triplets.  The three rows
// of each flagged triplet are cleared first (column b belongs to this workgroup), so zd
// holds z_j exactly where rb flags vector b and is never read elsewhere.
__global__ __launch_bounds__(256) void k_kzb_scatter(const KzBatch *__restrict__ bt, const int64_t *__restrict__ ztp,
                                                     const int32_t *__restrict__ zti, const double *__restrict__ ztv,
                                                     double *__restrict__ zd, uint32_t *rb) {
    const KzBatch B = bt[blockIdx.y];
    const int b = blockIdx.x;
    if (b >= B.ncol) return;
    const int64_t j = B.j0 + b;
    for (int64_t e = ztp[j] + threadIdx.x; e < ztp[j + 1]; e += 256) {
        const int64_t t = (int64_t)zti[e] - 3 * B.lo3;
        if (t < 0 || t >= 3 * B.w3) continue;
        const int64_t t3 = 3 * (t / 3);
        for (int r = 0; r < 3; ++r) zd[(3 * B.off3 + t3 + r) * kBatch + b] = 0.0;
    }
    __syncthreads();
    for (int64_t e = ztp[j] + threadIdx.x; e < ztp[j + 1]; e += 256) {
        const int64_t t = (int64_t)zti[e] - 3 * B.lo3;
        if (t < 0 || t >= 3 * B.w3) continue;
        zd[(3 * B.off3 + t) * kBatch + b] = ztv[e];
        atomicOr(&rb[B.moff + t / 3], 1u << b);
    }
}

// block structure of K z_j: every block column of the block rows of z_j's triplets.  A
// workgroup ORs the bits of its slice's block rows into an LDS window of the columns
// around the slice (kMarkHalo triplets on either side) and then ORs each nonzero window
// word into mk once; a column outside the window goes to mk directly.  Slices without a
// flagged triplet return at once.
constexpr int kMarkHalo = 7680;
constexpr int kMarkWindow = kSlice + 2 * kMarkHalo;  // 16384 words, 64 KB of LDS
constexpr int kMarkRun = 16;  // block columns of a row loaded together

__global__ __launch_bounds__(256) void k_kzb_mark(const KzBatch *__restrict__ bt, const int32_t *__restrict__ bptr,
                                                  const int32_t *__restrict__ bcol, const uint32_t *__restrict__ rb,
                                                  uint32_t *mk) {
    __shared__ uint32_t win[kMarkWindow];
    const KzBatch B = bt[blockIdx.y];
    if (blockIdx.x >= B.nslice) return;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = min<int64_t>(B.w3, t0 + kSlice);
    bool any = false;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 256) any = any || rb[B.moff + t] != 0u;
    if (!__syncthreads_or(any)) return;
    for (int i = threadIdx.x; i < kMarkWindow; i += 256) win[i] = 0u;
    __syncthreads();
    const int64_t w0 = t0 - kMarkHalo;  // window column of win[0] (may be negative)
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 256) {
        const uint32_t bits = rb[B.moff + t];
        if (!bits) continue;
        const int64_t R = B.lo3 + t;
        const int64_t q0 = bptr[R], q1 = bptr[R + 1];
        for (int64_t q = q0; q < q1; q += kMarkRun) {
            // a run of block columns loaded together, then their marks
            int32_t cr[kMarkRun];
#pragma unroll
            for (int u = 0; u < kMarkRun; ++u) cr[u] = q + u < q1 ? bcol[q + u] : -1;
#pragma unroll
            for (int u = 0; u < kMarkRun; ++u) {
                if (cr[u] < 0) continue;
                const int64_t c = (int64_t)cr[u] - B.lo3;
                if (c < 0 || c >= B.w3) continue;
                const int64_t l = c - w0;
                if (l >= 0 && l < kMarkWindow) atomicOr(&win[l], bits);
                else atomicOr(&mk[B.moff + c], bits);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kMarkWindow; i += 256) {
        const uint32_t v = win[i];
        const int64_t c = w0 + i;
        if (v && c >= 0 && c < B.w3) atomicOr(&mk[B.moff + c], v);
    }
}

// per (slice, vector) counts of rows (three per triplet of the mask), and per slice the
// number of triplets.  km null: the structure, and bit b of the batch's ends set where the
// structures of vectors b and b + 1 differ; else the triplets kept (km, set on mk's triplets).
__global__ __launch_bounds__(256) void k_kzb_count(const KzBatch *__restrict__ bt, const uint32_t *__restrict__ mk,
                                                   const uint32_t *__restrict__ km, int32_t *__restrict__ cnt,
                                                   int32_t *__restrict__ tcnt, uint32_t *__restrict__ ends) {
    __shared__ int32_t c_s[4][kBatch + 1];
    __shared__ uint32_t e_s;
    const KzBatch B = bt[blockIdx.y];
    if (blockIdx.x >= B.nslice) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x == 0) e_s = 0u;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice;
    uint32_t m[kSlice / 256], differ = 0u;
#pragma unroll
    for (int r = 0; r < kSlice / 256; ++r) {
        const int64_t t = t0 + 256 * r + threadIdx.x;
        m[r] = t < B.w3 ? mk[B.moff + t] : 0u;
    }
    if (km) {
#pragma unroll
        for (int r = 0; r < kSlice / 256; ++r)
            if (m[r]) m[r] = km[B.moff + t0 + 256 * r + threadIdx.x];
    }
    // a wave's counts by ballots, lane b taking vector b's and lane kBatch the triplets':
    // 6 us over the 3 x 23^3 problem, 37 with seventeen LDS adds per thread
    int32_t mine = 0;
#pragma unroll
    for (int r = 0; r < kSlice / 256; ++r) {
        differ |= m[r] ^ (m[r] >> 1);
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const int n = __popcll(__ballot((m[r] >> b) & 1u));
            mine += lane == b ? 3 * n : 0;
        }
        const int n = __popcll(__ballot(m[r] != 0u));
        mine += lane == kBatch ? n : 0;
    }
    if (lane <= kBatch) c_s[wv][lane] = mine;
    __syncthreads();
    if (!km && differ) atomicOr(&e_s, differ);
    if (threadIdx.x <= kBatch) {
        const int32_t n = (c_s[0][threadIdx.x] + c_s[1][threadIdx.x]) + (c_s[2][threadIdx.x] + c_s[3][threadIdx.x]);
        if (threadIdx.x < kBatch) cnt[(B.slice0 + blockIdx.x) * kBatch + threadIdx.x] = n;
        else tcnt[B.slice0 + blockIdx.x] = n;
    }
    if (km) return;
    __syncthreads();
    if (threadIdx.x == 0 && e_s) atomicOr(&ends[blockIdx.y], e_s);
}

// Per batch (kBatch + 1 threads): thread b < ncol forms the slice offsets within vector
// b's structure and the vector's total; thread kBatch forms each slice's first work item
// (exclusive prefix of the triplet counts) and the batch's number of items.
__global__ void k_kzb_offsets(const KzBatch *__restrict__ bt, int nbat, const int32_t *__restrict__ cnt,
                              const int32_t *__restrict__ tcnt, int32_t *__restrict__ soff,
                              int64_t *__restrict__ kzcnt, int32_t *__restrict__ icnt, int64_t *__restrict__ nitems) {
    const int bi = blockIdx.x;
    if (bi >= nbat) return;
    const KzBatch B = bt[bi];
    const int b = threadIdx.x;
    int64_t run = 0;
    if (b == kBatch) {
        for (int64_t sl = 0; sl < B.nslice; ++sl) {
            icnt[B.slice0 + sl] = (int32_t)run;
            run += tcnt[B.slice0 + sl];
        }
        nitems[bi] = run;
        return;
    }
    if (b >= B.ncol) return;
    for (int64_t sl = 0; sl < B.nslice; ++sl) {
        soff[(B.slice0 + sl) * kBatch + b] = (int32_t)run;
        run += cnt[(B.slice0 + sl) * kBatch + b];
    }
    kzcnt[B.j0 + b] = run;
}

// Every structure triplet of the slice gets a work item, stored densely per batch in slice
// order.
struct KzItem {
    int32_t t, mask;  // its triplet, its vectors
};

__global__ __launch_bounds__(256) void k_kzb_items(const KzBatch *__restrict__ bt, const uint32_t *__restrict__ mk,
                                                   const int32_t *__restrict__ icnt, KzItem *__restrict__ items) {
    __shared__ int32_t wave_cnt[kSlice / 64];
    const KzBatch B = bt[blockIdx.y];
    if (blockIdx.x >= B.nslice) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t item0 = B.off3 + icnt[B.slice0 + blockIdx.x];
    const int64_t t0 = (int64_t)blockIdx.x * kSlice;
    uint32_t m[kSlice / 256];
    int rank[kSlice / 256];
#pragma unroll
    for (int r = 0; r < kSlice / 256; ++r) {
        const int64_t t = t0 + 256 * r + threadIdx.x;
        m[r] = t < B.w3 ? mk[B.moff + t] : 0u;
        const unsigned long long bal = __ballot(m[r] != 0u);
        rank[r] = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wave_cnt[4 * r + wv] = __popcll(bal);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSlice / 256; ++r) {
        if (!m[r]) continue;
        int before = 0;
        for (int w = 0; w < 4 * r + wv; ++w) before += wave_cnt[w];
        items[item0 + before + rank[r]] = KzItem{(int32_t)(t0 + 256 * r + threadIdx.x), (int32_t)m[r]};
    }
}

// The kept triplets' entries of (KZ)^T from the dense K z, at their ranks within each vector.
__global__ __launch_bounds__(256) void k_kzb_store(const KzBatch *__restrict__ bt, const uint32_t *__restrict__ mk,
                                                   const uint32_t *__restrict__ km, const int32_t *__restrict__ soff,
                                                   const int64_t *__restrict__ kzp, const double *__restrict__ kd,
                                                   int32_t *__restrict__ kzi, double *__restrict__ kzv) {
    __shared__ int32_t wave_cnt[2][4][kBatch];
    const KzBatch B = bt[blockIdx.y];
    if (blockIdx.x >= B.nslice) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = min<int64_t>(B.w3, t0 + kSlice);
    int32_t carry[kBatch];  // rows of the slice's earlier chunks
#pragma unroll
    for (int b = 0; b < kBatch; ++b) carry[b] = 0;
    int buf = 0;
    for (int64_t c0 = t0; c0 < t1; c0 += 256, buf ^= 1) {
        const int64_t t = c0 + threadIdx.x;
        uint32_t m = t < t1 ? mk[B.moff + t] : 0u;
        if (m) m = km[B.moff + t];
        int32_t rank[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const unsigned long long bal = __ballot((m >> b) & 1u);
            rank[b] = __popcll(bal & ((1ull << lane) - 1ull));
            if (lane == 0) wave_cnt[buf][wv][b] = __popcll(bal);
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            int32_t before = carry[b];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                before += w < wv ? wave_cnt[buf][w][b] : 0;
                carry[b] += wave_cnt[buf][w][b];
            }
            if (!((m >> b) & 1u)) continue;
            const int64_t pos = kzp[B.j0 + b] + soff[(B.slice0 + blockIdx.x) * kBatch + b] + 3 * (before + rank[b]);
            for (int i = 0; i < 3; ++i) {
                kzi[pos + i] = (int32_t)(3 * (B.lo3 + t) + i);
                kzv[pos + i] = kd[(3 * (B.off3 + t) + i) * kBatch + b];
            }
        }
    }
}

// Compute pass: (K z_j) on the three rows of each structure triplet from the packed 3x3
// blocks.  Sixteen lanes per work item: lane bits 0-1 pick four of the batch's vectors,
// bits 2-3 a quarter of the block row's blocks; the quarters are combined by a fixed
// shuffle tree.  Writes the dense kd and the triplet's kept vectors km (see above), and flags
// the deflation vectors with a nonzero in a structure row as touched.
__global__ __launch_bounds__(256) void k_kzb_values(const KzBatch *__restrict__ bt, const int64_t *__restrict__ nitems,
                                                    const KzItem *__restrict__ items, const int32_t *__restrict__ bptr,
                                                    const int32_t *__restrict__ bcol, const double *__restrict__ bval,
                                                    const double *__restrict__ zd, const uint32_t *__restrict__ rb,
                                                    const int64_t *__restrict__ zp,
                                                    const int32_t *__restrict__ zc, double *__restrict__ kd,
                                                    uint32_t *__restrict__ km, const uint32_t *__restrict__ ends,
                                                    int words, uint32_t *touched) {
    __shared__ uint32_t tw[kTouchLds];
    const KzBatch B = bt[blockIdx.y];
    const int64_t n_it = nitems[blockIdx.y];
    const uint32_t run_ends = ends[blockIdx.y];
    const int sub = threadIdx.x & 3, part = (threadIdx.x >> 2) & 3;
    const bool lds_bits = words <= kTouchLds;
    if (lds_bits)
        for (int t = threadIdx.x; t < words; t += 256) tw[t] = 0u;
    __syncthreads();
    uint32_t *tb = lds_bits ? tw : touched + B.bit0;
    // a contiguous run of items per workgroup (neighbouring triplets, few deflation
    // vectors); the loop bound is uniform over the workgroup, so the shuffles stay in step
    const int64_t per = ((n_it + gridDim.x - 1) / gridDim.x + 15) / 16 * 16;
    const int64_t x0 = (int64_t)blockIdx.x * per, x1 = min(n_it, x0 + per);
    for (int64_t x = x0 + (threadIdx.x >> 4); x - (threadIdx.x >> 4) < x1; x += 16) {
        const bool live = x < x1;
        double acc[3][4], mag[3][4];  // (K z)_i and sum |K_ij| |z_j|
        for (int i = 0; i < 3; ++i)
            for (int b = 0; b < 4; ++b) acc[i][b] = mag[i][b] = 0.0;
        int64_t t = 0, R = 0;
        uint32_t mask = 0u;
        if (live) {
            t = items[B.off3 + x].t;
            mask = (uint32_t)items[B.off3 + x].mask;
            R = B.lo3 + t;
            const int64_t beg = bptr[R], mR = bptr[R + 1] - beg;
            const double *rv = bval + 9 * beg;
            for (int64_t q = beg + part; q < beg + mR; q += 4) {
                const int64_t c = (int64_t)bcol[q] - B.lo3;
                if (c < 0 || c >= B.w3) continue;
                const uint32_t zb = rb[B.moff + c] >> (4 * sub);
                if (!(zb & 15u)) continue;  // none of this lane's vectors has support on triplet c
                double v[9];
                for (int e = 0; e < 9; ++e) v[e] = rv[e * mR + (q - beg)];
                const double *z = zd + (3 * (B.off3 + c)) * kBatch + 4 * sub;
                for (int jj = 0; jj < 3; ++jj)
                    for (int b = 0; b < 4; ++b) {
                        const double zz = ((zb >> b) & 1u) ? z[jj * kBatch + b] : 0.0;
                        for (int i = 0; i < 3; ++i) {
                            acc[i][b] = fma(v[3 * i + jj], zz, acc[i][b]);
                            mag[i][b] = fma(fabs(v[3 * i + jj]), fabs(zz), mag[i][b]);
                        }
                    }
            }
            // the vectors of the triplet's three rows of Z, over the item's sixteen lanes: a
            // chain of loads and adds on one lane took the kernel from 95 to 104 us (23^3)
            const int64_t e1 = zp[3 * R + 3];
            for (int64_t e = zp[3 * R] + (threadIdx.x & 15); e < e1; e += 16) {
                const int32_t col = zc[e];
                atomicOr(&tb[col / 32], 1u << (col % 32));
            }
        }
        uint32_t keep = 0u;  // the lane's vectors with an entry above the rounding of its sum
        for (int i = 0; i < 3; ++i)
            for (int b = 0; b < 4; ++b) {
                acc[i][b] += __shfl_xor(acc[i][b], 4);
                acc[i][b] += __shfl_xor(acc[i][b], 8);
                mag[i][b] += __shfl_xor(mag[i][b], 4);
                mag[i][b] += __shfl_xor(mag[i][b], 8);
                // (a NaN is kept, and what no finite bound covers)
                if (!(fabs(acc[i][b]) <= 4.0 * DBL_EPSILON * mag[i][b] && isfinite(mag[i][b])))
                    keep |= 1u << (4 * sub + b);
            }
        keep |= (uint32_t)__shfl_xor((int)keep, 1);
        keep |= (uint32_t)__shfl_xor((int)keep, 2);
        if (!live || part != 0) continue;
        if (sub == 0) {  // all vectors of a run with one to keep
            for (int b = 1; b < kBatch; ++b) keep |= ((keep & ~run_ends) >> (b - 1) & 1u) << b;
            for (int b = kBatch - 2; b >= 0; --b) keep |= ((keep >> (b + 1)) & ~(run_ends >> b) & 1u) << b;
            km[B.moff + t] = keep & mask;
        }
        double *o = kd + (3 * (B.off3 + t)) * kBatch + 4 * sub;
        for (int i = 0; i < 3; ++i)
            for (int b = 0; b < 4; ++b) o[i * kBatch + b] = acc[i][b];
    }
    if (!lds_bits) return;
    __syncthreads();
    for (int t = threadIdx.x; t < words; t += 256)
        if (tw[t]) atomicOr(&touched[B.bit0 + t], tw[t]);
}

// E_raw[j0+b, i] = sum over the structure rows t of the batch in the rows of z_i of
// Z[t, i] (K z_{j0+b})_t, for the vectors i flagged as touched.  One wave per (i,
// batch); lanes stride over the rows of z_i inside the window, then a fixed-order
// wave reduction.
// First index in [a, e) whose entry is >= key (e if none), for an increasing array, by
// the whole wave: each round tests 64 evenly spaced entries and keeps the one gap that
// holds the answer, so a range of L entries takes about log_64 L rounds of one load.
__device__ __forceinline__ int64_t wave_lower_bound(const int32_t *__restrict__ v, int64_t a, int64_t e,
                                                    int64_t key) {
    const int lane = threadIdx.x & 63;
    int64_t lo = a, hi = e;  // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t step = (hi - lo + 63) / 64;
        const int64_t idx = lo + lane * step;
        const bool below = idx < hi && (int64_t)v[idx] < key;
        const int nless = __popcll(__ballot(below));  // the samples below key form a prefix
        if (nless == 0) {
            hi = lo;
        } else {
            const int64_t nlo = lo + (int64_t)(nless - 1) * step + 1;
            hi = min(hi, lo + (int64_t)nless * step);
            lo = nlo;
        }
    }
    return lo;
}

constexpr int kErowRun = 4;  // entries per lane whose rows and masks are loaded together

__global__ __launch_bounds__(256) void k_kzb_erows(const KzBatch *__restrict__ bt, int32_t k,
                                                   const int64_t *__restrict__ ztp, const int32_t *__restrict__ zti,
                                                   const double *__restrict__ ztv, const double *__restrict__ kd,
                                                   const uint32_t *__restrict__ mk, const uint32_t *__restrict__ touched,
                                                   double *__restrict__ eraw, int64_t ld) {
    const KzBatch B = bt[blockIdx.y];
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= k || B.w3 == 0) return;
    if (!((touched[B.bit0 + i / 32] >> (i % 32)) & 1u)) return;
    const int64_t lo = 3 * B.lo3, w = 3 * B.w3;
    int64_t a = ztp[i], e = ztp[i + 1];
    if (a == e || zti[e - 1] < lo || zti[a] >= lo + w) return;
    // the entries of z_i with rows in the window: [first row >= lo, first row >= lo + w)
    e = wave_lower_bound(zti, a, e, lo + w);
    a = wave_lower_bound(zti, a, e, lo);
    double acc[kBatch];
    for (int b = 0; b < kBatch; ++b) acc[b] = 0.0;
    for (int64_t q0 = a + lane; q0 < e; q0 += 64 * kErowRun) {
        // a run of the lane's entries: rows, then their structure masks, loaded together
        int64_t tr[kErowRun];
        bool on[kErowRun];
#pragma unroll
        for (int u = 0; u < kErowRun; ++u) tr[u] = q0 + 64 * u < e ? (int64_t)zti[q0 + 64 * u] - lo : -1;
#pragma unroll
        for (int u = 0; u < kErowRun; ++u) on[u] = tr[u] >= 0 && mk[B.moff + tr[u] / 3] != 0u;
        for (int u = 0; u < kErowRun; ++u) {
            if (!on[u]) continue;  // (K z_j)_t is structurally zero for every vector of the batch
            const double z = ztv[q0 + 64 * u];
            const double *kdr = kd + (3 * B.off3 + tr[u]) * kBatch;
            for (int b = 0; b < kBatch; ++b) acc[b] = fma(z, kdr[b], acc[b]);
        }
    }
    for (int b = 0; b < kBatch; ++b) {
        double v = acc[b];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        acc[b] = v;
    }
    if (lane == 0)
        for (int b = 0; b < kBatch; ++b)
            if (b < B.ncol) eraw[(B.j0 + b) * ld + i] = acc[b];
}

// A = S (E + E^T)/2 S with S = diag(1 / sqrt(E_ii)), padded to ld x ld with an identity
// tail; diag0 = diagonal of A; scale = the diagonal of S (1 where E_ii <= 0, whose
// pivot then fails the SPD test).  Inverting the Jacobi-scaled matrix is exact
// (E^-1 = S (S E S)^-1 S) and much better conditioned when the deflation vectors' scales
// differ (rigid-body rotations against translations, enriched against standard DoFs);
// the Schur pivots scale with the diagonal, so the SPD test is the unscaled one.
__global__ void k_symmetrise(int32_t k, int64_t ld, const double *__restrict__ eraw, double *__restrict__ A,
                             double *__restrict__ diag0, double *__restrict__ scale) {
    const int64_t total = ld * ld;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = t / ld, j = t % ld;
        double v;
        if (i < k && j < k) {
            const double di = eraw[i * ld + i], dj = eraw[j * ld + j];
            const double si = di > 0.0 ? 1.0 / sqrt(di) : 1.0, sj = dj > 0.0 ? 1.0 / sqrt(dj) : 1.0;
            v = (0.5 * (eraw[i * ld + j] + eraw[j * ld + i]) * si) * sj;
            if (i == j) scale[i] = si;
        } else {
            v = (i == j) ? 1.0 : 0.0;
        }
        A[t] = v;
        if (i == j) diag0[i] = v;
    }
}

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- symmetric sweeps
// The coarse matrix and the dense block-Jacobi blocks are symmetric positive definite, so
// their block Gauss-Jordan inverses are run as the symmetric sweep operator on the lower
// triangle of 64 x 64 tiles only, Jacobi-scaled.  Gauss-Jordan elimination without pivoting:
// its pivots are the Schur complement pivots of the Cholesky factorisation.  Step k, pivot
// p = a_kk:  a_rc -= a_rk a_kc / p (r, c != k),  a_kc /= p,  a_rk = -a_rk / p,  a_kk = 1 / p.
// After
// the sweeps over pivot blocks 0 .. p-1 the working matrix is symmetric up to signs: its
// entry (i, j) equals sigma_i sigma_j times entry (j, i), sigma = -1 on the rows of the
// pivot blocks already swept and +1 on the others, so every tile above the diagonal is a
// signed transpose of one below it, and a diagonal tile is symmetric (its upper half is
// always taken from its lower half).  Sweep p, with P = A_pp^-1 (symmetrised):
//   new row p:        T_J  = P A_pJ                       (panel kernel, every J)
//   new column p:     B_Ip = -A_Ip P = -T_I^T   (I > p)
//   new pivot tile:   B_pp = P
//   every other tile: B_IJ = A_IJ - A_Ip T_J
// so each lower tile costs one 64 x 64 x 64 product on the matrix cores, and a sweep
// reads and writes the lower triangle once: a quarter of the work of the full 32-wide
// sweeps over every tile.  The panel kernel stores T and the column panel C_I = A_Ip in
// buffers of their own, so the sweep updates the matrix in place.  (The dense blocks, whose
// sweeps are bound by that traffic and not by the chain of pivot inverses, run two at a time.)  In a numpy model on
// the Jacobi-scaled coarse matrices of the 40^3 and 80^3 workloads this form leaves
// max |I - E E^-1| at the level of the full 32-wide sweeps (80^3: 2.6e-3 against 2.9e-3).
constexpr int kCb = 64;
constexpr int kCbLd = kCb + 1;  // LDS row stride: a column's 16 rows in distinct banks

// v from lane K of each row of 16 lanes, in every lane of the row (one DPP move per half)
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + K, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + K, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// v from row G of 16 lanes, lane by lane, in every row: the row swaps of gfx950 with both
// operands the same register (odd rows of one against even rows of the other, then the
// halves)
template <int G>
__device__ __forceinline__ int rows_bcast_b32(int v) {
    const auto h = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const unsigned x = h[G & 1];
    const auto w = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return (int)w[G >> 1];
}
template <int G>
__device__ __forceinline__ double rows_bcast(double v) {
    return __hiloint2double(rows_bcast_b32<G>(__double2hiint(v)), rows_bcast_b32<G>(__double2loint(v)));
}

// Steps K .. 15 of the in-place Gauss-Jordan elimination of a symmetric 16 x 16 block a held by
// one wave, with the block b beside it in the same rows: b becomes a^-1 b, and u keeps the rows
// of b as they were when their pivot came, w those rows over their pivots, so that
// b^T a^-1 b' = w^T u'.  Lane l keeps elements (l / 16 + 4 v, l % 16), v < 4, the layout of the
// matrix instruction's result.  Row K and column K travel by lane moves within the vector unit
// (through the LDS crossbar a step took 0.2 us), no barrier.  An update of a forms the product
// of its two factors first, so that a stays symmetric (up to the signs of the steps) to the
// last bit.  Pivot K is kept in the lanes of column K.
template <int K>
__device__ __forceinline__ void gj16_steps(double (&a)[4], double (&b)[4], double (&u)[4], double (&w)[4],
                                           double &pivots) {
    if constexpr (K < 16) {
        const int l = threadIdx.x & 63, c = l & 15, g = l >> 4;
        const double rowk = rows_bcast<K % 4>(a[K / 4]), rowb = rows_bcast<K % 4>(b[K / 4]);
        const double p = row_bcast<K>(rowk);
        pivots = c == K ? p : pivots;
        // 1/p: hardware reciprocal refined by two Newton steps
        double ip = __builtin_amdgcn_rcp(p);
        ip = fma(ip, fma(-p, ip, 1.0), ip);
        ip = fma(ip, fma(-p, ip, 1.0), ip);
        const double rip = rowk * ip, ribp = rowb * ip;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double col = row_bcast<K>(a[v]), m = -col * ip;
            double x = fma(-(col * rowk), ip, a[v]), y = fma(m, rowb, b[v]);
            x = c == K ? m : x;
            if (v == K / 4) {
                const bool mine = g == K % 4;
                x = mine ? (c == K ? ip : rip) : x;
                y = mine ? ribp : y;
                u[v] = mine ? rowb : u[v];
                w[v] = mine ? ribp : w[v];
            }
            a[v] = x;
            b[v] = y;
        }
        gj16_steps<K + 1>(a, b, u, w, pivots);
    }
}

// P = S^-1 (symmetrised, in place) for the 64 x 64 SPD pivot block S in LDS (row stride
// kCbLd) by Gauss-Jordan elimination without pivoting, in four stages of 16 pivots.  Stage q
// of the 256 threads: every wave eliminates the 16 x 16 block S_qq in its own registers, wave w
// with S_qw beside it, which gives the new row block T_w = S_qq^-1 S_qw and, S being symmetric up
// to the signs of the sweeps, the new column block -+T_w^T; the rows the elimination went
// through give the update S_wJ -= S_wq S_qq^-1 S_qJ on the matrix cores, as the factors of a
// Cholesky factorisation would.  That keeps the accuracy of one pivot after the other (in a
// model with condition 1e6 |I - S P| is 1.9e-10 against 1.8e-10; with T_w and the update as
// products with an explicit inverse of S_qq it was 1.1e-9, and the preconditioner's error
// against a factorisation 1.5 to 2.4 times larger on meshes of 16 and 20 elements).  Three
// barriers a stage: what bounds the routine is one wave's chain of 64 pivot steps.  A barrier
// per pivot step over the whole block took 38 us in all, this 15; a sweep of the coarse
// inversion, which ends with the next pivot's inverse, went from 44 to 21 us up to k = 1000
// and from 57 to 46.5 us at k = 4528.  Pivot j is tested against kdim * DBL_EPSILON times the
// original diagonal entry gcol0 + j; returns whether one failed (in every thread).
__device__ __forceinline__ bool pivot_inverse64(double *S, const double *__restrict__ diag0, int64_t gcol0,
                                                int32_t kdim) {
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, c = l & 15, g = l >> 4;
    double floors[4];  // of pivots 16 q + c
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t gmine = gcol0 + 16 * q + c;
        floors[q] = gmine < kdim ? (double)kdim * DBL_EPSILON * fabs(diag0[gmine]) : 0.0;
    }
    bool bad = false;
    // one stage's code for all four: unrolled, the fetch of 64 steps of code costs as much as
    // running them
    const int stages = (int)min((int64_t)4, (kdim - gcol0 + 15) / 16);  // the identity tail inverts to itself
#pragma unroll 1
    for (int q = 0; q < stages; ++q) {
        const double fl = q < 2 ? (q == 0 ? floors[0] : floors[1]) : (q == 2 ? floors[2] : floors[3]);
        double inv[4], row[4], u[4], w[4], pivots = 1.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = g + 4 * v;
            inv[v] = S[(16 * q + max(r, c)) * kCbLd + 16 * q + min(r, c)];  // the lower half
            row[v] = S[(16 * q + r) * kCbLd + 16 * wv + c];
            u[v] = w[v] = 0.0;
        }
        gj16_steps<0>(inv, row, u, w, pivots);
        bad = bad || !(pivots > fl) || !isfinite(pivots);
        const double sign = wv < q ? -1.0 : 1.0;  // S_wq = sign S_qw^T
        if (wv != q)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[(16 * q + g + 4 * v) * kCbLd + 16 * wv + c] = u[v];
        __syncthreads();
        if (wv != q)
#pragma unroll
            for (int j = 1; j < 4; ++j) {  // the column blocks other than q
                const int J = (q + j) & 3;
                dbl4 x;
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = S[(16 * wv + g + 4 * v) * kCbLd + 16 * J + c];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    x = __builtin_amdgcn_mfma_f64_16x16x4f64(-sign * w[v],
                                                             S[(16 * q + g + 4 * v) * kCbLd + 16 * J + c], x, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) S[(16 * wv + g + 4 * v) * kCbLd + 16 * J + c] = x[v];
            }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = g + 4 * v;
            S[(16 * q + r) * kCbLd + 16 * wv + c] = wv != q ? row[v] : inv[v];
            if (wv != q) S[(16 * wv + c) * kCbLd + 16 * q + r] = -sign * row[v];
        }
        __syncthreads();
    }
    const int r0 = wv * 16;
    double a[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) a[q] = 0.5 * (S[(r0 + q) * kCbLd + l] + S[l * kCbLd + r0 + q]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) S[(r0 + q) * kCbLd + l] = a[q];
    __syncthreads();
    return __any(bad);
}

// X Y for 64 x 64 tiles X, Y in LDS (row stride kCbLd) on the matrix cores: wave w of the
// 256 threads computes the 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 blocks of 16 x 16,
// sixteen v_mfma_f64_16x16x4f64 steps each.  Result item v of block b = 2 bi + bj of lane
// l is element (cb_row(b, v), cb_col(b)) of the product.  XT, YT: X or Y is kept transposed.
__device__ __forceinline__ int cb_row(int b, int v) {
    return ((threadIdx.x >> 6) >> 1) * 32 + (b >> 1) * 16 + ((threadIdx.x & 63) >> 4) + 4 * v;
}
__device__ __forceinline__ int cb_col(int b) { return ((threadIdx.x >> 6) & 1) * 32 + (b & 1) * 16 + (threadIdx.x & 15); }

template <bool XT = false, bool YT = false>
__device__ __forceinline__ void cb_mfma(const double *X, const double *Y, dbl4 (&acc)[4]) {
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, kq = l >> 4;
    const int r0 = (wv >> 1) * 32 + (l & 15), c0 = (wv & 1) * 32 + (l & 15);
    auto x = [&](int r, int k) { return XT ? X[k * kCbLd + r] : X[r * kCbLd + k]; };
    auto y = [&](int k, int c) { return YT ? Y[c * kCbLd + k] : Y[k * kCbLd + c]; };
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int s4 = 0; s4 < kCb; s4 += 4) {
        const double x0 = x(r0, s4 + kq), x1 = x(r0 + 16, s4 + kq);
        const double y0 = y(s4 + kq, c0), y1 = y(s4 + kq, c0 + 16);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y0, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y1, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y0, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y1, acc[3], 0, 0, 0);
    }
}

// acc += X^T Y for 64 x 64 tiles X, Y in memory, both with the summed index first, in
// cb_mfma's split with the rows and the columns of a quadrant's two 16-wide blocks
// interleaved: a lane's operands, like its results, are pairs of neighbours, read from memory
// 256 contiguous bytes per 16 lanes without LDS.
__device__ __forceinline__ int fma_row(int b, int v) {
    return ((threadIdx.x >> 6) >> 1) * 32 + 2 * (((threadIdx.x & 63) >> 4) + 4 * v) + (b >> 1);
}
__device__ __forceinline__ int fma_col(int b) { return ((threadIdx.x >> 6) & 1) * 32 + 2 * (threadIdx.x & 15) + (b & 1); }

__device__ __forceinline__ void cb_fma(const double *__restrict__ X, const double *__restrict__ Y, dbl4 (&acc)[4]) {
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, kq = l >> 4;
    X += kq * kCb + (wv >> 1) * 32 + 2 * (l & 15);
    Y += kq * kCb + (wv & 1) * 32 + 2 * (l & 15);
#pragma unroll 2
    for (int s4 = 0; s4 < kCb; s4 += 4) {
        const dbl2 x = *(const dbl2 *)(X + s4 * kCb), y = *(const dbl2 *)(Y + s4 * kCb);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.y, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.y, acc[3], 0, 0, 0);
    }
}

// The lower tiles (I, J), I >= J, of a matrix under inversion: row-major ld x ld (the coarse
// matrix) or packed tile after tile (a dense block).
struct RowTiles {
    double *A;
    int64_t ld;
    __device__ __forceinline__ double *tile(int I, int J) const { return A + (int64_t)I * kCb * ld + J * kCb; }
    __device__ __forceinline__ int64_t stride() const { return ld; }
};
struct PackedTiles {
    double *A;
    __device__ __forceinline__ double *tile(int I, int J) const {
        return A + ((int64_t)I * (I + 1) / 2 + J) * (kCb * kCb);
    }
    __device__ __forceinline__ int64_t stride() const { return kCb; }
};

// a failed pivot sets *fail to 1 (failval < 0) or lowers it to failval
__device__ __forceinline__ void pivot_failed(int *fail, int failval) {
    if (failval < 0) atomicOr(fail, 1);
    else atomicMin(fail, failval);
}

// (I, J) of lower tile number tid = I (I + 1) / 2 + J
__device__ __forceinline__ void lower_tile(int64_t tid, int &I, int &J) {
    I = (int)((sqrt(8.0 * (double)tid + 1.0) - 1.0) * 0.5);
    while ((int64_t)(I + 1) * (I + 2) / 2 <= tid) ++I;
    while ((int64_t)I * (I + 1) / 2 > tid) --I;
    J = (int)(tid - (int64_t)I * (I + 1) / 2);
}

// P_0 = A_00^-1 (symmetrised) from the first diagonal tile's lower half; A_00 whole to orig when
// given.
template <class M>
__device__ __forceinline__ void first_pivot_body(const M &mat, int32_t kdim, const double *__restrict__ diag0,
                                                 double *__restrict__ P, double *__restrict__ orig, int *fail,
                                                 int failval) {
    __shared__ double S[kCb * kCbLd];
    const double *A = mat.tile(0, 0);
    const int64_t ld = mat.stride();
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;  // element (ta + 4 q, tb)
    double sv[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) sv[q] = A[(ta + 4 * q) * ld + tb];
#pragma unroll
    for (int q = 0; q < 16; ++q) S[(ta + 4 * q) * kCbLd + tb] = sv[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = ta + 4 * q;
        sv[q] = a >= tb ? S[a * kCbLd + tb] : S[tb * kCbLd + a];
        if (orig) orig[a * kCb + tb] = sv[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) S[(ta + 4 * q) * kCbLd + tb] = sv[q];
    __syncthreads();
    const bool bad = pivot_inverse64(S, diag0, 0, kdim);
#pragma unroll
    for (int q = 0; q < 16; ++q) P[(ta + 4 * q) * kCb + tb] = S[(ta + 4 * q) * kCbLd + tb];
    if (bad && threadIdx.x == 0) pivot_failed(fail, failval);
}

__global__ __launch_bounds__(256) void k_cgj_first_pivot(double *A, int64_t ld, int32_t kdim,
                                                         const double *__restrict__ diag0, double *__restrict__ P,
                                                         int *fail) {
    first_pivot_body(RowTiles{A, ld}, kdim, diag0, P, nullptr, fail, -1);
}

// Panel of sweep p, workgroup J != p: the tile A_pJ (stored below the diagonal for J < p;
// for J > p the transpose of the stored (J, p), sign +1), T_J = P A_pJ into tbuf[J], and
// the column tile A_Jp = s A_pJ^T into cbuf[J] (s = +1 for J > p, -1 for J < p: block row
// J is swept, block row p not yet).  Both buffers hold nt tiles of 64 x 64, row-major.
__global__ __launch_bounds__(256) void k_cgj_panel(int p, double *A0, int64_t ld, const double *__restrict__ P,
                                                   double *__restrict__ cbuf, double *__restrict__ tbuf) {
    const int J = blockIdx.x;
    __shared__ double S[kCb * kCbLd], Y[kCb * kCbLd];
    if (J == p) return;
    // all loads (coalesced, row-major) before the first LDS store: P, and the stored
    // tile (p, J) for J < p or (J, p) for J > p, which is A_pJ transposed
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;  // element (ta + 4 q, tb)
    const RowTiles mat{A0, ld};
    const double *A = J < p ? mat.tile(p, J) : mat.tile(J, p);
    double pv[16], yv[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = ta + 4 * q;
        pv[q] = P[a * kCb + tb];
        yv[q] = A[a * ld + tb];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = ta + 4 * q;
        S[a * kCbLd + tb] = pv[q];
        if (J < p) Y[a * kCbLd + tb] = yv[q];
        else Y[tb * kCbLd + a] = yv[q];
    }
    __syncthreads();
    const double s = J > p ? 1.0 : -1.0;
    double *cj_out = cbuf + (int64_t)J * kCb * kCb;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = ta + 4 * q;
        cj_out[a * kCb + tb] = s * Y[tb * kCbLd + a];
    }
    dbl4 acc[4];
    cb_mfma(S, Y, acc);
    double *tj = tbuf + (int64_t)J * kCb * kCb;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) tj[cb_row(b, v) * kCb + cb_col(b)] = acc[b][v];
}

// Sweep p of the lower tiles, in place, one workgroup each.  The workgroup of the next pivot
// tile (p + 1, p + 1) also inverts it into Pnext (P and Pnext are distinct buffers).  The
// tiles, numbered row by row, are rotated so that this one is dispatched first: its inverse is
// the critical path of the sweep, overlapped with the other tiles.
__global__ __launch_bounds__(256) void k_cgj_sweep(int p, int nt, double *A0, int64_t ld, int32_t kdim,
                                                   const double *__restrict__ P, double *__restrict__ Pnext,
                                                   const double *__restrict__ cbuf, const double *__restrict__ tbuf,
                                                   const double *__restrict__ diag0, int *fail) {
    __shared__ double X[kCb * kCbLd], Y[kCb * kCbLd];
    const int64_t ntl = (int64_t)nt * (nt + 1) / 2;
    const int64_t first = p + 1 < nt ? (int64_t)(p + 1) * (p + 2) / 2 + (p + 1) : 0;
    int I, J;
    lower_tile((blockIdx.x + first) % ntl, I, J);
    double *A = RowTiles{A0, ld}.tile(I, J);
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;  // element (ta + 4 q, tb)
    if (I == p || J == p) {
        // pivot tile P; row p: T_J; column p: -T_I^T (transposed through LDS)
        const double *src = I == p && J == p ? P : tbuf + (int64_t)(I == p ? J : I) * kCb * kCb;
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = src[(ta + 4 * q) * kCb + tb];
        if (J == p && I != p) {
#pragma unroll
            for (int q = 0; q < 16; ++q) X[(ta + 4 * q) * kCbLd + tb] = v[q];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = -X[tb * kCbLd + ta + 4 * q];
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) A[(ta + 4 * q) * ld + tb] = v[q];
        return;
    }
    // all loads before the first LDS store
    const double *xi = cbuf + (int64_t)I * kCb * kCb, *yj = tbuf + (int64_t)J * kCb * kCb;
    double sr[16], xr[16], yr[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        xr[q] = xi[(ta + 4 * q) * kCb + tb];
        yr[q] = yj[(ta + 4 * q) * kCb + tb];
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int a = cb_row(b, v), c = cb_col(b);
            sr[4 * b + v] = I == J && a < c ? A[c * ld + a] : A[a * ld + c];  // a diagonal tile's lower half
        }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        X[(ta + 4 * q) * kCbLd + tb] = xr[q];
        Y[(ta + 4 * q) * kCbLd + tb] = yr[q];
    }
    __syncthreads();
    dbl4 acc[4];
    cb_mfma(X, Y, acc);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sr[4 * b + v] -= acc[b][v];
            A[cb_row(b, v) * ld + cb_col(b)] = sr[4 * b + v];
        }
    if (I == p + 1 && J == p + 1) {
        __syncthreads();  // every wave is done with X
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) X[cb_row(b, v) * kCbLd + cb_col(b)] = sr[4 * b + v];
        __syncthreads();
        // the symmetric block from the lower half
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int a = ta + 4 * q;
            Y[a * kCbLd + tb] = a >= tb ? X[a * kCbLd + tb] : X[tb * kCbLd + a];
        }
        __syncthreads();
        const bool bad = pivot_inverse64(Y, diag0, (int64_t)I * kCb, kdim);
#pragma unroll
        for (int q = 0; q < 16; ++q) Pnext[(ta + 4 * q) * kCb + tb] = Y[(ta + 4 * q) * kCbLd + tb];
        if (bad && threadIdx.x == 0) pivot_failed(fail, -1);
    }
}

// The final E^-1 from the lower tiles of the inverse X of the scaled matrix: F = S X S,
// entry (i, j) from X's entry (max(i, j), min(i, j)), written to the dense array (both
// triangles) and as the packed lower-triangle tiles of the solve; one workgroup per
// lower tile of kCoarseTile^2.  The two scale factors are applied in index order, so the
// dense result is exactly symmetric.
__global__ __launch_bounds__(256) void k_einv_from_lower(int32_t k, int64_t ld, const double *__restrict__ scale,
                                                         const double *__restrict__ X, double *__restrict__ einv,
                                                         double *__restrict__ tiles) {
    constexpr int T = kCoarseTile;
    __shared__ double F[T][T + 1];
    const int64_t tid = blockIdx.x;
    int I, J;
    lower_tile(tid, I, J);
    double *out = tiles + tid * T * T;
    for (int e = threadIdx.x; e < T * T; e += 256) {
        const int a = e / T, b = e % T;
        const int ra = I * T + a, cb = J * T + b;
        double f = 0.0;
        if (ra < k && cb < k) {
            const int hi = max(ra, cb), lo = min(ra, cb);
            f = (X[(int64_t)hi * ld + lo] * scale[lo]) * scale[hi];
            einv[(int64_t)ra * ld + cb] = f;
        }
        out[e] = f;
        F[a][b] = f;
    }
    if (I != J) {  // the mirrored tile (J, I) of the dense array, written row by row
        __syncthreads();
        for (int e = threadIdx.x; e < T * T; e += 256) {
            const int a = e / T, b = e % T;
            const int rb = J * T + a, ca = I * T + b;
            if (rb < k && ca < k) einv[(int64_t)rb * ld + ca] = F[b][a];
        }
    }
}

// ---------------------------------------------------------------- dense blocks
// Block-Jacobi blocks of more than kMaxBlock DoFs (subdomain-sized blocks).  The lower
// triangle of K_BB, Jacobi-scaled, is inverted as 64 x 64 tiles (the identity beyond the block's
// size): blocks of one or two tiles each by a workgroup in LDS (k_gjb_small), larger ones
// gathered into packed tiles and inverted by the symmetric sweeps above, batched over the
// blocks: the table is sorted by tiles, most first, so the blocks that still have a pivot tile
// p form a prefix, and a sweep of pivot tiles p and p + 1 runs the tiles of that prefix in one
// launch.  A failed pivot lowers the flag to the block's index.
struct GjMat {
    int64_t tile0;  // first lower tile (prefix of nt (nt + 1) / 2), also its place in the work buffer
    int64_t row0;   // first tile row (prefix of nt): its panels, its diagonal and scale (64 each)
    int64_t out;    // first entry of its inverse in dinv
    int32_t nt, size, start, block;
    int64_t buf0, piv0;  // first tile of its row buffers and of its pivot inverses
};

// last matrix whose first tile (row) is <= wg
template <int64_t GjMat::*FIRST>
__device__ __forceinline__ int gj_find(const GjMat *__restrict__ m, int count, int64_t wg) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (m[mid].*FIRST <= wg) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// scale_i = 1 / sqrt(K_ii) of the matrices' rows (1 where K_ii <= 0 or is absent, whose pivot
// then fails the SPD test, and beyond the block's size), one thread per row, which searches its
// increasing columns (a wave per row that read all of them took 85 us for 180,000 rows, this 14)
__global__ __launch_bounds__(256) void k_dense_scale(const GjMat *__restrict__ mats, int count,
                                                     const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                                     const double *__restrict__ val, double *__restrict__ scale) {
    for (int mi = blockIdx.y; mi < count; mi += gridDim.y) {
        const GjMat G = mats[mi];
        for (int i = blockIdx.x * 256 + threadIdx.x; i < G.nt * kCb; i += gridDim.x * 256) {
            double d = 0.0;
            if (i < G.size) {
                const int64_t g = (int64_t)G.start + i, end = ptr[g + 1];
                int64_t lo = ptr[g], hi = end;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (idx[mid] < g) lo = mid + 1;
                    else hi = mid;
                }
                if (lo < end && idx[lo] == g) d = val[lo];
            }
            scale[G.row0 * kCb + i] = d > 0.0 ? 1.0 / sqrt(d) : 1.0;
        }
    }
}

// rows of matrix blockIdx.y (grid-stride), sixteen lanes each: the scaled lower-triangle entries
// of K_BB, their diagonal to diag0, the identity beyond the block's size (73 -> 40 us against a
// wave each).  W and diag0 are zero on entry.
__global__ __launch_bounds__(256) void k_dense_gather(const GjMat *__restrict__ mats, int count,
                                                      const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                                      const double *__restrict__ val,
                                                      const double *__restrict__ scale, double *__restrict__ W,
                                                      double *__restrict__ diag0) {
    const int lane = threadIdx.x & 15;
    for (int mi = blockIdx.y; mi < count; mi += gridDim.y) {
        const GjMat G = mats[mi];
        const PackedTiles T{W + G.tile0 * (kCb * kCb)};
        const double *sc = scale + G.row0 * kCb;
        for (int i = blockIdx.x * 16 + (threadIdx.x >> 4); i < G.nt * kCb; i += gridDim.x * 16) {
            if (i >= G.size) {
                if (lane == 0) {
                    T.tile(i / kCb, i / kCb)[(i % kCb) * (kCb + 1)] = 1.0;
                    diag0[G.row0 * kCb + i] = 1.0;
                }
                continue;
            }
            const int64_t g = (int64_t)G.start + i;
            for (int64_t e = ptr[g] + lane; e < ptr[g + 1]; e += 16) {
                const int64_t c = (int64_t)idx[e] - G.start;
                if (c < 0 || c > i) continue;
                const double v = (val[e] * sc[i]) * sc[c];
                T.tile(i / kCb, (int)c / kCb)[(i % kCb) * kCb + c % kCb] = v;
                if (c == i) diag0[G.row0 * kCb + i] = v;
            }
        }
    }
}

// The dense blocks take two pivot tiles p and q = p + 1 at a time (one where a matrix ends):
// a sweep reads and writes every tile once, so two in one pass halve that traffic.  With
// L = A_qp, the second sweep's rows are formed from the first's,
//   P = A_pp^-1,  T1_J = P A_pJ,  B_qJ = A_qJ - L T1_J,  P' = B_qq^-1,  T2_J = P' B_qJ,
// B_qp being -L P, and a tile's update is the two products together,
//   B_IJ = A_IJ - A_Ip T1_J - B_Iq T2_J;
// in row p it starts from T1_J, in column p from -T1_I^T, in the pivot tile from P, all without
// the first product; row q is T2_J, column q -T2_I^T, its pivot tile P'.  The column tiles
// A_Ip and B_Iq are signed transposes of row tiles, so -s A_pI and -s B_qI are kept (s = +1
// for I > p, else -1): the summed index first, as cb_fma reads them.
//
// T1_J = P A_pJ by the explicit inverse leaves the residual A_pJ - A_pp T1_J at eps cond(A_pp),
// which the tiles not yet swept take over: errors grew with the square of the condition.  One
// step of refinement, T1_J += P (A_pJ - A_pp T1_J), and the same for T2_J, for the rows J still
// to be swept keeps elimination's accuracy (in a model further refinement changes nothing).
// Error of M^-1 r, blocks of 80 / 129 / 256 / 800 unknowns with condition 1e6: 8.9e-12, 1.5e-11,
// 1.5e-11, 1.2e-11; without 1.1e-8, 7.6e-10, 5.7e-11, 1.6e-11 (sweeps of 32 pivots: 2.0e-10,
// 3.0e-11, 9.3e-12, 5.8e-12).
struct GjBufs {
    double *c1, *t1, *c2, *t2;  // a matrix's tiles: -s A_pJ, T1_J, -s B_qJ, T2_J
};
__device__ __forceinline__ GjBufs gj_bufs(const GjMat &G, double *cbuf, double *tbuf) {
    const int64_t o = G.buf0 * (kCb * kCb), n = (int64_t)G.nt * (kCb * kCb);
    return {cbuf + o, tbuf + o, cbuf + o + n, tbuf + o + n};
}
// P of pivot tile p (i = 0) or P' (i = 1): two pairs per matrix, used in turn (as many tiles of
// them as it has pivots)
// (and, in an array of the same layout, of A_pp and B_qq)
__device__ __forceinline__ double *gj_pivot(double *P, const GjMat &G, int p, int i) {
    return P + (G.piv0 + (p & 2) + i) * (kCb * kCb);
}

__global__ __launch_bounds__(256) void k_gjb_first_pivot(const GjMat *__restrict__ mats, int count, double *W,
                                                         const double *__restrict__ diag0, double *__restrict__ P,
                                                         double *__restrict__ orig, int *fail) {
    for (int mi = blockIdx.x; mi < count; mi += gridDim.x) {
        const GjMat G = mats[mi];
        __syncthreads();
        first_pivot_body(PackedTiles{W + G.tile0 * (kCb * kCb)}, G.size, diag0 + G.row0 * kCb,
                         gj_pivot(P, G, 0, 0), gj_pivot(orig, G, 0, 0), fail, G.block);
    }
}

__device__ __forceinline__ void cb_to_lds(const dbl4 (&acc)[4], double *S) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) S[cb_row(b, v) * kCbLd + cb_col(b)] = acc[b][v];
}

// S becomes the symmetric matrix of its lower half
__device__ __forceinline__ void mirror_lower(double *S) {
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;
    double v[16];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = ta + 4 * q;
        v[q] = a >= tb ? S[a * kCbLd + tb] : S[tb * kCbLd + a];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) S[(ta + 4 * q) * kCbLd + tb] = v[q];
    __syncthreads();
}

// the LDS tile Y in a product's result layout
__device__ __forceinline__ void cb_from_lds(const double *Y, dbl4 (&y)[4]) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[b][v] = Y[cb_row(b, v) * kCbLd + cb_col(b)];
}

// S (LDS) becomes the 64 x 64 tile A in memory
__device__ __forceinline__ void tile_to_lds(const double *__restrict__ A, double *S) {
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = A[(ta + 4 * q) * kCb + tb];
#pragma unroll
    for (int q = 0; q < 16; ++q) S[(ta + 4 * q) * kCbLd + tb] = v[q];
}

// t += P (y - A t), t and y in the result layout, P and A = P^-1 tiles in memory; S and Y are
// LDS tiles to use, which the caller may still be reading.  Ends without a barrier.
__device__ __forceinline__ void refine(const double *__restrict__ P, const double *__restrict__ A,
                                       const dbl4 (&y)[4], dbl4 (&t)[4], double *S, double *Y) {
    dbl4 x[4];
    __syncthreads();
    tile_to_lds(A, S);
    cb_to_lds(t, Y);
    __syncthreads();
    cb_mfma(S, Y, x);
    __syncthreads();
    tile_to_lds(P, S);
#pragma unroll
    for (int b = 0; b < 4; ++b) x[b] = y[b] - x[b];
    cb_to_lds(x, Y);
    __syncthreads();
    cb_mfma(S, Y, x);
#pragma unroll
    for (int b = 0; b < 4; ++b) t[b] += x[b];
}

// P' of the first count matrices (those with a pivot tile p + 1), and T1_q
__global__ __launch_bounds__(256, 2) void k_gjb_pivot2(int p, const GjMat *__restrict__ mats, int count,
                                                    const double *__restrict__ W, double *Pm, double *orig,
                                                    double *cbuf, double *tbuf, const double *__restrict__ diag0,
                                                    int *fail) {
    __shared__ double S[kCb * kCbLd], Y[kCb * kCbLd];
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;  // element (ta + 4 q, tb)
    for (int mi = blockIdx.x; mi < count; mi += gridDim.x) {
        const GjMat G = mats[mi];
        const double *A = W + G.tile0 * (kCb * kCb);
        const int64_t row = (int64_t)(p + 1) * (p + 2) / 2;
        const double *L = A + (row + p) * (kCb * kCb), *Aqq = L + kCb * kCb;
        const double *P = gj_pivot(Pm, G, p, 0);
        double *P2 = gj_pivot(Pm, G, p, 1), *O2 = gj_pivot(orig, G, p, 1);
        double *t1 = gj_bufs(G, cbuf, tbuf).t1 + (int64_t)(p + 1) * (kCb * kCb);
        double lv[16];
        __syncthreads();
        tile_to_lds(P, S);
#pragma unroll
        for (int q = 0; q < 16; ++q) lv[q] = L[(ta + 4 * q) * kCb + tb];
#pragma unroll
        for (int q = 0; q < 16; ++q) Y[tb * kCbLd + ta + 4 * q] = lv[q];
        __syncthreads();
        dbl4 t[4], y[4], acc[4];
        cb_mfma(S, Y, t);  // T1_q = P L^T
        cb_from_lds(Y, y);
        refine(P, gj_pivot(orig, G, p, 0), y, t, S, Y);
        __syncthreads();
        cb_to_lds(t, Y);
#pragma unroll
        for (int q = 0; q < 16; ++q) S[(ta + 4 * q) * kCbLd + tb] = lv[q];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                t1[cb_row(b, v) * kCb + cb_col(b)] = t[b][v];
                y[b][v] = Aqq[cb_row(b, v) * kCb + cb_col(b)];
            }
        __syncthreads();
        cb_mfma(S, Y, acc);
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b] = y[b] - acc[b];
        cb_to_lds(acc, S);
        mirror_lower(S);
#pragma unroll
        for (int q = 0; q < 16; ++q) O2[(ta + 4 * q) * kCb + tb] = S[(ta + 4 * q) * kCbLd + tb];
        __syncthreads();
        const bool bad = pivot_inverse64(S, diag0 + G.row0 * kCb, (int64_t)(p + 1) * kCb, G.size);
#pragma unroll
        for (int q = 0; q < 16; ++q) P2[(ta + 4 * q) * kCb + tb] = S[(ta + 4 * q) * kCbLd + tb];
        if (bad && threadIdx.x == 0) pivot_failed(fail, G.block);
    }
}

// Row tiles J of the pivot tiles p and p + 1, one workgroup each, over the first count
// matrices (those with more than p pivot tiles)
__global__ __launch_bounds__(256) void k_gjb_panel(int p, const GjMat *__restrict__ mats, int count,
                                                   const double *__restrict__ W, double *Pm, double *orig,
                                                   double *cbuf, double *tbuf) {
    __shared__ double S[kCb * kCbLd], Y[kCb * kCbLd];
    const int mi = gj_find<&GjMat::row0>(mats, count, blockIdx.x);
    const GjMat G = mats[mi];
    const int J = (int)(blockIdx.x - G.row0);
    const bool two = p + 1 < G.nt;
    if (two ? J == p + 1 : J == p) return;
    const PackedTiles T{const_cast<double *>(W) + G.tile0 * (kCb * kCb)};
    const GjBufs B = gj_bufs(G, cbuf, tbuf);
    const double *P = gj_pivot(Pm, G, p, 0), *P2 = gj_pivot(Pm, G, p, 1), *L = T.tile(p + 1, p);
    const int64_t o = (int64_t)J * (kCb * kCb);
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;  // element (ta + 4 q, tb)
    const double s = J > p ? 1.0 : -1.0;
    // loads coalesced, row-major: the stored tile (p, J) or (J, p), the latter A_pJ transposed,
    // and the same of row p + 1, or T1_q where J = p: B_qp = -T1_q^T
    const double *A1 = J < p ? T.tile(p, J) : T.tile(J, p), *A2 = J < p ? T.tile(p + 1, J) : T.tile(J, p + 1);
    if (J == p) A2 = B.t1 + (int64_t)(p + 1) * (kCb * kCb);
    double yv[16], wv2[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int e = (ta + 4 * q) * kCb + tb;
        yv[q] = J != p ? A1[e] : 0.0;
        wv2[q] = two ? A2[e] : 0.0;
    }
    dbl4 acc[4], y[4];
    if (J != p) {
        tile_to_lds(P, S);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int a = ta + 4 * q;
            if (J < p) Y[a * kCbLd + tb] = yv[q];
            else Y[tb * kCbLd + a] = yv[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int a = ta + 4 * q;
            B.c1[o + a * kCb + tb] = -s * Y[a * kCbLd + tb];
        }
        cb_mfma(S, Y, acc);  // T1_J
        if (J > p) {
            cb_from_lds(Y, y);
            refine(P, gj_pivot(orig, G, p, 0), y, acc, S, Y);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) B.t1[o + cb_row(b, v) * kCb + cb_col(b)] = acc[b][v];
        if (!two) return;
        __syncthreads();
        cb_to_lds(acc, Y);
        tile_to_lds(L, S);
        __syncthreads();
        cb_mfma(S, Y, acc);  // L T1_J
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = ta + 4 * q;
        if (J < p) S[a * kCbLd + tb] = wv2[q];
        else S[tb * kCbLd + a] = wv2[q];
    }
    __syncthreads();
    cb_from_lds(S, y);
#pragma unroll
    for (int b = 0; b < 4; ++b) y[b] = J != p ? y[b] - acc[b] : -y[b];  // B_qJ
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) B.c2[o + cb_row(b, v) * kCb + cb_col(b)] = -s * y[b][v];
    cb_to_lds(y, Y);
    __syncthreads();
    tile_to_lds(P2, S);
    __syncthreads();
    cb_mfma(S, Y, acc);  // T2_J
    if (J > p + 1) refine(P2, gj_pivot(orig, G, p, 1), y, acc, S, Y);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) B.t2[o + cb_row(b, v) * kCb + cb_col(b)] = acc[b][v];
}

// The first count workgroups take the matrices' next pivot tiles (the longest ones: they also
// invert them), the others every other tile.  A tile is read and written once per two pivot
// tiles, past the caches (the row and column tiles, which every tile's products read, stay
// there), the products' operands come from memory and the four workgroups a CU holds hide it:
// eight blocks of 4150 unknowns take 337 us a pair, panel and second pivot 98 (as first written
// 350; operands staged through LDS, one pivot tile a pass: 605; without the bound on registers
// 455; with cached tiles 367).  Matrix cores and traffic alone would take 250 and 220.
__global__ __launch_bounds__(256, 4) void k_gjb_sweep(int p, const GjMat *__restrict__ mats, int count, double *W,
                                                   double *Pm, double *orig, double *cbuf, double *tbuf,
                                                   const double *__restrict__ diag0, int *fail) {
    __shared__ double S[kCb * kCbLd];
    const bool pivots = (int)blockIdx.x < count;
    const int64_t t = pivots ? 0 : xcd_remap((int)blockIdx.x - count, (int)gridDim.x - count);
    const int mi = pivots ? (int)blockIdx.x : gj_find<&GjMat::tile0>(mats, count, t);
    const GjMat G = mats[mi];
    int I = p + 2, J = p + 2;
    if (pivots) {
        if (I >= G.nt) return;
    } else {
        lower_tile(t - G.tile0, I, J);
        if (I == p + 2 && J == p + 2) return;
    }
    const bool two = p + 1 < G.nt;
    double *A = PackedTiles{W + G.tile0 * (kCb * kCb)}.tile(I, J);
    const GjBufs B = gj_bufs(G, cbuf, tbuf);
    const int64_t oi = (int64_t)I * (kCb * kCb), oj = (int64_t)J * (kCb * kCb);
    const int tb = threadIdx.x & 63, ta = threadIdx.x >> 6;  // element (ta + 4 q, tb)
    const int last = two ? p + 1 : p;  // the pivot row and column with no product after it
    if (I == last || J == last) {
        // pivot tile; row: T_J; column: -T_I^T (transposed through LDS)
        const double *tl = two ? B.t2 : B.t1;
        const double *src = I == last && J == last ? gj_pivot(Pm, G, p, two ? 1 : 0) : tl + (I == last ? oj : oi);
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = src[(ta + 4 * q) * kCb + tb];
        if (J == last && I != last) {
#pragma unroll
            for (int q = 0; q < 16; ++q) S[(ta + 4 * q) * kCbLd + tb] = v[q];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = -S[tb * kCbLd + ta + 4 * q];
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) A[(ta + 4 * q) * kCb + tb] = v[q];
        return;
    }
    const double *base = A;
    if (I == p) base = J == p ? gj_pivot(Pm, G, p, 0) : B.t1 + oj;
    else if (J == p) base = B.t1 + oi;
    const bool column = J == p && I != p;
    // of a diagonal tile only the lower half is kept: the wave of the quarter above it would start
    // from the quarter below, which another wave is overwriting, and has nothing to do
    const bool above = I == J && __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 1;
    // The products are summed by themselves and added to the tile at the end, one rounding at
    // its magnitude: sums that began with the tile made errors of M^-1 r at 800 unknowns three
    // times as large.
    dbl4 acc[4] = {};
    if (!above) {
        if (I != p && J != p) cb_fma(B.c1 + oi, B.t1 + oj, acc);
        if (two) cb_fma(B.c2 + oi, B.t2 + oj, acc);
        if (column || I == J) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int a = fma_row(b, v), c = fma_col(b);
                    // a diagonal tile's lower half
                    const double x = base[column || a < c ? c * kCb + a : a * kCb + c];
                    acc[b][v] += column ? -x : x;
                }
        } else {
#pragma unroll
            for (int b = 0; b < 4; b += 2)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const dbl2 x = __builtin_nontemporal_load((const dbl2 *)(base + fma_row(b, v) * kCb + fma_col(b)));
                    acc[b][v] += x.x;
                    acc[b + 1][v] += x.y;
                }
        }
#pragma unroll
        for (int b = 0; b < 4; b += 2)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                __builtin_nontemporal_store(dbl2{acc[b][v], acc[b + 1][v]},
                                            (dbl2 *)(A + fma_row(b, v) * kCb + fma_col(b)));
    }
    if (pivots) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[fma_row(b, v) * kCbLd + fma_col(b)] = acc[b][v];
        mirror_lower(S);
        double *Pn = gj_pivot(Pm, G, p + 2, 0), *On = gj_pivot(orig, G, p + 2, 0);
#pragma unroll
        for (int q = 0; q < 16; ++q) On[(ta + 4 * q) * kCb + tb] = S[(ta + 4 * q) * kCbLd + tb];
        __syncthreads();
        const bool bad = pivot_inverse64(S, diag0 + G.row0 * kCb, (int64_t)I * kCb, G.size);
#pragma unroll
        for (int q = 0; q < 16; ++q) Pn[(ta + 4 * q) * kCb + tb] = S[(ta + 4 * q) * kCbLd + tb];
        if (bad && threadIdx.x == 0) pivot_failed(fail, G.block);
    }
}

// Tile (I, J) of the inverse S X S (S the scale) from X's lower triangle (X: the 64 x 64 tile,
// row stride ldx, times sign), as the apply reads it: lower tiles of kDenseTile^2, diagonal
// ones whole, zero beyond the block.
__device__ __forceinline__ void store_inverse(const GjMat &G, int I, int J, const double *X, int ldx, double sign,
                                              const double *sc, double *__restrict__ dinv) {
    constexpr int T = kDenseTile;
    const int ntd = (G.size + T - 1) / T;
    for (int e = threadIdx.x; e < kCb * kCb; e += 256) {
        const int sub = e / (T * T), a = e / T % T, b = e % T;
        const int It = 2 * I + (sub >> 1), Jt = 2 * J + (sub & 1);
        if (It >= ntd || Jt > It) continue;
        const int r = It * T + a, c = Jt * T + b, hi = max(r, c), lo = min(r, c);
        double v = 0.0;
        if (hi < G.size) v = (sign * X[(hi - I * kCb) * ldx + lo - J * kCb] * sc[lo]) * sc[hi];
        dinv[G.out + ((int64_t)It * (It + 1) / 2 + Jt) * (T * T) + a * T + b] = v;
    }
}

// one workgroup per 64 x 64 tile
__global__ __launch_bounds__(256) void k_gjb_finish(const GjMat *__restrict__ mats, int count,
                                                    const double *__restrict__ W, const double *__restrict__ scale,
                                                    double *__restrict__ dinv) {
    const int mi = gj_find<&GjMat::tile0>(mats, count, blockIdx.x);
    const GjMat G = mats[mi];
    int I, J;
    lower_tile(blockIdx.x - G.tile0, I, J);
    store_inverse(G, I, J, W + (int64_t)blockIdx.x * (kCb * kCb), kCb, 1.0, scale + G.row0 * kCb, dinv);
}

// Rows [r0, min(r0 + 64, size)) of the block into the 64 x 64 tile S of columns [c0, c0 + 64),
// the entries with column <= row, zero elsewhere; with diag the rows' diagonal entries go there.
// Sixteen lanes per row.  Starts and ends with a barrier.
__device__ __forceinline__ void gather_tile(const GjMat &G, int r0, int c0, const int64_t *__restrict__ ptr,
                                            const int32_t *__restrict__ idx, const double *__restrict__ val,
                                            double *S, double *diag) {
    __syncthreads();
    for (int e = threadIdx.x; e < kCb * kCbLd; e += 256) S[e] = 0.0;
    __syncthreads();
    for (int i = r0 + (threadIdx.x >> 4); i < min(r0 + kCb, G.size); i += 16) {
        const int64_t g = (int64_t)G.start + i, e1 = ptr[g + 1];
        for (int64_t e = ptr[g] + (threadIdx.x & 15); e < e1; e += 16) {
            const int64_t c = (int64_t)idx[e] - G.start;
            if (c < c0 || c > i || (c >= c0 + kCb && c != i)) continue;
            const double v = val[e];
            if (c < c0 + kCb) S[(i - r0) * kCbLd + (int)c - c0] = v;
            if (diag && c == i) diag[i] = v;
        }
    }
    __syncthreads();
}

// S scaled, as gathered; a diagonal tile (r0 == c0) also gets the identity beyond the block and
// its upper half.  Ends with a barrier.
__device__ __forceinline__ void scale_tile(const GjMat &G, int r0, int c0, const double *sc, double *S) {
    for (int e = threadIdx.x; e < kCb * kCb; e += 256) {
        const int a = e / kCb, b = e % kCb, i = r0 + a, c = c0 + b;
        if (i < G.size) S[a * kCbLd + b] = (S[a * kCbLd + b] * sc[i]) * sc[c];
        else if (r0 == c0 && a == b) S[a * kCbLd + b] = 1.0;
    }
    if (r0 == c0) mirror_lower(S);
    else __syncthreads();
}

// The blocks of up to 64 (NT = 1) and up to 128 unknowns (NT = 2), one workgroup each from K's
// rows to the stored inverse with everything in LDS: no work buffers, one launch.  With
// A = [A_00, L^T; L, A_11] and P = A_00^-1, T = L P (refined once, as the sweeps' rows, with
// A_00 gathered again), P' = (A_11 - T L^T)^-1, V = P' T the inverse is [P + T^T V, -V^T; -V, P'].  Bound by the pivot inverses' chains; registers are not
// bounded further (spilling for four workgroups per CU took 0.1 ms more, blocks of 19 to 64).
// Setup of 180,000 unknowns in blocks of one size, in ms: here / by the 64-wide sweeps above /
// by sweeps of 32 pivots before them:
//   19: 0.83 / 1.41 / 1.00   32: 0.63 / 0.97 / 0.74   64: 0.58 / 0.75 / 0.89
//   65: 0.86 / 1.36 / 1.09   96: 0.77 / 1.11 / 0.88  128: 0.74 / 1.01 / 1.94
template <int NT>
__global__ __launch_bounds__(256, 2) void k_gjb_small(const GjMat *__restrict__ mats,
                                                      const int64_t *__restrict__ ptr,
                                                      const int32_t *__restrict__ idx,
                                                      const double *__restrict__ val, double *__restrict__ dinv,
                                                      int *fail) {
    __shared__ double S[NT][kCb * kCbLd], sc[NT * kCb], dg[NT * kCb];
    const GjMat G = mats[blockIdx.x];
    const int t = threadIdx.x;
    if (t < NT * kCb) dg[t] = 0.0;
    gather_tile(G, 0, 0, ptr, idx, val, S[0], dg);
    if constexpr (NT == 2) gather_tile(G, kCb, 0, ptr, idx, val, S[1], dg);
    if (t < NT * kCb) {
        const double d = dg[t];
        sc[t] = d > 0.0 ? 1.0 / sqrt(d) : 1.0;  // as k_dense_scale
        dg[t] = (d * sc[t]) * sc[t];
    }
    __syncthreads();
    scale_tile(G, 0, 0, sc, S[0]);
    if constexpr (NT == 2) scale_tile(G, kCb, 0, sc, S[1]);
    bool bad = pivot_inverse64(S[0], dg, 0, G.size);
    if constexpr (NT == 2) {
        dbl4 p[4], l[4], tt[4], acc[4];
        cb_from_lds(S[0], p);
        cb_from_lds(S[1], l);
        cb_mfma(S[1], S[0], tt);  // T = L P
        __syncthreads();
        cb_to_lds(tt, S[1]);
        gather_tile(G, 0, 0, ptr, idx, val, S[0], nullptr);
        scale_tile(G, 0, 0, sc, S[0]);
        cb_mfma(S[1], S[0], acc);  // T A_00
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b] = l[b] - acc[b];
        cb_to_lds(acc, S[1]);
        cb_to_lds(p, S[0]);
        __syncthreads();
        cb_mfma(S[1], S[0], acc);  // (L - T A_00) P
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 4; ++b) tt[b] += acc[b];
        cb_to_lds(tt, S[0]);
        cb_to_lds(l, S[1]);
        __syncthreads();
        cb_mfma<false, true>(S[0], S[1], acc);  // T L^T
        gather_tile(G, kCb, kCb, ptr, idx, val, S[1], nullptr);
        scale_tile(G, kCb, kCb, sc, S[1]);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[1][cb_row(b, v) * kCbLd + cb_col(b)] -= acc[b][v];
        mirror_lower(S[1]);
        bad |= pivot_inverse64(S[1], dg, kCb, G.size);
        store_inverse(G, 1, 1, S[1], kCbLd, 1.0, sc, dinv);
        cb_mfma(S[1], S[0], acc);  // V = P' T
        __syncthreads();
        cb_to_lds(acc, S[1]);
        __syncthreads();
        store_inverse(G, 1, 0, S[1], kCbLd, -1.0, sc, dinv);
        cb_mfma<true, false>(S[0], S[1], acc);  // T^T V
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 4; ++b) p[b] += acc[b];
        cb_to_lds(p, S[0]);
        __syncthreads();
    }
    store_inverse(G, 0, 0, S[0], kCbLd, 1.0, sc, dinv);
    if (bad && t == 0) pivot_failed(fail, G.block);
}

__global__ void k_to_i64(const int32_t *__restrict__ a, int64_t n, int64_t *__restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = a[i];
}

__global__ void k_to_f32_s(const double *__restrict__ a, int64_t n, float *__restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (float)a[i];
}

// flag = first block row whose block count differs from the stored row pointer
__global__ void k_cmp_counts(int32_t nb, const int64_t *__restrict__ cnt, const int32_t *__restrict__ bptr,
                             int *flag) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < nb; r += (int64_t)gridDim.x * blockDim.x)
        if (cnt[r] != (int64_t)(bptr[r + 1] - bptr[r])) atomicMin(flag, (int)r);
}

// flag = 0 when a[i] != b[i] for some i
__global__ void k_cmp_i32(int64_t n, const int32_t *__restrict__ a, const int32_t *__restrict__ b, int *flag) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        if (a[i] != b[i]) atomicMin(flag, 0);
}

// ---------------------------------------------------------------- host helpers
// Scratch of one setup call; released (to the cache) once the stream is idle.
struct Pool {
    dpcg_ctx *c;
    std::vector<void *> scratch;
    std::vector<void *> pinned;  // host read-back buffers (pinned, so the copies stay asynchronous)
    // work enqueued on the side stream after fork() runs beside the main stream from that
    // point on; join() makes the main stream wait for all of it
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    bool pending = false;
    ~Pool() {
        if (pending) (void)hipStreamSynchronize(side);
        (void)hipStreamSynchronize(c->stream);
        for (void *p : scratch) dev_release(p);
        for (void *p : pinned) host_release(p);
        sync_event_give(ev_fork);
        sync_event_give(ev_join);
    }
    hipError_t fork(hipStream_t *sb) {
        hipError_t e = side_stream(&side);
        if (e == hipSuccess && !ev_fork) e = sync_event_take(&ev_fork);
        if (e == hipSuccess && !ev_join) e = sync_event_take(&ev_join);
        if (e == hipSuccess) e = hipEventRecord(ev_fork, c->stream);
        if (e == hipSuccess) e = hipStreamWaitEvent(side, ev_fork, 0);
        if (e != hipSuccess) return e;
        pending = true;
        *sb = side;
        return hipSuccess;
    }
    hipError_t join() {
        if (!pending) return hipSuccess;
        hipError_t e = hipEventRecord(ev_join, side);
        if (e == hipSuccess) e = hipStreamWaitEvent(c->stream, ev_join, 0);
        if (e == hipSuccess) pending = false;
        return e;
    }
    template <class T>
    hipError_t host(T **p, size_t count) {
        void *q = nullptr;
        hipError_t e = host_alloc(&q, std::max<size_t>(1, count) * sizeof(T));
        if (e == hipSuccess) pinned.push_back(q);
        *p = (T *)q;
        return e;
    }
    template <class T>
    hipError_t tmp(T **p, size_t count) {
        void *q = nullptr;
        hipError_t e = dev_alloc(&q, std::max<size_t>(1, count) * sizeof(T));
        if (e == hipSuccess) scratch.push_back(q);
        *p = (T *)q;
        return e;
    }
};

template <class T>
hipError_t keep(dpcg_ctx *c, T **p, size_t count) {
    void *q = nullptr;
    const size_t bytes = std::max<size_t>(1, count) * sizeof(T);
    hipError_t e = dev_alloc(&q, bytes);
    if (e == hipSuccess) {
        c->allocations.push_back(q);
        c->device_bytes += (int64_t)bytes;
    }
    *p = (T *)q;
    return e;
}

int grid_for(int64_t work, int per = 256, int cap = 8192) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(cap, (work + per - 1) / per));
}

// Checks a CSR matrix (rows x cols, nnz entries) into *flag; with mx, also max |value|
// into (*mx)[0] (scratch from the pool).
hipError_t check_csr(hipStream_t s, Pool &pool, int64_t rows, int64_t cols, const int64_t *ptr, const int32_t *idx,
                     const double *val, int64_t nnz, int *flag, double **mx) {
    uint32_t *bits = nullptr;
    hipError_t e = pool.tmp(&bits, nnz / 32 + 1);
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(bits, 0, sizeof(uint32_t) * (size_t)(nnz / 32 + 1), s);
    if (e != hipSuccess) return e;
    const int ge = grid_for(nnz, 256, 4096);
    double *part = nullptr;
    if (mx) {
        e = pool.tmp(&part, ge);
        if (e != hipSuccess) return e;
        *mx = part;
    }
    hipLaunchKernelGGL(k_csr_rows, dim3(grid_for(rows, 256, 4096)), dim3(256), 0, s, rows, ptr, nnz, bits, flag);
    hipLaunchKernelGGL(k_csr_entries, dim3(ge), dim3(256), 0, s, rows, cols, ptr, idx, val, nnz,
                       (const uint32_t *)bits, flag, part);
    if (mx) hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(256), 0, s, part, ge);
    return hipGetLastError();
}

// out[0..n] = exclusive scan of a[0..n); tmp holds the chunk partials.
hipError_t scan(hipStream_t s, const int64_t *a, int64_t n, int64_t *out, int64_t *part) {
    const int chunks = (int)std::max<int64_t>(1, (n + kScanChunk - 1) / kScanChunk);
    hipLaunchKernelGGL(k_scan_partials, dim3(chunks), dim3(256), 0, s, a, n, part);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, s, part, chunks);
    hipLaunchKernelGGL(k_scan_apply, dim3(chunks), dim3(256), 0, s, a, n, part, out);
    return hipGetLastError();
}

#define HT(expr)                                       \
    do {                                               \
        if ((expr) != hipSuccess) return DPCG_EHIP;    \
    } while (0)

// K Z (as (KZ)^T) and E = Z^T K Z in batches of kBatch deflation vectors, then E^-1 by
// blocked Gauss-Jordan sweeps.  Inputs: Z (int64 row pointer), Z^T (int64 pointer), the
// row windows of K z_j (wlo on the device, ws on the host).  reuse: the arrays of a
// previous build are overwritten (same structure) instead of allocated.
int coarse_operator(dpcg_ctx *c, Pool &pool, int32_t k, const int64_t *zp, const int32_t *zc, const int64_t *ztp,
                    const int32_t *zti, const double *ztv, const int64_t *wl, const int64_t *ws, int64_t *part,
                    int *flags, int64_t *bad, bool reuse) {
    hipStream_t s = c->stream;
    int *fl = nullptr;  // pinned read-backs: fl[0..4), nkz, cf
    int64_t *nkzp = nullptr;
    HT(pool.host(&fl, 5));
    HT(pool.host(&nkzp, 1));
    {
        // ---- K Z and E, in batches of kBatch vectors; batch groups bound the scratch ----
        // (wl, ws: host copies of the row windows of K z_j)
        const int nbat = (k + kBatch - 1) / kBatch;
        const int words = (k + 31) / 32;
        std::vector<KzBatch> bt(nbat);
        int64_t slices = 0;
        for (int bi = 0; bi < nbat; ++bi) {
            KzBatch &B = bt[bi];
            B.j0 = (int64_t)bi * kBatch;
            B.ncol = std::min<int64_t>(kBatch, k - B.j0);
            int64_t lo = INT64_MAX, hi = -1;
            for (int64_t j = B.j0; j < B.j0 + B.ncol; ++j)
                if (ws[j] > 0) {
                    lo = std::min(lo, wl[j]);
                    hi = std::max(hi, wl[j] + ws[j]);
                }
            B.lo3 = hi > 0 ? lo / 3 : 0;
            B.w3 = hi > 0 ? (hi + 2) / 3 - B.lo3 : 0;
            B.nslice = std::max<int64_t>(1, (B.w3 + kSlice - 1) / kSlice);
            B.slice0 = slices;
            slices += B.nslice;
        }
        // group consecutive batches so that a group's scratch (the dense z and K z of its
        // windows) stays under the budget: 8 GB, under 3% of the device's memory, so that
        // a large system takes few groups, whose launches fill the device better (at 80^3
        // two groups instead of sixteen with 1 GB: 4.7 against 7.7 ms of these kernels)
        const int64_t per_triplet = 2 * 3 * kBatch * sizeof(double) + 3 * sizeof(uint32_t);
        const int64_t budget = int64_t(8) << 30;
        std::vector<int> gcut{0};
        int64_t acc_w = 0, max_group_w = 0, total_w = 0;
        int max_group_nb = 0;
        for (int bi = 0; bi < nbat; ++bi) {
            if (acc_w > 0 && (acc_w + bt[bi].w3) * per_triplet > budget) {
                gcut.push_back(bi);
                acc_w = 0;
            }
            bt[bi].off3 = acc_w;
            bt[bi].moff = total_w;
            total_w += bt[bi].w3;
            bt[bi].bit0 = (int64_t)(bi - gcut.back()) * words;
            acc_w += bt[bi].w3;
            max_group_w = std::max(max_group_w, acc_w);
            max_group_nb = std::max(max_group_nb, bi - gcut.back() + 1);
        }
        gcut.push_back(nbat);
        KzBatch *bt_d = nullptr;
        int32_t *scnt = nullptr, *soff = nullptr, *tcnt = nullptr;
        int64_t *kzcnt = nullptr, *kzp = nullptr;
        double *zd = nullptr, *kd = nullptr;
        uint32_t *mk = nullptr, *rbits = nullptr, *km = nullptr, *ends = nullptr, *touched = nullptr;
        HT(pool.tmp(&bt_d, nbat));
        HT(hipMemcpyAsync(bt_d, bt.data(), sizeof(KzBatch) * nbat, hipMemcpyHostToDevice, s));
        HT(pool.tmp(&scnt, slices * kBatch));
        HT(pool.tmp(&tcnt, slices));
        HT(pool.tmp(&soff, slices * kBatch));
        HT(pool.tmp(&kzcnt, k));
        HT(pool.tmp(&kzp, k + 1));
        HT(pool.tmp(&zd, 3 * max_group_w * kBatch));
        HT(pool.tmp(&kd, 3 * max_group_w * kBatch));
        // the structure masks of every batch at once (4 bytes per window triplet each):
        // the values pass of a call with several groups then needs no second marking
        HT(pool.tmp(&mk, std::max<int64_t>(1, total_w)));
        HT(pool.tmp(&rbits, std::max<int64_t>(1, total_w)));
        HT(pool.tmp(&km, std::max<int64_t>(1, total_w)));
        HT(pool.tmp(&ends, nbat));
        HT(pool.tmp(&touched, (int64_t)max_group_nb * words));
        int32_t *icnt = nullptr;
        int64_t *nitems = nullptr;
        KzItem *items = nullptr;
        HT(pool.tmp(&icnt, slices));
        HT(pool.tmp(&nitems, nbat));
        HT(pool.tmp(&items, max_group_w));
        auto max_slices = [&](int g0, int g1) {
            int64_t m = 1;
            for (int bi = g0; bi < g1; ++bi) m = std::max(m, bt[bi].nslice);
            return (int)m;
        };
        // full: the count pass (masks cleared, z scattered, structure marked); otherwise the
        // values pass of a later group, which only needs its z rows again (the scatter's
        // bits are already in rbits) and clear touched bits
        auto prepare = [&](int g0, int g1, bool full) {
            const dim3 gs(max_slices(g0, g1), g1 - g0);
            hipLaunchKernelGGL(k_kzb_init, gs, dim3(256), 0, s, bt_d + g0, words, mk, rbits, touched,
                               ends + g0, full ? 1 : 0);
            hipLaunchKernelGGL(k_kzb_scatter, dim3(kBatch, g1 - g0), dim3(256), 0, s, bt_d + g0, ztp, zti, ztv, zd,
                               rbits);
            if (full) hipLaunchKernelGGL(k_kzb_mark, gs, dim3(256), 0, s, bt_d + g0, c->brow_ptr, c->bcol, rbits, mk);
        };
        for (size_t g = 0; g + 1 < gcut.size(); ++g) {
            prepare(gcut[g], gcut[g + 1], true);
            hipLaunchKernelGGL(k_kzb_count, dim3(max_slices(gcut[g], gcut[g + 1]), gcut[g + 1] - gcut[g]), dim3(256),
                               0, s, bt_d + gcut[g], mk, (const uint32_t *)nullptr, scnt, tcnt, ends + gcut[g]);
        }
        hipLaunchKernelGGL(k_kzb_offsets, dim3(nbat), dim3(kBatch + 1), 0, s, bt_d, nbat, scnt, tcnt, soff, kzcnt,
                           icnt, nitems);
        HT(scan(s, kzcnt, k, kzp, part));
        HT(hipMemcpyAsync(nkzp, kzp + k, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        int64_t *zp_h = nullptr, *kp_h = nullptr;  // list lengths for the restriction's column order
        if (!reuse) {
            HT(pool.host(&zp_h, k + 1));
            HT(pool.host(&kp_h, k + 1));
            HT(hipMemcpyAsync(zp_h, ztp, sizeof(int64_t) * (k + 1), hipMemcpyDeviceToHost, s));
            HT(hipMemcpyAsync(kp_h, kzp, sizeof(int64_t) * (k + 1), hipMemcpyDeviceToHost, s));
        }
        HT(pool.join());  // the symmetry and block flags are read here
        HT(hipMemcpyAsync(fl, flags, sizeof(int) * 4, hipMemcpyDeviceToHost, s));
        HT(hipStreamSynchronize(s));
        const int64_t nkz = *nkzp;
        if (fl[3] != INT32_MAX) return DPCG_ENOTSYM;
        if (fl[1] != INT32_MAX) {
            *bad = fl[1];
            return DPCG_EBLOCK_NOT_SPD;
        }
        if (nkz > (int64_t)INT32_MAX) return DPCG_EINVAL;
        if (reuse && nkz != c->kz_structure) return DPCG_EINVAL;  // the structure of K Z must not change
        c->kz_structure = nkz;
        if (!reuse) {
            // the restriction's column order: columns needing more rounds of its loads first,
            // launch order kept within each class (neighbouring columns share their gathers)
            // (a counting sort: classes of 0 .. 63 rounds and one of 64 or more)
            constexpr int kCls = 64;
            std::vector<int32_t> cls(k), start(kCls + 2, 0);
            for (int32_t j = 0; j < k; ++j) {
                const int64_t len = zp_h[j + 1] - zp_h[j] + kp_h[j + 1] - kp_h[j];
                const int64_t r = std::min<int64_t>((len + kRestrictRound - 1) / kRestrictRound, kCls);
                cls[j] = kCls - (int32_t)r;  // more rounds, earlier class
                ++start[cls[j] + 1];
            }
            for (int q = 0; q <= kCls; ++q) start[q + 1] += start[q];
            c->rs_order_h.resize(k);
            for (int32_t j = 0; j < k; ++j) c->rs_order_h[start[cls[j]]++] = j;
        }
        if (!reuse) {
            HT(keep(c, &c->kzt_idx, nkz));
            HT(keep(c, &c->kzt_val, nkz));
        }
        const int64_t ld = ((int64_t)k + kCb - 1) / kCb * kCb;
        c->einv_ld = ld;
        double *eraw = nullptr, *ga = nullptr, *diag0 = nullptr, *pv = nullptr;
        HT(pool.tmp(&eraw, ld * ld));
        HT(hipMemsetAsync(eraw, 0, sizeof(double) * ld * ld, s));
        for (size_t g = 0; g + 1 < gcut.size(); ++g) {
            const int g0 = gcut[g], g1 = gcut[g + 1];
            if (gcut.size() > 2) prepare(g0, g1, false);  // one group: the count pass left it ready
            const dim3 gs(max_slices(g0, g1), g1 - g0);
            hipLaunchKernelGGL(k_kzb_items, gs, dim3(256), 0, s, bt_d + g0, mk, icnt, items);
            hipLaunchKernelGGL(k_kzb_values, dim3(512, g1 - g0), dim3(256),
                               0, s, bt_d + g0, nitems + g0, items, c->brow_ptr, c->bcol, c->bval, zd, rbits, zp, zc,
                               kd, km, ends + g0, words, touched);
            // the kept entries' places (those of later groups' vectors come after them)
            hipLaunchKernelGGL(k_kzb_count, gs, dim3(256), 0, s, bt_d + g0, mk, (const uint32_t *)km, scnt, tcnt,
                               (uint32_t *)nullptr);
            hipLaunchKernelGGL(k_kzb_offsets, dim3(g1 - g0), dim3(kBatch + 1), 0, s, bt_d + g0, g1 - g0, scnt, tcnt,
                               soff, kzcnt, icnt, nitems + g0);
            HT(scan(s, kzcnt, k, kzp, part));
            hipLaunchKernelGGL(k_kzb_store, gs, dim3(256), 0, s, bt_d + g0, mk, km, soff, kzp, kd, c->kzt_idx,
                               c->kzt_val);
            hipLaunchKernelGGL(k_kzb_erows, dim3((k + 3) / 4, g1 - g0), dim3(256), 0, s, bt_d + g0, k, ztp, zti, ztv,
                               kd, mk, touched, eraw, ld);
        }
        HT(hipGetLastError());
        // ---- E^-1 ----
        HT(pool.tmp(&ga, ld * ld));
        if (!reuse) HT(keep(c, &c->einv, ld * ld));
        double *esc = nullptr;
        HT(pool.tmp(&diag0, ld));
        HT(pool.tmp(&esc, ld));
        HT(pool.tmp(&pv, 2 * kCb * kCb));
        hipLaunchKernelGGL(k_symmetrise, dim3(grid_for(ld * ld)), dim3(256), 0, s, k, ld, eraw, ga, diag0, esc);
        int *cfail = flags + 2;
        HT(hipMemsetAsync(cfail, 0, sizeof(int), s));
        const int nt = (int)(ld / kCb);
        double *cbuf = nullptr, *tbuf = nullptr;
        HT(pool.tmp(&cbuf, ld * kCb));
        HT(pool.tmp(&tbuf, ld * kCb));
        hipLaunchKernelGGL(k_cgj_first_pivot, dim3(1), dim3(256), 0, s, ga, ld, k, diag0, pv, cfail);
        for (int p = 0; p < nt; ++p) {
            const double *pc = pv + (p & 1) * kCb * kCb;
            hipLaunchKernelGGL(k_cgj_panel, dim3(nt), dim3(256), 0, s, p, ga, ld, pc, cbuf, tbuf);
            hipLaunchKernelGGL(k_cgj_sweep, dim3((unsigned)coarse_tile_count(nt)), dim3(256), 0, s, p, nt, ga, ld, k, pc,
                               pv + ((p + 1) & 1) * kCb * kCb, (const double *)cbuf, (const double *)tbuf, diag0,
                               cfail);
        }
        // E^-1 from the lower tiles, and its lower-triangle tiles for the solve's coarse product
        const int32_t cnt = (int32_t)((k + kCoarseTile - 1) / kCoarseTile);
        c->coarse_nt = cnt;
        if (!reuse) HT(keep(c, &c->einv_tiles, coarse_tile_count(cnt) * kCoarseTile * kCoarseTile));
        hipLaunchKernelGGL(k_einv_from_lower, dim3((unsigned)coarse_tile_count(cnt)), dim3(256), 0, s, k, ld,
                           (const double *)esc, (const double *)ga, c->einv, c->einv_tiles);
        HT(hipGetLastError());
        if (!reuse) HT(keep(c, &c->kzt_ptr, k + 1));
        hipLaunchKernelGGL(k_to_i32, dim3(grid_for(k + 1)), dim3(256), 0, s, kzp, (int64_t)k + 1, c->kzt_ptr);
        HT(hipMemcpyAsync(nkzp, kzp + k, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        if (c->bws) c->bws->stale = true;  // its restriction lists follow (KZ)^T's pattern
        if (!reuse) {
            HT(keep(c, &c->rs_order, k));
            HT(hipMemcpyAsync(c->rs_order, c->rs_order_h.data(), sizeof(int32_t) * k, hipMemcpyHostToDevice, s));
        }
        HT(hipMemcpyAsync(fl + 4, cfail, sizeof(int), hipMemcpyDeviceToHost, s));
        HT(hipStreamSynchronize(s));
        c->nnz_kz = *nkzp;
        if (fl[4]) return DPCG_ECOARSE_NOT_SPD;
        return DPCG_OK;
    }
}

// Inverses of the dense blocks which[] (indices into c->dense_h), written to c->dinv.
// A block that is not SPD to working precision lowers *bad_flag to its block index.
int dense_inverses(dpcg_ctx *c, Pool &pool, const int64_t *kp, const int32_t *kc, const double *kv,
                   const std::vector<int32_t> &which, int *bad_flag) {
    hipStream_t s = c->stream;
    const int count = (int)which.size();
    if (count == 0) return DPCG_OK;
    std::vector<GjMat> m(count);
    for (int i = 0; i < count; ++i) {
        const DenseBlk &D = c->dense_h[which[i]];
        m[i] = GjMat{0, 0, D.off, (D.size + kCb - 1) / kCb, D.size, D.start, D.block};
    }
    std::stable_sort(m.begin(), m.end(), [](const GjMat &a, const GjMat &b) { return a.nt > b.nt; });
    // most tiles first: [0, big) take the sweeps, then the blocks of two tiles and of one
    int big = 0, one = count;
    while (big < count && m[big].nt > 2) ++big;
    while (one > big && m[one - 1].nt == 1) --one;
    std::vector<int64_t> tiles(big + 1, 0), rows(big + 1, 0);
    int64_t bufs = 0, pivs = 0;
    for (int i = 0; i < big; ++i) {
        m[i].tile0 = tiles[i];
        m[i].row0 = rows[i];
        m[i].buf0 = bufs;
        m[i].piv0 = pivs;
        bufs += 2 * m[i].nt;
        pivs += std::min(m[i].nt, 4);
        tiles[i + 1] = tiles[i] + coarse_tile_count(m[i].nt);
        rows[i + 1] = rows[i] + m[i].nt;
    }
    GjMat *md = nullptr;
    HT(pool.tmp(&md, count));
    HT(hipMemcpyAsync(md, m.data(), sizeof(GjMat) * count, hipMemcpyHostToDevice, s));
    if (one > big)
        hipLaunchKernelGGL(k_gjb_small<2>, dim3(one - big), dim3(256), 0, s, (const GjMat *)md + big, kp, kc, kv,
                           c->dinv, bad_flag);
    if (count > one)
        hipLaunchKernelGGL(k_gjb_small<1>, dim3(count - one), dim3(256), 0, s, (const GjMat *)md + one, kp, kc, kv,
                           c->dinv, bad_flag);
    HT(hipGetLastError());
    if (big == 0) return DPCG_OK;
    constexpr int64_t kTile = kCb * kCb;
    double *W = nullptr, *diag0 = nullptr, *scale = nullptr, *pv = nullptr, *orig = nullptr, *cbuf = nullptr,
           *tbuf = nullptr;
    HT(pool.tmp(&W, tiles[big] * kTile));
    HT(pool.tmp(&diag0, rows[big] * kCb));
    HT(pool.tmp(&scale, rows[big] * kCb));
    HT(pool.tmp(&pv, pivs * kTile));
    HT(pool.tmp(&orig, pivs * kTile));
    HT(pool.tmp(&cbuf, bufs * kTile));
    HT(pool.tmp(&tbuf, bufs * kTile));
    HT(hipMemsetAsync(diag0, 0, sizeof(double) * rows[big] * kCb, s));
    HT(hipMemsetAsync(W, 0, sizeof(double) * tiles[big] * kTile, s));
    const int gy = std::min(big, 65535);
    hipLaunchKernelGGL(k_dense_scale, dim3((m[0].nt * kCb + 255) / 256, gy), dim3(256), 0, s, md, big, kp, kc, kv,
                       scale);
    hipLaunchKernelGGL(k_dense_gather, dim3((m[0].nt * kCb + 15) / 16, gy), dim3(256), 0, s, md, big, kp, kc, kv, scale, W, diag0);
    hipLaunchKernelGGL(k_gjb_first_pivot, dim3(gy), dim3(256), 0, s, md, big, W, diag0, pv, orig,
                       bad_flag);
    int active = big, active2 = big;
    for (int p = 0; p < m[0].nt; p += 2) {
        while (active > 0 && m[active - 1].nt <= p) --active;
        while (active2 > 0 && m[active2 - 1].nt <= p + 1) --active2;
        if (active2 > 0)
            hipLaunchKernelGGL(k_gjb_pivot2, dim3(std::min(active2, 65535)), dim3(256), 0, s, p, md, active2, W, pv,
                               orig, cbuf, tbuf, diag0, bad_flag);
        hipLaunchKernelGGL(k_gjb_panel, dim3((unsigned)rows[active]), dim3(256), 0, s, p, md, active, W, pv, orig,
                           cbuf, tbuf);
        hipLaunchKernelGGL(k_gjb_sweep, dim3((unsigned)(tiles[active] + active)), dim3(256), 0, s, p, md, active, W, pv,
                           orig, cbuf, tbuf, diag0, bad_flag);
    }
    hipLaunchKernelGGL(k_gjb_finish, dim3((unsigned)tiles[big]), dim3(256), 0, s, md, big, W, scale, c->dinv);
    HT(hipGetLastError());
    return DPCG_OK;
}

// The dense-block tables from the host copy of the partition: extents, offsets in dinv, and
// the apply's strips and tile rows.
int dense_tables(dpcg_ctx *c, const int32_t *bph, int32_t nblocks) {
    hipStream_t s = c->stream;
    c->dense_h.clear();
    int64_t tiles = 0;
    for (int32_t b = 0; b < nblocks; ++b) {
        const int32_t m = bph[b + 1] - bph[b];
        if (m <= kMaxBlock) continue;
        c->dense_h.push_back(DenseBlk{tiles * kDenseTile * kDenseTile, tiles, bph[b], m, (int32_t)b, 0});
        tiles += coarse_tile_count((m + kDenseTile - 1) / kDenseTile);
    }
    std::vector<DenseStrip> st;
    std::vector<DenseRow> rows;
    for (size_t i = 0; i < c->dense_h.size(); ++i) {
        const int32_t nt = (c->dense_h[i].size + kDenseTile - 1) / kDenseTile;
        for (int32_t I = 0; I < nt; ++I) {
            rows.push_back(DenseRow{(int32_t)i, I, (int32_t)st.size(), 0});
            for (int32_t j = 0; j <= I; j += kDenseStrip) st.push_back(DenseStrip{(int32_t)i, I, j, 0});
            rows.back().strip1 = (int32_t)st.size();
        }
    }
    c->ndense = (int32_t)c->dense_h.size();
    c->ndstrips = (int32_t)st.size();
    c->ndrows = (int32_t)rows.size();
    c->dense_tiles = tiles;
    c->dinv_len = tiles * kDenseTile * kDenseTile;
    HT(keep(c, &c->dense, c->ndense));
    HT(keep(c, &c->dstrip, c->ndstrips));
    HT(keep(c, &c->drow, c->ndrows));
    HT(keep(c, &c->dinv, c->dinv_len));
    HT(keep(c, &c->dpart, (tiles + c->ndstrips) * kDenseTile));
    HT(hipMemcpyAsync(c->dense, c->dense_h.data(), sizeof(DenseBlk) * c->ndense, hipMemcpyHostToDevice, s));
    HT(hipMemcpyAsync(c->dstrip, st.data(), sizeof(DenseStrip) * c->ndstrips, hipMemcpyHostToDevice, s));
    HT(hipMemcpyAsync(c->drow, rows.data(), sizeof(DenseRow) * c->ndrows, hipMemcpyHostToDevice, s));
    HT(hipStreamSynchronize(s));  // st and rows are host temporaries
    return DPCG_OK;
}

}  // namespace

int gpu_setup(dpcg_ctx *c, int64_t n, const int64_t *kp, const int32_t *kc, const double *kv, int32_t k,
              const int64_t *zp, const int32_t *zc, const double *zv, int32_t nblocks, const int32_t *bp,
              int64_t *bad) {
    hipStream_t s = c->stream;
    Pool pool{c, {}};
    // ---- sizes ----
    int64_t *ends = nullptr;  // pinned read-backs of the setup
    int *fl = nullptr;
    int64_t *tot = nullptr;
    HT(pool.host(&ends, 4));
    HT(pool.host(&fl, 5));
    HT(pool.host(&tot, 2));
    ends[2] = ends[3] = 0;
    HT(hipMemcpyAsync(&ends[0], kp, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HT(hipMemcpyAsync(&ends[1], kp + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    if (k > 0) {
        HT(hipMemcpyAsync(&ends[2], zp, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        HT(hipMemcpyAsync(&ends[3], zp + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    }
    HT(hipStreamSynchronize(s));
    const int64_t nnz = ends[1], nnz_z = k > 0 ? ends[3] : 0;
    if (ends[0] != 0 || nnz < 0 || nnz > (int64_t)INT32_MAX || ends[2] != 0 || nnz_z < 0 ||
        nnz_z > (int64_t)INT32_MAX)
        return DPCG_EINVAL;
    c->nnz = nnz;
    c->nnz_z = nnz_z;
    // ---- validation ----
    const double *maxpart = nullptr;
    int nmaxpart = 0;
    int *flags = nullptr;
    HT(pool.tmp(&flags, 5));
    const int init_flags[5] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX, 0};  // [4]: largest block above kMaxBlock
    HT(hipMemcpyAsync(flags, init_flags, sizeof(init_flags), hipMemcpyHostToDevice, s));
    double *mxk = nullptr;
    HT(check_csr(s, pool, n, n, kp, kc, kv, nnz, flags, &mxk));
    if (k > 0) HT(check_csr(s, pool, n, (int64_t)k, zp, zc, zv, nnz_z, flags + 1, nullptr));
    hipLaunchKernelGGL(k_check_blocks, dim3(grid_for(nblocks)), dim3(256), 0, s, nblocks, bp, n, flags + 2,
                       flags + 4);
    HT(hipGetLastError());
    HT(hipMemcpyAsync(fl, flags, sizeof(int) * 5, hipMemcpyDeviceToHost, s));
    HT(hipStreamSynchronize(s));
    if (fl[2] != INT32_MAX) *bad = fl[2];
    if (fl[0] != INT32_MAX || fl[1] != INT32_MAX || fl[2] != INT32_MAX) return DPCG_EINVAL;
    if (fl[4] > kMaxBlock) {
        int32_t *bph = nullptr;
        HT(pool.host(&bph, nblocks + 1));
        HT(hipMemcpyAsync(bph, bp, sizeof(int32_t) * (nblocks + 1), hipMemcpyDeviceToHost, s));
        HT(hipStreamSynchronize(s));
        const int st = dense_tables(c, bph, nblocks);
        if (st != DPCG_OK) return st;
    }
    maxpart = mxk;
    nmaxpart = 1;  // the maximum of |K| over all entries, in mxk[0]
    // ---- block-CSR counts, block-Jacobi offsets, Z^T, windows ----
    const int32_t nb = c->nb;
    int64_t *cnt = nullptr, *bptr64 = nullptr, *part = nullptr;
    const int64_t scan_parts = std::max<int64_t>({nb, nblocks, (int64_t)k, 1}) / kScanChunk + 2;
    HT(pool.tmp(&cnt, std::max<int64_t>({nb, nblocks, (int64_t)k}) + 1));
    HT(pool.tmp(&bptr64, nb + 1));
    HT(pool.tmp(&part, scan_parts));
    hipLaunchKernelGGL((k_bsr<false>), dim3(grid_for(nb, 4)), dim3(256), 0, s, nb, kp, kc, kv, cnt, nullptr, nullptr,
                       nullptr, nullptr);
    HT(scan(s, cnt, nb, bptr64, part));
    int64_t *moff = nullptr, *sq = nullptr;
    HT(pool.tmp(&moff, nblocks + 1));
    HT(pool.tmp(&sq, nblocks));
    hipLaunchKernelGGL(k_block_sq, dim3(grid_for(nblocks)), dim3(256), 0, s, nblocks, bp, sq);
    int64_t *part2 = nullptr;
    HT(pool.tmp(&part2, scan_parts));
    HT(scan(s, sq, nblocks, moff, part2));
    int64_t *ztp = nullptr, *wlo = nullptr, *wsize = nullptr;
    int32_t *zti = nullptr;
    double *ztv = nullptr;
    if (k > 0) {
        // chunks of Z's entries: at most 1024, and at most 4M (column, chunk) pairs
        const int64_t nch_cap = std::max<int64_t>(1, std::min<int64_t>(1024, ((int64_t)1 << 22) / k));
        const int64_t per = std::max<int64_t>(256, (nnz_z + nch_cap - 1) / nch_cap);
        const int nch = (int)std::max<int64_t>(1, (nnz_z + per - 1) / per);
        const int nranges = (int)((k + kZtCols - 1) / kZtCols);
        const int64_t pairs = (int64_t)k * nch;
        int64_t *cnt = nullptr, *off = nullptr, *part3 = nullptr;
        int32_t *erow = nullptr;
        HT(pool.tmp(&cnt, pairs));
        HT(pool.tmp(&off, pairs + 1));
        HT(pool.tmp(&part3, pairs / kScanChunk + 2));
        HT(pool.tmp(&erow, nnz_z));
        HT(pool.tmp(&ztp, k + 1));
        HT(keep(c, &c->zt_idx, nnz_z));
        HT(keep(c, &c->zt_val, nnz_z));
        zti = c->zt_idx;
        ztv = c->zt_val;
        const int cols_lds = std::min<int>(k, kZtCols);
        hipLaunchKernelGGL(k_entry_rows, dim3(grid_for(n)), dim3(256), 0, s, n, zp, erow);
        hipLaunchKernelGGL(k_zt_count, dim3(nch, nranges), dim3(256), sizeof(int32_t) * cols_lds, s, nnz_z, per, nch,
                           k, zc, cnt);
        HT(scan(s, cnt, pairs, off, part3));
        hipLaunchKernelGGL(k_zt_ptr, dim3(grid_for(k + 1)), dim3(256), 0, s, k, nch, off, ztp);
        hipLaunchKernelGGL(k_zt_place, dim3(nch, nranges), dim3(64), sizeof(int64_t) * cols_lds, s, nnz_z, per, nch, k,
                           zc, zv, erow, off, zti, ztv);
        HT(pool.tmp(&wlo, k));
        HT(pool.tmp(&wsize, k));
        hipLaunchKernelGGL(k_kz_window, dim3(k), dim3(256), 0, s, k, ztp, zti, kp, kc, wlo, wsize);
        HT(hipGetLastError());
    }
    int64_t *ws = nullptr, *wl = nullptr;
    HT(pool.host(&ws, k));
    HT(pool.host(&wl, k));
    HT(hipMemcpyAsync(&tot[0], bptr64 + nb, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HT(hipMemcpyAsync(&tot[1], moff + nblocks, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HT(hipMemcpyAsync(fl, flags, sizeof(int) * 5, hipMemcpyDeviceToHost, s));
    if (k > 0) {
        HT(hipMemcpyAsync(ws, wsize, sizeof(int64_t) * k, hipMemcpyDeviceToHost, s));
        HT(hipMemcpyAsync(wl, wlo, sizeof(int64_t) * k, hipMemcpyDeviceToHost, s));
    }
    HT(hipStreamSynchronize(s));
    const int64_t nnzb = tot[0];
    if (nnzb > (int64_t)INT32_MAX || tot[1] > (int64_t)INT32_MAX) return DPCG_EINVAL;
    c->nnzb = nnzb;
    c->bj_values = tot[1];
    // ---- block-CSR, block-Jacobi, tiles ----
    HT(keep(c, &c->brow_ptr, nb + 1));
    hipLaunchKernelGGL(k_to_i32, dim3(grid_for(nb + 1)), dim3(256), 0, s, bptr64, (int64_t)nb + 1, c->brow_ptr);
    HT(keep(c, &c->bcol, nnzb));
    HT(keep(c, &c->bval, 9 * (size_t)nnzb));
    HT(hipMemsetAsync(c->bval, 0, sizeof(double) * 9 * (size_t)nnzb, s));
    int32_t *brow = nullptr;
    HT(pool.tmp(&brow, nnzb));
    hipLaunchKernelGGL((k_bsr<true>), dim3(grid_for(nb, 4)), dim3(256), 0, s, nb, kp, kc, kv, nullptr, c->brow_ptr,
                       c->bcol, c->bval, brow);
    // block columns as 16-bit offsets from their row for the iteration SpMV (kept when
    // every offset fits: read back at the end of setup)
    int *b16bad = nullptr;  // [1]: the longest row
    HT(pool.tmp(&b16bad, 2));
    HT(keep(c, &c->bcol16, nnzb));
    HT(hipMemsetAsync(b16bad, 0, 2 * sizeof(int), s));
    hipLaunchKernelGGL(k_bcol16, dim3(grid_for(nnzb)), dim3(256), 0, s, nnzb, (const int32_t *)brow,
                       (const int32_t *)c->bcol, c->bcol16, b16bad);
    if (nnzb <= (int64_t)kLongRowMean * nb)
        hipLaunchKernelGGL(k_longest_row, dim3(grid_for(nb, 256, 64)), dim3(256), 0, s, nb,
                           (const int32_t *)c->brow_ptr, b16bad + 1);
    // The symmetry test and the small block-Jacobi inverses do not feed K Z, E or E^-1:
    // they run on the side stream beside that chain (whose kernels are latency bound and
    // leave most of the chip idle), joined before their flags are read.  Dense blocks
    // keep one stream.
    hipStream_t sb = s;
    if (c->ndense == 0) HT(pool.fork(&sb));
    const int gsym = (grid_for(nnzb, 256, 16384) + 7) / 8 * 8;
    int64_t *sympart = nullptr;
    int *need = nullptr;
    HT(pool.tmp(&sympart, 2 * (int64_t)gsym));
    HT(pool.tmp(&need, 1));
    HT(keep(c, &c->minv, tot[1]));
    HT(keep(c, &c->bj_rowoff, n));
    HT(keep(c, &c->bj_meta, n));
    hipLaunchKernelGGL(k_check_sym, dim3(gsym), dim3(256), 0, sb, c->brow_ptr, brow, c->bcol, c->bval, nnzb, maxpart,
                       nmaxpart, flags, sympart);
    hipLaunchKernelGGL(k_sym_reduce, dim3(1), dim3(256), 0, sb, sympart, gsym, need);
    hipLaunchKernelGGL(k_check_sym_lower, dim3(gsym), dim3(256), 0, sb, c->brow_ptr, brow, c->bcol, c->bval, nnzb,
                       maxpart, nmaxpart, flags, need);
    int *bjbad = flags + 1;  // reuse: Z's flag is known to be clear
    if (c->ndense > 0) {  // the DoFs of dense blocks take no part in the small-block kernels
        HT(hipMemsetAsync(c->bj_meta, 0, sizeof(int32_t) * n, s));
        HT(hipMemsetAsync(c->bj_rowoff, 0, sizeof(int32_t) * n, s));
    }
    hipLaunchKernelGGL(k_bj_small, dim3(grid_for(nblocks)), dim3(256), 0, sb, nblocks, bp, kp, kc, kv, moff, c->minv,
                       c->bj_rowoff, c->bj_meta, bjbad, (const int32_t *)nullptr, 0);
    hipLaunchKernelGGL(k_bj_factor, dim3(std::min<int32_t>(nblocks, 4096)), dim3(64), 0, sb, nblocks, bp, kp, kc, kv,
                       moff, c->minv, c->bj_rowoff, c->bj_meta, bjbad, (const int32_t *)nullptr, 0);
    HT(hipGetLastError());
    if (c->ndense > 0) {
        std::vector<int32_t> all(c->ndense);
        for (int32_t i = 0; i < c->ndense; ++i) all[i] = i;
        const int st = dense_inverses(c, pool, kp, kc, kv, all, bjbad);
        if (st != DPCG_OK) return st;
    }
    // kept for value updates: the partition and each block's offset in minv
    HT(keep(c, &c->block_ptr, nblocks + 1));
    HT(keep(c, &c->bj_moff, nblocks + 1));
    HT(hipMemcpyAsync(c->block_ptr, bp, sizeof(int32_t) * (nblocks + 1), hipMemcpyDeviceToDevice, s));
    HT(hipMemcpyAsync(c->bj_moff, moff, sizeof(int64_t) * (nblocks + 1), hipMemcpyDeviceToDevice, s));
    c->bj_ntiles = (int32_t)((n + kTileDofs - 1) / kTileDofs);
    HT(keep(c, &c->bj_wg_start, c->bj_ntiles + 1));
    hipLaunchKernelGGL(k_tiles, dim3(grid_for((int64_t)nblocks + 1)), dim3(256), 0, s, c->bj_ntiles, nblocks, bp, n,
                       kTileDofs, c->bj_wg_start);
    // the multi-RHS kernels stage tiles of <= kBatchTileDofs DoFs times 32 columns
    c->bjb_ntiles = (int32_t)((n + kBatchTileWindow - 1) / kBatchTileWindow);
    HT(keep(c, &c->bjb_start, c->bjb_ntiles + 1));
    hipLaunchKernelGGL(k_tiles, dim3(grid_for((int64_t)nblocks + 1)), dim3(256), 0, s, c->bjb_ntiles, nblocks, bp, n,
                       kBatchTileWindow, c->bjb_start);
    // Z by rows (int32 row pointer) for the prolongation
    HT(keep(c, &c->z_ptr, n + 1));
    if (k > 0) {
        hipLaunchKernelGGL(k_to_i32, dim3(grid_for(n + 1)), dim3(256), 0, s, zp, n + 1, c->z_ptr);
        HT(keep(c, &c->z_col, nnz_z));
        HT(keep(c, &c->z_val, nnz_z));
        HT(hipMemcpyAsync(c->z_col, zc, sizeof(int32_t) * nnz_z, hipMemcpyDeviceToDevice, s));
        HT(hipMemcpyAsync(c->z_val, zv, sizeof(double) * nnz_z, hipMemcpyDeviceToDevice, s));
    } else {
        HT(hipMemsetAsync(c->z_ptr, 0, sizeof(int32_t) * (n + 1), s));
    }
    HT(hipGetLastError());
    if (k > 0) {
        const int st = coarse_operator(c, pool, k, zp, zc, ztp, zti, ztv, wl, ws, part, flags, bad, false);
        if (st != DPCG_OK) return st;
        // transposed pointers as int32
        HT(keep(c, &c->zt_ptr, k + 1));
        hipLaunchKernelGGL(k_to_i32, dim3(grid_for(k + 1)), dim3(256), 0, s, ztp, (int64_t)k + 1, c->zt_ptr);
        HT(hipStreamSynchronize(s));
    } else {
        HT(pool.join());
        HT(hipMemcpyAsync(fl, flags, sizeof(int) * 4, hipMemcpyDeviceToHost, s));
        HT(hipStreamSynchronize(s));
        if (fl[3] != INT32_MAX) return DPCG_ENOTSYM;
        if (fl[1] != INT32_MAX) {
            *bad = fl[1];
            return DPCG_EBLOCK_NOT_SPD;
        }
    }
    int b16[2] = {};
    HT(hipMemcpy(b16, b16bad, sizeof(b16), hipMemcpyDeviceToHost));
    if (b16[0]) c->bcol16 = nullptr;  // an offset does not fit: the SpMV reads the int32 columns
    c->longest_row = b16[1];
    return DPCG_OK;
}

// New values of K on the same sparsity pattern: block values, the symmetry test, the
// inverses of the listed blocks (all when list is null), K Z, E and E^-1 again.
int gpu_update_values(dpcg_ctx *c, const int64_t *kp, const int32_t *kc, const double *kv, int32_t nlist,
                      const int32_t *list_host, int64_t *bad) {
    hipStream_t s = c->stream;
    Pool pool{c, {}};
    const int64_t n = c->n;
    const int32_t nb = c->nb, k = c->k, nblocks = c->nblocks;
    if (list_host)
        for (int32_t i = 0; i < nlist; ++i)
            if (list_host[i] < 0 || list_host[i] >= nblocks) return DPCG_EINVAL;
    int64_t *ends = nullptr;  // pinned read-backs
    int *fl = nullptr;
    HT(pool.host(&ends, 2));
    HT(pool.host(&fl, 4));
    HT(hipMemcpyAsync(&ends[0], kp, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HT(hipMemcpyAsync(&ends[1], kp + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HT(hipStreamSynchronize(s));
    if (ends[0] != 0 || ends[1] != c->nnz) return DPCG_EINVAL;
    const int64_t nnz = c->nnz, nnzb = c->nnzb;
    int *flags = nullptr;
    HT(pool.tmp(&flags, 4));
    const int init_flags[4] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX};
    HT(hipMemcpyAsync(flags, init_flags, sizeof(init_flags), hipMemcpyHostToDevice, s));
    double *mxp = nullptr;
    HT(check_csr(s, pool, n, n, kp, kc, kv, nnz, flags, &mxp));
    HT(hipMemcpyAsync(fl, flags, sizeof(int) * 4, hipMemcpyDeviceToHost, s));
    HT(hipStreamSynchronize(s));
    if (fl[0] != INT32_MAX) return DPCG_EINVAL;
    // the CSR arrays are valid: the block structure must be the stored one
    int64_t *cnt = nullptr;
    HT(pool.tmp(&cnt, nb));
    hipLaunchKernelGGL((k_bsr<false>), dim3(grid_for(nb, 4)), dim3(256), 0, s, nb, kp, kc, kv, cnt, nullptr, nullptr,
                       nullptr, nullptr);
    hipLaunchKernelGGL(k_cmp_counts, dim3(grid_for(nb)), dim3(256), 0, s, nb, cnt, c->brow_ptr, flags + 2);
    HT(hipMemcpyAsync(fl, flags, sizeof(int) * 4, hipMemcpyDeviceToHost, s));
    HT(hipStreamSynchronize(s));
    if (fl[2] != INT32_MAX) return DPCG_EINVAL;
    // max |K| for the symmetry tolerance: mxp[0], from the checks above
    // block values; the block columns must be the stored ones
    int32_t *bcol2 = nullptr, *brow = nullptr;
    HT(pool.tmp(&bcol2, nnzb));
    HT(pool.tmp(&brow, nnzb));
    HT(hipMemsetAsync(c->bval, 0, sizeof(double) * 9 * (size_t)nnzb, s));
    hipLaunchKernelGGL((k_bsr<true>), dim3(grid_for(nb, 4)), dim3(256), 0, s, nb, kp, kc, kv, nullptr, c->brow_ptr,
                       bcol2, c->bval, brow);
    hipLaunchKernelGGL(k_cmp_i32, dim3(grid_for(nnzb)), dim3(256), 0, s, nnzb, bcol2, c->bcol, flags + 2);
    {
        const int gsym = (grid_for(nnzb, 256, 16384) + 7) / 8 * 8;
        int64_t *sympart = nullptr;
        int *need = nullptr;
        HT(pool.tmp(&sympart, 2 * (int64_t)gsym));
        HT(pool.tmp(&need, 1));
        hipLaunchKernelGGL(k_check_sym, dim3(gsym), dim3(256), 0, s, c->brow_ptr, brow, c->bcol, c->bval, nnzb, mxp,
                           1, flags, sympart);
        hipLaunchKernelGGL(k_sym_reduce, dim3(1), dim3(256), 0, s, sympart, gsym, need);
        hipLaunchKernelGGL(k_check_sym_lower, dim3(gsym), dim3(256), 0, s, c->brow_ptr, brow, c->bcol, c->bval, nnzb,
                           mxp, 1, flags, need);
    }
    // block-Jacobi inverses of the listed blocks
    int32_t *list_d = nullptr;
    if (list_host && nlist > 0) {
        HT(pool.tmp(&list_d, nlist));
        HT(hipMemcpyAsync(list_d, list_host, sizeof(int32_t) * nlist, hipMemcpyHostToDevice, s));
    }
    if (!list_host || nlist > 0) {
        const int32_t count = list_host ? nlist : nblocks;
        hipLaunchKernelGGL(k_bj_small, dim3(grid_for(count)), dim3(256), 0, s, nblocks, c->block_ptr, kp, kc, kv,
                           c->bj_moff, c->minv, c->bj_rowoff, c->bj_meta, flags + 1, (const int32_t *)list_d, nlist);
        hipLaunchKernelGGL(k_bj_factor, dim3(std::min<int32_t>(std::max(count, 1), 4096)), dim3(64), 0, s, nblocks,
                           c->block_ptr, kp, kc, kv, c->bj_moff, c->minv, c->bj_rowoff, c->bj_meta, flags + 1,
                           (const int32_t *)list_d, nlist);
    }
    if (c->ndense > 0) {  // the listed dense blocks (all without a list)
        std::vector<int32_t> which;
        if (!list_host) {
            for (int32_t i = 0; i < c->ndense; ++i) which.push_back(i);
        } else {
            std::vector<char> seen(c->ndense, 0);
            for (int32_t i = 0; i < nlist; ++i) {
                auto it = std::lower_bound(c->dense_h.begin(), c->dense_h.end(), list_host[i],
                                           [](const DenseBlk &d, int32_t b) { return d.block < b; });
                if (it != c->dense_h.end() && it->block == list_host[i] && !seen[it - c->dense_h.begin()]) {
                    seen[it - c->dense_h.begin()] = 1;
                    which.push_back((int32_t)(it - c->dense_h.begin()));
                }
            }
        }
        const int st = dense_inverses(c, pool, kp, kc, kv, which, flags + 1);
        if (st != DPCG_OK) return st;
    }
    HT(hipGetLastError());
    HT(hipMemcpyAsync(fl, flags, sizeof(int) * 4, hipMemcpyDeviceToHost, s));
    HT(hipStreamSynchronize(s));
    if (fl[2] != INT32_MAX) return DPCG_EINVAL;
    if (k > 0) {
        int64_t *ztp = nullptr, *zp = nullptr, *wlo = nullptr, *wsize = nullptr, *part = nullptr;
        HT(pool.tmp(&ztp, k + 1));
        HT(pool.tmp(&zp, n + 1));
        HT(pool.tmp(&wlo, k));
        HT(pool.tmp(&wsize, k));
        HT(pool.tmp(&part, (int64_t)k / kScanChunk + 2));
        hipLaunchKernelGGL(k_to_i64, dim3(grid_for(k + 1)), dim3(256), 0, s, c->zt_ptr, (int64_t)k + 1, ztp);
        hipLaunchKernelGGL(k_to_i64, dim3(grid_for(n + 1)), dim3(256), 0, s, c->z_ptr, n + 1, zp);
        hipLaunchKernelGGL(k_kz_window, dim3(k), dim3(256), 0, s, k, ztp, c->zt_idx, kp, kc, wlo, wsize);
        int64_t *ws = nullptr, *wl = nullptr;
        HT(pool.host(&ws, k));
        HT(pool.host(&wl, k));
        HT(hipMemcpyAsync(ws, wsize, sizeof(int64_t) * k, hipMemcpyDeviceToHost, s));
        HT(hipMemcpyAsync(wl, wlo, sizeof(int64_t) * k, hipMemcpyDeviceToHost, s));
        HT(hipStreamSynchronize(s));
        const int st = coarse_operator(c, pool, k, zp, c->z_col, ztp, c->zt_idx, c->zt_val, wl, ws, part, flags, bad,
                                       true);
        if (st != DPCG_OK) return st;
    } else {
        if (fl[3] != INT32_MAX) return DPCG_ENOTSYM;
        if (fl[1] != INT32_MAX) {
            *bad = fl[1];
            return DPCG_EBLOCK_NOT_SPD;
        }
    }
    // binary32 copies of a handle that has run mixed solves
    if (c->bval32) {
        hipLaunchKernelGGL(k_to_f32_s, dim3(grid_for(9 * nnzb, 256, 8192)), dim3(256), 0, s, c->bval, 9 * nnzb, c->bval32);
        hipLaunchKernelGGL(k_to_f32_s, dim3(grid_for(c->bj_values, 256, 8192)), dim3(256), 0, s, c->minv,
                           c->bj_values, c->minv32);
        if (c->ndense > 0)
            hipLaunchKernelGGL(k_to_f32_s, dim3(grid_for(c->dinv_len, 256, 8192)), dim3(256), 0, s, c->dinv,
                               c->dinv_len, c->dinv32);
    }
    HT(hipGetLastError());
    HT(hipStreamSynchronize(s));
    return DPCG_OK;
}

}  // namespace dpcg
