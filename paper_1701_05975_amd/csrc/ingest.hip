// ingest.hip -- graph ingest from device arrays (bc_create_graph_device).
//
// The caller's CSR (row offsets int64[n+1], heads int32[nnz], weights
// int32[nnz], Sec. 3.1) is validated, renumbered, packed and transposed on
// the device, and the result has the same device layout as the host ingest
// of bc_create_graph builds from the same arrays: the same renumbering by
// decreasing in-degree (ties by id), the same arc order in every row of the
// transpose (by arc index), the same pairing of reverse arcs.  The building
// blocks are a stable least-significant-digit radix sort of (64-bit key,
// 32-bit value) pairs and an exclusive scan, both written for 64-lane waves.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <vector>

#include "bc_internal.h"
#include "dev_common.h"
#include "kernels.h"

namespace {

constexpr int SCAN_NT = 1024;        // threads of a scan block
constexpr int SCAN_PER = 4;          // items per thread
constexpr int SCAN_TILE = SCAN_NT * SCAN_PER;
constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int RADIX_CHUNKS = 16;     // 64-element chunks per wave tile
constexpr int RADIX_TILE = WAVE * RADIX_CHUNKS;
constexpr int RADIX_WAVES = 4;       // waves (tiles) per workgroup

int blocks_for(size_t items, int per_block, int cap = 1 << 20)
{
    size_t b = (items + (size_t)per_block - 1) / (size_t)per_block;
    return (int)std::max<size_t>(1, std::min<size_t>(b, (size_t)cap));
}

// ---------------------------------------------------------------------------
// Exclusive scan of uint32 (totals below 2^32)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t x)
{
    const int lane = lane_id();
    for (int o = 1; o < WAVE; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o)
            x += y;
    }
    return x;
}

// Scans one tile of SCAN_TILE items per block; the block's total goes to
// sums[blockIdx.x].
__global__ __launch_bounds__(SCAN_NT) void k_scan_tiles(const uint32_t *in, uint32_t *out,
                                                       size_t count, uint32_t *sums)
{
    __shared__ uint32_t wsum[SCAN_NT / WAVE];
    const size_t base = (size_t)blockIdx.x * SCAN_TILE + (size_t)threadIdx.x * SCAN_PER;
    uint32_t v[SCAN_PER];
    uint32_t t = 0;
#pragma unroll
    for (int j = 0; j < SCAN_PER; ++j) {
        v[j] = base + j < count ? in[base + j] : 0u;
        t += v[j];
    }
    const int w = threadIdx.x / WAVE;
    const uint32_t incl = wave_incl_scan_u32(t);
    if (lane_id() == WAVE - 1)
        wsum[w] = incl;
    __syncthreads();
    if (w == 0) {
        const uint32_t x = lane_id() < SCAN_NT / WAVE ? wsum[lane_id()] : 0u;
        const uint32_t xi = wave_incl_scan_u32(x);
        if (lane_id() < SCAN_NT / WAVE)
            wsum[lane_id()] = xi - x; // exclusive prefix of each wave
        if (lane_id() == SCAN_NT / WAVE - 1)
            sums[blockIdx.x] = xi;
    }
    __syncthreads();
    uint32_t run = wsum[w] + incl - t;
#pragma unroll
    for (int j = 0; j < SCAN_PER; ++j) {
        if (base + j < count)
            out[base + j] = run;
        run += v[j];
    }
}

__global__ void k_scan_add(uint32_t *out, size_t count, const uint32_t *offs)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count)
        out[i] += offs[i / SCAN_TILE];
}

// Words of scratch that a scan of `count` items needs.
size_t scan_scratch(size_t count)
{
    const size_t tiles = (count + SCAN_TILE - 1) / SCAN_TILE;
    return tiles > 1 ? tiles + scan_scratch(tiles) : 2;
}

// out[i] = sum of in[0 .. i-1]; in and out may be the same array.
void scan_exclusive(const uint32_t *in, uint32_t *out, size_t count, uint32_t *scratch,
                    hipStream_t st)
{
    const size_t tiles = std::max<size_t>((count + SCAN_TILE - 1) / SCAN_TILE, 1);
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)tiles), dim3(SCAN_NT), 0, st, in, out, count,
                       scratch);
    hip_check(hipGetLastError(), "scan");
    if (tiles > 1) {
        scan_exclusive(scratch, scratch, tiles, scratch + tiles, st);
        hipLaunchKernelGGL(k_scan_add, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                           out, count, scratch);
        hip_check(hipGetLastError(), "scan add");
    }
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort of (key, value u32) pairs, 8 bits per pass; the keys
// are 32-bit where their bits fit.
//
// Each wave owns a tile of RADIX_TILE consecutive items, read in 64-item
// chunks in order; the digit histograms are stored digit-major over the
// tiles, so one exclusive scan gives every (digit, tile) its first output
// position, and inside a tile an item's rank among the equal digits before
// it comes from ballots.  Equal digits keep their input order: the sort is
// stable, so a sort by a secondary key followed by one by the primary key
// orders by both.
// ---------------------------------------------------------------------------
template <class K>
__global__ __launch_bounds__(WAVE * RADIX_WAVES) void k_radix_hist(const K *keys,
                                                                  uint32_t count, int shift,
                                                                  uint32_t ntiles, uint32_t *hist)
{
    __shared__ uint32_t h[RADIX_WAVES][RADIX];
    const int w = threadIdx.x / WAVE, lane = lane_id();
    const uint32_t tile = blockIdx.x * RADIX_WAVES + w;
    for (int d = lane; d < RADIX; d += WAVE)
        h[w][d] = 0;
    __syncthreads();
    if (tile < ntiles) {
        const uint32_t base = tile * RADIX_TILE;
        for (int c = 0; c < RADIX_CHUNKS; ++c) {
            const uint32_t i = base + c * WAVE + lane;
            if (i < count)
                atomicAdd(&h[w][(keys[i] >> shift) & (RADIX - 1)], 1u);
        }
    }
    __syncthreads();
    if (tile < ntiles)
        for (int d = lane; d < RADIX; d += WAVE)
            hist[(size_t)d * ntiles + tile] = h[w][d];
}

template <class K>
__global__ __launch_bounds__(WAVE * RADIX_WAVES) void k_radix_scatter(
    const K *keys, const uint32_t *vals, K *okeys, uint32_t *ovals, uint32_t count, int shift,
    uint32_t ntiles, const uint32_t *offs)
{
    __shared__ uint32_t pos[RADIX_WAVES][RADIX];
    const int w = threadIdx.x / WAVE, lane = lane_id();
    const uint32_t tile = blockIdx.x * RADIX_WAVES + w;
    if (tile >= ntiles)
        return; // whole wave: the tile index is uniform in the wave
    for (int d = lane; d < RADIX; d += WAVE)
        pos[w][d] = offs[(size_t)d * ntiles + tile];
    const uint32_t base = tile * RADIX_TILE;
    for (int c = 0; c < RADIX_CHUNKS; ++c) {
        const uint32_t i = base + c * WAVE + lane;
        const bool valid = i < count;
        K k = 0;
        uint32_t v = 0, d = 0;
        if (valid) {
            k = keys[i];
            v = vals[i];
            d = (uint32_t)(k >> shift) & (RADIX - 1);
        }
        // lanes holding the same digit
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < RADIX_BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = lanes_below(peers);
        const uint32_t at = valid ? pos[w][d] + rank : 0u;
        // the last of the peers advances the digit's position for the next chunk
        const bool last = valid && (peers >> lane) == 1ull;
        __builtin_amdgcn_wave_barrier();
        if (last)
            pos[w][d] = at + 1u;
        __builtin_amdgcn_wave_barrier();
        if (valid) {
            okeys[at] = k;
            ovals[at] = v;
        }
    }
}

int bit_width_u64(uint64_t x)
{
    int b = 0;
    while (x) {
        ++b;
        x >>= 1;
    }
    return b;
}

// Sorts (keys, vals) by the key bits [0, bits), through the scratch pair;
// returns the buffer that the sorted values end in (vals or the scratch).
struct SortBufs {
    DevBuf keys, vals, k2, v2, hist, scan;
    void reserve(size_t count, size_t key_bytes, size_t scans)
    {
        auto at_least = [](DevBuf &b, size_t bytes) {
            if (b.bytes < bytes)
                b.alloc(bytes);
        };
        const size_t tiles = (count + RADIX_TILE - 1) / RADIX_TILE;
        at_least(keys, count * key_bytes);
        at_least(k2, count * key_bytes);
        at_least(vals, count * 4);
        at_least(v2, count * 4);
        at_least(hist, tiles * RADIX * 4);
        at_least(scan, scan_scratch(std::max(scans, tiles * RADIX)) * 4);
    }
};

template <class K>
uint32_t *radix_sort(SortBufs &b, uint32_t count, int bits, hipStream_t st)
{
    uint32_t *va = (uint32_t *)b.vals.p, *vb = (uint32_t *)b.v2.p;
    if (count < 2 || bits <= 0)
        return va;
    const uint32_t ntiles = (count + RADIX_TILE - 1) / RADIX_TILE;
    K *ka = (K *)b.keys.p, *kb = (K *)b.k2.p;
    uint32_t *hist = (uint32_t *)b.hist.p;
    const unsigned blocks = (ntiles + RADIX_WAVES - 1) / RADIX_WAVES;
    for (int shift = 0; shift < bits; shift += RADIX_BITS) {
        hipLaunchKernelGGL(k_radix_hist<K>, dim3(blocks), dim3(WAVE * RADIX_WAVES), 0, st, ka,
                           count, shift, ntiles, hist);
        hip_check(hipGetLastError(), "radix histogram");
        scan_exclusive(hist, hist, (size_t)ntiles * RADIX, (uint32_t *)b.scan.p, st);
        hipLaunchKernelGGL(k_radix_scatter<K>, dim3(blocks), dim3(WAVE * RADIX_WAVES), 0, st, ka,
                           va, kb, vb, count, shift, ntiles, hist);
        hip_check(hipGetLastError(), "radix scatter");
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    return va;
}

// ---------------------------------------------------------------------------
// Ingest kernels
// ---------------------------------------------------------------------------
struct IngestSummary {
    unsigned long long bad_row;  // smallest row whose offsets decrease (ULLONG_MAX: none)
    unsigned long long bad_col;  // smallest arc whose head is out of range
    unsigned long long bad_w;    // smallest arc whose weight is below 1
    unsigned long long wsum;     // sum of the weights
    unsigned long long deg_sum, deg_squares; // of the degrees, at most DEG_CAP each
    unsigned int maxdeg, wmax, nz_rows, max_indeg;
    int32_t bad_w_value, bad_col_value;
    long long row0, rown;        // row_ptr[0], row_ptr[n]
};

// Validation (the checks of the host ingest) and the per-vertex in-degrees.
// Atomics on the summary's one line follow one another at about 12 ns each, so
// workgroups are few and add once: with a wave's four each from 8192 workgroups
// they were 1.5 ms of the kernel (ER 500k, 4M arcs 1.57 -> 0.18 ms).
constexpr int CHECK_NT = 256, CHECK_WGS = 1024;

__global__ __launch_bounds__(CHECK_NT) void k_ingest_check(int32_t n, uint32_t nnz, const int64_t *row_ptr,
                               const int32_t *col, const int32_t *w, uint32_t *indeg,
                               IngestSummary *sum)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t span = std::max<size_t>((size_t)n, (size_t)nnz);
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid == 0) {
        sum->row0 = row_ptr[0];
        sum->rown = row_ptr[n];
    }
    // every lane of a wave runs the same number of iterations (wave reductions)
    const size_t iters = (span + stride - 1) / stride;
    uint32_t maxdeg = 0, wmax = 0, nz = 0;
    unsigned long long wsum = 0;
    for (size_t it = 0; it < iters; ++it) {
        const size_t i = tid + it * stride;
        if (i < (size_t)n) {
            const long long d = row_ptr[i + 1] - row_ptr[i];
            if (d < 0)
                atomicMin(&sum->bad_row, (unsigned long long)i);
            else if (d > 0) {
                nz += 1;
                const uint32_t dd = d > 0xffffffffll ? 0xffffffffu : (uint32_t)d;
                maxdeg = dd > maxdeg ? dd : maxdeg;
            }
        }
        if (i < (size_t)nnz) {
            const int32_t c = col[i];
            const int32_t x = w[i];
            if (c < 0 || c >= n)
                atomicMin(&sum->bad_col, (unsigned long long)i);
            else
                atomicAdd(&indeg[c], 1u);
            if (x < 1)
                atomicMin(&sum->bad_w, (unsigned long long)i);
            else {
                wmax = (uint32_t)x > wmax ? (uint32_t)x : wmax;
                wsum += (unsigned long long)x;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t a = __shfl_xor(maxdeg, o), b = __shfl_xor(wmax, o);
        maxdeg = a > maxdeg ? a : maxdeg;
        wmax = b > wmax ? b : wmax;
        nz += __shfl_xor(nz, o);
        wsum += __shfl_xor(wsum, o);
    }
    __shared__ uint32_t wg[3][CHECK_NT / WAVE];
    __shared__ unsigned long long wg_wsum[CHECK_NT / WAVE];
    if (lane_id() == 0) {
        const int j = threadIdx.x / WAVE;
        wg[0][j] = maxdeg;
        wg[1][j] = wmax;
        wg[2][j] = nz;
        wg_wsum[j] = wsum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 1; j < CHECK_NT / WAVE; ++j) {
            maxdeg = wg[0][j] > maxdeg ? wg[0][j] : maxdeg;
            wmax = wg[1][j] > wmax ? wg[1][j] : wmax;
            nz += wg[2][j];
            wsum += wg_wsum[j];
        }
        atomicMax(&sum->maxdeg, maxdeg);
        atomicMax(&sum->wmax, wmax);
        atomicAdd(&sum->nz_rows, nz);
        atomicAdd(&sum->wsum, wsum);
    }
}

__global__ void k_ingest_bad_values(const int32_t *col, const int32_t *w, IngestSummary *sum)
{
    if (sum->bad_col != ~0ull)
        sum->bad_col_value = col[sum->bad_col];
    if (sum->bad_w != ~0ull)
        sum->bad_w_value = w[sum->bad_w];
}

// The largest in-degree and the sums for the spread of the degrees; few workgroups,
// which add once each (see k_ingest_check).
__global__ __launch_bounds__(CHECK_NT) void k_degrees(const uint32_t *indeg, const int64_t *row_ptr,
                                                      int32_t n, IngestSummary *sum)
{
    uint32_t m = 0;
    unsigned long long ds = 0, dq = 0;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)n; i += stride) {
        m = indeg[i] > m ? indeg[i] : m;
        const long long d = row_ptr[i + 1] - row_ptr[i];
        const unsigned long long x = d < 0 ? 0 : d < DEG_CAP ? d : DEG_CAP;
        ds += x;
        dq += x * x;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t y = __shfl_xor(m, o);
        m = y > m ? y : m;
        ds += __shfl_xor(ds, o);
        dq += __shfl_xor(dq, o);
    }
    __shared__ unsigned long long wg[3][CHECK_NT / WAVE];
    if (lane_id() == 0) {
        const int j = threadIdx.x / WAVE;
        wg[0][j] = m;
        wg[1][j] = ds;
        wg[2][j] = dq;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 1; j < CHECK_NT / WAVE; ++j) {
            m = wg[0][j] > m ? (uint32_t)wg[0][j] : m;
            ds += wg[1][j];
            dq += wg[2][j];
        }
        atomicMax(&sum->max_indeg, m);
        atomicAdd(&sum->deg_sum, ds);
        atomicAdd(&sum->deg_squares, dq);
    }
}

// Sort keys of the renumbering: decreasing in-degree; the stable sort keeps
// equal in-degrees in id order, as the host's stable sort does.
__global__ void k_renumber_keys(const uint32_t *indeg, int32_t n, uint32_t maxin, uint32_t *keys,
                                uint32_t *vals)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x; v < (size_t)n; v += stride) {
        keys[v] = maxin - indeg[v];
        vals[v] = (uint32_t)v;
    }
}

// Sum of the in-degrees of the first `top` vertices of the order.
__global__ void k_top_sum(const uint32_t *indeg, const uint32_t *order, int32_t top,
                          unsigned long long *out)
{
    unsigned long long s = 0;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)top; i += stride)
        s += indeg[order[i]];
    for (int o = 32; o > 0; o >>= 1)
        s += __shfl_xor(s, o);
    if (lane_id() == 0 && s)
        atomicAdd(out, s);
}

// perm[i] = order[i] (internal -> caller), iperm[order[i]] = i, and the
// internal out-degrees (deg[i] = out-degree of order[i]) and in-degrees.
__global__ void k_apply_order(const uint32_t *order, int32_t n, const int64_t *row_ptr,
                              const uint32_t *indeg, int32_t *perm, int32_t *iperm, uint32_t *deg,
                              uint32_t *tdeg)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)n; i += stride) {
        const uint32_t o = order[i];
        perm[i] = (int32_t)o;
        iperm[o] = (int32_t)i;
        deg[i] = (uint32_t)(row_ptr[o + 1] - row_ptr[o]);
        tdeg[i] = indeg[o];
    }
}

__global__ void k_row_u32(const int64_t *row_ptr, int32_t n, uint32_t *row)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i <= (size_t)n; i += stride)
        row[i] = (uint32_t)row_ptr[i];
}

// The row holding arc position p: the last v with row[v] <= p.
template <class T>
__device__ __forceinline__ uint32_t row_of(const T *row, int32_t n, uint32_t p)
{
    uint32_t lo = 0, hi = (uint32_t)n; // row[lo] <= p < row[hi]
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (row[mid] <= (T)p)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Internal arcs: arc position p of internal row i comes from caller arc
// src = row_ptr[perm[i]] + (p - row[i]) (src = p without renumbering); its
// head is renumbered.  Writes the graph's arc words, the weights (null: not
// wanted), the caller arc index (edge betweenness, else null), and for the
// sorts the head and the internal tail (null: no sort follows).
__global__ void k_internal_arcs(int32_t n, uint32_t nnz, const uint32_t *row,
                                const int64_t *row_ptr, const int32_t *col, const int32_t *w,
                                const int32_t *perm, const int32_t *iperm, int packed,
                                uint32_t wshift, uint32_t wmask, uint32_t *arc, int32_t *wt,
                                uint32_t *ce, uint32_t *head, uint32_t *tail)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < (size_t)nnz; p += stride) {
        uint32_t i = 0;
        size_t src = p;
        if (perm || tail)
            i = row_of(row, n, (uint32_t)p);
        if (perm)
            src = (size_t)row_ptr[perm[i]] + (p - row[i]);
        const int32_t c = col[src], x = w[src];
        const uint32_t h = (uint32_t)(iperm ? iperm[c] : c);
        arc[p] = packed ? (h << wshift) | ((uint32_t)(x - 1) & wmask) : h;
        if (wt)
            wt[p] = x;
        if (ce)
            ce[p] = (uint32_t)src;
        if (tail) {
            head[p] = h;
            tail[p] = i;
        }
    }
}

// Keys of a directed graph's transpose: the head; values: the arc's word in the
// in-row of its head (tail and weight), so that the sorted values are the
// transpose itself.
__global__ void k_transpose_keys(int32_t n, uint32_t nnz, const uint32_t *row, const uint32_t *arc,
                                 uint32_t wshift, uint32_t wmask, uint32_t *keys, uint32_t *vals)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < (size_t)nnz; p += stride) {
        const uint32_t x = arc[p];
        keys[p] = x >> wshift;
        vals[p] = row_of(row, n, (uint32_t)p) << wshift | (x & wmask);
    }
}

// Keys (primary << shift | secondary) over the arcs, values = arc positions.
template <class K>
__global__ void k_pair_keys(uint32_t nnz, const uint32_t *a, const uint32_t *b, int shift,
                            K *keys, uint32_t *vals, const uint32_t *order)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)nnz; i += stride) {
        const uint32_t p = order ? order[i] : (uint32_t)i;
        keys[i] = b ? (K)(((uint64_t)a[p] << shift) | b[p]) : (K)a[p];
        vals[i] = p;
    }
}

__global__ void k_weight_keys(uint32_t nnz, const int32_t *wt, uint32_t *keys, uint32_t *vals)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)nnz; i += stride) {
        keys[i] = (uint32_t)wt[i];
        vals[i] = (uint32_t)i;
    }
}

// Transpose entries: in-row position q holds the arc sorted[q] (tail, weight).
__global__ void k_transpose_arcs(uint32_t nnz, const uint32_t *sorted, const uint32_t *tail,
                                 const int32_t *wt, int packed, uint32_t wshift, uint32_t wmask,
                                 uint32_t *tarc, int32_t *twt)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < (size_t)nnz; q += stride) {
        const uint32_t p = sorted[q];
        const uint32_t t = tail[p];
        const int32_t x = wt[p];
        tarc[q] = packed ? (t << wshift) | ((uint32_t)(x - 1) & wmask) : t;
        if (twt)
            twt[q] = x;
    }
}

// (head, weight) of caller arc e, as one number.
__device__ __forceinline__ uint64_t arc_key(const int32_t *col, const int32_t *w, size_t e)
{
    return (uint64_t)(uint32_t)col[e] << 32 | (uint32_t)w[e];
}

// The first arc of [lo, hi) whose key is not below k, if they are in order.
__device__ __forceinline__ size_t first_arc(const int32_t *col, const int32_t *w, size_t lo,
                                            size_t hi, uint64_t k)
{
    while (lo < hi) {
        const size_t mid = lo + (hi - lo) / 2;
        if (arc_key(col, w, mid) < k)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Undirected check and reverse-arc pairing on the caller's arrays, for rows in
// (head, weight) order: the i-th of the equal arcs (u, v, w) in row u pairs with
// the i-th (v, u, w) in row v, which a search in row v finds.  If every arc has
// its partner the graph is symmetric.  flags[0]: a row is out of order (the
// other outputs say nothing then, and the sorts below decide); flags[1]: an arc
// without a partner.  A few random reads per arc take the place of two sorts of
// all arcs by (tail, head, weight) (22 to 24 passes over 12 to 16 bytes):
// Barabasi-Albert 1M, 10M arcs, the whole build of the graph 12.3 -> 4.4 ms;
// ER 500k, 4M arcs 6.6 -> 2.4 ms.
__global__ void k_reverse_arcs(int32_t n, uint32_t nnz, const int64_t *row_ptr,
                               const int32_t *col, const int32_t *w, uint32_t *rev,
                               unsigned int *flags)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    bool disorder = false, bad = false;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < (size_t)nnz; p += stride) {
        const uint32_t u = row_of(row_ptr, n, (uint32_t)p);
        const size_t beg = (size_t)row_ptr[u];
        const int32_t v = col[p], x = w[p];
        const uint64_t own = arc_key(col, w, p);
        size_t rank = 0;
        if (p > beg) {
            const uint64_t before = arc_key(col, w, p - 1);
            disorder |= before > own;
            if (before == own)
                rank = p - first_arc(col, w, beg, p, own);
        }
        const uint64_t want = (uint64_t)u << 32 | (uint32_t)x;
        const size_t end = (size_t)row_ptr[v + 1];
        const size_t q = first_arc(col, w, (size_t)row_ptr[v], end, want) + rank;
        const bool found = q < end && arc_key(col, w, q) == want;
        bad |= !found;
        if (rev && found)
            rev[p] = (uint32_t)q;
    }
    if (__ballot(disorder) && lane_id() == 0)
        atomicOr(&flags[0], 1u);
    if (__ballot(bad) && lane_id() == 0)
        atomicOr(&flags[1], 1u);
}

// The same for rows in any order: fwd lists the arcs sorted by
// (tail, head, weight, position), bwd by (head, tail, weight, position).  The
// graph is symmetric iff the i-th entries agree as (tail, head, weight) vs
// (head, tail, weight) for every i; then rev[fwd[i]] = bwd[i].
__global__ void k_pair_reverse(uint32_t nnz, const uint32_t *fwd, const uint32_t *bwd,
                               const uint32_t *head, const uint32_t *tail, const int32_t *wt,
                               uint32_t *rev, unsigned int *mismatch)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)nnz; i += stride) {
        const uint32_t f = fwd[i], b = bwd[i];
        bad |= tail[f] != head[b] || head[f] != tail[b] || wt[f] != wt[b];
        if (rev)
            rev[f] = b;
    }
    if (__ballot(bad) && lane_id() == 0)
        atomicOr(mismatch, 1u);
}

__global__ void k_emap(uint32_t nnz, const uint32_t *through, const uint32_t *ce, uint32_t *emap)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < (size_t)nnz; p += stride) {
        const uint32_t a = through[p];
        emap[p] = ce ? ce[a] : a;
    }
}

#define GRID(items) dim3((unsigned)blocks_for((size_t)(items), 256, 8192)), dim3(256), 0

// Sorts the arc positions stably by (a << shift | b) after a stable sort by
// the weight (when wbits > 0): the result lists the arcs ordered by
// (a, b, weight, position).  by_w: nnz words when wbits > 0.
uint32_t *sort_arcs(uint32_t nnz, const uint32_t *a, const uint32_t *b, int shift, int key_bits,
                    const int32_t *wt, int wbits, uint32_t *by_w, SortBufs &tmp, hipStream_t st)
{
    const uint32_t *order = nullptr;
    uint32_t *const vals = (uint32_t *)tmp.vals.p;
    if (wbits > 0) {
        hipLaunchKernelGGL(k_weight_keys, GRID(nnz), st, nnz, wt, (uint32_t *)tmp.keys.p, vals);
        const uint32_t *sorted = radix_sort<uint32_t>(tmp, nnz, wbits, st);
        hip_check(hipMemcpyAsync(by_w, sorted, (size_t)nnz * 4, hipMemcpyDeviceToDevice, st),
                  "copy");
        order = by_w;
    }
    if (key_bits <= 32) {
        hipLaunchKernelGGL(k_pair_keys<uint32_t>, GRID(nnz), st, nnz, a, b, shift,
                           (uint32_t *)tmp.keys.p, vals, order);
        return radix_sort<uint32_t>(tmp, nnz, key_bits, st);
    }
    hipLaunchKernelGGL(k_pair_keys<uint64_t>, GRID(nnz), st, nnz, a, b, shift,
                       (uint64_t *)tmp.keys.p, vals, order);
    return radix_sort<uint64_t>(tmp, nnz, key_bits, st);
}

bc_error not_symmetric()
{
    return bc_error(BC_E_GRAPH,
                    "undirected graph is not symmetric (every arc needs a reverse arc of "
                    "equal weight); pass BC_DIRECTED for one-way arcs");
}

} // namespace

// Builds graph g (fields already zeroed) from the caller's device CSR.
void create_graph_device(int32_t n, int64_t nnz64, const int64_t *row_ptr, const int32_t *col,
                         const int32_t *w, uint32_t flags, hipStream_t st, bc_graph *g)
{
    const uint32_t nnz = (uint32_t)nnz64;
    const bool directed = (flags & BC_DIRECTED) != 0;
    const bool want_edges = (flags & BC_EDGE_BC) != 0;

    // 1. validation and in-degrees
    DevBuf sumb, indegb;
    sumb.alloc(sizeof(IngestSummary));
    indegb.alloc((size_t)n * 4);
    {
        IngestSummary init;
        memset(&init, 0, sizeof init);
        init.bad_row = init.bad_col = init.bad_w = ~0ull;
        hip_check(hipMemcpyAsync(sumb.p, &init, sizeof init, hipMemcpyHostToDevice, st), "init");
    }
    hip_check(launch_fill_u32((uint32_t *)indegb.p, (size_t)n, 0u, st), "clear");
    IngestSummary *dsum = (IngestSummary *)sumb.p;
    uint32_t *indeg = (uint32_t *)indegb.p;
    hipLaunchKernelGGL(k_ingest_check,
                       dim3((unsigned)blocks_for(std::max<size_t>((size_t)n, nnz), CHECK_NT,
                                                 CHECK_WGS)),
                       dim3(CHECK_NT), 0, st, n, nnz, row_ptr, col, w, indeg, dsum);
    hipLaunchKernelGGL(k_ingest_bad_values, dim3(1), dim3(1), 0, st, col, w, dsum);
    hipLaunchKernelGGL(k_degrees, dim3((unsigned)blocks_for((size_t)n, CHECK_NT, 256)),
                       dim3(CHECK_NT), 0, st, indeg, row_ptr, n, dsum);
    hip_check(hipGetLastError(), "ingest check");
    IngestSummary S;
    hip_check(hipMemcpyAsync(&S, dsum, sizeof S, hipMemcpyDeviceToHost, st), "summary");
    hip_check(hipStreamSynchronize(st), "ingest check");
    if (S.row0 != 0 || S.rown != nnz64)
        throw bc_error(BC_E_GRAPH, "row_ptr[0] must be 0 and row_ptr[n] must equal nnz");
    if (S.bad_row != ~0ull)
        throw bc_error(BC_E_GRAPH, "row_ptr decreases at row %lld", (long long)S.bad_row);
    if (S.bad_col != ~0ull && S.bad_col <= S.bad_w)
        throw bc_error(BC_E_GRAPH, "col[%lld] = %d out of range", (long long)S.bad_col,
                       S.bad_col_value);
    if (S.bad_w != ~0ull)
        throw bc_error(BC_E_WEIGHT, "w[%lld] = %d is below 1", (long long)S.bad_w, S.bad_w_value);
    const int32_t wmax = nnz ? (int32_t)S.wmax : 1;
    if ((int64_t)(n - 1) * (int64_t)wmax > (int64_t)INT32_MAX - 1)
        throw bc_error(BC_E_DIST_OVERFLOW, "(n-1)*max weight = %lld does not fit in int32",
                       (long long)(n - 1) * wmax);

    g->n = n;
    g->nnz = nnz64;
    g->directed = directed;
    g->wmax = wmax;
    g->maxdeg = (int32_t)std::min<uint32_t>(S.maxdeg, INT32_MAX);
    const int colbits = bit_width_u64((uint64_t)(n - 1));
    const int wbits = bit_width_u64((uint64_t)(wmax - 1));
    g->packed = colbits + wbits <= 32 && wbits < 32;
    g->wshift = g->packed ? (uint32_t)wbits : 0u;
    g->wmask = g->packed ? (wbits == 0 ? 0u : (uint32_t)((1ull << wbits) - 1)) : 0u;
    g->wbytes = wmax <= 255 ? 1 : (wmax <= 65535 ? 2 : 4);
    g->avg_deg = S.nz_rows ? (double)nnz64 / (double)S.nz_rows : 0.0;
    g->wmean = nnz ? (double)S.wsum / (double)nnz64 : 1.0;
    g->deg_spread = spread_of((double)S.nz_rows, (double)S.deg_sum, (double)S.deg_squares);

    SortBufs tmp;
    const uint32_t *order = nullptr; // the renumbering, if any
    // 2. renumbering by decreasing in-degree when the in-degrees are skewed
    bool renumber = false;
    DevBuf topb;
    if (!(flags & BC_KEEP_ORDER) && n > 1 && nnz > 0) {
        tmp.reserve((size_t)n, 4, (size_t)n + 1);
        hipLaunchKernelGGL(k_renumber_keys, GRID(n), st, indeg, n, S.max_indeg,
                           (uint32_t *)tmp.keys.p, (uint32_t *)tmp.vals.p);
        order = radix_sort<uint32_t>(tmp, (uint32_t)n, bit_width_u64(S.max_indeg), st);
        topb.alloc(8);
        hip_check(launch_fill_u64((unsigned long long *)topb.p, 1, 0ull, st), "clear");
        const int32_t top = std::max<int32_t>(1, n / 100);
        hipLaunchKernelGGL(k_top_sum, GRID(top), st, indeg, order, top,
                           (unsigned long long *)topb.p);
        unsigned long long top_arcs = 0;
        hip_check(hipMemcpyAsync(&top_arcs, topb.p, 8, hipMemcpyDeviceToHost, st), "top");
        hip_check(hipStreamSynchronize(st), "renumbering");
        renumber = (double)top_arcs > 0.05 * (double)nnz64;
    }
    DevBuf degb, tdegb;
    degb.alloc(((size_t)n + 1) * 4);
    tdegb.alloc(((size_t)n + 1) * 4);
    g->row.alloc(((size_t)n + 1) * 4);
    uint32_t *row = (uint32_t *)g->row.p;
    if (renumber) {
        g->renumbered = true;
        g->perm.alloc((size_t)n * 4);
        g->iperm.alloc((size_t)n * 4);
        hipLaunchKernelGGL(k_apply_order, GRID(n), st, order, n, row_ptr, indeg,
                           (int32_t *)g->perm.p, (int32_t *)g->iperm.p, (uint32_t *)degb.p,
                           (uint32_t *)tdegb.p);
        hip_check(hipGetLastError(), "renumber");
        hip_check(launch_fill_u32((uint32_t *)degb.p + n, 1, 0u, st), "clear");
        scan_exclusive((const uint32_t *)degb.p, row, (size_t)n + 1, (uint32_t *)tmp.scan.p, st);
        g->host_iperm.resize((size_t)n);
        hip_check(hipMemcpyAsync(g->host_iperm.data(), g->iperm.p, (size_t)n * 4,
                                 hipMemcpyDeviceToHost, st),
                  "numbering");
    } else {
        hipLaunchKernelGGL(k_row_u32, GRID((size_t)n + 1), st, row_ptr, n, row);
        hip_check(hipGetLastError(), "rows");
    }

    // 3. undirected: the reverse arcs, if the rows are in order
    DevBuf through; // per in-row position: the arc it stands for (edge map)
    DevBuf rev;     // or, of rows in order, per caller arc: its reverse arc
    // step 5 sorts the arcs' positions (packed arcs of a transpose without an edge
    // map are sorted themselves, without the four arrays of positions, tails, weights
    // and heads: 1.6 ms of 7.8 less for R-MAT scale 20, 16M arcs)
    bool sorts = nnz > 0 && !(directed && g->packed && !want_edges);
    if (!directed && nnz > 0) {
        DevBuf flag;
        flag.alloc(8);
        hip_check(launch_fill_u32((uint32_t *)flag.p, 2, 0u, st), "clear");
        if (want_edges)
            rev.alloc((size_t)nnz * 4);
        hipLaunchKernelGGL(k_reverse_arcs, GRID(nnz), st, n, nnz, row_ptr, col, w,
                           (uint32_t *)rev.p, (unsigned int *)flag.p);
        hip_check(hipGetLastError(), "symmetry");
        unsigned int got[2] = {0, 0};
        hip_check(hipMemcpyAsync(got, flag.p, 8, hipMemcpyDeviceToHost, st), "symmetry");
        hip_check(hipStreamSynchronize(st), "symmetry");
        if (got[0])
            rev.release();
        else if (got[1])
            throw not_symmetric();
        else
            sorts = false;
    }

    // 4. internal arcs (heads renumbered), packed
    DevBuf headb, tailb, wtb, ceb;
    if (sorts) {
        headb.alloc((size_t)nnz * 4);
        tailb.alloc((size_t)nnz * 4);
        if (g->packed)
            wtb.alloc((size_t)nnz * 4);
    }
    if (want_edges && renumber)
        ceb.alloc(std::max<size_t>(nnz, 1) * 4);
    uint32_t *head = (uint32_t *)headb.p, *tail = (uint32_t *)tailb.p;
    uint32_t *ce = (uint32_t *)ceb.p;
    int32_t *wt = (int32_t *)wtb.p;
    if (nnz > 0) {
        g->arc.alloc((size_t)nnz * 4);
        if (!g->packed) {
            g->wt.alloc((size_t)nnz * 4);
            wt = (int32_t *)g->wt.p;
        }
        hipLaunchKernelGGL(k_internal_arcs, GRID(nnz), st, n, nnz, row, row_ptr, col, w,
                           renumber ? (const int32_t *)g->perm.p : nullptr,
                           renumber ? (const int32_t *)g->iperm.p : nullptr, (int)g->packed,
                           g->wshift, g->wmask, (uint32_t *)g->arc.p, wt, ce, head, tail);
        hip_check(hipGetLastError(), "arcs");
    }

    // 5. transpose (directed) or, of rows in any order, symmetry check and
    // reverse arcs (undirected)
    if (directed) {
        g->trow.alloc(((size_t)n + 1) * 4);
        uint32_t *tdeg = renumber ? (uint32_t *)tdegb.p : indeg;
        if (!renumber) {
            hip_check(hipMemcpyAsync(tdegb.p, indeg, (size_t)n * 4, hipMemcpyDeviceToDevice, st),
                      "in-degrees");
            tdeg = (uint32_t *)tdegb.p;
        }
        hip_check(launch_fill_u32(tdeg + n, 1, 0u, st), "clear");
        tmp.reserve(nnz, 4, (size_t)n + 1);
        scan_exclusive(tdeg, (uint32_t *)g->trow.p, (size_t)n + 1, (uint32_t *)tmp.scan.p, st);
        // arcs stably by head: every in-row lists its arcs by arc position
        if (nnz > 0 && !sorts) {
            hipLaunchKernelGGL(k_transpose_keys, GRID(nnz), st, n, nnz, row,
                               (const uint32_t *)g->arc.p, g->wshift, g->wmask,
                               (uint32_t *)tmp.keys.p, (uint32_t *)tmp.vals.p);
            const uint32_t *sorted = radix_sort<uint32_t>(tmp, nnz, colbits, st);
            DevBuf &from = sorted == tmp.vals.p ? tmp.vals : tmp.v2;
            if (from.bytes == (size_t)nnz * 4) {
                std::swap(g->tarc.p, from.p);
                std::swap(g->tarc.bytes, from.bytes);
            } else { // sized for the renumbering's n keys
                g->tarc.alloc((size_t)nnz * 4);
                hip_check(hipMemcpyAsync(g->tarc.p, from.p, (size_t)nnz * 4,
                                         hipMemcpyDeviceToDevice, st),
                          "copy");
            }
        } else if (nnz > 0) {
            const uint32_t *vals =
                sort_arcs(nnz, head, nullptr, 0, colbits, nullptr, 0, nullptr, tmp, st);
            g->tarc.alloc((size_t)nnz * 4);
            if (!g->packed)
                g->twt.alloc((size_t)nnz * 4);
            hipLaunchKernelGGL(k_transpose_arcs, GRID(nnz), st, nnz, vals, tail, wt,
                               (int)g->packed, g->wshift, g->wmask, (uint32_t *)g->tarc.p,
                               g->packed ? nullptr : (int32_t *)g->twt.p);
            hip_check(hipGetLastError(), "transpose");
            if (want_edges) {
                through.alloc((size_t)nnz * 4);
                hip_check(hipMemcpyAsync(through.p, vals, (size_t)nnz * 4,
                                         hipMemcpyDeviceToDevice, st),
                          "copy");
            }
        }
    } else if (sorts) {
        const int wb = bit_width_u64((uint64_t)wmax);
        DevBuf fwd, by_w;
        fwd.alloc((size_t)nnz * 4);
        by_w.alloc((size_t)nnz * 4);
        tmp.reserve(nnz, 2 * colbits <= 32 ? 4 : 8, 0);
        const uint32_t *vals = sort_arcs(nnz, tail, head, colbits, 2 * colbits, wt, wb,
                                         (uint32_t *)by_w.p, tmp, st);
        hip_check(hipMemcpyAsync(fwd.p, vals, (size_t)nnz * 4, hipMemcpyDeviceToDevice, st),
                  "copy");
        vals = sort_arcs(nnz, head, tail, colbits, 2 * colbits, wt, wb, (uint32_t *)by_w.p, tmp,
                         st);
        DevBuf mis;
        mis.alloc(4);
        hip_check(launch_fill_u32((uint32_t *)mis.p, 1, 0u, st), "clear");
        if (want_edges)
            through.alloc((size_t)nnz * 4);
        hipLaunchKernelGGL(k_pair_reverse, GRID(nnz), st, nnz, (const uint32_t *)fwd.p, vals, head,
                           tail, wt, want_edges ? (uint32_t *)through.p : nullptr,
                           (unsigned int *)mis.p);
        hip_check(hipGetLastError(), "symmetry");
        unsigned int bad = 0;
        hip_check(hipMemcpyAsync(&bad, mis.p, 4, hipMemcpyDeviceToHost, st), "symmetry");
        hip_check(hipStreamSynchronize(st), "symmetry");
        if (bad)
            throw not_symmetric();
    }

    // 6. edge map: in-row position -> caller arc index
    if (want_edges && nnz > 0) {
        g->emap.alloc((size_t)nnz * 4);
        // in-row position p of an undirected graph holds the reverse of arc p
        const uint32_t *const pairs = (const uint32_t *)rev.p;
        const uint32_t *const via = pairs && renumber ? ce : pairs;
        hipLaunchKernelGGL(k_emap, GRID(nnz), st, nnz, pairs ? via : (const uint32_t *)through.p,
                           !renumber ? nullptr : pairs ? pairs : ce, (uint32_t *)g->emap.p);
        hip_check(hipGetLastError(), "edge map");
    }
    g->edges_ready = want_edges;
    set_inarc_bound(g, st);
}
