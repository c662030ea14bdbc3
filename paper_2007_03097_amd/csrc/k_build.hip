// Keys, sort and snapshot (Sec. 2.1 "Tree topology" of arXiv:2007.03097, Fig. 1).
//
//  * k_bbox      exact per-segment bounding box (ordered-integer atomics, order independent)
//  * k_keys      quantise to B bits inside the cubic root cell, interleave (x lowest) or
//                Hilbert index, sentinel bit 63, segment number in bits 54..62 for
//                segmented sets
//  * merge sort  (key, value) with ties by particle ID: the (key, ID) order of the paper
#include <utility>

#include "common.h"

// ---------------------------------------------------------------------------------------
// fills
__global__ void k_fill_i32(int* p, int v, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}
static int grid_for(int n, int bs = 256, int cap = 4096) {
    int g = (n + bs - 1) / bs;
    return g < 1 ? 1 : (g > cap ? cap : g);
}
void launch_fill_i32(hipStream_t s, int* p, int v, int n) {
    if (n > 0) hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n)), dim3(256), 0, s, p, v, n);
}

// ---------------------------------------------------------------------------------------
// bounding box per segment.  The chunk table splits [0, n) into pieces that never cross a
// segment boundary; one block reduces a chunk and folds it into the segment's box with
// exact atomic min/max on an order-preserving integer encoding.
__global__ void k_box_init(DevCtl* ctl, int n_seg) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < n_seg) {
        for (int c = 0; c < 3; ++c) {
            ctl->box_enc[6 * s + c] = ~0ull;
            ctl->box_enc[6 * s + 3 + c] = 0ull;
        }
    }
}

// With all atomics on one box 4M positions took 104 us, of which reading them is 20 (4,096 workgroups
// x 6 atomics on the same addresses); over 64 boxes 28 us (1M: 28 -> 9 us).
__global__ void __launch_bounds__(256) k_bbox(DevCtl* ctl, const int4* chunk, int batched, const double* __restrict__ x,
                                               const double* __restrict__ y, const double* __restrict__ z) {
    const int4 ch = chunk[blockIdx.x];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i0 = ch.x; i0 < ch.y; i0 += 1024) {
        double v[4][3];
#pragma unroll
        for (int k = 0; k < 4; ++k) {  // twelve loads in flight; past the end the chunk's last particle again
            const int i = min(i0 + k * 256 + (int)threadIdx.x, ch.y - 1);
            v[k][0] = x[i];
            v[k][1] = y[i];
            v[k][2] = z[i];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lo[c] = fmin(lo[c], v[k][c]);
                hi[c] = fmax(hi[c], v[k][c]);
            }
    }
    box_block_merge(ctl, batched ? ch.z : (int)(blockIdx.x & (BOX_SLOTS - 1)), lo, hi, ch.y > ch.x);
}

void launch_box_init(hipStream_t s, const DevPtrs& d, const Dims& dm) {
    hipLaunchKernelGGL(k_box_init, dim3((dm.n_seg + 255) / 256), dim3(256), 0, s, d.ctl, dm.n_seg);
}

void launch_bbox(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* x, const double* y, const double* z) {
    const int slots = dm.batched ? dm.n_seg : BOX_SLOTS;
    hipLaunchKernelGGL(k_box_init, dim3((slots + 255) / 256), dim3(256), 0, s, d.ctl, slots);
    if (dm.n_chunks > 0)
        hipLaunchKernelGGL(k_bbox, dim3(dm.n_chunks), dim3(256), 0, s, d.ctl, d.chunk, dm.batched, x, y, z);
}

// Decode the boxes (unless the caller supplied them) and derive L and S = 2^B / L.
__global__ void k_set_box(DevCtl* ctl, int n_seg, int bits, int from_host) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (!from_host && bits == 21) {  // one set: merge the BOX_SLOTS accumulators
        for (int c = 0; c < 6; ++c) {
            u64 e = c < 3 ? ~0ull : 0ull;
            if (threadIdx.x < BOX_SLOTS) e = ctl->box_enc[6 * threadIdx.x + c];
            for (int d = 32; d >= 1; d >>= 1) {
                const u64 o = __shfl_xor(e, d, 64);
                e = c < 3 ? (o < e ? o : e) : (o > e ? o : e);
            }
            if (threadIdx.x == 0) ctl->box[c] = dec_double(e);
        }
    }
    if (s >= n_seg) return;
    if (!from_host && bits != 21)
        for (int c = 0; c < 6; ++c) ctl->box[6 * s + c] = dec_double(ctl->box_enc[6 * s + c]);
    double L = 0.0;
    for (int c = 0; c < 3; ++c) {
        double e = ctl->box[6 * s + 3 + c] - ctl->box[6 * s + c];
        if (e > L) L = e;
    }
    double S = 0.0;
    if (L > 0.0) {
        S = (double)(1u << bits) / L;   // one IEEE division
        if (!isfinite(S)) S = 0.0;
    }
    ctl->scale[s] = S;
    ctl->side[s] = L;
}

void launch_set_box(hipStream_t s, const DevPtrs& d, const Dims& dm, int from_host_box) {
    hipLaunchKernelGGL(k_set_box, dim3((dm.n_seg + 255) / 256), dim3(256), 0, s, d.ctl, dm.n_seg,
                       dm.batched ? 18 : 21, from_host_box);
}

// ---------------------------------------------------------------------------------------
// keys
__device__ __forceinline__ u64 spread3(u32 v) {
    u64 x = v & 0x1fffffu;
    x = (x | (x << 32)) & 0x001f00000000ffffull;
    x = (x | (x << 16)) & 0x001f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Hilbert index of grid cell (x, y, z) on a 2^bits grid: Skilling's transposition
// (J. Skilling, AIP Conf. Proc. 707, 381 (2004)) unrolled for three axes, then one 3-bit
// digit per level with x in its high bit.
__device__ __forceinline__ u64 hilbert3(u32 x, u32 y, u32 z, int bits) {
    const u32 top = 1u << (bits - 1);
    for (u32 q = top; q > 1u; q >>= 1) {
        const u32 low = q - 1u;
        if (x & q) x ^= low;
        if (y & q) {
            x ^= low;
        } else {
            const u32 t = (x ^ y) & low;
            x ^= t;
            y ^= t;
        }
        if (z & q) {
            x ^= low;
        } else {
            const u32 t = (x ^ z) & low;
            x ^= t;
            z ^= t;
        }
    }
    y ^= x;
    z ^= y;
    u32 flip = 0u;
    for (u32 q = top; q > 1u; q >>= 1)
        if (z & q) flip ^= q - 1u;
    x ^= flip;
    y ^= flip;
    z ^= flip;
    return spread3(z) | (spread3(y) << 1) | (spread3(x) << 2);
}

__device__ __forceinline__ u64 make_key(double x, double y, double z, const double* lo, double S, int seg,
                                        int batched, int curve) {
    const int bits = batched ? 18 : 21;
    const u32 top = (1u << bits) - 1u;
    const u32 qx = quantise(x, lo[0], S, top), qy = quantise(y, lo[1], S, top), qz = quantise(z, lo[2], S, top);
    const u64 m = curve ? hilbert3(qx, qy, qz, bits) : (spread3(qx) | (spread3(qy) << 1) | (spread3(qz) << 2));
    u64 k = (1ull << 63) | m;
    if (batched) k |= (u64)seg << 54;
    return k;
}

// Caller-order keys + input validation.  Each particle is also written as one 64-byte record
// (x, y, z, h), (vx, vy, vz, m) in caller order, from which the gather into key order reads it: one
// line per particle and u instead of nine (InputMove in k_tree.hip).
__global__ void __launch_bounds__(256) k_keys(DevCtl* ctl, const int4* chunk, int batched, int curve,
                                               const double* __restrict__ x, const double* __restrict__ y,
                                               const double* __restrict__ z, const double* __restrict__ vx,
                                               const double* __restrict__ vy, const double* __restrict__ vz,
                                               const double* __restrict__ m, const double* __restrict__ h,
                                               const double* __restrict__ u, u64* key, u64* key_out,
                                               double4* __restrict__ rec) {
    const int4 ch = chunk[blockIdx.x];
    u32 bad = 0;
    for (int i = ch.x + threadIdx.x; i < ch.y; i += blockDim.x) {
        double px = x[i], py = y[i], pz = z[i];
        const double wx = vx[i], wy = vy[i], wz = vz[i], hh = h[i], mm = m[i];
        if (!isfinite(px) || !isfinite(py) || !isfinite(pz) || !isfinite(wx) || !isfinite(wy) ||
            !isfinite(wz) || !isfinite(u[i]))
            bad |= ERR_NONFINITE;
        if (!(hh > 0.0) || !(mm > 0.0) || !isfinite(hh) || !isfinite(mm)) bad |= ERR_NONPOSITIVE;
        rec[2 * (size_t)i] = make_double4(px, py, pz, hh);
        rec[2 * (size_t)i + 1] = make_double4(wx, wy, wz, mm);
        u64 k = make_key(px, py, pz, ctl->box + 6 * ch.z, ctl->scale[ch.z], ch.z, batched, curve);
        key[i] = k;
        if (key_out) key_out[i] = k;
    }
    if (bad) set_err(ctl, bad);
}

void launch_keys(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* x, const double* y,
                 const double* z, const double* vx, const double* vy, const double* vz, const double* m,
                 const double* h, const double* u, u64* keys_out_caller) {
    if (dm.n_chunks > 0)
        hipLaunchKernelGGL(k_keys, dim3(dm.n_chunks), dim3(256), 0, s, d.ctl, d.chunk, dm.batched, dm.curve, x, y, z, vx, vy,
                           vz, m, h, u, d.key_b, keys_out_caller, d.rec);
}

// Step-loop keys, in the previous key order, which the sort takes as it is (it orders equal
// keys by ID itself): nearly sorted input, and no scatter to the caller's order.  The positions
// were checked for non-finite values by the kick-drift that wrote them.  (Made in the sort's tile
// kernel instead, the keys of 4,096 particles keep one CU busy for 7 us, against 3 us for this launch.)
__global__ void __launch_bounds__(256) k_step_keys(DevCtl* ctl, const int4* chunk, int batched, int curve,
                                                    const double* __restrict__ x, const double* __restrict__ y,
                                                    const double* __restrict__ z, u64* key) {
    const int4 ch = chunk[blockIdx.x];
    // the segment's box from the merged encodings, L and S = 2^B / L (one IEEE division);
    // the segment's first chunk publishes them for the tree build
    double box[6];
    for (int c = 0; c < 6; ++c) box[c] = dec_double(ctl->box_enc[6 * ch.z + c]);
    double L = 0.0;
    for (int c = 0; c < 3; ++c) L = fmax(L, box[3 + c] - box[c]);
    double S = 0.0;
    if (L > 0.0) {
        S = (double)(1u << (batched ? 18 : 21)) / L;
        if (!isfinite(S)) S = 0.0;
    }
    if (ch.w && threadIdx.x < 6) {
        ctl->box[6 * ch.z + threadIdx.x] = box[threadIdx.x];
        if (threadIdx.x == 0) {
            ctl->scale[ch.z] = S;
            ctl->side[ch.z] = L;
        }
    }
    for (int p = ch.x + threadIdx.x; p < ch.y; p += blockDim.x)
        key[p] = make_key(x[p], y[p], z[p], box, S, ch.z, batched, curve);
}

static void launch_step_keys(hipStream_t s, const DevPtrs& d, const Dims& dm) {
    if (dm.n_chunks > 0)
        hipLaunchKernelGGL(k_step_keys, dim3(dm.n_chunks), dim3(256), 0, s, d.ctl, d.chunk, dm.batched, dm.curve, d.x,
                           d.y, d.z, d.key_b);
}

// ---------------------------------------------------------------------------------------
// scans (exclusive), 256 threads x 8 items per block
constexpr int SC_THREADS = 256, SC_ITEMS = 8, SC_TILE = SC_THREADS * SC_ITEMS;

template <typename T>
__device__ T block_excl_scan(T v, T* total) {
    __shared__ T wsum[SC_THREADS / 64];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        T t = __shfl_up(x, d, 64);
        if (lane >= d) x += t;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    T off = 0, tot = 0;
    for (int k = 0; k < SC_THREADS / 64; ++k) {
        if (k < w) off += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

template <typename T>
__global__ void __launch_bounds__(SC_THREADS) k_scan_reduce(const T* __restrict__ in, int n, T* sums) {
    const int base = blockIdx.x * SC_TILE + threadIdx.x * SC_ITEMS;
    T s = 0;
#pragma unroll
    for (int k = 0; k < SC_ITEMS; ++k)
        if (base + k < n) s += in[base + k];
    T tot;
    block_excl_scan<T>(s, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

template <typename T>
__global__ void __launch_bounds__(SC_THREADS) k_scan_top(T* sums, int nb) {
    T carry = 0;
    for (int b0 = 0; b0 < nb; b0 += SC_TILE) {
        T v[SC_ITEMS];
        T s = 0;
#pragma unroll
        for (int k = 0; k < SC_ITEMS; ++k) {
            int i = b0 + threadIdx.x * SC_ITEMS + k;
            v[k] = (i < nb) ? sums[i] : (T)0;
            s += v[k];
        }
        T tot;
        T e = block_excl_scan<T>(s, &tot) + carry;
#pragma unroll
        for (int k = 0; k < SC_ITEMS; ++k) {
            int i = b0 + threadIdx.x * SC_ITEMS + k;
            if (i < nb) sums[i] = e;
            e += v[k];
        }
        carry += tot;
        __syncthreads();
    }
}

template <typename T>
__global__ void __launch_bounds__(SC_THREADS) k_scan_down(const T* __restrict__ in, T* out, int n,
                                                          const T* __restrict__ sums, int write_total) {
    const int base = blockIdx.x * SC_TILE + threadIdx.x * SC_ITEMS;
    T v[SC_ITEMS];
    T s = 0;
#pragma unroll
    for (int k = 0; k < SC_ITEMS; ++k) {
        v[k] = (base + k < n) ? in[base + k] : (T)0;
        s += v[k];
    }
    T tot;
    T e = block_excl_scan<T>(s, &tot) + sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < SC_ITEMS; ++k) {
        if (base + k < n) out[base + k] = e;
        if (write_total && base + k == n - 1) out[n] = e + v[k];
        e += v[k];
    }
}

// Down-sweep that first sums the block totals of the blocks before it (sums[] holds the
// totals of k_scan_reduce, not yet scanned): for up to SCAN_FUSE_MAX blocks this costs less
// than a separate one-workgroup launch over the totals.
constexpr int SCAN_FUSE_MAX = 4096;

template <typename T>
__global__ void __launch_bounds__(SC_THREADS) k_scan_down_fused(const T* __restrict__ in, T* out, int n,
                                                                const T* __restrict__ sums, int write_total) {
    T pre = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += SC_THREADS) pre += sums[i];
    T pre_tot;
    block_excl_scan<T>(pre, &pre_tot);
    const int base = blockIdx.x * SC_TILE + threadIdx.x * SC_ITEMS;
    T v[SC_ITEMS];
    T s = 0;
#pragma unroll
    for (int k = 0; k < SC_ITEMS; ++k) {
        v[k] = (base + k < n) ? in[base + k] : (T)0;
        s += v[k];
    }
    T tot;
    T e = block_excl_scan<T>(s, &tot) + pre_tot;
#pragma unroll
    for (int k = 0; k < SC_ITEMS; ++k) {
        if (base + k < n) out[base + k] = e;
        if (write_total && base + k == n - 1) out[n] = e + v[k];
        e += v[k];
    }
}

template <typename T>
__global__ void k_zero_one(T* p) {
    if (threadIdx.x == 0) p[0] = (T)0;
}

template <typename T>
static void scan_impl(hipStream_t s, const T* in, T* out, int n, void* tmp, int write_total) {
    if (n <= 0) {
        if (write_total) hipLaunchKernelGGL(k_zero_one<T>, dim3(1), dim3(64), 0, s, out);
        return;
    }
    const int nb = (n + SC_TILE - 1) / SC_TILE;
    T* sums = (T*)tmp;
    hipLaunchKernelGGL(k_scan_reduce<T>, dim3(nb), dim3(SC_THREADS), 0, s, in, n, sums);
    if (nb <= SCAN_FUSE_MAX) {
        hipLaunchKernelGGL(k_scan_down_fused<T>, dim3(nb), dim3(SC_THREADS), 0, s, in, out, n, (const T*)sums,
                           write_total);
        return;
    }
    hipLaunchKernelGGL(k_scan_top<T>, dim3(1), dim3(SC_THREADS), 0, s, sums, nb);
    hipLaunchKernelGGL(k_scan_down<T>, dim3(nb), dim3(SC_THREADS), 0, s, in, out, n, (const T*)sums, write_total);
}

// out[0..n) = exclusive scan, out[n] = total
void scan_i64_inplace(hipStream_t s, int64_t* a, int n, void* tmp) {
    scan_impl<long long>(s, (const long long*)a, (long long*)a, n, tmp, 1);
}

// ---------------------------------------------------------------------------------------
// Merge sort of (u64 key, u32 value), value = the input index: tiles of MS_TILE keys sorted in
// LDS by one workgroup each (two resident per CU), then merge passes: 2-way over runs that double (merge path:
// every workgroup finds where its MS_OUT outputs start in both runs and merges them in LDS), or by rank
// over four or eight runs (k_ms_rank below).  Sets of up to RANK_MAX keys skip both (k_rank_sort).
//
// Equal keys are ordered by `tie[value]` (the particle ID; tie == nullptr: the value itself), in
// the comparison, so the input may be in any order: the step sorts from the previous key order,
// which needs no scatter of its keys to the caller's order, and nearly sorted input makes most
// merge tiles plain copies.
//
// What bounds it: launches for small sets; LDS reads in the tiles, memory in the passes for
// large ones.  Measured per sort against an LSD radix sort of 8-bit digits (8 passes of three
// kernels at any size, for 63 key bits): 4,096 keys 134 -> 15-21 us (6.5 us by rank, below), 123K 144 -> 59 us
// (43 by more ways), 1M 183 -> 101 us (a pass 8.9 us, 2.7 TB/s; the tiles 30 us; 95 by four ways), 4M 400 -> 365 us
// (a pass 28 us, 3.6 TB/s).
// Tiles of 8,192 keys save a pass and lose as much (47 us at 1M); 8 keys a thread instead of 4
// leave fewer waves to hide the LDS latency (tiles 34 us, a pass 10.3 us at 1M).
constexpr int MS_ITEMS = 4, MS_TILE = 1024 * MS_ITEMS, MS_TILE_MID = 256 * MS_ITEMS;
constexpr int MM_ITEMS = 4, MM_THREADS = 512, MS_OUT = MM_THREADS * MM_ITEMS;
constexpr u32 MS_PAD = 0xffffffffu;  // value of a filler entry past the end of the last tile

// Slot of item i in LDS: one spare slot after every 8 items, so that the lanes of a wave, whose
// items lie MS_ITEMS apart, start in different banks.
__device__ __forceinline__ int ms_slot(int i) { return i + (i >> 3); }

// Order of two items with equal keys (rare: duplicates, and the fillers of the last tile).
template <bool TIE>
__device__ __forceinline__ bool ms_tie_less(u32 va, u32 vb, const u32* __restrict__ tie) {
    if (va == MS_PAD || vb == MS_PAD) return va != MS_PAD;  // fillers come last
    if constexpr (TIE) return tie[va] < tie[vb];
    else return va < vb;
}

// Merges ITEMS outputs of the sorted runs A = [a, ae) and B = [b, be) of LDS items, from the
// split (a, b) on.  One LDS read per output and no branch on which run it comes from; the read
// past a run's end is in bounds (the arrays have a spare slot) and unused.
template <int ITEMS, bool TIE>
__device__ __forceinline__ void ms_merge_items(const u64* sk, const u32* sv, int a, int ae, int b, int be,
                                               const u32* __restrict__ tie, u64* k, u32* v) {
    u64 ka = sk[ms_slot(a)], kb = sk[ms_slot(b)];
    u32 va = sv[ms_slot(a)], vb = sv[ms_slot(b)];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        bool b_less = kb < ka;
        if (kb == ka && a < ae && b < be) b_less = ms_tie_less<TIE>(vb, va, tie);
        const bool from_a = a < ae && (b >= be || !b_less);
        k[r] = from_a ? ka : kb;
        v[r] = from_a ? va : vb;
        a += from_a ? 1 : 0;
        b += from_a ? 0 : 1;
        const int i = ms_slot(min(from_a ? a : b, from_a ? ae : be));
        const u64 nk = sk[i];
        const u32 nv = sv[i];
        ka = from_a ? nk : ka;
        va = from_a ? nv : va;
        kb = from_a ? kb : nk;
        vb = from_a ? vb : nv;
    }
}

// Number of items that the first d outputs of the merge take from A = [a0, a0 + na) (the rest
// come from B = [b0, b0 + nb)); items of LDS.
template <bool TIE>
__device__ __forceinline__ int ms_split(const u64* sk, const u32* sv, int a0, int na, int b0, int nb, int d,
                                        const u32* __restrict__ tie) {
    int lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int ia = ms_slot(a0 + mid), ib = ms_slot(b0 + d - 1 - mid);
        const u64 ka = sk[ia], kb = sk[ib];
        bool b_less = kb < ka;
        if (kb == ka) b_less = ms_tie_less<TIE>(sv[ib], sv[ia], tie);
        hi = b_less ? mid : hi;
        lo = b_less ? lo : mid + 1;
    }
    return lo;
}

// One tile: every thread sorts MS_ITEMS keys in registers, then runs of that size merge in LDS.
template <bool TIE, int TILE>
__global__ void __launch_bounds__(TILE / MS_ITEMS) k_ms_tile(const u64* key, u64* kout, u32* vout, int n,
                                                        const u32* __restrict__ tie) {
    __shared__ u64 sk[TILE + TILE / 8 + 1];
    __shared__ u32 sv[TILE + TILE / 8 + 1];
    const int t0 = blockIdx.x * TILE;
    const int cnt = n - t0 < TILE ? n - t0 : TILE;
    const int i0 = threadIdx.x * MS_ITEMS;
#pragma unroll
    for (int r = 0; r < MS_ITEMS; ++r) {  // consecutive lanes read consecutive keys
        const int i = r * (TILE / MS_ITEMS) + threadIdx.x;
        if (i < cnt) sk[ms_slot(i)] = key[t0 + i];
    }
    __syncthreads();
    u64 k[MS_ITEMS];
    u32 v[MS_ITEMS];
#pragma unroll
    for (int r = 0; r < MS_ITEMS; ++r) {
        const bool ok = i0 + r < cnt;
        k[r] = ok ? sk[ms_slot(i0 + r)] : ~0ull;
        v[r] = ok ? (u32)(t0 + i0 + r) : MS_PAD;
    }
    __syncthreads();
    if (i0 < cnt) {
#pragma unroll
        for (int s = 0; s < MS_ITEMS; ++s) {  // odd-even transposition network
#pragma unroll
            for (int r = s & 1; r + 1 < MS_ITEMS; r += 2) {
                const u64 ka = k[r], kb = k[r + 1];
                const u32 va = v[r], vb = v[r + 1];
                bool b_less = kb < ka;
                if (kb == ka) b_less = ms_tie_less<TIE>(vb, va, tie);
                k[r] = b_less ? kb : ka;
                v[r] = b_less ? vb : va;
                k[r + 1] = b_less ? ka : kb;
                v[r + 1] = b_less ? va : vb;
            }
        }
    }
    const int pad = (cnt + MS_ITEMS - 1) / MS_ITEMS * MS_ITEMS;  // items with fillers up to a whole thread
    for (int run = MS_ITEMS; run < pad; run *= 2) {
        if (i0 < pad) {
#pragma unroll
            for (int r = 0; r < MS_ITEMS; ++r) {
                sk[ms_slot(i0 + r)] = k[r];
                sv[ms_slot(i0 + r)] = v[r];
            }
        }
        __syncthreads();
        if (i0 < pad) {
            const int a0 = i0 & ~(2 * run - 1);
            const int b0 = min(a0 + run, pad), e = min(a0 + 2 * run, pad);
            const int d = i0 - a0;
            // nearly sorted input (a step's): the thread's items stay where they are when all
            // of them precede the other run (in A) or follow it (in B)
            const bool in_a = i0 < b0;
            const bool stays = b0 == e || (in_a ? k[MS_ITEMS - 1] < sk[ms_slot(b0)] : sk[ms_slot(b0 - 1)] < k[0]);
            if (!stays) {
                const int a = ms_split<TIE>(sk, sv, a0, b0 - a0, b0, e - b0, d, tie);
                ms_merge_items<MS_ITEMS, TIE>(sk, sv, a0 + a, b0, b0 + d - a, e, tie, k, v);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < MS_ITEMS; ++r) {
        if (i0 + r < cnt) {
            kout[t0 + i0 + r] = k[r];
            vout[t0 + i0 + r] = v[r];
        }
    }
}

// Splits of two diagonals of the same pair of runs in global memory, one per half wave: 32
// probes per round, so a run of 2^20 keys takes four dependent rounds of loads.
template <bool TIE>
__device__ __forceinline__ int ms_split_global(const u64* __restrict__ key, const u32* __restrict__ val, int a0, int na,
                                               int b0, int nb, int d, const u32* __restrict__ tie) {
    const int half = lane_id() >> 5, j = lane_id() & 31;
    int lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    while (__ballot(lo < hi)) {  // both halves take part until both are done
        const int step = (hi - lo + 31) / 32;
        const int c = lo + (j + 1) * step - 1;
        bool past = false;  // A's item c is not among the first d outputs
        if (lo < hi && c < hi) {
            const int ia = a0 + c, ib = b0 + d - 1 - c;
            const u64 ka = key[ia], kb = key[ib];
            past = kb < ka;
            if (kb == ka) past = ms_tie_less<TIE>(val[ib], val[ia], tie);
        }
        const u32 m = (u32)(__ballot(past) >> (32 * half));
        if (lo < hi) {
            if (m) {
                const int f = __ffs((int)m) - 1;
                hi = lo + (f + 1) * step - 1;
                lo = lo + f * step;
            } else {  // every probe below hi is taken from A
                lo = min(hi, lo + ((hi - lo) / step) * step);
            }
        }
    }
    return lo;
}

// Small sets: the place of a key is the number of keys before it.  A workgroup holds RANK_KEYS keys
// in RANK_PARTS lanes each, every lane counting over its part of all keys, which are staged in LDS
// together; equal keys (rare) are told apart by a second pass over the lanes concerned.  n^2 work on
// the whole chip against the tile sort's n log^2 n on one or two CUs: 4,096 keys 15-21 -> 6.5 us, 8,192
// (a tile sort and a merge) 34 -> 16 us; at 16,384 it would take 64 us against 40.
constexpr int RANK_THREADS = 1024, RANK_KEYS = 16, RANK_PARTS = RANK_THREADS / RANK_KEYS;
constexpr int RANK_MAX = 8192;  // keys of the largest set, which LDS holds

template <bool TIE>
__global__ void __launch_bounds__(RANK_THREADS) k_rank_sort(const u64* __restrict__ key, u64* __restrict__ kout,
                                                            u32* __restrict__ vout, int n,
                                                            const u32* __restrict__ tie) {
    __shared__ u64 sk[RANK_MAX];
    __shared__ int part[RANK_THREADS / 64][RANK_KEYS];
    // lanes l and l + 16 m of a wave hold key l % 16; wave w, lane group m: part 4 w + m
    const int kk = threadIdx.x % RANK_KEYS, p = threadIdx.x / RANK_KEYS;
    const int i = blockIdx.x * RANK_KEYS + kk;
    for (int j = threadIdx.x; j < n; j += RANK_THREADS) sk[j] = key[j];
    __syncthreads();
    const u64 mine = i < n ? sk[i] : 0ull;
    int less = 0, same = 0;
#pragma unroll 4
    for (int j = p; j < n; j += RANK_PARTS) {
        const u64 k = sk[j];
        less += k < mine ? 1 : 0;
        same += k == mine ? 1 : 0;
    }
    if (i < n && same > (i % RANK_PARTS == p ? 1 : 0)) {  // other keys equal to this one
        for (int j = p; j < n; j += RANK_PARTS)
            if (sk[j] == mine && j != i && (TIE ? tie[j] < tie[i] : j < i)) ++less;
    }
    less += __shfl_xor(less, 16, 64);
    less += __shfl_xor(less, 32, 64);
    if (lane_id() < RANK_KEYS) part[threadIdx.x >> 6][kk] = less;
    __syncthreads();
    if (threadIdx.x < RANK_KEYS && i < n) {
        int r = 0;
#pragma unroll
        for (int w = 0; w < RANK_THREADS / 64; ++w) r += part[w][kk];
        kout[r] = mine;
        vout[r] = (u32)i;
    }
}

// One merge pass: pairs of runs of `run` keys.
template <bool TIE>
__global__ void __launch_bounds__(MM_THREADS) k_ms_merge(const u64* __restrict__ kin, const u32* __restrict__ vin,
                                                         u64* __restrict__ kout, u32* __restrict__ vout, int n, int run,
                                                         const u32* __restrict__ tie) {
    __shared__ u64 sk[MS_OUT + MS_OUT / 8 + 1];
    __shared__ u32 sv[MS_OUT + MS_OUT / 8 + 1];
    __shared__ int split[2];
    const int o = blockIdx.x * MS_OUT;
    const int on = n - o < MS_OUT ? n - o : MS_OUT;
    const int p0 = (int)((long long)o / (2ll * run) * (2ll * run));  // first key of the pair of runs
    const int na = min(run, n - p0), nb = min(run, n - p0 - na);
    const int d0 = o - p0;
    if (threadIdx.x < 64) {
        const int d = (lane_id() >> 5) ? d0 + on : d0;
        const int a = ms_split_global<TIE>(kin, vin, p0, na, p0 + na, nb, d, tie);
        if ((lane_id() & 31) == 0) split[lane_id() >> 5] = a;
    }
    __syncthreads();
    const int a0 = split[0], ca = split[1] - a0, cb = on - ca, b0 = d0 - a0;
    const u64* ka = kin + p0 + a0;
    const u32* va = vin + p0 + a0;
    const u64* kb = kin + p0 + na + b0;
    const u32* vb = vin + p0 + na + b0;
    if (ca == 0 || cb == 0) {  // the tile comes from one run
        const u64* ks = cb == 0 ? ka : kb;
        const u32* vs = cb == 0 ? va : vb;
        for (int i = threadIdx.x; i < on; i += MM_THREADS) {
            kout[o + i] = ks[i];
            vout[o + i] = vs[i];
        }
        return;
    }
    for (int i = threadIdx.x; i < on; i += MM_THREADS) {
        const bool A = i < ca;
        sk[ms_slot(i)] = A ? ka[i] : kb[i - ca];
        sv[ms_slot(i)] = A ? va[i] : vb[i - ca];
    }
    __syncthreads();
    const int i0 = threadIdx.x * MM_ITEMS;
    u64 k[MM_ITEMS];
    u32 v[MM_ITEMS];
    if (i0 < on) {
        const int a = ms_split<TIE>(sk, sv, 0, ca, ca, cb, i0, tie);
        ms_merge_items<MM_ITEMS, TIE>(sk, sv, a, ca, ca + i0 - a, on, tie, k, v);
    }
    __syncthreads();
    if (i0 < on) {
#pragma unroll
        for (int r = 0; r < MM_ITEMS; ++r) {
            if (i0 + r < on) {
                sk[ms_slot(i0 + r)] = k[r];
                sv[ms_slot(i0 + r)] = v[r];
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < on; i += MM_THREADS) {
        kout[o + i] = sk[ms_slot(i)];
        vout[o + i] = sv[ms_slot(i)];
    }
}

// One K-way merge pass over runs of `run` (a power of two, at least MR_THREADS) keys.  A workgroup takes
// MR_THREADS consecutive keys of a run.  Where its first and last key belong in the other K - 1 runs is found
// by half waves, 32 probes a round; the keys between go to LDS, where every thread finds the places of its
// own key by K - 1 binary searches side by side.  Its place is the sum.  Keys that crowd in few places of
// other runs (more than MR_STAGE of them) are searched in memory.
constexpr int MR_THREADS = 512, MR_STAGE = 4608;  // (one spare item: a run without items reads there)

template <bool TIE, int K>
__global__ void __launch_bounds__(MR_THREADS) k_ms_rank(const u64* __restrict__ kin, const u32* __restrict__ vin,
                                                        u64* __restrict__ kout, u32* __restrict__ vout, int n, int run,
                                                        const u32* __restrict__ tie) {
    __shared__ u64 sk[MR_STAGE + 1];
    __shared__ int bound[2][K - 1];
    const int i0 = blockIdx.x * MR_THREADS, i = i0 + threadIdx.x;
    const int p0 = (int)((long long)i0 / ((long long)K * run) * ((long long)K * run));  // first key of the K runs
    const int own = (i0 - p0) / run;
    auto start = [&](int r) { return (int)min(p0 + (long long)(r < own ? r : r + 1) * run, (long long)n); };
    u64 mine = 0;
    u32 v = 0;
    if (i < n) {
        mine = kin[i];
        v = vin[i];
    }
    {
        const int half = lane_id() >> 5, j = lane_id() & 31;
        const int e = half ? min(i0 + MR_THREADS, n) - 1 : i0;  // the last or the first key
        const u64 ke = kin[e];
        const u32 ve = vin[e];
        for (int r = threadIdx.x >> 6; r < K - 1; r += MR_THREADS / 64) {
            const int at = start(r);
            int lo = 0, hi = min(run, n - at);
            while (__ballot(lo < hi)) {  // both halves take part until both are done
                const int step = (hi - lo + 31) / 32;
                const int c = lo + (j + 1) * step - 1;
                bool past = false;  // item c does not precede the key
                if (lo < hi && c < hi) {
                    const u64 k = kin[at + c];
                    past = ke < k;
                    if (k == ke) past = ms_tie_less<TIE>(ve, vin[at + c], tie);
                }
                const u32 m = (u32)(__ballot(past) >> (32 * half));
                if (lo < hi) {
                    if (m) {
                        const int f = __ffs((int)m) - 1;
                        hi = lo + (f + 1) * step - 1;
                        lo = lo + f * step;
                    } else {
                        lo = min(hi, lo + ((hi - lo) / step) * step);
                    }
                }
            }
            if (j == 0) bound[half][r] = lo;
        }
    }
    __syncthreads();
    int at[K - 1], len[K - 1], off[K - 1], total = 0, longest = 1;
    int o = p0 + (i - p0) % run;
#pragma unroll
    for (int r = 0; r < K - 1; ++r) {
        const int lo = __builtin_amdgcn_readfirstlane(bound[0][r]);
        at[r] = start(r) + lo;
        len[r] = __builtin_amdgcn_readfirstlane(bound[1][r]) - lo;
        off[r] = total;
        total += len[r];
        longest = max(longest, len[r]);
        o += lo;
    }
    const bool staged = total <= MR_STAGE;
    if (staged) {
        constexpr int U = 4;  // loads in flight
        for (int x0 = threadIdx.x; x0 < total; x0 += U * MR_THREADS) {
            u64 k[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int x = min(x0 + q * MR_THREADS, total - 1);
                int from = at[0];
#pragma unroll
                for (int r = 1; r < K - 1; ++r) from = x >= off[r] ? at[r] - off[r] : from;
                k[q] = kin[from + x];
            }
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (x0 + q * MR_THREADS < total) sk[x0 + q * MR_THREADS] = k[q];
        }
    }
    __syncthreads();
    if (i >= n) return;
    auto search = [&](auto&& item) {
        int pos[K - 1];
#pragma unroll
        for (int r = 0; r < K - 1; ++r) pos[r] = 0;
        for (int step = 1 << (31 - __clz(longest)); step > 0; step >>= 1) {
            u64 k[K - 1];
            u32 same = 0;
#pragma unroll
            for (int r = 0; r < K - 1; ++r) k[r] = item(r, max(min(pos[r] + step, len[r]) - 1, 0));
#pragma unroll
            for (int r = 0; r < K - 1; ++r) {
                const int c = pos[r] + step;
                same |= c <= len[r] && k[r] == mine ? 1u << r : 0u;
                pos[r] = c <= len[r] && k[r] < mine ? c : pos[r];
            }
            if (same) {  // rare
#pragma unroll
                for (int r = 0; r < K - 1; ++r)
                    if (((same >> r) & 1u) && ms_tie_less<TIE>(vin[at[r] + pos[r] + step - 1], v, tie)) pos[r] += step;
            }
        }
#pragma unroll
        for (int r = 0; r < K - 1; ++r) o += pos[r];
    };
    if (staged) search([&](int r, int c) { return sk[off[r] + c]; });
    else search([&](int r, int c) { return kin[min(at[r] + c, n - 1)]; });
    kout[o] = mine;
    vout[o] = v;
}

// Sorts the keys in key_b (any order) into key_a, with the input index of each in val_a.
template <bool TIE>
static void sort_keys(hipStream_t s, const DevPtrs& d, int n, const u32* tie) {
    if (n <= 0) return;
    if (n <= RANK_MAX) {
        hipLaunchKernelGGL(k_rank_sort<TIE>, dim3((n + RANK_KEYS - 1) / RANK_KEYS), dim3(RANK_THREADS), 0, s, d.key_b,
                           d.key_a, d.val_a, n, tie);
        return;
    }
    // Middling sets do not fill the chip with tiles of 4,096 keys, and the 7 us that a pass takes there are
    // latency: tiles of 1,024 (16 us against 28) and passes of up to eight ways (8: 10-14 us, 4: 7-12 us).  Sorts,
    // us, before and so: 20,011 keys 48 -> 32, 50,021 56 -> 38, 123,480 (a step's) 58 -> 43, 200,003 75 ->
    // 57; up to 2^19 keys.  Then memory counts: four-way passes of 16 us at 1M for two of 9 up to 2^21 keys
    // (4M: 68 us for two of 28).
    const bool mid = n <= (1 << 19);
    const int tile = mid ? MS_TILE_MID : MS_TILE, most = mid ? 8 : n <= (1 << 21) ? 4 : 2;
    // the fewest passes of at most `most` ways, each with no more ways than these need
    int passes = 0, ways[32];
    for (long long run = tile; run < n; ++passes) {
        int left = 1, w = 2;
        for (long long r = most * run; r < n; r *= most) ++left;
        auto reach = [&] {
            long long r = run;
            for (int p = 0; p < left; ++p) r *= w;
            return r;
        };
        while (reach() < n) w *= 2;
        ways[passes] = w;
        run *= w;
    }
    // the tile sort starts in the buffer from which the passes end in _a
    u64 *ki = (passes & 1) ? d.key_b : d.key_a, *ko = (passes & 1) ? d.key_a : d.key_b;
    u32 *vi = (passes & 1) ? d.val_b : d.val_a, *vo = (passes & 1) ? d.val_a : d.val_b;
    auto sort_tiles = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((n + tile - 1) / tile), dim3(tile / MS_ITEMS), 0, s, d.key_b, ki, vi, n, tie);
    };
    if (mid) sort_tiles(k_ms_tile<TIE, MS_TILE_MID>);
    else sort_tiles(k_ms_tile<TIE, MS_TILE>);
    int run = tile;
    for (int p = 0; p < passes; ++p) {
        auto pass = [&](auto kern, int threads, int keys) {
            hipLaunchKernelGGL(kern, dim3((n + keys - 1) / keys), dim3(threads), 0, s, ki, vi, ko, vo, n, run, tie);
        };
        if (ways[p] == 8) pass(k_ms_rank<TIE, 8>, MR_THREADS, MR_THREADS);
        else if (ways[p] == 4) pass(k_ms_rank<TIE, 4>, MR_THREADS, MR_THREADS);
        else pass(k_ms_merge<TIE>, MM_THREADS, MS_OUT);
        run *= ways[p];
        std::swap(ki, ko);
        std::swap(vi, vo);
    }
}

// The keys in key_b, in caller order: equal keys by index.
void sort_caller_keys(hipStream_t s, const DevPtrs& d, int n) { sort_keys<false>(s, d, n, nullptr); }

// The keys of the step's new positions, in the previous key order: equal keys by particle ID.
void sort_step_keys(hipStream_t s, const DevPtrs& d, const Dims& dm) {
    launch_step_keys(s, d, dm);
    sort_keys<true>(s, d, dm.n, d.id);
}
