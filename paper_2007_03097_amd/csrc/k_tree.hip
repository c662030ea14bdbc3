// Octree over sorted keys (Sec. 2.1 "Tree topology" of arXiv:2007.03097, Fig. 1).
//
// A cell at level l is the run of sorted particles sharing the first l 3-bit digits of
// their keys.  The root (level 0) is a node; a cell is a node when its parent cell is a
// node holding more than leaf_size particles (and l <= 21); a node is a leaf when it holds
// at most leaf_size particles, or at level 21.  This is the paper's refine-until-isolated
// rule with "isolated" widened to leaf_size particles.
//
// Data-parallel construction, no recursion:
//   lcp[i]   = leading equal digits of keys i-1 and i (-1 at i = 0 and i = n): cell
//              boundaries at level l are the positions with lcp < l.
//   lvl[i]   = level of the leaf holding i = 1 + min{v : the nearest boundaries with
//              lcp <= v on both sides of i are at most leaf_size apart}, found in one
//              pass over a window of lcp values in LDS (see window_level).
//   position i starts the nodes of levels lcp[i]+1 .. lvl[i].  Breadth-first order is level by
//   level, by position within a level, so a node's index is the number of nodes at lower levels
//   plus the number of positions before it that start a node at its level: per-level counts
//   of each tile of positions, one scan of them per level, and ballots within the tile.  The
//   children of a node are then contiguous, the first one starting at the node's own position.
//   Leaves get their geometry and moments with the topology, internal nodes bottom-up from their
//   children.
//   The largest nodes holding at most 4 * group_size particles form compact "group cells";
//   each is split into target groups of at most group_size consecutive particles, so a
//   group never spans two distant cells of the space-filling curve.
#include <algorithm>
#include <type_traits>

#include "common.h"

constexpr int MAX_WIN = 64;      // largest supported leaf_size
// Positions per workgroup and tile of the kernels that number the nodes: few for small sets, which
// would not fill the chip otherwise, more for larger ones, whose tile counts are then shorter.
constexpr int TB_SMALL = 256, TB_LARGE = 1024;
constexpr int TREE_ROWS = MAX_LEVEL + 2;  // counts of a tile: nodes at levels 0 .. 21, and leaves
constexpr int GROUP_TILE = 1024;          // positions per group count

int tree_tile(int64_t n) { return n <= (1 << 18) ? TB_SMALL : TB_LARGE; }
int64_t tree_hist_words(int64_t n) {
    const int64_t small = std::min<int64_t>(n, 1 << 18);
    return TREE_ROWS * (std::max((n + TB_LARGE - 1) / TB_LARGE, (small + TB_SMALL - 1) / TB_SMALL) + 1);
}
int64_t group_hist_words(int64_t n) { return (n + GROUP_TILE - 1) / GROUP_TILE + 1; }

// Level of the smallest cell around position ci that holds at most win particles:
// 1 + min{v : the nearest boundaries with lcp <= v on both sides are at most win apart}.
// With ML(t) = min c[ci-t .. ci] and MR(k) = min c[ci+1 .. ci+k], a level v qualifies
// exactly when ML(t) <= v and MR(k) <= v for some t < win, k >= 1, t + k <= win; both
// minima only fall as t, k grow, so the smallest v is min over t of max(ML(t), MR(win - t)).
// One branch-free pass; this thread's MR(k) sits at mr[(k - 1) * TB] in LDS (threads of a
// wave write neighbouring bytes).
template <int TB>
__device__ __forceinline__ int window_level(const signed char* c, int ci, int win, signed char* mr) {
    int m = 127;
    for (int k = 1; k <= win; ++k) {
        const int v = c[ci + k];
        m = v < m ? v : m;
        mr[(k - 1) * TB] = (signed char)m;
    }
    int best = 127, ml = 127;
    for (int t = 0; t < win; ++t) {
        const int v = c[ci - t];
        ml = v < ml ? v : ml;
        const int r = mr[(win - 1 - t) * TB];
        const int x = ml > r ? ml : r;
        best = x < best ? x : best;
    }
    const int L = best + 1;
    return L > MAX_LEVEL ? MAX_LEVEL : L;
}

// window_level with the leaf capacity W known at compile time: the running minima MR(k) stay
// in registers (the same values, the same pairing of ML(t) with MR(W - t)).
template <int W>
__device__ __forceinline__ int window_level_w(const signed char* c, int ci) {
    int mr[W];
    int m = 127;
#pragma unroll
    for (int k = 1; k <= W; ++k) {
        const int v = c[ci + k];
        m = v < m ? v : m;
        mr[k - 1] = m;
    }
    int best = 127, ml = 127;
#pragma unroll
    for (int t = 0; t < W; ++t) {
        const int v = c[ci - t];
        ml = v < ml ? v : ml;
        const int r = mr[W - 1 - t];
        const int x = ml > r ? ml : r;
        best = x < best ? x : best;
    }
    const int L = best + 1;
    return L > MAX_LEVEL ? MAX_LEVEL : L;
}

// Nodes per level (lane l < 22) and leaves (lane 22) that the wave's positions start, position
// (c, L) starting one node at each of the levels c+1 .. L, the last one a leaf (none if L <= c).
__device__ __forceinline__ int wave_level_counts(int c, int L) {
    const int lane = lane_id();
    int mine = 0;
#pragma unroll
    for (int l = 0; l <= MAX_LEVEL; ++l) {
        const int k = __popcll(__ballot(c < l && l <= L));
        if (lane == l) mine = k;
    }
    const int k = __popcll(__ballot(L > c));
    return lane == MAX_LEVEL + 1 ? k : mine;
}

// What a sort is followed by: the data of sorted position q fetched from where the sort found it.
//
// Caller-order input -> key-ordered snapshot.  The caller's order is arbitrary: gathered array by
// array, every 8-byte read costs a line, and the records of k_keys cost one line for eight of
// the nine fields.  4M particles in random order: the gather 784 -> 245 us and the keys, which
// write the records, 83 -> 150 us; 1M: 179 -> 57 us and 18 -> 38 us.
struct InputMove {
    DevPtrs d;
    const double* u;
    int64_t* order_out;
    __device__ __forceinline__ void begin() const {}
    __device__ __forceinline__ void move(int q) const {
        const u32 i = d.val_a[q];
        const double4 p = d.rec[2 * (size_t)i], v = d.rec[2 * (size_t)i + 1];
        const double pu = u[i];
        d.id[q] = i;
        d.x[q] = p.x; d.y[q] = p.y; d.z[q] = p.z;
        d.vx[q] = v.x; d.vy[q] = v.y; d.vz[q] = v.z;
        d.m[q] = v.w; d.h[q] = p.w; d.u[q] = pu;
        d.pos4[q] = p;
        d.vel4[q] = v;
        if (order_out) order_out[q] = (int64_t)i;
    }
};
// New key order of a step: q <- old position val[q] (the sort carried the positions); the second
// buffer set receives the data, and the pair kernels' records pos4 = (x, h),
// vel4 = (predicted v, m) are written too.  The predicted velocities enter vel4 only: the
// next kick-drift writes them anew before anything reads them.  The step's keys are made, so
// the first workgroup also resets the box accumulators of every set for the next step's kick-drift
// (a run's first step resets them itself: other calls may use them in between).
struct StepMove {
    DevPtrs d;
    __device__ __forceinline__ void begin() const {
        if (blockIdx.x != 0) return;
        constexpr int NB = (int)(sizeof(d.ctl->box_enc) / sizeof(u64));
        for (int i = threadIdx.x; i < NB; i += blockDim.x) d.ctl->box_enc[i] = (i % 6) < 3 ? ~0ull : 0ull;
    }
    __device__ __forceinline__ void move(int q) const {
        const u32 p = d.val_a[q];
        d.id2[q] = d.id[p];
        const double px = d.x[p], py = d.y[p], pz = d.z[p], hh = d.h[p], mm = d.m[p];
        const double wx = d.vpx[p], wy = d.vpy[p], wz = d.vpz[p];
        d.x2[q] = px; d.y2[q] = py; d.z2[q] = pz;
        d.vx2[q] = d.vx[p]; d.vy2[q] = d.vy[p]; d.vz2[q] = d.vz[p];
        d.u2[q] = d.u[p]; d.m2[q] = mm; d.h2[q] = hh;
        d.up2[q] = d.up[p];
        d.pos4[q] = make_double4(px, py, pz, hh);
        d.vel4[q] = make_double4(wx, wy, wz, mm);
    }
};

// Per sorted position: its data moved into place, lcp and leaf level (leaf capacity win); per
// tile: nodes per level and leaves, hist[row * (ntiles + 1) + tile].  Also clears what later kernels
// of the build count into: the group sizes of every position and the group counts.  W > 0: the
// leaf capacity is W (= win) and the window runs in registers; W = 0: any win, through LDS.  The
// move (memory) and the window (vector ALU) share a launch:
// 62 us for 987,840 particles in a step where two kernels took 55 + 16 us, and one launch fewer.
template <int W, int TB, typename Move>
__global__ void __launch_bounds__(TB) k_order_levels(Move mv, const u64* __restrict__ key, int n, int win, int min_level,
                                                     signed char* lcp, unsigned char* lvl, int* hist, int ntiles,
                                                     u32* gsize, int* gcount) {
    __shared__ signed char c[TB + 2 * MAX_WIN + 2];
    __shared__ signed char mrow[W > 0 ? 1 : TB * MAX_WIN];
    __shared__ int wcnt[TB / 64][TREE_ROWS];
    const int b0 = blockIdx.x * TB;
    const int i = b0 + threadIdx.x;
    mv.begin();
    if (i < n) mv.move(i);
    if (threadIdx.x == 0 && b0 % GROUP_TILE == 0) gcount[b0 / GROUP_TILE] = 0;
    const int lo = b0 - win;                      // c[j] holds position lo + j
    const int cnt = TB + 2 * win + 1;
    for (int j = threadIdx.x; j < cnt; j += TB) {
        const int p = lo + j;
        int v = -1;
        if (p > 0 && p < n) v = lcp_digits(key[p - 1], key[p]);
        c[j] = (signed char)v;
    }
    __syncthreads();
    const int ci = i - lo;
    int L = -1, cc = MAX_LEVEL;
    if (i < n) {
        if constexpr (W > 0) L = window_level_w<W>(c, ci);
        else L = window_level<TB>(c, ci, win, mrow + threadIdx.x);
        if (L < min_level) L = min_level;
        cc = c[ci];
        lcp[i] = (signed char)cc;
        lvl[i] = (unsigned char)L;
        gsize[i] = 0u;
        if (i == n - 1) lcp[n] = -1;
    }
    const int mine = wave_level_counts(cc, L);
    if (lane_id() < TREE_ROWS) wcnt[threadIdx.x >> 6][lane_id()] = mine;
    __syncthreads();
    if (threadIdx.x < TREE_ROWS) {
        int t = 0;
        for (int w = 0; w < TB / 64; ++w) t += wcnt[w][threadIdx.x];
        hist[threadIdx.x * (ntiles + 1) + blockIdx.x] = t;
    }
}

// Exclusive scan over a workgroup of up to 16 full waves; total gets the sum.
__device__ __forceinline__ int block_scan(int v, int& total) {
    __shared__ int wsum[16];
    const int incl = wave_incl_scan(v), w = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
    if (lane_id() == 63) wsum[w] = incl;
    __syncthreads();
    int off = 0, tot = 0;
    for (int k = 0; k < nw; ++k) {
        if (k < w) off += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    total = tot;
    return off + incl - v;
}

// One workgroup per row: its tile counts become offsets, their total goes to the row's last word.
__global__ void __launch_bounds__(1024) k_level_scan(int* hist, int ntiles) {
    int* h = hist + (size_t)blockIdx.x * (ntiles + 1);
    const int per = (ntiles + (int)blockDim.x - 1) / (int)blockDim.x;
    const int a = min(ntiles, (int)threadIdx.x * per), e = min(ntiles, a + per);
    int t = 0;
    for (int k = a; k < e; ++k) t += h[k];
    int total;
    int off = block_scan(t, total);
    for (int k = a; k < e; ++k) {
        const int v = h[k];
        h[k] = off;
        off += v;
    }
    if (threadIdx.x == 0) h[ntiles] = total;
}

// Nodes in breadth-first order: level, first position, and the first child's index or, for a
// leaf, ~(its number among the leaves); the leaf tables; the level table of the control block.
// A tile's base index per level comes from the scanned counts, the rank within it from ballots.
// Launch latency bounds the numbering of small sets and the leaf-level window that of large ones:
// levels, counts and emission take 13 us at 4,096 particles and 34 us at 1M, where a pre-order
// numbering (scan in two launches) sorted by level (three more) took 27 and 60 us.
template <int TB>
__global__ void __launch_bounds__(TB) k_emit_nodes(int n, const signed char* __restrict__ lcp,
                                                   const unsigned char* __restrict__ lvl, const int* __restrict__ hist,
                                                   int ntiles, int scanned, unsigned char* node_level, int* node_start,
                                                   int* node_first, int* leaf_start, int* leaf_node, DevCtl* ctl,
                                                   int node_cap) {
    __shared__ int base[TREE_ROWS], offs[TREE_ROWS], tots[TREE_ROWS];
    __shared__ int wcnt[TB / 64][TREE_ROWS];
    const int w = threadIdx.x >> 6, lane = lane_id();
    const u64 lt = lanemask_lt();
    const int i = blockIdx.x * TB + threadIdx.x;
    int c = MAX_LEVEL, L = -1;
    if (i < n) {
        c = lcp[i];
        L = lvl[i];
    }
    if (!scanned) {  // few tiles: this one's offsets and the totals straight from the counts
        for (int r = w; r < TREE_ROWS; r += TB / 64) {
            int before = 0, all = 0;
            for (int t = lane; t < ntiles; t += 64) {
                const int v = hist[(size_t)r * (ntiles + 1) + t];
                all += v;
                if (t < (int)blockIdx.x) before += v;
            }
            before = wave_last(wave_incl_scan(before));
            all = wave_last(wave_incl_scan(all));
            if (lane == 0) {
                offs[r] = before;
                tots[r] = all;
            }
        }
        __syncthreads();
    }
    if (w == 0) {
        const int r = min(lane, TREE_ROWS - 1);
        const int* row = hist + (size_t)r * (ntiles + 1);
        const int tot = lane < TREE_ROWS ? (scanned ? row[ntiles] : tots[r]) : 0;
        const int nodes = lane <= MAX_LEVEL ? tot : 0;
        const int off = wave_incl_scan(nodes) - nodes;  // nodes at lower levels; all of them past the last
        if (lane < TREE_ROWS) base[lane] = (scanned ? row[blockIdx.x] : offs[r]) + (lane <= MAX_LEVEL ? off : 0);
        if (blockIdx.x == 0) {
            if (lane < 24) {
                ctl->level_count[lane] = nodes;
                ctl->level_off[lane] = off;
            }
            if (lane == TREE_ROWS - 1) {
                ctl->n_nodes = off < node_cap ? off : node_cap;
                ctl->n_leaves = tot;
                ctl->n_sub = ctl->n_big = 0;
                leaf_start[tot] = n;
                if (off > node_cap) set_err(ctl, ERR_NODE_CAP);
            }
        }
    }
    const int mine = wave_level_counts(c, L);
    if (lane < TREE_ROWS) wcnt[w][lane] = mine;
    __syncthreads();
    if (threadIdx.x < TREE_ROWS) {
        int t = base[threadIdx.x];
        for (int k = 0; k < TB / 64; ++k) {
            const int v = wcnt[k][threadIdx.x];
            wcnt[k][threadIdx.x] = t;
            t += v;
        }
    }
    __syncthreads();
    int prev = -1;
    for (int l = 0; l <= MAX_LEVEL; ++l) {
        const bool in = c < l && l <= L;
        const u64 bal = __ballot(in);
        if (!in) continue;
        const int idx = wcnt[w][l] + __popcll(bal & lt);
        if (idx < node_cap) {
            node_level[idx] = (unsigned char)l;
            node_start[idx] = i;
        }
        if (prev >= 0 && prev < node_cap) node_first[prev] = idx;
        prev = idx;
    }
    const u64 bal = __ballot(L > c);
    if (L > c) {
        const int lf = wcnt[w][MAX_LEVEL + 1] + __popcll(bal & lt);
        if (prev < node_cap) node_first[prev] = ~lf;
        leaf_start[lf] = i;
        leaf_node[lf] = prev;
    }
}

// Group cells: the largest nodes holding at most gcap particles (at or below min_level),
// plus leaves that hold more (runs of equal keys).  They partition the sorted particles.
// Each is cut into target groups of at most gsz consecutive particles: the group's size is
// recorded at its first position, and the groups of each tile of positions are counted: one atomic
// for the lanes of a wave whose cells start in the same tile (nodes are in breadth-first order, so
// these are neighbours; one atomic a group took 36 us for 100,000 groups of 16, 5.5 so).
__global__ void k_group_starts(const DevCtl* __restrict__ ctl, int gcap, int gsz, int min_level,
                               const int4* __restrict__ topo, const int* __restrict__ parent,
                               const int2* __restrict__ range, u32* gsize, int* gcount) {
    const int nn = ctl->n_nodes;
    for (int b0 = blockIdx.x * blockDim.x; b0 < nn; b0 += gridDim.x * blockDim.x) {
        const int b = b0 + threadIdx.x;
        int tile = -1, count = 0;
        if (b < nn) {
            const int4 tp = topo[b];
            const int2 r = range[b];
            const int p = parent[b];
            const bool fits = r.y <= gcap && tp.z >= min_level;
            bool pfits = false;
            if (p >= 0) pfits = range[p].y <= gcap && topo[p].z >= min_level;
            if ((fits || tp.w) && !pfits) {
                const int e = r.x + r.y;
                tile = r.x / GROUP_TILE;
                for (int k = r.x; k < e; k += gsz) {
                    gsize[k] = (u32)min(gsz, e - k);
                    if (k / GROUP_TILE == tile) ++count;
                    else atomicAdd(&gcount[k / GROUP_TILE], 1);
                }
            }
        }
        u64 todo = __ballot(count > 0);
        while (todo) {
            const int t = __builtin_amdgcn_readlane(tile, __builtin_ctzll(todo));
            const bool same = count > 0 && tile == t;
            const u64 m = __ballot(same);
            const int sum = wave_last(wave_incl_scan(same ? count : 0));
            if (lane_id() == 0) atomicAdd(&gcount[t], sum);
            todo &= ~m;
        }
    }
}

// Target groups in sorted order; a tile's first group follows those of the tiles before it, which
// the workgroup adds up itself.
__global__ void __launch_bounds__(GROUP_TILE) k_emit_groups(int n, int batched, DevCtl* ctl,
                                                            const u32* __restrict__ gsize,
                                                            const int* __restrict__ gcount,
                                                            const u64* __restrict__ key,
                                                            const int* __restrict__ seg_root_rank, int4* group) {
    const int i = blockIdx.x * GROUP_TILE + threadIdx.x;
    const u32 sz = i < n ? gsize[i] : 0u;
    int before = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += GROUP_TILE) before += gcount[t];
    int first, own;
    block_scan(before, first);
    const int at = first + block_scan(sz ? 1 : 0, own);
    if (sz) {
        const int rank = batched ? seg_root_rank[(int)((key[i] >> 54) & 511ull)] : -1;
        group[at] = make_int4(i, (int)sz, rank, 0);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) ctl->n_groups = first + own;
}

// Order in which the workgroups take their units (target groups, or leaves for leaf_info): within each
// XCD's contiguous share, the units of most targets first, so that what is left at the end is short (a
// unit takes 100 to 400 us whatever the set's size).  Before them the heavy leaves: the at most 16
// coarsest ones that lie two levels or more above the share's average, and with at most wide_leaves leaves in
// all every one of 16 particles and more (launch_fmm).  One workgroup per share counts
// and places its units.  Gravity, 1,000,003 particles in groups of 64, FP32C: 1.96 -> 1.80 ms; 131,101 in
// groups of 32, FP64: 0.451 -> 0.370 ms; 4,194,304: 12.78 -> 12.61.  What is left of its own time are the passes
// over a share's units, a load each: a leaf's level and particle count come in one word (k_fmm_cells) in
// leaf order, where the leaf's node and its record took two dependent ones (560,000 leaves 168 -> 121 us).
__global__ void __launch_bounds__(1024) k_unit_order(DevCtl* ctl, const int4* __restrict__ group,
                                                     const u32* __restrict__ leaf_info, int wide_leaves,
                                                     int* __restrict__ order) {
    __shared__ int at[65], lev[MAX_LEVEL + 1], heavy_at, cut;
    const int tid = threadIdx.x;
    if (tid < 65) at[tid] = 0;
    if (tid <= MAX_LEVEL) lev[tid] = 0;
    int u0, u1, step;  // (eight workgroups: step 1 from the share's first unit)
    group_range(leaf_info ? ctl->n_leaves : ctl->n_groups, u0, u1, step);
    __syncthreads();
    if (leaf_info) {
        for (int u = u0 + tid; u < u1; u += 1024) atomicAdd(&lev[leaf_info[u] >> 8], 1);
        __syncthreads();
    }
    if (tid == 0) {
        cut = -1;
        heavy_at = 0;
        if (leaf_info) {
            long long sum = 0, n = u1 - u0;
            for (int l = 0; l <= MAX_LEVEL; ++l) sum += (long long)l * lev[l];
            int k = 0;
            for (int l = 0; l <= MAX_LEVEL && (l + 2) * n <= sum; ++l) {
                k += lev[l];
                if (k > 16) break;
                cut = l;
            }
        }
    }
    __syncthreads();
    const int c = cut;
    const int wide = leaf_info && ctl->n_leaves <= wide_leaves ? 16 : INT_MAX;
    auto size = [&](int u) {  // 0: heavy
        if (!leaf_info) return group[u].y;
        const u32 t = leaf_info[u];
        return (int)(t >> 8) <= c || (int)(t & 0xff) >= wide ? 0 : (int)(t & 0xff);
    };
    for (int u = u0 + tid; u < u1; u += 1024) atomicAdd(&at[size(u)], 1);
    __syncthreads();
    if (tid == 0 && leaf_info) ctl->fmm_heavy[blockIdx.x] = at[0];
    if (tid < 64) {  // first place of size 64 - tid
        const int k = at[64 - tid];
        const int incl = wave_incl_scan(k);
        at[64 - tid] = at[0] + incl - k;
    }
    __syncthreads();
    for (int u = u0 + tid; u < u1; u += 1024) {
        const int z = size(u);
        order[u0 + atomicAdd(z ? &at[z] : &heavy_at, 1)] = u;
    }
}

void launch_unit_order(hipStream_t s, DevCtl* ctl, const int4* group, const u32* leaf_info, int wide_leaves, int* order) {
    hipLaunchKernelGGL(k_unit_order, dim3(8), dim3(1024), 0, s, ctl, group, leaf_info, wide_leaves, order);
}

// ---- nodes in breadth-first order: eight lanes per node
//
// Eight lanes read a node's children (at most eight), or an eighth of a leaf's particles, at
// once: the work per node is short and what it costs is the latency of its loads, which one
// thread per node paid in turn, child by child and particle by particle.  The sums stay those of
// one thread, term by term in child or particle order: the lanes put their terms of up to six
// sums into LDS and lane q adds up the eight of sum q.
constexpr int NODE_LANES = 8;
constexpr int NODE_SUMS = 6;
struct NodeSums {
    double v[NODE_SUMS][NODE_LANES + 1];  // (a spare column against bank conflicts)
};

// acc (of lane q < Q) plus the eight lanes' terms t[q], in lane order.
template <int Q>
__device__ __forceinline__ void add_in_order(NodeSums& S, int j, const double (&t)[Q], double& acc) {
    static_assert(Q <= NODE_SUMS, "one lane per sum");
#pragma unroll
    for (int q = 0; q < Q; ++q) S.v[q][j] = t[q];
    wave_lds_fence();
    const int q = j < Q ? j : 0;
#pragma unroll
    for (int k = 0; k < NODE_LANES; ++k) acc += S.v[q][k];
    wave_lds_fence();
}
__device__ __forceinline__ double min8(double v) {
#pragma unroll
    for (int d = 1; d < NODE_LANES; d <<= 1) v = fmin(v, __shfl_xor(v, d, NODE_LANES));
    return v;
}
__device__ __forceinline__ double max8(double v) {
#pragma unroll
    for (int d = 1; d < NODE_LANES; d <<= 1) v = fmax(v, __shfl_xor(v, d, NODE_LANES));
    return v;
}

struct NodeArgs {
    DevCtl* ctl;
    int n;
    int sub_max;  // largest number of particles of a subtree that one workgroup finishes; 0: cut at a level
    int* list;    // their roots and, from the end, {level, node} of the nodes above them
    int batched;
    int mass;  // build masses and moments too (gravity on), else only boxes, h_max and ranges
    const u64* key;
    int4* topo;
    int* parent;
    const double4* pos4;
    const double* m;
    double4 *nbox_lo, *nbox_hi, *mom0, *mom1, *mom2;
    int2* range;
};

// Cell side of a node at level l whose first particle is at sorted position s.
__device__ __forceinline__ double node_side(const NodeArgs& A, int s, int l) {
    const int seg = A.batched ? (int)((A.key[s] >> 54) & 511ull) : 0;
    return ldexp(A.ctl->side[seg], -l);
}

// Mass, centre of mass and second moments of node b; lane q < 6 holds second moment q in acc.
__device__ __forceinline__ void store_moments(const NodeArgs& A, int b, double M, double cx, double cy, double cz,
                                              double acc, int j) {
    const double I0 = __shfl(acc, 0, NODE_LANES), I1 = __shfl(acc, 1, NODE_LANES), I2 = __shfl(acc, 2, NODE_LANES),
                 I3 = __shfl(acc, 3, NODE_LANES), I4 = __shfl(acc, 4, NODE_LANES), I5 = __shfl(acc, 5, NODE_LANES);
    if (j != 0) return;
    A.mom0[b] = make_double4(M, cx, cy, cz);
    A.mom1[b] = make_double4(I0, I1, I2, I0 + I1 + I2);
    A.mom2[b] = make_double4(I3, I4, I5, 0.0);
}

// Leaf geometry and moments from its particles [s, s + c); lane j of the node's eight.
__device__ __forceinline__ void leaf_node(const NodeArgs& A, NodeSums& S, int b, int s, int c, double side, int j) {
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    double hmax = 0.0, acc = 0.0;
    const int e = s + c;
    for (int i0 = s; i0 < e; i0 += NODE_LANES) {
        const bool has = i0 + j < e;  // lanes past the end add zeros and repeat the first particle
        const int i = has ? i0 + j : s;
        const double4 p = A.pos4[i];
        lo[0] = fmin(lo[0], p.x); lo[1] = fmin(lo[1], p.y); lo[2] = fmin(lo[2], p.z);
        hi[0] = fmax(hi[0], p.x); hi[1] = fmax(hi[1], p.y); hi[2] = fmax(hi[2], p.z);
        hmax = fmax(hmax, p.w);
        if (A.mass) {
            const double mi = has ? A.m[i] : 0.0;
            add_in_order<4>(S, j, {mi, mi * p.x, mi * p.y, mi * p.z}, acc);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = min8(lo[k]);
        hi[k] = max8(hi[k]);
    }
    hmax = max8(hmax);
    if (j == 0) {
        A.nbox_lo[b] = make_double4(lo[0], lo[1], lo[2], hmax);
        A.nbox_hi[b] = make_double4(hi[0], hi[1], hi[2], side);
    }
    if (!A.mass) return;
    const double M = __shfl(acc, 0, NODE_LANES);
    const double cx = __shfl(acc, 1, NODE_LANES) / M, cy = __shfl(acc, 2, NODE_LANES) / M,
                 cz = __shfl(acc, 3, NODE_LANES) / M;
    acc = 0.0;
    for (int i0 = s; i0 < e; i0 += NODE_LANES) {
        const bool has = i0 + j < e;
        const int i = has ? i0 + j : s;
        const double4 p = A.pos4[i];
        const double mi = has ? A.m[i] : 0.0;
        const double dx = p.x - cx, dy = p.y - cy, dz = p.z - cz;
        add_in_order<6>(S, j, {mi * dx * dx, mi * dy * dy, mi * dz * dz, mi * dx * dy, mi * dx * dz, mi * dy * dz}, acc);
    }
    store_moments(A, b, M, cx, cy, cz, acc, j);
}

// Internal node p from its finished children: box, largest h, particle range, mass, centre of
// mass, and second moments about it (parallel-axis shifts of the children's); lane j has child j.
__device__ __forceinline__ void internal_node(const NodeArgs& A, NodeSums& S, int p, const int4 tp, int j) {
    const bool has = j < tp.y;
    const int c = tp.x + (has ? j : 0);
    const double4 a = A.nbox_lo[c], b = A.nbox_hi[c];
    const int2 r = A.range[c];
    double4 m0 = make_double4(0, 0, 0, 0), m1 = m0, m2 = m0;
    if (A.mass) {
        m0 = A.mom0[c];
        m1 = A.mom1[c];
        m2 = A.mom2[c];
    }
    int cnt = has ? r.y : 0;
#pragma unroll
    for (int d = 1; d < NODE_LANES; d <<= 1) cnt += __shfl_xor(cnt, d, NODE_LANES);
    const int s = __shfl(r.x, 0, NODE_LANES);
    // an absent child's lane repeats child 0, which changes no minimum or maximum
    const double lx = min8(a.x), ly = min8(a.y), lz = min8(a.z), hm = max8(a.w);
    const double hx = max8(b.x), hy = max8(b.y), hz = max8(b.z);
    if (j == 0) {
        A.range[p] = make_int2(s, cnt);
        A.nbox_lo[p] = make_double4(lx, ly, lz, hm);
        A.nbox_hi[p] = make_double4(hx, hy, hz, node_side(A, s, tp.z));
    }
    if (!A.mass) return;
    const double mc = has ? m0.x : 0.0;
    double acc = 0.0;
    add_in_order<4>(S, j, {mc, mc * m0.y, mc * m0.z, mc * m0.w}, acc);
    const double M = __shfl(acc, 0, NODE_LANES);
    const double cx = __shfl(acc, 1, NODE_LANES) / M, cy = __shfl(acc, 2, NODE_LANES) / M,
                 cz = __shfl(acc, 3, NODE_LANES) / M;
    const double dx = m0.y - cx, dy = m0.z - cy, dz = m0.w - cz;
    acc = 0.0;
    add_in_order<6>(S, j,
                    {has ? m1.x + mc * dx * dx : 0.0, has ? m1.y + mc * dy * dy : 0.0, has ? m1.z + mc * dz * dz : 0.0,
                     has ? m2.x + mc * dx * dy : 0.0, has ? m2.y + mc * dx * dz : 0.0, has ? m2.z + mc * dy * dz : 0.0},
                    acc);
    store_moments(A, p, M, cx, cy, cz, acc, j);
}

// A node at level l whose first particle is at sorted position s holds more than sub_max particles: so far
// on, the keys still share its digits.
__device__ __forceinline__ bool node_is_big(const NodeArgs& A, int s, int l) {
    return A.n - s > A.sub_max && lcp_digits(A.key[s], A.key[s + A.sub_max]) >= l;
}

// Appends v of the active lanes with `add` to the list of subtree roots: one atomic for all of them.
__device__ __forceinline__ void add_root(const NodeArgs& A, bool add, int v) {
    const u64 m = __ballot(add);
    if (!add) return;
    const int leader = __builtin_ctzll(m);
    int at = 0;
    if (lane_id() == leader) at = atomicAdd(&A.ctl->n_sub, (int)__popcll(m));
    A.list[__shfl(at, leader, 64) + __popcll(m & lanemask_lt())] = v;
}

// Topology of every node (leaf -> particle range; internal -> children range) and the leaves'
// geometry and moments, whatever their level: the bottom-up kernels below then only combine
// children.  With sub_max also how they share the internal nodes: those that hold more particles are
// done last, by one workgroup; the subtrees below them are handed out whole.
__global__ void __launch_bounds__(256) k_finalize(NodeArgs A, const unsigned char* __restrict__ node_level,
                                                   const int* __restrict__ node_start, const int* __restrict__ node_first,
                                                   const signed char* __restrict__ lcp,
                                                   const int* __restrict__ leaf_start) {
    __shared__ NodeSums sums[256 / NODE_LANES];
    NodeSums& S = sums[threadIdx.x / NODE_LANES];
    const int nn = A.ctl->n_nodes;
    const int j = threadIdx.x & (NODE_LANES - 1);
    const int stride = gridDim.x * (blockDim.x / NODE_LANES);
    for (int b = blockIdx.x * (blockDim.x / NODE_LANES) + threadIdx.x / NODE_LANES; b < nn; b += stride) {
        const int l = node_level[b], s = node_start[b], f = node_first[b];
        if (b == 0 && j == 0) A.parent[0] = -1;
        if (f < 0) {
            const int cnt = leaf_start[~f + 1] - s;
            if (j == 0) {
                A.topo[b] = make_int4(s, cnt, l, 1);
                A.range[b] = make_int2(s, cnt);
            }
            leaf_node(A, S, b, s, cnt, node_side(A, s, l), j);
        } else if (f >= nn) {  // only with a truncated (over-capacity) tree
            if (j == 0) {
                A.topo[b] = make_int4(s, 0, l, 1);
                A.range[b] = make_int2(s, 0);
            }
            leaf_node(A, S, b, s, 0, node_side(A, s, l), j);
        } else {
            const int end = min(nn, A.ctl->level_off[l + 1] + A.ctl->level_count[l + 1]);
            const bool child = j == 0 || (f + j < end && lcp[node_start[f + j]] >= l);
            const u32 mask = (u32)(__ballot(child) >> (lane_id() & ~(NODE_LANES - 1))) & 0xffu;
            const int nc = __ffs((int)~mask) - 1;  // children are the leading run (1 .. 8)
            if (j < nc) A.parent[f + j] = b;
            if (j == 0) A.topo[b] = make_int4(f, nc, l, 0);
            if (A.sub_max == 0) continue;
            const bool big = node_is_big(A, s, l);
            if (big && j == 0) {
                const int at = A.n - 2 - 2 * atomicAdd(&A.ctl->n_big, 1);
                A.list[at] = l;
                A.list[at + 1] = b;
            }
            bool root = b == 0 && j == 0 && !big;
            if (big && j < nc) {
                const int cf = node_first[f + j];
                root = cf >= 0 && cf < nn && !node_is_big(A, node_start[f + j], l + 1);
            }
            add_root(A, root, big ? f + j : b);
        }
    }
}

// Which subtrees are handed out whole, one workgroup each.  Sets of up to SUB_LISTED particles: those of
// the first level with at least SUB_ROOTS nodes, so that flat sets (a tube fills 64 cells at level 4) still
// occupy the chip and the levels above, which one workgroup finishes, hold few nodes.  Larger ones: those of at
// most a 128th of the particles (between the 64th and the 256th or 512th that two levels' cells hold
// in flat and in full sets); cut at a level, a cluster of half the particles within one of its cells was
// one workgroup's: 4,194,304 particles 1,365 -> 142 us.  Finding them costs 3-8 us, more than
// it saves in ordinary smaller sets.  The lists fit: at most 127 nodes a level lie above the subtrees, two words
// each, and no more than 8 roots below each, some 27,000 words of n.
constexpr int SUB_ROOTS = 256, SUB_SHARE = 128;
constexpr int TOP_MAX = (MAX_LEVEL + 1) * SUB_SHARE;
constexpr int64_t SUB_LISTED = 1 << 18;
constexpr int SUB_THREADS = 256;
__device__ __forceinline__ int subtree_cut(const DevCtl* ctl) {
    int l = 3;
    while (l < MAX_LEVEL && ctl->level_count[l] < SUB_ROOTS && ctl->level_count[l + 1] > 0) ++l;
    return l;
}

// Internal nodes of the subtrees: one workgroup finishes a whole subtree
// bottom-up.  A subtree's nodes at each level are one contiguous run in breadth-first order
// (from the first child of its first internal node to the last child of its last internal
// node), so the runs are found top-down, then the levels are done deepest first with the
// workgroup's own results as inputs.  The internal nodes are few (about one per 100 particles):
// the levels' latency bounds this kernel and k_top_moments.  Moments and finalize together,
// before (one thread per node, leaves summed in the level order, one launch per level between
// a fixed cut and the top) and now: 105 -> 32 us (131K polytrope), 337 -> 83 us (1M Evrard
// sphere), 125 -> 43 us (1.2M particles in 64 boxes), 63 -> 37 us (987,840 tube), 306 -> 245 us (4M
// polytrope).  Workgroups of 1,024 threads lose on flat sets (tube 12 -> 17 us) and gain little
// at 4M (107 -> 87 us).
__global__ void __launch_bounds__(SUB_THREADS) k_subtree_moments(NodeArgs A) {
    __shared__ NodeSums S[SUB_THREADS / NODE_LANES];
    __shared__ int run_lo[MAX_LEVEL + 1], run_hi[MAX_LEVEL + 1], deepest;
    const int lane = lane_id(), j = threadIdx.x & (NODE_LANES - 1);
    const bool listed = A.sub_max > 0;
    const int level = listed ? 0 : subtree_cut(A.ctl);
    const int nroot = listed ? A.ctl->n_sub : A.ctl->level_count[level], r0 = A.ctl->level_off[level];
    for (int ri = blockIdx.x; ri < nroot; ri += gridDim.x) {
        const int root = listed ? A.list[ri] : r0 + ri, cut = listed ? A.topo[root].z : level;
        if (threadIdx.x < 64) {  // internal nodes of each level of the subtree lie in run_lo .. run_hi
            int lo = root, hi = lo, deep = cut - 1;
            for (int l = cut; l < MAX_LEVEL; ++l) {
                int first = -1, cfirst = 0, last = -1, clast = 0;
                for (int k0 = lo; k0 <= hi && first < 0; k0 += 64) {
                    const int4 t = A.topo[min(k0 + lane, hi)];
                    const u64 bl = __ballot(k0 + lane <= hi && !t.w);
                    if (!bl) continue;
                    const int f = __ffsll((long long)bl) - 1;
                    first = k0 + f;
                    cfirst = __shfl(t.x, f, 64);
                    if (hi - k0 < 64) {  // the chunk ends the run: it holds the last one too
                        const int g = 63 - __clzll((long long)bl);
                        last = k0 + g;
                        clast = __shfl(t.x + t.y - 1, g, 64);
                    }
                }
                if (first < 0) break;
                for (int k1 = hi; last < 0; k1 -= 64) {
                    const int4 t = A.topo[max(k1 - lane, lo)];
                    const u64 bl = __ballot(k1 - lane >= lo && !t.w);
                    if (!bl) continue;
                    const int g = __ffsll((long long)bl) - 1;
                    last = k1 - g;
                    clast = __shfl(t.x + t.y - 1, g, 64);
                }
                deep = l;
                if (lane == 0) {
                    run_lo[l] = first;
                    run_hi[l] = last;
                }
                lo = cfirst;
                hi = clast;
            }
            if (lane == 0) deepest = deep;
        }
        __syncthreads();
        for (int l = deepest; l >= cut; --l) {
            const int a = run_lo[l], e = run_hi[l];
            for (int k = a + threadIdx.x / NODE_LANES; k <= e; k += SUB_THREADS / NODE_LANES) {
                const int4 tp = A.topo[k];
                if (!tp.w) internal_node(A, S[threadIdx.x / NODE_LANES], k, tp, j);
            }
            __syncthreads();
        }
        __syncthreads();  // the runs are free for the next subtree
    }
}

// Internal nodes above the subtrees in one workgroup, a barrier between levels.
// Also finds (in its last wavefront, which seldom has nodes) the level at which the neighbour walks start: the last
// one with at most WALK_START nodes and no leaf above it.
__global__ void __launch_bounds__(1024) k_top_moments(NodeArgs A, DevCtl* ctl) {
    __shared__ NodeSums S[1024 / NODE_LANES];
    __shared__ int node[TOP_MAX];
    __shared__ unsigned char level[TOP_MAX];
    __shared__ u32 levels;
    const int j = threadIdx.x & (NODE_LANES - 1);
    const bool listed = A.sub_max > 0;
    const int nb = listed ? min(ctl->n_big, TOP_MAX) : 0;
    if (listed) {
        if (threadIdx.x == 0) levels = 0u;
        __syncthreads();
        for (int k = threadIdx.x; k < nb; k += 1024) {
            const int l = A.list[A.n - 2 - 2 * k];
            node[k] = A.list[A.n - 1 - 2 * k];
            level[k] = (unsigned char)l;
            atomicOr(&levels, 1u << l);
        }
    }
    if (threadIdx.x >= 960) {
        int l = 0;
        while (l < MAX_LEVEL && A.ctl->level_count[l + 1] > 0 && A.ctl->level_count[l + 1] <= WALK_START) {
            const int b0 = A.ctl->level_off[l], nl = A.ctl->level_count[l];  // at most WALK_START nodes
            if (__ballot(lane_id() < nl && A.topo[b0 + min(lane_id(), nl - 1)].w)) break;
            ++l;
        }
        if (threadIdx.x == 960) ctl->walk_level = l;
    }
    if (!listed) {
        for (int l = subtree_cut(A.ctl) - 1; l >= 0; --l) {
            const int b0 = A.ctl->level_off[l], nl = A.ctl->level_count[l];
            for (int k = threadIdx.x / NODE_LANES; k < nl; k += 1024 / NODE_LANES) {
                const int4 tp = A.topo[b0 + k];
                if (!tp.w) internal_node(A, S[threadIdx.x / NODE_LANES], b0 + k, tp, j);
            }
            __syncthreads();
        }
        return;
    }
    __syncthreads();
    for (u32 todo = levels; todo;) {
        const int l = 31 - __clz((int)todo);
        todo &= ~(1u << l);
        for (int k = threadIdx.x / NODE_LANES; k < nb; k += 1024 / NODE_LANES)
            if (level[k] == l) internal_node(A, S[threadIdx.x / NODE_LANES], node[k], A.topo[node[k]], j);
        __syncthreads();
    }
}

static int grid_cap(int n, int bs, int cap) {
    int g = (n + bs - 1) / bs;
    return g < 1 ? 1 : (g > cap ? cap : g);
}

template <typename Move>
static void build_octree(hipStream_t s, const DevPtrs& d, const Dims& dm, const Move& mv) {
    const int n = dm.n;
    if (n <= 0) return;
    const int tb = tree_tile(n), ntiles = (n + tb - 1) / tb;
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(ntiles), dim3(tb), 0, s, mv, d.key_a, n, dm.leaf_size, dm.min_level, d.lcp, d.lvl,
                           d.tree_hist, ntiles, d.gsize, d.gcount);
    };
    auto levels = [&](auto w) {
        if (tb == TB_SMALL) run(k_order_levels<decltype(w)::value, TB_SMALL, Move>);
        else run(k_order_levels<decltype(w)::value, TB_LARGE, Move>);
    };
    switch (dm.leaf_size) {  // the autotuner's leaf sizes (its 48 for the node-node scheme takes the general form)
        case 8: levels(std::integral_constant<int, 8>()); break;
        case 12: levels(std::integral_constant<int, 12>()); break;
        case 16: levels(std::integral_constant<int, 16>()); break;
        case 24: levels(std::integral_constant<int, 24>()); break;
        case 32: levels(std::integral_constant<int, 32>()); break;
        case 64: levels(std::integral_constant<int, 64>()); break;
        default: levels(std::integral_constant<int, 0>()); break;
    }
    // up to 64 tiles every workgroup of the emission adds the counts itself (one load a lane and row):
    // 6.0 us at 4,096 particles against 4.4 + 3.9 us with the scan (196 tiles: 9.7 against 5.6 + 4.1)
    const int scanned = ntiles > 64;
    if (scanned)
        hipLaunchKernelGGL(k_level_scan, dim3(TREE_ROWS), dim3(ntiles <= 1024 ? 256 : 1024), 0, s, d.tree_hist, ntiles);
    auto emit = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(ntiles), dim3(tb), 0, s, n, d.lcp, d.lvl, d.tree_hist, ntiles, scanned, d.node_level,
                           d.node_start, d.node_first, d.leaf_start, d.leaf_node, d.ctl, dm.node_cap);
    };
    if (tb == TB_SMALL) emit(k_emit_nodes<TB_SMALL>);
    else emit(k_emit_nodes<TB_LARGE>);
    const int sub_max = n > SUB_LISTED ? (n + SUB_SHARE - 1) / SUB_SHARE : 0;
    const NodeArgs A{d.ctl, n, sub_max, d.gorder, dm.batched, dm.mass_moments, d.key_a, d.topo, d.parent, d.pos4, d.m,
                     d.nbox_lo, d.nbox_hi, d.mom0, d.mom1, d.mom2, d.range};
    // about 4 n / leaf_size nodes of eight lanes; the kernel loops over any beyond that
    hipLaunchKernelGGL(k_finalize, dim3(grid_cap(4 * (n / dm.leaf_size) + 64, 256 / NODE_LANES, 8192)), dim3(256), 0, s,
                       A, d.node_level, d.node_start, d.node_first, d.lcp, d.leaf_start);
    hipLaunchKernelGGL(k_subtree_moments, dim3(grid_cap(n, 16, 2048)), dim3(SUB_THREADS), 0, s, A);
    hipLaunchKernelGGL(k_top_moments, dim3(1), dim3(1024), 0, s, A, d.ctl);
    // target groups: cells of at most 4 * group_size particles, cut into runs of group_size
    const int gcap = 4 * dm.group_size;
    const int g = grid_cap(dm.node_cap, 256, 2048);
    hipLaunchKernelGGL(k_group_starts, dim3(g), dim3(256), 0, s, d.ctl, gcap, dm.group_size, dm.min_level, d.topo,
                       d.parent, d.range, d.gsize, d.gcount);
    hipLaunchKernelGGL(k_emit_groups, dim3((n + GROUP_TILE - 1) / GROUP_TILE), dim3(GROUP_TILE), 0, s, n, dm.batched,
                       d.ctl, d.gsize, d.gcount, d.key_a, d.seg_root_rank, d.group);
    if (dm.group_gravity || group_order(d, dm)) launch_unit_order(s, d.ctl, d.group, nullptr, 0, d.gorder);
}

void build_input_tree(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* u, int64_t* order_out) {
    build_octree(s, d, dm, InputMove{d, u, order_out});
}
void build_step_tree(hipStream_t s, const DevPtrs& a, const DevPtrs& b, const Dims& dm) {
    build_octree(s, b, dm, StepMove{a});
}

// Export (test path): node keys etc. in breadth-first order.
__global__ void k_tree_export(const DevCtl* __restrict__ ctl, int n, const u64* __restrict__ key,
                              const int4* __restrict__ topo,
                              const int2* __restrict__ range, u64* okey, int32_t* olevel, int32_t* oleaf,
                              int64_t* ostart, int64_t* ocount) {
    const int nn = ctl->n_nodes;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nn; b += gridDim.x * blockDim.x) {
        const int4 t = topo[b];
        int2 r = range[b];
        if (r.x < 0 || r.x >= n) r.x = 0;
        const int l = t.z;
        const u64 body = key[r.x] & 0x7fffffffffffffffull;
        const u64 digits = l == 0 ? 0ull : (body >> (3 * (MAX_LEVEL - l)));
        if (okey) okey[b] = (1ull << (3 * l)) | digits;
        if (olevel) olevel[b] = l;
        if (oleaf) oleaf[b] = t.w;
        if (ostart) ostart[b] = r.x;
        if (ocount) ocount[b] = r.y;
    }
}

void launch_tree_export(hipStream_t s, const DevPtrs& d, const Dims& dm, u64* key, int32_t* level, int32_t* leaf,
                        int64_t* start, int64_t* count) {
    hipLaunchKernelGGL(k_tree_export, dim3(grid_cap(dm.node_cap, 256, 2048)), dim3(256), 0, s, d.ctl, dm.n, d.key_a,
                       d.topo, d.range, key, level, leaf, start, count);
}
