// Neighbour search (Sec. 2.1 of arXiv:2007.03097, last paragraph: the traversal runs for
// a group of particles, prunes with the node bounds and builds one neighbour list per
// particle).
//
// One wavefront per target group (at most group_size consecutive particles of one compact
// octree cell), or two or four where groups are few, in an XCD-aware loop over the groups (one group
// per workgroup at the default grid, which holds a workgroup per expected group).
//  1. Group box and largest h by wave reductions.
//  2. Wide tree walk: up to 64 nodes are tested at once, one per lane, against the group
//     box.  A node survives when the squared gap between the boxes, summed in the same
//     operation order as the pair test, is below (hmax_group + hmax_node)^2; rounding is
//     monotone in every operation, so no true neighbour pair is ever pruned.  Surviving
//     leaves go to a candidate list, surviving internal nodes push their children.  The
//     candidate list is matched (step 3) whenever it fills, so any number of candidates
//     is handled with fixed LDS.
//  3. Each candidate particle is tested against the group box (conservatively, as the
//     nodes are); survivors are staged in an LDS ring and matched 64 at a time with the exact
//     predicate fl(fl(fl(dx dx) + fl(dy dy)) + fl(dz dz)) < fl(t t).  The predicate is screened
//     on the matrix cores (see Screen below): the screen decides every pair outside a proven
//     error margin, the few pairs inside it take the FP64 expression, so the lists are those of
//     the FP64 predicate bit for bit.  The OR of all targets' hits is the tile's part of the
//     group's source union U (sources that are a neighbour of at least one target), appended to
//     U in staging order.  The 64 / group_size lanes of a target then take consecutive source
//     ranges of the tile and write, for each hit, the source's index in U.
// Outputs per group (n_g targets starting at sorted position s):
//   uni[s*cap + i], i < ucnt[group]: particle index of the i-th member of U;
//   nbr[s*cap + k*n_g + t]: slot k of target t, a 16-bit index into U (|U| <= UNION_MAX),
//   ascending in k; the blocks of all groups tile exactly n * cap entries, and consumers
//   reading slot k of consecutive targets read consecutive entries.
// The pair kernels stage U in LDS and read their sources there.
#include "common.h"

constexpr int WALK_STACK = 512;
constexpr int WALK_CAND = 256;

constexpr int TILE_RING = 128;

// Group-level state of the matching step.
struct GroupBox {
    double lo[3], hi[3], hg;
};

// Screen of the exact predicate: the signed margin t^2 - r^2 (t = h_a + h_b) of 32 targets against 32
// sources is a contraction over six terms,
//   t^2 - r^2 = a . 2b + h_a 2h_b + c_a + c_b,   c = h^2 - |x|^2,
// of offsets a, b from the centre of the group's box, and runs on the matrix cores in FP32
// (v_mfma_f32_32x32x2_f32, three per 1,024 pairs: K = 6).  Error of the computed value D: with
// u = 2^-24 and S = (|a| + |b|)^2 + (h_a + h_b)^2, which bounds the sum of the terms' magnitudes, the
// rounded inputs give at most 4u S (offsets and h are formed in FP64 and rounded once, c likewise)
// and six accumulations, taken at 2u each so that any order or truncation is covered, 12u S; FP32
// underflow less than 2^-100.  The margin
//   M = 2^-19 S' + 2^-100,   S' >= S for every pair of the tile,
// is twice that.  It is added to c_a, so that D' = D + M: D' < 0 means t^2 - r^2 < 0 and D' > 2M
// means t^2 - r^2 > 0, each by more than the FP64 expression's own rounding (O(2^-53) S), and a
// D' between is undecided.  S' takes the half diagonal R of the group box, the largest h of the
// group hg and of the tile's sources hm: |a| <= R, and a source that passed the group-box filter
// has |b| <= R + hg + hm.  Lengths are in units of the group's reach 2 R + hg, rounded to a power of two (exact),
// so the screen decides as much in any unit of the input; in the input's own, the FP32 range left lists of
// coordinates above 1e18 or below 1e-13 to the exact predicate (600,000 particles 216 -> 541 us at 1e19).  Where M
// is not below 2^100 (or NaN; sources whose h dwarfs the group, or a reach whose square is hardly
// representable) every pair is undecided; below, nothing overflows.
//
// The former screen ran on the vector ALUs, 12 instructions a pair test, and bound the kernel
// (about 780 of some 1,400 vector instructions per tile of 64 sources and 64 targets); a D'
// costs 1.5 of them here, its sign shifted into the hit mask and its bits into the running
// minimum that finds undecided pairs.  Lists of the 987,840 tube 357 -> 288 us, of 123K particles 114 ->
// 79 us, of 1.2M in 64 boxes 443 -> 363 us; with the slot loop below in eight 32-bit instructions an
// entry (no range checks inside, one 32-bit offset from the group's block) 250, 66 and 317 us.  What
// bounds it now is vector instruction issue (73% of the quad-cycles before that change), spread over
// the walk, the candidates' filter, the masks and the slots; the matrix pipe is busy 14% of the time.
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int TILE_COMP = 5;  // staged per source: 2 b (three), 2 h, c
template <int W>
struct Tile {
    static constexpr int RING = TILE_RING * W;
    float v[TILE_COMP][RING];
    int src[RING];
};

// What W wavefronts that match a tile each tell one another.
template <int W>
struct Exchange {
    int pass[W];      // candidates that passed the box filter
    int uni[W];       // union members of the wavefront's tile
    int hits[W][64];  // hits of a target in it
    int walked[3];    // candidates listed, nodes left on the stack, overflow
};

struct Screen {
    double k;      // power of two near 1 / (2 R + hg): the unit of all below
    double o[3];   // centre of the group's box
    float reach;   // 2 R + hg, rounded up
    float hg;      // rounded up
};

__device__ __forceinline__ float next_up(double v) { return (float)(v * (1.0 + 0x1p-20)); }

// Stages source b at ring slot r.
template <int W>
__device__ __forceinline__ void stage_source(Tile<W>& tile, int r, const double4& b, int src, const Screen& S) {
    const double x = fma(b.x, S.k, -S.o[0]), y = fma(b.y, S.k, -S.o[1]), z = fma(b.z, S.k, -S.o[2]), h = b.w * S.k;
    tile.v[0][r] = 2.0f * (float)x;
    tile.v[1][r] = 2.0f * (float)y;
    tile.v[2][r] = 2.0f * (float)z;
    tile.v[3][r] = 2.0f * (float)h;
    tile.v[4][r] = (float)(h * h - ((x * x + y * y) + z * z));
    tile.src[r] = src;
}

// Targets of a group of at most T.  Matrix columns: the lane's column of block k is target
// 32 k + lane % 32, of which it supplies the terms 2q + lane / 32 (q = 0 .. 2).  Lists: the lane writes
// for target lane % T, with the P = 64 / T lanes of a target splitting the tile's sources.
template <int T>
struct LaneTargets {
    static constexpr int P = 64 / T, NC = T == 64 ? 2 : 1;
    float b0[NC], b1[NC], b2[NC];
    int t, p, cnt;
};

template <int T>
__device__ __forceinline__ void load_targets(LaneTargets<T>& L, const double4* __restrict__ pos4, int gx, int gy,
                                             const Screen& S) {
    const int lane = lane_id();
    const bool odd = lane >= 32;
#pragma unroll
    for (int k = 0; k < L.NC; ++k) {
        const int col = 32 * k + (lane & 31);
        const double4 A = pos4[gx + (col < gy ? col : 0)];  // columns past the group repeat its first target
        const double x = fma(A.x, S.k, -S.o[0]), y = fma(A.y, S.k, -S.o[1]), z = fma(A.z, S.k, -S.o[2]), h = A.w * S.k;
        L.b0[k] = odd ? (float)y : (float)x;
        L.b1[k] = odd ? (float)h : (float)z;
        L.b2[k] = odd ? (float)(h * h - ((x * x + y * y) + z * z)) : 1.0f;
    }
}

// The exact predicate for undecided elements of a 32 x 32 block (bit i of und = element i, matrix row
// (i & 3) + 8 (i >> 2) + 4 half); rows from `rows` on are stale.
template <int W>
__device__ u32 resolve_exact(u32 und, u32 hits, const double4 A, int half, int rows, int slot0, const Tile<W>& tile,
                             const double4* __restrict__ pos4) {
    while (und) {
        const int i = __ffs(und) - 1;
        und &= und - 1;
        const int m = (i & 3) + 8 * (i >> 2) + 4 * half;
        if (m >= rows) continue;
        const double4 s = pos4[tile.src[(slot0 + m) & (Tile<W>::RING - 1)]];
        const double dx = A.x - s.x, dy = A.y - s.y, dz = A.z - s.z;
        double r2 = dx * dx + dy * dy;
        r2 = r2 + dz * dz;
        const double tt = A.w + s.w;
        hits = r2 < tt * tt ? hits | (1u << i) : hits & ~(1u << i);
    }
    return hits;
}

// Matches the n sources (1 .. 64 W) at ring positions first .. against the group's targets, 64 per
// wavefront: hits go to the group's union and to the targets' lists, in the order of the sources.
template <int T, int W>
__device__ __forceinline__ void test_tile(int first, int n, const Tile<W>& tile, LaneTargets<T>& L, const Screen& S,
                                          const double4* __restrict__ pos4, int gx, int gy, int cap, u16* mylist,
                                          int* myuni, int ulim, int& ucnt, Exchange<W>& X) {
    const int lane = lane_id(), col = lane & 31, half = lane >> 5, wave = W > 1 ? threadIdx.x >> 6 : 0;
    const int head = first + 64 * wave, tn = W > 1 ? min(n - 64 * wave, 64) : n;  // (none left: no hits)
    // largest |h| of the tile: non-negative floats order as unsigned integers, a NaN above them
    const u32 hv = lane < tn ? __float_as_uint(fabsf(tile.v[3][(head + lane) & (Tile<W>::RING - 1)])) : 0u;
    const float hm = 0.5f * __uint_as_float(wave_reduce_u32(hv, [](u32 a, u32 b) { return max(a, b); }));
    const float R = S.reach + hm, tt = S.hg + hm;
    const float M = fmaf(fmaf(R, R, tt * tt), 0x1p-19f * (1.0f + 0x1p-18f), 0x1p-100f);
    const bool all = !(M < 0x1p100f);
    const u32 lim = __float_as_uint(2.0f * M * (1.0f + 0x1p-18f));
    // matrix rows: the terms 2q + half of source 32 r + lane % 32 (head is a multiple of 64)
    float a0[2], a1[2], a2[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int j = (head + 32 * r + col) & (Tile<W>::RING - 1);
        a0[r] = tile.v[half][j];
        a1[r] = tile.v[2 + half][j];
        a2[r] = half ? 1.0f : tile.v[4][j];
    }
    u32 w[LaneTargets<T>::NC][2];  // the column's hits, source 32 r + bit (the same in both halves)
#pragma unroll
    for (int k = 0; k < LaneTargets<T>::NC; ++k) {
        w[k][0] = w[k][1] = 0u;
        if (32 * k >= gy) continue;
        const bool exists = 32 * k + col < gy;
        const float b2 = L.b2[k] + (half ? M : 0.0f);
        f32x16 D[2] = {};
        D[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[0], L.b0[k], D[0], 0, 0, 0);
        D[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[1], L.b0[k], D[1], 0, 0, 0);
        D[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[0], L.b1[k], D[0], 0, 0, 0);
        D[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[1], L.b1[k], D[1], 0, 0, 0);
        D[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a2[0], b2, D[0], 0, 0, 0);
        D[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a2[1], b2, D[1], 0, 0, 0);
        u32 hits[2], low = 0xffffffffu;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            u32 miss = 0u;
#pragma unroll
            for (int i = 15; i >= 0; --i) {
                const u32 v = __float_as_uint(D[r][i]);
                miss = __builtin_amdgcn_alignbit(miss, v, 31);  // miss << 1 | sign
                low = min(low, v);                              // negative values lie above all others
            }
            hits[r] = ~miss & 0xffffu;
        }
        if (__ballot(low <= lim) || all) {  // rare: undecided pairs take the FP64 expression
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                u32 und = 0u;
#pragma unroll
                for (int i = 15; i >= 0; --i) und = und + und + (__float_as_uint(D[r][i]) <= lim || all ? 1u : 0u);
                if (exists && und)
                    hits[r] = resolve_exact(und, hits[r], pos4[gx + 32 * k + col], half, tn - 32 * r, head + 32 * r,
                                            tile, pos4);
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            // nibble n of the half's hits holds rows 8 n + 4 half ..; both halves' rows together
            u32 h = hits[r];
            h = (h | (h << 8)) & 0x00ff00ffu;
            h = (h | (h << 4)) & 0x0f0f0f0fu;
            const auto both = __builtin_amdgcn_permlane32_swap(h << (4 * half), h << (4 * half), false, false);
            const int rows = tn - 32 * r;
            const u32 valid = rows >= 32 ? 0xffffffffu : (rows > 0 ? (1u << rows) - 1u : 0u);
            w[k][r] = exists ? (both[0] | both[1]) & valid : 0u;
        }
    }
    u32 w0 = w[0][0], w1 = w[0][1];  // hits of the lane's list target
    if constexpr (T == 64) {
        w0 = half ? w[1][0] : w0;
        w1 = half ? w[1][1] : w1;
    } else if constexpr (T < 32) {
        w0 = (u32)__shfl((int)w0, L.t, 64);
        w1 = (u32)__shfl((int)w1, L.t, 64);
    }
    auto either = [](u32 a, u32 b) { return a | b; };
    const u32 u0 = wave_reduce_u32(w0, either), u1 = wave_reduce_u32(w1, either);  // union of the tile
    const u64 ub = (u64)u0 | ((u64)u1 << 32);
    int ufirst = ucnt, slot = L.cnt;  // after those of the wavefronts before this one
    if constexpr (W > 1) {
        if (L.p == 0) X.hits[wave][L.t] = (int)(__popc(w0) + __popc(w1));
        if (lane == 0) X.uni[wave] = (int)__popcll(ub);
        __syncthreads();
#pragma unroll
        for (int v = 0; v < W; ++v) {
            const int h = X.hits[v][L.t], u = X.uni[v];
            L.cnt += h;
            ucnt += u;
            if (v < wave) {
                slot += h;
                ufirst += u;
            }
        }
    } else {
        L.cnt += (int)(__popc(w0) + __popc(w1));
        ucnt += (int)__popcll(ub);
    }
    if ((ub >> lane) & 1ull) {
        const int r = ufirst + __popcll(ub & lanemask_lt());
        if (r < ulim) myuni[r] = tile.src[(head + lane) & (Tile<W>::RING - 1)];
    }
    // the lane's share of its target's hits: sources p T .. p T + T - 1, after those before them
    u32 m0 = w0, m1 = w1;
    if constexpr (T < 64) {
        const int j0 = L.p * T;
        const u32 below = (1u << (j0 & 31)) - 1u, range = T == 32 ? 0xffffffffu : ((1u << (T & 31)) - 1u) << (j0 & 31);
        if (j0 < 32) {
            slot += __popc(w0 & below);
            m0 &= range;
            m1 = 0u;
        } else {
            slot += __popc(w0) + __popc(w1 & below);
            m0 = 0u;
            m1 &= range;
        }
    }
    const int end = slot + (int)__popc(m0) + (int)__popc(m1);
    if (__ballot(end > cap)) {  // an overflow the kernel reports: only the slots below cap are written
        while (slot + (int)__popc(m0) + (int)__popc(m1) > cap && (m0 | m1)) {
            if (m1) m1 &= ~(1u << (31 - __clz((int)m1)));
            else m0 &= ~(1u << (31 - __clz((int)m0)));
        }
    }
    // entries past UNION_MAX (likewise reported) stay at the last index, in bounds
    const u32 last = UNION_MAX - 1, stride = 2u * (u32)gy;
    u32 at = 2u * ((u32)slot * (u32)gy + (u32)L.t);  // byte offset in the group's block, below 2 x 64 x 4,096
    auto append = [&](u32 bits, u32 uw, u32 first) {
        while (bits) {
            const u32 before = __builtin_amdgcn_ubfe(uw, 0u, (u32)__builtin_ctz(bits));
            bits &= bits - 1;
            const u32 e = first + __popc(before);
            *reinterpret_cast<u16*>(reinterpret_cast<char*>(mylist) + at) = (u16)(e < last ? e : last);
            at += stride;
        }
    };
    append(m0, u0, (u32)ufirst);
    append(m1, u1, (u32)ufirst + __popc(u0));
}

// Matching of the group's targets against the particles of the nc candidate leaves, whose first
// particles are in cand[] and particle counts in coff[] (which become offsets).  Each candidate
// particle is first tested against the group box, in the same monotone operation order as the node
// test (gap^2 < (hmax_group + h_b)^2), so no true neighbour is dropped; survivors enter an
// LDS ring and are matched 64 at a time.  Sources left in the ring (< 64) are matched by
// the caller's final flush.  The next 64 candidates are loaded before a tile is matched.
template <int T, int W>
__device__ void match_candidates(int nc, int* cand, int* coff, Tile<W>& tile, int& head, int& tail, const GroupBox& gb,
                                 const Screen& S, const double4* __restrict__ pos4, LaneTargets<T>& L, int gx, int gy,
                                 int cap, u16* mylist, int* myuni, int ulim, int& ucnt, Exchange<W>& X) {
    const int lane = lane_id(), wave = W > 1 ? threadIdx.x >> 6 : 0;
    const u64 lt = lanemask_lt();
    int total = 0;
    if (W == 1 || wave == 0) {
        for (int j0 = 0; j0 < nc; j0 += 64) {
            const int j = j0 + lane;
            const int c = j < nc ? coff[j] : 0;
            const int incl = wave_incl_scan(c);
            if (j < nc) coff[j] = total + incl - c;
            total += wave_last(incl);
        }
        if (W > 1 && lane == 0) coff[nc] = total;
    }
    unit_sync<W>();
    if (W > 1) total = coff[nc];
    int last = -1, src = 0;
    double4 b;
    auto fetch = [&](int p0) {
        int a = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int own = tile_owner(coff, nc, p0 + 64 * w, last);
            if (w == wave) a = own;
        }
        const int p = p0 + 64 * wave + lane;
        if (p < total) {
            src = cand[a] + (p - coff[a]);
            b = pos4[src];
        }
    };
    if (total > 0) fetch(0);
    for (int p0 = 0; p0 < total; p0 += 64 * W) {
        bool pass = false;
        if (p0 + 64 * wave + lane < total) {
            const double gx = fmax(0.0, fmax(b.x - gb.hi[0], gb.lo[0] - b.x));
            const double gy2 = fmax(0.0, fmax(b.y - gb.hi[1], gb.lo[1] - b.y));
            const double gz = fmax(0.0, fmax(b.z - gb.hi[2], gb.lo[2] - b.z));
            double r2 = gx * gx + gy2 * gy2;
            r2 = r2 + gz * gz;
            const double tt = gb.hg + b.w;
            pass = r2 < tt * tt;
        }
        const u64 bal = __ballot(pass);
        int at = tail;
        if constexpr (W > 1) {
            if (lane == 0) X.pass[wave] = (int)__popcll(bal);
            __syncthreads();
#pragma unroll
            for (int v = 0; v < W; ++v) {
                const int c = X.pass[v];
                if (v < wave) at += c;
                tail += c;
            }
        } else {
            tail += __popcll(bal);
        }
        if (pass) stage_source(tile, (at + __popcll(bal & lt)) & (Tile<W>::RING - 1), b, src, S);
        unit_sync<W>();
        if (p0 + 64 * W < total) fetch(p0 + 64 * W);
        if (tail - head >= 64 * W) {
            test_tile(head, 64 * W, tile, L, S, pos4, gx, gy, cap, mylist, myuni, ulim, ucnt, X);
            head += 64 * W;
        }
        unit_sync<W>();
    }
}

// W wavefronts per group: the first one walks the tree, all of them match the candidates, a tile each.
template <int T, int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W == 1 ? 5 : 1))) k_nbr_lists(
    DevCtl* ctl, const int* __restrict__ order, const int4* __restrict__ group, int cap, const int4* __restrict__ topo,
    const double4* __restrict__ nbox_lo, const double4* __restrict__ nbox_hi, const double4* __restrict__ pos4,
    u16* __restrict__ nbr, int* __restrict__ nbr_cnt, int* __restrict__ list_base, int* __restrict__ uni,
    int* __restrict__ ucnt_out) {
    __shared__ int stack[WALK_STACK];
    __shared__ int cand[WALK_CAND];
    __shared__ int coff[WALK_CAND + 1];
    __shared__ Tile<W> tile;
    __shared__ Exchange<W> X;
    const int lane = lane_id(), wave = W > 1 ? threadIdx.x >> 6 : 0;
    const u64 lt = lanemask_lt();
    LaneTargets<T> L;
    L.t = lane % T;
    L.p = lane / T;
    int g0, g1, gstep;
    group_range(ctl->n_groups, g0, g1, gstep);
    for (int ui = g0; ui < g1; ui += gstep) {
        const int gi = order ? order[ui] : ui;
        const int4 g = group[gi];
        GroupBox gb;
        {
            const double4 A = pos4[g.x + (L.t < g.y ? L.t : 0)];  // lanes past the group repeat its first target
            gb.lo[0] = wave_min(A.x);
            gb.lo[1] = wave_min(A.y);
            gb.lo[2] = wave_min(A.z);
            gb.hi[0] = wave_max(A.x);
            gb.hi[1] = wave_max(A.y);
            gb.hi[2] = wave_max(A.z);
            gb.hg = wave_max(A.w);
        }
        Screen S;
        {
            double d2 = 0.0;
            for (int c = 0; c < 3; ++c) {
                S.o[c] = 0.5 * (gb.lo[c] + gb.hi[c]);
                const double e = fmax(gb.hi[c] - S.o[c], S.o[c] - gb.lo[c]);
                d2 += e * e;
            }
            const double reach = 2.0 * sqrt(d2) + gb.hg;
            S.k = inv_pow2(reach);
            for (int c = 0; c < 3; ++c) S.o[c] *= S.k;
            // squares in range: near its ends the FP64 predicate rounds to 0 or overflows, and every pair takes it
            S.reach = reach > 0x1p-400 && reach < 0x1p400 ? next_up(reach * S.k) : INFINITY;
            S.hg = next_up(gb.hg * S.k);
        }
        load_targets(L, pos4, g.x, g.y, S);
        L.cnt = 0;
        const double* lo = gb.lo;
        const double* hi = gb.hi;
        const double hg = gb.hg;
        u16* mylist = nbr + (size_t)g.x * (size_t)cap;
        int* myuni = uni + (size_t)g.x * (size_t)cap;
        const int ulim = min(g.y * cap, UNION_MAX);
        int ucnt = 0, head = 0, tail = 0;
        // a segment's walk starts at its root, a single set's at the nodes of walk_level (those
        // above it would all be opened, or their whole subtrees pruned)
        const bool single = g.z < 0;
        const int wl = ctl->walk_level;
        const int first = single ? ctl->level_off[wl] : ctl->level_off[3] + g.z;
        int sp = single ? ctl->level_count[wl] : 1, iters = 0;
        bool overflow = false;
        unit_sync<W>();
        if ((int)threadIdx.x < sp && (W == 1 || wave == 0)) stack[lane] = first + lane;
        wave_lds_fence();
        while (true) {
            int nc = 0;
            // until the list may not hold another round or the walk has ended
            while ((W == 1 || wave == 0) && sp > 0 && nc + 64 <= WALK_CAND) {
                if (++iters > (1 << 20)) {  // bounded: every wave leaves the loop
                    overflow = true;
                    break;
                }
                // pop at most as many nodes as the free stack can take the children of (8 each)
                int k = sp < 64 ? sp : 64;
                const int room = (WALK_STACK - sp) / 8;
                if (k > room) k = room > 1 ? room : 1;
                const int node = lane < k ? stack[sp - k + lane] : -1;
                wave_lds_fence();
                sp -= k;
                bool hit = false;
                int4 tp = make_int4(0, 0, 0, 0);
                if (node >= 0) {
                    tp = topo[node];
                    const double4 a = nbox_lo[node], b = nbox_hi[node];
                    const double gx = fmax(0.0, fmax(a.x - hi[0], lo[0] - b.x));
                    const double gy = fmax(0.0, fmax(a.y - hi[1], lo[1] - b.y));
                    const double gz = fmax(0.0, fmax(a.z - hi[2], lo[2] - b.z));
                    double r2 = gx * gx + gy * gy;
                    r2 = r2 + gz * gz;
                    const double tt = hg + a.w;
                    hit = r2 < tt * tt;
                }
                const bool isleaf = hit && tp.w;
                const u64 bl = __ballot(isleaf);
                if (isleaf) {
                    cand[nc + __popcll(bl & lt)] = tp.x;
                    coff[nc + __popcll(bl & lt)] = tp.y;
                }
                nc += __popcll(bl);
                const int nch = (hit && !tp.w) ? tp.y : 0;
                const int incl = wave_incl_scan(nch);
                const int tot = wave_last(incl);
                if (sp + tot > WALK_STACK) {
                    overflow = true;
                    break;
                }
                for (int j = 0; j < nch; ++j) stack[sp + incl - nch + j] = tp.x + j;
                sp += tot;
                wave_lds_fence();
            }
            if (W > 1) {
                if (threadIdx.x == 0) {
                    X.walked[0] = nc;
                    X.walked[1] = sp;
                    X.walked[2] = overflow;
                }
                __syncthreads();
                nc = X.walked[0];
                sp = X.walked[1];
                overflow = X.walked[2];
            }
            if (overflow) break;
            unit_sync<W>();
            match_candidates(nc, cand, coff, tile, head, tail, gb, S, pos4, L, g.x, g.y, cap, mylist, myuni, ulim,
                             ucnt, X);
            unit_sync<W>();
            if (sp <= 0) break;
        }
        if (!overflow) {
            if (tail > head)
                test_tile(head, tail - head, tile, L, S, pos4, g.x, g.y, cap, mylist, myuni, ulim, ucnt, X);
            unit_sync<W>();
        } else if (threadIdx.x == 0)
            set_err(ctl, ERR_WALK_STACK);
        if (threadIdx.x == 0) {
            ucnt_out[gi] = overflow ? 0 : (ucnt < ulim ? ucnt : ulim);
            if (ucnt > UNION_MAX) set_err(ctl, ERR_UNION_CAP);
        }
        if (L.p == 0 && L.t < g.y && (W == 1 || wave == 0)) {
            const int q = g.x + L.t;
            nbr_cnt[q] = overflow ? 0 : (L.cnt < cap ? L.cnt : cap);
            list_base[q] = overflow ? -1 : gi;
            if (L.cnt > cap) {
                set_err(ctl, ERR_NBR_CAP);
                atomicMax(&ctl->nbr_max, L.cnt);
            }
        }
    }
}

void launch_nbr_lists(hipStream_t s, const DevPtrs& d, const Dims& dm) {
    if (dm.n <= 0) return;
    auto go = [&](auto kern, int waves) {
        const int grid = std::min(dm.group_grid, 8 * std::max(1, dm.wave_cap / (8 * waves)));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * waves), 0, s, d.ctl, group_order(d, dm), d.group, dm.nbr_cap,
                           d.topo, d.nbox_lo, d.nbox_hi, d.pos4, d.nbr, d.nbr_cnt, d.nbr_base, d.uni, d.ucnt);
    };
    // Wavefronts a group: with few groups a wavefront's own latencies (25 us at 4,096 particles) are the
    // kernel's time, and the matching, though not the walk, is shared.  Lists alone, us, for 1 / 2 / 4: 4,096
    // particles in groups of 32 25.9 / 20.7 / 19.0; 50,021 in groups of 32 47 / 43 / 55; 123,480 in groups of
    // 64 65 / 69 / 78; with build, density and forces 20,011 in groups of 64 178 / 168 / 163, 100,003 in groups
    // of 64 266 / 256 / 268, 50,021 in groups of 16 240 / 258 / 276.
    const int64_t units = dm.n / std::max(1, dm.group_size);
    // Sets of up to 64 particles are one tile, which one wavefront matches (512 sets of 8: 8.0 -> 6.8 us).
    const int W = units > 1600 || tiny_sets(dm) ? 1 : (units > 512 ? 2 : 4);
    auto size = [&](auto t) {
        constexpr int T = decltype(t)::value;
        if (W == 4) go(k_nbr_lists<T, 4>, 4);
        else if (W == 2) go(k_nbr_lists<T, 2>, 2);
        else go(k_nbr_lists<T, 1>, 1);
    };
    switch (dm.group_size) {  // validated at context creation: 8, 16, 32 or 64
        case 8: size(std::integral_constant<int, 8>()); break;
        case 16: size(std::integral_constant<int, 16>()); break;
        case 32: size(std::integral_constant<int, 32>()); break;
        default: size(std::integral_constant<int, 64>()); break;
    }
}

// ---- CSR export in caller order (test and inspection path)
__global__ void k_csr_count(int n, const u32* __restrict__ id, const int* __restrict__ cnt, int64_t* counts) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) counts[id[q]] = cnt[q];
}

void launch_csr_count(hipStream_t s, const DevPtrs& d, const Dims& dm, int64_t* counts_caller) {
    if (dm.n > 0) hipLaunchKernelGGL(k_csr_count, dim3((dm.n + 255) / 256), dim3(256), 0, s, dm.n, d.id, d.nbr_cnt,
                                     counts_caller);
}

// One workgroup per group, one wave per target, or 16 or 8 lanes where no list of the group is longer (200,003
// particles of one neighbour in groups of 64, whole query: 96 -> 77 us).  The targets' neighbour IDs are distinct, so an
// entry's place in its list is the number of smaller IDs in it: each lane holds one entry and
// counts them against the others broadcast from their lanes, without LDS sorts or divergence.
// The former one-thread insertion sort in global memory was bound by its chains of dependent
// loads and stores: 1,070 us for 200,003 particles of 38 neighbours, now 84 us (30 MB of lists: 0.4 TB/s; the
// counting bounds it).
template <int CSR_THREADS>
__global__ void __launch_bounds__(CSR_THREADS) k_csr_fill(const DevCtl* __restrict__ ctl, int cap,
                                                          const int4* __restrict__ group, const u32* __restrict__ id,
                                                          const int* __restrict__ cnt, const int* __restrict__ gidx,
                                                          const u16* __restrict__ nbr, const int* __restrict__ uni,
                                                          const int* __restrict__ ucnt,
                                                          const int64_t* __restrict__ off, int32_t* __restrict__ idx) {
    constexpr int CSR_UNION = 16 * CSR_THREADS;  // union IDs staged in LDS; larger unions read them from memory
    __shared__ int uid[CSR_UNION];
    __shared__ int64_t toff[64];  // per target: its place in idx and its count
    __shared__ int tcnt[64], longest;
    const int lane = lane_id(), w = threadIdx.x >> 6;
    int g0, g1, gstep;
    group_range(ctl->n_groups, g0, g1, gstep);
    for (int gi = g0; gi < g1; gi += gstep) {
        const int4 g = group[gi];
        const int* un = uni + (size_t)g.x * cap;
        const int nu = ucnt[gi];
        const bool staged = nu <= CSR_UNION;
        __syncthreads();
        if (staged)
            for (int i = threadIdx.x; i < nu; i += CSR_THREADS) uid[i] = (int)id[un[i]];
        if (threadIdx.x < 64) {  // at most 64 targets
            int c = 0;
            if (threadIdx.x < g.y) {
                const int q = g.x + threadIdx.x;
                toff[threadIdx.x] = off[id[q]];
                tcnt[threadIdx.x] = c = gidx[q] < 0 ? 0 : cnt[q];
            }
            c = (int)wave_reduce_u32((u32)c, [](u32 a, u32 b) { return max(a, b); });
            if (threadIdx.x == 0) longest = c;
        }
        __syncthreads();
        auto few = [&](auto width) {  // width lanes a target, an entry each
            constexpr int N = decltype(width)::value;
            const int k = threadIdx.x % N;
            for (int t = threadIdx.x / N; t < g.y; t += CSR_THREADS / N) {
                const int c = tcnt[t];
                int v = 0x7fffffff;
                if (k < c) {
                    const int u = nbr[(size_t)g.x * cap + t + k * g.y];
                    v = staged ? uid[u] : (int)id[un[u]];
                }
                int rank = 0;
#pragma unroll
                for (int j = 0; j < N; ++j) rank += __shfl(v, j, N) < v ? 1 : 0;
                if (k < c) idx[toff[t] + rank] = v;
            }
        };
        const int most = longest;
        if (most <= 16) {
            if (most <= 8) few(std::integral_constant<int, 8>());
            else few(std::integral_constant<int, 16>());
            continue;
        }
        for (int t = w; t < g.y; t += CSR_THREADS / 64) {
            const int c = __builtin_amdgcn_readfirstlane(tcnt[t]);
            const u16* lst = nbr + (size_t)g.x * cap + t;
            int32_t* out = idx + toff[t];
            auto entry = [&](int k) -> int {  // caller index of list slot k; above all of them past the end
                if (k >= c) return 0x7fffffff;
                const int u = lst[k * g.y];
                return staged ? uid[u] : (int)id[un[u]];
            };
            for (int i0 = 0; i0 < c; i0 += 64) {
                const int v = entry(i0 + lane);
                int rank = 0;
                for (int j0 = 0; j0 < c; j0 += 64) {
                    const int o = j0 == i0 ? v : entry(j0 + lane);
                    const int jn = min(64, c - j0);
                    for (int j = 0; j < jn; j += 8) {  // entries past the end are above every other
#pragma unroll
                        for (int k = 0; k < 8; ++k) rank += __builtin_amdgcn_readlane(o, j + k) < v ? 1 : 0;
                    }
                }
                if (i0 + lane < c) out[rank] = v;
            }
        }
    }
}

void launch_csr_fill(hipStream_t s, const DevPtrs& d, const Dims& dm, const int64_t* offsets, int32_t* idx,
                     int64_t total) {
    if (dm.n <= 0) return;
    auto go = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(dm.pair_grid), dim3(threads), 0, s, d.ctl, dm.nbr_cap, d.group, d.id, d.nbr_cnt,
                           d.nbr_base, d.nbr, d.uni, d.ucnt, offsets, idx);
    };
    // Many small groups of short lists: a wavefront each.  200,003 particles of a lattice, whole query, us, 256 / 64
    // threads: one neighbour each, groups of 8 100 / 81, of 16 84 / 76; 58 neighbours, of 8 214 / 204, of 16
    // 198 / 212; 60,000 of 58, of 8 112 / 123.
    if (dm.group_size <= 16 && dm.n / dm.group_size > 4096 && total <= 24 * (int64_t)dm.n) go(k_csr_fill<64>, 64);
    else go(k_csr_fill<256>, 256);
}
