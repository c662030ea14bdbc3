// Internal header of the gfx950 SPH + octree library: device helpers, the device-side
// workspace layout and the kernel launchers shared between translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned long long u64;
typedef unsigned int u32;
typedef unsigned short u16;

// ---------------------------------------------------------------------------------------
// Sticky device error bits (read back by sph_sync / synchronous calls).
enum : u32 {
    ERR_NONFINITE = 1u,      // non-finite position, velocity or energy
    ERR_NONPOSITIVE = 2u,    // h <= 0 or m <= 0
    ERR_NBR_CAP = 4u,        // a particle has more neighbours than nbr_capacity
    ERR_WALK_STACK = 8u,     // tree-walk stack or candidate list overflow
    ERR_NODE_CAP = 16u,      // octree node capacity exceeded
    ERR_GRAV_LIST = 32u,     // gravity walk stack overflow
    ERR_UNION_CAP = 64u,     // a walk group's source union exceeds UNION_MAX particles
};

// List entries are 16-bit indices into their group's source union, so a union holds at most
// this many particles (unions of a few thousand are typical).
constexpr int UNION_MAX = 65536;

constexpr int MAX_LEVEL = 21;   // 21 three-bit digits below the sentinel bit 63
constexpr double M_1_PI_D = 0.318309886183790671537767526745028724;
constexpr double M_1_PI_LO = -1.9678676675182486e-17;  // 1/pi - M_1_PI_D (6e-17 of it)

// Accumulators of a single set's bounding box in k_bbox: workgroups spread their atomics over
// them, and k_set_box merges them (a segmented set has one per segment).
constexpr int BOX_SLOTS = 64;

// Nodes of the starting level of the neighbour walks: as many as one round of a walk pops (it keeps
// room for eight children of each on its 512-entry stack), so that starting there visits the same
// nodes in the same order as starting at the root.
constexpr int WALK_START = 56;

// Counter slots of the gravity pass's term counts, one 128-byte line each.
constexpr int GRAV_SLOTS = 64;

// Control block living in device memory.
struct DevCtl {
    // read back in one copy at the end of a call (CtlHead)
    u32 err;
    int nbr_max;                  // largest neighbour count seen (for overflow reports)
    double diag[16];              // step diagnostics
    int n_nodes;
    int n_leaves;
    int n_groups;                 // target groups
    int level_count[24];          // nodes per level
    int level_off[24];            // exclusive prefix of level_count
    int walk_level;               // level at which a single set's neighbour walks start (k_top_moments)
    int n_sub, n_big;             // subtrees handed out whole, nodes above them (k_finalize)
    int fmm_heavy[8];             // leaves of an XCD's share that a whole workgroup takes (node-node gravity)
    u64 box_enc[512 * 6];         // per segment: ordered-integer min x,y,z then max x,y,z
    double box[512 * 6];          // decoded per-segment box lo.xyz, hi.xyz
    double scale[512];            // 2^B / L per segment (0 when L == 0)
    double side[512];             // L (root cell side) per segment
    double seg_dt[512];           // step size of each segment (read by the kick kernels)
    u64 dtb_enc[512];             // per segment: ordered-integer min of the time-step bound
    // last quadrupole gravity pass: particle-cell terms ([s][0]) and particle-particle terms
    // ([s][1], each target's own pair included) evaluated, summed over the slots s; a group
    // adds its counts to slot (group % GRAV_SLOTS), so the atomics spread over 64 lines
    u64 grav_cnt[GRAV_SLOTS][16];
    int skip_phi;                 // nonzero: the gravity passes leave phi unevaluated
};

// The part of DevCtl that the host reads back, a prefix of it.
struct CtlHead {
    u32 err;
    int nbr_max;
    double diag[10];
};
static_assert(offsetof(DevCtl, err) == offsetof(CtlHead, err) && offsetof(DevCtl, nbr_max) == offsetof(CtlHead, nbr_max) &&
                  offsetof(DevCtl, diag) == offsetof(CtlHead, diag),
              "CtlHead is a prefix of DevCtl");

// Device pointers of one context.  All arrays are carved out of the caller's workspace.
struct DevPtrs {
    DevCtl* ctl;
    // sort
    u64 *key_a, *key_b;           // n_cap: sorted keys; keys to sort (and scratch of the sort)
    u32 *val_a, *val_b;           // n_cap
    void* scan_tmp;               // 8 * scan_blocks_cap (u64)
    // Morton-ordered particle data (SoA FP64)
    double *x, *y, *z, *vx, *vy, *vz, *m, *h, *u;
    double *vpx, *vpy, *vpz, *up;  // predictors (step)
    double *ax, *ay, *az, *du;
    double *rho, *P, *cs, *hnext;
    double *gx, *gy, *gz, *phi;
    // second copies used while reordering between steps
    double *x2, *y2, *z2, *vx2, *vy2, *vz2, *m2, *h2, *u2, *vpx2, *vpy2, *vpz2, *up2;
    u32* id;                      // caller index of each Morton position
    u32* id2;
    double4* rec;                 // 2 n_cap, over the second copies: caller-order records of a build
    double4* pos4;                // x, y, z, h (Morton order)
    double4* vel4;                // vx(pred), vy, vz, m
    double4* thr4;                // rho, P/rho^2, c, u
    float4* thrf;                 // FP32 copy for the compensated path: rho, P/rho^2, c, h
    // tree
    signed char* lcp;             // n_cap + 1: shared leading digits with the previous key
    unsigned char* lvl;           // n_cap: leaf level of each sorted position
    int* tree_hist;               // tree_hist_words(n_cap): per-level node counts of the position tiles
    int* leaf_start;              // n_cap + 1 (sorted position of each leaf, then n)
    int* leaf_node;               // n_cap: breadth-first node of each leaf
    unsigned char* node_level;    // node_cap (breadth-first, as all node arrays)
    int* node_start;              // node_cap: first sorted position
    int* node_first;              // node_cap: first child, or ~(number among the leaves)
    int4* topo;                   // node_cap: {first, count, level, is_leaf}
    int* parent;                  // node_cap
    int2* range;                  // node_cap: {start, count} in sorted order
    double4* nbox_lo;             // node_cap: lo.xyz, hmax
    double4* nbox_hi;             // node_cap: hi.xyz, cell side
    double4* mom0;                // node_cap: M, com.xyz
    double4* mom1;                // node_cap: Ixx, Iyy, Izz, tr I
    double4* mom2;                // node_cap: Ixy, Ixz, Iyz, cell (bits; node-node gravity only)
    // groups and neighbour lists
    int4* group;                  // group_cap: {start, count, segment root rank (-1 = root), 0}
    u32* gsize;                   // n_cap: size of the target group starting at a position, else 0; after the groups'
                                  // emission the order of the leaves in node-node gravity (k_unit_order)
    int* gorder;                  // n_cap: order in which the group kernels take the groups (k_unit_order); in the
                                  // build the roots of the subtrees handed out whole and, from its end, the nodes above
    int* gcount;                  // group_hist_words(n_cap): groups starting in each tile of positions
    u16* nbr;                     // n_cap * nbr_cap: list slots, indices into the group's union
    int* nbr_cnt;                 // n_cap
    int* nbr_base;                // n_cap: group whose lists hold the particle (-1 = none)
    int* uni;                     // n_cap * nbr_cap: per group, particles of its source union
    int* ucnt;                    // group_cap: size of each group's union
    // seg / chunk tables
    int4* chunk;                  // chunk_cap: {begin, end, seg, 0} in caller/Morton order
    int* seg_root_rank;           // seg_cap: rank of the segment among non-empty segments
    // diagnostics partials
    double* diag_part;            // 16 * diag_blocks
    // CSR export
    int64_t* csr_tmp;             // n_cap + 1 (counts / offsets in caller order)
};

struct Dims {
    int n;            // particles
    int n_seg;        // 1 = one set
    int batched;      // n_seg > 1
    int leaf_size;
    int group_size;
    int nbr_cap;
    int group_grid;   // grid (multiple of 8) of the per-group kernels of one to four waves (lists, gravity)
    int pair_grid;    // the same for the pair kernels (density, forces)
    int wave_cap;     // wavefronts that a per-group grid may hold
    int n_sets;       // non-empty sets
    int n_chunks;
    int node_cap;
    int min_level;    // 3 when batched, else 0
    int curve;        // 0 Morton, 1 Hilbert keys
    int mass_moments; // node masses and moments are built (only the gravity kernels read them)
    int group_gravity; // gravity is the walk over target groups (quadrupole scheme)
};

// Key quantisation of one coordinate (Sec. 2.1): one subtraction, one multiplication, then
// truncation into 0 .. top (the cell index inside the cubic root cell at the finest level).
__device__ __forceinline__ u32 quantise(double x, double lo, double S, u32 top) {
    double t = (x - lo) * S;
    if (!(t > 0.0)) return 0u;
    if (t >= (double)top) return top;
    return (u32)t;
}

// ---------------------------------------------------------------------------------------
// Wave helpers (wave64 on gfx950)

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ u64 lanemask_lt() { return (1ull << lane_id()) - 1ull; }

// Scans and reductions over a full wave (all 64 lanes active) go through DPP operands of the vector
// ALU: six short dependent steps, where __shfl's LDS permutes cost an LDS round trip each (the
// one-wave walks do one scan a round and several reductions a group or tile).
// Lanes without a source in a step keep `old`.
template <int CTRL, int ROWS>
__device__ __forceinline__ u32 dpp_move(u32 old, u32 v) {
    return (u32)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
constexpr int DPP_SHR1 = 0x111, DPP_SHR2 = 0x112, DPP_SHR4 = 0x114, DPP_SHR8 = 0x118, DPP_BCAST15 = 0x142,
              DPP_BCAST31 = 0x143;

__device__ __forceinline__ int wave_incl_scan(int x) {
    u32 v = (u32)x;
    v += dpp_move<DPP_SHR1, 0xf>(0u, v);
    v += dpp_move<DPP_SHR2, 0xf>(0u, v);
    v += dpp_move<DPP_SHR4, 0xf>(0u, v);
    v += dpp_move<DPP_SHR8, 0xf>(0u, v);
    v += dpp_move<DPP_BCAST15, 0xa>(0u, v);  // rows 1 and 3 add the row before
    v += dpp_move<DPP_BCAST31, 0xc>(0u, v);  // rows 2 and 3 add the first half
    return (int)v;
}
// The last lane's value (an inclusive scan's total), in a scalar register.
__device__ __forceinline__ int wave_last(int v) { return __builtin_amdgcn_readlane(v, 63); }

// Reduction of 32-bit words by an idempotent op (a lane without a source combines with itself); the
// result is in scalar registers.
template <typename Op>
__device__ __forceinline__ u32 wave_reduce_u32(u32 v, Op op) {
    v = op(v, dpp_move<DPP_SHR1, 0xf>(v, v));
    v = op(v, dpp_move<DPP_SHR2, 0xf>(v, v));
    v = op(v, dpp_move<DPP_SHR4, 0xf>(v, v));
    v = op(v, dpp_move<DPP_SHR8, 0xf>(v, v));
    v = op(v, dpp_move<DPP_BCAST15, 0xa>(v, v));
    v = op(v, dpp_move<DPP_BCAST31, 0xc>(v, v));
    return (u32)__builtin_amdgcn_readlane((int)v, 63);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move_d(double v) {
    const u64 b = (u64)__double_as_longlong(v);
    const u32 lo = dpp_move<CTRL, ROWS>((u32)b, (u32)b), hi = dpp_move<CTRL, ROWS>((u32)(b >> 32), (u32)(b >> 32));
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
template <typename Op>
__device__ __forceinline__ double wave_reduce_d(double v, Op op) {
    v = op(v, dpp_move_d<DPP_SHR1, 0xf>(v));
    v = op(v, dpp_move_d<DPP_SHR2, 0xf>(v));
    v = op(v, dpp_move_d<DPP_SHR4, 0xf>(v));
    v = op(v, dpp_move_d<DPP_SHR8, 0xf>(v));
    v = op(v, dpp_move_d<DPP_BCAST15, 0xa>(v));
    v = op(v, dpp_move_d<DPP_BCAST31, 0xc>(v));
    const u64 b = (u64)__double_as_longlong(v);
    const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)b, 63), hi = (u32)__builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
__device__ __forceinline__ double wave_min(double v) {
    return wave_reduce_d(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ double wave_max(double v) {
    return wave_reduce_d(v, [](double a, double b) { return fmax(a, b); });
}

// Orders LDS accesses of one wave (its lanes run in step and LDS serves them in order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// W wavefronts work on one unit: the thread's index among them, and their barrier (one wavefront alone
// needs none, only its LDS accesses in order).
template <int W>
__device__ __forceinline__ int unit_thread() {
    return W == 1 ? lane_id() : (int)threadIdx.x;
}
template <int W>
__device__ __forceinline__ void unit_sync() {
    if constexpr (W == 1) wave_lds_fence();
    else __syncthreads();
}

// Owner of each of 64 consecutive items p0 + lane of a concatenation whose parts start at the
// ascending LDS offsets off[0 .. n): the last part that starts at or before the item.  `last` is the
// owner of item p0 - 1 (-1 at the start; updated): no part is empty, so at most 64 parts start among
// these items, the next ones after `last`, and an item's owner is `last` plus the starts up to it.
// One LDS read in place of a binary search's eight dependent ones.
__device__ __forceinline__ int tile_owner(const int* off, int n, int p0, int& last) {
    const int lane = lane_id();
    const int j = last + 1 + lane;
    const int o = j < n ? off[j] - p0 : 64;
    const u64 bit = o < 64 ? 1ull << o : 0ull;
    auto either = [](u32 a, u32 b) { return a | b; };
    const u64 starts = (u64)wave_reduce_u32((u32)bit, either) | ((u64)wave_reduce_u32((u32)(bit >> 32), either) << 32);
    const int own = last + __popcll(starts & (lanemask_lt() | (1ull << lane)));
    last += __popcll(starts);
    return own;
}

// Sum over the 64/gsz lanes that serve one target (lanes t, t+gsz, ...), fixed order.
__device__ __forceinline__ double lanes_sum_d(double v, int gsz) {
    for (int off = gsz; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Persistent, XCD-aware loop over groups.  Workgroups are dispatched round-robin over the
// 8 XCDs (blockIdx % 8); the workgroups of one XCD take one contiguous eighth of the groups,
// so neighbouring groups -- which read the same neighbour particles -- share an L2.
__device__ __forceinline__ void group_range(int n_groups, int& g0, int& g1, int& step) {
    const int nx = 8;
    const int xcd = (int)(blockIdx.x % nx), j = (int)(blockIdx.x / nx);
    step = (int)(gridDim.x / nx);
    const int chunk = (n_groups + nx - 1) / nx;
    g0 = xcd * chunk + j;
    g1 = min(n_groups, (xcd + 1) * chunk);
}

// Ordered-integer encoding of doubles for exact atomic min/max.
__device__ __forceinline__ u64 enc_double(double d) {
    u64 b = (u64)__double_as_longlong(d);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double dec_double(u64 e) {
    u64 b = (e >> 63) ? (e & 0x7fffffffffffffffull) : ~e;
    return __longlong_as_double((long long)b);
}

__device__ __forceinline__ void set_err(DevCtl* ctl, u32 bits) { atomicOr(&ctl->err, bits); }

// Block-wide min/max of a chunk's positions (blockDim.x a multiple of 64, at most 1024),
// merged into the segment's box with order-independent atomics on the encoded values.
__device__ __forceinline__ void box_block_merge(DevCtl* ctl, int seg, double lo[3], double hi[3], bool any) {
    __shared__ double red[16][6];
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lo[c] = wave_min(lo[c]);
        hi[c] = wave_max(hi[c]);
    }
    if (lane_id() == 0) {
        for (int c = 0; c < 3; ++c) {
            red[w][c] = lo[c];
            red[w][3 + c] = hi[c];
        }
    }
    __syncthreads();
    if (threadIdx.x < 6 && any) {
        const int c = threadIdx.x;
        double v = red[0][c];
        for (int k = 1; k < (int)(blockDim.x >> 6); ++k) v = (c < 3) ? fmin(v, red[k][c]) : fmax(v, red[k][c]);
        u64* slot = &ctl->box_enc[6 * seg + c];
        if (c < 3) atomicMin(slot, enc_double(v));
        else atomicMax(slot, enc_double(v));
    }
}

// Leading equal 3-bit digits (0..21) of two keys below the sentinel.
__device__ __forceinline__ int lcp_digits(u64 a, u64 b) {
    u64 x = (a ^ b) & 0x7fffffffffffffffull;
    if (x == 0) return MAX_LEVEL;
    return (__clzll(x) - 1) / 3;
}

// ---------------------------------------------------------------------------------------
// M4 cubic spline (support 2h): W = w(q) / (pi h^3), grad_a W_ab = r_ab g(q) / (pi h^5),
// g = w'(q) / q; and compensated FP32 accumulators.  Both pieces of w are evaluated and one is
// selected, so a wavefront never splits on q.

// g(q) given 1/q (unused, and may be inf or NaN, for q < 1)
__device__ __forceinline__ float m4_wf(float q) {
    const float t = fmaxf(2.0f - q, 0.0f);
    const float wo = 0.25f * (t * t * t);
    const float wi = fmaf(q * q, fmaf(0.75f, q, -1.5f), 1.0f);
    return q < 1.0f ? wi : wo;
}

// FP64 reciprocal and reciprocal square root of positive, normal arguments for the pair sums: the
// hardware estimates refined by one third-order step, r (1 + e + e^2) and y (1 + e/2 + 3 e^2/8) with e the
// estimate's residual (about 1e-7); within 1 ulp, not correctly rounded.
__device__ __forceinline__ double rcp_nr3(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(fma(e, e, e), r, r);
}
__device__ __forceinline__ double rsq_nr3(double a) {
    const double y = __builtin_amdgcn_rsq(a);
    const double e = fma(-a * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}
// One Newton step only: the hardware estimate (~5e-8 relative) refined to ~4e-15, for sums
// whose own approximation error is far larger (tree gravity).
__device__ __forceinline__ double rsq_nr1(double a) {
    const double y = __builtin_amdgcn_rsq(a);
    return y * fma(-0.5 * a * y, y, 1.5);
}
// 2/sqrt(a) likewise, in one operation less.
__device__ __forceinline__ double rsq2_nr1(double a) {
    const double y = __builtin_amdgcn_rsq(a);
    return y * fma(-a, y * y, 3.0);
}

// The power of two k with k v in [1, 2) (v > 0; the nearest power there is at the ends of the range).
__device__ __forceinline__ double inv_pow2(double v) {
    const int e = (int)((u64)__double_as_longlong(v) >> 52) & 0x7ff;
    return __longlong_as_double((long long)max(2046 - e, 1) << 52);
}

// Kahan accumulator (explicit operation order; the library is built without floating-point
// contraction, so it is not fused).
struct Kahan {
    float s = 0.0f, c = 0.0f;
    __device__ __forceinline__ void add(float x) {
        const float y = x - c;
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    }
    __device__ __forceinline__ double value() const { return (double)s - (double)c; }
};


// The order of k_unit_order for the list and pair kernels, where the list kernel's tail counts for more than
// the order's 4-6 us and the neighbours it parts (gravity takes it at every size).  Lists, us, in position
// order and by size: 200,003 particles in groups of 32 92 / 81, a 131,101-particle star in groups of 32
// 88 / 74, 123,480 of the tube in groups of 64 65 / 60, 50,021 in groups of 32 43 / 42, 987,840 in groups
// of 64 250 / 250, a star of 4,194,304 in groups of 32 1600 / 1670.
inline const int* group_order(const DevPtrs& d, const Dims& dm) {
    const int64_t units = dm.n / std::max(1, dm.group_size);
    return units > 2048 && units <= 8192 ? d.gorder : nullptr;
}

// Sets of 64 particles at most on average.
inline bool tiny_sets(const Dims& dm) { return dm.n <= 64 * (int64_t)dm.n_sets; }

// ---------------------------------------------------------------------------------------
// Launchers (defined in the .hip files)

// k_build.hip
void launch_fill_i32(hipStream_t s, int* p, int v, int n);
void launch_bbox(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* x, const double* y, const double* z);
void launch_set_box(hipStream_t s, const DevPtrs& d, const Dims& dm, int from_host_box);
void launch_keys(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* x, const double* y,
                 const double* z, const double* vx, const double* vy, const double* vz, const double* m,
                 const double* h, const double* u, u64* keys_out_caller);
void sort_caller_keys(hipStream_t s, const DevPtrs& d, int n);
void sort_step_keys(hipStream_t s, const DevPtrs& d, const Dims& dm);
// k_tree.hip
int64_t tree_hist_words(int64_t n);
int64_t group_hist_words(int64_t n);
// after sort_caller_keys: snapshot of the caller's particles in key order, octree and groups
void build_input_tree(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* u, int64_t* order_out);
// after sort_step_keys: the resident state moves from set a to set b = swapped(a), octree and groups
void build_step_tree(hipStream_t s, const DevPtrs& a, const DevPtrs& b, const Dims& dm);
void launch_unit_order(hipStream_t s, DevCtl* ctl, const int4* group, const u32* leaf_info, int wide_leaves, int* order);
void launch_tree_export(hipStream_t s, const DevPtrs& d, const Dims& dm, u64* key, int32_t* level,
                        int32_t* leaf, int64_t* start, int64_t* count);
// k_walk.hip
// neighbour lists + density, EOS and h_next (u_eos: the energy the EOS uses)
void launch_nbr_lists(hipStream_t s, const DevPtrs& d, const Dims& dm);
void launch_density(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double gamma, double h_coeff,
                    const double* u_eos, int kinetic_in_u);
void launch_csr_count(hipStream_t s, const DevPtrs& d, const Dims& dm, int64_t* counts_caller);
void scan_i64_inplace(hipStream_t s, int64_t* a, int n, void* tmp);
void launch_csr_fill(hipStream_t s, const DevPtrs& d, const Dims& dm, const int64_t* offsets, int32_t* idx,
                     int64_t total);
// k_sph.hip
void launch_thermo_from_caller(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* rho,
                               const double* P, const double* cs);
void launch_forces(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double alpha, double beta,
                  double eps_av, int thermokinetic);
// k_grav.hip
void launch_gravity(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double G, double eps,
                    double theta, int accumulate, int thermokinetic);
void launch_fmm(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double G, double eps, double theta,
                int accumulate, int thermokinetic);
// k_step.hip
struct ScatterArgs {
    const double* src[4];
    double* dst[4];
};
void launch_scatter_caller(hipStream_t s, const DevPtrs& d, int n, const ScatterArgs& a);
void launch_fill_zero(hipStream_t s, int n, double* dst);
void launch_box_init(hipStream_t s, const DevPtrs& d, const Dims& dm);
void launch_kick_drift(hipStream_t s, const DevPtrs& d, const Dims& dm, bool pre_kick, int adaptive_h);
void launch_kick(hipStream_t s, const DevPtrs& d, const Dims& dm, int adaptive_h);
void launch_set_hnext(hipStream_t s, const DevPtrs& d, int n);
void launch_diag(hipStream_t s, const DevPtrs& d, const Dims& dm, int with_phi, int kinetic_in_u, double eps_grav);
void launch_write_back(hipStream_t s, const DevPtrs& d, int n, double* x, double* y, double* z, double* vx,
                       double* vy, double* vz, double* h, double* u, double* ax, double* ay, double* az,
                       double* du, int kinetic_in_u);
void launch_dt_bound(hipStream_t s, const DevPtrs& d, const Dims& dm, double eps_grav);
void launch_resident_export(hipStream_t s, const DevPtrs& d, int n, u64* keys_caller, int64_t* order);
void launch_add_kinetic(hipStream_t s, const DevPtrs& d, int n);
void launch_load_accel(hipStream_t s, const DevPtrs& d, int n, const double* ax, const double* ay,
                       const double* az, const double* du);
