// Octree self-gravity (Sec. 2.2.2 of arXiv:2007.03097, eq. (10), with Plummer softening
// and quadrupole moments).
//
// One, two or four wavefronts per target group, two targets per lane.  The wide walk (by the first of them)
// tests up to 64 nodes at once against the group's box: a cell B is accepted for the whole group when its
// particle box does not touch the group box and b_B < theta d, b_B being the distance from B's centre of mass to the
// farthest corner of its particle box (B's radius about the centre of mass) and d the
// distance from the centre of mass to the group box (theta = 0 opens everything: the exact
// direct sum).  Accepted
// cells act through the second-order expansion of the softened potential about their
// centre of mass (monopole + quadrupole; the dipole vanishes there):
//   phi += -G [M/s + (3/2) R.I.R/s^5 - (1/2) tr(I)/s^3]
//   g   +=  G [-M R/s^3 + 3 I.R/s^5 - (15/2) (R.I.R) R/s^7 + (3/2) tr(I) R/s^5]
// with R = r_a - R_B, s^2 = |R|^2 + eps^2, I = sum m y y^T about R_B.  Unaccepted leaves
// contribute softened particle sums with the target itself skipped.  Cell and leaf lists
// live in LDS and are evaluated whenever they fill, so the walk needs no global scratch;
// the evaluation stages cell moments (32 a wavefront at a time in FP64, 64 in FP32C) and leaf
// particles (64 a wavefront at a time) through LDS.
#include "common.h"

constexpr int GW_STACK = 768;
constexpr int GW_CELLS = 448;
constexpr int GW_LEAVES = 256;
constexpr int GW_FOLD = 16;  // partial sums of a target that one lane adds
// Stack headroom kept free of wide rounds: popping one entry at a time (depth first), the
// stack grows by at most 7 per tree level below the popped node, so rounds of 64 entries
// stop DFS_HEADROOM entries short of the top and single-entry rounds cannot overflow it.
constexpr int DFS_HEADROOM = 7 * MAX_LEVEL + 8;
static_assert(GW_STACK > 2 * DFS_HEADROOM, "room for wide rounds above the headroom");

// LDS staging of one evaluation by W wavefronts: cell moments in the cell phase, particles in the leaf
// phase.  FP32C stages FP32 records, 64 W cells per round; FP64 stages 32 W cells of 96 bytes per round.
// With one wavefront the walk's LDS stays near 10 KB per workgroup (16 workgroups per CU).
template <bool FP32C, int W>
struct GravStage;
template <int W>
struct GravStage<false, W> {
    union {
        struct {
            double4 c0[32 * W], c1[32 * W], c2[32 * W];  // the record of cell_term
        } cell;
        struct {
            double4 pm[64 * W];  // (x, y, z, m)
            int src[64 * W];     // particle index (self test without softening)
        } part;
        double red[4][64 * W];   // a target's partial sums
    };
    int loff[GW_LEAVES + 1];  // particle offsets of the staged leaves
};
template <int W>
struct GravStage<true, W> {
    union {
        struct {             // positions as offsets from the group origin
            float4 c0[64 * W], c1[64 * W], c2[64 * W];
        } cellf;
        struct {
            float4 pm[64 * W];
            int src[64 * W];
        } partf;
    };
    int loff[GW_LEAVES + 1];
};

// Kahan-compensated FP32 sum of FP32 partial sums (one add per staged tile).
struct KahanF {
    float s = 0.0f, c = 0.0f;
    __device__ __forceinline__ void add(float x) {
        const float y = x - c;
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    }
    __device__ __forceinline__ double value() const { return (double)s - (double)c; }
};

// Per-target accumulators: FP64 sums, or FP32 sums of one staged tile (t*) that enter
// Kahan-compensated FP32 accumulators (k*) once per tile.
struct TargetSums {
    double gx = 0, gy = 0, gz = 0, ph = 0;
    float tx = 0, ty = 0, tz = 0, tph = 0;
    KahanF kx, ky, kz, kp;
    __device__ __forceinline__ void flush_tile() {
        kx.add(tx); ky.add(ty); kz.add(tz); kp.add(tph);
        tx = ty = tz = tph = 0.0f;
    }
};

// Monopole + quadrupole of a staged cell (FP64).  With the traceless Q = 3 I - tr(I) 1 the trace terms
// of the expansion cancel but for the softening's share: with u = R.Q.R - tr(I) eps^2,
//   g += -R (M/s^3 + (5/2) u/s^7) + Q.R/s^5,   phi -= M/s + (1/2) u/s^5
// (3 R.I.R = R.Q.R + tr(I) (s^2 - eps^2)), so u takes its constant from the record and starts the
// sum for free.  With 2/s for 1/s (an operation less) the powers of two go into the record,
// a = (M/8, com), b = (Qxx, Qyy, Qzz, -tr(I) eps^2)/32, d = (Qxy, Qxz, Qyz, -)/32, and the sum holds phi/4.
// The kernel is bound by its FP64 instructions (at 4M particles it runs at what the FMA probe
// sustains of the issue rate): 35 per term, 37 with the potential, against 39 and 44 with the
// trace carried along (15.7 -> 14.2 ms) and 1/s itself (node-node gravity of 262,144 particles 1.61 -> 1.58 ms,
// the walk of 4M unchanged).
template <bool PH = true>
__device__ __forceinline__ void cell_term(const double4 me, const double4 a, const double4 b, const double4 d,
                                          double e2, TargetSums& S) {
    const double Rx = me.x - a.y, Ry = me.y - a.z, Rz = me.z - a.w;
    const double QRx = fma(b.x, Rx, fma(d.x, Ry, d.y * Rz));
    const double QRy = fma(d.x, Rx, fma(b.y, Ry, d.z * Rz));
    const double QRz = fma(d.y, Rx, fma(d.z, Ry, b.z * Rz));
    const double u = fma(Rx, QRx, fma(Ry, QRy, fma(Rz, QRz, b.w)));
    const double s2 = fma(Rx, Rx, fma(Ry, Ry, fma(Rz, Rz, e2)));
    const double i1 = rsq2_nr1(s2);  // 2/s
    const double i2 = i1 * i1, i3 = i1 * i2, i5 = i3 * i2, u5 = u * i5;
    const double cR = fma(-0.625, u5 * i2, -a.x * i3);
    S.gx = fma(cR, Rx, fma(i5, QRx, S.gx));
    S.gy = fma(cR, Ry, fma(i5, QRy, S.gy));
    S.gz = fma(cR, Rz, fma(i5, QRz, S.gz));
    if constexpr (PH) S.ph = fma(-0.125, u5, fma(-a.x, i1, S.ph));
}

// Softened particle term of source sb = (x, y, z, m), m/8 in FP64 (as in cell_term).
template <bool FP32C, bool PH = true>
__device__ __forceinline__ void part_term(const double4 me, const double4 sb, double e2, TargetSums& S) {
    if (!FP32C) {
        const double dx = me.x - sb.x, dy = me.y - sb.y, dz = me.z - sb.z;
        const double s2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, e2)));
        const double i1 = rsq2_nr1(s2);  // 2/s
        const double mi1 = sb.w * i1, mi3 = mi1 * (i1 * i1);
        S.gx = fma(-mi3, dx, S.gx);
        S.gy = fma(-mi3, dy, S.gy);
        S.gz = fma(-mi3, dz, S.gz);
        if constexpr (PH) S.ph -= mi1;
    } else {
        const float dx = (float)(me.x - sb.x), dy = (float)(me.y - sb.y), dz = (float)(me.z - sb.z);
        const float s2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, (float)e2)));
        const float i1 = __builtin_amdgcn_rsqf(s2);
        const float mb = (float)sb.w;
        const float mi3 = mb * i1 * i1 * i1;
        S.tx = fmaf(-mi3, dx, S.tx);
        S.ty = fmaf(-mi3, dy, S.ty);
        S.tz = fmaf(-mi3, dz, S.tz);
        if constexpr (PH) S.tph = fmaf(-mb, i1, S.tph);
    }
}

// FP32C forms; the cell record has the constants folded in: a = (M, com), b = (3 Ixx, 3 Iyy, 3 Izz,
// 3/2 tr I), d = (3 Ixy, 3 Ixz, 3 Iyz, 1/2 tr I), so with Q = 3 I: g += -M R/s^3 + Q.R/s^5
// - (5/2) (R.Q.R) R/s^7 + (3/2) tr(I) R/s^5 and phi -= M/s + (1/2) R.Q.R/s^5 - (1/2) tr(I)/s^3.
// They work on group-origin offsets: the target and the cell's centre of mass (or the
// source particle) are FP32 offsets from the group's first target, each formed in FP64 and
// rounded once, so one FP32 subtraction gives R (its error is within u (|r_a - o| + |R_B - o|),
// small against |R| for accepted cells, and softened for near particle pairs).
template <bool PH = true>
__device__ __forceinline__ void cell_term_f(const float4 me, const float4 a, const float4 b, const float4 d, float e2,
                                            TargetSums& S) {
    const float Rx = me.x - a.y, Ry = me.y - a.z, Rz = me.z - a.w;
    const float QRx = fmaf(b.x, Rx, fmaf(d.x, Ry, d.y * Rz));
    const float QRy = fmaf(d.x, Rx, fmaf(b.y, Ry, d.z * Rz));
    const float QRz = fmaf(d.y, Rx, fmaf(d.z, Ry, b.z * Rz));
    const float RQR = fmaf(Rx, QRx, fmaf(Ry, QRy, Rz * QRz));
    const float s2 = fmaf(Rx, Rx, fmaf(Ry, Ry, fmaf(Rz, Rz, e2)));
    const float i1 = __builtin_amdgcn_rsqf(s2);
    const float i2 = i1 * i1, i3 = i1 * i2, i5 = i3 * i2, i7 = i5 * i2;
    const float cR = fmaf(b.w, i5, fmaf(-2.5f * RQR, i7, -a.x * i3));
    S.tx = fmaf(cR, Rx, fmaf(i5, QRx, S.tx));
    S.ty = fmaf(cR, Ry, fmaf(i5, QRy, S.ty));
    S.tz = fmaf(cR, Rz, fmaf(i5, QRz, S.tz));
    if constexpr (PH) S.tph -= fmaf(a.x, i1, fmaf(0.5f * RQR, i5, -d.w * i3));
}

template <bool PH = true>
__device__ __forceinline__ void part_term_f(const float4 me, const float4 sb, float e2, TargetSums& S) {
    const float dx = me.x - sb.x, dy = me.y - sb.y, dz = me.z - sb.z;
    const float s2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, e2)));
    const float i1 = __builtin_amdgcn_rsqf(s2);
    const float mi3 = sb.w * i1 * i1 * i1;
    S.tx = fmaf(-mi3, dx, S.tx);
    S.ty = fmaf(-mi3, dy, S.ty);
    S.tz = fmaf(-mi3, dz, S.tz);
    if constexpr (PH) S.tph = fmaf(-sb.w, i1, S.tph);
}

// Two targets per lane: tp and tp + TP; the P lanes with the same tp split every staged tile, so each LDS
// read of a cell or particle feeds two evaluations.  FP64: TP is half the group's targets, rounded up,
// and P = 64 W / TP over all W wavefronts (lanes past P TP idle).  FP32C, whose sums depend in their last
// bits on how the tiles are split: TP the fewest power of two that holds the targets, P = 64 / TP, and
// with W = 2 each wavefront serves one of the lane's two targets.
struct GravTargets {
    double4 a, b;
    float4 fa, fb;  // FP32C: offsets from the group origin o
    double o[3];
    int qa, qb;
    bool va, vb;
    int tp, phi, TP, P;
};

// Accepted cells (monopole + quadrupole) for the lane's targets, staged CS at a time (one
// lane loads one cell).
// A compile-time flag passed as a value, to select a template from a run-time branch.
template <bool B>
struct BoolC {
    static constexpr bool value = B;
};

template <bool FP32C, int W>
__device__ void eval_cells(int ncell, const int* cells, GravStage<FP32C, W>& St, const double4* __restrict__ mom0,
                           const double4* __restrict__ mom1, const double4* __restrict__ mom2, const GravTargets& T,
                           double e2, bool phi, TargetSums& A, TargetSums& B) {
    const int tid = unit_thread<W>();
    const bool any = T.va || T.vb;
    constexpr bool TWO = !(FP32C && W > 1);
    constexpr int CS = (FP32C ? 64 : 32) * W;  // cells staged per round
    for (int k0 = 0; k0 < ncell; k0 += CS) {
        unit_sync<W>();
        if (tid < CS && k0 + tid < ncell) {
            const int c = cells[k0 + tid];
            const double4 c0 = mom0[c], c1 = mom1[c], c2 = mom2[c];
            if constexpr (FP32C) {
                St.cellf.c0[tid] = make_float4((float)c0.x, (float)(c0.y - T.o[0]), (float)(c0.z - T.o[1]),
                                               (float)(c0.w - T.o[2]));
                St.cellf.c1[tid] = make_float4((float)(3.0 * c1.x), (float)(3.0 * c1.y), (float)(3.0 * c1.z),
                                               (float)(1.5 * c1.w));
                St.cellf.c2[tid] = make_float4((float)(3.0 * c2.x), (float)(3.0 * c2.y), (float)(3.0 * c2.z),
                                               (float)(0.5 * c1.w));
            } else {  // see cell_term
                constexpr double q = 3.0 / 32.0;
                const double tr = c1.w / 32.0;
                St.cell.c0[tid] = make_double4(0.125 * c0.x, c0.y, c0.z, c0.w);
                St.cell.c1[tid] = make_double4(fma(q, c1.x, -tr), fma(q, c1.y, -tr), fma(q, c1.z, -tr), -e2 * tr);
                St.cell.c2[tid] = make_double4(q * c2.x, q * c2.y, q * c2.z, 0.0);
            }
        }
        unit_sync<W>();
        const int cn = ncell - k0 < CS ? ncell - k0 : CS;
        auto run = [&](auto ph) {
            constexpr bool PH = decltype(ph)::value;
            if constexpr (FP32C) {
                const float e2f = (float)e2;
                for (int s = 0; s < cn; s += 64) {  // tile by tile, whatever W
                    const int e = min(s + 64, cn);
#pragma unroll TWO ? 1 : 4
                    for (int k = s + T.phi; k < e; k += T.P) {
                        const float4 a = St.cellf.c0[k], b = St.cellf.c1[k], d = St.cellf.c2[k];
                        cell_term_f<PH>(T.fa, a, b, d, e2f, A);
                        if constexpr (TWO) cell_term_f<PH>(T.fb, a, b, d, e2f, B);
                    }
                    A.flush_tile();
                    if constexpr (TWO) B.flush_tile();
                }
            } else {
                for (int k = T.phi; k < cn; k += T.P) {
                    const double4 a = St.cell.c0[k], b = St.cell.c1[k], d = St.cell.c2[k];
                    cell_term<PH>(T.a, a, b, d, e2, A);
                    cell_term<PH>(T.b, a, b, d, e2, B);
                }
            }
        };
        if (any) {
            if (phi) run(BoolC<true>());
            else run(BoolC<false>());
        }
    }
}

// Particles of the listed leaves (first particles in leaves[], counts in St.loff[], which become
// offsets), concatenated and staged through LDS 64 W at a time (one load per lane per round):
// put(slot, position, mass, index) writes the staged record, tile(tn) evaluates each staged tile of
// tn particles.  Returns the number of particles.
template <int W, typename Stage, typename Tile, typename Put>
__device__ int stage_leaves_put(int nleaf, int* leaves, Stage& St, const double4* __restrict__ pos4,
                                const double* __restrict__ m, Tile&& tile, Put&& put) {
    const int lane = lane_id(), wave = W > 1 ? threadIdx.x >> 6 : 0;
    int total = 0;
    if (W == 1 || wave == 0) {
        for (int j0 = 0; j0 < nleaf; j0 += 64) {  // particle counts of the leaves -> offsets
            const int j = j0 + lane;
            const int c = j < nleaf ? St.loff[j] : 0;
            const int incl = wave_incl_scan(c);
            if (j < nleaf) St.loff[j] = total + incl - c;
            total += wave_last(incl);
        }
        if (W > 1 && lane == 0) St.loff[nleaf] = total;
    }
    unit_sync<W>();
    if (W > 1) total = St.loff[nleaf];
    int last = -1;
    for (int p0 = 0; p0 < total; p0 += 64 * W) {
        unit_sync<W>();
        int a = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int own = tile_owner(St.loff, nleaf, p0 + 64 * w, last);
            if (w == wave) a = own;
        }
        const int p = p0 + unit_thread<W>();
        if (p < total) {
            const int src = leaves[a] + (p - St.loff[a]);
            put(unit_thread<W>(), pos4[src], m[src], src);
        }
        unit_sync<W>();
        tile(total - p0 < 64 * W ? total - p0 : 64 * W);
    }
    return total;
}

// stage_leaves_put with (x, y, z, m) records in FP64, m/8 for FP64 sums.
template <bool FP32C, int W, typename Stage, typename Tile>
__device__ int stage_leaves(int nleaf, int* leaves, Stage& St, const double4* __restrict__ pos4,
                            const double* __restrict__ m, Tile&& tile) {
    return stage_leaves_put<W>(nleaf, leaves, St, pos4, m, tile, [&](int i, const double4& ps, double mass, int src) {
        St.part.pm[i] = make_double4(ps.x, ps.y, ps.z, FP32C ? mass : 0.125 * mass);
        St.part.src[i] = src;
    });
}

// Leaves evaluated by softened particle sums (self excluded) for the lane's two targets.
// With softening the self pair is evaluated like any other (it adds no force) and its
// potential term -m_q/eps is taken out by the caller.  Returns the number of sources.
template <bool FP32C, int W>
__device__ int eval_leaves(int nleaf, int* leaves, GravStage<FP32C, W>& St, const double4* __restrict__ pos4,
                           const double* __restrict__ m, const GravTargets& T, double e2, bool phi, TargetSums& A,
                           TargetSums& B) {
    const bool any = T.va || T.vb;
    constexpr bool TWO = !(FP32C && W > 1);
    const bool soft = e2 > 0.0;
    if constexpr (FP32C) {
        const float e2f = (float)e2;
        auto run = [&](int j0, int j1, auto ph) {
            constexpr bool PH = decltype(ph)::value;
            if (soft) {
#pragma unroll TWO ? 1 : 4
                for (int j = j0 + T.phi; j < j1; j += T.P) {
                    const float4 sb = St.partf.pm[j];
                    part_term_f<PH>(T.fa, sb, e2f, A);
                    if constexpr (TWO) part_term_f<PH>(T.fb, sb, e2f, B);
                }
            } else {
                for (int j = j0 + T.phi; j < j1; j += T.P) {
                    const float4 sb = St.partf.pm[j];
                    const int s = St.partf.src[j];
                    if (s != T.qa) part_term_f<PH>(T.fa, sb, e2f, A);
                    if constexpr (TWO)
                        if (s != T.qb) part_term_f<PH>(T.fb, sb, e2f, B);
                }
            }
        };
        return stage_leaves_put<W>(
            nleaf, leaves, St, pos4, m,
            [&](int tn) {
                if (!any) return;
                for (int s = 0; s < tn; s += 64) {  // tile by tile, whatever W
                    if (phi) run(s, min(s + 64, tn), BoolC<true>());
                    else run(s, min(s + 64, tn), BoolC<false>());
                    A.flush_tile();
                    if constexpr (TWO) B.flush_tile();
                }
            },
            [&](int i, const double4& ps, double mass, int src) {
                St.partf.pm[i] = make_float4((float)(ps.x - T.o[0]), (float)(ps.y - T.o[1]), (float)(ps.z - T.o[2]),
                                             (float)mass);
                St.partf.src[i] = src;
            });
    } else {
        auto run = [&](int tn, auto ph) {
            constexpr bool PH = decltype(ph)::value;
            if (soft) {
                for (int j = T.phi; j < tn; j += T.P) {
                    const double4 sb = St.part.pm[j];
                    part_term<false, PH>(T.a, sb, e2, A);
                    part_term<false, PH>(T.b, sb, e2, B);
                }
            } else {
                for (int j = T.phi; j < tn; j += T.P) {
                    const double4 sb = St.part.pm[j];
                    const int s = St.part.src[j];
                    if (s != T.qa) part_term<false, PH>(T.a, sb, e2, A);
                    if (s != T.qb) part_term<false, PH>(T.b, sb, e2, B);
                }
            }
        };
        return stage_leaves<false, W>(nleaf, leaves, St, pos4, m, [&](int tn) {
            if (!any) return;
            if (phi) run(tn, BoolC<true>());
            else run(tn, BoolC<false>());
        });
    }
}

// The targets of one octree leaf: lane tp + TP ph serves target tp and (TWO) target tp + TP, the
// P = 64 / TP lanes of a target splitting the staged sources.  Two targets a lane halve the LDS reads
// and fill more lane slots (18 targets: 126 of 128, one a lane: 54 of 64; 40 targets: 120 of 128 and
// 40 of 64), but have twice the sums to combine and more registers: FP64 takes them for leaf
// sizes over 16, at wide angles (theta >= 0.7, short lists) over 32.  Polytropes, ms, one / two: 262,144 particles
// in leaves of 64 at theta = 0.5 1.61 / 1.37, of 32 1.57 / 1.57 and at theta = 0.8 0.40 / 0.43, of 16 2.45 / 2.59;
// 4,194,304 at theta = 1 in leaves of 64 5.24 / 5.15, of 32 6.43 / 6.96, of 16 8.73 / 9.63.  The FP32C sums, whose
// last bits depend on the split, keep one target.
struct LaneTarget {
    double4 a, b;
    int qa, qb;
    bool va, vb;
    int ph, P, TP;
};

template <bool FP32C, bool TWO, int W, typename Stage>
__device__ void eval_leaves1(int nleaf, int* leaves, Stage& St, const double4* __restrict__ pos4,
                             const double* __restrict__ m, const LaneTarget& T, double e2, bool phi, TargetSums& A,
                             TargetSums& B) {
    const bool soft = e2 > 0.0;
    auto run = [&](int tn, auto ph) {
        constexpr bool PH = decltype(ph)::value;
        if (soft) {
            for (int j = T.ph; j < tn; j += T.P) {
                const double4 s = St.part.pm[j];
                part_term<FP32C, PH>(T.a, s, e2, A);
                if constexpr (TWO) part_term<FP32C, PH>(T.b, s, e2, B);
            }
        } else {
            for (int j = T.ph; j < tn; j += T.P) {
                const int src = St.part.src[j];
                if (src != T.qa) part_term<FP32C, PH>(T.a, St.part.pm[j], e2, A);
                if constexpr (TWO)
                    if (src != T.qb) part_term<FP32C, PH>(T.b, St.part.pm[j], e2, B);
            }
        }
    };
    stage_leaves<FP32C, W>(nleaf, leaves, St, pos4, m, [&](int tn) {
        if (!T.va) return;
        if (phi) run(tn, BoolC<true>());
        else run(tn, BoolC<false>());
        if (FP32C) A.flush_tile();
    });
}

__global__ void k_zero_grav_counts(DevCtl* ctl) {
    const int s = threadIdx.x;
    if (s < GRAV_SLOTS) {
        ctl->grav_cnt[s][0] = 0;
        ctl->grav_cnt[s][1] = 0;
    }
}

// Evaluates the lists: ncell cells and the particles of nleaf leaves, each against the group's ng
// targets, and adds these numbers of terms to the group's running counts (the same in every
// lane).  A group adds them to the pass's counters once, at its end: a returnless atomic still
// holds the wave's next memory wait, and one per flush on two addresses shared by the whole
// grid cost ~12% of the 4M-particle pass.
template <bool FP32C, int W>
__device__ void eval_lists(int ncell, int nleaf, const int* cells, int* leaves, GravStage<FP32C, W>& St,
                           const double4* __restrict__ mom0,
                           const double4* __restrict__ mom1, const double4* __restrict__ mom2,
                           const double4* __restrict__ pos4, const double* __restrict__ m, const GravTargets& T,
                           double eps, bool phi, TargetSums& A, TargetSums& B, int ng, u64& n_cells, u64& n_pairs) {
    eval_cells<FP32C, W>(ncell, cells, St, mom0, mom1, mom2, T, eps * eps, phi, A, B);
    n_cells += (u64)ncell * (u64)ng;
    n_pairs += (u64)eval_leaves<FP32C, W>(nleaf, leaves, St, pos4, m, T, eps * eps, phi, A, B) * (u64)ng;
}

// W wavefronts per target group: the first one walks the tree and fills the lists, all of them evaluate.
template <bool FP32C, int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(FP32C ? 1 : 4))) k_gravity(
    DevCtl* ctl, const int* __restrict__ order, const int4* __restrict__ group, int gsz, const int4* __restrict__ topo,
    const double4* __restrict__ nbox_lo, const double4* __restrict__ nbox_hi, const double4* __restrict__ mom0,
    const double4* __restrict__ mom1, const double4* __restrict__ mom2, const double4* __restrict__ pos4,
    const double* __restrict__ m, double G, double eps, double theta, int accumulate, double* __restrict__ gxo,
    double* __restrict__ gyo, double* __restrict__ gzo, double* __restrict__ pho, const double4* __restrict__ vel4,
    double* __restrict__ deo) {
    constexpr bool TWO = !(FP32C && W > 1);
    __shared__ int stack[GW_STACK];
    __shared__ int cells[GW_CELLS];
    __shared__ int leaves[GW_LEAVES];
    __shared__ GravStage<FP32C, W> St;
    __shared__ int walked[3];  // cells and leaves listed, nodes left on the stack
    const int lane = lane_id(), wave = W > 1 ? threadIdx.x >> 6 : 0;
    GravTargets T;
    // the potential is evaluated (and written) unless the step sequence has switched it off:
    // inside a run of steps only the last step's value is read (by the energy diagnostic)
    const bool phi = pho != nullptr && ctl->skip_phi == 0;
    int g0, g1, gstep;
    group_range(ctl->n_groups, g0, g1, gstep);
    for (int ui = g0; ui < g1; ui += gstep) {
        const int4 g = group[order[ui]];
        // TP target pairs per wave: with few targets, more lanes split the tiles.  Halving the
        // targets fills 92-94% of the lane slots (groups of at most 32, 23 on average at 4M),
        // powers of two 87%.
        if (FP32C) {
            T.TP = 1;
            while (2 * T.TP < g.y && T.TP < (gsz >> 1)) T.TP <<= 1;
        } else {
            T.TP = (g.y + 1) >> 1;
        }
        const int slot = FP32C ? lane : (int)threadIdx.x;
        T.P = (FP32C ? 64 : 64 * W) / T.TP;
        T.tp = slot % T.TP;
        T.phi = slot / T.TP;
        const bool works = T.phi < T.P;
        const int ta = TWO ? T.tp : T.tp + wave * T.TP;
        T.qa = g.x + ta;
        T.qb = g.x + T.tp + T.TP;
        T.va = works && ta < g.y;
        T.vb = TWO && works && T.tp + T.TP < g.y;
        T.a = T.va ? pos4[T.qa] : make_double4(0, 0, 0, 0);
        T.b = T.vb ? pos4[T.qb] : make_double4(0, 0, 0, 0);
        if (FP32C) {
            const double4 o = pos4[g.x];
            T.o[0] = o.x;
            T.o[1] = o.y;
            T.o[2] = o.z;
            T.fa = make_float4((float)(T.a.x - o.x), (float)(T.a.y - o.y), (float)(T.a.z - o.z), 0.0f);
            T.fb = make_float4((float)(T.b.x - o.x), (float)(T.b.y - o.y), (float)(T.b.z - o.z), 0.0f);
        }
        double lo[3], hi[3];  // the group's box, for the walking wavefront
        if (W == 1 || wave == 0) {
            const double4 p = pos4[g.x + min(lane, g.y - 1)];
            lo[0] = wave_min(p.x);
            lo[1] = wave_min(p.y);
            lo[2] = wave_min(p.z);
            hi[0] = wave_max(p.x);
            hi[1] = wave_max(p.y);
            hi[2] = wave_max(p.z);
        }
        const double th2 = theta * theta;
        const u64 lt = lanemask_lt();
        TargetSums A, B;
        const int root = g.z < 0 ? 0 : ctl->level_off[3] + g.z;
        __syncthreads();
        if (threadIdx.x == 0) stack[0] = root;
        int sp = 1, iters = 0;
        u64 n_cells = 0, n_pairs = 0;
        wave_lds_fence();
        while (true) {
            int nc = 0, nl = 0;
            // until the lists may not hold another round or the walk has ended
            while ((W == 1 || wave == 0) && sp > 0 && nc + 64 <= GW_CELLS && nl + 64 <= GW_LEAVES) {
                if (++iters > (1 << 22)) {  // bounded: every wave leaves the loop
                    if (lane == 0) set_err(ctl, ERR_GRAV_LIST);
                    sp = 0;
                    break;
                }
                // pop as many nodes as the stack can take the children of (8 each) while keeping
                // the depth-first headroom; past it, one node per round
                int k = sp < 64 ? sp : 64;
                const int room = (GW_STACK - DFS_HEADROOM - sp) / 8;
                if (k > room) k = room > 1 ? room : 1;
                const int node = lane < k ? stack[sp - k + lane] : -1;
                wave_lds_fence();
                sp -= k;
                int kind = 0;  // 1 = accepted cell, 2 = leaf to open, 3 = open children
                int4 tp = make_int4(0, 0, 0, 0);
                if (node >= 0) {
                    tp = topo[node];
                    const double4 a = nbox_lo[node], b = nbox_hi[node], m0 = mom0[node];
                    const double com[3] = {m0.y, m0.z, m0.w};
                    double d2 = 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double gp = com[c] < lo[c] ? lo[c] - com[c] : (com[c] > hi[c] ? com[c] - hi[c] : 0.0);
                        d2 += gp * gp;
                    }
                    const bool apart =
                        a.x > hi[0] || b.x < lo[0] || a.y > hi[1] || b.y < lo[1] || a.z > hi[2] || b.z < lo[2];
                    const double ux = fmax(com[0] - a.x, b.x - com[0]), uy = fmax(com[1] - a.y, b.y - com[1]),
                                 uz = fmax(com[2] - a.z, b.z - com[2]);
                    const double b2 = (ux * ux + uy * uy) + uz * uz;  // radius^2 about the centre of mass
                    if (apart && b2 < th2 * d2) kind = 1;
                    else kind = tp.w ? 2 : 3;
                }
                const u64 bc = __ballot(kind == 1), bl = __ballot(kind == 2);
                if (kind == 1) cells[nc + __popcll(bc & lt)] = node;
                if (kind == 2) {
                    leaves[nl + __popcll(bl & lt)] = tp.x;
                    St.loff[nl + __popcll(bl & lt)] = tp.y;
                }
                nc += __popcll(bc);
                nl += __popcll(bl);
                const int nch = kind == 3 ? tp.y : 0;
                const int incl = wave_incl_scan(nch);
                const int tot = wave_last(incl);
                if (sp + tot > GW_STACK) {
                    if (lane == 0) set_err(ctl, ERR_GRAV_LIST);
                    sp = 0;
                    break;
                }
                for (int j = 0; j < nch; ++j) stack[sp + incl - nch + j] = tp.x + j;
                sp += tot;
                wave_lds_fence();
            }
            if (W > 1) {
                if (threadIdx.x == 0) {
                    walked[0] = nc;
                    walked[1] = nl;
                    walked[2] = sp;
                }
                __syncthreads();
                nc = walked[0];
                nl = walked[1];
                sp = walked[2];
            }
            eval_lists<FP32C, W>(nc, nl, cells, leaves, St, mom0, mom1, mom2, pos4, m, T, eps, phi, A, B, g.y, n_cells,
                                 n_pairs);
            __syncthreads();
            if (sp <= 0) break;
        }
        // per target: lanes tp + TP*phi combine in a fixed order
        double r[8];
        if constexpr (FP32C) {
            r[0] = A.kx.value(); r[1] = A.ky.value(); r[2] = A.kz.value(); r[3] = A.kp.value();
            r[4] = B.kx.value(); r[5] = B.ky.value(); r[6] = B.kz.value(); r[7] = B.kp.value();
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] = G * lanes_sum_d(r[i], T.TP);  // (B: zero if !TWO)
        } else {
            // With more than GW_FOLD sums a target, the first GW_FOLD of its lanes add the others' first: a group
            // of one target has up to 256, and one lane took 17 us to add them (a set of one particle 25 -> 41
            // us, 512 sets of two particles 68 -> 278 us).
            double v[8] = {A.gx, A.gy, A.gz, 4.0 * A.ph, B.gx, B.gy, B.gz, 4.0 * B.ph};
            const int tid = threadIdx.x, last = 64 * W - 1;
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                int P = T.P;
                while (true) {
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < 4; ++i) St.red[i][tid] = v[h + i];
                    __syncthreads();
                    if (P <= GW_FOLD) break;
                    if (T.phi < GW_FOLD)
                        for (int k = GW_FOLD; T.phi + k < P; k += GW_FOLD)
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[h + i] += St.red[i][tid + k * T.TP];
                    P = GW_FOLD;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    double t = v[h + i];  // the lanes with phi = 0 use it
                    for (int k = 1; k < P; ++k) t += St.red[i][min(tid + k * T.TP, last)];
                    r[h + i] = G * t;
                }
            }
        }
        if (T.phi == 0) {
            for (int s = 0; s < 2; ++s) {
                if (!(s ? T.vb : T.va)) continue;
                const int q = s ? T.qb : T.qa;
                double gx = r[4 * s], gy = r[4 * s + 1], gz = r[4 * s + 2], ph = r[4 * s + 3];
                if (eps > 0.0) {  // take out the self pair's potential term (see eval_lists)
                    const double e2 = eps * eps;
                    const double is = FP32C ? (double)__builtin_amdgcn_rsqf((float)e2) : 0.5 * rsq2_nr1(e2);
                    ph += G * (m[q] * is);
                }
                if (accumulate) {
                    gxo[q] += gx;
                    gyo[q] += gy;
                    gzo[q] += gz;
                    if (deo) {  // thermokinetic form: the work of gravity on e = u + v^2/2
                        const double4 v = vel4[q];
                        deo[q] += fma(v.x, gx, fma(v.y, gy, v.z * gz));
                    }
                } else {
                    gxo[q] = gx;
                    gyo[q] = gy;
                    gzo[q] = gz;
                }
                if (phi) pho[q] = ph;
            }
        }
        if (threadIdx.x == 0) {  // last, so that no later memory wait of the group holds for it
            u64* slot = ctl->grav_cnt[ui & (GRAV_SLOTS - 1)];
            atomicAdd(&slot[0], n_cells);
            atomicAdd(&slot[1], n_pairs);
        }
    }
}

void launch_gravity(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double G, double eps, double theta,
                    int accumulate, int thermo) {
    if (dm.n <= 0) return;
    double* gx = accumulate ? d.ax : d.gx;
    double* gy = accumulate ? d.ay : d.gy;
    double* gz = accumulate ? d.az : d.gz;
    double* de = (accumulate && thermo) ? d.du : nullptr;
    hipLaunchKernelGGL(k_zero_grav_counts, dim3(1), dim3(64), 0, s, d.ctl);
    auto go = [&](auto kern, int waves) {
        const int grid = std::min(dm.group_grid, 8 * std::max(1, dm.wave_cap / (8 * waves)));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * waves), 0, s, d.ctl, d.gorder, d.group, dm.group_size, d.topo,
                           d.nbox_lo, d.nbox_hi, d.mom0, d.mom1, d.mom2, d.pos4, d.m, G, eps, theta, accumulate, gx, gy,
                           gz, d.phi, d.vel4, de);
    };
    // Wavefronts a group: with few groups the chip is not full of single wavefronts.  With the tree, us,
    // for 1 / 2 / 4 (FP32C 1 / 2): 20,011 particles in groups of 32, FP64 254 / 229 / 210, FP32C 240 / 209;
    // 50,000 in groups of 32, 331 / 304 / 341 and 290 / 270; 262,144 in groups of 64, 1197 / 1078 / 1132 and
    // 875 / 816; 131,101 in groups of 32, 534 / 538 and 445 / 456; 500,000 in groups of 64, 1638 / 1639 and
    // 1114 / 1217.  Groups of 16 lack the targets for four (8,000 particles: 153 / 146 / 155).
    const int64_t units = dm.n / std::max(1, dm.group_size);
    // Sets of up to 64 particles are one tile, which one wavefront evaluates.
    const bool one = units > 64 * dm.group_size || tiny_sets(dm);
    const int W = one ? 1 : (units > 1024 || dm.group_size <= 16 || fp32c ? 2 : 4);
    if (fp32c) {
        // FP32C sums are the same bit for bit by one and by two wavefronts, so a cap on the wavefronts that leaves
        // fewer than two a group goes to more groups at once (50,000 particles, one a CU: 618 -> 456 us).  FP64 sums
        // are not, and results do not depend on the cap: there it costs up to twice the time of one a group.
        if (W > 1 && dm.group_grid <= dm.wave_cap / 2) go(k_gravity<true, 2>, 2);
        else go(k_gravity<true, 1>, 1);
    } else {
        if (W > 2) go(k_gravity<false, 4>, 4);
        else if (W > 1) go(k_gravity<false, 2>, 2);
        else go(k_gravity<false, 1>, 1);
    }
}

// ---------------------------------------------------------------------------------------
// Symmetric node-node gravity: the paper's own scheme (Sec. 2.2.2, eq. (10), after Dehnen
// 2000).
//
// Interaction set: the mutual recursion over node pairs.  A node paired with itself splits
// into its children's self pairs and every unordered pair of children (a leaf sums its
// particle pairs).  A pair (A, B) of distinct nodes is one node-node term when the opening
// test accepts it; else every particle pair when both are leaves; else the larger node
// (lower level; on equal levels the one whose particles come first in key order) is split,
// unless it is a leaf, in which case the other one is.
//
// Opening test: every octree cell (the cells of the key quantisation) lies inside the
// sphere of radius (sqrt 3 / 2) side about its centre; (A, B) is accepted when
// r_A + r_B < theta |c_A - c_B|.  In integer units of half the finest cell this reads
// 3 T^2 < 4 theta^2 |D|^2 with T = 2 (s_A + s_B) and D = 2 (c_A - c_B), so every decision is
// exact and independent of rounding.  theta = 0 accepts nothing: the direct sum.
//
// Node-node term: first order in the Taylor expansion of the potential about each centre
// of mass, with monopole sources.  Node Y acts on node X through g = -G M_Y R / s^3 at R_X
// (R = R_X - R_Y, s^2 = |R|^2 + eps^2), constant across X, and the potential
// -G M_Y / s - g . (r - R_X).  R flips sign bit for bit between the two directions of a
// pair, so the forces two nodes exert on each other are opposite and central: linear and
// angular momentum are conserved up to rounding.
//
// GPU form: every leaf of the tree is a target of one wavefront (or four), which replays the part of
// the recursion that involves the leaf's ancestors X_0 (root) .. X_D (the leaf): each self
// pair (X_e, X_e) yields the pairs (X_e+1, C) for the other children C of X_e, and a pair
// (X_e, Y) either ends (term or particle pairs), moves down the path (X split) or fans out
// over Y's children.  Every node-node term of an ancestor is evaluated once per leaf below
// it -- no scatter, no atomics, a fixed summation order.  The lanes evaluate 64 accepted
// pairs at a time (one each) and sum the constant fields across the wave at the end;
// the particle pairs of unaccepted leaf pairs go through eval_leaves1 (a leaf fills a wave
// poorly, so several lanes share each of its targets).  The
// potential's linear part is referred to the leaf's centre of mass.
constexpr int FM_STACK = 672;
constexpr int FM_TERMS = 192;
constexpr int FM_LEAVES = 192;
constexpr int FM_TARGETS = 64;    // targets per pass over a leaf
static_assert(7 * MAX_LEVEL + DFS_HEADROOM <= FM_STACK, "the initial pairs of a path and the headroom fit");

// LDS staging of the particle sums (the node-node walk has no cell tiles).
template <int W>
struct FmmStage {
    struct {
        double4 pm[64 * W];  // (x, y, z, m)
        int src[64 * W];     // particle index (self test without softening)
    } part;
    int loff[FM_LEAVES + 1];  // particle offsets of the staged leaves
};

struct FmmPath {
    double4 com[MAX_LEVEL + 1];  // (M, centre of mass) of the ancestor at each depth
    int4 topo[MAX_LEVEL + 1];    // its topology record
    int node[MAX_LEVEL + 1];
    int start[MAX_LEVEL + 1];    // its first particle (key order)
    int cell[MAX_LEVEL + 1][3];  // its integer cell coordinates at its level
};

// Integer coordinates of the cell of every node: its first particle, quantised as for the
// keys and truncated to the node's level; packed 21 bits per axis into the free fourth
// component of mom2 (the walk then reads them with the node's topology, not after it).  Also each leaf's
// level and particle count (at most 64) for k_unit_order, in leaf order: level << 8 | count.
__global__ void __launch_bounds__(256) k_fmm_cells(const DevCtl* __restrict__ ctl, const int4* __restrict__ topo,
                                                    const int2* __restrict__ range, const double4* __restrict__ pos4,
                                                    const int* __restrict__ node_first, double4* mom2, u32* leaf_info) {
    const double lo[3] = {ctl->box[0], ctl->box[1], ctl->box[2]};
    const double S = ctl->scale[0];
    const u32 top = (1u << MAX_LEVEL) - 1u;
    const int nn = ctl->n_nodes;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nn; b += gridDim.x * blockDim.x) {
        const double4 p = pos4[range[b].x];
        const int4 t = topo[b];
        const int f = node_first[b];
        if (f < 0) leaf_info[~f] = ((u32)t.z << 8) | (u32)min(t.y, 64);
        const int sh = MAX_LEVEL - t.z;
        const u64 c = (u64)(quantise(p.x, lo[0], S, top) >> sh) | ((u64)(quantise(p.y, lo[1], S, top) >> sh) << 21) |
                      ((u64)(quantise(p.z, lo[2], S, top) >> sh) << 42);
        mom2[b].w = __longlong_as_double((long long)c);
    }
}

__device__ __forceinline__ void fmm_unpack(u64 c, int* v) {
    v[0] = (int)(c & 0x1fffff);
    v[1] = (int)((c >> 21) & 0x1fffff);
    v[2] = (int)(c >> 42);
}

// 3 T^2 < 4 theta^2 |D|^2: coordinates and sides are below 2^23, so their differences are exact in 32 bits
// and the squares and sums (below 2^48) exact in FP64, at a fraction of 64-bit integer products.
__device__ __forceinline__ bool fmm_accept(int la, const int* ca, int lb, const int* cb, double th4) {
    const double T = (double)((1 << (MAX_LEVEL - la + 1)) + (1 << (MAX_LEVEL - lb + 1)));
    double D2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int a = (2 * ca[d] + 1) << (MAX_LEVEL - la);
        const int b = (2 * cb[d] + 1) << (MAX_LEVEL - lb);
        const double e = (double)(a - b);
        D2 = fma(e, e, D2);
    }
    return 3.0 * (T * T) < th4 * D2;
}

// Accepted pairs (tnode[k], depth tdep[k]): lane k evaluates pair k, k + 64, ... and keeps
// its own partial sums of the field (fg) and of the potential referred to the leaf's
// centre of mass (fc); the caller sums them across the wave.
template <bool PH, int W>
__device__ __forceinline__ void fmm_eval_terms(int nt, const int* tnode, const unsigned char* tdep, const FmmPath& P,
                                               int D, const double4* __restrict__ mom0, double e2, double& fgx,
                                               double& fgy, double& fgz, double& fc) {
    const double4 cl = P.com[D];
    for (int k = unit_thread<W>(); k < nt; k += 64 * W) {
        const double4 cx = P.com[tdep[k]];
        const double4 cy = mom0[tnode[k]];
        const double Rx = cx.y - cy.y, Ry = cx.z - cy.z, Rz = cx.w - cy.w;
        const double s2 = fma(Rx, Rx, fma(Ry, Ry, fma(Rz, Rz, e2)));
        const double i1 = rsq_nr1(s2);
        const double mi1 = cy.x * i1;
        const double mi3 = mi1 * i1 * i1;
        const double gx = -mi3 * Rx, gy = -mi3 * Ry, gz = -mi3 * Rz;
        fgx += gx;
        fgy += gy;
        fgz += gz;
        if constexpr (PH) fc -= mi1 + fma(gx, cl.y - cx.y, fma(gy, cl.z - cx.z, gz * (cl.w - cx.w)));
    }
}

// LDS of W wavefronts that work on one leaf.
template <int W>
struct FmmLds {
    int stk[FM_STACK];
    int tnode[FM_TERMS];
    int leaves[FM_LEAVES];
    unsigned char sdep[FM_STACK], tdep[FM_TERMS];
    int walked[3];   // pairs and leaves listed, pairs left on the stack
    double4 far[W];  // the waves' constant fields
    FmmStage<W> St;
    FmmPath Pth;
};

struct FmmArgs {
    DevCtl* ctl;
    const int* order;
    const int* leaf_node;
    const int* parent;
    const int4* topo;
    const int2* range;
    const double4* mom0;
    const double* ncell;
    const double4* pos4;
    const double* m;
    double G, eps, th4;
    int accumulate;
    double *gxo, *gyo, *gzo, *pho;
    const double4* vel4;
    double* deo;
};

// Leaf L by W wavefronts: the first one replays the recursion and fills the lists, all of them evaluate.
template <bool FP32C, bool TWO, int W>
__device__ __forceinline__ void fmm_leaf(const FmmArgs& K, FmmLds<W>& S, int L, bool phi) {
    DevCtl* ctl = K.ctl;
    const int* __restrict__ parent = K.parent;
    const int4* __restrict__ topo = K.topo;
    const int2* __restrict__ range = K.range;
    const double4* __restrict__ mom0 = K.mom0;
    const double* __restrict__ ncell = K.ncell;
    const double4* __restrict__ pos4 = K.pos4;
    const double* __restrict__ m = K.m;
    const double G = K.G, eps = K.eps, th4 = K.th4, e2 = eps * eps;
    const int lane = lane_id(), tid = unit_thread<W>(), wave = W > 1 ? threadIdx.x >> 6 : 0;
    const u64 lt = lanemask_lt();
    const int4 tl = topo[L];
    const int D = tl.z;  // one set: the root is at level 0
    unit_sync<W>();
    if (tid == 0) {
        int b = L;
        for (int e = D; e >= 0; --e) {
            S.Pth.node[e] = b;
            b = e > 0 ? parent[b] : -1;
        }
    }
    unit_sync<W>();
    if ((W == 1 || wave == 0) && lane <= D) {
        const int b = S.Pth.node[lane];
        const int4 t = topo[b];
        const int st = range[b].x;
        S.Pth.topo[lane] = t;
        S.Pth.start[lane] = st;
        S.Pth.com[lane] = mom0[b];
        fmm_unpack((u64)__double_as_longlong(ncell[4 * b]), S.Pth.cell[lane]);
    }
    unit_sync<W>();
    const double4 cl = S.Pth.com[D];
    for (int t0 = 0; t0 < tl.y; t0 += FM_TARGETS) {
        const int cc = min(FM_TARGETS, tl.y - t0);
        LaneTarget T;
        T.TP = TWO ? (cc + 1) >> 1 : cc;
        T.P = 64 * W / T.TP;
        T.ph = tid / T.TP;
        const int tp = tid - T.ph * T.TP;
        T.qa = tl.x + t0 + tp;
        T.qb = T.qa + T.TP;
        T.va = T.ph < T.P;
        T.vb = TWO && T.va && tp + T.TP < cc;
        T.a = T.va ? pos4[T.qa] : make_double4(0, 0, 0, 0);
        T.b = T.vb ? pos4[T.qb] : make_double4(0, 0, 0, 0);  // (not T.a: a choice of addresses puts T in scratch memory)
        // initial pairs: (X_e+1, C) for every other child C of every ancestor X_e
        const int n0 = lane < D ? S.Pth.topo[lane].y - 1 : 0;
        const int incl = wave_incl_scan(n0);
        int sp = wave_last(incl);
        if ((W == 1 || wave == 0) && lane < D) {
            const int4 t = S.Pth.topo[lane];
            const int nxt = S.Pth.node[lane + 1];
            int o = incl - n0;
            for (int j = 0; j < t.y; ++j) {
                const int ch = t.x + j;
                if (ch != nxt) {
                    S.stk[o] = ch;
                    S.sdep[o] = (unsigned char)(lane + 1);
                    ++o;
                }
            }
        }
        if (tid == 0) {  // the leaf's own particle pairs
            S.leaves[0] = tl.x;
            S.St.loff[0] = tl.y;
        }
        int nt = 0, nl = 1, iters = 0;
        TargetSums A, B;
        double fgx = 0.0, fgy = 0.0, fgz = 0.0, fc = 0.0;
        unit_sync<W>();
        while (true) {
            // until a list may not hold another round or the walk has ended
            while ((W == 1 || wave == 0) && sp > 0 && nt + 64 <= FM_TERMS && nl + 64 <= FM_LEAVES) {
                if (++iters > (1 << 22)) {  // bounded: every wave leaves the loop
                    if (lane == 0) set_err(ctl, ERR_GRAV_LIST);
                    sp = 0;
                    break;
                }
                int k = sp < 64 ? sp : 64;  // wide rounds only above the depth-first headroom
                const int room = (FM_STACK - DFS_HEADROOM - sp) / 8;
                if (k > room) k = room > 1 ? room : 1;
                int Y = -1, e = 0;
                if (lane < k) {
                    Y = S.stk[sp - k + lane];
                    e = S.sdep[sp - k + lane];
                }
                wave_lds_fence();
                sp -= k;
                int kind = 0;  // 1 = node-node term, 2 = leaf pair, 3 = split X, 4 = split Y
                int4 ty = make_int4(0, 0, 0, 0);
                if (Y >= 0) {
                    ty = topo[Y];
                    const int sy = range[Y].x;
                    int cy[3];
                    fmm_unpack((u64)__double_as_longlong(ncell[4 * Y]), cy);
                    const int4 tx = S.Pth.topo[e];
                    if (fmm_accept(tx.z, S.Pth.cell[e], ty.z, cy, th4)) {
                        kind = 1;
                    } else if (tx.w && ty.w) {
                        kind = 2;
                    } else {
                        bool split_x = tx.z < ty.z || (tx.z == ty.z && S.Pth.start[e] < sy);
                        if (split_x ? tx.w : ty.w) split_x = !split_x;
                        kind = split_x ? 3 : 4;
                    }
                }
                const u64 bt = __ballot(kind == 1), bl = __ballot(kind == 2);
                if (kind == 1) {
                    const int o = nt + __popcll(bt & lt);
                    S.tnode[o] = Y;
                    S.tdep[o] = (unsigned char)e;
                }
                if (kind == 2) {
                    S.leaves[nl + __popcll(bl & lt)] = ty.x;
                    S.St.loff[nl + __popcll(bl & lt)] = ty.y;
                }
                nt += __popcll(bt);
                nl += __popcll(bl);
                const int np = kind == 3 ? 1 : (kind == 4 ? ty.y : 0);
                const int pin = wave_incl_scan(np);
                const int tot = wave_last(pin);
                if (sp + tot > FM_STACK) {
                    if (lane == 0) set_err(ctl, ERR_GRAV_LIST);
                    sp = 0;
                    break;
                }
                if (kind == 3) {
                    S.stk[sp + pin - 1] = Y;
                    S.sdep[sp + pin - 1] = (unsigned char)(e + 1);
                } else if (kind == 4) {
                    for (int j = 0; j < np; ++j) {
                        S.stk[sp + pin - np + j] = ty.x + j;
                        S.sdep[sp + pin - np + j] = (unsigned char)e;
                    }
                }
                sp += tot;
                wave_lds_fence();
            }
            if (W > 1) {
                if (tid == 0) {
                    S.walked[0] = nt;
                    S.walked[1] = nl;
                    S.walked[2] = sp;
                }
                unit_sync<W>();
                nt = S.walked[0];
                nl = S.walked[1];
                sp = S.walked[2];
            }
            // each list by itself, when it is full: FP32C sums depend on how a list's tiles are cut
            if (nt + 64 > FM_TERMS || sp <= 0) {
                if (phi) fmm_eval_terms<true, W>(nt, S.tnode, S.tdep, S.Pth, D, mom0, e2, fgx, fgy, fgz, fc);
                else fmm_eval_terms<false, W>(nt, S.tnode, S.tdep, S.Pth, D, mom0, e2, fgx, fgy, fgz, fc);
                nt = 0;
            }
            if (nl + 64 > FM_LEAVES || sp <= 0) {
                eval_leaves1<FP32C, TWO, W>(nl, S.leaves, S.St, pos4, m, T, e2, phi, A, B);
                nl = 0;
            }
            unit_sync<W>();
            if (sp <= 0) break;
        }
        fgx = lanes_sum_d(fgx, 1);
        fgy = lanes_sum_d(fgy, 1);
        fgz = lanes_sum_d(fgz, 1);
        fc = lanes_sum_d(fc, 1);
        if (W > 1) {
            if (lane == 0) S.far[wave] = make_double4(fgx, fgy, fgz, fc);
            unit_sync<W>();
            double4 f = S.far[0];
            for (int w = 1; w < W; ++w) {
                f.x += S.far[w].x;
                f.y += S.far[w].y;
                f.z += S.far[w].z;
                f.w += S.far[w].w;
            }
            fgx = f.x; fgy = f.y; fgz = f.z; fc = f.w;
        }
        // each target's P partial sums (lanes tp + TP ph) combined in phase order
        for (int h = 0; h < (TWO ? 2 : 1); ++h) {
            unit_sync<W>();
            if (FP32C) S.St.part.pm[tid] = make_double4(A.kx.value(), A.ky.value(), A.kz.value(), A.kp.value());
            else if (TWO && h) S.St.part.pm[tid] = make_double4(B.gx, B.gy, B.gz, 4.0 * B.ph);
            else S.St.part.pm[tid] = make_double4(A.gx, A.gy, A.gz, 4.0 * A.ph);
            unit_sync<W>();
            if (!(h ? T.vb : T.va) || T.ph != 0) continue;
            double4 r = S.St.part.pm[tid];
            for (int k = 1; k < T.P; ++k) {
                const double4 o = S.St.part.pm[tid + k * T.TP];
                r.x += o.x;
                r.y += o.y;
                r.z += o.z;
                r.w += o.w;
            }
            const int q = h ? T.qb : T.qa;
            const double4 me = h ? T.b : T.a;
            const double lin = fma(fgx, me.x - cl.y, fma(fgy, me.y - cl.z, fgz * (me.z - cl.w)));
            const double gx = G * (r.x + fgx), gy = G * (r.y + fgy), gz = G * (r.z + fgz);
            double ph = G * (r.w + (fc - lin));
            if (eps > 0.0) {  // take out the self pair's potential term (see eval_leaves1)
                const double is = FP32C ? (double)__builtin_amdgcn_rsqf((float)e2) : 0.5 * rsq2_nr1(e2);
                ph += G * (m[q] * is);
            }
            if (K.accumulate) {
                K.gxo[q] += gx;
                K.gyo[q] += gy;
                K.gzo[q] += gz;
                if (K.deo) {  // thermokinetic form: the work of gravity on e = u + v^2/2
                    const double4 v = K.vel4[q];
                    K.deo[q] += fma(v.x, gx, fma(v.y, gy, v.z * gz));
                }
            } else {
                K.gxo[q] = gx;
                K.gyo[q] = gy;
                K.gzo[q] = gz;
            }
            if (phi) K.pho[q] = ph;
        }
    }
}

// One workgroup of four wavefronts takes one heavy leaf, or four others, one each.  A leaf that is far larger
// than its neighbours' (few particles at the edge of a set, next to many small cells) opens everything
// around it down to the particles: eight such leaves of the 262,144-particle polytrope ran 0.7 ms longer
// than all other work in one wavefront each.  With at most 4,096 leaves (four
// workgroups a CU hold 1,024 at once) leaves of 16 targets and more count as heavy too; smaller ones are
// bound by the walk, which one wavefront does.  Where the angle is wide, leaves have less to evaluate beside
// their walk, and the limit is 3,072.  At theta = 0.5, us, for limits of 0 / 1,024 / 2,048 / 4,096 leaves: 3,000
// particles in leaves of 48 176 / 71 / 72 / 71, 20,011 in leaves of 32 210 / 209 / 170 / 170, 35,000
// in leaves of 64 517 / 519 / 309 / 314, 50,000 in leaves of 64 655 / 656 / 655 / 450; at theta = 1, 3,072 / 4,096:
// a flat 60,000 in leaves of 32 42 / 73.
// Four leaves a workgroup, sizes in order and the heavy leaves together: 262,144 particles 2.18 -> 1.56 ms.
// The FP32C sums, whose last bits depend on the split, keep one wavefront a leaf.
template <bool FP32C, bool TWO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FP32C ? 1 : 4))) k_fmm(const FmmArgs K) {
    __shared__ __align__(32) char lds[4 * sizeof(FmmLds<1>)];
    static_assert(sizeof(FmmLds<4>) <= sizeof(lds), "the workgroup's form fits the four wavefronts' areas");
    const bool phi = K.pho != nullptr && K.ctl->skip_phi == 0;  // as in k_gravity
    int l0, l1, step;
    group_range(K.ctl->n_leaves, l0, l1, step);
    const int first = l0 - (int)(blockIdx.x / 8);  // the share's first leaf
    const int heavy = FP32C ? 0 : K.ctl->fmm_heavy[blockIdx.x & 7];
    for (int j = blockIdx.x / 8;; j += step) {
        if (j < heavy) {
            if constexpr (!FP32C)
                fmm_leaf<FP32C, TWO, 4>(K, *reinterpret_cast<FmmLds<4>*>(lds), K.leaf_node[K.order[first + j]], phi);
            __syncthreads();
            continue;
        }
        const int u = first + heavy + 4 * (j - heavy);
        if (u >= l1) break;
        const int w = u + (int)(threadIdx.x >> 6);
        if (w < l1)
            fmm_leaf<FP32C, TWO, 1>(K, reinterpret_cast<FmmLds<1>*>(lds)[threadIdx.x >> 6], K.leaf_node[K.order[w]], phi);
    }
}

void launch_fmm(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double G, double eps, double theta,
                int accumulate, int thermo) {
    if (dm.n <= 0) return;
    double* gx = accumulate ? d.ax : d.gx;
    double* gy = accumulate ? d.ay : d.gy;
    double* gz = accumulate ? d.az : d.gz;
    double* de = (accumulate && thermo) ? d.du : nullptr;
    const double th4 = 4.0 * (theta * theta);
    const double* ncell = &d.mom2[0].w;  // stride 4 doubles
    const int cg = std::min(2048, (dm.node_cap + 255) / 256);
    u32* leaf_info = d.val_b;  // the sort's scratch: free from one build to the next
    hipLaunchKernelGGL(k_fmm_cells, dim3(cg), dim3(256), 0, s, d.ctl, d.topo, d.range,
                       d.pos4, d.node_first, d.mom2, leaf_info);
    int* order = reinterpret_cast<int*>(d.gsize);  // free once the groups are emitted
    const bool wide_angle = theta >= 0.7;
    const int wide_leaves = wide_angle ? 3072 : 4096;
    launch_unit_order(s, d.ctl, nullptr, leaf_info, wide_leaves, order);
    // four leaves a workgroup, about 3 n / leaf_size of them; the kernel loops over any beyond that.  Few leaves
    // may all be heavy, one a workgroup (8,000 uniform particles in leaves of 64 on a quarter of the workgroups:
    // 209 -> 110 us).
    const int fours = dm.n / std::max(1, dm.leaf_size);
    const int ones = fp32c ? 0 : (int)std::min<int64_t>(3ll * fours, wide_leaves);
    const int grid = std::min(8 * ((std::max(fours, ones) + 23) / 8), 8 * std::max(1, dm.wave_cap / 32));
    const FmmArgs K{d.ctl, order, d.leaf_node, d.parent, d.topo, d.range, d.mom0, ncell, d.pos4, d.m, G, eps, th4,
                    accumulate, gx, gy, gz, d.phi, d.vel4, de};
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, s, K); };
    if (fp32c) go(k_fmm<true, false>);
    else if (dm.leaf_size > (wide_angle ? 32 : 16)) go(k_fmm<false, true>);  // see LaneTarget
    else go(k_fmm<false, false>);
}
