// SPH pair sums (Sec. 2.2.1 of arXiv:2007.03097):
//   density (eq. (7)):  rho_a = sum_b m_b W(r_ab, h_ab), self included; ideal-gas EOS
//                       P = (gamma - 1) rho u, c = sqrt(gamma P / rho); h_next (eq. (9))
//   momentum (eq. (6)): dv_a/dt = -sum_b m_b ((P_a/rho_a^2 + P_b/rho_b^2) + Pi_ab) grad_a W_ab
//   energy (eq. (5)):   du_a/dt =  sum_b m_b (P_a/rho_a^2 + Pi_ab/2) v_ab . grad_a W_ab
//   or, thermokinetic (eq. (8)), e = u + v^2/2:
//                       de_a/dt = -sum_b m_b (P_a v_b/rho_a^2 + P_b v_a/rho_b^2
//                                             + (v_a + v_b)/2 Pi_ab) . grad_a W_ab
//   viscosity:          Pi_ab = (-alpha cbar mu + beta mu^2)/rhobar if v_ab . r_ab < 0,
//                       mu = h_ab v_ab . r_ab / (r^2 + eps h_ab^2)
// with the M4 cubic spline, W = w(q)/(pi h^3), grad_a W_ab = r_ab g(q)/(pi h^5), g = w'(q)/q.
//
// One workgroup of NT = 256 threads (128 for small groups in FP64) per target group, in an XCD-aware loop
// over the groups.  The group's
// source union (built with the lists) is staged in LDS in chunks; each of the group's n_g
// targets is served by PL = NT/n_g threads that take every PL-th entry of its list --
// entries are ascending union indices, so each thread walks its entries once across the
// chunks --
// and read the source records from LDS.  The partial sums of a target are added in a
// fixed order, so results are bitwise reproducible.  The pair sums are not a dense
// contraction (each target has its own irregular list), so they run on the vector ALUs,
// not on the matrix cores.
//
// FP32C: in the density pass positions enter as FP32 offsets from the group's first particle
// (each offset formed in FP64, then rounded), so a pair's difference is one FP32 subtraction
// of two nearby offsets; the force pass forms r_ab, v_ab and the support-edge margin
// (h_a + h_b)^2 - r^2 in FP64 and rounds them once (their rounding in FP32 would dominate the
// terms near the edge of the support and in smooth flows); everything
// else of the pair term is FP32, summed per thread with Kahan
// compensation (its error stays within about 2u times the sum of the terms' magnitudes,
// whatever their signs); the partial sums combine in FP64 and results are stored in FP64.
#include "common.h"

// rho, P, c given by the caller (caller order) -> key-ordered thermo records
__global__ void k_thermo_from_caller(int n, const u32* __restrict__ id, const double4* __restrict__ pos4,
                                     const double* __restrict__ rho, const double* __restrict__ P,
                                     const double* __restrict__ cs, double* drho, double* dP, double* dcs,
                                     double4* thr4, float4* thrf) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const u32 i = id[q];
    const double r_ = rho[i], p_ = P[i], c_ = cs[i];
    const double pr2 = p_ / (r_ * r_);
    drho[q] = r_;
    dP[q] = p_;
    dcs[q] = c_;
    thr4[q] = make_double4(r_, pr2, c_, 0.0);
    thrf[q] = make_float4((float)r_, (float)pr2, (float)c_, (float)pos4[q].w);
}

void launch_thermo_from_caller(hipStream_t s, const DevPtrs& d, const Dims& dm, const double* rho, const double* P,
                               const double* cs) {
    if (dm.n > 0)
        hipLaunchKernelGGL(k_thermo_from_caller, dim3((dm.n + 255) / 256), dim3(256), 0, s, dm.n, d.id, d.pos4, rho, P,
                           cs, d.rho, d.P, d.cs, d.thr4, d.thrf);
}

// A thread's entries of its target's list: slots phi, phi + PL, ... of a list whose slots lie n_g entries
// apart, as byte offsets from the group's (uniform) base.
struct Entries {
    const char* base;
    u32 off, step, end, last;
    int a0, a1, a2, a3;  // the entries of the next four slots
    __device__ __forceinline__ Entries(const u16* b, int ng, int t, int phi, int PL, int cnt)
        : base(reinterpret_cast<const char*>(b)) {
        off = 2u * (u32)(phi * ng + t);
        step = 2u * (u32)(PL * ng);
        end = 2u * (u32)(cnt * ng + t);
        last = cnt > 0 ? end - 2u * (u32)ng : 2u * (u32)t;  // slot 0 of an empty list exists too
        load();
    }
    __device__ __forceinline__ int at(u32 o) const { return *reinterpret_cast<const u16*>(base + min(o, last)); }
    __device__ __forceinline__ void load() {
        a0 = at(off);
        a1 = at(off + step);
        a2 = at(off + 2 * step);
        a3 = at(off + 3 * step);
    }
    // Hands the entries below ce (those of the staged round; entries ascend) to add, in batches of four
    // that are read one batch ahead.  A batch that ends early ends the round too: the next batch's
    // entries are beyond ce as well, or INT_MAX.  The next batch is carried by the loop, or the
    // compiler sinks each load to the test that uses it.
    template <typename Add>
    __device__ __forceinline__ void round(int ce, Add&& add) {
        auto take = [&](int r) {
            if (!(off < end && r < ce)) return false;
            add(r);
            off += step;
            return true;
        };
        while (off < end && a0 < ce) {
            int b0 = INT_MAX, b1 = INT_MAX, b2 = INT_MAX, b3 = INT_MAX;
            if (off + 4 * step < end) {
                b0 = at(off + 4 * step);
                b1 = at(off + 5 * step);
                b2 = at(off + 6 * step);
                b3 = at(off + 7 * step);
            }
            add(a0);
            off += step;
            if (take(a1))
                if (take(a2)) take(a3);
            a0 = b0;
            a1 = b1;
            a2 = b2;
            a3 = b3;
        }
    }
};

// Both passes are bound by VALU issue (FP64 at 987,840 particles: 65-76% of the issue slots, the rest waits
// for list entries and at the group's ends), so the pair term is written for few instructions: density
// 145 -> 129 us (119 without DensAcc's residual), forces 279 -> 214 us with PairGeo, the byte offsets and
// batches of Entries and the force pass's one round.
//
// Geometry of one pair in FP64 from one reciprocal square root: with T = h_a + h_b = 2 h_ab,
// y = 1/(r T) gives r/T = r^2 y and 1/T^2 = (r^2 y) y, without a square root or a reciprocal of its own.
// r^2 is held above 1e-180 (a pair at the same place: r/T then vanishes beside 1 and the direction is 0).
// r^2 T^2 has to stay a normal number: T from 1.5e-64 to 1e77, more than the force terms' 1/T^5 leaves (1e-61
// to 1e61).  The density, whose 1/T^3 reaches from 1e-102 to 1e102, takes lengths in units of the
// group's own h (inv_pow2).
struct PairGeo {
    double T, s, r2, y, qh, iT2;  // s = T^2, qh = r/T = q/2, iT2 = 1/T^2
    __device__ __forceinline__ PairGeo(double dx, double dy, double dz, double ha, double hb) {
        T = ha + hb;
        s = T * T;
        r2 = fmax(fma(dx, dx, fma(dy, dy, dz * dz)), 1e-180);
        y = rsq_nr3(r2 * s);
        qh = r2 * y;
        iT2 = qh * y;
    }
};

// Density term of one pair: FP64, or FP32 on group-origin offsets with Kahan compensation.  One term is
// m_b w(r/h_ab) / h_ab^3 (1/pi applied at the end); in FP64, with x = r/T and u = 1 - x, m_b w'/T^3 with
// w' = 6 x^3 - 6 x^2 + 1 for x < 1/2, else 2 u^3, that is 1/8 of it.  1/T^3 counts the error of 1/T^2 twice, so
// the residual e of 1/T^2 corrects the product (in 1/T^2 itself the correction's rounding would be the same
// for every pair of a set with one h, and add up).  RMS error of a sum, in 1e-16, with u^3 - v^3/2 (which cancels
// for x < 1/2) and no residual / as here / from a square root and a reciprocal of their own: h spread by two
// 1.78 / 1.44 / 1.59, lattices of one h 1.52 / 1.39 / 1.54, one h and random positions 1.71 / 1.47 / 1.61.
template <bool FP32C>
struct DensAcc;
template <>
struct DensAcc<false> {
    double s = 0.0;
    __device__ __forceinline__ void add(const double4 me, const double4 b, double mb) {
        const PairGeo g(me.x - b.x, me.y - b.y, me.z - b.z, me.w, b.w);
        const double u = 1.0 - g.qh;
        const double wi = fma(g.qh * g.qh, fma(6.0, g.qh, -6.0), 1.0), wo = (u + u) * (u * u);
        const double e = fma(-g.s, g.iT2, 1.0);
        const double t3 = g.iT2 * (g.iT2 * g.T);
        s = fma(mb * (g.qh < 0.5 ? wi : wo), fma(e + e, t3, t3), s);
    }
    __device__ __forceinline__ double value() const { return 8.0 * s; }
};
template <>
struct DensAcc<true> {
    Kahan k;
    // me, b: (x, y, z offsets from the group origin, h) in FP32
    __device__ __forceinline__ void add(const float4 me, const float4 b, float mb) {
        const float dx = me.x - b.x, dy = me.y - b.y, dz = me.z - b.z;
        const float r = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
        const float ih = __builtin_amdgcn_rcpf(0.5f * (me.w + b.w));
        k.add(mb * m4_wf(r * ih) * (ih * ih * ih));
    }
    __device__ __forceinline__ double value() const { return k.value(); }
};

// FP32 offset record of a position from the group origin o: (x - o, y - o, z - o, h).
__device__ __forceinline__ float4 offset_rec(const double4 p, const double4 o) {
    return make_float4((float)(p.x - o.x), (float)(p.y - o.y), (float)(p.z - o.z), (float)p.w);
}


// An array of 32-byte records kept as two arrays of their 16-byte halves.  Read with 16-byte
// loads at random indices, records 32 bytes apart put the first half of every record in the
// same half of the LDS banks (a two-way conflict at least); at a 16-byte stride the halves of
// different records spread over all banks.
template <int N>
struct Split4 {
    double2 lo[N], hi[N];
    __device__ __forceinline__ void put(int i, const double4& v) {
        lo[i] = make_double2(v.x, v.y);
        hi[i] = make_double2(v.z, v.w);
    }
    __device__ __forceinline__ double4 get(int i) const {
        const double2 a = lo[i], b = hi[i];
        return make_double4(a.x, a.y, b.x, b.y);
    }
};

// Density sources staged in LDS: FP64 (x, y, z, h), times the group's unit k, and m, or FP32 offset records and m.
template <bool FP32C, int CH>
struct DensSrc;
template <int CH>
struct DensSrc<false, CH> {
    Split4<CH> pos;
    double mass[CH];
    using Rec = double4;
    using Mass = double;
    __device__ __forceinline__ void put(int i, const double4 p, double mb, const double4&, double k) {
        pos.put(i, target(p, p, k));
        mass[i] = mb;
    }
    __device__ __forceinline__ double4 rec(int i) const { return pos.get(i); }
    __device__ __forceinline__ static double4 target(const double4 p, const double4&, double k) {
        return make_double4(k * p.x, k * p.y, k * p.z, k * p.w);
    }
};
template <int CH>
struct DensSrc<true, CH> {
    float4 pos[CH];
    float mass[CH];
    using Rec = float4;
    using Mass = float;
    __device__ __forceinline__ void put(int i, const double4 p, double mb, const double4& o, double) {
        pos[i] = offset_rec(p, o);
        mass[i] = (float)mb;
    }
    __device__ __forceinline__ float4 rec(int i) const { return pos[i]; }
    __device__ __forceinline__ static float4 target(const double4 p, const double4& o, double) {
        return offset_rec(p, o);
    }
};
// Sets whose workgroups (256 threads, 40 KB) are resident at once.
static bool few_groups(const Dims& dm) { return dm.n <= 512 * (int64_t)dm.group_size; }
// FP64 sums over small groups take 128 threads: with 256 a thread would have three or four entries of its
// target's list, too few beside what it does once.  1.0M particles in 56 boxes, groups of 16: density 216
// -> 171 us, forces 363 -> 300 us; 123,480 of the tube 33 -> 27 and 52 -> 40 us; groups of 32 keep 256
// (density 148 and 143, forces 248 and 297 us).  Where lists may be long (by their capacity) it takes more groups
// until the chip is as full with 128 threads each: 20,011 particles in groups of 16, forces, us, 256 / 128
// threads: 39 neighbours 18 / 14, 160 25 / 35, 610 65 / 101.  The FP32C sums, whose last bits depend on the
// split, keep 256.
static bool narrow_groups(const Dims& dm) {
    return dm.group_size <= 16 && dm.n > (dm.nbr_cap > 192 ? 2048 : 512) * (int64_t)dm.group_size;
}

template <bool FP32C, int NT, int CH>
__global__ void __launch_bounds__(NT) k_density(
    const DevCtl* __restrict__ ctl, const int* __restrict__ order, const int4* __restrict__ group, int cap,
    const u16* __restrict__ nbr, const int* __restrict__ nbr_cnt, const int* __restrict__ uni,
    const int* __restrict__ ucnt,
    const double4* __restrict__ pos4, const double4* __restrict__ vel4, const double* __restrict__ m,
    const double* __restrict__ u_eos, int kin, double gamma, double h_coeff, double* __restrict__ rho,
    double* __restrict__ P, double* __restrict__ cs, double* __restrict__ hnext, double4* __restrict__ thr4,
    float4* __restrict__ thrf) {
    __shared__ DensSrc<FP32C, CH> S;  // CH union members a round
    static_assert(sizeof(S) >= NT * sizeof(double), "the reduction reuses the staging");
    const int tid = threadIdx.x;
    int g0, g1, gstep;
    group_range(ctl->n_groups, g0, g1, gstep);
    for (int ui = g0; ui < g1; ui += gstep) {
        const int gi = order ? order[ui] : ui;
        const int4 g = group[gi];
        // PL = NT / n_g threads per target, so a group with few targets still fills the
        // workgroup; thread tid serves target tid mod n_g (the last NT mod n_g threads idle)
        const int PL = NT / g.y;
        const int t = tid % g.y, phi = tid / g.y;
        const bool tv = phi < PL;
        const int q = g.x + t;
        const double4 org = pos4[g.x];  // group origin (FP32C offsets)
        const double k = FP32C ? 1.0 : inv_pow2(org.w);  // FP64: lengths in units of h (exact, a power of two)
        const double4 mp = tv ? pos4[q] : make_double4(org.x, org.y, org.z, 1);
        const typename DensSrc<FP32C, CH>::Rec me = DensSrc<FP32C, CH>::target(mp, org, k);
        const int cnt = tv ? nbr_cnt[q] : 0;
        Entries E(nbr + (size_t)g.x * cap, g.y, t, phi, PL, cnt);
        const int* un = uni + (size_t)g.x * cap;
        const int nu = ucnt[gi];
        const double mq = m[q], uq = u_eos[q];  // for the end: in flight during the sums
        DensAcc<FP32C> acc;
        for (int c0 = 0; c0 < nu; c0 += CH) {  // union members c0 .. c0 + cn - 1 through LDS
            const int cn = nu - c0 < CH ? nu - c0 : CH;
            __syncthreads();
            for (int i = tid; i < cn; i += NT) {
                const int b = un[c0 + i];
                S.put(i, pos4[b], m[b], org, k);
            }
            if (c0) E.load();
            __syncthreads();
            E.round(c0 + cn, [&](int r) { acc.add(me, S.rec(r - c0), S.mass[r - c0]); });
        }
        __syncthreads();
        double* red = reinterpret_cast<double*>(&S);
        red[tid] = acc.value();
        __syncthreads();
        if (tv && phi == 0) {
            double sum = red[t];
            for (int f = 1; f < PL; ++f) sum += red[t + g.y * f];
            const double r_ = FP32C ? sum * M_1_PI_D : fma(sum, M_1_PI_D, sum * M_1_PI_LO) * k * k * k;
            double ue = uq;
            const double4 mpos = mp;
            if (kin) {  // u_eos holds the total energy e = u + v^2/2 (thermokinetic form)
                const double4 v = vel4[q];
                ue -= 0.5 * (v.x * v.x + v.y * v.y + v.z * v.z);
            }
            const double p_ = (gamma - 1.0) * r_ * ue;
            const double c_ = sqrt(gamma * p_ / r_);
            const double pr2 = p_ / (r_ * r_);
            rho[q] = r_;
            P[q] = p_;
            cs[q] = c_;
            hnext[q] = h_coeff * cbrt(mq / r_);
            thr4[q] = make_double4(r_, pr2, c_, ue);
            thrf[q] = make_float4((float)r_, (float)pr2, (float)c_, (float)mpos.w);
        }
    }
}

void launch_density(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double gamma, double h_coeff,
                    const double* u_eos, int kin) {
    if (dm.n <= 0) return;
    auto go = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(dm.pair_grid), dim3(threads), 0, s, d.ctl, group_order(d, dm), d.group, dm.nbr_cap,
                           d.nbr, d.nbr_cnt, d.uni, d.ucnt, d.pos4, d.vel4, d.m, u_eos, kin, gamma, h_coeff, d.rho, d.P,
                           d.cs, d.hnext, d.thr4, d.thrf);
    };
    if (fp32c) go(k_density<true, 256, 512>, 256);
    else if (narrow_groups(dm)) go(k_density<false, 128, 256>, 128);
    else go(k_density<false, 256, 512>, 256);
}

// Source records in LDS for the force sums: FP64 (x, h), (v, m), (rho, P/rho^2, c), or
// FP32C (x, h) and (v, m) in FP64 and (rho, P/rho^2, c, h) in FP32.
template <bool FP32C, int CH>
struct ForceSrc;
template <int CH>
struct ForceSrc<false, CH> {
    Split4<CH> pos, vel;
    double2 rp[CH];  // rho, P/rho^2
    double c[CH];    // -(alpha/2) c
};
template <int CH>
struct ForceSrc<true, CH> {
    Split4<CH> pos, vel;  // x, y, z, h and predicted v, m in FP64: the pair's differences
    float4 thr[CH];       // and its support-edge margin are formed in FP64
};
template <bool FP32C, bool THERMO, int NT, int CH>
__global__ void __launch_bounds__(NT) k_forces(
    const DevCtl* __restrict__ ctl, const int* __restrict__ order, const int4* __restrict__ group, int cap,
    const u16* __restrict__ nbr, const int* __restrict__ nbr_cnt, const int* __restrict__ uni,
    const int* __restrict__ ucnt,
    const double4* __restrict__ pos4, const double4* __restrict__ vel4, const double4* __restrict__ thr4,
    const float4* __restrict__ thrf, double alpha, double beta, double eps_av,
    double* __restrict__ ax, double* __restrict__ ay, double* __restrict__ az, double* __restrict__ du) {
    __shared__ ForceSrc<FP32C, CH> S;  // CH union members a round
    static_assert(sizeof(S) >= 4 * NT * sizeof(double), "the reduction reuses the staging");
    const int tid = threadIdx.x;
    int g0, g1, gstep;
    group_range(ctl->n_groups, g0, g1, gstep);
    for (int ui = g0; ui < g1; ui += gstep) {
        const int gi = order ? order[ui] : ui;
        const int4 g = group[gi];
        // PL = NT / n_g threads per target, so a group with few targets still fills the
        // workgroup; thread tid serves target tid mod n_g (the last NT mod n_g threads idle)
        const int PL = NT / g.y;
        const int t = tid % g.y, phi = tid / g.y;
        const bool tv = phi < PL;
        const int q = g.x + t;
        const double4 me = tv ? pos4[q] : make_double4(0, 0, 0, 1);
        const int cnt = tv ? nbr_cnt[q] : 0;
        Entries E(nbr + (size_t)g.x * cap, g.y, t, phi, PL, cnt);
        const int* un = uni + (size_t)g.x * cap;
        const int nu = ucnt[gi];
        double fx, fy, fz, fu;
        if constexpr (!FP32C) {
            const double4 mv = tv ? vel4[q] : make_double4(0, 0, 0, 0);
            const double4 mt = tv ? thr4[q] : make_double4(1, 0, 0, 0);
            const double al2 = -0.5 * alpha, be2 = 0.5 * beta, ep4 = 0.25 * eps_av;
            const double mc = al2 * mt.z;
            double sx = 0, sy = 0, sz = 0, su = 0;
            for (int c0 = 0; c0 < nu; c0 += CH) {
                const int cn = nu - c0 < CH ? nu - c0 : CH;
                __syncthreads();
                for (int i = tid; i < cn; i += NT) {
                    const int b = un[c0 + i];
                    S.pos.put(i, pos4[b]);
                    S.vel.put(i, vel4[b]);
                    const double4 tb = thr4[b];
                    S.rp[i] = make_double2(tb.x, tb.y);
                    S.c[i] = al2 * tb.z;
                }
                if (c0) E.load();
                __syncthreads();
                E.round(c0 + cn, [&](int e) {
                    const int j = e - c0;
                    const double4 sb = S.pos.get(j);
                    const double4 vb = S.vel.get(j);
                    const double2 tb = S.rp[j];
                    const double dx = me.x - sb.x, dy = me.y - sb.y, dz = me.z - sb.z;
                    const PairGeo p(dx, dy, dz, me.w, sb.w);
                    // g(q)/h_ab^5 = -48 G/T^5: G = 2 - 3 r/T for q < 1, else u^2/(r/T) with u = 1 - r/T
                    const double u = 1.0 - p.qh;
                    const double G = p.qh < 0.5 ? fma(-3.0, p.qh, 2.0) : (u * u) * (p.s * p.y);
                    const double i2 = fma(p.iT2, fma(-p.s, p.iT2, 1.0), p.iT2);  // its third power counts
                    const double F = (vb.w * G) * ((i2 * i2) * (i2 * p.T));
                    const double wx = mv.x - vb.x, wy = mv.y - vb.y, wz = mv.z - vb.z;
                    const double vr = fma(wx, dx, fma(wy, dy, wz * dz));
                    double Pi = 0.0;
                    if (vr < 0.0) {  // one reciprocal of den (rho_a + rho_b) gives 1/den and 1/(rho_a + rho_b)
                        const double den = fma(ep4, p.s, p.r2);
                        const double rs = mt.x + tb.x;
                        const double inv = rcp_nr3(den * rs);
                        const double mu2 = (p.T * vr) * (rs * inv);  // 2 mu
                        Pi = (fma(be2, mu2, mc + S.c[j]) * mu2) * (den * inv);
                    }
                    const double c = F * ((mt.y + tb.y) + Pi);
                    sx = fma(c, dx, sx);
                    sy = fma(c, dy, sy);
                    sz = fma(c, dz, sz);
                    if (THERMO) {  // eq. (8): P_a v_b/rho_a^2 + P_b v_a/rho_b^2 + (v_a + v_b)/2 Pi
                        const double var = fma(mv.x, dx, fma(mv.y, dy, mv.z * dz));
                        const double vbr = fma(vb.x, dx, fma(vb.y, dy, vb.z * dz));
                        su = fma(F, fma(mt.y, vbr, fma(tb.y, var, 0.5 * Pi * (var + vbr))), su);
                    } else {
                        su = fma(-F * fma(0.5, Pi, mt.y), vr, su);
                    }
                });
            }
            constexpr double K = 48.0 * M_1_PI_D;
            fx = K * sx; fy = K * sy; fz = K * sz; fu = K * su;
        } else {
            const double4 mv = tv ? vel4[q] : make_double4(0, 0, 0, 0);
            const float4 mt = tv ? thrf[q] : make_float4(1, 0, 0, 1);
            const float alf = (float)alpha, bef = (float)beta, epf = (float)eps_av;
            const float ipi = (float)M_1_PI_D;
            Kahan sx, sy, sz, su;
            for (int c0 = 0; c0 < nu; c0 += CH) {
                const int cn = nu - c0 < CH ? nu - c0 : CH;
                __syncthreads();
                for (int i = tid; i < cn; i += NT) {
                    const int b = un[c0 + i];
                    S.pos.put(i, pos4[b]);
                    S.vel.put(i, vel4[b]);
                    S.thr[i] = thrf[b];
                }
                if (c0) E.load();
                __syncthreads();
                E.round(c0 + cn, [&](int e) {
                    const int j = e - c0;
                    const double4 sb = S.pos.get(j);
                    const double4 vb = S.vel.get(j);
                    const float4 tb = S.thr[j];
                    // the pair's separation, relative velocity and margin to the support edge
                    // in FP64, rounded once to FP32: D = (h_a + h_b)^2 - r^2 has no
                    // cancellation, so 2 - q = D/((T + r) h_ab) keeps FP32 relative accuracy as
                    // q -> 2 (2 - q formed from an FP32 q loses digits there), and r_ab, v_ab
                    // keep it however large the positions and velocities are against their
                    // differences; the rest of the pair term is FP32
                    const double ex = me.x - sb.x, ey = me.y - sb.y, ez = me.z - sb.z;
                    const double r2d = fma(ex, ex, fma(ey, ey, ez * ez));
                    const double Td = me.w + sb.w;
                    const float Dm = (float)fma(Td, Td, -r2d);
                    const float dx = (float)ex, dy = (float)ey, dz = (float)ez;
                    const float r2 = (float)r2d;
                    const float r = __builtin_amdgcn_sqrtf(r2);
                    const float T = (float)Td;
                    const float hab = 0.5f * T;
                    const float ih = __builtin_amdgcn_rcpf(hab);
                    const float ih2 = ih * ih;
                    const float qq = r * ih;
                    const float tq = Dm * __builtin_amdgcn_rcpf((T + r) * hab);
                    const float gq = qq < 1.0f ? fmaf(2.25f, qq, -3.0f) : -0.75f * (tq * tq) * __builtin_amdgcn_rcpf(qq);
                    const float gw = gq * (ih2 * ih2 * ih) * ipi;
                    const float wx = (float)(mv.x - vb.x), wy = (float)(mv.y - vb.y), wz = (float)(mv.z - vb.z);
                    const float vr = fmaf(wx, dx, fmaf(wy, dy, wz * dz));
                    float Pi = 0.0f;
                    if (vr < 0.0f) {
                        const float mu = hab * vr * __builtin_amdgcn_rcpf(fmaf(epf * hab, hab, r2));
                        Pi = fmaf(-alf * 0.5f * (mt.z + tb.z), mu, bef * mu * mu) *
                             __builtin_amdgcn_rcpf(0.5f * (mt.x + tb.x));
                    }
                    const float mb = (float)vb.w;
                    const float term = mb * ((mt.y + tb.y) + Pi) * gw;
                    sx.add(-term * dx);
                    sy.add(-term * dy);
                    sz.add(-term * dz);
                    if (THERMO) {  // eq. (8) takes the absolute velocities
                        const float var = fmaf((float)mv.x, dx, fmaf((float)mv.y, dy, (float)mv.z * dz));
                        const float vbr = fmaf((float)vb.x, dx, fmaf((float)vb.y, dy, (float)vb.z * dz));
                        su.add(-mb * gw * fmaf(mt.y, vbr, fmaf(tb.y, var, 0.5f * Pi * (var + vbr))));
                    } else {
                        su.add(mb * fmaf(0.5f, Pi, mt.y) * gw * vr);
                    }
                });
            }
            fx = sx.value(); fy = sy.value(); fz = sz.value(); fu = su.value();
        }
        __syncthreads();
        double* red = reinterpret_cast<double*>(&S);  // 4 NT doubles
        red[tid] = fx;
        red[NT + tid] = fy;
        red[2 * NT + tid] = fz;
        red[3 * NT + tid] = fu;
        __syncthreads();
        if (tv && phi == 0) {
            double s0 = red[t], s1 = red[NT + t], s2 = red[2 * NT + t], s3 = red[3 * NT + t];
            for (int f = 1; f < PL; ++f) {
                const int i = t + g.y * f;
                s0 += red[i];
                s1 += red[NT + i];
                s2 += red[2 * NT + i];
                s3 += red[3 * NT + i];
            }
            ax[q] = s0;
            ay[q] = s1;
            az[q] = s2;
            du[q] = s3;
        }
    }
}

void launch_forces(hipStream_t s, const DevPtrs& d, const Dims& dm, int fp32c, double alpha, double beta,
                   double eps_av, int thermo) {
    if (dm.n <= 0) return;
    auto go = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(dm.pair_grid), dim3(threads), 0, s, d.ctl, group_order(d, dm), d.group,
                           dm.nbr_cap, d.nbr, d.nbr_cnt, d.uni, d.ucnt, d.pos4, d.vel4, d.thr4, d.thrf, alpha,
                           beta, eps_av, d.ax, d.ay, d.az, d.du);
    };
    // Union members staged a round.  A wave runs each round as long as its busiest target, so a union in one
    // round wastes fewer lanes, but the records (88 bytes, 80 in FP32C) bound the workgroups a CU holds.
    // Forces alone, us, at 256 / 320 / 464 (FP32C 512): 987,840 particles in groups of 64, FP64 239 / - / 204 (214 with
    // the correction of 1/T^2); 1.2M in 64 boxes, groups of 64, FP32C 306 / 289 / 276; 1.0M in 56 boxes, groups of 32,
    // FP64 269 / 249 / 269; the same in groups of 16, FP32C 316 / 338 / 441, FP64 365 / 391 / 451 and with 128
    // threads 326 (192: 300).  Few groups take the largest: 3,375 in groups of 32, FP32C 9.0 / 8.2 / 7.2.
    auto pick = [&](auto f, auto th) {
        constexpr bool F = decltype(f)::value, TH = decltype(th)::value;
        if (dm.group_size > 32 || few_groups(dm) || (!F && dm.group_size <= 16 && !narrow_groups(dm)))
            go(k_forces<F, TH, 256, F ? 512 : 464>, 256);
        else if (dm.group_size > 16) go(k_forces<F, TH, 256, 320>, 256);
        else if constexpr (F) go(k_forces<F, TH, 256, 256>, 256);
        else go(k_forces<F, TH, 128, 192>, 128);
    };
    if (fp32c) {
        if (thermo) pick(std::true_type(), std::true_type());
        else pick(std::true_type(), std::false_type());
    } else {
        if (thermo) pick(std::false_type(), std::true_type());
        else pick(std::false_type(), std::false_type());
    }
}
