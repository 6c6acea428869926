// mc_stretch.hpp -- several fixed steps of a population in one launch (gfx950).
//
// Between two space-charge updates (or sorts, or snapshots) nothing couples
// the packs, so a launch may take each pack through all of those steps with
// its state in registers, and give it G lanes (k_stretch):
//
//  - A small population cannot fill the chip with one lane per pack (1e4
//    packs are 157 wavefronts for 1024 SIMDs), and a wavefront alone on its
//    SIMD takes some 6.5 clocks per instruction of the collision loop.  What
//    a candidate draws -- its three Philox blocks and the logarithms, roots,
//    sines and cosines of them, 390 instructions in the FP64 form -- does not
//    depend on the pack's state, so the G lanes of a pack draw G candidates
//    at once and leave the results in LDS; the part that does depend on it
//    (wait, acceptance, velocity and internal-energy update, 270
//    instructions) then runs through them in order, the same on every lane
//    of the group.
//  - A launch per step ends with its slowest wavefront (the Poisson count of
//    a step's candidates, 23 on average at 1e5 Pa, reaches 38 somewhere among
//    1e4 packs); over a stretch the counts of a wavefront's steps even out.
//  - On the Langevin branch the state of a population stays in registers
//    instead of streaming through HBM every step.
//
// Measured (per step, 32 or 64 steps, against one launch of k_step per
// step): FP64 form at 1e5 Pa, 1e3 packs 67 -> 20 us, 1e4 70 -> 31 us, 3.2e4
// 78 -> 43 us, 1e5 113 -> 88 us; at 1000 to 20 Pa, 1e4 packs 17.2 -> 6.3 us,
// 2e5 45 -> 26 us.  FP32 form at 1e5 Pa, 8e3 packs 45 -> 18 us, 3.2e4 49 ->
// 25 us, 1e5 59 -> 46 us.  Langevin branch, 1e6 packs: FP32 29 -> 20.5 us,
// FP64 112 -> 37 us.
//
// Every value is computed by the expressions of k_step (mc_kernels.hpp), in
// the same order, so the two kernels agree bit for bit; which of them a
// population takes is a matter of speed alone (lanes_for in mc_plan.hpp).
#pragma once
#include "mc_kernels.hpp"

namespace mc {

// Steps of one launch at most: their coefficients travel as kernel arguments.
constexpr int kStretchMax = 32;

// Per step of the stretch: its start, the RF coefficients of its stages and
// the slots that exist in it (a slot filled by the emission of step j takes
// part from step j on).
struct StretchSteps {
    int32_t n;
    double t0[kStretchMax], c0[kStretchMax], ch[kStretchMax], c1[kStretchMax];
    int64_t n_slots[kStretchMax];
};

template <class P, class Tab>
struct StretchArgs {
    StepArgs<P, Tab> a;
    StretchSteps st;
};

// The four nodes of the table cell a pack is in, read when the cell changes.
// (Read in every gather instead, the records of 1e6 packs spread over the
// 256x1024 grid kept the FP32 form's Langevin step at 36 us; held, 21 us.
// The FP64 form, four times the bytes per record: 97 and 37 us.)
template <class T, class Tab>
struct CellNodes {
    int32_t i = -1, j = -1;
    Tab n[4];

    __device__ __forceinline__ Q4<T> gather(const Tab *tab, const float *sc, const Cell<T> &c, int32_t nr) {
        if (c.i != i || c.j != j) {
            const int64_t k = (int64_t)c.j * nr + c.i;
            n[0] = tab[k];
            n[1] = tab[k + 1];
            n[2] = tab[k + nr];
            n[3] = tab[k + nr + 1];
            i = c.i;
            j = c.j;
        }
        Q4<T> q = interp(Nodes4<T>{load4(&n[0], 0, sc), load4(&n[1], 0, sc), load4(&n[2], 0, sc), load4(&n[3], 0, sc)},
                         c);
        if constexpr (sizeof(Tab) == sizeof(bf16x4)) {
            q.a *= sc[0];
            q.b *= sc[1];
            q.c *= sc[2];
            q.d *= sc[3];
        }
        return q;
    }
};

// Orders a wavefront's LDS accesses for the compiler (the hardware keeps a
// wavefront's LDS accesses in order).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// What one candidate draws: the wait's -ln u, the branch uniform, the
// partner's speed on the flux-weighted and on the Maxwellian branch and its
// direction, the acceptance uniform, the scattering direction and the
// logarithm of the exchange.  One column per lane.
enum { DR_WAIT, DR_BRANCH, DR_WFLUX, DR_WMAXW, DR_ST, DR_SPH, DR_CPH, DR_CT, DR_ACC, DR_CCHI, DR_SCHI, DR_SPS, DR_CPS,
       DR_LNX, DR_N };

template <class T>
struct Draws {
    T v[DR_N];
};

template <class P, class Tab>
__device__ __forceinline__ Draws<typename P::T> draw_candidate(const StepArgs<P, Tab> &a, int64_t id, uint32_t c,
                                                               uint32_t k0, uint32_t k1, typename P::T ag) {
    using T = typename P::T;
    Draws<T> d;
    const W4 wa = draw(id, a.step, kPurposeCollide, 3 * c, k0, k1);
    const W4 wb = draw(id, a.step, kPurposeCollide, 3 * c + 1, k0, k1);
    const W4 wc = draw(id, a.step, kPurposeCollide, 3 * c + 2, k0, k1);
    d.v[DR_WAIT] = -P::ln_word(wa.w0);
    d.v[DR_BRANCH] = P::u01(wa.w1);
    const T cc = P::cos2pi_word(wb.w0);
    const T la = P::ln_word(wa.w2), lb = P::ln_word(wa.w3);
    const T ef = -la - lb * (T)1, em = -la - lb * (cc * cc);
    d.v[DR_WFLUX] = ag * P::sqrt_pos((T)2 * ef);
    d.v[DR_WMAXW] = ag * P::sqrt_pos((T)2 * em);
    const T ct = P::sym_word(wb.w1);
    d.v[DR_ST] = P::sqrt_pos((T)1 - ct * ct);
    d.v[DR_CT] = ct;
    P::sc2pi_word(wb.w2, &d.v[DR_SPH], &d.v[DR_CPH]);
    d.v[DR_ACC] = P::u01(wb.w3);
    const T cchi = P::sym_word(wc.w0);
    d.v[DR_SCHI] = P::sqrt_pos((T)1 - cchi * cchi);
    d.v[DR_CCHI] = cchi;
    P::sc2pi_word(wc.w1, &d.v[DR_SPS], &d.v[DR_CPS]);
    d.v[DR_LNX] = P::ln_words(wc.w2, wc.w3);
    return d;
}

// collide_explicit with the draws shared out over the G lanes of the pack
// (a power of two, at least 2).  sub is the lane's place in its group, col
// the LDS column of the group's first lane.  te enters and leaves as the
// effective temperature of e: it changes with e only, and is refreshed as
// soon as e is known, off the chain that ends in the next wait.
template <class P, class Tab, int G>
__device__ __forceinline__ void collide_group(const StepArgs<P, Tab> &a, const Species &sp, int64_t id, uint32_t k0,
                                              uint32_t k1, const GasAt<typename P::T> &g, typename P::T ag,
                                              typename P::T abar, typename P::T sv, typename P::T lam,
                                              typename P::T &vx, typename P::T &vy, typename P::T &vz,
                                              typename P::T &e, typename P::T &el, typename P::T &te, PackCount &pc,
                                              typename P::T (*lds)[64], int sub, int col) {
    using T = typename P::T;
    const T dt = (T)a.dt, m = (T)sp.m, mg = (T)a.mg;
    const T M = m + mg, fm = P::div(mg, M), fi = P::div(m, M), mu = mg * fi;
    const T two_mu = P::div((T)2, mu);
    const T alpha = (T)sp.alpha, skt = (T)sp.skt, theta = (T)sp.theta;
    const T alpha2 = alpha * alpha;
    const T ux = g.ux, uy = g.uy, uz = g.uz, ngs = g.ngs;
    T rx = vx - ux, ry = vy - uy, rz = vz - uz;
    const T nexp = lam * dt;
    const int32_t cap = (nexp < (T)1e6) ? 64 + 8 * (int32_t)ceil(nexp) : (nexp >= (T)1e6 ? 8000064 : 0);
    T tleft = dt;
    T inv_lam = P::rcp(lam);
    bool live = true;
    for (int32_t base = 0; live; base += G) {
        {
            const Draws<T> d = draw_candidate<P, Tab>(a, id, (uint32_t)(base + sub), k0, k1, ag);
#pragma unroll
            for (int k = 0; k < DR_N; ++k) lds[k][col + sub] = d.v[k];
        }
        wave_lds_order();
#pragma unroll 1
        for (int j = 0; j < G; ++j) {
            Draws<T> d;
#pragma unroll
            for (int k = 0; k < DR_N; ++k) d.v[k] = lds[k][col + j];
            const T tau = d.v[DR_WAIT] * inv_lam;
            const bool capped = base + j == cap;
            if (capped || !(tau < tleft)) {
                if (capped) ++pc.cap;
                live = false;
                break;
            }
            tleft -= tau;
            ++pc.cand;
            const bool maxw = d.v[DR_BRANCH] * (sv + abar) < sv;
            const T wn = maxw ? d.v[DR_WMAXW] : d.v[DR_WFLUX];
            const T st = d.v[DR_ST], sph = d.v[DR_SPH], cph = d.v[DR_CPH], ct = d.v[DR_CT];
            const T wx = wn * st * cph, wy = wn * st * sph, wz = wn * ct;
            const T gx = rx - wx, gy = ry - wy, gz = rz - wz;
            const T g2 = gx * gx + gy * gy + gz * gz;
            const T lhs = d.v[DR_ACC] * (sv + wn);
            const T lhs2 = lhs * lhs;
            if (lhs2 < g2) {
                ++pc.acc;
                const T vcx = fi * vx + fm * (ux + wx), vcy = fi * vy + fm * (uy + wy), vcz = fi * vz + fm * (uz + wz);
                const T et = (T)0.5 * mu * g2;
                T etp = et;
                if (lhs2 < alpha2 * g2) {
                    ++pc.exch;
                    etp = -(T)kB * te * d.v[DR_LNX];
                    const T de = et - etp;
                    if (e + el + de < (T)0) {
                        etp = e + el + et;
                        e = 0;
                        el = 0;
                        ++pc.clamp;
                    } else {
                        acc2(e, el, de);
                    }
                    te = einstein_t<P>(e + el, skt, theta);
                }
                const T cchi = d.v[DR_CCHI], schi = d.v[DR_SCHI], sps = d.v[DR_SPS], cps = d.v[DR_CPS];
                const T f = fm * P::sqrt_(etp * two_mu);
                vx = vcx + f * schi * cps;
                vy = vcy + f * schi * sps;
                vz = vcz + f * cchi;
                rx = vx - ux;
                ry = vy - uy;
                rz = vz - uz;
                sv = P::sqrt_(rx * rx + ry * ry + rz * rz);
                lam = ngs * (sv + abar);
                inv_lam = P::rcp(lam);
            }
        }
        wave_lds_order();
    }
}

// Adaptive steps (Eq. 1) without the host: a launch takes one step of the
// length that the packs' limits allow.  Every block reduces the limits that
// the launch before left (kDtLines replica lines) and finds the same step,
//   dt = min(dt_max, limit, rf_cap, lv_cap if a pack takes the Langevin
//            branch, t_pic - t)
// (the caps are +inf where they do not apply), takes its packs through it and
// leaves their limits for the launch after; the first block writes the record.
// Records and lines change places from launch to launch: two records, three
// sets of lines (read, filled, cleared).  A step below `collapse` halts the
// run; one that would start at t_pause or later is not taken (the host's
// space-charge update comes first): then the launches that follow only hand
// the record on.  One launch instead of three (limits, their reduction, step):
// 1e5 packs 24.5 -> 15.1 us a step in the FP32 form (Langevin branch), 36.8 ->
// 22.1 in FP64; 1e6 FP64 packs 166 -> 125.  Below 1e5 packs what is
// left is the launch and the chain of loads, limits and step in each.
constexpr int kDtLines = 64;  // a lane of the reducing wavefront per line
static_assert(kDtLines <= kHotRep);
struct DtArgs {
    const unsigned long long *limits;
    unsigned long long *next, *clear;
    const DtRecord *in;
    DtRecord *out;
    double dt_max, rf_cap, lv_cap, t_pic, t_pause, collapse, v_rf, w2, phase;
    int64_t step;
};

template <class P, class Tab>
struct AdaptiveArgs {
    StretchArgs<P, Tab> s;
    DtArgs d;
};

struct DtStep {
    double t0, dt, c0, ch, c1;
    bool go;
};

// Lane l's value, in scalar registers.
__device__ __forceinline__ double from_lane(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// The step from record r whose limits' smallest is mn over the lanes (lang: some
// pack takes the Langevin branch), with the record after it.  A whole wavefront.
__device__ __forceinline__ DtStep dt_of(const DtArgs &d, const DtRecord &r, unsigned long long mn, bool lang,
                                        DtRecord &o) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    o = r;
    DtStep s{r.t, 0.0, r.c, 0.0, 0.0, false};
#pragma unroll
    for (int o2 = 32; o2 > 0; o2 >>= 1) {
        const unsigned long long other = __shfl_xor(mn, o2, 64);
        mn = other < mn ? other : mn;
    }
    double dt = fmin(d.dt_max, __longlong_as_double((long long)mn));
    dt = fmin(dt, d.rf_cap);
    if (lang) dt = fmin(dt, d.lv_cap);
    dt = fmin(dt, d.t_pic - r.t);
    if (dt > d.collapse) {
        s.go = true;
        s.dt = from_lane(dt, 0);
        const double t1 = r.t + dt;
        // both RF coefficients by one cosine: every wavefront pays for it
        const double c = d.v_rf * cos(d.w2 * (lane & 1 ? t1 : r.t + 0.5 * dt) + d.phase);
        s.ch = from_lane(c, 0);
        s.c1 = from_lane(c, 1);
        o.t = t1;
        o.c = s.c1;
        o.dt = dt;
        ++o.steps;
    } else {
        o.halted = (unsigned long long)d.step + 1ull;
    }
    return s;
}

__device__ __forceinline__ DtStep dt_step(const DtArgs &d) {
    const int lane = threadIdx.x & 63;
    const DtRecord r = *d.in;
    DtRecord o = r;
    DtStep s{r.t, 0.0, r.c, 0.0, 0.0, false};
    if (!r.halted && r.t < d.t_pause) {
        const bool lang = __ballot(d.limits[(int64_t)lane * kHotStride + 1] != 0ull) != 0ull;
        s = dt_of(d, r, d.limits[(int64_t)lane * kHotStride], lang, o);
    }
    if (blockIdx.x == 0) {
        if (lane == 0) *d.out = o;
        d.clear[(int64_t)lane * kHotStride] = kInfBits;
        d.clear[(int64_t)lane * kHotStride + 1] = 0ull;
    }
    return s;
}

// Counters of a stretch: totals over its steps, kept below 2^25 per lane
// (a step adds less than 2^23 + 64 to any of them) so that a wavefront's sum
// fits 32 bits.
__device__ __forceinline__ void flush_stretch(const TallyPtrs &t, StepCount &n) {
    const uint32_t v[HOT_N] = {n.act, n.cand, n.acc, n.cap, n.clamp, n.lang, n.exch};
    unsigned long long *rep = t.hot + (int64_t)(blockIdx.x & (kHotRep - 1)) * kHotStride;
#pragma unroll
    for (int k = 0; k < HOT_N; ++k) {
        if (__ballot(v[k] != 0u) == 0ull) continue;
        const uint32_t sum = wave_total_u32(v[k]);
        if (threadIdx.x == 0) atomicAdd(&rep[k], (unsigned long long)sum);
    }
    n = StepCount{0, 0, 0, 0, 0, 0, 0};
}

// Wavefronts per SIMD the kernel is compiled for: what its registers allow
// without spilling (FP64 form 256, FP32 form 168).  One more, with the spills
// it takes, made the small runs 3 to 15 % slower, and so did one fewer.
template <class P>
constexpr int stretch_waves() {
    return P::kTwo ? 3 : 2;
}

// One wavefront, 64 / G packs: those of place `block` of the launch.  The
// arguments are read afresh in every step, through a pointer that the compiler
// cannot see through: left to itself it keeps all of them, and what it makes
// of them, in registers across the steps (some 130 scalar registers spilled;
// 40 this way in the FP64 form and 8 in the FP32 form).
template <class P, class Tab>
using ConstArgs = const __attribute__((address_space(4))) StretchArgs<P, Tab> *;

template <class P, class Tab, int G, bool kAdaptive = false>
__device__ __forceinline__ void stretch_packs(ConstArgs<P, Tab> from, int64_t block, const DtArgs *dt = nullptr) {
    using T = typename P::T;
    __shared__ T lds[G > 1 ? DR_N : 1][64];
    const auto &args = *(const StretchArgs<P, Tab> *)from;
    DtStep now_dt{};
    if constexpr (kAdaptive) {  // (a single step)
        now_dt = dt_step(*dt);
        if (!now_dt.go) return;
    }
    const int32_t n_steps = args.st.n;
    P::prepare_tables(args.a.tables);
    const int lane = threadIdx.x & 63, sub = lane & (G - 1), col = lane & ~(G - 1);
    const int64_t s = block * (64 / G) + lane / G;
    StepCount n{0, 0, 0, 0, 0, 0, 0};
    int32_t status = -1, tag = 0;
    Motion<T> m{};
    T e = 0, el = 0, h = 0;
    int64_t id = 0;
    if (s < args.st.n_slots[n_steps - 1]) {
        const PackPtrs<T> &p = args.a.p;
        status = p.status[s];
        tag = p.tag[s];
        m.x = p.x[s];
        m.y = p.y[s];
        m.z = p.z[s];
        if constexpr (P::kTwo) {
            m.xl = p.xl[s];
            m.yl = p.yl[s];
            m.zl = p.zl[s];
            el = p.el[s];
        }
        m.vx = p.vx[s];
        m.vy = p.vy[s];
        m.vz = p.vz[s];
        e = p.e[s];
        h = p.h[s];
        id = p.id[s];
    }
    const bool mine = status == ST_ACTIVE;
    if (!mine) tag = 0;
    CellNodes<T, Tab> ecell, gcell;
    int32_t hi = -1, hj = -1;
    bool hmetal = false;
    T te = (T)0;
    if (mine) te = einstein_t<P>(e + el, (T)args.a.sp[tag].skt, (T)args.a.sp[tag].theta);
    for (int32_t j = 0; j < n_steps; ++j) {
        asm volatile("" : "+s"(from));
        const auto &now = *(const StretchArgs<P, Tab> *)from;
        StepArgs<P, Tab> a = now.a;
        const StretchSteps &st = now.st;
        const uint32_t k0 = a.k0, k1 = a.k1;
        const Species &sp = a.sp[tag];
        a.step += j;
        if constexpr (kAdaptive) {
            a.t0 = now_dt.t0;
            a.dt = now_dt.dt;
            a.c0 = now_dt.c0;
            a.ch = now_dt.ch;
            a.c1 = now_dt.c1;
        } else {
            a.t0 = st.t0[j];
            a.c0 = st.c0[j];
            a.ch = st.ch[j];
            a.c1 = st.c1[j];
        }
        if (status == ST_ACTIVE && s < st.n_slots[j]) {
            PackCount pc{0, 0, 0, 0, 0, 0};
            const double X0 = (double)m.x + (double)m.xl, Y0 = (double)m.y + (double)m.yl,
                         Zo = (double)m.z + (double)m.zl;
            push_rk4(a, [&](const Cell<T> &c) { return ecell.gather(a.etab, a.esc, c, a.nr); }, (T)sp.qm, m);
            const double X1 = (double)m.x + (double)m.xl, Y1 = (double)m.y + (double)m.yl,
                         Z1 = (double)m.z + (double)m.zl;
            double r1;
            {
#pragma clang fp contract(off)
                r1 = sqrt(X1 * X1 + Y1 * Y1);
            }
            GasAt<T> g{};
            if (a.collisions_on)
                g = gas_at(a, sp, [&](const Cell<T> &c) { return gcell.gather(a.gtab, a.gsc, c, a.nr); }, (T)r1, m.x, m.y,
                           m.z);
            // terminal classification, as in step_one
            int32_t cls = ST_ACTIVE, in = -1, jn = -1;
            double tcross = 0.0, rcross = 0.0;
            {
#pragma clang fp contract(off)
                const bool finite = isfinite(X1) && isfinite(Y1) && isfinite(Z1) && isfinite((double)m.vx) &&
                                    isfinite((double)m.vy) && isfinite((double)m.vz);
                if (!finite) {
                    cls = ST_NUMERIC;
                } else if (Z1 >= a.z_det || Z1 < 0.0) {
                    const double zp = Z1 >= a.z_det ? a.z_det : 0.0;
                    const double fr = (Z1 != Zo) ? (zp - Zo) / (Z1 - Zo) : 1.0;
                    const double xc = X0 + fr * (X1 - X0), yc = Y0 + fr * (Y1 - Y0);
                    rcross = sqrt(xc * xc + yc * yc);
                    tcross = a.t0 + fr * a.dt;
                    cls = (Z1 >= a.z_det && rcross <= a.r_det) ? ST_TRANSMITTED : ST_AXIAL;
                } else if (r1 > a.R) {
                    cls = ST_RADIAL;
                } else {
                    const int32_t ii = (int32_t)floor(r1 * a.inv_dr + 0.5), jj = (int32_t)floor(Z1 * a.inv_dz + 0.5);
                    if (ii != hi || jj != hj) {
                        hmetal = ii < a.nr && jj < a.nz && a.hit[(int64_t)jj * a.nr + ii];
                        hi = ii;
                        hj = jj;
                    }
                    if (hmetal) {
                        cls = ST_ELECTRODE;
                        in = ii;
                        jn = jj;
                    }
                }
            }
            bool lang = false;
            if (cls == ST_ACTIVE && a.collisions_on && g.gas) {
                const T ag = P::sqrt_(P::div((T)kB * g.tg, (T)a.mg));
                const T abar = ag * (T)1.5957691216057308;  // sqrt(8/pi)
                const T rx = m.vx - g.ux, ry = m.vy - g.uy, rz = m.vz - g.uz;
                const T sv = P::sqrt_(rx * rx + ry * ry + rz * rz);
                const T lam = g.ngs * (sv + abar);
                lang = takes_langevin(a, Z1, lam);
                if (lang) {
                    langevin_relax(a, sp, id, k0, k1, g, m.vx, m.vy, m.vz);
                    ++pc.lang;
                } else if constexpr (G > 1) {
                    collide_group<P, Tab, G>(a, sp, id, k0, k1, g, ag, abar, sv, lam, m.vx, m.vy, m.vz, e, el, te, pc,
                                             lds, sub, col);
                } else {
                    collide_explicit(a, sp, id, k0, k1, g, ag, abar, sv, lam, m.vx, m.vy, m.vz, e, el, pc);
                    if (pc.exch) te = einstein_t<P>(e + el, (T)sp.skt, (T)sp.theta);
                }
            }
            if (cls == ST_ACTIVE) {
                if (!lang) h = h + rate<P>(sp.act_kind, (T)sp.act_a, (T)sp.act_b, te) * (T)a.dt;
            } else {
                if (sub == 0)
                    record_exit(a, s, cls, in, jn, X1, Y1, Z1, (double)m.vx, (double)m.vy, (double)m.vz, tcross, rcross,
                                (double)e + (double)el, (double)h, sp);
                status = cls;
            }
            if (sub == 0) {
                ++n.act;
                n.cand += pc.cand;
                n.acc += pc.acc;
                n.cap += pc.cap;
                n.clamp += pc.clamp;
                n.lang += pc.lang;
                n.exch += pc.exch;
            }
        }
        if (__ballot(n.cand >> 24) != 0ull) flush_stretch(a.t, n);
        if constexpr (kAdaptive) {  // the limits of the step after this one
            double lim = HUGE_VAL;
            bool lang = false;
            if (status == ST_ACTIVE)
                lim = pack_limit(
                    a, sp, [&](const Cell<T> &c) { return ecell.gather(a.etab, a.esc, c, a.nr); },
                    [&](const Cell<T> &c) { return gcell.gather(a.gtab, a.gsc, c, a.nr); }, m.x, m.y, m.z,
                    (double)m.z + (double)m.zl, m.vx, m.vy, m.vz, a.c1, lang);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) lim = fmin(lim, __shfl_xor(lim, o, 64));
            const bool any = __ballot(lang) != 0ull;
            if (lane == 0) {
                unsigned long long *line = dt->next + (int64_t)(blockIdx.x & (kDtLines - 1)) * kHotStride;
                if (lim < HUGE_VAL) atomicMin(line, (unsigned long long)__double_as_longlong(lim));
                if (any) atomicOr(line + 1, 1ull);
            }
        }
    }
    const StepArgs<P, Tab> &a = ((const StretchArgs<P, Tab> *)from)->a;
    if (mine && sub == 0) {
        const PackPtrs<T> &p = a.p;
        p.x[s] = m.x;
        p.y[s] = m.y;
        p.z[s] = m.z;
        if constexpr (P::kTwo) {
            p.xl[s] = m.xl;
            p.yl[s] = m.yl;
            p.zl[s] = m.zl;
            p.el[s] = el;
        }
        p.vx[s] = m.vx;
        p.vy[s] = m.vy;
        p.vz[s] = m.vz;
        p.e[s] = e;
        p.h[s] = h;
        if (status != ST_ACTIVE) p.status[s] = status;
    }
    flush_stretch(a.t, n);
}

template <class P, class Tab, int G>
__global__ __launch_bounds__(64, (stretch_waves<P>())) void k_stretch(StretchArgs<P, Tab> args) {
    stretch_packs<P, Tab, G>((ConstArgs<P, Tab>)__builtin_amdgcn_kernarg_segment_ptr(),
                             args.a.from_last ? gridDim.x - 1 - blockIdx.x : blockIdx.x);
}

// Its FP64 form: a single step of the stretch kernel, one pack a lane (an
// adaptive step draws 0.1 candidates a pack), whose limits come from the state
// and the cell in registers.
template <class P, class Tab>
__global__ __launch_bounds__(64, (stretch_waves<P>())) void k_stretch_adaptive(AdaptiveArgs<P, Tab> args) {
    stretch_packs<P, Tab, 1, true>((ConstArgs<P, Tab>)__builtin_amdgcn_kernarg_segment_ptr(),
                                   args.s.a.from_last ? gridDim.x - 1 - blockIdx.x : blockIdx.x, &args.d);
}

// Its FP32 form: the step by k_step's code, which leaves five wavefronts a SIMD
// where the stretch kernel's leaves three, the limits from the state just
// written; one wavefront of a block looks for the step.  Us a step at 3e4 /
// 1e5 / 3e5 / 1e6 packs: FP32 11.5 / 14.1 / 22.8 / 56.1 here, 14.1 / 15.1 /
// 26.9 / 65.8 the other way; FP64 20.4 / 28.9 / 57.7 / 157 against 17.2 /
// 22.1 / 47.8 / 125.
template <class P, class Tab, bool kOneSpecies>
__global__ __launch_bounds__(256, (step_waves<P, Tab>())) void k_step_adaptive(StepArgs<P, Tab> a, DtArgs d) {
    __shared__ DtStep found;
    if (threadIdx.x < 64) {
        const DtStep s = dt_step(d);
        if (threadIdx.x == 0) found = s;
    }
    __syncthreads();
    if (!found.go) return;
    a.t0 = from_lane(found.t0, 0);
    a.dt = from_lane(found.dt, 0);
    a.c0 = from_lane(found.c0, 0);
    a.ch = from_lane(found.ch, 0);
    a.c1 = from_lane(found.c1, 0);
    P::prepare_tables(a.tables);
    StepCount n{0, 0, 0, 0, 0, 0, 0};
    const unsigned block = !kOneSpecies && a.from_last ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    const int64_t s = (int64_t)block * blockDim.x + threadIdx.x;
    step_one<P, Tab, kOneSpecies>(a, s, n, a.k0, a.k1);
    flush_counts(a.t, n);
    block_limits(a, s, a.c1, d.next, kDtLines);
}

// Other adaptive steps take three launches: the packs' limits, the step from
// them and from the record (d.in, or null for a batch's first step, whose record
// r the host holds; the lines are left cleared), the step's kernel.
//
// Batches of up to kAdaptiveShort steps, which are too short for the limits that
// every launch leaves and the last one leaves to none: 2e5 FP32 packs took 51 us
// a call of one step that way and 1.4e4 FP64 packs 44, so 46 and 41.
//
// The FP32 form above kAdaptivePacks32 packs, where the look for the step at the
// start of every block, in each round of blocks, costs more than the launches:
// 1e6 packs spread over 0.3 mm 51.5 us a step so against 54.0 in one launch, on
// the Langevin branch 53.7 against 54.8.  (Three launches with a pass of their
// own for the reduction took 4e5 packs 35 to 38 us, one launch 28.)
constexpr int64_t kAdaptiveShort = 2;
constexpr int64_t kAdaptivePacks32 = 800'000;

static __global__ __launch_bounds__(64) void k_dt_single(DtArgs d, DtRecord r, unsigned long long *lines,
                                                         DtStep *found) {
    const int lane = threadIdx.x & 63;
    if (d.in) r = *d.in;
    unsigned long long *line = lines + (int64_t)lane * kHotStride;
    const unsigned long long mn = line[0];
    const bool lang = __ballot(line[1] != 0ull) != 0ull;
    line[0] = kInfBits;
    line[1] = 0ull;
    DtRecord o = r;
    DtStep s{r.t, 0.0, r.c, 0.0, 0.0, false};
    if (!r.halted && r.t < d.t_pause) s = dt_of(d, r, mn, lang, o);
    if (lane == 0) {
        *found = s;
        *d.out = o;
    }
}

// (Not held to five wavefronts as k_step is: with that the kernel of several
// species took 1e6 packs 41.8 us, without 38.7.)
template <class P, class Tab, bool kOneSpecies>
__global__ __launch_bounds__(256, (step_waves<P, Tab>())) void k_step_found(StepArgs<P, Tab> a, const DtStep *found) {
    if (!found->go) return;
    a.t0 = found->t0;
    a.dt = found->dt;
    a.c0 = found->c0;
    a.ch = found->ch;
    a.c1 = found->c1;
    P::prepare_tables(a.tables);
    StepCount n{0, 0, 0, 0, 0, 0, 0};
    const unsigned block = !kOneSpecies && a.from_last ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    step_one<P, Tab, kOneSpecies>(a, (int64_t)block * blockDim.x + threadIdx.x, n, a.k0, a.k1);
    flush_counts(a.t, n);
}

// The resident queries of a server, each over its own steps; each block
// belongs to one query (descriptors in device memory).
template <class P, class Tab, int G>
__global__ __launch_bounds__(64, (stretch_waves<P>())) void k_stretch_multi(const StretchArgs<P, Tab> *descs,
                                                                            const int32_t *prefix, int32_t nq) {
    const int q = __builtin_amdgcn_readfirstlane(block_query(prefix, nq));
    stretch_packs<P, Tab, G>((ConstArgs<P, Tab>)(uintptr_t)(descs + q), (int64_t)blockIdx.x - prefix[q]);
}

// Emission of one source over the steps of a stretch in one launch: step j
// emits the packs [first[j], first[j + 1]) of this launch into the slots from
// slot0[j] on.
struct EmitSteps {
    int32_t n;
    int64_t first[kStretchMax + 1], slot0[kStretchMax];
};

// Pack k of the launch.
template <class P, class Tab>
__device__ __forceinline__ void emit_in_stretch(EmitArgs<P, Tab> a, const EmitSteps &st, int64_t k) {
    if (k >= st.first[st.n]) return;
    int32_t j = 0;
    while (k >= st.first[j + 1]) ++j;
    // the pack's place in its step's emission
    a.step += j;
    a.slot0 = st.slot0[j] - st.first[j];
    emit_one(a, k);
}

template <class P, class Tab>
__global__ __launch_bounds__(256) void k_emit_stretch(EmitArgs<P, Tab> a, EmitSteps st) {
    emit_in_stretch(a, st, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// The sources of a server's queries.
template <class P, class Tab>
struct EmitStretchArgs {
    EmitArgs<P, Tab> a;
    EmitSteps st;
};

template <class P, class Tab>
__global__ __launch_bounds__(256) void k_emit_stretch_multi(const EmitStretchArgs<P, Tab> *descs,
                                                            const int32_t *prefix, int32_t nq) {
    const int q = block_query(prefix, nq);
    emit_in_stretch(descs[q].a, descs[q].st, (int64_t)(blockIdx.x - prefix[q]) * blockDim.x + threadIdx.x);
}

}  // namespace mc
