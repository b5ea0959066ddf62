// Collisions and sampling of the DSMC step for gfx950 (paper section 2.1:
// pair selection and collisions in each cell; eq. dsmc_temperatures for the
// sums), with the launch wrapper that picks the kernel's instance.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "slots.h"

namespace dsmcx {

// ---------------------------------------------------------------------------
// collisions and sampling
// ---------------------------------------------------------------------------
// A workgroup of four waves (one where the cells are sparse) works on some
// consecutive cells (64; 16 on a small mesh or of dense cells) whose particles
// it stages in LDS (see k_collide_sample).

// Velocities (and rotational energies) of a window of cells, staged in LDS
// in slot order and written back as a whole (deferred sort: a changed value
// goes to the particle store at once, the window's particles lying apart).  A
// particle is named by 3 x its slot (the element of its velocity, so that no
// access multiplies); ord: logical (pid) position -> that, from a cell's
// first slot.
template <class VT, bool IND>
struct Staged {
    typedef VT value;
    typedef uint16_t handle;
    VT* lv;               // [slots][3]
    double* li;           // [slots]
    const uint16_t* ord;
    const uint32_t* idx;  // slot -> particle (deferred sort, as the rest)
    VT* v;                // particle store
    double* ir;
    __device__ __forceinline__ int at(int s0, int k) const { return ord[s0 + k]; }
    static __device__ __forceinline__ int slot(int h) { return (int)(((uint32_t)h * 43691u) >> 17); }  // h / 3
    __device__ __forceinline__ VT get(int h, int comp) const { return lv[h + comp]; }
    __device__ __forceinline__ void put(int h, VT x, VT y, VT z) const {
        lv[h] = x;
        lv[h + 1] = y;
        lv[h + 2] = z;
        if (IND) {
            VT* g = v + 3 * (int64_t)idx[slot(h)];
            g[0] = x;
            g[1] = y;
            g[2] = z;
        }
    }
    __device__ __forceinline__ double getI(int h) const { return li[slot(h)]; }
    __device__ __forceinline__ void putI(int h, double e) const {
        const int l = slot(h);
        li[l] = e;
        if (IND) ir[idx[l]] = e;
    }
};

// The same for a cell that exceeds the LDS stage: the particle store itself
// through a global order table (particles named by their index).
template <class VT>
struct Stored {
    typedef VT value;
    typedef int32_t handle;
    VT* v;
    const int32_t* perm;
    double* ir;
    __device__ __forceinline__ int at(int, int k) const { return perm[k]; }
    __device__ __forceinline__ VT get(int l, int comp) const { return v[3 * (int64_t)l + comp]; }
    __device__ __forceinline__ void put(int l, VT x, VT y, VT z) const {
        VT* g = v + 3 * (int64_t)l;
        g[0] = x;
        g[1] = y;
        g[2] = z;
    }
    __device__ __forceinline__ double getI(int l) const { return ir[l]; }
    __device__ __forceinline__ void putI(int l, double e) const { ir[l] = e; }
};

// Particles from which a cell's ids are ranked by all lanes of the workgroup
// instead of the few that are the cell's.  These make a pass over the N ids per
// 48 or 64 of them, the workgroup one per 1,024, but cell after cell, up to
// some 3,000 ids a window: as much as N^2 / 64 at this N.  Six FP32 cells of
// 2,000 particles: 3.7 ms a step against 27.1 with their own lanes alone, of
// 1,000 1.13 against 4.18, of 500 0.46 against 0.87; of 400 0.34 either way.
constexpr int kRankAll = 448;

// r[t] += o < p[t] for four ids.  Written out because a compare's lane mask
// may not be read by the next two instructions: interleaved by four, none of
// the slots in between is idle (compiled from the plain form, half are).
__device__ __forceinline__ void rank4(uint32_t o, const uint32_t* p, int* r) {
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_lt_u32_e64 %[m0], %[o], %[p0]\n\t"
        "v_cmp_lt_u32_e64 %[m1], %[o], %[p1]\n\t"
        "v_cmp_lt_u32_e64 %[m2], %[o], %[p2]\n\t"
        "v_cmp_lt_u32_e64 %[m3], %[o], %[p3]\n\t"
        "v_addc_co_u32_e64 %[r0], %[m0], 0, %[r0], %[m0]\n\t"
        "v_addc_co_u32_e64 %[r1], %[m1], 0, %[r1], %[m1]\n\t"
        "v_addc_co_u32_e64 %[r2], %[m2], 0, %[r2], %[m2]\n\t"
        "v_addc_co_u32_e64 %[r3], %[m3], 0, %[r3], %[m3]"
        : [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3), [r0] "+&v"(r[0]), [r1] "+&v"(r[1]),
          [r2] "+&v"(r[2]), [r3] "+&v"(r[3])
        : [o] "v"(o), [p0] "v"(p[0]), [p1] "v"(p[1]), [p2] "v"(p[2]), [p3] "v"(p[3]));
}

// What the candidate pairs of a round need besides the velocities: it
// depends on the generator alone, so it is computed one candidate per lane,
// the candidates of all the cells packed together.
template <int CC, int S, bool VSS, bool ROT, class H>
struct PairSlots {
    static constexpr int kCells = CC, kSlots = S;
    typedef H handle;
    // VHS: cos(theta), sin(theta) cos(eps), sin(theta) sin(eps); VSS:
    // cos(chi), sin(chi), cos(eps), sin(eps); then, rotating gas, the
    // translational shares of the two partners (-1: no exchange)
    static constexpr int kDir = VSS ? 4 : 3;
    static constexpr int kVals = kDir + (ROT ? 2 : 0);
    double U[S];
    double val[kVals][S];
    H pi[S], pj[S];                          // the partners
    int32_t first[CC];                       // first slot of each cell
    int32_t base[CC];                        // candidate index of slot 0, per cell
    int total;
};

// Per-cell values that the candidate lanes read.
template <int CC>
struct CellTable {
    int N[CC], s0[CC];
    uint32_t subj[CC], k0[CC], k1[CC];
};

// Slot s of a round: partners, acceptance deviate, and the scattering of two
// uniform deviates R1 (deflection) and R2 (azimuth eps = 2 pi R2).  VHS:
// isotropic, cos(theta) = 2 R1 - 1 measured from the x axis.  VSS (section
// 2.1, the model of Bird 1994): cos(chi) = 2 R1^(1/alpha) - 1 from the
// relative velocity.
template <bool VSS, bool ROT, class Acc, class Slots, class Table>
__device__ __forceinline__ void pair_draw(const Acc& cv, Slots& ps, int s, const CollideParams& cp, const Table& tab,
                                          uint32_t step) {
    // the slot's cell: the last whose first slot is at most s
    int o = 0;
#pragma unroll
    for (int x = Slots::kCells / 2; x > 0; x >>= 1)
        if (ps.first[o + x] <= s) o += x;
    const RngKey key{tab.k0[o], tab.k1[o]};
    const uint32_t subj = tab.subj[o];
    const int N = tab.N[o], s0 = tab.s0[o];
    const uint64_t k = (uint64_t)(ps.base[o] + s);
    const Rand4 w = draw(key, subj, step, kPurposePair, k);
    const uint32_t i = pick(w.w[0], (uint32_t)N);
    uint32_t j = pick(w.w[1], (uint32_t)(N - 1));
    if (j >= i) ++j;
    ps.pi[s] = (typename Acc::handle)cv.at(s0, (int)i);
    ps.pj[s] = (typename Acc::handle)cv.at(s0, (int)j);
    ps.U[s] = u01(w.w[2], w.w[3]);
    const Rand4 q = draw(key, subj, step, kPurposeScatter, k);
    const double R1 = u01(q.w[0], q.w[1]), R2 = u01(q.w[2], q.w[3]);
    const double eps = DSMC_TWO_PI * R2;
    double se, ce;
    sincos(eps, &se, &ce);
    if constexpr (VSS) {
        const double cc = 2.0 * pow(R1, cp.inv_alpha) - 1.0;
        ps.val[0][s] = cc;
        ps.val[1][s] = sqrt(1.0 - cc * cc);
        ps.val[2][s] = ce;
        ps.val[3][s] = se;
    } else {
        const double cx = 2.0 * R1 - 1.0;
        const double sx = sqrt(1.0 - cx * cx);
        ps.val[0][s] = cx;
        ps.val[1][s] = sx * ce;
        ps.val[2][s] = sx * se;
    }
    if constexpr (ROT) {
        constexpr int d = VSS ? 4 : 3;  // the translational shares follow the scattering
        // one copy of the power for both partners
#pragma unroll 1
        for (int x = 0; x < 2; ++x) {
            const Rand4 r = draw(key, subj, step, x ? kPurposeInelasticJ : kPurposeInelasticI, k);
            ps.val[d + x][s] = u01(r.w[0], r.w[1]) < cp.pinel ? pow(u01(r.w[2], r.w[3]), cp.ex_bl) : -1.0;
        }
    }
}

// Post-collision relative velocity g' (|g'| = cr) from slot s.  VSS: g' =
// cos(chi) g + sin(chi) c_r (cos(eps) e1 + sin(eps) e2) in the frame e1 =
// (0, g_z, -g_y) / g_yz, e2 = (g_yz^2, -g_x g_y, -g_x g_z) / (c_r g_yz),
// g_yz = |(g_y, g_z)|; with g along x (g_yz = 0) e1 and e2 are the y and z
// axes.
template <bool VSS, class Slots>
__device__ __forceinline__ void scatter(const Slots& ps, int s, double gx, double gy, double gz,
                                        double cr, double& o0, double& o1, double& o2) {
    if constexpr (!VSS) {
        o0 = cr * ps.val[0][s];
        o1 = cr * ps.val[1][s];
        o2 = cr * ps.val[2][s];
    } else {
        const double cc = ps.val[0][s], sc = ps.val[1][s], ce = ps.val[2][s], se = ps.val[3][s];
        const double gyz = sqrt(gy * gy + gz * gz);
        double e10 = 0.0, e11 = 1.0, e12 = 0.0, e20 = 0.0, e21 = 0.0, e22 = 1.0;
        if (gyz > 0.0) {
            e11 = gz / gyz;
            e12 = -gy / gyz;
            e20 = gyz / cr;
            e21 = -(gx * gy) / (cr * gyz);
            e22 = -(gx * gz) / (cr * gyz);
        }
        const double scr = sc * cr;
        o0 = cc * gx + scr * (se * e20 + ce * e10);
        o1 = cc * gy + scr * (se * e21 + ce * e11);
        o2 = cc * gz + scr * (se * e22 + ce * e12);
    }
}

// The m candidates of the lane's cell in slots base ..., in order:
// acceptance against (sigma c)_max and the velocity update.  (sigma
// c)/(sigma c)_max = K cr2^ex / sm is first estimated in FP32 (hardware
// log2/exp2, relative error of about 1e-5); when the estimate is below 1 and
// U lies outside it by a relative margin of 1e-4 each, both the acceptance
// and the (sigma c)_max update (only values above sm matter) are decided
// without the FP64 power (taken by a wave when any of its lanes needs it), and
// decided as the FP64 expression would.  The next candidate's velocities are
// read before this one is decided, and replaced by this one's results where
// they are the same particles, so that the reads are not in the chain.
template <bool VSS, bool ROT, class Acc, class Slots>
__device__ __forceinline__ void ntc_round(const Acc& cv, const Slots& ps, int base, int m, const CollideParams& cp,
                                          double sm, float lk, double& seen, int& acc) {
    typedef typename Acc::value VT;
    if (m <= 0) return;
    const float ex32 = (float)cp.ex;
    const int last = base + m - 1;
    int i = ps.pi[base], j = ps.pj[base];
    int in = ps.pi[min(base + 1, last)], jn = ps.pj[min(base + 1, last)];
    double U = ps.U[base];
    VT a[3], b[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        a[x] = cv.get(i, x);
        b[x] = cv.get(j, x);
    }
    for (int s = base; s <= last; ++s) {
        const int sn = min(s + 1, last), sn2 = min(s + 2, last);
        VT na[3], nb[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            na[x] = cv.get(in, x);
            nb[x] = cv.get(jn, x);
        }
        const double Un = ps.U[sn];
        const int in2 = ps.pi[sn2], jn2 = ps.pj[sn2];
        const double a0 = (double)a[0], a1 = (double)a[1], a2 = (double)a[2];
        const double b0 = (double)b[0], b1 = (double)b[1], b2 = (double)b[2];
        const double gx = a0 - b0, gy = a1 - b1, gz = a2 - b2;
        const double cr2 = gx * gx + gy * gy + gz * gz;
        const float c2f = (float)cr2, Uf = (float)U;
        const float est = __builtin_amdgcn_exp2f(fmaf(ex32, __builtin_amdgcn_logf(c2f), lk));
        bool take = Uf < est;
        // (the hardware logarithm takes a subnormal argument as zero)
        if (!(est < 0.9999f && fabsf(Uf - est) > 1e-4f * est && c2f > 1e-30f)) {
            const double sc = cp.K * pow(cr2, cp.ex);
            if (sc > seen) seen = sc;
            take = U < sc / sm;
        }
        // the results are formed for refused pairs too (some lane of the wave
        // takes its pair nearly always), so that their chain runs beside the
        // decision's
        double hx = gx, hy = gy, hz = gz, cn2 = cr2;
        if constexpr (ROT) {
            // Borgnakke-Larsen, partner by partner: with probability pinel
            // the partner's rotational energy and the relative translational
            // energy E_t = m c_r^2 / 4 are pooled and the translation keeps
            // E_c R^(1/(5/2 - omega)) (two rotational degrees of freedom);
            // the relative velocity keeps its direction and takes the new
            // speed
            constexpr int d = VSS ? 4 : 3;  // the translational shares follow the scattering
            const double fi = ps.val[d][s], fj = ps.val[d + 1][s];
            if (take && (fi >= 0.0 || fj >= 0.0)) {
                double Et = (0.25 * cp.mass) * cr2;
                double Ii = cv.getI(i), Ij = cv.getI(j);
                if (fi >= 0.0) {
                    const double Ec = Et + Ii;
                    Et = Ec * fi;
                    Ii = Ec - Et;
                }
                if (fj >= 0.0) {
                    const double Ec = Et + Ij;
                    Et = Ec * fj;
                    Ij = Ec - Et;
                }
                cv.putI(i, Ii);
                cv.putI(j, Ij);
                cn2 = (4.0 * Et) / cp.mass;
                const double f = sqrt(cn2 / cr2);
                hx = gx * f;
                hy = gy * f;
                hz = gz * f;
            }
        }
        double g0, g1, g2;
        scatter<VSS>(ps, s, hx, hy, hz, sqrt(cn2), g0, g1, g2);
        const double cm0 = 0.5 * (a0 + b0), cm1 = 0.5 * (a1 + b1), cm2 = 0.5 * (a2 + b2);
        const double h0 = 0.5 * g0, h1 = 0.5 * g1, h2 = 0.5 * g2;
        const VT w[3] = {(VT)(cm0 + h0), (VT)(cm1 + h1), (VT)(cm2 + h2)};
        const VT z[3] = {(VT)(cm0 - h0), (VT)(cm1 - h1), (VT)(cm2 - h2)};
        if (take) {
            ++acc;
            cv.put(i, w[0], w[1], w[2]);
            cv.put(j, z[0], z[1], z[2]);
        }
        const bool ai = take && in == i, aj = take && in == j, bi = take && jn == i, bj = take && jn == j;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            na[x] = ai ? w[x] : aj ? z[x] : na[x];
            nb[x] = bi ? w[x] : bj ? z[x] : nb[x];
        }
        i = in;
        j = jn;
        in = in2;
        jn = jn2;
        U = Un;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            a[x] = na[x];
            b[x] = nb[x];
        }
    }
}

// The sums of a cell are shared out over the workgroup's waves, one lane per
// cell in each: wave 0 takes S3, wave 1 the diagonal S2, wave 2 the
// off-diagonal S2, wave 3 S1, the particle count S0 and (rotating gas) sum
// I_r and sum v_i I_r (a workgroup of one wave takes the four shares one after
// another).  Rows of the accumulators: g ... g + 2.
__device__ __forceinline__ int sum_rows(int wave) { return wave == 0 ? 10 : wave == 1 ? 4 : wave == 2 ? 7 : 1; }

// Old values of the accumulators that this lane updates, requested ahead of
// the collisions.
template <bool ROT>
struct CellSums {
    double s[3], e[3], s0, e0;
    double r[ROT ? 4 : 1], f[ROT ? 4 : 1];
    int m, local;
};

template <bool ROT>
__device__ __forceinline__ void load_sums(CellSums<ROT>& a, int c, int wave, const CollideParams& cp, bool steady) {
    const int64_t nt = cp.nt;
    const int64_t g = sum_rows(wave) * nt + c;
    if (steady) {
#pragma unroll
        for (int x = 0; x < 3; ++x) a.s[x] = cp.acc[g + x * nt];
        if (wave == 3) {
            a.s0 = cp.acc[c];
            if constexpr (ROT)
                for (int x = 0; x < 4; ++x) a.r[x] = cp.racc[x * nt + c];
        }
    }
    if (cp.ewma_on) {
        a.m = cp.ewma_m[c];
        a.local = cp.local_acc[c];
#pragma unroll
        for (int x = 0; x < 3; ++x) a.e[x] = cp.ewma[g + x * nt];
        if (wave == 3) {
            a.e0 = cp.ewma[c];
            if constexpr (ROT)
                for (int x = 0; x < 4; ++x) a.f[x] = cp.rewma[x * nt + c];
        }
    }
}

// Moment sums of the lane's cell, each sum over the particles in logical
// order, added to the accumulators.
template <bool ROT, class Acc>
__device__ __forceinline__ void sample_cell(const Acc& cv, int s0, int N, int c, int wave, const CollideParams& cp,
                                            bool steady, const CellSums<ROT>& a) {
    double t[3] = {0.0, 0.0, 0.0}, r[4] = {0.0, 0.0, 0.0, 0.0};
    // one loop per wave's sums (the wave index is uniform)
#define DSMC_SAMPLE_LOOP(BODY)                                                                     \
    _Pragma("unroll 4") for (int k = 0; k < N; ++k) {                                              \
        const int l = cv.at(s0, k);                                                                \
        const double vx = (double)cv.get(l, 0), vy = (double)cv.get(l, 1), vz = (double)cv.get(l, 2); \
        BODY                                                                                       \
    }
    if (wave == 0) {
        DSMC_SAMPLE_LOOP(const double v2 = vx * vx + vy * vy + vz * vz;
                         t[0] += vx * v2; t[1] += vy * v2; t[2] += vz * v2;)
    } else if (wave == 1) {
        DSMC_SAMPLE_LOOP(t[0] += vx * vx; t[1] += vy * vy; t[2] += vz * vz;)
    } else if (wave == 2) {
        DSMC_SAMPLE_LOOP(t[0] += vx * vy; t[1] += vx * vz; t[2] += vy * vz;)
    } else if constexpr (ROT) {
        // rotational sums: sum I_r, sum v_i I_r (rotational temperature and
        // heat flux of eq. dsmc_temperatures)
        DSMC_SAMPLE_LOOP(const double I = cv.getI(l);
                         t[0] += vx; t[1] += vy; t[2] += vz;
                         r[0] += I; r[1] += vx * I; r[2] += vy * I; r[3] += vz * I;)
    } else {
        DSMC_SAMPLE_LOOP(t[0] += vx; t[1] += vy; t[2] += vz;)
    }
#undef DSMC_SAMPLE_LOOP
    const int64_t nt = cp.nt;
    const int64_t g = sum_rows(wave) * nt + c;
    const double n1 = (double)N;
    if (cp.inst) {
#pragma unroll
        for (int x = 0; x < 3; ++x) cp.inst[g + x * nt] = t[x];
        if (wave == 3) cp.inst[c] = n1;
    }
    if (steady) {
#pragma unroll
        for (int x = 0; x < 3; ++x) cp.acc[g + x * nt] = a.s[x] + t[x];
        if (wave == 3) cp.acc[c] = a.s0 + n1;
    }
    double wo = 0.0, wn = 0.0;
    if (cp.ewma_on) {
        const int m = a.m + 1;
        const int n = (a.local || m < cp.n_a) ? m : cp.n_a;
        wo = (double)(n - 1) / (double)n;
        wn = 1.0 / (double)n;
#pragma unroll
        for (int x = 0; x < 3; ++x) cp.ewma[g + x * nt] = wo * a.e[x] + wn * t[x];
        if (wave == 3) {
            cp.ewma[c] = wo * a.e0 + wn * n1;
            cp.ewma_m[c] = m;
        }
    }
    if constexpr (ROT) {
        if (wave == 3) {
            for (int x = 0; x < 4; ++x) {
                if (cp.rinst) cp.rinst[x * nt + c] = r[x];
                if (steady) cp.racc[x * nt + c] = a.r[x] + r[x];
                if (cp.ewma_on) cp.rewma[x * nt + c] = wo * a.f[x] + wn * r[x];
            }
        }
    }
}

// What the collisions of a cell read besides its particles.
struct CellInfo {
    double sm, vol, FN, dt;
    RngKey key;
    uint32_t subj;
};

__device__ __forceinline__ void load_info(CellInfo& f, int c, const CollideParams& cp) {
    f.sm = cp.smax[c];
    f.vol = cp.vol[c];
    f.subj = (uint32_t)cp.orig[c];
    f.key = cp.key;
    f.FN = cp.FN;
    f.dt = cp.dt;
    if (cp.cell_case) {
        const CaseDev& cs = cp.cases[cp.cell_case[c]];
        f.key.k0 = cs.k0;
        f.key.k1 = cs.k1;
        f.FN = cs.FN;
        f.dt = cs.dt;
        f.subj -= (uint32_t)cs.cell0;
    }
}

// Collisions of the cells of a window (lane l of every wave: cell l, `live`
// when it is one of them, its N particles in cv from s0), then their sums.
// Candidate pairs are taken in rounds of at most a lane each: drawn one per
// lane by all waves, then decided and applied cell by cell, one cell per
// lane, by wave 0.
template <bool VSS, bool ROT, class Acc, class Slots, class Table>
__device__ __forceinline__ void collide_cells(const Acc& cv, bool live, int s0, int N, int c, int wave, Slots& ps,
                                              Table& tab, const CollideParams& cp, uint32_t step, int do_collide,
                                              int do_sample, const CellInfo& f, const CellSums<ROT>& sums) {
    const int lane = threadIdx.x & 63;
    if (do_collide) {
        int M = 0, acc = 0, left = 0;
        double seen = 0.0;
        float lk = 0.f;
        if (wave == 0) {
            if (live && N >= 2) {
                const Rand4 r = draw(f.key, f.subj, step, kPurposeNtcCount, 0);
                const double Nd = (double)N;
                const double mean = ((((0.5 * Nd) * (Nd - 1.0)) * f.FN) * f.sm) * f.dt / f.vol;
                M = (int)floor(mean + u01(r.w[0], r.w[1]));
                lk = log2f((float)cp.K) - log2f((float)f.sm);
                tab.N[lane] = N;
                tab.s0[lane] = s0;
                tab.subj[lane] = f.subj;
                tab.k0[lane] = f.key.k0;
                tab.k1[lane] = f.key.k1;
            }
            left = M > 0 ? M : 0;
        }
#pragma unroll 1
        for (int kb = 0;;) {
            int m = 0, base = 0;
            if (wave == 0) {
                int total;
                m = share_slots<Slots::kSlots>(left, &base, &total);
                if (lane < Slots::kCells) {
                    ps.first[lane] = base;
                    ps.base[lane] = kb - base;
                }
                if (lane == 0) ps.total = total;
            }
            __syncthreads();
            const int total = ps.total;
            if (total == 0) break;
            if ((int)threadIdx.x < total) pair_draw<VSS, ROT>(cv, ps, (int)threadIdx.x, cp, tab, step);
            __syncthreads();
            if (wave == 0) {
                ntc_round<VSS, ROT>(cv, ps, base, m, cp, f.sm, lk, seen, acc);
                left -= m;
                kb += m;
            }
        }
        if (live && wave == 0) {
            if (seen > f.sm) cp.smax[c] = seen;
            cp.ncand[c] = M;
            cp.nacc[c] = acc;
        }
    }
    const bool steady = (int64_t)step > (int64_t)cp.n_ss;
    if constexpr (Slots::kSlots > 64) {
        if (do_sample && live) sample_cell<ROT>(cv, s0, N, c, wave, cp, steady, sums);
    } else if (do_sample && live) {
        // one wave: the four shares of the sums one after another
        CellSums<ROT> a[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) load_sums<ROT>(a[x], c, x, cp, steady);
#pragma unroll
        for (int x = 0; x < 4; ++x) sample_cell<ROT>(cv, s0, N, c, x, cp, steady, a[x]);
    }
}

// Particles that fit when `wg` workgroups of L lanes share a CU's LDS: 128 units
// of 1,280 bytes (gfx950 hands it out in these; a workgroup a few bytes over a
// third of it leaves room for two only).
template <class VT, int CC, int L, bool IND, bool VSS, bool ROT>
constexpr int stage_cap(int wg) {
    // the ids share the candidate slots' memory, or have it to themselves
    // where they need more
    const int slots = (int)sizeof(PairSlots<CC, L, VSS, ROT, uint16_t>);
    const int room = (128 / wg) * 1280 - (int)sizeof(CellTable<CC>) - 4 * (CC + 1) - 64;
    const int per = 3 * (int)sizeof(VT) + 2 + (IND ? 4 : 0) + (ROT ? 8 : 0);
    const int cap = (room - slots) / per;
    return (4 * cap <= slots ? cap : std::max(slots / 4, room / (per + 4))) & ~31;
}

// A workgroup of L lanes works on CC consecutive cells.  Per window of them whose
// particles fit the stage (one window as a rule) the particles' ids and
// velocities (rotational energies) are staged in LDS with one round of
// coalesced loads, and four lanes a cell (16 in workgroups of 16 cells, all of
// them where the cell is large) rank its ids; then the candidate pairs, the
// collisions and the sums (collide_cells).  A single cell beyond the stage
// works on the particle store through a global order table.
// With FUSED, the cells' slots of the sorted buffer p are filled from the
// unsorted buffer src through the gather permutation (slot -> source index):
// velocities and ids go through the stage, the rest passes through once the
// window has been worked on, while other workgroups compute.  With IND
// (deferred sort) nothing is moved: slot d of the sorted order is particle
// sortperm[d] of p.
// On the 40^3 cavity (11.52M particles, Kn 0.1) FUSED takes 461 us, against 367
// for a gather of its own and 281 for this kernel without (and 35 more in the
// permutation, which then writes the cells).  Bound: its 2.2 GB of HBM traffic
// at 4.7 TB/s (a copy reaches 5.2) and, beside it, the waits for the one
// deciding wave.  Without the gather it moves 408 MB, and VALU issue (16,200
// wave instructions per 64 cells: a quarter the ranking, a quarter the
// candidates' draws, a fifth each the decisions and the sums; 159 us at full
// issue) takes 54 % of its time, those waits the rest.  One wave per 64 cells
// that drew, decided and summed cell by cell, a lane each, at 47-63 % lane
// efficiency and two waves per SIMD, took 360 us; nitrogen on 73,000 cells 133
// against 209 us.
// (For sparse cells there are workgroups of one wave here too: L = 64.)
template <class VT, int CC, int L, int WG, int GM, bool VSS, bool ROT>
__global__ __launch_bounds__(L) __attribute__((amdgpu_waves_per_eu(WG * L / 256))) void k_collide_sample(
    PartDev<VT> p, const int32_t* offsets, CollideParams cp, const Scalars* sc, int32_t* perm, int do_collide,
    int do_sample, PartDev<VT> src, const int32_t* sortperm) {
    constexpr bool FUSED = GM == kGatherFused;
    constexpr bool IND = GM == kGatherIndirect;
    constexpr int CAP = stage_cap<VT, CC, L, IND, VSS, ROT>(WG);
    constexpr int kStageBatch = L == 64 ? 4 : 8;  // particles per lane loaded together
    // also the candidate slots of a cell beyond the stage, whose candidates
    // name particles by 32-bit index
    typedef PairSlots<CC, L, VSS, ROT, int32_t> StoredSlots;
    constexpr int kStage = std::max(3 * CAP, (int)(sizeof(StoredSlots) / sizeof(VT)) + 1);
    __shared__ __attribute__((aligned(16))) VT lv[kStage];
    __shared__ double li[ROT ? CAP : 1];
    __shared__ uint16_t ord[CAP];
    __shared__ uint32_t idx[IND ? CAP : 1];
    // the ids are read before the candidate slots are written
    __shared__ union {
        PairSlots<CC, L, VSS, ROT, uint16_t> ps;
        uint32_t ids[CAP];
    } u;
    __shared__ CellTable<CC> tab;
    __shared__ int32_t soff[CC + 1];
    const int nt = cp.nt;
    const int tid = threadIdx.x, lane = tid & 63;
    // the wave that takes part 0 below works while the others wait: not the
    // same SIMD's in each workgroup of a CU
    const int wave = L == 64 ? 0 : __builtin_amdgcn_readfirstlane(((tid >> 6) + (blockIdx.x >> 8)) & 3);
    // Workgroups go round-robin over the 8 XCDs: eight consecutive ones of an
    // XCD take eight consecutive pieces of the cells, so that its L2 holds the
    // source lines that neighbouring cells' gathers share (40^3 cavity: 1.52 GB
    // fetched against 2.15, 2.5 % less time; one slice per XCD 3 % more, and
    // 132 us against 107 on a mesh whose busy cells lie together).  gridDim.x is a
    // multiple of 64; the last workgroups may be past the last cell.
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    const int c0 = ((seq >> 3) * 64 + xcd * 8 + (seq & 7)) * CC;
    if (c0 >= cp.nt) return;
    const int c = c0 + lane;
    const int64_t a = offsets[c0];
    for (int i = tid; i <= CC; i += L) soff[i] = offsets[min(c0 + i, nt)] - (int32_t)a;
    const uint32_t step = sc->step;
    // requested ahead of their use after the ranking
    CellInfo f{};
    CellSums<ROT> sums{};
    if (lane < CC && c < nt) {
        if (wave == 0) load_info(f, c, cp);
        if (L > 64 && do_sample) load_sums<ROT>(sums, c, wave, cp, (int64_t)step > (int64_t)cp.n_ss);
    }
    __syncthreads();
#pragma unroll 1
    for (int k0 = 0; k0 < CC;) {
        // the cells from k0 on that fit the stage together (lane l looks at
        // cell l; offsets do not fall, so the fitting ones are consecutive)
        const int w0 = soff[k0];
        const int lo = soff[min(lane, CC - 1)], hi = soff[min(lane, CC - 1) + 1];
        const int k1 = k0 + __popcll(__ballot(lane >= k0 && lane < CC && hi - w0 <= CAP));
        uint64_t large = __ballot(lane >= k0 && lane < k1 && hi - lo > kRankAll);
        const int64_t base = a + w0;
        if (k1 == k0) {
            // one cell beyond the stage: its order by comparison of all ids
            const int N = soff[k0 + 1] - w0;
            if (FUSED) {
                for (int k = tid; k < N; k += L) {
                    const int64_t d = base + k, j = sortperm[d];
                    for (int q = 0; q < 3; ++q) {
                        p.pos[3 * d + q] = src.pos[3 * j + q];
                        p.vel[3 * d + q] = src.vel[3 * j + q];
                    }
                    p.pid[d] = src.pid[j];
                    p.cell[d] = c0 + k0;
                    if (ROT) p.ir[d] = src.ir[j];
                }
                __syncthreads();
            }
            for (int k = tid; k < N; k += L) {
                const int32_t l = IND ? sortperm[base + k] : (int32_t)(base + k);
                const uint32_t pk = p.pid[l];
                int r = 0;
                for (int x = 0; x < N; ++x) r += p.pid[IND ? (int64_t)sortperm[base + x] : base + x] < pk ? 1 : 0;
                perm[base + r] = l;
            }
            __syncthreads();
            const Stored<VT> cv{p.vel, perm + base, p.ir};
            collide_cells<VSS, ROT>(cv, lane == k0 && c < nt, 0, N, c, wave, *(StoredSlots*)lv, tab, cp, step,
                                    do_collide, do_sample, f, sums);
            ++k0;
            __syncthreads();
            continue;
        }
        const int wn = soff[k1] - w0;
        for (int i0 = tid; i0 < wn; i0 += kStageBatch * L) {
            // kStageBatch particles per lane in flight
            int64_t x[kStageBatch];
            uint32_t id[kStageBatch];
            VT v[kStageBatch][3];
            double I[kStageBatch];
#pragma unroll
            for (int b = 0; b < kStageBatch; ++b) {
                // past the window: its last particle again (no branch around a load)
                x[b] = base + min(i0 + b * L, wn - 1);
                if (IND || FUSED) x[b] = sortperm[x[b]];
            }
            const PartDev<VT>& from = FUSED ? src : p;
#pragma unroll
            for (int b = 0; b < kStageBatch; ++b) {
                id[b] = from.pid[x[b]];
                v[b][0] = from.vel[3 * x[b]];
                v[b][1] = from.vel[3 * x[b] + 1];
                v[b][2] = from.vel[3 * x[b] + 2];
                if (ROT) I[b] = from.ir[x[b]];
            }
#pragma unroll
            for (int b = 0; b < kStageBatch; ++b) {
                const int i = i0 + b * L;
                if (i < wn) {
                    u.ids[i] = id[b];
                    lv[3 * i] = v[b][0];
                    lv[3 * i + 1] = v[b][1];
                    lv[3 * i + 2] = v[b][2];
                    if (ROT) li[i] = I[b];
                    if (IND) idx[i] = (uint32_t)x[b];
                    if (FUSED) p.pid[base + i] = id[b];
                }
            }
        }
        __syncthreads();
        {
            // logical order: lane q of a cell's `lanes` ranks the ids q, q +
            // lanes, ..., `batch` of them against one pass over the cell
            auto rank = [&](int lc, int N, int q, auto lanes, auto batch) {
                constexpr int G = decltype(lanes)::value, B = decltype(batch)::value;
                const int s0 = soff[lc] - w0;
                for (int b0 = q; b0 < N; b0 += G * B) {
                    uint32_t pk[B];
                    int r[B];
#pragma unroll
                    for (int t = 0; t < B; ++t) {
                        const int x = b0 + G * t;
                        pk[t] = x < N ? u.ids[s0 + x] : 0u;
                        r[t] = s0;
                    }
#pragma unroll 4
                    for (int x = 0; x < N; ++x) {
                        const uint32_t o = u.ids[s0 + x];
#pragma unroll
                        for (int t = 0; t < B; t += 4) rank4(o, pk + t, r + t);
                    }
#pragma unroll
                    for (int t = 0; t < B; ++t) {
                        const int x = b0 + G * t;
                        if (x < N) {
                            ord[r[t]] = (uint16_t)(3 * (s0 + x));
                            if (FUSED) p.cell[base + s0 + x] = c0 + lc;
                        }
                    }
                }
            };
            constexpr int kLanes = L / CC, kBatch = kLanes <= 4 ? 12 : kLanes == 8 ? 8 : 4;
            const int lc = tid / kLanes;
            const int N = lc >= k0 && lc < k1 ? soff[lc + 1] - soff[lc] : 0;
            rank(lc, N <= kRankAll ? N : 0, tid & (kLanes - 1), std::integral_constant<int, kLanes>{},
                 std::integral_constant<int, kBatch>{});
            // the large cells by all lanes, one after another
            for (; large; large &= large - 1) {
                const int k = __builtin_ctzll(large);
                rank(k, soff[k + 1] - soff[k], tid, std::integral_constant<int, L>{},
                     std::integral_constant<int, 4>{});
            }
        }
        __syncthreads();
        const bool live = lane >= k0 && lane < k1 && c < nt;
        const int s0 = live ? soff[lane] - w0 : 0;
        const int N = live ? soff[lane + 1] - soff[lane] : 0;
        const Staged<VT, IND> cv{lv, li, ord, idx, p.vel, p.ir};
        collide_cells<VSS, ROT>(cv, live, s0, N, c, wave, u.ps, tab, cp, step, do_collide, do_sample, f, sums);
        if (FUSED || (!IND && do_collide)) {
            // whole lines: written where they changed, 12 bytes here and
            // there, the same velocities took the memory several times as long
            for (int i = tid; i < 3 * wn; i += L) p.vel[3 * base + i] = lv[i];
            if (ROT)
                for (int i = tid; i < wn; i += L) p.ir[base + i] = li[i];
        }
        if (FUSED) {
            // positions only pass through (next read by the following step's move)
            for (int i0 = tid; i0 < wn; i0 += kStageBatch * L) {
                double x[kStageBatch][3];
#pragma unroll
                for (int b = 0; b < kStageBatch; ++b) {
                    const int64_t j = sortperm[base + min(i0 + b * L, wn - 1)];
                    x[b][0] = src.pos[3 * j];
                    x[b][1] = src.pos[3 * j + 1];
                    x[b][2] = src.pos[3 * j + 2];
                }
#pragma unroll
                for (int b = 0; b < kStageBatch; ++b) {
                    const int i = i0 + b * L;
                    if (i < wn) {
                        double* d = p.pos + 3 * (base + i);
                        __builtin_nontemporal_store(x[b][0], d);
                        __builtin_nontemporal_store(x[b][1], d + 1);
                        __builtin_nontemporal_store(x[b][2], d + 2);
                    }
                }
            }
        }
        k0 = k1;
        __syncthreads();  // the stage is filled again
    }
}

// Particles that the instance with wg workgroups per CU stages at once.
template <class VT, int CC, int L, bool VSS, bool ROT>
static int collide_cap(int wg, int gmode) {
    return gmode == kGatherIndirect ? stage_cap<VT, CC, L, true, VSS, ROT>(wg)
                                    : stage_cap<VT, CC, L, false, VSS, ROT>(wg);
}

bool collide_fuses_gather(int variant) { return variant != kCollideApart3; }

template <class VT, int CC, int L, int WG, bool VSS, bool ROT>
static void launch_collide_g(hipStream_t s, PartDev<VT> p, const int32_t* offsets, const CollideParams& cp,
                             const Scalars* sc, int32_t* perm, int do_collide, int do_sample, int gmode,
                             PartDev<VT> src, const int32_t* sortperm) {
    const dim3 gr(((cp.nt + CC - 1) / CC + 63) / 64 * 64), bl(L);
    if (gmode == kGatherIndirect) {
        hipLaunchKernelGGL((k_collide_sample<VT, CC, L, WG, kGatherIndirect, VSS, ROT>), gr, bl, 0, s, p, offsets, cp,
                           sc, perm, do_collide, do_sample, src, sortperm);
        return;
    }
    if (gmode == kGatherFused) {
        hipLaunchKernelGGL((k_collide_sample<VT, CC, L, WG, kGatherFused, VSS, ROT>), gr, bl, 0, s, p, offsets, cp, sc,
                           perm, do_collide, do_sample, src, sortperm);
        return;
    }
    hipLaunchKernelGGL((k_collide_sample<VT, CC, L, WG, kGatherNone, VSS, ROT>), gr, bl, 0, s, p, offsets, cp, sc, perm,
                       do_collide, do_sample, src, sortperm);
}

template <class VT, bool VSS, bool ROT>
static void launch_collide_v(hipStream_t s, PartDev<VT> p, const int32_t* offsets, const CollideParams& cp,
                             const Scalars* sc, int32_t* perm, int do_collide, int do_sample, int variant, int gmode,
                             PartDev<VT> src, const int32_t* sortperm, int64_t np, int64_t bound) {
    const int64_t need = np * 64 * 12 / (11 * (int64_t)std::max(cp.nt, 1));
    // Cells per workgroup: 64, a lane of the deciding wave each, keep that
    // wave full; where they would give the device's 256 CUs fewer than two
    // workgroups each, 16 (1,296 cells, FP64: 20.0 against 24.5 us; 24,500
    // cells, VSS: 104 against 130 us; but 73,000 cells of nitrogen 194
    // against 133 us, 384,000 of argon 707 against 281 us).  Also 16 where 64
    // cells' particles exceed even three of the largest stage: in windows of a few
    // cells most lanes of the deciding waves idle, and three of these waves a
    // CU decide more than two (35,000 cells, a step: FP32 250 particles a cell
    // 1.77 against 2.70 ms, 450 5.2 against 10.3; FP64 450 7.4 against 16.9;
    // 162,000 cells, FP64, 125 a cell 3.49 against 3.84).  Below, some meshes
    // gain and some lose (nitrogen, FP64: 162,000 cells of 80 2.47 against 2.33;
    // 83,000 of 15 and 165 at random, without the move, 1.72 against 1.53).
    if ((variant == kCollideAuto && cp.nt <= 64 * 512) || need > 3 * collide_cap<VT, 64, 256, VSS, ROT>(2, gmode)) {
        launch_collide_g<VT, 16, 256, 3, VSS, ROT>(s, p, offsets, cp, sc, perm, do_collide, do_sample, gmode, src,
                                                   sortperm);
        return;
    }
    // Few particles a cell on many cells: the phases of a workgroup are a serial
    // chain whatever it holds, and eight one-wave workgroups a CU have more of
    // them under way than three or four of four waves (384,000 cells, us a step,
    // FP32 / FP64 / FP64 nitrogen: one particle a cell 143 / 145 / 159 against
    // 175 / 182 / 274, six 356 / 374 against 387 / 396 and nitrogen beyond the
    // stage; 83,000 cells of six 122 / 124 against 124 / 126, of nine 146 / 147
    // against 143 / 145; 35,000 cells of four 82 against 76).  Twelve a CU have
    // registers spilled (216 for the nitrogen).
    // The particles are counted by their upper bound: an inflow can fill the mesh
    // before the count is next seen, or in replays of a graph captured now.
    if (variant == kCollideAuto && cp.nt >= 64 * 1024 && bound <= 6 * (int64_t)cp.nt &&
        bound * 64 * 12 / (11 * (int64_t)cp.nt) <= collide_cap<VT, 64, 64, VSS, ROT>(8, gmode)) {
        launch_collide_g<VT, 64, 64, 8, VSS, ROT>(s, p, offsets, cp, sc, perm, do_collide, do_sample, gmode, src,
                                                  sortperm);
        return;
    }
    // Workgroups per CU: the most for which the stage holds a workgroup's
    // particles at the mean occupancy and an eleventh more (a workgroup with
    // more takes its cells in several windows): the waves wait at barriers
    // for a good half of their time, so more of them are worth more than
    // spare room (11.52M particles, 384,000 cells: 281 us with four, 318 with
    // three, 415 with two).  The schedules other than the default fix it.
    // FP64 velocities or rotational energies: three at most (four stages would
    // hold a dozen particles a cell, and the registers of four spill: 384,000
    // cells of 12 FP64 particles 659 us a step against 624).
    constexpr int kMost = sizeof(VT) == 4 && !ROT ? 4 : 3;
    int wg = 2;
    if (variant == kCollideWg3 || variant == kCollideApart3) wg = 3;
    else if (variant == kCollideWg4) wg = kMost;
    else if (variant != kCollideWg2)
        while (wg < kMost && need <= collide_cap<VT, 64, 256, VSS, ROT>(wg + 1, gmode)) ++wg;
    if constexpr (kMost == 4) {
        if (wg == 4) {
            launch_collide_g<VT, 64, 256, 4, VSS, ROT>(s, p, offsets, cp, sc, perm, do_collide, do_sample, gmode, src,
                                                  sortperm);
            return;
        }
    }
    if (wg == 3)
        launch_collide_g<VT, 64, 256, 3, VSS, ROT>(s, p, offsets, cp, sc, perm, do_collide, do_sample, gmode, src,
                                                   sortperm);
    else
        launch_collide_g<VT, 64, 256, 2, VSS, ROT>(s, p, offsets, cp, sc, perm, do_collide, do_sample, gmode, src,
                                                   sortperm);
}

template <class VT>
void launch_collide_sample(hipStream_t s, PartDev<VT> p, const int32_t* offsets, const CollideParams& cp,
                           const Scalars* sc, int32_t* perm, int do_collide, int do_sample, int variant, int gmode,
                           PartDev<VT> src, const int32_t* sortperm, int64_t np, int64_t bound) {
    if (cp.rot) {
        if (cp.vss)
            launch_collide_v<VT, true, true>(s, p, offsets, cp, sc, perm, do_collide, do_sample, variant, gmode, src,
                                             sortperm, np, bound);
        else
            launch_collide_v<VT, false, true>(s, p, offsets, cp, sc, perm, do_collide, do_sample, variant, gmode, src,
                                              sortperm, np, bound);
    } else if (cp.vss) {
        launch_collide_v<VT, true, false>(s, p, offsets, cp, sc, perm, do_collide, do_sample, variant, gmode, src,
                                          sortperm, np, bound);
    } else {
        launch_collide_v<VT, false, false>(s, p, offsets, cp, sc, perm, do_collide, do_sample, variant, gmode, src,
                                           sortperm, np, bound);
    }
}

#define INSTANTIATE(VT)                                                                                      \
    template void launch_collide_sample<VT>(hipStream_t, PartDev<VT>, const int32_t*, const CollideParams&, \
                                            const Scalars*, int32_t*, int, int, int, int, PartDev<VT>,      \
                                            const int32_t*, int64_t, int64_t);

INSTANTIATE(float)
INSTANTIATE(double)

}  // namespace dsmcx
