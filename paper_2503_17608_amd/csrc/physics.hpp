// Device physics of the electromagnetic step loop: table interpolation,
// process cross sections, final-state samplers and annihilation at rest.
//
// The paper (arXiv 2503.17608) states only that the transport covers EM
// processes of photons, electrons and positrons.  The models used are named
// textbook forms: Klein-Nishina Compton with Butcher-Messel sampling, Born
// K-shell photoelectric (x 5/4), complete-screening Bethe-Heitler pair
// production, Moller and Bhabha delta rays above the cut, Tsai complete-
// screening bremsstrahlung above the cut, restricted continuous loss through
// a range table, annihilation at rest into two back-to-back photons.
//
// Template parameter R is the precision of energies, directions, cross
// sections and tables (double, or float in the mixed mode); positions and
// path lengths are always double.
#pragma once
#include "common.hpp"

namespace ems {

template <class R>
struct Tables {
    const R* v;        // [n_mat][8][181]
    R ln_e0;
    R inv_dlog;
    R dlog;
    __device__ __forceinline__ const R* tab(int mat, int which) const
    {
        return v + (mat * kTabPerMat + which) * kNodes;
    }
};

// interpolation location of energy T on the log grid
template <class R>
struct Loc {
    int i;
    R f;
};

template <class R>
__device__ __forceinline__ Loc<R> locate(const Tables<R>& tb, R T)
{
    const R x = m_log(T) - tb.ln_e0;
    R t = x * tb.inv_dlog;
    R fl = m_floor(t);
    int i = (int)fl;
    if (fl < R(0)) i = 0;
    if (fl > R(kNodes - 2)) i = kNodes - 2;
    Loc<R> l;
    l.i = i;
    // written as the fused operation, which the compiler makes of t - i where
    // it sees both, so that every use gets the same bits
    l.f = m_fma(x, tb.inv_dlog, -R(i));
    return l;
}

template <class R>
__device__ __forceinline__ R interp(const R* v, const Loc<R>& l)
{
    R a = v[l.i], b = v[l.i + 1];
    return a + l.f * (b - a);
}

// processes of each particle, in selection order
__device__ __forceinline__ int n_proc(int type) { return type == kGamma ? 3 : 2; }
__device__ __forceinline__ int proc_of(int type, int n)
{
    if (type == kGamma) return n;                       // Compton, photoelectric, pair
    if (type == kElectron) return n == 0 ? P_MOLLER : P_BREMS;
    return n == 0 ? P_BHABHA : P_BREMS;
}

// Macroscopic cross sections of a particle's processes at T, in selection
// order, zero at and below their thresholds.  Every table is read whatever
// the thresholds say, so that the loads are in flight together.
template <class R>
struct ProcXs {
    R x[3];       // [2]: photons only
};

template <class R>
__device__ __forceinline__ ProcXs<R> proc_xs(const Tables<R>& tb, int mat, int typ, R T, const Loc<R>& l, R ecut)
{
    ProcXs<R> s;
    if (typ == kGamma) {
        s.x[0] = interp(tb.tab(mat, TB_COMPTON), l);
        s.x[1] = interp(tb.tab(mat, TB_PHOTO), l);
        const R pair = interp(tb.tab(mat, TB_PAIR), l);
        s.x[2] = T <= R(2.0 * kMe) ? R(0) : pair;
    } else {
        const bool ele = typ == kElectron;
        const R delta = interp(tb.tab(mat, ele ? TB_MOLLER : TB_BHABHA), l);
        const R brems = interp(tb.tab(mat, TB_BREMS), l);
        s.x[0] = T <= (ele ? R(2) * ecut : ecut) ? R(0) : delta;
        s.x[1] = T <= ecut ? R(0) : brems;
        s.x[2] = R(0);
    }
    return s;
}

template <class R>
__device__ __forceinline__ R total_xs(const ProcXs<R>& s, int typ)
{
    const R two = s.x[0] + s.x[1];
    return typ == kGamma ? two + s.x[2] : two;
}

template <class R>
__device__ __forceinline__ const R* range_tab(const Tables<R>& tb, int mat, int type)
{
    return tb.tab(mat, type == kPositron ? TB_RANGE_EP : TB_RANGE_EM);
}

// Exact inverse of the piecewise-linear range map: the interval is the one an
// upper-bound search on the node ranges finds (first node with R > r, minus
// one); ln T is linear in R inside it.  The search starts at interval i0 of
// the pre-step energy; a step loses at most a fifth of the range (below the
// final range more), so the interval is i0 or one of the two below, whose
// nodes are read together; else it walks on from i0 node by node.
template <class R>
__device__ __forceinline__ R inverse_range(const Tables<R>& tb, const R* Rt, R r, int i0)
{
    const R r1 = Rt[i0 + 1], r0 = Rt[i0], rm = Rt[i0 > 0 ? i0 - 1 : 0], rn = Rt[i0 > 1 ? i0 - 2 : 0];
    int i = i0;
    R lo = r0, hi = r1;
    if (!(r1 > r) || (r0 > r && !(i0 > 0 && !(rm > r)) && !(i0 > 1 && !(rn > r)))) {
        int j = i0 + 1;
        while (j < kNodes && !(Rt[j] > r)) ++j;
        while (j > 0 && Rt[j - 1] > r) --j;
        i = j - 1;
        if (i < 0) i = 0;
        if (i > kNodes - 2) i = kNodes - 2;
        lo = Rt[i];
        hi = Rt[i + 1];
    } else if (r0 > r) {
        const bool one = !(rm > r);
        i = one ? i0 - 1 : i0 - 2;
        lo = one ? rm : rn;
        hi = one ? r0 : rm;
    }
    R t = R(i) + (r - lo) / (hi - lo);
    return m_exp(tb.ln_e0 + t * tb.dlog);
}

// rotate direction u by polar cosine c and azimuth phi (phi given as sin/cos)
template <class R>
__device__ __forceinline__ void rotate(const R u[3], R c, R sp, R cp, R out[3])
{
    if (c > R(1)) c = R(1);
    if (c < R(-1)) c = R(-1);
    R s = m_sqrt(R(1) - c * c);
    R a = m_sqrt(R(1) - u[2] * u[2]);
    if (a > R(1.0e-10)) {
        out[0] = u[0] * c + s * (u[0] * u[2] * cp - u[1] * sp) / a;
        out[1] = u[1] * c + s * (u[1] * u[2] * cp + u[0] * sp) / a;
        out[2] = u[2] * c - a * s * cp;
    } else {
        out[0] = s * cp;
        out[1] = s * sp;
        out[2] = (u[2] >= R(0) ? R(1) : R(-1)) * c;
    }
}

template <class R>
__device__ __forceinline__ void normalize3(R v[3])
{
    R n = m_sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    v[0] /= n; v[1] /= n; v[2] /= n;
}

// up to three secondaries produced by one track step, kept in registers
// (fixed slots, selected with compile-time indices after unrolling)
template <class R>
struct Sec {
    R T;
    R ux, uy, uz;       // scalars, not an array: the buffer must stay in registers
    uint64_t key;
    int type;
};

template <class R>
struct SecBuf {
    int n;
    Sec<R> s0, s1, s2;
    // every field of every slot is written through a value select: branches
    // or whole-struct copies chosen at run time would be merged into stores
    // through a selected pointer, which puts the buffer on the stack
    __device__ __forceinline__ static void put(Sec<R>& s, bool here, int t, R e, const R d[3], uint64_t k)
    {
        s.T = here ? e : s.T;
        s.ux = here ? d[0] : s.ux;
        s.uy = here ? d[1] : s.uy;
        s.uz = here ? d[2] : s.uz;
        s.key = here ? k : s.key;
        s.type = here ? t : s.type;
    }
    __device__ __forceinline__ void add(int t, R e, const R d[3], uint64_t k)
    {
        put(s0, n == 0, t, e, d, k);
        put(s1, n == 1, t, e, d, k);
        put(s2, n >= 2, t, e, d, k);
        ++n;
    }
    // Visit the stored secondaries in order, by name (no run-time index, so
    // the buffer stays in registers): f(secondary, ordinal).
    template <class F>
    __device__ __forceinline__ void each(F&& f) const
    {
        if (n > 0) f(s0, 0);
        if (n > 1) f(s1, 1);
        if (n > 2) f(s2, 2);
    }
};

// per-step tallies of one track
struct StepTally {
    double edep;
    int n_pair, n_annih, capped;
};

struct PhysParams {
    uint64_t seed;
    uint64_t event;    // Philox key word 1 of the track's event
    double ecut;
};

// annihilation at rest of a positron with key `key` in step `step`: two
// photons of m c^2, back to back, isotropic (Philox domain 4, block 0);
// deposited locally when m c^2 is below the cut
template <class R>
__device__ __forceinline__ void annihilate(const PhysParams& pp, uint64_t key, uint64_t step, SecBuf<R>& sb, StepTally& tl)
{
    tl.n_annih += 1;
    if (kMe < pp.ecut) {
        tl.edep += 2.0 * kMe;
        return;
    }
    U64x4 w = philox4x64_10(key, step, 0, 4, pp.seed, pp.event);
    R cost = R(2) * unit_from<R>(w.w[0]) - R(1);
    R phi = R(2.0 * kPi) * unit_from<R>(w.w[1]);
    R sp, cp;
    m_sincos(phi, &sp, &cp);
    R sint = m_sqrt(R(1) - cost * cost);
    R v[3] = {sint * cp, sint * sp, cost};
    R mv[3] = {-v[0], -v[1], -v[2]};
    sb.add(kGamma, R(kMe), v, child_key(pp.seed, pp.event, key, step, 2));
    sb.add(kGamma, R(kMe), mv, child_key(pp.seed, pp.event, key, step, 3));
}

// in/out state of the interacting track
template <class R>
struct Prim {
    R T;
    R u[3];
    uint64_t key;
    uint32_t step;
    int type;
    bool alive;
};

// The lepton stops: its kinetic energy is deposited; a positron annihilates.
// Returns true when its annihilation at rest is still to be done.
template <class R>
__device__ __forceinline__ bool stop_lepton(Prim<R>& t, StepTally& tl)
{
    tl.edep += (double)t.T;
    t.T = R(0);
    t.alive = false;
    return t.type == kPositron;
}

// Sampled variable of process `proc` for a track of kinetic energy T (or a
// photon's energy): Compton's energy ratio, the pair's electron share, the
// delta ray's share of T, the photon's share of E.  One trial loop for all of
// them, so that the drawing of the uniforms is in the code once.
template <class R>
__device__ __forceinline__ R sample_share(int proc, R T, R ec, StepRng<R>& rng, StepTally& tl)
{
    R c0 = R(0), c1 = R(0), c2 = R(0), c3 = R(0), c4 = R(0), c5 = R(0);
    // (sums of products that several branches use are written as fused
    // operations: whether the compiler fuses one depends on the code around it)
    if (proc == P_COMPTON) {                    // kappa, e0^2, a1, a2, 1 - e0^2
        const R kap = T / R(kMe);
        const R e0 = R(1) / (R(1) + R(2) * kap), e0sq = e0 * e0;
        c0 = kap;
        c1 = e0sq;
        c2 = -m_log(e0);
        c4 = m_fma(-e0, e0, R(1));
        c3 = R(0.5) * c4;
    } else if (proc == P_PAIR) {                // m / E
        c0 = R(kMe) / T;
    } else if (proc == P_MOLLER) {              // cut / T, C1, C2, bound
        const R g = (T + R(kMe)) / R(kMe);
        c0 = ec / T;
        c1 = ((g - R(1)) / g) * ((g - R(1)) / g);
        c2 = (R(2) * g - R(1)) / (g * g);
        c3 = R(1) + c1 / R(4) + m_max(R(0), R(1) - c2);
    } else if (proc == P_BHABHA) {              // cut / T, beta^2, B1..B4
        const R g = (T + R(kMe)) / R(kMe);
        const R y = R(1) / (R(1) + g);
        c0 = ec / T;
        c1 = R(1) - R(1) / (g * g);
        c2 = R(2) - y * y;
        c3 = (R(1) - R(2) * y) * (R(3) + y * y);
        c5 = (R(1) - R(2) * y) * (R(1) - R(2) * y) * (R(1) - R(2) * y);
        c4 = c5 + (R(1) - R(2) * y) * (R(1) - R(2) * y);
    } else {                                    // cut / E, ln(T / cut)
        const R E = T + R(kMe);
        c0 = ec / E;
        c1 = m_log((T / E) / c0);
    }
    R x = R(0);
    const int n = proc == P_COMPTON ? 3 : 2;
    for (int trial = 0; trial < kMaxTrials; ++trial) {
        R a = R(0), b = R(0), c = R(0);          // the trial's uniforms, the last ones in b and c
#pragma unroll 1
        for (int k = 0; k < n; ++k) {
            a = b;
            b = c;
            c = rng.next();
        }
        bool ok;
        if (proc == P_COMPTON) {
            if (a * (c2 + c3) < c2) x = m_exp(-c2 * b);
            else x = m_sqrt(m_fma(c4, b, c1));
            const R omc = (R(1) - x) / (c0 * x);
            const R sin2 = omc * (R(2) - omc);
            ok = c <= R(1) - x * sin2 / (R(1) + x * x);
        } else if (proc == P_PAIR) {
            x = c0 + (R(1) - R(2) * c0) * b;
            ok = c <= R(1) - R(4) / R(3) * x * (R(1) - x);
        } else if (proc == P_MOLLER) {
            x = c0 / (R(1) - b * (R(1) - R(2) * c0));
            const R f = x * x * (c1 + R(1) / (x * x) + R(1) / ((R(1) - x) * (R(1) - x)) - c2 / (x * (R(1) - x)));
            ok = c * c3 <= f;
        } else if (proc == P_BHABHA) {
            x = c0 / (R(1) - b * (R(1) - c0));
            ok = c <= R(1) - c1 * (c2 * x - c3 * x * x + c4 * x * x * x - c5 * x * x * x * x);
        } else {
            x = c0 * m_exp(b * c1);
            ok = c <= R(1) - x + R(0.75) * x * x;
        }
        if (ok) break;
        if (trial == kMaxTrials - 1) tl.capped = 1;
    }
    return x;
}

// Discrete interaction `proc` of a track (P_ANNIH: at rest, the kinetic energy
// deposited before), whose next unused uniform of the step is j0.  The
// processes share their parts -- the trial loop, the rotation by the sampled
// angle and the recoil, the keys of the secondaries, the annihilation -- so
// that the code of all seven fits the instruction cache.
template <class R>
__device__ __forceinline__ void interact(const PhysParams& pp, int proc, Prim<R>& t, uint32_t j0, SecBuf<R>& sb,
                                         StepTally& tl)
{
    const R ec = R(pp.ecut);
    const R T = t.T;
    const bool delta = proc == P_MOLLER || proc == P_BHABHA;
    const uint64_t key0 = proc == P_ANNIH ? 0 : child_key(pp.seed, pp.event, t.key, t.step, 0);
    uint64_t key_at = t.key, step_at = t.step;       // of the annihilating positron
    bool annih = proc == P_ANNIH;
    if (proc == P_PHOTO) {
        if (T >= ec) sb.add(kElectron, T, t.u, key0);
        else tl.edep += (double)T;
        t.T = R(0);
        t.alive = false;
    } else if (proc != P_ANNIH) {
        StepRng<R> rng(pp.seed, pp.event, t.key, t.step, j0);
        const R x = rounded(sample_share<R>(proc, T, ec, rng, tl));
        if (proc == P_COMPTON || delta) {
            // the scattered photon, or the delta ray, at the sampled angle about the
            // track; the electron, or the track, takes the rest of the momentum
            const R phi = R(2.0 * kPi) * rng.next();
            R sp, cp;
            m_sincos(phi, &sp, &cp);
            R part, cosine, p_in = T, p_out;        // the sampled part of T; momenta before and of it
            if (delta) {
                part = x * T;
                const R t2 = T + R(2.0 * kMe), q2 = m_fma(x, T, R(2.0 * kMe));
                cosine = m_sqrt(part * t2 / (T * q2));
                p_in = m_sqrt(T * t2);
                p_out = m_sqrt(part * q2);
            } else {
                part = x * T;
                cosine = R(1) - (R(1) - x) / (T / R(kMe) * x);
                p_out = part;
            }
            part = rounded(part);
            p_in = rounded(p_in);
            p_out = rounded(p_out);
            cosine = rounded(cosine);
            R dir[3];
            rotate<R>(t.u, cosine, sp, cp, dir);
            R rest[3] = {p_in * t.u[0] - p_out * dir[0], p_in * t.u[1] - p_out * dir[1],
                         p_in * t.u[2] - p_out * dir[2]};
            // (the order of the squares' sum is fixed: x and y change places
            // between the two, which is how each was rounded when on its own)
            const R first = delta ? rest[1] : rest[0], second = delta ? rest[0] : rest[1];
            const R norm = m_sqrt(m_fma(rest[2], rest[2], m_fma(first, first, second * second)));
            rest[0] /= norm; rest[1] /= norm; rest[2] /= norm;
            // what is left of T: for Compton the fused difference
            const R left = delta ? T - part : m_fma(-x, T, T);
            const R T_sec = delta ? part : left, T_prim = delta ? left : part;
            for (int k = 0; k < 3; ++k) {
                const R d0 = dir[k], d1 = rest[k];
                dir[k] = delta ? d0 : d1;           // of the secondary
                rest[k] = delta ? d1 : d0;          // of the track
            }
            if (T_sec >= ec) sb.add(kElectron, T_sec, dir, key0);
            else tl.edep += (double)T_sec;
            t.T = T_prim;
            if (T_prim >= ec) {
                t.u[0] = rest[0]; t.u[1] = rest[1]; t.u[2] = rest[2];
            } else {
                annih = stop_lepton<R>(t, tl);      // (a photon: deposited like a lepton)
            }
        } else if (proc == P_PAIR) {
            const R Tp = m_fma(x, T, -R(kMe)), Tm = m_fma(R(1) - x, T, -R(kMe));
            if (Tm >= ec) sb.add(kElectron, Tm, t.u, key0);
            else tl.edep += (double)Tm;
            const uint64_t kp = child_key(pp.seed, pp.event, t.key, t.step, 1);
            if (Tp >= ec) {
                sb.add(kPositron, Tp, t.u, kp);
            } else {
                // a positron below the cut is not tracked: it deposits and annihilates
                // at the vertex with its own key at step 0
                tl.edep += (double)Tp;
                annih = true;
                key_at = kp;
                step_at = 0;
            }
            tl.n_pair += 1;
            t.T = R(0);
            t.alive = false;
        } else {                                    // bremsstrahlung
            const R k = rounded(x * (T + R(kMe)));
            if (k >= ec) sb.add(kGamma, k, t.u, key0);
            else tl.edep += (double)k;
            t.T = T - k;
            if (t.T < ec) annih = stop_lepton<R>(t, tl);
        }
    }
    if (annih) {
        annihilate<R>(pp, key_at, step_at, sb, tl);
        if (proc == P_ANNIH) {
            t.T = R(0);
            t.alive = false;
        }
    }
}

}  // namespace ems
