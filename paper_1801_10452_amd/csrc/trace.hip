// trace.hip -- the fused geodesic + radiative-transfer kernel and the flux reduction.
//
// One lane traces one ray (one camera pixel) backward from the camera: RK4 step of the null
// geodesic in Kerr-Schild coordinates (FP64, Sec. 2.2), termination tests, and at every
// accepted step inside the plasma the fluid sample, the fluid frame, the closure and the
// backward formal-solution update of every frequency (Sec. 3.1).  Waves are persistent: each
// starts with a tile of its own (64 rays, 8 x 8 pixels, or fewer) and takes the rays behind those
// from a global counter shared by every image of the launch.
#include "device_types.hpp"
#include "ks_geodesic.hpp"
#include "plasma.hpp"
#include "launch.hpp"
#include "mlp_device.hpp"

#include <type_traits>

namespace {

__device__ inline int find_job(const DevJob* jobs, int n_jobs, long long tile)
{
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].tile_base <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The kernel's arguments read afresh from the argument segment: what a refill, a sample round or a
// finished ray needs is loaded there (scalar loads, cached) instead of being held in scalar
// registers across the step, where it would spill into vector-register lanes.
__device__ inline const TraceParams& fresh_params()
{
    auto* k = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return *(const TraceParams*)k;
}

// A lane index the compiler takes for a new value: addresses formed from it are not kept.
__device__ inline int fresh(int lane)
{
    asm volatile("" : "+v"(lane));
    return lane;
}

__device__ inline unsigned lane_rank(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Transfer arithmetic in precision TT (double or float); the closure inputs come in FP64.
template <class TT>
struct Transfer;

template <>
struct Transfer<double> {
    // per-sample, frequency-independent part
    double ne, the, bf, sinb, ln_k2, ds, inr3, nr;
    bool emits;
    bool live;   // the sample contributes (a positive fluid-frame frequency)
    // the state as doubles: a record's words while several lanes share its sample
    static constexpr int WORDS = 9;
    __device__ inline void to_words(double* w) const
    {
        w[0] = ne; w[1] = the; w[2] = bf; w[3] = sinb; w[4] = ln_k2; w[5] = ds; w[6] = inr3; w[7] = nr;
        w[8] = __hiloint2double((int)live, (int)emits);
    }
    __device__ inline void from_words(const double* w)
    {
        ne = w[0]; the = w[1]; bf = w[2]; sinb = w[3]; ln_k2 = w[4]; ds = w[5]; inr3 = w[6]; nr = w[7];
        emits = __double2loint(w[8]) != 0;
        live = __double2hiint(w[8]) != 0;
    }
    __device__ inline void setup(const TraceParams& p, const double fl[4], double nr_, double cosb, double dsv)
    {
        ne = fl[0]; the = fl[1]; bf = fl[2];
        nr = nr_;
        ds = dsv;
        inr3 = rt::rcp_nr(nr * nr * nr);
        const double s2 = 1.0 - cosb * cosb;
        sinb = s2 > 0.0 ? s2 * rt::rsqrt_nr(s2) : 0.0;
        emits = (ne > 0.0 && the > 0.0 && bf > 0.0 && sinb > 0.0);
        ln_k2 = 0.0;
        if (emits && p.closure != CL_CONST)
            ln_k2 = (p.closure == CL_K2_PAPER) ? ::log(2.0 * the * the) : pl::ln_k2_theta(p.k2, the);
    }
    __device__ inline void contribution(const TraceParams& p, double nu_obs, double& A, double& dtau) const
    {
        double j, al, S;
        if (p.closure == CL_CONST) {
            j = p.const_j;
            al = p.const_alpha;
            S = al > 0.0 ? j / al : 0.0;
        } else if (emits) {
            pl::closure_exact(nu_obs * nr, ne, the, bf, sinb, ln_k2, &j, &al, &S);
        } else {
            return;
        }
        pl::step_source(j, al, S, ds, inr3, A, dtau);
    }
    // frequencies nu_obs[0 .. cnt) of up to G (entries g >= cnt are left untouched)
    // (nothing for a sample that does not contribute, see `live`)
    template <int G, bool BRANCHES = (G == 1)>
    __device__ inline void contributions(const TraceParams& p, const double* nu_obs, int cnt, double* A,
                                         double* dtau) const
    {
        if (!live) return;
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g < cnt) contribution(p, nu_obs[g], A[g], dtau[g]);
    }
};

// FP32 transfer.  The coefficients j, alpha, S and the step's contribution are float
// mantissas; the arguments of the exponentials whose size amplifies rounding -- X^1/3 in the
// emissivity (up to ~40 where the flux matters) and ln K2 -- are formed in double.  The
// factor 1/K2 exp(-X^1/3) = exp(-(ln K2 + X^1/3)) is split exactly into 2^-n 2^-f: the float
// arithmetic carries the mantissa 2^-f and the power of two 2^-n is applied in double at the
// end, so emission far below the float range (X^1/3 > 87, common at high frequencies) keeps its
// value instead of flushing to zero, and so does the large 1/K2 of cold plasma (Theta_e below
// ~0.01, where 1/K2 alone exceeds the float range).  The results (contribution and optical
// depth of the step) are doubles.
template <>
struct Transfer<float> {
    float ne, the, inv_the, nu_s, ds, inr3;
    double ln_k2;        // ln K2(1/Theta_e) (ln 2 Theta_e^2 for the paper's closure)
    double nr_inv_nus;   // nu_r / nu_s: X = nu_obs nu_r / nu_s in double
    double nr;
    bool emits;
    bool live;   // the sample contributes (a positive fluid-frame frequency)
    static constexpr int WORDS = 7;
    __device__ static inline double pack(float a, float b)
    {
        return __hiloint2double((int)__float_as_uint(b), (int)__float_as_uint(a));
    }
    __device__ inline void to_words(double* w) const
    {
        w[0] = pack(ne, the); w[1] = pack(inv_the, nu_s); w[2] = pack(ds, inr3);
        w[3] = ln_k2; w[4] = nr_inv_nus; w[5] = nr;
        w[6] = __hiloint2double((int)live, (int)emits);
    }
    __device__ inline void from_words(const double* w)
    {
        ne = __uint_as_float((unsigned)__double2loint(w[0])); the = __uint_as_float((unsigned)__double2hiint(w[0]));
        inv_the = __uint_as_float((unsigned)__double2loint(w[1])); nu_s = __uint_as_float((unsigned)__double2hiint(w[1]));
        ds = __uint_as_float((unsigned)__double2loint(w[2])); inr3 = __uint_as_float((unsigned)__double2hiint(w[2]));
        ln_k2 = w[3]; nr_inv_nus = w[4]; nr = w[5];
        emits = __double2loint(w[6]) != 0;
        live = __double2hiint(w[6]) != 0;
    }
    __device__ inline void setup(const TraceParams& p, const double fl[4], double nr_, double cosb, double dsv)
    {
        ne = (float)fl[0];
        the = (float)fl[1];
        inv_the = rt::rcpf_nr(the);
        nr = nr_;
        ds = (float)dsv;
        inr3 = rt::rcpf_nr((float)(nr_ * nr_ * nr_));
        const double s2 = 1.0 - cosb * cosb;
        const double sb = s2 > 0.0 ? s2 * rt::rsqrt_nr(s2) : 0.0;
        emits = (fl[0] > 0.0 && fl[1] > 0.0 && fl[2] > 0.0 && sb > 0.0);
        const double nus = (2.0 / 9.0) * pl::NUC_PER_GAUSS * fl[2] * fl[1] * fl[1] * sb;
        nu_s = (float)nus;
        nr_inv_nus = emits ? nr_ * rt::rcp_nr(nus) : 0.0;
        ln_k2 = 0.0;
        if (emits && p.closure != CL_CONST)
            ln_k2 = (p.closure == CL_K2_PAPER) ? rt::log_pos(2.0 * fl[1] * fl[1]) : pl::ln_k2_theta(p.k2, fl[1]);
    }
    // One frequency's coefficients from tt = X^1/3 (X = nu_obs nu_r / nu_s): the power of two
    // 2^-n of exp(-(ln K2 + tt)) = 2^-n 2^-f, the float mantissas of j (jm, j = jm 2^-n) and of
    // the source S = B_nu, and the step's optical depth dt in double.
    struct Terms {
        double scale, dt;
        float jm, S;
    };
    __device__ inline Terms terms(double tt, double nu_obs) const
    {
        // exp(-(ln K2 + tt)) = 2^-n 2^-f, |f| <= 1/2; beyond 2^-1100 the emission is zero in
        // double too, and the exponent is kept above -1000 so that the scale stays finite
        const double z = ::fmax(::fmin((tt + ln_k2) * 1.4426950408889634, 1100.0), -1000.0);
        const double n = __builtin_rint(z);
        const float em = __builtin_amdgcn_exp2f(-(float)(z - n));
        Terms T;
        T.scale = __builtin_ldexp(1.0, -(int)n);
        const float t = (float)tt;
        const float tc = t + 1.8877486253633868f;                 // 2^(11/12)
        T.jm = 1.1396857174835936e-29f * ne * nu_s * t * tc * tc * em;   // j = jm 2^-n
        const float nuf = (float)(nu_obs * nr);
        const float q = nuf * 2.45215662654257e-16f;              // nu (2h/c^2)^(1/3)
        const float q3 = q * q * q;                               // 2 h nu^3 / c^2
        const float em1 = rt::expm1_f((float)pl::H_OVER_MEC2 * nuf * inv_the);
        T.S = q3 * rt::rcpf_nr(em1);                              // B_nu
        const float dtm = T.jm * em1 * rt::rcpf_nr(q3) * ds;      // dtau = dtm 2^-n
        T.dt = (double)dtm * T.scale;
        return T;
    }
    __device__ inline void contribution(const TraceParams& p, double nu_obs, double& A, double& dtau) const
    {
        contributions<1>(p, &nu_obs, 1, &A, &dtau);
    }
    // Frequencies nu_obs[0 .. cnt) of up to G at once, written without branches (unless G = 1
    // and BRANCHES) so that the G dependency chains interleave, and so that consecutive calls in
    // a loop stay free of branches; entries g >= cnt, frequencies whose emission is below
    // exp(-1e8), and every entry of a sample that does not emit or contribute (`live`), are
    // left untouched.
    template <int G, bool BRANCHES = (G == 1)>
    __device__ inline void contributions(const TraceParams& p, const double* nu_obs, int cnt, double* A,
                                         double* dtau) const
    {
        if (p.closure == CL_CONST) {
            if (!live) return;
            const float j = (float)p.const_j, al = (float)p.const_alpha;
            float Af, dtf;
            pl::step_source(j, al, al > 0.0f ? j / al : 0.0f, ds, inr3, Af, dtf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (g < cnt) {
                    A[g] = Af;
                    dtau[g] = dtf;
                }
            }
            return;
        }
        if constexpr (G == 1 && BRANCHES) {
            // one frequency: branches skip the work that the selects below would only discard
            if (!(emits && live) || cnt < 1) return;
            const double X = nu_obs[0] * nr_inv_nus;
            if (!(X < 1e24)) return;   // exp(-X^1/3) < exp(-1e8): no emission, no absorption
            const Terms T = terms(rt::cbrt_refined(X), nu_obs[0]);
            dtau[0] = T.dt;
            if (T.dt > 1e-8)
                A[0] = (double)(T.S * -rt::expm1_f(-(float)T.dt) * inr3);
            else
                A[0] = (double)(T.jm * ds * inr3) * T.scale;   // S dtau = j ds to float precision
            return;
        }
        // a sample that does not emit goes through the same instructions, its results discarded
        const bool on = emits && live;
        bool ok[G];
        double tt[G], An[G], Dt[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const double X = nu_obs[g] * nr_inv_nus;
            ok[g] = on && g < cnt && X < 1e24;   // beyond, exp(-X^1/3) < exp(-1e8): no emission, no absorption
            tt[g] = rt::cbrt_refined(ok[g] ? X : 1.0);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const Terms T = terms(tt[g], nu_obs[g]);
            // 1 - exp(-dtau) = dtau (1 - dtau/2 + ...): below 1e-8, S dtau = j ds to float precision
            const double a_thick = (double)(T.S * -rt::expm1_f(-(float)T.dt) * inr3);
            const double a_thin = (double)(T.jm * ds * inr3) * T.scale;
            An[g] = T.dt > 1e-8 ? a_thick : a_thin;
            Dt[g] = T.dt;
        }
        // The G results are consumed here, unconditionally, by empty asm statements: without
        // that the compiler sinks each chain into a branch on ok[g], one after another, and the
        // chains no longer interleave.
#pragma unroll
        for (int g = 0; g < G; ++g) asm volatile("" ::"v"(An[g]), "v"(Dt[g]));
#pragma unroll
        for (int g = 0; g < G; ++g) {
            A[g] = ok[g] ? An[g] : A[g];
            dtau[g] = ok[g] ? Dt[g] : dtau[g];
        }
    }
};

// Attenuation e^-tau of the accumulated optical depth (held in double in both precisions).
template <class TT>
__device__ inline TT attenuation(double tau);
template <>
__device__ inline double attenuation<double>(double tau) { return ::exp(-tau); }
template <>
__device__ inline float attenuation<float>(double tau) { return rt::exp_mixed(-tau); }

// ---------------------------------------------------------------------------------------
// Sample compaction.  A lane whose ray takes a step inside the plasma does not evaluate the
// sample at once: the wave appends it to a ring of sample records in LDS, first in first out,
// whichever lanes the samples come from.  Once 64 are queued the wave evaluates the oldest 64
// together, one per lane, so the expensive part (MKS map, gather, fluid frame, closure) runs on
// full waves; it evaluates fewer only when the next step's samples would not fit, when no ray is
// left running, when as many rays wait for their last samples as still run, or when a ray has as many
// samples waiting as the optical-depth cut-off allows.  The samples of a ray are chained through
// their records; after a round each ray folds its evaluated samples into (I, tau) in the order they
// were taken, which keeps the backward transfer identical to evaluating every sample right after its
// step.  A ray that has ended waits in its lane until its samples are folded.
//
// The optical-depth-aware step needs each sample before its ray goes on: its kernels (EACH) queue
// nothing and evaluate and fold the samples of a step at once, one per ray.  Launches whose rounds the
// ring does not fill, or whose folds outweigh them (launch_geometry), run there too.
//
// A ring shared by the wave, against a queue of K samples per lane (K = 1 to 3) whose first full
// lane forced a round: a lone long ray at the end of a wave's work has a round every 64 of its
// steps instead of every K, a round of several frequencies is full where it held the samples of a
// single step, and with fewer rays per wave a round serves several steps of each.
// ---------------------------------------------------------------------------------------
constexpr int N_FIELDS = 10;   // t, r, theta, phi, k^t, k^r, k^phi, sin, cos, |dlambda|
constexpr int F_DL = 9;
// A sample record: the ten fields, then a word with the owner's lane (byte 0, with DROPPED once the
// cut-off has stopped the ray before this sample), the slot of the owner's next sample (byte 1) and
// the ray's pole crossings so far (byte 2, modulo 256), and the step number of the sample.  Eleven
// doubles: an odd stride lets consecutive lanes access consecutive records without bank conflicts.
// After the evaluation the fields hold its results: contributions in [0, FREQ_GROUP), optical depths
// behind them (the step length stays).
constexpr int REC = 11;
constexpr int REC_LINK = 80, REC_STEP = 84;   // byte offsets
constexpr unsigned char DROPPED = 128;

// Frequencies evaluated together (independent dependency chains) by one lane.
constexpr int FREQ_GROUP = 4;
// Cut-off: samples a ray may have waiting (those behind the one that makes it opaque are dropped).
constexpr int CUT_PENDING = 8;
static_assert(2 * FREQ_GROUP <= F_DL, "the results of a group fit the record below the step length");
static_assert(Transfer<double>::WORDS <= F_DL && Transfer<float>::WORDS <= F_DL,
              "the transfer set-up fits the record below the step length");

// What the evaluation of a queued sample needs from its ray's job.
struct LaneInfo {
    double a;
    int grid, fast_snap, nu_base;
};

__device__ inline LaneInfo lane_info(const TraceParams& p, int job)
{
    const DevJob& J = p.jobs[job];
    return LaneInfo{J.a, J.grid, J.fast_snap, J.nu_base};
}

// The LDS of a wave: job and pixel index of each lane [64 each], three byte tables of the rays in a
// round [64 each], counts of ended rays by status and of pole crossings [8], the sample ring
// [slots][REC], and a row per ray: its intensity and its optical depth at every frequency, and the
// rate of the optical-depth-aware step.  What a ray needs only once a round or less lives here, not
// in registers: the step and the evaluation leave none free at three waves per SIMD.
template <int NNU, bool MLPC, int WPE>
struct Queue {
    // words of each kind in a row: as the launch has frequencies, so that the rows of 5 to 8, 12 or
    // 24 take no more LDS (waves) than they need
    __host__ __device__ static constexpr int cols(int n_nu) { return NNU > FREQ_GROUP ? n_nu : NNU; }
    __host__ __device__ static constexpr int row(int n_nu) { return 2 * cols(n_nu) + 1; }   // odd, as REC
    static constexpr size_t HEAD = 128 * sizeof(int) + 192 + 8 * sizeof(unsigned);
    __host__ __device__ static constexpr size_t per_wave(int rays, int slots, int n_nu)
    {
        return (HEAD + (size_t)slots * REC * 8 + (size_t)rays * row(n_nu) * 8 + 15) / 16 * 16;
    }
    // Ring size: 64 slots for a round and one for each ray, so that a step never has to force a
    // round, as far as the variant's waves then fit a compute unit's LDS (beside one copy of the
    // network for the learned closure), and no fewer than the 64 that a round takes.
    static constexpr int slots(int rays, int n_nu)
    {
        const size_t used = HEAD + (size_t)rays * row(n_nu) * 8 + 15, least = used + 64 * REC * 8;
        size_t budget = MLPC ? (LDS_BYTES - mlp::LDS_NET_BYTES) / 8 : 0;
        for (int w = WPE; !MLPC && w >= 1 && budget < least; --w)
            budget = LDS_BYTES / w / LDS_GRANULE * LDS_GRANULE / 4;   // w work-groups of four waves
        const int fit = budget > least ? (int)((budget - used) / (REC * 8)) : 64;
        return fit >= 64 + rays ? 64 + rays : fit;
    }
};

__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline unsigned char* link_of(double* rec) { return reinterpret_cast<unsigned char*>(rec) + REC_LINK; }
__device__ inline unsigned char* link_of(double* ring, int slot) { return link_of(ring + slot * REC); }

// The frequency-independent part of a queued sample's evaluation: fluid state, fluid frame and
// the transfer set-up.  A sample whose fluid-frame frequency is not positive (integration error
// of a low-order integrator in the last step before the horizon) has no defined emission: its
// transfer stays non-emitting and it adds nothing.  Returns whether the fluid frame fell back to
// the ZAMO.
template <class TT>
__device__ inline bool setup_sample(const TraceParams& p, const double* q, const LaneInfo& li, Transfer<TT>& tr)
{
    const DevGrid& G = p.grids[li.grid];
    const double y[8] = {q[0], q[1], q[2], q[3], q[4], q[5], 0.0, q[6]};
    double fl[4];
    pl::sample_fluid(G, p.slow_light, li.fast_snap, y, fl);
    double nr, cb;
    const bool zamo = pl::fluid_frame(li.a, li.a * li.a, p.M, y, q[7], q[8], fl[3], &nr, &cb);
    tr.emits = false;
    tr.live = nr > 0.0;
    if (tr.live) tr.setup(p, fl, nr, cb, nr * q[F_DL] * p.length_unit);
    return zamo;
}

// The learned closure's step contribution in FP32 transfer, by the scheme of Transfer<float>: the
// network gives ln j_hat + X^1/3 and ln alpha_hat + X^1/3 (standardised); the cut-off factor
// exp(-X^1/3), common to j and alpha, is split exactly into 2^-n 2^-f, the float arithmetic
// carries 2^-f and the power of two is applied in double to the step's optical depth and
// contribution.  j = n_e nu_c J0 e^(ln j_hat), alpha = n_e J0 / (2 m_e nu_c) e^(ln alpha_hat)
// B_RJ/B_nu, and the source is their ratio.
__device__ inline void mlp_contribution_f32(const Transfer<float>& tr, float y0, float y1, double nu_obs, double nuc,
                                            double& A, double& dtau)
{
    const double X = nu_obs * tr.nr_inv_nus;
    if (!(X < 1e24)) return;   // exp(-X^1/3) < exp(-1e8): no emission, no absorption
    const double tt = rt::cbrt_refined(X);
    const double z = ::fmin(tt * 1.4426950408889634, 1100.0);
    const double n = __builtin_rint(z);
    const float em = __builtin_amdgcn_exp2f(-(float)(z - n));
    const double scale = __builtin_ldexp(1.0, -(int)n);
    const float ej = __expf(y0 * mlp::SIGMA_J + mlp::MU_J), ea = __expf(y1 * mlp::SIGMA_A + mlp::MU_A);
    const float nucf = (float)nuc;
    const float yy = (float)pl::H_OVER_MEC2 * (float)(nu_obs * tr.nr) * tr.inv_the;
    const float planck = (yy > 1e-4f) ? rt::expm1_f(yy) * rt::rcpf_nr(yy) : 1.0f + 0.5f * yy;   // B_RJ / B_nu
    const float jm = tr.ne * nucf * (float)pl::J_PREF * ej * em;                                 // j = jm 2^-n
    const float am = tr.ne * (float)(pl::J_PREF / (2.0 * pl::ME_CGS)) * rt::rcpf_nr(nucf) * ea * em * planck;
    const float dtm = am * tr.ds;                                                                // dtau = dtm 2^-n
    dtau = (double)dtm * scale;
    if (dtau > 1e-8) {
        A = (double)(jm * rt::rcpf_nr(am) * -rt::expm1_f(-(float)dtau) * tr.inr3);
    } else {
        // 1 - exp(-dtau) = dtau (1 - dtau/2 + ...): S dtau = j ds to float precision
        A = (double)(jm * tr.ds * tr.inr3) * scale;
    }
}

// Learned closure: the frequency-independent part of a sample, and its contribution at one
// frequency.  Every lane of the wave takes part in the network evaluations; lanes without a sample
// feed zeros.  Samples whose closure inputs leave the training box use the exact closure, except
// where the exact closure itself gives exactly zero: where X^1/3 + ln K2(1/Theta_e) exceeds
// MLP_ZERO_EXP, the factor exp(-(X^1/3 + ln K2)) lies below the smallest double, so j and alpha
// vanish in both transfer precisions (the FP32 transfer's power of two 2^-n has n >= 1076 there).
// Those samples are skipped (counted as dropped) at no change to any result.
constexpr double MLP_ZERO_EXP = 746.0;

template <class TT>
struct MlpSample {
    Transfer<TT> tr;
    double fl[4], nr, cb, nuc, ds, inr3, nus;
    float lth;
    bool has;
    __device__ inline bool setup(const TraceParams& p, bool has_, const double* q, const LaneInfo& li)
    {
        fl[0] = 0.0; fl[1] = 1.0; fl[2] = 1.0; fl[3] = 0.0;
        nr = 1.0;
        cb = 0.0;
        has = has_;
        bool zamo = false;
        tr.emits = false;
        tr.live = false;
        if (has) {
            const DevGrid& G = p.grids[li.grid];
            const double y[8] = {q[0], q[1], q[2], q[3], q[4], q[5], 0.0, q[6]};
            pl::sample_fluid(G, p.slow_light, li.fast_snap, y, fl);
            zamo = pl::fluid_frame(li.a, li.a * li.a, p.M, y, q[7], q[8], fl[3], &nr, &cb);
            // a non-positive fluid-frame frequency has no defined emission (see setup_sample): the
            // transfer stays non-emitting and the sample adds nothing
            tr.live = nr > 0.0;
            if (tr.live) tr.setup(p, fl, nr, cb, nr * q[F_DL] * p.length_unit);
        }
        nuc = pl::NUC_PER_GAUSS * fl[2];
        lth = (float)rt::log_pos(fl[1] > 0.0 ? fl[1] : 1.0);
        ds = nr * q[F_DL] * p.length_unit;
        inr3 = has ? rt::rcp_nr(nr * nr * nr) : 0.0;
        // nu_s / nu: X = nu / nu_s, nu_s = (2/9) nu_c Theta_e^2 sin(theta_B)
        nus = (2.0 / 9.0) * nuc * fl[1] * fl[1] * ::sqrt(::fmax(1.0 - cb * cb, 0.0));
        return zamo;
    }
    // fallback, dropped: whether the exact closure took the sample, and whether it was skipped
    __device__ inline void contribution(const TraceParams& p, const unsigned char* lds_net, double nu_obs, double& A,
                                        double& dtau, bool& fallback, bool& dropped)
    {
        const double nu = has ? nu_obs * nr : nuc;
        const float lx = (float)rt::log_pos(nu / nuc);
        const bool inb = has && tr.emits && mlp::in_box(lx, lth, (float)cb);
        // X^1/3 + ln K2 > MLP_ZERO_EXP  <=>  X > t_lim^3, t_lim = MLP_ZERO_EXP - ln K2 (X^1/3 >= 0)
        const double t_lim = MLP_ZERO_EXP - tr.ln_k2;
        dropped = has && tr.emits && !inb && (t_lim <= 0.0 || nu > t_lim * t_lim * t_lim * nus);
        fallback = has && tr.emits && !inb && !dropped;
        const float x0 = inb ? mlp::norm_lx(lx) : 0.0f, x1 = inb ? mlp::norm_lt(lth) : 0.0f,
                    x2 = inb ? mlp::norm_cb((float)cb) : 0.0f;
        float y0, y1;
        if (p.closure == CL_MLP_BF16)
            mlp::forward_wave_lds<false>(lds_net, inb, x0, x1, x2, &y0, &y1);
        else
            mlp::forward_wave_lds<true>(lds_net, inb, x0, x1, x2, &y0, &y1);
        A = 0.0;
        dtau = 0.0;
        if (!has) return;
        if (inb) {
            if constexpr (std::is_same<TT, float>::value) {
                mlp_contribution_f32(tr, y0, y1, nu_obs, nuc, A, dtau);
            } else {
                // the network gives ln j_hat + X^1/3 and ln alpha_hat + X^1/3 (standardised); the
                // coefficients are formed in double from them (their logs span hundreds)
                const double sb2 = 1.0 - cb * cb;
                const double tc = rt::cbrt_refined(nu / ((2.0 / 9.0) * nuc * fl[1] * fl[1] * ::sqrt(sb2)));
                const double lnj = y0 * mlp::SIGMA_J + mlp::MU_J - tc, lna = y1 * mlp::SIGMA_A + mlp::MU_A - tc;
                const double ne = fl[0];
                const double j = ne * nuc * pl::J_PREF * ::exp(lnj);
                const double yy = pl::H_OVER_MEC2 * nu / fl[1];
                const double planck = (yy > 1e-4) ? ::expm1(yy) / yy : 1.0 + 0.5 * yy;   // B_RJ / B_nu
                const double al = ne * pl::J_PREF / (2.0 * pl::ME_CGS * nuc) * ::exp(lna) * planck;
                pl::step_source(j, al, j / al, ds, inr3, A, dtau);
            }
        } else if (fallback) {
            tr.contribution(p, nu_obs, A, dtau);
        }
    }
};

// Work-groups of up to 256 lanes; up to 512 for the learned closure's 2-waves-per-SIMD variant,
// whose eight waves share one LDS copy of the network (a 512-lane group caps a kernel at 256
// registers per lane, which that variant fits anyway).
template <int NNU, class TT, int WPE, bool MLPC, int INTEG, bool EACH>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, (MLPC && WPE >= 2) ? 512 : 256),
                               amdgpu_waves_per_eu(WPE, 8)))
trace_kernel(TraceParams args)
{
    const TraceParams& p = args;
    using Q = Queue<NNU, MLPC, WPE>;
    constexpr int G = NNU < FREQ_GROUP ? NNU : FREQ_GROUP;
    // lanes [0, RAYS) trace rays; with fewer than 64 rays per wave the other lanes only work in the
    // sample rounds
    const int RAYS = p.rays_per_wave;
    const int SLOTS = p.slots;
    const int COLS = Q::cols(p.n_nu), ROW = Q::row(p.n_nu);
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const size_t per_wave = Q::per_wave(RAYS, SLOTS, p.n_nu);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char* wbase = smem + wid * (int)per_wave;
    int* lane_job = reinterpret_cast<int*>(wbase);                                  // [64]
    int* lane_pix = lane_job + 64;                                                  // [64]
    unsigned char* ray_tab = wbase + 128 * sizeof(int);                             // [64] lane of the n-th ray
    unsigned char* ray_next = ray_tab + 64;                                         // [64] per lane
    unsigned char* ray_left = ray_next + 64;                                        // [64]
    unsigned* tally = reinterpret_cast<unsigned*>(ray_left + 64);                   // [8] by status; [0]: poles
    double* ring = reinterpret_cast<double*>(wbase + Q::HEAD);                      // [SLOTS][REC]
    double* rows = ring + (size_t)SLOTS * REC;                                      // [RAYS][ROW]
    const double M = p.M;
    // learned closure: the work-group's copy of the network, after the areas of its waves
    unsigned char* lds_net = smem + (size_t)(blockDim.x >> 6) * per_wave;
    if (MLPC) {
        const mlp::Net net{p.mlp_P, p.mlp_W, p.mlp_Wlo, nullptr};
        mlp::stage_weights(net, lds_net, threadIdx.x, blockDim.x);
        __syncthreads();
    }

    // ray state of this lane (Verlet also carries dk/dlambda at y, valid when have_acc)
    double y[8];
    double vacc[4] = {0.0, 0.0, 0.0, 0.0};
    bool have_acc = false;
    double a = 0.0, r_stop = 0.0, r_esc = 0.0, sth = 0.0, cth = 1.0;
    int steps = 0;
    // this ray's queued samples: oldest slot in bits 0-7, newest in 8-15, their number in 16-23; in
    // 24-31 the pole crossings of the lane's rays, modulo 256
    unsigned queued = 0;
    int lead = NNU > FREQ_GROUP ? (p.n_nu - 1) / G * G : 0;   // cut-off: the group looked at first in a round
    const auto first = [&] { return (int)(queued & 255u); };
    const auto pending = [&] { return (int)(queued >> 16 & 255u); };
    int status = RAY_IDLE;
    // the ray's accumulated intensities and optical depths (doubles; the per-sample terms are TT),
    // and a last word: the step length between a step and the queueing of its sample, and with EACH,
    // from the sample to the next step, d tau / d|lambda| of the sample at its most absorbing frequency
    // (0: no transfer limit on the next step).
    const int RATE = 2 * COLS;
    // this lane's row (for the lanes below RAYS); as the other per-lane LDS addresses formed where it
    // is used, from `fresh(lane)`, so that no register holds it across the step
    const auto row_of = [&](int l) { return rows + l * ROW; };
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = 0.0;

    // wave-level statistics: ballot counts in scalar registers, and the tally of rarer events
    unsigned long long c_steps = 0, c_samples = 0, c_zamo = 0, c_fallback = 0, c_dropped = 0;
    if (lane < 8) tally[lane] = 0u;

    // Rays of the current tile not yet handed out (wave-uniform).  The first tile of a wave is its
    // own index, so that a launch does not begin with an atomic of every wave on one counter, and one
    // with fewer tiles than waves has none; the counter starts behind them.
    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + wid;
    const long long n_waves = (long long)gridDim.x * (blockDim.x >> 6);
    long long next = wave * RAYS, end = wave < p.n_tiles ? next + RAYS : next;
    bool drained = n_waves >= p.n_tiles;
    int head = 0, total = 0;       // the ring: oldest slot, samples queued (wave-uniform)

    // The lanes with a running ray and those whose ended ray waits for its samples, as scalar masks:
    // an iteration in which no ray starts or ends asks the lanes for two ballots only (a ballot
    // that a branch depends on costs a lone wave about 60 cycles).
    const unsigned long long ray_lanes = RAYS == 64 ? ~0ull : (1ull << RAYS) - 1ull;
    unsigned long long run = 0, wait = 0;
    bool idle_changed = true;

    while (true) {
        // ------------------------------------------------------------ refill idle lanes
        if (idle_changed) {
            idle_changed = false;
            const TraceParams& p = fresh_params();
            unsigned long long idle = ray_lanes & ~(run | wait);
            int n_idle = __popcll(idle);
            if (n_idle < p.refill_threshold && n_idle < RAYS) n_idle = 0;
            while (n_idle > 0) {
                if (next == end) {
                    if (drained) break;
                    // a tile's worth of rays at once, and near the end of the launch about as many as
                    // there are idle lanes: a wave hands out what it holds over hundreds of steps,
                    // while other waves run out
                    const long long total_rays = p.n_tiles * RAYS;
                    const int tail = n_idle > 8 ? n_idle : 8 < RAYS ? 8 : RAYS;
                    const int chunk = total_rays - end > n_waves * RAYS ? RAYS : tail;
                    unsigned long long t = 0;
                    if (lane == 0) t = atomicAdd(p.ray_counter, (unsigned long long)chunk);
                    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)t);
                    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(t >> 32));
                    next = (long long)(((unsigned long long)hi << 32) | lo);
                    end = next + chunk < total_rays ? next + chunk : total_rays;
                    if (next >= total_rays) {
                        next = end;
                        drained = true;
                        break;
                    }
                }
                const long long avail = end - next;
                const unsigned rank = lane_rank(idle);
                bool started = false;
                if (__builtin_amdgcn_inverse_ballot_w64(idle) && (long long)rank < avail) {
                    const long long ray = next + rank;
                    const long long tile = ray >> p.rays_shift;
                    const int slot = (int)(ray & (RAYS - 1));
                    const int job = find_job(p.jobs, p.n_jobs, tile);
                    const DevJob& J = p.jobs[job];
                    const long long lt = tile - J.tile_base;
                    const int tw = 1 << p.tile_shift;
                    const int px = (int)(lt % J.tiles_x) * tw + (slot & (tw - 1));
                    const int py = (int)(lt / J.tiles_x) * (RAYS >> p.tile_shift) + (slot >> p.tile_shift);
                    if (px < J.nx && py < J.ny) {
                        const double alpha = __builtin_fma(px + 0.5, J.dalpha, -J.fov);
                        const double beta = __builtin_fma(py + 0.5, J.dbeta, -J.fov);
                        a = J.a;
                        rk::camera_ray(J.cam, alpha, beta, y);
                        sth = J.sin_th;
                        cth = J.cos_th;
                        r_stop = J.r_stop;
                        r_esc = J.cam.r;
                        const int l = fresh(lane);
                        double* my_row = row_of(l);
                        lane_job[l] = job;
                        lane_pix[l] = py * J.nx + px;
                        steps = 0;
                        have_acc = false;
                        for (int f = 0; f < ROW; ++f) my_row[f] = 0.0;
                        status = RAY_RUNNING;
                        started = true;
                    }
                }
                next += (avail < n_idle) ? avail : n_idle;
                run |= __ballot(started);
                idle = ray_lanes & ~(run | wait);
                n_idle = __popcll(idle);
            }
        }
        if ((run | (unsigned long long)total) == 0ull) break;   // nothing running or queued: the tiles are drained

        // ------------------------------------------------------------ one step of every running ray
        bool event = false, reflected = false, want = false;
        if (__builtin_amdgcn_inverse_ballot_w64(run)) {
            const rk::Spin<double> sp = rk::make_spin(a, M);
            double h = rk::step_size(p.eps, y);
            if constexpr (EACH) {
                double* my_row = row_of(fresh(lane));
                const double rate = my_row[RATE];
                if (rate > 0.0) h = ::fmin(h, p.tau_step / rate);
                my_row[RATE] = 0.0;
            }
            const double dl = -h;
            [[maybe_unused]] const double th0 = y[2], s0 = sth, c0 = cth;
            if (INTEG == INTEG_RK2) {
                rk::rk2_step(sp, y, dl, sth, cth);
            } else if (INTEG == INTEG_VERLET) {
                if (!have_acc) rk::ks_accel<true>(sp, y, sth, cth, vacc);
                rk::verlet_step(sp, y, vacc, dl, p.integrator == INTEG_VERLET_CORR, sth, cth);
                have_acc = true;
            } else {
                rk::rk4_step_angles<false>(sp, y, dl, p.eps <= rk::EPS_CHAINED, &sth, &cth);
            }
            ++steps;
            // What ends a ray or reflects it at the axis is rare: one test covers it all.  (A
            // non-finite derivative reaches the wave vector whichever stage it arises in, and the sum
            // of the four components is finite only if each is.)
            const bool plain = y[2] >= 0.0 && y[2] <= M_PI && y[1] >= r_stop && y[1] <= r_esc &&
                               steps < p.max_steps && ::isfinite((y[4] + y[5]) + (y[6] + y[7]));
            if (!plain) {
                event = true;
                bool fin = true;
#pragma unroll
                for (int i = 4; i < 8; ++i) fin = fin && ::isfinite(y[i]);
                if (!fin) {
                    status = RAY_NUMERIC;
                } else {
                    reflected = rk::reflect_pole(y);
                    if (reflected) {
                        have_acc = false;   // the carried derivative belongs to the old chart
                        rt::sincos_small(y[2], &sth, &cth);
                    }
                    if (y[1] < r_stop)
                        status = RAY_HORIZON;
                    else if (y[1] > r_esc)
                        status = RAY_ESCAPED;
                    else if (steps >= p.max_steps)
                        status = RAY_MAXSTEP;
                }
            }
            // sin and cos of the new theta from those of the old one (the step moves theta little;
            // RK4 has them already, a reflection forms them from scratch)
            if (INTEG != INTEG_RK4)
                if (!reflected && status != RAY_NUMERIC) rk::sincos_shift(th0, s0, c0, y[2], &sth, &cth);
            if (status == RAY_RUNNING) {
                // the radial range of the fluid: one for the launch, or the one of the ray's grid
                double lo = p.r_in, hi = p.r_out;
                if (!(lo < hi)) {
                    const DevGrid& gr = p.grids[p.jobs[lane_job[fresh(lane)]].grid];
                    lo = gr.r_in;
                    hi = gr.r_out;
                }
                want = y[1] >= lo && y[1] <= hi;
                // the step length waits here for the sample's record (a round may come first)
                if (want) row_of(fresh(lane))[RATE] = h;
            }
        }
        c_steps += __popcll(run);
        const unsigned long long events = __ballot(event);
        if (events) {
            if (reflected) {
                atomicAdd(tally, 1u);
                queued += 1u << 24;
            }
            const unsigned long long ended = __ballot(status > RAY_RUNNING) & run;
            run &= ~ended;
            wait |= ended;
        }

        unsigned long long adds = __ballot(want);
        const int n_want = __popcll(adds);
        // this ray's sample into its record, with the lane and the pole crossings
        const auto put = [&](double* rec, int lane) {
            rec[0] = y[0];
            rec[1] = y[1];
            rec[2] = y[2];
            rec[3] = y[3];
            rec[4] = y[4];
            rec[5] = y[5];
            rec[6] = y[7];
            rec[7] = sth;
            rec[8] = cth;
            rec[F_DL] = row_of(lane)[RATE];
            *reinterpret_cast<int*>(rec + N_FIELDS) = lane | (int)(queued >> 8 & 0xff0000u);
        };

        // ------------------------------------------------------------ evaluate and fold the step's samples
        if (EACH && adds) {
            // One sample per ray.  Lane i sets up sample i and leaves the set-up in its record; then
            // `per` consecutive lanes share each sample, lane c of them taking its frequencies
            // [c m, (c + 1) m), m = ceil(n_nu / per): contribution and fold, I += exp(-tau) A, tau +=
            // dtau, straight into the owner's row.  (As rounds of the ring, a group of frequencies
            // after another on the lanes with a sample, 256^2 at 4 and 24 frequencies took 79.6 and
            // 280 ms against 68 and 207, FP64 transfer, and with the cut-off, whose groups are looked
            // at before they are folded, 81 and 478 against 66 and 192.)
            const TraceParams& p = fresh_params();
            const int lane = fresh(threadIdx.x & 63);
            double* my_rec = ring + lane_rank(adds) * REC;
            if (__builtin_amdgcn_inverse_ballot_w64(adds)) put(my_rec, lane);
            wave_lds_sync();
            const bool has = lane < n_want;
            double* rec = ring + (has ? lane : 0) * REC;
            const int owner = link_of(rec)[0];
            const LaneInfo li = lane_info(p, lane_job[owner]);
            double q[N_FIELDS];
#pragma unroll
            for (int f = 0; f < N_FIELDS; ++f) q[f] = MLPC && !has ? 1.0 : rec[f];
            double* row = rows + owner * ROW;
            double tmin = 1e300, dmax = 0.0;   // over the frequencies of this lane
            const auto fold = [&](int f, double t0, TT att, double A, double dt) {
                row[f] = __builtin_fma((double)att, A, row[f]);
                const double t1 = t0 + dt;
                row[COLS + f] = t1;
                tmin = ::fmin(tmin, t1);
                dmax = ::fmax(dmax, dt);
            };
            if (MLPC) {
                MlpSample<TT> ms;
                c_zamo += __popcll(__ballot(ms.setup(p, has, q, li)));
#pragma unroll 1
                for (int f = 0; f < p.n_nu; ++f) {
                    double A, dt;
                    bool fb, dr;
                    ms.contribution(p, lds_net, p.nu[li.nu_base + f], A, dt, fb, dr);
                    c_fallback += __popcll(__ballot(fb));
                    c_dropped += __popcll(__ballot(dr));
                    if (has) {
                        const double t0 = row[COLS + f];
                        fold(f, t0, attenuation<TT>(t0), A, dt);
                    }
                }
                if (has) {
                    rec[0] = tmin;
                    rec[1] = dmax;
                }
            } else {
                Transfer<TT> tr;
                bool zamo = false;
                if (has) zamo = setup_sample<TT>(p, q, li, tr);
                c_zamo += __popcll(__ballot(zamo));
                const unsigned share = 64u / (unsigned)n_want;
                const unsigned per = NNU == 1 ? 1u : share < (unsigned)p.n_nu ? share : (unsigned)p.n_nu;
                unsigned is = lane, c = 0;
                int nu_base = li.nu_base, f = 0, f1 = 1;
                if (NNU > 1) {
                    double w[Transfer<TT>::WORDS];
                    if (has) {
                        tr.to_words(w);
#pragma unroll
                        for (int k = 0; k < Transfer<TT>::WORDS; ++k) rec[k] = w[k];
                    }
                    wave_lds_sync();
                    const unsigned mul = (65535u + per) / per;   // x / per = (x mul) >> 16 for x < 1024
                    is = (unsigned)lane * mul >> 16;
                    c = (unsigned)lane - is * per;
                    rec = ring + (is < (unsigned)n_want ? is : 0u) * REC;
#pragma unroll
                    for (int k = 0; k < Transfer<TT>::WORDS; ++k) w[k] = rec[k];
                    tr.from_words(w);
                    const int o = link_of(rec)[0];
                    row = rows + o * ROW;
                    nu_base = p.jobs[lane_job[o]].nu_base;
                    const int m = (int)(((unsigned)p.n_nu + per - 1u) * mul >> 16);
                    f = (int)c * m;
                    f1 = f + m < p.n_nu ? f + m : p.n_nu;
                }
                if (is < (unsigned)n_want) {
                    if (NNU > 1) {
                        for (; f + G <= f1; f += G) {
                            double nu[G], A[G], dt[G], t0[G];
                            TT att[G];   // formed before the contributions, so that the chains overlap
#pragma unroll
                            for (int g = 0; g < G; ++g) {
                                nu[g] = p.nu[nu_base + f + g];
                                A[g] = 0.0;
                                dt[g] = 0.0;
                                t0[g] = row[COLS + f + g];
                                att[g] = attenuation<TT>(t0[g]);
                            }
                            tr.template contributions<G>(p, nu, G, A, dt);
#pragma unroll
                            for (int g = 0; g < G; ++g) fold(f + g, t0[g], att[g], A[g], dt[g]);
                        }
                    }
                    for (; f < f1; ++f) {   // the rest one at a time
                        double A = 0.0, dt = 0.0;
                        const double nu1 = p.nu[nu_base + f], t0 = row[COLS + f];
                        tr.template contributions<1, NNU == 1>(p, &nu1, 1, &A, &dt);
                        fold(f, t0, attenuation<TT>(t0), A, dt);
                    }
                }
                // over the sample's lanes onto its first, which leaves them in the record
                for (unsigned off = 1; off < per; off <<= 1) {
                    const double tm = __shfl_down(tmin, off, 64), dm = __shfl_down(dmax, off, 64);
                    if (c + off < per) {
                        tmin = ::fmin(tmin, tm);
                        dmax = ::fmax(dmax, dm);
                    }
                }
                wave_lds_sync();
                if (is < (unsigned)n_want && c == 0) {
                    rec[0] = tmin;
                    rec[1] = dmax;
                }
            }
            wave_lds_sync();
            c_samples += n_want;
            if (__builtin_amdgcn_inverse_ballot_w64(adds)) {
                row_of(lane)[RATE] = my_rec[1] / my_rec[F_DL];
                if (p.tau_cutoff > 0.0 && my_rec[0] >= p.tau_cutoff) status = RAY_OPAQUE;
            }
            const unsigned long long ended = __ballot(status > RAY_RUNNING) & run;
            run &= ~ended;
            wait |= ended;
            wave_lds_sync();
        }

        // ------------------------------------------------------------ evaluate queued samples
        bool round = EACH ? adds != 0ull : total >= 64 || total + n_want > SLOTS;
        if (!EACH && !round && total > 0)
            round = __popcll(wait) >= __popcll(run) ||
                    (p.tau_cutoff > 0.0 && __ballot(pending() >= CUT_PENDING) != 0ull);
        if (!EACH && round) {
            const TraceParams& p = fresh_params();
            const int lane = fresh(threadIdx.x & 63);
            double* my_row = row_of(lane);
            const int n_eval = total < 64 ? total : 64;
            int slot = head + (lane < n_eval ? lane : 0);
            slot = slot >= SLOTS ? slot - SLOTS : slot;
            double* rec = ring + slot * REC;
            // (a lane without a sample reads the oldest one's owner: a lane with a job)
            const unsigned char link = link_of(ring, slot)[0];
            const int owner = link & 63;
            const bool has = lane < n_eval && !(link & DROPPED);
            double q[N_FIELDS];
#pragma unroll
            for (int f = 0; f < N_FIELDS; ++f) q[f] = MLPC && !has ? 1.0 : rec[f];
            Transfer<TT> tr;
            MlpSample<TT> ms;
            int nu_base = 0;
            bool zamo = false;
            if (MLPC) {
                const LaneInfo li = lane_info(p, lane_job[owner]);
                nu_base = li.nu_base;
                zamo = ms.setup(p, has, q, li);
            } else if (has) {
                const LaneInfo li = lane_info(p, lane_job[owner]);
                nu_base = li.nu_base;
                zamo = setup_sample<TT>(p, q, li, tr);
            }
            int fallback = 0, dropped = 0;   // of this lane's sample, over the frequencies folded

            // whether slot s lies among the evaluated samples
            auto evaluated = [&](int s) {
                const int d = s - head;
                return (d < 0 ? d + SLOTS : d) < n_eval;
            };
            const bool mine = pending() > 0 && evaluated(first());
            const unsigned long long rays = __ballot(mine);
            const int n_rays = __popcll(rays);
            // Each ray folds its evaluated samples in order, I += exp(-tau) A, tau += dtau: one lane
            // per ray takes all frequencies of a group, or, when there are lanes for it, one lane per
            // (ray, frequency).  The cut-off looks at every frequency of a sample, so its rays fold in
            // one lane.
            const bool spread = NNU > 1 && n_rays * G <= 64 && !(p.tau_cutoff > 0.0);
            if (spread && mine) ray_tab[lane_rank(rays)] = (unsigned char)lane;
            int stop = -1;                 // cut-off: slot of the sample that made the ray opaque
            int nxt = first(), taken = 0;  // after the walk: the ray's oldest sample left and the number folded
            // The cut-off stops a ray at the first sample behind which every frequency is beyond it.
            // With several groups that sample (stop_n, counted along the walk) has to be known before
            // anything is folded.  The group `lead` decides nearly every round by itself: a ray with a
            // frequency there below the cut-off after all its samples does not stop.  If one is left
            // in question the other groups are evaluated too, and then all of them again to be folded.
            const bool groups = NNU > FREQ_GROUP && p.tau_cutoff > 0.0 && p.n_nu > G;
            bool probe = groups, question = mine;
            int stop_n = 0;
            for (int k = 0, f0 = groups ? lead : 0; k < p.n_nu;) {
                const int cnt = p.n_nu - f0;
                double A[G], dt[G];
                int group_fb = 0, group_dr = 0;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    A[g] = 0.0;
                    dt[g] = 0.0;
                }
                if (MLPC) {
                    bool fb, dr;
                    if (NNU == 1) {
                        ms.contribution(p, lds_net, p.nu[nu_base], A[0], dt[0], fb, dr);
                        group_fb = fb;
                        group_dr = dr;
                    } else {
#pragma unroll 1
                        for (int g = 0; g < G && g < cnt; ++g) {
                            double Ag, dg;
                            ms.contribution(p, lds_net, p.nu[nu_base + f0 + g], Ag, dg, fb, dr);
                            group_fb += fb;
                            group_dr += dr;
#pragma unroll
                            for (int k = 0; k < G; ++k) {
                                A[k] = k == g ? Ag : A[k];
                                dt[k] = k == g ? dg : dt[k];
                            }
                        }
                    }
                } else if (has) {
                    if (NNU == 1) {
                        tr.contribution(p, p.nu[nu_base], A[0], dt[0]);
                    } else {
                        double nu[G];
#pragma unroll
                        for (int g = 0; g < G; ++g) nu[g] = g < cnt ? p.nu[nu_base + f0 + g] : 1.0;
                        tr.template contributions<G>(p, nu, cnt, A, dt);
                    }
                }
                if (has) {
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        rec[g] = A[g];
                        rec[G + g] = dt[g];
                    }
                }
                wave_lds_sync();
                if (NNU > FREQ_GROUP && probe) {
                    double t0[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) t0[g] = question && g < cnt ? my_row[f0 + COLS + g] : 0.0;
                    int s = first(), n = 0;
                    bool more = question, opaque = false;
                    while (__ballot(more)) {
                        if (more) {
                            const double* r = ring + s * REC;
                            double t1 = 1e300;
#pragma unroll
                            for (int g = 0; g < G; ++g) {
                                t0[g] = t0[g] + r[G + g];
                                t1 = g < cnt ? ::fmin(t1, t0[g]) : t1;
                            }
                            ++n;
                            opaque = t1 >= p.tau_cutoff;
                            s = link_of(ring, s)[1];
                            more = !opaque && pending() > n && evaluated(s);
                        }
                    }
                    question = question && opaque;
                    if (question) stop_n = n > stop_n ? n : stop_n;
                    wave_lds_sync();
                    const bool none = __ballot(question) == 0ull;
                    if (none && k == 0) {
                        probe = false;   // this evaluation is folded at once
                    } else {
                        if (none) lead = f0;
                        probe = !none && k + G < p.n_nu;
                        k = probe ? k + G : 0;
                        f0 = probe ? (f0 + G < p.n_nu ? f0 + G : 0) : lead;
                        continue;
                    }
                }
                fallback += group_fb;
                dropped += group_dr;
                if (spread) {
                    const int j = lane / G, g = lane % G;
                    const bool on = j < n_rays && g < cnt;
                    const int o = on ? ray_tab[j] : 0;
                    const unsigned oq = __shfl(queued, o, 64);
                    int s = (int)(oq & 255u), left = (int)(oq >> 16 & 255u);
                    double* row = rows + o * ROW + f0 + g;
                    double It = 0.0, t0 = 0.0;
                    if (on) {
                        It = row[0];
                        t0 = row[COLS];
                    }
                    bool more = on;
                    while (__ballot(more)) {
                        if (more) {
                            const double* r = ring + s * REC;
                            It = __builtin_fma((double)attenuation<TT>(t0), r[g], It);
                            t0 = t0 + r[G + g];
                            s = link_of(ring, s)[1];
                            more = --left > 0 && evaluated(s);
                        }
                    }
                    if (on) {
                        row[0] = It;
                        row[COLS] = t0;
                        if (f0 == 0 && g == 0) {
                            ray_next[o] = (unsigned char)s;
                            ray_left[o] = (unsigned char)left;
                        }
                    }
                } else {
                    double* row = my_row + f0;
                    double It[G], t0[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        It[g] = mine && g < cnt ? row[g] : 0.0;
                        t0[g] = mine && g < cnt ? row[COLS + g] : 0.0;
                    }
                    nxt = first();
                    taken = 0;
                    bool more = mine;
                    while (__ballot(more)) {
                        if (more) {
                            const int s = nxt;
                            const double* r = ring + s * REC;
                            nxt = link_of(ring, s)[1];
                            double t1 = 1e300;
#pragma unroll
                            for (int g = 0; g < G; ++g) {
                                It[g] = __builtin_fma((double)attenuation<TT>(t0[g]), r[g], It[g]);
                                t0[g] = t0[g] + r[G + g];
                                t1 = g < cnt ? ::fmin(t1, t0[g]) : t1;
                            }
                            ++taken;
                            more = pending() > taken && evaluated(nxt);
                            // cut-off: with one group, every frequency of the sample is known here
                            if (groups ? question && taken == stop_n : p.tau_cutoff > 0.0 && t1 >= p.tau_cutoff) {
                                stop = s;
                                more = false;
                            }
                        }
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (mine && g < cnt) {
                            row[g] = It[g];
                            row[COLS + g] = t0[g];
                        }
                    }
                }
                wave_lds_sync();
                k += G;
                f0 = f0 + G < p.n_nu ? f0 + G : 0;
            }
            // each ray leaves the folded samples behind; one found opaque stops at that sample: its
            // later ones are dropped, and the counters hold what it took up to there
            if (mine) {
                const int left = spread ? ray_left[lane] : pending() - taken;
                queued = (queued & 0xff00ff00u) | ((unsigned)left << 16) | (unsigned)(spread ? ray_next[lane] : nxt);
                if (stop >= 0) {
                    const unsigned char* l = link_of(ring, stop);
                    const int at = *reinterpret_cast<const int*>(l + REC_STEP - REC_LINK);
                    atomicAdd(p.stats + ST_STEPS, (unsigned long long)(at - steps));   // steps beyond the stop
                    atomicSub(tally, (queued >> 24) - l[2] & 255u);                    // crossings beyond it
                    for (int s = nxt, n = left; n > 0; --n) {
                        unsigned char* d = link_of(ring, s);
                        *d |= DROPPED;
                        s = d[1];
                    }
                    status = RAY_OPAQUE;
                    steps = at;
                    queued &= 0xff000000u;
                }
            }
            bool folded = has;
            if (p.tau_cutoff > 0.0) {
                wave_lds_sync();
                folded = has && !(link_of(ring, slot)[0] & DROPPED);
                c_samples += __popcll(__ballot(folded));
            } else {
                c_samples += n_eval;
            }
            c_zamo += __popcll(__ballot(folded && zamo));
            if (MLPC) {
#pragma unroll
                for (int b = 0; 1 << b <= NNU; ++b) {
                    c_fallback += (unsigned long long)__popcll(__ballot(folded && (fallback >> b & 1))) << b;
                    c_dropped += (unsigned long long)__popcll(__ballot(folded && (dropped >> b & 1))) << b;
                }
            }
            if (p.tau_cutoff > 0.0) {
                const unsigned long long ended = __ballot(status > RAY_RUNNING) & run;
                run &= ~ended;
                wait |= ended;
                adds &= run;   // a ray found opaque at an earlier sample queues no more
            }
            head += n_eval;
            head = head >= SLOTS ? head - SLOTS : head;
            total -= n_eval;
            wave_lds_sync();
        }

        // ------------------------------------------------------------ queue this step's samples
        if (!EACH && __builtin_amdgcn_inverse_ballot_w64(adds)) {
            const int lane = fresh(threadIdx.x & 63);
            int s = head + total + (int)lane_rank(adds);
            s = s >= SLOTS ? s - SLOTS : s;
            double* rec = ring + s * REC;
            put(rec, lane);
            *reinterpret_cast<int*>(link_of(rec) + REC_STEP - REC_LINK) = steps;
            if (pending() > 0)
                link_of(ring, (int)((queued >> 8) & 255u))[1] = (unsigned char)s;
            else
                queued = (queued & 0xff000000u) | (unsigned)s;
            queued = ((queued + 0x10000u) & ~0xff00u) | ((unsigned)s << 8);
        }
        if (!EACH) {
            total += __popcll(adds);
            wave_lds_sync();
        }

        // ------------------------------------------------------------ finished rays
        if (wait != 0ull && (events != 0ull || round)) {
            const bool finished = status > RAY_RUNNING && pending() == 0;
            const unsigned long long done = __ballot(finished);
            const TraceParams& p = fresh_params();
            if (finished) {
                const int lane = fresh(threadIdx.x & 63);
                const double* my_row = row_of(lane);
                const DevJob& J = p.jobs[lane_job[lane]];
                const int pix = lane_pix[lane];
                const long long npix = (long long)J.nx * J.ny;
                double* o = p.out + J.out_base + pix;
                for (int f = 0; f < p.n_nu; ++f) o[f * npix] = (status == RAY_NUMERIC) ? 0.0 : my_row[f];
                if (p.ray_status) p.ray_status[J.pix_base + pix] = status;
                if (p.ray_steps) p.ray_steps[J.pix_base + pix] = steps;
                atomicAdd(tally + status, 1u);
                status = RAY_IDLE;
            }
            wait &= ~done;
            idle_changed = done != 0ull;
        }
    }

    // ------------------------------------------------------------ statistics, one atomic per counter per wave
    wave_lds_sync();
    if (lane == 0) {
        const TraceParams& p = fresh_params();
        unsigned long long rays = 0;
#pragma unroll
        for (int i = RAY_HORIZON; i <= RAY_OPAQUE; ++i) rays += tally[i];
        const unsigned long long st[ST_COUNT] = {rays, c_steps, c_samples, tally[RAY_HORIZON], tally[RAY_ESCAPED],
                                                 tally[RAY_MAXSTEP], tally[0], tally[RAY_NUMERIC], c_fallback, c_zamo,
                                                 tally[RAY_OPAQUE], c_dropped};
#pragma unroll
        for (int i = 0; i < ST_COUNT; ++i)
            if (st[i]) atomicAdd(p.stats + i, st[i]);
    }
}

// Flux density per (job, frequency): the sum of the job's image times the pixel solid angle
// and 1e23 (erg/s/cm^2/Hz -> Jy).  Pass 1: FLUX_SPLIT blocks per (job, frequency), block b
// summing the pixels b * 256 + t + k * 256 * FLUX_SPLIT of every thread t in order and
// combining its threads in a fixed tree.  Pass 2: one thread per (job, frequency) adds the
// FLUX_SPLIT partial sums in order.  The result does not depend on scheduling.

__global__ void __launch_bounds__(256) flux_partial_kernel(const DevJob* jobs, const double* out, double* part,
                                                           int max_nu)
{
    const int b = blockIdx.x % FLUX_SPLIT;
    const int jf = blockIdx.x / FLUX_SPLIT;
    const int job = jf / max_nu, f = jf % max_nu;
    const DevJob& J = jobs[job];
    __shared__ double red[256];
    double s = 0.0;
    if (f < J.n_nu) {
        const long long npix = (long long)J.nx * J.ny;
        const double* img = out + J.out_base + f * npix;
        for (long long i = (long long)b * 256 + threadIdx.x; i < npix; i += 256ll * FLUX_SPLIT) s += img[i];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void flux_final_kernel(const DevJob* jobs, const double* part, const double* pix_sr, double* flux,
                                  int n_jobs, int max_nu)
{
    const int jf = blockIdx.x * blockDim.x + threadIdx.x;
    if (jf >= n_jobs * max_nu) return;
    const int job = jf / max_nu, f = jf % max_nu;
    if (f >= jobs[job].n_nu) return;
    double s = 0.0;
    for (int b = 0; b < FLUX_SPLIT; ++b) s += part[(size_t)jf * FLUX_SPLIT + b];
    flux[jf] = s * pix_sr[job] * 1e23;
}

__global__ void reset_kernel(unsigned long long* ray_counter, unsigned long long first, unsigned long long* stats)
{
    if (threadIdx.x == 0) *ray_counter = first;
    if (threadIdx.x < ST_COUNT) stats[threadIdx.x] = 0ull;
}

// Instantiations: RK4 with every register budget (1, 2 or 3 waves per SIMD), the learned
// closure with 1 or 2, the second-order integrators with 2 or 3; all with the sample ring and with the
// optical-depth-aware step (EACH), whose RK4 kernels hold their registers at 2 waves per SIMD without
// scratch (at 3, tau_step = 0.1, FP32 transfer, ms at 2 and 3: 512^2, one frequency 6.56 6.66, four
// 7.94 8.46; 256^2, 24 frequencies 104.4 107.4).
}  // namespace

int kernel_wpe(int wpe, bool mlpc, int integ, bool each)
{
    if (integ != INTEG_RK4) return wpe >= 3 ? 3 : 2;   // RK2 and Verlet: two or three waves per SIMD
    if (mlpc || each) return wpe >= 2 ? 2 : 1;
    return wpe >= 3 ? 3 : wpe == 2 ? 2 : 1;
}

namespace {

template <int NNU, class TT, bool EACH>
const void* symbol_of(int wpe, bool mlpc, int integ)
{
    const int w = kernel_wpe(wpe, mlpc, integ, EACH);
    if (integ == INTEG_RK2)
        return w == 3 ? (const void*)trace_kernel<NNU, TT, 3, false, INTEG_RK2, EACH>
                      : (const void*)trace_kernel<NNU, TT, 2, false, INTEG_RK2, EACH>;
    if (integ == INTEG_VERLET || integ == INTEG_VERLET_CORR)
        return w == 3 ? (const void*)trace_kernel<NNU, TT, 3, false, INTEG_VERLET, EACH>
                      : (const void*)trace_kernel<NNU, TT, 2, false, INTEG_VERLET, EACH>;
    if (mlpc)
        return w == 2 ? (const void*)trace_kernel<NNU, TT, 2, true, INTEG_RK4, EACH>
                      : (const void*)trace_kernel<NNU, TT, 1, true, INTEG_RK4, EACH>;
    if constexpr (!EACH)
        if (w == 3) return (const void*)trace_kernel<NNU, TT, 3, false, INTEG_RK4, false>;
    return w == 2 ? (const void*)trace_kernel<NNU, TT, 2, false, INTEG_RK4, EACH>
                  : (const void*)trace_kernel<NNU, TT, 1, false, INTEG_RK4, EACH>;
}

template <class TT, bool EACH>
const void* symbol_tt(int max_nu, int wpe, bool mlpc, int integ)
{
    if (max_nu <= 1) return symbol_of<1, TT, EACH>(wpe, mlpc, integ);
    if (max_nu <= 4) return symbol_of<4, TT, EACH>(wpe, mlpc, integ);
    return symbol_of<32, TT, EACH>(wpe, mlpc, integ);
}

}  // namespace

hipError_t launch_reset(unsigned long long* ray_counter, unsigned long long first, unsigned long long* stats,
                        hipStream_t st)
{
    hipLaunchKernelGGL(reset_kernel, dim3(1), dim3(64), 0, st, ray_counter, first, stats);
    return hipGetLastError();
}

hipError_t launch_trace(const TraceParams& p, int max_nu, bool fp32, int wpe, int blocks, int threads, hipStream_t st)
{
    const bool each = p.tau_step > 0.0;
    const void* fn = trace_kernel_symbol(max_nu, fp32, wpe, p.closure >= CL_MLP, p.integrator, each);
    void* args[] = {const_cast<TraceParams*>(&p)};
    return hipLaunchKernel(fn, dim3(blocks), dim3(threads), args,
                           trace_kernel_lds(p.n_nu, wpe, threads, p.closure >= CL_MLP, p.integrator,
                                            p.rays_per_wave, each),
                           st);
}

size_t flux_partials(int n_jobs, int max_nu) { return (size_t)n_jobs * max_nu * FLUX_SPLIT; }

hipError_t launch_flux(const DevJob* jobs, int n_jobs, const double* out, const double* pix_sr, double* part,
                       double* flux, int max_nu, hipStream_t st)
{
    hipLaunchKernelGGL(flux_partial_kernel, dim3(n_jobs * max_nu * FLUX_SPLIT), dim3(256), 0, st, jobs, out, part,
                       max_nu);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int n = n_jobs * max_nu;
    hipLaunchKernelGGL(flux_final_kernel, dim3((n + 255) / 256), dim3(256), 0, st, jobs, part, pix_sr, flux, n_jobs,
                       max_nu);
    return hipGetLastError();
}

// Visit the queue type of the instantiation that trace_kernel_symbol picks for the same arguments.
template <class F>
auto with_queue(int n_nu, int wpe, bool mlpc, int integ, F f)
{
    const int w = kernel_wpe(wpe, mlpc, integ, false);   // with EACH any does: the slots are given
    auto per_w = [&](auto m, auto w) {
        constexpr bool M = decltype(m)::value;
        constexpr int W = decltype(w)::value;
        if (n_nu <= 1) return f(Queue<1, M, W>{});
        if (n_nu <= 4) return f(Queue<4, M, W>{});
        return f(Queue<32, M, W>{});
    };
    auto per = [&](auto m) {
        return w == 3 ? per_w(m, std::integral_constant<int, 3>{})
             : w == 2 ? per_w(m, std::integral_constant<int, 2>{}) : per_w(m, std::integral_constant<int, 1>{});
    };
    return mlpc ? per(std::true_type{}) : per(std::false_type{});
}

bool trace_plan_takes_rays(int max_nu, int wpe, bool mlpc, int integ)
{
    return !mlpc && (max_nu > 4 || (max_nu > 1 && kernel_wpe(wpe, mlpc, integ, false) == 3));
}

int trace_kernel_slots(int n_nu, int wpe, bool mlpc, int integ, int rays, bool each)
{
    if (each) return rays;   // one sample per ray
    return with_queue(n_nu, wpe, mlpc, integ, [&](auto q) { return decltype(q)::slots(rays, n_nu); });
}

size_t trace_kernel_lds(int n_nu, int wpe, int threads, bool mlpc, int integ, int rays, bool each)
{
    const int slots = trace_kernel_slots(n_nu, wpe, mlpc, integ, rays, each);
    const size_t per_wave =
        with_queue(n_nu, wpe, mlpc, integ, [&](auto q) { return decltype(q)::per_wave(rays, slots, n_nu); });
    return (size_t)(threads / 64) * per_wave + (mlpc ? (size_t)mlp::LDS_NET_BYTES : 0);
}

const void* trace_kernel_symbol(int max_nu, bool fp32, int wpe, bool mlpc, int integ, bool each)
{
    if (each)
        return fp32 ? symbol_tt<float, true>(max_nu, wpe, mlpc, integ) : symbol_tt<double, true>(max_nu, wpe, mlpc, integ);
    return fp32 ? symbol_tt<float, false>(max_nu, wpe, mlpc, integ) : symbol_tt<double, false>(max_nu, wpe, mlpc, integ);
}

hipError_t trace_kernel_attributes(int max_nu, bool fp32, int wpe, bool mlpc, int integ, int* vgprs,
                                   int* spill_bytes, int* max_threads)
{
    hipFuncAttributes at;
    const hipError_t e = hipFuncGetAttributes(&at, trace_kernel_symbol(max_nu, fp32, wpe, mlpc, integ));
    if (e != hipSuccess) return e;
    if (vgprs) *vgprs = at.numRegs;
    if (spill_bytes) *spill_bytes = (int)at.localSizeBytes;
    if (max_threads) *max_threads = at.maxThreadsPerBlock;
    return hipSuccess;
}
