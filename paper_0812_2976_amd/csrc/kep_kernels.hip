// gfx950 kernels for batched Keplerian radial-velocity models (Ford 2008).
//
// Dense batches (every system sees the same n_obs observations) use one
// wavefront per system at a time with the 64 lanes spread over observations:
// lane l evaluates observations l, l + 64, ... (NCH chunks held in registers
// for the whole launch), so every parameter a lane needs is wave-uniform and
// the eccentricity schedule of the Kepler solve is uniform across the wave.
// Per-planet constants (reciprocal period, phase offset, amplitudes) are
// computed with the lanes spread over a batch's (planet, system) pairs instead
// and handed over through the wave's slice of LDS, so that setup is paid once
// per system rather than once per lane.
// The chi-square is reduced across the wave in binary64 (Sec. 4.4's final sum).
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "kep_device.h"
#include "kep_internal.h"
#include "kep_grad.h"
#include "kep_policy.h"
#include "kep_root64.h"

namespace kep {

// Residency target of the dense kernels: the mixed-precision variants with up
// to four chunks per lane are held to five wavefronts per SIMD (at most 102
// VGPRs).  With four chunks the compiler would otherwise use 126 VGPRs (four
// wavefronts); the extra wavefront lets the SIMD issue binary32 arithmetic
// from more wavefronts at once: 4% (1,048,576 x 4 x 256, 1.757 against 1.688 ms,
// when the jitter's and the further groups' registers put 52 bytes per lane in
// scratch).  Compiled without them (JIT, the one group that a launch without
// teams has) the four-chunk chi-square keeps 12 bytes there and takes 1.535 ms.
// It issues vector instructions for nearly all of that time.
template <class Pol, int NCH>
constexpr int dense_waves_per_simd()
{
    return NCH > 4 ? 1 : Pol::kMixed ? 5 : Pol::kTables == 2 ? 4 : 1;
}

// The mixed and the default binary64 kernels start the Kepler solve from the
// table of kep_start_tab.h, copied once into each block's LDS behind the
// records; the binary64 ones have the sin/cos knots behind it.

__host__ __device__ inline size_t dense_table_offset(int wpb, int sb, int n_pl, size_t rec_size)
{
    return ((size_t)wpb * sb * n_pl * rec_size + (size_t)wpb * sb * sizeof(int) + 15) & ~(size_t)15;
}

template <class Pol>
constexpr size_t dense_table_bytes()
{
    static_assert(sizeof(kep_start_tab) % 16 == 0, "the knots after the table are 16-byte aligned");
    return (Pol::kTables >= 1 ? sizeof(kep_start_tab) : 0) + (Pol::kTables == 2 ? kSc64Bytes : 0);
}

// k_dense_team: the block's records, every wavefront's sums and the domain flags,
// then the tables.
__host__ __device__ inline size_t team_table_offset(int W, int sb, int n_pl, size_t rec_size)
{
    return ((size_t)sb * n_pl * rec_size + (size_t)W * sb * sizeof(double) + (size_t)sb * sizeof(int) + 15) &
           ~(size_t)15;
}

// JIT: chi-squares with a jitter per system (other modes: false).
template <class Pol, int NCH, int MODE, bool JIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(dense_waves_per_simd<Pol, NCH>())))
k_dense(DenseArgs a)
{
    using Rec = typename Pol::Rec;
    using Obs = typename Pol::Obs;
    using ModelAcc = typename Pol::ModelAcc;
    extern __shared__ __align__(16) unsigned char smem[];

    const int lane = __lane_id();
    const int wpb = blockDim.x >> 6;
    const int wib = uniform_int(threadIdx.x >> 6);
    Rec *recs = reinterpret_cast<Rec *>(smem) + (size_t)wib * a.sb * a.n_pl;
    int *sysbad = reinterpret_cast<int *>(smem + (size_t)wpb * a.sb * a.n_pl * sizeof(Rec)) + wib * a.sb;
    // the block's copies of the starting-value table and the knots after the records
    const uint32_t *tab = nullptr;
    const double2 *knots = nullptr;
    if constexpr (Pol::kTables >= 1) {
        uint32_t *t = reinterpret_cast<uint32_t *>(smem + dense_table_offset(wpb, a.sb, a.n_pl, sizeof(Rec)));
        if constexpr (Pol::kTables == 2) {
            double2 *k = reinterpret_cast<double2 *>(t + kTabWords);
            load_knots64(k);
            knots = k;
        }
        start_table_begin(t);      // arrives while the observations and the first records are made
        tab = t;
    }

    const int64_t gw = (int64_t)blockIdx.x * wpb + wib;
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    // chi-squares with the table hold every observation in one group (more go to
    // k_dense_team); knowing it spares the group loop's registers (four chunks: 48
    // bytes of scratch a lane with it)
    constexpr bool kOne = MODE == kChi2 && Pol::kTables >= 1;
    const int n_groups = kOne ? 1 : (int)((a.n_obs + 64 * NCH - 1) / (64 * NCH));

    constexpr bool MODEL = MODE != kChi2;
    Obs o[NCH];
    auto load_group = [&](int g) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            int64_t k = (int64_t)g * 64 * NCH + c * 64 + lane;
            if (MODE != kChi2) Pol::load_obs_model(a, k, o[c]);
            else Pol::load_obs(a, k, o[c]);
        }
    };
    if (n_groups <= 1) load_group(0);
    bool obs_bad = !MODEL && !JIT && n_groups <= 1 && __any(pol_obs_bad<Pol, NCH>(o));

    // Velocities need no reduction over observations, so their work items are
    // (batch, observation group) pairs: a few systems with very many
    // observations still spread over the whole chip.
    const int64_t n_items = MODEL ? a.bt.n_batches * n_groups : a.bt.n_batches;
    int64_t prev_bt = -1;
    auto make_batch = [&](int64_t s0, int nb) {
        wave_sync_lds();
        if (lane < nb) {
            const int64_t sys = s0 + lane;
            bool ok = isfinite(a.t0);
            if (a.offset) ok = ok && isfinite(a.offset[sys]);
            if (a.jitter) ok = ok && isfinite(a.jitter[sys]) && a.jitter[sys] >= 0.0;
            sysbad[lane] = ok ? 0 : 1;
        }
        wave_sync_lds();
        // planet records with the lanes over the batch's (planet, system) pairs,
        // planet-major (each parameter plane read in one run)
        for (int q = lane; q < nb * a.n_pl; q += 64) {
            const int j = q / nb, sq = q - j * nb;
            const int64_t p = (int64_t)j * a.n_sys + s0 + sq;
            Rec r;
            if (!Pol::setup(a, a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], r)) sysbad[sq] = 1;
            recs[sq * a.n_pl + j] = r;
        }
        wave_sync_lds();
    };
    // The first records are made while the table arrives.  The kernels that write
    // velocities wait for it before the loop, where the wait is passed once: inside,
    // their LDS reads also waited for the stores of the systems before (models of
    // 1,048,576 x 4 x 256 1.68 against 1.55 ms).  The chi-square has no such stores
    // and one copy of the setup in its code (1.54 against 1.61 ms with two).
    bool table_here = Pol::kTables == 0;
    if constexpr (MODEL && Pol::kTables >= 1) {
        if (gw < n_items) {
            int nb;
            prev_bt = gw / n_groups;
            const int64_t s0 = a.bt.first(prev_bt, a.n_sys, nb);
            make_batch(s0, nb);
        }
        start_table_end();
        table_here = true;
    }
    for (int64_t item = gw; item < n_items; item += n_waves) {
        const int64_t bt = MODEL ? item / n_groups : item;
        const int g_first = MODEL ? (int)(item - bt * n_groups) : 0;
        const int g_end = MODEL ? g_first + 1 : n_groups;
        int nb;
        const int64_t s0 = a.bt.first(bt, a.n_sys, nb);
        if (bt != prev_bt) {
            prev_bt = bt;
            make_batch(s0, nb);
        }
        if (!MODEL && !table_here) {
            start_table_end_uncounted();     // (every wavefront passes one, here or after the loop)
            table_here = true;
        }

        for (int s = 0; s < nb; ++s) {
            const int64_t sys = s0 + s;
            const double gam = a.offset ? a.offset[sys] : 0.0;
            const double jit = JIT ? a.jitter[sys] : 0.0;
            const bool sbad = uniform_int(sysbad[s]) != 0;
            typename Pol::ChiAcc chi;
            Pol::chi_init(chi);
            bool bad_obs = false;
            for (int g = g_first; g < g_end; ++g) {
                if (n_groups > 1) {
                    load_group(g);
                    if (!MODEL && !JIT) bad_obs = bad_obs || pol_obs_bad<Pol, NCH>(o);
                }
                if constexpr (MODE == kAnomalies) {
                    // the same solve as the velocities' (so E is the root the model uses)
                    for (int j = 0; j < a.n_pl; ++j) {
                        const Rec &rr = recs[s * a.n_pl + j];
                        float *row = a.dv + ((int64_t)j * a.n_sys + sys) * a.n_obs;
                        float M[NCH], E[NCH], sv[NCH], omc[NCH];
#pragma unroll
                        for (int c = 0; c < NCH; ++c) M[c] = mean_anomaly32(o[c].tt, rr.ph);
                        PolMixed::solve<NCH, false>(rr.k, uniform_int(rr.niter), uniform_int(rr.check) != 0, rr.tp, M,
                                                    E, sv, omc, a.max_iter, tab);
#pragma unroll
                        for (int c = 0; c < NCH; ++c) {
                            if (o[c].in) {
                                const int64_t k = (int64_t)g * 64 * NCH + c * 64 + lane;
                                // streamed out: nontemporal stores (3.5% at c2)
                                __builtin_nontemporal_store((sbad || !o[c].ok) ? __builtin_nanf("") : E[c], row + k);
                            }
                        }
                    }
                    continue;
                }
                ModelAcc m[NCH];
                if (MODE == kPlanets) {
                    for (int j = 0; j < a.n_pl; ++j) {
#pragma unroll
                        for (int c = 0; c < NCH; ++c) Pol::model_init(m[c]);
                        pol_add_planet<Pol, NCH>(recs[s * a.n_pl + j], o, m, a, tab, knots);
                        float *row = a.dv + ((int64_t)j * a.n_sys + sys) * a.n_obs;
#pragma unroll
                        for (int c = 0; c < NCH; ++c) {
                            if (o[c].in) {
                                const int64_t k = (int64_t)g * 64 * NCH + c * 64 + lane;
                                __builtin_nontemporal_store(
                                    (sbad || !o[c].ok) ? __builtin_nanf("") : (float)Pol::model_value(m[c]), row + k);
                            }
                        }
                    }
                    continue;
                }
#pragma unroll
                for (int c = 0; c < NCH; ++c) Pol::model_init(m[c]);
                for (int j = 0; j < a.n_pl; ++j) pol_add_planet<Pol, NCH>(recs[s * a.n_pl + j], o, m, a, tab, knots);
                if (MODEL) {
#pragma unroll
                    for (int c = 0; c < NCH; ++c) {
                        if (o[c].in) {
                            int64_t k = (int64_t)g * 64 * NCH + c * 64 + lane;
                            double val = Pol::model_value(m[c]) + gam;
                            a.out[sys * a.n_obs + k] = (sbad || !o[c].ok) ? __builtin_nan("") : val;
                        }
                    }
                } else {
                    pol_chi_add<Pol, NCH, JIT>(chi, m, o, gam, jit, bad_obs);
                }
            }
            if (!MODEL) {
                double tot = wave_sum(Pol::chi_value(chi));
                const bool bad = sbad || obs_bad || __any(bad_obs);
                if (lane == 0) a.out[sys] = bad ? __builtin_nan("") : tot;
            }
        }
    }
    if (!table_here) start_table_end_uncounted();
}

// Chi-square with several wavefronts over a system's observations: wavefront w of
// a team of W holds groups w, w + W, ... of NCH x 64 observations, the team's
// wavefronts evaluate the same systems, and the block adds their sums in wavefront
// order.  A block of T teams shares the tables and a batch of systems (records
// built by all its threads, systems dealt to the teams in turn).  For two kinds of
// call:
//   - more than 256 observations: one wavefront per system held eight chunks
//     (212 VGPRs, two wavefronts per SIMD, and a whole eight for the last few),
//     or beyond 512 loaded and converted every observation again for every
//     system; here each wavefront keeps its group in registers for the launch (up to
//     16 x 4 x 64 observations), or loads it once per batch;
//   - few systems: a system's observations one wavefront after another leave most
//     SIMDs idle.
// Every observation is evaluated as by k_dense, so results differ from its only
// in the order of the binary64 sums.  Before and after: 60,000 x 4 x 300 257 ->
// 152 us, 30,000 x 4 x 700 262 -> 164, 5,000 x 2 x 5,000 169 -> 105; few systems,
// bound by the launch and one pass of dependent work: 1 x 4 x 1,000 17.4 -> 8.3,
// 16 x 4 x 300 12.4 -> 7.6.
template <class Pol, int NCH, bool JIT>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(dense_waves_per_simd<Pol, NCH>())))
k_dense_team(DenseArgs a, int W)
{
    using Rec = typename Pol::Rec;
    using Obs = typename Pol::Obs;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = __lane_id();
    const int T = uniform_int((int)(blockDim.x >> 6) / W);
    const int team = uniform_int((int)(threadIdx.x >> 6) / W);
    const int w = uniform_int((int)(threadIdx.x >> 6)) - team * W;
    Rec *recs = reinterpret_cast<Rec *>(smem);
    double *part = reinterpret_cast<double *>(recs + (size_t)a.sb * a.n_pl);    // [W][sb]
    int *sysbad = reinterpret_cast<int *>(part + (size_t)W * a.sb);
    uint32_t *tab = reinterpret_cast<uint32_t *>(smem + team_table_offset(W, a.sb, a.n_pl, sizeof(Rec)));
    double2 *knots = nullptr;
    const int n_groups = (int)((a.n_obs + 64 * NCH - 1) / (64 * NCH));

    start_table_begin(tab);
    if constexpr (Pol::kTables == 2) {
        knots = reinterpret_cast<double2 *>(tab + kTabWords);
        load_knots64(knots);
    }
    Obs o[NCH];
    auto load_group = [&](int g) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) Pol::load_obs(a, (int64_t)g * 64 * NCH + c * 64 + lane, o[c]);
    };
    bool obs_bad = false;
    if (n_groups <= W) {
        load_group(w);
        obs_bad = !JIT && __any(pol_obs_bad<Pol, NCH>(o));
    }

    for (int64_t bt = blockIdx.x; bt < a.bt.n_batches; bt += gridDim.x) {
        int nb;
        const int64_t s0 = a.bt.first(bt, a.n_sys, nb);
        __syncthreads();                                   // the previous batch's sums are written out
        for (int q = threadIdx.x; q < nb; q += blockDim.x) {
            const int64_t sys = s0 + q;
            bool ok = isfinite(a.t0);
            if (a.offset) ok = ok && isfinite(a.offset[sys]);
            if (JIT) ok = ok && isfinite(a.jitter[sys]) && a.jitter[sys] >= 0.0;
            sysbad[q] = ok ? 0 : 1;
        }
        __syncthreads();
        for (int q = threadIdx.x; q < nb * a.n_pl; q += blockDim.x) {
            const int j = q / nb, sq = q - j * nb;
            const int64_t p = (int64_t)j * a.n_sys + s0 + sq;
            Rec r;
            if (!Pol::setup(a, a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], r)) sysbad[sq] = 1;
            recs[sq * a.n_pl + j] = r;
        }
        start_table_end();         // (the wait is for the first batch's sake)

        for (int g = w; g < n_groups; g += W) {
            if (n_groups > W) {
                load_group(g);
                obs_bad = !JIT && __any(pol_obs_bad<Pol, NCH>(o));
            }
            for (int s = team; s < nb; s += T) {
                const double gam = a.offset ? a.offset[s0 + s] : 0.0;
                const double jit = JIT ? a.jitter[s0 + s] : 0.0;
                typename Pol::ModelAcc m[NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) Pol::model_init(m[c]);
                for (int j = 0; j < a.n_pl; ++j) pol_add_planet<Pol, NCH>(recs[s * a.n_pl + j], o, m, a, tab, knots);
                typename Pol::ChiAcc chi;
                Pol::chi_init(chi);
                bool bad_obs = false;
                pol_chi_add<Pol, NCH, JIT>(chi, m, o, gam, jit, bad_obs);
                double tot = wave_sum(Pol::chi_value(chi));
                if (obs_bad || __any(bad_obs)) tot = __builtin_nan("");
                if (lane == 0) part[w * a.sb + s] = g == w ? tot : part[w * a.sb + s] + tot;
            }
        }
        __syncthreads();
        for (int q = threadIdx.x; q < nb; q += blockDim.x) {
            double tot = part[q];
            for (int v = 1; v < W; ++v) tot += part[v * a.sb + q];
            a.out[s0 + q] = sysbad[q] != 0 ? __builtin_nan("") : tot;
        }
    }
}

// Second kernel of the separate-function form: planet sums, residuals and the
// chi-square (binary64 sums) from the velocities written by kPlanets.
template <int NCH>
__global__ void __launch_bounds__(256) k_chisq_from_dv(DenseArgs a)
{
    const int lane = __lane_id();
    const int wpb = blockDim.x >> 6;
    const int64_t gw = (int64_t)blockIdx.x * wpb + uniform_int(threadIdx.x >> 6);
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    const bool has_jit = a.jitter != nullptr;
    ObsMixed o[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) PolMixed::load_obs(a, c * 64 + lane, o[c]);
    for (int64_t sys = gw; sys < a.n_sys; sys += n_waves) {
        const double gam = a.offset ? a.offset[sys] : 0.0;
        const double jit = a.jitter ? a.jitter[sys] : 0.0;
        bool bad = !isfinite(a.t0) || (a.offset && !isfinite(gam)) || (has_jit && !(isfinite(jit) && jit >= 0.0));
        PolMixed::ModelAcc m[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) PolMixed::model_init(m[c]);
        // every planet's row is requested before the first is summed (one row at a
        // time left too few bytes in flight to fill HBM); the sum keeps planet order
        float dv[kMaxPl][NCH];
#pragma unroll
        for (int j = 0; j < kMaxPl; ++j) {
            if (j < a.n_pl) {
                const float *row = a.dv + ((int64_t)j * a.n_sys + sys) * a.n_obs;
#pragma unroll
                for (int c = 0; c < NCH; ++c)  // read once: nontemporal loads (4% at c2)
                    dv[j][c] = o[c].in ? __builtin_nontemporal_load(row + c * 64 + lane) : 0.0f;
            }
        }
#pragma unroll
        for (int j = 0; j < kMaxPl; ++j) {
            if (j < a.n_pl) {
#pragma unroll
                for (int c = 0; c < NCH; ++c) m[c].add(dv[j][c]);
            }
        }
        PolMixed::ChiAcc chi;
        PolMixed::chi_init(chi);
        bool bad_obs = false;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (o[c].in) {
                bool okw = PolMixed::chi_add(chi, m[c], o[c], gam, jit, has_jit);
                bad_obs = bad_obs || !okw || !o[c].ok;
            }
        }
        const double tot = wave_sum(PolMixed::chi_value(chi));
        bad = bad || __any(bad_obs);
        if (lane == 0) a.out[sys] = bad ? __builtin_nan("") : tot;
    }
}

// ------------------------------------------------------------------ Kepler only
// Standalone Kepler solve (the paper's Kepler-only mode): one lane per pair.
// M is reduced to [-pi, pi] with 2 pi as a double-double; the root is returned
// on the input's branch.  kKepMixed: from the starting-value table (the block's
// LDS copy) and one quartic step where e <= KEP_TAB_EMAX, else the schedule;
// kKepRoot64: that binary32 value corrected in binary64 (kep_root64.h);
// kKepDanby64: Danby's plain binary64 iteration (fixed_iter != 0).
enum { kKepDanby64 = 0, kKepMixed = 1, kKepRoot64 = 2 };

// ANY: every finite M; else |M| < kOneTurnStep (ok: such an M, and e in the domain).
template <int KIND, bool ANY>
__device__ __forceinline__ double kepler_one(double M, double e, int fixed, int max_iter, const uint32_t *tab,
                                             const double2 *knots, bool &ok)
{
    ok = (ANY ? isfinite(M) : fabs(M) < kOneTurnStep) && e >= 0.0 && e < 1.0;
    // from 2^54 on e sin E is less than half a unit in the last place of M: E rounds to M
    const bool whole = ANY && fabs(M) >= 0x1p54;
    const double M_in = M;
    if (!ok || whole) { M = 0.0; e = 0.0; }
    double kq, k2, Mr;
    if constexpr (ANY) {
        Mr = centre_turns(M, kq, k2);
    } else {
        kq = rint(M * kInvTwoPi);
        Mr = fma(-kq, kTwoPiHi, M);
        Mr = fma(-kq, kTwoPiLo, Mr);
    }
    double E;
    if (KIND == kKepDanby64) {
        E = kepler64(Mr, e, Mr >= 0.0 ? 1.0 : -1.0, fixed, max_iter);
    } else {
        const Ecc32 k = make_ecc32(e);
        const int niter = fixed > 0 ? fixed : sched32(k.e);
        const TabPlace tp = table_place(e, fixed <= 0);
        float sE, omcE;   // unused here: the standalone solve returns E only
        const float E32 = kepler32_start((float)Mr, k, tp, tab, niter, max_iter, fixed > 0, sE, omcE);
        E = (double)E32;
        if (KIND == kKepRoot64) {
            Root64 r;
            refine_root64(e, E32, Mr, tp.toff < 0, knots, r);
            E = r.E;
        }
    }
    if constexpr (ANY) {
        E = fma(k2, kTwoPiHi, E);
        E = fma(k2, kTwoPiLo, E);
    }
    E = fma(kq, kTwoPiHi, E);
    E = fma(kq, kTwoPiLo, E);
    return !ok ? __builtin_nan("") : whole ? M_in : E;
}

// Each thread takes KU pairs per tile (KU x blockDim consecutive pairs per
// block), issuing all of their loads before solving, so that more memory
// requests are in flight than one pair per thread would allow.
template <int KIND, int KU>
__global__ void __launch_bounds__(256) k_kepler(const double *__restrict__ Mv, const double *__restrict__ ev,
                                               double *__restrict__ Ev, int64_t n, int fixed, int max_iter)
{
    const uint32_t *tab = nullptr;
    const double2 *knots = nullptr;
    if constexpr (KIND != kKepDanby64) {
        __shared__ __align__(16) uint32_t tab_s[kTabWords];    // Kepler starting values
        start_table_begin(tab_s);
        tab = tab_s;
        if constexpr (KIND == kKepRoot64) {
            __shared__ double2 knots_s[kSc64Knots];
            load_knots64(knots_s);
            knots = knots_s;
        }
        start_table_end();
    }
    const int64_t tile = (int64_t)blockDim.x * KU;
    const int64_t stride = (int64_t)gridDim.x * tile;
    for (int64_t base = (int64_t)blockIdx.x * tile + threadIdx.x; base < n; base += stride) {
        double M[KU], e[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int64_t i = base + (int64_t)u * blockDim.x;
            // streamed once: nontemporal loads and stores (2^26 pairs: 4.74 -> 5.07 TB/s)
            M[u] = i < n ? __builtin_nontemporal_load(Mv + i) : 0.0;
            e[u] = i < n ? __builtin_nontemporal_load(ev + i) : 0.0;
        }
        bool all_ok = true;
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int64_t i = base + (int64_t)u * blockDim.x;
            bool ok;
            const double E = kepler_one<KIND, false>(M[u], e[u], fixed, max_iter, tab, knots, ok);
            all_ok = all_ok && ok;
            if (i < n) __builtin_nontemporal_store(E, Ev + i);
        }
        // Then the pairs with a large M, through the general reduction (in the loop above
        // it would cost 3 to 5%: 2^26 pairs mixed 298 against 306 us, binary64 331 against
        // 351)
        if (__any(!all_ok)) {
#pragma nounroll
            for (int u = 0; u < KU; ++u) {
                const int64_t i = base + (int64_t)u * blockDim.x;
                if (i < n && fabs(Mv[i]) >= kOneTurnStep) {
                    bool ok;
                    Ev[i] = kepler_one<KIND, true>(Mv[i], ev[i], fixed, max_iter, tab, knots, ok);
                }
            }
        }
    }
}

// ------------------------------------------------------------------ ragged
// Persistent kernel over CSR systems.  Work items are runs of `sb` systems of
// the plan's work order (decreasing work, grouped by planet count within
// short windows); each wavefront takes the next item from an atomic counter
// until the items run out.  Setup runs with the lanes over the item's (system, planet) pairs.
// Each system's whole groups of 64 observations are evaluated one system at a
// time with the lanes over its observations (uniform planet records, groups
// of up to 4 x 64 loaded with coalesced reads).  The remaining n_obs mod 64
// observations of all the item's systems are then packed back to back into
// one stream of lanes, each lane with its own system's planet records, and a
// segmented scan over each group of 64 lanes returns every system's share: a
// system's last partial group no longer leaves the rest of its wavefront idle.
// Observations of one unit of a system's whole groups (up to G groups of 64),
// as loaded.
template <int G>
struct RawObs {
    double t[G], v[G], s[G];
};

template <int G>
__device__ __forceinline__ void load_unit(const RaggedArgs &a, int64_t k0, int64_t left, RawObs<G> &r)
{
    const int lane = __lane_id();
#pragma unroll
    for (int c = 0; c < G; ++c) {
        const int64_t k = c * 64 + lane;
        const bool in = k < left;
        // read once per launch: nontemporal loads (c3 0.593-0.598 -> 0.588 ms)
        r.t[c] = in ? __builtin_nontemporal_load(a.t + k0 + k) : a.t0;
        r.v[c] = in ? __builtin_nontemporal_load(a.v + k0 + k) : 0.0;
        r.s[c] = in ? __builtin_nontemporal_load(a.sigma + k0 + k) : 1.0;
    }
}

// One unit (the first NCH of its groups) of a system's whole groups, with the
// lanes over its observations and uniform planet records.
template <int NCH, int G, bool JIT>
__device__ __forceinline__ void ragged_unit(const RaggedArgs &a, const RecMixed *recs, int npl, const RawObs<G> &r,
                                            int64_t left, double gam, double jit, PolMixed::ChiAcc &chi,
                                            bool &bad_obs, const uint32_t *tab)
{
    const int lane = __lane_id();
    ObsMixed o[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        o[c].in = c * 64 + lane < left;
        o[c].ok = isfinite(r.t[c]) && isfinite(r.v[c]) && isfinite(r.s[c]) && r.s[c] >= 0.0;
        o[c].tt = r.t[c] - a.t0;
        o[c].v = r.v[c];
        o[c].s2 = (float)(r.s[c] * r.s[c]);
        o[c].w = rcp32(o[c].s2);
    }
    PolMixed::ModelAcc m[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) PolMixed::model_init(m[c]);
    // (before the planets, so that sigma^2 need not be held for them)
    if constexpr (!JIT) bad_obs = bad_obs || pol_obs_bad<PolMixed, NCH>(o);
    for (int j = 0; j < npl; ++j) PolMixed::add_planet<NCH>(recs[j], o, m, a.max_iter, 0, tab);
    pol_chi_add<PolMixed, NCH, JIT>(chi, m, o, gam, jit, bad_obs);
}

// One planet's velocity (the arithmetic of PolMixed::add_planet) from this
// lane's own planet record: lanes of different systems differ in step count.
__device__ __forceinline__ float ragged_vel_lane(const RecMixed &r, double tt, int max_iter, const uint32_t *tab)
{
    const float M = mean_anomaly32(tt, r.ph);
    float s, omc;
    kepler32_start(M, r.k, r.tp, tab, r.niter, max_iter, r.check != 0, s, omc);
    const float D = fmaf(r.k.e, omc, r.k.ome);           // 1 - e cos E
    const float num = fmaf(r.B, s, fmaf(-r.A, omc, r.A));  // A cos E + B sin E
    return num * rcp32(D);
}

// LDS of one wavefront for sb systems: planet records [sb][kMaxPl]; per
// system the first planet offset, the global index of its first tail
// observation and its chi-square so far; its first observation and the
// length of its whole groups [sb] each; its offset and jitter [sb][2];
// (code, system) pairs [sb][2], where code is the planet count, negative for
// an invalid system; per-planet domain flags [sb][kMaxPl]; prefix sums of the
// tail lengths [sb + 1]; bad-data flags [sb].
// With COOP one such slice serves a block, which adds each wavefront's share of
// the systems' chi-square [sb] after it.
__host__ __device__ inline size_t ragged_lds_per_wave(int sb)
{
    const size_t b = (size_t)sb * kMaxPl * sizeof(RecMixed) + (size_t)sb * 2 * sizeof(int64_t) +
                     (size_t)sb * sizeof(double) + (size_t)sb * 2 * sizeof(int64_t) + (size_t)sb * 2 * sizeof(double) +
                     (size_t)sb * 2 * sizeof(int) + (size_t)sb * kMaxPl * sizeof(int) +
                     (size_t)(sb + 1) * sizeof(int) + (size_t)sb * sizeof(int);
    return (b + 15) & ~(size_t)15;
}

__device__ __forceinline__ int64_t uniform_i64(int64_t x)
{
    const int lo = __builtin_amdgcn_readfirstlane((int)(x & 0xffffffff));
    const int hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
    return ((int64_t)hi << 32) | (uint32_t)lo;
}

// GMAX: largest observation group in 64-lane chunks (2 or 4): fewer chunks in
// flight need fewer registers and allow more resident waves; the plan's
// autotuner picks it.  Five wavefronts per SIMD with two chunks (96 VGPRs, 16
// bytes of scratch), four with four (128 VGPRs, 72 bytes): at c3 the four-chunk
// form at four wavefronts runs 3% faster than the two-chunk one at four.
//
// COOP: a block takes an item, not a wavefront: its wavefronts build the item's
// records together, take its units and its tail groups in turn, each keeping its
// own sums, which are added in wavefront order at the end.  For batches of fewer
// items than the chip has wavefronts (30,011 systems in items of 16: 1,876
// items), where one wavefront per item left most of the chip idle for as long as
// the largest item takes.  The evaluations are the same: units, and groups of 64
// tail lanes, hold the same observations in either form.
template <int GMAX, bool COOP, bool JIT>
__global__ void __launch_bounds__(COOP ? 1024 : 256) __attribute__((amdgpu_waves_per_eu(GMAX == 2 ? 5 : 4)))
k_ragged_mixed(RaggedArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = __lane_id();
    const int wib = uniform_int(threadIdx.x >> 6);
    const int wpb = blockDim.x >> 6;
    const int sb = a.sb;
    // the threads that share an item: tid of nthr
    const int tid = COOP ? (int)threadIdx.x : lane, nthr = COOP ? (int)blockDim.x : 64;
    auto sync_item = [] {
        if constexpr (COOP) __syncthreads();
        else wave_sync_lds();
    };
    unsigned char *mine = smem + (COOP ? 0 : (size_t)wib * ragged_lds_per_wave(sb));
    RecMixed *recs = reinterpret_cast<RecMixed *>(mine);
    int64_t *pofs = reinterpret_cast<int64_t *>(recs + sb * kMaxPl);
    int64_t *tail0 = pofs + sb;
    double *acc0 = reinterpret_cast<double *>(tail0 + sb);
    int64_t *obs0 = reinterpret_cast<int64_t *>(acc0 + sb);
    int64_t *nfl = obs0 + sb;
    double *gj = reinterpret_cast<double *>(nfl + sb);
    int *meta = reinterpret_cast<int *>(gj + 2 * sb);
    int *okpl = meta + 2 * sb;
    int *tpre = okpl + sb * kMaxPl;
    int *bad = tpre + sb + 1;
    // this wavefront's sums: the slice's own, or one of the block's wavefronts'
    double *acc = COOP ? reinterpret_cast<double *>(smem + ragged_lds_per_wave(sb)) + wib * sb : acc0;
    __shared__ __align__(16) uint32_t tab[kTabWords];    // Kepler starting values
    __shared__ unsigned int drained;       // bit q: a wave of this block found queue q drained
    __shared__ unsigned int waves_out;     // the block's waves that have left the item loop
    if (threadIdx.x == 0) {
        drained = 0u;
        waves_out = 0u;
    }
    load_start_table(tab);                 // (its barrier also orders the stores above)

    // this block's XCD queue first (blocks go to the XCDs round-robin), then the
    // others.  Device-scope atomics on one address complete one after another, so
    // probes of a drained queue delay the takes still to come: a wave that finds a
    // queue drained marks it in the block's LDS, and the block's other waves skip it
    // (c3: 0.611 -> 0.599 ms together with the block-level exit count below).
    const int home = (int)(blockIdx.x % kRaggedQueues);
    int tried = 0;
    bool first_item = true;
    __shared__ int64_t taken;              // COOP: the block's item
    for (;;) {
        int64_t item = -1;
        if constexpr (COOP) {
            // block b's first item is b; items past the grid come from one counter
            // (a probe of eight drained queues, one after another, was 8 us of a
            // launch of 28)
            if (!first_item && (int64_t)gridDim.x >= a.n_items) break;
            __syncthreads();                          // every wavefront is done with the previous item
            if (threadIdx.x == 0)
                taken = first_item ? (int64_t)blockIdx.x
                                   : (int64_t)gridDim.x + (int64_t)atomicAdd(a.queue, 1u);
            first_item = false;
            __syncthreads();
            item = uniform_i64(taken);
            if (item >= a.n_items) item = -1;
        }
        while (!COOP && tried < kRaggedQueues) {      // uniform: every lane takes part in the shuffle
            const int q = (home + tried) % kRaggedQueues;
            // a relaxed read: a mark not yet seen costs one more probe, nothing else
            const unsigned int seen = __hip_atomic_load(&drained, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if ((uniform_int((int)seen) >> q) & 1) {
                ++tried;
                continue;
            }
            unsigned int k = 0;
            if (lane == 0) k = atomicAdd(a.queue + q * kQueueStride, 1u);
            k = (unsigned int)uniform_int(__shfl((int)k, 0, 64));
            const int64_t it = (int64_t)k * kRaggedQueues + q;
            if (it < a.n_items) {
                item = it;
                break;
            }
            if (lane == 0) atomicOr(&drained, 1u << q);
            ++tried;
        }
        if (item < 0) break;
        const int64_t i0 = item * sb;
        const int nb = (int)min((int64_t)sb, a.n_sys - i0);
        wave_sync_lds();
        int rem = 0;
        // (COOP: every wavefront reads them for the prefix sums, the first one writes)
        if (lane < nb) {
            const int32_t code = a.order[i0 + lane];
            if (COOP && wib != 0) {
                if (code >= 0) rem = (int)((a.obs_off[code + 1] - a.obs_off[code]) & 63);
            } else if (code >= 0) {
                const int64_t sys = code;
                const int64_t p0 = a.pl_off[sys];
                const int64_t o0 = a.obs_off[sys], n = a.obs_off[sys + 1] - o0;
                // the system's offset and jitter with its offsets, not behind the
                // planet parameters (one dependent round trip fewer per item)
                gj[2 * lane] = a.offset ? a.offset[sys] : 0.0;
                gj[2 * lane + 1] = JIT ? a.jitter[sys] : 0.0;
                meta[2 * lane] = (int)(a.pl_off[sys + 1] - p0);
                meta[2 * lane + 1] = (int)sys;
                pofs[lane] = p0;
                rem = (int)(n & 63);
                tail0[lane] = o0 + (n - rem);
                obs0[lane] = o0;
                nfl[lane] = n - rem;
            } else {
                // a system whose offsets failed the on-device check (-1 - index):
                // its offsets are not read again and its chi-square is NaN
                meta[2 * lane] = 0;
                meta[2 * lane + 1] = -1 - code;
                gj[2 * lane] = 0.0;
                gj[2 * lane + 1] = 0.0;
                pofs[lane] = 0;
                tail0[lane] = 0;
                obs0[lane] = 0;
                nfl[lane] = 0;
            }
            acc[lane] = 0.0;
            if (!COOP || wib == 0) bad[lane] = 0;
        }
        // prefix sums of the tail lengths over the item's systems
        int incl = rem;
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(incl, d, 64);
            if (lane >= d) incl += u;
        }
        if (!COOP || wib == 0) {
            if (lane < nb) tpre[lane + 1] = incl;
            if (lane == 0) tpre[0] = 0;
        }
        const int ntail = uniform_int(__shfl(incl, nb - 1, 64));
        sync_item();
        DenseArgs dummy;
        dummy.fixed_iter = a.fixed_iter;
        for (int q = tid; q < nb * kMaxPl; q += nthr) {
            const int s = q / kMaxPl, j = q - s * kMaxPl;
            if (j < meta[2 * s]) {
                const int64_t p = pofs[s] + j;
                RecMixed r;
                okpl[q] = PolMixed::setup(dummy, a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], r) ? 1 : 0;
                recs[q] = r;
            }
        }
        sync_item();
        if (lane < nb && (!COOP || wib == 0)) {
            const int npl = meta[2 * lane];
            bool ok = isfinite(a.t0) && npl >= 1 && npl <= kMaxPl;
            for (int j = 0; j < kMaxPl; ++j)
                if (j < npl) ok = ok && okpl[lane * kMaxPl + j] != 0;
            const double g = gj[2 * lane], sj = gj[2 * lane + 1];
            if (a.offset) ok = ok && isfinite(g);
            if (JIT) ok = ok && isfinite(sj) && sj >= 0.0;
            meta[2 * lane] = ok ? npl : -npl;
        }
        sync_item();
        // whole groups of 64 observations, one system at a time, in units of up to
        // GMAX groups.  Each unit's observations are loaded when it starts: the
        // other resident wavefronts cover the wait, and loading the next unit's
        // ahead (registers for two units) cost a wavefront per SIMD, 3% at c3.
        {
            auto has_units = [&](int q) { return uniform_int(meta[2 * q]) > 0 && uniform_i64(nfl[q]) > 0; };
            int us = 0, turn = 0;                        // COOP: units go to the wavefronts in turn
            while (us < nb && !has_units(us)) ++us;
            int64_t ug = 0;
            RawObs<GMAX> cur;
            PolMixed::ChiAcc chi;
            PolMixed::chi_init(chi);
            bool bad_obs = false;
            while (us < nb) {
                const int64_t nf = uniform_i64(nfl[us]);
                int ns = us;
                int64_t ng = ug + 64 * GMAX;
                if (ng >= nf) {
                    ns = us + 1;
                    while (ns < nb && !has_units(ns)) ++ns;
                    ng = 0;
                }
                const bool my_turn = !COOP || turn == wib;
                if (COOP && ++turn == wpb) turn = 0;
                if (!my_turn && ns == us) {
                    ug = ng;
                    continue;
                }
                if (my_turn) {
                load_unit<GMAX>(a, uniform_i64(obs0[us]) + ug, nf - ug, cur);
                const int64_t left = nf - ug;
                const int code = uniform_int(meta[2 * us]);
                const double gam = gj[2 * us], jit = gj[2 * us + 1];
                const RecMixed *rs = recs + us * kMaxPl;
                if (left <= 64) ragged_unit<1, GMAX, JIT>(a, rs, code, cur, left, gam, jit, chi, bad_obs, tab);
                else if (GMAX == 2 || left <= 128)
                    ragged_unit<2, GMAX, JIT>(a, rs, code, cur, left, gam, jit, chi, bad_obs, tab);
                else if (left <= 192) ragged_unit<3, GMAX, JIT>(a, rs, code, cur, left, gam, jit, chi, bad_obs, tab);
                else ragged_unit<GMAX, GMAX, JIT>(a, rs, code, cur, left, gam, jit, chi, bad_obs, tab);
                }
                if (ns != us) {
                    const double tot = wave_sum(PolMixed::chi_value(chi));
                    const bool b = __any(bad_obs);
                    if (lane == 0) {
                        acc[us] = tot;
                        if (b) bad[us] = 1;             // every writer stores the same value
                    }
                    PolMixed::chi_init(chi);
                    bad_obs = false;
                }
                us = ns;
                ug = ng;
            }
        }
        wave_sync_lds();
        // the packed tails: lane position p of the stream belongs to system s
        // with tpre[s] <= p < tpre[s + 1].  Positions only grow along the
        // stream, so each lane moves its system cursor forward; the next
        // group's observations are loaded before the current group is
        // evaluated.
        if (ntail > 0) {
            int s = 0;
            auto seek = [&](int pos) {
                while (s + 1 < nb && tpre[s + 1] <= pos) ++s;
            };
            auto fetch = [&](int pos, bool in, double &t, double &v, double &sg) {
                t = a.t0;
                v = 0.0;
                sg = 1.0;
                if (in && meta[2 * s] > 0) {
                    const int64_t k = tail0[s] + (pos - tpre[s]);
                    t = __builtin_nontemporal_load(a.t + k);
                    v = __builtin_nontemporal_load(a.v + k);
                    sg = __builtin_nontemporal_load(a.sigma + k);
                }
            };
            const int first = COOP ? 64 * wib : 0, step = COOP ? 64 * wpb : 64;
            bool in = first + lane < ntail;
            int pp = in ? first + lane : ntail - 1;
            seek(pp);
            double t, v, sg;
            fetch(pp, in, t, v, sg);
            for (int c0 = first; c0 < ntail; c0 += step) {
                const int sc = s;
                const bool inc = in;
                const double tc = t, vc = v, sgc = sg;
                if (c0 + step < ntail) {                // next group: cursor and loads
                    in = c0 + step + lane < ntail;
                    pp = in ? c0 + step + lane : ntail - 1;
                    seek(pp);
                    fetch(pp, in, t, v, sg);
                }
                const int code = meta[2 * sc];
                const int npl = inc && code > 0 ? code : 0;
                double x = 0.0;
                if (npl > 0) {
                    ObsMixed o;
                    o.in = true;
                    o.ok = isfinite(tc) && isfinite(vc) && isfinite(sgc) && sgc >= 0.0;
                    o.tt = tc - a.t0;
                    o.v = vc;
                    o.s2 = (float)(sgc * sgc);
                    o.w = rcp32(o.s2);
                    PolMixed::ModelAcc m;
                    PolMixed::model_init(m);
                    const RecMixed *rs = recs + sc * kMaxPl;
                    for (int j = 0; j < npl; ++j) m.add(ragged_vel_lane(rs[j], o.tt, a.max_iter, tab));
                    const double gam = gj[2 * sc], jit = gj[2 * sc + 1];
                    PolMixed::ChiAcc cx;
                    PolMixed::chi_init(cx);
                    bool okw;
                    if constexpr (JIT) {
                        okw = PolMixed::chi_add(cx, m, o, gam, jit, true) && o.ok;
                    } else {
                        okw = PolMixed::obs_valid(o);
                        PolMixed::chi_add_plain(cx, m, o, gam);
                    }
                    x = PolMixed::chi_value(cx);
                    if (!okw) bad[sc] = 1;              // every writer stores the same value
                }
                // segmented scan: a lane adds only partial sums that start inside
                // its own system's run of lanes (from `head`), so the lane that
                // ends the run holds that system's share of this group, and a
                // non-finite value stays within its own system
                const int head = max(tpre[sc] - c0, 0);
                const int last = min(tpre[sc + 1] - c0, 64) - 1;
                double sum = x;
                for (int d = 1; d < 64; d <<= 1) {
                    const double u = __shfl_up(sum, d, 64);
                    if (lane - d >= head) sum += u;
                }
                if (inc && lane == last && code > 0) acc[sc] += sum;
                wave_sync_lds();
            }
        }
        if constexpr (COOP) __syncthreads();
        if (lane < nb && (!COOP || wib == 0)) {
            const int code = meta[2 * lane];
            double tot = acc[lane];
            if constexpr (COOP)
                for (int w = 1; w < wpb; ++w) tot += acc[w * sb + lane];
            a.out[meta[2 * lane + 1]] = (code <= 0 || bad[lane] != 0) ? __builtin_nan("") : tot;
        }
    }
    // The last wave to leave resets the counters for the next launch, so no
    // reset launch is needed between launches: every wave counts itself out
    // after its last (failed) take from the queue, the last of a block counts
    // the block out (one global atomic per block, not per wave: 0.627 -> 0.611
    // ms at c3), so when the count reaches the number of blocks no wave of this
    // launch touches the queue again.
    if (COOP && (int64_t)gridDim.x >= a.n_items) return;     // the queue was not used
    if (lane == 0 && atomicAdd(&waves_out, 1u) == (blockDim.x >> 6) - 1) {
        if (atomicAdd(a.queue + kQueueDone, 1u) == gridDim.x - 1) {
            for (int q = 0; q < kRaggedQueues; ++q) atomicExch(a.queue + q * kQueueStride, 0u);
            atomicExch(a.queue + kQueueDone, 0u);
        }
    }
}

// ------------------------------------------------------- ragged, no allocation
// Device memory of the allocation-free ragged entry point: the work-queue
// and exit counters in the first 2 KiB, the blocks' counts of systems per planet
// count, then the int32 work order of up to kStaticMaxSys systems.  One copy per
// GPU, kept until the process ends; every call on a GPU shares it (calls that
// overlap in time on one GPU race).
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// The work order: systems by decreasing planet count (so that the systems of a
// work item share their planet count), index order within a count (a stable
// counting sort: the order, and so every result, is the same on every call), the
// systems whose CSR offsets fail the check (0 <= o0 <= o1 <= n_obs_total,
// 0 <= p0 < p1 <= n_pl_total, p1 - p0 <= kMaxPl) last as -1 - index.
//
// Two launches of one block per kPrepTile systems: the first checks the offsets
// and counts the tile's systems per key (and zeroes the queue counters), the
// second sums the counts before its tile and places its systems.  Within a tile
// the lanes read consecutive systems; ballots rank them.  One block that walked
// all systems twice, each thread over a run of its own, took 93 us at 30,011
// systems (strided 8-byte reads, one load in flight per thread): more than half
// of the whole call.
// Up to kStaticOneTile systems a single block of 1,024 threads does both (one
// launch of 5 us instead of two).
constexpr int kPrepThreads = 256;
constexpr int kPrepKeys = kMaxPl + 1;      // planet counts 8 .. 1, then rejected systems
constexpr int kPrepRounds = kStaticTile / kPrepThreads;
constexpr int kOneThreads = 1024, kOneRounds = 8;
constexpr int64_t kStaticOneTile = kOneThreads * kOneRounds;
static_assert(kStaticCountBytes == (size_t)kPrepKeys * kStaticMaxTiles * sizeof(int), "counts fill their area");

struct StaticOrderArgs {
    const int64_t *obs_off, *pl_off;
    int64_t n_sys, n_obs_total, n_pl_total;
    int n_tiles;
    int *counts;               // [kPrepKeys][n_tiles]
    int32_t *order;
    unsigned int *queue;
};

// Key of system i: 0 for 8 planets ... 7 for one, 8 rejected.
__device__ __forceinline__ int static_key(const StaticOrderArgs &a, int64_t i)
{
    const int64_t o0 = a.obs_off[i], o1 = a.obs_off[i + 1], p0 = a.pl_off[i], p1 = a.pl_off[i + 1];
    const bool ok = o0 >= 0 && o0 <= o1 && o1 <= a.n_obs_total && p0 >= 0 && p0 < p1 && p1 <= a.n_pl_total &&
                    p1 - p0 <= kMaxPl;
    return ok ? kMaxPl - (int)(p1 - p0) : kMaxPl;
}

// The keys of this thread's ROUNDS systems (-1 past the last), and in LDS how
// many of each key every (round, wavefront) segment of the block's tile of
// THREADS x ROUNDS systems holds.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void static_tile_keys(const StaticOrderArgs &a, int (&key)[ROUNDS], int (*seg)[kPrepKeys])
{
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * (THREADS * ROUNDS);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = base + r * THREADS + threadIdx.x;
        key[r] = i < a.n_sys ? static_key(a, i) : -1;
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        int n = 0;
#pragma unroll
        for (int k = 0; k < kPrepKeys; ++k) {
            const int c = __popcll(__ballot(key[r] == k));
            n = lane == k ? c : n;
        }
        if (lane < kPrepKeys) seg[r * (THREADS / 64) + w][lane] = n;
    }
    __syncthreads();
}

__global__ void __launch_bounds__(kPrepThreads) k_ragged_static_count(StaticOrderArgs a)
{
    constexpr int kSegs = kStaticTile / 64;
    __shared__ int seg[kSegs][kPrepKeys];
    int key[kPrepRounds];
    if (blockIdx.x == 0)
        for (int q = threadIdx.x; q < kQueueWords; q += kPrepThreads) a.queue[q] = 0u;
    static_tile_keys<kPrepThreads, kPrepRounds>(a, key, seg);
    if (threadIdx.x < kPrepKeys) {
        int n = 0;
        for (int q = 0; q < kSegs; ++q) n += seg[q][threadIdx.x];
        a.counts[threadIdx.x * a.n_tiles + blockIdx.x] = n;
    }
}

// ONE: a single tile, whose own counts are all there are (no counting launch).
template <int THREADS, int ROUNDS, bool ONE>
__global__ void __launch_bounds__(THREADS) k_ragged_static_place(StaticOrderArgs a)
{
    constexpr int kWaves = THREADS / 64, kSegs = ROUNDS * kWaves;
    __shared__ int seg[kSegs][kPrepKeys];
    __shared__ int tot[kPrepKeys], before[kPrepKeys];
    const int lane = __lane_id(), w = threadIdx.x >> 6, tile = blockIdx.x;
    int key[ROUNDS];
    if constexpr (ONE) {
        for (int q = threadIdx.x; q < kQueueWords; q += THREADS) a.queue[q] = 0u;
    } else {
        // each key's count over all tiles and over the tiles before this one
        for (int k = w; k < kPrepKeys; k += kWaves) {
            int t = 0, b = 0;
            for (int q = lane; q < a.n_tiles; q += 64) {
                const int c = a.counts[k * a.n_tiles + q];
                t += c;
                b += q < tile ? c : 0;
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                t += __shfl_xor(t, o, 64);
                b += __shfl_xor(b, o, 64);
            }
            if (lane == 0) {
                tot[k] = t;
                before[k] = b;
            }
        }
    }
    static_tile_keys<THREADS, ROUNDS>(a, key, seg);
    // every (segment, key)'s first slot within the key, in place of its count: one
    // wavefront per key, lanes over the segments
    for (int k = w; k < kPrepKeys; k += kWaves) {
        int carry = 0;
        for (int q0 = 0; q0 < kSegs; q0 += 64) {
            const int n = q0 + lane < kSegs ? seg[q0 + lane][k] : 0;
            int incl = n;
            for (int d = 1; d < 64; d <<= 1) {
                const int u = __shfl_up(incl, d, 64);
                if (lane >= d) incl += u;
            }
            if (q0 + lane < kSegs) seg[q0 + lane][k] = carry + incl - n;
            carry += __shfl(incl, 63, 64);
        }
        if (ONE && lane == 0) {
            tot[k] = carry;
            before[k] = 0;
        }
    }
    __syncthreads();
    const uint64_t below_me = (1ull << lane) - 1ull;
    int base[kPrepKeys];                       // first slot of this tile's systems of each key
#pragma unroll
    for (int k = 0, sum = 0; k < kPrepKeys; ++k) {
        base[k] = sum + before[k];
        sum += tot[k];
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = (int64_t)tile * (THREADS * ROUNDS) + r * THREADS + threadIdx.x;
        uint64_t same = 0;
        int slot = 0;
#pragma unroll
        for (int k = 0; k < kPrepKeys; ++k) {
            const uint64_t m = __ballot(key[r] == k);
            same = key[r] == k ? m : same;
            slot = key[r] == k ? base[k] : slot;
        }
        if (key[r] >= 0) {
            slot += seg[r * kWaves + w][key[r]] + __popcll(same & below_me);
            a.order[slot] = key[r] < kMaxPl ? (int32_t)i : (int32_t)(-1 - i);
        }
    }
}

// The scratch array's device address on each GPU (host code must not use the
// array's name: on the host it is a stand-in, not a device address).
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[64];

hipError_t static_scratch(void **ptr)
{
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return err;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

static size_t ragged_coop_lds(int block, int sb);

// One block per item (k_ragged_mixed's COOP form, two-chunk units: five blocks a
// CU where four-chunk units leave four; 30,011 systems 69 -> 64 us).  Eight
// wavefronts a block while two blocks a CU hold every item, else four (32 items:
// 25 against 35 us, 501: 29 against 38, 1,876: 84 against 64).
static hipError_t launch_ragged_coop(RaggedArgs a, LaunchShape shape, hipStream_t st)
{
    a.gmax = 2;
    const int block = shape.block > 0 ? shape.block : a.n_items <= 2 * (int64_t)device_cu_count() ? 512 : 256;
    const size_t lds = ragged_coop_lds(block, a.sb);
    int per_cu = shape.blocks_per_cu;
    void (*kern)(RaggedArgs) = a.jitter ? k_ragged_mixed<2, true, true> : k_ragged_mixed<2, true, false>;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)kern, block, lds);
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    const int grid = (int)(a.n_items < cap ? a.n_items : cap);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_ragged_static(RaggedArgs a, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0) return hipSuccess;
    if (a.n_sys > kStaticMaxSys) return hipErrorInvalidValue;
    void *base = nullptr;
    hipError_t err = static_scratch(&base);
    if (err != hipSuccess) return err;
    unsigned char *area = reinterpret_cast<unsigned char *>(base);
    unsigned int *queue = reinterpret_cast<unsigned int *>(area);
    int32_t *order = reinterpret_cast<int32_t *>(area + kStaticQueueBytes + kStaticCountBytes);
    StaticOrderArgs o;
    o.obs_off = a.obs_off;
    o.pl_off = a.pl_off;
    o.n_sys = a.n_sys;
    o.n_obs_total = a.n_obs_total;
    o.n_pl_total = a.n_pl_total;
    o.n_tiles = (int)((a.n_sys + kStaticTile - 1) / kStaticTile);
    o.counts = reinterpret_cast<int *>(area + kStaticQueueBytes);
    o.order = order;
    o.queue = queue;
    if (a.n_sys <= kStaticOneTile) {
        hipLaunchKernelGGL((k_ragged_static_place<kOneThreads, kOneRounds, true>), dim3(1), dim3(kOneThreads), 0, st, o);
    } else {
        hipLaunchKernelGGL(k_ragged_static_count, dim3(o.n_tiles), dim3(kPrepThreads), 0, st, o);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL((k_ragged_static_place<kPrepThreads, kPrepRounds, false>), dim3(o.n_tiles),
                           dim3(kPrepThreads), 0, st, o);
    }
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    a.order = order;
    a.queue = queue;
    a.n_items = (a.n_sys + a.sb - 1) / a.sb;
    const int wpb = (shape.block > 0 ? shape.block : 256) / 64;
    const int64_t cap = ragged_max_grid(shape, a.sb, a.gmax);
    // a block per item up to two items for every three resident wavefronts (256
    // threads, items of 16: 30,011 systems 84 against 111 us a call, 65,536 systems
    // 144 against 134, 262,144 systems 721 against 644)
    if (wpb > 1 && 3 * a.n_items < 2 * cap * wpb) return launch_ragged_coop(a, shape, st);
    const int64_t need = (a.n_items + wpb - 1) / wpb;
    const int grid = (int)(need < cap ? need : cap);
    return launch_ragged(a, shape, grid, st);
}

// ------------------------------------------------------------------ launchers
static int g_cu_count = 0;

int device_cu_count()
{
    if (g_cu_count == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
        g_cu_count = cus;
    }
    return g_cu_count;
}

// Occupancy per (device, kernel, block size, LDS bytes), looked up once: the
// runtime query costs microseconds, as much as a small launch.
int cached_occupancy(const void *kern, int block, size_t lds)
{
    struct Entry { int dev; const void *kern; int block; size_t lds; int occ; };
    static std::mutex mu;
    static std::vector<Entry> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    {
        std::lock_guard<std::mutex> lock(mu);
        for (const Entry &e : cache)
            if (e.dev == dev && e.kern == kern && e.block == block && e.lds == lds) return e.occ;
    }
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, block, lds) != hipSuccess || occ <= 0) occ = 1;
    std::lock_guard<std::mutex> lock(mu);
    if (cache.size() < 4096) cache.push_back(Entry{dev, kern, block, lds, occ});
    return occ;
}

hipError_t launch_kepler_solve(const double *M, const double *e, double *E, int64_t n, Prec prec, int fixed_iter,
                               int max_iter, LaunchShape shape, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int block = shape.block > 0 ? shape.block : 256;
    const int per_cu = shape.blocks_per_cu > 0 ? shape.blocks_per_cu : 8 * (256 / block);
    constexpr int KU = 4;
    const int64_t need = (n + (int64_t)block * KU - 1) / ((int64_t)block * KU);
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    const int grid = (int)(need < cap ? need : cap);
    if (prec == Prec::Mixed)
        hipLaunchKernelGGL((k_kepler<kKepMixed, KU>), dim3(grid), dim3(block), 0, st, M, e, E, n, fixed_iter, max_iter);
    else if (fixed_iter == 0)
        hipLaunchKernelGGL((k_kepler<kKepRoot64, KU>), dim3(grid), dim3(block), 0, st, M, e, E, n, 0, max_iter);
    else
        hipLaunchKernelGGL((k_kepler<kKepDanby64, KU>), dim3(grid), dim3(block), 0, st, M, e, E, n,
                           fixed_iter < 0 ? 0 : fixed_iter, max_iter);
    return hipGetLastError();
}

// How many chunks a wavefront takes (NCH) and how many wavefronts share a
// system's observations (W): the least of rounds x instructions x the time each
// takes.  A wavefront's instructions per system are about 62 a planet and chunk,
// 25 a planet, 10 a chunk and 45 more (the mixed kernel's; the proportions are
// what matters); a SIMD issues for its wavefronts in turn, and a lone one at half
// that rate.  Large batches get the NCH that fits n_obs with the fewest empty
// chunks (157 observations: three, not four), small ones more wavefronts per
// system.
DenseSplit dense_split(int64_t n_sys, int n_pl, int64_t n_obs, int most)
{
    const int64_t need = n_obs > 64 ? (n_obs + 63) / 64 : 1;
    const double simds = 4.0 * device_cu_count();
    DenseSplit best{most, 1};
    double best_cost = 0.0;
    for (int nch = most; nch >= 1; --nch) {
        const int64_t groups = (need + nch - 1) / nch;
        const int W = (int)(groups < 16 ? groups : 16);
        const double instr = n_pl * (62.0 * nch + 25.0) + 10.0 * nch + 45.0;
        const double cost = (double)((groups + W - 1) / W) * instr * fmax(2.0, (double)n_sys * W / simds);
        if (nch == most || cost < best_cost) {
            best = DenseSplit{nch, W};
            best_cost = cost;
        }
    }
    return best;
}

template <class Pol, bool JIT>
static hipError_t launch_dense_team(DenseArgs a, DenseSplit split, LaunchShape shape, hipStream_t st)
{
    int W = shape.block > 0 ? shape.block / 64 : split.W;
    const int64_t groups = (a.n_obs + 64 * split.nch - 1) / (64 * split.nch);
    if (W > groups) W = (int)(groups > 0 ? groups : 1);
    auto lds_of = [&](int64_t sb) {
        return team_table_offset(W, (int)sb, a.n_pl, sizeof(typename Pol::Rec)) + dense_table_bytes<Pol>();
    };
    // teams per block: four wavefronts share the tables (two teams of two: one team
    // left no room for records, 60,000 x 4 x 300 256 us against 152; two teams of
    // three, six wavefronts on four SIMDs, 30,000 x 4 x 700 228 against 162), unless
    // the systems do not fill the chip that way or the caller's blocks are smaller.
    // Systems per batch: the blocks that the registers allow (four or five
    // wavefronts per SIMD) share a CU's LDS, at most sixteen systems a team (whole
    // 128-byte lines of the parameter planes)
    const int64_t cus = device_cu_count();
    const int T = W <= 2 && (shape.block > 0 ? shape.block >= 256 : a.n_sys >= 8 * cus) ? 4 / W : 1;
    int blocks = 4 * dense_waves_per_simd<Pol, 4>() / (T * W);
    blocks = blocks > 8 ? 8 : blocks;
    int64_t sb_cap = 16 * T;
    while (sb_cap > 1 && (int64_t)lds_of(sb_cap) > lds_budget(blocks > 1 ? blocks : 1)) --sb_cap;
    void (*kern)(DenseArgs, int) = split.nch == 1   ? k_dense_team<Pol, 1, JIT>
                                   : split.nch == 2 ? k_dense_team<Pol, 2, JIT>
                                   : split.nch == 3 ? k_dense_team<Pol, 3, JIT>
                                                    : k_dense_team<Pol, 4, JIT>;
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)kern, 64 * T * W, lds_of(sb_cap));
    const int64_t cap = cus * per_cu;
    // a multiple of T systems keeps the teams level
    a.bt = make_batches(a.n_sys, cap, sb_cap, T);
    a.sb = a.bt.sb;
    const int64_t grid = a.bt.n_batches < cap ? a.bt.n_batches : cap;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * T * W), lds_of(a.sb), st, a, W);
    return hipGetLastError();
}

template <class Pol, int MODE, bool JIT>
static hipError_t launch_dense_jit(DenseArgs a, LaunchShape shape, hipStream_t st)
{
    const int block = shape.block > 0 ? shape.block : 256;
    const int wpb = block / 64;
    const size_t rec_bytes = (size_t)wpb * a.n_pl * sizeof(typename Pol::Rec) + (size_t)wpb * sizeof(int);
    constexpr bool table = Pol::kTables >= 1;
    auto lds_of = [&](int64_t sb) {
        return table ? dense_table_offset(wpb, (int)sb, a.n_pl, sizeof(typename Pol::Rec)) + dense_table_bytes<Pol>()
                     : rec_bytes * (size_t)sb;
    };
    // systems per setup batch: at most kMaxSB and at most 48 KiB of LDS per block
    // (with the table, five blocks of four wavefronts share a CU's LDS; with the
    // knots too, four)
    const int64_t budget = table ? lds_budget(Pol::kTables == 2 ? 4 : 5) - (int64_t)dense_table_bytes<Pol>() - 16
                                 : (int64_t)(48 * 1024);
    int64_t sb_cap = budget / (int64_t)rec_bytes;
    sb_cap = sb_cap < 1 ? 1 : (sb_cap > kMaxSB ? kMaxSB : sb_cap);
    // a multiple of 16 systems reads whole 128-byte lines of every parameter plane:
    // a line split between two batches may be fetched by two XCDs' L2s
    if (sb_cap > 16) sb_cap &= ~(int64_t)15;
    size_t lds = lds_of(sb_cap);
    const int64_t need = a.n_obs > 64 ? (a.n_obs + 63) / 64 : 1;
    void (*kern)(DenseArgs);
    int nch;
    if constexpr (table) {
        // one to four chunks a lane (velocities of more observations go out in equal
        // groups of at most four, each a work item)
        const int64_t groups = (need + 3) / 4;
        nch = (int)((need + groups - 1) / groups);
        if constexpr (MODE == kChi2) {
            const DenseSplit split = dense_split(a.n_sys, a.n_pl, a.n_obs, 4);
            if (groups > 1 || (split.W > 1 && shape.block == 0)) return launch_dense_team<Pol, JIT>(a, split, shape, st);
        }
        kern = nch == 1   ? k_dense<Pol, 1, MODE, JIT>
               : nch == 2 ? k_dense<Pol, 2, MODE, JIT>
               : nch == 3 ? k_dense<Pol, 3, MODE, JIT>
                          : k_dense<Pol, 4, MODE, JIT>;
    } else {
        nch = need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 8;
        kern = nch == 1   ? k_dense<Pol, 1, MODE, JIT>
               : nch == 2 ? k_dense<Pol, 2, MODE, JIT>
               : nch == 4 ? k_dense<Pol, 4, MODE, JIT>
                          : k_dense<Pol, 8, MODE, JIT>;
    }
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) {
        per_cu = cached_occupancy((const void *)kern, block, lds);
    }
    const int64_t n_groups = (a.n_obs + 64 * nch - 1) / (64 * nch);
    const int64_t workers = (int64_t)device_cu_count() * per_cu * wpb;
    a.bt = make_batches(a.n_sys, workers, sb_cap);
    if (MODE != kChi2) {
        // equal batches, an item for each of a batch's groups: what bounds these is the
        // streaming of their results, which a partly filled last round does not slow,
        // while a round of smaller batches sets up more often (400,000 x 2 x 128
        // anomalies 142 against 136 us)
        const int64_t share = workers / (n_groups > 0 ? n_groups : 1), w = share > 0 ? share : 1;
        int64_t sb = (a.n_sys + w - 1) / w;
        sb = sb < 1 ? 1 : sb > sb_cap ? sb_cap : sb;
        const int64_t n = (a.n_sys + sb - 1) / sb;
        a.bt = Batches{(int)sb, (int)sb, n, n};
    }
    a.sb = a.bt.sb;
    lds = lds_of(a.sb);
    const int64_t n_batches = a.bt.n_batches;
    const int64_t n_items = MODE != kChi2 ? n_batches * (n_groups > 0 ? n_groups : 1) : n_batches;
    int64_t grid = (n_items + wpb - 1) / wpb;
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    if (grid > cap) grid = cap;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(block), lds, st, a);
    return hipGetLastError();
}

template <class Pol, int MODE>
static hipError_t launch_dense_t(DenseArgs a, LaunchShape shape, hipStream_t st)
{
    if constexpr (MODE == kChi2)
        if (a.jitter) return launch_dense_jit<Pol, MODE, true>(a, shape, st);
    return launch_dense_jit<Pol, MODE, false>(a, shape, st);
}

hipError_t launch_dense(DenseArgs a, Prec prec, bool model, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0) return hipSuccess;
    if (model && a.n_obs <= 0) return hipSuccess;
    if (prec == Prec::Mixed)
        return model ? launch_dense_t<PolMixed, kModel>(a, shape, st) : launch_dense_t<PolMixed, kChi2>(a, shape, st);
    if (a.fixed_iter == 0)
        return model ? launch_dense_t<Pol64R, kModel>(a, shape, st) : launch_dense_t<Pol64R, kChi2>(a, shape, st);
    return model ? launch_dense_t<Pol64, kModel>(a, shape, st) : launch_dense_t<Pol64, kChi2>(a, shape, st);
}

hipError_t launch_planet_velocities(DenseArgs a, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0 || a.n_obs <= 0) return hipSuccess;
    return launch_dense_t<PolMixed, kPlanets>(a, shape, st);
}

hipError_t launch_eccentric_anomalies(DenseArgs a, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0 || a.n_obs <= 0) return hipSuccess;
    return launch_dense_t<PolMixed, kAnomalies>(a, shape, st);
}

hipError_t launch_chisq_from_velocities(DenseArgs a, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0) return hipSuccess;
    const int block = shape.block > 0 ? shape.block : 256;
    const int wpb = block / 64;
    const int nch_needed = (int)((a.n_obs + 63) / 64);
    void (*kern)(DenseArgs);
    if (nch_needed <= 1) kern = k_chisq_from_dv<1>;
    else if (nch_needed <= 2) kern = k_chisq_from_dv<2>;
    else if (nch_needed <= 4) kern = k_chisq_from_dv<4>;
    else if (nch_needed <= 8) kern = k_chisq_from_dv<8>;
    else if (nch_needed <= 16) kern = k_chisq_from_dv<16>;
    else return hipErrorInvalidValue;
    const int per_cu = shape.blocks_per_cu > 0 ? shape.blocks_per_cu : 8;
    int64_t grid = (a.n_sys + wpb - 1) / wpb;
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(block), 0, st, a);
    return hipGetLastError();
}

}  // namespace kep

namespace kep {

static size_t ragged_lds(int block, int sb)
{
    return (size_t)(block / 64) * ragged_lds_per_wave(sb);
}

static size_t ragged_coop_lds(int block, int sb)
{
    return ragged_lds_per_wave(sb) + (size_t)(block / 64) * sb * sizeof(double);
}

// The block's LDS is the waves' dynamic slices plus the static copy of the
// Kepler starting-value table and the block's two queue words (16 bytes
// allowed for them and their alignment).
bool ragged_shape_fits(int block, int sb) { return ragged_lds(block, sb) + sizeof(kep_start_tab) + 16 <= 64 * 1024; }

int ragged_max_grid(LaunchShape shape, int sb, int gmax)
{
    const int block = shape.block > 0 ? shape.block : 256;
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) {
        void (*kern)(RaggedArgs) = gmax == 2 ? k_ragged_mixed<2, false, true> : k_ragged_mixed<4, false, true>;
        per_cu = cached_occupancy((const void *)kern, block, ragged_lds(block, sb));
    }
    return device_cu_count() * per_cu;
}

hipError_t launch_ragged(RaggedArgs a, LaunchShape shape, int grid, hipStream_t st)
{
    const int block = shape.block > 0 ? shape.block : 256;
    void (*kern)(RaggedArgs) = a.gmax == 2 ? (a.jitter ? k_ragged_mixed<2, false, true> : k_ragged_mixed<2, false, false>)
                                           : (a.jitter ? k_ragged_mixed<4, false, true> : k_ragged_mixed<4, false, false>);
    hipLaunchKernelGGL(kern, dim3(grid > 0 ? grid : 1), dim3(block), ragged_lds(block, a.sb), st, a);
    return hipGetLastError();
}

}  // namespace kep
