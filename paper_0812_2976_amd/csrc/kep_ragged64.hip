// Plain binary64 chi-square of a ragged (CSR) batch: the paper's
// double-precision variant (Sec. 5.1, Eq. 1-5) over systems that each have
// their own planet and observation counts.  A wavefront takes batches of up to
// kRag64Batch consecutive positions of the work order (or of the systems in
// their own order when there is none), grid-stride: eight lanes per system read
// its offsets and build its planet records (into the wavefront's LDS slice),
// then the systems are evaluated one at a time with the lanes over the
// observations in groups of up to four 64-lane chunks, every planet as in the
// dense binary64 kernel and the chi-square summed in binary64.
//
// Every system's offsets are checked against the CSR totals before anything
// else of it is read, so the kernel also runs on offsets that no host code has
// checked: a system whose offsets are inconsistent (decreasing, beyond the
// totals, planet count outside [1, kMaxPl]) gets a NaN chi-square and none of
// its arrays is read.
#include <hip/hip_runtime.h>

#include "kep_device.h"
#include "kep_internal.h"
#include "kep_policy.h"
#include "kep_root64.h"

namespace kep {

namespace {

// Systems of a batch: 4 x 8 lanes build their records together, and four
// wavefronts' records and the two tables leave four blocks a CU's 160 KiB.
constexpr int kRag64Batch = 4;

// One group of up to 64 NC observations of a system (starting at index g0 of
// its n): loads, every planet, and the chi-square terms of the lanes in range.
template <class Pol, int NC>
__device__ __forceinline__ void ragged64_group(const RaggedArgs &a, const DenseArgs &d, const typename Pol::Rec *recs,
                                               int npl, int64_t o0, int64_t n, int64_t g0, double gam, double jit,
                                               bool has_jit, const uint32_t *tab, const double2 *knots,
                                               typename Pol::ChiAcc &chi, bool &bad_obs)
{
    const int lane = __lane_id();
    Obs64 o[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t i = g0 + c * 64 + lane;
        o[c].in = i < n;
        const double t = o[c].in ? a.t[o0 + i] : a.t0;
        const double v = o[c].in ? a.v[o0 + i] : 0.0;
        const double s = o[c].in ? a.sigma[o0 + i] : 1.0;
        o[c].ok = isfinite(t) && isfinite(v) && isfinite(s) && s >= 0.0;
        o[c].tt = t - a.t0;
        o[c].v = v;
        o[c].s2 = s * s;
        o[c].w = 1.0 / (s * s);
    }
    typename Pol::ModelAcc m[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) Pol::model_init(m[c]);
    for (int j = 0; j < npl; ++j) pol_add_planet<Pol, NC>(recs[j], o, m, d, tab, knots);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (o[c].in) {
            const bool okw = Pol::chi_add(chi, m[c], o[c], gam, jit, has_jit);
            bad_obs = bad_obs || !okw || !o[c].ok;
        }
    }
}

__device__ __forceinline__ int lane_int(int x, int l) { return __builtin_amdgcn_readlane(x, l); }

__device__ __forceinline__ int64_t lane_i64(int64_t x, int l)
{
    return ((int64_t)lane_int((int)(x >> 32), l) << 32) | (uint32_t)lane_int((int)(x & 0xffffffff), l);
}

__device__ __forceinline__ double lane_f64(double x, int l)
{
    return __longlong_as_double(lane_i64(__double_as_longlong(x), l));
}

template <class Pol>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Pol::kTables == 2 ? 4 : 1)))
k_ragged64(RaggedArgs a)
{
    using Rec = typename Pol::Rec;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = __lane_id();
    const int wpb = blockDim.x >> 6;
    const int wib = uniform_int(threadIdx.x >> 6);
    Rec *recs = reinterpret_cast<Rec *>(smem) + (size_t)wib * a.sb * kMaxPl;
    const uint32_t *tab = nullptr;
    const double2 *knots = nullptr;
    if constexpr (Pol::kTables == 2) {
        __shared__ __align__(16) uint32_t tab_s[kTabWords];
        __shared__ double2 knots_s[kSc64Knots];
        start_table_begin(tab_s);
        load_knots64(knots_s);
        start_table_end();
        tab = tab_s;
        knots = knots_s;
    }
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    const bool has_jit = a.jitter != nullptr;
    const double nan = __builtin_nan("");
    DenseArgs d{};                           // the policies read only the step counts
    d.fixed_iter = a.fixed_iter;
    d.max_iter = a.max_iter;
    const int ls = lane >> 3, lj = lane & 7;

    for (int64_t pos0 = ((int64_t)blockIdx.x * wpb + wib) * a.sb; pos0 < a.n_sys; pos0 += n_waves * a.sb) {
        const int nb = (int)min((int64_t)a.sb, a.n_sys - pos0);
        wave_sync_lds();
        int64_t sys = 0, o0 = 0, n = 0;
        int npl = 0;
        bool bad = true, pok = true;
        double gam = 0.0, jit = 0.0;
        if (ls < nb) {
            sys = pos0 + ls;
            bad = false;
            if (a.order) {
                const int32_t code = a.order[pos0 + ls];
                sys = code >= 0 ? (int64_t)code : -1 - (int64_t)code;   // negative: failed an earlier check
                bad = code < 0;
            }
            o0 = a.obs_off[sys];
            const int64_t o1 = a.obs_off[sys + 1], p0 = a.pl_off[sys], p1 = a.pl_off[sys + 1];
            bad = bad || !(o0 >= 0 && o0 <= o1 && o1 <= a.n_obs_total && p0 >= 0 && p1 - p0 >= 1 &&
                           p1 - p0 <= kMaxPl && p1 <= a.n_pl_total);
            if (!bad) {
                n = o1 - o0;
                npl = (int)(p1 - p0);
                gam = a.offset ? a.offset[sys] : 0.0;
                jit = has_jit ? a.jitter[sys] : 0.0;
                if (lj < npl) {
                    const int64_t p = p0 + lj;
                    Rec r;
                    pok = Pol::setup(d, a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], r);
                    recs[ls * kMaxPl + lj] = r;
                }
                bad = !isfinite(a.t0) || (a.offset && !isfinite(gam)) ||
                      (has_jit && !(isfinite(jit) && jit >= 0.0));
            }
        }
        const uint64_t bads = __ballot(bad || !pok);
        wave_sync_lds();

        for (int s = 0; s < nb; ++s) {
            const int64_t sy = lane_i64(sys, 8 * s);
            if ((bads >> (8 * s)) & 0xff) {
                if (lane == 0) a.out[sy] = nan;
                continue;
            }
            const int64_t so = lane_i64(o0, 8 * s), sn = lane_i64(n, 8 * s);
            const int np = lane_int(npl, 8 * s);
            const double sg = lane_f64(gam, 8 * s), sj = lane_f64(jit, 8 * s);
            const Rec *rs = recs + s * kMaxPl;
            typename Pol::ChiAcc chi;
            Pol::chi_init(chi);
            bool bad_obs = false;
            // groups of four 64-lane chunks; the last takes only the chunks it needs
            for (int64_t g0 = 0; g0 < sn; g0 += 256) {
                const int64_t left = sn - g0;
#define KEP_RAG64(NC) ragged64_group<Pol, NC>(a, d, rs, np, so, sn, g0, sg, sj, has_jit, tab, knots, chi, bad_obs)
                if (left > 192) KEP_RAG64(4);
                else if (left > 128) KEP_RAG64(3);
                else if (left > 64) KEP_RAG64(2);
                else KEP_RAG64(1);
#undef KEP_RAG64
            }
            const double tot = wave_sum(Pol::chi_value(chi));
            const bool b = __any(bad_obs);
            if (lane == 0) a.out[sy] = b ? nan : tot;
        }
    }
}

struct Ragged64Shape {
    int block, sb, grid;
    size_t lds;
};

template <class Pol>
Ragged64Shape ragged64_shape(LaunchShape shape, int64_t n_sys)
{
    Ragged64Shape r;
    r.block = shape.block > 0 ? shape.block : 256;
    const int wpb = r.block / 64;
    auto lds_of = [&](int sb) { return (size_t)wpb * sb * kMaxPl * sizeof(typename Pol::Rec); };
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)k_ragged64<Pol>, r.block, lds_of(kRag64Batch));
    const int64_t cap = (int64_t)device_cu_count() * (per_cu > 0 ? per_cu : 1);
    // the smallest batch that takes no more rounds than the largest would
    const int64_t waves = cap * wpb, rounds = (n_sys + waves * kRag64Batch - 1) / (waves * kRag64Batch);
    r.sb = (int)((n_sys + waves * rounds - 1) / (waves * (rounds > 0 ? rounds : 1)));
    if (r.sb < 1) r.sb = 1;
    int64_t grid = ((n_sys + r.sb - 1) / r.sb + wpb - 1) / wpb;
    r.grid = (int)(grid > cap ? cap : grid < 1 ? 1 : grid);
    r.lds = lds_of(r.sb);
    return r;
}

template <class Pol>
hipError_t launch_ragged64_t(RaggedArgs a, LaunchShape shape, hipStream_t st)
{
    const Ragged64Shape r = ragged64_shape<Pol>(shape, a.n_sys);
    a.sb = r.sb;
    hipLaunchKernelGGL(k_ragged64<Pol>, dim3((unsigned)r.grid), dim3(r.block), r.lds, st, a);
    return hipGetLastError();
}

}  // namespace

int ragged64_grid(LaunchShape shape, int64_t n_sys, int fixed_iter)
{
    return fixed_iter == 0 ? ragged64_shape<Pol64R>(shape, n_sys).grid : ragged64_shape<Pol64>(shape, n_sys).grid;
}

hipError_t launch_ragged64(RaggedArgs a, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0) return hipSuccess;
    const int block = shape.block > 0 ? shape.block : 256;
    if (block % 64 != 0 || block > 256) return hipErrorInvalidValue;
    return a.fixed_iter == 0 ? launch_ragged64_t<Pol64R>(a, shape, st) : launch_ragged64_t<Pol64>(a, shape, st);
}

}  // namespace kep
