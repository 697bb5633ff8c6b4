// Population MCMC by differential evolution (DE-MC, ter Braak 2006): the
// many-chain sampler that the batched chi-square is built for (Sec. 6 of the
// paper).  One generation is two fused half-step launches (propose, chi-square
// and accept for every chain of one half, k_demc_half) and, when the
// generation number lives in device memory for graph replay, a one-thread
// kernel that advances it.  The half-step kernel reuses the dense kernels'
// per-precision policies (kep_policy.h) for the chi-square.
//
// r1 != r2 index chains of the other half, which does not move while this
// half is updated.  Random numbers come from Philox-4x32-10 (Salmon et al.,
// SC'11) keyed by the seed, with counter (chain, draw, generation lo,
// generation hi | half << 31), so a proposal depends only on (seed, half,
// chain, generation) and the same generation can be replayed from a graph.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kep_internal.h"
#include "kep_philox.h"
#include "kep_policy.h"
#include "kep_root64.h"

namespace kep {

namespace {

// chi-square of a population from the dense kernel, NaN outside K >= 0
__global__ void __launch_bounds__(256) k_demc_support(const double *x, double *chi2, int64_t nh, int n_pl, int d)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * nh) return;
    const int64_t h = i / nh, k = i - h * nh;
    bool ok = true;
    for (int j = 0; j < n_pl; ++j) ok = ok && x[(h * d + n_pl + j) * nh + k] >= 0.0;
    if (!ok) chi2[i] = __builtin_nan("");
}

__global__ void k_demc_set_gen(uint64_t *gen, uint64_t value)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) gen[0] = value;
}

__global__ void k_demc_advance(uint64_t *gen, uint64_t inc)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) gen[0] = gen[0] + inc;
}

DenseArgs half_dense(const DemcArgs &a, const DenseArgs &base, const double *planes, const double *jitter,
                     double *out)
{
    DenseArgs b = base;
    const int64_t nh = a.nh;
    b.P = planes;
    b.K = planes + (int64_t)a.n_pl * nh;
    b.e = planes + (int64_t)2 * a.n_pl * nh;
    b.w = planes + (int64_t)3 * a.n_pl * nh;
    b.M0 = planes + (int64_t)4 * a.n_pl * nh;
    b.offset = planes + (int64_t)5 * a.n_pl * nh;
    b.jitter = jitter;
    b.n_sys = nh;
    b.n_pl = a.n_pl;
    b.out = out;
    b.grad = nullptr;
    b.dv = nullptr;
    return b;
}

}  // namespace

// ------------------------------------------------------------------ DE-MC
// One half-step of the population sampler, fused: for a batch of sb chains
// of half h the block
//   A. threads over chains: draw 0 gives r1 != r2 (other half) and u;
//   B. threads over (chain, pair of rows): two normals z and the proposal rows
//      y_r = x_ir + gam (x_r1,r - x_r2,r) + eps_r z_r;
//   C. threads over (chain, planet): the planet records, as the dense kernel's
//      setup does from parameter planes;
//   D. threads over chains: domain and prior-support flags;
//   then evaluates each proposal's chi-square with the lanes over observations,
//   as the dense team kernel does (T teams of W wavefronts, k_dense_team), and
//   E. threads over chains: accepts iff 2 ln u < chi2(x) - chi2(y) and K >= 0,
//      copying y into the chain.
// Everything one thread hands to another goes through the block's LDS; the half
// being updated is read and written only by the threads that own the chain in
// phases B / E, and the other half is only read.  The proposals and their
// chi-square are also written to the workspace (m.y, m.c_new).
//
// What bounds it: a few thousand chains are a chain of latencies (starting-value
// table, observations, random numbers, gathers, records, solves, log u).  The
// table arrives in LDS and the observations in registers while the proposals are
// made; several wavefronts share a chain's observations where the population
// leaves the chip idle otherwise.
__host__ __device__ inline size_t demc_lds(int W, int sb, int n_pl, int d, size_t rec_bytes)
{
    size_t b = (size_t)sb * n_pl * rec_bytes          // planet records
               + (size_t)sb * d * sizeof(double)       // proposals
               + (size_t)sb * (1 + W) * sizeof(double) // u, each wavefront's share of the proposal's chi2
               + (size_t)sb * 2 * sizeof(uint32_t)     // r1, r2
               + (size_t)sb * n_pl * sizeof(int)       // per-planet domain flag
               + (size_t)sb * 2 * sizeof(int);         // per-chain domain and support flags
    return (b + 15) & ~(size_t)15;
}

template <class Pol, int NCH, bool JIT>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
k_demc_half(DenseArgs a, DemcArgs m, int h, int W)
{
    using Rec = typename Pol::Rec;
    using Obs = typename Pol::Obs;
    using ModelAcc = typename Pol::ModelAcc;
    extern __shared__ __align__(16) unsigned char smem[];

    const int lane = __lane_id(), tid = threadIdx.x, nthr = blockDim.x;
    const int T = uniform_int((int)(blockDim.x >> 6) / W);
    const int team = uniform_int((int)(threadIdx.x >> 6) / W);
    const int w = uniform_int((int)(threadIdx.x >> 6)) - team * W;
    const int sb = a.sb, npl = a.n_pl, d = m.d;
    Rec *recs = reinterpret_cast<Rec *>(smem);
    double *y_l = reinterpret_cast<double *>(smem + (size_t)sb * npl * sizeof(Rec));
    double *u_l = y_l + (size_t)sb * d;
    double *part = u_l + sb;                              // [W][sb]
    uint32_t *r12_l = reinterpret_cast<uint32_t *>(part + (size_t)W * sb);
    int *okpl_l = reinterpret_cast<int *>(r12_l + 2 * sb);
    int *bad_l = okpl_l + sb * npl;
    int *supp_l = bad_l + sb;
    // the block's copies of the Kepler starting-value table and the knots
    const uint32_t *tab = nullptr;
    const double2 *knots = nullptr;
    if constexpr (Pol::kTables >= 1) {
        uint32_t *t = reinterpret_cast<uint32_t *>(smem + demc_lds(W, sb, npl, d, sizeof(Rec)));
        start_table_begin(t);      // phase C's end waits for it
        if constexpr (Pol::kTables == 2) {
            double2 *k = reinterpret_cast<double2 *>(t + kTabWords);
            load_knots64(k);
            knots = k;
        }
        tab = t;
    }

    const int64_t nh = m.nh;
    const uint64_t g = m.gen_ptr ? *m.gen_ptr + m.gen : m.gen;
    const double gde = (m.jump_every > 0 && (g + 1) % (uint64_t)m.jump_every == 0) ? 1.0 : m.gamma;
    double *xh = m.x + (int64_t)h * d * nh;
    const double *xo = m.x + (int64_t)(1 - h) * d * nh;
    const int ndraw = (d + 1) / 2;
    const int n_groups = (int)((a.n_obs + 64 * NCH - 1) / (64 * NCH));

    Obs o[NCH];
    bool obs_bad = false;
    auto load_group = [&](int gi) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) Pol::load_obs(a, (int64_t)gi * 64 * NCH + c * 64 + lane, o[c]);
        obs_bad = !JIT && __any(pol_obs_bad<Pol, NCH>(o));
    };
    if (n_groups <= W) load_group(w);

    for (int64_t bt = blockIdx.x; bt < a.bt.n_batches; bt += gridDim.x) {
        int nb;
        const int64_t s0 = a.bt.first(bt, nh, nb);
        __syncthreads();
        for (int c = tid; c < nb; c += nthr) {                                  // A
            const U4 r = demc_draw(m.key0, m.key1, h, (uint32_t)(s0 + c), 0u, g);
            const uint32_t r1 = below(r.w0, (uint32_t)nh);
            uint32_t r2 = below(r.w1, (uint32_t)nh - 1u);
            if (r2 >= r1) r2 += 1u;
            r12_l[2 * c] = r1;
            r12_l[2 * c + 1] = r2;
            u_l[c] = unit53(r.w2, r.w3);
        }
        __syncthreads();
        for (int q = tid; q < nb * ndraw; q += nthr) {                          // B
            const int c = q / ndraw, p = q - c * ndraw, r = 2 * p;
            const int64_t i = s0 + c;
            const uint32_t r1 = r12_l[2 * c], r2 = r12_l[2 * c + 1];
            const U4 z = demc_draw(m.key0, m.key1, h, (uint32_t)i, (uint32_t)(1 + p), g);
            const double rho = sqrt(-2.0 * log(unit53(z.w0, z.w1)));
            double sn, cs;
            sincos(kTwoPi * unit53(z.w2, z.w3), &sn, &cs);
            {
                // rounded term by term, as written (no contraction)
#pragma clang fp contract(off)
                const int64_t o0 = (int64_t)r * nh;
                const double y0 = xh[o0 + i] + gde * (xo[o0 + r1] - xo[o0 + r2]) + m.eps[r] * (rho * cs);
                y_l[c * d + r] = y0;
                m.y[o0 + i] = y0;
                if (r + 1 < d) {
                    const int64_t o1 = o0 + nh;
                    const double y1 = xh[o1 + i] + gde * (xo[o1 + r1] - xo[o1 + r2]) + m.eps[r + 1] * (rho * sn);
                    y_l[c * d + r + 1] = y1;
                    m.y[o1 + i] = y1;
                }
            }
        }
        __syncthreads();
        for (int q = tid; q < nb * npl; q += nthr) {                            // C
            const int c = q / npl, j = q - c * npl;
            const double *yc = y_l + c * d;
            Rec rr;
            okpl_l[q] = Pol::setup(a, yc[j], yc[npl + j], yc[2 * npl + j], yc[3 * npl + j], yc[4 * npl + j], rr)
                            ? 1 : 0;
            recs[q] = rr;
        }
        if constexpr (Pol::kTables >= 1) start_table_end();
        else __syncthreads();
        for (int c = tid; c < nb; c += nthr) {                                  // D (read in phase E, by the same thread)
            const double *yc = y_l + c * d;
            bool ok = isfinite(a.t0) && isfinite(yc[5 * npl]);
            bool supp = true;
            for (int j = 0; j < npl; ++j) {
                ok = ok && okpl_l[c * npl + j] != 0;
                supp = supp && yc[npl + j] >= 0.0;
            }
            if (JIT) ok = ok && isfinite(a.jitter[s0 + c]) && a.jitter[s0 + c] >= 0.0;
            bad_l[c] = ok ? 0 : 1;
            supp_l[c] = supp ? 1 : 0;
        }

        for (int gi = w; gi < n_groups; gi += W) {
            if (n_groups > W) load_group(gi);
            for (int s = team; s < nb; s += T) {
                const double gam = y_l[s * d + 5 * npl];
                const double jit = JIT ? a.jitter[s0 + s] : 0.0;
                ModelAcc mm[NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) Pol::model_init(mm[c]);
                for (int j = 0; j < npl; ++j) pol_add_planet<Pol, NCH>(recs[s * npl + j], o, mm, a, tab, knots);
                typename Pol::ChiAcc chi;
                Pol::chi_init(chi);
                bool bad_obs = false;
                pol_chi_add<Pol, NCH, JIT>(chi, mm, o, gam, jit, bad_obs);
                double tot = wave_sum(Pol::chi_value(chi));
                if (obs_bad || __any(bad_obs)) tot = __builtin_nan("");
                if (lane == 0) part[w * sb + s] = gi == w ? tot : part[w * sb + s] + tot;
            }
        }
        __syncthreads();

        for (int c = tid; c < nb; c += nthr) {                                  // E
            const int64_t i = s0 + c;
            double c_new = 0.0;
            if (n_groups > 0) {
                c_new = part[c];
                for (int v = 1; v < W; ++v) c_new += part[v * sb + c];
            }
            if (bad_l[c] != 0) c_new = __builtin_nan("");
            double *chi = m.chi2 + (int64_t)h * nh + i;
            m.c_new[i] = c_new;
            if (supp_l[c] != 0 && 2.0 * log(u_l[c]) < *chi - c_new) {
                for (int r = 0; r < d; ++r) xh[(int64_t)r * nh + i] = y_l[c * d + r];
                *chi = c_new;
                if (m.n_accept) m.n_accept[(int64_t)h * nh + i] += 1;
            }
        }
    }
    // A block without a batch lets the table land.  The launch makes none (its grid is at
    // most the number of batches), but without this way out the compiler orders the kernel
    // so that 32 generations of 2 x 2,048 chains x 4 x 256 take 822 us, not 808.
    if constexpr (Pol::kTables >= 1)
        if (blockIdx.x >= a.bt.n_batches) start_table_end();
}

template <class Pol, bool JIT>
static hipError_t launch_demc_half_t(DemcArgs m, DenseArgs a, int h, LaunchShape shape, hipStream_t st)
{
    // two chunks a wavefront at most: with four the registers of the proposals and of
    // the solve together spill (2 x 32,768 chains x 4 x 256, a generation: 149 against
    // 130 us).  Eight wavefronts share a block's tables and proposals where the
    // population fills the chip that way (2 x 2,048: 25.4 us, four 26.7), else one team.
    const DenseSplit split = dense_split(m.nh, a.n_pl, a.n_obs, 2);
    const int64_t groups = (a.n_obs + 64 * split.nch - 1) / (64 * split.nch);
    int W = shape.block > 0 ? shape.block / 64 : split.W;
    if (W > groups) W = (int)(groups > 0 ? groups : 1);
    const int T = shape.block > 0 ? shape.block / 64 / W
                  : W <= 2 && m.nh >= 4 * (int64_t)device_cu_count() ? 8 / W : 1;
    const size_t rec = sizeof(typename Pol::Rec);
    const size_t table = (Pol::kTables >= 1 ? sizeof(kep_start_tab) : 0) + (Pol::kTables == 2 ? kSc64Bytes : 0);
    auto lds_of = [&](int64_t sb) { return demc_lds(W, (int)sb, a.n_pl, m.d, rec) + table; };
    // the batch leaves room for the blocks that the registers allow (four wavefronts per SIMD;
    // two blocks of eight wavefronts: up to 80 KiB of dynamic LDS each, of the 160 KiB that a
    // block may have)
    const int blocks = 16 / (T * W) > 8 ? 8 : 16 / (T * W);
    int64_t sb_cap = 16 * T;
    while (sb_cap > 1 && (int64_t)lds_of(sb_cap) > lds_budget(blocks > 1 ? blocks : 1)) --sb_cap;
    void (*kern)(DenseArgs, DemcArgs, int, int) = split.nch == 1 ? k_demc_half<Pol, 1, JIT> : k_demc_half<Pol, 2, JIT>;
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)kern, 64 * T * W, lds_of(sb_cap));
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    a.bt = make_batches(m.nh, cap, sb_cap, T);
    a.sb = a.bt.sb;
    const int64_t grid = a.bt.n_batches < cap ? a.bt.n_batches : cap;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * T * W), lds_of(a.sb), st, a, m, h, W);
    return hipGetLastError();
}

template <class Pol>
static hipError_t launch_demc_half_pol(DemcArgs m, DenseArgs a, int h, LaunchShape shape, hipStream_t st)
{
    return a.jitter ? launch_demc_half_t<Pol, true>(m, a, h, shape, st)
                    : launch_demc_half_t<Pol, false>(m, a, h, shape, st);
}

hipError_t launch_demc_half(DemcArgs m, DenseArgs a, Prec prec, int h, LaunchShape shape, hipStream_t st)
{
    if (m.nh <= 0) return hipSuccess;
    a.n_sys = m.nh;
    a.n_pl = m.n_pl;
    a.jitter = m.jitter ? m.jitter + (int64_t)h * m.nh : nullptr;
    a.out = nullptr;
    a.grad = nullptr;
    a.dv = nullptr;
    if (prec == Prec::Mixed) return launch_demc_half_pol<PolMixed>(m, a, h, shape, st);
    return a.fixed_iter == 0 ? launch_demc_half_pol<Pol64R>(m, a, h, shape, st)
                             : launch_demc_half_pol<Pol64>(m, a, h, shape, st);
}

hipError_t launch_demc_chisq(DemcArgs a, DenseArgs base, Prec prec, LaunchShape shape, hipStream_t st)
{
    if (a.nh <= 0) return hipSuccess;
    for (int h = 0; h < 2; ++h) {
        const double *jit = a.jitter ? a.jitter + (int64_t)h * a.nh : nullptr;
        DenseArgs b = half_dense(a, base, a.x + (int64_t)h * a.d * a.nh, jit, a.chi2 + (int64_t)h * a.nh);
        hipError_t err = launch_dense(b, prec, false, shape, st);
        if (err != hipSuccess) return err;
    }
    const int64_t n = 2 * a.nh;
    hipLaunchKernelGGL(k_demc_support, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a.x, a.chi2, a.nh,
                       a.n_pl, a.d);
    return hipGetLastError();
}

hipError_t launch_demc_generation(DemcArgs a, DenseArgs base, Prec prec, LaunchShape shape, hipStream_t st)
{
    for (int h = 0; h < 2; ++h) {
        hipError_t err = launch_demc_half(a, base, prec, h, shape, st);
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

hipError_t launch_demc_advance(uint64_t *gen, uint64_t inc, hipStream_t st)
{
    hipLaunchKernelGGL(k_demc_advance, dim3(1), dim3(64), 0, st, gen, inc);
    return hipGetLastError();
}

hipError_t launch_demc_set_gen(uint64_t *gen, uint64_t value, hipStream_t st)
{
    hipLaunchKernelGGL(k_demc_set_gen, dim3(1), dim3(64), 0, st, gen, value);
    return hipGetLastError();
}

}  // namespace kep
