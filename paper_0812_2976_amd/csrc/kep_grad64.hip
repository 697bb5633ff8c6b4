// Binary64 chi-square gradient (the implicit-function adjoint, Sec. 6) and the
// Gaussian likelihood with jitter.  One wavefront per system at a time, lanes
// over its observations in groups of NCH x 64, planet records built with the
// lanes over the (planet, system) pairs of a batch, the 5 n_pl + 1 sums kept in
// binary64 per lane over all observations and reduced across the wavefront once
// per system.
//
// Why lanes over observations: with one lane per system, as this kernel's
// predecessor had it, 2,000 systems are 32 wavefronts on 1,024 SIMDs and every
// lane walks all observations one after another (2,000 x 2 x 75: 1.48 ms, of
// which thirty Danby steps a solve were 0.97); here the same batch is 2,000
// wavefronts of one group of two chunks each.  What bounds a large batch is VALU
// issue.
#include <hip/hip_runtime.h>

#include "kep_device.h"
#include "kep_internal.h"
#include "kep_policy.h"
#include "kep_root64.h"

namespace kep {

namespace {

constexpr int pow2_at_least(int n) { return n <= 1 ? 1 : 2 * pow2_at_least((n + 1) / 2); }

// Sum over the 64 lanes of R per-lane binary64 rows (R a power of two <= 64),
// each row's total left in the lanes l with l / (64 / R) equal to the row: every
// step halves the rows a lane holds (rows_reduce_scatter in kep_grad.h).
__device__ __forceinline__ double lane_select64(uint64_t mask, double if_clear, double if_set)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, if_clear), b = __builtin_bit_cast(uint64_t, if_set);
    const uint32_t lo = __float_as_uint(lane_select(mask, __uint_as_float((uint32_t)a), __uint_as_float((uint32_t)b)));
    const uint32_t hi = __float_as_uint(
        lane_select(mask, __uint_as_float((uint32_t)(a >> 32)), __uint_as_float((uint32_t)(b >> 32))));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int R>
__device__ __forceinline__ double rows_reduce_scatter64(double (&x)[R])
{
#pragma unroll
    for (int h = R / 2, o = 32; h >= 1; h >>= 1, o >>= 1) {
        const uint64_t up = __ballot((__lane_id() & o) != 0);     // lanes keeping the upper half
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const double keep = lane_select64(up, x[i], x[i + h]);
            const double send = lane_select64(up, x[i + h], x[i]);
            x[i] = keep + __shfl_xor(send, o, 64);
        }
    }
    double v = x[0];
#pragma unroll
    for (int o = 32 / R; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__host__ __device__ inline size_t grad64_table_offset(int wpb, int sb, int npl)
{
    return ((size_t)wpb * sb * npl * sizeof(RecG64) + (size_t)wpb * sb * sizeof(int) + 15) & ~(size_t)15;
}

constexpr size_t kGrad64TableBytes = sizeof(kep_start_tab) + kSc64Bytes;

template <bool ROOT, int NPL, int NCH>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NPL <= 2 ? 3 : 2)))
k_grad64(DenseArgs a, int nll)
{
    constexpr int NROW = 5 * NPL + 1;
    constexpr int R = pow2_at_least(NROW);
    constexpr int SPAN = 64 / R;              // lanes holding one row after the reduction
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = __lane_id();
    const int wpb = blockDim.x >> 6;
    const int wib = uniform_int(threadIdx.x >> 6);
    RecG64 *recs = reinterpret_cast<RecG64 *>(smem) + (size_t)wib * a.sb * NPL;
    int *sysbad = reinterpret_cast<int *>(smem + (size_t)wpb * a.sb * NPL * sizeof(RecG64)) + wib * a.sb;
    uint32_t *tab = nullptr;
    double2 *knots = nullptr;
    if constexpr (ROOT) {
        tab = reinterpret_cast<uint32_t *>(smem + grad64_table_offset(wpb, a.sb, NPL));
        knots = reinterpret_cast<double2 *>(tab + kTabWords);
        start_table_begin(tab);
        load_knots64(knots);
    }

    const int64_t group = 64 * NCH;
    const bool has_jit = a.jitter != nullptr;
    const int fixed = fixed64(a.fixed_iter);
    const int row = lane / SPAN;
    const double nan = __builtin_nan("");

    Obs64 o[NCH];
    auto load_group = [&](int64_t k0) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) Pol64::load_obs(a, k0 + c * 64 + lane, o[c]);
    };
    if (a.n_obs <= group) load_group(0);
    if constexpr (ROOT) start_table_end();

    // batches in turn over the grid's wavefronts: the whole grid sweeps the systems in
    // order (contiguous shares per wavefront or block ran 2-7% slower: the grid then
    // writes all over every output row at once)
    for (int64_t bt = (int64_t)blockIdx.x * wpb + wib; bt < a.bt.n_batches; bt += (int64_t)gridDim.x * wpb) {
        int nb;
        const int64_t first = a.bt.first(bt, a.n_sys, nb);
        wave_sync_lds();
        if (lane < nb) {
            const int64_t sys = first + lane;
            bool ok = isfinite(a.t0);
            if (a.offset) ok = ok && isfinite(a.offset[sys]);
            if (has_jit) ok = ok && isfinite(a.jitter[sys]) && a.jitter[sys] >= 0.0;
            sysbad[lane] = ok ? 0 : 1;
        }
        wave_sync_lds();
#pragma nounroll
        for (int q = lane; q < nb * NPL; q += 64) {
            const int j = q / nb, sq = q - j * nb;
            const int64_t p = (int64_t)j * a.n_sys + first + sq;
            RecG64 r;
            if (!setup_g64(a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], r)) sysbad[sq] = 1;
            recs[sq * NPL + j] = r;
        }
        wave_sync_lds();

        for (int sl = 0; sl < nb; ++sl) {
            const int64_t sys = first + sl;
            const double gam = a.offset ? a.offset[sys] : 0.0;
            const double jit = has_jit ? a.jitter[sys] : 0.0;
            const bool sbad = uniform_int(sysbad[sl]) != 0;
            const RecG64 *rs = recs + sl * NPL;
            double acc[R];
#pragma unroll
            for (int i = 0; i < R; ++i) acc[i] = 0.0;
            double chi = 0.0, sum_lv = 0.0, sum_w = 0.0, sum_wr2 = 0.0;
            bool bad_obs = false;
            for (int64_t k0 = 0; k0 < a.n_obs; k0 += group) {
                if (a.n_obs > group) load_group(k0);
                // velocities; sin E, cos E, 1/D (and q) kept for the derivative terms
                double m[NCH], sE[NPL][NCH], cE[NPL][NCH], rD[NPL][NCH];
                double tt[NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    m[c] = 0.0;
                    tt[c] = o[c].tt;
                }
#pragma nounroll
                for (int j = 0; j < NPL; ++j) {
                    Root64 r[NCH];
                    double q[NCH];
                    roots_g64<ROOT, NCH>(rs[j], tt, fixed, a.max_iter, tab, knots, r, q);
                    const double K = rs[j].K;
#pragma unroll
                    for (int c = 0; c < NCH; ++c) m[c] += K * dvdk_g64(rs[j], r[c]);
#pragma unroll
                    for (int jj = 0; jj < NPL; ++jj) {
                        if (jj == j) {
#pragma unroll
                            for (int c = 0; c < NCH; ++c) {
                                sE[jj][c] = r[c].s;
                                cE[jj][c] = r[c].c;
                                rD[jj][c] = r[c].rD;
                            }
                        }
                    }
                }
                double c2[NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    const double r = m[c] + gam - o[c].v;
                    const double var = o[c].s2 + jit * jit;
                    c2[c] = 0.0;
                    if (o[c].in) {
                        bad_obs = bad_obs || !o[c].ok || !(var > 0.0);
                        const double w = has_jit ? 1.0 / var : o[c].w;
                        const double wr = w * r;
                        chi = fma(wr, r, chi);
                        c2[c] = 2.0 * wr;
                        if (nll) {
                            sum_lv += log(var);
                            sum_w += w;
                            sum_wr2 = fma(wr, wr, sum_wr2);
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < NPL; ++j) {
                    lds_reload_barrier();
                    const RecG64 &p = rs[j];
#pragma unroll
                    for (int c = 0; c < NCH; ++c) {
                        double x[3];
                        terms_g64(p, sE[j][c], cE[j][c], rD[j][c], x);
                        const double dvdK = p.b * fma(p.b * p.cw, cE[j][c], -(p.sw * sE[j][c])) * rD[j][c];
                        const double q = p.ph.rP == p.ph.rP ? o[c].tt * p.ph.rP : o[c].tt / p.ph.P;
                        acc[5 * j] = fma(c2[c], x[0] * q, acc[5 * j]);
                        acc[5 * j + 1] = fma(c2[c], dvdK, acc[5 * j + 1]);
                        acc[5 * j + 2] = fma(c2[c], x[1], acc[5 * j + 2]);
                        acc[5 * j + 3] = fma(c2[c], x[2], acc[5 * j + 3]);
                        acc[5 * j + 4] = fma(c2[c], x[0], acc[5 * j + 4]);
                    }
                }
#pragma unroll
                for (int c = 0; c < NCH; ++c) acc[5 * NPL] += c2[c];
            }
            const double tot = rows_reduce_scatter64<R>(acc);
            chi = wave_sum(chi);
            if (nll) {
                sum_lv = wave_sum(sum_lv);
                sum_w = wave_sum(sum_w);
                sum_wr2 = wave_sum(sum_wr2);
            }
            const bool bad = sbad || __any(bad_obs);
            if (lane % SPAN == 0 && row < NROW) {
                double gv = tot;                     // the offset row, and K rows: factor 1
                if (row < 5 * NPL) {
                    const int j = row / 5, i = row - 5 * (row / 5);
                    const double K = rs[j].K;
                    // (tot / P first: 2 pi K / P overflows for the smallest P, where tot may be 0)
                    gv = i == 0 ? tot / rs[j].ph.P * (kTwoPi * K) : i == 1 ? tot : i == 2 ? K * tot : -K * tot;
                }
                a.grad[(int64_t)row * a.n_sys + sys] = bad ? nan : gv;
            }
            if (lane == 0) {
                a.out[sys] = bad ? nan : chi + sum_lv;
                if (nll) a.grad[(int64_t)NROW * a.n_sys + sys] = bad ? nan : 2.0 * jit * (sum_w - sum_wr2);
            }
        }
    }
}

template <bool ROOT, int NPL, int NCH>
hipError_t launch_grad64_t(DenseArgs a, bool nll, LaunchShape shape, hipStream_t st)
{
    const int block = shape.block > 0 ? shape.block : 256;
    const int wpb = block / 64;
    const size_t rec_bytes = (size_t)wpb * (NPL * sizeof(RecG64) + sizeof(int));
    const size_t tables = ROOT ? kGrad64TableBytes : 0;
    // systems per setup batch: four blocks of four wavefronts share a CU's LDS
    int64_t sb_cap = (lds_budget(4) - (int64_t)tables - 16) / (int64_t)rec_bytes;
    sb_cap = sb_cap < 1 ? 1 : (sb_cap > kMaxSB ? kMaxSB : sb_cap);
    auto lds_of = [&](int64_t sb) { return grad64_table_offset(wpb, (int)sb, NPL) + tables; };
    void (*kern)(DenseArgs, int) = k_grad64<ROOT, NPL, NCH>;
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)kern, block, lds_of(sb_cap));
    a.bt = make_batches(a.n_sys, (int64_t)device_cu_count() * per_cu * wpb, sb_cap);
    a.sb = a.bt.sb;
    int64_t grid = (a.bt.n_batches + wpb - 1) / wpb;
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    if (grid > cap) grid = cap;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(block), lds_of(a.sb), st, a, nll ? 1 : 0);
    return hipGetLastError();
}

// Two chunks per lane where n_obs fills them and the registers allow.
template <int NPL>
hipError_t launch_grad64_npl(DenseArgs a, bool nll, LaunchShape shape, hipStream_t st)
{
    if (a.fixed_iter != 0) return launch_grad64_t<false, NPL, 1>(a, nll, shape, st);
    if constexpr (NPL <= 4)
        if (a.n_obs > 64) return launch_grad64_t<true, NPL, 2>(a, nll, shape, st);
    return launch_grad64_t<true, NPL, 1>(a, nll, shape, st);
}

}  // namespace

hipError_t launch_grad64(DenseArgs a, bool nll, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0) return hipSuccess;
    switch (a.n_pl) {
        case 1: return launch_grad64_npl<1>(a, nll, shape, st);
        case 2: return launch_grad64_npl<2>(a, nll, shape, st);
        case 3: return launch_grad64_npl<3>(a, nll, shape, st);
        case 4: return launch_grad64_npl<4>(a, nll, shape, st);
        case 5: return launch_grad64_npl<5>(a, nll, shape, st);
        case 6: return launch_grad64_npl<6>(a, nll, shape, st);
        case 7: return launch_grad64_npl<7>(a, nll, shape, st);
        case 8: return launch_grad64_npl<8>(a, nll, shape, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kep
