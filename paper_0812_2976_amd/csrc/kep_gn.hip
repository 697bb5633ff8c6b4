// Gauss-Newton products of the chi-square on the matrix cores: for each
// system, with J the Jacobian of the model velocities (one row per
// observation, one column per parameter P, K, e, omega, M0 of each planet and
// the offset) and W = diag(1/(sigma^2 + s^2)),
//   J^T W J (packed upper triangle),  J^T W r,  chi2 = r^T W r.
// These feed Levenberg-Marquardt and Newton-type optimisers (the paper asks
// for derivatives for optimisers, Sec. 6).  J^T W J is a dense contraction
// over the observations, so it runs on MFMA: each lane (one observation)
// forms its row of the augmented matrix sqrt(w) [J | 1 | r] from the
// implicit-function derivative terms of the adjoint (kep_grad.h) and stores it
// in the wavefront's slice of LDS; the wavefront then accumulates 16 x 16
// blocks that cover the upper triangle of its Gram matrix, four observations
// per product.  The augmented column gives J^T W r and chi2 from the same
// products.
//
// binary64 path (k_gn64): rows in binary64, v_mfma_f64_16x16x4_f64.
// Mixed path (k_gn_obs): rows in binary32 (the derivative terms are binary32
// already), v_mfma_f32_16x16x4_f32 over each chunk of 64 observations, and
// each chunk's sums added into binary64 accumulators, so one rounding error
// spans at most 64 terms.  The binary32 tile halves the LDS per wavefront
// (more resident wavefronts) and the binary32 products issue at twice the
// binary64 rate.
#include <hip/hip_runtime.h>

#include "kep_device.h"
#include "kep_grad.h"
#include "kep_internal.h"
#include "kep_policy.h"
#include "kep_root64.h"

namespace kep {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// Stores block (bi, bj) of the Gram matrix of sqrt(w) [J | 1 | r]: the packed
// upper triangle of J^T W J, J^T W r from the last column, chi2 from the
// corner.  (i, j) is this lane's entry q of the block.
__device__ __forceinline__ void gn_store(const DenseArgs &a, double *jtwr, double *jtwj, int64_t sys, int np, int i,
                                         int j, double val)
{
    if (i <= j && j < np) jtwj[(int64_t)(i * np - i * (i - 1) / 2 + (j - i)) * a.n_sys + sys] = val;
    else if (j == np && i < np) jtwr[(int64_t)i * a.n_sys + sys] = val;
    else if (i == np && j == np) a.out[sys] = val;
}

// ------------------------------------------------------------------ binary64
// Binary64 path (k_gn64): one chunk of 64 observations at a time, each lane's
// row of sqrt(w) [J | 1 | r] in the wavefront's column-major tile (the layout
// and the block products of the mixed path, in binary64), four observations per
// v_mfma_f64_16x16x4_f64.  The binary64 product returns row l/16 + 4 q of its
// block in accumulator q (the binary32 one row 4 (l/16) + q).  ROOT: the default
// step count (kep_root64.h; its starting-value table is read through the cache,
// as in the mixed kernel, the sin/cos knots from LDS); else Danby's plain
// iteration.
//
// What bounds it: at 262,144 x 4 x 256 the products (64 cycles each, two per
// four observations) and the row arithmetic take about the same time and add
// up, as in the mixed kernel.
constexpr int kGn64Col = 66;   // 64 observations + 2: consecutive columns start 4 banks apart

template <int NPL>
__host__ __device__ inline size_t gn64_lds_per_wave()
{
    return ((size_t)(5 * NPL + 2) * kGn64Col + 0) * sizeof(double) + ((NPL * sizeof(RecG64) + 15) & ~(size_t)15);
}

template <bool ROOT, int NPL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NPL <= 6 ? 3 : 2)))
k_gn64(DenseArgs a, double *jtwr, double *jtwj)
{
    constexpr int NC = 5 * NPL + 2;          // parameters, offset, residual
    constexpr int NP = NC - 1;
    constexpr int NB = (NC + 15) / 16;
    constexpr bool TWO = NC > 16 && NC <= 24;
    constexpr int GX = NC - 16;
    constexpr int NOP = TWO ? 3 : NB;
    constexpr int NPAIR = TWO ? 2 : NB * (NB + 1) / 2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = __lane_id();
    const int wpb = blockDim.x >> 6;
    const int wib = uniform_int(threadIdx.x >> 6);
    unsigned char *mine = smem + (size_t)wib * gn64_lds_per_wave<NPL>();
    double *T = reinterpret_cast<double *>(mine);
    RecG64 *pl = reinterpret_cast<RecG64 *>(T + (size_t)NC * kGn64Col);
    const double2 *knots = nullptr;
    if constexpr (ROOT) {
        double2 *k = reinterpret_cast<double2 *>(smem + (size_t)wpb * gn64_lds_per_wave<NPL>());
        load_knots64(k);
        __syncthreads();
        knots = k;
    }

    const int fixed = fixed64(a.fixed_iter);
    const bool has_jit = a.jitter != nullptr;
    const int n_chunks = (int)((a.n_obs + 63) / 64);
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    const double nan = __builtin_nan("");
    double *col = T + lane;
    const int li = lane & 15;
    const double *src[NOP];                  // this lane's operand columns (as k_gn_obs)
#pragma unroll
    for (int b = 0; b < NOP; ++b) {
        int c;
        if constexpr (TWO) c = b == 0 ? li : b == 1 ? (li < GX ? li : (li + 8 < NC ? li + 8 : li)) : GX + li;
        else c = 16 * b + li < NC ? 16 * b + li : NC - 1;
        src[b] = T + c * kGn64Col + 16 * (lane >> 4);
    }

    for (int64_t sys = (int64_t)blockIdx.x * wpb + wib; sys < a.n_sys; sys += n_waves) {
        wave_sync_lds();
        bool pok = true;
        if (lane < NPL) {
            const int64_t p = (int64_t)lane * a.n_sys + sys;
            RecG64 q;
            pok = setup_g64(a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], q);
            pl[lane] = q;
        }
        const double gam = a.offset ? a.offset[sys] : 0.0;
        const double jit = has_jit ? a.jitter[sys] : 0.0;
        bool ok = isfinite(a.t0) && !__any(!pok);
        if (a.offset) ok = ok && isfinite(gam);
        if (has_jit) ok = ok && isfinite(jit) && jit >= 0.0;
        wave_sync_lds();

        d4 acc[NPAIR];
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) acc[p] = d4{0.0, 0.0, 0.0, 0.0};
        bool bad_obs = false;
        for (int ch = 0; ch < n_chunks; ++ch) {
            const int64_t k = (int64_t)ch * 64 + lane;
            const bool in = k < a.n_obs;
            const double t = in ? a.t[k] : a.t0, vo = in ? a.v[k] : 0.0, sg = in ? a.sigma[k] : 1.0;
            const double var = sg * sg + jit * jit;
            const bool ook = isfinite(t) && isfinite(vo) && isfinite(sg) && sg >= 0.0 && var > 0.0;
            const bool use = in && ook;
            bad_obs = bad_obs || (in && !ook);
            const double sw = use ? sqrt(1.0 / var) : 0.0;   // sqrt(w) = 1 / sqrt(sigma^2 + s^2)
            const double tt[1] = {use ? t - a.t0 : 0.0};     // rows past the last observation stay finite
            double model = 0.0;
#pragma nounroll
            for (int j = 0; j < NPL; ++j) {
                const RecG64 &p = pl[j];
                Root64 r[1];
                double q[1], x[3];
                roots_g64<ROOT, 1>(p, tt, fixed, a.max_iter, kep_start_tab, knots, r, q);
                const double dvdK = dvdk_g64(p, r[0]);
                terms_g64(p, r[0].s, r[0].c, r[0].rD, x);
                const double swK = sw * p.K;
                model += p.K * dvdK;
                double *cj = col + 5 * j * kGn64Col;
                // (where 1/P overflows q may be 0: at the epoch, and past the last observation)
                const double qP = kTwoPi * q[0];
                cj[0 * kGn64Col] = swK * x[0] * (p.ph.rP == p.ph.rP ? qP * p.ph.rP : qP / p.ph.P);
                cj[1 * kGn64Col] = sw * dvdK;
                cj[2 * kGn64Col] = swK * x[1];
                cj[3 * kGn64Col] = -swK * x[2];
                cj[4 * kGn64Col] = -swK * x[0];
            }
            col[(NP - 1) * kGn64Col] = sw;
            col[NP * kGn64Col] = use ? sw * ((model + gam) - vo) : 0.0;
            wave_sync_lds();
#pragma unroll
            for (int s2 = 0; s2 < 8; ++s2) {
                double2 av[NOP];
#pragma unroll
                for (int b = 0; b < NOP; ++b) av[b] = *reinterpret_cast<const double2 *>(src[b] + 2 * s2);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    double op[NOP];
#pragma unroll
                    for (int b = 0; b < NOP; ++b) op[b] = u == 0 ? av[b].x : av[b].y;
                    if constexpr (TWO) {
                        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(op[0], op[1], acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(op[2], op[2], acc[1], 0, 0, 0);
                    } else {
                        int p = 0;
#pragma unroll
                        for (int bi = 0; bi < NB; ++bi) {
#pragma unroll
                            for (int bj = bi; bj < NB; ++bj) {
                                acc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(op[bi], op[bj], acc[p], 0, 0, 0);
                                ++p;
                            }
                        }
                    }
                }
            }
            wave_sync_lds();
        }
        ok = ok && !__any(bad_obs);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = (lane >> 4) + 4 * q;
            if constexpr (TWO) {
                // X+Y by X+Z, then Y+Z squared (as k_gn_obs)
                const int c = li < GX ? li : li + 8;
                if (i < GX + 8 && li < GX + 8 && !(i < GX && c < GX && i > c))
                    gn_store(a, jtwr, jtwj, sys, NP, i < c ? i : c, i < c ? c : i, ok ? acc[0][q] : nan);
                const int p2 = GX + i, c2 = GX + li;
                if (p2 <= c2 && !(p2 < GX + 8 && c2 >= GX + 8))
                    gn_store(a, jtwr, jtwj, sys, NP, p2, c2, ok ? acc[1][q] : nan);
            } else {
                int p = 0;
#pragma unroll
                for (int bi = 0; bi < NB; ++bi) {
#pragma unroll
                    for (int bj = bi; bj < NB; ++bj) {
                        gn_store(a, jtwr, jtwj, sys, NP, 16 * bi + i, 16 * bj + li, ok ? acc[p][q] : nan);
                        ++p;
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------------ mixed

// Mixed path (k_gn_obs): the observations of a system in NCH chunks of 64
// per lane, like the mixed adjoint (kep_adjoint.hip): pass 1 over the chunks
// (binary64 phase, binary32 Kepler solve from the starting-value table,
// binary64 correction of E and the velocity) gives every chunk's sin E and
// cos E - e per planet and its binary64 residual; then, one chunk at a time,
// each lane writes its row of sqrt(w) [J | 1 | r] (the derivative terms of the
// corrected root) into the wavefront's tile and the tile's Gram matrix is
// accumulated with v_mfma_f32_16x16x4_f32, each chunk's sums added into
// binary64 accumulators.  The tile is column-major, T[c * kGnCol + obs]: a
// lane writes its row with unit stride across the wavefront, and the matrix
// operands are read as runs of four consecutive observations (128-bit loads).
// Observation 16 g + 4 s + u of the chunk feeds step u of lane group g = l/16
// in the s-th run: the Gram matrix sums over all observations, so any fixed
// assignment of observations to (step, k) slots, the same for both operands,
// gives the same products.  Only the 5 n_pl + 2 live columns are stored.  An
// operand lane past the live columns reads some live column instead: output
// row i of a product depends only on row i of its first operand and output
// column j only on column j of its second, so such lanes change nothing but
// entries that are never stored.
//
// Block products per step of four observations: every pair of 16-column
// blocks, except for 17 to 24 columns (three or four planets), where two
// products cover the upper triangle: with the columns in groups
// X = [0, g), Y = [g, g + 8), Z = [g + 8, NC), g = NC - 16, the product of the
// operands X+Y (rows) and X+Z (columns) holds the pairs XX, XY, XZ and YZ, and
// the square of Y+Z holds YY and ZZ (against three products for two blocks;
// NC <= 24 makes each operand at most 16 columns).
constexpr int kGnCol = 68;   // 64 observations + 4: consecutive columns start 4 banks apart

template <int NPL>
__host__ __device__ constexpr int gn_cols() { return 5 * NPL + 2; }

template <int NPL>
__host__ __device__ inline size_t gn_obs_lds_per_wave(int sb)
{
    const size_t b = (size_t)gn_cols<NPL>() * kGnCol * sizeof(float) + (size_t)sb * NPL * sizeof(RecGrad) +
                     (size_t)sb * sizeof(int);
    return (b + 15) & ~(size_t)15;
}

// GROUPS: kOneGroup where one group of NCH chunks holds every observation,
// kOddChunks where the last group's last chunk is empty, else kGroups.
enum { kOneGroup = 0, kGroups = 1, kOddChunks = 2 };

template <int NPL, int NCH, int GROUPS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) k_gn_obs(DenseArgs a, double *jtwr,
                                                                                       double *jtwj)
{
    constexpr int NC = gn_cols<NPL>();       // parameters, offset, residual
    constexpr int NP = NC - 1;               // parameters and offset
    constexpr int NB = (NC + 15) / 16;       // 16-column blocks
    constexpr bool TWO = NC > 16 && NC <= 24;
    constexpr int GX = NC - 16;              // TWO: group X = [0, GX), Y = [GX, GX + 8), Z = [GX + 8, NC)
    constexpr int NOP = TWO ? 3 : NB;        // operand column sets (TWO: X+Y, X+Z, Y+Z)
    constexpr int NPAIR = TWO ? 2 : NB * (NB + 1) / 2;   // products per step
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = __lane_id();
    const int wpb = blockDim.x >> 6;
    const int wib = uniform_int(threadIdx.x >> 6);
    unsigned char *mine = smem + (size_t)wib * gn_obs_lds_per_wave<NPL>(a.sb);
    float *T = reinterpret_cast<float *>(mine);
    RecGrad *recs = reinterpret_cast<RecGrad *>(mine + (size_t)NC * kGnCol * sizeof(float));
    int *sysbad = reinterpret_cast<int *>(recs + (size_t)a.sb * NPL);
    double2 *knots = reinterpret_cast<double2 *>(smem + (size_t)wpb * gn_obs_lds_per_wave<NPL>(a.sb));
    fill_sincos64_knots(knots);
    __syncthreads();

    // Block b takes runs b, b + G, ... of wpb x sb systems (G blocks); wavefront w of
    // the block holds systems run + w + wpb i (i < nb), so the block's wavefronts
    // write neighbouring systems' entries of every output row at about the same time
    // and the L2 merges them into longer pieces (with consecutive systems per
    // wavefront each row's line stays partly written for a whole batch and goes
    // back to HBM in pieces; contiguous shares ran slower too).
    const int64_t run_step = (int64_t)gridDim.x * wpb * a.sb;
    const int n_groups = GROUPS == kOneGroup ? 1 : (int)((a.n_obs + 64 * NCH - 1) / (64 * NCH));
    const bool has_jit = a.jitter != nullptr;
    const double nan = __builtin_nan("");
    float *col = T + lane;                   // this lane's observation in column 0
    // operand columns of this lane, li = l%16: 16 b + li in block b, or with TWO
    // li (X+Y), li or li + 8 (X+Z) and GX + li (Y+Z); lanes past the live
    // columns read a live one
    const int li = lane & 15;
    const float *src[NOP];
#pragma unroll
    for (int b = 0; b < NOP; ++b) {
        int c;
        if constexpr (TWO) c = b == 0 ? li : b == 1 ? (li < GX ? li : (li + 8 < NC ? li + 8 : li)) : GX + li;
        else c = 16 * b + li < NC ? 16 * b + li : NC - 1;
        src[b] = T + c * kGnCol + 16 * (lane >> 4);
    }

    ObsG o[NCH];
    auto load_group = [&](int g) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) load_obs_g(a, (int64_t)g * 64 * NCH + c * 64 + lane, o[c]);
    };
    if (n_groups <= 1) load_group(0);

    for (int64_t run0 = (int64_t)blockIdx.x * wpb * a.sb; run0 < a.n_sys; run0 += run_step) {
        const int64_t first = run0 + wib, left = a.n_sys - first;
        const int nb = left <= 0 ? 0 : (int)min((int64_t)a.sb, (left + wpb - 1) / wpb);
        wave_sync_lds();
        if (lane < nb) {
            const int64_t sys = first + (int64_t)wpb * lane;
            bool ok = isfinite(a.t0);
            if (a.offset) ok = ok && isfinite(a.offset[sys]);
            if (has_jit) ok = ok && isfinite(a.jitter[sys]) && a.jitter[sys] >= 0.0;
            sysbad[lane] = ok ? 0 : 1;
        }
        wave_sync_lds();
        // planet records with the lanes over the run's (planet, system) pairs
#pragma nounroll
        for (int q = lane; q < nb * NPL; q += 64) {
            const int j = q / nb, sq = q - j * nb;
            const int64_t p = (int64_t)j * a.n_sys + first + (int64_t)wpb * sq;
            RecGrad r;
            if (!grad_setup_rec(a.fixed_iter, a.P[p], a.K[p], a.e[p], a.w[p], a.M0[p], r)) sysbad[sq] = 1;
            // the column factors 2 pi K/P and K as the binary32 pair that the rows use (read as
            // binary64 and converted for every chunk: 262,144 x 4 x 256 1.822 against 1.815 ms)
            r.fP = __hiloint2double(__float_as_int((float)r.fK), __float_as_int((float)r.fP));
            recs[sq * NPL + j] = r;
        }
        wave_sync_lds();

        for (int s = 0; s < nb; ++s) {
            const int64_t sys = first + (int64_t)wpb * s;
            const double gam = a.offset ? a.offset[sys] : 0.0;
            const double jit = has_jit ? a.jitter[sys] : 0.0;
            const float jit2 = (float)(jit * jit);
            const bool sbad = uniform_int(sysbad[s]) != 0;
            const RecGrad *rs = recs + s * NPL;
            d4 acc[NPAIR];
#pragma unroll
            for (int p = 0; p < NPAIR; ++p) acc[p] = d4{0.0, 0.0, 0.0, 0.0};
            bool bad_obs = false;
            for (int g = 0; g < n_groups; ++g) {
                if (n_groups > 1) load_group(g);
                // pass 1 (as the mixed adjoint): corrected velocities; sin E and
                // cos E - e kept per planet and chunk
                double model[NCH];
                float sE[NPL][NCH], cme[NPL][NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) model[c] = gam;
#pragma nounroll
                for (int j = 0; j < NPL; ++j) {
                    const RecGrad &rr = rs[j];
                    double M64[NCH];
                    float M[NCH], E[NCH], sv[NCH], omc[NCH], sj[NCH], cj[NCH];
#pragma unroll
                    for (int c = 0; c < NCH; ++c) {
                        M64[c] = mean_anomaly64_exact(o[c].tt, rr.ph);
                        M[c] = (float)M64[c];
                    }
                    PolMixed::solve<NCH, false>(rr.k, uniform_int(rr.niter), uniform_int(rr.check) != 0, rr.tp, M, E,
                                                sv, omc, a.max_iter, kep_start_tab);
#pragma unroll
                    for (int c = 0; c < NCH; ++c) model[c] += refine_velocity(rr, E[c], M64[c], knots, sj[c], cj[c]);
#pragma unroll
                    for (int jj = 0; jj < NPL; ++jj) {
                        if (jj == j) {
#pragma unroll
                            for (int c = 0; c < NCH; ++c) {
                                sE[jj][c] = sj[c];
                                cme[jj][c] = cj[c];
                            }
                        }
                    }
                }
                // pass 2, one chunk at a time: the rows of sqrt(w) [J | 1 | r] into
                // the tile, then the tile's Gram matrix
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    // the last group's empty chunk has no rows
                    if constexpr (GROUPS == kOddChunks)
                        if (c == NCH - 1 && g == n_groups - 1) break;
                    const float var = o[c].s2 + jit2;
                    const bool use = o[c].in && o[c].ok && var > 0.0f;
                    if (o[c].in) bad_obs = bad_obs || !o[c].ok || !(var > 0.0f);
                    const float sw = use ? __builtin_amdgcn_rsqf(var) : 0.0f;   // sqrt(w)
                    const double r = model[c] - o[c].v;                          // residual in binary64
#pragma unroll
                    for (int j = 0; j < NPL; ++j) {
                        lds_reload_barrier();
                        const RecGrad &rr = rs[j];
                        float x[5];
                        grad_terms_ce(rr, sE[j][c], cme[j][c], (float)(o[c].tt * rr.ph.rP), x);
                        const double f = rr.fP;
                        const float fP = __int_as_float(__double2loint(f)), fK = __int_as_float(__double2hiint(f));
                        float *cj = col + 5 * j * kGnCol;
                        cj[0 * kGnCol] = sw * (fP * x[0]);
                        cj[1 * kGnCol] = sw * x[1];
                        cj[2 * kGnCol] = sw * (fK * x[2]);
                        cj[3 * kGnCol] = -sw * (fK * x[3]);
                        cj[4 * kGnCol] = -sw * (fK * x[4]);
                    }
                    col[(NP - 1) * kGnCol] = sw;
                    col[NP * kGnCol] = use ? sw * (float)r : 0.0f;
                    wave_sync_lds();
                    f4 accf[NPAIR];
#pragma unroll
                    for (int p = 0; p < NPAIR; ++p) accf[p] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4) {
                        f4 av[NOP];
#pragma unroll
                        for (int b = 0; b < NOP; ++b) av[b] = *reinterpret_cast<const f4 *>(src[b] + 4 * s4);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if constexpr (TWO) {
                                accf[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[0][u], av[1][u], accf[0], 0, 0, 0);
                                accf[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[2][u], av[2][u], accf[1], 0, 0, 0);
                            } else {
                                int p = 0;
#pragma unroll
                                for (int bi = 0; bi < NB; ++bi) {
#pragma unroll
                                    for (int bj = bi; bj < NB; ++bj) {
                                        accf[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[bi][u], av[bj][u], accf[p],
                                                                                        0, 0, 0);
                                        ++p;
                                    }
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int p = 0; p < NPAIR; ++p)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[p][q] += (double)accf[p][q];
                    wave_sync_lds();
                }
            }
            const bool ok = !sbad && !__any(bad_obs);
            // lane l holds entry (4 (l/16) + q, l%16) of each product in acc[.][q]
            // (the binary32 16x16x4 product keeps four consecutive output rows per lane)
            if constexpr (TWO) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 4 * (lane >> 4) + q;
                    // X+Y by X+Z: XX (upper triangle), YX (as XY), XZ and YZ
                    const int c = li < GX ? li : li + 8;
                    if (i < GX + 8 && li < GX + 8 && !(i < GX && c < GX && i > c))
                        gn_store(a, jtwr, jtwj, sys, NP, i < c ? i : c, i < c ? c : i, ok ? acc[0][q] : nan);
                    // Y+Z squared: YY and ZZ (upper triangles; YZ came from the first)
                    const int p2 = GX + i, c2 = GX + li;
                    if (p2 <= c2 && !(p2 < GX + 8 && c2 >= GX + 8))
                        gn_store(a, jtwr, jtwj, sys, NP, p2, c2, ok ? acc[1][q] : nan);
                }
            } else {
                int p = 0;
#pragma unroll
                for (int bi = 0; bi < NB; ++bi) {
#pragma unroll
                    for (int bj = bi; bj < NB; ++bj) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            gn_store(a, jtwr, jtwj, sys, NP, 16 * bi + 4 * (lane >> 4) + q, 16 * bj + li,
                                     ok ? acc[p][q] : nan);
                        ++p;
                    }
                }
            }
        }
    }
}

template <int NPL, int NCH, int GROUPS>
hipError_t launch_gn_obs_t(DenseArgs a, double *jtwr, double *jtwj, LaunchShape shape, hipStream_t st)
{
    const int block = shape.block > 0 ? shape.block : 256;
    const int wpb = block / 64;
    // systems per setup batch: tiles and records within 40 KiB per block (four
    // blocks of four wavefronts on a CU's 160 KiB), at most kMaxSB; the
    // block's sin/cos knots come on top
    int sb_cap = kMaxSB;
    while (sb_cap > 1 && (size_t)wpb * gn_obs_lds_per_wave<NPL>(sb_cap) > 40 * 1024) --sb_cap;
    auto lds_of = [&](int sbv) { return (size_t)wpb * gn_obs_lds_per_wave<NPL>(sbv) + kSc64Bytes; };
    void (*kern)(DenseArgs, double *, double *) = k_gn_obs<NPL, NCH, GROUPS>;
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)kern, block, lds_of(sb_cap));
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    const int64_t max_waves = cap * wpb;
    int64_t sb = (a.n_sys + max_waves - 1) / (max_waves > 0 ? max_waves : 1);
    sb = sb < 1 ? 1 : (sb > sb_cap ? sb_cap : sb);
    a.sb = (int)sb;
    const size_t lds = lds_of(a.sb);
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    // one block per wpb x sb systems, at most the resident count
    int64_t grid = (a.n_sys + (int64_t)wpb * sb - 1) / ((int64_t)wpb * sb);
    if (grid > cap) grid = cap;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(block), lds, st, a, jtwr, jtwj);
    return hipGetLastError();
}

// Observation chunks per lane: one for n_obs <= 64, else two (at c4, 262,144 x 4
// x 256: one chunk 2.74 ms, two 2.50 ms, four 2.65 ms).
template <int NPL>
hipError_t launch_gn_obs_npl(DenseArgs a, double *jtwr, double *jtwj, LaunchShape shape, hipStream_t st)
{
    const int64_t need = (a.n_obs + 63) / 64;
    if (need <= 1) return launch_gn_obs_t<NPL, 1, kOneGroup>(a, jtwr, jtwj, shape, st);
    if (need == 2) return launch_gn_obs_t<NPL, 2, kOneGroup>(a, jtwr, jtwj, shape, st);
    return need % 2 ? launch_gn_obs_t<NPL, 2, kOddChunks>(a, jtwr, jtwj, shape, st)
                    : launch_gn_obs_t<NPL, 2, kGroups>(a, jtwr, jtwj, shape, st);
}

hipError_t launch_gn_mixed(DenseArgs a, double *jtwr, double *jtwj, LaunchShape shape, hipStream_t st)
{
    switch (a.n_pl) {
        case 1: return launch_gn_obs_npl<1>(a, jtwr, jtwj, shape, st);
        case 2: return launch_gn_obs_npl<2>(a, jtwr, jtwj, shape, st);
        case 3: return launch_gn_obs_npl<3>(a, jtwr, jtwj, shape, st);
        case 4: return launch_gn_obs_npl<4>(a, jtwr, jtwj, shape, st);
        case 5: return launch_gn_obs_npl<5>(a, jtwr, jtwj, shape, st);
        case 6: return launch_gn_obs_npl<6>(a, jtwr, jtwj, shape, st);
        case 7: return launch_gn_obs_npl<7>(a, jtwr, jtwj, shape, st);
        case 8: return launch_gn_obs_npl<8>(a, jtwr, jtwj, shape, st);
        default: return hipErrorInvalidValue;
    }
}

template <bool ROOT, int NPL>
hipError_t launch_gn64_t(DenseArgs a, double *jtwr, double *jtwj, LaunchShape shape, hipStream_t st)
{
    // four wavefronts a block while their tiles and the knots leave three blocks a
    // CU its 160 KiB (up to three planets; four without the knots), else two
    const size_t per_wave = gn64_lds_per_wave<NPL>(), knots = ROOT ? kSc64Bytes : 0;
    const int wpb = shape.block > 0 ? shape.block / 64 : (4 * per_wave + knots <= 53 * 1024 ? 4 : 2);
    const size_t lds = (size_t)wpb * per_wave + knots;
    void (*kern)(DenseArgs, double *, double *) = k_gn64<ROOT, NPL>;
    int per_cu = shape.blocks_per_cu;
    if (per_cu <= 0) per_cu = cached_occupancy((const void *)kern, wpb * 64, lds);
    int64_t grid = (a.n_sys + wpb - 1) / wpb;
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    if (grid > cap) grid = cap;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(wpb * 64), lds, st, a, jtwr, jtwj);
    return hipGetLastError();
}

template <int NPL>
hipError_t launch_gn64_npl(DenseArgs a, double *jtwr, double *jtwj, LaunchShape shape, hipStream_t st)
{
    // a caller's block size whose row-major binary64 tiles (the layout before the
    // live-column one) did not fit 64 KiB was refused, and stays so
    constexpr int nb = (5 * NPL + 2 + 15) / 16;
    constexpr size_t refused_per_wave = ((size_t)64 * (16 * nb + 1) * sizeof(double) + 8 * 64 + 15) & ~(size_t)15;
    if (shape.block > 0 && (size_t)(shape.block / 64) * refused_per_wave > 64 * 1024) return hipErrorInvalidValue;
    return a.fixed_iter == 0 ? launch_gn64_t<true, NPL>(a, jtwr, jtwj, shape, st)
                             : launch_gn64_t<false, NPL>(a, jtwr, jtwj, shape, st);
}

hipError_t launch_gn64(DenseArgs a, double *jtwr, double *jtwj, LaunchShape shape, hipStream_t st)
{
    switch (a.n_pl) {
        case 1: return launch_gn64_npl<1>(a, jtwr, jtwj, shape, st);
        case 2: return launch_gn64_npl<2>(a, jtwr, jtwj, shape, st);
        case 3: return launch_gn64_npl<3>(a, jtwr, jtwj, shape, st);
        case 4: return launch_gn64_npl<4>(a, jtwr, jtwj, shape, st);
        case 5: return launch_gn64_npl<5>(a, jtwr, jtwj, shape, st);
        case 6: return launch_gn64_npl<6>(a, jtwr, jtwj, shape, st);
        case 7: return launch_gn64_npl<7>(a, jtwr, jtwj, shape, st);
        case 8: return launch_gn64_npl<8>(a, jtwr, jtwj, shape, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_gn(DenseArgs a, double *jtwr, double *jtwj, Prec prec, LaunchShape shape, hipStream_t st)
{
    if (a.n_sys <= 0) return hipSuccess;
    if (prec == Prec::Mixed) return launch_gn_mixed(a, jtwr, jtwj, shape, st);
    return launch_gn64(a, jtwr, jtwj, shape, st);
}

}  // namespace kep
