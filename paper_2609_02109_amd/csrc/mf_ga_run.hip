// Whole GA generations in one launch (Section IV-C): one workgroup per
// scenario carries its population through generations [g0, g1] in LDS.
//
// A generation as two launches (fitness, operators) costs about 20 us whatever
// it does: the launches, and their dependent reads of memory.  Scenarios never
// exchange anything, so a workgroup needs no other to go on: tournaments read
// fitness and population from LDS, and a child's fitness is formed by the
// thread that built it.
//
// The random draws do not depend on the population either: ga_draws_kernel
// computes every Philox block of a span of generations beforehand, over the
// whole chip, and keeps only what the operators use (winner candidates, swap
// bits, new genes, repair words: 40 bytes a pair instead of 13 blocks of 32).
//
// Fitness, canonical as everywhere:
//   FIXED  the observed state is held fixed: a prediction depends on the
//          option row only, so each individual's J is a chain over a table of
//          rows (sum K_i canonical forwards per run).
//   else   the fitness of every VRAM-feasible configuration is tabulated per
//          scenario before the first generation (ga_fitness_pre_kernel over
//          the feasible list; no other configuration enters a population).
#include "mf_ga_device.h"

namespace mfi {

// ---------------------------------------------------------------- draws

// A pair's record, in 32-bit words; genes are bytes, model i's at byte i (as
// the digits of an individual are kept), dw = ceil(N / 8) 64-bit words of them:
//   0            per child the digits of its repair draw [2 dw]
//   4 dw         swap bytes (255: swap) [2 dw]
//   6 dw         per child the mutated bytes (255: mutated) [2 dw] and their
//                new values [2 dw]
//   14 dw        crossover (0, 1)
//   14 dw + 1    16-bit tournament candidates, two words per selection block
// Word w of every pair of a generation and scenario are neighbours.
struct GaRecord {
    int nsel, nswap, nmut, dw, swap, mut, cx, sel, words;
    __host__ __device__ GaRecord(int tk, int N)
        : nsel((2 * tk + 3) / 4), nswap((N + 3) / 4), nmut((N + 1) / 2), dw((N + 7) / 8), swap(4 * dw), mut(6 * dw),
          cx(14 * dw), sel(14 * dw + 1), words(14 * dw + 1 + 2 * nsel)
    {
    }
    __host__ __device__ int blocks() const { return nsel + 1 + nswap + 2 * nmut + 2; }
};

int ga_record_bytes(int tk, int N) { return GaRecord(tk, N).words * 4; }

constexpr int kDrawThreads = 256;

// One thread per Philox block: blocks of one kind are neighbours, and the
// generation and scenario of a workgroup are uniform (part of the first two
// rounds then runs on the scalar unit).
__global__ void __launch_bounds__(kDrawThreads) ga_draws_kernel(const GAConst c, uint64_t seed, int S, int P, int tk,
                                                                float p_cx, float p_swap, float p_mut, int gen0,
                                                                int wgs_per, const uint32_t *fl,
                                                                const unsigned long long *n_fl, uint8_t *recs)
{
    const GaRecord R(tk, c.N);
    const int gs = (int)(blockIdx.x / (unsigned)wgs_per), wg = (int)(blockIdx.x % (unsigned)wgs_per);
    const int g = gs / S, s = gs - g * S;   // generation gen0 + g builds the next one
    const int np = P / 2;
    const int t = wg * kDrawThreads + (int)threadIdx.x;
    if (t >= np * R.blocks()) return;
    const int b = t / np, q = t - b * np;
    uint32_t *rec = reinterpret_cast<uint32_t *>(recs) + (int64_t)gs * np * R.words + q;   // word w at rec[w np]
    uint64_t item = (uint64_t)q, purpose;
    int kind, x = 0;   // 0 selection, 1 crossover, 2 swap, 3 mutation, 4 repair; x: block, child
    const int child0 = R.nsel + 1 + R.nswap;
    if (b < R.nsel) {
        kind = 0;
        x = b;
        purpose = kPSel + b;
    } else if (b == R.nsel) {
        kind = 1;
        purpose = kPCx;
    } else if (b < child0) {
        kind = 2;
        x = b - R.nsel - 1;
        purpose = kPSwap + x;
    } else if (b < child0 + 2 * R.nmut) {
        kind = 3;
        x = b - child0;
        const int ch = x >= R.nmut ? 1 : 0;
        item = 1 + 2 * (uint64_t)q + ch;
        purpose = kPMut + (x - ch * R.nmut);
    } else {
        kind = 4;
        x = b - child0 - 2 * R.nmut;
        item = 1 + 2 * (uint64_t)q + x;
        purpose = kPRep;
    }
    const Philox4 r = philox4x64_10(item, (uint64_t)(gen0 + g) + 1, (uint64_t)s, purpose, seed, 0);
    if (kind == 0) {
        rec[(R.sel + 2 * x) * np] =
            (uint32_t)ga_below(r.w[0], (uint64_t)P) | (uint32_t)ga_below(r.w[1], (uint64_t)P) << 16;
        rec[(R.sel + 2 * x + 1) * np] =
            (uint32_t)ga_below(r.w[2], (uint64_t)P) | (uint32_t)ga_below(r.w[3], (uint64_t)P) << 16;
    } else if (kind == 1) {
        rec[R.cx * np] = ga_uni(r.w[0]) < (double)p_cx ? 1u : 0u;
    } else if (kind == 2) {
        uint32_t bytes = 0;
#pragma unroll
        for (int w = 0; w < 4; w++) bytes |= (ga_uni(r.w[w]) < (double)p_swap ? 255u : 0u) << (8 * w);
        rec[(R.swap + x) * np] = bytes;
        // the other half of the last 64-bit word when N ends in its first
        if (x == R.nswap - 1 && (R.nswap & 1)) rec[(R.swap + x + 1) * np] = 0u;
    } else if (kind == 3) {
        // genes 2 blk and 2 blk + 1 of the child: 16 bits of a word each
        const int ch = x >= R.nmut ? 1 : 0, blk = x - ch * R.nmut;
        uint32_t mask = 0, val = 0;
#pragma unroll
        for (int w = 0; w < 2; w++) {
            const int i = 2 * blk + w;
            if (i < c.N && ga_uni(r.w[2 * w]) < (double)p_mut) {
                mask |= 255u << (8 * w);
                val |= (uint32_t)ga_below(r.w[2 * w + 1], (uint64_t)c.K[i]) << (8 * w);
            }
        }
        const int m0 = R.mut + ch * 4 * R.dw, v0 = m0 + 2 * R.dw;
        auto put = [&](int base, int h, uint32_t y) {
            reinterpret_cast<uint16_t *>(rec + (base + h / 2) * np)[h & 1] = (uint16_t)y;
        };
        put(m0, blk, mask);
        put(v0, blk, val);
        if (blk == R.nmut - 1)   // the rest of the last 64-bit word
            for (int z = R.nmut; z < 4 * R.dw; z++) {
                put(m0, z, 0);
                put(v0, z, 0);
            }
    } else {
        // the repair: a uniform draw from the feasible list (index 0 when none
        // is feasible), as digits
        const unsigned long long nf = *n_fl;
        int32_t d[kMaxN];
        ga_digits(c, nf ? fl[ga_below(r.w[0], nf)] : 0, d);
        for (int w = 0; w < 2 * R.dw; w++) {
            uint32_t y = 0;
            for (int z = 0; z < 4; z++)
                if (4 * w + z < c.N) y |= (uint32_t)d[4 * w + z] << (8 * z);
            rec[(x * 2 * R.dw + w) * np] = y;
        }
    }
}

hipError_t launch_ga_draws(const GAConst &c, uint64_t seed, int S, int P, int tk, float p_cx, float p_swap, float p_mut,
                           int gen0, int gens, const uint32_t *fl, const unsigned long long *n_fl, uint8_t *recs,
                           hipStream_t st)
{
    const int wgs = (P / 2 * GaRecord(tk, c.N).blocks() + kDrawThreads - 1) / kDrawThreads;
    hipLaunchKernelGGL(ga_draws_kernel, dim3((unsigned)((int64_t)gens * S * wgs)), dim3(kDrawThreads), 0, st, c, seed, S,
                       P, tk, p_cx, p_swap, p_mut, gen0, wgs, fl, n_fl, recs);
    return hipGetLastError();
}

// ---------------------------------------------------------------- generations

constexpr int kRunMaxThreads = 1024;

// Dynamic LDS of the run kernel, in this order: per individual the fitness,
// the digits (8 bits per model) and the joint index; per option row its term.
struct RunLds {
    size_t fit, dig, rows, pens, idx, total;
    __host__ __device__ RunLds(const GAConst &c, int P, bool fixed)
    {
        size_t o = 0;
        fit = o; o += (size_t)P * 8;
        dig = o; o += (size_t)P * 8 * ((c.N + 7) / 8);
        rows = o; o += (size_t)c.sumK * sizeof(FixedRow);
        pens = o; o += fixed && c.obj.kind != 0 ? (size_t)c.sumK * sizeof(FixedPen) : 0;
        idx = o; o += (size_t)P * 4;
        total = o;
    }
};

// Largest fitness over the wave's lanes and the lowest joint index that has it.
__device__ __forceinline__ void wave_best(double &f, uint32_t &x)
{
    double m = f;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double y = __longlong_as_double((long long)shfl_xor64((unsigned long long)__double_as_longlong(m), o));
        m = y > m ? y : m;
    }
    const unsigned long long at = __ballot(f == m);
    uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)x, at ? (int)__ffsll((long long)at) - 1 : 0);
    if (__ballot(f == m && x != b)) {   // several configurations with the best fitness
        uint32_t y = f == m ? x : 0xFFFFFFFFu;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t z = xor_lane32(y, o);
            y = z < y ? z : y;
        }
        b = y;
    }
    f = m;
    x = b;
}

// FIXED: fitness from the table of option rows; otherwise from the table of
// configurations.  QP: parent pairs per thread.  MAXN: bound on the number of
// models.
//
// Bound by latency and, at 1,024 pairs, by the instructions of one CU per
// scenario: individuals are kept as packed digits, so that crossover and
// mutation are a few 64-bit masks, and a generation's candidates, parents and
// rows are read in three dependent LDS steps.  64 scenarios, 2,048 x 100
// generations: 5.1 us per generation here (35 us as two launches), 1.55 ms for
// the whole run with the draws (0.78 ms) and the table (0.19 ms), 3.75 ms
// before; one scenario, 100 x 30: 3.9 us per generation, 225 us against 739 us.
template <bool FIXED, int QP, int MAXN>
__global__ void __launch_bounds__(kRunMaxThreads) ga_run_kernel(const GARunArgs r)
{
    const GAConst &c = r.c;
    constexpr int DW = (MAXN + 7) / 8, SELW = 8, SWAP = 4 * DW, MUT = 6 * DW, CX = 14 * DW, SEL = CX + 1,
                  WORDS = SEL + SELW;
    extern __shared__ float4 dyn4[];
    char *dyn = reinterpret_cast<char *>(dyn4);
    __shared__ float s_tau[kMaxN];
    __shared__ int32_t s_prev[kMaxN];
    __shared__ double s_inv[kMaxN];
    __shared__ double s_ef[kRunMaxThreads / 64];
    __shared__ uint32_t s_ei[kRunMaxThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, threads = (int)blockDim.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), waves = threads >> 6;
    const int N = c.N, P = r.P, S = r.S, np = P / 2, s = blockIdx.x;
    const bool eq3 = c.obj.kind != 0;
    const RunLds ly(c, P, FIXED);
    double *fit = reinterpret_cast<double *>(dyn + ly.fit);
    uint64_t *dig = reinterpret_cast<uint64_t *>(dyn + ly.dig);      // [P][DW]
    uint32_t *idx = reinterpret_cast<uint32_t *>(dyn + ly.idx);
    FixedRow *rows = reinterpret_cast<FixedRow *>(dyn + ly.rows);    // FIXED: q, VRAM, flags; else VRAM only
    FixedPen *pens = reinterpret_cast<FixedPen *>(dyn + ly.pens);

    // ---- the scenario's tables
#pragma unroll
    for (int i = 0; i < kMaxN; i++)   // compile-time index into the argument block
        if (tid == i) {
            s_tau[i] = c.obj.tau[i];
            s_prev[i] = c.obj.prev[i];
            s_inv[i] = i < N ? 1.0 / (double)c.K[i] : 0.0;
        }
    double om[MAXN];
    float bound[MAXN];
    uint32_t stride[MAXN];   // joint index = sum of digit x stride
    {
        uint32_t st = 1;
#pragma unroll
        for (int i = MAXN - 1; i >= 0; i--) {
            om[i] = i < N ? (double)r.omega[(int64_t)s * N + i] : 0.0;
            bound[i] = i < N ? r.sla[(int64_t)s * N + i] : 0.f;
            stride[i] = i < N ? st : 0u;
            st *= i < N ? (uint32_t)c.K[i] : 1u;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MAXN; i++)
        if (i < N)
            for (int o = tid; o < c.K[i]; o += threads) {
                const int row = c.opt_off[i] + o;
                FixedRow x = {0.0, c.features[(int64_t)row * c.L + c.vram_col], 0u};
                if (FIXED) {
                    const double2 y = r.lat_thr[row];
                    x.q = y.y;
                    x.flags = y.x <= (double)bound[i] ? 0u : kRowBad;
                    if (eq3) {
                        FixedPen pp = {0.0, 0.0};
                        bool do_P, do_pen;
                        if (!canon_eq3(c.obj, row, y.y, s_tau[i], s_prev[i], x.q, pp.P, do_P, pp.pen, do_pen))
                            x.flags = kRowBad;
                        // +0 where a penalty does not apply: subtracting it
                        // changes no value, so the chain has no test
                        pens[row] = FixedPen{do_P ? pp.P : 0.0, do_pen ? pp.pen : 0.0};
                    }
                }
                rows[row] = x;
            }
    const unsigned long long n_fl = *r.n_fl;
    double bestJ = -INFINITY;
    uint64_t bestI = ~0ull;
    if (!r.init && tid == 0) {
        bestJ = r.best_J[s];
        bestI = r.best_idx[s];
    }
    __syncthreads();

    auto gene = [&](const uint64_t (&d)[DW], int i) { return (uint32_t)(d[i / 8] >> (8 * (i % 8))) & 0xFFu; };
    // digits of a joint index, by a reciprocal (the half added keeps the
    // product clear of the integers: exact below 2^32)
    auto digits_of = [&](uint32_t x, uint64_t (&d)[DW]) {
#pragma unroll
        for (int w = 0; w < DW; w++) d[w] = 0;
#pragma unroll
        for (int i = MAXN - 1; i >= 0; i--)
            if (i < N) {
                const uint32_t q = (uint32_t)(((double)x + 0.5) * s_inv[i]);
                d[i / 8] |= (uint64_t)(x - q * (uint32_t)c.K[i]) << (8 * (i % 8));
                x = q;
            }
    };
    auto index_of = [&](const uint64_t (&d)[DW]) {
        uint32_t x = 0;
#pragma unroll
        for (int i = 0; i < MAXN; i++)
            if (i < N) x += gene(d, i) * stride[i];
        return x;
    };
    auto vram_of = [&](const uint64_t (&d)[DW]) {
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < MAXN; i++)
            if (i < N) v = v + rows[(uint32_t)c.opt_off[i] + gene(d, i)].vram;
        return v;
    };
    // canonical J of a configuration within the VRAM cap: the models' terms in
    // order, from the table of rows, or its entry in the table of configurations
    auto fitness = [&](uint32_t x, const uint64_t (&d)[DW]) {
        double J = 0.0;
        bool ok = n_fl != 0;   // none feasible: index 0 throughout, never scored
        if constexpr (FIXED) {
            uint32_t fl = 0u;
#pragma unroll
            for (int i = 0; i < MAXN; i++)
                if (i < N) {
                    const uint32_t row = (uint32_t)c.opt_off[i] + gene(d, i);
                    const FixedRow y = rows[row];
                    fl |= y.flags;
                    J = fma(om[i], y.q, J);
                    if (eq3) {
                        const FixedPen pp = pens[row];
                        J = (J - pp.P) - pp.pen;
                    }
                }
            ok = ok && (int32_t)fl >= 0;
        } else {
            return ok ? r.fit_table[(int64_t)s * (int64_t)c.space + x] : -INFINITY;
        }
        return ok ? J : -INFINITY;
    };

    // each thread's own records, read one generation ahead
    const int words = GaRecord(r.tk, N).words;   // (N > 8 exactly when DW == 2)
    uint32_t rec[QP][WORDS];
    auto fetch = [&](int g) {
#pragma unroll
        for (int qp = 0; qp < QP; qp++) {
            const int q = qp * threads + tid;
            const uint32_t *gr = reinterpret_cast<const uint32_t *>(r.recs) + ((int64_t)(g - r.g0) * S + s) * np * words + q;
            if (q < np)
#pragma unroll
                for (int w = 0; w < WORDS; w++)
                    if (w < words) rec[qp][w] = gr[(int64_t)w * np];
        }
    };
    if (r.g0 < r.g1) fetch(r.g0);

    // ---- the first generation's population and its fitness
    double slot0 = 0.0;   // thread 0: the fitness in slot 0
    double ef = -INFINITY;
    uint32_t ei = 0xFFFFFFFFu;
    auto offer = [&](double f, uint32_t x) {   // the lane's best (f desc, index asc)
        if (f > ef || (f == ef && x < ei)) {
            ef = f;
            ei = x;
        }
    };
    for (int j = tid; j < P; j += threads) {
        uint32_t x;
        if (r.init)
            // no VRAM-feasible configuration: index 0 throughout
            x = n_fl ? r.fl[ga_below(ga_draw(r.seed, (uint64_t)j, 0, (uint64_t)s, kPInit, 0), n_fl)] : 0u;
        else
            x = (uint32_t)r.pop[(int64_t)s * P + j];
        uint64_t d[DW];
        digits_of(x, d);
        const double f = fitness(x, d);
        idx[j] = x;
        fit[j] = f;
        if (j == 0) slot0 = f;
#pragma unroll
        for (int w = 0; w < DW; w++) dig[j * DW + w] = d[w];
        offer(f, x);
    }
    __syncthreads();

    for (int g = r.g0;; g++) {
        // elite: the best of the generation, from what each lane built of it
        wave_best(ef, ei);
        if (lane == 0) {
            s_ef[wv] = ef;
            s_ei[wv] = ei;
        }
        const bool last = g == r.g1;
        uint32_t ci[QP][2];
        uint64_t cd[QP][2][DW];
        double cf[QP][2];
        ef = -INFINITY;
        ei = 0xFFFFFFFFu;
        if (!last) {
#pragma unroll
            for (int qp = 0; qp < QP; qp++) {
                const int q = qp * threads + tid;
                if (q >= np) continue;
                // tournaments: best (f desc, index asc), the earliest of equals
                uint64_t par[2][DW];
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    double fp = 0.0;
                    uint32_t xp = 0, jp = 0;
                    // candidates t k .. t k + k - 1 (16 bits each)
                    auto cand = [&](int m) {
                        uint32_t w = 0;
#pragma unroll
                        for (int z = 0; z < SELW; z++) w = (m >> 1) == z ? rec[qp][SEL + z] : w;
                        return (w >> (16 * (m & 1))) & 0xFFFFu;
                    };
                    if (r.tk == 3) {   // the usual size: candidates read together
                        const uint32_t j0 = t ? rec[qp][SEL + 1] >> 16 : rec[qp][SEL] & 0xFFFFu;
                        const uint32_t j1 = t ? rec[qp][SEL + 2] & 0xFFFFu : rec[qp][SEL] >> 16;
                        const uint32_t j2 = t ? rec[qp][SEL + 2] >> 16 : rec[qp][SEL + 1] & 0xFFFFu;
                        const double f0 = fit[j0], f1 = fit[j1], f2 = fit[j2];
                        const uint32_t x0 = idx[j0], x1 = idx[j1], x2 = idx[j2];
                        fp = f0;
                        xp = x0;
                        jp = j0;
                        if (f1 > fp || (f1 == fp && x1 < xp)) {
                            fp = f1;
                            xp = x1;
                            jp = j1;
                        }
                        if (f2 > fp || (f2 == fp && x2 < xp)) jp = j2;
                    } else {
                        for (int m = 0; m < r.tk; m++) {
                            const uint32_t j = cand(t * r.tk + m);
                            const double f = fit[j];
                            const uint32_t x = idx[j];
                            if (m == 0 || f > fp || (f == fp && x < xp)) {
                                fp = f;
                                xp = x;
                                jp = j;
                            }
                        }
                    }
#pragma unroll
                    for (int w = 0; w < DW; w++) par[t][w] = dig[jp * DW + w];
                }
                const bool cx = rec[qp][CX] != 0u;
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int w = 0; w < DW; w++) {
                        auto u64 = [&](int at) {
                            return (uint64_t)rec[qp][at + 2 * w] | (uint64_t)rec[qp][at + 2 * w + 1] << 32;
                        };
                        const uint64_t sm = cx ? u64(SWAP) : 0ull;
                        const uint64_t mm = u64(MUT + t * 4 * DW), mv = u64(MUT + t * 4 * DW + 2 * DW);
                        cd[qp][t][w] = ((((par[t][w] & ~sm) | (par[1 - t][w] & sm)) & ~mm) | mv);
                    }
                float v[2];
#pragma unroll
                for (int t = 0; t < 2; t++) v[t] = vram_of(cd[qp][t]);
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    const bool over = !((double)v[t] <= (double)c.vram_cap);   // repaired
#pragma unroll
                    for (int w = 0; w < DW; w++)
                        if (over)
                            cd[qp][t][w] = (uint64_t)rec[qp][t * 2 * DW + 2 * w] |
                                           (uint64_t)rec[qp][t * 2 * DW + 2 * w + 1] << 32;
                    ci[qp][t] = index_of(cd[qp][t]);
                }
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    cf[qp][t] = fitness(ci[qp][t], cd[qp][t]);
                    if (1 + 2 * q + t < P) offer(cf[qp][t], ci[qp][t]);
                }
            }
            if (g + 1 < r.g1) fetch(g + 1);
        }
        __syncthreads();
        // every read of this generation is done
        if (wv == 0) {
            double f = lane < waves ? s_ef[lane] : -INFINITY;
            uint32_t x = lane < waves ? s_ei[lane] : 0xFFFFFFFFu;
            wave_best(f, x);
            if (f > -INFINITY && ga_better(f, (uint64_t)x, bestJ, bestI)) {
                bestJ = f;
                bestI = (uint64_t)x;
            }
            // slot 0 goes to the elite.  A NaN there stays (nothing compares
            // above it), also when every fitness is NaN and x is no index
            if (tid == 0 && !last && slot0 == slot0) {
                slot0 = f;
                fit[0] = f;
                idx[0] = x;
                uint64_t d[DW];
                digits_of(x, d);
#pragma unroll
                for (int w = 0; w < DW; w++) dig[w] = d[w];
                offer(f, x);   // slot 0 of the next generation
            }
        }
        if (last) break;
#pragma unroll
        for (int qp = 0; qp < QP; qp++) {
            const int q = qp * threads + tid;
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const int j = 1 + 2 * q + t;
                if (q < np && j < P) {
                    idx[j] = ci[qp][t];
                    fit[j] = cf[qp][t];
#pragma unroll
                    for (int w = 0; w < DW; w++) dig[j * DW + w] = cd[qp][t][w];
                }
            }
        }
        __syncthreads();
    }
    if (r.g1 == r.gens) {
        if (r.final_pop)
            for (int j = tid; j < P; j += threads) r.final_pop[(int64_t)s * P + j] = n_fl ? (uint64_t)idx[j] : ~0ull;
    } else {
        for (int j = tid; j < P; j += threads) r.pop[(int64_t)s * P + j] = idx[j];
    }
    if (tid == 0) {
        r.best_J[s] = bestJ;
        r.best_idx[s] = bestI;
    }
}

// A thread per pair, up to 1,024 (then two pairs per thread: populations go
// up to 4,096).
static int run_threads(int P)
{
    const int t = (P / 2 + 63) & ~63;
    return t > kRunMaxThreads ? kRunMaxThreads : t;
}

constexpr size_t kRunLdsMax = 163840 - 1024;   // its static LDS takes below 1 KiB

bool ga_run_supported(const GAConst &c, int P, int tk) { return RunLds(c, P, c.fixed != 0).total <= kRunLdsMax; }

hipError_t launch_ga_run(const GARunArgs &r, hipStream_t st)
{
    const bool fixed = r.c.fixed != 0;
    const int threads = run_threads(r.P), N = r.c.N;
    const size_t lds = RunLds(r.c, r.P, fixed).total;
    const bool two = r.P / 2 > threads;   // at most two pairs per thread (populations up to 4,096)
    auto pick = [&](auto f6, auto f8, auto f16) { return N <= 6 ? f6 : (N <= 8 ? f8 : f16); };
    auto fn = fixed ? (two ? pick(ga_run_kernel<true, 2, 6>, ga_run_kernel<true, 2, 8>, ga_run_kernel<true, 2, 16>)
                           : pick(ga_run_kernel<true, 1, 6>, ga_run_kernel<true, 1, 8>, ga_run_kernel<true, 1, 16>))
                    : (two ? pick(ga_run_kernel<false, 2, 6>, ga_run_kernel<false, 2, 8>, ga_run_kernel<false, 2, 16>)
                           : pick(ga_run_kernel<false, 1, 6>, ga_run_kernel<false, 1, 8>, ga_run_kernel<false, 1, 16>));
    const hipError_t e = ensure_dyn_lds((const void *)fn, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(r.S), dim3(threads), lds, st, r);
    return hipGetLastError();
}

}  // namespace mfi
