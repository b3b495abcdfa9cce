// Separable searches by meet in the middle: the fixed-state search (Section
// III-B) and the static search over T steps (Section IV-C), whole blocks, no
// per-configuration output.
//
// With the observed state held fixed every configuration's value is a chain
// of per-option terms, so the joint space factors into a prefix (models 0 ..
// j0 - 1) and a suffix (the rest, S <= 4,096 combinations).  Scanning all
// prefix x suffix pairs (the general scan) costs one chain step per
// configuration; here each prefix costs one binary search:
//
//   VRAM   fl(x + v) is monotone in x, so the fp32 chain of the suffix stays
//          within the cap exactly when the prefix's sum is at most a
//          threshold of the suffix, found by inverting the rounded additions
//          from the cap backwards (vram_inverse).  With the suffixes sorted by
//          threshold, a prefix's VRAM-feasible suffixes are the first `pos`.
//   counts pos, and the number of good suffixes (no service constraint
//          failed; a constraint depends on one row only) among the first pos.
//   top-k  a prefix's best J is within `slack` of its own sum of terms plus
//          the largest sum of terms over the good suffixes among the first
//          pos (a running maximum): slack bounds the rounding of every chain
//          involved.  The k prefixes of the largest bounds give a lower bound
//          theta of the k-th J; only prefixes whose bound reaches theta are
//          looked into, and in them only the suffixes whose own sum reaches
//          it are evaluated, by the canonical chain.
//
// One launch: every workgroup of 1,024 threads builds and sorts the suffix
// table in LDS (its own copy: cheaper than a launch that builds it once) and
// its lanes take prefixes.  The last workgroup to finish (a ticket, no
// waiting) takes the largest bounds the waves hand on, selects the candidate
// prefixes, evaluates their hits and writes the result.  When a wave of a grid
// may have kept back a prefix that reaches theta (many equal bounds), when more
// prefixes reach it than the last workgroup takes, or a term is not finite, the
// result says so and the host runs the general scan.
//
// Bound by latency: some 15 dependent LDS phases of 2-4 us each, no unit busy.
// Whole searches, call to host result, general scan before -> now (MI355X):
// 24^6 configurations, top-1: 153 us -> 76-79 us (kernel 48); 16^8, top-64:
// 2,610 us -> 112-230 us by the input (kernel 78 and more: the evaluation of
// what reaches theta); 104,976 (Eq. 3, top-1): 78 us -> 54-58 us (kernel 26);
// the same over 12 steps: 276 us -> 93-100 us (kernel 28).
#include <type_traits>

#include "mf_canon.h"

namespace mfi {

constexpr int kMitmThreads = 1024;
constexpr int kMitmWaves = kMitmThreads / 64;
constexpr int kMitmCand = 1024;      // candidate prefixes the last workgroup takes
constexpr int kMitmHits = 512;       // configurations evaluated a thread each
// One workgroup whose list is full of bounds that reach the cut (prefixes that
// tie: models of no weight, equal options) takes its candidates from all its
// prefixes again.  Where the tie goes through the suffixes too, every one of
// them is a hit: beyond this many (about 2 ns each at 8 models) the search is
// left to the scan.  12x12x9x9x9 with two models of no weight, k = 1: 107 us a
// call; 140 when a full list goes to the scan, 127 for the scan alone.  Every J
// equal (no model has a weight): 147 against 126, lost before the scan.
constexpr uint32_t kMitmTieHits = 4096;

// Dynamic LDS.  While the suffixes are built level by level, their thresholds
// alternate between lst and G and their sums between M and Bs.
struct MitmLds {
    FixedRow *rows;               // [sumK] per option row: sum over steps of its terms, VRAM, flags
    FixedRow *raw;                // [n_steps][sumK] the rows as given (when staged)
    FixedPen *rawpen;             // [n_steps][sumK] (Eq. 3, when staged)
    unsigned long long *key;      // [spad] threshold (order-preserving bits) << 32 | ~u, descending
    double *Bs;                   // [spad] sum of terms by sorted position (-inf: a constraint fails)
    double *M;                    // [spad + 2] largest Bs of the first i positions
    unsigned long long *lst;      // [waves][128] list merge; then the exact keys
    uint32_t *G;                  // [spad + 4] good suffixes among the first i positions
};

__device__ __forceinline__ MitmLds mitm_lds(float4 *smem, int n_steps, int sumK, uint32_t spad, uint32_t raw_bytes)
{
    MitmLds l;
    l.rows = reinterpret_cast<FixedRow *>(smem);
    l.raw = l.rows + sumK;
    l.rawpen = reinterpret_cast<FixedPen *>(l.raw + (size_t)n_steps * sumK);
    l.key = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(l.raw) + raw_bytes);
    l.Bs = reinterpret_cast<double *>(l.key + spad);
    l.M = l.Bs + spad;
    l.lst = reinterpret_cast<unsigned long long *>(l.M + spad + 2);
    l.G = reinterpret_cast<uint32_t *>(l.lst + kMitmWaves * 128);
    return l;
}

size_t mitm_lds_bytes(int sumK, uint32_t spad)
{
    return (size_t)sumK * sizeof(FixedRow) + (size_t)spad * 16 + (size_t)(spad + 2) * 8 + kMitmWaves * 128 * 8 +
           (size_t)(spad + 4) * 4;
}

// Rows as given are staged up to this many bytes, where the tables leave room
// (read from memory otherwise: they are used once for the sums and for the few
// configurations evaluated).
constexpr size_t kMitmRawBytes = 32768;

uint32_t mitm_raw_bytes(int n_steps, int sumK, uint32_t spad, bool eq3)
{
    const size_t b = (size_t)n_steps * sumK * (sizeof(FixedRow) + (eq3 ? sizeof(FixedPen) : 0));
    return b <= kMitmRawBytes && mitm_lds_bytes(sumK, spad) + b <= kMitmLdsMax ? (uint32_t)b : 0;
}

// A prefix of the launch: its exact VRAM sum (fp32, model order), the sum of
// its terms and its flags.
struct Prefix {
    float v;
    double B;
    uint32_t fl;
};

// Per model in LDS: option count, magic quotient, first row, digit of the
// launch's first prefix.
struct MitmModel {
    uint32_t K, magic, off, base;
};

// t / K for t < 2^24.
__device__ __forceinline__ uint32_t mitm_div(const MitmModel &m, uint32_t t) { return m.magic ? __umulhi(t, m.magic) : t; }

template <int MAXN>
__device__ __forceinline__ Prefix mitm_prefix(const MitmArgs &a, const MitmModel *mm, const FixedRow *rows, uint32_t prel)
{
    Prefix p = {0.f, 0.0, 0u};
    uint32_t d[MAXN];
    uint32_t carry = prel;
#pragma unroll
    for (int j = MAXN - 1; j >= 0; j--) {
        d[j] = 0;
        if (j < a.j0) {
            const MitmModel m = mm[j];
            const uint32_t t = m.base + carry, q = mitm_div(m, t);
            d[j] = m.off + (t - q * m.K);
            carry = q;
        }
    }
#pragma unroll
    for (int j = 0; j < MAXN; j++)
        if (j < a.j0) {
            const FixedRow r = rows[d[j]];
            p.v += r.vram;
            p.B += r.q;
            p.fl |= r.flags;
        }
    return p;
}

// The number of sorted suffixes whose threshold is at least v.
__device__ __forceinline__ uint32_t mitm_pos(const unsigned long long *key, uint32_t spad, float v)
{
    const uint32_t o = ord_f32(v + 0.f);   // -0 compares as +0
    uint32_t pos = 0;
    for (uint32_t b = spad >> 1; b > 0; b >>= 1)
        if (o <= (uint32_t)(key[pos + b - 1] >> 32)) pos += b;
    if (o <= (uint32_t)(key[pos] >> 32)) pos++;
    return pos;
}

// The canonical value of configuration (prefix, suffix) over steps [t0, t1)
// and its flags: each step's chain over all models in order, summed in step
// order.
template <int MAXN, bool EQ3>
__device__ inline double mitm_exact(const MitmArgs &a, const MitmModel *mm, const FixedRow *rows, const FixedPen *pens,
                                    int t0, int t1, uint32_t prel, uint32_t u, float &v, uint32_t &fl)
{
    uint64_t dig[MAXN / 8] = {};   // 8 bits per model
    uint32_t carry = prel, uu = u;
#pragma unroll
    for (int j = MAXN - 1; j >= 0; j--)
        if (j < a.n_models) {
            const MitmModel m = mm[j];
            const uint32_t t = j >= a.j0 ? uu : m.base + carry, q = mitm_div(m, t);
            dig[j / 8] |= (uint64_t)(t - q * m.K) << (8 * (j % 8));
            if (j >= a.j0) uu = q;
            else carry = q;
        }
    v = 0.f;
    fl = 0u;
    double S = 0.0;
    for (int t = t0; t < t1; t++) {
        const FixedRow *rs = rows + (int64_t)t * a.sumK;
        const FixedPen *ps = pens + (int64_t)t * a.sumK;
        const float *om = a.omega + t * a.n_models;
        double J = 0.0;
#pragma unroll 4
        for (int j = 0; j < a.n_models; j++) {
            uint64_t w = dig[0];
            if (MAXN > 8 && j >= 8) w = dig[MAXN / 8 - 1];
            const uint32_t row = mm[j].off + (uint32_t)((w >> (8 * (j & 7))) & 0xFFu);
            const FixedRow r = rs[row];
            if (t == t0) v += r.vram;
            fl |= r.flags;
            J = fma((double)om[j], r.q, J);
            if (EQ3) {
                const FixedPen pp = ps[row];
                if (r.flags & kRowP) J = J - pp.P;
                if (r.flags & kRowPen) J = J - pp.pen;
            }
        }
        S = t == t0 ? J : S + J;
    }
    return S;
}

template <int MAXN, int NS, bool EQ3>
__global__ void __launch_bounds__(kMitmThreads) mitm_kernel(const MitmArgs a)
{
    extern __shared__ float4 smem4[];
    constexpr int kp = 64 * NS;
    __shared__ unsigned long long s_mag[kMaxN];      // largest magnitude of a row's terms, per model (bits)
    __shared__ unsigned long long s_cnt[2 * kMitmWaves];
    __shared__ double s_segmax[64];                  // largest Bs per 64 sorted positions
    __shared__ double s_wmax[kMitmWaves];
    __shared__ uint32_t s_wcnt[kMitmWaves];
    __shared__ double s_theta;
    __shared__ unsigned long long s_cut;
    __shared__ uint32_t s_last, s_ncand, s_bad, s_nhit, s_full;
    __shared__ unsigned long long s_hit[kMitmHits];
    __shared__ uint32_t s_cand[kMitmCand];
    __shared__ unsigned long long s_t0;
    __shared__ MitmModel s_m[kMaxN];
    __shared__ float s_hi[kMitmWaves], s_lo[kMitmWaves];
    __shared__ uint32_t s_big;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = a.n_models, T = a.n_steps, sumK = a.sumK, k = a.top_k;
    const uint32_t S = a.S, spad = a.spad;
    const MitmLds l = mitm_lds(smem4, T, sumK, spad, a.raw_bytes);
    const bool staged = a.raw_bytes != 0u;
    unsigned long long t_start = 0;
    if (tid == 0) {
        t_start = (unsigned long long)wall_clock64();
        s_ncand = 0;
        s_bad = 0;
        s_nhit = 0;
        s_t0 = t_start;
        s_big = 0;
    }
    if (tid < kMaxN) s_mag[tid] = 0ull;
#pragma unroll
    for (int j = 0; j < MAXN; j++)   // compile-time index into the argument block
        if (tid == j) s_m[j] = MitmModel{(uint32_t)a.K[j], a.magic[j], (uint32_t)a.opt_off[j], a.base_digits[j]};
    if (tid < 64) s_segmax[tid] = -INFINITY;
    if (staged)
        for (int e = tid; e < T * sumK; e += kMitmThreads) {
            l.raw[e] = a.rows[e];
            if (EQ3) l.rawpen[e] = a.pens[e];
        }
    const FixedRow *rows_x = staged ? l.raw : a.rows;
    const FixedPen *pens_x = staged ? l.rawpen : a.pens;
    __syncthreads();

    // ---- every option row's terms summed over the steps
    for (int r = tid; r < sumK; r += kMitmThreads) {
        const int i = a.row_model[r];
        double B = 0.0, mag = 0.0;
        float v = 0.f;
        uint32_t fl = 0u;
#pragma unroll 4
        for (int t = 0; t < T; t++) {
            const FixedRow x = rows_x[(int64_t)t * sumK + r];
            const double q = (double)a.omega[t * N + i] * x.q;
            B += q;
            mag += fabs(q);
            if (EQ3) {
                const FixedPen pp = pens_x[(int64_t)t * sumK + r];
                if (x.flags & kRowP) {
                    B -= pp.P;
                    mag += fabs(pp.P);
                }
                if (x.flags & kRowPen) {
                    B -= pp.pen;
                    mag += fabs(pp.pen);
                }
            }
            v = x.vram;
            fl |= x.flags;
        }
        l.rows[r] = FixedRow{B, v, fl};
        atomicMax(&s_mag[i], (unsigned long long)__double_as_longlong(mag));   // NaN bits exceed every finite value's
    }
    __syncthreads();
    // slack: no chain (prefix + suffix sums, or the canonical one) rounds more
    // than 3 T N + T + N times, each by at most 2^-53 of what it holds
    double mag = 0.0;
    for (int i = 0; i < N; i++) mag += __longlong_as_double((long long)s_mag[i]);
    const double slack = mag * ((double)(4 * T * N + 2 * T + 2 * N + 16) * 0x1p-51);
    const bool finite = mag < 1e290;

    // ---- the suffixes, one model at a time from the last: threshold and sum
    // of terms (-inf when a constraint fails) of every combination so far
    float *thr_a = reinterpret_cast<float *>(l.lst), *thr_b = reinterpret_cast<float *>(l.G);
    double *sum_a = l.M, *sum_b = l.Bs;
    if ((N - a.j0) & 1) {   // the last level ends in lst and M
        float *x = thr_a;
        thr_a = thr_b;
        thr_b = x;
        double *y = sum_a;
        sum_a = sum_b;
        sum_b = y;
    }
    if (tid == 0) {
        thr_a[0] = a.vram_cap;
        sum_a[0] = 0.0;
    }
    uint32_t size = 1;
    for (int j = N - 1; j >= a.j0; j--) {
        const uint32_t K = s_m[j].K, off = s_m[j].off, next = size * K;
        __syncthreads();
        for (uint32_t u = tid; u < next; u += kMitmThreads) {
            const uint32_t d = u / size, w = u - d * size;
            const FixedRow r = l.rows[off + d];
            thr_b[u] = vram_inverse(thr_a[w], r.vram);
            sum_b[u] = (int32_t)r.flags >= 0 ? r.q + sum_a[w] : -INFINITY;
        }
        size = next;
        float *x = thr_a;
        thr_a = thr_b;
        thr_b = x;
        double *y = sum_a;
        sum_a = sum_b;
        sum_b = y;
    }
    __syncthreads();
    // ---- sorted by threshold, descending: a counting sort over spad equal
    // intervals between the extremes, then each interval's few keys by one
    // thread.  (One bitonic sort over the keys took 12 us at 1,024 and 34 us
    // at 4,096; it remains for thresholds that crowd into one interval.)
    {
        const float *thr = thr_a;
        float hi = -INFINITY, lo = INFINITY;
        for (uint32_t u = tid; u < S; u += kMitmThreads) {
            const float x = thr[u];
            hi = x > hi ? x : hi;
            lo = x < lo && x > -INFINITY ? x : lo;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const float h2 = __shfl_xor(hi, o), l2 = __shfl_xor(lo, o);
            hi = h2 > hi ? h2 : hi;
            lo = l2 < lo ? l2 : lo;
        }
        if (lane == 0) {
            s_hi[wv] = hi;
            s_lo[wv] = lo;
        }
        for (uint32_t u = tid; u < spad; u += kMitmThreads) l.G[u] = 0u;
        __syncthreads();
        for (int w = 0; w < kMitmWaves; w++) {
            hi = s_hi[w] > hi ? s_hi[w] : hi;
            lo = s_lo[w] < lo ? s_lo[w] : lo;
        }
        const float range = hi - lo, top = (float)(spad - 1);
        const float scale = range > 1e-30f && range < INFINITY ? top / range : 0.f;
        // monotone in the threshold, the infinite ones at the end
        auto bucket = [&](float x) {
            const float y = (hi - x) * scale;
            return x == -INFINITY ? spad - 1 : (uint32_t)(y < top ? y : top);
        };
        for (uint32_t u = tid; u < S; u += kMitmThreads) atomicAdd(&l.G[bucket(thr[u])], 1u);
        __syncthreads();
        const uint32_t per = spad > kMitmThreads ? spad / kMitmThreads : 1, b0 = tid * per;
        uint32_t c = 0, big = 0;
        for (uint32_t i = b0; i < b0 + per && i < spad; i++) {
            const uint32_t x = l.G[i];
            c += x;
            big = x > big ? x : big;
        }
        uint32_t wc = c;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t oc = __shfl_up(wc, o);
            if (lane >= o) wc += oc;
        }
        if (lane == 63) s_wcnt[wv] = wc;
        if (big > 24) atomicOr(&s_big, 1u);
        __syncthreads();
        uint32_t at = wc - c;
        for (int w = 0; w < wv; w++) at += s_wcnt[w];
        for (uint32_t i = b0; i < b0 + per && i < spad; i++) {
            const uint32_t x = l.G[i];
            l.G[i] = at;
            at += x;
        }
        __syncthreads();
        for (uint32_t u = tid; u < spad; u += kMitmThreads) {
            if (u < S) {
                const float x = thr[u];
                l.key[atomicAdd(&l.G[bucket(x)], 1u)] =
                    ((unsigned long long)ord_f32(x) << 32) | (unsigned long long)(0xFFFFFFFFu - u);
            } else {
                l.key[u] = 0ull;
            }
        }
        __syncthreads();
        if (s_big == 0u) {
            // G[b] is now the end of interval b
            for (uint32_t b = tid; b < spad; b += kMitmThreads) {
                const uint32_t e0 = b ? l.G[b - 1] : 0u, e1 = l.G[b];
                for (uint32_t i = e0 + 1; i < e1; i++) {
                    const unsigned long long x = l.key[i];
                    uint32_t q = i;
                    while (q > e0 && l.key[q - 1] < x) {
                        l.key[q] = l.key[q - 1];
                        q--;
                    }
                    l.key[q] = x;
                }
            }
        } else {
            // pairs at distance 64 or less stay within a wave's own 128 keys
            for (uint32_t kk = 2; kk <= spad; kk <<= 1)
                for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
                    for (uint32_t t = tid; t < spad / 2; t += kMitmThreads) {
                        const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), o = i | j;
                        const unsigned long long x = l.key[i], y = l.key[o];
                        if ((x < y) == ((i & kk) == 0)) {
                            l.key[i] = y;
                            l.key[o] = x;
                        }
                    }
                    if (j > 64 || (j == 1 && kk >= 128)) __syncthreads();
                    else __builtin_amdgcn_wave_barrier();
                }
        }
        __syncthreads();
    }
    // sums of terms in sorted order, their running maximum and the running
    // count of good suffixes: `per` consecutive positions per thread
    {
        constexpr uint32_t kPer = kMitmSuffixMax / kMitmThreads;
        const uint32_t per = spad > kMitmThreads ? spad / kMitmThreads : 1, b0 = tid * per;
        double m = -INFINITY, B[kPer];
        uint32_t c = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPer; q++) {
            const uint32_t i = b0 + q;
            B[q] = q < per && i < S ? sum_a[0xFFFFFFFFu - (uint32_t)(l.key[i] & 0xFFFFFFFFull)] : -INFINITY;
            m = B[q] > m ? B[q] : m;
            c += B[q] > -INFINITY ? 1u : 0u;
        }
        // exclusive scan over the threads
        double wm = m;
        uint32_t wc = c;
        for (int o = 1; o < 64; o <<= 1) {
            const double om = __shfl_up(wm, o);
            const uint32_t oc = __shfl_up(wc, o);
            if (lane >= o) {
                wm = om > wm ? om : wm;
                wc += oc;
            }
        }
        if (lane == 63) {
            s_wmax[wv] = wm;
            s_wcnt[wv] = wc;
        }
        double em = __shfl_up(wm, 1);
        uint32_t ec = __shfl_up(wc, 1);
        if (lane == 0) {
            em = -INFINITY;
            ec = 0;
        }
        __syncthreads();   // sum_a is M: every thread has read its sums
        for (int w = 0; w < wv; w++) {
            em = s_wmax[w] > em ? s_wmax[w] : em;
            ec += s_wcnt[w];
        }
#pragma unroll
        for (uint32_t q = 0; q < kPer; q++) {
            const uint32_t i = b0 + q;
            if (q < per && i < spad) {
                l.M[i] = em;
                l.G[i] = ec;
                l.Bs[i] = B[q];
                em = B[q] > em ? B[q] : em;
                ec += B[q] > -INFINITY ? 1u : 0u;
                if (i == spad - 1) {
                    l.M[spad] = em;
                    l.G[spad] = ec;
                }
            }
        }
        __syncthreads();
    }

    // ---- the prefixes.  One workgroup: each wave keeps a sorted list of its
    // largest bounds.  A grid: prefixes go to the waves in turn, each round
    // rotated by a fixed step (prefixes that share options have the best
    // bounds together: a run of neighbours, or a stride of whole digits,
    // would give one wave many of them), each lane keeps its two largest bounds and the largest it dropped, and the
    // wave hands on the `a.list` largest of the kept ones (descending), then the
    // largest of all the others: sorted lists of 128 in every wave and their merges took 70 of
    // 145 us at 2^20 prefixes.
    const int grid = (int)gridDim.x;
    // a prefix's key: an upper bound of its best J, its order-preserving bits
    // rounded up to 40, then the lowest prefix (0: no feasible suffix); pos
    // suffixes meet the cap, g of them the service constraints too
    auto prefix_key = [&](uint32_t p, uint32_t &pos, uint32_t &g) {
        const Prefix x = mitm_prefix<MAXN>(a, s_m, l.rows, p);
        pos = mitm_pos(l.key, spad, x.v);
        g = (int32_t)x.fl >= 0 ? l.G[pos] : 0u;
        return g ? (((ord_f64((x.B + l.M[pos]) + slack) >> 24) + 1) << 24) | (unsigned long long)(0xFFFFFFu - p) : 0ull;
    };
    WaveList<NS> L;
    wl_init(L);
    unsigned long long cv = 0, cf = 0, m1 = 0ull, m2 = 0ull, m3 = 0ull;
    const uint32_t n_waves = (uint32_t)grid * kMitmWaves, gw = blockIdx.x * kMitmWaves + wv;
    const uint32_t n_whole = a.whole_hi - a.whole_lo;
    const uint32_t step = (uint32_t)(0.618034f * (float)n_waves);
    for (uint32_t i0 = 0; grid > 1 ? i0 * n_waves < n_whole : i0 * n_waves + gw * 64u < n_whole; i0 += 64u) {
        // below 2^32: the rounds number at most 2^23 / n_waves + 64
        const uint32_t round = i0 + lane;
        const uint32_t r = grid > 1 ? round * n_waves + (gw + round * step) % n_waves : i0 * n_waves + gw * 64u + lane;
        unsigned long long key = 0ull;
        if (r < n_whole) {
            uint32_t pos, g;
            key = prefix_key(a.whole_lo + r, pos, g);
            cv += pos;
            cf += g;
        }
        if (grid == 1) {
            wl_offer_many(L, key, lane, kp);
        } else {
            m3 = key > m2 ? m2 : (key > m3 ? key : m3);
            m2 = key > m1 ? m1 : (key > m2 ? key : m2);
            m1 = key > m1 ? key : m1;
        }
    }
    cv = wave_sum64(cv);
    cf = wave_sum64(cf);
    if (lane == 0) {
        s_cnt[wv] = cv;
        s_cnt[kMitmWaves + wv] = cf;
    }
    if (grid == 1) {
#pragma unroll
        for (int j = 0; j < NS; j++) l.lst[wv * kp + j * 64 + lane] = L.s[j];
        wl_tree_merge<NS, kMitmWaves>(L, l.lst, kp, wv, lane, kp);
    } else {
        unsigned long long mine = 0ull;
        for (int t = 0; t <= a.list; t++) {
            unsigned long long y = m1;
            if (t == a.list) y = m1 > m3 ? m1 : m3;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long z = shfl_xor64(y, o);
                y = z > y ? z : y;
            }
            if (m1 == y) {   // keys are distinct, so one lane (or none has any)
                m1 = m2;
                m2 = 0ull;
            }
            if (lane == t) mine = y;
        }
        if (lane <= a.list) a.wg_lists[(uint64_t)gw * (a.list + 1) + lane] = mine;
        __builtin_amdgcn_s_waitcnt(0);   // in the L2 before wave 0's release below
        __syncthreads();
    }
    unsigned long long tv = 0, tf = 0;   // wave 0, lanes 0 and 1: this workgroup's counts
    if (wv == 0) {
        unsigned long long c = 0;
        if (lane < 2)
            for (int w = 0; w < kMitmWaves; w++) c += s_cnt[lane * kMitmWaves + w];
        if (lane == 0) tv = c;
        if (lane == 1) tf = c;
        if (grid > 1) {
            if (lane < 2) a.wg_counts[4 * (uint64_t)blockIdx.x + lane] = c;
            if (lane == 0) a.wg_counts[4 * (uint64_t)blockIdx.x + 2] = t_start;
            // one wave releases the workgroup's results (every wave fencing
            // took 50 us over 256 workgroups: each fence writes back the L2)
            __threadfence();
            if (lane == 0) s_last = atomicAdd(a.ticket, 1u) == (uint32_t)(grid - 1) ? 1u : 0u;
        } else if (lane == 0) {
            s_last = 1u;
        }
    }
    __syncthreads();
    if (!s_last) return;

    // ==== the last workgroup: candidates, exact values, the result
    constexpr int kRec = kMitmMaxGrid * kMitmWaves / kMitmThreads;   // wave records per thread
    unsigned long long x[kRec] = {}, rest = 0ull;   // the thread's records: largest keys; largest key not handed on
    WaveList<NS> Q;   // wave 0: the largest bounds of all workgroups
    wl_init(Q);
    if (grid > 1) {
        __threadfence();
        unsigned long long best = 0ull;
#pragma unroll
        for (int q = 0; q < kRec; q++) {
            const uint32_t w = (uint32_t)(q * kMitmThreads + tid);
            unsigned long long y = 0ull;
            if (w < n_waves) {
                x[q] = a.wg_lists[(uint64_t)w * (a.list + 1)];
                y = a.wg_lists[(uint64_t)w * (a.list + 1) + a.list];
            }
            best = x[q] > best ? x[q] : best;
            rest = y > rest ? y : rest;
        }
        tv = tf = 0;
        if (tid < grid) {
            tv = a.wg_counts[4 * (uint64_t)tid];
            tf = a.wg_counts[4 * (uint64_t)tid + 1];
            atomicMin(&s_t0, a.wg_counts[4 * (uint64_t)tid + 2]);
        }
        // the 64 largest of the threads' maxima (distinct prefixes): the
        // k-th bounds the k-th largest bound of all from below
        wl_offer_many(Q, best, lane, kp);
#pragma unroll
        for (int j = 0; j < NS; j++) l.lst[wv * kp + j * 64 + lane] = Q.s[j];
        wl_tree_merge<NS, kMitmWaves>(Q, l.lst, kp, wv, lane, kp);
    } else if (wv == 0) {
#pragma unroll
        for (int j = 0; j < NS; j++) Q.s[j] = L.s[j];
    }
    if (wv == 0) {
        const unsigned long long kth = readlane64(Q.s[0], k - 1);   // k <= 64
        if (lane == 0) {
            // the k-th prefix holds a configuration at least this good
            const double w = kth ? unord_f64((((kth >> 24) - 1) << 24)) - 2.5 * slack : -INFINITY;
            s_theta = w;
            s_cut = kth ? ((ord_f64(w) >> 24) + 1) << 24 : 1ull;
        }
        // a full list whose last key reaches the cut may have dropped others
        const unsigned long long last = readlane64(Q.s[NS - 1], 63);
        if (lane == 0) s_full = grid == 1 && last >= s_cut ? 1u : 0u;
    }
    // the largest sum per 64 sorted positions
    for (uint32_t s = wv; s < (spad + 63) / 64; s += kMitmWaves) {
        double y = s * 64 + lane < spad ? l.Bs[s * 64 + lane] : -INFINITY;
        for (int o = 32; o > 0; o >>= 1) {
            const double z = __shfl_xor(y, o);
            y = z > y ? z : y;
        }
        if (lane == 0) s_segmax[s] = y;
    }
    __syncthreads();
    const double theta = s_theta;
    const unsigned long long cut = s_cut;
    const bool full = s_full != 0u;
    auto take = [&](unsigned long long key) {
        const uint32_t at = atomicAdd(&s_ncand, 1u);
        if (at < kMitmCand) s_cand[at] = 0xFFFFFFu - (uint32_t)(key & 0xFFFFFFull);
    };
    if (grid > 1) {
        // a lane's third key is in no list, so a wave may have kept back a key
        // above some that it handed on: the rest is tested whatever the list
        // holds
        if (rest >= cut) atomicOr(&s_bad, 1u);
#pragma unroll
        for (int q = 0; q < kRec; q++) {
            // the wave's keys from the cut up
            const unsigned long long *rec = a.wg_lists + (uint64_t)(q * kMitmThreads + tid) * (a.list + 1);
            unsigned long long key = x[q];
            for (int t = 1; key >= cut; t++) {
                take(key);
                if (t == a.list) break;
                key = rec[t];
            }
        }
    } else if (full) {
        for (uint32_t r = tid; r < n_whole; r += kMitmThreads) {
            uint32_t pos, g;
            const unsigned long long key = prefix_key(a.whole_lo + r, pos, g);
            if (key >= cut) take(key);
        }
    } else if (wv == 0) {
#pragma unroll
        for (int j = 0; j < NS; j++)
            if (Q.s[j] >= cut) take(Q.s[j]);
    }
    __syncthreads();
    const uint32_t ncand = s_ncand;
    bool general = ncand > kMitmCand || s_bad != 0u || !finite;   // the host runs the general scan
    // a thread per candidate prefix: its VRAM sum's position and its sum
    double *cand_B = reinterpret_cast<double *>(l.lst);                     // [kMitmCand]
    uint32_t *cand_pos = reinterpret_cast<uint32_t *>(cand_B + kMitmCand);  // [kMitmCand]
    static_assert(kMitmCand * 12 <= kMitmWaves * 128 * 8 && kMitmCand <= kMitmThreads, "candidates fit the list buffer");
    if (!general && (uint32_t)tid < ncand) {
        const Prefix c = mitm_prefix<MAXN>(a, s_m, l.rows, s_cand[tid]);
        cand_B[tid] = c.B;
        cand_pos[tid] = mitm_pos(l.key, spad, c.v);
    }
    __syncthreads();
    // a wave per candidate: the segments, then the suffixes, whose sum reaches
    // theta; f takes each group of 64 with the hits marked
    // (tie: stop once they are too many)
    auto each_hit = [&](auto tie, const double &bar, auto f) {
        for (uint32_t c = wv; !general && c < ncand; c += kMitmWaves) {
            const double B = cand_B[c];
            const uint32_t pos = cand_pos[c];
            unsigned long long segs = __ballot((uint32_t)lane * 64u < pos && (B + s_segmax[lane]) + slack >= bar);
            while (segs) {
                if (tie.value && *(volatile uint32_t *)&s_nhit > kMitmTieHits) return;
                const uint32_t i = ((uint32_t)__ffsll((long long)segs) - 1u) * 64u + lane;
                segs &= segs - 1;
                const bool hit = i < pos && l.Bs[i] > -INFINITY && (B + l.Bs[i]) + slack >= bar;
                if (__ballot(hit)) f(hit, s_cand[c], hit ? 0xFFFFFFFFu - (uint32_t)(l.key[i] & 0xFFFFFFFFull) : 0u);
            }
        }
    };
    K128 slot = {0ull, 0ull}, thr = {0ull, 0ull};
    double thrJ = theta;
    const bool parts = a.part_hi[0] != 0u || a.part_hi[1] != 0u;
    const auto count = [&](bool hit, uint32_t prel, uint32_t u) {
        if (hit) {
            const uint32_t at = atomicAdd(&s_nhit, 1u);
            if (at < kMitmHits) s_hit[at] = ((unsigned long long)prel << 32) | u;
        }
    };
    if (full) each_hit(std::true_type{}, theta, count);
    else each_hit(std::false_type{}, theta, count);
    __syncthreads();
    const uint32_t nhit = s_nhit;
    general = general || (full && nhit > kMitmTieHits);
    const bool few = nhit <= kMitmHits && !parts;
    if (!general && few) {
        // every hit's canonical value: T = 1 a thread per hit; otherwise a
        // wave per hit, a lane per step, the sum in step order
        if (T == 1) {
            if ((uint32_t)tid < nhit) {
                const uint32_t prel = (uint32_t)(s_hit[tid] >> 32), u = (uint32_t)s_hit[tid];
                float v;
                uint32_t fl;
                const double J = mitm_exact<MAXN, EQ3>(a, s_m, rows_x, pens_x, 0, 1, prel, u, v, fl);
                slot = K128{ord_f64(J), ~((a.prefix0 + prel) * (uint64_t)S + u)};
            }
        } else {
            K128 *hk = reinterpret_cast<K128 *>(l.lst);   // the candidates are done
            for (uint32_t h = wv; h < nhit; h += kMitmWaves) {
                const uint32_t prel = (uint32_t)(s_hit[h] >> 32), u = (uint32_t)s_hit[h];
                float v;
                uint32_t fl;
                const int t = lane < T ? lane : T - 1;
                const double J = mitm_exact<MAXN, EQ3>(a, s_m, rows_x, pens_x, t, t + 1, prel, u, v, fl);
                double sum = readlane_f64(J, 0);
                for (int q = 1; q < T; q++) sum = sum + readlane_f64(J, q);
                if (lane == 0) hk[h] = K128{ord_f64(sum), ~((a.prefix0 + prel) * (uint64_t)S + u)};
            }
            __syncthreads();
            if ((uint32_t)tid < nhit) slot = hk[tid];
        }
        slot = sort128_desc(slot, lane);
    } else if (!general) {
        // many (fewer than k prefixes feasible, or equal values): each wave's
        // running top-k
        each_hit(std::false_type{}, thrJ, [&](bool hit, uint32_t prel, uint32_t u) {
            K128 key = {0ull, 0ull};
            if (hit) {
                float v;
                uint32_t fl;
                const double J = mitm_exact<MAXN, EQ3>(a, s_m, rows_x, pens_x, 0, T, prel, u, v, fl);
                key = K128{ord_f64(J), ~((a.prefix0 + prel) * (uint64_t)S + u)};
            }
            list128_offer_many(slot, key, lane, k, thr);
            if (nz128(thr)) {
                const double kj = unord_f64(thr.hi);
                thrJ = kj > thrJ ? kj : thrJ;
            }
        });
    }
    // the blocks the range covers in part: every configuration evaluated
    for (int b = 0; !general && b < 2; b++) {
        const uint32_t ua = a.part_lo[b], ub = a.part_hi[b];
        for (uint32_t u0 = ua + wv * 64u; u0 < ub; u0 += kMitmThreads) {
            const uint32_t u = u0 + lane;
            K128 key = {0ull, 0ull};
            if (u < ub) {
                float v;
                uint32_t fl;
                const double J = mitm_exact<MAXN, EQ3>(a, s_m, rows_x, pens_x, 0, T, a.part_prefix[b], u, v, fl);
                const bool vok = v <= a.vram_cap, ok = vok && (int32_t)fl >= 0;
                tv += vok ? 1u : 0u;
                tf += ok ? 1u : 0u;
                if (ok && J >= thrJ) key = K128{ord_f64(J), ~((a.prefix0 + a.part_prefix[b]) * (uint64_t)S + u)};
            }
            list128_offer_many(slot, key, lane, k, thr);
            if (nz128(thr)) {
                const double kj = unord_f64(thr.hi);
                thrJ = kj > thrJ ? kj : thrJ;
            }
        }
    }
    tv = wave_sum64(tv);
    tf = wave_sum64(tf);
    __syncthreads();
    if (lane == 0) {
        s_cnt[wv] = tv;
        s_cnt[kMitmWaves + wv] = tf;
    }
    K128 *kl = reinterpret_cast<K128 *>(l.lst);   // [waves][64]
    kl[wv * 64 + lane] = key_if(lane < k, slot);
    if (few && nhit <= 64) {
        __syncthreads();   // wave 0 holds every key, sorted
        slot = key_if(lane < k, slot);
    } else {
#pragma unroll
        for (int h = kMitmWaves / 2; h >= 1; h >>= 1) {
            __syncthreads();
            if (wv < h) {
                list128_merge_sorted(slot, kl[(wv + h) * 64 + lane], lane, k, thr);
                if (h > 1) kl[wv * 64 + lane] = slot;
            }
        }
    }
    if (wv == 0) {
        const int n_top = __popcll(__ballot(lane < k && nz128(slot)));
        unsigned long long c = 0;
        if (lane < 2)
            for (int w = 0; w < kMitmWaves; w++) c += s_cnt[lane * kMitmWaves + w];
        const unsigned long long nv = readlane64(c, 0), nf = readlane64(c, 1);
        const bool ok = lane < n_top;
        const unsigned long long ti = ok ? ~slot.lo : ~0ull;
        const double tj = ok ? unord_f64(slot.hi) : -INFINITY;
        DevResult *dst[2] = {a.res, a.res_host};
#pragma unroll
        for (int q = 0; q < 2; q++)
            if (DevResult *R = dst[q]) {
                R->top_idx[lane] = ti;
                R->top_J[lane] = tj;
                if (lane == 0) {
                    R->n_vram = nv;
                    R->n_feas_sure = nf;
                    R->n_top = n_top;
                    R->status = general ? 0u : kStatVerified;
                    R->fast_ticks = (unsigned long long)wall_clock64() - s_t0;
                }
            }
        if (lane == 0) *a.ticket = 0u;   // the next launch of the call
        if (a.res_host) {
            __threadfence_system();
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) *reinterpret_cast<volatile unsigned long long *>(&a.res_host->done_seq) = a.seq;
        }
    }
}

hipError_t launch_mitm(const MitmArgs &a, int grid, hipStream_t s)
{
    const size_t lds = mitm_lds_bytes(a.sumK, a.spad) + a.raw_bytes;
    // one workgroup, more than 32 best: lists of 128
    const bool big = grid == 1 && a.top_k > 32;
    auto pick = [&](auto f1, auto f2, auto f3, auto f4) { return a.eq3 ? (big ? f4 : f3) : (big ? f2 : f1); };
    auto fn = a.n_models <= 8 ? pick(mitm_kernel<8, 1, false>, mitm_kernel<8, 2, false>, mitm_kernel<8, 1, true>,
                                     mitm_kernel<8, 2, true>)
                              : pick(mitm_kernel<16, 1, false>, mitm_kernel<16, 2, false>, mitm_kernel<16, 1, true>,
                                     mitm_kernel<16, 2, true>);
    const hipError_t e = ensure_dyn_lds((const void *)fn, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kMitmThreads), lds, s, a);
    return hipGetLastError();
}

}  // namespace mfi
