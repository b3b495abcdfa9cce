// Fast path of the exhaustive surrogate search (fp32 MFMA), gfx950.
//
// One wave evaluates tiles of 32 joint indices, one per step in a small range
// (small_kernel), two in a large one (scan_kernel):
//   decode       mixed-radix digits (Eq. 1): by reciprocals from the offset, or,
//                in a small range with a dump, by odometer
//   aggregate    fp32 sum in model order of every model's option row
//                (the aggregate field of Section III-B), from LDS; slot 0 is
//                the VRAM sum, compared with the cap (Eq. 4)
//   surrogate    per model (Eq. 6): layer 1 = per-option precompute
//                P[row] = b1 + W1_local x (the option's own columns, done once
//                per option) as the accumulator init, plus W1_agg a on MFMA;
//                layer 2 on binary16 matrix cores at fp32-level accuracy: the
//                layer-1 accumulator registers are split into two binary16
//                pieces each (x1 = x truncated, x2 = the rest truncated), W2
//                into two precomputed pieces (w1 + w2), and the three leading
//                cross products x1 w1 + x1 w2 + x2 w1 run on
//                v_mfma_f32_32x32x16_f16 with fp32 accumulation (the dropped
//                term and the pieces' truncation are below 2^-20 relative, and
//                go into the a-priori bound); power-of-two scales folded into
//                the layer-1, b2 and W3 tables keep every piece inside the
//                binary16 range without changing any fp32 rounding; the
//                accumulator row order is absorbed into W2's A-operand layout;
//                layer 3 (2 outputs) on VALU with one cross-half add
//   mask/score   latency bound per model decided with an a-priori error bound:
//                sure pass, sure fail, or "left to canonical re-evaluation";
//                J = fma chain over models of omega_i thr_i
//   top-K'       sure-feasible keys (J, lowest index) kept in a sorted
//                register list per wave (lane l holds slot l), merged per
//                workgroup at the end
// Everything the kernel reads per configuration lives in LDS; the only HBM
// traffic is the image load in the prologue and O(K') results.
#pragma once

#include "mf_canon.h"

namespace mfi {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f16x8 as_f16x8(uint4 v)
{
    f16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

__device__ __forceinline__ uint32_t pk_f16_rtz(float a, float b)
{
    const auto h = __builtin_amdgcn_cvt_pkrtz(a, b);
    uint32_t u;
    __builtin_memcpy(&u, &h, 4);
    return u;
}

// x - x1 for the binary16 value x1 in the low (HI = false) or high half of
// the packed register p: one mixed-precision fma, exact (x1 is x truncated).
// Its result feeds only vector instructions the compiler emits itself (the
// packing below), so the compiler's own wait states cover every matrix-core
// read of the pieces.
template <bool HI>
__device__ __forceinline__ float f16_residual(uint32_t p, float x)
{
    float r;
    if constexpr (HI)
        asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    else
        asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
    return r;
}

// The pair (a, b) as binary16 pieces: *x1 = (a, b) rounded toward zero,
// return (a - a1, b - b1) rounded to nearest.  |x - x1 - x2| <= 2^-21 |x| +
// 2^-24 (binary16 subnormals are kept, by the conversions under the kernel's
// denormal mode and by the matrix cores).
__device__ __forceinline__ uint32_t split_f16_pair(float a, float b, uint32_t *x1)
{
    const uint32_t h = pk_f16_rtz(a, b);
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const f16x2 l = {(_Float16)f16_residual<false>(h, a), (_Float16)f16_residual<true>(h, b)};
    uint32_t u;
    __builtin_memcpy(&u, &l, 4);
    *x1 = h;
    return u;
}

// Eight fp32 values v[r0 .. r0 + 7] as two binary16 B operands (x1, x2).
__device__ __forceinline__ void split_f16x8(const floatx16 &v, int r0, f16x8 &hi, f16x8 &lo)
{
    uint32_t h[4], l[4];
#pragma unroll
    for (int t = 0; t < 4; t++) l[t] = split_f16_pair(v[r0 + 2 * t], v[r0 + 2 * t + 1], &h[t]);
    __builtin_memcpy(&hi, h, 16);
    __builtin_memcpy(&lo, l, 16);
}


// One model's surrogate (Eq. 6) on canonical semantics, by one wave with no
// barriers: one configuration (lane u computes hidden unit u, H <= 64), or,
// when PAIR (H <= 32 and at most 32 inputs), two configurations of the same
// model, one per 32-lane half.  Each unit's chain takes its inputs in
// ascending order.  The inputs of a layer (z, then h1, then h2: input k of a
// half in its lane k) pass through the wave's 64 doubles of LDS, xb, and are
// read back at one address per half (a broadcast read), so that the VALU
// issues the chains themselves.  cb is the model's canonical fp32 block
// (W1T[nin][H], b1[H], W2T[H][H], b2[H], W3[2][H], b3[2]; LDS or global):
// lane u reads column u of a transposed matrix, consecutive lanes consecutive
// words.  fp32 weights are exact in fp64.  A wave's LDS accesses complete in
// program order; wave barriers keep the compiler from moving them across a
// layer's store.  Outputs: (lat, thr) of the configuration of half h in lanes
// 32 h and 32 h + 1 of y.
template <int H, bool PAIR>
__device__ inline double canon_forward_block(const float *cb, int nin, double z, int lane, bool sigmoid, double *xb)
{
    static_assert(!PAIR || H <= 32, "two configurations per wave need H <= 32");
    const int uu = PAIR ? (lane & 31) : lane;
    const int u = uu < H ? uu : H - 1;   // lanes past H repeat the last unit and are ignored
    const int hb = PAIR ? (lane & 32) : 0;
    const float *c1 = cb, *w2t = cb + nin * H + H, *b2 = w2t + H * H, *w3 = b2 + H, *b3 = w3 + 2 * H;
    xb[lane] = z;
    __builtin_amdgcn_wave_barrier();
    double c = (double)c1[nin * H + u];
    int k = 0;
    for (; k + 8 <= nin; k += 8) {
        float wv[8];
        double zk[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            wv[j] = c1[(k + j) * H + u];
            zk[j] = xb[hb + k + j];
        }
#pragma unroll
        for (int j = 0; j < 8; j++) c = fma((double)wv[j], zk[j], c);
    }
    for (; k < nin; k++) c = fma((double)c1[k * H + u], xb[hb + k], c);
    __builtin_amdgcn_wave_barrier();
    xb[lane] = c > 0.0 ? c : 0.0;   // h1
    __builtin_amdgcn_wave_barrier();
    c = (double)b2[u];
#pragma unroll
    for (int u0 = 0; u0 < H; u0 += 8) {
        float wv[8];
        double2 hk[4];
#pragma unroll
        for (int j = 0; j < 8; j++) wv[j] = w2t[(u0 + j) * H + u];
#pragma unroll
        for (int j = 0; j < 4; j++) hk[j] = *reinterpret_cast<const double2 *>(xb + hb + u0 + 2 * j);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            c = fma((double)wv[2 * j], hk[j].x, c);
            c = fma((double)wv[2 * j + 1], hk[j].y, c);
        }
    }
    __builtin_amdgcn_wave_barrier();
    xb[lane] = c > 0.0 ? c : 0.0;   // h2
    __builtin_amdgcn_wave_barrier();
    // layer 3: lanes 32 h + o, W3[o][v] contiguous in v
    const int o = lane & 1;
    c = (double)b3[o];
#pragma unroll
    for (int v0 = 0; v0 < H; v0 += 8) {
        float wv[8];
        double2 hk[4];
#pragma unroll
        for (int j = 0; j < 8; j++) wv[j] = w3[o * H + v0 + j];
#pragma unroll
        for (int j = 0; j < 4; j++) hk[j] = *reinterpret_cast<const double2 *>(xb + hb + v0 + 2 * j);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            c = fma((double)wv[2 * j], hk[j].x, c);
            c = fma((double)wv[2 * j + 1], hk[j].y, c);
        }
    }
    return sigmoid ? canon_sigmoid(c) : c;
}

// Small ranges, after the scan: the workgroup evaluates canonically (the
// defining semantics) its first eval_top list entries and the configurations
// of its certification segment, one wave per (entry, model), then each
// entry's constraints and J in model order (Section II, Eq. 3 and 4).  The
// image stays in LDS; the tail's buffers follow the workgroup lists.
// listkey: wave 0 holds the workgroup's sorted list, slot lane.
template <int H, int WAVES, bool OBJ, bool SIG>
__device__ inline void small_certify(const FastArgs &args, const FastConst &fc, float *smem, float *par,
                                     unsigned long long listkey, int kp, unsigned int n_offered, int lane, int wv,
                                     unsigned long long t_start)
{
    const FastLayout &Ly = args.lay;
    const int N = fc.n_models, L = args.n_local, A = Ly.A, nin = L + A, T = args.eval_top;
    const uint64_t g = blockIdx.x;
    const int *pK = reinterpret_cast<const int *>(par + 112), *pOff = reinterpret_cast<const int *>(par + 48);
    const int *pPrev = reinterpret_cast<const int *>(par + 80);
    unsigned long long *ekey = reinterpret_cast<unsigned long long *>(par + kFastPar) +
                               (args.lst_off == 0 ? 0 : WAVES * kp);   // [64]
    unsigned int *estat = reinterpret_cast<unsigned int *>(ekey + 64);                               // status, rest
    double *eout = reinterpret_cast<double *>(ekey + 66);                                            // [chunk][N][2]
    int *erow = reinterpret_cast<int *>(eout + (size_t)kCertChunk * N * 2);                          // [chunk][kMaxN]
    static_assert(WAVES <= kSearchWavesWide, "one 64-double forward buffer per wave");
    double *xb = reinterpret_cast<double *>(erow + kCertChunk * kMaxN) + wv * 64;
    // the chunk's canonical keys (J, joint index; 0 when infeasible)
    K128 *eck = reinterpret_cast<K128 *>(reinterpret_cast<double *>(erow + kCertChunk * kMaxN) + kSearchWavesWide * 64);
    if (wv == 0) {
        ekey[lane] = lane < T ? listkey : 0ull;
        // a bound on the upper bound U of every sure-feasible configuration
        // of the workgroup left unevaluated: list entry T when the list goes
        // past T, its last entry (itself evaluated) when T covers the whole
        // list; 0 when the list ends before (nothing left)
        const unsigned long long rest = readlane64(listkey, T < kp ? T : kp - 1);
        if (lane == 0) {
            estat[0] = 0;
            estat[1] = (uint32_t)(rest >> 32);
            estat[2] = 0;   // segment entries found feasible
        }
    }
    __syncthreads();
    // wave 0: the workgroup's best wg_k canonical keys so far
    K128 tslot = {0ull, 0ull}, tthr = {0ull, 0ull};
    const int n_list = __popcll(__ballot(lane < T && ekey[lane] != 0ull));
    const int n_seg = (int)(n_offered < args.seg_cap ? n_offered : args.seg_cap);
    const int n_ent = n_list + n_seg;
    const int *pCols = reinterpret_cast<const int *>(par + 144);
    const float *feat = Ly.off_feat >= 0 ? smem + Ly.off_feat : args.features;
    const bool pair = H <= 32 && nin <= 32;
    for (int c0 = 0; c0 < n_ent; c0 += kCertChunk) {
        const int nc = n_ent - c0 < kCertChunk ? n_ent - c0 : kCertChunk;
        // each entry's option rows (model order)
        for (int t = threadIdx.x; t < nc; t += WAVES * 64) {
            const int e = c0 + t;
            uint64_t x = args.lo + (e < n_list ? 0xFFFFFFFFu - (uint32_t)(ekey[e] & 0xFFFFFFFFull)
                                               : (uint32_t)args.seg[g * args.seg_cap + (e - n_list)]);
            for (int j = N - 1; j >= 0; j--) {
                const uint64_t kj = (uint64_t)pK[j];
                erow[t * kMaxN + j] = pOff[j] + (int)(x % kj);
                x /= kj;
            }
        }
        __syncthreads();
        // items (entry group, model): one entry per wave, or two (one per
        // half) when the model fits a half
        const int per = pair ? 2 : 1;
        const int n_grp = (nc + per - 1) / per;
        for (int q = wv; q < n_grp * N; q += WAVES) {
            const int p = q / N, i = q % N;
            const int half = pair ? (lane >> 5) : 0, kl = pair ? (lane & 31) : lane;
            const int t_raw = p * per + half;
            const int t = t_raw < nc ? t_raw : nc - 1;   // a spare half repeats the last entry
            const int *rows = erow + t * kMaxN;
            double z = 0.0;
            if (kl < L) {
                z = (double)feat[rows[i] * L + kl];
            } else if (kl < nin) {
                const int col = pCols[kl - L];
                int rj[kMaxN];
#pragma unroll
                for (int j = 0; j < kMaxN; j++) rj[j] = j < N ? rows[j] : 0;
                float sa = 0.f;
#pragma unroll
                for (int j = 0; j < kMaxN; j++)
                    if (j < N) sa = sa + feat[rj[j] * L + col];
                z = (double)sa;
            }
            const float *cb = Ly.off_c1 >= 0 ? smem + Ly.off_c1 + i * Ly.c1_stride
                                             : args.canon + (int64_t)i * args.wstride;
            double y;
            if constexpr (H <= 32) {
                y = pair ? canon_forward_block<H, true>(cb, nin, z, lane, SIG, xb)
                         : canon_forward_block<H, false>(cb, nin, z, lane, SIG, xb);
            } else {
                y = canon_forward_block<H, false>(cb, nin, z, lane, SIG, xb);
            }
            const double lat0 = readlane_f64(y, 0), thr0 = readlane_f64(y, 1);
            const double lat1 = readlane_f64(y, 32), thr1 = readlane_f64(y, 33);
            if (lane == 0) {
                const int tq = p * per;
                eout[2 * (tq * N + i)] = lat0;
                eout[2 * (tq * N + i) + 1] = thr0;
                if (pair && tq + 1 < nc) {
                    eout[2 * ((tq + 1) * N + i)] = lat1;
                    eout[2 * ((tq + 1) * N + i) + 1] = thr1;
                }
            }
        }
        __syncthreads();
        for (int t = threadIdx.x; t < nc; t += WAVES * 64) {
            const int e = c0 + t;
            const uint32_t off = e < n_list ? 0xFFFFFFFFu - (uint32_t)(ekey[e] & 0xFFFFFFFFull)
                                            : (uint32_t)args.seg[g * args.seg_cap + (e - n_list)];
            const int vcol = pCols[args.vram_slot];
            float va = 0.f;
            for (int j = 0; j < N; j++) va = va + feat[erow[t * kMaxN + j] * L + vcol];
            const bool vram_ok = (double)va <= (double)fc.vram_cap;
            bool sla_ok = true;
            double J = 0.0;
            for (int i = 0; i < N; i++) {
                const double lat = eout[2 * (t * N + i)], thr = eout[2 * (t * N + i) + 1];
                if (!(lat <= (double)par[128 + i])) sla_ok = false;
                if constexpr (OBJ) {
                    double qv, P, pen;
                    bool do_P, do_pen;
                    if (!canon_eq3(args.obj, erow[t * kMaxN + i], thr, par[64 + i], pPrev[i], qv, P, do_P, pen,
                                   do_pen))
                        sla_ok = false;
                    J = fma((double)par[32 + i], qv, J);
                    if (do_P) J = J - P;
                    if (do_pen) J = J - pen;
                } else {
                    J = fma((double)par[32 + i], thr, J);
                }
            }
            const bool feas = vram_ok && sla_ok;
            eck[t] = feas ? K128{ord_f64(J), ~(args.lo + (uint64_t)off)} : K128{0ull, 0ull};
            if (e < n_list) {
                // a sure-feasible fast decision must be canonically feasible,
                // and the key's U must bound the canonical J
                const double U = (double)unord_f32((uint32_t)(ekey[e] >> 32));
                if (!feas || !(U - J >= 0.0)) atomicOr(&estat[0], kStatSelfCheck);
            } else {
                if (feas) atomicAdd(&estat[2], 1u);
                if (args.mask)
                    args.mask[off] = (uint8_t)((vram_ok ? 1u : 0u) | (sla_ok ? 2u : 0u) | (feas ? 4u : 0u) | 8u);
            }
        }
        __syncthreads();
        // wave 0 takes the chunk's keys (kCertChunk = 64: one per lane); the
        // next chunk writes eck only after two more barriers
        static_assert(kCertChunk == 64, "one key per lane");
        if (wv == 0) list128_offer_many(tslot, lane < nc ? eck[lane] : K128{0ull, 0ull}, lane, args.wg_k, tthr);
    }
    if (wv == 0 && lane < args.wg_k) args.wg_top[g * (uint64_t)args.wg_k + lane] = tslot;
    if (threadIdx.x == 0) {
        unsigned long long *r = args.wg_rec + 8 * g;
        r[0] = n_offered;
        r[1] = t_start;
        r[2] = (unsigned long long)wall_clock64();
        r[3] = ((unsigned long long)estat[0] << 32) | estat[1];
        r[4] = estat[2];
    }
}

// Per-model parameters of a search after the image in LDS:
// [0,16) sla_lo  [16,32) sla_hi  [32,48) omega  [48,64) first option row per model (int)
// [64,80) floor tau  [80,96) previous variant (int)  [96,112) throughput bound
// [112,128) option count per model (int)  [128,144) latency bound  [144,160) aggregate column (int)
// OBJ: score with the full utility of Eq. 3 (otherwise the linear objective).
// SIG: the surrogates' outputs pass a sigmoid; the latency decision then
// compares the pre-activation with logit thresholds.
template <bool OBJ, bool SIG>
__device__ __forceinline__ void fast_params(const FastArgs &args, const FastConst &fc, float *par)
{
    const int N = fc.n_models;
    int *par_off = reinterpret_cast<int *>(par + 48);
    int *par_prev = reinterpret_cast<int *>(par + 80);
#pragma unroll
    for (int i = 0; i < kMaxN; i++) {
        // compile-time index into the argument block (keeps it out of scratch)
        if (threadIdx.x == (unsigned)i && i < N) {
            const double s = (double)args.sla[i], b = fc.bound_lat[i];
            if constexpr (SIG) {
                // canonical sigmoid within 2^-49 relative of the exact one:
                // pre-activation <= logit(s (1 - 2^-49)) gives a sure pass,
                // > logit(s (1 + 2^-48)) a sure miss (outputs lie in [0, 1])
                auto logit = [](double p) {
                    return p <= 0.0 ? -INFINITY : (p >= 1.0 ? INFINITY : log(p / (1.0 - p)));
                };
                const double lo = s >= 1.0 ? INFINITY : logit(s * (1.0 - 0x1p-49));
                const double hi = s >= 1.0 ? INFINITY : logit(s * (1.0 + 0x1p-48));
                par[i] = isinf(lo) ? (float)lo : (float)(lo - b - ((fabs(lo) + b) * 0x1p-22 + 1e-12));
                par[16 + i] = isinf(hi) ? (float)hi : (float)(hi + b + ((fabs(hi) + b) * 0x1p-22 + 1e-12));
            } else {
                const double slack = (fabs(s) + b) * 0x1p-22 + 1e-30;
                const bool inf = isinf(s);
                par[i] = inf ? (float)s : (float)(s - b - slack);       // lat <= this  => canonical lat <= sla
                par[16 + i] = inf ? (float)s : (float)(s + b + slack);  // lat >  this  => canonical lat >  sla
            }
            par[32 + i] = args.omega[i];
            par_off[i] = fc.opt_off[i];
            reinterpret_cast<int *>(par + 112)[i] = fc.K[i];
            par[128 + i] = args.sla[i];
            if constexpr (OBJ) {
                par[64 + i] = args.obj.tau[i];
                par_prev[i] = args.obj.prev[i];
                par[96 + i] = f32_up(fc.bound_thr[i]);
            }
        }
    }
}

// After the scan: the workgroup's counts and its merged candidate list (the
// merge kernel, or the finish of a small range, takes them on).
template <int WAVES>
__device__ __forceinline__ void write_wg_result(WaveList<1> &wl, uint32_t c_vram, uint32_t c_feas,
                                                unsigned long long *lst, const FastArgs &args, int kp, int lane, int wv)
{
    __shared__ unsigned long long s_cnt[2 * WAVES];
    const unsigned long long sv = wave_sum64(c_vram), sf = wave_sum64(c_feas);
    if (lane == 0) {
        s_cnt[wv] = sv;
        s_cnt[WAVES + wv] = sf;
    }
    if (args.lst_off == 0) __syncthreads();   // the lists overwrite the weights: every wave's scan is done
    if (lane < kp) lst[wv * kp + lane] = wl.s[0];
    wl_tree_merge<1, WAVES>(wl, lst, kp, wv, lane, kp);
    if (wv == 0) {
        if (lane < kp) args.wg_lists[(uint64_t)blockIdx.x * kp + lane] = wl.s[0];
        if (lane < 2) {
            unsigned long long t = 0;
            for (int w = 0; w < WAVES; w++) t += s_cnt[lane * WAVES + w];
            args.wg_counts[2 * (uint64_t)blockIdx.x + lane] = t;
        }
    }
}

// One 32-configuration tile's state in the scan of large ranges.
template <int MB>
struct ScanTile {
    uint32_t xh[MB * 8], xl[MB * 8];   // h1 as binary16 pairs: x1, x2 of registers 2 p, 2 p + 1
    floatx16 h1[MB];                   // layer-1 accumulators
    floatx16 acc;                      // layer 2, one output block
    float pl, pt;                      // layer-3 partial sums (lat, thr)
};

// The lane's 16 accumulator rows of a 32-row block, in accumulator order.
__device__ __forceinline__ floatx16 scan_load16(const float *p)
{
    floatx16 v;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const float4 f = *reinterpret_cast<const float4 *>(p + 8 * q);
        v[4 * q + 0] = f.x;
        v[4 * q + 1] = f.y;
        v[4 * q + 2] = f.z;
        v[4 * q + 3] = f.w;
    }
    return v;
}

// relu and binary16 pieces of the pair p of h1.
template <int MB>
__device__ __forceinline__ void scan_split(ScanTile<MB> &t, int p)
{
    const int mb = p >> 3, r = 2 * (p & 7);
    t.xl[p] = split_f16_pair(relu_f32(t.h1[mb][r]), relu_f32(t.h1[mb][r + 1]), &t.xh[p]);
}

__device__ __forceinline__ f16x8 pairs_f16x8(const uint32_t *v)
{
    f16x8 r;
    __builtin_memcpy(&r, v, 16);
    return r;
}

// Row r of the tile's layer-2 block into the layer-3 sums.
template <int MB>
__device__ __forceinline__ void scan_l3(ScanTile<MB> &t, const floatx16 &acc, int r, const float4 (&wl)[4],
                                        const float4 (&wt)[4])
{
    const float h = relu_f32(acc[r]);
    const float4 a = wl[r >> 2], b = wt[r >> 2];
    const int j = r & 3;
    t.pl = fmaf(j == 0 ? a.x : j == 1 ? a.y : j == 2 ? a.z : a.w, h, t.pl);
    t.pt = fmaf(j == 0 ? b.x : j == 1 ? b.y : j == 2 ? b.z : b.w, h, t.pt);
}

// Large ranges, the collect pass and lists: two tiles of 32 configurations per
// wave, 8 waves per workgroup (2 per SIMD, up to 256 registers).  What bounds
// it is the vector and matrix issue of a SIMD: per (tile, model) at H = 64 28
// matrix instructions (17.4 ns each, 490 ns) and about 215 vector ones (2 ns
// each beside the matrix cores, whatever their kind).  A tile's vector work
// (the split of h1, layer 3) lies between the other tile's matrix
// instructions, the operands both tiles share (W1, W2, b2, W3) are read from
// LDS once, and a lane decides one configuration: lane l of a step holds
// configuration l, tile l / 32 column l % 32 (decode, tail and lists once per
// 64 configurations).  One tile per wave and 4 waves per SIMD took 872 ns per
// (tile, model); two tiles in a fixed order of steps 790; steps taken from a
// counter and the decode without branches 720.
template <int MAXN, int A, int H, bool OBJ, bool SIG>
__global__ void __launch_bounds__(kSearchWaves * 64, 1)
scan_kernel(const FastArgs args, const FastConst fc, const int mode, const int kp)
{
    constexpr int MB = H / 32, WAVES = kSearchWaves, NW = (MAXN + 3) / 4;
    static_assert(A <= 8, "layer 1 takes at most 4 aggregate slots per lane half");
    constexpr bool L1ONE = A <= 4;     // two slots per lane half: one layer-1 instruction per block
    constexpr int AP = 8;              // aggregate row stride in LDS: [half][4]
    extern __shared__ float4 smem4[];
    float *smem = reinterpret_cast<float *>(smem4);
    const FastLayout &Ly = args.lay;
    const int N = fc.n_models;
    for (int t = threadIdx.x; t < args.image_f4; t += blockDim.x) smem4[t] = args.image[t];
    float *par = smem + Ly.total_floats;
    const int *par_off = reinterpret_cast<const int *>(par + 48), *par_prev = reinterpret_cast<const int *>(par + 80);
    unsigned long long *lst = reinterpret_cast<unsigned long long *>(smem + args.lst_off);
    fast_params<OBJ, SIG>(args, fc, par);
    // decode constants per model: 1 / K; K and the first index's digit (the
    // unused models decode to digit 0 and add a row of zeros)
    __shared__ double s_inv[MAXN];
    __shared__ uint2 s_kd[MAXN];
    __shared__ alignas(16) float s_zero[AP];
    __shared__ unsigned int s_next;   // the workgroup's steps handed out
#pragma unroll
    for (int i = 0; i < MAXN; i++)
        if (threadIdx.x == (unsigned)i) {   // a compile-time index keeps the argument block out of scratch
            s_inv[i] = i < N ? 1.0 / (double)fc.K[i] : 1.0;
            s_kd[i] = i < N ? uint2{(uint32_t)fc.K[i], args.digits[i]} : uint2{1u, 0u};
        }
    if (threadIdx.x < AP) s_zero[threadIdx.x] = 0.f;
    if (threadIdx.x == 0) s_next = WAVES;
    // global bound on |fast J - canonical J|: keys and certification entries
    // carry the upper bound U = J + eJ
    const double eJ = bound_eJ(fc, args.omega);
    if (mode == kModeSearch && blockIdx.x == 0 && threadIdx.x == 0) args.res->eJ = eJ;
    __syncthreads();

    const int lane = threadIdx.x & 63, half = lane >> 5;
    const float4 *cen_p = reinterpret_cast<const float4 *>(smem + Ly.off_c + 4 * half);
    const float sx_s[4] = {half ? fc.agg_scale[1][0] : fc.agg_scale[0][0], half ? fc.agg_scale[1][1] : fc.agg_scale[0][1],
                           half ? fc.agg_scale[1][2] : fc.agg_scale[0][2], half ? fc.agg_scale[1][3] : fc.agg_scale[0][3]};
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
    const uint64_t n = args.n;
    const uint64_t n_steps = (n + 63) >> 6;

    WaveList<1> wl;
    wl_init(wl);
    uint32_t c_vram = 0, c_feas = 0;
    WorkBuf wbuf;   // certification entries
    wbuf.e = 0ull;
    wbuf.j = 0.f;
    wbuf.n = 0;

    // The workgroup's steps are blockIdx.x, + gridDim.x, ...; its waves take
    // them one by one: of the two waves of a SIMD one is served first and runs
    // a third faster (12.4 us a step against 17 at six models).  With equal
    // shares the slower one set the time (29.1 ms against 26.6).
    uint64_t step = (uint64_t)wv * gridDim.x + blockIdx.x;
    while (step < n_steps) {
        unsigned int taken = 0;
        if (lane == 0) taken = atomicAdd(&s_next, 1u);
        const uint64_t off = step * 64u + (uint64_t)lane;
        const bool valid = off < n;
        // digits of the lane's configuration, 8 bits each, four to a word
        uint32_t dg[NW] = {};
        if (mode == kModeList) {
            uint64_t x = args.idx_list[valid ? off : n - 1];
#pragma unroll
            for (int j = MAXN - 1; j >= 0; j--)
                if (j < N) {
                    const uint64_t k = (uint64_t)fc.K[j];
                    dg[j / 4] |= (uint32_t)(x % k) << (8 * (j % 4));
                    x /= k;
                }
        } else {
            // offset (below 2^32) by reciprocals, the half added keeping the
            // product clear of the integers; then the first index's digits
            uint32_t x = valid ? (uint32_t)off : 0u, carry = 0;
#pragma unroll
            for (int j = MAXN - 1; j >= 0; j--) {
                const uint2 kd = s_kd[j];
                const uint32_t q = (uint32_t)(((double)x + 0.5) * s_inv[j]);
                const uint32_t t = x - q * kd.x + kd.y + carry;
                x = q;
                carry = t >= kd.x ? 1u : 0u;
                dg[j / 4] |= (t - (carry ? kd.x : 0u)) << (8 * (j % 4));
            }
        }
        // both tiles' digits in every lane: column l % 32 of tile t
        uint32_t dt[2][NW];
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const auto r = __builtin_amdgcn_permlane32_swap(dg[w], dg[w], false, false);
            dt[0][w] = r[0];
            dt[1][w] = r[1];
        }

        // aggregate field (model order, fp32).  Lane half h accumulates the
        // slots it feeds to layer 1 as B operand: internal slots 2s + h.
        // Slot 0 (half 0, s 0) is the VRAM sum.
        float ah[2][4] = {};
#pragma unroll
        for (int j = 0; j < MAXN; j++) {
            const float *g = (j < N ? smem + Ly.off_g + fc.opt_off[j] * AP : s_zero) + 4 * half;
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const float4 v = *reinterpret_cast<const float4 *>(g + ((dt[t][j / 4] >> (8 * (j % 4))) & 0xFFu) * AP);
                ah[t][0] += v.x;
                ah[t][1] += v.y;
                ah[t][2] += v.z;
                ah[t][3] += v.w;
            }
        }
        bool vram_ok;
        {
            // the lane's own sum: both lower halves hold slot 0
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(ah[0][0]), __float_as_uint(ah[1][0]), false,
                                                            false);
            vram_ok = __uint_as_float(r[0]) <= fc.vram_cap;
        }
        // layer 1's B operands, shared by every model of the step: the lane's
        // slots s (2s + half) as x = 2^ex (a - c) in binary16 pieces x1 + x2.
        // Four slots (A > 4): in k = 8 half + j, j and j + 4 both hold slot
        // j, bx1 its x1, bx2 its x2.  Two slots: one operand, j = 0, 1 and
        // 2, 3 hold x1 of slots 0, 1, j = 4, 5 and 6, 7 their x2.
        f16x8 bx1[2], bx2[2];
        {
            const float4 cen = cen_p[0];
#pragma unroll
            for (int t = 0; t < 2; t++) {
                uint32_t q[2], r[2];
                r[0] = split_f16_pair((ah[t][0] - cen.x) * sx_s[0], (ah[t][1] - cen.y) * sx_s[1], &q[0]);
                if constexpr (L1ONE) {
                    const uint32_t w1[4] = {q[0], q[0], r[0], r[0]};
                    __builtin_memcpy(&bx1[t], w1, 16);
                    bx2[t] = bx1[t];
                } else {
                    r[1] = split_f16_pair((ah[t][2] - cen.z) * sx_s[2], (ah[t][3] - cen.w) * sx_s[3], &q[1]);
                    const uint32_t w1[4] = {q[0], q[1], q[0], q[1]}, w2[4] = {r[0], r[1], r[0], r[1]};
                    __builtin_memcpy(&bx1[t], w1, 16);
                    __builtin_memcpy(&bx2[t], w2, 16);
                }
            }
        }

        float J = 0.f, EJ = 0.f, MJ = 0.f;   // fast J; under Eq. 3 its bound and magnitude
        bool anyfail = false;
        uint32_t umask = 0;   // models whose service decision is left to the canonical pass
        // Loads run ahead of their use, held in place by scheduling barriers: a
        // register pair of W2 operands is reloaded for the next output block
        // (or the next model's first) as soon as its last instruction is
        // issued, layer-3 weights likewise, the next model's layer-1 rows
        // beside the last block.  Left to itself the compiler sinks them to
        // their use, and the LDS latency showed at every block.
        ScanTile<MB> T[2];
        f16x8 a1[MB], wa[2 * MB], wb[2 * MB];
        floatx16 bias;
        const auto load_rows = [&](int i) {
            const int sh = 8 * (i & 3), base = par_off[i];
            uint32_t w0 = dt[0][0], w1 = dt[1][0];
#pragma unroll
            for (int w = 1; w < NW; w++)
                if (i >= 4 * w) {
                    w0 = dt[0][w];
                    w1 = dt[1][w];
                }
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const uint32_t row = (uint32_t)base + (((t ? w1 : w0) >> sh) & 0xFFu);
                const float *prow = smem + Ly.off_p + row * (uint32_t)Ly.PST + 4 * half;
#pragma unroll
                for (int mb = 0; mb < MB; mb++)
                    T[t].h1[mb] = scan_load16(prow + 32 * mb);
            }
            // W1_agg 2^(e1 - ex) in binary16 pieces w1 + w2, row 32 mb + l%32
            // of lane l.  Four slots: 16 bytes per lane and block, w1 (j < 4)
            // then w2 (j >= 4) of the slots 2 (j % 4) + l/32; one A operand
            // for both instructions, w1 x1 + w2 x1, then w1 x2 + w2 x2.  Two
            // slots: 8 bytes, w1 then w2 of slots l/32 and 2 + l/32, read
            // twice into one operand, all four products in one instruction.
#pragma unroll
            for (int mb = 0; mb < MB; mb++) {
                if constexpr (L1ONE) {
                    const uint2 p = (reinterpret_cast<const uint2 *>(smem + Ly.off_w1a + i * (MB * 64 * 2)) + lane)[mb * 64];
                    a1[mb] = as_f16x8(uint4{p.x, p.y, p.x, p.y});
                } else {
                    a1[mb] = as_f16x8((reinterpret_cast<const uint4 *>(smem + Ly.off_w1a + i * (MB * 64 * 4)) + lane)[mb * 64]);
                }
            }
        };
        load_rows(0);
        {
            const uint4 *w2p = reinterpret_cast<const uint4 *>(smem + Ly.off_w2) + lane;
#pragma unroll
            for (int kb = 0; kb < 2 * MB; kb++) {
                wa[kb] = as_f16x8(w2p[(kb * 2 + 0) * 64]);
                wb[kb] = as_f16x8(w2p[(kb * 2 + 1) * 64]);
            }
            bias = scan_load16(smem + Ly.off_b2 + 4 * half);
        }
        for (int i = 0; i < N; i++) {
            const int nx = i + 1 < N ? i + 1 : i;
            const uint4 *w2p = reinterpret_cast<const uint4 *>(smem + Ly.off_w2 + i * (H * H)) + lane;
            const uint4 *w2n = reinterpret_cast<const uint4 *>(smem + Ly.off_w2 + nx * (H * H)) + lane;
            const float *w3 = smem + Ly.off_w3 + i * (2 * H) + 4 * half;
            // the tail's values
            const float2 b3 = *reinterpret_cast<const float2 *>(smem + Ly.off_b3 + 4 * i);
            const float p_lo = par[i], p_hi = par[16 + i], p_om = par[32 + i];
            float4 vr0, vr1;
            if constexpr (OBJ) {
                uint32_t w = dg[0];
#pragma unroll
                for (int q = 1; q < NW; q++) w = i >= 4 * q ? dg[q] : w;
                const uint32_t row = (uint32_t)par_off[i] + ((w >> (8 * (i & 3))) & 0xFFu);
                vr0 = args.obj.vrow[2 * row];
                vr1 = args.obj.vrow[2 * row + 1];
            }
            // ---- layer 1: P[row] + W1_agg a
#pragma unroll
            for (int t = 0; t < 2; t++) {
                T[t].pl = 0.f;
                T[t].pt = 0.f;
#pragma unroll
                for (int mb = 0; mb < MB; mb++) {
                    T[t].h1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[mb], bx1[t], T[t].h1[mb], 0, 0, 0);
                    if constexpr (!L1ONE)
                        T[t].h1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[mb], bx2[t], T[t].h1[mb], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // layer-3 weights of the block whose sums are due
            float4 w3l[4], w3t[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                w3l[q] = *reinterpret_cast<const float4 *>(w3 + (0 * MB * 4 + q) * 8);
                w3t[q] = *reinterpret_cast<const float4 *>(w3 + (1 * MB * 4 + q) * 8);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < 8 * MB; p++) scan_split(T[0], p);
            __builtin_amdgcn_sched_barrier(0);
            // ---- layer 2: b2 + W2 h1, one output block at a time.  h1 (the
            // relu'd layer-1 accumulators) as binary16 pieces, x1 = x
            // truncated, x2 = (x - x1) rounded to nearest.  W2 as two binary16
            // pieces (w1 + w2 ~ 2^e2 W2) in the A-operand order of
            // v_mfma_f32_32x32x16_f16: per (mb2, mb1, kh) 1 KB of w1 then 1 KB
            // of w2, lane l's 16 bytes holding K-block elements 0..7.  The
            // small cross products first, while the accumulator holds only the
            // bias (each matrix instruction's error grows with the accumulator
            // it adds to), then the leading ones.
            constexpr int NM = 6 * MB;          // matrix instructions per tile and block
#pragma unroll
            for (int mb2 = 0; mb2 < MB; mb2++) {
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    floatx16 acc = bias;
                    const floatx16 prev = T[1 - t].acc;
#pragma unroll
                    for (int m = 0; m < NM; m++) {
                        const int kb = m < 4 * MB ? m >> 1 : m - 4 * MB;
                        const bool lo2 = m < 4 * MB && (m & 1);         // w1 x2
                        const bool hi2 = m < 4 * MB && !(m & 1);        // w2 x1
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(hi2 ? wb[kb] : wa[kb],
                                                                     pairs_f16x8((lo2 ? T[t].xl : T[t].xh) + 4 * kb),
                                                                     acc, 0, 0, 0);
                        // the other tile's vector work beside it
                        if (t == 0 && mb2 == 0) {
#pragma unroll
                            for (int p = m * 8 * MB / NM; p < (m + 1) * 8 * MB / NM; p++) scan_split(T[1], p);
                        } else {
#pragma unroll
                            for (int r = m * 16 / NM; r < (m + 1) * 16 / NM; r++) {
                                scan_l3(T[1 - t], prev, r, w3l, w3t);
                                if (t == 0 && (r & 3) == 3) {   // tile 1 was the last to need these
                                    const int q = r >> 2;
                                    w3l[q] = *reinterpret_cast<const float4 *>(w3 + ((0 * MB + mb2) * 4 + q) * 8);
                                    w3t[q] = *reinterpret_cast<const float4 *>(w3 + ((1 * MB + mb2) * 4 + q) * 8);
                                }
                            }
                        }
                        if (t == 1) {
                            const bool last = mb2 + 1 == MB;
                            const uint4 *src = last ? w2n : w2p + (mb2 + 1) * MB * 4 * 64;
                            if (hi2) wb[kb] = as_f16x8(src[(kb * 2 + 1) * 64]);
                            if (m >= 4 * MB) wa[kb] = as_f16x8(src[(kb * 2 + 0) * 64]);
                            if (m == 1)
                                bias = scan_load16(last ? smem + Ly.off_b2 + nx * H + 4 * half
                                                        : smem + Ly.off_b2 + i * H + 4 * half + 32 * (mb2 + 1));
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    T[t].acc = acc;
                }
            }
            load_rows(nx);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 16; r++) scan_l3(T[1], T[1].acc, r, w3l, w3t);
            // each half's sums join: tile 0's in lanes 0..31, tile 1's above
            const auto sl = __builtin_amdgcn_permlane32_swap(__float_as_uint(T[0].pl), __float_as_uint(T[1].pl), false, false);
            const auto st = __builtin_amdgcn_permlane32_swap(__float_as_uint(T[0].pt), __float_as_uint(T[1].pt), false, false);
            const float lat = (__uint_as_float(sl[0]) + __uint_as_float(sl[1])) + b3.x;
            const float pre = (__uint_as_float(st[0]) + __uint_as_float(st[1])) + b3.y;
            const float thr = SIG ? sigmoid_f32(pre) : pre;
            bool pass = lat <= p_lo, fail = lat > p_hi;
            if constexpr (OBJ) {
                const Eq3Term t = eq3_term(vr0, vr1, thr, par[96 + i], p_om, par[64 + i], par_prev[i], args.obj.alpha,
                                           args.obj.beta, args.obj.delta);
                fail = fail || t.fail;
                pass = pass && t.pass;
                J += t.c;
                EJ += t.e;
                MJ += t.mag;
            } else {
                J = fmaf(p_om, thr, J);
            }
            anyfail |= fail;
            umask |= (pass || fail) ? 0u : (1u << i);
            if (args.pred && valid) {
                args.pred[(off * (uint64_t)N + (uint64_t)i) * 2u + 0u] = SIG ? sigmoid_f32(lat) : lat;
                args.pred[(off * (uint64_t)N + (uint64_t)i) * 2u + 1u] = thr;
            }
        }

        if (mode != kModeList) {
            const bool anyunc = umask != 0u;
            const bool sla_sure = !anyfail && !anyunc;
            const bool feas_sure = valid && vram_ok && sla_sure;
            // a latency decision the bound cannot settle: re-evaluated
            // canonically when it can change the count (VRAM ok) or, in dump
            // mode, the mask
            const bool unc = valid && !anyfail && anyunc && (vram_ok || args.mask != nullptr);
            // Eq. 3: the sum of per-model bounds, plus the fp32 sum over models
            // (N u relative to the magnitudes)
            const float U = OBJ ? f32_up((double)J + (double)EJ * (1.0 + 0x1p-10) + (double)MJ * N * 0x1p-22 + 1e-30)
                                : f32_up((double)J + eJ);
            if (mode == kModeSearch) {
                c_vram += (valid && vram_ok) ? 1u : 0u;
                c_feas += feas_sure ? 1u : 0u;
                const unsigned long long went = (unsigned long long)(uint32_t)off | ((unsigned long long)umask << 32);
                wb_append(wbuf, unc, went, U, lane, &args.res->n_work, args.work, args.work_J, args.work_cap);
                const unsigned long long key = feas_sure
                    ? (((unsigned long long)ord_f32(U) << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)off))
                    : 0ull;
                wl_offer_many(wl, key, lane, kp);
                if (args.mask && valid)
                    args.mask[off] = (uint8_t)((vram_ok ? 1u : 0u) | (sla_sure ? 2u : 0u) |
                                               (feas_sure ? 4u : 0u) | (unc ? 8u : 0u));
            } else {
                list_append(feas_sure && (double)U >= args.theta, (uint32_t)off, lane, &args.res->n_collect,
                            args.collect, args.collect_cap);
            }
        }
        step = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)taken) * gridDim.x + blockIdx.x;
    }

    if (mode == kModeSearch) {
        wb_flush(wbuf, lane, &args.res->n_work, args.work, args.work_J, args.work_cap);
        write_wg_result<WAVES>(wl, c_vram, c_feas, lst, args, kp, lane, wv);
    }
}

// Where round h of a dealt range begins among n workgroups: a hash of h, so
// that configurations a whole number of rounds apart (the options of a model,
// where the counts are powers of two) do not meet in one workgroup.
__device__ __forceinline__ uint32_t deal_rotation(uint32_t h, uint32_t n)
{
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return __umulhi(h, n);
}

// Small ranges: a tile of 32 configurations per wave (latency counts here, so
// the range goes to as many waves as there are tiles), then the certification.
// Also short lists (predictions only), their tiles dealt over the workgroups
// so that few waves share a SIMD.
template <int MAXN, int A, int H, int WAVES, bool OBJ, bool SIG>
__global__ void __launch_bounds__(WAVES * 64, 1)
small_kernel(const FastArgs args, const FastConst fc, const int kp)
{
    const uint32_t spread = args.spread;
    const uint64_t *list = args.idx_list;
    constexpr int MB = H / 32;         // 32-row blocks of a hidden layer
    static_assert(A <= 8, "layer 1 takes at most 4 aggregate slots per lane half");
    constexpr bool L1ONE = A <= 4;     // two slots per lane half: one layer-1 instruction per block
    constexpr int AP = 8;              // aggregate row stride in LDS: [half][4]
    extern __shared__ float4 smem4[];
    float *smem = reinterpret_cast<float *>(smem4);
    const FastLayout &Ly = args.lay;
    const int N = fc.n_models;
    __shared__ unsigned int s_nwork;   // small ranges: certification entries of the workgroup
    __shared__ double s_inv[MAXN];     // 1 / K (spread ranges)

    for (int t = threadIdx.x; t < args.image_f4; t += blockDim.x) smem4[t] = args.image[t];
    float *par = smem + Ly.total_floats;
    int *par_off = reinterpret_cast<int *>(par + 48);
    int *par_prev = reinterpret_cast<int *>(par + 80);
    unsigned long long *lst = reinterpret_cast<unsigned long long *>(smem + args.lst_off);
    fast_params<OBJ, SIG>(args, fc, par);
    {
        // (a compile-time index keeps the argument block out of scratch)
#pragma unroll
        for (int i = 0; i < MAXN; i++)
            if (threadIdx.x == (unsigned)i && i < N) s_inv[i] = 1.0 / (double)fc.K[i];
    }
    if (threadIdx.x < (unsigned)Ly.A)
        reinterpret_cast<int *>(par + 144)[threadIdx.x] = args.agg_cols[threadIdx.x];
    constexpr bool eq3 = OBJ;
    // global bound on |fast J - canonical J|: keys and certification entries
    // carry the upper bound U = J + eJ
    const double eJ = bound_eJ(fc, args.omega);
    // small ranges: certification entries counted per workgroup in LDS
    unsigned long long t_start = 0;
    if (threadIdx.x == 0) {
        s_nwork = 0;
        t_start = (unsigned long long)wall_clock64();
    }
    __syncthreads();

    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    // aggregate centre and power-of-two scale of the slots this lane feeds
    // to layer 1 (read per tile: registers are the kernel's limit)
    const float4 *cen_p = reinterpret_cast<const float4 *>(smem + Ly.off_c + 4 * half);
    const float sx_s[4] = {half ? fc.agg_scale[1][0] : fc.agg_scale[0][0], half ? fc.agg_scale[1][1] : fc.agg_scale[0][1],
                           half ? fc.agg_scale[1][2] : fc.agg_scale[0][2], half ? fc.agg_scale[1][3] : fc.agg_scale[0][3]};
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
    const int gw = blockIdx.x * WAVES + wv;
    const uint64_t n = args.n;
    const uint32_t n_tiles = ((spread ? spread : (uint32_t)n) + 31) >> 5;   // n <= 2^20

    uint32_t bd[MAXN] = {};
    if (spread == 0u && !list) {
        uint64_t x = args.lo + (uint64_t)gw * 32u;
#pragma unroll
        for (int j = MAXN - 1; j >= 0; j--) {
            if (j < N) {
                const uint64_t k = (uint64_t)fc.K[j];
                bd[j] = (uint32_t)(x % k);
                x /= k;
            } else {
                bd[j] = 0;
            }
        }
    }

    WaveList<1> wl;
    wl_init(wl);
    uint32_t c_vram = 0, c_feas = 0;

    const uint32_t tile_step = spread ? (uint32_t)WAVES : (uint32_t)args.total_waves;
    for (uint32_t tile = spread ? wv : list ? wv * gridDim.x + blockIdx.x : gw; tile < n_tiles; tile += tile_step) {
        uint32_t o = tile * 32u + (uint32_t)col;   // in order, or the round
        if (spread) {
            const uint32_t at = (uint32_t)blockIdx.x + deal_rotation(o, gridDim.x);
            o = o < spread ? o * gridDim.x + (at < gridDim.x ? at : at - gridDim.x) : 0xFFFFFFFFu;
        }
        const uint64_t off = o;
        const bool valid = off < n;
        uint32_t d[MAXN];
        if (spread) {
            // quotients by a reciprocal: the half added keeps the product
            // clear of the integers (exact below 2^32)
            uint32_t x = (uint32_t)(args.lo + (valid ? off : 0ull));
#pragma unroll
            for (int j = MAXN - 1; j >= 0; j--) {
                d[j] = 0;
                if (j < N) {
                    const uint32_t q = (uint32_t)(((double)x + 0.5) * s_inv[j]);
                    d[j] = x - q * (uint32_t)fc.K[j];
                    x = q;
                }
            }
        } else if (list) {
            uint64_t x = list[valid ? off : n - 1];
#pragma unroll
            for (int j = MAXN - 1; j >= 0; j--) {
                d[j] = 0;
                if (j < N) {
                    const uint64_t k = (uint64_t)fc.K[j];
                    d[j] = (uint32_t)(x % k);
                    x /= k;
                }
            }
        } else {
            uint32_t carry = (uint32_t)col;
#pragma unroll
            for (int j = MAXN - 1; j >= 0; j--) {
                if (j < N) {
                    const uint32_t t = bd[j] + carry;
                    const uint32_t q = fc.magic[j] ? __umulhi(t, fc.magic[j]) : t;
                    d[j] = t - q * (uint32_t)fc.K[j];
                    carry = q;
                } else {
                    d[j] = 0;
                }
            }
        }

        // aggregate field (model order, fp32).  Lane half h accumulates the
        // slots it feeds to layer 1 as B operand: internal slots 2s + h.
        // Slot 0 (half 0, s 0) is the VRAM sum.
        float ah[4] = {0.f, 0.f, 0.f, 0.f};
        uint64_t dig0 = 0, dig1 = 0;   // digits packed 8 bits each: models 0..7, 8..15
#pragma unroll
        for (int j = 0; j < MAXN; j++) {
            if (j < N) {
                if (j < 8) dig0 |= (uint64_t)d[j] << (8 * j);
                else dig1 |= (uint64_t)d[j] << (8 * (j - 8));
                const uint32_t row = (uint32_t)fc.opt_off[j] + d[j];
                const float4 v = *reinterpret_cast<const float4 *>(smem + Ly.off_g + row * AP + 4 * half);
                ah[0] += v.x;
                ah[1] += v.y;
                ah[2] += v.z;
                ah[3] += v.w;
            }
        }
        const bool vram_ok = ah[0] <= fc.vram_cap;
        // layer 1's B operands, shared by every model of the tile: the lane's
        // slots s (2s + half) as x = 2^ex (a - c) in binary16 pieces x1 + x2.
        // Four slots (A > 4): in k = 8 half + j, j and j + 4 both hold slot
        // j, bx1 its x1, bx2 its x2.  Two slots: one operand, j = 0, 1 and
        // 2, 3 hold x1 of slots 0, 1, j = 4, 5 and 6, 7 their x2.
        f16x8 bx1, bx2;
        {
            const float4 cen = cen_p[0];
            uint32_t q[2], r[2];
            r[0] = split_f16_pair((ah[0] - cen.x) * sx_s[0], (ah[1] - cen.y) * sx_s[1], &q[0]);
            if constexpr (L1ONE) {
                const uint32_t w1[4] = {q[0], q[0], r[0], r[0]};
                __builtin_memcpy(&bx1, w1, 16);
                bx2 = bx1;
            } else {
                r[1] = split_f16_pair((ah[2] - cen.z) * sx_s[2], (ah[3] - cen.w) * sx_s[3], &q[1]);
                const uint32_t w1[4] = {q[0], q[1], q[0], q[1]}, w2[4] = {r[0], r[1], r[0], r[1]};
                __builtin_memcpy(&bx1, w1, 16);
                __builtin_memcpy(&bx2, w2, 16);
            }
        }

        float J = 0.f, EJ = 0.f, MJ = 0.f;   // fast J; under Eq. 3 its bound and magnitude
        bool anyfail = false;
        uint32_t umask = 0;   // models whose service decision is left to the canonical pass
        for (int i = 0; i < N; i++) {
            const uint64_t sel = (uint64_t)0 - (uint64_t)(i >= 8);
            const uint64_t dw = dig0 ^ ((dig0 ^ dig1) & sel);
            const uint32_t row = (uint32_t)par_off[i] + (uint32_t)((dw >> (8 * (i & 7))) & 0xFFu);
            // ---- layer 1: P[row] + W1_agg a
            floatx16 acc1[MB];
            const float *prow = smem + Ly.off_p + row * (uint32_t)Ly.PST + 4 * half;
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const float4 v = *reinterpret_cast<const float4 *>(prow + 32 * mb + 8 * q);
                    acc1[mb][4 * q + 0] = v.x;
                    acc1[mb][4 * q + 1] = v.y;
                    acc1[mb][4 * q + 2] = v.z;
                    acc1[mb][4 * q + 3] = v.w;
                }
            // W1_agg 2^(e1 - ex) in binary16 pieces w1 + w2, row 32 mb + l%32
            // of lane l.  Four slots: 16 bytes per lane and block, w1 (j < 4)
            // then w2 (j >= 4) of the slots 2 (j % 4) + l/32; one A operand
            // for both instructions, w1 x1 + w2 x1, then w1 x2 + w2 x2.  Two
            // slots: 8 bytes, w1 then w2 of slots l/32 and 2 + l/32, read
            // twice into one operand, all four products in one instruction.
            if constexpr (L1ONE) {
                const uint2 *w1a = reinterpret_cast<const uint2 *>(smem + Ly.off_w1a + i * (MB * 64 * 2)) + lane;
#pragma unroll
                for (int mb = 0; mb < MB; mb++) {
                    const uint2 p = w1a[mb * 64];
                    const uint4 a = {p.x, p.y, p.x, p.y};
                    acc1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a), bx1, acc1[mb], 0, 0, 0);
                }
            } else {
                const uint4 *w1a = reinterpret_cast<const uint4 *>(smem + Ly.off_w1a + i * (MB * 64 * 4)) + lane;
#pragma unroll
                for (int mb = 0; mb < MB; mb++) {
                    const f16x8 a = as_f16x8(w1a[mb * 64]);
                    acc1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bx1, acc1[mb], 0, 0, 0);
                    acc1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bx2, acc1[mb], 0, 0, 0);
                }
            }
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc1[mb][r] = relu_f32(acc1[mb][r]);
            // ---- layer 2: b2 + W2 h1.  h1 (the relu'd layer-1 accumulators)
            // becomes binary16 pieces first, K-block by K-block (accumulator
            // registers 8 kh .. 8 kh + 7 of block mb1): x1 = x truncated, x2
            // = (x - x1) rounded to nearest, as many registers as h1 itself
            f16x8 xh[MB][2], xl[MB][2];
#pragma unroll
            for (int mb1 = 0; mb1 < MB; mb1++)
#pragma unroll
                for (int kh = 0; kh < 2; kh++) split_f16x8(acc1[mb1], 8 * kh, xh[mb1][kh], xl[mb1][kh]);
            // W2 as two binary16 pieces (w1 + w2 ~ 2^e2 W2) in the A-operand
            // order of v_mfma_f32_32x32x16_f16: per (mb2, mb1, kh) 1 KB of w1
            // then 1 KB of w2, lane l's 16 bytes holding K-block elements 0..7;
            // the products x1 w1 + x1 w2 + x2 w1 accumulate in fp32.  One
            // output block at a time: block mb2's relu and layer-3 rows (VALU)
            // are independent of block mb2 + 1's matrix instructions.
            const float *b2 = smem + Ly.off_b2 + i * H + 4 * half;
            const uint4 *w2p = reinterpret_cast<const uint4 *>(smem + Ly.off_w2 + i * (H * H)) + lane;
            const float *w3 = smem + Ly.off_w3 + i * (2 * H) + 4 * half;
            float pl = 0.f, pt = 0.f;
#pragma unroll
            for (int mb2 = 0; mb2 < MB; mb2++) {
                floatx16 acc2;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const float4 v = *reinterpret_cast<const float4 *>(b2 + 32 * mb2 + 8 * q);
                    acc2[4 * q + 0] = v.x;
                    acc2[4 * q + 1] = v.y;
                    acc2[4 * q + 2] = v.z;
                    acc2[4 * q + 3] = v.w;
                }
                // the small cross products first, while the accumulator holds
                // only the bias (each matrix instruction's error grows with
                // the accumulator it adds to), then the leading ones, K-block
                // by K-block
                f16x8 wa[MB][2];   // the w1 pieces, kept for the leading products
#pragma unroll
                for (int mb1 = 0; mb1 < MB; mb1++)
#pragma unroll
                    for (int kh = 0; kh < 2; kh++) {
                        wa[mb1][kh] = as_f16x8(w2p[(((mb2 * MB + mb1) * 2 + kh) * 2 + 0) * 64]);
                        const f16x8 wb = as_f16x8(w2p[(((mb2 * MB + mb1) * 2 + kh) * 2 + 1) * 64]);
                        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(wb, xh[mb1][kh], acc2, 0, 0, 0);
                        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(wa[mb1][kh], xl[mb1][kh], acc2, 0, 0, 0);
                    }
#pragma unroll
                for (int mb1 = 0; mb1 < MB; mb1++)
#pragma unroll
                    for (int kh = 0; kh < 2; kh++)
                        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(wa[mb1][kh], xh[mb1][kh], acc2, 0, 0, 0);
                // ---- layer 3 (2 outputs) on VALU, this block's rows
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const float4 wl = *reinterpret_cast<const float4 *>(w3 + ((0 * MB + mb2) * 4 + q) * 8);
                    const float4 wt = *reinterpret_cast<const float4 *>(w3 + ((1 * MB + mb2) * 4 + q) * 8);
                    const float h0 = relu_f32(acc2[4 * q + 0]), h1 = relu_f32(acc2[4 * q + 1]);
                    const float h2 = relu_f32(acc2[4 * q + 2]), h3 = relu_f32(acc2[4 * q + 3]);
                    pl = fmaf(wl.x, h0, pl); pt = fmaf(wt.x, h0, pt);
                    pl = fmaf(wl.y, h1, pl); pt = fmaf(wt.y, h1, pt);
                    pl = fmaf(wl.z, h2, pl); pt = fmaf(wt.z, h2, pt);
                    pl = fmaf(wl.w, h3, pl); pt = fmaf(wt.w, h3, pt);
                }
            }
            pl += __shfl_xor(pl, 32);
            pt += __shfl_xor(pt, 32);
            const float *b3 = smem + Ly.off_b3 + 4 * i;
            const float lat = pl + b3[0];
            const float thr = SIG ? sigmoid_f32(pt + b3[1]) : pt + b3[1];
            bool pass = lat <= par[i], fail = lat > par[16 + i];
            if constexpr (eq3) {
                const Eq3Term t = eq3_term(args.obj.vrow[2 * row], args.obj.vrow[2 * row + 1], thr, par[96 + i],
                                           par[32 + i], par[64 + i], par_prev[i], args.obj.alpha, args.obj.beta,
                                           args.obj.delta);
                fail = fail || t.fail;
                pass = pass && t.pass;
                J += t.c;
                EJ += t.e;
                MJ += t.mag;
            } else {
                J = fmaf(par[32 + i], thr, J);
            }
            anyfail |= fail;
            umask |= (pass || fail) ? 0u : (1u << i);
            if (args.pred && valid && half == 0) {
                args.pred[(off * (uint64_t)N + (uint64_t)i) * 2u + 0u] = SIG ? sigmoid_f32(lat) : lat;
                args.pred[(off * (uint64_t)N + (uint64_t)i) * 2u + 1u] = thr;
            }
        }

        if (list) continue;   // predictions only
        const bool mine = valid && half == 0;
        const bool anyunc = umask != 0u;
        const bool sla_sure = !anyfail && !anyunc;
        const bool feas_sure = mine && vram_ok && sla_sure;
        // a latency decision the bound cannot settle: re-evaluated
        // canonically when it can change the count (VRAM ok) or, in dump
        // mode, the mask
        const bool unc = mine && !anyfail && anyunc && (vram_ok || args.mask != nullptr);
        // Eq. 3: the sum of per-model bounds, plus the fp32 sum over models
        // (N u relative to the magnitudes)
        const float U = eq3 ? f32_up((double)J + (double)EJ * (1.0 + 0x1p-10) + (double)MJ * N * 0x1p-22 + 1e-30)
                            : f32_up((double)J + eJ);
        c_vram += (mine && vram_ok) ? 1u : 0u;
        c_feas += feas_sure ? 1u : 0u;
        const unsigned long long went = (unsigned long long)(uint32_t)off | ((unsigned long long)umask << 32);
        const unsigned long long m = __ballot(unc);
        if (m) {
            unsigned int base = 0;
            if (lane == 0) base = atomicAdd(&s_nwork, (unsigned int)__popcll(m));
            base = (unsigned int)__builtin_amdgcn_readfirstlane((int)base);
            const unsigned int slot = base + (unsigned int)__popcll(m & ((1ull << lane) - 1ull));
            if (unc && slot < args.seg_cap) {
                const uint64_t at = (uint64_t)blockIdx.x * args.seg_cap + slot;
                args.seg[at] = went;
                args.seg_J[at] = U;
            }
        }
        const unsigned long long key = feas_sure
            ? (((unsigned long long)ord_f32(U) << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)off))
            : 0ull;
        wl_offer_many(wl, key, lane, kp);
        if (args.mask && mine)
            args.mask[off] = (uint8_t)((vram_ok ? 1u : 0u) | (sla_sure ? 2u : 0u) | (feas_sure ? 4u : 0u) |
                                       (unc ? 8u : 0u));

        if (spread == 0u) {
            // advance the tile base by the grid stride, in mixed radix
            uint32_t carry = 0;
#pragma unroll
            for (int j = MAXN - 1; j >= 0; j--) {
                if (j < N) {
                    uint32_t t = bd[j] + args.digits[j] + carry;
                    carry = t >= (uint32_t)fc.K[j] ? 1u : 0u;
                    bd[j] = carry ? t - (uint32_t)fc.K[j] : t;
                }
            }
        }
    }

    if (list) return;
    write_wg_result<WAVES>(wl, c_vram, c_feas, lst, args, kp, lane, wv);
    // s_nwork is final: every wave's appends precede the tree merge's barriers
    small_certify<H, WAVES, OBJ, SIG>(args, fc, smem, par, wl.s[0], kp, s_nwork, lane, wv, t_start);
}

// The small kernel has 16 waves per workgroup where its registers and LDS allow
// (a.waves), the scan always 8.
template <int MAXN, int A, int H, bool SIG>
static hipError_t launch_fast_t(const FastArgs &a, const FastConst &fc, int grid, int kp, int mode, hipStream_t s)
{
    FastArgs b = a;
    const bool eq3 = a.obj.kind != 0;
    const int waves = a.small ? a.waves : kSearchWaves;
    b.lst_off = fast_lists_in_image(a.lay, waves, kp) ? 0 : a.lay.total_floats + kFastPar;
    const size_t lds = fast_dyn_lds(a.lay, waves, kp, (size_t)a.ep_bytes);
    if (a.small) {
        if (mode != kModeSearch && mode != kModeList) return hipErrorInvalidValue;
        auto fn = eq3 ? small_kernel<MAXN, A, H, kSearchWaves, true, SIG>
                      : small_kernel<MAXN, A, H, kSearchWaves, false, SIG>;
        if (waves != kSearchWaves) {
            if constexpr (MAXN <= 8 && !SIG)
                fn = eq3 ? small_kernel<MAXN, A, H, kSearchWavesWide, true, SIG>
                         : small_kernel<MAXN, A, H, kSearchWavesWide, false, SIG>;
            else
                return hipErrorInvalidValue;
        }
        hipError_t e = ensure_dyn_lds((const void *)fn, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fn, dim3(grid), dim3(waves * 64), lds, s, b, fc, kp);
        return hipGetLastError();
    }
    auto fn = eq3 ? scan_kernel<MAXN, A, H, true, SIG> : scan_kernel<MAXN, A, H, false, SIG>;
    hipError_t e = ensure_dyn_lds((const void *)fn, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(waves * 64), lds, s, b, fc, mode, kp);
    return hipGetLastError();
}

// The kernels of one model-count class and hidden width (a source file each,
// so that they compile in parallel).  Sigmoid outputs run on the 16-model
// kernels.
template <int MAXN, int H>
hipError_t launch_fast_for(const FastArgs &a, const FastConst &fc, int grid, int kp, int mode, hipStream_t s)
{
#define MF_FAST_CASE(AA)                                                                                       \
    if (a.lay.A == AA) {                                                                                       \
        if (!fc.act) return launch_fast_t<MAXN, AA, H, false>(a, fc, grid, kp, mode, s);                       \
        if constexpr (MAXN == kMaxN) return launch_fast_t<MAXN, AA, H, true>(a, fc, grid, kp, mode, s);        \
    }
    MF_FAST_CASE(2) MF_FAST_CASE(4) MF_FAST_CASE(6) MF_FAST_CASE(8)
#undef MF_FAST_CASE
    return hipErrorInvalidValue;
}

}  // namespace mfi
