// fp32 fast path, host side: support, LDS budget and dispatch to the kernel
// instantiations (mf_fast_kernel.h); the per-workgroup list merge and the
// per-option layer-1 precompute.
#include "mf_canon.h"

namespace mfi {

// Bytes of LDS (after the workgroup lists) the certification tail needs: the
// evaluated list keys, a status word, per (entry, model) predictions of one
// chunk of kCertChunk entries, and each chunk entry's option rows.
size_t fast_small_epilogue_bytes(int n_models)
{
    return 64 * 8 + 16 + (size_t)kCertChunk * n_models * 16 + (size_t)kCertChunk * kMaxN * 4 +
           (size_t)kSearchWavesWide * 64 * 8 + (size_t)kCertChunk * sizeof(K128);
}

// ---------------------------------------------------------------------------
// Merge the per-workgroup lists into one sorted top-kp list (one workgroup).
// ---------------------------------------------------------------------------
constexpr int kMergeWaves = 16;

constexpr int kMergeStageKeys = 4096;   // keys staged in LDS per pass

// Each per-workgroup list is sorted: the lists are staged in LDS a batch at a
// time (every thread loading), wave w merges lists w, w + 16, ... of the
// batch into its own, then wave 0 merges the 16.  The workgroups' counts are
// summed into counts_out[0..1] (VRAM-feasible, surely feasible).
template <int NS>
__global__ void __launch_bounds__(kMergeWaves * 64)
merge_lists_kernel(const unsigned long long *lists, int n_lists, int kp, unsigned long long *out,
                   const unsigned long long *wg_counts, unsigned long long *counts_out)
{
    __shared__ unsigned long long stage[kMergeStageKeys];
    __shared__ unsigned long long lst[kMergeWaves * 64 * NS];
    __shared__ unsigned long long s_cnt[2 * kMergeWaves];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    WaveList<NS> L, L2;   // two independent merge chains per wave
    wl_init(L);
    wl_init(L2);
    const int per_pass = kMergeStageKeys / kp;   // kp <= 128: at least 32 lists
    for (int l0 = 0; l0 < n_lists; l0 += per_pass) {
        const int nl = n_lists - l0 < per_pass ? n_lists - l0 : per_pass;
        __syncthreads();
        for (int t = threadIdx.x; t < nl * kp; t += kMergeWaves * 64) stage[t] = lists[(uint64_t)l0 * kp + t];
        __syncthreads();
        for (int i = wv; i < nl; i += 2 * kMergeWaves) {
            const int i2 = i + kMergeWaves;
            unsigned long long b[NS], b2[NS];
#pragma unroll
            for (int j = 0; j < NS; j++) {
                const bool in = j * 64 + lane < kp;
                b[j] = in ? stage[i * kp + j * 64 + lane] : 0ull;
                b2[j] = in && i2 < nl ? stage[i2 * kp + j * 64 + lane] : 0ull;
            }
            wl_merge_sorted(L, b, lane, kp);
            wl_merge_sorted(L2, b2, lane, kp);
        }
    }
    wl_merge_sorted(L, L2.s, lane, kp);
    unsigned long long cv = 0, cf = 0;
    if (wg_counts)
        for (int i = threadIdx.x; i < n_lists; i += kMergeWaves * 64) {
            cv += wg_counts[2 * (uint64_t)i];
            cf += wg_counts[2 * (uint64_t)i + 1];
        }
    cv = wave_sum64(cv);
    cf = wave_sum64(cf);
    if (lane == 0) {
        s_cnt[wv] = cv;
        s_cnt[kMergeWaves + wv] = cf;
    }
#pragma unroll
    for (int j = 0; j < NS; j++) lst[(wv * NS + j) * 64 + lane] = L.s[j];
    wl_tree_merge<NS, kMergeWaves>(L, lst, NS * 64, wv, lane, kp);
    if (wv == 0) {
#pragma unroll
        for (int j = 0; j < NS; j++)
            if (j * 64 + lane < kp) out[j * 64 + lane] = L.s[j];
        if (wg_counts && lane < 2) {
            unsigned long long t = 0;
            for (int w = 0; w < kMergeWaves; w++) t += s_cnt[lane * kMergeWaves + w];
            counts_out[lane] = t;
        }
    }
}

int fast_kernel_supported(int n_models, int A, int H, int kp)
{
    if (n_models < 1 || n_models > 16) return 0;
    if (!(A == 2 || A == 4 || A == 6 || A == 8)) return 0;
    if (!(H == 32 || H == 64)) return 0;
    if (kp < 1 || kp > 64) return 0;
    return 1;
}

// 16 waves per workgroup (4 per SIMD) when the per-wave registers fit 128
// VGPRs (up to 8 models) and the image plus 16 candidate lists fit in LDS.
int fast_waves_for(int n_models, const FastLayout &lay, int kp, int act)
{
    const size_t lds = fast_dyn_lds(lay, kSearchWavesWide, kp, 0);
    return (n_models <= 8 && lds <= (size_t)kFastLdsMax && !act) ? kSearchWavesWide : kSearchWaves;
}

hipError_t launch_fast_impl(const FastArgs &a, const FastConst &fc, int grid, int kp, int mode, hipStream_t s)
{
    // sigmoid outputs run on the generic kernel (16 models)
    const bool n8 = fc.n_models <= 8 && !fc.act;
    switch (a.lay.H) {
        case 32: return n8 ? launch_fast_n8_h32(a, fc, grid, kp, mode, s) : launch_fast_n16_h32(a, fc, grid, kp, mode, s);
        case 64: return n8 ? launch_fast_n8_h64(a, fc, grid, kp, mode, s) : launch_fast_n16_h64(a, fc, grid, kp, mode, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_merge_lists(const unsigned long long *lists, int n_lists, int kp, unsigned long long *out,
                              const unsigned long long *wg_counts, unsigned long long *counts_out, hipStream_t s)
{
    if (kp <= 64)
        hipLaunchKernelGGL(merge_lists_kernel<1>, dim3(1), dim3(kMergeWaves * 64), 0, s, lists, n_lists, kp, out,
                           wg_counts, counts_out);
    else
        hipLaunchKernelGGL(merge_lists_kernel<2>, dim3(1), dim3(kMergeWaves * 64), 0, s, lists, n_lists, kp, out,
                           wg_counts, counts_out);
    return hipGetLastError();
}

}  // namespace mfi

namespace mfi {

// Per-option first-layer precompute (the option's own columns, Eq. 6, plus
// the aggregate centre c the fast path subtracts from the aggregate):
// P[row][h] = b1[h] + sum_k W1[h][k] x[row][k] + sum_k W1_agg[h][k] c[k],
// one fp64 fma chain, rounded to fp32.  Reads the canonical image (W1T[k][h]).
__global__ void precompute_p_kernel(const float *features, const float *canon_w, const float *centre, int n_rows,
                                    int L, int A, int H, int64_t wstride, const int32_t *row_model, float *image_p,
                                    int pst, Pow2Scales sc)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n_rows * H) return;
    const int row = (int)(t / H), h = (int)(t % H);
    const int nin = L + A;
    const float *w = canon_w + (int64_t)row_model[row] * wstride;
    const float *W1T = w, *b1 = w + (int64_t)nin * H;
    double c = (double)b1[h];
    for (int k = 0; k < L; k++) c = fma((double)W1T[(int64_t)k * H + h], (double)features[(int64_t)row * L + k], c);
    for (int k = 0; k < A; k++) c = fma((double)W1T[(int64_t)(L + k) * H + h], (double)centre[k], c);
    // the fast image's layer-1 scale 2^e (exact: rounding commutes with it)
    image_p[(int64_t)row * pst + h] = (float)ldexp(c, sc.e[row_model[row]]);
}

hipError_t launch_precompute_p(const float *features, const float *weights, const float *centre, int n_rows, int L,
                               int A, int H, int64_t wstride, const int32_t *row_model, float *image_p, int pst,
                               const Pow2Scales &sc, hipStream_t s)
{
    const int64_t total = (int64_t)n_rows * H;
    const int blk = 256;
    const int grid = (int)((total + blk - 1) / blk);
    hipLaunchKernelGGL(precompute_p_kernel, dim3(grid), dim3(blk), 0, s, features, weights, centre, n_rows, L, A, H,
                       wstride, row_model, image_p, pst, sc);
    return hipGetLastError();
}

}  // namespace mfi
