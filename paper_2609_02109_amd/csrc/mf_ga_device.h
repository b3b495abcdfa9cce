// Device code shared by the GA's kernels (mf_ga.hip, mf_ga_run.hip): the
// counter-based draws, the fitness terms and the order of individuals.
#pragma once

#include "mf_canon.h"

namespace mfi {

enum { kPInit = 1, kPSel = 2, kPCx = 8, kPSwap = 9, kPMut = 16, kPRep = 32 };

struct Philox4 {
    uint64_t w[4];
};

// The 128-bit product a b: its high and low 64 bits from four 32 x 32 -> 64
// multiply-adds (no partial sum overflows 64 bits).
__device__ __forceinline__ void mulhilo64(uint64_t a, uint64_t b, uint64_t &hi, uint64_t &lo)
{
    const uint64_t a0 = (uint32_t)a, a1 = a >> 32, b0 = (uint32_t)b, b1 = b >> 32;
    const uint64_t p00 = a0 * b0;
    const uint64_t t1 = a0 * b1 + (p00 >> 32);
    const uint64_t t2 = a1 * b0 + (t1 & 0xFFFFFFFFull);
    hi = a1 * b1 + (t1 >> 32) + (t2 >> 32);
    lo = (t2 << 32) | (p00 & 0xFFFFFFFFull);
}

__device__ __forceinline__ Philox4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                                 uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; r++) {
        if (r) { k0 += W0; k1 += W1; }
        uint64_t h0, l0, h1, l1;
        mulhilo64(M0, c0, h0, l0);
        mulhilo64(M1, c2, h1, l1);
        const uint64_t y0 = h1 ^ c1 ^ k0, y2 = h0 ^ c3 ^ k1;
        c0 = y0; c1 = l1; c2 = y2; c3 = l0;
    }
    return Philox4{{c0, c1, c2, c3}};
}

__device__ __forceinline__ uint64_t ga_draw(uint64_t seed, uint64_t item, uint64_t gen, uint64_t scen,
                                            uint64_t purpose, int word)
{
    const Philox4 p = philox4x64_10(item, gen, scen, purpose, seed, 0);
    return p.w[word & 3];
}
__device__ __forceinline__ double ga_uni(uint64_t r) { return (double)(r >> 11) * 0x1p-53; }
__device__ __forceinline__ uint64_t ga_below(uint64_t r, uint64_t n) { return ((r >> 32) * n) >> 32; }

// Mixed-radix digits of a joint index, model 0 most significant (the decode of
// Eq. 1's configuration vector); 32-bit divisions when the space fits 32 bits.
__device__ __forceinline__ void ga_digits(const GAConst &c, uint64_t idx, int32_t *d)
{
    if (c.space <= 0x100000000ull) {
        uint32_t x = (uint32_t)idx;
        for (int i = c.N - 1; i >= 0; i--) {
            const uint32_t k = (uint32_t)c.K[i], q = x / k;
            d[i] = (int32_t)(x - q * k);
            x = q;
        }
    } else {
        for (int i = c.N - 1; i >= 0; i--) {
            d[i] = (int32_t)(idx % (uint64_t)c.K[i]);
            idx /= (uint64_t)c.K[i];
        }
    }
}

// One model's term of the canonical fitness, in the order every fitness
// kernel takes it: the service constraint (Eq. 4), then J = fma(omega, thr,
// J) or, under Eq. 3, the utility's terms (throughput floor as a constraint).
__device__ __forceinline__ void ga_term(const GAConst &c, int s, int i, int64_t row, double lat, double thr,
                                        const float *sla, const float *omega, const float *tau,
                                        const int32_t *prev, double &J, bool &ok)
{
    if (!(lat <= (double)sla[(int64_t)s * c.N + i])) ok = false;
    const double om = (double)omega[(int64_t)s * c.N + i];
    if (c.obj.kind != 0) {
        double q, Pr, pen;
        bool do_P, do_pen;
        if (!canon_eq3(c.obj, row, thr, tau[i], prev[i], q, Pr, do_P, pen, do_pen)) ok = false;
        J = fma(om, q, J);
        if (do_P) J = J - Pr;
        if (do_pen) J = J - pen;
    } else {
        J = fma(om, thr, J);
    }
}

__device__ __forceinline__ bool ga_better(double fa, uint64_t ia, double fb, uint64_t ib)
{
    return fa > fb || (fa == fb && ia < ib);
}

// The Philox blocks of a parent pair, in a fixed order: the
// selection blocks (2k draws), the crossover block, the swap blocks (one
// word per gene), the mutation blocks of child 1 + 2q and of child 2 + 2q
// (two words per gene).  A child's repair block is drawn where it is needed.
struct OpBlocks {
    int nsel, nswap, nmut, total;
    __host__ __device__ OpBlocks(int tk, int N)
        : nsel((2 * tk + 3) / 4), nswap((N + 3) / 4), nmut((N + 1) / 2), total(nsel + 1 + nswap + 2 * nmut)
    {
    }
    __host__ __device__ int cx() const { return nsel; }
    __host__ __device__ int swap() const { return nsel + 1; }
    __host__ __device__ int mut(int t) const { return nsel + 1 + nswap + t * nmut; }
};

}  // namespace mfi
