// The active experts of one token from its logits, shared by every kernel that routes a token in one lane.  Nothing here
// needs a GPU: the host can compile it, with the qualifiers and the exp2 builtin defined away.
#pragma once

#include <math.h>
#include <stdint.h>

namespace swimba {

// Top-k over E logits read through `load(e)`, in (logit descending, index
// ascending) order; softmax over all E, no renormalisation.
// exp(v) for v <= 0 through the hardware exp2 (about 1 ulp; the product v * log2(e) adds a
// relative error of |v| * 2^-24, far inside the 1e-5 the routing weights are held to)
__device__ __forceinline__ float route_exp(float v) { return __builtin_amdgcn_exp2f(v * 1.4426950408889634f); }

// Only a NaN among the logits, outside the contract, leaves a pick without a candidate.  The result is undefined then, but the
// index stays a valid one, which addresses the expert rows, and one that the token has not picked yet: an expert's list of the
// projection has a place for every token, not two.  First expert behind the last pick, cyclically, that is still open.
__device__ __forceinline__ int route_open(uint32_t picked, int pi, int E)        // one bit an expert
{
    const uint32_t open = ~picked & ((1u << E) - 1), behind = open & ~((2u << pi) - 1);
    return __builtin_ctz(behind ? behind : open);
}
__device__ __forceinline__ int route_open(const int32_t *idx, int r, int pi, int E)      // idx[0 .. r) are picked
{
    int e = pi + 1 < E ? pi + 1 : 0;
    for (int q = 0; q < r;)
        if (idx[q] == e) { e = e + 1 < E ? e + 1 : 0; q = 0; }
        else ++q;
    return e;
}

// E <= EM experts, their logits in registers: a loop that loads one after the other waits for each.  KM: most picks, where these
// are registers, too.
template <int EM, int KM = 0, typename Load>           // EM < 32
__device__ __forceinline__ void route_few(Load load, int E, int K, int32_t *idx, float *w)
{
    float v[EM], m = -INFINITY, Z = 0.f;
#pragma unroll
    for (int e = 0; e < EM; ++e) v[e] = load(e < E ? e : E - 1);
#pragma unroll
    for (int e = 0; e < EM; ++e) m = fmaxf(m, v[e]);
#pragma unroll
    for (int e = 0; e < EM; ++e) Z += e < E ? route_exp(v[e] - m) : 0.f;
    const float invZ = 1.0f / Z;
    float pv = 0.f;
    int pi = -1;
    uint32_t picked = 0;
    auto pick = [&](int r) __attribute__((always_inline)) {
        int best = -1;
        float bv = 0.f;
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            const bool after = (r == 0) || (v[e] < pv) || (v[e] == pv && e > pi);
            if (e < E && after && (best < 0 || v[e] > bv)) { best = e; bv = v[e]; }
        }
        if (best < 0) { best = route_open(picked, pi, E); bv = NAN; }      // no candidate for the picks behind it either
        picked |= 1u << best;
        idx[r] = best;
        w[r] = route_exp(bv - m) * invZ;
        pv = bv;
        pi = best;
    };
    if constexpr (KM > 0) {
#pragma unroll
        for (int r = 0; r < KM; ++r)
            if (r < K) pick(r);
    } else {
        for (int r = 0; r < K; ++r) pick(r);
    }
}

constexpr int ROUTE_FEW = 16;                          // most experts whose logits lie in registers

template <typename Load>
__device__ __forceinline__ void route_many(Load load, int E, int K, int32_t *idx, float *w)
{
    float m = -INFINITY;
    for (int e = 0; e < E; ++e) m = fmaxf(m, load(e));
    float Z = 0.f;
    for (int e = 0; e < E; ++e) Z += route_exp(load(e) - m);
    const float invZ = 1.0f / Z;
    float pv = 0.f;
    int pi = -1;
    for (int r = 0; r < K; ++r) {
        int best = -1;
        float bv = 0.f;
        for (int e = 0; e < E; ++e) {
            const float v = load(e);
            // candidates are the experts that come after the previous pick in the order
            const bool after = (r == 0) || (v < pv) || (v == pv && e > pi);
            if (after && (best < 0 || v > bv)) { best = e; bv = v; }
        }
        if (best < 0) { best = route_open(idx, r, pi, E); bv = NAN; }
        idx[r] = best;
        w[r] = route_exp(bv - m) * invZ;
        pv = bv;
        pi = best;
    }
}

template <typename Load>
__device__ __forceinline__ void route_token(Load load, int E, int K, int32_t *idx, float *w)
{
    if (E <= 8) return route_few<8>(load, E, K, idx, w);
    if (E <= ROUTE_FEW) return route_few<ROUTE_FEW>(load, E, K, idx, w);
    route_many(load, E, K, idx, w);
}

}  // namespace swimba
