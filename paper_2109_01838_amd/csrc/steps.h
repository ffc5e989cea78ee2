// Arithmetic of single steps that more than one kernel takes: the signs of the costs, the six min-marginal updates of a
// triangle and the rank of an edge in the matching.  One definition, so that every path rounds and breaks ties alike.
#pragma once

#include "prim.h"

namespace rama {

// both sign counters in one scan: attractive edges count in the low word, repulsive ones in the high word
struct SignFlags {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "SignFlags";
    const float *c;
    __device__ __forceinline__ uint64_t operator()(size_t e) const
    {
        const float w = c[e];
        return w > 0.0f ? 1ull : (w < 0.0f ? (1ull << 32) : 0ull);
    }
};

// order of the candidate edges: larger cost first, then earlier position
__device__ __forceinline__ uint32_t ordered_bits(float x)
{
    uint32_t u = __float_as_uint(x + 0.0f);   // -0 and +0 rank alike
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ unsigned long long edge_rank(float cost, uint32_t e)
{
    return ((unsigned long long)ordered_bits(cost) << 32) | (unsigned long long)(0xFFFFFFFFu - e);
}

// costs of the four non-trivial labelings of M_T = {000,110,101,011,111}
struct TriCosts {
    float l110, l101, l011, l111;
};
__device__ __forceinline__ TriCosts labeling_costs(float a, float b, float c)
{
    TriCosts r;
    r.l110 = a + b;
    r.l101 = a + c;
    r.l011 = b + c;
    r.l111 = (a + b) + c;
    return r;
}
// min-marginal of slot s: min over labelings that cut s minus min over those that do not
__device__ __forceinline__ float min_marginal(float a, float b, float c, int s)
{
    TriCosts l = labeling_costs(a, b, c);
    if (s == 0) return fminf(fminf(l.l110, l.l101), l.l111) - fminf(0.0f, l.l011);
    if (s == 1) return fminf(fminf(l.l110, l.l011), l.l111) - fminf(0.0f, l.l101);
    return fminf(fminf(l.l101, l.l011), l.l111) - fminf(0.0f, l.l110);
}

// the six updates of one triangle (slot, weight) = (0,1/3),(1,1/2),(2,1),(0,1/2),(1,1),(0,1), each on the current
// costs; oa, ob, oc: what its edges get
__device__ __forceinline__ void triangle_to_edges(float &a, float &b, float &c, float &oa, float &ob, float &oc)
{
    const float third = 1.0f / 3.0f, half = 1.0f / 2.0f;
    float d;
    oa = 0.0f; ob = 0.0f; oc = 0.0f;
    d = third * min_marginal(a, b, c, 0); a = a - d; oa = oa + d;
    d = half * min_marginal(a, b, c, 1);  b = b - d; ob = ob + d;
    d = 1.0f * min_marginal(a, b, c, 2);  c = c - d; oc = oc + d;
    d = half * min_marginal(a, b, c, 0);  a = a - d; oa = oa + d;
    d = 1.0f * min_marginal(a, b, c, 1);  b = b - d; ob = ob + d;
    d = 1.0f * min_marginal(a, b, c, 0);  a = a - d; oa = oa + d;
}

}  // namespace rama
