// Device code shared by the kernels of the library: wave helpers, candidate
// thresholds, the fp64 re-evaluation of a plan, index decoding and the
// per-level recurrence of a row.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>

#include <type_traits>

#include "dyplan_internal.h"

namespace dyp {


// Descriptors and tables never change while a kernel runs: reading them
// through the constant address space lets wave-uniform reads become scalar
// loads (and the inner-sweep trip counts stay uniform).
#if defined(__HIP_DEVICE_COMPILE__)
#define CS __attribute__((address_space(4)))
#else
#define CS
#endif
typedef const CS ProbDev* PD;
typedef const CS JobDev* JD;

template <class T>
__device__ __forceinline__ const CS T* cs(const T* p) {
    return (const CS T*)p;
}

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t mdiv(uint32_t x, const CS Magic& g) {
    uint32_t t = __umulhi(g.m, x);
    return (t + ((x - t) >> g.sh1)) >> g.sh2;
}

// Wave-wide max of an unsigned key with DPP row shifts and row broadcasts
// (lane 63 ends with the maximum); the result is read back uniformly.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x113, 0xf, 0xf, false));  // row_shr:3
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xe, false));  // row_shr:4
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xc, false));  // row_shr:8
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Candidate threshold from the fp32 corr `s` of a certainly-feasible plan.
// With |corr32 - corr64| <= g corr64 + eta for every plan (g = (2N+1) 2^-24,
// eta = N 2^-148), the exact winner W satisfies corr32_W >= returned value.
__device__ __forceinline__ float cand_threshold(float s, int n) {
    if (!(s >= 0.0f)) return -INFINITY;
    const double g = (2.0 * n + 1.0) * 0x1p-24;
    const double eta = (double)n * 0x1p-148;
    double t = ((double)s - eta) * (1.0 - g) / (1.0 + g) - eta;
    t = t - fabs(t) * 0x1p-48;
    return __double2float_rd(t);
}

// ---- objective mode: keys and thresholds ----------------------------------------

// Order-preserving unsigned key of a float (a greater number has a greater
// key; no number maps to 0, which marks "none").
__device__ __forceinline__ uint32_t fkey(float x) {
    const uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float fkey_value(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__device__ __forceinline__ uint64_t dkey(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// An fp32 value <= a - b (exact real difference): the fp64 difference, lowered
// by more than its rounding error, rounded down.
__device__ __forceinline__ float sub_rd(double a, double b) {
    double x = a - b;
    x = x - (fabs(a) + fabs(b)) * 0x1p-50;
    return __double2float_rd(x);
}

// Candidate threshold of level k from the best estimate s of any plan's J_k:
// every estimate is within err2/2 of the plan's fp64 J_k, so the winner's
// estimate is >= s - err2.
__device__ __forceinline__ float obj_threshold(float s, double err2) {
    return sub_rd((double)s, err2);
}

// fp32 estimate of a plan's J_k.  The weight m may lie beyond fp32 where D is
// small enough (+inf here): a plan of D = 0 has J_k = G, one of D > 0 an
// estimate of -inf, which raises no seed.
__device__ __forceinline__ float obj_estimate(float m, float D, float G) { return D > 0.0f ? fmaf(-m, D, G) : G; }

// Prefilter bin threshold: an fp32 value <= thr + m D_low (exact), m >= 0.
__device__ __forceinline__ float obj_bin_threshold(float thr, double m, float dlow) {
    if (thr == -INFINITY) return -INFINITY;
    const double md = m * (double)dlow;
    double x = (double)thr + md;
    x = x - (fabs((double)thr) + md) * 0x1p-50;
    return __double2float_rd(x);
}

// exact test of the scoring passes: some level's J_k estimate G - m_k D (one
// rounding) reaches its threshold
__device__ __forceinline__ bool is_candidate_obj(PD P, JD J, float G, float D) {
    for (int k = 0; k < P->k; ++k)
        if (fma(-P->m64[k], (double)D, (double)G) >= (double)J->thr[k]) return true;
    return false;
}

// J_k = U - lambda_l T - m_k D in fp64, operation by operation as the definition
// writes it (no contraction into fused multiply-adds).
__device__ __forceinline__ double obj_j(double lam_l, double m, double U, double T, double D) {
#pragma clang fp contract(off)
    double j = lam_l * T;
    j = U - j;
    const double q = m * D;
    return j - q;
}

// ---- fp64 re-evaluation ------------------------------------------------------
// The per-node terms (1 - w(1-p), tau/(1-rho), tau*size) are precomputed on the
// host in fp64 with the same operations as the definition, so the products,
// sums and maxima below reproduce an fp64 evaluation of the definition in
// node order bit for bit.  ids / f are strided per-thread columns.

__device__ double ex_corr(PD P, const uint8_t* ids, int is) {
    const CS double* a = cs(P->a64);
    double c = 1.0;
    for (int n = 0; n < P->n; ++n) c = c * a[n * P->rmax + ids[n * is]];
    return c;
}

__device__ double ex_cp(PD P, const uint8_t* ids, int is, int k, double* f, int fs) {
    const CS double* lat = cs(P->lat64) + (size_t)k * P->n * P->rmax;
    double cp = 0.0;
    for (int n = 0; n < P->n; ++n) {
        double m = 0.0;
        uint32_t pm = P->pred[n];
        while (pm) {
            const int u = __builtin_ctz(pm);
            pm &= pm - 1;
            const double fu = f[u * fs];
            if (fu > m) m = fu;
        }
        const double fn = lat[n * P->rmax + ids[n * is]] + m;
        f[n * fs] = fn;
        if ((P->sinks >> n & 1u) && fn > cp) cp = fn;
    }
    return cp;
}

// Objective mode: U (returned), T and D in fp64, node order (the definition's).
__device__ double ex_obj(PD P, const uint8_t* ids, int is, double* f, int fs, double& T, double& D) {
    const CS double* u64 = cs(P->a64);
    const CS double* d64 = cs(P->dem64);
    const CS double* t64 = cs(P->lat64);
    double U = 0.0, d = 0.0, t = 0.0;
    for (int n = 0; n < P->n; ++n) {
        const int e = n * P->rmax + ids[n * is];
        if (P->llm >> n & 1u) {
            U = U + u64[e];
            d = d + d64[e];
        }
        double m = 0.0;
        uint32_t pm = P->pred[n];
        while (pm) {
            const int u = __builtin_ctz(pm);
            pm &= pm - 1;
            const double fu = f[u * fs];
            if (fu > m) m = fu;
        }
        const double fn = t64[e] + m;
        f[n * fs] = fn;
        if ((P->sinks >> n & 1u) && fn > t) t = fn;
    }
    T = t;
    D = d;
    return U;
}

__device__ double ex_demand(PD P, const uint8_t* ids, int is) {
    const CS double* d64 = cs(P->dem64);
    double d = 0.0;
    for (int n = 0; n < P->n; ++n) d = d + d64[n * P->rmax + ids[n * is]];
    return d;
}

// Implementation ids of plan `index` of the problem (node N-1 least significant).
__device__ void decode64(PD P, uint64_t index, uint8_t* ids, int is) {
    if (index <= 0xffffffffull) {
        uint32_t x = (uint32_t)index;
        for (int n = P->n - 1; n >= 0; --n) {
            const uint32_t q = mdiv(x, P->rmag[n]);
            ids[n * is] = (uint8_t)(x - q * (uint32_t)P->radix[n]);
            x = q;
        }
        return;
    }
    for (int n = P->n - 1; n >= 0; --n) {
        const uint64_t r = (uint64_t)P->radix[n];
        ids[n * is] = (uint8_t)(index % r);
        index /= r;
    }
}

// ids of a candidate or of a fallback unit; returns false for a bad row id
__device__ bool job_ids(JD J, PD P, uint64_t index, uint8_t* ids, int is) {
    if (J->kind == DY_SOURCE_RANGE) {
        decode64(P, index, ids, is);
        return true;
    }
    const uint8_t* row = J->rows + (index - J->index_base) * J->stride;
    const int N = P->n;
    bool ok = true;
    // eight byte loads in flight at a time (a lane otherwise waits on each)
    for (int n0 = 0; n0 < N; n0 += 8) {
        uint8_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = n0 + j < N ? row[n0 + j] : (uint8_t)0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = n0 + j;
            if (n < N) {
                uint8_t x = v[j];
                if (x >= (uint32_t)P->radix[n]) {
                    ok = false;
                    x = 0;
                }
                ids[n * is] = x;
            }
        }
    }
    return ok;
}

__device__ __forceinline__ void append_cand(JD J, uint64_t index, float c, float cp) {
    uint32_t slot = atomicAdd(J->ncand, 1u);
    if (slot < J->cap) {
        Cand* d = J->cand + slot;
        d->index = index;
        d->corr = c;
        d->cp = cp;
    } else {
        atomicOr(J->flags, (int32_t)JF_OVERFLOW);
    }
}

// exact per-level candidate test of the scoring pass (levels in P->k)
__device__ __forceinline__ bool is_candidate(PD P, JD J,
                                             float cp, float c) {
    for (int k = 0; k < P->k; ++k)
        if (cp <= P->hi[k] && c >= J->thr[k]) return true;
    return false;
}

// Digit of prefix node n in block index b (node 0 most significant).
__device__ __forceinline__ uint32_t prefix_digit(PD P, int n, uint64_t b, int big) {
    if (!big) {
        const uint32_t q = P->pv_big[n] ? 0u : mdiv((uint32_t)b, P->pvmag[n]);
        return q - mdiv(q, P->rmag[n]) * (uint32_t)P->radix[n];
    }
    return (uint32_t)((b / P->pv64[n]) % (uint64_t)P->radix[n]);
}

// Per-backend pressure (not uniform): the level-k state of a row of the
// sweep, for the exact per-level tests of the seeding pass and of the rare
// path.  `dg` holds the prefix digits of the block.  NPRE > 0: the prefix has
// exactly NPRE nodes, the recurrence is unrolled with every f_n in a register;
// NPRE == 0: any length, f_n in the thread's LDS column s_f.  Returns M (the
// path into y other than through y's own duration) and S2 (the longest path
// ending at another sink), as the sweep forms them at level 0.
template <int NPRE>
__device__ __forceinline__ void level_row(PD P, const CS float* lat, const uint32_t* dg, uint64_t b, int big, int ix,
                          float* __restrict__ s_f, float& M, float& S2) {
    const int R = P->rmax, xn = P->xnode;
    const uint32_t pmx = xn >= 0 ? P->pred[xn] : 0u;
    const uint32_t pmy = P->pred[P->ynode] & (xn >= 0 ? ~(1u << xn) : ~0u);
    float px = 0.0f, py = 0.0f, s = 0.0f;
    if constexpr (NPRE > 0) {
        float f[NPRE];
#pragma unroll
        for (int n = 0; n < NPRE; ++n) {
            float m = 0.0f;
            const uint32_t pm = P->pred[n];
#pragma unroll
            for (int u = 0; u < n; ++u)
                if (pm >> u & 1u) m = fmaxf(m, f[u]);
            f[n] = lat[n * R + dg[n]] + m;
        }
#pragma unroll
        for (int u = 0; u < NPRE; ++u) {
            if (pmx >> u & 1u) px = fmaxf(px, f[u]);
            if (pmy >> u & 1u) py = fmaxf(py, f[u]);
            if (P->pre_sinks >> u & 1u) s = fmaxf(s, f[u]);
        }
    } else {
        const int tid = threadIdx.x;
        for (int n = 0; n < P->npre; ++n) {
            const uint32_t d = prefix_digit(P, n, b, big);
            float m = 0.0f;
            uint32_t pm = P->pred[n];
            while (pm) {
                const int u = __builtin_ctz(pm);
                pm &= pm - 1;
                m = fmaxf(m, s_f[u * WG + tid]);
            }
            s_f[n * WG + tid] = lat[n * R + d] + m;
        }
        auto pmax = [&](uint32_t pm) {
            float v = 0.0f;
            while (pm) {
                const int u = __builtin_ctz(pm);
                pm &= pm - 1;
                v = fmaxf(v, s_f[u * WG + tid]);
            }
            return v;
        };
        px = pmax(pmx);
        py = pmax(pmy);
        s = pmax(P->pre_sinks);
    }
    const float fx = (xn >= 0 ? lat[xn * R + ix] : 0.0f) + px;
    const bool exy = P->edge_xy != 0;
    M = exy ? fmaxf(py, fx) : py;
    S2 = exy ? s : fmaxf(s, fx);
}

template <int NPRE>
__device__ __forceinline__ void prefix_digits(PD P, uint64_t b, int big, uint32_t* dg) {
    if constexpr (NPRE > 0) {
#pragma unroll
        for (int n = 0; n < NPRE; ++n) dg[n] = prefix_digit(P, n, b, big);
    }
}

// Work unit of sample j: one unit of the window [j S, min((j+1) S, n)), at a
// hashed offset.  A fixed offset would alias with the mixed-radix digits (a
// stride sharing factors with the radices visits only some implementation ids
// of the low-order prefix nodes).
__device__ __forceinline__ uint64_t sample_unit(uint64_t j, uint64_t S, uint64_t n) {
    const uint64_t start = j * S;
    const uint32_t width = (uint32_t)min(S, n - start);
    const uint32_t h = (uint32_t)(j * 0x9E3779B1ull) >> 16;
    return start + (uint64_t)(h % width);
}

__device__ __forceinline__ bool better(double c1, uint64_t i1, double c2, uint64_t i2) {
    return c1 > c2 || (c1 == c2 && i1 < i2);
}

}  // namespace dyp
