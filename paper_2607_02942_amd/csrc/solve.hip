// Selection over RANGE sources in one launch: seeds, thresholds, the sweep of
// the plan space and the certified choices (gfx950).
//
// The space is swept by heads, a head being one assignment of every node but
// the last three (w = N-3, x = N-2, y = N-1).  Whether any of a head's plans
// can win a level depends on its product, on the longest paths into w, x and
// y, and on the longest path that ends at a sink before them.  Each workgroup
// folds y, then x, then w into tables over the bins of those paths
// (build_tables): the least product a row (all but y fixed), a block (all but
// x and y) and a head must have for some plan of it to reach the threshold of
// the CP bin it falls in.  A head then costs its own recurrence, three table
// reads and a compare; the few that pass are unfolded from queues in LDS, by
// dense lists of pairs: (head, w) into blocks, (block, x) into rows, (row, y)
// into plans, which take the exact per-level test.  Every plan of the source
// is covered by a test that it fails only if it cannot be a candidate, so the
// candidates are those that scoring each plan would give.
//
// Objective mode runs the same steps on its additive terms: the bins are
// those of D, and the tables hold the least U - lambda_l (path).  Under
// per-backend pressure every level has its own durations and takes a sweep of
// its own (but those whose candidates an earlier level's sweep has listed).
#include "device_common.h"

namespace dyp {

// Values are scaled down before they pick a bin of a folded table, the more
// the further it is folded (thresholds by row, block, head): a value then lies
// in bin b only if it exceeds the bin's low edge by so much that the sums the
// tables are formed of, with their roundings, reach the same bin of the table
// below.  (Without, each fold read one bin lower.)
constexpr float BIN_ROW = 1.0f - 0x1p-20f, BIN_BLK = 1.0f - 2 * 0x1p-20f, BIN_HEAD = 1.0f - 3 * 0x1p-20f;

// Pointers into LDS, held in structs and passed to functions.
#if defined(__HIP_DEVICE_COMPILE__)
#define LS __attribute__((address_space(3)))
#else
#define LS
#endif

constexpr int SOLVE_HEAD = 8;      // longest unrolled head
constexpr int SOLVE_Q = 320;       // queue entries (a round adds at most WG; drained above SOLVE_Q - WG)
constexpr int SOLVE_PAIRS = 1280;  // (candidate, level) pairs gathered per certification round
constexpr int SOLVE_REBUILD = 512; // rows unfolded before the tables are rebuilt on the raised seeds
constexpr int SOLVE_OWN = 32;      // candidates kept in LDS as well
constexpr int SOLVE_LAT = 4096;    // per-backend pressure: durations of all levels kept in LDS for the seeding up to this many

constexpr int SEED_LEVELS = 8;     // per-backend pressure: levels seeded at a time, at most
constexpr int SEED_NEAR = 3;       // ... and levels on each side that a level's plans are tried at

constexpr uint32_t CAND_LEVEL = 0x7fc00000u;  // per-backend pressure: a candidate's level, in place of its CP

enum { SV_LEVEL = 0, SV_CLASS = 1, SV_OBJ = 2 };

// Dynamic LDS, in bytes from its start.  The certification reuses all of it.
struct SolveLds {
    int at, dm, e3, q3, d3, col, sc, nt, lat, id, hx, hv, bq, rq, total;
};

__host__ __device__ inline SolveLds solve_lds(int ent, int rmax, int nlat, int ncol, int nmax, bool obj, bool cls) {
    SolveLds L;
    int o = 0;
    auto take = [&](int bytes) {
        const int r = o;
        o += (bytes + 15) / 16 * 16;
        return r;
    };
    L.at = take(ent * 8);                // every node's (a, tau) (objective: (u, tau))
    L.dm = take(obj ? ent * 4 : 0);      // objective: every node's d
    L.e3 = take(3 * rmax * 8);           // (a, tau) of w, x and y
    L.q3 = take(3 * rmax * 8);           // reciprocal factors of w, x and y (objective: two offsets each)
    L.d3 = take(obj ? 3 * rmax * 4 : 0); // objective: d of w, x and y
    L.col = take(ncol * WG * 4);         // recurrence columns
    L.sc = o;                            // seeding only, where the queues follow: a recurrence column per node,
    L.nt = o + nmax * WG * 4;            // every node's (-ln a, tau) (objective: (u_max - u, tau)),
    L.lat = L.nt + ent * 8;              // and (per-backend pressure) the durations at every level and an id
    L.id = L.lat + nlat * 4;             // column per node
    L.hx = take(SOLVE_Q * 8);            // parked heads: index, then product, paths, (sum of d)
    L.hv = take(SOLVE_Q * 4 * (obj ? 6 : 5));
    L.bq = take(SOLVE_Q * 4);            // parked blocks: head slot, w
    L.rq = take(SOLVE_Q * 4);            // parked rows: head slot, w, x
    const int seeding = L.id + (cls ? nmax * WG : 0);
    if (o < seeding) o = seeding;
    L.total = o;
    return L;
}

// Threads that re-evaluate (candidate, level) pairs: each needs nf doubles and
// nf id bytes of LDS beside the pair list.
__host__ __device__ inline int solve_cert_threads(int nf, int lds) {
    int t = (lds - SOLVE_PAIRS * 4) / (nf * 9) / 64 * 64;
    return t < 64 ? 64 : (t > WG ? WG : t);
}

// An fp32 r <= 1 / (a (1 + 2^-22)), at most 2^-21 relative below (see
// div_threshold): the quotient errs by 2^-24, the product too.  Below 2^-20:
// 2^-126, far below 1 / a, and T = +inf stays +inf.
__device__ __forceinline__ float down_reciprocal(float a) {
    return a >= 0x1p-20f ? (1.0f / a) * (1.0f - 0x1p-21f) : 0x1p-126f;
}

// Threshold on c given one on fp32(c a), r = down_reciprocal(a): fp32(c a) >=
// T implies c >= the value returned.  For T > 2^-60, fp32(c a) >= T gives
// c a >= T / (1 + 2^-24) (both normal), and fp32(T r) <= T r (1 + 2^-24) <=
// T / (a (1 + 2^-24)); smaller T give 0, which every c >= 0 meets.
__device__ __forceinline__ float div_threshold(float T, float r) { return T > 0x1p-60f ? T * r : 0.0f; }

// An fp32 value <= t - c (c finite), -inf for t = -inf: the difference is
// within half an ulp of the exact one and is lowered by at least an ulp (2^-23
// relative; 2^-149 where it is subnormal).
__device__ __forceinline__ float lower_by(float t, float c) {
    const float x = t - c;
    return fmaf(-fabsf(x), 0x1p-23f, x) - 0x1p-149f;
}

// An fp32 value >= w + e (e >= 0).
__device__ __forceinline__ float raise_by(double w, double e) {
    return __double2float_ru(w + e + (fabs(w) + e) * 0x1p-50);
}

// What the nodes before w give: the product of their factors (objective: sum
// of u) and the sum of their d; the longest paths into w, x and y; the longest
// path ending at a sink among them.
struct SHead {
    float pc, pd, m, px, py, s;
};

struct SBlock {  // ... with w
    float pc, pd, px, py, s;
};

struct SRow {  // ... with w and x: product (sum of u), sum of d, path into y, longest path to another sink
    float c, d, M, S2;
};

// One workgroup's view of its source.
template <int NB>
struct SolveT {
    PD P;
    JD J;
    const LS float2* s_at;
    const LS float* s_dm;
    const LS float2* s_e;     // (a, tau) of w, x, y: rows 0, 1, 2 of rmax entries
    const LS float2* s_q;
    const LS float* s_d;
    LS float* s_col;
    const CS float* lat;      // per-backend pressure: durations at the level of the pass
    const LS uint32_t* t_bin;   // tables (fp32), NB bins each
    const LS uint32_t* t_row;
    const LS uint32_t* t_blk;
    const LS uint32_t* t_head;
    const LS uint32_t* t_rowu;  // objective: row without y's path, block and head off the path to x
    const LS uint32_t* t_blky;
    const LS uint32_t* t_headx;
    const LS uint32_t* t_heady;
    const LS float* s_thr;
    const LS float* s_lo;
    const LS float* s_hi;
    int stg;                  // the node tables are staged (per-backend pressure: with the level's durations)
    int rmax, sh;             // sh: shift of a bin's byte offset
    float lo, top;            // least CP (D); a value in the first bin that no level admits
    float dy, dxy, dw;        // least parts of y, of x and y, and of w and what follows it
    float aw, ax, ay;         // largest factors
    float nl;                 // objective: -lambda_l
    uint32_t mx, my, ms;      // w feeds x, feeds y, is a sink: all ones, else 0
    uint32_t sinks;           // sinks before w

    __device__ __forceinline__ float2 ent(int e) const {
        if (stg) return make_float2(s_at[e].x, s_at[e].y);
        float2 v = cs(P->at)[e];
        if (lat) v.y = lat[e];
        return v;
    }
    __device__ __forceinline__ float dem(int e) const { return stg ? s_dm[e] : cs(P->dem)[e]; }
    __device__ __forceinline__ float2 e3(int row, int i) const {
        const LS float2* q = s_e + row * rmax + i;
        return make_float2(q->x, q->y);
    }
    __device__ __forceinline__ float2 q3(int row, int i) const {
        const LS float2* q = s_q + row * rmax + i;
        return make_float2(q->x, q->y);
    }
    __device__ __forceinline__ float d3(int row, int i) const { return s_d[row * rmax + i]; }
    __device__ __forceinline__ uint32_t off(float v) const {
        return (__float_as_uint(__builtin_amdgcn_fmed3f(v, lo, top)) >> sh) & (uint32_t)((NB - 1) * 4);
    }
};

__device__ __forceinline__ float tab(const LS uint32_t* t, uint32_t off) {
    return *(const LS float*)((const LS char*)t + off);
}

// Head x (mixed radix over its nodes, the last least significant) of exactly
// NH nodes; the same operations in the same order as a plan's own evaluation.
template <int NH, bool OBJ, class SV>
__device__ __forceinline__ SHead head_nh(const SV& S, uint64_t x, int big) {
    PD P = S.P;
    SHead h{OBJ ? 0.0f : 1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (NH > 0) {
        uint32_t dg[NH];
        float f[NH];
        if (!big) {
            uint32_t q = (uint32_t)x;
#pragma unroll
            for (int n = NH - 1; n >= 0; --n) {
                const uint32_t t = mdiv(q, P->rmag[n]);
                dg[n] = q - t * (uint32_t)P->radix[n];
                q = t;
            }
        } else {
#pragma unroll
            for (int n = NH - 1; n >= 0; --n) {
                const uint64_t r = (uint64_t)P->radix[n];
                dg[n] = (uint32_t)(x % r);
                x /= r;
            }
        }
#pragma unroll
        for (int n = 0; n < NH; ++n) {
            const int e = n * S.rmax + (int)dg[n];
            const float2 v = S.ent(e);
            if (OBJ) {
                h.pc = h.pc + v.x;
                h.pd = h.pd + S.dem(e);
            } else {
                h.pc = h.pc * v.x;
            }
            float m = 0.0f;
            const uint32_t pm = P->pred[n];
#pragma unroll
            for (int u = 0; u < n; ++u)
                if (pm >> u & 1u) m = fmaxf(m, f[u]);
            f[n] = v.y + m;
        }
        const uint32_t pmw = P->pred[NH], pmx = P->pred[NH + 1], pmy = P->pred[NH + 2], pms = S.sinks;
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            if (pmw >> u & 1u) h.m = fmaxf(h.m, f[u]);
            if (pmx >> u & 1u) h.px = fmaxf(h.px, f[u]);
            if (pmy >> u & 1u) h.py = fmaxf(h.py, f[u]);
            if (pms >> u & 1u) h.s = fmaxf(h.s, f[u]);
        }
    }
    return h;
}

__device__ __forceinline__ float col_max(const LS float* f, uint32_t pm) {
    float v = 0.0f;
    while (pm) {
        const int u = __builtin_ctz(pm);
        pm &= pm - 1;
        v = fmaxf(v, f[u * WG]);
    }
    return v;
}

// Any number of nodes: the f_n in the thread's LDS column.
template <bool OBJ, class SV>
__device__ __forceinline__ SHead head_any(const SV& S, uint64_t x, int big) {
    PD P = S.P;
    const int nh = P->npre - 1;
    LS float* f = S.s_col + threadIdx.x;
    SHead h{OBJ ? 0.0f : 1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    const uint64_t b = x * (uint64_t)P->radix[nh];  // its first block
    for (int n = 0; n < nh; ++n) {
        const int e = n * S.rmax + (int)prefix_digit(P, n, b, big);
        const float2 v = S.ent(e);
        if (OBJ) {
            h.pc = h.pc + v.x;
            h.pd = h.pd + S.dem(e);
        } else {
            h.pc = h.pc * v.x;
        }
        f[n * WG] = v.y + col_max(f, P->pred[n]);
    }
    const uint32_t mask = (1u << nh) - 1u;
    h.m = col_max(f, P->pred[nh]);
    h.px = col_max(f, P->pred[nh + 1] & mask);
    h.py = col_max(f, P->pred[nh + 2] & mask);
    h.s = col_max(f, S.sinks);
    return h;
}

template <bool OBJ, class SV>
__device__ __forceinline__ SHead head_of(const SV& S, uint64_t x, int big) {
    switch (S.P->npre) {
        case 0:
        case 1: return head_nh<0, OBJ>(S, x, big);
        case 2: return head_nh<1, OBJ>(S, x, big);
        case 3: return head_nh<2, OBJ>(S, x, big);
        case 4: return head_nh<3, OBJ>(S, x, big);
        case 5: return head_nh<4, OBJ>(S, x, big);
        case 6: return head_nh<5, OBJ>(S, x, big);
        case 7: return head_nh<6, OBJ>(S, x, big);
        case 8: return head_nh<7, OBJ>(S, x, big);
        case 9: return head_nh<SOLVE_HEAD, OBJ>(S, x, big);
        default: return head_any<OBJ>(S, x, big);
    }
}

template <bool OBJ, class SV>
__device__ __forceinline__ SBlock block_of(const SV& S, const SHead& h, int g) {
    const float2 v = S.e3(0, g);
    const uint32_t fl = __float_as_uint(v.y + h.m);
    SBlock q;
    q.pc = OBJ ? h.pc + v.x : h.pc * v.x;
    q.pd = OBJ ? h.pd + S.d3(0, g) : 0.0f;
    q.px = fmaxf(h.px, __uint_as_float(fl & S.mx));
    q.py = fmaxf(h.py, __uint_as_float(fl & S.my));
    q.s = fmaxf(h.s, __uint_as_float(fl & S.ms));
    return q;
}

template <bool OBJ, class SV>
__device__ __forceinline__ SRow row_of(const SV& S, const SBlock& q, int ix) {
    const float2 v = S.e3(1, ix);
    const bool exy = S.P->edge_xy != 0;
    const float fx = v.y + q.px;
    SRow r;
    r.c = OBJ ? q.pc + v.x : q.pc * v.x;
    r.d = OBJ ? q.pd + S.d3(1, ix) : 0.0f;
    r.M = exy ? fmaxf(q.py, fx) : q.py;
    r.S2 = exy ? q.s : fmaxf(q.s, fx);
    return r;
}

// Can some plan of the head (block, row) be a candidate?  Never false for one
// that holds a candidate (see build_tables).  A factor is bounded by its
// node's largest: fp32 products are monotone.
template <int MODE, class SV>
__device__ __forceinline__ bool head_test(const SV& S, const SHead& h) {
    if (MODE == SV_OBJ) {
        const uint32_t o = S.off((h.pd + S.dw) * BIN_HEAD);
        return fmaf(S.nl, h.px, h.pc) >= tab(S.t_headx, o) && fmaf(S.nl, h.py, h.pc) >= tab(S.t_heady, o) &&
               fmaf(S.nl, h.m, h.pc) >= tab(S.t_head, o);
    }
    const float c = h.pc * S.aw, cx = c * S.ax;
    const float tx = tab(S.t_blk, S.off((h.px + S.dxy) * BIN_BLK));
    const float ty = tab(S.t_row, S.off((h.py + S.dy) * BIN_ROW));
    const float tw = tab(S.t_head, S.off((h.m + S.dw) * BIN_HEAD));
    bool in = h.pc >= tw && c >= tx && cx >= ty;
    if (S.sinks) in = in && cx * S.ay >= tab(S.t_bin, S.off(h.s));
    return in;
}

template <int MODE, class SV>
__device__ __forceinline__ bool block_test(const SV& S, const SBlock& q) {
    if (MODE == SV_OBJ) {
        const uint32_t o = S.off((q.pd + S.dxy) * BIN_BLK);
        return fmaf(S.nl, q.px, q.pc) >= tab(S.t_blk, o) && fmaf(S.nl, q.py, q.pc) >= tab(S.t_blky, o);
    }
    const float cx = q.pc * S.ax;
    return q.pc >= tab(S.t_blk, S.off((q.px + S.dxy) * BIN_BLK)) &&
           cx >= tab(S.t_row, S.off((q.py + S.dy) * BIN_ROW)) && cx * S.ay >= tab(S.t_bin, S.off(q.s));
}

template <int MODE, class SV>
__device__ __forceinline__ bool row_test(const SV& S, const SRow& r) {
    if (MODE == SV_OBJ) return fmaf(S.nl, r.M, r.c) >= tab(S.t_row, S.off((r.d + S.dy) * BIN_ROW));
    return r.c >= tab(S.t_row, S.off((r.M + S.dy) * BIN_ROW)) && r.c * S.ay >= tab(S.t_bin, S.off(r.S2));
}

// Append to the source's candidate list: the workgroup's count is n (LDS), the
// source's, where it has several, in device memory.  A list that overflowed
// takes no more: a source may have 2^40 candidates, and a count of them all
// would wrap.  (Past the capacity, at most 2^26, come at most the threads that
// had found room: one a thread of the source's at most 2^10 workgroups.)
__device__ __forceinline__ void solve_append(JD J, LS uint32_t* n, LS Cand* own, uint64_t index, float c, float cp) {
    if (*(volatile LS uint32_t*)n > J->cap) return;
    uint32_t slot = __hip_atomic_fetch_add(n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (J->nwg > 1) {
        slot = atomicAdd(J->wk, 1u);
        if (slot >= J->cap)
            __hip_atomic_fetch_max(n, J->cap + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (slot < (uint32_t)SOLVE_OWN) {  // (read back from here by a source's only workgroup)
        own[slot].index = index;
        own[slot].corr = c;
        own[slot].cp = cp;
    }
    if (slot < J->cap) {
        Cand* d = J->cand + slot;
        d->index = index;
        d->corr = c;
        d->cp = cp;
    }
}

__device__ __forceinline__ void raise_seed(LS uint32_t* seed, uint32_t key) {
    if (key > *(volatile LS uint32_t*)seed)
        __hip_atomic_fetch_max(seed, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Exact test of plan j of row (block b, ix); a candidate is appended, a
// certainly feasible one raises its levels' seeds.  Per-backend pressure: at
// the level kk of the pass.
template <int MODE, class SV>
__device__ __forceinline__ void plan_exact(const SV& S, uint64_t b, int ix, const SRow& r, int j, int kk,
                                           LS uint32_t* s_seed, LS uint32_t* n, LS Cand* own) {
    PD P = S.P;
    JD J = S.J;
    const uint64_t idx = (b * (uint64_t)P->rx + (uint64_t)ix) * (uint64_t)P->ry + (uint64_t)j;
    if (!(idx - J->begin < J->count)) return;
    const float2 v = S.e3(2, j);
    const float T = fmaxf(v.y + r.M, r.S2);
    bool cand = false;
    if (MODE == SV_OBJ) {
        const float G = fmaf(S.nl, T, r.c + v.x);
        const float D = r.d + S.d3(2, j);
        for (int k = 0; k < P->k; ++k)
            if (fma(-P->m64[k], (double)D, (double)G) >= (double)S.s_thr[k]) {
                cand = true;
                raise_seed(s_seed + k, fkey(obj_estimate(P->m32[k], D, G)));
            }
        if (cand) solve_append(J, n, own, idx, G, D);
        return;
    }
    const float c = r.c * v.x;
    if (MODE == SV_CLASS) {
        if (T <= P->ghi && c >= S.s_thr[kk]) {
            if (T <= P->glo) raise_seed(s_seed + kk, __float_as_uint(c) + 1u);
            // No CP is kept: its only use was a seed for other levels, and the
            // recurrence column it took (a float per node and thread) cost
            // occupancy: 1,000 mixed requests 337 us with it, 251 without.
            // The level takes its place, as a NaN, which passes no test of a CP.
            solve_append(J, n, own, idx, c, __uint_as_float(CAND_LEVEL | (uint32_t)kk));
        }
        return;
    }
    for (int k = 0; k < P->k; ++k)
        if (T <= S.s_hi[k] && c >= S.s_thr[k]) {
            cand = true;
            if (T <= S.s_lo[k]) raise_seed(s_seed + k, __float_as_uint(c) + 1u);
        }
    if (cand) solve_append(J, n, own, idx, c, T);
}

// fp64 corr, CP and demand (objective: U, T, D) of candidate ids, as cert_eval
// of the certification kernel: the definition's operations in node order.
template <bool OBJ>
__device__ __forceinline__ void pair_eval(PD P, const uint8_t* ids, double* f, int st, int k, double& x, double& cp,
                                          double& d) {
    const int N = P->n, R = P->rmax;
    const CS double* a64 = cs(P->a64);
    const CS double* d64 = cs(P->dem64);
    const CS double* lat = cs(P->lat64) + (OBJ ? (size_t)0 : (size_t)k * N * R);
    x = OBJ ? 0.0 : 1.0;
    cp = 0.0;
    d = 0.0;
    for (int n0 = 0; n0 < N; n0 += 8) {
        double va[8], vl[8], vd[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {  // the loads of eight nodes in flight together
            const int n = n0 + j;
            const int e = n < N ? n * R + ids[n * st] : 0;
            va[j] = a64[e];
            vl[j] = lat[e];
            vd[j] = d64[e];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = n0 + j;
            if (n < N) {
                if (!OBJ) {
                    x = x * va[j];
                    d = d + vd[j];
                } else if (P->llm >> n & 1u) {
                    x = x + va[j];
                    d = d + vd[j];
                }
                double m = 0.0;
                uint32_t pm = P->pred[n];
                while (pm) {
                    const int u = __builtin_ctz(pm);
                    pm &= pm - 1;
                    const double fu = f[u * st];
                    if (fu > m) m = fu;
                }
                const double fn = vl[j] + m;
                f[n * st] = fn;
                if ((P->sinks >> n & 1u) && fn > cp) cp = fn;
            }
        }
    }
}

// Grid (workgroups per source, sources).  A source's heads are spread over its
// J->nwg workgroups; each takes an evenly spaced share, after seeding the
// thresholds (every workgroup of a source the same) and building the tables.
// The workgroup that ends last certifies the candidates in fp64 and writes
// the choices.
// Bound by latency: a workgroup is one serial chain (seeding, three folds,
// heads, unfolding, the 64-bit recurrences) of dependent reads.  Per CU and
// cycle it issues 0.36 vector instructions on 4,096 six-node requests (1 is the
// rate of the four SIMDs), 0.10 and 0.18 on single ranges of 4.3e8 and 4.3e9
// plans, and 0.05, 0.01 and 0.02 LDS instructions; HBM is idle.  us a pass, the
// separate sampling, table, plan-by-plan sweep and certification launches and
// this one, timed in turn: 4,096 six-node requests 1,563 / 211, their objective
// 1,106 / 163, 512 mixed 432 / 116, 1,000 under per-backend pressure 501 / 154,
// one fork-join of 4.3e8 plans 111 / 42, one layered space of 4.3e9 717 / 56.
// Five waves per SIMD: with one more register group the batches, whose
// workgroups wait on LDS chains most of the time, ran 9 % longer; at six (80
// registers, spills) small sources run 3 to 10 % longer.
template <int MODE>
__global__ void __launch_bounds__(WG, 5) k_solve(const JobDev* __restrict__ jobs, const LaunchSizes sizes, int ent,
                                              int rmax_all, int nlat, int ncol, int nf, int lds) {
    constexpr bool OBJ = MODE == SV_OBJ;
    constexpr int NB = OBJ ? SOLVE_BINS_OBJ : SOLVE_BINS, Q = NB / WG;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    __shared__ uint32_t s_tab[OBJ ? 8 : 4][NB];
    __shared__ float s_thr[KMAX], s_lo[KMAX], s_hi[KMAX];
    __shared__ uint32_t s_seed[KMAX];
    __shared__ uint8_t s_b0[NMAX], s_b1[NMAX];
    __shared__ SeedBox s_box[SEED_BOXES];
    __shared__ uint32_t s_cnt[WG / 64];
    __shared__ Cand s_own[SOLVE_OWN];
    __shared__ uint32_t s_nh, s_nb, s_nr, s_nc, s_flag, s_rows;
    if (gridDim.y <= (unsigned)LAUNCH_SIZES && blockIdx.x >= sizes.n[blockIdx.y]) return;
    JD J = cs(jobs + blockIdx.y);
    PD P = cs(J->prob);
    const uint32_t nwg = (uint32_t)J->nwg;
    if (blockIdx.x >= nwg) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int K = P->k, N = P->n, R = P->rmax, rx = P->rx, ry = P->ry, npre = P->npre;
    const int rw = npre > 0 ? P->radix[npre - 1] : 1;
    const int big = J->big;
    const SolveLds L = solve_lds(ent, rmax_all, nlat, ncol, nf, OBJ, MODE == SV_CLASS);

    // ---- the source's tables in LDS
    SolveT<NB> S;
    S.P = P;
    S.J = J;
    S.stg = N * R <= ent;
    S.s_at = (const LS float2*)(s_dyn + L.at);
    S.s_dm = (const LS float*)(s_dyn + L.dm);
    S.s_e = (const LS float2*)(s_dyn + L.e3);
    S.s_q = (const LS float2*)(s_dyn + L.q3);
    S.s_d = (const LS float*)(s_dyn + L.d3);
    S.s_col = (LS float*)(s_dyn + L.col);
    S.lat = nullptr;
    S.t_bin = (const LS uint32_t*)s_tab[0];
    S.t_row = (const LS uint32_t*)s_tab[1];
    S.t_blk = (const LS uint32_t*)s_tab[2];
    S.t_head = (const LS uint32_t*)s_tab[3];
    S.t_rowu = (const LS uint32_t*)s_tab[OBJ ? 4 : 0];
    S.t_blky = (const LS uint32_t*)s_tab[OBJ ? 5 : 0];
    S.t_headx = (const LS uint32_t*)s_tab[OBJ ? 6 : 0];
    S.t_heady = (const LS uint32_t*)s_tab[OBJ ? 7 : 0];
    S.s_thr = (const LS float*)s_thr;
    S.s_lo = (const LS float*)s_lo;
    S.s_hi = (const LS float*)s_hi;
    S.rmax = R;
    int bsh = P->wsh;
    S.sh = bsh - 2;
    S.lo = __uint_as_float(P->cp_lo_bits);
    S.top = INFINITY;
    S.dy = P->dmin_y;
    S.dxy = P->dmin_xy;
    S.dw = P->dmin_w;
    S.aw = P->aw_max;
    S.ax = P->ax_max;
    S.ay = P->ay_max;
    S.nl = OBJ ? -P->lam_l : 0.0f;
    S.mx = P->w_feeds & 1u ? ~0u : 0u;
    S.my = P->w_feeds & 2u ? ~0u : 0u;
    S.ms = P->w_feeds & 4u ? ~0u : 0u;
    S.sinks = npre > 1 ? P->pre_sinks & ((1u << (npre - 1)) - 1u) : 0u;
    if (S.stg)
        for (int i = tid; i < N * R; i += WG) {
            const float2 v = cs(P->at)[i];
            ((float2*)(s_dyn + L.at))[i] = v;
            if (OBJ) ((float*)(s_dyn + L.dm))[i] = cs(P->dem)[i];
            ((float2*)(s_dyn + L.nt))[i] = make_float2(OBJ ? P->u_top - v.x : -__logf(v.x), v.y);
        }
    const LS float* s_lat = MODE == SV_CLASS && K * N * R <= nlat ? (const LS float*)(s_dyn + L.lat) : nullptr;
    if (s_lat)
        for (int i = tid; i < K * N * R; i += WG) ((float*)(s_dyn + L.lat))[i] = cs(P->lat)[i];
    auto class_lat = [&](int e) __attribute__((always_inline)) { return s_lat ? s_lat[e] : cs(P->lat)[e]; };
    // w, x and y: entries (a missing node: one neutral entry) and reciprocals
    // of the factors (objective: what an implementation adds to U - lambda_l
    // (path), with its own duration on the path and without)
    for (int i = tid; i < 3 * R; i += WG) {
        const int row = i / R, j = i - row * R, n = N - 3 + row;
        float2 v = make_float2(OBJ ? 0.0f : 1.0f, 0.0f);
        float d = 0.0f;
        if (n >= 0) {
            v = cs(P->at)[n * R + j];
            if (OBJ) d = cs(P->dem)[n * R + j];
        }
        ((float2*)(s_dyn + L.e3))[i] = v;
        float2 q = make_float2(down_reciprocal(v.x), 0.0f);
        if (OBJ) {
            q.x = raise_by((double)v.x - P->lam_l64 * (double)v.y, P->eshift);
            q.y = raise_by((double)v.x, P->eshift);
            ((float*)(s_dyn + L.d3))[i] = d;
        }
        ((float2*)(s_dyn + L.q3))[i] = q;
    }
    if (tid < K) {
        s_lo[tid] = P->lo[tid];
        s_hi[tid] = P->hi[tid];
        uint32_t e = 0;
        if (J->seeded) e = J->scert[tid * NSLOT];
        s_seed[tid] = e;
    }
    if (tid < N) {  // digits of the source's first and last plan
        s_b0[tid] = J->dig0[tid];
        s_b1[tid] = J->dig1[tid];
    }
    if (tid < SEED_BOXES) {
        s_box[tid].end = J->box[tid].end;
        s_box[tid].n = J->box[tid].n;
        s_box[tid].lo = J->box[tid].lo;
        s_box[tid].hi = J->box[tid].hi;
    }
    if (tid == 0) {
        s_nh = 0;
        s_nb = 0;
        s_nr = 0;
        s_nc = 0;
        s_rows = 0;
    }
    LS uint32_t* ncand = (LS uint32_t*)&s_nc;
    LS uint32_t* seeds = (LS uint32_t*)s_seed;
    uint64_t* hx = (uint64_t*)(s_dyn + L.hx);
    float* hv = (float*)(s_dyn + L.hv);
    uint32_t* bq = (uint32_t*)(s_dyn + L.bq);
    uint32_t* rq = (uint32_t*)(s_dyn + L.rq);
    __syncthreads();

    auto set_thr = [&]() __attribute__((always_inline)) {
        if (tid < K) {
            const uint32_t e = s_seed[tid];
            float t = -INFINITY;
            if (e) t = OBJ ? obj_threshold(fkey_value(e), P->err2[tid]) : cand_threshold(__uint_as_float(e - 1u), N);
            s_thr[tid] = t;
        }
    };
    // Thresholds from the seeds, then the folded tables, Q bins per thread.
    // Bin b's entries hold for every value v of the quantity indexed whose
    // fp32 (v + d) c (d: the least that the folded nodes add) lies in b: they are
    // formed at a value `least` not above any such v, with the sweep's own fp32
    // operations, which are monotone; the CP (D) bins they read then lie at or
    // below those of the plans, and bin thresholds do not fall with the bin.
    // Corr: a factor a is divided out by div_threshold.  Objective: G and the
    // folded sums take at most four roundings between two levels, bounded by
    // eshift (part of the offsets, see lower_by).  256 bins, one a thread:
    // 1,024 let no fewer rows through and took longer to build.
    int kk = 0;  // per-backend pressure: the level of the pass
    auto build_tables = [&]() __attribute__((always_inline)) {
        set_thr();
        __syncthreads();
        // bin i covers fp32 patterns [B << bsh, (B + 1) << bsh), B = i (mod NB)
        const uint32_t blo = __float_as_uint(S.lo) >> bsh;
        bool first[Q];
        float low[Q], g[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t Bn = blo + (((uint32_t)(tid + q * WG) - blo) & (uint32_t)(NB - 1));
            first[q] = Bn == blo;
            low[q] = first[q] ? S.lo : __uint_as_float(Bn << bsh);
            g[q] = INFINITY;
        }
        if (MODE == SV_CLASS) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (P->ghi >= low[q]) g[q] = s_thr[kk];
        } else {
            for (int k = 0; k < K; ++k) {
                const float t = s_thr[k];
                const float h = OBJ ? 0.0f : s_hi[k];
                const double m = OBJ ? P->m64[k] : 0.0;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (OBJ)
                        g[q] = fminf(g[q], obj_bin_threshold(t, m, low[q]));
                    else
                        g[q] = fminf(g[q], h >= low[q] ? t : INFINITY);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) s_tab[0][tid + q * WG] = __float_as_uint(g[q]);
        __syncthreads();
        // no value v of the bin with fp32(fp32(v + d) c) >= low is below this
        auto least = [&](int q, float d, float c) __attribute__((always_inline)) {
            const double v = (double)low[q] * (1.0 + (1.0 - (double)c) - 0x1p-22) - (double)d;
            return !first[q] && v > 0.0 ? __double2float_rd(v) : 0.0f;  // (the first bin: any value below the bins)
        };
        const bool exy = P->edge_xy != 0;
        float at[Q], r0[Q], r1[Q], r2[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            at[q] = least(q, S.dy, BIN_ROW);
            r0[q] = r1[q] = INFINITY;
        }
#pragma unroll 4
        for (int j = 0; j < ry; ++j) {
            const float2 c = S.q3(2, j);
            const float e = OBJ ? S.d3(2, j) : S.e3(2, j).y;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float t = tab(S.t_bin, S.off(at[q] + e));
                if (OBJ) {
                    r0[q] = fminf(r0[q], lower_by(t, c.x));
                    r1[q] = fminf(r1[q], lower_by(t, c.y));
                } else {
                    r0[q] = fminf(r0[q], div_threshold(t, c.x));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            s_tab[1][tid + q * WG] = __float_as_uint(r0[q]);
            if (OBJ) s_tab[OBJ ? 4 : 0][tid + q * WG] = __float_as_uint(r1[q]);
        }
        __syncthreads();
        const float ray = down_reciprocal(S.ay);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            at[q] = least(q, S.dxy, BIN_BLK);
            r0[q] = r1[q] = INFINITY;
        }
        auto fold_x = [&](auto&& bound) __attribute__((always_inline)) {
#pragma unroll 4
            for (int i = 0; i < rx; ++i) {
                const float2 c = S.q3(1, i);
                const float e = OBJ ? S.d3(1, i) : S.e3(1, i).y;
#pragma unroll
                for (int q = 0; q < Q; ++q) bound(q, at[q] + e, c);
            }
        };
        if (OBJ) {
            const LS uint32_t* t_x = exy ? S.t_row : S.t_rowu;  // x off y's paths: its own path bounds T
            fold_x([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                const uint32_t o = S.off((p + S.dy) * BIN_ROW);
                r1[q] = fminf(r1[q], lower_by(tab(S.t_row, o), c.y));
                r0[q] = fminf(r0[q], lower_by(tab(t_x, o), c.x));
            });
        } else if (exy) {
            fold_x([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                r0[q] = fminf(r0[q], div_threshold(tab(S.t_row, S.off((p + S.dy) * BIN_ROW)), c.x));
            });
        } else {
            fold_x([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                r0[q] = fminf(r0[q], div_threshold(div_threshold(tab(S.t_bin, S.off(p)), ray), c.x));
            });
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            s_tab[2][tid + q * WG] = __float_as_uint(r0[q]);
            if (OBJ) s_tab[OBJ ? 5 : 0][tid + q * WG] = __float_as_uint(r1[q]);
        }
        __syncthreads();
        const float rax = down_reciprocal(S.ax);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            at[q] = least(q, S.dw, BIN_HEAD);
            r0[q] = r1[q] = r2[q] = INFINITY;
        }
        // w's bound by what it feeds, the loop per case (a branch inside keeps the
        // LDS reads of its iterations apart)
        auto fold_w = [&](auto&& bound) __attribute__((always_inline)) {
#pragma unroll 4
            for (int i = 0; i < rw; ++i) {
                const float2 c = S.q3(0, i);
                const float e = OBJ ? S.d3(0, i) : S.e3(0, i).y;
#pragma unroll
                for (int q = 0; q < Q; ++q) bound(q, at[q] + e, c);
            }
        };
        if (OBJ) {
            const bool mx = S.mx != 0, my = S.my != 0;
            fold_w([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                const uint32_t o = S.off((p + S.dxy) * BIN_BLK);
                const float tx = tab(S.t_blk, o), ty = tab(S.t_blky, o);
                r1[q] = fminf(r1[q], lower_by(tx, c.y));
                r2[q] = fminf(r2[q], lower_by(ty, c.y));
                // w on a path to x or to y; a sink: no bound
                r0[q] = fminf(r0[q], fmaxf(mx ? lower_by(tx, c.x) : -INFINITY, my ? lower_by(ty, c.x) : -INFINITY));
            });
        } else {
            auto tx = [&](float p) __attribute__((always_inline)) { return tab(S.t_blk, S.off((p + S.dxy) * BIN_BLK)); };
            auto ty = [&](float p) __attribute__((always_inline)) {
                return div_threshold(tab(S.t_row, S.off((p + S.dy) * BIN_ROW)), rax);
            };
            if (S.mx && S.my)
                fold_w([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                    r0[q] = fminf(r0[q], div_threshold(fmaxf(tx(p), ty(p)), c.x));
                });
            else if (S.mx)
                fold_w([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                    r0[q] = fminf(r0[q], div_threshold(tx(p), c.x));
                });
            else if (S.my)
                fold_w([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                    r0[q] = fminf(r0[q], div_threshold(ty(p), c.x));
                });
            else if (S.ms)
                fold_w([&](int q, float p, const float2& c) __attribute__((always_inline)) {
                    const float t = div_threshold(div_threshold(tab(S.t_bin, S.off(p)), ray), rax);
                    r0[q] = fminf(r0[q], div_threshold(t, c.x));
                });
            else  // no such node
                for (int q = 0; q < Q; ++q) r0[q] = -INFINITY;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            s_tab[3][tid + q * WG] = __float_as_uint(r0[q]);
            if (OBJ) {
                s_tab[OBJ ? 6 : 0][tid + q * WG] = __float_as_uint(r1[q]);
                s_tab[OBJ ? 7 : 0][tid + q * WG] = __float_as_uint(r2[q]);
            }
        }
        __syncthreads();
    };

    // ---- unfolding of what passed, by every thread
    auto load_head = [&](uint32_t i) __attribute__((always_inline)) {
        SHead h;
        h.pc = hv[i];
        h.m = hv[SOLVE_Q + i];
        h.px = hv[2 * SOLVE_Q + i];
        h.py = hv[3 * SOLVE_Q + i];
        h.s = hv[4 * SOLVE_Q + i];
        h.pd = OBJ ? hv[5 * SOLVE_Q + i] : 0.0f;
        return h;
    };
    // queue entries: head slot << 16 | w << 8 | x
    auto drain_rows = [&]() __attribute__((always_inline)) {
        const uint32_t n = s_nr;
        for (uint32_t p = tid; p < n * (uint32_t)ry; p += WG) {
            const uint32_t i = p / (uint32_t)ry, j = p - i * (uint32_t)ry;
            const uint32_t e = rq[i], slot = e >> 16;
            const int g = (int)(e >> 8 & 255u), ix = (int)(e & 255u);
            const SRow r = row_of<OBJ>(S, block_of<OBJ>(S, load_head(slot), g), ix);
            plan_exact<MODE>(S, hx[slot] * (uint64_t)rw + (uint64_t)g, ix, r, (int)j, kk, seeds, ncand,
                             (LS Cand*)s_own);
        }
        __syncthreads();
        if (tid == 0) {
            s_nr = 0;
            s_rows += n;
        }
        __syncthreads();
    };
    auto drain_blocks = [&]() __attribute__((always_inline)) {
        const uint32_t n = s_nb * (uint32_t)rx;
        for (uint32_t p0 = 0; p0 < n; p0 += WG) {
            const uint32_t p = p0 + tid;
            if (p < n) {
                const uint32_t i = p / (uint32_t)rx, ix = p - i * (uint32_t)rx;
                const uint32_t e = bq[i];
                const SRow r =
                    row_of<OBJ>(S, block_of<OBJ>(S, load_head(e >> 16), (int)(e >> 8 & 255u)), (int)ix);
                if (row_test<MODE>(S, r)) rq[atomicAdd(&s_nr, 1u)] = e | ix;
            }
            __syncthreads();
            const bool go = s_nr > (uint32_t)(SOLVE_Q - WG) || (p0 + WG >= n && s_nr > 0);
            __syncthreads();
            if (go) drain_rows();
        }
        if (tid == 0) s_nb = 0;
        __syncthreads();
    };
    // The parked heads, WG (head, w) pairs at a time.  Where many rows come
    // through, the tables are rebuilt on the seeds they raised before the next
    // pairs (heads are parked in a fixed order, and what a round leaves does
    // not depend on the order of its work, so a call repeats exactly).
    auto drain = [&]() __attribute__((always_inline)) {
        const uint32_t n = s_nh * (uint32_t)rw;
        for (uint32_t p0 = 0; p0 < n; p0 += WG) {
            const uint32_t p = p0 + tid;
            if (p < n) {
                const uint32_t i = p / (uint32_t)rw, g = p - i * (uint32_t)rw;
                if (block_test<MODE>(S, block_of<OBJ>(S, load_head(i), (int)g)))
                    bq[atomicAdd(&s_nb, 1u)] = i << 16 | g << 8;
            }
            __syncthreads();
            const bool any = s_nb > 0;
            __syncthreads();
            if (any) {
                drain_blocks();
                set_thr();  // (here, not after each round of rows, whose make-up varies)
            }
            if (s_rows > (uint32_t)SOLVE_REBUILD) {
                __syncthreads();
                if (tid == 0) s_rows = 0;
                build_tables();
            }
        }
        if (tid == 0) s_nh = 0;
        __syncthreads();
    };

    // ---- seeds: one constructed plan per thread.  A node takes the
    // implementation that maximises ln a - lambda phi tau (objective: u -
    // phi lambda_l tau - m_k d), phi the share of a unit flow from the sources
    // to the sinks that passes through the node (split evenly at forks: a
    // dual solution of the longest path, so that parallel branches share the
    // weight), times a random factor in all but the first set of threads; the
    // threads run through lambda (and the levels, where they differ).  Such
    // plans lie on or next to the front of corr against CP: on the recipes'
    // workloads the best of them is the level's optimum more often than not,
    // and 0 to 3 % below it otherwise (256 sampled rows of plans: 2 to 13 %).
    // A range that is not the whole space is constructed in by parts, whole
    // subtrees of it (seed_boxes), which the sets of threads take in turn.
    // Per-backend pressure: at most SEED_LEVELS levels share the threads (with
    // all of 32 the 8 plans a level had were 2.7 % below its optimum in the
    // mean, now 0.3 %), and a plan serves the levels about its own as well.
    const int rounds = MODE == SV_CLASS ? (K + SEED_LEVELS - 1) / SEED_LEVELS : 1;
    for (int rd = 0; rd < rounds; ++rd) {
        const int lpr = MODE == SV_LEVEL ? 1 : (K + rounds - 1) / rounds, per = WG / lpr;  // levels, plans of each
        const int gl = min(tid / per, lpr - 1);
        const int sk = min(rd * lpr + gl, K - 1);
        const int v = tid - gl * per;
        const int nl = OBJ ? 4 : (per >= 32 ? (MODE == SV_LEVEL ? 32 : 16) : per);  // values of lambda
        const int q = v % nl, set = v / nl;
        float lam;
        if (OBJ)
            lam = P->lam_l * (q == 0 ? 1.0f : q == 1 ? 0.5f : q == 2 ? 1.5f : 0.25f);
        else if (q == nl - 1)
            lam = 1e30f;  // about every node's fastest (ids within 2^-15 of it tie): a level of
                          // few feasible plans may stay without a seed all the same (threshold -inf)
        else
            lam = P->lam0 * exp2f((MODE == SV_CLASS ? -13.0f : -7.0f) +
                                  (MODE == SV_CLASS ? 20.0f : 14.0f) * (float)q / (float)max(nl - 2, 1));
        const float mk = OBJ ? P->m32[sk] : 0.0f;
        LS float* f = (LS float*)(s_dyn + L.sc) + tid;
        const LS float2* nt = (const LS float2*)(s_dyn + L.nt);
        LS uint8_t* ids = (LS uint8_t*)(s_dyn + L.id) + tid;
        const bool whole = J->whole != 0;
        const int nbox = J->nbox;
        const SeedBox box = s_box[(MODE == SV_CLASS ? set + sk : set) % nbox];  // (few sets a level)
        const uint8_t* ends = box.end ? s_b1 : s_b0;
        float c = OBJ ? 0.0f : 1.0f, cp = 0.0f, D = 0.0f;
        const uint32_t sinks = P->sinks;
        for (int n = 0; n < N; ++n) {
            float w = lam * P->flow[n];
            const int r = P->radix[n], e0 = n * R, lat = MODE == SV_CLASS ? sk * N * R + e0 : 0;
            const uint32_t pm = P->pred[n];
            if (set >= nbox) {
                const uint32_t hash = ((uint32_t)(rd * WG + tid) * 32u + (uint32_t)n + 1u) * 0x9E3779B1u;
                w *= __builtin_amdgcn_exp2f((float)(hash >> 8) * (3.0f * 0x1p-24f) - 1.5f);
            }
            // the cost w tau - ln a (objective: w tau + m_k d + u_max - u) is not
            // negative, so its pattern orders as it does; the last eight bits
            // carry the id, and the least key is the choice
            uint32_t key = ~0u;
            int i0 = 0, span = 255;  // ids i0 .. i0 + span
            if (!whole && n <= (int)box.n) {
                i0 = n < (int)box.n ? (int)ends[n] : (int)box.lo;
                span = n < (int)box.n ? 0 : (int)box.hi - i0;
            }
            if (S.stg) {
                const LS float2* q = nt + e0;
                auto cost = [&](int i) __attribute__((always_inline)) {
                    float y = fmaf(w, MODE == SV_CLASS ? class_lat(lat + i) : q[i].y, q[i].x);
                    if (OBJ) y = fmaf(mk, S.s_dm[e0 + i], y);
                    return (__float_as_uint(y) & 0x7fffff00u) | (uint32_t)i;
                };
                if (whole) {
#pragma unroll 6
                    for (int i = 0; i < r; ++i) key = min(key, cost(i));
                } else {
#pragma unroll 6
                    for (int i = 0; i < r; ++i)
                        key = min(key, cost(i) | ((uint32_t)(i - i0) <= (uint32_t)span ? 0u : 0x80000000u));
                }
            } else {
                for (int i = i0; i <= min(i0 + span, r - 1); ++i) {
                    const float2 x = S.ent(e0 + i);
                    float y = fmaf(w, MODE == SV_CLASS ? class_lat(lat + i) : x.y, OBJ ? P->u_top - x.x : -__logf(x.x));
                    if (OBJ) y = fmaf(mk, S.dem(e0 + i), y);
                    key = min(key, (__float_as_uint(y) & 0x7fffff00u) | (uint32_t)i);
                }
            }
            const int e = e0 + (int)(key & 255u);
            const float2 x = S.ent(e);
            const float t = MODE == SV_CLASS ? class_lat(lat + (int)(key & 255u)) : x.y;
            c = OBJ ? c + x.x : c * x.x;
            if (OBJ) D = D + S.dem(e);
            const float fn = t + col_max(f, pm);
            f[n * WG] = fn;
            if (sinks >> n & 1u) cp = fmaxf(cp, fn);
            if (MODE == SV_CLASS) ids[n * WG] = (uint8_t)key;
        }
        // the fp32 values are the sweep's own (the same operations in node order)
        if (MODE == SV_CLASS) {  // at the level it was made for and at those about it
            if (cp <= P->glo) raise_seed(seeds + sk, __float_as_uint(c) + 1u);
            for (int k = max(sk - SEED_NEAR, 0); k <= min(sk + SEED_NEAR, K - 1); ++k) {
                if (k == sk || *(volatile LS uint32_t*)(seeds + k) > __float_as_uint(c)) continue;
                float cpk = 0.0f;
                for (int n = 0; n < N; ++n) {
                    const float fn = class_lat((k * N + n) * R + (int)ids[n * WG]) + col_max(f, P->pred[n]);
                    f[n * WG] = fn;
                    if (sinks >> n & 1u) cpk = fmaxf(cpk, fn);
                }
                if (cpk <= P->glo) raise_seed(seeds + k, __float_as_uint(c) + 1u);
            }
            continue;
        }
        const float G = OBJ ? fmaf(S.nl, cp, c) : 0.0f;
        for (int k = 0; k < K; ++k) {
            uint32_t e = 0;
            if (OBJ)
                e = fkey(obj_estimate(P->m32[k], D, G));
            else if (cp <= s_lo[k])
                e = __float_as_uint(c) + 1u;
            e = wave_max_u32(e);
            if (lane == 0 && e) atomicMax(s_seed + k, e);
        }
    }
    __syncthreads();

    // ---- the sweep (per-backend pressure: of each level)
    const uint64_t units = J->units;
    const uint64_t threads = (uint64_t)nwg * WG;
    const uint64_t steps = (units + threads - 1) / threads;
    const uint64_t gid = (uint64_t)tid * nwg + blockIdx.x;
    uint32_t swept = 0, skipped = 0;
    for (kk = 0; kk < (MODE == SV_CLASS ? K : 1); ++kk) {
        if (MODE == SV_CLASS) {
            // a level whose durations are nowhere below those of a level swept
            // before, and whose threshold is no lower than that level's last,
            // has its candidates among that level's; a level above whose bound every CP lies has none
            set_thr();
            __syncthreads();
            bool skip = P->cplo[kk] > P->ghi;
            uint32_t m = swept & P->nest[kk];
            while (m) {
                const int j = __builtin_ctz(m);
                m &= m - 1;
                skip = skip || s_thr[j] <= s_thr[kk];
            }
            if (skip) skipped |= 1u << kk;
            if (skip) continue;
            swept |= 1u << kk;
            // the level's durations in the tables, and its bins: [cplo, ghi]
            S.lat = cs(P->lat) + (size_t)kk * N * R;
            if (S.stg)
                for (int i = tid; i < N * R; i += WG) ((float2*)(s_dyn + L.at))[i].y = S.lat[i];
            for (int i = tid; i < 3 * R; i += WG) {
                const int n = N - 3 + i / R;
                if (n >= 0) ((float2*)(s_dyn + L.e3))[i].y = S.lat[(N - 3) * R + i];
            }
            S.lo = P->cplo[kk];
            bsh = P->csh[kk];
            S.sh = bsh - 2;
            S.top = __uint_as_float(min(((__float_as_uint(P->ghi) >> bsh) + 1u) << bsh, 0x7f800000u));
            S.dy = P->cdmin[kk][0];
            S.dxy = P->cdmin[kk][1];
            S.dw = P->cdmin[kk][2];
            __syncthreads();
        }
        build_tables();
        for (uint64_t it = 0; it < steps; ++it) {
            const uint64_t u = it * threads + gid;
            const bool live = u < units;
            const uint64_t x = J->ublk0 + (live ? u : 0);
            const SHead h = head_of<OBJ>(S, x, big);
            const bool hit = live && head_test<MODE>(S, h);
            const uint64_t m = __ballot(hit);
            if (lane == 0) s_cnt[tid >> 6] = (uint32_t)__popcll(m);
            __syncthreads();
            uint32_t o = s_nh, all = s_nh;
            for (int v = 0; v < WG / 64; ++v) {
                if (v < tid >> 6) o += s_cnt[v];
                all += s_cnt[v];
            }
            if (hit) {
                o += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                hx[o] = x;
                hv[o] = h.pc;
                hv[SOLVE_Q + o] = h.m;
                hv[2 * SOLVE_Q + o] = h.px;
                hv[3 * SOLVE_Q + o] = h.py;
                hv[4 * SOLVE_Q + o] = h.s;
                if (OBJ) hv[5 * SOLVE_Q + o] = h.pd;
            }
            __syncthreads();
            if (tid == 0) s_nh = all;
            __syncthreads();
            if (all > (uint32_t)(SOLVE_Q - WG) || (it + 1 == steps && all > 0)) drain();
        }
    }

    // ---- the candidates of every workgroup of the source, then the choices
    bool last = true;
    if (nwg > 1) {
        // seeds go to slot 1 of each level (slot 0 holds those given to the
        // launch); counters in two stages, same-address atomics serialise.  A
        // workgroup without a candidate has written nothing, and its seeds are
        // every workgroup's, so it publishes and fences nothing.
        if (s_nc) {
            if (tid < K && s_seed[tid]) atomicMax(J->scert + tid * NSLOT + 1, s_seed[tid]);
            if (MODE == SV_CLASS && tid == 0) atomicOr(J->wk + 2, skipped);
            __threadfence();
        }
        __syncthreads();
        if (tid == 0) {
            const uint32_t grp = blockIdx.x % 16u;
            const uint32_t members = (nwg - grp + 15u) / 16u;
            uint32_t f = 0;
            if (atomicAdd(J->wk + 16 + grp, 1u) + 1u == members) {
                __threadfence();
                f = atomicAdd(J->wk + 1, 1u) + 1u == min(nwg, 16u) ? 1u : 0u;
            }
            s_flag = f;
        }
        __syncthreads();
        last = s_flag != 0u;
        if (last) {
            __threadfence();
            if (tid == 0) s_nc = __hip_atomic_load(J->wk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (MODE == SV_CLASS) skipped = __hip_atomic_load(J->wk + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid < K) {
                uint32_t* slot = J->scert + tid * NSLOT + 1;
                s_seed[tid] = max(s_seed[tid], __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                *slot = 0u;
            }
        }
    }
    if (!last) return;
    __syncthreads();
    // (a list that overflowed decides nothing: the host sweeps again, or decides
    // the source exhaustively; one workgroup certified 65,536 plans in 5 ms)
    const uint32_t total = s_nc, nc = total > J->cap ? 0u : total;
    if (nwg > 1 && tid < 32) J->wk[tid] = 0u;
    // a list that overflowed: its seeds serve the next sweep of the source
    if (tid < K && total > J->cap) J->scert[tid * NSLOT] = s_seed[tid];

    // certification: thresholds from the best seeds of all, then every
    // (candidate, level) that can still win is re-evaluated in fp64
    __shared__ uint64_t s_bv[KMAX], s_bi[KMAX], s_cv[KMAX], s_ci[KMAX];
    __shared__ double s_bp[KMAX], s_bd[KMAX], s_bx[KMAX];
    __shared__ double s_cp[KMAX], s_cd[KMAX], s_cx[KMAX];
    __shared__ double s_ct[KMAX];  // objective: fp64 threshold on the estimate
    uint32_t* pairs = (uint32_t*)s_dyn;
    const int T = solve_cert_threads(nf, lds);
    double* f64 = (double*)(s_dyn + SOLVE_PAIRS * 4);
    uint8_t* ids = (uint8_t*)(f64 + (size_t)nf * T);
    if (OBJ) {
        if (tid < K) {
            double t = -INFINITY;
            if (s_seed[tid]) {
                const double sb = (double)fkey_value(s_seed[tid]), e2 = P->err2[tid];
                t = sb - e2;
                t = t - (fabs(sb) + e2) * 0x1p-50;
            }
            s_ct[tid] = t;
        }
    } else {
        set_thr();
    }
    if (tid < K) {
        s_bv[tid] = 0ull;
        s_bi[tid] = ~0ull;
    }
    if (tid == 0) s_nh = 0;
    __syncthreads();
    auto certify = [&]() __attribute__((always_inline)) {  // the gathered pairs, T at a time; called by every thread
        const uint32_t n = s_nh;
        for (uint32_t p0 = 0; p0 < n; p0 += (uint32_t)T) {
            if (tid < K) {
                s_cv[tid] = 0ull;
                s_ci[tid] = ~0ull;
            }
            __syncthreads();
            const uint32_t p = p0 + tid;
            int k = 0;
            uint64_t key = 0, idx = 0;
            double x = 0.0, cp = 0.0, d = 0.0;
            if (tid < T && p < n) {
                k = (int)(pairs[p] >> 27);
                const uint32_t i = pairs[p] & 0x7ffffffu;
                idx = nwg == 1 && i < (uint32_t)SOLVE_OWN ? s_own[i].index : J->cand[i].index;
                decode64(P, idx, ids + tid, T);
                pair_eval<OBJ>(P, ids + tid, f64 + tid, T, k, x, cp, d);
                if (OBJ) {
                    x = obj_j(P->lam_l64, P->m64[k], x, cp, d);
                    key = dkey(x);
                } else if (cp <= P->slo) {
                    key = dkey(x);
                }
                if (key) atomicMax((unsigned long long*)&s_cv[k], (unsigned long long)key);
            }
            __syncthreads();
            const bool tie = key && s_cv[k] == key;
            if (tie) atomicMin((unsigned long long*)&s_ci[k], (unsigned long long)idx);
            __syncthreads();
            if (tie && s_ci[k] == idx) {  // (a plan listed twice writes the same values)
                s_cx[k] = x;
                s_cp[k] = cp;
                s_cd[k] = d;
            }
            __syncthreads();
            if (tid < K && s_cv[tid] &&
                (s_cv[tid] > s_bv[tid] || (s_cv[tid] == s_bv[tid] && s_ci[tid] < s_bi[tid]))) {
                s_bv[tid] = s_cv[tid];
                s_bi[tid] = s_ci[tid];
                s_bx[tid] = s_cx[tid];
                s_bp[tid] = s_cp[tid];
                s_bd[tid] = s_cd[tid];
            }
            __syncthreads();
        }
        if (tid == 0) s_nh = 0;
        __syncthreads();
    };
    // per-backend pressure: a level's candidates are those its own sweep has
    // listed, or any sweep where some workgroup left the level's out (without
    // it every candidate took part at every level of no higher threshold:
    // 512 requests of 2^14 plans at 32 levels 857 us, with it 386)
    auto pass = [&](const Cand& c, int k) __attribute__((always_inline)) {
        return (__float_as_uint(c.cp) & 31u) == (uint32_t)k || (skipped >> k & 1u);
    };
    for (uint32_t c0 = 0; c0 < nc; c0 += WG)
        for (int k0 = 0; k0 < K; k0 += 4) {
            const uint32_t i = c0 + tid;
            if (i < nc) {
                const Cand c = nwg == 1 && i < (uint32_t)SOLVE_OWN ? s_own[i] : J->cand[i];
                for (int k = k0; k < min(K, k0 + 4); ++k) {
                    const bool in = OBJ ? fma(-P->m64[k], (double)c.cp, (double)c.corr) >= s_ct[k]
                                        : c.corr >= s_thr[k] && (MODE == SV_CLASS ? pass(c, k) : c.cp <= s_hi[k]);
                    if (in) pairs[atomicAdd(&s_nh, 1u)] = (uint32_t)k << 27 | i;
                }
            }
            __syncthreads();
            const bool go = s_nh > (uint32_t)(SOLVE_PAIRS - 4 * WG) || (c0 + WG >= nc && k0 + 4 >= K);
            __syncthreads();
            if (go) certify();
        }
    __shared__ dy_choice s_out[KMAX];
    if (tid < K) {
        dy_choice c;
        if (s_bv[tid]) {
            c.index = (int64_t)s_bi[tid];
            c.feasible = 1;
            c.corr = (float)s_bx[tid];
            c.cp = (float)s_bp[tid];
            c.demand = (float)s_bd[tid];
        } else {
            c.index = -1;
            c.feasible = 0;
            c.corr = NAN;
            c.cp = NAN;
            c.demand = NAN;
        }
        J->out[tid] = c;
        s_out[tid] = c;
    }
    // A source that was given seeds leaves every slot clear (a generated sweep,
    // whose overflow this launch recovers, has sampled into all of them): the
    // next call may give the job slot to another source without clearing it.
    if (J->seeded && total <= J->cap)
        for (int i = tid; i < KMAX * NSLOT; i += WG) J->scert[i] = 0u;
    const int32_t flags = total > J->cap ? (int32_t)JF_OVERFLOW : 0;
    if (tid == 0) {
        *J->ncand = total;
        *J->flags = flags;
    }
    if (!J->hout) return;
    // the host-mapped copy, then the completion word behind a system fence
    __syncthreads();
    const uint32_t* src = (const uint32_t*)s_out;
    uint32_t* dst = (uint32_t*)J->hout;
    for (int i = tid; i < K * 6; i += WG) dst[i] = src[i];
    if (tid == 0) {
        *J->hncand = total;
        *J->hflags = flags;
    }
    if (J->hdone) {
        __threadfence_system();
        __syncthreads();
        if (tid == 0) __hip_atomic_store(J->hdone, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// mode: SV_LEVEL, SV_CLASS or SV_OBJ.  ent: the largest node table (N x R_max)
// of the sources, rmax their largest R_max, nmax their most nodes, lat: the
// most durations of all levels of one (per-backend pressure), col: the most
// prefix nodes of a source that needs recurrence columns, 0 for none.
hipError_t launch_solve(const JobDev* d_jobs, const LaunchSizes& sz, int n, int mode, int nwg, int ent, int rmax,
                        int nmax, int lat, int col, hipStream_t s) {
    if (n == 0) return hipSuccess;
    constexpr int kEntMax = 1024;
    const int e = std::min(ent, kEntMax);
    const int nl = mode == SV_CLASS ? std::min(lat, SOLVE_LAT) : 0;
    const SolveLds L = solve_lds(e, rmax, nl, col, nmax, mode == SV_OBJ, mode == SV_CLASS);
    const int lds = std::max(L.total, SOLVE_PAIRS * 4 + nmax * 9 * 64);
    const dim3 grid((unsigned)nwg, (unsigned)n);
    if (mode == SV_OBJ)
        hipLaunchKernelGGL(k_solve<SV_OBJ>, grid, dim3(WG), lds, s, d_jobs, sz, e, rmax, nl, col, nmax, lds);
    else if (mode == SV_CLASS)
        hipLaunchKernelGGL(k_solve<SV_CLASS>, grid, dim3(WG), lds, s, d_jobs, sz, e, rmax, nl, col, nmax, lds);
    else
        hipLaunchKernelGGL(k_solve<SV_LEVEL>, grid, dim3(WG), lds, s, d_jobs, sz, e, rmax, nl, col, nmax, lds);
    return hipGetLastError();
}

}  // namespace dyp
