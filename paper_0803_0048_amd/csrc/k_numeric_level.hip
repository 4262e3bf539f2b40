// Phase II for rows of up to 64 entries, several rows per wavefront: G lanes
// per row (8, 16, 32 or 64), lane t of a row owning its entry t in a register,
// the 64 / G rows of a wavefront all of one dependency level (parts of the
// chunks of the forward solve, k_solve_level.hip).
//
// k_numeric.hip keeps a row in LDS and walks the update pairs of each pivot:
// per pivot the LDS round trips of the row, and 60 of 64 lanes idle on a short
// row.  Here Phase I lays down one byte per row, pivot and entry (the "plan"):
// where in the pivot's row of U~ the f_ht of this entry stands, so that one
// load per pivot brings every lane the value it needs, the lane of the pivot's
// own entry its diagonal, and the elimination is, per pivot, a division, a
// broadcast among the row's lanes and one update, all in registers.  Pivots go
// in ascending order, so every entry takes its updates in that order; an update
// that the pattern does not have is not made.  Two kernels:
//   k_numeric_group  final values handed over through one XCD's L2 (narrow
//                    levels) or across the device: a hand-off, a round of loads
//                    and 50 to 90 ns per pivot a level
//   k_numeric_lds    small systems of short rows on one compute unit, U~ in its
//                    LDS: 0.33 us for the pivots of a 2-D ILU(1) level and 0.17
//                    to store
// Measured (us, a wavefront per row -> here): 2-D 64 x 64 ILU(1) 429 -> 121, 400
// x 400 ILU(1) 2788 -> 984 and ILU(3) 4725 -> 2081, 7-point 64^3 ILU(0) 805 ->
// 366, ILU(1) 1264 -> 756, ILU(2) 2258 -> 1756, 110^3 ILU(0) 3470 -> 798; 27-point
// 50^3 ILU(0) 1147 -> 922, ILU(1) 2711 -> 2253.  (A lane per row with 64 rows a
// wavefront, in LDS or in registers, took 2.3 to 15 us a level: its 16 to 63
// gathers of 64 lines each, and a branch for every absent update.)
#include "kernels.h"

namespace tpilu {

namespace {
constexpr uint32_t kNone = 255u;
// bytes of a row's plan: dwords [KP / 4][G], four pivots each; the diagonal of
// each pivot [G] (its slot in F, or its place in LDS); the place of every entry
// in A's row [G]
constexpr size_t plan_bytes(int G, int KP) { return (size_t)G * (KP + 4 + 1); }
}  // namespace

// The value of lane k of every group of G lanes (k < G, a constant).
template <int G, int K>
__device__ __forceinline__ uint32_t bcast32(uint32_t v) {
    if constexpr (G == 64) {
        return __builtin_amdgcn_readlane(v, K);
    } else if constexpr (G == 32) {
        const uint32_t a = __builtin_amdgcn_readlane(v, K), b = __builtin_amdgcn_readlane(v, K + 32);
        return lane_id() & 32 ? b : a;
    } else if constexpr (G == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + K, 0xf, 0xf, true);  // row_newbcast
    } else {
        const uint32_t a = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + K, 0xf, 0xf, true);
        const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x158 + K, 0xf, 0xf, true);
        return lane_id() & 8 ? b : a;
    }
}
template <int G, int K>
__device__ __forceinline__ double bcast(double v) {
    const uint64_t u = as_u64(v);
    const uint32_t lo = bcast32<G, K>((uint32_t)u), hi = bcast32<G, K>((uint32_t)(u >> 32));
    return as_f64(((uint64_t)hi << 32) | lo);
}

// for constants K = 0 .. N - 1, until f returns false
template <int N, int K = 0, class Fn>
__device__ __forceinline__ void unrolled(Fn&& f) {
    if constexpr (K < N) {
        f(std::integral_constant<int, K>{});
        unrolled<N, K + 1>(static_cast<Fn&&>(f));
    }
}

// One wavefront per 64 / G rows; position p's plan at plan + p * plan_bytes, its
// record (row, first slot, pivots and length << 16, first entry of A).  ucum
// (null: slots in F): entries of L~ before row i, a diagonal's place among the
// entries of U~ being its slot minus those up to its row.
template <int G, int KP>
__global__ __launch_bounds__(64) void k_numeric_plan(PatDev P, LevelSched L, const int32_t* __restrict__ ucum,
                                                     uint8_t* __restrict__ plan, int4* __restrict__ rec) {
    constexpr int R = kWave / G;
    __shared__ uint8_t tab[R * KP * G];
    __shared__ uint8_t aat[R * G];
    const int lane = lane_id(), g = lane / G, t = lane % G;
    for (int64_t p0 = (int64_t)blockIdx.x * R; p0 < P.n; p0 += (int64_t)gridDim.x * R) {
        const int64_t p = p0 + g;
        wave_sync();
#pragma unroll
        for (int k = 0; k < KP; ++k) tab[(g * KP + k) * G + t] = (uint8_t)kNone;
        aat[lane] = (uint8_t)kNone;
        wave_sync();
        if (p < P.n) {
            const int4 r = L.rec[p];
            const int32_t rs = r.y;
            const int64_t a0 = P.rpA[r.x], a1 = P.rpA[r.x + 1];
            for (int64_t a = a0 + t; a < a1; a += G) aat[g * G + (P.a2f[a] - rs)] = (uint8_t)(a - a0);
            int32_t place = 0;
            if (t < r.z) {
                const int32_t dh = P.lsd[rs + t];
                place = ucum ? dh - ucum[P.ciF[rs + t] + 1] : dh;
                tab[(g * KP + t) * G + t] = 0;
                for (int64_t e = P.sptr[rs + t]; e < P.sptr[rs + t + 1]; ++e)
                    tab[(g * KP + t) * G + (P.sp[e] - rs)] = (uint8_t)(P.sq[e] - dh);
            }
            reinterpret_cast<int32_t*>(plan + p * plan_bytes(G, KP))[KP / 4 * G + t] = place;
            if (t == 0)
                rec[p] = make_int4(r.x, rs, r.z | (int32_t)(P.rpF[r.x + 1] - rs) << 16, (int32_t)a0);
        }
        wave_sync();
        if (p < P.n) {
            uint8_t* out = plan + p * plan_bytes(G, KP);
            for (int q = 0; q < KP / 4; ++q) {
                uint32_t w = 0;
                for (int b = 0; b < 4; ++b) w |= (uint32_t)tab[(g * KP + 4 * q + b) * G + t] << (8 * b);
                reinterpret_cast<uint32_t*>(out)[q * G + t] = w;
            }
            out[G * (KP + 4) + t] = aat[lane];
        }
    }
}

// What a lane knows of its row before the wait; a part's rows are positions
// h.x .. h.y - 1.
template <int G, int KP>
struct GroupRow {
    int32_t j, rs, nl, len, a0;
    uint32_t rel[KP / 4];
    int32_t dh;  // lane k < nl: diagonal of pivot k
    uint32_t at;
};

template <int G, int KP>
__device__ __forceinline__ GroupRow<G, KP> group_load(const NumericPlan& N, const int4& h) {
    const int t = lane_id() % G;
    const int32_t p = h.x + lane_id() / G;
    GroupRow<G, KP> x;
    x.j = x.rs = x.nl = x.len = x.dh = x.a0 = 0;
    x.at = kNone;
#pragma unroll
    for (int q = 0; q < KP / 4; ++q) x.rel[q] = 0xffffffffu;
    if (p < h.y) {
        const int4 r = N.rec[p];
        const uint8_t* pl = N.plan + p * plan_bytes(G, KP);
#pragma unroll
        for (int q = 0; q < KP / 4; ++q) x.rel[q] = reinterpret_cast<const uint32_t*>(pl)[q * G + t];
        x.dh = reinterpret_cast<const int32_t*>(pl)[KP / 4 * G + t];
        x.at = pl[G * (KP + 4) + t];
        x.j = r.x;
        x.rs = r.y;
        x.nl = r.z & 0xffff;
        x.len = r.z >> 16;
        x.a0 = r.w;
    }
    return x;
}
// the entry's value in A
template <int G, int KP>
__device__ __forceinline__ double group_a(const GroupRow<G, KP>& x, const double* __restrict__ a_val) {
    return x.at != kNone ? a_val[x.a0 + (int32_t)x.at] : 0.0;
}

constexpr int kGroupAhead = 4;  // pivots polled together

// Pivot k of the wavefront's rows: w the lane's entry, v its value from pivot k.
template <int G, int KP, bool kFused, int k>
__device__ __forceinline__ double group_step(double w, const uint32_t (&rel)[KP / 4], double v) {
    const double l = w / v;
    const double x = ikj_update<kFused>(w, bcast<G, k>(l), v);
    const bool has = ((rel[k / 4] >> (8 * (k & 3))) & 255u) != kNone;  // (the pivot's own lane has one too)
    return has ? (lane_id() % G == k ? l : x) : w;
}

__device__ __forceinline__ int32_t wave_max(int32_t v) {
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off));
    return uniform(v);
}

// Parts (the rows of one level, 64 / G at a time) are drawn in order from the
// position counters (next_pos), and not before the last one is done: a part
// held back behind another of its own wavefront was late by a whole level
// (2-D 400^2 ILU(1), a ticket drawn ahead: 3.0 ms, 1.1 so).  A wavefront waits
// pivot by pivot, so that only what comes after the last value's pivot is left
// to do when that arrives.
template <Scope S, int G, int KP, bool kFused>
__global__ __launch_bounds__(64) void k_numeric_group(PatDev P, LevelSched L, NumericPlan N,
                                                      const double* __restrict__ a_val, double* F, Ctl* ctl,
                                                      uint64_t limit, int64_t skip_row) {
    if constexpr (S == Scope::Xcd) {
        if (!xcd_member(ctl)) return;
    }
    const int lane = lane_id(), t = lane % G;
    PosRun run;
    uint32_t c;
    while (next_pos(ctl, (uint32_t)N.nparts, 1u, S == Scope::Xcd ? 1u : (uint32_t)P.parts, run, c)) {
        const int4 h = N.part[c];
        const GroupRow<G, KP> x = group_load<G, KP>(N, h);
        const double a = group_a<G, KP>(x, a_val);
        const bool mine = t < x.len;  // (no entries: no row)
        trace_mark_lane(P.trace, x.j, mine && t == 0);
        const int32_t hint = uniform(L.rec[h.x].w), hd = hint >= 0 ? uniform(P.diagF[hint]) : 0;
        const int32_t most = wave_max(x.nl);
        double w = sanitize_input(a, ctl);
        const double* src[KP];
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const uint32_t rel = (x.rel[k / 4] >> (8 * (k & 3))) & 255u;
            // no update: the pivot's diagonal, which the row waits for anyway
            src[k] = F + ((int32_t)bcast32<G, (k < G ? k : 0)>((uint32_t)x.dh) + (int32_t)(rel == kNone ? 0u : rel));
        });
        // a single value first (k_level_recs), then all of them at once
        uint32_t polls = 0;
        uint64_t t0 = 0;
        bool stop = false;
        if (hint >= 0)
            while (!stop && __any(ld_poll<S>(F + hd) == kPending)) stop = wait_expired(polls, t0, ctl, limit);
        uint64_t v[KP];
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (k < most) v[k] = ld_poll<S>(src[k]);
        });
        trace_mark_lane(P.trace, 2 * (int64_t)P.n + x.j, mine && t == 0);
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (k >= most) return;
            polls = 0;
            while (__any((k < x.nl) & (v[k] == kPending))) {
                if (stop) {
                    if (v[k] == kPending) v[k] = kQNaN;
                    break;
                }
                // this pivot's and the next ones' in one round trip
                uint64_t f[kGroupAhead];
                unrolled<kGroupAhead>([&](auto uc) {
                    constexpr int m = k + decltype(uc)::value;
                    if constexpr (m < KP)
                        if (m < most) f[m - k] = ld_poll<S>(src[m]);
                });
                unrolled<kGroupAhead>([&](auto uc) {
                    constexpr int m = k + decltype(uc)::value;
                    if constexpr (m < KP)
                        if (m < most) v[m] = f[m - k];
                });
                stop = wait_expired(polls, t0, ctl, limit);
            }
            w = group_step<G, KP, kFused, k>(w, x.rel, as_f64(v[k]));
        });
        trace_mark_lane(P.trace, 3 * (int64_t)P.n + x.j, mine && t == 0);
        if (mine && (int64_t)x.j != skip_row) {
            // other rows wait on the U part; the L part is only read by later kernels
            if (t >= x.nl) st_final<S>(F + x.rs + t, w);
            else F[x.rs + t] = w;
        }
        if (mine && t == x.nl && w == 0.0) atomicMin(&ctl->bad_row, (unsigned long long)x.j);
        trace_mark_lane(P.trace, (int64_t)P.n + x.j, mine && t == 0);
    }
}

// Batches of patterns of short rows: lanes are instances (as in
// k_numeric_batch), a wavefront's row in registers, KW entries and KP pivots at
// most, and everything about the row scalar: its plan (laid out for G lanes and
// GK pivots), so that an absent update costs a scalar test.  Waits go pivot by
// pivot.  The fused forward substitution (bvec, xout) is k_numeric_batch's.
// Bound by the hand-off across the device and the scalar tests and pivots after
// the last value to arrive.  Factorization alone, k_numeric_batch -> here (ms):
// 2-D 128^2 ILU(2) x 256 1.23 -> 0.96, x 1024 2.20 -> 1.73, ILU(0) x 256 0.69 ->
// 0.48, ILU(1) x 64 0.81 -> 0.57, 7-point 32^3 ILU(1) x 16 0.76 -> 0.72.  (One XCD
// per team of instance groups gained nothing: the same 0.98 at x 256.)
template <int KP, int KW, int G, int GK, bool kFused>
__global__ __launch_bounds__(64) void k_numeric_batch_plan(PatDev P, NumericPlan N, const double* __restrict__ a_val,
                                                           int32_t B, double* F, Ctl* ctl, uint64_t limit,
                                                           int64_t skip_row, const double* __restrict__ bvec,
                                                           double* xout) {
    const int lane = lane_id();
    const int32_t groups = (B + kWave - 1) / kWave;
    const uint32_t ntask = (uint32_t)P.n * (uint32_t)groups;
    PosRun run;
    uint32_t task;
    while (next_pos(ctl, ntask, 1u, (uint32_t)P.parts, run, task)) {
        const int32_t pos = (int32_t)(task / (uint32_t)groups), g = (int32_t)(task % (uint32_t)groups);
        const bool act = g * kWave + lane < B;
        // this instance's byte in a line of B values (in bounds for inactive lanes too)
        const uint32_t own = (uint32_t)(act ? g * kWave + lane : B - 1) << 3;
        auto line = [&](const double* base, int32_t slot) {  // scalar base, 32-bit lane offset
            return reinterpret_cast<const double*>(reinterpret_cast<const char*>(base + (int64_t)slot * B) + own);
        };
        const int4 r = N.rec[pos];
        const int32_t j = uniform(r.x), rs = uniform(r.y), nl = uniform(r.z) & 0xffff, len = uniform(r.z) >> 16,
                      a0 = uniform(r.w);
        const uint32_t* pl = reinterpret_cast<const uint32_t*>(N.plan + (int64_t)pos * plan_bytes(G, GK));
        uint32_t rel[KP / 4 * KW], at[KW / 4];
        int32_t dh[KP];
        unrolled<KP / 4 * KW>([&](auto xc) {
            constexpr int x = decltype(xc)::value;
            rel[x] = (uint32_t)uniform((int32_t)pl[x / KW * G + x % KW]);
        });
        unrolled<KW / 4>([&](auto xc) {
            constexpr int x = decltype(xc)::value;
            at[x] = (uint32_t)uniform((int32_t)pl[G * (GK + 4) / 4 + x]);
        });
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            dh[k] = k < nl ? uniform(P.lsd[rs + k]) : 0;
        });
        auto byte = [&](auto kc, auto tc) {
            constexpr int k = decltype(kc)::value, t = decltype(tc)::value;
            return (rel[k / 4 * KW + t] >> (8 * (k & 3))) & 255u;
        };
        uint32_t has[KP];  // entries that pivot k updates
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            has[k] = 0u;
            unrolled<KW>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if constexpr (t > k) has[k] |= byte(kc, tc) != kNone ? 1u << t : 0u;
            });
        });
        double w[KW];
        unrolled<KW>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const uint32_t x = (at[t / 4] >> (8 * (t & 3))) & 255u;
            w[t] = 0.0;
            if (x != kNone) w[t] = *line(a_val, a0 + (int32_t)x);
        });
        uint64_t u[KP], v[KP * KW];  // (place k * KW + t; those of t <= k are never used)
        auto fetch = [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            u[k] = ld_coherent(line(F, dh[k]));
            unrolled<KW>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if constexpr (t > k)
                    if (has[k] >> t & 1u) v[k * KW + t] = ld_coherent(line(F, dh[k] + (int32_t)byte(kc, tc)));
            });
        };
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            unrolled<KW>([&](auto tc) { v[k * KW + decltype(tc)::value] = 0ull; });
            if (k < nl) fetch(kc);
        });
        unrolled<KW>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            w[t] = sanitize_input(w[t], ctl);
        });
        bool stop = false;
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (k >= nl) return;
            uint32_t polls = 0;
            uint64_t t0 = 0;
            for (;;) {
                bool pend = u[k] == kPending;
                unrolled<KW>([&](auto tc) {
                    constexpr int t = decltype(tc)::value;
                    if constexpr (t > k) pend |= v[k * KW + t] == kPending;
                });
                if (!__any(pend)) break;
                if (stop || wait_expired(polls, t0, ctl, limit)) {
                    stop = true;
                    if (u[k] == kPending) u[k] = kQNaN;
                    unrolled<KW>([&](auto tc) {
                        constexpr int t = decltype(tc)::value;
                        if (v[k * KW + t] == kPending) v[k * KW + t] = kQNaN;
                    });
                    break;
                }
                fetch(kc);
                if constexpr (k + 1 < KP)
                    if (k + 1 < nl) fetch(std::integral_constant<int, k + 1>{});
            }
            const double l = w[k] / as_f64(u[k]);
            unrolled<KW>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if constexpr (t > k)
                    if (has[k] >> t & 1u) w[t] = ikj_update<kFused>(w[t], l, as_f64(v[k * KW + t]));
            });
            w[k] = l;
        });
        if (act && (int64_t)j != skip_row) {
            // the U part first: other rows wait on it
            unrolled<KW>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t >= nl && t < len) st_publish(const_cast<double*>(line(F, rs + t)), w[t]);
            });
            unrolled<KP>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t < nl) *const_cast<double*>(line(F, rs + t)) = w[t];
            });
        }
        bool zero = false;
        unrolled<KP + 1>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            zero |= (t == nl) & (w[t] == 0.0);
        });
        if (act && zero) atomicMin(&ctl->bad_row, (unsigned long long)j);
        if (xout) {
            double sx = sanitize_input(*line(bvec, j), ctl);
            uint64_t xv[KP];
            int32_t h[KP];
            unrolled<KP>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                if (k >= nl) return;
                h[k] = uniform(P.ciF[rs + k]);
                xv[k] = ld_coherent(line(xout, h[k]));
            });
            unrolled<KP>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                if (k >= nl) return;
                uint32_t polls = 0;
                uint64_t t0 = 0;
                while (__any(xv[k] == kPending)) {
                    if (stop || wait_expired(polls, t0, ctl, limit)) {
                        stop = true;
                        if (xv[k] == kPending) xv[k] = kQNaN;
                        break;
                    }
                    xv[k] = ld_coherent(line(xout, h[k]));
                }
                sx = sx - w[k] * as_f64(xv[k]);
            });
            if (act && (int64_t)j != skip_row) st_publish(const_cast<double*>(line(xout, j)), sx);
        }
    }
}

typedef __attribute__((address_space(3))) volatile double LdsDouble;
typedef __attribute__((address_space(3))) volatile int32_t LdsInt;
constexpr int kLdsWaves = 16;

// Part c belongs to wavefront c mod kLdsWaves; `done` counts finished parts,
// and the parts of a level may start once every part before the level's first
// is finished (as in k_solve_lds).  A wavefront has the plans of its next two
// parts and the values of A of the next one on their way while it works on one.
template <int G, int KP, bool kFused>
__global__ __launch_bounds__(kLdsWaves * 64) void k_numeric_lds(PatDev P, NumericPlan N,
                                                                const double* __restrict__ a_val, double* F,
                                                                int64_t skip_row, Ctl* ctl) {
    extern __shared__ double ush[];
    __shared__ int32_t sh_done;
    LdsDouble* U = (LdsDouble*)ush;
    LdsInt* done = (LdsInt*)&sh_done;
    if (threadIdx.x == 0) {
        ctl->abort = 0;
        ctl->status = 0;
        ctl->bad_row = ~0ull;
        *done = 0;
    }
    __syncthreads();
    const int t = lane_id() % G;
    auto part = [&](int32_t q) { return q < N.nparts ? N.part[q] : make_int4(0, 0, 0, 0); };
    int32_t c = uniform((int32_t)(threadIdx.x / kWave));
    int4 h = part(c), h1 = part(c + kLdsWaves), h2 = part(c + 2 * kLdsWaves);
    GroupRow<G, KP> x = group_load<G, KP>(N, h), x1 = group_load<G, KP>(N, h1);
    double a = group_a<G, KP>(x, a_val);
    int32_t at = x.rs - N.ucum[x.j] - x.nl;  // place of the row's first entry of U~, minus its pivots
    while (c < N.nparts) {
        const GroupRow<G, KP> x2 = group_load<G, KP>(N, h2);
        const double a1 = group_a<G, KP>(x1, a_val);
        const int32_t at1 = x1.rs - N.ucum[x1.j] - x1.nl;
        const int4 h3 = part(c + 3 * kLdsWaves);
        const bool mine = t < x.len;
        trace_mark_lane(P.trace, x.j, mine && t == 0);
        const int32_t most = wave_max(x.nl);
        double w = sanitize_input(a, ctl);
        LdsDouble* src[KP];
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const uint32_t rel = (x.rel[k / 4] >> (8 * (k & 3))) & 255u;
            src[k] = U + ((int32_t)bcast32<G, k>((uint32_t)x.dh) + (int32_t)(rel == kNone ? 0u : rel));
        });
        while (uniform(*done) < h.z) {}
        trace_mark_lane(P.trace, 2 * (int64_t)P.n + x.j, mine && t == 0);
        double v[KP];
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            v[k] = *src[k];
        });
        unrolled<KP>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (k < most) w = group_step<G, KP, kFused, k>(w, x.rel, v[k]);
        });
        trace_mark_lane(P.trace, 3 * (int64_t)P.n + x.j, mine && t == 0);
        jitter((uint32_t)c);
        if (mine && t >= x.nl) U[at + t] = w;
        // the wavefront's LDS operations complete in order: the count rises after the values are there
        if (lane_id() == 0) __hip_atomic_fetch_add((int32_t*)done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (mine && (int64_t)x.j != skip_row) F[x.rs + t] = w;
        if (mine && t == x.nl && w == 0.0) atomicMin(&ctl->bad_row, (unsigned long long)x.j);
        trace_mark_lane(P.trace, (int64_t)P.n + x.j, mine && t == 0);
        c += kLdsWaves;
        h = h1; h1 = h2; h2 = h3;
        x = x1; x1 = x2;
        a = a1;
        at = at1;
    }
}

namespace {
struct Config {
    int g, kp;
};
constexpr Config kConfigs[] = {{8, 4}, {16, 8}, {32, 16}, {64, 32}};
}  // namespace

int numeric_plan_config(int32_t max_row, int32_t max_lrow) {
    for (int i = 0; i < 4; ++i)
        if (max_row <= kConfigs[i].g && max_lrow <= kConfigs[i].kp) return i;
    return -1;
}
int numeric_plan_rows(int config) { return kWave / kConfigs[config].g; }
size_t numeric_plan_bytes(int config) { return plan_bytes(kConfigs[config].g, kConfigs[config].kp); }

__global__ __launch_bounds__(1024) void k_lower_before(int32_t n, const int64_t* __restrict__ rpF,
                                                       const int32_t* __restrict__ diagF,
                                                       int32_t* __restrict__ before) {
    __shared__ int32_t sh[1024];
    const int tid = threadIdx.x;
    int32_t base = 0;
    for (int32_t i0 = 0; i0 < n; i0 += 1024) {
        const int32_t i = i0 + tid, own = i < n ? diagF[i] - (int32_t)rpF[i] : 0;
        sh[tid] = own;
        __syncthreads();
        for (int w = 1; w < 1024; w <<= 1) {
            const int32_t v = tid >= w ? sh[tid - w] : 0;
            __syncthreads();
            sh[tid] += v;
            __syncthreads();
        }
        if (i < n) before[i] = base + sh[tid] - own;
        base += sh[1023];
        __syncthreads();
    }
    if (tid == 0) before[n] = base;
}

hipError_t launch_lower_before(int32_t n, const int64_t* rpF, const int32_t* diagF, int32_t* before, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_lower_before, dim3(1), dim3(1024), 0, s, n, rpF, diagF, before);
    return hipGetLastError();
}

hipError_t launch_numeric_plan(const PatDev& P, const LevelSched& L, const NumericPlan& N, hipStream_t s) {
    if (P.n <= 0) return hipSuccess;
    const int64_t rows = numeric_plan_rows(N.config);
    auto go = [&](auto kern) {
        const int grid = (int)std::min<int64_t>((P.n + rows - 1) / rows, 65536);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64), 0, s, P, L, N.ucum, N.plan, N.rec);
    };
    if (N.config == 0) go(k_numeric_plan<8, 4>);
    else if (N.config == 1) go(k_numeric_plan<16, 8>);
    else if (N.config == 2) go(k_numeric_plan<32, 16>);
    else go(k_numeric_plan<64, 32>);
    return hipGetLastError();
}

int numeric_batch_plan_shape(const NumericPlan& N, int32_t max_row, int32_t max_lrow) {
    if (!N.plan || N.config > 1) return -1;
    return N.config == 0 ? 0 : max_row <= 12 && max_lrow <= 4 ? 1 : 2;
}

hipError_t launch_numeric_batch_plan(const PatDev& P, const NumericPlan& N, int shape, const double* a_val,
                                     int32_t batch, double* f_val, bool fused, Ctl* ctl, uint64_t spin_limit,
                                     int64_t skip_row, int32_t grid, const double* bvec, double* xout, hipStream_t s) {
    if (P.n <= 0) return hipSuccess;
    auto go = [&](auto plain, auto fma) {
        hipLaunchKernelGGL(fused ? fma : plain, dim3(grid), dim3(kWave), 0, s, P, N, a_val, batch, f_val, ctl, spin_limit,
                           skip_row, bvec, xout);
    };
    if (shape == 0) go(k_numeric_batch_plan<4, 8, 8, 4, false>, k_numeric_batch_plan<4, 8, 8, 4, true>);
    else if (shape == 1) go(k_numeric_batch_plan<4, 12, 16, 8, false>, k_numeric_batch_plan<4, 12, 16, 8, true>);
    else go(k_numeric_batch_plan<8, 16, 16, 8, false>, k_numeric_batch_plan<8, 16, 16, 8, true>);
    return hipGetLastError();
}

hipError_t launch_numeric_level(const PatDev& P, const LevelSched& L, const NumericPlan& N, const double* a_val,
                                double* f_val, bool fused, Ctl* ctl, uint64_t spin_limit, int64_t skip_row,
                                hipStream_t s) {
    if (P.n <= 0) return hipSuccess;
    if (N.ucum) {
        const size_t lds = (size_t)N.nnz_u * sizeof(double);
        auto go = [&](auto plain, auto fma) {
            hipLaunchKernelGGL(fused ? fma : plain, dim3(1), dim3(kLdsWaves * kWave), lds, s, P, N, a_val, f_val,
                               skip_row, ctl);
        };
        N.config == 0 ? go(k_numeric_lds<8, 4, false>, k_numeric_lds<8, 4, true>)
                      : go(k_numeric_lds<16, 8, false>, k_numeric_lds<16, 8, true>);
        return hipGetLastError();
    }
    auto go = [&](auto xplain, auto xfma, auto plain, auto fma) {
        const int grid = N.one_xcd ? N.waves * kXcds : N.waves;
        hipLaunchKernelGGL(N.one_xcd ? (fused ? xfma : xplain) : (fused ? fma : plain), dim3(grid), dim3(kWave), 0, s,
                           P, L, N, a_val, f_val, ctl, spin_limit, skip_row);
    };
    auto pick = [&](auto gc, auto kc) {
        constexpr int G = decltype(gc)::value, K = decltype(kc)::value;
        go(k_numeric_group<Scope::Xcd, G, K, false>, k_numeric_group<Scope::Xcd, G, K, true>,
           k_numeric_group<Scope::Device, G, K, false>, k_numeric_group<Scope::Device, G, K, true>);
    };
    if (N.config == 0) pick(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{});
    else if (N.config == 1) pick(std::integral_constant<int, 16>{}, std::integral_constant<int, 8>{});
    else if (N.config == 2) pick(std::integral_constant<int, 32>{}, std::integral_constant<int, 16>{});
    else pick(std::integral_constant<int, 64>{}, std::integral_constant<int, 32>{});
    return hipGetLastError();
}

}  // namespace tpilu
