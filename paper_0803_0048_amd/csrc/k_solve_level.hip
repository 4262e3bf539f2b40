// The triangular solves of Eq. 1 by level chunks: lane per row, the rows of a
// wavefront all of one dependency level.
//
// A chunk is up to 64 consecutive positions of the level order that lie in
// one level, so the rows of a chunk never wait on each other and the
// wavefront can take their entries in lockstep: entry k of every row, then
// entry k + 1, with no per-lane bookkeeping.  Per position the schedule holds
// one 16-byte record (row, first slot, entries, diagonal slot), read
// coalesced, in place of a chain of dependent loads (level order -> row
// bounds and diagonal).
//
// Two kernels use it; both are bound by the step from level to level:
//   k_solve_lds     both substitutions of a small system in one launch, on one
//                   compute unit with x in its LDS: a level costs an LDS
//                   write, the count of finished chunks and the LDS reads of
//                   the next level, about 0.18 us against 0.7 us through the
//                   L2 (2-D 64 x 64 ILU(1), 190 levels, both sweeps: 0.281 ->
//                   0.079 ms).  On larger systems the loads of one compute
//                   unit bound it, about 1 ns per entry of F.
//   k_solve_chunks  one substitution on one XCD, values handed over through
//                   its L2 (see Scope::Xcd), for rows of at most 16 entries:
//                   0.45 us a level for up to 4 entries, 0.6 for 8, 0.97 for
//                   16 (2-D 400 x 400 ILU(1), both sweeps: 5.00 -> 1.16 ms;
//                   7-point 64^3 ILU(1): 1.78 -> 0.70 ms, ILU(2): 5.05 -> 1.65
//                   ms).  The former kernel for this shape polled across XCDs and
//                   kept every lane at an entry of its own.
// The order of every row's subtractions is that of k_solve.hip: forward
// ascending columns, backward right to left and then the division.
#include "kernels.h"

namespace tpilu {

// ----------------------------------------------------------------------------------
// the schedule: level bounds -> chunks, and one record per position
// ----------------------------------------------------------------------------------
// off[l] .. off[l + 1]: positions of level l (0-based).  head[c] of chunk c =
// (first position, end, first chunk of its level, 0); depth comes from device
// memory, the chunk count goes there.
// The second block does the same in parts of `rows` positions, when wanted.
__global__ __launch_bounds__(1024) void k_level_chunks(const int64_t* __restrict__ off,
                                                       const int32_t* __restrict__ depth, int4* __restrict__ heads,
                                                       int32_t* __restrict__ nheads, int32_t rows,
                                                       int4* __restrict__ part, int32_t* __restrict__ nparts) {
    const int32_t size = blockIdx.x ? rows : kWave;
    int4* __restrict__ head = blockIdx.x ? part : heads;
    int32_t* __restrict__ nchunk = blockIdx.x ? nparts : nheads;
    __shared__ int32_t sh[1024];
    const int tid = threadIdx.x;
    const int32_t levels = *depth;
    int32_t base = 0;
    for (int32_t l0 = 0; l0 < levels; l0 += 1024) {
        const int32_t l = l0 + tid;
        const int32_t a = l < levels ? (int32_t)off[l] : 0, b = l < levels ? (int32_t)off[l + 1] : 0;
        const int32_t c = (b - a + size - 1) / size;
        sh[tid] = c;
        __syncthreads();
        for (int w = 1; w < 1024; w <<= 1) {
            const int32_t v = tid >= w ? sh[tid - w] : 0;
            __syncthreads();
            sh[tid] += v;
            __syncthreads();
        }
        const int32_t first = base + sh[tid] - c;
        for (int32_t k = 0; k < c; ++k)
            head[first + k] = make_int4(a + k * size, min(a + (k + 1) * size, b), first, 0);
        base += sh[1023];
        __syncthreads();
    }
    if (tid == 0) *nchunk = base;
}

// rec[p] of position p: row, first slot of its half in subtraction order,
// entries, hint row (the last position's row kHintLevels levels earlier, or -1).
// A wavefront first waits for its hint row alone, one line per poll, and only
// then polls the values it needs, 64 lines per entry: with all waiting
// wavefronts polling those, their requests slow the hand-offs of the rows in
// work (7-point 64^3 ILU(1), 192 wavefronts, 8 entries: 2.35 -> 1.13 ms; one
// level off costs latency, 3 gain nothing more).
constexpr int kHintLevels = 2;
template <bool kBackward>
__global__ void k_level_recs(int32_t n, const int64_t* __restrict__ off, const int32_t* __restrict__ depth,
                             const int32_t* __restrict__ perm, const int64_t* __restrict__ rpF,
                             const int32_t* __restrict__ diagF, int4* __restrict__ rec) {
    const int32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int32_t i = perm[p], d = diagF[i], l = depth[i] - 1;
    const int32_t q = (int32_t)(kBackward ? rpF[i + 1] - 1 : rpF[i]);
    rec[p] = make_int4(i, q, kBackward ? q - d : d - q, l >= kHintLevels ? perm[off[l - kHintLevels + 1] - 1] : -1);
}

hipError_t launch_level_sched(int32_t n, const int64_t* off, const int32_t* depth, const int32_t* max_depth,
                              const int32_t* perm, const int64_t* rpF, const int32_t* diagF, bool backward, int4* rec,
                              int4* head, int32_t* nchunk, int32_t part_rows, int4* part, int32_t* nparts,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_level_chunks, dim3(part ? 2 : 1), dim3(1024), 0, s, off, max_depth, head, nchunk, part_rows, part,
                       nparts);
    const dim3 g((n + 255) / 256);
    if (backward)
        hipLaunchKernelGGL(k_level_recs<true>, g, dim3(256), 0, s, n, off, depth, perm, rpF, diagF, rec);
    else
        hipLaunchKernelGGL(k_level_recs<false>, g, dim3(256), 0, s, n, off, depth, perm, rpF, diagF, rec);
    return hipGetLastError();
}

typedef __attribute__((address_space(3))) volatile double LdsDouble;
typedef __attribute__((address_space(3))) volatile int32_t LdsInt;

// ----------------------------------------------------------------------------------
// one compute unit, x in LDS
// ----------------------------------------------------------------------------------
// One sweep: chunk c belongs to wavefront c mod W.  `done` in LDS counts
// finished chunks; the chunks of a level may start once every chunk before
// the level's first is finished (all of those finish before any of the
// level's own can, so the count says so exactly).  A wavefront loads the
// entries of its next chunk when it is done with one (about W levels ahead on
// a narrow graph), and the head and records of the ones after, so that memory
// latency never sits between two levels.  Entries past a row's end multiply
// +0.0 by the +0.0 kept in xs[n], which leaves every running difference as it
// is, its sign of zero included.
// kKeepX: the caller sees x.  Rows of the first level have no entries, and their
// x is b to the bit, where the +0.0 subtracted makes a signalling NaN quiet.  (In
// instances of its own: beside any code for it the loop is a few percent slower,
// 2-D 64^2 ILU(1) 76 -> 78 us.)
template <bool kBackward, int KE, bool kKeepX>
__device__ __forceinline__ void lds_sweep(const LevelSched& L, const double* __restrict__ F,
                                          const int32_t* __restrict__ ci, const double* __restrict__ in, double* out,
                                          LdsDouble* xs, LdsInt* done, Ctl* ctl, unsigned long long* trace,
                                          int64_t tr0, int32_t n, bool in_lds) {
    const int32_t waves = (int32_t)(blockDim.x / kWave);
    const int lane = lane_id();
    int32_t c = uniform((int32_t)(threadIdx.x / kWave));
    int4 h = chunk_head(L, c), h1 = chunk_head(L, c + waves), h2 = chunk_head(L, c + 2 * waves);
    int4 r = chunk_rec(L, h), r1 = chunk_rec(L, h1);
    double f[KE], s = 0.0, fii = 1.0;
    int32_t cc[KE];
    auto load = [&]() {
#pragma unroll
        for (int k = 0; k < KE; ++k) {
            cc[k] = n;
            f[k] = 0.0;
            if (k < r.z) {
                const int32_t q = kBackward ? r.y - k : r.y + k;
                cc[k] = ci[q];
                f[k] = F[q];
            }
        }
        if (r.z >= 0) {
            if (!kBackward || !in_lds) s = in[r.x];
            if (kBackward) fii = F[r.y - r.z];
        }
    };
    load();
    while (c < L.nchunk) {
        const bool act = r.z >= 0;
        if (!kBackward && act) s = sanitize_input(s, ctl);
        trace_mark_lane(trace, tr0 + r.x, act);
        while (uniform(*done) < h.z) {}
        double xv[KE];
#pragma unroll
        for (int k = 0; k < KE; ++k) xv[k] = xs[cc[k]];
        double a = s;
        if (kBackward && in_lds) a = xs[act ? r.x : n];
#pragma unroll
        for (int k = 0; k < KE; ++k) a = a - f[k] * xv[k];
        if (kBackward) a = a / fii;
        jitter((uint32_t)r.x);
        if (act) xs[r.x] = a;
        // the wavefront's LDS operations complete in order: the count rises after the values are there
        if (lane == 0) __hip_atomic_fetch_add((int32_t*)done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if constexpr (kKeepX && !kBackward)
            if (uniform(h.z) == 0) a = s;  // the first level
        if (act && out) out[r.x] = a;
        trace_mark_lane(trace, tr0 + n + r.x, act);
        c += waves;
        h = h1;
        h1 = h2;
        r = r1;
        load();
        r1 = chunk_rec(L, h1);
        h2 = chunk_head(L, c + 2 * waves);
    }
}

template <int KE, bool kKeepX>
__global__ __launch_bounds__(1024) void k_solve_lds(int32_t n, LevelSched Lo, LevelSched Up,
                                                    const double* __restrict__ F, const int32_t* __restrict__ ci,
                                                    const double* __restrict__ b, double* x, double* y, int sweeps,
                                                    int reset, Ctl* ctl, unsigned long long* trace, const int32_t* skip) {
    if (skip && *skip) return;  // a GMRES cycle that has stopped
    extern __shared__ double xsh[];  // [n]: x, then y in its place; [n + 1]: 0.0
    __shared__ int32_t sh_done;
    LdsDouble* xs = (LdsDouble*)xsh;
    LdsInt* done = (LdsInt*)&sh_done;
    if (threadIdx.x == 0) {
        if (reset) {
            ctl->abort = 0;
            ctl->status = 0;
            ctl->bad_row = ~0ull;
        }
        xs[n] = 0.0;
        *done = 0;
    }
    __syncthreads();
    if (sweeps & 1) lds_sweep<false, KE, kKeepX>(Lo, F, ci, b, x, xs, done, ctl, trace, 0, n, false);
    if (sweeps == 3) {
        __syncthreads();
        if (threadIdx.x == 0) *done = 0;
        __syncthreads();
    }
    if (sweeps & 2) lds_sweep<true, KE, kKeepX>(Up, F, ci, x, y, xs, done, ctl, trace, 2 * (int64_t)n, n, (sweeps & 1) != 0);
}

hipError_t launch_solve_lds(int32_t n, const LevelSched& Lo, const LevelSched& Up, int32_t max_half,
                            const double* f_val, const int32_t* ci, const double* b, double* x, double* y, int sweeps,
                            bool reset, Ctl* ctl, unsigned long long* trace, hipStream_t s, const int32_t* skip) {
    if (n <= 0) return hipSuccess;
    const size_t lds = ((size_t)n + 1) * sizeof(double);
    const int rs = reset ? 1 : 0;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(1), dim3(1024), lds, s, n, Lo, Up, f_val, ci, b, x, y, sweeps, rs, ctl, trace,
                           skip);
    };
    auto pick = [&](auto keep) {
        constexpr bool K = decltype(keep)::value;
        if (max_half <= 4) go(k_solve_lds<4, K>);
        else if (max_half <= 8) go(k_solve_lds<8, K>);
        else go(k_solve_lds<16, K>);
    };
    if (x && (sweeps & 1)) pick(std::true_type{});
    else pick(std::false_type{});
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// one XCD, values handed over through its L2
// ----------------------------------------------------------------------------------
// Chunks are drawn in order from one counter, the next when the last is done: a
// chunk drawn ahead waits behind its wavefront's own and starts late (7-point
// 64^3 ILU(1), both sweeps, 0.84 ms so, 0.70 here; with 63 chunks a level, 110^3
// ILU(0), 1.18 and 1.28).  Deadlock-free: the smallest unfinished chunk is
// always in work, and it only waits on smaller ones.
// KE: entries of a row whose loads are in flight together.  The smallest that
// holds a whole row half is the fastest (7-point 64^3 ILU(1), 6 entries: 0.77
// ms with 8, 1.06 with 4, 0.96 with 16).
// kKeepX: the caller sees x (see lds_sweep); never backward.
template <bool kBackward, int KE, bool kKeepX = false>
__global__ __launch_bounds__(64) void k_solve_chunks(LevelSched L, const double* __restrict__ F,
                                                     const int32_t* __restrict__ ci, const double* __restrict__ in,
                                                     double* out, Ctl* ctl, uint64_t limit,
                                                     unsigned long long* trace, int64_t tr0, int32_t n) {
    if (!xcd_member(ctl)) return;
    const int lane = lane_id();
    for (;;) {
        int32_t c = 0;
        if (lane == 0) c = (int32_t)atomicAdd(&ctl->part[0], 1u);
        c = uniform(c);
        if (c >= L.nchunk) break;
        const int4 h = chunk_head(L, c), r = chunk_rec(L, h);
        const bool act = r.z >= 0;
        trace_mark_lane(trace, tr0 + r.x, act);
        if constexpr (kKeepX) {
            if (uniform(h.z) == 0) {  // the first level: no entries, x is b to the bit
                if (act) st_final<Scope::Xcd>(out + r.x, sanitize_input(in[r.x], ctl));
                trace_mark_lane(trace, tr0 + n + r.x, act);
                continue;
            }
        }
        double s = 0.0, fii = 1.0;
        if (act) {
            s = in[r.x];
            if (kBackward) fii = F[r.y - r.z];
        }
        uint32_t polls = 0;
        uint64_t t0 = 0;
        bool stop = false;
        int32_t k0 = 0;
        do {  // at least once: the input is checked in the first round
            double f[KE];
            int32_t cc[KE];
            uint64_t v[KE];
#pragma unroll
            for (int k = 0; k < KE; ++k) {
                cc[k] = 0;
                f[k] = 0.0;
                if (k0 + k < r.z) {
                    const int32_t q = kBackward ? r.y - (k0 + k) : r.y + (k0 + k);
                    cc[k] = ci[q];
                    f[k] = F[q];
                }
            }
            const int32_t hint = uniform(r.w);
            if (k0 == 0 && hint >= 0)
                while (!stop && __any(ld_poll<Scope::Xcd>(out + hint) == kPending))
                    stop = wait_expired(polls, t0, ctl, limit);
#pragma unroll
            for (int k = 0; k < KE; ++k) v[k] = k0 + k < r.z ? ld_poll<Scope::Xcd>(out + cc[k]) : 0ull;
            polls = 0;
            while (!stop) {
                bool pend = false;
#pragma unroll
                for (int k = 0; k < KE; ++k) pend |= v[k] == kPending;
                if (!__any(pend)) break;
#pragma unroll
                for (int k = 0; k < KE; ++k)
                    if (v[k] == kPending) v[k] = ld_poll<Scope::Xcd>(out + cc[k]);
                stop = wait_expired(polls, t0, ctl, limit);
            }
            if (!kBackward && k0 == 0 && act) s = sanitize_input(s, ctl);
#pragma unroll
            for (int k = 0; k < KE; ++k) s = s - f[k] * as_f64(v[k]);  // past the row's end +0.0 * +0.0
            k0 += KE;
        } while (__any(k0 < r.z));
        if (act) st_final<Scope::Xcd>(out + r.x, stop ? as_f64(kQNaN) : kBackward ? s / fii : s);
        trace_mark_lane(trace, tr0 + n + r.x, act);
    }
}

hipError_t launch_solve_chunks(const PatDev& P, const LevelSched& L, int32_t max_half, const double* f_val,
                               const double* in, double* out, bool backward, bool keep_x, int32_t grid, Ctl* ctl,
                               uint64_t spin_limit, hipStream_t s) {
    if (P.n <= 0) return hipSuccess;
    const int64_t tr0 = backward ? 2 * (int64_t)P.n : 0;
    auto go = [&](auto fwd, auto keep, auto bwd) {
        hipLaunchKernelGGL(backward ? bwd : keep_x ? keep : fwd, dim3(grid * kXcds), dim3(64), 0, s, L, f_val, P.ciF, in, out, ctl,
                           spin_limit, P.trace, tr0, P.n);
    };
    if (max_half <= 4) go(k_solve_chunks<false, 4>, k_solve_chunks<false, 4, true>, k_solve_chunks<true, 4>);
    else if (max_half <= 8) go(k_solve_chunks<false, 8>, k_solve_chunks<false, 8, true>, k_solve_chunks<true, 8>);
    else go(k_solve_chunks<false, 16>, k_solve_chunks<false, 16, true>, k_solve_chunks<true, 16>);
    return hipGetLastError();
}

}  // namespace tpilu
