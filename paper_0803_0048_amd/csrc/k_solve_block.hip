// The triangular solves of Eq. 1 by blocks of 64 consecutive rows, for deep,
// narrow dependency graphs whose rows depend on few of their near neighbours
// (general sparse matrices).
//
// A wavefront per row costs such a graph one hand-off through the L2 per
// dependency level.  Here a wavefront owns 64 consecutive rows, a lane per
// row, and the blocks follow each other in natural order: n / 64 hand-offs
// instead of one per level.  The order of Eq. 3b makes this exact: a row's
// subtractions run over ascending columns, so those of earlier blocks come
// first and those inside the block last (backward: right to left, later
// blocks first).  A row's entries fall in two parts:
//   outer   columns more than kWinBlocks blocks away: their values are nearly
//           always there already; all 64 rows take them in lockstep, entry by
//           entry, straight from memory (no row of the block is among them, so
//           the lockstep cannot wait for itself);
//   window  the kWinBlocks nearest blocks and the block itself: entries and
//           values in LDS.  A second wavefront of the workgroup polls the
//           neighbour blocks' values (64 consecutive ones per load) into the
//           LDS window, where the block's own rows put theirs, and every lane
//           walks its row there, two entries a round.  (With the polls in the
//           walking wavefront every round waited for them and for the
//           acknowledgement of its stores: 23 ms instead of 6.4 below.)
// What bounds a block is the walk inside it, about 0.12 us per round (LDS
// reads, two dependent subtractions, the choice of the next two entries), and
// one hand-off through the L2 of the XCD that all wavefronts run on
// (Scope::Xcd), about 0.23 us.  Random banded n=160,000 ILU(2) (9 rounds a
// block, 12,281 levels), both sweeps: 16.6 ms by a wavefront per row, 6.7 ms
// here; ILU(1) 4.9 -> 3.0 ms; n=10,000 ILU(2) 1.39 -> 0.56 ms.  Rows that
// depend on their direct predecessor (stencils) walk 64 rounds a block and
// stay with the other kernels.
#include "kernels.h"

namespace tpilu {

// ----------------------------------------------------------------------------------
// per row: entries in the window; per direction: the most of any row and the
// rounds of the walks summed over the blocks (in half rounds)
// ----------------------------------------------------------------------------------
// A block whose walk has not settled after kStatSteps steps counts as one of
// 64 rounds (a row waiting on its predecessor, and so on): far beyond what the
// block kernel is chosen for.
constexpr int kStatSteps = 24;

template <bool kBackward>
__device__ __forceinline__ void block_stats(int32_t n, const int64_t* __restrict__ rpF,
                                            const int32_t* __restrict__ ciF, const int32_t* __restrict__ diagF,
                                            uint8_t* __restrict__ wcnt, int32_t* fin, unsigned long long* rounds,
                                            int32_t* max_win) {
    const int lane = lane_id();
    const int32_t nb = (n + kWave - 1) / kWave;
    unsigned long long sum = 0ull;
    int32_t most = 0;
    for (int32_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int32_t base = b * kWave, i = base + lane;
        int32_t q = 0, z = 0, w = 0;
        if (i < n) {
            const int32_t d = diagF[i];
            q = (int32_t)(kBackward ? rpF[i + 1] - 1 : rpF[i]);
            z = kBackward ? q - d : d - q;
            // the window entries are the last ones of the row's chain
            while (w < z && w <= kWinEntries) {
                const int32_t c = ciF[kBackward ? q - (z - 1 - w) : q + (z - 1 - w)];
                if (kBackward ? c >= base + (kWinBlocks + 1) * kWave : c < base - kWinBlocks * kWave) break;
                ++w;
            }
            wcnt[i] = (uint8_t)w;
        }
        fin[lane] = 0;
        wave_sync();
        int32_t mine = 0;
        bool settled = false;
        // (half the rows waiting on their predecessor is enough to know)
        const bool chain = w > 0 && ciF[kBackward ? q - (z - 1) : q + (z - 1)] == (kBackward ? i + 1 : i - 1);
        const bool hopeless = __popcll(__ballot(chain)) > kWave / 2;
        for (int step = 0; step < kStatSteps && !settled && !hopeless; ++step) {
            int32_t t = 0;
            for (int32_t k = z - w; k < z; ++k) {
                const int32_t l = ciF[kBackward ? q - k : q + k] - base;
                if (l >= 0 && l < kWave) t = max(t + 1, fin[l] + 2);
                else if (kBackward ? l < 2 * kWave : l >= -kWave) t = t + 1;
            }
            settled = !__any(t != mine);
            mine = t;
            wave_sync();
            fin[lane] = t;
            wave_sync();
        }
        for (int off = 32; off > 0; off >>= 1) mine = max(mine, __shfl_xor(mine, off));
        sum += (unsigned long long)(settled ? mine : 2 * kWave);
        most = max(most, w);
    }
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off));
    if (lane == 0) {
        if (sum) atomicAdd(rounds, sum);
        if (most) atomicMax(max_win, most);
    }
}

// blockIdx.y: 0 the forward sweep's blocks, 1 the backward sweep's
__global__ __launch_bounds__(64) void k_block_stats(int32_t n, const int64_t* __restrict__ rpF,
                                                    const int32_t* __restrict__ ciF,
                                                    const int32_t* __restrict__ diagF, uint8_t* __restrict__ wcntL,
                                                    uint8_t* __restrict__ wcntU, BlockStats* st) {
    __shared__ int32_t fin[kWave];
    if (blockIdx.y == 0) block_stats<false>(n, rpF, ciF, diagF, wcntL, fin, &st->rounds_l, &st->max_win_l);
    else block_stats<true>(n, rpF, ciF, diagF, wcntU, fin, &st->rounds_u, &st->max_win_u);
}

hipError_t launch_block_stats(int32_t n, const int64_t* rpF, const int32_t* ciF, const int32_t* diagF, uint8_t* wcntL,
                              uint8_t* wcntU, BlockStats* st, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int grid = std::min((n + kWave - 1) / kWave, 1024);  // two atomics a wavefront, on one address
    hipLaunchKernelGGL(k_block_stats, dim3(grid, 2), dim3(64), 0, s, n, rpF, ciF, diagF, wcntL, wcntU, st);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// one sweep
// ----------------------------------------------------------------------------------
constexpr int kOuterChunk = 8;  // outer entries of a row in flight together

typedef __attribute__((address_space(3))) volatile uint64_t LdsWord;

template <bool kBackward>
__global__ __launch_bounds__(128) void k_solve_blocks(int32_t n, const int64_t* __restrict__ rpF,
                                                     const int32_t* __restrict__ ci, const int32_t* __restrict__ diagF,
                                                     const uint8_t* __restrict__ wcnt, const double* __restrict__ F,
                                                     const double* __restrict__ in, double* out, Ctl* ctl,
                                                     uint64_t limit, unsigned long long* trace) {
    __shared__ double fw[(kWinEntries + 4) * kWave];
    __shared__ int32_t cw[(kWinEntries + 4) * kWave];
    __shared__ uint64_t xsh[(kWinBlocks + 1) * kWave];
    __shared__ uint32_t sh_ticket;
    __shared__ int32_t sh_walk;
    LdsWord* xw = (LdsWord*)xsh;
    LdsWord32* walk = (LdsWord32*)&sh_walk;
    if (threadIdx.x == 0) *walk = 0;
    if (!xcd_member(ctl)) return;
    const int lane = lane_id();
    const bool solver = uniform((int32_t)(threadIdx.x / kWave)) == 0;
    const int32_t nb = (n + kWave - 1) / kWave;
    const int64_t tr0 = kBackward ? 2 * (int64_t)n : 0;
    // window-local place of this block and of the neighbours' values
    constexpr int kOwn = kBackward ? 0 : kWinBlocks * kWave;
    constexpr int kNear = kBackward ? kWave : 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) sh_ticket = atomicAdd(&ctl->ticket, 1u);
        if (solver)
#pragma unroll
            for (int u = 0; u <= kWinBlocks; ++u) xw[u * kWave + lane] = kPending;
        __syncthreads();
        const uint32_t t = __builtin_amdgcn_readfirstlane(sh_ticket);
        if (t >= (uint32_t)nb) break;
        const int32_t b = kBackward ? nb - 1 - (int32_t)t : (int32_t)t;
        const int32_t base = b * kWave, i = base + lane;
        const bool has = i < n;
        const int32_t wbase = base - kOwn;  // row of window place 0
        uint32_t polls = 0;
        uint64_t t0 = 0;
        if (!solver) {
            // the neighbour blocks' values into the LDS window, as they come
#pragma unroll
            for (int u = 0; u < kWinBlocks; ++u) {
                // farthest block first: it is complete first
                const int32_t o = kNear + (kBackward ? kWinBlocks - 1 - u : u) * kWave + lane;
                const int32_t r = wbase + o;
                uint64_t v = r >= 0 && r < n ? kPending : 0ull;
                for (;;) {
                    const bool pend = v == kPending;
                    if (!__any(pend)) break;
                    if (pend) {
                        v = ld_poll<Scope::Xcd>(out + r);
                        if (v != kPending) xw[o] = v;
                    }
                    if (wait_expired(polls, t0, ctl, limit)) {
                        if (v == kPending) xw[o] = kQNaN;  // the walk ends, with NaNs
                        break;
                    }
                }
            }
            watch_walk(walk, (int32_t)t, ctl, limit, [&]() {
                for (int u = 0; u <= kWinBlocks; ++u)
                    if (xw[u * kWave + lane] == kPending) xw[u * kWave + lane] = kQNaN;
            });
            continue;
        }
        trace_mark_lane(trace, tr0 + i, has);
        int32_t q = 0, z = 0, w = 0;
        double s = 0.0, fii = 1.0;
        if (has) {
            const int32_t d = diagF[i];
            q = (int32_t)(kBackward ? rpF[i + 1] - 1 : rpF[i]);
            z = kBackward ? q - d : d - q;
            w = wcnt[i];
            s = in[i];
            if constexpr (kBackward) fii = F[d];
        }
        const int32_t outer = z - w;
        int32_t wmax = w, omax = outer;
        for (int off = 32; off > 0; off >>= 1) {
            wmax = max(wmax, __shfl_xor(wmax, off));
            omax = max(omax, __shfl_xor(omax, off));
        }
        wmax = uniform(wmax);
        // rounds of kOuterChunk; the rows end together, so that the values that
        // come last are in everyone's last round
        const int32_t orounds = (uniform(omax) + kOuterChunk - 1) / kOuterChunk;
        const int32_t pad = orounds * kOuterChunk - outer;
        // window entries to LDS; past the row's end +0.0 at the row's own place
        for (int32_t k0 = 0; k0 < wmax + 4; k0 += 4) {
            double f4[4];
            int32_t c4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                f4[u] = 0.0;
                c4[u] = i;
                if (k0 + u < w) {
                    const int32_t e = outer + k0 + u, sl = kBackward ? q - e : q + e;
                    f4[u] = F[sl];
                    c4[u] = ci[sl];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u < wmax + 4) {
                    fw[(k0 + u) * kWave + lane] = f4[u];
                    cw[(k0 + u) * kWave + lane] = c4[u] - wbase;
                }
        }
        if constexpr (!kBackward) s = sanitize_input(s, ctl);
        const double s0 = s;

        // outer entries, the next chunk's loaded before this one's values are waited for
        bool stop = false;
        double f[kOuterChunk], fn[kOuterChunk];
        int32_t c[kOuterChunk], cn[kOuterChunk];
        auto load = [&](int32_t k0) {
#pragma unroll
            for (int k = 0; k < kOuterChunk; ++k) {
                fn[k] = 0.0;
                cn[k] = 0;
                const int32_t x = k0 + k - pad;
                if (x >= 0 && x < outer) {
                    const int32_t sl = kBackward ? q - x : q + x;
                    fn[k] = F[sl];
                    cn[k] = ci[sl];
                }
            }
        };
        load(0);
        for (int32_t k0 = 0; k0 < orounds * kOuterChunk; k0 += kOuterChunk) {
            uint64_t v[kOuterChunk];
#pragma unroll
            for (int k = 0; k < kOuterChunk; ++k) {
                f[k] = fn[k];
                c[k] = cn[k];
            }
#pragma unroll
            for (int k = 0; k < kOuterChunk; ++k) v[k] = k0 + k >= pad ? ld_poll<Scope::Xcd>(out + c[k]) : 0ull;
            load(k0 + kOuterChunk);
            for (;;) {
                bool pend = false;
#pragma unroll
                for (int k = 0; k < kOuterChunk; ++k) pend |= v[k] == kPending;
                if (!__any(pend)) break;
                if (wait_expired(polls, t0, ctl, limit)) {
                    stop = true;
                    break;
                }
#pragma unroll
                for (int k = 0; k < kOuterChunk; ++k)
                    if (v[k] == kPending) v[k] = ld_poll<Scope::Xcd>(out + c[k]);
            }
            if (stop) break;
            polls = 0;
#pragma unroll
            for (int k = 0; k < kOuterChunk; ++k) s = s - f[k] * as_f64(v[k]);  // before the row's start +0.0 * +0.0
        }

        if (!kBackward && z == 0) s = s0;  // nothing to subtract: every bit stays

        // window: every lane walks its row, two entries a round
        int32_t e = 0;
        bool done = !has;
        uint64_t left = __ballot(has);  // rows not finished
        double f0 = fw[lane], f1 = fw[kWave + lane];
        int32_t c0 = cw[lane], c1 = cw[kWave + lane];
        if (lane == 0) *walk = 2 * (int32_t)t + 1;
        if (!stop) do {
            // the two entries after this round's, then the values of this round's
            const double* fp = fw + (e + 2) * kWave + lane;
            const int32_t* cp = cw + (e + 2) * kWave + lane;
            const double f2 = fp[0], f3 = fp[kWave];
            const int32_t c2 = cp[0], c3 = cp[kWave];
            __builtin_amdgcn_sched_barrier(0);
            const uint64_t v0 = xw[c0], v1 = xw[c1];
            const bool ok0 = e < w && v0 != kPending, ok1 = ok0 && e + 1 < w && v1 != kPending;
            const double s1 = s - f0 * as_f64(v0);
            const double s2 = s1 - f1 * as_f64(v1);
            s = ok1 ? s2 : ok0 ? s1 : s;
            e += ok1 ? 2 : ok0 ? 1 : 0;
            f0 = ok1 ? f2 : ok0 ? f1 : f0;
            c0 = ok1 ? c2 : ok0 ? c1 : c0;
            f1 = ok1 ? f3 : ok0 ? f2 : f1;
            c1 = ok1 ? c3 : ok0 ? c2 : c1;
            const bool fin = !done && e == w;
            const uint64_t m = __ballot(fin);
            if (m) {
                const double r = kBackward ? s / fii : s;
                if (fin) {
                    xw[kOwn + lane] = as_u64(r);
                    st_final<Scope::Xcd>(out + i, r);
                    trace_mark_lane(trace, tr0 + n + i, true);
                }
                done = done || fin;
            }
            left &= ~m;
        } while (left);
        if (lane == 0) *walk = 2 * (int32_t)t + 2;
        if (stop && !done) st_final<Scope::Xcd>(out + i, as_f64(kQNaN));
    }
}

hipError_t launch_solve_blocks(const PatDev& P, const uint8_t* wcnt, const double* f_val, const double* in, double* out,
                               bool backward, int32_t grid, Ctl* ctl, uint64_t spin_limit, hipStream_t s) {
    if (P.n <= 0) return hipSuccess;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid * kXcds), dim3(2 * kWave), 0, s, P.n, P.rpF, P.ciF, P.diagF, wcnt, f_val, in,
                           out, ctl, spin_limit, P.trace);
    };
    backward ? go(k_solve_blocks<true>) : go(k_solve_blocks<false>);
    return hipGetLastError();
}

}  // namespace tpilu
