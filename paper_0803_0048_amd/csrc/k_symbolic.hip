// Phase I on gfx950: the level-of-fill pattern (Def. 2.3, Algorithm 1), the
// map from A's entries to F's slots, and the per-row update schedule that
// Phase II replays.
//
// Algorithm 1 merges rows in ascending order, so row j can only be built
// after every row it pivots on.  On the GPU every row is built on its own,
// from the graph of A, using the fill-path form of the same levels: level(i,j)
// equals the least number of interior vertices of a path i -> j in the graph
// of A (edge u -> v for every stored a_uv) whose interior vertices are all
// smaller than min(i, j).  (Each term level(i,h) + level(h,j) + 1 of Def. 2.3
// joins a path to h and a path from h through vertex h itself, which is
// smaller than both ends.)  Algorithm 1 only minimises over entries that are
// themselves kept, but a path through an entry of level > k is already too
// long, so the two agree on every entry of level <= k.  Rows are therefore
// independent (the observation Sec. 3.3 makes for k = 1 holds for every k in
// this form) and one wavefront builds one row:
//
//   frontier_1 = { (v, v) : a_iv stored, v < i }      (vertex, largest interior)
//   depth d = 1..k:  every (v, M) in frontier_d and stored a_vj with j > M
//                    gives entry (i, j) a level candidate d;
//                    frontier_{d+1} = { (w, max(M, w)) : a_vw stored, w < i },
//                    keeping per w the smallest M, and dropping w when a
//                    shorter walk already reached it with an interior maximum
//                    no larger (that state can only lead to higher levels).
//   level 0 for every stored a_ij.
//
// Per-row sets live in LDS hash maps; a row that does not fit is redone by
// the same code with the maps in global memory sized for any row.
#include "kernels.h"

namespace tpilu {

// ------------------------------------------------------------------------------------
// validation
// ------------------------------------------------------------------------------------
__global__ void k_validate(int32_t n, int64_t nnz, const int64_t* __restrict__ rp,
                           const int32_t* __restrict__ ci, uint32_t* status) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i > n) return;
    uint32_t bad = 0;
    if (i == 0 && rp[0] != 0) bad |= kValBadRowptr;
    if (i == n) {
        if (rp[n] != nnz) bad |= kValBadRowptr;
    } else {
        int64_t a = rp[i], b = rp[i + 1];
        if (a > b || a < 0 || b > nnz) {
            bad |= kValBadRowptr;
        } else {
            bool diag = false;
            int32_t prev = -1;
            for (int64_t p = a; p < b; ++p) {
                int32_t c = ci[p];
                if (c < 0 || c >= n) { bad |= kValBadCol; break; }
                if (c <= prev) bad |= kValUnsorted;
                if (c == i) diag = true;
                prev = c;
            }
            if (!diag) bad |= kValNoDiag;
        }
    }
    if (bad) atomicOr(status, bad);
}

hipError_t launch_validate(int32_t n, int64_t nnz, const int64_t* rp, const int32_t* ci,
                           uint32_t* status, hipStream_t s) {
    int64_t threads = (int64_t)n + 1;
    int blocks = (int)((threads + 255) / 256);
    hipLaunchKernelGGL(k_validate, dim3(blocks), dim3(256), 0, s, n, nnz, rp, ci, status);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// hash maps (open addressing, linear probing) keyed by a vertex, value = min
// ------------------------------------------------------------------------------------
constexpr int32_t kEmpty = -1;
constexpr int32_t kBig = 0x7fffffff;

__device__ __forceinline__ uint32_t hslot(int32_t key, uint32_t mask) {
    uint32_t h = static_cast<uint32_t>(key) * 0x9E3779B1u;
    h ^= h >> 15;
    return h & mask;
}

// insert key (if absent) and lower its value to min(value, val); false if full
__device__ __forceinline__ bool map_min(int32_t* keys, int32_t* vals, uint32_t mask, int32_t key,
                                        int32_t val) {
    uint32_t h = hslot(key, mask);
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        int32_t old = atomicCAS(&keys[h], kEmpty, key);
        if (old == kEmpty || old == key) {
            atomicMin(&vals[h], val);
            return true;
        }
        h = (h + 1) & mask;
    }
    return false;
}

// map_min on the endpoint map of an LDS tier: an insert that finds no slot
// within kProbeMax probes fails, which the row then reports as overflowing
// (and the next tier builds it).  A linear-probing table near full makes
// every probe sequence long; giving up early keeps a row that will not fit
// from paying for a full table.
constexpr uint32_t kProbeMax = 64;
__device__ __forceinline__ bool map_min_bounded(int32_t* keys, int32_t* vals, uint32_t mask, int32_t key,
                                                int32_t val, uint32_t max_probe) {
    uint32_t h = hslot(key, mask);
    const uint32_t lim = min(max_probe, mask + 1u);
    for (uint32_t probe = 0; probe < lim; ++probe) {
        int32_t old = atomicCAS(&keys[h], kEmpty, key);
        if (old == kEmpty || old == key) {
            atomicMin(&vals[h], val);
            return true;
        }
        h = (h + 1) & mask;
    }
    return false;
}

__device__ __forceinline__ int32_t map_get(const int32_t* keys, const int32_t* vals, uint32_t mask,
                                           int32_t key) {
    uint32_t h = hslot(key, mask);
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        int32_t k = keys[h];
        if (k == key) return vals[h];
        if (k == kEmpty) return kBig;
        h = (h + 1) & mask;
    }
    return kBig;
}

struct SymWs {
    int32_t *ek, *ev;  // endpoint map: column -> level
    int32_t *bk, *bv;  // best interior maximum per vertex over all depths so far
    int32_t *ck, *cv;  // candidates of the next frontier
    int32_t *fv[2], *fm[2];  // frontier lists (vertex, interior maximum)
    int32_t *ok, *ol;  // compacted row (column, level)
    int32_t* ctr;      // [0],[1] frontier sizes, [2] overflow, [3] output size
    uint32_t emask, fmask, fcap;
    uint32_t eprobe;   // most probes of an endpoint insert before the row counts as overflowing
    uint32_t* bm;      // LDS tiers: the space of ok, reused as a bitmap of bm_bits columns
    uint32_t bm_bits;  //   (0: the global tier, which sorts its compacted row instead)
};

constexpr int32_t kSymSortMax = 512;  // longest row the sorting network orders
constexpr int32_t kSymRankMax = 256;  // longest row ordered by counting smaller columns

// exclusive prefix sum over the wavefront's lanes
__device__ __forceinline__ int32_t wave_excl_sum(int32_t v, int32_t& total) {
    const int lane = lane_id();
    int32_t x = v;
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    total = __shfl(x, kWave - 1);
    return x - v;
}

// Write row i of F (column, level) in ascending column order straight from
// the endpoint map: the map's columns are marked in a bitmap over a window
// of bm_bits columns, each lane takes a block of the window's words, a
// prefix over the lanes' bit counts gives every block its first output
// position, and the lane emits its block's columns in order, looking each
// level up in the map.  Windows follow each other from the row's smallest
// column to its largest.  O(row + column range / 32), against the
// O(row log^2 row) of a sorting network.
__device__ __forceinline__ void sym_emit_sorted(int32_t i, const int64_t* __restrict__ rpF, int32_t* __restrict__ ciF,
                                uint8_t* __restrict__ lvF, int32_t* __restrict__ diagF, const SymWs& W) {
    const int lane = lane_id();
    int32_t cmin = kBig, cmax = -1;
    for (uint32_t sl = lane; sl <= W.emask; sl += kWave) {
        const int32_t c = W.ek[sl];
        if (c != kEmpty) {
            cmin = min(cmin, c);
            cmax = max(cmax, c);
        }
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        cmin = min(cmin, __shfl_xor(cmin, off));
        cmax = max(cmax, __shfl_xor(cmax, off));
    }
    const int64_t base = rpF[i];
    int64_t out = base;
    for (int64_t w0 = cmin; w0 <= cmax; w0 += W.bm_bits) {
        const int32_t span = (int32_t)min<int64_t>(W.bm_bits, (int64_t)cmax - w0 + 1);
        const int32_t nw = (span + 31) >> 5;
        for (int32_t x = lane; x < nw; x += kWave) W.bm[x] = 0u;
        wave_sync();
        for (uint32_t sl = lane; sl <= W.emask; sl += kWave) {
            const int32_t c = W.ek[sl];
            if (c != kEmpty && c >= w0 && c < w0 + span) {
                const int32_t o = (int32_t)(c - w0);
                atomicOr(&W.bm[o >> 5], 1u << (o & 31));
            }
        }
        wave_sync();
        const int32_t per = (nw + kWave - 1) / kWave;
        const int32_t wb = min(lane * per, nw), we = min(wb + per, nw);
        int32_t mine = 0;
        for (int32_t x = wb; x < we; ++x) mine += __popc(W.bm[x]);
        int32_t total = 0;
        int64_t r = out + wave_excl_sum(mine, total);
        for (int32_t x = wb; x < we; ++x) {
            uint32_t bits = W.bm[x];
            while (bits) {
                const int32_t b = __builtin_ctz(bits);
                bits &= bits - 1u;
                const int32_t c = (int32_t)(w0 + x * 32 + b);
                const int32_t lev = map_get(W.ek, W.ev, W.emask, c);
                ciF[r] = c;
                lvF[r] = static_cast<uint8_t>(min(lev, 255));
                if (c == i) diagF[i] = static_cast<int32_t>(r);
                ++r;
            }
        }
        out += total;
        wave_sync();
    }
}

// false: the row does not fit in the maps
__device__ __forceinline__ bool sym_row(int32_t i, const int64_t* __restrict__ rpA,
                                        const int32_t* __restrict__ ciA, int32_t k, int mode,
                                        int32_t* __restrict__ cnt, const int64_t* __restrict__ rpF,
                                        int32_t* __restrict__ ciF, uint8_t* __restrict__ lvF,
                                        int32_t* __restrict__ diagF, const SymWs& W) {
    const int lane = lane_id();
    for (uint32_t s = lane; s <= W.emask; s += kWave) { W.ek[s] = kEmpty; W.ev[s] = kBig; }
    for (uint32_t s = lane; s <= W.fmask; s += kWave) {
        W.bk[s] = kEmpty; W.bv[s] = kBig; W.ck[s] = kEmpty; W.cv[s] = kBig;
    }
    if (lane < 4) W.ctr[lane] = 0;
    wave_sync();
    const int64_t a0 = rpA[i], a1 = rpA[i + 1];
    for (int64_t p = a0 + lane; p < a1; p += kWave) {
        int32_t c = ciA[p];
        bool ok = map_min_bounded(W.ek, W.ev, W.emask, c, 0, W.eprobe);
        if (c < i) {
            int32_t slot = atomicAdd(&W.ctr[0], 1);
            if (slot < (int32_t)W.fcap) { W.fv[0][slot] = c; W.fm[0][slot] = c; }
            else ok = false;
            ok = map_min(W.bk, W.bv, W.fmask, c, c) && ok;
        }
        if (!ok) W.ctr[2] = 1;
    }
    wave_sync();
    int cur = 0;
    for (int32_t d = 1; d <= k; ++d) {
        const int32_t nf = uniform(min(W.ctr[cur], (int32_t)W.fcap));
        if (nf == 0 || uniform(W.ctr[2])) break;
        // endpoints reachable from this frontier in one more edge
        for (int32_t f = lane; f < nf; f += kWave) {
            if (W.ctr[2]) break;  // overflowing: the next tier builds this row
            int32_t v = (cur ? W.fv[1] : W.fv[0])[f], M = (cur ? W.fm[1] : W.fm[0])[f];
            for (int64_t p = rpA[v]; p < rpA[v + 1]; ++p) {
                int32_t j = ciA[p];
                if (j > M && !map_min_bounded(W.ek, W.ev, W.emask, j, d, W.eprobe)) {
                    W.ctr[2] = 1;
                    break;
                }
            }
        }
        if (d == k) break;
        wave_sync();
        if (uniform(W.ctr[2])) break;
        // next frontier
        for (int32_t f = lane; f < nf; f += kWave) {
            int32_t v = (cur ? W.fv[1] : W.fv[0])[f], M = (cur ? W.fm[1] : W.fm[0])[f];
            for (int64_t p = rpA[v]; p < rpA[v + 1]; ++p) {
                int32_t w = ciA[p];
                if (w < i && !map_min(W.ck, W.cv, W.fmask, w, max(M, w))) W.ctr[2] = 1;
            }
        }
        const int nxt = cur ^ 1;
        if (lane == 0) W.ctr[nxt] = 0;
        wave_sync();
        for (uint32_t s = lane; s <= W.fmask; s += kWave) {
            int32_t w = W.ck[s];
            if (w == kEmpty) continue;
            int32_t c = W.cv[s];
            W.ck[s] = kEmpty;
            W.cv[s] = kBig;
            if (c < map_get(W.bk, W.bv, W.fmask, w)) {
                bool ok = map_min(W.bk, W.bv, W.fmask, w, c);
                int32_t slot = atomicAdd(&W.ctr[nxt], 1);
                if (slot < (int32_t)W.fcap) { (nxt ? W.fv[1] : W.fv[0])[slot] = w; (nxt ? W.fm[1] : W.fm[0])[slot] = c; }
                else ok = false;
                if (!ok) W.ctr[2] = 1;
            }
        }
        wave_sync();
        cur = nxt;
    }
    wave_sync();
    if (uniform(W.ctr[2])) return false;
    if (W.bm_bits) {
        int32_t mine = 0;
        for (uint32_t sl = lane; sl <= W.emask; sl += kWave) mine += W.ek[sl] != kEmpty;
        for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
        if (mode == 0) {
            if (lane == 0) cnt[i] = mine;
            return true;
        }
        // long rows: through the bitmap; short ones: the sorting network
        // below costs less than a pass over the column range
        if (mine > kSymSortMax) {
            sym_emit_sorted(i, rpF, ciF, lvF, diagF, W);
            return true;
        }
    }
    // compact the row
    for (uint32_t s = lane; s <= W.emask; s += kWave) {
        int32_t c = W.ek[s];
        if (c != kEmpty) {
            int32_t idx = atomicAdd(&W.ctr[3], 1);
            W.ok[idx] = c;
            W.ol[idx] = W.ev[s];
        }
    }
    wave_sync();
    const int32_t len = uniform(W.ctr[3]);
    if (mode == 0) {
        if (lane == 0) cnt[i] = len;
        return true;
    }
    // short rows: every lane counts the columns smaller than its own, four to
    // a broadcast read.  (The network below takes len log^2 len / 64 dependent
    // exchanges: random banded n=160,000 ILU(2), rows of 164 entries, fill
    // pass of the 1,024-entry tier 6.0 ms; by counting, in the smaller tiers,
    // 2.0 ms.)
    if (W.bm_bits && len <= kSymRankMax) {
        if (lane < 3 && len + lane < ((len + 3) & ~3)) W.ok[len + lane] = kBig;
        wave_sync();
        const int64_t base = rpF[i];
        for (int32_t e0 = 0; e0 < len; e0 += kWave) {
            const int32_t key = e0 + lane < len ? W.ok[e0 + lane] : kBig;
            int32_t r = 0;
            for (int32_t x = 0; x < len; x += 4) {
                const int4 o = *reinterpret_cast<const int4*>(W.ok + x);
                r += (o.x < key) + (o.y < key) + (o.z < key) + (o.w < key);
            }
            if (key != kBig) {
                ciF[base + r] = key;
                lvF[base + r] = static_cast<uint8_t>(min(W.ol[e0 + lane], 255));
                if (key == i) diagF[i] = static_cast<int32_t>(base + r);
            }
        }
        return true;
    }
    // sort (column, level) by column: bitonic network over the next power of
    // two, padded with kBig (it fits: the map's capacity is a power of two)
    uint32_t np2 = 1;
    while (np2 < (uint32_t)len) np2 <<= 1;
    for (uint32_t e = len + lane; e < np2; e += kWave) { W.ok[e] = kBig; W.ol[e] = 0; }
    wave_sync();
    for (uint32_t kk = 2; kk <= np2; kk <<= 1) {
        for (uint32_t jj = kk >> 1; jj > 0; jj >>= 1) {
            for (uint32_t e = lane; e < np2; e += kWave) {
                const uint32_t f = e ^ jj;
                if (f > e) {
                    const int32_t a = W.ok[e], b = W.ok[f];
                    if ((a > b) == ((e & kk) == 0)) {
                        W.ok[e] = b;
                        W.ok[f] = a;
                        const int32_t la = W.ol[e];
                        W.ol[e] = W.ol[f];
                        W.ol[f] = la;
                    }
                }
            }
            wave_sync();
        }
    }
    const int64_t base = rpF[i];
    for (int32_t e = lane; e < len; e += kWave) {
        const int32_t key = W.ok[e];
        ciF[base + e] = key;
        lvF[base + e] = static_cast<uint8_t>(min(W.ol[e], 255));
        if (key == i) diagF[i] = static_cast<int32_t>(base + e);
    }
    return true;
}

// A tier's LDS maps: kEnd the capacity of the endpoint map (and of the
// compacted row), kFront of the frontier maps and lists.  A wavefront clears
// its maps for every row and walks A's rows with dependent loads, so the
// smallest maps that hold a row are the fastest twice over: least to clear,
// most wavefronts on a CU (kSymWaves).  7-point 64^3 ILU(1), count + fill:
// 3.5 ms with 1,024-entry maps for every row, 0.65 here; random banded
// n=160,000 ILU(2) 8.7 -> 3.3 ms.  The compacted row and the bitmap of
// the long rows take the place of the frontier maps, which are done by then.
// In the count pass a row that does not fit goes to the next tier's list.
template <int kEnd, int kFront>
__global__ __launch_bounds__(64) void k_sym_rows_lds(const int64_t* __restrict__ rpA,
                                                     const int32_t* __restrict__ ciA, int32_t k,
                                                     SymLists lists, int mode, int32_t* __restrict__ cnt,
                                                     const int64_t* __restrict__ rpF,
                                                     int32_t* __restrict__ ciF,
                                                     uint8_t* __restrict__ lvF,
                                                     int32_t* __restrict__ diagF, int tier) {
    constexpr int kOut = kEnd > 4 * kFront ? 2 * kEnd : 0;  // (column, level) when the frontier space is too small
    __shared__ int32_t ek[kEnd], ev[kEnd];
    __shared__ __attribute__((aligned(16))) int32_t front[8 * kFront];
    __shared__ __attribute__((aligned(16))) int32_t outsh[kOut ? kOut : 4];
    __shared__ int32_t ctr[4];
    SymWs W;
    W.ek = ek; W.ev = ev;
    W.bk = front; W.bv = front + kFront; W.ck = front + 2 * kFront; W.cv = front + 3 * kFront;
    W.fv[0] = front + 4 * kFront; W.fm[0] = front + 5 * kFront;
    W.fv[1] = front + 6 * kFront; W.fm[1] = front + 7 * kFront;
    W.ok = kOut ? outsh : front;
    W.ol = W.ok + kEnd;
    W.ctr = ctr;
    W.emask = kEnd - 1; W.fmask = kFront - 1; W.fcap = kFront;
    W.eprobe = kProbeMax;
    W.bm = reinterpret_cast<uint32_t*>(W.ok);
    W.bm_bits = (uint32_t)kEnd * 32u;
    const int32_t* list = lists.rows + (size_t)tier * lists.n;
    const int32_t n_rows = lists.count[tier];
    for (int32_t r = blockIdx.x; r < n_rows; r += gridDim.x) {
        const int32_t i = list[r];
        if (mode == 1 && lists.tier_of[i] != tier) continue;  // built by a later tier
        const bool fits = sym_row(i, rpA, ciA, k, mode, cnt, rpF, ciF, lvF, diagF, W);
        if (!fits && mode == 0 && lane_id() == 0) {
            lists.rows[(size_t)(tier + 1) * lists.n + atomicAdd(&lists.count[tier + 1], 1)] = i;
            lists.tier_of[i] = static_cast<uint8_t>(tier + 1);
        }
        wave_sync();
    }
}

__host__ __device__ size_t sym_global_scratch_ints(int32_t n, uint32_t gcap) {
    // ek ev (gcap) bk bv ck cv (gcap) f0v f0m f1v f1m (n) ok ol (gcap) ctr (4, padded)
    return (size_t)gcap * 8 + (size_t)n * 4 + 64;
}

__global__ __launch_bounds__(64) void k_sym_rows_global(int32_t n, const int64_t* __restrict__ rpA,
                                                        const int32_t* __restrict__ ciA, int32_t k,
                                                        SymLists lists, int mode, int32_t* __restrict__ cnt,
                                                        const int64_t* __restrict__ rpF,
                                                        int32_t* __restrict__ ciF,
                                                        uint8_t* __restrict__ lvF,
                                                        int32_t* __restrict__ diagF,
                                                        int32_t* gscratch, uint32_t gcap) {
    int32_t* base = gscratch + (size_t)blockIdx.x * sym_global_scratch_ints(n, gcap);
    SymWs W;
    W.ek = base; W.ev = base + gcap;
    W.bk = base + 2 * (size_t)gcap; W.bv = base + 3 * (size_t)gcap;
    W.ck = base + 4 * (size_t)gcap; W.cv = base + 5 * (size_t)gcap;
    W.ok = base + 6 * (size_t)gcap; W.ol = base + 7 * (size_t)gcap;
    int32_t* fl = base + 8 * (size_t)gcap;
    W.fv[0] = fl; W.fm[0] = fl + n; W.fv[1] = fl + 2 * (size_t)n; W.fm[1] = fl + 3 * (size_t)n;
    W.ctr = fl + 4 * (size_t)n;
    W.emask = gcap - 1; W.fmask = gcap - 1; W.fcap = (uint32_t)n;
    W.eprobe = gcap;  // sized for any row (gcap >= 2n + 2): never gives up
    W.bm = nullptr;
    W.bm_bits = 0;
    const int32_t* list = lists.rows + (size_t)kSymGlobal * lists.n;
    const int32_t n_rows = lists.count[kSymGlobal];
    for (int32_t r = blockIdx.x; r < n_rows; r += gridDim.x) {
        sym_row(list[r], rpA, ciA, k, mode, cnt, rpF, ciF, lvF, diagF, W);
        wave_sync();
    }
}

hipError_t launch_sym_rows(int tier, int32_t n, const int64_t* rpA, const int32_t* ciA, int32_t k,
                           const SymLists& lists, int mode, int32_t* cnt, const int64_t* rpF, int32_t* ciF,
                           uint8_t* lvF, int32_t* diagF, int32_t* gscratch, uint32_t gcap, int32_t grid,
                           hipStream_t s) {
    if (n <= 0 || grid <= 0) return hipSuccess;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64), 0, s, rpA, ciA, k, lists, mode, cnt, rpF, ciF, lvF, diagF, tier);
    };
    if (tier == 0) go(k_sym_rows_lds<128, 64>);
    else if (tier == 1) go(k_sym_rows_lds<512, 256>);
    else if (tier == kSymMid) go(k_sym_rows_lds<1024, 512>);
    else if (tier == kSymLong) go(k_sym_rows_lds<4096, 512>);
    else
        hipLaunchKernelGGL(k_sym_rows_global, dim3(grid), dim3(64), 0, s, n, rpA, ciA, k, lists, mode, cnt, rpF, ciF,
                           lvF, diagF, gscratch, gcap);
    return hipGetLastError();
}

// Routing of rows to the tiers before the count pass.  ub_i = |row i of A| +
// sum over stored a_ih, h < i, of the entries of row h right of h: every
// position of level <= 1 of row i is one of those terms (Def. 2.3 with one
// interior vertex), so for k = 1 it bounds the row's length, counting
// duplicates (k = 0: the row's length itself).  For k > 1 the length is
// guessed as ub k^2 / 2.  Rows whose ub passes the capacity of tier kSymMid
// go straight to the larger maps: built there they would only fill its map
// and be given up.  The routing only changes where a row is built, never what
// it holds (a row that a tier cannot hold goes on to the next).
__global__ void k_row_upper(int32_t n, const int64_t* __restrict__ rpA, const int32_t* __restrict__ ciA,
                            int32_t* __restrict__ nup) {
    const int32_t h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= n) return;
    int64_t lo = rpA[h], hi = rpA[h + 1];
    const int64_t end = hi;
    while (lo < hi) {  // first entry right of the diagonal
        const int64_t mid = (lo + hi) >> 1;
        if (ciA[mid] <= h) lo = mid + 1;
        else hi = mid;
    }
    nup[h] = (int32_t)(end - lo);
}

// most expected entries of a row that starts in a tier: half of tier 0's map,
// seven eighths of tier 1's (for k > 1 twice that, the guess being high for
// stencils), and kSymMid's limit on ub
constexpr int64_t kSymRoute0 = 64, kSymRoute1 = 448, kSymRouteMid = (1024 - 1024 / 8) * 5 / 4;

__global__ __launch_bounds__(256) void k_route_rows(int32_t n, const int64_t* __restrict__ rpA,
                                                    const int32_t* __restrict__ ciA,
                                                    const int32_t* __restrict__ nup, int32_t k, SymLists lists) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int tier = -1;
    if (i < n) {
        const int64_t a0 = rpA[i], a1 = rpA[i + 1];
        int64_t ub = a1 - a0;
        for (int64_t p = a0; k > 0 && p < a1 && ub <= kSymRouteMid; ++p) {
            const int32_t h = ciA[p];
            if (h >= i) break;
            ub += nup[h];
        }
        const int64_t guess = k > 1 ? ub * min(k, 64) * min(k, 64) / 2 : ub;
        tier = ub > kSymRouteMid ? kSymLong
               : guess <= kSymRoute0 ? 0
               : guess <= (k > 1 ? 2 * kSymRoute1 : kSymRoute1) ? 1 : kSymMid;
        lists.tier_of[i] = static_cast<uint8_t>(tier);
    }
    // one atomic per wavefront and tier
    for (int t = 0; t <= kSymLong; ++t) {
        const uint64_t m = __ballot(tier == t);
        if (!m) continue;
        int32_t at = 0;
        if (lane_id() == __builtin_ctzll(m)) at = atomicAdd(&lists.count[t], __popcll(m));
        at = __shfl(at, __builtin_ctzll(m));
        if (tier == t)
            lists.rows[(size_t)t * lists.n + at + __popcll(m & ((1ull << lane_id()) - 1ull))] = i;
    }
}

hipError_t launch_route_rows(int32_t n, const int64_t* rpA, const int32_t* ciA, int32_t* nup, int32_t k,
                             const SymLists& lists, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (k > 0) hipLaunchKernelGGL(k_row_upper, dim3((n + 255) / 256), dim3(256), 0, s, n, rpA, ciA, nup);
    hipLaunchKernelGGL(k_route_rows, dim3((n + 255) / 256), dim3(256), 0, s, n, rpA, ciA, nup, k, lists);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// exclusive scan int32 -> int64 (three passes, 1024 elements per block)
// ------------------------------------------------------------------------------------
constexpr int kScanTile = 1024;

size_t scan_tmp_elems(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile) + 1; }

__global__ __launch_bounds__(256) void k_scan_reduce(const int32_t* __restrict__ in, int64_t n,
                                                     int64_t* __restrict__ bsum) {
    __shared__ int64_t sh[256];
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t acc = 0;
    for (int e = threadIdx.x; e < kScanTile; e += 256) {
        int64_t idx = base + e;
        if (idx < n) acc += in[idx];
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(1024) void k_scan_blocks(int64_t* bsum, int64_t nb) {
    // exclusive scan of nb block sums in place; bsum[nb] = total
    __shared__ int64_t sh[1024];
    int64_t per = (nb + 1023) / 1024;
    int64_t lo = threadIdx.x * per, hi = min(nb, lo + per);
    int64_t acc = 0;
    for (int64_t e = lo; e < hi; ++e) acc += bsum[e];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 1; w < 1024; w <<= 1) {
        int64_t v = (int)threadIdx.x >= w ? sh[threadIdx.x - w] : 0;
        __syncthreads();
        sh[threadIdx.x] += v;
        __syncthreads();
    }
    int64_t run = threadIdx.x ? sh[threadIdx.x - 1] : 0;
    for (int64_t e = lo; e < hi; ++e) {
        int64_t v = bsum[e];
        bsum[e] = run;
        run += v;
    }
    if (threadIdx.x == 1023) bsum[nb] = sh[1023];
}

__global__ __launch_bounds__(256) void k_scan_final(const int32_t* __restrict__ in, int64_t n,
                                                    const int64_t* __restrict__ boff,
                                                    int64_t* __restrict__ out, int64_t nb) {
    __shared__ int64_t sh[256];
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int32_t v[4];
    int64_t loc = 0;
    for (int e = 0; e < 4; ++e) {
        int64_t idx = base + threadIdx.x * 4 + e;
        v[e] = idx < n ? in[idx] : 0;
        loc += v[e];
    }
    sh[threadIdx.x] = loc;
    __syncthreads();
    for (int w = 1; w < 256; w <<= 1) {
        int64_t t = (int)threadIdx.x >= w ? sh[threadIdx.x - w] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    int64_t run = boff[blockIdx.x] + (threadIdx.x ? sh[threadIdx.x - 1] : 0);
    for (int e = 0; e < 4; ++e) {
        int64_t idx = base + threadIdx.x * 4 + e;
        if (idx < n) out[idx] = run;
        run += v[e];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = boff[nb];
}

hipError_t launch_scan(const int32_t* in, int64_t n, int64_t* out, int64_t* tmp, hipStream_t s) {
    int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 0) {
        hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, s, tmp, (int64_t)0);
        hipLaunchKernelGGL(k_scan_final, dim3(1), dim3(256), 0, s, in, n, tmp, out, (int64_t)0);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(256), 0, s, in, n, tmp);
    hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, s, tmp, nb);
    hipLaunchKernelGGL(k_scan_final, dim3((unsigned)nb), dim3(256), 0, s, in, n, tmp, out, nb);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// A -> F slot map: sixteen lanes per row, each searching its entries in the
// sorted row of F (a thread merging two whole rows read them lane by lane in
// lines of its own: 0.24 ms against 0.035 at random banded n=160,000 ILU(2))
// ------------------------------------------------------------------------------------
constexpr int kA2fLanes = 16;
__global__ __launch_bounds__(256) void k_a2f(int32_t n, const int64_t* __restrict__ rpA,
                                             const int32_t* __restrict__ ciA, const int64_t* __restrict__ rpF,
                                             const int32_t* __restrict__ ciF, int32_t* __restrict__ a2f,
                                             uint32_t* status) {
    const int64_t stride = gridDim.x * (int64_t)(blockDim.x / kA2fLanes);
    for (int64_t i = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kA2fLanes; i < n; i += stride) {
        const int64_t qb = rpF[i], qe = rpF[i + 1], pe = rpA[i + 1];
        for (int64_t p = rpA[i] + threadIdx.x % kA2fLanes; p < pe; p += kA2fLanes) {
            const int32_t c = ciA[p];
            int64_t lo = qb, hi = qe;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (ciF[mid] < c) lo = mid + 1;
                else hi = mid;
            }
            if (lo < qe && ciF[lo] == c) {
                a2f[p] = static_cast<int32_t>(lo);
            } else {
                a2f[p] = -1;
                atomicOr(status, kValBadCol);
            }
        }
    }
}

hipError_t launch_a2f(int32_t n, const int64_t* rpA, const int32_t* ciA, const int64_t* rpF,
                      const int32_t* ciF, int32_t* a2f, uint32_t* status, hipStream_t s) {
    // (a launch holds fewer than 2^32 threads)
    const int64_t blocks = std::min<int64_t>(((int64_t)n * kA2fLanes + 255) / 256, 1 << 22);
    hipLaunchKernelGGL(k_a2f, dim3((unsigned)blocks), dim3(256), 0, s, n, rpA, ciA, rpF, ciF, a2f, status);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Update schedule.  For every pivot slot s = (j, h) of F (h < j), the pairs
// (q, p) with q the slot of f_ht in row h and p the slot of f_jt in row j,
// for every t > h stored in both rows, in ascending t.  Phase II replays them
// (f_jt <- f_jt - f_jh * f_ht); their number is the number of updates.
// One wavefront per row j; row j's columns are staged in LDS, and every
// candidate t of a pivot row is looked up among them.  Most candidates are no
// column of row j (random banded n=160,000 ILU(2): 1 in 35), so a lookup is two
// steps: a bit of a filter (the row's columns folded into 64 or more bits per
// column), and, for the few that pass, a search of the sorted columns.
// Those are queued in LDS in order and searched 64 at a time, all lanes busy.
// Candidates are loaded four wavefront-wide rounds ahead of their test; pivot
// rows of at most 8, 16 or 32 candidates share a round.  What bounds the
// kernel is the instructions per candidate: with a search of a column
// directory by every candidate Phase I's two passes took 2.2 ms at 7-point
// 64^3 ILU(1), 0.4 here; paper-scale ILU(1) (1,276 entries a row, 55 candidates
// per pair) one pass of 330 ms, 210 here.
// ------------------------------------------------------------------------------------
constexpr int kSchedAhead = 4;    // rounds of candidates loaded together
constexpr int kSchedQueue = 128;  // candidates that passed the filter, a ring
constexpr size_t kSchedStaticLds = kSchedQueue * 9 + kWave * 4;  // qt, qq, qp, pcnt of k_sched

// filter bits for rows of up to max_row entries (rows too long for the LDS
// beside a larger one get a small one, and search nearly every candidate)
static int32_t sched_filter_bits(int32_t max_row) {
    if (max_row > 16384) return 8192;
    int32_t bits = 2048;
    while (bits < 65536 && bits < 64 * (int64_t)max_row) bits <<= 1;
    return bits;
}

// Modes: 0 counts the pairs of every pivot slot (scount) and records its
// pivot's diagonal slot (lsd); 1 writes them at sptr (the scan of the
// counts); 2 does both in one pass: the counts as mode 0, and the pairs, in
// order, to a pool.  A wavefront takes the pool a chunk of pool.chunk pairs
// at a time (one atomic per chunk) and writes each round's pairs straight
// into its chunk; a run of one row's pairs inside one chunk is a segment
// (row, index of its first pair within the row, pool position, count),
// closed when the row ends or the chunk is full.  Atomics on one address cost
// about 25 ns each across the device: the chunks are about a wavefront's whole
// share, and a row's first segments have places of their own (an atomic for
// every row and smaller chunk: random banded n=160,000 ILU(2) 7.7 ms instead of 2.4).  k_sched_copy then moves
// each segment to sptr[first slot of its row] + that index.  If the pool or
// the segment list is too small, mode 2 raises *overflow and stops storing
// (the counts stay exact): the caller then runs mode 1.  Mode 3 only adds
// the sampled rows' pair count into sample[0] and their candidate count into
// sample[2] (rows j with j % stride == 0), to size the pool and to decide
// whether one pass pays.
// split > 1 (mode 3): each sampled row is shared by `split` wavefronts, each
// taking every split-th block of 64 pivots, so the few sampled rows still
// fill the device.
__global__ __launch_bounds__(64) void k_sched(int32_t n, const int64_t* __restrict__ rpF,
                                              const int32_t* __restrict__ ciF,
                                              const int32_t* __restrict__ diagF, int mode,
                                              int32_t* __restrict__ scount, int32_t* __restrict__ lsd,
                                              const int64_t* __restrict__ sptr,
                                              int32_t* __restrict__ sq, int32_t* __restrict__ sp,
                                              SchedPool pool, int32_t max_bits, int32_t stride,
                                              int32_t split) {
    extern __shared__ uint32_t sched_sh[];
    uint32_t* filter = sched_sh;                                          // [max_bits / 32]
    int32_t* colsj = reinterpret_cast<int32_t*>(sched_sh + max_bits / 32);  // [max_row]
    // the queue: column, slot in the pivot row, pivot (of the 64 at hand)
    __shared__ int32_t qt[kSchedQueue], qq[kSchedQueue];
    __shared__ uint8_t qp[kSchedQueue];
    __shared__ int32_t pcnt[kWave];
    const int lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    const bool counts = mode == 0 || mode == 2;
    int64_t cbase = -1;          // mode 2: pool position of the wavefront's chunk (-2: pool exhausted)
    int32_t used = 0, seg0 = 0;  // pairs used in the chunk; start of the open segment
    int64_t ncand = 0, nfound = 0;  // mode 3
    const int64_t nsampled = ((int64_t)n + stride - 1) / stride;
    for (int64_t task = blockIdx.x; task < nsampled * split; task += gridDim.x) {
        const int32_t j = (int32_t)((task / split) * stride);
        const int32_t part = (int32_t)(task % split);
        const int32_t rs = (int32_t)rpF[j], re = (int32_t)rpF[j + 1], dj = diagF[j];
        const int32_t len = re - rs;
        // mode 2: the open segment is [seg0, used) of the current chunk
        int64_t row_done = 0;  // pairs of this row in closed segments
        int32_t nseg = 0;      // closed segments
        auto close_seg = [&]() {
            if (cbase >= 0 && used > seg0) {
                // the row's first kSchedSegs segments have their places, the others draw one
                int64_t g = (int64_t)j * kSchedSegs + nseg;
                if (nseg >= kSchedSegs) {
                    unsigned long long a = 0;
                    if (lane == 0) a = atomicAdd(pool.ctr + 1, 1ull);
                    g = (int64_t)n * kSchedSegs + (int64_t)__shfl(a, 0);
                }
                if (g < pool.seg_cap) {
                    if (lane == 0) pool.seg[g] = make_longlong4(j, row_done, cbase + seg0, used - seg0);
                } else if (lane == 0) {
                    atomicOr(pool.overflow, 1u);
                }
                ++nseg;
                row_done += used - seg0;
            }
            seg0 = used;
        };
        if (counts)
            for (int32_t s = dj + lane; s < re; s += kWave) scount[s] = 0;
        // (a row of no pivots has nothing else to do)
        if (dj == rs) {
            if (mode == 2 && lane < kSchedSegs) pool.seg[(int64_t)j * kSchedSegs + lane].w = 0;
            continue;
        }
        int32_t logm = 11;
        while ((1 << logm) < max_bits && (1 << logm) < 64 * len) ++logm;
        const uint32_t mask = (1u << logm) - 1u;
        // neighbouring columns fall on neighbouring bits, and those a multiple
        // of the filter's size apart (the planes of a grid) on different ones
        auto fold = [&](int32_t t) { return ((uint32_t)t + ((uint32_t)t >> logm) * 67u) & mask; };
        for (int32_t w = lane; w < (1 << logm) / 32; w += kWave) filter[w] = 0u;
        wave_sync();
        for (int32_t e = lane; e < len; e += kWave) {
            const int32_t c = ciF[rs + e];
            colsj[e] = c;
            const uint32_t h = fold(c);
            atomicOr(&filter[h >> 5], 1u << (h & 31u));
        }
        wave_sync();
        int32_t top = 1;  // the largest power of two in len
        while (2 * top <= len) top *= 2;
        int64_t out = mode == 1 ? sptr[rs] : 0;  // the row's pairs follow each other
        int32_t head = 0, qn = 0;
        // search the first cnt candidates of the queue
        auto drain = [&](int32_t cnt) {
            wave_sync();
            const bool on = lane < cnt;
            const int32_t at = (head + lane) & (kSchedQueue - 1);
            const int32_t t = qt[at], q = qq[at];
            int32_t pos = 0;  // columns smaller than t
            for (int32_t h = top; h > 0; h >>= 1)
                if (pos + h <= len && colsj[pos + h - 1] < t) pos += h;
            const bool hit = on && pos < len && colsj[min(pos, len - 1)] == t;
            const uint64_t m = __ballot(hit);
            const int32_t c = __popcll(m), rank = __popcll(m & below);
            if (counts && hit) atomicAdd(&pcnt[qp[at]], 1);
            if (mode == 1) {
                if (hit) {
                    sq[out + rank] = q;
                    sp[out + rank] = rs + pos;
                }
                out += c;
            }
            if (mode == 3) nfound += c;
            if (mode == 2 && m && cbase != -2) {
                if (cbase < 0 || used + c > pool.chunk) {
                    close_seg();
                    unsigned long long a = 0;
                    if (lane == 0) a = atomicAdd(pool.ctr, (unsigned long long)pool.chunk);
                    a = __shfl(a, 0);
                    if (a + (unsigned long long)pool.chunk > (unsigned long long)pool.cap) {
                        if (lane == 0) atomicOr(pool.overflow, 1u);
                        cbase = -2;
                    } else {
                        cbase = (int64_t)a;
                    }
                    used = 0;
                    seg0 = 0;
                }
                if (cbase >= 0) {
                    if (hit) {
                        pool.q[cbase + used + rank] = q;
                        pool.p[cbase + used + rank] = rs + pos;
                    }
                    used += c;
                }
            }
            head = (head + cnt) & (kSchedQueue - 1);
            qn -= cnt;
            wave_sync();
        };
        auto test = [&](bool on, int32_t t, int32_t q, int32_t p) {
            const uint32_t h = fold(t);
            const bool pass = on && ((filter[h >> 5] >> (h & 31u)) & 1u);
            const uint64_t m = __ballot(pass);
            if (!m) return;
            if (pass) {
                const int32_t at = (head + qn + __popcll(m & below)) & (kSchedQueue - 1);
                qt[at] = t;
                qq[at] = q;
                qp[at] = (uint8_t)p;
            }
            qn += __popcll(m);
            if (qn >= kWave) drain(kWave);
        };
        for (int32_t s0 = rs + part * kWave; s0 < dj; s0 += kWave * split) {
            const int32_t np = min(kWave, dj - s0);
            int32_t pd = 0, pe = 0;  // this lane's pivot: its candidates' slots
            if (lane < np) {
                const int32_t h = colsj[s0 - rs + lane];
                const int32_t dh = diagF[h];
                pd = dh + 1;
                pe = (int32_t)rpF[h + 1];
                if (counts) lsd[s0 + lane] = dh;
            }
            pcnt[lane] = 0;
            wave_sync();
            if (mode == 3) ncand += pe - pd;
            const int shift = __any(pe - pd > 32) ? 6 : __any(pe - pd > 16) ? 5 : __any(pe - pd > 8) ? 4 : 3;
            int32_t tv[kSchedAhead], tq[kSchedAhead], tp[kSchedAhead];
            bool on[kSchedAhead];
            if (shift < 6) {
                // every pivot's candidates in one go, several pivots a round
                for (int32_t p0 = 0; p0 < np; p0 += kSchedAhead << (6 - shift)) {
#pragma unroll
                    for (int u = 0; u < kSchedAhead; ++u) {
                        tp[u] = p0 + (u << (6 - shift)) + (lane >> shift);
                        const int32_t a = __shfl(pd, tp[u] & (kWave - 1)), e = __shfl(pe, tp[u] & (kWave - 1));
                        tq[u] = (int32_t)((uint32_t)a + (uint32_t)(lane & ((1 << shift) - 1)));
                        on[u] = tp[u] < np && (uint32_t)tq[u] < (uint32_t)e;  // (lanes past the end can pass 2^31)
                        tv[u] = on[u] ? ciF[tq[u]] : 0;
                    }
#pragma unroll
                    for (int u = 0; u < kSchedAhead; ++u) test(on[u], tv[u], tq[u], tp[u]);
                }
            } else {
                int32_t p = 0;
                uint32_t q0 = __builtin_amdgcn_readlane(pd, 0), he = __builtin_amdgcn_readlane(pe, 0);
                while (p < np) {
#pragma unroll
                    for (int u = 0; u < kSchedAhead; ++u) {
                        while (p < np && q0 >= he) {
                            ++p;
                            q0 = __builtin_amdgcn_readlane(pd, p & (kWave - 1));
                            he = __builtin_amdgcn_readlane(pe, p & (kWave - 1));
                        }
                        tp[u] = p;
                        tq[u] = (int32_t)(q0 + (uint32_t)lane);
                        on[u] = p < np && (uint32_t)tq[u] < he;
                        tv[u] = on[u] ? ciF[tq[u]] : 0;
                        q0 += kWave;
                    }
#pragma unroll
                    for (int u = 0; u < kSchedAhead; ++u) test(on[u], tv[u], tq[u], tp[u]);
                }
            }
            if (qn > 0) drain(qn);
            if (counts && lane < np) scount[s0 + lane] = pcnt[lane];
            wave_sync();
        }
        if (mode == 2) {
            close_seg();
            if (lane >= nseg && lane < kSchedSegs) pool.seg[(int64_t)j * kSchedSegs + lane].w = 0;
        }
        wave_sync();
    }
    if (mode == 3) {
        for (int off = 32; off > 0; off >>= 1) ncand += __shfl_xor(ncand, off);
        if (lane == 0 && ncand) {
            atomicAdd(pool.sample, (unsigned long long)nfound);
            atomicAdd(pool.sample + 2, (unsigned long long)ncand);
        }
    }
}

// mode 2's segments to their places: one wavefront per segment
__global__ __launch_bounds__(64) void k_sched_copy(SchedPool pool, int64_t nseg, const int64_t* __restrict__ rpF,
                                                   const int64_t* __restrict__ sptr, int32_t* __restrict__ sq,
                                                   int32_t* __restrict__ sp) {
    const int lane = lane_id();
    for (int64_t g = blockIdx.x; g < nseg; g += gridDim.x) {
        const longlong4 d = pool.seg[g];
        if (d.w == 0) continue;
        const int64_t dst = sptr[rpF[d.x]] + d.y;
        for (int64_t e = lane; e < d.w; e += kWave) {
            sq[dst + e] = pool.q[d.z + e];
            sp[dst + e] = pool.p[d.z + e];
        }
    }
}

hipError_t launch_sched_copy(const SchedPool& pool, int64_t nseg, const int64_t* rpF, const int64_t* sptr,
                             int32_t* sq, int32_t* sp, hipStream_t s) {
    if (nseg <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(nseg, 65536);
    hipLaunchKernelGGL(k_sched_copy, dim3(grid), dim3(64), 0, s, pool, nseg, rpF, sptr, sq, sp);
    return hipGetLastError();
}

// a workgroup's LDS holds the columns of a row of max_row entries and the filter,
// the queue and the counts included (a little more ends the queue instead of
// failing the launch)
bool sched_row_fits(int32_t max_row) {
    return (size_t)std::max(max_row, 1) * sizeof(int32_t) + (size_t)sched_filter_bits(max_row) / 8 + kSchedStaticLds <=
           160 * 1024;
}

hipError_t launch_sched(int32_t n, const int64_t* rpF, const int32_t* ciF, const int32_t* diagF,
                        int mode, int32_t* scount, int32_t* lsd, const int64_t* sptr,
                        int32_t* sq, int32_t* sp, int32_t max_row, hipStream_t s, const SchedPool* pool,
                        int32_t stride) {
    const int32_t bits = sched_filter_bits(max_row);
    const size_t lds = (size_t)std::max(max_row, 1) * sizeof(int32_t) + (size_t)bits / 8;
    if (!sched_row_fits(max_row)) return hipErrorInvalidValue;
    stride = max(stride, 1);
    const int32_t split = mode == 3 ? kSchedSampleSplit : 1;
    const int64_t tasks = ((int64_t)n + stride - 1) / stride * split;
    int grid = (int)std::min<int64_t>(tasks, mode == 2 ? pool->waves : 8 * kSchedWaves);
    if (grid <= 0) return hipSuccess;
    const SchedPool none{};
    hipLaunchKernelGGL(k_sched, dim3(grid), dim3(64), lds, s, n, rpF, ciF, diagF, mode, scount, lsd, sptr, sq, sp,
                       pool ? *pool : none, bits, stride, split);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Target-major copy of the update schedule: for every F slot p of row j, the
// updates it receives (row-local slot of the pivot entry f_jh, slot of f_ht)
// in ascending h.  One wavefront per row.  mode 0 counts per slot into
// tcount; mode 1 fills, walking the pivots in ascending order so that each
// slot's list comes out sorted (a pivot updates distinct slots).
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_tsched(int32_t n, const int64_t* __restrict__ rpF,
                                               const int32_t* __restrict__ diagF,
                                               const int64_t* __restrict__ sptr,
                                               const int32_t* __restrict__ sq,
                                               const int32_t* __restrict__ sp, int mode,
                                               int32_t* __restrict__ tcount, const int64_t* __restrict__ tptr,
                                               int32_t* __restrict__ tsl, int32_t* __restrict__ tq) {
    extern __shared__ int64_t tsh[];
    const int lane = lane_id();
    for (int32_t j = blockIdx.x; j < n; j += gridDim.x) {
        const int64_t rs = rpF[j], re = rpF[j + 1], dj = diagF[j];
        const int32_t len = (int32_t)(re - rs), dl = (int32_t)(dj - rs);
        int64_t* Tp = tsh;                                  // [len] next place of each of the row's slots
        int64_t* Sp = tsh + len;                            // [dl + 1] sptr of its L slots
        int32_t* cur = reinterpret_cast<int32_t*>(tsh + len + dl + 1);  // [len] counts (mode 0)
        for (int32_t e = lane; e < len; e += kWave) {
            cur[e] = 0;
            if (mode == 1) Tp[e] = tptr[rs + e];
        }
        for (int32_t e = lane; e <= dl; e += kWave) Sp[e] = sptr[rs + e];
        wave_sync();
        if (mode == 0) {
            for (int64_t e = Sp[0] + lane; e < Sp[dl]; e += kWave) atomicAdd(&cur[sp[e] - rs], 1);
            wave_sync();
            for (int32_t e = lane; e < len; e += kWave) tcount[rs + e] = cur[e];
        } else {
            // the row's pairs 64 at a time, the next ones loading meanwhile; a
            // pivot updates distinct slots, so the pivots of a round take turns
            // in LDS alone (a pivot at a time with its loads: 1.13 ms at random
            // banded n=160,000 ILU(2), 0.71 here)
            const int64_t e1 = Sp[dl];
            int64_t e = Sp[0] + lane;
            int32_t h = 0, p = 0, q = 0;
            if (e < e1) {
                p = sp[e];
                q = sq[e];
            }
            for (int64_t e0 = Sp[0]; e0 < e1; e0 += kWave) {
                int32_t pn = 0, qn = 0;
                if (e + kWave < e1) {
                    pn = sp[e + kWave];
                    qn = sq[e + kWave];
                }
                const int64_t end = min(e0 + kWave, e1);
                for (;;) {
                    const int64_t lo = Sp[h], hi = Sp[h + 1];
                    if (e >= lo && e < min(hi, end)) {
                        const int64_t pos = Tp[p - rs];
                        Tp[p - rs] = pos + 1;
                        tsl[pos] = h;
                        tq[pos] = q;
                    }
                    wave_sync();
                    if (hi >= end) break;
                    ++h;
                }
                e += kWave;
                p = pn;
                q = qn;
            }
        }
        wave_sync();
    }
}

size_t tsched_lds_bytes(int32_t max_row, int32_t max_lrow) {
    return (size_t)max_row * 8 + ((size_t)max_lrow + 1) * 8 + (size_t)max_row * 4;
}

hipError_t launch_tsched(int32_t n, const int64_t* rpF, const int32_t* diagF, const int64_t* sptr,
                         const int32_t* sq, const int32_t* sp, int mode, int32_t* tcount, const int64_t* tptr,
                         int32_t* tsl, int32_t* tq, int32_t max_row, int32_t max_lrow, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const size_t lds = tsched_lds_bytes(std::max(max_row, 1), max_lrow);
    hipLaunchKernelGGL(k_tsched, dim3(std::min(n, 65536)), dim3(64), lds, s, n, rpF, diagF, sptr, sq, sp, mode,
                       tcount, tptr, tsl, tq);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// pattern statistics
// ------------------------------------------------------------------------------------
// (one atomic per wavefront and quantity, not per row: those took 0.12 ms at
// 160,000 rows, on one address)
__global__ __launch_bounds__(256) void k_stats(int32_t n, const int64_t* __restrict__ rpF,
                                               const int32_t* __restrict__ diagF, PatStats* st) {
    int32_t mrow = 0, ml = 0, mu = 0;
    int64_t nl = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t rs = rpF[i], re = rpF[i + 1], d = diagF[i];
        mrow = max(mrow, static_cast<int32_t>(re - rs));
        ml = max(ml, static_cast<int32_t>(d - rs));
        mu = max(mu, static_cast<int32_t>(re - d - 1));
        nl += d - rs;
    }
    for (int off = 32; off > 0; off >>= 1) {
        mrow = max(mrow, __shfl_xor(mrow, off));
        ml = max(ml, __shfl_xor(ml, off));
        mu = max(mu, __shfl_xor(mu, off));
        nl += __shfl_xor(nl, off);
    }
    if (lane_id() == 0) {
        atomicMax(&st->max_row, mrow);
        atomicMax(&st->max_lrow, ml);
        atomicMax(&st->max_upart, mu);
        atomicAdd(&st->nnz_l, static_cast<unsigned long long>(nl));
    }
}

hipError_t launch_stats(int32_t n, const int64_t* rpF, const int32_t* diagF, PatStats* st,
                        hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_stats, dim3(std::min((n + 255) / 256, 64)), dim3(256), 0, s, n, rpF, diagF, st);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// dependency levels: level_i = 1 + max level_h over the nodes h that node i
// depends on (-1 = not yet known).  Up to two independent graphs are walked in
// one launch (the forward and the backward DAG), alternate wavefronts taking
// nodes of either, so their two dependency chains overlap in time.
// ------------------------------------------------------------------------------------
// The dependencies of node i: mode 0 the strict lower part of row i of F,
// mode 1 the strict upper part, mode 2 entries [ptr[i], ptr[i+1]) of a
// column structure (idx = row indices).
__device__ __forceinline__ void dep_range(const DepGraph& G, int32_t i, int64_t& a, int64_t& b) {
    if (G.mode == 0) { a = G.ptr[i]; b = G.diag[i]; }
    else if (G.mode == 1) { a = G.diag[i] + 1; b = G.ptr[i + 1]; }
    else { a = G.ptr[i]; b = G.ptr[i + 1]; }
}

__device__ __forceinline__ int32_t ld_level(const int32_t* p) {
    const int32_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    jitter((uint32_t)v);
    return v;
}

// watchdog over polling rounds without progress; true = give up
__device__ __forceinline__ bool level_watchdog(uint32_t& polls, uint64_t& t0, Ctl* ctl, uint64_t limit) {
    ++polls;
    if ((polls & 31u) != 0u) return false;
    bool stop = (polls & 255u) == 0u && ld_u32_coherent(&ctl->abort) != 0u;
    const uint64_t now = wall_clock64();
    if (polls == 32u) {
        t0 = now;
    } else if (now - t0 > limit) {
        if (lane_id() == 0) {
            atomicOr(&ctl->status, kStTimeout);
            __hip_atomic_store(&ctl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        stop = true;
    }
    return __any(stop);
}

typedef __attribute__((address_space(3))) volatile int32_t LdsLevel;

// One node, one wavefront.  The maximum does not depend on order, so every
// round re-polls all of a chunk's unknown dependencies at once.
constexpr int kLevelPer = 4;  // dependencies per lane and chunk

// S == Scope::Xcd: every wavefront of the job runs on one XCD and the levels
// are stored with workgroup scope (they stay in that XCD's L2, where the
// agent-scope polls of the job's other wavefronts find them)
template <Scope S>
__device__ __forceinline__ void level_row(const DepGraph& G, int32_t* depth, Ctl* ctl, uint64_t limit, int32_t i) {
    const int lane = lane_id();
    int64_t a, b;
    dep_range(G, i, a, b);
    int32_t best = 0;
    bool stop = false;
    for (int64_t base = a; base < b && !stop; base += kWave * kLevelPer) {
        int32_t src[kLevelPer], dv[kLevelPer];
        bool need[kLevelPer];
#pragma unroll
        for (int u = 0; u < kLevelPer; ++u) {
            const int64_t q = base + u * kWave + lane;
            need[u] = q < b;
            src[u] = need[u] ? G.idx[q] : 0;
            dv[u] = need[u] ? __hip_atomic_load(depth + src[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT) : 0;
        }
        uint32_t polls = 0;
        uint64_t t0 = 0;
        for (;;) {
            bool pend = false;
#pragma unroll
            for (int u = 0; u < kLevelPer; ++u) {
                if (need[u]) {
                    if (dv[u] >= 0) {
                        best = max(best, dv[u]);
                        need[u] = false;
                    } else {
                        pend = true;
                    }
                }
            }
            if (!__any(pend)) break;
#pragma unroll
            for (int u = 0; u < kLevelPer; ++u)
                if (need[u]) dv[u] = ld_level(depth + src[u]);
            if (level_watchdog(polls, t0, ctl, limit)) {
                stop = true;
                break;
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) best = max(best, __shfl_xor(best, off));
    if (lane == 0) {
        jitter((uint32_t)i);
        if constexpr (S == Scope::Xcd)
            __hip_atomic_store(depth + i, best + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_store(depth + i, best + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// S == Scope::Xcd: each job elects its own XCD through its control block (the
// first of its workgroups to start names it); the job's workgroups elsewhere
// leave at once
template <Scope S>
__global__ __launch_bounds__(64) void k_depth(int32_t n, LevelJob j0, LevelJob j1, int32_t njobs, Ctl* ctl,
                                              uint64_t spin_limit) {
    const LevelJob J = (njobs > 1 && (blockIdx.x & 1)) ? j1 : j0;
    if constexpr (S == Scope::Xcd) {
        if (!xcd_member(J.tctl)) return;
    }
    for (;;) {
        const uint32_t t = wave_ticket(J.tctl);
        if (t >= (uint32_t)n) break;
        const int32_t i = J.desc ? n - 1 - (int32_t)t : (int32_t)t;
        level_row<S>(J.G, J.depth, ctl, spin_limit, i);
    }
}

// Lane per node: a ticket hands a wavefront 64 consecutive nodes (in the
// sweep's order), so the whole graph can be in flight at once and wide
// graphs are not throttled by the ticket.  A lane looks at its first
// kLaneBatch dependencies not known yet at a time, in whatever order they
// become known (a maximum), so that little is left when the last one comes;
// dependencies on the wavefront's own nodes (the chains of a
// stencil's grid lines) go through LDS.  The wavefront keeps looping until
// every lane published, so lanes that depend on other lanes of the same
// wavefront cannot deadlock.  Bound by one hand-off per level and the polls
// of the wavefronts that wait: one that has found nothing new watches a single
// value, up to kLaneWatch loads, before all its lanes look again (27-point
// 90^3 ILU(1), Phase I, 4096 wavefronts: 89 ms without, 53 / 35 / 32 with 4 /
// 16 / 64 loads; 2-D 400^2 ILU(1) 3.3 / 3.6 / 3.5 / 4.2).  Phase I with one
// load at a time, nothing through LDS and every lane polling -> here: 2-D
// 400^2 ILU(3) 7.5 -> 6.0 ms, 7-point 64^3 ILU(2) 14.4 -> 6.2 ms.
constexpr int kLaneBatch = 8;
constexpr int kLaneWatch = 16;

__global__ __launch_bounds__(64) void k_depth_lanes(int32_t n, LevelJob j0, LevelJob j1, int32_t njobs, Ctl* ctl,
                                                    uint64_t spin_limit) {
    __shared__ int32_t lvsh[kWave];
    LdsLevel* lv = (LdsLevel*)lvsh;
    const int lane = lane_id();
    const LevelJob J = (njobs > 1 && (blockIdx.x & 1)) ? j1 : j0;
    const int32_t* __restrict__ ciF = J.G.idx;
    for (;;) {
        const uint32_t t = wave_ticket(J.tctl);
        const int64_t r = (int64_t)t * kWave + lane;
        if ((int64_t)t * kWave >= n) break;
        const bool valid = r < n;
        const int32_t i = valid ? (J.desc ? n - 1 - (int32_t)r : (int32_t)r) : 0;
        const int32_t first = J.desc ? n - 1 - (int32_t)t * kWave : (int32_t)t * kWave;  // lane 0's node
        int64_t q = 0, b = 0;
        if (valid) dep_range(J.G, i, q, b);
        // the dependencies not known yet, 64 at a time
        auto window = [&](int64_t from) {
            return from >= b ? 0ull : b - from >= kWave ? ~0ull : (1ull << (b - from)) - 1ull;
        };
        uint64_t open = window(q);
        int32_t best = 0;
        bool done = !valid;
        lv[lane] = -1;
        uint32_t polls = 0;
        uint64_t t0 = 0;
        int idle = 0;
        // the first kLaneBatch dependencies not known yet; they stay as they are
        // until one of them has come
        int32_t id[kLaneBatch], c[kLaneBatch];
        bool fresh = true;
        auto level_of = [&](int32_t c) {
            const uint32_t x = (uint32_t)(J.desc ? first - c : c - first);  // its lane, if below 64
            int32_t v;
            if (x < (uint32_t)kWave) v = lv[x];
            else v = ld_level(J.depth + c);
            return v;
        };
        for (;;) {
            bool prog = false;
            if (!done) {
                if (fresh) {
                    uint64_t m = open;
#pragma unroll
                    for (int u = 0; u < kLaneBatch; ++u) {
                        id[u] = m ? __builtin_ctzll(m) : -1;
                        m &= m - 1ull;
                        c[u] = id[u] >= 0 ? ciF[q + id[u]] : first;
                    }
                    fresh = false;
                }
                int32_t v[kLaneBatch];  // all loads in flight together
#pragma unroll
                for (int u = 0; u < kLaneBatch; ++u) v[u] = id[u] >= 0 ? level_of(c[u]) : -1;
#pragma unroll
                for (int u = 0; u < kLaneBatch; ++u)
                    if (v[u] >= 0) {
                        best = max(best, v[u]);
                        open &= ~(1ull << id[u]);
                        prog = true;
                    }
                fresh = prog;
                if (open == 0ull) {
                    q += kWave;
                    open = window(q);
                    prog = true;
                    if (open == 0ull) {
                        jitter((uint32_t)i);
                        lv[lane] = best + 1;
                        __hip_atomic_store(J.depth + i, best + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        done = true;
                    }
                }
            }
            const uint64_t left = __ballot(!done);
            if (!left) break;
            if (__any(prog)) {
                polls = 0;
                idle = 0;
                continue;
            }
            // nothing new: watch the first waiting lane's dependency alone for a
            // while, longer each time
            const int f = __builtin_ctzll(left);
            const int64_t qw = q + (open ? __builtin_ctzll(open) : 0);
            const int32_t c = ciF[((int64_t)__builtin_amdgcn_readlane((int32_t)(qw >> 32), f) << 32) |
                                  (uint32_t)__builtin_amdgcn_readlane((int32_t)qw, f)];
            if ((uint32_t)(J.desc ? first - c : c - first) >= (uint32_t)kWave) {
                for (int w = min(4 << idle, kLaneWatch); w > 0 && uniform(ld_level(J.depth + c)) < 0; --w) {}
                idle = min(idle + 1, 3);
            }
            if (wait_expired(polls, t0, ctl, spin_limit)) {
                // the status tells; a level all the same, so that the order sorted
                // by level next still holds every node once
                if (!done)
                    __hip_atomic_store(J.depth + i, best + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
    }
}

// Block of 64 consecutive nodes per workgroup, a lane per node, for rows of F
// that depend on few of their near neighbours: the blocks follow each other in
// the sweep's order, so the chain has n / 64 hand-offs through one XCD's L2
// instead of one per level.  As in the substitutions by blocks (which also
// count the window entries, wcnt), far dependencies are taken in lockstep from
// memory, 8 loads in flight; those in the kWinBlocks nearest blocks and the
// block itself stand in LDS, where a second wavefront puts the neighbours'
// levels as they come.  The maximum does not depend on order, so a lane walks
// four strided parts of its window at a time.  Bound by one hand-off and the walk of
// each block.  Random banded n=160,000 ILU(2), both DAGs, beside the update
// schedule: 16.2 ms by a wavefront per node, 5.8 ms here (the whole of Phase I
// 27.6 -> 22.6 ms; ILU(1) 11.2 -> 9.3, ILU(0) 6.9 -> 4.0 ms).
// The two DAGs of a launch take alternate workgroups, which the dispatcher
// deals to the XCDs in turn: each elects an XCD of its own.
constexpr int kDepthSlots = 4;
constexpr int kDepthOuter = 8;

template <bool kBackward>
__device__ __forceinline__ void depth_blocks(int32_t n, const LevelJob& J, const uint8_t* __restrict__ wcnt, Ctl* ctl,
                                             uint64_t limit, int32_t* cw, LdsLevel* lw, uint32_t* sh_ticket,
                                             LdsWord32* walk) {
    const int32_t* __restrict__ ci = J.G.idx;
    const int lane = lane_id();
    const bool walker = uniform((int32_t)(threadIdx.x / kWave)) == 0;
    const int32_t nb = (n + kWave - 1) / kWave;
    // window-local place of the block itself and of its neighbours
    constexpr int kOwn = kBackward ? 0 : kWinBlocks * kWave;
    constexpr int kNear = kBackward ? kWave : 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) *sh_ticket = atomicAdd(&J.tctl->ticket, 1u);
        if (walker)
#pragma unroll
            for (int u = 0; u <= kWinBlocks; ++u) lw[u * kWave + lane] = -1;
        __syncthreads();
        const uint32_t t = __builtin_amdgcn_readfirstlane(*sh_ticket);
        if (t >= (uint32_t)nb) break;
        const int32_t b = kBackward ? nb - 1 - (int32_t)t : (int32_t)t;
        const int32_t base = b * kWave, i = base + lane;
        const bool has = i < n;
        const int32_t wbase = base - kOwn;  // node of window place 0
        uint32_t polls = 0;
        uint64_t t0 = 0;
        if (!walker) {
#pragma unroll
            for (int u = 0; u < kWinBlocks; ++u) {
                // farthest block first: it is complete first
                const int32_t o = kNear + (kBackward ? kWinBlocks - 1 - u : u) * kWave + lane;
                const int32_t r = wbase + o;
                int32_t v = r >= 0 && r < n ? -1 : 0;
                for (;;) {
                    const bool pend = v < 0;
                    if (!__any(pend)) break;
                    if (pend) {
                        v = ld_level(J.depth + r);
                        if (v >= 0) lw[o] = v;
                    }
                    if (wait_expired(polls, t0, ctl, limit)) {
                        if (v < 0) lw[o] = 0;  // the walk ends; the status tells
                        break;
                    }
                }
            }
            watch_walk(walk, (int32_t)t, ctl, limit, [&]() {
                for (int u = 0; u <= kWinBlocks; ++u)
                    if (lw[u * kWave + lane] < 0) lw[u * kWave + lane] = 0;
            });
            continue;
        }
        int32_t q = 0, z = 0, w = 0;
        if (has) {
            const int32_t d = J.G.diag[i];
            q = (int32_t)(kBackward ? J.G.ptr[i + 1] - 1 : J.G.ptr[i]);
            z = kBackward ? q - d : d - q;
            w = wcnt[i];
        }
        const int32_t outer = z - w;
        int32_t wmax = w, omax = outer;
        for (int off = 32; off > 0; off >>= 1) {
            wmax = max(wmax, __shfl_xor(wmax, off));
            omax = max(omax, __shfl_xor(omax, off));
        }
        wmax = uniform(wmax);
        const int32_t rounds = (uniform(omax) + kDepthOuter - 1) / kDepthOuter;
        for (int32_t k0 = 0; k0 < wmax; k0 += 8) {
            int32_t c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = k0 + u < w ? ci[kBackward ? q - (outer + k0 + u) : q + outer + k0 + u] : i;
#pragma unroll
            for (int u = 0; u < 8; ++u) cw[(k0 + u) * kWave + lane] = c[u] - wbase;
        }
        // outer dependencies, the last ones of every row in the last round
        int32_t best = 0;
        bool stop = false;
        const int32_t pad = rounds * kDepthOuter - outer;
        for (int32_t k0 = 0; k0 < rounds * kDepthOuter && !stop; k0 += kDepthOuter) {
            int32_t c[kDepthOuter], v[kDepthOuter];
#pragma unroll
            for (int k = 0; k < kDepthOuter; ++k) {
                const int32_t x = k0 + k - pad;
                c[k] = x >= 0 ? ci[kBackward ? q - x : q + x] : 0;
            }
#pragma unroll
            for (int k = 0; k < kDepthOuter; ++k) v[k] = k0 + k >= pad ? ld_level(J.depth + c[k]) : 0;
            for (;;) {
                bool pend = false;
#pragma unroll
                for (int k = 0; k < kDepthOuter; ++k) pend |= v[k] < 0;
                if (!__any(pend)) break;
                if (wait_expired(polls, t0, ctl, limit)) {
                    stop = true;
                    break;
                }
#pragma unroll
                for (int k = 0; k < kDepthOuter; ++k)
                    if (v[k] < 0) v[k] = ld_level(J.depth + c[k]);
            }
            polls = 0;
#pragma unroll
            for (int k = 0; k < kDepthOuter; ++k) best = max(best, v[k]);
        }
        int32_t e[kDepthSlots], c[kDepthSlots];
#pragma unroll
        for (int u = 0; u < kDepthSlots; ++u) {
            e[u] = u;
            c[u] = u < w ? cw[u * kWave + lane] : kOwn + lane;
        }
        bool done = !has;
        uint64_t left = __ballot(has);
        if (lane == 0) *walk = 2 * (int32_t)t + 1;
        if (!stop) do {
            int32_t cn[kDepthSlots], v[kDepthSlots];
#pragma unroll
            for (int u = 0; u < kDepthSlots; ++u) cn[u] = cw[(e[u] + kDepthSlots) * kWave + lane];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kDepthSlots; ++u) v[u] = lw[c[u]];
            bool more = false;
#pragma unroll
            for (int u = 0; u < kDepthSlots; ++u) {
                const bool ok = e[u] < w && v[u] >= 0;
                best = max(best, ok ? v[u] : 0);
                e[u] += ok ? kDepthSlots : 0;
                more |= e[u] < w;
                c[u] = ok && e[u] < w ? cn[u] : c[u];
            }
            const bool fin = !done && !more;
            const uint64_t m = __ballot(fin);
            if (m && fin) {
                jitter((uint32_t)i);
                lw[kOwn + lane] = best + 1;
                __hip_atomic_store(J.depth + i, best + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            done = done || fin;
            left &= ~m;
        } while (left);
        if (lane == 0) *walk = 2 * (int32_t)t + 2;
        if (stop && !done) __hip_atomic_store(J.depth + i, best + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

__global__ __launch_bounds__(128) void k_depth_blocks(int32_t n, LevelJob j0, LevelJob j1, Ctl* ctl,
                                                      uint64_t spin_limit) {
    // entries + one slot round past the last + the fill's rounding
    __shared__ int32_t cw[(kWinEntries + 2 * kDepthSlots) * kWave];
    __shared__ int32_t lwsh[(kWinBlocks + 1) * kWave];
    __shared__ uint32_t sh_ticket;
    const LevelJob J = (blockIdx.x & 1) ? j1 : j0;
    if (!xcd_member(J.tctl)) return;
    __shared__ int32_t sh_walk;
    LdsLevel* lw = (LdsLevel*)lwsh;
    LdsWord32* walk = (LdsWord32*)&sh_walk;
    if (threadIdx.x == 0) *walk = 0;
    if (J.desc) depth_blocks<true>(n, J, J.wcnt, ctl, spin_limit, cw, lw, &sh_ticket, walk);
    else depth_blocks<false>(n, J, J.wcnt, ctl, spin_limit, cw, lw, &sh_ticket, walk);
}

// Rows sorted by level (counting sort): hist, scan (shared scan kernel),
// scatter.  Every depth is in 1 .. n, also after a wait that ran out: each
// level kernel then stores 1 + the largest level that it saw.  The order inside a level is whatever the atomics give; any
// order that lists every level before the next is a valid schedule, and the
// results never depend on it.
__global__ void k_level_hist(int32_t n, const int32_t* __restrict__ depth, int32_t* hist, int32_t* most) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t d = i < n ? depth[i] : 0;
    if (i < n) atomicAdd(&hist[d - 1], 1);
    for (int off = 32; off > 0; off >>= 1) d = max(d, __shfl_xor(d, off));
    if (lane_id() == 0 && d > *(volatile int32_t*)most) atomicMax(most, d);
}

__global__ void k_level_scatter(int32_t n, const int32_t* __restrict__ depth,
                                const int64_t* __restrict__ off, int32_t* cursor, int32_t* perm) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t d = depth[i] - 1;
    perm[off[d] + atomicAdd(&cursor[d], 1)] = i;
}

hipError_t launch_level_order(int32_t n, const int32_t* depth, int32_t max_depth, int32_t* hist, int32_t* most,
                              int64_t* off, int64_t* scan_tmp, int32_t* perm, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_level_hist, dim3((n + 255) / 256), dim3(256), 0, s, n, depth, hist, most);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_scan(hist, max_depth, off, scan_tmp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_level_scatter, dim3((n + 255) / 256), dim3(256), 0, s, n, depth, off,
                       hist + max_depth, perm);
    return hipGetLastError();
}

hipError_t launch_depth_blocks(int32_t n, const LevelJob& j0, const LevelJob& j1, Ctl* ctl, uint64_t spin_limit,
                               int32_t grid, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_depth_blocks, dim3(grid * kXcds), dim3(2 * kWave), 0, s, n, j0, j1, ctl, spin_limit);
    return hipGetLastError();
}

hipError_t launch_depth(int32_t n, const LevelJob& j0, const LevelJob* j1, Ctl* ctl, uint64_t spin_limit,
                        int32_t grid, bool one_xcd, hipStream_t s) {
    if (n <= 0 || grid == 0) return hipSuccess;
    const int32_t njobs = j1 ? 2 : 1;
    const LevelJob b = j1 ? *j1 : j0;
    auto go = [&](auto kern, int32_t groups) {
        hipLaunchKernelGGL(kern, dim3(groups), dim3(64), 0, s, n, j0, b, njobs, ctl, spin_limit);
    };
    if (grid < 0) go(k_depth_lanes, -grid * njobs);
    else if (one_xcd) go(k_depth<Scope::Xcd>, grid * njobs * kXcds);
    else go(k_depth<Scope::Device>, grid * njobs);
    return hipGetLastError();
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int blocks = (int)std::min<int64_t>((n + 255) / 256, 16384);
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

}  // namespace tpilu
