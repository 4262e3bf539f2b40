// Krylov building blocks for right-preconditioned restarted GMRES and
// BiCGSTAB on gfx950.
//
// The paper keeps inner products sequential so that their bits do not depend
// on the number of threads (Sec. 3.5).  Here every reduction instead has one
// fixed shape that depends only on the vector length: 16384 lanes each sum a
// strided subsequence in ascending order from +0.0, then lanes are combined
// pairwise at strides 1, 2, 4, ..., 8192 (IEEE addition is commutative, so
// which lane of a pair does the add, or whether both do, does not matter).  The launch is
// 64 blocks x 256 threads = 16384 threads; strides 1..32 are combined inside a
// wavefront with shuffles, 64 and 128 through LDS, 256..8192 over the 64
// block partials by whichever kernel consumes the result.  SpMV sums every
// row from +0.0 in ascending column order.
#include "kernels.h"

namespace tpilu {

// Rows in tiles (row_products): a thread per row read its entries in lines of
// its own (random banded n=160,000, 11 entries a row: 19.3 us, about 7 here).
template <int kTile, int kRows>
__global__ __launch_bounds__(64) void k_spmv(int32_t n, const int64_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                             const double* __restrict__ v, const double* __restrict__ x,
                                             const double* __restrict__ b_minus, double* __restrict__ y) {
    __shared__ double tv[kRows * (kTile + 1)];
    row_products<kTile, kRows>(
        n, ci, v, x, tv,
        [&](int32_t i, int32_t& a, int32_t& b) {
            a = (int32_t)rp[i];
            b = (int32_t)rp[i + 1];
        },
        [&](int32_t i, double s) { y[i] = b_minus ? b_minus[i] - s : s; });
}

hipError_t launch_spmv(int32_t n, int64_t nnz, int32_t longest, const int64_t* rp, const int32_t* ci, const double* v,
                       const double* x, const double* b_minus, double* y, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    auto go = [&](auto kern, int rows) {
        const int grid = std::min((n + rows - 1) / rows, 65536);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64), 0, s, n, rp, ci, v, x, b_minus, y);
    };
    // 8, 16 or 32 entries a round (us a call, launch included, random banded
    // 11.2 / 10.7 / 12.9; 7-point 110^3 30.5 / 32.7 / 54.3; 27-point 50^3 16.5 /
    // 15.0 / 11.3)
    // and fewer for the shortest rows (1 / 4 / 8: diagonal n=8,000,000, nnz = n, 46 /
    // 69 / 101; bidiagonal n=4,000,000 34 / 32 / 38; tridiagonal n=1,000,000 14.5 /
    // 12.1 / 13.2), unless a long row sets the time (one of 6,000 entries 765 with
    // 4, 640 with 8, 351 with 32)
    const bool uneven = longest >= 1024 && (int64_t)longest * 64 >= nnz;
    if (nnz <= n) go(k_spmv<1, 64>, 64);
    else if (uneven) go(k_spmv<32, 16>, 16);
    else if (nnz <= 3 * (int64_t)n && longest <= 64) go(k_spmv<4, 64>, 64);
    else if (nnz <= 8 * (int64_t)n) go(k_spmv<8, 64>, 64);
    else if (nnz <= 20 * (int64_t)n) go(k_spmv<16, 32>, 32);
    else go(k_spmv<32, 16>, 16);
    return hipGetLastError();
}

template <int kCtrl>
__device__ __forceinline__ double dpp_move(double v) {
    const uint64_t u = as_u64(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), kCtrl, 0xf, 0xf, true);
    return as_f64(((uint64_t)hi << 32) | lo);
}

// pairwise tree over the 16 lanes of a row, strides 1, 2, 4, 8: every lane gets
// the sum (once the lanes of a quad, then of half a row, agree, a mirror image
// is as good as the lane a stride away)
__device__ __forceinline__ double row_tree(double s) {
    s = s + dpp_move<0xB1>(s);   // lane ^ 1
    s = s + dpp_move<0x4E>(s);   // lane ^ 2
    s = s + dpp_move<0x141>(s);  // 7 - lane, in the half row
    return s + dpp_move<0x140>(s);  // 15 - lane
}

// pairwise tree inside a wavefront, strides 1 .. 32 (every lane gets the sum)
__device__ __forceinline__ double wave_tree(double s) {
    s = row_tree(s);
    return (bcast_lane(s, 0) + bcast_lane(s, 16)) + (bcast_lane(s, 32) + bcast_lane(s, 48));
}

__global__ __launch_bounds__(256) void k_dot_partial(int64_t n, const double* __restrict__ x,
                                                     const double* __restrict__ y,
                                                     double* __restrict__ partial) {
    __shared__ double sh[4];
    const int64_t l = (int64_t)blockIdx.x * kDotThreads + threadIdx.x;
    double s = 0.0;
    for (int64_t e = l; e < n; e += kDotLanes) s = s + x[e] * y[e];
    s = wave_tree(s);
    const int wv = threadIdx.x / kWave;
    if (lane_id() == 0) sh[wv] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double a = sh[0] + sh[1];  // stride 64
        const double c = sh[2] + sh[3];
        partial[blockIdx.x] = a + c;     // stride 128
    }
}

// strides 256..8192: tree over the 64 block partials
__device__ __forceinline__ double tree64(const double* __restrict__ partial) {
    double p[kDotBlocks];
#pragma unroll
    for (int b = 0; b < kDotBlocks; ++b) p[b] = partial[b];
#pragma unroll
    for (int w = 1; w < kDotBlocks; w <<= 1) {
#pragma unroll
        for (int b = 0; b < kDotBlocks; b += 2 * w) p[b] = p[b] + p[b + w];
    }
    return p[0];
}

hipError_t launch_dot_partial(int64_t n, const double* x, const double* y, double* partial,
                              hipStream_t s) {
    hipLaunchKernelGGL(k_dot_partial, dim3(kDotBlocks), dim3(kDotThreads), 0, s, n, x, y, partial);
    return hipGetLastError();
}

__global__ void k_dot_final(const double* __restrict__ partial, double* out, int sqrt_it) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        double r = tree64(partial);
        if (sqrt_it) r = __builtin_sqrt(r);
        *out = r;
    }
}

hipError_t launch_dot_final(const double* partial, double* out, int sqrt_it, hipStream_t s) {
    hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(64), 0, s, partial, out, sqrt_it);
    return hipGetLastError();
}

// scalar of a finished reduction, computed once per block and broadcast
__device__ __forceinline__ double block_scalar(const double* partial, int sqrt_it) {
    __shared__ double sc;
    if (threadIdx.x == 0) {
        double r = tree64(partial);
        sc = sqrt_it ? __builtin_sqrt(r) : r;
    }
    __syncthreads();
    return sc;
}

// The rotation that zeroes b against a: rho = sqrt(a*a + b*b) (each product
// and the sum rounded on its own, no hypot), c = a / rho, s = b / rho, all
// correctly rounded binary64 operations.
struct Rotation {
    double rho, c, s;
};
__device__ __forceinline__ Rotation givens_rotation(double a, double b) {
    Rotation r;
    r.rho = __builtin_sqrt(a * a + b * b);
    r.c = a / r.rho;
    r.s = b / r.rho;
    return r;
}

// The step's outcome to the host, which polls the slot for the step's number.
__device__ __forceinline__ void gm_report(const GmStep& a, int32_t iters, int32_t stop) {
    if (threadIdx.x != 0) return;
    volatile int32_t* slot = gm_report_slot(a.flags, a.seq);
    slot[0] = iters;
    slot[1] = stop;
    slot[2] = (int32_t)ld_u32_coherent(&a.ctl->status);
    __hip_atomic_store(const_cast<int32_t*>(slot) + 3, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Givens, by one workgroup: apply rotations 0..j-1 to column j of H, form
// rotation j, update g, count the iteration and decide whether the cycle stops
// (|g_{j+1}| <= tol, maxit reached, or breakdown).  H is (m+1) x m, row-major:
// H[i * m + j].  hn = h_{j+1,j}.  The chain runs in one thread, its operands
// through LDS (from memory it took 3 to 5 us).
__device__ __forceinline__ void gm_givens(const GmStep& a, double hn) {
    constexpr int kPart = 256;
    __shared__ double hc[kPart], rc[kPart], rsn[kPart];
    const int t = threadIdx.x;
    const int32_t m = a.m, j = a.j;
    __syncthreads();  // column j of H is there
    double run = a.H[j];
    for (int32_t i0 = 0; i0 < j; i0 += kPart) {
        const int32_t cnt = min(kPart, j - i0);
        if (t < cnt) {
            hc[t] = a.H[(int64_t)(i0 + t + 1) * m + j];
            rc[t] = a.cs[i0 + t];
            rsn[t] = a.sn[i0 + t];
        }
        __syncthreads();
        if (t == 0)
            for (int32_t i = 0; i < cnt; ++i) {
                const double x = hc[i], c = rc[i], s = rsn[i];
                hc[i] = c * run + s * x;
                run = c * x - s * run;
            }
        __syncthreads();
        if (t < cnt) a.H[(int64_t)(i0 + t) * m + j] = hc[t];
        __syncthreads();
    }
    if (t != 0) return;
    const Rotation rot = givens_rotation(run, hn);
    a.cs[j] = rot.c;
    a.sn[j] = rot.s;
    a.H[(int64_t)j * m + j] = rot.rho;
    a.H[(int64_t)(j + 1) * m + j] = 0.0;
    const double gj = a.g[j], gn = -rot.s * gj;
    a.g[j + 1] = gn;
    a.g[j] = rot.c * gj;
    const int32_t it = *a.iters;
    const double res = __builtin_fabs(gn);
    if (a.hist) a.hist[it] = res;
    *a.iters = it + 1;
    const int32_t stop = (res <= a.tol || it + 1 >= a.maxit || hn == 0.0) ? 1 : 0;
    a.iters[1] = stop;
    gm_report(a, it + 1, stop);
}

// h = <w, v> (from its partials); H slot <- h; w <- w - h v; then the partials
// of <w, vn> (vn null: of <w, w>), for the next step: a launch per MGS step.
// Every lane of the fixed shape owns its elements, so what it subtracts is
// what it sums next.  The loads of kGmAhead elements are in flight together
// (64 x 256 threads are few).  n=160,000: a dot and an axpy launch 5.7 + 4.9
// us, 4.7 here.
constexpr int kGmAhead = 8;
__global__ __launch_bounds__(256) void k_gm_axpy_dot(int64_t n, const int32_t* __restrict__ iters,
                                                     const double* __restrict__ pin, double* hslot,
                                                     double* __restrict__ w, const double* __restrict__ v,
                                                     const double* vn, double* __restrict__ pout) {
    __shared__ double sh[4];
    if (iters[1]) return;
    const double h = block_scalar(pin, 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) *hslot = h;
    double s = 0.0;
    for (int64_t e0 = (int64_t)blockIdx.x * kDotThreads + threadIdx.x; e0 < n; e0 += (int64_t)kGmAhead * kDotLanes) {
        double x[kGmAhead], y[kGmAhead], z[kGmAhead];
#pragma unroll
        for (int u = 0; u < kGmAhead; ++u) {
            const int64_t e = e0 + (int64_t)u * kDotLanes;
            x[u] = y[u] = z[u] = 0.0;
            if (e < n) {
                x[u] = w[e];
                y[u] = v[e];
                if (vn) z[u] = vn[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kGmAhead; ++u) {
            const int64_t e = e0 + (int64_t)u * kDotLanes;
            if (e < n) {
                const double r = x[u] - h * y[u];
                w[e] = r;
                s = s + r * (vn ? z[u] : r);
            }
        }
    }
    s = wave_tree(s);
    if (lane_id() == 0) sh[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double a = sh[0] + sh[1];
        const double c = sh[2] + sh[3];
        pout[blockIdx.x] = a + c;
    }
}

// h_{j+1,j} = ||w||; v_{j+1} = w / h_{j+1,j} when it is not zero; block 0 also
// applies the rotations
__global__ __launch_bounds__(256) void k_gm_finish(GmStep a, const double* __restrict__ partial) {
    if (a.iters[1]) {
        if (blockIdx.x == 0) gm_report(a, *a.iters, 1);
        return;
    }
    const double hn = block_scalar(partial, 1);
    double* vnext = a.V + (int64_t)(a.j + 1) * a.n;
    if (hn != 0.0)
        for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < a.n;
             e += (int64_t)gridDim.x * blockDim.x)
            vnext[e] = a.w[e] / hn;
    // (a block that starts after this may find the cycle stopped: v_{j+1} is then not used)
    if (blockIdx.x == 0) gm_givens(a, hn);
}

// The fixed-shape sum of one value per lane of the shape, lanes 1024 C .. being
// +0.0 (no sum of lanes that start from +0.0 is -0.0, so adding them changes
// nothing): thread t holds lanes C t .. C t + C - 1, so the first strides are
// its own; the strides inside the wavefront move through the VALU (shuffles
// through LDS took twice as long), and every wavefront sums the 16 wavefront
// sums for itself after the one barrier.  All threads get the sum.
template <int C>
__device__ __forceinline__ double gm_sum(const double (&in)[C], double* sh) {
    double p[C];
#pragma unroll
    for (int c = 0; c < C; ++c) p[c] = in[c];
#pragma unroll
    for (int w = 1; w < C; w <<= 1)
#pragma unroll
        for (int c = 0; c < C; c += 2 * w) p[c] = p[c] + p[c + w];
    const double s = wave_tree(p[0]);
    if (lane_id() == 0) sh[threadIdx.x / kWave] = s;
    __syncthreads();
    return bcast_lane(row_tree(sh[lane_id() & 15]), 0);
}

// A whole Arnoldi step of a small system in one workgroup: all MGS steps, the
// norm, v_{j+1} and the rotations; w stays in registers, the next v loads
// while the sum of this one goes through its stages.  Bound by those stages,
// about 1 us each (4,096 rows, 16 columns on average: 17 us a step, 26 with the
// sums through LDS shuffles; with a
// launch for every sum and every axpy about 110).
template <int C>
__global__ __launch_bounds__(1024) void k_gm_step(GmStep a) {
    __shared__ double sh[2][16];
    if (a.iters[1]) {  // the cycle stopped: this step was launched ahead
        gm_report(a, *a.iters, 1);
        return;
    }
    const int32_t n = (int32_t)a.n, e0 = (int32_t)threadIdx.x * C;
    double w[C], v[C], vn[C], p[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        w[c] = e0 + c < n ? a.w[e0 + c] : 0.0;
        v[c] = e0 + c < n ? a.V[e0 + c] : 0.0;
        vn[c] = 0.0;
    }
    for (int32_t i = 0; i <= a.j; ++i) {
        const double* __restrict__ next = a.V + (int64_t)(i + 1) * n;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (i < a.j && e0 + c < n) vn[c] = next[e0 + c];
            p[c] = 0.0 + w[c] * v[c];
        }
        const double h = gm_sum<C>(p, sh[i & 1]);
        if (threadIdx.x == 0) a.H[(int64_t)i * a.m + a.j] = h;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            w[c] = e0 + c < n ? w[c] - h * v[c] : 0.0;
            v[c] = vn[c];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) p[c] = 0.0 + w[c] * w[c];
    const double hn = __builtin_sqrt(gm_sum<C>(p, sh[(a.j + 1) & 1]));
    if (hn != 0.0) {
        double* vnext = a.V + (int64_t)(a.j + 1) * n;
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (e0 + c < n) vnext[e0 + c] = w[c] / hn;
    }
    gm_givens(a, hn);
}

hipError_t launch_gm_step(const GmStep& a, double* partial, hipStream_t s) {
    if (a.n <= kGmSmall) {
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(1), dim3(1024), 0, s, a); };
        if (a.n <= 1024) go(k_gm_step<1>);
        else if (a.n <= 2048) go(k_gm_step<2>);
        else if (a.n <= 4096) go(k_gm_step<4>);
        else go(k_gm_step<8>);
        return hipGetLastError();
    }
    hipError_t e = launch_dot_partial(a.n, a.w, a.V, partial, s);
    for (int32_t i = 0; e == hipSuccess && i <= a.j; ++i) {
        // all blocks read one set of partials while they write the other
        double *pin = partial + (i & 1) * kDotBlocks, *pout = partial + ((i + 1) & 1) * kDotBlocks;
        const double* v = a.V + (int64_t)i * a.n;
        hipLaunchKernelGGL(k_gm_axpy_dot, dim3(kDotBlocks), dim3(kDotThreads), 0, s, a.n, a.iters, pin,
                           a.H + (int64_t)i * a.m + a.j, a.w, v, i < a.j ? v + a.n : nullptr, pout);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    const int blocks = (int)std::min<int64_t>((a.n + 255) / 256, 2048);
    hipLaunchKernelGGL(k_gm_finish, dim3(blocks), dim3(256), 0, s, a, partial + ((a.j + 1) & 1) * kDotBlocks);
    return hipGetLastError();
}

// cycle start: beta = ||r||, g_0 = beta, v_0 = r / beta
__global__ __launch_bounds__(256) void k_gm_start(int64_t n, const double* __restrict__ partial,
                                                  double* beta_slot, double* g0, int32_t* stop,
                                                  const double* __restrict__ r,
                                                  double* __restrict__ v0) {
    const double beta = block_scalar(partial, 1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *beta_slot = beta;
        *g0 = beta;
        *stop = 0;
    }
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        v0[e] = r[e] / beta;
}

hipError_t launch_gm_start(int64_t n, const double* partial, double* beta_slot, double* g0, int32_t* stop,
                           const double* r, double* v0, hipStream_t s) {
    int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 2048));
    hipLaunchKernelGGL(k_gm_start, dim3(blocks), dim3(256), 0, s, n, partial, beta_slot, g0, stop, r, v0);
    return hipGetLastError();
}

__global__ void k_givens_batch(int64_t n, const double* __restrict__ a, const double* __restrict__ b,
                               double* rho, double* c, double* s) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const Rotation r = givens_rotation(a[i], b[i]);
        rho[i] = r.rho;
        c[i] = r.c;
        s[i] = r.s;
    }
}

hipError_t launch_givens_batch(int64_t n, const double* a, const double* b, double* rho, double* c, double* s,
                               hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_givens_batch, dim3(blocks), dim3(256), 0, st, n, a, b, rho, c, s);
    return hipGetLastError();
}

// back substitution H(0:jj, 0:jj) y = g, i descending, running subtraction
// in ascending l
__global__ void k_gm_backsub(const double* H, const double* g, double* yv, int32_t m, int32_t jj) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    for (int32_t i = jj - 1; i >= 0; --i) {
        double s = g[i];
        for (int32_t l = i + 1; l < jj; ++l) s = s - H[i * m + l] * yv[l];
        yv[i] = s / H[i * m + i];
    }
}

hipError_t launch_gm_backsub(const double* H, const double* g, double* yv, int32_t m, int32_t jj,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_gm_backsub, dim3(1), dim3(64), 0, s, H, g, yv, m, jj);
    return hipGetLastError();
}

// u_e = sum_i y_i v_{i,e}, from +0.0 in ascending i
__global__ void k_gm_combine(int64_t n, const double* __restrict__ V, const double* __restrict__ yv,
                             int32_t jj, double* __restrict__ u) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int32_t i = 0; i < jj; ++i) s = s + yv[i] * V[(int64_t)i * n + e];
        u[e] = s;
    }
}

hipError_t launch_gm_combine(int64_t n, const double* V, const double* yv, int32_t jj, double* u,
                             hipStream_t s) {
    int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_gm_combine, dim3(blocks), dim3(256), 0, s, n, V, yv, jj, u);
    return hipGetLastError();
}

__global__ void k_axpy1(int64_t n, double* __restrict__ x, const double* __restrict__ z) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        x[e] = x[e] + z[e];
}

hipError_t launch_axpy1(int64_t n, double* x, const double* z, hipStream_t s) {
    int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_axpy1, dim3(blocks), dim3(256), 0, s, n, x, z);
    return hipGetLastError();
}

__global__ void k_copy(double* __restrict__ dst, const double* __restrict__ src, int64_t n) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        dst[e] = src[e];
}

hipError_t launch_copy(double* dst, const double* src, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192));
    hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(256), 0, s, dst, src, n);
    return hipGetLastError();
}

}  // namespace tpilu

namespace tpilu {

// ----------------------------------------------------------------------------------
// BiCGSTAB steps.  Scalars live in sc[] on the device (kBi* slots); every
// thread that needs one derives it from the same stored values with the same
// expression, so all of them hold the same bits.
// ----------------------------------------------------------------------------------
// rho_old <- rho, rho <- (rs, r) from its partials
__global__ void k_bi_rho(const double* __restrict__ partial, double* sc) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        sc[kBiRhoOld] = sc[kBiRho];
        sc[kBiRho] = tree64(partial);
    }
}

// p <- r (first pass) or p_e <- r_e + beta * (p_e - omega * v_e),
// beta = (rho / rho_old) * (alpha / omega)
__global__ __launch_bounds__(256) void k_bi_p(int64_t n, int first, const double* __restrict__ sc,
                                              const double* __restrict__ r, double* __restrict__ p,
                                              const double* __restrict__ v) {
    const double omega = sc[kBiOmega];
    const double beta = (sc[kBiRho] / sc[kBiRhoOld]) * (sc[kBiAlpha] / omega);
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        p[e] = first ? r[e] : r[e] + beta * (p[e] - omega * v[e]);
}

// rv = (rs, v); alpha = rho / rv (rv == 0: breakdown flag, alpha left alone)
__global__ void k_bi_alpha(const double* __restrict__ partial, double* sc) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const double rv = tree64(partial);
        sc[kBiRv] = rv;
        if (rv != 0.0) sc[kBiAlpha] = sc[kBiRho] / rv;
    }
}

// s_e = r_e - alpha * v_e (skipped after a breakdown)
__global__ __launch_bounds__(256) void k_bi_s(int64_t n, const double* __restrict__ sc, const double* __restrict__ r,
                                              const double* __restrict__ v, double* __restrict__ s) {
    if (sc[kBiRv] == 0.0) return;
    const double alpha = sc[kBiAlpha];
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        s[e] = r[e] - alpha * v[e];
}

// x_e = x_e + alpha * ph_e (the exit after the first half of a step)
__global__ __launch_bounds__(256) void k_bi_x_half(int64_t n, const double* __restrict__ sc, double* __restrict__ x,
                                                   const double* __restrict__ ph) {
    const double alpha = sc[kBiAlpha];
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        x[e] = x[e] + alpha * ph[e];
}

// ts = (t, s), tt = (t, t); omega = ts / tt (tt == 0: breakdown, omega left alone)
__global__ void k_bi_omega(const double* __restrict__ pts, const double* __restrict__ ptt, double* sc) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const double ts = tree64(pts), tt = tree64(ptt);
        sc[kBiTt] = tt;
        if (tt != 0.0) sc[kBiOmega] = ts / tt;
    }
}

// x_e = (x_e + alpha * ph_e) + omega * sh_e; r_e = s_e - omega * t_e (skipped after a breakdown)
__global__ __launch_bounds__(256) void k_bi_xr(int64_t n, const double* __restrict__ sc, double* __restrict__ x,
                                               double* __restrict__ r, const double* __restrict__ ph,
                                               const double* __restrict__ sh, const double* __restrict__ s,
                                               const double* __restrict__ t) {
    if (sc[kBiTt] == 0.0) return;
    const double alpha = sc[kBiAlpha], omega = sc[kBiOmega];
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        x[e] = (x[e] + alpha * ph[e]) + omega * sh[e];
        r[e] = s[e] - omega * t[e];
    }
}

namespace {
int vec_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 2048)); }
}  // namespace

hipError_t launch_bi(int op, int64_t n, int first, const double* pa, const double* pb, double* sc, double* x,
                     double* r, const double* a1, const double* a2, const double* a3, const double* a4,
                     hipStream_t s) {
    switch (op) {
        case kBiOpRho:
            hipLaunchKernelGGL(k_bi_rho, dim3(1), dim3(64), 0, s, pa, sc);
            break;
        case kBiOpP:  // r = a1, p = x (in/out), v = a2
            hipLaunchKernelGGL(k_bi_p, dim3(vec_blocks(n)), dim3(256), 0, s, n, first, sc, a1, x, a2);
            break;
        case kBiOpAlpha:
            hipLaunchKernelGGL(k_bi_alpha, dim3(1), dim3(64), 0, s, pa, sc);
            break;
        case kBiOpS:  // r = a1, v = a2, s = x
            hipLaunchKernelGGL(k_bi_s, dim3(vec_blocks(n)), dim3(256), 0, s, n, sc, a1, a2, x);
            break;
        case kBiOpXHalf:  // x, ph = a1
            hipLaunchKernelGGL(k_bi_x_half, dim3(vec_blocks(n)), dim3(256), 0, s, n, sc, x, a1);
            break;
        case kBiOpOmega:
            hipLaunchKernelGGL(k_bi_omega, dim3(1), dim3(64), 0, s, pa, pb, sc);
            break;
        case kBiOpXR:  // x, r, ph = a1, sh = a2, s = a3, t = a4
            hipLaunchKernelGGL(k_bi_xr, dim3(vec_blocks(n)), dim3(256), 0, s, n, sc, x, r, a1, a2, a3, a4);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace tpilu
