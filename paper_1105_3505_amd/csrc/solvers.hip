// The two applications of the lattice convolution in Section 10, on top of resident plans:
//
//  * a lattice with inclusions (Section 10.1): (A + B) u = 0, u -> v = c1 m1 + c2 m2 at
//    infinity, reduced to mu + B S mu = -B S B v on the nodes the modified bars touch
//    (eq. 10.4), then u = v - S (B v + mu);
//  * a Dirichlet problem on a finite lattice (Section 10.2): u = D q with the double-layer-like
//    operator D of eq. 10.6 (a dipole across each boundary node along its outward normal), q
//    from D q = g on the boundary (eq. 10.7).
//
// S and D are applied by lattice FMM plans (the sources of D are the dipole ends); the dense
// equations are solved by restarted GMRES whose vector operations (classical Gram-Schmidt run
// twice, updates, norms) are kernels on the device.  The small Hessenberg least-squares
// problem (Givens rotations) is solved on the host from one read-back per iteration.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <limits>
#include <memory>
#include <numeric>
#include <string>
#include <unordered_map>
#include <vector>

#include "api_common.h"
#include "lfmm.h"

using namespace lfmm;

namespace {

constexpr int kThreads = 256;

inline unsigned blocks_for(int64_t n) { return unsigned(std::max<int64_t>(1, (n + kThreads - 1) / kThreads)); }

// ---- vector kernels -------------------------------------------------------------------------

typedef double double2_t __attribute__((ext_vector_type(2)));

constexpr int kGsThreads = 1024, kGsWaves = kGsThreads / 64;
constexpr int kGsTile = 512;     // elements: 32 a wave
constexpr int kGsBlocks = 256;   // at most: one per CU

// One step of the Gram-Schmidt passes: a block's slice [per * block, per * (block + 1)) of the vectors.
// UPDATE: w -= V h with the k coefficients h summed from part_in (the nb blocks' partials of a step before;
// block 0 writes them to h_out).  Then NORM: the slice's share of |w|^2 into part_out[block]; otherwise
// its shares of V^T w into part_out[block * kp + j], j < k.
//
// V has rows of ld elements, ld a multiple of the tile, and its rows and w are zero from n on (NORM: w
// may end at n).  For V^T w, lane l of a wave holds row l % 16 of a group of V, eight consecutive
// elements at a time, so that nothing is exchanged between lanes before the end.  (On the matrix cores,
// with w as the other operand, 15 of 16 columns are idle: 2.6 us of FP64 pipe a step against 0.2.)
// A step is bound by reading V, from L2 up to some 10 MB.
// Before, a kernel for the partials (V row by row, nine barriers a row), one that added a vector's 256
// partials in turn and one for the update took 17 + 7 + 7 us on 50,000 elements and 18 vectors; now
// 5.8 us for V^T w, 9.4 with the update before it, 6.7 for the update and |w|^2.
// The order of the sums depends on n and k alone.
template <bool UPDATE, bool NORM>
__global__ __launch_bounds__(kGsThreads) void k_gs(const double* V, int64_t ld, int k, int kp, double* w, int64_t n,
                                                   int64_t per, int nb, const double* part_in, double* h_out,
                                                   double* part_out, double* part_copy) {
    __shared__ double hs[576];   // restart + 1 <= 513 coefficients, in whole rounds of 64
    __shared__ double red[kGsWaves][64];
    const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const int64_t i0 = int64_t(blockIdx.x) * per, i1 = i0 + per < ld ? i0 + per : ld;
    if (UPDATE) {
        for (int j0 = 0; j0 < k; j0 += 64) {
            double a = 0.0;
            #pragma unroll 4
            for (int b = wave; b < nb; b += kGsWaves) a += part_in[size_t(b) * kp + j0 + lane];
            red[wave][lane] = a;
            __syncthreads();
            if (tid < 64) {
                double h = 0.0;
                for (int q = 0; q < kGsWaves; ++q) h += red[q][tid];
                hs[j0 + tid] = h;
                if (blockIdx.x == 0 && j0 + tid < k) h_out[j0 + tid] = h;
            }
            __syncthreads();
        }
    }
    double sq = 0.0;
    if (UPDATE || NORM) {
        // two threads an element: the even and the odd vectors
        const int e = tid & (kGsTile - 1), odd = tid / kGsTile;
        for (int64_t t0 = i0; t0 < i1; t0 += kGsTile) {
            const int64_t i = t0 + e;
            double a = 0.0;
            if (UPDATE) {
                const double* v = V + size_t(i);
                #pragma unroll 8
                for (int j = odd; j < k; j += 2) a += hs[j] * v[size_t(j) * size_t(ld)];
                double* sum = &red[0][0];
                if (odd) sum[e] = a;
                __syncthreads();
                a += sum[e];
            }
            if (!odd && i < n) {
                const double x = UPDATE ? w[i] - a : w[i];
                if (UPDATE) w[i] = x;
                sq += x * x;
            }
            __syncthreads();   // w is read by the block's other waves below, the sums' array written again
        }
    }
    if (NORM) {
        red[wave][lane] = sq;
        __syncthreads();
        if (tid < 64) {
            double a = 0.0;
            for (int q = 0; q < kGsWaves; ++q) a += red[q][tid];
            for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
            if (tid == 0) {
                part_out[blockIdx.x] = a;
                if (part_copy) part_copy[blockIdx.x] = a;
            }
        }
    } else {
        for (int j0 = 0; j0 < k; j0 += 64) {   // up to four groups of 16 vectors a pass
            const int groups = (min(k - j0, 64) + 15) / 16;
            // waves: group wave % G of G = 1, 2 or 4 and an equal part of the tile
            const int G = groups > 2 ? 4 : groups, g = wave & (G - 1), len = 32 * G;
            const int row = min(j0 + 16 * g + (lane & 15), k - 1);   // rows past the last repeat it
            const int64_t first = i0 + (wave / G) * len + 8 * (lane >> 4);
            const double2_t* v = reinterpret_cast<const double2_t*>(V + size_t(row) * size_t(ld) + first);
            const double2_t* x = reinterpret_cast<const double2_t*>(w + first);
            double a0 = 0.0, a1 = 0.0;
            if (g < groups)
                for (int64_t t0 = i0; t0 < i1; t0 += kGsTile) {
                    #pragma unroll 2
                    for (int q = 0; q < len; q += 32) {
                        double2_t a[4], b[4];
                        #pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            a[u] = v[q / 2 + u];
                            b[u] = x[q / 2 + u];
                        }
                        #pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            a0 = fma(a[u].x, b[u].x, a0);
                            a1 = fma(a[u].y, b[u].y, a1);
                        }
                    }
                    v += kGsTile / 2;
                    x += kGsTile / 2;
                }
            red[wave][lane] = a0 + a1;
            __syncthreads();
            if (tid < 16 * groups) {   // vector j0 + tid: its group's waves, four lanes each
                double h = 0.0;
                for (int q = tid >> 4; q < kGsWaves; q += G)
                    for (int u = 0; u < 4; ++u) h += red[q][16 * u + (tid & 15)];
                part_out[size_t(blockIdx.x) * kp + j0 + tid] = h;
            }
            __syncthreads();
        }
    }
}

// zero elements n .. ld - 1 of the rows of V
__global__ void k_pad_rows(double* V, int64_t ld, int64_t n) {
    const int64_t i = n + int64_t(threadIdx.x);
    if (i < ld) V[size_t(blockIdx.x) * size_t(ld) + size_t(i)] = 0.0;
}

// w += sign * sum_j h[j] V[j]
__global__ void k_combine(const double* V, int64_t ldv, int k, const double* h, double sign, double* w, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int j = 0; j < k; ++j) s += h[j] * V[size_t(j) * size_t(ldv) + size_t(i)];
    w[i] += sign * s;
}

__global__ void k_fill(double* out, double v, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = v;
}

__global__ void k_scale_copy(const double* a, double s, double* out, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = s * a[i];
}

// out = w / |w|, with |w|^2 the sum of the nb <= kGsBlocks shares sq, added in turn as on the host
__global__ __launch_bounds__(kThreads) void k_normalise(const double* w, const double* sq, int nb, double* out, int64_t n) {
    static_assert(kGsBlocks <= kThreads, "a share per thread");
    __shared__ double p[kGsBlocks], s;
    if (int(threadIdx.x) < nb) p[threadIdx.x] = sq[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0;
        #pragma unroll 8
        for (int b = 0; b < nb; ++b) a += p[b];
        s = 1.0 / sqrt(max(a, 0.0));
    }
    __syncthreads();
    const int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) out[i] = s * w[i];
}

// out = a - b
__global__ void k_sub(const double* a, const double* b, double* out, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] - b[i];
}

// ---- operators of Section 10 ------------------------------------------------------------------

// out[i] = cb * base[i] + cs * sum over the bars at node i of delta (s[i] - s[other end])
// (B applied to s, Section 10.1: each bar adds delta (e_a - e_b)(e_a - e_b)^T); base may be null
__global__ void k_bars(const int32_t* rowptr, const int32_t* col, const double* dlt, const double* s,
                       const double* base, double cb, double cs, double* out, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double si = s[i];
    double acc = 0.0;
    for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e) acc += dlt[e] * (si - s[col[e]]);
    out[i] = (base ? cb * base[i] : 0.0) + cs * acc;
}

// v(m) = c1 m1 + c2 m2 at the points xy (the far-field condition of eq. 10.2)
__global__ void k_linear(const int2* xy, double c1, double c2, double* out, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = c1 * double(xy[i].x) + c2 * double(xy[i].y);
}

// u[i] = c1 x_i + c2 y_i - u[i]  (u = v - S(...) in place)
__global__ void k_linear_minus(const int2* xy, double c1, double c2, double* u, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) u[i] = c1 * double(xy[i].x) + c2 * double(xy[i].y) - u[i];
}

// loads of the dipoles of D: +q at n + nu(n) (first half), -q at n (second half)
__global__ void k_dipole_loads(const double* q, double* f2, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) {
        f2[i] = q[i];
        f2[n + i] = -q[i];
    }
}

// ---- device buffers ---------------------------------------------------------------------------

struct HipError {
    std::string msg;
};

#define SOLVER_HIP(call)                                                                         \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess) throw HipError{std::string(#call) + ": " + hipGetErrorString(e_)}; \
    } while (0)

template <class T>
struct DevBuf {
    T* p = nullptr;
    size_t n = 0;
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    void alloc(size_t count) {
        free();
        if (count == 0) count = 1;
        SOLVER_HIP(hipMalloc(reinterpret_cast<void**>(&p), count * sizeof(T)));
        n = count;
    }
    void free() {
        if (p) (void)hipFree(p);
        p = nullptr;
        n = 0;
    }
    ~DevBuf() { free(); }
};

struct Status {
    lfmm_status s;
    std::string msg;
};

void check(lfmm_status s) {
    if (s < 0) throw Status{s, lfmm_last_error()};
}

// ---- restarted GMRES ----------------------------------------------------------------------------

// Solves A x = b (device vectors of n) by GMRES(m) with x0 = 0; apply(in, out) enqueues A in
// on the stream.  Stops when the relative residual |b - A x| / |b| estimated by the Givens
// recurrence is <= tol, or after max_iter iterations; then reports the true relative residual.
struct Gmres {
    lfmm_ctx* ctx;
    hipStream_t st;
    int64_t n;
    int m;
    int64_t ld, per;   // elements of a row of V, of a block's slice
    int kp, nb;        // coefficients a block's partials hold room for; blocks
    // V: m + 1 rows and w; part, part2: the blocks' shares of either pass's coefficients; rhs: room for the
    // caller's right-hand side
    double *V = nullptr, *w = nullptr, *part = nullptr, *part2 = nullptr, *y = nullptr, *r = nullptr, *rhs = nullptr;
    // pinned, written by the kernels: coefficients of both passes and the blocks' shares of |w|^2 (a
    // copy to pageable memory behind them left the device idle for 30 us more an iteration), of the even
    // and of the odd iterations, and what tells that they are there
    double* h = nullptr;
    hipEvent_t ready[2] = {nullptr, nullptr};

    // The workspace of one solve.  Up to kPooledBytes it is a block of the context's pool, so that solves
    // one after another, of this object or others, neither allocate (hipMalloc and hipFree on every solve,
    // with the copies named above: 35 iterations on 50,000 elements 7.1 ms, without 6.2) nor hold more than
    // one such block between them; above, it is allocated and freed.
    static constexpr size_t kPooledBytes = size_t(128) << 20;
    void* dev = nullptr;
    size_t dev_class = 0, host_class = 0;   // of the pooled blocks; dev_class 0: not pooled

    Gmres(lfmm_ctx* ctx_, int64_t n_, int restart, hipStream_t st_)
        : ctx(ctx_), st(st_), n(n_), m(int(std::min<int64_t>(restart, n_))) {
        const int64_t tiles = (n + kGsTile - 1) / kGsTile;
        ld = tiles * kGsTile;
        per = (tiles + kGsBlocks - 1) / kGsBlocks * kGsTile;
        nb = int((ld + per - 1) / per);
        kp = (m + 1 + 63) / 64 * 64;
        const size_t basis = size_t(m + 2) * size_t(ld), share = size_t(nb) * size_t(kp);
        const size_t bytes = (basis + 2 * share + size_t(kp) + 2 * size_t(ld)) * sizeof(double);
        try {
            if (bytes <= kPooledBytes) check(ctx_acquire(ctx, bytes, false, &dev, &dev_class));
            else SOLVER_HIP(hipMalloc(&dev, bytes));
            V = static_cast<double*>(dev);   // (all pieces are whole tiles or whole rounds of 64)
            w = V + size_t(m + 1) * size_t(ld);
            part = V + basis;
            part2 = part + share;
            y = part2 + share;
            r = y + kp;
            rhs = r + ld;
            void* p = nullptr;
            check(ctx_acquire(ctx, 2 * size_t(2 * kp + nb) * sizeof(double), true, &p, &host_class));
            h = static_cast<double*>(p);
            for (hipEvent_t& e : ready) SOLVER_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        } catch (...) {
            release();
            throw;
        }
        hipLaunchKernelGGL(k_pad_rows, dim3(unsigned(m + 2)), dim3(kGsTile), 0, st, V, ld, n);
    }
    Gmres(const Gmres&) = delete;
    Gmres& operator=(const Gmres&) = delete;
    // After an error in a solve, kernels (an iteration sent ahead among them) may still write the workspace
    ~Gmres() {
        (void)hipStreamSynchronize(st);
        release();
    }

    void release() {
        for (hipEvent_t e : ready)
            if (e) (void)hipEventDestroy(e);
        if (h) ctx_release(ctx, h, host_class, true);
        if (dev && dev_class) ctx_release(ctx, dev, dev_class, false);
        else if (dev) (void)hipFree(dev);
    }

    // part = the blocks' shares of V[0..k)^T w
    void dots(int k) {
        hipLaunchKernelGGL((k_gs<false, false>), dim3(unsigned(nb)), dim3(kGsThreads), 0, st, V, ld, k, kp, w, n, per,
                           nb, nullptr, nullptr, part, nullptr);
    }

    double norm(const double* x) {
        hipLaunchKernelGGL((k_gs<false, true>), dim3(unsigned(nb)), dim3(kGsThreads), 0, st, V, ld, 0, kp,
                           const_cast<double*>(x), n, per, nb, nullptr, nullptr, h, nullptr);
        SOLVER_HIP(hipStreamSynchronize(st));
        return std::sqrt(std::max(std::accumulate(h, h + nb, 0.0), 0.0));
    }

    lfmm_solver_stats run(const std::function<void(const double*, double*)>& apply, const double* b, double* x,
                          double tol, int max_iter, bool ahead) {
        lfmm_solver_stats out{};
        hipLaunchKernelGGL(k_fill, dim3(blocks_for(n)), dim3(kThreads), 0, st, x, 0.0, n);
        const double bn = norm(b);
        if (bn == 0.0) {
            out.converged = 1;
            return out;
        }
        std::vector<double> H(size_t(m + 1) * m), cs(m), sn(m), g(m + 1);
        auto Hat = [&](int i, int j) -> double& { return H[size_t(i) * m + size_t(j)]; };
        SOLVER_HIP(hipMemcpyAsync(r, b, size_t(n) * sizeof(double), hipMemcpyDeviceToDevice, st));
        double beta = bn;
        int iters = 0;
        bool done = false;
        while (!done) {
            hipLaunchKernelGGL(k_scale_copy, dim3(blocks_for(n)), dim3(kThreads), 0, st, r, 1.0 / beta, V, n);
            std::fill(g.begin(), g.end(), 0.0);
            g[0] = beta;
            // Iteration j's kernels: classical Gram-Schmidt, twice: h = V^T w; w -= V h (both passes
            // summed); the two coefficient sets and |w|^2 come back together
            auto enqueue = [&](int j) {
                double* hj = h + (j & 1) * (2 * kp + nb);
                apply(V + size_t(j) * size_t(ld), w);
                dots(j + 1);
                hipLaunchKernelGGL((k_gs<true, false>), dim3(unsigned(nb)), dim3(kGsThreads), 0, st, V, ld, j + 1, kp,
                                   w, n, per, nb, part, hj, part2, nullptr);
                hipLaunchKernelGGL((k_gs<true, true>), dim3(unsigned(nb)), dim3(kGsThreads), 0, st, V, ld, j + 1, kp,
                                   w, n, per, nb, part2, hj + kp, hj + 2 * kp, part);
                SOLVER_HIP(hipEventRecord(ready[j & 1], st));
            };
            auto enqueue_next = [&](int j) {
                hipLaunchKernelGGL(k_normalise, dim3(blocks_for(n)), dim3(kThreads), 0, st, w, part, nb,
                                   V + size_t(j + 1) * size_t(ld), n);
                enqueue(j + 1);
            };
            enqueue(0);
            int j = 0;
            for (; j < m; ++j) {
                // The next iteration goes out before this one's results are read, so that the device does
                // not wait for the host (a third of an iteration on 50,000 unknowns), unless the residual's
                // last step, taken again, would end the solve: then it would be in vain
                const bool likely_last = j > 0 && g[size_t(j)] * g[size_t(j)] <= tol * bn * std::fabs(g[size_t(j) - 1]);
                const bool sent = ahead && j + 1 < m && iters + 1 < max_iter && !likely_last;
                if (sent) enqueue_next(j);
                const double* hj = h + (j & 1) * (2 * kp + nb);
                SOLVER_HIP(hipEventSynchronize(ready[j & 1]));
                SOLVER_HIP(hipGetLastError());
                const double wn = std::sqrt(std::max(std::accumulate(hj + 2 * kp, hj + 2 * kp + nb, 0.0), 0.0));
                for (int i = 0; i <= j; ++i) Hat(i, j) = hj[i] + hj[kp + i];
                Hat(j + 1, j) = wn;
                // previous rotations, then a new one that zeroes H(j+1, j)
                for (int i = 0; i < j; ++i) {
                    const double a = Hat(i, j), c = Hat(i + 1, j);
                    Hat(i, j) = cs[size_t(i)] * a + sn[size_t(i)] * c;
                    Hat(i + 1, j) = -sn[size_t(i)] * a + cs[size_t(i)] * c;
                }
                const double a = Hat(j, j), c = Hat(j + 1, j);
                const double rho = std::hypot(a, c);
                cs[size_t(j)] = rho > 0.0 ? a / rho : 1.0;
                sn[size_t(j)] = rho > 0.0 ? c / rho : 0.0;
                Hat(j, j) = rho;
                Hat(j + 1, j) = 0.0;
                g[size_t(j) + 1] = -sn[size_t(j)] * g[size_t(j)];
                g[size_t(j)] = cs[size_t(j)] * g[size_t(j)];
                ++iters;
                if (std::fabs(g[size_t(j) + 1]) <= tol * bn || iters >= max_iter || wn == 0.0) {
                    ++j;
                    done = true;
                    break;
                }
                if (!sent && j + 1 < m) enqueue_next(j);
            }
            if (!done) j = m;
            // y = H(0..j, 0..j)^-1 g; x += V y
            std::vector<double> c(size_t(j), 0.0);
            for (int i = j - 1; i >= 0; --i) {
                double s = g[size_t(i)];
                for (int k = i + 1; k < j; ++k) s -= Hat(i, k) * c[size_t(k)];
                c[size_t(i)] = Hat(i, i) != 0.0 ? s / Hat(i, i) : 0.0;
            }
            SOLVER_HIP(hipMemcpyAsync(y, c.data(), size_t(j) * sizeof(double), hipMemcpyHostToDevice, st));
            hipLaunchKernelGGL(k_combine, dim3(blocks_for(n)), dim3(kThreads), 0, st, V, ld, j, y, 1.0, x, n);
            // true residual r = b - A x (also the next cycle's start)
            apply(x, w);
            hipLaunchKernelGGL(k_sub, dim3(blocks_for(n)), dim3(kThreads), 0, st, b, w, r, n);
            beta = norm(r);
            if (beta <= tol * bn) done = true;
            if (iters >= max_iter) done = true;
        }
        out.iterations = iters;
        out.rel_residual = beta / bn;
        out.converged = out.rel_residual <= tol ? 1 : 0;
        return out;
    }
};

lfmm_status check_solver_options(const lfmm_solver_options* o, double* tol, int* max_iter, int* restart) {
    *tol = 1e-12;
    *max_iter = 500;
    *restart = 50;
    if (!o) return LFMM_OK;
    if (o->tol > 0.0) *tol = o->tol;
    if (o->max_iter > 0) *max_iter = o->max_iter;
    if (o->restart > 0) *restart = o->restart;
    if (!(*tol < 1.0) || *restart > 512 || *max_iter > 1000000)
        return fail(LFMM_E_INVAL, "solver options: tol in (0, 1), restart <= 512, max_iter <= 1e6");
    return LFMM_OK;
}

template <class F>
lfmm_status run_guarded(F&& f) {
    (void)hipGetLastError();
    try {
        return f();
    } catch (const HipError& e) {
        return fail(LFMM_E_HIP, e.msg);
    } catch (const Status& e) {
        return fail(e.s, e.msg);
    } catch (const std::bad_alloc&) {
        return fail(LFMM_E_NOMEM, "host allocation failed");
    }
}

// executes that check their loads read them back, and would refuse those of an iteration sent in vain
bool runs_ahead(const lfmm_ctx* ctx) { return !(ctx_flags(ctx) & LFMM_FLAG_CHECK_LOADS); }

hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

}  // namespace

// ---- lattice with inclusions ----------------------------------------------------------------------

struct lfmm_inclusions {
    lfmm_ctx* ctx = nullptr;
    int device = 0;
    int64_t nn = 0;                       // nodes touched by the bars (Omega_inc)
    std::vector<int32_t> nodes;           // host copy, [nn][2]
    DevBuf<int32_t> xy, rowptr, col;
    DevBuf<double> dlt, v, s, t;
    lfmm_plan* plan = nullptr;            // the nodes, targets = sources: S on Omega_inc
    ~lfmm_inclusions() {
        if (plan) lfmm_plan_destroy(plan);
    }
};

struct lfmm_dirichlet {
    lfmm_ctx* ctx = nullptr;
    int device = 0;
    int64_t n = 0;                        // boundary nodes
    DevBuf<int32_t> src;                  // [2n][2]: n + nu(n) first, then n
    DevBuf<int32_t> gam;                  // [n][2]
    DevBuf<double> f2;                    // dipole loads
    lfmm_plan* plan = nullptr;            // sources: the dipole ends; targets: the boundary
    ~lfmm_dirichlet() {
        if (plan) lfmm_plan_destroy(plan);
    }
};

extern "C" {

lfmm_status lfmm_inclusions_create(lfmm_ctx* ctx, int64_t n_bars, const int32_t* bars, const double* delta,
                                   void* stream, lfmm_inclusions** out) {
    if (!ctx || !bars || !delta || !out || n_bars < 1) return fail(LFMM_E_INVAL, "null argument or no bar");
    if (n_bars > (int64_t(1) << 28)) return fail(LFMM_E_INVAL, "too many bars");
    *out = nullptr;
    for (int64_t k = 0; k < n_bars; ++k) {
        if (!std::isfinite(delta[k])) return fail(LFMM_E_INVAL, "non-finite conductance change");
        if (bars[4 * k] == bars[4 * k + 2] && bars[4 * k + 1] == bars[4 * k + 3])
            return fail(LFMM_E_INVAL, "a bar joins a node to itself");
    }
    return run_guarded([&]() -> lfmm_status {
        auto inc = std::make_unique<lfmm_inclusions>();
        inc->ctx = ctx;
        inc->device = ctx_device(ctx);
        SOLVER_HIP(hipSetDevice(inc->device));
        // nodes in first-appearance order; per node its bars as (other end, delta)
        std::unordered_map<uint64_t, int32_t> index;
        index.reserve(size_t(2 * n_bars));
        std::vector<int32_t> ends(size_t(2 * n_bars));
        for (int64_t k = 0; k < 2 * n_bars; ++k) {
            const uint64_t key = (uint64_t(uint32_t(bars[2 * k])) << 32) | uint32_t(bars[2 * k + 1]);
            auto it = index.find(key);
            if (it == index.end()) {
                it = index.emplace(key, int32_t(inc->nodes.size() / 2)).first;
                inc->nodes.push_back(bars[2 * k]);
                inc->nodes.push_back(bars[2 * k + 1]);
            }
            ends[size_t(k)] = it->second;
        }
        const int64_t nn = int64_t(inc->nodes.size() / 2);
        inc->nn = nn;
        std::vector<int32_t> rp(size_t(nn) + 1, 0), cl(size_t(2 * n_bars));
        std::vector<double> dl(size_t(2 * n_bars));
        for (int64_t k = 0; k < n_bars; ++k) {
            ++rp[size_t(ends[size_t(2 * k)]) + 1];
            ++rp[size_t(ends[size_t(2 * k + 1)]) + 1];
        }
        for (int64_t i = 0; i < nn; ++i) rp[size_t(i) + 1] += rp[size_t(i)];
        std::vector<int32_t> fill(rp.begin(), rp.end() - 1);
        for (int64_t k = 0; k < n_bars; ++k) {
            const int32_t a = ends[size_t(2 * k)], b = ends[size_t(2 * k + 1)];
            cl[size_t(fill[size_t(a)])] = b;
            dl[size_t(fill[size_t(a)]++)] = delta[k];
            cl[size_t(fill[size_t(b)])] = a;
            dl[size_t(fill[size_t(b)]++)] = delta[k];
        }
        inc->xy.alloc(size_t(2 * nn));
        inc->rowptr.alloc(size_t(nn) + 1);
        inc->col.alloc(cl.size());
        inc->dlt.alloc(dl.size());
        inc->v.alloc(size_t(nn));
        inc->s.alloc(size_t(nn));
        inc->t.alloc(size_t(nn));
        SOLVER_HIP(hipMemcpy(inc->xy.p, inc->nodes.data(), size_t(2 * nn) * 4, hipMemcpyHostToDevice));
        SOLVER_HIP(hipMemcpy(inc->rowptr.p, rp.data(), rp.size() * 4, hipMemcpyHostToDevice));
        SOLVER_HIP(hipMemcpy(inc->col.p, cl.data(), cl.size() * 4, hipMemcpyHostToDevice));
        SOLVER_HIP(hipMemcpy(inc->dlt.p, dl.data(), dl.size() * 8, hipMemcpyHostToDevice));
        check(lfmm_plan_create(ctx, nn, inc->xy.p, 0, nullptr, stream, &inc->plan));
        *out = inc.release();
        return LFMM_OK;
    });
}

lfmm_status lfmm_inclusions_nodes(const lfmm_inclusions* inc, int64_t* n_nodes, int32_t* nodes_xy_host) {
    if (!inc || !n_nodes) return fail(LFMM_E_INVAL, "null argument");
    *n_nodes = inc->nn;
    if (nodes_xy_host) std::memcpy(nodes_xy_host, inc->nodes.data(), inc->nodes.size() * sizeof(int32_t));
    return LFMM_OK;
}

lfmm_status lfmm_inclusions_solve(lfmm_inclusions* inc, double c1, double c2, const lfmm_solver_options* opt,
                                  double* mu_dev, lfmm_solver_stats* stats, void* stream) {
    if (!inc || !mu_dev) return fail(LFMM_E_INVAL, "null argument");
    if (!std::isfinite(c1) || !std::isfinite(c2)) return fail(LFMM_E_INVAL, "non-finite field");
    double tol = 0.0;
    int max_iter = 0, restart = 0;
    lfmm_status s = check_solver_options(opt, &tol, &max_iter, &restart);
    if (s != LFMM_OK) return s;
    return run_guarded([&]() -> lfmm_status {
        SOLVER_HIP(hipSetDevice(inc->device));
        hipStream_t st = as_stream(stream);
        const int64_t nn = inc->nn;
        const unsigned gb = blocks_for(nn);
        const int2* xy = reinterpret_cast<const int2*>(inc->xy.p);
        // right-hand side of eq. 10.4: -B S B v
        Gmres gm(inc->ctx, nn, restart, st);
        hipLaunchKernelGGL(k_linear, dim3(gb), dim3(kThreads), 0, st, xy, c1, c2, inc->v.p, nn);
        hipLaunchKernelGGL(k_bars, dim3(gb), dim3(kThreads), 0, st, inc->rowptr.p, inc->col.p, inc->dlt.p, inc->v.p,
                           nullptr, 0.0, 1.0, inc->t.p, nn);
        check(lfmm_execute(inc->plan, inc->t.p, inc->s.p, stream));
        hipLaunchKernelGGL(k_bars, dim3(gb), dim3(kThreads), 0, st, inc->rowptr.p, inc->col.p, inc->dlt.p, inc->s.p,
                           nullptr, 0.0, -1.0, gm.rhs, nn);
        // operator: mu -> mu + B S mu
        auto apply = [&](const double* in, double* o) {
            check(lfmm_execute(inc->plan, in, inc->s.p, stream));
            hipLaunchKernelGGL(k_bars, dim3(gb), dim3(kThreads), 0, st, inc->rowptr.p, inc->col.p, inc->dlt.p,
                               inc->s.p, in, 1.0, 1.0, o, nn);
        };
        const lfmm_solver_stats r = gm.run(apply, gm.rhs, mu_dev, tol, max_iter, runs_ahead(inc->ctx));
        SOLVER_HIP(hipStreamSynchronize(st));
        if (stats) *stats = r;
        return LFMM_OK;
    });
}

lfmm_status lfmm_inclusions_potential(lfmm_inclusions* inc, double c1, double c2, const double* mu_dev,
                                      int64_t n_tgt, const int32_t* tgt_xy_dev, double* u_dev, void* stream) {
    if (!inc || !mu_dev || !tgt_xy_dev || !u_dev || n_tgt < 1) return fail(LFMM_E_INVAL, "null argument or no target");
    return run_guarded([&]() -> lfmm_status {
        SOLVER_HIP(hipSetDevice(inc->device));
        hipStream_t st = as_stream(stream);
        const int64_t nn = inc->nn;
        const unsigned gb = blocks_for(nn);
        // loads B v + mu on the nodes, their field at the targets, u = v - that field
        hipLaunchKernelGGL(k_linear, dim3(gb), dim3(kThreads), 0, st, reinterpret_cast<const int2*>(inc->xy.p), c1, c2,
                           inc->v.p, nn);
        hipLaunchKernelGGL(k_bars, dim3(gb), dim3(kThreads), 0, st, inc->rowptr.p, inc->col.p, inc->dlt.p, inc->v.p,
                           mu_dev, 1.0, 1.0, inc->t.p, nn);
        lfmm_plan* pt = nullptr;
        check(lfmm_plan_create(inc->ctx, nn, inc->xy.p, n_tgt, tgt_xy_dev, stream, &pt));
        lfmm_status s = lfmm_execute(pt, inc->t.p, u_dev, stream);
        lfmm_plan_destroy(pt);
        check(s);
        hipLaunchKernelGGL(k_linear_minus, dim3(blocks_for(n_tgt)), dim3(kThreads), 0, st,
                           reinterpret_cast<const int2*>(tgt_xy_dev), c1, c2, u_dev, n_tgt);
        SOLVER_HIP(hipGetLastError());
        return LFMM_OK;
    });
}

lfmm_status lfmm_inclusions_destroy(lfmm_inclusions* inc) {
    if (!inc) return LFMM_OK;
    (void)hipSetDevice(inc->device);
    (void)hipDeviceSynchronize();
    delete inc;
    return LFMM_OK;
}

// ---- Dirichlet problem ------------------------------------------------------------------------------

lfmm_status lfmm_dirichlet_create(lfmm_ctx* ctx, int64_t n, const int32_t* gamma_xy, const int8_t* normal,
                                  void* stream, lfmm_dirichlet** out) {
    if (!ctx || !gamma_xy || !normal || !out || n < 1) return fail(LFMM_E_INVAL, "null argument or no boundary node");
    if (n > (int64_t(1) << 28)) return fail(LFMM_E_INVAL, "too many boundary nodes");
    *out = nullptr;
    static const int32_t step[4][2] = {{1, 0}, {-1, 0}, {0, 1}, {0, -1}};
    std::vector<int32_t> src(size_t(4 * n));
    for (int64_t i = 0; i < n; ++i) {
        const int c = normal[i];
        if (c < 0 || c > 3) return fail(LFMM_E_INVAL, "normal codes are 0..3 (+x, -x, +y, -y)");
        const int64_t x = int64_t(gamma_xy[2 * i]) + step[c][0], y = int64_t(gamma_xy[2 * i + 1]) + step[c][1];
        if (x < INT32_MIN || x > INT32_MAX || y < INT32_MIN || y > INT32_MAX)
            return fail(LFMM_E_RANGE, "a normal step leaves the int32 lattice");
        src[size_t(2 * i)] = int32_t(x);
        src[size_t(2 * i + 1)] = int32_t(y);
        src[size_t(2 * (n + i))] = gamma_xy[2 * i];
        src[size_t(2 * (n + i) + 1)] = gamma_xy[2 * i + 1];
    }
    return run_guarded([&]() -> lfmm_status {
        auto dir = std::make_unique<lfmm_dirichlet>();
        dir->ctx = ctx;
        dir->device = ctx_device(ctx);
        dir->n = n;
        SOLVER_HIP(hipSetDevice(dir->device));
        dir->src.alloc(size_t(4 * n));
        dir->gam.alloc(size_t(2 * n));
        dir->f2.alloc(size_t(2 * n));
        SOLVER_HIP(hipMemcpy(dir->src.p, src.data(), src.size() * 4, hipMemcpyHostToDevice));
        SOLVER_HIP(hipMemcpy(dir->gam.p, gamma_xy, size_t(2 * n) * 4, hipMemcpyHostToDevice));
        check(lfmm_plan_create(ctx, 2 * n, dir->src.p, n, dir->gam.p, stream, &dir->plan));
        *out = dir.release();
        return LFMM_OK;
    });
}

lfmm_status lfmm_dirichlet_apply(lfmm_dirichlet* dir, const double* q_dev, double* out_dev, void* stream) {
    if (!dir || !q_dev || !out_dev) return fail(LFMM_E_INVAL, "null argument");
    return run_guarded([&]() -> lfmm_status {
        SOLVER_HIP(hipSetDevice(dir->device));
        hipLaunchKernelGGL(k_dipole_loads, dim3(blocks_for(dir->n)), dim3(kThreads), 0, as_stream(stream), q_dev,
                           dir->f2.p, dir->n);
        check(lfmm_execute(dir->plan, dir->f2.p, out_dev, stream));
        SOLVER_HIP(hipGetLastError());
        return LFMM_OK;
    });
}

lfmm_status lfmm_dirichlet_solve(lfmm_dirichlet* dir, const double* g_dev, const lfmm_solver_options* opt,
                                 double* q_dev, lfmm_solver_stats* stats, void* stream) {
    if (!dir || !g_dev || !q_dev) return fail(LFMM_E_INVAL, "null argument");
    double tol = 0.0;
    int max_iter = 0, restart = 0;
    lfmm_status s = check_solver_options(opt, &tol, &max_iter, &restart);
    if (s != LFMM_OK) return s;
    return run_guarded([&]() -> lfmm_status {
        SOLVER_HIP(hipSetDevice(dir->device));
        hipStream_t st = as_stream(stream);
        auto apply = [&](const double* in, double* o) {
            hipLaunchKernelGGL(k_dipole_loads, dim3(blocks_for(dir->n)), dim3(kThreads), 0, st, in, dir->f2.p, dir->n);
            check(lfmm_execute(dir->plan, dir->f2.p, o, stream));
        };
        Gmres gm(dir->ctx, dir->n, restart, st);
        const lfmm_solver_stats r = gm.run(apply, g_dev, q_dev, tol, max_iter, runs_ahead(dir->ctx));
        SOLVER_HIP(hipStreamSynchronize(st));
        if (stats) *stats = r;
        return LFMM_OK;
    });
}

lfmm_status lfmm_dirichlet_potential(lfmm_dirichlet* dir, const double* q_dev, int64_t n_tgt,
                                     const int32_t* tgt_xy_dev, double* u_dev, void* stream) {
    if (!dir || !q_dev || !tgt_xy_dev || !u_dev || n_tgt < 1) return fail(LFMM_E_INVAL, "null argument or no target");
    return run_guarded([&]() -> lfmm_status {
        SOLVER_HIP(hipSetDevice(dir->device));
        hipLaunchKernelGGL(k_dipole_loads, dim3(blocks_for(dir->n)), dim3(kThreads), 0, as_stream(stream), q_dev,
                           dir->f2.p, dir->n);
        lfmm_plan* pt = nullptr;
        check(lfmm_plan_create(dir->ctx, 2 * dir->n, dir->src.p, n_tgt, tgt_xy_dev, stream, &pt));
        lfmm_status s = lfmm_execute(pt, dir->f2.p, u_dev, stream);
        lfmm_plan_destroy(pt);
        check(s);
        SOLVER_HIP(hipGetLastError());
        return LFMM_OK;
    });
}

lfmm_status lfmm_dirichlet_destroy(lfmm_dirichlet* dir) {
    if (!dir) return LFMM_OK;
    (void)hipSetDevice(dir->device);
    (void)hipDeviceSynchronize();
    delete dir;
    return LFMM_OK;
}

}  // extern "C"
