// k_reduce.hip -- FP64 reductions (Krylov dot products, norms) and the
// streaming vector updates of PCG.  Reductions are two-stage and
// deterministic: a fixed number of workgroups accumulate FP64 partial sums
// in grid-stride order and one workgroup adds the partials in index order.
#include "internal.h"

namespace clh {

namespace {

constexpr int TPB = 256;

__global__ __launch_bounds__(TPB) void k_dot(const float *__restrict__ a, const float *__restrict__ b, size_t n,
                                             double *__restrict__ partials)
{
    double acc = 0.0;
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t p = (size_t)blockIdx.x * TPB + threadIdx.x; p < n; p += stride)
        acc += (double)a[p] * (double)b[p];
    acc = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

// Counts the values that are not finite and copies them on the way (copy may be
// NULL).  W values per access: 4 where the pointers allow it, else 1.  One pass
// instead of two: a 256^3 velocity 75 us against 40 + 80 us.
template <int W>
__global__ __launch_bounds__(TPB) void k_count_nonfinite(const float *__restrict__ a, float *__restrict__ copy, size_t n,
                                                         double *__restrict__ partials)
{
    typedef float fw __attribute__((ext_vector_type(W)));
    int bad = 0;
    const size_t stride = (size_t)gridDim.x * TPB, nw = n / W;
    for (size_t p = (size_t)blockIdx.x * TPB + threadIdx.x; p < nw; p += stride) {
        const fw x = ((const fw *)a)[p];
#pragma unroll
        for (int i = 0; i < W; ++i) bad += isfinite(x[i]) ? 0 : 1;
        if (copy) ((fw *)copy)[p] = x;
    }
    const double acc = block_sum((double)bad);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

// Sum of nb partials in a fixed order, valid in thread 0 of the one
// workgroup that runs it: thread t adds the partials t, t + T, ... of T threads
// (so a wavefront reads consecutive values), then block_sum.  Every finalize below
// is a launch of one small workgroup between two dependent kernels, bound by
// its latency: with a serial sum of 256 thread values it took 3.0 us at
// nb = 192 and 5 us at nb = 2048.
__device__ __forceinline__ double sum_partials(const double *__restrict__ partials, int nb)
{
    double acc = 0.0;
    for (int q = threadIdx.x; q < nb; q += blockDim.x) acc += partials[q];
    return block_sum(acc);
}

// threads for nb partials of the sums that a transform's workgroups leave behind
// (6912 at 256^3: 13.0 us with 256 threads, 5.5 us with 1024)
constexpr int FIN = 1024;
int finalize_threads(int nb) { return nb > 2048 ? FIN : TPB; }

__global__ __launch_bounds__(FIN) void k_finalize(const double *__restrict__ partials, int nb, double scale,
                                                  double *__restrict__ out)
{
    const double t = sum_partials(partials, nb);
    if (threadIdx.x == 0) out[0] = scale * t;
}

// out[c] = sum of row c of nb partials, one workgroup per row
__global__ __launch_bounds__(TPB) void k_finalize_rows(const double *__restrict__ partials, int nb,
                                                       double *__restrict__ out)
{
    const double t = sum_partials(partials + (size_t)blockIdx.x * nb, nb);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// min and max of the wavefronts' values over a workgroup (valid in thread 0);
// any bad thread turns both into NaN
template <typename T> __device__ __forceinline__ void block_minmax(T &lo, T &hi, bool bad)
{
    __shared__ T slo[TPB / 64], shi[TPB / 64];
    __shared__ int sbad[TPB / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, __shfl_xor(lo, off, 64));
        hi = max(hi, __shfl_xor(hi, off, 64));
    }
    const int w = threadIdx.x >> 6;
    const bool any = __any(bad);
    if ((threadIdx.x & 63) == 0) {
        slo[w] = lo;
        shi[w] = hi;
        sbad[w] = any;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int b = sbad[0];
        for (int q = 1; q < TPB / 64; ++q) {
            lo = min(lo, slo[q]);
            hi = max(hi, shi[q]);
            b |= sbad[q];
        }
        if (b) lo = hi = (T)NAN;
    }
}

// per-block min and max (a non-finite value turns both into NaN)
__global__ __launch_bounds__(TPB) void k_minmax(const float *__restrict__ a, size_t n, double *__restrict__ partials)
{
    float lo = INFINITY, hi = -INFINITY;
    bool bad = false;
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t p = (size_t)blockIdx.x * TPB + threadIdx.x; p < n; p += stride) {
        const float x = a[p];
        bad |= !isfinite(x);
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
    }
    block_minmax(lo, hi, bad);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = lo;
        partials[2 * blockIdx.x + 1] = hi;
    }
}

// min and max over the nb blocks of k_minmax.  One workgroup reading the
// partials in parallel: at 128^3 (1024 blocks) a single thread walking them
// took 150 us, and the serial end of k_minmax 30 of its 37 us.
__global__ __launch_bounds__(TPB) void k_minmax_final(const double *__restrict__ partials, int nb,
                                                      double *__restrict__ out)
{
    double lo = INFINITY, hi = -INFINITY;
    bool bad = false;
    for (int q = threadIdx.x; q < nb; q += TPB) {
        const double l = partials[2 * q], h = partials[2 * q + 1];
        bad |= isnan(l) || isnan(h);
        lo = fmin(lo, l);
        hi = fmax(hi, h);
    }
    block_minmax(lo, hi, bad);
    if (threadIdx.x == 0) {
        out[0] = lo;
        out[1] = hi;
    }
}

__global__ __launch_bounds__(TPB) void k_axpy(float *y, const float *a, const float *b, float alpha,
                                              size_t n)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n; q += stride) y[q] = fmaf(alpha, b[q], a[q]);
}

__global__ __launch_bounds__(TPB) void k_scale(float *__restrict__ y, const float *__restrict__ a, float alpha,
                                               size_t n)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n; q += stride) y[q] = alpha * a[q];
}

// per-component sums of a 3-field vector: partials[c * nb + block]
__global__ __launch_bounds__(TPB) void k_comp_sums(const float *__restrict__ a, size_t n, double *__restrict__ partials)
{
    const int c = blockIdx.y;
    const float *x = a + c * n;
    double acc = 0.0;
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t p = (size_t)blockIdx.x * TPB + threadIdx.x; p < n; p += stride) acc += (double)x[p];
    acc = block_sum(acc);
    if (threadIdx.x == 0) partials[c * gridDim.x + blockIdx.x] = acc;
}

// The kernels on component c = blockIdx.y of a vector field take four values per
// access: n is a multiple of 4 and the fields are allocations of their own.
typedef float f4 __attribute__((ext_vector_type(4)));

// y_c = r_c - sum_c / n for the 3 components (sums on device)
__global__ __launch_bounds__(TPB) void k_mean_free(f4 *__restrict__ y, const f4 *__restrict__ r,
                                                   const double *__restrict__ sums, size_t n)
{
    const float mean = (float)(sums[blockIdx.y] / (double)n);
    const size_t off = blockIdx.y * (n / 4), stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n / 4; q += stride) y[off + q] = r[off + q] - mean;
}

// Fused PCG kernels.  Device scalars (FP64) in sc[]: see the PCG_* slots in
// internal.h.

// pHp = scale * (sum of the partials), alpha = rz / pHp; a non-positive
// curvature sets the flag and alpha = 0, so the update that follows leaves x
// and r unchanged
__global__ __launch_bounds__(TPB) void k_finalize_alpha(const double *__restrict__ partials, int nb, double scale,
                                                        double *__restrict__ sc)
{
    const double t = sum_partials(partials, nb);
    if (threadIdx.x != 0) return;
    const double pHp = scale * t, rz = sc[PCG_RZ];
    const bool ok = pHp > 0.0;
    sc[PCG_PHP] = pHp;
    sc[PCG_ALPHA] = ok ? rz / pHp : 0.0;
    sc[PCG_NEG] = ok ? 0.0 : 1.0;
}

// rz_new = scale * (sum of the partials), beta = rz_new / rz, then rz = rz_new
__global__ __launch_bounds__(FIN) void k_finalize_beta(const double *__restrict__ partials, int nb, double scale,
                                                       double *__restrict__ sc)
{
    const double t = sum_partials(partials, nb);
    if (threadIdx.x != 0) return;
    const double rznew = scale * t;
    sc[PCG_RZNEW] = rznew;
    sc[PCG_BETA] = rznew / sc[PCG_RZ];
    sc[PCG_RZ] = rznew;
}

// ||r||^2 (scaled) and the three component sums of r from the partials of
// k_pcg_update3, one workgroup per scalar
__global__ __launch_bounds__(TPB) void k_finalize_update3(const double *__restrict__ partials, int nb, double rscale,
                                                          double *__restrict__ sc)
{
    const int c = blockIdx.x;
    const double t = c == 0 ? sum_partials(partials, 3 * nb) : sum_partials(partials + (size_t)(2 + c) * nb, nb);
    if (threadIdx.x == 0) {
        if (c == 0) sc[PCG_RR] = rscale * t;
        else sc[PCG_SUMR + c - 1] = t;
    }
}

// x += alpha p, r -= alpha Hp on component c = blockIdx.y; per-block partial
// sums of r^2 (partials[c nb + b]) and of r (partials[(3 + c) nb + b]).  On small
// grids a chain of dependent loads and two block sums: one access a thread instead
// of four, 64^3 7.9 -> 6.6 us.
__global__ __launch_bounds__(TPB) void k_pcg_update3(f4 *__restrict__ x, f4 *__restrict__ r, const f4 *__restrict__ p,
                                                     const f4 *__restrict__ Hp, const double *__restrict__ sc, size_t n,
                                                     double *__restrict__ partials)
{
    const int c = blockIdx.y, nb = gridDim.x;
    const float alpha = (float)sc[PCG_ALPHA];
    double a2 = 0.0, a1 = 0.0;
    const size_t off = c * (n / 4), stride = (size_t)nb * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n / 4; q += stride) {
        f4 rq = r[off + q], xq = x[off + q];              // requested beside alpha
        const f4 pq = p[off + q], hq = Hp[off + q];
        if (alpha != 0.0f) {          // alpha = 0: curvature exit, x and r stay as they are
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xq[i] = fmaf(alpha, pq[i], xq[i]);
                rq[i] = fmaf(-alpha, hq[i], rq[i]);
            }
            x[off + q] = xq;
            r[off + q] = rq;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a2 += (double)rq[i] * (double)rq[i];
            a1 += (double)rq[i];
        }
    }
    a2 = block_sum(a2);
    if (threadIdx.x == 0) partials[c * nb + blockIdx.x] = a2;
    a1 = block_sum(a1);
    if (threadIdx.x == 0) partials[(3 + c) * nb + blockIdx.x] = a1;
}

__global__ void k_pcg_beta_flex(double *sc)
{
    sc[PCG_BETA] = (sc[PCG_RZNEW] - sc[PCG_RZOLD]) / sc[PCG_RZ];
    sc[PCG_RZ] = sc[PCG_RZNEW];
}

__global__ __launch_bounds__(TPB) void k_pcg_direction_lz(float *__restrict__ p, float *__restrict__ q,
                                                          const float *__restrict__ z, const float *__restrict__ Lz,
                                                          const double *__restrict__ sc, size_t n3)
{
    const float beta = (float)sc[PCG_BETA];
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n3; e += stride) {
        p[e] = fmaf(beta, p[e], z[e]);
        q[e] = Lz[e] + beta * q[e];
    }
}

// First inner step of the zero-velocity preconditioner: p = z, q = r (q = L_0 p),
// out = q + (G . p) G, and p . out per block
__global__ __launch_bounds__(TPB) void k_h0_apply(float *__restrict__ p, float *__restrict__ q,
                                                  const float *__restrict__ z, const float *__restrict__ r,
                                                  const float *__restrict__ G, float *__restrict__ out, size_t n,
                                                  double *__restrict__ partials)
{
    double acc = 0.0;
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n; e += stride) {
        float pn[3], qn[3], g[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t i = c * n + e;
            pn[c] = z[i];
            qn[c] = r[i];
            g[c] = G[i];
            p[i] = pn[c];
            q[i] = qn[c];
        }
        const float gp = g[0] * pn[0] + g[1] * pn[1] + g[2] * pn[2];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float o = fmaf(gp, g[c], qn[c]);
            out[c * n + e] = o;
            acc += (double)pn[c] * o;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

// Inner step of the zero-velocity preconditioner, the solution's update of the
// step before (which reads the same p), direction and operator in one pass: x +=
// alpha p, p = z + beta p, q = r + beta q (q = L_0 p), out = q + (G . p) G,
// per-block partials of p . out.  Streaming, 30 fields of 4 n bytes: 417 us at
// 256^3 (4.8 TB/s).  With the update of x beside that of r instead, the two
// passes of a step move 42 fields against 39.  FIRST: x = alpha p (no x before).
template <bool FIRST>
__global__ __launch_bounds__(TPB) void k_h0_direction_apply(float *__restrict__ x, float *__restrict__ p,
                                                            float *__restrict__ q, const float *__restrict__ z,
                                                            const float *__restrict__ r, const float *__restrict__ G,
                                                            float *__restrict__ out, const double *__restrict__ sc,
                                                            size_t n, double *__restrict__ partials)
{
    const float alpha = (float)sc[PCG_ALPHA], beta = (float)sc[PCG_BETA];
    double acc = 0.0;
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n; e += stride) {
        float pn[3], qn[3], g[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t i = c * n + e;
            const float po = p[i];
            x[i] = fmaf(alpha, po, FIRST ? 0.0f : x[i]);
            pn[c] = fmaf(beta, po, z[i]);
            qn[c] = r[i] + beta * q[i];
            p[i] = pn[c];
            q[i] = qn[c];
            g[c] = G[i];
        }
        const float gp = g[0] * pn[0] + g[1] * pn[1] + g[2] * pn[2];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float o = fmaf(gp, g[c], qn[c]);
            out[c * n + e] = o;
            acc += (double)pn[c] * o;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

// out = r - alpha H over 3 n values (alpha = sc[PCG_ALPHA]; no reductions), where
// the transform that follows does not form it while it reads
__global__ __launch_bounds__(TPB) void k_h0_residual(const float *r, const float *__restrict__ H,
                                                     const double *__restrict__ sc, float *out, size_t n3)
{
    const float alpha = (float)sc[PCG_ALPHA];
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n3; e += stride) out[e] = fmaf(-alpha, H[e], r[e]);
}

// x += alpha p, or x = alpha p, over 3 n values
template <bool FIRST>
__global__ __launch_bounds__(TPB) void k_h0_step(float *__restrict__ x, const float *__restrict__ p,
                                                 const double *__restrict__ sc, size_t n3)
{
    const float alpha = (float)sc[PCG_ALPHA];
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n3; e += stride)
        x[e] = fmaf(alpha, p[e], FIRST ? 0.0f : x[e]);
}

// p = z + beta p and q = (r - mean r) + beta q on component c = blockIdx.y (q is
// beta A p carried by recurrence; means from the component sums in sc, one FP64
// division a thread): 64^3 5.7 -> 5.0 us against a division per value
__global__ __launch_bounds__(TPB) void k_pcg_direction(f4 *__restrict__ p, f4 *__restrict__ q, const f4 *__restrict__ z,
                                                       const f4 *__restrict__ r, const double *__restrict__ sc,
                                                       size_t n)
{
    const float beta = (float)sc[PCG_BETA];
    const float mean = (float)(sc[PCG_SUMR + blockIdx.y] / (double)n);
    const size_t off = blockIdx.y * (n / 4), stride = (size_t)gridDim.x * TPB;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n / 4; e += stride) {
        f4 pe = p[off + e], qe = q[off + e];
        const f4 ze = z[off + e], re = r[off + e];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pe[i] = fmaf(beta, pe[i], ze[i]);
            qe[i] = (re[i] - mean) + beta * qe[i];
        }
        p[off + e] = pe;
        q[off + e] = qe;
    }
}

template <typename To>
__global__ __launch_bounds__(TPB) void k_convert(To *__restrict__ out, const float *__restrict__ in, size_t n)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n; q += stride) stf(out + q, in[q]);
}

template <typename Ti>
__global__ __launch_bounds__(TPB) void k_to_f32(const Ti *__restrict__ in, float *__restrict__ out, size_t n)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n; q += stride) out[q] = ldf(in + q);
}

// Streaming copy, 16 bytes per lane per iteration when aligned.
__global__ __launch_bounds__(TPB) void k_copy4(const float4 *__restrict__ src, float4 *__restrict__ dst, size_t n4)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n4; q += stride) dst[q] = src[q];
}

__global__ __launch_bounds__(TPB) void k_copy1(const float *__restrict__ src, float *__restrict__ dst, size_t n)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n; q += stride) dst[q] = src[q];
}

__global__ __launch_bounds__(TPB) void k_fill(float *__restrict__ dst, float v, size_t n)
{
    const size_t stride = (size_t)gridDim.x * TPB;
    for (size_t q = (size_t)blockIdx.x * TPB + threadIdx.x; q < n; q += stride) dst[q] = v;
}

inline dim3 stream_grid(size_t n)
{
    size_t b = (n + TPB - 1) / TPB;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    return dim3((unsigned)b);
}

} // namespace

int reduce_blocks(size_t n)
{
    size_t b = (n + TPB * 4 - 1) / (TPB * 4);
    if (b > 2048) b = 2048;
    if (b < 1) b = 1;
    return (int)b;
}

void launch_dot(const float *a, const float *b, size_t n, double *partials, int nblocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_dot, dim3(nblocks), dim3(TPB), 0, s, a, b, n, partials);
}

void launch_count_nonfinite(const float *a, float *copy, size_t n, double *partials, int nblocks, hipStream_t s)
{
    if ((((uintptr_t)a | (uintptr_t)copy) & 15) == 0 && n % 4 == 0)
        hipLaunchKernelGGL(k_count_nonfinite<4>, dim3(nblocks), dim3(TPB), 0, s, a, copy, n, partials);
    else
        hipLaunchKernelGGL(k_count_nonfinite<1>, dim3(nblocks), dim3(TPB), 0, s, a, copy, n, partials);
}

void launch_minmax(const float *a, size_t n, double *partials, int nblocks, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_minmax, dim3(nblocks), dim3(TPB), 0, s, a, n, partials);
    hipLaunchKernelGGL(k_minmax_final, dim3(1), dim3(TPB), 0, s, partials, nblocks, out);
}

void launch_finalize(const double *partials, int nblocks, double scale, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(finalize_threads(nblocks)), 0, s, partials, nblocks, scale, out);
}

void launch_axpy(float *y, const float *a, const float *b, float alpha, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_axpy, stream_grid(n), dim3(TPB), 0, s, y, a, b, alpha, n);
}

void launch_scale(float *y, const float *a, float alpha, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_scale, stream_grid(n), dim3(TPB), 0, s, y, a, alpha, n);
}

void launch_comp_sums3(const float *a, size_t n, double *partials, int nblocks, double *sums_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_comp_sums, dim3(nblocks, 3), dim3(TPB), 0, s, a, n, partials);
    hipLaunchKernelGGL(k_finalize_rows, dim3(3), dim3(TPB), 0, s, partials, nblocks, sums_out);
}

void launch_mean_free(float *y, const float *r, const double *sums, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_mean_free, dim3(reduce_blocks(n), 3), dim3(TPB), 0, s, (f4 *)y, (const f4 *)r, sums, n);
}

void launch_finalize_alpha(const double *partials, int nblocks, double scale, double *sc, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize_alpha, dim3(1), dim3(TPB), 0, s, partials, nblocks, scale, sc);
}

void launch_finalize_beta(const double *partials, int nblocks, double scale, double *sc, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize_beta, dim3(1), dim3(finalize_threads(nblocks)), 0, s, partials, nblocks, scale, sc);
}

void launch_pcg_update3(float *x, float *r, const float *p, const float *Hp, double *sc, size_t n, double *partials,
                        int nblocks, double rscale, hipStream_t s)
{
    hipLaunchKernelGGL(k_pcg_update3, dim3(nblocks, 3), dim3(TPB), 0, s, (f4 *)x, (f4 *)r, (const f4 *)p,
                       (const f4 *)Hp, sc, n, partials);
    hipLaunchKernelGGL(k_finalize_update3, dim3(4), dim3(TPB), 0, s, partials, nblocks, rscale, sc);
}

void launch_pcg_beta_flex(double *sc, hipStream_t s)
{
    hipLaunchKernelGGL(k_pcg_beta_flex, dim3(1), dim3(1), 0, s, sc);
}

void launch_pcg_direction_lz(float *p, float *q, const float *z, const float *Lz, const double *sc, size_t n,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_pcg_direction_lz, stream_grid(3 * n), dim3(TPB), 0, s, p, q, z, Lz, sc, 3 * n);
}

void launch_h0_direction_apply(float *x, bool first, float *p, float *q, const float *z, const float *r, const float *G,
                               float *out, const double *sc, size_t n, double *partials, int nblocks, hipStream_t s)
{
    if (first)
        hipLaunchKernelGGL(k_h0_direction_apply<true>, dim3(nblocks), dim3(TPB), 0, s, x, p, q, z, r, G, out, sc, n,
                           partials);
    else
        hipLaunchKernelGGL(k_h0_direction_apply<false>, dim3(nblocks), dim3(TPB), 0, s, x, p, q, z, r, G, out, sc, n,
                           partials);
}

void launch_h0_residual(const float *r, const float *H, const double *sc, float *out, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_h0_residual, stream_grid(3 * n), dim3(TPB), 0, s, r, H, sc, out, 3 * n);
}

void launch_h0_step(float *x, bool first, const float *p, const double *sc, size_t n, hipStream_t s)
{
    if (first) hipLaunchKernelGGL(k_h0_step<true>, stream_grid(3 * n), dim3(TPB), 0, s, x, p, sc, 3 * n);
    else hipLaunchKernelGGL(k_h0_step<false>, stream_grid(3 * n), dim3(TPB), 0, s, x, p, sc, 3 * n);
}

void launch_h0_apply(float *p, float *q, const float *z, const float *r, const float *G, float *out, size_t n,
                     double *partials, int nblocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_h0_apply, dim3(nblocks), dim3(TPB), 0, s, p, q, z, r, G, out, n, partials);
}

void launch_pcg_direction(float *p, float *q, const float *z, const float *r, const double *sc, size_t n,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_pcg_direction, dim3(reduce_blocks(n), 3), dim3(TPB), 0, s, (f4 *)p, (f4 *)q, (const f4 *)z,
                       (const f4 *)r, sc, n);
}

void launch_convert(int dt_out, void *out, const float *in, size_t n, hipStream_t s)
{
    with_dtype(dt_out, [&](auto to) {
        using To = decltype(to);
        hipLaunchKernelGGL((k_convert<To>), stream_grid(n), dim3(TPB), 0, s, (To *)out, in, n);
    });
}

void launch_to_f32(int dt_in, const void *in, float *out, size_t n, hipStream_t s)
{
    with_dtype(dt_in, [&](auto ti) {
        using Ti = decltype(ti);
        hipLaunchKernelGGL((k_to_f32<Ti>), stream_grid(n), dim3(TPB), 0, s, (const Ti *)in, out, n);
    });
}

void launch_copy_f32(const float *src, float *dst, size_t n, hipStream_t s)
{
    if (((uintptr_t)src % 16) == 0 && ((uintptr_t)dst % 16) == 0 && n % 4 == 0)
        hipLaunchKernelGGL(k_copy4, stream_grid(n / 4), dim3(TPB), 0, s, (const float4 *)src, (float4 *)dst, n / 4);
    else
        hipLaunchKernelGGL(k_copy1, stream_grid(n), dim3(TPB), 0, s, src, dst, n);
}

void launch_fill_f32(float *dst, float v, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill, stream_grid(n), dim3(TPB), 0, s, dst, v, n);
}

} // namespace clh
