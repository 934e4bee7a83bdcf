// k_fft.hip -- 3D real FFT spectral operators for gfx950 (Section 2.2: a
// spectral operator costs two FFTs and one Hadamard product; Section 3 uses
// a vendor 3D FFT on one GPU, here it is written from scratch).
//
// Layout: real fields [n1][n2][n3]; half spectrum [n1][n2][np]: nh = n3/2+1
// values per row at a row pitch np of nh rounded up to 16 (128-byte rows).
// One spectral apply is five passes, each a single read and a single write
// of the field:
//   x3 R2C    rows of n3 reals packed as M = n3/2 complex, complex FFT of
//             length M, split into the half spectrum of the real row;
//   x2 C2C    columns of a fixed-x1 plane;
//   x1 fused  columns along x1: forward FFT, Hadamard multiply by the
//             symbol, inverse FFT, all in one LDS tile;
//   x2 C2C    inverse;
//   x3 C2R    Hermitian merge, inverse FFT of length M, unpack to reals,
//             optional fused add.
// Columns of 64 ... 1024 and rows of 128 ... 1024 points take register-resident
// passes (below); the generic passes for shorter lines work on LDS tiles: a workgroup owns a
// tile of nl lines x L points (nl L <= 2048 complex, 16 KB), coalesced
// batched loads into LDS, then Stockham stages of radix 8 (and one of
// radix 2/4 for the remainder) with every group's R values in registers,
// twiddles from FP64-computed tables staged in LDS, and a coalesced store.
// The LDS tile is stored as [q][l] with pitch nl + 1 so that both row-wise and
// column-wise accesses are conflict-free.  Grids of such lines are small and
// a pass lasts as long as one tile: radix 16 on tiles of 4096 values left half
// the threads of a stage idle behind the other half's longer chains.  Planes of
// at most 64 x 64 points, up to 2048 of them, do their x3 and x2 passes in one kernel (k_fft_plane),
// three passes in all: a 64^3 vector 49 -> 29 us (26 with the x1
// pass in registers), 32^3 35 -> 18 us.
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace clh {

namespace {

constexpr int TPB = 256;
constexpr int TILE = 2048;   // complex values per LDS tile of the Stockham passes
constexpr int EPT = TILE / TPB;

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }

// cos / sin of 2 pi k / 16, k = 0..7 (folded at compile time)
__device__ __forceinline__ constexpr float c16(int k)
{
    return k == 0 ? 1.0f : k == 1 ? 0.92387953251128674f : k == 2 ? 0.70710678118654752f
         : k == 3 ? 0.38268343236508977f : k == 4 ? 0.0f : k == 5 ? -0.38268343236508977f
         : k == 6 ? -0.70710678118654752f : -0.92387953251128674f;
}
__device__ __forceinline__ constexpr float s16(int k)
{
    return k == 0 ? 0.0f : k == 1 ? 0.38268343236508977f : k == 2 ? 0.70710678118654752f
         : k == 3 ? 0.92387953251128674f : k == 4 ? 1.0f : k == 5 ? 0.92387953251128674f
         : k == 6 ? 0.70710678118654752f : 0.38268343236508977f;
}

template <int R> __device__ constexpr int brev_c(int i)
{
    int r = 0;
    for (int b = 1; b < R; b <<= 1) {
        r <<= 1;
        if (i & b) r |= 1;
    }
    return r;
}

// y * e^{-+2 pi i k / 16}; k is a compile-time constant after unrolling
template <bool INV> __device__ __forceinline__ float2 rot16(float2 y, int k)
{
    if (k == 0) return y;
    if (k == 4) return INV ? make_float2(-y.y, y.x) : make_float2(y.y, -y.x);
    const float c = c16(k), s = INV ? s16(k) : -s16(k);
    return make_float2(y.x * c - y.y * s, y.x * s + y.y * c);
}

// In-register DFT of length R (2, 4, 8, 16), natural order in and out:
// radix-2 DIT after a compile-time bit-reversal (register renaming only).
template <int R, bool INV> __device__ __forceinline__ void dft_reg(float2 *v)
{
    float2 a[R];
#pragma unroll
    for (int i = 0; i < R; ++i) a[i] = v[brev_c<R>(i)];
#pragma unroll
    for (int len = 2; len <= R; len <<= 1) {
#pragma unroll
        for (int s = 0; s < R; s += len) {
#pragma unroll
            for (int k = 0; k < len / 2; ++k) {
                const float2 x = a[s + k];
                const float2 y = rot16<INV>(a[s + k + len / 2], k * (16 / len));
                a[s + k] = cadd(x, y);
                a[s + k + len / 2] = csub(x, y);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = a[i];
}

// One Stockham radix-R stage in place on the LDS tile (element (l, q) at
// q * P + l), for nl = 2^lognl lines of length L = 2^logL; Ns = 2^logNs is
// the product of the radices of the earlier stages.  tw[t] = e^{-2 pi i t / L}
// (t < L).  Every thread reads all its groups, the workgroup synchronises,
// then the results are written back, so the stage is safe in place.
template <int R, bool INV, int NT>
__device__ __forceinline__ void stage(float2 *lds, int P, int lognl, int logL, int logNs, const float2 *tw)
{
    constexpr int LOGR = R == 2 ? 1 : R == 4 ? 2 : 3;
    constexpr int G = EPT / R;          // groups per thread (the tile holds EPT values per thread)
    const int nl = 1 << lognl, L = 1 << logL, Ns = 1 << logNs;
    const int ngroups = nl << (logL - LOGR);
    const int LR = L >> LOGR;
    float2 v[G][R];
#pragma unroll
    for (int gq = 0; gq < G; ++gq) {
        const int gi = gq * NT + threadIdx.x;
        if (gi < ngroups) {
            const int l = gi & (nl - 1), j = gi >> lognl;
#pragma unroll
            for (int r = 0; r < R; ++r) v[gq][r] = lds[(j + r * LR) * P + l];
        }
    }
    __syncthreads();
#pragma unroll
    for (int gq = 0; gq < G; ++gq) {
        const int gi = gq * NT + threadIdx.x;
        if (gi < ngroups) {
            const int l = gi & (nl - 1), j = gi >> lognl;
            const int jm = j & (Ns - 1);
            if (logNs > 0) {
                const int tsh = logL - logNs - LOGR;
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    float2 w = tw[(r * jm) << tsh];
                    if (INV) w.y = -w.y;
                    v[gq][r] = cmul(v[gq][r], w);
                }
            }
            dft_reg<R, INV>(v[gq]);
            const int base = ((j >> logNs) << (logNs + LOGR)) + jm;
#pragma unroll
            for (int r = 0; r < R; ++r) lds[(base + r * Ns) * P + l] = v[gq][r];
        }
    }
    __syncthreads();
}

// Full FFT of the tile's lines: radix-8 stages, then one radix-2/4 stage.
// NT threads per workgroup, EPT values per thread.
template <bool INV, int NT = TPB> __device__ void fft_lines(float2 *lds, int P, int lognl, int logL, const float2 *tw)
{
    int logNs = 0;
    while (logL - logNs >= 3) {
        stage<8, INV, NT>(lds, P, lognl, logL, logNs, tw);
        logNs += 3;
    }
    const int rem = logL - logNs;
    if (rem == 2) stage<4, INV, NT>(lds, P, lognl, logL, logNs, tw);
    else if (rem == 1) stage<2, INV, NT>(lds, P, lognl, logL, logNs, tw);
}

template <int NT = TPB> __device__ __forceinline__ void load_table(float2 *dst, const float2 *__restrict__ src, int n)
{
    for (int t = threadIdx.x; t < n; t += NT) dst[t] = src[t];
}

// --- x3 forward: real rows -> half spectrum.  nl = 2^lognl rows per tile.
__global__ __launch_bounds__(TPB) void k_fft_x3_r2c(const float *__restrict__ in, float2 *__restrict__ spec,
                                                    const float2 *__restrict__ twM, const float2 *__restrict__ tw3,
                                                    int logM, int lognl, int nrows, size_t in_cs, size_t spec_cs,
                                                    int np)
{
    extern __shared__ float2 sm[];
    const int M = 1 << logM, nl = 1 << lognl, P = nl + 1, nh = M + 1;
    float2 *twm = sm;                 // M: e^{-2 pi i t / M}
    float2 *tws = sm + M;             // M + 1: e^{-2 pi i k / n3}, k <= M
    float2 *lds = tws + M + 1;        // M * P
    const int comp = blockIdx.y;
    const float2 *src = (const float2 *)(in + comp * in_cs);
    float2 *dst = spec + comp * spec_cs;
    const int row0 = blockIdx.x * nl;
    load_table(twm, twM, M);
    load_table(tws, tw3, M + 1);
    const int tot = nl << logM;
    float2 buf[EPT];
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = it * TPB + threadIdx.x;
        if (e < tot) buf[it] = src[(size_t)row0 * M + e];
    }
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = it * TPB + threadIdx.x;
        if (e < tot) lds[(e & (M - 1)) * P + (e >> logM)] = buf[it];
    }
    __syncthreads();
    fft_lines<false>(lds, P, lognl, logM, twm);
    // X[k] = E[k] + w^k O[k], E = (Z[k] + conj Z[M-k]) / 2, O = -i (Z[k] - conj Z[M-k]) / 2
    const int totk = nl * nh;
    for (int e = threadIdx.x; e < totk; e += TPB) {
        const int r = e / nh, k = e - r * nh;
        const float2 zk = lds[(k & (M - 1)) * P + r];
        const float2 zc = cconj(lds[((M - k) & (M - 1)) * P + r]);
        const float2 E = make_float2(0.5f * (zk.x + zc.x), 0.5f * (zk.y + zc.y));
        const float2 O = make_float2(0.5f * (zk.y - zc.y), -0.5f * (zk.x - zc.x));
        dst[(size_t)(row0 + r) * np + k] = cadd(E, cmul(tws[k], O));
    }
}

// --- x3 inverse: half spectrum -> real rows (unnormalised), optional add; the
// values k >= kmax are zero and not read.
__global__ __launch_bounds__(TPB) void k_fft_x3_c2r(const float2 *__restrict__ spec, float *__restrict__ out,
                                                    const float *__restrict__ add, const float2 *__restrict__ twM,
                                                    const float2 *__restrict__ tw3, int logM, int lognl, int nrows,
                                                    size_t out_cs, size_t spec_cs, int np, int kmax)
{
    extern __shared__ float2 sm[];
    const int M = 1 << logM, nl = 1 << lognl, P = nl + 1, nh = M + 1;
    float2 *twm = sm;
    float2 *tws = sm + M;
    float2 *lds = tws + M + 1;
    const int comp = blockIdx.y;
    const float2 *src = spec + comp * spec_cs;
    float2 *dst = (float2 *)(out + comp * out_cs);
    const float2 *ad = add ? (const float2 *)(add + comp * out_cs) : nullptr;
    const int row0 = blockIdx.x * nl;
    load_table(twm, twM, M);
    load_table(tws, tw3, M + 1);
    // stage the half-spectrum rows (nh values each) at lds[k * P + r], k <= M
    // (row M of the tile doubles as the Nyquist slot; the tile has M + 1 rows).
    // nl * nh = TILE + nl <= TILE + TILE / 8 values (M >= 8), i.e. at most
    // EPT + EPT / 8 = EPT + 1 per thread, all of them in use at M = 8.
    const int totk = nl * nh;
    {
        constexpr int NB = EPT + EPT / 8;
        static_assert(NB * TPB >= TILE + TILE / 8, "a thread's buffer holds its share of the widest tile");
        float2 buf[NB];
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            const int e = it * TPB + threadIdx.x;
            if (e < totk) {
                const int r = e / nh, k = e - r * nh;
                buf[it] = k < kmax ? src[(size_t)(row0 + r) * np + k] : make_float2(0.f, 0.f);
            }
        }
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            const int e = it * TPB + threadIdx.x;
            if (e < totk) {
                const int r = e / nh, k = e - r * nh;
                lds[k * P + r] = buf[it];
            }
        }
    }
    __syncthreads();
    // Z[k] = (X[k] + conj X[M-k]) + i e^{+2 pi i k / n3} (X[k] - conj X[M-k]),  k < M
    float2 z[EPT];
    const int tot = nl << logM;
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = it * TPB + threadIdx.x;
        if (e < tot) {
            const int r = e & (nl - 1), k = e >> lognl;
            const float2 a = lds[k * P + r], b = cconj(lds[(M - k) * P + r]);
            const float2 sum = cadd(a, b), dif = csub(a, b);
            const float2 wd = cmul(cconj(tws[k]), dif);
            z[it] = make_float2(sum.x - wd.y, sum.y + wd.x);
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = it * TPB + threadIdx.x;
        if (e < tot) lds[(e >> lognl) * P + (e & (nl - 1))] = z[it];
    }
    __syncthreads();
    fft_lines<true>(lds, P, lognl, logM, twm);
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = it * TPB + threadIdx.x;
        if (e < tot) {
            const int r = e >> logM, n = e & (M - 1);
            float2 v = lds[n * P + r];
            const size_t o = (size_t)row0 * M + e;
            if (ad) {
                const float2 a = ad[o];
                v.x += a.x;
                v.y += a.y;
            }
            dst[o] = v;
        }
    }
}

// --- x3 and x2 passes of one x1 plane in one workgroup (planes of at most 64 x
// 64 points), forward: real rows -> half spectrum -> columns; inverse the other
// way, with the optional add, from the values k < kmax of the rows |k2| < m2
// (the others are zero and not read).  Same line transforms as the separate passes; the
// plane stays in LDS between them, as rows [q][row] (pitch n2 + 1) and as
// columns [row][k] (pitch NL + 1, NL >= n3 / 2 + 1 a power of two).
// Separate passes at 64^3: 11 + 7 us forward, 7 + 12 us inverse; one kernel 10
// and 9 us, bound by the latency of its stages.
constexpr int NTP = 512;            // threads, EPT = 8 values each: 64 x 64

template <bool INV>
__global__ __launch_bounds__(NTP) void k_fft_plane(const float *__restrict__ in, float *__restrict__ out,
                                                   const float *__restrict__ add, float2 *__restrict__ spec,
                                                   const float2 *__restrict__ twM, const float2 *__restrict__ tw3,
                                                   const float2 *__restrict__ tw2, int logM, int logn2, int logNL,
                                                   size_t cs, size_t spec_cs, int np, int kmax, int m2)
{
    extern __shared__ float2 sm[];
    const int M = 1 << logM, n2 = 1 << logn2, NL = 1 << logNL, PR = n2 + 1, PC = NL + 1;
    float2 *twm = sm;                 // M: e^{-2 pi i t / M}
    float2 *tws = twm + M;            // M + 1: e^{-2 pi i k / n3}
    float2 *twc = tws + M + 1;        // n2
    float2 *lds = twc + n2;
    const int comp = blockIdx.y;
    const size_t row0 = (size_t)blockIdx.x << logn2;
    float2 *sp = spec + comp * spec_cs + row0 * np;
    load_table<NTP>(twm, twM, M);
    load_table<NTP>(tws, tw3, M + 1);
    load_table<NTP>(twc, tw2, n2);
    const int rows = n2 << logM, cols = n2 << logNL;   // values as rows, as columns
    float2 v[EPT];
    if (!INV) {
        const float2 *src = (const float2 *)(in + comp * cs) + row0 * M;
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < rows) v[it] = src[e];
        }
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < rows) lds[(e & (M - 1)) * PR + (e >> logM)] = v[it];
        }
        __syncthreads();
        fft_lines<false, NTP>(lds, PR, logn2, logM, twm);
        // X[k] = E[k] + w^k O[k] (see k_fft_x3_r2c), k <= M
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x, k = e & (NL - 1), r = e >> logNL;
            v[it] = make_float2(0.f, 0.f);
            if (e < cols && k <= M) {
                const float2 zk = lds[(k & (M - 1)) * PR + r];
                const float2 zc = cconj(lds[((M - k) & (M - 1)) * PR + r]);
                const float2 E = make_float2(0.5f * (zk.x + zc.x), 0.5f * (zk.y + zc.y));
                const float2 O = make_float2(0.5f * (zk.y - zc.y), -0.5f * (zk.x - zc.x));
                v[it] = cadd(E, cmul(tws[k], O));
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < cols) lds[(e >> logNL) * PC + (e & (NL - 1))] = v[it];
        }
        __syncthreads();
        fft_lines<false, NTP>(lds, PC, logNL, logn2, twc);
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x, k = e & (NL - 1), r = e >> logNL;
            if (e < cols && k <= M) sp[(size_t)r * np + k] = lds[r * PC + k];
        }
    } else {
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x, k = e & (NL - 1), r = e >> logNL;
            v[it] = e < cols && k < kmax && (r < m2 || r > n2 - m2) ? sp[(size_t)r * np + k] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < cols) lds[(e >> logNL) * PC + (e & (NL - 1))] = v[it];
        }
        __syncthreads();
        fft_lines<true, NTP>(lds, PC, logNL, logn2, twc);
        // Z[k] (see k_fft_x3_c2r), k < M
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < rows) {
                const int k = e & (M - 1), r = e >> logM;
                const float2 a = lds[r * PC + k], b = cconj(lds[r * PC + M - k]);
                const float2 sum = cadd(a, b), dif = csub(a, b);
                const float2 wd = cmul(cconj(tws[k]), dif);
                v[it] = make_float2(sum.x - wd.y, sum.y + wd.x);
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < rows) lds[(e & (M - 1)) * PR + (e >> logM)] = v[it];
        }
        __syncthreads();
        fft_lines<true, NTP>(lds, PR, logn2, logM, twm);
        float2 *dst = (float2 *)(out + comp * cs) + row0 * M;
        const float2 *ad = add ? (const float2 *)(add + comp * cs) + row0 * M : nullptr;
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = it * NTP + threadIdx.x;
            if (e < rows) {
                float2 x = lds[(e & (M - 1)) * PR + (e >> logM)];
                if (ad) {
                    const float2 a = ad[e];
                    x.x += a.x;
                    x.y += a.y;
                }
                dst[e] = x;
            }
        }
    }
}

// <in, out> of a spectral operation from its x1 pass (Parseval): the sum of w
// |X|^2 sym over the half spectrum, w = 2 off the planes k3 = 0 and k3 = n3 / 2,
// in FP64, one partial per workgroup (sym carries the transform's 1 / N).  A dot
// product of the two fields reads both again: 402 MB, 102 us at 256^3, against 1.5 us
// more in this pass (75.0 -> 76.5).
__device__ __forceinline__ double dot_term(float2 x, float sym, bool edge)
{
    const double m = (double)x.x * x.x + (double)x.y * x.y;
    return (edge ? 1.0 : 2.0) * (double)sym * m;
}
__device__ __forceinline__ void dot_store(double acc, double *__restrict__ partials)
{
    acc = block_sum(acc);
    if (threadIdx.x == 0)
        partials[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = acc;
}

// Pruned column passes (spectral resampling): of the La-point lines of a source
// spectrum only the rows |k| < m are read, as the rows |k| < m of lines of L
// points, the others are zero; and only the planes |k| < mp are visited.  A
// pass with m = mp = L and dplane = 0 is the plain one.
struct ColSrc {
    const float2 *src;   // spectrum read, components cs apart, planes ps, rows rs
    size_t cs, ps, rs;
    int La, m;           // points of a source line, kept rows
    int mp, skip;        // kept planes, planes left out (N - (2 mp - 1), or 0)
    int dplane;          // source planes minus planes (for negative k)
    float scale;         // of every value read
};

// plane of the j-th kept one, and its source plane
__device__ __forceinline__ int kept_plane(const ColSrc &c, int j) { return j < c.mp ? j : j + c.skip; }
__device__ __forceinline__ const float2 *src_plane(const ColSrc &c, int comp, int j, int c0)
{
    return c.src + comp * c.cs + (size_t)(j < c.mp ? j : j + c.skip + c.dplane) * c.ps + c0;
}
// row q of an L-point line
__device__ __forceinline__ float2 src_row(const ColSrc &c, const float2 *__restrict__ base, int q, int L, int l, bool ok)
{
    if (!ok || (q >= c.m && q <= L - c.m)) return make_float2(0.f, 0.f);
    const float2 v = base[(size_t)(q < c.m ? q : q + c.La - L) * c.rs + l];
    return make_float2(v.x * c.scale, v.y * c.scale);
}

// --- column tile load/store for the x2 and x1 passes: element (l, q) of
// the tile is base[q * rs + l], l < cw valid columns; NT threads.  A thread
// keeps its column l and steps through the rows q0, q0 + NT / C, ...: the
// row part of an address is wave-uniform (a scalar base), the thread's part a
// 32-bit byte offset of at most NT / C - 1 = 7 rows, below half of one component's
// half spectrum (lines of 16 or 32 points: at most 138 MB, 32 x 1024 x 1024).
template <int NT>
__device__ __forceinline__ void load_cols(float2 *lds, const float2 *__restrict__ base, size_t rs, int logC, int logL,
                                          int cw, int P)
{
    const int C = 1 << logC, L = 1 << logL;
    const int l = threadIdx.x & (C - 1), q0 = threadIdx.x >> logC, QS = NT >> logC;
    const unsigned off = (unsigned)(((size_t)q0 * rs + l) * sizeof(float2));
    float2 buf[EPT];
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const char *row = (const char *)(base + (size_t)it * QS * rs);
        if (q0 + it * QS < L) buf[it] = l < cw ? *(const float2 *)(row + off) : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int it = 0; it < EPT; ++it)
        if (q0 + it * QS < L) lds[(q0 + it * QS) * P + l] = buf[it];
    __syncthreads();
}

// the same through a ColSrc
template <int NT>
__device__ __forceinline__ void load_cols_src(float2 *lds, const ColSrc &c, const float2 *__restrict__ base, int logC,
                                              int logL, int cw, int P)
{
    const int C = 1 << logC, L = 1 << logL;
    const int l = threadIdx.x & (C - 1), q0 = threadIdx.x >> logC, QS = NT >> logC;
    float2 buf[EPT];
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int q = q0 + it * QS;
        if (q < L) buf[it] = src_row(c, base, q, L, l, l < cw);
    }
#pragma unroll
    for (int it = 0; it < EPT; ++it)
        if (q0 + it * QS < L) lds[(q0 + it * QS) * P + l] = buf[it];
    __syncthreads();
}

template <int NT>
__device__ __forceinline__ void store_cols(const float2 *lds, float2 *__restrict__ base, size_t rs, int logC, int logL,
                                           int cw, int P)
{
    const int C = 1 << logC, L = 1 << logL;
    const int l = threadIdx.x & (C - 1), q0 = threadIdx.x >> logC, QS = NT >> logC;
    const unsigned off = (unsigned)(((size_t)q0 * rs + l) * sizeof(float2));
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        char *row = (char *)(base + (size_t)it * QS * rs);
        if (q0 + it * QS < L && l < cw) *(float2 *)(row + off) = lds[(q0 + it * QS) * P + l];
    }
}

// --- x2 C2C in place on the half spectrum: plane i1 = blockIdx.y, columns
// [c0, c0 + C) of the nh per row; NT threads hold the tile of NT EPT values.
template <bool INV, int NT, bool PR>
__global__ __launch_bounds__(NT) void k_fft_x2(float2 *spec, const float2 *__restrict__ tw2, int logn2,
                                                int n2, int nh, int np, int logC, size_t spec_cs, ColSrc from)
{
    extern __shared__ float2 sm[];
    const int C = 1 << logC, P = C + 1;
    float2 *tw = sm;
    float2 *lds = sm + n2;
    const int comp = blockIdx.z, i1 = blockIdx.y, c0 = blockIdx.x * C;
    const int cw = min(C, nh - c0);
    float2 *base = spec + comp * spec_cs + (size_t)i1 * n2 * np + c0;
    load_table<NT>(tw, tw2, n2);
    if (PR) load_cols_src<NT>(lds, from, src_plane(from, comp, i1, c0), logC, logn2, cw, P);
    else load_cols<NT>(lds, base, np, logC, logn2, cw, P);
    fft_lines<INV, NT>(lds, P, logC, logn2, tw);
    store_cols<NT>(lds, base, np, logC, logn2, cw, P);
}

// --- x1 fused: forward FFT along x1, symbol multiply, inverse FFT.
// plane i2 = blockIdx.y, columns [c0, c0 + C).
// mode 0: forward, multiply, inverse; 1: forward only; 2: inverse only
template <int NT, bool PR>
__global__ __launch_bounds__(NT) void k_fft_x1_mult(float2 *spec, const float2 *__restrict__ tw1,
                                                     int logn1, int n1, int n2, int nh, int np, int logC, int kind,
                                                     float beta, float scale, size_t spec_cs, int mode, ColSrc from,
                                                     double *__restrict__ dot)
{
    extern __shared__ float2 sm[];
    const int C = 1 << logC, P = C + 1;
    float2 *tw = sm;
    float2 *lds = sm + n1;
    const int comp = blockIdx.z, i2 = PR ? kept_plane(from, blockIdx.y) : blockIdx.y, c0 = blockIdx.x * C;
    const int cw = min(C, nh - c0);
    float2 *base = spec + comp * spec_cs + (size_t)i2 * np + c0;
    const size_t rs = (size_t)n2 * np;
    load_table<NT>(tw, tw1, n1);
    if (PR) load_cols_src<NT>(lds, from, src_plane(from, comp, blockIdx.y, c0), logC, logn1, cw, P);
    else load_cols<NT>(lds, base, rs, logC, logn1, cw, P);
    if (mode == 2) {
        fft_lines<true, NT>(lds, P, logC, logn1, tw);
        store_cols<NT>(lds, base, rs, logC, logn1, cw, P);
        return;
    }
    fft_lines<false, NT>(lds, P, logC, logn1, tw);
    if (mode == 1) {
        store_cols<NT>(lds, base, rs, logC, logn1, cw, P);
        return;
    }
    const float k2 = (float)(i2 < (n2 >> 1) ? i2 : i2 - n2);
    const int tot = C << logn1;
    double acc = 0.0;
    for (int e = threadIdx.x; e < tot; e += NT) {
        const int l = e & (C - 1), q = e >> logC;
        const float k1 = (float)(q < (n1 >> 1) ? q : q - n1);
        const float k3 = (float)(c0 + l);
        const float ksq = k1 * k1 + k2 * k2 + k3 * k3;
        float sym;
        if (kind == 0) sym = beta * ksq;
        else if (kind == 1) sym = 1.0f / (beta * fmaxf(ksq, 1.0f));
        else sym = 1.0f;
        sym *= scale;
        float2 &x = lds[q * P + l];
        if (dot && l < cw) acc += dot_term(x, sym, c0 + l == 0 || c0 + l == nh - 1);
        x.x *= sym;
        x.y *= sym;
    }
    if (dot) dot_store(acc, dot);
    __syncthreads();
    fft_lines<true, NT>(lds, P, logC, logn1, tw);
    store_cols<NT>(lds, base, rs, logC, logn1, cw, P);
}

// --- register-resident column passes for lines of L = 16 R2 points (R2 =
// 4, 8 or 16, i.e. L = 64, 128 or 256; 512 and 1024 below) in tiles of C = 256 /
// R2 columns.  On small grids a pass lasts as long as one tile: lines of 64 points
// cross LDS twice here, eight times in the Stockham pass, 11.2 -> 8.3 us at 64^3
// with the sum of <x, P x>, and an operation on 64 x 256 x 256 116 -> 100 us; lines
// of 32 took 5.8 us either way and stay there
// (tiles of 128 columns, of which a 32^3 row fills 17).  With
// n = R2 a + b and k = c + 16 d,
//   X[c + 16 d] = sum_b W_R2^{bd} W_L^{bc} sum_a x[R2 a + b] W_16^{ac},
// so each thread holds 16 (or 2 x R2) values in registers: the length-16
// DFTs over a run on the "b" layout (thread = column l, residue b), the
// length-R2 DFTs over b on the "c" layout (thread = column l, c), and one
// LDS exchange [c][b][l] (pitch 272 complex per c: row reads and writes of a
// half-wavefront hit distinct banks) connects them.  The inverse runs the
// same steps backwards.  A tile therefore crosses LDS twice per transform
// (Stockham stages in LDS cross it four times plus the staging).
// MODE 0: forward, symbol multiply (x1 pass), inverse; 1: forward only;
// 2: inverse only.  Element (row q, column l) of the tile is base[q rs + l].
constexpr int CSC = 272;   // LDS pitch per c (R2 C + 16 complex)

template <int R2>
__device__ __forceinline__ void cols_load_b(float2 (&v)[16], const float2 *__restrict__ base, size_t rs, int l, int b,
                                            bool ok)
{
#pragma unroll
    for (int a = 0; a < 16; ++a) v[a] = ok ? base[(size_t)(R2 * a + b) * rs + l] : make_float2(0.f, 0.f);
}

template <int R2, int MODE, bool PR, bool DOT>
__global__ __launch_bounds__(TPB) void k_fft_cols(float2 *spec, const float2 *__restrict__ twL,
                                                  int nh, size_t plane_stride, size_t rs, size_t spec_cs, int kind,
                                                  float beta, float scale, int n1, int n2, ColSrc from,
                                                  double *__restrict__ dot)
{
    constexpr int L = 16 * R2, C = 256 / R2, P2 = C / 16;   // P2: (l, c) pairs per thread
    __shared__ float2 tw[L];
    __shared__ float2 ex[16 * CSC];
    const int comp = blockIdx.z, pl = PR ? kept_plane(from, blockIdx.y) : blockIdx.y, c0 = blockIdx.x * C;
    const int cw = min(C, nh - c0);
    float2 *base = spec + comp * spec_cs + pl * plane_stride + c0;
    const float2 *sb = PR ? src_plane(from, comp, blockIdx.y, c0) : base;
    for (int t = threadIdx.x; t < L; t += TPB) tw[t] = twL[t];
    const int l = threadIdx.x % C, r = threadIdx.x / C;     // r: b (b layout) or the first c (c layout)
    const bool ok = l < cw;
    float2 v[16];
    if (MODE != 2) {
        // forward: b layout, DFT-16 over a, twiddle W_L^{bc}, exchange
        if (PR) {
#pragma unroll
            for (int a = 0; a < 16; ++a) v[a] = src_row(from, sb, R2 * a + r, L, l, ok);
        } else {
            cols_load_b<R2>(v, base, rs, l, r, ok);
        }
        __syncthreads();                                      // twiddle table
        dft_reg<16, false>(v);
#pragma unroll
        for (int c = 1; c < 16; ++c) v[c] = cmul(v[c], tw[r * c]);
#pragma unroll
        for (int c = 0; c < 16; ++c) ex[c * CSC + r * C + l] = v[c];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < P2; ++u) {
            const int c = r + (256 / C) * u;
            float2 w[R2];
#pragma unroll
            for (int b = 0; b < R2; ++b) w[b] = ex[c * CSC + b * C + l];
            dft_reg<R2, false>(w);                            // w[d] = X[c + 16 d]
#pragma unroll
            for (int d = 0; d < R2; ++d) v[u * R2 + d] = w[d];
        }
        if (MODE == 1) {
#pragma unroll
            for (int u = 0; u < P2; ++u) {
                const int c = r + (256 / C) * u;
#pragma unroll
                for (int d = 0; d < R2; ++d)
                    if (ok) base[(size_t)(c + 16 * d) * rs + l] = v[u * R2 + d];
            }
            return;
        }
        // symbol of the x1 pass: k1 = c + 16 d, k2 = plane, k3 = c0 + l
        const float k2 = (float)(pl < (n2 >> 1) ? pl : pl - n2);
        const float k3 = (float)(c0 + l);
        const bool edge = c0 + l == 0 || c0 + l == nh - 1;
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < P2; ++u) {
            const int c = r + (256 / C) * u;
#pragma unroll
            for (int d = 0; d < R2; ++d) {
                const int q = c + 16 * d;
                const float k1 = (float)(q < (n1 >> 1) ? q : q - n1);
                const float ksq = k1 * k1 + k2 * k2 + k3 * k3;
                float sym;
                if (kind == 0) sym = beta * ksq;
                else if (kind == 1) sym = 1.0f / (beta * fmaxf(ksq, 1.0f));
                else sym = 1.0f;
                sym *= scale;
                if (DOT) acc += dot_term(v[u * R2 + d], sym, edge);   // zero past the last column
                v[u * R2 + d].x *= sym;
                v[u * R2 + d].y *= sym;
            }
        }
        if (DOT) dot_store(acc, dot);
        __syncthreads();                                      // exchange buffer free again
    } else {
        // inverse only: c layout loads X[c + 16 d]
#pragma unroll
        for (int u = 0; u < P2; ++u) {
            const int c = r + (256 / C) * u;
#pragma unroll
            for (int d = 0; d < R2; ++d)
                v[u * R2 + d] = PR ? src_row(from, sb, c + 16 * d, L, l, ok)
                                   : ok ? base[(size_t)(c + 16 * d) * rs + l] : make_float2(0.f, 0.f);
        }
        __syncthreads();                                      // twiddle table
    }
    // inverse: c layout, DFT-R2 over d, twiddle W_L^{-bc}, exchange, DFT-16 over c
#pragma unroll
    for (int u = 0; u < P2; ++u) {
        const int c = r + (256 / C) * u;
        float2 w[R2];
#pragma unroll
        for (int d = 0; d < R2; ++d) w[d] = v[u * R2 + d];
        dft_reg<R2, true>(w);                                 // w[b] = sum_d X[c + 16 d] W_R2^{-bd}
#pragma unroll
        for (int b = 0; b < R2; ++b) ex[c * CSC + b * C + l] = b ? cmul(w[b], cconj(tw[b * c])) : w[b];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = ex[c * CSC + r * C + l];
    dft_reg<16, true>(v);                                     // v[a] = x[r + R2 a]
    if (ok) {
#pragma unroll
        for (int a = 0; a < 16; ++a) base[(size_t)(R2 * a + r) * rs + l] = v[a];
    }
}

// --- register-resident column passes for lines of L = 256 E points (E = 2
// or 4: 512 or 1024 points) in tiles of C = 32 / E columns, 512 threads.
// The split n = R2 a + b, k = c + 16 d (R2 = 16 E) of k_fft_cols leaves a
// length-R2 DFT over b for every (column, c); it is split again as
// b = E beta + eps, d = d' + 16 m:
//   X[c + 16 d' + 256 m] = sum_eps W_E^{eps m} W_R2^{eps d'} Z_eps[d'],
//   Z_eps[d'] = sum_beta y_c[E beta + eps] W_16^{beta d'},
// so a thread holds 16 values in both layouts: the E lanes eps of a
// (column, c) pair are neighbours, each runs one length-16 DFT, and the
// length-E DFT over eps runs across them (radix-2 lane exchanges; with E = 4
// lane eps ends with m = the bit reverse of eps).  The inverse applies the
// same steps backwards with conjugate twiddles.  Tiles of 16 (512 points) or
// 8 columns (1024 points) keep row pieces of 128 or 64 bytes and 66 KB of
// exchange buffer, so that two workgroups fit a CU.
constexpr int NTX = 512;

// length-E DFT over the lanes eps S, in place on 16 values (eps = (lane / S)
// mod E: the partners of a lane are lane ^ S and lane ^ 2S)
template <int E, bool INV, int S = 1> __device__ __forceinline__ void cross_dft(float2 (&v)[16], int eps)
{
    auto bfly = [&](int bit) {        // lane bit 0: own + partner; bit 1: partner - own
        const bool hi = (eps & bit) != 0;
        const int mask = bit * S;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float px = __shfl_xor(v[i].x, mask), py = __shfl_xor(v[i].y, mask);
            v[i] = hi ? make_float2(px - v[i].x, py - v[i].y) : make_float2(v[i].x + px, v[i].y + py);
        }
    };
    if (E == 2) {
        bfly(1);
        return;
    }
    bfly(INV ? 1 : 2);
    if (eps == 3) {                   // W_4^{+-1}
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = INV ? make_float2(-v[i].y, v[i].x) : make_float2(v[i].y, -v[i].x);
    }
    bfly(INV ? 2 : 1);
}

template <int E, int MODE, bool PR, bool DOT>
__global__ __launch_bounds__(NTX, 4) void k_fft_colsx(float2 *spec, const float2 *__restrict__ twL,
                                                      int nh, size_t plane_stride, size_t rs, size_t spec_cs, int kind,
                                                      float beta, float scale, int n1, int n2, ColSrc from,
                                                      double *__restrict__ dot)
{
    constexpr int R2 = 16 * E, L = 16 * R2, C = NTX / R2, LOGC = C == 16 ? 4 : 3, LOGE = E == 2 ? 1 : 2;
    constexpr int CS = R2 * C + 16;   // exchange pitch per c
    __shared__ float2 tw[L];
    __shared__ float2 ex[16 * CS];
    const int comp = blockIdx.z, pl = PR ? kept_plane(from, blockIdx.y) : blockIdx.y, c0 = blockIdx.x * C;
    const int cw = min(C, nh - c0);
    float2 *base = spec + comp * spec_cs + pl * plane_stride + c0;
    const float2 *sb = PR ? src_plane(from, comp, blockIdx.y, c0) : base;
    for (int t = threadIdx.x; t < L; t += NTX) tw[t] = twL[t];
    // b layout: thread (column lb, b); c layout: thread (eps, column lc, c), eps fastest
    const int lb = threadIdx.x & (C - 1), b = threadIdx.x >> LOGC;
    const int eps = threadIdx.x & (E - 1), lc = (threadIdx.x >> LOGE) & (C - 1), c = threadIdx.x >> (LOGE + LOGC);
    const int m = E == 4 ? ((eps & 1) << 1 | eps >> 1) : eps;
    const bool okb = lb < cw, okc = lc < cw;
    float2 v[16];
    if (MODE != 2) {
        if (PR) {
#pragma unroll
            for (int a = 0; a < 16; ++a) v[a] = src_row(from, sb, R2 * a + b, L, lb, okb);
        } else {
            cols_load_b<R2>(v, base, rs, lb, b, okb);        // v[a] = x[R2 a + b]
        }
        __syncthreads();                                      // twiddle table
        dft_reg<16, false>(v);
#pragma unroll
        for (int k = 1; k < 16; ++k) v[k] = cmul(v[k], tw[b * k]);
#pragma unroll
        for (int k = 0; k < 16; ++k) ex[k * CS + b * C + lb] = v[k];
        __syncthreads();
#pragma unroll
        for (int bt = 0; bt < 16; ++bt) v[bt] = ex[c * CS + (E * bt + eps) * C + lc];
        dft_reg<16, false>(v);                                // Z_eps[d']
#pragma unroll
        for (int k = 1; k < 16; ++k)
            if (eps) v[k] = cmul(v[k], tw[16 * eps * k]);
        cross_dft<E, false>(v, eps);                          // v[d'] = X[c + 16 d' + 256 m]
        if (MODE == 1) {
            if (okc) {
#pragma unroll
                for (int k = 0; k < 16; ++k) base[(size_t)(c + 16 * k + 256 * m) * rs + lc] = v[k];
            }
            return;
        }
        // symbol of the x1 pass: k1 = c + 16 d' + 256 m, k2 = plane, k3 = c0 + lc
        const float k2 = (float)(pl < (n2 >> 1) ? pl : pl - n2);
        const float k3 = (float)(c0 + lc);
        const bool edge = c0 + lc == 0 || c0 + lc == nh - 1;
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int q = c + 16 * k + 256 * m;
            const float k1 = (float)(q < (n1 >> 1) ? q : q - n1);
            const float ksq = k1 * k1 + k2 * k2 + k3 * k3;
            float sym;
            if (kind == 0) sym = beta * ksq;
            else if (kind == 1) sym = 1.0f / (beta * fmaxf(ksq, 1.0f));
            else sym = 1.0f;
            sym *= scale;
            if (DOT) acc += dot_term(v[k], sym, edge);        // zero past the last column
            v[k].x *= sym;
            v[k].y *= sym;
        }
        if (DOT) dot_store(acc, dot);
        __syncthreads();                                      // exchange buffer free again
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k)
            v[k] = PR ? src_row(from, sb, c + 16 * k + 256 * m, L, lc, okc)
                      : okc ? base[(size_t)(c + 16 * k + 256 * m) * rs + lc] : make_float2(0.f, 0.f);
        __syncthreads();                                      // twiddle table
    }
    // inverse: lanes, twiddle W_R2^{-eps d'}, DFT-16 over d', exchange,
    // twiddle W_L^{-b c}, DFT-16 over c
    cross_dft<E, true>(v, eps);
#pragma unroll
    for (int k = 1; k < 16; ++k)
        if (eps) v[k] = cmul(v[k], cconj(tw[16 * eps * k]));
    dft_reg<16, true>(v);                                     // v[beta] = y_c[E beta + eps]
#pragma unroll
    for (int bt = 0; bt < 16; ++bt) ex[c * CS + (E * bt + eps) * C + lc] = v[bt];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = ex[k * CS + b * C + lb];
#pragma unroll
    for (int k = 1; k < 16; ++k) v[k] = cmul(v[k], cconj(tw[b * k]));
    dft_reg<16, true>(v);                                     // v[a] = x[R2 a + b]
    if (okb) {
#pragma unroll
        for (int a = 0; a < 16; ++a) base[(size_t)(R2 * a + b) * rs + lb] = v[a];
    }
}

// --- register-resident x3 passes for rows of M = 16 R2 complex values (M =
// 64 ... 512, i.e. n3 = 128 ... 1024), NR = 256 / R2 rows per tile.  With
// input index n = c + 16 d and output index k = b + R2 a (M = 16 R2),
//   X[b + R2 a] = sum_c W_16^{ac} W_M^{bc} sum_d x[c + 16 d] W_R2^{bd}
// (conjugate twiddles for the inverse): the length-R2 DFTs over d run on the
// "c" layout (thread = row, c; 16 / R2 pairs per thread; R2 = 32 below),
// the length-16 DFTs over c on the "b" layout (thread = row, b), joined by one LDS exchange
// [row][c][b] (row pitch 17 R2 + 16 complex).  Loads on the c layout read
// 16 consecutive complex values per row per instruction.
// Rows of M = 512 complex values (n3 = 1024, R2 = 32, NR = 8 rows per tile)
// split the length-32 DFTs over d once more, d = 2 delta + eps, b = b' + 16 m:
//   Y_c[b' + 16 m] = sum_eps (-1)^{eps m} W_32^{eps b'}
//                    sum_delta x[c + 16 (2 delta + eps)] W_16^{delta b'},
// so the c layout holds (row, c, eps) with eps = bit 4 of the lane, every
// thread runs one length-16 DFT, and the length-2 DFT over eps is a lane
// exchange (lane ^ 16).
template <int R2> constexpr int rows_pitch() { return 17 * R2 + 16; }

// Lane i of each 16-lane row receives x of lane 16 - i of the same row
// (DPP row mirror, i -> 15 - i, then a shift by one lane); lane 0 receives 0.
__device__ __forceinline__ float row_reflect16(float x)
{
    const int m = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xf, 0xf, false);   // row_mirror
    return __int_as_float(__builtin_amdgcn_update_dpp(0, m, 0x111, 0xf, 0xf, false));         // row_shr:1
}

template <int R2, bool INV>
__device__ __forceinline__ void rows_cb(float2 (&v)[16], float2 *ex, const float2 *tw)
{
    constexpr int PP = 16 / R2, RS = rows_pitch<R2>();
    const int c = threadIdx.x & 15, r0 = threadIdx.x >> 4;
#pragma unroll
    for (int u = 0; u < PP; ++u) {
        const int row = r0 + 16 * u;
        float2 w[R2];
#pragma unroll
        for (int d = 0; d < R2; ++d) w[d] = v[u * R2 + d];
        dft_reg<R2, INV>(w);
#pragma unroll
        for (int b = 0; b < R2; ++b) {
            float2 t = w[b];
            if (b) t = cmul(t, INV ? cconj(tw[b * c]) : tw[b * c]);
            ex[row * RS + c * (R2 + 1) + b] = t;
        }
    }
    __syncthreads();
    const int b = threadIdx.x % R2, row = threadIdx.x / R2;
#pragma unroll
    for (int cc = 0; cc < 16; ++cc) v[cc] = ex[row * RS + cc * (R2 + 1) + b];
    dft_reg<16, INV>(v);                                      // v[a] = X[b + R2 a]
}

// rows_cb for R2 = 32: v[delta] = x[c + 16 (2 delta + eps)] on the c layout
// (c = lane bits 0-3, eps = bit 4, row = thread / 32) in, v[a] = X[b + 32 a]
// on the b layout out
template <bool INV> __device__ __forceinline__ void rows_cbx(float2 (&v)[16], float2 *ex, const float2 *tw)
{
    constexpr int R2 = 32, RS = rows_pitch<32>();
    const int c = threadIdx.x & 15, eps = (threadIdx.x >> 4) & 1, row = threadIdx.x >> 5;
    dft_reg<16, INV>(v);                                      // v[b'] = sum_delta ... W_16^{delta b'}
    if (eps) {
#pragma unroll
        for (int k = 1; k < 16; ++k) v[k] = cmul(v[k], INV ? cconj(tw[16 * k]) : tw[16 * k]);   // W_32^{b'}
    }
    cross_dft<2, INV, 16>(v, eps);                            // v[b'] = Y_c[b' + 16 eps]
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int b = k + 16 * eps;
        float2 t = v[k];
        if (b * c) t = cmul(t, INV ? cconj(tw[b * c]) : tw[b * c]);
        ex[row * RS + c * (R2 + 1) + b] = t;
    }
    __syncthreads();
    const int bb = threadIdx.x % R2, rb = threadIdx.x / R2;
#pragma unroll
    for (int cc = 0; cc < 16; ++cc) v[cc] = ex[rb * RS + cc * (R2 + 1) + bb];
    dft_reg<16, INV>(v);                                      // v[a] = X[b + R2 a]
}

// x3 forward: real rows -> half spectrum.  UPD: of r - alpha H in place of in,
// also stored to out, which may be r (a thread stores the values that it has
// read).  Bound by its traffic: the residual formed here instead of in a pass of
// its own takes 174 us at 256^3, 12 fields of 4 n bytes, against 120 + 80 us and 15.
template <int R2, bool UPD>
__global__ __launch_bounds__(TPB) void k_fft_rows_r2c(const float *__restrict__ in, float2 *__restrict__ spec,
                                                      const float2 *__restrict__ twM, const float2 *__restrict__ tw3,
                                                      size_t in_cs, size_t spec_cs, SpecUpdate upd)
{
    constexpr int M = 16 * R2, NR = 256 / R2, NP = M + 16;   // NP: spectrum row pitch
    __shared__ float2 twm[M], tws[M + 1];
    __shared__ float2 ex[NR * rows_pitch<R2>()];
    const int comp = blockIdx.y;
    const size_t row0 = (size_t)blockIdx.x * NR;
    const float2 *src = (const float2 *)((UPD ? upd.r : in) + comp * in_cs) + row0 * M;
    float2 *dst = spec + comp * spec_cs + row0 * NP;
    for (int t = threadIdx.x; t < M; t += TPB) twm[t] = twM[t];
    for (int t = threadIdx.x; t <= M; t += TPB) tws[t] = tw3[t];
    const int c = threadIdx.x & 15, r0 = threadIdx.x >> 4;
    // offset of value j of the thread in its tile of rows
    auto off = [&](int j) {
        return R2 == 32 ? (size_t)(r0 >> 1) * M + c + 16 * (r0 & 1) + 32 * j
                        : (size_t)(r0 + 16 * (j / R2)) * M + c + 16 * (j % R2);
    };
    float2 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = src[off(j)];
    if constexpr (UPD) {
        const float alpha = (float)*upd.alpha;
        const float2 *h = (const float2 *)(upd.H + comp * in_cs) + row0 * M;
        float2 *o = (float2 *)(upd.out + comp * in_cs) + row0 * M;
        float2 w[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = h[off(j)];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            v[j] = make_float2(fmaf(-alpha, w[j].x, v[j].x), fmaf(-alpha, w[j].y, v[j].y));
            o[off(j)] = v[j];
        }
    }
    __syncthreads();                                          // twiddle tables
    if constexpr (R2 == 32) {
        rows_cbx<false>(v, ex, twm);
    } else {
        rows_cb<R2, false>(v, ex, twm);
    }
    // X[k] = E + W_n3^k O with E = (Z[k] + conj Z[M-k]) / 2, O = -i (Z[k] -
    // conj Z[M-k]) / 2; Z[M-k] of k = b + R2 a is v[15 - a] of the lane with
    // b' = R2 - b (b > 0) or this lane's v[(16 - a) mod 16] (b = 0)
    const int b = threadIdx.x % R2, row = threadIdx.x / R2;
    const int lane = threadIdx.x & 63, partner = lane - b + ((R2 - b) & (R2 - 1));
    float2 *drow = dst + (size_t)row * NP;
#pragma unroll
    for (int a = 0; a < 16; ++a) {
        float2 zc;
        zc.x = __shfl(v[15 - a].x, partner, 64);
        zc.y = __shfl(v[15 - a].y, partner, 64);
        if (b == 0) zc = v[(16 - a) & 15];
        zc = cconj(zc);
        const float2 zk = v[a];
        const int k = b + R2 * a;
        const float2 E = make_float2(0.5f * (zk.x + zc.x), 0.5f * (zk.y + zc.y));
        const float2 O = make_float2(0.5f * (zk.y - zc.y), -0.5f * (zk.x - zc.x));
        drow[k] = cadd(E, cmul(tws[k], O));
    }
    if (b == 0) {
        // k = M: Z[M mod M] = Z[0]
        const float2 zk = v[0], zc = cconj(v[0]);
        const float2 E = make_float2(0.5f * (zk.x + zc.x), 0.5f * (zk.y + zc.y));
        const float2 O = make_float2(0.5f * (zk.y - zc.y), -0.5f * (zk.x - zc.x));
        drow[M] = cadd(E, cmul(tws[M], O));
    }
}

// x3 inverse: half spectrum -> real rows (unnormalised), optional add
template <int R2, bool PR>
__global__ __launch_bounds__(TPB) void k_fft_rows_c2r(const float2 *__restrict__ spec, float *__restrict__ out,
                                                      const float *__restrict__ add, const float2 *__restrict__ twM,
                                                      const float2 *__restrict__ tw3, size_t out_cs, size_t spec_cs,
                                                      int kmax)
{
    constexpr int M = 16 * R2, NR = 256 / R2, PP = 16 / R2, NP = M + 16;   // NP: spectrum row pitch
    __shared__ float2 twm[M], tws[M + 1];
    __shared__ float2 ex[NR * rows_pitch<R2>()];
    const int comp = blockIdx.y;
    const size_t row0 = (size_t)blockIdx.x * NR;
    // value k of a row (PR: zero from kmax on, not read)
    auto val = [&](const float2 *row, int k) { return !PR || k < kmax ? row[k] : make_float2(0.f, 0.f); };
    const float2 *src = spec + comp * spec_cs + row0 * NP;
    float2 *dst = (float2 *)(out + comp * out_cs) + row0 * M;
    const float2 *ad = add ? (const float2 *)(add + comp * out_cs) + row0 * M : nullptr;
    for (int t = threadIdx.x; t < M; t += TPB) twm[t] = twM[t];
    for (int t = threadIdx.x; t <= M; t += TPB) tws[t] = tw3[t];
    const int c = threadIdx.x & 15, r0 = threadIdx.x >> 4;
    float2 v[16];
    if constexpr (R2 == 32) {
        // X[k] and X[M - k] for k = c + 16 (2 delta + eps), both read from
        // the row (k = 0 pairs with the Nyquist value X[M])
        const int eps = r0 & 1, rw = r0 >> 1;
        const float2 *srow = src + (size_t)rw * NP;
        float2 xa[16], xb[16];
#pragma unroll
        for (int dl = 0; dl < 16; ++dl) {
            const int k = c + 16 * eps + 32 * dl;
            xa[dl] = val(srow, k);
            xb[dl] = val(srow, M - k);
        }
        __syncthreads();                                      // twiddle tables
#pragma unroll
        for (int dl = 0; dl < 16; ++dl) {
            const int k = c + 16 * eps + 32 * dl;
            const float2 a = xa[dl], bb = cconj(xb[dl]);
            const float2 sum = cadd(a, bb), dif = csub(a, bb);
            const float2 wd = cmul(cconj(tws[k]), dif);
            v[dl] = make_float2(sum.x - wd.y, sum.y + wd.x);
        }
        rows_cbx<true>(v, ex, twm);
    } else {
        float2 xa[16], xb[16], nyq[PP];
#pragma unroll
        for (int u = 0; u < PP; ++u) {
            const float2 *srow = src + (size_t)(r0 + 16 * u) * NP;
#pragma unroll
            for (int d = 0; d < R2; ++d) xa[u * R2 + d] = val(srow, c + 16 * d);
            nyq[u] = c == 0 ? val(srow, M) : make_float2(0.f, 0.f);
        }
        // X[M - k] for k = c + 16 d: for c > 0 it is X[(16 - c) + 16 (R2 - 1 - d)],
        // held by lane 16 - c of the same 16-lane row (a row reflection by DPP);
        // for c = 0 it is this lane's X[16 (R2 - d)], or the Nyquist value at d = 0
#pragma unroll
        for (int u = 0; u < PP; ++u)
#pragma unroll
            for (int d = 0; d < R2; ++d) {
                const float2 o = xa[u * R2 + R2 - 1 - d];
                const float2 m = make_float2(row_reflect16(o.x), row_reflect16(o.y));
                xb[u * R2 + d] = c ? m : (d ? xa[u * R2 + R2 - d] : nyq[u]);
            }
        __syncthreads();                                      // twiddle tables
        // Z[k] = (X[k] + conj X[M-k]) + i e^{+2 pi i k / n3} (X[k] - conj X[M-k])
#pragma unroll
        for (int u = 0; u < PP; ++u)
#pragma unroll
            for (int d = 0; d < R2; ++d) {
                const int k = c + 16 * d;
                const float2 a = xa[u * R2 + d], bb = cconj(xb[u * R2 + d]);
                const float2 sum = cadd(a, bb), dif = csub(a, bb);
                const float2 wd = cmul(cconj(tws[k]), dif);
                v[u * R2 + d] = make_float2(sum.x - wd.y, sum.y + wd.x);
            }
        rows_cb<R2, true>(v, ex, twm);
    }
    const int b = threadIdx.x % R2, row = threadIdx.x / R2;
#pragma unroll
    for (int a = 0; a < 16; ++a) {
        const size_t o = (size_t)row * M + b + R2 * a;
        float2 val = v[a];
        if (ad) {
            const float2 t = ad[o];
            val.x += t.x;
            val.y += t.y;
        }
        dst[o] = val;
    }
}

// Per-mode 3x3 operators of the near-incompressible regularisation on the
// half spectrum of a vector field (three components spec_cs apart), scaled
// by 1/N.  With a = beta_v |k|^2, c = beta_w (1 + |k|^2) and kappa the
// derivative wavenumber (k_d, 0 at the Nyquist index):
//   kind 0: L = a I + c kappa kappa^T (Hessian of the regularisation)
//   kind 1: L^-1 = (I - c/(a + c |kappa|^2) kappa kappa^T) / a, 1/beta_v at k = 0
//   kind 3: K = beta_v A L^-1 = I - c/(a + c |kappa|^2) kappa kappa^T, I at k = 0
// (Sherman-Morrison on the rank-one term).
__global__ __launch_bounds__(TPB) void k_spec_mult3(float2 *__restrict__ spec, int n1, int n2, int nh, int np,
                                                    int kind, float beta_v, float beta_w, float scale, size_t spec_cs)
{
    const size_t m = (size_t)blockIdx.x * TPB + threadIdx.x;   // mode index over the n1 n2 nh modes
    if (m >= (size_t)n1 * n2 * nh) return;
    const int q3 = (int)(m % nh);
    const int q2 = (int)((m / nh) % n2);
    const int q1 = (int)(m / ((size_t)nh * n2));
    const size_t e = ((size_t)q1 * n2 + q2) * np + q3;
    const float k1 = (float)(q1 < (n1 >> 1) ? q1 : q1 - n1);
    const float k2 = (float)(q2 < (n2 >> 1) ? q2 : q2 - n2);
    const float k3 = (float)q3;
    const float c1 = q1 == (n1 >> 1) ? 0.f : k1, c2 = q2 == (n2 >> 1) ? 0.f : k2, c3 = q3 == nh - 1 ? 0.f : k3;
    const float ksq = k1 * k1 + k2 * k2 + k3 * k3;
    const float a = beta_v * ksq, c = beta_w * (1.0f + ksq);
    float2 x0 = spec[e], x1 = spec[spec_cs + e], x2 = spec[2 * spec_cs + e];
    const float pr = c1 * x0.x + c2 * x1.x + c3 * x2.x;   // kappa . x
    const float pi = c1 * x0.y + c2 * x1.y + c3 * x2.y;
    float d, f;   // y = d x + f kappa (kappa . x)
    if (kind == 0) {
        d = a;
        f = c;
    } else if (ksq == 0.f) {
        d = kind == 1 ? 1.0f / beta_v : 1.0f;
        f = 0.f;
    } else {
        const float r = c / (a + c * (c1 * c1 + c2 * c2 + c3 * c3));
        d = kind == 1 ? 1.0f / a : 1.0f;
        f = -r * d;
    }
    d *= scale;
    f *= scale;
    x0 = make_float2(fmaf(f * c1, pr, d * x0.x), fmaf(f * c1, pi, d * x0.y));
    x1 = make_float2(fmaf(f * c2, pr, d * x1.x), fmaf(f * c2, pi, d * x1.y));
    x2 = make_float2(fmaf(f * c3, pr, d * x2.x), fmaf(f * c3, pi, d * x2.y));
    spec[e] = x0;
    spec[spec_cs + e] = x1;
    spec[2 * spec_cs + e] = x2;
}

int ilog2(int n)
{
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

} // namespace

size_t fft_spec_bytes(int n1, int n2, int n3, int ncomp)
{
    return (size_t)ncomp * n1 * n2 * fft_row_pitch(n3) * sizeof(float2);
}

void fft_make_twiddles(float2 *host, int n, int count)
{
    const double two_pi = 6.283185307179586476925286766559;
    for (int t = 0; t < count; ++t) {
        const double a = -two_pi * t / n;
        host[t] = make_float2((float)std::cos(a), (float)std::sin(a));
    }
}

namespace {
struct PassGeom;
void coupled3(const FFTPlan &P, int kind, float beta_v, float beta_w, const float *in, float *out, hipStream_t s);
} // namespace

namespace {

bool cols_ok(int L) { return L == 64 || L == 128 || L == 256 || L == 512 || L == 1024; }

// columns per tile of the register-resident column passes
int cols_width(int L) { return L <= 256 ? 4096 / L : 8192 / L; }

// from: pruned source (NULL: the spectrum itself, in full)
template <int MODE>
void launch_cols(int L, dim3 grid, float2 *spec, const float2 *tw, int nh, size_t plane_stride, size_t rs,
                 size_t spec_cs, int kind, float beta, float scale, int n1, int n2, const ColSrc *from, double *dot,
                 hipStream_t s)
{
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, spec, tw, nh, plane_stride, rs, spec_cs, kind, beta,
                           scale, n1, n2, from ? *from : ColSrc{}, dot);
    };
    auto size = [&](auto pruned, auto dotted) {
        constexpr bool PR = decltype(pruned)::value, DOT = decltype(dotted)::value;
        if (L == 1024) go(k_fft_colsx<4, MODE, PR, DOT>, NTX);
        else if (L == 512) go(k_fft_colsx<2, MODE, PR, DOT>, NTX);
        else if (L == 256) go(k_fft_cols<16, MODE, PR, DOT>, TPB);
        else if (L == 128) go(k_fft_cols<8, MODE, PR, DOT>, TPB);
        else go(k_fft_cols<4, MODE, PR, DOT>, TPB);
    };
    if constexpr (MODE == 0) {
        if (dot) return size(std::false_type{}, std::true_type{});
    } else {
        if (from) return size(std::true_type{}, std::false_type{});
    }
    size(std::false_type{}, std::false_type{});
}

bool rows_ok(int n3) { return n3 == 128 || n3 == 256 || n3 == 512 || n3 == 1024; }

// register-resident row kernel for rows of n3 reals (R2 = n3 / 32, NR = 256 / R2 rows per tile)
template <int R2>
void launch_rows_r2c(const FFTPlan &P, const float *in, int nc, size_t N, size_t spec_cs, const SpecUpdate *upd,
                     hipStream_t s)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(P.n1 * P.n2 / (256 / R2), nc), dim3(TPB), 0, s, in, P.spec, P.twM, P.twS, N,
                           spec_cs, upd ? *upd : SpecUpdate{});
    };
    if (upd) go(k_fft_rows_r2c<R2, true>);
    else go(k_fft_rows_r2c<R2, false>);
}

bool rows_fit(const FFTPlan &P) { return rows_ok(P.n3) && P.n1 * P.n2 % (256 / (P.n3 / 32)) == 0; }

template <int R2>
void launch_rows_c2r(const FFTPlan &P, float *out, const float *add, int nc, size_t N, size_t spec_cs, int kmax,
                     hipStream_t s)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(P.n1 * P.n2 / (256 / R2), nc), dim3(TPB), 0, s, P.spec, out, add, P.twM, P.twS,
                           N, spec_cs, kmax);
    };
    if (kmax < P.nh) go(k_fft_rows_c2r<R2, true>);
    else go(k_fft_rows_c2r<R2, false>);
}

// x3 forward pass (real rows -> half spectrum), nc components
void pass_r2c(const FFTPlan &P, const float *in, int nc, int logM, int lognl3, size_t lds3, size_t spec_cs,
              const SpecUpdate *upd, hipStream_t s)
{
    const size_t N = (size_t)P.n1 * P.n2 * P.n3;
    const int nrows = P.n1 * P.n2;
    if (rows_fit(P)) {
        if (P.n3 == 1024) launch_rows_r2c<32>(P, in, nc, N, spec_cs, upd, s);
        else if (P.n3 == 512) launch_rows_r2c<16>(P, in, nc, N, spec_cs, upd, s);
        else if (P.n3 == 256) launch_rows_r2c<8>(P, in, nc, N, spec_cs, upd, s);
        else launch_rows_r2c<4>(P, in, nc, N, spec_cs, upd, s);
        return;
    }
    hipLaunchKernelGGL(k_fft_x3_r2c, dim3(nrows >> lognl3, nc), dim3(TPB), lds3, s, in, P.spec, P.twM, P.twS, logM,
                       lognl3, nrows, N, spec_cs, P.np);
}

// x3 inverse pass (half spectrum -> real rows, optional add), nc components;
// values k >= kmax are taken as zero
void pass_c2r(const FFTPlan &P, float *out, const float *add, int nc, int logM, int lognl3, size_t lds3,
              size_t spec_cs, int kmax, hipStream_t s)
{
    const size_t N = (size_t)P.n1 * P.n2 * P.n3;
    const int nrows = P.n1 * P.n2;
    if (rows_fit(P)) {
        if (P.n3 == 1024) launch_rows_c2r<32>(P, out, add, nc, N, spec_cs, kmax, s);
        else if (P.n3 == 512) launch_rows_c2r<16>(P, out, add, nc, N, spec_cs, kmax, s);
        else if (P.n3 == 256) launch_rows_c2r<8>(P, out, add, nc, N, spec_cs, kmax, s);
        else launch_rows_c2r<4>(P, out, add, nc, N, spec_cs, kmax, s);
        return;
    }
    hipLaunchKernelGGL(k_fft_x3_c2r, dim3(nrows >> lognl3, nc), dim3(TPB), lds3, s, P.spec, out, add, P.twM, P.twS,
                       logM, lognl3, nrows, N, spec_cs, P.np, kmax);
}

// x3 and x2 passes of small planes (of nc components) in one kernel, one workgroup a
// plane.  With 3072 of them, 1024 planes of three components, the workgroups come in
// rounds and the separate passes' full tiles take less: 1024 x 16 x 32 77 -> 60 us,
// 1024 x 64 x 64 172 -> 148 us.  At 1536 the two are within 10 % of each other either
// way, below one kernel takes 0.5-0.9 of the time.
bool planes_ok(const FFTPlan &P, int nc) { return P.n2 <= 64 && P.n3 <= 64 && P.n1 * nc <= 2048; }

template <bool INV>
void launch_planes(const FFTPlan &P, const float *in, float *out, const float *add, int nc, size_t spec_cs, int kmax,
                   int m2, hipStream_t s)
{
    const int M = P.n3 / 2, NL = 2 * M;   // NL >= nh = M + 1; n2 NL <= 64 x 64 values
    const size_t lds = (size_t)(2 * M + 1 + P.n2 + std::max(M * (P.n2 + 1), P.n2 * (NL + 1))) * sizeof(float2);
    hipLaunchKernelGGL((k_fft_plane<INV>), dim3(P.n1, nc), dim3(NTP), lds, s, in, out, add, P.spec, P.twM, P.twS, P.tw2,
                       ilog2(M), ilog2(P.n2), ilog2(NL), (size_t)P.n1 * P.n2 * P.n3, spec_cs, P.np,
                       kmax, m2);
}

// Stockham column passes (lines of 16 and 32 points; longer ones take the
// register-resident passes): a 256-thread tile of at most 2048 values holds 32
// columns.
struct ColGeom {
    int logC;
    size_t lds;   // twiddle table + tile at pitch C + 1
};

ColGeom col_geom(int L)
{
    ColGeom c;
    const int logT = ilog2(TPB * EPT);
    c.logC = logT - ilog2(L) > 5 ? 5 : logT - ilog2(L);
    c.lds = (size_t)(L + (size_t)L * ((1 << c.logC) + 1)) * sizeof(float2);
    return c;
}


// x2 pass over every x1 plane (forward or inverse), nc components: the columns
// k3 < kmax; from: pruned rows of an inverse pass
void pass_x2(const FFTPlan &P, bool inv, int nc, size_t spec_cs, int kmax, const ColSrc *from, hipStream_t s)
{
    const size_t ps = (size_t)P.n2 * P.np;
    if (cols_ok(P.n2)) {
        const int C = cols_width(P.n2);
        const dim3 grid((kmax + C - 1) / C, P.n1, nc);
        if (inv) launch_cols<2>(P.n2, grid, P.spec, P.tw2, kmax, ps, P.np, spec_cs, 2, 0.f, 1.f, P.n1, P.n2, from,
                                nullptr, s);
        else launch_cols<1>(P.n2, grid, P.spec, P.tw2, kmax, ps, P.np, spec_cs, 2, 0.f, 1.f, P.n1, P.n2, nullptr,
                            nullptr, s);
        return;
    }
    const ColGeom cg = col_geom(P.n2);
    const int C2 = 1 << cg.logC;
    const dim3 grid((kmax + C2 - 1) / C2, P.n1, nc);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(TPB), cg.lds, s, P.spec, P.tw2, ilog2(P.n2), P.n2, kmax, P.np, cg.logC,
                           spec_cs, from ? *from : ColSrc{});
    };
    if (!inv) go(k_fft_x2<false, TPB, false>);
    else if (from) go(k_fft_x2<true, TPB, true>);
    else go(k_fft_x2<true, TPB, false>);
}

// x1 pass over every x2 plane: mode 0 forward, symbol, inverse; 1 forward; 2
// inverse.  kmax, from: the columns k3 < kmax of the planes that from keeps
// (modes 1 and 2), read through it; dot (mode 0, may be NULL): partials of <in, out>.
void pass_x1(const FFTPlan &P, int mode, int kind, float beta, float scale, int nc, size_t spec_cs, int kmax,
             const ColSrc *from, double *dot, hipStream_t s)
{
    const int planes = from ? P.n2 - from->skip : P.n2;
    if (cols_ok(P.n1)) {
        const int C = cols_width(P.n1);
        const dim3 grid((kmax + C - 1) / C, planes, nc);
        const size_t rs = (size_t)P.n2 * P.np;
        if (mode == 0) launch_cols<0>(P.n1, grid, P.spec, P.tw1, kmax, P.np, rs, spec_cs, kind, beta, scale, P.n1, P.n2, nullptr, dot, s);
        else if (mode == 1) launch_cols<1>(P.n1, grid, P.spec, P.tw1, kmax, P.np, rs, spec_cs, kind, beta, scale, P.n1, P.n2, from, nullptr, s);
        else launch_cols<2>(P.n1, grid, P.spec, P.tw1, kmax, P.np, rs, spec_cs, kind, beta, scale, P.n1, P.n2, from, nullptr, s);
        return;
    }
    const ColGeom cg = col_geom(P.n1);
    const int C1 = 1 << cg.logC;
    const dim3 grid((kmax + C1 - 1) / C1, planes, nc);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(TPB), cg.lds, s, P.spec, P.tw1, ilog2(P.n1), P.n1, P.n2, kmax, P.np,
                           cg.logC, kind, beta, scale, spec_cs, mode, from ? *from : ColSrc{}, dot);
    };
    if (from) go(k_fft_x1_mult<TPB, true>);
    else go(k_fft_x1_mult<TPB, false>);
}

} // namespace

int spectral_dot_blocks(const FFTPlan &P)
{
    const int C = cols_ok(P.n1) ? cols_width(P.n1) : 1 << col_geom(P.n1).logC;
    return (P.nh + C - 1) / C * P.n2 * P.ncomp_max;
}

// (the rows that can are longer than those of a plane)
bool spectral_takes_update(const FFTPlan &P) { return rows_fit(P); }

void spectral_apply(const FFTPlan &P, int kind, float beta, float beta_w, int ncomp, const float *in, float *out,
                    const float *add, hipStream_t s, double *dot, const SpecUpdate *upd)
{
    if (beta_w != 0.f && ncomp == 3 && kind != 2) {
        // the three components are coupled per mode: forward transforms,
        // one 3x3 pass over the half spectrum, inverse transforms
        coupled3(P, kind, beta, beta_w, in, out, s);
        if (add) launch_axpy(out, out, add, 1.0f, 3 * (size_t)P.n1 * P.n2 * P.n3, s);
        return;
    }
    if (kind == 3) kind = 2;   // K = I without the divergence term
    const int n1 = P.n1, n2 = P.n2, n3 = P.n3;
    const int M = n3 / 2, logM = ilog2(M);
    const size_t N = (size_t)n1 * n2 * n3;
    const size_t spec_cs = (size_t)n1 * n2 * P.np;
    const float scale = (float)(1.0 / (double)N);
    const int nrows = n1 * n2;
    const int logT = ilog2(TILE);
    // x3: nl rows of M per tile
    int lognl3 = logT - logM;            // M >= 8, so nl <= TILE / 8
    if ((1 << lognl3) > nrows) lognl3 = ilog2(nrows);
    const size_t lds3 = (size_t)(M + M + 1 + ((size_t)M + 1) * ((1 << lognl3) + 1)) * sizeof(float2);
    for (int c0 = 0; c0 < ncomp; c0 += P.ncomp_max) {
        const int nc = ncomp - c0 < P.ncomp_max ? ncomp - c0 : P.ncomp_max;
        const float *inc = in + c0 * N;
        float *outc = out + c0 * N;
        const float *addc = add ? add + c0 * N : nullptr;
        if (planes_ok(P, nc)) {
            launch_planes<false>(P, inc, nullptr, nullptr, nc, spec_cs, P.nh, P.n2, s);
            pass_x1(P, 0, kind, beta, scale, nc, spec_cs, P.nh, nullptr, dot, s);
            launch_planes<true>(P, nullptr, outc, addc, nc, spec_cs, P.nh, P.n2, s);
            continue;
        }
        const SpecUpdate u = upd ? SpecUpdate{upd->r + c0 * N, upd->H + c0 * N, upd->alpha, upd->out + c0 * N} : SpecUpdate{};
        pass_r2c(P, inc, nc, logM, lognl3, lds3, spec_cs, upd ? &u : nullptr, s);
        pass_x2(P, false, nc, spec_cs, P.nh, nullptr, s);
        pass_x1(P, 0, kind, beta, scale, nc, spec_cs, P.nh, nullptr, dot, s);
        pass_x2(P, true, nc, spec_cs, P.nh, nullptr, s);
        pass_c2r(P, outc, addc, nc, logM, lognl3, lds3, spec_cs, P.nh, s);
    }
}

namespace {

struct PassGeom {
    int logM, lognl3, nrows;
    size_t lds3, N, spec_cs;
};

PassGeom geom(const FFTPlan &P)
{
    PassGeom G;
    const int logT = ilog2(TILE);
    G.logM = ilog2(P.n3 / 2);
    G.nrows = P.n1 * P.n2;
    G.lognl3 = logT - G.logM;
    if ((1 << G.lognl3) > G.nrows) G.lognl3 = ilog2(G.nrows);
    const int M = P.n3 / 2;
    G.lds3 = (size_t)(M + M + 1 + ((size_t)M + 1) * ((1 << G.lognl3) + 1)) * sizeof(float2);
    G.N = (size_t)P.n1 * P.n2 * P.n3;
    G.spec_cs = (size_t)P.n1 * P.n2 * P.np;
    return G;
}

// Forward and inverse transforms of nc components, in full or for the modes
// |k_d| < m_d alone (full: m_d = n_d and kmax = nh): a forward pass visits the
// columns and planes that are kept, an inverse pass reads the others as zero.
struct Keep {
    int m1, m2, kmax;
};

ColSrc whole(const FFTPlan &P, const PassGeom &G, const float2 *src, size_t ps, size_t rs)
{
    return ColSrc{src, G.spec_cs, ps, rs, 0, 1 << 30, 1 << 30, 0, 0, 1.0f};
}

void forward3(const FFTPlan &P, const PassGeom &G, int nc, const float *in, const Keep &k, hipStream_t s)
{
    if (planes_ok(P, nc)) {
        launch_planes<false>(P, in, nullptr, nullptr, nc, G.spec_cs, P.nh, P.n2, s);
    } else {
        pass_r2c(P, in, nc, G.logM, G.lognl3, G.lds3, G.spec_cs, nullptr, s);
        pass_x2(P, false, nc, G.spec_cs, k.kmax, nullptr, s);
    }
    if (k.m2 >= P.n2) {
        pass_x1(P, 1, 2, 0.f, 1.f, nc, G.spec_cs, k.kmax, nullptr, nullptr, s);
    } else {
        ColSrc c = whole(P, G, P.spec, P.np, (size_t)P.n2 * P.np);
        c.mp = k.m2;
        c.skip = P.n2 - (2 * k.m2 - 1);
        pass_x1(P, 1, 2, 0.f, 1.f, nc, G.spec_cs, k.kmax, &c, nullptr, s);
    }
}

// from: source of the x1 pass (NULL: this plan's spectrum, in full)
void inverse3(const FFTPlan &P, const PassGeom &G, int nc, float *out, const Keep &k, const ColSrc *from, hipStream_t s)
{
    pass_x1(P, 2, 2, 0.f, 1.f, nc, G.spec_cs, k.kmax, from, nullptr, s);
    if (planes_ok(P, nc)) {
        launch_planes<true>(P, nullptr, out, nullptr, nc, G.spec_cs, k.kmax, k.m2, s);
        return;
    }
    if (k.m2 >= P.n2) {
        pass_x2(P, true, nc, G.spec_cs, k.kmax, nullptr, s);
    } else {
        ColSrc c = whole(P, G, P.spec, (size_t)P.n2 * P.np, P.np);
        c.La = P.n2;
        c.m = k.m2;
        pass_x2(P, true, nc, G.spec_cs, k.kmax, &c, s);
    }
    pass_c2r(P, out, nullptr, nc, G.logM, G.lognl3, G.lds3, G.spec_cs, k.kmax, s);
}

void coupled3(const FFTPlan &P, int kind, float beta_v, float beta_w, const float *in, float *out, hipStream_t s)
{
    // every plan of the library holds three components of spectrum
    const PassGeom G = geom(P);
    const Keep all{P.n1, P.n2, P.nh};
    forward3(P, G, 3, in, all, s);
    const size_t modes = (size_t)P.n1 * P.n2 * P.nh;
    hipLaunchKernelGGL(k_spec_mult3, dim3((unsigned)((modes + TPB - 1) / TPB)), dim3(TPB), 0, s, P.spec, P.n1, P.n2,
                       P.nh, P.np, kind, beta_v, beta_w, (float)(1.0 / (double)G.N), G.spec_cs);
    inverse3(P, G, 3, out, all, nullptr, s);
}

} // namespace

// The modes |k_d| < m_d = min(a_d, b_d) / 2 go straight from A's spectrum into
// B's x1 pass, scaled by 1 / N_A (a power of two); every pass visits only the
// columns and planes that hold them.  128^3 -> 256^3 (3 fields): with a copy
// into a zero-filled spectrum, full inverse passes and a scaling pass 434 us,
// 155 us so; the real rows written (201 MB) bound the last pass (60 us).
void spectral_resample(const FFTPlan &A, const FFTPlan &B, int ncomp, const float *in, float *out, hipStream_t s)
{
    const PassGeom GA = geom(A), GB = geom(B);
    for (int c0 = 0; c0 < ncomp; c0 += min(A.ncomp_max, B.ncomp_max)) {
        const int nc = min(ncomp - c0, min(A.ncomp_max, B.ncomp_max));
        const Keep k{min(A.n1, B.n1) / 2, min(A.n2, B.n2) / 2, min(A.n3, B.n3) / 2};
        forward3(A, GA, nc, in + c0 * GA.N, k, s);
        const ColSrc from{A.spec, GA.spec_cs, (size_t)A.np, (size_t)A.n2 * A.np, A.n1, k.m1, k.m2,
                          B.n2 - (2 * k.m2 - 1), A.n2 - B.n2, (float)(1.0 / (double)GA.N)};
        inverse3(B, GB, nc, out + c0 * GB.N, k, &from, s);
    }
}

} // namespace clh
