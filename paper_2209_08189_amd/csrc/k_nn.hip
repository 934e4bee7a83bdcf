// k_nn.hip -- kernels of the learned warm-start network: a 3D convolutional
// encoder-decoder that predicts an initial stationary velocity from the
// image pair (restricted to a coarser grid); the registration solve stays
// the judge of its output.
//
// Activations are BF16 tensors of C channels (a multiple of 16), by 16-channel
// chunks [C / 16][D][H][W][16] inside the network and channels last, [D][H][W][C],
// at the single-layer entry points (NNLayout); arithmetic is FP32.  3x3x3
// convolutions run on the matrix cores as an
// implicit GEMM with v_mfma_f32_16x16x32_bf16 (K = two taps x 16 input
// channels, below).  Weights are packed once per update into fragment order, so
// a fragment is one 16-byte load per lane.  The transpose needed by the
// backward data pass is the same convolution with flipped taps and swapped
// channel roles, i.e. the same kernel with a differently packed weight.
#include "internal.h"
#include "nn.h"

#include <algorithm>
#include <type_traits>

namespace clh {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

constexpr int TPB = 256;

__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }
__device__ __forceinline__ unsigned short f2bf(float f)
{
    // round to nearest even (inputs are finite)
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// two values rounded to nearest even and packed, lo in the low half (one
// v_cvt_pk_bf16_f32)
__device__ __forceinline__ unsigned pack_bf2(float lo, float hi)
{
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f2{lo, hi}, bf2));
}

// --- weight packing -------------------------------------------------------
// The 3x3x3 convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16:
// M = 16 voxels, N = 16 output channels, K = 32 = two taps x 16 input
// channels.  Lane l supplies row/column l % 16 of A/B and the 8 K values
// (l / 16, j): tap 2 tp + (l / 32), channel 8 ((l / 16) % 2) + j of the
// 16-channel chunk.  The same (lane, j) -> K assignment is used for both
// operands, so the product is the K sum whatever order the hardware takes
// the K values in.  27 taps are padded to 14 tap pairs with a zero tap.
// Forward packing (flip = 0): K = Ci, N = Co,
//   out[(((kc * 14 + tp) * NT + nt) * 64 + l) * 8 + j] = w[tap][kc*16 + c][nt*16 + l%16]
// Backward-data packing (flip = 1): K = Co, N = Ci, tap 26 - tap,
//   out[...] = w[26 - tap][nt*16 + l%16][kc*16 + c]
// with tap = 2 tp + l / 32, c = 8 ((l / 16) % 2) + j; zero for tap 27.
constexpr int NTP = 14;   // tap pairs

__global__ __launch_bounds__(TPB) void k_pack_w(const float *__restrict__ w, unsigned short *__restrict__ out, int Ci,
                                               int Co, int flip)
{
    const int K = flip ? Co : Ci, Nn = flip ? Ci : Co;
    const int KC = K / 16, NT = Nn / 16;
    const int total = KC * NTP * NT * 512;
    const int e = blockIdx.x * TPB + threadIdx.x;
    if (e >= total) return;
    const int j = e & 7, l = (e >> 3) & 63;
    int r = e >> 9;                  // (kc * NTP + tp) * NT + nt
    const int nt = r % NT;
    r /= NT;
    const int tp = r % NTP, kc = r / NTP;
    const int tap = 2 * tp + (l >> 5);
    const int k = kc * 16 + 8 * ((l >> 4) & 1) + j, n = nt * 16 + (l & 15);
    float val = 0.f;
    if (tap < 27) {
        if (!flip) val = w[((size_t)tap * Ci + k) * Co + n];
        else val = w[((size_t)(26 - tap) * Ci + n) * Co + k];
    }
    out[e] = f2bf(val);
}

__device__ __forceinline__ bf8 as_bf8(u4 v) { return __builtin_bit_cast(bf8, v); }

__device__ __forceinline__ float lo_bf(unsigned v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float hi_bf(unsigned v) { return __uint_as_float(v & 0xffff0000u); }

// LeakyReLU backward of a BF16-rounded gradient, from the sign of the output y
__device__ __forceinline__ float lrelu_bwd1(float g, float y, float slope) { return y > 0.f ? g : slope * g; }
__device__ __forceinline__ f4 lrelu_bwd4(f4 v, u2 y, float slope)
{
    const unsigned a = pack_bf2(v[0], v[1]), b = pack_bf2(v[2], v[3]);
    return f4{lrelu_bwd1(lo_bf(a), lo_bf(y[0]), slope), lrelu_bwd1(hi_bf(a), hi_bf(y[0]), slope),
              lrelu_bwd1(lo_bf(b), lo_bf(y[1]), slope), lrelu_bwd1(hi_bf(b), hi_bf(y[1]), slope)};
}

// four consecutive channels of one voxel; wide: the address is a multiple of
// their size (a caller's buffer may start at any element)
__device__ __forceinline__ void store4(unsigned short *o, f4 v, int wide)
{
    const u2 r = u2{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    if (wide) {
        *(u2 *)o = r;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (unsigned short)(r[j >> 1] >> (16 * (j & 1)));
    }
}
__device__ __forceinline__ void store4(float *o, f4 v, int wide)
{
    if (wide) {
        *(f4 *)o = v;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = v[j];
    }
}

// --- 3x3x3 convolution (zero padding), LDS-staged MFMA implicit GEMM -------
// in: BF16, voxels in order vs elements apart and 16-channel chunks cs elements
// apart (Layout; channels last: Ci and 16); wp: packed (K = Ci); bias FP32 [Co]
// or NULL; act: 0 none, 1 LeakyReLU(slope).  out: BF16 or FP32, laid out
// likewise.  mask (BF16 output only, laid out as out, or NULL): the activation
// whose LeakyReLU lies below the output, so that the rounded output v becomes
// v or slope v (rounded again) by its sign: dZ of the layer below.
// Work items: a 16 (x) x YR (y) x 8 MT / YR (z) output brick, YR = 8 or 4, times
// NTS of the NTT 16-channel output tiles, times the 16-channel input chunks.  A
// workgroup (4 wavefronts, each two rows of MT planes) walks its items in a
// loop: the input halo of the next item (one voxel more on every side) is requested
// into registers before the current one is computed from LDS, so the matrix
// cores do not wait for memory, and the weight fragments of a chunk (14 NTS,
// one per tap pair) sit in registers.
// Fragment reuse: a fragment is the voxels of one tap (lanes 0-31) and of the
// next tap (lanes 32-63), so there are five kinds per halo row, by the place of
// the first tap and the step to the second:
//   P0, P1: x offset 0 or 1, next voxel;  Q: x offset 2, next row;
//   R: x offset 2, next plane (taps 8, 9);  L: tap 26 and the zero tap.
// A wavefront streams the halo planes and reads each kind of each of its four
// halo rows once (15 LDS reads) for the up to 28 products of its two output
// rows and three output planes; with a read per product the LDS bandwidth
// bound the 16 -> 16 layers (24 us of a 128^3 launch against 12 us of MFMA).
// Weights are the A operand, voxels the B operand: a lane then holds four
// consecutive channels of one voxel and stores them with one instruction.
// The product order of an output (chunks, then tap pairs) is that of the
// packing, whatever MT and NTS.
// Measured (one MI355X, launch): 16 -> 16 at 128^3 91 -> 47 us, 48 -> 16 200 ->
// 130 us, 32 -> 32 at 64^3 31 -> 24 us; what is left is LDS reads (53 us of the
// 130) and staging that only the other workgroup of the CU overlaps.  Loads
// straight to LDS with three or four workgroups per CU and no prefetch: 65 and
// 167 us; three workgroups per CU with the prefetch: 17-60 spilled registers,
// 67 and 195 us.
// IN2: in holds the first two of 16 channels, the others are zero (the network's
// two images; vs = 2): they are filled in as the halo is staged, so the first
// layer reads 4 bytes a voxel instead of 32.  128^3: 55 -> 54 us (bound by
// its LDS reads), and the pass that packs the images 19 -> 7.6 us.
// Off: unsigned where a brick's halo spans less than 4 GiB of the input (each
// access is then a wave-uniform base plus a 32-bit offset), else size_t.
__device__ const u4 conv_zero = {0u, 0u, 0u, 0u};

template <int MT, int NTS, int YR, typename To, typename Off, bool MASK, bool IN2>
__global__ __launch_bounds__(TPB, 2) void k_conv3(const unsigned short *__restrict__ in, const u4 *__restrict__ wp,
                                                  const float *__restrict__ bias, To *__restrict__ out,
                                                  const unsigned short *__restrict__ mask, NNLayout li, NNLayout lo,
                                                  int D, int H, int W, int Ci, int act, float slope, int nbx, int nby,
                                                  int ntile, int NTT, int wide)
{
    constexpr int ZR = MT * 8 / YR;       // planes of a brick
    constexpr int XS = 18, YS = YR + 2, ZS = ZR + 2, NV = XS * YS * ZS, NQ = 2 * NV, NCH = (NQ + TPB - 1) / TPB;
    // two planes of 8 channels: the 16 lanes of a quarter of a fragment read
    // read 256 contiguous bytes; a plane pitch of 8 (mod 16) items puts the two
    // halves that neighbouring lanes stage on different banks
    constexpr int NP = NV + (24 - NV % 16) % 16;
    __shared__ u4 tile[2 * NP];
    const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = l & 15, half = (l >> 4) & 1, tsel = l >> 5;
    const int KC = Ci >> 4, ngrp = NTT / NTS;
    // tiles of this workgroup: first, stride, end.  Workgroups are dealt to the 8
    // XCDs round robin; each XCD takes a contiguous range of tiles, which share
    // input halos, so that they share its L2
    int t = blockIdx.x, tstep = gridDim.x, tend = ntile;
    if (((ntile | gridDim.x) & 7) == 0) {
        const int per = ntile >> 3;
        tend = ((t & 7) + 1) * per;
        t = (t & 7) * per + (t >> 3);
        tstep >>= 3;
    }
    // halo items of this thread (voxel q / 2, half q % 2): byte offset from the
    // halo origin, and its place: bits 0-5 first / last x, y, z of the halo
    // (bit 6: past the end)
    Off rel[NCH];
    unsigned edge[(NCH + 3) / 4] = {};
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int q = ch * TPB + tid, v = q >> 1, xt = v % XS, r = v / XS;
        const int yt = r % YS, zt = r / YS;
        rel[ch] = ((((Off)zt * H + yt) * W + xt) * li.vs + (IN2 ? 0 : (q & 1) * 8)) * 2;
        const unsigned e = (xt == 0) | (xt == XS - 1) << 1 | (yt == 0) << 2 | (yt == YS - 1) << 3 | (zt == 0) << 4 |
                           (zt == ZS - 1) << 5 | (q >= NQ) << 6;
        edge[ch >> 2] |= e << (8 * (ch & 3));
    }
    int x0, y0, z0, g;
    auto origin = [&](int tt) {
        g = tt % ngrp;
        tt /= ngrp;
        x0 = (tt % nbx) * 16;
        tt /= nbx;
        y0 = (tt % nby) * YR;
        z0 = (tt / nby) * ZR;
    };
    u4 st[NCH];
    auto request = [&](int kc) {
        const char *org = (const char *)(in + (((long)(z0 - 1) * H + (y0 - 1)) * W + (x0 - 1)) * li.vs + kc * (long)li.cs);
        // which faces of the halo lie outside the grid; a ragged brick (more
        // than its last face outside) compares coordinates.  Items outside
        // read a zero, so that no load depends on a branch.
        const bool ragged = x0 + 16 > W || y0 + YR > H || z0 + ZR > D;
        unsigned ok = 0;
        if (!ragged) {
            const unsigned faces = (x0 == 0) | (x0 + 16 == W) << 1 | (y0 == 0) << 2 | (y0 + YR == H) << 3 |
                                   (z0 == 0) << 4 | (z0 + ZR == D) << 5 | 1u << 6;
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch)
                ok |= (((edge[ch >> 2] >> (8 * (ch & 3))) & faces) == 0 ? 1u : 0u) << ch;
        } else {
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                const int q = ch * TPB + tid, v = q >> 1, r = v / XS;
                const int x = x0 - 1 + v % XS, y = y0 - 1 + r % YS, z = z0 - 1 + r / YS;
                ok |= (q < NQ && (unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H && (unsigned)z < (unsigned)D
                           ? 1u : 0u) << ch;
            }
        }
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            if constexpr (IN2)   // the other half's channels are zero
                st[ch] = u4{*(const unsigned *)((ok >> ch) & ~tid & 1 ? org + rel[ch] : (const char *)&conv_zero), 0u, 0u,
                            0u};
            else
                st[ch] = *(const u4 *)((ok >> ch) & 1 ? org + rel[ch] : (const char *)&conv_zero);
        }
    };
    f4 acc[MT][2][NTS];
    u4 bw[NTP][NTS];
    // rows wy, wy + 1 and planes wz ... wz + MT - 1 of the brick
    const int wy = 2 * (wv % (YR / 2)), wz = wv / (YR / 2) * MT;
    const u4 *base0 = tile + half * NP + (wz * YS + wy) * XS + m;
    const u4 *baseP = base0 + tsel, *baseQ = base0 + (XS - 2) * tsel + 2,
             *baseR = base0 + (YS * XS - 2 * XS - 2) * tsel + 2, *baseL = base0 + 2;
    u4 *put = tile + (tid & 1) * NP + (tid >> 1);
    if (t >= tend) return;
    origin(t);
    request(0);
    int kc = 0;
    bool first = true;
    for (;;) {
        const int cx = x0, cy = y0, cz = z0, cg = g;
        // weights first: their latency hides behind the staging (a workgroup
        // whose every item has the same chunk and group keeps them)
        if (first || KC > 1 || ngrp > 1) {
            const u4 *wk = wp + ((size_t)kc * NTP * NTT + cg * NTS) * 64 + l;
#pragma unroll
            for (int tp = 0; tp < NTP; ++tp)
#pragma unroll
                for (int nt = 0; nt < NTS; ++nt) bw[tp][nt] = wk[(tp * NTT + nt) * 64];
            first = false;
        }
        __syncthreads();
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
            if ((ch + 1) * TPB <= NQ || ch * TPB + tid < NQ) put[ch * (TPB / 2)] = st[ch];
        if (kc == 0) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int yi = 0; yi < 2; ++yi)
#pragma unroll
                    for (int nt = 0; nt < NTS; ++nt) acc[i][yi][nt] = f4{0.f, 0.f, 0.f, 0.f};
        }
        // the next item
        const bool last_kc = kc + 1 == KC;
        const bool more = !last_kc || t + tstep < tend;
        if (more) {
            if (last_kc) {
                t += tstep;
                origin(t);
                kc = 0;
            } else {
                ++kc;
            }
            request(kc);
        }
        __syncthreads();
        // the mask of the item's outputs, in flight while they are computed
        // (with two output tiles the registers do not allow it)
        constexpr bool PRE = MASK && NTS == 1;
        u2 mk[PRE ? MT : 1][2];
        if (PRE && last_kc) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int yi = 0; yi < 2; ++yi) {
                    const int z = min(cz + wz + i, D - 1), y = min(cy + wy + yi, H - 1), x = min(m, W - 1 - cx);
                    mk[PRE ? i : 0][yi] = *(const u2 *)(mask + (((size_t)z * H + y) * W + cx) * lo.vs + cg * lo.cs +
                                                        x * lo.vs + 4 * (l >> 4));
                }
        }
        // the fragments of step (plane zz, k) are read one step ahead of its
        // products, so that LDS latency hides behind them (left to itself the
        // compiler reads each pair just before its use and waits)
        bf8 P0[2][4], P1[2][4], Q[2][3], R[2][2], L[2][2];
        auto row = [&](const u4 *b, int zz, int r, int dx) { return as_bf8(b[(zz * YS + r) * XS + dx]); };
        auto fetch = [&](int zz, int k) {
            const bool d0 = zz < MT, d1 = zz >= 1 && zz <= MT, d2 = zz >= 2;
            const int u = zz & 1;
            if (k == 0) {
                if (d0 || d2) P0[u][0] = row(baseP, zz, 0, 0);
                P0[u][1] = row(baseP, zz, 1, 0);
                if (d1) P1[u][0] = row(baseP, zz, 0, 1);
                P1[u][1] = row(baseP, zz, 1, 1);
            } else if (k == 1) {
                if (d0 || d2) Q[u][0] = row(baseQ, zz, 0, 0);
                Q[u][1] = row(baseQ, zz, 1, 0);
                P0[u][2] = row(baseP, zz, 2, 0);
            } else if (k == 2) {
                P1[u][2] = row(baseP, zz, 2, 1);
                if (d1) Q[u][2] = row(baseQ, zz, 2, 0);
            } else if (k == 3) {
                if (d0 || d2) P0[u][3] = row(baseP, zz, 3, 0);
                if (d1) P1[u][3] = row(baseP, zz, 3, 1);
            } else {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    if (d0) R[u][r] = row(baseR, zz, 2 + r, 0);
                    if (d2) L[u][r] = row(baseL, zz, 2 + r, 0);
                }
            }
        };
        fetch(0, 0);
#pragma unroll
        for (int zk = 0; zk < 5 * (MT + 2); ++zk) {
            const int zz = zk / 5, k = zk % 5, u = zz & 1;
            const bool d0 = zz < MT, d1 = zz >= 1 && zz <= MT, d2 = zz >= 2;
            if (zk + 1 < 5 * (MT + 2)) fetch((zk + 1) / 5, (zk + 1) % 5);
            __builtin_amdgcn_sched_barrier(0);
            // tap pairs 0-4, 5-8 and 9-13 of the output planes zz, zz - 1 and zz - 2
#pragma unroll
            for (int yi = 0; yi < 2; ++yi) {
                const bf8 a02 = k == 0 ? P0[u][yi] : k == 1 ? Q[u][yi] : k == 2 ? P1[u][yi + 1] : P0[u][yi + 2];
                const bf8 a1 = k == 0 ? P1[u][yi] : k == 1 ? P0[u][yi + 1] : k == 2 ? Q[u][yi + 1] : P1[u][yi + 2];
                bf8 al = a02;
                if (k == 4 && d2) {
                    u4 raw = __builtin_bit_cast(u4, L[u][yi]);
                    if (tsel) raw = u4{0u, 0u, 0u, 0u};   // tap 27 does not exist
                    al = as_bf8(raw);
                }
#pragma unroll
                for (int nt = 0; nt < NTS; ++nt) {
                    auto mac = [&](int i, int tp, bf8 v) {
                        acc[i][yi][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(bw[tp][nt]), v,
                                                                                 acc[i][yi][nt], 0, 0, 0);
                    };
                    if (d0) mac(d0 ? zz : 0, k, k == 4 ? R[u][yi] : a02);
                    if (d1 && k < 4) mac(d1 ? zz - 1 : 0, 5 + (k & 3), a1);
                    if (d2) mac(d2 ? zz - 2 : 0, 9 + k, al);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (last_kc) {
            // D[m][n]: n = l % 16 (voxel along x), m = 4 (l / 16) + j (channel);
            // row bases are wave-uniform
            const int cl = 4 * (l >> 4), lane_off = m * lo.vs + cl;
#pragma unroll
            for (int nt = 0; nt < NTS; ++nt) {
                const int co = (cg * NTS + nt) * 16;
                f4 bb = f4{0.f, 0.f, 0.f, 0.f};
                if (bias) bb = f4{bias[co + cl], bias[co + cl + 1], bias[co + cl + 2], bias[co + cl + 3]};
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int yi = 0; yi < 2; ++yi) {
                        const int z = cz + wz + i, y = cy + wy + yi;
                        if (y >= H || z >= D) continue;
                        f4 v = acc[i][yi][nt] + bb;
                        if (act) {
#pragma unroll
                            for (int j = 0; j < 4; ++j) v[j] = v[j] > 0.f ? v[j] : slope * v[j];
                        }
                        const size_t row = (((size_t)z * H + y) * W + cx) * lo.vs + (cg * NTS + nt) * lo.cs;
                        if (cx + m >= W) continue;
                        if constexpr (MASK)
                            v = lrelu_bwd4(v, PRE ? mk[PRE ? i : 0][yi] : *(const u2 *)(mask + row + lane_off), slope);
                        store4(out + row + lane_off, v, wide);
                    }
            }
        }
        if (!more) break;
    }
}

// --- weight gradient --------------------------------------------------------
// part[chunk] = (gw partial [t][Ci][Co], gb partial [Co]): sums over the
// chunk's voxels p of X[p + t - 1][i] dZ[p][o] and of dZ[p][o].  GEMM with
// M = 16 input channels (chunk kc), N = 16 output channels (tile ct), K = 32
// voxels: two rows of 16 x; lane group g = l / 16, item j holds row g / 2,
// x = 8 (g % 2) + j.
// A workgroup owns one (kc, ct) pair and a run of 16 (x) x 4 (y) x 4 (z) voxel
// tiles.  The x shift of a tap is taken on dZ, so X is staged without an x halo
// (16 x 6 x 6 voxels) and dZ with one (18 x 4 x 4); both go straight to LDS as
// they lie in memory, and the transposing LDS read (ds_read_b64_tr_b16: lane i
// of 16 receives channel i of 4 voxels) forms the fragments.  Two buffers: the
// next tile is in flight while the current one is computed.
// Wavefront w owns two rows of two planes and all 27 taps (108 accumulators):
// 12 X fragments and 6 dZ fragments serve 54 products, a third of an LDS read
// per product.  The wavefronts' sums are added in a fixed order at the end; the bias
// sums use an all-ones X operand.
// Measured (one MI355X, with the sum of the partials): 16 -> 16 at 128^3 165 ->
// 42 us, 48 -> 16 365 -> 116 us (channels last).  Before, X was transposed into three shifted
// copies by 2-byte LDS writes (24 per staged 16 bytes).
typedef short s4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4 lds_s4;
typedef __attribute__((address_space(3))) void lds_void;

// fragment of 8 voxels 32 bytes apart from LDS byte address a (of this lane)
__device__ __forceinline__ bf8 frag_tr(unsigned a)
{
    struct {
        s4 lo, hi;
    } f;
    f.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(uintptr_t)a);
    f.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(uintptr_t)(a + 128));
    return __builtin_bit_cast(bf8, f);
}

// DMA: X and dZ on 16-byte boundaries, which the loads straight to LDS need; else
// through registers.
template <bool DMA>
__global__ __launch_bounds__(TPB, 2) void k_conv3_dw(const unsigned short *__restrict__ X,
                                                     const unsigned short *__restrict__ dZ, float *__restrict__ part,
                                                     NNLayout lx, NNLayout lz, int D, int H, int W, int Ci, int Co,
                                                     int ntx, int nty, int ntiles, int tpc)
{
    constexpr int XQ = 16 * 6 * 6 * 2, ZQ = 18 * 4 * 4 * 2, NCH = (XQ + ZQ + TPB - 1) / TPB, BUF = NCH * TPB;
    __shared__ u4 tile[2 * BUF];
    const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = l >> 4, ln = l & 15;
    const int KC = Ci >> 4, npair = KC * (Co >> 4);
    // the pairs of a run of tiles share its data: consecutive on one XCD
    int b = blockIdx.x;
    const int nb = gridDim.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int pair = b % npair, chunk = b / npair;
    const int kc = pair % KC, ct = pair / KC;
    const int t0 = chunk * tpc, t1 = min(ntiles, t0 + tpc);
    // items of this thread: [voxel][half] of X, then of dZ; byte offset from the
    // tile's first voxel in its tensor, and place (bits 0-5: first / last x, y,
    // z of a halo; bit 6: past the end)
    long rel[NCH];
    unsigned edge[(NCH + 3) / 4] = {};
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int q = ch * TPB + tid;
        const bool isx = q < XQ;
        const int v = (isx ? q : q - XQ) >> 1, xt = isx ? v & 15 : v % 18, r = isx ? v >> 4 : v / 18;
        const int yt = isx ? r % 6 : r & 3, zt = isx ? r / 6 : r >> 2;
        const int vs = isx ? lx.vs : lz.vs;
        rel[ch] = ((((long)zt * H + yt) * W + xt) * vs + (q & 1) * 8) * 2;
        const unsigned e = isx ? (yt == 0) << 2 | (yt == 5) << 3 | (zt == 0) << 4 | (zt == 5) << 5
                               : (xt == 0) | (xt == 17) << 1 | (q >= XQ + ZQ) << 6;
        edge[ch >> 2] |= e << (8 * (ch & 3));
    }
    auto request = [&](int tI, int buf) {
        const int x0 = (tI % ntx) * 16, y0 = ((tI / ntx) % nty) * 4, z0 = (tI / (ntx * nty)) * 4;
        const char *xo = (const char *)(X + (((long)(z0 - 1) * H + (y0 - 1)) * W + x0) * lx.vs + kc * (long)lx.cs);
        const char *zo = (const char *)(dZ + (((long)z0 * H + y0) * W + (x0 - 1)) * lz.vs + ct * (long)lz.cs);
        unsigned ok = 0;
        if (x0 + 16 <= W && y0 + 4 <= H && z0 + 4 <= D) {
            const unsigned faces = (x0 == 0) | (x0 + 16 == W) << 1 | (y0 == 0) << 2 | (y0 + 4 == H) << 3 |
                                   (z0 == 0) << 4 | (z0 + 4 == D) << 5 | 1u << 6;
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch)
                ok |= (((edge[ch >> 2] >> (8 * (ch & 3))) & faces) == 0 ? 1u : 0u) << ch;
        } else {
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                const int q = ch * TPB + tid;
                const bool isx = q < XQ;
                const int v = (isx ? q : q - XQ) >> 1, r = isx ? v >> 4 : v / 18;
                const int x = isx ? x0 + (v & 15) : x0 - 1 + v % 18, y = isx ? y0 - 1 + r % 6 : y0 + (r & 3),
                          z = isx ? z0 - 1 + r / 6 : z0 + (r >> 2);
                ok |= (q < XQ + ZQ && (unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H && (unsigned)z < (unsigned)D
                           ? 1u : 0u) << ch;
            }
        }
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            const char *src = (ch * TPB + tid < XQ ? xo : zo) + rel[ch];
            const void *from = (ok >> ch) & 1 ? src : (const char *)&conv_zero;
            if constexpr (DMA) {
                __builtin_amdgcn_global_load_lds(from, (lds_void *)(tile + buf * BUF + ch * TPB + wv * 64), 16, 0, 0);
            } else {
                u4 v;
                __builtin_memcpy(&v, from, sizeof(v));
                tile[buf * BUF + ch * TPB + tid] = v;
            }
        }
    };
    f4 acc[27], accb = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 27; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    const bool do_bias = kc == 0;
    // rows yp, yp + 1 of planes zb, zb + 1
    const int yp = (wv & 1) * 2, zb = (wv >> 1) * 2;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void *)tile;
    const unsigned ax = lds0 + (((zb * 6 + yp + (g >> 1)) * 16 + 8 * (g & 1) + (ln >> 2)) * 32 + (ln & 3) * 8);
    const unsigned az = lds0 + XQ * 16 + (((zb * 4 + yp + (g >> 1)) * 18 + 8 * (g & 1) + (ln >> 2)) * 32 + (ln & 3) * 8);
    if (t0 < t1) request(t0, 0);
    for (int tI = t0; tI < t1; ++tI) {
        const int buf = (tI - t0) & 1;
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        // every fragment first, then the request: an LDS read after it would
        // wait for it (the compiler does not tell the two buffers apart)
        const unsigned bo = buf * BUF * 16;
        bf8 bz[2][3], a[12];
#pragma unroll
        for (int zi = 0; zi < 2; ++zi)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) bz[zi][dx] = frag_tr(az + bo + ((zi * 4) * 18 + 2 - dx) * 32);
#pragma unroll
        for (int s = 0; s < 12; ++s) a[s] = frag_tr(ax + bo + ((s / 3) * 6 + s % 3) * 512);
        __builtin_amdgcn_sched_barrier(0);
        if (tI + 1 < t1) request(tI + 1, buf ^ 1);
#pragma unroll
        for (int s = 0; s < 12; ++s) {
            const int zq = s / 3, dy = s % 3;
#pragma unroll
            for (int zi = 0; zi < 2; ++zi) {
                const int dz = zq - zi;
                if (dz < 0 || dz > 2) continue;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[dz * 9 + dy * 3 + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], bz[zi][dx],
                                                                                       acc[dz * 9 + dy * 3 + dx], 0, 0, 0);
            }
        }
        if (do_bias) {
            const bf8 ones = as_bf8(u4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
#pragma unroll
            for (int zi = 0; zi < 2; ++zi) accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, bz[zi][1], accb, 0, 0, 0);
        }
    }
    // sum over the wavefronts, half of the 27 taps and the bias at a time: wavefront
    // w adds and stores the sums w, w + 4, ... (one wavefront adding and storing all of
    // them: 8.3 -> 7.6 us where a run is one tile)
    f4 *red = (f4 *)tile;                 // 4 wavefronts x 14 x 64 values
    float *dst = part + (size_t)chunk * (27 * Ci * Co + Co);
#pragma unroll
    for (int h = 0; h < 28; h += 14) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 14; ++t) red[(wv * 14 + t) * 64 + l] = h + t < 27 ? acc[h + t < 27 ? h + t : 0] : accb;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = wv + 4 * u;
            if (t >= 14) break;
            const f4 *r = red + t * 64 + l;
            const f4 v = (r[0] + r[2 * 14 * 64]) + (r[14 * 64] + r[3 * 14 * 64]);
            // D[m][n]: m = 4 g + j (input channel), n = ln (output channel)
            if (h + t < 27) {
#pragma unroll
                for (int j = 0; j < 4; ++j) dst[((size_t)(h + t) * Ci + kc * 16 + 4 * g + j) * Co + ct * 16 + ln] = v[j];
            } else if (do_bias && g == 0) {
                dst[27 * (size_t)Ci * Co + ct * 16 + ln] = v[0];
            }
        }
    }
}

// Element (tap t, channels i, o) of a chunk's weight gradient as plain sums of
// the products inside the grid.  k_conv3_dw stages zeros outside the grid, and
// zero times a value that is not finite is NaN in taps that do not see it.
struct DwOperands {
    const unsigned short *X, *dZ;
    NNLayout lx, lz;
    int D, H, W, Ci, Co, ntx, nty, ntiles, tpc;
};
__device__ float dw_element(const DwOperands &a, int chunk, int t, int i, int o)
{
    const unsigned short *x = a.X + (size_t)(i >> 4) * a.lx.cs + (i & 15);
    const unsigned short *dz = a.dZ + (size_t)(o >> 4) * a.lz.cs + (o & 15);
    const int sx = t % 3 - 1, sy = t / 3 % 3 - 1, sz = t / 9 - 1, t1 = min(a.ntiles, (chunk + 1) * a.tpc);
    double s = 0.0;
    for (int tI = chunk * a.tpc; tI < t1; ++tI) {
        const int x0 = tI % a.ntx * 16, y0 = tI / a.ntx % a.nty * 4, z0 = tI / (a.ntx * a.nty) * 4;
        // the tiles are those of X along x, of dZ along y and z
        for (int z = max(z0, -sz); z < min(z0 + 4, min(a.D, a.D - sz)); ++z)
            for (int y = max(y0, -sy); y < min(y0 + 4, min(a.H, a.H - sy)); ++y) {
                for (int v = max(x0, sx); v < min(x0 + 16, min(a.W, a.W + sx)); ++v)
                    s += (double)bf2f(x[(((size_t)(z + sz) * a.H + y + sy) * a.W + v) * a.lx.vs]) *
                         bf2f(dz[(((size_t)z * a.H + y) * a.W + v - sx) * a.lz.vs]);
                if (isnan(s)) return NAN;
            }
    }
    return (float)s;
}

// Fixed-order sum of the chunk partials: row c of partial holds nw weight
// values then nb bias values (row stride nw + nb).  A workgroup owns 64
// consecutive outputs; wave w of NW sums the chunks c = w (mod NW) in order,
// eight loads in flight, then the wave sums are added in order.  16 waves
// where there are more chunks than 4 waves take in one go, 4 else: the 16 -> 16
// layers have 27 KB rows and 512 chunks, few outputs whose rows are split
// over many waves (4 waves with one load in flight: 48 us), the wide layers of
// small grids have up to 2.6 MB rows and a few chunks (128 -> 128 at 6^3, 4 chunks:
// 16 waves 14 us, 4 waves 5 us).  A sum that is not
// finite is taken again, with dw_element in place of the weight partials that are
// not (masked operands in k_conv3_dw would take 5-38 % of its time).
constexpr int SUM_LOADS = 8;
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_sum_partials(const float *__restrict__ partial, int nchunk, int nw, int nb,
                                                          float *__restrict__ gw, float *__restrict__ gb, DwOperands a)
{
    __shared__ float red[NW][64];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + l;
    const int rs = nw + nb;
    float s = 0.f;
    if (e < rs) {
        for (int c = w; c < nchunk; c += SUM_LOADS * NW) {
            float v[SUM_LOADS];
#pragma unroll
            for (int u = 0; u < SUM_LOADS; ++u)
                if (c + u * NW < nchunk) v[u] = partial[(size_t)(c + u * NW) * rs + e];
#pragma unroll
            for (int u = 0; u < SUM_LOADS; ++u)
                if (c + u * NW < nchunk) s += v[u];
        }
        if (!isfinite(s) && e < nw) {
            s = 0.f;
            for (int c = w; c < nchunk; c += NW) {
                const float v = partial[(size_t)c * rs + e];
                s += isfinite(v) ? v : dw_element(a, c, e / (a.Ci * a.Co), e / a.Co % a.Ci, e % a.Co);
            }
        }
    }
    red[w][l] = s;
    __syncthreads();
    if (w == 0 && e < rs) {
        float t = red[0][l];
#pragma unroll
        for (int u = 1; u < NW; ++u) t += red[u][l];
        if (e < nw) gw[e] = t;
        else if (gb) gb[e - nw] = t;
    }
}

// The network keeps its activations by 16-channel chunks, [C / 16][D][H][W][16]:
// a convolution stages one chunk at a time, so each staged row is contiguous
// (channels last, a 48-channel voxel's 96 bytes were fetched three times, a
// third of every cache line used: dW of 48 -> 16 at 128^3 115 -> 98 us), a
// skip connection is written by its convolution into its place in the
// concatenated tensor, and the elementwise layers see 16-channel tensors with
// the chunks stacked along z.  They work on 8-channel groups (one 16-byte load
// per tensor and thread).
__device__ __forceinline__ void unpack8(u4 v, float (&f)[8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = lo_bf(v[i]);
        f[2 * i + 1] = hi_bf(v[i]);
    }
}
__device__ __forceinline__ u4 pack8(const float (&f)[8])
{
    u4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = pack_bf2(f[2 * i], f[2 * i + 1]);
    return v;
}
// LeakyReLU backward of 8 gradients (rounded to BF16 first), from the output y
__device__ __forceinline__ u4 lrelu_bwd8(const float (&g)[8], u4 y, float slope)
{
    float f[8], yy[8];
    unpack8(pack8(g), f);
    unpack8(y, yy);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = lrelu_bwd1(f[i], yy[i], slope);
    return pack8(f);
}

// sums of the 2 x 2 x 2 children of a coarse voxel (H, W of the fine grid)
__device__ __forceinline__ void children8(const u4 *__restrict__ in, int x, int y, int z, int H, int W, int c,
                                          float (&s)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float f[8];
                unpack8(in[((((size_t)(2 * z + a)) * H + 2 * y + b) * W + 2 * x + q) * 2 + c], f);
#pragma unroll
                for (int i = 0; i < 8; ++i) s[i] += f[i];
            }
}

// 2x2x2 average pooling (D, H, W of the input, D over all chunks)
__global__ __launch_bounds__(TPB) void k_pool2(const u4 *__restrict__ in, u4 *__restrict__ out, int D, int H, int W)
{
    const int d = D / 2, h = H / 2, w = W / 2;
    const size_t e = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (e >= (size_t)d * h * w * 2) return;
    const int c = e & 1;
    const size_t v = e >> 1;
    const int x = v % w, y = (v / w) % h, z = v / ((size_t)w * h);
    float s[8];
    children8(in, x, y, z, H, W, c, s);
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] *= 0.125f;
    out[e] = pack8(s);
}

// the gradient of an activation Y that is both pooled and skipped, through its
// LeakyReLU: g[fine] <- bwd(g[fine] + gpool[coarse] / 8)
__global__ __launch_bounds__(TPB) void k_pool2_bwd(const u4 *__restrict__ gpool, u4 *__restrict__ g,
                                                   const u4 *__restrict__ Y, float slope, int D, int H, int W)
{
    const size_t e = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (e >= (size_t)D * H * W * 2) return;
    const int c = e & 1;
    const size_t v = e >> 1;
    const int x = v % W, y = (v / W) % H, z = v / ((size_t)W * H);
    float p[8], f[8];
    unpack8(gpool[((((size_t)z / 2) * (H / 2) + y / 2) * (W / 2) + x / 2) * 2 + c], p);
    unpack8(g[e], f);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = f[i] + p[i] * 0.125f;
    g[e] = lrelu_bwd8(f, Y[e], slope);
}

// nearest 2x upsampling (D, H, W of the output)
__global__ __launch_bounds__(TPB) void k_up2(const u4 *__restrict__ a, u4 *__restrict__ out, int D, int H, int W)
{
    const size_t e = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (e >= (size_t)D * H * W * 2) return;
    const int c = e & 1;
    const size_t v = e >> 1;
    const int x = v % W, y = (v / W) % H, z = v / ((size_t)W * H);
    out[e] = a[((((size_t)z / 2) * (H / 2) + y / 2) * (W / 2) + x / 2) * 2 + c];
}

// backward of up2, through the LeakyReLU of Y: ga[coarse] <- bwd(sum of its
// children) (D, H, W of the fine grid)
__global__ __launch_bounds__(TPB) void k_up2_bwd(const u4 *__restrict__ g, u4 *__restrict__ ga,
                                                 const u4 *__restrict__ Y, float slope, int D, int H, int W)
{
    const int d = D / 2, h = H / 2, w = W / 2;
    const size_t e = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (e >= (size_t)d * h * w * 2) return;
    const int c = e & 1;
    const size_t v = e >> 1;
    const int x = v % w, y = (v / w) % h, z = v / ((size_t)w * h);
    float s[8];
    children8(g, x, y, z, H, W, c, s);
    ga[e] = lrelu_bwd8(s, Y[e], slope);
}

// head: 1x1x1 convolution Ci -> 3, FP32 output as SoA [3][P]
__global__ __launch_bounds__(TPB) void k_head(const unsigned short *__restrict__ in, const float *__restrict__ w,
                                              const float *__restrict__ b, float *__restrict__ out, size_t P, int Ci)
{
    const size_t p = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (p >= P) return;
    float s0 = b[0], s1 = b[1], s2 = b[2];
    const u4 *src = (const u4 *)(in + p * Ci);
    for (int i8 = 0; i8 < Ci / 8; ++i8) {
        float x[8];
        unpack8(src[i8], x);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i8 * 8 + u;
            s0 = fmaf(w[i * 3 + 0], x[u], s0);
            s1 = fmaf(w[i * 3 + 1], x[u], s1);
            s2 = fmaf(w[i * 3 + 2], x[u], s2);
        }
    }
    out[p] = s0;
    out[P + p] = s1;
    out[2 * P + p] = s2;
}

// head backward, through the LeakyReLU of its input Y: gin[p][i] =
// bwd(sum_o w[i][o] gout[o][p]), 8 channels per thread
__global__ __launch_bounds__(TPB) void k_head_bwd_x(const float *__restrict__ gout, const float *__restrict__ w,
                                                    const u4 *__restrict__ Y, float slope, u4 *__restrict__ gin,
                                                    size_t P)
{
    const size_t e = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (e >= P * 2) return;
    const size_t p = e >> 1;
    const int i0 = 8 * (int)(e & 1);
    const float g0 = gout[p], g1 = gout[P + p], g2 = gout[2 * P + p];
    float f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float *wi = w + (i0 + i) * 3;
        f[i] = wi[0] * g0 + wi[1] * g1 + wi[2] * g2;
    }
    gin[e] = lrelu_bwd8(f, Y[e], slope);
}

// head weight gradient: every workgroup sums, over its voxels, the 16 x 3
// products in[p][i] gout[o][p] and the 3 bias terms gout[o][p] (FP64), then
// writes them as partials[c][block], c = i * 3 + o (bias: 48 + o)
constexpr int HEAD_CI = 16, HEAD_NC = HEAD_CI * 3 + 3;

__global__ __launch_bounds__(TPB) void k_head_bwd_w(const unsigned short *__restrict__ in,
                                                    const float *__restrict__ gout, size_t P,
                                                    double *__restrict__ partials)
{
    double acc[HEAD_NC];
#pragma unroll
    for (int c = 0; c < HEAD_NC; ++c) acc[c] = 0.0;
    for (size_t p = (size_t)blockIdx.x * TPB + threadIdx.x; p < P; p += (size_t)gridDim.x * TPB) {
        const float g0 = gout[p], g1 = gout[P + p], g2 = gout[2 * P + p];
        const u4 lo = *(const u4 *)(in + p * HEAD_CI), hi = *(const u4 *)(in + p * HEAD_CI + 8);
        const unsigned short *e0 = (const unsigned short *)&lo, *e1 = (const unsigned short *)&hi;
#pragma unroll
        for (int i = 0; i < HEAD_CI; ++i) {
            const double x = bf2f(i < 8 ? e0[i] : e1[i - 8]);
            acc[i * 3 + 0] += x * g0;
            acc[i * 3 + 1] += x * g1;
            acc[i * 3 + 2] += x * g2;
        }
        acc[48] += g0;
        acc[49] += g1;
        acc[50] += g2;
    }
    // one barrier for all 51 sums
    __shared__ double red[TPB / 64][HEAD_NC];
#pragma unroll
    for (int c = 0; c < HEAD_NC; ++c) {
        double v = acc[c];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][c] = v;
    }
    __syncthreads();
    if (threadIdx.x < HEAD_NC) {
        double v = red[0][threadIdx.x];
        for (int q = 1; q < TPB / 64; ++q) v += red[q][threadIdx.x];
        partials[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = v;
    }
}

// out[c] = sum_b partials[c][b] in a fixed order, one workgroup per c
__global__ __launch_bounds__(TPB) void k_finalize_rows(const double *__restrict__ partials, int nb,
                                                       double *__restrict__ out)
{
    const double *row = partials + (size_t)blockIdx.x * nb;
    double acc = 0.0;
    for (int q = threadIdx.x; q < nb; q += TPB) acc += row[q];
    acc = block_sum(acc);
    if (threadIdx.x == 0) out[blockIdx.x] = acc;
}

// loss = 0.5 / P sum (pred - label)^2 over 3 components; grad = (pred - label) / P.
// W values per access: 4 where label allows it, else 1.  Two streams read and one
// written by 512 workgroups, bound by the loads they have in flight: 128^3 30 -> 14
// us.
template <int W>
__global__ __launch_bounds__(TPB) void k_mse(const float *__restrict__ pred, const float *__restrict__ label, size_t n,
                                             float inv, float *__restrict__ grad, double *__restrict__ partials)
{
    typedef float fw __attribute__((ext_vector_type(W)));
    double s = 0.0;
    for (size_t e = (size_t)blockIdx.x * TPB + threadIdx.x; e < n / W; e += (size_t)gridDim.x * TPB) {
        const fw r = ((const fw *)pred)[e] - ((const fw *)label)[e];
        ((fw *)grad)[e] = r * inv;
#pragma unroll
        for (int i = 0; i < W; ++i) s += (double)r[i] * r[i];
    }
    s = block_sum(s);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// Adam on FP32 master parameters
__global__ __launch_bounds__(TPB) void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, size_t n, float lr, float b1, float b2, float eps,
                                              float c1, float c2)
{
    const size_t e = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (e >= n) return;
    const float gg = g[e];
    const float mm = b1 * m[e] + (1.f - b1) * gg;
    const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
    m[e] = mm;
    v[e] = vv;
    p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

// two FP32 scalar fields [P] -> BF16 channels-last [P][16] (channels 2..15 zero)
__global__ __launch_bounds__(TPB) void k_pack_input(const float *__restrict__ a, const float *__restrict__ b,
                                                    u4 *__restrict__ out, size_t P)
{
    const size_t p = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (p >= P) return;
    out[2 * p] = u4{(unsigned)f2bf(a[p]) | ((unsigned)f2bf(b[p]) << 16), 0u, 0u, 0u};
    out[2 * p + 1] = u4{0u, 0u, 0u, 0u};
}

// the same as two channels per voxel
__global__ __launch_bounds__(TPB) void k_pack_two(const float *__restrict__ a, const float *__restrict__ b,
                                                  unsigned *__restrict__ out, size_t P)
{
    const size_t p = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (p >= P) return;
    out[p] = (unsigned)f2bf(a[p]) | ((unsigned)f2bf(b[p]) << 16);
}

inline unsigned nblk(size_t n) { return (unsigned)((n + TPB - 1) / TPB); }

} // namespace

size_t nn_packed_weight_elems(int Ci, int Co) { return (size_t)NTP * 2 * Ci * Co; }

void nn_pack_weights(const float *w, unsigned short *out, int Ci, int Co, int flip, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack_w, dim3(nblk(nn_packed_weight_elems(Ci, Co))), dim3(TPB), 0, s, w, out, Ci, Co, flip);
}

template <int MT, int NTS, int YR, typename To, typename Off = unsigned, bool IN2 = false>
static void conv3_launch(const unsigned short *in, const void *wp, const float *bias, To *out, const unsigned short *mask, NNLayout li, NNLayout lo, int D, int H, int W,
                         int Ci, int NT, int act, float slope, hipStream_t s)
{
    constexpr int ZR = MT * 8 / YR;
    const int nbx = (W + 15) / 16, nby = (H + YR - 1) / YR, nbz = (D + ZR - 1) / ZR;
    const int ntile = nbx * nby * nbz * (NT / NTS);
    const int wide = ((uintptr_t)out % (4 * sizeof(To))) == 0;
    // two resident workgroups per CU (of 160-250 VGPRs) walk the tiles
    const int grid = ntile < 512 ? ntile : 512;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(TPB), 0, s, in, (const u4 *)wp, bias, out, mask, li, lo, D, H, W,
                           Ci, act, slope, nbx, nby, ntile, NT, wide);
    };
    if constexpr (sizeof(To) == 2 && !IN2 && YR == 8) {
        if (mask) return go(k_conv3<MT, NTS, YR, To, Off, true, false>);
    }
    go(k_conv3<MT, NTS, YR, To, Off, false, IN2>);
}

// Brick depth and output tiles per workgroup (MT, NTS) by the time of their items:
// rounds of 512 walkers, two per CU.  Times per item and 16-channel input chunk in
// 0.1 us, fitted to 340 launches of ragged and whole sizes in each variant (one
// MI355X): one walker per CU, two, and two in the rounds after the first.  A deep
// brick reads less halo for its work, a flat one gives more items and less work past
// the last plane.  On average this is 0.4 % off the best variant; the rule "the
// largest brick with 512 items" was 4.6 % off: two rounds of flat bricks for one of
// deeper ones (30^3 64 -> 64 22.6 -> 16.9 us), bricks of four planes for grids of
// one (1 x 40 x 200 128 -> 192 66 -> 34 us).
struct ConvBrick {
    int mt, nts;
    double alone, paired, later;
    int rows;
    double time(int items) const
    {
        const int last = items % 512;
        double t = last == 0 ? 0.0 : last <= 256 ? alone : alone + (paired - alone) * (last - 256) / 256.0;
        if (items >= 512) t += paired + (items / 512 - 1) * later;
        return t;
    }
};
// Bricks of 4 rows and twice the planes (four: they are built) where they are 10 %
// better by fewer rows past the last one: 100 x 4 x 100 64 -> 128 55 -> 33 us, 60 x 12
// x 60 44 -> 37 us.  Their halo has shorter runs of memory (113 x 60 x 83 48 -> 16, as
// many items: 48 -> 57 us).
static ConvBrick conv3_brick(int D, int H, int W, int NT, bool two, bool four)
{
    constexpr ConvBrick bricks[] = {{2, 2, 31., 47., 48.}, {4, 1, 31., 50., 50.}, {2, 1, 19., 28., 31.}, {1, 1, 15., 18., 24.}};
    ConvBrick best{};
    double tbest = 0.0;
    for (int yr = 8; yr >= (four ? 4 : 8); yr -= 4)
        for (const ConvBrick &b : bricks) {
            if (b.nts == 2 && (two || NT % 2)) continue;
            const int zr = b.mt * 8 / yr;
            const double t = b.time(((W + 15) / 16) * ((H + yr - 1) / yr) * ((D + zr - 1) / zr) * (NT / b.nts)) *
                             (yr == 4 ? 1.1 : 1.0);
            if (best.mt && t >= tbest) continue;
            best = b;
            best.rows = yr;
            tbest = t;
        }
    return best;
}

template <typename To, bool IN2 = false>
static void conv3_dispatch(const unsigned short *in, const void *wp, const float *bias, To *out, const unsigned short *mask, NNLayout li, NNLayout lo, int D, int H, int W,
                           int Ci, int Co, int act, float slope, hipStream_t s)
{
    const int NT = Co / 16;
    // 32-bit offsets within the halo of the deepest brick of 4 rows and of 8
    const double voxel = W * li.vs * 2.0;
    const bool four = !IN2 && !mask && (10.0 * H + 10.0) * voxel < 4294967296.0;
    const ConvBrick b = conv3_brick(D, H, W, NT, IN2, four);
    auto go = [&](auto rows) {
        constexpr int YR = decltype(rows)::value;
        if constexpr (!IN2)
            if (b.nts == 2)
                return conv3_launch<2, 2, YR, To>(in, wp, bias, out, mask, li, lo, D, H, W, Ci, NT, act, slope, s);
        if (b.mt == 4)
            conv3_launch<4, 1, YR, To, unsigned, IN2>(in, wp, bias, out, mask, li, lo, D, H, W, Ci, NT, act, slope, s);
        else if (b.mt == 2)
            conv3_launch<2, 1, YR, To, unsigned, IN2>(in, wp, bias, out, mask, li, lo, D, H, W, Ci, NT, act, slope, s);
        else
            conv3_launch<1, 1, YR, To, unsigned, IN2>(in, wp, bias, out, mask, li, lo, D, H, W, Ci, NT, act, slope, s);
    };
    // (the network's grids, the only ones of two channels, are far below 4 GiB)
    if constexpr (!IN2) {
        if ((6.0 * H + 10.0) * voxel >= 4294967296.0)
            return conv3_launch<1, 1, 8, To, size_t>(in, wp, bias, out, mask, li, lo, D, H, W, Ci, NT, act, slope, s);
        if (b.rows == 4) return go(std::integral_constant<int, 4>{});
    }
    go(std::integral_constant<int, 8>{});
}

void nn_conv3(const unsigned short *in, const void *wp, const float *bias, void *out, int out_f32,
              const unsigned short *mask, NNLayout li, NNLayout lo, int D, int H, int W, int Ci, int Co, int act, float slope, hipStream_t s)
{
    if (out_f32) conv3_dispatch(in, wp, bias, (float *)out, mask, li, lo, D, H, W, Ci, Co, act, slope, s);
    else conv3_dispatch(in, wp, bias, (unsigned short *)out, mask, li, lo, D, H, W, Ci, Co, act, slope, s);
}

void nn_conv3_two(const unsigned short *in, const void *wp, const float *bias, unsigned short *out, NNLayout lo, int D,
                  int H, int W, int Co, int act, float slope, hipStream_t s)
{
    conv3_dispatch<unsigned short, true>(in, wp, bias, out, nullptr, NNLayout{2, 0}, lo, D, H, W, 16, Co, act, slope, s);
}

// Runs of voxel tiles that the workspace has room for.  Its size is a result of the
// ABI, and callers keep workspaces: it counts three resident workgroups per CU (one
// with output tiles by four) and tiles of 16 x 4 x 2 voxels, whatever the kernel's
// own split, which never takes more.
static int dw_room(int D, int H, int W, int Ci, int Co)
{
    const int nt = Co / 16, ng = nt % 4 == 0 ? 4 : nt % 3 == 0 ? 3 : nt, per = (Ci / 16) * (nt / ng);
    const int ntiles = ((W + 15) / 16) * ((H + 3) / 4) * ((D + 1) / 2);
    const int want = std::max(1, std::min(ntiles, ((ng == 4 ? 1 : 3) * 256 + per - 1) / per));
    const int tpc = (ntiles + want - 1) / want;
    return (ntiles + tpc - 1) / tpc;
}

// weight-gradient work split: the (input chunk, output tile) pairs times runs
// of tpc voxel tiles, at most the 512 workgroups that are resident at once (two
// per CU): 171 runs of three pairs, 513 workgroups, took twice the time of 170
struct DwPlan {
    int npair, ntx, nty, ntiles, tpc, nchunk;
};

static DwPlan dw_plan(int D, int H, int W, int Ci, int Co)
{
    DwPlan p{};
    p.npair = (Ci / 16) * (Co / 16);
    p.ntx = (W + 15) / 16;
    p.nty = (H + 3) / 4;
    p.ntiles = p.ntx * p.nty * ((D + 3) / 4);
    const int want = std::max(1, std::min({512 / p.npair, p.ntiles, dw_room(D, H, W, Ci, Co)}));
    p.tpc = (p.ntiles + want - 1) / want;
    p.nchunk = (p.ntiles + p.tpc - 1) / p.tpc;
    return p;
}

size_t nn_dw_workspace_floats(int D, int H, int W, int Ci, int Co)
{
    return (size_t)dw_room(D, H, W, Ci, Co) * (27 * (size_t)Ci * Co + Co);
}

void nn_conv3_dw(const unsigned short *X, const unsigned short *dZ, float *partial, float *gw, float *gb, NNLayout lx,
                 NNLayout lz, int D, int H, int W, int Ci, int Co, hipStream_t s)
{
    const DwPlan p = dw_plan(D, H, W, Ci, Co);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(p.nchunk * p.npair), dim3(TPB), 0, s, X, dZ, partial, lx, lz, D, H, W, Ci, Co,
                           p.ntx, p.nty, p.ntiles, p.tpc);
    };
    if ((((uintptr_t)X | (uintptr_t)dZ) & 15) == 0) go(k_conv3_dw<true>);
    else go(k_conv3_dw<false>);
    const int nw = 27 * Ci * Co;
    auto sum = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3((nw + Co + 63) / 64), dim3(64 * waves), 0, s, partial, p.nchunk, nw, Co, gw, gb,
                           DwOperands{X, dZ, lx, lz, D, H, W, Ci, Co, p.ntx, p.nty, p.ntiles, p.tpc});
    };
    if (p.nchunk > 4 * SUM_LOADS) sum(k_sum_partials<16>, 16);
    else sum(k_sum_partials<4>, 4);
}

void nn_pool2(const unsigned short *in, unsigned short *out, int D, int H, int W, hipStream_t s)
{
    hipLaunchKernelGGL(k_pool2, dim3(nblk((size_t)D * H * W / 4)), dim3(TPB), 0, s, (const u4 *)in, (u4 *)out, D, H, W);
}

void nn_pool2_bwd(const unsigned short *gpool, unsigned short *g, const unsigned short *Y, float slope, int D, int H,
                  int W, hipStream_t s)
{
    hipLaunchKernelGGL(k_pool2_bwd, dim3(nblk((size_t)D * H * W * 2)), dim3(TPB), 0, s, (const u4 *)gpool, (u4 *)g,
                       (const u4 *)Y, slope, D, H, W);
}

void nn_up2(const unsigned short *a, unsigned short *out, int D, int H, int W, hipStream_t s)
{
    hipLaunchKernelGGL(k_up2, dim3(nblk((size_t)D * H * W * 2)), dim3(TPB), 0, s, (const u4 *)a, (u4 *)out, D, H, W);
}

void nn_up2_bwd(const unsigned short *g, unsigned short *ga, const unsigned short *Y, float slope, int D, int H, int W,
                hipStream_t s)
{
    hipLaunchKernelGGL(k_up2_bwd, dim3(nblk((size_t)D * H * W / 4)), dim3(TPB), 0, s, (const u4 *)g, (u4 *)ga,
                       (const u4 *)Y, slope, D, H, W);
}

void nn_head(const unsigned short *in, const float *w, const float *b, float *out, size_t P, int Ci, hipStream_t s)
{
    hipLaunchKernelGGL(k_head, dim3(nblk(P)), dim3(TPB), 0, s, in, w, b, out, P, Ci);
}

void nn_head_bwd(const unsigned short *in, const float *gout, const float *w, float slope, unsigned short *gin,
                 double *partials, int nparts, double *dst_dev, size_t P, hipStream_t s)
{
    hipLaunchKernelGGL(k_head_bwd_x, dim3(nblk(P * 2)), dim3(TPB), 0, s, gout, w, (const u4 *)in, slope, (u4 *)gin, P);
    // partials holds HEAD_NC rows of nparts values
    hipLaunchKernelGGL(k_head_bwd_w, dim3(nparts), dim3(TPB), 0, s, in, gout, P, partials);
    hipLaunchKernelGGL(k_finalize_rows, dim3(HEAD_NC), dim3(TPB), 0, s, partials, nparts, dst_dev);
}

void nn_mse(const float *pred, const float *label, size_t n, float inv, float *grad, double *partials, int nparts,
            hipStream_t s)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nparts), dim3(TPB), 0, s, pred, label, n, inv, grad, partials);
    };
    if ((((uintptr_t)pred | (uintptr_t)label | (uintptr_t)grad) & 15) == 0 && n % 4 == 0) go(k_mse<4>);
    else go(k_mse<1>);
}

void nn_adam(float *p, const float *g, float *m, float *v, size_t n, float lr, float b1, float b2, float eps, float c1,
             float c2, hipStream_t s)
{
    hipLaunchKernelGGL(k_adam, dim3(nblk(n)), dim3(TPB), 0, s, p, g, m, v, n, lr, b1, b2, eps, c1, c2);
}

void nn_pack_input(const float *a, const float *b, unsigned short *out, size_t P, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack_input, dim3(nblk(P)), dim3(TPB), 0, s, a, b, (u4 *)out, P);
}

void nn_pack_two(const float *a, const float *b, unsigned short *out, size_t P, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack_two, dim3(nblk(P)), dim3(TPB), 0, s, a, b, (unsigned *)out, P);
}

} // namespace clh
