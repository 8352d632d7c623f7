// Learned warm start: a 3D convolutional network that predicts the Newton
// increment of a time step from the state at its start (an extension of the
// paper's Newton iteration, Algorithm 1: the prediction is only a first
// iterate, taken when it lowers the residual).
//
// Network (channels-last, [crop][z][y][x][channel], zero padding per crop):
//     h_0 = relu(conv(f, W_in)),  a_k = relu(conv(h_k, W_a,k)),
//     h_k+1 = h_k + conv(a_k, W_b,k)  (k < K),  out = conv(h_K, W_out),
// 3x3x3 taps, 32 channels.  Activations and weights are bfloat16 (rounded to
// nearest, ties to even), products accumulate in FP32; the input (6 feature
// channels) and output (2 channels) layers are stored padded to 32 channels
// with zero weights, so every layer is the same 32 -> 32 kernel.
//
// Device design.  A convolution is an implicit GEMM: for each of the 27 taps
// a wavefront multiplies 16-voxel x 32-channel blocks of shifted inputs by
// the tap's 32 x 32 weight block on the matrix cores
// (v_mfma_f32_16x16x32_bf16); a workgroup walks the planes of a 16 x 16 column
// with the weights in registers and the input planes in an LDS ring.  The
// input gradient is the same kernel
// on mirrored taps with per-tap transposed weights.  The weight gradient is a
// GEMM over voxels on the same tiles, its operands read from LDS transposed;
// workgroup partials are summed in a fixed order.
// Training keeps FP32 master weights with Adam moments.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "r2p_impl.h"

namespace {

constexpr int CH = 32;                      // channels of every layer (padded)
constexpr int TAPS = 27;
constexpr int WLAYER = TAPS * CH * CH;      // weights of one padded layer
constexpr int CBS = 256;                    // reduction workgroups
constexpr int NIN = 6, NOUT = 2;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

__host__ __device__ inline u16 to_bf16(float f) {
    unsigned u;
    memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}
__host__ __device__ inline float from_bf16(u16 h) {
    unsigned u = (unsigned)h << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

struct Geo {
    int nx, ny, nz, nb;
    __host__ __device__ long V() const { return (long)nx * ny * nz * nb; }
};

struct ConvArgs {
    const u16 *x;         // [V][32] input
    Geo g;
    const u16 *w;         // [27][32 out][32 in]
    const float *bias;    // [32] or NULL
    const u16 *addend;    // [V][32] or NULL: added to the result
    const u16 *mask;      // [V][32] or NULL: result kept where mask > 0
    int relu, flip;       // flip: taps mirrored (input-gradient form)
    int swap;             // the weights' taps are [dy][dz][dx] in g's axes (see launch_conv)
    u16 *out;             // [V][32] bf16 result, or NULL
    float *outf;          // [V][32] fp32 result, or NULL
    float *out2;          // [V][2] fp32 result (channels 0 and 1), or NULL
};

// Weight-gradient tiles: TZ x TY x TX voxels of one crop, read with a
// one-voxel halo.
constexpr int TZ = 2, TY = 8, TX = 32;
constexpr int HZ = TZ + 2, HY = TY + 2, HX = TX + 2, HV = HZ * HY * HX;

struct TileAt {
    long cb;            // first voxel of the tile's crop
    int x0, y0, z0;
};
// (32-bit arithmetic: the tile count is checked against 2^31 at launch)
__device__ __forceinline__ TileAt tile_at(int tile, const Geo &g) {
    const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + TZ - 1) / TZ;
    int rr = tile;
    TileAt T;
    T.x0 = (rr % ntx) * TX;
    rr /= ntx;
    T.y0 = (rr % nty) * TY;
    rr /= nty;
    T.z0 = (rr % ntz) * TZ;
    rr /= ntz;
    T.cb = (long)rr * ((long)g.nx * g.ny * g.nz);
    return T;
}

// Place of a 16-byte chunk of a staged row: the four chunks of voxel v of the
// row are permuted by v, so that reads of one chunk of consecutive voxels, 64
// bytes apart, fall on different LDS banks.
__device__ __forceinline__ int chunk_at(int v, int part) { return v * 4 + (part ^ ((v >> 2) & 3)); }

// out[v, o] = epilogue(bias[o] + sum_t sum_i x[v + s off_t, i] w[t, o, i]),
// s = -1 with FLIP.  A workgroup takes a column of CY x CX voxels of one crop
// and walks a range of its planes (downwards with FLIP).  Every input plane,
// with a one-voxel halo that is zero outside the crop, is staged once in LDS
// (two buffers, the plane after next in registers, one barrier a plane) and
// adds to the three output planes it meets, which are held in registers.
// Wavefront q owns rows ROWS (q mod 4) .. of the planes and output channels
// 16 (q / 4) .. + 15; the 27 weight blocks of those channels stay in its
// registers, so a 16-byte LDS read a lane (16 voxels x 32 channels) feeds nine
// v_mfma_f32_16x16x32_bf16.  The weights are the first operand, so a lane ends
// up with four consecutive channels of one voxel and the epilogue works
// straight from the registers.  Every output receives its taps in the order
// t = 0 .. 26.
// What bounds it: the matrix cores (2M voxels: 53 us at the 2.09 PFLOP/s that
// back-to-back matrix instructions reach here, 91 us at the rate of a large
// library product), then each step's epilogue, which the two wavefronts of a
// SIMD reach together.  Measured over the ten layers of a forward pass at 2M
// voxels: 115 us a layer.  Tiles of 2 x 8 x 32 voxels whose weights and input
// both came from LDS read six fragments for eight matrix instructions and
// took 200 us; the same column walk with all 32 output channels in each of
// four wavefronts needs 440 registers, which the compiler shuffles, 170 us;
// every halo plane at full cost, 118 us.
// Grids of up to 8 (4) rows take columns of 8 (4) rows, two (one) a wavefront:
// 1,000 x 8 x 8 voxels 143 us a forward pass, 185 with 16 rows; 300 crops of
// 4 x 5 x 7 236 and 322.
constexpr int CX = 16, PX = CX + 2;              // output voxels of a plane's row, staged
constexpr int CWG = 512;                         // eight wavefronts

template <int V>
using Int = std::integral_constant<int, V>;

// OUT2: the output layer; only its two channels are computed and stored.  ROWS:
// output rows per wavefront.
template <bool FLIP, bool OUT2, int ROWS>
__global__ __launch_bounds__(CWG, 1) void k_conv(ConvArgs A, int zc) {
    constexpr int CY = 4 * ROWS, PY = CY + 2, PV = PY * PX;
    constexpr int PCH = (PV * 4 + CWG - 1) / CWG;    // 16-byte chunks of a plane per thread
    __shared__ __attribute__((aligned(16))) u16 buf[2][PV * CH];
    const Geo g = A.g;
    const int ntx = (g.nx + CX - 1) / CX, nty = (g.ny + CY - 1) / CY, nzc = (g.nz + zc - 1) / zc;
    int rest = xcd_block(blockIdx.x, gridDim.x);
    const int x0 = (rest % ntx) * CX;
    rest /= ntx;
    const int y0 = (rest % nty) * CY;
    rest /= nty;
    const int z0 = (rest % nzc) * zc, z1 = min(z0 + zc, g.nz);
    const long cb = (long)(rest / nzc) * ((long)g.nx * g.ny * g.nz);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, kg = lane >> 4;
    const int rowq = wave & 3, ch = 16 * (wave >> 2) + 4 * kg;     // rows; this lane's channels

    // this thread's chunks of an input plane: place in the plane (-1: outside
    // the crop, zero) and in LDS
    int at[PCH], to[PCH];
#pragma unroll
    for (int u = 0; u < PCH; u++) {
        int c = (int)threadIdx.x + u * CWG, v = c >> 2, hx = v % PX, hy = v / PX;
        int gx = x0 + hx - 1, gy = y0 + hy - 1;
        bool in = c < PV * 4 && gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny;
        at[u] = in ? (gy * g.nx + gx) * CH + 8 * (c & 3) : -1;
        to[u] = c < PV * 4 ? hy * PX * 4 + chunk_at(hx, c & 3) : -1;
    }
    auto fetch = [&](uint4 (&p)[PCH], int z) {
        const u16 *src = A.x + (cb + (long)min(max(z, 0), g.nz - 1) * g.ny * g.nx) * CH;
        const bool zin = z >= 0 && z < g.nz;
#pragma unroll
        for (int u = 0; u < PCH; u++) {
            uint4 v = *reinterpret_cast<const uint4 *>(src + max(at[u], 0));
            p[u] = zin && at[u] >= 0 ? v : uint4{0u, 0u, 0u, 0u};
        }
    };
    auto stage = [&](const uint4 (&p)[PCH], int b) {
        uint4 *dst = reinterpret_cast<uint4 *>(buf[b]);
#pragma unroll
        for (int u = 0; u < PCH; u++)
            if (to[u] >= 0) dst[to[u]] = p[u];
    };
    // step k reads input plane zin(k) and completes output plane zin(k) - s
    const int n = z1 - z0;
    auto zin = [&](int k) { return FLIP ? z1 - k : z0 - 1 + k; };
    uint4 pr[PCH], p0[PCH];
    fetch(p0, zin(0));
    fetch(pr, zin(1));
    bf16x8 wr[TAPS];
#pragma unroll
    for (int t = 0; t < TAPS; t++) {
        const int tw = A.swap ? 9 * (t / 3 % 3) + 3 * (t / 9) + t % 3 : t;
        wr[t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(
                                               A.w + (tw * CH + 16 * (wave >> 2) + i) * CH + 8 * kg));
    }
    float bz[4];
#pragma unroll
    for (int u = 0; u < 4; u++) bz[u] = A.bias ? A.bias[ch + u] : 0.f;
    stage(p0, 0);
    // this lane's place in a staged row, by the tap's x step
    int xo[3];
#pragma unroll
    for (int e = 0; e < 3; e++) xo[e] = chunk_at(i + (FLIP ? 2 - e : e), kg) * 8;
    const int xi = x0 + i, yb = y0 + rowq * ROWS;
    f32x4 acc[3][ROWS];                 // output planes zin + s, zin, zin - s
#pragma unroll
    for (int d = 0; d < 3; d++)
#pragma unroll
        for (int r = 0; r < ROWS; r++) acc[d][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    // step k; LO .. HI: the output planes of acc that its plane adds to
    auto step = [&](int k, auto lo, auto hi) {
        constexpr int LO = decltype(lo)::value, HI = decltype(hi)::value;
        __syncthreads();        // this step's plane is staged; the other buffer is not read any more
        if (k < n + 1) stage(pr, (k + 1) & 1);
        if (k < n) fetch(pr, zin(k + 2));
        const int zo = FLIP ? zin(k) + 1 : zin(k) - 1;
        const long vb = cb + ((long)zo * g.ny + yb) * g.nx + xi;
        uint2 ad[ROWS], mk[ROWS];
        auto rows_of = [&](uint2 (&v)[ROWS], const u16 *src) {
#pragma unroll
            for (int r = 0; r < ROWS; r++)
                v[r] = *reinterpret_cast<const uint2 *>(
                    src + (xi < g.nx && yb + r < g.ny ? vb + (long)r * g.nx : cb) * CH + ch);
        };
        if (!OUT2 && A.addend && k >= 2) rows_of(ad, A.addend);
        if (!OUT2 && A.mask && k >= 2) rows_of(mk, A.mask);
        if (!OUT2 || wave < 4) {
            // fragments in order of use (input row, x step), each requested
            // three before its use; input row yy meets output row yy - a at
            // tap row a (rows reversed with FLIP)
            const u16 *pl = buf[k & 1] + rowq * ROWS * PX * CH;
            constexpr int NF = 3 * (ROWS + 2);
            uint4 fb[4];
            auto frag = [&](int f) {
                const int yy = f / 3;
                fb[f & 3] = *reinterpret_cast<const uint4 *>(
                    pl + (FLIP ? ROWS + 1 - yy : yy) * PX * CH + xo[f % 3]);
            };
#pragma unroll
            for (int f = 0; f < 3; f++) frag(f);
#pragma unroll
            for (int f = 0; f < NF; f++) {
                if (f + 3 < NF) frag(f + 3);
                const int yy = f / 3, e = f % 3;
                const bf16x8 b = __builtin_bit_cast(bf16x8, fb[f & 3]);
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    const int y = yy - a;
                    if (y < 0 || y >= ROWS) continue;
#pragma unroll
                    for (int d = LO; d <= HI; d++)
                        acc[d][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            wr[9 * d + 3 * a + e], b, acc[d][y], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (k >= 2) {
#pragma unroll
            for (int r = 0; r < ROWS; r++) {
                if (xi >= g.nx || yb + r >= g.ny) continue;
                const long vo = vb + (long)r * g.nx;
                const f32x4 v = acc[2][FLIP ? ROWS - 1 - r : r];
                float val[4];
#pragma unroll
                for (int u = 0; u < 4; u++) val[u] = v[u] + bz[u];
                if (OUT2) {
                    if (ch == 0) {
                        A.out2[2 * vo] = val[0];
                        A.out2[2 * vo + 1] = val[1];
                    }
                    continue;
                }
                if (A.addend) {
                    const u16 *ah = reinterpret_cast<const u16 *>(&ad[r]);
#pragma unroll
                    for (int u = 0; u < 4; u++) val[u] += from_bf16(ah[u]);
                }
                if (A.mask) {
                    const u16 *mh = reinterpret_cast<const u16 *>(&mk[r]);
#pragma unroll
                    for (int u = 0; u < 4; u++) val[u] = from_bf16(mh[u]) > 0.f ? val[u] : 0.f;
                }
                if (A.relu) {
#pragma unroll
                    for (int u = 0; u < 4; u++) val[u] = val[u] > 0.f ? val[u] : 0.f;
                }
                if (A.out) {
                    // nearest even, as to_bf16 (v_cvt_pk_bf16_f32)
                    bf16x4 o = {(__bf16)val[0], (__bf16)val[1], (__bf16)val[2], (__bf16)val[3]};
                    *reinterpret_cast<bf16x4 *>(A.out + vo * CH + ch) = o;
                }
                if (A.outf)
                    *reinterpret_cast<float4 *>(A.outf + vo * CH + ch) =
                        make_float4(val[0], val[1], val[2], val[3]);
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; r++) {
            acc[2][r] = acc[1][r];
            acc[1][r] = acc[0][r];
            acc[0][r] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // the halo planes at the ends of the range meet one output plane each
    step(0, Int<0>(), Int<0>());
    for (int k = 1; k <= n; k++) step(k, Int<0>(), Int<2>());
    step(n + 1, Int<2>(), Int<2>());
}

// Weight and bias gradients of a layer: dW[t, o, i] = sum_v gy[v, o] x[v + off_t, i],
// db[o] = sum_v gy[v, o].  A GEMM with the voxels as its inner dimension: a
// persistent workgroup takes tiles of TZ x TY x TX voxels, stages gy and x
// (with its halo) in LDS as they lie in memory, and reads both operands
// transposed (ds_read_b64_tr_b16: four voxels of one channel per lane), so a
// tap is only another start address.  Wavefront 3 (dz + 1) + (dx + 1) owns the
// three taps dy = -1, 0, 1: as it walks the tile's input rows, each row of x is
// read once and multiplied with the three rows of gy it meets, which stay in
// registers.  The tenth wavefront multiplies gy with ones for the bias.  The
// sums stay in registers over all tiles of the workgroup: one partial block
// per workgroup, added in workgroup order by k_sum_parts.
// What bounds it: the staging of a tile and the matrix cores in turn (45 us at
// 460,800 voxels, where the products alone are 10 us at peak).  One launch
// column per tap that read gy and x 27 times and transposed them through
// 2-byte LDS stores took 228 us, and the bias sums a pass of their own, 121 us.
constexpr int DWT = 640;                        // ten wavefronts
constexpr int TV = TZ * TY * TX;                // voxels of a tile
constexpr int DXC = (HV * 4 + DWT - 1) / DWT;   // 16-byte chunks of x, of gy per thread
constexpr int DGC = (TV * 4 + DWT - 1) / DWT;
typedef short s16x4 __attribute__((ext_vector_type(4)));

// Voxels v .. v + 31 of a staged row as a matrix operand of the 16 channels of
// `half`: lane (i, kg) gets channel 16 half + i of voxels v + 8 kg .. + 7, by
// two transposing reads of four voxels each.  The lane's offsets within a row
// (tr_off) do not depend on the row.
__device__ __forceinline__ int tr_off(int v, int half, int j) {
    const int lane = threadIdx.x & 63, q = lane & 3;
    const int vl = v + 8 * (lane >> 4) + ((lane & 15) >> 2) + 4 * j;
    return chunk_at(vl, 2 * half + (q >> 1)) * 8 + 4 * (q & 1);
}
__device__ __forceinline__ bf16x8 ld_tr(const u16 *row, const int (&off)[2]) {
    uint4 r;
    s16x4 *h = reinterpret_cast<s16x4 *>(&r);
#pragma unroll
    for (int j = 0; j < 2; j++)
        h[j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4 *)(row + off[j]));
    return __builtin_bit_cast(bf16x8, r);
}

__global__ __launch_bounds__(DWT) void k_conv_dw(const u16 *gy, const u16 *x, Geo g, float *part,
                                                 float *bpart) {
    __shared__ __attribute__((aligned(16))) u16 xl[HV * CH], gl[TV * CH];
    const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + TZ - 1) / TZ;
    const int ntile = g.nb * ntz * nty * ntx;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, kg = lane >> 4;
    const int dz = wave / 3 - 1, dx = wave % 3 - 1;
    int xo[2][2], go[2][2];             // this lane's offsets in a row of x and of gy
#pragma unroll
    for (int u = 0; u < 4; u++) {
        xo[u >> 1][u & 1] = tr_off(1 + dx, u >> 1, u & 1);
        go[u >> 1][u & 1] = tr_off(0, u >> 1, u & 1);
    }
    uint4 xr[DXC], gr[DGC];
    auto fetch = [&](int tile) {
        const TileAt T = tile_at(tile, g);
        // the chunks' places are worked out for every tile: kept across the
        // tile loop they would take more registers than there are
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int u = 0; u < DXC; u++) {
            int c = tid + u * DWT, hv = c >> 2;
            int gx = T.x0 + hv % HX - 1, gyy = T.y0 + (hv / HX) % HY - 1, gz = T.z0 + hv / (HX * HY) - 1;
            bool in = c < HV * 4 && gx >= 0 && gx < g.nx && gyy >= 0 && gyy < g.ny && gz >= 0 && gz < g.nz;
            long at = in ? (T.cb + ((long)gz * g.ny + gyy) * g.nx + gx) * CH + 8 * (c & 3) : 0;
            uint4 v = *reinterpret_cast<const uint4 *>(x + at);
            xr[u] = in ? v : uint4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < DGC; u++) {
            int c = tid + u * DWT, tv = c >> 2;
            int gx = T.x0 + tv % TX, gyy = T.y0 + (tv / TX) % TY, gz = T.z0 + tv / (TX * TY);
            bool in = c < TV * 4 && gx < g.nx && gyy < g.ny && gz < g.nz;
            long at = in ? (T.cb + ((long)gz * g.ny + gyy) * g.nx + gx) * CH + 8 * (c & 3) : 0;
            uint4 v = *reinterpret_cast<const uint4 *>(gy + at);
            gr[u] = in ? v : uint4{0u, 0u, 0u, 0u};
        }
    };
    f32x4 acc[3][2][2];
#pragma unroll
    for (int a = 0; a < 12; a++) acc[a / 4][(a >> 1) & 1][a & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
    if ((int)blockIdx.x < ntile) fetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        __syncthreads();                // the previous tile's reads are done
#pragma unroll
        for (int u = 0; u < DXC; u++) {
            int c = (int)threadIdx.x + u * DWT;
            int hv = c >> 2, v = hv % HX;
            if (c < HV * 4) reinterpret_cast<uint4 *>(xl)[(hv - v) * 4 + chunk_at(v, c & 3)] = xr[u];
        }
#pragma unroll
        for (int u = 0; u < DGC; u++) {
            int c = (int)threadIdx.x + u * DWT;
            int tv = c >> 2, v = tv % TX;
            if (c < TV * 4) reinterpret_cast<uint4 *>(gl)[(tv - v) * 4 + chunk_at(v, c & 3)] = gr[u];
        }
        __syncthreads();
        if (tile + (int)gridDim.x < ntile) fetch(tile + gridDim.x);
        if (wave < 9) {
            for (int z = 0; z < TZ; z++) {
                // rows of gy by row mod 3, of x by row mod 2; each is requested
                // one input row before its use
                bf16x8 ga[3][2], xb[2][2];
                auto row_x = [&](int yy) {
#pragma unroll
                    for (int n = 0; n < 2; n++)
                        xb[yy & 1][n] = ld_tr(xl + ((z + 1 + dz) * HY + yy) * HX * CH, xo[n]);
                };
                auto row_g = [&](int y) {
#pragma unroll
                    for (int m = 0; m < 2; m++)
                        ga[y % 3][m] = ld_tr(gl + (z * TY + y) * TX * CH, go[m]);
                };
                row_x(0);
                row_g(0);
#pragma unroll
                for (int yy = 0; yy < HY; yy++) {
                    if (yy + 1 < HY) row_x(yy + 1);
                    // input row yy - 1 of the tile meets gy row yy - 1 - dy, the
                    // oldest first: its registers take row yy + 1
#pragma unroll
                    for (int a = 2; a >= 0; a--) {
                        const int y = yy - a;
                        if (y < 0 || y >= TY) continue;
#pragma unroll
                        for (int m = 0; m < 2; m++)
#pragma unroll
                            for (int n = 0; n < 2; n++)
                                acc[a][m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    ga[y % 3][m], xb[yy & 1][n], acc[a][m][n], 0, 0, 0);
                    }
                    if (yy + 1 < TY) row_g(yy + 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            const bf16x8 one = {(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f,
                                (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f};
            for (int r = 0; r < TZ * TY; r++)
#pragma unroll
                for (int m = 0; m < 2; m++)
                    acc[0][m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        ld_tr(gl + r * TX * CH, go[m]), one, acc[0][m][0], 0, 0, 0);
        }
    }
    if (wave < 9) {
        float *out = part + (long)blockIdx.x * TAPS * CH * CH;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            int t = 9 * (dz + 1) + 3 * a + dx + 1;
#pragma unroll
            for (int m = 0; m < 2; m++)
#pragma unroll
                for (int n = 0; n < 2; n++)
#pragma unroll
                    for (int r = 0; r < 4; r++)
                        out[(t * CH + 16 * m + 4 * kg + r) * CH + 16 * n + i] = acc[a][m][n][r];
        }
    } else if (i == 0) {
#pragma unroll
        for (int m = 0; m < 2; m++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                bpart[(long)blockIdx.x * CH + 16 * m + 4 * kg + r] = acc[0][m][0][r];
    }
}

// dst[k] = sum over nparts of part[p * n + k], k < n (n a multiple of 32): a
// workgroup takes 32 values, eight groups of lanes a contiguous eighth of the
// parts each (eight loads in flight), then the eighths in order: 9 us for 256
// parts of a layer.  One thread per value walking every part was a chain of
// 225 loads, 80 us.
__global__ __launch_bounds__(CBS) void k_sum_parts(const float *part, int nparts, long n,
                                                   float *dst) {
    __shared__ float red[8][32];
    const int c = threadIdx.x & 31, q = threadIdx.x >> 5;
    const long k = (long)blockIdx.x * 32 + c;
    const int per = (nparts + 7) / 8, p1 = min(nparts, (q + 1) * per);
    float s = 0.f;
    int p = q * per;
    for (; p + 8 <= p1; p += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = part[(long)(p + u) * n + k];
#pragma unroll
        for (int u = 0; u < 8; u++) s += v[u];
    }
    for (; p < p1; p++) s += part[(long)p * n + k];
    red[q][c] = s;
    __syncthreads();
    if (q == 0) {
        float t = red[0][c];
        for (int u = 1; u < 8; u++) t += red[u][c];
        dst[k] = t;
    }
}

// Mean squared error over voxels and the NOUT output channels: gradient
// (bf16, padded to 32 channels) and per-workgroup partial loss sums.
__global__ __launch_bounds__(CBS) void k_mse(const float *out, const float *tgt, long V, float scale,
                                             u16 *gy, double *part) {
    __shared__ double red[CBS];
    long v = blockIdx.x * (long)CBS + threadIdx.x;
    double s = 0.0;
    if (v < V) {
        float d0 = out[NOUT * v] - tgt[NOUT * v], d1 = out[NOUT * v + 1] - tgt[NOUT * v + 1];
        s += (double)d0 * d0;
        s += (double)d1 * d1;
        unsigned g = (unsigned)to_bf16(2.f * d0 * scale) | ((unsigned)to_bf16(2.f * d1 * scale) << 16);
        uint4 *row = reinterpret_cast<uint4 *>(gy + v * CH);
        row[0] = uint4{g, 0u, 0u, 0u};
        row[1] = row[2] = row[3] = uint4{0u, 0u, 0u, 0u};
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = CBS / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Adam on the padded FP32 master weights; then bf16 copies in the forward
// layout [t][o][i] and the input-gradient layout [t][i][o].
__global__ void k_adam(long n, float *p, const float *g, float *m, float *vv, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    long k = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (k >= n) return;
    float gk = g[k];
    float mk = b1 * m[k] + (1.f - b1) * gk;
    float vk = b2 * vv[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    vv[k] = vk;
    p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

__global__ void k_weights_bf16(long nl, const float *w, u16 *wf, u16 *wt) {
    long k = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (k >= nl * WLAYER) return;
    long l = k / WLAYER;
    int r = (int)(k % WLAYER);
    int t = r / (CH * CH), o = (r / CH) % CH, i = r % CH;
    u16 h = to_bf16(w[k]);
    wf[k] = h;
    wt[l * WLAYER + (t * CH + i) * CH + o] = h;
}

// -------------------------------------------------------------- features
// Per cell of a state x at the start of a step of length dt (channels 0..5;
// 6..31 zero): scaled pressure, water saturation, scaled ln kh, scaled
// porosity, a well source term, ln dt.  The source of a perforated cell is
// log(1 + V) with V the pore-volume fraction its well could move in the
// step: the injected volume per perforation for a rate injector, the
// drawdown-driven volume W_i dt (p - p_bhp)^+ / PV for a BHP producer; signs
// mark injection (+) and production (-).
__global__ void k_features(int n, const double *x, double dt, const double *kx, const double *phi,
                           const int *cell_perf, const int *perf_well, const double *perf_wi,
                           const int *w_ptr, const int *w_kind, const int *w_ctrl,
                           const double *w_target, double vol, double alpha, u16 *feat) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    float f[CH];
    for (int k = 0; k < CH; k++) f[k] = 0.f;
    double p = x[2 * c], s = x[2 * c + 1];
    double pv = phi[c] * vol / alpha;
    f[0] = (float)((p - 4800.0) / 1000.0);
    f[1] = (float)s;
    f[2] = (float)((log(kx[c]) - 4.6) / 2.0);
    f[3] = (float)((phi[c] - 0.2) / 0.1);
    int pf = cell_perf[c];
    if (pf >= 0) {
        int w = perf_well[pf];
        int np = w_ptr[w + 1] - w_ptr[w];
        double q;
        if (w_ctrl[w] != R2P_BHP) q = fabs(w_target[w]) / np * dt / pv;
        else q = perf_wi[pf] * dt * fmax(fabs(p - w_target[w]), 0.0) / pv / 1000.0;
        f[4] = (float)((w_kind[w] == R2P_INJECTOR ? 1.0 : -1.0) * log1p(q));
    }
    f[5] = (float)log(dt);
    for (int k = 0; k < CH; k++) feat[(long)c * CH + k] = to_bf16(f[k]);
}

// Training target of a step x_old -> x_new: (dp / P_SCALE, ds_w / S_SCALE),
// so both channels are of order one.
constexpr double P_SCALE = 100.0, S_SCALE = 0.1;
__global__ void k_targets(int n, const double *xo, const double *xn, float *tgt) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    tgt[2 * c] = (float)((xn[2 * c] - xo[2 * c]) / P_SCALE);
    tgt[2 * c + 1] = (float)((xn[2 * c + 1] - xo[2 * c + 1]) / S_SCALE);
}

// First Newton iterate from a prediction: p += P_SCALE dp, s_w += S_SCALE ds
// (clipped to [0, 1]); a rate well's bottom-hole pressure moves by the mean
// pressure change of its perforated cells, a BHP well's stays at its target.
__global__ void k_apply_guess(int n, int nw, const double *x, const float *pred, const int *w_ptr,
                              const int *perf_cell, double *xg) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n) {
        xg[2 * c] = x[2 * c] + P_SCALE * (double)pred[2 * c];
        double s = x[2 * c + 1] + S_SCALE * (double)pred[2 * c + 1];
        xg[2 * c + 1] = s < 0.0 ? 0.0 : (s > 1.0 ? 1.0 : s);
    } else if (c < n + nw) {
        int w = c - n;
        double d = 0.0;
        for (int k = w_ptr[w]; k < w_ptr[w + 1]; k++) d += P_SCALE * (double)pred[2 * perf_cell[k]];
        int np = w_ptr[w + 1] - w_ptr[w];
        xg[2 * c] = x[2 * c] + (np > 0 ? d / np : 0.0);
        xg[2 * c + 1] = x[2 * c + 1];
    }
}

// Workgroups of a persistent tile kernel: one per CU (the staged tiles take
// most of the LDS), no more than tiles; -1 when the tile count overflows.
int tile_workgroups(const Geo &g) {
    long tiles = (long)g.nb * ((g.nz + TZ - 1) / TZ) * ((g.ny + TY - 1) / TY) * ((g.nx + TX - 1) / TX);
    if (tiles >= (1L << 31)) { r2p_set_error("convolution grid too large"); return -1; }
    return std::max(1, (int)std::min<long>(tiles, r2p_cu_count()));
}

// Planes per workgroup of k_conv.  A workgroup's time is its planes plus about
// two for the weights and the halo planes, and CUs take workgroups in rounds:
// the split of the columns' planes with the shortest rounds.
int conv_planes(const Geo &g, long columns, int cus) {
    long best = 0;
    int zc = g.nz;
    for (int c = 1; c <= g.nz; c++) {
        int p = (g.nz + c - 1) / c;
        long wgs = columns * ((g.nz + p - 1) / p);
        long cost = (wgs + cus - 1) / cus * (p + 2);
        if (best == 0 || cost < best) { best = cost; zc = p; }
        if (wgs >= 8L * cus) break;      // full rounds: a finer split only adds to each
    }
    return zc;
}

template <int ROWS>
int launch_conv_rows(const ConvArgs &A, hipStream_t s) {
    const Geo &g = A.g;
    constexpr int CY = 4 * ROWS;
    long columns = (long)g.nb * ((g.ny + CY - 1) / CY) * ((g.nx + CX - 1) / CX);
    int zc = conv_planes(g, columns, std::max(1, r2p_cu_count()));
    long wgs = columns * ((g.nz + zc - 1) / zc);
    if (wgs >= (1L << 31)) { r2p_set_error("convolution grid too large"); return R2P_EINVAL; }
    if (A.out2) k_conv<false, true, ROWS><<<(int)wgs, CWG, 0, s>>>(A, zc);
    else if (A.flip) k_conv<true, false, ROWS><<<(int)wgs, CWG, 0, s>>>(A, zc);
    else k_conv<false, false, ROWS><<<(int)wgs, CWG, 0, s>>>(A, zc);
    R2P_LAUNCH();
    return 0;
}

// A cross-section (ny = 1) is laid out like one plane of nz rows, so it is taken
// as that, with the taps of the two axes exchanged: the taps with dy = 0, the
// only ones that meet a voxel, keep their order.  (50 x 1 x 5,000 voxels: 439 us
// a forward pass, 1,755 as 50 planes of one row.)
int launch_conv(const ConvArgs &A0, hipStream_t s) {
    ConvArgs A = A0;
    A.swap = A.g.ny == 1 && A.g.nz > 1;
    if (A.swap) std::swap(A.g.ny, A.g.nz);
    if (A.g.ny <= 4) return launch_conv_rows<1>(A, s);
    if (A.g.ny <= 8) return launch_conv_rows<2>(A, s);
    return launch_conv_rows<4>(A, s);
}

}  // namespace

// ----------------------------------------------------------------- handle
struct r2p_cnn {
    int K = 4;                  // residual blocks
    int L = 0;                  // layers = 2K + 2
    DBuf<float> w, gw, mw, vw;  // padded FP32 master weights, gradients, Adam moments
    DBuf<float> b, gb, mb, vb;  // biases [L][32]
    DBuf<u16> wf, wt;           // bf16 weights: forward and input-gradient layouts
    long step = 0;
    // activations of the last forward pass ([V][32] each) and gradients
    std::vector<DBuf<u16>> act; // h0, a0, h1, a1, h2, ..., h_K
    DBuf<float> out2;           // [V][2]: the output of a training pass
    DBuf<u16> g0, g1, g2;       // gradient work tensors
    DBuf<float> part, bpart;
    DBuf<double> lpart;
    DBuf<float> pred;
    DBuf<u16> feat, fcopy;
    HostPinned pin;
};

namespace {

int ensure_acts(r2p_cnn *C, long V) {
    C->act.resize(2 * C->K + 1);
    for (auto &a : C->act) R2P_TRY(a.ensure((size_t)V * CH));
    return 0;
}

// The features where the kernels can read 16 bytes at a time: the caller's
// tensor, or a copy when that is not 16-byte aligned.
int aligned_features(r2p_cnn *C, const u16 *&feat, long V, hipStream_t s) {
    if (((uintptr_t)feat & 15) == 0) return 0;
    R2P_TRY(C->fcopy.ensure((size_t)V * CH));
    R2P_HIP(hipMemcpyAsync(C->fcopy.p, feat, sizeof(u16) * V * CH, hipMemcpyDeviceToDevice, s));
    feat = C->fcopy.p;
    return 0;
}

// Layer l: weights at wf + l * WLAYER, bias at b + l * 32.  Activation
// slots: act[0] = h0, then a_k at 1 + 2k, h_{k+1} at 2 + 2k; out: [V][2].
int forward_impl(r2p_cnn *C, const u16 *feat, Geo g, float *out, hipStream_t s) {
    ConvArgs A{};
    A.g = g;
    A.x = feat; A.w = C->wf.p; A.bias = C->b.p; A.relu = 1; A.out = C->act[0].p;
    R2P_TRY(launch_conv(A, s));
    for (int k = 0; k < C->K; k++) {
        int la = 1 + 2 * k, lb = 2 + 2 * k;
        ConvArgs Aa{};
        Aa.g = g;
        Aa.x = C->act[2 * k].p; Aa.w = C->wf.p + (long)la * WLAYER; Aa.bias = C->b.p + la * CH;
        Aa.relu = 1; Aa.out = C->act[1 + 2 * k].p;
        R2P_TRY(launch_conv(Aa, s));
        ConvArgs Ab{};
        Ab.g = g;
        Ab.x = C->act[1 + 2 * k].p; Ab.w = C->wf.p + (long)lb * WLAYER; Ab.bias = C->b.p + lb * CH;
        Ab.addend = C->act[2 * k].p; Ab.out = C->act[2 + 2 * k].p;
        R2P_TRY(launch_conv(Ab, s));
    }
    int lo = C->L - 1;
    ConvArgs Ao{};
    Ao.g = g;
    Ao.x = C->act[2 * C->K].p; Ao.w = C->wf.p + (long)lo * WLAYER; Ao.bias = C->b.p + lo * CH;
    Ao.out2 = out;
    return launch_conv(Ao, s);
}

// Weight and bias gradients of one layer into dw ([27][32][32]) and db ([32]);
// part, bpart: workspace.
int conv_dw(const u16 *gy, const u16 *x, Geo g, float *dw, float *db, DBuf<float> &part,
            DBuf<float> &bpart, hipStream_t s) {
    int nwg = tile_workgroups(g);
    if (nwg < 0) return R2P_EINVAL;
    R2P_TRY(part.ensure((size_t)nwg * WLAYER));
    R2P_TRY(bpart.ensure((size_t)nwg * CH));
    k_conv_dw<<<nwg, DWT, 0, s>>>(gy, x, g, part.p, bpart.p);
    R2P_LAUNCH();
    k_sum_parts<<<WLAYER / 32, CBS, 0, s>>>(part.p, nwg, WLAYER, dw);
    R2P_LAUNCH();
    k_sum_parts<<<1, CBS, 0, s>>>(bpart.p, nwg, CH, db);
    R2P_LAUNCH();
    return 0;
}

int weight_grad(r2p_cnn *C, const u16 *gy, const u16 *x, Geo g, int layer, hipStream_t s) {
    return conv_dw(gy, x, g, C->gw.p + (long)layer * WLAYER, C->gb.p + layer * CH, C->part, C->bpart,
                   s);
}

// Input gradient of layer l applied to gy, with an optional mask and addend.
int input_grad(r2p_cnn *C, const u16 *gy, Geo g, int layer, const u16 *mask, const u16 *addend,
               u16 *out, hipStream_t s) {
    ConvArgs A{};
    A.g = g;
    A.x = gy; A.w = C->wt.p + (long)layer * WLAYER; A.flip = 1;
    A.mask = mask; A.addend = addend; A.out = out;
    return launch_conv(A, s);
}

int refresh_bf16(r2p_cnn *C, hipStream_t s) {
    long n = (long)C->L * WLAYER;
    k_weights_bf16<<<r2p_blocks(n, 256), 256, 0, s>>>(C->L, C->w.p, C->wf.p, C->wt.p);
    R2P_LAUNCH();
    return 0;
}

Geo make_geo(int nb, int nz, int ny, int nx) { return Geo{nx, ny, nz, nb}; }

int check_geo(int nb, int nz, int ny, int nx) {
    if (nb < 1 || nz < 1 || ny < 1 || nx < 1 || (long)nb * nz * ny * nx > (1L << 31) / CH) {
        r2p_set_error("invalid network input shape");
        return R2P_EINVAL;
    }
    return 0;
}

// Compact parameter order: per layer W[t][cout][cin] then b[cout], with
// (cin, cout) = (6, 32) for the input layer, (32, 32) inside, (32, 2) last.
void layer_dims(const r2p_cnn *C, int l, int &cin, int &cout) {
    cin = l == 0 ? NIN : CH;
    cout = l == C->L - 1 ? NOUT : CH;
}

}  // namespace

extern "C" int r2p_cnn_param_count(int blocks, long *n_host) {
    if (blocks < 1 || blocks > 16 || !n_host) { r2p_set_error("invalid arguments"); return R2P_EINVAL; }
    *n_host = (long)TAPS * CH * NIN + CH + (long)blocks * 2 * (TAPS * CH * CH + CH) + TAPS * NOUT * CH + NOUT;
    return 0;
}

extern "C" int r2p_cnn_create(int blocks, r2p_cnn **out) {
    if (!out || blocks < 1 || blocks > 16) { r2p_set_error("invalid arguments"); return R2P_EINVAL; }
    r2p_cnn *C = new r2p_cnn();
    C->K = blocks;
    C->L = 2 * blocks + 2;
    long nw = (long)C->L * WLAYER, nb = (long)C->L * CH;
    int rc = 0;
    if ((rc = C->w.ensure(nw)) || (rc = C->gw.ensure(nw)) || (rc = C->mw.ensure(nw)) ||
        (rc = C->vw.ensure(nw)) || (rc = C->b.ensure(nb)) || (rc = C->gb.ensure(nb)) ||
        (rc = C->mb.ensure(nb)) || (rc = C->vb.ensure(nb)) || (rc = C->wf.ensure(nw)) ||
        (rc = C->wt.ensure(nw)) || (rc = C->pin.ensure(1 << 16))) {
        delete C;
        return rc;
    }
    hipMemset(C->w.p, 0, sizeof(float) * nw);
    hipMemset(C->b.p, 0, sizeof(float) * nb);
    hipMemset(C->mw.p, 0, sizeof(float) * nw);
    hipMemset(C->vw.p, 0, sizeof(float) * nw);
    hipMemset(C->mb.p, 0, sizeof(float) * nb);
    hipMemset(C->vb.p, 0, sizeof(float) * nb);
    hipMemset(C->gw.p, 0, sizeof(float) * nw);
    hipMemset(C->gb.p, 0, sizeof(float) * nb);
    if (refresh_bf16(C, nullptr)) { delete C; return R2P_EHIP; }
    if (hipDeviceSynchronize() != hipSuccess) { delete C; r2p_set_error("HIP error"); return R2P_EHIP; }
    *out = C;
    return 0;
}

extern "C" int r2p_cnn_destroy(r2p_cnn *C) {
    delete C;
    return 0;
}

extern "C" int r2p_cnn_set_params(r2p_cnn *C, const float *theta) {
    if (!C || !theta) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    std::vector<float> w((size_t)C->L * WLAYER, 0.f), b((size_t)C->L * CH, 0.f);
    long o = 0;
    for (int l = 0; l < C->L; l++) {
        int cin, cout;
        layer_dims(C, l, cin, cout);
        for (int t = 0; t < TAPS; t++)
            for (int co = 0; co < cout; co++)
                for (int ci = 0; ci < cin; ci++) w[(size_t)l * WLAYER + (t * CH + co) * CH + ci] = theta[o++];
        for (int co = 0; co < cout; co++) b[(size_t)l * CH + co] = theta[o++];
    }
    R2P_HIP(hipMemcpy(C->w.p, w.data(), sizeof(float) * w.size(), hipMemcpyHostToDevice));
    R2P_HIP(hipMemcpy(C->b.p, b.data(), sizeof(float) * b.size(), hipMemcpyHostToDevice));
    R2P_HIP(hipMemset(C->mw.p, 0, sizeof(float) * w.size()));
    R2P_HIP(hipMemset(C->vw.p, 0, sizeof(float) * w.size()));
    R2P_HIP(hipMemset(C->mb.p, 0, sizeof(float) * b.size()));
    R2P_HIP(hipMemset(C->vb.p, 0, sizeof(float) * b.size()));
    C->step = 0;
    R2P_TRY(refresh_bf16(C, nullptr));
    R2P_HIP(hipDeviceSynchronize());
    return 0;
}

static int pull_compact(r2p_cnn *C, const float *wdev, const float *bdev, float *theta) {
    std::vector<float> w((size_t)C->L * WLAYER), b((size_t)C->L * CH);
    R2P_HIP(hipDeviceSynchronize());
    R2P_HIP(hipMemcpy(w.data(), wdev, sizeof(float) * w.size(), hipMemcpyDeviceToHost));
    R2P_HIP(hipMemcpy(b.data(), bdev, sizeof(float) * b.size(), hipMemcpyDeviceToHost));
    long o = 0;
    for (int l = 0; l < C->L; l++) {
        int cin, cout;
        layer_dims(C, l, cin, cout);
        for (int t = 0; t < TAPS; t++)
            for (int co = 0; co < cout; co++)
                for (int ci = 0; ci < cin; ci++) theta[o++] = w[(size_t)l * WLAYER + (t * CH + co) * CH + ci];
        for (int co = 0; co < cout; co++) theta[o++] = b[(size_t)l * CH + co];
    }
    return 0;
}

extern "C" int r2p_cnn_get_params(r2p_cnn *C, float *theta) {
    if (!C || !theta) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    return pull_compact(C, C->w.p, C->b.p, theta);
}

extern "C" int r2p_cnn_get_grads(r2p_cnn *C, float *grad) {
    if (!C || !grad) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    return pull_compact(C, C->gw.p, C->gb.p, grad);
}

extern "C" int r2p_cnn_forward(r2p_cnn *C, const uint16_t *feat, int nb, int nz, int ny, int nx,
                               float *out, void *stream) {
    if (!C || !feat || !out) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    R2P_TRY(check_geo(nb, nz, ny, nx));
    hipStream_t s = (hipStream_t)stream;
    Geo g = make_geo(nb, nz, ny, nx);
    R2P_TRY(ensure_acts(C, g.V()));
    R2P_TRY(aligned_features(C, feat, g.V(), s));
    return forward_impl(C, feat, g, out, s);
}

extern "C" int r2p_cnn_backward(r2p_cnn *C, const uint16_t *feat, const float *target, int nb,
                                int nz, int ny, int nx, double *loss_host, void *stream) {
    if (!C || !feat || !target) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    R2P_TRY(check_geo(nb, nz, ny, nx));
    hipStream_t s = (hipStream_t)stream;
    Geo g = make_geo(nb, nz, ny, nx);
    long V = g.V();
    R2P_TRY(ensure_acts(C, V));
    R2P_TRY(C->out2.ensure(2 * (size_t)V));
    for (DBuf<u16> *t : {&C->g0, &C->g1, &C->g2}) R2P_TRY(t->ensure((size_t)V * CH));
    R2P_TRY(aligned_features(C, feat, V, s));
    R2P_TRY(forward_impl(C, feat, g, C->out2.p, s));
    int nbl = r2p_blocks(V, CBS);
    R2P_TRY(C->lpart.ensure(nbl));
    k_mse<<<nbl, CBS, 0, s>>>(C->out2.p, target, V, 1.0f / (float)(V * NOUT), C->g0.p, C->lpart.p);
    R2P_LAUNCH();
    // output layer
    int lo = C->L - 1, K = C->K;
    R2P_TRY(weight_grad(C, C->g0.p, C->act[2 * K].p, g, lo, s));
    R2P_TRY(input_grad(C, C->g0.p, g, lo, nullptr, nullptr, C->g1.p, s));   // gh
    u16 *gh = C->g1.p, *ga = C->g2.p, *spare = C->g0.p;
    for (int k = K - 1; k >= 0; k--) {
        int la = 1 + 2 * k, lb = 2 + 2 * k;
        const u16 *a = C->act[1 + 2 * k].p, *h = C->act[2 * k].p;
        R2P_TRY(weight_grad(C, gh, a, g, lb, s));
        R2P_TRY(input_grad(C, gh, g, lb, a, nullptr, ga, s));               // ga = (W_b^T gh) (a > 0)
        R2P_TRY(weight_grad(C, ga, h, g, la, s));
        // gh' = gh + W_a^T ga; the input layer needs it only where h0 > 0
        R2P_TRY(input_grad(C, ga, g, la, k == 0 ? h : nullptr, gh, spare, s));
        std::swap(gh, spare);
    }
    R2P_TRY(weight_grad(C, gh, feat, g, 0, s));
    if (loss_host) {
        std::vector<double> lp(nbl);
        R2P_HIP(hipStreamSynchronize(s));
        R2P_HIP(hipMemcpy(lp.data(), C->lpart.p, sizeof(double) * nbl, hipMemcpyDeviceToHost));
        double t = 0.0;
        for (int i = 0; i < nbl; i++) t += lp[i];
        *loss_host = t / (double)(V * NOUT);
    }
    return 0;
}

extern "C" int r2p_cnn_sgd_step(r2p_cnn *C, float lr, void *stream) {
    if (!C || !(lr > 0.f)) { r2p_set_error("invalid arguments"); return R2P_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    C->step++;
    float c1 = 1.f - powf(b1, (float)C->step), c2 = 1.f - powf(b2, (float)C->step);
    long nw = (long)C->L * WLAYER, nb = (long)C->L * CH;
    k_adam<<<r2p_blocks(nw, 256), 256, 0, s>>>(nw, C->w.p, C->gw.p, C->mw.p, C->vw.p, lr, b1, b2,
                                               eps, c1, c2);
    R2P_LAUNCH();
    k_adam<<<r2p_blocks(nb, 256), 256, 0, s>>>(nb, C->b.p, C->gb.p, C->mb.p, C->vb.p, lr, b1, b2,
                                               eps, c1, c2);
    R2P_LAUNCH();
    return refresh_bf16(C, s);
}

extern "C" int r2p_cnn_conv(const uint16_t *x, int nb, int nz, int ny, int nx, const uint16_t *w,
                            const float *bias, const uint16_t *addend, const uint16_t *mask,
                            int relu, int flip, uint16_t *out, float *outf, void *stream) {
    if (!x || !w || (!out && !outf)) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    R2P_TRY(check_geo(nb, nz, ny, nx));
    ConvArgs A{};
    A.x = x; A.g = make_geo(nb, nz, ny, nx); A.w = w; A.bias = bias; A.addend = addend;
    A.mask = mask; A.relu = relu; A.flip = flip; A.out = out; A.outf = outf;
    return launch_conv(A, (hipStream_t)stream);
}

extern "C" int r2p_cnn_conv_dw(const uint16_t *gy, const uint16_t *x, int nb, int nz, int ny,
                               int nx, float *dw, float *db, void *stream) {
    if (!gy || !x || !dw || !db) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    R2P_TRY(check_geo(nb, nz, ny, nx));
    hipStream_t s = (hipStream_t)stream;
    Geo g = make_geo(nb, nz, ny, nx);
    DBuf<float> part, bpart;
    R2P_TRY(conv_dw(gy, x, g, dw, db, part, bpart, s));
    R2P_HIP(hipStreamSynchronize(s));
    return 0;
}

extern "C" int r2p_cnn_features(r2p_model *m, const double *x, double dt, uint16_t *feat,
                                void *stream) {
    if (!m || !x || !feat || !(dt > 0)) { r2p_set_error("invalid arguments"); return R2P_EINVAL; }
    const Phys &ph = m->ph;
    k_features<<<r2p_blocks(ph.n, 256), 256, 0, (hipStream_t)stream>>>(
        ph.n, x, dt, m->kx.p, m->phi.p, m->cell_perf.p, m->perf_well.p, m->perf_wi.p, m->w_ptr.p,
        m->w_kind.p, m->w_ctrl.p, m->w_target.p, ph.dx * ph.dy * ph.dz, ph.alpha, feat);
    R2P_LAUNCH();
    return 0;
}

extern "C" int r2p_cnn_targets(r2p_model *m, const double *x_old, const double *x_new,
                               float *target, void *stream) {
    if (!m || !x_old || !x_new || !target) { r2p_set_error("NULL argument"); return R2P_EINVAL; }
    k_targets<<<r2p_blocks(m->ph.n, 256), 256, 0, (hipStream_t)stream>>>(m->ph.n, x_old, x_new,
                                                                          target);
    R2P_LAUNCH();
    return 0;
}

extern "C" int r2p_cnn_warm_start(r2p_model *m, r2p_cnn *C, const double *x, double dt,
                                  double *x_guess, void *stream) {
    if (!m || !C || !x || !x_guess || !(dt > 0)) { r2p_set_error("invalid arguments"); return R2P_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    const Phys &ph = m->ph;
    R2P_TRY(C->feat.ensure((size_t)ph.n * CH));
    R2P_TRY(C->pred.ensure(2L * ph.n));
    R2P_TRY(r2p_cnn_features(m, x, dt, C->feat.p, stream));
    R2P_TRY(r2p_cnn_forward(C, C->feat.p, 1, ph.nz, ph.ny, ph.nx, C->pred.p, stream));
    k_apply_guess<<<r2p_blocks(ph.n + ph.nw, 256), 256, 0, s>>>(ph.n, ph.nw, x, C->pred.p,
                                                                 m->w_ptr.p, m->perf_cell.p, x_guess);
    R2P_LAUNCH();
    return 0;
}
