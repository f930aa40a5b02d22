// Layers of the learned surrogate (a 3D convolutional U-Net) on CDNA4 matrix cores.
//
// The 3x3x3 convolutions are implicit GEMMs on v_mfma_f32_32x32x16_bf16 (BF16 operands, FP32
// accumulation), 16 input channels a step: the A operand is the channels-last activation (the 8 BF16
// values a lane supplies are contiguous channels of one voxel), through an LDS halo or straight from
// memory on small volumes, the B operand the weight rows.  Operand layout of the instruction (wave64),
// checked by sur_mfma_selftest:
//   A (32 x 16): lane l supplies A[l % 32][8 (l / 32) + j], j < 8
//   B (16 x 32): lane l supplies B[8 (l / 32) + j][l % 32]
//   D (32 x 32): lane l holds D[8 (i / 4) + 4 (l / 32) + i % 4][l % 32] in accumulator i < 16
// The weight gradient, whose reduction index is the voxel, first copies dY and X into a blocked layout
// ([voxel / 8][channel][8]: a lane's 8 voxels of one channel are one 16-byte word) and gives each wave
// the three taps of one (dz, dy) pair, over rows staged in an LDS ring.  It reduces over voxels in fixed
// chunks followed by a fixed-order two-level sum, so every result is deterministic.
#include <algorithm>
#include <cmath>
#include <utility>

#include "../../include/nslgf_surrogate.h"
#include "kernels.h"

namespace nslgf {

typedef unsigned short bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ bf16_t f2bf(float f) {
    unsigned u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
    return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float(((unsigned)b) << 16); }

__device__ __forceinline__ bf16x8 load8(const bf16_t* p) {
    const uint4 q = *(const uint4*)p;
    return __builtin_bit_cast(bf16x8, q);
}
__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)); }
__device__ __forceinline__ bf16x8 pack8(const bf16_t v[8]) {
    uint4 q;
    q.x = (unsigned)v[0] | ((unsigned)v[1] << 16);
    q.y = (unsigned)v[2] | ((unsigned)v[3] << 16);
    q.z = (unsigned)v[4] | ((unsigned)v[5] << 16);
    q.w = (unsigned)v[6] | ((unsigned)v[7] << 16);
    return __builtin_bit_cast(bf16x8, q);
}

// Y[v][n] = act(sum_tap sum_k X[v + SIGN off(tap)][k] Wn[tap][n][k]);  K % 16 == 0, N % 32 == 0.
// A workgroup of 9 wavefronts owns one 32 x 32 output tile; wave g sums the three dx taps of one (dz, dy) pair
// with its A rows gathered from the activation, and the nine partial tiles are added in LDS in a fixed order.
// For volumes too small to fill the chip with the LDS-staged kernel below, where a wave's chain of dependent
// steps is the time: one wave per tile over all 27 taps took 28 us forward and 51 us for the data gradient at
// 16^3, 96 -> 128 channels, and 27 and 48 us at 8^3; this takes 15 and 22, and 8 and 14.  MT = 2 gives a
// workgroup two tiles of voxels, which halves its weight reads (19 and 27 us with one at 16^3); below 256
// tiles that leaves CUs idle (12^3: 10.1 and 14.9 us with one, 10.8 and 20.9 with two).  Its six row pointers take it
// past its 96 registers: 8 spill.
__device__ __forceinline__ int split_row(int i, int half) { return 8 * (i / 4) + 4 * half + (i % 4); }
template <bool RELU, int SIGN, int MT>
__global__ void __launch_bounds__(576, MT == 1 ? 7 : 5) k_conv_split(const bf16_t* __restrict__ X, const bf16_t* __restrict__ Wn,
                                                    float* __restrict__ Y, int D, int H, int W, int K, int N,
                                                    long long nblocks) {
    __shared__ float part[9][MT * 1024];
    const int ntiles = N / 32;
    const int g = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int m = lane % 32, half = lane / 32;
    const long long nvox = (long long)D * H * W, wtap = (long long)N * K;
    for (long long blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        const int n0 = (int)(blk % ntiles) * 32;
        const long long v0 = blk / ntiles * (32 * MT);
        f32x16 acc[MT];
        const bf16_t* xp[MT][3];
        bool ok[MT][3];
#pragma unroll
        for (int r = 0; r < MT; ++r) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][i] = 0.f;
            const long long v = v0 + 32 * r + m;
            const int x = (int)(v % W), y = (int)((v / W) % H), z = (int)(v / ((long long)W * H));
            const int zz = z + SIGN * (g / 3 - 1), yy = y + SIGN * (g % 3 - 1);
            const bool row_ok = v < nvox && zz >= 0 && zz < D && yy >= 0 && yy < H;
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int xx = x + SIGN * (t - 1);
                ok[r][t] = row_ok && xx >= 0 && xx < W;
                xp[r][t] = X + (ok[r][t] ? ((long long)zz * H + yy) * W + xx : 0) * K + half * 8;
            }
        }
        const bf16_t* wp = Wn + ((long long)(3 * g) * N + n0 + m) * K + half * 8;
#pragma unroll 2
        for (int kc = 0; kc < K; kc += 16) {
            bf16x8 a[MT][3], b[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                b[t] = load8(wp + t * wtap + kc);
#pragma unroll
                for (int r = 0; r < MT; ++r) a[r][t] = ok[r][t] ? load8(xp[r][t] + kc) : zero8();
            }
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int r = 0; r < MT; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[r][t], b[t], acc[r], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < MT; ++r)
#pragma unroll
            for (int i = 0; i < 16; ++i) part[g][r * 1024 + i * 64 + lane] = acc[r][i];
        __syncthreads();
        for (int e = threadIdx.x; e < MT * 1024; e += 576) {
            float val = 0.f;
#pragma unroll
            for (int w = 0; w < 9; w += 3) val += (part[w][e] + part[w + 1][e]) + part[w + 2][e];
            if (RELU) val = fmaxf(val, 0.f);
            const long long v = v0 + e / 1024 * 32 + split_row(e / 64 % 16, (e / 32) % 2);
            if (v < nvox) Y[v * N + n0 + e % 32] = val;
        }
        __syncthreads();
    }
}

// The same convolution with the input staged in LDS.  A workgroup (4 waves) owns a block of TX x (4 TY) x 4
// voxels (TX TY = 32) and one tile of 32 output channels.  For every slice of 16 input channels it copies the
// slice's halo (zero outside the volume) into LDS once; the two 8-channel halves lie in planes of their own,
// so that a half-wave reads 16-byte words in a row.  Each wave owns TX x TY voxels (its matrix tile) of 4 z
// planes: for every (dy, dx) of the stencil it reads its tile of the 6 planes those 4 need and applies them
// for the three dz taps, so that an A operand read from LDS serves up to three taps, and a B operand (weights,
// read through the caches) serves the wave's 4 planes.  Any volume: voxels beyond it are computed from zeros
// and not stored.  The sum runs over slices, then dy, dx, dz (+1 first) in a fixed order:
// results are deterministic (dx before dy: 122 us at 128^3, 16 -> 32 channels, this 108).
// The time is the matrix operations and the latency of a slice's staging and of the weights, which the three
// workgroups of a CU overlap (128^3, 32 -> 32 channels: 183 to 194 us back to back, 590 to 635 TFLOP/s, and 153 to
// 166 between other passes, at a higher clock; a form with the weights in LDS and the next slice in registers ran
// two workgroups a CU and took 277).  Rows along y served three dy taps before, which tied the block to 32 voxels
// along x: widths that 32 does not divide went through the gathering kernel (112^3, 32 -> 32: 328 us, now 123;
// 56^3, 32 -> 64: 81 and 153 for the data gradient, now 39 and 50; 80^3: 121, now 47).
// The form Z = 2 owns TX x (8 TY) x 2 voxels: a wave takes two tiles of y in each of 2 planes, as many matrix
// operations in all.
template <int TX, int Z> struct LdsBlk {
    static constexpr int NY = 4 / Z, TY = 32 / TX, BY = 4 * TY * NY, HX = TX + 2, HY = BY + 2, HZ = Z + 2;
    static constexpr int HALO = HX * HY * HZ, PLANE = (HALO + 7) / 8 * 8 + 4;  // (halves 64 bytes apart in the banks)
};
template <bool RELU, int SIGN, int TX, int Z>
__global__ void __launch_bounds__(256) k_conv_lds(const bf16_t* __restrict__ X, const bf16_t* __restrict__ Wn,
                                                  float* __restrict__ Y, int D, int H, int W, int K, int N) {
    using B = LdsBlk<TX, Z>;
    __shared__ uint4 halo[2 * B::PLANE];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int m = lane % 32, half = lane / 32;
    const int xt = (W + TX - 1) / TX;
    const int x0 = (blockIdx.x % xt) * TX, nb = (blockIdx.x / xt) * 32;
    const int y0 = blockIdx.y * B::BY, z0 = blockIdx.z * Z;
    f32x16 acc[B::NY][Z];
#pragma unroll
    for (int t = 0; t < B::NY; ++t)
#pragma unroll
        for (int r = 0; r < Z; ++r)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][r][i] = 0.f;
    // this thread's halo elements (the same in every slice): offsets from the block's first voxel, in
    // BF16 elements (the host keeps 6 H W K below 2^31), and whether each lies inside the volume
    constexpr int kPer = (B::HALO * 2 + 255) / 256, kFirst = kPer / 2;
    const bf16_t* xblk = X + (((long long)z0 * H + y0) * W + x0) * K;
    int hoff[kPer];
    unsigned hok = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int q = tid + 256 * i;
        const int hv = q / 2, hh = q % 2;
        const int hx = hv % B::HX, hy = (hv / B::HX) % B::HY, hz = hv / (B::HX * B::HY);
        const int xx = x0 + hx - 1, yy = y0 + hy - 1, zz = z0 + hz - 1;
        hoff[i] = (((hz - 1) * H + (hy - 1)) * W + (hx - 1)) * K + hh * 8;
        if (q < B::HALO * 2 && xx >= 0 && xx < W && yy >= 0 && yy < H && zz >= 0 && zz < D) hok |= 1u << i;
    }
    uint4* hdst = halo + (tid % 2) * B::PLANE + tid / 2;
    const int ty = wave * B::TY + m / TX, tx = m % TX;  // this lane's voxel of the block
    const uint4* hsrc = halo + half * B::PLANE + (ty + 1) * B::HX + tx + 1;
    // the weights of the (dy, dx) two ahead are loaded while the current ones multiply, also across slices
    const bf16_t* wbase = Wn + ((long long)nb + m) * K + half * 8;
    const long long wtap = (long long)N * K;
    bf16x8 b[3][3];
    auto load_b = [&](int kc, int it, bf16x8 (&d)[3]) {
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) d[dz] = load8(wbase + (dz * 9 + it) * wtap + kc);
    };
    load_b(0, 0, b[0]);
    load_b(0, 1, b[1]);
    for (int kc = 0; kc < K; kc += 16) {
        // the slice's halo in two batches of loads, each issued whole before its LDS writes
        uint4 hr[kFirst];
#pragma unroll
        for (int i = 0; i < kFirst; ++i)
            hr[i] = (hok >> i) & 1 ? *(const uint4*)(xblk + kc + hoff[i]) : make_uint4(0, 0, 0, 0);
        __syncthreads();  // (the previous slice's reads are done)
#pragma unroll
        for (int i = 0; i < kFirst; ++i) hdst[128 * i] = hr[i];
        uint4 hr2[kPer - kFirst];
#pragma unroll
        for (int i = kFirst; i < kPer; ++i)
            hr2[i - kFirst] = (hok >> i) & 1 ? *(const uint4*)(xblk + kc + hoff[i]) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = kFirst; i < kPer; ++i)
            if (tid + 256 * i < B::HALO * 2) hdst[128 * i] = hr2[i - kFirst];
        __syncthreads();
        const int kn = kc + 16 < K ? kc + 16 : kc;  // (after the last slice: loaded and not used)
#pragma unroll 1
        for (int dy = 0; dy < 3; ++dy) {
            const uint4* hp = hsrc + SIGN * (dy - 1) * B::HX;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const int nx = 3 * dy + dx + 2;
                load_b(nx < 9 ? kc : kn, nx < 9 ? nx : nx - 9, b[(dx + 2) % 3]);
                bf16x8 a[B::NY][Z + 2];
#pragma unroll
                for (int t = 0; t < B::NY; ++t)
#pragma unroll
                    for (int j = 0; j < Z + 2; ++j)
                        a[t][j] = __builtin_bit_cast(bf16x8, hp[(j * B::HY + t * 4 * B::TY) * B::HX + SIGN * (dx - 1)]);
#pragma unroll
                for (int dz = 1; dz >= -1; --dz)
#pragma unroll
                    for (int t = 0; t < B::NY; ++t)
#pragma unroll
                        for (int r = 0; r < Z; ++r)
                            acc[t][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][r + SIGN * dz + 1], b[dx][dz + 1],
                                                                                acc[t][r], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < Z; ++r) {
        if (z0 + r >= D) break;
#pragma unroll
        for (int t = 0; t < B::NY; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = split_row(i, half);
                const int xx = x0 + row % TX, yy = y0 + (4 * t + wave) * B::TY + row / TX;
                float val = acc[t][r][i];
                if (RELU) val = fmaxf(val, 0.f);
                if (xx < W && yy < H) Y[(((long long)(z0 + r) * H + yy) * W + xx) * N + nb + m] = val;
            }
    }
}

template <int TX, int Z> static long long lds_blocks(int D, int H, int W) {
    return (long long)ceil_div(W, TX) * ceil_div(H, LdsBlk<TX, Z>::BY) * ceil_div(D, Z);
}
template <bool RELU, int SIGN, int TX, int Z>
static void launch_conv_lds(const bf16_t* x, const bf16_t* w, float* y, int D, int H, int W, int K, int N,
                            hipStream_t s) {
    // one output tile per workgroup: more workgroups on the small volumes, and more tiles would hold
    // 64 more accumulator registers per lane and tile
    const dim3 grid((unsigned)(ceil_div(W, TX) * (N / 32)), ceil_div(H, LdsBlk<TX, Z>::BY), ceil_div(D, Z));
    hipLaunchKernelGGL((k_conv_lds<RELU, SIGN, TX, Z>), grid, dim3(256), 0, s, x, w, y, D, H, W, K, N);
}
// The block shape with the fewest blocks (the least work beyond the volume's edges; 16 wide in a tie: 128^3,
// 32 -> 32: 194 us forward and 185 for the data gradient, 32 wide 193 and 195, 8 wide 195 and 198).  The split
// kernel below 48 workgroups, where most CUs would idle over 4 us a slice (16^3, 96 -> 128 with 32 workgroups:
// 24 us against 15; 24^3, 64 -> 96 with 108: 24 against 39), and where a block's offsets pass 32 bits or the
// grid its limits.  Two planes a workgroup where that saves 15 % of the blocks, which is on few planes that 4 does
// not divide (us with four and two: 2 x 128 x 128, 256 -> 256: 239 and 141, 96 -> 128: 46 and 34; 6 x 128 x 128,
// 256 -> 256: 485 and 404; where it saves less, 34 x 64 x 64, 32 -> 64 data gradient: 39 and 45).
template <bool RELU, int SIGN>
static void launch_conv(const bf16_t* x, const bf16_t* w, float* y, int D, int H, int W, int K, int N, hipStream_t s) {
    const long long nvox = (long long)D * H * W;
    using Form = std::pair<long long, void (*)(const bf16_t*, const bf16_t*, float*, int, int, int, int, int, hipStream_t)>;
    const auto fewest = [](const Form& p, const Form& q) { return p.first < q.first; };
    Form f = std::min({Form{lds_blocks<16, 4>(D, H, W), launch_conv_lds<RELU, SIGN, 16, 4>},
                       Form{lds_blocks<32, 4>(D, H, W), launch_conv_lds<RELU, SIGN, 32, 4>},
                       Form{lds_blocks<8, 4>(D, H, W), launch_conv_lds<RELU, SIGN, 8, 4>}}, fewest);
    const Form flat = std::min({Form{lds_blocks<16, 2>(D, H, W), launch_conv_lds<RELU, SIGN, 16, 2>},
                                Form{lds_blocks<32, 2>(D, H, W), launch_conv_lds<RELU, SIGN, 32, 2>},
                                Form{lds_blocks<8, 2>(D, H, W), launch_conv_lds<RELU, SIGN, 8, 2>}}, fewest);
    if (20 * flat.first <= 17 * f.first) f = flat;
    if (f.first * (N / 32) < 48 || 6LL * H * W * K >= (1LL << 31) || D / 2 >= 65535 || H / 4 >= 65535) {
        const long long nt = N / 32, tiles = nvox / 32 * nt, pairs = (nvox + 63) / 64 * nt, most = 1 << 22;
        if (tiles < 256)
            hipLaunchKernelGGL((k_conv_split<RELU, SIGN, 1>), dim3((unsigned)tiles), dim3(576), 0, s, x, w, y, D, H, W,
                               K, N, tiles);
        else
            hipLaunchKernelGGL((k_conv_split<RELU, SIGN, 2>), dim3((unsigned)(pairs < most ? pairs : most)), dim3(576),
                               0, s, x, w, y, D, H, W, K, N, pairs);
        return;
    }
    f.second(x, w, y, D, H, W, K, N, s);
}

// Channels-last [nvox][C] -> blocked [nvox / 8][C][8] (BF16): within each group of 8 consecutive voxels the
// channels become the slow index, so that the weight gradient's MFMA operands (whose reduction index is
// the voxel) read 8 consecutive voxels of one channel as one 16-byte load, and the 32 channels of a
// half-wave read 512 contiguous bytes.  One thread transposes 8 voxels x 8 channels in registers.
__global__ void __launch_bounds__(256) k_to_blocked8(const bf16_t* __restrict__ x, bf16_t* __restrict__ y,
                                                     long long ngroups, int C) {
    const int cgs = C / 8;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= ngroups * cgs) return;
    const long long g = e / cgs;
    const int cg = (int)(e % cgs) * 8;
    uint4 in[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) in[j] = *(const uint4*)(x + (g * 8 + j) * C + cg);
    const bf16_t* a = (const bf16_t*)in;  // a[j * 8 + c]: voxel j, channel cg + c
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        bf16_t o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = a[j * 8 + c];
        *(uint4*)(y + (g * C + cg + c) * 8) = *(const uint4*)o;
    }
}

// The same layout for rows of W voxels, W % 8 != 0: each x row starts a group of its own and its last group is
// filled with zeros, [row][ceil(W / 8)][C][8].
__global__ void __launch_bounds__(256) k_rows_to_blocked8(const bf16_t* __restrict__ x, bf16_t* __restrict__ y,
                                                          long long rows, int W, int C) {
    const int cgs = C / 8, nx = (W + 7) / 8;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * nx * cgs) return;
    const long long g = e / cgs, row = g / nx;
    const int cg = (int)(e % cgs) * 8, xg = (int)(g % nx) * 8;
    uint4 in[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        in[j] = xg + j < W ? *(const uint4*)(x + (row * W + xg + j) * C + cg) : make_uint4(0, 0, 0, 0);
    const bf16_t* a = (const bf16_t*)in;  // a[j * 8 + c]: voxel j, channel cg + c
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        bf16_t o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = a[j * 8 + c];
        *(uint4*)(y + (g * C + cg + c) * 8) = *(const uint4*)o;
    }
}

// FP32 -> BF16 cast of channels-last [nvox][C] with an optional ReLU backward and an optional blocked
// copy: val = src (0 where act is given and not > 0, as k_relu_bwd leaves it), y[v][c] = bf16(val) and
// yb[v / 8][c][v % 8] = bf16(val) (the layout of k_to_blocked8).
__device__ __forceinline__ uint2 cast4(float4 s, const float4* a) {
    if (a) {
        if (!(a->x > 0.f)) s.x = 0.f;
        if (!(a->y > 0.f)) s.y = 0.f;
        if (!(a->z > 0.f)) s.z = 0.f;
        if (!(a->w > 0.f)) s.w = 0.f;
    }
    return make_uint2(f2bf(s.x) | (unsigned)f2bf(s.y) << 16, f2bf(s.z) | (unsigned)f2bf(s.w) << 16);
}
// Without the blocked copy the layout does not matter: a workgroup takes 2048 values in a row (us at 128^3, in the
// tiles below and so: 32 channels 70 and 67, 48 channels 195 and 99, 64 channels 167 and 131; with act 122 and
// 117, 303 and 174, 295 and 239).
template <bool ACT>
__global__ void __launch_bounds__(256) k_cast_flat(const float4* __restrict__ src, const float4* __restrict__ act,
                                                   uint2* __restrict__ y, long long n4) {
    const long long e0 = (long long)blockIdx.x * 512 + threadIdx.x;
    float4 s[2], a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const long long e = min(e0 + 256 * i, n4 - 1);
        s[i] = src[e];
        if (ACT) a[i] = act[e];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (e0 + 256 * i < n4) y[e0 + 256 * i] = cast4(s[i], ACT ? &a[i] : nullptr);
}
// With it a workgroup takes 4096 / CW voxels x CW channels; a thread two times two voxels x 4 channels, so that
// CW / 4 lanes read 128 or 256 bytes of a row; the blocked copy goes through LDS and is written in rows of
// 16-byte words.  Bytes bound it (one thread per 8 voxels x 8 channels, which touched every line several times: at
// 128^3 x 32 channels 142 us, now 92, 5.9 TB/s; with act 198, now 165).
template <int CW>
__global__ void __launch_bounds__(256) k_cast_blocked(const float* __restrict__ src, const float* __restrict__ act,
                                                      bf16_t* __restrict__ y, bf16_t* __restrict__ yb, long long nvox,
                                                      int C, int chunks) {
    constexpr int VT = 4096 / CW, LR = CW / 4, NP = 256 / LR;  // voxels; lanes of a row; pairs of voxels at a time
    __shared__ unsigned tile[VT / 8][CW][4 + 1];  // [group][channel][pairs of voxels], one word of padding
    const int tid = threadIdx.x;
    // the chunks of one row on one XCD (workgroup b runs on XCD b mod 8)
    const int run = 8 * chunks, first = (int)blockIdx.x / run * run, r = (int)blockIdx.x - first;
    const int lg = first + run <= (int)gridDim.x ? first + r % 8 * chunks + r / 8 : (int)blockIdx.x;
    const long long v0 = (long long)(lg / chunks) * VT;
    const int c0 = lg % chunks * CW;
    const int cq = (tid % LR) * 4, c = c0 + cq;
    float4 s[2][2], a[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const long long v = v0 + 2 * NP * i + tid / LR * 2 + j;
            const bool ok = v < nvox && c < C;
            s[i][j] = ok ? *(const float4*)(src + v * C + c) : make_float4(0.f, 0.f, 0.f, 0.f);
            if (act) a[i][j] = ok ? *(const float4*)(act + v * C + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = NP * i + tid / LR;  // the pair of voxels
        uint2 w[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            w[j] = cast4(s[i][j], act ? &a[i][j] : nullptr);
            const long long v = v0 + 2 * p + j;
            if (v < nvox && c < C) *(uint2*)(y + v * C + c) = w[j];
        }
        unsigned* t = &tile[p / 4][cq][p % 4];
        t[0] = (w[0].x & 0xffffu) | w[1].x << 16;
        t[5] = w[0].x >> 16 | (w[1].x & 0xffff0000u);
        t[10] = (w[0].y & 0xffffu) | w[1].y << 16;
        t[15] = w[0].y >> 16 | (w[1].y & 0xffff0000u);
    }
    __syncthreads();
    const int nc = min(CW, C - c0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 256 * i, g = e / CW, ch = e % CW;
        if (v0 + 8 * g < nvox && ch < nc) {
            const unsigned* t = tile[g][ch];
            *(uint4*)(yb + ((v0 / 8 + g) * C + c0 + ch) * 8) = make_uint4(t[0], t[1], t[2], t[3]);
        }
    }
}

// Partial weight gradient of one chunk of the volume and one (cout, cin) tile pair:
//     P[chunk][tap][co][ci] = sum_{v in chunk} dY[v][co] X[v + off(tap)][ci],  tap = 3 (3 (dz + 1) + dy + 1) + dx + 1,
// from blocked copies (dYb [row][nx][cout][8], Xb [row][nx][cin][8], nx groups of 8 voxels a row).  A workgroup of 9
// wavefronts owns S groups of the rows y0 .. y0 + R - 1 of NZ planes and walks each plane RS rows at a time;
// wave g takes the three taps of one (dz, dy) pair.  The rows of X lie in an LDS ring (3 planes x 2 RS + 2
// rows of S groups and one on each side, zero outside the volume) beside two buffers of dY; the rows of the
// next step are loaded into registers while the current ones multiply.  A half-wave walks SH groups of a
// row, so that the voxel before and after a group (dx = -1 and +1) come from groups that it holds.
// PAIR: rows of one group (W <= 8); the half-waves take two neighbouring rows instead of two halves of one, of which
// the second would be empty, and a step is 8 rows (256 -> 256, 64 x 8 x 8: 91 us without, now 65; 32 x 32 x 8: 129, now
// 83; 96 -> 128 at 8^3: 21.4, now 20.5).
// PAD: rows of W voxels, W % 8 != 0, filled up with zeros; the one product that would pair such a filler with a
// voxel of the volume is masked, as are the groups that a half-wave lacks (an infinity there must not count).
// One workgroup a CU (its LDS, and waves of 140 to 168 registers, of which 4, padded 1, spill at eight groups a
// segment; the tenth wave only loads); the time is the matrix operations, 3 of the 9 waves on one SIMD, and a
// step's LDS latency.  The form before had every wave load its own operands and was bound by L2 (each XCD read all
// of both tensors for several of the nine pairs): 128^3, 32 -> 32: 276 us with the sums, now 174; 64^3, 32 -> 64:
// 79, now 63; 112^3: 223, now 144; 56^3, 32 -> 64: 192, now 55; rows that 8 does not divide, gathered voxel by
// voxel: 12^3, 96 -> 128: 193, now 28.  One row a step: 10 us more at 128^3; two workgroups a CU at 96 registers
// spilled and took 650.
constexpr int kWgThreads = 640;
struct WgradPlan {
    int nx, S, segs, SH, RS;  // groups of a row and of a segment, segments, groups of a half-wave, rows of a step
    int R, yb, NZ, zb;        // rows and planes of a chunk, and chunks along y and z
    int parts;                // partial sums of a chunk
    int chunks() const { return segs * yb * zb; }
    bool pair() const { return nx == 1; }
    size_t lds() const {
        const int sp = pair() ? 1 : 2 * SH;
        return (size_t)(3 * (2 * RS + 2) * (sp + 2) + 2 * RS * sp) * 512;
    }
};
template <int SH, int RS, bool PAD, bool PAIR>
__global__ void __launch_bounds__(kWgThreads)
k_conv_wgrad_ring(const bf16_t* __restrict__ dYb, const bf16_t* __restrict__ Xb, float* __restrict__ P, int D, int H, int W,
                  int cin, int cout, WgradPlan pl, int nblocks) {
    extern __shared__ uint4 wg_lds[];
    constexpr int NR = 2 * RS + 2;
    constexpr int SP = PAIR ? 1 : 2 * SH, S2 = SP + 2;  // groups of a row, and with their neighbours
    constexpr int NX = (3 * RS * S2 * 32 + kWgThreads - 1) / kWgThreads;  // 16-byte words of X of a thread and step
    // consecutive chunks, which share planes of X, on one XCD
    const int bid = (int)(blockIdx.x % 8) * ((int)gridDim.x / 8) + (int)blockIdx.x / 8;
    if (bid >= nblocks) return;
    const int tid = threadIdx.x, lane = tid % 64, g = tid / 64;
    const int cotiles = cout / 32, citiles = (cin + 31) / 32;
    int r = bid;
    const int cit = r % citiles;
    r /= citiles;
    const int cot = r % cotiles;
    const int chunk = r / cotiles;
    r = chunk;
    const int seg = r % pl.segs;
    r /= pl.segs;
    const int y0 = (r % pl.yb) * pl.R, y1 = min(H, y0 + pl.R);
    const int z0 = (r / pl.yb) * pl.NZ, z1 = min(D, z0 + pl.NZ);
    const int S = pl.S, nx = pl.nx, gx0 = seg * S;
    const int live = min(S, nx - gx0);  // groups of this segment
    const bool full = live == SP;
    uint4* const xr = wg_lds;                  // [plane][ring row][S2][32]
    uint4* const yr = wg_lds + 3 * NR * S2 * 32;  // [2][RS][SP][32]
    const int dz = g / 3 - 1, dy = g % 3 - 1;
    const int m = lane % 32, half = lane / 32;
    // a word of X: group (plane pz, row y, segment group gg - 1), channel ch of the tile
    auto x_word = [&](int zz, int yy, int gg, int ch) {
        const int gx = gx0 + gg - 1, ci = cit * 32 + ch;
        if (zz < 0 || zz >= D || yy < 0 || yy >= H || gx < 0 || gx >= nx || ci >= cin) return make_uint4(0, 0, 0, 0);
        return *(const uint4*)(Xb + ((((long long)zz * H + yy) * nx + gx) * cin + ci) * 8);
    };
    // this thread's words of a step: NX of the RS new rows of X in 3 planes, one of the RS rows of dY.  Of each:
    // its place in LDS (ring row 0, buffer 0), its place in its row (in words), its row of the step
    int xdst[NX], xpos[NX];
    unsigned xoff[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int e = tid + kWgThreads * i, ch = e % 32, t = e / 32;
        const int pz = t / (RS * S2), rr = (t / S2) % RS, gg = t % S2, gx = gx0 + gg - 1, ci = cit * 32 + ch;
        xdst[i] = (pz * NR * S2 + gg) * 32 + ch;
        xoff[i] = (unsigned)gx * cin + ci;
        xpos[i] = t < 3 * RS * S2 ? (gx >= 0 && gx < nx && ci < cin ? 4 * rr + pz : -1) : -2;
    }
    const int yt = tid / 32, yrr = yt / SP, ygx = gx0 + yt % SP;
    const int ydst = 3 * NR * S2 * 32 + tid;
    const unsigned yoff = (unsigned)ygx * cout + cot * 32 + tid % 32;
    const bool yhave = yt < RS * SP, yok = yhave && ygx < nx;
    const unsigned xrow = (unsigned)nx * cin, yrow = (unsigned)nx * cout;  // words of a row
    auto load_step = [&](int z, int y, uint4 (&w)[NX + 1]) {
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int zz = z + xpos[i] % 4 - 1, yy = y + 1 + xpos[i] / 4;
            w[i] = xpos[i] >= 0 && zz >= 0 && zz < D && yy < H
                       ? ((const uint4*)Xb)[((long long)zz * H + yy) * xrow + xoff[i]]
                       : make_uint4(0, 0, 0, 0);
        }
        w[NX] = yok && y + yrr < y1 ? ((const uint4*)dYb)[((long long)z * H + y + yrr) * yrow + yoff]
                                    : make_uint4(0, 0, 0, 0);
    };
    auto store_step = [&](int y, int buf, const uint4 (&w)[NX + 1]) {
        const int s0 = (y + 2) % NR;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            if (xpos[i] == -2) continue;
            int slot = s0 + (RS == 1 ? 0 : (tid + kWgThreads * i) / 32 / S2 % RS);
            if (slot >= NR) slot -= NR;
            wg_lds[xdst[i] + slot * S2 * 32] = w[i];
        }
        if (yhave) wg_lds[ydst + buf * RS * SP * 32] = w[NX];
    };
    f32x16 acc[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    // the sums of a long chunk's two halves are partials of their own: half the chain of FP32 additions
    const int ci = cit * 32 + m;
    const int steps = (z1 - z0) * ((y1 - y0 + RS - 1) / RS), mid = pl.parts == 2 ? (steps + 1) / 2 : 0;
    int step = 0, part = chunk * pl.parts;
    auto put = [&]() {
        if (ci >= cin || g >= 9) return;
        int cs = cin;
        asm volatile("" : "+s"(cs));  // (48 addresses formed here, not held through the loop)
        float* const out = P + (((long long)part * 27 + 3 * g) * cout + cot * 32 + 4 * half) * cs + ci;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) out[((long long)t * cout + 8 * (i / 4) + i % 4) * cs] = acc[t][i];
    };
    for (int z = z0; z < z1; ++z) {
        uint4 w[NX + 1];
        load_step(z, y0, w);
        __syncthreads();  // (the plane before is done)
        for (int e = tid; e < 3 * 2 * S2 * 32; e += kWgThreads) {  // rows y0 - 1 and y0
            const int ch = e % 32, gg = (e / 32) % S2, rr = (e / (32 * S2)) % 2, pz = e / (64 * S2);
            xr[((pz * NR + (y0 + rr) % NR) * S2 + gg) * 32 + ch] = x_word(z + pz - 1, y0 - 1 + rr, gg, ch);
        }
        store_step(y0, 0, w);
        __syncthreads();
        int buf = 0;
        for (int y = y0; y < y1; y += RS, buf ^= 1) {
            const bool more = y + RS < y1;
            if (more) load_step(z, y + RS, w);
#pragma unroll 1
            for (int rr = 0; rr < RS && y + rr < y1 && g < 9; rr += PAIR ? 2 : 1) {
                const int row = PAIR ? rr + half : rr, group = PAIR ? 0 : half * SH;  // of this half-wave
                const uint4* xp = xr + (((dz + 1) * NR + (y + row + dy + 1) % NR) * S2 + group) * 32 + m;
                const uint4* ap = yr + ((buf * RS + row) * SP + group) * 32 + m;
                unsigned pv = xp[0].w;
                uint4 q[SH + 1], av[SH];  // this half-wave's groups and the first words of the one after
#pragma unroll
                for (int j = 0; j < SH; ++j) {
                    q[j] = xp[(j + 1) * 32];
                    av[j] = ap[j * 32];
                }
                q[SH].x = xp[(SH + 1) * 32].x;
#pragma unroll
                for (int j = 0; j < SH; ++j) {
                    uint4 c = q[j];
                    unsigned nv = q[j + 1].x;
                    if (PAIR ? y + row >= y1 : !full && group + j >= live) {  // (no group here: both operands zero)
                        c = make_uint4(0, 0, 0, 0);
                        av[j] = c;
                        pv = 0;
                        nv = 0;
                    }
                    uint4 bm, bq;  // voxels x0 - 1 .. x0 + 6 and x0 + 1 .. x0 + 8
                    bm.x = (c.x << 16) | (pv >> 16);
                    bm.y = (c.y << 16) | (c.x >> 16);
                    bm.z = (c.z << 16) | (c.y >> 16);
                    bm.w = (c.w << 16) | (c.z >> 16);
                    bq.x = (c.x >> 16) | (c.y << 16);
                    bq.y = (c.y >> 16) | (c.z << 16);
                    bq.z = (c.z >> 16) | (c.w << 16);
                    bq.w = (c.w >> 16) | (nv << 16);
                    pv = c.w;
                    if (PAD && gx0 + group + j == nx - 1) {  // (the row's last voxel has no neighbour x + 1)
                        const unsigned keep = W % 2 ? 0xffffu : 0xffff0000u;
                        if (W % 8 / 2 == 0) bm.x &= keep;
                        if (W % 8 / 2 == 1) bm.y &= keep;
                        if (W % 8 / 2 == 2) bm.z &= keep;
                        if (W % 8 / 2 == 3) bm.w &= keep;
                    }
                    const bf16x8 a = __builtin_bit_cast(bf16x8, av[j]);
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, bm), acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, c), acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, bq), acc[2], 0, 0, 0);
                }
            }
            if (more) store_step(y + RS, buf ^ 1, w);
            if (++step == mid) {
                put();
                ++part;
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
            }
            __syncthreads();
        }
    }
    put();
}

// First level of the fixed-order chunk reduction: Q[g][i] = sum of the chunks g G .. g G + G - 1.
__global__ void k_sum_chunk_groups(const float* __restrict__ P, float* __restrict__ Q, long long n, int G, int nchunks) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int g = blockIdx.y;
    float s = 0.f;
    for (int c = g * G; c < min((g + 1) * G, nchunks); ++c) s += P[(long long)c * n + i];
    Q[(long long)g * n + i] = s;
}

__global__ void k_sum_chunks(const float* __restrict__ P, float* __restrict__ dW, long long n, int nchunks) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s = 0.f;
    for (int c = 0; c < nchunks; ++c) s += P[(long long)c * n + i];
    dW[i] = s;
}

__global__ void k_wtranspose(const bf16_t* __restrict__ w, bf16_t* __restrict__ wt, int cin, int cout) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n = 27LL * cin * cout;
    if (i >= n) return;
    const int ci = (int)(i % cin);
    const int co = (int)((i / cin) % cout);
    const int tap = (int)(i / ((long long)cin * cout));
    wt[((long long)tap * cin + ci) * cout + co] = w[i];
}

__global__ void k_cast_bf16(const float* __restrict__ x, bf16_t* __restrict__ y, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}
__global__ void k_relu_bwd(const float* __restrict__ y, float* __restrict__ g, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && !(y[i] > 0.f)) g[i] = 0.f;
}
__global__ void k_add(const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ o, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) o[i] = a[i] + b[i];
}

// coarse voxel index of fine (z, y, x)
__device__ __forceinline__ long long coarse_of(long long v, int D, int H, int W) {
    const int x = (int)(v % W), y = (int)((v / W) % H), z = (int)(v / ((long long)W * H));
    return ((long long)(z / 2) * (H / 2) + y / 2) * (W / 2) + x / 2;
}

// Fused resampling, skip sum and cast: val[v][c] = scale * coarse[parent(v)][c] + skip[v][c], parent(v)
// the voxel of the half-resolution grid that holds v (scale 1: the nearest-neighbour upsampling; scale
// 1/8: the adjoint of the 2x2x2 average pooling), then as k_cast_blocked: zero where act is given and not
// > 0, y[v][c] = bf16(val), and yb[v / 8][c][v % 8] = bf16(val) when yb is given.  The product and the
// sum are rounded one at a time, as the separate passes round them.  One thread: 8 voxels x 8 channels.
__global__ void __launch_bounds__(256) k_cast_up(const float* __restrict__ coarse, float scale,
                                                 const float* __restrict__ skip, const float* __restrict__ act,
                                                 bf16_t* __restrict__ y, bf16_t* __restrict__ yb, long long ngroups,
                                                 int C, int D, int H, int W) {
    const int cgs = C / 8;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= ngroups * cgs) return;
    const long long g = e / cgs;
    const int cg = (int)(e % cgs) * 8;
    // W % 8 == 0: the 8 voxels lie in one x row, so their parents follow from the first one's
    long long crow = 0;
    int x0 = 0;
    const bool row8 = W % 8 == 0;
    if (row8) {
        const long long v0 = g * 8;
        const long long zy = v0 / W;
        x0 = (int)(v0 - zy * W);
        const int y = (int)(zy % H), z = (int)(zy / H);
        crow = ((long long)(z / 2) * (H / 2) + y / 2) * (W / 2);
    }
    bf16_t o[64];  // o[j * 8 + c]: voxel j, channel cg + c
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const long long v = g * 8 + j;
        const long long parent = row8 ? crow + (x0 + j) / 2 : coarse_of(v, D, H, W);
        const long long base = v * C + cg, cb = parent * C + cg;
        const float4 c0 = *(const float4*)(coarse + cb), c1 = *(const float4*)(coarse + cb + 4);
        const float4 s0 = *(const float4*)(skip + base), s1 = *(const float4*)(skip + base + 4);
        const float cv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
        const float sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
        float v8[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v8[c] = __fadd_rn(__fmul_rn(scale, cv[c]), sv[c]);
        if (act) {
            const float4 a0 = *(const float4*)(act + base), a1 = *(const float4*)(act + base + 4);
            const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (!(a[c] > 0.f)) v8[c] = 0.f;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) o[j * 8 + c] = f2bf(v8[c]);
        *(uint4*)(y + base) = *(const uint4*)(o + j * 8);
    }
    if (yb) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            bf16_t t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) t[j] = o[j * 8 + c];
            *(uint4*)(yb + (g * C + cg + c) * 8) = *(const uint4*)t;
        }
    }
}

__global__ void k_pool2_fwd(const float* __restrict__ x, float* __restrict__ y, int D, int H, int W, int c) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nc = (long long)(D / 2) * (H / 2) * (W / 2) * c;
    if (i >= nc) return;
    const int ch = (int)(i % c);
    const long long vc = i / c;
    const int X = (int)(vc % (W / 2)), Y = (int)((vc / (W / 2)) % (H / 2)), Z = (int)(vc / ((long long)(W / 2) * (H / 2)));
    float s = 0.f;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b)
            for (int d = 0; d < 2; ++d) s += x[((((long long)(2 * Z + a) * H + 2 * Y + b) * W) + 2 * X + d) * c + ch];
    y[i] = 0.125f * s;
}
__global__ void k_pool2_bwd(const float* __restrict__ gy, float* __restrict__ gx, int D, int H, int W, int c) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nf = (long long)D * H * W * c;
    if (i >= nf) return;
    const int ch = (int)(i % c);
    gx[i] = 0.125f * gy[coarse_of(i / c, D, H, W) * c + ch];
}
__global__ void k_up2_fwd(const float* __restrict__ x, float* __restrict__ y, int D, int H, int W, int c) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nf = (long long)D * H * W * c;
    if (i >= nf) return;
    const int ch = (int)(i % c);
    y[i] = x[coarse_of(i / c, D, H, W) * c + ch];
}
__global__ void k_up2_bwd(const float* __restrict__ gy, float* __restrict__ gx, int D, int H, int W, int c) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nc = (long long)(D / 2) * (H / 2) * (W / 2) * c;
    if (i >= nc) return;
    const int ch = (int)(i % c);
    const long long vc = i / c;
    const int X = (int)(vc % (W / 2)), Y = (int)((vc / (W / 2)) % (H / 2)), Z = (int)(vc / ((long long)(W / 2) * (H / 2)));
    float s = 0.f;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b)
            for (int d = 0; d < 2; ++d) s += gy[((((long long)(2 * Z + a) * H + 2 * Y + b) * W) + 2 * X + d) * c + ch];
    gx[i] = s;
}

// VEC (c = 4 * 2^sh, grad on 16 bytes): one thread per 4 channels of a voxel (grid-stride), one
// 16-byte store each, so a wave writes contiguous rows; else one thread per voxel, one value at a time.
template <bool VEC>
__global__ void __launch_bounds__(256) k_mse(const float* __restrict__ pred, const float* __restrict__ tgt,
                                             float* __restrict__ grad, double* __restrict__ partial, long long nvox,
                                             int c, int used, int sh) {
    __shared__ double red[256];
    const double inv = 2.0 / ((double)nvox * used);
    double s = 0.0;
    if constexpr (VEC) {
        const long long n4 = nvox << sh;
        for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n4; e += (long long)gridDim.x * blockDim.x) {
            const long long v = e >> sh;
            const int c0 = (int)(e & ((1 << sh) - 1)) * 4;
            float o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int ch = c0 + k;
                o[k] = 0.f;
                if (ch < used) {
                    const double d = (double)pred[v * c + ch] - (double)tgt[v * used + ch];
                    s += d * d;
                    o[k] = (float)(inv * d);
                }
            }
            *(float4*)(grad + v * c + c0) = make_float4(o[0], o[1], o[2], o[3]);
        }
    } else {
        for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox;
             v += (long long)gridDim.x * blockDim.x) {
            for (int ch = 0; ch < c; ++ch) {
                if (ch < used) {
                    const double d = (double)pred[v * c + ch] - (double)tgt[v * used + ch];
                    s += d * d;
                    grad[v * c + ch] = (float)(inv * d);
                } else {
                    grad[v * c + ch] = 0.f;
                }
            }
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Squared error with the gradient written only as its BF16 copy y[v][c] and, when yb is given, the
// blocked copy yb[v / 8][c][v % 8] (the layout of k_to_blocked8): the gradient values are those of
// k_mse, rounded as sur_cast_bf16_ex rounds them.  One thread: 8 voxels x 8 channels (grid-stride); per-block
// FP64 partial sums of the squared error, in the order of this decomposition.
__global__ void __launch_bounds__(256) k_mse_cast(const float* __restrict__ pred, const float* __restrict__ tgt,
                                                  bf16_t* __restrict__ y, bf16_t* __restrict__ yb,
                                                  double* __restrict__ partial, long long nvox, int C, int used) {
    __shared__ double red[256];
    const double inv = 2.0 / ((double)nvox * used);
    const int cgs = C / 8;
    const long long ngroups = nvox / 8;
    double s = 0.0;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < ngroups * cgs;
         e += (long long)gridDim.x * blockDim.x) {
        const long long g = e / cgs;
        const int cg = (int)(e % cgs) * 8;
        bf16_t o[64];  // o[j * 8 + c]: voxel j, channel cg + c
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const long long v = g * 8 + j;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int ch = cg + c;
                float gv = 0.f;
                if (ch < used) {
                    const double d = (double)pred[v * C + ch] - (double)tgt[v * used + ch];
                    s += d * d;
                    gv = (float)(inv * d);
                }
                o[j * 8 + c] = f2bf(gv);
            }
            *(uint4*)(y + v * C + cg) = *(const uint4*)(o + j * 8);
        }
        if (yb) {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                bf16_t t[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) t[j] = o[j * 8 + c];
                *(uint4*)(yb + (g * C + cg + c) * 8) = *(const uint4*)t;
            }
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void k_adam(float* __restrict__ w, bf16_t* __restrict__ wb, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long long n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    wb[i] = f2bf(wi);
}

__global__ void k_pack_input(const double* __restrict__ om, bf16_t* __restrict__ x, long long nvox, double scale,
                             double feat) {
    const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    bf16_t out[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) out[k] = 0;
    for (int q = 0; q < 3; ++q) out[q] = f2bf((float)(om[q * nvox + v] * scale));
    out[3] = f2bf((float)feat);
    uint4* dst = (uint4*)(x + v * 16);
    dst[0] = __builtin_bit_cast(uint4, pack8(out));
    dst[1] = __builtin_bit_cast(uint4, pack8(out + 8));
}
// Input of the correction form: channels 0..2 = omega * scale, 3 = feat, 4..6 = delta * dscale.
__global__ void k_pack_input_pair(const double* __restrict__ om, const double* __restrict__ dl, bf16_t* __restrict__ x,
                                  long long nvox, double scale, double dscale, double feat) {
    const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    bf16_t out[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) out[k] = 0;
    for (int q = 0; q < 3; ++q) {
        out[q] = f2bf((float)(om[q * nvox + v] * scale));
        out[4 + q] = f2bf((float)(dl[q * nvox + v] * dscale));
    }
    out[3] = f2bf((float)feat);
    uint4* dst = (uint4*)(x + v * 16);
    dst[0] = __builtin_bit_cast(uint4, pack8(out));
    dst[1] = __builtin_bit_cast(uint4, pack8(out + 8));
}
// out = ca a + cb b + cc c (c may be null), FP64, n values.
__global__ void k_combine3(const double* __restrict__ a, const double* __restrict__ b, const double* __restrict__ c,
                           double* __restrict__ out, long long n, double ca, double cb, double cc) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double r = ca * a[i] + cb * b[i];
    if (c) r += cc * c[i];
    out[i] = r;
}
__global__ void k_pack_target(const double* __restrict__ f, float* __restrict__ t, long long nvox, double scale) {
    const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    for (int q = 0; q < 3; ++q) t[v * 3 + q] = (float)(f[q * nvox + v] * scale);
}
__global__ void k_unpack_update(const double* __restrict__ base, const float* __restrict__ y, double* __restrict__ out,
                                long long nvox, int c, double inv_scale) {
    const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    for (int q = 0; q < 3; ++q) out[q * nvox + v] = base[q * nvox + v] + (double)y[v * c + q] * inv_scale;
}

__global__ void k_mfma_selftest(const bf16_t* A, const bf16_t* B, float* C) {
    const int l = threadIdx.x;
    const int m = l % 32, half = l / 32;
    bf16_t av[8], bv[8];
    for (int j = 0; j < 8; ++j) {
        av[j] = A[m * 16 + 8 * half + j];
        bv[j] = B[(8 * half + j) * 32 + m];
    }
    f32x16 acc;
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pack8(av), pack8(bv), acc, 0, 0, 0);
    for (int i = 0; i < 16; ++i) C[(8 * (i / 4) + 4 * half + (i % 4)) * 32 + m] = acc[i];
}

static int grid1(long long n) { return ceil_div(n, 256); }

// Chunks of the weight gradient.  Cost in steps of RS rows (1 to 1.5 us each): the rounds of 256 workgroups
// (one a CU) times the steps of a chunk, two more for a plane's first rows, and 0.06 a workgroup for its
// partial sums, written and read once (110 KB).  Chunks of at least 8 rows.  Measured at 80^3, 32 -> 32: 160
// workgroups of a plane 99 us, what this rule takes 71.
static WgradPlan wgrad_plan(int D, int H, int W, int cin, int cout) {
    WgradPlan p;
    p.nx = ceil_div(W, 8);
    p.segs = ceil_div(p.nx, 8);
    p.S = ceil_div(p.nx, p.segs);
    p.segs = ceil_div(p.nx, p.S);
    p.SH = (p.S + 1) / 2;
    p.RS = p.pair() ? 8 : p.SH >= 3 ? 2 : 4;
    const long long per = (long long)(cout / 32) * ceil_div(cin, 32) * p.segs;
    double best = 0;
    p.R = H;
    p.NZ = D;
    for (int yb = 1; yb == 1 || ceil_div(H, yb) >= 8; ++yb) {
        const int R = ceil_div(ceil_div(H, yb), p.RS) * p.RS;
        const long long row = per * ceil_div(H, R);
        for (int rounds = 1; rounds <= 4; ++rounds) {
            const long long zmax = 256LL * rounds / row;
            if (zmax < 1 && rounds < 4) continue;
            const int NZ = zmax < 1 ? D : ceil_div(D, zmax < D ? zmax : D);
            const long long blocks = row * ceil_div(D, NZ);
            const double cost = (double)ceil_div(blocks, 256) * NZ * (R / p.RS + 2) + 0.06 * blocks;
            if (best == 0 || cost < best) {
                best = cost;
                p.R = R;
                p.NZ = NZ;
            }
        }
    }
    p.yb = ceil_div(H, p.R);
    p.zb = ceil_div(D, p.NZ);
    // two partials of a chunk of more than 768 voxels: the error against 64 bits stays at or below that of the
    // shorter chunks before (128^3: 4.2e-7, with one 5.8e-7), for 8 us of 174
    p.parts = (long long)p.R * p.NZ * p.S * 8 > 768 ? 2 : 1;
    return p;
}
// What the blocked form takes as it is: rows of whole groups.
static bool wgrad_blocked_ok(int W, long long nvox) { return W % 8 == 0 && nvox % 16 == 0; }
static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

template <int SH, int RS, bool PAD, bool PAIR>
static int launch_wgrad_ring(const WgradPlan& p, const bf16_t* dyc, const bf16_t* xc, float* part, int D, int H, int W,
                             int cin, int cout, hipStream_t s) {
    const int blocks = p.chunks() * (cout / 32) * ceil_div(cin, 32);
    hipLaunchKernelGGL((k_conv_wgrad_ring<SH, RS, PAD, PAIR>), dim3((unsigned)ceil_div(blocks, 8) * 8), dim3(kWgThreads), p.lds(), s,
                       dyc, xc, part, D, H, W, cin, cout, p, blocks);
    return NSLGF_OK;
}

}  // namespace nslgf

using namespace nslgf;

#define SUR_ENTER(h)                                                                               \
    do {                                                                                           \
        int rc_ = enter_handle(h);                                                                 \
        if (rc_ != NSLGF_OK) return rc_;                                                           \
    } while (0)

// The matrix-core and layout kernels move 16 bytes per access: their tensors must start on 16 bytes.
static bool a16(const void* p) { return p == nullptr || ((uintptr_t)p % 16) == 0; }

static int conv_shape_ok(int D, int H, int W, int cin, int cout) {
    NSLGF_CHECK_ARG(D >= 1 && H >= 1 && W >= 1 && (long long)D * H * W % 32 == 0, "surrogate: D*H*W must be a multiple of 32");
    NSLGF_CHECK_ARG(cin >= 16 && cin % 16 == 0 && cin <= 1024, "surrogate: cin must be a multiple of 16");
    NSLGF_CHECK_ARG(cout >= 32 && cout % 32 == 0 && cout <= 1024, "surrogate: cout must be a multiple of 32");
    return NSLGF_OK;
}

extern "C" {

int sur_conv3d_fwd(nslgf_t h, const void* x, const void* w, void* y, int D, int H, int W, int cin, int cout, int relu,
                   void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(conv_shape_ok(D, H, W, cin, cout));
    NSLGF_CHECK_ARG(x && w && y, "sur_conv3d_fwd: null pointer");
    NSLGF_CHECK_ARG(a16(x) && a16(w) && a16(y), "sur_conv3d_fwd: tensors must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    if (relu)
        launch_conv<true, 1>((const bf16_t*)x, (const bf16_t*)w, (float*)y, D, H, W, cin, cout, s);
    else
        launch_conv<false, 1>((const bf16_t*)x, (const bf16_t*)w, (float*)y, D, H, W, cin, cout, s);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_conv3d_bwd_data(nslgf_t h, const void* dy, const void* wt, void* dx, int D, int H, int W, int cin, int cout,
                        void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(conv_shape_ok(D, H, W, cin, cout));
    NSLGF_CHECK_ARG(cin % 32 == 0, "sur_conv3d_bwd_data: cin must be a multiple of 32");
    NSLGF_CHECK_ARG(dy && wt && dx, "sur_conv3d_bwd_data: null pointer");
    NSLGF_CHECK_ARG(a16(dy) && a16(wt) && a16(dx), "sur_conv3d_bwd_data: tensors must be 16-byte aligned");
    // GEMM with K = cout (inner) and N = cin (outputs), gathering dy at v - off
    launch_conv<false, -1>((const bf16_t*)dy, (const bf16_t*)wt, (float*)dx, D, H, W, cout, cin, (hipStream_t)stream);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

static size_t wgrad_work(int D, int H, int W, int cin, int cout) {
    // chunk partials, then the group sums of the partials
    const WgradPlan p = wgrad_plan(D, H, W, cin, cout);
    const int nch = p.chunks() * p.parts;
    return align256((size_t)nch * 27 * cin * cout * sizeof(float)) + (size_t)(nch / 32 + 1) * 27 * cin * cout * sizeof(float);
}

size_t sur_bwd_weight_work_bytes(int D, int H, int W, int cin, int cout) {
    if (D < 1 || H < 1 || W < 1 || cin < 1 || cout < 32) return 0;
    // the blocked copies of dY and X (rows filled up to 8 voxels), then what the blocked form needs
    const size_t nvox = (size_t)D * H * ceil_div(W, 8) * 8;
    return align256(nvox * cout * 2) + align256(nvox * cin * 2) + wgrad_work(D, H, W, cin, cout);
}

size_t sur_bwd_weight_blocked_work_bytes(int D, int H, int W, int cin, int cout) {
    if (D < 1 || H < 1 || W < 1 || cin < 1 || cout < 32) return 0;
    if (!wgrad_blocked_ok(W, (long long)D * H * W)) return 0;
    return wgrad_work(D, H, W, cin, cout);
}

// Weight gradient from the blocked copies, partials and their fixed-order sums in `work`.
static int wgrad_from_blocked(const bf16_t* dyc, const bf16_t* xc, float* dw, char* work, int D, int H, int W, int cin,
                              int cout, hipStream_t s) {
    const long long n = 27LL * cin * cout;
    const WgradPlan p = wgrad_plan(D, H, W, cin, cout);
    const int nch = p.chunks() * p.parts;
    float* part = (float*)work;
    const bool pad = W % 8 != 0;
#define WGRAD_RING(SH, RS, PAIR)                                                                    \
    (pad ? launch_wgrad_ring<SH, RS, true, PAIR>(p, dyc, xc, part, D, H, W, cin, cout, s)           \
         : launch_wgrad_ring<SH, RS, false, PAIR>(p, dyc, xc, part, D, H, W, cin, cout, s))
    NSLGF_TRY(p.pair() ? WGRAD_RING(1, 8, true) : p.SH == 4 ? WGRAD_RING(4, 2, false) : p.SH == 3 ? WGRAD_RING(3, 2, false)
              : p.SH == 2 ? WGRAD_RING(2, 4, false) : WGRAD_RING(1, 4, false));
#undef WGRAD_RING
    if (nch >= 64) {
        // two levels (groups of 32 chunks, then the groups), each in a fixed order
        const int G = 32, ng = ceil_div(nch, G);
        float* q = (float*)(work + align256((size_t)nch * 27 * cin * cout * sizeof(float)));
        hipLaunchKernelGGL(k_sum_chunk_groups, dim3(grid1(n), ng), dim3(256), 0, s, (const float*)part, q, n, G, nch);
        hipLaunchKernelGGL(k_sum_chunks, dim3(grid1(n)), dim3(256), 0, s, (const float*)q, dw, n, ng);
    } else {
        hipLaunchKernelGGL(k_sum_chunks, dim3(grid1(n)), dim3(256), 0, s, (const float*)part, dw, n, nch);
    }
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_conv3d_bwd_weight(nslgf_t h, const void* dy, const void* x, void* dw, void* work, int D, int H, int W, int cin,
                          int cout, void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(conv_shape_ok(D, H, W, cin, cout));
    NSLGF_CHECK_ARG(dy && x && dw && work, "sur_conv3d_bwd_weight: null pointer");
    NSLGF_CHECK_ARG(a16(dy) && a16(x) && a16(dw) && a16(work), "sur_conv3d_bwd_weight: tensors must be 16-byte aligned");
    const long long rows = (long long)D * H, groups = rows * ceil_div(W, 8);
    hipStream_t s = (hipStream_t)stream;
    bf16_t* dyc = (bf16_t*)work;
    bf16_t* xc = (bf16_t*)((char*)work + align256((size_t)groups * 8 * cout * 2));
    char* rest = (char*)xc + align256((size_t)groups * 8 * cin * 2);
    auto blocked = [&](const void* src, bf16_t* dst, int c) {
        const dim3 grid((unsigned)ceil_div(groups * (c / 8), 256));
        if (W % 8 == 0)
            hipLaunchKernelGGL(k_to_blocked8, grid, dim3(256), 0, s, (const bf16_t*)src, dst, groups, c);
        else
            hipLaunchKernelGGL(k_rows_to_blocked8, grid, dim3(256), 0, s, (const bf16_t*)src, dst, rows, W, c);
    };
    blocked(dy, dyc, cout);
    blocked(x, xc, cin);
    return wgrad_from_blocked(dyc, xc, (float*)dw, rest, D, H, W, cin, cout, s);
}

int sur_conv3d_bwd_weight_blocked(nslgf_t h, const void* dyb, const void* xb, void* dw, void* work, int D, int H, int W,
                                  int cin, int cout, void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(conv_shape_ok(D, H, W, cin, cout));
    NSLGF_CHECK_ARG(dyb && xb && dw && work, "sur_conv3d_bwd_weight_blocked: null pointer");
    NSLGF_CHECK_ARG(a16(dyb) && a16(xb) && a16(dw) && a16(work), "sur_conv3d_bwd_weight_blocked: tensors must be 16-byte aligned");
    NSLGF_CHECK_ARG(wgrad_blocked_ok(W, (long long)D * H * W), "sur_conv3d_bwd_weight_blocked: needs W % 8 == 0 and D*H*W % 16 == 0");
    return wgrad_from_blocked((const bf16_t*)dyb, (const bf16_t*)xb, (float*)dw, (char*)work, D, H, W, cin, cout,
                              (hipStream_t)stream);
}

int sur_cast_bf16_ex(nslgf_t h, const void* src, const void* act, void* y, void* yb, long long nvox, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(src && y && nvox >= 0 && nvox % 8 == 0 && c > 0 && c % 8 == 0,
                    "sur_cast_bf16_ex: need src, y, nvox % 8 == 0, c % 8 == 0");
    NSLGF_CHECK_ARG(a16(src) && a16(act) && a16(y) && a16(yb), "sur_cast_bf16_ex: tensors must be 16-byte aligned");
    if (nvox == 0) return NSLGF_OK;
    const float *x = (const float*)src, *a = (const float*)act;
    hipStream_t s = (hipStream_t)stream;
    // Tiles of 64 channels where they divide c, since a tile of 32 leaves half lines of y to the next workgroup (us at
    // 128^3, 64 channels, with the blocked copy: 219 in tiles of 32, 188 of 64; with act 378 and 295).
    const int wide = c % 64 == 0 ? 64 : 32, chunks = ceil_div(c, wide);
    const long long n4 = nvox * c / 4;
    const dim3 flat((unsigned)ceil_div(n4, 512));
    if (!yb && a)
        hipLaunchKernelGGL(k_cast_flat<true>, flat, dim3(256), 0, s, (const float4*)x, (const float4*)a, (uint2*)y, n4);
    else if (!yb)
        hipLaunchKernelGGL(k_cast_flat<false>, flat, dim3(256), 0, s, (const float4*)x, nullptr, (uint2*)y, n4);
    else if (wide == 64)
        hipLaunchKernelGGL(k_cast_blocked<64>, dim3((unsigned)(ceil_div(nvox, 64) * chunks)), dim3(256), 0, s, x, a,
                           (bf16_t*)y, (bf16_t*)yb, nvox, c, chunks);
    else
        hipLaunchKernelGGL(k_cast_blocked<32>, dim3((unsigned)(ceil_div(nvox, 128) * chunks)), dim3(256), 0, s, x, a,
                           (bf16_t*)y, (bf16_t*)yb, nvox, c, chunks);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_cast_bf16_up(nslgf_t h, const void* coarse, double scale, const void* skip, const void* act, void* y,
                     void* yb, int D, int H, int W, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(coarse && skip && y && D > 0 && H > 0 && W > 0 && D % 2 == 0 && H % 2 == 0 && W % 2 == 0 &&
                        c > 0 && c % 8 == 0 && ((long long)D * H * W) % 8 == 0,
                    "sur_cast_bf16_up: need coarse, skip, y, even D, H, W with D*H*W % 8 == 0, c % 8 == 0");
    NSLGF_CHECK_ARG(a16(coarse) && a16(skip) && a16(act) && a16(y) && a16(yb),
                    "sur_cast_bf16_up: tensors must be 16-byte aligned");
    const long long nvox = (long long)D * H * W;
    hipLaunchKernelGGL(k_cast_up, dim3(ceil_div(nvox / 8 * (c / 8), 256)), dim3(256), 0, (hipStream_t)stream,
                       (const float*)coarse, (float)scale, (const float*)skip, (const float*)act, (bf16_t*)y,
                       (bf16_t*)yb, nvox / 8, c, D, H, W);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_to_blocked8(nslgf_t h, const void* x, void* xb, long long nvox, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(x && xb && x != xb && nvox >= 0 && nvox % 8 == 0 && c > 0 && c % 8 == 0,
                    "sur_to_blocked8: need x != xb, nvox % 8 == 0, c % 8 == 0");
    NSLGF_CHECK_ARG(a16(x) && a16(xb), "sur_to_blocked8: tensors must be 16-byte aligned");
    if (nvox == 0) return NSLGF_OK;
    hipLaunchKernelGGL(k_to_blocked8, dim3(ceil_div(nvox / 8 * (c / 8), 256)), dim3(256), 0, (hipStream_t)stream,
                       (const bf16_t*)x, (bf16_t*)xb, nvox / 8, c);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_weight_transpose(nslgf_t h, const void* w, void* wt, int cin, int cout, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(w && wt && w != wt && cin > 0 && cout > 0, "sur_weight_transpose: bad arguments");
    const long long n = 27LL * cin * cout;
    hipLaunchKernelGGL(k_wtranspose, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const bf16_t*)w, (bf16_t*)wt,
                       cin, cout);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

#define SUR_ELEMWISE(call)                                                                         \
    SUR_ENTER(h);                                                                                  \
    NSLGF_CHECK_ARG(n >= 0, "surrogate: negative size");                                           \
    if (n == 0) return NSLGF_OK;                                                                   \
    call;                                                                                          \
    NSLGF_LAUNCH_CHECK();                                                                          \
    return NSLGF_OK;

int sur_cast_bf16(nslgf_t h, const void* x, void* y, long long n, void* stream) {
    SUR_ELEMWISE(hipLaunchKernelGGL(k_cast_bf16, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)x,
                                    (bf16_t*)y, n))
}
int sur_relu_bwd(nslgf_t h, const void* y, void* g, long long n, void* stream) {
    SUR_ELEMWISE(hipLaunchKernelGGL(k_relu_bwd, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)y,
                                    (float*)g, n))
}
int sur_add(nslgf_t h, const void* a, const void* b, void* o, long long n, void* stream) {
    SUR_ELEMWISE(hipLaunchKernelGGL(k_add, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)a,
                                    (const float*)b, (float*)o, n))
}

static int resample_ok(int D, int H, int W, int c) {
    NSLGF_CHECK_ARG(D >= 2 && H >= 2 && W >= 2 && D % 2 == 0 && H % 2 == 0 && W % 2 == 0 && c >= 1,
                    "surrogate: resampling needs even fine sizes");
    return NSLGF_OK;
}

int sur_pool2_fwd(nslgf_t h, const void* x, void* y, int D, int H, int W, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(resample_ok(D, H, W, c));
    const long long n = (long long)(D / 2) * (H / 2) * (W / 2) * c;
    hipLaunchKernelGGL(k_pool2_fwd, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)x, (float*)y, D, H,
                       W, c);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_pool2_bwd(nslgf_t h, const void* gy, void* gx, int D, int H, int W, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(resample_ok(D, H, W, c));
    const long long n = (long long)D * H * W * c;
    hipLaunchKernelGGL(k_pool2_bwd, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)gy, (float*)gx, D,
                       H, W, c);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_up2_fwd(nslgf_t h, const void* x, void* y, int D, int H, int W, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(resample_ok(D, H, W, c));
    const long long n = (long long)D * H * W * c;
    hipLaunchKernelGGL(k_up2_fwd, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)x, (float*)y, D, H, W,
                       c);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_up2_bwd(nslgf_t h, const void* gy, void* gx, int D, int H, int W, int c, void* stream) {
    SUR_ENTER(h);
    NSLGF_TRY(resample_ok(D, H, W, c));
    const long long n = (long long)(D / 2) * (H / 2) * (W / 2) * c;
    hipLaunchKernelGGL(k_up2_bwd, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const float*)gy, (float*)gx, D, H,
                       W, c);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_mse(nslgf_t h, const void* pred, const void* target, void* grad, void* partial, long long nvox, int c, int used,
            void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(pred && target && grad && partial && nvox > 0 && used >= 1 && used <= c, "sur_mse: bad arguments");
    int sh = 0;
    while (sh < 8 && (4 << sh) < c) ++sh;
    if ((4 << sh) == c && a16(grad))
        hipLaunchKernelGGL(k_mse<true>, dim3(1024), dim3(256), 0, (hipStream_t)stream, (const float*)pred,
                           (const float*)target, (float*)grad, (double*)partial, nvox, c, used, sh);
    else
        hipLaunchKernelGGL(k_mse<false>, dim3(1024), dim3(256), 0, (hipStream_t)stream, (const float*)pred,
                           (const float*)target, (float*)grad, (double*)partial, nvox, c, used, 0);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_mse_cast(nslgf_t h, const void* pred, const void* target, void* partial, void* y, void* yb, long long nvox,
                 int c, int used, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(pred && target && partial && y && nvox > 0 && nvox % 8 == 0 && c > 0 && c % 8 == 0 && used >= 1 &&
                        used <= c,
                    "sur_mse_cast: need pred, target, partial, y, nvox % 8 == 0, c % 8 == 0, 1 <= used <= c");
    NSLGF_CHECK_ARG(a16(y) && a16(yb), "sur_mse_cast: tensors must be 16-byte aligned");
    hipLaunchKernelGGL(k_mse_cast, dim3(1024), dim3(256), 0, (hipStream_t)stream, (const float*)pred,
                       (const float*)target, (bf16_t*)y, (bf16_t*)yb, (double*)partial, nvox, c, used);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_adam(nslgf_t h, void* w, void* wb, const void* g, void* m, void* v, long long n, float lr, float b1, float b2,
             float eps, int t, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(w && wb && g && m && v && n > 0 && t >= 1, "sur_adam: bad arguments");
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (float*)w, (bf16_t*)wb, (const float*)g,
                       (float*)m, (float*)v, n, lr, b1, b2, eps, c1, c2);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_pack_input(nslgf_t h, const void* om, void* x, int D, int H, int W, double scale, double feat, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(om && x && D > 0 && H > 0 && W > 0, "sur_pack_input: bad arguments");
    const long long nvox = (long long)D * H * W;
    hipLaunchKernelGGL(k_pack_input, dim3(grid1(nvox)), dim3(256), 0, (hipStream_t)stream, (const double*)om,
                       (bf16_t*)x, nvox, scale, feat);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_pack_input_pair(nslgf_t h, const void* om, const void* delta, void* x, int D, int H, int W, double scale,
                        double dscale, double feat, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(om && delta && x && D > 0 && H > 0 && W > 0, "sur_pack_input_pair: bad arguments");
    const long long nvox = (long long)D * H * W;
    hipLaunchKernelGGL(k_pack_input_pair, dim3(grid1(nvox)), dim3(256), 0, (hipStream_t)stream, (const double*)om,
                       (const double*)delta, (bf16_t*)x, nvox, scale, dscale, feat);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_combine3(nslgf_t h, const void* a, const void* b, const void* c, void* out, long long n, double ca, double cb,
                 double cc, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(a && b && out && n > 0, "sur_combine3: bad arguments");
    hipLaunchKernelGGL(k_combine3, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, (const double*)a,
                       (const double*)b, (const double*)c, (double*)out, n, ca, cb, cc);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_pack_target(nslgf_t h, const void* f, void* t, int D, int H, int W, double scale, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(f && t && D > 0 && H > 0 && W > 0, "sur_pack_target: bad arguments");
    const long long nvox = (long long)D * H * W;
    hipLaunchKernelGGL(k_pack_target, dim3(grid1(nvox)), dim3(256), 0, (hipStream_t)stream, (const double*)f, (float*)t,
                       nvox, scale);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int sur_unpack_update(nslgf_t h, const void* base, const void* y, void* out, int D, int H, int W, int c, double scale,
                      void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(base && y && out && c >= 3 && scale != 0.0, "sur_unpack_update: bad arguments");
    const long long nvox = (long long)D * H * W;
    hipLaunchKernelGGL(k_unpack_update, dim3(grid1(nvox)), dim3(256), 0, (hipStream_t)stream, (const double*)base,
                       (const float*)y, (double*)out, nvox, c, 1.0 / scale);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int sur_mfma_selftest(nslgf_t h, const void* a, const void* b, void* c, void* stream) {
    SUR_ENTER(h);
    NSLGF_CHECK_ARG(a && b && c, "sur_mfma_selftest: null pointer");
    hipLaunchKernelGGL(k_mfma_selftest, dim3(1), dim3(64), 0, (hipStream_t)stream, (const bf16_t*)a, (const bf16_t*)b,
                       (float*)c);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

}  // extern "C"
