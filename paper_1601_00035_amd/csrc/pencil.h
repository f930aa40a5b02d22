// Column (strided) FFT passes of the convolution: one kernel for every length.
//
// A length L = 8 R2 R3 transform is three radix passes over the digits of n = (R2 R3) a + R3 b + c
// (a < 8, b < R2, c < R3), k = k0 + 8 k1 + 8 R2 k2.  A workgroup takes a tile of 64 / R2 slots of
// 16 bytes (one complex double, or two neighbouring complex floats) and its digits are laid out so that
// only one exchange per transform leaves the wavefront:
//   pass 1  wave c, lane (b, slot), registers a -> k0;      exchange within the wave: b <-> k0
//   pass 2  wave c, lane (k0, slot), registers b -> k1;     exchange across waves:    c <-> k1
//   pass 3  wave k1, lane (k0, slot), registers c -> k2.
// (For R2 < 8 a lane holds 8 / R2 values of k0; for small R3 a wave of pass 3 takes several k1.)
// The inverse alone is the same with conjugate roots; behind the spectrum multiply it runs the passes
// backwards.  The exchange within a wave needs no barrier; the one across waves is written to a wave's own
// LDS region and read from the others', and the backward passes put their values back where the thread
// read them, so a whole forward, multiply, inverse takes two barriers (eight when every exchange left the
// wave).
//
// What bounds it: the y passes run at 4.7 to 5.2 TB/s of their algorithmic bytes at 256^3, the rate of a large
// copy (5.2), so memory; the fused z pass at 3.7 to 3.9 in FP64 and 3.4 in FP32, memory and, since a workgroup
// waits for all of its loads before it starts, their latency; the boxes that stay in the last-level cache are
// bound by LDS and issue.  Before (Stockham passes whose every exchange crossed the workgroup; lengths 320 and
// 384 in five passes through half-size LDS tiles) and now, fused z pass within a solve, us per launch of one /
// three components: FP64 256^3 359 / 975 -> 328 / 878, 192^3 196 / 554 -> 151 / 432, 160^3 115 / 323 -> 87 / 256;
// FP32 256^3 222 / 602 -> 176 / 501, 192^3 127 / 375 -> 75 / 239, 160^3 66 / 193 -> 44 / 137.  (At 256^3 in FP64
// the y inverse then takes 160 / 472 us instead of 153 / 455: it waits for the z pass's writes to drain.)
// Measured and left out: one resident grid that loads its next tile ahead (the compiler keeps the twiddles
// in registers and spills: 300 -> 665 us at 512; no gain where it does not spill), and column chunks small
// enough for the last-level cache (no faster: each chunk's launches are too small).
#pragma once

#include "fft.h"
#include "kernels.h"

namespace nslgf {

// Digits of each length; W3: waves of pass 3, each holding 8 / W3 transforms of radix R3 per lane.
template <int L> struct Pencil;
#define NSLGF_PENCIL(L_, R2_, R3_, W3_)                                                            \
    template <> struct Pencil<L_> {                                                                \
        static constexpr int R2 = R2_, R3 = R3_, W3 = W3_;                                         \
        static_assert(8 * R2 * R3 == L_, "digits");                                                \
    };
NSLGF_PENCIL(16, 2, 1, 1)
NSLGF_PENCIL(32, 4, 1, 1)
NSLGF_PENCIL(48, 2, 3, 4)
NSLGF_PENCIL(64, 8, 1, 1)
NSLGF_PENCIL(96, 4, 3, 4)
NSLGF_PENCIL(128, 8, 2, 2)
NSLGF_PENCIL(160, 4, 5, 8)
NSLGF_PENCIL(192, 8, 3, 4)
NSLGF_PENCIL(256, 8, 4, 4)
NSLGF_PENCIL(320, 8, 5, 8)
NSLGF_PENCIL(384, 8, 6, 8)
NSLGF_PENCIL(512, 8, 8, 8)
#undef NSLGF_PENCIL

// Columns per slot and per tile.
template <typename T> __host__ __device__ constexpr int slot_cols() { return sizeof(T) == 8 ? 1 : 2; }
template <typename T, int L> __host__ __device__ constexpr int pencil_cols() { return 64 / Pencil<L>::R2 * slot_cols<T>(); }
template <int L> __host__ __device__ constexpr int pencil_waves() {
    return Pencil<L>::R3 > Pencil<L>::W3 ? Pencil<L>::R3 : Pencil<L>::W3;
}

template <typename T> struct alignas(16) Slot {
    cplx<T> c[sizeof(T) == 8 ? 1 : 2];
};

template <typename T, int R, bool INV, int PRUNE = 0> __device__ __forceinline__ void dft(cplx<T>* v) {
    if constexpr (R == 1) {
    } else if constexpr (PRUNE == 1) {
        DFTHalfIn<T, R, INV>::run(v);
    } else if constexpr (PRUNE == 2) {
        DFTHalfOut<T, R, INV>::run(v);
    } else {
        DFT<T, R, INV>::run(v);
    }
}

// One tile of one pass.  FWD: n_in inputs (the rest zero) -> L outputs; INV: L inputs -> the first n_out
// outputs; CONV: forward, times the spectrum, inverse, in registers.  HALF: n_in <= L/2 (FWD, CONV) and
// n_out <= L/2 (INV, CONV), so the first or last butterflies do half the work.
// Batched form (da set): one problem spans `per` consecutive values of the grid's z index (FWD, INV:
// its components) or of the logical workgroup index (CONV) and takes the arguments da[p].
template <typename T, int L, int MODE, bool HALF>
__global__ void __launch_bounds__(64 * pencil_waves<L>()) __attribute__((amdgpu_waves_per_eu(4)))
k_pencil(ColPass a0, const ColPass* __restrict__ da, int per) {
    constexpr int R2 = Pencil<L>::R2, R3 = Pencil<L>::R3, W3 = Pencil<L>::W3, NW = pencil_waves<L>();
    constexpr int V = slot_cols<T>(), CB = 64 / R2, KL = 8 / R2, BF = 8 / W3, TB = CB * V;
    constexpr int NTW2 = (R2 - 1) * 8, NTW3 = (R3 - 1) * 8 * R2;
    __shared__ Slot<T> lds[R3 * 512];
    __shared__ cplx<T> tw2[NTW2 > 0 ? NTW2 : 1], tw3[NTW3 > 0 ? NTW3 : 1];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    int tile, outer, comp;
    ColPass a = a0;
    if constexpr (MODE == COL_CONV) {
        const int n = (int)gridDim.x, b = (int)blockIdx.x, x = b % 8;
        int lg = x * (n / 8) + min(x, n % 8) + b / 8;
        if (da) {
            a = da[lg / per];
            lg %= per;
        }
        comp = lg % a.ncomp;
        const int rest = lg / a.ncomp;
        const int sq = rest % a.nouter;
        tile = rest / a.nouter;
        outer = (sq & 1) ? a.nouter - 1 - (sq >> 1) : (sq >> 1);
    } else {
        // Consecutive workgroups go to different XCDs.  The forward pass writes twice what it reads: on launches
        // beyond the caches, groups of 4 tiles (512 bytes of every row) on one XCD make it 6 % faster (531 -> 501 us,
        // three FP64 components at 256^3, the solve 2348 -> 2340 us); on small ones they leave XCDs idle (54 x 26 x 79,
        // three components: 10.0 us grouped, 5.2 in the plain order), and at 128^3 to 192^3 the two are alike.  The
        // inverse gains nothing and keeps the plain order.
        constexpr int GRP = MODE == COL_FWD ? 4 : 1;
        const int nt = (int)gridDim.x, n = nt * (int)gridDim.y * (int)gridDim.z;
        int lg = (int)blockIdx.x + nt * ((int)blockIdx.y + (int)gridDim.y * (int)blockIdx.z);
        const int g = lg / (8 * GRP), r = lg % (8 * GRP);
        if (n >= 8192 && (g + 1) * 8 * GRP <= n) lg = g * 8 * GRP + (r % 8) * GRP + r / 8;
        tile = lg % nt;
        lg /= nt;
        outer = lg % (int)gridDim.y;
        comp = lg / (int)gridDim.y;
        if (da) {
            a = da[comp / per];
            comp %= per;
        }
    }
    // lane = (row digit, slot): the row digit is b in pass 1, the low digit of k0 in passes 2 and 3
    const int dl = lane / CB, col = tile * TB + (lane % CB) * V;
    const bool valid = col < a.ncols;
    const cplx<T>* in = (const cplx<T>*)a.in + comp * a.in_comp + (long long)outer * a.in_outer + (valid ? col : 0);
    cplx<T>* out = (cplx<T>*)a.out + comp * a.out_comp + (long long)outer * a.out_outer + (valid ? col : 0);
    Slot<T>* const own = lds + wave * 512;
    Slot<T> v[8], u[R3 * BF];
    auto zero = [](Slot<T>& s) {
#pragma unroll
        for (int i = 0; i < V; ++i) s.c[i] = mk<T>((T)0, (T)0);
    };
    auto load = [&](int row, int n, Slot<T>& s) {
        if (valid && row < n)
            s = *(const Slot<T>*)(in + (long long)row * a.in_row);
        else
            zero(s);
    };
    // ---- twiddles of passes 2 and 3, in the order their lanes read them
    constexpr int NT2 = (NTW2 + 64 * NW - 1) / (64 * NW), NT3 = (NTW3 + 64 * NW - 1) / (64 * NW);
    cplx<T> t2[NT2 > 0 ? NT2 : 1], t3[NT3 > 0 ? NT3 : 1];
#pragma unroll
    for (int i = 0; i < NT2; ++i) {
        const int e = min(tid + i * 64 * NW, NTW2 - 1);
        t2[i] = ((const cplx<T>*)a.tw)[(e / 8 + 1) * (e % 8) * R3];
    }
#pragma unroll
    for (int i = 0; i < NT3; ++i) {
        const int e = min(tid + i * 64 * NW, NTW3 - 1);
        t3[i] = ((const cplx<T>*)a.tw)[(e / (8 * R2) + 1) * (e % (8 * R2))];
    }
    // ---- loads in the layout of the first pass
    constexpr int NIN = MODE != COL_INV && HALF ? 4 : 8;
    if (wave < R3) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i >= NIN)
                zero(v[i]);
            else
                load(i * R2 * R3 + dl * R3 + wave, a.n_in, v[i]);
        }
    }
    constexpr bool LOW = MODE == COL_INV && HALF && prunable<R3>();  // pass 3 gives its lower half only
    T kv[MODE == COL_CONV ? R3 * BF * V : 1];
    if constexpr (MODE == COL_CONV) {
        if (wave < W3) {
            const int kyf = min(outer, a.outer_period - outer);
            const T* kh = (const T*)a.khat + ((long long)kyf * a.khat_tiles + tile) * (L / 2 + 1) * TB + (lane % CB) * V;
#pragma unroll
            for (int j = 0; j < BF; ++j) {
                const int q = wave + W3 * j, k01 = dl + R2 * (q % KL) + 8 * (q / KL);
#pragma unroll
                for (int k2 = 0; k2 < R3; ++k2) {
                    const int k = k01 + 8 * R2 * k2;
                    const T* kp = kh + min(k, L - k) * TB;
                    if constexpr (V == 2) {
                        const cplx<T> t = *(const cplx<T>*)kp;
                        kv[(j * R3 + k2) * 2] = t.x;
                        kv[(j * R3 + k2) * 2 + 1] = t.y;
                    } else {
                        kv[j * R3 + k2] = *kp;
                    }
                }
            }
        }
    }
    // (the pointers come from the arguments or from the batch's table, which the compiler addresses generically; such
    // loads count with the LDS operations too, so these writes wait for the data and the spectrum)
#pragma unroll
    for (int i = 0; i < NT2; ++i)
        if (tid + i * 64 * NW < NTW2) tw2[tid + i * 64 * NW] = t2[i];
#pragma unroll
    for (int i = 0; i < NT3; ++i)
        if (tid + i * 64 * NW < NTW3) tw3[tid + i * 64 * NW] = t3[i];
    __syncthreads();
    auto mul2 = [&](Slot<T>& s, const cplx<T> w, bool inv) {
#pragma unroll
        for (int i = 0; i < V; ++i) s.c[i] = inv ? cmulc<T>(s.c[i], w) : cmul<T>(s.c[i], w);
    };
    constexpr bool INV = MODE == COL_INV;  // the inverse alone: the same passes with the conjugate roots
    {
        if (wave < R3) {
            // pass 1, exchange b <-> k0 (rows of 64 slots per k0, rotated so that the reads spread over the banks)
#pragma unroll
            for (int i = 0; i < V; ++i) {
                cplx<T> x[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) x[r] = v[r].c[i];
                dft<T, 8, INV, NIN == 4 ? 1 : 0>(x);
#pragma unroll
                for (int r = 0; r < 8; ++r) v[r].c[i] = x[r];
            }
            if constexpr (R2 > 1) {
#pragma unroll
                for (int r = 0; r < 8; ++r) own[r * 64 + ((dl ^ (r % R2)) * CB + lane % CB)] = v[r];
                wave_sync();
#pragma unroll
                for (int b = 0; b < R2; ++b)
#pragma unroll
                    for (int kl = 0; kl < KL; ++kl)
                        v[b * KL + kl] = own[(dl + R2 * kl) * 64 + (b ^ dl) * CB + lane % CB];
                wave_sync();
                // pass 2
#pragma unroll
                for (int kl = 0; kl < KL; ++kl) {
#pragma unroll
                    for (int b = 1; b < R2; ++b) mul2(v[b * KL + kl], tw2[(b - 1) * 8 + dl + R2 * kl], INV);
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        cplx<T> x[R2];
#pragma unroll
                        for (int b = 0; b < R2; ++b) x[b] = v[b * KL + kl].c[i];
                        dft<T, R2, INV>(x);
#pragma unroll
                        for (int b = 0; b < R2; ++b) v[b * KL + kl].c[i] = x[b];
                    }
                }
            }
            if constexpr (R3 > 1) {
#pragma unroll
                for (int q = 0; q < 8; ++q) own[q * 64 + lane] = v[q];
            }
        }
        if constexpr (R3 > 1) {
            __syncthreads();
            if (wave < W3) {
#pragma unroll
                for (int j = 0; j < BF; ++j) {
                    const int q = wave + W3 * j, m = dl + R2 * (q % KL) + 8 * (q / KL);
#pragma unroll
                    for (int c = 0; c < R3; ++c) u[j * R3 + c] = lds[c * 512 + q * 64 + lane];
#pragma unroll
                    for (int c = 1; c < R3; ++c) mul2(u[j * R3 + c], tw3[(c - 1) * 8 * R2 + m], INV);
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        cplx<T> x[R3];
#pragma unroll
                        for (int c = 0; c < R3; ++c) x[c] = u[j * R3 + c].c[i];
                        dft<T, R3, INV, LOW ? 2 : 0>(x);
#pragma unroll
                        for (int c = 0; c < R3; ++c) u[j * R3 + c].c[i] = x[c];
                    }
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) u[q] = v[q];
        }
    }
    if constexpr (MODE == COL_CONV) {
        if (wave < W3) {
            const T sc = (T)a.scale;
#pragma unroll
            for (int e = 0; e < R3 * BF; ++e)
#pragma unroll
                for (int i = 0; i < V; ++i) u[e].c[i] = cscale<T>(u[e].c[i], kv[e * V + i] * sc);
        }
    }
    if constexpr (MODE != COL_CONV) {
        if (wave < W3 && valid) {
#pragma unroll
            for (int j = 0; j < BF; ++j) {
                const int q = wave + W3 * j, k01 = dl + R2 * (q % KL) + 8 * (q / KL);
#pragma unroll
                for (int k2 = 0; k2 < (LOW ? R3 / 2 : R3); ++k2) {
                    const int row = k01 + 8 * R2 * k2;
                    if (row < a.n_out) *(Slot<T>*)(out + (long long)row * a.out_row) = u[j * R3 + k2];
                }
            }
        }
    } else {
        // ---- the fused pass's inverse: pass 3 backwards, written to the places the forward transform read
        if constexpr (R3 > 1) {
            if (wave < W3) {
#pragma unroll
                for (int j = 0; j < BF; ++j) {
                    const int q = wave + W3 * j, m = dl + R2 * (q % KL) + 8 * (q / KL);
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        cplx<T> x[R3];
#pragma unroll
                        for (int c = 0; c < R3; ++c) x[c] = u[j * R3 + c].c[i];
                        dft<T, R3, true>(x);
#pragma unroll
                        for (int c = 0; c < R3; ++c) u[j * R3 + c].c[i] = x[c];
                    }
#pragma unroll
                    for (int c = 1; c < R3; ++c) mul2(u[j * R3 + c], tw3[(c - 1) * 8 * R2 + m], true);
#pragma unroll
                    for (int c = 0; c < R3; ++c) lds[c * 512 + q * 64 + lane] = u[j * R3 + c];
                }
            }
            __syncthreads();
        }
        if (wave < R3) {
            if constexpr (R3 > 1) {
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = own[q * 64 + lane];
                wave_sync();
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = u[q];
            }
            if constexpr (R2 > 1) {
                // pass 2 backwards, exchange k0 <-> b
#pragma unroll
                for (int kl = 0; kl < KL; ++kl) {
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        cplx<T> x[R2];
#pragma unroll
                        for (int b = 0; b < R2; ++b) x[b] = v[b * KL + kl].c[i];
                        dft<T, R2, true>(x);
#pragma unroll
                        for (int b = 0; b < R2; ++b) v[b * KL + kl].c[i] = x[b];
                    }
#pragma unroll
                    for (int b = 1; b < R2; ++b) mul2(v[b * KL + kl], tw2[(b - 1) * 8 + dl + R2 * kl], true);
                }
#pragma unroll
                for (int b = 0; b < R2; ++b)
#pragma unroll
                    for (int kl = 0; kl < KL; ++kl)
                        own[(dl + R2 * kl) * 64 + (b ^ dl) * CB + lane % CB] = v[b * KL + kl];
                wave_sync();
#pragma unroll
                for (int r = 0; r < 8; ++r) v[r] = own[r * 64 + ((dl ^ (r % R2)) * CB + lane % CB)];
            }
#pragma unroll
            for (int i = 0; i < V; ++i) {
                cplx<T> x[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) x[r] = v[r].c[i];
                dft<T, 8, true, HALF ? 2 : 0>(x);
#pragma unroll
                for (int r = 0; r < 8; ++r) v[r].c[i] = x[r];
            }
            if (valid) {
#pragma unroll
                for (int i = 0; i < (HALF ? 4 : 8); ++i) {
                    const int row = i * R2 * R3 + dl * R3 + wave;
                    if (row < a.n_out) *(Slot<T>*)(out + (long long)row * a.out_row) = v[i];
                }
            }
        }
    }
}

}  // namespace nslgf
