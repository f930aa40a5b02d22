// Zero-padded FFT convolution passes of the LGF solve (Sec. 2.2, Eq. dpoisson_conv).
//
// The box convolution y = dx^2 g * s equals, on the box, the cyclic convolution of the zero-padded
// source with the LGF wrapped onto a padded lattice of P >= 2n - 1 points per axis.  One scalar
// solve is five passes over HBM:
//   1. rows along x: real -> half spectrum (P/2 + 1 complex), n_x inputs, the rest implicit zeros;
//   2. columns along y: forward, n_y nonzero inputs -> P outputs;
//   3. columns along z: forward (n_z nonzero inputs), times the real even kernel spectrum,
//      inverse, keeping the n_z box outputs -- all in registers, one HBM round trip;
//   4. columns along y: inverse, keeping the n_y box outputs;
//   5. rows along x: half spectrum -> real, keeping the n_x box outputs.
// Rows are contiguous; the column passes work on tiles of TB adjacent columns (one 128-byte
// segment per transform element) so that every global access is coalesced without transposes.
#include <cmath>
#include <vector>

#include "fft.h"
#include "kernels.h"
#include "pencil.h"

namespace nslgf {

// ---------------------------------------------------------------------------------------------------
// Masked divergence of a face field at (x, y, z), in the order of operations of the divergence kernel but summed
// in FP64 and rounded once: the field is nearly solenoidal, so the FP32 sum's rounding, of the size of the
// terms, is white noise far above that of the result's own rounding, and the Green's function amplifies its
// lowest modes (relative error of the FP32 pressure after a step at 96^3: Scheme A 1.7e-6 to 3.0e-6 with the FP32
// sum, 0.7e-6 to 1.2e-6 so; Scheme B 3.0e-6 to 6.9e-6, 1.2e-6 to 1.9e-6).
template <typename T>
__device__ __forceinline__ T masked_div_at(const T* f, int x, int y, int z, int nx, int ny, int nz, int nbuf,
                                           const unsigned char* blocks, int nb, T idx) {
    if (!in_domain(x, y, z, nx, ny, nz, nbuf, blocks, nb)) return (T)0;
    const long long n = (long long)nx * ny * nz;
    const long long c = ((long long)z * ny + y) * nx + x;
    const double f0m = x > 0 ? f[c - 1] : (T)0;
    const double f1m = y > 0 ? f[n + c - nx] : (T)0;
    const double f2m = z > 0 ? f[2 * n + c - (long long)nx * ny] : (T)0;
    return (T)(((double)f[c] + f[n + c] + f[2 * n + c] - f0m - f1m - f2m) * idx);
}

// PAIRS: the real rows are read as pairs (x[2n], x[2n+1]) with one vector load each (the host sets it
// when the base is aligned, rows and components have even lengths, and n_io is even).  DIV: the rows
// are the masked divergence of RowPass::div_src, formed on load.
// Batched form (da set): the workgroups of grid z index p take the arguments da[p].
template <typename T, int LH, bool PAIRS, bool DIV>
__global__ void __launch_bounds__(256) k_row_r2c(RowPass a0, const RowPass* __restrict__ da) {
    RowPass a = a0;
    if (da) a = da[blockIdx.z];
    using P = Plan1D<LH>;
    constexpr int E = P::E, TP = LH / E, RPW = row_rpw<T, LH>();
    using RL = typename P::Fwd;
    constexpr int LD = row_lds_len<T, LH>();
    __shared__ cplx<T> lds[RPW * LD];
    const int tid = threadIdx.x;
    const int rl = tid / TP, t = tid % TP;
    const long long row = (long long)blockIdx.x * (blockDim.x / TP) + rl;
    const int comp = blockIdx.y;
    const bool valid = row < a.nrows;
    const T* in = (const T*)a.in + comp * a.in_comp + (valid ? row : 0) * a.in_row;
    cplx<T>* out = (cplx<T>*)a.out + comp * a.out_comp + (valid ? row : 0) * a.out_row;
    // the half-length root table goes to LDS (read by the transform's passes after the barrier below)
    __shared__ cplx<T> twh[LH];
    for (int m = tid; m < LH; m += blockDim.x) twh[m] = ((const cplx<T>*)a.tw_half)[m];
    const cplx<T>* twf = (const cplx<T>*)a.tw_full;
    RowAcc<T> acc{lds + rl * LD};
    cplx<T> v[E];
    constexpr int R1 = First<RL>::value;
#pragma unroll
    for (int b = 0; b < E / R1; ++b) {
        const int j = t + b * TP;
#pragma unroll
        for (int r = 0; r < R1; ++r) {
            const int m = 2 * (j + r * (LH / R1));  // z[n] = x[2n] + i x[2n+1]
            if constexpr (DIV) {
                const int y = (int)(row % a.div_ny), z = (int)(row / a.div_ny);
                const T* f = (const T*)a.div_src;
                const T idx = (T)a.div_idx;
                const T re = (valid && m < a.n_io)
                                 ? masked_div_at<T>(f, m, y, z, a.n_io, a.div_ny, a.div_nz, a.div_nbuf, a.div_blocks, a.div_nb, idx)
                                 : (T)0;
                const T im = (valid && m + 1 < a.n_io)
                                 ? masked_div_at<T>(f, m + 1, y, z, a.n_io, a.div_ny, a.div_nz, a.div_nbuf, a.div_blocks, a.div_nb,
                                                   idx)
                                 : (T)0;
                v[b * R1 + r] = mk<T>(re, im);
            } else if constexpr (PAIRS) {
                v[b * R1 + r] = (valid && m < a.n_io) ? *(const cplx<T>*)(in + m) : mk<T>((T)0, (T)0);
            } else {
                const T re = (valid && m < a.n_io) ? in[m] : (T)0;
                const T im = (valid && m + 1 < a.n_io) ? in[m + 1] : (T)0;
                v[b * R1 + r] = mk<T>(re, im);
            }
        }
    }
    __syncthreads();
    fft_regs<T, LH, false, RL>(v, t, twh, acc);
    constexpr int RLs = Last<RL>::value;
    wave_sync();
#pragma unroll
    for (int b = 0; b < E / RLs; ++b) {
        const int j = t + b * TP;
#pragma unroll
        for (int r = 0; r < RLs; ++r) acc(j + r * (LH / RLs)) = v[b * RLs + r];
    }
    wave_sync();
    if (valid) {
        // X[k] = E[k] + W_P^k O[k], E = (Z[k] + conj Z[-k]) / 2, O = -i (Z[k] - conj Z[-k]) / 2
        for (int k = t; k < LH; k += TP) {
            const cplx<T> zk = acc(k);
            const cplx<T> zm = acc(k == 0 ? 0 : LH - k);
            const T ex = (T)0.5 * (zk.x + zm.x), ey = (T)0.5 * (zk.y - zm.y);
            const cplx<T> o = mk<T>((T)0.5 * (zk.y + zm.y), (T)-0.5 * (zk.x - zm.x));
            const cplx<T> wo = cmul<T>(twf[k], o);
            out[k] = mk<T>(ex + wo.x, ey + wo.y);
        }
        if (t == 0) {
            const cplx<T> z0 = acc(0);
            out[LH] = mk<T>(z0.x - z0.y, (T)0);
        }
    }
}

// PAIRS: the real outputs are written as pairs with one vector store each (conditions as for r2c).
template <typename T, int LH, bool PAIRS>
__global__ void __launch_bounds__(256) k_row_c2r(RowPass a0, const RowPass* __restrict__ da) {
    RowPass a = a0;
    if (da) a = da[blockIdx.z];
    using P = Plan1D<LH>;
    constexpr int E = P::E, TP = LH / E, RPW = row_rpw<T, LH>();
    using RL = Reverse<typename P::Fwd>;
    constexpr int LD = row_lds_len<T, LH>();
    __shared__ cplx<T> lds[RPW * LD];
    const int tid = threadIdx.x;
    const int rl = tid / TP, t = tid % TP;
    const long long row = (long long)blockIdx.x * (blockDim.x / TP) + rl;
    const int comp = blockIdx.y;
    const bool valid = row < a.nrows;
    const cplx<T>* in = (const cplx<T>*)a.in + comp * a.in_comp + (valid ? row : 0) * a.in_row;
    T* out = (T*)a.out + comp * a.out_comp + (valid ? row : 0) * a.out_row;
    __shared__ cplx<T> twh[LH];  // the half-length root table, in LDS from the first barrier on
    for (int m = tid; m < LH; m += blockDim.x) twh[m] = ((const cplx<T>*)a.tw_half)[m];
    const cplx<T>* twf = (const cplx<T>*)a.tw_full;
    RowAcc<T> acc{lds + rl * LD};
    for (int k = t; k <= LH; k += TP) acc(k) = valid ? in[k] : mk<T>((T)0, (T)0);
    __syncthreads();
    cplx<T> v[E];
    constexpr int R1 = First<RL>::value;
#pragma unroll
    for (int b = 0; b < E / R1; ++b) {
        const int j = t + b * TP;
#pragma unroll
        for (int r = 0; r < R1; ++r) {
            const int k = j + r * (LH / R1);
            const cplx<T> xk = acc(k), xm = acc(LH - k);
            // Z = (X[k] + conj X[LH-k]) + i W_P^{-k} (X[k] - conj X[LH-k])
            const cplx<T> d = mk<T>(xk.x - xm.x, xk.y + xm.y);
            const cplx<T> o = cmulc<T>(d, twf[k]);
            v[b * R1 + r] = mk<T>(xk.x + xm.x - o.y, xk.y - xm.y + o.x);
        }
    }
    fft_regs<T, LH, true, RL>(v, t, twh, acc);
    constexpr int RLs = Last<RL>::value;
    if (valid) {
#pragma unroll
        for (int b = 0; b < E / RLs; ++b) {
            const int j = t + b * TP;
#pragma unroll
            for (int r = 0; r < RLs; ++r) {
                const int m = 2 * (j + r * (LH / RLs));
                if constexpr (PAIRS) {
                    if (m < a.n_io) *(cplx<T>*)(out + m) = v[b * RLs + r];
                } else {
                    if (m < a.n_io) out[m] = v[b * RLs + r].x;
                    if (m + 1 < a.n_io) out[m + 1] = v[b * RLs + r].y;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------
static const int kLengths[] = {16, 32, 48, 64, 96, 128, 160, 192, 256, 320, 384, 512};

bool fft_length_supported(int P) {
    for (int L : kLengths)
        if (L == P) return true;
    return false;
}

int next_supported_length(int n) {
    for (int L : kLengths)
        if (L >= n) return L;
    return -1;
}

template <int L> static int tb_of(int dtype) {
    return dtype == NSLGF_F32 ? pencil_cols<float, L>() : pencil_cols<double, L>();
}

int col_tile_width(int L, int dtype) {
    switch (L) {
#define NSLGF_CASE(L_) case L_: return tb_of<L_>(dtype);
        NSLGF_CASE(16) NSLGF_CASE(32) NSLGF_CASE(48) NSLGF_CASE(64) NSLGF_CASE(96) NSLGF_CASE(128)
        NSLGF_CASE(160) NSLGF_CASE(192) NSLGF_CASE(256) NSLGF_CASE(320) NSLGF_CASE(384) NSLGF_CASE(512)
#undef NSLGF_CASE
    }
    return -1;
}

int make_twiddles(int L, int dtype, void** dev_out) {
    const size_t esz = 2 * dtype_size(dtype);
    std::vector<unsigned char> host(esz * L);
    const long double two_pi = 6.283185307179586476925286766559005768L;
    for (int m = 0; m < L; ++m) {
        // exp(-2 pi i m / L) evaluated in extended precision and rounded once to the dtype
        // (accurately rounded twiddles); the exact quarter-period values are set directly
        const long double ang = two_pi * (long double)m / (long double)L;
        long double c = cosl(ang), s = sinl(ang);
        if (m == 0) { c = 1; s = 0; }
        if (4 * m == L) { c = 0; s = 1; }
        if (2 * m == L) { c = -1; s = 0; }
        if (4 * m == 3 * L) { c = 0; s = -1; }
        if (dtype == NSLGF_F32) {
            float* p = (float*)host.data();
            p[2 * m] = (float)c;
            p[2 * m + 1] = (float)-s;
        } else {
            double* p = (double*)host.data();
            p[2 * m] = (double)c;
            p[2 * m + 1] = (double)-s;
        }
    }
    void* d = nullptr;
    if (hipMalloc(&d, host.size()) != hipSuccess) {
        set_error("hipMalloc(twiddles) failed");
        return NSLGF_ENOMEM;
    }
    NSLGF_HIP_CHECK(hipMemcpy(d, host.data(), host.size(), hipMemcpyHostToDevice));
    *dev_out = d;
    return NSLGF_OK;
}

LaunchRecorder*& launch_recorder() {
    static thread_local LaunchRecorder* r = nullptr;
    return r;
}

// Batched launches of the row and column passes: nprob problems' argument tables, one problem's grid.
template <typename T, int LH, bool PAIRS, bool DIV>
static int batched_r2c(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_row_r2c<T, LH, PAIRS, DIV>), dim3(g.x, g.y, nprob), b, 0, s, RowPass{}, (const RowPass*)args);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T, int LH, bool PAIRS>
static int batched_c2r(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_row_c2r<T, LH, PAIRS>), dim3(g.x, g.y, nprob), b, 0, s, RowPass{}, (const RowPass*)args);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T, int L, int MODE, bool HALF>
static int batched_col(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    if (MODE == COL_CONV)
        hipLaunchKernelGGL((k_pencil<T, L, MODE, HALF>), dim3(g.x * nprob), b, 0, s, ColPass{}, (const ColPass*)args,
                           (int)g.x);
    else
        hipLaunchKernelGGL((k_pencil<T, L, MODE, HALF>), dim3(g.x, g.y, g.z * nprob), b, 0, s, ColPass{},
                           (const ColPass*)args, (int)g.z);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

template <typename T, int LH, bool PAIRS, bool DIV> static int issue_r2c(const RowPass& a, dim3 grid, dim3 block,
                                                                          hipStream_t s) {
    if (launch_recorder()) {
        record_launch(&batched_r2c<T, LH, PAIRS, DIV>, grid, block, a);
        return NSLGF_OK;
    }
    hipLaunchKernelGGL((k_row_r2c<T, LH, PAIRS, DIV>), grid, block, 0, s, a, nullptr);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T, int L, int MODE, bool HALF> static int issue_col(const ColPass& a, dim3 grid, dim3 block,
                                                                       hipStream_t s) {
    if (launch_recorder()) {
        record_launch(&batched_col<T, L, MODE, HALF>, grid, block, a);
        return NSLGF_OK;
    }
    hipLaunchKernelGGL((k_pencil<T, L, MODE, HALF>), grid, block, 0, s, a, nullptr, 0);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

template <typename T> static bool real_pairs(const void* p, long long row, long long comp, int n_io) {
    return ((uintptr_t)p % (2 * sizeof(T))) == 0 && row % 2 == 0 && comp % 2 == 0 && n_io % 2 == 0;
}
// Rows of a workgroup: one wave's worth where the launch is at most a wave a SIMD, so that it spreads over the
// CUs (32^3 solve, 64 waves: the two row passes 5.2 and 5.6 us in workgroups of four waves with a barrier at each
// exchange, 4.6 and 4.8 so, where the exchanges are a wave's own); full workgroups share the twiddle table.
template <typename T, int LH> static int row_rows(const RowPass& a) {
    constexpr int TP = LH / Plan1D<LH>::E, RPW = row_rpw<T, LH>();
    return a.nrows * a.ncomp * TP <= 1024 * 64 && RPW > 64 / TP ? 64 / TP : RPW;
}
template <typename T, int LH> static int do_r2c(const RowPass& a, hipStream_t s) {
    constexpr int TP = LH / Plan1D<LH>::E;
    const int RPW = row_rows<T, LH>(a);
    dim3 grid(ceil_div(a.nrows, RPW), a.ncomp);
    if (a.div_src) {
        if (a.ncomp != 1 || a.nrows != (long long)a.div_ny * a.div_nz) {
            set_error("row pass: the divergence input needs one component over ny * nz rows");
            return NSLGF_EINVAL;
        }
        return issue_r2c<T, LH, false, true>(a, grid, dim3(RPW * TP), s);
    }
    if (real_pairs<T>(a.in, a.in_row, a.in_comp, a.n_io)) return issue_r2c<T, LH, true, false>(a, grid, dim3(RPW * TP), s);
    return issue_r2c<T, LH, false, false>(a, grid, dim3(RPW * TP), s);
}
template <typename T, int LH> static int do_c2r(const RowPass& a, hipStream_t s) {
    constexpr int TP = LH / Plan1D<LH>::E;
    const int RPW = row_rows<T, LH>(a);
    dim3 grid(ceil_div(a.nrows, RPW), a.ncomp);
    const bool pairs = real_pairs<T>(a.out, a.out_row, a.out_comp, a.n_io);
    if (launch_recorder()) {
        record_launch(pairs ? &batched_c2r<T, LH, true> : &batched_c2r<T, LH, false>, grid, dim3(RPW * TP), a);
        return NSLGF_OK;
    }
    if (pairs)
        hipLaunchKernelGGL((k_row_c2r<T, LH, true>), grid, dim3(RPW * TP), 0, s, a, nullptr);
    else
        hipLaunchKernelGGL((k_row_c2r<T, LH, false>), grid, dim3(RPW * TP), 0, s, a, nullptr);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T, int L, int MODE> static int do_col(const ColPass& a, hipStream_t s) {
    if (a.nouter > 65535 || a.ncomp > 65535) {
        set_error("column pass grid too large");
        return NSLGF_EINVAL;
    }
    dim3 grid(ceil_div(a.ncols, pencil_cols<T, L>()), a.nouter, a.ncomp);
    const dim3 block(64 * pencil_waves<L>());
    const bool half_in = 2 * a.n_in <= L, half_out = 2 * a.n_out <= L;
    if constexpr (MODE == COL_CONV) {
        grid = dim3(grid.x * grid.y * grid.z);
        if (!half_in || !half_out) {
            set_error("column pass: the fused pass needs n_in, n_out <= L/2");
            return NSLGF_EINVAL;
        }
        return issue_col<T, L, MODE, true>(a, grid, block, s);
    } else {
        if (MODE == COL_FWD ? half_in : half_out) return issue_col<T, L, MODE, true>(a, grid, block, s);
        return issue_col<T, L, MODE, false>(a, grid, block, s);
    }
}

#define NSLGF_ROW_SWITCH(FN, T)                                                                    \
    switch (P) {                                                                                   \
        case 16: return FN<T, 8>(a, s);                                                            \
        case 32: return FN<T, 16>(a, s);                                                           \
        case 48: return FN<T, 24>(a, s);                                                           \
        case 64: return FN<T, 32>(a, s);                                                           \
        case 96: return FN<T, 48>(a, s);                                                           \
        case 128: return FN<T, 64>(a, s);                                                          \
        case 160: return FN<T, 80>(a, s);                                                          \
        case 192: return FN<T, 96>(a, s);                                                          \
        case 256: return FN<T, 128>(a, s);                                                         \
        case 320: return FN<T, 160>(a, s);                                                         \
        case 384: return FN<T, 192>(a, s);                                                         \
        case 512: return FN<T, 256>(a, s);                                                         \
    }

int launch_row_r2c(int P, int dtype, const RowPass& a, hipStream_t s) {
    if (dtype == NSLGF_F32) {
        NSLGF_ROW_SWITCH(do_r2c, float)
    } else {
        NSLGF_ROW_SWITCH(do_r2c, double)
    }
    set_error("unsupported padded length " + std::to_string(P));
    return NSLGF_EUNSUPPORTED;
}

int launch_row_c2r(int P, int dtype, const RowPass& a, hipStream_t s) {
    if (dtype == NSLGF_F32) {
        NSLGF_ROW_SWITCH(do_c2r, float)
    } else {
        NSLGF_ROW_SWITCH(do_c2r, double)
    }
    set_error("unsupported padded length " + std::to_string(P));
    return NSLGF_EUNSUPPORTED;
}

#define NSLGF_COL_SWITCH(T, MODE)                                                                  \
    switch (L) {                                                                                   \
        case 16: return do_col<T, 16, MODE>(a, s);                                                 \
        case 32: return do_col<T, 32, MODE>(a, s);                                                 \
        case 48: return do_col<T, 48, MODE>(a, s);                                                 \
        case 64: return do_col<T, 64, MODE>(a, s);                                                 \
        case 96: return do_col<T, 96, MODE>(a, s);                                                 \
        case 128: return do_col<T, 128, MODE>(a, s);                                               \
        case 160: return do_col<T, 160, MODE>(a, s);                                               \
        case 192: return do_col<T, 192, MODE>(a, s);                                               \
        case 256: return do_col<T, 256, MODE>(a, s);                                               \
        case 320: return do_col<T, 320, MODE>(a, s);                                               \
        case 384: return do_col<T, 384, MODE>(a, s);                                               \
        case 512: return do_col<T, 512, MODE>(a, s);                                               \
    }

template <typename T> static int col_dispatch(int L, ColMode mode, const ColPass& a, hipStream_t s) {
    if (mode == COL_FWD) {
        NSLGF_COL_SWITCH(T, COL_FWD)
    } else if (mode == COL_INV) {
        NSLGF_COL_SWITCH(T, COL_INV)
    } else {
        NSLGF_COL_SWITCH(T, COL_CONV)
    }
    set_error("unsupported transform length " + std::to_string(L));
    return NSLGF_EUNSUPPORTED;
}

int launch_col(int L, int dtype, ColMode mode, const ColPass& a, hipStream_t s) {
    return dtype == NSLGF_F32 ? col_dispatch<float>(L, mode, a, s) : col_dispatch<double>(L, mode, a, s);
}

bool col_variant_valid(int L, int v) { return L == 512 || L == 256 ? v >= 0 && v <= 2 : v == 0; }

// The plan number reported for a length, dtype and pass: a valid choice >= 0, else the default's number.
int col_variant_choice(int L, int dtype, int choice, bool zpass) {
    if (choice >= 0 && col_variant_valid(L, choice)) return choice;
    if (L != 512 && L != 256) return 0;
    if (dtype == NSLGF_F32) return zpass ? 1 : 0;
    return L == 512 ? 2 : 0;
}

}  // namespace nslgf
