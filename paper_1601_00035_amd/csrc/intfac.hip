// Integrating factor E(alpha) (Sec. 2.3): the kernel of the discrete heat semigroup is the product
// of three 1D factors w[k] = e^{-2 alpha} I_k(2 alpha) (Appendix B, Eq. lgf_intfac), so
// M E(alpha) M is applied as three masked 1D convolutions, one per axis, each reading its input
// with zero extension outside the box.  Every pass reads and writes each element of HBM once with
// coalesced accesses: rows through LDS for x, register windows over adjacent x-columns for y and z.
#include <algorithm>
#include <cmath>

#include "kernels.h"

namespace nslgf {

int if_weights(double alpha, int dtype, double* w, int wmax) {
    if (!(alpha >= 0.0) || !std::isfinite(alpha)) {
        set_error("if_apply: alpha must be a finite value >= 0");
        return -1;
    }
    if (alpha == 0.0) {
        w[0] = 1.0;
        return 0;
    }
    // I_k(2a) = sum_j a^{2j+k} / (j! (j+k)!), all terms positive; scaled by e^{-2a}
    const int kmax = 200;
    double vals[kmax + 1];
    const double ea = exp(-2.0 * alpha);
    double lead = 1.0;  // a^k / k!
    int last = kmax;    // (values below 1e-40 of the first change no sum)
    for (int k = 0; k <= kmax; ++k) {
        if (k > 0) lead *= alpha / k;
        double term = lead, sum = lead;
        for (int j = 1; j < 400; ++j) {
            term *= alpha * alpha / ((double)j * (double)(j + k));
            sum += term;
            if (term < 1e-19 * sum) break;
        }
        vals[k] = ea * sum;
        if (vals[k] < 1e-40 * vals[0]) {
            last = k;
            break;
        }
    }
    // smallest radius whose two-sided tail is below a quarter of the dtype's unit roundoff times w[0]
    const double tol = (dtype == NSLGF_F32 ? 5.960464477539063e-08 : 1.1102230246251565e-16) * 0.25 * vals[0];
    double tail = 0.0;
    int r = kmax;
    for (int k = last; k >= 1; --k) {
        if (2.0 * (tail + vals[k]) > tol) {
            r = k;
            break;
        }
        tail += vals[k];
    }
    if (r > wmax || r >= kmax) {
        set_error("if_apply: alpha too large for the supported kernel radius");
        return -1;
    }
    for (int k = 0; k <= r; ++k) w[k] = vals[k];
    return r;
}

struct IfWeights {
    double w[kIfMaxRadius + 1];
};

// x pass: whole rows staged in LDS (RPW rows of length nx per workgroup), each output summing its
// 2r+1 row neighbours from LDS; global reads and writes are contiguous.
constexpr int kIfRowElems = 2048;  // LDS elements per workgroup for the row pass

template <typename T>
__global__ void __launch_bounds__(256) k_if_rows(const T* __restrict__ in, T* __restrict__ out, int nx,
                                                 long long nrows, IfWeights wts, int radius) {
    __shared__ T lds[kIfRowElems];
    const int rpw = kIfRowElems / nx;
    const long long row0 = (long long)blockIdx.x * rpw;
    const int comp = blockIdx.y;
    const long long nrow_here = min((long long)rpw, nrows - row0);
    const long long base = comp * nrows * nx + row0 * nx;
    const int cnt = (int)(nrow_here * nx);
    for (int e = threadIdx.x; e < cnt; e += blockDim.x) lds[e] = in[base + e];
    __syncthreads();
    for (int e = threadIdx.x; e < cnt; e += blockDim.x) {
        const int i = e % nx;
        const int lo = max(-radius, -i), hi = min(radius, nx - 1 - i);
        double acc = 0.0;
        for (int d = max(-lo, hi); d >= 1; --d) {
            T s = 0;
            if (-d >= lo) s += lds[e - d];
            if (d <= hi) s += lds[e + d];
            acc += wts.w[d] * (double)s;
        }
        acc += wts.w[0] * (double)lds[e];
        out[base + e] = (T)acc;
    }
}

// x pass of the radii kIfFixedMaxRadius + 1 .. kIfWideMaxRadius: the same rows in LDS with R zeros (and a
// little more) on both sides, each thread 4 neighbouring outputs from one window of 4 + 2R values.  Same
// order of operations as k_if_rows (from the far neighbours inwards; a zero neighbour changes no sum), so
// the same bits.  One read per output and neighbour from LDS bounds k_if_rows: 147 us for 3 FP64 components
// of 177 x 144 x 160 at radius 15, against 70 us here (and 142 us for the y and the z pass each, against 55
// us in k_if_strided's register windows).
template <typename T, int R>
__global__ void __launch_bounds__(256) k_if_rows_wide(const T* __restrict__ in, T* __restrict__ out, int nx,
                                                      int rpw, int pitch, long long nrows, IfWeights wts) {
    constexpr int C = sizeof(T) == 8 ? 2 : 4;  // values per 16-byte LDS read
    constexpr int RP = (R + C - 1) / C * C;    // zeros in front (whole reads)
    constexpr int NV = (RP - R + 2 * R + 4 + C - 1) / C * C;
    struct alignas(16) Vec {
        T v[C];
    };
    extern __shared__ unsigned char smem[];
    T* lds = (T*)smem;  // [rpw][pitch]: RP zeros, the row, zeros
    const long long row0 = (long long)blockIdx.x * rpw;
    const int nr = (int)min((long long)rpw, nrows - row0);
    const long long base = blockIdx.y * nrows * nx + row0 * nx;
    for (int e = threadIdx.x; e < rpw * pitch; e += 256) {  // (one row per wave at a time measured 14 % slower)
        const int r = e / pitch, c = e - r * pitch - RP;
        lds[e] = (r < nr && c >= 0 && c < nx) ? in[base + (long long)r * nx + c] : (T)0;
    }
    __syncthreads();
    const int nq = (nx + 3) / 4;
    for (int e = threadIdx.x; e < nr * nq; e += 256) {
        const int r = e / nq, x = (e - r * nq) * 4;
        T v[NV];  // v[k] = value at x + k - RP
        const Vec* p = (const Vec*)(lds + r * pitch + x);
#pragma unroll
        for (int k = 0; k < NV / C; ++k) {
            const Vec t = p[k];
#pragma unroll
            for (int i = 0; i < C; ++i) v[k * C + i] = t.v[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double acc = 0.0;
#pragma unroll
            for (int d = R; d >= 1; --d) acc += wts.w[d] * (double)(v[RP + i - d] + v[RP + i + d]);
            acc += wts.w[0] * (double)v[RP + i];
            if (x + i < nx) out[base + (long long)r * nx + x + i] = (T)acc;
        }
    }
}

// y or z pass: a tile of TB adjacent x-columns times the full length along the axis is staged in
// LDS; each output sums its 2r+1 neighbours along the axis.  `stride` is the element distance
// between consecutive points along the axis, `outer_stride` between the tile groups of grid y.
template <typename T, int TB>
__global__ void __launch_bounds__(256) k_if_cols(const T* __restrict__ in, T* __restrict__ out, int nx, int len,
                                                 long long stride, long long outer_stride, long long comp_stride,
                                                 IfWeights wts, int radius) {
    extern __shared__ unsigned char smem[];
    T* lds = (T*)smem;  // [len][TB]
    const int c = threadIdx.x % TB;
    const int t = threadIdx.x / TB;
    constexpr int TPC = 256 / TB;  // threads per column
    const int col = blockIdx.x * TB + c;
    const bool valid = col < nx;
    const long long base = blockIdx.z * comp_stride + (long long)blockIdx.y * outer_stride + (valid ? col : 0);
    for (int k = t; k < len; k += TPC) lds[k * TB + c] = valid ? in[base + k * stride] : (T)0;
    __syncthreads();
    if (!valid) return;
    for (int k = t; k < len; k += TPC) {
        const int lo = max(-radius, -k), hi = min(radius, len - 1 - k);
        double acc = 0.0;
        for (int d = max(-lo, hi); d >= 1; --d) {
            T s = 0;
            if (-d >= lo) s += lds[(k - d) * TB + c];
            if (d <= hi) s += lds[(k + d) * TB + c];
            acc += wts.w[d] * (double)s;
        }
        acc += wts.w[0] * (double)lds[k * TB + c];
        out[base + k * stride] = (T)acc;
    }
}

// Fixed-radius passes (radius R known at compile time).  Outputs are formed in one order on every
// axis: w[0] v[k] + sum_{d = 1..R} w[d] (v[k - d] + v[k + d]), accumulated in FP64, with v = 0
// outside the box.  Input and output must not overlap.
//
// Input modes of the fused x-y pass.
enum IfInput { IF_IN_PLAIN = 0, IF_IN_COMB = 1, IF_IN_PROJ = 2 };
struct IfTerms {
    // IF_IN_COMB: v = c0 in + c1 in1 + c2 in2
    const void* in1;
    const void* in2;
    double c0, c1, c2;
    // IF_IN_PROJ: v = in - G dhat (component a of a 3-component field: the difference of dhat along axis
    // a); wnew = (v - (c_q q + c_w1 w1)) inv where wnew is given
    const void* dhat;
    const void* q;
    const void* w1;
    void* wnew;
    double idx, c_q, c_w1, inv;
};

// The operands of one input value of the fused x-y passes, and the value formed from them.  Loading and
// forming are separate so that a pass can have operands under way while it works on earlier rows: a
// combination or projection formed where it is loaded waits for memory there.
template <typename T, int MODE> struct IfOperands {
    static constexpr int N = MODE == IF_IN_PROJ ? 5 : MODE == IF_IN_COMB ? 3 : 1;
    T v[N];
};
template <typename T, int MODE>
__device__ __forceinline__ void if_load(IfOperands<T, MODE>& o, const T* __restrict__ in, const IfTerms& t, int comp,
                                        int z, int x, int y, int nx, int ny, int nz, long long pbase, bool inside,
                                        bool owned) {
#pragma unroll
    for (int i = 0; i < IfOperands<T, MODE>::N; ++i) o.v[i] = (T)0;
    if (!inside) return;
    const long long yx = (long long)y * nx + x, e = pbase + yx;  // (pbase: the plane's first element)
    o.v[0] = in[e];
    if constexpr (MODE == IF_IN_COMB) {
        o.v[1] = ((const T*)t.in1)[e];
        if (t.in2) o.v[2] = ((const T*)t.in2)[e];
    } else if constexpr (MODE == IF_IN_PROJ) {
        const T* D = (const T*)t.dhat;
        const long long c0 = (long long)z * ny * nx + yx;  // offset within one component
        o.v[1] = D[c0];
        const bool has = comp == 0 ? x + 1 < nx : comp == 1 ? y + 1 < ny : z + 1 < nz;
        const long long step = comp == 0 ? 1 : comp == 1 ? nx : (long long)nx * ny;
        if (has) o.v[2] = D[c0 + step];
        if (t.wnew && owned) {
            o.v[3] = ((const T*)t.q)[e];
            if (t.w1) o.v[4] = ((const T*)t.w1)[e];
        }
    }
}
// The roundings are written out (fused multiply-adds by name, nothing contracted beside them): left to the
// compiler, the product of a sum that is rounded first differs between the kernels and the loops that form a value,
// and the walk, the tiles and the batched forms have to agree bit for bit.
template <typename T, int MODE>
__device__ __forceinline__ T if_value(const IfOperands<T, MODE>& o, const IfTerms& t, int comp, int z, int x, int y,
                                      int nx, int ny, int nz, long long pbase, bool inside, bool owned) {
#pragma clang fp contract(off)
    if constexpr (MODE == IF_IN_COMB) {
        double v = fma(t.c0, (double)o.v[0], t.c1 * (double)o.v[1]);
        if (t.in2) v = fma(t.c2, (double)o.v[2], v);
        return inside ? (T)v : (T)0;
    } else if constexpr (MODE == IF_IN_PROJ) {
        const T v = fma(-(o.v[2] - o.v[1]), (T)t.idx, o.v[0]);
        if (t.wnew && inside && owned) {
            double base = t.c_q * (double)o.v[3];
            if (t.w1) base = fma(t.c_w1, (double)o.v[4], base);
            ((T*)t.wnew)[pbase + (long long)y * nx + x] = (T)(((double)v - base) * t.inv);
        }
        return inside ? v : (T)0;
    } else {
        return o.v[0];
    }
}

// One output of a filter of fixed radius R from its 2R + 1 neighbours v(-R) .. v(R), weights wd(0) .. wd(R): from the
// centre outwards, each step one rounding (written out for the same reason).
template <int R, class W, class V> __device__ __forceinline__ double if_filter(const W& wd, const V& v) {
    double acc = fma(wd(0), (double)v(0), wd(1) * (double)(v(-1) + v(1)));
#pragma unroll
    for (int d = 2; d <= R; ++d) acc = fma(wd(d), (double)(v(-d) + v(d)), acc);
    return acc;
}

// Fused x and y passes (fixed radius R): a workgroup owns one (component, z) plane and S consecutive
// output rows y0 .. y0 + S - 1 (the tile height, from the rows per workgroup the launch tuner sets per
// box), one thread per x (nx <= 256).  It walks the rows from y0 - R upwards,
// RB rows per step: each thread holds the operands of the next P steps in registers (loads issued
// P steps ahead; a projection formed where its operands were loaded waited for memory in every step: FP32
// 128^3 step 205 -> 151 us in these passes), the step's rows go through a double-buffered LDS tile with R zeros at both ends of
// each row (one barrier per step), each x-filtered value is rounded to the dtype and pushed into a
// register window of the last 2R + RB rows, and every row whose 2R + 1 neighbours are in the window
// is y-filtered and stored.  The values are the ones the separate x and y passes produce (same order
// of operations and roundings) without the intermediate field making a round trip through HBM.
// With IF_IN_COMB the raw value is the combination c0 in + c1 in1 + c2 in2, formed in FP64 and
// rounded once; with IF_IN_PROJ it is the projection r - G dhat of the stage (in the order of
// operations of the projection kernel), and the stage's new w is written on the way (each point by
// the workgroup that owns its output row).
// Workgroups are numbered so that all row blocks of one plane run on one XCD (the hardware hands
// workgroup b to XCD b mod 8) and share their halo rows through its L2.
// Arguments of one fused x-y pass (the batched form reads one table entry per problem).
struct IfXyArgs {
    const void* in;
    void* out;
    int nx, ny, nz, ntiles, S;
    IfWeights wts;
    IfTerms terms;
};
// BATCH: per consecutive logical workgroups make up one problem, whose arguments are da[problem].
template <typename T, int R, int RB, int P, int MODE, bool BATCH>
__global__ void __launch_bounds__(256) k_if_xy(IfXyArgs a0, const IfXyArgs* __restrict__ da, int per) {
    constexpr int W = 256 + 2 * R;  // LDS row length
    constexpr int NW = 2 * R + RB;  // register window (x-filtered rows)
    __shared__ T tile_lds[2][RB][W];
    const int nb = (int)gridDim.x, b = (int)blockIdx.x, xcd = b % 8;
    int lg = xcd * (nb / 8) + min(xcd, nb % 8) + b / 8;
    int pb = 0;
    if constexpr (BATCH) {
        pb = lg / per;
        lg -= pb * per;
    }
    const IfXyArgs* A = BATCH ? da + pb : nullptr;
    const T* __restrict__ in = (const T*)(BATCH ? A->in : a0.in);
    T* __restrict__ out = (T*)(BATCH ? A->out : a0.out);
    const int nx = BATCH ? A->nx : a0.nx, ny = BATCH ? A->ny : a0.ny, nz = BATCH ? A->nz : a0.nz;
    const int ntiles = BATCH ? A->ntiles : a0.ntiles, S = BATCH ? A->S : a0.S;
    const IfTerms terms = BATCH ? A->terms : a0.terms;
    auto wd = [&](int d) -> double {
        if constexpr (BATCH) return A->wts.w[d];
        else return a0.wts.w[d];
    };
    const int NSTEP = (S + 2 * R + RB - 1) / RB;
    const int tile = lg % ntiles, plane = lg / ntiles;  // plane = comp * nz + z
    const int x = threadIdx.x;
    const bool act = x < nx;
    const long long pbase = (long long)plane * nx * ny;
    const int y0 = tile * S, ylo = y0 - R;
    if (threadIdx.x < 2 * R) {
        const int h = threadIdx.x < R ? threadIdx.x : nx + threadIdx.x;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            tile_lds[0][i][h] = (T)0;
            tile_lds[1][i][h] = (T)0;
        }
    }
    const int comp = plane / nz, zpl = plane - comp * nz;
    using Ops = IfOperands<T, MODE>;
    Ops q[P][RB];
    auto fetch = [&](Ops& o, int y) {
        if_load<T, MODE>(o, in, terms, comp, zpl, x, y, nx, ny, nz, pbase, act && y >= 0 && y < ny, y >= y0 && y < y0 + S);
    };
    auto value = [&](const Ops& o, int y) -> T {
        return if_value<T, MODE>(o, terms, comp, zpl, x, y, nx, ny, nz, pbase, act && y >= 0 && y < ny, y >= y0 && y < y0 + S);
    };
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int i = 0; i < RB; ++i) fetch(q[j][i], ylo + j * RB + i);
    T win[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) win[i] = (T)0;
    for (int ks = 0; ks < NSTEP; ++ks) {
        T (*lt)[W] = tile_lds[ks & 1];
        if (act) {
#pragma unroll
            for (int i = 0; i < RB; ++i) lt[i][R + x] = value(q[0][i], ylo + ks * RB + i);
        }
#pragma unroll
        for (int j = 0; j < P - 1; ++j)
#pragma unroll
            for (int i = 0; i < RB; ++i) q[j][i] = q[j + 1][i];
#pragma unroll
        for (int i = 0; i < RB; ++i) fetch(q[P - 1][i], ylo + (ks + P) * RB + i);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) win[i] = win[i + RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            T xf = (T)0;
            if (act) {
                const T* p = &lt[i][R + x];
                xf = (T)if_filter<R>(wd, [&](int d) { return p[d]; });
            }
            win[2 * R + i] = xf;
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int kk = ks * RB + i;  // rows ylo .. ylo + kk are in; the row y = ylo + kk - R is complete
            const int y = ylo + kk - R;
            if (kk >= 2 * R && act && y < ny && y < y0 + S) {
                out[pbase + (long long)y * nx + x] = (T)if_filter<R>(wd, [&](int d) { return win[i + R + d]; });
            }
        }
    }
}

// Fused x and y passes on tiles of at most 64 x 32 outputs of one plane (any nx): the tile and its halo of
// R points come into LDS at once (independent loads, one memory latency), the x filter runs in place over
// the rows y0 - R .. y0 + ty + R - 1 (each thread 2 neighbouring outputs from R + 1 pair reads), the y
// filter reads columns (each thread 8 outputs of one column).  Same operations and roundings as the
// walking pass above, so the results are equal bit for bit.
struct IfTileArgs {
    const void* in;
    void* out;
    int nx, ny, nz, ntx, nty, tx, ty;
    IfWeights wts;
    IfTerms terms;
};
constexpr int kIfTileX = 64, kIfTileY = 32;

template <typename T> struct alignas(2 * sizeof(T)) IfPair {
    T a, b;
};

// Batched form (da set): `per` consecutive workgroups make up one problem, whose arguments are da[problem].
template <typename T, int R, int MODE>
__global__ void __launch_bounds__(256) k_if_tile(IfTileArgs a0, const IfTileArgs* __restrict__ da, int per) {
    constexpr int PITCH = kIfTileX + 2 * R + 2;  // (even; two spare elements keep the pair reads of a row inside it)
    constexpr int ROWS = kIfTileY + 2 * R;
    __shared__ IfPair<T> lds2[ROWS * PITCH / 2];
    T* const lds = (T*)lds2;
    const int nb = (int)gridDim.x, b = (int)blockIdx.x, xcd = b % 8;
    int lg = xcd * (nb / 8) + min(xcd, nb % 8) + b / 8;
    const IfTileArgs* A = &a0;
    if (da) {
        A = da + lg / per;
        lg %= per;
    }
    const T* __restrict__ in = (const T*)A->in;
    T* __restrict__ out = (T*)A->out;
    const int nx = A->nx, ny = A->ny, nz = A->nz, tx = A->tx, ty = A->ty;
    const IfTerms terms = A->terms;
    const int itx = lg % A->ntx, ity = (lg / A->ntx) % A->nty, plane = lg / (A->ntx * A->nty);  // plane = comp * nz + z
    const int comp = plane / nz, z = plane - comp * nz;
    const int x0 = itx * tx, y0 = ity * ty;
    const int txe = min(tx, nx - x0), tye = min(ty, ny - y0);  // this tile's outputs (none if the split left it empty)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long pbase = (long long)plane * nx * ny;
    using Ops = IfOperands<T, MODE>;
    auto inside = [&](int x, int y) { return x >= 0 && x < nx && y >= 0 && y < ny; };
    auto owned = [&](int x, int y) { return y >= y0 && y < y0 + tye && x >= x0 && x < x0 + txe; };
    auto fetch = [&](Ops& o, int x, int y) {
        if_load<T, MODE>(o, in, terms, comp, z, x, y, nx, ny, nz, pbase, inside(x, y), owned(x, y));
    };
    auto value = [&](const Ops& o, int x, int y) -> T {
        return if_value<T, MODE>(o, terms, comp, z, x, y, nx, ny, nz, pbase, inside(x, y), owned(x, y));
    };
    auto wd = [&](int d) -> double { return A->wts.w[d]; };
    // rows of the tile and its halo, one row per wave at a time; the columns beyond the first 64 (2R of them
    // at most) for several rows at once
    const int nrows = tye + 2 * R, ncols = txe + 2 * R;
    constexpr int CH = MODE == IF_IN_PROJ ? 4 : 6;  // rows whose loads are in flight together
    for (int r0 = wave; r0 < nrows; r0 += 4 * CH) {
        Ops t[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = r0 + 4 * i;
            fetch(t[i], (r < nrows && lane < ncols) ? x0 - R + lane : -1, y0 - R + r);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = r0 + 4 * i;
            if (r < nrows) lds[r * PITCH + lane] = value(t[i], lane < ncols ? x0 - R + lane : -1, y0 - R + r);
        }
    }
    constexpr int HL = 2 * R <= 8 ? 8 : 2 * R <= 16 ? 16 : 32, HR = 256 / HL;  // lanes per row, rows at a time
    if (ncols > 64) {
        const int hc = 64 + (int)threadIdx.x % HL;
        for (int r = (int)threadIdx.x / HL; r < nrows; r += HR) {
            Ops t;
            fetch(t, hc < ncols ? x0 - R + hc : -1, y0 - R + r);
            if (hc < PITCH) lds[r * PITCH + hc] = value(t, hc < ncols ? x0 - R + hc : -1, y0 - R + r);
        }
    }
    __syncthreads();
    // x filter in place: 32 pairs of outputs per row, 8 rows at a time
    constexpr int NP = (ROWS + 7) / 8;
    const int px = ((int)threadIdx.x & 31) * 2, pr = (int)threadIdx.x >> 5;
    IfPair<T> f[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int r = pr + 8 * i;
        if (r < nrows && px < txe) {
            T v[2 * R + 2];
#pragma unroll
            for (int k = 0; k <= R; ++k) {
                const IfPair<T> p = lds2[(r * PITCH + px) / 2 + k];
                v[2 * k] = p.a;
                v[2 * k + 1] = p.b;
            }
            f[i].a = (T)if_filter<R>(wd, [&](int d) { return v[R + d]; });
            f[i].b = (T)if_filter<R>(wd, [&](int d) { return v[R + 1 + d]; });
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int r = pr + 8 * i;
        if (r < nrows && px < txe) lds2[(r * PITCH + px) / 2] = f[i];
    }
    __syncthreads();
    // y filter: wave w takes the output rows 8 w .. 8 w + 7 of every column
    constexpr int NY = kIfTileY / 4;
    const int yr = wave * NY;
    if (lane < txe && yr < tye) {
        T v[NY + 2 * R];
#pragma unroll
        for (int k = 0; k < NY + 2 * R; ++k) v[k] = (yr + k < nrows) ? lds[(yr + k) * PITCH + lane] : (T)0;
#pragma unroll
        for (int k = 0; k < NY; ++k) {
            if (yr + k < tye) {
                out[pbase + (long long)(y0 + yr + k) * nx + x0 + lane] =
                    (T)if_filter<R>(wd, [&](int d) { return v[k + R + d]; });
            }
        }
    }
}

// y and z passes: a thread owns one x position (consecutive lanes take consecutive x, so every load
// and store of a wavefront is one contiguous row segment) and S consecutive outputs of its line; the
// S + 2R inputs go straight from memory into registers (neighbouring segments re-read their shared
// halo through the caches, not from HBM).  No LDS and no barriers.
struct IfStrArgs {
    const void* in;
    void* out;
    int nx, len, nouter;
    long long stride, outer_stride, comp_stride;
    IfWeights wts;
};
// BATCH: per consecutive values of the grid's z index make up one problem, whose arguments are da[problem].
template <typename T, int R, int S, bool BATCH>
__global__ void __launch_bounds__(256) k_if_strided(IfStrArgs a0, const IfStrArgs* __restrict__ da, int per) {
    int bz = blockIdx.z, pb = 0;
    if constexpr (BATCH) {
        pb = bz / per;
        bz -= pb * per;
    }
    const IfStrArgs* A = BATCH ? da + pb : nullptr;
    const T* __restrict__ in = (const T*)(BATCH ? A->in : a0.in);
    T* __restrict__ out = (T*)(BATCH ? A->out : a0.out);
    const int nx = BATCH ? A->nx : a0.nx, len = BATCH ? A->len : a0.len, nouter = BATCH ? A->nouter : a0.nouter;
    const long long stride = BATCH ? A->stride : a0.stride, outer_stride = BATCH ? A->outer_stride : a0.outer_stride;
    const long long comp_stride = BATCH ? A->comp_stride : a0.comp_stride;
    auto wd = [&](int d) -> double {
        if constexpr (BATCH) return A->wts.w[d];
        else return a0.wts.w[d];
    };
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int k0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * S;
    if (x >= nx || k0 >= len) return;
    const int o = bz % nouter, comp = bz / nouter;
    const long long base = comp * comp_stride + (long long)o * outer_stride + x;
    T v[S + 2 * R];
    if (k0 >= R && k0 + S + R <= len) {  // the whole window inside the line: loads without tests
#pragma unroll
        for (int j = 0; j < S + 2 * R; ++j) v[j] = in[base + (long long)(k0 - R + j) * stride];
    } else {
#pragma unroll
        for (int j = 0; j < S + 2 * R; ++j) {
            const int k = k0 - R + j;
            v[j] = (k >= 0 && k < len) ? in[base + (long long)k * stride] : (T)0;
        }
    }
    const bool full = k0 + S <= len;
#pragma unroll
    for (int m = 0; m < S; ++m) {
        if (full || k0 + m < len) {
            double acc;
            if constexpr (R > kIfFixedMaxRadius) {  // (the order of the runtime-radius passes)
                acc = 0.0;
#pragma unroll
                for (int d = R; d >= 1; --d) acc += wd(d) * (double)(v[m + R - d] + v[m + R + d]);
                acc += wd(0) * (double)v[m + R];
            } else {
                acc = if_filter<R>(wd, [&](int d) { return v[m + R + d]; });
            }
            out[base + (long long)(k0 + m) * stride] = (T)acc;
        }
    }
}

// Outputs per thread of the strided passes: 32 by default, 16 where the launch tuner finds it faster.
constexpr int kIfRowsPerStep = 4;    // rows per barrier of the fused x-y pass
constexpr int kIfPrefetch = 2;       // steps loaded ahead by the fused x-y pass

template <typename T, int R, int S>
static int batched_strided(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_if_strided<T, R, S, true>), dim3(g.x, g.y, g.z * nprob), b, 0, s, IfStrArgs{},
                       (const IfStrArgs*)args, (int)g.z);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
// Radii above the fixed ones up to kIfWideMaxRadius, one axis at a time (no batched form).
template <typename T, int R>
static void launch_wide(int axis, const T* in, T* out, int ncomp, int nx, int ny, int nz, const IfWeights& wts,
                        hipStream_t s) {
    const long long n = (long long)nx * ny * nz;
    if (axis == 0) {
        constexpr int C = sizeof(T) == 8 ? 2 : 4, RP = (R + C - 1) / C * C;
        // a row's last window starts at 4 (nq - 1) and holds at most 2 RP + 4 + C values
        const int pitch = ((nx + 3) / 4 * 4 + 2 * RP + 2 * C) / C * C;
        const int rpw = std::max(1, 2048 / pitch);
        hipLaunchKernelGGL((k_if_rows_wide<T, R>), dim3(ceil_div((long long)ny * nz, rpw), ncomp), dim3(256),
                           (size_t)rpw * pitch * sizeof(T), s, in, out, nx, rpw, pitch, (long long)ny * nz, wts);
        return;
    }
    const int len = axis == 1 ? ny : nz, nouter = axis == 1 ? nz : ny;
    const IfStrArgs a{in, out, nx, len, nouter, axis == 1 ? (long long)nx : (long long)nx * ny,
                      axis == 1 ? (long long)nx * ny : (long long)nx, n, wts};
    hipLaunchKernelGGL((k_if_strided<T, R, 32, false>), dim3(ceil_div(nx, 64), ceil_div(ceil_div(len, 32), 4), nouter * ncomp),
                       dim3(256), 0, s, a, nullptr, 0);
}
template <typename T, int R, int MODE>
static int batched_xy(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_if_xy<T, R, kIfRowsPerStep, kIfPrefetch, MODE, true>), dim3(g.x * nprob), b, 0, s,
                       IfXyArgs{}, (const IfXyArgs*)args, (int)g.x);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

template <typename T, int R, int S> static void issue_strided(const IfStrArgs& a, dim3 grid, hipStream_t s) {
    if (launch_recorder()) {
        record_launch(&batched_strided<T, R, S>, grid, dim3(256), a);
        return;
    }
    hipLaunchKernelGGL((k_if_strided<T, R, S, false>), grid, dim3(256), 0, s, a, nullptr, 0);
}

template <typename T, int R>
static void launch_fixed(int axis, const T* in, T* out, int ncomp, int nx, int ny, int nz, const IfWeights& wts,
                         hipStream_t s, int seg) {
    const long long n = (long long)nx * ny * nz;
    const int len = axis == 1 ? ny : nz;
    const long long stride = axis == 1 ? (long long)nx : (long long)nx * ny;
    const int nouter = axis == 1 ? nz : ny;
    const long long outer_stride = axis == 1 ? (long long)nx * ny : (long long)nx;
    const IfStrArgs a{in, out, nx, len, nouter, stride, outer_stride, n, wts};
    if (seg == 16)
        issue_strided<T, R, 16>(a, dim3(ceil_div(nx, 64), ceil_div(ceil_div(len, 16), 4), nouter * ncomp), s);
    else
        issue_strided<T, R, 32>(a, dim3(ceil_div(nx, 64), ceil_div(ceil_div(len, 32), 4), nouter * ncomp), s);
}

template <typename T, int R, int MODE>
static int batched_tile(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_if_tile<T, R, MODE>), dim3(g.x * nprob), b, 0, s, IfTileArgs{}, (const IfTileArgs*)args,
                       (int)g.x);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T, int R, int MODE>
static void issue_tile(const IfXyArgs& x, int ncomp, hipStream_t s) {
    // tiles of equal size along each axis (none empty: every split has at most one point per tile less than the first)
    IfTileArgs a{x.in, x.out, x.nx, x.ny, x.nz, ceil_div(x.nx, kIfTileX), ceil_div(x.ny, kIfTileY), 0, 0, x.wts, x.terms};
    a.tx = ceil_div(x.nx, a.ntx);
    a.ty = ceil_div(x.ny, a.nty);
    const dim3 grid((unsigned)((long long)a.ntx * a.nty * a.nz * ncomp)), block(256);
    if (launch_recorder()) {
        record_launch(&batched_tile<T, R, MODE>, grid, block, a);
        return;
    }
    hipLaunchKernelGGL((k_if_tile<T, R, MODE>), grid, block, 0, s, a, nullptr, 0);
}

template <typename T, int R, int MODE>
static void issue_xy(const IfXyArgs& a, dim3 grid, dim3 block, hipStream_t s) {
    if (launch_recorder()) {
        record_launch(&batched_xy<T, R, MODE>, grid, block, a);
        return;
    }
    hipLaunchKernelGGL((k_if_xy<T, R, kIfRowsPerStep, kIfPrefetch, MODE, false>), grid, block, 0, s, a, nullptr, 0);
}

// rows: at most this many output rows per workgroup; the ny rows of a plane are split into
// ntiles = ceil(ny / rows) tiles of height ceil(ny / ntiles) (the last at most ntiles - 1 rows shorter,
// never empty), so that no workgroup walks far past the plane's end or carries a long tail alone (halo
// rows re-read: 2R / height).  A workgroup has one thread per x rounded up to whole wavefronts.
template <typename T, int R>
static void launch_xy(const IfCombine& cb, T* out, int ncomp, int nx, int ny, int nz, const IfWeights& wts,
                      hipStream_t s, int rows) {
    const int ntiles = ceil_div(ny, rows);
    const int height = ceil_div(ny, ntiles);
    const dim3 grid((unsigned)((long long)ntiles * nz * ncomp)), block((unsigned)(ceil_div(nx, 64) * 64));
    IfXyArgs a{cb.p[0], out, nx, ny, nz, ntiles, height, wts, IfTerms{}};
    IfTerms& terms = a.terms;
    // Below two waves per SIMD (2048) the walk's chain of row steps is exposed and the tiles, which load
    // everything at once, win; above, the walk re-reads fewer halo points (us per plain / projecting launch at
    // radius 6 or 7, walk against tiles: FP64 48^3 18 / 26 against 11 / 14, 3 components at 96^3 29 against 26,
    // 6 components at 96^3 37 against 43; FP32 128^3 22 against 23; FP64 256^3 178 against 349).
    const long long waves = (long long)ntiles * nz * ncomp * ceil_div(nx, 64);
    const bool tile = waves * (launch_recorder() ? launch_recorder()->alike : 1) < 2048;
    if (cb.proj) {
        const IfProject& pj = *cb.proj;
        terms.dhat = pj.dhat;
        terms.q = pj.q;
        terms.w1 = pj.w1;
        terms.wnew = pj.wnew;
        terms.idx = pj.idx;
        terms.c_q = pj.c_q;
        terms.c_w1 = pj.c_w1;
        terms.inv = pj.inv;
        if (tile)
            issue_tile<T, R, IF_IN_PROJ>(a, ncomp, s);
        else
            issue_xy<T, R, IF_IN_PROJ>(a, grid, block, s);
    } else if (cb.p[1]) {
        terms.in1 = cb.p[1];
        terms.in2 = cb.p[2];
        terms.c0 = cb.c[0];
        terms.c1 = cb.c[1];
        terms.c2 = cb.c[2];
        if (tile)
            issue_tile<T, R, IF_IN_COMB>(a, ncomp, s);
        else
            issue_xy<T, R, IF_IN_COMB>(a, grid, block, s);
    } else {
        if (tile)
            issue_tile<T, R, IF_IN_PLAIN>(a, ncomp, s);
        else
            issue_xy<T, R, IF_IN_PLAIN>(a, grid, block, s);
    }
}

template <typename T>
static int if_axis_t(int axis, const void* in, void* out, int ncomp, int nx, int ny, int nz, const double* w,
                     int radius, hipStream_t s, int seg) {
    IfWeights wts;
    for (int k = 0; k <= kIfMaxRadius; ++k) wts.w[k] = k <= radius ? w[k] : 0.0;
    const long long n = (long long)nx * ny * nz;
    const T* src = (const T*)in;
    T* dst = (T*)out;
    if (axis != 0) {
        switch (radius) {
#define NSLGF_IF_R(R_) case R_: launch_fixed<T, R_>(axis, src, dst, ncomp, nx, ny, nz, wts, s, seg); NSLGF_LAUNCH_CHECK(); return NSLGF_OK;
            NSLGF_IF_R(1) NSLGF_IF_R(2) NSLGF_IF_R(3) NSLGF_IF_R(4) NSLGF_IF_R(5) NSLGF_IF_R(6) NSLGF_IF_R(7)
            NSLGF_IF_R(8) NSLGF_IF_R(9) NSLGF_IF_R(10) NSLGF_IF_R(11) NSLGF_IF_R(12)
#undef NSLGF_IF_R
            default: break;
        }
    }
    // wide and runtime-radius passes; no batched form
    if (recording_unsupported()) return NSLGF_OK;
    switch (radius) {
#define NSLGF_IF_R(R_) case R_: launch_wide<T, R_>(axis, src, dst, ncomp, nx, ny, nz, wts, s); NSLGF_LAUNCH_CHECK(); return NSLGF_OK;
        NSLGF_IF_R(13) NSLGF_IF_R(14) NSLGF_IF_R(15) NSLGF_IF_R(16) NSLGF_IF_R(17) NSLGF_IF_R(18) NSLGF_IF_R(19)
        NSLGF_IF_R(20) NSLGF_IF_R(21) NSLGF_IF_R(22) NSLGF_IF_R(23) NSLGF_IF_R(24)
#undef NSLGF_IF_R
        default: break;
    }
    if (axis == 0) {
        if (nx > kIfRowElems) {
            set_error("if_apply: rows longer than the LDS row buffer");
            return NSLGF_EUNSUPPORTED;
        }
        const long long nrows = (long long)ny * nz;
        const int rpw = kIfRowElems / nx;
        dim3 grid(ceil_div(nrows, rpw), ncomp);
        hipLaunchKernelGGL((k_if_rows<T>), grid, dim3(256), 0, s, src, dst, nx, nrows, wts, radius);
    } else {
        constexpr int TB = (int)(128 / sizeof(T));
        const int len = axis == 1 ? ny : nz;
        const long long stride = axis == 1 ? (long long)nx : (long long)nx * ny;
        const int nouter = axis == 1 ? nz : ny;
        const long long outer_stride = axis == 1 ? (long long)nx * ny : (long long)nx;
        const size_t lds = (size_t)len * TB * sizeof(T);
        dim3 grid(ceil_div(nx, TB), nouter, ncomp);
        hipLaunchKernelGGL((k_if_cols<T, TB>), grid, dim3(256), lds, s, src, dst, nx, len, stride, outer_stride, n,
                           wts, radius);
    }
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

template <typename T>
static int if_xy_t(const IfCombine& cb, void* out, int ncomp, int nx, int ny, int nz, const double* w, int radius,
                   hipStream_t s, int rows) {
    IfWeights wts;
    for (int k = 0; k <= kIfMaxRadius; ++k) wts.w[k] = k <= radius ? w[k] : 0.0;
    T* dst = (T*)out;
    switch (radius) {
#define NSLGF_IF_R(R_) case R_: launch_xy<T, R_>(cb, dst, ncomp, nx, ny, nz, wts, s, rows); NSLGF_LAUNCH_CHECK(); return NSLGF_OK;
        NSLGF_IF_R(1) NSLGF_IF_R(2) NSLGF_IF_R(3) NSLGF_IF_R(4) NSLGF_IF_R(5) NSLGF_IF_R(6) NSLGF_IF_R(7)
        NSLGF_IF_R(8) NSLGF_IF_R(9) NSLGF_IF_R(10) NSLGF_IF_R(11) NSLGF_IF_R(12)
#undef NSLGF_IF_R
        default: break;
    }
    set_error("if_apply: no fused x-y pass for this radius");
    return NSLGF_EUNSUPPORTED;
}

int launch_if_xy(int dtype, const IfCombine& cb, void* out, int ncomp, int nx, int ny, int nz, const double* w,
                 int radius, hipStream_t s, int rows) {
    if (!cb.p[0] || (cb.p[2] && !cb.p[1]) || (cb.proj && (cb.p[1] || ncomp != 3 || !cb.proj->dhat ||
                                                          (cb.proj->wnew && !cb.proj->q)))) {
        set_error("if_apply: bad input combination");
        return NSLGF_EINVAL;
    }
    if (nx > 256) {
        set_error("if_apply: the fused x-y pass needs nx <= 256");
        return NSLGF_EUNSUPPORTED;
    }
    if (rows != 32 && rows != 64 && rows != 128 && rows != 256) {
        set_error("if_apply: the fused x-y pass takes 32, 64, 128 or 256 rows per workgroup");
        return NSLGF_EINVAL;
    }
    if (dtype == NSLGF_F32) return if_xy_t<float>(cb, out, ncomp, nx, ny, nz, w, radius, s, rows);
    return if_xy_t<double>(cb, out, ncomp, nx, ny, nz, w, radius, s, rows);
}

int launch_if_axis(int axis, int dtype, const void* in, void* out, int ncomp, int nx, int ny, int nz, const double* w,
                   int radius, hipStream_t s, int seg) {
    if (seg != 16 && seg != 32) {
        set_error("if_apply: the strided pass takes 16 or 32 outputs per thread");
        return NSLGF_EINVAL;
    }
    if (dtype == NSLGF_F32) return if_axis_t<float>(axis, in, out, ncomp, nx, ny, nz, w, radius, s, seg);
    return if_axis_t<double>(axis, in, out, ncomp, nx, ny, nz, w, radius, s, seg);
}

}  // namespace nslgf
