// Staggered-grid point operators of Appendix A on one box, and the fused IF-HERK stage kernels.
//
// Every input is read with zero extension outside the box and every output is produced on the box
// only (the mask operators of Sec. 4.1).  Components (2) and (3) of each printed operator follow from
// component (1) by the cyclic permutation (component, axis): 1 -> 2 -> 3 -> 1 with x -> y -> z -> x.
#include <algorithm>
#include <cmath>

#include "kernels.h"

namespace nslgf {

// Boxes have at most 256 points per axis, so a point's offset within one component fits 32 bits.
template <typename T> struct Fld {
    const T* p;
    int nx, ny, nz;
    __device__ __forceinline__ T operator()(int i, int j, int k) const {
        return (i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz) ? p[(k * ny + j) * nx + i] : (T)0;
    }
};

// The same field read without bounds tests, for points whose neighbours are all inside the box (the
// tests would otherwise turn every load into a branch).
template <typename T> struct FldIn {
    const T* p;
    int nx, ny, nz;
    __device__ __forceinline__ T operator()(int i, int j, int k) const { return p[(k * ny + j) * nx + i]; }
};

template <typename T> struct Vec3 {
    Fld<T> c[3];
};
template <typename T> struct Vec3In {
    FldIn<T> c[3];
};
template <typename T> __device__ __forceinline__ Vec3In<T> unchecked(const Vec3<T>& v) {
    Vec3In<T> r;
    for (int q = 0; q < 3; ++q) r.c[q] = FldIn<T>{v.c[q].p, v.c[q].nx, v.c[q].ny, v.c[q].nz};
    return r;
}

template <typename T>
__device__ __forceinline__ Vec3<T> vec3(const T* p, int nx, int ny, int nz) {
    const long long n = (long long)nx * ny * nz;
    Vec3<T> v;
    for (int q = 0; q < 3; ++q) v.c[q] = Fld<T>{p + q * n, nx, ny, nz};
    return v;
}

// e = C f at edge (i, j, k), component q (0-based); the curl of the zero-extended face field, so
// it is also defined one layer outside the box.
template <typename T>
__device__ __forceinline__ T curl_at(const Vec3<T>& f, int q, int i, int j, int k, T idx) {
    if (q == 0) return (f.c[1](i, j, k) - f.c[1](i, j, k + 1) + f.c[2](i, j + 1, k) - f.c[2](i, j, k)) * idx;
    if (q == 1) return (f.c[2](i, j, k) - f.c[2](i + 1, j, k) + f.c[0](i, j, k + 1) - f.c[0](i, j, k)) * idx;
    return (f.c[0](i, j, k) - f.c[0](i, j + 1, k) + f.c[1](i + 1, j, k) - f.c[1](i, j, k)) * idx;
}

// Ntilde(f) at face (i, j, k), all three components (Eq. opr_def_nonlin and its cyclic images).
// The nine edge values of e = C f it needs (e1, e2, e3 at the cell and one step back along the
// other axes) use 24 distinct face values, each loaded once: component (1) at offsets
// (0,0,0), (0,0,+-1), (0,+-1,0), (-1,0,0), (-1,+1,0), (-1,0,+1) and the cyclic images for (2), (3).
// curl (when given): the three edge values at (i, j, k), as curl_at gives them.
template <typename T, class V>
__device__ __forceinline__ void nonlinear_at(const V& f, int i, int j, int k, T idx, T out[3], T* curl = nullptr) {
    const auto& F1 = f.c[0];
    const auto& F2 = f.c[1];
    const auto& F3 = f.c[2];
    const T a000 = F1(i, j, k), a00p = F1(i, j, k + 1), a00m = F1(i, j, k - 1), a0p0 = F1(i, j + 1, k),
            a0m0 = F1(i, j - 1, k), am00 = F1(i - 1, j, k), amp0 = F1(i - 1, j + 1, k), am0p = F1(i - 1, j, k + 1);
    const T b000 = F2(i, j, k), bp00 = F2(i + 1, j, k), bm00 = F2(i - 1, j, k), b00p = F2(i, j, k + 1),
            b00m = F2(i, j, k - 1), b0m0 = F2(i, j - 1, k), bpm0 = F2(i + 1, j - 1, k), b0mp = F2(i, j - 1, k + 1);
    const T c000 = F3(i, j, k), cp00 = F3(i + 1, j, k), cm00 = F3(i - 1, j, k), c0p0 = F3(i, j + 1, k),
            c0m0 = F3(i, j - 1, k), c00m = F3(i, j, k - 1), cp0m = F3(i + 1, j, k - 1), c0pm = F3(i, j + 1, k - 1);
    // edge values: e1 at (i,j,k), (i,j,k-1), (i,j-1,k); e2 at (i,j,k), (i,j,k-1), (i-1,j,k);
    // e3 at (i,j,k), (i,j-1,k), (i-1,j,k)
    const T e1_0 = (b000 - b00p + c0p0 - c000) * idx;
    const T e1_km = (b00m - b000 + c0pm - c00m) * idx;
    const T e1_jm = (b0m0 - b0mp + c000 - c0m0) * idx;
    const T e2_0 = (c000 - cp00 + a00p - a000) * idx;
    const T e2_km = (c00m - cp0m + a000 - a00m) * idx;
    const T e2_im = (cm00 - c000 + am0p - am00) * idx;
    const T e3_0 = (a000 - a0p0 + bp00 - b000) * idx;
    const T e3_jm = (a0m0 - a000 + bpm0 - b0m0) * idx;
    const T e3_im = (am00 - amp0 + b000 - bm00) * idx;
    if (curl) {
        curl[0] = e1_0;
        curl[1] = e2_0;
        curl[2] = e3_0;
    }
    out[0] = (T)0.25 * (e2_0 * (c000 + cp00) + e2_km * (c00m + cp0m) - e3_0 * (b000 + bp00) - e3_jm * (b0m0 + bpm0));
    out[1] = (T)0.25 * (e3_0 * (a000 + a0p0) + e3_im * (am00 + amp0) - e1_0 * (c000 + c0p0) - e1_km * (c00m + c0pm));
    out[2] = (T)0.25 * (e1_0 * (b000 + b00p) + e1_jm * (b0m0 + b0mp) - e2_0 * (a000 + a00p) - e2_im * (am00 + am0p));
}

// Point kernels run on 256-thread blocks tiling (x, y) (64 x 4 by default; the launch tuner may
// pick another of kCellShape), one z plane per grid z (no integer division); launch with cell_grid /
// cell_block.  (Renumbering the blocks so that each XCD works through a contiguous range of planes
// was measured slower for the stage kernels.)
#define NSLGF_CELL_INDEX_Z(KZ)                                                                     \
    const long long n = (long long)nx * ny * nz;                                                   \
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);                                    \
    const int j = (int)(blockIdx.y * blockDim.y + threadIdx.y);                                    \
    const int kz_ = (KZ);                                                                          \
    const int k = kz_ % nz;                                                                        \
    if (i >= nx || j >= ny) return;                                                                \
    const long long idx = (long long)((k * ny + j) * nx + i);
#define NSLGF_CELL_INDEX                                                                           \
    const long long n = (long long)nx * ny * nz;                                                   \
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);                                    \
    const int j = (int)(blockIdx.y * blockDim.y + threadIdx.y);                                    \
    const int kz_ = (int)blockIdx.z;                                                               \
    const int k = kz_ % nz;                                                                        \
    if (i >= nx || j >= ny) return;                                                                \
    const long long idx = (long long)((k * ny + j) * nx + i);

static const int kCellShape[kCellShapeCount][2] = {{64, 4}, {128, 2}, {32, 8}, {256, 1}};
static dim3 cell_block(int shape) {
    const int k = (shape >= 0 && shape < kCellShapeCount) ? shape : 0;
    return dim3(kCellShape[k][0], kCellShape[k][1]);
}
static dim3 cell_grid(int nx, int ny, int nz, int ncomp = 1, int shape = 0) {
    const dim3 b = cell_block(shape);
    return dim3(ceil_div(nx, b.x), ceil_div(ny, b.y), nz * ncomp);
}

template <typename T>
__global__ void __launch_bounds__(256) k_grad(const T* c, T* f, int nx, int ny, int nz, T idx_) {
    NSLGF_CELL_INDEX
    Fld<T> C{c, nx, ny, nz};
    const T v = C(i, j, k);
    f[idx] = (C(i + 1, j, k) - v) * idx_;
    f[n + idx] = (C(i, j + 1, k) - v) * idx_;
    f[2 * n + idx] = (C(i, j, k + 1) - v) * idx_;
}

template <typename T>
__global__ void __launch_bounds__(256) k_div(const T* f, T* c, int nx, int ny, int nz, T idx_, int nbuf) {
    NSLGF_CELL_INDEX
    Vec3<T> F = vec3(f, nx, ny, nz);
    const bool in_supp = i >= nbuf && i < nx - nbuf && j >= nbuf && j < ny - nbuf && k >= nbuf && k < nz - nbuf;
    T v = (F.c[0](i, j, k) + F.c[1](i, j, k) + F.c[2](i, j, k) - F.c[0](i - 1, j, k) - F.c[1](i, j - 1, k) -
           F.c[2](i, j, k - 1)) * idx_;
    c[idx] = in_supp ? v : (T)0;
}

// e = C f on the box; with nbuf > 0 or support blocks, e = M_supp C f: edges outside the support
// domain (the box shrunk by nbuf points, or the union of the marked blocks of nb^3 cells) are set to 0.
template <typename T>
__global__ void __launch_bounds__(256) k_curl(const T* f, T* e, int nx, int ny, int nz, T idx_, int nbuf,
                                              const unsigned char* blocks, int nb) {
    NSLGF_CELL_INDEX
    Vec3<T> F = vec3(f, nx, ny, nz);
    const bool in_supp = in_domain(i, j, k, nx, ny, nz, nbuf, blocks, nb);
    for (int q = 0; q < 3; ++q) e[q * n + idx] = in_supp ? curl_at(F, q, i, j, k, idx_) : (T)0;
}

template <typename T>
__global__ void __launch_bounds__(256) k_curl_bar(const T* e, T* f, int nx, int ny, int nz, T idx_) {
    NSLGF_CELL_INDEX
    Vec3<T> Ed = vec3(e, nx, ny, nz);
    f[idx] = (Ed.c[1](i, j, k - 1) - Ed.c[1](i, j, k) + Ed.c[2](i, j, k) - Ed.c[2](i, j - 1, k)) * idx_;
    f[n + idx] = (Ed.c[2](i - 1, j, k) - Ed.c[2](i, j, k) + Ed.c[0](i, j, k) - Ed.c[0](i, j, k - 1)) * idx_;
    f[2 * n + idx] = (Ed.c[0](i, j - 1, k) - Ed.c[0](i, j, k) + Ed.c[1](i, j, k) - Ed.c[1](i - 1, j, k)) * idx_;
}

template <typename T>
__global__ void __launch_bounds__(256) k_nonlinear(const T* f, T* out, int nx, int ny, int nz, T idx_) {
    NSLGF_CELL_INDEX
    Vec3<T> F = vec3(f, nx, ny, nz);
    T r[3];
    nonlinear_at(F, i, j, k, idx_, r);
    out[idx] = r[0];
    out[n + idx] = r[1];
    out[2 * n + idx] = r[2];
}

template <typename T>
__global__ void __launch_bounds__(256) k_laplacian(const T* a, T* out, int nx, int ny, int nz, T idx2) {
    NSLGF_CELL_INDEX
    const int comp = kz_ / nz;
    Fld<T> A{a + comp * n, nx, ny, nz};
    out[comp * n + idx] = (-(T)6 * A(i, j, k) + A(i + 1, j, k) + A(i - 1, j, k) + A(i, j + 1, k) + A(i, j - 1, k) +
                           A(i, j, k + 1) + A(i, j, k - 1)) * idx2;
}

// Arguments of the stage kernels (the batched forms read one table entry per problem: per consecutive
// values of the grid's z index make up one problem).
struct StageRhsArgs {
    const void* u;
    void* q;
    const void* w1;
    const void* w2;
    void* r;
    double idx;
    StageCoef c;
    int nx, ny, nz;
};
struct StageProjArgs {
    const void* r;
    void* rout;
    const void* dhat;
    const void* q;
    const void* w1;
    const void* w2;
    double c_q, c_w1, c_w2;
    void* wnew;
    double inv, idx;
    int nx, ny, nz;
    void* dout;  // (optional) dout = dscale dhat
    double dscale;
};
struct AxpbyArgs {
    void* out;
    const void* x;
    double a;
    const void* y;
    double b;
    const void* z;
    double c;
    long long n;
};

// r = c_q q + c_w1 w1 + c_w2 w2 + c_g M_soln Ntilde(u); optionally also copies u into q first
// (stage 1 starts the step with q^1 = u_k).
template <typename T, bool BATCH>
__global__ void __launch_bounds__(256) k_stage_rhs(StageRhsArgs a0, const StageRhsArgs* __restrict__ da, int per) {
    int bz = blockIdx.z, pb = 0;
    if constexpr (BATCH) {
        pb = bz / per;
        bz -= pb * per;
    }
    const StageRhsArgs& A = BATCH ? da[pb] : a0;
    const T* u = (const T*)A.u;
    T* q = (T*)A.q;
    const T* w1 = (const T*)A.w1;
    const T* w2 = (const T*)A.w2;
    T* r = (T*)A.r;
    const T idx_ = (T)A.idx;
    const StageCoef c = A.c;
    const int copy_q = c.copy_q, nx = A.nx, ny = A.ny, nz = A.nz;
    NSLGF_CELL_INDEX_Z(bz)
    Vec3<T> U = vec3(u, nx, ny, nz);
    const bool in_soln = in_domain(i, j, k, nx, ny, nz, c.nbuf, c.soln_blocks, c.nb);
    T nl[3] = {0, 0, 0};
    if (in_soln) {
        if (i >= 1 && i < nx - 1 && j >= 1 && j < ny - 1 && k >= 1 && k < nz - 1)
            nonlinear_at(unchecked(U), i, j, k, idx_, nl);
        else
            nonlinear_at(U, i, j, k, idx_, nl);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const long long p = a * n + idx;
        T qv;
        if (copy_q) {
            qv = u[p];
            q[p] = qv;
        } else {
            qv = q[p];
        }
        double v = c.c_q * (double)qv + c.c_g * (double)nl[a];
        if (w1) v += c.c_w1 * (double)w1[p];
        if (w2) v += c.c_w2 * (double)w2[p];
        r[p] = (T)v;
    }
}

// y = r - G dhat (into r); if wnew: wnew = (y - (c_q q + c_w1 w1 + c_w2 w2)) * inv
template <typename T, bool BATCH>
__global__ void __launch_bounds__(256) k_stage_project(StageProjArgs a0, const StageProjArgs* __restrict__ da,
                                                       int per) {
    int bz = blockIdx.z, pb = 0;
    if constexpr (BATCH) {
        pb = bz / per;
        bz -= pb * per;
    }
    const StageProjArgs& A = BATCH ? da[pb] : a0;
    const T* r = (const T*)A.r;
    T* rout = (T*)A.rout;
    const T* dhat = (const T*)A.dhat;
    const T* q = (const T*)A.q;
    const T* w1 = (const T*)A.w1;
    const T* w2 = (const T*)A.w2;
    const double c_q = A.c_q, c_w1 = A.c_w1, c_w2 = A.c_w2, inv = A.inv;
    T* wnew = (T*)A.wnew;
    const int nx = A.nx, ny = A.ny, nz = A.nz;
    const T idx_ = (T)A.idx;
    NSLGF_CELL_INDEX_Z(bz)
    Fld<T> D{dhat, nx, ny, nz};
    const T d0 = D(i, j, k);
    if (A.dout) ((T*)A.dout)[idx] = (T)(A.dscale * (double)d0);
    const T g[3] = {(D(i + 1, j, k) - d0) * idx_, (D(i, j + 1, k) - d0) * idx_, (D(i, j, k + 1) - d0) * idx_};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const long long p = a * n + idx;
        const T y = r[p] - g[a];
        rout[p] = y;
        if (wnew) {
            double base = c_q * (double)q[p];
            if (w1) base += c_w1 * (double)w1[p];
            if (w2) base += c_w2 * (double)w2[p];
            wnew[p] = (T)(((double)y - base) * inv);
        }
    }
}

// BATCH: the grid's y index is the problem.
template <typename T, bool BATCH>
__global__ void __launch_bounds__(256) k_axpby(AxpbyArgs a0, const AxpbyArgs* __restrict__ da) {
    const AxpbyArgs& A = BATCH ? da[blockIdx.y] : a0;
    T* out = (T*)A.out;
    const T* x = (const T*)A.x;
    const T* y = (const T*)A.y;
    const T* z = (const T*)A.z;
    const double a = A.a, b = A.b, c = A.c;
    const long long n = A.n;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    double v = a * (double)x[idx];
    if (y) v += b * (double)y[idx];
    if (z) v += c * (double)z[idx];
    out[idx] = (T)v;
}

// Plain streaming copy (16-byte vectors), the reference for hardware byte counters.
__global__ void __launch_bounds__(256) k_copy(const uint4* __restrict__ in, uint4* __restrict__ out, long long n16) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (long long)gridDim.x * blockDim.x)
        out[i] = in[i];
}

int launch_copy(const void* in, void* out, size_t bytes, hipStream_t s) {
    if (recording_unsupported()) return NSLGF_OK;
    if (bytes % 16 != 0 || ((uintptr_t)in % 16) != 0 || ((uintptr_t)out % 16) != 0) {
        set_error("copy: size and pointers must be multiples of 16 bytes");
        return NSLGF_EINVAL;
    }
    const long long n16 = (long long)(bytes / 16);
    hipLaunchKernelGGL(k_copy, dim3((unsigned)std::clamp((n16 + 255) / 256, 1LL, 4096LL)), dim3(256), 0, s,
                       (const uint4*)in, (uint4*)out, n16);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

// Largest cell-centred speed per workgroup; a wave walks whole rows (one index division per row), and the
// square root, monotone, is taken once of the largest square.
template <typename T>
__global__ void __launch_bounds__(256) k_max_speed(const T* u, int nx, int ny, int nz, double* partial) {
    const long long n = (long long)nx * ny * nz, sxy = (long long)nx * ny;
    __shared__ double red[256];
    double m = 0.0;
    const int nrows = ny * nz;
    for (int row = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6); row < nrows; row += (int)gridDim.x * 4) {
        const int k = row / ny, j = row - k * ny;
        const T* p = u + (long long)row * nx;
        for (int i = (int)threadIdx.x & 63; i < nx; i += 64) {
            const double a = 0.5 * ((double)p[i] + (double)(i > 0 ? p[i - 1] : (T)0));
            const double b = 0.5 * ((double)p[n + i] + (double)(j > 0 ? p[n + i - nx] : (T)0));
            const double c = 0.5 * ((double)p[2 * n + i] + (double)(k > 0 ? p[2 * n + i - sxy] : (T)0));
            m = fmax(m, a * a + b * b + c * c);
        }
    }
    red[threadIdx.x] = sqrt(m);
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Largest |u^(q)| over the three components on the solution domain (the box shrunk by nbuf points);
// one partial maximum per workgroup.
template <typename T>
__global__ void __launch_bounds__(256) k_max_abs(const T* u, int nx, int ny, int nz, int nbuf, double* partial) {
    const long long n = (long long)nx * ny * nz;
    __shared__ double red[256];
    double m = 0.0;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < 3 * n;
         idx += (long long)gridDim.x * blockDim.x) {
        const long long p = idx % n;
        const int i = (int)(p % nx);
        const int j = (int)((p / nx) % ny);
        const int k = (int)(p / ((long long)nx * ny));
        if (i >= nbuf && i < nx - nbuf && j >= nbuf && j < ny - nbuf && k >= nbuf && k < nz - nbuf)
            m = fmax(m, fabs((double)u[idx]));
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Volume integrals of an isolated vortex ring (Sec. 6.2, Eq. int_quantities) as 15 raw sums over the
// box, one set of partial sums per workgroup (partial[blockIdx.x * kDiagnosticSums + v]):
//   0..2   S_q    = sum (x cross w)_q              (I = dx^3 S / 2)
//   3..11  M_qp   = sum (x cross w)_q x_p          (X = dx^3 sum_q I_q M_q. / (2 |I|^2))
//   12     sum |w|^2                               (E = dx^3 sum / 2)
//   13     sum u_c . (x_c cross w_c)               (K = dx^3 sum)
//   14     sum u_c . w_c                           (J = dx^3 sum)
// with w = M_supp C u: zero outside the box and on edges closer than nbuf points to a face (there the
// curl of the zero-extended velocity sees a spurious jump).  The terms of S, M and |w|^2 are taken at the edge of
// each vorticity component (edge (q) is half a cell back along axis q); K and J average u (two faces)
// and w (four edges) to the cell centres.  Point (i, j, k) with offsets -1/2 on the flagged axes sits
// at origin + (i, j, k) dx - dx/2 on those axes.
// A workgroup takes a tile of 31 x 15 cells (32 x 16 threads: one more column and row below, whose edge
// values the averages need) and walks up to kDiagZ planes: every edge vorticity is formed once per tile,
// neighbours in the plane come through LDS and those of the plane below stay in registers.  (One thread per
// cell that formed its twelve edge values itself took 235 us at 192^3 in FP64, bound by instructions; this
// one 93.)  Small boxes are split along z until 256 workgroups or 4 planes each, as the walk's planes are its
// time there (a whole call: 48^3 42 us with a thread per cell, 54 in walks of 24 planes, 29 so; 96^3 68, 60, 46).
constexpr int kDiagX = 32, kDiagY = 16, kDiagZ = 24;
static dim3 diag_grid(int nx, int ny, int nz) {
    const int gx = ceil_div(nx, kDiagX - 1), gy = ceil_div(ny, kDiagY - 1);
    return dim3(gx, gy, std::max(ceil_div(nz, kDiagZ), std::min(ceil_div(nz, 4), ceil_div(256, gx * gy))));
}
int diagnostics_blocks(int nx, int ny, int nz) {
    const dim3 g = diag_grid(nx, ny, nz);
    return (int)(g.x * g.y * g.z);
}
template <typename T>
__global__ void __launch_bounds__(kDiagX* kDiagY) k_diagnostics(const T* u, int nx, int ny, int nz, int nbuf, T idx,
                                                               double dx, double ox, double oy, double oz,
                                                               double* partial) {
    const Vec3<T> U = vec3(u, nx, ny, nz);
    // tiles of equal size (none larger than 31 x 15 x kDiagZ)
    const int tx = (nx + gridDim.x - 1) / gridDim.x, ty = (ny + gridDim.y - 1) / gridDim.y,
              tz = (nz + gridDim.z - 1) / gridDim.z;
    const int lx = threadIdx.x % kDiagX, ly = threadIdx.x / kDiagX;
    const int i = (int)blockIdx.x * tx + lx - 1, j = (int)blockIdx.y * ty + ly - 1, k0 = (int)blockIdx.z * tz;
    const bool own = lx >= 1 && lx <= tx && i < nx && ly >= 1 && ly <= ty && j < ny;
    __shared__ T e[2][5][kDiagY][kDiagX];  // edge values (1), (2), (3), and the velocities u1, u2
    double acc[kDiagnosticSums];
#pragma unroll
    for (int v = 0; v < kDiagnosticSums; ++v) acc[v] = 0.0;
    const double xi = ox + i * dx, yj = oy + j * dx, h = 0.5 * dx;
    const bool in_xy = i >= nbuf && j >= nbuf && i < nx - nbuf && j < ny - nbuf && i >= 0 && j >= 0 && i < nx && j < ny;
    double s0 = 0.0, s1 = 0.0;  // sums over two edges of the plane below, for the cell-centre averages
    T u2m = (T)0;
    for (int k = k0 - 1; k < min(k0 + tz, nz); ++k) {
        T w[3] = {(T)0, (T)0, (T)0};
        if (in_xy && k >= nbuf && k < nz - nbuf && k >= 0)
#pragma unroll
            for (int q = 0; q < 3; ++q) w[q] = curl_at(U, q, i, j, k, idx);
        const T u0 = U.c[0](i, j, k), u1 = U.c[1](i, j, k), u2 = U.c[2](i, j, k);
        T(*p)[kDiagY][kDiagX] = e[k & 1];  // (two sets: one barrier per plane)
        p[0][ly][lx] = w[0];
        p[1][ly][lx] = w[1];
        p[2][ly][lx] = w[2];
        p[3][ly][lx] = u0;
        p[4][ly][lx] = u1;
        __syncthreads();
        if (own) {
            const double w0 = (double)w[0], w1 = (double)w[1], w2 = (double)w[2];
            const double t0 = w0 + (double)p[0][ly - 1][lx], t1 = w1 + (double)p[1][ly][lx - 1];
            if (k >= k0) {
                const double zk = oz + k * dx;
                const double we[3] = {w0, w1, w2};
                const double pe[3][3] = {{xi - h, yj, zk}, {xi, yj - h, zk}, {xi, yj, zk - h}};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int a = (q + 1) % 3, b = (q + 2) % 3;
                    // (x cross w)_q = x_a w_b - x_b w_a, each term at its own edge
                    const double tb = pe[b][a] * we[b], ta = pe[a][b] * we[a];
                    acc[q] += tb - ta;
#pragma unroll
                    for (int c = 0; c < 3; ++c) acc[3 + 3 * q + c] += tb * pe[b][c] - ta * pe[a][c];
                }
                acc[12] += w0 * w0 + w1 * w1 + w2 * w2;
                // cell centre
                const double uc[3] = {0.5 * ((double)u0 + (double)p[3][ly][lx - 1]),
                                      0.5 * ((double)u1 + (double)p[4][ly - 1][lx]), 0.5 * ((double)u2 + (double)u2m)};
                const double wc[3] = {0.25 * (t0 + s0), 0.25 * (t1 + s1),
                                      0.25 * ((w2 + (double)p[2][ly][lx - 1]) +
                                              ((double)p[2][ly - 1][lx] + (double)p[2][ly - 1][lx - 1]))};
                const double xc[3] = {xi - h, yj - h, zk - h};
                const double xw[3] = {xc[1] * wc[2] - xc[2] * wc[1], xc[2] * wc[0] - xc[0] * wc[2],
                                      xc[0] * wc[1] - xc[1] * wc[0]};
                acc[13] += uc[0] * xw[0] + uc[1] * xw[1] + uc[2] * xw[2];
                acc[14] += uc[0] * wc[0] + uc[1] * wc[1] + uc[2] * wc[2];
            }
            s0 = t0;
            s1 = t1;
            u2m = u2;
        }
    }
    // wave sums, then the waves' in order
    __shared__ double red[kDiagX * kDiagY / 64][kDiagnosticSums];
#pragma unroll
    for (int v = 0; v < kDiagnosticSums; ++v) {
        for (int o = 32; o > 0; o >>= 1) acc[v] += __shfl_xor(acc[v], o);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][v] = acc[v];
    }
    __syncthreads();
    if ((int)threadIdx.x < kDiagnosticSums) {
        double t = 0.0;
        for (int w = 0; w < kDiagX * kDiagY / 64; ++w) t += red[w][threadIdx.x];
        const long long b = ((long long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        partial[b * kDiagnosticSums + threadIdx.x] = t;
    }
}

// Block weights of the active domain (Sec. 4.3, Eq. weight_fun) per block of nb^3 cells (blocks tile the
// box from its origin; the last along an axis may be shorter): mu = the largest |(C u)^(q)| over the block's
// edges, nu = the largest |Dbar Ntilde(u)| over its cells (Ntilde(u) on the box, zero outside), both over
// the points at least nbuf away from every box face.
//
// A workgroup owns one layer of blocks of a tile of at most 16 x 16 points (whole blocks for nb <= 16, else a
// part of one block) and walks its planes from one below: Ntilde(u) of the tile and of one more column and
// row goes through LDS, the plane below stays in registers, so Ntilde(u) never reaches memory.  (A pass for
// Ntilde and one for the maxima took 94 + 92 us at 192^3 in FP64 with 16^3 blocks; this one 165, bound by
// the latency of its planes' loads, and it needs no temporary field.)  Parts of one block meet in
// an atomic maximum, exact in any order (mu and nu start at zero).
constexpr int kBwTile = 16, kBwThreads = 320;  // 17 x 17 points
template <typename T>
__global__ void __launch_bounds__(kBwThreads) k_block_weights(const T* u, int nx, int ny, int nz, int nb, int nbuf,
                                                             T idx, int tile, int parts, double* mu, double* nu) {
    const int bxn = (nx + nb - 1) / nb, byn = (ny + nb - 1) / nb;
    const Vec3<T> U = vec3(u, nx, ny, nz);
    // whole blocks: tiles side by side; parts of blocks: `parts` tiles per block and axis, the last one shorter
    const int px = (int)blockIdx.x / parts, py = (int)blockIdx.y / parts, step = parts > 1 ? nb : tile;
    const int i0 = px * step + ((int)blockIdx.x - px * parts) * tile, j0 = py * step + ((int)blockIdx.y - py * parts) * tile;
    const int i1 = min(min(px * step + step, i0 + tile), nx), j1 = min(min(py * step + step, j0 + tile), ny);
    const int k0 = (int)blockIdx.z * nb, k1 = min(k0 + nb, nz);
    const int ly = (int)threadIdx.x / (kBwTile + 1), lx = (int)threadIdx.x - ly * (kBwTile + 1);
    const int i = i0 + lx - 1, j = j0 + ly - 1;
    const bool here = i >= 0 && i < i1 && j >= 0 && j < j1;
    const bool own = here && lx >= 1 && ly >= 1 && i >= nbuf && j >= nbuf && i < nx - nbuf && j < ny - nbuf;
    const bool inner = i >= 1 && i < nx - 1 && j >= 1 && j < ny - 1;
    __shared__ T f[2][2][kBwTile + 1][kBwTile + 1];
    __shared__ unsigned long long red[2][kBwTile * kBwTile];
    for (int t = threadIdx.x; t < kBwTile * kBwTile; t += kBwThreads) red[0][t] = red[1][t] = 0ull;
    double m1 = 0.0, m2 = 0.0;
    T below = (T)0;
    for (int k = max(k0 - 1, 0); k < k1; ++k) {
        T nl[3] = {(T)0, (T)0, (T)0}, w[3] = {(T)0, (T)0, (T)0};
        if (here) {
            if (inner && k >= 1 && k < nz - 1)
                nonlinear_at(unchecked(U), i, j, k, idx, nl, w);
            else
                nonlinear_at(U, i, j, k, idx, nl, w);
        }
        T(*p)[kBwTile + 1][kBwTile + 1] = f[k & 1];  // (two sets: one barrier per plane)
        if (ly <= kBwTile) {
            p[0][ly][lx] = nl[0];
            p[1][ly][lx] = nl[1];
        }
        __syncthreads();
        if (own && k >= k0 && k >= nbuf && k < nz - nbuf) {
#pragma unroll
            for (int q = 0; q < 3; ++q) m1 = fmax(m1, fabs((double)w[q]));
            const T d = (nl[0] - p[0][ly][lx - 1] + nl[1] - p[1][ly - 1][lx] + nl[2] - below) * idx;
            m2 = fmax(m2, fabs((double)d));
        }
        below = nl[2];
    }
    // maxima per block of the tile (bit patterns of nonnegative doubles order like the values)
    const int per = parts == 1 ? tile / nb : 1;  // blocks per tile and axis
    if (own) {
        const int b = parts == 1 ? ((ly - 1) / nb) * per + (lx - 1) / nb : 0;
        atomicMax(&red[0][b], (unsigned long long)__double_as_longlong(m1));
        atomicMax(&red[1][b], (unsigned long long)__double_as_longlong(m2));
    }
    __syncthreads();
    for (int t = threadIdx.x; t < per * per; t += kBwThreads) {
        const int bi = i0 / nb + t % per, bj = j0 / nb + t / per;
        if (bi >= bxn || bj >= byn) continue;
        const long long b = ((long long)blockIdx.z * byn + bj) * bxn + bi;
        if (parts == 1) {
            mu[b] = __longlong_as_double((long long)red[0][t]);
            nu[b] = __longlong_as_double((long long)red[1][t]);
        } else {
            atomicMax((unsigned long long*)mu + b, red[0][t]);
            atomicMax((unsigned long long*)nu + b, red[1][t]);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
template <typename T>
static int stencil_t(int op, const void* src, void* dst, int ncomp, int nx, int ny, int nz, double dx, hipStream_t s,
                     int shape) {
    if (recording_unsupported()) return NSLGF_OK;
    const long long n = (long long)nx * ny * nz;
    const T idx_ = (T)(1.0 / dx);
    const dim3 grid = cell_grid(nx, ny, nz, 1, shape), block = cell_block(shape);
    switch (op) {
        case NSLGF_OP_GRAD: hipLaunchKernelGGL(k_grad<T>, grid, block, 0, s, (const T*)src, (T*)dst, nx, ny, nz, idx_); break;
        case NSLGF_OP_DIV: hipLaunchKernelGGL(k_div<T>, grid, block, 0, s, (const T*)src, (T*)dst, nx, ny, nz, idx_, 0); break;
        case NSLGF_OP_CURL: hipLaunchKernelGGL(k_curl<T>, grid, block, 0, s, (const T*)src, (T*)dst, nx, ny, nz, idx_, 0, nullptr, 0); break;
        case NSLGF_OP_CURL_BAR: hipLaunchKernelGGL(k_curl_bar<T>, grid, block, 0, s, (const T*)src, (T*)dst, nx, ny, nz, idx_); break;
        case NSLGF_OP_NONLINEAR: hipLaunchKernelGGL(k_nonlinear<T>, grid, block, 0, s, (const T*)src, (T*)dst, nx, ny, nz, idx_); break;
        case NSLGF_OP_LAPLACIAN:
            hipLaunchKernelGGL(k_laplacian<T>, cell_grid(nx, ny, nz, ncomp, shape), block, 0, s, (const T*)src, (T*)dst, nx,
                               ny, nz, (T)(1.0 / (dx * dx)));
            break;
        default: set_error("stencil_apply: unknown operator"); return NSLGF_EINVAL;
    }
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_stencil(int op, int dtype, const void* src, void* dst, int ncomp, int nx, int ny, int nz, double dx,
                   hipStream_t s, int shape) {
    if (dtype == NSLGF_F32) return stencil_t<float>(op, src, dst, ncomp, nx, ny, nz, dx, s, shape);
    return stencil_t<double>(op, src, dst, ncomp, nx, ny, nz, dx, s, shape);
}

// Batched launches: nprob problems' argument tables, one problem's grid (z extended by nprob).
template <typename T> static int batched_rhs(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_stage_rhs<T, true>), dim3(g.x, g.y, g.z * nprob), b, 0, s, StageRhsArgs{},
                       (const StageRhsArgs*)args, (int)g.z);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T> static int batched_proj(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_stage_project<T, true>), dim3(g.x, g.y, g.z * nprob), b, 0, s, StageProjArgs{},
                       (const StageProjArgs*)args, (int)g.z);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
template <typename T> static int batched_axpby(const void* args, int nprob, dim3 g, dim3 b, hipStream_t s) {
    hipLaunchKernelGGL((k_axpby<T, true>), dim3(g.x, nprob), b, 0, s, AxpbyArgs{}, (const AxpbyArgs*)args);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_stage_rhs(int dtype, const void* u, const void* q, const void* w1, const void* w2, void* r,
                     const StageCoef& c, int nx, int ny, int nz, double dx, hipStream_t s, int shape) {
    const StageRhsArgs a{u, (void*)q, w1, w2, r, 1.0 / dx, c, nx, ny, nz};
    const dim3 grid = cell_grid(nx, ny, nz, 1, shape), block = cell_block(shape);
    if (launch_recorder()) {
        record_launch(dtype == NSLGF_F32 ? &batched_rhs<float> : &batched_rhs<double>, grid, block, a);
        return NSLGF_OK;
    }
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL((k_stage_rhs<float, false>), grid, block, 0, s, a, nullptr, 0);
    else
        hipLaunchKernelGGL((k_stage_rhs<double, false>), grid, block, 0, s, a, nullptr, 0);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_masked_div(int dtype, const void* r, void* sdiv, int nbuf, int nx, int ny, int nz, double dx,
                      hipStream_t s) {
    if (recording_unsupported()) return NSLGF_OK;
    const long long n = (long long)nx * ny * nz;
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL(k_div<float>, cell_grid(nx, ny, nz), cell_block(0), 0, s, (const float*)r, (float*)sdiv, nx,
                           ny, nz, (float)(1.0 / dx), nbuf);
    else
        hipLaunchKernelGGL(k_div<double>, cell_grid(nx, ny, nz), cell_block(0), 0, s, (const double*)r, (double*)sdiv, nx,
                           ny, nz, 1.0 / dx, nbuf);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_stage_project(int dtype, const void* r, void* rout, const void* dhat, const void* q, const void* w1,
                         const void* w2, double c_q, double c_w1, double c_w2, void* wnew, double inv, int nx, int ny,
                         int nz, double dx, hipStream_t s, int shape, void* dout, double dscale) {
    const StageProjArgs a{r, rout, dhat, q, w1, w2, c_q, c_w1, c_w2, wnew, inv, 1.0 / dx, nx, ny, nz, dout, dscale};
    const dim3 grid = cell_grid(nx, ny, nz, 1, shape), block = cell_block(shape);
    if (launch_recorder()) {
        record_launch(dtype == NSLGF_F32 ? &batched_proj<float> : &batched_proj<double>, grid, block, a);
        return NSLGF_OK;
    }
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL((k_stage_project<float, false>), grid, block, 0, s, a, nullptr, 0);
    else
        hipLaunchKernelGGL((k_stage_project<double, false>), grid, block, 0, s, a, nullptr, 0);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_axpby(int dtype, void* out, const void* x, double a, const void* y, double b, const void* z, double c,
                 long long n, hipStream_t s) {
    const AxpbyArgs args{out, x, a, y, b, z, c, n};
    const dim3 grid(ceil_div(n, 256)), block(256);
    if (launch_recorder()) {
        record_launch(dtype == NSLGF_F32 ? &batched_axpby<float> : &batched_axpby<double>, grid, block, args);
        return NSLGF_OK;
    }
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL((k_axpby<float, false>), grid, block, 0, s, args, nullptr);
    else
        hipLaunchKernelGGL((k_axpby<double, false>), grid, block, 0, s, args, nullptr);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_masked_curl(int dtype, const void* f, void* e, int nbuf, const unsigned char* blocks, int nb, int nx, int ny,
                       int nz, double dx, hipStream_t s, int shape) {
    if (recording_unsupported()) return NSLGF_OK;
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL(k_curl<float>, cell_grid(nx, ny, nz, 1, shape), cell_block(shape), 0, s, (const float*)f, (float*)e, nx, ny,
                           nz, (float)(1.0 / dx), nbuf, blocks, nb);
    else
        hipLaunchKernelGGL(k_curl<double>, cell_grid(nx, ny, nz, 1, shape), cell_block(shape), 0, s, (const double*)f, (double*)e, nx,
                           ny, nz, 1.0 / dx, nbuf, blocks, nb);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_max_abs(int dtype, const void* u, int nbuf, int nx, int ny, int nz, double* dev_partial, int nblocks,
                   hipStream_t s) {
    if (recording_unsupported()) return NSLGF_OK;
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL(k_max_abs<float>, dim3(nblocks), dim3(256), 0, s, (const float*)u, nx, ny, nz, nbuf,
                           dev_partial);
    else
        hipLaunchKernelGGL(k_max_abs<double>, dim3(nblocks), dim3(256), 0, s, (const double*)u, nx, ny, nz, nbuf,
                           dev_partial);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

int launch_diagnostics(int dtype, const void* u, int nbuf, int nx, int ny, int nz, double dx, const double origin[3],
                       double* partial, hipStream_t s) {
    if (recording_unsupported()) return NSLGF_OK;
    const dim3 grid = diag_grid(nx, ny, nz), block(kDiagX * kDiagY);
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL(k_diagnostics<float>, grid, block, 0, s, (const float*)u, nx, ny, nz, nbuf, (float)(1.0 / dx),
                           dx, origin[0], origin[1], origin[2], partial);
    else
        hipLaunchKernelGGL(k_diagnostics<double>, grid, block, 0, s, (const double*)u, nx, ny, nz, nbuf, 1.0 / dx, dx,
                           origin[0], origin[1], origin[2], partial);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

template <typename T>
static int block_weights_t(const T* u, int nx, int ny, int nz, int nb, int nbuf, double dx, double* mu, double* nu,
                           hipStream_t s) {
    const int parts = ceil_div(nb, kBwTile);
    const int tile = parts == 1 ? kBwTile / nb * nb : ceil_div(nb, parts);
    const dim3 grid = parts == 1 ? dim3(ceil_div(nx, tile), ceil_div(ny, tile), ceil_div(nz, nb))
                                 : dim3(ceil_div(nx, nb) * parts, ceil_div(ny, nb) * parts, ceil_div(nz, nb));
    if (parts > 1) {
        const long long nblocks = (long long)ceil_div(nx, nb) * ceil_div(ny, nb) * ceil_div(nz, nb);
        NSLGF_TRY(launch_zero(NSLGF_F64, mu, nblocks, s));
        NSLGF_TRY(launch_zero(NSLGF_F64, nu, nblocks, s));
    }
    hipLaunchKernelGGL(k_block_weights<T>, grid, dim3(kBwThreads), 0, s, u, nx, ny, nz, nb, nbuf, (T)(1.0 / dx), tile, parts,
                       mu, nu);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}
int launch_block_weights(int dtype, const void* u, int nx, int ny, int nz, int nb, int nbuf, double dx, double* mu,
                         double* nu, hipStream_t s) {
    if (recording_unsupported()) return NSLGF_OK;
    if (dtype == NSLGF_F32) return block_weights_t<float>((const float*)u, nx, ny, nz, nb, nbuf, dx, mu, nu, s);
    return block_weights_t<double>((const double*)u, nx, ny, nz, nb, nbuf, dx, mu, nu, s);
}

int launch_max_speed(int dtype, const void* u, int nx, int ny, int nz, double* dev_partial, int nblocks,
                     hipStream_t s) {
    if (recording_unsupported()) return NSLGF_OK;
    if (dtype == NSLGF_F32)
        hipLaunchKernelGGL(k_max_speed<float>, dim3(nblocks), dim3(256), 0, s, (const float*)u, nx, ny, nz, dev_partial);
    else
        hipLaunchKernelGGL(k_max_speed<double>, dim3(nblocks), dim3(256), 0, s, (const double*)u, nx, ny, nz,
                           dev_partial);
    NSLGF_LAUNCH_CHECK();
    return NSLGF_OK;
}

}  // namespace nslgf
