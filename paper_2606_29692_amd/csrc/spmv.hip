// sigma = S psi with the FP64 energy reduction (Eq. 1) fused into the epilogue.
//
// Row-bucketed CSR-vector product: a sub-group of L lanes (L = 8..64, fixed
// per operator) owns one row, streams its column indices and values with
// coalesced loads (four strided loads in flight per lane), gathers psi from
// L2, multiplies in FP64 and reduces with a butterfly.  The sub-group leader
// writes sigma_r and accumulates conj(psi_r) sigma_r and |psi_r|^2; each
// workgroup writes one FP64 partial triple, and a one-wave-per-state kernel
// sums the partials in a fixed order.  The grid is either one state (block b
// -> rows of b) or a batch task table built so that all blocks of a state run
// on the same XCD (workgroup IDs are dealt round-robin over the 8 XCDs).
#include "kernels.hpp"

#include <algorithm>

// The LDS schedules hold the state in LDS, so one 16-wave workgroup fills a
// CU (4 waves per SIMD): the register allocator may use the whole budget.
#define VQE_LDS_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4, 4)))

namespace {

// V = entries per lane per pass.  V = 1: lane l of the sub-group takes
// entries k0 + l, k0 + l + L, ...  V = 4: lanes take aligned groups of four
// consecutive entries (one 16-byte index load and 32- or 64-byte value loads),
// masked to the row; a 64-lane sub-group covers 256 entries per pass.
template <int DT, int V> struct RowLoad;

template <int DT> struct RowLoad<DT, 1> {
    using T = typename Elem<DT>::T;
    static __device__ __forceinline__ void load(const int32_t *col, const T *val, int k, int k0,
                                                int k1, int64_t nnz, int c[1], T v[1])
    {
        (void)k0;
        (void)nnz;
        if (k < k1) {
            c[0] = __builtin_nontemporal_load(gmem(col) + k);
            v[0] = ldg(val, k);
        } else {
            c[0] = -1;
        }
    }
};

// Four consecutive values from a 32-byte (c64) or 64-byte (c128) aligned address.
__device__ __forceinline__ void load4(const float2 *p, float2 v[4])
{
    const vqe_v4f a = gmem(reinterpret_cast<const vqe_v4f *>(p))[0];
    const vqe_v4f b = gmem(reinterpret_cast<const vqe_v4f *>(p))[1];
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
}

__device__ __forceinline__ void load4(const double2 *p, double2 v[4])
{
#pragma unroll
    for (int u = 0; u < 4; u++)
        v[u] = ldg(p, u);
}

template <int DT> struct RowLoad<DT, 4> {
    using T = typename Elem<DT>::T;
    static __device__ __forceinline__ void load(const int32_t *col, const T *val, int k, int k0,
                                                int k1, int64_t nnz, int c[4], T v[4])
    {
        if (k >= k1) {
            // the whole group lies past the row: no load at all
#pragma unroll
            for (int u = 0; u < 4; u++)
                c[u] = -1;
            return;
        }
        if ((int64_t)k + 3 < nnz) {
            typedef int v4i __attribute__((ext_vector_type(4)));
            const v4i c4 = __builtin_nontemporal_load(gmem(reinterpret_cast<const v4i *>(col + k)));
            c[0] = c4.x;
            c[1] = c4.y;
            c[2] = c4.z;
            c[3] = c4.w;
            load4(val + k, v);
        } else {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if ((int64_t)(k + u) < nnz) {
                    c[u] = gmem(col)[k + u];
                    v[u] = ldg(val, k + u);
                } else {
                    c[u] = -1;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (k + u < k0 || k + u >= k1)
                c[u] = -1;
    }
};

// Wave wid (of four) of block blk: its rows of sigma, and its sums of the
// energy terms (each over the whole wave).
template <int DT, int L, int V>
__device__ __forceinline__ void spmv_energy_rows(const SpmvState &st, int blk, int wid, int lane, double &e_re,
                                                 double &e_im, double &e_n2)
{
    constexpr int G = VQE_WAVE / L;
    constexpr int RPB = spmv_rows_per_block(L);
    constexpr int U = V == 1 ? 4 : 1;     // passes issued together
    const int sub = lane / L, sl = lane % L;
    const int32_t *__restrict__ rowptr = st.rowptr;
    const int32_t *__restrict__ col = st.col;
    using T = typename Elem<DT>::T;
    const T *__restrict__ val = reinterpret_cast<const T *>(st.val);
    e_re = e_im = e_n2 = 0.0;
#pragma unroll
    for (int it = 0; it < SPMV_RPT; it++) {
        const int64_t r = (int64_t)blk * RPB + (it * 4 + wid) * G + sub;
        double are = 0.0, aim = 0.0;
        if (r < st.dim) {
            const int k0 = gmem(rowptr)[r], k1 = gmem(rowptr)[r + 1];
            const int first = V == 1 ? k0 + sl : (k0 & ~3) + 4 * sl;
            for (int k = first; k < k1; k += U * V * L) {
                int c[U * V];
                T v[U * V];
#pragma unroll
                for (int u = 0; u < U; u++)
                    RowLoad<DT, V>::load(col, val, k + u * V * L, k0, k1, st.nnz, c + u * V,
                                         v + u * V);
#pragma unroll
                for (int u = 0; u < U * V; u++) {
                    if (c[u] >= 0) {
                        const double2 x = Elem<DT>::ld(st.psi, c[u]);
                        const double ar = (double)v[u].x, ai = (double)v[u].y;
                        are += ar * x.x - ai * x.y;
                        aim += ar * x.y + ai * x.x;
                    }
                }
            }
        }
        are = group_sum<L>(are);
        aim = group_sum<L>(aim);
        if (sl == 0 && r < st.dim) {
            Elem<DT>::st(st.sigma, r, make_double2(are, aim));
            const double2 p = Elem<DT>::ld(st.psi, r);
            e_re += p.x * are + p.y * aim;
            e_im += p.x * aim - p.y * are;
            e_n2 += p.x * p.x + p.y * p.y;
        }
    }
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
}

template <int DT, int L, int V, bool BATCH>
__global__ void __launch_bounds__(256)
k_spmv_energy(SpmvState single, const SpmvState *__restrict__ states,
              const int2 *__restrict__ tasks)
{
    SpmvState st;
    int blk;
    if (BATCH) {
        int2 t = tasks[blockIdx.x];
        if (t.x < 0)
            return;
        st = states[t.x];
        blk = t.y;
        if (VQE_SKIP(st))
            return;
    } else {
        st = single;
        blk = blockIdx.x;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    double e_re, e_im, e_n2;
    spmv_energy_rows<DT, L, V>(st, blk, wid, lane, e_re, e_im, e_n2);
    __shared__ double s_part[4][3];
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int q = threadIdx.x;
        const double v = ((s_part[0][q] + s_part[1][q]) + s_part[2][q]) + s_part[3][q];
        gmem(st.partials)[(int64_t)blk * 3 + q] = v;
    }
}

// A small single state in one workgroup, product, block sums and energy (the
// same sums as k_spmv_energy and k_energy_finalize): up to SPMV_SMALL_DIM rows a
// call is two launches' cost on the host rather than work, as long as one
// workgroup has few entries to read (a call among others 8.4 us, one launch 5.0
// at 4 to 7 qubits of up to 16 entries a row, 5.7 at 6 of 64, 7.8 at 8 of 16;
// at 7 of 64, 8192 entries, level and alone 19.4 against 18.2, at 8 of 64
// 13.4 against 8.4).
#define SPMV_SMALL_DIM 256
#define SPMV_SMALL_NNZ 5120
template <int DT, int L>
__global__ void __launch_bounds__(1024)
k_spmv_energy_small(SpmvState st)
{
    constexpr int NB = (SPMV_SMALL_DIM + spmv_rows_per_block(L) - 1) / spmv_rows_per_block(L);
    static_assert(NB <= VQE_WAVE, "a block sum per lane");
    __shared__ double s_part[NB][4][3], s_sum[3];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int b = wid >> 2; b < st.nblocks; b += 4) {
        double e_re, e_im, e_n2;
        spmv_energy_rows<DT, L, 1>(st, b, wid & 3, lane, e_re, e_im, e_n2);
        if (lane == 0) {
            s_part[b][wid & 3][0] = e_re;
            s_part[b][wid & 3][1] = e_im;
            s_part[b][wid & 3][2] = e_n2;
        }
    }
    __syncthreads();
    if (wid < 3) {
        double v = 0.0;
        if (lane < st.nblocks)
            v = ((s_part[lane][0][wid] + s_part[lane][1][wid]) + s_part[lane][2][wid]) + s_part[lane][3][wid];
        v = wave_sum(v);
        if (lane == 0)
            s_sum[wid] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0 && st.energy_out) {
        st.energy_out[0] = st.shift + s_sum[0] / s_sum[2];
        st.energy_out[1] = s_sum[2];
        st.energy_out[2] = s_sum[1];
    }
}

// Loads of the LDS schedules: four consecutive entries from an aligned group
// k (16-byte index load, 32- or 64-byte value load).  Entries outside the
// row [k0, k1) get column zc, the index of a zero element kept after the
// state in LDS, so the multiply needs no per-entry select: their values are
// finite (entries of a neighbouring row, or zero) and multiply that zero.
// Only groups that reach past the end of the arrays (k + 4 > nnz) take the
// entry-by-entry path.  All index arithmetic is 32-bit (nnz < 2^31).
template <int DT>
__device__ __forceinline__ void lds_group_load(const int32_t *col, const typename Elem<DT>::T *val,
                                               int k, int k0, int k1, int nnz, int zc, int c[4],
                                               typename Elem<DT>::T v[4])
{
    using T = typename Elem<DT>::T;
    if (k >= k1) {
        // the whole group lies past the row: no load at all
#pragma unroll
        for (int u = 0; u < 4; u++) {
            c[u] = zc;
            v[u] = T{};
        }
        return;
    }
    if (k + 4 <= nnz) {
        typedef int v4i __attribute__((ext_vector_type(4)));
        const v4i c4 = __builtin_nontemporal_load(gmem(reinterpret_cast<const v4i *>(col + k)));
        c[0] = c4.x;
        c[1] = c4.y;
        c[2] = c4.z;
        c[3] = c4.w;
        load4(val + k, v);
    } else {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (k + u < nnz) {
                c[u] = gmem(col)[k + u];
                v[u] = ldg(val, k + u);
            } else {
                c[u] = zc;
                v[u] = T{};
            }
        }
    }
    // entry k + u belongs to the row iff 0 <= k + u - k0 < k1 - k0
    const unsigned len = (unsigned)(k1 - k0);
#pragma unroll
    for (int u = 0; u < 4; u++)
        c[u] = (unsigned)(k + u - k0) < len ? c[u] : zc;
}

// Gathers from the LDS copy of the state and FP64 multiply-accumulate.  All
// LDS reads issue back to back behind a single wait; masked entries read the
// zero element.
__device__ __forceinline__ float2 stage_load(const float2 *p, int64_t i) { return ldg(p, i); }
__device__ __forceinline__ double2 stage_load(const double2 *p, int64_t i) { return ldg(p, i); }
__device__ __forceinline__ int32_t stage_load(const int32_t *p, int64_t i) { return gmem(p)[i]; }

// Copy n elements from global memory to LDS with the workgroup's 1024
// threads: each thread issues SB loads before the batch's LDS writes, so it
// waits for memory once per batch instead of once per element.
template <int SB, typename T>
__device__ __forceinline__ void stage_lds(T *dst, const T *src, int64_t n, int tid)
{
    for (int64_t i0 = tid; i0 < n; i0 += 1024 * SB) {
        T v[SB];
#pragma unroll
        for (int u = 0; u < SB; u++) {
            const int64_t i = i0 + 1024 * (int64_t)u;
            if (i < n)
                v[u] = stage_load(src, i);
        }
#pragma unroll
        for (int u = 0; u < SB; u++) {
            const int64_t i = i0 + 1024 * (int64_t)u;
            if (i < n)
                dst[i] = v[u];
        }
    }
}

// The real parts of a state staged in LDS as FP64; returns nonzero when an
// element of this thread's share has a nonzero imaginary part.
template <int SB, typename T>
__device__ __forceinline__ int stage_real(double *dst, const T *src, int64_t n, int tid)
{
    int cplx = 0;
    for (int64_t i0 = tid; i0 < n; i0 += 1024 * SB) {
        T v[SB];
#pragma unroll
        for (int u = 0; u < SB; u++) {
            const int64_t i = i0 + (int64_t)u * 1024;
            if (i < n)
                v[u] = stage_load(src, i);
        }
#pragma unroll
        for (int u = 0; u < SB; u++) {
            const int64_t i = i0 + (int64_t)u * 1024;
            if (i < n) {
                dst[i] = (double)v[u].x;
                cplx |= v[u].y != 0;
            }
        }
    }
    return cplx;
}

// The real parts of a state staged in LDS in a given precision (FP32 real
// parts of FP32 storage stay exact); returns nonzero when an element of this
// thread's share has a nonzero imaginary part.
template <int SB, typename R, typename T>
__device__ __forceinline__ int stage_real_as(R *dst, const T *src, int64_t n, int tid)
{
    int cplx = 0;
    for (int64_t i0 = tid; i0 < n; i0 += 1024 * SB) {
        T v[SB];
#pragma unroll
        for (int u = 0; u < SB; u++) {
            const int64_t i = i0 + (int64_t)u * 1024;
            if (i < n)
                v[u] = stage_load(src, i);
        }
#pragma unroll
        for (int u = 0; u < SB; u++) {
            const int64_t i = i0 + (int64_t)u * 1024;
            if (i < n) {
                dst[i] = (R)v[u].x;
                cplx |= v[u].y != 0;
            }
        }
    }
    return cplx;
}

// One entry's product a * x added to (are, aim) in FP64: a complex value, or
// the real part alone when the operator is stored with real values.
template <typename T>
__device__ __forceinline__ void entry_fma(const float2 a, const T x, double &are, double &aim)
{
    const double ar = (double)a.x, ai = (double)a.y, xr = (double)x.x, xi = (double)x.y;
    are += ar * xr - ai * xi;
    aim += ar * xi + ai * xr;
}
template <typename T>
__device__ __forceinline__ void entry_fma(const double2 a, const T x, double &are, double &aim)
{
    const double ar = a.x, ai = a.y, xr = (double)x.x, xi = (double)x.y;
    are += ar * xr - ai * xi;
    aim += ar * xi + ai * xr;
}
template <typename T>
__device__ __forceinline__ void entry_fma(const float a, const T x, double &are, double &aim)
{
    are += (double)a * (double)x.x;
    aim += (double)a * (double)x.y;
}
template <typename T>
__device__ __forceinline__ void entry_fma(const double a, const T x, double &are, double &aim)
{
    are += a * (double)x.x;
    aim += a * (double)x.y;
}

// Entries against a real state (its real parts in FP64): the imaginary sum
// stays zero.
__device__ __forceinline__ void entry_fma(const float a, const double x, double &are, double &aim)
{
    (void)aim;
    are += (double)a * x;
}
__device__ __forceinline__ void entry_fma(const double a, const double x, double &are, double &aim)
{
    (void)aim;
    are += a * x;
}
__device__ __forceinline__ void entry_fma(const float a, const float x, double &are, double &aim)
{
    (void)aim;
    are += (double)a * (double)x;
}

// A row's terms of <psi|sigma> and <psi|psi> from its state element.
template <typename T>
__device__ __forceinline__ void energy_terms(const T ps, double are, double aim, double &e_re,
                                             double &e_im, double &e_n2)
{
    const double px = (double)ps.x, py = (double)ps.y;
    e_re += px * are + py * aim;
    e_im += px * aim - py * are;
    e_n2 += px * px + py * py;
}
__device__ __forceinline__ void energy_terms(const double px, double are, double aim, double &e_re,
                                             double &e_im, double &e_n2)
{
    (void)aim;
    (void)e_im;
    e_re += px * are;
    e_n2 += px * px;
}

template <typename T, typename V, int N>
__device__ __forceinline__ void lds_gather_fma(const T *s_x, const int c[N], const V v[N],
                                               double &are, double &aim)
{
    T xs[N];
#pragma unroll
    for (int u = 0; u < N; u++)
        xs[u] = s_x[c[u]];
#pragma unroll
    for (int u = 0; u < N; u++)
        entry_fma(v[u], xs[u], are, aim);
}

// The whole state vector staged in LDS (one 128 KB copy for 14 qubits in
// FP32 storage), so every gather of the product is an LDS read instead of an
// L2 request.  A workgroup of 16 waves owns SPMV_LDS_ROWS consecutive rows of
// one state; sub-groups of L lanes read their rows with the four-entry wide
// loads, U passes in flight.
template <int DT, int L, int U, bool BATCH>
__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_lds(SpmvState single, const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    SpmvState st;
    int blk;
    if (BATCH) {
        int2 t = tasks[blockIdx.x];
        if (t.x < 0)
            return;
        st = states[t.x];
        blk = t.y;
        if (VQE_SKIP(st))
            return;
    } else {
        st = single;
        blk = blockIdx.x;
    }
    using T = typename Elem<DT>::T;
    extern __shared__ unsigned char smem[];
    T *s_x = reinterpret_cast<T *>(smem);
    const int tid = threadIdx.x;
    const int64_t dim = st.dim;
    const T *__restrict__ psi = reinterpret_cast<const T *>(st.psi);
    const int64_t r0 = (int64_t)blk * SPMV_LDS_ROWS;
    const int64_t r1 = r0 + SPMV_LDS_ROWS < dim ? r0 + SPMV_LDS_ROWS : dim;
    // the state, one zero element (index dim), then the workgroup's row pointers
    int32_t *s_rp = reinterpret_cast<int32_t *>(smem + (size_t)(dim + 1) * sizeof(T));
    stage_lds<8>(s_x, psi, dim, tid);
    if (tid == 0)
        s_x[dim] = T{};
    stage_lds<4>(s_rp, st.rowptr + r0, r1 - r0 + 1, tid);
    __syncthreads();

    constexpr int G = VQE_WAVE / L;
    const int lane = tid & 63, wid = tid >> 6;
    const int sub = lane / L, sl = lane % L;
    const int32_t *__restrict__ col = st.col;
    const T *__restrict__ val = reinterpret_cast<const T *>(st.val);
    const int nnz = (int)st.nnz, zc = (int)dim;
    double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;
    for (int64_t base = r0 + wid * G; base < r1; base += 16 * G) {
        const int64_t r = base + sub;
        double are = 0.0, aim = 0.0;
        if (r < r1) {
            const int k0 = s_rp[r - r0], k1 = s_rp[r - r0 + 1];
            for (int k = (k0 & ~3) + 4 * sl; k < k1; k += U * 4 * L) {
                int c[U * 4];
                T v[U * 4];
#pragma unroll
                for (int u = 0; u < U; u++)
                    lds_group_load<DT>(col, val, k + u * 4 * L, k0, k1, nnz, zc, c + 4 * u,
                                       v + 4 * u);
                lds_gather_fma<T, T, U * 4>(s_x, c, v, are, aim);
            }
        }
        are = group_sum<L>(are);
        aim = group_sum<L>(aim);
        if (sl == 0 && r < r1) {
            Elem<DT>::st(st.sigma, r, make_double2(are, aim));
            const T ps = s_x[r];
            const double px = (double)ps.x, py = (double)ps.y;
            e_re += px * are + py * aim;
            e_im += px * aim - py * are;
            e_n2 += px * px + py * py;
        }
    }
    __shared__ double s_part[16][3];
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (tid < 3) {
        double v = 0.0;
        for (int w = 0; w < 16; w++)
            v += s_part[w][tid];
        gmem(st.partials)[(int64_t)blk * 3 + tid] = v;
    }
}

// Raw buffer resources (gfx9 descriptor word 3): a load whose offset lies at
// or past num_records returns zero and makes no memory request.
#define VQE_BUF_WORD3 0x00020000
#define VQE_BUF_OOB 0x80000000u

// Value streamed per entry: the complex value, or its real part alone (RV)
// when the plan stores the operator's real parts (an operator whose entries
// are all real).
template <int DT, bool RV> struct ValOf { using T = typename Elem<DT>::T; };
template <> struct ValOf<VQE_C64, true> { using T = float; };
template <> struct ValOf<VQE_C128, true> { using T = double; };

__device__ __forceinline__ float2 ldv(const float2 *p, int64_t i) { return ldg(p, i); }
__device__ __forceinline__ double2 ldv(const double2 *p, int64_t i) { return ldg(p, i); }
__device__ __forceinline__ float ldv(const float *p, int64_t i) { return gmem(p)[i]; }
__device__ __forceinline__ double ldv(const double *p, int64_t i) { return gmem(p)[i]; }

template <int DT, bool RV> struct BufVal;
template <> struct BufVal<VQE_C64, false> {
    // four consecutive complex64 values: two 16-byte loads
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned off, float2 v[4])
    {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const v4f a = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        const v4f b = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16, 0, 0);
        v[0] = make_float2(a.x, a.y);
        v[1] = make_float2(a.z, a.w);
        v[2] = make_float2(b.x, b.y);
        v[3] = make_float2(b.z, b.w);
    }
};
template <> struct BufVal<VQE_C128, false> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned off, double2 v[4])
    {
        typedef double v2d __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const v2d a = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * u, 0, 0);
            v[u] = make_double2(a.x, a.y);
        }
    }
};
template <> struct BufVal<VQE_C64, true> {
    // four consecutive real FP32 values: one 16-byte load
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned off, float v[4])
    {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const v4f a = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        v[0] = a.x;
        v[1] = a.y;
        v[2] = a.z;
        v[3] = a.w;
    }
};
template <> struct BufVal<VQE_C128, true> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned off, double v[4])
    {
        typedef double v2d __attribute__((ext_vector_type(2)));
        const v2d a = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        const v2d b = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16, 0, 0);
        v[0] = a.x;
        v[1] = a.y;
        v[2] = b.x;
        v[3] = b.y;
    }
};

// Real parts of an operator's values (for operators whose entries are all real).
template <int DT>
__global__ void __launch_bounds__(256)
k_val_real(const void *__restrict__ val, void *__restrict__ out, int64_t nnz)
{
    using T = typename Elem<DT>::T;
    using R = typename ValOf<DT, true>::T;
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < nnz)
        reinterpret_cast<R *>(out)[k] = ldg(reinterpret_cast<const T *>(val), k).x;
}

// Column codes of the 16-bit form: one wave per row, lanes over its entries.
__global__ void __launch_bounds__(256)
k_col_xor16(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
            uint16_t *__restrict__ col16, int64_t dim)
{
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= dim)
        return;
    const int32_t k1 = rowptr[r + 1];
    for (int32_t k = rowptr[r] + (int32_t)(threadIdx.x & 63); k < k1; k += 64)
        col16[k] = (uint16_t)((uint32_t)col[k] ^ (uint32_t)r);
}

// Row pointers of the padded layout, in which every row's length is rounded up
// to a multiple of SPMV_PAD.  One workgroup: each thread takes a contiguous run of
// rows, the workgroup scans the run totals, and each thread writes its run.
__global__ void __launch_bounds__(1024)
k_pad_rowptr(const int32_t *__restrict__ rowptr, int32_t *__restrict__ prow, int64_t dim)
{
    __shared__ int64_t s_sum[1024];
    const int tid = threadIdx.x;
    const int64_t per = (dim + 1023) / 1024;
    const int64_t a = (int64_t)tid * per < dim ? (int64_t)tid * per : dim;
    const int64_t b = a + per < dim ? a + per : dim;
    int64_t tot = 0;
    // the run's row pointers a batch at a time (independent loads)
    constexpr int NB = 16;
    for (int64_t r0 = a; r0 < b; r0 += NB) {
        int32_t p[NB + 1];
#pragma unroll
        for (int i = 0; i <= NB; i++)
            p[i] = r0 + i <= b ? rowptr[r0 + i] : 0;
#pragma unroll
        for (int i = 0; i < NB; i++)
            if (r0 + i < b)
                tot += (p[i + 1] - p[i] + SPMV_PAD - 1) & ~(SPMV_PAD - 1);
    }
    s_sum[tid] = tot;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t v = tid >= off ? s_sum[tid - off] : 0;
        __syncthreads();
        s_sum[tid] += v;
        __syncthreads();
    }
    int64_t run = s_sum[tid] - tot;
    for (int64_t r0 = a; r0 < b; r0 += NB) {
        int32_t p[NB + 1];
#pragma unroll
        for (int i = 0; i <= NB; i++)
            p[i] = r0 + i <= b ? rowptr[r0 + i] : 0;
#pragma unroll
        for (int i = 0; i < NB; i++)
            if (r0 + i < b) {
                prow[r0 + i] = (int32_t)run;
                run += (p[i + 1] - p[i] + SPMV_PAD - 1) & ~(SPMV_PAD - 1);
            }
    }
    if (tid == 1023)
        prow[dim] = (int32_t)s_sum[1023];
}

// Column codes and values in the padded layout, one wave per row: the real
// parts (RVAL) or the complex values themselves; a row's pad entries repeat
// its last column with the value zero.
template <int DT, bool RVAL>
__global__ void __launch_bounds__(256)
k_pad_fill(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
           const void *__restrict__ val, const int32_t *__restrict__ prow,
           uint16_t *__restrict__ code, void *__restrict__ vpad, int64_t dim)
{
    using T = typename Elem<DT>::T;
    using R = typename ValOf<DT, RVAL>::T;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= dim)
        return;
    const int32_t k0 = rowptr[r], len = rowptr[r + 1] - k0;
    const int32_t p0 = prow[r], plen = prow[r + 1] - p0;
    for (int32_t j = (int32_t)(threadIdx.x & 63); j < plen; j += 64) {
        const int32_t k = k0 + (j < len ? j : len - 1);
        code[p0 + j] = (uint16_t)((uint32_t)col[k] ^ (uint32_t)r);
        R v{};
        if (j < len) {
            if constexpr (RVAL)
                v = (R)ldg(reinterpret_cast<const T *>(val), k).x;
            else
                v = ldg(reinterpret_cast<const T *>(val), k);
        }
        reinterpret_cast<R *>(vpad)[p0 + j] = v;
    }
}

// Pipelined variant of the LDS schedule.  A sub-group of L lanes covers a row
// of up to U * GE * L = 256 entries in one pass (GE entries per lane group: 4,
// or 8 in the padded layout) and keeps the loads of its next
// D rows in flight: after a row's products it refills that row's registers
// with the row D sweeps ahead.  The loads are raw buffer loads issued by every
// lane without branches: groups past the row (or past the last whole group of
// the arrays) get an out-of-range offset and return zero without a memory
// request.  Because the number of loads per row is fixed, the wait before one
// row's products leaves the other rows' loads outstanding (the scheduling
// barriers keep each refill issued before the next row is consumed).  Rows
// longer than one pass finish with further passes, and the last nnz % 4
// entries of the arrays are added entry by entry.  With X16 the column of
// entry k of row r is read as the 16-bit code col16[k] = col[k] ^ r (8 bytes
// per group of four instead of 16), for states of at most 2^16 rows.  With
// PL the codes and values are the plan's padded layout: each row starts at a
// multiple of eight and is padded with zero values to whole groups (row
// pointers st.prow), so no entry needs a row mask and there is no tail, and a
// lane takes eight entries with one 16-byte code load.  With RV (operators
// whose entries are all real; always in the padded layout) the values are the
// real parts, 4 instead of 8 bytes per entry in FP32 storage, and a workgroup
// whose staged state has no imaginary part multiplies in real arithmetic (RX).  The kernel, k_spmv_lds_pf, stages
// and then runs pf_rows.

// The rows [r0, r1) of one workgroup of the pipelined LDS schedule, the state
// already staged in LDS at smem (complex, or with RX its real parts in FP64)
// and the row pointers at s_rp; writes sigma and the workgroup's energy
// partials.
template <int DT, int L, int D, bool X16, bool RV, bool RX, bool PL>
__device__ __forceinline__ void pf_rows(const SpmvState &st, int blk, const unsigned char *smem,
                                        const int32_t *s_rp, int64_t r0, int64_t r1)
{
    static_assert(!RV || PL, "real values come in the padded layout");
    using T = typename Elem<DT>::T;
    using X = typename std::conditional<RX, double, T>::type;
    // a lane's group: 4 entries, or 8 in the padded layout (one 16-byte code
    // load and 16-byte value loads)
    constexpr int GE = PL ? SPMV_PAD : 4;
    constexpr int U = 256 / (L * GE) > 0 ? 256 / (L * GE) : 1;
    constexpr int W = U * GE;                // entries per lane per pass
    constexpr int PASS = W * L;              // entries per sub-group per pass
    using V = typename ValOf<DT, RV>::T;
    constexpr unsigned EB = sizeof(V);
    const X *s_x = reinterpret_cast<const X *>(smem);
    const int tid = threadIdx.x;
    const int64_t dim = st.dim;
    constexpr int G = VQE_WAVE / L;
    const int lane = tid & 63, wid = tid >> 6;
    const int sub = lane / L, sl = lane % L;
    // the padded layout (PL) holds whole groups only, up to st.cap entries
    const int nnz = (int)(PL ? st.cap : st.nnz), zc = (int)dim;
    const int whole = PL ? 0x7fffffff : nnz & ~3;   // groups starting below this are whole
    const __amdgpu_buffer_rsrc_t rc =
        X16 ? __builtin_amdgcn_make_buffer_rsrc((void *)st.col16, (short)0, nnz * 2, VQE_BUF_WORD3)
            : __builtin_amdgcn_make_buffer_rsrc((void *)st.col, (short)0, nnz * 4, VQE_BUF_WORD3);
    const __amdgpu_buffer_rsrc_t rv =
        __builtin_amdgcn_make_buffer_rsrc((void *)(PL ? st.vre : st.val), (short)0, (int)(nnz * EB),
                                          VQE_BUF_WORD3);
    double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;

    // issue the loads of the pass starting at group kb of a row [k0, k1)
    auto issue = [&](int kb, int k1, int c[W], V v[W]) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int k = kb + u * GE * L;
            const bool ok = k < k1 && k < whole;
            if (X16 && GE == 8) {
                typedef unsigned v4u __attribute__((ext_vector_type(4)));
                const v4u c4 = __builtin_amdgcn_raw_buffer_load_b128(rc, ok ? (unsigned)k * 2u : VQE_BUF_OOB, 0, 0);
                const unsigned cw[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    c[GE * u + 2 * q] = (int)(cw[q] & 0xffffu);
                    c[GE * u + 2 * q + 1] = (int)(cw[q] >> 16);
                }
            } else if (X16) {
                typedef unsigned v2u __attribute__((ext_vector_type(2)));
                const v2u c2 = __builtin_amdgcn_raw_buffer_load_b64(rc, ok ? (unsigned)k * 2u : VQE_BUF_OOB, 0, 0);
                c[GE * u + 0] = (int)(c2.x & 0xffffu);
                c[GE * u + 1] = (int)(c2.x >> 16);
                c[GE * u + 2] = (int)(c2.y & 0xffffu);
                c[GE * u + 3] = (int)(c2.y >> 16);
            } else {
                typedef int v4i __attribute__((ext_vector_type(4)));
                const v4i c4 = __builtin_amdgcn_raw_buffer_load_b128(rc, ok ? (unsigned)k * 4u : VQE_BUF_OOB, 0, 0);
                c[GE * u + 0] = c4.x;
                c[GE * u + 1] = c4.y;
                c[GE * u + 2] = c4.z;
                c[GE * u + 3] = c4.w;
            }
#pragma unroll
            for (int h = 0; h < GE / 4; h++)
                BufVal<DT, RV>::load(rv, ok ? (unsigned)(k + 4 * h) * EB : VQE_BUF_OOB, v + GE * u + 4 * h);
        }
    };
    // products of one pass of row r; entries outside [k0, k1) read the zero
    // element
    auto consume = [&](int64_t r, int kb, int k0, int k1, const int c[W], const V v[W],
                       double &are, double &aim) {
        int cm[W];
        const unsigned len = (unsigned)(k1 - k0);
        const int rx = (int)r;
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int q = 0; q < GE; q++) {
                const int k = kb + u * GE * L + q;
                const int col = X16 ? (rx ^ c[GE * u + q]) : c[GE * u + q];
                cm[GE * u + q] = PL || (unsigned)(k - k0) < len ? col : zc;
            }
        lds_gather_fma<X, V, W>(s_x, cm, v, are, aim);
    };
    auto row_bounds = [&](int64_t r, int &k0, int &k1) {
        if (r < r1) {
            k0 = s_rp[r - r0];
            k1 = s_rp[r - r0 + 1];
        } else {
            k0 = k1 = 0;
        }
    };
    auto finish = [&](int64_t r, int k0, int k1, double are, double aim) {
        // further passes of a long row
        for (int kb = (k0 & ~(GE - 1)) + GE * sl + PASS; kb - GE * sl < k1; kb += PASS) {
            int c[W];
            V v[W];
            issue(kb, k1, c, v);
            consume(r, kb, k0, k1, c, v, are, aim);
        }
        // the entries after the last whole group of the arrays
        if (k1 > whole) {
            const int k = (k0 > whole ? k0 : whole) + sl;
            if (k < k1) {
                const V a = ldv(reinterpret_cast<const V *>(PL ? st.vre : st.val), k);
                const int col = X16 ? ((int)r ^ (int)gmem(st.col16)[k]) : gmem(st.col)[k];
                entry_fma(a, s_x[col], are, aim);
            }
        }
        are = group_sum<L>(are);
        if (!RX)
            aim = group_sum<L>(aim);
        if (sl == 0 && r < r1) {
            Elem<DT>::st(st.sigma, r, make_double2(are, aim));
            energy_terms(s_x[r], are, aim, e_re, e_im, e_n2);
        }
    };

    // D rows per sub-group in flight: each row's buffer is consumed and then
    // refilled with the sub-group's row D sweeps later
    int cb[D][W];
    V vb[D][W];
    int kb0[D], kb1[D];
    int64_t rr[D];
#pragma unroll
    for (int d = 0; d < D; d++) {
        rr[d] = r0 + (wid + 16 * d) * G + sub;
        row_bounds(rr[d], kb0[d], kb1[d]);
        issue((kb0[d] & ~(GE - 1)) + GE * sl, kb1[d], cb[d], vb[d]);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int64_t base = r0 + wid * G; base < r1; base += 16 * D * G) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            {
                double are = 0.0, aim = 0.0;
                consume(rr[d], (kb0[d] & ~(GE - 1)) + GE * sl, kb0[d], kb1[d], cb[d], vb[d], are, aim);
                finish(rr[d], kb0[d], kb1[d], are, aim);
            }
            rr[d] += 16 * D * G;
            row_bounds(rr[d], kb0[d], kb1[d]);
            issue((kb0[d] & ~(GE - 1)) + GE * sl, kb1[d], cb[d], vb[d]);
            // keep the refill ahead of the next row's products
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __shared__ double s_part[16][3];
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (tid < 3) {
        double v = 0.0;
        for (int w = 0; w < 16; w++)
            v += s_part[w][tid];
        gmem(st.partials)[(int64_t)blk * 3 + tid] = v;
    }
}

// The pipelined LDS schedule's kernel (described above pf_rows): one
// workgroup per (state, block of rows).
template <int DT, int L, int D, bool BATCH, bool X16, bool RV, bool PL>
__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_lds_pf(SpmvState single, const SpmvState *__restrict__ states,
              const int2 *__restrict__ tasks)
{
    SpmvState st;
    int blk;
    if (BATCH) {
        int2 t = tasks[blockIdx.x];
        if (t.x < 0)
            return;
        st = states[t.x];
        blk = t.y;
        if (VQE_SKIP(st))
            return;
    } else {
        st = single;
        blk = blockIdx.x;
    }
    using T = typename Elem<DT>::T;
    extern __shared__ unsigned char smem[];
    T *s_x = reinterpret_cast<T *>(smem);
    const int tid = threadIdx.x;
    const int64_t dim = st.dim;
    const T *__restrict__ psi = reinterpret_cast<const T *>(st.psi);
    const int64_t r0 = (int64_t)blk * SPMV_LDS_ROWS;
    const int64_t r1 = r0 + SPMV_LDS_ROWS < dim ? r0 + SPMV_LDS_ROWS : dim;
    int32_t *s_rp = reinterpret_cast<int32_t *>(smem + (size_t)(dim + 1) * sizeof(T));
    stage_lds<4>(s_rp, (PL ? st.prow : st.rowptr) + r0, r1 - r0 + 1, tid);
    if constexpr (RV) {
        // a real state (every imaginary part zero) runs in real arithmetic
        double *s_xr = reinterpret_cast<double *>(smem);
        const int cplx = stage_real<8>(s_xr, psi, dim, tid);
        if (tid == 0)
            s_xr[dim] = 0.0;
        if (!__syncthreads_or(cplx)) {
            pf_rows<DT, L, D, X16, RV, true, PL>(st, blk, smem, s_rp, r0, r1);
            return;
        }
    }
    stage_lds<8>(s_x, psi, dim, tid);
    if (tid == 0)
        s_x[dim] = T{};
    __syncthreads();
    pf_rows<DT, L, D, X16, RV, false, PL>(st, blk, smem, s_rp, r0, r1);
}


// ------------------------------------------------------------------ sliced layout
// VQE_SPMV_SLICED: one row per wave lane (the layout is described with
// SpmvState::scode).  Rows of a block are sorted by length so that the 64 rows
// of a slice are nearly equally long (the pads are a few percent of the
// entries at 14 qubits); a lane's loads of E entries sit next to its
// neighbours' (one contiguous run per wave and load), every lane sums its row
// in the CSR's column order with no cross-lane reduction, and the slice's
// length is uniform over the wave, so the loop has no row masks.

typedef unsigned sell_v2u __attribute__((ext_vector_type(2)));
typedef unsigned sell_v4u __attribute__((ext_vector_type(4)));
typedef int sell_v2i __attribute__((ext_vector_type(2)));

// Sort each block's rows by length, longest first (ties by row), and give
// each slice its length rounded up to E; one workgroup per block.
__global__ void __launch_bounds__(1024)
k_sell_sort(const int32_t *__restrict__ rowptr, int64_t dim, int E, uint16_t *__restrict__ srow,
            int32_t *__restrict__ slen)
{
    __shared__ uint32_t key[SPMV_LDS_ROWS];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * SPMV_LDS_ROWS;
    const int n = (int)(dim - r0 < SPMV_LDS_ROWS ? dim - r0 : SPMV_LDS_ROWS);
    for (int i = tid; i < SPMV_LDS_ROWS; i += 1024) {
        uint32_t k = 0xffffffffu;   // no row: sorts last
        if (i < n) {
            const uint32_t len = (uint32_t)(gmem(rowptr)[r0 + i + 1] - gmem(rowptr)[r0 + i]);
            k = ((0xffffu - len) << 16) | (uint32_t)i;
        }
        key[i] = k;
    }
    __syncthreads();
    // bitonic sort, ascending keys
    for (int k = 2; k <= SPMV_LDS_ROWS; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < SPMV_LDS_ROWS; i += 1024) {
                const int q = i ^ j;
                if (q > i) {
                    const uint32_t a = key[i], b = key[q];
                    if ((a > b) == ((i & k) == 0)) {
                        key[i] = b;
                        key[q] = a;
                    }
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < n; i += 1024)
        srow[r0 + i] = (uint16_t)(key[i] & 0xffffu);
    if (tid < SPMV_SLICES_PER_BLOCK) {
        int len = 0;
        if (tid * VQE_WAVE < n) {
            len = (int)(0xffffu - (key[tid * VQE_WAVE] >> 16));
            len = (len + E - 1) / E * E;
        }
        slen[(int64_t)blockIdx.x * SPMV_SLICES_PER_BLOCK + tid] = len;
    }
}

// Slice starts (entries) in slice order and the total; one wave per stream of
// slices (the entries, and with VQE_SPMV_VDICT the dictionary codes).
__global__ void __launch_bounds__(64)
k_sell_scan(const int32_t *__restrict__ slen, int64_t ns, int2 *__restrict__ sslice,
            int64_t *__restrict__ total)
{
    const int lane = threadIdx.x;
    slen += (int64_t)blockIdx.x * ns;
    sslice += (int64_t)blockIdx.x * ns;
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < ns; c0 += VQE_WAVE) {
        const int len = c0 + lane < ns ? slen[c0 + lane] : 0;
        int64_t inc = len;
#pragma unroll
        for (int o = 1; o < VQE_WAVE; o <<= 1) {
            const int64_t t = __shfl_up(inc, o, VQE_WAVE);
            if (lane >= o)
                inc += t;
        }
        if (c0 + lane < ns)
            sslice[c0 + lane] = make_int2((int)((carry + inc - len) * VQE_WAVE), len);
        carry += __shfl(inc, VQE_WAVE - 1, VQE_WAVE);
    }
    if (lane == 0)
        total[blockIdx.x] = carry * VQE_WAVE;
}

// Codes and values of one slice per wave (pads: column dim, value zero); RV:
// the values' real parts (an operator whose entries are all real).
template <int DT, bool RV>
__global__ void __launch_bounds__(64)
k_sell_fill(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
            const void *__restrict__ val, int64_t dim, int E, const uint16_t *__restrict__ srow,
            const int2 *__restrict__ sslice, uint16_t *__restrict__ code, void *__restrict__ sval)
{
    using T = typename Elem<DT>::T;
    using V = typename ValOf<DT, RV>::T;
    const int64_t c = blockIdx.x;
    const int64_t r0 = (c / SPMV_SLICES_PER_BLOCK) * SPMV_LDS_ROWS;
    const int n = (int)(dim - r0 < SPMV_LDS_ROWS ? dim - r0 : SPMV_LDS_ROWS);
    const int lane = threadIdx.x;
    const int i = (int)(c % SPMV_SLICES_PER_BLOCK) * VQE_WAVE + lane;
    const int2 sl = sslice[c];
    int64_t k0 = 0;
    int len = 0;
    if (i < n) {
        const int64_t row = r0 + srow[r0 + i];
        k0 = rowptr[row];
        len = rowptr[row + 1] - (int32_t)k0;
    }
    V *out = reinterpret_cast<V *>(sval);
    const T *in = reinterpret_cast<const T *>(val);
    for (int j = 0; j < sl.y; j++) {
        const int64_t at = (int64_t)sl.x + ((int64_t)(j / E) * VQE_WAVE + lane) * E + j % E;
        code[at] = j < len ? (uint16_t)col[k0 + j] : (uint16_t)dim;
        if constexpr (RV)
            out[at] = j < len ? in[k0 + j].x : V{};
        else
            out[at] = j < len ? in[k0 + j] : V{};
    }
}

// Flip-mask index form (VQE_SPMV_XIDX): the masks x = col ^ row an operator
// uses (Eq. 3: every Pauli string maps r to r ^ x), numbered in ascending
// order, and the slices' entries stored as those numbers.
__global__ void __launch_bounds__(256)
k_sell_fill32(uint32_t *__restrict__ p, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        p[i] = v;
}

// Rows of a workgroup of the kernels that read the whole CSR (a wave per row,
// 16 waves).  A row is a chain of dependent reads (bounds, columns, mask
// numbers), so waves in flight set their time: a 14-qubit H is 256 workgroups,
// and with four waves each the marks took 34 us, the magnitudes 70 and the
// rows' counts 26; with sixteen 12, 23 and 10.
#define SELL_SCAN_ROWS 64

// The masks the operator uses, a bit each in mark [dim / 32 words, at least
// one] (col and row are below dim = 2^N <= 2^16, so is their XOR); a
// workgroup's rows gather in LDS first.
__global__ void __launch_bounds__(1024)
k_sell_xmark(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int64_t dim,
             uint32_t *__restrict__ mark)
{
    __shared__ uint32_t s_mark[SPMV_X16_MAX_DIM / 32];
    const int tid = threadIdx.x, lane = tid & 63, words = (int)((dim + 31) / 32);
    for (int i = tid; i < words; i += 1024)
        s_mark[i] = 0u;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * SELL_SCAN_ROWS;
    for (int64_t r = r0 + (tid >> 6); r < r0 + SELL_SCAN_ROWS && r < dim; r += 16)
        for (int k = rowptr[r] + lane; k < rowptr[r + 1]; k += VQE_WAVE) {
            const uint32_t x = (uint32_t)col[k] ^ (uint32_t)r;
            if (!(s_mark[x >> 5] >> (x & 31u) & 1u))
                atomicOr(&s_mark[x >> 5], 1u << (x & 31u));
        }
    __syncthreads();
    for (int i = tid; i < words; i += 1024)
        if (s_mark[i])
            atomicOr(&mark[i], s_mark[i]);
}

// The masks' numbers xmap[x] (ascending x), the table xtab[number] = x for
// the first SPMV_XIDX_MAX numbers and the count; one workgroup (dim <= 2^16:
// at most two words of mark per thread).
__global__ void __launch_bounds__(1024)
k_sell_xscan(const uint32_t *__restrict__ mark, int64_t dim, uint16_t *__restrict__ xmap,
             uint16_t *__restrict__ xtab, int64_t *__restrict__ nx)
{
    __shared__ int part[1024];
    const int tid = threadIdx.x, words = (int)((dim + 31) / 32);
    const uint32_t w0 = 2 * tid < words ? mark[2 * tid] : 0u;
    const uint32_t w1 = 2 * tid + 1 < words ? mark[2 * tid + 1] : 0u;
    const int c = __popc(w0) + __popc(w1);
    part[tid] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int at = part[tid] - c;
#pragma unroll
    for (int h = 0; h < 2; h++)
        for (uint32_t w = h ? w1 : w0; w; w &= w - 1) {
            const uint32_t x = (uint32_t)(2 * tid + h) * 32u + (uint32_t)__builtin_ctz(w);
            xmap[x] = (uint16_t)at;
            if (at < SPMV_XIDX_MAX)
                xtab[at] = (uint16_t)x;
            at++;
        }
    if (tid == 1023)
        *nx = part[1023];
}

// ---- value dictionary (VQE_SPMV_VDICT): a flip mask whose entries take at
// most SPMV_VD_VALS magnitudes, all real (in a molecular Hamiltonian every
// two-electron mask: its entries are +- one integral, or one of three sums),
// has its entries stored as a code, the number of the (mask, magnitude) pair
// and the sign, beside a per-operator table of the pairs.  At 14 qubits 511 of
// 554 masks and 136.5 of 158.5 entries per row, in 651 pairs.
//
// What it is for: the sliced product streamed 9.3 bytes per entry at the rate
// HBM gives (64 states of 14 qubits: 1.6 GB, 275 us).  Twelve-bit codes for
// those entries and real parts for the others of a real H leave 0.4 GB; the
// product is then bound by the vector ALU (about ten operations an entry) and
// the LDS gathers about as much as by HBM: 96 us.  Sixteen-bit codes with the
// sign beside them took 113 us, twelve bits with an unsigned table 109 us.
#define SPMV_VD_EMPTY 0xffffffffu

// Collect each mask's magnitudes (bits of |re|): slots [SPMV_XIDX_MAX *
// SPMV_VD_VALS], all SPMV_VD_EMPTY before, and bad [SPMV_XIDX_MAX], zero
// before, set for a mask with more or with an imaginary part.  The set found
// does not depend on the order of the insertions.
__device__ __forceinline__ void vd_insert(uint32_t *slots, uint32_t *bad, int i, uint32_t v)
{
    for (int q = 0; q < SPMV_VD_VALS; q++) {
        uint32_t cur = __hip_atomic_load(&slots[i * SPMV_VD_VALS + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == SPMV_VD_EMPTY)
            cur = atomicCAS(&slots[i * SPMV_VD_VALS + q], SPMV_VD_EMPTY, v);
        if (cur == SPMV_VD_EMPTY || cur == v)
            return;
    }
    bad[i] = 1u;
}

__global__ void __launch_bounds__(1024)
k_vd_collect(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
             const float2 *__restrict__ val, int64_t dim, const uint16_t *__restrict__ xmap,
             uint32_t *__restrict__ slots, uint32_t *__restrict__ bad)
{
    __shared__ uint32_t s_slots[SPMV_XIDX_MAX * SPMV_VD_VALS];
    __shared__ uint32_t s_bad[SPMV_XIDX_MAX];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < SPMV_XIDX_MAX * SPMV_VD_VALS; i += 1024)
        s_slots[i] = SPMV_VD_EMPTY;
    for (int i = tid; i < SPMV_XIDX_MAX; i += 1024)
        s_bad[i] = 0u;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * SELL_SCAN_ROWS;
    for (int64_t r = r0 + (tid >> 6); r < r0 + SELL_SCAN_ROWS && r < dim; r += 16)
        for (int k = rowptr[r] + lane; k < rowptr[r + 1]; k += VQE_WAVE) {
            const int i = xmap[(uint32_t)col[k] ^ (uint32_t)r];
            const float2 v = val[k];
            if (i >= SPMV_XIDX_MAX || s_bad[i])     // (too many masks: refused later)
                continue;
            if (v.y != 0.f)
                s_bad[i] = 1u;
            else
                vd_insert(s_slots, s_bad, i, __float_as_uint(v.x) & 0x7fffffffu);
        }
    __syncthreads();
    for (int i = tid; i < SPMV_XIDX_MAX; i += 1024) {
        if (s_bad[i]) {
            bad[i] = 1u;
            continue;
        }
        for (int q = 0; q < SPMV_VD_VALS; q++)
            if (s_slots[i * SPMV_VD_VALS + q] != SPMV_VD_EMPTY)
                vd_insert(slots, bad, i, s_slots[i * SPMV_VD_VALS + q]);
    }
}

// Number the pairs, masks ascending and each one's magnitudes ascending:
// pair [SPMV_VD_PAIRS] = (magnitude, byte offset of the mask in a staged
// state), zero past the last (the pads' pair SPMV_VD_PAIRS - 1 among them),
// and base [SPMV_XIDX_MAX] the first pair of each mask, or SPMV_VD_NONE for a
// mask that keeps its entries as they are.
#define SPMV_VD_NONE 0xffffu
__global__ void __launch_bounds__(1024)
k_vd_number(const uint32_t *__restrict__ slots, const uint32_t *__restrict__ bad,
            const uint16_t *__restrict__ xtab, const int64_t *__restrict__ nx,
            uint2 *__restrict__ pair, uint16_t *__restrict__ base)
{
    static_assert(SPMV_XIDX_MAX == 1024 && SPMV_VD_PAIRS == 1024 && SPMV_VD_VALS == 4, "one thread each");
    __shared__ int part[1024];
    const int tid = threadIdx.x;
    uint32_t v[4] = {SPMV_VD_EMPTY, SPMV_VD_EMPTY, SPMV_VD_EMPTY, SPMV_VD_EMPTY};
    int c = 0;
    if (tid < *nx && !bad[tid]) {
#pragma unroll
        for (int q = 0; q < 4; q++)
            v[q] = slots[tid * 4 + q];
        // ascending (the empty ones last)
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int q = 0; q < 3 - a; q++)
                if (v[q] > v[q + 1]) {
                    const uint32_t t = v[q];
                    v[q] = v[q + 1];
                    v[q + 1] = t;
                }
#pragma unroll
        for (int q = 0; q < 4; q++)
            c += v[q] != SPMV_VD_EMPTY;
    }
    part[tid] = c;
    pair[tid] = make_uint2(0u, 0u);
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int t = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += t;
        __syncthreads();
    }
    const int at = part[tid] - c;
    const bool in = c > 0 && at + c <= SPMV_VD_PAIRS - 1;
    base[tid] = in ? (uint16_t)at : (uint16_t)SPMV_VD_NONE;
    if (in)
#pragma unroll
        for (int q = 0; q < 4; q++)
            if (q < c)
                pair[at + q] = make_uint2(v[q], (uint32_t)xtab[tid] * (uint32_t)sizeof(float2));
}

// Entries of each row in the dictionary (low half) and beside it (high half).
template <int MASKS>
__global__ void __launch_bounds__(1024)
k_vd_rows(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int64_t dim,
          const uint16_t *__restrict__ xmap, const uint16_t *__restrict__ base,
          uint32_t *__restrict__ len)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t r0 = (int64_t)blockIdx.x * SELL_SCAN_ROWS;
    for (int64_t r = r0 + (tid >> 6); r < r0 + SELL_SCAN_ROWS && r < dim; r += 16) {
        const int k0 = rowptr[r], k1 = rowptr[r + 1];
        int n = 0;
        for (int k = k0; k < k1; k += VQE_WAVE) {
            bool d = false;
            if (k + lane < k1) {
                const int i = xmap[(uint32_t)col[k + lane] ^ (uint32_t)r];
                d = i < MASKS && base[i] != SPMV_VD_NONE;
            }
            n += __popcll(__ballot(d));
        }
        if (lane == 0)
            len[r] = (uint32_t)n | (uint32_t)(k1 - k0 - n) << 16;
    }
}

// k_sell_sort for the two streams: rows by dictionary entries, then by the
// others (longest first, ties by row); slice lengths of the others, rounded up
// to E, then [at slen + slices] of the codes, rounded up to SPMV_VD_GROUP.
__global__ void __launch_bounds__(1024)
k_vd_sort(const uint32_t *__restrict__ len, int64_t dim, int E, uint16_t *__restrict__ srow,
          int32_t *__restrict__ slen, int64_t ns)
{
    __shared__ uint64_t key[SPMV_LDS_ROWS];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * SPMV_LDS_ROWS;
    const int n = (int)(dim - r0 < SPMV_LDS_ROWS ? dim - r0 : SPMV_LDS_ROWS);
    for (int i = tid; i < SPMV_LDS_ROWS; i += 1024) {
        uint64_t k = ~0ull;   // no row: sorts last
        if (i < n) {
            const uint32_t l = len[r0 + i];
            k = (uint64_t)(0xffffu - (l & 0xffffu)) << 32 | (uint64_t)(0xffffu - (l >> 16)) << 16 | (uint32_t)i;
        }
        key[i] = k;
    }
    __syncthreads();
    for (int k = 2; k <= SPMV_LDS_ROWS; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            // the lower row of each compared pair, one pair per thread
            const int i = ((tid & ~(j - 1)) << 1) | (tid & (j - 1)), q = i | j;
            const uint64_t a = key[i], b = key[q];
            if ((a > b) == ((i & k) == 0)) {
                key[i] = b;
                key[q] = a;
            }
            __syncthreads();
        }
    for (int i = tid; i < n; i += 1024)
        srow[r0 + i] = (uint16_t)(key[i] & 0xffffu);
    const int lane = tid & 63;
    for (int c = tid >> 6; c < SPMV_SLICES_PER_BLOCK; c += 16) {
        const int i = c * VQE_WAVE + lane;
        int d = 0, e = 0;
        if (i < n) {
            d = (int)(0xffffu - (uint32_t)(key[i] >> 32));
            e = (int)(0xffffu - (uint32_t)(key[i] >> 16 & 0xffffu));
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            d = max(d, __shfl_xor(d, o, VQE_WAVE));
            e = max(e, __shfl_xor(e, o, VQE_WAVE));
        }
        if (lane == 0) {
            const int64_t at = (int64_t)blockIdx.x * SPMV_SLICES_PER_BLOCK + c;
            slen[at] = (e + E - 1) / E * E;
            slen[ns + at] = (d + SPMV_VD_GROUP - 1) / SPMV_VD_GROUP * SPMV_VD_GROUP;
        }
    }
}

// A word of codes: one in bits 3 to 14 (in place for a byte offset into a
// table of 8-byte elements), one in bits 15 to 26, eight bits of a third in
// bits 27 to 31 and 0 to 2.
__device__ __forceinline__ uint32_t vd_word(uint32_t a, uint32_t b, uint32_t e)
{
    return a << 3 | b << 15 | e << 27 | e >> 5;
}
// The wave's accesses to LDS before this come before those after it.  A wave's
// LDS operations complete in order, so it only binds the compiler, which may
// otherwise take a lane's own last write for what another lane has overwritten.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ uint32_t vd_byte(uint32_t w) { return __builtin_amdgcn_alignbit(w, w, 27) & 0xffu; }

// Both streams of one slice per workgroup, a row per wave in turn.  A row's
// codes go in ascending pair order (neighbouring lanes then read neighbouring
// pairs), its other entries in column order.
template <bool RV, int E>
__global__ void __launch_bounds__(1024)
k_vd_fill(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
          const float2 *__restrict__ val, int64_t dim, const uint16_t *__restrict__ srow,
          const int2 *__restrict__ sslice, int64_t ns, const uint16_t *__restrict__ xmap,
          const uint16_t *__restrict__ base, const uint2 *__restrict__ pair,
          uint32_t *__restrict__ code, typename ValOf<VQE_C64, RV>::T *__restrict__ out,
          uint32_t *__restrict__ dcode)
{
    using V = typename ValOf<VQE_C64, RV>::T;
    // a row's codes, then its other entries' mask numbers (a row has one entry
    // per mask, so both fit)
    __shared__ uint32_t s_bits[16][SPMV_VD_PAIRS / 32];
    __shared__ uint16_t s_pre[16][SPMV_VD_PAIRS / 32];
    __shared__ uint16_t s_row[16][SPMV_XIDX_MAX];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t *bits = s_bits[wid];
    uint16_t *pre = s_pre[wid], *buf = s_row[wid];
    const int64_t c = blockIdx.x;
    const int64_t r0 = (c / SPMV_SLICES_PER_BLOCK) * SPMV_LDS_ROWS;
    const int n = (int)(dim - r0 < SPMV_LDS_ROWS ? dim - r0 : SPMV_LDS_ROWS);
    const int2 se = sslice[c], sd = sslice[ns + c];
    for (int lr = wid; lr < VQE_WAVE; lr += 16) {
        const int i = (int)(c % SPMV_SLICES_PER_BLOCK) * VQE_WAVE + lr;
        int64_t row = 0;
        int k0 = 0, k1 = 0;
        if (i < n) {
            row = r0 + srow[r0 + i];
            k0 = rowptr[row];
            k1 = rowptr[row + 1];
        }
        auto pair_of = [&](int k, int &m) -> int {     // the entry's pair, or -1; its mask's number
            m = xmap[(uint32_t)col[k] ^ (uint32_t)row];
            const uint32_t b = base[m];
            if (b == SPMV_VD_NONE)
                return -1;
            const uint32_t v = __float_as_uint(val[k].x) & 0x7fffffffu;
            int p = (int)b;
            for (int q = 0; q < SPMV_VD_VALS - 1 && pair[p].x != v; q++)
                p++;
            return p;
        };
        if (lane < SPMV_VD_PAIRS / 32)
            bits[lane] = 0u;
        wave_lds_order();
        for (int k = k0 + lane; k < k1; k += VQE_WAVE) {
            int m;
            const int p = pair_of(k, m);
            if (p >= 0)
                atomicOr(&bits[p >> 5], 1u << (p & 31));
        }
        wave_lds_order();
        int inc = lane < SPMV_VD_PAIRS / 32 ? __popc(bits[lane]) : 0;
        const int own = inc;
#pragma unroll
        for (int o = 1; o < VQE_WAVE; o <<= 1) {
            const int t = __shfl_up(inc, o, VQE_WAVE);
            if (lane >= o)
                inc += t;
        }
        if (lane < SPMV_VD_PAIRS / 32)
            pre[lane] = (uint16_t)(inc - own);
        wave_lds_order();
        const int nd = __shfl(inc, VQE_WAVE - 1, VQE_WAVE);
        auto eat = [&](int j) { return (int64_t)se.x + ((int64_t)(j / E) * VQE_WAVE + lr) * E + j % E; };
        int ne = 0;
        for (int kb = k0; kb < k1; kb += VQE_WAVE) {
            const int k = kb + lane;
            int m = 0, p = -1;
            const bool on = k < k1;
            if (on)
                p = pair_of(k, m);
            const uint64_t eb = __ballot(on && p < 0);
            if (on && p >= 0) {
                const int j = pre[p >> 5] + __popc(bits[p >> 5] & ((1u << (p & 31)) - 1u));
                buf[j] = (uint16_t)((uint32_t)p << 1 | __float_as_uint(val[k].x) >> 31);
            } else if (on) {
                const int j = ne + __popcll(eb & ((1ull << lane) - 1ull));
                buf[nd + j] = (uint16_t)m;
                if constexpr (RV)
                    out[eat(j)] = val[k].x;
                else
                    out[eat(j)] = val[k];
            }
            ne += __popcll(eb);
        }
        wave_lds_order();
        auto code_at = [&](int j) { return j < nd ? (uint32_t)buf[j] : 2u * (SPMV_VD_PAIRS - 1); };
        for (int w = lane; w < sd.y / SPMV_VD_GROUP * 4; w += VQE_WAVE) {
            const int g = w >> 2, q = w & 3, j = g * SPMV_VD_GROUP;
            const uint32_t x = code_at(j + 8 + (q >> 1));
            dcode[(int64_t)sd.x / SPMV_VD_GROUP * 4 + ((int64_t)g * VQE_WAVE + lr) * 4 + q] =
                vd_word(code_at(j + 2 * q), code_at(j + 2 * q + 1), q & 1 ? x >> 8 : x & 0xffu);
        }
        for (int j = ne + lane; j < se.y; j += VQE_WAVE)
            out[eat(j)] = V{};
        auto idx_at = [&](int j) { return j < ne ? (uint32_t)buf[nd + j] : 0u; };
        for (int w = lane; w < se.y / 3; w += VQE_WAVE)
            code[eat(3 * w) / 3] = idx_at(3 * w) | idx_at(3 * w + 1) << 10 | idx_at(3 * w + 2) << 20;
        wave_lds_order();      // the next row takes the buffers
    }
}

// Indices and values of one slice per wave (E = 3 or 6 entries per group,
// E / 3 words; pads: index 0, value zero); RV: the values' real parts.
template <int DT, bool RV, int E>
__global__ void __launch_bounds__(64)
k_sell_fill_x(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
              const void *__restrict__ val, int64_t dim, const uint16_t *__restrict__ srow,
              const int2 *__restrict__ sslice, const uint16_t *__restrict__ xmap,
              uint32_t *__restrict__ code, void *__restrict__ sval)
{
    using T = typename Elem<DT>::T;
    using V = typename ValOf<DT, RV>::T;
    static_assert(E == 3 || E == 6, "three indices to a word");
    const int64_t c = blockIdx.x;
    const int64_t r0 = (c / SPMV_SLICES_PER_BLOCK) * SPMV_LDS_ROWS;
    const int n = (int)(dim - r0 < SPMV_LDS_ROWS ? dim - r0 : SPMV_LDS_ROWS);
    const int lane = threadIdx.x;
    const int i = (int)(c % SPMV_SLICES_PER_BLOCK) * VQE_WAVE + lane;
    const int2 sl = sslice[c];
    int64_t k0 = 0, row = 0;
    int len = 0;
    if (i < n) {
        row = r0 + srow[r0 + i];
        k0 = rowptr[row];
        len = rowptr[row + 1] - (int32_t)k0;
    }
    V *out = reinterpret_cast<V *>(sval);
    const T *in = reinterpret_cast<const T *>(val);
    for (int g = 0; g < sl.y / E; g++) {
        // the group's first entry: a multiple of E, so its words start at a
        // multiple of E / 3
        const int64_t at = (int64_t)sl.x + ((int64_t)g * VQE_WAVE + lane) * E;
        uint32_t w[E / 3] = {};
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int j = g * E + e;
            const uint32_t idx = j < len ? xmap[(uint32_t)col[k0 + j] ^ (uint32_t)row] : 0u;
            w[e / 3] |= idx << (10 * (e % 3));
            if constexpr (RV)
                out[at + e] = j < len ? in[k0 + j].x : V{};
            else
                out[at + e] = j < len ? in[k0 + j] : V{};
        }
#pragma unroll
        for (int q = 0; q < E / 3; q++)
            code[at / 3 + q] = w[q];
    }
}

// One entry's product added to the row's sums in turn (each product with its
// own FMA): complex value and state; real value, complex state; real value,
// real state (FP64 real parts).
template <typename V, typename X>
__device__ __forceinline__ void sell_fma(const V a, const X x, double &are, double &aim)
{
    const double ar = (double)a.x, ai = (double)a.y, xr = (double)x.x, xi = (double)x.y;
    are = fma(ar, xr, are);
    are = fma(-ai, xi, are);
    aim = fma(ar, xi, aim);
    aim = fma(ai, xr, aim);
}
template <typename X>
__device__ __forceinline__ void sell_fma(const float a, const X x, double &are, double &aim)
{
    are = fma((double)a, (double)x.x, are);
    aim = fma((double)a, (double)x.y, aim);
}
template <typename X>
__device__ __forceinline__ void sell_fma(const double a, const X x, double &are, double &aim)
{
    are = fma(a, (double)x.x, are);
    aim = fma(a, (double)x.y, aim);
}
__device__ __forceinline__ void sell_fma(const float a, const double x, double &are, double &aim)
{
    (void)aim;
    are = fma((double)a, x, are);
}
__device__ __forceinline__ void sell_fma(const double a, const double x, double &are, double &aim)
{
    (void)aim;
    are = fma(a, x, are);
}

// E consecutive entries of one lane: their codes (two per word) and values
// (complex, or their real parts with RV).
template <int DT, int E, bool RV = false>
struct SellGroup {
    using T = typename Elem<DT>::T;
    using V = typename ValOf<DT, RV>::T;
    using C = uint16_t;     // the layout's code unit
    unsigned c[E / 2];
    V v[E];
    __device__ __forceinline__ void load(const uint16_t *__restrict__ code,
                                         const V *__restrict__ val, int64_t at)
    {
        if constexpr (E == 2) {
            c[0] = gmem(reinterpret_cast<const unsigned *>(code + at))[0];
        } else if constexpr (E == 4) {
            const sell_v2u w = gmem(reinterpret_cast<const sell_v2u *>(code + at))[0];
            c[0] = w.x;
            c[1] = w.y;
        } else {
            const sell_v4u w = gmem(reinterpret_cast<const sell_v4u *>(code + at))[0];
            c[0] = w.x;
            c[1] = w.y;
            c[2] = w.z;
            c[3] = w.w;
        }
        if constexpr (RV && DT == VQE_C64 && E == 2) {
            const vqe_v2f a = gmem(reinterpret_cast<const vqe_v2f *>(val + at))[0];
            v[0] = a.x;
            v[1] = a.y;
        } else if constexpr (RV && DT == VQE_C64) {
#pragma unroll
            for (int q = 0; q < E / 4; q++) {
                const vqe_v4f a = gmem(reinterpret_cast<const vqe_v4f *>(val + at))[q];
                v[4 * q] = a.x;
                v[4 * q + 1] = a.y;
                v[4 * q + 2] = a.z;
                v[4 * q + 3] = a.w;
            }
        } else if constexpr (RV) {
#pragma unroll
            for (int q = 0; q < E / 2; q++) {
                const vqe_v2d a = gmem(reinterpret_cast<const vqe_v2d *>(val + at))[q];
                v[2 * q] = a.x;
                v[2 * q + 1] = a.y;
            }
        } else if constexpr (DT == VQE_C64) {
#pragma unroll
            for (int q = 0; q < E / 2; q++) {
                const vqe_v4f a = gmem(reinterpret_cast<const vqe_v4f *>(val + at))[q];
                v[2 * q] = make_float2(a.x, a.y);
                v[2 * q + 1] = make_float2(a.z, a.w);
            }
        } else {
#pragma unroll
            for (int q = 0; q < E; q++)
                v[q] = ldg(val, at + q);
        }
    }
    // each product added to the row's sums in turn; X: the staged state's
    // element (complex, or the real parts in FP64)
    template <typename X>
    __device__ __forceinline__ void use(const X *s_x, double &are, double &aim) const
    {
#pragma unroll
        for (int q = 0; q < E; q++)
            sell_fma(v[q], s_x[(q & 1) ? c[q / 2] >> 16 : c[q / 2] & 0xffffu], are, aim);
    }
};

// The same for the flip-mask index form: E = 3 or 6 entries per lane, their
// indices in E / 3 32-bit words (three 10-bit fields each); an entry's column
// is the lane's row XOR the indexed mask.
template <int DT, bool RV, int E>
struct SellGroupX {
    using V = typename ValOf<DT, RV>::T;
    using C = uint32_t;
    static_assert(E == 3 || E == 6, "three indices to a word");
    unsigned c[E / 3];
    V v[E];
    // at: the group's first entry (a multiple of E: with E = 6 the words are
    // 8-byte and the values 16-byte aligned, 8-byte for FP32 real parts; with
    // E = 3 the values are aligned to their own size)
    __device__ __forceinline__ void load(const uint32_t *__restrict__ code, const V *__restrict__ val,
                                         int64_t at)
    {
        if constexpr (E == 3) {
            c[0] = gmem(code)[at / 3];
#pragma unroll
            for (int q = 0; q < E; q++) {
                if constexpr (RV)
                    v[q] = gmem(val)[at + q];
                else
                    v[q] = ldg(val, at + q);
            }
            return;
        }
        const sell_v2u w = gmem(reinterpret_cast<const sell_v2u *>(code + at / 3))[0];
        c[0] = w.x;
        c[1] = w.y;
        if constexpr (RV && DT == VQE_C64) {
#pragma unroll
            for (int q = 0; q < E / 2; q++) {
                const vqe_v2f a = gmem(reinterpret_cast<const vqe_v2f *>(val + at))[q];
                v[2 * q] = a.x;
                v[2 * q + 1] = a.y;
            }
        } else if constexpr (RV) {
#pragma unroll
            for (int q = 0; q < E / 2; q++) {
                const vqe_v2d a = gmem(reinterpret_cast<const vqe_v2d *>(val + at))[q];
                v[2 * q] = a.x;
                v[2 * q + 1] = a.y;
            }
        } else if constexpr (DT == VQE_C64) {
#pragma unroll
            for (int q = 0; q < E / 2; q++) {
                const vqe_v4f a = gmem(reinterpret_cast<const vqe_v4f *>(val + at))[q];
                v[2 * q] = make_float2(a.x, a.y);
                v[2 * q + 1] = make_float2(a.z, a.w);
            }
        } else {
#pragma unroll
            for (int q = 0; q < E; q++)
                v[q] = ldg(val, at + q);
        }
    }
    // each product added to the row's sums in turn; s_xt: the masks staged in
    // LDS, row: the lane's row
    template <typename X>
    __device__ __forceinline__ void use(const X *s_x, const uint16_t *s_xt, uint32_t row, double &are,
                                        double &aim) const
    {
#pragma unroll
        for (int q = 0; q < E; q++)
            sell_fma(v[q], s_x[row ^ (uint32_t)s_xt[(c[q / 3] >> (10 * (q % 3))) & 1023u]], are, aim);
    }
};

// One wave's share of a block of the sliced layout: its slices A and B (those
// the block has; a whole block: wid and wid + 16), taken as one stream of groups (A's,
// then B's) so that B's first groups load while A finishes; D groups of E
// entries per lane in flight.  Every load is issued (past the stream's end
// it repeats the last group, which is in cache), so no load sits under a
// branch and each group's wait leaves the later groups' loads in flight.
template <int DT, int E, int D, bool RV, bool XI = false>
struct SellWave {
    using V = typename ValOf<DT, RV>::T;
    using G = typename std::conditional<XI, SellGroupX<DT, RV, E>, SellGroup<DT, E, RV>>::type;
    static constexpr int64_t STEP = (int64_t)VQE_WAVE * E;
    const typename G::C *code;
    const V *val;
    int64_t r0, ata, atb;
    int n, ns, nga, ngb, ng, ra, rb;   // ra, rb: block-local rows of this lane
    int ka, kb;                        // the slices (none: past the block's)
    G g[D];

    __device__ __forceinline__ void init(const SpmvState &st, int blk, int lane, int a_slice, int b_slice)
    {
        ka = a_slice;
        kb = b_slice;
        code = reinterpret_cast<const typename G::C *>(st.scode);
        val = reinterpret_cast<const V *>(st.sval);
        r0 = (int64_t)blk * SPMV_LDS_ROWS;
        n = (int)(st.dim - r0 < SPMV_LDS_ROWS ? st.dim - r0 : SPMV_LDS_ROWS);
        ns = (n + VQE_WAVE - 1) / VQE_WAVE;
        const sell_v2i *sls = reinterpret_cast<const sell_v2i *>(st.sslice) + (int64_t)blk * SPMV_SLICES_PER_BLOCK;
        sell_v2i a = {0, 0}, b = {0, 0};
        if (ka < ns)
            a = gmem(sls)[ka];
        if (kb < ns)
            b = gmem(sls)[kb];
        nga = __builtin_amdgcn_readfirstlane(a.y) / E;
        ngb = __builtin_amdgcn_readfirstlane(b.y) / E;
        ng = nga + ngb;
        ata = (int64_t)__builtin_amdgcn_readfirstlane(a.x) + lane * E;
        atb = (int64_t)__builtin_amdgcn_readfirstlane(b.x) + lane * E - (int64_t)nga * STEP;
        const int ia = ka * VQE_WAVE + lane, ib = kb * VQE_WAVE + lane;
        ra = gmem(st.srow)[r0 + (ia < n ? ia : n - 1)];
        rb = gmem(st.srow)[r0 + (ib < n ? ib : n - 1)];
    }
    // stream group p (clamped to the last) and its first entry for this lane
    __device__ __forceinline__ int64_t addr(int p) const
    {
        const int pc = p < ng ? p : ng - 1;
        return (pc < nga ? ata : atb) + (int64_t)pc * STEP;
    }
    // the stream's first groups (a wave with groups only)
    __device__ __forceinline__ void prefetch()
    {
#pragma unroll
        for (int d = 0; d < D; d++)
            g[d].load(code, val, addr(d));
    }
    // the rows' sums for A and B against the staged state s_x (X: complex, or
    // the real parts in FP64 for a real state; s_xt: the staged flip masks of
    // the index form); prefetch() came first
    template <typename X>
    __device__ __forceinline__ void run(const X *s_x, const uint16_t *s_xt, double2 &sa, double2 &sb)
    {
        double are = 0.0, aim = 0.0;
        sa = make_double2(0.0, 0.0);
        sb = make_double2(0.0, 0.0);
        if (ng == 0)
            return;
        uint32_t row = (uint32_t)(r0 + ra);
        auto use = [&](const G &gr) {
            if constexpr (XI)
                gr.use(s_x, s_xt, row, are, aim);
            else
                gr.use(s_x, are, aim);
        };
        int q = 0;
        for (; q + D <= ng; q += D) {
#pragma unroll
            for (int d = 0; d < D; d++) {
                if (q + d == nga) {     // B's first group: A's sums are done
                    sa = make_double2(are, aim);
                    are = aim = 0.0;
                    row = (uint32_t)(r0 + rb);
                }
                use(g[d]);
                g[d].load(code, val, addr(q + D + d));
                // keep the refill ahead of the next group's products
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < D; d++)
            if (q + d < ng) {
                if (q + d == nga) {
                    sa = make_double2(are, aim);
                    are = aim = 0.0;
                    row = (uint32_t)(r0 + rb);
                }
                use(g[d]);
            }
        if (ngb == 0)
            sa = make_double2(are, aim);
        else
            sb = make_double2(are, aim);
    }
};

// One wave's share of a block's dictionary codes: its slices A and B as one stream of groups of SPMV_VD_GROUP codes (16 bytes per
// lane), D groups in flight, as SellWave.  An entry is one read of its signed
// pair, one of the state at row ^ mask and two FMAs (one for a real state).
template <int D> struct DictWave {
    const sell_v4u *code;
    int64_t ata, atb;
    int nga, ngb, ng;
    sell_v4u g[D];

    __device__ __forceinline__ void init(const SpmvState &st, int blk, int lane, int ka, int kb, int ns)
    {
        code = reinterpret_cast<const sell_v4u *>(st.dcode);
        const sell_v2i *sls = reinterpret_cast<const sell_v2i *>(st.dslice) + (int64_t)blk * SPMV_SLICES_PER_BLOCK;
        sell_v2i a = {0, 0}, b = {0, 0};
        if (ka < ns)
            a = gmem(sls)[ka];
        if (kb < ns)
            b = gmem(sls)[kb];
        nga = __builtin_amdgcn_readfirstlane(a.y) / SPMV_VD_GROUP;
        ngb = __builtin_amdgcn_readfirstlane(b.y) / SPMV_VD_GROUP;
        ng = nga + ngb;
        ata = __builtin_amdgcn_readfirstlane(a.x) / SPMV_VD_GROUP + lane;
        atb = __builtin_amdgcn_readfirstlane(b.x) / SPMV_VD_GROUP + lane - (int64_t)nga * VQE_WAVE;
    }
    __device__ __forceinline__ sell_v4u load(int p) const
    {
        const int pc = p < ng ? p : ng - 1;
        return gmem(code)[(pc < nga ? ata : atb) + (int64_t)pc * VQE_WAVE];
    }
    __device__ __forceinline__ void prefetch()
    {
#pragma unroll
        for (int d = 0; d < D; d++)
            g[d] = load(d);
    }
    template <typename X>
    static __device__ __forceinline__ void use(const sell_v4u c, const unsigned char *s_x,
                                               const unsigned char *s_pair, uint32_t row8, double &are, double &aim)
    {
        // byte offsets of the ten signed pairs (vd_word)
        uint32_t at[SPMV_VD_GROUP];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            at[2 * q] = c[q] & 0x7ff8u;
            at[2 * q + 1] = c[q] >> 12 & 0x7ff8u;
        }
#pragma unroll
        for (int q = 0; q < 2; q++)
            at[8 + q] = (vd_byte(c[2 * q]) | vd_byte(c[2 * q + 1]) << 8) << 3;
        uint2 pr[SPMV_VD_GROUP];
#pragma unroll
        for (int q = 0; q < SPMV_VD_GROUP; q++)
            pr[q] = *reinterpret_cast<const uint2 *>(s_pair + at[q]);
        X x[SPMV_VD_GROUP];
#pragma unroll
        for (int q = 0; q < SPMV_VD_GROUP; q++)
            x[q] = *reinterpret_cast<const X *>(s_x + (row8 ^ pr[q].y));
#pragma unroll
        for (int q = 0; q < SPMV_VD_GROUP; q++)
            sell_fma(__uint_as_float(pr[q].x), x[q], are, aim);
    }
    // the sums of rows ra (A) and rb (B) over their codes; X: 8-byte elements
    template <typename X>
    __device__ __forceinline__ void run(const X *s_xe, const uint2 *s_pairs, int64_t ra, int64_t rb,
                                        double2 &sa, double2 &sb)
    {
        static_assert(sizeof(X) == 8, "the pairs hold byte offsets of 8-byte elements");
        const unsigned char *s_x = reinterpret_cast<const unsigned char *>(s_xe);
        const unsigned char *s_pair = reinterpret_cast<const unsigned char *>(s_pairs);
        double are = 0.0, aim = 0.0;
        sa = make_double2(0.0, 0.0);
        sb = make_double2(0.0, 0.0);
        if (ng == 0)
            return;
        uint32_t row8 = (uint32_t)ra * 8u;
        int q = 0;
        for (; q + D <= ng; q += D) {
#pragma unroll
            for (int d = 0; d < D; d++) {
                if (q + d == nga) {
                    sa = make_double2(are, aim);
                    are = aim = 0.0;
                    row8 = (uint32_t)rb * 8u;
                }
                const sell_v4u c = g[d];
                g[d] = load(q + D + d);
                use<X>(c, s_x, s_pair, row8, are, aim);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < D; d++)
            if (q + d < ng) {
                if (q + d == nga) {
                    sa = make_double2(are, aim);
                    are = aim = 0.0;
                    row8 = (uint32_t)rb * 8u;
                }
                use<X>(g[d], s_x, s_pair, row8, are, aim);
            }
        if (ngb == 0)
            sa = make_double2(are, aim);
        else
            sb = make_double2(are, aim);
    }
};

// The block's rows from a wave's sums: sigma (FP32 storage: gathered in LDS
// and stored in row order), the energy terms and the block's partials.
template <int DT, int E, int D, bool RV, bool XI, typename X>
__device__ __forceinline__ void sell_finish(const SpmvState &st, int blk, const SellWave<DT, E, D, RV, XI> &w,
                                            const X *s_x, float2 *s_sig, double2 sa, double2 sb)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int k = wid + 16 * h;
        const int i = k * VQE_WAVE + lane;
        if (k < w.ns && i < w.n) {
            const int64_t row = w.r0 + (h ? w.rb : w.ra);
            const double2 a = h ? sb : sa;
            if constexpr (DT == VQE_C64)
                s_sig[row - w.r0] = make_float2((float)a.x, (float)a.y);
            else
                Elem<DT>::st(st.sigma, row, a);
            energy_terms(s_x[row], a.x, a.y, e_re, e_im, e_n2);
        }
    }
    if constexpr (DT == VQE_C64) {
        // the block's results leave in row order
        __syncthreads();
        for (int i = tid; i < w.n; i += 1024)
            stg(reinterpret_cast<float2 *>(st.sigma), w.r0 + i, s_sig[i]);
    }
    __shared__ double s_part[16][3];
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (tid < 3) {
        double v = 0.0;
        for (int q = 0; q < 16; q++)
            v += s_part[q][tid];
        gmem(st.partials)[(int64_t)blk * 3 + tid] = v;
    }
}

// The same for np parts (SPMV_VD_PART_ROWS sorted rows each) of a block from
// part p0 on, with a triple of partials per part: the sums' order is the same
// however the parts are split over workgroups.  A whole block's results leave
// in row order; a split one's rows lie all over the block and leave one by one.
// w: the wave's slices (as SellWave), x_at: the state's element of a row.
template <typename W, typename F>
__device__ __forceinline__ void vd_finish(const SpmvState &st, int blk, int p0, int np, const W &w, F x_at,
                                          float2 *s_sig, double2 sa, double2 sb)
{
    constexpr int SLICES = SPMV_VD_PART_ROWS / VQE_WAVE, PARTS = SPMV_LDS_ROWS / SPMV_VD_PART_ROWS;
    __shared__ double s_part[SPMV_SLICES_PER_BLOCK][3];
    const int tid = threadIdx.x, lane = tid & 63;
    const bool whole = np == PARTS;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int k = h ? w.kb : w.ka;
        if (k >= SPMV_SLICES_PER_BLOCK)
            continue;
        double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;
        const int i = k * VQE_WAVE + lane;
        if (k < w.ns && i < w.n) {
            const int64_t row = w.r0 + (h ? w.rb : w.ra);
            const double2 a = h ? sb : sa;
            if (whole)
                s_sig[row - w.r0] = make_float2((float)a.x, (float)a.y);
            else
                Elem<VQE_C64>::st(st.sigma, row, a);
            energy_terms(x_at(row), a.x, a.y, e_re, e_im, e_n2);
        }
        e_re = wave_sum(e_re);
        e_im = wave_sum(e_im);
        e_n2 = wave_sum(e_n2);
        if (lane == 0) {
            s_part[k][0] = e_re;
            s_part[k][1] = e_im;
            s_part[k][2] = e_n2;
        }
    }
    __syncthreads();
    if (whole)
        for (int i = tid; i < w.n; i += 1024)
            stg(reinterpret_cast<float2 *>(st.sigma), w.r0 + i, s_sig[i]);
    const int p = p0 + tid / 3, q = tid % 3;
    if (tid < 3 * np && p * SPMV_VD_PART_ROWS < w.n) {
        double v = 0.0;
        for (int k = 0; k < SLICES; k++)
            v += s_part[p * SLICES + k][q];
        gmem(st.partials)[((int64_t)blk * PARTS + p) * 3 + q] = v;
    }
}

// One workgroup per (state, block of SPMV_LDS_ROWS rows): the state staged in
// LDS (plus the zero element), then the block's slices; each wave's first
// groups are loaded together with the staged state.  With RV (the real parts
// of a real H) a state whose imaginary parts are all zero is staged as FP64
// real parts and multiplied in real arithmetic; any other state takes the
// complex staging in the same launch.  XI: the flip-mask index form, its
// masks staged after the block's results (every one of the SPMV_XIDX_MAX
// slots written, zero past the operator's count, so every index gives a
// column below dim).
template <int DT, int E, int D, bool RV, bool XI, bool VD, bool RS>
__device__ __forceinline__ void sell_block(const SpmvState &st, const int2 t)
{
    using T = typename Elem<DT>::T;
    extern __shared__ unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t dim = st.dim;
    const T *psi = reinterpret_cast<const T *>(st.psi);
    // FP32 storage: the block's results gather in LDS after the state
    float2 *s_sig = reinterpret_cast<float2 *>(smem + (size_t)(dim + 1) * sizeof(T));
    uint16_t *s_xt = reinterpret_cast<uint16_t *>(
        smem + (size_t)(dim + 1) * sizeof(T) + (DT == VQE_C64 ? SPMV_LDS_ROWS * sizeof(float2) : 0));
    // VD: the signed pairs where the results go later
    static_assert(2 * SPMV_VD_PAIRS * sizeof(uint2) == SPMV_LDS_ROWS * sizeof(float2), "pairs in the results' place");
    uint2 *s_pair = reinterpret_cast<uint2 *>(s_sig);
    // a task is a block, or with VD np of its parts from p0 on: one slice per
    // wave when they are fewer than all
    int blk = t.y, p0 = 0, np = 0, ka = wid, kb = wid + 16;
    if constexpr (VD) {
        constexpr int PARTS = SPMV_LDS_ROWS / SPMV_VD_PART_ROWS, SLICES = SPMV_VD_PART_ROWS / VQE_WAVE;
        np = t.y & 7;
        p0 = (t.y >> 3) % PARTS;
        blk = (t.y >> 3) / PARTS;
        if (np != PARTS) {
            ka = wid < np * SLICES ? p0 * SLICES + wid : SPMV_SLICES_PER_BLOCK;
            kb = SPMV_SLICES_PER_BLOCK;
        }
    }
    static_assert(!VD || DT == VQE_C64, "the dictionary form: FP32 storage");
    constexpr bool DICT = VD && XI;     // (VD alone: an operator past the index form)
    SellWave<DT, E, D, RV, XI> w;
    w.init(st, blk, lane, ka, kb);
    if constexpr (XI) {
        static_assert(SPMV_XIDX_MAX <= 1024, "one mask per thread");
        s_xt[tid] = tid < st.nx ? gmem(st.sxtab)[tid] : (uint16_t)0;
    }
    // DICT: the dictionary's codes run first, then the other entries, whose first
    // groups load meanwhile
    DictWave<SPMV_VD_DEPTH> dw;
    if constexpr (DICT) {
        const sell_v2u pr = gmem(reinterpret_cast<const sell_v2u *>(st.dpair))[tid];
        s_pair[2 * tid] = make_uint2(pr.x, pr.y);
        s_pair[2 * tid + 1] = make_uint2(pr.x ^ 0x80000000u, pr.y);
        dw.init(st, blk, lane, ka, kb, w.ns);
    }
    double2 sa, sb;
    auto products = [&](const auto *s_x) {
        if constexpr (DICT) {
            double2 da, db;
            if (w.ng > 0)
                w.prefetch();
            dw.run(s_x, s_pair, w.r0 + w.ra, w.r0 + w.rb, da, db);
            w.run(s_x, s_xt, sa, sb);
            sa = make_double2(sa.x + da.x, sa.y + da.y);
            sb = make_double2(sb.x + db.x, sb.y + db.y);
            __syncthreads();      // the results take the pairs' place
        } else {
            w.run(s_x, s_xt, sa, sb);
        }
    };
    auto finish = [&](const auto *s_x) {
        if constexpr (VD)
            vd_finish(st, blk, p0, np, w, [&](int64_t r) { return s_x[r]; }, s_sig, sa, sb);
        else
            sell_finish(st, blk, w, s_x, s_sig, sa, sb);
    };
    auto first_groups = [&]() {
        if constexpr (DICT) {
            if (dw.ng > 0)
                dw.prefetch();
        } else if (w.ng > 0) {
            w.prefetch();
        }
    };
    if constexpr (RS) {
        first_groups();
        double *s_xr = reinterpret_cast<double *>(smem);
        const int cplx = stage_real<8>(s_xr, psi, dim, tid);
        if (tid == 0)
            s_xr[dim] = 0.0;
        if (!__syncthreads_or(cplx)) {
            products(s_xr);
            finish(s_xr);
            return;
        }
    }
    // the state in 16-byte chunks (dim * sizeof(T) is a multiple of 16 and
    // psi 16-byte aligned): the first SP per thread loaded before the wave's
    // first groups, so both latencies overlap
    T *s_x = reinterpret_cast<T *>(smem);
    constexpr int SP = 8;
    const int64_t nch = dim * (int64_t)sizeof(T) / 16;
    const vqe_v4f *src = reinterpret_cast<const vqe_v4f *>(psi);
    vqe_v4f *dst = reinterpret_cast<vqe_v4f *>(s_x);
    vqe_v4f pre[SP];
#pragma unroll
    for (int u = 0; u < SP; u++) {
        const int64_t c = tid + 1024 * u;
        if (c < nch)
            pre[u] = gmem(src)[c];
    }
    if (!RS)
        first_groups();
#pragma unroll
    for (int u = 0; u < SP; u++) {
        const int64_t c = tid + 1024 * u;
        if (c < nch)
            dst[c] = pre[u];
    }
    for (int64_t c = tid + 1024 * SP; c < nch; c += 1024)
        dst[c] = gmem(src)[c];
    if (tid == 0)
        s_x[dim] = T{};
    __syncthreads();
    products(s_x);
    finish(s_x);
}

template <int DT, int E, int D, bool RV, bool XI, bool VD, bool RS>
__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_sell(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 t = tasks[blockIdx.x];
    if (t.x < 0)
        return;
    const SpmvState st = states[t.x];
    if (VQE_SKIP(st))
        return;
    // beside a dictionary the operator says whether its values are real parts;
    // past the index form (no codes) its entries are 16-bit columns, four a
    // group of real parts, two of complex values
    if constexpr (VD) {
        if (!st.dcode) {
            if constexpr (!RV) {
                if (!st.rvals) {
                    sell_block<DT, SPMV_VD_COLS(false), 4, false, false, true, RS>(st, t);
                    return;
                }
            }
            sell_block<DT, SPMV_VD_COLS(true), 3, true, false, true, RS>(st, t);
            return;
        }
        if constexpr (!RV) {
            if (st.rvals) {
                sell_block<DT, E, D, true, XI, VD, RS>(st, t);
                return;
            }
        }
    }
    sell_block<DT, E, D, RV, XI, VD, RS>(st, t);
}

// Column-tiled variant of the pipelined LDS schedule, for states larger than
// LDS.  A workgroup takes one block of rows and one column tile: it stages
// that tile of the state (SPMV_TILE_BYTES) and, per row, streams only the
// row's entries in the tile -- a contiguous sub-range, since columns are
// sorted within a row, bounded by the per-tile row pointers.  The row sums of
// a tile go to an FP64 partial array; the tile-sum kernel adds the tiles in
// ascending order and applies the energy epilogue.

// The rows [r0, r1) of one column tile t of the column-tiled schedule, the
// columns [c_lo, c_lo + tc) staged in LDS at smem (complex, or with RX the
// real parts in storage precision) and the rows' tile bounds at s_k0, s_k1;
// entries outside those columns are masked.  Writes the FP64 tile partials,
// or adds to them (accumulate).
template <int DT, int L, int D, int U, bool X16, bool RV, bool RX>
__device__ __forceinline__ void tiled_rows(const SpmvState &st, int t, int c_lo, int tc,
                                           bool accumulate, const unsigned char *smem,
                                           const int32_t *s_k0, const int32_t *s_k1, int64_t r0,
                                           int64_t r1)
{
    using X = typename std::conditional<RX, typename ValOf<DT, true>::T,
                                        typename Elem<DT>::T>::type;
    constexpr int W = U * 4;
    constexpr int PASS = W * L;
    using V = typename ValOf<DT, RV>::T;
    constexpr unsigned EB = sizeof(V);
    const X *s_x = reinterpret_cast<const X *>(smem);
    const int tid = threadIdx.x;
    const int64_t dim = st.dim;
    constexpr int G = VQE_WAVE / L;
    const int lane = tid & 63, wid = tid >> 6;
    const int sub = lane / L, sl = lane % L;
    const int nnz = (int)st.nnz, zc = tc;
    const int whole = nnz & ~3;
    const __amdgpu_buffer_rsrc_t rc =
        X16 ? __builtin_amdgcn_make_buffer_rsrc((void *)st.col16, (short)0, nnz * 2, VQE_BUF_WORD3)
            : __builtin_amdgcn_make_buffer_rsrc((void *)st.col, (short)0, nnz * 4, VQE_BUF_WORD3);
    const __amdgpu_buffer_rsrc_t rv =
        __builtin_amdgcn_make_buffer_rsrc((void *)(RV ? st.vre : st.val), (short)0, (int)(nnz * EB),
                                          VQE_BUF_WORD3);
    double *__restrict__ part = st.tile_part + (int64_t)t * dim * 2;

    auto issue = [&](int kb, int k1, int c[W], V v[W]) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int k = kb + u * 4 * L;
            const bool ok = k < k1 && k < whole;
            if (X16) {
                typedef unsigned v2u __attribute__((ext_vector_type(2)));
                const v2u c2 = __builtin_amdgcn_raw_buffer_load_b64(rc, ok ? (unsigned)k * 2u : VQE_BUF_OOB, 0, 0);
                c[4 * u + 0] = (int)(c2.x & 0xffffu);
                c[4 * u + 1] = (int)(c2.x >> 16);
                c[4 * u + 2] = (int)(c2.y & 0xffffu);
                c[4 * u + 3] = (int)(c2.y >> 16);
            } else {
                typedef int v4i __attribute__((ext_vector_type(4)));
                const v4i c4 = __builtin_amdgcn_raw_buffer_load_b128(rc, ok ? (unsigned)k * 4u : VQE_BUF_OOB, 0, 0);
                c[4 * u + 0] = c4.x;
                c[4 * u + 1] = c4.y;
                c[4 * u + 2] = c4.z;
                c[4 * u + 3] = c4.w;
            }
            BufVal<DT, RV>::load(rv, ok ? (unsigned)k * EB : VQE_BUF_OOB, v + 4 * u);
        }
    };
    // entries outside [k0, k1) (or not loaded) read the zero element; the
    // column test keeps every LDS index inside the tile
    auto consume = [&](int64_t r, int kb, int k0, int k1, const int c[W], const V v[W],
                       double &are, double &aim) {
        int cm[W];
        const unsigned len = (unsigned)(k1 - k0);
        const int rx = (int)r;
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int k = kb + u * 4 * L + q;
                const int cl = (X16 ? (rx ^ c[4 * u + q]) : c[4 * u + q]) - c_lo;
                cm[4 * u + q] = ((unsigned)(k - k0) < len && (unsigned)cl < (unsigned)tc) ? cl : zc;
            }
        lds_gather_fma<X, V, W>(s_x, cm, v, are, aim);
    };
    auto row_bounds = [&](int64_t r, int &k0, int &k1) {
        if (r < r1) {
            k0 = s_k0[r - r0];
            k1 = s_k1[r - r0];
        } else {
            k0 = k1 = 0;
        }
    };
    auto finish = [&](int64_t r, int k0, int k1, double are, double aim) {
        for (int kb = (k0 & ~3) + 4 * sl + PASS; kb - 4 * sl < k1; kb += PASS) {
            int c[W];
            V v[W];
            issue(kb, k1, c, v);
            consume(r, kb, k0, k1, c, v, are, aim);
        }
        if (k1 > whole) {
            const int k = (k0 > whole ? k0 : whole) + sl;
            if (k < k1) {
                const V a = ldv(reinterpret_cast<const V *>(RV ? st.vre : st.val), k);
                const int col = X16 ? ((int)r ^ (int)gmem(st.col16)[k]) : gmem(st.col)[k];
                if ((unsigned)(col - c_lo) < (unsigned)tc)
                    entry_fma(a, s_x[col - c_lo], are, aim);
            }
        }
        are = group_sum<L>(are);
        if (!RX)
            aim = group_sum<L>(aim);
        if (sl == 0 && r < r1) {
            if (accumulate) {
                are += gmem(part)[2 * r];
                aim += gmem(part)[2 * r + 1];
            }
            gmem(part)[2 * r] = are;
            gmem(part)[2 * r + 1] = aim;
        }
    };

    int cb[D][W];
    V vb[D][W];
    int kb0[D], kb1[D];
    int64_t rr[D];
#pragma unroll
    for (int d = 0; d < D; d++) {
        rr[d] = r0 + (wid + 16 * d) * G + sub;
        row_bounds(rr[d], kb0[d], kb1[d]);
        issue((kb0[d] & ~3) + 4 * sl, kb1[d], cb[d], vb[d]);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int64_t base = r0 + wid * G; base < r1; base += 16 * D * G) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            {
                double are = 0.0, aim = 0.0;
                consume(rr[d], (kb0[d] & ~3) + 4 * sl, kb0[d], kb1[d], cb[d], vb[d], are, aim);
                finish(rr[d], kb0[d], kb1[d], are, aim);
            }
            rr[d] += 16 * D * G;
            row_bounds(rr[d], kb0[d], kb1[d]);
            issue((kb0[d] & ~3) + 4 * sl, kb1[d], cb[d], vb[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}


template <int DT, int L, int D, int U, bool X16, bool RV>
__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_tiled(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 task = tasks[blockIdx.x];
    if (task.x < 0)
        return;
    const SpmvState st = states[task.x];
    if (VQE_SKIP(st))
        return;
    const int blk = task.y >> 8, t = task.y & 0xff;
    using T = typename Elem<DT>::T;
    extern __shared__ unsigned char smem[];
    T *s_x = reinterpret_cast<T *>(smem);
    const int tid = threadIdx.x;
    const int64_t dim = st.dim;
    const int tc = st.tile_cols;
    const int c_lo = t * tc;
    const T *__restrict__ psi = reinterpret_cast<const T *>(st.psi);
    const int64_t r0 = (int64_t)blk * SPMV_LDS_ROWS;
    const int64_t r1 = r0 + SPMV_LDS_ROWS < dim ? r0 + SPMV_LDS_ROWS : dim;
    // the tile, one zero element (index tc), then the block's tile bounds.
    // With real values (RV) the plan's tiles are twice as wide: a tile with no
    // imaginary part is staged as its real parts in storage precision; a
    // complex one runs as two half-width passes (complex elements), each over
    // the rows' whole segments with the columns outside its half masked, the
    // second adding to the first's partials
    const size_t x_bytes = (size_t)((RV ? tc / 2 : tc) + 1) * sizeof(T);
    int32_t *s_k0 = reinterpret_cast<int32_t *>(smem + x_bytes);
    int32_t *s_k1 = s_k0 + SPMV_LDS_ROWS;
    stage_lds<2>(s_k0, st.tptr + (int64_t)t * dim + r0, r1 - r0, tid);
    stage_lds<2>(s_k1, st.tptr + (int64_t)(t + 1) * dim + r0, r1 - r0, tid);
    if constexpr (RV) {
        using R = typename ValOf<DT, true>::T;
        R *s_xr = reinterpret_cast<R *>(smem);
        const int cplx = stage_real_as<8, R>(s_xr, psi + c_lo, (int64_t)tc, tid);
        if (tid == 0)
            s_xr[tc] = (R)0;
        if (!__syncthreads_or(cplx)) {
            tiled_rows<DT, L, D, U, X16, RV, true>(st, t, c_lo, tc, false, smem, s_k0, s_k1, r0, r1);
            return;
        }
        const int th = tc / 2;
        for (int h = 0; h < 2; h++) {
            stage_lds<8>(s_x, psi + c_lo + h * th, (int64_t)th, tid);
            if (tid == 0)
                s_x[th] = T{};
            __syncthreads();
            tiled_rows<DT, L, D, U, X16, RV, false>(st, t, c_lo + h * th, th, h == 1, smem, s_k0,
                                                    s_k1, r0, r1);
            __syncthreads();      // every wave is done with this half
        }
        return;
    }
    stage_lds<8>(s_x, psi + c_lo, (int64_t)tc, tid);
    if (tid == 0)
        s_x[tc] = T{};
    __syncthreads();
    tiled_rows<DT, L, D, U, X16, RV, false>(st, t, c_lo, tc, false, smem, s_k0, s_k1, r0, r1);
}

// sigma_r = sum over tiles (ascending) of the tile partials; the energy sums.
template <int DT>
__global__ void __launch_bounds__(256)
k_spmv_tile_sum(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 task = tasks[blockIdx.x];
    if (task.x < 0)
        return;
    const SpmvState st = states[task.x];
    if (VQE_SKIP(st))
        return;
    const int64_t dim = st.dim;
    const int64_t r0 = (int64_t)task.y * SPMV_SUM_ROWS;
    const int64_t r1 = r0 + SPMV_SUM_ROWS < dim ? r0 + SPMV_SUM_ROWS : dim;
    double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;
    for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
        double sr = 0.0, si = 0.0;
        for (int t = 0; t < st.ntiles; t++) {
            sr += gmem(st.tile_part)[((int64_t)t * dim + r) * 2];
            si += gmem(st.tile_part)[((int64_t)t * dim + r) * 2 + 1];
        }
        Elem<DT>::st(st.sigma, r, make_double2(sr, si));
        const double2 p = Elem<DT>::ld(st.psi, r);
        e_re += p.x * sr + p.y * si;
        e_im += p.x * si - p.y * sr;
        e_n2 += p.x * p.x + p.y * p.y;
    }
    __shared__ double s_part[4][3];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int q = threadIdx.x;
        gmem(st.partials)[(int64_t)task.y * 3 + q] =
            ((s_part[0][q] + s_part[1][q]) + s_part[2][q]) + s_part[3][q];
    }
}

// ------------------------------------------------------------------ blocked layout
// The column-tiled product of states larger than LDS, blocked: the plan lays
// H out per (row block, column tile) slab (the entries of the block's rows
// whose columns fall in the tile, rows in order, each slab starting at a
// multiple of four entries), with 16-bit tile-local column codes (any state
// size, since a tile holds fewer than 2^16 columns) and the values (complex,
// interleaved).  One workgroup owns a row block and walks every tile in
// ascending order: it stages the tile of the state and the slab's row
// pointers in LDS, streams the slab with the pipelined row loop, and adds each
// row's sum to the row's FP64 accumulator in LDS; after the last tile it
// writes sigma and the energy partials.  Each slab is one contiguous stream,
// so no line is shared between two workgroups' reads, and no per-tile partial
// sums go through device memory.

// first k in [lo, hi) with col[k] >= lim (columns ascend within a row)
__device__ __forceinline__ int first_col_at_least(const int32_t *col, int lo, int hi, int64_t lim)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)col[mid] < lim)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Step 1: the number of entries of row r in tile t, stored in the slab's
// row-pointer slot i + 1 (i = r - block * R); one thread per (row, tile),
// tiles fastest.  The slots start zeroed.
__global__ void __launch_bounds__(256)
k_blk_count(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int64_t dim,
            int32_t nt, int32_t tc, int32_t R, int32_t *__restrict__ brp)
{
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= dim * nt)
        return;
    const int64_t r = gid / nt;
    const int t = (int)(gid - r * nt);
    const int k0 = rowptr[r], k1 = rowptr[r + 1];
    const int lo = first_col_at_least(col, k0, k1, (int64_t)t * tc);
    const int hi = first_col_at_least(col, lo, k1, (int64_t)(t + 1) * tc);
    const int64_t b = r / R, i = r - b * R;
    brp[(b * nt + t) * (R + 1) + i + 1] = hi - lo;
}

// Step 2: per slab (one 256-thread workgroup), the row lengths in slots
// 1..R become the rows' starts (inclusive prefix sums: slot i = start of row
// i, slot R = the slab's length); the slab's length rounded up to four entries
// goes to blen.
__global__ void __launch_bounds__(256)
k_blk_scan(int32_t *__restrict__ brp, int32_t R, int64_t *__restrict__ blen)
{
    __shared__ int32_t s_tot[256];
    const int tid = threadIdx.x;
    int32_t *p = brp + (int64_t)blockIdx.x * (R + 1);
    const int per = (R + 255) / 256;
    const int a = 1 + tid * per;
    const int e = a + per < R + 1 ? a + per : R + 1;
    int32_t sum = 0;
    for (int i = a; i < e; i++)
        sum += p[i];
    s_tot[tid] = sum;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int32_t v = tid >= off ? s_tot[tid - off] : 0;
        __syncthreads();
        s_tot[tid] += v;
        __syncthreads();
    }
    int32_t run = s_tot[tid] - sum;
    for (int i = a; i < e; i++) {
        run += p[i];
        p[i] = run;
    }
    if (tid == 0)
        p[0] = 0;
    if (tid == 255)
        blen[blockIdx.x] = ((int64_t)s_tot[255] + 3) & ~(int64_t)3;
}

// Step 3: slab starts, the exclusive prefix sums of the rounded lengths
// (boff[n] = the total); one workgroup, each thread a contiguous run.
__global__ void __launch_bounds__(1024)
k_blk_offsets(const int64_t *__restrict__ blen, int64_t n, int64_t *__restrict__ boff)
{
    __shared__ int64_t s_sum[1024];
    const int tid = threadIdx.x;
    const int64_t per = (n + 1023) / 1024;
    const int64_t a = (int64_t)tid * per < n ? (int64_t)tid * per : n;
    const int64_t e = a + per < n ? a + per : n;
    int64_t tot = 0;
    for (int64_t i = a; i < e; i++)
        tot += blen[i];
    s_sum[tid] = tot;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t v = tid >= off ? s_sum[tid - off] : 0;
        __syncthreads();
        s_sum[tid] += v;
        __syncthreads();
    }
    int64_t run = s_sum[tid] - tot;
    for (int64_t i = a; i < e; i++) {
        boff[i] = run;
        run += blen[i];
    }
    if (tid == 1023)
        boff[n] = s_sum[1023];
}

// Step 4: copy row r's entries of tile t into its slab (codes col - t * tc),
// one thread per (row, tile); the entries between one slab's end and the next
// slab's start are set to zero by the thread of the block's last row.
template <int DT>
__global__ void __launch_bounds__(256)
k_blk_fill(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
           const void *__restrict__ val, int64_t dim, int32_t nt, int32_t tc, int32_t R,
           const int32_t *__restrict__ brp, const int64_t *__restrict__ boff,
           uint16_t *__restrict__ bcode, void *__restrict__ bval)
{
    using T = typename Elem<DT>::T;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= dim * nt)
        return;
    const int64_t r = gid / nt;
    const int t = (int)(gid - r * nt);
    const int k0 = rowptr[r], k1 = rowptr[r + 1];
    const int lo = first_col_at_least(col, k0, k1, (int64_t)t * tc);
    const int hi = first_col_at_least(col, lo, k1, (int64_t)(t + 1) * tc);
    const int64_t b = r / R, i = r - b * R;
    const int64_t slab = b * nt + t;
    const int32_t *rp = brp + slab * (R + 1);
    const int64_t dst = boff[slab] + rp[i];
    const T *v = reinterpret_cast<const T *>(val);
    T *bv = reinterpret_cast<T *>(bval);
    for (int k = lo; k < hi; k++) {
        bcode[dst + (k - lo)] = (uint16_t)(col[k] - t * tc);
        bv[dst + (k - lo)] = v[k];
    }
    const int64_t rows = dim - b * R < R ? dim - b * R : R;
    if (i == rows - 1)
        for (int64_t k = boff[slab] + rp[rows]; k < boff[slab + 1]; k++) {
            bcode[k] = 0;
            bv[k] = T{};
        }
}

// The rows of one slab of a blocked state (tile of the state at s_x, its
// zero element at index w; the slab's row pointers at s_rp): the pipelined row
// loop of the LDS schedule with L lanes per row, U groups of four entries per
// lane per pass and D rows in flight per sub-group; each row's sum is added to
// its FP64 accumulator in LDS.
template <int DT, int L, int D, int U>
__device__ __forceinline__ void blk_rows(const SpmvState &st, int64_t slab, int w,
                                         const typename Elem<DT>::T *s_x, const int32_t *s_rp,
                                         double2 *s_acc, int nrows)
{
    using T = typename Elem<DT>::T;
    constexpr int W = U * 4;                 // entries per lane per pass
    constexpr int PASS = W * L;              // entries per sub-group per pass
    constexpr unsigned EB = sizeof(T);
    constexpr int G = VQE_WAVE / L;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wid = tid >> 6;
    const int sub = lane / L, sl = lane % L;
    const int64_t base = st.boff[slab];
    const int nrec = (s_rp[nrows] + 3) & ~3;   // the slab's entries, whole groups
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(st.bcode + base), (short)0, nrec * 2, VQE_BUF_WORD3);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(reinterpret_cast<const T *>(st.bval) + base), (short)0, (int)(nrec * EB),
        VQE_BUF_WORD3);

    auto issue = [&](int kb, int k1, int c[W], T v[W]) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int k = kb + u * 4 * L;
            const bool ok = k < k1;
            typedef unsigned v2u __attribute__((ext_vector_type(2)));
            const v2u c2 = __builtin_amdgcn_raw_buffer_load_b64(rc, ok ? (unsigned)k * 2u : VQE_BUF_OOB, 0, 0);
            c[4 * u + 0] = (int)(c2.x & 0xffffu);
            c[4 * u + 1] = (int)(c2.x >> 16);
            c[4 * u + 2] = (int)(c2.y & 0xffffu);
            c[4 * u + 3] = (int)(c2.y >> 16);
            BufVal<DT, false>::load(rv, ok ? (unsigned)k * EB : VQE_BUF_OOB, v + 4 * u);
        }
    };
    // entries outside the row [k0, k1) read the zero element
    auto consume = [&](int kb, int k0, int k1, const int c[W], const T v[W], double &are,
                       double &aim) {
        int cm[W];
        const unsigned len = (unsigned)(k1 - k0);
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int k = kb + u * 4 * L + q;
                cm[4 * u + q] = (unsigned)(k - k0) < len ? c[4 * u + q] : w;
            }
        lds_gather_fma<T, T, W>(s_x, cm, v, are, aim);
    };
    auto row_bounds = [&](int i, int &k0, int &k1) {
        if (i < nrows) {
            k0 = s_rp[i];
            k1 = s_rp[i + 1];
        } else {
            k0 = k1 = 0;
        }
    };
    auto finish = [&](int i, int k0, int k1, double are, double aim) {
        for (int kb = (k0 & ~3) + 4 * sl + PASS; kb - 4 * sl < k1; kb += PASS) {
            int c[W];
            T v[W];
            issue(kb, k1, c, v);
            consume(kb, k0, k1, c, v, are, aim);
        }
        are = group_sum<L>(are);
        aim = group_sum<L>(aim);
        if (sl == 0 && i < nrows) {
            const double2 a = s_acc[i];
            s_acc[i] = make_double2(a.x + are, a.y + aim);
        }
    };

    int cb[D][W];
    T vb[D][W];
    int kb0[D], kb1[D], rr[D];
#pragma unroll
    for (int d = 0; d < D; d++) {
        rr[d] = (wid + 16 * d) * G + sub;
        row_bounds(rr[d], kb0[d], kb1[d]);
        issue((kb0[d] & ~3) + 4 * sl, kb1[d], cb[d], vb[d]);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int row = wid * G; row < nrows; row += 16 * D * G) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            {
                double are = 0.0, aim = 0.0;
                consume((kb0[d] & ~3) + 4 * sl, kb0[d], kb1[d], cb[d], vb[d], are, aim);
                finish(rr[d], kb0[d], kb1[d], are, aim);
            }
            rr[d] += 16 * D * G;
            row_bounds(rr[d], kb0[d], kb1[d]);
            issue((kb0[d] & ~3) + 4 * sl, kb1[d], cb[d], vb[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// The blocked product's kernel: one workgroup per (state, row block).
template <int DT, int L, int D, int U>
__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_blk(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 task = tasks[blockIdx.x];
    if (task.x < 0)
        return;
    const SpmvState st = states[task.x];
    if (VQE_SKIP(st))
        return;
    using T = typename Elem<DT>::T;
    extern __shared__ unsigned char smem[];
    const int tid = threadIdx.x;
    const int64_t dim = st.dim;
    const int R = st.blk_rows, tc = st.tile_cols, nt = st.ntiles;
    const int b = task.y;
    const int64_t r0 = (int64_t)b * R;
    const int nrows = (int)(dim - r0 < R ? dim - r0 : R);
    // LDS: the rows' accumulators, the tile (and its zero element), the
    // slab's row pointers
    double2 *s_acc = reinterpret_cast<double2 *>(smem);
    T *s_x = reinterpret_cast<T *>(smem + (size_t)R * sizeof(double2));
    int32_t *s_rp = reinterpret_cast<int32_t *>(smem + (size_t)R * sizeof(double2) +
                                                (size_t)(tc + 1) * sizeof(T));
    const T *__restrict__ psi = reinterpret_cast<const T *>(st.psi);
    for (int i = tid; i < nrows; i += 1024)
        s_acc[i] = make_double2(0.0, 0.0);
    for (int t = 0; t < nt; t++) {
        const int64_t c_lo = (int64_t)t * tc;
        const int w = (int)(dim - c_lo < tc ? dim - c_lo : tc);
        const int64_t slab = (int64_t)b * nt + t;
        __syncthreads();      // every wave is done with the previous tile
        stage_lds<2>(s_rp, st.brp + slab * (R + 1), nrows + 1, tid);
        stage_lds<8>(s_x, psi + c_lo, w, tid);
        if (tid == 0)
            s_x[w] = T{};
        __syncthreads();
        blk_rows<DT, L, D, U>(st, slab, w, s_x, s_rp, s_acc, nrows);
    }
    __syncthreads();
    double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;
    for (int i = tid; i < nrows; i += 1024) {
        const double2 a = s_acc[i];
        Elem<DT>::st(st.sigma, r0 + i, a);
        energy_terms(ldg(psi, r0 + i), a.x, a.y, e_re, e_im, e_n2);
    }
    __shared__ double s_part[16][3];
    const int lane = tid & 63, wid = tid >> 6;
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (tid < 3) {
        double v = 0.0;
        for (int q = 0; q < 16; q++)
            v += s_part[q][tid];
        gmem(st.partials)[(int64_t)b * 3 + tid] = v;
    }
}

// Per-tile row bounds: the first entry of row r with column >= t * tile_cols.
__global__ void __launch_bounds__(256)
k_tile_bounds(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 task = tasks[blockIdx.x];
    if (task.x < 0)
        return;
    const SpmvState st = states[task.x];
    const int64_t r = (int64_t)task.y * 256 + threadIdx.x;
    if (r >= st.dim)
        return;
    const int k0 = st.rowptr[r], k1 = st.rowptr[r + 1];
    int32_t *tp = const_cast<int32_t *>(st.tptr);
    tp[r] = k0;
    for (int t = 1; t < st.ntiles; t++) {
        const int lim = t * st.tile_cols;
        int lo = k0, hi = k1;   // first k in [k0, k1) with col[k] >= lim
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (st.col[mid] < lim)
                lo = mid + 1;
            else
                hi = mid;
        }
        tp[(int64_t)t * st.dim + r] = lo;
    }
    tp[(int64_t)st.ntiles * st.dim + r] = k1;
}

}  // namespace

// Fixed-order sum of the block partials, then out = {shift + re/n2, n2, im}; a
// wave for each of the three sums, 16 loads in flight per lane (one wave with
// one load of each in flight took 36 us for the 8192 blocks of 16 qubits).
__global__ void __launch_bounds__(192)
k_energy_finalize(SpmvState single)
{
    __shared__ double s_sum[3];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const double *p = single.partials + q;
    const int n = single.nblocks;
    double v = 0.0;
    for (int b0 = lane; b0 < n; b0 += 64 * 16) {
        double t[16];
#pragma unroll
        for (int u = 0; u < 16; u++)
            t[u] = b0 + 64 * u < n ? gmem(p)[(int64_t)(b0 + 64 * u) * 3] : 0.0;
#pragma unroll
        for (int u = 0; u < 16; u++)
            if (b0 + 64 * u < n)
                v += t[u];
    }
    v = wave_sum(v);
    if (lane == 0)
        s_sum[q] = v;
    __syncthreads();
    if (threadIdx.x == 0 && single.energy_out) {
        single.energy_out[0] = single.shift + s_sum[0] / s_sum[2];
        single.energy_out[1] = s_sum[2];
        single.energy_out[2] = s_sum[1];
    }
}

template <int DT, int L, int V>
static void launch_spmv_t(const SpmvState &single, const SpmvState *states, const int2 *tasks,
                          unsigned grid, hipStream_t s)
{
    if (tasks)
        k_spmv_energy<DT, L, V, true><<<grid, 256, 0, s>>>(single, states, tasks);
    else
        k_spmv_energy<DT, L, V, false><<<grid, 256, 0, s>>>(single, states, tasks);
}

template <int DT, int L, int U>
static void launch_spmv_lds_t(const SpmvState &single, const SpmvState *states, const int2 *tasks,
                              unsigned grid, hipStream_t s, size_t lds)
{
    if (tasks) {
        auto k = k_spmv_lds<DT, L, U, true>;
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        k<<<grid, 1024, lds, s>>>(single, states, tasks);
    } else {
        auto k = k_spmv_lds<DT, L, U, false>;
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        k<<<grid, 1024, lds, s>>>(single, states, tasks);
    }
}

template <int DT, int L, int D, bool X16 = false, bool RV = false, bool PL = RV>
static void launch_spmv_pf_t(const SpmvState &single, const SpmvState *states, const int2 *tasks,
                             unsigned grid, hipStream_t s, size_t lds)
{
    if (tasks) {
        auto k = k_spmv_lds_pf<DT, L, D, true, X16, RV, PL>;
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        k<<<grid, 1024, lds, s>>>(single, states, tasks);
    } else {
        auto k = k_spmv_lds_pf<DT, L, D, false, false, false, false>;
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        k<<<grid, 1024, lds, s>>>(single, states, tasks);
    }
}

// Sliced schedules: E entries per lane and load group, D groups in flight;
// rv: the real parts of the values (VQE_SPMV_REAL).
template <int DT, int E, int D, bool XI = false, bool VD = false>
static void launch_sell_t(const SpmvState *states, const int2 *tasks, unsigned grid, hipStream_t s,
                          size_t lds, int sched)
{
    // the state (with its zero element; lds counts it with the row pointers
    // of the other LDS schedules), in FP32 storage a block of results, and
    // the flip masks of the index form
    lds = lds - (SPMV_LDS_ROWS + 1) * sizeof(int32_t) +
          (DT == VQE_C64 ? SPMV_LDS_ROWS * sizeof(float2) : 0) + (XI ? SPMV_XIDX_MAX * sizeof(uint16_t) : 0);
    const bool rs = (sched & VQE_SPMV_REAL) != 0;
    auto k = rs ? k_spmv_sell<DT, E, D, true, XI, VD, true> : k_spmv_sell<DT, E, D, false, XI, VD, false>;
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k<<<grid, 1024, lds, s>>>(states, tasks);
}

template <int DT>
static void launch_spmv_dt(int sched, const SpmvState &single, const SpmvState *states,
                           const int2 *tasks, unsigned grid, hipStream_t s, size_t lds)
{
    if ((sched & VQE_SPMV_SLICED) && tasks) {
        // the sliced layout exists only in batch plans; E = 2, 4 or 8
        // (FP64 values keep half as many groups in flight: the registers)
        constexpr bool W = DT == VQE_C128;
        if constexpr (DT == VQE_C64)
            if (sched & VQE_SPMV_VDICT) {
                if ((sched & 0xff) == 3)
                    launch_sell_t<DT, 3, 4, true, true>(states, tasks, grid, s, lds, sched);
                else
                    launch_sell_t<DT, 6, 2, true, true>(states, tasks, grid, s, lds, sched);
                return;
            }
        if (sched & VQE_SPMV_XIDX) {
            if ((sched & 0xff) == 3)
                launch_sell_t<DT, 3, W ? 2 : 6, true>(states, tasks, grid, s, lds, sched);
            else
                launch_sell_t<DT, 6, W ? 1 : 3, true>(states, tasks, grid, s, lds, sched);
            return;
        }
        switch (sched & 0xff) {
        case 2: launch_sell_t<DT, 2, W ? 2 : 4>(states, tasks, grid, s, lds, sched); return;
        case 8: launch_sell_t<DT, 8, W ? 1 : 2>(states, tasks, grid, s, lds, sched); return;
        default: launch_sell_t<DT, 4, W ? 2 : 3>(states, tasks, grid, s, lds, sched); return;
        }
    }
    constexpr int D = VQE_SPMV_LDS | VQE_SPMV_DEEP;
    constexpr int P = VQE_SPMV_LDS | VQE_SPMV_PREFETCH;
    constexpr int X = P | VQE_SPMV_X16;
    constexpr int R = X | VQE_SPMV_REAL;
    constexpr int Q = X | VQE_SPMV_PAD;
    switch (sched) {
    // the 16-bit column form, the padded layout and the real values exist
    // only in batch plans (tasks non-null)
    case 16 | Q: launch_spmv_pf_t<DT, 16, 2, true, false, true>(single, states, tasks, grid, s, lds); return;
    case 32 | Q: launch_spmv_pf_t<DT, 32, 2, true, false, true>(single, states, tasks, grid, s, lds); return;
    case 64 | Q: launch_spmv_pf_t<DT, 64, 2, true, false, true>(single, states, tasks, grid, s, lds); return;
    case 32 | Q | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 32, 3, true, false, true>(single, states, tasks, grid, s, lds); return;
    case 64 | Q | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 64, 3, true, false, true>(single, states, tasks, grid, s, lds); return;
    case 16 | R: launch_spmv_pf_t<DT, 16, 2, true, true>(single, states, tasks, grid, s, lds); return;
    case 32 | R: launch_spmv_pf_t<DT, 32, 2, true, true>(single, states, tasks, grid, s, lds); return;
    case 64 | R: launch_spmv_pf_t<DT, 64, 2, true, true>(single, states, tasks, grid, s, lds); return;
    case 32 | R | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 32, 3, true, true>(single, states, tasks, grid, s, lds); return;
    case 64 | R | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 64, 3, true, true>(single, states, tasks, grid, s, lds); return;
    case 32 | X: launch_spmv_pf_t<DT, 32, 2, true>(single, states, tasks, grid, s, lds); return;
    case 64 | X: launch_spmv_pf_t<DT, 64, 2, true>(single, states, tasks, grid, s, lds); return;
    case 32 | X | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 32, 3, true>(single, states, tasks, grid, s, lds); return;
    case 64 | X | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 64, 3, true>(single, states, tasks, grid, s, lds); return;
    case 32 | P: launch_spmv_pf_t<DT, 32, 2>(single, states, tasks, grid, s, lds); return;
    case 64 | P: launch_spmv_pf_t<DT, 64, 2>(single, states, tasks, grid, s, lds); return;
    case 32 | P | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 32, 3>(single, states, tasks, grid, s, lds); return;
    case 64 | P | VQE_SPMV_DEEP: launch_spmv_pf_t<DT, 64, 3>(single, states, tasks, grid, s, lds); return;
    default: break;
    }
    switch (sched) {
    case 8 | VQE_SPMV_LDS: launch_spmv_lds_t<DT, 8, 2>(single, states, tasks, grid, s, lds); return;
    case 16 | VQE_SPMV_LDS: launch_spmv_lds_t<DT, 16, 2>(single, states, tasks, grid, s, lds); return;
    case 32 | VQE_SPMV_LDS: launch_spmv_lds_t<DT, 32, 2>(single, states, tasks, grid, s, lds); return;
    case 64 | VQE_SPMV_LDS: launch_spmv_lds_t<DT, 64, 1>(single, states, tasks, grid, s, lds); return;
    case 8 | D: launch_spmv_lds_t<DT, 8, 4>(single, states, tasks, grid, s, lds); return;
    case 16 | D: launch_spmv_lds_t<DT, 16, 4>(single, states, tasks, grid, s, lds); return;
    case 32 | D: launch_spmv_lds_t<DT, 32, 4>(single, states, tasks, grid, s, lds); return;
    case 64 | D: launch_spmv_lds_t<DT, 64, 2>(single, states, tasks, grid, s, lds); return;
    default: break;
    }
    switch (sched) {
    case 8: launch_spmv_t<DT, 8, 1>(single, states, tasks, grid, s); break;
    case 16: launch_spmv_t<DT, 16, 1>(single, states, tasks, grid, s); break;
    case 32: launch_spmv_t<DT, 32, 1>(single, states, tasks, grid, s); break;
    case 64: launch_spmv_t<DT, 64, 1>(single, states, tasks, grid, s); break;
    case 16 | VQE_SPMV_VEC4: launch_spmv_t<DT, 16, 4>(single, states, tasks, grid, s); break;
    case 32 | VQE_SPMV_VEC4: launch_spmv_t<DT, 32, 4>(single, states, tasks, grid, s); break;
    default: launch_spmv_t<DT, 64, 4>(single, states, tasks, grid, s); break;
    }
}

// ------------------------------------------------------------------ sliced, column-tiled
// VQE_SPMV_SLICED on a state larger than LDS: slabs of a block of
// SPMV_SELLT_ROWS rows against one column tile of SPMV_SELLT_TILE_BYTES are
// each sorted and sliced like the sliced layout, by the rows' segment lengths
// in the tile.  srow[slab * R + i] is the
// block-local row at sorted position i of the slab; sslice[slab *
// SPMV_SLICES_PER_BLOCK + k] = (start relative to the slab's boff[slab],
// entries per lane); codes are tile-local (col - t * tile_cols); a pad takes
// the column of its slice's first entry (so it reads a staged element) and
// the value zero.  One workgroup per row block walks the tiles with its rows'
// FP64 sums in LDS, as the blocked product.

// Layout step 1: per (row block, tile), the row's entries in the tile; one
// thread per row (tiles in turn; columns ascending).
__global__ void __launch_bounds__(256)
k_sellt_count(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int64_t dim,
              int32_t nt, int32_t tc, int32_t R, uint16_t *__restrict__ cnt)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= dim)
        return;
    const int64_t b = r / R, i = r - b * R;
    int k = rowptr[r];
    const int k1 = rowptr[r + 1];
    for (int t = 0; t < nt; t++) {
        const int k2 = first_col_at_least(col, k, k1, (int64_t)(t + 1) * tc);
        cnt[(b * nt + t) * R + i] = (uint16_t)(k2 - k);
        k = k2;
    }
}

// Step 2: one workgroup per slab sorts the block's rows by their entries in
// the tile (longest first, ties by row; in place: the counts become the row
// order) and writes the slab's slices (start in the slab, length rounded up
// to E) and its total entries, and clears its part mask.
__global__ void __launch_bounds__(1024)
k_sellt_sort(int64_t dim, int32_t nt, int E, uint16_t *__restrict__ cnt_row,
             int2 *__restrict__ sslice, int64_t *__restrict__ stot, uint32_t *__restrict__ smask)
{
    constexpr int R = SPMV_SELLT_ROWS, RK = 2048;   // rows, keys (a power of two)
    static_assert(R <= RK && (RK + VQE_WAVE - 1) / VQE_WAVE <= SPMV_SLICES_PER_BLOCK, "block size");
    __shared__ uint32_t key[RK];
    const int tid = threadIdx.x;
    const int64_t slab = blockIdx.x;
    const int64_t r0 = (slab / nt) * R;
    const int n = (int)(dim - r0 < R ? dim - r0 : R);
    uint16_t *c = cnt_row + slab * R;
    for (int i = tid; i < RK; i += 1024)
        key[i] = i < n ? ((0xffffu - (uint32_t)c[i]) << 16) | (uint32_t)i : 0xffffffffu;
    __syncthreads();
    for (int k = 2; k <= RK; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < RK; i += 1024) {
                const int q = i ^ j;
                if (q > i) {
                    const uint32_t a = key[i], b = key[q];
                    if ((a > b) == ((i & k) == 0)) {
                        key[i] = b;
                        key[q] = a;
                    }
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < n; i += 1024)
        c[i] = (uint16_t)(key[i] & 0xffffu);
    if (tid == 0) {
        int at = 0;
        for (int k = 0; k < SPMV_SLICES_PER_BLOCK; k++) {
            int len = 0;
            if (k * VQE_WAVE < n) {
                len = (int)(0xffffu - (key[k * VQE_WAVE] >> 16));
                len = (len + E - 1) / E * E;
            }
            sslice[slab * SPMV_SLICES_PER_BLOCK + k] = make_int2(at, len);
            at += len * VQE_WAVE;
        }
        stot[slab] = at;
        smask[slab] = 0;     // the fill sets the parts the codes reach
    }
}

// Step 3: the slabs' starts (exclusive prefix of their totals) and the
// layout's total entries; one workgroup.
__global__ void __launch_bounds__(1024)
k_sellt_scan(const int64_t *__restrict__ stot, int64_t nslab, int64_t *__restrict__ sbase,
             int64_t *__restrict__ total)
{
    __shared__ int64_t part[1024];
    const int tid = threadIdx.x;
    const int64_t per = (nslab + 1023) / 1024;
    const int64_t lo = (int64_t)tid * per < nslab ? (int64_t)tid * per : nslab;
    const int64_t hi = lo + per < nslab ? lo + per : nslab;
    int64_t sum = 0;
    for (int64_t j = lo; j < hi; j++)
        sum += stot[j];
    part[tid] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t at = part[tid] - sum;
    for (int64_t j = lo; j < hi; j++) {
        sbase[j] = at;
        at += stot[j];
    }
    if (tid == 1023)
        *total = part[1023];
}

// Step 4: codes and values, one wave per slice (empty slices return), and
// the tile parts the slice's columns reach, ORed into its slab's mask.
template <int DT>
__global__ void __launch_bounds__(64)
k_sellt_fill(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
             const void *__restrict__ val, int64_t dim, int32_t nt, int32_t tc, int E,
             const uint16_t *__restrict__ srow, const int2 *__restrict__ sslice,
             const int64_t *__restrict__ sbase, uint16_t *__restrict__ code, void *__restrict__ sval,
             uint32_t *__restrict__ smask)
{
    using T = typename Elem<DT>::T;
    constexpr int R = SPMV_SELLT_ROWS;
    const int64_t q = blockIdx.x;
    const int2 sl = sslice[q];
    if (sl.y == 0)
        return;
    const int64_t slab = q / SPMV_SLICES_PER_BLOCK;
    const int k = (int)(q - slab * SPMV_SLICES_PER_BLOCK);
    const int64_t b = slab / nt;
    const int t = (int)(slab - b * nt);
    const int64_t r0 = b * R;
    const int n = (int)(dim - r0 < R ? dim - r0 : R);
    const int lane = threadIdx.x;
    const int i = k * VQE_WAVE + lane;
    const int64_t c_lo = (int64_t)t * tc;
    int k0 = 0, len = 0;
    if (i < n) {
        const int64_t row = r0 + srow[slab * R + i];
        const int a = rowptr[row], e = rowptr[row + 1];
        k0 = first_col_at_least(col, a, e, c_lo);
        len = first_col_at_least(col, k0, e, c_lo + tc) - k0;
    }
    T *out = reinterpret_cast<T *>(sval);
    const T *in = reinterpret_cast<const T *>(val);
    const int64_t base = sbase[slab] + sl.x;
    constexpr int PART = SPMV_SELLT_PART_BYTES / (int)sizeof(T);
    // the pads' column: the slice's first entry (lane 0 holds its longest row)
    const int cpad = __shfl(len > 0 ? col[k0] - (int)c_lo : 0, 0);
    uint32_t parts = 0;
    for (int j = 0; j < sl.y; j++) {
        const int64_t at = base + ((int64_t)(j / E) * VQE_WAVE + lane) * E + j % E;
        const int c = j < len ? col[k0 + j] - (int)c_lo : cpad;
        code[at] = (uint16_t)c;
        out[at] = j < len ? in[k0 + j] : T{};
        if (j < len)
            parts |= 1u << (c / PART);
    }
    for (int off = VQE_WAVE / 2; off > 0; off >>= 1)
        parts |= (uint32_t)__shfl_xor((int)parts, off);
    if (lane == 0 && parts)
        atomicOr(smask + slab, parts);
}

// The product: one workgroup per (state, row block); per tile with entries,
// the parts of the tile that the slab reaches staged in LDS, each wave takes
// two of the slab's slices, every lane sums its
// row's segment with D groups of E entries in flight and adds it to the row's
// FP64 sums in LDS (each row once per slab, tiles in ascending order).
template <int DT, int E, int D, bool PF>
__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_sellt(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 task = tasks[blockIdx.x];
    if (task.x < 0)
        return;
    const SpmvState st = states[task.x];
    if (VQE_SKIP(st))
        return;
    using T = typename Elem<DT>::T;
    constexpr int R = SPMV_SELLT_ROWS;
    extern __shared__ unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t dim = st.dim;
    const int tc = st.tile_cols, nt = st.ntiles;
    const int b = task.y;
    const int64_t r0 = (int64_t)b * R;
    const int n = (int)(dim - r0 < R ? dim - r0 : R);
    double2 *s_acc = reinterpret_cast<double2 *>(smem);
    T *s_x = reinterpret_cast<T *>(smem + (size_t)R * sizeof(double2));
    const T *__restrict__ psi = reinterpret_cast<const T *>(st.psi);
    const uint16_t *__restrict__ code = st.scode;
    const T *__restrict__ val = reinterpret_cast<const T *>(st.sval);
    for (int i = tid; i < n; i += 1024)
        s_acc[i] = make_double2(0.0, 0.0);
    constexpr int64_t STEP = (int64_t)VQE_WAVE * E;
    // A tile is loaded into registers (16 bytes per thread and part) and
    // written to LDS between the tiles' barriers, only the parts of the tile
    // that the slab's columns reach; with PF the next tile's loads are issued
    // while the current tile is multiplied.  A tile's bytes are a multiple of
    // 16 (dim and the tile width are even) and start 16-byte aligned.
    constexpr int SP = SPMV_SELLT_TILE_BYTES / SPMV_SELLT_PART_BYTES;
    static_assert(SPMV_SELLT_PART_BYTES == 16 * 1024 && SP <= 32, "a part is 16 bytes per thread");
    vqe_v4f pre[SP];
    auto fetch = [&](int t, uint32_t parts) {
        const int64_t c_lo = (int64_t)t * tc;
        const int64_t nbytes = (dim - c_lo < tc ? dim - c_lo : tc) * (int64_t)sizeof(T);
        const vqe_v4f *src = reinterpret_cast<const vqe_v4f *>(psi + c_lo);
#pragma unroll
        for (int u = 0; u < SP; u++) {
            const int c = tid + 1024 * u;
            if (((parts >> u) & 1u) && (int64_t)c * 16 < nbytes)
                pre[u] = gmem(src)[c];
        }
        return nbytes;
    };
    // the slabs' part masks, 64 tiles at a time one per lane, and the tiles
    // with entries in this block as a bit mask of that window
    int win = -1;
    uint32_t pv = 0u;
    uint64_t live = 0ull;
    auto load_window = [&](int w) {
        win = w;
        const int tl = w * 64 + lane;
        pv = tl < nt ? gmem(st.smask)[(int64_t)b * nt + tl] : 0u;
        live = __builtin_amdgcn_ballot_w64(pv != 0u);
    };
    // the first tile at or after t with entries in this block (nt: none)
    auto next_tile = [&](int t) {
        while (t < nt) {
            if ((t >> 6) != win)
                load_window(t >> 6);
            const uint64_t m = live & (~0ull << (t & 63));
            if (m)
                return win * 64 + (int)__builtin_ctzll(m);
            t = (win + 1) * 64;
        }
        return nt;
    };
    auto parts_at = [&](int t) {   // t in the current window
        return (uint32_t)__builtin_amdgcn_readlane((int)pv, t & 63);
    };
    // wave w takes slices w and 31 - w of each slab (longest with shortest:
    // the slices are sorted longest first)
    static_assert(SPMV_SLICES_PER_BLOCK == 32, "two slices per wave");
    const int ka = wid, kb = SPMV_SLICES_PER_BLOCK - 1 - wid;
    int t = next_tile(0);
    uint32_t parts = 0u;
    int64_t staged = 0;
    if (PF && t < nt) {
        parts = parts_at(t);
        staged = fetch(t, parts);
    }
    while (t < nt) {
        const int64_t slab = (int64_t)b * nt + t;
        const uint32_t here = PF ? parts : parts_at(t);
        if (!PF)
            staged = fetch(t, here);
        // the slab's tables, loaded before the barriers: its start, the two
        // slices and the rows their lanes take (clamped to the block)
        const sell_v2i *sls = reinterpret_cast<const sell_v2i *>(st.sslice) + slab * SPMV_SLICES_PER_BLOCK;
        const int64_t base = gmem(st.boff)[slab];
        const sell_v2i sl2[2] = {gmem(sls)[ka], gmem(sls)[kb]};
        const uint16_t *srow = st.srow + slab * R;
        const int ia = ka * VQE_WAVE + lane, ib = kb * VQE_WAVE + lane;
        const int rl2[2] = {gmem(srow)[ia < n ? ia : n - 1], gmem(srow)[ib < n ? ib : n - 1]};
        __syncthreads();      // every wave is done with the previous tile
#pragma unroll
        for (int u = 0; u < SP; u++) {
            const int c = tid + 1024 * u;
            if (((here >> u) & 1u) && (int64_t)c * 16 < staged)
                reinterpret_cast<vqe_v4f *>(s_x)[c] = pre[u];
        }
        __syncthreads();
        const int tn = next_tile(t + 1);
        if (PF && tn < nt) {
            parts = parts_at(tn);
            staged = fetch(tn, parts);
        }
        // the wave's two slices as one stream of groups (the first slice's,
        // then the second's), so that the second slice's first groups load
        // while the first one finishes; each slice sums into its own pair
        const int nga = __builtin_amdgcn_readfirstlane(sl2[0].y) / E;
        const int ngb = __builtin_amdgcn_readfirstlane(sl2[1].y) / E;
        if (nga > 0) {
            const int ng = nga + ngb;
            const int64_t ata = base + __builtin_amdgcn_readfirstlane(sl2[0].x) + lane * E;
            const int64_t atb = base + __builtin_amdgcn_readfirstlane(sl2[1].x) + lane * E - (int64_t)nga * STEP;
            // stream group p (clamped to the last) and its address
            auto addr = [&](int p) {
                const int pc = p < ng ? p : ng - 1;
                return (pc < nga ? ata : atb) + (int64_t)pc * STEP;
            };
            // one running sum; at the second slice's first group the first
            // slice's sum is set aside and the sum restarts
            double are = 0.0, aim = 0.0;
            double2 sa = make_double2(0.0, 0.0), sb;
            SellGroup<DT, E> g[D];
#pragma unroll
            for (int d = 0; d < D; d++)
                g[d].load(code, val, addr(d));
            int q = 0;
            for (; q + D <= ng; q += D) {
#pragma unroll
                for (int d = 0; d < D; d++) {
                    if (q + d == nga) {
                        sa = make_double2(are, aim);
                        are = aim = 0.0;
                    }
                    g[d].use(s_x, are, aim);
                    g[d].load(code, val, addr(q + D + d));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int d = 0; d < D; d++)
                if (q + d < ng) {
                    if (q + d == nga) {
                        sa = make_double2(are, aim);
                        are = aim = 0.0;
                    }
                    g[d].use(s_x, are, aim);
                }
            if (ngb == 0)
                sa = make_double2(are, aim);
            sb = make_double2(are, aim);
            if (ka * VQE_WAVE + lane < n) {
                double2 a = s_acc[rl2[0]];
                a.x += sa.x;
                a.y += sa.y;
                s_acc[rl2[0]] = a;
            }
            if (ngb > 0 && kb * VQE_WAVE + lane < n) {
                double2 a = s_acc[rl2[1]];
                a.x += sb.x;
                a.y += sb.y;
                s_acc[rl2[1]] = a;
            }
        }
        t = tn;
    }
    __syncthreads();
    double e_re = 0.0, e_im = 0.0, e_n2 = 0.0;
    for (int i = tid; i < n; i += 1024) {
        const double2 a = s_acc[i];
        Elem<DT>::st(st.sigma, r0 + i, a);
        energy_terms(ldg(psi, r0 + i), a.x, a.y, e_re, e_im, e_n2);
    }
    // the waves' energy sums in the tile's space (the tiles are done): the
    // rows' sums and one tile fill the LDS
    double (*s_part)[3] = reinterpret_cast<double (*)[3]>(s_x);
    e_re = wave_sum(e_re);
    e_im = wave_sum(e_im);
    e_n2 = wave_sum(e_n2);
    if (lane == 0) {
        s_part[wid][0] = e_re;
        s_part[wid][1] = e_im;
        s_part[wid][2] = e_n2;
    }
    __syncthreads();
    if (tid < 3) {
        double v = 0.0;
        for (int q = 0; q < 16; q++)
            v += s_part[q][tid];
        gmem(st.partials)[(int64_t)b * 3 + tid] = v;
    }
}

// ------------------------------------------------------------------ column-tiled with a dictionary
// VQE_SPMV_VDICT on a state larger than LDS.  Column row ^ x lies in the tile
// (row >> 14) ^ (x >> 14), so a block of rows meets in one tile only masks of
// one x >> 14: the tables of signed pairs are per x >> 14 (at most 1023 pairs
// each; 651 of 2052 at 18 qubits in the largest), staged beside the tile, and a
// code is a 16-bit byte offset into the tile's table.  A block's rows are
// sorted once, by codes and other entries over all tiles, so a lane keeps its
// rows' FP64 sums in registers over the tiles; per tile a slice is padded to
// its longest row, codes to groups of four, other entries to pairs (18 qubits:
// 1.33 times the entries).  About 3 instead of 10 bytes per entry: two 18-qubit
// states 431 us, bound by HBM -> 217 us, sixteen of 16 qubits 525 -> 230,
// one of 20 qubits 1388 -> 736; bound now by the two LDS gathers of a code (26
// clocks per CU for 64 codes; about 22 where the state fits LDS) and each tile's
// staging and barriers.  Loads in flight: with two groups of codes and one of
// the others no register spills (three groups of codes 233 us, one 260).

// Marks of the masks the operator uses, as k_sell_xmark, for up to 2^20 rows:
// the bitmap (dynamic LDS) gathers `rows` rows per workgroup.
__global__ void __launch_bounds__(1024)
k_vdt_mark(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int64_t dim, int rows,
           uint32_t *__restrict__ mark)
{
    extern __shared__ uint32_t s_mark[];
    const int tid = threadIdx.x, lane = tid & 63, words = (int)(dim / 32);
    for (int i = tid; i < words; i += 1024)
        s_mark[i] = 0u;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * rows;
    for (int64_t r = r0 + (tid >> 6); r < r0 + rows && r < dim; r += 16)
        for (int k = rowptr[r] + lane; k < rowptr[r + 1]; k += VQE_WAVE) {
            const uint32_t x = (uint32_t)col[k] ^ (uint32_t)r;
            if (!(s_mark[x >> 5] >> (x & 31u) & 1u))
                atomicOr(&s_mark[x >> 5], 1u << (x & 31u));
        }
    __syncthreads();
    for (int i = tid; i < words; i += 1024)
        if (s_mark[i])
            atomicOr(&mark[i], s_mark[i]);
}

// Numbers of the masks, ascending: xmap[x] (0xffff past the SPMV_VDT_MASKS
// first), xtab[number] = x and the count kept; one workgroup.
__global__ void __launch_bounds__(1024)
k_vdt_scan(const uint32_t *__restrict__ mark, int64_t dim, uint16_t *__restrict__ xmap,
           uint32_t *__restrict__ xtab, int64_t *__restrict__ nx)
{
    __shared__ int part[1024];
    const int tid = threadIdx.x, words = (int)(dim / 32), per = (words + 1023) / 1024;
    const int lo = min(tid * per, words), hi = min(lo + per, words);
    int c = 0;
    for (int i = lo; i < hi; i++)
        c += __popc(mark[i]);
    part[tid] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int at = part[tid] - c;
    for (int i = lo; i < hi; i++)
        for (uint32_t w = mark[i]; w; w &= w - 1, at++) {
            const uint32_t x = (uint32_t)i * 32u + (uint32_t)__builtin_ctz(w);
            xmap[x] = at < SPMV_VDT_MASKS ? (uint16_t)at : (uint16_t)0xffffu;
            if (at < SPMV_VDT_MASKS)
                xtab[at] = x;
        }
    if (tid == 1023)
        *nx = min(part[1023], SPMV_VDT_MASKS);
}

// k_vd_collect for up to SPMV_VDT_MASKS masks (dynamic LDS: slots, bad).
__global__ void __launch_bounds__(1024)
k_vdt_collect(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
              const float2 *__restrict__ val, int64_t dim, int rows, const uint16_t *__restrict__ xmap,
              uint32_t *__restrict__ slots, uint32_t *__restrict__ bad)
{
    extern __shared__ uint32_t s_slots[];
    uint32_t *s_bad = s_slots + SPMV_VDT_MASKS * SPMV_VD_VALS;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < SPMV_VDT_MASKS * SPMV_VD_VALS; i += 1024)
        s_slots[i] = SPMV_VD_EMPTY;
    for (int i = tid; i < SPMV_VDT_MASKS; i += 1024)
        s_bad[i] = 0u;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * rows;
    for (int64_t r = r0 + (tid >> 6); r < r0 + rows && r < dim; r += 16)
        for (int k = rowptr[r] + lane; k < rowptr[r + 1]; k += VQE_WAVE) {
            const int i = xmap[(uint32_t)col[k] ^ (uint32_t)r];
            const float2 v = val[k];
            if (i >= SPMV_VDT_MASKS || s_bad[i])
                continue;
            if (v.y != 0.f)
                s_bad[i] = 1u;
            else
                vd_insert(s_slots, s_bad, i, __float_as_uint(v.x) & 0x7fffffffu);
        }
    __syncthreads();
    for (int i = tid; i < SPMV_VDT_MASKS; i += 1024) {
        if (s_bad[i]) {
            bad[i] = 1u;
            continue;
        }
        for (int q = 0; q < SPMV_VD_VALS; q++)
            if (s_slots[i * SPMV_VD_VALS + q] != SPMV_VD_EMPTY)
                vd_insert(slots, bad, i, s_slots[i * SPMV_VD_VALS + q]);
    }
}

// Number the pairs of each table h = x >> 14 (masks and magnitudes ascending):
// pair[h * SPMV_VD_PAIRS + i], zeroed before, and each mask's first number in
// its table, SPMV_VD_NONE for a mask outside the dictionary.
__global__ void __launch_bounds__(1024)
k_vdt_number(const uint32_t *__restrict__ slots, const uint32_t *__restrict__ bad,
             const uint32_t *__restrict__ xtab, const int64_t *__restrict__ nx,
             uint2 *__restrict__ pair, uint16_t *__restrict__ base)
{
    constexpr int PER = SPMV_VDT_MASKS / 1024;
    __shared__ int pre[SPMV_VDT_MASKS + 1];
    __shared__ int part[1024];
    const int tid = threadIdx.x, n = (int)*nx;
    int c[PER], own = 0;
    for (int q = 0; q < PER; q++) {
        const int i = tid * PER + q;
        c[q] = 0;
        if (i < n && !bad[i])
            for (int u = 0; u < SPMV_VD_VALS; u++)
                c[q] += slots[i * SPMV_VD_VALS + u] != SPMV_VD_EMPTY;
        own += c[q];
    }
    part[tid] = own;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int t = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += t;
        __syncthreads();
    }
    int at = part[tid] - own;
    for (int q = 0; q < PER; q++) {
        pre[tid * PER + q] = at;
        at += c[q];
    }
    __syncthreads();
    for (int q = 0; q < PER; q++) {
        const int i = tid * PER + q;
        base[i] = (uint16_t)SPMV_VD_NONE;
        if (i >= n || c[q] == 0)
            continue;
        // the table's first mask
        const uint32_t h = xtab[i] >> SPMV_VDT_BITS;
        int lo = 0, hi = i;
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (xtab[mid] >> SPMV_VDT_BITS < h)
                lo = mid + 1;
            else
                hi = mid;
        }
        const int local = pre[i] - pre[lo];
        if (local + c[q] > SPMV_VD_PAIRS - 1)
            continue;
        base[i] = (uint16_t)local;
        // the magnitudes ascending (each one's rank among the mask's)
        for (int u = 0; u < SPMV_VD_VALS; u++) {
            const uint32_t v = slots[i * SPMV_VD_VALS + u];
            if (v == SPMV_VD_EMPTY)
                continue;
            int rank = 0;
            for (int w = 0; w < SPMV_VD_VALS; w++)
                rank += slots[i * SPMV_VD_VALS + w] < v;
            pair[(int64_t)h * SPMV_VD_PAIRS + local + rank] =
                make_uint2(v, (xtab[i] & (uint32_t)(SPMV_VDT_COLS - 1)) * (uint32_t)sizeof(float2));
        }
    }
}

// Per slice and tile the longest row's codes and other entries, rounded up to
// their groups: len[0 / 1][(b * nt + t) * SPMV_SLICES_PER_BLOCK + k], and the
// parts of each tile that the block reaches (smask, zeroed before).
__global__ void __launch_bounds__(256)
k_vdt_count(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int64_t dim, int32_t nt,
            const uint16_t *__restrict__ srow, const uint16_t *__restrict__ xmap,
            const uint16_t *__restrict__ base, int32_t *__restrict__ len, int64_t nlen,
            uint32_t *__restrict__ smask)
{
    __shared__ uint32_t s_max[2][SPMV_VDT_TILES], s_parts[SPMV_VDT_TILES], s_cnt[4][2][SPMV_VDT_TILES];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t b = blockIdx.x / SPMV_SLICES_PER_BLOCK;
    const int k = (int)(blockIdx.x % SPMV_SLICES_PER_BLOCK);
    if (tid < SPMV_VDT_TILES)
        s_max[0][tid] = s_max[1][tid] = s_parts[tid] = 0u;
    __syncthreads();
    for (int lr = wid; lr < VQE_WAVE; lr += 4) {
        const int64_t row = b * SPMV_SELLT_ROWS + srow[b * SPMV_SELLT_ROWS + k * VQE_WAVE + lr];
        // (the counts of one row change lanes within the wave, without a barrier)
        volatile uint32_t *cd = s_cnt[wid][0], *ce = s_cnt[wid][1];
        cd[lane] = ce[lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        for (int e = rowptr[row] + lane; e < rowptr[row + 1]; e += VQE_WAVE) {
            const uint32_t c = (uint32_t)col[e], t = c >> SPMV_VDT_BITS;
            const int m = xmap[c ^ (uint32_t)row];
            const bool d = m < SPMV_VDT_MASKS && base[m] != SPMV_VD_NONE;
            atomicAdd(&s_cnt[wid][d ? 0 : 1][t], 1u);
            atomicOr(&s_parts[t], 1u << ((c & (SPMV_VDT_COLS - 1)) / (SPMV_SELLT_PART_BYTES / (int)sizeof(float2))));
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < nt) {
            atomicMax(&s_max[0][lane], cd[lane]);
            atomicMax(&s_max[1][lane], ce[lane]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (tid < nt) {
        const int64_t at = (b * nt + tid) * SPMV_SLICES_PER_BLOCK + k;
        len[at] = (int32_t)(s_max[0][tid] + SPMV_VDT_GROUP - 1) / SPMV_VDT_GROUP * SPMV_VDT_GROUP;
        len[nlen + at] = (int32_t)(s_max[1][tid] + 1) / 2 * 2;
        if (s_parts[tid])
            atomicOr(&smask[b * nt + tid], s_parts[tid]);
    }
}

// A block's slices: starts relative to the block (tiles ascending) and its
// total entries; grid (blocks, 2 streams).
__global__ void __launch_bounds__(1024)
k_vdt_offsets(const int32_t *__restrict__ len, int64_t nlen, int32_t nt, int2 *__restrict__ slice,
              int64_t *__restrict__ total)
{
    __shared__ int part[1024];
    const int tid = threadIdx.x, n = nt * SPMV_SLICES_PER_BLOCK, per = (n + 1023) / 1024;
    const int64_t at0 = blockIdx.y * nlen + (int64_t)blockIdx.x * n;
    const int lo = min(tid * per, n), hi = min(lo + per, n);
    int c = 0;
    for (int i = lo; i < hi; i++)
        c += len[at0 + i];
    part[tid] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int at = part[tid] - c;
    for (int i = lo; i < hi; i++) {
        slice[at0 + i] = make_int2(at * VQE_WAVE, len[at0 + i]);
        at += len[at0 + i];
    }
    if (tid == 1023)
        total[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = (int64_t)part[1023] * VQE_WAVE;
}

// Both streams of one slice per workgroup, a row per wave in turn; within a
// tile a row's codes, and its other entries, go in column order.
template <bool RV>
__global__ void __launch_bounds__(1024)
k_vdt_fill(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
           const float2 *__restrict__ val, int32_t nt, const uint16_t *__restrict__ srow,
           const int2 *__restrict__ slice, int64_t nlen, const int64_t *__restrict__ dbase,
           const int64_t *__restrict__ ebase, const uint16_t *__restrict__ xmap,
           const uint16_t *__restrict__ base, const uint2 *__restrict__ pair, uint16_t *__restrict__ dcode,
           uint16_t *__restrict__ code, typename ValOf<VQE_C64, RV>::T *__restrict__ out)
{
    using V = typename ValOf<VQE_C64, RV>::T;
    __shared__ uint32_t s_cnt[16][2][SPMV_VDT_TILES];     // a row's entries of each tile so far
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t b = blockIdx.x / SPMV_SLICES_PER_BLOCK;
    const int k = (int)(blockIdx.x % SPMV_SLICES_PER_BLOCK);
    const int64_t d0 = dbase[b], e0 = ebase[b];
    for (int lr = wid; lr < VQE_WAVE; lr += 16) {
        const int64_t row = b * SPMV_SELLT_ROWS + srow[b * SPMV_SELLT_ROWS + k * VQE_WAVE + lr];
        volatile uint32_t *cd = s_cnt[wid][0], *ce = s_cnt[wid][1];
        cd[lane] = ce[lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        const int k1 = rowptr[row + 1];
        for (int kb = rowptr[row]; kb < k1; kb += VQE_WAVE) {
            const bool on = kb + lane < k1;
            uint32_t c = 0u, t = 0xffffffffu, m = 0xffffu;
            float2 v = make_float2(0.f, 0.f);
            bool d = false;
            if (on) {
                c = (uint32_t)col[kb + lane];
                v = val[kb + lane];
                t = c >> SPMV_VDT_BITS;
                m = xmap[c ^ (uint32_t)row];
                d = m < SPMV_VDT_MASKS && base[m] != SPMV_VD_NONE;
            }
            // columns ascend, so a tile's lanes are a run: each entry's place is
            // its rank in the run after what earlier passes held of the tile
            const uint64_t db = __ballot(on && d), eb = __ballot(on && !d);
            const uint32_t tp = (uint32_t)__shfl_up((int)t, 1, VQE_WAVE);
            const uint64_t heads = __ballot(lane == 0 || t != tp);
            const uint64_t upto = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1ull;
            const int h0 = 63 - __clzll((long long)(heads & upto));
            const uint64_t run = ((1ull << lane) - 1ull) & ~((1ull << h0) - 1ull);
            if (on) {
                const int64_t sl = (b * nt + t) * SPMV_SLICES_PER_BLOCK + k;
                if (d) {
                    const int j = (int)cd[t] + __popcll(db & run);
                    const uint2 *pr = pair + (int64_t)((c ^ (uint32_t)row) >> SPMV_VDT_BITS) * SPMV_VD_PAIRS;
                    const uint32_t bits = __float_as_uint(v.x) & 0x7fffffffu;
                    uint32_t p = base[m];
                    for (int q = 0; q < SPMV_VD_VALS - 1 && pr[p].x != bits; q++)
                        p++;
                    dcode[d0 + slice[sl].x + ((int64_t)(j / SPMV_VDT_GROUP) * VQE_WAVE + lr) * SPMV_VDT_GROUP + j % SPMV_VDT_GROUP] =
                        (uint16_t)((p << 1 | __float_as_uint(v.x) >> 31) << 3);
                } else {
                    const int j = (int)ce[t] + __popcll(eb & run);
                    const int64_t at = e0 + slice[nlen + sl].x + ((int64_t)(j / 2) * VQE_WAVE + lr) * 2 + j % 2;
                    code[at] = (uint16_t)(c & (SPMV_VDT_COLS - 1));
                    if constexpr (RV)
                        out[at] = v.x;
                    else
                        out[at] = v;
                }
            }
            __builtin_amdgcn_wave_barrier();
            // the run's last lane adds the run to the tile's counts
            const uint32_t tn = (uint32_t)__shfl_down((int)t, 1, VQE_WAVE);
            if (on && (lane == 63 || tn != t)) {
                const uint64_t all = upto & ~((1ull << h0) - 1ull);
                cd[t] += (uint32_t)__popcll(db & all);
                ce[t] += (uint32_t)__popcll(eb & all);
            }
            __builtin_amdgcn_wave_barrier();
        }
        __builtin_amdgcn_wave_barrier();
        // pads: the table's zero pair; column 0 with the value zero
        for (int t = 0; t < nt; t++) {
            const int64_t sl = (b * nt + t) * SPMV_SLICES_PER_BLOCK + k;
            const int2 ds = slice[sl], es = slice[nlen + sl];
            for (int j = (int)cd[t] + lane; j < ds.y; j += VQE_WAVE)
                dcode[d0 + ds.x + ((int64_t)(j / SPMV_VDT_GROUP) * VQE_WAVE + lr) * SPMV_VDT_GROUP + j % SPMV_VDT_GROUP] =
                    (uint16_t)(2 * (SPMV_VD_PAIRS - 1) << 3);
            for (int j = (int)ce[t] + lane; j < es.y; j += VQE_WAVE) {
                const int64_t at = e0 + es.x + ((int64_t)(j / 2) * VQE_WAVE + lr) * 2 + j % 2;
                code[at] = 0;
                out[at] = V{};
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

struct SellRows {      // what vd_finish needs of a wave's slices
    int64_t r0;
    int n, ns, ka, kb, ra, rb;
};

// The groups (N in flight, STEP entries apart) of a wave's two slices of one
// stream, A then B.
template <int GROUP, int N, typename G>
struct TwoSlices {
    static constexpr int STEP = VQE_WAVE * GROUP;
    int nga, ngb;
    int ata, atb;       // (uniform offsets into a block's entries)
    G g[N];
    __device__ __forceinline__ int at(int p) const
    {
        const int pc = p < nga + ngb ? p : nga + ngb - 1;
        return (pc < nga ? ata : atb) + pc * STEP;
    }
    // a, b: the slices' (start, length); load(at): the lane's group of a slice's
    // 64 at an offset
    template <typename Load>
    __device__ __forceinline__ void start(const sell_v2i a, const sell_v2i b, Load load)
    {
        nga = __builtin_amdgcn_readfirstlane(a.y) / GROUP;
        ngb = __builtin_amdgcn_readfirstlane(b.y) / GROUP;
        ata = __builtin_amdgcn_readfirstlane(a.x);
        atb = __builtin_amdgcn_readfirstlane(b.x) - nga * STEP;
        if (nga + ngb > 0)
#pragma unroll
            for (int d = 0; d < N; d++)
                g[d] = load(at(d));
    }
    // use(group, whether it is A's, the row's sum)
    template <typename Load, typename Use>
    __device__ __forceinline__ void run(Load load, Use use, double2 &sa, double2 &sb)
    {
        const int ng = nga + ngb;
        if (ng == 0)
            return;
        double2 s = nga > 0 ? sa : sb;
        for (int q = 0; q < ng; q += N)
#pragma unroll
            for (int d = 0; d < N; d++) {
                if (q + d < ng) {
                    if (q + d == nga && nga > 0) {
                        sa = s;
                        s = sb;
                    }
                    const G c = g[d];
                    g[d] = load(at(q + d + N));
                    use(c, q + d < nga, s);
                }
            }
        (ngb > 0 ? sb : sa) = s;
    }
};

__global__ void __launch_bounds__(1024) VQE_LDS_OCCUPANCY
k_spmv_sellt_vd(const SpmvState *__restrict__ states, const int2 *__restrict__ tasks)
{
    const int2 task = tasks[blockIdx.x];
    if (task.x < 0)
        return;
    const SpmvState st = states[task.x];
    if (VQE_SKIP(st))
        return;
    constexpr int R = SPMV_SELLT_ROWS, PARTS = R / SPMV_VD_PART_ROWS, SLICES = SPMV_VD_PART_ROWS / VQE_WAVE;
    extern __shared__ unsigned char smem[];
    float2 *s_x = reinterpret_cast<float2 *>(smem);
    float2 *s_sig = reinterpret_cast<float2 *>(smem + SPMV_SELLT_TILE_BYTES);   // the pairs until the end
    uint2 *s_pair = reinterpret_cast<uint2 *>(s_sig);
    static_assert(2 * SPMV_VD_PAIRS * sizeof(uint2) <= R * sizeof(float2), "pairs in the results' place");
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    // np parts of a block from p0 on, as k_spmv_sell
    const int np = task.y & 7, p0 = (task.y >> 3) % PARTS, b = (task.y >> 3) / PARTS;
    SellRows w;
    w.r0 = (int64_t)b * R;
    w.n = R;
    w.ns = SPMV_SLICES_PER_BLOCK;
    w.ka = np == PARTS ? wid : wid < np * SLICES ? p0 * SLICES + wid : SPMV_SLICES_PER_BLOCK;
    w.kb = np == PARTS ? wid + 16 : SPMV_SLICES_PER_BLOCK;
    const bool has_a = w.ka < SPMV_SLICES_PER_BLOCK, has_b = w.kb < SPMV_SLICES_PER_BLOCK;
    w.ra = gmem(st.srow)[w.r0 + (has_a ? w.ka * VQE_WAVE : 0) + lane];
    w.rb = gmem(st.srow)[w.r0 + (has_b ? w.kb * VQE_WAVE : 0) + lane];
    const uint32_t mask8 = (SPMV_VDT_COLS - 1) * 8u;
    const uint32_t ra8 = ((uint32_t)(w.r0 + w.ra) * 8u) & mask8, rb8 = ((uint32_t)(w.r0 + w.rb) * 8u) & mask8;
    const float2 *__restrict__ psi = reinterpret_cast<const float2 *>(st.psi);
    const int nt = st.ntiles;
    const sell_v2u *dcode = reinterpret_cast<const sell_v2u *>(reinterpret_cast<const uint16_t *>(st.dcode) + gmem(st.dboff)[b]);
    const int64_t e0 = gmem(st.boff)[b];
    // a pad reads a staged element or what the space held before: zeros at
    // first, then an earlier tile's elements
    constexpr int SP = SPMV_SELLT_TILE_BYTES / SPMV_SELLT_PART_BYTES;
#pragma unroll
    for (int u = 0; u < SP; u++)
        reinterpret_cast<vqe_v4f *>(s_x)[tid + 1024 * u] = vqe_v4f{0.f, 0.f, 0.f, 0.f};
    double2 sa = make_double2(0.0, 0.0), sb = sa;
    const int hb = (int)(w.r0 >> SPMV_VDT_BITS);
    // the tiles that the block reaches; a tile's slices are read one tile ahead
    // and its first codes with its elements
    const int mine = lane < nt ? (int)gmem(st.smask)[(int64_t)b * nt + lane] : 0;
    uint64_t left = __ballot(mine != 0);
    const sell_v2i none = {0, 0};
    sell_v2i da, db, ea, eb;
    auto slices = [&](int t) {
        const int64_t sl = ((int64_t)b * nt + t) * SPMV_SLICES_PER_BLOCK;
        const sell_v2i *dsl = reinterpret_cast<const sell_v2i *>(st.dslice) + sl;
        const sell_v2i *esl = reinterpret_cast<const sell_v2i *>(st.sslice) + sl;
        da = has_a ? gmem(dsl)[w.ka] : none;
        db = has_b ? gmem(dsl)[w.kb] : none;
        ea = has_a ? gmem(esl)[w.ka] : none;
        eb = has_b ? gmem(esl)[w.kb] : none;
    };
    if (left)
        slices(__builtin_ctzll(left));
    while (left) {
        const int t = __builtin_ctzll(left);
        left &= left - 1;
        const uint32_t parts = (uint32_t)__builtin_amdgcn_readlane(mine, t);
        const vqe_v4f *src = reinterpret_cast<const vqe_v4f *>(psi + (int64_t)t * SPMV_VDT_COLS);
        vqe_v4f pre[SP];
#pragma unroll
        for (int u = 0; u < SP; u++)
            if ((parts >> u) & 1u)
                pre[u] = gmem(src)[tid + 1024 * u];
        const sell_v2u pr = gmem(reinterpret_cast<const sell_v2u *>(st.dpair))[(int64_t)(hb ^ t) * SPMV_VD_PAIRS + tid];
        auto load_codes = [&](int at) { return gmem(dcode + at / SPMV_VDT_GROUP)[lane]; };
        TwoSlices<SPMV_VDT_GROUP, SPMV_VDT_DEPTH, sell_v2u> codes;
        codes.start(da, db, load_codes);
        __syncthreads();      // every wave is done with the previous tile
#pragma unroll
        for (int u = 0; u < SP; u++)
            if ((parts >> u) & 1u)
                reinterpret_cast<vqe_v4f *>(s_x)[tid + 1024 * u] = pre[u];
        s_pair[2 * tid] = make_uint2(pr.x, pr.y);
        s_pair[2 * tid + 1] = make_uint2(pr.x ^ 0x80000000u, pr.y);
        __syncthreads();
        auto run = [&](auto real) {
            using E = SellGroup<VQE_C64, 2, decltype(real)::value>;
            const uint16_t *code = st.scode + e0;
            const typename E::V *val = reinterpret_cast<const typename E::V *>(st.sval) + e0;
            auto load = [&](int at) {
                E g;
                g.load(code + at, val + at, lane * 2);
                return g;
            };
            TwoSlices<2, SPMV_VDT_ODEPTH, E> others;
            others.start(ea, eb, load);
            if (left)
                slices(__builtin_ctzll(left));
            codes.run(load_codes, [&](const sell_v2u c, bool first, double2 &s) {
                const uint32_t row8 = first ? ra8 : rb8;
                uint2 q[SPMV_VDT_GROUP];
#pragma unroll
                for (int u = 0; u < SPMV_VDT_GROUP; u++)
                    q[u] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const unsigned char *>(s_pair) +
                                                            (u & 1 ? c[u / 2] >> 16 : c[u / 2] & 0xffffu));
                float2 x[SPMV_VDT_GROUP];
#pragma unroll
                for (int u = 0; u < SPMV_VDT_GROUP; u++)
                    x[u] = *reinterpret_cast<const float2 *>(smem + (row8 ^ q[u].y));
#pragma unroll
                for (int u = 0; u < SPMV_VDT_GROUP; u++)
                    sell_fma(__uint_as_float(q[u].x), x[u], s.x, s.y);
            }, sa, sb);
            others.run(load, [&](const E &g, bool, double2 &s) { g.use(s_x, s.x, s.y); }, sa, sb);
        };
        if (st.rvals)
            run(std::true_type{});
        else
            run(std::false_type{});
    }
    __syncthreads();      // the results take the pairs' place
    vd_finish(st, b, p0, np, w, [&](int64_t r) { return ldg(psi, r); }, s_sig, sa, sb);
}

int32_t spmv_blk_tile_cols(int dtype) { return (int32_t)(SPMV_BLK_TILE_BYTES / vqe_elem_bytes(dtype)); }
int32_t spmv_sellt_tile_cols(int dtype) { return (int32_t)(SPMV_SELLT_TILE_BYTES / vqe_elem_bytes(dtype)); }

size_t spmv_blk_lds(int dtype)
{
    return (size_t)SPMV_BLK_ROWS * 2 * sizeof(double) +
           (size_t)(spmv_blk_tile_cols(dtype) + 1) * vqe_elem_bytes(dtype) +
           (size_t)(SPMV_BLK_ROWS + 1) * sizeof(int32_t);
}

// Blocked schedules: L lanes per row (4, 8, 16, 32 or 64); VQE_SPMV_X16 gives
// each lane two groups of four entries per pass instead of one; VQE_SPMV_DEEP
// keeps four rows per sub-group in flight instead of two (short segments carry
// few bytes per row, so narrow sub-groups need many rows in flight).
template <int DT, int L, int D, int U>
static void launch_blk_t(const SpmvState *states, const int2 *tasks, unsigned grid, hipStream_t s)
{
    const size_t lds = spmv_blk_lds(DT);
    auto k = k_spmv_blk<DT, L, D, U>;
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k<<<grid, 1024, lds, s>>>(states, tasks);
}

template <int DT, int L>
static void launch_blk_l(int sched, const SpmvState *states, const int2 *tasks, unsigned grid,
                         hipStream_t s)
{
    const bool deep = (sched & VQE_SPMV_DEEP) != 0, wide = (sched & VQE_SPMV_X16) != 0;
    if (deep)
        wide ? launch_blk_t<DT, L, 4, 2>(states, tasks, grid, s)
             : launch_blk_t<DT, L, 4, 1>(states, tasks, grid, s);
    else
        wide ? launch_blk_t<DT, L, 2, 2>(states, tasks, grid, s)
             : launch_blk_t<DT, L, 2, 1>(states, tasks, grid, s);
}

template <int DT>
static void launch_blk_dt(int sched, const SpmvState *states, const int2 *tasks, unsigned grid,
                          hipStream_t s)
{
    switch (sched & 0xff) {
    case 4: launch_blk_l<DT, 4>(sched, states, tasks, grid, s); break;
    case 8: launch_blk_l<DT, 8>(sched, states, tasks, grid, s); break;
    case 16: launch_blk_l<DT, 16>(sched, states, tasks, grid, s); break;
    case 64: launch_blk_l<DT, 64>(sched, states, tasks, grid, s); break;
    default: launch_blk_l<DT, 32>(sched, states, tasks, grid, s); break;
    }
}

// Sliced schedules of column-tiled states: E entries per lane and load group,
// D groups in flight (FP64 values: half as many, the registers).
template <int DT, int E, int D>
static void launch_sellt_t(const SpmvState *states, const int2 *tasks, unsigned grid, hipStream_t s,
                           bool pf)
{
    const size_t lds = (size_t)SPMV_SELLT_ROWS * sizeof(double2) +
                       (size_t)spmv_sellt_tile_cols(DT) * vqe_elem_bytes(DT);
    auto k = pf ? k_spmv_sellt<DT, E, D, true> : k_spmv_sellt<DT, E, D, false>;
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k<<<grid, 1024, lds, s>>>(states, tasks);
}

template <int DT>
static void launch_sellt_dt(int sched, const SpmvState *states, const int2 *tasks, unsigned grid,
                            hipStream_t s)
{
    constexpr bool W = DT == VQE_C128;
    // VQE_SPMV_DEEP: the next column tile's loads in flight during each tile
    const bool pf = (sched & VQE_SPMV_DEEP) != 0;
    switch (sched & 0xff) {
    case 2: launch_sellt_t<DT, 2, W ? 2 : 4>(states, tasks, grid, s, pf); break;
    case 8: launch_sellt_t<DT, 8, W ? 1 : 2>(states, tasks, grid, s, pf); break;
    default: launch_sellt_t<DT, 4, W ? 2 : 3>(states, tasks, grid, s, pf); break;
    }
}

void launch_spmv_blk(int dtype, int sched, const SpmvState *states, const int2 *tasks,
                     unsigned grid, hipStream_t s)
{
    if ((sched & VQE_SPMV_SLICED) && (sched & VQE_SPMV_VDICT)) {
        const size_t lds = SPMV_SELLT_TILE_BYTES + SPMV_SELLT_ROWS * sizeof(float2);
        auto k = k_spmv_sellt_vd;
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        k<<<grid, 1024, lds, s>>>(states, tasks);
        return;
    }
    if (sched & VQE_SPMV_SLICED) {
        if (dtype == VQE_C128)
            launch_sellt_dt<VQE_C128>(sched, states, tasks, grid, s);
        else
            launch_sellt_dt<VQE_C64>(sched, states, tasks, grid, s);
        return;
    }
    if (dtype == VQE_C128)
        launch_blk_dt<VQE_C128>(sched, states, tasks, grid, s);
    else
        launch_blk_dt<VQE_C64>(sched, states, tasks, grid, s);
}

namespace {
__global__ void __launch_bounds__(256) k_zero_i32(int32_t *__restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        p[i] = 0;
}
}  // namespace

void launch_blk_layout(const vqe_csr *H, int32_t nt, int32_t tc, int32_t R, int32_t *brp,
                       int64_t *blen, int64_t *boff, uint16_t *bcode, void *bval, hipStream_t s)
{
    const int64_t dim = H->dim;
    const int64_t nb = (dim + R - 1) / R;
    const int64_t nslab = nb * nt;
    const int64_t nrp = nslab * (R + 1);
    const unsigned zgrid = (unsigned)std::min<int64_t>((nrp + 255) / 256, 65536);
    k_zero_i32<<<zgrid, 256, 0, s>>>(brp, nrp);
    const unsigned g = (unsigned)((dim * nt + 255) / 256);
    k_blk_count<<<g, 256, 0, s>>>(H->rowptr, H->col, dim, nt, tc, R, brp);
    k_blk_scan<<<(unsigned)nslab, 256, 0, s>>>(brp, R, blen);
    k_blk_offsets<<<1, 1024, 0, s>>>(blen, nslab, boff);
    if (H->dtype == VQE_C128)
        k_blk_fill<VQE_C128><<<g, 256, 0, s>>>(H->rowptr, H->col, H->val, dim, nt, tc, R, brp, boff,
                                               bcode, bval);
    else
        k_blk_fill<VQE_C64><<<g, 256, 0, s>>>(H->rowptr, H->col, H->val, dim, nt, tc, R, brp, boff,
                                              bcode, bval);
}

void launch_sell_layout(const vqe_csr *H, int E, uint16_t *srow, int32_t *slen, int2 *sslice,
                        int64_t *total, hipStream_t s)
{
    const int64_t nb = (H->dim + SPMV_LDS_ROWS - 1) / SPMV_LDS_ROWS;
    k_sell_sort<<<(unsigned)nb, 1024, 0, s>>>(H->rowptr, H->dim, E, srow, slen);
    k_sell_scan<<<1, VQE_WAVE, 0, s>>>(slen, nb * SPMV_SLICES_PER_BLOCK, sslice, total);
}

static void fill32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s)
{
    k_sell_fill32<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p, n, v);
}

void launch_sell_xtab(const vqe_csr *H, uint32_t *mark, uint16_t *xmap, uint16_t *xtab, int64_t *nx,
                      hipStream_t s)
{
    const unsigned g = (unsigned)((H->dim + SELL_SCAN_ROWS - 1) / SELL_SCAN_ROWS);
    fill32(mark, (H->dim + 31) / 32, 0u, s);
    k_sell_xmark<<<g, 1024, 0, s>>>(H->rowptr, H->col, H->dim, mark);
    k_sell_xscan<<<1, 1024, 0, s>>>(mark, H->dim, xmap, xtab, nx);
}

void launch_vd_layout(const vqe_csr *H, int E, const uint16_t *xmap, const uint16_t *xtab,
                      const int64_t *nx, uint32_t *scratch, uint2 *pair, uint16_t *base,
                      uint16_t *srow, int32_t *slen, int2 *sslice, int64_t *total, hipStream_t s)
{
    const unsigned g = (unsigned)((H->dim + SELL_SCAN_ROWS - 1) / SELL_SCAN_ROWS);
    const int64_t nb = (H->dim + SPMV_LDS_ROWS - 1) / SPMV_LDS_ROWS, ns = nb * SPMV_SLICES_PER_BLOCK;
    uint32_t *slots = scratch, *bad = slots + SPMV_XIDX_MAX * SPMV_VD_VALS, *len = bad + SPMV_XIDX_MAX;
    fill32(slots, SPMV_XIDX_MAX * SPMV_VD_VALS, SPMV_VD_EMPTY, s);
    fill32(bad, SPMV_XIDX_MAX, 0u, s);
    k_vd_collect<<<g, 1024, 0, s>>>(H->rowptr, H->col, (const float2 *)H->val, H->dim, xmap, slots, bad);
    k_vd_number<<<1, 1024, 0, s>>>(slots, bad, xtab, nx, pair, base);
    k_vd_rows<SPMV_XIDX_MAX><<<g, 1024, 0, s>>>(H->rowptr, H->col, H->dim, xmap, base, len);
    k_vd_sort<<<(unsigned)nb, 1024, 0, s>>>(len, H->dim, E, srow, slen, ns);
    k_sell_scan<<<2, VQE_WAVE, 0, s>>>(slen, ns, sslice, total);
}

void launch_vd_fill(const vqe_csr *H, int E, bool real, const uint16_t *srow, const int2 *sslice,
                    const uint16_t *xmap, const uint16_t *base, const uint2 *pair, uint32_t *code,
                    void *val, uint32_t *dcode, hipStream_t s)
{
    const int64_t nb = (H->dim + SPMV_LDS_ROWS - 1) / SPMV_LDS_ROWS, ns = nb * SPMV_SLICES_PER_BLOCK;
    auto go = [&](auto k, auto *out) {
        k<<<(unsigned)ns, 1024, 0, s>>>(H->rowptr, H->col, (const float2 *)H->val, H->dim, srow, sslice, ns,
                                        xmap, base, pair, code, out, dcode);
    };
    if (real)
        E == 3 ? go(k_vd_fill<true, 3>, (float *)val) : go(k_vd_fill<true, 6>, (float *)val);
    else
        E == 3 ? go(k_vd_fill<false, 3>, (float2 *)val) : go(k_vd_fill<false, 6>, (float2 *)val);
}

template <int E>
static void launch_sell_fill_x_e(const vqe_csr *H, bool real, const uint16_t *srow, const int2 *sslice,
                                 const uint16_t *xmap, uint32_t *code, void *val, hipStream_t s)
{
    const int64_t nb = (H->dim + SPMV_LDS_ROWS - 1) / SPMV_LDS_ROWS;
    const unsigned g = (unsigned)(nb * SPMV_SLICES_PER_BLOCK);
    auto k = H->dtype == VQE_C128
                 ? (real ? k_sell_fill_x<VQE_C128, true, E> : k_sell_fill_x<VQE_C128, false, E>)
                 : (real ? k_sell_fill_x<VQE_C64, true, E> : k_sell_fill_x<VQE_C64, false, E>);
    k<<<g, 64, 0, s>>>(H->rowptr, H->col, H->val, H->dim, srow, sslice, xmap, code, val);
}

void launch_sell_fill_x(const vqe_csr *H, int E, bool real, const uint16_t *srow, const int2 *sslice,
                        const uint16_t *xmap, uint32_t *code, void *val, hipStream_t s)
{
    if (E == 3)
        launch_sell_fill_x_e<3>(H, real, srow, sslice, xmap, code, val, s);
    else
        launch_sell_fill_x_e<6>(H, real, srow, sslice, xmap, code, val, s);
}

void launch_vdt_layout(const vqe_csr *H, const VdTiled &v, hipStream_t s)
{
    const int64_t dim = H->dim, nb = dim / SPMV_SELLT_ROWS, nt = dim / SPMV_VDT_COLS;
    const int64_t nlen = nb * nt * SPMV_SLICES_PER_BLOCK;
    const unsigned gs = (unsigned)((dim + SELL_SCAN_ROWS - 1) / SELL_SCAN_ROWS);
    // the whole CSR is read by 512 workgroups, so that few LDS tables are merged
    const int rows = (int)((dim + 511) / 512);
    const unsigned g = (unsigned)((dim + rows - 1) / rows);
    const size_t mark_lds = (size_t)(dim / 32) * 4, set_lds = (size_t)SPMV_VDT_MASKS * (SPMV_VD_VALS + 1) * 4;
    uint32_t *slots = v.slots, *bad = slots + SPMV_VDT_MASKS * SPMV_VD_VALS;
    fill32(v.mark, dim / 32, 0u, s);
    fill32(slots, SPMV_VDT_MASKS * SPMV_VD_VALS, SPMV_VD_EMPTY, s);
    fill32(bad, SPMV_VDT_MASKS, 0u, s);
    fill32((uint32_t *)v.pair, nt * SPMV_VD_PAIRS * 2, 0u, s);
    fill32(v.smask, nb * nt, 0u, s);
    (void)hipFuncSetAttribute((const void *)k_vdt_mark, hipFuncAttributeMaxDynamicSharedMemorySize, (int)mark_lds);
    k_vdt_mark<<<g, 1024, mark_lds, s>>>(H->rowptr, H->col, dim, rows, v.mark);
    k_vdt_scan<<<1, 1024, 0, s>>>(v.mark, dim, v.xmap, v.xtab, v.total + 2);
    (void)hipFuncSetAttribute((const void *)k_vdt_collect, hipFuncAttributeMaxDynamicSharedMemorySize, (int)set_lds);
    k_vdt_collect<<<g, 1024, set_lds, s>>>(H->rowptr, H->col, (const float2 *)H->val, dim, rows, v.xmap, slots, bad);
    k_vdt_number<<<1, 1024, 0, s>>>(slots, bad, v.xtab, v.total + 2, v.pair, v.base);
    k_vd_rows<SPMV_VDT_MASKS><<<gs, 1024, 0, s>>>(H->rowptr, H->col, dim, v.xmap, v.base, v.rowlen);
    k_vd_sort<<<(unsigned)nb, 1024, 0, s>>>(v.rowlen, dim, 2, v.srow, v.len, nb * SPMV_SLICES_PER_BLOCK);
    k_vdt_count<<<(unsigned)(nb * SPMV_SLICES_PER_BLOCK), 256, 0, s>>>(H->rowptr, H->col, dim, (int32_t)nt, v.srow,
                                                                      v.xmap, v.base, v.len, nlen, v.smask);
    k_vdt_offsets<<<dim3((unsigned)nb, 2), 1024, 0, s>>>(v.len, nlen, (int32_t)nt, v.slice, v.btot);
    for (int q = 0; q < 2; q++)
        k_sellt_scan<<<1, 1024, 0, s>>>(v.btot + q * nb, nb, v.bbase + q * nb, v.total + q);
}

void launch_vdt_fill(const vqe_csr *H, const VdTiled &v, bool real, uint16_t *dcode, uint16_t *code, void *val,
                     hipStream_t s)
{
    const int64_t nb = H->dim / SPMV_SELLT_ROWS, nt = H->dim / SPMV_VDT_COLS;
    const int64_t nlen = nb * nt * SPMV_SLICES_PER_BLOCK;
    auto go = [&](auto k, auto *out) {
        k<<<(unsigned)(nb * SPMV_SLICES_PER_BLOCK), 1024, 0, s>>>(
            H->rowptr, H->col, (const float2 *)H->val, (int32_t)nt, v.srow, v.slice, nlen, v.bbase, v.bbase + nb,
            v.xmap, v.base, v.pair, dcode, code, out);
    };
    real ? go(k_vdt_fill<true>, (float *)val) : go(k_vdt_fill<false>, (float2 *)val);
}

void launch_sellt_layout(const vqe_csr *H, int32_t nt, int32_t tc, int E, uint16_t *srow,
                         int2 *sslice, int64_t *stot, int64_t *sbase, int64_t *total, uint32_t *smask,
                         hipStream_t s)
{
    const int64_t nb = (H->dim + SPMV_SELLT_ROWS - 1) / SPMV_SELLT_ROWS, nslab = nb * nt;
    k_sellt_count<<<(unsigned)((H->dim + 255) / 256), 256, 0, s>>>(H->rowptr, H->col, H->dim, nt, tc,
                                                                  SPMV_SELLT_ROWS, srow);
    k_sellt_sort<<<(unsigned)nslab, 1024, 0, s>>>(H->dim, nt, E, srow, sslice, stot, smask);
    k_sellt_scan<<<1, 1024, 0, s>>>(stot, nslab, sbase, total);
}

void launch_sellt_fill(const vqe_csr *H, int32_t nt, int32_t tc, int E, const uint16_t *srow,
                       const int2 *sslice, const int64_t *sbase, uint16_t *code, void *val,
                       uint32_t *smask, hipStream_t s)
{
    const int64_t nb = (H->dim + SPMV_SELLT_ROWS - 1) / SPMV_SELLT_ROWS;
    const unsigned g = (unsigned)(nb * nt * SPMV_SLICES_PER_BLOCK);
    if (H->dtype == VQE_C128)
        k_sellt_fill<VQE_C128><<<g, 64, 0, s>>>(H->rowptr, H->col, H->val, H->dim, nt, tc, E, srow,
                                                sslice, sbase, code, val, smask);
    else
        k_sellt_fill<VQE_C64><<<g, 64, 0, s>>>(H->rowptr, H->col, H->val, H->dim, nt, tc, E, srow,
                                               sslice, sbase, code, val, smask);
}

void launch_sell_fill(const vqe_csr *H, int E, bool real, const uint16_t *srow,
                      const int2 *sslice, uint16_t *code, void *val, hipStream_t s)
{
    const int64_t nb = (H->dim + SPMV_LDS_ROWS - 1) / SPMV_LDS_ROWS;
    const unsigned g = (unsigned)(nb * SPMV_SLICES_PER_BLOCK);
    auto k = H->dtype == VQE_C128 ? (real ? k_sell_fill<VQE_C128, true> : k_sell_fill<VQE_C128, false>)
                                  : (real ? k_sell_fill<VQE_C64, true> : k_sell_fill<VQE_C64, false>);
    k<<<g, 64, 0, s>>>(H->rowptr, H->col, H->val, H->dim, E, srow, sslice, code, val);
}

void launch_spmv(int dtype, int sched, const SpmvState &single, const SpmvState *states,
                 const int2 *tasks, unsigned grid, hipStream_t s, int64_t max_dim)
{
    const size_t lds = (size_t)(max_dim + 1) * vqe_elem_bytes(dtype) + (SPMV_LDS_ROWS + 1) * sizeof(int32_t);
    if (dtype == VQE_C128)
        launch_spmv_dt<VQE_C128>(sched, single, states, tasks, grid, s, lds);
    else
        launch_spmv_dt<VQE_C64>(sched, single, states, tasks, grid, s, lds);
}

int32_t spmv_tile_cols(int dtype) { return (int32_t)(SPMV_TILE_BYTES / vqe_elem_bytes(dtype)); }
int32_t spmv_tile_cols_real(int dtype) { return 2 * spmv_tile_cols(dtype); }

// Tile passes see short row segments, so narrow sub-groups keep two groups of
// four entries per lane (U = 2) instead of covering 256 entries per pass.
// The real-value form comes only with the 16-bit codes.
template <int DT, int L, int D>
static void launch_tiled_t(const SpmvState *states, const int2 *tasks, unsigned grid, hipStream_t s,
                           bool x16, bool rv)
{
    const size_t lds = (size_t)(spmv_tile_cols(DT) + 1) * vqe_elem_bytes(DT) +
                       2 * SPMV_LDS_ROWS * sizeof(int32_t);
    constexpr int U = L >= 32 ? 64 / L : 2;
    auto k = rv ? k_spmv_tiled<DT, L, D, U, true, true>
                : x16 ? k_spmv_tiled<DT, L, D, U, true, false> : k_spmv_tiled<DT, L, D, U, false, false>;
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k<<<grid, 1024, lds, s>>>(states, tasks);
}

template <int DT>
static void launch_tiled_dt(int sched, const SpmvState *states, const int2 *tasks, unsigned grid,
                            const int2 *sum_tasks, unsigned sum_grid, hipStream_t s)
{
    const bool deep = (sched & VQE_SPMV_DEEP) != 0;
    const bool x = (sched & VQE_SPMV_X16) != 0;
    const bool r = (sched & VQE_SPMV_REAL) != 0;
    switch (sched & 0xff) {
    case 8: deep ? launch_tiled_t<DT, 8, 3>(states, tasks, grid, s, x, r)
                 : launch_tiled_t<DT, 8, 2>(states, tasks, grid, s, x, r); break;
    case 16: deep ? launch_tiled_t<DT, 16, 3>(states, tasks, grid, s, x, r)
                  : launch_tiled_t<DT, 16, 2>(states, tasks, grid, s, x, r); break;
    case 64: deep ? launch_tiled_t<DT, 64, 3>(states, tasks, grid, s, x, r)
                  : launch_tiled_t<DT, 64, 2>(states, tasks, grid, s, x, r); break;
    default: deep ? launch_tiled_t<DT, 32, 3>(states, tasks, grid, s, x, r)
                  : launch_tiled_t<DT, 32, 2>(states, tasks, grid, s, x, r); break;
    }
    k_spmv_tile_sum<DT><<<sum_grid, 256, 0, s>>>(states, sum_tasks);
}

void launch_spmv_tiled(int dtype, int sched, const SpmvState *states, const int2 *tasks,
                       unsigned grid, const int2 *sum_tasks, unsigned sum_grid, hipStream_t s)
{
    if (dtype == VQE_C128)
        launch_tiled_dt<VQE_C128>(sched, states, tasks, grid, sum_tasks, sum_grid, s);
    else
        launch_tiled_dt<VQE_C64>(sched, states, tasks, grid, sum_tasks, sum_grid, s);
}

void launch_tile_bounds(const SpmvState *states, const int2 *tasks, unsigned grid, hipStream_t s)
{
    k_tile_bounds<<<grid, 256, 0, s>>>(states, tasks);
}

bool vqe_valid_schedule(int sched)
{
    switch (sched) {
    case 8: case 16: case 32: case 64:
    case 16 | VQE_SPMV_VEC4: case 32 | VQE_SPMV_VEC4: case 64 | VQE_SPMV_VEC4:
    case 8 | VQE_SPMV_LDS: case 16 | VQE_SPMV_LDS: case 32 | VQE_SPMV_LDS: case 64 | VQE_SPMV_LDS:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_DEEP: case 16 | VQE_SPMV_LDS | VQE_SPMV_DEEP:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_DEEP: case 64 | VQE_SPMV_LDS | VQE_SPMV_DEEP:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH: case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP:
    // 8 and 16 lanes: pipelined only in the column-tiled form (else plain LDS)
    case 8 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH: case 16 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH:
    case 16 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16:
    case 16 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16 | VQE_SPMV_REAL:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16 | VQE_SPMV_REAL:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16 | VQE_SPMV_REAL:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16 | VQE_SPMV_REAL:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16 | VQE_SPMV_REAL:
    // narrow pipelined schedules with the codes (plain LDS for states that
    // fit, with at least eight lanes; the blocked product's narrow forms for
    // larger states)
    case 4 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH:
    case 4 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP:
    case 4 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16:
    case 4 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16:
    case 16 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16:
    case 16 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16:
    case 16 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16 | VQE_SPMV_PAD:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16 | VQE_SPMV_PAD:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16 | VQE_SPMV_PAD:
    case 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16 | VQE_SPMV_PAD:
    case 64 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16 | VQE_SPMV_PAD:
    case 2 | VQE_SPMV_LDS | VQE_SPMV_SLICED:
    case 4 | VQE_SPMV_LDS | VQE_SPMV_SLICED:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_SLICED:
    case 2 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_DEEP:
    case 4 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_DEEP:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_DEEP:
    case 2 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_REAL:
    case 4 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_REAL:
    case 8 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_REAL:
    case 3 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX:
    case 3 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX | VQE_SPMV_REAL:
    case 6 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX:
    case 6 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX | VQE_SPMV_REAL:
    case 3 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX | VQE_SPMV_VDICT:
    case 3 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX | VQE_SPMV_VDICT | VQE_SPMV_REAL:
    case 6 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX | VQE_SPMV_VDICT:
    case 6 | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_XIDX | VQE_SPMV_VDICT | VQE_SPMV_REAL:
        return true;
    default:
        return false;
    }
}

// Wide loads need 16-byte aligned column and 32-byte aligned value arrays; the
// LDS schedule also needs the state to fit in LDS.  Otherwise the plain
// schedule with the same lanes is used.
int vqe_effective_schedule(const vqe_csr *H, int sched)
{
    // the sliced layout needs a state that fits LDS (with its 16-bit columns);
    // otherwise the 32-lane pipelined schedule with the codes stands in
    if (sched & VQE_SPMV_SLICED) {
        if (H->dim * (int64_t)vqe_elem_bytes(H->dtype) > SPMV_LDS_MAX_BYTES || H->dim >= 65536)
            return vqe_effective_schedule(H, 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_X16);
        // the index form stages its masks too (states of up to 128 KiB)
        if ((sched & VQE_SPMV_XIDX) &&
            (H->dim + 1) * (int64_t)vqe_elem_bytes(H->dtype) + SPMV_LDS_ROWS * (int64_t)sizeof(float2) +
                    SPMV_XIDX_MAX * (int64_t)sizeof(uint16_t) > 160 * 1024)
            sched = (sched & ~(VQE_SPMV_XIDX | 0xff)) | 4;
        // the dictionary comes with the index form, in FP32 storage
        if (!(sched & VQE_SPMV_XIDX) || H->dtype != VQE_C64)
            sched &= ~VQE_SPMV_VDICT;
        // the real values need an operator flagged real
        return sched & (VQE_SPMV_SLICED | VQE_SPMV_LDS | VQE_SPMV_XIDX | VQE_SPMV_VDICT | 0xff |
                        ((H->flags & VQE_REAL) ? VQE_SPMV_REAL : 0));
    }
    // four lanes per row exist only in the blocked product of states larger
    // than LDS; elsewhere the same schedule runs with eight
    if ((sched & 0xff) == 4)
        sched = (sched & ~0xff) | 8;
    // the real-value form needs an operator flagged real, and the codes
    if (!(H->flags & VQE_REAL))
        sched &= ~VQE_SPMV_REAL;
    const bool wide = (sched & (VQE_SPMV_VEC4 | VQE_SPMV_LDS)) != 0;
    if (wide && ((((uintptr_t)H->col) & 15) != 0 || (((uintptr_t)H->val) & 31) != 0))
        return sched & 0xff;
    if ((sched & VQE_SPMV_LDS) && H->dim * (int64_t)vqe_elem_bytes(H->dtype) > SPMV_LDS_MAX_BYTES)
        return (sched & 0xff) == 8 ? 16 | VQE_SPMV_VEC4 : (sched & 0xff) | VQE_SPMV_VEC4;
    // the pipelined schedule addresses the arrays with 31-bit buffer offsets,
    // and runs with 32 or 64 lanes when the state fits LDS
    if ((sched & VQE_SPMV_PREFETCH) &&
        (!(sched & VQE_SPMV_LDS) || H->nnz * (int64_t)vqe_elem_bytes(H->dtype) > 0x7fffff00LL ||
         (sched & 0xff) < ((sched & (VQE_SPMV_REAL | VQE_SPMV_PAD)) ? 16 : 32)))
        return sched & ~(VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16 | VQE_SPMV_REAL |
                         VQE_SPMV_PAD);
    // the 16-bit column form needs column XOR row below 2^16; the padded
    // layout comes with it; the real values imply the padded layout
    if ((sched & VQE_SPMV_X16) && H->dim > SPMV_X16_MAX_DIM)
        return sched & ~(VQE_SPMV_X16 | VQE_SPMV_REAL | VQE_SPMV_PAD);
    if (!(sched & VQE_SPMV_X16))
        sched &= ~VQE_SPMV_PAD;
    if (sched & VQE_SPMV_REAL)
        sched &= ~VQE_SPMV_PAD;
    return sched;
}

// In a batch plan, a pipelined LDS schedule on a state too large for LDS
// becomes the column-tiled schedule with the same lanes and depth.
int vqe_batch_schedule(const vqe_csr *H, int sched)
{
    const bool big = H->dim * (int64_t)vqe_elem_bytes(H->dtype) > SPMV_LDS_MAX_BYTES;
    // a sliced schedule runs a state larger than LDS in the slabs of the
    // blocked layout, each sorted and sliced
    if ((sched & VQE_SPMV_SLICED) && big) {
        // (the index form's states fit LDS; larger ones take two entries per
        // group, with the dictionary up to the rows its builder's bitmap holds:
        // faster at every size it takes, 16 to 20 qubits by 1.9 to 2.4 times)
        int vd = 0;
        if ((sched & VQE_SPMV_VDICT) && (sched & VQE_SPMV_XIDX) && H->dtype == VQE_C64 &&
            H->dim <= SPMV_VDT_MAX_DIM && (H->dim & (H->dim - 1)) == 0)
            vd = VQE_SPMV_VDICT;
        if (sched & VQE_SPMV_XIDX)
            sched = (sched & ~(VQE_SPMV_XIDX | 0xff)) | 2;
        return (sched & (0xff | VQE_SPMV_LDS | VQE_SPMV_SLICED | VQE_SPMV_DEEP)) | vd | VQE_SPMV_TILED |
               VQE_SPMV_BLOCKED;
    }
    const bool aligned = ((((uintptr_t)H->col) & 15) == 0) && ((((uintptr_t)H->val) & 31) == 0);
    if (big && (sched & VQE_SPMV_LDS) && (sched & VQE_SPMV_PREFETCH) && H->dim <= ((int64_t)1 << 30)) {
        // the real-value form keeps the column-tiled CSR (16-bit col ^ row
        // codes, real parts, per-tile row bounds) where it applies
        if ((sched & VQE_SPMV_REAL) && (sched & VQE_SPMV_X16) && (H->flags & VQE_REAL) && aligned &&
            H->dim <= SPMV_X16_MAX_DIM && H->nnz * (int64_t)vqe_elem_bytes(H->dtype) <= 0x7fffff00LL)
            return (sched & ~VQE_SPMV_PAD) | VQE_SPMV_TILED;
        // otherwise the blocked layout (complex values, tile-local codes;
        // VQE_SPMV_X16 and VQE_SPMV_DEEP select the pass width and depth)
        return (sched & (0xff | VQE_SPMV_LDS | VQE_SPMV_PREFETCH | VQE_SPMV_DEEP | VQE_SPMV_X16)) |
               VQE_SPMV_TILED | VQE_SPMV_BLOCKED;
    }
    return vqe_effective_schedule(H, sched);
}

void launch_val_real(const vqe_csr *H, void *out, hipStream_t s)
{
    const unsigned grid = (unsigned)((H->nnz + 255) / 256);
    if (grid == 0)
        return;
    if (H->dtype == VQE_C128)
        k_val_real<VQE_C128><<<grid, 256, 0, s>>>(H->val, out, H->nnz);
    else
        k_val_real<VQE_C64><<<grid, 256, 0, s>>>(H->val, out, H->nnz);
}

void launch_pad_layout(const vqe_csr *H, int32_t *prow, uint16_t *code, void *vpad, bool real,
                       hipStream_t s)
{
    k_pad_rowptr<<<1, 1024, 0, s>>>(H->rowptr, prow, H->dim);
    const unsigned grid = (unsigned)((H->dim + 3) / 4);
    if (H->dtype == VQE_C128) {
        if (real)
            k_pad_fill<VQE_C128, true><<<grid, 256, 0, s>>>(H->rowptr, H->col, H->val, prow, code, vpad, H->dim);
        else
            k_pad_fill<VQE_C128, false><<<grid, 256, 0, s>>>(H->rowptr, H->col, H->val, prow, code, vpad, H->dim);
    } else {
        if (real)
            k_pad_fill<VQE_C64, true><<<grid, 256, 0, s>>>(H->rowptr, H->col, H->val, prow, code, vpad, H->dim);
        else
            k_pad_fill<VQE_C64, false><<<grid, 256, 0, s>>>(H->rowptr, H->col, H->val, prow, code, vpad, H->dim);
    }
}

void launch_col_xor16(const vqe_csr *H, uint16_t *col16, hipStream_t s)
{
    const unsigned grid = (unsigned)((H->dim + 3) / 4);
    k_col_xor16<<<grid, 256, 0, s>>>(H->rowptr, H->col, col16, H->dim);
}

int64_t spmv_blocks(int64_t dim, int sched)
{
    const int64_t rpb = (sched & VQE_SPMV_VDICT) ? SPMV_VD_PART_ROWS
                        : (sched & VQE_SPMV_LDS) ? SPMV_LDS_ROWS
                                                 : spmv_rows_per_block(sched);
    return (dim + rpb - 1) / rpb;
}

extern "C" int32_t vqe_default_schedule(const vqe_csr *H)
{
    if (!H || H->dim <= 0)
        return 32;
    const double avg = (double)H->nnz / (double)H->dim;
    // Long rows: sixteen lanes of four entries (two passes and more of a row, few
    // idle lanes in the last) where their blocks of 32 rows give every CU two,
    // from 2^14 rows on (14 and 16 qubits of molecules, FP64, 22.8 and 140 us
    // against 30.2 and 186 with 64 lanes), or one with rows of a few passes (13
    // qubits, 192 entries a row 13 against 17 us, 256 level, 512 35 against 27).
    // Fewer rows leave CUs idle and each lane a long chain: 64 lanes (FP64, 10
    // qubits of 512 entries a row 9 against 19 us, 12 of 2048 44 against 80).
    if (avg >= 96.0)
        return H->dim >= 16384 || (H->dim >= 8192 && avg < 256.0) ? 16 | VQE_SPMV_VEC4 : 64 | VQE_SPMV_VEC4;
    if (avg >= 40.0)
        return 32;
    if (avg >= 12.0)
        return 16;
    return 8;
}

int check_csr(vqe_ctx *ctx, const vqe_csr *M, const char *what)
{
    if (!M)
        return vqe_fail(ctx, VQE_EINVAL, "%s: null operator", what);
    if (M->n_qubits < 1 || M->n_qubits > 30 || M->dim != ((int64_t)1 << M->n_qubits))
        return vqe_fail(ctx, VQE_EINVAL, "%s: bad operator size", what);
    if (M->dtype != VQE_C128 && M->dtype != VQE_C64)
        return vqe_fail(ctx, VQE_EINVAL, "%s: bad operator dtype", what);
    if (!M->rowptr || (M->nnz > 0 && (!M->col || !M->val)))
        return vqe_fail(ctx, VQE_EINVAL, "%s: operator arrays not set", what);
    if (M->nnz < 0 || M->nnz > 0x7fffffff)
        return vqe_fail(ctx, VQE_ESIZE, "%s: bad nnz", what);
    return VQE_OK;
}

int vqe_spmv_energy_core(vqe_ctx *ctx, const vqe_csr *H, const void *psi, void *sigma,
                         double *out, int lanes, double *partials)
{
    const int64_t dim = H->dim;
    if (lanes & VQE_SPMV_SLICED)   // batch plans only
        lanes = 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH;
    lanes = vqe_effective_schedule(H, lanes);
    const int64_t nblk = spmv_blocks(dim, lanes);
    SpmvState st{};
    st.rowptr = H->rowptr;
    st.col = H->col;
    st.val = H->val;
    st.psi = psi;
    st.sigma = sigma;
    st.partials = partials;
    st.energy_out = out;
    st.dim = dim;
    st.shift = H->diag_shift;
    st.nblocks = (int32_t)nblk;
    st.lanes = lanes;
    st.nnz = H->nnz;
    if (dim <= SPMV_SMALL_DIM && H->nnz <= SPMV_SMALL_NNZ &&
        (lanes == 8 || lanes == 16 || lanes == 32 || lanes == 64)) {
        auto pick = [&](auto k8, auto k16, auto k32, auto k64) {
            return lanes == 8 ? k8 : lanes == 16 ? k16 : lanes == 32 ? k32 : k64;
        };
        auto k = H->dtype == VQE_C128
                     ? pick(k_spmv_energy_small<VQE_C128, 8>, k_spmv_energy_small<VQE_C128, 16>,
                            k_spmv_energy_small<VQE_C128, 32>, k_spmv_energy_small<VQE_C128, 64>)
                     : pick(k_spmv_energy_small<VQE_C64, 8>, k_spmv_energy_small<VQE_C64, 16>,
                            k_spmv_energy_small<VQE_C64, 32>, k_spmv_energy_small<VQE_C64, 64>);
        k<<<1, 1024, 0, ctx->stream>>>(st);
        VQE_LAUNCH_CHECK(ctx);
        return VQE_OK;
    }
    launch_spmv(H->dtype, lanes, st, nullptr, nullptr, (unsigned)nblk, ctx->stream, dim);
    k_energy_finalize<<<1, 192, 0, ctx->stream>>>(st);
    VQE_LAUNCH_CHECK(ctx);
    return VQE_OK;
}

size_t vqe_spmv_partials_bytes(int64_t dim, int lanes)
{
    // the larger of the two block counts, so any schedule fits
    const int64_t a = spmv_blocks(dim, lanes & 0xff), b = spmv_blocks(dim, lanes);
    return vqe_align((size_t)(a > b ? a : b) * 3 * sizeof(double));
}

int vqe_spmv_energy_launch(vqe_ctx *ctx, const vqe_csr *H, const void *psi, void *sigma,
                           double *out, int lanes)
{
    const size_t o_sigma = vqe_spmv_partials_bytes(H->dim, lanes);
    size_t need = o_sigma;
    if (!sigma)
        need += vqe_align(H->dim * vqe_elem_bytes(H->dtype));
    int rc = vqe_ws_reserve(ctx, need);
    if (rc)
        return rc;
    void *sg = sigma ? sigma : (char *)ctx->ws + o_sigma;
    return vqe_spmv_energy_core(ctx, H, psi, sg, out, lanes, (double *)ctx->ws);
}

extern "C" int energy(vqe_ctx *ctx, const vqe_csr *H, const void *psi, void *sigma_out,
                      double *out)
{
    if (!ctx)
        return VQE_EINVAL;
    int rc = check_csr(ctx, H, "energy");
    if (rc)
        return rc;
    if (!psi || !out)
        return vqe_fail(ctx, VQE_EINVAL, "energy: null psi or out");
    return vqe_spmv_energy_launch(ctx, H, psi, sigma_out, out, vqe_default_schedule(H));
}

extern "C" int energy_noalloc(vqe_ctx *ctx, const vqe_csr *H, const void *psi, void *sigma_out,
                              double *out)
{
    if (!ctx)
        return VQE_EINVAL;
    int rc = check_csr(ctx, H, "energy_noalloc");
    if (rc)
        return rc;
    if (!psi || !sigma_out || !out)
        return vqe_fail(ctx, VQE_EINVAL, "energy_noalloc: null psi, sigma_out or out");
    const int lanes = vqe_default_schedule(H);
    const size_t need = vqe_spmv_partials_bytes(H->dim, lanes);
    if (need > VQE_NOALLOC_SCRATCH_BYTES)
        return vqe_fail(ctx, VQE_ESIZE,
                        "energy_noalloc: the reduction of a %lld-row operator needs %zu bytes of "
                        "partial sums, more than the %u-byte scratch array",
                        (long long)H->dim, need, (unsigned)VQE_NOALLOC_SCRATCH_BYTES);
    if (!ctx->scratch)
        return vqe_fail(ctx, VQE_EHIP, "energy_noalloc: the scratch array's device address is "
                                       "unknown (%s)", ctx->err);
    return vqe_spmv_energy_core(ctx, H, psi, sigma_out, out, lanes, ctx->scratch);
}

extern "C" int vqe_time_spmv(vqe_ctx *ctx, const vqe_csr *H, const void *psi, void *sigma,
                             int32_t schedule, int32_t reps, float *ms_out)
{
    if (!ctx)
        return VQE_EINVAL;
    int rc = check_csr(ctx, H, "vqe_time_spmv");
    if (rc)
        return rc;
    if (!psi || !sigma || !ms_out || reps < 1)
        return vqe_fail(ctx, VQE_EINVAL, "vqe_time_spmv: bad arguments");
    if (!vqe_valid_schedule(schedule))
        return vqe_fail(ctx, VQE_EINVAL, "vqe_time_spmv: unknown schedule %d", schedule);
    // a single call has no 16-bit column codes, real values or sliced layout:
    // the same schedule without them (the 32-lane pipelined one for a sliced)
    const int lanes = (schedule & VQE_SPMV_SLICED) ? 32 | VQE_SPMV_LDS | VQE_SPMV_PREFETCH
                                                   : schedule & ~(VQE_SPMV_X16 | VQE_SPMV_REAL);
    // energy result goes after the partials in the workspace
    const size_t o_out = vqe_spmv_partials_bytes(H->dim, lanes);
    rc = vqe_ws_reserve(ctx, o_out + 256);
    if (rc)
        return rc;
    double *out = (double *)((char *)ctx->ws + o_out);
    hipEvent_t e0, e1;
    VQE_HIP(ctx, hipEventCreate(&e0));
    VQE_HIP(ctx, hipEventCreate(&e1));
    double *part = (double *)ctx->ws;
    rc = vqe_spmv_energy_core(ctx, H, psi, sigma, out, lanes, part);   // warm-up
    if (rc)
        return rc;
    VQE_HIP(ctx, hipEventRecord(e0, ctx->stream));
    for (int i = 0; i < reps && rc == VQE_OK; i++)
        rc = vqe_spmv_energy_core(ctx, H, psi, sigma, out, lanes, part);
    VQE_HIP(ctx, hipEventRecord(e1, ctx->stream));
    VQE_HIP(ctx, hipEventSynchronize(e1));
    float ms = 0.f;
    VQE_HIP(ctx, hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *ms_out = ms / (float)reps;
    return rc;
}
