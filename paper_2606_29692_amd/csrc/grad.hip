// Pool-gradient screen (Eq. 5) and the selection of Sec. III-D.
//
// g_j = <psi|[H, A_j]|psi> = 2 Re sum_r conj(sigma_r) (A_j psi)_r for
// anti-Hermitian A_j and Hermitian H, with sigma = H psi computed once by the
// energy kernel and shared by every generator.  A workgroup takes one
// generator and GRAD_ROWS rows per thread of it; psi and sigma are gathered
// from L2, and a second launch adds a generator's partial sums (FP64, fixed
// order: a thread's rows ascending, the workgroup's waves, then the chunks).
// What bounds it is the chain of dependent reads of a pair (row pointer,
// column, the partner's row pointer, values and amplitudes), so a thread's
// rows go through it together.  14 qubits, 204 generators, FP64: 25.6 us one
// row at a time -> 21.6 us; a workgroup for a whole generator, with no
// second launch, 43.9 us.
#include "kernels.hpp"

namespace {

constexpr int GRAD_ROWS = 4, GRAD_THREADS = 256, GRAD_CHUNK = GRAD_ROWS * GRAD_THREADS;

template <int DT>
__global__ void __launch_bounds__(GRAD_THREADS)
k_pool_grad(const vqe_csr *__restrict__ ops, const void *__restrict__ psi,
            const void *__restrict__ sigma, double shift, int64_t dim, double *__restrict__ partials,
            double *__restrict__ g_out)
{
    constexpr int nt = GRAD_THREADS;
    const int j = blockIdx.y;
    const int64_t r0 = (int64_t)blockIdx.x * GRAD_CHUNK + threadIdx.x;
    const vqe_csr op = ops[j];
    const VQE_GLOBAL int32_t *rowptr = gmem((const int32_t *)op.rowptr);
    const VQE_GLOBAL int32_t *col = gmem((const int32_t *)op.col);
    double acc = 0.0;
    if (op.flags & VQE_PAIRING) {
        // pair {r, c} with A[r,c] = a, A[c,r] = b, handled by its lower row:
        // conj(sigma_r) a psi_c + conj(sigma_c) b psi_r
        int k0[GRAD_ROWS], c[GRAD_ROWS], kb[GRAD_ROWS];
        bool on[GRAD_ROWS];
#pragma unroll
        for (int u = 0; u < GRAD_ROWS; u++) {
            const int64_t r = r0 + (int64_t)u * nt;
            on[u] = false;
            k0[u] = 0;
            if (r < dim) {
                k0[u] = rowptr[r];
                on[u] = rowptr[r + 1] != k0[u];
            }
        }
#pragma unroll
        for (int u = 0; u < GRAD_ROWS; u++)
            c[u] = on[u] ? col[k0[u]] : 0;
#pragma unroll
        for (int u = 0; u < GRAD_ROWS; u++) {
            on[u] = on[u] && c[u] >= r0 + (int64_t)u * nt;
            kb[u] = on[u] ? rowptr[c[u]] : 0;
        }
        double2 a[GRAD_ROWS], b[GRAD_ROWS], pr[GRAD_ROWS], pc[GRAD_ROWS], qr[GRAD_ROWS], qc[GRAD_ROWS];
#pragma unroll
        for (int u = 0; u < GRAD_ROWS; u++)
            if (on[u]) {
                const int64_t r = r0 + (int64_t)u * nt;
                a[u] = Elem<DT>::ld(op.val, k0[u]);
                b[u] = c[u] == r ? make_double2(0.0, 0.0) : Elem<DT>::ld(op.val, kb[u]);
                pr[u] = Elem<DT>::ld(psi, r);
                pc[u] = Elem<DT>::ld(psi, c[u]);
                qr[u] = Elem<DT>::ld(sigma, r);
                qc[u] = Elem<DT>::ld(sigma, c[u]);
            }
#pragma unroll
        for (int u = 0; u < GRAD_ROWS; u++)
            if (on[u]) {
                const double sr_x = qr[u].x + shift * pr[u].x, sr_y = qr[u].y + shift * pr[u].y;
                const double sc_x = qc[u].x + shift * pc[u].x, sc_y = qc[u].y + shift * pc[u].y;
                const double wr = a[u].x * pc[u].x - a[u].y * pc[u].y;
                const double wi = a[u].x * pc[u].y + a[u].y * pc[u].x;
                const double ur = b[u].x * pr[u].x - b[u].y * pr[u].y;
                const double ui = b[u].x * pr[u].y + b[u].y * pr[u].x;
                acc += (sr_x * wr + sr_y * wi) + (sc_x * ur + sc_y * ui);
            }
    } else {
        for (int64_t r = r0; r < dim && r < r0 + GRAD_CHUNK; r += nt) {
            const int k0 = rowptr[r], k1 = rowptr[r + 1];
            if (k0 == k1)
                continue;
            const double2 q = Elem<DT>::ld(sigma, r), p = Elem<DT>::ld(psi, r);
            const double sx = q.x + shift * p.x, sy = q.y + shift * p.y;
            for (int k = k0; k < k1; k++) {
                const double2 a = Elem<DT>::ld(op.val, k), x = Elem<DT>::ld(psi, col[k]);
                acc += sx * (a.x * x.x - a.y * x.y) + sy * (a.x * x.y + a.y * x.x);
            }
        }
    }
    __shared__ double s_red[GRAD_THREADS / VQE_WAVE];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0)
        s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double v = ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];
        if (gridDim.x == 1)
            g_out[j] = 2.0 * v;      // the only chunk: no second launch
        else
            partials[(int64_t)j * gridDim.x + blockIdx.x] = v;
    }
}

// g_j from its chunks' sums, one thread per generator.
__global__ void __launch_bounds__(64)
k_grad_fin(const double *__restrict__ partials, int M, int nchunks, double *__restrict__ g)
{
    const int j = (int)(blockIdx.x * 64 + threadIdx.x);
    if (j >= M)
        return;
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < nchunks; c++)
        s += partials[(int64_t)j * nchunks + c];
    g[j] = 2.0 * s;
}

template <bool BATCH>
__global__ void __launch_bounds__(64)
k_select_t(SelectState single, const SelectState *__restrict__ states, double rel_tie)
{
    const SelectState st = BATCH ? states[blockIdx.x] : single;
    if (VQE_SKIP(st))
        return;
    const int lane = threadIdx.x;
    double gmax = 0.0;
    for (int j = lane; j < st.M; j += 64)
        gmax = fmax(gmax, fabs(st.g[j]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        gmax = fmax(gmax, __shfl_xor(gmax, o, 64));
    const double thr = gmax * (1.0 - rel_tie);
    int best = 0x7fffffff;
    for (int j = lane; j < st.M; j += 64)
        if (fabs(st.g[j]) >= thr && j < best)
            best = j;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        best = min(best, __shfl_xor(best, o, 64));
    if (lane == 0) {
        st.k_out[0] = best == 0x7fffffff ? 0 : best;
        st.gmax_out[0] = gmax;
    }
}

}  // namespace

static int check_pool(vqe_ctx *ctx, const vqe_pool *pool, const vqe_csr *H)
{
    if (!pool || pool->M < 0 || (pool->M > 0 && (!pool->ops || !pool->ops_host)))
        return vqe_fail(ctx, VQE_EINVAL, "pool_gradients: bad pool");
    if (pool->n_qubits != H->n_qubits || pool->dtype != H->dtype)
        return vqe_fail(ctx, VQE_EINVAL, "pool_gradients: pool and H differ in size or dtype");
    for (int j = 0; j < pool->M; j++) {
        const vqe_csr &o = pool->ops_host[j];
        if (o.dim != H->dim || o.dtype != H->dtype || !o.rowptr || (o.nnz > 0 && (!o.col || !o.val)))
            return vqe_fail(ctx, VQE_EINVAL, "pool_gradients: generator %d does not match H", j);
    }
    return VQE_OK;
}

int vqe_pool_grad_launch(vqe_ctx *ctx, const vqe_csr *H, const vqe_pool *pool, const void *psi,
                         const void *sigma, double *g_out)
{
    const int64_t dim = H->dim;
    const int M = pool->M;
    if (M == 0)
        return VQE_OK;
    const int nchunks = (int)((dim + GRAD_CHUNK - 1) / GRAD_CHUNK);
    // workspace: [gradient partials][product partials][sigma][energy]
    const int lanes = vqe_effective_schedule(H, vqe_default_schedule(H));
    const size_t o_sp = vqe_align((size_t)M * nchunks * sizeof(double));
    const size_t o_sigma = o_sp + vqe_spmv_partials_bytes(dim, lanes);
    const size_t o_e = o_sigma + vqe_align(dim * vqe_elem_bytes(H->dtype));
    int rc = vqe_ws_reserve(ctx, sigma ? o_sp : o_e + 256);
    if (rc)
        return rc;
    char *ws = (char *)ctx->ws;
    if (!sigma) {
        rc = vqe_spmv_energy_core(ctx, H, psi, ws + o_sigma, (double *)(ws + o_e), lanes,
                                  (double *)(ws + o_sp));
        if (rc)
            return rc;
        sigma = ws + o_sigma;
    }
    auto k = H->dtype == VQE_C128 ? k_pool_grad<VQE_C128> : k_pool_grad<VQE_C64>;
    // (at most 65535 generators to a launch's second grid dimension)
    for (int j0 = 0; j0 < M; j0 += 65535) {
        const int m = M - j0 < 65535 ? M - j0 : 65535;
        k<<<dim3((unsigned)nchunks, (unsigned)m), GRAD_THREADS, 0, ctx->stream>>>(
            pool->ops + j0, psi, sigma, H->diag_shift, dim, (double *)ws + (size_t)j0 * nchunks,
            g_out + j0);
    }
    if (nchunks > 1)
        k_grad_fin<<<(unsigned)((M + 63) / 64), 64, 0, ctx->stream>>>((const double *)ws, M, nchunks, g_out);
    VQE_LAUNCH_CHECK(ctx);
    return VQE_OK;
}

extern "C" int pool_gradients(vqe_ctx *ctx, const vqe_csr *H, const vqe_pool *pool,
                              const void *psi, const void *sigma, double *g_out)
{
    if (!ctx)
        return VQE_EINVAL;
    int rc = check_csr(ctx, H, "pool_gradients");
    if (rc)
        return rc;
    rc = check_pool(ctx, pool, H);
    if (rc)
        return rc;
    if (!psi || (!g_out && pool->M > 0))
        return vqe_fail(ctx, VQE_EINVAL, "pool_gradients: null psi or g_out");
    return vqe_pool_grad_launch(ctx, H, pool, psi, sigma, g_out);
}

int vqe_select_launch(vqe_ctx *ctx, int32_t M, const double *g, double rel_tie, int32_t *k_out,
                      double *gmax_out)
{
    SelectState st{g, M, k_out, gmax_out};
    k_select_t<false><<<1, 64, 0, ctx->stream>>>(st, nullptr, rel_tie);
    VQE_LAUNCH_CHECK(ctx);
    return VQE_OK;
}

extern "C" int vqe_select(vqe_ctx *ctx, int32_t M, const double *g, double rel_tie,
                          int32_t *k_out, double *gmax_out)
{
    if (!ctx)
        return VQE_EINVAL;
    if (M < 1 || !g || !k_out || !gmax_out || !(rel_tie >= 0.0 && rel_tie < 1.0))
        return vqe_fail(ctx, VQE_EINVAL, "vqe_select: bad arguments");
    return vqe_select_launch(ctx, M, g, rel_tie, k_out, gmax_out);
}
