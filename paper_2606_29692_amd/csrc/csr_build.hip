// Pauli sum -> CSR on the GPU (Eq. 3 compiled as in Sec. III-E).
//
// Term t adds to entry (r, r ^ x_t) the value c_t * i^{|x_t & z_t|} *
// (-1)^{|z_t & (r ^ x_t)|}.  Terms with the same x land in the same column of
// every row, so the host groups the terms by x (stably: ascending t inside a
// group) and folds i^{|x & z|} into the coefficients (an exact permutation and
// negation of their parts).  A group's entry of a row is the sum of its terms
// in ascending t from +0.0 with plain additions, so it is bit-identical to any
// sequential evaluation in that order.
//
// One wave evaluates a group for 64 consecutive rows, a row per lane: the
// group's masks and coefficients are then uniform (scalar loads), and a term
// costs three integer operations and one FP64 FMA by +-1 (exact, so the FMA is
// the plain addition).  What bounds it is that arithmetic: terms x rows / 64
// waves of four operations, once to size the rows and twice to fill them.
//
// A row's columns r ^ x ascend without a sort.  With the low six bits of x
// apart, the 64 rows of a workgroup share their high bits rh, so the order of
// rh ^ (x >> 6) is the same for all of them and is found once per workgroup
// (rank of a group from the counts of the smaller subtrees of a dense prefix
// table over x >> 6); among groups of equal x >> 6 the columns differ in six
// bits, so a 64-bit mask of the kept ones and a population count give each
// entry its place.
//
// Measured (one MI355X, both calls and their allocations): H at 16 qubits, FP64,
// 18.2 M entries, 6.12 -> 0.61 ms, of which the sizing kernel is 0.10 ms and the
// fill 0.40 ms; the 92 generators of a 12-qubit pool 16.9 -> 3.2 ms.  Before, the
// terms were sorted on the device by one launch per bitonic step, one wave took
// one row with its groups over the lanes (a wave waits for its longest group) and
// the kept entries were sorted in LDS; that form of the kernels is left where
// few rows have many terms.
//
// This file is built with -ffp-contract=off.
#include "common.hpp"

#include <algorithm>
#include <numeric>
#include <vector>

namespace {

constexpr int kMaxRow = 2048;      // longest supported row (entries kept per row)
constexpr int kMaxGroups = 2048;   // groups of the 64-row kernels (LDS)
constexpr int kMaxDense = 20;      // qubits of the dense table over x >> 6
constexpr int kInline = 1536;      // operator bytes passed as a kernel argument

// A grouped operator: one blob holding, at these byte offsets, the groups' x
// (ascending), the groups' first terms [G + 1], the number of groups with a
// smaller x >> 6 for every value of x >> 6 [cells + 1], the terms' z and their
// folded coefficients (real parts only when every term is real).
struct OpLayout {
    uint64_t gs, cls, tz, tc;
    int32_t G;
};
struct OpInline {
    alignas(16) unsigned char b[kInline];
};
template <bool REAL, bool INL = false> struct OpView {
    const uint32_t *gx, *gs, *cls, *tz;
    const double *tc;
    __device__ __forceinline__ OpView(const unsigned char *b, const OpLayout &L)
    {
        gx = reinterpret_cast<const uint32_t *>(b);
        gs = reinterpret_cast<const uint32_t *>(b + L.gs);
        cls = reinterpret_cast<const uint32_t *>(b + L.cls);
        tz = reinterpret_cast<const uint32_t *>(b + L.tz);
        tc = reinterpret_cast<const double *>(b + L.tc);
    }
};

// +1.0 or -1.0: the sign (-1)^{|v|}.
__device__ __forceinline__ double parity_sign(uint32_t v)
{
    return __hiloint2double((int)(((uint32_t)__popc(v) << 31) | 0x3ff00000u), 0);
}

// Entry of column col contributed by group g, summed in ascending term order
// (+-1 * c is exact, so each FMA is one addition).  The kernel argument's terms
// are indexed (a moving pointer into it would have it copied to scratch memory);
// others, of which there may be more than 32-bit offsets reach, are walked by
// pointer (16 qubits: 608 us, with 64-bit indexes 748).
template <bool REAL, bool INL>
__device__ __forceinline__ double2 group_entry(const OpView<REAL, INL> &op, int g, uint32_t col)
{
    double re = 0.0, im = 0.0;
    const uint32_t i0 = op.gs[g], i1 = op.gs[g + 1];
    auto add = [&](uint32_t z, const double *c) {
        const double s = parity_sign(z & col);
        re = fma(s, c[0], re);
        if constexpr (!REAL)
            im = fma(s, c[1], im);
    };
    constexpr int W = REAL ? 1 : 2;
    if constexpr (INL) {
#pragma unroll 4
        for (int i = (int)i0; i < (int)i1; i++)
            add(op.tz[i], &op.tc[W * i]);
    } else {
        const uint32_t *z = op.tz + i0;
        const double *c = op.tc + (size_t)i0 * W;
#pragma unroll 4
        for (uint32_t i = i0; i < i1; i++, z++, c += W)
            add(*z, c);
    }
    return make_double2(re, im);
}

__device__ __forceinline__ bool keep_entry(double2 v, double tol, bool force)
{
    return force || !(fabs(v.x) <= tol && fabs(v.y) <= tol);
}

// A value that every lane holds, in scalar registers; and this lane's bit of a
// wave mask held so.
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
}
__device__ __forceinline__ int row_bit(uint64_t v)
{
    return __builtin_amdgcn_inverse_ballot_w64(uniform64(v)) ? 1 : 0;
}

// Phase 1: kept entries per row; for rows with exactly one entry, its column.
// A workgroup takes 64 rows, its waves take the groups in turn.
template <bool REAL, bool INL>
__global__ void __launch_bounds__(1024)
k_row_count(int64_t dim, OpInline inl, const unsigned char *__restrict__ mem, OpLayout L, double tol,
            int force_diag, int32_t *__restrict__ counts, int32_t *__restrict__ onecol)
{
    __shared__ int32_t s_cnt[16][64], s_col[16][64];
    const OpView<REAL, INL> op(INL ? inl.b : mem, L);
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = (int64_t)blockIdx.x * 64 + lane;
    int32_t cnt = 0, cols = 0;
    for (int g = wid; g < L.G; g += waves) {
        const uint32_t x = op.gx[g], col = (uint32_t)r ^ x;
        if (keep_entry(group_entry(op, g, col), tol, force_diag && x == 0)) {
            cnt++;
            cols += (int32_t)col;      // one entry: its column
        }
    }
    s_cnt[wid][lane] = cnt;
    s_col[wid][lane] = cols;
    __syncthreads();
    if (wid == 0 && r < dim) {
        for (int w = 1; w < waves; w++) {
            cnt += s_cnt[w][lane];
            cols += s_col[w][lane];
        }
        counts[r] = cnt;
        onecol[r] = cnt == 1 ? cols : -1;
    }
}

// Phase 2: the rows' kept entries in column order (see the top of the file).
// A workgroup takes 64 rows: its waves first mark which rows keep each group
// (bal), then fill runs of the ordered groups in turn, each behind the entries
// of the runs before it.
template <int DT, bool REAL, bool INL>
__global__ void __launch_bounds__(1024)
k_row_fill(int64_t dim, OpInline inl, const unsigned char *__restrict__ mem, OpLayout L, double tol,
           double shift, int force_diag, int run, const int32_t *__restrict__ rowptr,
           int32_t *__restrict__ col_out, void *__restrict__ val_out)
{
    extern __shared__ uint64_t bal[];                       // [G]
    uint16_t *order = reinterpret_cast<uint16_t *>(bal + L.G);   // [G]
    __shared__ int32_t s_cnt[2][16][64];
    const OpView<REAL, INL> op(INL ? inl.b : mem, L);
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = (int64_t)blockIdx.x * 64 + lane;
    const uint32_t rh = blockIdx.x;
    const int G = L.G;
    for (int g = wid; g < G; g += waves) {
        const uint32_t x = op.gx[g], col = (uint32_t)r ^ x;
        const uint64_t m =
            __ballot(r < dim && keep_entry(group_entry(op, g, col), tol, force_diag && x == 0));
        if (lane == 0)
            bal[g] = m;
    }
    // place of group g: the groups of smaller rh ^ (x >> 6), then its index in
    // its class.  Where bit b of rh ^ h is set, the sibling subtree at bit b
    // comes first.
    for (int g = threadIdx.x; g < G; g += blockDim.x) {
        const uint32_t h = op.gx[g] >> 6;
        uint32_t at = (uint32_t)g - op.cls[h], d = rh ^ h;
        while (d) {
            const uint32_t b = 31u - (uint32_t)__clz((int)d);
            const uint32_t lo = ((h >> b) ^ 1u) << b;
            at += op.cls[lo + (1u << b)] - op.cls[lo];
            d ^= 1u << b;
        }
        order[at] = (uint16_t)g;
    }
    __syncthreads();
    // Runs of about `run` ordered groups, whole classes each, go round the
    // waves: the workgroup's writes to a row then advance as one narrow front,
    // and a row's lines are whole before they leave L2 (a contiguous share of
    // the order per wave wrote 3.1 times the bytes at 16 qubits).
    auto start = [&](int c) {
        int p = c * run < G ? c * run : G;
        while (p > 0 && p < G && (op.gx[order[p]] >> 6) == (op.gx[order[p - 1]] >> 6))
            p--;
        return __builtin_amdgcn_readfirstlane(p);
    };
    const int runs = (G + run - 1) / run;
    int64_t row = r < dim ? rowptr[r] : 0;               // the round's first entry of this row
    const int64_t end = r < dim ? rowptr[r + 1] : 0;     // a row never writes past its own range
    for (int c0 = 0, buf = 0; c0 < runs; c0 += waves, buf ^= 1) {
        int p = G, p1 = G;
        if (c0 + wid < runs) {
            p = start(c0 + wid);
            p1 = start(c0 + wid + 1);
        }
        int32_t n = 0;
        for (int q = p; q < p1; q++)
            n += row_bit(bal[order[q]]);
        s_cnt[buf][wid][lane] = n;
        __syncthreads();
        int64_t base = row;
        for (int w = 0; w < waves; w++) {
            const int32_t k = s_cnt[buf][w][lane];
            base += w < wid ? k : 0;
            row += k;
        }
        while (p < p1) {
            // a class's groups are consecutive
            const int g0 = __builtin_amdgcn_readfirstlane((int)order[p]);
            const int g1 = (int)op.cls[(op.gx[g0] >> 6) + 1];
            // the kept columns of the class by their low six bits, as two
            // words: of this lane's half of the block and of the other
            uint32_t own = 0, other = 0;
            for (int g = g0; g < g1; g++) {
                const uint32_t x = op.gx[g];
                const uint32_t bit = (uint32_t)row_bit(bal[g]) << ((x ^ (uint32_t)lane) & 31u);
                if (x & 32u)
                    other |= bit;
                else
                    own |= bit;
            }
            const uint32_t lo = lane & 32 ? other : own, hi = lane & 32 ? own : other;
            for (int g = g0; g < g1; g++) {
                const uint64_t bg = uniform64(bal[g]);
                if (bg == 0)      // no row of the block keeps this group
                    continue;
                const uint32_t x = op.gx[g], col = (uint32_t)r ^ x;
                double2 v = group_entry(op, g, col);
                const uint32_t below = (1u << (col & 31u)) - 1u;
                const int64_t at = base + ((col & 32u) ? __popc(lo) + __popc(hi & below) : __popc(lo & below));
                if (row_bit(bg) && at < end) {
                    if (x == 0)
                        v.x = v.x - shift;
                    col_out[at] = (int32_t)col;
                    Elem<DT>::st(val_out, at, v);
                }
            }
            base += __popc(own) + __popc(other);
            p += g1 - g0;
        }
    }
}

// The same two phases with one wave per row, its groups over the lanes, and a
// bitonic sort of the kept entries in LDS: registers of more than kMaxDense
// qubits (no dense table over x >> 6), operators of more than kMaxGroups
// groups, and few rows of many terms.
template <bool REAL>
__global__ void __launch_bounds__(64)
k_wave_count(int64_t dim, const unsigned char *__restrict__ mem, OpLayout L, double tol,
             int force_diag, int32_t *__restrict__ counts, int32_t *__restrict__ onecol)
{
    const OpView<REAL> op(mem, L);
    const int64_t r = blockIdx.x;
    const int lane = threadIdx.x;
    if (r >= dim)
        return;
    int64_t cnt = 0;
    int64_t last_col = -1;
    for (int g0 = 0; g0 < L.G; g0 += 64) {
        const int g = g0 + lane;
        bool keep = false;
        int64_t col = -1;
        if (g < L.G) {
            const uint32_t c = (uint32_t)r ^ op.gx[g];
            col = (int64_t)c;
            keep = keep_entry(group_entry(op, g, c), tol, force_diag && col == r);
        }
        uint64_t m = __ballot(keep);
        if (m) {
            // column of the highest kept lane (used only when the row has one entry)
            int hi = 63 - __clzll(m);
            int64_t c = __shfl(col, hi, 64);
            last_col = c;
        }
        cnt += __popcll(m);
    }
    if (lane == 0) {
        counts[r] = (int32_t)(cnt > 0x7fffffff ? 0x7fffffff : cnt);
        onecol[r] = cnt == 1 ? (int32_t)last_col : -1;
    }
}

// Multi-block exclusive scan of int32 counts into int64 (3 kernels).
__global__ void __launch_bounds__(1024)
k_scan_block(const int32_t *__restrict__ in, int64_t n, int64_t *__restrict__ out,
             int64_t *__restrict__ block_sums)
{
    __shared__ int64_t s[1024];
    const int tid = threadIdx.x;
    int64_t i = (int64_t)blockIdx.x * 1024 + tid;
    int64_t v = i < n ? (int64_t)in[i] : 0;
    s[tid] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        int64_t t = tid >= o ? s[tid - o] : 0;
        __syncthreads();
        s[tid] += t;
        __syncthreads();
    }
    if (i < n)
        out[i] = s[tid] - v;   // exclusive within block
    if (tid == 1023)
        block_sums[blockIdx.x] = s[1023];
}

__global__ void __launch_bounds__(1024)
k_scan_sums(int64_t *__restrict__ sums, int64_t nb, int64_t *__restrict__ total,
            unsigned long long *__restrict__ stats)
{
    __shared__ int64_t s[1024];
    __shared__ int64_t carry;
    const int tid = threadIdx.x;
    if (tid == 0)
        carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < nb; base += 1024) {
        int64_t i = base + tid;
        int64_t v = i < nb ? sums[i] : 0;
        s[tid] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            int64_t t = tid >= o ? s[tid - o] : 0;
            __syncthreads();
            s[tid] += t;
            __syncthreads();
        }
        if (i < nb)
            sums[i] = carry + s[tid] - v;
        __syncthreads();
        if (tid == 1023)
            carry += s[1023];
        __syncthreads();
    }
    if (tid == 0) {
        *total = carry;
        stats[0] = stats[1] = 0;
    }
}

// rowptr[i] = exclusive prefix (int32, valid when the total fits), rowptr[n] = total;
// and the pairing check (every row has <= 1 entry and col(col(r)) == r: else
// stats[0] = 1) and stats[1] = the longest row.
__global__ void __launch_bounds__(1024)
k_scan_finish(const int64_t *__restrict__ part, const int64_t *__restrict__ sums, int64_t n,
              const int64_t *__restrict__ total, const int32_t *__restrict__ counts,
              const int32_t *__restrict__ onecol, int32_t *__restrict__ rowptr,
              unsigned long long *__restrict__ stats)
{
    __shared__ int32_t s_max[16];
    const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    bool bad = false;
    int32_t mx = 0;
    if (i < n) {
        const int64_t v = part[i] + sums[i / 1024];
        rowptr[i] = (int32_t)(v > 0x7fffffff ? 0x7fffffff : v);
        mx = counts[i];
        bad = mx > 1;
        if (mx == 1) {
            const int32_t c = onecol[i];
            bad = c < 0 || c >= n || onecol[c] != (int32_t)i;
        }
    } else if (i == n) {
        const int64_t t = *total;
        rowptr[n] = (int32_t)(t > 0x7fffffff ? 0x7fffffff : t);
    }
    if (__ballot(bad) && (threadIdx.x & 63) == 0)
        stats[0] = 1;      // every writer stores the same
    for (int o = 32; o > 0; o >>= 1)
        mx = max(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0)
        s_max[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; w++)
            mx = max(mx, s_max[w]);
        atomicMax(&stats[1], (unsigned long long)mx);
    }
}

// Row starts, the pairing check and the longest row of an operator of at most
// kScanRows rows, in one workgroup: a register-sized operator's sizing is
// launches and gaps, and this replaces five of them.  host (pinned) receives
// the entries, the violations of the pairing and the longest row.
constexpr int64_t kScanRows = 32768;
__global__ void __launch_bounds__(1024)
k_scan_rows(int64_t dim, const int32_t *__restrict__ counts, const int32_t *__restrict__ onecol,
            int32_t *__restrict__ rowptr, int64_t *__restrict__ host)
{
    __shared__ int64_t s_sum[16];
    __shared__ int32_t s_bad[16], s_max[16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int64_t carry = 0;
    int32_t bad = 0, mx = 0;
    for (int64_t r0 = 0; r0 < dim; r0 += 4096) {
        // four consecutive rows per thread
        int32_t c[4];
        int64_t own = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int64_t r = r0 + 4 * tid + q;
            c[q] = r < dim ? counts[r] : 0;
            own += c[q];
            mx = max(mx, c[q]);
            if (c[q] > 1)
                bad++;
            else if (c[q] == 1) {
                const int32_t o = onecol[r];
                bad += (o < 0 || o >= dim || onecol[o] != (int32_t)r);
            }
        }
        int64_t inc = own;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(inc, o, 64);
            if (lane >= o)
                inc += t;
        }
        if (lane == 63)
            s_sum[wid] = inc;
        __syncthreads();
        int64_t at = carry + inc - own;
        for (int w = 0; w < 16; w++) {
            if (w < wid)
                at += s_sum[w];
            carry += s_sum[w];
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int64_t r = r0 + 4 * tid + q;
            if (r < dim)
                rowptr[r] = (int32_t)(at > 0x7fffffff ? 0x7fffffff : at);
            at += c[q];
        }
        __syncthreads();
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        bad += __shfl_xor(bad, o, 64);
        mx = max(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
        s_bad[wid] = bad;
        s_max[wid] = mx;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 16; w++) {
            bad += s_bad[w];
            mx = max(mx, s_max[w]);
        }
        rowptr[dim] = (int32_t)(carry > 0x7fffffff ? 0x7fffffff : carry);
        host[0] = carry;
        host[1] = bad;
        host[2] = mx;
    }
}

// Phase 2: recompute each row's kept entries, sort by column in LDS, write.
template <int DT, bool REAL>
__global__ void __launch_bounds__(64)
k_wave_fill(int64_t dim, const unsigned char *__restrict__ mem, OpLayout L, double tol, double shift,
            int force_diag, int pad, const int32_t *__restrict__ rowptr,
            int32_t *__restrict__ col_out, void *__restrict__ val_out)
{
    extern __shared__ unsigned char smem[];
    const OpView<REAL> op(mem, L);
    int32_t *s_col = reinterpret_cast<int32_t *>(smem);
    double2 *s_val = reinterpret_cast<double2 *>(smem + vqe_align((size_t)pad * 4));
    const int64_t r = blockIdx.x;
    const int lane = threadIdx.x;
    if (r >= dim)
        return;
    int base = 0;
    for (int g0 = 0; g0 < L.G; g0 += 64) {
        const int g = g0 + lane;
        bool keep = false;
        double2 v = make_double2(0.0, 0.0);
        int32_t col = 0;
        if (g < L.G) {
            col = (int32_t)((uint32_t)r ^ op.gx[g]);
            v = group_entry(op, g, (uint32_t)col);
            keep = keep_entry(v, tol, force_diag && col == r);
        }
        uint64_t m = __ballot(keep);
        if (keep) {
            int pos = base + __popcll(m & ((1ull << lane) - 1ull));
            if (pos < pad) {
                s_col[pos] = col;
                s_val[pos] = v;
            }
        }
        base += __popcll(m);
    }
    // the kept count equals the sizing pass (same ordered sums); clamp anyway
    // so a row can never write past its own slot range
    const int64_t o = rowptr[r];
    const int64_t room = (int64_t)rowptr[r + 1] - o;
    int n = base < pad ? base : pad;
    if (n > room)
        n = (int)(room > 0 ? room : 0);
    for (int i = n + lane; i < pad; i += 64) {
        s_col[i] = 0x7fffffff;
        s_val[i] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    for (int k = 2; k <= pad; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = lane; i < pad; i += 64) {
                int l = i ^ j;
                if (l > i) {
                    int32_t ci = s_col[i], cl = s_col[l];
                    bool ascending = (i & k) == 0;
                    if ((ci > cl) == ascending) {
                        double2 vi = s_val[i];
                        s_col[i] = cl;
                        s_col[l] = ci;
                        s_val[i] = s_val[l];
                        s_val[l] = vi;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (int i = lane; i < n; i += 64) {
        double2 v = s_val[i];
        int32_t c = s_col[i];
        if (c == (int32_t)r)
            v.x = v.x - shift;
        col_out[o + i] = c;
        Elem<DT>::st(val_out, o + i, v);
    }
}

__global__ void k_row_max(int64_t dim, const int32_t *__restrict__ rowptr,
                          unsigned long long *__restrict__ mx)
{
    int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t len = r < dim ? rowptr[r + 1] - rowptr[r] : 0;
    for (int o = 32; o > 0; o >>= 1)
        len = max(len, __shfl_xor(len, o, 64));
    if ((threadIdx.x & 63) == 0)
        atomicMax(mx, (unsigned long long)len);
}

inline int64_t next_pow2(int64_t v)
{
    int64_t p = 1;
    while (p < v)
        p <<= 1;
    return p;
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

// ------------------------------------------------------------------ host side
namespace {

// Terms as flip mask << 32 | number, into ascending order: by mask, then as
// given.  Many of them by the digits of the mask (eleven bits a pass; the numbers
// ascend already): comparing made the two calls of 10^5 terms in no order 13 to
// 16 ms, of which this is 2; below kDigitSort terms the digits' tables cost more.
constexpr size_t kDigitSort = 512;
void sort_terms(std::vector<uint64_t> &key, int n_qubits)
{
    if (key.size() < kDigitSort) {
        std::sort(key.begin(), key.end());
        return;
    }
    std::vector<uint64_t> next(key.size());
    for (int at = 32; at < 32 + n_qubits; at += 11) {
        size_t start[2048] = {};
        for (const uint64_t k : key)
            start[(k >> at) & 2047u]++;
        size_t sum = 0;
        for (size_t &c : start) {
            const size_t n = c;
            c = sum;
            sum += n;
        }
        for (const uint64_t k : key)
            next[start[(k >> at) & 2047u]++] = k;
        key.swap(next);
    }
}

}  // namespace

extern "C" int csr_build_from_pauli(vqe_ctx *ctx, int32_t n_qubits, int64_t n_terms,
                                    const uint64_t *xmask, const uint64_t *zmask,
                                    const double *coeff, double drop_tol, int32_t dtype,
                                    double diag_shift, vqe_csr *inout, int64_t *nnz_out)
try {
    if (!ctx || !inout)
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: null context or descriptor");
    if (n_qubits < 1 || n_qubits > 30)
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: n_qubits %d outside [1, 30]",
                        n_qubits);
    if (n_terms < 0 || (n_terms > 0 && (!xmask || !zmask || !coeff)))
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: bad term arrays");
    if (n_terms >= ((int64_t)1 << 31))
        return vqe_fail(ctx, VQE_ESIZE, "csr_build_from_pauli: too many terms");
    if (dtype != VQE_C128 && dtype != VQE_C64)
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: unknown dtype %d", dtype);
    if (!std::isfinite(drop_tol) || drop_tol < 0 || !std::isfinite(diag_shift))
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: bad drop_tol or diag_shift");
    if (dtype == VQE_C128 && diag_shift != 0.0)
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: diag_shift needs VQE_C64");
    if (!inout->rowptr)
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: rowptr is null");
    const bool fill = inout->col != nullptr || inout->val != nullptr;
    if (fill && (!inout->col || !inout->val))
        return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: col and val must both be set");
    const uint64_t lim = ~(uint64_t)0 << n_qubits;
    for (int64_t t = 0; t < n_terms; t++)
        if ((xmask[t] | zmask[t]) & lim)
            return vqe_fail(ctx, VQE_EINVAL,
                            "csr_build_from_pauli: term %lld has a mask bit >= n_qubits",
                            (long long)t);
    for (int64_t t = 0; t < 2 * n_terms; t++)
        if (!std::isfinite(coeff[t]))
            return vqe_fail(ctx, VQE_EINVAL, "csr_build_from_pauli: non-finite coefficient");

    const int64_t dim = (int64_t)1 << n_qubits;
    const bool force_diag = diag_shift != 0.0;
    const int64_t nb = (dim + 1023) / 1024;
    hipStream_t s = ctx->stream;

    // Terms in group order: by x, then ascending t.  With a shift every row
    // needs its diagonal entry: an extra zero identity term (last, so the
    // order of the given terms is unchanged) makes sure the x = 0 group exists.
    const int64_t T = n_terms + (force_diag ? 1 : 0);
    std::vector<uint64_t> key;      // (none: the order as given)
    bool sorted = true;
    for (int64_t t = 1; t < n_terms && sorted; t++)
        sorted = xmask[t - 1] <= xmask[t];
    if (!sorted || force_diag) {
        key.reserve((size_t)T);
        for (int64_t t = 0; t < n_terms; t++)
            key.push_back(xmask[t] << 32 | (uint64_t)t);
        // the zero term joins the end of the x = 0 run
        if (force_diag)
            key.insert(sorted ? std::upper_bound(key.begin(), key.end(), (uint64_t)n_terms) : key.end(),
                       (uint64_t)n_terms);
        if (!sorted)
            sort_terms(key, n_qubits);
    }
    auto term = [&](int64_t i) { return key.empty() ? i : (int64_t)(uint32_t)key[(size_t)i]; };
    auto term_x = [&](int64_t i) { return key.empty() ? (uint32_t)xmask[i] : (uint32_t)(key[(size_t)i] >> 32); };
    // every entry is real when every term's c_t i^{|x_t & z_t|} is real
    bool real = true;
    for (int64_t t = 0; t < n_terms && real; t++) {
        const int k = __builtin_popcountll(xmask[t] & zmask[t]) & 3;
        real = (k & 1) ? coeff[2 * t] == 0.0 : coeff[2 * t + 1] == 0.0;
    }
    int64_t G = 0;
    for (int64_t i = 0; i < T; i++)
        G += i == 0 || term_x(i) != term_x(i - 1);
    // the 64-row kernels, unless few rows have many terms: 2^11 rows are 32 of
    // their workgroups, whose waves take a group's terms one after another, where
    // one wave per row has 32 times the waves and a group per lane (sizing and
    // fill, 8 qubits: 64 groups of 8 terms 71 us either way, of 200 742 against 386;
    // 11 qubits: 256 of 8 157 and 150, of 200 2004 and 1464; from 2^12 rows on the
    // 64-row kernels are the faster, or near).  Its sort of a row's entries
    // needs more terms to pay for rows of over 1024 (2000 groups of 8 882 and
    // 1118, of 30 2744 and 2132).
    const bool few_rows = n_qubits <= 11 && T >= 1024 && (G <= 1024 || T >= 24 * G);
    const bool wide = n_qubits <= kMaxDense && G <= kMaxGroups && !few_rows;
    const int64_t cells = wide ? std::max<int64_t>(dim >> 6, 1) : 0;
    OpLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 15) & ~(size_t)15; return o; };
    take((size_t)G * 4);
    const size_t o_gs = take((size_t)(G + 1) * 4), o_cls = take((size_t)(cells + 1) * 4);
    const size_t o_tz = take((size_t)T * 4), o_tc = take((size_t)T * (real ? 8 : 16));
    const size_t op_bytes = off;
    L.gs = o_gs;
    L.cls = o_cls;
    L.tz = o_tz;
    L.tc = o_tc;
    L.G = (int32_t)G;
    const bool inl = wide && op_bytes <= (size_t)kInline;
    // A small operator travels as a kernel argument, a larger one through the
    // context's pinned staging (its last copy waited for), beyond that from
    // pageable memory, which the copy is waited for.
    OpInline small;
    std::vector<unsigned char> blob;
    unsigned char *b = small.b;
    const bool staged = !inl && op_bytes <= VQE_STAGE_BYTES;
    if (staged) {
        if (!ctx->stage) {
            if (hipHostMalloc(&ctx->stage, VQE_STAGE_BYTES, hipHostMallocDefault) != hipSuccess) {
                ctx->stage = nullptr;
                (void)hipGetLastError();
                return vqe_fail(ctx, VQE_ENOMEM, "csr_build_from_pauli: staging allocation failed");
            }
        }
        if (!ctx->stage_ev)
            VQE_HIP(ctx, hipEventCreateWithFlags(&ctx->stage_ev, hipEventDisableTiming));
        VQE_HIP(ctx, hipEventSynchronize(ctx->stage_ev));
        b = (unsigned char *)ctx->stage;
    } else if (!inl) {
        blob.resize(op_bytes);
        b = blob.data();
    }
    uint32_t *h_gx = (uint32_t *)b, *h_cls = (uint32_t *)(b + o_cls), *h_tz = (uint32_t *)(b + o_tz);
    uint32_t *h_gs = (uint32_t *)(b + o_gs);
    double *h_tc = (double *)(b + o_tc);
    int64_t g = 0, cell = 0;
    for (int64_t i = 0; i < T; i++) {
        const int64_t t = term(i);
        const uint32_t x = term_x(i);
        if (g == 0 || x != h_gx[g - 1]) {
            for (; cells && cell <= (int64_t)(x >> 6); cell++)
                h_cls[cell] = (uint32_t)g;
            h_gx[g] = x;
            h_gs[g++] = (uint32_t)i;
        }
        // i^{|x & z|} folded into the coefficient (exact)
        double re = 0.0, im = 0.0;
        h_tz[i] = 0;
        if (t < n_terms) {
            h_tz[i] = (uint32_t)zmask[t];
            const double cr = coeff[2 * t], ci = coeff[2 * t + 1];
            switch (__builtin_popcountll(xmask[t] & zmask[t]) & 3) {
            case 0: re = cr; im = ci; break;
            case 1: re = -ci; im = cr; break;
            case 2: re = -cr; im = -ci; break;
            default: re = ci; im = -cr; break;
            }
        }
        if (real) {
            h_tc[i] = re;
        } else {
            h_tc[2 * i] = re;
            h_tc[2 * i + 1] = im;
        }
    }
    h_gs[G] = (uint32_t)T;
    for (; cells && cell <= cells; cell++)
        h_cls[cell] = (uint32_t)G;

    // workspace layout
    off = 0;
    auto ws_take = [&](size_t bytes) { size_t o = off; off += vqe_align(bytes); return o; };
    const size_t o_op = ws_take(op_bytes + 16);
    const size_t o_cnt = ws_take(dim * 4), o_one = ws_take(dim * 4), o_part = ws_take(dim * 8);
    const size_t o_bs = ws_take(nb * 8 + 8), o_tot = ws_take(24);   // the total, then two statistics
    int rc = vqe_ws_reserve(ctx, off);
    if (rc)
        return rc;
    char *ws = (char *)ctx->ws;
    unsigned char *d_op = (unsigned char *)(ws + o_op);
    int32_t *d_cnt = (int32_t *)(ws + o_cnt), *d_one = (int32_t *)(ws + o_one);
    int64_t *d_part = (int64_t *)(ws + o_part), *d_bs = (int64_t *)(ws + o_bs);
    int64_t *d_tot = (int64_t *)(ws + o_tot);
    unsigned long long *d_stats = (unsigned long long *)(d_tot + 1);
    if (!inl)
        VQE_HIP(ctx, hipMemcpyAsync(d_op, b, op_bytes, hipMemcpyHostToDevice, s));
    if (staged)
        VQE_HIP(ctx, hipEventRecord(ctx->stage_ev, s));
    else if (!inl)
        VQE_HIP(ctx, hipStreamSynchronize(s));
    const unsigned rows64 = (unsigned)((dim + 63) / 64);
    const int fd = force_diag ? 1 : 0;
    // waves per 64 rows: one for each group up to 16 (16 against 8 at 14 qubits: 0.99
    // against 1.07 ms for an admitted run; 4 against 16 for 30 groups of 200 terms at
    // 12 qubits: 616 against 298 us)
    const int waves = G < 2 ? 1 : G < 4 ? 2 : G < 8 ? 4 : G < 16 ? 8 : 16;

    if (!fill) {
        int64_t *h = ctx->host_scalars;
        if (wide) {
            auto k = real ? (inl ? k_row_count<true, true> : k_row_count<true, false>)
                          : (inl ? k_row_count<false, true> : k_row_count<false, false>);
            k<<<rows64, 64 * waves, 0, s>>>(dim, small, d_op, L, drop_tol, fd, d_cnt, d_one);
        } else {
            auto k = real ? k_wave_count<true> : k_wave_count<false>;
            k<<<(unsigned)dim, 64, 0, s>>>(dim, d_op, L, drop_tol, fd, d_cnt, d_one);
        }
        if (dim <= kScanRows) {
            k_scan_rows<<<1, 1024, 0, s>>>(dim, d_cnt, d_one, inout->rowptr, h);
            VQE_LAUNCH_CHECK(ctx);
        } else {
            k_scan_block<<<(unsigned)nb, 1024, 0, s>>>(d_cnt, dim, d_part, d_bs);
            k_scan_sums<<<1, 1024, 0, s>>>(d_bs, nb, d_tot, d_stats);
            k_scan_finish<<<grid_for(dim + 1, 1024), 1024, 0, s>>>(d_part, d_bs, dim, d_tot, d_cnt,
                                                                   d_one, inout->rowptr, d_stats);
            VQE_LAUNCH_CHECK(ctx);
            VQE_HIP(ctx, hipMemcpyAsync(h, d_tot, 24, hipMemcpyDeviceToHost, s));
        }
        VQE_HIP(ctx, hipStreamSynchronize(s));
        const int64_t nnz = h[0];
        const int64_t violations = h[1], maxrow = h[2];
        if (nnz > 0x7fffffff)
            return vqe_fail(ctx, VQE_ESIZE, "csr_build_from_pauli: nnz %lld exceeds INT32_MAX",
                            (long long)nnz);
        if (maxrow > kMaxRow)
            return vqe_fail(ctx, VQE_ESIZE,
                            "csr_build_from_pauli: a row holds %lld entries (max %d)",
                            (long long)maxrow, kMaxRow);
        inout->n_qubits = n_qubits;
        inout->dtype = dtype;
        inout->dim = dim;
        inout->nnz = nnz;
        inout->diag_shift = diag_shift;
        inout->flags = (violations == 0 ? VQE_PAIRING : 0u) | (real ? VQE_REAL : 0u);
        if (nnz_out)
            *nnz_out = nnz;
        return VQE_OK;
    }

    // phase 2
    if (inout->dim != dim || inout->dtype != dtype || inout->n_qubits != n_qubits)
        return vqe_fail(ctx, VQE_EINVAL,
                        "csr_build_from_pauli: descriptor does not match the sizing call");
    const bool d = dtype == VQE_C128;
    if (wide) {
        // (a row holds at most one entry per group, so no row is too long)
        const size_t lds = (size_t)G * 8 + (size_t)G * 2 + 16;
        // below 2^14 rows what is written stays in L2 whatever the order, and
        // one round of equal shares saves its barriers (12 qubits: 121 against
        // 132 us); above, rounds of 16 (16 qubits: 0.57 against 0.63 ms)
        const int run = dim < 16384 ? std::max((int)((G + waves - 1) / waves), 1) : 16;
        auto k = d ? (real ? (inl ? k_row_fill<VQE_C128, true, true> : k_row_fill<VQE_C128, true, false>)
                           : (inl ? k_row_fill<VQE_C128, false, true> : k_row_fill<VQE_C128, false, false>))
                   : (real ? (inl ? k_row_fill<VQE_C64, true, true> : k_row_fill<VQE_C64, true, false>)
                           : (inl ? k_row_fill<VQE_C64, false, true> : k_row_fill<VQE_C64, false, false>));
        k<<<rows64, 64 * waves, lds, s>>>(dim, small, d_op, L, drop_tol, diag_shift, fd, run, inout->rowptr,
                                          inout->col, inout->val);
        VQE_LAUNCH_CHECK(ctx);
        if (nnz_out)
            *nnz_out = inout->nnz;
        return VQE_OK;
    }
    VQE_HIP(ctx, hipMemsetAsync(d_stats, 0, 16, s));
    k_row_max<<<grid_for(dim, 256), 256, 0, s>>>(dim, inout->rowptr, d_stats);
    VQE_LAUNCH_CHECK(ctx);
    int64_t *h = ctx->host_scalars;
    VQE_HIP(ctx, hipMemcpyAsync(h, d_stats, 8, hipMemcpyDeviceToHost, s));
    VQE_HIP(ctx, hipStreamSynchronize(s));
    const int64_t maxrow = h[0];
    if (maxrow > kMaxRow)
        return vqe_fail(ctx, VQE_ESIZE, "csr_build_from_pauli: row too long");
    const int pad = (int)std::max<int64_t>(next_pow2(std::max<int64_t>(maxrow, 1)), 64);
    const size_t lds = vqe_align((size_t)pad * 4) + (size_t)pad * 16;
    auto k = d ? (real ? k_wave_fill<VQE_C128, true> : k_wave_fill<VQE_C128, false>)
               : (real ? k_wave_fill<VQE_C64, true> : k_wave_fill<VQE_C64, false>);
    k<<<(unsigned)dim, 64, lds, s>>>(dim, d_op, L, drop_tol, diag_shift, fd, pad, inout->rowptr,
                                     inout->col, inout->val);
    VQE_LAUNCH_CHECK(ctx);
    if (nnz_out)
        *nnz_out = inout->nnz;
    return VQE_OK;
} catch (const std::bad_alloc &) {
    return vqe_fail(ctx, VQE_ENOMEM, "csr_build_from_pauli: host allocation failed");
}
