// The launch functions of csrc/kernels.h that the GCN layer calls use, as
// plain loops over host memory, and a HIP runtime that copies at once: linked
// with csrc/digest_host.cpp they make a library whose layer calls run on the
// CPU, so that which kernel gets which operand is checked without a GPU.
#include <cmath>
#include <cstring>

#include "kernels.h"

namespace {
int n_sliced = 0, n_whole = 0, n_pending = 0;
constexpr hipError_t kNo = hipErrorNotSupported;
}  // namespace

extern "C" {
// Aggregations out of column slices, and of whole rows, since the last call.
void host_kernels_counts(int *sliced, int *whole)
{
    *sliced = n_sliced, *whole = n_whole;
    n_sliced = n_whole = 0;
}
// Copies that no synchronization has followed.
int host_kernels_pending() { return n_pending; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    ++n_pending;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "host kernels"; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { *d = 0; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { n_pending = 0; return hipSuccess; }
}

namespace digest {

hipError_t launch_copy_rows(const int32_t *sidx, const int32_t *didx, int32_t n, int32_t d,
                            const float *src, float *dst, hipStream_t, int32_t lds, int32_t ldd)
{
    lds = lds > 0 ? lds : d, ldd = ldd > 0 ? ldd : d;
    for (int64_t r = 0; r < n; ++r)
        std::memcpy(dst + (didx ? didx[r] : r) * (int64_t)ldd,
                    src + (sidx ? sidx[r] : r) * (int64_t)lds, sizeof(float) * d);
    return hipSuccess;
}

bool spmm_epilogue_ok(int32_t d, int32_t n2, const float *) { return d <= kNarrow && n2 > 0; }

hipError_t launch_spmm(const SpmmBlock *blocks, int32_t n_blocks, int32_t, const int32_t *rowptr,
                       const int32_t *col, const float *val, const float *src0, const float *src1,
                       int32_t n_src0, int32_t d, float *out0, hipStream_t,
                       const SpmmEpilogue *ep, float *out1, int32_t n_out0, bool relu, bool acc,
                       int32_t lds, int32_t out_ld, int32_t out_w)
{
    lds = lds > 0 ? lds : d, out_ld = out_ld > 0 ? out_ld : d, out_w = out_w > 0 ? out_w : d;
    ++n_whole;
#pragma omp parallel for
    for (int32_t b = 0; b < n_blocks; ++b)
        for (int32_t r = blocks[b].row; r < blocks[b].row + (blocks[b].nrows ? blocks[b].nrows : 1);
             ++r) {
            float *out = r < n_out0 ? out0 + (int64_t)r * out_ld
                                    : out1 + (int64_t)(r - n_out0) * out_ld;
            for (int32_t f = 0; f < out_w; ++f) {
                double sum = acc ? out[f] : 0.0;
                for (int32_t k = rowptr[r]; k < rowptr[r + 1]; ++k)
                    sum += (double)val[k] * (col[k] < n_src0
                                                 ? src0[(int64_t)col[k] * lds + f]
                                                 : src1[(int64_t)(col[k] - n_src0) * lds + f]);
                out[f] = relu && !(sum > 0) ? 0.f : (float)sum;
            }
            for (int32_t n = 0; ep && n < ep->n2; ++n) {
                float *to = r < ep->rows ? ep->out2 + (int64_t)r * ep->n2
                            : ep->out3   ? ep->out3 + (int64_t)(r - ep->rows) * ep->n2
                                         : nullptr;
                double sum = 0;
                for (int32_t k = 0; k < d; ++k)
                    sum += (double)out[k] * ep->w[(int64_t)n * d + k];
                if (to)
                    to[n] = (float)sum;
            }
        }
    return hipSuccess;
}

hipError_t launch_slice_rows(int32_t n, int32_t d, const float *src, int32_t lds, const float *h,
                             int32_t ldh, float *dst, hipStream_t)
{
    const int64_t W = kSliceFloats;
    for (int64_t r = 0; r < n; ++r)
        for (int64_t c = 0; c < (d + W - 1) / W * W; ++c)
            dst[c / W * n * W + r * W + c % W] =
                c < d && (!h || h[r * ldh + c] > 0) ? src[r * lds + c] : 0.f;
    return hipSuccess;
}

hipError_t launch_spmm_slice(const SpmmBlock *blocks, int32_t n_blocks, int32_t n_long,
                             const int32_t *rowptr, const int32_t *col, const float *val,
                             const float *src, int32_t n_src, const float *src1, int32_t ld1,
                             int32_t d, float *out, int32_t ldo, bool relu, hipStream_t)
{
    const int64_t W = kSliceFloats;
    ++n_sliced;
#pragma omp parallel for
    for (int32_t b = 0; b < n_blocks; ++b)
        for (int32_t r = blocks[b].row; r < blocks[b].row + (b < n_long ? 1 : blocks[b].nrows);
             ++r)
            for (int64_t f = 0; f < d; ++f) {
                double sum = 0;
                for (int32_t k = rowptr[r]; k < rowptr[r + 1]; ++k)
                    sum += col[k] < n_src
                               ? (double)val[k] * src[f / W * n_src * W + col[k] * W + f % W]
                               : (double)src1[(int64_t)(col[k] - n_src) * ld1 + f];
                out[(int64_t)r * ldo + f] = relu && !(sum > 0) ? 0.f : (float)sum;
            }
    return hipSuccess;
}

hipError_t launch_relu_mask(int64_t n, int32_t d, const float *g, int32_t ldg, const float *h,
                            int32_t ldh, float *out, int32_t ldo, hipStream_t,
                            const int32_t *idx)
{
    for (int64_t r = 0; r < n; ++r)
        for (int64_t c = 0, s = idx ? idx[r] : r; c < d; ++c)
            out[r * ldo + c] = h[s * ldh + c] > 0 ? g[s * ldg + c] : 0.f;
    return hipSuccess;
}

hipError_t launch_gemm(const GemmArgs &a, hipStream_t)
{
    for (int64_t z = 0; z < a.splits; ++z) {
        const int64_t kb = z * a.kchunk, ke = kb + a.kchunk < a.K ? kb + a.kchunk : a.K;
#pragma omp parallel for
        for (int64_t m = 0; m < a.M; ++m)
            for (int64_t n = 0; n < a.N; ++n) {
                double sum = 0;
                for (int64_t k = kb; k < ke; ++k) {
                    const int64_t ia = a.a_trans ? k * a.lda + m : m * a.lda + k;
                    const int64_t ib = a.b_trans ? n * a.ldb + k : k * a.ldb + n;
                    if ((!a.a_mask || a.a_mask[ia] > 0) && (!a.b_mask || a.b_mask[ib] > 0))
                        sum += (double)a.A[ia] * a.B[ib];
                }
                a.C[(a.splits > 1 ? z * a.M * a.ldc : 0) + m * a.ldc + n] =
                    a.relu && !(sum > 0) ? 0.f : (float)sum;
            }
    }
    return hipSuccess;
}

hipError_t launch_splitk_reduce(const float *part, int32_t splits, int64_t count, float *out,
                                hipStream_t)
{
    for (int64_t e = 0; e < count; ++e) {
        double sum = 0;
        for (int32_t z = 0; z < splits; ++z)
            sum += part[z * count + e];
        out[e] = (float)sum;
    }
    return hipSuccess;
}

size_t narrow_n_lds(int32_t K, int32_t N) { return sizeof(float) * narrow_n_stride(K) * N; }
hipError_t launch_narrow_n(int32_t M, int32_t m0, int32_t K, int32_t N, const float *A0,
                           const float *A1, int32_t lda, const float *B, float *C, int32_t ldc,
                           bool relu, hipStream_t s, int32_t lda1)
{
    GemmArgs g{m0 < M ? m0 : M, N, K, A0, lda, false, nullptr, B, N, false, nullptr, C, ldc,
               relu, 1, K};
    if (hipError_t e = launch_gemm(g, s))
        return e;
    g.M = M - g.M, g.A = A1, g.lda = lda1 > 0 ? lda1 : lda, g.C = C + (int64_t)m0 * ldc;
    return g.M > 0 ? launch_gemm(g, s) : hipSuccess;
}
hipError_t launch_narrow_k(int32_t M, int32_t N, int32_t K, const float *A, int32_t lda,
                           const float *W, float *C, int32_t ldc, hipStream_t s)
{
    return launch_gemm({M, N, K, A, lda, false, nullptr, W, K, true, nullptr, C, ldc, false, 1, K},
                       s);
}
size_t times_wt_lds(int32_t K, int32_t N) { return sizeof(float) * (K + 4) * N; }
hipError_t launch_times_wt(int32_t M, int32_t N, int32_t K, const float *A, int32_t lda,
                           const float *W, float *C, int32_t ldc, hipStream_t s)
{
    return launch_narrow_k(M, N, K, A, lda, W, C, ldc, s);
}
hipError_t launch_dw_narrow(int32_t R, int32_t m0, int32_t F, int32_t N, const float *H0,
                            const float *H1, int32_t ldh, const float *G, int32_t ldg,
                            int32_t chunk, int32_t splits, float *part, hipStream_t, int32_t ldh1)
{
    for (int64_t z = 0; z < splits; ++z)
        for (int64_t f = 0; f < F; ++f)
            for (int64_t n = 0; n < N; ++n) {
                double sum = 0;
                for (int64_t r = z * chunk; r < (z + 1) * chunk && r < R; ++r)
                    sum += (double)G[r * ldg + n] *
                           (r < m0 ? H0[r * ldh + f]
                                   : H1[(r - m0) * (ldh1 > 0 ? ldh1 : ldh) + f]);
                part[(z * F + f) * N + n] = (float)sum;
            }
    return hipSuccess;
}

// what these calls do not reach
bool spmm_tier_ok(int32_t, const float *, const float *, const float *) { return false; }
hipError_t launch_spmm_tier(const SpmmBlock *, int32_t, int32_t, const int32_t *, const int32_t *,
                            const float *, int64_t, const float *, const float *, int32_t,
                            int32_t, int32_t, float *, bool, hipStream_t) { return kNo; }
bool spmm_gemm_ok(int32_t, int32_t, int32_t, const float *, const float *, const float *,
                  const float *) { return false; }
hipError_t launch_spmm_gemm(int32_t, const int32_t *, const int32_t *, const float *,
                            const uint8_t *, const float *, const float *, int32_t, int32_t,
                            int32_t, float *, const float *, int32_t, const float *, int32_t,
                            float *, int32_t, bool, hipStream_t) { return kNo; }
hipError_t launch_transpose(int32_t, int32_t, const float *, float *, hipStream_t) { return kNo; }
hipError_t launch_add_rows(const int32_t *, const int32_t *, int32_t, int32_t, const float *,
                           float *, hipStream_t) { return kNo; }
hipError_t launch_add_clear_rows(const int32_t *, const int32_t *, int32_t, int32_t, float *,
                                 float *, hipStream_t) { return kNo; }
int32_t softmax_xent_blocks(int32_t, int32_t) { return 1; }
int32_t softmax_xent_rows_per_block(int32_t) { return 1; }
hipError_t launch_softmax_xent(const float *, const int32_t *, int32_t, int32_t, float *, float *,
                               hipStream_t) { return kNo; }
hipError_t launch_loss_mean(const float *, int32_t, int32_t, float *, hipStream_t) { return kNo; }
hipError_t launch_sgd_average(float *, const GradList &, int32_t, int64_t, float,
                              hipStream_t) { return kNo; }
hipError_t static_scratch(float **) { return kNo; }
hipError_t launch_fill_zero(float *p, int64_t n, hipStream_t)
{
    std::memset(p, 0, sizeof(float) * n);
    return hipSuccess;
}
hipError_t launch_gat_softmax(int32_t, const int32_t *, const int32_t *, const float *, float,
                              float *, float *, hipStream_t) { return kNo; }
hipError_t launch_gat_aggregate(const SpmmBlock *, int32_t, int32_t, bool, const int32_t *,
                                const int32_t *, const float *, const float *, int32_t, int32_t,
                                float *, bool, float *, hipStream_t) { return kNo; }
hipError_t launch_gat_rows(int32_t, int32_t, int32_t, const float *, const float *, const float *,
                           const float *, const float *, bool, float, float *, float *,
                           hipStream_t) { return kNo; }
hipError_t launch_gat_backward(const SpmmBlock *, int32_t, int32_t, bool, const int32_t *,
                               const int32_t *, const float *, const float *, const float *,
                               const float *, int32_t, int32_t, float, int32_t, float *, float *,
                               hipStream_t) { return kNo; }

}  // namespace digest
