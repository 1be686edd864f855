// Export of a quantized layer for serving: bit-packed codes and the outliers
// in CSR form.  The paper leaves serving kernels out of scope (Sec. 4.3,
// "Structured Outliers"); the layouts are this library's (see qe.h).
#include "qe_internal.h"

namespace qe {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4a1 __attribute__((aligned(1)));
typedef uint32_t u32a1 __attribute__((aligned(1)));

// One thread per 32 codes of a row: two 16-byte loads, BITS whole words out.  Rows
// and words need no alignment (row i starts at byte i * row_bytes).  The last
// codes of a row that fill no 32 are read one by one and end at the row's last
// byte.  Bound by the codes' read and the stream's write: 11008 x 4096 codes at 3
// bits, 62 MB, 77 us with a thread per output byte (up to nine one-byte loads and
// a 64-bit division each), 12 us so.
template <int BITS>
__global__ __launch_bounds__(256) void pack_codes_kernel(const uint8_t* __restrict__ codes, int64_t q,
                                                         int64_t p, int64_t groups, int64_t row_bytes,
                                                         uint8_t* packed)
{
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    const int64_t t = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
    if (t >= q * groups) return;
    // (the quotient in 32 bits where it fits)
    const int64_t i = q * groups < (int64_t(1) << 32) ? (int64_t)((uint32_t)t / (uint32_t)groups) : t / groups;
    const int64_t j0 = 32 * (t - i * groups);
    const uint8_t* src = codes + i * p + j0;
    uint8_t* dst = packed + i * row_bytes + j0 / 8 * BITS;
    uint32_t in[8];
    const int have = (int)min((int64_t)32, p - j0);
    if (have == 32) {
        const u32x4 a = *reinterpret_cast<const u32x4a1*>(src), b = *reinterpret_cast<const u32x4a1*>(src + 16);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            in[u] = a[u];
            in[4 + u] = b[u];
        }
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            in[u] = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * u + e < have) in[u] |= (uint32_t)src[4 * u + e] << (8 * e);
        }
    }
    uint32_t out[BITS + 1];
#pragma unroll
    for (int w = 0; w <= BITS; ++w) out[w] = 0;
#pragma unroll
    for (int c = 0; c < 32; ++c) {
        const uint32_t v = (in[c / 4] >> (8 * (c % 4))) & MASK;
        const int w = c * BITS / 32, sh = c * BITS % 32;
        out[w] |= v << sh;
        if (sh + BITS > 32) out[w + 1] |= v >> (32 - sh);
    }
    if (have == 32) {
#pragma unroll
        for (int w = 0; w < BITS; ++w) *reinterpret_cast<u32a1*>(dst + 4 * w) = out[w];
    } else {
        const int bytes = (have * BITS + 7) / 8;
#pragma unroll
        for (int b = 0; b < 4 * BITS; ++b)
            if (b < bytes) dst[b] = (uint8_t)(out[b / 4] >> (8 * (b % 4)));
    }
}

// CSR of the support entries (ascending linear indices) of H.  The first `entry_wgs`
// workgroups take the entries; the others the row pointers, 16 lanes per row: each
// step of the search narrows the range 17-fold (five dependent loads for 450000
// entries, where one lane's binary search takes 19: the launch 14.7 -> 11.7 us at 11008 x
// 4096 with 450000 entries).
__global__ __launch_bounds__(256) void csr_kernel(const float* __restrict__ H,
                                                  const int64_t* __restrict__ support,
                                                  const int64_t* nnz_p, int64_t cap, int64_t q,
                                                  int64_t p, int entry_wgs, int64_t* rowptr,
                                                  int32_t* cols, float* vals)
{
    int64_t n = *nnz_p;
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (wg < entry_wgs) {
        const bool small = q * p < (int64_t(1) << 32);
        const int64_t G = (int64_t)entry_wgs * blockDim.x;
        for (int64_t e = wg * blockDim.x + threadIdx.x; e < n; e += G) {
            int64_t k = support[e];
            k = k < 0 ? 0 : (k >= q * p ? q * p - 1 : k);
            cols[e] = small ? (int32_t)((uint32_t)k % (uint32_t)p) : (int32_t)(k % p);
            vals[e] = H[k];
        }
        return;
    }
    const int64_t i = (wg - entry_wgs) * 16 + (threadIdx.x >> 4);
    const int g = threadIdx.x & 15;
    const int64_t key = i * p;
    // the first position with support >= key lies in [lo, hi]
    int64_t lo = 0, hi = i <= q ? n : 0;
    while (__any(lo < hi)) {
        // 16 probes that cut [lo, hi) into 17 parts (the same ones again once it is short)
        const int64_t len = hi - lo;
        const int64_t at = lo + (len * (g + 1)) / 17;
        const bool below = len > 0 && at < hi && support[at] < key;
        const uint32_t m = (uint32_t)(__ballot(below) >> (threadIdx.x & 48)) & 0xffffu;
        const int c = __popc(m);                 // probes 0 .. c - 1 lie below the key
        if (len > 0) {
            const int64_t nlo = c > 0 ? lo + (len * c) / 17 + 1 : lo;
            const int64_t nhi = c < 16 ? lo + (len * (c + 1)) / 17 : hi;
            lo = nlo;
            hi = nhi < nlo ? nlo : nhi;
        }
    }
    if (i <= q && g == 0) rowptr[i] = lo;
}

int64_t packed_row_bytes(int64_t p, int bits) { return (p * bits + 7) / 8; }

qe_status launch_pack_codes(const uint8_t* codes, int64_t q, int64_t p, int bits,
                            uint8_t* packed, hipStream_t s)
{
    const int64_t rb = packed_row_bytes(p, bits);
    const int64_t groups = cdiv(p, 32);
    if (q * rb == 0) return QE_OK;
    const dim3 grid = grid_xy(cdiv(q * groups, 256), 256);
#define QE_PACK(B)                                                                               \
    case B:                                                                                      \
        hipLaunchKernelGGL(pack_codes_kernel<B>, grid, dim3(256), 0, s, codes, q, p, groups, rb, \
                           packed);                                                              \
        break
    switch (bits) {
        QE_PACK(1);
        QE_PACK(2);
        QE_PACK(3);
        QE_PACK(4);
        QE_PACK(5);
        QE_PACK(6);
        QE_PACK(7);
        QE_PACK(8);
    }
#undef QE_PACK
    return hipGetLastError() == hipSuccess ? QE_OK : QE_ERR_HIP;
}

qe_status launch_outliers_csr(const float* H, int64_t q, int64_t p, const int64_t* support,
                              const int64_t* nnz, int64_t cap, int64_t* rowptr, int32_t* cols,
                              float* vals, hipStream_t s)
{
    const int entry_wgs = (int)std::min<int64_t>(1024, cdiv(cap, 256));
    hipLaunchKernelGGL(csr_kernel, grid_xy(entry_wgs + cdiv(q + 1, 16), 256), dim3(256), 0, s, H,
                       support, nnz, cap, q, p, entry_wgs, rowptr, cols, vals);
    return hipGetLastError() == hipSuccess ? QE_OK : QE_ERR_HIP;
}

}  // namespace qe
