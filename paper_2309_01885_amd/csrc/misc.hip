// Grid, exact objective and lambda_max kernels (gfx950).
#include <algorithm>
#include <cmath>

#include "nt_x3.h"
#include "qe_internal.h"

namespace qe {

// ---------------------------------------------------------------- grid
// Per-row asymmetric min/max grid (Sec. 2.1: uniformly spaced levels per output
// channel; the paper does not print the formula, see qe.h): one workgroup per
// row, min/max reductions (exact in any order), then the scale and zero point
// in fp32.  Entries with H != 0 are excluded (outlier-aware grid, Sec. 4.3).
__global__ __launch_bounds__(256) void grid_minmax_kernel(const float* __restrict__ W,
                                                          const float* __restrict__ H, int64_t p,
                                                          float maxq, float* scale, float* zero)
{
    __shared__ float slo[256], shi[256];
    const int64_t i = blockIdx.x;
    float lo = 0.f, hi = 0.f;
    for (int64_t j = threadIdx.x; j < p; j += blockDim.x) {
        if (H && H[i * p + j] != 0.f) continue;
        const float w = W[i * p + j];
        lo = fminf(lo, w);
        hi = fmaxf(hi, w);
    }
    slo[threadIdx.x] = lo;
    shi[threadIdx.x] = hi;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            slo[threadIdx.x] = fminf(slo[threadIdx.x], slo[threadIdx.x + s]);
            shi[threadIdx.x] = fmaxf(shi[threadIdx.x], shi[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        lo = slo[0];
        hi = shi[0];
        if (lo == 0.f && hi == 0.f) {
            lo = -1.f;
            hi = 1.f;
        }
        const float s = (hi - lo) / maxq;
        scale[i] = s;
        zero[i] = rintf(-lo / s);
    }
}

// ---------------------------------------------------------------- input checks
// Any NaN or infinity among `count` floats sets QE_ERR_NONFINITE.
__global__ __launch_bounds__(256) void nonfinite_scan_kernel(const float* __restrict__ a,
                                                             int64_t count, int vec4, int* status)
{
    const int64_t G = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // exponent field all ones: infinity or NaN
    auto bad = [](float x) { return (int)((__float_as_uint(x) & 0x7f800000u) == 0x7f800000u); };
    int found = 0;
    int64_t tail = 0;
    if (vec4) {
        const f32x4* a4 = reinterpret_cast<const f32x4*>(a);
        const int64_t n4 = count / 4;
        for (int64_t e = tid; e < n4; e += G) {
            const f32x4 v = a4[e];
            found |= bad(v[0]) | bad(v[1]) | bad(v[2]) | bad(v[3]);
        }
        tail = n4 * 4;
    }
    for (int64_t e = tail + tid; e < count; e += G) found |= bad(a[e]);
    if (found) set_status(status, QE_ERR_NONFINITE);
}

qe_status launch_nonfinite_scan(const float* a, int64_t count, int* status, hipStream_t s)
{
    if (!a || count <= 0) return QE_OK;
    const int64_t wgs = std::min<int64_t>(2048, std::max<int64_t>(1, cdiv(count / 4, 256)));
    hipLaunchKernelGGL(nonfinite_scan_kernel, dim3((unsigned)wgs), dim3(256), 0, s, a, count,
                       aligned16(a) ? 1 : 0, status);
    return hipGetLastError() == hipSuccess ? QE_OK : QE_ERR_HIP;
}

qe_status launch_grid_minmax(const float* W, const float* H, int64_t q, int64_t p, int bits,
                             float* scale, float* zero, hipStream_t s)
{
    if (q == 0) return QE_OK;
    hipLaunchKernelGGL(grid_minmax_kernel, dim3((unsigned)q), dim3(256), 0, s, W, H, p,
                       (float)((1 << bits) - 1), scale, zero);
    return hipGetLastError() == hipSuccess ? QE_OK : QE_ERR_HIP;
}

// ---------------------------------------------------------------- exact objective
// <A, A Sigma> for A = What (+ H) - W and for A = W, on the bf16 matrix cores with
// the exact three-way split.  Sigma is symmetric, so with column tiles C
//     <A, A Sigma> = sum_C ( 2 <A_C, sum_{K < C} A_K Sigma_{K,C}> + <A_C, A_C Sigma_{C,C}> ),
// half the products of the full square.  The sum over K needs no common
// accumulator: every workgroup forms A_K Sigma_{K,C} for one row tile, one C and
// a run of at most `chunk` tiles K <= C (twice the tiles before K = C), dots it
// with its tile of A in fp64 at once, and writes one partial; the partials are
// summed in a fixed order.  Both forms share one launch.
//
// Tiles are 256 x 256 (eight waves, nt_tile_x3_wide) or, where those leave the
// chip idle, 128 x 128 (four waves); the runs are as long as the number of
// workgroups allows (see quad_plan).  Rows past the end repeat the last one and
// are left out of the dot product; rows need no 16-byte alignment.
template <bool P2, bool P3>
struct X3Quad {
    const float *p1, *p2, *p3;
    int64_t off, kvalid;          // this thread's row and half stage, from the bases
    __device__ inline X3Quad(const float* q1, const float* q2, const float* q3, int64_t ld, int64_t rows,
                             int64_t row0, int64_t kv)
        : p1(q1), p2(q2), p3(q3),
          off(min(row0 + (int)(threadIdx.x >> 1), rows - 1) * ld + 8 * (threadIdx.x & 1)), kvalid(kv)
    {
    }
    __device__ inline f32x4 at(int64_t e) const
    {
        f32x4 v = *reinterpret_cast<const f32x4a4*>(p1 + e);
        if constexpr (P2) v = v + *reinterpret_cast<const f32x4a4*>(p2 + e);
        if constexpr (P3) v = v - *reinterpret_cast<const f32x4a4*>(p3 + e);
        return v;
    }
    static __device__ inline float one(const float* p1, const float* p2, const float* p3, int64_t e)
    {
        float a = p1[e];
        if constexpr (P2) a = a + p2[e];
        if constexpr (P3) a = a - p3[e];
        return a;
    }
    // a stage inside the row's columns (the row is the constructor's)
    __device__ inline void load_full(int64_t, int64_t k0, X3Stage& st) const
    {
        st.v[0] = at(off + k0);
        st.v[1] = at(off + k0 + 4);
    }
    // any stage: columns from kvalid on read as 0
    __device__ inline void load(int64_t, int64_t k0, X3Stage& st) const
    {
        const int64_t k = k0 + 8 * (threadIdx.x & 1);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            st.v[u >> 2][u & 3] = k + u < kvalid ? one(p1, p2, p3, off + k0 + u) : 0.f;
    }
    __device__ inline void store(uint32_t* op, const X3Stage& st) const { x3_store_row8(op, st); }
};

struct QuadArgs {
    const float *Wh, *H, *W, *Sigma;
    int64_t q, p, tm, tn;         // row tiles, column tiles
    int64_t full;                 // runs of `chunk` tiles over all C
    int64_t units;                // all runs
    int chunk;
    double* partial;              // 2 x units x tm
    const int* status;
};

// One workgroup's unit of form A: rows row0.., columns 256 or 128 from col0, the
// tiles K in [k0, col0) twice and, with `diag`, those of K = C once.
template <int TILE, bool P2, bool P3>
__device__ __forceinline__ double quad_unit(const QuadArgs& a, const float* p1, const float* p2,
                                            const float* p3, int64_t row0, int64_t col0, int64_t k0,
                                            int64_t k1, uint32_t* lds)
{
    constexpr int NI = TILE == 256 ? 4 : 2;
    f32x16 acc[2][NI];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
#pragma unroll 1
    for (int part = 0; part < 2; ++part) {
        const int64_t b = part ? max(k0, col0) : k0, e = part ? k1 : min(k1, col0);
        if (e > b) {
            const X3Quad<P2, P3> A(p1 + b, P2 ? p2 + b : nullptr, P3 ? p3 + b : nullptr, a.p, a.q, row0, e - b);
            const X3Quad<false, false> B(a.Sigma + b, nullptr, nullptr, a.p, a.p, col0, e - b);
            if constexpr (TILE == 256)
                nt_tile_x3_wide(A, row0, B, col0, e - b, lds, acc);
            else if ((e - b) % (2 * kX3KC) == 0)
                nt_tile_x3_full(A, row0, B, col0, e - b, lds, acc);
            else
                nt_tile_x3_edge(A, row0, B, col0, e - b, lds, acc);
        }
        if (part == 0) {
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[mi][ni][v] *= 2.f;
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double d = 0.0;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t r = row0 + (wave >> 1) * 64 + 32 * mi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                const int64_t c = col0 + (wave & 1) * (32 * NI) + 32 * ni + (lane & 31);
                // unconditional loads, all in flight together
                const float av =
                    X3Quad<P2, P3>::one(p1, p2, p3, min(r, a.q - 1) * a.p + min(c, a.p - 1));
                d += (double)av * (double)(r < a.q && c < a.p ? acc[mi][ni][v] : 0.f);
            }
    return d;
}

template <int TILE, bool HASH>
__global__ __launch_bounds__(2 * TILE, TILE == 256 ? 1 : 2) void quad_kernel(QuadArgs a)
{
    if (failed(a.status)) return;
    __shared__ __attribute__((aligned(16))) uint32_t lds[TILE == 256 ? kX3wLdsDw : kX3LdsDw];
    __shared__ double sh[TILE / 32];
    // rows fastest: the workgroups at work at one time share their run of Sigma
    const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t unit = wg / (2 * a.tm), slot = wg % (2 * a.tm);
    if (unit >= a.units) return;                  // uniform: the whole workgroup leaves
    const bool isw = slot >= a.tm;
    const int64_t row0 = (slot - (isw ? a.tm : 0)) * TILE;
    // whole runs first, those of the same K tiles side by side (they share their
    // tiles of A in L2), then the remainders
    const int64_t ch = a.chunk;
    int64_t C, first = 0;
    if (unit < a.full) {
        int64_t u = unit, n;
        for (; u >= (n = a.tn - first - ch + 1); first += ch) u -= n;
        C = first + ch - 1 + u;
    } else {
        int64_t v = unit - a.full, n;
        for (; v >= (n = min(ch - 1, a.tn - first)); first += ch) v -= n;
        C = first + n - 1 - v;
    }
    const int64_t k0 = first * TILE, k1 = min(a.p, min(first + ch, C + 1) * TILE);
    double d = isw ? quad_unit<TILE, false, false>(a, a.W, nullptr, nullptr, row0, C * TILE, k0, k1, lds)
                   : quad_unit<TILE, HASH, true>(a, a.Wh, a.H, a.W, row0, C * TILE, k0, k1, lds);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < TILE / 32; ++w) t += sh[w];
        a.partial[(isw ? a.units * a.tm : 0) + unit * a.tm + row0 / TILE] = t;
    }
}

// Workgroup f: out[f] = the sum of form f's n partials.
__global__ __launch_bounds__(1024) void quad_sum_kernel(const double* partial, int64_t n, double* out,
                                                        const int* status)
{
    if (failed(status)) return;
    __shared__ double sh[16];
    const double* src = partial + blockIdx.x * n;
    double acc = 0.0;
#pragma unroll 4
    for (int64_t e = threadIdx.x; e < n; e += 1024) acc += src[e];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < 16; ++w) t += sh[w];
        out[blockIdx.x] = t;
    }
}

struct QuadPlan {
    int tile, chunk;
    int64_t tm, tn, full, units;
};

// Tile and run length.  256 x 256 tiles (one workgroup per CU) need p to be a
// multiple of 32 and at least 256 units, the others run on 128 x 128 tiles (two
// per CU).  The run minimises, in tiles of K, the work per slot (or the longest
// unit) and kQuadUnit for every unit: its pipeline fill and its tile of A, whose
// 16 us no other workgroup of the CU hides with 256 x 256 tiles (52 us against 37
// us for a tile of K).  4096 x 4096: 1.21 ms as two launches over the full square,
// 0.87 ms with runs of 4, 0.75 ms with runs of 16 (the whole C).

static QuadPlan quad_plan(int64_t q, int64_t p)
{
    QuadPlan best{};
    for (int tile : {256, 128}) {
        if (tile == 256 && p % (2 * kX3KC) != 0) continue;
        const double slots = tile == 256 ? 256.0 : 512.0;
        const double kQuadUnit = tile == 256 ? 1.4 : 0.5;
        double best_cost = 0.0;
        for (int chunk = 1; chunk <= 32; ++chunk) {
            QuadPlan pl{tile, chunk, cdiv(q, tile), cdiv(p, tile), 0, 0};
            for (int64_t C = 0; C < pl.tn; ++C) {
                pl.full += (C + 1) / chunk;
                pl.units += cdiv(C + 1, (int64_t)chunk);
            }
            const double units = 2.0 * (double)(pl.tm * pl.units);
            const double work = (double)(pl.tm * pl.tn) * (double)(pl.tn + 1);
            const double cost = std::max(work / slots, (double)std::min<int64_t>(chunk, pl.tn)) +
                                kQuadUnit * units / slots;
            if (chunk == 1 || cost < best_cost) {
                best = pl;
                best_cost = cost;
            }
            if (chunk == 1 && units < 256.0) break;
        }
        if (tile == 256 && 2 * best.tm * best.units >= 256) break;
    }
    return best;
}

size_t objective_ws_bytes(int64_t q, int64_t p)
{
    const QuadPlan pl = quad_plan(q, p);
    return kStatusBytes + align256(sizeof(double) * 2 * pl.tm * pl.units);
}

qe_status launch_objective(const float* W, const float* Wh, const float* H, const float* Sigma,
                           int64_t q, int64_t p, double* out, void* ws, hipStream_t s)
{
    int* status = static_cast<int*>(ws);
    Ws w(ws);
    const QuadPlan pl = quad_plan(q, p);
    const int64_t n = pl.tm * pl.units;
    double* part = w.take<double>(2 * n);
    const QuadArgs a{Wh, H, W, Sigma, q, p, pl.tm, pl.tn, pl.full, pl.units, pl.chunk, part, status};
    const dim3 grid = grid_xy(2 * n, 2 * pl.tile), block((unsigned)(2 * pl.tile));
    if (pl.tile == 256 && H)
        hipLaunchKernelGGL((quad_kernel<256, true>), grid, block, 0, s, a);
    else if (pl.tile == 256)
        hipLaunchKernelGGL((quad_kernel<256, false>), grid, block, 0, s, a);
    else if (H)
        hipLaunchKernelGGL((quad_kernel<128, true>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((quad_kernel<128, false>), grid, block, 0, s, a);
    hipLaunchKernelGGL(quad_sum_kernel, dim3(2), dim3(1024), 0, s, part, n, out, status);
    return hipGetLastError() == hipSuccess ? QE_OK : QE_ERR_HIP;
}

// ---------------------------------------------------------------- lambda_max
// Power method (Sec. 4.3): v_k = y_{k-1} / ||y_{k-1}|| (v_0 = 1/sqrt(p)),
// y_k = Sigma v_k, lambda_k = v_k . y_k (Rayleigh quotient of the unit v_k).
// One kernel per iteration: every workgroup forms 8 rows of Sigma y_{k-1} (two per
// wavefront, processed together so that each float4 of y_{k-1} serves two rows of
// Sigma; fp64 dot products against y_{k-1} itself), then 1/||y_{k-1}|| from the
// previous iteration's per-workgroup partials (same fixed-order sum in every
// workgroup), applies it once per row, and writes its partials of ||y_k||^2 and
// v_k . y_k.  Workgroup 0 also records
// lambda_{k-1}.  Sigma is read once per iteration: the kernel is bound by
// that stream (HBM or, for Sigma within the die-level cache, that cache).
constexpr int kSymvRows = 8;
constexpr int kLambdaCheck = 32;   // iterations per host check (the stop is still per iteration)

// The per-workgroup partials (|Sv|^2, v'Sv, |v|^2) of one iteration: early() fetches
// this thread's first kEarly of each, before the iteration's own loads are waited
// for, and sum() adds all of them in a fixed order (every thread gets the sums).
struct Partials3 {
    static constexpr int kEarly = 2;
    double v[kEarly][3];
    __device__ inline void early(const double* part, int n)
    {
#pragma unroll
        for (int k = 0; k < kEarly; ++k) {
            const int e = threadIdx.x + 256 * k;
#pragma unroll
            for (int c = 0; c < 3; ++c) v[k][c] = e < n ? part[3 * e + c] : 0.0;
        }
    }
    __device__ inline void sum(const double* part, int n, double (&sh)[4][3], double (&out)[3]) const
    {
        double a[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = v[0][c] + v[1][c];
        for (int e = threadIdx.x + 256 * kEarly; e < n; e += 256)
#pragma unroll
            for (int c = 0; c < 3; ++c) a[c] += part[3 * e + c];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int c = 0; c < 3; ++c) a[c] += __shfl_xor(a[c], o, 64);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int c = 0; c < 3; ++c) sh[threadIdx.x >> 6][c] = a[c];
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 3; ++c) out[c] = ((sh[0][c] + sh[1][c]) + sh[2][c]) + sh[3][c];
    }
};

// Quotient rho = v'Sv / v'v and squared inclusion radius |Sv - rho v|^2 / |v|^2
// (= (|Sv|^2 - (v'Sv)^2 / v'v) / v'v) of one iteration, into lam_hist.
__device__ inline void put_hist(double* lam_hist, int slot, double yy, double vy, double vv)
{
    lam_hist[2 * slot] = vv > 0.0 ? vy / vv : 0.0;
    lam_hist[2 * slot + 1] = vv > 0.0 ? fmax(0.0, yy - vy * vy / vv) / vv : 0.0;
}

// One power iteration y = Sigma v with v = yprev / |S v_prev| (the first: all
// ones / sqrt(p)); the products and the partial sums are fp64, y is stored in
// fp32 for the next iteration.
__global__ __launch_bounds__(256) void power_step_kernel(const float* __restrict__ Sigma,
                                                         int64_t p, const float* __restrict__ yprev,
                                                         const double* __restrict__ pprev,
                                                         int first, int vec4, float* y,
                                                         double* part, double* lam_hist, int slot)
{
    __shared__ double sh[4][3];
    __shared__ double wpart[4][3];
    const int nwg = (int)gridDim.x;
    Partials3 prev;
    prev.early(pprev, first ? 0 : nwg);
    auto wj = [&](int64_t j) -> float { return first ? 1.f : yprev[j]; };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int RW = kSymvRows / 4;            // rows per wavefront
    const int64_t r0 = (int64_t)blockIdx.x * kSymvRows + wave * RW;
    const float* srow[RW];
    bool ok[RW];
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
        ok[rr] = r0 + rr < p;
        srow[rr] = Sigma + (ok[rr] ? r0 + rr : 0) * p;
    }
    double acc[RW];
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) acc[rr] = 0.0;
    int64_t tail = 0;
    if (vec4) {
        const int64_t n4 = p / 4;
#pragma unroll 4
        for (int64_t f = lane; f < n4; f += 64) {
            const f32x4 wv = first ? f32x4{1.f, 1.f, 1.f, 1.f}
                                   : *reinterpret_cast<const f32x4*>(yprev + 4 * f);
#pragma unroll
            for (int rr = 0; rr < RW; ++rr) {
                const f32x4 sv = *reinterpret_cast<const f32x4*>(srow[rr] + 4 * f);
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[rr] += (double)sv[u] * (double)wv[u];
            }
        }
        tail = 4 * n4;
    }
    for (int64_t j = tail + lane; j < p; j += 64) {
        const double wv = (double)wj(j);
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) acc[rr] += (double)srow[rr][j] * wv;
    }
    // v_k = yprev * inv (the first iteration: yprev taken as all ones).  Only now,
    // behind the stream of Sigma: it is not needed before.
    double inv;
    if (first) {
        inv = 1.0 / sqrt((double)p);
    } else {
        double t[3];
        prev.sum(pprev, nwg, sh, t);
        inv = t[0] > 0.0 ? 1.0 / sqrt(t[0]) : 0.0;
        if (blockIdx.x == 0 && threadIdx.x == 0 && slot > 0) put_hist(lam_hist, slot - 1, t[0], t[1], t[2]);
    }
    double pyy = 0.0, pvy = 0.0, pvv = 0.0;
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
        double a = acc[rr];
        for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
        if (!ok[rr]) continue;
        const double yd = a * inv;               // (S v)_r in fp64
        if (lane == 0) y[r0 + rr] = (float)yd;
        const double vr = (double)wj(r0 + rr) * inv;
        pyy += yd * yd;
        pvy += vr * yd;
        pvv += vr * vr;
    }
    if (lane == 0) {
        wpart[wave][0] = pyy;
        wpart[wave][1] = pvy;
        wpart[wave][2] = pvv;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            part[3 * blockIdx.x + c] = ((wpart[0][c] + wpart[1][c]) + wpart[2][c]) + wpart[3][c];
    }
}

// Quotient and radius of the last iteration of a batch.
__global__ __launch_bounds__(256) void power_last_kernel(const double* part, int nwg,
                                                         double* lam_hist, int slot)
{
    __shared__ double sh[4][3];
    Partials3 last;
    last.early(part, nwg);
    double t[3];
    last.sum(part, nwg, sh, t);
    if (threadIdx.x == 0) put_hist(lam_hist, slot, t[0], t[1], t[2]);
}

// ---- the same with Sigma kept on the chip (p <= 4096)
// One launch runs a whole batch of iterations: workgroup b holds rows 8 RW b .. 8 RW b
// + 8 RW - 1 of Sigma in registers (RW rows per wavefront, 4 NC values of each per
// lane; RW = 2 above 2048 channels), so that an iteration moves only y.  y travels
// between the workgroups as 64-bit words of a value and the iteration that made it,
// stored and polled with agent-scope atomics: the word carries its own flag, so no
// other ordering is needed.  Two buffers alternate; a workgroup writes iteration k + 1 only after it has read all of
// k, when every other one has done with k - 1.  The launch is cooperative (all
// workgroups resident), and a wait that lasts kMaxPolls polls gives up: the batch
// then reports it and the call starts over with a launch per iteration of this same
// kernel, where every word is there before it is read: the same sums in the same order,
// so the result does not depend on what else the device was doing.
// Bound by the exchange of y (about 2.7 us an iteration) and, at 4096, by the
// conversions of the fp64 products: 12.7 -> 5.5 us an iteration at 4096 (Sigma, 67 MB,
// streamed before), 6.7 -> 2.0 us at 1025, the call 5.0 -> 2.5 ms and 3.2 -> 1.0 ms.
constexpr int64_t kChipMaxP = 4096;          // 256 workgroups of 128 values per lane

__global__ __launch_bounds__(256) void power_clear_kernel(uint64_t* y, int64_t n, int* gave_up)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < n) y[t] = 0;
    if (t == 0) *gave_up = 0;
}

template <int NC, int RW>
__global__ __launch_bounds__(512, 1) void power_batch_kernel(const float* Sigma, int p, uint64_t* ybuf, int it0,
                                                          int iters, double* part, int* gave_up, int max_polls)
{
    __shared__ __attribute__((aligned(16))) float y[256 * NC];
    __shared__ double wsum[8], wpart[8][3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = RW * (8 * (int)blockIdx.x + wave);
    f32x4 sv[RW][NC];
#pragma unroll
    for (int rr = 0; rr < RW; ++rr)
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int c = 256 * i + 4 * lane;
            const float* src = Sigma + (int64_t)min(r0 + rr, p - 1) * p + c;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (c + 4 <= p) {
                v = *reinterpret_cast<const f32x4a4*>(src);
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (c + e < p) v[e] = src[e];
            }
            sv[rr][i] = v;
        }
    for (int k = 0; k < iters; ++k) {
        const uint32_t tag = (uint32_t)(it0 + k);        // y of iteration tag - 1
        const uint64_t* yin = ybuf + (tag & 1) * (int64_t)kChipMaxP;
        uint64_t* yout = ybuf + ((tag + 1) & 1) * (int64_t)kChipMaxP;
        // this thread's values: all loads of a poll in flight together
        constexpr int NV = (256 * NC + 511) / 512;
        uint64_t w[NV];
        int late = 0;
        if (tag != 0) {
            int polls = 0;
            do {
                late = 0;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int c = threadIdx.x + 512 * v;
                    w[v] = (uint64_t)tag << 32;
                    if (c < p) w[v] = __hip_atomic_load(yin + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int v = 0; v < NV; ++v) late |= (uint32_t)(w[v] >> 32) != tag;
            } while (late && ++polls < max_polls);
        }
        double sq = 0.0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int c = threadIdx.x + 512 * v;
            const float val = tag != 0 ? __uint_as_float((uint32_t)w[v]) : c < p ? 1.f : 0.f;
            if (c < 256 * NC) y[c] = val;
            sq += (double)val * (double)val;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
        if (lane == 0) wsum[wave] = sq;
        if (__syncthreads_or(late)) {                    // uniform: the workgroup leaves
            if (threadIdx.x == 0) atomicExch(gave_up, 1);
            return;
        }
        double yy = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) yy += wsum[w];
        const double inv = yy > 0.0 ? 1.0 / sqrt(yy) : 0.0;
        double acc[RW] = {};
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const f32x4 yv = *reinterpret_cast<const f32x4*>(y + 256 * i + 4 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int rr = 0; rr < RW; ++rr) {
                    // (opaque, or the conversions to fp64 would be hoisted out of the
                    // loop, twice the registers)
                    float a = sv[rr][i][e];
                    asm volatile("" : "+v"(a));
                    acc[rr] += (double)a * (double)yv[e];
                }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int rr = 0; rr < RW; ++rr) acc[rr] += __shfl_xor(acc[rr], o, 64);
        if (lane == 0) {
            double pyy = 0.0, pvy = 0.0, pvv = 0.0;
#pragma unroll
            for (int rr = 0; rr < RW; ++rr) {
                if (r0 + rr >= p) continue;
                const double yd = acc[rr] * inv;         // (S v)_r in fp64
                __hip_atomic_store(yout + r0 + rr,
                                   ((uint64_t)(tag + 1) << 32) | __float_as_uint((float)yd),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const double vr = (double)y[r0 + rr] * inv;
                pyy += yd * yd;
                pvy += vr * yd;
                pvv += vr * vr;
            }
            wpart[wave][0] = pyy;
            wpart[wave][1] = pvy;
            wpart[wave][2] = pvv;
        }
        __syncthreads();                                 // y, wsum and wpart are free again below
        if (threadIdx.x < 3) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < 8; ++w) t += wpart[w][threadIdx.x];
            part[((int64_t)k * gridDim.x + blockIdx.x) * 3 + threadIdx.x] = t;
        }
    }
}

// Quotients and radii of a batch: workgroup k sums iteration k's partials.
__global__ __launch_bounds__(256) void power_hist_kernel(const double* part, int nwg, double* lam_hist)
{
    __shared__ double sh[4][3];
    const double* src = part + (int64_t)blockIdx.x * nwg * 3;
    Partials3 s;
    s.early(src, nwg);
    double t[3];
    s.sum(src, nwg, sh, t);
    if (threadIdx.x == 0) put_hist(lam_hist, blockIdx.x, t[0], t[1], t[2]);
}

static int64_t chip_wgs(int64_t p) { return cdiv(p, p > 2048 ? 16 : 8); }

size_t lambda_ws_bytes(int64_t p)
{
    const int64_t nwg = cdiv(p, kSymvRows);
    size_t b = kStatusBytes + 2 * align256(sizeof(float) * p) +
               2 * align256(sizeof(double) * 3 * nwg) + align256(sizeof(double) * 2 * kLambdaCheck + 8);
    if (p <= kChipMaxP)
        b += align256(sizeof(uint64_t) * 2 * kChipMaxP) +
             align256(sizeof(double) * 3 * chip_wgs(p) * kLambdaCheck);
    return b;
}

// One batch: as one cooperative launch (false if the runtime does not take it), or with
// one launch per iteration.
static bool launch_chip_batch(const float* Sigma, int p, uint64_t* ybuf, int it0, int iters, double* part,
                              int* gave_up, int max_polls, bool coop, hipStream_t s)
{
    const void* f = p <= 512    ? reinterpret_cast<const void*>(power_batch_kernel<2, 1>)
                    : p <= 1024 ? reinterpret_cast<const void*>(power_batch_kernel<4, 1>)
                    : p <= 2048 ? reinterpret_cast<const void*>(power_batch_kernel<8, 1>)
                    : p <= 3072 ? reinterpret_cast<const void*>(power_batch_kernel<12, 2>)
                                : reinterpret_cast<const void*>(power_batch_kernel<16, 2>);
    const dim3 grid((unsigned)chip_wgs(p)), block(512);
    if (coop) {
        void* args[] = {&Sigma, &p, &ybuf, &it0, &iters, &part, &gave_up, &max_polls};
        if (hipLaunchCooperativeKernel(f, grid, block, args, 0, s) == hipSuccess) return true;
        (void)hipGetLastError();
        return false;
    }
    int one = 1;
    for (int b = 0; b < iters; ++b, ++it0, part += 3 * chip_wgs(p)) {
        void* args[] = {&Sigma, &p, &ybuf, &it0, &one, &part, &gave_up, &max_polls};
        if (hipLaunchKernel(f, grid, block, args, 0, s) != hipSuccess) return false;
    }
    return true;
}

qe_status launch_lambda(const float* Sigma, int64_t p, int max_iters, float tol, float* out,
                        void* ws, int max_polls, hipStream_t s)
{
    Ws w(ws);
    const int64_t nwg = cdiv(p, kSymvRows);
    float* y[2] = {w.take<float>(p), w.take<float>(p)};
    double* part[2] = {w.take<double>(3 * nwg), w.take<double>(3 * nwg)};
    double* hist = w.take<double>(2 * kLambdaCheck + 1);  // (rho, radius^2) per iteration; gave_up
    int* const gave_up = reinterpret_cast<int*>(hist + 2 * kLambdaCheck);
    const bool chip = p <= kChipMaxP;
    bool coop = max_polls >= 0;
    uint64_t* ybuf = nullptr;
    double* cpart = nullptr;
    if (chip) {
        ybuf = w.take<uint64_t>(2 * kChipMaxP);
        cpart = w.take<double>(3 * chip_wgs(p) * kLambdaCheck);
    }
    auto clear = [&] {
        hipLaunchKernelGGL(power_clear_kernel, dim3((unsigned)cdiv(2 * kChipMaxP, 256)), dim3(256), 0, s,
                           ybuf, 2 * kChipMaxP, gave_up);
    };
    if (chip) clear();
    const int vec4 = (aligned16(Sigma) && p % 4 == 0) ? 1 : 0;
    double last = 0.0, prev = 0.0, last_r2 = 0.0;
    int it = 0, cur = 0;
    while (it < max_iters) {
        const int batch = std::min(kLambdaCheck, max_iters - it);
        if (chip) {
            if (!launch_chip_batch(Sigma, (int)p, ybuf, it, batch, cpart, gave_up,
                                   coop ? max_polls : kMaxPolls, coop, s)) {
                if (!coop) return QE_ERR_HIP;
                coop = false;                            // not taken: from here launch by launch
                continue;
            }
            hipLaunchKernelGGL(power_hist_kernel, dim3((unsigned)batch), dim3(256), 0, s, cpart,
                               (int)chip_wgs(p), hist);
        } else {
            for (int b = 0; b < batch; ++b) {
                const int nxt = cur ^ 1;
                hipLaunchKernelGGL(power_step_kernel, dim3((unsigned)nwg), dim3(256), 0, s, Sigma, p,
                                   y[cur], part[cur], it + b == 0 ? 1 : 0, vec4, y[nxt], part[nxt],
                                   hist, b);
                cur = nxt;
            }
            hipLaunchKernelGGL(power_last_kernel, dim3(1), dim3(256), 0, s, part[cur], (int)nwg, hist,
                               batch - 1);
        }
        it += batch;
        if (hipGetLastError() != hipSuccess) return QE_ERR_HIP;
        double h[2 * kLambdaCheck + 1];
        if (hipMemcpyAsync(h, hist, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess) return QE_ERR_HIP;
        if (hipStreamSynchronize(s) != hipSuccess) return QE_ERR_HIP;
        if (chip && *reinterpret_cast<const int*>(h + 2 * kLambdaCheck) != 0) {
            if (!coop) return QE_ERR_HIP;
            coop = false;                                // a wait gave up: start over, launch by launch
            it = 0;
            last = 0.0;
            clear();
            continue;
        }
        // the first iteration of the batch whose quotient moved by <= tol relative
        bool done = false;
        for (int b = 0; b < batch && !done; ++b) {
            prev = last;
            last = h[2 * b];
            last_r2 = h[2 * b + 1];
            done = it - batch + b > 0 && last > 0.0 && fabs(last - prev) <= (double)tol * last;
        }
        if (done) break;
    }
    // Upper bound: for v and rho = v'Sv / v'v some eigenvalue of the symmetric
    // Sigma lies within |Sv - rho v| / |v| of rho, and v approximates the
    // leading eigenvector, so rho plus that radius bounds lambda_max from
    // above.  Both come from fp64 sums of the fp64 product S v; a relative
    // 2^-30 covers their rounding, and the result is rounded up to fp32.  The
    // IHT step 1 / (2 lambda) then stays within the Lipschitz bound of Lemma 3.
    const double bound = (last + sqrt(last_r2)) * (1.0 + 0x1p-30);
    float f = (float)bound;
    if ((double)f < bound) f = std::nextafter(f, INFINITY);
    *out = f;
    return QE_OK;
}

}  // namespace qe
