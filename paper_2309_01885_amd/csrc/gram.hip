// Gram matrix Sigma = X X^T on the matrix cores of gfx950.
//
// Products: by default, on the 256 x 256 tiles, on the fp16 matrix cores with
// every channel scaled by a power of two and split into two fp16 values, three
// products kept per fp32 product (gram_x3w_kernel with F2, see nt_f2.h); on
// the other tiles, or with QE_GRAM_BF16X3, on the bf16 matrix cores with every
// fp32 operand split exactly into three bf16 values and six products kept
// (gram_x3_kernel and gram_x3w_kernel, see nt_x3.h); with QE_GRAM_FP32 on the
// fp32 matrix cores (gram_kernel).  All share the work split and the
// reductions below.
//
// Lemma 1 (Sec. 3.2) needs X only through Sigma, a p x p statistic whose size
// does not grow with the token count n.  Work split: 128 x 128 tiles of the
// upper triangle (ti <= tj) x token splits of at most kSplitTokensMax tokens,
// their count chosen to fill the last round of workgroups (gram_splits).
// Each workgroup sums its split in the fp32 matrix-core accumulators (a
// running sum of at most 32768 products), writes the partial tile to the
// workspace, and a finalize kernel adds the splits in a fixed order in fp64.
// When the split partials would not fit the workspace budget (very large p),
// one workgroup per tile sums all tokens with a two-level accumulator (inner
// sums of 512 tokens added into a second fp32 accumulator) and writes Sigma
// directly.  The lower triangle is
// written as an exact mirror through an LDS transpose.
#include "nt_f2.h"
#include "nt_x3.h"
#include "qe_internal.h"

namespace qe {

constexpr int kInnerChunks = 16;          // two-level mode: 16 x 32 = 512 tokens per inner sum
constexpr int64_t kSplitTokensMax = 32768;  // longest single fp32 running sum allowed
constexpr size_t kSplitBudget = size_t(2) << 30;   // bytes of split partials allowed
constexpr int kTileFloats = kTile * kTile;
constexpr int kTStride = kTile + 1;       // LDS transpose tile row stride

__device__ inline void tri_index(int64_t t, int64_t nt, int64_t& ti, int64_t& tj)
{
    // row ti of the upper triangle starts at ti * nt - ti * (ti - 1) / 2
    const double b = 2.0 * nt + 1.0;
    int64_t r = (int64_t)((b - sqrt(b * b - 8.0 * (double)t)) * 0.5);
    if (r < 0) r = 0;
    auto start = [nt](int64_t i) { return i * nt - i * (i - 1) / 2; };
    while (r > 0 && start(r) > t) --r;
    while (r + 1 < nt && start(r + 1) <= t) ++r;
    ti = r;
    tj = r + (t - start(r));
}

__device__ inline int64_t tri_row_start(int64_t i, int64_t nt) { return i * nt - i * (i - 1) / 2; }

// Tile t of the upper triangle in banded order: bands of 8 tile rows, each
// band ordered by tile column, so that consecutive tiles share their row
// panels (and, within a band, their column panel).
__device__ inline void band_index(int64_t t, int64_t nt, int64_t& ti, int64_t& tj)
{
    int64_t r, c;
    tri_index(t, nt, r, c);
    const int64_t b0 = (r / 8) * 8;
    const int64_t bh = min((int64_t)8, nt - b0);
    const int64_t u = t - tri_row_start(b0, nt);
    const int64_t tri = bh * (bh + 1) / 2;
    if (u < tri) {
        int64_t m = (int64_t)((sqrt(8.0 * (double)u + 1.0) - 1.0) * 0.5);
        while (m > 0 && m * (m + 1) / 2 > u) --m;
        while ((m + 1) * (m + 2) / 2 <= u) ++m;
        tj = b0 + m;
        ti = b0 + (u - m * (m + 1) / 2);
    } else {
        const int64_t v = u - tri;
        tj = b0 + bh + v / bh;
        ti = b0 + v % bh;
    }
}

// Writes rows [r0, r0 + nr) of the 128 x 128 tile (held in LDS as rows
// 0 .. nr-1, row stride kTStride) to Sigma's upper block (ti, tj) and their
// mirror in block (tj, ti).  On a diagonal tile only the entries with
// row <= col are taken and the rest mirrored, so Sigma is exactly symmetric.
// With `accumulate`, the old upper value is added first.
__device__ void write_symmetric(float* tileLds, int64_t ti, int64_t tj, float* Sigma, int64_t p,
                                int accumulate, int r0, int nr)
{
    const int64_t a0 = ti * kTile + r0, b0 = tj * kTile;
    const bool diag = ti == tj;
    for (int e = threadIdx.x; e < nr * kTile; e += blockDim.x) {
        const int r = e / kTile, c = e % kTile;
        const int64_t a = a0 + r, b = b0 + c;
        if (a < p && b < p && (!diag || r0 + r <= c)) {
            float v = tileLds[r * kTStride + c];
            if (accumulate) v += Sigma[a * p + b];
            Sigma[a * p + b] = v;
            tileLds[r * kTStride + c] = v;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nr * kTile; e += blockDim.x) {
        const int c = e / nr, r = e % nr;            // consecutive threads: consecutive a
        const int64_t a = a0 + r, b = b0 + c;
        if (a < p && b < p && (!diag || r0 + r < c)) Sigma[b * p + a] = tileLds[r * kTStride + c];
    }
}

template <bool TRANS, bool TWO_LEVEL>
__global__ __launch_bounds__(256, TWO_LEVEL ? 1 : 2) void gram_kernel(
    const float* __restrict__ X, int64_t p, int64_t n, int64_t nt, int64_t split_len,
    float* __restrict__ out, int accumulate, int x_vec4, const int* status)
{
    if (failed(status)) return;
    __shared__ __attribute__((aligned(16))) float lds[kNTLdsFloats];
    int64_t ti, tj;
    tri_index(blockIdx.x, nt, ti, tj);
    const int64_t k0 = (int64_t)blockIdx.y * split_len;
    const int64_t k1 = min(n, k0 + split_len);

    f32x16 acc[2][2];
    auto run = [&](int64_t kb, int64_t ke) {
        if (TRANS) {
            // X is n x p: element (channel r, token k) at X[k * p + r]
            const ColOp op{X + kb * p, p, p, ke - kb, x_vec4 != 0};
            nt_tile(op, ti * kTile, op, tj * kTile, ke - kb, lds, acc);
        } else {
            const RowOp op{X + kb, n, p, ke - kb, x_vec4 != 0};
            nt_tile(op, ti * kTile, op, tj * kTile, ke - kb, lds, acc);
        }
    };
    if constexpr (TWO_LEVEL) {
        f32x16 outer[2][2];
        zero_acc(outer);
        const int64_t inner = (int64_t)kInnerChunks * kKC;
        for (int64_t kb = k0; kb < k1; kb += inner) {
            zero_acc(acc);
            run(kb, min(k1, kb + inner));
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) outer[a][b] += acc[a][b];
        }
        float* tl = lds;   // reuse the pipeline LDS (nt_tile ended with a barrier)
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    tl[acc_row(mi, v) * kTStride + acc_col(ni)] = outer[mi][ni][v];
        __syncthreads();
        write_symmetric(tl, ti, tj, out, p, accumulate, 0, kTile);
    } else {
        zero_acc(acc);
        run(k0, k1);
        float* dst = out + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kTileFloats;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    dst[acc_row(mi, v) * kTile + acc_col(ni)] = acc[mi][ni][v];
    }
}

// The same work on the bf16 matrix cores with the exact three-way split of
// each fp32 operand (six bf16 products per fp32 product, fp32 accumulation).
// Work items (tile, split) are dealt to the 8 XCDs in contiguous ranges (the
// hardware places workgroup b on XCD b % 8), split-major and in banded tile
// order inside a split, so the workgroups resident on one XCD at a time share
// their X panels through that XCD's L2.
// FULL launches (every 128-row panel inside X, every K range a multiple of
// 32, aligned rows) take the unguarded two-stage-prefetch loop; any other
// shape takes the guarded loop for every tile.
template <bool TRANS, bool TWO_LEVEL, bool FULL>
__global__ __launch_bounds__(256, TWO_LEVEL ? 1 : 2) void gram_x3_kernel(
    const float* __restrict__ X, int64_t p, int64_t n, int64_t nt, int64_t tiles,
    int64_t splits, int64_t split_len, float* __restrict__ out, int accumulate, const int* status)
{
    if (failed(status)) return;
    // the two-level mode also stages the finished 128 x kTStride tile here
    constexpr int kLds = TWO_LEVEL && kTile * kTStride > kX3LdsDw ? kTile * kTStride : kX3LdsDw;
    __shared__ __attribute__((aligned(16))) uint32_t lds[kLds];
    const int64_t items = tiles * splits;
    const int64_t per = cdiv(items, 8);
    const int64_t item = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (item >= items) return;                    // uniform: the whole workgroup leaves
    const int64_t sp = item / tiles;
    int64_t ti, tj;
    band_index(item % tiles, nt, ti, tj);
    const int64_t k0 = sp * split_len;
    const int64_t k1 = min(n, k0 + split_len);

    f32x16 acc[2][2];
    auto run = [&](int64_t kb, int64_t ke) {
        const int64_t K = ke - kb;
        if constexpr (TRANS) {
            const X3Col op{X + kb * p, p, p, K};
            if constexpr (FULL) nt_tile_x3_full<true>(op, ti * kTile, op, tj * kTile, K, lds, acc);
            else nt_tile_x3_edge(op, ti * kTile, op, tj * kTile, K, lds, acc);
        } else {
            const X3Row op{X + kb, n, p, K};
            if constexpr (FULL) nt_tile_x3_full<true>(op, ti * kTile, op, tj * kTile, K, lds, acc);
            else nt_tile_x3_edge(op, ti * kTile, op, tj * kTile, K, lds, acc);
        }
    };
    float* tl = reinterpret_cast<float*>(lds);
    if constexpr (TWO_LEVEL) {
        f32x16 outer[2][2];
        zero_acc(outer);
        const int64_t inner = (int64_t)kInnerChunks * kKC;
        for (int64_t kb = k0; kb < k1; kb += inner) {
            zero_acc(acc);
            run(kb, min(k1, kb + inner));
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) outer[a][b] += acc[a][b];
        }
        // the K loop ended with a barrier: the stage area is free
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    tl[acc_row(mi, v) * kTStride + acc_col(ni)] = outer[mi][ni][v];
        __syncthreads();
        write_symmetric(tl, ti, tj, out, p, accumulate, 0, kTile);
    } else {
        zero_acc(acc);
        run(k0, k1);
        const int64_t slot = tri_row_start(ti, nt) + (tj - ti);
        float* dst = out + (sp * tiles + slot) * kTileFloats;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    dst[acc_row(mi, v) * kTile + acc_col(ni)] = acc[mi][ni][v];
    }
}

// Split mode on 256 x 256 tiles: one workgroup of eight waves per CU, each
// wave a 64 x 128 block, so that every staged operand value feeds twice the
// matrix-core work of the 128 x 128 tile (half the split work, LDS traffic
// and L2 traffic per product), with the operand reads pipelined through three
// LDS stage buffers (nt_tile_x3_wide).  Used when every 256-row panel lies
// inside X (p a multiple of 256, aligned rows, token ranges multiples of 32),
// in either layout (channel-major rows through X3Row, token-major through
// X3Col).  Each wave's 64 x 128 block lies in one 128 x 128 tile of the
// upper triangle, so the partials use the same slots as gram_x3_kernel and
// the same finalize.
constexpr int kWide = 256;

__device__ inline void band_index_wide(int64_t t, int64_t nt, int64_t& ti, int64_t& tj)
{
    // bands of 4 tile rows: about the 32 workgroups an XCD holds at a time
    int64_t r, c;
    tri_index(t, nt, r, c);
    const int64_t b0 = (r / 4) * 4;
    const int64_t bh = min((int64_t)4, nt - b0);
    const int64_t u = t - tri_row_start(b0, nt);
    const int64_t tri = bh * (bh + 1) / 2;
    if (u < tri) {
        int64_t m = (int64_t)((sqrt(8.0 * (double)u + 1.0) - 1.0) * 0.5);
        while (m > 0 && m * (m + 1) / 2 > u) --m;
        while ((m + 1) * (m + 2) / 2 <= u) ++m;
        tj = b0 + m;
        ti = b0 + (u - m * (m + 1) / 2);
    } else {
        const int64_t v = u - tri;
        tj = b0 + bh + v / bh;
        ti = b0 + v % bh;
    }
}

// DIRECT: one token range per launch (n <= kSplitTokensMax, a single fp32
// running sum), written to Sigma itself (with accumulate) through the same
// LDS-transposed symmetric writes as the two-level mode, 128 x 128 quadrant
// by quadrant; the large-p replacement of the two-level mode for streamed
// token chunks.
//
// F2: the two-way fp16 split of nt_f2.h, channel i scaled by 2^chexp[i] on the
// way in and every sum scaled back by 2^-(chexp[i] + chexp[j]) on the way out
// (exact); otherwise the three-way bf16 split of nt_x3.h (chexp unused).
//
// EDGE (F2 only): p is no multiple of 256, or token counts are none of 32, or
// channel-major rows are not 16-byte aligned.  The tiles then reach past p;
// channels there take some other channel's values (in bounds), their sums are
// not stored, and tokens past the end read as 0.  Token-major loads guard
// themselves through their descriptor in either case.
template <bool DIRECT, bool TRANS, bool F2, bool EDGE>
__global__ __launch_bounds__(512, 1) void gram_x3w_kernel(
    const float* __restrict__ X, int64_t p, int64_t n, int64_t ntw, int64_t tiles_w, int64_t nt,
    int64_t tiles, int64_t splits, int64_t split_len, float* __restrict__ out, int accumulate,
    const int* __restrict__ chexp, const int* status)
{
    if (failed(status)) return;
    // the direct mode also stages a finished 128 x kTStride quadrant here
    static_assert(kTile * kTStride <= 3 * kF2BufDw && kTile * kTStride <= kX3wLdsDw, "quadrant fits");
    __shared__ __attribute__((aligned(16))) uint32_t lds[F2 ? (TRANS ? 4 : 3) * kF2BufDw : kX3wLdsDw];
    const int64_t items = tiles_w * splits;
    const int64_t per = cdiv(items, 8);
    const int64_t item = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (item >= items) return;                    // uniform: the whole workgroup leaves
    const int64_t sp = item / tiles_w;
    int64_t ti, tj;
    band_index_wide(item % tiles_w, ntw, ti, tj);
    const int64_t k0 = sp * split_len;
    const int64_t kv = min(n, k0 + split_len) - k0;
    const int64_t K = EDGE ? cdiv(kv, 2 * kX3KC) * (2 * kX3KC) : kv;
    // exponent of channel c (EDGE: those past the end repeat the last one)
    auto cexp = [&](int64_t c) { return chexp[EDGE ? min(c, p - 1) : c]; };
    f32x16 acc[2][4];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    if constexpr (F2 && TRANS) {
        // X is n x p; this thread stages channel t / 2 of both panels (eight
        // tokens, buffer loads); four stage buffers
        const int r = threadIdx.x >> 1;
        const F2ColB<EDGE> A{X + k0 * p, p, ldexpf(1.f, cexp(ti * kWide + r)), kv};
        const F2ColB<EDGE> B{X + k0 * p, p, ldexpf(1.f, cexp(tj * kWide + r)), kv};
        nt_tile_f2_wide<4>(A, ti * kWide, B, tj * kWide, K, lds, acc);
    } else if constexpr (F2 && EDGE) {
        const int r = threadIdx.x >> 2;
        const F2RowQE A(X + k0, n, ldexpf(1.f, cexp(ti * kWide + r)),
                        ldexpf(1.f, cexp(ti * kWide + r + 128)), p, ti * kWide, kv);
        const F2RowQE B(X + k0, n, ldexpf(1.f, cexp(tj * kWide + r)),
                        ldexpf(1.f, cexp(tj * kWide + r + 128)), p, tj * kWide, kv);
        nt_tile_f2_wide<3>(A, ti * kWide, B, tj * kWide, K, lds, acc);
    } else if constexpr (F2) {
        // this thread stages channels t / 4 and t / 4 + 128 of both panels
        // (four tokens each); three stage buffers, which keep the loop free of
        // register spills
        const int r = threadIdx.x >> 2;
        const F2RowQ A{X + k0, n, {ldexpf(1.f, chexp[ti * kWide + r]),
                                   ldexpf(1.f, chexp[ti * kWide + r + 128])}};
        const F2RowQ B{X + k0, n, {ldexpf(1.f, chexp[tj * kWide + r]),
                                   ldexpf(1.f, chexp[tj * kWide + r + 128])}};
        nt_tile_f2_wide<3>(A, ti * kWide, B, tj * kWide, K, lds, acc);
    } else if constexpr (TRANS) {
        // X is n x p: element (channel r, token k) at X[k * p + r]
        const X3Col op{X + k0 * p, p, 0, K};
        nt_tile_x3_wide(op, ti * kWide, op, tj * kWide, K, lds, acc);
    } else {
        const X3Row op{X + k0, n, 0, K};
        nt_tile_x3_wide(op, ti * kWide, op, tj * kWide, K, lds, acc);
    }
    // wave (wm, wn): rows 64 wm .. of the tile, columns 128 wn ..
    const int wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t qi = 2 * ti + wm / 2, qj = 2 * tj + wn;
    const int lane = threadIdx.x & 63;
    const int r0 = (wm & 1) * 64;
    if constexpr (F2) {
        int ec[4];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) ec[ni] = cexp(tj * kWide + wn * 128 + 32 * ni + (lane & 31));
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int er = cexp(ti * kWide + wm * 64 + 32 * mi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3));
#pragma unroll
                for (int ni = 0; ni < 4; ++ni) acc[mi][ni][v] = ldexpf(acc[mi][ni][v], -(er + ec[ni]));
            }
    }
    if constexpr (DIRECT) {
        // the K loop ended with a barrier: its LDS holds a 128 x kTStride tile
        float* tl = reinterpret_cast<float*>(lds);
#pragma unroll 1
        for (int quad = 0; quad < 4; ++quad) {
            const int a = quad >> 1, b = quad & 1;          // rows 128 a.., columns 128 b..
            const int64_t gi = 2 * ti + a, gj = 2 * tj + b;
            if (gi > gj || (EDGE && gj >= nt)) continue;     // uniform across the workgroup
            if (wm / 2 == a && wn == b) {
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            tl[(r0 + 32 * mi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * kTStride +
                               32 * ni + (lane & 31)] = acc[mi][ni][v];
            }
            __syncthreads();
            write_symmetric(tl, gi, gj, out, p, accumulate, 0, kTile);
            __syncthreads();
        }
        return;
    }
    // below the diagonal of a diagonal tile, or past the last 128 channels
    if (qi > qj || (EDGE && qj >= nt)) return;
    float* dst = out + (sp * tiles + tri_row_start(qi, nt) + (qj - qi)) * kTileFloats;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                dst[(r0 + 32 * mi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * kTile + 32 * ni +
                    (lane & 31)] = acc[mi][ni][v];
}

// Adds the split partial tiles in fixed split order (fp64) and writes Sigma.
// Workgroup (tile, y): rows [ROWS y, ROWS (y + 1)) of the tile, one float4 column
// group per thread and pass, eight splits in flight.  ROWS = 32 keeps the
// mirrored writes in whole 128-byte lines; few tiles (small p, many splits) take
// ROWS = 8 for four times the workgroups and a quarter of the serial loads: 512
// channels x 64 splits 18.4 us with ROWS = 32 and four splits in flight.
template <int ROWS>
__global__ __launch_bounds__(256) void gram_finalize_kernel(const float* __restrict__ parts,
                                                            int64_t ntiles, int splits,
                                                            int64_t nt, float* Sigma, int64_t p,
                                                            int accumulate, const int* status)
{
    if (failed(status)) return;
    __shared__ float tl[ROWS * kTStride];
    int64_t ti, tj;
    tri_index(blockIdx.x, nt, ti, tj);
    const int r0 = (int)blockIdx.y * ROWS;
    const float* src0 = parts + (int64_t)blockIdx.x * kTileFloats + r0 * kTile;
    const int64_t sstride = ntiles * kTileFloats;
#pragma unroll
    for (int u = 0; u < ROWS * kTile / 4 / 256; ++u) {
        const int f = threadIdx.x + 256 * u;
        const int r = f / (kTile / 4), c = 4 * (f % (kTile / 4));
        const float* src = src0 + r * kTile + c;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll 8
        for (int sp = 0; sp < splits; ++sp) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(src + sp * sstride);
            s0 += (double)v[0];
            s1 += (double)v[1];
            s2 += (double)v[2];
            s3 += (double)v[3];
        }
        float* d = tl + r * kTStride + c;
        d[0] = (float)s0;
        d[1] = (float)s1;
        d[2] = (float)s2;
        d[3] = (float)s3;
    }
    __syncthreads();
    write_symmetric(tl, ti, tj, Sigma, p, accumulate, r0, ROWS);
}

// Sigma_jj += damp * mean_j(Sigma_jj): one workgroup, fp64 mean.
__global__ __launch_bounds__(256) void damp_kernel(float* Sigma, int64_t p, float damp,
                                                   const int* status)
{
    if (failed(status)) return;
    __shared__ double sh[256];
    double s = 0.0;
    for (int64_t j = threadIdx.x; j < p; j += blockDim.x) s += (double)Sigma[j * p + j];
    const double total = block_sum_f64(s, sh);
    const float add = (float)((double)damp * (total / (double)p));
    for (int64_t j = threadIdx.x; j < p; j += blockDim.x) Sigma[j * p + j] += add;
}

// Channel exponents of the fp16 split: e with the channel's largest |x| times
// 2^e in [2^14, 2^15) (frexp: amax = f 2^ex, f in [1/2, 1)), at most 127 (2^e
// a normal float; e >= -113 holds for any finite amax); 0 for an all-zero or
// non-finite channel (a non-finite value reaches Sigma as in fp32).
__device__ inline int chan_exp(float amax)
{
    if (!(amax > 0.f) || !isfinite(amax)) return 0;
    int ex;
    (void)frexpf(amax, &ex);
    return min(15 - ex, 127);
}

__device__ inline float absmax4(float m, f32x4 v)
{
    return fmaxf(m, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
}

// Channel-major X (p x n): workgroup (channel, slice y of the tokens).  One slice
// writes the channel's exponent, several their largest |x| to part[y * p + channel];
// chan_exp_np_kernel reduces those.  Rows need no alignment beyond their four bytes.
__global__ __launch_bounds__(256) void chan_exp_pn_kernel(const float* __restrict__ X, int64_t n,
                                                          int64_t slice, int* __restrict__ chexp,
                                                          float* __restrict__ part, const int* status)
{
    if (failed(status)) return;
    __shared__ float sh[4];
    const int64_t t0 = blockIdx.y * slice, len = min(slice, n - t0);
    const float* row = X + (int64_t)blockIdx.x * n + t0;
    float m = 0.f;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < len / 4; i += 256)
        m = absmax4(m, *reinterpret_cast<const f32x4a4*>(row + 4 * i));
    if (threadIdx.x < len % 4) m = fmaxf(m, fabsf(row[len / 4 * 4 + threadIdx.x]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x != 0) return;
    m = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
    if (gridDim.y == 1)
        chexp[blockIdx.x] = chan_exp(m);
    else
        part[blockIdx.y * gridDim.x + blockIdx.x] = m;
}

// Token-major X (n x p): workgroup (column block of 256, token slice y), lane l of
// each wave four columns; wave w takes the tokens 4 y + w, 4 (y + slices) + w, ...
// and the waves' largest |x| go to part[y * p + column]; chan_exp_np_kernel
// reduces over the slices.  Rows need no alignment beyond their four bytes.
__global__ __launch_bounds__(256) void chan_absmax_np_kernel(const float* __restrict__ X, int64_t p,
                                                             int64_t n, float* __restrict__ part,
                                                             const int* status)
{
    if (failed(status)) return;
    __shared__ f32x4 sh[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 256 + 4 * lane;
    const int64_t step = 4 * (int64_t)gridDim.y;
    float m[4] = {0.f, 0.f, 0.f, 0.f};
    if (c + 4 <= p) {
#pragma unroll 8
        for (int64_t t = 4 * (int64_t)blockIdx.y + wave; t < n; t += step) {
            const f32x4 v = *reinterpret_cast<const f32x4a4*>(X + t * p + c);
#pragma unroll
            for (int u = 0; u < 4; ++u) m[u] = fmaxf(m[u], fabsf(v[u]));
        }
    } else if (c < p) {
        for (int64_t t = 4 * (int64_t)blockIdx.y + wave; t < n; t += step)
#pragma unroll
            for (int u = 0; u < 3; ++u)
                if (c + u < p) m[u] = fmaxf(m[u], fabsf(X[t * p + c + u]));
    }
    sh[wave][lane] = f32x4{m[0], m[1], m[2], m[3]};
    __syncthreads();
    const int k = threadIdx.x;                         // channel of the block
    const int64_t cc = (int64_t)blockIdx.x * 256 + k;
    if (cc >= p) return;
    float best = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) best = fmaxf(best, sh[w][k >> 2][k & 3]);
    part[blockIdx.y * p + cc] = best;
}

// Workgroup: 64 channels, wave w every fourth slice.
__global__ __launch_bounds__(256) void chan_exp_np_kernel(const float* __restrict__ part, int64_t p,
                                                          int slices, int* __restrict__ chexp,
                                                          const int* status)
{
    if (failed(status)) return;
    __shared__ float sh[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * 64 + lane;
    float m = 0.f;
    if (j < p) {
#pragma unroll 8
        for (int y = wave; y < slices; y += 4) m = fmaxf(m, part[y * p + j]);
    }
    sh[wave][lane] = m;
    __syncthreads();
    if (wave == 0 && j < p)
        chexp[j] = chan_exp(fmaxf(fmaxf(sh[0][lane], sh[1][lane]), fmaxf(sh[2][lane], sh[3][lane])));
}

// Token slices of chan_absmax_np_kernel: about 2048 workgroups, at most 512 slices
// (the partials then hold at most 8 MB), and at least 256 tokens a slice, or 64
// where that leaves fewer than 256 workgroups.
static int64_t chan_slices(int64_t p, int64_t n)
{
    const int64_t blocks = cdiv(p, 256);
    const int64_t few = std::min(cdiv(n, 64), cdiv(256, blocks));
    return std::max<int64_t>(
        1, std::min<int64_t>(std::min<int64_t>(512, 2048 / blocks), std::max(cdiv(n, 256), few)));
}

// Token slices of chan_exp_pn_kernel: one workgroup per channel where channels fill the
// chip, else about 1024 of them, at least 16384 tokens a slice (no more slices than
// chan_slices gives, whose partials they share).
static int64_t chan_slices_pn(int64_t p, int64_t n)
{
    return p >= 512 ? 1 : std::max<int64_t>(1, std::min<int64_t>(cdiv(1024, p), n / 16384));
}

// Workspace of the channel exponents: p ints and the token-major partials (room for
// as many slices as with 1024 channels a workgroup, the layout's documented size).
static size_t chan_ws_bytes(int64_t p, int64_t n)
{
    const int64_t wide = std::max<int64_t>(
        1, std::min<int64_t>(std::min<int64_t>(512, 2048 / cdiv(p, 1024)), cdiv(n, 256)));
    return align256((size_t)p * sizeof(int)) +
           align256((size_t)std::max(wide, chan_slices(p, n)) * p * sizeof(float));
}

// Number of token splits, or 0 for the two-level direct mode.
//
// The tile kernels hold one workgroup per slot (256 slots for the 256 x 256
// tiles at one workgroup per CU, 512 for the 128 x 128 tiles at two, on the 256
// CUs of the MI355X), so a launch of items = tiles x splits workgroups of
// ceil(n / splits) tokens takes ceil(items / slots) rounds.  The count chosen
// minimises, in units of one workgroup's time per token, rounds x (tokens per
// split + a fixed cost per workgroup) + the finalize's reads of the partials,
// over the counts whose splits hold at most tokens_max tokens and whose
// partials fit kSplitBudget; ties keep the fewer splits.
constexpr int64_t kGramSlotsWide = 256, kGramSlotsNarrow = 512;
constexpr double kGramWgCostTokens = 32.0;        // prologue, pipeline fill, partial-tile store
constexpr double kGramFinalizeTokensPerTile = 0.11;   // one 64 KB partial tile read in finalize

static int64_t gram_splits(int64_t p, int64_t n, bool wide, int64_t tokens_max)
{
    const int64_t nt = cdiv(p, kTile);
    const int64_t tiles = nt * (nt + 1) / 2;
    const int64_t ntw = cdiv(p, kWide);
    const int64_t items = wide ? ntw * (ntw + 1) / 2 : tiles;
    const int64_t slots = wide ? kGramSlotsWide : kGramSlotsNarrow;
    const int64_t s_min = cdiv(n, tokens_max);
    const int64_t s_max = std::min<int64_t>(
        (int64_t)(kSplitBudget / ((size_t)tiles * kTileFloats * sizeof(float))), cdiv(n, kKC));
    if (s_min > s_max) return 0;
    int64_t best = s_min;
    double best_cost = 0.0;
    for (int64_t sp = s_min; sp <= s_max; ++sp) {
        const int64_t len = cdiv(cdiv(n, sp), kKC) * kKC;
        const int64_t used = cdiv(n, len);
        const double cost = (double)cdiv(items * used, slots) * ((double)len + kGramWgCostTokens) +
                            kGramFinalizeTokensPerTile * (double)(used * tiles);
        if (sp == s_min || cost < best_cost) {
            best = sp;
            best_cost = cost;
        }
        // no count from here on costs less than rounds and partials that waste nothing
        // (long token ranges of few channels have thousands of counts)
        if ((double)items / (double)slots * ((double)n + kGramWgCostTokens * (double)used) +
                kGramFinalizeTokensPerTile * (double)(used * tiles) >
            best_cost)
            break;
    }
    return best;
}

// Token-major X with a token count that is not a multiple of 32 is taken as
// an aligned part on the 256 x 256 tiles and a short tail (launch_gram), where
// those tiles need aligned token ranges.
constexpr int64_t kTokAlign = 2 * kX3KC;

// Which calls take the fp16 split on the 256 x 256 tiles.  Shapes of whole tiles and
// stages always do.  The others do from the amount of work on (p^2 n) from which the pass
// for the channel scales and the padding to 256 channels cost less than the
// 128 x 128 tiles of the bf16 split lose (times in us, 128 x 128 tiles and here):
//  - those tiles' guarded loop, the most of them: from 3e9 on (1100 x 2049 token-major
//    49 and 48, 700 x 8193 68 and 58, 4544 x 16384 3880 and 1320; below, 995 x 2049
//    44 and 50, 896 x 993 33 and 42);
//  - their unguarded loop (p a multiple of 128, whole stages, aligned rows), twice as
//    fast: from 1e10 on (896 x 8192 55 and 56, 1152 x 8192 78 and 70, 640 x 16384 57
//    and 61), and never at p = 384, where both do the same number of products and the
//    scale pass comes on top (384 x 180000 198 and 241).
constexpr double kF2Guarded = 3e9, kF2Unguarded = 1e10;

static bool gram_f2(int64_t p, int64_t n, int layout, bool x_vec4)
{
    // (the token-major loader's buffer offsets are 32-bit)
    if ((layout & (QE_GRAM_FP32 | QE_GRAM_BF16X3)) != 0 || p > (int64_t(1) << 24)) return false;
    const bool stages = x_vec4 && n % kTokAlign == 0;
    // (token-major rows of whole tiles: only the last stage is short)
    if (p % kWide == 0 && (stages || (layout == QE_LAYOUT_NP && x_vec4 && n > kTokAlign))) return true;
    const double work = (double)p * (double)p * (double)n;
    if (p % kTile == 0 && p % kWide != 0 && stages) return p > 3 * kTile && work >= kF2Unguarded;
    return p > kTile && work >= kF2Guarded;
}

// Token splits of a call.  Work that would do for the fp16 split but runs on the bf16
// split's unguarded tiles keeps its running sums as short as they would be there: the
// six products of the bf16 split round twice as often, 384 x 180000 is 1.1e-6 off
// (Frobenius) with 2144 tokens in a sum, 3.4e-7 with 704 and 6% more time.
constexpr int64_t kShortSum = 1024;

static int64_t gram_call_splits(int64_t p, int64_t n, int layout, bool f2)
{
    if (!f2 && (layout & (QE_GRAM_FP32 | QE_GRAM_BF16X3)) == 0 && p % kWide != 0 && p > kTile &&
        (double)p * (double)p * (double)n >= kF2Guarded) {
        const int64_t splits = gram_splits(p, n, false, kShortSum);
        if (splits != 0) return splits;          // (0: their partials would not fit)
    }
    return gram_splits(p, n, f2 || p % kWide == 0, kSplitTokensMax);
}

static size_t gram_ws_one(int64_t p, int64_t n)
{
    const int64_t nt = cdiv(p, kTile);
    const int64_t tiles = nt * (nt + 1) / 2;
    // whatever the layout, the flags and X's alignment choose
    int64_t splits = 0;
    for (bool aligned : {false, true}) {
        const bool f2 = gram_f2(p, n, QE_LAYOUT_PN, aligned);
        splits = std::max(splits, gram_call_splits(p, n, QE_LAYOUT_PN, f2));
    }
    splits = std::max(splits, gram_call_splits(p, n, QE_GRAM_BF16X3, false));
    return kStatusBytes + align256((size_t)splits * tiles * kTileFloats * sizeof(float)) +
           chan_ws_bytes(p, n);
}

size_t gram_ws_bytes(int64_t p, int64_t n)
{
    size_t b = gram_ws_one(p, n);
    if (n > kTokAlign && n % kTokAlign != 0)
        b = std::max(b, std::max(gram_ws_one(p, n - n % kTokAlign), gram_ws_one(p, n % kTokAlign)));
    return b;
}

// 16-byte loads need an aligned base and a row stride that keeps them aligned.
static bool x_vec4(const float* X, int64_t p, int64_t n, bool trans)
{
    return aligned16(X) && (trans ? p : n) % 4 == 0;
}

static qe_status launch_gram_one(const float* X, int64_t p, int64_t n, int layout, float* Sigma,
                                 int accumulate, float damp, void* ws, hipStream_t s);

qe_status launch_gram(const float* X, int64_t p, int64_t n, int layout, float* Sigma,
                      int accumulate, float damp, void* ws, hipStream_t s)
{
    const bool trans = (layout & ~(QE_GRAM_FP32 | QE_GRAM_BF16X3)) == QE_LAYOUT_NP;
    const bool whole = gram_f2(p, n, layout, x_vec4(X, p, n, trans)) &&
                       (n <= kSplitTokensMax || gram_call_splits(p, n, layout, true) != 0);
    if (trans && !(layout & QE_GRAM_FP32) && !whole && p % kWide == 0 && n > kTokAlign &&
        n % kTokAlign != 0) {
        // token rows are contiguous: the tail is X's last n % 32 token rows
        const int64_t tail = n % kTokAlign, main = n - tail;
        const qe_status st = launch_gram_one(X, p, main, layout, Sigma, accumulate, 0.f, ws, s);
        if (st != QE_OK) return st;
        return launch_gram_one(X + main * p, p, tail, layout, Sigma, 1, damp, ws, s);
    }
    return launch_gram_one(X, p, n, layout, Sigma, accumulate, damp, ws, s);
}

static qe_status launch_gram_one(const float* X, int64_t p, int64_t n, int layout, float* Sigma,
                                 int accumulate, float damp, void* ws, hipStream_t s)
{
    int* status = static_cast<int*>(ws);
    const int64_t nt = cdiv(p, kTile);
    const int64_t tiles = nt * (nt + 1) / 2;
    const bool fp32 = (layout & QE_GRAM_FP32) != 0;
    const bool trans = (layout & ~(QE_GRAM_FP32 | QE_GRAM_BF16X3)) == QE_LAYOUT_NP;
    const bool vec4 = x_vec4(X, p, n, trans);
    const bool f2 = gram_f2(p, n, layout, vec4);
    const int64_t splits = gram_call_splits(p, n, layout, f2);
    // split length: a multiple of the K chunk, at most kSplitTokensMax
    const int64_t split_len = splits == 0 ? n : cdiv(cdiv(n, splits), kKC) * kKC;
    const int64_t used = splits == 0 ? 1 : cdiv(n, split_len);
    float* parts = reinterpret_cast<float*>(static_cast<char*>(ws) + kStatusBytes);
    float* dst = splits == 0 ? Sigma : parts;
    // channel exponents (fp16 split) after the split partials
    char* const chws = static_cast<char*>(ws) + kStatusBytes +
                       align256((size_t)splits * tiles * kTileFloats * sizeof(float));
    int* const chexp = reinterpret_cast<int*>(chws);
    float* const chpart = reinterpret_cast<float*>(chws + align256((size_t)p * sizeof(int)));
    if (fp32) {
        dim3 grid((unsigned)tiles, (unsigned)used);
        if (splits == 0) {
            if (trans)
                hipLaunchKernelGGL((gram_kernel<true, true>), grid, dim3(256), 0, s, X, p, n, nt,
                                   n, Sigma, accumulate, vec4 ? 1 : 0, status);
            else
                hipLaunchKernelGGL((gram_kernel<false, true>), grid, dim3(256), 0, s, X, p, n, nt,
                                   n, Sigma, accumulate, vec4 ? 1 : 0, status);
        } else {
            if (trans)
                hipLaunchKernelGGL((gram_kernel<true, false>), grid, dim3(256), 0, s, X, p, n, nt,
                                   split_len, parts, accumulate, vec4 ? 1 : 0, status);
            else
                hipLaunchKernelGGL((gram_kernel<false, false>), grid, dim3(256), 0, s, X, p, n,
                                   nt, split_len, parts, accumulate, vec4 ? 1 : 0, status);
        }
    } else {
        const unsigned grid = (unsigned)(8 * cdiv(tiles * used, 8));
        // every panel inside X, every K range a multiple of 32 (split_len is)
        const bool full = vec4 && p % kTile == 0 && n % (2 * kX3KC) == 0;
#define QE_GRAM_X3(T, L, F)                                                                     \
    hipLaunchKernelGGL((gram_x3_kernel<T, L, F>), dim3(grid), dim3(256), 0, s, X, p, n, nt, tiles, \
                       used, split_len, dst, accumulate, status)
        const bool two = splits == 0;
        const bool aligned = full && p % kWide == 0;
        if ((aligned || f2) && (!two || n <= kSplitTokensMax)) {
            const int64_t ntw = cdiv(p, kWide);
            const int64_t tiles_w = ntw * (ntw + 1) / 2;
            const dim3 grid((unsigned)(8 * cdiv(tiles_w * used, 8)));
            if (f2) {
                if (trans) {
                    const int64_t sl = chan_slices(p, n);
                    hipLaunchKernelGGL(chan_absmax_np_kernel,
                                       dim3((unsigned)cdiv(p, 256), (unsigned)sl), dim3(256), 0, s,
                                       X, p, n, chpart, status);
                    hipLaunchKernelGGL(chan_exp_np_kernel, dim3((unsigned)cdiv(p, 64)), dim3(256),
                                       0, s, chpart, p, (int)sl, chexp, status);
                } else {
                    const int64_t slice = cdiv(cdiv(n, chan_slices_pn(p, n)), 4) * 4;
                    const int64_t sl = cdiv(n, slice);
                    hipLaunchKernelGGL(chan_exp_pn_kernel, dim3((unsigned)p, (unsigned)sl), dim3(256), 0, s,
                                       X, n, slice, chexp, chpart, status);
                    if (sl > 1)
                        hipLaunchKernelGGL(chan_exp_np_kernel, dim3((unsigned)cdiv(p, 64)), dim3(256),
                                           0, s, chpart, p, (int)sl, chexp, status);
                }
                if (hipGetLastError() != hipSuccess) return QE_ERR_HIP;
            }
#define QE_GRAM_X3W(T, F, E)                                                                    \
    do {                                                                                        \
        if (two)                                                                                \
            hipLaunchKernelGGL((gram_x3w_kernel<true, T, F, E>), grid, dim3(512), 0, s, X, p, n,   \
                               ntw, tiles_w, nt, tiles, (int64_t)1, n, Sigma, accumulate,       \
                               chexp, status);                                                  \
        else                                                                                    \
            hipLaunchKernelGGL((gram_x3w_kernel<false, T, F, E>), grid, dim3(512), 0, s, X, p, n,  \
                               ntw, tiles_w, nt, tiles, used, split_len, parts, accumulate,     \
                               chexp, status);                                                  \
    } while (0)
            if (f2 && aligned && trans) QE_GRAM_X3W(true, true, false);
            else if (f2 && aligned) QE_GRAM_X3W(false, true, false);
            else if (f2 && trans) QE_GRAM_X3W(true, true, true);
            else if (f2) QE_GRAM_X3W(false, true, true);
            else if (trans) QE_GRAM_X3W(true, false, false);
            else QE_GRAM_X3W(false, false, false);
#undef QE_GRAM_X3W
        } else if (trans) {
            if (two) { if (full) QE_GRAM_X3(true, true, true); else QE_GRAM_X3(true, true, false); }
            else { if (full) QE_GRAM_X3(true, false, true); else QE_GRAM_X3(true, false, false); }
        } else {
            if (two) { if (full) QE_GRAM_X3(false, true, true); else QE_GRAM_X3(false, true, false); }
            else { if (full) QE_GRAM_X3(false, false, true); else QE_GRAM_X3(false, false, false); }
        }
#undef QE_GRAM_X3
    }
    if (hipGetLastError() != hipSuccess) return QE_ERR_HIP;
    if (splits != 0) {
        if (tiles < 128)
            hipLaunchKernelGGL(gram_finalize_kernel<8>, dim3((unsigned)tiles, kTile / 8), dim3(256), 0, s,
                               parts, tiles, (int)used, nt, Sigma, p, accumulate, status);
        else
            hipLaunchKernelGGL(gram_finalize_kernel<32>, dim3((unsigned)tiles, kTile / 32), dim3(256), 0, s,
                               parts, tiles, (int)used, nt, Sigma, p, accumulate, status);
        if (hipGetLastError() != hipSuccess) return QE_ERR_HIP;
    }
    if (damp > 0.f) {
        hipLaunchKernelGGL(damp_kernel, dim3(1), dim3(256), 0, s, Sigma, p, damp, status);
        if (hipGetLastError() != hipSuccess) return QE_ERR_HIP;
    }
    return QE_OK;
}

}  // namespace qe
