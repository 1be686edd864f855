// Sweeps from valid codes, one workgroup per row (gfx950).
//
// From the second sweep on most coordinates keep their level, and a kept
// coordinate changes nothing: neither its code, nor R.  Rows are independent
// (Sec. 3.2), so such a sweep is, for one row, a search for the next column
// whose level moves, followed by that column's rank-1 update
// R_i += delta Sigma_j over all p columns.  Its cost goes with the number of
// moves instead of with p column steps and a q x p x p product.
//
// The row's residual stays in registers over all the sweeps of a launch: wave
// w of the workgroup owns 256 G consecutive columns, lane l the columns
// 256 g + 4 l .. + 3 of its groups g.  The waves take turns in column order.
// The wave whose turn it is looks at one group of 256 columns at a time: every
// lane decides its four coordinates, ballots give the first column that
// moves, its update is applied to the wave's own columns, and the search goes
// on behind that column.  The moves are listed in LDS; after the turn (one
// barrier; two lists alternate, so that the next turn may write while slower
// waves still read) the other waves apply the list to their columns.
//
// Bound: each move reads one row of Sigma, 4 p bytes.  At 4096 x 4096 and 5% moves
// 858000 of them take 1.5 ms (9.4 TB/s, Sigma from the die-level cache), at 4096 x
// 11008 (Sigma 485 MB, from HBM) 1.57 million take 9.9 ms (7 TB/s); below about
// 0.1% the launch's own reads and writes of R, What and the codes remain (0.11
// ms at 4096 x 4096, paid once per launch and not per sweep).  The blocked sweep
// takes 0.4 to 1.1 ms there and 2.2 to 6.9 ms at 4096 x 11008.  Ten sweeps from
// What = W: 8.06 -> 3.04 ms (4096 x 4096), 45.4 -> 20.0 ms (4096 x 11008), 26.7
// -> 14.7 ms (11008 x 4096), 8.69 -> 2.05 ms (1003 x 3001).
// 1024 columns per wave keep a lane's state (16 values of R, 16 codes) at 78
// registers: six waves per SIMD, which hide the latency of the serial search of
// one row behind the other rows.  Turns of 256 columns in place of 1024 (more
// barriers, more reuse of Sigma rows in L2) took 10 to 30% longer, and 8 waves
// of 1536 columns at p = 11008 (139 registers) 25% longer than 11 of 1024.
#include <algorithm>
#include <utility>

#include "qe_internal.h"

namespace qe {

struct RowsArgs {
    const float* Sigma;
    const float* inv_d;
    const float* scale;
    const float* zero;
    const float* inv_s;
    float* Wh;
    uint8_t* codes;
    float* R;
    int64_t q, p;
    float maxq;
    int k0, k1;           // sweeps of the call that this launch may run
    const int* first;     // the optional sweep that was given to this form (see cd_sample_kernel)
    int opt1;             // the first sweep that is not optional
    double* fpart;        // (k1 - k0) x q: objective change of each row and sweep (or null)
    const int* status;
};

// The first sweep of a launch that runs here.
__device__ __forceinline__ int first_sweep(const RowsArgs& a) { return max(a.k0, min(*a.first, a.opt1)); }

// Four consecutive floats; those at or past the end of the row read as 0.
template <bool FULL>
__device__ __forceinline__ f32x4 load4(const float* row, int c, int n)
{
    if (FULL || c + 4 <= n) return *reinterpret_cast<const f32x4a4*>(row + c);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 3; ++e)
        if (c + e < n) v[e] = row[c + e];
    return v;
}

// The wave's columns: L += delta Sigma_j.
template <int G, bool FULL>
__device__ __forceinline__ void apply_move(f32x4 (&L)[G], const float* srow, int c0, int n, float delta)
{
    f32x4 v[G];
#pragma unroll
    for (int g = 0; g < G; ++g) v[g] = load4<FULL>(srow, c0 + 256 * g, n);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) L[g][e] = fmaf(delta, v[g][e], L[g][e]);
}

// Moves [k, k + N) of another wave's turn, all their rows of Sigma in flight together.
template <int G, bool FULL, int N>
__device__ __forceinline__ void apply_listed(f32x4 (&L)[G], const RowsArgs& a, const int2* li, int k, int c0)
{
    f32x4 v[N][G];
    float delta[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int2 en = li[k + u];
        const float* srow = a.Sigma + (int64_t)__builtin_amdgcn_readfirstlane(en.x) * a.p;
        delta[u] = __int_as_float(en.y);
#pragma unroll
        for (int g = 0; g < G; ++g) v[u][g] = load4<FULL>(srow, c0 + 256 * g, (int)a.p);
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) L[g][e] = fmaf(delta[u], v[u][g][e], L[g][e]);
}

// The moves of another wave's turn, in order; AHEAD: four of them at a time.
template <int G, bool FULL, bool AHEAD>
__device__ __forceinline__ void apply_list(f32x4 (&L)[G], const RowsArgs& a, const int2* li, int cnt, int c0)
{
    int k = 0;
    if constexpr (AHEAD) {
        for (; k + 4 <= cnt; k += 4) apply_listed<G, FULL, 4>(L, a, li, k, c0);
        if (k + 2 <= cnt) {
            apply_listed<G, FULL, 2>(L, a, li, k, c0);
            k += 2;
        }
    }
    for (; k < cnt; ++k) {
        const int2 en = li[k];
        const int j = __builtin_amdgcn_readfirstlane(en.x);
        apply_move<G, FULL>(L, a.Sigma + (int64_t)j * a.p, c0, (int)a.p, __int_as_float(en.y));
    }
}

// One group of 256 columns of the wave's turn.  Returns the number of moves so far.
// KEEP: the group's codes stay unpacked over its moves (four more registers, which
// cost workgroups of many waves one of two places on a CU: 2.3 -> 2.9 ms for a
// sweep of 0.7% at 4096 x 11008).
template <int G, int g, bool FULL, bool KEEP>
__device__ __forceinline__ int take_group(const RowsArgs& a, f32x4 (&L)[G], uint32_t (&code)[G], int c0,
                                          int wcol, float s, float inv_s, int2* list, double& f, int cnt)
{
    const int lane = threadIdx.x & 63;
    const int n = (int)a.p;
    if (!FULL && wcol + 256 * g >= n) return cnt;
    f32x4 u = load4<FULL>(a.inv_d, c0 + 256 * g, n);
    auto unpack = [&](int e) { return (float)((code[g] >> (8 * e)) & 0xffu); };
    float kc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        u[e] *= inv_s;
        if constexpr (KEEP) kc[e] = unpack(e);
    }
    // the columns still to be taken: inside the row, behind the last move
    uint64_t open[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) open[e] = FULL ? ~0ull : __ballot(c0 + 256 * g + e < n);
    for (;;) {
        float d[4];
        uint64_t m[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // Lemma 1's minimiser on the grid axis, its nearest level; a valid,
            // equally near current level is kept (Sec. 3.3)
            if constexpr (!KEEP) kc[e] = unpack(e);
            const float t = fmaf(-L[g][e], u[e], kc[e]);
            const float kn = __builtin_amdgcn_fmed3f(rintf(t), 0.f, a.maxq);
            d[e] = kn - kc[e];
            m[e] = __ballot(!(fabsf(t - kc[e]) <= fabsf(t - kn))) & open[e];
        }
        const uint64_t any = m[0] | m[1] | m[2] | m[3];
        if (any == 0) break;
        const int ls = __builtin_ctzll(any);
        const int es = (m[0] >> ls) & 1 ? 0 : (m[1] >> ls) & 1 ? 1 : (m[2] >> ls) & 1 ? 2 : 3;
        const float dsel = es == 0 ? d[0] : es == 1 ? d[1] : es == 2 ? d[2] : d[3];
        const float dm = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dsel), ls));
        const float delta = s * dm;
        const int j = wcol + 256 * g + 4 * ls + es;
        const uint64_t at = 1ull << ls, behind = (~0ull << ls) << 1;
        const float r0 = es == 0 ? L[g][0] : es == 1 ? L[g][1] : es == 2 ? L[g][2] : L[g][3];
        const float mine = lane == ls ? dm : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            open[e] &= behind | (e > es ? at : 0ull);
            if constexpr (KEEP) kc[e] += e == es ? mine : 0.f;
        }
        if constexpr (!KEEP) code[g] += (uint32_t)((int)mine << (8 * es));
        if (list && lane == 0) list[cnt] = make_int2(j, __float_as_int(delta));
        apply_move<G, FULL>(L, a.Sigma + (int64_t)j * a.p, c0, n, delta);
        const float r1 = es == 0 ? L[g][0] : es == 1 ? L[g][1] : es == 2 ? L[g][2] : L[g][3];
        // the move changes f by delta (2 R + delta Sigma_jj) = delta (R + R')
        f += (double)(s * mine) * ((double)r0 + (double)r1);
        ++cnt;
    }
    if constexpr (KEEP) {
        code[g] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) code[g] |= (uint32_t)kc[e] << (8 * e);
    }
    return cnt;
}

// One turn: the wave's columns in order.  Returns the number of moves.
template <int G, bool FULL, bool KEEP, int... g>
__device__ __forceinline__ int take_turn(std::integer_sequence<int, g...>, const RowsArgs& a, f32x4 (&L)[G],
                                         uint32_t (&code)[G], int c0, int wcol, float s, float inv_s,
                                         int2* list, double& f)
{
    int cnt = 0;
    ((cnt = take_group<G, g, FULL, KEEP>(a, L, code, c0, wcol, s, inv_s, list, f, cnt)), ...);
    return cnt;
}

// MULTI: several waves per row, 1024 columns each; else one wave.
template <int G, bool MULTI, bool AHEAD>
__global__ __launch_bounds__(MULTI ? 1024 : 64) void cd_rows_kernel(RowsArgs a)
{
    if (failed(a.status)) return;
    const int start = first_sweep(a);
    if (start >= a.k1) return;
    __shared__ int2 list[2][MULTI ? 256 * G : 1];
    __shared__ int count[2];
    __shared__ double fw[16];
    const int W = MULTI ? (int)blockDim.x >> 6 : 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = blockIdx.x;
    const int n = (int)a.p;
    const int wcol = 256 * G * wave;
    const int c0 = wcol + 4 * lane;
    const bool full = wcol + 256 * G <= n;
    const float s = a.scale[i], z = a.zero[i], inv_s = a.inv_s[i];
    float* Rrow = a.R + i * a.p;
    float* Wrow = a.Wh + i * a.p;
    uint8_t* crow = a.codes + i * a.p;
    f32x4 L[G];
    uint32_t code[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        L[g] = load4<false>(Rrow, c0 + 256 * g, n);
        const f32x4 w = load4<false>(Wrow, c0 + 256 * g, n);
        // the current code is recovered exactly from What (|k - z| <= 255 keeps
        // the rounding error far below 1/2)
        code[g] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c0 + 256 * g + e < n)
                code[g] |= (uint32_t)__builtin_amdgcn_fmed3f(rintf(fmaf(w[e], inv_s, z)), 0.f, 255.f)
                           << (8 * e);
    }
    constexpr auto groups = std::make_integer_sequence<int, G>{};
    int turn = 0;
    for (int sw = start; sw < a.k1; ++sw) {
        double f = 0.0;
        int moves = 0;
        for (int w = 0; w < W; ++w, turn ^= 1) {
            int2* li = MULTI ? list[turn] : nullptr;
            if (wave == w) {
                const int cnt = full ? take_turn<G, true, !MULTI>(groups, a, L, code, c0, wcol, s, inv_s, li, f)
                                     : take_turn<G, false, !MULTI>(groups, a, L, code, c0, wcol, s, inv_s, li, f);
                if (lane == 0) count[turn] = cnt;
            }
            __syncthreads();
            const int cnt = count[turn];
            moves += cnt;
            if (wave != w) {
                if (full)
                    apply_list<G, true, AHEAD>(L, a, li, cnt, c0);
                else if (wcol < n)
                    apply_list<G, false, AHEAD>(L, a, li, cnt, c0);
            }
        }
        if (a.fpart) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) f += __shfl_xor(f, o, 64);
            if (lane == 0) fw[wave] = f;
            __syncthreads();
            if (threadIdx.x == 0) {
                double t = 0.0;
                for (int w = 0; w < W; ++w) t += fw[w];
                a.fpart[(int64_t)(sw - a.k0) * a.q + i] = t;
            }
        }
        if (moves == 0) {       // a fixed point: no later sweep moves anything
            if (a.fpart && threadIdx.x == 0)
                for (int k = sw + 1; k < a.k1; ++k) a.fpart[(int64_t)(k - a.k0) * a.q + i] = 0.0;
            break;
        }
    }
    const bool words = (n & 3) == 0 && (reinterpret_cast<uintptr_t>(a.codes) & 3) == 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int c = c0 + 256 * g;
        f32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = s * ((float)((code[g] >> (8 * e)) & 0xffu) - z);
        if (c + 4 <= n) {
            *reinterpret_cast<f32x4a4*>(Rrow + c) = L[g];
            *reinterpret_cast<f32x4a4*>(Wrow + c) = w;
            if (words) {
                *reinterpret_cast<uint32_t*>(crow + c) = code[g];
                continue;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < n) {
                Rrow[c + e] = L[g][e];
                Wrow[c + e] = w[e];
                crow[c + e] = (uint8_t)(code[g] >> (8 * e));
            }
    }
}

// obj[k] = the objective before sweep k + its change, for the sweeps of a
// cd_rows_kernel launch.  Workgroup b sums sweep k0 + b's changes over the rows in a
// fixed order, in place of the first row's; the second kernel adds them up.  f0: the
// objective before the call's first sweep (null: 0).
__global__ __launch_bounds__(256) void rows_sum_kernel(RowsArgs a)
{
    if (failed(a.status)) return;
    const int k = a.k0 + blockIdx.x;
    if (k < first_sweep(a)) return;
    __shared__ double sh[256];
    double* part = a.fpart + (int64_t)blockIdx.x * a.q;
    double acc = 0.0;
#pragma unroll 4
    for (int64_t e = threadIdx.x; e < a.q; e += 256) acc += part[e];
    const double t = block_sum_f64(acc, sh);
    if (threadIdx.x == 0) part[0] = t;
}

__global__ void rows_objective_kernel(RowsArgs a, const double* f0, double* obj, int stride)
{
    if (failed(a.status) || threadIdx.x != 0) return;
    const int start = first_sweep(a);
    if (start >= a.k1) return;
    double f = start > 0 ? obj[(int64_t)(start - 1) * stride] : (f0 ? *f0 : 0.0);
    for (int k = start; k < a.k1; ++k) {
        f += a.fpart[(int64_t)(k - a.k0) * a.q];
        obj[(int64_t)k * stride] = f;
    }
}

// Whether sweep k runs row by row: no more than `limit` coordinates of a sample of
// rows (every q / gridDim.x-th) would move from the present state.  The last workgroup
// to count decides, sets choice->first and leaves the count at 0 (one 64-bit atomic
// carries both sums, so nothing has to be ordered).  Once a sweep has been given to the
// row form, so are the later ones of the call.
__global__ __launch_bounds__(256) void cd_sample_kernel(const float* __restrict__ R,
                                                        const float* __restrict__ Wh,
                                                        const float* __restrict__ inv_d,
                                                        const float* __restrict__ scale,
                                                        const float* __restrict__ zero,
                                                        const float* __restrict__ inv_s, int64_t q,
                                                        int64_t p, float maxq, int k, int limit,
                                                        RowsChoice* choice, const int* status)
{
    if (failed(status) || choice->first < k) return;
    __shared__ int sh[4];
    const int64_t i = (int64_t)blockIdx.x * q / gridDim.x;
    const float z = zero[i], is = inv_s[i];
    int n = 0;
#pragma unroll 4
    for (int64_t j = threadIdx.x; j < p; j += blockDim.x) {
        const float kc = rintf(fmaf(Wh[i * p + j], is, z));
        const float t = fmaf(-R[i * p + j], inv_d[j] * is, kc);
        const float kn = __builtin_amdgcn_fmed3f(rintf(t), 0.f, maxq);
        n += kn != kc && !(fabsf(t - kc) <= fabsf(t - kn));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x != 0) return;
    constexpr unsigned long long kOne = 1ull << 40;
    const unsigned long long add = kOne + (unsigned)(sh[0] + sh[1] + sh[2] + sh[3]);
    const unsigned long long all = atomicAdd(&choice->count, add) + add;
    if (all < kOne * gridDim.x) return;
    if ((long long)(all % kOne) <= limit) choice->first = k;
    choice->count = 0;
}

constexpr int64_t kRowsMaxP = 16384;     // 16 waves of 1024 columns
constexpr int64_t kOneWave = 1024;       // up to here one wave holds a row
constexpr int kSampleRows = 256;
// Layers of few rows apply another wave's moves four at a time: nothing but the loads in
// flight hides the latency of a row of Sigma there (384 x 1792, five sweeps of a layer of
// 1472 tokens: 1.73 -> 1.65 ms, 1003 x 3001, rho = 0.9, ten sweeps 1.84 -> 1.67, 300 x 6000
// 2.74 -> 2.58, 1280 x 3000 1.35 -> 1.30).  That takes 125 registers, four waves per SIMD;
// where the workgroups then no longer fit the chip at once, more waves hide it better (1282
// x 3000 1.36 against 1.53 ms).  More than four waves load the SIMDs unevenly (768 x 5000
// 2.72 against 3.11 ms): there each SIMD counts as many as the fullest one.
constexpr int64_t kCus = 256, kAheadWaves = 16;

static int rows_threads(int64_t p) { return p <= kOneWave ? 64 : (int)(64 * cdiv(p, 1024)); }

static bool rows_ahead(int64_t q, int64_t p)
{
    const int64_t waves = rows_threads(p) / 64;
    return q <= kCus * (kAheadWaves / (waves <= 4 ? waves : 4 * cdiv(waves, (int64_t)4)));
}

bool cd_rows_fits(int64_t q, int64_t p) { return p <= kRowsMaxP && q <= max_grid(rows_threads(p)); }

constexpr double kFewRows = 0.12;
constexpr double kManyWork = 1.5e11;     // q p^2

// The share of moves at which the blocked sweep costs what the bytes of the row form do
// (see cd_rows_limit).
static double rows_line(int64_t q, int64_t p)
{
    const double work = (double)q * (double)p * (double)p;
    const double bw = 4.0 * (double)p * (double)p <= 2.0e8 ? 9.0e12 : 7.0e12;
    const double dense = std::max(2.0 * work / 135.0e12, (double)(cdiv(p, 256) + 1) * 50.0e-6);
    return dense * bw / (4.0 * work);
}

// The most moves in the sample with which the row form is taken, or -1: always.
// The row form costs 4 p bytes per move, at 9 TB/s while Sigma fits the die-level
// cache and 7 TB/s beyond; the blocked form its products, at 135 TFLOP/s (fp32
// products; 125 to 144 measured over 4096 x 4096, 11008 x 4096 and 4096 x 11008),
// or the column steps of its launches, 50 us for 256 columns, where rows are few.
// The line lies where the two are equal: 3.3% at 4096 x 4096 (measured: 5.1%,
// 1.60 against 1.13 ms; 0.9%, 0.38 against 1.06 ms), 2.6% at 4096 x 11008 (3.5%,
// 9.9 against 6.9 ms; 0.7%, 2.3 against 6.6 ms).
// Strongly coupled channels move less than the sample says (the first move
// settles its neighbours): the blocked form is then kept a few sweeps longer.
//
// Above 12%, where rows are few, the bytes do not bound a move any more but the
// search's chain does: 20 us and 0.45 us per move for one wave (128 x 300, 56%: 0.11
// against 0.08 ms; 16 x 1024, 59%: 0.27 against 0.15), 0.87 us for several (16 x 4096,
// 62%: 2.24 against 0.56 ms; 64 x 12000, 74%: 7.5 against 1.8), and 38 us for 256
// columns of the blocked form.  A layer of less than one panel, 16 rows, is always taken
// row by row (8 x 4096 from rounded weights: 17% move, 0.84 against 0.55 ms, and ten
// sweeps 6.9 against 6.0 ms).
int cd_rows_limit(int64_t q, int64_t p)
{
    double f = rows_line(q, p);
    if (f > kFewRows) {
        if (q < 16) return -1;
        const double move = p <= kOneWave ? 0.45e-6 : 0.87e-6;
        f = std::min(f, ((double)cdiv(p, 256) * 38.0e-6 - 20.0e-6) / ((double)p * move));
        if (f >= 1.0) return -1;
    }
    return (int)(f * (double)std::min<int64_t>(q, kSampleRows) * (double)p);
}

// The sweeps from What = W on (the first counted) up to which the choice is offered.
// The first leaves few codes to move: 10 to 40% move in the second, 4 to 16% in the third,
// 1 to 5% in the fifth, on every layer, bit width and conditioning tried, and from there on
// the row form took at most 1.15 times the blocked sweep (large layers: the line lies
// lower, and the launches weigh less).  Where rows are few the row form loses in the second
// sweep only (layers of as many tokens as channels, 1152 x 1664: 41.6%, 0.79 against 0.26
// ms; third 16%, 0.35; fourth 8%, 0.20), and the empty launches of one optional sweep
// cost up to 5% of a call that did not need them (1003 x 3001, 4.5%: 0.23 against 0.50 ms
// and 0.05 for the launches).  One wave per row loses less (1152 x 1024, 38%: 0.25
// against 0.16 ms) and gains it back in the next sweeps: nothing is offered.
int cd_rows_offered(int64_t q, int64_t p)
{
    if ((double)q * (double)p * (double)p >= kManyWork) return 8;
    if (rows_line(q, p) <= kFewRows) return 4;
    return p > kOneWave ? 2 : 1;
}

qe_status launch_cd_sample(const float* R, const float* Wh, const float* inv_d, const float* scale,
                           const float* zero, const float* inv_s, int64_t q, int64_t p, float maxq,
                           int k, int limit, RowsChoice* choice, const int* status, hipStream_t s)
{
    hipLaunchKernelGGL(cd_sample_kernel, dim3((unsigned)std::min<int64_t>(q, kSampleRows)), dim3(256), 0,
                       s, R, Wh, inv_d, scale, zero, inv_s, q, p, maxq, k, limit, choice, status);
    return hipGetLastError() == hipSuccess ? QE_OK : QE_ERR_HIP;
}

// Sweeps [opt0, sweeps) of a call, of which [opt0, opt1) are optional (those before
// *first have run in the blocked form).  fpart: room for fpart_count doubles (at least
// one sweep of q).
qe_status launch_cd_rows(const float* Sigma, int64_t q, int64_t p, const float* inv_d, const float* scale,
                         const float* zero, const float* inv_s, float maxq, float* Wh, uint8_t* codes,
                         float* R, int sweeps, const int* first, int opt0, int opt1, double* obj, int obj_stride,
                         const double* f0, double* fpart, int64_t fpart_count, const int* status, hipStream_t s)
{
    const int per = obj ? (int)std::max<int64_t>(1, std::min<int64_t>(sweeps, fpart_count / q)) : sweeps;
    for (int k = opt0; k < sweeps; k += per) {
        RowsArgs a{Sigma, inv_d, scale, zero, inv_s, Wh, codes, R, q, p, maxq, k, std::min(k + per, sweeps),
                   first, opt1, obj ? fpart : nullptr, status};
        const dim3 grid((unsigned)q);
#define QE_ROWS(G, M, A) \
    hipLaunchKernelGGL((cd_rows_kernel<G, M, A>), grid, dim3((unsigned)rows_threads(p)), 0, s, a)
        if (p <= 256) QE_ROWS(1, false, false);
        else if (p <= 512) QE_ROWS(2, false, false);
        else if (p <= kOneWave) QE_ROWS(4, false, false);
        else if (rows_ahead(q, p)) QE_ROWS(4, true, true);
        else QE_ROWS(4, true, false);
#undef QE_ROWS
        if (obj)
        {
            hipLaunchKernelGGL(rows_sum_kernel, dim3((unsigned)(a.k1 - a.k0)), dim3(256), 0, s, a);
            hipLaunchKernelGGL(rows_objective_kernel, dim3(1), dim3(64), 0, s, a, f0, obj, obj_stride);
        }
        if (hipGetLastError() != hipSuccess) return QE_ERR_HIP;
    }
    return QE_OK;
}

}  // namespace qe
