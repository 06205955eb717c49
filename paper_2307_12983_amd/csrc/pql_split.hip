// Row-tile learner kernels on the 16-bit matrix cores at 32-bit precision.
//
// Every operand of a matrix product is an fp32 value times a power of two, written as the sum of two fp16 terms
// (hi = fp16(x s), lo = fp16(2^11 (x s - hi)): 22 significant bits and the sign of lo), and a product is three fp16 MFMAs
// (lo w_hi + hi w_lo with sums of their own, hi w_hi; the left-out lo w_lo is below 2^-22 of the product) with fp32 sums.
// What the pairs miss of the weights averages out over the row tiles (split_weights_kernel).
// The scales keep the terms inside fp16's range whatever the data: one per batch row of an activation tile (its largest
// magnitude goes to [2^14, 2^15), found anew for every layer), one per 32 output columns of a weight matrix.  Values down
// to 2^-28 of their row's (their tile's) largest keep their relative precision, smaller ones are off by 2^-50 of that largest
// one.  Infinite inputs and NaN stay in their row, infinite weights in their column.
// Measured against double precision a K = 256 product is off by 1.2e-7 (2-norm) where a chain of fp32 MFMAs is off by
// 2.8e-7: one rounding of the large sums per 32 products instead of sixteen outweighs the missing bit of the operands.
// v_mfma_f32_16x16x32_f16 multiplies at 13 times the rate of v_mfma_f32_32x32x2_f32 (2.0 PFLOP/s against 0.15), so
// three of them are 4.4 times as fast and take a quarter of the energy, which matters as much: the chip holds
// 2.4 GHz only below its power limit.
//
// A workgroup (eight wavefronts, two per SIMD) owns 32 batch rows and carries them through a whole chain of layers, the
// twin critics side by side (four wavefronts each) where the layers are at most 512 wide, one after the other up to 1024.
// (Sixteen wavefronts of 128 registers, weights one step ahead: 68 us per launch at 256-256 and 8192 rows, 55 with eight.)  A
// wavefront owns 32 output columns of one network.  The product is computed as W^T X^T (weights are the A operand): a lane
// then holds four consecutive output columns of one batch row, which is the order in which the next layer's B operand
// wants them, so an epilogue packs its results with no exchange between lanes and writes them to LDS as 16-byte pieces,
// and row maxima, output heads and their gradients come from registers.
//
// What bounds it: with 32 rows per workgroup the weights (4 bytes each, once per workgroup) come from L2 at about 50 bytes per clock
// and compute unit (a loop that only reads reaches 56 with all compute units running), more than twice the time of the matrix work: a
// paired 256 x 256 layer takes 5 us, where the fp32 MFMA kernels take 18.8.  That is a third of the launch (2.3 MB, 18 - 20 of 55 us at
// 256-256 and 8192 rows); the rest is what lies between the products, phases in which a wavefront waits for LDS, barriers and memory or
// issues one instruction every nine cycles.
//
// The weights are brought into fragment order by split_weights_kernel at the start of every call (zero-padded to whole
// tiles, so any layer width works): a lane's operand is one 16-byte load, a wavefront's a contiguous kilobyte.
#include "pql_pairs.h"
#include "pql_rowtile.h"

#include <float.h>

namespace pql {

enum Variant : int { VAR_PLAIN = 0, VAR_SAC = 1, VAR_DIST = 2 };
constexpr int SW = 8;                // wavefronts per workgroup
constexpr int ST = 64 * SW;          // threads per workgroup
constexpr int PT = 1024;             // threads per workgroup of the preparation
constexpr int PREP_ITEMS = SPLIT_MAXK / 256;   // pieces of eight values per thread
constexpr int STEP_UNITS = 384;      // 16-byte units of one k-step of a prepared 32-column tile
constexpr int CS = 33;               // 16-byte units per k-chunk of a tile: 32 rows and one of padding against bank conflicts

// ---- layouts ----------------------------------------------------------------------------------------
// A prepared matrix (K x N): fragments [N/32][K/32][hi, lo, other lo][16-column half][lane] of 16 bytes (see
// split_weights_kernel; workgroups with odd numbers read the other lo terms), then the bias padded with zeros to whole tiles,
// then the inverse scale of every 32-column tile.  Lane (l15 = lane & 15,
// q = lane >> 4) holds column 16 half + l15 for the eight k-values k_slot(step, q, i).
__host__ __device__ __forceinline__ int k_slot(int step, int q, int i) { return 32 * step + 16 * (i >> 2) + 4 * q + (i & 3); }
size_t split_mat_floats(int K, int N) {
    const size_t ks = (size_t)((K + 31) / 32), tiles = (size_t)((N + 31) / 32);
    return tiles * ks * (4 * STEP_UNITS) + tiles * 33;
}
struct MatView { const u32x4* frag; const float* inv; const float* bias; int ks, tiles; };
__device__ __forceinline__ MatView mat_view(const float* base, int K, int N) {
    MatView m;
    m.ks = (K + 31) >> 5; m.tiles = (N + 31) >> 5;
    m.frag = reinterpret_cast<const u32x4*>(base);
    m.bias = base + (unsigned)(m.tiles * m.ks * (4 * STEP_UNITS));
    m.inv = m.bias + (unsigned)(m.tiles * 32);
    return m;
}

__device__ __forceinline__ void split16x8(const f32x4& a, const f32x4& b, float s, u32x4& hi, u32x4& lo) {
    unsigned h[4], l[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        split16x2(a[2 * i], a[2 * i + 1], s, h[i], l[i]);
        split16x2(b[2 * i], b[2 * i + 1], s, h[2 + i], l[2 + i]);
    }
    hi = u32x4{h[0], h[1], h[2], h[3]};
    lo = u32x4{l[0], l[1], l[2], l[3]};
}

// The lo terms of two values at the same distance from the exact remainders as the given ones, on the other side.
__device__ __forceinline__ unsigned other_lo(float x0, float x1, float s, unsigned hi, unsigned lo) {
    const f16x2 h = __builtin_bit_cast(f16x2, hi), l = __builtin_bit_cast(f16x2, lo);
    const float r0 = __fmaf_rn((float)h[0], -PAIR_LO, x0 * s * PAIR_LO), r1 = __fmaf_rn((float)h[1], -PAIR_LO, x1 * s * PAIR_LO);
    const f16x2 o = {(_Float16)__fmaf_rn(2.f, r0, -(float)l[0]), (_Float16)__fmaf_rn(2.f, r1, -(float)l[1])};
    return __builtin_bit_cast(unsigned, o);
}

// Reductions across the four 16-lane rows of a wavefront (same l15) and inside one of them.
__device__ __forceinline__ float quarters_max(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quarters_sum(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float row16_sum(float x) {
    x += dpp_move<0x128>(x);     // row_ror 8, 4, 2, 1
    x += dpp_move<0x124>(x);
    x += dpp_move<0x122>(x);
    return x + dpp_move<0x121>(x);
}
__device__ __forceinline__ float half_max(float x) {          // over the 32 lanes of a half wavefront
    x = fmaxf(x, dpp_move<0x128>(x));
    x = fmaxf(x, dpp_move<0x124>(x));
    x = fmaxf(x, dpp_move<0x122>(x));
    x = fmaxf(x, dpp_move<0x121>(x));
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}

// ---- weights into fragment order ------------------------------------------------------------------------
// One workgroup per 32-column tile: every element is read once (all requests in flight together), kept in registers while
// the tile's largest magnitude is found, and written as fragments.  Latency-bound: one round trip each way.
//
// Two fp16 terms and the sign of lo hold 23 of a weight's 24 significant bits; half of the weights whose lo is in its upper
// octave lie exactly between two pairs.  Rounded the same way for all rows of a batch, those errors add up in the gradients,
// where the errors of activations average out: 1.1e-7 of a policy gradient of 512-256-128 at 8192 rows where the fp32 MFMA
// kernels were off by 0.9e-7.  So there are two sets of lo terms, the second rounded to the other neighbour (lo' =
// fp16(2 r - lo), r the exact remainder), and every second row tile takes the second: on average over the batch the weights are
// exact (0.7e-7).  Workgroups go round the eight XCDs, so an L2 still holds one set.  The Actor step, whose rows stand alone,
// takes the first throughout.
__global__ __launch_bounds__(PT) void split_weights_kernel(const SplitPrepArgs) {
    const SplitPrepArgs& P = kernel_args<SplitPrepArgs>();
    __shared__ float red[PT / 64];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int first = P.first[lane];
    const int pi = __builtin_amdgcn_readfirstlane(__popcll(__ballot(b >= first)) - 1);
    const SplitPrepArgs::Mat M = P.m[pi];
    const int tile = b - __builtin_amdgcn_readlane(first, pi), K = M.K, N = M.N;
    const float* src = M.src;
    float* dst = P.dst + M.dst;
    if (M.kind == SPLIT_VECTOR) {        // a vector padded with zeros to whole tiles
        for (int i = tid; i < (N + 31) / 32 * 32; i += PT) dst[i] = i < N ? src[i] : 0.f;
        return;
    }
    const int ks = (K + 31) >> 5, tiles = (N + 31) >> 5;
    const int items = ks * 128;
    const int l15 = lane & 15, q = lane >> 4;
    const bool trans = M.kind == SPLIT_TRANSPOSED;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(src), 0, K * N * (int)sizeof(float), 0x00020000);
    // element (k, n) at k sk + n sn; what lies outside the matrix is requested outside the descriptor and reads as zero
    const int sk = trans ? 1 : N, sn = trans ? K : 1;
    f32x4 v[PREP_ITEMS][2];
    float mx = 0.f;
#pragma unroll
    for (int it = 0; it < PREP_ITEMS; ++it) {
        if (it * PT >= items) break;
        const int e = it * PT + tid;
        const int n = tile * 32 + ((e >> 6) & 1) * 16 + l15;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = k_slot(e >> 7, q, i);
            v[it][i >> 2][i & 3] = buf_load(rs, k < K && n < N ? (unsigned)(k * sk + n * sn) * 4u : 0x7ffffffcu, 0);
        }
    }
    float bias = 0.f;
    if (tid < 32 && M.bias != nullptr && tile * 32 + tid < N) bias = M.bias[tile * 32 + tid];
#pragma unroll
    for (int it = 0; it < PREP_ITEMS; ++it) {
        if (it * PT >= items) break;
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(v[it][i >> 2][i & 3]));
    }
    // element i of piece e of this tile
    auto offset = [&](int e, int i) {
        const int k = k_slot(e >> 7, (e >> 4) & 3, i), n = tile * 32 + ((e >> 6) & 1) * 16 + (e & 15);
        return k < K && n < N ? (unsigned)(k * sk + n * sn) * 4u : 0x7ffffffcu;
    };
    bool infinite = false;
    while (true) {
        mx = quarters_max(half_max(mx));
        if (lane == 0) red[tid >> 6] = mx;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < PT / 64; ++w) mx = fmaxf(mx, red[w]);
        if (infinite || !(mx > FLT_MAX)) break;
        // an infinite weight: the scale is that of the finite ones, so that the columns beside it keep their values
        infinite = true;
        mx = 0.f;
#pragma unroll 1
        for (int j = tid; j < items * 8; j += PT) {
            const float x = fabsf(buf_load(rs, offset(j >> 3, j & 7), 0));
            mx = fmaxf(mx, x <= FLT_MAX ? x : 0.f);
        }
        __syncthreads();
    }
    float inv;
    const float s = scale_for(mx, inv);
    u32x4* frag = reinterpret_cast<u32x4*>(dst) + (size_t)tile * ks * STEP_UNITS;
    float* tail = dst + (size_t)tiles * ks * (4 * STEP_UNITS);
    auto place = [&](int e) { return frag + (size_t)(e >> 7) * STEP_UNITS + ((e >> 6) & 1) * 64 + lane; };       // piece e's hi terms
#pragma unroll
    for (int it = 0; it < PREP_ITEMS; ++it) {
        const int e = it * PT + tid;
        if (e >= items) break;
        u32x4 hi, lo, lo2;
        split16x8(v[it][0], v[it][1], s, hi, lo);
        u32x4* d = place(e);
        d[0] = hi;
        d[128] = lo;
        if (!P.both) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) lo2[i] = other_lo(v[it][i >> 1][2 * (i & 1)], v[it][i >> 1][2 * (i & 1) + 1], s, hi[i], lo[i]);
        d[256] = lo2;
    }
    if (infinite) {          // as hi = 0, lo = +-inf: one product with the sign of x_hi, none with x_lo
#pragma unroll 1
        for (int e = tid; e < items; e += PT)                    // (the pieces this thread has just written)
#pragma unroll 1
            for (int i = 0; i < 8; ++i) {
                const float x = buf_load(rs, offset(e, i), 0);
                if (!(fabsf(x) > FLT_MAX)) continue;
                char* d = reinterpret_cast<char*>(place(e)) + 2 * i;
                const uint16_t hi = 0, lo = x > 0.f ? 0x7c00 : 0xfc00;
                __builtin_memcpy(d, &hi, 2);
                __builtin_memcpy(d + 128 * 16, &lo, 2);
                if (P.both) __builtin_memcpy(d + 256 * 16, &lo, 2);
            }
    }
    if (tid == 0) tail[tiles * 32 + tile] = inv;
    if (tid < 32) tail[tile * 32 + tid] = bias;
}

hipError_t split_weights_launch(SplitPrepArgs& a, bool both, int kid, hipStream_t stream) {
    a.both = both ? 1 : 0;
    int blocks = 0;
    double bytes = 0.0;
    for (int i = 0; i < 64; ++i) {
        a.first[i] = i < a.n ? blocks : 0x7fffffff;
        if (i >= a.n) continue;
        if (a.m[i].kind != SPLIT_VECTOR && a.m[i].K > SPLIT_MAXK) return hipErrorInvalidValue;
        blocks += a.m[i].kind == SPLIT_VECTOR ? 1 : (a.m[i].N + 31) / 32;
        bytes += (both ? 10.0 : 8.0) * a.m[i].K * a.m[i].N;
    }
    if (blocks == 0) return hipSuccess;
    const ProfSlot ps = prof_slot();
    PQL_LAUNCH(ps, split_weights_kernel, dim3(blocks), dim3(PT), 0, stream, a);
    prof_commit(ps, kid, 0.0, kid == KID_SPLIT_WEIGHTS ? bytes : 0.0);
    return hipGetLastError();
}

// ---- a layer on the tile --------------------------------------------------------------------------------
struct Wv { int tid, lane, wave, l15, q; unsigned hi, lo; };        // hi, lo: this lane's byte offsets into a k-step's fragments
// R: what is rare is not compiled in (an input of more than XV steps or in the place of the activations, widths that are no
// multiples of four): a wavefront issues an instruction every nine cycles (4.5 where two share a SIMD), and the tests, scalars and
// registers kept (and spilled) for paths not taken lengthen every phase.  us per launch with / without them: critic update 256-256
// 58 / 55, policy update 51 / 48, critic update 512-256-128 125 / 120, 64-64 at 256 rows 23.6 / 22; with the input in the place of
// the activations critic update 1024-512-256 at 4096 rows 364 / 328, policy update 512-512-256 at 16384 385 / 373.  Kernels with the
// critics one after the other still spill: 76 (critic) and 53 - 63 (policy) vector registers, 140 - 148 bytes of scratch a lane, and
// with everything 191 - 204 and 181 - 197.
enum Shapes : int { GENERAL = 0, REGULAR = 1, REGULAR_ALIAS = 2 };      // REGULAR_ALIAS: the input may lie in the place of the activations
template <bool R>
struct WvOf : Wv { static constexpr bool regular = R; };

// Barrier for data in LDS only: __syncthreads() would also wait for every store to memory and every weight request that
// is meant to stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ u32x4* lds_units() { return reinterpret_cast<u32x4*>(smem); }

// Activation tile in LDS: k-chunks of eight values (chunk 4 step + q holds k_slot(step, q, 0..7)), 32 rows each, hi terms
// then lo terms.  base and plane in 16-byte units.
struct Tile { int base, plane; };

// The fragments of two k-steps of a 32-column tile (4 KB each, hi and lo of its halves): the requests run two steps ahead of the matrix work, also
// from one product to the next (over the epilogue and its barriers), so every product is told where the following one begins.
template <int D>
struct AheadOf { u32x4 w[D][4]; };
typedef AheadOf<2> Ahead;
struct Begin { const u32x4* first; const u32x4* second; };
__device__ __forceinline__ Begin begin_of(const MatView& W, int tile, int s0, int ds) {
    const int t = tile < W.tiles ? tile : 0, a = s0 < W.ks ? s0 : 0, b = s0 + ds < W.ks ? s0 + ds : a;     // (an idle wavefront requests something valid)
    return {W.frag + (unsigned)((t * W.ks + a) * STEP_UNITS), W.frag + (unsigned)((t * W.ks + b) * STEP_UNITS)};
}
__device__ __forceinline__ Begin begin_at(const float* mat) {
    return {reinterpret_cast<const u32x4*>(mat), reinterpret_cast<const u32x4*>(mat)};
}
template <int D>
__device__ __forceinline__ void request(AheadOf<D>& a, const Begin& p, const Wv& T) {
#pragma unroll
    for (int st = 0; st < D; ++st) {
        const char* step = reinterpret_cast<const char*>(st == 0 ? p.first : p.second);
#pragma unroll
        for (int m = 0; m < 2; ++m) a.w[st][m] = *reinterpret_cast<const u32x4*>(step + T.hi + m * 1024);
#pragma unroll
        for (int m = 0; m < 2; ++m) a.w[st][2 + m] = *reinterpret_cast<const u32x4*>(step + T.lo + m * 1024);
    }
}

// acc[m][n] = 16x16 products of weight columns 32 tile + 16 m .. with batch rows 16 n .., steps s0, s0 + ds, ...  `cur`
// holds the first two steps' fragments and leaves with those at `next` (the fences keep the requests ahead of the MFMAs).
// The cross products have sums of their own, 2^11 too large like their lo terms, which join at the end.
// NB blocks of 16 rows (tiles of 32 rows: 2), D steps ahead.
template <int NB, int D>
__device__ __forceinline__ void mac_steps(f32x4 (&acc)[2][NB], const MatView& W, int tile, const Tile& X, const Wv& T, int s0, int ds,
                                          AheadOf<D>& cur, const Begin& next) {
    const u32x4* p = W.frag + (unsigned)(tile * W.ks * STEP_UNITS);
    f32x4 low[2][NB];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) { acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f}; low[m][n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    auto mac = [&](int s, const u32x4 (&w)[4]) {
        const int at = X.base + (4 * s + T.q) * (16 * NB + 1) + T.l15;
        f16x8 xh[NB], xl[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            xh[n] = __builtin_bit_cast(f16x8, lds_units()[at + 16 * n]);
            xl[n] = __builtin_bit_cast(f16x8, lds_units()[at + X.plane + 16 * n]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const f16x8 a = __builtin_bit_cast(f16x8, c == 0 ? w[2 + m] : w[m]);
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    if (c == 0) low[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xh[n], low[m][n], 0, 0, 0);
                    if (c == 1) low[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xl[n], low[m][n], 0, 0, 0);
                    if (c == 2) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xh[n], acc[m][n], 0, 0, 0);
                }
            }
    };
    // D steps from s on out of `have`, the D after them requested into `get`
    auto step = [&](int s, AheadOf<D>& have, AheadOf<D>& get) {
        const int s2 = s + D * ds, s3 = s + (2 * D - 1) * ds;
        Begin b = next;
        if (s2 < W.ks) b = {p + (unsigned)(s2 * STEP_UNITS), p + (unsigned)((s3 < W.ks ? s3 : s2) * STEP_UNITS)};
        request(get, b, T);
        __builtin_amdgcn_sched_barrier(0);
        mac(s, have.w[0]);
        if (D > 1 && s + ds < W.ks) mac(s + ds, have.w[D - 1]);
        __builtin_amdgcn_sched_barrier(0);
        return s2 < W.ks;
    };
    AheadOf<D> other;
    for (int s = s0; ; s += 2 * D * ds) {
        if (!step(s, cur, other)) { cur = other; break; }
        if (!step(s + D * ds, other, cur)) break;
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[m][n][r] = __fmaf_rn(low[m][n][r], 1.f / PAIR_LO, acc[m][n][r]);
}

template <int NB>
__device__ __forceinline__ void clear(f32x4 (&z)[2][NB]) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) z[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// (PAST: stores bypass the caches' retention.  The one-launch kernels leave their results in the caches, where a row's two
// 64-byte pieces of a line meet and the next kernel finds them: policy update 512-512-256 395 / 369 us, critic update 512-256-128
// 140 / 131, 256-256 59.8 / 58.2 and its weight gradients 23.2 / 22.3.  The layer kernel's results are larger than the
// caches: no difference there, and the weight gradients after it are 1 % faster without them.)
// The 32 x 32 results of one tile to / from a row-major [B][N] array: this lane's rows r0 + 16 n + l15, columns
// 32 tile + 16 m + 4 q .. + 3.  Through a descriptor of the tile's rows, which drops what lies past them: no branches, so that all
// requests leave together and none waits for another (as masked loads the compiler waited for each before the next one:
// four round trips a tile).  Widths that are no multiples of four pay for the branch-free form with requests past the descriptor: with
// masked loads policy updates of such networks above 512 wide were 3 - 5 % faster (514-31 at 4096 rows 115.5 / 118.8 us, 1023-510-255
// 359 / 370, stochastic 641-201 at 3000 rows 175 / 184), all others slower (critic updates 127.4 / 126.3, 421 / 419, 191 / 186; 301-62
// at 4096 rows critic 82.3 / 76.1, policy 76.0 / 72.1).
constexpr int NOWHERE = 0x7ffffffc;          // a buffer offset past any descriptor used here: a load returns zero, a store is dropped
template <int NB>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rows(const float* g, int N, int r0, int B) {
    const int rows = B - r0 < 16 * NB ? B - r0 : 16 * NB;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g) + (size_t)r0 * (size_t)N, 0, rows * N * (int)sizeof(float), 0x00020000);
}
template <int NB = 2, bool PAST = false, typename WV>
__device__ __forceinline__ void store_tile(float* g, int N, int tile, const f32x4 (&z)[2][NB], int r0, int B, const WV& T) {
    const __amdgpu_buffer_rsrc_t rs = tile_rows<NB>(g, N, r0, B);
    const int col = 32 * tile + 4 * T.q;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int at = ((16 * n + T.l15) * N + col + 16 * m) * (int)sizeof(float);
            if (WV::regular || (N & 3) == 0) {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, z[m][n]), rs, col + 16 * m < N ? at : NOWHERE, 0, PAST ? 2 : 0);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(z[m][n][r]), rs, col + 16 * m + r < N ? at + 4 * r : NOWHERE, 0, 0);
            }
        }
}
template <int NB = 2, typename WV>
__device__ __forceinline__ void load_tile(const float* g, int N, int tile, f32x4 (&z)[2][NB], int r0, int B, const WV& T) {
    const __amdgpu_buffer_rsrc_t rs = tile_rows<NB>(g, N, r0, B);
    const int col = 32 * tile + 4 * T.q;
    const bool vec = WV::regular || (N & 3) == 0;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int at = ((16 * n + T.l15) * N + col + 16 * m) * (int)sizeof(float);
            z[m][n] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vec && col + 16 * m < N ? at : NOWHERE, 0, 0));
        }
    if (vec) return;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int at = ((16 * n + T.l15) * N + col + 16 * m) * (int)sizeof(float);
#pragma unroll
            for (int r = 0; r < 4; ++r) z[m][n][r] = buf_load(rs, (unsigned)(col + 16 * m + r < N ? at + 4 * r : NOWHERE), 0);
        }
}
// Sums of a[..] over the tile's rows (this lane's share of them) to out[N].  Eight columns' values meet in a butterfly that
// halves what a lane holds at every exchange (lane l15 of a quarter ends with column l15 / 2 of its eight), so that one store
// takes all 32 columns.
__device__ __forceinline__ void store_colsum(float* out, int N, int tile, const f32x4 (&a)[2], const Wv& T) {
    const bool b3 = (T.l15 & 8) != 0, b2 = (T.l15 & 4) != 0, b1 = (T.l15 & 2) != 0;
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = (b3 ? a[1][r] : a[0][r]) + dpp_move<0x128>(b3 ? a[0][r] : a[1][r]);          // row_ror 8
    float u[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) u[r] = (b2 ? v[2 + r] : v[r]) + dpp_move<0x141>(b2 ? v[r] : v[2 + r]);              // row_half_mirror
    float s = (b1 ? u[1] : u[0]) + dpp_move<0x4E>(b1 ? u[0] : u[1]);                                                // quad_perm [2, 3, 0, 1]
    s += dpp_move<0xB1>(s);                                                                                         // quad_perm [1, 0, 3, 2]
    const int col = 32 * tile + 16 * (T.l15 >> 3) + 4 * T.q + ((T.l15 >> 1) & 3);
    if ((T.l15 & 1) == 0 && col < N) out[col] = s;
}

// Which of the workgroup's networks and output tiles a wavefront works on.
struct Share { int net, slot, waves; };      // tiles slot, slot + waves, ...
template <typename WV>
__device__ __forceinline__ void load_ahead(const float* h, int N, f32x4 (&hv)[2][2], const Share& S, int r0, int B, const WV& T) {
    load_tile(h, N, S.slot, hv, r0, B, T);
}

// Small per-tile arrays in LDS (floats from `sm`).
struct SmallMem {
    int max, part, inv, logp, act;           // of 16 NB rows: row maxima and head partials of eight wavefronts, inverse scales of X, log pi, [as] actions
    int as;
};
__host__ __device__ constexpr int small_floats(int nb, int as) { return 288 * nb + 16 * nb * as; }
template <int NB>
__device__ __forceinline__ SmallMem small_mem(int sm, int as) {
    SmallMem m;
    m.max = sm; m.part = sm + 128 * NB; m.inv = sm + 256 * NB; m.logp = sm + 272 * NB; m.act = sm + 288 * NB; m.as = as;
    return m;
}

// Puts the wavefronts' results (z, TPW tiles of 32 columns each) into the activation tile `out`, in place over the layer's
// input: row maxima meet in LDS; the barrier they need is also the one after which nobody reads the input any more.
template <int TPW, int NB>
__device__ __forceinline__ void put_tile(const f32x4 (&z)[TPW][2][NB], int tiles, const Tile& out, const Share& S, const SmallMem& M,
                                float (&inv)[NB], const Wv& T) {
    float mx[NB] = {};
#pragma unroll
    for (int t = 0; t < TPW; ++t)
        if (S.slot + t * S.waves < tiles) {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mx[n] = fmaxf(mx[n], fabsf(z[t][m][n][r]));
        }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        mx[n] = quarters_max(mx[n]);
        if (T.q == 0) smem[M.max + (S.net * 16 * NB + 16 * n + T.l15) * S.waves + S.slot] = mx[n];
    }
    lds_barrier();
    float sc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const f32x4* src = reinterpret_cast<const f32x4*>(smem) + (M.max + (S.net * 16 * NB + 16 * n + T.l15) * S.waves) / 4;
        f32x4 a = src[0];
        float m = fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));
        if (S.waves > 4) {
            a = src[1];
            m = fmaxf(m, fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])));
        }
        sc[n] = scale_for(m, inv[n]);
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int tile = S.slot + t * S.waves;
        if (tile < tiles) {
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                u32x4 hi, lo;
                split16x8(z[t][0][n], z[t][1][n], sc[n], hi, lo);
                const int at = out.base + (4 * tile + T.q) * (16 * NB + 1) + 16 * n + T.l15;
                lds_units()[at] = hi;
                lds_units()[at + out.plane] = lo;
            }
        }
    }
    lds_barrier();
}

// z = ELU(X W + b) for this wavefront's tiles; inv = inverse row scales of the input tile.
template <int TPW, int NB, int D>
__device__ __forceinline__ void forward(f32x4 (&z)[TPW][2][NB], const MatView& W, const Tile& X, const Share& S, const float (&inv)[NB],
                               const Wv& T, AheadOf<D>& cur, const Begin& next) {
    if (S.slot >= W.tiles) request(cur, next, T);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int tile = S.slot + t * S.waves;
        if (tile >= W.tiles) { clear(z[t]); continue; }
        const bool more = t + 1 < TPW && tile + S.waves < W.tiles;
        f32x4 b[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) b[m] = *reinterpret_cast<const f32x4*>(W.bias + 32 * tile + 16 * m + 4 * T.q);
        const float iw = W.inv[tile];
        f32x4 acc[2][NB];
        mac_steps(acc, W, tile, X, T, 0, 1, cur, more ? begin_of(W, tile + S.waves, 0, 1) : next);
        float f[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) f[n] = inv[n] * iw;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) z[t][m][n][r] = elu_f(__fmaf_rn(acc[m][n][r], f[n], b[m][r]));
    }
}

// z = (D W^T) * ELU'(.) with the activations h [B][N] read back from memory (each lane reads what it wrote in the forward
// pass: those of the first tile the caller has requested into hv before the deltas were put into the tile); the deltas go to
// d_out and their column sums to col_out where given.
template <int TPW, typename WV>
__device__ __forceinline__ void backward(f32x4 (&z)[TPW][2][2], const MatView& W, const Tile& X, const Share& S, const float (&inv)[2],
                                const float* h, float* d_out, float* col_out, int N, int r0, int B, const WV& T, Ahead& cur,
                                const Begin& next, f32x4 (&hv)[2][2]) {
    if (S.slot >= W.tiles) request(cur, next, T);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int tile = S.slot + t * S.waves;
        if (tile >= W.tiles) { clear(z[t]); continue; }
        const bool more = t + 1 < TPW && tile + S.waves < W.tiles;
        f32x4 acc[2][2];
        const float iw = W.inv[tile];
        if (t > 0) load_tile(h, N, tile, hv, r0, B, T);
        mac_steps(acc, W, tile, X, T, 0, 1, cur, more ? begin_of(W, tile + S.waves, 0, 1) : next);
        const float f[2] = {inv[0] * iw, inv[1] * iw};
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) z[t][m][n][r] = acc[m][n][r] * f[n] * delu_h(hv[m][n][r]);
        if (d_out != nullptr) store_tile(d_out, N, tile, z[t], r0, B, T);
        if (col_out != nullptr) {
            const f32x4 cs[2] = {z[t][0][0] + z[t][0][1], z[t][1][0] + z[t][1][1]};
            store_colsum(col_out, N, tile, cs, T);
        }
    }
}

// ---- input rows --------------------------------------------------------------------------------------------
// Rows r0 .. r0 + 16 NB - 1 of concat(obs[o], act[a]) as a tile: half a wavefront takes NB rows, one after the other, so that their
// largest magnitudes are found without leaving the registers.  `floor`: lower bound of that magnitude (actions in [-1, 1] that are inserted later must
// fit the row's scale).  Up to 256 columns are requested ahead of time into v.
struct InputRows { __amdgpu_buffer_rsrc_t obs, act, mean, rstd; int o, a, act_lds, as, last; bool norm; };   // act_lds >= 0: actions in LDS; last: last row
constexpr int XV = 8;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const float* p, int cols, int r0, int B, int most) {
    const int rows = B - r0 < most ? B - r0 : most;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + (size_t)r0 * (size_t)cols, 0,
                                             p != nullptr ? rows * cols * (int)sizeof(float) : 0, 0x00020000);
}
template <int NB>
__device__ __forceinline__ InputRows input_rows(const float* obs, int o, const float* act, int act_lds, int a, int as, int r0, int B) {
    InputRows in;
    in.obs = rows_of(obs, o, r0, B, 16 * NB); in.act = rows_of(act, a, r0, B, 16 * NB); in.mean = in.obs; in.rstd = in.obs;
    in.o = o; in.a = a; in.act_lds = act_lds; in.as = as; in.last = (B - r0 < 16 * NB ? B - r0 : 16 * NB) - 1; in.norm = false;
    return in;
}
// Places of rows beyond the batch hold its last row: their results go nowhere, but enter sums with a factor of zero, so they
// have to be finite where those of the batch are (a row of zeros is not, at an infinite weight).  Columns beyond the row are
// requested past the descriptor and read as zero.
__device__ __forceinline__ float input_value(const InputRows& in, int row, int col) {
    float x = buf_load(in.obs, (unsigned)(col < in.o ? (row * in.o + col) * 4 : NOWHERE), 0);
    if (in.norm) {
        const unsigned at = (unsigned)(col < in.o ? col * 4 : NOWHERE);
        x = (x - buf_load(in.mean, at, 0)) * buf_load(in.rstd, at, 0);
    }
    return x;
}
__device__ __forceinline__ float input_action(const InputRows& in, int row, int col) {
    const int c = col - in.o;
    const bool live = c >= 0 && c < in.a;
    if (in.act_lds >= 0) {
        const float y = smem[in.act_lds + row * in.as + (live ? c : 0)];
        return live ? y : 0.f;
    }
    return buf_load(in.act, (unsigned)(live ? (row * in.a + c) * 4 : NOWHERE), 0);
}
// Requested rows: columns c + 32 j of the states (and their statistics), and the action columns, which lie in the steps j0 and
// j0 + 1.  They come together where they are put: put together here, the request would wait for its own answers.
template <int NB>
struct Rows { float v[NB][XV], y[NB][2], mean[XV], rstd[XV]; };
__device__ __forceinline__ int input_row(const Wv& T, int i) { return 2 * T.wave + (T.lane >> 5) + 16 * i; }
__device__ __forceinline__ int source_row(const InputRows& in, int row) { return row < in.last ? row : in.last; }
// Element j of a row that begins at byte offset `base` (this lane's first column included): whole steps need no mask.
__device__ __forceinline__ float step_value(__amdgpu_buffer_rsrc_t r, int base, int j, int j0, int o, int c) {
    const int at = j < j0 || (j == j0 && c + 32 * j0 < o) ? base : NOWHERE - 32 * 4 * XV;
    return buf_load(r, (unsigned)(at + 128 * j), 0);
}
template <int NB, typename WV>
__device__ __forceinline__ void request_rows(Rows<NB>& x, const InputRows& in, int steps, const WV& T) {
    if (!WV::regular && steps > XV) return;
    const int c = T.lane & 31, j0 = in.o >> 5;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = source_row(in, input_row(T, i)), base = (row * in.o + c) * 4;
#pragma unroll
        for (int j = 0; j < XV; ++j)
            if (j < steps) x.v[i][j] = step_value(in.obs, base, j, j0, in.o, c);
        if (in.a > 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) x.y[i][j] = input_action(in, row, c + 32 * (j0 + j));
        }
    }
    if (in.norm) {
#pragma unroll
        for (int j = 0; j < XV; ++j)
            if (j < steps) { x.mean[j] = step_value(in.mean, c * 4, j, j0, in.o, c); x.rstd[j] = step_value(in.rstd, c * 4, j, j0, in.o, c); }
    }
}
__device__ __forceinline__ float input_any(const InputRows& in, int row, int col) {
    const float x = input_value(in, row, col);
    return in.a > 0 && col >= in.o ? input_action(in, row, col) : x;
}
template <int NB>
__device__ __forceinline__ int tile_half(const Tile& X, int row, int k) {      // position of (row, k) in 2-byte units
    return (X.base + ((k >> 5) * 4 + ((k >> 2) & 3)) * (16 * NB + 1) + row) * 8 + (k & 3) + 4 * ((k >> 4) & 1);
}
__device__ __forceinline__ void put_at(const Tile& X, int at, float x, float s) {
    _Float16* h = reinterpret_cast<_Float16*>(smem);
    _Float16 hi, lo;
    split16(x, s, hi, lo);
    h[at] = hi;
    h[at + X.plane * 8] = lo;
}
template <int NB>
__device__ __forceinline__ void put_value(const Tile& X, int row, int k, float x, float s) { put_at(X, tile_half<NB>(X, row, k), x, s); }
template <int NB, typename WV>
__device__ __forceinline__ void put_rows(const Rows<NB>& x, const InputRows& in, int steps, const Tile& X, int inv_at, float floor_,
                                         const WV& T) {
    const int c = T.lane & 31, j0 = in.o >> 5;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = input_row(T, i);
        float mx = floor_, v[XV];
        if (WV::regular || steps <= XV) {
            // states and actions come together here, not where they are requested: that would wait for both
#pragma unroll
            for (int j = 0; j < XV; ++j) {
                if (j >= steps) break;
                v[j] = in.norm ? (x.v[i][j] - x.mean[j]) * x.rstd[j] : x.v[i][j];
                if (in.a > 0 && j >= j0) v[j] = c + 32 * j >= in.o ? (j > j0 ? x.y[i][1] : x.y[i][0]) : v[j];
                mx = fmaxf(mx, fabsf(v[j]));
            }
        } else {
            for (int j = 0; j < steps; ++j) mx = fmaxf(mx, fabsf(input_any(in, source_row(in, row), c + 32 * j)));
        }
        float inv;
        const float s = scale_for(half_max(mx), inv);
        if (c == 0) smem[inv_at + row] = inv;
        if (WV::regular || steps <= XV) {
#pragma unroll
            for (int j = 0; j < XV; ++j) {
                if (j >= steps) break;
                put_at(X, tile_half<NB>(X, row, c) + j * 4 * (16 * NB + 1) * 8, v[j], s);
            }
        } else {
            for (int j = 0; j < steps; ++j) put_value<NB>(X, row, c + 32 * j, input_any(in, source_row(in, row), c + 32 * j), s);
        }
    }
}
template <int NB>
__device__ __forceinline__ void row_inv(float (&inv)[NB], int at, const Wv& T) {
#pragma unroll
    for (int n = 0; n < NB; ++n) inv[n] = smem[at + 16 * n + T.l15];
}

// ---- action-wide products --------------------------------------------------------------------------------
// At most 32 output columns: the wavefronts of a network split the contraction, every one leaves its partial tile
// in LDS, over the input tile (hence the first barrier); afterwards element (row, col) is the sum of the partial tiles.
template <int NB>
__device__ __forceinline__ void put_partial(const f32x4 (&acc)[2][NB], int at, int part, bool mine, const Wv& T) {
    lds_barrier();
    if (mine) {
        f32x4* p = reinterpret_cast<f32x4*>(smem) + at + part * (128 * NB) + T.lane;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n) p[(NB * m + n) * 64] = acc[m][n];
    }
    lds_barrier();
}
template <int NB>
__device__ __forceinline__ float sum_partials(int at, int parts, int row, int col) {
    const int e = (((col >> 4) * NB + (row >> 4)) * 64 + ((col >> 2) & 3) * 16 + (row & 15)) * 4 + (col & 3);
    float s = 0.f, x[SW];
#pragma unroll
    for (int p = 0; p < SW; ++p) x[p] = smem[at * 4 + (p < parts ? p : 0) * (512 * NB) + e];      // (all requests before the first sum)
#pragma unroll
    for (int p = 0; p < SW; ++p) s += p < parts ? x[p] : 0.f;
    return s;
}
template <int NB>
__device__ __forceinline__ void scaled(f32x4 (&acc)[2][NB], const float (&inv)[NB], float iw) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[m][n][r] *= inv[n] * iw;
}

// A sample of the tanh-Gaussian policy for element (row, col) of the output tile; the 32 lanes of a row add their shares of
// log pi, which every lane returns.
template <int NB>
__device__ __forceinline__ float sample_action(int at, int parts, int row, int col, int a, const float* bias, int r0, const FusedSac& sc,
                                      float& act, float& eps, float& raw) {
    float lp = 0.f;
    act = 0.f; eps = 0.f; raw = 0.f;
    if (col < a) {
        const float mu = sum_partials<NB>(at, parts, row, col) + bias[col];
        raw = sum_partials<NB>(at, parts, row, col + a) + bias[col + a];
        eps = std_normal_f((uint32_t)((r0 + row) * a + col), sc);
        const float ls = fminf(fmaxf(raw, SAC_LOG_STD_MIN), SAC_LOG_STD_MAX);
        const float u = mu + expf(ls) * eps;
        const float x = -2.f * u;
        const float softplus = fmaxf(x, 0.f) + log1pf(expf(-fabsf(x)));
        lp = -0.5f * eps * eps - ls - 0.91893853320467274178f - 2.f * (0.69314718055994530942f - u - softplus);
        act = tanhf(u);
    }
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) lp += __shfl_xor(lp, o);
    return lp;
}

// The policy's hidden layers on the tile (all wavefronts on one network), its output layer as partial tiles.
// keep: h_l go to hA[l]; returns the number of partial tiles at H.
template <int TPW, int NB, int D, typename WV>
__device__ __forceinline__ int policy_forward(const SplitShape& P, const float* const* mats, const Tile& X, const Tile& H, const SmallMem& M,
                                     bool keep, float* const* hA, int aw, int r0, int B, const WV& T, AheadOf<D>& cur,
                                     const Begin& next) {
    const Share S = {0, T.wave, SW};
    float inv[NB];
    row_inv(inv, M.inv, T);
    f32x4 z[TPW][2][NB];
    for (int l = 0; l < P.L; ++l) {
        const int N = P.H[l];
        const MatView W = mat_view(mats[l], l == 0 ? P.o : P.H[l - 1], N);
        const MatView V = mat_view(mats[l + 1], N, l + 1 < P.L ? P.H[l + 1] : aw);
        forward(z, W, l == 0 ? X : H, S, inv, T, cur, l + 1 < P.L ? begin_of(V, S.slot, 0, 1) : begin_of(V, 0, T.wave, SW));
        if (keep) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
                if (S.slot + t * SW < W.tiles) store_tile(hA[l + 1], N, S.slot + t * SW, z[t], r0, B, T);
        }
        put_tile(z, W.tiles, H, S, M, inv, T);
    }
    const MatView W = mat_view(mats[P.L], P.H[P.L - 1], aw);
    f32x4 acc[2][NB];
    clear(acc);
    if (T.wave < W.ks) mac_steps(acc, W, 0, H, T, T.wave, SW, cur, next);
    else request(cur, next, T);
    scaled(acc, inv, W.inv[0]);
    const int parts = W.ks < SW ? W.ks : SW;
    put_partial(acc, H.base, T.wave, T.wave < parts, T);
    return parts;
}

// Scalar output head: partial dot products of this wavefront's tiles of the last hidden layer with the output weights meet in
// LDS; q[i][n] = Q_i of this lane's rows (all networks the workgroup carries; one: q[0]).
template <int NN, int TPW>
__device__ __forceinline__ void head_values(const f32x4 (&z)[TPW][2][2], const f32x4 (&wo)[TPW][2], const Share& S, const SmallMem& M,
                                   const float (&bias)[NN], float (&q)[NN][2], const Wv& T) {
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) s += z[t][m][n][r] * wo[t][m][r];
        s = quarters_sum(s);
        if (T.q == 0) smem[M.part + (S.net * 32 + 16 * n + T.l15) * S.waves + S.slot] = s;
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NN; ++i)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const f32x4* src = reinterpret_cast<const f32x4*>(smem) + (M.part + (i * 32 + 16 * n + T.l15) * S.waves) / 4;
            f32x4 v = src[0];
            if (S.waves > 4) v += src[1];
            q[i][n] = (v[0] + v[1]) + (v[2] + v[3]) + bias[i];
        }
}
template <int TPW>
__device__ __forceinline__ void head_weights(f32x4 (&wo)[TPW][2], const float* w, int tiles, const Share& S, const Wv& T) {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int tile = S.slot + t * S.waves;
            wo[t][m] = tile < tiles ? *reinterpret_cast<const f32x4*>(w + 32 * tile + 16 * m + 4 * T.q) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
}

// Hidden layers of the critics on (X): leaves z = h_L in registers.  h_l of layers l <= kept go to h[net][l].
template <int NN, int TPW, typename WV>
__device__ __forceinline__ void critic_forward(f32x4 (&z)[TPW][2][2], const SplitShape& P, const float* const (*mats)[PQL_MAX_HIDDEN + 1],
                                      int net, const Tile& X, const Tile& H, const Share& S, const SmallMem& M, int kept,
                                      float* const (*h)[PQL_MAX_HIDDEN + 1], int r0, int B, const WV& T, Ahead& cur,
                                      const Begin& next, Rows<2>& xv, const InputRows& following, bool fetch) {
    float inv[2];
    row_inv(inv, M.inv, T);
    for (int l = 0; l < P.L; ++l) {
        const int N = P.H[l];
        const MatView W = mat_view(mats[net][l], l == 0 ? P.o + P.a : P.H[l - 1], N);
        Begin n = next;
        if (l + 1 < P.L) n = begin_of(mat_view(mats[net][l + 1], N, P.H[l + 1]), S.slot, 0, 1);
        forward(z, W, l == 0 ? X : H, S, inv, T, cur, n);
        if (l == 0 && fetch) request_rows(xv, following, (P.o + P.a + 31) >> 5, T);    // the next chain's input
        if (l < kept) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
                if (S.slot + t * S.waves < W.tiles) store_tile(h[net][l + 1], N, S.slot + t * S.waves, z[t], r0, B, T);
        }
        if (l < P.L - 1) put_tile(z, W.tiles, H, S, M, inv, T);
    }
}

// ---- distributional critics (PQL-D) on the tile ------------------------------------------------------------------------
// Logits of a network from its last hidden tile: atoms <= 64 columns in two 32-column tiles, the wavefronts of a network take
// one tile and every second k-step; the partial tiles go to LDS over the activations.  A row is then handled by one
// wavefront, lane = atom.
constexpr int DIST_PARTS = 4;        // partial tiles per network: (k-step mod 2) * 2 + tile
constexpr int LOGIT_STEP = 2;
constexpr int DR = 32 / SW;          // rows per wavefront
__device__ __forceinline__ void put_logits(const MatView& W, const Tile& H, int at, const Share& S, const float (&inv)[2], const Wv& T,
                                  Ahead& cur, const Begin& next) {
    const int tile = S.slot & 1, part = S.slot >> 1;
    f32x4 acc[2][2];
    clear(acc);
    if (tile < W.tiles && part < W.ks) {
        mac_steps(acc, W, tile, H, T, part, LOGIT_STEP, cur, next);
        scaled(acc, inv, W.inv[tile]);
    } else {
        request(cur, next, T);
    }
    put_partial(acc, at, S.net * DIST_PARTS + S.slot, true, T);
}
__device__ __forceinline__ float logit(int at, int net, int row, int k) {
    const int col = k & 31;
    const int e = (((col >> 4) * 2 + (row >> 4)) * 64 + ((col >> 2) & 3) * 16 + (row & 15)) * 4 + (col & 3);
    const int p = at * 4 + (net * DIST_PARTS + (k >> 5)) * 1024 + e;
    return smem[p] + smem[p + 2048];
}
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_move<0x128>(x));
    x = fmaxf(x, dpp_move<0x124>(x));
    x = fmaxf(x, dpp_move<0x122>(x));
    return quarters_max(fmaxf(x, dpp_move<0x121>(x)));
}
// Softmax over the lanes < atoms (lane = atom): returns p and, through logp, log p (0 for idle lanes).
__device__ __forceinline__ float lane_softmax(float x, bool live, float& logp) {
    const float mx = wave_max(live ? x : -3.0e38f);
    const float e = live ? expf(x - mx) : 0.f;
    const float s = wsum(e);
    logp = live ? (x - mx) - logf(s) : 0.f;
    return e / s;
}
// The gradients at the logits (DR rows per wavefront, both networks) as a two-step tile per network at `at`, each row with
// its own scale (inverse scales to smem[inv_at + 32 net + row]).
__device__ __forceinline__ Tile logit_tile(int at, int net) { return Tile{at + net * 2 * 8 * CS, 8 * CS}; }
__device__ __forceinline__ void put_dlogits(const float (&dl)[2][DR], int at, int inv_at, const Wv& T) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int rr = 0; rr < DR; ++rr) {
            const int row = DR * T.wave + rr;
            float inv;
            const float s = scale_for(wave_max(fabsf(dl[i][rr])), inv);
            put_value<2>(logit_tile(at, i), row, T.lane, dl[i][rr], s);
            if (T.lane == 0) smem[inv_at + 32 * i + row] = inv;
        }
}

template <bool R = false>
__device__ __forceinline__ WvOf<R> wave_of(int other) {        // other: whether the workgroup reads the other lo terms
    WvOf<R> T;
    T.tid = threadIdx.x; T.lane = T.tid & 63; T.wave = __builtin_amdgcn_readfirstlane(T.tid >> 6);
    T.l15 = T.lane & 15; T.q = T.lane >> 4;
    T.hi = (unsigned)T.lane * 16u; T.lo = T.hi + 2048u + (unsigned)other * 2048u;
    return T;
}

// =============================================================================================
// V-learner step on one row tile (Algorithm 3; Section 3.2 for the lagged target policy): a' = pi^v(s'),
// t_i = Q'_i(s', a'), y = ret + boot * min(t_1, t_2); q_i = Q_i(s, a); loss partials, output deltas, and the deltas of
// every hidden layer of both critics.  NN networks side by side, TPW output tiles per wavefront.
// =============================================================================================
template <int NN, int TPW, int VAR, int R>
__device__ __forceinline__ void critic_step(const SplitCriticArgs& A) {
    warm_args<SplitCriticArgs>();
    constexpr bool SAC = VAR == VAR_SAC, DIST = VAR == VAR_DIST;
    const auto T = wave_of<R != GENERAL>(blockIdx.x & 1);
    const SplitShape& P = A.shape;
    const int B = A.B, L = P.L, a = P.a, HL = P.H[L - 1];
    const int r0 = blockIdx.x * 32, wg = blockIdx.x, nwg = gridDim.x;
    const int aw = SAC ? 2 * a : a;
    const Share S = NN == 2 ? Share{T.wave >> 2, T.wave & 3, 4} : Share{0, T.wave, SW};
    const Tile X = {P.x0, P.xplane}, H0 = {P.h0, P.hplane};
    const Tile H = {P.h0 + S.net * 2 * P.hplane, P.hplane};
    const SmallMem M = small_mem<2>(P.sm, P.as);
    const int steps = (P.o + a + 31) >> 5;
    Rows<2> xv;
    InputRows in = input_rows<2>(A.next_obs, P.o, nullptr, -1, a, P.as, r0, B);
    request_rows(xv, in, steps, T);
    Ahead cur;
    request(cur, begin_of(mat_view(A.pi[0], P.o, P.H[0]), T.wave, 0, 1), T);
    auto critic_begin = [&](const float* const (&mats)[2][PQL_MAX_HIDDEN + 1], int net) {
        return begin_of(mat_view(mats[net][0], P.o + a, P.H[0]), S.slot, 0, 1);
    };
    float ret[2], boot[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int row = r0 + 16 * n + T.l15;
        ret[n] = row < B ? A.ret[row] : 0.f;
        boot[n] = row < B ? A.boot[row] : 0.f;
    }
    put_rows(xv, in, steps, X, M.inv, 1.f, T);
    lds_barrier();
    // ---- a' from the lagged policy
    {
        const int parts = policy_forward<NN == 2 ? TPW / 2 : TPW, 2>(P, A.pi, X, H0, M, false, nullptr, aw, r0, B, T,
                                                                             cur, critic_begin(A.qt, S.net));
        const int col = T.tid & 31;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int row = (T.tid >> 5) + 16 * e;
            float act = 0.f;
            if (SAC) {      // a' ~ pi^v(.|s') with its log-density (soft target)
                float eps, raw;
                const float lp = sample_action<2>(H0.base, parts, row, col, a, A.pi_bias, r0, A.sac, act, eps, raw);
                if (col == 0) smem[M.logp + row] = lp;
            } else if (col < a) {
                act = tanhf(sum_partials<2>(H0.base, parts, row, col) + A.pi_bias[col]);
            }
            if (col < a) {
                if (R != REGULAR && P.alias) smem[M.act + row * M.as + col] = act;
                else put_value<2>(X, row, P.o + col, act, __uint_as_float(0x7F000000u - __float_as_uint(smem[M.inv + row])));
            }
        }
        lds_barrier();
        if (SAC) {      // y = ret + boot (min Q' - alpha log pi): the entropy term joins the reward part here
            const float alpha = expf(A.sac.log_alpha[0]);
#pragma unroll
            for (int n = 0; n < 2; ++n) ret[n] = ret[n] - boot[n] * (alpha * smem[M.logp + 16 * n + T.l15]);
        }
    }
    // ---- target critics, y
    f32x4 z[TPW][2][2], wo[TPW][2];
    const int tilesL = (HL + 31) >> 5;
    float y[2], mass[DR];                     // TD target of this lane's rows / projected target distribution of this wavefront's (lane = atom)
    const int atoms = DIST ? A.atoms : 2;
    const bool live = T.lane < atoms;
    const float dz = (A.v_max - A.v_min) / (float)(atoms - 1), zk = A.v_min + (float)T.lane * dz;
    auto dist_begin = [&](const float* const (&mats)[2][PQL_MAX_HIDDEN + 1]) {
        return begin_of(mat_view(mats[S.net][L], HL, atoms), S.slot & 1, S.slot >> 1, LOGIT_STEP);
    };
    const InputRows online = input_rows<2>(A.obs, P.o, A.act, -1, a, P.as, r0, B);
    {
        float tq[2][2];
#pragma unroll 1
        for (int ni = 0; ni < (NN == 2 ? 1 : 2); ++ni) {
            const int net = NN == 2 ? S.net : ni;
            if (ni > 0) lds_barrier();      // every wavefront has read the other critic's head partials (and activations)
            if (R != REGULAR && P.alias) {      // the input tile shares its place with the activations: bring the rows in again
                in.act_lds = M.act;
                request_rows(xv, in, steps, T);
                put_rows(xv, in, steps, X, M.inv, 1.f, T);
                lds_barrier();
            }
            if (!DIST && TPW <= 2) head_weights<TPW>(wo, A.wo_t[net], tilesL, S, T);      // (wider layers: no registers to spare until the products are done)
            const bool last = NN == 2 || ni == 1;
            critic_forward<NN>(z, P, A.qt, net, X, H, S, M, 0, nullptr, r0, B, T, cur,
                                    DIST ? dist_begin(A.qt) : (last ? critic_begin(A.q, S.net) : critic_begin(A.qt, 1)), xv, online,
                                    last);
            if (DIST) {
                // the target critic with the smaller mean supplies the next-state distribution; its atoms move to
                // clip(ret + boot z) and are projected back onto the support (lane k gathers atom k's mass)
                float inv[2];
                put_tile(z, tilesL, H, S, M, inv, T);
                put_logits(mat_view(A.qt[net][L], HL, atoms), H, H0.base, S, inv, T, cur, critic_begin(A.q, S.net));
                const float b0 = live ? A.bo_t[0][T.lane] : 0.f, b1 = live ? A.bo_t[1][T.lane] : 0.f;
#pragma unroll
                for (int rr = 0; rr < DR; ++rr) {
                    const int row = DR * T.wave + rr;
                    float unused;
                    const float t0 = lane_softmax(logit(H0.base, 0, row, T.lane) + b0, live, unused);
                    const float t1 = lane_softmax(logit(H0.base, 1, row, T.lane) + b1, live, unused);
                    const float pn = wsum(t0 * zk) <= wsum(t1 * zk) ? t0 : t1;
                    const bool rv = r0 + row < B;
                    const float rt = rv ? A.ret[r0 + row] : 0.f, bt = rv ? A.boot[r0 + row] : 0.f;
                    const float pos = (fminf(fmaxf(rt + bt * zk, A.v_min), A.v_max) - A.v_min) / dz;
                    float mm = 0.f;
                    for (int j = 0; j < atoms; ++j)         // j is wave-uniform: lane j's values come as scalars
                        mm += lane_value(pn, j) * fminf(fmaxf(1.f - fabsf(lane_value(pos, j) - (float)T.lane), 0.f), 1.f);
                    mass[rr] = live ? mm : 0.f;
                }
                continue;
            }
            float bias[NN], q[NN][2];
#pragma unroll
            for (int i = 0; i < NN; ++i) bias[i] = A.bo_t[NN == 2 ? i : net][0];
            if (TPW > 2) head_weights<TPW>(wo, A.wo_t[net], tilesL, S, T);
            head_values(z, wo, S, M, bias, q, T);
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                if (NN == 2) { tq[0][n] = q[0][n]; tq[1][n] = q[NN - 1][n]; }
                else if (ni == 0) tq[0][n] = q[0][n];
                else tq[1][n] = q[0][n];
            }
        }
#pragma unroll
        for (int n = 0; n < 2 && !DIST; ++n) {
            y[n] = ret[n] + boot[n] * fminf(tq[0][n], tq[1][n]);
            const int row = r0 + 16 * n + T.l15;
            if (T.wave == 0 && T.q == 0 && row < B) A.y[row] = y[n];
        }
    }
    // ---- online critics: forward, head, backward data path
    const float invB = 1.f / (float)B;
    in = online;
#pragma unroll 1
    for (int ni = 0; ni < (NN == 2 ? 1 : 2); ++ni) {
        const int net = NN == 2 ? S.net : ni;
        if (NN == 2 || (R != REGULAR && P.alias) || ni == 0) {
            if (ni > 0) request_rows(xv, in, steps, T);       // (else requested during the target critics)
            lds_barrier();     // the head partials of the networks before have been read, and so has their input
            put_rows(xv, in, steps, X, M.inv, 0.f, T);
        }
        lds_barrier();
        if (!DIST && TPW <= 2) head_weights<TPW>(wo, A.wo_q[net], tilesL, S, T);
        const Begin after = NN == 1 && ni == 0 ? critic_begin(A.q, 1) : begin_at(A.q[0][0]);
        const Begin back = L > 1 ? begin_of(mat_view(A.qT[net][L - 1], HL, P.H[L - 2]), S.slot, 0, 1) : after;
        critic_forward<NN>(z, P, A.q, net, X, H, S, M, DIST ? L : L - 1, A.h, r0, B, T, cur, DIST ? dist_begin(A.q) : back, xv, in,
                                false);
        if (DIST) {
            // cross-entropy against the projected target, dLoss/dlogits, and through the output layer to h_L
            float inv[2];
            const MatView WT = mat_view(A.qT[net][L], atoms, HL);
            put_tile(z, tilesL, H, S, M, inv, T);
            put_logits(mat_view(A.q[net][L], HL, atoms), H, H0.base, S, inv, T, cur, begin_of(WT, S.slot, 0, 1));
            float dl[2][DR], lsum[2] = {0.f, 0.f}, dsum[2] = {0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float b = live ? A.bo_q[i][T.lane] : 0.f;
#pragma unroll
                for (int rr = 0; rr < DR; ++rr) {
                    const int row = DR * T.wave + rr;
                    const bool rv = r0 + row < B;
                    float lp;
                    const float p = lane_softmax(logit(H0.base, i, row, T.lane) + b, live, lp);
                    const float sum = wsum(mass[rr]), ce = wsum(mass[rr] * lp);
                    if (rv) lsum[i] -= ce;
                    dl[i][rr] = (rv && live) ? (p * sum - mass[rr]) * invB : 0.f;
                    dsum[i] += dl[i][rr];
                    if (rv && live) A.dlg[i][(size_t)(r0 + row) * atoms + T.lane] = dl[i][rr];
                }
            }
            lds_barrier();                                   // the partial tiles have been read
            put_dlogits(dl, H0.base, M.part, T);
            float* sums = &smem[(H0.base + 4 * 8 * CS) * 4];  // [2][SW][64] output-bias gradients, behind the two tiles
            sums[T.wave * 64 + T.lane] = dsum[0];
            sums[(SW + T.wave) * 64 + T.lane] = dsum[1];
            if (T.lane == 0) { smem[M.part + 64 + T.wave] = lsum[0]; smem[M.part + 64 + SW + T.wave] = lsum[1]; }
            lds_barrier();
            if (T.tid < 128) {
                const int i = T.tid >> 6, k = T.tid & 63;
                float s = 0.f;
                for (int w = 0; w < SW; ++w) s += sums[(i * SW + w) * 64 + k];
                if (k < atoms) A.p_dbo[i][(size_t)wg * atoms + k] = s;
            } else if (T.tid < 130) {
                const int i = T.tid - 128;
                float s = 0.f;
                for (int w = 0; w < SW; ++w) s += smem[M.part + 64 + SW * i + w];
                A.p_loss[i * nwg + wg] = s;
            }
            row_inv(inv, M.part + 32 * net, T);
            f32x4 hl[2][2];
            load_ahead(A.h[net][L], HL, hl, S, r0, B, T);
            backward(z, WT, logit_tile(H0.base, net), S, inv, A.h[net][L], A.d[net][L], A.col[net][L] + (size_t)wg * HL, HL, r0, B, T,
                          cur, back, hl);
        } else {
        float bias[NN], q[NN][2];
#pragma unroll
        for (int i = 0; i < NN; ++i) bias[i] = A.bo_q[NN == 2 ? i : net][0];
        if (TPW > 2) head_weights<TPW>(wo, A.wo_q[net], tilesL, S, T);
        head_values(z, wo, S, M, bias, q, T);
        float d[2], loss = 0.f, db = 0.f;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int row = r0 + 16 * n + T.l15;
            const bool rv = row < B;
            const float qv = NN == 2 ? (S.net == 0 ? q[0][n] : q[NN - 1][n]) : q[0][n];
            const float e = rv ? qv - y[n] : 0.f;
            d[n] = 2.f * e * invB;
            loss += e * e;
            db += d[n];
            if (S.slot == 0 && T.q == 0 && rv) A.q_out[net][row] = qv;
        }
        if (S.slot == 0) {
            loss = row16_sum(loss);
            db = row16_sum(db);
            if (T.lane == 0) { A.p_loss[net * nwg + wg] = loss; A.p_db[net][wg] = db; }
        }
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const int tile = S.slot + t * S.waves;
            if (tile >= tilesL) continue;
            f32x4 dw[2], cs[2];
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    dw[m][r] = d[0] * z[t][m][0][r] + d[1] * z[t][m][1][r];
#pragma unroll
                    for (int n = 0; n < 2; ++n) z[t][m][n][r] = d[n] * wo[t][m][r] * delu_h(z[t][m][n][r]);
                    cs[m][r] = z[t][m][0][r] + z[t][m][1][r];
                }
            store_tile(A.d[net][L], HL, tile, z[t], r0, B, T);
            store_colsum(A.p_dw[net] + (size_t)wg * HL, HL, tile, dw, T);
            store_colsum(A.p_dbh[net] + (size_t)wg * HL, HL, tile, cs, T);
        }
        }
        float inv[2];
        f32x4 hv[2][2];
        for (int l = L; l >= 2; --l) {
            const int Hl = P.H[l - 1], Hp = P.H[l - 2];
            load_ahead(A.h[net][l - 1], Hp, hv, S, r0, B, T);
            put_tile(z, (Hl + 31) >> 5, H, S, M, inv, T);
            const MatView W = mat_view(A.qT[net][l - 1], Hl, Hp);
            backward(z, W, H, S, inv, A.h[net][l - 1], A.d[net][l - 1], A.col[net][l - 1] + (size_t)wg * Hp, Hp, r0, B, T, cur,
                          l > 2 ? begin_of(mat_view(A.qT[net][l - 2], Hp, P.H[l - 3]), S.slot, 0, 1) : after, hv);
        }
    }
}

// =============================================================================================
// P-learner step on one row tile (Algorithm 2: maximise min_i Q_i(s, pi(s))): a = pi(s), both critics on (s, a), the
// gradient -1/B through the smaller critic down to its action input, through tanh' and back through the policy.
// =============================================================================================
template <int NN, int TPW, int VAR, int R>
__device__ __forceinline__ void policy_step(const SplitPolicyArgs& A) {
    warm_args<SplitPolicyArgs>();
    constexpr bool SAC = VAR == VAR_SAC, DIST = VAR == VAR_DIST;
    const auto T = wave_of<R != GENERAL>(blockIdx.x & 1);
    const SplitShape& P = A.shape;
    constexpr int TPA = NN == 2 ? TPW / 2 : TPW;       // the policy's tiles per wavefront
    const int B = A.B, L = P.L, a = P.a, HL = P.H[L - 1], H1 = P.H[0];
    const int r0 = blockIdx.x * 32, wg = blockIdx.x;
    const int aw = SAC ? 2 * a : a;
    const Share S = NN == 2 ? Share{T.wave >> 2, T.wave & 3, 4} : Share{0, T.wave, SW};
    const Tile X = {P.x0, P.xplane}, H0 = {P.h0, P.hplane};
    const Tile H = {P.h0 + S.net * 2 * P.hplane, P.hplane};
    const SmallMem M = small_mem<2>(P.sm, P.as);
    const int atoms = DIST ? A.atoms : 2;
    const int steps = (P.o + a + 31) >> 5;
    const int col = T.tid & 31;                              // this thread's elements of an action-wide tile: rows row_of(e)
    auto row_of = [&](int e) { return (T.tid >> 5) + 16 * e; };
    Rows<2> xv;
    InputRows in = input_rows<2>(A.obs, P.o, nullptr, -1, a, P.as, r0, B);
    request_rows(xv, in, steps, T);
    Ahead cur;
    request(cur, begin_of(mat_view(A.pi[0], P.o, P.H[0]), T.wave, 0, 1), T);
    auto critic_begin = [&](int net) { return begin_of(mat_view(A.q[net][0], P.o + a, P.H[0]), S.slot, 0, 1); };
    // the first of the backward products of critic `net`: from its last hidden layer down, or its action gradient
    auto action_begin = [&](int net) { return begin_of(mat_view(A.w1aT[net], H1, a), 0, S.slot, S.waves); };
    auto back_begin = [&](int net) {
        return L > 1 ? begin_of(mat_view(A.qT[net][L - 1], HL, P.H[L - 2]), S.slot, 0, 1) : action_begin(net);
    };
    put_rows(xv, in, steps, X, M.inv, 1.f, T);
    lds_barrier();
    float act[2] = {0.f, 0.f}, eps[2] = {0.f, 0.f}, raw[2] = {0.f, 0.f}, logp[2] = {0.f, 0.f};
    {
        const int parts = policy_forward<TPA, 2>(P, A.pi, X, H0, M, true, A.hA, aw, r0, B, T, cur, critic_begin(S.net));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int row = row_of(e);
            if (SAC) logp[e] = sample_action<2>(H0.base, parts, row, col, a, A.pi_bias, r0, A.sac, act[e], eps[e], raw[e]);
            else if (col < a) act[e] = tanhf(sum_partials<2>(H0.base, parts, row, col) + A.pi_bias[col]);
            if (col < a) {
                if (R != REGULAR && P.alias) smem[M.act + row * M.as + col] = act[e];
                else put_value<2>(X, row, P.o + col, act[e], __uint_as_float(0x7F000000u - __float_as_uint(smem[M.inv + row])));
            }
        }
        lds_barrier();
    }
    // ---- both critics on (s, a)
    f32x4 z[TPW][2][2], wo[TPW][2];
    const int tilesL = (HL + 31) >> 5;
    float qv[2][2];
#pragma unroll 1
    for (int ni = 0; ni < (NN == 2 ? 1 : 2); ++ni) {
        const int net = NN == 2 ? S.net : ni;
        if (ni > 0) lds_barrier();          // every wavefront has read the other critic's head partials (and activations)
        if (R != REGULAR && P.alias) {
            in.act_lds = M.act;
            request_rows(xv, in, steps, T);
            put_rows(xv, in, steps, X, M.inv, 1.f, T);
            lds_barrier();
        }
        if (!DIST && TPW <= 2) head_weights<TPW>(wo, A.wo[net], tilesL, S, T);
        critic_forward<NN>(z, P, A.q, net, X, H, S, M, NN == 2 && !DIST ? L - 1 : L, A.h, r0, B, T, cur,
                                DIST ? begin_of(mat_view(A.q[net][L], HL, atoms), S.slot & 1, S.slot >> 1, LOGIT_STEP)
                                     : (NN == 1 && ni == 0 ? critic_begin(1) : back_begin(S.net)), xv, in, false);
        if (DIST) continue;
        float bias[NN], q[NN][2];
#pragma unroll
        for (int i = 0; i < NN; ++i) bias[i] = A.bo[NN == 2 ? i : net][0];
        if (TPW > 2) head_weights<TPW>(wo, A.wo[net], tilesL, S, T);
        head_values(z, wo, S, M, bias, q, T);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            if (NN == 2) { qv[0][n] = q[0][n]; qv[1][n] = q[NN - 1][n]; }
            else if (ni == 0) qv[0][n] = q[0][n];
            else qv[1][n] = q[0][n];
        }
    }
    const float invB = 1.f / (float)B;
    float pick0[2], pick1[2], loss = 0.f;
    if (DIST) {
        // Q_i = mean of critic i's distribution; the smaller one receives dJ/dlogit_k = -(1/B) p_k (z_k - Q), and from
        // there through its output layer to h_L
        const int net = S.net;
        const bool live = T.lane < atoms;
        const float zk = A.v_min + (float)T.lane * ((A.v_max - A.v_min) / (float)(atoms - 1));
        float inv[2];
        const MatView WT = mat_view(A.qT[net][L], atoms, HL);
        put_tile(z, tilesL, H, S, M, inv, T);
        put_logits(mat_view(A.q[net][L], HL, atoms), H, H0.base, S, inv, T, cur, begin_of(WT, S.slot, 0, 1));
        const float b0 = live ? A.bo[0][T.lane] : 0.f, b1 = live ? A.bo[1][T.lane] : 0.f;
        float dl[2][DR];
#pragma unroll
        for (int rr = 0; rr < DR; ++rr) {
            const int tr = DR * T.wave + rr;
            const bool rv = r0 + tr < B;
            float unused;
            const float p0 = lane_softmax(logit(H0.base, 0, tr, T.lane) + b0, live, unused);
            const float p1 = lane_softmax(logit(H0.base, 1, tr, T.lane) + b1, live, unused);
            const float q0 = wsum(p0 * zk), q1 = wsum(p1 * zk);
            const bool first = q0 <= q1;
            if (rv) loss += first ? q0 : q1;
            if (T.lane == 0 && rv) { A.q_out[0][r0 + tr] = q0; A.q_out[1][r0 + tr] = q1; }
            dl[0][rr] = (rv && live && first) ? -invB * p0 * (zk - q0) : 0.f;
            dl[1][rr] = (rv && live && !first) ? -invB * p1 * (zk - q1) : 0.f;
        }
        lds_barrier();                                       // the partial tiles have been read
        put_dlogits(dl, H0.base, M.part, T);
        if (T.lane == 0) smem[M.part + 64 + T.wave] = loss;
        lds_barrier();
        if (T.tid == 0) {
            float s = 0.f;
            for (int w = 0; w < SW; ++w) s += smem[M.part + 64 + w];
            A.p_loss[wg] = s;
        }
        row_inv(inv, M.part + 32 * net, T);
        f32x4 hl[2][2];
        load_ahead(A.h[net][L], HL, hl, S, r0, B, T);
        backward(z, WT, logit_tile(H0.base, net), S, inv, A.h[net][L], nullptr, nullptr, HL, r0, B, T, cur, back_begin(net), hl);
    }
#pragma unroll
    for (int n = 0; n < 2 && !DIST; ++n) {
        const int rr = r0 + 16 * n + T.l15;
        const bool rv = rr < B, first = qv[0][n] <= qv[1][n];
        pick0[n] = rv && first ? -invB : 0.f;
        pick1[n] = rv && !first ? -invB : 0.f;
        if (rv) loss += first ? qv[0][n] : qv[1][n];
        if (T.wave == 0 && T.q == 0 && rv) { A.q_out[0][rr] = qv[0][n]; A.q_out[1][rr] = qv[1][n]; }
    }
    if (!DIST && T.wave == 0) {
        loss = row16_sum(loss);
        if (T.lane == 0) A.p_loss[wg] = loss;
    }
    // ---- down to the critics' action input
    const int ks1 = (H1 + 31) >> 5;
    const int per = ks1 < S.waves ? ks1 : S.waves;           // partial tiles per network
    float gs[2] = {0.f, 0.f};                                       // dJ/da of this thread's elements
    float inv[2];
#pragma unroll 1
    for (int ni = 0; ni < (NN == 2 ? 1 : 2); ++ni) {
        const int net = NN == 2 ? S.net : ni;
        if (NN == 1) {
            head_weights<TPW>(wo, A.wo[net], tilesL, S, T);
#pragma unroll
            for (int t = 0; t < TPW; ++t)
                if (S.slot + t * S.waves < tilesL) load_tile(A.h[net][L], HL, S.slot + t * S.waves, z[t], r0, B, T);
                else clear(z[t]);
        }
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int n = 0; n < 2 && !DIST; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        z[t][m][n][r] = (net == 0 ? pick0[n] : pick1[n]) * wo[t][m][r] * delu_h(z[t][m][n][r]);
        f32x4 hv[2][2];
        for (int l = L; l >= 2; --l) {
            const int Hl = P.H[l - 1], Hp = P.H[l - 2];
            load_ahead(A.h[net][l - 1], Hp, hv, S, r0, B, T);
            put_tile(z, (Hl + 31) >> 5, H, S, M, inv, T);
            const MatView W = mat_view(A.qT[net][l - 1], Hl, Hp);
            backward(z, W, H, S, inv, A.h[net][l - 1], nullptr, nullptr, Hp, r0, B, T, cur,
                          l > 2 ? begin_of(mat_view(A.qT[net][l - 2], Hp, P.H[l - 3]), S.slot, 0, 1) : action_begin(net), hv);
        }
        put_tile(z, (H1 + 31) >> 5, H, S, M, inv, T);
        const MatView W = mat_view(A.w1aT[net], H1, a);
        const Begin after = NN == 1 && ni == 0 ? back_begin(1) : begin_of(mat_view(A.waT[L], aw, HL), T.wave, 0, 1);
        f32x4 acc[2][2];
        clear(acc);
        if (S.slot < W.ks) mac_steps(acc, W, 0, H, T, S.slot, S.waves, cur, after);
        else request(cur, after, T);
        scaled(acc, inv, W.inv[0]);
        put_partial(acc, H0.base, S.net * per + S.slot, S.slot < per, T);
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (col < a) gs[e] += sum_partials<2>(H0.base, NN * per, row_of(e), col);
    }
    float g[2] = {0.f, 0.f}, g2[2] = {0.f, 0.f};             // gradient at the output layer: column col, and a + col (raw)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int row = row_of(e);
        const bool rv = r0 + row < B;
        const float s = gs[e];
        if (!SAC) {
            g[e] = (col < a && rv) ? s * (1.f - act[e] * act[e]) : 0.f;
        } else if (col < a && rv) {
            // J = mean(alpha log pi - min Q): dJ/dmu = dJ/du = g + (alpha/B) 2a; dJ/draw = dJ/du sigma eps - alpha/B
            // inside the clip of log sigma, 0 outside
            const float ab = expf(A.sac.log_alpha[0]) / (float)B;
            const float ls = fminf(fmaxf(raw[e], SAC_LOG_STD_MIN), SAC_LOG_STD_MAX);
            g[e] = s * (1.f - act[e] * act[e]) + ab * 2.f * act[e];
            g2[e] = (raw[e] > SAC_LOG_STD_MIN && raw[e] < SAC_LOG_STD_MAX) ? g[e] * expf(ls) * eps[e] - ab : 0.f;
        }
        if (col < a && rv) {
            A.dPre[(size_t)(r0 + row) * aw + col] = g[e];
            if (SAC) A.dPre[(size_t)(r0 + row) * aw + a + col] = g2[e];
        }
    }
    lds_barrier();                                         // the partial tiles have been read
    // one k-step of 32 columns at the place of the activations, with its own row scales; column sums for the output bias
    const Tile D = {P.h0, 4 * CS};
    float* sums = &smem[P.h0 * 4 + 2 * 4 * CS * 4];          // [32][33] behind that tile
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int row = row_of(e);
        float inv_d;
        const float s = scale_for(half_max(fmaxf(fabsf(g[e]), fabsf(g2[e]))), inv_d);
        if (col == 0) smem[M.inv + row] = inv_d;
        if (!SAC || col < a || col >= aw) put_value<2>(D, row, col, g[e], s);
        if (SAC && col < a) put_value<2>(D, row, a + col, g2[e], s);
        if (!SAC || col < a) sums[row * 33 + col] = g[e];
        if (SAC && col < a) sums[row * 33 + a + col] = g2[e];
        if (SAC && col == 0) smem[M.logp + row] = r0 + row < B ? logp[e] : 0.f;
    }
    lds_barrier();
    if (T.tid < aw) {
        float s = 0.f;
        for (int r = 0; r < 32; ++r) s += sums[r * 33 + T.tid];
        A.colA[L + 1][(size_t)wg * aw + T.tid] = s;
    }
    if (SAC && T.tid == 64) {
        float s = 0.f;
        for (int r = 0; r < 32; ++r) s += smem[M.logp + r];
        A.p_logp[wg] = s;
    }
    // ---- back through the policy
    {
        const Share SA = {0, T.wave, SW};
        f32x4 za[TPA][2][2], hv[2][2];
        row_inv(inv, M.inv, T);
        load_ahead(A.hA[L], HL, hv, SA, r0, B, T);
        for (int l = L; l >= 1; --l) {
            const int N = P.H[l - 1];
            const MatView W = mat_view(A.waT[l], l == L ? aw : P.H[l], N);
            backward(za, W, l == L ? D : H0, SA, inv, A.hA[l], A.dA[l], A.colA[l] + (size_t)wg * N, N, r0, B, T, cur,
                          l > 1 ? begin_of(mat_view(A.waT[l - 1], N, P.H[l - 2]), T.wave, 0, 1) : begin_at(A.pi[0]), hv);
            if (l > 1) {
                load_ahead(A.hA[l - 1], P.H[l - 2], hv, SA, r0, B, T);
                put_tile(za, W.tiles, H0, SA, M, inv, T);
            }
        }
    }
}

// =============================================================================================
// Actor step on one row tile (Section 3.3, Algorithm 1): a = clip(pi(s) + sigma_i * eps, -1, 1).
// =============================================================================================
template <int TPW, int VAR, int NB = 2>
__device__ __forceinline__ void act_step(const SplitActArgs& A) {
    warm_args<SplitActArgs>();
    constexpr bool SAC = VAR == VAR_SAC;
    const auto T = wave_of<NB == 4>(0);          // tiles of 64 rows: states of up to XV steps
    const SplitShape& P = A.shape;
    const int B = A.B, a = P.a, r0 = blockIdx.x * 16 * NB;
    const int aw = SAC ? 2 * a : a;
    const Tile X = {P.x0, P.xplane}, H = {P.h0, P.hplane};
    const SmallMem M = small_mem<NB>(P.sm, P.as);
    const int steps = (P.o + 31) >> 5;
    Rows<NB> xv;
    InputRows in = input_rows<NB>(A.obs, P.o, nullptr, -1, 0, P.as, r0, B);
    if (A.nmean != nullptr) {
        in.norm = true;
        in.mean = rows_of(A.nmean, P.o, 0, 1, 1); in.rstd = rows_of(A.nrstd, P.o, 0, 1, 1);
    }
    request_rows(xv, in, steps, T);
    AheadOf<NB == 2 ? 2 : 1> cur;
    request(cur, begin_of(mat_view(A.pi[0], P.o, P.H[0]), T.wave, 0, 1), T);
    put_rows(xv, in, steps, X, M.inv, 0.f, T);
    lds_barrier();
    const int parts = policy_forward<TPW, NB>(P, A.pi, X, H, M, false, nullptr, aw, r0, B, T, cur, begin_at(A.pi[0]));
    const int col = T.tid & 31;
#pragma unroll
    for (int e = 0; e < NB; ++e) {
        const int row = (T.tid >> 5) + 16 * e, env = r0 + row;
        if (SAC) {
            float act, eps, raw;
            (void)sample_action<NB>(H.base, parts, row, col, a, A.pi_bias, r0, A.sac, act, eps, raw);
            if (col < a && env < B) A.act_out[(size_t)env * a + col] = act;
        } else if (col < a && env < B) {
            const GemmNoise& nz = A.noise;
            uint32_t w0, w1;
            philox4x32_10_f((uint32_t)(env * a + col), 2u, nz.ctr2, nz.ctr3, nz.key0, nz.key1, w0, w1);
            // double precision: (w >> 8) + 0.5 needs 25 significant bits
            const double u1 = ((double)(w0 >> 8) + 0.5) * 0x1p-24;
            const double u2 = ((double)(w1 >> 8) + 0.5) * 0x1p-24;
            const double eps = sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925286766559 * u2);
            double sigma = (double)nz.sigma_min;
            if (nz.sigma_rows > 1)
                sigma += ((double)env / (double)(nz.sigma_rows - 1)) * ((double)nz.sigma_max - (double)nz.sigma_min);
            const float x = tanhf(sum_partials<NB>(H.base, parts, row, col) + A.pi_bias[col]) + (float)(sigma * eps);
            A.act_out[(size_t)env * a + col] = fminf(fmaxf(x, -1.f), 1.f);
        }
    }
}

// =============================================================================================
// One wide layer for a list of networks (networks too wide or batches too large for the one-launch kernels; the twin
// critics, the target critics and the policy share launches): Y = ELU(X W + b), X W + b, or (D W^T) * ELU'(.) with column
// sums.  A workgroup brings 16 NB input rows into LDS as pairs, each row with its own scale, and its eight wavefronts sweep
// the output columns, 32 each per pass, the weights streaming from L2 in fragment order.  64 rows where they fit (inputs up
// to about 600 wide) read the weights half as often: at 32 rows they take twice the time of the matrix work, at 64 about as
// long.  Eight launches of 1024-512-256 at 32768 rows: 427 us each on fp32 MFMAs, 220 so, 212 with the requests of all rows
// together (222 TFLOP/s); one workgroup fits a compute unit, so what it reads first and writes last overlaps little.
// =============================================================================================
constexpr int LAYER_PIECES = 4;      // 16-byte pieces a lane brings in per row at once (1024 columns per half wavefront)
template <int NB>
__device__ __forceinline__ void layer_rows(const GemmProb& P, int K, int ks, int r0, int plane, float* inv_rows, const Wv& T) {
    const int K0 = P.seg[0].K, K1 = K - K0, c0 = T.lane & 31, chunks = 4 * ks;
    const int rows = P.M - r0 < 16 * NB ? P.M - r0 : 16 * NB;
    const __amdgpu_buffer_rsrc_t s0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P.seg[0].A) + (size_t)r0 * (size_t)K0, 0,
                                                                        rows * K0 * (int)sizeof(float), 0x00020000);
    const __amdgpu_buffer_rsrc_t s1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P.seg[K1 > 0 ? 1 : 0].A) + (size_t)r0 * (size_t)(K1 > 0 ? K1 : K0), 0,
                                                                        K1 > 0 ? rows * K1 * (int)sizeof(float) : 0, 0x00020000);
    const bool vec = K1 == 0 && (K0 & 3) == 0 && (reinterpret_cast<uintptr_t>(P.seg[0].A) & 15) == 0;
    auto piece = [&](int row, int chunk, f32x4 (&v)[2]) {      // chunk 4 step + q: columns k_slot(step, q, 0..7)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = k_slot(chunk >> 2, chunk & 3, 4 * h);
            if (vec) {
                v[h] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(s0, k < K0 ? (row * K0 + k) * 4 : NOWHERE, 0, 0));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = k + i - K0;
                    const float x = buf_load(s0, (unsigned)(c < 0 ? (row * K0 + k + i) * 4 : NOWHERE), 0);
                    const float y = K1 > 0 ? buf_load(s1, (unsigned)(c >= 0 && c < K1 ? (row * K1 + c) * 4 : NOWHERE), 0) : 0.f;
                    v[h][i] = c < 0 ? x : y;
                }
            }
        }
    };
    // 2 SW = 16 rows at a time; rows of up to RP pieces per lane: all NB rows' requests go out together (one row after the
    // other, a workgroup waited NB times before its first product)
    constexpr int RP = 4 * LAYER_PIECES / (2 * NB);              // NB = 4: 512 columns, NB = 2: 1024
    if (chunks <= 32 * RP) {
        f32x4 v[NB][RP][2];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int p = 0; p < RP; ++p)
                if (32 * p < chunks) piece(16 * i + 2 * T.wave + (T.lane >> 5), 32 * p + c0, v[i][p]);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int row = 16 * i + 2 * T.wave + (T.lane >> 5);
            float mx = 0.f;
#pragma unroll
            for (int p = 0; p < RP; ++p)
                if (32 * p < chunks) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(v[i][p][e >> 2][e & 3]));
                }
            float inv;
            const float s = scale_for(half_max(mx), inv);
            if (c0 == 0) inv_rows[row] = inv;
#pragma unroll
            for (int p = 0; p < RP; ++p) {
                const int chunk = 32 * p + c0;
                if (chunk >= chunks) continue;
                u32x4 hi, lo;
                split16x8(v[i][p][0], v[i][p][1], s, hi, lo);
                lds_units()[chunk * (16 * NB + 1) + row] = hi;
                lds_units()[plane + chunk * (16 * NB + 1) + row] = lo;
            }
        }
        return;
    }
    for (int i = 0; i < NB; ++i) {
        const int row = 16 * i + 2 * T.wave + (T.lane >> 5);
        f32x4 v[LAYER_PIECES][2];
        float mx = 0.f;
        for (int p0 = 0; p0 < chunks; p0 += 32 * LAYER_PIECES) {
#pragma unroll
            for (int p = 0; p < LAYER_PIECES; ++p)
                if (p0 + 32 * p < chunks) piece(row, p0 + 32 * p + c0, v[p]);
#pragma unroll
            for (int p = 0; p < LAYER_PIECES; ++p)
                if (p0 + 32 * p < chunks) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(v[p][e >> 2][e & 3]));
                }
        }
        float inv;
        const float s = scale_for(half_max(mx), inv);
        if (c0 == 0) inv_rows[row] = inv;
        for (int p0 = 0; p0 < chunks; p0 += 32 * LAYER_PIECES) {
            const bool again = chunks > 32 * LAYER_PIECES;       // rows of more than 1024 columns come twice
#pragma unroll
            for (int p = 0; p < LAYER_PIECES; ++p) {
                const int chunk = p0 + 32 * p + c0;
                if (p0 + 32 * p >= chunks) continue;
                if (again) piece(row, chunk, v[p]);
                if (chunk >= chunks) continue;
                u32x4 hi, lo;
                split16x8(v[p][0], v[p][1], s, hi, lo);
                lds_units()[chunk * (16 * NB + 1) + row] = hi;
                lds_units()[plane + chunk * (16 * NB + 1) + row] = lo;
            }
        }
    }
}

template <int NB>
__global__ __launch_bounds__(ST) void layer_rowtile_kernel(const GemmGroup) {
    const GemmGroup& G = kernel_args<GemmGroup>();
    const auto T = wave_of(blockIdx.x & 1);
    const int b = blockIdx.x;
    const GemmProb& P = G.p[record_of(G.p, &GemmProb::tile_begin, G.nprob, b)];
    const int K = P.seg[0].K + (P.nseg > 1 ? P.seg[1].K : 0), N = P.N, M = P.M;
    const int r0 = (b - P.tile_begin) * 16 * NB;
    const MatView W = mat_view(P.frag, K, N);
    const Tile X = {0, W.ks * 4 * (16 * NB + 1)};
    float* inv_rows = &smem[2 * X.plane * 4];
    Ahead cur;
    request(cur, begin_of(W, T.wave, 0, 1), T);
    layer_rows<NB>(P, K, W.ks, r0, X.plane, inv_rows, T);
    lds_barrier();
    float inv[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) inv[n] = inv_rows[16 * n + T.l15];
    const int epi = P.epi;
    for (int tile = T.wave; tile < W.tiles; tile += SW) {
        f32x4 acc[2][NB], hv[2][NB], bias[2];
        const float iw = W.inv[tile];
#pragma unroll
        for (int m = 0; m < 2; ++m) bias[m] = *reinterpret_cast<const f32x4*>(W.bias + 32 * tile + 16 * m + 4 * T.q);
        if (NB == 2 && epi == EPI_MUL_DELU) load_tile<NB>(P.aux, N, tile, hv, r0, M, T);      // (64 rows: too many registers)
        mac_steps(acc, W, tile, X, T, 0, 1, cur, begin_of(W, tile + SW, 0, 1));
        if (NB != 2 && epi == EPI_MUL_DELU) load_tile<NB>(P.aux, N, tile, hv, r0, M, T);
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const float f = inv[n] * iw;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (epi == EPI_MUL_DELU) {
                        acc[m][n][r] = acc[m][n][r] * f * delu_h(hv[m][n][r]);
                    } else {
                        const float x = __fmaf_rn(acc[m][n][r], f, bias[m][r]);
                        acc[m][n][r] = epi == EPI_BIAS_ELU ? elu_f(x) : x;
                    }
                }
        }
        store_tile<NB, true>(P.C, N, tile, acc, r0, M, T);
        if (P.colsum != nullptr) {      // one partial row per 32 batch rows
#pragma unroll
            for (int h = 0; h < NB / 2; ++h)
                if (r0 + 32 * h < M) {
                    const f32x4 cs[2] = {acc[0][2 * h] + acc[0][2 * h + 1], acc[1][2 * h] + acc[1][2 * h + 1]};
                    store_colsum(P.colsum + (size_t)(r0 / 32 + h) * (size_t)N, N, tile, cs, T);
                }
        }
    }
}

// LDS of a layer's input tile of `rows` rows.
static size_t layer_lds(const GemmProb& p, int rows) {
    const int K = p.seg[0].K + (p.nseg > 1 ? p.seg[1].K : 0);
    return 2 * (size_t)((K + 31) / 32 * 4) * (rows + 1) * 16 + rows * sizeof(float);
}

bool layer_rowtile_ok(const GemmGroup& g) {
    long wgs = 0;
    for (int i = 0; i < g.nprob; ++i) {
        const GemmProb& p = g.p[i];
        if (p.frag == nullptr) return false;
        if (p.epi != EPI_BIAS_ELU && p.epi != EPI_BIAS && p.epi != EPI_MUL_DELU) return false;
        if (p.epi == EPI_MUL_DELU ? (p.aux == nullptr || p.ldaux != p.N) : (p.bias == nullptr || p.colsum != nullptr)) return false;
        if (p.nseg < 1 || p.nseg > 2 || p.ldc != p.N) return false;
        if (p.N < 128 || p.M < 1) return false;
        for (int s = 0; s < p.nseg; ++s)
            if (p.seg[s].K < 1 || p.seg[s].lda != p.seg[s].K) return false;
        if (layer_lds(p, 32) > SPLIT_LDS) return false;
        wgs += (p.M + 31) / 32;
    }
    return wgs >= 256;
}

hipError_t layer_rowtile_launch(GemmGroup& g, hipStream_t stream) {
    if (!layer_rowtile_ok(g)) return hipErrorInvalidValue;
    long wgs64 = 0;
    bool fits = true;
    for (int i = 0; i < g.nprob; ++i) {
        wgs64 += (g.p[i].M + 63) / 64;
        if (layer_lds(g.p[i], 64) > SPLIT_LDS) fits = false;
    }
    const int rows = fits && wgs64 >= 256 ? 64 : 32;             // (a workgroup for every compute unit comes first)
    int total = 0;
    size_t lds = 0;
    double flops = 0.0;
    for (int i = 0; i < g.nprob; ++i) {
        GemmProb& p = g.p[i];
        p.tile_begin = total;
        p.tiles_m = (p.M + rows - 1) / rows; p.tiles_n = 1; p.splits = 1; p.k_chunk = 0;
        total += p.tiles_m;
        for (int s = 0; s < p.nseg; ++s) flops += 2.0 * p.M * (double)p.N * p.seg[s].K;
        const size_t bytes = layer_lds(p, rows);
        if (bytes > lds) lds = bytes;
    }
    g.total_tiles = total;
    static LdsLimit configured, configured64;
    const hipError_t e = rows == 64 ? set_lds_limit(reinterpret_cast<const void*>(layer_rowtile_kernel<4>), lds, configured64)
                                    : set_lds_limit(reinterpret_cast<const void*>(layer_rowtile_kernel<2>), lds, configured);
    if (e != hipSuccess) return e;
    const ProfSlot ps = prof_slot();
    if (rows == 64) PQL_LAUNCH(ps, layer_rowtile_kernel<4>, dim3(total), dim3(ST), lds, stream, g);
    else            PQL_LAUNCH(ps, layer_rowtile_kernel<2>, dim3(total), dim3(ST), lds, stream, g);
    prof_commit(ps, KID_LAYER_ROWTILE, ps.on ? flops : 0.0, 0.0);
    return hipGetLastError();
}

// ---- host side ------------------------------------------------------------------------------------------------
// LDS plan of a shape: the activation tiles of `nets` networks, the input tile behind them or, where that does not fit, in
// their place, and the small arrays.  Returns the bytes, 0 if the shape does not fit at all.
static size_t plan_lds(SplitShape& p, int nets, int in_cols, bool dist = false, int nb = 2) {
    int w = 0;
    for (int l = 0; l < p.L; ++l) w = p.H[l] > w ? p.H[l] : w;
    p.hplane = (w + 31) / 32 * 4 * (16 * nb + 1);
    p.xplane = (in_cols + 31) / 32 * 4 * (16 * nb + 1);
    p.as = p.a | 1;
    const int h_units = nets * 2 * p.hplane;
    const size_t small = sizeof(float) * (size_t)small_floats(nb, p.as);
    // the policy step's output-layer tile and its column sums also live in the place of the activations
    // (distributional critics: eight partial tiles of logits)
    const int least = dist ? 2 * DIST_PARTS * 256 : 2 * 4 * (16 * nb + 1) + 16 * nb * 33 / 4;
    p.h0 = 0; p.x0 = h_units < least ? least : h_units; p.alias = 0;
    size_t units = (size_t)p.x0 + 2 * (size_t)p.xplane;
    if (units * 16 + small > SPLIT_LDS) {
        p.x0 = 0; p.alias = 1;
        units = (size_t)(h_units > 2 * p.xplane ? h_units : 2 * p.xplane);
        if (units < (size_t)least) units = (size_t)least;
    }
    p.sm = (int)units * 4;
    const size_t bytes = units * 16 + small;
    return bytes <= SPLIT_LDS ? bytes : 0;
}
static int widest(const SplitShape& p) {
    int w = 0;
    for (int l = 0; l < p.L; ++l) w = p.H[l] > w ? p.H[l] : w;
    return w;
}

bool split_shape_ok(int o, int a, int aw, const int* H, int L, bool dist) {
    if (aw > FUSED_MAX_ACT || o > SPLIT_MAXW) return false;
    SplitShape p;
    p.o = o; p.a = a; p.L = L;
    for (int l = 0; l < L; ++l) {
        if (H[l] > SPLIT_MAXW) return false;
        p.H[l] = H[l];
    }
    if (dist && widest(p) > 512) return false;
    return plan_lds(p, widest(p) <= 512 ? 2 : 1, o + a, dist) != 0;
}

// ---- kernels ------------------------------------------------------------------------------------------------------
// fused_*: every layer at most 256 wide (two output tiles per wavefront); chain_*: at most 512, scalar critics and deterministic
// policy (four); split_*: at most 512 with the other variants, and layers above 512 with the critics one after the other.
template <int VAR, int R>
__global__ __launch_bounds__(ST) void fused_critic_kernel(const SplitCriticArgs) { critic_step<2, 2, VAR, R>(kernel_args<SplitCriticArgs>()); }
template <int VAR, int R>
__global__ __launch_bounds__(ST) void chain_critic_kernel(const SplitCriticArgs) { critic_step<2, 4, VAR, R>(kernel_args<SplitCriticArgs>()); }
template <int NN, int TPW, int VAR, int R>
__global__ __launch_bounds__(ST) void split_critic_kernel(const SplitCriticArgs) { critic_step<NN, TPW, VAR, R>(kernel_args<SplitCriticArgs>()); }
template <int VAR, int R>
__global__ __launch_bounds__(ST) void fused_policy_kernel(const SplitPolicyArgs) { policy_step<2, 2, VAR, R>(kernel_args<SplitPolicyArgs>()); }
template <int VAR, int R>
__global__ __launch_bounds__(ST) void chain_policy_kernel(const SplitPolicyArgs) { policy_step<2, 4, VAR, R>(kernel_args<SplitPolicyArgs>()); }
template <int NN, int TPW, int VAR, int R>
__global__ __launch_bounds__(ST) void split_policy_kernel(const SplitPolicyArgs) { policy_step<NN, TPW, VAR, R>(kernel_args<SplitPolicyArgs>()); }
template <int VAR, int NB>
__global__ __launch_bounds__(ST) void fused_act_kernel(const SplitActArgs) { act_step<1, VAR, NB>(kernel_args<SplitActArgs>()); }
template <int NB>
__global__ __launch_bounds__(ST) void chain_act_kernel(const SplitActArgs) { act_step<2, VAR_PLAIN, NB>(kernel_args<SplitActArgs>()); }

#define SPLIT_LAUNCH_ROWS(KERNEL, KID, ROWS)                                                                       \
    do {                                                                                                           \
        static LdsLimit configured;                                                                                \
        const hipError_t le = set_lds_limit(reinterpret_cast<const void*>(KERNEL), lds, configured);               \
        if (le != hipSuccess) return le;                                                                           \
        const ProfSlot ps = prof_slot();                                                                           \
        PQL_LAUNCH(ps, (KERNEL), dim3((a.B + (ROWS) - 1) / (ROWS)), dim3(ST), lds, stream, a);                     \
        prof_commit(ps, KID, flops, 0.0);                                                                          \
        return hipGetLastError();                                                                                  \
    } while (0)
#define SPLIT_LAUNCH(KERNEL, KID) SPLIT_LAUNCH_ROWS(KERNEL, KID, 32)
// Picks the kernel of one step: shape and policy variant are fixed at compile time, one kernel for each pair that occurs (the
// class only decides what a launch is filed under).
#define SPLIT_PICK(STEP, VAR)                                                                                      \
    do {                                                                                                           \
        const bool r = regular(p);                                                                                 \
        if (w <= 256 && r && !p.alias)                                                                             \
            SPLIT_LAUNCH((fused_##STEP##_kernel<VAR, REGULAR>), kind == SPLIT_FUSED ? fused_kid : split_kid);      \
        if (w <= 256) SPLIT_LAUNCH((fused_##STEP##_kernel<VAR, GENERAL>), kind == SPLIT_FUSED ? fused_kid : split_kid);\
        if (w <= 512 && VAR == VAR_PLAIN && r && !p.alias)                                                         \
            SPLIT_LAUNCH((chain_##STEP##_kernel<VAR_PLAIN, REGULAR>), kind == SPLIT_CHAIN ? chain_kid : split_kid);\
        if (w <= 512 && VAR == VAR_PLAIN && r)                                                                     \
            SPLIT_LAUNCH((chain_##STEP##_kernel<VAR_PLAIN, REGULAR_ALIAS>), kind == SPLIT_CHAIN ? chain_kid : split_kid);\
        if (w <= 512 && VAR == VAR_PLAIN)                                                                          \
            SPLIT_LAUNCH((chain_##STEP##_kernel<VAR_PLAIN, GENERAL>), kind == SPLIT_CHAIN ? chain_kid : split_kid);\
        constexpr int V2 = VAR == VAR_PLAIN ? VAR_SAC : VAR, V1 = VAR == VAR_DIST ? VAR_PLAIN : VAR;               \
        if (w <= 512 && r) SPLIT_LAUNCH((split_##STEP##_kernel<2, 4, V2, REGULAR_ALIAS>), split_kid);              \
        if (w <= 512) SPLIT_LAUNCH((split_##STEP##_kernel<2, 4, V2, GENERAL>), split_kid);                         \
        if (VAR != VAR_DIST && r) SPLIT_LAUNCH((split_##STEP##_kernel<1, 4, V1, REGULAR_ALIAS>), split_kid);       \
        if (VAR != VAR_DIST) SPLIT_LAUNCH((split_##STEP##_kernel<1, 4, V1, GENERAL>), split_kid);                  \
    } while (0)

// Whether the kernels without the rare paths take this shape (after plan_lds).
static bool regular(const SplitShape& p) {
    for (int l = 0; l < p.L; ++l)
        if (p.H[l] & 3) return false;
    return p.o + p.a <= 32 * XV;
}
// Multiply-adds of the policy for one state.
static double policy_weights(const SplitShape& p, int aw) {
    double n = (double)p.o * p.H[0] + (double)p.H[p.L - 1] * aw;
    for (int l = 1; l < p.L; ++l) n += (double)p.H[l - 1] * p.H[l];
    return n;
}
// Whether the Actor step takes tiles of 64 rows, which read the weights half as often: a tile takes five thirds of the time of one
// of 32, one tile at a time fits a compute unit, and the launch takes as many rounds of 256 as it has tiles for.  us per call with 32
// / 64 rows at 8193, 16384, 20000, 24576, 28000 and 32768 environments: 256-256 25.7 / 23.6, 28.0 / 24.4, 37.3 / 41.4, 38.0 / 41.3,
// 47.1 / 41.3, 48.2 / 41.8; 512-256-128 41.4 / 36.1, 45.0 / 38.7, 62.6 / 66.6, 64.2 / 66.5, 81.3 / 67.1, 83.0 / 70.5.
// What does not get cheaper is the output: a lane draws the noise of its action column for two or four rows, one after the other, and
// each takes 0.6 - 0.8 us longer where a row has at most four.  With so few actions, or one narrow layer, that and the input are most
// of a tile: 64 rows take 11 / 6 of the time of 32 (one narrow layer: twice), and a last round of a few tiles half a round.  us at
// 8193, 16384, 24577, 32768, 40961, 49153, 57344 and 65537 environments: 250-64-4 18.8 / 22.2, 23.1 / 22.1, 34.5 / 37.3, 38.6 / 37.9,
// 50.0 / 53.0, 58.2 / 59.3, 62.4 / 68.6, 73.7 / 74.4; 20-64-32-4 17.5 / 20.4, 22.2 / 20.5, 32.2 / 33.6, 36.2 / 33.9, 45.7 / 47.1,
// 52.6 / 51.5, 57.4 / 60.6, 66.7 / 64.5.  The bounds on weights, at 8193: 60-256-256-4 (82 k) 25.7 / 26.4, 108-256-256-256-4 (160 k)
// 35.3 / 34.4; stochastic, 20-64-32-4 (4 k) 19.7 / 20.8, 60-64-64-4 (8 k) 22.2 / 21.7.
static bool takes_64_rows(const SplitShape& p, int B, bool sac) {
    auto rounds = [&](int rows) { return ((B + rows - 1) / rows + 255) / 256; };
    const bool narrow = p.L == 1 && p.H[0] <= 64, few = p.a <= 4;
    const double weights = policy_weights(p, sac ? 2 * p.a : p.a);
    if (!(few && (narrow || weights < (sac ? 4096 : 98304))) && !(narrow && !sac)) return 5 * rounds(64) < 3 * rounds(32);
    auto halves = [&](int rows) {
        const int tiles = (B + rows - 1) / rows, last = tiles % 256;
        return 2 * (tiles / 256) + (last == 0 ? 0 : (last <= 32 ? 1 : 2));
    };
    return narrow ? 2 * halves(64) <= halves(32) : 11 * halves(64) < 6 * halves(32);
}
// Rows per tile of the Actor step (0: its tiles do not fit) and its LDS plan.  Its input is the states alone; the kernels on tiles of
// 64 rows have no path for states of more than XV steps.
static int plan_act(SplitShape& p, int B, bool sac, size_t& lds) {
    if (p.o <= 32 * XV && takes_64_rows(p, B, sac) && (lds = plan_lds(p, 1, p.o, false, 4)) != 0) return 64;
    return (lds = plan_lds(p, 1, p.o)) != 0 ? 32 : 0;
}
int split_act_rows(SplitShape p, int B, bool sac) {
    size_t lds;
    return plan_act(p, B, sac, lds);
}
static bool kind_fits(int kind, int w) {
    return kind == SPLIT_FUSED ? w <= 256 : (kind == SPLIT_CHAIN ? w <= 512 : true);
}

hipError_t split_critic_launch(SplitCriticArgs& a, int kind, hipStream_t stream) {
    SplitShape& p = a.shape;
    const int w = widest(p), aw = a.sac.on ? 2 * p.a : p.a;
    if (!split_shape_ok(p.o, p.a, aw, p.H, p.L) || !kind_fits(kind, w) || (a.atoms >= 2 && (w > 512 || a.sac.on))) return hipErrorInvalidValue;
    const size_t lds = plan_lds(p, w <= 512 ? 2 : 1, p.o + p.a, a.atoms >= 2);
    const double outs = a.atoms >= 2 ? (double)a.atoms : 1.0;
    double pa = (double)p.o * p.H[0], pc = (double)(p.o + p.a) * p.H[0], pb = 0.0;
    for (int l = 1; l < p.L; ++l) { const double x = (double)p.H[l - 1] * p.H[l]; pa += x; pc += x; pb += x; }
    pa += (double)p.H[p.L - 1] * aw; pc += p.H[p.L - 1] * outs; pb += p.H[p.L - 1] * outs;
    const double flops = 2.0 * a.B * (pa + 4.0 * pc + 2.0 * pb);
    const int fused_kid = KID_FUSED_CRITIC, chain_kid = KID_CHAIN_CRITIC, split_kid = KID_SPLIT_CRITIC;
    if (a.sac.on) SPLIT_PICK(critic, VAR_SAC);
    if (a.atoms >= 2) SPLIT_PICK(critic, VAR_DIST);
    SPLIT_PICK(critic, VAR_PLAIN);
    return hipErrorInvalidValue;
}

hipError_t split_policy_launch(SplitPolicyArgs& a, int kind, hipStream_t stream) {
    SplitShape& p = a.shape;
    const int w = widest(p), aw = a.sac.on ? 2 * p.a : p.a;
    if (!split_shape_ok(p.o, p.a, aw, p.H, p.L) || !kind_fits(kind, w) || (a.atoms >= 2 && (w > 512 || a.sac.on))) return hipErrorInvalidValue;
    const size_t lds = plan_lds(p, w <= 512 ? 2 : 1, p.o + p.a, a.atoms >= 2);
    const double outs = a.atoms >= 2 ? (double)a.atoms : 1.0;
    double pa = (double)p.o * p.H[0], pc = (double)(p.o + p.a) * p.H[0], pb = (double)p.a * p.H[0], pab = 0.0;
    for (int l = 1; l < p.L; ++l) { const double x = (double)p.H[l - 1] * p.H[l]; pa += x; pc += x; pb += x; pab += x; }
    pa += (double)p.H[p.L - 1] * aw; pab += (double)p.H[p.L - 1] * aw; pc += p.H[p.L - 1] * outs; pb += p.H[p.L - 1] * outs;
    const double flops = 2.0 * a.B * (pa + 2.0 * pc + 2.0 * pb + pab);
    const int fused_kid = KID_FUSED_POLICY, chain_kid = KID_CHAIN_POLICY, split_kid = KID_SPLIT_POLICY;
    if (a.sac.on) SPLIT_PICK(policy, VAR_SAC);
    if (a.atoms >= 2) SPLIT_PICK(policy, VAR_DIST);
    SPLIT_PICK(policy, VAR_PLAIN);
    return hipErrorInvalidValue;
}

hipError_t split_act_launch(SplitActArgs& a, int kind, hipStream_t stream) {
    SplitShape& p = a.shape;
    const int w = widest(p), aw = a.sac.on ? 2 * p.a : p.a;
    if (!split_shape_ok(p.o, p.a, aw, p.H, p.L) || w > 512) return hipErrorInvalidValue;
    size_t lds;
    const int rows = plan_act(p, a.B, a.sac.on != 0, lds);
    if (rows == 0) return hipErrorInvalidValue;
    const double flops = 2.0 * a.B * policy_weights(p, aw);
    if (kind != SPLIT_FUSED) {
        if (a.sac.on) return hipErrorInvalidValue;          // (no class of stochastic policies takes this kernel)
        if (rows == 64) SPLIT_LAUNCH_ROWS(chain_act_kernel<4>, KID_CHAIN_ACT, 64);
        SPLIT_LAUNCH(chain_act_kernel<2>, KID_CHAIN_ACT);
    }
    if (a.sac.on) {
        if (rows == 64) SPLIT_LAUNCH_ROWS((fused_act_kernel<VAR_SAC, 4>), KID_FUSED_ACT, 64);
        SPLIT_LAUNCH((fused_act_kernel<VAR_SAC, 2>), KID_FUSED_ACT);
    }
    if (rows == 64) SPLIT_LAUNCH_ROWS((fused_act_kernel<VAR_PLAIN, 4>), KID_FUSED_ACT, 64);
    SPLIT_LAUNCH((fused_act_kernel<VAR_PLAIN, 2>), KID_FUSED_ACT);
}

}  // namespace pql
