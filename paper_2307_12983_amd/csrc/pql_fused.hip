// One launch per layer on 32-row tiles with fp32 MFMAs, for networks and batches that the one-launch kernels
// (pql_split.hip) leave to a launch per layer: wide layers, and the action-wide products around them.
#include "pql_rowtile.h"

namespace pql {


// =============================================================================================
// One wide layer on row tiles, for networks whose layers are too wide for the one-launch
// kernels: Y = act(X W + b), or delta W^T * ELU'(.) with W^T materialised by transpose_kernel, for a
// list of problems (the twin critics, the target critics and the policy share launches).  A
// workgroup stages 32 input rows in LDS once and its eight wavefronts sweep the output columns, 32
// each per pass, with the weights streamed from L2 as in the chained kernels; nothing but the input
// rows and the output tile touches memory.  Two workgroups fit a compute unit while the input tile
// stays below 80 KB (sixteen wavefronts: the kernel is held to 128 registers, and has none to
// spare: requesting the first weight chunks ahead of the input rows spilled and ran 6 % slower).
// =============================================================================================
__global__ __launch_bounds__(FT, 4) void layer_rowtile_kernel(const GemmGroup g) {
    Lanes T;
    T.tid = threadIdx.x; T.lane = T.tid & 63; T.wave = __builtin_amdgcn_readfirstlane(T.tid >> 6); T.l32 = T.lane & 31; T.half = T.lane >> 5;
    const int b = blockIdx.x;
    int pi = 0;
    for (int i = 1; i < g.nprob; ++i)
        if (b >= g.p[i].tile_begin) pi = i;
    const GemmProb& P = g.p[pi];
    // tiles_n holds the row tiles per workgroup: 2 for layers of at most 128 columns (four wavefronts
    // cover those, the other four take a second row tile), else 1
    const int RT = P.tiles_n, CW = FW / RT;
    const int rt = T.wave / CW, cw = T.wave - rt * CW;
    const int M = P.M, N = P.N;
    const int K0 = P.seg[0].K, K1 = P.nseg > 1 ? P.seg[1].K : 0;
    const int S0 = ((K0 + 7) & ~7) + 4, S1 = K1 > 0 ? ((K1 + 7) & ~7) + 4 : 0;
    const int rw = (b - P.tile_begin) * BMF * RT;
    for (int t = 0; t < RT; ++t) {
        load_rows(T, t * BMF * S0, S0, P.seg[0].A, K0, rw + t * BMF, M);
        if (K1 > 0) load_rows(T, RT * BMF * S0 + t * BMF * S1, S1, P.seg[1].A, K1, rw + t * BMF, M);
    }
    __syncthreads();
    const int r0 = rw + rt * BMF;
    if (r0 >= M) return;                 // (no barrier follows)
    const int XA = rt * BMF * S0, XB = RT * BMF * S0 + rt * BMF * S1;
    const int epi = P.epi;
    const int ldc = P.ldc, ldaux = P.ldaux;
    const int lrow = 4 * T.half;
    const bool full = r0 + BMF <= M;
    for (int n0 = cw * 32; n0 < N; n0 += 32 * CW) {
        const int n = n0 + T.l32;
        const bool n_ok = n < N;
        const int ncol = n_ok ? n : N - 1;
        const float bv = epi == EPI_MUL_DELU ? 0.f : P.bias[ncol];
        floatx16 acc[1];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = 0.f;
        const int in0[1] = {XA};
        const float* const W0[1] = {P.seg[0].B};
        if (K1 > 0) {
            float bs[1][16], bf[1][16];
            const int in1[1] = {XB};
            const float* const W1[1] = {P.seg[1].B};
            prefetch_first_chunk<1>(bs, W1, K1, P.seg[1].ldb, ncol, T, 0, 1);
            prefetch_first_chunk<1>(bf, W0, K0, P.seg[0].ldb, ncol, T, 0, 1);
            mac_segment<1>(acc, in1, S1, K1, W1, P.seg[1].ldb, ncol, T, 0, 1, true, bs);
            mac_segment<1>(acc, in0, S0, K0, W0, P.seg[0].ldb, ncol, T, 0, 1, true, bf);
        } else {
            mac_segment<1>(acc, in0, S0, K0, W0, P.seg[0].ldb, ncol, T, 0, 1);
        }
        float* __restrict__ gbase = P.C + (size_t)(r0 + lrow) * (size_t)ldc + n;
        if (epi == EPI_MUL_DELU) {
            // backward data path: delta = acc * ELU'(z) with the activation read from memory; the
            // tile's column sums are one partial row of the bias gradient
            const float* __restrict__ abase = P.aux + (size_t)(r0 + lrow) * (size_t)ldaux + ncol;
            float h[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r >> 2) + (r & 3);
                h[r] = (full || r0 + lrow + dr < M) ? abase[(size_t)dr * (size_t)ldaux] : 0.f;
            }
            float cs = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r >> 2) + (r & 3);
                const bool rv = full || r0 + lrow + dr < M;
                const float x = rv ? acc[0][r] * delu_h(h[r]) : 0.f;
                if (n_ok && rv) gbase[(size_t)dr * (size_t)ldc] = x;
                cs += x;
            }
            if (P.colsum != nullptr) {
                cs += __shfl_xor(cs, 32);
                if (T.half == 0 && n_ok) P.colsum[(size_t)((b - P.tile_begin) * RT + rt) * (size_t)N + n] = cs;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r >> 2) + (r & 3);
                float x = acc[0][r] + bv;
                if (epi == EPI_BIAS_ELU) x = elu_f(x);
                if (n_ok && (full || r0 + lrow + dr < M)) gbase[(size_t)dr * (size_t)ldc] = x;
            }
        }
    }
}

// Whether a launch of X W products (B operand [K][N] row-major) can take the row-tile layer kernel:
// bias (+ ELU) epilogues, or the backward data path's ELU' epilogue with column sums (one partial
// row per 32 batch rows); dense input rows (row stride = width), enough columns to occupy the eight wavefronts, enough rows to
// fill the chip, input tiles that fit LDS, and weights within reach of a 32-bit buffer offset.
bool layer_rowtile_ok(const GemmGroup& g) {
    long wgs = 0;
    for (int i = 0; i < g.nprob; ++i) {
        const GemmProb& p = g.p[i];
        if (p.epi != EPI_BIAS_ELU && p.epi != EPI_BIAS && p.epi != EPI_MUL_DELU) return false;
        if (p.epi == EPI_MUL_DELU ? (p.aux == nullptr || p.ldaux < p.N) : (p.bias == nullptr || p.colsum != nullptr)) return false;
        if (p.nseg < 1 || p.nseg > 2 || p.ldc < p.N) return false;
        if (p.N < 128 || p.M < 1) return false;
        size_t floats = 0;
        for (int s = 0; s < p.nseg; ++s) {
            const GemmSeg& q = p.seg[s];
            if (q.K < 1 || q.lda != q.K || q.ldb < p.N) return false;
            if ((size_t)q.K * (size_t)q.ldb * sizeof(float) >= ((size_t)1 << 31)) return false;
            floats += (size_t)BMF * (size_t)(((q.K + 7) & ~7) + 4);
        }
        if (floats * sizeof(float) > 150 * 1024) return false;
        wgs += (p.M + BMF - 1) / BMF;
    }
    return wgs >= 256;
}

static size_t layer_tile_floats(const GemmProb& p) {
    size_t floats = 0;
    for (int s = 0; s < p.nseg; ++s) floats += (size_t)BMF * (size_t)(((p.seg[s].K + 7) & ~7) + 4);
    return floats;
}

hipError_t layer_rowtile_launch(GemmGroup& g, hipStream_t stream) {
    // Narrow layers (at most 128 columns) take two row tiles per workgroup, if the launch still has
    // a workgroup for every compute unit and the two input tiles fit LDS.
    long wgs2 = 0;
    bool fits2 = true;
    for (int i = 0; i < g.nprob; ++i) {
        const GemmProb& p = g.p[i];
        const int rt = p.N <= 128 ? 2 : 1;
        wgs2 += (p.M + BMF * rt - 1) / (BMF * rt);
        if (rt == 2 && 2 * layer_tile_floats(p) * sizeof(float) > 150 * 1024) fits2 = false;
    }
    const bool pair_rows = fits2 && wgs2 >= 256;
    int total = 0;
    size_t lds = 0;
    double flops = 0.0;
    for (int i = 0; i < g.nprob; ++i) {
        GemmProb& p = g.p[i];
        const int rt = (pair_rows && p.N <= 128) ? 2 : 1;
        p.tile_begin = total;
        p.tiles_m = (p.M + BMF * rt - 1) / (BMF * rt); p.tiles_n = rt; p.splits = 1; p.k_chunk = 0;
        total += p.tiles_m;
        for (int s = 0; s < p.nseg; ++s) flops += 2.0 * p.M * (double)p.N * p.seg[s].K;
        const size_t bytes = rt * layer_tile_floats(p) * sizeof(float);
        if (bytes > lds) lds = bytes;
    }
    g.total_tiles = total;
    if (total == 0) return hipSuccess;
    static LdsLimit configured;
    const hipError_t e = set_lds_limit(reinterpret_cast<const void*>(layer_rowtile_kernel), lds, configured);
    if (e != hipSuccess) return e;
    const ProfSlot ps = prof_slot();
    PQL_LAUNCH(ps, layer_rowtile_kernel, dim3(total), dim3(FT), lds, stream, g);
    prof_commit(ps, KID_LAYER_ROWTILE, ps.on ? flops : 0.0, 0.0);
    return hipGetLastError();
}

// =============================================================================================
// Action-wide products of the layered path (at most 32 output columns): the policy's output layer
// (with the Actor's exploration noise where asked for) and the gradient with respect to the action.  One wavefront's 32 columns already cover the
// output, so the eight wavefronts of a row tile split the contraction instead (every eighth chunk
// of 32 k-values each, as in the chained kernels' narrow layers) and their partial tiles meet in
// LDS.  Segments (the twin critics' first-layer deltas) pass through the same input tile one after
// the other.  B operands are row-major [K][N].
// =============================================================================================
__global__ __launch_bounds__(FT, 2) void narrow_rowtile_kernel(const GemmGroup g) {
    Lanes T;
    T.tid = threadIdx.x; T.lane = T.tid & 63; T.wave = __builtin_amdgcn_readfirstlane(T.tid >> 6); T.l32 = T.lane & 31; T.half = T.lane >> 5;
    const int b = blockIdx.x;
    int pi = 0;
    for (int i = 1; i < g.nprob; ++i)
        if (b >= g.p[i].tile_begin) pi = i;
    const GemmProb& P = g.p[pi];
    const int part = b - P.tile_begin, r0 = part * BMF, M = P.M, N = P.N;
    int kmax = P.seg[0].K;
    if (P.nseg > 1 && P.seg[1].K > kmax) kmax = P.seg[1].K;
    const int S = ((kmax + 7) & ~7) + 4;
    // input tile; the partial tiles and the 32 x 33 output tile take its place once the products are done
    const int XA = 0, scratch = 0, red = SCRATCH_F;
    const int ncol = T.l32 < N ? T.l32 : N - 1;
    floatx16 acc[1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = 0.f;
    for (int sg = 0; sg < P.nseg; ++sg) {
        if (sg > 0) __syncthreads();                                     // the tile is reused
        load_rows(T, XA, S, P.seg[sg].A, P.seg[sg].K, r0, M);
        __syncthreads();
        const int ins[1] = {XA};
        const float* const ws[1] = {P.seg[sg].B};
        mac_segment<1>(acc, ins, S, P.seg[sg].K, ws, P.seg[sg].ldb, ncol, T, T.wave, FW);
    }
    __syncthreads();                                                     // every wavefront is done with the input tile
#pragma unroll
    for (int r = 0; r < 16; ++r) smem[scratch + T.wave * 1024 + r * 64 + T.lane] = acc[0][r];
    __syncthreads();
    const int epi = P.epi;
    for (int e = T.tid; e < 1024; e += FT) {
        int row, col;
        float x = small_sum(scratch, e, row, col);
        const bool ok = col < N && r0 + row < M;
        if (ok) {
            if (epi == EPI_MUL_DTANH) {
                const float t = P.aux[(size_t)(r0 + row) * (size_t)P.ldaux + col];
                x *= 1.f - t * t;
            } else {
                x = tanhf(x + P.bias[col]);
                if (epi == EPI_BIAS_TANH_NOISE) {
                    // Actor step (Section 3.3): a = clip(pi(s) + sigma_i * eps, -1, 1), sigma_i linear in the
                    // environment index, eps from Philox-4x32-10 (stream 2) by Box-Muller, as in fused_act_kernel
                    const GemmNoise& nz = g.noise;
                    const int env = r0 + row;
                    uint32_t w0, w1;
                    philox4x32_10_f((uint32_t)(env * nz.act_dim + col), 2u, nz.ctr2, nz.ctr3, nz.key0, nz.key1, w0, w1);
                    const double u1 = ((double)(w0 >> 8) + 0.5) * 0x1p-24;
                    const double u2 = ((double)(w1 >> 8) + 0.5) * 0x1p-24;
                    const double eps = sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925286766559 * u2);
                    double sigma = (double)nz.sigma_min;
                    if (nz.sigma_rows > 1)
                        sigma += ((double)env / (double)(nz.sigma_rows - 1)) * ((double)nz.sigma_max - (double)nz.sigma_min);
                    x = fminf(fmaxf(x + (float)(sigma * eps), -1.f), 1.f);
                }
            }
            P.C[(size_t)(r0 + row) * (size_t)P.ldc + col] = x;
        } else {
            x = 0.f;
        }
        smem[red + row * 33 + col] = x;
    }
    if (P.colsum != nullptr) {
        __syncthreads();
        if (T.tid < N) {
            float cs = 0.f;
            for (int row = 0; row < BMF; ++row) cs += smem[red + row * 33 + T.tid];
            P.colsum[(size_t)part * (size_t)N + T.tid] = cs;
        }
    }
}

static size_t narrow_lds_bytes(const GemmProb& p) {
    int kmax = p.seg[0].K;
    if (p.nseg > 1 && p.seg[1].K > kmax) kmax = p.seg[1].K;
    const size_t tile = (size_t)BMF * (size_t)(((kmax + 7) & ~7) + 4), tail = (size_t)SCRATCH_F + BMF * 33;
    return sizeof(float) * (tile > tail ? tile : tail);
}

// Whether a launch of X W products (B operand [K][N] row-major) can take the narrow row-tile kernel.
bool narrow_rowtile_ok(const GemmGroup& g) {
    long wgs = 0;
    for (int i = 0; i < g.nprob; ++i) {
        const GemmProb& p = g.p[i];
        if (p.epi != EPI_BIAS_TANH && p.epi != EPI_BIAS_TANH_NOISE && p.epi != EPI_MUL_DTANH) return false;
        if (p.epi == EPI_BIAS_TANH_NOISE && (g.nprob != 1 || g.noise.act_dim != p.N)) return false;
        if (p.epi == EPI_MUL_DTANH ? (p.aux == nullptr || p.ldaux < p.N) : (p.bias == nullptr || p.colsum != nullptr)) return false;
        if (p.N < 1 || p.N > 32 || p.M < 1 || p.nseg < 1 || p.nseg > 2 || p.ldc < p.N) return false;
        for (int s = 0; s < p.nseg; ++s) {
            const GemmSeg& q = p.seg[s];
            if (q.K < 1 || q.lda != q.K || q.ldb < p.N) return false;
            if ((size_t)q.K * (size_t)q.ldb * sizeof(float) >= ((size_t)1 << 31)) return false;
        }
        if (narrow_lds_bytes(p) > 150 * 1024) return false;
        wgs += (p.M + BMF - 1) / BMF;
    }
    return wgs >= 256;
}

hipError_t narrow_rowtile_launch(GemmGroup& g, hipStream_t stream) {
    int total = 0;
    size_t lds = 0;
    double flops = 0.0;
    for (int i = 0; i < g.nprob; ++i) {
        GemmProb& p = g.p[i];
        p.tile_begin = total;
        p.tiles_m = (p.M + BMF - 1) / BMF; p.tiles_n = 1; p.splits = 1; p.k_chunk = 0;
        total += p.tiles_m;
        for (int s = 0; s < p.nseg; ++s) flops += 2.0 * p.M * (double)p.N * p.seg[s].K;
        if (narrow_lds_bytes(p) > lds) lds = narrow_lds_bytes(p);
    }
    g.total_tiles = total;
    if (total == 0) return hipSuccess;
    static LdsLimit configured;
    const hipError_t e = set_lds_limit(reinterpret_cast<const void*>(narrow_rowtile_kernel), lds, configured);
    if (e != hipSuccess) return e;
    const ProfSlot ps = prof_slot();
    PQL_LAUNCH(ps, narrow_rowtile_kernel, dim3(total), dim3(FT), lds, stream, g);
    prof_commit(ps, KID_NARROW_ROWTILE, ps.on ? flops : 0.0, 0.0);
    return hipGetLastError();
}

// =============================================================================================
// Batched 2-D transposes: dst[c][r] = src[r][c] for a list of small matrices.
// =============================================================================================
__global__ __launch_bounds__(256) void transpose_kernel(const TransposeArgs a) {
    __shared__ float tile[32][33];
    int b = blockIdx.x, mi = 0;
    for (int i = 1; i < a.n; ++i)
        if (b >= a.m[i].block_begin) mi = i;
    const TransposeArgs::Mat& M = a.m[mi];
    b -= M.block_begin;
    const int tiles_c = (M.cols + 31) / 32;
    const int tr = b / tiles_c, tc = b - tr * tiles_c;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int j = ty; j < 32; j += 8) {
        const int r = tr * 32 + j, c = tc * 32 + tx;
        tile[j][tx] = (r < M.rows && c < M.cols) ? M.src[(size_t)r * M.cols + c] : 0.f;
    }
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
        const int c = tc * 32 + j, r = tr * 32 + tx;
        if (r < M.rows && c < M.cols) M.dst[(size_t)c * M.rows + r] = tile[tx][j];
    }
}

hipError_t transpose_launch(TransposeArgs& a, hipStream_t stream) {
    int blocks = 0;
    double bytes = 0.0;
    for (int i = 0; i < a.n; ++i) {
        a.m[i].block_begin = blocks;
        blocks += ((a.m[i].rows + 31) / 32) * ((a.m[i].cols + 31) / 32);
        bytes += 8.0 * a.m[i].rows * a.m[i].cols;
    }
    if (blocks == 0) return hipSuccess;
    const ProfSlot ps = prof_slot();
    PQL_LAUNCH(ps, transpose_kernel, dim3(blocks), dim3(256), 0, stream, a);
    prof_commit(ps, KID_TRANSPOSE, 0.0, bytes);
    return hipGetLastError();
}

}  // namespace pql
