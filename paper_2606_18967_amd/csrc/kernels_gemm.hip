// kernels_gemm.hip -- the bf16 projections: C[M][N] (fp32) = or += A[M][K] W^T.
//
// Weights are row-major [N][K] (K contiguous), activations [M][K].
//   - gemm_dma (N a multiple of 128): tiles of 64 to 320 rows, both operands
//     brought into LDS by DMA; see k_gemm_dma.
//   - gemm_stream (N an odd multiple of 64): weights streamed from HBM into
//     registers, v_mfma_f32_16x16x32_bf16; see k_gemm_stream.
//   - gemm_f32 / gemm_q4_f32: plain VALU versions for fp32 models (the int4
//     one reads the packed layout of kernels_q4.hip).
#include "common.h"
#include "kernels.h"

namespace {

// ------------------------------------------------------------------ fp32 VALU
constexpr int FT = 64, FK = 16;

__global__ void __launch_bounds__(256) k_gemm_f32(const float* __restrict__ A, const float* __restrict__ W,
                                                  float* __restrict__ C, int M, int N, int K, int ldc, int mode)
{
    __shared__ float As[FK][FT + 1];
    __shared__ float Ws[FK][FT + 1];
    int tid = threadIdx.x;
    int tm = tid >> 4, tn = tid & 15;   // 16 x 16 threads, 4 x 4 outputs each
    int m0 = blockIdx.y * FT, n0 = blockIdx.x * FT;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += FK) {
        for (int t = tid; t < FT * FK; t += 256) {
            int row = t / FK, kk = t % FK;
            int gm = m0 + row;
            As[kk][row] = gm < M ? A[(size_t)gm * K + k0 + kk] : 0.f;
            Ws[kk][row] = W[(size_t)(n0 + row) * K + k0 + kk];
        }
        lds_barrier();
#pragma unroll
        for (int kk = 0; kk < FK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = As[kk][tm * 4 + i]; b[i] = Ws[kk][tn * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        lds_barrier();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int row = m0 + tm * 4 + i;
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float* cp = C + (size_t)row * ldc + n0 + tn * 4 + j;
            *cp = mode == GEMM_ADD ? *cp + acc[i][j] : acc[i][j];
        }
    }
}

// The same for few rows (decode and verify batches): a wave takes two columns,
// its lanes four consecutive k each (whole 1 KB lines of a weight row), MR rows
// per pass, and sums over its lanes at the end.  The tiled kernel above walks
// K in steps of 16 with a barrier and a memory round trip each, on as many
// work-groups as there are 64-column tiles (47.6 us per launch of the two-layer
// hidden-256 decoder at 4 and 20 rows, against 6.0 at 20 rows and 3.3 at 4 here).
template <int MR>
__global__ void __launch_bounds__(256) k_gemm_f32_rows(const float* __restrict__ A, const float* __restrict__ W,
                                                       float* __restrict__ C, int M, int N, int K, int ldc, int mode)
{
    const int lane = threadIdx.x & 63, n0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 2, m0 = blockIdx.y * MR;
    float acc[MR][2];
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[m][0] = acc[m][1] = 0.f;
    auto dot = [](float v, float4 a, float4 b) { return v + a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; };
    for (int k = 4 * lane; k < K; k += 256) {
        const float4 w0 = *(const float4*)(W + (size_t)n0 * K + k), w1 = *(const float4*)(W + (size_t)(n0 + 1) * K + k);
        float4 a[MR];
#pragma unroll
        for (int m = 0; m < MR; ++m) a[m] = *(const float4*)(A + (size_t)min(m0 + m, M - 1) * K + k);
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            acc[m][0] = dot(acc[m][0], a[m], w0);
            acc[m][1] = dot(acc[m][1], a[m], w1);
        }
    }
    float mine = 0.f;                                       // lane 2 m + j keeps output (m, j)
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float v = wave_sum(acc[m][j]);
            if (lane == 2 * m + j) mine = v;
        }
    const int row = m0 + (lane >> 1);
    if (lane < 2 * MR && row < M) {
        float* cp = C + (size_t)row * ldc + n0 + (lane & 1);
        *cp = mode == GEMM_ADD ? *cp + mine : mine;
    }
}

__device__ __forceinline__ float f16_bits_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

// ------------------------------------------------------------------ weight-streaming bf16 MFMA GEMM
// C[M][N] = A[M][K] W^T where N is an odd multiple of 64 (an LM head of such a
// vocabulary).  A work-group covers a 64-row m-tile, 64 columns (16 per wave, 4
// waves) and a range of K split into chunks of 128.  The A chunk is staged in LDS
// (double-buffered) and shared by the four waves; each wave streams its weight
// columns from HBM straight into registers through a ring of RD register sets (RD - 1
// chunks in flight), so every weight byte is read once per m-tile.  Lane l
// covers k = 128g + 32j + 8(l/16) + 0..7 of chunk g in k-step j
// (v_mfma_f32_16x16x32_bf16): each load instruction reads 64 contiguous
// bytes of 16 weight rows; A is read from LDS in the same k order.  With several K splits
// the partial sums go to P[s][M][N] for the consumer (or k_splitk_reduce).
// Work items are laid out so that consecutive ones (the m-tiles of one
// column tile) land on the same XCD and share its L2.
constexpr int SK = 128;          // k per chunk
constexpr int ALD = SK + 8;      // LDS row stride in 2-byte elements
constexpr int SM = 64;           // rows per m-tile

template <int MT>
__global__ void __launch_bounds__(256) k_gemm_stream(const uint16_t* __restrict__ A, const uint16_t* __restrict__ Wt,
                                                     float* __restrict__ C, float* __restrict__ P, int M, int N, int K,
                                                     int ldc, int mode, int S, int msup, int total)
{
    constexpr int RD = 3;                                   // register sets in the load ring
    __shared__ __attribute__((aligned(16))) uint16_t As[2][SM * ALD];
    const int per_xcd = gridDim.x >> 3;                     // gridDim.x is a multiple of 8
    const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (w >= total) return;
    const int ms = w % msup, rest = w / msup;
    const int s = rest % S, tile = rest / S;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m0 = ms * SM;
    const int G = K / SK, Gs = G / S, g0 = s * Gs, g1 = g0 + Gs;
    const int nb = tile * 4 + wv;                           // this wave's 16-column block
    const int rows = min(M - m0, MT * 16);                  // rows staged (others stay zero)
    // each work item walks its chunks from a different starting offset: in
    // lockstep they would all read the same 256-byte column of the weight
    // rows at once and crowd a few HBM channels
    const int rot = (tile * 5 + s) % Gs;
    auto phys = [&](int g) { const int i = g - g0 + rot; return g0 + (i >= Gs ? i - Gs : i); };

    // A tiles travel through a ring of register sets too (same depth as the
    // weights): the tile of chunk c + 1 is requested RD - 2 chunks before it
    // is stored to LDS
    constexpr int AP = 4;                                 // 16-byte A pieces per thread per chunk
    u32x4 ar[RD][AP];
    auto load_a = [&](int g, u32x4 (&a)[AP]) {
#pragma unroll
        for (int t = 0; t < AP; ++t) {
            const int pidx = tid + t * 256;
            const int row = pidx >> 4, col = (pidx & 15) * 8;
            a[t] = *(const u32x4*)(A + (size_t)(m0 + min(row, rows - 1)) * K + (size_t)phys(g) * SK + col);
        }
    };
    // a tile of a chunk past the split (valid false) is stored as zeros, so
    // the padded iterations of the main loop add nothing
    auto store_a = [&](int buf, const u32x4 (&a)[AP], bool valid) {
#pragma unroll
        for (int t = 0; t < AP; ++t) {
            const int pidx = tid + t * 256;
            const int row = pidx >> 4, col = (pidx & 15) * 8;
            if (row < MT * 16)
                *(u32x4*)(&As[buf][row * ALD + col]) = (valid && row < rows) ? a[t] : (u32x4){0u, 0u, 0u, 0u};
        }
    };
    u32x4 wr[RD][4];
    auto load_w = [&](int g, u32x4 (&wq)[4]) {
        const uint16_t* wp = Wt + (size_t)(nb * 16 + (lane & 15)) * K + (size_t)phys(g) * SK + 8 * (lane >> 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) wq[j] = *(const u32x4*)(wp + 32 * j);   // j, j + 1 share a 128-byte line: cached
    };

    floatx4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = (floatx4){0.f, 0.f, 0.f, 0.f};

    auto compute = [&](int buf, const u32x4 (&wq)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint16_t* ab = &As[buf][(lane & 15) * ALD + 32 * j + 8 * (lane >> 4)];
            const bf16x8 bb = __builtin_bit_cast(bf16x8, wq[j]);
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, *(const u32x4*)(ab + t * 16 * ALD)), bb, acc[t], 0, 0, 0);
        }
    };

    // prologue: A and weights of the first RD - 1 chunks in flight, A of chunk g0 in LDS
    // (chunk indices past the split are clamped: those loads are redundant but
    // unconditional, which keeps the compiler's wait counts exact)
#pragma unroll
    for (int u = 0; u < RD - 1; ++u) {
        load_a(min(g0 + u, g1 - 1), ar[u]);
        load_w(min(g0 + u, g1 - 1), wr[u]);
    }
    store_a(0, ar[0], true);
    lds_barrier();

    // chunk c uses ring slot u = (c - g0) % RD and LDS buffer (c - g0) & 1; it
    // requests chunk c + RD - 1 (A before weights, so waiting for an A tile
    // leaves the newer loads in flight) and stores the A tile of c + 1.  The
    // chunk count is rounded up to a multiple of RD so the unrolled body has
    // no branches: a conditional chunk would make the compiler's wait counts
    // conservative at the merge and drain the whole ring every chunk.
    const int gend = g0 + (Gs + RD - 1) / RD * RD;
    for (int gb = g0; gb < gend; gb += RD) {
#pragma unroll
        for (int u = 0; u < RD; ++u) {
            const int c = gb + u;
            const int buf = (gb - g0 + u) & 1;
            const int nx = (u + RD - 1) % RD;
            load_a(min(c + RD - 1, g1 - 1), ar[nx]);
            load_w(min(c + RD - 1, g1 - 1), wr[nx]);
            compute(buf, wr[u]);
            store_a(buf ^ 1, ar[(u + 1) % RD], c + 1 < g1);
            lds_barrier();
        }
    }

    // ---- epilogue
    const int col = nb * 16 + (lane & 15);
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = m0 + t * 16 + (lane >> 4) * 4 + r;
            if (row >= M) continue;
            if (S == 1) {
                float* cp = C + (size_t)row * ldc + col;
                *cp = mode == GEMM_ADD ? *cp + acc[t][r] : acc[t][r];
            } else {
                P[((size_t)s * M + row) * N + col] = acc[t][r];
            }
        }
}

// ------------------------------------------------------------------ tiled bf16 MFMA GEMM, register-staged
// C[M][N] = A[M][K] W^T with both operands staged through registers into LDS:
// the reference form of the 320-row DMA-fed tiles below (debug switch).  Block
// tile (32*MTW) x 128, four waves in a 2 x 2 grid, each wave (16*MTW) x 64 =
// MTW/2 x 2 blocks of v_mfma_f32_32x32x16_bf16; lane l reads row or column
// l % 32 and k 8 (l / 32) + 0..7 of each 16-k step.  K advances in stages of
// 64 with double-buffered LDS and the global loads of stage k + 2 in flight
// while stage k is multiplied.  LDS rows are padded to 72 elements (bank-
// conflict free 16-byte fragment reads).  Split-K partials as in k_gemm_stream.
constexpr int TBK = 64, TLD = TBK + 8, TBN = 128;

// SW: the SwiGLU epilogue.  W is [2F][K], gate rows then up rows; column tile
// t loads gate rows 64t..64t+63 (waves wn = 0) and up rows F + 64t.. (wn = 1),
// runs without split-K and writes out[m][f] = SiLU(g) u (type out_t).
template <int MTW, bool SW>
__global__ void __launch_bounds__(256) k_gemm_t32(const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
                                                    float* __restrict__ C, float* __restrict__ P, int M, int N, int K,
                                                    int ldc, int mode, int S, int mtiles, int total,
                                                    void* __restrict__ out, int out_t)
{
    constexpr int BM = 32 * MTW;
    constexpr int AP = MTW;      // 16-byte A pieces per thread per stage (BM*8/256)
    constexpr int WP = 4;        // 16-byte W pieces per thread per stage (128*8/256)
    __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * TLD];
    __shared__ __attribute__((aligned(16))) uint16_t Ws[2][TBN * TLD];
    const int per_xcd = gridDim.x >> 3;
    const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (w >= total) return;
    const int mt = w % mtiles, rest = w / mtiles;
    const int s = rest % S, nt = rest / S;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wm = wv >> 1, wn = wv & 1;
    const int m0 = mt * BM, n0 = nt * TBN;
    const int KS = K / TBK, Ks = KS / S, k0 = s * Ks, k1 = k0 + Ks;
    const int rows = min(M - m0, BM);

    u32x4 ra[2][AP], rw[2][WP];
    auto load = [&](int kb, u32x4 (&a)[AP], u32x4 (&b)[WP]) {
#pragma unroll
        for (int t = 0; t < AP; ++t) {
            const int pidx = tid + t * 256, row = pidx >> 3, col = (pidx & 7) * 8;
            a[t] = *(const u32x4*)(A + (size_t)(m0 + min(row, rows - 1)) * K + (size_t)kb * TBK + col);
        }
#pragma unroll
        for (int t = 0; t < WP; ++t) {
            const int pidx = tid + t * 256, row = pidx >> 3, col = (pidx & 7) * 8;
            const int wrow = SW ? (row < 64 ? nt * 64 + row : N / 2 + nt * 64 + row - 64) : n0 + row;
            b[t] = *(const u32x4*)(W + (size_t)wrow * K + (size_t)kb * TBK + col);
        }
    };
    auto store = [&](int buf, const u32x4 (&a)[AP], const u32x4 (&b)[WP]) {
#pragma unroll
        for (int t = 0; t < AP; ++t) {
            const int pidx = tid + t * 256, row = pidx >> 3, col = (pidx & 7) * 8;
            *(u32x4*)(&As[buf][row * TLD + col]) = row < rows ? a[t] : (u32x4){0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int t = 0; t < WP; ++t) {
            const int pidx = tid + t * 256, row = pidx >> 3, col = (pidx & 7) * 8;
            *(u32x4*)(&Ws[buf][row * TLD + col]) = b[t];
        }
    };

    floatx16 acc[MTW / 2][2];
#pragma unroll
    for (int i = 0; i < MTW / 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    load(k0, ra[0], rw[0]);
    if (k0 + 1 < k1) load(k0 + 1, ra[1], rw[1]);
    store(0, ra[0], rw[0]);
    lds_barrier();
    for (int kb = k0; kb < k1; kb += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = kb + u;
            if (k < k1) {
                const int buf = (k - k0) & 1;
                if (k + 2 < k1) load(k + 2, ra[u], rw[u]);      // slot u is free: stage k is in LDS
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int kk = ks * 16 + (lane >> 5) * 8;
                    u32x4 af[MTW / 2], bw[2];
#pragma unroll
                    for (int i = 0; i < MTW / 2; ++i)
                        af[i] = *(const u32x4*)(&As[buf][(wm * 16 * MTW + 32 * i + (lane & 31)) * TLD + kk]);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        bw[j] = *(const u32x4*)(&Ws[buf][(wn * 64 + 32 * j + (lane & 31)) * TLD + kk]);
#pragma unroll
                    for (int i = 0; i < MTW / 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i]),
                                                                               __builtin_bit_cast(bf16x8, bw[j]),
                                                                               acc[i][j], 0, 0, 0);
                }
                if (k + 1 < k1) store(buf ^ 1, ra[u ^ 1], rw[u ^ 1]);
                lds_barrier();
            }
        }
    }
    if constexpr (SW) {
        // the up half hands its products to the gate half of the same features
        static_assert(2 * (MTW / 2) * 2 * 16 * 64 * 4 <= sizeof(As), "SwiGLU exchange does not fit the A buffers");
        float* ys = (float*)&As[0][0];                 // [wm][i][j][r][64 lanes]
        auto yi = [&](int i, int j, int r) { return (((wm * (MTW / 2) + i) * 2 + j) * 16 + r) * 64 + lane; };
        if (wn == 1) {
#pragma unroll
            for (int i = 0; i < MTW / 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) ys[yi(i, j, r)] = acc[i][j][r];
        }
        lds_barrier();
        if (wn == 1) return;
        const int F = N / 2;
#pragma unroll
        for (int i = 0; i < MTW / 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int feat = nt * 64 + 32 * j + (lane & 31);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = m0 + wm * 16 * MTW + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    if (row >= M) continue;
                    const float v = swiglu(acc[i][j][r], ys[yi(i, j, r)]);
                    const size_t oi = (size_t)row * F + feat;
                    if (out_t == ACT_F16) store_act<_Float16>(out, oi, v);
                    else if (out_t == ACT_BF16) store_act<uint16_t>(out, oi, v);
                    else store_act<float>(out, oi, v);
                }
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < MTW / 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn * 64 + 32 * j + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + wm * 16 * MTW + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row >= M) continue;
                if (S == 1) {
                    float* cp = C + (size_t)row * ldc + col;
                    *cp = mode == GEMM_ADD ? *cp + acc[i][j][r] : acc[i][j][r];
                } else {
                    P[((size_t)s * M + row) * N + col] = acc[i][j][r];
                }
            }
        }
}

// ------------------------------------------------------------------ tiles fed by LDS DMA
// C[M][N] = A[M][K] W^T, tile (32 MT) x (64 WCN), WM x WCN waves, each wave
// (32 MT / WM) x 64 as MT / WM x 2 blocks of v_mfma_f32_32x32x16_bf16 (k in
// ascending 16-k steps).  Both operands come into LDS by
// global_load_lds_dwordx4: an instruction puts 64 lanes x 16 bytes straight
// into 1 KB of LDS, whole 128-byte lines of eight rows, so no registers stage
// the tiles and the waves issue no LDS stores.  K advances in stages of 64
// through a ring of NST buffers: NST - 1 stages are in flight, the next one
// requested right after the barrier that opens a stage.  The 16-byte chunk c
// of row r sits at position c ^ sw(r), sw(r) = (r ^ r / 8) % 8, which keeps the
// fragment reads (rows r..r+7 or r..r+15 at one chunk) free of bank conflicts;
// a DMA lane therefore fetches chunk pos ^ sw(r) of its row.  Rows past M
// repeat row M - 1 (never stored).
// SW: the SwiGLU epilogue; the tile takes 32 WCN features, and wave column
// wn's two 32-column blocks are the gate rows and the up rows of the same 32
// features, so SiLU(g) u is formed in registers (no split-K there).  With S
// K splits the partial sums go to P[s][M][N] as in k_gemm_stream.
// The weights' loads are non-temporal, also where several m-tiles read them (8B
// gate/up at 1280 rows 278 us against 286, LM head at 640 626 against 644).
// What bounds it: the weights' stream up to about 200 rows, so the ring is as
// deep as LDS allows (three stages of 160 x 256 are 156 KB); the matrix cores
// and the wait for the next stage at 320 rows (two stages).
constexpr int DBK = 64, DRB = DBK * 2;                  // k per stage, bytes per tile row

__device__ __forceinline__ void lds_dma16(const void* src, uint32_t lds_byte)
{
    asm volatile("global_load_lds_dwordx4 %0, off" : : "v"(src), "{m0}"(lds_byte) : "memory");
}

// the same for data read once (weights): non-temporal
__device__ __forceinline__ void lds_dma16_nt(const void* src, uint32_t lds_byte)
{
    asm volatile("global_load_lds_dwordx4 %0, off nt" : : "v"(src), "{m0}"(lds_byte) : "memory");
}

// s_waitcnt vmcnt(N) with the other counters left free (gfx9 field layout)
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt field is 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// ROT: the stage a tile starts its K range with (it goes round).  The gate and
// the up columns of a feature start alike, in the plain form and in the SwiGLU
// form (whose tile takes half as many features), so that both sum in one order.
__device__ __forceinline__ int dma_rot(int nt, int s, int tiles, int Ks, bool sw)
{
    const int t = sw ? nt >> 1 : (tiles % 2 == 0 && nt >= tiles / 2 ? nt - tiles / 2 : nt);
    return tiles % 2 ? 0 : (t * 5 + s) % Ks;
}

// Where tiles rotate: rows are K elements apart, so with a K of a multiple of
// 4096 all rows of all tiles lie at one k in the same few memory channels, and
// tiles that walk K in step crowd them (8B gate/up at 2, 64 and 65 rows: 42, 46
// and 52 us, rotated 38, 41 and 45).  With other K the first round of tiles does
// better in step (32B gate/up at 2, 64 and 128 rows: 87, 93 and 108 us, rotated
// 93, 100 and 114); launches of several rounds gain between 65 and 160 rows (32B
// LM head at 96 and 128: 317 and 332 us, rotated 304 and 326; at 64 and 256
// within 1%).  From 161 rows on it makes no difference.
static bool dma_rotates(int mt, long long tiles, int K)
{
    return mt <= 5 && (K % 4096 == 0 || (mt >= 3 && tiles > 256));
}

__device__ __forceinline__ int dma_sw(int r) { return (r ^ (r >> 3)) & 7; }

template <int MT, int WM, int WCN, int NST, bool SW, bool ROT>
__global__ void __launch_bounds__(64 * WM * WCN) k_gemm_dma(const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
                                                            float* __restrict__ C, float* __restrict__ P, int M, int N,
                                                            int K, int ldc, int mode, int S, int mtiles, int total,
                                                            void* __restrict__ out, int out_t,
                                                            const int32_t* __restrict__ live)
{
    constexpr int BM = 32 * MT, BN = 64 * WCN, NWAVE = WM * WCN, RT = MT / WM;   // RT row blocks per wave
    constexpr int NA = BM / 8, NI = NA + BN / 8;               // 1 KB pieces (8 rows) per stage
    constexpr int STG = (BM + BN) * DRB;
    constexpr int CNT = NI / NWAVE;                            // pieces per wave per stage
    static_assert(MT % WM == 0 && NI % NWAVE == 0, "every wave has the same rows and pieces");
    static_assert(NST >= 2 && NST <= 5 && NST * STG <= 160 * 1024 && CNT * (NST - 2) < 64, "LDS, vmcnt");
    constexpr int FT = 32 * WCN;                               // features per tile of the SwiGLU form
    __shared__ __attribute__((aligned(1024))) uint8_t sm[NST * STG];
    const uint32_t sbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)sm;
    const int per_xcd = gridDim.x >> 3;                        // gridDim.x is a multiple of 8
    const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (w >= total) return;
    const int mt = w % mtiles, rest = w / mtiles;
    const int s = rest % S, nt = rest / S;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv / WCN, wn = wv % WCN;
    const int m0 = mt * BM, n0 = nt * BN;
    if (live && m0 >= *live) return;                           // a row tile without a live row
    const int Ks = K / DBK / S, k0 = s * Ks;
    const int rows = min(M - m0, BM);

    // this lane's source row and chunk for each of its pieces
    const uint16_t* src[CNT];
    uint32_t dst[CNT];
#pragma unroll
    for (int q = 0; q < CNT; ++q) {
        const int t = wv + q * NWAVE, rl = lane >> 3, pos = lane & 7;
        if (t < NA) {
            const int row = 8 * t + rl;
            src[q] = A + (size_t)(m0 + min(row, rows - 1)) * K + (size_t)k0 * DBK + 8 * (pos ^ dma_sw(row));
            dst[q] = t * 1024;
        } else {
            const int row = 8 * (t - NA) + rl;
            int wrow = n0 + row;
            if constexpr (SW) {
                const int f = nt * FT + (row >> 6) * 32 + (row & 31);   // wave column row/64, block (row/32)%2
                wrow = ((row >> 5) & 1) ? N / 2 + f : f;
            }
            src[q] = W + (size_t)wrow * K + (size_t)k0 * DBK + 8 * (pos ^ dma_sw(row));
            dst[q] = BM * DRB + (t - NA) * 1024;
        }
    }
    const int rot = ROT ? dma_rot(nt, s, N / BN, Ks, SW) : 0;
    auto issue = [&](int kb) {
        const uint32_t buf = sbase + (kb % NST) * STG;
        const size_t at = (size_t)(ROT && kb + rot >= Ks ? kb + rot - Ks : kb + rot) * DBK;
#pragma unroll
        for (int q = 0; q < CNT; ++q) {
            if (wv + q * NWAVE < NA) lds_dma16(src[q] + at, buf + dst[q]);
            else lds_dma16_nt(src[q] + at, buf + dst[q]);
        }
    };

    floatx16 acc[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
    for (int u = 0; u < NST - 1; ++u)
        if (u < Ks) issue(u);
    for (int kb = 0; kb < Ks; ++kb) {
        // this wave's pieces of stage kb are in once those of the later stages are all that is outstanding
        const int later = min(NST - 2, Ks - 1 - kb);
        if (NST >= 5 && later == 3) wait_vmcnt<3 * CNT>();
        else if (NST >= 4 && later == 2) wait_vmcnt<2 * CNT>();
        else if (NST >= 3 && later == 1) wait_vmcnt<CNT>();
        else wait_vmcnt<0>();
        lds_barrier();                      // everyone's are, and stage kb - 1 is no longer read
        if (kb + NST - 1 < Ks) issue(kb + NST - 1);
        const uint8_t* sa = sm + (kb % NST) * STG;
        const uint8_t* sw = sa + BM * DRB;
#pragma unroll
        for (int ks = 0; ks < DBK / 16; ++ks) {
            const int c = 2 * ks + (lane >> 5);
            u32x4 af[RT], bw[2];
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int r = (wm * RT + i) * 32 + (lane & 31);
                af[i] = *(const u32x4*)(sa + r * DRB + ((c ^ dma_sw(r)) << 4));
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = wn * 64 + 32 * j + (lane & 31);
                bw[j] = *(const u32x4*)(sw + r * DRB + ((c ^ dma_sw(r)) << 4));
            }
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i]),
                                                                       __builtin_bit_cast(bf16x8, bw[j]), acc[i][j],
                                                                       0, 0, 0);
        }
    }
    if constexpr (SW) {
        const int F = N / 2, feat = nt * FT + wn * 32 + (lane & 31);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + (wm * RT + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row >= M) continue;
                const float v = swiglu(acc[i][0][r], acc[i][1][r]);
                const size_t oi = (size_t)row * F + feat;
                if (out_t == ACT_F16) store_act<_Float16>(out, oi, v);
                else if (out_t == ACT_BF16) store_act<uint16_t>(out, oi, v);
                else store_act<float>(out, oi, v);
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn * 64 + 32 * j + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + (wm * RT + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row >= M) continue;
                if (S == 1) {
                    float* cp = C + (size_t)row * ldc + col;
                    *cp = mode == GEMM_ADD ? *cp + acc[i][j][r] : acc[i][j][r];
                } else {
                    P[((size_t)s * M + row) * N + col] = acc[i][j][r];
                }
            }
        }
}

// C[m][n] (+)= sum_s P[s][m][n]
__global__ void __launch_bounds__(256) k_splitk_reduce(const float* __restrict__ P, float* __restrict__ C, int M, int N,
                                                       int ldc, int S, int mode)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t MN = (size_t)M * N;
    if (idx >= MN) return;
    const float v = add_splits(0.f, P, S, MN, idx);
    int row = (int)(idx / N), col = (int)(idx % N);
    float* cp = C + (size_t)row * ldc + col;
    *cp = mode == GEMM_ADD ? *cp + v : v;
}

// ------------------------------------------------------------------ int4 x fp32 VALU
// Work-group (32-column block, MR rows), lane l as in the packed layout of
// kernels_q4.hip: column l % 32, k-half l / 32.  The four waves take the groups
// of 128 k in turn; a wave stages its group's MR x 128 activations in LDS,
// reads its codes with 16-byte loads and multiplies k-step by k-step; the
// halves and the waves are summed at the end.  (One thread per output, decoding
// each code from its own load, took 59.2 us per launch of the two-layer
// hidden-256 decoder at 4 rows, against 5.4 us.)
template <int MR, int FMT>
__global__ void __launch_bounds__(256) k_gemm_q4_f32(const float* __restrict__ A, const uint32_t* __restrict__ Wq,
                                                     const uint16_t* __restrict__ Sc, const uint8_t* __restrict__ Z,
                                                     float* __restrict__ C, int M, int N, int K, int ldc, int mode)
{
    constexpr int NL = FMT == QF_W8 ? 4 : 2;                // 16-byte code pieces per lane and group
    __shared__ __attribute__((aligned(16))) float sa[4][MR][128];
    __shared__ float sum[4][MR][32];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nb = blockIdx.x, m0 = blockIdx.y * MR;
    const int G = K / 128, h = lane >> 5;
    float acc[MR];
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[m] = 0.f;
    for (int g = wv; g < G; g += 4) {
        u32x4 w[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) w[i] = *((const u32x4*)Wq + ((size_t)nb * G + g) * (64 * NL) + 64 * i + lane);
        const size_t si = ((size_t)nb * G + g) * 32 + (lane & 31);
        const float sc = f16_bits_to_f32(Sc[si]);
        const float z = FMT == QF_W8 ? 128.f : (FMT == QF_W4A ? (float)Z[si] : 8.f);
        float4 a4[MR / 2];
#pragma unroll
        for (int i = 0; i < MR / 2; ++i) {
            const int m = 2 * i + h;
            a4[i] = *(const float4*)(A + (size_t)min(m0 + m, M - 1) * K + (size_t)g * 128 + 4 * (lane & 31));
        }
#pragma unroll
        for (int i = 0; i < MR / 2; ++i) *(float4*)&sa[wv][2 * i + h][4 * (lane & 31)] = a4[i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        float part[MR];
#pragma unroll
        for (int m = 0; m < MR; ++m) part[m] = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            float q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (FMT == QF_W8) {
                    const int j = 2 * st + (e >> 2);
                    q[e] = (float)((w[j >> 2][j & 3] >> (8 * (e & 3))) & 255u) - z;
                } else {
                    q[e] = (float)((w[st >> 2][st & 3] >> (4 * (e >> 1) + 16 * (e & 1))) & 15u) - z;
                }
            }
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                const float* ar = &sa[wv][m][16 * st + 8 * h];
                const float4 a = *(const float4*)ar, c = *(const float4*)(ar + 4);
                part[m] += a.x * q[0] + a.y * q[1] + a.z * q[2] + a.w * q[3] + c.x * q[4] + c.y * q[5] + c.z * q[6] + c.w * q[7];
            }
        }
#pragma unroll
        for (int m = 0; m < MR; ++m) acc[m] += sc * part[m];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();                    // the group's activations are read before the next replace them
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        const float v = acc[m] + __shfl_xor(acc[m], 32, WAVE);
        if (lane < 32) sum[wv][m][lane] = v;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < MR * 32; t += 256) {
        const int m = t >> 5, c = t & 31;
        if (m0 + m >= M) continue;
        const float v = sum[0][m][c] + sum[1][m][c] + sum[2][m][c] + sum[3][m][c];
        float* cp = C + (size_t)(m0 + m) * ldc + nb * 32 + c;
        *cp = mode == GEMM_ADD ? *cp + v : v;
    }
}

}  // namespace

// K splits of the weight-streaming kernel: doubled until the launch has
// GEMM_SPLIT_TARGET work-groups, with at most GEMM_MAX_SPLIT splits and at least
// two chunks per split.
#ifndef GEMM_SPLIT_TARGET
#define GEMM_SPLIT_TARGET 256
#endif
#ifndef GEMM_MAX_SPLIT
#define GEMM_MAX_SPLIT 8
#endif

static int stream_splits(int M, int N, int K)
{
    const int tiles = N / 64, msup = (M + SM - 1) / SM, G = K / SK;
    int s = 1;
    while (tiles * s * msup < GEMM_SPLIT_TARGET && G % (2 * s) == 0 && G / (2 * s) >= 2 && 2 * s <= GEMM_MAX_SPLIT)
        s *= 2;
    return s;
}

// The DMA-fed tiles' plan: tile height 32 mt, width 64 wcn, S splits of the
// K / 64 stages.
struct dma_tile { int mt, wcn, S; };

// N a multiple of 128, K of 64 (at least two stages)
static bool use_dma(int N, int K) { return N % 128 == 0 && K % DBK == 0 && K >= 2 * DBK; }

#ifndef DMA_MAX_SPLIT
#define DMA_MAX_SPLIT 32
#endif

// Height: the lowest of 64, 96, 128, 160, 192, 256 and 320 rows that holds M;
// more rows take 320-row tiles (fewer passes over the weights at a higher rate
// per pass: 8B gate/up at 640 rows 154 us, in 256-row tiles 236).  Width and
// split: the least of rounds of 256 work-groups x (stages + a ring's to start) x
// a stage's time, plus, with splits, 8 us and the partial sums' write and read at
// 5 TB/s (an unsplit gate/up forms SwiGLU in its epilogue).
// A stage of 128 columns takes about .42 + .125 mt us with all CUs at work
// (measured .67, .9, 1.4 and 1.7 at mt 2, 4, 8 and 10), one of 256 columns
// 1.65 times that, 1.45 at 320 rows: half as many activation bytes per weight,
// but half as many work-groups, so wide tiles go to large N (LM head at M = 128:
// 195 against 283 us) and to the projections past 320 rows (32B QKV with the
// read of its partials at M = 400 and 640: 69 and 77 us, narrow with half the
// splits 76 and 81), narrow ones elsewhere (8B gate/up at M = 128: 58 against
// 71; down projections with half the splits).  Heights of 96 and 160 rows are
// built at 256 columns only (LM head at M = 148: 214 us, in a 192-row tile 241).
// The times are estimates: past one round they are up to a third too long, for
// every choice alike.
static dma_tile dma_plan(int M, int N, int K)
{
    const int KB = K / DBK;
    dma_tile best = {0, 0, 1};
    double least = 0;
    for (int wcn = 4; wcn >= 2; wcn -= 2) {
        if (N % (64 * wcn)) continue;
        int mt = M <= 64 ? 2 : M > 256 ? 10 : M > 192 ? 8 : M > 160 ? 6 : (M + 31) / 32;
        if (wcn == 2 && mt % 2) ++mt;
        const long long tiles = (long long)(N / (64 * wcn)) * ((M + 32 * mt - 1) / (32 * mt));
        const double stage = (.42 + .125 * mt) * (wcn == 2 ? 1. : mt == 10 ? 1.45 : 1.65);
        const int start = mt == 10 ? 2 : 3;
        for (int S = 1; S <= DMA_MAX_SPLIT && 2 * S <= KB; ++S) {
            if (KB % S) continue;
            const double wgs = (double)tiles * S, rounds = wgs <= 256 ? 1. : wgs / 256 + .35;
            const double t = rounds * (KB / S + start) * stage + (S > 1 ? 8 + 8e-6 / 5 * S * M * N : 0.);
            if (!best.mt || t < least) best = {mt, wcn, S}, least = t;
        }
    }
    return best;
}

size_t gemm_part_floats(int M, int N, int K)
{
    const int S = use_dma(N, K) ? dma_plan(M, N, K).S : stream_splits(M, N, K);
    return S > 1 ? (size_t)S * M * N : 0;
}

// args of k_gemm_dma, launched as the plan's instance
struct dma_args {
    const uint16_t *A, *W;
    float *C, *P;
    int M, N, K, ldc, mode;
    void* out;
    int out_t;
    const int32_t* live;
};

template <int MT, int WM, int WCN, int NST, bool SW>
static void dma_go(const dma_args& a, int S, hipStream_t s)
{
    const int mtiles = (a.M + 32 * MT - 1) / (32 * MT);
    const int total = a.N / (64 * WCN) * mtiles * S;
    auto go = [&](auto kern) {
        kern<<<dim3((total + 7) / 8 * 8), 64 * WM * WCN, 0, s>>>(a.A, a.W, a.C, a.P, a.M, a.N, a.K, a.ldc, a.mode, S, mtiles,
                                                               total, a.out, a.out_t, a.live);
    };
    if constexpr (MT <= 5)
        if (dma_rotates(MT, (long long)(a.N / (64 * WCN)) * mtiles, a.K)) return go(k_gemm_dma<MT, WM, WCN, NST, SW, true>);
    go(k_gemm_dma<MT, WM, WCN, NST, SW, false>);
}

template <bool SW>
static void dma_launch(const dma_args& a, dma_tile p, hipStream_t s)
{
    if (p.wcn == 4) {
        switch (p.mt) {
            case 2: dma_go<2, 2, 4, 3, SW>(a, p.S, s); break;
            case 3: dma_go<3, 1, 4, 3, SW>(a, p.S, s); break;
            case 4: dma_go<4, 2, 4, 3, SW>(a, p.S, s); break;
            case 5: dma_go<5, 1, 4, 3, SW>(a, p.S, s); break;
            case 6: dma_go<6, 2, 4, 2, SW>(a, p.S, s); break;
            case 8: dma_go<8, 2, 4, 2, SW>(a, p.S, s); break;
            default: dma_go<10, 2, 4, 2, SW>(a, p.S, s); break;
        }
    } else {
        switch (p.mt) {
            case 2: dma_go<2, 2, 2, 5, SW>(a, p.S, s); break;
            case 4: dma_go<4, 2, 2, 5, SW>(a, p.S, s); break;
            case 6: dma_go<6, 2, 2, 3, SW>(a, p.S, s); break;
            case 8: dma_go<8, 2, 2, 3, SW>(a, p.S, s); break;
            default: dma_go<10, 2, 2, 2, SW>(a, p.S, s); break;
        }
    }
}

static void reduce_splits(const float* part, float* C, int M, int N, int ldc, int S, int mode, hipStream_t s)
{
    const size_t MN = (size_t)M * N;
    k_splitk_reduce<<<(unsigned)((MN + 255) / 256), 256, 0, s>>>(part, C, M, N, ldc, S, mode);
}

int launch_gemm_bf16(const uint16_t* A, const uint16_t* W, float* C, float* part, size_t part_cap, int M, int N, int K,
                     int ldc, gemm_mode mode, bool defer_reduce, hipStream_t s, bool lds_dma, const int32_t* live)
{
    if (use_dma(N, K)) {
        dma_tile p = dma_plan(M, N, K);
        if (p.S > 1 && (size_t)p.S * M * N > part_cap) p.S = 1;   // workspace too small: no split
        if (lds_dma || p.mt != 10) {
            dma_launch<false>({A, W, C, part, M, N, K, ldc, mode, nullptr, 0, live}, p, s);
        } else {
            const int mtiles = (M + 319) / 320, total = N / TBN * mtiles * p.S;
            k_gemm_t32<10, false><<<dim3((total + 7) / 8 * 8), 256, 0, s>>>(A, W, C, part, M, N, K, ldc, mode, p.S, mtiles,
                                                                            total, nullptr, 0);
        }
        if (p.S > 1 && !defer_reduce) reduce_splits(part, C, M, N, ldc, p.S, mode, s);
        return p.S;
    }
    int S = stream_splits(M, N, K);
    if (S > 1 && (size_t)S * M * N > part_cap) S = 1;   // workspace too small: no split
    const int msup = (M + SM - 1) / SM, total = N / 64 * S * msup;
    auto go = [&](auto kern) {
        kern<<<dim3((total + 7) / 8 * 8), 256, 0, s>>>(A, W, C, part, M, N, K, ldc, mode, S, msup, total);
    };
    switch (msup > 1 ? 4 : (M + 15) / 16) {
        case 1: go(k_gemm_stream<1>); break;
        case 2: go(k_gemm_stream<2>); break;
        case 3: go(k_gemm_stream<3>); break;
        default: go(k_gemm_stream<4>); break;
    }
    if (S > 1 && !defer_reduce) reduce_splits(part, C, M, N, ldc, S, mode, s);
    return S;
}

int launch_gemm_bf16_swiglu(const uint16_t* A, const uint16_t* W, void* out, act_t out_t, int M, int F, int K,
                            size_t part_cap, hipStream_t s, bool lds_dma, const int32_t* live)
{
    const int N = 2 * F;
    if (!use_dma(N, K) || F % 64) return 0;
    // fused only where the plain projection runs unsplit (the same products
    // summed in the same order either way)
    dma_tile p = dma_plan(M, N, K);
    if ((p.S > 1 && (size_t)p.S * M * N <= part_cap) || F % (32 * p.wcn)) return 0;
    p.S = 1;
    if (lds_dma || p.mt != 10) {
        dma_launch<true>({A, W, nullptr, nullptr, M, N, K, 0, 0, out, (int)out_t, live}, p, s);
    } else {
        const int mtiles = (M + 319) / 320, total = F / 64 * mtiles;
        k_gemm_t32<10, true><<<dim3((total + 7) / 8 * 8), 256, 0, s>>>(A, W, nullptr, nullptr, M, N, K, 0, 0, 1, mtiles,
                                                                       total, out, out_t);
    }
    return 1;
}

// Rows up to which the row kernel's passes of 4 or 8 rows over the weights (which
// the caches hold) are the faster ones on every decoder measured: verify of 64,
// 128, 192 and 256 rows 102, 134, 165 and 197 us at hidden 256 (two layers), 150,
// 250, 354 and 458 at hidden 1024 (one), 1840, 3600, 5370 and 7130 at hidden 4096
// (one), in tiles 590, 597, 601 and 601; 1140, 1155, 1165 and 1172; 4930, 5100,
// 5490 and 5730.
constexpr int F32_ROWS = 192;

void launch_gemm_f32(const float* A, const float* W, float* C, int M, int N, int K, int ldc, gemm_mode mode,
                     hipStream_t s)
{
    if (M <= 4) k_gemm_f32_rows<4><<<dim3(N / 8, 1), 256, 0, s>>>(A, W, C, M, N, K, ldc, mode);
    else if (M <= F32_ROWS) k_gemm_f32_rows<8><<<dim3(N / 8, (M + 7) / 8), 256, 0, s>>>(A, W, C, M, N, K, ldc, mode);
    else k_gemm_f32<<<dim3(N / FT, (M + FT - 1) / FT), 256, 0, s>>>(A, W, C, M, N, K, ldc, mode);
}

template <int FMT>
static void q4_f32_go(const float* A, const uint32_t* Wq, const uint16_t* Sc, const uint8_t* Z, float* C, int M, int N,
                      int K, int ldc, int mode, hipStream_t s)
{
    if (M <= 4) k_gemm_q4_f32<4, FMT><<<dim3(N / 32, 1), 256, 0, s>>>(A, Wq, Sc, Z, C, M, N, K, ldc, mode);
    else k_gemm_q4_f32<8, FMT><<<dim3(N / 32, (M + 7) / 8), 256, 0, s>>>(A, Wq, Sc, Z, C, M, N, K, ldc, mode);
}

void launch_gemm_q4_f32(const float* A, const uint32_t* Wq, const uint16_t* Sc, const uint8_t* Z, int fmt, float* C,
                        int M, int N, int K, int ldc, gemm_mode mode, hipStream_t s)
{
    if (fmt == QF_W8) q4_f32_go<QF_W8>(A, Wq, Sc, Z, C, M, N, K, ldc, mode, s);
    else if (fmt == QF_W4A) q4_f32_go<QF_W4A>(A, Wq, Sc, Z, C, M, N, K, ldc, mode, s);
    else q4_f32_go<QF_W4>(A, Wq, Sc, Z, C, M, N, K, ldc, mode, s);
}
