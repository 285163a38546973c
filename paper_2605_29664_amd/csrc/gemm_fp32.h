// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, products
// and sums), any shape, any strides: the products of fp32 stages.
//
// What bounds it: the small stages that run in fp32 have products of a few dozen
// tiles with contractions of 32 to 512, so a launch is a chain of memory latencies.
// Two tilings of the same code:
//   split: 32x32 outputs per workgroup, every chunk of 128 k divided over its four
//          waves, whose sums are added in wave order at the end. A wave loads what it
//          alone needs into its own part of LDS: no barrier until that sum, and a
//          128-long contraction is one round trip to memory;
//   tile:  64x64 outputs per workgroup, 32x32 per wave, chunks of 32 k through two
//          LDS buffers: half the loads per product, for outputs with enough tiles.
// Loads of the next chunk are in flight during the matrix instructions of the current one.
// Products of one window on MI355X against the vector-unit kernel with 64x64 tiles and loads
// waited for in every chunk of 16: 128 wide, 128 tokens 2.4 -> 0.59 ms; 512 wide, 2048 tokens
// 10 -> 52 TFLOP/s. Partial sums per wave and chunk also bring the results closer to those
// in 64 bits (worst gradient of a 256-wide stage 1.2e-6 -> 6.0e-7).
#pragma once
#include "common.h"
#include "gemm_mfma.h"

namespace amdp {

constexpr int F32_KC = 32;     // k per wave and chunk
// 64x64 tiles from this many per compute unit on. One layer's accumulation windows (four minibatches),
// always tiled / always split: 128 wide, 128 tokens 0.95 / 0.84 ms; 512 wide, 512 tokens 1.96 / 1.17;
// 512 wide, 2048 tokens 2.87 / 2.89 and 2.66 with the line at 2 or at 4.
constexpr int F32_TILE_MIN_PER_CU = 2;

// ROWS x 32 k of one operand, loaded by NT lanes into registers and stored to LDS as
// [k][ROWS + 4]: a k row's elements are consecutive for the fragment reads, and the 4
// make the scattered stores of a k-contiguous operand (16 lanes a k, 4 k apart) hit
// different banks. KC: k is contiguous in memory, else the row index (m or n) is.
// VEC: 16-byte loads (a vector never straddles the operand's end).
template <int ROWS, int NT, bool KC, bool VEC>
struct F32Tile {
    static constexpr int S = ROWS + 4, NP = ROWS * F32_KC / 4 / NT;
    f32x4 r[NP];
    __device__ static __forceinline__ void pos(int t, int p, int& row, int& k) {
        if constexpr (KC) {
            constexpr int RPP = NT / 4, HALVES = ROWS / RPP;
            row = t / 4 + RPP * (p % HALVES);
            k = 4 * (t % 4) + 16 * (p / HALVES);
        } else {
            constexpr int VR = ROWS / 4;
            row = 4 * (t % VR);
            k = t / VR + (NT / VR) * p;
        }
    }
    // src: element (row 0, k 0) of the tile; `rows` rows and `ks` k exist from there on
    __device__ __forceinline__ void fetch(const float* src, long ld, int t, int rows, int ks) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            int row, k;
            pos(t, p, row, k);
            const float* q = src + (KC ? row * ld + k : k * ld + row);
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if constexpr (VEC) {
                if (row < rows && k < ks) v = *(const f32x4*)q;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (row + (KC ? 0 : e) < rows && k + (KC ? e : 0) < ks) v[e] = q[e];
            }
            r[p] = v;
        }
    }
    __device__ __forceinline__ void store(lds_f32* tile, int t) const {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            int row, k;
            pos(t, p, row, k);
            if constexpr (KC) {
#pragma unroll
                for (int e = 0; e < 4; ++e) tile[(k + e) * S + row] = r[p][e];
            } else {
                *(lds_f32x4*)(tile + k * S + row) = r[p];
            }
        }
    }
};

template <bool SPLIT, bool A_KC, bool B_KC, bool VEC>
__global__ __launch_bounds__(256) void gemm_fp32_kernel(GemmArgs g) {
    constexpr int T = SPLIT ? 32 : 64, NT = SPLIT ? 64 : 256, STEP = SPLIT ? 4 * F32_KC : F32_KC;
    typedef F32Tile<T, NT, A_KC, VEC> TA;
    typedef F32Tile<T, NT, B_KC, VEC> TB;
    constexpr int TILE = F32_KC * (T + 4);                 // floats of one operand's tile
    __shared__ __attribute__((aligned(16))) float smem[(SPLIT ? 4 : 2) * 2 * TILE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = SPLIT ? lane : tid;
    lds_f32* lds = (lds_f32*)smem + (SPLIT ? wave * 2 * TILE : 0);

    const long zo = blockIdx.z / g.batch_inner, zi = blockIdx.z % g.batch_inner;
    const int tiles_n = (g.N + T - 1) / T;
    const int m0 = (int)(blockIdx.x / tiles_n) * T, n0 = (int)(blockIdx.x % tiles_n) * T;
    if (g.causal == 1 && n0 > m0 + T - 1) return;
    const int k_lo = g.causal == 3 ? m0 : 0, k_hi = g.causal == 2 ? min(g.K, m0 + T) : g.K;

    const long a_ld = A_KC ? g.a_rs : g.a_cs, b_ld = B_KC ? g.b_cs : g.b_rs;
    const float* A = (const float*)g.A + zo * g.a_bo + zi * g.a_bi + m0 * g.a_rs;
    const float* B = (const float*)g.B + zo * g.b_bo + zi * g.b_bi + n0 * g.b_cs;
    TA ta;
    TB tb;
    int k0 = k_lo + (SPLIT ? wave * F32_KC : 0);           // first k of this wave's next chunk
    auto fetch = [&]() {
        ta.fetch(A + k0 * g.a_cs, a_ld, t, g.M - m0, k_hi - k0);
        tb.fetch(B + k0 * g.b_rs, b_ld, t, g.N - n0, k_hi - k0);
        k0 += STEP;
    };
    // this wave's 32x32 outputs inside the tile
    const int wm = SPLIT ? 0 : (wave >> 1) * 32, wn = SPLIT ? 0 : (wave & 1) * 32;
    const int ra = wm + (lane & 31) + (lane >> 5) * TA::S, rb = wn + (lane & 31) + (lane >> 5) * TB::S;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;

    const int chunks = (k_hi - k_lo + STEP - 1) / STEP;    // the same for every wave
    if (chunks > 0) fetch();
    for (int c = 0; c < chunks; ++c) {
        // split: a wave's LDS operations complete in order, so its stores cannot overtake the
        // previous chunk's reads; tile: the other buffer's readers are behind the last barrier
        lds_f32* la = lds + (SPLIT ? 0 : (c & 1) * 2 * TILE);
        lds_f32* lb = la + TILE;
        __builtin_amdgcn_wave_barrier();
        ta.store(la, t);
        tb.store(lb, t);
        if constexpr (SPLIT) __builtin_amdgcn_wave_barrier(); else __syncthreads();
        if (c + 1 < chunks) fetch();
#pragma unroll
        for (int k = 0; k < F32_KC; k += 2)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(la[k * TA::S + ra], lb[k * TB::S + rb], acc, 0, 0, 0);
    }

    void* C = (float*)g.C + zo * g.c_bo + zi * g.c_bi;
    const int n = n0 + wn + (lane & 31);
    if constexpr (SPLIT) {
        __syncthreads();
        lds_f32* sum = (lds_f32*)smem;
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[(wave * 16 + v) * 64 + lane] = acc[v];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = wave * 4 + i;
            float x = sum[v * 64 + lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) x += sum[(w * 16 + v) * 64 + lane];
            const int m = m0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (m < g.M && n < g.N) epilogue_store<float>(g.epi, C, g.ldc, m, n, x);
        }
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + wm + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (m < g.M && n < g.N) epilogue_store<float>(g.epi, C, g.ldc, m, n, acc[v]);
        }
    }
}

// One of each operand's two strides is 1 (all layouts of a stage); n_cu: compute units.
inline hipError_t launch_gemm_fp32(const GemmArgs& g, int n_cu, hipStream_t st) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    const bool a_kc = g.a_cs == 1, b_kc = g.b_rs == 1;
    const long a_ld = a_kc ? g.a_rs : g.a_cs, b_ld = b_kc ? g.b_cs : g.b_rs;
    const bool vec = (((uintptr_t)g.A | (uintptr_t)g.B) & 15) == 0 &&
                     ((a_ld | b_ld | g.a_bo | g.a_bi | g.b_bo | g.b_bi) & 3) == 0 && (a_kc ? g.K : g.M) % 4 == 0 &&
                     (b_kc ? g.K : g.N) % 4 == 0;
    auto tiles = [&](int t) { return (long)((g.M + t - 1) / t) * ((g.N + t - 1) / t); };
    const bool split = tiles(64) * g.batch < F32_TILE_MIN_PER_CU * n_cu;
    const dim3 grid((unsigned)tiles(split ? 32 : 64), 1, g.batch);
#define F32_GEMM(S, A, B, V) hipLaunchKernelGGL((gemm_fp32_kernel<S, A, B, V>), grid, dim3(256), 0, st, g)
#define F32_VEC(S, A, B) do { if (vec) F32_GEMM(S, A, B, true); else F32_GEMM(S, A, B, false); } while (0)
#define F32_LAYOUT(S)                                                                          \
    do {                                                                                       \
        if (a_kc) { if (b_kc) F32_VEC(S, true, true); else F32_VEC(S, true, false); }          \
        else { if (b_kc) F32_VEC(S, false, true); else F32_VEC(S, false, false); }             \
    } while (0)
    if (split) F32_LAYOUT(true); else F32_LAYOUT(false);
#undef F32_LAYOUT
#undef F32_VEC
#undef F32_GEMM
    return hipGetLastError();
}

}  // namespace amdp
