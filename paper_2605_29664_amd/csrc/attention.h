// Fused attention for bf16 stages (any sequence length, even head widths up to
// 128): scores, mask, softmax and the value product in one kernel, so the s x s
// score / probability matrices never touch HBM. Forward saves one fp32 number
// per (sequence, head, query): the log-sum-exp of its scores.
//
// Each kernel exists for tiles of 64 and 128 head columns, and in a RAGGED form
// for heads narrower than the tile and sequences that end inside a block: its
// loads fill missing rows and columns with zeros, which add nothing to any
// product, missing keys are masked, and only what exists is stored. Head rows of
// an even width start at multiples of 4 bytes, which 16-byte loads accept. Whole
// tiles have a form of their own, without the guards.
// Before, a sequence that was no multiple of 128 kept its scores in memory and went
// through the generic product, and heads of 50 were repacked to 64 in memory. On
// MI355X, a whole accumulation window then -> now: 768 wide, 3 x 1000 tokens, 2 layers
// 12.4 -> 3.2 ms; 192 wide, 2 x 200 tokens, 2 layers 7.7 -> 4.1 ms; 1600 wide with 32
// heads of 50, 4 x 1024 tokens, 6 layers 59.8 -> 55.5 ms.
//
// Layout trick (all three kernels): every matrix product is set up so that the
// index a row-wise quantity belongs to (the query for max / sum / LSE / delta)
// is the MFMA *column* index n = lane % 32. Then each lane owns one query, its
// 16 accumulator registers per 32x32 tile hold 16 different keys, and the
// probabilities can be fed straight back into the next MFMA as its B operand
// without leaving registers: in a 32-key tile, lane half h = lane / 32 holds
// keys {4h..4h+3, 8+4h.., 16+4h.., 24+4h..}; taking registers 0..7 as the first
// 16-wide k-step and 8..15 as the second fixes a permutation of the keys, and
// the A operand (V^T, read from the [key][dh] LDS tile with the transposing
// read, 4 consecutive keys per read) is fetched in the same permuted order.
//
// What bounds them: per 32x32 tile of scores and wave a kernel spends 256 to 512 cycles
// of matrix instructions and as many of vector instructions (an exponential costs four
// others); the rest of a step is latency. So the fragments a product needs are read from
// LDS together, ahead of it and behind a scheduling fence: the value fragments before the
// softmax, the transposed ones of the backward before the exponentials. Left to the
// compiler every pair of matrix instructions waited for its own reads. The backward
// kernels' accumulators start at -lse and -delta instead of zero, which leaves two vector
// instructions per score besides the exponential and the packing. Kernel times without
// other work, before -> now (forward, dQ, dK/dV in us): 16 heads of 64, 4 x 1024 tokens,
// causal 26.2 / 30.2 / 38.8 -> 26.4 / 29.0 / 34.2; 32 heads of 64, 2 x 2048, causal
// 59.4 / 78.6 / 102 -> 58.7 / 75.0 / 93.8; 32 heads of 128, 2048, causal 66.8 / 96.5 / 146
// -> 63.5 / 93.3 / 128. With the exponentials taken out the second case takes 43 / 60 / 72,
// with the tile loads taken out 52 / 68 / 87.
#pragma once
#include "common.h"
#include "gemm_mfma.h"
#include <type_traits>

namespace amdp {

// LDS placement of a [rows][DH] bf16 tile that is read both ways: by 128-bit
// row reads (a 16-lane group reads 16 consecutive rows, 16 bytes each) and by
// transposing reads (half a wave reads 4 consecutive rows, 64 bytes each).
// With 64 banks of 4 bytes the first wants the 16 rows 4 banks apart, the
// second wants the 4 rows 16 banks apart. Both hold when the row stride is
// DH*2 + 16 bytes (4 banks past a multiple of 32 banks) and, inside every
// group of 16 rows, row 4a + i is stored at position 4i + a.
template <int DH> struct AttnTile { static constexpr int STRIDE = DH * 2 + 16; };
__device__ __forceinline__ int tile_pos(int row) { return (row & ~15) | ((row & 3) << 2) | ((row >> 2) & 3); }

constexpr float LOG2E = 1.4426950408889634f;

// 2^x as the bare hardware instruction. The library exp2f wraps it in a range
// test and a rescale for results below the normal range (four more vector
// instructions per call); here x <= 0 always and a result that small is a
// probability that rounds to zero in bf16 anyway.
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8 pack8(const f32x16& p, int first) {
    bf16x8 out;
#pragma unroll
    for (int j = 0; j < 8; ++j) out[j] = (bf16)p[first + j];
    return out;
}

// Nothing is moved across it by the compiler's scheduler.
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// A-operand fragment (rows = 32 consecutive columns c0.. of the tile, k = the
// permuted 16 keys of k-step `ks` inside the 32-row group starting at row r0).
template <int STRIDE>
__device__ __forceinline__ bf16x8 frag_tr(lds_u8* tile, int r0, int ks, int c0, int lane) {
    // rows 16ks + 4h + j (h = lane / 32, j = 0..3) sit at positions 16ks + 4j + h,
    // the rows 8 further on at positions 2 further on
    const int q = lane >> 4, i = lane & 15;
    lds_u8* p = tile + (r0 + 16 * ks + 4 * (i >> 2) + (q >> 1)) * STRIDE + (c0 + 16 * (q & 1) + 4 * (i & 3)) * 2;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 2 * STRIDE));
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// A-operand fragment with rows = 32 consecutive tile rows r0.., k = 16 consecutive columns at 16*kk.
template <int STRIDE>
__device__ __forceinline__ bf16x8 frag_row(lds_u8* tile, int r0, int kk, int lane) {
    return *(lds_bf16x8*)(tile + (r0 + tile_pos(lane & 31)) * STRIDE + (kk * 16 + 8 * (lane >> 5)) * 2);
}
// Columns [c, c + 8) of a head row of dh columns (dh even, the row 4-byte aligned):
// zeros where the row does not exist (`ok` false) and past its end, which is never read.
typedef u32x4 __attribute__((aligned(4))) u32x4_a4;
template <bool RAGGED>
__device__ __forceinline__ u32x4 load_head8(const bf16* row, int c, int dh, bool ok) {
    if constexpr (!RAGGED) {
        return *(const u32x4*)(row + c);
    } else {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (ok && c + 8 <= dh) v = *(const u32x4_a4*)(row + c);
        if (dh & 7) {                                  // the same for every lane
            if (ok && c < dh && c + 8 > dh) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if (c + 2 * j < dh) v[j] = *(const uint32_t*)(row + c + 2 * j);
            }
        }
        return v;
    }
}

// A fragment that stays in registers over a kernel's whole loop: waits for its load here.
// Left to its first use inside the loop, the wait there (memory counters complete in
// order) is one for every load before that use, each step's prefetch among them.
__device__ __forceinline__ bf16x8 arrived(u32x4 v) {
    asm volatile("" : "+v"(v));
    return __builtin_bit_cast(bf16x8, v);
}

// Cooperative copy of ROWS x DH bf16 (row stride ld elements in memory, `rows` rows
// of dh columns exist) into an LDS tile, split in two so the global loads of the next
// tile can be in flight while the current one is being multiplied.
template <int DH, int ROWS, int NT, bool RAGGED>
struct TileCopy {
    static constexpr int VPR = DH / 8, NV = ROWS * VPR / NT, STRIDE = AttnTile<DH>::STRIDE;
    u32x4 r[NV];
    __device__ __forceinline__ void fetch(const bf16* src, long ld, int tid, int rows, int dh) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int v = tid + i * NT, row = v / VPR, c = v % VPR;
            r[i] = load_head8<RAGGED>(src + (long)row * ld, c * 8, dh, row < rows);
        }
    }
    __device__ __forceinline__ void store(lds_u8* tile, int tid) const {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int v = tid + i * NT, row = v / VPR, c = v % VPR;
            *(lds_u32x4*)(tile + tile_pos(row) * STRIDE + c * 16) = r[i];
        }
    }
};

// Work order. The grid is one-dimensional over (128-row block, sequence*head).
// Under a causal mask a block's work grows with its position, so blocks are
// numbered heaviest first (rank 0 = most work; the dispatcher hands them out
// in order as slots free up). When the whole grid is resident at once
// (total <= resident) that does nothing; there the compute unit that takes
// block i also takes block i + total/2, so the second half is numbered lightest
// first and every unit gets a heavy and a light block.
__device__ __forceinline__ void attn_block(int i, int nq, int nz, int resident, bool causal, int& rank, int& z) {
    if (!causal) { rank = i % nq; z = i / nq; return; }
    const int total = nq * nz;
    int j = i;
    if (total <= resident && i >= total / 2) j = total - 1 - (i - total / 2);
    rank = j / nz;
    z = j % nz;
}

// Row of a head from the accumulators of its 32-column tiles (this lane: its half's columns).
template <int NTILES, bool RAGGED, int NACC>
__device__ __forceinline__ void store_headrow(bf16* row, const f32x16 (&acc)[NACC], int half, float mul, int dh) {
    typedef bf16x4 __attribute__((aligned(4))) bf16x4_a4;
#pragma unroll
    for (int t = 0; t < NTILES; ++t)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)(acc[t][4 * gq + e] * mul);
            const int c = t * 32 + 8 * gq + 4 * half;
            if constexpr (!RAGGED) {
                *(bf16x4*)(row + c) = o;
            } else if (c + 4 <= dh) {
                *(bf16x4_a4*)(row + c) = o;
            } else if (c + 2 <= dh) {
                row[c] = o[0];
                row[c + 1] = o[1];
            }
        }
}

// ---------------------------------------------------------------- forward
// grid ceil(s/128) * (b*H) blocks, see attn_block; 4 waves, each owns 32 queries; keys in blocks of 64.
// qkv: [b*s, 3D] (Q | K | V column blocks, heads of dh <= DH); O: [b*s, D];
// lse2: [b*H, s] = log2-domain log-sum-exp of scale*scores.
template <int DH, bool CAUSAL, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void flash_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ O,
                                                        float* __restrict__ lse2,
                                                        const int32_t* __restrict__ valid_len, int s, int H,
                                                        int D, int dh, float scale_log2e, int nz, int resident) {
    constexpr int STRIDE = AttnTile<DH>::STRIDE, BKV = 64, KQ = DH / 16, DT = DH / 32;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BKV * STRIDE];
    lds_u8* tK = (lds_u8*)smem;
    lds_u8* tV = tK + BKV * STRIDE;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int rank, z;
    attn_block(blockIdx.x, (s + 127) / 128, nz, resident, CAUSAL, rank, z);
    const int qb = CAUSAL ? (s + 127) / 128 - 1 - rank : rank;      // late queries see the most keys
    const int b = z / H, h = z % H;
    const long ld = 3L * D;
    if constexpr (!RAGGED) dh = DH;
    const bf16* base = qkv + (long)b * s * ld + (long)h * dh;
    const int q_blk = qb * 128, q_wave = q_blk + wave * 32, q = q_wave + (lane & 31);
    const int half = lane >> 5;

    bf16x8 bq[KQ];   // B operand: n = query, k = head dimension
    {
        u32x4 raw[KQ];
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) raw[kk] = load_head8<RAGGED>(base + (long)q * ld, kk * 16 + 8 * half, dh, q < s);
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) bq[kk] = arrived(raw[kk]);
    }

    f32x16 acc[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    int kend = s;
    if (CAUSAL) kend = RAGGED ? min(q_blk + 128, s) : q_blk + 128;
    if (valid_len) kend = min(kend, (max(valid_len[b], 1) + BKV - 1) / BKV * BKV);
    const int klimit = valid_len ? min(valid_len[b], s) : s;

    TileCopy<DH, BKV, 256, RAGGED> cK, cV;
    if (kend > 0) {
        cK.fetch(base + D, ld, tid, s, dh);
        cV.fetch(base + 2 * D, ld, tid, s, dh);
    }
    for (int k0 = 0; k0 < kend; k0 += BKV) {
        __syncthreads();                              // everyone is done with the previous tiles
        cK.store(tK, tid);
        cV.store(tV, tid);
        __syncthreads();
        if (k0 + BKV < kend) {                        // next tiles travel while this one is used
            cK.fetch(base + D + (long)(k0 + BKV) * ld, ld, tid, s - k0 - BKV, dh);
            cV.fetch(base + 2 * D + (long)(k0 + BKV) * ld, ld, tid, s - k0 - BKV, dh);
        }
        if (RAGGED && q_wave >= s) continue;          // none of this wave's queries exists
        if (CAUSAL && k0 > q_wave + 31) continue;     // every key of the block is hidden from this wave

        f32x16 st[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) st[kt][v] = 0.f;
#pragma unroll
        for (int r = 0; r < DH / 64; ++r) {
            bf16x8 ka[KQ / (DH / 64)][2];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) ka[kk][kt] = frag_row<STRIDE>(tK, kt * 32, 4 * r + kk, lane);
            sched_fence();
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
                    st[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk][kt], bq[4 * r + kk], st[kt], 0, 0, 0);
        }
        sched_fence();
        bf16x8 va[2][2][DT];       // of the first 32 keys for wide heads, of all 64 for narrow ones
        auto read_v = [&](int kt) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int t = 0; t < DT; ++t) va[DH == 64 ? kt : 0][ks][t] = frag_tr<STRIDE>(tV, kt * 32, ks, t * 32, lane);
        };
        read_v(0);
        if constexpr (DH == 64) read_v(1);
        sched_fence();
        // Softmax in the log2 domain on the raw scores: x = c*s, p = exp2(c*s - m).
        // Masks only where a block touches the diagonal or the padding edge
        // (wave-uniform test); everything else is one max, one fma, one exp2 and
        // one add per score.
        const bool edge = (CAUSAL && k0 + BKV - 1 > q_wave) || k0 + BKV > klimit;
        if (edge) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = k0 + kt * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                    if ((CAUSAL && key > q) || key >= klimit) st[kt][v] = -INFINITY;
                }
        }
        float mloc = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) mloc = fmaxf(mloc, st[kt][v]);
        mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64)) * scale_log2e;      // scale > 0 commutes with max
        const float m_new = fmaxf(m_run, mloc);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        float lsum = 0.f;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = exp2_raw(fmaf(st[kt][v], scale_log2e, -m_use));
                st[kt][v] = p;
                lsum += p;
            }
        if (m_new != m_run) {          // most blocks leave the running maximum alone
            const float alpha = exp2_raw(m_run - m_use);
            l_run *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][v] *= alpha;
            m_run = m_new;
        }
        l_run += lsum;
        // O^T += V^T P^T
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            if constexpr (DH != 64)
                if (kt) { sched_fence(); read_v(1); sched_fence(); }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const bf16x8 pb = pack8(st[kt], 8 * ks);
#pragma unroll
                for (int t = 0; t < DT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[DH == 64 ? kt : 0][ks][t], pb, acc[t], 0, 0, 0);
            }
        }
    }

    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (RAGGED && q >= s) return;
    store_headrow<DT, RAGGED>(O + ((long)b * s + q) * D + (long)h * dh, acc, half, inv, dh);
    if (half == 0) lse2[(long)z * s + q] = m_run + log2f(l_tot);
}


// ---------------------------------------------------------------- backward
// dK, dV. Same grid; each wave owns 32 keys (lane % 32) and walks the
// query tiles of 64 that can see them. dqkv: [b*s, 3D], K block at +D, V at +2D.
template <int DH, bool CAUSAL, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DH == 64 ? 2 : 1))) void flash_bwd_dkv_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dO,
                                                            const float* __restrict__ lse2,
                                                            const float* __restrict__ delta, bf16* __restrict__ dqkv,
                                                            const int32_t* __restrict__ valid_len, int s, int H,
                                                            int D, int dh, float scale, int nz, int resident) {
    constexpr int STRIDE = AttnTile<DH>::STRIDE, BQ = 64, KQ = DH / 16, DT = DH / 32;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BQ * STRIDE];
    __shared__ __attribute__((aligned(16))) float sstat[2][BQ];
    lds_u8* tQ = (lds_u8*)smem;
    lds_u8* tdO = tQ + BQ * STRIDE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    int rank, z;
    attn_block(blockIdx.x, (s + 127) / 128, nz, resident, CAUSAL, rank, z);     // early keys are seen by the most queries
    const int b = z / H, h = z % H;
    const long ld = 3L * D;
    if constexpr (!RAGGED) dh = DH;
    const bf16* base = qkv + (long)b * s * ld + (long)h * dh;
    const bf16* dObase = dO + (long)b * s * D + (long)h * dh;
    const int k_blk = rank * 128, k_wave = k_blk + wave * 32, key = k_wave + (lane & 31);
    const int klimit = valid_len ? min(valid_len[b], s) : s;
    const float sl2 = scale * LOG2E;
    const bool key_dead = key >= klimit;     // padding: this lane's key is visible to nobody

    bf16x8 bk[KQ], bv[KQ];      // B operands: n = key, k = head dimension
    {
        const bf16* krow = base + D + (long)key * ld;
        u32x4 rk[KQ], rv[KQ];
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            rk[kk] = load_head8<RAGGED>(krow, kk * 16 + 8 * half, dh, key < s);
            rv[kk] = load_head8<RAGGED>(krow + D, kk * 16 + 8 * half, dh, key < s);
        }
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) { bk[kk] = arrived(rk[kk]); bv[kk] = arrived(rv[kk]); }
    }
    f32x16 dk[4], dv[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) { dk[t][v] = 0.f; dv[t][v] = 0.f; }

    const int q_begin = CAUSAL ? k_blk : 0;
    const bool block_live = k_blk < klimit;
    TileCopy<DH, BQ, 256, RAGGED> cQ, cdO;
    float stat_next = 0.f;      // threads 0..63: lse of query tid; 64..127: delta of query tid-64
    const float* stat_src = tid < BQ ? lse2 + (long)z * s + tid : delta + (long)z * s + (tid - BQ);
    const float stat_mul = tid < BQ ? -1.0f / sl2 : -1.0f;
    // a query past the end gets probability 0 from an infinite log-sum-exp, and delta 0
    auto stat_at = [&](int q0) {
        if (RAGGED && q0 + tid % BQ >= s) return tid < BQ ? INFINITY : 0.f;
        return stat_src[q0];
    };
    if (block_live && q_begin < s) {
        cQ.fetch(base + (long)q_begin * ld, ld, tid, s - q_begin, dh);
        cdO.fetch(dObase + (long)q_begin * D, D, tid, s - q_begin, dh);
        if (tid < 2 * BQ) stat_next = stat_at(q_begin);
    }
    for (int q0 = q_begin; q0 < s && block_live; q0 += BQ) {
        __syncthreads();
        cQ.store(tQ, tid);
        cdO.store(tdO, tid);
        if (tid < 2 * BQ) sstat[tid / BQ][tid % BQ] = stat_next * stat_mul;
        __syncthreads();
        if (q0 + BQ < s) {
            cQ.fetch(base + (long)(q0 + BQ) * ld, ld, tid, s - q0 - BQ, dh);
            cdO.fetch(dObase + (long)(q0 + BQ) * D, D, tid, s - q0 - BQ, dh);
            if (tid < 2 * BQ) stat_next = stat_at(q0 + BQ);
        }
        if (RAGGED && k_wave >= s) continue;
        if (CAUSAL && q0 + BQ - 1 < k_wave) continue;      // none of these queries sees this wave's keys
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            // The accumulators start at -lse / (scale log2 e) and -delta, so that one product each gives
            // the exponent's argument and dP - delta.
            f32x16 sc, dp;
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const f32x4 l4 = *(const f32x4*)&sstat[0][qt * 32 + 8 * gq + 4 * half];
                const f32x4 d4 = *(const f32x4*)&sstat[1][qt * 32 + 8 * gq + 4 * half];
#pragma unroll
                for (int e = 0; e < 4; ++e) { sc[4 * gq + e] = l4[e]; dp[4 * gq + e] = d4[e]; }
            }
#pragma unroll
            for (int r = 0; r < DH / 64; ++r) {
                bf16x8 aq[4], ado[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    aq[kk] = frag_row<STRIDE>(tQ, qt * 32, 4 * r + kk, lane);
                    ado[kk] = frag_row<STRIDE>(tdO, qt * 32, 4 * r + kk, lane);
                }
                sched_fence();
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[kk], bk[4 * r + kk], sc, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ado[kk], bv[4 * r + kk], dp, 0, 0, 0);
                }
            }
            sched_fence();
            bf16x8 tq[2][DT], tdo[2][DT];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    tdo[ks][t] = frag_tr<STRIDE>(tdO, qt * 32, ks, t * 32, lane);
                    tq[ks][t] = frag_tr<STRIDE>(tQ, qt * 32, ks, t * 32, lane);
                }
            sched_fence();
            // masks only where this wave's keys meet the diagonal or the padding edge
            // (wave-uniform test): elsewhere one fma, one exp2, one sub, one mul per score
            const bool edge = CAUSAL ? (q0 + qt * 32 < k_wave + 31) : (k_wave + 31 >= klimit);
            auto probabilities = [&](auto masked) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = sc[v] * sl2;
                    if constexpr (decltype(masked)::value) {
                        const int q = q0 + qt * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                        x = ((CAUSAL && key > q) || key_dead) ? -INFINITY : x;     // before the exponential: a select, no branch
                    }
                    sc[v] = exp2_raw(x);
                    dp[v] *= sc[v];          // the factor `scale` of dS is applied to dK at the end
                }
            };
            if (edge) probabilities(std::true_type{}); else probabilities(std::false_type{});
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const bf16x8 pb = pack8(sc, 8 * ks), dsb = pack8(dp, 8 * ks);
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    dv[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tdo[ks][t], pb, dv[t], 0, 0, 0);
                    dk[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tq[ks][t], dsb, dk[t], 0, 0, 0);
                }
            }
        }
    }
    if (RAGGED && key >= s) return;
    bf16* out = dqkv + ((long)b * s + key) * ld + (long)h * dh;
    store_headrow<DT, RAGGED>(out + D, dk, half, scale, dh);
    store_headrow<DT, RAGGED>(out + 2 * D, dv, half, 1.0f, dh);
}

// dQ. Same grid; each wave owns 32 queries and walks the key blocks of 64 it can see.
// It also computes delta[z][q] = sum_d dO[q, d] * O[q, d] (z = sequence*H + head), which the
// dK / dV kernel reads: a lane already holds half of its query's dO row, so only O has
// to be read (a pass over dO and O of its own took 8-11 us a layer at 4096 tokens x 1024).
template <int DH, bool CAUSAL, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void flash_bwd_dq_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dO,
                                                           const bf16* __restrict__ O, const float* __restrict__ lse2,
                                                           float* __restrict__ delta, bf16* __restrict__ dqkv,
                                                           const int32_t* __restrict__ valid_len, int s, int H,
                                                           int D, int dh, float scale, int nz, int resident) {
    constexpr int STRIDE = AttnTile<DH>::STRIDE, BKV = 64, KQ = DH / 16, DT = DH / 32;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BKV * STRIDE];
    lds_u8* tK = (lds_u8*)smem;
    lds_u8* tV = tK + BKV * STRIDE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    int rank, z;
    attn_block(blockIdx.x, (s + 127) / 128, nz, resident, CAUSAL, rank, z);
    const int qb = CAUSAL ? (s + 127) / 128 - 1 - rank : rank;
    const int b = z / H, h = z % H;
    const long ld = 3L * D;
    if constexpr (!RAGGED) dh = DH;
    const bf16* base = qkv + (long)b * s * ld + (long)h * dh;
    const int q_blk = qb * 128, q_wave = q_blk + wave * 32, q = q_wave + (lane & 31);
    const int klimit = valid_len ? min(valid_len[b], s) : s;
    const float sl2 = scale * LOG2E;
    const bool q_ok = !RAGGED || q < s;

    bf16x8 bq[KQ], bdo[KQ];     // B operands: n = query, k = head dimension
    float delta_q = 0.f;
    {
        const bf16* dorow = dO + ((long)b * s + q) * D + (long)h * dh;
        const bf16* orow = O + ((long)b * s + q) * D + (long)h * dh;
        u32x4 rq[KQ], rdo[KQ], ro[KQ];
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            rq[kk] = load_head8<RAGGED>(base + (long)q * ld, kk * 16 + 8 * half, dh, q_ok);
            rdo[kk] = load_head8<RAGGED>(dorow, kk * 16 + 8 * half, dh, q_ok);
            ro[kk] = load_head8<RAGGED>(orow, kk * 16 + 8 * half, dh, q_ok);
        }
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            bq[kk] = arrived(rq[kk]);
            bdo[kk] = arrived(rdo[kk]);
            const bf16x8 o = arrived(ro[kk]);
#pragma unroll
            for (int e = 0; e < 8; ++e) delta_q += (float)bdo[kk][e] * (float)o[e];
        }
    }
    delta_q += __shfl_xor(delta_q, 32, 64);
    // As in the dK / dV kernel the accumulators start at -lse / (scale log2 e) and -delta. Two sets of
    // 16 registers hold these over the loop, which 128 columns do not leave free (70 spilled).
    constexpr bool FOLD = DH == 64;
    const float neg_lse = q_ok ? -lse2[(long)z * s + q] / (FOLD ? sl2 : 1.0f) : 0.f;
    if (half == 0 && q_ok) delta[(long)z * s + q] = delta_q;
    f32x16 dq[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) dq[t][v] = 0.f;

    int kend = s;
    if (CAUSAL) kend = RAGGED ? min(q_blk + 128, s) : q_blk + 128;
    if (valid_len) kend = min(kend, (max(klimit, 1) + BKV - 1) / BKV * BKV);
    TileCopy<DH, BKV, 256, RAGGED> cK, cV;
    if (kend > 0) {
        cK.fetch(base + D, ld, tid, s, dh);
        cV.fetch(base + 2 * D, ld, tid, s, dh);
    }
    for (int k0 = 0; k0 < kend; k0 += BKV) {
        __syncthreads();
        cK.store(tK, tid);
        cV.store(tV, tid);
        __syncthreads();
        if (k0 + BKV < kend) {
            cK.fetch(base + D + (long)(k0 + BKV) * ld, ld, tid, s - k0 - BKV, dh);
            cV.fetch(base + 2 * D + (long)(k0 + BKV) * ld, ld, tid, s - k0 - BKV, dh);
        }
        if (RAGGED && q_wave >= s) continue;          // none of this wave's queries exists
        if (CAUSAL && k0 > q_wave + 31) continue;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            f32x16 sc, dp;
#pragma unroll
            for (int v = 0; v < 16; ++v) { sc[v] = FOLD ? neg_lse : 0.f; dp[v] = FOLD ? -delta_q : 0.f; }
            bf16x8 tk[2][DT];
            auto read_tk = [&](int ks) {
#pragma unroll
                for (int t = 0; t < DT; ++t) tk[ks][t] = frag_tr<STRIDE>(tK, kt * 32, ks, t * 32, lane);
            };
            if constexpr (DH == 64) {
                bf16x8 ak[KQ], av[KQ];
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    ak[kk] = frag_row<STRIDE>(tK, kt * 32, kk, lane);
                    av[kk] = frag_row<STRIDE>(tV, kt * 32, kk, lane);
                }
                sched_fence();
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak[kk], bq[kk], sc, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[kk], bdo[kk], dp, 0, 0, 0);
                }
                sched_fence();
                read_tk(0);
                read_tk(1);
                sched_fence();
            } else {          // no registers left to read ahead (tried: 82 spilled, 95 -> 180 us at 32 heads of 128, 2048 tokens)
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row<STRIDE>(tK, kt * 32, kk, lane), bq[kk], sc, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_row<STRIDE>(tV, kt * 32, kk, lane), bdo[kk], dp, 0, 0, 0);
                }
            }
            // masks only where the key tile meets this wave's diagonal or the padding edge (wave-uniform)
            const bool edge = CAUSAL ? (k0 + kt * 32 + 31 > q_wave) : (k0 + kt * 32 + 31 >= klimit);
            auto dscores = [&](auto masked) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = FOLD ? sc[v] * sl2 : fmaf(sc[v], sl2, neg_lse);
                    if constexpr (decltype(masked)::value) {
                        const int key = k0 + kt * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                        x = (CAUSAL ? key > q : key >= klimit) ? -INFINITY : x;   // causal stages carry no padding mask
                    }
                    dp[v] = exp2_raw(x) * (FOLD ? dp[v] : dp[v] - delta_q);       // the factor `scale` of dS is applied to dQ at the end
                }
            };
            // (at head dimension 128 the second copy of the loop body costs 14 spilled registers
            // and 13 % of the kernel's time: there every tile takes the masked form)
            if (DH == 128 || edge) dscores(std::true_type{}); else dscores(std::false_type{});
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                if constexpr (DH != 64) read_tk(ks);
                const bf16x8 dsb = pack8(dp, 8 * ks);
#pragma unroll
                for (int t = 0; t < DT; ++t)
                    dq[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tk[ks][t], dsb, dq[t], 0, 0, 0);
            }
        }
    }
    if (RAGGED && q >= s) return;
    store_headrow<DT, RAGGED>(dqkv + ((long)b * s + q) * ld + (long)h * dh, dq, half, scale, dh);
}

}  // namespace amdp
