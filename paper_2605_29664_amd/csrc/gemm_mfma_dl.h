// bf16 GEMM on the matrix cores with tiles loaded from global memory STRAIGHT
// INTO LDS (buffer_load_dwordx4 ... lds): no staging registers, no LDS-write
// instructions, and the data of a tile is in flight for at least a whole k-tile
// of matrix work. Same tiling, fragment double buffering, XCD-aware tile order and
// epilogue as gemm_mfma_kernel; no batch, no causal band, but any M, N and K that
// are multiples of 8 (the row kernels' vector width, so every shape a bf16 stage
// can have): the loads go through buffer descriptors that end where the operand
// ends, and a lane past the end writes zeros into the tile. An operand whose k rows
// lie apart may be of any length: its descriptor starts at the k-tile being loaded.
//
// One such load moves 64 lanes x 16 bytes = 1 KB to consecutive LDS addresses
// (lane l's 16 bytes land at base + 16 l), so a tile row cannot be padded.
// Bank conflicts are avoided by a swizzle instead, which costs nothing at load
// time (a lane simply fetches the piece of memory that belongs at the LDS
// position it writes) and a few precomputed lane offsets at read time:
//   * k-contiguous operand, tile [rows][64 k], 128 bytes per row = 8 chunks of
//     16 bytes: chunk c of row r sits at chunk position c ^ ((r >> 1) & 7); a
//     128-bit fragment read by 16 consecutive rows touches all 64 banks once;
//   * m/n-contiguous operand, tile [64 k][R], R*2 bytes per row: the 64-byte
//     block b of row k sits at block position b ^ (k & 3), with R = 64 (two
//     blocks to a row) at b ^ ((k >> 1) & 1); the transposing read of half a
//     wave (4 consecutive k, 64 bytes each) touches all banks once.
#pragma once
#include "gemm_mfma.h"
#include <type_traits>

namespace amdp {

// Buffer descriptor of `bytes` bytes at p (raw: range check on the byte offset).
__device__ __forceinline__ u32x4 buffer_rsrc(const void* p, unsigned bytes) {
    const uint64_t a = (uint64_t)p;
    u32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xFFFFu);
    r[2] = __builtin_amdgcn_readfirstlane(bytes);
    r[3] = 0x00020000u;
    return r;
}
constexpr unsigned BUF_OOB = 0x80000000u;      // a lane offset past the end of every descriptor used here (< 2 GiB)

// 16 bytes per lane from rsrc + voff + soff to LDS: lane l's data lands at
// lds_addr + 16 l (lds_addr uniform, in M0); zeros for a lane whose
// 16 bytes are not inside the descriptor. Written as an asm statement on
// purpose: with the compiler's own builtin its wait-count pass puts a full
// vmcnt(0) wait in front of every transposing LDS read that follows (it cannot
// tell that those read another LDS slot), which serialises the loads with the
// matrix work. The waits that are needed are written out below. M0 is an operand of
// the statement, so the compiler sets it and knows its value (saving and restoring it
// around a move inside the statement cost 3 to 10 % of a 256x256 product's main loop
// in issue slots).
__device__ __forceinline__ void load16_to_lds(u32x4 rsrc, unsigned voff, unsigned soff, lds_u8* lds_addr) {
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "{m0}"((unsigned)(__UINTPTR_TYPE__)lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory");
}
// s_barrier without the waits and fences of __syncthreads: what has to have
// arrived is waited for explicitly; the compiler moves no memory access across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// s_waitcnt vmcnt(N) alone (immediate: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64);
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// One operand's tile: R rows (m or n) by 64 k. NW = waves in the workgroup.
template <int R, bool KM, int NW>
struct DlTile {
    static constexpr int BYTES = R * MF_BK * 2;
    static constexpr int ROWB = KM ? R * 2 : MF_BK * 2;       // bytes per LDS row
    static constexpr int CHUNK_ROWS = 1024 / ROWB;            // LDS rows per 1 KB load
    static constexpr int PW = BYTES / 1024 / NW;              // loads per wave
    static_assert(BYTES % (1024 * NW) == 0, "tile must split into whole 1 KB loads per wave");
    static_assert(NW % 2 == 0 && (!KM || R == 64 || R == 128 || R == 256), "swizzle terms assume these shapes");
    __device__ static __forceinline__ int block_swizzle(int k) { return R == 64 ? (k >> 1) & 1 : k & 3; }

    // Byte offset, from the tile's first element (row 0, k 0), of what this lane
    // fetches in pass p; ld = elements between the operand's memory rows (m/n rows
    // of a k-contiguous operand, k rows of an m/n-contiguous one). `k_chunk`
    // receives the lane's first k inside the tile (k-contiguous operand only; the
    // same in every pass).
    __device__ static __forceinline__ unsigned lane_goff(int wave, int lane, int p, unsigned ld, int& k_chunk) {
        if constexpr (!KM) {
            const int row = 8 * (wave + NW * p) + (lane >> 3), pos = lane & 7;
            const int c = pos ^ ((row >> 1) & 7);
            k_chunk = 8 * c;
            return (unsigned)row * ld * 2 + c * 16;
        } else {
            const int o = 16 * lane;                          // LDS byte inside the 1 KB chunk
            const int krow = CHUNK_ROWS * (wave + NW * p) + o / ROWB, pb = o % ROWB;
            k_chunk = 0;
            return (unsigned)krow * ld * 2 + ((((pb >> 6) ^ block_swizzle(krow)) << 6) | (pb & 63));
        }
    }
    // Bytes from the descriptor's start to the end of what may be read through it:
    // `rows` m/n rows and `ks` k exist from there on. A k-contiguous operand keeps its
    // descriptor and moves the scalar offset by 128 bytes a k-tile; an m/n-contiguous
    // one, whose k rows would take that offset past 2 GiB (65536 tokens of a 16384-wide
    // FFN), moves the descriptor itself and covers one k-tile.
    __device__ static __forceinline__ unsigned extent(int rows, int ks, unsigned ld) {
        if constexpr (!KM) return ((unsigned)(min(rows, R) - 1) * ld + (unsigned)ks) * 2;
        else return ((unsigned)(min(ks, MF_BK) - 1) * ld + (unsigned)rows) * 2;
    }
    // The descriptor and scalar offset of the k-tile that starts at k; `last`: first k of the last
    // tile; `whole`, `tail`: extents of a whole k-tile and of the last one. Past that the descriptor
    // is empty and the offset 0 (zeros, no memory traffic). Scalar selects, no branch.
    __device__ static __forceinline__ void advance(u32x4& rsrc, unsigned& soff, int k, int last, unsigned ld, unsigned whole,
                                                   unsigned tail) {
        if constexpr (!KM) {
            soff = k <= last ? soff + MF_BK * 2 : 0;
            if (k > last) rsrc[2] = 0;
        } else {
            const uint64_t a = ((uint64_t)rsrc[1] << 32 | rsrc[0]) + (uint64_t)MF_BK * 2 * ld;
            rsrc[0] = (uint32_t)a;
            rsrc[1] = (uint32_t)(a >> 32);
            const unsigned e = k == last ? tail : whole;
            rsrc[2] = k <= last ? e : 0;
        }
    }

    // Fragment addressing. `origin` = first row of the wave's part of the tile.
    // !KM: index = k-step (4 lane offsets), sub-tile j is an immediate.
    //  KM: index = sub-tile (up to 4 lane offsets), k-step is an immediate.
    __device__ static __forceinline__ int frag_off(int origin, int lane, int idx) {
        if constexpr (!KM) {
            const int r = lane & 31, f = (r >> 1) & 7, half = lane >> 5;
            return (origin + r) * ROWB + (((2 * idx + half) ^ f) * 16);
        } else {
            const int q = lane >> 4, i = lane & 15;
            const int krow = 8 * (q >> 1) + (i >> 2);
            const int blk = ((origin + 32 * idx) * 2 / 64) & (ROWB / 64 - 1);   // idx past the tile is never read
            return krow * ROWB + ((blk ^ block_swizzle(krow)) << 6) + (16 * (q & 1) + 4 * (i & 3)) * 2;
        }
    }
    // f[] = lds + operand base + frag_off(origin, lane, 0..3)
    __device__ static __forceinline__ bf16x8 frag(lds_u8* const (&f)[4], int stage, int j, int kk) {
        if constexpr (!KM) {
            return *(lds_bf16x8*)(f[kk] + stage + j * 32 * ROWB);
        } else {
            lds_u8* p = f[j] + stage + kk * 16 * ROWB;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * ROWB));
            typedef __attribute__((ext_vector_type(8))) short s16x8;
            return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    }
};

// ---- epilogue ------------------------------------------------------------------
// Each wave parks one 32-row strip of its tile in LDS as fp32 and reads it back
// row-wise, so that a lane handles 8 consecutive columns (fp32 output: 4) and the
// wave writes whole row segments. The strip is private to its wave and a wave's LDS
// operations complete in issue order: no workgroup barrier between the passes. A
// lane's columns are the same in every pass, so the bias is read once; what is read
// per element (residual, GELU argument, the sum that is added to) is requested one
// strip ahead, otherwise every pass waits for memory: with one workgroup per compute
// unit the GELU' epilogue of a 4096 x 4096 product cost 28 us of its 53.
enum EpiKind { EPI_BF16, EPI_RES, EPI_GELU_OUT, EPI_GELU_GRAD, EPI_F32, EPI_F32_ACC, EPI_MIXED };
__device__ __forceinline__ EpiKind epilogue_kind(const Epilogue& e) {
    if (e.out_f32) return e.bias || e.res || e.gelu_u || e.aux_out ? EPI_MIXED : e.accumulate ? EPI_F32_ACC : EPI_F32;
    if (!e.res && !e.gelu_u && !e.aux_out) return EPI_BF16;
    if (e.res && !e.gelu_u && !e.aux_out) return EPI_RES;
    if (!e.res && !e.gelu_u && e.aux_out) return EPI_GELU_OUT;
    if (!e.res && e.gelu_u && !e.aux_out && !e.bias) return EPI_GELU_GRAD;
    return EPI_MIXED;
}

// acc: the wave's TM x TN accumulators; (m0, n0): its first row and column.
template <int KIND, int TM, int TN>
__device__ __forceinline__ void dl_epilogue(const GemmArgs& g, void* C, const f32x16 (&acc)[TM][TN], lds_f32* strip, int m0,
                                            int n0, int lane) {
    constexpr int WN = TN * 32, SW = WN + 4;
    constexpr bool F32 = KIND == EPI_F32 || KIND == EPI_F32_ACC, SIDE = KIND == EPI_RES || KIND == EPI_GELU_GRAD;
    constexpr int COLS = F32 ? 4 : 8, CPR = WN / COLS, RPP = 64 / CPR, NP = 32 / RPP;   // rows per pass, passes per strip
    const int n = n0 + lane % CPR * COLS, r0 = lane / CPR;
    const bool n_ok = n < g.N;
    const Epilogue& e = g.epi;
    float bias[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) bias[k] = 0.f;
    if constexpr (!F32 && KIND != EPI_MIXED && KIND != EPI_GELU_GRAD)
        if (e.bias && n_ok) {
            const bf16x8 b = *(const bf16x8*)((const bf16*)e.bias + n);
#pragma unroll
            for (int k = 0; k < 8; ++k) bias[k] = (float)b[k];
        }
    // what is read per element, one strip ahead (half a strip for the fp32 sum, which is twice as wide)
    constexpr int NS = KIND == EPI_F32_ACC ? (NP > 8 ? 8 : NP) : NP;
    bf16x8 side[2][SIDE ? NS : 1];
    f32x4 sum[2][KIND == EPI_F32_ACC ? NS : 1];
    const bf16* sp = KIND == EPI_RES ? (const bf16*)e.res : (const bf16*)e.gelu_u;
    const long sld = KIND == EPI_RES ? e.ldr : e.ldu;
    auto fetch = [&](int buf, int chunk) {        // chunk: NS passes
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            const long m = m0 + r0 + (chunk * NS + p) * RPP;
            if constexpr (SIDE) side[buf][p] = n_ok && m < g.M ? *(const bf16x8*)(sp + m * sld + n) : bf16x8{};
            if constexpr (KIND == EPI_F32_ACC)
                sum[buf][p] = n_ok && m < g.M ? *(const f32x4*)((const float*)C + m * g.ldc + n) : f32x4{};
        }
    };
    constexpr bool AHEAD = SIDE || KIND == EPI_F32_ACC;
    if constexpr (AHEAD) fetch(0, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                strip[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * SW + j * 32 + (lane & 31)] = acc[i][j][v];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int chunk = i * (NP / NS) + p / NS, buf = chunk & 1;
            if constexpr (AHEAD)
                if (p % NS == 0 && chunk + 1 < TM * (NP / NS)) fetch(buf ^ 1, chunk + 1);
            const int row = r0 + p * RPP;
            const long m = m0 + i * 32 + row;
            if constexpr (F32) {
                f32x4 v = *(lds_f32x4*)(strip + row * SW + lane % CPR * 4) * e.alpha;
                if constexpr (KIND == EPI_F32_ACC) v = sum[buf][p % NS] + v;
                if (n_ok && m < g.M) *(f32x4*)((float*)C + m * g.ldc + n) = v;
            } else {
                const f32x4 lo = *(lds_f32x4*)(strip + row * SW + lane % CPR * 8);
                const f32x4 hi = *(lds_f32x4*)(strip + row * SW + lane % CPR * 8 + 4);
                float v8[8];
#pragma unroll
                for (int k = 0; k < 4; ++k) { v8[k] = lo[k]; v8[4 + k] = hi[k]; }
                if constexpr (KIND == EPI_MIXED) {
                    if (n_ok && m < g.M) epilogue_store8(e, C, g.ldc, m, n, v8);
                } else {
                    bf16x8 o, h;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        float v = v8[k] * e.alpha;
                        if constexpr (KIND != EPI_GELU_GRAD) v += bias[k];
                        if constexpr (KIND == EPI_RES) v += (float)side[buf][p % NS][k];
                        if constexpr (KIND == EPI_GELU_GRAD) v *= gelu_grad_fast((float)side[buf][p % NS][k]);
                        o[k] = (bf16)v;
                        if constexpr (KIND == EPI_GELU_OUT) h[k] = (bf16)gelu_fast(v);
                    }
                    if (n_ok && m < g.M) {
                        *(bf16x8*)((bf16*)C + m * g.ldc + n) = o;
                        if constexpr (KIND == EPI_GELU_OUT) *(bf16x8*)((bf16*)e.aux_out + m * g.ldc + n) = h;
                    }
                }
            }
        }
    }
}

// ---- kernel --------------------------------------------------------------------
// Workgroup: WGM x WGN waves over the BM x BN tile. LDS: RA slots for A tiles and RB
// for B tiles (RA >= RB), refilled round robin. FD k-steps (16 k each) form a group;
// a wave holds the fragments of two groups and reads the next one while the matrix
// cores work on the current one.
//
// Schedule. Per k-tile kt there is ONE barrier, before its last group. By then every
// wave has the rest of tile kt in registers, so its two slots are free, and tile
// kt+1 has landed. The loads that fill them (B of tile kt+RB first: it is needed
// soonest; then A of tile kt+RA) are spread one by one over a whole k-tile of
// matrix instructions, and the LDS reads over the first three quarters of each
// group; sched_barrier keeps the compiler from bunching them again. Both spreads
// matter: a compute unit takes one 1 KB load per 16 cycles (64 bytes per cycle into
// LDS), loads issued faster stall the wave and with it its matrix instructions.
// LDS reads (256 bytes per cycle) and the loads' LDS writes do not disturb each
// other. Measured on 8192^3, random data, same box: compiler-scheduled predecessor
// (two stages, loads at once behind the barrier) 1205-1270 TFLOP/s by layout, this
// schedule 1355-1400; matrix instructions alone 1740 (power-limited clock).
//
// grid.z parts: part z contracts k in [z * k_part, min(K, (z+1) * k_part)) into C + z * c_bo.
template <int BM, int BN, bool A_KM, bool B_KM, int WGM, int WGN, int RA, int RB, int FD>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_mfma_dl_kernel(GemmArgs g, int k_part) {
    constexpr int NW = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 32, TN = WN / 32;
    using TA = DlTile<BM, A_KM, NW>;
    using TB = DlTile<BN, B_KM, NW>;
    static_assert(RA >= RB && RB >= 2);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    lds_u8* lds = (lds_u8*)smem_raw;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    // tile id -> (pm, pn): a contiguous run of tiles per XCD (workgroups are dealt round
    // robin to the 8 XCDs, each with its own L2), then groups of 8 row-tiles walked
    // column by column so that neighbours share operand tiles
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN, ntiles = tiles_m * tiles_n;
    const int xcd = blockIdx.x % 8;
    const int pid = xcd * (ntiles / 8) + min(xcd, ntiles % 8) + blockIdx.x / 8;
    constexpr int GROUP = 8;
    const int per_group = GROUP * tiles_n;
    const int first_m = (pid / per_group) * GROUP;
    const int gsize = min(tiles_m - first_m, GROUP);
    const int pm = first_m + (pid % per_group) % gsize;
    const int pn = (pid % per_group) / gsize;
    const int m0 = pm * BM, n0 = pn * BN;

    const int k_lo = blockIdx.z * k_part, K = min(k_part, g.K - k_lo);
    const unsigned lda = (unsigned)(A_KM ? g.a_cs : g.a_rs), ldb = (unsigned)(B_KM ? g.b_rs : g.b_cs);
    // A tile's missing rows lie past its descriptor's end. So do the missing k of an
    // m/n-contiguous operand; those of a k-contiguous one are the next row's first
    // elements, so its lanes past K are sent past the end.
    u32x4 ra = buffer_rsrc((const bf16*)g.A + (long)m0 * g.a_rs + (long)k_lo * g.a_cs, TA::extent(g.M - m0, K, lda));
    u32x4 rb = buffer_rsrc((const bf16*)g.B + (long)n0 * g.b_cs + (long)k_lo * g.b_rs, TB::extent(g.N - n0, K, ldb));
    unsigned va_off[TA::PW], vb_off[TB::PW];
    int ka, kb;
#pragma unroll
    for (int p = 0; p < TA::PW; ++p) va_off[p] = TA::lane_goff(wave, lane, p, lda, ka);
#pragma unroll
    for (int p = 0; p < TB::PW; ++p) vb_off[p] = TB::lane_goff(wave, lane, p, ldb, kb);
    unsigned sa_off = 0, sb_off = 0;
    const int nk = (K + MF_BK - 1) / MF_BK, k_last = (nk - 1) * MF_BK;
    const unsigned a_whole = TA::extent(g.M - m0, MF_BK, lda), a_tail = TA::extent(g.M - m0, K - k_last, lda);
    const unsigned b_whole = TB::extent(g.N - n0, MF_BK, ldb), b_tail = TB::extent(g.N - n0, K - k_last, ldb);
    constexpr int NVM = TA::PW + TB::PW;
    constexpr int A_BYTES = RA * TA::BYTES;
    int ka_issue = 0, kb_issue = 0;            // first k of the operand tile being issued
    int a_slot = 0, b_slot = A_BYTES;          // where it goes
    auto issue_a = [&](int p) {
        const unsigned v = (!A_KM && ka_issue + ka >= K) ? BUF_OOB : va_off[p];
        load16_to_lds(ra, v, sa_off, lds + a_slot + (wave + NW * p) * 1024);
    };
    auto issue_b = [&](int p) {
        const unsigned v = (!B_KM && kb_issue + kb >= K) ? BUF_OOB : vb_off[p];
        load16_to_lds(rb, v, sb_off, lds + b_slot + (wave + NW * p) * 1024);
    };
    // tiles past the last are issued too: the loop body has no branches and the count of
    // loads in flight is fixed
    auto next_a = [&]() {
        ka_issue += MF_BK;
        TA::advance(ra, sa_off, ka_issue, k_last, lda, a_whole, a_tail);
        a_slot = a_slot + TA::BYTES == A_BYTES ? 0 : a_slot + TA::BYTES;
    };
    auto next_b = [&]() {
        kb_issue += MF_BK;
        TB::advance(rb, sb_off, kb_issue, k_last, ldb, b_whole, b_tail);
        b_slot = b_slot + TB::BYTES == A_BYTES + RB * TB::BYTES ? A_BYTES : b_slot + TB::BYTES;
    };

    lds_u8* fa[4];
    lds_u8* fb[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        fa[x] = lds + TA::frag_off(wm * WM, lane, x);
        fb[x] = lds + A_BYTES + TB::frag_off(wn * WN, lane, x);
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    constexpr int G = 4 / FD;                  // groups per k-tile
    constexpr int NR = FD * (TM + TN);         // fragments per group
    constexpr int NM = FD * TM * TN;           // matrix instructions per group
    bf16x8 va[2][FD][TM], vb[2][FD][TN];
    auto read_frag = [&](int set, int sa, int sb, int grp, int r) {     // fragment r of group grp
        const int f = r / (TM + TN), x = r % (TM + TN), kk = grp * FD + f;
        if (x < TM) va[set][f][x] = TA::frag(fa, sa, x, kk);
        else vb[set][f][x - TM] = TB::frag(fb, sb, x - TM, kk);
    };

    // Loads that may still be on their way at the barrier of k-tile kt, before which A and B of tile
    // kt+1 must have landed: those issued behind them (B(j+RB), then A(j+RA) per barrier j < kt).
    constexpr int IN_FLIGHT = (RA > RB ? TA::PW : 0) + (RB - 2) * NVM;
    static_assert(IN_FLIGHT + NVM < 64, "vmcnt counts to 63");
#pragma unroll
    for (int j = -RA; j < 0; ++j) {
        const int upto = j == -1 ? NVM / G : NVM;      // the rest of barrier -1's loads go out in the first groups below
        if (j + RB >= 0) {
#pragma unroll
            for (int p = 0; p < TB::PW; ++p)
                if (p < upto) issue_b(p);
            if (upto >= TB::PW) next_b();
        }
#pragma unroll
        for (int p = 0; p < TA::PW; ++p)
            if (TB::PW + p < upto) issue_a(p);
        if (upto == NVM) next_a();
    }
    wait_vmcnt<IN_FLIGHT + NVM / G>();
    lds_barrier();
#pragma unroll
    for (int r = 0; r < NR; ++r) read_frag(0, 0, 0, 0, r);

    int cur_a = 0, nxt_a = TA::BYTES, cur_b = 0, nxt_b = TB::BYTES;     // slots of tiles kt and kt+1
    auto group = [&](auto set_c, auto grp_c) {
        constexpr int S = decltype(set_c)::value, GR = decltype(grp_c)::value;
        constexpr bool last = GR == G - 1;
        if constexpr (last) {
            __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): this wave's reads of tile kt, issued a group ago
            wait_vmcnt<IN_FLIGHT>();                 // tile kt+1 has landed
            lds_barrier();
            __builtin_amdgcn_sched_barrier(0);
        }
        const int rsa = last ? nxt_a : cur_a, rsb = last ? nxt_b : cur_b;
        constexpr int rgrp = last ? 0 : GR + 1;
        constexpr int POS = last ? 0 : GR + 1, L0 = POS * NVM / G, L1 = (POS + 1) * NVM / G;
        int r = 0, l = L0;
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            const int f = t / (TM * TN), i = t % (TM * TN) / TN, j = t % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[S][f][i], vb[S][f][j], acc[i][j], 0, 0, 0);
            const int r_to = min(NR, ((t + 1) * NR * 4 + 3 * NM - 1) / (3 * NM));
            for (; r < r_to; ++r) read_frag(S ^ 1, rsa, rsb, rgrp, r);
            const int l_to = min(L1, L0 + ((t + 1) * (L1 - L0) + NM - 1) / NM);
            for (; l < l_to; ++l) { if (l < TB::PW) issue_b(l); else issue_a(l - TB::PW); }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (L0 < TB::PW && L1 >= TB::PW) next_b();
        if constexpr (L1 == NVM) next_a();
    };
    auto advance = [&]() {
        cur_a = nxt_a; nxt_a = nxt_a + TA::BYTES == A_BYTES ? 0 : nxt_a + TA::BYTES;
        cur_b = nxt_b; nxt_b = nxt_b + TB::BYTES == RB * TB::BYTES ? 0 : nxt_b + TB::BYTES;
    };
    using std::integral_constant;
    typedef integral_constant<int, 0> I0;
    typedef integral_constant<int, 1> I1;
    if constexpr (FD == 4) {
        int kt = 0;
        for (; kt + 1 < nk; kt += 2) {
            group(I0{}, I0{}); advance();
            group(I1{}, I0{}); advance();
        }
        if (kt < nk) group(I0{}, I0{});
    } else {
        static_assert(FD == 1, "one k-step or a whole k-tile to a group");
        for (int kt = 0; kt < nk; ++kt) {
            group(I0{}, I0{});
            group(I1{}, I1{});
            group(I0{}, integral_constant<int, 2>{});
            group(I1{}, integral_constant<int, 3>{}); advance();
        }
    }
    wait_vmcnt<0>();           // the empty tiles' zeros are in LDS before the epilogue reuses it
    __syncthreads();

    void* C = g.epi.out_f32 ? (void*)((float*)g.C + blockIdx.z * g.c_bo) : (void*)((bf16*)g.C + blockIdx.z * g.c_bo);
    lds_f32* strip = (lds_f32*)lds + wave * (32 * (WN + 4));
    const int mw = m0 + wm * WM, nw = n0 + wn * WN;
    // the kinds a layout is used with get their own code; anything else takes the mixed form
    const EpiKind kind = epilogue_kind(g.epi);
    if constexpr (A_KM) {
        if (kind == EPI_F32) { dl_epilogue<EPI_F32, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }
        if (kind == EPI_F32_ACC) { dl_epilogue<EPI_F32_ACC, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }
    } else {
        if (kind == EPI_BF16) { dl_epilogue<EPI_BF16, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }
        if (kind == EPI_RES) { dl_epilogue<EPI_RES, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }
        if (kind == EPI_F32) { dl_epilogue<EPI_F32, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }     // parts of a split contraction
        if (B_KM && kind == EPI_GELU_OUT) { dl_epilogue<EPI_GELU_OUT, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }
        if (!B_KM && kind == EPI_GELU_GRAD) { dl_epilogue<EPI_GELU_GRAD, TM, TN>(g, C, acc, strip, mw, nw, lane); return; }
    }
    dl_epilogue<EPI_MIXED, TM, TN>(g, C, acc, strip, mw, nw, lane);
}

// True when the problem satisfies every assumption of gemm_mfma_dl_kernel (any tile):
// whole 16-byte vectors along every row, and every descriptor below 2 GiB (rows of a k-contiguous
// operand below 8 MiB, of an m/n-contiguous one below 32 MiB).
inline bool mfma_dl_shape_ok(const GemmArgs& g, bool a_km, bool b_km) {
    GemmArgs t = g;
    if (g.M % 8 || g.N % 8 || g.K % 8 || g.M <= 0 || g.N <= 0 || g.K <= 0 || g.batch != 1 || g.causal) return false;
    t.M = t.N = 64; t.K = MF_BK;
    if (!mfma_shape_ok<64, 64>(t, a_km, b_km)) return false;
    const long lda = a_km ? g.a_cs : g.a_rs, ldb = b_km ? g.b_rs : g.b_cs;
    // elements that one descriptor covers: a k-tile of an m/n-contiguous operand, a tile's rows of a k-contiguous one
    const long ea = a_km ? MF_BK * lda : 256 * lda + g.K, eb = b_km ? MF_BK * ldb : 256 * ldb + g.K;
    constexpr long LIM = (1L << 30) - 4096 * 64;      // 2 GiB less the scalar offset's overshoot
    return ea < LIM && eb < LIM;
}

// parts > 1: split contraction, fp32 parts at C + z * g.c_bo; k_part a multiple of MF_BK with
// (parts - 1) * k_part < K.
template <int BM, int BN, bool A_KM, bool B_KM, int WGM, int WGN, int RA, int RB, int FD>
inline hipError_t launch_gemm_mfma_dl(const GemmArgs& g, hipStream_t st, int parts = 1, int k_part = 0) {
    constexpr size_t lds = (size_t)(RA * BM + RB * BN) * MF_BK * 2;
    static_assert(lds <= 160 * 1024, "tile does not fit the 160 KB LDS of a CDNA4 compute unit");
    static_assert((size_t)WGM * WGN * 32 * (BN / WGN + 4) * 4 <= lds, "the epilogue's strips reuse the slots");
    constexpr auto kern = gemm_mfma_dl_kernel<BM, BN, A_KM, B_KM, WGM, WGN, RA, RB, FD>;
    if (hipError_t e = allow_dynamic_lds<kern>((int)lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN), 1, parts), dim3(64 * WGM * WGN), lds, st, g,
                       parts > 1 ? k_part : g.K);
    return hipGetLastError();
}

}  // namespace amdp
