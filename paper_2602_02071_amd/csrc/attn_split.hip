// Split-key passes of the fused BAPS attention forward, for few query rows
// per key/value head and few (batch, key/value head) streams (single-sequence
// or small-batch decode over long contexts), where one workgroup per stream
// would leave most of the GPU idle.
//
// Alg. 1 visits the key blocks of a row in order, but its state after block j
// (the integer running maximum m and the block reference) depends on the keys
// only through each block's row maximum.  So:
//   1. scores: every key split in parallel streams K and writes the raw dot
//      products acc = q.k (fp32, as the MFMA accumulates them) and the raw
//      row maximum of every block;
//   2. pv: every split in parallel first replays Alg. 1's B0 / restart rule
//      and integer maximum over the block maxima of its rows, from block 0 to
//      its own last block -- the same per-block decision as the one-pass
//      kernels, many blocks per step, serial only where m changes -- then
//      streams V, forms P = HiF8(2^HiF8(T)) with T = fl32(acc*c - ref_j), and
//      accumulates X and dX relative to its latest reference;
//   3. combine: per row, the splits' X and dX brought to the largest
//      reference with exact powers of two (references never decrease along a
//      row) and summed: O = sum X / sum dX, and lse.
// Every T, P and reference equals the one-pass kernels'; O differs only by
// the order of the fp32 additions.

#include <type_traits>

#include "common.hpp"

namespace baps {

namespace {

typedef __bf16 bf16x2 __attribute__((__vector_size__(2 * sizeof(__bf16))));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

constexpr int kRows = 16;            // query rows per workgroup (16x16x32 MFMA columns)
constexpr int kSlotKeys = 32;        // keys per wave and block, and per ring slot

// A workgroup's W waves are KW key slots (wave % KW takes 32 keys of a block)
// times BG block groups (wave / KW takes every BG-th block of the split: the
// blocks are independent once the references are known), with 16 KiB of ring
// each.  launch_split_rt picks four waves, two workgroups of which share a CU,
// or, where the grid holds at most one per CU, eight; or one group alone.
template <int D, int BLK, int W>
struct SCfg {
    static constexpr int kWaves = W;
    static constexpr int kKeySlots = BLK / kSlotKeys;
    static constexpr int kGroups = kWaves / kKeySlots;
    static constexpr int kRowBytes = 2 * D;
    static constexpr int kCPR = D / 8;                          // 16-byte chunks per row
    static constexpr int kSlotBytes = kSlotKeys * kRowBytes;
    static constexpr int kIPS = kSlotBytes / 1024;              // wave-wide loads per slot
    static constexpr int kRW = 16 * 1024 / kSlotBytes;          // ring slots per wave
    static constexpr int kLdsBytes = kWaves * kRW * kSlotBytes;
    static_assert(kGroups >= 1 && kWaves == kGroups * kKeySlots, "whole block groups");
    static_assert(kRW >= 2 && kRW <= 4 && kRW * kIPS <= 63, "ring slots");
};

template <int D>
__device__ __forceinline__ int k_swz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D>
__device__ __forceinline__ int v_swz(int r) { return D == 128 ? 2 * (r & 3) : 2 * ((r >> 1) & 1); }
// FP8 K rows (D bytes), read 16 rows at a time at one logical chunk
template <int D>
__device__ __forceinline__ int k8_swz(int r) { return D == 128 ? ((r ^ ((r >> 3) & 1)) & 7) : ((r >> 2) & 3); }

typedef int i32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ i32x8 cat8(u32x4 a, u32x4 b)
{
    return i32x8{(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)b[0], (int)b[1], (int)b[2], (int)b[3]};
}

// one wave-wide non-temporal global->LDS load of 1 KiB (every byte read once)
__device__ __forceinline__ void lds_dma_16(const void* gptr, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :
                 : "v"(gptr), "s"(lds_base)
                 : "memory", "m0");
}

// wait until at most n wave-wide loads of this wave are outstanding (n is
// rounded down to a multiple of 4: waiting longer is always safe)
__device__ __forceinline__ void wait_vm(int n)
{
    switch (n < 0 ? 0 : (n > 60 ? 60 : (n & ~3))) {
#define W(N) case N: __builtin_amdgcn_s_waitcnt(0xF70 | ((N) & 15) | ((((N) >> 4) & 3) << 14)); break;
        W(0) W(4) W(8) W(12) W(16) W(20) W(24) W(28) W(32) W(36) W(40) W(44) W(48) W(52) W(56) W(60)
#undef W
    default: __builtin_amdgcn_s_waitcnt(0xF70); break;
    }
    asm volatile("" ::: "memory");            // LDS written by the loads is read after this
}

// Rows of the workgroup: flat index f = r * G + h_local of its 16-row tile.
struct RowInfo {
    int f, r, h, kmax;
    bool ok;
};

__device__ __forceinline__ RowInfo row_info(const AttnParams& p, int tile, int g, int c16)
{
    const int G = p.Hq / p.Hkv;
    const int flat = p.Sq * G;
    RowInfo ri;
    ri.f = tile * kRows + c16;
    ri.ok = ri.f < flat;
    ri.r = ri.ok ? ri.f / G : 0;
    ri.h = g * G + (ri.ok ? ri.f % G : 0);
    ri.kmax = ri.ok ? (p.causal ? min(p.Sk - 1, ri.r + (p.Sk - p.Sq)) : p.Sk - 1) : -1;
    return ri;
}

// ---------------------------------------------------------------------------
// 1. scores: acc and block maxima of one key split
// ---------------------------------------------------------------------------
template <int D, int BLK, bool F8, int RT, int W>
__global__ __launch_bounds__(64 * W, 2) void split_scores_kernel(SplitParams sp)
{
    using C = SCfg<D, BLK, W>;
    constexpr int NW = C::kWaves, KW = C::kKeySlots, BG = C::kGroups;
    constexpr int RW = C::kRW;
    constexpr int kDK = D / 32;
    constexpr int kTR = RT * kRows;              // rows of the workgroup
    // row maxima of this wave's keys of every block of the split; the waves
    // meet once, after the last block
    __shared__ float wmax[kSplitMaxBps / RT][KW][kTR];
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    const uint32_t ring_lds = (uint32_t)(uintptr_t)LDS_PTR(char, ring);
    const AttnParams& p = sp.a;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave % KW, bg0 = wave / KW;    // key slot and block group of this wave
    const int c16 = lane & 15;
    const int grp = lane >> 4;
    const int split = blockIdx.x % sp.nsplit;
    const int tile = blockIdx.x / sp.nsplit;
    const int g = blockIdx.y;
    const int b = blockIdx.z;
    const int flat = p.Sq * (p.Hq / p.Hkv);
    const long long bg = (long long)b * p.Hkv + g;
    const uint16_t* kbase = p.k + bg * (long long)p.Sk * D;
    const uint8_t* kbase8 = reinterpret_cast<const uint8_t*>(p.k) + bg * (long long)p.Sk * D;
    const int j0 = split * sp.bps;
    const int j1 = min(sp.nblk, j0 + sp.bps);
    const int nslots = max(0, j1 - j0);                  // blocks of the split, and of this wave
    const int mine = max(0, (nslots - bg0 + BG - 1) / BG);
    constexpr int kIPS = F8 ? kSlotKeys * D / 1024 : C::kIPS;     // loads per slot (FP8 K: rows of D bytes)

    const uint32_t my_ring_lds = ring_lds + (uint32_t)(wave * RW * C::kSlotBytes);
    const char* my_ring = ring + wave * RW * C::kSlotBytes;
    auto issue_slot = [&](int n) {               // K keys [32*kw, +32) of this wave's n-th block
        const int key0 = (j0 + bg0 + BG * n) * BLK + kw * kSlotKeys;
        const uint32_t dst = my_ring_lds + (uint32_t)((n % RW) * C::kSlotBytes);
        if constexpr (F8) {
#pragma unroll
            for (int t = 0; t < kIPS; ++t) {
                const int rr = t * (1024 / D) + lane / (D / 16);
                const int ch = (lane % (D / 16)) ^ k8_swz<D>(rr);
                const int key = min(key0 + rr, p.Sk - 1);
                lds_dma_16(kbase8 + (long long)key * D + ch * 16, dst + t * 1024);
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < C::kIPS; ++t) {
            const int rr = t * (1024 / C::kRowBytes) + lane / C::kCPR;
            const int ch = (lane % C::kCPR) ^ k_swz<D>(rr);
            const int key = min(key0 + rr, p.Sk - 1);
            lds_dma_16(kbase + (long long)key * D + ch * 8, dst + t * 1024);
        }
    };
    int issued = 0;
    for (; issued < min(mine, RW); ++issued) issue_slot(issued);

    RowInfo ri[RT];
    int kmax_lo = 0x7fffffff;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        ri[rt] = row_info(p, tile * RT + rt, g, c16);
        if (ri[rt].ok) kmax_lo = min(kmax_lo, ri[rt].kmax);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) kmax_lo = min(kmax_lo, __shfl_xor(kmax_lo, o, 64));
    kmax_lo = __builtin_amdgcn_readfirstlane(kmax_lo);
    u32x4 qop[RT][F8 ? 1 : kDK];
    i32x8 qop8[RT] = {};                          // FP8: Q[row][32*grp .. +32], zeros past D
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const long long qoff = (((long long)b * p.Hq + ri[rt].h) * p.Sq + ri[rt].r) * D;
        if constexpr (F8) {
            const uint8_t* qrow = reinterpret_cast<const uint8_t*>(p.q) + qoff;
            if (ri[rt].ok && 32 * grp < D)
                qop8[rt] = cat8(*reinterpret_cast<const u32x4*>(qrow + 32 * grp),
                                *reinterpret_cast<const u32x4*>(qrow + 32 * grp + 16));
        } else {
            const uint16_t* qrow = p.q + qoff;
#pragma unroll
            for (int kk = 0; kk < kDK; ++kk)
                qop[rt][kk] = ri[rt].ok ? *reinterpret_cast<const u32x4*>(qrow + kk * 32 + grp * 8) : u32x4{0, 0, 0, 0};
        }
    }
    const float ninf = -__builtin_huge_valf();
    const int kx = k_swz<D>(c16);
    const uint32_t krow = c16 * C::kRowBytes;
    const long long nkeys = (long long)sp.nblk * BLK;
    const long long row0 = bg * flat + (long long)tile * kTR;    // the workgroup's first row
    float* acc_row[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc_row[rt] = sp.acc + (bg * flat + (ri[rt].ok ? ri[rt].f : 0)) * nkeys;

    for (int n = 0; n < mine; ++n) {
        const int nb = bg0 + BG * n;              // block of the split
        const int key0 = (j0 + nb) * BLK + kw * kSlotKeys;
        f32x4 sacc[RT][2];
        wait_vm((issued - 1 - n) * kIPS);
        const char* slot = my_ring + (n % RW) * C::kSlotBytes;
        if constexpr (F8) {
            const int kx8 = k8_swz<D>(c16);
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                i32x8 a8 = {};
                if (32 * grp < D) {
                    const char* kr = slot + (16 * t2 + c16) * D;
                    a8 = cat8(*reinterpret_cast<const u32x4*>(kr + 16 * ((2 * grp) ^ kx8)),
                              *reinterpret_cast<const u32x4*>(kr + 16 * ((2 * grp + 1) ^ kx8)));
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    sacc[rt][t2] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, qop8[rt], f32x4{}, 0, 0, 0, 127, 0, 127);
            }
        } else {
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) sacc[rt][t2] = f32x4{};
#pragma unroll
                for (int kk = 0; kk < kDK; ++kk) {
                    const u32x4 a = *reinterpret_cast<const u32x4*>(
                        slot + krow + t2 * 16 * C::kRowBytes + 16 * ((4 * kk + grp) ^ kx));
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        sacc[rt][t2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(qop[rt][kk]),
                                                                              sacc[rt][t2], 0, 0, 0);
                }
            }
        }
        // one block group: its waves stay on one block, whose rows are neighbours
        // in memory (D = 128, block 128, 268 MB of K and V: 0.5 us of 24)
        if constexpr (BG == 1 && KW > 1 && D == 128) __builtin_amdgcn_s_barrier();
        if (issued < mine) { issue_slot(issued); ++issued; }
        // mask keys past kmax; register i of tile t2 holds key key0 + 16*t2 + 4*grp + i
        if (key0 + kSlotKeys - 1 > kmax_lo) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int lim = ri[rt].kmax - key0 - 4 * grp;
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (16 * t2 + i > lim) sacc[rt][t2][i] = ninf;
            }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if (ri[rt].ok) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2)
                    *reinterpret_cast<f32x4*>(acc_row[rt] + key0 + 16 * t2 + 4 * grp) = sacc[rt][t2];
            }
            const f32x4 *s0 = &sacc[rt][0], *s1 = &sacc[rt][1];
            float pm = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf((*s0)[0], (*s0)[1]), (*s0)[2]),
                                       __builtin_fmaxf(__builtin_fmaxf((*s0)[3], (*s1)[0]), (*s1)[1]));
            pm = __builtin_fmaxf(pm, __builtin_fmaxf((*s1)[2], (*s1)[3]));
            pm = __builtin_fmaxf(pm, __shfl_xor(pm, 16, 64));
            pm = __builtin_fmaxf(pm, __shfl_xor(pm, 32, 64));
            if (grp == 0) wmax[nb][kw][rt * kRows + c16] = pm;
        }
    }
    __syncthreads();
    const int nr = min(kTR, flat - tile * kTR);
    for (int i = tid; i < nr * nslots; i += 64 * NW) {
        const int row = i / nslots, n = i - row * nslots;
        float m = wmax[n][0][row];
#pragma unroll
        for (int w = 1; w < KW; ++w) m = __builtin_fmaxf(m, wmax[n][w][row]);
        sp.bmax[(row0 + row) * sp.bstride + j0 + n] = m;
    }
}

// ---------------------------------------------------------------------------
// 2. pv: Alg. 1's per-block decisions up to the split, then P V of the split
// ---------------------------------------------------------------------------
constexpr int kWinFloats = 256;      // block maxima per LDS window of the replay

// RT tiles of 16 rows per workgroup share every V (and, in the scores pass, K) read.
template <int D, int BLK, int RT, int W>
__global__ __launch_bounds__(64 * W, 2) void split_pv_kernel(SplitParams sp)
{
    using C = SCfg<D, BLK, W>;
    constexpr int NW = C::kWaves, KW = C::kKeySlots, BG = C::kGroups;
    constexpr int RW = C::kRW;
    constexpr int kDT = D / 16;
    constexpr int NT = 64 * NW;
    constexpr int PS = D + 4;                     // floats per partial: X, dX, reference, two spare
    constexpr int kTR = RT * kRows;              // rows of the workgroup
    constexpr int kMaxBps = kSplitMaxBps / RT;
    // The ring carries the split's raw dot products beside V: one slot holds
    // those of kRun blocks (32 keys x kTR rows x 4 B per block and wave), in
    // front of the V slots of the same blocks.
    constexpr int kAccBytes = kSlotKeys * kTR * 4;
    constexpr int kRun = C::kSlotBytes / kAccBytes;
    static_assert(kRun >= 1 && kRun * kAccBytes == C::kSlotBytes, "a slot holds whole blocks of dot products");
    __shared__ __attribute__((aligned(1024))) uint8_t ctab[kCodeTableBytes];   // entry i at [i - kCodeLo]
    __shared__ unsigned s_cnt[kTR][2];
    constexpr int kWinBufs = 2;                   // windows in flight per wave
    __shared__ __attribute__((aligned(1024))) float s_win[NW][kWinBufs][kWinFloats];
    __shared__ float refs_l[kTR * kMaxBps];                                          // block references
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    const uint32_t ring_lds = (uint32_t)(uintptr_t)LDS_PTR(char, ring);
    const AttnParams& p = sp.a;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave % KW, bg0 = wave / KW;    // key slot and block group of this wave
    const int c16 = lane & 15;
    const int grp = lane >> 4;
    const int split = blockIdx.x % sp.nsplit;
    const int tile = blockIdx.x / sp.nsplit;
    const int g = blockIdx.y;
    const int b = blockIdx.z;
    const int flat = p.Sq * (p.Hq / p.Hkv);
    const long long bg = (long long)b * p.Hkv + g;
    const uint16_t* vbase = p.v + bg * (long long)p.Sk * D;
    const int j0 = split * sp.bps;
    const int j1 = min(sp.nblk, j0 + sp.bps);
    const int nslots = max(0, j1 - j0);
    const float ninf = -__builtin_huge_valf();
    const float c = p.c;

    // -- block-maximum windows of the replay: a wave replays RPW rows at a
    //    time, L = 64/RPW lanes per row, and one wave-wide 1 KiB DMA brings the
    //    maxima of 4 L blocks of each of them
    const int nr = min(kTR, flat - tile * kTR);             // rows of the workgroup (at least one)
    const int rpw = nr <= NW ? 1 : (nr <= 2 * NW ? 2 : 4);
    const int npass = (nr + NW * rpw - 1) / (NW * rpw);
    const int wblk = kWinFloats / rpw;                       // blocks per window and row
    const int nwin = (j1 + wblk - 1) / wblk;
    const int nall = npass * nwin;                           // windows of this wave, pass by pass
    const uint32_t win_lds = (uint32_t)(uintptr_t)LDS_PTR(float, &s_win[wave][0][0]);
    int ndma = 0;                                 // DMA ops of this wave issued so far
    {
        const uint32_t ctab_lds = (uint32_t)(uintptr_t)LDS_PTR(uint8_t, ctab);
        for (int i = wave; i < kCodeTableBytes / 1024; i += NW) {
            lds_dma_16(p.ctab + i * 1024 + 16 * lane, ctab_lds + (uint32_t)(i * 1024));
            ++ndma;
        }
    }
    const int tagc = ndma;                        // ndma after this wave's part of the code table
    auto issue_win = [&](int i) {
        const int lpr = 64 / rpw;
        const int srow = min((i / nwin * NW + wave) * rpw + lane / lpr, nr - 1);
        const float* src = sp.bmax + (bg * flat + tile * kTR + srow) * sp.bstride + (i % nwin) * wblk + 4 * (lane % lpr);
        lds_dma_16(src, win_lds + (uint32_t)((i % kWinBufs) * 1024));
        ++ndma;
    };
    const int nearly = min(nall, kWinBufs);       // windows issued ahead of the V ring
    for (int i = 0; i < nearly; ++i) issue_win(i);

    // -- the ring of this wave (blocks bg0 + BG*i of the split): slot q holds
    //    the raw dot products of run q / (kRun + 1) (q % (kRun + 1) == 0) or V
    //    of one block of that run
    const int mine = max(0, (nslots - bg0 + BG - 1) / BG);
    const long long nkeys = (long long)sp.nblk * BLK;
    const long long row0 = bg * flat + (long long)tile * kTR;    // the workgroup's first row
    const uint32_t my_ring_lds = ring_lds + (uint32_t)(wave * RW * C::kSlotBytes);
    const char* my_ring = ring + wave * RW * C::kSlotBytes;
    const int nrg = min(kTR / 8, (nr + 7) / 8);              // groups of 8 rows with a row
    uint64_t tags = 0;                            // ndma after each of the last four slots, the latest lowest
    auto issue_slot = [&](int q) {               // keys [32*kw, +32) of the blocks
        const int run = q / (kRun + 1), u = q % (kRun + 1);
        const uint32_t dst = my_ring_lds + (uint32_t)((q % RW) * C::kSlotBytes);
        if (u == 0) {
            // 8 rows of 128 B per load; the 16-byte chunks of a row XOR-swizzled
#pragma unroll
            for (int t = 0; t < C::kIPS; ++t) {
                if (run * kRun + t / (kTR / 8) >= mine) break;   // (the last run may hold fewer blocks)
                if (t % (kTR / 8) >= nrg) continue;
                const int n = bg0 + BG * (run * kRun + t / (kTR / 8));
                const int rr = (t % (kTR / 8)) * 8 + lane / 8;
                const int ch = (lane % 8) ^ (rr & 7);
                lds_dma_16(sp.acc + (row0 + min(rr, nr - 1)) * nkeys + (j0 + n) * BLK + kw * kSlotKeys + 4 * ch,
                           dst + t * 1024);
                ++ndma;
            }
        } else {
            const int key0 = (j0 + bg0 + BG * (run * kRun + u - 1)) * BLK + kw * kSlotKeys;
#pragma unroll
            for (int t = 0; t < C::kIPS; ++t) {
                const int rr = t * (1024 / C::kRowBytes) + lane / C::kCPR;
                const int ch = (lane % C::kCPR) ^ v_swz<D>(rr);
                const int key = min(key0 + rr, p.Sk - 1);
                lds_dma_16(vbase + (long long)key * D + ch * 8, dst + t * 1024);
            }
            ndma += C::kIPS;
        }
        tags = tags << 16 | (uint16_t)ndma;
    };
    const int nseq = mine + (mine + kRun - 1) / kRun;
    int issued = 0;
    for (; issued < min(nseq, RW); ++issued) issue_slot(issued);

    // -- the replay: Alg. 1's decision for every block of [0, j1) of a row, L
    //    blocks (one per lane) per step.  The integer maximum is nearly always
    //    the running maximum of the blocks' own ceil(row maximum): every lane
    //    takes that as its guess of m before its block (a prefix maximum),
    //    applies the rule of Alg. 1 to it, and the blocks up to the first one
    //    whose result is not the next lane's guess are settled; the step
    //    repeats from there with the true m.  This runs in front of P V, so it
    //    is kept short: up to four rows share a wave where there are more rows
    //    than waves (6 queries of 4 heads on 3000 keys, 4 sequences, kernel
    //    time: 33 us with a row per wave at a time and a step per change of m,
    //    18.8 us with four rows per wave, 11.4 us with eight waves and the
    //    prefix maximum).
    const int tagv = ndma;                        // ndma after the V ring's first loads
    auto wait_win = [&](int i) { wait_vm(ndma - (i < nearly ? tagc + i + 1 : tagv + (i - nearly) + 1)); };
    const float* win = &s_win[wave][0][0];
    const float x_still = p.dec_x0 > 0.0f ? 0.0f : ninf;   // (lambda < 0 restarts below m as well)
    auto replay = [&](auto rows_per_wave) {
        constexpr int RPW = decltype(rows_per_wave)::value;
        constexpr int L = 64 / RPW, kWB = kWinFloats / RPW;
        const int sl = lane % L, sg = lane / L;   // this lane's block of the step, and its row
        for (int pass = 0; pass < npass; ++pass) {
            const int srow = (pass * NW + wave) * RPW + sg;
            const bool row_ok = srow < nr;
            const int last_blk = row_ok ? row_info(p, tile * RT + srow / kRows, g, srow % kRows).kmax / BLK : -1;   // B0 with b0_last
            float m = ninf;
            unsigned n_restart = 0, n_visit = 0;
            for (int w = 0; w < nwin; ++w) {
                const int i = pass * nwin + w;
                wait_win(i);
                const float* wl = win + (i % kWinBufs) * kWinFloats + sg * kWB;
#pragma unroll 1
                for (int kk = 0; kk < kWB / L; ++kk) {
                    const int cb = w * kWB + L * kk;
                    if (cb >= j1) break;
                    const int jb = cb + sl;
                    float amax = wl[L * kk + sl];
                    if (!(row_ok && jb < j1)) amax = ninf;
                    const bool vis = amax != ninf;
                    const float ceil_ac = ceilf(amax * c);
                    const bool in_b0 = jb < p.n_b0 || (p.b0_last && jb == last_blk);
                    const bool in_split = row_ok && jb >= j0 && jb < j1;
                    // no block above m (nearly every step of a long row): none
                    // restarts or moves it, and m is the reference of them all
                    // (131072 keys, block 128: 109.1 -> 106.4 us a call; 32
                    // rows gain less, and 0.25 us of 28.3 is lost on 24 blocks)
                    if constexpr (RT == 1) {
                        if (!__any(vis && !(__builtin_fmaf(amax, c, -m) <= x_still))) {
                            if (in_split) {
                                refs_l[srow * kMaxBps + (jb - j0)] = vis ? m : ninf;
                                n_visit += vis && !in_b0 ? 1u : 0u;
                            }
                            continue;
                        }
                    }
                    const float h = vis ? ceil_ac : ninf;
                    int lo = 0;
                    for (;;) {
                        // (the restart test and the increment as in the
                        // prefill kernel: lambda <= kCodeMaxLambda here)
                        const float g = __builtin_fmaxf(m, prefix_max_before<L>(sl >= lo ? h : ninf));
                        const bool forced = in_b0 || (g == ninf);
                        const float xt = __builtin_fmaf(amax, c, -g);
                        const bool restart = forced || (xt >= p.dec_x0);
                        const float m_hi = __builtin_fmaxf(g, ceil_ac);
                        const float m_new = vis ? (restart ? m_hi : g + hif8_ceil_below9(xt)) : g;
                        const float ref_new = vis ? (restart ? m_hi : g) : ninf;
                        const bool pend = sl >= lo;
                        const unsigned long long bal = __ballot(pend && m_new != __builtin_fmaxf(g, h));
                        const unsigned long long gb = RPW == 1 ? bal : (bal >> (sg * L)) & ((1ull << (L & 63)) - 1);
                        const int f = gb ? (int)__builtin_ctzll(gb) : L - 1;   // this row's last settled block
                        if (pend && sl <= f && in_split) {
                            refs_l[srow * kMaxBps + (jb - j0)] = ref_new;   // -inf: no visible key
                            const bool b1 = vis && !in_b0;
                            n_visit += b1 ? 1u : 0u;
                            n_restart += (b1 && restart) ? 1u : 0u;
                        }
                        // (a row whose step is done has lo = L: its lanes hold
                        // g = m, and m stays)
                        const float at = __shfl(m_new, sg * L + f, 64);
                        m = lo < L ? at : m;
                        lo = f + 1;
                        if (!__any(lo < L)) break;
                    }
                }
                if (i + kWinBufs < nall) issue_win(i + kWinBufs);
            }
#pragma unroll
            for (int o = 1; o < L; o <<= 1) {
                n_visit += __shfl_xor(n_visit, o, 64);
                n_restart += __shfl_xor(n_restart, o, 64);
            }
            if (sl == 0 && row_ok) {
                s_cnt[srow][0] = n_restart;
                s_cnt[srow][1] = n_visit;
            }
        }
    };
    if (rpw == 1) replay(std::integral_constant<int, 1>{});
    else if (rpw == 2) replay(std::integral_constant<int, 2>{});
    else replay(std::integral_constant<int, 4>{});
    wait_vm(ndma - tagc);                         // this wave's part of the code table has landed

    bool ok[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) ok[rt] = rt * kRows + c16 < nr;
    float cur[RT], dl[RT];                        // X and dX are relative to the reference cur
    f32x4 oacc[RT][kDT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        cur[rt] = ninf;
        dl[rt] = 0.0f;
#pragma unroll
        for (int t = 0; t < kDT; ++t) oacc[rt][t] = f32x4{};
    }
    const int vrow0 = 4 * grp + c16 / 4;
    const int vx = v_swz<D>(vrow0);
    const int vd0 = 4 * (c16 & 3);
    const uint32_t vrow = vrow0 * C::kRowBytes + 2 * (vd0 & 7);
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    __syncthreads();                              // code table, references and counts published

    int q = 0;                                    // ring slot to consume next
    auto wait_slot = [&]() {
        wait_vm((uint16_t)(ndma - (int)(tags >> 16 * (issued - 1 - q))));
    };
    auto next_slot = [&]() {
        if (issued < nseq) { issue_slot(issued); ++issued; }
        ++q;
    };
    for (int n0 = 0; n0 < mine; n0 += kRun) {
        // P of the run's blocks from their dot products and references (the
        // partials follow the references with exact rescales), all ahead of
        // their P V: the dot products landed in front of V, so this overlaps
        // V's way from memory
        float fac[kRun][RT];
        u32x4 pop[kRun][RT];
        f32x4 sacc[kRun][RT][2];
        wait_slot();
        const char* aslot = my_ring + (q % RW) * C::kSlotBytes;
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
            if (n0 + u >= mine) break;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    const int row = rt * kRows + c16;
                    sacc[u][rt][t2] = *reinterpret_cast<const f32x4*>(aslot + u * kAccBytes + row * 128 + 16 * ((4 * t2 + grp) ^ (row & 7)));
                }
        }
        // the slot goes back as soon as it is read: V streams on behind the
        // gathers (4 sequences on 16384 keys, block 128: 26.4 -> 25.2 us)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        next_slot();
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
            if (n0 + u >= mine) break;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int row = rt * kRows + c16;
                const float rj = ok[rt] ? refs_l[row * kMaxBps + bg0 + BG * (n0 + u)] : ninf;
                fac[u][rt] = (cur[rt] == ninf || rj == ninf) ? 1.0f : exp2_int(cur[rt] - rj);
                dl[rt] *= fac[u][rt];
                if (rj != ninf) cur[rt] = rj;
                const float nref = (cur[rt] == ninf) ? 0.0f : -cur[rt];
                if (!ok[rt]) sacc[u][rt][0] = sacc[u][rt][1] = f32x4{ninf, ninf, ninf, ninf};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int t2 = e >> 1;
                    const float t0 = __builtin_fmaf(sacc[u][rt][t2][2 * (e & 1)], c, nref);
                    const float t1 = __builtin_fmaf(sacc[u][rt][t2][2 * (e & 1) + 1], c, nref);
                    const uint32_t i0 = min(max(hif8::f2u(t0) >> kTabShift, (uint32_t)kCodeLo), (uint32_t)kCodeHi);
                    const uint32_t i1 = min(max(hif8::f2u(t1) >> kTabShift, (uint32_t)kCodeLo), (uint32_t)kCodeHi);
                    const uint32_t w = ((uint32_t)ctab[i0 - kCodeLo] | ((uint32_t)ctab[i1 - kCodeLo] << 16)) << 4;
                    pop[u][rt][e] = w;
                    dl[rt] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, dl[rt], false);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
            if (n0 + u >= mine) break;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                if (__any(fac[u][rt] != 1.0f)) {
#pragma unroll
                    for (int t = 0; t < kDT; ++t)
#pragma unroll
                        for (int i = 0; i < 4; ++i) oacc[rt][t][i] *= fac[u][rt];
                }
            wait_slot();
            const char* slot = my_ring + (q % RW) * C::kSlotBytes;
            // (every operand read of the block ahead of its MFMAs)
            u32x4 va[kDT];
#pragma unroll
            for (int t = 0; t < kDT; ++t) {
                const char* pa = slot + vrow + 16 * (((16 * t + vd0) >> 3) ^ vx);
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, pa));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, pa + 16 * C::kRowBytes));
                va[t] = u32x4{__builtin_bit_cast(u32x2, lo)[0], __builtin_bit_cast(u32x2, lo)[1],
                              __builtin_bit_cast(u32x2, hi)[0], __builtin_bit_cast(u32x2, hi)[1]};
            }
#pragma unroll
            for (int t = 0; t < kDT; ++t)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    oacc[rt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va[t]), as_bf16x8(pop[u][rt]), oacc[rt][t], 0, 0, 0);
            next_slot();
        }
    }

    // -- one sum over the waves through the ring (chunks of 4 values of d
    //    swizzled by row), the block groups brought to the latest reference of
    //    the row; this split's partial: X, dX and that reference
    constexpr int QD = D / 4;                     // chunks per row
    static_assert(C::kLdsBytes >= NW * kTR * D * 4, "merge buffer fits the ring");
    static_assert(sizeof(float) * (NW + BG) * kTR <= sizeof(s_win), "denominators and references fit the windows");
    f32x4* mb = reinterpret_cast<f32x4*>(ring);                  // [NW][kTR][QD]
    float* db = &s_win[0][0][0];                                 // [NW][kTR], then the references [BG][kTR]
    float* rb = db + NW * kTR;
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int row = rt * kRows + c16;
#pragma unroll
        for (int t = 0; t < kDT; ++t) mb[(wave * kTR + row) * QD + ((4 * t + grp) ^ (c16 & (QD - 1)))] = oacc[rt][t];
        float dw = dl[rt] + __shfl_xor(dl[rt], 16, 64);
        dw += __shfl_xor(dw, 32, 64);
        if (grp == 0) db[wave * kTR + row] = dw;
        if (grp == 0 && kw == 0) rb[bg0 * kTR + row] = cur[rt];
    }
    __syncthreads();
    float* prow0 = sp.part + split * ((long long)p.B * p.Hkv * flat * PS) + row0 * PS;
    for (int i = tid; i < nr * QD; i += NT) {
        const int row = i / QD, ch = i % QD;
        float top = rb[row];
#pragma unroll
        for (int g2 = 1; g2 < BG; ++g2) top = __builtin_fmaxf(top, rb[g2 * kTR + row]);
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
        float d = 0.0f;
#pragma unroll
        for (int g2 = 0; g2 < BG; ++g2) {
            f32x4 y = mb[(g2 * KW * kTR + row) * QD + (ch ^ (row & 15 & (QD - 1)))];
            float e1 = db[g2 * KW * kTR + row];
#pragma unroll
            for (int w = 1; w < KW; ++w) {
                const f32x4 z = mb[((g2 * KW + w) * kTR + row) * QD + (ch ^ (row & 15 & (QD - 1)))];
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] += z[e];
                e1 += db[(g2 * KW + w) * kTR + row];
            }
            // (a group that saw no key adds nothing)
            const float rg = rb[g2 * kTR + row];
            const float f = rg == ninf ? 0.0f : exp2_int(rg - top);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] += f * y[e];
            d += f * e1;
        }
        *reinterpret_cast<f32x4*>(prow0 + row * PS + 4 * ch) = x;
        if (ch == 0) {
            prow0[row * PS + D] = d;
            prow0[row * PS + D + 1] = top;
        }
    }
    // restart counters of this split's blocks (a tile is one row here)
    if (tid < nr) {
        const RowInfo cr = row_info(p, tile * RT + tid / kRows, g, tid % kRows);
        if (s_cnt[tid][1]) {
            if (p.counters) {
                unsigned long long* cp = p.counters + 2 * ((long long)b * p.Hq + cr.h);
                atomicAdd(cp + 0, (unsigned long long)s_cnt[tid][0]);
                atomicAdd(cp + 1, (unsigned long long)s_cnt[tid][1]);
            }
            if (p.tile_counts) {
                unsigned long long* tc = p.tile_counts + 2 * (((long long)b * p.Hq + cr.h) * p.Sq + cr.r);
                atomicAdd(tc + 0, (unsigned long long)s_cnt[tid][0]);
                atomicAdd(tc + 1, (unsigned long long)s_cnt[tid][1]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 3. combine: one workgroup per row; groups of threads take every SG-th split
//    of 4 values of d each, and their sums meet in LDS
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void split_combine_kernel(SplitParams sp)
{
    constexpr int QD = D / 4;                     // threads per split group (4 values of d each)
    constexpr int SG = 256 / QD;                  // split groups
    constexpr int PS = D + 4;
    constexpr int kU = 8;                         // splits in flight per thread
    __shared__ float red[256][6];
    const AttnParams& p = sp.a;
    const int tid = threadIdx.x;
    const int q4 = tid % QD;
    const int sg = tid / QD;
    const int f = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    const int G = p.Hq / p.Hkv;
    const int flat = p.Sq * G;
    const long long row = ((long long)b * p.Hkv + g) * flat + f;
    const long long pstride = (long long)p.B * p.Hkv * flat * PS;
    const float* pcol = sp.part + row * PS;
    const float ninf = -__builtin_huge_valf();
    float rr = ninf, dx = 0.0f;
    f32x4 xs = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = sg; s0 < sp.nsplit; s0 += kU * SG) {
        float rv[kU], dv[kU];
        f32x4 xv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {           // straight-line loads (a clamped split, masked below)
            const float* prow = pcol + min(s0 + u * SG, sp.nsplit - 1) * pstride;
            xv[u] = *reinterpret_cast<const f32x4*>(prow + 4 * q4);
            dv[u] = prow[D];
            rv[u] = prow[D + 1];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (s0 + u * SG >= sp.nsplit) rv[u] = ninf;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (rv[u] == ninf) continue;          // no visible key in that split
            if (rv[u] > rr) {
                const float fa = exp2_int(rr - rv[u]);   // 0 while rr is -inf (nothing summed yet)
#pragma unroll
                for (int e = 0; e < 4; ++e) xs[e] *= fa;
                dx *= fa;
                rr = rv[u];
            }
            const float fb = exp2_int(rv[u] - rr);
#pragma unroll
            for (int e = 0; e < 4; ++e) xs[e] += fb * xv[u][e];
            dx += fb * dv[u];
        }
    }
    red[tid][0] = rr;
    red[tid][1] = dx;
    red[tid][2] = xs[0];
    red[tid][3] = xs[1];
    red[tid][4] = xs[2];
    red[tid][5] = xs[3];
    __syncthreads();
    if (sg != 0) return;
    for (int o = 1; o < SG; ++o) {
        const float* th = red[tid + o * QD];
        const float r2 = th[0];
        if (r2 == ninf) continue;
        const float top = __builtin_fmaxf(rr, r2);
        const float fa = (rr == ninf) ? 0.0f : exp2_int(rr - top);
        const float fb = exp2_int(r2 - top);
        dx = dx * fa + th[1] * fb;
#pragma unroll
        for (int e = 0; e < 4; ++e) xs[e] = xs[e] * fa + th[2 + e] * fb;
        rr = top;
    }
    const int r = f / G;
    const int h = g * G + f % G;
    const bool empty = rr == ninf;
    const float inv = empty ? 0.0f : 1.0f / dx;
    const long long orow_off = (((long long)b * p.Hq + h) * p.Sq + r) * D + 4 * q4;
    if (p.out_bf16) {
        typedef __bf16 bf16x2 __attribute__((__vector_size__(2 * sizeof(__bf16))));
        const bf16x2 lo = {(__bf16)(xs[0] * inv), (__bf16)(xs[1] * inv)};
        const bf16x2 hi = {(__bf16)(xs[2] * inv), (__bf16)(xs[3] * inv)};
        *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(p.o) + orow_off) =
            u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    } else {
        *reinterpret_cast<f32x4*>(p.o + orow_off) = f32x4{xs[0] * inv, xs[1] * inv, xs[2] * inv, xs[3] * inv};
    }
    if (q4 == 0 && p.lse)
        p.lse[((long long)b * p.Hq + h) * p.Sq + r] =
            empty ? ninf : 0.69314718055994531f * (rr + (log2f(dx) + (float)kCodeBiasLog2));
}

template <int D, int BLK, int RT, int W>
hipError_t launch_split_waves(const SplitParams& sp, hipStream_t st)
{
    using C = SCfg<D, BLK, W>;
    static DeviceOnce attr_set;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (!attr_set.is_done(dev)) {
        const void* fns[] = {reinterpret_cast<const void*>(&split_scores_kernel<D, BLK, false, RT, W>),
                             reinterpret_cast<const void*>(&split_scores_kernel<D, BLK, true, RT, W>),
                             reinterpret_cast<const void*>(&split_pv_kernel<D, BLK, RT, W>)};
        for (const void* fn : fns) {
            e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
            if (e != hipSuccess) return e;
        }
        attr_set.mark(dev);
    }
    const AttnParams& p = sp.a;
    const long long flat = (long long)p.Sq * (p.Hq / p.Hkv);
    const unsigned tiles = (unsigned)((flat + RT * kRows - 1) / (RT * kRows));
    const dim3 grid(tiles * (unsigned)sp.nsplit, (unsigned)p.Hkv, (unsigned)p.B), block(64 * C::kWaves);
    if (p.qk_f8) hipLaunchKernelGGL((split_scores_kernel<D, BLK, true, RT, W>), grid, block, C::kLdsBytes, st, sp);
    else hipLaunchKernelGGL((split_scores_kernel<D, BLK, false, RT, W>), grid, block, C::kLdsBytes, st, sp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((split_pv_kernel<D, BLK, RT, W>), grid, block, C::kLdsBytes, st, sp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((split_combine_kernel<D>), dim3((unsigned)flat, (unsigned)p.Hkv, (unsigned)p.B), dim3(256), 0,
                       st, sp);
    return hipGetLastError();
}

// The waves of a workgroup.  Where the grid holds at most one per CU, eight
// share the replay of the rows and hide each other's latency (32 rows: 1.03 to
// 1.2 times as fast as four over 1600 shapes).  16 rows on so few workgroups
// means that a split is a single block; then only many rows on many blocks give
// eight waves work (8 rows on 256 blocks: 19.6 us a call, with four waves 21.2;
// otherwise four are 2 % faster), and of blocks of 32 or 64 keys one group is
// enough for a row per wave (8 heads on 1500 keys, block 32: 17.0 us a call with
// four waves, 16.2 with one) or up to four rows on few blocks (16 heads on 130
// keys, block 32: 14.9 and 14.0; on many the replay takes longer on one group:
// 4 rows on 212 blocks of 64 21.1 and 21.6, of 32 21.2 and 24.6).
template <int D, int BLK, int RT>
hipError_t launch_split_rt(const SplitParams& sp, hipStream_t st)
{
    int ncu = 0;
    const hipError_t e = cu_count(&ncu);
    if (e != hipSuccess) return e;
    const AttnParams& p = sp.a;
    const long long flat = (long long)p.Sq * (p.Hq / p.Hkv);
    const long long wgs = (flat + RT * kRows - 1) / (RT * kRows) * sp.nsplit * p.Hkv * p.B;
    if (wgs <= ncu && (RT == 2 || (flat > 4 && sp.nblk >= 128))) return launch_split_waves<D, BLK, RT, 8>(sp, st);
    if constexpr (RT == 1 && BLK < 128) {
        constexpr int kFew = D == 64 && BLK == 64 ? 8 : 32;
        if (sp.bps == 1 && (flat <= BLK / kSlotKeys || (flat <= 4 && sp.nblk <= kFew)))
            return launch_split_waves<D, BLK, RT, BLK / kSlotKeys>(sp, st);
    }
    return launch_split_waves<D, BLK, RT, 4>(sp, st);
}

template <int D, int BLK>
hipError_t launch_split_db(const SplitParams& sp, hipStream_t st)
{
    const AttnParams& p = sp.a;
    if (sp.bps < 1 || sp.bps > kSplitMaxBps || sp.bstride % kWinFloats || sp.bstride < sp.nblk ||
        (long long)sp.nsplit * sp.bps < sp.nblk || (long long)(sp.nsplit - 1) * sp.bps >= sp.nblk)
        return hipErrorInvalidValue;
    // more than 16 rows per key/value head: 32 per workgroup, so that K and V
    // are streamed once for both tiles (8 sequences, 32 rows, 4000 keys: scores
    // 31.7 -> 20.9 us, pv 36.6 -> 23.5 us); the references of the split's
    // blocks then fit in LDS up to 16 blocks
    if ((long long)p.Sq * (p.Hq / p.Hkv) > kRows && sp.bps <= kSplitMaxBps / 2) return launch_split_rt<D, BLK, 2>(sp, st);
    return launch_split_rt<D, BLK, 1>(sp, st);
}

}  // namespace

hipError_t launch_attention_split(const SplitParams& sp, int D, int block, hipStream_t st)
{
    if (D == 64 && block == 32) return launch_split_db<64, 32>(sp, st);
    if (D == 64 && block == 64) return launch_split_db<64, 64>(sp, st);
    if (D == 64 && block == 128) return launch_split_db<64, 128>(sp, st);
    if (D == 128 && block == 32) return launch_split_db<128, 32>(sp, st);
    if (D == 128 && block == 64) return launch_split_db<128, 64>(sp, st);
    if (D == 128 && block == 128) return launch_split_db<128, 128>(sp, st);
    return hipErrorInvalidValue;
}

}  // namespace baps
