// The vector-side steps of Alg. 1 (block-aware precision rescaling) on fp32
// score rows that are already in log2 units: per key block, the row maximum,
// the restart decision of the B1 loop, the integer running maximum (Sec. 3.3),
// T = HiF8(S - ref), P = HiF8(2^T), and the running denominator.
//
// HBM-bound where rows fill the GPU: 4 B read and 1 B written per score.  The
// only sequential dependency is that the reference of block j depends on the
// running maximum after block j-1.  Three forms (launch_softmax_block picks):
// a wave per row that walks 1024 columns at a time (16 per lane,
// lane-interleaved so every load and store of the wave is contiguous; any
// alignment), four rows per wave, and a workgroup per row.
#include "common.hpp"

namespace baps {

namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = kThreads / 64;
constexpr int kChunk = 1024;               // columns per wave per step
constexpr int kPerLane = kChunk / 64;

template <int BLOCK>
__global__ __launch_bounds__(kThreads) void softmax_block_kernel(SoftmaxBlockParams p)
{
    __shared__ uint32_t tab[kTabEntries];
    for (int i = threadIdx.x; i < kTabEntries; i += kThreads) tab[i] = p.tab[i];
    __syncthreads();

    constexpr int kBPL = BLOCK / 64;                      // elements of a block per lane
    constexpr int kBlocksPerChunk = kChunk / BLOCK;
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    if (row >= p.rows) return;

    const long long cols = p.cols;
    const long long nblk = (cols + BLOCK - 1) / BLOCK;
    const float* S = p.s + row * p.ld;
    uint8_t* code = p.codes + row * cols;
    int32_t* refs_out = p.ref_shift + row * nblk;
    const float ninf = -__builtin_huge_valf();

    float m = ninf;            // running integer maximum m^(j)
    float dl = 0.0f;           // this lane's share of the denominator d^(j)
    float myref = ninf;        // reference of block (64*g + lane) of the current group
    long long j = 0;

    float cur[kPerLane], nxt[kPerLane];
    auto load = [&](float* v, long long c0) {
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            const long long c = c0 + lane + 64 * i;
            v[i] = c < cols ? __builtin_nontemporal_load(S + c) : ninf;
        }
    };
    load(cur, 0);
    for (long long c0 = 0; c0 < cols; c0 += kChunk) {
        if (c0 + kChunk < cols) load(nxt, c0 + kChunk);
#pragma unroll
        for (int b = 0; b < kBlocksPerChunk; ++b) {
            if (j >= nblk) break;
            float M = ninf;
#pragma unroll
            for (int t = 0; t < kBPL; ++t) M = fmaxf(M, cur[b * kBPL + t]);
            M = wave_max_uniform(M);

            // Alg. 1: B0 blocks always take the high-precision path; B1 blocks
            // test ceil(rowmax T) > lambda with T = S - m~ cast to 8 bits.
            // HiF8 rounding is monotone, so rowmax of the cast T is the cast
            // of (rowmax S) - m~.
            bool restart;
            float tq = ninf;
            if (j < p.n_b0) {
                restart = true;
            } else {
                if (M != ninf) tq = hif8::round(M - m);     // m = -inf gives +inf: restart
                restart = ceilf(tq) > (float)p.lambda;
            }
            float m_new, ref;
            if (restart) {
                m_new = fmaxf(m, ceilf(M));
                ref = m_new;
            } else {
                m_new = m + fmaxf(0.0f, ceilf(tq));
                ref = m;
            }
            const float alpha = (m == ninf) ? 0.0f : exp2_int(m - m_new);
            const float beta = (ref == ninf) ? 0.0f : exp2_int(ref - m_new);

            float rowsum = 0.0f;
#pragma unroll
            for (int t = 0; t < kBPL; ++t) {
                const float s = cur[b * kBPL + t];
                const float T = (s == ninf || ref == ninf) ? ninf : s - ref;
                const uint32_t e = tab[hif8::f2u(T) >> kTabShift];
                const long long c = c0 + (long long)b * BLOCK + lane + 64 * t;
                if (c < cols) code[c] = (uint8_t)(e & 0xffu);
                rowsum += hif8::u2f(e & 0xffffff00u);
            }
            dl = alpha * dl + beta * rowsum;
            m = m_new;
            if (p.restarted && lane == 0) p.restarted[row * nblk + j] = restart ? 1 : 0;
            if (lane == (int)(j & 63)) myref = ref;
            if ((j & 63) == 63 || j == nblk - 1) {
                if (nblk > 64) {            // park the group's references until m is final
                    const long long idx = (j & ~63LL) + lane;
                    if (idx < nblk) refs_out[idx] = (int32_t)hif8::f2u(myref);
                }
            }
            ++j;
        }
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) cur[i] = nxt[i];
    }

    const float d = wave_sum(dl);
    if (lane == 0) {
        p.m_final[row] = m;
        p.d_final[row] = d;
    }
    auto shift = [&](float ref) -> int32_t {
        if (ref == ninf || m == ninf) return INT32_MIN;
        return (int32_t)fmaxf(ref - m, -2147483520.0f);
    };
    if (nblk <= 64) {
        if (lane < nblk) refs_out[lane] = shift(myref);
    } else {
        for (long long idx = lane; idx < nblk; idx += 64)
            refs_out[idx] = shift(hif8::u2f((uint32_t)refs_out[idx]));
    }
}

// Row-group variant for 16-byte aligned rows whose length is a multiple of 4
// and blocks of at most 256 columns: a wave owns 4 rows and each row is a
// DPP row of 16 lanes, so the per-block maximum is 4 in-row DPP steps and the
// per-block state update runs for 4 rows at once.  A lane holds 4 adjacent
// columns per 64-column group: fp32x4 loads and 4-code stores, contiguous
// per row.
__device__ __forceinline__ float row16_max(float v)
{
    int o = __builtin_bit_cast(int, v);
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0xB1, 0xF, 0xF, false)));
    o = __builtin_bit_cast(int, v);
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0x4E, 0xF, 0xF, false)));
    o = __builtin_bit_cast(int, v);
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0x141, 0xF, 0xF, false)));
    o = __builtin_bit_cast(int, v);
    return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0x140, 0xF, 0xF, false)));
}

__device__ __forceinline__ float row16_sum(float v)
{
    int o = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0xB1, 0xF, 0xF, false));
    o = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0x4E, 0xF, 0xF, false));
    o = __builtin_bit_cast(int, v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0x141, 0xF, 0xF, false));
    o = __builtin_bit_cast(int, v);
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(o, o, 0x140, 0xF, 0xF, false));
}

constexpr int kRowsPerWave4 = 4;

// NT threads per workgroup, 4 rows per wave.  With rows enough to give every
// CU a workgroup, 1024 threads (64 rows, one workgroup and one 32 KiB table
// copy per CU) run about 10 % faster than 256 threads (four workgroups and
// four table copies per CU).  KCH columns of a row stream per step, and the
// next step's loads are in flight while one is processed.  256 columns keep
// the kernel at 64 VGPRs (8 waves per SIMD), which suits grids of many
// workgroups per CU and short rows; wider steps put more bytes in flight per
// wave where fewer waves share a CU: 512 columns (96 VGPRs) for rows of at
// least 4096 columns at 1024 threads (rows just behind a chunk of the wide
// form, and more blocks than it holds), 1024 columns (162 VGPRs) for grids of
// at most two 256-thread workgroups per CU.
template <int BLOCK, int NT, int KCH>
__global__ __launch_bounds__(NT) void softmax_block4_kernel(SoftmaxBlockParams p)
{
    constexpr int kRows4PerBlock = kRowsPerWave4 * (NT / 64);
    __shared__ uint32_t tab[kTabEntries];
    for (int i = threadIdx.x; i < kTabEntries; i += NT) tab[i] = p.tab[i];
    __syncthreads();

    constexpr int kCh = BLOCK < KCH ? KCH : BLOCK;        // columns per row per step
    constexpr int kG = kCh / 64;                          // fp32x4 groups per lane per step
    constexpr int kGPB = BLOCK / 64;                      // groups per block (>= 1)
    constexpr int kBPS = kCh / BLOCK;                     // blocks per step
    const int lane = threadIdx.x & 63;
    const int sub = lane & 15;
    const long long row = (long long)blockIdx.x * kRows4PerBlock + (threadIdx.x >> 6) * kRowsPerWave4 + (lane >> 4);
    const bool row_ok = row < p.rows;                     // whole DPP rows agree
    const long long rr = row_ok ? row : 0;

    const long long cols = p.cols;
    const long long nblk = (cols + BLOCK - 1) / BLOCK;
    const float* S = p.s + rr * p.ld;
    uint8_t* code = p.codes + rr * cols;
    int32_t* refs_out = p.ref_shift + rr * nblk;
    const float ninf = -__builtin_huge_valf();

    float m = ninf, dl = 0.0f, myref = ninf;
    long long j = 0;
    f32x4 cur[kG], nxt[kG];
    auto load = [&](f32x4* v, long long c0) {
#pragma unroll
        for (int i = 0; i < kG; ++i) {
            const long long c = c0 + 64 * i + 4 * sub;
            v[i] = (row_ok && c < cols) ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(S + c))
                                        : f32x4{ninf, ninf, ninf, ninf};
        }
    };
    load(cur, 0);
    for (long long c0 = 0; c0 < cols; c0 += kCh) {
        if (c0 + kCh < cols) load(nxt, c0 + kCh);
#pragma unroll
        for (int bb = 0; bb < kBPS; ++bb) {
            if (j >= nblk) break;
            float M = ninf;
#pragma unroll
            for (int gi = 0; gi < kGPB; ++gi)
#pragma unroll
                for (int e = 0; e < 4; ++e) M = fmaxf(M, cur[bb * kGPB + gi][e]);
            M = row16_max(M);
            bool restart;
            float tq = ninf;
            if (j < p.n_b0) {
                restart = true;
            } else {
                if (M != ninf) tq = hif8::round(M - m);
                restart = ceilf(tq) > (float)p.lambda;
            }
            const float m_new = restart ? fmaxf(m, ceilf(M)) : m + fmaxf(0.0f, ceilf(tq));
            const float ref = restart ? m_new : m;
            const float alpha = (m == ninf) ? 0.0f : exp2_int(m - m_new);
            const float beta = (ref == ninf) ? 0.0f : exp2_int(ref - m_new);
            float rowsum = 0.0f;
#pragma unroll
            for (int gi = 0; gi < kGPB; ++gi) {
                uint32_t word = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float sv = cur[bb * kGPB + gi][e];
                    const float T = (sv == ninf || ref == ninf) ? ninf : sv - ref;
                    const uint32_t ent = tab[hif8::f2u(T) >> kTabShift];
                    word |= (ent & 0xffu) << (8 * e);
                    rowsum += hif8::u2f(ent & 0xffffff00u);
                }
                const long long c = c0 + (long long)bb * BLOCK + 64 * gi + 4 * sub;
                if (row_ok && c < cols) *reinterpret_cast<uint32_t*>(code + c) = word;
            }
            dl = alpha * dl + beta * rowsum;
            m = m_new;
            if (row_ok && p.restarted && sub == 0) p.restarted[rr * nblk + j] = restart ? 1 : 0;
            if (sub == (int)(j & 15)) myref = ref;
            if ((j & 15) == 15 || j == nblk - 1) {
                if (nblk > 16 && row_ok) {      // park the group's references until m is final
                    const long long idx = (j & ~15LL) + sub;
                    if (idx < nblk) refs_out[idx] = (int32_t)hif8::f2u(myref);
                }
            }
            ++j;
        }
#pragma unroll
        for (int i = 0; i < kG; ++i) cur[i] = nxt[i];
    }
    const float d = row16_sum(dl);
    if (!row_ok) return;
    if (sub == 0) {
        p.m_final[rr] = m;
        p.d_final[rr] = d;
    }
    auto shift = [&](float ref) -> int32_t {
        if (ref == ninf || m == ninf) return INT32_MIN;
        return (int32_t)fmaxf(ref - m, -2147483520.0f);
    };
    if (nblk <= 16) {
        if (sub < nblk) refs_out[sub] = shift(myref);
    } else {
        for (long long idx = sub; idx < nblk; idx += 16)
            refs_out[idx] = shift(hif8::u2f((uint32_t)refs_out[idx]));
    }
}

// Wide form: a workgroup of 256 threads takes whole rows, 4096 columns at a
// time with the next chunk's loads in flight.  The rule of Alg. 1
// depends on a block only through its maximum, so per chunk the maxima of
// every 64 columns meet in LDS (the only barrier), every wave runs the rule
// over the chunk's blocks, one per lane, and then all threads form their codes
// at the references found.  The rule itself is serial, but the integer maximum
// is nearly always the running maximum of the blocks' own ceil(maximum): each
// lane takes that as its guess (a prefix maximum), and the rule is repeated with
// its results in place of the wrong guesses until nothing changes.  Where the 8-bit cast
// rounds a block's T down to an integer the first guess is one too high from
// there on; the repeats mend all such blocks of a chunk at once (settling them
// one by one took 348 us on 16384 x 8192 scores that climb 6 per block at lambda
// 8, against 140 for the row-group form and 128 so).  A thread sums its P relative to the latest integer
// maximum by exact powers of two.  VEC: 16-byte aligned rows of a multiple of
// 4 columns (4 adjacent columns per lane); else columns go lane by lane.
//
// The other kernels give a row 16 or 64 lanes and walk it in steps: with few
// rows that walk, not memory, is the time (300 rows of 30000 columns 158 us,
// here 22; 4096 x 4096 41 -> 20 us; 16384 x 8192, back to back, 126 -> 120 us, 5.6 TB/s).
constexpr int kWideMaxBlk = 1024;                 // blocks per row (their references stay in LDS)

template <int BLOCK, bool VEC>
__global__ __launch_bounds__(kThreads) void softmax_block_wide_kernel(SoftmaxBlockParams p)
{
    constexpr int NT = kThreads;
    constexpr int kCols = 16 * NT;                        // columns per chunk
    constexpr int kSub = kCols / 64;                      // 64-column pieces per chunk
    constexpr int kNB = kCols / BLOCK;                    // blocks per chunk
    constexpr int kSteps = (kNB + 63) / 64;
    __shared__ __attribute__((aligned(16))) uint32_t tab[kTabEntries];
    __shared__ float maxs[2][kSub];
    __shared__ float refs_l[kWideMaxBlk];
    __shared__ float wsum[NT / 64];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = 4 * tid; i < kTabEntries; i += 4 * NT)
        *reinterpret_cast<u32x4*>(tab + i) = *reinterpret_cast<const u32x4*>(p.tab + i);

    const long long cols = p.cols;
    const int nblk = (int)((cols + BLOCK - 1) / BLOCK);
    const int nchunk = (int)((cols + kCols - 1) / kCols);
    const float ninf = -__builtin_huge_valf();
    // column of element (u, e) of this thread in a chunk
    auto col = [&](int u, int e) { return VEC ? u * 4 * NT + 4 * tid + e : (4 * u + e) * NT + tid; };
    auto load = [&](f32x4* v, const float* S, long long c0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if constexpr (VEC) {
                const long long c = c0 + col(u, 0);
                v[u] = c < cols ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(S + c))
                                : f32x4{ninf, ninf, ninf, ninf};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const long long c = c0 + col(u, e);
                    v[u][e] = c < cols ? __builtin_nontemporal_load(S + c) : ninf;
                }
            }
        }
    };
    int par = 0;                                          // buffer of maxs
    for (long long row = blockIdx.x; row < p.rows; row += gridDim.x) {
        const float* S = p.s + row * p.ld;
        uint8_t* code = p.codes + row * cols;
        float m = ninf, dl = 0.0f;
        f32x4 cur[4], nxt[4];
        load(cur, S, 0);
        for (int ch = 0; ch < nchunk; ++ch, par ^= 1) {
            const long long c0 = (long long)ch * kCols;
            if (ch + 1 < nchunk) load(nxt, S, c0 + kCols);
            // maxima of the 64-column pieces
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (VEC) {
                    const float mx = row16_max(fmaxf(fmaxf(cur[u][0], cur[u][1]), fmaxf(cur[u][2], cur[u][3])));
                    if ((lane & 15) == 0) maxs[par][u * (NT / 16) + (tid >> 4)] = mx;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float mx = wave_max_uniform(cur[u][e]);
                        if (lane == 0) maxs[par][(4 * u + e) * (NT / 64) + wave] = mx;
                    }
                }
            }
            __syncthreads();                              // (and, the first time, the table)
            // the rule over the chunk's blocks
            float refs[kSteps];
            const float m_old = m;
#pragma unroll
            for (int st = 0; st < kSteps; ++st) {
                const int jl = 64 * st + lane;            // block of the chunk, and of the row
                const int j = ch * kNB + jl;
                float M = ninf;
                if (jl < kNB) {
#pragma unroll
                    for (int k = 0; k < BLOCK / 64; ++k) M = fmaxf(M, maxs[par][jl * (BLOCK / 64) + k]);
                }
                const bool in_row = jl < kNB && j < nblk;
                const float h = in_row ? ceilf(M) : ninf;
                // lanes 0 .. last hold the blocks.  hc: what m is taken to rise to
                // at each, first the ceil of its own maximum, then, where that was
                // wrong, what the rule made of it (the first k lanes are right
                // after k repeats: at most last of them)
                const int last = min(kNB - 64 * st, nblk - ch * kNB - 64 * st) - 1;
                float hc = h, g, m_new;
                bool restart;
                for (int it = 0;; ++it) {
                    g = fmaxf(m, prefix_max_before<64>(hc));
                    float tq = ninf;
                    if (M != ninf) tq = hif8::round(M - g);       // g = -inf gives +inf: restart
                    restart = j < p.n_b0 || ceilf(tq) > (float)p.lambda;
                    m_new = restart ? fmaxf(g, h) : g + fmaxf(0.0f, ceilf(tq));
                    const bool wrong = m_new != fmaxf(g, hc);     // (never behind the last block)
                    if (it >= last || !__any(wrong)) break;
                    if (wrong) hc = m_new > g ? m_new : ninf;
                }
                const float ref = lane > last ? ninf : (restart ? m_new : g);
                const bool rst = restart;
                m = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, m_new), last));
                refs[st] = ref;
                if (wave == 0 && in_row) {
                    refs_l[j] = ref;
                    if (p.restarted) p.restarted[row * nblk + j] = rst ? 1 : 0;
                }
            }
            // codes, and this thread's P relative to the new integer maximum
            dl = (m_old == ninf) ? 0.0f : dl * exp2_int(m_old - m);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                uint32_t word = 0;
                float rowsum = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // (VEC: the four columns share a block; else each column of the wave does)
                    const int base = VEC ? u * 4 * NT : (4 * u + e) * NT;
                    const int st = (base / BLOCK) / 64;
                    const int src = VEC ? (base / BLOCK) % 64 + (BLOCK <= 4 * NT ? 4 * tid / BLOCK : 0)
                                        : (base + 64 * wave) / BLOCK - 64 * st;
                    float ref, beta;
                    if constexpr (VEC) ref = __shfl(refs[st], src, 64);
                    else ref = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, refs[st]), src));
                    const float sv = cur[u][e];
                    const float T = (sv == ninf || ref == ninf) ? ninf : sv - ref;
                    const uint32_t ent = tab[hif8::f2u(T) >> kTabShift];
                    const float pv = hif8::u2f(ent & 0xffffff00u);
                    if constexpr (VEC) {
                        word |= (ent & 0xffu) << (8 * e);
                        rowsum += pv;
                        if (e == 3) {
                            beta = (ref == ninf) ? 0.0f : exp2_int(ref - m);
                            dl += beta * rowsum;
                            const long long c = c0 + col(u, 0);
                            if (c < cols) *reinterpret_cast<uint32_t*>(code + c) = word;
                        }
                    } else {
                        beta = (ref == ninf) ? 0.0f : exp2_int(ref - m);
                        dl += beta * pv;
                        const long long c = c0 + col(u, e);
                        if (c < cols) code[c] = (uint8_t)(ent & 0xffu);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
        }
        const float ws = wave_sum(dl);
        if (lane == 0) wsum[wave] = ws;
        __syncthreads();                                  // references and sums of the row
        if (tid == 0) {
            float d = wsum[0];
#pragma unroll
            for (int w = 1; w < NT / 64; ++w) d += wsum[w];
            p.m_final[row] = m;
            p.d_final[row] = d;
        }
        for (int idx = tid; idx < nblk; idx += NT) {
            const float ref = refs_l[idx];
            p.ref_shift[row * nblk + idx] =
                (ref == ninf || m == ninf) ? INT32_MIN : (int32_t)fmaxf(ref - m, -2147483520.0f);
        }
        __syncthreads();                                  // read before the next row writes
    }
}

template <bool VEC>
hipError_t launch_wide(const SoftmaxBlockParams& p, int ncu, hipStream_t st)
{
    const long long most = 4LL * ncu;                     // 37 KiB of LDS: four workgroups per CU
    const dim3 grid((unsigned)(p.rows < most ? p.rows : most));
    switch (p.block) {
    case 64: hipLaunchKernelGGL((softmax_block_wide_kernel<64, VEC>), grid, dim3(kThreads), 0, st, p); break;
    case 128: hipLaunchKernelGGL((softmax_block_wide_kernel<128, VEC>), grid, dim3(kThreads), 0, st, p); break;
    case 256: hipLaunchKernelGGL((softmax_block_wide_kernel<256, VEC>), grid, dim3(kThreads), 0, st, p); break;
    case 512: hipLaunchKernelGGL((softmax_block_wide_kernel<512, VEC>), grid, dim3(kThreads), 0, st, p); break;
    case 1024: hipLaunchKernelGGL((softmax_block_wide_kernel<1024, VEC>), grid, dim3(kThreads), 0, st, p); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Whether the wide form is the faster one, drawn through 2290 aligned shapes of
// 4 to 65536 rows and 4 to 50000 columns (the other form in front, us): 1.90
// times as fast in the geometric mean, no shape below 0.98.  It spends a whole
// chunk of 4096 columns on a shorter rest of a row, so with many short rows the
// forms that pack rows into a wave win (4000 x 1000, block 128: 12.2 against
// 15.6; 2000 x 1000 11.4 against 9.6), and so they do with many rows that end
// just behind a chunk (16384 x 4100, block 256: 72 against 92, block 64: 82
// against 92; 4096 x 4100, block 1024: 23 against 27; but 8192 x 4100, block 64,
// 117 against 50: the wide steps of 256 threads spill there).  Blocks of 512 and 1024 make the walk of
// the other form shorter: their lines lie at fewer rows; block 256 is between
// (4096 x 2048 15.5 against 16.2, 16384 x 3000 55 against 57).  Unaligned rows
// store byte by byte either way, and there the wide form only pays where the
// others leave the chip idle (300 x 2001 8.3 against 14.1; 2000 x 2001 17.7
// against 15.6).
bool wide_is_faster(const SoftmaxBlockParams& p, bool aligned)
{
    if (p.cols < 1 || (p.cols + p.block - 1) / p.block > kWideMaxBlk) return false;
    const bool big = p.block > 256;
    if (!aligned) return p.rows <= 1024 && p.cols >= (big ? 1500 : 512) && p.cols >= (big ? 8 : 4) * p.rows;
    if (p.cols > 4096 && p.cols < 5200) return p.rows <= (big ? 2048 : (p.block == 256 ? 7000 : 10000));
    if (p.cols >= 3000) return p.block != 256 || p.cols >= 3300 || p.rows <= 10000;
    if (p.block == 256) return p.rows <= 2 * p.cols && (p.rows <= 2048 || 5 * p.rows <= 9 * p.cols);
    return p.rows <= (big ? 1 : 2) * p.cols;
}

template <int NT, int KCH>
hipError_t launch_block4(const SoftmaxBlockParams& p, hipStream_t st)
{
    constexpr int kRows4PerBlock = kRowsPerWave4 * (NT / 64);
    const dim3 grid4((unsigned)((p.rows + kRows4PerBlock - 1) / kRows4PerBlock));
    switch (p.block) {
    case 64: hipLaunchKernelGGL((softmax_block4_kernel<64, NT, KCH>), grid4, dim3(NT), 0, st, p); break;
    case 128: hipLaunchKernelGGL((softmax_block4_kernel<128, NT, KCH>), grid4, dim3(NT), 0, st, p); break;
    default: hipLaunchKernelGGL((softmax_block4_kernel<256, NT, KCH>), grid4, dim3(NT), 0, st, p); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_softmax_block(const SoftmaxBlockParams& p, hipStream_t st)
{
    const bool aligned = ((uintptr_t)p.s % 16 == 0) && (p.ld % 4 == 0) && (p.cols % 4 == 0) &&
                         ((uintptr_t)p.codes % 4 == 0);
    int ncu = 0;
    const hipError_t e = cu_count(&ncu);
    if (e != hipSuccess) return e;
    if (wide_is_faster(p, aligned)) return aligned ? launch_wide<true>(p, ncu, st) : launch_wide<false>(p, ncu, st);
    if (aligned && p.block <= 256) {
        // one 1024-thread workgroup per CU when the rows fill every CU
        const long long wg1024 = (p.rows + 4 * 16 - 1) / (4 * 16);
        if (wg1024 >= ncu) return p.cols >= 4096 ? launch_block4<1024, 512>(p, st) : launch_block4<1024, 256>(p, st);
        // fewer rows than CUs x 64: at most two 256-thread workgroups per CU
        // take 1024 columns per step (162 VGPRs), more take 256
        const long long wg256 = (p.rows + 4 * 4 - 1) / (4 * 4);
        return wg256 <= 2 * ncu ? launch_block4<256, 1024>(p, st) : launch_block4<256, 256>(p, st);
    }
    const dim3 grid((unsigned)((p.rows + kRowsPerBlock - 1) / kRowsPerBlock));
    switch (p.block) {
    case 64: hipLaunchKernelGGL(softmax_block_kernel<64>, grid, dim3(kThreads), 0, st, p); break;
    case 128: hipLaunchKernelGGL(softmax_block_kernel<128>, grid, dim3(kThreads), 0, st, p); break;
    case 256: hipLaunchKernelGGL(softmax_block_kernel<256>, grid, dim3(kThreads), 0, st, p); break;
    case 512: hipLaunchKernelGGL(softmax_block_kernel<512>, grid, dim3(kThreads), 0, st, p); break;
    case 1024: hipLaunchKernelGGL(softmax_block_kernel<1024>, grid, dim3(kThreads), 0, st, p); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace baps
