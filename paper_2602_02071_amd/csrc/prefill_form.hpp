// Which form of the fused attention kernel a call takes (host only, no HIP:
// the tests compile this header by itself).
#pragma once

namespace baps {

// NW waves per workgroup, KW of them on the same rows: 32 * NW / KW query rows
// per work item.
struct PrefillForm {
    int nw, kw;
};

struct PrefillShape {
    int D, block;
    long long Sq, Sk, group, heads;   // heads: (batch, key/value head) pairs; group: query heads of each
    bool causal, fp8;                 // fp8: FP8 Q/K
    bool alg1, full_table, ties_even; // Alg. 1 (not eq. 2); the full score table (lambda > 8); ties to even
    int ncu;
};

// 128 rows on four waves against 256 on eight, where two such workgroups share
// a CU: the same waves at work, half the step when items run out, and two
// barriers of four waves instead of one of eight.  n256, n128: their items.
// Measured in 12 classes of 32 shapes (times of 256 over 128 rows).  D * block
// = 8192: causal at D = 128 0.97 to 1.34, mean 1.11 (the longest item ends
// earlier); not causal 0.90 to 1.59, so only where the last round thins out:
// fewer rounds (480 items for 288: 1.38 and 1.59), or at most half a second
// round of 256-row items on rows long enough that an item's start does not
// weigh (384 items of 1369 keys 1.06 and 1.14; of 300 keys 0.94).  FP8 Q/K
// under a causal mask at D = 64: 0.98 to 1.23, mean 1.10.  Past four rounds
// the two are alike.
inline bool four_waves_are_faster(const PrefillShape& s, long long n256, long long n128)
{
    const int size = s.D * s.block;
    const long long ncu = s.ncu;
    if (n256 > 4 * ncu) return false;
    if (s.causal && (s.fp8 ? (s.D == 64 || s.block == 64) : (s.D == 128 && s.block == 64))) return true;
    if (size != 8192) return false;
    return (n256 + ncu - 1) / ncu > (n128 + 2 * ncu - 1) / (2 * ncu) ||
           (n256 > ncu && 2 * n256 <= 3 * ncu && s.Sk >= 8 * s.block);
}

// The rows of a work item, by how many items that leaves for the CUs.  A wave
// is bound by the latency of its own chain (QK^T, row maximum, decision, table
// reads, PV), so a key block takes 3.0 us with eight waves on 256 rows, 2.2 us
// with eight on 128 rows (each block's keys split over two waves of the same
// rows) and 1.8 us with four on 64 rows (likewise) at D = 128, block 128: the
// smallest tile wins while all its items run at once, the largest once the
// items queue.  64 rows: up to three workgroups per CU at D * block = 4096, two
// at 8192 and one at 16384, where the K/V buffers fill the LDS; 128 rows: one.
// Measured over 340 shapes (1 to 16 sequences of 100 to 4096 queries, contexts
// to 9000 keys): 1.27x 256 rows alone in the geometric mean, at most 6 %
// slower anywhere (GQA 32/8, D = 128: 512 queries 19.3 -> 11.5 us, 512 queries
// on 4096 keys 101.5 -> 56.8 us, 1024 queries 33.2 -> 25.8 us).
inline PrefillForm prefill_form(const PrefillShape& s)
{
    const PrefillForm rows256{8, 1}, rows128{8, 2}, rows64{4, 2}, four_waves{4, 1};
    if (s.block < 64) return rows256;
    const int size = s.D * s.block;
    const long long ncu = s.ncu, flat = s.Sq * s.group;
    const long long n64 = (flat + 63) / 64 * s.heads, n128 = (flat + 127) / 128 * s.heads,
                    n256 = (flat + 255) / 256 * s.heads;
    const int per_cu = size <= 4096 ? 3 : (size <= 8192 ? 2 : 1);
    if (n64 <= per_cu * ncu) return rows64;
    // (with two or three 64-row workgroups per CU the 128-row items never fit when the 64-row ones do not)
    if (per_cu == 1 && n128 <= ncu) return rows128;
    if (s.alg1 && !s.full_table && !s.ties_even && per_cu > 1 && four_waves_are_faster(s, n256, n128))
        return four_waves;
    return rows256;
}

}  // namespace baps
