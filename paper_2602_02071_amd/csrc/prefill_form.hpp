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
// items queue (GQA 32/8, D = 128: 512 queries 19.3 -> 11.5 us, 512 queries on
// 4096 keys 101.5 -> 56.8 us, 1024 queries 33.2 -> 25.8 us).  Below, D * block
// names the K/V buffers' size: 4096, 8192 or 16384.  Factors are times of 256
// rows over the form's.
inline PrefillForm prefill_form(const PrefillShape& s)
{
    const PrefillForm rows256{8, 1}, rows128{8, 2}, rows64{4, 2}, four_waves{4, 1};
    if (s.block < 64) return rows256;
    const int size = s.D * s.block;
    const long long ncu = s.ncu, flat = s.Sq * s.group, Sk = s.Sk;
    const long long q = s.Sq < Sk ? s.Sq : Sk;              // query positions that see a key, causal
    const long long n64 = (flat + 63) / 64 * s.heads, n128 = (flat + 127) / 128 * s.heads,
                    n256 = (flat + 255) / 256 * s.heads;
    // 64-row workgroups whose LDS fits a CU: K/V buffers, the table (8 KiB, or 16
    // for ties to even and the full one; none in eq. (2)'s fp32 setup, which fits
    // as often) and the exchanged row maxima
    const int lds64 = 8 * size + (s.ties_even || s.full_table ? 16 : 8) * 1024 + 1024 + 256;
    const int fit64 = 160 * 1024 / lds64;
    // One 256-row item holds a head's rows and more than half of the CUs have
    // one: smaller items read K/V again (256 heads, 128 rows, 5000 keys, D = 64,
    // block 128: 0.79; 200 heads, 500 keys 0.92 at 16384).  Short causal rows at
    // D = 64 still gain (133 heads of 150 positions 1.22), and so do ties to
    // even at 16384, whose lookups weigh more than the reads (200 heads, 128
    // rows, 1500 keys 1.2).
    const bool held = flat <= 256 && 2 * s.heads > ncu && n256 <= ncu && !(s.ties_even && size == 16384) &&
                      !(s.causal && s.D == 64 && flat > 128 && Sk <= 2 * flat);
    if (!s.full_table && !held) {
        if (n64 <= ncu) return rows64;
        // A second one per CU, if its LDS fits there (ties to even at 8192: 81
        // KiB, not); if not, where causal items end at very different times
        // (700 positions of 24 heads 1.4; not causal 0.6 to 0.9).
        const bool uneven = s.causal && (3 * q >= 2 * Sk ? Sk >= 500 || (Sk >= 300 && 2 * n64 <= 3 * ncu)
                                                         : 5 * q >= 2 * Sk && Sk >= 1500);
        if (size < 16384 && n64 <= 2 * ncu && (fit64 >= 2 || uneven)) return rows64;
        // A third: causal (1.05 to 1.4; 150 positions 0.97 unless the 256-row
        // items do not fit at once, 1.12), 256-row items that do not (144 heads
        // of 257 positions 1.14), or long rows (4096 positions of 12 heads 1.04)
        // whose K/V stay on one XCD, are few or have as many queries to share
        // them (65 heads, 512 on 6000 keys: 0.87).  Other short ones lose: 197
        // positions of 192 heads 0.94, 256 of 170 0.81.
        const bool local = s.heads % 8 == 0 || s.heads <= 32 || 2 * s.Sq >= Sk;
        if (fit64 >= 3 && n64 <= 3 * ncu &&
            ((s.causal && 3 * q >= Sk && (flat > 192 || n256 > ncu)) ||
             (flat > 256 && (n256 > ncu || (Sk >= 1024 && local)))))
            return rows64;
        // (at 8192 and below 128-row items never all fit when 64-row ones do not)
        if (size == 16384 && n128 <= ncu) return rows128;
    }
    if (s.full_table && !held) {
        // The full table costs a workgroup 2 us before its first block: more,
        // smaller workgroups only where rows are long or many and a head's K/V
        // stay on one XCD, are few, or are long enough to hide that (one per
        // CU: 256 positions of 48 heads 1.3 at 16384, 300 of 51 heads 0.86; two
        // at 8192, where they do not fit at once: 500 positions of 37 heads
        // 0.58, 3000 causal positions of 8 heads 1.5).
        const bool local = s.heads % 8 == 0 || s.heads <= 32;      // K/V stay on one XCD, or are few
        const bool ramp = s.causal && 3 * q >= 2 * Sk;
        if (n64 <= ncu && (flat > 128 ? Sk >= 1024 || flat > 512 || (local && (size > 4096 || Sk >= 256)) : Sk >= 4096))
            return rows64;
        if (size == 4096 && n64 <= 2 * ncu && ((flat > 256 && Sk >= 1024) || (flat > 512 && local))) return rows64;
        if (size == 4096 && n64 <= 3 * ncu && ((ramp && Sk >= 1500) || (s.causal && 3 * q >= Sk && Sk >= 700 && local)))
            return rows64;
        if (size == 8192 && n64 <= 2 * ncu && ramp && (Sk >= 2048 || (Sk >= 600 && 2 * n64 <= 3 * ncu))) return rows64;
        if (size == 16384 && n128 <= ncu && flat > 128) return rows128;
    }
    // (four waves: two items of a head's 129 to 256 rows, short causal ones only)
    if (held && !(s.causal && flat > 128 && Sk <= 2 * flat)) return rows256;
    if (s.alg1 && !s.full_table && !s.ties_even && size < 16384 && four_waves_are_faster(s, n256, n128))
        return four_waves;
    return rows256;
}

}  // namespace baps
