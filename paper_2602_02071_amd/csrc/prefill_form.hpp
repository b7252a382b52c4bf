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

// A wave is bound by the latency of its own chain (QK^T, row maximum, decision,
// table reads, PV), so a key block takes 3.5 us with eight waves on 256 rows,
// 2.2 us with eight on 128 rows (each block's keys split over two waves of the
// same rows) and 1.5 us with four on 64 rows (likewise) at D = 128, block 128
// (bf16, one workgroup on every CU, 64 blocks against 32):
// the smallest item wins while all items run at once, the largest once they
// queue (GQA 32/8, D = 128: 512 queries 19.3 -> 11.5 us, 512 queries on 4096
// keys 101.5 -> 56.8 us, 1024 queries 33.2 -> 25.8 us); four waves on 128 rows,
// two workgroups per CU, win where a round of 256-row items runs thin.  The
// lines were drawn through 14800 shapes with every form timed (2 to 400 heads,
// 64 to 4096 queries, to 10000 keys, all setups): 1.160 times the speed of 256
// rows alone in the geometric mean (the best form of each shape: 1.172), 11
// shapes below 0.98, the least 0.93.  D * block names the K/V buffers' size
// (4096, 8192 or 16384); factors are times of 256 rows over the form's.
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
    // block 128: 0.79; 200 heads, 500 keys 0.92 at 16384).  Short rows at D = 64
    // still gain (133 heads of 150 positions 1.12, causal 1.22), and so do ties
    // to even at 16384, whose lookups weigh more than the reads (200 heads, 128
    // rows, 1500 keys 1.2).
    const bool held = flat <= 256 && 2 * s.heads > ncu && n256 <= ncu && !(s.ties_even && size == 16384) &&
                      !(s.D == 64 && flat > 128 && Sk <= 2 * flat);
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
    // 128 rows on four waves, two workgroups per CU: the same waves at work,
    // half the step when items run out, two barriers of four waves instead of
    // one of eight; a pair is 2 to 8 % slower than eight waves on the same rows
    // where nothing runs out.  Measured on bf16 and FP8 Q/K of the canonical
    // setup only (the others are not built); past four rounds it is level.
    if (!s.alg1 || s.full_table || s.ties_even || size == 16384 || n256 > 4 * ncu) return rows256;
    if (held && !(s.causal && flat > 128 && Sk <= 2 * flat)) return rows256;
    const bool fewer = (n256 + ncu - 1) / ncu > (n128 + 2 * ncu - 1) / (2 * ncu);      // rounds
    const bool thin = fewer || (n256 > ncu && 2 * n256 <= 3 * ncu && Sk >= 8 * s.block);
    // Not causal: a thin last round (480 items for 288: 1.38 to 1.59; 288 to 384
    // items of 1024 keys and more 1.04 to 1.2).  At 4096, where two 256-row
    // workgroups share a CU anyway, FP8 gains as much in a round as thin (1.07
    // to 1.18) and is not taken; bf16 is not built.
    if (!s.causal) return size == 8192 && thin ? four_waves : rows256;
    // Causal: what the CUs have on average, in units of the longest item.
    // Below 0.63 that item sets the time and a half-size one ends earlier (1.1
    // to 1.2); near 1 the long-and-short pairs of the 256-row schedule fill the
    // GPU and four waves lose (GQA 32/8, 4096 positions, D = 128: 0.93).
    const double load = (double)n256 * (double)(2 * Sk - q) / (2.0 * (double)Sk * (double)ncu);
    const bool lead = 3 * q >= Sk && load <= (3 * q >= 2 * Sk ? 0.70 : 0.63);
    bool four;
    if (size == 4096)          // FP8 only: 1.0 to 1.2; cached keys in front and many items 0.97
        four = s.fp8 && (n128 <= 3 * ncu || (5 * q >= 2 * Sk && n256 <= 2 * ncu) || 4 * q >= 3 * Sk);
    else if (s.D == 128)       // also heads of few items unless those nearly fill two rounds or four (512 positions
                               // 1.2, 700 1.12), and rows that 256-row tiles pad by a twelfth (1369 positions 1.1)
        four = lead || (3 * q >= Sk && flat <= 1024 && (4 * n256 < 7 * ncu || (n256 > 2 * ncu && 2 * n256 <= 7 * ncu))) ||
               (24 * n256 >= 13 * n128 && 3 * q >= Sk);
    else                       // D = 64, block 128
        four = (s.fp8 && load <= 0.70 && 3 * q >= Sk && (load <= 0.55 || flat <= 768 || Sk >= 8 * s.block)) ||
               (thin && (load <= 0.74 || 2 * q < Sk)) || (fewer && 10 * n256 >= 6 * n128);
    return four ? four_waves : rows256;
}

}  // namespace baps
