// Which calls run on the kernels that take whole chunks (gla_onepass.hip, gla_onepass_bwd.hip), and how they are cut: host rules on sizes
// alone, in plain C++ (the tests compile this file by itself).
#pragma once
#include <stddef.h>

namespace gla {

// Most spans per (batch, head) that the output pass chains by itself: work-group r reads the r local states
// before it, so the reads grow with the square of the span count while a carry kernel's grow linearly.
constexpr int kMaxChainedSpans = 128; // beyond this the reads of a slowly decaying chain outgrow the carry kernel

// A call that those kernels cover, in bf16 rows
struct OnePassCall {
    long long bh;       // sequences
    int nchunks;        // 64-token chunks of one
    bool small;         // heads of up to 32 / 64 channels
    bool two_sided, prologue, epilogue;
};

// Bytes of the flags of a single-launch plan (two waves a chunk), which lie behind the sums of the gates
inline size_t onepass_flag_bytes(size_t bh, size_t nspans, int chunks) { return (bh * nspans * 2 * chunks * sizeof(unsigned long long) + 255) / 256 * 256; }

// The next three functions: chunks that a work-group of the single-launch forward kernels holds (4 or 8), or 0 where the call stays on the others.  Eight chunks fill
// a compute unit, so up to 2048 are one round of work-groups, all loads in flight at once.  Below: time of the two-pass kernels over
// that of these, in sequences x chunks (36 / 72 channels; S: 32 / 64 channels), bf16 row scan and fp32 column scan where there are two.

// With the output epilogue (the two-pass kernels take two fills and a pass for it):
//     4 chunks      16 1.34, 256 1.16, 512 1.11, 1920 1.03 (S 16 1.50, 510 1.19, 1920 1.23); 3 chunks 64 1.10, 192 1.06, but 288 0.95, 384 0.98
//                   (S 192 1.20, 288 0.97); 2 chunks 192 0.89 (S 0.96)
//     groups of 4   3 x 16 1.11 1.04, 6 x 12 1.14 1.06, 16 x 8 1.05, 48 x 5 1.02, 32 x 12 1.36, but 16 x 5 0.99, 16 x 6 1.01 0.98, 32 x 5 0.99
//                   (S 12 x 6 1.14 1.07); 160 x 9 1.35
//     groups of 8   192 x 6 1.11, 256 x 6 1.10, 256 x 8 1.28, but 192 x 5 1.00 (S 1.34); 6 x 300 1.49
//     rounds        16 x 256 1.07 1.12, 32 x 128 1.08 1.18, 128 x 24 1.07 1.15, 160 x 24 1.20 1.28, 192 x 16 1.15 1.12, but 64 x 43 1.01 1.03, 256 x 32
//                   0.94 0.92, 256 x 12 0.87, and where the second round is less than half full, or a few long sequences (row scans, z = 0 and 3) 16 x 160 0.89 0.94,
//                   32 x 80 0.93 0.97, 48 x 48 0.94 0.98, 16 x 192 0.95 0.97, 32 x 96 0.99 1.02, 16 x 208 0.99 1.05; in fours 192 x 12 1.14, but 192 x 9 0.95, 256 x 12 1.03 0.97, 32 x 128 with slow gates 0.81, 512 x 8 0.89,
//                   304 x 6 0.97 (sequences from 256 on stay in one pass each, 304 x 12 1.22 for all that); S, in fours: 96 x 32 1.47, 192 x 16 1.58, 126 x 32 1.18, 252 x 9 1.24, 510 x 8 1.09, but 510 x 6 0.95, 510 x 5 0.80
inline int onepass_epilogue_chunks(const OnePassCall &p) {
    const int nchunks = p.nchunks;
    const long long bh = p.bh, total = bh * nchunks;
    const bool small = p.small;
    auto groups = [&](int chunks) { return bh * ((nchunks + chunks - 1) / chunks); };
    if (nchunks <= 4) return (nchunks == 4 && bh * 512 < (1LL << 32)) || (nchunks == 3 && bh <= 256) ? 4 : 0;
    if (total < (small ? 48 : nchunks >= 8 ? 72 : 192)) return 0;
    if (groups(4) <= 256) return 4;
    if (bh > 128 && nchunks <= 8) {
        if (bh <= 256) return small || nchunks >= 6 ? 8 : 0;
        return small && nchunks == 8 && bh <= 512 ? 4 : 0;
    }
    if (groups(8) <= 256) return 8;
    if (groups(4) <= 512) return 4;
    if (small) return groups(4) <= 1024 ? 4 : 0;
    if (bh >= 256) return 0;
    // three groups of four with at most one place empty (9 and 10 chunks leave more of them idle, 13 to 15 begin a fourth)
    if (nchunks < 16) return (nchunks == 11 || nchunks == 12) && groups(4) <= 1024 ? 4 : 0;
    // (a second round that is at least half full; of long sequences somewhat more, since its groups look back further)
    return groups(8) <= 512 && total >= (nchunks > 128 ? 3300 : 2990) ? 8 : 0;
}

// With the two-sided gate there is room for four chunks on a compute unit, in one group: 16 x 4 1.29 (S 1.05), 256 x 4 1.17 (S 1.01), 512 x 4
// 1.17 (S 0.83), 16 x 16 1.02 (column scan 0.87), 32 x 9 1.28 (S 1.13), 64 x 16 1.73 (S 1.52), and in several rounds 128 x 9 1.17 (S 1.00),
// 32 x 64 1.43, 16 x 256 1.38, 128 x 32 1.40 (S 1.16), but 192 x 5 0.74 and 256 x 16 0.87, whose sequences the other kernels walk in one pass.
inline int onepass_two_sided_chunks(const OnePassCall &p) {
    const int nchunks = p.nchunks;
    const long long bh = p.bh;
    if (nchunks <= 4) return nchunks == 4 && (bh <= 128 || !p.small) && bh * 512 < (1LL << 32) ? 4 : 0;
    return bh <= 128 && bh * nchunks >= 288 ? 4 : 0;
}

// Of the plain call the backward call may take the span states, so this is a matter of both:
//     4 chunks      16 1.14, 128 1.10, but 192 1.02 0.97, 256 0.97 0.94 (S 96 1.15, 240 1.05, 360 1.03, 600 1.10; both calls 1.05 to 1.01)
//     groups of 4   64 x 8 1.18, 32 x 32 1.16, 128 x 8 1.29; S: 16 x 20 1.14, 16 x 32 1.16; two groups on a unit 96 x 17 1.16 to 1.31
//     groups of 8   16 x 100 1.20, 32 x 64 1.26, 128 x 16 1.38, 128 x 5 1.13; 136 x 6 1.35 1.57, 168 x 6 1.33 1.57, 168 x 7 1.46 1.64 (both calls 1.11 and
//                   1.24), where the other plan has one round and a half, but 176 x 6 0.96 1.03, 144 x 5 0.96, 256 x 7 0.93 1.04 (S 0.94);
//                   192 x 7 1.00 1.08, 224 x 8 1.01 1.10 (S 1.02 1.04)
//     two rounds    32 x 100 1.08, 32 x 128 1.15 1.18, 64 x 64 1.14, 96 x 32 1.15 1.14, 16 x 256 1.10 1.16, but 64 x 43 0.93,
//                   128 x 17 0.91, 192 x 16 1.29 0.95; three and more 0.87 to 1.11; S (z = 0, 3, 6) 12 x 256 1.02 0.95 0.90, 10 x 320 1.01 0.94 0.85, 8 x 400
//                   1.00 0.96 0.86, but 14 x 240 1.05 1.03 0.96, 18 x 200 1.13 1.12 1.07, 12 x 320 1.09 1.04 0.93
// Sequences of up to three chunks, which would leave waves idle, take 0.6 to 1.0.  Of longer ones, smaller calls stay with the others
// although the forward call alone would gain (16 x 8 16.2 us, 14.6 here; 16 x 20 19.8, 17.4): the walks of the backward call that takes the
// span states want spans of one or two chunks there (both calls: 16 x 8 39.9 us, here 44.4; 16 x 20 52.5, here 52.5 to 58; [B,T,H,d]
// 32 x 13 55.5 and 64.4), and in spans that short these kernels gain nothing (16 x 8 18.0 us, 16 x 20 19.3, 16 x 27 22.8 for 20.7) but for
// few of them a sequence (64 x 5 1.11, both calls 1.03) and small heads (16 x 20, both calls: 44.6 us, here 42.8).
inline int onepass_plain_chunks(const OnePassCall &p) {
    const int nchunks = p.nchunks;
    const long long bh = p.bh, total = bh * nchunks;
    const bool small = p.small;
    auto groups = [&](int chunks) { return bh * ((nchunks + chunks - 1) / chunks); };
    if (nchunks <= 4) return nchunks == 4 && bh <= (small ? 640 : 128) ? 4 : 0;
    if (total < (small ? 288 : nchunks <= 10 ? 320 : 513)) return 0;
    if (groups(4) <= 256) return 4;
    // One group of eight a sequence, one round.  What it costs does not fall with the places that are empty, so six chunks pay only while the other plan
    // cuts them into three spans (up to 512 of them, 170 sequences; then into two), seven a little longer
    if (bh > 128) return nchunks <= 8 && bh <= (nchunks == 8 ? 256 : nchunks == 7 ? 192 : nchunks == 6 ? 170 : 0) ? 8 : 0;
    if (groups(8) <= 256) return 8;
    if (groups(4) <= 512) return 4;
    // (a second round that is about half full: 2048 chunks and 942 more; of long sequences of small heads somewhat more, as with the epilogue)
    return groups(8) <= 512 && total >= (small && nchunks > 128 ? 3300 : 2990) && !p.prologue ? 8 : 0;
}

constexpr int onepass_resident(int chunks, bool two_sided) { return chunks == 8 || two_sided ? 256 : 512; }     // groups at once

// Most spans of a sequence where all groups are resident at once.  With gates that decay by nothing (z = 6) every earlier span is looked at,
// four a trip to memory (of about 1 us) in groups of eight, two in groups of four; the two-pass kernels take 16 or 32, and a kernel of its own above
// kMaxChainedSpans.  Their time over that of these, z = 0, 3 and 6, fours and in their place eights:
//     36 / 72 channels   4 x 192 (48 spans of 4) 1.20 1.06 0.99 (1.03 1.17 1.28), 3 x 256 (64) 1.29 1.01 0.90 (1.11 1.14 1.23), 2 x 320 (80) 1.30 1.06 0.90
//                        (1.17 1.25 1.38), 2 x 512 (128) 1.19 1.00 0.73 (1.12 1.18 1.29); eights 2 x 700 (88) 1.18 1.21 1.11, 2 x 1024 (128) 1.26 1.23 0.98
//     32 / 64            2 x 256 (64) 1.30 1.04 1.00 (0.94 1.00 1.15), 2 x 320 (80) 1.40 1.07 0.89 (1.06 1.01 1.03), 2 x 512 (128) 1.37 1.04 0.72
//                        (1.03 0.97 0.93), 1 x 512 (128) 3.14 2.01 0.89 (2.20 1.89 1.19); eights 4 x 512 (64) 1.25 1.21 1.03, but 2 x 700 (88) 1.15 1.11
//                        0.88, 2 x 1024 (128) 1.25 1.21 0.80
//     epilogue           2 x 256 (64) 1.45 1.23 1.13, 3 x 320 (80) 1.38 1.17 0.97 (1.16 1.23 1.33), 1 x 512 (128) 2.33 1.60 0.68 (1.81 1.63 1.09), eights
//                        2 x 1024 (128) 1.38 1.39 1.16; 32 / 64: 2 x 512 (128) 2.67 1.96 1.04, eights 2 x 1024 2.16 2.00 1.11
//     two-sided gate     2 x 400 (100) 1.80 1.41 1.01, 2 x 512 (128) 1.72 1.38 0.94, and one sequence, which the others cut into more than
//                        kMaxChainedSpans spans, 1 x 320 (80) 2.18 1.45 0.77; 32 / 64: 1 x 400 (100) 2.39 1.83 1.03, 1 x 512 (128) 2.62 2.00 0.97
inline int onepass_most_spans(const OnePassCall &p, int chunks) {
    if (p.two_sided) return p.bh > 1 || p.small ? 100 : 0;
    if (p.epilogue) return chunks == 4 && !p.small ? 64 : kMaxChainedSpans;
    return p.small ? 64 : chunks == 4 ? 48 : kMaxChainedSpans;
}

// The same in several rounds, where a group that looks back keeps its place on a unit from the groups of the next round.  `aligned`: the
// sequences lie whole within the ranges of spans that the XCDs work through (onepass_block).  z = 0, 3 and 6:
//     two-sided gate   aligned 24 x 192 (48 spans) 1.39 1.14 1.03 (S 1.20 1.07 1.02), 16 x 256 (64) 1.36 1.07 0.84 (kept for the former two); else, in two rounds,
//                      12 x 160 (40) 1.49 1.18 1.00 (S 1.33 1.15 1.04), and in more 26 x 96 (24) 1.38 1.17 1.17 (S 1.21 1.09 1.09), 60 x 128 (32) 1.32
//                      0.96 0.91, 18 x 256 (64) 1.31 0.94 0.73
//     epilogue, S      up to a round and a half 12 x 224 (56 spans) 1.25 1.03 0.94; in more, aligned 24 x 160 (40) 1.27 1.10 1.05, 16 x 256 (64)
//                      1.22 1.01 0.85 (in eights 1.16 1.15 1.09), else 26 x 128 (32) 1.25 1.04 0.97, 18 x 192 (48) 1.27 1.01 0.89 (1.16 1.11 1.10)
//     eights           aligned 8 x 512 (64) 1.13 1.13 1.07 (S 1.11 1.11 0.97); else 12 x 320 (40) 1.10 1.08 0.99 (S 1.10 1.05 0.94), 10 x 384 (48)
//                      1.10 1.06 0.96 (S 1.10 1.03 0.91)
inline int onepass_most_spans_in_rounds(const OnePassCall &p, int chunks) {
    const bool aligned = p.bh % 8 == 0;
    if (chunks == 8) return aligned ? 64 : 40;
    if (p.two_sided) return aligned ? 64 : p.bh * ((p.nchunks + 3) / 4) <= 512 ? 40 : 24;
    return p.bh * ((p.nchunks + 3) / 4) <= 768 ? 56 : aligned ? 40 : 32;
}

inline int onepass_chunks_per_group(const OnePassCall &p) {
    const int nchunks = p.nchunks, c = p.two_sided ? onepass_two_sided_chunks(p) : p.epilogue ? onepass_epilogue_chunks(p) : onepass_plain_chunks(p);
    if (c == 0 || nchunks <= c) return c;
    auto spans = [&](int chunks) { return (nchunks + chunks - 1) / chunks; };
    if (p.bh * spans(c) > onepass_resident(c, p.two_sided)) {
        if (p.bh < 8) return 0;
        if (spans(c) <= onepass_most_spans_in_rounds(p, c)) return c;
        const bool eights = c == 4 && !p.two_sided && p.bh * nchunks >= 2990 && p.bh * spans(8) <= 2 * onepass_resident(8, p.two_sided);
        return eights && spans(8) <= onepass_most_spans_in_rounds(p, 8) ? 8 : 0;
    }
    if (spans(c) <= onepass_most_spans(p, c)) return c;
    const bool eights = c == 4 && !p.two_sided && spans(4) <= kMaxChainedSpans && p.bh * spans(8) <= onepass_resident(8, p.two_sided);
    return eights && spans(8) <= onepass_most_spans(p, 8) ? 8 : 0;
}

// The span that a work-group takes, of all sequences' spans one behind the other.  Work-groups go to the eight XCDs in turn, and each XCD starts its own in
// the order of their numbers.  `ranges`: an XCD gets a contiguous eighth of the spans, so that what neighbours share comes from one L2.  The
// first spans of a range then look back at the last ones of the range before, which is well while all groups are resident, or where no sequence
// goes over from one range to the next; else those are a round away or more, and places on an XCD's units wait for them: up to a round and a half
// a few, in more all (forward call over that of two passes, z = 3, in ranges and with spans in the order of the work-groups: two-sided 18 x 62, 288
// groups, 1.12 and 1.01, 12 x 128, 384, 1.18 and 1.07, 18 x 96, 432, 0.95 and 1.12, 12 x 160, 480, 0.90 and 1.17, 126 x 16, 504, 1.14 and 1.56, 30 x 256
// 0.49 and 0.95; one gate 36 x 112, 504, 0.92 and 1.18, 12 x 320, 480, 0.88 and 1.08).  Whole sequences in order: 16 x 256 with slow gates 0.96, in ranges 1.08.
constexpr bool onepass_in_ranges(int bh, int spans, int resident) { return bh * spans <= resident * 3 / 2 || (bh & 7) == 0; }
constexpr int onepass_block(int block, int blocks, bool ranges) { return ranges && (blocks & 7) == 0 ? (block & 7) * (blocks >> 3) + (block >> 3) : block; }

// Whether the backward pass takes whole chunks although the forward call's states are there.  Forward and backward call, with the walks
// over spans cut for them and with these kernels: 6 x 100 61.8 and 58.2 us, 16 x 43 61.8 and 59.3, 32 x 32 68.9 and 66.5, 64 x 16 66.0 and
// 64.4, 64 x 10 56.9 and 56.0, but 64 x 6 46.5 and 50.6, 32 x 16 55.9 and 55.7 ([B,T,H,d] 32 x 13 55.5 and 64.4), 128 x 5 53.4 and 55.4;
// 32 / 64 channels: 32 x 24 53.4 and 50.3, 128 x 8 52.3 and 51.6, 6 x 75 58.4 and 54.6, but 64 x 10 46.1 and 48.1, 6 x 52 46.0 and 49.
inline bool onepass_back_with_states(const OnePassCall &p) {
    const long long nchunks = p.nchunks, total = p.bh * nchunks;
    return p.small ? total >= 720 || (nchunks >= 64 && total >= 400) : total >= 560 && nchunks >= 8;
}

// Whether the backward pass runs on the kernels that take whole chunks, four on a compute unit (`reuse`: the other kernels would
// find the forward states in the forward call's workspace).  Time of the walks over that of these (36 / 72 channels, sequences x
// chunks; S: 32 / 64 channels, R: with the forward call's states, that call included):
//     one span     16 x 4 1.40 (S 1.31, R 1.27), 256 x 4 1.26 (R 1.21), 512 x 4 1.13 (S 1.02), 16 x 3 1.20, 256 x 3 1.10, 320 x 3 0.98,
//                  two chunks and fewer leave waves idle: 16 x 2 0.97, 1 chunk 0.7
//     several      32 x 9 1.07 (S 0.89), 16 x 24 1.12 (S 1.04), 32 x 32 1.27, 16 x 64 1.30, 128 x 8 1.21, but 16 x 16 0.96 and 16 x 5
//                  0.87, where two launches are all there is (R: onepass_back_with_states)
//     more groups than compute units 0.6 to 0.98: what a group loads and stores has nothing beside it there
inline bool onepass_back_takes(const OnePassCall &p, bool reuse) {
    if (p.two_sided) return false;
    const long long bh = p.bh, nchunks = p.nchunks, total = bh * nchunks;
    if (nchunks <= 4) return nchunks == 4 ? bh <= 512 : nchunks == 3 && bh <= 256;
    return bh * ((nchunks + 3) / 4) <= 256 && (reuse ? onepass_back_with_states(p) : total >= (p.small ? 384 : 288));
}

// How the call is cut: chunks that a group holds (0: the call stays on the other kernels) and chunks of a span, of which a group takes one.
// What a group holds is the fastest for the forward call (64 x 24 24.1 us in spans of 8, 26.3 of 6).  Where the walks of the backward pass may
// follow, which go back over these spans, they are as short as leaves one group a compute unit (64 x 24, both calls: 81.6 us in spans of 6, 89.1
// of 8; 64 x 5 46.1 of 2, 54.9 of 4; S: 32 x 12 43.0 and 46.2), but not so many that looking back takes longer (S, both calls, z = 3: 3 x 128 63.4
// us in 64 spans of 2, 54.7 in 43 of 3; 1 x 320 in 107 of 3 and 46 of 7, forward call 29.6 and 22.3).  A few sequences where the two do not
// agree stay on the other kernels (S, z = 3: 2 x 192 63.4 us in 96 of 2, 60.0 in 48 of 4, 56.4 there; 3 x 400 86.9 in 50 of 8, 77.3 there).
struct OnePassPlan {
    int chunks, span;
};
inline OnePassPlan onepass_plan(const OnePassCall &p) {
    const int nchunks = p.nchunks, chunks = onepass_chunks_per_group(p);
    if (chunks == 0 || nchunks <= chunks) return {chunks, chunks > 0 ? nchunks : 0};
    const bool walks = !p.two_sided && !p.epilogue && p.bh <= 256 && !(chunks == 4 && onepass_back_with_states(p)) && !onepass_back_takes(p, true);
    if (!walks) return {chunks, chunks};
    auto cut = [&](int parts) { return (nchunks + parts - 1) / parts; };
    int span = cut((int)(256 / p.bh));
    span = span < 2 ? 2 : span < chunks ? span : chunks;                      // (spans of one chunk leave no room for the flags)
    if (chunks == 4 && span == 2 && cut(span) > 30) {
        if (p.bh > 5) return {0, 0};      // (S, z = 3: 6 x 63 in 32 spans of 2 49.7 us, in 21 of 3 51.9, 48.3 there)
        ++span;
    }
    if (chunks == 8 && p.bh == 1 && span < cut(48)) span = cut(48) < chunks ? cut(48) : chunks;
    if (cut(span) > (chunks == 4 ? 48 : onepass_most_spans(p, 8))) return {0, 0};
    return {chunks, span};
}

}  // namespace gla
