// How attention is split over workgroups and wavefronts (host side): which cross-attention sequences are cut into several
// work items, the list of items, and how many wavefronts an item's workgroup has.
#pragma once
#include <limits.h>

#include <algorithm>
#include <vector>

#include "kernels.h"

namespace aed {

// Float32 rows: one workgroup of 8 wavefronts fills a CU.  Up to so many of them, two rounds, longest first, come out even
// enough by themselves.
constexpr long long kF32TwoRounds = 512;

// no sequence is longer than 4/3 of the mean
inline bool even_lengths(long long total_keys, int longest_len, int batch) { return 3ll * longest_len * batch <= 4 * total_keys; }

// Cross-attention work items.  A sequence of more than `longest` keys is cut into pieces of about `piece` keys.
struct CrossCut { int longest, piece; };
// Which ones, from the batch's lengths and the bytes of a cached element (4: float32).  `share`: the keys of a CU if the
// batch's were dealt evenly, of two CUs in float32.
//  * Batches of more than 4096 are left whole: a CU has 32 workgroups and more then, and with the pieces a prompt pass's list
//    (kMaxPrefillPositions times as long) could pass what a launch grid holds in y.
//  * So are those of even lengths and of more than 96 (8-bit caches 48) and at most 256
//    workgroups: all of their sequences would be cut, and merging all of them takes longer than the idle CUs are worth.  24
//    layers, 8 heads of 128, us a launch, whole / cut by the last rule:
//      sequences           8            14           16           20           24            28            32
//      200 keys     5.96  5.95   6.22  7.05   6.28  7.13   6.52  7.83   6.92   8.08   7.26   8.83   7.73   9.14
//      350 keys     7.55  7.39   7.92  8.22   8.05  8.77   8.48  9.27   9.04  10.40   9.79  11.12  10.58  11.71
//      500 keys     9.02  8.42   9.50  9.55   9.68 10.54  10.22 11.46  11.05  12.21  12.19  14.30  13.35  15.34
//      300 to 500   8.76  7.94   9.20  9.06   9.20  9.38   9.65 10.31  10.10  11.15  10.99  12.69  11.81  13.09
//      12 to 500    8.54  6.98   8.99  8.00   8.89  7.38   9.07  8.00   9.24   8.50   9.84  10.24  10.05  10.21
//      8-bit, 200   5.29  5.80   5.44  6.78   5.48  6.88   5.63  7.55   5.78   7.81   5.92   8.36   6.12   8.52
//      8-bit, 500   7.05  7.87   7.31  8.89   7.45  9.29   7.58  9.88   7.97   9.92   8.47  11.31   8.98  11.73
//    Beyond 256 workgroups some CUs have two sequences and others one, and pieces even that out (36 of 350 keys 14.3 and 13.5).
//    Float32 rows are twice as long: 16 of 200 / 350 / 500 keys 11.0 and 9.9, 16.5 and 14.2, 22.5 and 18.7.
//  * Else sequences of more than 7/8 of a share are cut into pieces of half of that, at least 192 and 64 keys: one of 500 keys
//    among 31 / 127 of 40 8.9 and 5.9, 10.9 and 8.0; log-normal lengths (mean 115), batch 16 / 32 / 64 9.0 and 6.4, 9.4 and 6.9,
//    11.0 and 8.9; from batch 128 on little is cut (15.8 and 15.6).  Float32 is cut from 7/8 of two CUs' share up to kF32TwoRounds,
//    of one beyond: log-normal lengths, from two / one CU's share, batch 80 25.1 and 18.9, 96 26.9 and 21.0, 128 30.3 and 28.7; 12 to
//    500 keys, batch 40 22.4 and 25.9, 48 22.0 and 27.6, 64 29.9 and 32.3, 80 37.1 and 37.1.
constexpr CrossCut kWhole{INT_MAX, INT_MAX};
inline CrossCut cross_cut(long long total_keys, int longest_len, int batch, int n_heads, int kv_bytes) {
    const long long wgs = (long long)batch * n_heads;
    if (batch > 4096) return kWhole;
    if (kv_bytes <= 2 && wgs > 48 * kv_bytes && wgs <= 256 && even_lengths(total_keys, longest_len, batch)) return kWhole;
    const long long share = total_keys * n_heads / 256 * (kv_bytes == 4 ? 2 : 1);
    CrossCut c;
    c.longest = (int)std::min<long long>(std::max<long long>(192, (kv_bytes == 4 && wgs > kF32TwoRounds ? share / 2 : share) * 7 / 8), INT_MAX);
    c.piece = (int)std::min<long long>(std::max<long long>(64, share * 7 / 16 / 32 * 32), INT_MAX);
    return c;
}
inline int cross_pieces(int len, const CrossCut& c) {
    return len <= c.longest ? 1 : std::min(kMaxChunks, (len + c.piece - 1) / c.piece);
}
inline int piece_keys(int len, const CrossCut& c) {
    const int n = cross_pieces(len, c);
    return ((len + n - 1) / n + 15) / 16 * 16;
}
// most keys of an item of a sequence of len keys
inline int item_keys(int len, const CrossCut& c) { return std::min(len, piece_keys(len, c)); }
// the work items of sequence b of len keys, the first at frame first_frame of the packed layout
inline void add_items(std::vector<int4>& items, int b, int len, int first_frame, const CrossCut& c) {
    const int per = piece_keys(len, c), n = (len + per - 1) / per;
    for (int k = 0; k < n; ++k) {
        int4 it;
        it.x = b; it.y = (k * per) | (k << 16); it.z = std::min(per, len - k * per) | (n << 16); it.w = first_frame;
        items.push_back(it);
    }
}
// Cut sequences first, so that their merge is over when the rest is; then longest first.  Stable, so that the list is a
// function of the lengths alone.
inline void order_items(std::vector<int4>& items) {
    std::stable_sort(items.begin(), items.end(), [](const int4& p, const int4& q) {
        const bool pc = p.z >> 16 > 1, qc = q.z >> 16 > 1;
        return pc != qc ? pc : (p.z & 0xFFFF) > (q.z & 0xFFFF);
    });
}

// Whether cross-attention of a batch reads the frames (attn_frames.hip) instead of keys and values.
// Half the bytes per frame against two products per sequence and what a workgroup needs to begin and end; one workgroup per
// sequence, so the longest must not take longer than all together.  A whole step of 4 layers, us, keys and values / frames:
//   sequences         260           300           400           512           600           700          1000
//   100 frames     306   385    321   402    366   434    410   468    511   612    547   625    686    771
//   200            375   427    395   451    464   488    534   531    658   695    715   724    928    905
//   300            436   483    466   499    559   543    659   604    802   788    884   826   1168   1046
//   500            564   572    614   594    751   646    906   733   1090   953   1217  1006   1644   1284
//   12 to 500      414   459    433   485    518   538    617   593    748   734    814   774   1088    982
//   log-normal     324   460    340   476    396   513    438   546    556   661    599   680    765    819
// The batch's start computes and stores its keys and values all the same, for aed_read_cross_kv and kernel timing (1024 sequences of 500
// frames: 2.04 ms a layer); the figures are of steps alone.
constexpr int kFramesMinBatch = 288;
constexpr long long frames_min_keys(int batch) { return 140ll * batch + 60000; }
inline bool frames_attention(long long total_keys, int longest_len, int batch) {
    return batch >= kFramesMinBatch && total_keys >= frames_min_keys(batch) && 256ll * longest_len <= total_keys;
}

// Wavefronts per workgroup, 4 or 8, of a launch of wgs workgroups over caches of kv_bytes an element.  What counts is that
// every workgroup is resident from the start (4096 wavefronts fit the 256 CUs, of float32 rows 2048) and that a wavefront has
// a block or two to itself: with 8 wavefronts where 8 do not fit, a second round of workgroups starts when the first is over
// (self-attention, 24 layers, batch 128, 33 positions: 44.4 ms with 8, 42.9 with 4; batch 64 125.0 and 125.4 for 131), and
// wavefronts without a block still cost the merge (one utterance, cross- and self-attention on 16 and on 4: 92.6 and 90.1 ms).
// Items that are long on average (kLongItem) keep memory busy in two rounds as well, and 8 wavefronts are through with the last
// ones sooner (24 layers, batch 128 of 12 to 500 frames, half of whose sequences are through on average: 357 and 350 ms; us a
// launch on 4 / 8, batch 72 / 96 / 128: 12 to 500 keys 18.4 / 17.4, 20.0 / 18.0, 23.3 / 21.7; 100 to 400 17.5 / 15.8, 19.1 / 18.0, 22.9 /
// 22.0; 500 each 27.8 / 27.5, 32.0 / 32.0, 41.4 / 41.3; but 200 each 14.0 / 14.1, 15.5 / 16.0, 19.3 / 19.8).
// 16 are nowhere better than 8 (bfloat16, 8 heads of 128, us a launch on 16 / 8 / 4: cross-attention of 350 keys, batch 16 8.8 /
// 8.1 / 8.1, batch 32 11.4 / 10.6 / 10.3; 500 keys 11.3 / 9.7 / 10.1 and 15.1 / 13.3 / 13.4; self-attention over 440 positions,
// batch 16 8.4 / 7.9 / 7.8, batch 32 11.6 / 11.1 / 11.0; 4 heads of 64, 500 keys, batch 64 9.1 / 7.7 / 8.0): the keys of 8 are as
// many as a CU has under way, and the merge of 16 takes longer.
// Float32 cross-attention of uneven lengths has 8 up to kF32TwoRounds (sequence, head) pairs (us on 4 / 8: log-normal lengths,
// batch 48 16.5 and 14.3, 64 21.8 and 18.9; 12 to 250 keys, batch 48 16.4 and 13.8; but batch 128 of log-normal ones 29.8 and 31.1,
// 100 keys each, batch 64 12.4 and 13.6).
// Items of at most 64 keys are 4 blocks.  (Taken for as long as a sequence that is just not cut, they had 8: one utterance of
// 200 / 350 / 500 keys 5.18 / 5.27 / 5.40 us, 5.12 / 5.19 / 5.32 on 4; 8-bit caches, batch 16 of 200 keys 7.7 and 6.8.)
// pairs: of cross-attention sequences and heads, 0: self-attention; even: even_lengths of the batch.
inline int attn_wavefronts(long long wgs, long long pairs, int kv_bytes, int most_keys, bool long_items, bool even) {
    if (most_keys <= 64) return 4;
    if (kv_bytes == 4 && !long_items && !even && pairs > 256 && pairs <= kF32TwoRounds) return 8;
    const long long resident = kv_bytes <= 2 ? 4096 : 2048;
    return wgs * 8 > (long_items ? 2 * resident : resident) ? 4 : 8;
}

}  // namespace aed
