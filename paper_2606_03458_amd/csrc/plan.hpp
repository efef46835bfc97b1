// The launch plan of a decode: how a (sequence, kv head, head chunk) is split over workgroups and
// waves.  Host code only, from the sizes of a call alone, so that it can be looked at without a GPU.
#pragma once

#include <algorithm>

namespace kvarn {

constexpr int kG = 128;  // tokens per quantization group / body tile
constexpr int kRC = 32;  // bf16 tokens (sink / residual) per chunk
// Waves of one workgroup at most: one workgroup then fills a CU (three waves per SIMD for the
// 2-bit kernels of up to four heads, two for the others).
constexpr int kMaxGroup3 = 12, kMaxGroup2 = 8;
constexpr int kOrderBatch = 128;  // sequences that a wave ranks by length (two per lane)

struct DecodePlan {
    int n_chunk, g_chunk;  // query heads of a group taken in n_chunk chunks of up to g_chunk (<= 8)
    int n_wg, group;       // workgroups per (sequence, kv head, chunk) and waves per workgroup
    int order;             // 1: the longest sequences first
    int ws_parts;          // partials per query head that the workspace has room for (n_wg <= ws_parts or n_wg == 1)
};

// Partials per query head that kvarn_decode_workspace_bytes leaves room for: one for each share
// of at least two body tiles and one per sink or residual chunk, of the streams (sequence, kv
// head, head chunk) that are too few to fill the card.  Callers keep buffers of this size, so it is
// part of the interface; a plan takes fewer, at most 32, or none.  Where this is 0 it takes none.
inline int workspace_parts(long long streams, int nb, int max_len, int n_sink, int per_simd) {
    const long long slots = 1024LL * per_simd;
    if (streams * 4 >= 1024) return 0;
    const int want = (int)std::min<long long>((slots + streams - 1) / streams, nb / 2);
    if (want < 2) return 0;
    const int bps = (nb + want - 1) / want, body = (nb + bps - 1) / bps;
    const int chunks = (std::min(n_sink, std::max(max_len, 0)) + kRC - 1) / kRC + kG / kRC;
    const int parts = body + (streams * (body + chunks) <= slots ? chunks : streams * (body + 1) <= slots ? 1 : 0);
    return parts <= 4 ? 0 : parts;
}

// equal: the sequences are known to be equally long (a lock-step step); else any of them may be up to
// max_len.
inline DecodePlan plan_decode(int batch, int n_kv, int n_q, int bits, int max_len, int n_sink, int max_blocks, bool equal) {
    DecodePlan p;
    const int nb = std::min(max_len > n_sink ? (max_len - n_sink) / kG : 0, max_blocks);
    const int g = n_kv > 0 ? n_q / n_kv : 1;
    // Groups above 8 query heads go to the kernels in chunks of at most 8 heads (as even as
    // possible); the chunks of a stream read the same tiles.
    p.n_chunk = (g + 7) / 8;
    p.g_chunk = (g + p.n_chunk - 1) / p.n_chunk;
    const long long streams = (long long)batch * n_kv * p.n_chunk;
    const int per_simd = bits == 2 && p.g_chunk <= 4 ? 3 : 2, per_cu = 4 * per_simd;
    p.ws_parts = workspace_parts(streams, nb, max_len, n_sink, per_simd);
    const int units = nb + (std::min(n_sink, std::max(max_len, 0)) + kRC - 1) / kRC + kG / kRC;
    // Waves per workgroup: a CU holds per_cu waves, and a workgroup merges its waves' parts in LDS.
    // The lines below were measured with 1 and 8 kv heads, every plan in turn; times in us at 2 bits, group
    // size 4 unless said otherwise; "ragged": lengths from a 16th to all of the tokens named.  A rule that
    // is there for ragged batches leaves equally long ones no slower than the plan of at most four waves over
    // fixed spans that these rules replaced, and the other way round ("before").
    p.n_wg = 1;
    // More workgroups than CUs: the longest sequences go first, so that no long one starts when the
    // others are done (ragged 384 streams at 16k tokens: 58 -> 50).  Ranking a ragged batch costs a wave
    // up to 3 us, so only where a sequence may hold 32 tiles or more.  A wave ranks two sequences per lane;
    // larger batches go as they come, and lose what ranking gains (832 ragged streams at 8k: 49 -> 46 and
    // 54 -> 47 of two draws).
    p.order = !equal && streams > 256 && batch > 1 && batch <= kOrderBatch && nb >= 32;
    const long long round = 1024LL * per_simd;  // waves that the card holds
    if (streams >= round) {
        p.group = 1;  // a round of waves and more: nothing to share
    } else if (streams > 1024 || (streams > 768 && 2 * streams <= round)) {
        // One wave leaves the longest sequences of a ragged batch alone on the card, and two the second round
        // nearly empty, so four from 16 tiles on (ragged 8k tokens: 1792 streams 142 / 110 / 97 with 1 / 2 / 4
        // waves, equal 206 / 213 / 202, before 120 and 219; 4 bits, 1152 streams: ragged 128 / 115 / 102, before
        // 113).  Below that the waves' set-up and merge count for more than they share (in a
        // step below 32: 2560 streams at 2k 89 / 93 with 1 / 4).  Where two waves per
        // stream fit the round they are as good on equal lengths (16k tokens, 1024 streams: 226 with 2, 229 with
        // 4), and four only pay at three waves per SIMD and well off the round's end (ragged 1024 streams at
        // 16k: 136 with 2, 101 with 4; 1536 at 8k, equal: 171 and 174).
        if (2 * streams <= round)
            p.group = per_simd == 3 && (streams <= 1024 ? nb >= 32 : streams <= 1472 && nb >= 16) ? 4 : 2;
        else
            p.group = nb >= (equal ? 32 : 16) || (per_simd == 2 && streams <= 1280 && nb >= 4) ? 4 : 1;
    } else if (streams > 256) {
        // Four waves, one per SIMD, so that workgroups share a CU (512 streams, 1.1k tokens: 23 / 21 / 28
        // / 30 with 3 / 4 / 6 / 12 waves; groups that are not a multiple of four load the SIMDs
        // unevenly).  Long sequences of few streams take a whole CU in turn where they may be ragged, since a
        // sequence then takes as long as its own tiles (384 streams at 16k: ragged 67 with 4 waves, 50 with
        // 12), unless the second round of workgroups is nearly empty: equally long ones at 16k then take
        // longer than before (264 streams: 87 / 96 with 4 / 12 waves, before 93; 328 at 33k, compact aux: 154 /
        // 166, before 159; not so at two waves per SIMD, 4 bits, 264: 144 / 150, before 151).
        const int whole_cu_from = per_simd == 3 ? 352 : 256;
        p.group = !equal && streams > whole_cu_from && streams <= 512 && nb * per_simd >= 192 ? per_cu : 4;
    } else {
        // A CU or more per stream.  Few units: eight waves of one or two units each (8 streams, 1k
        // tokens: 9.5 / 7.9 / 8.8 with 4 / 8 / 12 waves); more: all the CU's waves (2k tokens: 12.4 /
        // 10.2 / 10.0).
        p.group = units <= 16 ? std::min(8, units) : per_cu;
        // Several workgroups of four waves per stream, as many as fill the card with waves or leave
        // each a unit per wave: they cost a merge launch (about 4 us) and pay by the units they take off the
        // CU, less what the card's memory rate then allows (8 streams: 2k tokens 10.0 alone and shared,
        // 4k 15.1 and 11.0; 64 streams: 4k 15.4 and 14.3, 8k 24.8 and 17.6; 128 streams: 4k 15.8 and 17.9, 8k
        // 25.4 and 24.2, ragged 24.0 and 19.3; 192 streams: 8k 28.2 and 33.4).
        bool share = units * (512 - 3 * streams) > 7680;
        int n = (int)(256 * per_simd / std::max(streams, 1LL));
        // A ragged batch of more streams leaves the CUs of its short ones idle, and pays by that, with four
        // workgroups (group size 8, 192 streams at 33k tokens: 120 alone, 75 shared, before 102, equal 129 and
        // 117; 4 bits, 176 streams: 108 and 74, before 92, equal 138 and 144, before 173).
        if (!equal && !share && units * ((per_simd == 3 ? 256 : 264) - streams) > 3072 * per_simd) {
            share = true;
            if (streams > 170) n = 4;
        }
        n = std::min({n, (units + 3) / 4, 32, p.ws_parts});
        if (n > 1 && share) {
            p.n_wg = n;
            p.group = 4;
        }
    }
    return p;
}

}  // namespace kvarn
