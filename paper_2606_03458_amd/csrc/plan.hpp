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
// head, head chunk) that are too few to fill the card; 0 where no plan writes partials.  Callers
// keep buffers of this size, so it is part of the interface; a plan takes fewer.
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

inline DecodePlan plan_decode(int batch, int n_kv, int n_q, int bits, int max_len, int n_sink, int max_blocks) {
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
    // The lines below were measured with 8 kv heads, every plan in turn; times in us at 2 bits, group
    // size 4 unless said otherwise; "ragged": lengths from a 16th to all of the tokens named.
    p.n_wg = 1;
    // More workgroups than CUs: the longest sequences go first, so that no long one starts when the
    // others are done (ragged 384 streams at 16k tokens: 58 -> 50).  Ranking a ragged batch costs a wave
    // up to 3 us, so only where a sequence may hold 32 tiles or more.
    p.order = streams > 256 && batch > 1 && batch <= kOrderBatch && nb >= 32;
    if (streams > 1024 || (streams > 768 && !(p.order && per_simd == 3))) {
        // enough streams to fill the card with one or two waves each (16k tokens: 1024 streams 231 /
        // 226 / 229 with 1 / 2 / 4 waves, 2048 streams 446 / 490 / 453; group size 5 276 / 244 / 246)
        p.group = 2 * streams <= 1024LL * per_simd ? 2 : 1;
    } else if (streams > 256) {
        // Four waves, one per SIMD, so that workgroups share a CU (512 streams, 1.1k tokens: 23 / 21 / 28
        // / 30 with 3 / 4 / 6 / 12 waves; groups that are not a multiple of four load the SIMDs
        // unevenly; ragged 1024 streams at 16k: 136 with 2, 101 with 4).  Long sequences of few streams
        // take a whole CU in turn (384 streams at 16k: 4 % slower where all are equally long, ragged 67
        // with 4 waves, 50 with 12), since a sequence then takes as long as its own tiles.
        p.group = streams <= 512 && nb * per_simd >= 192 ? per_cu : 4;
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
        const int n = std::min({(int)(256 * per_simd / std::max(streams, 1LL)), (units + 3) / 4, 32, p.ws_parts});
        if (n > 1 && units * (512 - 3 * streams) > 7680) {
            p.n_wg = n;
            p.group = 4;
        }
    }
    return p;
}

}  // namespace kvarn
