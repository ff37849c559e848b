// Host side of the chunk-parallel backward schedules: how a workspace is divided and which calls they take.
#pragma once
#include <stddef.h>

#include <algorithm>

#include "sla.h"
#include "sla_gdn_block.h"

namespace sla {

constexpr int kChunkTokens = 64;  // tokens per chunk

inline size_t chunk_round4(size_t n) { return (n + 3) & ~(size_t)3; }

// ---- RetNet and GLA (sla_chunk_backward.hip)

// The parts a call is worked off in, one after the other: whole heads of nb sequences or nh heads of one.  Packed batches:
// nh heads of all sequences.
struct ChunkParts {
    int nb, nh, slots;  // of a part; slots: chunks per head
    size_t floats;      // of its states, both directions
};
inline ChunkParts chunk_parts(const sla_params& p, bool packed, size_t budget) {
    const int nchunk = (p.T + kChunkTokens - 1) / kChunkTokens, all = p.T / kChunkTokens + p.B + 1;
    const size_t per = (size_t)p.dk * p.dv;  // two bf16 states
    ChunkParts r;
    if (packed) {
        r.nb = p.B;
        r.slots = all;
        r.nh = (int)std::min<size_t>(p.H, std::max<size_t>(1, budget / (per * all)));
    } else {
        const size_t heads = std::max<size_t>(1, budget / (per * nchunk));
        r.nh = (int)std::min<size_t>(p.H, heads);
        r.nb = r.nh == p.H ? (int)std::min<size_t>(p.B, heads / p.H) : 1;
        r.slots = r.nb * nchunk;
    }
    r.floats = (size_t)r.slots * r.nh * per;
    return r;
}

// Floats of states a part may hold: as many as the workspace has room for, of which the query asks for no more than
// kMostStates and the call is content with kLeastStates.  Large parts are better: B=6 T=5690 H=8 128 x 256 RetNet takes
// 498 us in parts of 1 GiB, 746 in parts of 128 MiB (a launch ends with a partly filled chip, and the intermediate states'
// stay in the memory-side cache gains less than that); below kLeastStates launches are too small to fill the chip at all.
constexpr size_t kMostStates = (size_t)1 << 28, kLeastStates = (size_t)1 << 24;

// Gates and their gradients [B,T,H], and behind the states Args::end.
inline size_t backward_chunks_fixed_floats(const sla_params& p, bool packed) {
    return 4 * chunk_round4((packed ? (size_t)p.T : (size_t)p.B * p.T) * p.H);
}
inline size_t backward_chunks_end_floats(const sla_params& p) {
    return p.variant == SLA_GLA ? (size_t)p.B * p.H * p.dk * (p.dv / 32) : 0;
}
// How a workspace of that many floats is used: Args::end and as many states as there is room for, kMostStates of them at most.
inline ChunkParts backward_chunks_parts(const sla_params& p, bool packed, size_t floats) {
    const size_t taken = backward_chunks_fixed_floats(p, packed) + backward_chunks_end_floats(p);
    return chunk_parts(p, packed, floats > taken ? std::min(kMostStates, floats - taken) : 0);
}
inline size_t backward_chunks_floats(const sla_params& p, bool packed, const ChunkParts& parts) {
    return backward_chunks_fixed_floats(p, packed) + backward_chunks_end_floats(p) + parts.floats;
}
inline size_t backward_chunks_workspace_floats(const sla_params& p, bool packed) {
    return backward_chunks_floats(p, packed, chunk_parts(p, packed, kMostStates));
}
// Whether a call runs chunk-parallel in a workspace of that many floats: they have to be enough, and the schedule has to be
// faster than what runs otherwise, nseg segments or (nseg == 1) the sweeps in one pass.  A part's states are carried over the
// chunks one after another, 0.65 us a chunk (RetNet) or 1.15 (GLA) whatever the number of heads, which is what it loses by on
// long rows with few heads; it wins by 0.6 and 0.9 ns a token and head of 128 x 128, and by the segments' launches.
//     us, segments -> chunks, B=1 128 x 128      T=4096       8192       16384      32768
//         RetNet H=2                              97 ->  65  106 -> 108  123 -> 197  167 -> 376
//                H=8                             111 ->  76  155 -> 135  235 -> 264  435 -> 572
//                H=16                            151 ->  93  231 -> 179  430 -> 393  819 -> 781
//         GLA    H=2                             115 -> 105  128 -> 181  148 -> 338  205 -> 661
//                H=8                             130 -> 111  185 -> 204  301 -> 404  571 -> 830
//                H=16                            179 -> 137  296 -> 270  567 -> 541 1081 -> 1066
//     and in parts: GLA B=1 T=16384 H=32 8 segments 1110 -> 2104 (8 parts), B=8 T=4096 H=4 128 x 256 543 -> 498 (4).
// Against the sweeps, whose own walk takes 8 us in place of a chunk's, a few parts are no matter where those leave compute
// units idle (RetNet B=4 T=8192 H=16 1027 -> 538 in one part, 562 in four, 1202 in 16); where they fill the chip a part costs
// its walk (B=16 T=4096 H=16: 1187 -> 1067, 1107 in four parts, 1601 in 16; GLA 1555 -> 1503, 1580 in two).
inline bool backward_chunks_take(const sla_params& p, bool packed, int nseg, size_t floats) {
    if (p.dtype != SLA_BF16 || p.T == 0 || p.B == 0) return false;
    const size_t least = backward_chunks_fixed_floats(p, packed) + kLeastStates;
    if (backward_chunks_floats(p, packed, backward_chunks_parts(p, packed, least)) > floats) return false;
    if (p.dk < 64) return true;  // the others run them on copies padded to 64 (GLA B=1 T=16384 H=8 32 x 64 1997 -> 210 us)
    const bool gla = p.variant == SLA_GLA;
    const double heads = (double)p.B * p.H * p.dk * p.dv / (128. * 128.);  // of 128 x 128
    const int64_t rows = (int64_t)p.B * p.H;
    // Sequences of a 16-token block: the sweeps do one step of their walk, a chunk all its work.  That is slower for numbers
    // that fill the chip about once, and GLA's kernel pays for it in larger numbers too, but for keys of 128 with up to 128 values.
    // Packed, 3 and 14 tokens each, H=8, sweeps -> chunks:
    //     GLA     64 x 128   32 sequences 30 -> 34, 31 -> 34   64 34 -> 50, 36 -> 50   256 92 -> 109, 104 -> 109   1024 327 -> 367, 377 -> 381
    //             128 x 128  16 31 -> 32, 31 -> 34   64 54 -> 68, 58 -> 65   128 94 -> 99, 103 -> 98   256 172 -> 164, 199 -> 168
    //             128 x 256  16 31 -> 42, 32 -> 47   64 69 -> 91, 77 -> 91   256 235 -> 260, 278 -> 266   1024 917 -> 1027, 1088 -> 1114
    //     RetNet  64 x 256   16 25 -> 27, 26 -> 28   64 35 -> 48, 38 -> 43   128 58 -> 63, 63 -> 61   256 102 -> 95, 118 -> 101
    //             128 x 128  16 25 -> 27, 25 -> 28   32 29 -> 35, 31 -> 35   64 46 -> 52, 50 -> 47   128 80 -> 67, 87 -> 65
    if ((packed ? (int64_t)p.T <= (int64_t)16 * p.B : p.T < 16) && heads >= 128. &&
        (gla ? p.dk == 64 || p.dv == 256 || rows < 1536 : rows < (p.dk == 64 ? 1536 : 768)))
        return false;
    const ChunkParts parts = backward_chunks_parts(p, packed, floats);
    const int64_t count = ((int64_t)p.B + parts.nb - 1) / parts.nb * (((int64_t)p.H + parts.nh - 1) / parts.nh);
    if (nseg > 1) return (double)((p.T + kChunkTokens - 1) / kChunkTokens) * (count - heads / (gla ? 20. : 24.)) <= (gla ? 58. : 90.);
    if (rows * std::min(p.dk, p.dv) / 64 < 240) return count <= 4;
    // RetNet's 64 x 256 keeps states as large as the rows they stand for.  Where the sweeps fill the chip in every round it loses on
    // all but short rows: B=16 H=16 T=448 139 -> 131, T=576 169 -> 179, T=1024 305 -> 328; two rounds, B=32, T=704 444 -> 437,
    // T=2500 1517 -> 1595; one and a quarter, B=20, T=1024 470 -> 394.
    if (!gla && !packed && p.dk == 64 && p.dv == 256) {
        const int64_t rounds = (rows + 255) / 256;
        if (16 * rows >= 15 * 256 * rounds && p.T >= (rounds == 1 ? 576 : 1024)) return false;
    }
    return (double)(count - 1) <= heads / (gla ? 400. : 92.);
}

// ---- delta rule (sla_chunk_gdn.hip)

struct GdnChunkSizes {
    size_t rows, n, slots, state, rest, wide, ends;  // n: floats of a [rows,H] array; state: of S or X; wide: of res, half of du
    size_t floats;
};
inline GdnChunkSizes gdn_chunk_sizes(const sla_params& p, bool packed) {
    GdnChunkSizes z;
    z.rows = packed ? (size_t)p.T : (size_t)p.B * p.T;
    z.n = chunk_round4(z.rows * p.H);
    z.slots = packed ? (size_t)p.T / kGdnChunk + p.B + 1 : (size_t)p.B * ((p.T + kGdnChunk - 1) / kGdnChunk);
    z.state = z.slots * p.H * p.dk * p.dv / 2;
    z.wide = z.rows * p.H * p.dv / 2;
    z.rest = gdn_anchor_count(z.rows) * p.H * p.dk * p.dv / 2;
    z.ends = gdn_anchor_count(z.rows) * p.H * (kGdnAnchor / kGdnChunk) + (size_t)p.B * p.H * (p.dv / 16);
    z.floats = 5 * z.n + z.ends + 2 * (z.state + z.rest) + 3 * z.wide + gdn_pair_workspace_floats(p.B, p.T, p.H, packed);
    return z;
}

// Where the sweeps have a workgroup for each of 256 compute units in every round, or nearly, the schedules are close, and heads
// of 256 values are cheaper in the sweeps (the chunk kernel takes 256 registers for them, and spills).  Backward call, us,
// sweeps -> chunks:
//     128 x 256  B=6 H=16 T=1024 389 -> 371   B=7 403 -> 445   B=8 415 -> 500   B=10 663 -> 587   B=12 674 -> 699   B=16 839 -> 948
//                B=7 T=256 140 -> 120         B=8 T=512 225 -> 258              32 packed rows of 256 488 -> 524
//     64 x 256   B=16 H=16 T=1024 618 -> 645  B=24 951 -> 894  B=32 1220 -> 1229
//     128 x 128  B=8 H=15 T=2048 492 -> 468   B=8 H=16 489 -> 500, T=1024 261 -> 251, T=4096 942 -> 940; two rounds, B=16 T=4096
//                1873 -> 1790, three, B=24 T=2048, 1426 -> 1343
//     others     64 x 128 B=8 H=32 T=2048 749 -> 703, 128 x 64 B=16 H=16 T=4096 1261 -> 1158, 64 x 64 B=16 942 -> 821
inline bool gdn_sweeps_are_faster(const sla_params& p, bool packed) {
    const int64_t cus = 256, wgs = (int64_t)p.B * p.H * std::min(p.dk, p.dv) / 64, rounds = (wgs + cus - 1) / cus;
    const int64_t mean = packed ? p.T / p.B : p.T;  // tokens of a sequence
    if (p.dv == 256 && p.dk == 128) return mean >= (rounds > 1 ? 256 : 384) && 16 * wgs >= 12 * cus * rounds;
    if (p.dv == 256) return !packed && mean >= 256 && 16 * wgs >= 15 * cus * rounds;
    return !packed && p.dk == 128 && p.dv == 128 && mean >= 1536 && wgs <= cus && 32 * wgs > 31 * cus;
}

// 0: this call does not run chunk-parallel (heads of width 32 are padded by sla_backward_narrow.hip, which runs the sweeps).
// Its states may take a GiB, as in sla_chunk_backward.hip.
inline size_t backward_gdn_chunks_workspace_floats(const sla_params& p, bool packed) {
    if (p.dtype != SLA_BF16 || p.dk < 64 || p.T == 0 || p.B == 0 || gdn_sweeps_are_faster(p, packed)) return 0;
    const GdnChunkSizes z = gdn_chunk_sizes(p, packed);
    return 2 * z.state <= (size_t)1 << 28 ? z.floats : 0;
}

}  // namespace sla
