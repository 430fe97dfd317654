// launch_rules.hpp -- the rules that choose a kernel or cut its work from a call's sizes, in
// plain C++ (no HIP), so that they can be checked over the whole range of the sizes that the
// entry points accept. Sizes are valid arguments: S = 64 / G queries side by side in a wave
// (G component lanes each, a power of two from 4 to 64), ns >= 1 draws per query.
#pragma once

#include <cstdint>

namespace sdmm {

// Whether the draws of a wave's S queries fit its 64 lanes, one draw each (the lanes
// kernels' phase B). ns has no upper limit, so ns * S may not fit 32 bits.
constexpr bool lanes_fit(int S, int ns) { return ns <= 64 / S; }

// rounds of S queries whose draws share one pass of the 64 lanes, at most `most`; for calls
// that lanes_fit
constexpr int rounds_per_pass(int S, int ns, int most)
{
    const int fit = 64 / (S * ns);
    return fit < most ? fit : most;
}

// Whether separate draws (conditioned before) run on the lanes kernel. It scans a query's
// CDF once for its draws and draws on all lanes, but reads the picked component's row once
// more per draw. With two draws or more that pays from a table that fits one XCD's L2
// (4 MB): 400,000 queries of 16 components in random order, 2 draws 48-53 us, 79-80 by the
// group kernel, 4 draws 56-59 and 152. With one draw it costs up to a third in random
// order (1M queries of 4 components 48.0 against 35.9 us, of 32 288 and 231) and gives 13%
// at most in the order of the cells, which the host doesn't know. From a larger table those
// reads leave the L2 (500,009 queries of one draw, 8 MB: 79.9 against 61.7 us).
constexpr bool sample_by_lanes(int S, int ns, int64_t table_bytes)
{
    return ns >= 2 && lanes_fit(S, ns) && table_bytes <= (4 << 20);
}

// batches of G draws of a query, the last of what is left (a counter that advances by G
// would pass 2^31 where ns is within G of it, and never end)
constexpr int draw_batches(int ns, int G) { return ns / G + (ns % G != 0 ? 1 : 0); }

constexpr int kLanesRounds = 4;  // most rounds of S queries per pass of the query kernels

// wave groups below which the passes of a launch take fewer rounds (four waves per SIMD, so
// that a small call spreads out)
constexpr int64_t kFewGroups = 4096;

// Whether the condition and pdf kernels take kRounds rounds of S items per wave pass, all their
// loads ahead (else one). That pays where the rows miss the L2: 16 components, 524,288
// queries in random order over 8192 cells 71.4 against 73.2 us, over 2048 35.0 against 37.2; in
// the order of the cells it is level (35.1 against 34.8). Below 16 wave groups per SIMD the
// longer passes even out badly (pdf of 85,000 to 110,000 directions up to 10% slower), and
// the pdf of groups of 4 lanes loses up to 7% at any size.
constexpr int kRounds = 4;
constexpr int64_t kRoundsGroups = 16384;
constexpr bool condition_in_rounds(int S, int64_t nq) { return nq >= kRoundsGroups * S * kRounds; }
constexpr bool pdf_in_rounds(int S, int64_t items) { return S <= 8 && items >= kRoundsGroups * S * kRounds; }

// rounds of the query kernels' passes: as many as fill the lanes, at most kLanesRounds (more
// take the LDS of one wave less per SIMD: 4% slower in path order), fewer where the call is
// too small to give every SIMD four waves of that many
constexpr int lanes_rounds(int64_t nq, int S, int ns)
{
    int nqr = rounds_per_pass(S, ns, kLanesRounds);
    while (nqr > 1 && nq < kFewGroups * S * nqr) nqr >>= 1;
    return nqr;
}

// Whether a product pdf call stages the BSDF components of kStagedQueries queries per wave
// pass. It needs passes enough to hide a second chain of loads and to even out the last
// ones, which a query's directions lengthen: time against the unstaged kernel, worst and best
// of 1 to 16 directions per query in random order and in that of the cells, at 131,072
// queries of 16 components 0.96 to 1.15, at 262,144 0.88 to 1.02, at 400,000 0.90 to 1.02,
// at 1.5 M 0.82 to 0.85; of 32 components 0.91 to 1.14, 0.86 to 1.01, 0.85 to 1.01 and 0.80 to
// 0.84; of 64 (32 rounds a pass) 0.94 to 1.25, 0.90 to 1.35, 0.89 to 0.94 and 0.79 to 0.80. Of
// up to 8 components the lanes that rotate in vain are few: 8 take 0.94 to 1.08 from
// 262,144 queries on, 4 take 0.97 to 1.11, so these never stage.
constexpr int kStagedQueries = 32, kStagedGroup = 16;
constexpr bool staged_pdf(int G, int64_t nq) { return G >= kStagedGroup && nq >= (G == 64 ? 400000 : 262144); }

// The chunks (work items) of a leaf of a tree refinement: `count` records, up to 2^31 - 1,
// in chunks of at most `most` (a multiple of 64), all of one size, a multiple of 64, but the
// last, which takes what is left. Nothing here may add to a count before it divides: a leaf
// within a chunk of 2^31 records would leave 32 bits.
constexpr int32_t chunks_of(int32_t count, int32_t most) { return count / most + (count % most != 0 ? 1 : 0); }

constexpr int32_t chunk_size(int32_t count, int32_t n_chunks)
{
    return (count / n_chunks + (count % n_chunks != 0 ? 1 : 0) + 63) & ~63;
}

// records [begin, end) of chunk q < n_chunks = chunks_of(count, most)
constexpr int32_t chunk_begin(int32_t count, int32_t n_chunks, int32_t q)
{
    const int32_t at = q * chunk_size(count, n_chunks);
    return at < count ? at : count;
}

constexpr int32_t chunk_end(int32_t count, int32_t n_chunks, int32_t q)
{
    const int32_t begin = chunk_begin(count, n_chunks, q), size = chunk_size(count, n_chunks);
    return count - begin < size ? count : begin + size;
}

}  // namespace sdmm
