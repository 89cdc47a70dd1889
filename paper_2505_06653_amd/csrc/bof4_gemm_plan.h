// bof4_gemm_plan.h - how bof4_gemm takes a product on: its tiles' sizes, which kernel takes which shape, how its columns are
// split, where its chains of additions are cut, and the workspace that follows.  Host only and without the GPU's headers.
#pragma once
#include <cstddef>
#include <cstdint>
#include <initializer_list>

namespace bof4 {

constexpr size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

constexpr uint32_t GEMM_ROWS = 32;    // rows per tile (M of the matrix-core product)
constexpr uint32_t GEMM_MAX_R = 2;    // tiles of rows per workgroup: each word of x read serves up to 64 rows
constexpr uint32_t GEMM_TOKENS = 32;  // tokens per tile (N of the matrix-core product)
constexpr uint32_t GEMM_MAX_TILES = 4;  // token tiles per launch: the codes are decoded once per 128 tokens
constexpr uint32_t GEMM_CHUNK = 64;   // columns per wave and step: four products of K = 16
constexpr uint32_t GEMM_MAX_WAVES = 8;
constexpr uint32_t GEMM_MAX_COLS = 32768, GEMM_MAX_TOKENS = 65536;  // of a product; sizes are told for any
// Workgroups wanted before the columns are also split over workgroups: three quarters of the 256 compute units.
// Measured: splitting further (to 256, 512 or 1024 workgroups) costs more in partial results and in the epilogue per
// workgroup than the fuller chip gains; fewer than 192 leave too much of it idle.
constexpr uint32_t GEMM_TARGET_WGS = 192;
constexpr uint32_t GEMM_WIDE_WAVES = 8, GEMM_WIDE_TOK_TILES = 4;  // a row tile per wave; token tiles per workgroup
constexpr uint32_t GEMM_WIDE_MAX_SPLIT = 16;
constexpr uint32_t GEMM_TILE_WORDS = 4 * 64;                      // 16-byte words of one tile's bfloat16 operand

// Tiles of 32 rows per wave: with two, every word of x read serves 64 rows, at twice the accumulators.  Measured
// better for more than 32 tokens on all but small matrices, and for very large ones at any number of tokens.
inline uint32_t gemm_row_tiles_per_wg(uint64_t rows, uint64_t cols, uint64_t n_tokens) {
    return ((n_tokens > GEMM_TOKENS && (rows >= 8192 || cols >= 8192)) || rows * cols >= (1ull << 27)) ? 2 : 1;
}
inline uint64_t gemm_row_tiles(uint64_t rows) {  // in the packed matrix: a multiple of GEMM_MAX_R
    return (rows + GEMM_ROWS * GEMM_MAX_R - 1) / (GEMM_ROWS * GEMM_MAX_R) * GEMM_MAX_R;
}
// How many workgroups share the columns of their rows: the fewest that put GEMM_TARGET_WGS workgroups on the chip,
// each with at least one chunk per wave.
inline uint32_t gemm_split(uint64_t rows, uint64_t cols, uint64_t n_tokens) {
    const uint64_t groups = gemm_row_tiles(rows) / gemm_row_tiles_per_wg(rows, cols, n_tokens);
    const uint64_t chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK;
    uint64_t split = (GEMM_TARGET_WGS + groups - 1) / groups;
    const uint64_t most = chunks / GEMM_MAX_WAVES;
    if (split > most) split = most;
    return (uint32_t)(split < 1 ? 1 : split);
}

// Where gemm_wide_kernel takes the product over from gemm_kernel, and over how many workgroups it splits the columns: by a
// model of both kernels' times (us, from 21 shapes of 1 M to 470 M weights at 64 to 2000 tokens without a list, which it
// gives to 7 and 6 %).  gemm_kernel takes up to four token tiles per launch, gemm_wide_kernel whole groups of 128
// tokens at the same time for one token of a group as for 128; both go in rounds of 256 workgroups.  gemm_kernel / the wide
// kernel, measured:
//   2000 tokens: 4096 x 4096 261 / 100, 22016 x 4096 827 / 517, 8192 x 28672 1378 / 1219, 28672 x 512 309 / 138
//    640 tokens: 13824 x 5120 209 / 256 (two rounds), 8192 x 28672 430 / 405, 24576 x 6144 356 / 258
//    340 tokens: 22016 x 4096 152 / 168, 8000 x 1024 26 / 31, 10240 x 8192 160 / 99, 4096 x 4096 50 / 38
//    128 tokens: 10240 x 8192 60 / 46, 57344 x 8192 184 / 165, 22016 x 4096 55 / 56, 4096 x 4096 18 / 29
// With a list both take longer, gemm_kernel by some 10 % more:
//    128 tokens: 22016 x 4096 71 / 64, 4096 x 11008 42 / 36;  256 tokens: 12288 x 4096 75 / 65, 32000 x 4096 148 / 108
inline double gemm_kernel_time(uint64_t rows, uint64_t cols, uint64_t tok_tiles) {
    const uint64_t n_tokens = tok_tiles * GEMM_TOKENS, per_wg_tiles = gemm_row_tiles_per_wg(rows, cols, n_tokens);
    const uint64_t split = gemm_split(rows, cols, n_tokens), chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK;
    const uint64_t per_wg = (chunks + split - 1) / split, waves = per_wg < GEMM_MAX_WAVES ? per_wg : GEMM_MAX_WAVES;
    const double rounds = (double)((gemm_row_tiles(rows) / per_wg_tiles * split + 255) / 256);
    const double chain = (double)((per_wg + waves - 1) / waves);
    auto launch = [&](uint64_t nt) {  // start, sums and stores per tile, steps; the partial results at 4.7 TB/s
        const double step = per_wg_tiles == 2 ? 0.97 + 0.33 * (double)nt : 0.83 + 0.17 * (double)nt;
        return 3.0 + rounds * (0.7 * (double)(per_wg_tiles * nt) + chain * step) +
               (split > 1 ? 2.0 + (double)((split + 1) * nt * GEMM_TOKENS * rows) * 4.0 / 4.7e6 : 0.0);
    };
    return (double)(tok_tiles / GEMM_MAX_TILES) * launch(GEMM_MAX_TILES) +
           (tok_tiles % GEMM_MAX_TILES ? launch(tok_tiles % GEMM_MAX_TILES) : 0.0) + 3e-6 * (double)(n_tokens * cols);
}
struct GemmWideSplit {
    uint32_t split, per_split;  // workgroups along the columns, chunks each
    double time;                // with x reordered and the partial results added
};
inline GemmWideSplit gemm_wide_split(uint64_t rows, uint64_t cols, uint64_t tok_tiles) {
    const uint64_t tok_groups = (tok_tiles + GEMM_WIDE_TOK_TILES - 1) / GEMM_WIDE_TOK_TILES;
    const uint64_t groups = (rows + GEMM_WIDE_WAVES * GEMM_ROWS - 1) / (GEMM_WIDE_WAVES * GEMM_ROWS) * tok_groups;
    const uint64_t chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK, slots = tok_groups * GEMM_WIDE_TOK_TILES * GEMM_TOKENS;
    GemmWideSplit best = {1, (uint32_t)chunks, 0.0};
    for (uint64_t want = 1; want <= GEMM_WIDE_MAX_SPLIT && (want == 1 || want * 8 <= chunks); ++want) {
        const uint64_t per = (chunks + want - 1) / want, split = (chunks + per - 1) / per;
        const double sums = split > 1 ? (double)((2 * split + 1) * slots * rows) * 4.0 / 7e6 : 0.0;
        if (want > 1 && sums >= best.time) break;  // (more in every wider split)
        const double time = (double)((groups * split + 255) / 256) * (9.2 + 1.15 * (double)per) + sums;
        if (want == 1 || time < best.time) best = {(uint32_t)split, (uint32_t)per, time};
    }
    best.time += 3.5 + 0.8e-6 * (double)(tok_tiles * GEMM_TOKENS * cols);
    return best;
}
// The split where the wide kernel takes the product, else split = 0.  4 % and 1.5 us in hand for what the models do not
// know: of the 462 measured cases without a list the wide kernel is chosen where it is more than 1 % slower in one (1.4 %),
// of those with one in seven (14 % at most); the other kernel where that is more than 5 % slower in eight and seventeen.
inline GemmWideSplit gemm_wide_choice(uint64_t rows, uint64_t cols, uint64_t tok_tiles, bool list) {
    const GemmWideSplit narrow = {0, 0, 0.0};
    const uint64_t wg_rows = GEMM_WIDE_WAVES * GEMM_ROWS;
    const uint64_t tok_groups = (tok_tiles + GEMM_WIDE_TOK_TILES - 1) / GEMM_WIDE_TOK_TILES;
    if (cols < 512 || (rows + wg_rows - 1) / wg_rows * tok_groups >= (1ull << 23)) return narrow;  // 2^32 lanes a launch
    const GemmWideSplit wide = gemm_wide_split(rows, cols, tok_tiles);
    return 1.04 * wide.time + 1.5 < (list ? 1.1 : 1.0) * gemm_kernel_time(rows, cols, tok_tiles) ? wide : narrow;
}

// Where gemm_kernel reads x as it stands instead of in a copy reordered by a kernel of its own (3 us): tokens of one tile, and
// matrices so small that the launch is what counts - a wave's load then touches a line per token and not 8 in all -, or so
// few tokens that there are few lines.  Copy / in place, us:
//   up to 2^24 weights, 75 shapes: 1.07 to 1.4 times as fast at 8 and 16 tokens (4096 x 4096, 8 and 32 tokens 12.8 / 10.0, 12.9 /
//   10.7), at 32 too except where the second workgroup of a compute unit is there for some only: 257 to 330 workgroups and
//   14 M weights and more 0.88 to 0.95 (4160 x 4032, 3000 x 5568, 10000 x 1664), 376 1.02 and with a list 0.96, 10 M 1.1
//   above that, no list: 8 tokens 12288 x 4096 14.6 / 12.8, 28672 x 8192 42.2 / 37.4, 8192 x 28672 45.3 / 42.0, 57344 x 8192 1.00; with
//   one workgroup per compute unit, eight waves, the lines are waited for (8192 x 8192 15.3 / 16.9, 8192 x 12288 0.89, 8192 x
//   4096 1.01 - 1.14); 16 tokens 8256 x 4096 0.98, 32 tokens 12288 x 4096 0.69; with a list, 8 tokens 22016 x 4096 0.92
// (Turning whole lines into the products' order through LDS: 12288 x 4096, 8 / 32 tokens 14.7 / 16.3, 22016 x 4096 22.7 / 26.1.)
inline bool gemm_x_in_place(uint64_t rows, uint64_t cols, uint64_t n_tokens, bool list) {
    if (n_tokens > GEMM_TOKENS) return false;
    const uint64_t wgs = gemm_row_tiles(rows) / gemm_row_tiles_per_wg(rows, cols, n_tokens) * gemm_split(rows, cols, n_tokens);
    if (rows * cols <= (1ull << 24))
        return n_tokens <= 16 || wgs <= 256 || wgs >= 384 || rows * cols <= (3ull << 22);
    return !list && n_tokens <= 8 && rows >= 8192 && (wgs > 256 || cols <= 4096 || rows * cols >= (1ull << 27));
}

// Chunks in one chain of additions.  gemm_kernel: with a list half of what a wave takes, which holds its error to that of
// adding the entries apart where they carry half of the sums' energy (measured 0.94 to 1.04 of it over twelve shapes;
// 0.56 to 0.75 with the entries of Student-t weights).  Additions over more workgroups were that many more roundings, in
// binary32; in binary64 they leave room for a chunk more per two of them (per four in longer chains).
// The 256 x 128 tile: without a list and where gemm_kernel does not split the columns, sums of eight runs as long as its
// eight waves' lose what those lose.  Else the sums carry (without a list over a chunk more than gemm_kernel's waves take,
// whose own sums are rounded).
struct GemmChains {
    uint32_t waves, list_flush, n_runs;  // gemm_kernel
    uint32_t wide_flush;                 // gemm_wide_kernel, gemm_decoded_kernel
    bool wide_carry;
};
inline GemmChains gemm_chains(uint64_t rows, uint64_t cols, uint64_t n_tokens, bool list) {
    const uint32_t split = gemm_split(rows, cols, n_tokens);
    const uint32_t chunks = (uint32_t)((cols + GEMM_CHUNK - 1) / GEMM_CHUNK), per_wg = (chunks + split - 1) / split;
    GemmChains C;
    C.waves = per_wg < GEMM_MAX_WAVES ? per_wg : GEMM_MAX_WAVES;
    const uint32_t chain = (per_wg + C.waves - 1) / C.waves;  // that a wave of gemm_kernel takes, at most
    const uint32_t half_chain = chain > 3 ? chain / 2 : 1;
    C.list_flush = half_chain + (split - 1) / (chain > 3 ? 4 : 2);
    C.n_runs = list && chain > C.list_flush ? 2 : 1;
    C.wide_carry = list || split > 1;
    C.wide_flush = list ? half_chain + (split - 1) / 4 : C.wide_carry ? 1 + chain + (split - 1) / 4 : chain;
    return C;
}

// Where the matrix is decoded first (gemm_decode_kernel, gemm_decoded_kernel), in slabs of whole row groups of at most
// GEMM_DECODED_BYTES: what is decoded should still be in the 256 MB cache behind the L2s when it is multiplied (0.46 ps per
// weight to decode 180 MB, 0.9 for 300 MB and more).  By a model of its time (us; 15 shapes at 192 to 2500 tokens): on nine
// matrices of 16 M to 470 M weights it takes all products from 384 to 1056 tokens on with a list, 544 to 1568 without one,
// on large ones with some stretches before that (57344 x 8192 with a list: 544 to 768, then from 1056).  The other kernel / decoded first, measured:
//   with a list      4096 x 4096, 512 / 1000 / 2000 tokens 52 / 81 / 127 -> 49 / 71 / 102, 12288 x 4096 106 / 213 / 353 -> 90 /
//                    161 / 252, 22016 x 4096 215 / 331 / 649 -> 180 / 261 / 482, 8192 x 28672 320 / 648 / 1305 -> 371 / 573 / 1042
//   without a list   4096 x 4096, 512 / 1000 / 2000 tokens 45 / 67 / 103 -> 48 / 66 / 93, 12288 x 4096 86 / 174 / 286 -> 85 /
//                    151 / 236, 22016 x 4096 172 / 273 / 522 -> 162 / 239 / 442, 8192 x 28672 297 / 569 / 1185 -> 362 / 557 / 1020
constexpr uint64_t GEMM_DECODED_BYTES = 256ull << 20;
struct GemmDecodedPlan {
    uint32_t slab_tiles;        // row tiles per slab, 0: not this way
    uint32_t split, per_split;  // workgroups along the columns, chunks each
    double time;
    size_t slab_bytes;
    uint32_t flush;  // chunks in one chain of additions
    bool carry;
};
inline GemmDecodedPlan gemm_decoded_plan(uint64_t rows, uint64_t cols, uint64_t tok_tiles) {
    const uint64_t tok_groups = (tok_tiles + GEMM_WIDE_TOK_TILES - 1) / GEMM_WIDE_TOK_TILES;
    const uint64_t groups = (rows + GEMM_WIDE_WAVES * GEMM_ROWS - 1) / (GEMM_WIDE_WAVES * GEMM_ROWS);
    const uint64_t chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK, slots = tok_groups * GEMM_WIDE_TOK_TILES * GEMM_TOKENS;
    const uint64_t group_bytes = chunks * GEMM_WIDE_WAVES * GEMM_TILE_WORDS * 16, most = GEMM_DECODED_BYTES / group_bytes;
    const uint64_t least_slabs = (groups + most - 1) / most;
    GemmDecodedPlan best = {0, 0, 0, 0.0, 0, 0, false};
    for (uint64_t n_slabs = least_slabs; n_slabs <= least_slabs + 2 && n_slabs <= groups; ++n_slabs) {
        const uint64_t slab = (groups + n_slabs - 1) / n_slabs, last = groups - (n_slabs - 1) * slab;
        if ((n_slabs - 1) * slab >= groups) continue;
        for (uint64_t want = 1; want <= GEMM_WIDE_MAX_SPLIT && (want == 1 || want * 8 <= chunks); ++want) {
            const uint64_t per = (chunks + want - 1) / want, split = (chunks + per - 1) / per;
            const double sums = split > 1 ? 2.0 + (double)((2 * split + 1) * slots * rows) * 4.0 / 7e6 : 0.0;
            if (best.slab_tiles != 0 && sums >= best.time) break;  // (more in every wider split)
            const uint64_t rounds = (n_slabs - 1) * ((slab * tok_groups * split + 255) / 256) + (last * tok_groups * split + 255) / 256;
            const double time = sums + 4.0 * (double)n_slabs + (double)rounds * (7.5 + 0.82 * (double)per) +
                                (slab * group_bytes > (200ull << 20) ? 0.9e-6 : 0.46e-6) * (double)(rows * cols);
            if (best.slab_tiles == 0 || time < best.time)
                best = {(uint32_t)(slab * GEMM_WIDE_WAVES), (uint32_t)split, (uint32_t)per, time, (size_t)(slab * group_bytes), 0, false};
        }
    }
    best.time += 6.0 + 0.8e-6 * (double)(tok_tiles * GEMM_TOKENS * cols);
    return best;
}
// The plan where the product is decoded first, else slab_tiles = 0.  W: gemm_wide_choice's answer.
inline GemmDecodedPlan gemm_decoded_choice(uint64_t rows, uint64_t cols, uint64_t tok_tiles, bool list, const GemmWideSplit& W) {
    const GemmDecodedPlan no = {0, 0, 0, 0.0, 0, 0, false};
    const uint64_t wg_rows = GEMM_WIDE_WAVES * GEMM_ROWS, tok_groups = (tok_tiles + GEMM_WIDE_TOK_TILES - 1) / GEMM_WIDE_TOK_TILES;
    if (tok_groups < 2 || cols < 512 || cols > GEMM_MAX_COLS || (rows + wg_rows - 1) / wg_rows * tok_groups >= (1ull << 23)) return no;
    // (what carrying costs: 21 % of the wide kernel's time where a chain is four chunks, 11 % at eight)
    const GemmChains C = gemm_chains(rows, cols, tok_tiles * GEMM_TOKENS, list);
    const double flush = (double)C.wide_flush;
    const double other = W.split > 0 ? W.time * (list ? 1.0 + 0.85 / (flush < 3.0 ? 3.0 : flush) : 1.0)
                                     : (list ? 1.1 : 1.0) * gemm_kernel_time(rows, cols, tok_tiles);
    // (every plan's least: the decoding at its best rate and the products without what a round costs to start)
    const uint64_t chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK, groups = (rows + wg_rows - 1) / wg_rows;
    if (0.98 * (10.0 + 0.46e-6 * (double)(rows * cols) + 0.82 / 256.0 * (double)(groups * tok_groups * chunks)) >= other) return no;
    GemmDecodedPlan D = gemm_decoded_plan(rows, cols, tok_tiles);
    // The error stays that of the kernel which would take the product otherwise.  Where that is the wide tile with the columns
    // split alike, by the same additions.  Else the sums are carried, over chains no longer than that kernel's in the mean (with a
    // list gemm_kernel's are no shorter than wide_flush; it adds its waves' sums in binary64, so eight uncarried runs are 35 / 8
    // roundings more), a chunk shorter for every three workgroups more that share the columns.  Error over the other kernel's:
    // 12288 x 4096 with 700 tokens 1.10 if not carried, 13264 x 1632 with 562 1.29, 5970 x 23808 with 1065 and a list in two parts
    // 1.025 without the shorter chain; now 0.9 to 1.0, at 1 to 4 % more time.
    D.flush = C.wide_flush;
    D.carry = C.wide_carry;
    if (D.split != W.split) {
        const uint32_t split = W.split > 0 ? W.split : gemm_split(rows, cols, tok_tiles * GEMM_TOKENS);
        uint32_t chain = C.wide_flush;
        if (W.split > 0) chain = W.per_split / ((W.per_split + chain - 1) / chain);
        if (!list && W.split == 0) chain = (uint32_t)((chunks + split - 1) / split - 1) / C.waves;
        const uint32_t shorter = D.split > split ? (D.split - split + 2) / 3 : 0;
        D.flush = chain > shorter ? chain - shorter : 1;
        D.carry = true;
    }
    const double cost = list || (D.carry && (!C.wide_carry || W.split == 0)) ? 1.0 + 0.3 / (double)D.flush : 1.0;
    // Decoding first has to save 1 us and may be 2 % slower by the models, without a list and carried sums, where they are too
    // kind to it, has to save 3 %: of 82 such products measured from 0.98 on, other kernel / decoded first is 0.94 to 1.09
    // below 1.03 (28 of them, 1.01 in the mean; 28672 x 8192 with 1200 tokens 743 / 784 us) and 0.99 to 1.32 from there on.
    const bool kind = !list && !C.wide_carry && D.split >= W.split && W.split + D.split > 1;
    return (kind ? 1.03 : 0.98) * D.time * cost + 1.0 < other ? D : no;
}

// Workspace of bof4_gemm: x in the order of the products, then the partial results of the workgroups that share a row.
// gemm_kernel's lie behind `part`; the wide kernel's - all but the first part's, which goes to y - behind `wide_part`.
// `total` is what a call cannot do without and what gemm_kernel takes; it holds room for a second copy of x that only the
// wide kernel's partial results use (x transposed once stood there: buffers of that size are in use).
struct GemmWsLayout {
    size_t xp, part, wide_part, total;
    size_t decoded(uint64_t split, uint64_t n_tokens, uint64_t rows) const {  // behind the partial results of the 256 x 128 tile
        return align_up(wide_part + (split - 1) * n_tokens * rows * 4, 256);
    }
};
inline GemmWsLayout gemm_ws_layout(uint64_t rows, uint64_t cols, uint64_t n_tokens) {
    const uint64_t n_pad = (n_tokens + GEMM_TOKENS - 1) / GEMM_TOKENS * GEMM_TOKENS;
    const uint64_t chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK, split = gemm_split(rows, cols, n_tokens);
    const uint64_t per_launch = n_pad < GEMM_TOKENS * GEMM_MAX_TILES ? n_pad : GEMM_TOKENS * GEMM_MAX_TILES;
    GemmWsLayout L;
    L.xp = 0;
    L.wide_part = align_up(L.xp + n_pad * chunks * GEMM_CHUNK * 2, 256);
    L.part = align_up(L.wide_part + cols * n_pad * 2, 256);
    L.total = L.part + (split > 1 ? split * per_launch * rows * 4 : 0);
    return L;
}
// What bof4_gemm_workspace_bytes returns: enough for every kernel, with and without a list, at this and at every smaller token
// count that a product takes (the split falls as the token groups grow in number, so the largest need is not that of the most
// tokens).  Splits and slabs are the same for all token tiles of a group, so the most tokens of a group for which a kernel is
// chosen need the most: 8192 x 28672 at 2000 / 65536 tokens 29 us / 0.37 ms, 4096 x 4096 15 us / 0.18 ms (45 / 1500 and 30 / 1000
// where every token tile is asked about).
inline size_t gemm_ws_bytes(uint64_t rows, uint64_t cols, uint64_t n_tokens) {
    size_t need = gemm_ws_layout(rows, cols, n_tokens).total;
    const uint64_t most = n_tokens < GEMM_MAX_TOKENS ? n_tokens : GEMM_MAX_TOKENS;
    const uint64_t all_tiles = (most + GEMM_TOKENS - 1) / GEMM_TOKENS;
    for (uint64_t below = 0; below < all_tiles; below += GEMM_WIDE_TOK_TILES) {  // the token tiles before a group
        bool has_wide = false, has_decoded = false;
        for (uint64_t tiles = below + GEMM_WIDE_TOK_TILES < all_tiles ? below + GEMM_WIDE_TOK_TILES : all_tiles;
             tiles > below && !(has_wide && has_decoded); --tiles) {
            const uint64_t t = tiles * GEMM_TOKENS < most ? tiles * GEMM_TOKENS : most;  // the most tokens in them
            for (const bool list : {true, false}) {  // (which kernel is chosen depends on it, neither way the other's superset)
                const GemmWideSplit W = gemm_wide_choice(rows, cols, tiles, list);
                if (W.split > 0 && !has_wide) {
                    const size_t bytes = gemm_ws_layout(rows, cols, t).wide_part + (uint64_t)(W.split - 1) * t * rows * 4;
                    if (bytes > need) need = bytes;
                    has_wide = true;
                }
                if (has_decoded) continue;
                const GemmDecodedPlan D = gemm_decoded_choice(rows, cols, tiles, list, W);
                if (D.slab_tiles == 0) continue;
                const size_t bytes = gemm_ws_layout(rows, cols, t).decoded(D.split, t, rows) + D.slab_bytes;
                if (bytes > need) need = bytes;
                has_decoded = true;
            }
        }
    }
    return need;
}

// How a call is carried out with a workspace of ws_bytes (at least gemm_ws_layout's total): a smaller one gets the next
// kernel that it has room for, down to gemm_kernel.
enum GemmWay { GEMM_NARROW, GEMM_WIDE, GEMM_DECODED };  // gemm_kernel, gemm_wide_kernel, gemm_decoded_kernel
struct GemmPlan {
    GemmWay way;
    GemmWsLayout ws;
    GemmWideSplit wide;       // split = 0: not with the 256 x 128 tile
    GemmDecodedPlan decoded;  // slab_tiles = 0: not decoded first
    GemmChains chains;
    bool x_in_place;
};
inline GemmPlan gemm_plan(uint64_t rows, uint64_t cols, uint64_t n_tokens, bool list, size_t ws_bytes) {
    const uint64_t tok_tiles = (n_tokens + GEMM_TOKENS - 1) / GEMM_TOKENS;
    GemmPlan P;
    P.ws = gemm_ws_layout(rows, cols, n_tokens);
    P.wide = gemm_wide_choice(rows, cols, tok_tiles, list);
    P.decoded = gemm_decoded_choice(rows, cols, tok_tiles, list, P.wide);
    P.chains = gemm_chains(rows, cols, n_tokens, list);
    P.x_in_place = P.wide.split == 0 && gemm_x_in_place(rows, cols, n_tokens, list);
    P.way = GEMM_NARROW;
    if (P.decoded.slab_tiles > 0 && ws_bytes >= P.ws.decoded(P.decoded.split, n_tokens, rows) + P.decoded.slab_bytes)
        P.way = GEMM_DECODED;
    else if (P.wide.split > 0 && ws_bytes >= P.ws.wide_part + (uint64_t)(P.wide.split - 1) * n_tokens * rows * 4)
        P.way = GEMM_WIDE;
    return P;
}

}  // namespace bof4
