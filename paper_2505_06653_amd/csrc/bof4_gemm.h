// bof4_gemm.h - the decoder inside a matrix product for many tokens (the paper's inference path decodes the matrix to
// bfloat16 and multiplies in bfloat16; section 2.1 eq. 3, outliers of section 3.3):
//
//   y[t][r] = sum_c W^[r][c] x[t][c],   W^ = bfloat16(m_b * level[code]), outliers as stored - what bof4_dequantize
//   returns, never written to memory.
//
// The codes are still read once (0.5 + 2/I bytes per weight) and decoded once per 32 tokens, so per weight the cost is
// that of the matrix-vector kernel (extract, look the level up, one multiply, one conversion); the 32 multiply-adds
// per weight that follow are a dense contraction and go to the matrix cores: v_mfma_f32_32x32x16_bf16, A = 32 rows x
// 16 columns of decoded weights, B = the same 16 columns of 32 tokens, binary32 accumulators; up to four tiles of
// 32 tokens share one decoded A.  Codes, constants and x are read in that order from copies laid out for it (the
// matrix once, x per call unless it is small), so that every load of a wave is one run of consecutive bytes.  Lane l supplies
// row l % 32 of A and token l % 32 of B, eight consecutive columns each; which eight is the same for both (half
// l / 32 of a 64-column chunk takes its columns 32 (l / 32) + 8 j .. + 7 in the j-th of four products), so a lane
// decodes one 16-byte load of its row per chunk.
// A workgroup owns 32 or 64 rows (one or two tiles per wave: with two, every word of x read serves both); its waves
// take the 64-column chunks in turn and their 32 x 32 partial results are added in wave order through LDS.
// Outliers: the list, sorted once per matrix into the products' tiles (32 rows x 64 columns), overwrites the decoded
// placeholders on their way into the product, so it costs the same for one token and for 128.  When the columns of a
// matrix with few rows are split over several workgroups to fill the chip, a second small kernel adds their partial
// results.  Every order is fixed: the result is bit-reproducible.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "bof4_device.h"
#include "bof4_segment.h"
#include "bof4_gemv.h"
#include "bof4_gemm_plan.h"

namespace bof4 {

typedef __bf16 gemm_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 gemm_bf16x2 __attribute__((ext_vector_type(2)));
typedef float gemm_f32x2 __attribute__((ext_vector_type(2)));
typedef float gemm_f32x2_any __attribute__((ext_vector_type(2), aligned(4)));  // two floats anywhere
typedef float gemm_f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t gemm_pack_bf16(float lo, float hi) {
    gemm_f32x2 v = {lo, hi};
    gemm_bf16x2 r = __builtin_convertvector(v, gemm_bf16x2);
    uint32_t u;
    __builtin_memcpy(&u, &r, 4);
    return u;
}

// The codes and block constants in the order the products read them, made once per matrix: per tile of 32 rows and
// chunk of 64 columns GEMM_TILE_BYTES consecutive bytes - one 16-byte word of codes per lane (row = lane % 32 of the
// tile, columns 32 (lane / 32) .. + 31 of the chunk), then one binary16 constant per lane (that of the lane's 32
// columns).  Rows past the matrix and columns past its width hold code 0 and constant 0: they add nothing.
constexpr uint32_t GEMM_TILE_BYTES = 64 * 16 + 64 * 2;
__global__ __launch_bounds__(256) void gemm_pack_weights_kernel(const uint4* __restrict__ codes,
                                                                const uint16_t* __restrict__ scales, uint32_t rows,
                                                                uint32_t cols, uint32_t log2_block, uint32_t n_chunks,
                                                                uint64_t n_tiles, char* __restrict__ packed) {
    const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_tiles * 64) return;
    const uint32_t lane = (uint32_t)(idx & 63);
    const uint64_t tile = idx >> 6;
    const uint32_t ch = (uint32_t)(tile % n_chunks), rt = (uint32_t)(tile / n_chunks);
    const uint32_t row = rt * GEMM_ROWS + (lane & 31), c = ch * GEMM_CHUNK + 32 * (lane >> 5);
    uint4 q = make_uint4(0u, 0u, 0u, 0u);
    uint16_t m = 0;
    if (row < rows && c < cols) {
        const uint64_t e = (uint64_t)row * cols + c;
        q = codes[e >> 5];
        m = scales[e >> log2_block];
    }
    char* out = packed + tile * GEMM_TILE_BYTES;
    reinterpret_cast<uint4*>(out)[lane] = q;
    reinterpret_cast<uint16_t*>(out + 1024)[lane] = m;
}

// x in the order the products read it, made once per call: for every tile of 32 tokens, chunk of 64 columns and
// product j one 16-byte word per lane (token = lane % 32 of the tile, columns 32 (lane / 32) + 8 j .. + 7 of the
// chunk), so that a wave's load is 1 KiB of consecutive memory; zeros past the last token and the last column.
__global__ __launch_bounds__(256) void gemm_pack_x_kernel(const uint16_t* __restrict__ x, uint32_t n_tokens,
                                                          uint32_t cols, uint32_t n_chunks, uint32_t n_pad,
                                                          uint4* __restrict__ xp) {
    const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint64_t total = (uint64_t)(n_pad / 32) * n_chunks * 256;
    if (idx >= total) return;
    const uint32_t lane = (uint32_t)(idx & 63), j = (uint32_t)((idx >> 6) & 3);
    const uint64_t tc = idx >> 8;
    const uint32_t ch = (uint32_t)(tc % n_chunks), tile = (uint32_t)(tc / n_chunks);
    const uint32_t n = tile * 32 + (lane & 31), c = ch * GEMM_CHUNK + 32 * (lane >> 5) + 8 * j;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (n < n_tokens && c < cols) v = *reinterpret_cast<const uint4*>(x + (uint64_t)n * cols + c);
    xp[idx] = v;
}

// The outlier list in the order of the products' tiles, made once per matrix.  ptr[rt * n_groups + g] is where the
// entries of row tile rt and column group g begin (a group: 2^log2_group chunks of 64 columns, as fine as the room that
// the size of the table leaves for a rows x cols matrix - one chunk wherever the last row tile is full, at most two for
// any other matrix of 32 rows or more), with one closing value; an entry is one 32-bit word:
//   bits 0 .. 15 the value as the decoder stores it (bfloat16), bits 16 .. 26 where it goes in the tile's decoded
//   operand - 16-byte word (product j, lane) and place in it, j * 512 + lane * 8 + column % 8 -, bits 27 .. 31 which
//   chunk of its group it belongs to.
// The list ascends, so the entries of 32 rows are one run of it and every workgroup sorts its own run: it counts the
// run's entries per group, turns the counts into places, and deals the entries out.  (Within a tile their order does
// not matter: they go to different places.)  Entries outside the matrix lie before or behind all runs.
struct GemmListGeometry {
    uint32_t n_groups, log2_group;
};
// Where the entries of one group begin (lo) and end (hi): never past the list, never more than the group has positions,
// and never backwards, whatever the table holds - the products take hi - lo as a count, so a table of another matrix
// costs wrong numbers and no read outside the list.
__device__ __forceinline__ void gemm_list_range(const uint32_t* __restrict__ p, uint32_t n_out, uint32_t log2_group,
                                                uint32_t& lo, uint32_t& hi) {
    lo = min(p[0], n_out);
    hi = min(max(p[1], lo), lo + min(2048u << log2_group, n_out - lo));
}
__device__ __forceinline__ uint32_t list_lower_bound(const int64_t* __restrict__ out_idx, uint32_t n_out, int64_t target) {
    uint32_t lo = 0, hi = n_out;  // first entry >= target
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (out_idx[mid] < target) lo = mid + 1; else hi = mid;
    }
    return lo;
}
constexpr uint32_t GEMM_MAX_CHUNKS = GEMM_MAX_COLS / GEMM_CHUNK;  // 512
static_assert(GEMM_MAX_COLS == GEMV_MAX_STRIPS * GEMV_STRIP, "both products take the same widths");
// A grid of at most GEMM_LIST_WGS workgroups (a launch holds fewer than 2^32 lanes, a matrix up to 2^27 row tiles); 1024
// lanes each where there are fewer row tiles than compute units, else 256.  An entry's distance from the first
// position of its row tile is below 2^20, so rows and columns come from a 32-bit division: 500 x 28672 with 0.7 %
// outliers took 21 us with 64-bit divisions and 256 lanes.
constexpr uint32_t GEMM_LIST_WGS = 1u << 20;
__global__ __launch_bounds__(1024) void gemm_list_kernel(const int64_t* __restrict__ out_idx,
                                                         const uint16_t* __restrict__ out_val, uint32_t n_out,
                                                         uint64_t rows, uint32_t cols, uint32_t row_tiles,
                                                         GemmListGeometry lg, uint32_t* __restrict__ ptr,
                                                         uint32_t* __restrict__ entries) {
    __shared__ uint32_t place[GEMM_MAX_CHUNKS];
    __shared__ uint32_t range[2];
    const uint32_t tid = threadIdx.x, group_cols = GEMM_CHUNK << lg.log2_group;
    for (uint32_t rt = blockIdx.x; rt < row_tiles; rt += gridDim.x) {
        if (tid < 2) {
            const uint64_t r = min((uint64_t)(rt + tid) * GEMM_ROWS, rows);
            range[tid] = list_lower_bound(out_idx, n_out, (int64_t)(r * cols));
        }
        for (uint32_t i = tid; i < lg.n_groups; i += blockDim.x) place[i] = 0u;
        __syncthreads();
        const uint32_t a = range[0], b = range[1];
        const uint64_t first = (uint64_t)rt * GEMM_ROWS * cols;
        for (uint64_t k = (uint64_t)a + tid; k < b; k += blockDim.x) {
            const uint32_t c = (uint32_t)((uint64_t)out_idx[k] - first) % cols;
            atomicAdd(&place[c / group_cols], 1u);
        }
        __syncthreads();
        if (tid < 64) {  // exclusive prefix sum over the groups, eight per lane
            uint32_t v[GEMM_MAX_CHUNKS / 64], sum = 0;
#pragma unroll
            for (uint32_t i = 0; i < GEMM_MAX_CHUNKS / 64; ++i) {
                const uint32_t g = tid * (GEMM_MAX_CHUNKS / 64) + i;
                v[i] = g < lg.n_groups ? place[g] : 0u;
                sum += v[i];
            }
            uint32_t at = a + wave_inclusive_scan_u32(sum) - sum;
#pragma unroll
            for (uint32_t i = 0; i < GEMM_MAX_CHUNKS / 64; ++i) {
                const uint32_t g = tid * (GEMM_MAX_CHUNKS / 64) + i;
                if (g < lg.n_groups) {
                    place[g] = at;
                    ptr[(uint64_t)rt * lg.n_groups + g] = at;
                }
                at += v[i];
            }
        }
        if (tid == 0 && rt == row_tiles - 1) ptr[(uint64_t)row_tiles * lg.n_groups] = b;
        __syncthreads();
        for (uint64_t k = (uint64_t)a + tid; k < b; k += blockDim.x) {
            const uint32_t off = (uint32_t)((uint64_t)out_idx[k] - first);
            const uint32_t r = off / cols, c = off % cols, cc = c % GEMM_CHUNK;
            const uint32_t lane = 32 * (cc >> 5) + r, j = (cc >> 3) & 3u;
            const uint32_t val = f32_to_bf16_rne(f16_bits_to_f32(out_val[k]));
            entries[atomicAdd(&place[c / group_cols], 1u)] =
                val | ((j * 512 + lane * 8 + (cc & 7u)) << 16) | ((c % group_cols / GEMM_CHUNK) << 27);
        }
        __syncthreads();  // place and range are the next row tile's
    }
}

// Adds an accumulator to its sum and leaves in the accumulator what the addition rounded away (exactly where the sum is the
// larger of the two, to within a rounding of the smaller elsewhere), so that cutting a chain of additions there costs
// nothing of the sum.  The clamp is for sums that are not finite: an infinite sum stays what it is (inf - inf
// would make it NaN), a NaN is in the sum already; no residue of finite numbers reaches 2^104.
__device__ __forceinline__ void gemm_carry(gemm_f32x16& sum, gemm_f32x16& acc, int i) {
    const float s0 = sum[i], a0 = acc[i], s1 = s0 + a0;
    sum[i] = s1;
    acc[i] = __builtin_amdgcn_fmed3f(a0 - (s1 - s0), -0x1p104f, 0x1p104f);
}

// Workgroup (b, s): R tiles of 32 rows (32 R b ..), the chunks s * waves + wave, + n_split * waves, ... of the row,
// NT tiles of 32 tokens (tile0 ..).  Its sum goes to dst[(s * n_tokens + token) * rows + row], token counted from
// the first of tile0: the result itself when n_split is 1, else one of n_split partial results that gemm_sum_kernel
// adds.  With a list the wave parks the decoded operand of a tile in LDS, writes the tile's entries over their
// placeholders and reads the operand back (one wave, one buffer: no barrier).  Against adding (value - placeholder) *
// x per entry and token to the row sums afterwards, as this kernel did before: 12288 x 4096 with 0.7 % outliers, 8 /
// 32 / 64 / 128 tokens 20.2 / 20.4 / 31.1 / 49.7 -> 18.3 / 17.9 / 24.2 / 38.2 us.
//   Outliers put half of a row's energy into a hundredth of its terms, and the roundings of a chain of additions grow
// with what it has added up: with the entries inside the product the error of the sums was 1.03 to 1.4 times that of
// adding them apart.  So with a list the matrix cores' chain is cut: after `flush` chunks the accumulators are added to a
// second set (CARRY, where there are registers for one: 4 instructions per accumulator), or the chunks are taken in
// n_runs = 2 runs with the workgroup's sum after each (RUNS: the largest tiles, and two tiles of rows with one of tokens,
// which would lose its second workgroup per compute unit).  Without the cuts 128 tokens on 12288 x 4096 took 32 us.
//   The waves' sums are added in binary64: 8 additions of 1 in 24 bits are as many roundings as a short chain has.  Two
// buffers in turn save a barrier per tile, which pays for it: 28672 x 512 without a list, 128 tokens 21.0 -> 20.2 us.
// The packed matrix holds a multiple of GEMM_MAX_R row tiles.
template <int R, int NT>
constexpr bool GEMM_CARRY = R == 1 || NT == 2;
template <int R, int NT, bool OUTLIERS, bool X_IN_PLACE>
__global__ __launch_bounds__(64 * GEMM_MAX_WAVES, X_IN_PLACE ? 4 : 2) void gemm_kernel(
    const char* __restrict__ packed, uint32_t rows, uint32_t cols, CodebookArgs cb, const uint32_t* __restrict__ list_ptr,
    const uint32_t* __restrict__ entries, uint32_t n_out, GemmListGeometry lg, uint32_t row_tiles,
    const uint4* __restrict__ xp, const uint16_t* __restrict__ x, uint32_t tile0, uint32_t n_tokens, uint32_t flush,
    uint32_t n_runs, float* __restrict__ dst) {
    static_assert(!X_IN_PLACE || NT == 1, "one tile of tokens");
    constexpr uint32_t N_RED = R * NT > 1 && !(OUTLIERS && R * NT > 6) ? 2 : 1;  // (the largest one would spill)
    struct Shared {
        float tab[16];
        // per wave: accumulator registers 4 k .. 4 k + 3 of lane l at [(k * 64 + l) * 4], for two tiles in turn; in the
        // loop over chunks, with a list, the wave's decoded operand
        float red[N_RED][GEMM_MAX_WAVES * 16 * 64];
        float half[OUTLIERS && !GEMM_CARRY<R, NT> ? R * NT * 16 * 64 : 2];  // the workgroup's sums over the first run
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63, n_waves = blockDim.x >> 6;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 16) sh.tab[tid] = cb.lv32[tid];
    __syncthreads();
    const char* tab = reinterpret_cast<const char*>(sh.tab);
    const uint32_t n_chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK;
    const uint32_t stride = gridDim.y * n_waves;

    constexpr bool CARRY = OUTLIERS && GEMM_CARRY<R, NT>, RUNS = OUTLIERS && !GEMM_CARRY<R, NT>;
    gemm_f32x16 acc[R][NT], sum[CARRY ? R : 1][CARRY ? NT : 1];

    // What the chunk after this one needs (codes, constants and - where the registers allow it - x) is on its way
    // while this one is decoded and multiplied, in two sets of registers used in turn.  Past the last chunk the last
    // one is read again and not used.
    constexpr bool X_AHEAD = R * NT <= 2;
    struct Operands {
        uint4 q[R], xb[NT][4];
        uint16_t m[R];
        uint32_t en[R], n_en[R];  // this lane's list entry of the tile, and how many entries the tile has
    };
    // X_IN_PLACE: a single tile of tokens is read where it stands.  A lane's four words of a chunk are 64 consecutive bytes of its
    // token's row, and what the wave reads of a row is one line.  (Lanes past the last token take the last one's and
    // their results are not stored; columns past the width are zero.)
    const char* x_tile = reinterpret_cast<const char*>(x);
    const uint32_t my_x = (min(lane & 31u, n_tokens - 1) * cols + 32 * (lane >> 5)) * 2;  // 2 MB at most
    auto fetch_x = [&](Operands& o, uint32_t chunk) {
        if constexpr (X_IN_PLACE) {
            const bool inside = chunk * GEMM_CHUNK + 32 * (lane >> 5) < cols;
            const uint4* p = reinterpret_cast<const uint4*>(x_tile + chunk * (GEMM_CHUNK * 2) + my_x);
#pragma unroll
            for (int j = 0; j < 4; ++j) o.xb[0][j] = inside ? p[j] : make_uint4(0u, 0u, 0u, 0u);
            return;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                o.xb[t][j] = xp[((uint64_t)(tile0 + t) * n_chunks + chunk) * 256 + j * 64 + lane];
    };
    const char* my_tiles = packed + (uint64_t)blockIdx.x * R * n_chunks * GEMM_TILE_BYTES;
    const uint32_t ch_first = blockIdx.y * n_waves + wave;
    // Where the entries of the wave's tiles begin and end: lane i holds those of the i-th chunk it takes (a wave takes
    // at most 64 chunks: 512 in all, and fewer than eight waves only where each takes one).
    uint32_t e_lo[R], e_hi[R];
    if (OUTLIERS) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t rt = blockIdx.x * R + r, chunk = ch_first + lane * stride;
            e_lo[r] = e_hi[r] = 0u;
            if (rt < row_tiles && chunk < n_chunks) {
                const uint32_t* p = list_ptr + (uint64_t)rt * lg.n_groups + (chunk >> lg.log2_group);
                gemm_list_range(p, n_out, lg.log2_group, e_lo[r], e_hi[r]);
            }
        }
    }
    auto fetch = [&](Operands& o, uint32_t chunk, uint32_t nth) {  // this lane's 32 columns of the chunk, in each tile of rows
        if (OUTLIERS) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)e_lo[r], (int)nth);
                o.n_en[r] = (uint32_t)__builtin_amdgcn_readlane((int)e_hi[r], (int)nth) - lo;
                o.en[r] = lane < o.n_en[r] ? entries[lo + lane] : 0u;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const char* tile = my_tiles + ((uint64_t)r * n_chunks + chunk) * GEMM_TILE_BYTES;
            o.q[r] = load_stream(reinterpret_cast<const uint4*>(tile) + lane);
            o.m[r] = __builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(tile + 1024) + lane);
        }
        if (X_AHEAD) fetch_x(o, chunk);
    };
    uint16_t* parked = reinterpret_cast<uint16_t*>(sh.red[0] + wave * 16 * 64);
    auto patch = [&](uint32_t e, uint32_t chunk) {
        if ((e >> 27) == (chunk & ((1u << lg.log2_group) - 1u))) parked[(e >> 16) & 2047u] = (uint16_t)e;
    };
    auto multiply = [&](Operands& o, uint32_t chunk, uint32_t nth) {
        if (!X_AHEAD) {
            fetch_x(o, chunk);
            __builtin_amdgcn_sched_barrier(0);  // x is on its way while the first tile of rows is decoded
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float msc = f16_bits_to_f32(o.m[r]);
            const uint32_t w[4] = {o.q[r].x, o.q[r].y, o.q[r].z, o.q[r].w};
            gemm_bf16x8 A[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // byte i of `even` = 4 * code of element 2 i of the word, of `odd` = 4 * code of element 2 i + 1
                const uint32_t even = (w[j] << 2) & 0x3c3c3c3cu, odd = (w[j] >> 2) & 0x3c3c3c3cu;
                const uint32_t oe[4] = {byte_of<0>(even), byte_of<1>(even), byte_of<2>(even), byte_of<3>(even)};
                const uint32_t oo[4] = {byte_of<0>(odd), byte_of<1>(odd), byte_of<2>(odd), byte_of<3>(odd)};
                uint32_t a[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float le = *reinterpret_cast<const float*>(tab + oe[i]);
                    const float lo = *reinterpret_cast<const float*>(tab + oo[i]);
                    a[i] = gemm_pack_bf16(msc * le, msc * lo);  // the decoder's product and rounding
                }
                __builtin_memcpy(&A[j], a, 16);
            }
            if (OUTLIERS && o.n_en[r] != 0u) {  // wave-uniform
                gemm_bf16x8* word = reinterpret_cast<gemm_bf16x8*>(parked) + lane;
                wave_lds_fence();
#pragma unroll
                for (int j = 0; j < 4; ++j) word[64 * j] = A[j];
                wave_lds_fence();
                if (lane < o.n_en[r]) patch(o.en[r], chunk);
                if (o.n_en[r] > 64u) {  // a tile with more entries than lanes
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)e_lo[r], (int)nth);
                    for (uint32_t k = 64u + lane; k < o.n_en[r]; k += 64u) patch(entries[lo + k], chunk);
                }
                wave_lds_fence();
#pragma unroll
                for (int j = 0; j < 4; ++j) A[j] = word[64 * j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    gemm_bf16x8 B;
                    const uint32_t bw[4] = {o.xb[t][j].x, o.xb[t][j].y, o.xb[t][j].z, o.xb[t][j].w};
                    __builtin_memcpy(&B, bw, 16);
                    acc[r][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[j], B, acc[r][t], 0, 0, 0);
                }
        }
    };
    // Adds the waves' accumulators of every tile, in wave order and in binary64, and stores the sums: for the second
    // half of the chunks (or all of them) the result, for the first half the record that the second half starts from.
    // Accumulator i of lane l: row 8 (i / 4) + 4 (l / 32) + i % 4 of the tile, token l % 32; a thread adds two
    // neighbouring rows of one token.
    float* out = dst + (uint64_t)blockIdx.y * n_tokens * rows;
    auto reduce = [&](const uint32_t run, const bool last_run) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t r0 = (blockIdx.x * R + r) * GEMM_ROWS;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                // what stood here has been read: with two buffers the barrier of the tile in between says so
                if (N_RED == 1 && (r > 0 || t > 0)) __syncthreads();
                float* red = sh.red[(r * NT + t) % N_RED];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 v = make_float4(acc[r][t][4 * k], acc[r][t][4 * k + 1], acc[r][t][4 * k + 2], acc[r][t][4 * k + 3]);
                    *reinterpret_cast<float4*>(red + ((wave * 4 + k) * 64 + lane) * 4) = v;
                }
                __syncthreads();
                for (uint32_t p = tid; p < 8 * 64; p += blockDim.x) {
                    double s0 = 0.0, s1 = 0.0;
                    float2* first = reinterpret_cast<float2*>(sh.half) + (RUNS ? (r * NT + t) * 8 * 64 + p : 0);
                    if (RUNS && run > 0u) {
                        s0 = first->x;
                        s1 = first->y;
                    }
                    const float2* v = reinterpret_cast<const float2*>(red) + p;
                    if (n_waves == GEMM_MAX_WAVES) {  // all reads under way at once
                        float2 w[GEMM_MAX_WAVES];
#pragma unroll
                        for (uint32_t wv = 0; wv < GEMM_MAX_WAVES; ++wv) w[wv] = v[wv * 8 * 64];
#pragma unroll
                        for (uint32_t wv = 0; wv < GEMM_MAX_WAVES; ++wv) {
                            s0 += w[wv].x;
                            s1 += w[wv].y;
                        }
                    } else {
                        for (uint32_t wv = 0; wv < n_waves; ++wv) {
                            s0 += v[wv * 8 * 64].x;
                            s1 += v[wv * 8 * 64].y;
                        }
                    }
                    if (!last_run) {
                        *first = make_float2((float)s0, (float)s1);
                        continue;
                    }
                    const uint32_t l = (p >> 1) & 63, row = r0 + 8 * (p >> 7) + 4 * (l >> 5) + 2 * (p & 1), n = 32 * t + (l & 31);
                    if (n >= n_tokens) continue;
                    float* o = out + (uint64_t)n * rows + row;
                    if (row + 1 < rows) {
                        const gemm_f32x2_any v = {(float)s0, (float)s1};
                        *reinterpret_cast<gemm_f32x2_any*>(o) = v;
                    } else if (row < rows) {
                        *o = (float)s0;
                    }
                }
            }
        }
    };

    uint32_t ch = ch_first;
    const uint32_t last = n_chunks - 1;
    const uint32_t n_iter = ch < n_chunks ? (last - ch) / stride + 1 : 0;
    uint32_t nth = 0;  // how many chunks this wave has taken
    uint32_t until_flush = flush;
    auto carry = [&]() __attribute__((always_inline)) {
        if constexpr (CARRY) {
            if (--until_flush == 0u) {
                until_flush = flush;
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int i = 0; i < 16; ++i) gemm_carry(sum[r][t], acc[r][t], i);
            }
        }
    };
    Operands o0, o1;
    fetch(o0, min(ch, last), 0);
    for (uint32_t run = 0; run < (RUNS ? n_runs : 1u); ++run) {  // o0 holds chunk ch
        const bool last_run = !RUNS || run + 1 == n_runs;
        const uint32_t todo = last_run ? n_iter - nth : (n_iter + 1) / 2;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    acc[r][t][i] = 0.0f;
                    if constexpr (CARRY) sum[r][t][i] = 0.0f;
                }
        if (todo & 1u) {  // an odd one first, so that the rest goes in pairs
            multiply(o0, ch, nth);
            carry();
            ch += stride;
            nth += 1;
            fetch(o0, min(ch, last), min(nth, 63u));
        }
        for (uint32_t it = todo >> 1; it > 0; --it) {  // o0 holds chunk ch
            fetch(o1, ch + stride, nth + 1);
            __builtin_amdgcn_sched_barrier(0);  // the loads first, then the arithmetic
            multiply(o0, ch, nth);
            carry();
            fetch(o0, min(ch + 2 * stride, last), min(nth + 2, 63u));
            __builtin_amdgcn_sched_barrier(0);
            multiply(o1, ch + stride, nth + 1);
            carry();
            ch += 2 * stride;
            nth += 2;
        }
        if constexpr (CARRY) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[r][t] += sum[r][t];
        }
        reduce(run, last_run);
        if (!last_run) __syncthreads();  // `red` is the waves' own again
    }
}

// Many tokens: the same product with a tile of 256 rows x 128 tokens per workgroup of eight waves.  gemm_kernel reads
// all of x once per 64 rows (0.8 GB per 128 tokens through a Llama-7B-shaped block, and it ran at the rate at which the
// caches deliver that); here the decoded weights and x are shared through LDS, so x is read once per 256 rows and a
// weight is decoded once per 128 tokens by one wave.
//   A step is one chunk of 64 columns.  Each wave decodes its one row tile of the chunk after the next into LDS (list
// entries are written over their placeholders there: a wave's LDS accesses are carried out in order, so nothing is
// waited for), carries its share of that chunk's x over, and multiplies two row tiles with two token tiles of the
// current chunk (four waves by two).  The step goes in quarters - one 16-byte word of every operand -, and the LDS
// reads of a quarter are under way while the one before is multiplied, across the step's barrier too: that is what the
// third buffer is for.
//   The matrix cores' chain of additions is cut every `flush` chunks and added to a second set of accumulators, which with
// CARRY keeps what the addition rounds away (gemm_carry).  `flush` follows the chunks that a wave of gemm_kernel takes for
// the same matrix, so the error of the sums is at most that kernel's.  Carrying is for what would be worse without: a
// list, and matrices whose columns gemm_kernel splits; its four instructions per accumulator instead of two are 7 % of the
// time where `flush` is nine chunks, 10 % at four (4096 columns with a list) and 40 % at one (512 columns with a list).
//   What bounds it: of a chunk's 2745 clocks the LDS unit is busy 1440, the vector units 1135, the matrix cores 1024
// (12288 x 4096, 2000 tokens; with a list 3515, 1470, 1695, 1024); two waves per SIMD overlap them in part.
//   2000 tokens, gemm_kernel -> this: without a list 22016 x 4096 850 -> 488 us, 57344 x 8192 2860 -> 2250 (835
// TFLOP/s), 4096 x 4096 257 -> 100; with one 22016 x 4096 1087 -> 589, 57344 x 8192 3503 -> 2590, 4096 x 4096 305 -> 122.
// The weights are the second operand here: accumulator i of lane l is token 8 (i / 4) + 4 (l / 32) + i % 4 and row
// l % 32, so that a store of a wave writes two runs of 128 bytes.
template <bool OUTLIERS, bool CARRY>
__global__ __launch_bounds__(64 * GEMM_WIDE_WAVES, 2) void gemm_wide_kernel(
    const char* __restrict__ packed, uint32_t rows, uint32_t cols, CodebookArgs cb, const uint32_t* __restrict__ list_ptr,
    const uint32_t* __restrict__ entries, uint32_t n_out, GemmListGeometry lg, uint32_t row_tiles, uint32_t packed_tiles,
    const uint4* __restrict__ xp, uint32_t tok_tiles, uint32_t tok_groups, uint32_t per_split, uint32_t flush,
    uint32_t n_tokens, float* __restrict__ y, float* __restrict__ parts) {
    struct Shared {
        float tab[16];
        uint16_t unused[GEMM_WIDE_WAVES][64];  // where lanes without an entry write
        uint4 a[3][GEMM_WIDE_WAVES][GEMM_TILE_WORDS];
        uint4 b[3][GEMM_WIDE_TOK_TILES][GEMM_TILE_WORDS];
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 16) sh.tab[tid] = cb.lv32[tid];
    __syncthreads();
    const char* tab = reinterpret_cast<const char*>(sh.tab);
    const uint32_t n_chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK;

    // Workgroups go to the eight dies in turn; each die takes a contiguous run of tiles, token groups fastest, so
    // that the workgroups on one die share rows and tokens in its cache.
    uint32_t id = blockIdx.x;
    {
        const uint32_t total = gridDim.x, q = total / 8, rem = total % 8, die = id % 8;
        id = die * q + min(die, rem) + id / 8;
    }
    const uint32_t tg = id % tok_groups, rg = (id / tok_groups) % ((row_tiles + 7) / 8),
                   part = id / (tok_groups * ((row_tiles + 7) / 8));
    const uint32_t ch0 = part * per_split, ch1 = min(n_chunks, ch0 + per_split), n_steps = ch1 - ch0;
    const uint32_t my_rt = rg * GEMM_WIDE_WAVES + wave;
    // a row tile or token tile past the last is read from the last one and not stored
    const char* my_tile = packed + (uint64_t)min(my_rt, packed_tiles - 1) * n_chunks * GEMM_TILE_BYTES;
    const uint32_t my_tt = min(tg * GEMM_WIDE_TOK_TILES + (wave >> 1), tok_tiles - 1);
    const uint4* my_x = xp + (uint64_t)my_tt * n_chunks * GEMM_TILE_WORDS + (wave & 1) * 128 + lane;

    struct Ahead {  // what a wave brings into LDS for one chunk: the codes of its row tile and its share of x
        uint4 q, x0, x1;
        uint16_t m;
        uint32_t en, lo, n_en;  // this lane's list entry of the tile; where the tile's entries begin, how many
    };
    uint32_t e_lo = 0, e_hi = 0;  // lane i: where the entries of the i-th of 64 chunks begin and end
    auto fetch = [&](uint32_t nth) __attribute__((always_inline)) {  // called for nth = 0, 1, 2, ...
        Ahead o = {};
        const uint32_t chunk = min(ch0 + nth, ch1 - 1);
        if (OUTLIERS) {
            if ((nth & 63u) == 0u) {
                const uint32_t c = ch0 + nth + lane;
                e_lo = e_hi = 0u;
                if (my_rt < row_tiles && c < ch1) {
                    const uint32_t* p = list_ptr + (uint64_t)my_rt * lg.n_groups + (c >> lg.log2_group);
                    gemm_list_range(p, n_out, lg.log2_group, e_lo, e_hi);
                }
            }
            o.lo = (uint32_t)__builtin_amdgcn_readlane((int)e_lo, (int)(nth & 63u));
            o.n_en = (uint32_t)__builtin_amdgcn_readlane((int)e_hi, (int)(nth & 63u)) - o.lo;
            o.en = lane < o.n_en ? entries[o.lo + lane] : 0u;
        }
        const char* tile = my_tile + (uint64_t)chunk * GEMM_TILE_BYTES;
        o.q = reinterpret_cast<const uint4*>(tile)[lane];
        o.m = reinterpret_cast<const uint16_t*>(tile + 1024)[lane];
        const uint4* p = my_x + (uint64_t)chunk * GEMM_TILE_WORDS;
        o.x0 = p[0];
        o.x1 = p[64];
        return o;
    };
    // Decoding in quarters (one 16-byte word of the operand each): the look-ups, then products, rounding and the store.
    struct Levels {
        float v[8];
    };
    auto look_up = [&](const uint32_t w) __attribute__((always_inline)) {
        const uint32_t even = (w << 2) & 0x3c3c3c3cu, odd = (w >> 2) & 0x3c3c3c3cu;
        const uint32_t oe[4] = {byte_of<0>(even), byte_of<1>(even), byte_of<2>(even), byte_of<3>(even)};
        const uint32_t oo[4] = {byte_of<0>(odd), byte_of<1>(odd), byte_of<2>(odd), byte_of<3>(odd)};
        Levels l;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            l.v[2 * i] = *reinterpret_cast<const float*>(tab + oe[i]);
            l.v[2 * i + 1] = *reinterpret_cast<const float*>(tab + oo[i]);
        }
        return l;
    };
    auto store_word = [&](const Levels l, float msc, uint32_t buf, int j) __attribute__((always_inline)) {
        uint32_t a[4];  // the decoder's product and rounding
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = gemm_pack_bf16(msc * l.v[2 * i], msc * l.v[2 * i + 1]);
        sh.a[buf][wave][64 * j + lane] = make_uint4(a[0], a[1], a[2], a[3]);
    };
    auto patch = [&](const Ahead o, uint32_t nth, uint32_t buf) __attribute__((always_inline)) {
        const uint32_t my_parked = (uint32_t)offsetof(Shared, a) + (buf * GEMM_WIDE_WAVES + wave) * GEMM_TILE_WORDS * 16;
        const uint32_t my_unused = (uint32_t)offsetof(Shared, unused) + (wave * 64 + lane) * 2;
        const uint32_t place = min(ch0 + nth, ch1 - 1) & ((1u << lg.log2_group) - 1u);
        wave_lds_fence();  // the entries after what they overwrite
        const bool mine = lane < o.n_en && (o.en >> 27) == place;
        const uint32_t at = mine ? my_parked + 2 * ((o.en >> 16) & 2047u) : my_unused;
        *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(&sh) + at) = (uint16_t)o.en;
        if (o.n_en > 64u) {  // a tile with more entries than lanes
            uint16_t* parked = reinterpret_cast<uint16_t*>(sh.a[buf][wave]);
            for (uint32_t k = 64u + lane; k < o.n_en; k += 64u) {
                const uint32_t e = entries[o.lo + k];
                if ((e >> 27) == place) parked[(e >> 16) & 2047u] = (uint16_t)e;
            }
        }
    };

    gemm_f32x16 acc[2][2], sum[2][2];  // [row tile][token tile]
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][t][i] = sum[r][t][i] = 0.0f;
    const uint32_t wr = 2 * (wave & 3), wt = 2 * (wave >> 2);  // first row tile and token tile that the wave multiplies
    struct Operands {
        gemm_bf16x8 a[2], b[2];
    };
    auto read_operands = [&](uint32_t buf, int j) __attribute__((always_inline)) {
        const gemm_bf16x8* a = reinterpret_cast<const gemm_bf16x8*>(sh.a[buf][wr]) + lane;
        const gemm_bf16x8* b = reinterpret_cast<const gemm_bf16x8*>(sh.b[buf][wt]) + lane;
        const Operands o = {{a[64 * j], a[GEMM_TILE_WORDS + 64 * j]}, {b[64 * j], b[GEMM_TILE_WORDS + 64 * j]}};
        return o;
    };
    auto multiply = [&](const Operands o) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[r][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.b[t], o.a[r], acc[r][t], 0, 0, 0);
    };
    auto store_x = [&](const uint4 v0, const uint4 v1, uint32_t buf) __attribute__((always_inline)) {
        uint4* p = sh.b[buf][wave >> 1] + (wave & 1) * 128 + lane;
        p[0] = v0;
        p[64] = v1;
    };

    uint32_t until_flush = flush;
    // Before step s: buffer s % 3 holds chunk s and buffer (s + 1) % 3 chunk s + 1; `o` is what chunk s + 2 needs; what
    // chunk s + 3 needs is on its way, that of chunk s + 4 is asked for during the step; `op` and `lv` are the operands
    // and the look-ups of the step's first quarter.
    Operands op;
    Levels lv;
    auto step = [&](uint32_t s, const uint32_t buf, const Ahead o, uint32_t next_word) __attribute__((always_inline)) {
        const uint32_t buf1 = buf == 2u ? 0u : buf + 1u, buf2 = buf == 0u ? 2u : buf - 1u;
        const Ahead asked = fetch(s + 4);
        const float msc = f16_bits_to_f32(o.m);
        const uint32_t w[5] = {o.q.x, o.q.y, o.q.z, o.q.w, next_word};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // the next quarter's LDS reads are on their way while this one is multiplied and stored
            const Operands op_next = read_operands(j < 3 ? buf : buf1, (j + 1) & 3);
            const Levels lv_next = look_up(w[j + 1]);
            __builtin_amdgcn_sched_barrier(0);
            multiply(op);
            store_word(lv, msc, buf2, j);
            if (j == 2) store_x(o.x0, o.x1, buf2);
            __builtin_amdgcn_sched_barrier(0);
            lv = lv_next;
            op = op_next;
        }
        if (OUTLIERS) patch(o, s + 2, buf2);
        if (--until_flush == 0u) {
            until_flush = flush;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        if (CARRY) {
                            gemm_carry(sum[r][t], acc[r][t], i);
                        } else {
                            sum[r][t][i] += acc[r][t][i];
                            acc[r][t][i] = 0.0f;
                        }
                    }
        }
        __syncthreads();
        return asked;
    };
    Ahead o2, o3;
    {
        const Ahead first = fetch(0), second = fetch(1);
        o2 = fetch(2);
        o3 = fetch(3);
        const uint32_t w[8] = {first.q.x, first.q.y, first.q.z, first.q.w, second.q.x, second.q.y, second.q.z, second.q.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) store_word(look_up(w[j]), f16_bits_to_f32(j < 4 ? first.m : second.m), j >> 2, j & 3);
        if (OUTLIERS) {
            patch(first, 0, 0);
            patch(second, 1, 1);
        }
        store_x(first.x0, first.x1, 0);
        store_x(second.x0, second.x1, 1);
        lv = look_up(o2.q.x);
        __syncthreads();
        op = read_operands(0, 0);
    }
    // Three steps to a round, so that neither the buffers' places nor the registers of what is on its way move: a copy
    // of a register that is being loaded would wait for the load, and each step would take as long as memory's latency
    // (keeping them in place made the largest matrices 3 to 5 % faster).
    uint32_t s = 0;
    for (uint32_t rounds = n_steps / 3; rounds > 0; --rounds, s += 3) {
        const Ahead o4 = step(s, 0, o2, o3.q.x);
        o2 = step(s + 1, 1, o3, o4.q.x);
        o3 = step(s + 2, 2, o4, o2.q.x);
    }
    if (s < n_steps) {
        const Ahead o4 = step(s, 0, o2, o3.q.x);
        if (s + 1 < n_steps) step(s + 1, 1, o3, o4.q.x);
    }

    // the first part goes to the result itself, where gemm_sum_kernel adds the others to it
    float* out = part == 0 ? y : parts + (uint64_t)(part - 1) * n_tokens * rows;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint32_t row = (rg * GEMM_WIDE_WAVES + wr + r) * GEMM_ROWS + (lane & 31);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t tok0 = (tg * GEMM_WIDE_TOK_TILES + wt + t) * GEMM_TOKENS + 4 * (lane >> 5);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t tok = tok0 + 8 * (i >> 2) + (i & 3);
                if (row < rows && tok < n_tokens) out[(uint64_t)tok * rows + row] = sum[r][t][i] + acc[r][t][i];
            }
        }
    }
}

// Many more tokens: the matrix is decoded once, to bfloat16 in the order of the products' operands (gemm_decode_kernel, a
// 4096-byte tile per 32 rows and 64 columns, list entries in place), and multiplied by gemm_decoded_kernel, which has
// nothing to decode.  gemm_wide_kernel decodes a weight once per 128 tokens.
// One wave per GEMM_DECODE_TILES tiles of one row tile, all of whose codes are on their way at once.  Bound by memory: 50 M
// weights in 23 us (5.7 TB/s) where what it writes stays in the 256 MB cache behind the L2s, half of that beyond.
constexpr uint32_t GEMM_DECODE_TILES = 4, GEMM_DECODE_WAVES = 4;
template <bool OUTLIERS>
__global__ __launch_bounds__(64 * GEMM_DECODE_WAVES) void gemm_decode_kernel(
    const char* __restrict__ packed, uint32_t first_rt, uint32_t n_rt, uint32_t n_chunks, CodebookArgs cb,
    const uint32_t* __restrict__ list_ptr, const uint32_t* __restrict__ entries, uint32_t n_out, GemmListGeometry lg,
    uint32_t row_tiles, uint4* __restrict__ decoded) {
    struct Shared {
        float tab[16];
        uint4 parked[OUTLIERS ? GEMM_DECODE_WAVES : 1][OUTLIERS ? 4 * 64 : 1];
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 16) sh.tab[tid] = cb.lv32[tid];
    __syncthreads();
    const char* tab = reinterpret_cast<const char*>(sh.tab);
    const uint32_t runs = (n_chunks + GEMM_DECODE_TILES - 1) / GEMM_DECODE_TILES;
    const uint64_t job = (uint64_t)blockIdx.x * GEMM_DECODE_WAVES + wave;
    if (job >= (uint64_t)n_rt * runs) return;
    const uint32_t rt_local = (uint32_t)(job / runs), ch0 = (uint32_t)(job % runs) * GEMM_DECODE_TILES;
    const uint32_t n = min(GEMM_DECODE_TILES, n_chunks - ch0), rt = first_rt + rt_local;
    uint4 q[GEMM_DECODE_TILES];
    uint16_t m[GEMM_DECODE_TILES];
#pragma unroll
    for (uint32_t i = 0; i < GEMM_DECODE_TILES; ++i) {
        const char* tile = packed + ((uint64_t)rt * n_chunks + ch0 + min(i, n - 1)) * GEMM_TILE_BYTES;
        q[i] = load_stream(reinterpret_cast<const uint4*>(tile) + lane);
        m[i] = __builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(tile + 1024) + lane);
    }
    uint32_t e_lo = 0, e_hi = 0, en[GEMM_DECODE_TILES], lo[GEMM_DECODE_TILES], n_en[GEMM_DECODE_TILES];
    if (OUTLIERS) {
        if (rt < row_tiles && lane < n)
            gemm_list_range(list_ptr + (uint64_t)rt * lg.n_groups + ((ch0 + lane) >> lg.log2_group), n_out, lg.log2_group, e_lo, e_hi);
#pragma unroll
        for (uint32_t i = 0; i < GEMM_DECODE_TILES; ++i) {
            lo[i] = (uint32_t)__builtin_amdgcn_readlane((int)e_lo, (int)i);
            n_en[i] = (uint32_t)__builtin_amdgcn_readlane((int)e_hi, (int)i) - lo[i];
            en[i] = lane < n_en[i] ? entries[lo[i] + lane] : 0u;
        }
    }
    uint4* out = decoded + ((uint64_t)rt_local * n_chunks + ch0) * GEMM_TILE_WORDS + lane;
#pragma unroll
    for (uint32_t i = 0; i < GEMM_DECODE_TILES; ++i) {
        if (i >= n) break;  // wave-uniform
        const float msc = f16_bits_to_f32(m[i]);
        const uint32_t w[4] = {q[i].x, q[i].y, q[i].z, q[i].w};
        uint4 A[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t even = (w[j] << 2) & 0x3c3c3c3cu, odd = (w[j] >> 2) & 0x3c3c3c3cu;
            const uint32_t oe[4] = {byte_of<0>(even), byte_of<1>(even), byte_of<2>(even), byte_of<3>(even)};
            const uint32_t oo[4] = {byte_of<0>(odd), byte_of<1>(odd), byte_of<2>(odd), byte_of<3>(odd)};
            uint32_t a[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float le = *reinterpret_cast<const float*>(tab + oe[k]);
                const float lv = *reinterpret_cast<const float*>(tab + oo[k]);
                a[k] = gemm_pack_bf16(msc * le, msc * lv);  // the decoder's product and rounding
            }
            A[j] = make_uint4(a[0], a[1], a[2], a[3]);
        }
        if (OUTLIERS && n_en[i] != 0u) {  // wave-uniform
            uint4* word = sh.parked[wave] + lane;
            uint16_t* parked = reinterpret_cast<uint16_t*>(sh.parked[wave]);
            const uint32_t place = (ch0 + i) & ((1u << lg.log2_group) - 1u);
            wave_lds_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j) word[64 * j] = A[j];
            wave_lds_fence();
            if (lane < n_en[i] && (en[i] >> 27) == place) parked[(en[i] >> 16) & 2047u] = (uint16_t)en[i];
            for (uint32_t k = 64u + lane; k < n_en[i]; k += 64u) {  // a tile with more entries than lanes
                const uint32_t e = entries[lo[i] + k];
                if ((e >> 27) == place) parked[(e >> 16) & 2047u] = (uint16_t)e;
            }
            wave_lds_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j) A[j] = word[64 * j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) out[i * GEMM_TILE_WORDS + 64 * j] = A[j];
    }
}

// The product over the decoded tiles, with the tile and the steps of gemm_wide_kernel: 256 rows x 128 tokens per
// workgroup of eight waves, one chunk of 64 columns per step, three LDS buffers, each wave bringing in one row tile of the
// chunk after the next and its share of x, the quarter's LDS reads under way while the one before is multiplied.  The same
// additions in the same order: where the columns are split alike, the results are gemm_wide_kernel's bit for bit.
//   What bounds it: of a chunk's 2150 clocks the matrix cores are busy 1024, the LDS unit 912, the vector units 767 (12288 x
// 4096, 2000 tokens, with a list, at the 1.81 GHz that the card holds meanwhile); 1.04 to 1.19 PFLOP/s, where a large product
// of the library reaches 1.17 to 1.22.  One product per two LDS reads in the order of issue: 2 to 3 % faster than four products
// after four reads; the waves' priority raised for the products 4 to 8 % slower; the tiles' sums carried in turns no difference.
//   2000 tokens with a list, gemm_wide_kernel -> decoding and this: 4096 x 4096 127 -> 102 us, 12288 x 4096 353 -> 252, 22016 x
// 4096 649 -> 482, 8192 x 28672 1305 -> 1042.
template <bool CARRY>
__global__ __launch_bounds__(64 * GEMM_WIDE_WAVES, 2) void gemm_decoded_kernel(
    const uint4* __restrict__ decoded, uint32_t first_row, uint32_t n_rt, uint32_t rows, uint32_t n_chunks,
    const uint4* __restrict__ xp, uint32_t tok_tiles, uint32_t tok_groups, uint32_t per_split, uint32_t flush,
    uint32_t n_tokens, float* __restrict__ y, float* __restrict__ parts) {
    struct Shared {
        uint4 a[3][GEMM_WIDE_WAVES][GEMM_TILE_WORDS];
        uint4 b[3][GEMM_WIDE_TOK_TILES][GEMM_TILE_WORDS];
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (as in gemm_wide_kernel: each die takes a contiguous run of tiles, token groups fastest)
    uint32_t id = blockIdx.x;
    {
        const uint32_t total = gridDim.x, q = total / 8, rem = total % 8, die = id % 8;
        id = die * q + min(die, rem) + id / 8;
    }
    const uint32_t row_groups = (n_rt + GEMM_WIDE_WAVES - 1) / GEMM_WIDE_WAVES;
    const uint32_t tg = id % tok_groups, rg = (id / tok_groups) % row_groups, part = id / (tok_groups * row_groups);
    const uint32_t ch0 = part * per_split, ch1 = min(n_chunks, ch0 + per_split), n_steps = ch1 - ch0;
    // a row tile or token tile past the last is read from the last one and not stored
    const uint4* my_a = decoded + (uint64_t)min(rg * GEMM_WIDE_WAVES + wave, n_rt - 1) * n_chunks * GEMM_TILE_WORDS + lane;
    const uint4* my_x = xp + (uint64_t)min(tg * GEMM_WIDE_TOK_TILES + (wave >> 1), tok_tiles - 1) * n_chunks * GEMM_TILE_WORDS +
                        (wave & 1) * 128 + lane;
    struct Ahead {  // what a wave brings into LDS for one chunk
        uint4 a0, a1, a2, a3, x0, x1;
    };
    auto fetch = [&](uint32_t nth) __attribute__((always_inline)) {
        const uint64_t at = (uint64_t)min(ch0 + nth, ch1 - 1) * GEMM_TILE_WORDS;
        const uint4 *a = my_a + at, *x = my_x + at;
        Ahead o;
        o.a0 = a[0];
        o.a1 = a[64];
        o.a2 = a[128];
        o.a3 = a[192];
        o.x0 = x[0];
        o.x1 = x[64];
        return o;
    };
    gemm_f32x16 acc[2][2], sum[2][2];  // [row tile][token tile]
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][t][i] = sum[r][t][i] = 0.0f;
    const uint32_t wr = 2 * (wave & 3), wt = 2 * (wave >> 2);  // first row tile and token tile that the wave multiplies
    struct Operands {
        gemm_bf16x8 a[2], b[2];
    };
    auto read_operands = [&](uint32_t buf, int j) __attribute__((always_inline)) {
        const gemm_bf16x8* a = reinterpret_cast<const gemm_bf16x8*>(sh.a[buf][wr]) + lane;
        const gemm_bf16x8* b = reinterpret_cast<const gemm_bf16x8*>(sh.b[buf][wt]) + lane;
        const Operands o = {{a[64 * j], a[GEMM_TILE_WORDS + 64 * j]}, {b[64 * j], b[GEMM_TILE_WORDS + 64 * j]}};
        return o;
    };
    auto store_quarter = [&](const Ahead o, uint32_t buf, int j) __attribute__((always_inline)) {
        sh.a[buf][wave][64 * j + lane] = j == 0 ? o.a0 : j == 1 ? o.a1 : j == 2 ? o.a2 : o.a3;
        if (j >= 2) sh.b[buf][wave >> 1][(wave & 1) * 128 + 64 * (j - 2) + lane] = j == 2 ? o.x0 : o.x1;
    };
    uint32_t until_flush = flush;
    // Before step s: buffer s % 3 holds chunk s and buffer (s + 1) % 3 chunk s + 1; `o` is chunk s + 2, on its way since the
    // step before; chunk s + 3 is asked for during the step; `op` are the operands of the step's first quarter.
    Operands op;
    auto step = [&](uint32_t s, const uint32_t buf, const Ahead o) __attribute__((always_inline)) {
        const uint32_t buf1 = buf == 2u ? 0u : buf + 1u, buf2 = buf == 0u ? 2u : buf - 1u;
        const Ahead asked = fetch(s + 3);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const Operands next = read_operands(j < 3 ? buf : buf1, (j + 1) & 3);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[r][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.b[t], op.a[r], acc[r][t], 0, 0, 0);
            store_quarter(o, buf2, j);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            op = next;
        }
        if (--until_flush == 0u) {
            until_flush = flush;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        if (CARRY) {
                            gemm_carry(sum[r][t], acc[r][t], i);
                        } else {
                            sum[r][t][i] += acc[r][t][i];
                            acc[r][t][i] = 0.0f;
                        }
                    }
        }
        __syncthreads();
        return asked;
    };
    Ahead o0;
    {
        const Ahead first = fetch(0), second = fetch(1);
        o0 = fetch(2);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            store_quarter(first, 0, j);
            store_quarter(second, 1, j);
        }
        __syncthreads();
        op = read_operands(0, 0);
    }
    // Six steps to a round, so that neither the buffers' places nor the registers of what is on its way move (a copy of a
    // register that is being loaded waits for the load).
    uint32_t s = 0;
    for (uint32_t rounds = n_steps / 6; rounds > 0; --rounds, s += 6) {
        const Ahead o1 = step(s, 0, o0);
        const Ahead o2 = step(s + 1, 1, o1);
        const Ahead o3 = step(s + 2, 2, o2);
        const Ahead o4 = step(s + 3, 0, o3);
        const Ahead o5 = step(s + 4, 1, o4);
        o0 = step(s + 5, 2, o5);
    }
    if (s < n_steps) {
        const Ahead o1 = step(s, 0, o0);
        if (s + 1 < n_steps) {
            const Ahead o2 = step(s + 1, 1, o1);
            if (s + 2 < n_steps) {
                const Ahead o3 = step(s + 2, 2, o2);
                if (s + 3 < n_steps) {
                    const Ahead o4 = step(s + 3, 0, o3);
                    if (s + 4 < n_steps) step(s + 4, 1, o4);
                }
            }
        }
    }
    // the first part goes to the result itself, where gemm_sum_kernel adds the others to it
    float* out = part == 0 ? y : parts + (uint64_t)(part - 1) * n_tokens * rows;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint32_t rt = rg * GEMM_WIDE_WAVES + wr + r, row = first_row + rt * GEMM_ROWS + (lane & 31);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t tok0 = (tg * GEMM_WIDE_TOK_TILES + wt + t) * GEMM_TOKENS + 4 * (lane >> 5);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t tok = tok0 + 8 * (i >> 2) + (i & 3);
                if (rt < n_rt && row < rows && tok < n_tokens) out[(uint64_t)tok * rows + row] = sum[r][t][i] + acc[r][t][i];
            }
        }
    }
}

// y = the partial results in order (count elements each): the first, which may stand in y itself, and n_more others.
__global__ __launch_bounds__(256) void gemm_sum_kernel(const float* first, const float* __restrict__ more, uint32_t n_more,
                                                       uint64_t count, float* y) {
    const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= count) return;
    double s = first[idx];
    for (uint32_t k = 0; k < n_more; ++k) s += more[k * count + idx];
    y[idx] = (float)s;
}

}  // namespace bof4
