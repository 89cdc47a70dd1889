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
// matrix once, x per call), so that every load of a wave is one run of consecutive bytes.  Lane l supplies
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

#include <cstdint>

#include "bof4_device.h"
#include "bof4_segment.h"
#include "bof4_gemv.h"

namespace bof4 {

constexpr uint32_t GEMM_ROWS = 32;    // rows per tile (M of the matrix-core product)
constexpr uint32_t GEMM_MAX_R = 2;    // tiles of rows per workgroup: each word of x read serves up to 64 rows
constexpr uint32_t GEMM_TOKENS = 32;  // tokens per tile (N of the matrix-core product)
constexpr uint32_t GEMM_MAX_TILES = 4;  // token tiles per launch: the codes are decoded once per 128 tokens
constexpr uint32_t GEMM_CHUNK = 64;   // columns per wave and step: four products of K = 16
constexpr uint32_t GEMM_MAX_WAVES = 8;
// Workgroups wanted before the columns are also split over workgroups: three quarters of the 256 compute units.
// Measured: splitting further (to 256, 512 or 1024 workgroups) costs more in partial results and in the epilogue per
// workgroup than the fuller chip gains; fewer than 192 leave too much of it idle.
constexpr uint32_t GEMM_TARGET_WGS = 192;

typedef __bf16 gemm_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 gemm_bf16x2 __attribute__((ext_vector_type(2)));
typedef float gemm_f32x2 __attribute__((ext_vector_type(2)));
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
// entries of row tile rt and column group g begin (a group: 2^log2_group chunks of 64 columns, as fine as the table's
// size allows - one chunk for all but a few odd row counts), with one closing value; an entry is one 32-bit word:
//   bits 0 .. 15 the value as the decoder stores it (bfloat16), bits 16 .. 26 where it goes in the tile's decoded
//   operand - 16-byte word (product j, lane) and place in it, j * 512 + lane * 8 + column % 8 -, bits 27 .. 31 which
//   chunk of its group it belongs to.
// The list ascends, so the entries of 32 rows are one run of it and every workgroup sorts its own run: it counts the
// run's entries per group, turns the counts into places, and deals the entries out.  (Within a tile their order does
// not matter: they go to different places.)  Entries outside the matrix lie before or behind all runs.
struct GemmListGeometry {
    uint32_t n_groups, log2_group;
};
__device__ __forceinline__ uint32_t list_lower_bound(const int64_t* __restrict__ out_idx, uint32_t n_out, int64_t target) {
    uint32_t lo = 0, hi = n_out;  // first entry >= target
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (out_idx[mid] < target) lo = mid + 1; else hi = mid;
    }
    return lo;
}
constexpr uint32_t GEMM_MAX_CHUNKS = GEMV_MAX_STRIPS * GEMV_STRIP / GEMM_CHUNK;  // 512: 32768 columns
__global__ __launch_bounds__(256) void gemm_list_kernel(const int64_t* __restrict__ out_idx,
                                                        const uint16_t* __restrict__ out_val, uint32_t n_out,
                                                        uint64_t rows, uint32_t cols, GemmListGeometry lg,
                                                        uint32_t* __restrict__ ptr, uint32_t* __restrict__ entries) {
    __shared__ uint32_t place[GEMM_MAX_CHUNKS];
    __shared__ uint32_t range[2];
    const uint32_t tid = threadIdx.x, rt = blockIdx.x, group_cols = GEMM_CHUNK << lg.log2_group;
    if (tid < 2) {
        const uint64_t r = min((uint64_t)(rt + tid) * GEMM_ROWS, rows);
        range[tid] = list_lower_bound(out_idx, n_out, (int64_t)(r * cols));
    }
    for (uint32_t i = tid; i < lg.n_groups; i += 256) place[i] = 0u;
    __syncthreads();
    const uint32_t a = range[0], b = range[1];
    const uint64_t row0 = (uint64_t)rt * GEMM_ROWS;
    for (uint64_t k = (uint64_t)a + tid; k < b; k += 256) {
        const uint32_t c = (uint32_t)(((uint64_t)out_idx[k] - row0 * cols) % cols);
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
    if (tid == 0 && rt == gridDim.x - 1) ptr[(uint64_t)gridDim.x * lg.n_groups] = b;
    __syncthreads();
    for (uint64_t k = (uint64_t)a + tid; k < b; k += 256) {
        const uint64_t off = (uint64_t)out_idx[k] - row0 * cols;
        const uint32_t r = (uint32_t)(off / cols), c = (uint32_t)(off % cols), cc = c % GEMM_CHUNK;
        const uint32_t lane = 32 * (cc >> 5) + r, j = (cc >> 3) & 3u;
        const uint32_t val = f32_to_bf16_rne(f16_bits_to_f32(out_val[k]));
        entries[atomicAdd(&place[c / group_cols], 1u)] =
            val | ((j * 512 + lane * 8 + (cc & 7u)) << 16) | ((c % group_cols / GEMM_CHUNK) << 27);
    }
}

// Workgroup (b, s): R tiles of 32 rows (32 R b ..), the chunks s * waves + wave, + n_split * waves, ... of the row,
// NT tiles of 32 tokens (tile0 ..).  Its sum goes to dst[(s * n_tokens + token) * rows + row], token counted from
// the first of tile0: the result itself when n_split is 1, else one of n_split partial results that gemm_sum_kernel
// adds.  With a list the wave parks the decoded operand of a tile in LDS, writes the tile's entries over their
// placeholders and reads the operand back (one wave, one buffer: no barrier).  Against adding (value - placeholder) *
// x per entry and token to the row sums afterwards, as this kernel did before, four matrices of a
// Llama-70B-shaped layer with 0.9 % outliers take 388 us instead of 643 for 128 tokens.
// The packed matrix holds a multiple of GEMM_MAX_R row tiles.
template <int R, int NT, bool OUTLIERS>
__global__ __launch_bounds__(64 * GEMM_MAX_WAVES) void gemm_kernel(
    const char* __restrict__ packed, uint32_t rows, uint32_t cols, CodebookArgs cb, const uint32_t* __restrict__ list_ptr,
    const uint32_t* __restrict__ entries, uint32_t n_out, GemmListGeometry lg, uint32_t row_tiles,
    const uint4* __restrict__ xp, uint32_t tile0, uint32_t n_tokens, float* __restrict__ dst) {
    struct Shared {
        float tab[16];
        float red[GEMM_MAX_WAVES * 16 * 64];         // per wave: accumulator register i of lane l at [i * 64 + l]; in
                                                     // the loop over chunks, with a list, the wave's decoded operand
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63, n_waves = blockDim.x >> 6;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 16) sh.tab[tid] = cb.lv32[tid];
    __syncthreads();
    const char* tab = reinterpret_cast<const char*>(sh.tab);
    const uint32_t n_chunks = (cols + GEMM_CHUNK - 1) / GEMM_CHUNK;
    const uint32_t stride = gridDim.y * n_waves;

    gemm_f32x16 acc[R][NT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][t][i] = 0.0f;

    // What the chunk after this one needs (codes, constants and - where the registers allow it - x) is on its way
    // while this one is decoded and multiplied, in two sets of registers used in turn.  Past the last chunk the last
    // one is read again and not used.
    constexpr bool X_AHEAD = R * NT <= 2;
    struct Operands {
        uint4 q[R], xb[NT][4];
        uint16_t m[R];
        uint32_t en[R], n_en[R];  // this lane's list entry of the tile, and how many entries the tile has
    };
    auto fetch_x = [&](Operands& o, uint32_t chunk) {
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
                e_lo[r] = min(p[0], n_out);
                e_hi[r] = min(p[1], n_out);
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
    float* mine = sh.red + wave * 16 * 64;
    uint16_t* parked = reinterpret_cast<uint16_t*>(mine);
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
    Operands o0, o1;
    uint32_t ch = ch_first;
    const uint32_t last = n_chunks - 1;
    const uint32_t n_iter = ch < n_chunks ? (last - ch) / stride + 1 : 0;
    uint32_t nth = 0;  // how many chunks this wave has taken
    fetch(o0, min(ch, last), 0);
    if (n_iter & 1u) {  // an odd one first, so that the rest goes in pairs
        multiply(o0, ch, 0);
        ch += stride;
        nth = 1;
        fetch(o0, min(ch, last), min(nth, 63u));
    }
    for (uint32_t it = n_iter >> 1; it > 0; --it) {  // o0 holds chunk ch
        fetch(o1, ch + stride, nth + 1);
        __builtin_amdgcn_sched_barrier(0);  // the loads first, then the arithmetic
        multiply(o0, ch, nth);
        fetch(o0, min(ch + 2 * stride, last), min(nth + 2, 63u));
        __builtin_amdgcn_sched_barrier(0);
        multiply(o1, ch + stride, nth + 1);
        ch += 2 * stride;
        nth += 2;
    }

    float* out = dst + (uint64_t)blockIdx.y * n_tokens * rows;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t r0 = (blockIdx.x * R + r) * GEMM_ROWS;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (r > 0 || t > 0) __syncthreads();  // the sums of the round before have been read
#pragma unroll
            for (int i = 0; i < 16; ++i) mine[i * 64 + lane] = acc[r][t][i];
            __syncthreads();
            // The waves' results in wave order.  Accumulator i of lane l: row 8 (i / 4) + 4 (l / 32) + i % 4 of the
            // tile, token l % 32.
            for (uint32_t idx = tid; idx < 16 * 64; idx += blockDim.x) {
                float s = 0.0f;
                for (uint32_t wv = 0; wv < n_waves; ++wv) s += sh.red[wv * 16 * 64 + idx];
                const uint32_t i = idx >> 6, l = idx & 63;
                const uint32_t mr = 8 * (i >> 2) + 4 * (l >> 5) + (i & 3u), n = 32 * t + (l & 31);
                if (r0 + mr < rows && n < n_tokens) out[(uint64_t)n * rows + r0 + mr] = s;
            }
        }
    }
}

// y = the n_split partial results in order (count elements each).
__global__ __launch_bounds__(256) void gemm_sum_kernel(const float* __restrict__ part, uint32_t n_split, uint64_t count,
                                                       float* __restrict__ y) {
    const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= count) return;
    float s = 0.0f;
    for (uint32_t k = 0; k < n_split; ++k) s += part[k * count + idx];
    y[idx] = s;
}

}  // namespace bof4
