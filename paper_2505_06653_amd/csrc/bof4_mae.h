// bof4_mae.h - Lloyd step under the MAE criterion (section 3.2 eq. 7-8, appendix B.4): per region the weighted
// median of the normalised weights, weighted by the absolute block maximum - or, on request, the plain median of
// appendix D (every weight one unit).
//
// A weighted median over 10^8 samples is found without sorting, by a radix search on an order-preserving integer
// key of x.  Region l can only hold keys between klo[l] (its lower threshold) and its upper threshold, so the search
// runs on sub = key - klo[l], which has bits[l] <= 31 significant bits; every pass over the weights fixes the next 8
// of them: a histogram of the weight that falls on each value of those 8 bits (among the elements that agree with
// the bits fixed so far), then the smallest value d for which twice the weight up to and including d reaches the
// region's total.  Three passes settle an ordinary region, four the one that contains zero (its keys span both
// signs).  Weights are exact integers, |block constant| * 2^24 (the constant is a binary16 number), added in 64
// bits; additions of integers commute, so the result does not depend on the order of the atomics.
// The second pass also writes every element that agrees with the first digit of its region (about one in 200) to a
// list - key, region and block constant in 8 bytes - and the passes after it read that list instead of the weights.
// Every wave appends to a region of its own; if one of them runs full (a tensor of equal numbers), the later passes
// scan the weights as before.
// Large tensors get by with ONE pass over all the weights: a first-digit histogram over one tile in 8 to 64 (picked by a
// hash of the tile number) says where every region's median will be to within a few digits; the full pass
// (mae_window_kernel) then adds up what lies below that window and in all, and writes the elements inside to the list.
// If the exact first digit of every region falls inside its window (it does unless the sampled tiles differ from the
// rest), all later passes read the list.  If not, the first pass follows after all, without the sums and counts that
// mae_window_kernel has taken already; and then, or if the list ran full, the second pass writes the list anew.
//
// What is computed is "the smallest x_k with 2 * sum_{x_j <= x_k} a_j >= sum_j a_j" - the lower weighted median,
// which minimises sum a_j |x_j - c|.  (The closing formula of appendix B.4 names the element before it; its own
// derivation puts the minimum where this rule does.)
#pragma once
#include "bof4_segment.h"

namespace bof4 {

// Search state of one region, in the workspace.
struct MaeLevelState {
    uint32_t klo;     // key of the region's lower bound
    uint32_t hi;      // bits [hi, 32) of sub are fixed to `prefix`; 0 = finished
    uint32_t prefix;  // their value
    uint32_t pad;     // 1: the caller does not want this region's median (no search after the first pass)
    unsigned long long base;   // weight of the elements whose sub lies below prefix << hi
    unsigned long long total;  // weight of the whole region
    uint32_t win_lo;   // first digits win_lo .. win_lo + win_len - 1: what mae_window_kernel writes to the list
    uint32_t win_len;
};
// Per-region constants from the host: key range of the region.
struct MaeLevelConst {
    uint32_t klo[16];
    uint32_t bits[16];  // significant bits of (key of upper bound - klo)
};
constexpr int MAE_REC = 51;  // doubles of the result record (layout of bof4_mae_stats)
constexpr uint32_t MAE_PASS_WAVES = 8;  // waves that share one histogram in mae_pass_kernel: one workgroup per compute unit
constexpr uint32_t MAE_MAX_WGS = 768;  // most workgroups of a pass: the stride of the counts' records
// Tile t belongs to slot t mod n_slots.  The two floating-point sums are added up per slot, in ascending order of its
// tiles, and then over the slots in order, so that they do not depend on which kernel read the weights: a wave of
// mae_pass_kernel takes 3 slots, one of mae_window_kernel (whose grid holds half as many waves again) 2.
constexpr uint32_t MAE_SLOTS_PER_PASS_WAVE = 3;
constexpr uint32_t MAE_SLOTS_PER_WINDOW_WAVE = 2;
constexpr uint32_t MAE_WINDOW_WAVES = 3072;  // three per SIMD
// What became of the list, in the workspace.  Words after the first are there only where the step samples.
enum MaeListWord {
    MAE_LIST_UNUSABLE,   // 1: scan the weights
    MAE_DIGITS_MISSING,  // 1: mae_window_kernel did not find the regions' first digits
    MAE_DECLINED,        // 1: the sample says that the windows would take in too much: mae_window_kernel does not run
    MAE_NO_LIST_AT_ALL,  // 1: nor would the second pass's find room (few values)
    MAE_WINDOW_OUTCOME,  // MaeOutcome of mae_window_kernel's list, for who looks into it
    MAE_LIST_WORDS
};
enum MaeOutcome { MAE_LIST_SERVED, MAE_WINDOW_MISSED, MAE_STRETCH_FULL, MAE_LIST_DECLINED };
// Bins of all regions' windows together in mae_window_kernel.
constexpr uint32_t MAE_WINDOW_BINS = 1024;
// A wave-uniform number to scalar registers (divisions leave it in vector registers).
__device__ __forceinline__ uint64_t wave_uniform(uint64_t v) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
}
struct MaeTiles {
    uint64_t t, slot;  // the wave's next tile and its slot; slot >= n_slots: none
    uint64_t n_waves, n_slots, step, end;
    // Which tiles the sampling pass looks at: one in (sample_mask + 1), spread by a multiplicative hash so that the choice
    // does not follow the rows and columns of the matrices behind the tensor.  Its waves take contiguous stretches, in
    // which the hash is spread evenly (its sums are not used).
    uint32_t sample_mask;
    __device__ __forceinline__ bool more() const { return slot < n_slots; }
    __device__ __forceinline__ void settle() {  // to the first tile from t on that counts
        while (more()) {
            if (t >= end) t = slot = slot + n_waves;
            else if (sample_mask != 0u && (((uint32_t)t * 0x9E3779B1u) >> 16 & sample_mask) != 0u) t += step;
            else break;
        }
    }
    __device__ __forceinline__ MaeTiles next() const {
        MaeTiles m = *this;
        m.t += step;
        m.settle();
        return m;
    }
};
__device__ __forceinline__ MaeTiles mae_tiles(uint64_t wave, uint64_t n_waves, uint32_t slots_per_wave, uint64_t n_tiles,
                                              uint32_t sample_mask) {
    MaeTiles m = {wave, wave, n_waves, n_waves * slots_per_wave, n_waves * slots_per_wave, n_tiles, sample_mask};
    if (sample_mask != 0u) {
        m.t = wave_uniform(n_tiles * wave / n_waves);
        m.end = wave_uniform(n_tiles * (wave + 1) / n_waves);
        m.step = 1;
        m.n_slots = n_waves;
    }
    m.settle();
    return m;
}
struct MaeSlotSums {
    uint64_t slot;
    double sae, w_est;
    // The wave goes on in `next_slot`: store the sums of the slots before it (all lanes), of which it worked on `slot`.
    __device__ __forceinline__ void close_until(uint64_t next_slot, uint64_t n_waves, uint32_t lane, double* __restrict__ sae_part) {
        if (slot >= next_slot) return;
        double s = sae, we = w_est;
#pragma unroll
        for (int mk = 32; mk >= 1; mk >>= 1) {
            s += __shfl_xor(s, mk, 64);
            we += __shfl_xor(we, mk, 64);
        }
        for (; slot < next_slot; slot += n_waves) {
            if (lane == 0) {
                sae_part[2 * slot] = s;
                sae_part[2 * slot + 1] = we;
            }
            s = we = 0.0;
        }
        sae = w_est = 0.0;
    }
};

// Order-preserving map from binary32 to uint32 (negative numbers reversed below the positive ones).
__device__ __forceinline__ uint32_t order_key(float x) {
    const uint32_t b = __float_as_uint(x);
    return b ^ ((uint32_t)((int)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

// Sets up the search (state from the host's constants) and clears the accumulators.
__global__ __launch_bounds__(256) void mae_init_kernel(MaeLevelConst lc, MaeLevelState* __restrict__ state,
                                                       unsigned long long* __restrict__ hist) {
    const uint32_t t = blockIdx.x * 256 + threadIdx.x;
    if (t < 16 * 256) hist[t] = 0ull;
    if (t < 16) {
        MaeLevelState s;
        s.klo = lc.klo[t];
        s.hi = lc.bits[t];
        s.prefix = 0;
        s.pad = 0;
        s.base = 0ull;
        s.total = 0ull;
        s.win_lo = 0;
        s.win_len = 0;
        state[t] = s;
    }
}

// One pass over the weights, by KIND: the first one also counts the regions' elements and accumulates the error sum
// sum |block constant| |x - level| at the current codebook; the sampling pass is a first one over the sampled tiles
// without either (a third of its vector work).  A later pass reads the list where there is one and the words at `list` say
// that it can be used, and the weights where not: a stretch of at most cand_cap entries for every wave of a pass, or of
// window_cap for every wave of mae_window_kernel (0: that did not write it), cand_count of them filled.
enum MaePass { MAE_SAMPLE, MAE_FIRST, MAE_LATER };
template <int I, bool FAST, bool OPQ, MaePass KIND>
__global__ __launch_bounds__(64 * MAE_PASS_WAVES, 2) void mae_pass_kernel(const uint4* __restrict__ w, uint64_t n_seg, CodebookArgs cb,
                                                           BinTable bt, int signed_norm, double T2,
                                                           const MaeLevelState* __restrict__ state,
                                                           unsigned long long* __restrict__ hist_g,
                                                           unsigned long long* __restrict__ cnt_part,
                                                           double* __restrict__ sae_part,
                                                           unsigned long long* __restrict__ cand,
                                                           uint32_t* __restrict__ cand_count, uint32_t cand_cap,
                                                           const uint32_t* __restrict__ list, uint32_t window_cap,
                                                           int unweighted, uint32_t sample_mask, int second) {
    using C = SegCfg<I>;
    constexpr bool FIRST = KIND != MAE_LATER, SUMS = KIND == MAE_FIRST;
    // list != nullptr, a first pass: it follows mae_window_kernel, whose sums stand if it ran.  The second pass, where it
    // reads no list: append the elements that still count to this wave's stretch of it.
    if (FIRST && list != nullptr && list[MAE_DIGITS_MISSING] == 0u) return;
    const bool sums_too = SUMS && (list == nullptr || list[MAE_DECLINED] != 0u);
    const bool from_list = KIND == MAE_LATER && list != nullptr && list[MAE_LIST_UNUSABLE] == 0u;
    struct Shared {  // one object, so that the table sits at LDS offset 0 (reachable by an immediate offset)
        uint2 tab[BIN_TABLE_ENTRIES];
        uint4 info[16];    // per region: klo, (lo | hi << 8 | digit mask << 16), then prefix and active flag; in
                           // the first pass (no prefix yet, every region active, its key range has exactly hi bits):
                           // klo, lo, the region's level as binary64
        unsigned long long hist[16 * 256];
        uint32_t cntcol[MAE_PASS_WAVES * 8 * 64];  // per lane, two 16-bit counters per word: regions 2p and 2p + 1
        unsigned long long cnt[17];              // the workgroup's counts of the regions, and of outliers
        char stage[MAE_PASS_WAVES * C::STAGE_BYTES] __attribute__((aligned(16)));  // (off 16 bytes: 35 % slower)
        uint16_t tie[MAE_PASS_WAVES * TIE_BUF_HALFWORDS] __attribute__((aligned(16)));
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    bin_table_fill(sh.tab, bt, tid, blockDim.x);
    if (tid < 17) sh.cnt[tid] = 0ull;
    if (tid < 16) {
        const MaeLevelState s = state[tid];
        const uint32_t hi = s.hi, lo = hi > 8 ? hi - 8 : 0;
        const uint32_t packed = lo | (hi << 8) | (((1u << (hi - lo)) - 1u) << 16);
        if (FIRST) {
            const unsigned long long lv = (unsigned long long)__double_as_longlong(cb.cb64[tid]);
            sh.info[tid] = make_uint4(s.klo, lo, (uint32_t)lv, (uint32_t)(lv >> 32));
        } else {
            sh.info[tid] = make_uint4(s.klo, packed, s.prefix, (hi != 0 && s.total != 0ull && s.pad == 0u) ? 1u : 0u);
        }
    }
    for (uint32_t i = tid; i < 16 * 256; i += 64 * MAE_PASS_WAVES) sh.hist[i] = 0ull;
    uint32_t* cntcol = sh.cntcol + wave * 8 * 64;
    if (SUMS) {
#pragma unroll
        for (int p = 0; p < 8; ++p) cntcol[p * 64 + lane] = 0u;
    }
    __syncthreads();
    if (from_list) {
        const uint64_t n_waves = (uint64_t)gridDim.x * MAE_PASS_WAVES;
        const bool by_windows = window_cap != 0u && list[MAE_WINDOW_OUTCOME] == MAE_LIST_SERVED;
        const uint64_t n_stretches = by_windows ? MAE_WINDOW_WAVES : n_waves;
        const uint32_t cap = by_windows ? window_cap : cand_cap;
        // every stretch in two halves, its even and odd runs of 512 entries: 3072 stretches deal out evenly to 2048 waves
        constexpr uint32_t AHEAD = 8, RUN = 64 * AHEAD;  // loads in flight per lane
        for (uint64_t half = (uint64_t)blockIdx.x * MAE_PASS_WAVES + wave; half < 2 * n_stretches; half += n_waves) {
            const uint32_t count = cand_count[half >> 1];  // at most cap, or the list would count as full
            const unsigned long long* mine = cand + (half >> 1) * cap;
            for (uint32_t i0 = ((uint32_t)half & 1u) * RUN + lane; i0 < count; i0 += 2 * RUN) {
                unsigned long long e[AHEAD];
#pragma unroll
                for (uint32_t u = 0; u < AHEAD; ++u) e[u] = mine[min(i0 + 64 * u, count - 1)];
#pragma unroll
                for (uint32_t u = 0; u < AHEAD; ++u) {
                    const uint32_t sub = (uint32_t)e[u], l = (uint32_t)(e[u] >> 32) & 15u, m15 = (uint32_t)(e[u] >> 36) & 0x7fffu;
                    const uint4 inf = sh.info[l];
                    const uint32_t lo = inf.y & 0xffu, hi = (inf.y >> 8) & 0xffu, dmask = inf.y >> 16;
                    if (i0 + 64 * u < count && inf.w != 0u && (sub >> hi) == inf.z) {
                        const float a = f16_bits_to_f32(m15);
                        const unsigned long long W =
                            (a < 65536.0f) ? (unweighted ? 1ull : (unsigned long long)((double)a * 16777216.0)) : 0ull;
                        atomicAdd(&sh.hist[l * 256 + ((sub >> lo) & dmask)], W);
                    }
                }
            }
        }
        __syncthreads();
        for (uint32_t i = tid; i < 16 * 256; i += 64 * MAE_PASS_WAVES) {
            const unsigned long long v = sh.hist[i];
            if (v != 0ull) atomicAdd(&hist_g[i], v);
        }
        return;
    }
    const bool writes_list = KIND == MAE_LATER && second != 0 && (list == nullptr || list[MAE_NO_LIST_AT_ALL] == 0u);
    const uint2* tab = sh.tab;
    const uint32_t lane_off = bin_lane_offset(threadIdx.x & 63u);
    char* stage = sh.stage + wave * C::STAGE_BYTES;
    uint16_t* tie_buf = sh.tie + wave * TIE_BUF_HALFWORDS;
    const uint64_t n_vec = n_seg * C::NV;
    const uint64_t n_tiles = (n_seg + 63) / 64;
    const uint64_t n_waves = (uint64_t)gridDim.x * MAE_PASS_WAVES;
    const uint64_t gw = (uint64_t)blockIdx.x * MAE_PASS_WAVES + wave;

    // outliers were zeroed: they ran through the loop as x = +0 of the zero region and are taken out again
    const uint32_t cz = bt.code_of_zero;
    const uint32_t key0 = order_key(0.0f);
    MaeTiles at = mae_tiles(gw, n_waves, MAE_SLOTS_PER_PASS_WAVE, n_tiles, sample_mask);
    MaeSlotSums sums = {gw, 0.0, 0.0};
    uint32_t kout = 0, tiles_since_flush = 0;
    uint32_t wave_cand = 0;  // entries this wave has appended to the list (wave-uniform; may pass the capacity)
    uint2* my_cand = reinterpret_cast<uint2*>(cand) + gw * cand_cap;  // this wave's stretch of the list
    // The 16-bit lane counters are added up over the wave before they can overflow; lane l < 16 keeps the wave's count
    // of region l.  (Every wave adding its counts to 17 words in memory at the end of the kernel cost more than the pass.)
    unsigned long long wave_cnt = 0ull;
    auto flush_counts = [&]() {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const uint32_t v = cntcol[p * 64 + lane];
            cntcol[p * 64 + lane] = 0u;
            uint32_t c0 = v & 0xffffu, c1 = v >> 16;  // at most 65535 each: the wave's sum fits 32 bits
#pragma unroll
            for (int mk = 32; mk >= 1; mk >>= 1) {
                c0 += (uint32_t)__shfl_xor((int)c0, mk, 64);
                c1 += (uint32_t)__shfl_xor((int)c1, mk, 64);
            }
            if (lane == 2u * p) wave_cnt += c0;
            if (lane == 2u * p + 1u) wave_cnt += c1;
        }
    };
    uint4 G[C::NV];
    uint32_t R[C::NR];
    if (at.more()) tile_issue_loads<I>(w, at.t * 64 * C::NV, n_vec, lane, G);
    if (SUMS && sums_too) sums.close_until(at.slot, n_waves, lane, sae_part);
    for (MaeTiles next; at.more(); at = next) {  // wave-uniform
        next = at.next();
        const uint64_t t = at.t;
        wave_lds_fence();
        tile_stage<I>(stage, lane, G);
        if (next.more()) tile_issue_loads<I>(w, next.t * 64 * C::NV, n_vec, lane, G);
        wave_lds_fence();
        tile_fetch<I>(stage, lane, R);
        const uint64_t seg = t * 64 + lane;
        const bool active = seg < n_seg;
        uint32_t k_out = 0;
        if (OPQ) {
            uint32_t omap[2];
            opq_zero_outliers<I>(R, opq_theta<I>(R, T2), omap);
            k_out = opq_count(omap);
        }
        uint32_t maxabs, sign;
        block_constant<I>(R, lane, signed_norm != 0, maxabs, sign, tie_buf);
        const float m = bf16_bits_to_f32(maxabs | (sign << 15));
        const float m_eff = f16_bits_to_f32(f32_to_f16_bits(m));
        const float a = fabsf(m_eff);
        // |block constant| in units of 2^-24; a constant beyond binary16 (infinite) carries no weight
        // (unweighted: the plain median of the normalised weights - every element of such a block weighs one unit)
        const unsigned long long W =
            (a < 65536.0f) ? (unweighted ? 1ull : (unsigned long long)((double)a * 16777216.0)) : 0ull;
        const double a_sum = unweighted ? 1.0 : (double)a;  // what an element's |x - level| counts with in the error sum
        const bool fast = FAST && __builtin_amdgcn_ballot_w64(!maxabs_is_ordinary(maxabs)) == 0;
        const uint32_t m15_shifted = (f32_to_f16_bits(a) & 0x7fffu) << 4;
        if (active) {
            const BlockDiv dv = make_block_div(m_eff);
            double dsum = 0.0;
            // batches of 8: the table reads of a batch are issued together, then the reads of the regions' search
            // state, then the (few) histogram additions - two dependent LDS round trips per batch instead of per weight
#pragma unroll
            for (int b0 = 0; b0 < C::SEG; b0 += 8) {
                float x[8];
                uint32_t code[8];
                if (fast) {
                    uint2 en[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        x[e] = div_fast(seg_f32(R, b0 + e), dv);
                        en[e] = bin_lookup(tab, x[e], lane_off);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) code[e] = en[e].y + (x[e] > __uint_as_float(en[e].x) ? 1u : 0u);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float f = seg_f32(R, b0 + e);
                        x[e] = (m_eff == 0.0f) ? 0.0f : f / m_eff;
                        code[e] = (uint32_t)assign_code_generic(x[e], cb);
                    }
                }
                uint4 inf[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) inf[e] = sh.info[code[e]];
                uint32_t bin[8], subk[8];
                bool counts[8], any = false;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t sub = order_key(x[e]) - inf[e].x;
                    subk[e] = sub;
                    if (FIRST) {
                        // the region's keys span exactly its hi bits, of which the first pass takes the top 8 (all of
                        // them if there are fewer): sub >> lo is the digit, and every element counts
                        bin[e] = code[e] * 256 + (sub >> (inf[e].y & 31u));
                        counts[e] = false;
                    } else {
                        const uint32_t lo = inf[e].y & 0xffu, hi = (inf[e].y >> 8) & 0xffu, dmask = inf[e].y >> 16;
                        counts[e] = inf[e].w != 0u && (sub >> hi) == inf[e].z;
                        bin[e] = code[e] * 256 + ((sub >> lo) & dmask);
                    }
                    any = any || counts[e];
                }
                if (FIRST) {  // every weight lands in some bin: no branches
#pragma unroll
                    for (int e = 0; e < 8; ++e) atomicAdd(&sh.hist[bin[e]], W);
                    if (SUMS && sums_too) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            atomicAdd(&cntcol[(code[e] >> 1) * 64 + lane], 1u << ((code[e] & 1u) * 16u));
                            dsum += fabs((double)x[e] - __hiloint2double((int)inf[e].w, (int)inf[e].z));
                            // pin the addition here: left alone, the compiler sinks all of them below the loop and keeps
                            // every x and level alive until then (it spilled 300 registers)
                            asm volatile("" : "+v"(dsum));
                        }
                    }
                } else if (__builtin_amdgcn_ballot_w64(any) != 0) {  // later passes: one weight in 256 still counts
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const unsigned long long who = __builtin_amdgcn_ballot_w64(counts[e]);
                        if (who == 0ull) continue;  // wave-uniform: three times out of four nobody's element e counts
                        if (counts[e]) atomicAdd(&sh.hist[bin[e]], W);
                        if (writes_list) {  // wave-uniform
                            const uint32_t pos = wave_cand + __builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
                            if (counts[e] && pos < cand_cap)  // entry: key | region << 32 | constant << 36
                                my_cand[pos] = make_uint2(subk[e], code[e] | m15_shifted);
                            wave_cand += (uint32_t)__builtin_popcountll(who);
                        }
                    }
                }
            }
            if (OPQ && k_out != 0u) {
                const uint4 inf = sh.info[cz];
                const uint32_t sub = key0 - inf.x;
                const uint32_t lo = FIRST ? (inf.y & 31u) : (inf.y & 0xffu), hi = (inf.y >> 8) & 0xffu;
                const uint32_t dmask = FIRST ? 0xffu : (inf.y >> 16);
                const bool counts = FIRST ? true : (inf.w != 0u && (sub >> hi) == inf.z);
                if (counts)
                    atomicAdd(&sh.hist[cz * 256 + ((sub >> lo) & dmask)], 0ull - (unsigned long long)k_out * W);
                if (SUMS && sums_too) {
                    atomicAdd(&cntcol[(cz >> 1) * 64 + lane], 0u - (k_out << ((cz & 1u) * 16u)));
                    dsum -= (double)k_out * fabs(__hiloint2double((int)inf.w, (int)inf.z));
                    kout += k_out;
                }
            }
            if (SUMS && sums_too) {
                sums.sae = fma(a_sum, dsum, sums.sae);
                sums.w_est = fma(a_sum, (double)(C::SEG - k_out), sums.w_est);
            }
        }
        if (SUMS && sums_too) sums.close_until(next.slot, n_waves, lane, sae_part);
        if (SUMS && sums_too && ++tiles_since_flush == 65535u / C::SEG) {
            flush_counts();
            tiles_since_flush = 0;
        }
    }
    if (SUMS && sums_too) {
        flush_counts();
        // counts leave as one record per workgroup, [17][MAE_MAX_WGS]
        uint32_t kc = kout;
#pragma unroll
        for (int mk = 32; mk >= 1; mk >>= 1) kc += (uint32_t)__shfl_xor((int)kc, mk, 64);
        if (lane < 17) atomicAdd(&sh.cnt[lane], lane == 16 ? (unsigned long long)kc : wave_cnt);
        __syncthreads();
        if (tid < 17) cnt_part[tid * MAE_MAX_WGS + blockIdx.x] = sh.cnt[tid];
    }
    if (writes_list && lane == 0) cand_count[gw] = wave_cand;
    __syncthreads();
    // 64-bit integer atomics: exact and order-free.  Eight waves share a histogram: with four, twice the atomics, a step on
    // 16.8 M weights took 97 us instead of 90.
    for (uint32_t i = tid; i < 16 * 256; i += 64 * MAE_PASS_WAVES) {
        const unsigned long long v = sh.hist[i];
        if (v != 0ull) atomicAdd(&hist_g[i], v);
    }
}

// bits = 2 bits + the lane's bit of `who` (an addition with carry; all lanes active).
__device__ __forceinline__ void shift_in(uint32_t& bits, uint64_t who) {
    uint64_t carry;
    asm("v_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(bits), "=s"(carry) : "s"(who));
}
// The one pass over all the weights of a large tensor.  The windows tell which elements can still be a median, so of
// all the others only the weight in all and below the window is needed, per region; both follow from counts per block,
// because a block's elements weigh the same.  Per weight one 32-bit LDS addition to a lane-private column (16 regions x
// 64 lanes: no two lanes share a bank) counts the element, and in the upper half-word whether it lies below its
// region's window; once per tile the columns are folded, with the block's weight, into binary64 registers that hold
// whole numbers below 2^53, and every 31 tiles those go to 64-bit integers.  Elements inside the window (about one in 100)
// are marked in a bit map per lane; after the tile the wave lists them, one lane takes each, reads its weight again, adds
// it to the histogram of first digits and writes it to the list.  At the end what lies below and above the window joins the
// bins beside it, so that the selection finds an ordinary first-digit histogram.
//   What bounds it: vector instructions, 21.8 per weight (17 for the weight itself, the rest for the fold, the block constant
// and the list), which keep the vector units busy for 83 % of the time; the LDS unit for 36 %.  855 M weights, block 64: 1043
// to 1093 us with a histogram of all elements (a 64-bit addition to a random bin and one for the count: 42 clocks of the LDS
// unit per 64 weights), now 655 to 680; the whole step 1240 -> 785 us.  Four waves per SIMD spill, and every reload waits for
// the next tile's pieces: 870 us.
template <int I, bool FAST, bool OPQ>
__global__ __launch_bounds__(256, 3) void mae_window_kernel(const uint4* __restrict__ w, uint64_t n_seg, CodebookArgs cb,
                                                            BinTable bt, int signed_norm, double T2,
                                                            const MaeLevelState* __restrict__ state,
                                                            unsigned long long* __restrict__ hist_g,
                                                            unsigned long long* __restrict__ cnt_part,
                                                            double* __restrict__ sae_part,
                                                            unsigned long long* __restrict__ cand,
                                                            uint32_t* __restrict__ cand_count, uint32_t cand_cap,
                                                            const uint32_t* __restrict__ list, int unweighted) {
    using C = SegCfg<I>;
    if (list[MAE_DECLINED] != 0u) return;
    struct Shared {  // one object, so that the table sits at LDS offset 0 (reachable by an immediate offset)
        uint2 tab[BIN_TABLE_ENTRIES];
        u32x4 info[16];  // per region: the level as binary64, the window's first value and the first one past it
        uint4 key[16];   // per region: klo, lo, the digit of its first bin, that bin's place
        unsigned long long hist[MAE_WINDOW_BINS];
        unsigned long long mass[16], below[16], cnt[17];
        uint32_t cols[WAVES_PER_WG * 16 * 64];
        uint16_t tie[WAVES_PER_WG * TIE_BUF_HALFWORDS] __attribute__((aligned(16)));
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    bin_table_fill(sh.tab, bt, tid, blockDim.x);
    if (tid < 17) sh.cnt[tid] = 0ull;
    if (tid < 16) {
        const MaeLevelState s = state[tid];
        const uint32_t lo = s.hi > 8 ? s.hi - 8 : 0;
        // The window as binary32 numbers, which compare -0 and +0 as equal: where an edge lies between the two zeros both
        // belong to the window.  No window: nothing is below, nothing inside.
        constexpr uint64_t KEY_INF = 0xff800000ull, KEY_ZERO = 0x80000000ull;
        float first = -__builtin_inff(), past = -__builtin_inff();
        if (s.win_len != 0u) {
            const uint64_t k0 = s.klo + ((uint64_t)s.win_lo << lo), k1 = s.klo + ((uint64_t)(s.win_lo + s.win_len) << lo);
            first = key_to_float((uint32_t)min(k0, KEY_INF));
            past = k1 == KEY_ZERO ? __uint_as_float(1u) : key_to_float((uint32_t)min(k1, KEY_INF));
        }
        const unsigned long long lv = (unsigned long long)__double_as_longlong(cb.cb64[tid]);
        sh.info[tid] = u32x4{(uint32_t)lv, (uint32_t)(lv >> 32), __float_as_uint(first), __float_as_uint(past)};
        uint32_t place = 0;  // a bin for each digit of the window and for the digits next to it
        for (uint32_t l = 0; l < tid; ++l) place += state[l].win_len + 2;
        sh.key[tid] = make_uint4(s.klo, lo, s.win_lo - 1, place);
        sh.mass[tid] = sh.below[tid] = 0ull;
    }
    for (uint32_t i = tid; i < MAE_WINDOW_BINS; i += 256) sh.hist[i] = 0ull;
    uint32_t* col = sh.cols + wave * 16 * 64;
#pragma unroll
    for (int l = 0; l < 16; ++l) col[l * 64 + lane] = 0u;
    __syncthreads();
    constexpr uint32_t ONE = 1u, ONE_BELOW = 0x10001u;
    const uint2* tab = sh.tab;
    const uint32_t lane_off = bin_lane_offset(lane);
    uint16_t* tie_buf = sh.tie + wave * TIE_BUF_HALFWORDS;
    const uint64_t n_tiles = (n_seg + 63) / 64;
    const uint64_t n_waves = (uint64_t)gridDim.x * WAVES_PER_WG;
    const uint64_t gw = (uint64_t)blockIdx.x * WAVES_PER_WG + wave;
    // fold: regions 4 p + k (k = 0 .. 3) of the blocks of lanes lane ^ c (c = 0 .. 3), as in the Lloyd pass
    const uint32_t p4 = (lane & 3u) * 4u;
    uint32_t* fold_col[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) fold_col[c] = col + p4 * 64 + (lane ^ (uint32_t)c);

    MaeTiles tiles = mae_tiles(gw, n_waves, MAE_SLOTS_PER_WINDOW_WAVE, n_tiles, 0u);
    MaeSlotSums sums = {gw, 0.0, 0.0};
    double mass[4], below[4];  // in units of 2^-24 (unweighted: of one), whole numbers
    uint32_t cnt[4], kout = 0, tiles_since_flush = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        mass[k] = below[k] = 0.0;
        cnt[k] = 0;
    }
    auto flush_masses = [&]() {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            atomicAdd(&sh.mass[p4 + k], (unsigned long long)mass[k]);
            atomicAdd(&sh.below[p4 + k], (unsigned long long)below[k]);
            mass[k] = below[k] = 0.0;
        }
    };
    uint32_t wave_cand = 0;  // entries this wave has appended to the list (wave-uniform; may pass the capacity)
    uint2* my_cand = reinterpret_cast<uint2*>(cand) + gw * cand_cap;  // this wave's stretch of the list
    // What a block's elements weigh: |block constant| in units of 2^-24; a constant beyond binary16 (infinite) carries no
    // weight (unweighted: every element of a block with a finite constant weighs one).
    auto weight_of = [&](float a) { return a < 65536.0f ? (unweighted ? 1.0 : (double)a * 16777216.0) : 0.0; };
    // An element inside its window: to the histogram and to place `pos` of the list.
    auto capture = [&](uint32_t raw, float m_own, bool fast, uint32_t pos) {
        const float f = bf16_bits_to_f32(raw);
        float x;
        uint32_t code;
        if (fast) {  // wave-uniform
            x = div_fast(f, make_block_div(m_own));
            const uint2 en = bin_lookup(tab, x, lane_off);
            code = en.y + (x > __uint_as_float(en.x) ? 1u : 0u);
        } else {
            x = (m_own == 0.0f) ? 0.0f : f / m_own;
            code = (uint32_t)assign_code_generic(x, cb);
        }
        const float a = fabsf(m_own);
        const uint4 key = sh.key[code];
        const uint32_t sub = order_key(x) - key.x;
        atomicAdd(&sh.hist[key.w + (sub >> key.y) - key.z], (unsigned long long)weight_of(a));
        if (pos < cand_cap)  // entry: key | region << 32 | constant << 36
            my_cand[pos] = make_uint2(sub, code | ((f32_to_f16_bits(a) & 0x7fffu) << 4));
    };

    uint32_t R[C::NR], Rn[C::NR];
    if (tiles.more()) {
        const uint4* p = own_segment<I>(w, tiles.t, n_seg, lane);
#pragma unroll
        for (int k = 0; k < C::NV; ++k) {
            const uint4 q = p[k];
            R[4 * k] = q.x;
            R[4 * k + 1] = q.y;
            R[4 * k + 2] = q.z;
            R[4 * k + 3] = q.w;
        }
    }
    sums.close_until(tiles.slot, n_waves, lane, sae_part);
    // The last tile's elements inside their windows, one per lane: their weights are sent for again (their lines were
    // fetched a moment ago) before the next tile's pieces and used after that tile.  Loads come back in order: sent for
    // after those pieces, each tile would wait for the next one to arrive from memory.
    uint32_t pend_n = 0, pend_entry = 0;
    float pend_m = 0.0f;
    bool pend_fast = false;
    const uint16_t* pend_w = nullptr;
    for (MaeTiles next; tiles.more(); tiles = next) {  // wave-uniform
        next = tiles.next();
        const uint64_t t = tiles.t;
        // (after the wave's last tile this requests that tile once more: cached, and never used)
        const uint4* pn = own_segment<I>(w, next.more() ? next.t : t, n_seg, lane);
        uint32_t pend_raw = 0;
        if (pend_n != 0u) pend_raw = pend_w[(pend_entry >> 6) * C::SEG + (pend_entry & 63u)];
        __builtin_amdgcn_sched_barrier(0);
        const bool active = t * 64 + lane < n_seg;
        uint32_t k_out = 0;
        if (OPQ) {
            uint32_t omap[2];
            opq_zero_outliers<I>(R, opq_theta<I>(R, T2), omap);
            k_out = active ? opq_count(omap) : 0u;
        }
        uint32_t maxabs, sign;
        block_constant<I>(R, lane, signed_norm != 0, maxabs, sign, tie_buf);
        const float m = bf16_bits_to_f32(maxabs | (sign << 15));
        const float m_eff = f16_bits_to_f32(f32_to_f16_bits(m));
        const float a = fabsf(m_eff);
        const double a_sum = unweighted ? 1.0 : (double)a;  // what an element's |x - level| counts with in the error sum
        const bool fast = FAST && __builtin_amdgcn_ballot_w64(!maxabs_is_ordinary(maxabs)) == 0;
        const BlockDiv dv = make_block_div(m_eff);
        double dsum = 0.0;
        uint32_t inside[2] = {0, 0};  // element 32 h + i: bit 31 - i of word h
        // Batches of four weights in a pipeline: while the regions of one batch are read, the next one's bins are; two
        // dependent LDS reads per weight, and neither is waited for right after it is sent.
        constexpr int B = 4;
        auto region_work = [&](const int b0, const float (&x)[B], const uint32_t (&code)[B], u32x4 (&inf)[B])
            __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < B; ++e) {
                asm volatile("" : "+v"(inf[e]));  // one read of 16 bytes (the compiler reads the level a second time)
                const bool from_first = x[e] >= __uint_as_float(inf[e].z);
                const uint64_t in = __builtin_amdgcn_ballot_w64(from_first) &
                                    __builtin_amdgcn_ballot_w64(x[e] < __uint_as_float(inf[e].w));
                atomicAdd(&col[code[e] * 64 + lane], from_first ? ONE : ONE_BELOW);
                shift_in(inside[b0 >> 5], in);
                dsum += fabs((double)x[e] - __hiloint2double((int)inf[e].y, (int)inf[e].x));
                // pin the addition here: left alone, the compiler sinks all of them below the loop and keeps every x and
                // level alive until then (it spilled 300 registers)
                asm volatile("" : "+v"(dsum));
            }
        };
        auto next_piece = [&](const int b0) __attribute__((always_inline)) {
            if (b0 % 8 == 0) {  // (these registers of R are free after the batch: the next tile's piece moves in)
                const uint4 q = pn[b0 / 8];
                Rn[b0 / 2] = q.x;
                Rn[b0 / 2 + 1] = q.y;
                Rn[b0 / 2 + 2] = q.z;
                Rn[b0 / 2 + 3] = q.w;
            }
        };
        if (fast) {
            float x[B], xn[B];
            uint2 en[B];
            auto send = [&](const int b0, float (&to)[B]) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < B; ++e) {
                    to[e] = div_fast(seg_f32(R, b0 + e), dv);
                    en[e] = bin_lookup(tab, to[e], lane_off);
                }
            };
            send(0, x);
#pragma unroll
            for (int b0 = 0; b0 < C::SEG; b0 += B) {
                uint32_t code[B];
                u32x4 inf[B];
#pragma unroll
                for (int e = 0; e < B; ++e) {
                    code[e] = en[e].y + (x[e] > __uint_as_float(en[e].x) ? 1u : 0u);
                    inf[e] = sh.info[code[e]];
                }
                __builtin_amdgcn_sched_barrier(0);
                if (b0 + B < C::SEG) send(b0 + B, xn);
                if (b0 % 8 == 8 - B) next_piece(b0 + B - 8);
                __builtin_amdgcn_sched_barrier(0);
                region_work(b0, x, code, inf);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < B; ++e) x[e] = xn[e];
            }
        } else {
#pragma unroll
            for (int b0 = 0; b0 < C::SEG; b0 += B) {
                float x[B];
                uint32_t code[B];
                u32x4 inf[B];
#pragma unroll
                for (int e = 0; e < B; ++e) {
                    const float f = seg_f32(R, b0 + e);
                    x[e] = (m_eff == 0.0f) ? 0.0f : f / m_eff;
                    code[e] = (uint32_t)assign_code_generic(x[e], cb);
                    inf[e] = sh.info[code[e]];
                }
                if (b0 % 8 == 8 - B) next_piece(b0 + B - 8);
                region_work(b0, x, code, inf);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (OPQ && k_out != 0u) {  // the zeroed outliers ran through as x = +0: take them out again
            uint32_t cz = bt.code_of_zero;
            asm volatile("" : "+s"(cz));  // (the address here, not in a spilled register: its load would wait for the next tile)
            const u32x4 info_z = sh.info[cz];
            const uint32_t inc_z = 0.0f >= __uint_as_float(info_z.z) ? ONE : ONE_BELOW;
            atomicAdd(&col[cz * 64 + lane], 0u - k_out * inc_z);
            dsum -= (double)k_out * fabs(__hiloint2double((int)info_z.y, (int)info_z.x));
            kout += k_out;
        }
        if (t * 64 + 64 > n_seg) {  // wave-uniform: the ragged last tile of the tensor
            wave_lds_fence();
            if (!active) {
#pragma unroll
                for (int l = 0; l < 16; ++l) col[l * 64 + lane] = 0u;
                inside[0] = inside[1] = 0u;
            }
        }
        if (active) {
            sums.sae = fma(a_sum, dsum, sums.sae);
            sums.w_est = fma(a_sum, (double)(C::SEG - k_out), sums.w_est);
        }
        // fold (all lanes)
        wave_lds_fence();
        {
            const float aw = a < 65536.0f ? (unweighted ? 0x1p-24f : a) : 0.0f;
            const float aq[4] = {aw, quad_xor<1>(aw), quad_xor<2>(aw), quad_xor<3>(aw)};
            uint32_t v[16];
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * c + k] = atomicExch(fold_col[c] + k * 64, 0u);  // read and clear
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double ac = (double)aq[c] * 16777216.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t n = v[4 * c + k] & 0xffffu;
                    mass[k] = fma(ac, (double)n, mass[k]);
                    below[k] = fma(ac, (double)(v[4 * c + k] >> 16), below[k]);
                    cnt[k] += n;
                }
            }
        }
        // a tile adds at most 4 blocks x 64 elements x 2^40 to a sum: 31 tiles stay below 2^53
        if (++tiles_since_flush == 31u) {
            flush_masses();
            tiles_since_flush = 0;
        }
        if (pend_n != 0u) {  // wave-uniform
            if (lane < pend_n) capture(pend_raw, pend_m, pend_fast, wave_cand + lane);
            wave_cand += pend_n;
        }
        // List this tile's elements inside their windows, (lane, element) in order, in the tie buffer (free here).
        uint32_t k_in = (uint32_t)__builtin_popcount(inside[0]) + (uint32_t)__builtin_popcount(inside[1]);
        const uint32_t incl = wave_inclusive_scan_u32(k_in);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        pend_n = min(total, 64u);
        if (total != 0u) {  // wave-uniform
            auto pop = [&]() {  // the first marked element
                const uint32_t h = inside[0] != 0u ? 0u : 1u, word = h == 0u ? inside[0] : inside[1];
                const uint32_t i = (uint32_t)__builtin_clz(word), cleared = word & ~(0x80000000u >> i);
                if (h == 0u) inside[0] = cleared;
                else inside[1] = cleared;
                return 32u * h + i;
            };
            pend_w = reinterpret_cast<const uint16_t*>(w) + t * 64 * C::SEG;
            pend_fast = fast;
            // up to TIE_BUF_HALFWORDS at a time: the last 64 of them wait, the others are done with here
            uint32_t at = incl - k_in;
            for (uint32_t from = 0; from < total; from += TIE_BUF_HALFWORDS) {
                while ((inside[0] | inside[1]) != 0u && at < from + TIE_BUF_HALFWORDS)
                    tie_buf[at++ - from] = (uint16_t)(pop() | (lane << 6));
                wave_lds_fence();
                const uint32_t n = min(total - from, (uint32_t)TIE_BUF_HALFWORDS);
                for (uint32_t i0 = 0; i0 < n; i0 += 64) {
                    pend_entry = i0 + lane < n ? tie_buf[i0 + lane] : 0u;
                    pend_m = __shfl(m_eff, (int)(pend_entry >> 6), 64);
                    pend_n = min(n - i0, 64u);
                    if (from + i0 + 64 < total) {
                        if (lane < pend_n)
                            capture(pend_w[(pend_entry >> 6) * C::SEG + (pend_entry & 63u)], pend_m, fast, wave_cand + lane);
                        wave_cand += pend_n;
                    }
                }
                wave_lds_fence();  // the buffer is read: it is filled again, or the search for the block constants uses it
            }
        }
        sums.close_until(next.slot, n_waves, lane, sae_part);
#pragma unroll
        for (int d = 0; d < C::NR; ++d) R[d] = Rn[d];
    }
    if (pend_n != 0u) {
        if (lane < pend_n)
            capture(pend_w[(pend_entry >> 6) * C::SEG + (pend_entry & 63u)], pend_m, pend_fast, wave_cand + lane);
        wave_cand += pend_n;
    }
    flush_masses();
#pragma unroll
    for (int k = 0; k < 4; ++k) atomicAdd(&sh.cnt[p4 + k], (unsigned long long)cnt[k]);
    atomicAdd(&sh.cnt[16], (unsigned long long)kout);
    if (lane == 0) cand_count[gw] = wave_cand;
    __syncthreads();
    if (tid < 17) cnt_part[tid * MAE_MAX_WGS + blockIdx.x] = sh.cnt[tid];
    // what lies below the window to the bin before it, what lies above to the bin behind it: 16 lanes per region
    const uint32_t l = tid >> 4, n_bins = state[l].win_len + 2, place = sh.key[l].w;
    unsigned long long in = 0ull;
    for (uint32_t i = tid & 15u; i < n_bins; i += 16) in += sh.hist[place + i];
#pragma unroll
    for (int mk = 8; mk >= 1; mk >>= 1) in += (unsigned long long)__shfl_xor((long long)in, mk, 64);
    __syncthreads();
    if ((tid & 15u) == 0u) {
        sh.hist[place] += sh.below[l];
        sh.hist[place + n_bins - 1] += sh.mass[l] - sh.below[l] - in;
    }
    __syncthreads();
    for (uint32_t i = tid & 15u; i < n_bins; i += 16) {
        const unsigned long long v = sh.hist[place + i];
        const uint32_t digit = state[l].win_lo + i - 1;  // (the bins outside 0 .. 255 stay empty)
        if (v != 0ull && digit < 256u) atomicAdd(&hist_g[l * 256 + digit], v);
    }
}

// After the sampling pass (over `sampled` elements): one wave per region reads the sampled first-digit histogram and sets the
// window of first digits that mae_window_kernel will capture: from the digit below which half of the sample's weight lies less
// six standard deviations of a sampled quantile (0.5 / sqrt(samples), widened by half for the unequal weights) to the one
// with as much more, and half a digit to either side of the sample's median.  (Not so many digits as the median's
// weight makes of six deviations: around zero a digit is an octave and holds next to nothing, and between the atoms of a
// tensor of some hundred values there are digits without any.  That took in most of the region or missed the next atom:
// 537 M Gaussian weights with the region around zero wanted 1992 us, now 660.)  Clears the bins.  The search state proper
// is left alone.  If the windows would take in more than 6 % of the weights (few values, many of them equal) or have more
// digits than mae_window_kernel has bins, it does not run: capturing would cost more than the first pass's histogram.  (Not
// already where they would fill the list: the digits it finds and its sums stand if a stretch runs full.)  And if the
// medians' digits alone would fill the list, no pass writes one.
__global__ __launch_bounds__(1024) void mae_predict_kernel(MaeLevelState* __restrict__ state,
                                                           unsigned long long* __restrict__ hist,
                                                           double sampled, uint32_t skip_mask, double list_room,
                                                           uint32_t* __restrict__ list) {
    __shared__ double expected[16], least[16];
    __shared__ uint32_t bins[16];
    __shared__ double share[16];
    const uint32_t lane = threadIdx.x & 63, l = threadIdx.x >> 6;  // wave l = region l
    unsigned long long b[4], sum = 0ull;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        b[k] = hist[l * 256 + 4 * lane + k];
        hist[l * 256 + 4 * lane + k] = 0ull;
        sum += b[k];
    }
    unsigned long long incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long up = (unsigned long long)__shfl_up((long long)incl, d, 64);
        if (lane >= (uint32_t)d) incl += up;
    }
    const unsigned long long total = (unsigned long long)__shfl((long long)incl, 63, 64);
    // the region's elements, by its share of the weight
    if (lane == 0) share[l] = (double)total;
    __syncthreads();
    double all = 0.0;
    for (int i = 0; i < 16; ++i) all += share[i];
    const double samples = all > 0.0 ? sampled * ((double)total / all) : 0.0;
    uint32_t win_lo = 0, win_len = 0;
    double captured = 0.0, median_digits = 0.0;  // elements of the sample inside the window, and in the median's digit
    if (total != 0ull && ((skip_mask >> l) & 1u) == 0u) {  // wave-uniform
        const unsigned long long ballot = __builtin_amdgcn_ballot_w64(2ull * incl >= total);
        const uint32_t L = ballot ? (uint32_t)__builtin_ctzll(ballot) : 63u;
        unsigned long long c = incl - sum;  // weight below this lane's four bins
        uint32_t k_sel = 3;
        unsigned long long below = c, mass = b[3];
        bool found = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!found && 2ull * (c + b[k]) >= total) {
                found = true;
                k_sel = (uint32_t)k;
                below = c;
                mass = b[k];
            }
            c += b[k];
        }
        const uint32_t digit = (uint32_t)__shfl((int)(4 * lane + k_sel), (int)L, 64);
        const double below_d = (double)(unsigned long long)__shfl((long long)below, (int)L, 64);
        const double mass_d = (double)(unsigned long long)__shfl((long long)mass, (int)L, 64);
        const double tot = (double)total;
        const double place = (double)digit + (mass_d > 0.0 ? (0.5 * tot - below_d) / mass_d : 0.5);
        const double six_sigma = 6.0 * 0.75 / sqrt(samples);
        auto digit_of = [&](double weight) {  // the first digit up to and including which there is at least that much
            const unsigned long long reached = __builtin_amdgcn_ballot_w64((double)incl >= weight);
            if (reached == 0ull) return 255;
            unsigned long long below_k = incl - sum;
            int k_at = 3;
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                unsigned long long up_to = below_k;
#pragma unroll
                for (int i = 0; i <= k; ++i) up_to += b[i];
                if ((double)up_to >= weight) k_at = k;
            }
            return __shfl((int)(4 * lane) + k_at, (int)__builtin_ctzll(reached), 64);
        };
        const int from = min(digit_of((0.5 - six_sigma) * tot), (int)floor(place - 0.5));
        const int to = max(digit_of((0.5 + six_sigma) * tot), (int)floor(place + 0.5));
        const int lo_i = max(from, 0), hi_i = min(to, 255);
        win_lo = (uint32_t)lo_i;
        win_len = (uint32_t)(hi_i - lo_i + 1);
        median_digits = mass_d / tot * samples;
        double inside = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (4 * lane + k - win_lo < win_len) inside += (double)b[k];
#pragma unroll
        for (int mk = 32; mk >= 1; mk >>= 1) inside += __shfl_xor(inside, mk, 64);
        captured = inside / tot * samples;
    }
    if (lane == 0) {
        state[l].win_lo = win_lo;
        state[l].win_len = win_len;
        expected[l] = captured;
        least[l] = median_digits;
        bins[l] = win_len + 2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum_captured = 0.0, sum_least = 0.0;
        uint32_t sum_bins = 0;
        for (int i = 0; i < 16; ++i) {
            sum_captured += expected[i];
            sum_least += least[i];
            sum_bins += bins[i];
        }
        const uint32_t declined = sum_captured > 0.06 * sampled || sum_bins > MAE_WINDOW_BINS ? 1u : 0u;
        list[MAE_LIST_UNUSABLE] = list[MAE_DIGITS_MISSING] = list[MAE_DECLINED] = declined;
        list[MAE_NO_LIST_AT_ALL] = sum_least > 0.95 * list_room ? 1u : 0u;
        list[MAE_WINDOW_OUTCOME] = declined ? MAE_LIST_DECLINED : MAE_LIST_SERVED;
    }
}

// After a pass: one wave per region reads its 256 bins, fixes the next digit and clears the bins.  FIRST also takes
// the region's total from the bins.  `wrote` says what the pass before it did to the list.  LAST writes the result record (layout of bof4_mae_stats): [0..15] median,
// [16..31] den, [32..47] cnt (integers), [48] sae, [49] n_used, [50] n_outliers (integers); word 49 is stored last, at
// system scope, so that a host watching it may read the record as soon as it changes.
enum MaeWrote {
    MAE_NO_LIST,
    MAE_AFTER_LIST,     // the second pass of a step that does not sample
    MAE_AFTER_WINDOWS,  // mae_window_kernel
    MAE_AFTER_RERUN,    // the first pass, where mae_window_kernel did not find the first digits
    MAE_AFTER_SECOND    // the second pass after these: it has written the list where that could not be used
};
__global__ __launch_bounds__(1024) void mae_select_kernel(MaeLevelState* __restrict__ state,
                                                          unsigned long long* __restrict__ hist,
                                                          const unsigned long long* __restrict__ cnt_part,
                                                          const double* __restrict__ sae_part, uint32_t n_part,
                                                          uint32_t n_part_scan, uint32_t n_slots,
                                                          int first, int last, uint32_t skip_mask, int wrote,
                                                          const uint32_t* __restrict__ cand_count,
                                                          uint32_t cand_waves, uint32_t cand_cap,
                                                          uint32_t* __restrict__ list,
                                                          double* __restrict__ out, int unweighted) {
    const uint32_t lane = threadIdx.x & 63, l = threadIdx.x >> 6;  // wave l = region l
    // as for the passes: this launch follows one that did nothing
    if (wrote == MAE_AFTER_WINDOWS && list[MAE_DECLINED] != 0u) return;
    if (wrote == MAE_AFTER_RERUN && list[MAE_DIGITS_MISSING] == 0u) return;
    // after the pass that wrote the list: did every wave's stretch hold its entries?  (and, below, if the list was
    // captured by windows: does every region's digit lie inside its window?  If not, the state stays as it is: a first pass
    // over all the weights starts the search again.)
    const bool check_window = wrote == MAE_AFTER_WINDOWS;
    const bool written = wrote == MAE_AFTER_LIST || check_window ||
                         (wrote == MAE_AFTER_SECOND && list[MAE_LIST_UNUSABLE] != 0u && list[MAE_NO_LIST_AT_ALL] == 0u);
    uint32_t stretch_full = 0, missed = 0;
    if (written)
        for (uint32_t i = threadIdx.x; i < cand_waves; i += 1024) stretch_full |= cand_count[i] > cand_cap ? 1u : 0u;
    MaeLevelState s = state[l];
    unsigned long long b[4], sum = 0ull;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        b[k] = hist[l * 256 + 4 * lane + k];
        hist[l * 256 + 4 * lane + k] = 0ull;
        sum += b[k];
    }
    unsigned long long incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long up = (unsigned long long)__shfl_up((long long)incl, d, 64);
        if (lane >= (uint32_t)d) incl += up;
    }
    if (first) s.total = (unsigned long long)__shfl((long long)incl, 63, 64);
    const bool skipped = ((skip_mask >> l) & 1u) != 0u;  // only the region's mass was wanted: no search
    if (skipped) s.pad = 1u;
    if (!skipped && s.hi != 0u && s.total != 0ull) {  // wave-uniform
        const uint32_t lo = s.hi > 8 ? s.hi - 8 : 0;
        // smallest digit d with 2 (base + weight of digits <= d) >= total; totals stay below 2^62 (checked below)
        const bool reached = 2ull * (s.base + incl) >= s.total;
        const unsigned long long ballot = __builtin_amdgcn_ballot_w64(reached);
        // the bins of this pass hold all the weight between base and the end of the prefix's range, and the prefix
        // was chosen because the total is reached inside it: some lane has reached it
        const uint32_t L = ballot ? (uint32_t)__builtin_ctzll(ballot) : 63u;
        unsigned long long c = s.base + incl - sum;  // weight below this lane's four bins
        uint32_t k_sel = 3;
        unsigned long long below = 0ull;
        bool found = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!found && 2ull * (c + b[k]) >= s.total) {
                found = true;
                k_sel = (uint32_t)k;
                below = c;
            }
            c += b[k];
        }
        if (!found) below = c - b[3];
        const uint32_t digit = (uint32_t)__shfl((int)(4 * lane + k_sel), (int)L, 64);
        const unsigned long long nb = (unsigned long long)__shfl((long long)below, (int)L, 64);
        s.prefix = (s.prefix << (s.hi - lo)) | digit;
        s.base = nb;
        s.hi = lo;
        if (check_window && !((digit - s.win_lo) < s.win_len)) missed = 1u;
    }
    if (written) {  // uniform
        const uint32_t any_full = (uint32_t)__syncthreads_or((int)stretch_full);
        if (check_window) missed = (uint32_t)__syncthreads_or((int)missed);
        if (threadIdx.x == 0) {
            list[MAE_LIST_UNUSABLE] = any_full != 0u || missed != 0u ? 1u : 0u;
            if (check_window) {
                list[MAE_DIGITS_MISSING] = missed != 0u ? 1u : 0u;
                list[MAE_WINDOW_OUTCOME] = missed != 0u ? MAE_WINDOW_MISSED : any_full != 0u ? MAE_STRETCH_FULL : MAE_LIST_SERVED;
            }
        }
    }
    if (lane == 0 && !(check_window && missed != 0u)) state[l] = s;
    if (!last) return;
    __shared__ double med[16], den[16];
    __shared__ unsigned long long cnt[17];
    // the records of mae_window_kernel, or of mae_pass_kernel where that did not run
    const uint32_t n_rec = (n_part_scan != 0u && list[MAE_DECLINED] != 0u) ? n_part_scan : n_part;
    unsigned long long k_l = 0ull, k_out = 0ull;
    for (uint32_t i0 = lane; i0 < n_rec; i0 += 64 * 4) {  // four independent loads in flight (integers: any order)
        unsigned long long a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = i0 + 64 * u;
            a[u] = i < n_rec ? cnt_part[l * MAE_MAX_WGS + i] : 0ull;
            b[u] = (l == 15 && i < n_rec) ? cnt_part[16 * MAE_MAX_WGS + i] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            k_l += a[u];
            k_out += b[u];
        }
    }
#pragma unroll
    for (int mk = 32; mk >= 1; mk >>= 1) {
        k_l += (unsigned long long)__shfl_xor((long long)k_l, mk, 64);
        k_out += (unsigned long long)__shfl_xor((long long)k_out, mk, 64);
    }
    if (lane == 0) {
        med[l] = (s.total != 0ull && s.hi == 0u && s.pad == 0u) ? (double)key_to_float(s.klo + s.prefix)
                                                                  : __builtin_nan("");
        den[l] = (double)s.total * (unweighted ? 1.0 : 0x1p-24);  // correctly rounded conversion of the integer
        cnt[l] = k_l;
        if (l == 15) cnt[16] = k_out;
    }
    // the slots' sums in a fixed order: thread i adds its run of them, a butterfly the lanes of a wave, thread 0 the waves
    __shared__ double part_sum[16][2];
    {
        const uint32_t per = (n_slots + 1023) / 1024;
        double s0 = 0.0, s1 = 0.0;
        for (uint32_t p = per * threadIdx.x; p < min(per * (threadIdx.x + 1), n_slots); ++p) {
            s0 += sae_part[2 * p];
            s1 += sae_part[2 * p + 1];
        }
#pragma unroll
        for (int mk = 32; mk >= 1; mk >>= 1) {
            s0 += __shfl_xor(s0, mk, 64);
            s1 += __shfl_xor(s1, mk, 64);
        }
        if (lane == 0) {
            part_sum[l][0] = s0;
            part_sum[l][1] = s1;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sae = 0.0, w_est = 0.0;
        for (int i = 0; i < 16; ++i) {
            sae += part_sum[i][0];
            w_est += part_sum[i][1];
        }
        unsigned long long used = 0ull;
        const bool too_large = !(w_est < 0x1p38);  // 64-bit weight sums need sum |constant| < 2^39 (NaN counts too)
        for (int q = 0; q < 16; ++q) {
            out[q] = too_large ? __builtin_nan("") : med[q];
            out[16 + q] = den[q];
            out[32 + q] = __longlong_as_double((long long)cnt[q]);
            used += cnt[q];
        }
        out[48] = too_large ? __builtin_nan("") : sae;
        out[50] = __longlong_as_double((long long)cnt[16]);
        __hip_atomic_store(reinterpret_cast<unsigned long long*>(&out[49]), used, __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace bof4
