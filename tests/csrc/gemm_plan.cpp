// paper_2505_06653_amd/csrc/bof4_gemm_plan.h for tests on the CPU: compiled and called by tests/test_host_gemm_plan.py.
#include "bof4_gemm_plan.h"

using namespace bof4;

struct Plan {
    uint32_t way, wide_split, decoded_split, decoded_slab_tiles, kernel_split, carry, flush, decoded_carry, decoded_flush, x_in_place;
    uint64_t need;  // workspace without which the call takes another way
};

extern "C" void plan(uint64_t rows, uint64_t cols, uint32_t n_tokens, int list, uint64_t ws_bytes, Plan* out) {
    const GemmPlan P = gemm_plan(rows, cols, n_tokens, list != 0, (size_t)ws_bytes);
    *out = {(uint32_t)P.way, P.wide.split, P.decoded.split, P.decoded.slab_tiles, gemm_split(rows, cols, n_tokens),
            P.chains.wide_carry ? 1u : 0u, P.chains.wide_flush, P.decoded.carry ? 1u : 0u, P.decoded.flush, P.x_in_place ? 1u : 0u, P.ws.total};
    if (P.way == GEMM_WIDE) out->need = P.ws.wide_part + (uint64_t)(P.wide.split - 1) * n_tokens * rows * 4;
    if (P.way == GEMM_DECODED) out->need = P.ws.decoded(P.decoded.split, n_tokens, rows) + P.decoded.slab_bytes;
}
extern "C" uint64_t workspace_bytes(uint64_t rows, uint64_t cols, uint32_t n_tokens) { return gemm_ws_bytes(rows, cols, n_tokens); }
