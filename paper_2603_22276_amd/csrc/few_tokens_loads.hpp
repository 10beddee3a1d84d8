// Which bytes the global -> LDS loads of the few-token kernel fetch.  Plain C++ without HIP, so that a host program can hold
// every load against the extent of its tensor.
#pragma once

#include <stdint.h>

namespace dora {

// A ring slot holds STEP_K k of MR blocks of 16 weight rows, then of TB blocks of 16 token rows.  A load of a slot brings 16
// bytes (eight k) per lane, LOAD_ROWS rows for the whole wave.
//
// The K advance travels in the scalar offset of the load and everything else in the vector offset, because the range check
// of a raw buffer load is specified for the vector offset alone: a row past the end has to be pushed out of range there.
template <int TB, int MR>
struct FewTokensLoads {
    static constexpr int STEP_K = 64;
    static constexpr int ROWS = MR * 16, TOK = TB * 16;
    static constexpr int LANES_PER_ROW = STEP_K / 8, LOAD_ROWS = 64 / LANES_PER_ROW;
    static constexpr int COUNT = (ROWS + TOK) / LOAD_ROWS;      // loads of a slot
    static constexpr uint32_t OUTSIDE = 0xFFFFFFFFu;            // beyond every descriptor: loads zeros

    static constexpr bool weights(int load) { return load < ROWS / LOAD_ROWS; }
    // row, inside its operand's part of the slot, that a lane of a load brings in
    static constexpr int row(int load, int lane)
    {
        return (weights(load) ? load : load - ROWS / LOAD_ROWS) * LOAD_ROWS + lane / LANES_PER_ROW;
    }
    // bytes from the operand's first row to k of that row; `rows` of its rows exist, K elements each.  For a row that
    // exists this fits 32 bits unsigned (no tensor has 2^31 elements); for the others the product may wrap and is not used.
    static constexpr uint32_t vector_offset(int row, int rows, int k, int K)
    {
        return row < rows ? ((uint32_t)row * (uint32_t)K + (uint32_t)k) * 2u : OUTSIDE;
    }
    // the same for the step that starts at k0, its k past the end masked
    static constexpr uint32_t step_offset(uint32_t offset, int k, int k0, int K) { return k0 + k < K ? offset : OUTSIDE; }
    static constexpr uint32_t scalar_offset(int k0) { return (uint32_t)k0 * 2u; }
};

}  // namespace dora
