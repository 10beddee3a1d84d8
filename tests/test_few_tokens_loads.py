"""The global -> LDS loads of the few-token kernel, held on the host against the extents of x and of W: its offset arithmetic
is plain C++, compiled here into a program that walks every lane of every load.

A raw buffer load checks its vector offset against the descriptor and adds the scalar offset unchecked, so that is what
the program does: a load whose vector offset lies in range reads 16 bytes at vector + scalar offset, which must lie inside
the tensor and hold the row and k that the slot wants there; any other load reads nothing, and must not be wanted."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <utility>
#include "few_tokens_loads.hpp"

using namespace dora;

static long loads = 0;

// one operand of `rows` rows (of which a group sees at most `part`), K elements each, walked step by step
template <class L>
void walk(const char* what, bool weights, int rows, int part, int K, bool first_and_last_step_only)
{
    const int64_t bytes = (int64_t)rows * K * 2;               // extent of the descriptor
    const int steps = (K + L::STEP_K - 1) / L::STEP_K;
    for (int s = 0; s <= steps; ++s) {                         // the last one lies past the end
        if (first_and_last_step_only && s > 0 && s < steps - 1) continue;
        const int k0 = s * L::STEP_K;
        std::set<std::pair<int, int>> seen;
        for (int i = 0; i < L::COUNT; ++i) {
            if (L::weights(i) != weights) continue;
            for (int lane = 0; lane < 64; ++lane)
                for (int k = 0; k < L::STEP_K; k += 8) {       // whichever chunk of the row the swizzle gives the lane
                    const int row = L::row(i, lane);
                    if (row < 0 || row >= part) { printf("%s: row %d outside the slot\n", what, row); exit(1); }
                    const uint32_t v = L::step_offset(L::vector_offset(row, rows, k, K), k, k0, K);
                    ++loads;
                    if ((int64_t)v >= bytes) continue;         // out of the descriptor's range: zeros
                    const int64_t at = (int64_t)v + L::scalar_offset(k0);
                    if (at + 16 > bytes || at != ((int64_t)row * K + k0 + k) * 2 || row >= rows || k0 + k >= K) {
                        printf("%s: rows %d K %d: load %d lane %d k0 %d reads bytes %lld..+16 of %lld\n", what, rows, K, i, lane, k0,
                               (long long)at, (long long)bytes);
                        exit(1);
                    }
                    seen.insert({row, k});
                }
        }
        const int wanted = k0 < K ? (K - k0 < L::STEP_K ? K - k0 : L::STEP_K) / 8 : 0;
        if ((int)seen.size() != rows * wanted) { printf("%s: rows %d K %d k0 %d: %zu chunks\n", what, rows, K, k0, seen.size()); exit(1); }
    }
}

template <int TB, int MR>
void variant()
{
    typedef FewTokensLoads<TB, MR> L;
    static_assert(L::COUNT * 1024 == (L::ROWS + L::TOK) * L::STEP_K * 2, "a slot is filled exactly");
    const int ks[] = {8, 56, 64, 72, 200};
    for (int K : ks) {
        for (int T = 1; T <= L::TOK; ++T) walk<L>("x", false, T, L::TOK, K, false);
        for (int N = 8; N <= 16 * L::ROWS; N += 8)             // d_out of 8200 ends like 8 of these, and so on
            walk<L>("W", true, N % L::ROWS ? N % L::ROWS : L::ROWS, L::ROWS, K, false);
    }
    // the largest tensors: below 2^31 elements
    for (int T : {1, 2, 15, 16, 17, 33, 48, 49, 63, 64})
        if (T <= L::TOK) walk<L>("x", false, T, L::TOK, (int)(((((int64_t)1 << 31) - 1) / T < (1 << 28) - 8 ? (((int64_t)1 << 31) - 1) / T : (1 << 28) - 8) / 8 * 8), true);
    for (int rows : {8, 16, 24, 56, 64})
        if (rows <= L::ROWS) walk<L>("W", true, rows, L::ROWS, (int)((((int64_t)1 << 31) - 1) / rows / 8 * 8), true);
}

int main()
{
    variant<1, 1>(); variant<2, 1>(); variant<4, 1>(); variant<4, 2>(); variant<1, 4>(); variant<2, 4>(); variant<4, 4>();
    printf("%ld\n", loads);
    return 0;
}
"""


def test_every_load_lies_inside_its_tensor(tmp_path):
    source, program = tmp_path / "loads.cpp", tmp_path / "loads"
    source.write_text(PROGRAM)
    include = os.path.join(ROOT, "paper_2603_22276_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", include, "-o", str(program), str(source)])
    proc = subprocess.run([str(program)], stdout=subprocess.PIPE, text=True)
    assert proc.returncode == 0, proc.stdout
    assert int(proc.stdout) > 10 ** 6
