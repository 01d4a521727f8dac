// Paley's Hadamard matrices of order 12, 20 and 28, at compile time.
#pragma once

namespace qvggt {

// Sizes whose bf16 activation rows are quantized in rotate_quant_paley.hip
constexpr bool paley_size(int K) { return K == 768 || K == 1536 || K == 3072 || K == 6144 || K == 2560 || K == 5120 || K == 8192; }

namespace gen {

// entry (r, c) in {+1, -1}, from the squares of GF(q) found by enumeration
template <int Q>
constexpr bool is_square_mod(int x)
{
    x %= Q;
    if (x < 0) x += Q;
    for (int k = 1; k < Q; ++k)
        if ((k * k) % Q == x) return true;
    return false;
}

template <int MM>
constexpr int paley_entry(int r, int c)
{
    static_assert(MM == 12 || MM == 20 || MM == 28, "Paley matrices of order 12, 20 and 28");
    if constexpr (MM == 28) {
        // type II, q = 13: symmetric conference matrix of order 14 blown up by 2 x 2 blocks
        const int i = r / 2, j = c / 2, u = r % 2, v = c % 2;
        if (i == j) return (u == 0 && v == 0) ? 1 : -1;                       // the zero diagonal becomes [[1, -1], [-1, -1]]
        const int cc = (i == 0 || j == 0) ? 1 : (is_square_mod<13>(i - j) ? 1 : -1);
        return (u == 1 && v == 1) ? -cc : cc;                                 // +-1 becomes +-[[1, 1], [1, -1]]
    } else {
        // type I, q = MM - 1: identity plus the skew matrix bordered by +1 (first row) and -1 (first column)
        if (r == c) return 1;
        if (r == 0) return 1;
        if (c == 0) return -1;
        return is_square_mod<MM - 1>(r - c) ? 1 : -1;
    }
}

}  // namespace gen
}  // namespace qvggt
