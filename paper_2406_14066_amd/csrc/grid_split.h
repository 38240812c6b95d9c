// How the rows of a launch that holds both halves are mixed (host only; a row is 8 consecutive
// blocks, one per XCD, of one role).
#pragma once

// The attention rows among which the rejection rows are spread evenly; the other attention rows
// follow (the rejection stages of a request wait for each other, so the last rejection item sits
// well before the end of the grid: the tail of the launch is attention only).
//
// Spread evenly, every `period`-th row is an attention row.  The hardware deals an XCD's blocks to its 32
// compute units in turn, so with a period near 2, 4, 6 or 8 the attention blocks always fall on the same
// compute units, and the others are left to the rejection's short ones.  64/8 heads, V = 32000, k = 4, 96
// requests of 300 to 1700 tokens, by period: 93.2 us at 4.3, 93.4 at 4.2, 122.4 at 4.04, 130.5 at
// 3.98, 97.4 at 3.86, 92.2 at 3.75; k = 7, 96 requests: 103 at 4.16, 156 at 4.03, 106 at 5.95, 98 at 5.74;
// k = 2, 128 requests: 78.8 at 2.1, 90.7 at 2.0; odd and fractional periods do no harm.  So a period within a
// twentieth of one of them becomes the one a twentieth above (fewer attention rows among the rejection's), or 3.7 instead
// of 3.7 to 4.2 where there are enough attention rows (V = 8192, k = 4, 96 requests: 83 us at 3.4, 84 at 3.7, 89 at 4.2).
inline int attention_rows_mixed(int rows_attn, int rows_reject, double span)
{
    int rows = (int)(rows_attn * span);
    if (rows < 1) rows = 1;
    if (rows > rows_attn) rows = rows_attn;
    const double period = 1.0 + (double)rows_reject / rows;
    const int even = 2 * (int)(period / 2.0 + 0.5);
    if (even >= 2 && even <= 8 && period > (even == 4 ? 3.7 : 0.95 * even) && period < 1.05 * even) {
        const int more = (int)(rows_reject / 2.7) + 1;
        if (even == 4 && more <= rows_attn) return more;
        rows = (int)(rows_reject / (1.05 * even - 1.0));
        if (rows < 1) rows = 1;
    }
    return rows;
}
