// Where the lanes of predict_split find the key rows of their ranges.  Constant expressions only, so that the host can count them
// out for every length (tests/test_key_rows_host.py): no request may depend on what lies behind K~.
#pragma once

namespace dsa {

// A lane range is Lr keys, four ranges to a wavefront.  Matrix row c = lane % 16 of a row operand is key c % 4 of a tile of range
// 4 wv + c / 4, and R tiles (keys 4 apart) lie side by side in it, 64 / R columns each; lane / 16 is the 16-byte column.
constexpr unsigned key_row_offset(int wv, int lane, int Lr, int k, int R)
{
    const int c = lane & 15, g = lane >> 4, sub = R == 4 ? g : R == 2 ? g >> 1 : 0;
    return (unsigned)((4 * wv + (c >> 2)) * Lr + 4 * sub + (c & 3)) * (unsigned)k;
}
// Byte of that row that step s of the contraction takes, or -1 where the row has ended.
constexpr int key_piece_offset(int lane, int k, int R, int s)
{
    const int g = lane >> 4, part = R == 4 ? 0 : R == 2 ? g & 1 : g, byte = 64 * s + 16 * part;
    return byte < k ? byte : -1;
}
// Row operands of one batch of requests, of the `all` that hold 8 tiles; one batch is on its way while another is used.  Groups of rows
// need a second unit operand and the sums of two matrix instructions: with four, 6 to 33 of their registers went through scratch.
// Groups of 8, four and two: k = 32, N = 32, L = 8192, keep = 82 102.4 and 99.8 us, k = 64, N = 4, L = 12288, keep = 246 60.0 and 57.5.
// Two tiles of groups use what they fetch twice and want the four: k = 64, N = 16, L = 8192, keep = 82 66.2 and 71.8.  (k = 16 has
// two in all: one at a time 95.1 and 96.2, N = 32, L = 8192.  k = 48 has the registers for four, and with few wavefronts two are waited
// for: N = 14, L = 1976, keep = 66, groups of 4, 18.8 and 21.0.)
constexpr int key_batch_slots(int all, int steps, bool fewer) { return steps == 2 || fewer || all < 4 ? 2 : 4; }
// Bytes from row operand to row operand, and from the head to batch b of them (beyond the range: to its last batch).
constexpr int key_slot_step(int k, int R) { return 4 * R * k; }
constexpr int key_batch_offset(int b, int batches, int slots, int step) { return (b < batches ? b : batches - 1) * slots * step; }
// Bytes that K~ of the head still has there: the length of the descriptor that batch's loads go through.  Base and length carry the
// batch because the scalar offset of a buffer load does not: whether its range check counts it differs between descriptions, and
// where it does, it is taken off the length, which fails as soon as it is the larger (28 k bytes are, for L < 28).
constexpr int key_bytes_left(int L, int k, int offset) { return offset < L * k ? L * k - offset : 0; }

}  // namespace dsa
