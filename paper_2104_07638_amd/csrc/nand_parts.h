// nand_parts.h -- NAND minors of kNandRowMin blocks and more: what the three launches of a call
// tell each other about the parts of a matrix.
//
// A part is one choice for each of the last L = N - 6 blocks (levels 0 .. L - 1 of the tree): a
// node of order 12 with its 729 minors, contiguous in the output.  A word and a code per part:
//   * nand_row.h forms every part without pivot shifts and says in the word whether a shift is
//     due: kPartRedo, with the first of the L levels whose pivot is shifted (L: none of these,
//     but one inside the part).  Up to that level every part below the shifted node has made
//     the same test on the same numbers; behind it a shifted tree has other numbers.  It
//     counts and lists the parts so marked.
//   * nand_part_kernel (xor.hip) forms the marked parts again, with the shifts the word asks for
//     and, behind the first, those of its own tests (which the parts below one node agree on,
//     all of them being formed there), and leaves the codes of the shifts in the L levels, the
//     number of shifts and the scale of the matrix.
//   * nand_fix_kernel (xor.hip) applies the corrections of those levels, whose nodes span several
//     parts, deepest first, and completes info.
// So a shift costs the parts below its node and not the whole matrix, and they are spread over
// wavefronts; a call without shifts ends the last two launches after one load.
#pragma once
#include <stdint.h>

namespace apm {

// 7 is the fewest blocks with a level above a part; with fewer the LDS kernel of xor.hip is
// launch-bound or nearly so (1000 complex matrices of 6 blocks 26 us).
constexpr int kNandRowMin = 7;

constexpr int nand_levels(int N) { return N - 6; }

// The word of a part.  nand_row.h: first | kPartRedo | kPartBad.  After nand_part_kernel also
// the shifts made (those in the L levels counted in the first part below) and the exponent of
// the matrix's largest magnitude.
constexpr uint32_t kPartFirst = 7u;        // first shifted level, or L
constexpr uint32_t kPartRedo = 8u;         // formed again with shifts
constexpr uint32_t kPartBad = 16u;         // a non-finite minor (finite input)
constexpr int kPartShifts = 8;             // 12 bits: at most 1 + 2 (1 + 3 + 9 + 27 + 81)
constexpr int kPartScale = 20;             // 12 bits
constexpr int kPartScaleBias = 2048;
static_assert(nand_levels(13) <= (int)kPartFirst, "the level fits");

// The head: the lengths of the lists (wavefront i of the register kernel appends to list i mod
// subs: an atomic takes 12 ns on one address, 50 us for the 4000 wavefronts of 16000 shifted
// matrices) and its count of parts with a non-finite minor, both cleared by the last launch; and
// what the second launch passes on to the last: the counts, and the levels inside its groups.
constexpr int kSubLists = 64, kHeadStride = 32;
constexpr int kHeadBad = kSubLists * kHeadStride, kHeadRedo2 = kHeadBad + 1, kHeadBad2 = kHeadBad + 2, kHeadGroup = kHeadBad + 3;
constexpr int kRowParts = 12;              // parts of a wavefront of the register kernel

// Wavefronts of the register kernel: one for four units (3^(N - 8) a matrix above 8 blocks) and,
// from 8 blocks on, one of the three choices of the block below them.
constexpr int64_t nand_row_waves(int N, int64_t batch)
{
    int64_t units = batch;
    for (int k = 8; k < N; ++k) units *= 3;
    return (units + 3) / 4 * (N >= 8 ? 3 : 1);
}

}  // namespace apm
