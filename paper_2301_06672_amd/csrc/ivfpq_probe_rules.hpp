// Which kernels rank clusters, by sizes alone.  Plain C++, so that a test can ask the same rules.
#pragma once

namespace ivfpq {

// Tile choice of the ranking product: 128 x 128 tiles on the bf16 kernel when they cover the chip four times (256 compute units), else 64 x 64 in
// fp32: the products of the operands as they are.  The bf16 halves carry 16 of an operand's 24 bits, which nobody has asked for; below that
// line they stay out, though the selection as a whole would take less from about 512 tiles on (us, fp32 / bf16, 1,024 clusters of 128
// components, 10 probes: 504 tiles 47 / 43, 704 60 / 51, 1,000 79 / 62).
inline bool coarse_big_tiles(int nq, int n_lists) {
    return (long)((n_lists + 127) / 128) * ((nq + 127) / 128) >= 1024;
}
inline int coarse_strip_width(int nq, int n_lists) { return coarse_big_tiles(nq, n_lists) ? 64 : 32; }
// whether a selection of the k smallest per row should work from strip summaries instead of all keys
inline bool coarse_use_strips(int nq, int n_lists, int k) {
    const int w = coarse_strip_width(nq, n_lists);
    return n_lists > 1024 && (n_lists + w - 1) / w >= 2 * k;
}

}  // namespace ivfpq
