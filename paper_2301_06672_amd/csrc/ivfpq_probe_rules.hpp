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

// Whether the selection from stored ranking values takes a wave per query (select_probes_wave_kernel) instead of a workgroup: from the batch on
// whose workgroups the chip does not hold at once.  The workgroup kernel's 25,648 bytes of LDS leave room for six in a compute unit, 1,536 in
// all.  Ranking and selection, us, workgroups / waves, n_probes 10, 64 (centred vectors of 128 components where no other number stands):
//   1,024 clusters    513 queries 18.0 / 17.0, 19.8 / 23.8; 1,200 21.5 / 19.8, 29.0 / 29.1; 1,536 22.5 / 20.8, 29.9 / 30.4;
//                     1,600 27.3 / 20.7, 37.5 / 30.4; 3,000 35.7 / 27.8, 45.5 / 39.8; 10,000 89.7 / 57.9, 111.8 / 81.3
//   2,000 clusters    64 probes: 513 24.2 / 27.6, 1,536 38.1 / 37.8, 1,600 44.0 / 39.7, 3,000 58.0 / 50.4, 10,000 139.3 / 95.0
//   512 components    1,024 clusters: 1,536 43.2 / 42.6, 62.1 / 65.6; 1,600 53.5 / 42.9, 70.0 / 66.4; 2,100 62.9 / 52.5, 86.7 / 85.0
//   960 components    513 52.9 / 54.7, 73.2 / 98.5; 1,600 85.1 / 72.8, 120.2 / 118.5; 2,100 102.2 / 91.3, 146.0 / 158.4; 3,000 107.1 / 94.9, 168.9 / 162.2
//   offset by 400     1,536 23.8 / 25.2, 37.1 / 48.9; 1,600 29.0 / 25.2, 46.0 / 49.0; 2,100 33.0 / 29.5, 54.9 / 52.8
//   offset by 2,000   (every cluster is a candidate) 1,536 78.1 / 107.5, 78.7 / 133.2; 3,000 136 / 144, 139 / 160; 10,000 397 / 405, 400 / 423
constexpr int kWaveProbes = 64;
inline bool select_by_waves(int nq, int n_probes) { return nq > 6 * 256 && n_probes <= kWaveProbes; }

}  // namespace ivfpq
