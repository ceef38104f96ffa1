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
// A wave takes its candidates 192 at a time, and where there are many its chain is the longer one.  By the number of clusters within the error
// bound that a sample of the centroids finds at upload (rank_crowd), waves' time over workgroups', mean (least ... most), 32 to 512 components,
// 300 to 4,000 clusters, offsets of 0 to 1,000:
//   sampled number             below 40          80 to 120         120 to 160        160 to 192        224 to 256        400 to 600
//   1,600 queries, 10 probes   0.92 (0.75 1.02)  0.98 (0.97 1.00)  1.07 (0.95 1.21)  1.26 (1.16 1.36)                    1.03 (0.95 1.13)
//                  64                            0.96 (0.85 1.07)  1.06 (0.94 1.26)  1.14 (0.89 1.46)  1.33 (1.03 1.71)  1.59 (1.24 2.36)
//   3,000          10          0.90 (0.75 1.01)  0.99 (0.96 1.00)  0.99 (0.88 1.09)  1.13 (1.05 1.21)                    0.99 (0.97 1.02)
//                  64                            0.88 (0.74 0.99)  0.94 (0.81 1.12)  1.05 (0.90 1.33)  1.25 (1.01 1.56)  1.43 (1.19 2.09)
//   10,000         10          0.79 (0.57 1.00)  0.97 (0.95 0.99)  0.77 (0.68 0.89)  0.86 (0.78 0.93)                    1.00 (0.97 1.04)
//                  64                            0.72 (0.67 0.83)  0.81 (0.69 0.98)  0.83 (0.73 0.97)  0.99 (0.75 1.16)  1.10 (0.94 1.45)
constexpr int kWaveProbes = 64;
inline bool select_by_waves(int nq, int n_probes, double crowd) {
    return nq > 6 * 256 && n_probes <= kWaveProbes && crowd <= (nq < 5000 ? 120.0 : 192.0);
}

// The error bound of a ranking value over |q|^2 + max |c|^2 (rank_error_bound).
constexpr float rank_error_share(int d) { return (float)(3 * d + 8) * 2.3841858e-07f + 5.0e-05f; }

}  // namespace ivfpq
