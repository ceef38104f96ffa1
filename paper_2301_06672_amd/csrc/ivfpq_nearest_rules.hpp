// How the nearest probes of a large batch are scanned and bounded, by sizes alone.  Plain C++, so that a test can ask the same rules.
#pragma once

namespace ivfpq {

// bound_wave_kernel: the largest k that it takes, the minima whose k-th is the first bound, and the room for the values that are not above that.
// Their expected number is S * ln(S / (S - k)) for S = kBoundShares minima of a long list, with a deviation of about sqrt(k): 127 at k = 100
// (the room is never short), 177 at 128, where 0.4 / 1.3 / 4 % of the lists of 2,000 / 4,000 / 20,000 values have more than 192.  Such a query keeps the
// first bound and lists up to half as many values again.  Room for 256 (a fourth register of every lane in each of the bisection's 31 steps) was
// measured: 10,000 queries, lists of 1,000 to 2,000, k of 100 to 128 one to two us slower, lists of 8,000 and k of 120 to 128 one to nine faster of 600.
constexpr int kBoundWaveK = 128, kBoundShares = 256, kBoundCand = 192;

// Whether a batch's nearest probes are scanned by the group kernel, up to four queries of a cluster a workgroup, and bounded by a wave each, instead
// of a workgroup a query that does both.  The order (5 us), the bound (10 to 30) and two launches have to be won back by tables that are built
// and codes that are fetched once for several queries, and the fewer workgroups have to fill the chip.  Gain (-) or loss (+) of the nearest probes,
// us, beside what a workgroup a query takes (lists of equal length, 20 probes, k = 10):
//   number x length of lists               1,000 x 500               1,000 x 1,000             500 x 2,000               2,000 x 2,000             100 x 8,000
//   queries                                4,500   10,000   16,000   4,500   6,500   10,000    3,000   4,500   10,000    4,500   6,500   10,000    3,000     10,000
//   eight waves a workgroup
//     64 codes, e5m3                       51 +8   98  0    147 -5   71 +3   96 -1   138 -10   78 -2   127 -31 241 -69   140 -16 187 -30 269 -69   229 -43   764 -260
//     64 codes, half                       64 +1   126 -11  189 -19  85 -1   115 -7  167 -20   91 -5   129 -18 269 -76   131  0  182 -16 269 -45   268 -46   820 -248
//   four waves, tables of 24 KB and more
//     32 codes, e5m3                       50 +5   96 -13   146 -31  61 +4   81 -4   114 -18   59 +1   90 -13  158 -42   92 +1   116 -8  170 -23   145 -7    434 -94
//     48 codes, e5m3                       43 +7   78 +4    115 -3   58 +4   76 +2   109 -6    63 +2   98 -12  184 -44   100 -9  137 -22 200 -42   180 -10   588 -146
//     64 codes of 7 bits, e5m3             45 +8   86 -5    129 -18  64 +6   87 -3   126 -15   72 -4   109 -10 202 -41   115 -5  150 -12 221 -41   214 -21   659 -152
//     64 codes of 7 bits, half             47 +8   91  0    137 -8   68 +7   92 +1   135 -5    77 +9   145 -32 281 -86   149 -22 200 -43 299 -90   233 +17   904 -299
//   smaller tables: the codes alone bound the scan, of which a workgroup a query has more under way
//     64 codes of 4 bits, half             32 +8   59  0    87 -11   47 +7   62 -1   89 -13    54 +25  78 +8   142 -18   78 +30  102 +15 148 +2    162 +47   493 -69
//     64 codes of 4 bits, float            31 +8   58  0    86 -10   46 +6   61 -1   88 -15    51 +24  73 +1   135 -22   75 +26  96 +16  143 +10   152 +36   515 -76
//     64 codes of 4 bits, e5m3             33 +12  61 +6    91 +2    50 +12  66 +7   95  0     58 +33  86 +22  157 +12   87 +40  110 +30 161 +27   181 +86   551 +18
//     64 codes of 6 bits, half             40 +9   75 +6    111 +2   59 +9   80 +5   115 -1    68 +27  103 +33 189 -2    104 +33 138 +33 196 +2    208 +101  660 +16
//     16 codes, e5m3                       35 +4   63 -4    93 -14   42 +4   56 -2   79 -12    40 +14  57 +2   98 -6    59 +13  72 +11  102 +1    91 +30    267  0
//     32 codes of 4 bits, float            27 +26  49 +33   74 +42   36 +32  48 +35  69 +41    38 +39  52 +44  91 +74    53 +49  65 +61  94 +103   98 +117   295 +282
//     32 codes of 7 bits, half             33 +8   61 +6    90  0    44 +7   59 +4   84 -5     47 +15  67 +17  122 -3    69 +16  87 +13  128 +10   132 +43   397 +44
// Hence a number of queries by the table, and 2,000 and more times the lists' number over their length (queries of many short lists share
// none; lists of uneven length count by sum of len^2 / n, as queries that are like the vectors meet them).  Lists that are much
// longer than the others keep one workgroup, and then one wave, at work after all others have ended: among 1,024 of which the others have
// 1,000, one of 32,000 / 64,000 / 134,000: us a search of 6,500 (10,000) queries, spread like the vectors; evenly over the lists
//     64 codes, e5m3, eight waves          410 -35 (456 -68), 319 -11 (388 -11) / 726 +7 (885 -26), 468 +65 (517 +55) / 1,738 -108 (2,028 -274), 773 +195 (867 +157)
//     64 codes of 7 bits, e5m3, four       382 +40 (481 +49), 317 +95 (400 +52) / 803 -62 (934 +5), 522 +183 (576 +164) / 1,898 -367 (2,143 -51), 955 +414 (1,034 +357)
// and of lengths that are log-normal, the longest 13.7 times the mean, 64 codes of 7 bits 303 +41 (418 +2): 200 queries more for every mean
// length above eight that the longest list has, 380 with four waves.
struct NearestSizes {
    long long nq;
    int k;
    long long n;                   // vectors of the index
    double mean, typical;          // length of a list that is not empty; of the list that a vector lies in
    double longest;
    int bits, pq_dim, elem_bytes;  // elem_bytes: of a table's entry
    int pairs;                     // queries of a workgroup of the group kernel, 0: it does not apply
    bool eight_waves;              // its workgroups have eight waves, of which two share a compute unit
};
// queries that one launch orders: sixteen of a thread (a search of more, or a tile of more, takes a workgroup a query)
constexpr int kNearestPerThread = 16, kNearestThreads = 1024;
inline bool nearest_by_groups(const NearestSizes& s) {
    if (s.pairs == 0 || s.k > kBoundWaveK || s.nq > kNearestPerThread * kNearestThreads || s.n <= 0) return false;
    const bool whole = s.bits == 8 || s.bits == 4;
    const int table = (s.pq_dim << s.bits) * s.pairs * s.elem_bytes;
    double from = 9000, short_lists = 2000;
    if (s.bits == 4 && s.elem_bytes == 1) return false;                                      // never faster by a twelfth
    else if (s.eight_waves) { from = 2500; if (s.elem_bytes == 1) short_lists = 4000; }
    else if (table >= 24 * 1024) { from = 3500; if (!whole && s.elem_bytes == 1) { from = 3000; short_lists = 6500; } }
    else if (s.pq_dim == 32 && s.elem_bytes == (whole ? 4 : 2)) return false;               // never faster by an eighth
    else if (s.pq_dim > 32 && (s.elem_bytes == 4 || (s.bits == 4 && s.elem_bytes == 2))) from = 5000;
    const double over = s.longest / s.mean - 8.0;
    return (double)s.nq >= from + short_lists * (double)s.n / (s.typical * s.typical) + (over > 0.0 ? (s.eight_waves ? 200.0 : 380.0) * over : 0.0);
}

}  // namespace ivfpq
