// How the nearest probes of a large batch are scanned and bounded, by sizes alone.  Plain C++, so that a test can ask the same rules.
#pragma once

namespace ivfpq {

// bound_wave_kernel: the largest k that it takes, the minima whose k-th is the first bound, and the room for the values that are not above that.
// Their expected number is S * ln(S / (S - k)) for S = kBoundShares minima of a long list, with a deviation of about sqrt(k): 127 at k = 100
// (the room is never short), 177 at 128, where 0.4 / 1.3 / 4 % of the lists of 2,000 / 4,000 / 20,000 values have more than 192.  Such a query keeps the
// first bound and lists up to half as many values again.  Room for 256 (a fourth register of every lane in each of the bisection's 31 steps) was
// measured: 10,000 queries, lists of 1,000 to 2,000, k of 100 to 128 one to two us slower, lists of 8,000 and k of 120 to 128 one to nine faster of 600.
constexpr int kBoundWaveK = 128, kBoundShares = 256, kBoundCand = 192;

}  // namespace ivfpq
