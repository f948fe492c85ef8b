// Failure word of a blocked factorization whose wavefronts run ahead of each
// other by up to one panel: it is 0, or the mark of the panel that broke down.
// A wavefront reads it after the barrier that ends panel q; by then a faster
// one may have set it in panel q + 1, which the reader must not see as its own
// panel's failure, or it would leave one barrier before the others.
#pragma once

namespace btc {

constexpr int panel_mark(int q) { return q + 1; }
// Word read after panel q's barrier: did a panel up to q break down?
constexpr bool panel_failed(int word, int q) { return word != 0 && word <= panel_mark(q); }

}  // namespace btc
