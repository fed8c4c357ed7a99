// The source lists' limit and a block's walk over its stretch in the 32-bit
// arithmetic of the kernel, built with g++ by tests/test_source_walk.py.
#include "../paper_2112_05051_amd/csrc/source_walk.hpp"

extern "C" {
int sw_fits(long long nnz, long long values) { return rich::source_lists_fit(nnz, values); }
int sw_piece() { return rich::GS_PIECE; }
// pieces of the walk over [t0, t1); -1 when it has not ended after `most`
int sw_pieces(uint32_t t0, uint32_t t1, int most) {
    int pieces = 0;
    for (uint32_t base = t0; base < t1; base += rich::GS_PIECE)
        if (++pieces > most) return -1;
    return pieces;
}
}
