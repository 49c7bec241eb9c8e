// Host build of the GEMM kernels' work decomposition (layout.hpp), for tests/test_gemm_blocks.py.
#include "../paper_2508_00441_amd/csrc/layout.hpp"

using namespace ozaki;

extern "C" {

// 0 if the workgroups 0 ... total - 1 take every item (group, block row, block column) exactly once
int work_items_cover(unsigned groups, unsigned blocks_m, unsigned blocks_n, int unit, int height) {
    const unsigned total = groups * blocks_m * blocks_n;
    unsigned char* seen = new unsigned char[total]();
    int bad = 0;
    for (unsigned b = 0; b < total; ++b) {
        const WorkItem w = work_item(b, total, WorkOrder{unit, height}, blocks_m, blocks_n);
        if (w.gi >= groups || w.bm >= blocks_m || w.bn >= blocks_n) { bad = 1; break; }
        if (seen[(w.gi * blocks_n + w.bn) * blocks_m + w.bm]++) { bad = 2; break; }
    }
    delete[] seen;
    return bad;
}

// 0 if the groups of the pass g_hi ... g_lo hold every pair of it once, each in its slot, none longer than len, start where
// the accumulation expects them, and the list for the kernels holds the same groups, longest first
int groups_cover(int s, int full, int len, int g_hi, int g_lo) {
    const PairOrder o{s, full, len};
    Pass ps{g_hi, g_lo, 0, 0};
    for (int g = g_hi; g >= g_lo; --g) { ps.npairs += diag_len(o, g); ps.ngroups += diag_groups(o, g); }
    static GroupList list;
    list_groups(o, ps, list);
    if (list.listed != (ps.ngroups <= MAX_LISTED_GROUPS ? ps.ngroups : 0)) return 5;
    for (int listed = 0; listed < 2; ++listed) {
        int seen[MAX_PAIRS] = {}, last = MAX_SLICES;
        for (int gi = 0; gi < ps.ngroups; ++gi) {
            const Group r = listed ? listed_group(list, o, ps, gi) : pass_group(o, ps, gi);
            if (r.len < 1 || r.len > len) return 1;
            if (listed && list.listed && r.len > last) return 6;
            last = r.len;
            int slot = 0, g = g_hi;
            for (; g > r.p0 + r.q0; --g) slot += diag_len(o, g);
            if (g < g_lo || slot + r.p0 - diag_first_p(o, g) != r.slot) return 2;
            for (int j = 0; j < r.len; ++j) {
                if (r.p0 + j > s || r.q0 - j < 1) return 3;
                if (((r.p0 - diag_first_p(o, g) + j) % len == 0) != (j == 0)) return 7;
                ++seen[r.slot + j];
            }
        }
        for (int z = 0; z < ps.npairs; ++z)
            if (seen[z] != 1) return 4;
    }
    return 0;
}

}  // extern "C"
