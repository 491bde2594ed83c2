// What the walks ask of a caller's tree, found on the host before anything is staged.
#ifndef GBT_TREE_SHAPE_H
#define GBT_TREE_SHAPE_H
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "gbt.h"

namespace {

struct TreeShape {
    int bad_node = -1;      // the first split whose feature or children do not exist: the tree is refused, nothing else is set
    bool compact = true;    // every split has right == left + 1, feature < 2^20 and bin < 4096, and the tree is in order
    bool in_order = true;   // children come after their parents
    bool proper = true;     // in order, and no node is the child of two splits
    int depth = 0;          // in order: steps of the longest walk from the root
};
// scratch: any vector, reused from tree to tree.
// A node of two parents is legal (two splits may lead to the same subtree); its depth is that of the longer way to it.
inline TreeShape tree_shape(const gbt_tree &T, int32_t F, std::vector<int> &scratch) {
    TreeShape s;
    scratch.assign((size_t)T.n_nodes, 0);
    int *__restrict__ depth_of = scratch.data();   // (a child's is at least 1)
    const int32_t *__restrict__ feature = T.feature, *__restrict__ bin = T.bin, *__restrict__ left = T.left, *__restrict__ right = T.right;
    const int n = T.n_nodes;
    int splits = 0, depth = 0;
    bool compact = true, in_order = true;
    for (int i = 0; i < n; ++i) {
        const int32_t f = feature[i];
        if (f < 0) continue;
        const int32_t l = left[i], r = right[i];
        if (f >= F || l < 0 || l >= n || r < 0 || r >= n) {
            s.bad_node = i;
            return s;
        }
        compact &= r == l + 1 && f < (1 << 20) && (uint32_t)bin[i] < 4096u;
        in_order &= l > i && r > i;
        ++splits;
        const int d = depth_of[i] + 1;
        depth_of[l] = depth_of[r] = d;
        depth = std::max(depth, d);
    }
    s.in_order = in_order;
    s.compact = compact && in_order;
    s.proper = in_order;
    if (!in_order) return s;
    s.depth = depth;
    int children = 0;   // (two to a split where none is shared)
    for (int i = 0; i < n; ++i) children += depth_of[i] != 0;
    if (children == 2 * splits) return s;
    s.proper = false;
    s.depth = 0;
    scratch.assign((size_t)n, 0);
    for (int i = 0; i < n; ++i) {
        if (feature[i] < 0) continue;
        const int32_t l = left[i], r = right[i], d = depth_of[i] + 1;
        depth_of[l] = std::max(depth_of[l], d);
        depth_of[r] = std::max(depth_of[r], d);
        s.depth = std::max(s.depth, d);
    }
    return s;
}

// Places for the many-trees kernel, where every left child stands at an odd place of its tree and the right one behind it.
// Returns true where the tree's own ids have that form (grown trees have them: pairs of children are allocated behind the
// root); else place[i] is node i's place, -1 for one that no walk reaches.  The tree is compact and proper: a reachable
// split then takes two places that nothing else takes, so that places stay below n_nodes.
inline bool tree_places(const gbt_tree &T, std::vector<int32_t> &place) {
    bool odd = true;
    for (int i = 0; i < T.n_nodes; ++i) odd = odd && (T.feature[i] < 0 || (T.left[i] & 1));
    place.clear();
    if (odd) return true;
    place.assign((size_t)T.n_nodes, -1);
    place[0] = 0;
    int next = 1;
    for (int i = 0; i < T.n_nodes; ++i)
        if (T.feature[i] >= 0 && place[(size_t)i] >= 0) {
            place[(size_t)T.left[i]] = next;
            place[(size_t)T.right[i]] = next + 1;
            next += 2;
        }
    return false;
}

}  // namespace
#endif
