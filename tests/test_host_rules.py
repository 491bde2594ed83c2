"""Rules the library's host side decides by, compiled apart from it and checked without a GPU: what a walk may assume of a
caller's tree (csrc/tree_shape.h), and how many histogram jobs and
evaluation records a level planned on the device can have (csrc/gbt_internal.h)."""
import ctypes as C
import subprocess

import numpy as np
import pytest

import hist_tiles

SOURCE = r"""
#include "gbt_internal.h"
#include "kernels_split.hip"
#include "tree_shape.h"

#define API extern "C" __attribute__((visibility("default")))

// The most jobs a level can have beyond gbt_plan_jobs_max (<= 0), over `count` numbers of rows its `splits` built children
// have in all and every candidate length; each child has one row more than whole pieces.
API long long jobs_over_bound(int num_cu, int per_cu, int tiles, long long max_rows, double merge, long long n, long long splits,
                              const long long *rows, int count) {
    PlanHistRule r{};
    r.pieces_max = std::max<int64_t>(1, (int64_t)num_cu * per_cu / tiles);
    r.min_rows = 256;
    r.max_rows = max_rows;
    r.merge = merge;
    r.num_cu = num_cu;
    r.tiles = tiles;
    const long long bound = gbt_plan_jobs_max(r, n, splits);
    long long over = -bound;
    for (int k = 0; k < count; ++k)
        for (int c = 0; c < kPieceCandidates; ++c) {
            const long long length = gbt_piece_candidate(r, rows[k], c), with_rows = std::min(splits, rows[k]);
            over = std::max(over, ((rows[k] - with_rows) / length + with_rows) * tiles - bound);
        }
    return over;
}

API int tile_columns(int F, int bits, int ft_max, double gathered) { return gbt_tile_columns(F, bits, ft_max, gathered); }
API int window(int bits) { return gbt_histw_window(bits); }
API int eval_chunks(int F, int n_nodes, long long budget) { return gbt_eval_chunks(F, n_nodes, (size_t)budget); }
API long long eval_records_max(long long n_nodes) { return gbt_eval_records_max(n_nodes); }
API long long split_bytes() { return (long long)sizeof(gbt_split); }

// out: bad_node, compact, in_order, proper, depth, odd; place: n_nodes places (where the tree is compact, proper and not odd)
API void shape_of(int n_nodes, int F, int *feature, int *bin, int *left, int *right, int *out, int *place) {
    gbt_tree T{};
    T.capacity = T.n_nodes = n_nodes;
    T.feature = feature;
    T.bin = bin;
    T.left = left;
    T.right = right;
    std::vector<int> scratch(3, 7);
    const TreeShape s = tree_shape(T, F, scratch);
    out[0] = s.bad_node;
    out[1] = s.compact;
    out[2] = s.in_order;
    out[3] = s.proper;
    out[4] = s.depth;
    out[5] = -1;
    if (s.bad_node >= 0 || !s.compact || !s.proper) return;
    std::vector<int32_t> p(5, 3);
    out[5] = tree_places(T, p);
    for (size_t i = 0; i < p.size(); ++i) place[i] = p[i];
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    from paper_1806_11248_amd import build
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.hip", d / "librules.so"
    src.write_text(SOURCE)
    r = subprocess.run([build._hipcc(), *build.FLAGS, "-shared", "-o", str(lib), str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return C.CDLL(str(lib))


def _shape(rules, F, splits, n_nodes):
    """splits: {node: (feature, left, right)}"""
    feature, left, right = (np.full(n_nodes, -1, np.int32) for _ in range(3))
    for i, (f, l, r) in splits.items():
        feature[i], left[i], right[i] = f, l, r
    out, place = np.zeros(6, np.int32), np.full(n_nodes, -9, np.int32)
    p = [a.ctypes.data_as(C.c_void_p) for a in (feature, np.zeros(n_nodes, np.int32), left, right, out, place)]
    rules.shape_of(n_nodes, F, *p)
    return dict(zip(("bad_node", "compact", "in_order", "proper", "depth", "odd"), out.tolist())), place


def _longest(splits, i=0):
    return 1 + max(_longest(splits, c) for c in splits[i][1:]) if i in splits else 0


# splits that lead to the same pair of children, or to pairs that overlap
SHARED = {
    "even ids": ({0: (0, 2, 3), 2: (1, 4, 5), 3: (2, 4, 5)}, 6),
    "odd ids": ({0: (0, 1, 2), 1: (1, 3, 4), 2: (2, 3, 4)}, 5),
    "overlapping pairs": ({0: (0, 1, 2), 1: (1, 3, 4), 2: (2, 4, 5)}, 6),
    # 13 and 14 are four and three steps below the root; only the longer way counts
    "two depths": ({0: (0, 1, 2), 1: (1, 3, 4), 2: (2, 11, 12), 3: (0, 5, 6), 5: (1, 13, 14), 11: (2, 13, 14),
                    13: (0, 15, 16)}, 17),
    # many parents of one pair: places handed out per parent would run far past the tree
    "many parents": ({0: (0, 2, 3), 2: (1, 4, 5), 3: (1, 6, 7), 4: (0, 8, 9), 5: (0, 8, 9), 6: (0, 8, 9), 7: (0, 8, 9)}, 10),
}


@pytest.mark.parametrize("name", SHARED)
def test_shared_children_are_no_proper_tree(rules, name):
    splits, n_nodes = SHARED[name]
    s, _ = _shape(rules, 3, splits, n_nodes)
    assert s["bad_node"] == -1 and s["compact"] and s["in_order"] and not s["proper"]
    assert s["depth"] == _longest(splits)


def test_trees_that_are_refused_or_out_of_order(rules):
    assert _shape(rules, 3, {0: (3, 1, 2)}, 3)[0]["bad_node"] == 0                   # no such feature
    assert _shape(rules, 3, {0: (0, 1, 2), 2: (0, 3, 4)}, 4)[0]["bad_node"] == 2     # no such child
    s, _ = _shape(rules, 3, {0: (0, 3, 4), 3: (1, 1, 2)}, 5)                         # a child before its parent
    assert s["bad_node"] == -1 and not s["in_order"] and not s["proper"] and not s["compact"]
    s, _ = _shape(rules, 3, {0: (0, 1, 1)}, 2)                                       # both children the same node
    assert s["bad_node"] == -1 and not s["proper"] and not s["compact"]


@pytest.mark.parametrize("gaps", [0.0, 0.3])
def test_places_of_proper_trees(rules, gaps):
    """Whatever the ids: every reachable node has a place of its own below n_nodes, a left child an odd one with its sibling
    behind it, the root the first."""
    rng = np.random.default_rng(5)
    for n_splits in (0, 1, 2, 7, 40, 300):
        splits, open_, at = {}, [0], 1
        for _ in range(n_splits):
            i = open_.pop(int(rng.integers(0, len(open_))))
            at += int(rng.random() < gaps)
            splits[i] = (0, at, at + 1)
            open_ += [at, at + 1]
            at += 2
        s, place = _shape(rules, 1, splits, at)
        assert s["compact"] and s["proper"] and s["depth"] == _longest(splits)
        assert s["odd"] == all(l % 2 for _, l, _ in splits.values())
        if s["odd"]:
            continue
        reached = {0} | {c for v in splits.values() for c in v[1:]}
        assert place[0] == 0 and sorted(place[list(reached)]) == list(range(len(reached)))
        assert all(place[i] == -1 for i in range(at) if i not in reached)
        assert all(place[l] % 2 == 1 and place[r] == place[l] + 1 for _, l, r in splits.values())


@pytest.mark.parametrize("kind", ["dense", "sparse"])
def test_bound_of_a_levels_histogram_jobs(rules, kind):
    """No level makes more jobs than its launch and its table hold, for any number of rows the built children can have (half
    the matrix): near every power of two and square (where the candidate lengths round), near the most, and at random."""
    rng = np.random.default_rng(3)
    rules.jobs_over_bound.restype = C.c_longlong
    rules.jobs_over_bound.argtypes = [C.c_int] * 3 + [C.c_longlong, C.c_double] + [C.c_longlong] * 2 + [C.c_void_p, C.c_int]
    for _ in range(3000):
        n = int(np.exp(rng.uniform(0, np.log(4e9))))
        most = n // 2
        rows = np.concatenate([2 ** np.arange(32), np.arange(1, 65536, 257) ** 2, most - np.arange(64),
                               np.exp(rng.uniform(0, np.log(most + 1), 300)).astype(np.int64)])
        rows = np.unique(np.concatenate([rows - 1, rows, rows + 1]))
        rows = np.ascontiguousarray(rows[(rows >= 0) & (rows <= most)], np.int64)
        tiles = int(rng.choice([1, 1, 2, 3, 8, 40, 700]))
        if kind == "dense":
            per_cu, max_rows = int(rng.choice([1, 8, 64])), int(rng.choice([2 ** 18 - 1, 2 ** 21]))
            merge = 0.15 * int(rng.integers(2, 4097)) * float(rng.choice([1, 96, 100_000])) / 96.0
        else:
            per_cu, max_rows = 16 * int(rng.choice([1, 64])), int(rng.choice([2 ** 18 - 1, 2 ** 24]))
            merge = float(rng.choice([0.08, 0.25])) * int(rng.integers(64, 20_000)) / (8 + 300 * rng.random()) * rng.random() + 1e-3
        splits = int(2 ** rng.integers(0, 16))
        over = rules.jobs_over_bound(256, per_cu, tiles, max_rows, merge, n, splits, rows.ctypes.data, len(rows))
        assert over <= 0, (n, tiles, per_cu, max_rows, merge, splits, over)


def test_bound_of_a_levels_evaluation_records(rules):
    """The table of a planned level's split records holds every number of nodes and chunks; a budget that holds less (one
    record per node is the least) is kept."""
    rules.eval_records_max.restype = rules.split_bytes.restype = C.c_longlong
    rules.eval_records_max.argtypes = [C.c_longlong]
    rules.eval_chunks.argtypes = [C.c_int, C.c_int, C.c_longlong]
    size = rules.split_bytes()
    nodes = sorted({v for k in range(17) for v in (2 ** k - 1, 2 ** k, 2 ** k + 1) if 0 < v <= 65536} | set(range(1, 9000, 97)))
    for level_nodes in (1, 64, 4096, 65536):
        room = rules.eval_records_max(level_nodes)
        for n_nodes in [v for v in nodes if v <= level_nodes]:
            for F in (1, 4, 5, 13, 253, 2000, 1 << 20):
                assert n_nodes * rules.eval_chunks(F, n_nodes, 1 << 60) <= room, (level_nodes, n_nodes, F)
                tight = 3 * n_nodes * size
                assert n_nodes * rules.eval_chunks(F, n_nodes, tight) * size <= tight


@pytest.mark.parametrize("bits", [b for b in range(1, 17) if b != 8])
def test_column_tiles_by_the_slots_the_kernel_issues(rules, bits):
    """A tile costs the slots of its lanes, one, two or four, less where all are full, and ten per lane; at least its line of a long
    row, and one more where the rows come from HBM; the last tile no less than the others.  No even split up to eight tiles past
    the fewest, nor full windows, cost less than the tiles taken."""
    rules.tile_columns.argtypes = [C.c_int] * 3 + [C.c_double]
    E = rules.window(bits)
    full = {1: 0.67, 2: 0.69, 4: 0.74 if E <= 24 else 0.85}

    def cost(F, ft, far):
        def tile(t):
            lanes = 1 if t <= E else 2 if t <= 2 * E else 4
            slots = lanes * (10 + -(-t // lanes)) * (full[lanes] if t == lanes * E else 1)
            row = F * bits / 8
            return max(slots, 35 * min(1, row / 256) + 10 * min(1, row / 1500)) + 30 * far
        return (-(-F // ft) - 1) * tile(ft) + max(tile(ft), tile((F - 1) % ft + 1))

    for F in [*range(1, 420), 700, 1000, 2000, 5001, 1 << 20]:
        for ft_max in {min(F, m) for m in (1, 2, 5, E - 1, E, E + 7, 2 * E, 4 * E)} - {0}:
            least = -(-F // ft_max)
            others = [-(-F // nt) for nt in range(least, min(least + 8, F) + 1)] + [w * E for w in full if w * E <= ft_max]
            for far in (False, True):
                ft = rules.tile_columns(F, bits, ft_max, 1e9 * far)
                assert 1 <= ft <= ft_max <= 4 * E
                assert cost(F, ft, far) <= min(cost(F, o, far) for o in others) * (1 + 1e-12), (F, ft_max, ft)


def test_column_tiles_of_known_shapes(rules):
    rules.tile_columns.argtypes = [C.c_int] * 3 + [C.c_double]
    # full windows with a ragged last tile: 36 and 52 columns of 9 bits, 100 of 6, a wide matrix
    assert [rules.tile_columns(*a, 0.0) for a in ((36, 9, 20), (52, 9, 20), (100, 6, 78), (40, 6, 40), (1000, 6, 78), (2000, 6, 80))] == \
        [13, 13, 20, 20, 40, 80]
    # ... that has no more to wait for than the others: 150 columns of 4 and 1 bits, not in tiles of 124 or 128 and what is left
    assert [rules.tile_columns(*a, 0.0) for a in ((150, 4, 124), (150, 1, 128), (124, 4, 124), (1000, 4, 124))] == [31, 32, 31, 62]
    # gathered from past the caches: half as many tiles
    assert [rules.tile_columns(50, 9, 25, b) for b in (0.0, 168e6, 560e6)] == [13, 13, 25]
    # bytes: more tiles than needed only where they save a fifth of the slots
    assert [rules.tile_columns(*a, 0.0) for a in ((33, 8, 19), (50, 8, 19), (70, 8, 64), (400, 8, 38))] == [11, 13, 35, 31]


def test_column_tiles_the_kernel_tests_count_on(rules):
    rules.tile_columns.argtypes = [C.c_int] * 3 + [C.c_double]
    for table, windows, gathered in ((hist_tiles.TWO, 2, 0), (hist_tiles.FOUR, 4, 0), (hist_tiles.FOUR_GATHERED, 4, hist_tiles.GATHERED_BYTES)):
        for bits, F in table.items():
            E = rules.window(bits)
            ft = rules.tile_columns(F, bits, min(F, 4 * E), gathered)
            assert ft == windows * E and windows * E > F % ft > windows // 2 * E, (bits, F, ft)
