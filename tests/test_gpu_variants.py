"""GPU parity at the sizes where a kernel variant or a launch rule changes: each test names the
edge it stands on.  Same oracle, same bounds as test_gpu_parity."""
import numpy as np
import pytest
import torch

from oracle import sga_oracle as orc
from paper_2512_02541_amd import binding as agg
from paper_2512_02541_amd import harness, inputs
from test_gpu_parity import (TILE_EDGE_COUNTS, _idx_case, check_list_case, check_output,
                             check_subsample, oshape, run_case)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H", [(1, 1), (1, 7), (1, 8), (3, 3), (1, 12), (2, 10)])
@pytest.mark.parametrize("nq", [200, 600])
def test_pairs_around_the_xcd_count(B, H, nq):
    """(batch, head) pairs below, at and above a multiple of the eight XCDs, at one and at three
    query tiles per pair: the pairs beyond the multiple share the XCDs, and their tiles do not
    divide evenly among them."""
    shape = agg.make_shape(B, 1, 1, nq, 0, H, 64, 1, 3, 0)
    q, k, v = inputs.iid_qkv(B, nq, H, 64, seed=5000 + 100 * B + H, device="cuda")
    run_case(shape, q, k, v, what="pairs %d" % (B * H))
    _idx_case(shape, q, k, v, "pairs %d" % (B * H))


# (B, queries, H, column stride): the strides leave 70 to 520 keys, so that every row can be checked
TAILS = [
    (1, 1000, 16, 9),      # at most a workgroup per CU: the keys are shared by two groups
    (1, 9192, 16, 97),     # narrow workgroups only (192 queries)
    (1, 13740, 16, 97),    # whole rounds of full-width workgroups, then 192-query ones
    (1, 24984, 12, 301),   # ... over pairs that share the XCDs
    (1, 8193, 16, 97),     # narrow workgroups only (192), the last of 129 queries
    (2, 2049, 8, 31),      # two batch elements
    # nine key tiles
    (1, 2600, 16, 5),
    (1, 4096, 16, 8),      # full-width workgroups only
    (1, 13740, 16, 27),
]


@pytest.mark.parametrize("extreme", [False, True])
@pytest.mark.parametrize("case", TAILS)
def test_narrow_tail_workgroups(case, extreme):
    """Launches that end in narrow workgroups, compacted and index-driven.  `extreme`: one query in
    211 leaves the fast path's range, so that full-width and narrow workgroups alike are redone.
    Those queries are 32 times their own key: their own logit is 32 |k|^2 / 8, about 256 and above
    128, every other one at most 32 |k| |k'| cos / 8, a normal of deviation 32.  A rounding of the
    query operand moves a logit by 2^-9 of that, at most 1, so their own column keeps all the
    weight (an arbitrary query scaled up would not: it ties two columns up to that error)."""
    B, nq, H, s_w = case
    shape = agg.make_shape(B, 1, 1, nq, 0, H, 64, 1, s_w, 0)
    q, k, v = inputs.iid_qkv(B, nq, H, 64, seed=6100 + nq, device="cuda")
    if extreme:
        q[:, ::211] = 32 * k[:, ::211]
    run_case(shape, q, k, v, what="tail %s" % (case,))
    _idx_case(shape, q, k, v, "tail %s" % (case,))


@pytest.mark.parametrize("L", [449, 600, 700, 769])
def test_narrow_tail_per_frame(L):
    """A pair per CU and more: each pair's narrow workgroup (128 queries at 600 and 769, 192 at 700)
    follows its full-width ones.  449 keys, the fewest that may take this order, stay at full width."""
    shape = agg.make_shape(1, 16, 1, L, 0, 16, 64, 1, 1, 0, flags=0)
    q, k, v = inputs.iid_qkv(1, shape.NQ, 16, 64, seed=6600 + L, device="cuda")
    O, lse = harness.frame_forward(shape, q, k, v)
    torch.cuda.synchronize()
    rows = np.concatenate([f * L + np.arange(256 * (L // 256) - 40, L) for f in (0, 7, 15)])
    qb, kb, vb = (inputs.bf16_bits(t) for t in (q, k, v))
    want_o, want_lse = orc.frame_rows(oshape(shape), qb, kb, vb, rows)
    got_lse = lse.permute(1, 0, 2).reshape(1, 16, shape.NQ)
    check_output(O, got_lse, want_o, want_lse, rows, "frame tail %d" % L, q, k, shape.scale)


def _bf16(t):
    return t.to(torch.bfloat16).double()


# (heads, rows) -> the tiles of the Q, K and V projections and of the output projection, the one with the
# residual (plan_linear; test_launch_plan.py checks them without a GPU).  "256+64": the rows of whole rounds
# in tiles of 256, the others in tiles of 64, in a launch of their own.
PROJECTIONS = {
    (1, 3): ("64", "64"), (1, 129): ("64", "64"),
    (1, 30000): ("128", "64"),
    (3, 999): ("64", "64"),
    (4, 66048): ("128", "128"),         # every tile whole
    (5, 261): ("64", "64"),
    (16, 21999): ("256+64", "128"),
    (16, 34353): ("256", "256+64"),
    (16, 17319): ("256+128", "256+64"),
    (16, 38631): ("256+64", "256+128"),
    (33, 30000): ("256", "256+128"),    # 2112 channels: the last large tile of every matrix is a quarter full
    (1, 33000): ("128", "128"),         # one k step, at most one tile per workgroup with the residual
    (1, 99999): ("128", "128"),         # ... and several
    (2, 69999): ("128", "128"),         # two k steps, several tiles per workgroup
    (3, 12000): ("128", "128"),         # 192 channels: the last tile of every matrix is half empty
    (3, 64998): ("256", "256"),         # three k steps, and a quarter of every large tile empty
    (5, 45000): ("128", "128"),         # 320 channels, several tiles per workgroup
    (8, 65286): ("256", "256"),         # tiles of 256, whole but for the last tokens, several per workgroup
}


@pytest.mark.parametrize("H,rows", PROJECTIONS)
def test_projection_tiles(H, rows):
    """Projections at the sizes where their tiles change, in a block of three-token frames (their
    attention is three columns) against float64 with the five bf16 roundings that the interface
    states.  Bounds: those of test_global_block."""
    C, L = 64 * H, 3
    shape = agg.make_shape(1, rows // L, 1, L, 0, H, 64, 1, 1, 0)
    assert shape.NQ == rows
    wts = inputs.block_weights(C, seed=rows + H, device="cuda")
    x = inputs.block_input(1, rows, C, seed=rows + H, device="cuda")
    y, _ = harness.block_forward(shape, agg.AGG_BLOCK_FRAME, wts, x)
    x64 = x.double().view(rows, C)
    ln = _bf16(torch.nn.functional.layer_norm(x64, (C,), wts["ln_gamma"].double(),
                                              wts["ln_beta"].double(), wts["ln_eps"]))
    q, k, v = (_bf16(ln @ wts["w_" + n].double().t().contiguous() + wts["b_" + n].double())
               .view(rows // L, L, H, 64).permute(0, 2, 1, 3).contiguous() for n in "qkv")
    s = (q[:, :, :, None, :] * k[:, :, None, :, :]).sum(-1) * 0.125
    o = _bf16((torch.softmax(s, -1)[..., None] * v[:, :, None, :, :]).sum(3))
    o = o.permute(0, 2, 1, 3).reshape(rows, C)
    want = _bf16(x64 + o @ wts["w_o"].double().t().contiguous() + wts["b_o"].double())
    err = (y.double().view(rows, C) - want).abs()
    assert bool(torch.isfinite(y).all())
    assert float(err.max()) <= 6e-2 and float(err.mean()) <= 4e-3, (float(err.max()), float(err.mean()))


# The same around the sizes at which a projection changes from tiles of 64 to larger ones
FEW_PROJECTIONS = {
    # one to five k steps (the ring has four) around whole tiles
    (1, 63): ("64", "64"), (2, 66): ("64", "64"), (3, 192): ("64", "64"), (4, 195): ("64", "64"), (5, 66): ("64", "64"),
    (16, 639): ("64", "64"), (16, 642): ("128", "64"),  # the most token tiles of Q, K and V, and one more
    (33, 192): ("64", "64"),    # 33 k steps
    (3, 9999): ("128", "64"),   # tiles of 128: the last of every matrix half empty
    (2, 16383): ("128", "64"), (2, 16386): ("128", "128"),  # the most token tiles of the output, and one more
}


@pytest.mark.parametrize("H,rows", FEW_PROJECTIONS)
def test_projection_few_tokens(H, rows):
    """The same check around the sizes at which a projection changes from tiles of 64 to larger ones."""
    test_projection_tiles(H, rows)


# (heads, rows) -> tiles, as above: calls whose rows are computed again, 66 at a time, in tiles of 64
SAME_BITS = {
    (2, 16386): ("128", "128"), (5, 7002): ("128", "128"), (16, 3000): ("128", "128"),
    (3, 64998): ("256", "256"), (16, 17319): ("256+128", "256+64"), (16, 38631): ("256+64", "256+128"),
}


@pytest.mark.parametrize("H,rows", SAME_BITS)
def test_projection_bits_do_not_depend_on_the_tiles(H, rows):
    """Every tile size adds a channel's products in the same order.  Frames of three tokens attend to
    nothing else, so a call with some of them gives those rows' bits of the whole call: the first ones, those on
    both sides of the end of whole rounds of tiles of 256, and the last."""
    C, L, few = 64 * H, 3, 66
    wts = inputs.block_weights(C, seed=rows + H, device="cuda")
    x = inputs.block_input(1, rows, C, seed=rows + H, device="cuda")

    def block(x):
        shape = agg.make_shape(1, x.shape[1] // L, 1, L, 0, H, 64, 1, 1, 0)
        return harness.block_forward(shape, agg.AGG_BLOCK_FRAME, wts, x)[0].view(torch.int16)

    y = block(x)
    for at in {0, rows - few} | {end // L * L - 33 for end in (16384, 32768, 38144, rows // 256 * 256)}:
        if at <= rows - few:
            assert torch.equal(block(x[:, at:at + few].contiguous()), y[:, at:at + few]), at


@pytest.mark.parametrize("H", [1, 3, 16, 33])
@pytest.mark.parametrize("B,nq", [(1, 1024), (2, 1026), (1, 70000)])
def test_mean_split_by_heads(H, B, nq):
    """Few partial sums: their rows are shared out by heads.  512 dropped rows are one partial, whose
    workgroups write the means themselves; 513 are two; 35 000 are enough partials that a workgroup
    takes several heads (and at 33 heads the last one fewer)."""
    if nq > 10000 and H == 33:
        nq = 35000
    shape = agg.make_shape(B, 1, 1, nq, 0, H, 64, 1, 2, 0)
    q, k, v = inputs.iid_qkv(B, nq, H, 64, seed=8100 + nq + H, device="cuda")
    buf = harness.alloc(shape, "cuda", poison=True)
    harness.subsample(buf, k, v)
    again = harness.alloc(shape, "cuda", poison=True)
    agg.agg_kv_subsample(shape, k, v, None, None, again.idx, again.kmean, again.vmean,
                         again.workspace, again.workspace.numel())
    torch.cuda.synchronize()
    check_subsample(shape, buf, inputs.bf16_bits(k), inputs.bf16_bits(v))
    assert torch.equal(buf.kmean, again.kmean) and torch.equal(buf.vmean, again.vmean)


@pytest.mark.parametrize("extreme", [False, True])
@pytest.mark.parametrize("nq,s_w", [(66, 1), (130, 1), (250, 1), (257, 1), (3073, 1), (3200, 1), (4160, 3)])
def test_keys_shared_by_two_groups(nq, s_w, extreme):
    """At most one workgroup per CU: two groups of wavefronts share the key tiles, an even and an odd
    number of them: 2 (the fewest that are shared), 3, 4, 5, 49, 50 and 22.  `extreme`: rows that leave
    the fast path's range, as in test_narrow_tail_workgroups; the same launch redoes them."""
    shape = agg.make_shape(1, 1, 1, nq, 0, 2, 64, 1, s_w, 0)
    q, k, v = inputs.iid_qkv(1, nq, 2, 64, seed=6900 + nq, device="cuda")
    if extreme:
        q[:, ::211] = 32 * k[:, ::211]
    run_case(shape, q, k, v, what="shared keys %d" % nq)
    _idx_case(shape, q, k, v, "shared keys %d" % nq)


# ---- the kernels of four wavefronts, which do nearly all the work of larger calls ---------------
# Launches of at most one narrow workgroup per CU go to eight wavefronts that share the keys, so
# the sweeps below stay beyond that.  tests/test_launch_plan.py checks, without a GPU, that each size
# here is cut as it says.
QUERIES_BY_WIDTH = {0: 4096, 192: 2748, 128: 4122}  # last workgroups' width -> queries, with 16 heads


def _shape_of_keys(B, nq, nkeys, H):
    """nq queries, nkeys kept rows: all but one of them special tokens."""
    return agg.make_shape(B, 1, 1, nq - nkeys + 1, nkeys - 1, H, 64, 1, nq, 0)


def _some_rows(nq):
    """Both sides of every 64th row of the last two workgroups' worth, and every 61st row."""
    end = {r + d for r in range(nq - nq % 64, max(0, nq - 600), -64) for d in (-1, 0, 1)}
    return np.array(sorted(r for r in end | set(range(0, nq, 61)) | {nq - 2, nq - 1} if 0 <= r < nq))


@pytest.mark.parametrize("nkeys", TILE_EDGE_COUNTS)
def test_key_counts_of_four_wavefront_kernels(nkeys):
    """1 to 8, 24, 25 and 26 key tiles, the last one of 1, 63 and 64 keys, at each width, compacted and
    index-driven; and the same counts as rows in place, by per-frame attention."""
    for width, nq in QUERIES_BY_WIDTH.items():
        shape = _shape_of_keys(1, nq, nkeys, 16)
        assert agg.agg_kv_count(shape)[0] == nkeys
        q, k, v = inputs.iid_qkv(1, nq, 16, 64, seed=9100 + nkeys + width, device="cuda")
        run_case(shape, q, k, v, rows=_some_rows(nq), what="%d keys, width %d" % (nkeys, width))
        _idx_case(shape, q, k, v, "%d keys, width %d" % (nkeys, width))
    _frame_case(33, nkeys, 8, 9400 + nkeys)


@pytest.mark.parametrize("nkeys", [31, 32, 33, 96, 97, 1568, 1569])
def test_half_filled_last_tiles(nkeys):
    """A last tile of up to 32 keys is walked half: 31, 32 and 33 keys in it, as the only tile, the second
    and the 25th, at each width, in the launches whose wavefronts share the keys, and redone."""
    for width, nq in QUERIES_BY_WIDTH.items():
        shape = _shape_of_keys(1, nq, nkeys, 16)
        q, k, v = inputs.iid_qkv(1, nq, 16, 64, seed=9700 + nkeys + width, device="cuda")
        run_case(shape, q, k, v, rows=_some_rows(nq), what="%d keys, width %d" % (nkeys, width))
        _idx_case(shape, q, k, v, "%d keys, width %d" % (nkeys, width))
    shape = _shape_of_keys(1, nkeys + 70, nkeys, 2)
    q, k, v = inputs.iid_qkv(1, shape.NQ, 2, 64, seed=9800 + nkeys, device="cuda")
    run_case(shape, q, k, v, what="%d shared keys" % nkeys)
    _idx_case(shape, q, k, v, "%d shared keys" % nkeys)
    _frame_case(33, nkeys, 8, 9900 + nkeys)
    _frame_case(33, nkeys, 8, 9900 + nkeys, _spoil("own"))


def _frame_case(N, L, H, seed, spoil=None):
    shape = agg.make_shape(1, N, 1, L, 0, H, 64, 1, 1, 0, flags=0)
    q, k, v = inputs.iid_qkv(1, shape.NQ, H, 64, seed=seed, device="cuda")
    if spoil:
        q, k = spoil(q, k)
    O, lse = harness.frame_forward(shape, q, k, v)
    torch.cuda.synchronize()
    rows = np.concatenate([f * L + _some_rows(L) for f in (0, N // 2, N - 1)] +
                          [np.arange(0, shape.NQ, 211)])
    rows = np.unique(rows)
    want_o, want_lse = orc.frame_rows(oshape(shape), *(inputs.bf16_bits(t) for t in (q, k, v)), rows)
    got_lse = lse.permute(1, 0, 2).reshape(1, H, shape.NQ)
    check_output(O, got_lse, want_o, want_lse, rows, "%d frames of %d" % (N, L), q, k, shape.scale)


# 261 pairs.  Up to six key tiles: full width throughout; with 520 keys a pair may end in a narrow
# workgroup, by its queries beyond 1024.
QUERY_EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513]
QUERY_EDGES_BY_PAIR = {1025: 128, 1087: 128, 1151: 128, 1152: 128, 1153: 192, 1215: 192, 1216: 192,
                       1217: 0, 1280: 0}


@pytest.mark.parametrize("nq", QUERY_EDGES + list(QUERY_EDGES_BY_PAIR))
def test_query_counts_of_four_wavefront_kernels(nq):
    """Query counts around the tile of 16, the wavefront of 32, 48 or 64 and the workgroup of 128, 192
    or 256, at 9 batch elements of 29 heads."""
    B, H = 9, 29
    nkeys = 520 if nq in QUERY_EDGES_BY_PAIR else (nq + 2) // 3
    shape = _shape_of_keys(B, nq, nkeys, H)
    q, k, v = inputs.iid_qkv(B, nq, H, 64, seed=7200 + nq, device="cuda")
    run_case(shape, q, k, v, rows=_some_rows(nq), what="%d queries" % nq)
    _idx_case(shape, q, k, v, "%d queries" % nq)


# Rows that leave the fast path's range, on every route that redoes them: (queries, heads, keys, width
# of the last workgroups).  Up to 127 key tiles they are redone in place, beyond that by the second
# launch; from 25 tiles on a sum that overflows ends the fast pass at the 24th.
REDO = {
    "keys": [(4096, 16, 30, 0), (2748, 16, 300, 192), (4122, 16, 300, 128),       # in place
             (4096, 16, 600, 0), (2748, 16, 600, 192), (4122, 16, 600, 128),
             (4096, 16, 2500, 0), (2748, 16, 2500, 192), (4122, 16, 2500, 128),   # in place, early
             (8448, 12, 8200, 0), (8500, 8, 8200, 128), (8560, 16, 8200, 192)],   # second launch, early
    "list": [(2748, 16, 300, 192), (4096, 16, 600, 0), (2748, 16, 600, 192), (4122, 16, 600, 128),
             (4096, 16, 8200, 0), (2748, 16, 8200, 192), (4122, 16, 8200, 128)],
    "dense": [(2600, 16, 2600, 192), (3700, 16, 3700, 0), (4122, 16, 4122, 128),  # in place, early
              (8193, 16, 8193, 192), (8448, 12, 8448, 0), (8500, 8, 8500, 128)],  # second launch, early
    # 256 pairs: 16 frames of 16 heads
    "frame": [(50, 256, 50, 0), (300, 256, 300, 0), (768, 256, 768, 0), (700, 256, 700, 192),
              (1374, 256, 1374, 128), (2000, 256, 2000, 0)],                      # in place
}


def _spoil(extreme):
    """Queries (and keys) of which some rows, or all, leave the fast path's range: `own` and `few` as
    in test_narrow_tail_workgroups, one row in 211 or two in all; `low`: every logit near -240, so that
    every sum is below the range and no sum overflows."""
    def own(q, k):
        q[:, ::211] = 32 * k[:, ::211]
        return q, k

    def few(q, k):
        for r in (3, q.shape[1] - 2):
            q[:, r] = 32 * k[:, r]
        return q, k

    def low(q, k):
        u = torch.ones(64, device="cuda")
        return (-30.0 * u).expand_as(q).to(torch.bfloat16).contiguous(), (u + 0.05 * k.float()).to(torch.bfloat16)

    return {"own": own, "few": few, "low": low}[extreme]


@pytest.mark.parametrize("extreme", ["own", "few", "low"])
@pytest.mark.parametrize("kind,case", [(kind, c) for kind, cases in REDO.items() for c in cases])
def test_rows_redone_on_every_route(kind, case, extreme):
    nq, H, nkeys, width = case
    seed = 7700 + nq + nkeys
    if kind == "frame":
        return _frame_case(16, nq, H // 16, seed, _spoil(extreme))
    q, k, v = inputs.iid_qkv(1, nq, H, 64, seed=seed, device="cuda")
    q, k = _spoil(extreme)(q, k)
    rows = np.unique(np.concatenate([_some_rows(nq)[::2], np.arange(0, nq, 211), [3, nq - 2]]))
    what = "%s %s %s" % (kind, case, extreme)
    if kind == "keys":
        shape = _shape_of_keys(1, nq, nkeys, H)
        run_case(shape, q, k, v, rows=rows, what=what)
        _idx_case(shape, q, k, v, what)
    elif kind == "list":
        shape = agg.make_shape(1, 1, 1, nq, 0, H, 64, 1, 3, 0)
        gen = torch.Generator().manual_seed(seed)
        # (a list longer than the sequence names tokens more than once)
        lst = torch.cat([torch.randperm(nq, generator=gen) for _ in range(-(-nkeys // nq))])
        lst = lst[:nkeys].to(torch.int32).view(1, nkeys).cuda()
        check_list_case(shape, lst, q, k, v, rows[::2], what)
    else:
        shape = agg.make_shape(1, 1, 1, nq, 0, H, 64, 1, 1, 0, flags=0)
        O, lse = harness.dense_forward(shape, q, k, v)
        torch.cuda.synchronize()
        want_o, want_lse = orc.dense_rows(oshape(shape), *(inputs.bf16_bits(t) for t in (q, k, v)), rows)
        check_output(O, lse, want_o, want_lse, rows, what, q, k, shape.scale)
