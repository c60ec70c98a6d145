"""The prefill's attention over tiles of rows (bf16, 64 rows and more) against
the split kernels that fewer rows take (selected by an explicit attention
split): the same arithmetic up to the order of the sums and the split of the
keys, so cache rows agree within the storage tolerance, and NaN rows are the
same ones."""
import numpy as np
import pytest

from fe_synth import configs as C
from fe_synth import make_update_rows, make_weights
from fe_synth.gen import float_tensor
from tests.parity import TOL, assert_rows_close

pytestmark = pytest.mark.gpu
SELF = lambda c: c.with_(cascade_ctx="self", name=c.name + "_self")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _update(cfg, w, up, split, max_prefix, chunk_rows=1024):
    """Caches (fp64 values) after one update; split 0 takes the tiles."""
    import torch
    from paper_2509_20416_amd import Drafter
    from paper_2509_20416_amd.drafter import to_device
    dr = Drafter(cfg, w, max_batch=1, max_prefix=max_prefix, max_topk=cfg.topk)
    dr.set_attention_split(split)
    shape = (up.cache_rows, cfg.n_kv_heads, cfg.head_dim)
    kv = [[to_device(float_tensor(f"tiles.{n}{l}", shape, 5, cfg.dtype), cfg.dtype, dr.device)
           for l in range(cfg.n_layers)] for n in "kv"]
    dr.kv_update(to_device(up.features, cfg.dtype, dr.device), to_device(up.tokens, "i32", dr.device),
                 to_device(up.positions, "i32", dr.device), to_device(up.dst_rows, "i32", dr.device),
                 *kv, chunk_rows=chunk_rows)
    torch.cuda.synchronize()
    got = [t.double().cpu().numpy().reshape(up.cache_rows, -1) for side in kv for t in side]
    dr.close()
    return got


# A tile is 64 (row, head) columns: 64, 32, 16 and 8 rows where a KV head has 1,
# 2, 4 and 8 query heads.
CASES = [  # rows per sequence, prefix per sequence
    (SELF(C.SMALL_GQA_BF16), [64], [0]),                        # the fewest rows; 16-row tiles
    (SELF(C.SMALL_GQA_BF16), [33, 1, 31, 65, 2], [0, 700, 31, 32, 1]),  # runs across tile edges
    (SELF(C.SMALL_GQA8_BF16_D128), [17, 100], [0, 333]),        # 8-row tiles, head dim 128
    (SELF(C.SMALL_MHA_BF16_D128), [129, 140], [5, 0]),          # 64-row tiles
    (SELF(C.SMALL_GQA2_BF16), [70, 63], [0, 64]),               # 32-row tiles
    (SELF(C.SMALL_GQA_BF16), [1] * 70, list(range(70))),        # every row a run of its own
    (SELF(C.SMALL_GQA_BF16), [1100], [0]),                      # one run over two chunks
    # one row short of a tile, a tile, one row more, one more than two tiles
    (SELF(C.SMALL_GQA8_BF16_D128), [7, 8, 9, 17, 25], [40, 0, 3, 31, 32]),
    (SELF(C.SMALL_GQA_BF16), [15, 16, 17, 33], [0, 33, 64, 5]),
    (SELF(C.SMALL_GQA2_BF16), [31, 32, 33, 65], [9, 0, 65, 30]),
    (SELF(C.SMALL_MHA_BF16_D128), [63, 64, 65, 129], [0, 31, 7, 100]),
]


@pytest.mark.parametrize("cfg,acc,plens", CASES, ids=[f"{c.name}-{len(a)}x{a[0]}" for c, a, _ in CASES])
def test_tiles_match_split_kernels(cfg, acc, plens):
    acc, plens = np.asarray(acc, np.int32), np.asarray(plens, np.int32)
    cap = int((acc + plens).max())
    up = make_update_rows(cfg, acc, plens, capacity=cap, seed=11)
    w = make_weights(cfg, 3)
    for i, (a, b) in enumerate(zip(_update(cfg, w, up, 0, cap), _update(cfg, w, up, 4, cap))):
        assert_rows_close(f"array {i}", a[up.dst_rows], b[up.dst_rows], TOL["bf16"])


# More rows than one scan of the plan: the run that a round leaves off in goes on
# in the next, at rows 1024 and 2048 that are inside a tile, and the tiles are
# numbered on; more tiles than one round lists
ROUNDS = [
    (SELF(C.SMALL_GQA_BF16), [5, 2200, 3], [0, 7, 2]),
    (SELF(C.SMALL_GQA8_BF16_D128), [1021, 1, 2, 1050], [0, 3, 9, 1]),
    (SELF(C.SMALL_GQA2_BF16), [1, 2] * 760, [3, 0, 1, 6] * 380),
]


@pytest.mark.parametrize("cfg,acc,plens", ROUNDS, ids=[f"{c.name}-{len(a)}x{a[0]}" for c, a, _ in ROUNDS])
def test_plan_of_several_rounds(cfg, acc, plens):
    acc, plens = np.asarray(acc, np.int32), np.asarray(plens, np.int32)
    cap = int((acc + plens).max())
    up = make_update_rows(cfg, acc, plens, capacity=cap, seed=15)
    assert len(up.tokens) > 2048
    for row in (1023, 1024, 2047, len(up.tokens) - 1):
        up.positions[row] = cap + row  # no such position: a tile of its own, NaN
    w = make_weights(cfg, 3)
    tiles, split = (_update(cfg, w, up, s, cap, chunk_rows=2600) for s in (0, 4))
    for i, (a, b) in enumerate(zip(tiles, split)):
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b), err_msg=f"array {i}")
        ok = up.dst_rows[~np.isnan(b[up.dst_rows]).any(1)]
        assert len(ok) > 1000
        assert_rows_close(f"array {i}", a[ok], b[ok], TOL["bf16"])


# Histories that are cut into pieces over several workgroups (more than 32
# stages of 32 keys), next to short ones and to the longest that stay whole;
# the cut tiles' heights as above, and pieces that most columns of a wave see
# none of
LONG = [
    (SELF(C.SMALL_GQA_BF16), [60, 3, 1, 9], [4200, 0, 1024, 1025]),
    (SELF(C.SMALL_GQA8_BF16_D128), [9, 70, 1], [2500, 0, 1900]),
    (SELF(C.SMALL_MHA_BF16_D128), [65, 2], [1100, 3000]),
    (SELF(C.SMALL_GQA2_BF16), [40, 33], [990, 1023]),
    (SELF(C.SMALL_GQA_BF16), [1] * 64, [2400] + [20] * 63),
]


@pytest.mark.parametrize("cfg,acc,plens", LONG, ids=[f"{c.name}-{len(a)}x{a[0]}" for c, a, _ in LONG])
def test_long_ragged_histories_match_oracle(cfg, acc, plens):
    from tests.test_gpu_kv_update_self import _run
    acc, plens = np.asarray(acc), np.asarray(plens)
    cap = int((acc + plens).max())
    _run(cfg.with_(n_layers=3), make_update_rows(cfg, acc, plens, capacity=cap, seed=16), 1024, max_prefix=cap)


@pytest.mark.parametrize("split", [0, 4])
def test_infinite_values_in_a_history_stay_apart(split):
    """A cached value row of infinities makes NaN or infinite the rows that see
    it, in whichever piece of the history it lies, and no other row."""
    import torch
    from paper_2509_20416_amd import Drafter
    from paper_2509_20416_amd.drafter import to_device
    cfg = SELF(C.SMALL_GQA_BF16).with_(n_layers=2)
    up = make_update_rows(cfg, np.array([70, 20]), np.array([2000, 2000]), capacity=2100, seed=17)
    dr = Drafter(cfg, make_weights(cfg, 3), max_batch=1, max_prefix=2100, max_topk=cfg.topk)
    dr.set_attention_split(split)
    shape = (up.cache_rows, cfg.n_kv_heads, cfg.head_dim)
    kv = [[to_device(float_tensor(f"inf.{n}{l}", shape, 5, cfg.dtype), cfg.dtype, dr.device)
           for l in range(2)] for n in "kv"]
    kv[1][0][1300] = float("inf")                       # the first sequence's history, layer 1
    dr.kv_update(to_device(up.features, cfg.dtype, dr.device), to_device(up.tokens, "i32", dr.device),
                 to_device(up.positions, "i32", dr.device), to_device(up.dst_rows, "i32", dr.device), *kv)
    last = kv[0][1][torch.from_numpy(up.dst_rows.astype(np.int64)).to(dr.device)].float().cpu().numpy()
    dr.close()
    assert np.isnan(last[:70]).all((1, 2)).all() and np.isfinite(last[70:]).all()


def test_tiles_keep_nan_rows_apart():
    """A row whose token is outside the vocabulary is NaN, and with it the later
    rows of its sequence (they see its key), but no earlier row of its tile; a
    row whose position-0 row lies before the cache is NaN by itself."""
    cfg = SELF(C.SMALL_GQA_BF16)
    up = make_update_rows(cfg, np.array([80, 40]), np.array([0, 9]), capacity=96, seed=12)
    up.tokens[50] = cfg.target_vocab + 5
    up.positions[3] = 60          # dst 3 - 60 < 0
    w = make_weights(cfg, 3)
    tiles, split = (_update(cfg, w, up, s, 96) for s in (0, 4))
    for i, (a, b) in enumerate(zip(tiles, split)):
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b), err_msg=f"array {i}")
        ok = up.dst_rows[~np.isnan(b[up.dst_rows]).any(1)]
        assert_rows_close(f"array {i}", a[ok], b[ok], TOL["bf16"])
    last = np.isnan(tiles[cfg.n_layers - 1][up.dst_rows]).any(1)  # the deepest layer's keys
    assert last[50:80].all() and last[3] and not last[:3].any() and not last[80:].any()


# MLP widths whose gate/up GEMM (512 wide K) takes each tile shape at 300 rows:
# 128 x 128, 128 x 192, 128 x 256, 256 x 224 and 256 x 256, with a ragged last
# row block and last column tile; the fusion and down FCs (K above 1024) run as
# summed K slices, 1088 wide also the down FC with a ragged share of chunks
@pytest.mark.parametrize("inter", [1088, 6016, 9056, 12000, 29984])
def test_tile_shapes_match_oracle(inter):
    from tests.test_gpu_kv_update_self import _run
    cfg = SELF(C.SMALL_GQA_BF16).with_(intermediate=inter, n_layers=2)
    up = make_update_rows(cfg, np.array([290, 10]), np.array([0, 3]), capacity=290, seed=13)
    _run(cfg, up, 1024, max_prefix=290)


@pytest.mark.parametrize("layers", [5, 7])
def test_cascade_rows_over_tiles_match_oracle(layers):
    """Every layer's K/V rows in one launch of 256 x 224 (5 layers) and
    256 x 256 (7) tiles."""
    from tests.test_gpu_kv_update import _run
    cfg = C.SMALL_MHA_BF16_D128.with_(n_q_heads=16, n_kv_heads=16, n_layers=layers, name="wide_kv")
    up = make_update_rows(cfg, np.array([400, 77]), np.array([0, 5]), capacity=400, seed=14)
    _run(cfg, up, 1024)


# 17 to 256 rows: one row block of 64, 96, 128 or 160 rows, 64 columns wide for
# two layers' K/V and 128 wide for seven; above 160 rows two blocks
@pytest.mark.parametrize("rows", [17, 64, 65, 96, 128, 129, 160, 161, 256])
@pytest.mark.parametrize("layers", [2, 7])
def test_few_rows_over_tiles_match_oracle(layers, rows):
    from tests.test_gpu_kv_update import _run
    cfg = C.SMALL_MHA_BF16_D128.with_(n_q_heads=16, n_kv_heads=16, n_layers=layers, name="wide_kv")
    up = make_update_rows(cfg, np.array([rows - 5, 5]), np.array([0, 40]), capacity=256, seed=rows)
    _run(cfg, up, 1024)
