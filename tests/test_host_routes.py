"""CPU-side checks of the sizes and routes the library chooses on the host (nothing is launched, no device is touched)."""
import random

import pytest

import paper_2509_15148_amd as A
from synth import WORKLOADS, ModelConfig

MODELS = {
    "tiny": WORKLOADS["tiny"].model,
    "7b": ModelConfig(28, 3584, 28, 4, 128, 18944, 152064, "bf16"),
    "32b": ModelConfig(64, 5120, 40, 8, 128, 27648, 152064, "bf16"),
    "70b": ModelConfig(80, 8192, 64, 8, 128, 28672, 128256, "bf16"),
    "hd64": ModelConfig(2, 1024, 16, 4, 64, 2816, 32000, "bf16"),
    "odd": ModelConfig(2, 136, 4, 1, 24, 200, 515, "bf16"),
    "narrow_ffn": ModelConfig(2, 2048, 16, 16, 128, 64, 50304, "bf16"),
    "odd_vocab": ModelConfig(2, 768, 6, 6, 128, 3072, 384 * 131, "bf16"),
}


def _bytes(cfg, kind, P, K, T, n_new=1):
    return A.atts_pass_routes(cfg, kind, P, K, T, n_new).workspace_bytes


@pytest.mark.parametrize("name", MODELS)
def test_a_larger_call_never_needs_a_smaller_workspace(name):
    """A program allocates for its largest prefix, draft count and draft length and then makes smaller calls."""
    cfg, rng = MODELS[name], random.Random(name)
    for _ in range(3000):
        P, K, T = (int(2 ** rng.uniform(0, 11)) for _ in range(3))
        K = min(K, 64)
        more = [x + (rng.choice((0, 1, 7, 40, 300)) if rng.random() < 0.6 else 0) for x in (P, K, T)]
        assert _bytes(cfg, A.PASS_SCORE, *more) >= _bytes(cfg, A.PASS_SCORE, P, K, T), (P, K, T, more)
        n = rng.choice((1, 2, 33))
        assert _bytes(cfg, A.PASS_CONTINUE, *more, n + rng.choice((0, 1, 20))) >= _bytes(cfg, A.PASS_CONTINUE, P, K, T, n), (P, K, T, more)
    rows = [_bytes(cfg, A.PASS_SCORE, 512, 1, T) for T in range(1, 2600)]            # every row count: tile and split boundaries
    assert all(a <= b for a, b in zip(rows, rows[1:]))


@pytest.mark.parametrize("name", ["7b", "32b", "70b"])
def test_the_published_widths_have_room_for_every_split(name):
    """Splits are chosen by rows and shape; at these widths the room for their sums never takes slices away."""
    cfg = MODELS[name]
    for rows in list(range(1, 400)) + list(range(400, 4100, 37)):
        a, b = (A.atts_pass_routes(cfg, A.PASS_SCORE_CACHED, P, 1, rows) for P in (4, 8000))
        for product in ("qkv", "o", "down"):
            assert getattr(a, product).slices == getattr(b, product).slices, (rows, product)


def test_route_entry_points_validate_arguments():
    cfg = MODELS["7b"]
    for bad in (lambda: A.atts_pass_routes(cfg, 3, 1, 1, 1), lambda: A.atts_pass_routes(cfg, 0, 0, 1, 1),
                lambda: A.atts_pass_routes(cfg, A.PASS_CONTINUE, 1, 769, 1, 1), lambda: A.atts_pass_routes(cfg, A.PASS_CONTINUE, 1, 1, 1, 0),
                lambda: A.atts_gemm_routes(cfg.torch_dtype, 0, 1, 8)):
        with pytest.raises(A.AttsError) as e:
            bad()
        assert e.value.code == A.ERR_INVALID_ARG
    with pytest.raises(A.AttsError) as e:
        A.atts_pass_routes(ModelConfig(1, 66, 4, 2, 16, 128, 100, "bf16"), 0, 1, 1, 1)
    assert e.value.code == A.ERR_SHAPE


@pytest.mark.parametrize("rows,vocab,d,exchanged", [
    (300, 768, 4096, False), (300, 9216, 1024, True), (300, 9216, 1536, False), (600, 12288, 4096, False), (1000, 6144, 4096, False),
    (256, 2304, 768, True), (256, 3072, 4096, False), (160, 32256, 1536, True), (300, 32256, 4096, True), (385, 152064, 3584, True)])
def test_lm_head_with_few_tiles_keeps_the_faster_kernel(rows, vocab, d, exchanged):
    """More than 128 unpadded scoring rows: vocabulary entries as rows of 384 x 256 tiles where that was measured faster, and
    not where a partly filled round of them is the longer chain."""
    _, head = A.atts_gemm_routes(MODELS["7b"].torch_dtype, rows, vocab, d)
    assert (head.kernel == A.KERNEL_EXCHANGED) == exchanged


@pytest.mark.parametrize("name,rows,exchanged", [
    ("7b", 300, True), ("32b", 300, True), ("70b", 300, False),          # one row of 384 x 256 tiles in the other orientation
    ("70b", 513, True), ("70b", 600, True),                              # ... a second launch of lower tiles there
    ("7b", 1090, True), ("32b", 1025, False), ("32b", 1152, False), ("70b", 1090, False), ("70b", 1800, False), ("32b", 1800, True)])
def test_lm_head_of_padded_rows_takes_the_faster_orientation(name, rows, exchanged):
    """Each was timed in both orientations (1.2 to 17 % apart)."""
    head = A.atts_pass_routes(MODELS[name], A.PASS_SCORE, 4, 1, rows).lm_head
    assert (head.kernel == A.KERNEL_EXCHANGED) == exchanged


@pytest.mark.parametrize("rows,vocab,d,head,tail", [
    (256, 152064, 3584, 256 * 384, 256), (385, 152064, 3584, 384 * 384, 128), (800, 152064, 3584, 384 * 384, 128),
    (300, 24576, 3584, 0, 0), (4096, 152064, 3584, 0, 0), (128, 152064, 3584, 0, 0)])
def test_lm_head_second_launch(rows, vocab, d, head, tail):
    """A last round of 384 x 256 tiles that would leave most compute units idle goes to smaller tiles of the last vocabulary entries."""
    _, r = A.atts_gemm_routes(MODELS["7b"].torch_dtype, rows, vocab, d)
    assert (r.head_rows, r.tail_rows) == (head, tail)


@pytest.mark.parametrize("name,rows,product,tile,tail,seam", [
    ("7b", 776, "gate_up", 384, 256, 85 * 128), ("7b", 385, "gate_up", 256, 128, 128 * 128), ("7b", 1500, "gate_up", 384, 128, 128 * 128),
    ("7b", 4608, "gate_up", 384, 0, 0), ("70b", 4608, "down", 384, 256, 21 * 256), ("7b", 8192, "o", 256, 0, 0),
    # 384-row tiles and 128-row ones for the rest: not where the model has them only little faster
    ("7b", 700, "gate_up", 256, 0, 0), ("7b", 8192, "down", 256, 0, 0), ("70b", 1100, "gate_up", 384, 0, 0), ("70b", 4900, "o", 384, 0, 0),
    ("32b", 15800, "down", 384, 128, 18 * 256), ("70b", 4900, "down", 384, 128, 19 * 256)])
def test_last_columns_of_a_projection(name, rows, product, tile, tail, seam):
    """Whole rounds of tall tiles over the first columns, lower ones over the last, where the last round would be partly filled."""
    r = getattr(A.atts_pass_routes(MODELS[name], A.PASS_SCORE, 4, 1, rows - 4), product)
    assert (r.kernel, r.tile_rows, r.head_rows, r.tail_rows, r.head_cols) == (A.KERNEL_ALIGNED, tile, 0, tail, seam)


def test_second_launches_and_first_ones_have_work():
    """A call in two launches is cut either by rows or by columns, inside them: neither launch is empty.  Shapes around whole rounds
    of tiles, down to one column of tiles, long and short inner dimensions."""
    cut = set()
    bf16 = MODELS["7b"].torch_dtype
    for K in (768, 4096, 28672):
        for N in [256 * n for n in (1, 2, 3, 5, 8, 14, 21, 32, 55, 85, 112, 148, 257)]:
            for M in [128 * m for m in (2, 3, 4, 6, 7, 9, 12, 18, 20, 36, 64, 90, 129, 258, 600, 771, 774, 1538)]:
                for r in A.atts_gemm_routes(bf16, M, N, K):
                    assert (r.head_rows != 0) + (r.head_cols != 0) == (r.tail_rows != 0), (M, N, K)
                    assert 0 <= r.head_rows < (N if r.kernel == A.KERNEL_EXCHANGED else M) and 0 <= r.head_cols < N
                    if r.tail_rows:
                        cut.add((r.kernel, r.head_cols != 0))
    assert cut == {(A.KERNEL_ALIGNED, False), (A.KERNEL_ALIGNED, True), (A.KERNEL_EXCHANGED, False)}


@pytest.mark.parametrize("cfg,rows,rope,norm", [
    (MODELS["tiny"], 320, 1, 1), (MODELS["7b"], 320, 0, 0),
    (ModelConfig(2, 2048, 64, 16, 32, 8192, 8000, "fp32"), 16, 1, 1), (ModelConfig(2, 2048, 64, 16, 32, 8192, 8000, "fp32"), 1500, 0, 0),
    (ModelConfig(2, 512, 8, 8, 64, 1536, 4000, "fp32"), 100, 0, 1), (ModelConfig(2, 60, 5, 5, 12, 40, 100, "fp32"), 20, 0, 1)])
def test_passes_inside_small_products(cfg, rows, rope, norm):
    """fp32 passes whose products are small: rotation (heads of a power of two of at most 32 columns) and norms ride in them."""
    r = A.atts_pass_routes(cfg, A.PASS_SCORE, 4, 1, rows - 4)
    assert (r.rope_in_qkv, r.norm_in_gate_up) == (rope, norm)
    assert A.atts_pass_routes(cfg, A.PASS_CONTINUE, 4, 4, rows - 4).norm_in_gate_up == 0


@pytest.mark.parametrize("dtype,shape,small", [
    ("fp32", (1024, 2048, 256), True), ("fp32", (2000, 1000, 1024), False), ("fp32", (1000, 1900, 2048), True), ("fp32", (300, 12000, 2048), False),
    ("fp32", (129, 16600, 8192), True), ("fp32", (260, 11000, 512), True), ("fp32", (260, 11000, 2048), False),
    ("bf16", (17, 33000, 2048), True), ("bf16", (17, 33000, 8192), False), ("bf16", (17, 49000, 8192), True), ("bf16", (33, 24000, 2048), False),
    ("fp32", (1 << 30, 32, 8), False)])
def test_products_of_few_tiles(dtype, shape, small):
    gemm, _ = A.atts_gemm_routes({"fp32": MODELS["tiny"], "bf16": MODELS["7b"]}[dtype].torch_dtype, *shape)
    assert (gemm.kernel == A.KERNEL_SMALL) == small


@pytest.mark.parametrize("shape,small", [((2000, 1000, 2048), True), ((300, 12000, 2048), True), ((300, 12000, 8192), False), ((260, 11000, 8192), True),
                                         ((1024, 2080, 512), False)])
def test_fp32_lm_head_of_few_tiles(shape, small):
    """Its 32 x 64 tiles stay ahead of the general kernel for longer than the plain product's 32 x 32."""
    _, head = A.atts_gemm_routes(MODELS["tiny"].torch_dtype, *shape)
    assert (head.kernel == A.KERNEL_SMALL) == small
