"""Which kernels, and how many splits, the entry points launch for a shape.  The calls are recorded and never run, so
the results they would compute are the concern of the parity tests."""
import pytest
import torch

pytestmark = pytest.mark.gpu
TDT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2506_20187_amd as lib
    return lib


def one_call(L, kernels_of, dtype, G, units, budget, n_ctx=16384, c_max=512, k_max=None, max_chunks=0, given=False):
    """Kernels of chunk_select_attention_decode over `units` (sequence, kv head) pairs."""
    shape = L.make_shape(units, G, 1, 128, n_ctx, c_max, k_max or c_max, L.binding.Q8Q4 if dtype == "q8q4" else TDT[dtype])
    t = torch.zeros(64, device="cuda")
    ws = torch.zeros((L.leoam_fused_workspace_bytes(shape, budget) + 15) // 16 * 16, dtype=torch.uint8, device="cuda")
    return kernels_of(lambda: L.chunk_select_attention_decode(
        shape, None if given else t, t, t, t, t, t, max_chunks, budget, 1.0, t, t, t, t, t, ws,
        qmeta=t if dtype == "q8q4" else None))


@pytest.mark.parametrize("given", [False, True], ids=["select", "given"])
@pytest.mark.parametrize("dtype,G,units,budget,splits", [
    ("bf16", 4, 128, 1024, 2), ("f16", 1, 128, 512, 2), ("bf16", 2, 96, 512, 2), ("f32", 4, 128, 512, 2),
    ("bf16", 8, 8, 256, 2), ("bf16", 8, 80, 768, 3), ("bf16", 4, 80, 1536, 3), ("bf16", 4, 40, 3072, 6),
    ("q8q4", 4, 8, 512, 2), ("q8q4", 1, 128, 2048, 2), ("q8q4", 4, 80, 2048, 3),
    # one granule or less, more than half of the compute units, more pairs than compute units
    ("bf16", 4, 8, 256, 1), ("bf16", 4, 8, 1, 1), ("bf16", 4, 129, 4096, 1), ("f32", 1, 192, 4096, 1), ("q8q4", 4, 256, 8192, 1),
    ("bf16", 4, 512, 4096, 1)])
def test_splits_fill_one_round_of_workgroups(L, kernels_of, dtype, G, units, budget, splits, given):
    (name, grid), = one_call(L, kernels_of, dtype, G, units, budget, given=given)
    assert "select_attention" in name and grid == (splits, 1, units), (name, grid)


@pytest.mark.parametrize("dtype,units,tokens,chunks", [
    # the most tokens of a step
    ("bf16", 8, 32768, 512), ("f16", 32, 8192, 128), ("bf16", 256, 1024, 12), ("f32", 32, 20480, 320), ("f32", 256, 2560, 40),
    ("bf16", 512, 256, 3), ("f32", 512, 512, 8),
    # the most tokens of a workgroup's share
    ("bf16", 86, 2400, 37), ("bf16", 129, 1200, 14), ("f16", 200, 1200, 14), ("f32", 129, 3072, 48), ("f32", 86, 6144, 96),
    ("bf16", 257, 320, 3), ("f16", 384, 320, 3), ("f32", 257, 800, 12), ("f32", 327, 800, 12), ("bf16", 769, 96, 1)])
def test_eight_heads_per_group_leave_the_one_launch_kernel_for_large_steps(L, kernels_of, dtype, units, tokens, chunks):
    """The largest budget and, without a budget, the largest chunk limit (chunks of n_ctx / c_max = 64 tokens)."""
    for budget, max_chunks, fused in ((tokens, 0, True), (tokens + 1, 0, False), (0, chunks, True), (0, chunks + 1, False)):
        names = [n for n, _ in one_call(L, kernels_of, dtype, 8, units, budget, n_ctx=65536, c_max=1024, max_chunks=max_chunks)]
        assert (len(names) == 1 and "select_attention" in names[0]) == fused, (budget, max_chunks, names)
        assert ("topk_select" in names[0]) != fused, names


@pytest.mark.parametrize("G,units,budget,max_chunks,fused", [
    # one round: uneven lists, little more than half as many as compute units
    (1, 128, 0, 512, True), (1, 129, 0, 512, False), (1, 152, 0, 16, False), (1, 152, 0, 15, True), (1, 153, 0, 512, True),
    (2, 140, 0, 32, False), (2, 140, 0, 31, True), (2, 141, 0, 512, True), (4, 129, 0, 512, True), (1, 129, 8192, 0, True),
    (1, 256, 8192, 0, True),
    # two and three rounds: few workgroups in the last
    (1, 257, 192, 0, False), (1, 257, 191, 0, True), (1, 384, 8192, 0, False), (1, 385, 8192, 0, True),
    (2, 257, 384, 0, False), (2, 257, 383, 0, True), (2, 336, 8192, 0, False), (2, 337, 8192, 0, True),
    (4, 257, 768, 0, False), (4, 257, 767, 0, True), (4, 288, 8192, 0, False), (4, 289, 8192, 0, True),
    (1, 512, 64, 0, True), (1, 513, 200, 0, False), (1, 640, 8192, 0, False), (1, 641, 97, 0, True), (1, 641, 96, 0, False),
    (2, 513, 97, 0, True), (2, 768, 96, 0, False), (4, 768, 64, 0, True),
    # more rounds: short lists
    (1, 769, 512, 0, False), (1, 769, 513, 0, True), (2, 1100, 256, 0, False), (2, 1100, 257, 0, True),
    (4, 800, 96, 0, False), (4, 800, 97, 0, True)])
def test_fp32_leaves_the_one_launch_kernel_where_it_would_wait_for_few_workgroups(L, kernels_of, G, units, budget, max_chunks, fused):
    names = [n for n, _ in one_call(L, kernels_of, "f32", G, units, budget, n_ctx=65536, c_max=1024, max_chunks=max_chunks)]
    assert (len(names) == 1 and "select_attention" in names[0]) == fused, names
    assert ("topk_select" in names[0]) != fused, names
    assert len(one_call(L, kernels_of, "f16", G, units, budget, n_ctx=65536, c_max=1024, max_chunks=max_chunks)) == 1


@pytest.mark.parametrize("dtype,G,units,m0,apart", [
    ("bf16", 4, 8, 513, True), ("bf16", 4, 8, 512, False), ("f32", 1, 8, 257, True), ("f32", 1, 8, 256, False),
    ("bf16", 8, 8, 2048, False),
    ("bf16", 4, 192, 2048, True), ("f16", 1, 193, 2048, False), ("bf16", 2, 256, 2048, False), ("bf16", 4, 320, 1024, True),
    ("bf16", 4, 512, 2048, False), ("f32", 1, 128, 512, True), ("f32", 1, 129, 512, False), ("f32", 4, 160, 513, True),
    ("f32", 4, 161, 2048, False)])
def test_tree_initial_chunks_apart_where_compute_units_are_idle(L, kernels_of, dtype, G, units, m0, apart):
    shape = L.make_shape(1, units * G, units, 128, 4 * m0, m0, m0, TDT[dtype])
    t = torch.zeros(64, device="cuda")
    ws = torch.empty(L.leoam_tree_workspace_bytes(shape, m0), dtype=torch.uint8, device="cuda")
    launched = kernels_of(lambda: L.chunk_tree_refine(shape, t, t, t, 4, 16, 1, m0, t, t, t, t, t, ws))
    assert ["tree_leaves" in n for n, _ in launched] == ([True, False] if apart else [False])
    assert "tree_refine" in launched[-1][0] and launched[-1][1] == (units, 1, 1)
