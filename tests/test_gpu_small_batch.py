"""The FFN's split kernels (batches of at most 64 tokens): tile edges of the
tokens, contractions shorter than the wavefronts' shares, slots of several
passes, kept sets that the caller brings."""
import numpy as np
import pytest

import workloads as W
from oracle import carith, method
from test_gpu_parity import Y_TOL, check_plan, gu, run_case  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("B", [1, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65])
@pytest.mark.parametrize("d,E,K,I,ns,budget", [
    (256, 8, 2, 64, 0, 3),       # eight k-steps of d, two of I: most shares of I empty
    (768, 24, 5, 192, 2, 9),     # shares of unequal length, shared experts
    (2048, 16, 4, 1408, 1, 16),  # several rounds of k-steps per share
])
def test_token_tiles(gu, B, d, E, K, I, ns, budget):  # noqa: F811
    inp = W.custom_layer(d, E, K, I, B, seed=700 + B, n_shared=ns, shared_gate=ns == 2)
    run_case(gu, inp, budget, flags=1, with_residual=True)


def _forward(gu, inp, logits, ids, sel, n_sel, slot, budget, flags):  # noqa: F811
    """base_moe_forward on a given plan against the oracle."""
    from paper_2609_36222_amd import binding as bd
    sh, B = inp["shape"], inp["x"].shape[0]
    ex, n_ex = method.backfill(logits, ids, slot, n_sel, sh.K, flags)
    gates = method.gates_c(logits, ids, ex, n_ex, 1, flags)
    offsets, pair_tok, pair_gate, pair_of = method.compact(ex, n_ex, slot, gates, budget)
    y_ref = method.moe_restricted64(inp["x"], ex, n_ex, gates,
                                    method.Experts(inp["w13"], inp["w2"], sh.bf16))
    for packed in (False, True) if sh.bf16 else (False,):
        gl = gu.GpuLayer(inp, packed=packed)
        ws, y = gl.workspace(B, budget), gl.y_like(B)

        def i32(a):
            return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()

        plan = bd.base_moe_forward(gl.desc, gl.x(inp["x"]), B, gu.dev_f32(logits), i32(ids),
                                   i32(sel), i32([n_sel]), i32(slot), budget, flags, None, y, ws)
        torch.cuda.synchronize()
        got = gu.plan_arrays(plan, ws, B, sh.K, sh.E, budget, full=False)
        check_plan(got, dict(exec_ids=ex, exec_gates=gates, offsets=offsets, pair_tok=pair_tok,
                             pair_gate=pair_gate, pair_of=pair_of))
        err = np.max(np.abs(gu.to_np_f32(y).astype(np.float64) - y_ref))
        assert err <= Y_TOL[sh.bf16], err
    return offsets


@pytest.mark.parametrize("B", [16, 29, 60])
def test_slot_of_several_passes(gu, B):  # noqa: F811
    """Routes that name one expert up to four times, executed as they are
    (drop): a slot then holds more pairs than one pass's token tiles."""
    inp = W.custom_layer(512, 12, 4, 128, B, seed=41)
    logits, ids, _ = carith.route(inp["x"], inp["w_router"], inp["b_router"], 4, 1)
    ids = ids.copy()
    ids[:, :] = 3
    ids[::5, 1] = 7
    slot = np.full(12, -1, np.int32)
    slot[[3, 7]] = [1, 0]
    offsets = _forward(gu, inp, logits, ids, np.array([7, 3]), 2, slot, 2, 2)
    assert offsets[2] - offsets[1] > 16 * (1 if B <= 16 else 2 if B <= 32 else 4)


def test_kept_set_beyond_the_routes(gu):  # noqa: F811
    """A kept set of the caller's own, larger than the batch has routes: the
    token's experts may sit in any slot."""
    inp = W.custom_layer(256, 40, 2, 128, 1, seed=42)
    logits, ids, _ = carith.route(inp["x"], inp["w_router"], inp["b_router"], 2, 1)
    sel = np.setdiff1d(np.arange(40)[::-1], ids[0][:1])[::-1][:30]
    slot = np.full(40, -1, np.int32)
    slot[sel] = np.arange(30)
    _forward(gu, inp, logits, ids, sel, 30, slot, 30, 0)


@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 8, 9, 33])
@pytest.mark.parametrize("d,I", [(256, 64), (768, 320), (1280, 1088)])
def test_fp32_rows(gu, B, d, I):  # noqa: F811
    """fp32 layers: token batches of 1, 2, 4 and 8 and their remainders, a row of
    I shorter than a wavefront's pass and ones with a remainder."""
    run_case(gu, W.custom_layer(d, 6, 3, I, B, bf16=False, seed=80 + B), 4, flags=2)


@pytest.mark.parametrize("B", [1, 2, 4])
def test_fp32_slot_of_several_passes(gu, B):  # noqa: F811
    """Routes that name one expert three times (drop): a slot then holds more
    pairs than the batch has tokens."""
    inp = W.custom_layer(512, 12, 4, 128, B, bf16=False, seed=43)
    logits, ids, _ = carith.route(inp["x"], inp["w_router"], inp["b_router"], 4, 1)
    ids = np.full_like(ids, 3)
    ids[:, 1] = 7
    slot = np.full(12, -1, np.int32)
    slot[[3, 7]] = [1, 0]
    offsets = _forward(gu, inp, logits, ids, np.array([7, 3]), 2, slot, 2, 2)
    assert offsets[2] - offsets[1] == 3 * B


@pytest.mark.parametrize("B", [1, 4, 5, 16, 17, 63, 64, 65])
@pytest.mark.parametrize("d,E,bf16,sg", [(256, 3, True, 1), (768, 37, False, 0), (1024, 256, True, 0),
                                         (1280, 6, True, 1), (2304, 8, True, 1)])
def test_small_scores(gu, B, d, E, bf16, sg):  # noqa: F811
    _small_scores(gu, B, d, E, bf16, sg)


@pytest.mark.parametrize("B,E", [(81, 100), (82, 100), (100, 64), (128, 64), (129, 64), (1000, 8),
                                 (300, 3)])
def test_small_scores_of_many_tokens(gu, B, E):  # noqa: F811
    """More token groups than dies: every row of a group on its own die."""
    _small_scores(gu, B, 512, E, True, 1)


@pytest.mark.parametrize("B,d,E", [(8, 256, 129), (8, 768, 129), (8, 512, 128), (9, 512, 128),
                                   (9, 768, 128), (9, 768, 129)])
def test_scores_lines(gu, B, d, E):  # noqa: F811
    """Either side of the lines between the scoring kernels, with the
    predictor's rows in the same launch and without; a gate alone."""
    _small_scores(gu, B, d, E, True, 1)
    _small_scores(gu, B, d, E, False, 0)


def _small_scores(gu, B, d, E, bf16, sg):  # noqa: F811
    """Router, predictor and extra rows in one launch: token and row
    remainders, chunks of the contraction that do not fill a pass."""
    inp = W.custom_layer(d, E, min(E, 5), 64, B, bf16=bf16, seed=98, n_shared=sg,
                         shared_gate=bool(sg), zero_token=True)
    run_case(gu, inp, max(1, E // 2))


@pytest.mark.parametrize("B", [1, 32, 33, 64])
@pytest.mark.parametrize("E,K,rule,flags", [(40, 3, 1, 0), (65, 16, 0, 3), (256, 16, 4, 1),
                                            (130, 9, 2, 2)])
def test_one_launch_plan(gu, B, E, K, rule, flags):  # noqa: F811
    """Selection, backfill and compaction in one launch: every plan array
    against the oracle and the staged calls, over the chunk widths of the
    experts and the tokens, ties of the binary rule, all the gate and fill
    flags."""
    inp = W.custom_layer(256, E, K, 64, B, seed=95 + K, n_shared=K % 2)
    run_case(gu, inp, max(1, E // 3), flags=flags, score_rule=rule, norm_topk=K % 2)
    run_case(gu, inp, E, flags=flags, score_rule=rule, norm_topk=K % 2)


def test_long_contraction(gu):  # noqa: F811
    """A long contraction of I: the split kernels' bound, and down's row
    groups of two, four and eight tiles."""
    for B in (32, 33, 120, 400):
        run_case(gu, W.custom_layer(256, 5, 2, 2112, B, seed=97), 3)
    run_case(gu, W.custom_layer(2048, 4, 2, 2112, 70, seed=97), 2)


def test_full_slots_either_side_of_the_line(gu):  # noqa: F811
    """Every slot full of pairs: the split kernels, their plan in one launch, up
    to (pairs - 16 slots) d I = 1.8e9, beyond it the unit kernels; every plan
    array against the oracle, staged equal to fused and packed to row-major."""
    from paper_2609_36222_amd import binding as bd
    inp = W.custom_layer(2048, 12, 12, 1024, 64, seed=44, n_shared=6)
    for B, compacts in ((60, False), (64, True)):
        part = dict(inp, x=inp["x"][:B])
        desc = gu.GpuLayer(part).desc
        assert ("compact" in bd.layer_stages(desc, B, 12)) == compacts
        run_case(gu, part, 12)


@pytest.mark.parametrize("B", [511, 513, 600])
def test_selection_workgroups(gu, B):  # noqa: F811
    """Where the fused selection takes more tokens per workgroup."""
    run_case(gu, W.custom_layer(256, 24, 3, 64, B, seed=90), 7)


@pytest.mark.parametrize("B", [3, 130])
def test_graph_replay_either_side_of_the_line(gu, B):  # noqa: F811
    """A captured layer on the small batches' launches and on the general
    ones: replays on new tokens, over a workspace of junk, equal eager calls
    bit for bit."""
    from paper_2609_36222_amd import binding as bd
    inp = W.custom_layer(512, 32, 4, 128, B, seed=99, n_shared=1, shared_gate=True)
    gl = gu.GpuLayer(inp, packed=True)
    xs = [gl.x(W.decode_tokens(inp["shape"], 0, data_seed=s)) for s in range(3)]
    x, ws, y = xs[0].clone(), gl.workspace(B, 9), gl.y_like(B)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        bd.base_decode_layer(gl.desc, x, B, 9, 0, None, y, ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bd.base_decode_layer(gl.desc, x, B, 9, 0, None, y, ws)
    for rep in range(5):
        xk, ws_e, y_e = xs[rep % 3], gl.workspace(B, 9), gl.y_like(B)
        bd.base_decode_layer(gl.desc, xk, B, 9, 0, None, y_e, ws_e)
        x.copy_(xk)
        ws.fill_(0xA5)
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(gu.to_np_f32(y), gu.to_np_f32(y_e)), rep
