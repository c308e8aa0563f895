"""GPU parity of the forward under every shard-step grouping (tsp_shape.group_steps):
one step per launch, groups that divide D, groups that leave a smaller last group, and
more shards than one group holds.  Whatever the grouping, the result is the sum of
Algorithm 1's and Algorithm 2's shard terms in schedule order, so each run is checked
element by element against the fp64 oracle at the usual tolerance, and the groupings
against each other (they differ only in fp32 summation order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2604_26294_amd import inputs as I  # noqa: E402
from paper_2604_26294_amd import tsp as T  # noqa: E402
from paper_2604_26294_amd.harness import RankProblem, local_rows, to_device_bf16  # noqa: E402
from tests.gpu_common import (DEG12, DEG16, MID_GQA64, MID_MHA128, ODD3, SUBL,  # noqa: E402
                              WIDE, assert_close, gen, oracle_blocks)

# (workload, rank, group_steps values); 0 is the library default, min(D, 8)
CASES = [(MID_GQA64, 3, (1, 2, 3)), (MID_GQA64.with_layout(1), 1, (1, 3)),
         (ODD3, 2, (1, 2)), (ODD3.with_layout(1), 0, (2,)), (MID_MHA128, 1, (1,)),
         (DEG16, 13, (0, 5)), (DEG16.with_layout(1), 6, (0,))]
_IDS = [f"{w.name}-{w.layout_name}-r{p}" for w, p, _ in CASES]
_cache = {}


def _inputs(wl):
    if wl.name not in _cache:
        _cache[wl.name] = gen(wl)
    return _cache[wl.name]


@pytest.mark.parametrize("wl,p,groups", CASES, ids=_IDS)
@pytest.mark.parametrize("block", ["mlp", "attn", "layer"])
def test_grouping_parity(wl, p, groups, block):
    x_bits, w_bits = _inputs(wl)
    ref = oracle_blocks(wl, x_bits, w_bits, p, blocks=(block,))[block]
    outs = {}
    for g in groups:
        print(f"[grouping] {wl.name} {wl.layout_name} rank {p} {block} group_steps={g}",
              flush=True)
        prob = RankProblem(wl, x_bits, w_bits, p, group_steps=g)
        prob.prefill_kv()
        y = {"mlp": prob.mlp, "attn": prob.attn_fwd, "layer": prob.layer}[block]()
        torch.cuda.synchronize()
        outs[g] = y.double().cpu().numpy()
        assert_close(outs[g], ref, f"{wl.name} r{p} {block} G={g}")
    # every grouping against the default one (all steps together where D <= 8)
    prob = RankProblem(wl, x_bits, w_bits, p)
    prob.prefill_kv()
    base = {"mlp": prob.mlp, "attn": prob.attn_fwd, "layer": prob.layer}[block]()
    torch.cuda.synchronize()
    base = base.double().cpu().numpy()
    scale = np.max(np.abs(base))
    for g, y in outs.items():
        assert np.max(np.abs(y - base)) <= 1e-2 * scale, f"G={g} vs default"


@pytest.mark.parametrize("wl,p", [(SUBL, 2), (SUBL.with_layout(1), 1)],
                         ids=["paired-contiguous-r2", "paired-zigzag-r1"])
@pytest.mark.parametrize("block", ["attn", "layer"])
def test_attention_with_paired_query_tiles(wl, p, block):
    """A group's attention with two query tiles per workgroup (the i-th most and the i-th
    fewest keys), as the launch plan takes it for shapes with many work items per shard;
    launches over part of a group's shards (heads' columns inside group-wide Q and A rows)
    are covered at full size (7B S=65536, 70B: 4 of 8 shards per launch)."""
    print(f"[grouping] {wl.name} {wl.layout_name} rank {p} {block}", flush=True)
    x_bits, w_bits = _inputs(wl)
    prob = RankProblem(wl, x_bits, w_bits, p)
    prob.prefill_kv()
    y = {"attn": prob.attn_fwd, "layer": prob.layer}[block]()
    torch.cuda.synchronize()
    ref = oracle_blocks(wl, x_bits, w_bits, p, blocks=(block,))[block]
    assert_close(y.double().cpu().numpy(), ref, f"{wl.name} r{p} {block}")


@pytest.mark.parametrize("wl,p", [(WIDE, 2), (WIDE.with_layout(1), 1)],
                         ids=["contiguous-r2", "zigzag-r1"])
def test_paired_launch_over_more_shards_than_fill_the_gpu(wl, p):
    """One paired launch over all four shards where two already fill every CU, because its
    rounds waste less of the last one; against the oracle, and every shard for itself."""
    print(f"[grouping] {wl.name} {wl.layout_name} rank {p}", flush=True)
    x_bits, w_bits = _inputs(wl)
    outs = []
    for steps in (0, 1):
        prob = RankProblem(wl, x_bits, w_bits, p, group_steps=steps)
        prob.prefill_kv()
        T.tsp_profile_enable(True)
        try:
            y = prob.attn_fwd()
            torch.cuda.synchronize()
            launches = T.tsp_profile_read(T.KERNELS.index("attn"))[1]
        finally:
            T.tsp_profile_enable(False)
        assert launches == (4 if steps else 1)
        outs.append(y.double().cpu().numpy())
    assert_close(outs[0], oracle_blocks(wl, x_bits, w_bits, p, blocks=("attn",))["attn"],
                 f"{wl.name} r{p}")
    assert np.max(np.abs(outs[0] - outs[1])) <= 1e-2 * np.max(np.abs(outs[1]))


@pytest.mark.parametrize("wl,p,steps", [(MID_GQA64, 2, 1), (MID_MHA128.with_layout(1), 0, 1),
                                        (ODD3, 2, 2), (DEG12, 7, 1), (DEG12, 7, 5)],
                         ids=["gqa64-1", "mha128-zigzag-1", "odd3-2", "deg12-1", "deg12-5"])
def test_backward_in_the_smallest_workspace(wl, p, steps):
    """Every backward call in the smallest workspace that group_steps allows (one shard at a
    time without partial sums, groups that leave a smaller last one) gives the gradients of the
    default groups, which the oracle checks elsewhere, and writes nothing past it."""
    print(f"[bounded bwd] {wl.name} {wl.layout_name} rank {p} group_steps={steps}", flush=True)
    x_bits, w_bits = _inputs(wl)
    dy = to_device_bf16(local_rows(I.make_dy_full(wl), wl, p))
    dkl, dvl = (to_device_bf16(t) for t in I.make_dkv_own(wl, p))
    outs = []
    for g in (0, steps):
        prob = RankProblem(wl, x_bits, w_bits, p, group_steps=g)
        prob.prefill_kv()
        prob.attn_fwd_train()
        calls = {"mlp": (T.OP_MLP_BWD, "ws_bwd", lambda: prob.mlp_bwd(dy)),
                 "attn": (T.OP_ATTN_BWD, "ws_abwd", lambda: prob.attn_bwd(dy)),
                 "saved": (T.OP_ATTN_BWD, "ws_abwd", lambda: prob.attn_bwd_saved(dy)),
                 "kv": (T.OP_ATTN_KV_BWD, "ws_abwd", lambda: prob.attn_kv_bwd(dkl, dvl, False))}
        got = {}
        for name, (op, buf, call) in calls.items():
            call()  # allocates the gradients and a full workspace
            if g:
                n = T.workspace_bytes(prob.shape, op | T.WS_MIN)
                assert n < T.workspace_bytes(prob.shape, op)
                held = torch.full((n + 4096,), 255, dtype=torch.uint8, device="cuda")
                setattr(prob, buf, held[:n])
            flat = [t for o in call() for t in (o if isinstance(o, list) else [o])]
            got[name] = [t.double().cpu().numpy() for t in flat]
            if g:
                assert bool((held[n:] == 255).all()), f"{name} past the workspace"
        outs.append(got)
    for name, ref in outs[0].items():
        for a, b in zip(outs[1][name], ref):
            assert_close(a, b, f"{wl.name} r{p} {name} G={steps}")


@pytest.mark.parametrize("wl,p", [(MID_GQA64, 2), (DEG12, 7)], ids=["one-group", "two-groups"])
def test_shards_that_share_a_gradient_buffer(wl, p):
    """One weight-gradient buffer given for every shard: with accumulate it ends as the sum of
    the shards' gradients, without as the last shard's in the schedule's order (the products of
    a launch run at the same time, so these go in launches of their own).  Same products as with
    a buffer each, so only the fp32 order of the running sums differs."""
    print(f"[shared dw] {wl.name} rank {p}", flush=True)
    x_bits, w_bits = _inputs(wl)
    prob = RankProblem(wl, x_bits, w_bits, p)
    prob.prefill_kv(include_self=True)
    dy = to_device_bf16(local_rows(I.make_dy_full(wl), wl, p))
    dkl, dvl = (to_device_bf16(t) for t in I.make_dkv_own(wl, p))
    calls = {"mlp": lambda acc: prob.mlp_bwd(dy, acc), "attn": lambda acc: prob.attn_bwd(dy, acc),
             "kv": lambda acc: prob.attn_kv_bwd(dkl, dvl, acc)}
    prob.mlp_bwd(dy), prob.attn_bwd(dy)  # (allocate the gradient buffers)
    own = {"dw": [list(t) for t in prob.dw], "adw": list(prob.adw)}
    for name, call in calls.items():
        prob.dw, prob.adw = own["dw"], own["adw"]
        for t in prob.adw + [t for ts in prob.dw for t in ts]:
            t.zero_()
        call(False)
        each = [list(ts) for ts in prob.dw] if name == "mlp" else [prob.adw]
        each = [[t.double() for t in ts] for ts in each]
        last = (p + 1) % wl.degree if name == "mlp" else wl.degree - 1  # of ring step D - 1
        for acc in (True, False):
            prob.dw = [[torch.zeros_like(ts[0])] * wl.degree for ts in own["dw"]]
            prob.adw = [torch.zeros_like(own["adw"][0])] * wl.degree
            call(acc)
            shared = [ts[0] for ts in prob.dw] if name == "mlp" else [prob.adw[0]]
            for got, ts in zip(shared, each):
                ref = sum(ts) if acc else ts[last]
                assert torch.allclose(got.double(), ref, rtol=1e-5, atol=1e-6 * ref.abs().max().item())
