"""Steps that carry their selections and their controller inside the attention's and the projection's launches, against the same steps with
both in launches of their own on the side streams (which the oracle follows elsewhere): the same arithmetic in the same order, bit for bit."""
import pytest

pytestmark = pytest.mark.gpu

# batch, heads, d, hidden, K, R, S, dtype, rescore, rope; what the second launch looks like
CASES = [
    (1, 4, 64, 256, 64, 8, 128, "f32", False, 0.0),        # fp32 tiles of 16, no splits
    (3, 5, 128, 384, 300, 7, 321, "f32", False, 0.0),      # ... rows cut into splits, merged in the tail
    (9, 16, 128, 512, 40, 3, 30, "f32", False, 0.0),       # ... tiles of 32 at the end; a cache that fills up first (steps without a projection)
    (1, 2, 64, 128, 20, 2, 10, "bf16", False, 0.0),        # the narrowest projection; fills up first
    (3, 12, 64, 768, 203, 13, 333, "bf16", True, 10000.0),  # rescoring, rows turned by a pass of their own
    (17, 12, 64, 640, 130, 9, 200, "bf16", False, 0.0),    # a ragged block of 16 sequences, more than 8 tails in front of the tiles
    (16, 8, 128, 1024, 96, 32, 300, "bf16", False, 10000.0),  # 256 narrow tiles: the tail behind them, or wider tiles
    (4, 32, 128, 4096, 128, 32, 200, "bf16", False, 0.0),  # the tail behind 256 narrow tiles, splits merged there
    (2, 8, 128, 392, 150, 5, 180, "bf16", True, 0.0),      # a width the projection's tiles do not take: launches of its own
    # sequences whose choice is made in parts of 1024 tokens: five heads, one, parts that begin within the run, the most slots and
    # tokens to rebuild, scores that are made anew, fp32, fewer candidates than ranks in a part
    (2, 5, 64, 128, 64, 8, 7164, "bf16", False, 0.0), (1, 1, 64, 128, 20, 4, 40955, "bf16", False, 0.0),
    (2, 2, 128, 256, 1024, 300, 6000, "bf16", False, 0.0), (1, 4, 64, 128, 130, 48, 5117, "bf16", True, 0.0),
    (3, 4, 64, 128, 200, 17, 6140, "f32", False, 0.0), (1, 3, 64, 128, 1000, 40, 5116, "bf16", False, 0.0),
    (2, 4, 64, 128, 300, 8, 1996, "bf16", False, 0.0),     # from one workgroup to parts within the run
]


def _of_state(state, n):
    """What a snapshot at position n defines: rows of free slots hold whatever was there."""
    free = (state["slot_pos"] < 0)[None, ..., None]
    return [state["slot_pos"], state["z"], state["cache_k"].masked_fill(free, 0), state["cache_v"].masked_fill(free, 0),
            state["scores"][:, :n].clone()]


def _run(case, carried, ordered, monkeypatch, steps, coarse=False):
    import torch
    from paper_2407_02328_amd import Adore, make_config
    B, H, d, D, K, R, S, dtype, rescore, rope = case
    monkeypatch.setenv("ADORE_STEP_STREAMS", "0" if carried else "1")
    monkeypatch.setenv("ADORE_NO_RIDE", "0" if carried else "1")
    st = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(B * 1009 + H * 31 + K)
    n = lambda shape, std, dt: torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, std, generator=g)
    f, N, dp = torch.float32, S + steps, 128
    w = {"w_kv": n((1, 2 * H * d, D), 0.05, st), "gru_w_ih": n((3 * dp, D), D ** -0.5, st), "gru_w_hh": n((3 * dp, dp), dp ** -0.5, st),
         "gru_b_ih": n((3 * dp,), 0.1, f), "gru_b_hh": n((3 * dp,), 0.1, f), "pos_w": n((dp,), 1.0, f), "pos_b": n((dp,), 0.1, f),
         "mlp_w1": n((dp, dp), dp ** -0.5, f), "mlp_b1": n((dp,), 0.1, f), "out_w": n((dp,), 4.0 * dp ** -0.5, f), "out_b": n((1,), 0.1, f)}
    a = Adore(make_config(layers=1, batch=B, heads=H, head_dim=d, hidden=D, cache_slots=K, rebuild_budget=R, max_positions=N,
                          ctrl_hidden=dp, dtype=dtype, pos_scale=2.0 ** -12, score_mode=1 if rescore else 0, rope_base=rope), w)
    a.set_input_order(ordered)
    pk, pv, hid = n((1, B, H, S, d), 1.0, st), n((1, B, H, S, d), 1.0, st), n((1, B, N, D), 1.0, st)
    qkv = n((steps, 3, B, H, d), 1.0, st)
    given = torch.rand((steps, (B + 3) // 4 * 4), device="cuda", generator=g)
    xs = hid[0][:, S:].transpose(0, 1).contiguous()
    prompt_scores = None
    if coarse:                                                         # eight values in all, the caller's own at every step
        given = (given * 8).floor() / 8
        prompt_scores = (torch.rand((B, S), device="cuda", generator=g) * 8).floor() / 8
    a.init_cache(pk, pv, hid, hid[0][:, :S].contiguous(), prompt_scores, S)
    torch.cuda.synchronize()
    a.set_timing(True)
    seen = []
    for t in range(steps):
        out = torch.empty((B, H, d), dtype=f, device="cuda")
        maps = torch.empty((B, H, K), dtype=torch.int32, device="cuda")
        ov = given[t, :B] if coarse or (not rescore and t % 3 == 2) else None     # now and then the caller's own scores
        a.decode_step(qkv[t, 0], qkv[t, 1], qkv[t, 2], hid[0], xs[t], ov, out, maps)
        seen += [out, maps]
    state = a.empty_state()
    a.get_state(**state)
    torch.cuda.synchronize()
    launches = {name: count for name, (_, count) in a.read_timing().items()}
    a.close()
    return seen + _of_state(state, S + steps), launches


@pytest.mark.parametrize("ordered", [True, False])
@pytest.mark.parametrize("case", CASES)
def test_carried_steps_are_the_steps(case, ordered, monkeypatch):
    import torch
    steps = 9
    carried, launches = _run(case, True, ordered, monkeypatch, steps)
    # what is carried is no launch of its own: the selections in every step, the controller and the merge of the splits in every step
    # with a projection (all of them but where a cache fills up first) that can carry them
    assert launches["attend"] == steps and launches["release"] == launches["rebuild_select"] == 0
    own = steps if case[3] == 392 else 0
    if case[6] >= case[4]:
        assert launches["ctrl_input"] == launches["ctrl_cell"] == own and (own or launches["attend_combine"] == 0)
    else:
        assert launches["ctrl_input"] == launches["ctrl_cell"] < steps
    apart, launches = _run(case, False, ordered, monkeypatch, steps)
    assert launches["ctrl_input"] == launches["ctrl_cell"] == launches["release"] == steps
    for i, (x, y) in enumerate(zip(carried, apart)):
        same = torch.equal(x.view(torch.int16 if x.dtype == torch.bfloat16 else torch.int32), y.view(torch.int16 if y.dtype == torch.bfloat16 else torch.int32))
        assert same, f"{case}: tensor {i} of {len(carried)}"


# Equal scores: positions decide, in the low word of the keys.  A workgroup per head with one, two and four keys a thread, a wave per head; the
# choice by all of a workgroup, by its waves, in parts, and with more ranks than four waves rank.
@pytest.mark.parametrize("case", [(2, 3, 64, 128, 150, 9, 400, "bf16", False, 0.0), (4, 32, 64, 128, 400, 32, 700, "bf16", False, 0.0),
                                  (1, 4, 128, 256, 1024, 64, 1500, "bf16", False, 0.0), (9, 16, 64, 128, 500, 17, 700, "bf16", False, 0.0),
                                  (2, 4, 64, 128, 700, 65, 1000, "bf16", False, 0.0), (2, 3, 64, 128, 1000, 40, 5000, "bf16", False, 0.0),
                                  (1, 2, 64, 128, 40, 12, 37, "f32", False, 0.0)])
def test_carried_steps_with_equal_scores(case, monkeypatch):
    import torch
    carried, launches = _run(case, True, True, monkeypatch, 7, coarse=True)
    assert launches["release"] == launches["rebuild_select"] == 0
    apart, _ = _run(case, False, True, monkeypatch, 7, coarse=True)
    for i, (x, y) in enumerate(zip(carried, apart)):
        same = torch.equal(x.view(torch.int16 if x.dtype == torch.bfloat16 else torch.int32), y.view(torch.int16 if y.dtype == torch.bfloat16 else torch.int32))
        assert same, f"{case}: tensor {i} of {len(carried)}"
