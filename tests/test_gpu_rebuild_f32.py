"""The fp32 projections (rebuilt K/V rows, input projection of a prompt) against 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# fewer rows than a tile and whole tiles (16x16), a row length that ends inside a step of 16, more k than one trip of the four
# waves; from 256 tiles of 32x32 on: whole ones and a last one of 1 row
@pytest.mark.parametrize("batch,heads,d,D,R", [(1, 2, 64, 64, 1), (1, 2, 64, 72, 16), (3, 2, 128, 136, 11), (2, 4, 64, 520, 8),
                                               (4, 16, 64, 1024, 40), (3, 32, 64, 264, 43), (1, 1, 64, 8, 3)])
def test_rebuilt_rows(batch, heads, d, D, R):
    from paper_2407_02328_amd import Adore, make_config
    g = torch.Generator().manual_seed(batch * 1000 + D)

    def normal(shape, std):
        return (torch.randn(shape, generator=g) * std).cuda()
    DP, K, S = 16, R + 9, 2 * R + 20
    n_max = S + 4
    w = {"w_kv": normal((1, 2 * heads * d, D), D ** -0.5), "gru_w_ih": normal((3 * DP, D), D ** -0.5),
         "gru_w_hh": normal((3 * DP, DP), DP ** -0.5), "gru_b_ih": normal((3 * DP,), 0.1), "gru_b_hh": normal((3 * DP,), 0.1),
         "pos_w": normal((DP,), 1.0), "pos_b": normal((DP,), 0.1), "mlp_w1": normal((DP, DP), DP ** -0.5),
         "mlp_b1": normal((DP,), 0.1), "out_w": normal((DP,), 0.3), "out_b": normal((1,), 0.1)}
    job = Adore(make_config(layers=1, batch=batch, heads=heads, head_dim=d, hidden=D, cache_slots=K, rebuild_budget=R,
                            max_positions=n_max, ctrl_hidden=DP, dtype="f32", pos_scale=2.0 ** -12), w, "cuda")
    hidden = normal((1, batch, n_max, D), 1.0)
    kv = normal((1, batch, heads, S, d), 1.0)
    job.init_cache(kv, kv, hidden, hidden[0, :, :S].contiguous(), None, S)
    slots = torch.empty((batch, heads, K), dtype=torch.int32, device="cuda")
    ck, cv = (torch.empty((1, batch, heads, K, d), device="cuda") for _ in range(2))
    job.get_state(slot_pos=slots, cache_k=ck, cache_v=cv)
    torch.cuda.synchronize()
    m = K - R - 1                                          # the residents' slots come first, then the R rebuilt tokens'
    pos = slots[:, 0, m:m + R].cpu().long()
    assert (pos >= 0).all() and (slots[:, :, m:m + R] == slots[:, :1, m:m + R]).all()
    x = hidden[0].cpu().double().gather(1, pos[:, :, None].expand(-1, -1, D))
    wkv = w["w_kv"][0].cpu().double()
    shape = (batch, R, 2, heads, d)
    want, size = (x @ wkv.t()).view(shape), (x.abs() @ wkv.abs().t()).view(shape)
    got = torch.stack([c[0, :, :, m:m + R].cpu().double() for c in (ck, cv)]).permute(1, 3, 0, 2, 4)   # [b][rank][K, V][h][d]
    # eight products and their sum in fp32, rounded at most 16 times, then 64 bits and one rounding
    n = 17
    err = (got - want).abs()
    print(f"B{batch} H{heads} d{d} D{D} R{R}: relative error {float((got - want).norm() / want.norm()):.2e}", flush=True)
    assert (err <= n * 2.0 ** -24 * size).all()
    job.close()


# just below and above the least number of tokens for the tiles, one chunk and two
@pytest.mark.parametrize("batch,S,D", [(1, 15, 200), (1, 16, 200), (3, 33, 264), (2, 520, 1024)])
def test_controller_over_an_fp32_prompt(batch, S, D):
    from paper_2407_02328_amd import Adore, make_config
    from tests.test_gpu_controller import _reference
    g = torch.Generator().manual_seed(S + D)
    DP, H, d = 128, 2, 64

    def normal(shape, std):
        return (torch.randn(shape, generator=g) * std).cuda()
    w = {"w_kv": normal((1, 2 * H * d, D), 0.02), "gru_w_ih": normal((3 * DP, D), D ** -0.5),
         "gru_w_hh": normal((3 * DP, DP), DP ** -0.5), "gru_b_ih": normal((3 * DP,), 0.1), "gru_b_hh": normal((3 * DP,), 0.1),
         "pos_w": normal((DP,), 1.0), "pos_b": normal((DP,), 0.1), "mlp_w1": normal((DP, DP), DP ** -0.5),
         "mlp_b1": normal((DP,), 0.1), "out_w": normal((DP,), 0.3), "out_b": normal((1,), 0.1)}
    pos_scale = 2.0 ** -12
    job = Adore(make_config(layers=1, batch=batch, heads=H, head_dim=d, hidden=D, cache_slots=24, rebuild_budget=3,
                            max_positions=S + 4, ctrl_hidden=DP, dtype="f32", pos_scale=pos_scale), w, "cuda")
    hidden = normal((1, batch, S + 4, D), 1.0)
    kv = normal((1, batch, H, S, d), 1.0)
    x = hidden[0, :, :S].contiguous()
    scores, z = torch.zeros((batch, S + 4), device="cuda"), torch.zeros((batch, DP), device="cuda")
    job.init_cache(kv, kv, hidden, x, None, S)
    job.get_state(scores=scores, z=z)
    torch.cuda.synchronize()
    want_scores, want_z = _reference(w, x, pos_scale)
    print(f"B{batch} S{S} D{D}: error of z {float((z.cpu().double() - want_z).norm() / want_z.norm()):.2e}", flush=True)
    # as for bf16 weights: a pre-activation is a sum of D + 128 fp32 products of order one, and |z| <= 1
    assert (z.cpu().double() - want_z).abs().max() <= 4e-6
    assert (scores[:, :S].cpu().double() - want_scores).abs().max() <= 4e-6
    job.close()


# decode steps of many sequences: the plain projection and the tiles on either side of the line between them (16 tokens, and
# 24 * D outputs), a ragged last tile
@pytest.mark.parametrize("batch,D", [(15, 256), (16, 256), (16, 264), (63, 1024), (64, 1024), (17, 2048), (131, 2080)])
def test_controller_over_fp32_steps(batch, D):
    from paper_2407_02328_amd import Adore, make_config
    from tests.test_gpu_controller import _reference
    g = torch.Generator().manual_seed(batch + D)
    DP, H, d, K, S, T = 128, 1, 64, 8, 5, 4

    def normal(shape, std):
        return (torch.randn(shape, generator=g) * std).cuda()
    w = {"w_kv": normal((1, 2 * H * d, D), 0.02), "gru_w_ih": normal((3 * DP, D), D ** -0.5),
         "gru_w_hh": normal((3 * DP, DP), DP ** -0.5), "gru_b_ih": normal((3 * DP,), 0.1), "gru_b_hh": normal((3 * DP,), 0.1),
         "pos_w": normal((DP,), 1.0), "pos_b": normal((DP,), 0.1), "mlp_w1": normal((DP, DP), DP ** -0.5),
         "mlp_b1": normal((DP,), 0.1), "out_w": normal((DP,), 0.3), "out_b": normal((1,), 0.1)}
    pos_scale = 2.0 ** -12
    job = Adore(make_config(layers=1, batch=batch, heads=H, head_dim=d, hidden=D, cache_slots=K, rebuild_budget=2,
                            max_positions=S + T, ctrl_hidden=DP, dtype="f32", pos_scale=pos_scale), w, "cuda")
    hidden, kv, out = normal((1, batch, S + T, D), 1.0), normal((1, batch, H, S, d), 1.0), normal((batch, H, d), 1.0)
    qkv = [normal((T, batch, H, d), 1.0) for _ in range(3)]
    scores, z = torch.zeros((batch, S + T), device="cuda"), torch.zeros((batch, DP), device="cuda")
    job.init_cache(kv, kv, hidden, hidden[0, :, :S].contiguous(), None, S)
    for t in range(T):
        job.decode_step(*(a[t] for a in qkv), hidden[0], hidden[0, :, S + t].contiguous(), None, out, None)
    job.get_state(scores=scores, z=z)
    torch.cuda.synchronize()
    want_scores, want_z = _reference(w, hidden[0], pos_scale)
    # as over a prompt
    assert (z.cpu().double() - want_z).abs().max() <= 4e-6
    assert (scores.cpu().double() - want_scores).abs().max() <= 4e-6
    job.close()
