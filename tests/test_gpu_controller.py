"""The controller over a prompt against the same recurrence in 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _reference(w, x, pos_scale):
    DP = w["gru_w_hh"].shape[1]
    f = {k: v.double().cpu() for k, v in w.items()}
    x = x.double().cpu()
    gi = x @ f["gru_w_ih"].t() + f["gru_b_ih"]
    h = torch.zeros(x.shape[0], DP, dtype=torch.float64)
    scores = []
    for t in range(x.shape[1]):
        g, gh = gi[:, t], h @ f["gru_w_hh"].t() + f["gru_b_hh"]
        r = torch.sigmoid(g[:, :DP] + gh[:, :DP])
        u = torch.sigmoid(g[:, DP:2 * DP] + gh[:, DP:2 * DP])
        h = (1 - u) * torch.tanh(g[:, 2 * DP:] + r * gh[:, 2 * DP:]) + u * h
        p = f["pos_w"] * (t * pos_scale) + f["pos_b"]
        scores.append(torch.sigmoid(torch.tanh((p + h) @ f["mlp_w1"].t() + f["mlp_b1"]) @ f["out_w"] + f["out_b"]))
    return torch.stack(scores, 1), h


# one token (the step's kernels), around the read-ahead of 8 tokens and the staged blocks of 16 (few tokens: sliced
# projection), more than 256 tokens (whole projection), across two chunks of 512; the last without a sliced projection's widths
@pytest.mark.parametrize("batch,S,D", [(2, 1, 512), (1, 2, 512), (3, 7, 512), (2, 8, 512), (2, 9, 512), (1, 16, 512), (2, 17, 512),
                                       (1, 33, 1024), (2, 129, 512), (3, 263, 384), (1, 515, 512), (2, 1100, 256), (2, 40, 200),
                                       (1, 300, 200), (2, 1025, 256), (1, 2100, 128)])
def test_scores_and_state_after_a_prompt(batch, S, D):
    _check_prompt(batch, S, D, 128)


# the general cell kernel, one chunk and several
@pytest.mark.parametrize("batch,S,D,DP", [(2, 9, 256, 64), (1, 600, 128, 64), (2, 1030, 64, 20)])
def test_scores_and_state_after_a_prompt_other_controller_widths(batch, S, D, DP):
    _check_prompt(batch, S, D, DP)


def _prompt(batch, S, D, DP, H=2, K=24, change=None, change_x=None):
    """An init behind random prompts; change(w) and change_x(x) may alter weights and prompts.  -> weights, prompts, scores, z, position scale"""
    from paper_2407_02328_amd import Adore, make_config
    g = torch.Generator().manual_seed(1000 * S + D)

    def normal(shape, std, dtype):
        return (torch.randn(shape, generator=g) * std).to(dtype).cuda()
    d, R, n_max = 64, 3, S + 4
    bf, f32 = torch.bfloat16, torch.float32
    w = {"w_kv": normal((1, 2 * H * d, D), 0.02, bf), "gru_w_ih": normal((3 * DP, D), D ** -0.5, bf),
         "gru_w_hh": normal((3 * DP, DP), DP ** -0.5, bf), "gru_b_ih": normal((3 * DP,), 0.1, f32),
         "gru_b_hh": normal((3 * DP,), 0.1, f32), "pos_w": normal((DP,), 1.0, f32), "pos_b": normal((DP,), 0.1, f32),
         "mlp_w1": normal((DP, DP), DP ** -0.5, f32), "mlp_b1": normal((DP,), 0.1, f32), "out_w": normal((DP,), 0.3, f32),
         "out_b": normal((1,), 0.1, f32)}
    if change:
        change(w)
    pos_scale = 2.0 ** -12
    job = Adore(make_config(layers=1, batch=batch, heads=H, head_dim=d, hidden=D, cache_slots=K, rebuild_budget=R,
                            max_positions=n_max, ctrl_hidden=DP, dtype="bf16", pos_scale=pos_scale), w, "cuda")
    x = normal((batch, S, D), 1.0, bf)
    if change_x:
        change_x(x)
    hidden = torch.zeros((1, batch, n_max, D), dtype=bf, device="cuda")
    hidden[0, :, :S] = x
    kv = normal((1, batch, H, S, d), 1.0, bf)
    scores = torch.zeros((batch, n_max), device="cuda")
    z = torch.zeros((batch, DP), device="cuda")
    job.init_cache(kv, kv, hidden, x.contiguous(), None, S)
    job.get_state(scores=scores, z=z)
    torch.cuda.synchronize()
    job.close()
    return w, x, scores[:, :S].cpu(), z.cpu(), pos_scale


def _check_prompt(batch, S, D, DP, H=2, K=24, change=None):
    w, x, scores, z, pos_scale = _prompt(batch, S, D, DP, H, K, change)
    want_scores, want_z = _reference(w, x, pos_scale)
    # |z| <= 1; a pre-activation is a sum of D + 128 fp32 products of order one (error about 2^-24 sqrt(D) < 2e-6), the gates
    # damp what earlier tokens bring along, and the scores are as smooth: 4e-6 leaves a factor of two
    assert (z.double() - want_z).abs().max() <= 4e-6
    assert (scores.double() - want_scores).abs().max() <= 4e-6


def _opened(by):
    """Update gates opened by so much: a state keeps more of itself from one token to the next."""
    def change(w):
        w["gru_b_ih"][128:256] += by
    return change


def _slow_units(w):
    """A few units that hardly forget and take in next to nothing."""
    w["gru_b_ih"][128:136] += 11.5
    w["gru_w_ih"][256:264] *= 1e-4
    w["gru_w_hh"][256:264] *= 1e-4
    for name in ("gru_b_ih", "gru_b_hh"):
        w[name][256:264] *= 1e-4


def _small_states(w):
    w["gru_w_ih"][256:] *= 2e-5
    for name in ("gru_b_ih", "gru_b_hh"):
        w[name][256:] *= 2e-5
    w["gru_b_ih"][128:256] += 1.0


# The recurrence in pieces: chunks just long enough for two of them and just too short, the most there are, sliced projections, a last chunk
# as one chain; update gates so far open (6: a state keeps 0.997 of itself) that no piece begins where the one before it ended, or some do (2).
@pytest.mark.parametrize("batch,S,D,H", [(2, 130, 512, 4), (1, 161, 1024, 4), (2, 163, 512, 4), (3, 300, 384, 1), (2, 512, 256, 4), (1, 1200, 256, 4),
                                         (40, 600, 128, 4), (2, 200, 200, 4)])
@pytest.mark.parametrize("slow", [0.0, 2.0, 6.0])
def test_prompts_in_pieces(batch, S, D, H, slow):
    _check_prompt(batch, S, D, 128, H=H, change=_opened(slow))


# Whatever keeps more of itself over a warm-up than fp32 would show takes the steps of one chain, bit for bit: gates opened to where the
# pieces' ends come close, units that lose a part of the state at every joint that is too small to see there, states as small.  64 sequences
# leave the pieces no room next to the projection of the chunk behind theirs: some start when the ones before them are through.
@pytest.mark.parametrize("batch,S,D", [(2, 512, 256), (1, 163, 512), (3, 200, 128), (2, 1100, 256), (64, 1100, 1024)])
@pytest.mark.parametrize("change", [_opened(0.9), _opened(1.0), _opened(1.1), _slow_units, _small_states],
                         ids=["opened 0.9", "opened 1.0", "opened 1.1", "slow units", "small states"])
def test_prompts_that_are_remembered(batch, S, D, change, monkeypatch):
    _, _, scores, z, _ = _prompt(batch, S, D, 128, H=4, change=change)
    monkeypatch.setenv("ADORE_NO_PIECES", "1")
    _, _, one_scores, one_z, _ = _prompt(batch, S, D, 128, H=4, change=change)
    assert torch.equal(scores.view(torch.int32), one_scores.view(torch.int32)) and torch.equal(z.view(torch.int32), one_z.view(torch.int32))


# What slow units take in adds up over chunks: a state of 512 tokens behind one of 4096 is not lost.  |z| is the sum of 4608 candidates of at
# most 3e-4 x 1e-5; an fp32 sum of so many is off by 4608 x 2^-24 of it at most, 4e-9, the other units' states by 5e-7.
def test_prompts_with_slow_units_against_64_bits():
    w, x, _, z, pos_scale = _prompt(1, 4608, 128, 128, H=4, change=_slow_units)
    _, want = _reference(w, x, pos_scale)
    assert (z.double() - want).abs().max() <= 1e-6
    assert (z.double() - want)[:, :8].abs().max() <= 1e-8, (z[:, :8], want[:, :8])


# Pieces that stand differ from one chain by its own rounding: errors against 64 bits of the same size (2-norm over all scores)
@pytest.mark.parametrize("batch,S,D", [(4, 512, 256), (2, 1100, 256)])
@pytest.mark.parametrize("slow", [0.0, 0.3, 0.5, 0.65, 0.75])
def test_prompts_in_pieces_are_as_exact_as_one_chain(batch, S, D, slow, monkeypatch):
    w, x, scores, z, pos_scale = _prompt(batch, S, D, 128, H=4, change=_opened(slow))
    again = _prompt(batch, S, D, 128, H=4, change=_opened(slow))    # whichever workgroup worked through the pieces that did not stand
    assert torch.equal(again[2], scores) and torch.equal(again[3], z)
    monkeypatch.setenv("ADORE_NO_PIECES", "1")
    _, _, one_scores, one_z, _ = _prompt(batch, S, D, 128, H=4, change=_opened(slow))
    want_scores, want_z = _reference(w, x, pos_scale)
    off, one_off = (scores.double() - want_scores).norm(), (one_scores.double() - want_scores).norm()
    assert off <= 1.05 * one_off, (off, one_off)
    assert (scores - one_scores).abs().max() <= 1e-6 and (z - one_z).abs().max() <= 1e-6


# Pieces that forgot where they started, and yet did not start where the one before them ended: a few units fall from zero to the lower
# of two states and stay in the upper one once a token has put them there, until another takes them down (some of them inside a
# piece, behind which its states are met again; the last one stays up).
@pytest.mark.parametrize("batch,S", [(2, 512), (3, 250), (2, 1100)])
def test_prompts_in_pieces_that_start_elsewhere(batch, S, monkeypatch):
    def latch(w):
        w["gru_w_hh"][:, :8] = 0
        for gate, bias in ((0, 8.0), (1, -2.0), (2, -0.9)):
            rows = slice(gate * 128, gate * 128 + 8)
            w["gru_w_hh"][rows] = 0
            w["gru_w_ih"][rows] = 0
            w["gru_b_ih"][rows] = bias
            w["gru_b_hh"][rows] = 0
        for i in range(8):
            w["gru_w_hh"][256 + i, i] = 3.0
            w["gru_w_ih"][256 + i, 0] = 1.0

    def pulses(x):
        x[:, :, 0] = 0
        for b in range(x.shape[0]):
            for up, down in ((20, 101 + 3 * b), (140, 207 + b), (333, 480 - b), (500, 700), (840 + b, 1060)):
                if up < S:
                    x[b, up, 0] = 6.0
                if down < S:
                    x[b, down, 0] = -6.0

    w, x, scores, z, pos_scale = _prompt(batch, S, 256, 128, H=4, change=latch, change_x=pulses)
    want_scores, want_z = _reference(w, x, pos_scale)
    assert (z.double() - want_z).abs().max() <= 4e-6 and (scores.double() - want_scores).abs().max() <= 4e-6   # as in _check_prompt
    monkeypatch.setenv("ADORE_NO_PIECES", "1")
    _, _, one_scores, one_z, _ = _prompt(batch, S, 256, 128, H=4, change=latch, change_x=pulses)
    assert (scores - one_scores).abs().max() <= 1e-6 and (z - one_z).abs().max() <= 1e-6


# 24 sequences go over the wide tiles of the input projection, 12 over the narrow ones: the same sums
def test_prompts_over_wide_and_narrow_tiles_are_the_same(monkeypatch):
    randn = torch.randn
    _, x, scores, z, _ = _prompt(24, 512, 2048, 128, H=2)

    def again(*shape, generator=None):
        out = randn(*shape, generator=generator)
        return x[:12].float().cpu() if shape[0] == tuple(x[:12].shape) else out
    monkeypatch.setattr(torch, "randn", again)
    _, x12, few_scores, few_z, _ = _prompt(12, 512, 2048, 128, H=2)
    assert torch.equal(x12, x[:12])
    assert torch.equal(few_scores, scores[:12]) and torch.equal(few_z, z[:12])


# The chunks' second copy in the cache (undivided with sliced tails, and at the smallest cache that holds it), behind everything else, and
# missing; with the guard words of the debug layout, which tests/conftest.py counts when the job closes.
@pytest.mark.parametrize("guards", [False, True])
@pytest.mark.parametrize("batch,S,D,H,K,without", [(1, 1100, 512, 16, 512, False), (1, 770, 1024, 12, 512, False),
                                                   (3, 1537, 256, 12, 512, False), (2, 1100, 256, 2, 24, False),
                                                   (2, 1100, 256, 2, 24, True), (1, 700, 512, 2, 24, True),
                                                   # a cache with room for exactly the whole prompt in one chunk (682, 1365 tokens a
                                                   # sequence), for one token less, and for chunks of half the room (680)
                                                   (1, 682, 256, 16, 512, False), (1, 683, 256, 16, 512, False),
                                                   (2, 1365, 256, 16, 1024, False), (2, 1366, 256, 16, 1024, False),
                                                   (1, 2040, 128, 16, 1024, False), (3, 2041, 128, 16, 1024, False),
                                                   # halves of 520 rows with a sliced last chunk in the lower one (35 chunks), in the upper (34)
                                                   (1, 17921, 2048, 16, 780, False), (1, 17410, 1024, 16, 780, False)])
def test_places_of_the_chunks_second_copy(batch, S, D, H, K, without, guards, monkeypatch):
    import os
    from paper_2407_02328_amd import binding
    if guards:
        monkeypatch.setenv("ADORE_GUARD_WORDS", "1")
    guards = os.environ.get("ADORE_GUARD_WORDS", "0") != "0"
    if without:
        lib = binding.load_library()
        second = max(512 * batch, 4096) * 3 * 128 * 4 + 512 * batch * 128 * 4 + (512 if guards else 0)

        class Smaller:
            def __getattr__(self, name):
                return getattr(lib, name)

            def adore_workspace_bytes(self, cfg):
                return lib.adore_workspace_bytes(cfg) - second
        monkeypatch.setattr(binding, "load_library", lambda: Smaller())
    _check_prompt(batch, S, D, 128, H, K)
