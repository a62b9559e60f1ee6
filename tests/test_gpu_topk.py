"""GPU parity of adore_topk_attention (top-K attention over a whole sequence) against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _mods():
    import torch
    from oracle import adore_oracle as O
    from paper_2407_02328_amd import topk_attention
    return torch, O, topk_attention


def _to_gpu(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda:0").to(torch.bfloat16).contiguous()


def _bf16_values(torch, a):
    """The values a bf16 tensor holds, as fp64 (so that the oracle sees what the GPU sees)."""
    return _to_gpu(torch, a).float().cpu().numpy().astype(np.float64)


def _row_err(got, want):
    return np.abs(got - want).max(axis=-1) / np.maximum(np.abs(want).max(axis=-1), 1e-30)


BAND = 1e-3      # weights closer than this may change places between fp32 and fp64 accumulation (a hundred times the
                 # fp32 error of a d-term sum of products of unit-variance values)
TOL = 2e-3 + 2.0 ** -8      # the attention tolerance + the rounding of the bf16 output


def _check_rows_allowing_swaps_at_the_cut(O, q, k, v, got, top_k, what):
    """q, k, v, got: [rows, S, d] fp64.  The GPU decides on fp32 weights, the oracle on fp64 ones.  A query whose
    K-th and (K+1)-th largest weights are more than BAND apart has one kept set, and its row must meet TOL against
    the oracle's.  For the others the kept sets a decision on weights perturbed by less than BAND / 2 can reach are
    listed: a key stays for certain if fewer than K others come within BAND of it from above, goes for certain if K
    others beat it by more than BAND, and the keys in between fill the remaining places in every combination; the
    GPU's row must meet TOL against the oracle's softmax and value sum over ONE of these sets."""
    import itertools
    rows, S, d = q.shape
    want, _ = O.topk_attention(q, k, v, top_k)
    e = _row_err(got, want)
    unclear, worst_unclear = 0, 0.0
    for r in range(rows):
        for i in range(top_k, S):
            w = k[r, :i + 1] @ q[r, i]
            srt = np.sort(w)[::-1]
            if srt[top_k - 1] - srt[top_k] > BAND:
                assert e[r, i] < TOL, f"{what}: row {r} query {i}: {e[r, i]}"
                continue
            unclear += 1
            n_ge = lambda x: int(np.searchsorted(-srt, -x, side="right"))       # how many weights are >= x
            n_gt = lambda x: int(np.searchsorted(-srt, -x, side="left"))        # ... > x
            sure = [j for j in range(i + 1) if n_ge(w[j] - BAND) <= top_k]
            band = [j for j in range(i + 1) if n_ge(w[j] - BAND) > top_k and n_gt(w[j] + BAND) < top_k]
            need = top_k - len(sure)
            assert 0 <= need <= len(band) and len(band) <= 12, (len(sure), len(band))
            best = np.inf
            for comb in itertools.combinations(band, need):
                sel = np.array(sorted(sure + list(comb)))
                out = O.softmax_row(w[sel] / np.sqrt(np.float64(d))) @ v[r, sel]
                best = min(best, float(np.abs(got[r, i] - out).max() / np.abs(out).max()))
            worst_unclear = max(worst_unclear, best)
            assert best < TOL, f"{what}: row {r} query {i}: no kept set within the band gives the GPU's row ({best})"
        for i in range(min(top_k, S)):
            assert e[r, i] < TOL, f"{what}: row {r} query {i}: {e[r, i]}"
    print(f"{what}: worst row {e.max():.2e} against the oracle's own sets; {unclear} queries with a tie within {BAND} at "
          f"the cut, worst of them against their best admissible set {worst_unclear:.2e}", flush=True)
    assert unclear <= 0.1 * rows * S


GRID_CASES = [
    # rows, S, d, top_k
    (2, 1, 64, 1),            # a single token
    (3, 17, 64, 5),           # one ragged query block
    (2, 100, 128, 1),         # K = 1: the value row of the largest weight
    (2, 100, 128, 32),
    (1, 257, 128, 96),        # ragged tail of one query and one key
    (2, 600, 64, 96),         # several query blocks, every wave has several key blocks
    (1, 300, 128, 1000),      # K beyond the sequence: plain causal attention
    (1, 1024, 128, 96),       # whole steps of 128 keys
    (1, 1100, 64, 200),       # ... and a ragged last one
    (1, 2048, 128, 300),      # the longest sequence adore_topk_attention_static takes
    (1, 2049, 64, 300),       # one more
    (2, 3000, 128, 96),       # long sequences
    (2, 200, 64, 64),         # K a multiple of the wave
    (11, 70, 64, 20),         # one whole group of 8 rows (one per XCD) and a tail of 3
]


@pytest.mark.parametrize("rows,S,d,top_k", GRID_CASES)
def test_topk_attention_on_exactly_representable_weights(rows, S, d, top_k):
    """q and k on a grid of quarters in [-2, 2]: every product sum is exact in fp32 and in fp64, so both sides
    select from identical weights, equal weights abound (the tie rule decides many rows) and the kept sets are
    the same; the outputs then differ by the arithmetic of the softmax and the second product only."""
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(1000 * S + top_k)
    q = rng.integers(-8, 9, size=(rows, S, d)) / 4.0
    k = rng.integers(-8, 9, size=(rows, S, d)) / 4.0
    v = _bf16_values(torch, rng.standard_normal((rows, S, d)))
    want, kept = O.topk_attention(q, k, v, top_k)
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), top_k)
    torch.cuda.synchronize()
    e = _row_err(got.float().cpu().numpy().astype(np.float64), want)
    print(f"grid rows={rows} S={S} d={d} K={top_k}: worst row error {e.max():.2e}", flush=True)
    assert e.max() < TOL


@pytest.mark.parametrize("rows,S,d,top_k", [(2, 500, 128, 96), (2, 333, 64, 48), (1, 1500, 128, 512), (1, 2600, 128, 700)])
def test_topk_attention_on_gaussian_inputs(rows, S, d, top_k):
    """Gaussian q, k, v.  The GPU takes its decision on fp32 weights, the oracle on fp64 ones: where the K-th and
    the (K+1)-th largest weight of a query are further apart than the fp32 accumulation error can bridge, the kept
    sets are the same and the output must agree to the attention tolerance; for the few other queries the GPU's row
    must be the oracle's attention over one of the kept sets that differ only in keys within that distance of the cut."""
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(7 * S + top_k)
    q, k, v = (_bf16_values(torch, rng.standard_normal((rows, S, d))) for _ in range(3))
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), top_k).float().cpu().numpy().astype(np.float64)
    torch.cuda.synchronize()
    _check_rows_allowing_swaps_at_the_cut(O, q, k, v, got, top_k, f"gauss rows={rows} S={S} K={top_k}")


def test_topk_attention_at_the_benchmark_shape_sampled_rows():
    """B16 x H32 rows of 1024 tokens, head_dim 128, K = 96 (the paper's fine-tuning setting), as bench.py
    --topk-attention times it: eight rows checked in full against the oracle, Gaussian inputs drawn on the device."""
    torch, O, topk_attention = _mods()
    from gen import DeviceNormals
    rows, S, d, top_k = 512, 1024, 128, 96
    drawer = DeviceNormals(20240702, "cuda:0")
    q, k, v = (drawer.normal((rows, S, d), 1.0, torch.bfloat16) for _ in range(3))
    got = topk_attention(q, k, v, top_k)
    torch.cuda.synchronize()
    pick = [0, 1, 63, 200, 255, 256, 400, 511]
    sel = torch.tensor(pick, device="cuda:0")
    q64, k64, v64 = (t[sel].float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    _check_rows_allowing_swaps_at_the_cut(O, q64, k64, v64, got[sel].float().cpu().numpy().astype(np.float64), top_k,
                                          "benchmark shape")


def test_topk_attention_rejects_what_it_does_not_take():
    torch, O, topk_attention = _mods()
    from paper_2407_02328_amd import AdoreError
    q = torch.zeros((1, 8, 96), dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(AdoreError):
        topk_attention(q, q, q, 4)                      # head_dim 96
    q = torch.zeros((1, 32769, 64), dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(AdoreError):
        topk_attention(q, q, q, 4)                      # sequence longer than the entry point takes
    q = torch.zeros((1, 8, 64), dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(AdoreError):
        topk_attention(q, q, q, 0)
    with pytest.raises(AdoreError):
        topk_attention(q, q, q, 4, workspace=torch.empty(16, dtype=torch.uint8, device="cuda:0"))


def _random_topk_cases(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(count):
        S = int(rng.integers(1, 700))
        out.append((int(rng.integers(1, 12)), S, int(rng.choice([64, 128])), int(rng.integers(1, S + 40)),
                    int(rng.choice([1, 2, 4, 8]))))
    return out


@pytest.mark.parametrize("rows,S,d,top_k,levels", _random_topk_cases(24, 2407))
def test_topk_attention_random_shapes_on_exactly_representable_weights(rows, S, d, top_k, levels):
    """Random shapes; q and k on grids of `levels` steps per unit (coarse grids: most weights of a query tie, so
    the cut among equal weights decides nearly every row; fine grids: few ties)."""
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(rows * 100003 + S * 17 + top_k)
    q = rng.integers(-2 * levels, 2 * levels + 1, size=(rows, S, d)) / float(levels)
    k = rng.integers(-2 * levels, 2 * levels + 1, size=(rows, S, d)) / float(levels)
    if levels == 1:                        # very coarse: make whole runs of keys identical
        k[:, ::3] = k[:, :1]
    v = _bf16_values(torch, rng.standard_normal((rows, S, d)))
    want, kept = O.topk_attention(q, k, v, top_k)
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), top_k)
    torch.cuda.synchronize()
    e = _row_err(got.float().cpu().numpy().astype(np.float64), want)
    assert e.max() < TOL, f"rows={rows} S={S} d={d} K={top_k} levels={levels}: {e.max()}"


@pytest.mark.timeout(900)
def test_topk_attention_at_the_long_context_shape_sampled_rows():
    """B4 x H32 rows of 8192 tokens (the long-context workload's prompts), K = 96.  Two rows that sit on different XCDs
    checked in full against the oracle; what the call asks for as a workspace (and does not touch) stays below 1 GiB."""
    torch, O, topk_attention = _mods()
    from gen import DeviceNormals
    from paper_2407_02328_amd import load_library
    rows, S, d, top_k = 128, 8192, 128, 96
    assert load_library().adore_topk_attention_workspace_bytes(rows, S, d) < (1 << 30)
    drawer = DeviceNormals(20240703, "cuda:0")
    q, k, v = (drawer.normal((rows, S, d), 1.0, torch.bfloat16) for _ in range(3))
    got = topk_attention(q, k, v, top_k)
    torch.cuda.synchronize()
    pick = [77, 122]
    sel = torch.tensor(pick, device="cuda:0")
    q64, k64, v64 = (t[sel].float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    _check_rows_allowing_swaps_at_the_cut(O, q64, k64, v64, got[sel].float().cpu().numpy().astype(np.float64), top_k,
                                          "long-context shape")


@pytest.mark.parametrize("rows,S,d,top_k,same", [
    (1, 1, 64, 1, 0), (2, 31, 64, 8, 0), (1, 33, 128, 32, 0), (2, 129, 64, 17, 0),   # query blocks of 32, key steps of 128
    (1, 161, 128, 40, 0),        # the last query block samples its keys, the ones before it see all of them
    (1, 257, 64, 256, 0), (1, 320, 128, 400, 0),                                      # top_k at and beyond the sequence
    (512, 40, 64, 12, 0), (260, 65, 128, 20, 0),                                      # query blocks of 64, key steps of 64
    (512, 64, 128, 63, 0), (176, 129, 128, 40, 0), (128, 193, 64, 50, 0), (56, 577, 128, 96, 0), (104, 300, 64, 30, 250),
    (7, 193, 64, 20, 0), (15, 290, 128, 30, 0), (61, 330, 128, 40, 0),                # rows that make up no group of eight, which go first
    (1, 300, 128, 50, 300), (2, 200, 64, 30, 60),   # (runs of) identical keys: more equal weights than are ranked directly
])
def test_topk_attention_at_the_edges_of_its_blocks(rows, S, d, top_k, same):
    """Exactly representable weights, as above; up to four rows of a launch are checked, the first and the last among them."""
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(rows * 7919 + S * 31 + top_k)
    q = rng.integers(-8, 9, size=(rows, S, d)) / 4.0
    k = rng.integers(-8, 9, size=(rows, S, d)) / 4.0
    if same:
        k[:, :same] = k[:, :1]
    v = _bf16_values(torch, rng.standard_normal((rows, S, d)))
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), top_k).float().cpu().numpy().astype(np.float64)
    pick = sorted({0, rows // 3, rows // 2, rows - 1})
    want, _ = O.topk_attention(q[pick], k[pick], v[pick], top_k)
    e = _row_err(got[pick], want)
    assert e.max() < TOL, f"rows={rows} S={S} d={d} K={top_k}: {e.max()}"


def _checked_rows(O, torch, topk_attention, q, k, top_k, rng, what):
    """Exactly representable weights: the kept sets are the oracle's.  The first, the last and two other rows are checked."""
    rows = q.shape[0]
    v = _bf16_values(torch, rng.standard_normal(q.shape))
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), top_k).float().cpu().numpy().astype(np.float64)
    pick = sorted({0, rows // 3, rows // 2, rows - 1})
    want, _ = O.topk_attention(q[pick], k[pick], v[pick], top_k)
    e = _row_err(got[pick], want)
    print(f"{what}: worst row error {e.max():.2e}", flush=True)
    assert e.max() < TOL, f"{what}: {e.max()}"


# 32 and 64 queries per workgroup.  The weights are multiples of 2^(2 exponent - 4): down to the smallest normal numbers, where
# their squares vanish, and up to where these overflow and the softmax is that of the largest weight or the ties with it
@pytest.mark.parametrize("rows,S,d,top_k", [(2, 300, 64, 40), (260, 200, 128, 33)])
@pytest.mark.parametrize("exponent", [-60, -52, -46, -25, 8, 14, 18, 33, 57])
def test_topk_attention_far_from_unit_scale(rows, S, d, top_k, exponent):
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(100 * S - exponent)
    q, k = (rng.integers(-8, 9, size=(rows, S, d)) / 4.0 * 2.0 ** exponent for _ in range(2))
    _checked_rows(O, torch, topk_attention, q, k, top_k, rng, f"rows={rows} exponent={exponent}")


# Keys whose weights crowd one value (and so go by position) or lead the sampled range astray, for both workgroup sizes.
# From position 512 on a query block samples every fourth key (multiples of four) or fewer.
KEYS = {
    "zeroed": lambda k, rng: np.where(rng.random(k.shape[:2])[..., None] < 0.6, 0.0, k),           # the K-th weight is often 0
    "zeroed tail": lambda k, rng: np.where((np.arange(k.shape[1]) >= k.shape[1] // 2)[None, :, None], 0.0, k),
    "runs": lambda k, rng: np.where((np.arange(k.shape[1]) % 5 < 3)[None, :, None], k[:, :1], k),
    "whole numbers": lambda k, rng: np.rint(k),
    "samples zero": lambda k, rng: np.where((np.arange(k.shape[1]) % 4 == 0)[None, :, None], 0.0, k),
    "samples large": lambda k, rng: np.where((np.arange(k.shape[1]) % 4 == 0)[None, :, None], 64.0 * k, k),
    "samples equal": lambda k, rng: np.where((np.arange(k.shape[1]) % 4 == 0)[None, :, None], k[:, :1], k),
}


@pytest.mark.parametrize("rows,S,d,top_k", [(2, 620, 64, 200), (56, 620, 64, 50), (2, 580, 128, 290), (56, 580, 128, 20)])
@pytest.mark.parametrize("keys", list(KEYS))
def test_topk_attention_with_crowded_or_misleading_keys(rows, S, d, top_k, keys):
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(rows * 31 + S + len(keys))
    q, k = (rng.integers(-8, 9, size=(rows, S, d)) / 4.0 for _ in range(2))
    _checked_rows(O, torch, topk_attention, q, KEYS[keys](k, rng), top_k, rng, f"rows={rows} {keys}")


@pytest.mark.parametrize("S,d,levels,top_k,offset", [
    (32768, 64, 1, 33, 0),        # 32735 equal keys in one bin: the fullest a histogram's 16 bits get
    (32768, 64, 1, 33, 1),        # ... and one of them stays
    (32768, 64, 1, 33, -1),       # one of the crowded upper bin goes
    (700, 128, 40, 350, 0),       # a cut between two crowded bins, odd and even ones: the bin above it stays whole
    (700, 128, 41, 350, 0),
    (700, 64, 40, 350, 7),        # ... and inside one
    (200, 128, 200, 50, 0),       # bins of a single weight
])
def test_bins_that_stay_whole_and_bins_that_are_full(S, d, levels, top_k, offset):
    """Keys whose weights are whole numbers 0 .. levels, the same for every query (q is the first unit vector): how many of them a
    bin holds is known.  Every query's kept set is the top_k highest, equal ones by position; the last queries are checked in 64
    bits (the bound of the other tests)."""
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(S + levels + top_k)
    level = np.zeros(S)
    if levels == 1:
        level[rng.permutation(S - 64)[:top_k]] = 1.0             # top_k keys above all others
    else:
        level = rng.integers(0, levels + 1, size=S).astype(np.float64)
        above = np.sort(level)[::-1]
        top_k = int(np.searchsorted(-above, -above[top_k - 1], side="right"))   # every key down to one level: the cut between two
    keep = top_k + offset
    q, k = np.zeros((1, S, d)), np.zeros((1, S, d))
    q[..., 0], k[0, :, 0] = 1.0, level
    v = _bf16_values(torch, rng.standard_normal((1, S, d)))
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), keep).float().cpu().numpy().astype(np.float64)
    for i in range(S - 40, S):
        sel = np.sort(np.argsort(-level[:i + 1], kind="stable")[:keep])
        want = O.softmax_row(level[sel] / np.sqrt(np.float64(d))) @ v[0, sel]
        e = np.abs(got[0, i] - want).max() / np.abs(want).max()
        assert e < TOL, f"S={S} K={keep}: query {i}: {e}"


@pytest.mark.parametrize("rows,d", [(5, 64), (5, 128), (600, 64), (600, 128)])
def test_weights_that_stay_are_within_half_a_place(rows, d):
    """Two keys stay of which the first's probability is 1, and their values cancel to 2^-8 of them and less: what is left shows
    the second's probability to its last bits.  P goes into the product as two bf16 terms, the upper 8 bits and the rest, below 2^-7 P,
    rounded to 8 bits: within 2^-16 P.  Exponential, sums and the division are off by a few 2^-23 (2^-20 allowed).  The output is
    rounded to 8 bits, half a unit of the last of which is up to 2^-8 of it."""
    torch, _, topk_attention = _mods()
    rng = np.random.default_rng(rows + d)
    S = 70
    k = np.zeros((rows, S, d))
    k[..., 0] = -8.0 + 4.0 * rng.random((rows, S))               # far below
    k[:, 0, 0], k[:, 1, 0] = 8.0, 8.0 - 8.0 * rng.random(rows)
    k = _bf16_values(torch, k)
    q = np.zeros((rows, S, d))
    q[..., 0] = 1.0
    p = np.exp((k[:, 1, 0] - 8.0) / np.sqrt(np.float64(d)))[:, None]
    v = _bf16_values(torch, rng.standard_normal((rows, S, d)))
    v[:, 1] = _bf16_values(torch, 1.0 + rng.random((rows, d)))
    v[:, 0] = -_bf16_values(torch, p * v[:, 1])
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), 2).float().cpu().numpy().astype(np.float64)
    want = ((v[:, 0] + p * v[:, 1]) / (1.0 + p))[:, None]
    off = ((2.0 ** -16 + 2.0 ** -20) * p * v[:, 1] / (1.0 + p))[:, None]
    over = np.abs(got[:, 2:] - want) / (off + 2.0 ** -8 * (np.abs(want) + off))
    assert over.max() <= 1.0, over.max()


@pytest.mark.parametrize("rows,d", [(2, 64), (150, 64), (2, 128), (90, 128)])
@pytest.mark.parametrize("top_k", [17, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191, 192, 193])
def test_equal_weights_stay_up_to_the_last_position(rows, d, top_k):
    """All keys equal: the first top_k positions stay, which end before, at and behind the edges of a wave's block of 32 keys, of a
    step's and of a workgroup's queries; a query's result is the mean of their values."""
    torch, O, topk_attention = _mods()
    rng = np.random.default_rng(rows + d + top_k)
    S = 230
    q, k = (np.broadcast_to(rng.integers(-8, 9, size=(rows, 1, d)) / 4.0, (rows, S, d)) for _ in range(2))
    v = _bf16_values(torch, rng.standard_normal((rows, S, d)))
    got = topk_attention(_to_gpu(torch, q), _to_gpu(torch, k), _to_gpu(torch, v), top_k).float().cpu().numpy().astype(np.float64)
    last = np.minimum(np.arange(S), top_k - 1)
    want = np.cumsum(v, axis=1)[:, last] / (last + 1.0)[:, None]
    assert _row_err(got, want).max() < TOL
