"""Batches of more than 64 tokens (the tiled matrix-core products) against the
oracle: rows and columns at the edges of their tiles and of the 16-row blocks,
stacks, both routes, and passes of unequal length.  Tolerances are those of
tests/harness.py: p and the output are rounded to bf16 (2^-9 each) and the
sums are float32, well inside the 2e-2 bound on the largest element."""
import numpy as np
import pytest

from harness import check_against_oracle, from_dev, run_gpu, to_dev, weights_dev
from test_gpu_parity import case_thresholds
from workloads import synth

pytestmark = pytest.mark.gpu

CASES = [
    # seed, layers, d, d_ff, tokens
    (101, 1, 128, 64, 65),       # one column tile, the fewest rows
    (102, 2, 128, 192, 127),     # a ragged row block
    (103, 1, 256, 1024, 128),
    (104, 2, 384, 448, 129),     # k of 12 steps, a second row tile of one row
    (105, 2, 256, 1024, 256),
    (106, 3, 640, 1536, 257),    # k of 20 steps
    (107, 1, 2048, 6144, 700),
]


@pytest.mark.parametrize("seed,L,d,dff,n", CASES)
def test_prefill_matches_oracle_and_inspection_changes_nothing(seed, L, d, dff, n):
    print(f"prefill case seed={seed} L={L} d={d} d_ff={dff} n={n}", flush=True)
    c = synth.small_case(seed, L, d, dff, "bf16", n, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    ts = case_thresholds(c, "bf16", seed=seed)
    tokens = sorted({0, 15, 16, 63, 64, n // 2, min(n - 1, 127), min(n - 1, 128), min(n - 1, 255), n - 1})
    for lut in (None, c["route_lut"]):
        res = run_gpu(c, ts, lut, "bf16")
        worst = check_against_oracle(c, ts, lut, "bf16", res, tokens=tokens)
        fwd = run_gpu(c, ts, lut, "bf16", inspect=False, out_is_x=lut is None)
        np.testing.assert_array_equal(fwd["out"], res["out"])
        print(f"  lut={'yes' if lut is not None else 'no'} worst rel err {worst:.3g}", flush=True)


def test_prefill_in_two_passes_gives_each_half_alone():
    """2600 tokens run as passes of 1536 and 1064 rows; each gives the bits of
    a call on its rows alone."""
    import torch
    import paper_2607_08991_amd as sats
    d, dff, n, cut = 128, 256, 2600, 1536
    c = synth.small_case(111, 1, d, dff, "bf16", n, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    ts = case_thresholds(c, "bf16", seed=111)
    x, w = to_dev(c["x"], "bf16"), list(weights_dev(c, "bf16"))
    ids, lut = to_dev(np.asarray(c["token_ids"], np.int32), "bf16"), to_dev(c["route_lut"], "bf16")
    thr = torch.tensor(np.asarray(ts, np.float32)).cuda()
    out = torch.empty_like(x)
    sats.sats_mlp_forward(x, ids, *w, thr, lut, out, n, d, dff, 1)
    parts = []
    for a, b in ((0, cut), (cut, n)):
        o = torch.empty((b - a, d), dtype=torch.bfloat16, device="cuda")
        sats.sats_mlp_forward(x[a:b], ids[a:b], *w, thr, lut, o, b - a, d, dff, 1)
        parts.append(from_dev(o))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(from_dev(out), np.concatenate(parts))
