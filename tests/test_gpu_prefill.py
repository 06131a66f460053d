"""The tiled matrix-core products (batches of more than 64 tokens, batches of
shapes that are on no whole tile, and float32 batches) against the oracle: rows and columns at
the edges of their tiles and of the 16-row blocks, widths in 16-byte pieces
only, stacks, both routes, and passes of unequal length.  Tolerances are those of
tests/harness.py: p and the output are rounded to bf16 (2^-9 each) and the
sums are float32, well inside the 2e-2 bound on the largest element; float32
batches keep float32 throughout (1e-5)."""
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
    # widths of 16-byte rows only: p in three terms
    (120, 2, 24, 41, 2),         # less than one step of k, less than one tile
    (121, 2, 264, 333, 7),
    (122, 1, 1000, 2730, 66),    # k ends in the first half of a weight stage
    (123, 3, 200, 77, 130),
    (124, 1, 384, 1000, 16),     # only d_ff off the tiles
    (125, 2, 520, 1600, 300),    # only d off the tiles
    (126, 1, 2056, 5999, 520),
    # one token, d_ff in no whole 16-byte pieces: the single-token kernels
    (127, 2, 256, 1001, 1),
]


# float32 batches (passes of up to 64 rows)
F32 = [
    (140, 2, 20, 37, 2),         # less than one stage of k, less than one tile
    (141, 2, 260, 333, 7),
    (142, 1, 1028, 2730, 16),
    (143, 3, 128, 512, 17),
    (144, 1, 512, 1536, 48),
    (145, 2, 384, 1001, 64),
    (146, 2, 132, 200, 67),      # a second pass of 3 rows
    (147, 1, 4096, 1024, 33),
]


@pytest.mark.parametrize("dtype,seed,L,d,dff,n", [("bf16", *c) for c in CASES] + [("f32", *c) for c in F32])
def test_prefill_matches_oracle_and_inspection_changes_nothing(dtype, seed, L, d, dff, n):
    print(f"prefill case seed={seed} L={L} d={d} d_ff={dff} n={n} {dtype}", flush=True)
    c = synth.small_case(seed, L, d, dff, dtype, n, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    ts = case_thresholds(c, dtype, seed=seed)
    tokens = sorted({t for t in (0, 15, 16, 63, 64, n // 2, 127, 128, 255, n - 1) if t < n})
    for lut in (None, c["route_lut"]):
        res = run_gpu(c, ts, lut, dtype)
        worst = check_against_oracle(c, ts, lut, dtype, res, tokens=tokens)
        fwd = run_gpu(c, ts, lut, dtype, inspect=False, out_is_x=lut is None)
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


@pytest.mark.parametrize("d,dff,n", [(264, 333, 7), (128, 256, 100)])
def test_allocation_free_call_takes_the_same_kernels(d, dff, n):
    """A batch whose workspace fits the fixed scratch gives sats_mlp_forward's bits."""
    import torch
    import paper_2607_08991_amd as sats
    c = synth.small_case(131, 2, d, dff, "bf16", n, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    ts = case_thresholds(c, "bf16", seed=131)
    assert sats.sats_query_path(n, d, dff, 2) == sats.SATS_PATH_BATCH_MFMA
    x, w = to_dev(c["x"], "bf16"), list(weights_dev(c, "bf16"))
    ids, lut = to_dev(np.asarray(c["token_ids"], np.int32), "bf16"), to_dev(c["route_lut"], "bf16")
    thr = torch.tensor(np.asarray(ts, np.float32)).cuda()
    outs = []
    for call in (sats.sats_mlp_forward, sats.sats_mlp_forward_noalloc):
        o = torch.empty_like(x)
        call(x, ids, *w, thr, lut, o, n, d, dff, 2)
        outs.append(from_dev(o))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(*outs)


# LoRA batches above two passes of 64: adapters as further k of the gate/up product
LORA = [
    # seed, layers, d, d_ff, tokens, rank
    (151, 2, 256, 1024, 129, 16),
    (152, 1, 128, 512, 200, 8),    # the further k fill half a weight stage
    (153, 1, 512, 1536, 300, 64),  # ... and four
    (154, 3, 384, 448, 257, 32),
]


@pytest.mark.parametrize("seed,L,d,dff,n,rank", LORA)
def test_lora_prompt_matches_oracle(seed, L, d, dff, n, rank):
    from test_gpu_lora import check_lora, run_lora, scale_for, thresholds_for
    print(f"lora prompt seed={seed} L={L} d={d} d_ff={dff} n={n} rank={rank}", flush=True)
    w_std = 1.0 / np.sqrt(d)
    c = synth.small_case(seed, L, d, dff, "bf16", n, vocab=40, n_dense_ids=12, w_std=w_std)
    ad = synth.stack_lora_adapters(seed, L, d, dff, rank, "bf16")
    s = scale_for(w_std, rank)
    ts = thresholds_for(c, "bf16", seed)
    for lut in (None, c["route_lut"]):
        res = run_lora(c, ad, rank, s, ts, lut, "bf16")
        worst = check_lora(c, ad, s, ts, lut, "bf16", res)
        again = run_lora(c, ad, rank, s, ts, lut, "bf16", inspect=False)
        np.testing.assert_array_equal(again["out"], res["out"])
        print(f"  lut={'yes' if lut is not None else 'no'} worst rel err {worst:.3g}", flush=True)


def test_captured_prompts_keep_their_buffers():
    """Under capture a prompt takes the passes of 64 where only those are
    reserved (nothing is allocated), and the tiled products once a prompt is;
    longer eager prompts between the replays move no buffer of either graph."""
    import torch
    import paper_2607_08991_amd as sats
    d, dff, n, longer = 256, 1024, 130, 700
    c = synth.small_case(161, 2, d, dff, "bf16", longer, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    ts = case_thresholds(c, "bf16", seed=161)
    x, w = to_dev(c["x"], "bf16"), list(weights_dev(c, "bf16"))
    ids, lut = to_dev(np.asarray(c["token_ids"], np.int32), "bf16"), to_dev(c["route_lut"], "bf16")
    thr = torch.tensor(np.asarray(ts, np.float32)).cuda()
    torch.cuda.synchronize()
    outs = [torch.zeros_like(x) for _ in range(4)]

    def call(o, a, b):
        sats.sats_mlp_forward(x[a:b], ids[a:b], *w, thr, lut, o[a:b], b - a, d, dff, 2)

    stream, graphs = torch.cuda.Stream(), []
    with torch.cuda.stream(stream):
        for reserve, o in ((64, outs[0]), (n, outs[1])):
            sats.sats_reserve(reserve, d, dff, 2, 2)
            torch.cuda.synchronize()
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[-1], stream=stream):
                call(o, 0, n)
        for a in range(0, n, 64):
            call(outs[2], a, min(n, a + 64))  # the passes of 64, eagerly
        call(outs[3], 0, n)
        torch.cuda.synchronize()
        want = [from_dev(outs[2][:n]), from_dev(outs[3][:n])]
        for _ in range(3):
            call(outs[3], 0, longer)
            for g, o, y in zip(graphs, outs, want):
                o.zero_()
                g.replay()
                torch.cuda.synchronize()
                np.testing.assert_array_equal(from_dev(o[:n]), y)


@pytest.mark.parametrize("dtype,d,n", [("f32", 260, 5), ("f32", 260, 40), ("bf16", 264, 7), ("bf16", 264, 70)])
@pytest.mark.parametrize("where", ["gate", "gate product", "p", "p rounds up", "y"])
def test_an_overflow_stays_an_infinity(dtype, d, n, where):
    """Sums past float32's range are infinite, as in the compacted kernels (same keep
    sets, same outputs bit for bit: one row and one neuron carry the values, so no
    order of summation matters), and p between the largest bf16 and the largest
    float32 stays finite."""
    import torch
    import paper_2607_08991_amd as sats
    dff, dt = 333, torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.zeros((n, d), dtype=dt, device="cuda")
    wg, wu, wd = (torch.zeros((dff, d), dtype=dt, device="cuda") for _ in range(3))
    j, r = 201, n - 2                       # the neuron and the row
    x[r, :] = 2.0 ** 32
    wg[j, 0] = 2.0 ** 33                    # a = 2^65
    wd[j, :] = 2.0 ** -10
    if where == "gate":                     # ten terms of 2^125
        wg[j, :10] = 2.0 ** 93
        wu[j, 0] = 2.0 ** -40
    elif where == "gate product":
        wg[j, 7] = 2.0 ** 97
        wu[j, 0] = 2.0 ** -40
    elif where == "p":
        wu[j, :] = 2.0 ** 32
    elif where == "p rounds up":            # 1.998046875 2^127: bf16 ends at 1.9921875 2^127
        wu[j, 0], wu[j, 1] = 255 / 128 * 2.0 ** 30, 1.5 * 2.0 ** 22
    else:
        wu[j, 0] = 2.0 ** 28                # p = 2^125
        wd[j, :] = 2.0 ** 10
    thr = torch.ones(1, device="cuda")
    got = []
    for path in (sats.SATS_BATCH_AUTO, sats.SATS_BATCH_COMPACT):
        out = torch.empty_like(x)
        cnt = torch.empty((1, n), dtype=torch.int32, device="cuda")
        with sats.options(batch_path=path):
            sats.sats_mlp_forward_inspect(x, None, wg, wu, wd, thr, None, out, n, d, dff, 1, active_count=cnt)
        torch.cuda.synchronize()
        got.append((from_dev(out), cnt.cpu().numpy()))
        want = 255.75 / 128 * 2.0 ** 117 if where == "p rounds up" else np.inf
        assert (out[r].float().cpu().numpy() == np.float32(torch.tensor(want).to(dt).float())).all(), (path, out[r, :4])
        assert cnt[0, r].item() == 1
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("d,dff,n,level", [(4096, 4096, 2, 0.9), (4096, 4096, 3, 0.97), (512, 16400, 5, 0.95),
                                           (1028, 9001, 8, 0.97), (512, 17001, 6, 0.5), (4096, 2048, 2, None)])
def test_float32_batches_read_no_row_that_nothing_keeps(d, dff, n, level):
    """W_down rows that no token keeps are not read (NaN there changes no bit) but for
    the first two stages (64 rows) of a workgroup's chunk, which are loaded before the
    flags are there; every kept row counts (float64 sums over the call's keep sets)."""
    import torch
    import paper_2607_08991_amd as sats
    print(f"float32 rows nothing keeps d={d} d_ff={dff} n={n} level={level}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(d + dff + n)
    x = torch.randn((n, d), generator=g, device="cuda")
    wg, wu, wd = (torch.randn((dff, d), generator=g, device="cuda") / d ** 0.5 for _ in range(3))
    a = x.double() @ wg.double().T
    p = a * torch.sigmoid(a) * (x.double() @ wu.double().T)
    mag = (a * torch.sigmoid(a)).abs().reshape(-1)
    thr = torch.tensor([np.inf if level is None else float(torch.quantile(mag[:1 << 20], level))], device="cuda").float()

    def call(w):
        out, cnt = torch.empty_like(x), torch.empty((1, n), dtype=torch.int32, device="cuda")
        idx = torch.empty((1, n, dff), dtype=torch.int32, device="cuda")
        sats.sats_mlp_forward_inspect(x, None, wg, wu, w, thr, None, out, n, d, dff, 1, active_count=cnt, active_idx=idx)
        torch.cuda.synchronize()
        keep = torch.zeros((n, dff), dtype=torch.bool, device="cuda")
        for m in range(n):
            keep[m, idx[0, m, :int(cnt[0, m])].long()] = True
        return out, keep

    out, keep = call(wd)
    y = (p * keep) @ wd.double()
    assert float((out - y).abs().max()) <= 1e-5 * max(float(y.abs().max()), 1e-30)
    # d_ff in chunks of whole stages of 32 rows, a workgroup per compute unit and 128 columns, at most 16
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    chunk = -(-dff // min(16, max(1, cus // -(-d // 128)))) + 31 & -32
    rows = ~keep.any(0) & (torch.arange(dff, device="cuda") % chunk >= 64)
    assert int(rows.sum()) > dff // 100
    poisoned = wd.clone()
    poisoned[rows] = float("nan")
    np.testing.assert_array_equal(from_dev(call(poisoned)[0]), from_dev(out))


def _picked(c, res, rows):
    """`rows` of a case and of an inspect run of it."""
    sub = dict(c, x=c["x"][rows], token_ids=np.asarray(c["token_ids"])[rows])
    return sub, dict(route=res["route"][rows], count=res["count"][:, rows], idx=res["idx"][:, rows],
                     layer_in=res["layer_in"][:, rows], out=res["out"][rows])


# passes of at most 2048 rows, equal shares in whole tiles of 256: 2100 tokens are 1280 and
# 820, 16385 eight of 2048 and one of a single row
@pytest.mark.parametrize("seed,L,d,dff,n,rank", [
    (180, 1, 8, 8, 66, 0),           # less than one step of k
    (181, 2, 24, 41, 70, 0),
    (182, 2, 264, 333, 2100, 0),     # off the tiles
    (183, 1, 128, 64, 16385, 0),     # a last pass of one row
    (184, 1, 136, 72, 16385, 0),     # ... off the tiles: on the kernels of up to 64 rows
    (185, 2, 128, 128, 2100, 16),    # adapters
    (186, 1, 128, 64, 16385, 8),
])
def test_prompts_at_the_edges_of_their_passes(seed, L, d, dff, n, rank):
    from test_gpu_lora import check_lora, run_lora, scale_for, thresholds_for
    print(f"pass edges seed={seed} L={L} d={d} d_ff={dff} n={n} rank={rank}", flush=True)
    w_std = 1.0 / np.sqrt(d)
    c = synth.small_case(seed, L, d, dff, "bf16", n, vocab=40, n_dense_ids=12, w_std=w_std)
    rows = sorted({t for t in (0, 17, 65, 1279, 1280, 1281, 2047, 2048, 16383, n - 2, n - 1) if t < n})
    for lut in (None, c["route_lut"]):
        if rank:
            ad, s, ts = synth.stack_lora_adapters(seed, L, d, dff, rank, "bf16"), scale_for(w_std, rank), \
                thresholds_for(c, "bf16", seed)
            res = run_lora(c, ad, rank, s, ts, lut, "bf16")
            sub, part = _picked(c, res, rows)
            check_lora(sub, ad, s, ts, lut, "bf16", part)
            fwd = run_lora(c, ad, rank, s, ts, lut, "bf16", inspect=False)
        else:
            ts = case_thresholds(c, "bf16", seed=seed)
            res = run_gpu(c, ts, lut, "bf16")
            check_against_oracle(c, ts, lut, "bf16", res, tokens=rows)
            fwd = run_gpu(c, ts, lut, "bf16", inspect=False)
        np.testing.assert_array_equal(fwd["out"], res["out"])


@pytest.mark.parametrize("dtype,d,dff,n", [("bf16", 128, 192, 70), ("bf16", 264, 333, 70), ("bf16", 264, 333, 7),
                                           ("f32", 260, 333, 7), ("f32", 4096, 2048, 3)])
def test_an_infinite_threshold_removes_every_column(dtype, d, dff, n):
    """Sparse-path rows are exactly zero, base-path rows those of the dense call."""
    c = synth.small_case(190, 2, d, dff, dtype, n, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    c["token_ids"] = np.asarray(c["token_ids"]).copy()
    lut = np.asarray(c["route_lut"])
    c["token_ids"][:2] = np.flatnonzero(lut)[0], np.flatnonzero(lut == 0)[0]  # both routes
    base = lut[c["token_ids"]] != 0
    got = run_gpu(c, [np.inf, np.inf], c["route_lut"], dtype)
    dense = run_gpu(c, [np.inf, np.inf], None, dtype, dense=True)
    assert (got["count"][:, ~base] == 0).all() and (got["count"][:, base] == dff).all()
    assert not (got["out"][~base] if dtype == "f32" else got["out"][~base] & 0x7fff).any()
    np.testing.assert_array_equal(got["out"][base], dense["out"][base])


@pytest.mark.parametrize("dtype,d,dff,n", [("f32", 260, 1001, 9), ("bf16", 264, 333, 9), ("bf16", 264, 333, 100)])
def test_a_captured_batch_without_its_matrix_core_workspace(dtype, d, dff, n):
    """Where only the other kernels' workspace is there a captured batch takes those
    kernels, and after a reserve the usual ones; each replay gives its eager call's bits."""
    import torch
    import paper_2607_08991_amd as sats
    c = synth.small_case(191, 2, d, dff, dtype, n, vocab=40, n_dense_ids=12, w_std=1.0 / np.sqrt(d))
    ts = case_thresholds(c, dtype, seed=191)
    x, w = to_dev(c["x"], dtype), list(weights_dev(c, dtype))
    ids, lut = to_dev(np.asarray(c["token_ids"], np.int32), dtype), to_dev(c["route_lut"], dtype)
    thr = torch.tensor(np.asarray(ts, np.float32)).cuda()
    outs = [torch.zeros_like(x) for _ in range(4)]
    torch.cuda.synchronize()

    def call(o):
        sats.sats_mlp_forward(x, ids, *w, thr, lut, o, n, d, dff, 2)

    stream, graphs = torch.cuda.Stream(), []
    sats.sats_release()
    with torch.cuda.stream(stream):
        with sats.options(batch_path=sats.SATS_BATCH_COMPACT):
            call(outs[0])
        for o in outs[1:3]:
            torch.cuda.synchronize()
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[-1], stream=stream):
                call(o)
            sats.sats_reserve(n, d, dff, 2, x.element_size())
        call(outs[3])
        torch.cuda.synchronize()
        want = [from_dev(outs[0]), from_dev(outs[3])]
        for _ in range(3):
            call(outs[3])
            for g, o, y in zip(graphs, outs[1:3], want):
                o.zero_()
                g.replay()
                torch.cuda.synchronize()
                np.testing.assert_array_equal(from_dev(o), y)
