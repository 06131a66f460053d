"""Dispatch and workspaces of the forward calls, on the host side alone (see hostside.py)."""
import pytest

import hostside


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = hostside.build_fake(tmp_path_factory.mktemp("fake"))
    return lambda body: hostside.run(so, body)


@pytest.mark.parametrize("dtype,d,dff,first,second,rank", [
    ("bf16", 256, 1024, 100, 10, 0),    # on the 64-row kernels' tiles: a prompt, then a decode batch
    ("bf16", 256, 1024, 100, 1, 0),
    ("bf16", 256, 1000, 100, 10, 0),    # off them
    ("bf16", 256, 1000, 10, 1, 0),
    ("f32", 256, 1024, 16, 1, 0),
    ("bf16", 256, 1024, 200, 10, 16),   # adapters
    ("bf16", 3072, 5999, 2, 1, 0),      # the single-token kernels would need more than two tokens did
])
def test_a_shorter_call_can_be_captured_after_an_eager_one(run, dtype, d, dff, first, second, rank):
    rc1, rc2, lines = run(f"""
a = fwd({first}, {d}, {dff}, "{dtype}", rank={rank}); log()
fake.fake_capture(1)
b = fwd({second}, {d}, {dff}, "{dtype}", rank={rank})
print(json.dumps([a, b, log()]))""")
    assert rc1 == 0 and rc2 == 0
    assert [l for l in lines if l[0] != "launch"] == []


def test_a_longer_call_keeps_the_buffers_of_a_captured_one(run):
    """The graph of a captured token (or batch) points at its buffers, so a later call
    that needs larger ones frees none of them; sats_release does."""
    freed, held = run("""
fwd(1, 512, 4096); log()
fake.fake_capture(1); fwd(1, 512, 4096); fake.fake_capture(0)
fwd(64, 512, 4096); fwd(300, 512, 4096)
freed = [l for l in log() if l[0] == "free"]
lib.sats_release()
print(json.dumps([freed, fake.fake_held()]))""")
    assert freed == [] and held == 0


def test_a_call_that_can_do_without_the_shorter_ones_workspace_runs_and_does_not_try_again(run):
    """Memory for the tiled products but not for the other kernels' workspace: every
    call runs, and only the first one tries to allocate it."""
    rcs, tries = run("""
fwd(300, 2048, 8192)
sizes = [int(l[2]) for l in log() if l[0] == "malloc"]
lib.sats_release(); log()
fake.fake_limit(sizes[0] + 4096)
rcs = [fwd(300, 2048, 8192) for _ in range(3)]
print(json.dumps([rcs, len([l for l in log() if l[0] in ("malloc-failed", "sync")])]))""")
    assert rcs == [0, 0, 0] and tries <= 4


BIG = (4096, 14336)   # 12 MB for 65 tokens, 166 MB for any prompt


def test_a_prompt_allocates_what_it_needs(run):
    """65 tokens take the buffer of 65 (12.4 MB at this shape), not that of 2048 rows
    with adapters, and the next lengths grow it in few steps."""
    first, grown = run(f"""
def tiled(lines):  # (the tiled buffer is the one that is cleared with its counters)
    big = {{l[1]: int(l[2]) for l in lines if l[0] == "malloc"}}
    return [big[l[1]] for l in lines if l[0] == "memset" and big.get(l[1], 0) > 1 << 20]
fwd(65, *{BIG}); first = tiled(log())
for n in range(66, 1000, 9): fwd(n, *{BIG})
print(json.dumps([first, tiled(log())]))""")
    assert len(first) == 1 and first[0] < 13 << 20
    assert len(grown) <= 4 and sum(grown) < 512 << 20


def test_a_larger_buffer_is_there_before_the_smaller_one_goes(run):
    lines = run(f"""
fwd(65, *{BIG}); log(); fwd(300, *{BIG}); print(json.dumps([l[0] for l in log()]))""")
    assert lines.index("malloc") < lines.index("sync") < lines.index("free")


def test_without_memory_the_passes_of_64_run_and_nothing_is_tried_twice(run):
    """A prompt whose buffer cannot be allocated runs on the 64-row kernels; the
    calls after it neither synchronise nor allocate, the smaller prompt's buffer
    stays, and a reserve with memory at hand brings the tiled products back."""
    r = run(f"""
fwd(100, *{BIG}); log()
fake.fake_limit(fake.fake_held() + (1 << 20))
out = []
for n in (1000, 1000, 900, 100):
    out.append([fwd(n, *{BIG}), log()])
lib.sats_release(); log()
fake.fake_limit(1 << 40)
out.append([reserve(1000, *{BIG}), log()]); out.append([fwd(1000, *{BIG}), log()])
print(json.dumps([[rc, [l[0] for l in lines if l[0] != "launch"], launches(lines)] for rc, lines in out]))""")
    assert [rc for rc, _, _ in r] == [0] * 6
    assert "malloc-failed" in r[0][1] and "free" not in r[0][1]
    assert r[1][1] == [] and all("dense" in k or "route" in k for k in r[0][2] + r[1][2])
    assert r[3][1] == [] and any("pf_gateup" in k for k in r[3][2])
    assert r[5][1] == [] and any("pf_gateup" in k for k in r[5][2])


def test_reserve_without_memory_still_allows_every_call_without_allocating(run):
    rc, calls = run(f"""
fwd(64, *{BIG}); lines = log(); held = fake.fake_held()
lib.sats_release(); log()
fake.fake_limit(held + (24 << 20))   # the 64-row kernels' workspace and little more
rc = reserve(1000, *{BIG}); log()
calls = [[fwd(n, *{BIG}), [l[0] for l in log() if l[0] != "launch"]] for n in (1000, 65, 64, 1)]
print(json.dumps([rc, calls]))""")
    assert rc == 0 and calls == [[0, []]] * 4


def test_adapters_take_memory_only_where_they_are_used(run):
    plain, lora = run("""
fwd(300, 256, 1024); a = fake.fake_held(); lib.sats_release()
fwd(300, 256, 1024, rank=64); b = fake.fake_held()
print(json.dumps([a, b]))""")
    assert plain < lora


@pytest.mark.parametrize("dtype,d,dff", [("f32", 256, 1024), ("bf16", 256, 1000)])
def test_a_captured_batch_takes_the_kernels_of_the_eager_one(run, dtype, d, dff):
    """After an eager prompt of a shape whose short batches run on kernels of the same
    family, a batch under capture runs on those, not on others with other roundings."""
    eager, captured = run(f"""
fwd(100, {d}, {dff}, "{dtype}"); log()
fake.fake_capture(1); fwd(9, {d}, {dff}, "{dtype}"); b = launches(log())
fake.fake_capture(0); fwd(9, {d}, {dff}, "{dtype}")
print(json.dumps([launches(log()), b]))""")
    assert eager == captured and any("sm_gateup" in k for k in eager)


@pytest.mark.parametrize("dtype,d,dff", [("f32", 256, 1024), ("f32", 256, 1001), ("bf16", 256, 1000),
                                         ("bf16", 256, 1024)])
def test_the_batch_path_option_holds_for_every_type(run, dtype, d, dff):
    """SATS_BATCH_COMPACT takes the compacted kernels for float32 as for bf16 (and so
    does SATS_BATCH_SPLIT where no matrix-core group applies); the default does not."""
    got = run(f"""
out = dict()
for name, path in (("auto", AUTO), ("mfma", MFMA), ("split", SPLIT), ("compact", COMPACT)):
    options(path)
    for n in (2, 64, 100):
        assert fwd(n, {d}, {dff}, "{dtype}") == 0
        out[name + str(n)] = launches(log())
print(json.dumps(out))""")
    for key, names in got.items():
        compacted = any("4sats11gate_kernel" in k for k in names)
        tiled = any("sm_gateup" in k or "pf_gateup" in k or "dense_gateup" in k for k in names)
        if key.startswith(("auto", "mfma")):
            assert tiled and not compacted, (key, names)
        elif key.startswith("compact") or dtype == "f32":
            assert compacted and not tiled, (key, names)
