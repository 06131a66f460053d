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
