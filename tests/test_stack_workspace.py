"""The binding's stack workspace, without a GPU: a stubbed library stands for
libeb.so and records the workspace each call gets.  A cached plan keeps its
launch tables in the workspace that its call passed, so that memory stays with
the op array for as long as the array lives."""

import weakref

import pytest


class FakeLib:
    """Ops with m < 0 are invalid; an op needs 1024 bytes per row."""

    def __init__(self, eb):
        self.eb, self.calls = eb, []

    def _need(self, ops, n):
        return -1 if any(ops[i].m < 0 for i in range(n)) else 1024 * sum(ops[i].m for i in range(n))

    def eb_qlinear_stack_workspace_bytes(self, ops, n):
        return max(0, self._need(ops, n))

    def eb_qlinear_stack(self, ops, n, wp, wb, stream):
        need = self._need(ops, n)
        self.calls.append((wp, wb))
        return self.eb.EB_OK if 0 <= need <= wb else self.eb.EB_ERR_INVALID

    def eb_status_str(self, st):
        return b"status %d" % st


@pytest.fixture
def stack(monkeypatch):
    from paper_2607_02501_amd import eb

    fake = FakeLib(eb)
    monkeypatch.setattr(eb, "lib", fake)
    monkeypatch.setattr(eb, "_stream", lambda device: 0)
    return eb, fake


def _ops(eb, *ms):
    arr = (eb.eb_qlinear_op * len(ms))()
    for o, m in zip(arr, ms):
        o.m = m
    return arr


def test_rejected_call_keeps_the_workspace(stack):
    eb, fake = stack
    ops = _ops(eb, 4, 3)
    eb.qlinear_stack(ops, "cpu")
    ws = ops._eb_workspace
    assert ws.numel() == 7168 and fake.calls[-1] == (ws.data_ptr(), 7168)
    ops[1].m = -1
    with pytest.raises(eb.EBError):
        eb.qlinear_stack(ops, "cpu")
    assert ops._eb_workspace is ws
    ops[1].m = 3
    eb.qlinear_stack(ops, "cpu")
    assert ops._eb_workspace is ws and fake.calls[-1] == (ws.data_ptr(), 7168)


def test_rejected_first_call_and_no_workspace(stack):
    eb, fake = stack
    ops = _ops(eb, -1)
    with pytest.raises(eb.EBError):
        eb.qlinear_stack(ops, "cpu")
    ops[0].m = 0  # needs none
    for _ in range(2):
        eb.qlinear_stack(ops, "cpu")
        assert fake.calls[-1] == (None, 0)
    ops[0].m = 2  # and now some
    eb.qlinear_stack(ops, "cpu")
    assert fake.calls[-1] == (ops._eb_workspace.data_ptr(), 2048)


def test_changed_ops_ask_for_their_size_before_the_call(stack):
    """Under a stream capture the library runs the ops plainly and takes any
    workspace (an op may then run unsplit or be refused), so a list that has
    grown gets its larger workspace before it is passed on, not on an error."""
    eb, fake = stack
    ops = _ops(eb, 1, 0)
    eb.qlinear_stack(ops, "cpu")
    asked = []
    size = fake.eb_qlinear_stack_workspace_bytes
    fake.eb_qlinear_stack_workspace_bytes = lambda o, n: asked.append(1) or size(o, n)
    eb.qlinear_stack(ops, "cpu")
    assert not asked  # the same ops: the size is known
    n = len(fake.calls)
    ops[1].m = 5
    eb.qlinear_stack(ops, "cpu")
    assert [wb for _, wb in fake.calls[n:]] == [6144]
    ops[1].m = 0  # smaller again: the larger workspace serves
    eb.qlinear_stack(ops, "cpu")
    assert fake.calls[-1][1] == 6144


def test_too_small_for_another_setting_is_asked_again(stack):
    """The EB_STACK_* settings change what the same ops need."""
    eb, fake = stack
    ops = _ops(eb, 2)
    eb.qlinear_stack(ops, "cpu")
    need = fake._need
    fake._need = lambda o, n: 2 * need(o, n)
    eb.qlinear_stack(ops, "cpu")
    assert fake.calls[-1] == (ops._eb_workspace.data_ptr(), 4096)


def test_an_outgrown_workspace_stays_with_the_array(stack):
    """The plan of the smaller list is still cached and has its tables there."""
    eb, fake = stack
    ops = _ops(eb, 1)
    eb.qlinear_stack(ops, "cpu")
    first = weakref.ref(ops._eb_workspace)
    ops[0].m = 4
    eb.qlinear_stack(ops, "cpu")
    assert ops._eb_workspace.numel() == 4096 and first() is not None
    del ops
    assert first() is None


def test_an_outgrown_tick_workspace_stays_with_the_modules(stack):
    eb, fake = stack
    mods, need = eb.make_modules([(_ops(eb, 1), 1, 0, 1)]), [1024]
    fake.eb_multirate_workspace_bytes = lambda m, n: need[0]
    fake.eb_multirate_tick = lambda m, n, tick, wp, wb, stream: eb.EB_OK
    eb.multirate_tick(mods, 0, "cpu")
    first = weakref.ref(mods._eb_workspace)
    need[0] = 2048
    eb.multirate_tick(mods, 1, "cpu")
    assert mods._eb_workspace.numel() == 2048 and first() is not None
