"""When the input gradient's Python call takes scratch memory from torch's allocator, decided on the host.  No GPU is used."""
import pytest

torch = pytest.importorskip("torch")

TOTAL = 288 << 30
NBYTES = 1 << 30


@pytest.fixture
def card(monkeypatch):
    """A card that is not there: what the decision asks about it, and the allocations that it makes."""
    from paper_2104_10949_amd import binding as b
    state = {"free": TOTAL, "fraction": 1.0, "capturing": False, "current": 0, "allocated": [], "mode": 0}

    def exchange(mode):
        before, state["mode"] = state["mode"], mode
        return before
    monkeypatch.setattr(b, "_exchange_capture_mode", exchange)
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (state["free"], TOTAL))
    monkeypatch.setattr(torch.cuda, "get_per_process_memory_fraction", lambda device=None: state["fraction"])
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: state["capturing"])
    monkeypatch.setattr(torch.cuda, "current_device", lambda: state["current"])
    real_empty = torch.empty

    def empty(n, dtype=None, device=None):
        state["allocated"].append((n, state["mode"]))
        return real_empty(8, dtype=dtype)
    monkeypatch.setattr(torch, "empty", empty)
    return state


def takes(state, nbytes=NBYTES, stream=None):
    from paper_2104_10949_amd import binding as b
    state["allocated"].clear()
    taken = b._scratch(nbytes, torch.device("cuda", 0), stream) is not None
    # nothing is asked for where nothing is used; what is asked for, in the relaxed capture mode, and the thread's own is back after it
    assert state["allocated"] == ([(nbytes, b.HIP_STREAM_CAPTURE_MODE_RELAXED)] if taken else []) and state["mode"] == 0
    return taken


def test_scratch_is_taken_where_it_is_free(card):
    assert takes(card)
    card["free"] = TOTAL // 8 + NBYTES
    assert takes(card)


def test_no_memory_is_asked_for_where_it_is_short(card):
    """The allocator would release its whole cache before it says that there is none."""
    for free in (TOTAL // 8 + NBYTES - 1, NBYTES, 0):
        card["free"] = free
        assert not takes(card)


def test_no_memory_is_asked_for_by_a_program_that_limits_its_share(card):
    card["fraction"] = 0.5
    assert not takes(card)


@pytest.mark.parametrize("what", ["nothing to take", "beyond the limit", "named stream", "capturing", "another device"])
def test_calls_that_take_none(card, what):
    from paper_2104_10949_amd import binding as b
    card["capturing"] = what == "capturing"
    card["current"] = 1 if what == "another device" else 0
    assert not takes(card, {"nothing to take": 0, "beyond the limit": b.SCRATCH_LIMIT + 1}.get(what, NBYTES),
                     object() if what == "named stream" else None)
