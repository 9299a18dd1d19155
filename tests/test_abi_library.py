"""CPU-side checks of the C ABI library: it is built, loads, and exports every function include/bagpipe.h
declares; argument checks that need no GPU return the documented errors."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "bagpipe.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bp_[a-z_0-9]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    import paper_2202_12429_amd as bp
    if not os.path.exists(bp.library_path()):
        from paper_2202_12429_amd.build import build
        build(verbose=False)
    return bp.load_library()


def test_header_declares_the_four_operations():
    names = declared_functions()
    for n in ("bp_oracle_plan", "bp_cache_apply", "bp_embbag_fwd", "bp_embbag_bwd_update"):
        assert n in names


def test_library_exports_every_declared_symbol(lib):
    for name in declared_functions():
        assert hasattr(lib, name), f"{name} is declared in bagpipe.h but not exported"


def test_binding_has_the_same_names():
    import paper_2202_12429_amd as bp
    for n in ("bp_oracle_plan", "bp_cache_apply", "bp_embbag_fwd", "bp_embbag_bwd_update",
              "bp_oracle_plan_workspace_bytes", "bp_embbag_bwd_update_workspace_bytes"):
        assert callable(getattr(bp, n))


def test_config_struct_layout_matches_header():
    import paper_2202_12429_amd as bp
    assert ctypes.sizeof(bp.bp_config) == 64
    assert bp.bp_config.lookahead.offset == 28 and bp.bp_config.lr.offset == 32 and bp.bp_config.reserve.offset == 40
    assert bp.bp_config.cache_w_stride.offset == 48 and bp.bp_config.cache_state_stride.offset == 56


def test_argument_errors_without_gpu(lib):
    import paper_2202_12429_amd as bp
    assert bp.bp_version() >= 100
    assert "capacity" in bp.bp_error_string(-2)
    good = bp.make_config(1000, 64, 16)
    assert bp.bp_oracle_plan_workspace_bytes(good, 4096, 10) > 0
    assert bp.bp_embbag_bwd_update_workspace_bytes(good, 4096, 4096) > 0
    for bad in (bp.make_config(1000, 64, 6),              # 24-byte rows: not a multiple of 16 bytes
                bp.make_config(1000, 0, 16),               # no capacity
                bp.make_config(0, 64, 16),                 # no rows
                bp.make_config(1000, 64, 16, lookahead=-1),
                bp.make_config(1000, 64, 16, reserve=64),  # nothing left to plan with
                bp.make_config(1000, 64, 16, reserve=-1)):
        with pytest.raises(bp.BagpipeError) as e:
            bp.bp_embbag_bwd_update_workspace_bytes(bad, 128, 128)
        assert e.value.status == -1
    with pytest.raises(bp.BagpipeError) as e:
        bp.bp_embbag_bwd_update_workspace_bytes(bp.make_config(1000, 64, 512), 128, 128)   # 2 KiB rows
    assert e.value.status == -6
    with pytest.raises(bp.BagpipeError) as e:
        bp.bp_oracle_plan_workspace_bytes(good, 4096, 10_000)                               # too many batches
    assert e.value.status == -6
    # bf16 rows need dim % 8 == 0
    with pytest.raises(bp.BagpipeError):
        bp.bp_embbag_bwd_update_workspace_bytes(bp.make_config(1000, 64, 12, "bf16"), 128, 128)


@pytest.mark.parametrize("around", [1 << 10, 1 << 18, 1 << 21])
def test_plan_workspace_for_more_lookups_is_enough_for_fewer(lib, around):
    """Short traces are cut into smaller tiles, of which they may have more than a longer trace has of its own."""
    import paper_2202_12429_amd as bp
    cfg = bp.make_config(10_000, 512, 16, lookahead=8)
    sizes = [around + d for d in (-4097, -1, 0, 1, 4097) if around + d > 0]
    for grouping in (False, True):
        need = [bp.bp_oracle_plan_workspace_bytes(cfg, n, 10, grouping) for n in sizes]
        assert need == sorted(need)


def test_backward_workspace_for_more_lookups_is_enough_for_fewer(lib):
    """The sort takes larger tiles, and so less scratch, from 2^21 lookups on; a caller that sizes its workspace once for
    the largest batch passes it for the smaller ones too."""
    import paper_2202_12429_amd as bp
    cfg = bp.make_config(10_000, 512, 16)
    sizes = sorted({max(0, around + d) for around in (1 << 10, 1 << 18, 1 << 21) for d in (-4097, -1, 0, 1, 4097)} | {2_200_000})
    need = [bp.bp_embbag_bwd_update_workspace_bytes(cfg, n, n) for n in sizes]
    assert need == sorted(need)


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_torch_internals(monkeypatch, missing):
    """A torch that lacks one of the internal calls still tells its current stream, by the public one."""
    import types
    import torch
    from paper_2202_12429_amd import binding
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert binding._stream(None) == 77


def test_spans_are_slices():
    """A span names what the tensor's slice would, whatever the bounds; anything not contiguous stays a slice."""
    import torch
    from paper_2202_12429_amd import binding
    for t in (torch.arange(40, dtype=torch.int64), torch.arange(160, dtype=torch.int32).view(40, 4), torch.zeros(0, dtype=torch.int32)):
        for a, b in ((0, 0), (0, 40), (3, 17), (17, 3), (-5, 40), (0, -1), (35, 60), (60, 70)):
            want, got = t[a:b], binding._span(t, a, b)
            assert (got.numel(), got.shape[0], binding._count(got), binding._rows(got)) == (want.shape[0],) * 4, (a, b)
            assert want.numel() == 0 or binding._ptr(got) == want.data_ptr()
    strided = torch.arange(40).view(20, 2)[:, 0]
    assert torch.equal(binding._span(strided, 2, 5), strided[2:5])
    assert binding._count(None) == binding._rows(None) == 0


def test_lists_a_call_cannot_do_without(lib):
    """A plan made without the slot map or the grouping carries None for these lists: no call takes that for an empty batch."""
    import torch
    import paper_2202_12429_amd as bp
    cfg = bp.make_config(1000, 64, 16)
    w, ws, tickets = torch.zeros((64, 16)), torch.zeros(1 << 16, dtype=torch.uint8), torch.zeros(64, dtype=torch.int32)
    grad, off, none = torch.zeros((4, 16)), torch.zeros(5, dtype=torch.int64), torch.zeros(0, dtype=torch.int32)
    for b in (None, off):
        with pytest.raises(AttributeError):
            bp.bp_embbag_fwd(cfg, w, None, b, 4, torch.zeros((4, 16)), stream=0)
        with pytest.raises(AttributeError):
            bp.bp_embbag_bwd_update(cfg, w, None, None, b, 4, grad, ws, tickets, stream=0)
        for lookups, rows in ((None, none.view(0, 4)), (none, None), (None, None)):
            with pytest.raises(AttributeError):
                bp.bp_embbag_bwd_update_grouped(cfg, w, None, lookups, rows, None, b, 4, grad, ws, tickets, stream=0)
            with pytest.raises(AttributeError):
                bp.bp_embbag_bwd_update_grouped_static(cfg, w, None, lookups, rows, None, b, 4, grad, stream=0)
    for lookups, rows in ((None, none.view(0, 4)), (none, None), (None, None)):
        with pytest.raises(AttributeError):
            bp.bp_embbag_fwd_grouped(cfg, w, lookups, rows, None, 0, torch.zeros((0, 16)), stream=0)


def test_ticket_bytes_are_the_librarys(lib):
    from paper_2202_12429_amd import binding
    for n in (0, 1, 255, 256, 257, 1 << 20, (1 << 31) - 1):
        assert binding._ticket_bytes(n) == lib.bp_embbag_bwd_ticket_bytes(n)
