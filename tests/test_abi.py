"""The C-ABI library loads without a GPU and exports every function `include/mebptt.h` declares;
the size queries (pure host arithmetic) behave."""
import ctypes
import os
import re

import pytest

from paper_1606_03401_amd import binding as mb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "mebptt.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"\b(mebptt_[a-z_0-9]+)\s*\(", text)
    return sorted(set(names))


def test_every_declared_symbol_is_exported_and_bound():
    names = _declared_functions()
    assert "mebptt_plan" in names and "mebptt_run" in names and len(names) >= 18
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_1606_03401_amd", "libmebptt.so"))
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in the header but not exported"
        assert n in mb.SIGNATURES, f"{n} has no binding"
    assert set(mb.SIGNATURES) == set(names)
    assert "gfx950" in mb.mebptt_version()


def test_recomputation_stage_in_the_workspace():
    """The workspace carries a stage for recomputed internal states exactly on the shapes whose way
    back through stored hidden states is a forward-batch launch plus a backward-only sweep launch:
    bf16 operands, a shape a backward-only sweep kernel covers (with a copy of the weights per XCD or
    spread over several), and no sweep launch that recomputes internal states itself (the LSTM has
    those up to H = 512; the GRU has none).  As many states as a sweep launch carries (32), at most
    48 MiB, three units each."""
    def desc(B, I, H, cell=0, dtype=1):
        return mb.make_desc(B, I, H, 100, dtype, 0, 1, cell)
    unit = lambda B, H: mb.mebptt_unit_bytes(desc(B, 64, H))
    assert mb.mebptt_stage_steps(desc(64, 256, 1024)) == 32 and 32 * 3 * unit(64, 1024) == 48 << 20
    assert mb.mebptt_stage_steps(desc(128, 64, 1024)) == 16 and 16 * 3 * unit(128, 1024) == 48 << 20
    for B, I, H in ((256, 128, 512), (64, 256, 256), (64, 128, 128)):      # the sweep launch recomputes the states itself
        assert mb.mebptt_stage_steps(desc(B, I, H)) == 0
        assert mb.mebptt_stage_steps(desc(B, I, H, cell=1)) > 0           # the GRU has no such launch
    for B, I, H in ((128, 512, 2048), (200, 64, 1024), (32, 1024, 4096)):  # weights spread over several XCDs
        want = min(32, (48 << 20) // (3 * unit(B, H)))
        assert want > 0 and mb.mebptt_stage_steps(desc(B, I, H)) == want == mb.mebptt_stage_steps(desc(B, I, H, cell=1))
    for B, I, H in ((129, 512, 2048), (257, 64, 1024), (33, 1024, 4096), (16, 64, 4100), (64, 7, 2048)):  # no backward-only sweep launch
        assert mb.mebptt_stage_steps(desc(B, I, H)) == 0 and mb.mebptt_stage_steps(desc(B, I, H, cell=1)) == 0
    assert mb.mebptt_stage_steps(desc(64, 256, 1024, dtype=0)) == 0       # fp32 operands: launch-per-step kernels only
    # the stage is part of the workspace, which does not depend on t
    with_stage, without = desc(64, 256, 1024), desc(64, 256, 1024, dtype=0)
    assert mb.mebptt_workspace_bytes(with_stage) == mb.mebptt_workspace_bytes(mb.make_desc(64, 256, 1024, 5, 1, 0, 1, 0))
    assert mb.mebptt_workspace_bytes(with_stage) > 48 << 20 and without is not None


def test_size_queries():
    d = mb.make_desc(64, 256, 1024, 1000, 1, 0, 1)
    unit = 2 * 64 * 1024 * 4
    assert mb.mebptt_unit_bytes(d) == unit
    p = mb.mebptt_plan(1000, 50, mb.HSM)
    assert mb.mebptt_slot_pool_bytes(d, p) == 50 * unit
    p = mb.mebptt_plan(1000, 100, mb.ISM)
    assert mb.mebptt_slot_pool_bytes(d, p) == 100 * 4 * unit
    ws = mb.mebptt_workspace_bytes(d)
    assert 0 < ws < 192 << 20          # operand copies, chunk buffers of the batched GEMMs, recomputation stage (<= 48 MiB)
    # independent of t
    assert mb.mebptt_workspace_bytes(mb.make_desc(64, 256, 1024, 7, 1, 0, 1)) == ws
    assert mb.mebptt_units_for_bytes(d, mb.MSM, 4_000_000_000) == 4_000_000_000 // unit
    assert mb.mebptt_units_for_bytes(d, mb.ISM, 4_000_000_000) == 4_000_000_000 // (4 * unit)
    assert mb.mebptt_units_for_bytes(d, mb.HSM, unit - 1) == 0
    assert mb.mebptt_workspace_bytes(mb.make_desc(0, 256, 1024, 7, 1, 0, 1)) == 0


def test_dense_chain_workspace_holds_two_activations_and_two_gradients():
    desc = mb.make_chain_desc([70, 2047, 65], 510, 4096)
    slab = (510 * 2047 * 4 + 255) // 256 * 256
    assert mb.mebptt_chain_workspace_bytes(desc) == 4 * slab


def _round_up(v, n):
    return (v + n - 1) // n * n


def _wide_operands_fit(desc):
    """The arrays that the launches with weights spread over several XCDs address by 32-bit byte offsets -- the gate weights and
    the two transposed operands of the weight gradient -- below 2 GiB, and x of one step within its staging."""
    KX, KH, NX = _round_up(desc.I, 32), _round_up(desc.H, 32), _round_up(desc.I, 16)
    KC = _round_up(mb.mebptt_chunk_steps(desc) * desc.B, 32)
    largest = max(4 * KH * (KX + KH) * 2, (NX + KH + 16) * KC * 2, 4 * KH * KC * 2)
    return largest < 1 << 31 and _round_up(desc.B, 16) * KX * 2 <= 32 << 20


def test_launches_that_address_by_32_bits_are_not_used_beyond_them():
    """Inputs so wide that an operand reaches 2 GiB are accepted, and run by the launch-per-step kernels, whose offsets are
    64 bits wide.  (The recomputation stage is there exactly where the other launches are: these shapes have no copy of the weights
    per XCD.)"""
    for B, H in ((32, 4096), (9, 2100), (128, 2048), (70, 1056), (16, 1100), (200, 1024), (129, 600)):
        def desc(I):
            return mb.make_desc(B, I, H, 10, 1, 0, 1, 0)
        lo, hi = 64, (1 << 31) // (4 * H) - H                     # hi: the widest input that is accepted
        assert _wide_operands_fit(desc(lo)) and not _wide_operands_fit(desc(hi))
        while hi - lo > 1:
            mid = (lo + hi) // 2
            if _wide_operands_fit(desc(mid)):
                lo = mid
            else:
                hi = mid
        assert mb.mebptt_stage_steps(desc(lo)) > 0 and mb.mebptt_stage_steps(desc(hi)) == 0, (B, H, lo)
        for I in (2 * hi, 3 * hi, (1 << 31) // (4 * H) - H):
            if 4 * H * (I + H) <= 1 << 31:
                assert mb.mebptt_stage_steps(desc(I)) == 0 and mb.mebptt_workspace_bytes(desc(I)) > 0, (B, H, I)


def test_small_batches_of_very_wide_inputs_have_no_wide_launches():
    """The line beyond which streaming the input's weights through them is slower than a launch per step."""
    def stage(B, I, H):
        return mb.mebptt_stage_steps(mb.make_desc(B, I, H, 10, 1, 0, 1, 0))
    for B, H in ((1, 2048), (16, 1281), (9, 1600), (17, 2048), (32, 1537 + 127), (32, 1770)):
        assert stage(B, 4096, H) > 0 and stage(B, 4097, H) == 0
    for B, H in ((33, 2048), (16, 1280), (32, 1536), (32, 1600), (20, 2000), (32, 2049), (130, 1000)):
        assert stage(B, 4097, H) > 0 and stage(B, 30000, H) > 0


def _common_workspace_bytes(desc):
    """What the workspace of a bf16 LSTM holds on any shape, without the weight-gradient accumulator (which does not depend on B)."""
    KX, KH, NX, BP = _round_up(desc.I, 32), _round_up(desc.H, 32), _round_up(desc.I, 16), _round_up(desc.B, 16)
    G4, CH = 4 * KH, mb.mebptt_chunk_steps(desc)
    KC = _round_up(CH * desc.B, 32)
    weights = 2 * G4 * (KX + KH) + 4 * G4 + 2 * KH * G4 + 2 * NX * G4
    return (weights + 9 * mb.mebptt_unit_bytes(desc) + 4 * desc.B * desc.H
            + 2 * 2 * (CH * BP * G4 + G4 * KC + (NX + KH + 16) * KC))


def test_staged_input_of_a_launch_is_at_most_32_mib():
    """Chain launches with weights spread over several XCDs read x of all their steps as operands from the workspace: as
    many steps as 32 MiB hold.  Seen in the workspace of the largest such batch, against that of a batch one larger, which has no
    resident launches."""
    for B, H, groups, nr in ((128, 2048, 2, 4), (256, 1024, 4, 4)):
        for I in (512, 8192, 16384, 30000, 60000):
            d, beyond = mb.make_desc(B, I, H, 10, 1, 0, 1, 0), mb.make_desc(B + 1, I, H, 10, 1, 0, 1, 0)
            assert mb.mebptt_stage_steps(d) > 0 and mb.mebptt_stage_steps(beyond) == 0
            more = (mb.mebptt_workspace_bytes(d) - _common_workspace_bytes(d)
                    - mb.mebptt_workspace_bytes(beyond) + _common_workspace_bytes(beyond))
            part = groups * (H // (16 * nr)) * 16 * (4 * nr * 64) * 4
            rings = 8 * B * H * 2 + 8 * B * 4 * H * 2 + 4 * part + 4 * B * H
            staged = more - rings - 3 * mb.mebptt_unit_bytes(d) * mb.mebptt_stage_steps(d)
            step = B * _round_up(I, 32) * 2
            assert abs(staged - min(192, (32 << 20) // step) * step) < 8192 and staged < (32 << 20) + 8192, (B, I, H, staged)


def test_static_workspace_takes_the_shapes_it_took():
    """Shapes whose workspace fits the static array as long as the weight gradient has no more accumulators than 1.5 workgroups per
    compute unit need: a plan that splits K further would have them refused.  (Without a device, and without arrays, what comes
    back is another error.)"""
    import torch
    plan = mb.mebptt_plan(8, 3, mb.HSM)

    def refused(B, I, H, dtype):
        args = [mb.make_desc(B, I, H, 8, dtype, 1, 1, 0), plan] + [None] * 7 + [torch.zeros(0)] + [None] * 7
        with pytest.raises(mb.MebpttError) as e:
            mb.mebptt_run_static(*args, stream=0)
        return e.value.code == mb.EWORKSPACE
    for shape in ((2, 319, 317, 1), (2, 307, 291, 1), (1, 314, 311, 1), (1, 307, 307, 1), (4, 1494, 141, 1), (2, 1204, 170, 1)):
        assert not refused(*shape), shape
    assert refused(64, 256, 1024, 1)
