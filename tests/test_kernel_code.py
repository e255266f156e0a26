"""What the compiler made of the kernels: properties of the device code that the
kernels' speed rests on and that a small change of the source can lose."""

import re

import pytest

import code_objects


def _vector_products_read_back(body):
    """v_readfirstlane of a value that a vector multiply (or a choice of one) made shortly before."""
    found = []
    made = {}  # VGPR -> index of the instruction that made it a product
    for i, line in enumerate(body):
        op, _, args = line.partition(" ")
        regs = [r.strip() for r in args.split(",")]
        if op == "v_readfirstlane_b32":
            if i - made.get(regs[1], -99) < 16:
                found.append(line)
        elif op.startswith("v_") and regs:
            if op == "v_mul_lo_u32" or any(i - made.get(r, -99) < 16 for r in regs[1:]):
                made[regs[0]] = i
            else:
                made.pop(regs[0], None)
    return found


@pytest.mark.parametrize("seg", [4, 8, 16, 32, 64])
def test_streaming_step_offsets_are_scalar(seg):
    """A step's row offsets are products of uniform values: scalar multiplies, not vector
    ones (quarter rate) whose result is read back into a scalar register."""
    bodies = code_objects.disassembly(rf"bitcos_(fast|diag)_kernel<\d+, {seg}, ")
    assert len(bodies) >= 2 * (16 + 8) * 2
    bad = {name: found for name, body in bodies.items() if (found := _vector_products_read_back(body))}
    assert not bad, f"{len(bad)} of {len(bodies)} kernels, e.g. {next(iter(bad.items()))}"


def test_bitcos_kernels_do_not_spill():
    """Every instantiation of the default layout's kernels keeps its state in registers: a
    spilled scalar register is read back with a vector instruction inside the step loop, and
    a spilled activation load is waited for before its data is needed."""
    found = {name: (k[".sgpr_spill_count"], k[".vgpr_spill_count"]) for name, k in code_objects.kernels().items()
             if re.search(r"bitcos_(fast|diag|mfma)_kernel<", name)}
    assert len(found) > 500
    spilled = {name: n for name, n in found.items() if any(n)}
    assert not spilled, f"{len(spilled)} of {len(found)} kernels: {sorted(spilled.items())[:5]}"


def test_light_2bit_int8_kernels_start_without_lds():
    """2-bit kernels with int8 activations of a few words a lane hold nothing in LDS and
    wait at no barrier: each wave starts by itself."""
    ks = code_objects.kernels()
    light = {n: k for n, k in ks.items() if (m := re.search(r"bit2_gemv_kernel<(\d+), \d+, false, (true|false)>", n))
             and int(m.group(1)) < (6 if m.group(2) == "true" else 4)}
    assert len(light) == 5 * (5 + 3)
    held = {n: k[".group_segment_fixed_size"] for n, k in light.items() if k[".group_segment_fixed_size"]}
    assert not held, f"{len(held)} of {len(light)}: {sorted(held.items())[:3]}"


def test_2bit_int8_steps_do_not_wait_for_the_last_store():
    """A batch's 2-bit int8 step waits for its words where it masks them, so nothing in front of
    the next step's loads waits for all memory accesses (the last step's store is among them)."""
    bodies = code_objects.disassembly(r"bit2_gemv_kernel<(8|12|16), 64, false, true>")
    assert len(bodies) == 3
    waits = {}
    for name, body in bodies.items():
        at = body.index("s_setprio 1")
        while not body[at].startswith("buffer_load"):
            at -= 1
        while any(line.startswith("buffer_load") for line in body[at - 16:at]):  # the step's first load
            at -= 1
        waits[name] = [line for line in body[at - 60:at] if line.startswith("s_waitcnt") and "vmcnt(0)" in line]
    assert not any(waits.values()), waits
