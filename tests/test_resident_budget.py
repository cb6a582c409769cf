"""Registers of the kernels whose workgroups wait for each other, from the built library: a compute unit that holds as many
of their workgroups as are counted on must still have room for the waves that wait for room (amq_resident.h), or such a
wave could sit where a grid that has its room already needs to go."""
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SIMD_REGISTERS = 512   # per lane, both kinds together
WAITERS = 4            # hardware queues of a process: at most that many kernels wait, all on one SIMD at worst


def kernels():
    """Name -> metadata of every kernel in the library's code objects."""
    msgpack = pytest.importorskip("msgpack")
    from paper_1802_00150_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    blob = open(build.LIB, "rb").read()
    found = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        n, = struct.unpack_from("<Q", blob, m.end())
        at = m.end() + 8
        if n > 16:
            continue  # (the word by itself, no bundle)
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", blob, at)
            target = blob[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in target:
                continue
            code = blob[m.start() + offset:m.start() + offset + size]
            for note in re.finditer(b"AMDGPU\0\0", code):
                namesz, descsz, kind = struct.unpack_from("<III", code, note.start() - 12)
                if namesz == 7 and kind == 32:
                    meta = msgpack.unpackb(code[note.end():note.end() + descsz])
                    found.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
    return found


@pytest.fixture(scope="module")
def registers():
    """Kernel name -> registers a wave is given (handed out in eights)."""
    return {name: (k[".vgpr_count"] + 7) // 8 * 8 for name, k in kernels().items()}


def test_large_steps_spill_nothing():
    # recurrent steps with several tiles per wave, every number of bits (amq_mfma4w.hip)
    hits = {n: k for n, k in kernels().items() if "14mfma4wc_kernel" in n}
    assert len(hits) == 38, sorted(hits)
    for name, k in hits.items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, (name, k[".vgpr_spill_count"])


def test_large_products_spill_little():
    # several tiles per wave (amq_mfma4w.hip): a few coefficients where 96 accumulators are held, no operands
    hits = {n: k for n, k in kernels().items() if "13mfma4w_kernel" in n}
    assert len(hits) == 74, sorted(hits)
    for name, k in hits.items():
        assert k[".vgpr_spill_count"] <= 8, (name, k[".vgpr_spill_count"])


def of(registers, pattern, count):
    hits = {k: v for k, v in registers.items() if re.search(pattern, k)}
    assert len(hits) == count, sorted(hits)
    return hits


def test_waiting_kernels_hold_few_registers(registers):
    for name, r in of(registers, "seq[gw]_reset_kernel", 2).items():
        assert r <= 8, (name, r)


def test_room_for_waiting_kernels_beside_a_full_claim(registers):
    # one workgroup of 8 waves per compute unit: two waves on every SIMD
    for name, r in of(registers, "11seqw_kernel", 36).items():
        assert 2 * r + WAITERS * 8 <= SIMD_REGISTERS, (name, r)


def test_room_for_waiting_kernels_beside_light_claims(registers):
    # three workgroups of 4 waves per compute unit: three waves on every SIMD
    for name, r in of(registers, "16lstm_seqg_kernel", 4).items():
        assert 3 * r + WAITERS * 8 <= SIMD_REGISTERS, (name, r)


def test_room_for_waiting_kernels_beside_single_sequences(registers):
    # one workgroup of 4 waves per compute unit: a wave on every SIMD
    for name, r in of(registers, "11seq1_kernel", 104).items():
        assert r + WAITERS * 8 <= SIMD_REGISTERS, (name, r)


def test_room_for_waiting_kernels_beside_light_single_sequences(registers):
    # (four waves quantize together, one unit per lane: the forms whose claim is light) three workgroups of 4 waves per unit
    for name, r in of(registers, r"11seq1_kernelI(Li\dE){3}Li4ELi\dELi1E", 16).items():
        assert 3 * r + WAITERS * 8 <= SIMD_REGISTERS, (name, r)


def test_room_for_waiting_kernels_beside_tiled_sequences(registers):
    # one workgroup of 8 waves per compute unit, as amq_seqw.hip
    for name, r in of(registers, "17seqw_tiles_kernel", 12).items():
        assert 2 * r + WAITERS * 8 <= SIMD_REGISTERS, (name, r)


def test_room_for_waiting_kernels_beside_sequences_with_long_inputs(registers):
    # one workgroup of 8 waves per compute unit, as the other kernel of amq_seqw.hip
    for name, r in of(registers, "17seqw_apart_kernel", 18).items():
        assert 2 * r + WAITERS * 8 <= SIMD_REGISTERS, (name, r)
