"""The pass of csrc/gen_dispatch.py that moves a block's weights to vector registers, executed on
the wavefront model (tests/gcn_model.py) in place of the program it rewrites, against the oracle.
The moves are given to the model as additions of a zero register."""

import numpy as np
import pytest

import gcn_model
import test_interpreter_model as tim
from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl


class VectorWave(gcn_model.Wave):
    def __init__(self, *a):
        super().__init__(*a)
        self.v["zero"] = np.zeros(gcn_model.WAVE, np.uint32)

    def rd32(self, a):
        key = self.vkey(a)
        if key in self.v:                    # a weight: the same value in every lane
            v = self.vreg(a)
            assert (v == v[0]).all()
            return int(v[0])
        return super().rd32(a)


@pytest.mark.parametrize("c_out,c_in,n,h,w,ck,patterns", [(8, 6, 1, 7, 16, 6, 8), (11, 9, 1, 9, 18, 4, 8), (8, 16, 1, 7, 16, 8, 56)])
def test_weights_in_vector_registers(oracle, monkeypatch, c_out, c_in, n, h, w, ck, patterns):
    import gen_dispatch
    plain = gen_dispatch.program

    def shipped(*key):
        lines, g = plain(*key)
        assert g["vector"]
        lines = gen_dispatch.vector_weights(lines, g)
        assert not any(l.startswith("v_fmac") and ", s" in l for l in lines)
        return [l.replace("v_mov_b32", "v_add_u32") + ", %[zero]" if l.startswith("v_mov_b32") else l for l in lines], g

    monkeypatch.setattr(gen_dispatch, "program", shipped)
    monkeypatch.setattr(gcn_model, "Wave", VectorWave)
    monkeypatch.setattr(tim, "_programs", {})
    rng = np.random.default_rng(c_out + c_in)
    lib = wl.pattern_library(wl.PATTERN_SEED) if patterns < 56 else wl.pattern_universe()
    d = {"weights": rng.standard_normal((c_out, c_in, 3, 3)).astype(np.float32), "pattern_masks": lib,
         "pattern_ids": rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8),
         "kernel_mask": (rng.random((c_out, c_in)) < 0.5).astype(np.uint8),
         "bias": rng.standard_normal(c_out).astype(np.float32)}
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    name = "t_g8_p7x2_s1_x8_thw1b"
    assert name in [B.patdnn_variant_name(v) for v in range(B.patdnn_num_variants())]
    tim._check(oracle, d, x, ck, only=(name,))


def test_blocks_fill_their_slots():
    """Blocks lie where the encoder's offsets put them, and those of the largest variant close to each
    other: the instruction cache has to hold what a layer's patterns use."""
    import gen_dispatch
    from paper_2001_00138_amd import buildlib
    for key in buildlib.sparse_geometries():
        lines, g = gen_dispatch.program(*key)
        if g["vector"]:
            lines = gen_dispatch.vector_weights(lines, g)
        starts = [i for i, l in enumerate(lines) if l.startswith(".Lblk")]
        table = starts[-g["sets"] * key[0] * 56:]
        for a, b in zip(table, table[1:]):
            code = 4 * sum(not l.startswith(".") for l in lines[a:b])      # instructions of four bytes all
            assert lines[b - 1] == f".org {lines[a][:-1]}+{g['block_bytes']}"
            assert 0 <= g["block_bytes"] - code < (16 if g["vector"] else g["block_bytes"] // 2)
        assert g["table_off"] % 512 == 0
