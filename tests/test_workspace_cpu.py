"""Sizes of the training workspace (lst_mlp_workspace_bytes), on the CPU."""
import paper_2209_13711_amd as lst
from synth import weights as W


def test_workspace_holds_the_chunks_that_are_used():
    """64 rows a chunk: up to 4096 rows no more than 64 chunks, above 128; it
    never shrinks with more rows"""
    size = lst.load_library().lst_mlp_workspace_bytes
    last = 0
    for n in [0, 1, 64, 65, 4095, 4096, 4097, 5000, 8192, 8193, 200003]:
        chunks = 64 if n <= 4096 else 128
        assert size(n) == 4 * (n + chunks * W.N_PARAM), n
        assert size(n) >= last
        last = size(n)
    assert size(-1) == 0
