"""How score calls are split into key chunks (host only, nothing is launched)."""
import pytest

from score_layout import CHUNK_CASES, chunk_dims, fuses, layout
import paper_2609_04971_amd as bkv


@pytest.mark.parametrize("case", CHUNK_CASES, ids=lambda c: "-".join(map(str, c[:7])))
def test_chunk_cases_are_what_they_are_meant_to_be(case):
    L = layout(chunk_dims(case), mean=case[7])
    assert (L.groups, L.key_chunk, L.nch, L.in_scores) == case[9:]


def test_chunks_cover_the_head_and_their_statistics_fit():
    # every form of the rule, over sizes, rows and head counts: the chunks cover
    # the head, none is empty, none longer than the kernels' LDS holds, and the
    # statistics fit the workspace or, per head, the room of its scores
    for P in (1, 2, 7, 36, 61, 64, 65, 200, 513, 5000):
        for N in (1, 33, 255, 256, 257, 1151, 1153, 1665, 4224, 6657, 16384, 29999, 65536):
            if P * N > 1 << 25:
                continue
            for R in (1, 16, 40, 80, 96, 144, 145, 192, 288, 384, 464, 576, 1024):
                for mean in (False, True):
                    d = bkv.dims(B=P, Hq=1, Hkv=1, D=128, N=N, W=R, C=0, budget=R, dtype="bf16")
                    L = layout(d, mean)
                    at = (P, N, R, mean, L.key_chunk, L.nch)
                    assert L.key_chunk % 128 == 0 and 0 <= L.nch * L.key_chunk - N < L.key_chunk, at
                    assert L.key_chunk <= (1664 if L.groups == 1 else 1152), at
                    assert L.nch <= L.nch_ws or 2 * L.nch * L.R_pad_max <= N, at
                    other = layout(d, not mean)  # one workspace serves both forms
                    assert (L.evict_end, L.part_z, L.lse2) == (other.evict_end, other.part_z, other.lse2), at
                    # the fused launch reads its own scores back: its statistics stay in the workspace
                    assert not (fuses(d) and other.in_scores), at


@pytest.mark.parametrize("P,N,R,budget,dtype,want", [
    (128, 32768, 144, 4096, "bf16", True), (33, 32768, 24, 4096, "bf16", True), (32, 32768, 24, 4096, "bf16", False),
    (53, 20000, 80, 2500, "bf16", True), (52, 20000, 80, 2500, "bf16", False), (60, 19999, 80, 2500, "bf16", False),
    (98, 15361, 16, 2048, "bf16", True), (97, 15361, 16, 2048, "bf16", False), (256, 15360, 16, 2048, "bf16", False),
    (128, 32769, 144, 4096, "bf16", False), (128, 32768, 145, 4096, "bf16", False), (128, 32768, 144, 16384, "bf16", True),
    (128, 32768, 144, 16385, "bf16", False), (128, 32768, 144, 4096, "fp32", False)])
def test_where_the_eviction_is_one_launch(P, N, R, budget, dtype, want):
    assert fuses(bkv.dims(B=P, Hq=1, Hkv=1, D=128, N=N, W=R, C=0, budget=budget, dtype=dtype)) == want
