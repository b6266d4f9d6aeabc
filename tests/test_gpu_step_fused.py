"""The step's quantisation and scan in one launch (no flush, up to 256 blocks of 1024 keys, 512 at 64 dimensions,
groups of up to 4 heads) against the two launches it replaces (the separate calls): bitwise, at the edges of its blocks and of its range."""
import pytest
import torch

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,D,n,compact", [
    (1, 1, 1, 128, 1, False), (1, 4, 1, 128, 255, True), (3, 2, 1, 64, 257, False), (1, 8, 8, 128, 513, True),
    (2, 32, 8, 128, 4096, False),      # 256 blocks of one key per lane
    (2, 32, 8, 128, 4097, False),      # two keys per lane
    (2, 32, 8, 64, 8193, True),        # four
    (4, 16, 8, 128, 8192, False),      # 256 blocks: the largest
    (4, 16, 8, 128, 8193, False),      # past it: two launches
    (8, 16, 8, 64, 8192, False),       # 512 blocks at 64 dimensions
    (8, 16, 8, 64, 8193, False),
    (1, 8, 1, 128, 3000, False),       # a group of 8: two launches
    (70, 8, 8, 64, 31, False),         # more groups than blocks allowed: two launches
])
def test_same_as_the_separate_calls(B, Hq, Hkv, D, n, compact):
    from paper_2606_31519_amd import pipeline
    wl = gen.random_case(B, Hq, Hkv, n, D=D, seed=n, kv_dtype="bf16", w=5, c_q_scale=0.0 if compact else 0.5)
    st = pipeline.DecodeState.from_workload(wl, compact=compact)
    st.build_index()
    got = {}
    for name, step in (("calls", st.step_calls), ("step", st.step)):
        for t in (st.qplanes, st.qscal, st.scores, st.out):
            t.zero_()
        step(0.9, flush=False)
        torch.cuda.synchronize()
        got[name] = [t.clone() for t in (st.qplanes, st.qscal, st.scores, st.sel_count, st.out, st.lse)]
    for x, y in zip(got["calls"], got["step"]):
        assert torch.equal(x, y)
