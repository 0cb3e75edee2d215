"""Long linear-attention calls run in segments of the sequence, short ones in
one pass; the route follows from the sizes and never changes a bit.  Each case
computes one long call and the same tokens in 64-token calls that hand the
state on, and compares o, every chunk state and the final state bit for bit;
o also against the token recurrence of the oracle."""
import pytest
import torch

import paper_2606_20537_amd as cap
from gpu_util import SPLIT_TOL, dev_inputs, rel_err, scan_case

pytestmark = pytest.mark.gpu

CASES = [
    # (T, H, dk, dv, dtype, chunk states, entering state)
    (1024, 1, 128, 128, "bf16", False, True),    # the first segmented length, whole chunks
    (1025, 3, 128, 16, "bf16", False, True),     # a one-token tail, hand-over rows short of dk
    (1151, 2, 128, 48, "bf16", False, False),    # 63-token tail; a wave without columns
    (1087, 2, 128, 80, "bf16", True, True),      # a second column group of 16
    (1600, 5, 128, 256, "bf16", True, False),    # row blocks of 64, four column groups
    (2049, 9, 128, 176, "bf16", False, True),    # 2049 x 9 heads x 11 slices: below 128 slices
    (4161, 20, 128, 128, "bf16", False, True),   # heads not a multiple of 8, whole-head row blocks
    (6200, 32, 128, 256, "bf16", False, True),   # 128-column workgroups, more slices than CUs
    (1024, 2, 64, 64, "bf16", True, True),
    (1100, 16, 64, 96, "bf16", False, True),
    (512, 2, 64, 64, "f32", True, True),         # fp32: the first segmented length
    (577, 3, 64, 112, "f32", False, True),
    (1600, 16, 64, 128, "f32", False, False),
]


@pytest.mark.parametrize("T,H,dk,dv,dtype,states,with_s0", CASES, ids=["%d_%d_%d_%d_%s" % c[:5] for c in CASES])
def test_segments_equal_single_chunks(orc, T, H, dk, dv, dtype, states, with_s0):
    print("case", T, H, dk, dv, dtype, flush=True)
    inp = scan_case(300 + T + H, T, H, dk, dv, dtype)
    d = dev_inputs(inp)
    kind = cap.CAP_DTYPE_F32 if dtype == "f32" else cap.CAP_DTYPE_BF16
    gen = torch.Generator(device="cuda").manual_seed(T)
    s0 = torch.randn((H, dk, dv), generator=gen, device="cuda") if with_s0 else None
    n, nan = (T + 63) // 64, float("nan")

    def buffers():
        return (torch.full((T, H, dv), nan, device="cuda"), torch.full((n, H, dk, dv), nan, device="cuda"),
                torch.full((H, dk, dv), nan, device="cuda") if s0 is None else s0.clone())

    o, cs, fs = buffers()  # the state is updated in place where there is one
    cap.linattn_chunked_prefill(d["q"], d["k"], d["v"], d["g"], o, state_in=None if s0 is None else fs,
                                chunk_states=cs if states else None, final_state=fs, in_dtype=kind)
    o1, cs1, fs1 = buffers()
    for c in range(n):
        t0, t1 = 64 * c, min(64 * c + 64, T)
        cap.linattn_chunked_prefill(d["q"][t0:t1], d["k"][t0:t1], d["v"][t0:t1], d["g"][t0:t1], o1[t0:t1],
                                    state_in=None if c == 0 and s0 is None else fs1, chunk_states=cs1[c:],
                                    final_state=fs1, T=t1 - t0, H=H, dk=dk, dv=dv, in_dtype=kind)
    o2 = torch.full((T, H, dv), nan, device="cuda")
    cap.linattn_chunked_prefill(d["q"], d["k"], d["v"], d["g"], o2, state_in=s0, in_dtype=kind)
    torch.cuda.synchronize()
    assert torch.equal(o, o1) and torch.equal(fs, fs1)
    assert not states or torch.equal(cs, cs1)
    assert torch.equal(o2, o)  # neither a final state nor chunk states wanted
    if T * H <= 12000:
        o_ref, _ = orc.sequential(inp["q"], inp["k"], inp["v"], inp["g"], S0=None if s0 is None else s0.cpu().numpy())
        assert rel_err(o.cpu().numpy(), o_ref) <= SPLIT_TOL
