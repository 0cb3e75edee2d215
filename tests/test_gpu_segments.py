"""Long linear-attention calls run in segments of the sequence, short ones in
one pass; the route follows from the sizes and never changes a bit.  Each case
computes one long call and the same tokens in 64-token calls that hand the
state on, and compares o, every chunk state and the final state bit for bit;
o also against the token recurrence of the oracle.  The plan of each case is
checked on the host (test_launch_rules.py), so that none runs in one pass."""
import pytest
import torch

import paper_2606_20537_amd as cap
from gpu_util import SPLIT_TOL, dev_inputs, rel_err, scan_case

pytestmark = pytest.mark.gpu

CASES = [
    # (T, H, dk, dv, dtype, chunk states, entering state, (columns per workgroup, segments, chunks in each))
    (1024, 1, 128, 128, "bf16", False, True, (64, 8, 2)),         # the first segmented length, whole chunks
    (1665, 3, 128, 16, "bf16", False, True, (64, 13, 2)),         # a one-token tail, hand-over rows short of dk
    (1791, 2, 128, 48, "bf16", False, False, (64, 13, 2)),        # 63-token tail; a wave without columns
    (1087, 2, 128, 80, "bf16", True, True, (64, 17, 1)),          # a second column group of 16
    (1800, 5, 128, 256, "bf16", True, False, (64, 15, 2)),        # row blocks of 64, four column groups
    (2049, 9, 128, 176, "bf16", False, True, (64, 16, 2)),        # 9 heads x 11 slices: below 128 slices
    (6200, 20, 128, 128, "bf16", False, True, (64, 11, 9)),       # heads not a multiple of 8, whole-head row blocks
    (6200, 32, 128, 256, "bf16", False, True, (128, 8, 13)),      # 128-column workgroups, more slices than CUs
    (1024, 2, 64, 64, "bf16", True, True, (64, 16, 1)),
    (3160, 16, 64, 96, "bf16", False, True, (64, 13, 4)),         # hand-over in o at dk 64
    (512, 2, 64, 64, "f32", True, True, (64, 8, 1)),              # fp32: the first segmented length
    (833, 3, 64, 112, "f32", False, True, (64, 13, 1)),           # a one-token tail
    (2780, 16, 64, 128, "f32", False, False, (64, 15, 3)),        # several chunks a segment
]
# inputs made on the device, o compared with the single chunks only
LARGE = [
    (12325, 16, 128, 128, "bf16", True, True, (128, 28, 7)),      # 128-column workgroups with chunk states
    (9850, 10, 128, 176, "bf16", True, False, (128, 22, 7)),      # the same, columns short of the second group
    (6200, 32, 128, 176, "bf16", False, True, (128, 8, 13)),      # without chunk states
    (6200, 64, 128, 80, "bf16", False, True, (128, 8, 13)),       # one column group, not whole
    (3100, 64, 64, 144, "bf16", False, False, (128, 4, 13)),      # 128-column workgroups at dk 64
    (2050, 257, 128, 64, "bf16", False, True, (64, 1, 33)),       # one segment: no first launch, the state updated in place
    (3100, 264, 64, 128, "bf16", False, True, (128, 1, 49)),      # the same at dk 64 with 128-column workgroups
]
IDS = "%d_%d_%d_%d_%s"


@pytest.mark.parametrize("T,H,dk,dv,dtype,states,with_s0,plan", CASES, ids=[IDS % c[:5] for c in CASES])
def test_segments_equal_single_chunks(orc, T, H, dk, dv, dtype, states, with_s0, plan):
    print("case", T, H, dk, dv, dtype, flush=True)
    inp = scan_case(300 + T + H, T, H, dk, dv, dtype)
    o, s0 = compare(dev_inputs(inp), T, H, dk, dv, dtype, states, with_s0)
    if T * H <= 12000:
        o_ref, _ = orc.sequential(inp["q"], inp["k"], inp["v"], inp["g"], S0=None if s0 is None else s0.cpu().numpy())
        assert rel_err(o.cpu().numpy(), o_ref) <= SPLIT_TOL


@pytest.mark.parametrize("T,H,dk,dv,dtype,states,with_s0,plan", LARGE, ids=[IDS % c[:5] for c in LARGE])
def test_large_segments_equal_single_chunks(T, H, dk, dv, dtype, states, with_s0, plan):
    print("case", T, H, dk, dv, dtype, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + H)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    d = {n: torch.nn.functional.normalize(randn(T, H, dk), dim=-1).bfloat16() for n in ("q", "k")}
    d["v"], d["g"] = randn(T, H, dv).bfloat16(), torch.nn.functional.logsigmoid(3 + randn(T, H))
    compare(d, T, H, dk, dv, dtype, states, with_s0)


@pytest.mark.parametrize("states", [False, True])
def test_segments_in_a_graph(states):
    """Both launches recorded in one graph: every replay, on new inputs and with
    eager work in between, equals the eager call."""
    T, H, dk, dv = 1800, 3, 128, 48
    gen = torch.Generator(device="cuda").manual_seed(5)

    def tokens():
        q, k = (torch.nn.functional.normalize(torch.randn((T, H, dk), generator=gen, device="cuda"), dim=-1).bfloat16()
                for _ in range(2))
        return [q, k, torch.randn((T, H, dv), generator=gen, device="cuda").bfloat16(),
                torch.nn.functional.logsigmoid(3 + torch.randn((T, H), generator=gen, device="cuda"))]

    def outputs():
        return [torch.full(s, float("nan"), device="cuda") for s in ((T, H, dv), (H, dk, dv), ((T + 63) // 64, H, dk, dv))]

    def call(x, out):
        cap.linattn_chunked_prefill(*x, out[0], final_state=out[1], chunk_states=out[2] if states else None)

    x, out = tokens(), outputs()
    call(x, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, out)
    for _ in range(3):
        for a, b in zip(x, tokens()):
            a.copy_(b)
        want = outputs()
        call(x, want)
        for t in out:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out[:2 + states], want))


def compare(d, T, H, dk, dv, dtype, states, with_s0):
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
    return o, s0
