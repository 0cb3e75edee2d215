"""Head counts that 8 does not divide: the scans and the decode steps place a
head's workgroups by head count, and every head must still get all its
workgroups exactly once -- each head of a call equals, bit for bit, the same
head computed in a call of its own."""
import pytest
import torch

import paper_2606_20537_amd as cap

pytestmark = pytest.mark.gpu


# 20 x 176, 17 x 192: by XCD the slices of three heads, 33 or 36, would not fit 32 CUs
@pytest.mark.parametrize("H,dv", [(8, 48), (10, 48), (11, 48), (12, 48), (17, 48), (31, 48), (20, 176), (17, 192)])
@pytest.mark.parametrize("T", [1, 130])
@pytest.mark.parametrize("mixer", ["linattn", "gdn"])
def test_every_head_alone(mixer, T, H, dv):
    print("case", mixer, T, H, dv, flush=True)
    dk, nan = 128, float("nan")
    gen = torch.Generator(device="cuda").manual_seed(100 * T + H)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    q, k = (torch.nn.functional.normalize(randn(T, H, dk), dim=-1).bfloat16() for _ in range(2))
    v, s0 = randn(T, H, dv).bfloat16(), randn(H, dk, dv)
    gates = [torch.nn.functional.logsigmoid(3 + randn(T, H))] + ([torch.sigmoid(randn(T, H))] if mixer == "gdn" else [])
    fns = [getattr(cap, mixer + "_chunked_prefill")] + ([getattr(cap, mixer + "_decode_step")] if T == 1 else [])
    for fn in fns:
        o, fs = torch.full((T, H, dv), nan, device="cuda"), torch.full((H, dk, dv), nan, device="cuda")
        fn(q, k, v, *gates, o, state_in=s0, final_state=fs)
        for h in range(H):
            one = slice(h, h + 1)
            oh, fh = torch.full((T, 1, dv), nan, device="cuda"), torch.full((1, dk, dv), nan, device="cuda")
            fn(*(x[:, one].clone(memory_format=torch.contiguous_format) for x in (q, k, v, *gates)), oh, state_in=s0[one].clone(), final_state=fh)
            torch.cuda.synchronize()
            assert torch.equal(o[:, one], oh) and torch.equal(fs[one], fh), (fn.__name__, h)
