"""vsh_generate_into adds to the caller's histogram by plain loads and stores,
whatever the size of the call: a histogram in pinned host memory, which
hardware FP64 atomics do not reach, receives what one in device memory does.
Entries are counts (exact); the sums of weights agree within the order of
their additions: n terms of one sign, each rounded to 2^-53 relative, either
side, and once more per call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


SIZES = [(1, 64), (100, 64), (5003, 64), (16_385, 256), (32_768, 64), (32_769, 64)]


@pytest.mark.parametrize("fixed", [False, True])
@pytest.mark.parametrize("form,n,cap", [(form, n, cap) for n, cap in SIZES for form in ("plain", "batched", "static")
                                        if form != "static" or n <= 5003])  # the static workspace holds 10^4
def test_histogram_in_host_memory(form, n, cap, fixed):
    import torch

    import paper_2403_08692_amd as P

    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    with P.Context(0) as ctx:
        flags = (P.VSH_FORM_PERSISTENT if form == "batched" else P.VSH_FORM_PLAIN) | \
            (P.VSH_HIST_FIXEDPOINT if fixed else 0)
        req, _ = P.make_request(n, 9, 0, 91.2, 1.0, cap, flags)
        size = ctx.workspace_size(req)
        ws = torch.empty(size, dtype=torch.uint8, device=dev)
        hists = [torch.full((P.HIST_DOUBLES,), 2.0, dtype=torch.float64, device=dev),
                 torch.full((P.HIST_DOUBLES,), 2.0, dtype=torch.float64, pin_memory=True)]
        for h in hists:
            print(f"case histogram form={form} n={n} cap={cap} fixed={fixed} on {h.device}", flush=True)
            for _ in range(2):  # accumulated into
                if form == "static":
                    ctx.generate_into_static(req, stream, h.data_ptr())
                else:
                    ctx.generate_into(req, stream, ws.data_ptr(), size, h.data_ptr())
            torch.cuda.synchronize()
        a, b = (h.cpu().numpy().reshape(P.NOBS, P.NHCOL, 3) for h in hists)
    np.testing.assert_array_equal(a[..., 2], b[..., 2])
    assert ((a[..., 2] - 2.0).sum(axis=1) >= 2 * 0.999 * n).all()  # both calls' events are there
    np.testing.assert_allclose(a, b, rtol=2 * (n + 2) * 2.0 ** -53, atol=0)
