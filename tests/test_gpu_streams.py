"""The binding's default stream: calls go to torch's current stream of the
current device, also inside a stream context and on another thread."""
import threading

import numpy as np
import pytest
import torch

import synth
from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def test_default_stream_is_torchs_current_one():
    import paper_1203_5737_amd as ac
    torch.cuda.init()
    assert ac._stream_handle(None) == torch.cuda.current_stream().cuda_stream
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        assert ac._stream_handle(None) == st.cuda_stream
        got = []
        th = threading.Thread(target=lambda: got.append(ac._stream_handle(None)))
        th.start()
        th.join()
        assert got == [torch.cuda.default_stream().cuda_stream]
    assert ac._stream_handle(st) == st.cuda_stream
    assert ac._stream_handle(None) == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("side", [3, 64, 300])
def test_product_follows_its_stream(side):
    import paper_1203_5737_amd as ac
    A = synth.laplace2d(side)
    M = ac.convert(ac.to_device_csr(A.rp, A.col, A.val, A.n_cols), 64, 1)
    want = ac.spmv(M, torch.ones(A.n_cols, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        x = torch.zeros(A.n_cols, dtype=torch.float64, device="cuda")
        for _ in range(50):                 # x is ready only in this stream's order
            x = x * 0.5
        x = x + 1.0
        y = ac.spmv(M, x)
    st.synchronize()
    assert np.array_equal(y.cpu().numpy(), want.cpu().numpy())


def test_calls_that_wait_are_refused_under_capture_and_spoil_nothing():
    """Conversion, staging, planning and binning wait for their stream: on a
    stream that captures a graph they are refused before they queue anything,
    the graph goes on, and the same calls work again afterwards."""
    import paper_1203_5737_amd as ac
    A = synth.laplace2d(120)                 # 14 400 rows: grouped on the device
    dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols)
    M = ac.convert(dev, 64, 1)
    want = M.columns.clone()
    a = torch.ones(1000, device="cuda")
    torch.cuda.synchronize()
    calls = [lambda: ac.convert(dev, 64, 1), lambda: ac.convert(dev, 64, 1, device_grouping=True),
             lambda: ac.convert(dev, 64, 0, region_rows=100, region_desired=np.ones(144, np.int32)),
             lambda: ac.plan_device(dev.row_ptr, 64, 1), lambda: ac.stage(M), lambda: ac.csr_bins(dev)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b = a * 2
        codes = []
        for call in calls:
            with pytest.raises(ac.ArgCsrError) as e:
                call()
            codes.append(e.value.code)
        b = b + 1
    assert codes == [ac._lib.EHIP] * len(calls)
    for k in range(3):
        a.fill_(float(k))
        g.replay()
        torch.cuda.synchronize()
        assert b.tolist() == [2.0 * k + 1.0] * 1000
        assert torch.equal(ac.convert(dev, 64, 1).columns, want)
    ac.stage(M)
    ac.csr_bins(dev)
