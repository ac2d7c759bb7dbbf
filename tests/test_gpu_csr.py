"""GPU: the plain-CSR baselines (Sec. 2 definition) against the oracle --
the binned variant (rows grouped by length, a lane count per bin) must bin
every row once, in ascending order within its bin, sum a row of bin k < 7
bitwise as the uniform kernel with 2^k lanes per row does, and stay within
the FP64 bound (reduced types: gamma_{L+1}(2^-24)) everywhere."""
import numpy as np
import pytest
import torch

import oracle
import synth
from conftest import gpu_available
from helpers import powerlaw_sample
from test_gpu_parity import check_f64, check_reduced

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ac():
    import paper_1203_5737_amd as ac
    ac._lib.lib()
    return ac


def bins_of(rp):
    """Bin of every row: the smallest k with L <= 2^k, 7 above 64."""
    L = np.diff(rp.astype(np.int64))
    k = np.zeros(L.shape, np.int64)
    for b in range(1, 8):
        k[L > (1 << (b - 1))] = b
    return k


def with_rows(A, lengths_at):
    """A copy of A with the given rows replaced by rows of given lengths
    (columns 0..L-1, values 1/(1+j))."""
    L = np.diff(A.rp).astype(np.int64)
    cols, vals = [], []
    for r in range(A.n_rows):
        if r in lengths_at:
            n = lengths_at[r]
            cols.append(np.arange(n, dtype=np.int32) % A.n_cols)
            vals.append(1.0 / (1.0 + np.arange(n)))
            L[r] = n
        else:
            cols.append(A.col[A.rp[r]:A.rp[r + 1]])
            vals.append(A.val[A.rp[r]:A.rp[r + 1]])
    rp = np.zeros(A.n_rows + 1, np.int32)
    rp[1:] = np.cumsum(L)
    return synth.Csr(A.n_rows, A.n_cols, rp, np.concatenate(cols).astype(np.int32),
                     np.concatenate(vals))


def stored_values(ac, A, dtype):
    """A's values rounded to the storage type as the oracle rounds them
    (nearest-even from FP64), as a device tensor of that type."""
    bits = oracle.round_array(A.val, dtype)
    t = torch.from_numpy(bits.view(np.int16) if bits.dtype == np.uint16 else bits)
    return t.view(ac.storage_dtype(dtype)).to(DEV)


def test_binning_is_a_stable_partition(ac):
    A, x = powerlaw_sample(50_000, seed=12)
    dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV)
    b = ac.csr_bins(dev)
    k = bins_of(A.rp)
    want = np.argsort(k, kind="stable").astype(np.int32)
    assert np.array_equal(b.rows.cpu().numpy(), want)
    counts = np.bincount(k, minlength=8)
    assert np.array_equal(b.bin_start, np.concatenate([[0], np.cumsum(counts)]))


@pytest.mark.parametrize("dtype", [0, 1, 2, 3])
def test_binned_matches_oracle_and_uniform_kernel(ac, dtype):
    A0, x = powerlaw_sample(40_000, seed=13)
    # rows of every bin, long rows for the workgroup bin, empty rows
    A = with_rows(A0, {5: 65, 6: 255, 7: 256, 8: 257, 9: 3000, 10: 0, 11: 0, 39_999: 64})
    dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV)
    bins = ac.csr_bins(dev)
    vt = ac.vector_dtype(dtype)
    xd = torch.from_numpy(x).to(DEV, vt)
    vals = dev.val if dtype == 0 else stored_values(ac, A, dtype)
    y = ac.csr_spmv_binned(dev, xd, bins, values=vals, dtype=dtype)
    yn = y.cpu().numpy().astype(np.float64)
    if dtype == 0:
        check_f64(A, x, yn)
    else:
        check_reduced(A, x, yn, dtype)
    k = bins_of(A.rp)
    for b in range(7):
        yu = ac.csr_spmv(dev, xd, values=vals, dtype=dtype, lanes_per_row=1 << b).cpu()
        rows = np.nonzero(k == b)[0]
        assert torch.equal(y.cpu()[rows], yu[rows]), f"bin {b}"


def test_binned_full_powerlaw_and_stencil(ac):
    for A, x in (synth.workload_powerlaw(), synth.workload_stencil27(64)):
        dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV)
        bins = ac.csr_bins(dev)
        y = ac.csr_spmv_binned(dev, torch.from_numpy(x).to(DEV), bins)
        check_f64(A, x, y.cpu().numpy())


# launches of every make-up: one bin alone (teams of four rows), bins of about
# equal work (teams of one), bin 7 around the 1024 nonzeros of one wave, fewer
# rows than a workgroup or a region holds, and remainders
@pytest.mark.parametrize("lengths", ["one_bin", "equal_bins", "long", "few", "odd"])
@pytest.mark.parametrize("dtype", [0, 1])
def test_binned_launch_shapes(ac, lengths, dtype):
    rng = np.random.default_rng(5)
    L = {"one_bin": rng.integers(17, 33, 20_011),
         "equal_bins": np.repeat([1, 2, 4, 8, 16, 32, 64], 40_000 >> np.arange(7)),
         "long": np.array([65, 1023, 1024, 1025, 64, 1026, 2049, 0, 3000, 70, 4000]),
         "few": np.array([3, 0, 1]),
         "odd": rng.integers(0, 130, 1537)}[lengths].astype(np.int64)
    rng.shuffle(L)
    A = synth.random_csr(L, 6000, rng, rng)
    x = rng.uniform(-1.0, 1.0, A.n_cols)
    if dtype == 1:
        x = x.astype(np.float32).astype(np.float64)
    dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV)
    xd = torch.from_numpy(x).to(DEV, ac.vector_dtype(dtype))
    vals = dev.val if dtype == 0 else stored_values(ac, A, dtype)
    y = ac.csr_spmv_binned(dev, xd, ac.csr_bins(dev), values=vals, dtype=dtype)
    yn = y.cpu().numpy().astype(np.float64)
    if dtype == 0:
        check_f64(A, x, yn)
    else:
        check_reduced(A, x, yn, dtype)


# both batch sizes of bin 7 (16 elements a lane up to 4096 such rows, 8 beyond)
# at the edges of a wave, a round of 256 lanes and a whole batch
@pytest.mark.parametrize("rows", [60, 4096, 4097])
@pytest.mark.parametrize("dtype", [0, 2])
def test_binned_long_row_batches(ac, rows, dtype):
    rng = np.random.default_rng(rows)
    edges = [65, 127, 128, 129, 255, 256, 257, 511, 512, 513]
    for batch in (8 * 256, 16 * 256):
        edges += [batch - 193, batch - 192, batch - 1, batch, batch + 1, batch + 63, batch + 64,
                  batch + 65, batch + 257]
    edges += [2 * 8 * 256 + 8 * 256 - 1, 2 * 16 * 256 - 193, 2 * 16 * 256 + 300]
    L = np.full(rows, 65, np.int64)
    L[:len(edges)] = edges
    rng.shuffle(L)
    L = np.concatenate([L, [0, 1, 64, 3]])
    A = synth.random_csr(L, 9000, rng, rng)
    x = rng.uniform(-1.0, 1.0, A.n_cols).astype(np.float32).astype(np.float64)
    dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV)
    xd = torch.from_numpy(x).to(DEV, ac.vector_dtype(dtype))
    vals = dev.val if dtype == 0 else stored_values(ac, A, dtype)
    y = ac.csr_spmv_binned(dev, xd, ac.csr_bins(dev), values=vals, dtype=dtype)
    yn = y.cpu().numpy().astype(np.float64)
    if dtype == 0:
        check_f64(A, x, yn)
    else:
        check_reduced(A, x, yn, dtype)


def test_bins_of_another_matrix_still_cover_the_rows(ac):
    """Bins are a partition of the rows: a matrix whose rows have other
    lengths than the ones they were made from gives the right result too."""
    rng = np.random.default_rng(6)
    L = rng.integers(0, 90, 3000).astype(np.int64)
    A = synth.random_csr(L, 4000, rng, rng)
    B = synth.random_csr(L[::-1].copy(), 4000, rng, rng)
    x = rng.uniform(-1.0, 1.0, 4000)
    bins = ac.csr_bins(ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV))
    dev = ac.to_device_csr(B.rp, B.col, B.val, B.n_cols, DEV)
    y = ac.csr_spmv_binned(dev, torch.from_numpy(x).to(DEV), bins)
    check_f64(B, x, y.cpu().numpy())


def test_binned_edge_cases(ac):
    E = synth.Csr(0, 0, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0))
    dev = ac.to_device_csr(E.rp, E.col, E.val, 0, DEV)
    b = ac.csr_bins(dev)
    assert list(b.bin_start) == [0] * 9
    # all rows empty
    Z = synth.Csr(300, 10, np.zeros(301, np.int32), np.zeros(0, np.int32), np.zeros(0))
    dz = ac.to_device_csr(Z.rp, Z.col, Z.val, 10, DEV)
    bz = ac.csr_bins(dz)
    y = ac.csr_spmv_binned(dz, torch.ones(10, dtype=torch.float64, device=DEV), bz)
    assert torch.count_nonzero(y).item() == 0
    # bins that do not cover the rows are refused
    bz.bin_start[8] = 299
    with pytest.raises(ac.ArgCsrError):
        ac.csr_spmv_binned(dz, torch.ones(10, dtype=torch.float64, device=DEV), bz)


# how the rows of bin 7 are read: singly up to 4096 elements (1024 beside other
# rows) and in batches above, in one launch (a matrix the Infinity Cache holds); from 100 MB of
# elements on singly up to 256 (512 in 2-byte values), in batches of 4 up to
# 1024 and of 8 above, streamed; from 75 MB on where x is over 4 MB
@pytest.mark.parametrize("dtype,n_cols,mb,beside", [
    (0, 9000, 2, 0), (0, 9000, 99, 0), (0, 9000, 101, 0), (0, 530_000, 74, 0), (0, 530_000, 76, 0),
    (1, 9000, 99, 0), (1, 9000, 101, 0), (1, 1_060_000, 76, 0), (2, 9000, 2, 0), (2, 9000, 101, 0),
    (0, 9000, 3, 9000), (1, 9000, 2, 9000), (3, 9000, 2, 9000)])
def test_binned_long_row_paths(ac, dtype, n_cols, mb, beside):
    rng = np.random.default_rng(mb)
    edges = np.array([65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095,
                      4096, 4097, 4096 + 255, 4096 + 256, 4096 + 257, 6143, 6144, 6145, 8191,
                      8192, 8193])
    elements = mb * 1_000_000 // (4 + [8, 4, 2, 2][dtype]) + 1
    L = np.concatenate([edges, np.full((elements - edges.sum() - 600) // 2500, 2500),
                        rng.integers(0, 65, 20 + beside)])
    L = np.append(L, max(0, elements - L.sum())).astype(np.int64)
    rng.shuffle(L)
    A = synth.random_csr(L, n_cols, rng, rng)
    x = rng.uniform(-1.0, 1.0, A.n_cols).astype(np.float32).astype(np.float64)
    dev = ac.to_device_csr(A.rp, A.col, A.val, A.n_cols, DEV)
    xd = torch.from_numpy(x).to(DEV, ac.vector_dtype(dtype))
    vals = dev.val if dtype == 0 else stored_values(ac, A, dtype)
    y = ac.csr_spmv_binned(dev, xd, ac.csr_bins(dev), values=vals, dtype=dtype)
    yn = y.cpu().numpy().astype(np.float64)
    if dtype == 0:
        check_f64(A, x, yn)
    else:
        check_reduced(A, x, yn, dtype)
