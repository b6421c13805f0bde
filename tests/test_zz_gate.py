"""The parity gate's kernels at the sizes and alignments where they can go wrong: fewer elements than a wave, one more or
less than a workgroup's, the grid's and the unrolled loop's share, arrays that start at any 4-byte offset, rows shorter
than a wave and of odd length.  The maximum is a quotient of the same two doubles on both sides, so it is compared exactly;
the norms differ by the order of an fp64 sum over at most 5e6 terms (1e-12 is 1000 times the rounding of a pairwise sum)."""
import numpy as np
import pytest

import paper_2006_05664_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def data():
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    c = torch.randn(1 << 22, generator=g, device="cuda")
    return c, c + 1e-3 * torch.randn(1 << 22, generator=g, device="cuda"), torch.cuda.current_stream().cuda_stream, g


def _expected(c, ref):
    c, ref = c.double(), ref.double()
    return float(((c - ref).abs() / (ref.abs() + 1.0)).max()), float((c - ref).norm() / ref.norm())


def _check(got, want):
    assert got[0] == want[0] and abs(got[1] - want[1]) <= 1e-12 * want[1], (got, want)


@pytest.mark.parametrize("offset", [0, 1, 2, 4])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 255, 257, 1023, 1025, 4099, (1 << 20) - 1, (1 << 20) + 5, 3000001])
def test_whole_output(data, n, offset):
    buf, refs, stream, _ = data
    c, ref = buf[offset:offset + n], refs[offset:offset + n]
    _check(P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), n, stream), _expected(c, ref))
    for place in {0, n // 2, n - 1}:       # what can never pass does not, wherever it is
        for bad in (float("nan"), float("inf")):
            kept = float(buf[offset + place])
            buf[offset + place] = bad
            got = P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), n, stream)
            buf[offset + place] = kept
            assert np.isinf(got[0]), (place, bad, got)
            kept = float(refs[offset + place])
            refs[offset + place] = bad
            got = P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), n, stream)
            refs[offset + place] = kept
            assert np.isinf(got[0]), (place, bad, got)


@pytest.mark.parametrize("row_len", [1, 3, 4, 64, 100, 729, 4096])
def test_sampled_rows(data, row_len):
    import torch
    buf, _, stream, g = data
    total = 2000000 // row_len
    c = buf[:total * row_len].view(total, row_len)
    for n_rows in (1, 2, 5, total // 3, total):
        index = torch.randperm(total, generator=g, device="cuda")[:n_rows].to(torch.int32)
        ref = c[index.long()] + 1e-3 * torch.randn((n_rows, row_len), generator=g, device="cuda")
        _check(P.opevo_compare_rows_f32(c.data_ptr(), ref.data_ptr(), index.data_ptr(), n_rows, row_len, stream),
               _expected(c[index.long()], ref))
        ref[n_rows - 1, row_len - 1] = float("nan")
        assert np.isinf(P.opevo_compare_rows_f32(c.data_ptr(), ref.data_ptr(), index.data_ptr(), n_rows, row_len, stream)[0])


def test_equal_arrays_and_a_reference_of_zeros(data):
    import torch
    stream = data[2]
    zeros, ones = torch.zeros(1000, device="cuda"), torch.ones(1000, device="cuda")
    assert P.opevo_compare_f32(zeros.data_ptr(), zeros.data_ptr(), 1000, stream) == (0.0, 0.0)
    assert P.opevo_compare_f32(ones.data_ptr(), ones.data_ptr(), 1000, stream) == (0.0, 0.0)
    mx, fro = P.opevo_compare_f32(ones.data_ptr(), zeros.data_ptr(), 1000, stream)
    assert mx == 1.0 and np.isinf(fro)


def test_a_stream_under_capture_is_refused_and_keeps_its_capture(data):
    import torch
    c, ref = data[0][:4099], data[1][:4099]
    want = P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), 4099, data[2])      # a workspace is there
    out, graph = torch.zeros(2, dtype=torch.float64, device="cuda"), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        stream = torch.cuda.current_stream().cuda_stream
        for _ in range(3):
            with pytest.raises(P.OpevoError) as e:
                P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), 4099, stream)
            assert e.value.status == P.OPEVO_E_HIP and "captured" in e.value.message
        P.opevo_compare_f32_static(c.data_ptr(), ref.data_ptr(), 4099, stream, out.data_ptr())
    for _ in range(3):                                                            # what was recorded beside the refused calls runs
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert tuple(out.tolist()) == want == P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), 4099, data[2])
