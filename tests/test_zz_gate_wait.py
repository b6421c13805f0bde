"""Comparisons that return to the host: the stream is synchronised then, sizes on either side of the single workgroup's share, behind work that takes long, from
several threads and streams at a time."""
import threading

import pytest

import paper_2006_05664_amd as P

pytestmark = pytest.mark.gpu


def _pair(n, seed, scale=1e-3):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    c = torch.randn(n, generator=g, device="cuda")
    return c, c + scale * torch.randn(n, generator=g, device="cuda")


def _expected(c, ref):
    c, ref = c.double(), ref.double()
    return float(((c - ref).abs() / (ref.abs() + 1.0)).max()), float((c - ref).norm() / ref.norm())


def _check(got, want):
    assert got[0] == want[0] and abs(got[1] - want[1]) <= 1e-12 * want[1], (got, want)


@pytest.mark.parametrize("n", [4095, 4096, 4097, 5000])
@pytest.mark.parametrize("offset", [0, 1])
def test_either_side_of_a_single_workgroup(n, offset):
    import torch
    c, ref = _pair(n + 1, n)
    c, ref = c[offset:offset + n], ref[offset:offset + n]
    stream = torch.cuda.current_stream().cuda_stream
    want = _expected(c, ref)
    result = torch.zeros(2, dtype=torch.float64, device="cuda")
    for _ in range(3):
        _check(P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), n, stream), want)
        P.opevo_compare_f32_static(c.data_ptr(), ref.data_ptr(), n, stream, result.data_ptr())
        torch.cuda.synchronize()
        assert tuple(result.tolist()) == P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), n, stream)


@pytest.mark.parametrize("n", [1, 4096, 4097, 65536, 3000000])
@pytest.mark.parametrize("rows", [False, True])
def test_the_stream_is_synchronised(n, rows):
    """The runtime itself calls the stream finished, on a stream of the caller's and on the default one, without being asked to wait."""
    import torch
    c, ref = _pair(n, n)
    index = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for stream in (torch.cuda.Stream(), torch.cuda.current_stream()):
        for _ in range(20):
            if rows:
                P.opevo_compare_rows_f32(c.data_ptr(), ref.data_ptr(), index.data_ptr(), 1, n, stream.cuda_stream)
            else:
                P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), n, stream.cuda_stream)
            assert stream.query()


def test_behind_work_that_takes_longer():
    import torch
    a = torch.randn(4096, 4096, device="cuda")
    c, ref = _pair(3000, 1)
    want = _expected(c, ref)
    for _ in range(3):
        b = a
        for _ in range(6):                                 # some ms of products in front of the comparison
            b = a @ b
        c2 = c + 0.0 * b.flatten()[:3000].nan_to_num(0.0, 0.0, 0.0)      # what is compared is the last of it
        _check(P.opevo_compare_f32(c2.data_ptr(), ref.data_ptr(), 3000, torch.cuda.current_stream().cuda_stream), want)


def test_several_threads_and_streams():
    import torch
    data = [_pair(n, n, s) for n, s in ((700, 1e-3), (4096, 1e-2), (50000, 1e-4), (3000000, 1e-1))]
    want = [_expected(*d) for d in data]
    torch.cuda.synchronize()
    failed = []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            for _ in range(200):
                _check(P.opevo_compare_f32(data[i][0].data_ptr(), data[i][1].data_ptr(), data[i][0].numel(), stream.cuda_stream), want[i])
        except BaseException as e:                          # noqa: B036 -- reported by the test's own thread
            failed.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
