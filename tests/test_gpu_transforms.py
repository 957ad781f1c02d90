"""GPU parity of the data-free offline transforms (channel salience, order, gather, reordered activation
quantizer, Hadamard rotation) against the CPU oracle, through the C ABI.  Everything here is exact: indices,
FP16 bit patterns, INT8 codes, INT32 accumulators."""
import ctypes
import math

import numpy as np
import pytest
import torch

from oracle import gemm as ogemm
from oracle import qoq_quant as qq
from oracle import transforms as tr
from paper_2405_04532_amd import api, workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bits(a):
    return np.asarray(a).view(np.uint16)


@pytest.mark.parametrize("M,K", [(100, 1024), (1, 128), (257, 4096)])
def test_salience_and_order(M, K):
    x = wl.make_activations(M, K, 60 + M, DEV)
    x[:, 7] = x[:, 3]                                            # exact ties in salience
    sal = api.channel_absmax(x)
    ref = tr.channel_salience(x.cpu().numpy())
    assert np.array_equal(sal.cpu().numpy(), ref)
    perm = api.channel_order(sal)
    assert np.array_equal(perm.cpu().numpy(), tr.channel_order(ref))
    assert not api.channel_absmax(x[:0]).any()                   # no tokens: zeros


@pytest.mark.parametrize("K", [1, 63, 64, 65, 8191, 8193, 14336, 32768, 32776])
def test_channel_order_on_the_device(K):
    """Ranks at the edges of a workgroup's 64 channels and of a tile of keys, many ties, both zeros, negative numbers; the
    last size is sorted on the host."""
    s = torch.randint(-3, 40, (K,), generator=torch.Generator().manual_seed(K)).to(torch.float32) * 0.25
    s[::7] = -0.0
    perm = api.channel_order(s.to(DEV))
    assert perm.dtype == torch.int32 and perm.is_cuda
    assert np.array_equal(perm.cpu().numpy(), tr.channel_order(s.numpy()))
    for bad in (float("nan"), float("inf"), float("-inf")):
        t = s.clone()
        t[K // 2] = bad
        with pytest.raises(api.QoqError):
            api.channel_order(t.to(DEV))


def test_channel_order_behind_other_work_and_under_capture():
    """The verdict on the salience comes from the kernel while the host waits: behind work of milliseconds on a stream of its own, good
    and bad in turn; a stream that is being captured cannot be waited for, and the capture goes on."""
    s = torch.rand(5000, generator=torch.Generator().manual_seed(3))
    bad = s.clone()
    bad[4999] = float("nan")
    ref = tr.channel_order(s.numpy())
    good, worse = s.to(DEV), bad.to(DEV)
    big = torch.ones(1 << 28, dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(3):
            for _ in range(4):
                big.mul_(1.0)                                    # 2 GiB each: 0.4 ms
            assert np.array_equal(api.channel_order(good).cpu().numpy(), ref)
            big.mul_(1.0)
            with pytest.raises(api.QoqError):
                api.channel_order(worse)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        out = torch.zeros(8, device=DEV)
        with torch.cuda.graph(graph, stream=side):
            with pytest.raises(RuntimeError):
                api.channel_order(good)
            out += 1
        graph.replay()
    torch.cuda.synchronize()
    assert (out == 1).all()


def test_channel_order_is_complete_when_the_call_returns():
    """Read on another stream without an event between, and salience overwritten there: 32768 channels of one value, which all meet in one counter
    and take the sort longest, so that its verdict on the salience is there long before the order is; the order's memory held other values."""
    K = 32768
    want = torch.arange(K, dtype=torch.int32)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(4):
        with torch.cuda.stream(side):
            sal = torch.full((K,), 2.5, device=DEV)
            stale = torch.full((K,), -1, dtype=torch.int32, device=DEV)
            side.synchronize()
            del stale
            perm = api.channel_order(sal)
        with torch.cuda.stream(other):
            sal.fill_(float("nan"))
            seen = perm.clone()
        other.synchronize()
        assert torch.equal(seen.cpu(), want)


@pytest.mark.parametrize("blocking", [False, True])
def test_channel_order_on_the_default_stream_beside_a_capture(blocking):
    """While another stream is captured: beside one that the default stream does not wait for, the order; beside one that it does, an error before
    anything is launched.  Neither the capture nor the next launch is the worse for it."""
    sal = torch.rand(300, device=DEV)
    want = torch.argsort(sal, descending=True, stable=True).to(torch.int32)
    out = torch.zeros(8, device=DEV)
    handle = ctypes.c_ulonglong(0)
    if blocking:
        assert int(torch.cuda.cudart().cudaStreamCreate(ctypes.addressof(handle))) == 0
    side = torch.cuda.ExternalStream(handle.value) if blocking else torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    assert torch.equal(api.channel_order(sal), want)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        out += 1
        with torch.cuda.stream(torch.cuda.default_stream()):
            if blocking:
                with pytest.raises(RuntimeError):
                    api.channel_order(sal)
            else:
                order = api.channel_order(sal)
        out += 2
    for n in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert (out == 3 * n).all()
        assert torch.equal(api.channel_order(sal), want) and (blocking or torch.equal(order, want))
    torch.cuda.synchronize()
    del graph
    if blocking:
        assert int(torch.cuda.cudart().cudaStreamDestroy(handle.value)) == 0


@pytest.mark.parametrize("rows,K", [(1, 8), (5, 8192), (3, 8200), (7, 16392), (2, 32768), (2, 32776)])
def test_gather_and_salience_edges(rows, K):
    """Four, two and one rows in LDS with a remainder, and rows that do not fit; row slabs of the salience."""
    x = wl.make_activations(rows, K, 71, DEV)
    perm = torch.randperm(K, generator=torch.Generator().manual_seed(K)).to(torch.int32).to(DEV)
    got = api.gather_channels(x, perm).cpu().numpy()
    assert np.array_equal(_bits(got), _bits(tr.reorder_channels(x.cpu().numpy(), perm.cpu().numpy())))
    y = wl.make_activations(128 * rows + 1, 264, 72, DEV)
    assert np.array_equal(api.channel_absmax(y).cpu().numpy(), tr.channel_salience(y.cpu().numpy()))


@pytest.mark.parametrize("K", [8, 256, 264, 4104])
@pytest.mark.parametrize("M", [1, 2, 127, 128, 129, 257])
def test_salience_of_one_slab_of_rows_and_of_several(M, K):
    """One slab of rows stores every channel itself, whatever the output held; a channel of NaNs and one of zeros are 0."""
    x = wl.make_activations(M, K, 74, DEV)
    x[:, 3], x[:, 5], x[M - 1, 6] = float("nan"), 0.0, float("inf")
    out = torch.full((K,), float("nan"), device=DEV)
    ref = np.nan_to_num(np.abs(x.float().cpu().numpy()), nan=0.0, posinf=np.inf).max(axis=0)
    assert api.lib().qoq_channel_absmax(x.data_ptr(), M, K, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert np.array_equal(out.cpu().numpy(), ref)


@pytest.mark.parametrize("rows,K", [(3, 256), (3, 264), (511, 264), (513, 264), (2047, 264), (2050, 264), (513, 8184), (159, 8192), (160, 8192),
                                    (81, 16392), (41, 32768)])
def test_gather_on_either_side_of_its_rules(rows, K):
    """Short rows and few long ones gathered from memory, the others through LDS with one, two and four rows at a time."""
    x = wl.make_activations(rows, K, 73, DEV)
    perm = torch.randperm(K, generator=torch.Generator().manual_seed(K)).to(torch.int32).to(DEV)
    assert torch.equal(api.gather_channels(x, perm), x[:, perm.long()])


@pytest.mark.parametrize("M,K", [(129, 8), (130, 72), (255, 4104), (1000, 64), (1024, 520), (1025, 520)])
def test_salience_in_one_pass_over_the_rows(M, K):
    """Up to 1024 rows by columns: a part of a 64-channel workgroup, rows past the last multiple of 128, the maximum in the last
    row, infinities taken and NaN not; 1025 rows by slabs."""
    x = torch.randn(M, K, generator=torch.Generator(device=DEV).manual_seed(M), device=DEV).half()
    x[M - 1, K - 1], x[M // 2, 0] = -60000.0, float("-inf")
    x[:, 1] = float("nan")
    x[M - 1, 1] = 0.25
    out = torch.full((K,), -1.0, device=DEV)
    assert api.lib().qoq_channel_absmax(x.data_ptr(), M, K, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(out, torch.nan_to_num(x.float(), nan=0.0, posinf=math.inf, neginf=-math.inf).abs().amax(0))


@pytest.mark.parametrize("M", [65535 * 128, 65535 * 128 + 1, 65535 * 128 + 128, 65535 * 128 + 129])
def test_salience_of_more_rows_than_a_launch_takes(M):
    """The last launch has no rows, one row, one slab and two slabs of its own: it adds to the maxima of the one before."""
    x = torch.zeros(M, 8, dtype=torch.float16, device=DEV)
    x[0, 0], x[M // 2, 1], x[M - 1, 2] = 3.0, -5.0, 7.0
    out = torch.full((8,), -1.0, device=DEV)
    assert api.lib().qoq_channel_absmax(x.data_ptr(), M, 8, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert out.tolist() == [3.0, 5.0, 7.0] + [0.0] * 5


def test_gather_and_reordered_quantizer_bit_exact():
    M, K, N = 70, 2048, 192
    x = wl.make_activations(M, K, 61, DEV)
    w = wl.make_weights(N, K, 61, DEV)
    perm = api.channel_order(api.channel_absmax(x))
    p = perm.cpu().numpy()
    wr = api.gather_channels(w, perm)
    assert np.array_equal(_bits(wr.cpu().numpy()), _bits(tr.reorder_channels(w.cpu().numpy(), p)))
    qx, sx, rowsum, tx = api.quant_act_per_token_reordered(x, perm, want_tx=True)
    oqx, osx, ors, otx = qq.act_quant(tr.reorder_channels(x.cpu().numpy(), p))
    assert np.array_equal(qx.cpu().numpy(), oqx) and np.array_equal(_bits(sx.cpu().numpy()), _bits(osx))
    assert np.array_equal(rowsum.cpu().numpy(), ors)
    # the fused gather equals gather-then-quantize on the GPU as well
    qx2, sx2, _, _ = api.quant_act_per_token(api.gather_channels(x, perm))
    assert torch.equal(qx, qx2) and torch.equal(sx, sx2)
    # whole reordered layer: INT32 accumulators bit-exact, FP16 output within the GEMM tolerance
    blob = api.pack_weights(wr)
    acc = api.w4a8_gemm_i32(qx, blob, N).cpu().numpy().astype(np.int64)
    out = api.w4a8_gemm(qx, sx, blob, N).cpu().numpy().astype(np.float64)
    ref = ogemm.forward_group(tr.reorder_channels(w.cpu().numpy(), p), tr.reorder_channels(x.cpu().numpy(), p))
    assert np.array_equal(acc, ref["acc"])
    assert np.all(np.abs(out - ref["out64"]) <= 1e-3 * np.abs(ref["out64"]) + 2.0 ** -24)


def test_reordering_clamps_bad_indices():
    x = wl.make_activations(4, 256, 62, DEV)
    perm = torch.arange(256, dtype=torch.int32, device=DEV)
    perm[5], perm[9] = -7, 100000
    g = api.gather_channels(x, perm).cpu().numpy()
    xc = x.cpu().numpy()
    assert np.array_equal(_bits(g[:, 5]), _bits(xc[:, 0])) and np.array_equal(_bits(g[:, 9]), _bits(xc[:, 255]))
    assert np.array_equal(_bits(g[:, 10:]), _bits(xc[:, 10:]))


@pytest.mark.parametrize("rows,K,block", [(5, 64, 2), (3, 256, 64), (70, 4096, 4096), (2, 8192, 8192), (9, 11008, 256),
                                          (4, 512, 1)])
def test_hadamard_rotation_bit_exact(rows, K, block):
    x = wl.make_activations(rows, K, 63 + block % 97, DEV)
    got = api.hadamard_rotate(x, block)
    ref = tr.rotate_fp16(x.cpu().numpy(), block)
    assert np.array_equal(_bits(got.cpu().numpy()), _bits(ref))
    y = x.clone()
    api.hadamard_rotate(y, block, out=y)                         # in place
    assert torch.equal(y, got)


@pytest.mark.parametrize("rows,K,block", [(1, 8, 8), (3, 24, 8), (1, 4104, 8), (257, 16, 16), (33, 128, 128), (7, 2048, 2048),
                                          (3, 12288, 4096), (3, 24576, 8192), (5, 20, 4), (3, 5, 1),
                                          (512, 8, 8), (513, 8, 8), (514, 32, 16), (600, 128, 128), (2, 65536, 128), (2, 65792, 256), (1, 4104, 4),
                                          (2, 512, 512)])
def test_hadamard_segment_edges_bit_exact(rows, K, block):
    """Tensors that end inside a segment of the kernel, every group of stages present and absent, few short blocks, and tensors
    that are no whole number of 16-byte chunks; exact, because FP64 sums of FP16 numbers are."""
    x = wl.make_activations(rows, K, 70 + block % 89, DEV)
    ref = tr.rotate_fp16(x.cpu().numpy(), block)
    assert np.array_equal(_bits(api.hadamard_rotate(x, block).cpu().numpy()), _bits(ref))
    odd = torch.empty(rows * K + 1, dtype=torch.float16, device=DEV)[1:].view(rows, K)      # 2-byte aligned only
    odd.copy_(x)
    assert np.array_equal(_bits(api.hadamard_rotate(odd, block, out=odd).cpu().numpy()), _bits(ref))


def _butterflies(x, block):
    """The rotation in FP64 with the stages in the order in which the segment kernel takes them, which sign of a zero can depend on."""
    v = x.cpu().numpy().astype(np.float64).reshape(-1, block)
    with np.errstate(invalid="ignore"):                          # infinities
        for h in (1, 2, 4, 2048, 4096) + tuple(8 << i for i in range(8)):
            if h < block:
                p = v.reshape(-1, block // (2 * h), 2, h)
                v = np.stack([p[:, :, 0] + p[:, :, 1], p[:, :, 0] - p[:, :, 1]], axis=2).reshape(-1, block)
        return (v * (1.0 / math.sqrt(block))).reshape(x.shape).astype(np.float16)


@pytest.mark.parametrize("signed_zeros", [False, True])
@pytest.mark.parametrize("rows,K,block", [(3, 4096, 4096), (2, 8192, 8192), (9, 2048, 2048), (5, 4096, 512), (3, 4104, 8), (3, 4096, 4)])
def test_hadamard_small_magnitudes_bit_exact(rows, K, block, signed_zeros):
    """Rows whose magnitudes add up to just less and just more than 128 (whole numbers, FP64), with subnormals, blocks of zeros
    (of both signs: FP64), an infinity and a NaN in the last row; against FP64, zeros with their signs."""
    g = torch.Generator(device=DEV).manual_seed(K + block)
    x = torch.randn(rows, K, generator=g, device=DEV)
    seg = 4096 if block <= 4096 else 8192
    x = x * (torch.tensor([127.0, 127.95, 129.0] * rows, device=DEV)[:rows, None] / (seg * (2 / math.pi) ** 0.5))
    x = x.half()
    x[0, ::7] *= 2.0 ** -12                                      # subnormals
    x = torch.where(x == 0, torch.zeros_like(x), x)              # (subnormals rounded to -0)
    x[0, :8] = -0.0 if signed_zeros else 0.0                     # a chunk of nothing but -0
    if rows > 1:
        x[1, block // 2:block] = 0.0
        x[1, :block // 2] = -0.0 if signed_zeros else 0.0
    x[-1, -1], x[-1, -2] = float("inf"), float("nan")
    ref = _butterflies(x, block)
    got = api.hadamard_rotate(x, block).cpu().numpy()
    nan = np.isnan(ref)
    assert np.array_equal(np.isnan(got), nan)
    assert np.array_equal(_bits(got)[~nan], _bits(ref)[~nan])
    if block == 8 and signed_zeros:                              # a sum of nothing but -0, and differences of such
        assert _bits(got)[0, :8].tolist() == [0x8000] + 7 * [0]


@pytest.mark.parametrize("block,others", [(8, 0.01), (8, 1000.0), (512, 0.01), (4096, 0.01)])
def test_hadamard_signs_of_zero(block, others):
    """Blocks of zeros of both signs and pairs that cancel give the zeros of FP64 sums, whatever the sum of the other magnitudes in
    their segment."""
    x = torch.full((4, 8192), others, dtype=torch.float16, device=DEV)
    pos, neg, v = torch.tensor([0.0, -0.0, 0.01], dtype=torch.float16, device=DEV)
    for at, eight in ((0, (neg, neg, v, -v, pos, pos, pos, pos)), (8, (neg, pos, v, v, pos, pos, pos, pos)),
                      (4096, (neg,) * 8), (4104, (neg, pos) * 4), (4112, (pos,) * 8)):     # two segments
        x[:2, at:at + 8] = torch.stack(eight)
    if block > 8:                                                # the whole block cancels
        x[2, :block] = 0.0
        x[2, :4] = torch.stack((neg, neg, v, -v))
        x[3, 4096:4096 + block] = -0.0
    got = _bits(api.hadamard_rotate(x, block).cpu().numpy())
    ref = _bits(_butterflies(x, block))
    assert (ref == 0x8000).any() and np.array_equal(got, ref)


def test_rotated_layer_matches_the_oracle_and_the_unrotated_product():
    M, K, N = 33, 1024, 128
    x = wl.make_activations(M, K, 64, DEV)
    w = wl.make_weights(N, K, 64, DEV)
    xr, wr = api.hadamard_rotate(x), api.hadamard_rotate(w)      # default block: the whole row (1024)
    blob = api.pack_weights(wr)
    qx, sx, _, _ = api.quant_act_per_token(xr)
    acc = api.w4a8_gemm_i32(qx, blob, N).cpu().numpy().astype(np.int64)
    ref = ogemm.forward_group(tr.rotate_fp16(w.cpu().numpy(), K), tr.rotate_fp16(x.cpu().numpy(), K))
    assert np.array_equal(acc, ref["acc"])
    exact = x.cpu().numpy().astype(np.float64) @ w.cpu().numpy().astype(np.float64).T
    plain = ogemm.forward_group(w.cpu().numpy(), x.cpu().numpy())["out64"]
    err_rot = np.sqrt(np.mean((ref["out64"] - exact) ** 2))
    err_plain = np.sqrt(np.mean((plain - exact) ** 2))
    assert err_rot < err_plain                                   # what the rotation is for, on outlier activations


def test_transform_argument_validation():
    L = api.lib()
    x = torch.zeros((4, 256), dtype=torch.float16, device=DEV)
    out = torch.empty_like(x)
    perm = torch.arange(256, dtype=torch.int32, device=DEV)
    assert L.qoq_hadamard_rotate(x.data_ptr(), 4, 256, 48, out.data_ptr(), None) == 2        # not a power of two
    assert L.qoq_hadamard_rotate(x.data_ptr(), 4, 256, 512, out.data_ptr(), None) == 2       # does not divide K
    assert L.qoq_hadamard_rotate(x.data_ptr(), 4, 1 << 15, 1 << 14, out.data_ptr(), None) == 2   # block too large
    assert L.qoq_hadamard_rotate(None, 4, 256, 256, out.data_ptr(), None) == 1
    assert L.qoq_gather_channels(x.data_ptr(), perm.data_ptr(), 4, 256, x.data_ptr(), None) == 2  # in place
    assert L.qoq_gather_channels(x.data_ptr(), perm.data_ptr(), 4, 252, out.data_ptr(), None) == 2
    assert L.qoq_quant_act_per_token_reordered(x.data_ptr(), None, 4, 256, out.data_ptr(), out.data_ptr(), None, None, None) == 1
    assert L.qoq_channel_order_host(None, 16, None) == 1
