"""fp16 rows of a decode call (the window, 16-bit layers): the values go through the matrix cores, their numerators as two fp16
parts.  Against the oracle with the bars of the parity tests, and where those parts could matter against 64 bits.  And the order in which a
call takes its blocks."""
import os

import numpy as np
import pytest
import torch

import kvq_workloads as W
from test_gpu_parity import assert_outputs_close, kvq_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def _odd(x):
    """A contiguous copy on the GPU that begins two bytes behind an aligned address."""
    t = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape)
    return t.copy_(x)


@pytest.mark.parametrize("kb,vb", [(4, 2), (8, 16), (16, 4), (16, 16)])
@pytest.mark.parametrize("gq,hkv,batch,T,residual", [
    (1, 2, 1, 1, 32), (4, 2, 1, 31, 32), (3, 2, 1, 33, 32),              # window only: one row, one chunk less one, two chunks
    (5, 1, 2, 32 * 6 + 7, 128), (8, 2, 1, 32 * 5 + 31, 64), (12, 1, 1, 70, 32),
    (4, 8, 160, 40, 32), (7, 4, 300, 32 + 9, 32),                        # more work-groups than are resident: one pair of waves each
])
def test_rows_and_appended_rows(kvq_mod, oracle_mod, gq, hkv, batch, T, residual, kb, vb):
    """Every kind of row position: rows of the ring, the appended one (from the caller's tensors, at odd addresses), rows past the end."""
    w = W.Workload("rows", 1, batch, gq * hkv, hkv, 128, T, [kb], [vb], seed=7 + T + gq, outlier_channels=3)
    g = kvq_mod.KVQ(1, batch, gq * hkv, hkv, 128, T + 40, [kb], [vb], residual=residual)
    g.workspace.fill_(0xff)                                              # a row that was never written reads as NaN
    o = oracle_mod.OracleCache(1, batch, gq * hkv, hkv, 128, [kb], [vb], residual=residual)
    K, V = W.kv_tokens(w, 0, 0, T + 2)
    if T > 1:
        g.quantize_append(0, _odd(K[:, :, :T - 1].contiguous()), _odd(V[:, :, :T - 1].contiguous()))
        o.quantize_append(0, K[:, :, :T - 1].numpy().copy(), V[:, :, :T - 1].numpy().copy())
    q = W.query(w, 0)
    for t in range(T - 1, T + 2):
        k, v = K[:, :, t:t + 1].contiguous(), V[:, :, t:t + 1].contiguous()
        out = g.append_decode_attention(0, _odd(k), _odd(v), _odd(q), _odd(torch.zeros_like(q)))
        o.quantize_append(0, k.numpy(), v.numpy())
        assert_outputs_close(out, *o.decode_attention(0, q.numpy()), "append %d" % t)
    assert_outputs_close(g.decode_attention(0, _odd(q)), *o.decode_attention(0, q.numpy()), "from the ring")
    g.close()


@pytest.mark.parametrize("vb", [4, 16])
def test_small_numerators_count(kvq_mod, vb):
    """One token takes nearly all of the weight and has zeros as values; the others weigh 2^-14 .. 2^-34 of it and hold values up to
    6e4, so the outputs are made of small numerators alone, whose high parts are down to fp16 subnormals without the lift.  A numerator
    keeps 24 bits, or 2^-47 where its two parts end; |error| <= sum_t (2^-20 p_t + 2^-47) |v_t| / l, and the fp16 rounding."""
    T, D = 32 + 23, 128
    g = torch.Generator().manual_seed(5)
    q = torch.zeros(1, 4, D, dtype=torch.float16)
    q[..., 0] = 16.0
    K = torch.zeros(1, 1, T, D, dtype=torch.float16)
    logit = -(14 + 20 * torch.arange(T) / T)                             # in powers of two
    logit[7] = 0
    K[0, 0, :, 0] = (logit * np.log(2) * np.sqrt(D) / 16).half()
    V = (torch.rand(1, 1, T, D, generator=g) * 6e4).half()
    V[0, 0, 7] = 0
    cache = kvq_mod.KVQ(1, 1, 4, 1, D, 128, [16], [vb], residual=64 if vb < 16 else 0)     # all of it in the window, or one unit of a 16-bit layer and the rest
    cache.quantize_append(0, K.cuda(), V.cuda())
    out = cache.decode_attention(0, q.cuda()).cpu().double()
    s = (q.double()[0] @ K.double()[0, 0].T) / np.sqrt(D)
    p = torch.exp(s - s.amax(1, keepdim=True))
    ref = (p @ V.double()[0, 0]) / p.sum(1, keepdim=True)
    bound = ((2.0 ** -20 * p + 2.0 ** -47) @ V.double()[0, 0].abs()) / p.sum(1, keepdim=True) + 2.0 ** -11 * ref.abs() + 2.0 ** -24
    assert ref.abs().min() > 1e-3 and ((out[0] - ref).abs() <= bound).all(), ((out[0] - ref).abs() / bound).max()
    cache.close()


@pytest.mark.parametrize("vb", [4, 16])
@pytest.mark.parametrize("gq", [4, 7])
def test_infinite_values_stay_infinite(kvq_mod, gq, vb):
    """An infinite value makes its channel of the output infinite, with the value's sign, also where a numerator is one fp16 number
    (no low part); other channels are untouched."""
    T, D = 32 + 9, 128
    g = torch.Generator().manual_seed(6)
    q, K, V = (torch.randn(1, h, n, D, generator=g).half() for h, n in ((gq, 1), (1, T), (1, T)))
    K[0, 0, 3] = 0
    plain = None
    for bad in (False, True):
        if bad:
            V[0, 0, 3, 5], V[0, 0, T - 1, 77] = float("inf"), float("-inf")
            V[0, 0, 9, 100] = float("nan")
        cache = kvq_mod.KVQ(1, 1, gq, 1, D, 128, [16], [vb], residual=64 if vb < 16 else 0)
        cache.set_decode_options(0, 1)                                   # (several: the next test)
        cache.quantize_append(0, K[:, :, :T - 1].contiguous().cuda(), V[:, :, :T - 1].contiguous().cuda())
        out = cache.append_decode_attention(0, K[:, :, T - 1:].contiguous().cuda(), V[:, :, T - 1:].contiguous().cuda(), q[:, :, 0].contiguous().cuda()).cpu()
        cache.close()
        if not bad:
            plain = out
    assert (out[0, :, 5] == float("inf")).all()
    # (rows past the end repeat the last one with weight zero, and its infinity times zero is no number, but for the high parts, which are never zero)
    assert not torch.isfinite(out[0, :, 77]).any() and torch.isnan(out[0, :, 100]).all()
    rest = [c for c in range(D) if c not in (5, 77, 100)]
    assert torch.equal(out[0][:, rest], plain[0][:, rest])


@pytest.mark.parametrize("vb", [4, 16])
@pytest.mark.parametrize("gq", [3, 5, 7, 8, 12])
def test_infinite_values_stay_infinite_in_merged_splits(kvq_mod, gq, vb):
    """Several splits, merged by the last work-group: an infinity in one split's record reaches every head's output as it is, from 2
    splits to as many as are merged that way, and nothing of it reaches another head's record or another channel."""
    T, D = 32 * 17 + 9, 128
    g = torch.Generator().manual_seed(6)
    q, K, V = (torch.randn(1, h, n, D, generator=g).half().cuda() for h, n in ((gq, 1), (1, T), (1, T)))
    rest = [c for c in range(D) if c != 5]
    for splits in list(range(2, 10)) + [15, 16, 17]:
        outs = []
        for value in (1.0, float("-inf")):
            V[0, 0, T - 3, 5] = value                                    # (in the window: the last split's)
            cache = kvq_mod.KVQ(1, 1, gq, 1, D, T, [16], [vb], residual=32 if vb < 16 else 0)
            cache.set_decode_options(0, splits)
            cache.quantize_append(0, K, V)
            outs.append(cache.decode_attention(0, q[:, :, 0].contiguous()).cpu())
            cache.close()
        assert (outs[1][0, :, 5] == float("-inf")).all(), (splits, outs[1][0, :, 5])
        assert torch.equal(outs[0][0][:, rest], outs[1][0][:, rest]), splits


@pytest.mark.parametrize("batch,gq,splits", [(300, 4, s) for s in (2, 3, 5, 8, 9, 13, 16, 17)] + [(1, 7, 17), (1, 8, 19), (1, 4, 49), (1, 1, 63), (2, 7, 65), (1, 7, 70)])
def test_infinite_values_stay_infinite_where_a_launch_merges(kvq_mod, batch, gq, splits):
    """The same for splits that a launch of their own merges: one sequence's first and last split hold an infinity each, which its outputs show in their
    channels and nothing else does, whatever number of records the launch's threads have room for."""
    T, D = 32 * 72 + 9 if batch < 10 else 32 * 20 + 9, 128
    g = torch.Generator().manual_seed(7)
    q, K, V = (torch.randn(1, h, n, D, generator=g).half().cuda().expand(batch, h, n, D).contiguous() for h, n in ((gq, 1), (1, T), (1, T)))
    outs = []
    for bad in (False, True):
        if bad:
            V[0, 0, 3, 5], V[0, 0, T - 3, 77] = float("inf"), float("-inf")
        cache = kvq_mod.KVQ(1, batch, gq, 1, D, T, [16], [16])
        cache.set_decode_options(0, splits)
        cache.quantize_append(0, K, V)
        outs.append(cache.decode_attention(0, q[:, :, 0].contiguous()).cpu())
        cache.close()
    plain, out = outs
    assert (out[0, :, 5] == float("inf")).all() and (out[0, :, 77] == float("-inf")).all(), (out[0, :, 5], out[0, :, 77])
    plain[0, :, 5], plain[0, :, 77] = float("inf"), float("-inf")
    assert torch.equal(out, plain)


@pytest.mark.parametrize("vb", [4, 16])
@pytest.mark.parametrize("gq", [1, 4, 7])
def test_numerators_far_below_the_largest(kvq_mod, gq, vb):
    """One token takes nearly all of the weight and has zeros as values; the others weigh 2^-37 to 2^-39 of it and hold values of
    3e4 to 6e4, so each output is a few 2^-18: a numerator keeps 2^-47 where its bits end, and |error| <= sum_t 2^-47 |v_t| / l,
    half of the outputs' spacing (fp16 subnormals: 2^-24), and 2^-18 of the sum (scores of 39 in fp32, exponentiated)."""
    T, D = 32 + 31, 128
    g = torch.Generator().manual_seed(8)
    q = torch.zeros(1, gq, D, dtype=torch.float16)
    q[..., 0] = 32.0
    K = torch.zeros(1, 1, T, D, dtype=torch.float16)
    logit = -(37 + 2 * torch.arange(T) / T)                              # in powers of two
    logit[7] = 0
    K[0, 0, :, 0] = (logit * np.log(2) * np.sqrt(D) / 32).half()
    V = (3e4 * (1 + torch.rand(1, 1, T, D, generator=g))).half()
    V[0, 0, 7] = 0
    cache = kvq_mod.KVQ(1, 1, gq, 1, D, 128, [16], [vb], residual=64 if vb < 16 else 0)     # all of it in the window, or one unit of a 16-bit layer and the rest
    cache.set_decode_options(0, 1)
    cache.quantize_append(0, K.cuda(), V.cuda())
    out = cache.decode_attention(0, q.cuda()).cpu().double()
    cache.close()
    s = (q.double()[0] @ K.double()[0, 0].T) / np.sqrt(D)
    p = torch.exp(s - s.amax(1, keepdim=True))
    ref = (p @ V.double()[0, 0]) / p.sum(1, keepdim=True)
    bound = (2.0 ** -47 * V.double()[0, 0].abs().sum(0)) / p.sum(1, keepdim=True) + 2.0 ** -25 + 2.0 ** -18 * ref.abs()
    assert ref.min() > 2.0 ** -19 and ((out[0] - ref).abs() <= bound).all(), ((out[0] - ref).abs() / bound).max()


@pytest.mark.parametrize("vb", [4, 16])
@pytest.mark.parametrize("power", [-3, -25, -38, -50, -80])
def test_infinite_values_under_small_weights(kvq_mod, power, vb):
    """An infinite value under a weight of 2^power of the largest: infinite, with the value's sign, next to another infinite one under a large weight,
    and where a chunk of rows follows another.  Infinities of both signs, or a value that is no number, give no number."""
    T, D, gq = 32 + 29, 128, 4
    q = torch.zeros(1, gq, D, dtype=torch.float16)
    q[..., 0] = 64.0
    K = torch.zeros(1, 1, T, D, dtype=torch.float16)
    small = [5, 40]
    K[0, 0, small, 0] = power * np.log(2) * np.sqrt(D) / 64
    V = torch.ones(1, 1, T, D, dtype=torch.float16)
    V[0, 0, 5, 1], V[0, 0, 40, 2], V[0, 0, 5, 3], V[0, 0, 11, 3] = float("inf"), float("-inf"), float("inf"), float("inf")
    V[0, 0, 40, 4], V[0, 0, 11, 4], V[0, 0, 5, 5], V[0, 0, 40, 5], V[0, 0, 5, 6] = float("-inf"), float("-inf"), float("inf"), float("-inf"), float("nan")
    cache = kvq_mod.KVQ(1, 1, gq, 1, D, 128, [16], [vb], residual=64 if vb < 16 else 0)
    cache.set_decode_options(0, 1)
    cache.quantize_append(0, K.cuda(), V.cuda())
    out = cache.decode_attention(0, q.cuda()).cpu()[0]
    cache.close()
    inf = float("inf")
    for channel, value in ((1, inf), (2, -inf), (3, inf), (4, -inf)):
        assert (out[:, channel] == value).all(), (channel, out[:, channel])
    assert torch.isnan(out[:, 5:7]).all() and torch.isfinite(out[:, 7:]).all() and torch.isfinite(out[:, 0]).all()


SWEEPS = {"short": (1, 8, 2, 4133, 4, 2), "streaming": (64, 8, 2, 2000, 4, 4), "tiles of 8": (16, 14, 2, 3000, 8, 2)}


def _bell(rows, seed):
    """fp16 [rows, 128] of unit variance, by whole numbers: the same on every machine."""
    with np.errstate(over="ignore"):
        x = np.arange(rows * 128, dtype=np.uint64) + np.uint64(seed << 40)
        for shift, factor in ((30, 0xBF58476D1CE4E5B9), (27, 0x94D049BB133111EB), (31, 0x9E3779B97F4A7C15), (29, 0xBF58476D1CE4E5B9)):
            x = (x ^ (x >> np.uint64(shift))) * np.uint64(factor)
    total = sum(((x >> np.uint64(16 * k)) & np.uint64(0xffff)).astype(np.int64) for k in range(4))       # of four uniform numbers
    return torch.from_numpy(((total - 131070) / 37837.0).astype(np.float16)).view(rows, 128)


def sweep_outputs(module, batch, hq, hkv, T, kb, vb):
    """Outputs of one layer's decode attention, of the last sequence."""
    K, V, q = _bell(hkv * T, 1).cuda(), _bell(hkv * T, 2).cuda(), _bell(hq, 3).cuda()
    cache = module.KVQ(1, batch, hq, hkv, 128, T, [kb], [vb])
    # every sequence is the same one, its tokens rolled by another 131
    roll = lambda x: torch.stack([torch.roll(x.view(hkv, T, 128), 131 * b, 1) for b in range(batch)])     # noqa: E731
    cache.quantize_append(0, roll(K), roll(V))
    out = cache.decode_attention(0, q.view(1, hq, 128).expand(batch, hq, 128).contiguous())
    cache.close()
    return out[-1].cpu().numpy()


@pytest.mark.parametrize("name", list(SWEEPS))
def test_sweeps_start_where_they_did(kvq_mod, name):
    """A pair of waves starts its sweep at block (40503 * cache + 9973 * split) mod blocks.  The start decides the order of all sums and, with the running
    maximum, how the operands round, so another one moves the outputs by 5e-5 to 1e-4 of their size, as far from 64 bits as before but not what they were.
    Against outputs of that order kept in a file: sums that only differ in their own last bits turn the rounding of one output in several
    hundred (2-norm: 2^-11 of the value, so 1e-5 where one in a thousand turns)."""
    kept = np.load(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "decode_sweep_outputs.npz"))
    want, got = kept[name].astype(np.float64), sweep_outputs(kvq_mod, *SWEEPS[name]).astype(np.float64)
    assert np.linalg.norm(got - want) <= 2e-5 * np.linalg.norm(want), np.linalg.norm(got - want) / np.linalg.norm(want)
