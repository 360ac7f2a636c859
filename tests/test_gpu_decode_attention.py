"""Attention of a decoding step through tfm_op_decode_attention, against its definition in 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UNIT = {"fp16": 2.0 ** -11, "bf16": 2.0 ** -8, "fp32": 2.0 ** -24}     # a result's rounding to the type, relative


def _dtype(prec):
    import torch
    return {"fp16": torch.float16, "bf16": torch.bfloat16, "fp32": torch.float32}[prec]


def _check(q, k, v, beam, places, sample, prec):
    """q [rows, H, dh], k and v [positions, H, dh] on the GPU; places: an ancestry table [rows, n] of the history (position s of row r in line places[r, s]
    of the caches) or the offsets of the sources (a list).  Compares the rows in `sample` and returns the largest result.

    The bound: the result's own rounding; a score's products of 2-byte values are exact and their sum is good to 16 roundings of the size of its terms,
    which two scores bring into a weight; a weight to 2^-20 (exponent, exponential, division), and the sum of n weighted values to n roundings."""
    import torch
    import paper_1904_01038_amd as T
    rows, H, dh = q.shape
    q, k, v = (x.reshape(x.shape[0], H * dh).to(_dtype(prec)) for x in (q, k, v))
    o = torch.zeros_like(q)
    if isinstance(places, list):
        n = max(b - a for a, b in zip(places, places[1:]))
        T.ops.decode_attention(q, k, v, o, H, dh, beam=beam, src_off=torch.tensor(places, dtype=torch.int32).cuda(), n_max=n)
        at = [torch.arange(places[r // beam], places[r // beam + 1]) for r in sample]
    else:
        n, steps = places.shape[1], k.shape[0] // rows
        anc = np.full((rows, steps), -10 ** 6, np.int32)     # (what lies behind position t is not looked at)
        anc[:, :n] = places
        T.ops.decode_attention(q, k, v, o, H, dh, beam=beam, anc=torch.tensor(anc).cuda(), t=n - 1)
        at = [torch.tensor(places[r].astype(np.int64) * steps + np.arange(n)) for r in sample]
    largest = 0.0
    for r, where in zip(sample, at):
        got, qr = (x[r].cpu().double().view(H, 1, dh) for x in (o, q))
        kr, vr = (x[where.cuda()].cpu().double().view(-1, H, dh).transpose(0, 1) for x in (k, v))         # [H, positions, dh]
        w = torch.softmax((qr * kr).sum(2, keepdim=True) * dh ** -0.5, 1)
        size = (qr.abs() * kr.abs()).sum(2, keepdim=True).amax(1, keepdim=True) * dh ** -0.5
        ref, weighted = (w * vr).sum(1, keepdim=True), (w * vr.abs()).sum(1, keepdim=True)
        bound = UNIT[prec] * ref.abs() + 2.0 ** -25 + (2 * 16 * 2.0 ** -24 * size + 2.0 ** -20 + n * 2.0 ** -24) * weighted
        assert bool(((got - ref).abs() <= bound).all()), (n, int(r), float(((got - ref).abs() / bound).max()))
        largest = max(largest, float(ref.abs().max()))
    return largest


def _lines(rng, rows, beam, n):
    return (np.arange(rows)[:, None] // beam * beam + rng.integers(0, beam, (rows, n))).astype(np.int32)


@pytest.mark.parametrize("prec", ["fp16", "bf16", "fp32"])
@pytest.mark.parametrize("over", ["history", "source"])
@pytest.mark.parametrize("scale", [3e-6, 2e-4, 1.0, 8.0])
def test_scores_are_formed_in_32_bits(prec, over, scale):
    """Values of +1 and -1 on two positions whose scores nearly cancel: the result is half the difference of the scores, to some 2^-11 of itself.  Keys of
    3e-6 are subnormal in fp16; a 16-bit dot product loses 1.6e-5 of a score there."""
    import torch
    rng = np.random.default_rng(int(scale * 1e6))
    rows, H, dh, beam = 40, 2, 64, 4
    lines = rows if over == "history" else rows // beam
    q = np.clip(rng.standard_normal((rows, H, dh)) * min(2.0 / scale, 2e4), -6e4, 6e4)
    k = np.repeat(rng.standard_normal((lines, 1, H, dh)) * scale, 2, axis=1)
    k[:, 1] *= np.where(rng.random((lines, H, dh)) < 0.05, 1.25, 1.0)
    v = np.broadcast_to(np.array([1.0, -1.0])[:, None, None], k.shape)
    # the two positions of a row lie side by side: in one line of the caches, or as a sentence of their own
    places = np.repeat(_lines(rng, rows, beam, 1), 2, axis=1) if over == "history" else list(range(0, 2 * lines + 1, 2))
    on_gpu = [torch.tensor(np.ascontiguousarray(x).reshape(-1, H, dh)).cuda() for x in (q, k, v)]
    assert _check(*on_gpu, beam, places, range(rows), prec) > 1e-3


# 64, 1020, 2048, 2052, 3072, 4096 and 4288 wavefronts: on either side of the lines from which chunks of 32 positions are taken instead of 64
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("over", ["history", "source"])
@pytest.mark.parametrize("rows,H,beam", [(16, 4, 4), (255, 4, 5), (512, 4, 1), (513, 4, 9), (192, 16, 4), (256, 16, 4), (268, 16, 4)])
def test_chunks_of_positions_for_all_numbers_of_wavefronts(prec, over, rows, H, beam):
    import torch
    rng, gen = np.random.default_rng(rows), torch.Generator(device="cuda").manual_seed(rows)
    dh, sentences = 64, rows // beam
    sample = np.unique(np.r_[0, rows - 1, rng.integers(0, rows, 20)])
    for n in (1, 31, 32, 33, 48, 63, 64, 65, 96, 97, 128, 129):
        if over == "history":
            count, places = rows * (n + 1), _lines(rng, rows, beam, n)
        else:                                            # lengths up to n, the first and the last one n
            lens = rng.integers(max(1, n - 40), n + 1, sentences)
            lens[[0, -1]] = n
            places = [0] + np.cumsum(lens).tolist()
            count = places[-1]
        q, k, v = (torch.randn(c, H, dh, generator=gen, device="cuda") for c in (rows, count, count))
        _check(2 * q, k, v, beam, places, sample, prec)


def test_arguments_are_checked():
    import torch
    import paper_1904_01038_amd as T
    q, k, o = (torch.zeros(n, 128, dtype=torch.float16, device="cuda") for n in (8, 64, 8))
    off = torch.tensor([0, 32, 64], dtype=torch.int32, device="cuda")
    anc = torch.zeros(8, 8, dtype=torch.int32, device="cuda")
    good = dict(H=2, dh=64, beam=4, src_off=off, n_max=32)
    T.ops.decode_attention(q, k, k, o, **good)
    for change in (dict(beam=3), dict(H=3), dict(dh=60), dict(n_max=0), dict(n_max=5000), dict(src_off=None), dict(anc=anc)):
        with pytest.raises(T.TfmError):
            T.ops.decode_attention(q, k, k, o, **{**good, **change})
    with pytest.raises(T.TfmError):                      # past the caches' last step
        T.ops.decode_attention(q, k, k, o, H=2, dh=64, beam=4, anc=anc, t=8)
    with pytest.raises(T.TfmError):                      # rows 2 bytes off a multiple of 16
        T.ops.decode_attention(q.reshape(-1)[1:897].view(7, 128), k, k, o, **{**good, "beam": 7})
