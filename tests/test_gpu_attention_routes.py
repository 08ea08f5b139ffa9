"""bf16 attention along each of its kernels at the sizes where they hand over to
one another: 16 queries per wave (few query tiles), the single-block kernels
above it, and the block-pair kernel (long rows of long sequences).  Every case against the oracle, with the general list forms (empty,
unsorted, out of range, repeated, the partial last block) and with a block whose
logits overflow the fixed reference.
"""
import numpy as np
import pytest

import oracle
import paper_2606_23743_amd as sva
from paper_2606_23743_amd import inputs, workloads

from . import parity
from .gpu_cases import device_inputs, say, scale_of, takes_pairs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SC = workloads.small_case


def _check(out, lse, f64, rows_of, S, scale, sample):
    """Query blocks `sample` = [(h, i)] of out, lse [1, H, N(, D)] against the oracle
    on the entries of rows_of(h, i) that are in range."""
    H, N = lse.shape[1:]
    nb = -(-N // S)
    o, s = out.float().cpu().numpy(), lse.cpu().numpy()
    for h, i in sample:
        kept = [j for j in rows_of(h, i) if 0 <= j < nb]
        one = {n: x[:, h:h + 1] for n, x in f64.items()}
        ref, rlse = oracle.block_sparse_attention(one["q"], one["k"], one["v"], [[{i: kept}]], S, scale,
                                                  rows=[(0, 0, i)])
        sl = slice(i * S, min(N, (i + 1) * S))
        if not kept:
            assert np.all(o[0, h, sl] == 0) and np.all(np.isneginf(s[0, h, sl])), (h, i)
            continue
        mx, mean = parity.attention_errors(o[0, h, sl], ref[0, 0, sl], np.ones(ref[0, 0, sl].shape, dtype=bool))
        assert mx <= parity.MAX_ABS and mean <= parity.MEAN_ABS, (h, i, mx, mean)
        err = np.abs(s[0, h, sl] - rlse[0, 0, sl])
        assert np.all(err <= parity.LSE_TOL + 1e-5 * np.abs(rlse[0, 0, sl])), (h, i, err.max())


def _general_rows(nb, kmax, rng):
    last = nb - 1
    kinds = [[], [last], [last] * kmax, list(range(min(kmax, nb)))[::-1], [-1, 0, nb, 1 << 30, last],
             [0, 0, last], list(rng.permutation(nb)[:kmax])]
    return lambda i: [int(j) for j in kinds[i % len(kinds)][:kmax]]


def _arrays(rows, H, nb, kmax):
    idx = np.full((1, H, nb, kmax), -1, dtype=np.int32)
    cnt = np.zeros((1, H, nb), dtype=np.int32)
    for i in range(nb):
        idx[0, :, i, :len(rows(i))] = rows(i)
        cnt[0, :, i] = len(rows(i))
    return torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()


# (D, S, heads, grid, kmax): both sides of 512 tiles; the last block holds 5
# tokens or the sequence is under one block
@pytest.mark.parametrize("D,S,H,grid,kmax", [
    (64, 64, 2, (3, 43, 5), 8), (112, 64, 2, (3, 43, 5), 7), (112, 64, 2, (3, 43, 5), 11), (128, 64, 2, (1, 1, 901), 12),
    (128, 64, 2, (1, 1, 901), 15), (112, 128, 2, (1, 1, 901), 4), (128, 128, 2, (1, 1, 901), 8), (128, 128, 2, (1, 1, 901), 3),
    (64, 128, 1, (1, 1, 901), 7), (128, 128, 1, (1, 3, 1), 1), (128, 64, 18, (1, 1, 901), 8),
    (64, 128, 34, (1, 1, 901), 4), (112, 64, 35, (1, 1, 901), 8), (128, 128, 35, (1, 1, 901), 6)])
def test_narrow_and_wide_general_lists(D, S, H, grid, kmax):
    wl = SC(f"routes_{D}_{S}_{H}_{kmax}", 1, H, D, grid, S, "topk", topk=1, seed=500 + kmax)
    bits = inputs.generate(wl)
    dev = device_inputs(bits)
    N = wl.seq_len
    nb = -(-N // S)
    rows = _general_rows(nb, kmax, np.random.default_rng(kmax))
    idx, cnt = _arrays(rows, H, nb, kmax)
    f64 = {n: oracle.bf16_bits_to_f64(bits[n]) for n in ("q", "k", "v")}
    prob = sva.problem_for(wl)
    say(f"[routes] D={D} S={S} tiles={H * -(-N // 64)} chunks={min(kmax, nb) * S // 32}")
    out, lse = sva.sparse_attention(prob, dev["q"], dev["k"], dev["v"], idx, cnt, want_lse=True)
    torch.cuda.synchronize()
    _check(out, lse, f64, lambda h, i: rows(i), S, scale_of(wl), [(h, i) for h in {0, H - 1} for i in range(nb)])
    out, lse = sva.dense_attention(prob, dev["q"], dev["k"], dev["v"], want_lse=True)
    torch.cuda.synchronize()
    _check(out, lse, f64, lambda h, i: range(nb), S, scale_of(wl), [(h, i) for h in {0, H - 1} for i in range(nb)])


@pytest.mark.parametrize("D,S", [(64, 64), (112, 64), (128, 64), (64, 128), (112, 128), (128, 128)])
@pytest.mark.parametrize("f32", [False, True])
def test_a_head_does_not_depend_on_its_call(D, S, f32):
    """One head alone (25 query tiles), in a call of 22 heads (550 tiles, past the
    512 from which 32 queries share a wave) and, sparse, with its lists in
    longer rows: the same bits, dense and sparse."""
    H, N = 22, 1560
    say(f"[routes one head D={D} S={S} f32={f32}]")
    g = torch.Generator(device="cuda").manual_seed(D + S)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda").bfloat16() for _ in "qkv")
    nb = -(-N // S)
    kept = 5
    idx = torch.rand((1, H, nb, nb), generator=g, device="cuda").argsort(-1)[..., :kept].sort(-1)[0].int().contiguous()
    cnt = torch.full((1, H, nb), kept, dtype=torch.int32, device="cuda")
    dt = "f32" if f32 else "bf16"
    every, one = (sva.problem(1, h, N, D, (1, 1, N), S, out_dtype=dt) for h in (H, 1))
    dense = sva.dense_attention(every, q, k, v, want_lse=True)
    sparse = sva.sparse_attention(every, q, k, v, idx, cnt, want_lse=True)
    for h in (0, H - 1):
        qh, kh, vh = (x[:, h:h + 1].contiguous() for x in (q, k, v))
        for x, y in zip(dense, sva.dense_attention(one, qh, kh, vh, want_lse=True)):
            assert torch.equal(x[:, h:h + 1], y), h
        for kmax in (kept, nb, 4 * nb):
            rows = torch.full((1, 1, nb, kmax), -1, dtype=torch.int32, device="cuda")
            rows[..., :kept] = idx[:, h:h + 1]
            got = sva.sparse_attention(one, qh, kh, vh, rows, cnt[:, h:h + 1].contiguous(), want_lse=True)
            for x, y in zip(sparse, got):
                assert torch.equal(x[:, h:h + 1], y), (h, kmax)


@pytest.mark.parametrize("D,S,H", [(128, 64, 65), (64, 128, 65), (112, 64, 65), (128, 128, 65), (128, 64, 2),
                                   (64, 64, 1), (112, 128, 1)])
def test_overflow_is_walked_again(D, S, H):
    """A later kept block whose logits exceed the first chunk's reference by
    about 1000 (log2 units), with more than 512 query tiles (65 heads) and fewer."""
    wl = SC(f"routes_over_{D}_{S}_{H}", 1, H, D, (4, 8, 16), S, "topk", topk=2, seed=520)
    bits = inputs.generate(wl)
    f = {n: inputs.bf16_bits_to_f32(bits[n]).copy() for n in ("q", "k", "v")}
    f["k"][0, :, 0:S] *= 1e-3
    f["q"][0, :, 128:256] = 8.0 * (128 / D)
    f["k"][0, :, 384:512] = 8.0
    bits = {n: inputs._round_bf16(f[n]) for n in f}
    dev = device_inputs(bits)
    nb = 512 // S
    hot = list(range(384 // S, nb))
    rows = lambda i: [0] + hot + [1] if i * S >= 128 else [0, 1]   # noqa: E731
    idx, cnt = _arrays(rows, H, nb, 1024 // S)
    out, lse = sva.sparse_attention(sva.problem_for(wl), dev["q"], dev["k"], dev["v"], idx, cnt, want_lse=True)
    torch.cuda.synchronize()
    assert lse.max().item() > 400.0                  # the regime this test is about
    f64 = {n: oracle.bf16_bits_to_f64(bits[n]) for n in ("q", "k", "v")}
    _check(out, lse, f64, lambda h, i: rows(i), S, scale_of(wl), [(h, i) for h in {0, H - 1} for i in range(nb)])


@pytest.mark.parametrize("D,S,H", [(112, 64, 2), (112, 128, 2), (112, 64, 40), (112, 128, 40), (64, 64, 2),
                                   (128, 128, 40)])
def test_infinite_keys_and_values(D, S, H):
    """Keys with -Inf in one of the first eight channels (the piece that stands in
    for the padding of D = 112) against queries that are positive there: logits of
    -Inf, weight zero.  Then an Inf in V at the first row of the last chunk (which
    stands in for the rows past the end): that channel is Inf, the others finite.
    Some lists begin with a block of which every key is -Inf.
    In calls of 30 and of 600 query tiles."""
    N = 901
    wl = SC(f"routes_inf_{D}_{S}_{H}", 1, H, D, (1, 1, N), S, "topk", topk=1, seed=540)
    f = {n: inputs.bf16_bits_to_f32(x).copy() for n, x in inputs.generate(wl).items()}
    f["q"][..., 3] = np.abs(f["q"][..., 3]) + 0.5
    f["k"][0, :, [40, 130, 900], 3] = -np.inf
    f["k"][0, :, 5 * S:6 * S, 3] = -np.inf
    nb = -(-N // S)
    rows = lambda i: [[nb - 1, 0], [0, 130 // S, nb - 1], [5, 0, nb - 1]][i % 3]   # noqa: E731
    idx, cnt = _arrays(rows, H, nb, 4)
    prob, every = sva.problem_for(wl), lambda h, i: range(nb)
    say(f"[routes inf D={D} S={S} H={H}]")

    def run(v):
        bits = {n: inputs._round_bf16(x) for n, x in dict(f, v=v).items()}
        dev = device_inputs(bits)
        got = [sva.sparse_attention(prob, dev["q"], dev["k"], dev["v"], idx, cnt, want_lse=True),
               sva.dense_attention(prob, dev["q"], dev["k"], dev["v"], want_lse=True)]
        torch.cuda.synchronize()
        return got, {n: oracle.bf16_bits_to_f64(bits[n]) for n in ("q", "k", "v")}

    sample = [(h, i) for h in {0, H - 1} for i in range(nb)]
    got, f64 = run(f["v"])
    for (out, lse), lists in zip(got, (lambda h, i: rows(i), every)):
        _check(out, lse, f64, lists, S, scale_of(wl), sample)
    v = f["v"].copy()
    v[0, :, N // 32 * 32, 5] = np.inf
    got, f64 = run(v)
    f64["v"][0, :, N // 32 * 32, 5] = 0.0            # the other channels of the oracle
    for (out, lse), lists in zip(got, (lambda h, i: rows(i), every)):
        assert torch.isposinf(out[..., 5]).all()
        out[..., 5] = 0
        f64["v"][..., 5] = 0.0
        _check(out, lse, f64, lists, S, scale_of(wl), sample)


@pytest.mark.parametrize("nb,dtype", [(902, "bf16"), (901, "bf16"), (901, "f32")])
def test_pairs_of_long_sequences(nb, dtype):
    """The block-pair kernel, the last pair with one block at 901.  Ascending and
    general lists match the single-block kernel (the same lists in short rows) bit
    for bit and the oracle; lists too long for a pair's union and overflowing
    blocks match the oracle."""
    S, D, H, N = 64, 128, 2, (nb - 1) * 64 + 37
    say(f"[routes pairs nB={nb} {dtype}]")
    wl = SC("routes_pairs", 1, H, D, (1, 1, N), S, "topk", topk=1, seed=530)
    bits = inputs.generate(wl)
    assert takes_pairs(H, N, S, D, nb) and not takes_pairs(H, N, S, D, 12)
    rng = np.random.default_rng(5)
    asc = {i: sorted({int(j) for j in rng.integers(0, nb, 10)} | ({nb - 1} if i % 3 == 0 else set()))
           for i in range(nb)}
    prob, f64 = sva.problem_for(wl, out_dtype=dtype), {n: oracle.bf16_bits_to_f64(bits[n]) for n in ("q", "k", "v")}
    dev = device_inputs(bits)
    for rows in (asc.__getitem__, _general_rows(nb, 12, rng)):
        wide, cnt = _arrays(rows, H, nb, nb)
        o1, l1 = sva.sparse_attention(prob, dev["q"], dev["k"], dev["v"], wide, cnt, want_lse=True)
        o2, l2 = sva.sparse_attention(prob, dev["q"], dev["k"], dev["v"], wide[..., :12].contiguous(), cnt, want_lse=True)
        torch.cuda.synchronize()
        assert torch.equal(o1, o2) and torch.equal(l1, l2)
        _check(o1, l1, f64, lambda h, i: rows(i), S, scale_of(wl), [(0, i) for i in list(range(14)) + [nb - 2, nb - 1]])

    many = {i: [int(j) for j in rng.integers(-1, nb, n)] for i, n in ((2, 2100), (3, 2100), (nb - 1, 4200))}
    rows = lambda i: many.get(i, [i])   # noqa: E731
    idx, cnt = _arrays(rows, H, nb, 4200)
    out, lse = sva.sparse_attention(prob, dev["q"], dev["k"], dev["v"], idx, cnt, want_lse=True)
    torch.cuda.synchronize()
    _check(out, lse, f64, lambda h, i: rows(i), S, scale_of(wl), [(0, i) for i in (1, 2, 3, nb - 2, nb - 1)])

    f = {n: inputs.bf16_bits_to_f32(bits[n]).copy() for n in ("q", "k", "v")}
    f["k"][0, :, 0:64] *= 1e-3
    f["q"][0, :, 128:256] = 8.0                      # query blocks 2 and 3
    f["q"][0, :, (nb - 1) * 64:] = 8.0               # and the last
    f["k"][0, :, 384:512] = 8.0                      # key blocks 6 and 7
    bits = {n: inputs._round_bf16(f[n]) for n in f}
    dev, f64 = device_inputs(bits), {n: oracle.bf16_bits_to_f64(bits[n]) for n in ("q", "k", "v")}
    rows = lambda i: [0, 6, 7] if i in (2, 3, 5, nb - 1) else [0, 1]   # noqa: E731
    idx, cnt = _arrays(rows, H, nb, nb)
    out, lse = sva.sparse_attention(prob, dev["q"], dev["k"], dev["v"], idx, cnt, want_lse=True)
    torch.cuda.synchronize()
    assert lse[0, 0, 128].item() > 400.0 and lse[0, 0, -1].item() > 400.0      # the regime this part is about
    _check(out, lse, f64, lambda h, i: rows(i), S, scale_of(wl), [(0, i) for i in list(range(8)) + [nb - 2, nb - 1]])
