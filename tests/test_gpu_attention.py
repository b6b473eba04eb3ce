"""GPU parity of p4q_attention_prefill against the oracle (float64 softmax
attention).  Tolerance, from the arithmetic: the softmax weights are rounded
to the input dtype before the P V product (at most half an ulp each, so at
most 2^-11 (fp16) / 2^-8 (bf16) of max|v| in total), and both results are
rounded to that dtype (one ulp of |o| between them); the bound used is twice
that: |o - ref| <= 2^-10 max|v| + 2^-9 |ref| (fp16), 2^-7 max|v| + 2^-6 |ref|
(bf16)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34867_amd as p4q
from workload import random_features
from gpu_util import Guarded, check_canaries, to_gpu, to_np

pytestmark = pytest.mark.gpu
D = 128


def make_qkv(seed, B, L, H, dtype, std=1.0):
    """One fused [B*L, 3*H*D] q|k|v buffer, as the q|k|v projection writes it."""
    return random_features(seed, B * L, 3 * H * D, dtype, outliers=0, std=std)


def tol(dtype):
    return (2.0 ** -10, 2.0 ** -9) if dtype == "fp16" else (2.0 ** -7, 2.0 ** -6)


def check(qkv, B, L, H, causal=True, dtype="fp16", samples=None):
    t = to_gpu(qkv, dtype)
    HD = H * D
    go = Guarded((B * L, HD), t.dtype, "out")
    out = p4q.attention_prefill(t[:, :HD], t[:, HD:2 * HD], t[:, 2 * HD:], B, H, causal, out=go.t)
    torch.cuda.synchronize()
    check_canaries(go)
    got = oracle.as_f32(to_np(out), dtype).astype(np.float64).reshape(B, L, H, D)
    a, r = tol(dtype)
    for b in (range(B) if samples is None else samples):
        blk = qkv[b * L:(b + 1) * L].reshape(L, 3, H, D)
        ref = oracle.attention_prefill(blk[:, 0], blk[:, 1], blk[:, 2], causal, dtype)
        ref = oracle.as_f32(ref, dtype).astype(np.float64)
        vmax = np.abs(oracle.as_f32(blk[:, 2], dtype)).max(axis=(0, 2))          # per head
        err = np.abs(got[b] - ref)
        bound = a * vmax[None, :, None] + r * np.abs(ref)
        bad = np.argwhere(err > bound)
        assert bad.size == 0, (f"b={b}: {len(bad)} elements out of tolerance, first {tuple(bad[0])}: "
                               f"{got[b][tuple(bad[0])]} vs {ref[tuple(bad[0])]}")


@pytest.mark.parametrize("L", [1, 5, 32, 33, 127, 128, 129, 300])
def test_lengths_causal(L):
    check(make_qkv(61, 2, L, 3, "fp16"), 2, L, 3)


@pytest.mark.parametrize("L", [7, 200])
def test_non_causal(L):
    check(make_qkv(62, 1, L, 2, "fp16"), 1, L, 2, causal=False)


def test_bf16_and_large_logits():
    check(make_qkv(63, 1, 257, 2, "bf16", std=2.0), 1, 257, 2, dtype="bf16")
    check(make_qkv(64, 1, 160, 2, "fp16", std=3.0), 1, 160, 2)


def test_separate_buffers_and_strided_output():
    B, L, H = 2, 96, 2
    q, k, v = (to_gpu(random_features(65 + i, B * L, H * D, "fp16", outliers=0)) for i in range(3))
    out = torch.zeros((B * L, H * D + 64), dtype=torch.float16, device=q.device)
    p4q.attention_prefill(q, k, v, B, H, True, out=out[:, :H * D])
    torch.cuda.synchronize()
    assert torch.count_nonzero(out[:, H * D:]) == 0
    fused = np.concatenate([to_np(q), to_np(k), to_np(v)], axis=1)
    got = to_np(out[:, :H * D]).reshape(B, L, H, D).astype(np.float64)
    for b in range(B):
        blk = fused[b * L:(b + 1) * L].reshape(L, 3, H, D)
        ref = oracle.attention_prefill(blk[:, 0], blk[:, 1], blk[:, 2], True).astype(np.float64)
        assert np.all(np.abs(got[b] - ref) <= 2.0 ** -10 * 4 + 2.0 ** -9 * np.abs(ref))


def test_llava_next_b16_layer_sampled():
    """The bench shape: 16 samples x 704 tokens (640 kept + 64 text), 32 heads;
    first and last samples checked."""
    B, L, H = 16, 704, 32
    check(make_qkv(66, B, L, H, "fp16"), B, L, H, samples=[0, B - 1])


@pytest.mark.parametrize("L,causal,dtype", [(63, True, "bf16"), (64, True, "fp16"), (65, True, "fp16"),
                                            (192, False, "bf16"), (257, False, "fp16"), (450, True, "bf16")])
def test_tile_edges(L, causal, dtype):
    """Token counts at the edges of a 64-key tile and of a work-group's 128
    queries (wavefronts without queries among them)."""
    check(make_qkv(67 + L, 3, L, 2, dtype), 3, L, 2, causal=causal, dtype=dtype)


def test_output_rows_without_16_byte_alignment():
    """Output rows that allow 8-byte stores only: the same values, nothing
    between the rows touched."""
    B, L, H = 2, 130, 2
    t = to_gpu(make_qkv(68, B, L, H, "fp16"))
    HD = H * D
    ref = p4q.attention_prefill(t[:, :HD], t[:, HD:2 * HD], t[:, 2 * HD:], B, H, True)
    out = torch.zeros((B * L, HD + 12), dtype=torch.float16, device=t.device)
    p4q.attention_prefill(t[:, :HD], t[:, HD:2 * HD], t[:, 2 * HD:], B, H, True, out=out[:, :HD])
    assert torch.equal(out[:, :HD], ref)
    assert torch.count_nonzero(out[:, HD:]) == 0


def test_more_work_groups_than_one_grid_dimension():
    """Over 2^20 work-groups (single-token samples): the output is v."""
    B, H = 65535, 17
    HD = H * D
    g = torch.Generator(device="cuda:0").manual_seed(3)
    t = torch.randn((B, 3 * HD), generator=g, device="cuda:0", dtype=torch.float16)
    out = p4q.attention_prefill(t[:, :HD], t[:, HD:2 * HD], t[:, 2 * HD:], B, H, True)
    assert torch.equal(out, t[:, 2 * HD:])


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_nonfinite_rows_stay_behind_the_diagonal(dtype):
    """Rows of V with infinities and NaN reach no query of an earlier group of
    32 (the wavefront's queries): keys past a wavefront's last query are not
    multiplied, not even by weights of 0."""
    B, L, H = 1, 300, 2
    HD = H * D
    clean = to_gpu(make_qkv(71, B, L, H, dtype), dtype)
    ref = p4q.attention_prefill(clean[:, :HD], clean[:, HD:2 * HD], clean[:, 2 * HD:], B, H, True)
    for row, bad in ((32, float("inf")), (96, float("nan")), (160, -float("inf")), (64, float("inf")), (299, float("nan"))):
        t = clean.clone()
        t[row, 2 * HD:] = bad
        out = p4q.attention_prefill(t[:, :HD], t[:, HD:2 * HD], t[:, 2 * HD:], B, H, True)
        n = row // 32 * 32
        assert torch.equal(out[:n], ref[:n]), row
        assert not torch.isfinite(out[row]).any()


def test_fp16_output_is_rounded_once():
    """Equal scores (q = 0) and integer V: every weight is 1 and the sums are
    exact, so the output is sum * fl32(1 / L) rounded to fp16 -- once, not to
    fp32 in between.  The two differ where sum / L is a tie of fp16: the fp32
    product falls on it, the exact one beside it."""
    B, L, H = 16, 37, 40
    HD = H * D
    g = torch.Generator(device="cuda:0").manual_seed(9)

    def ints(rows, lo, hi):
        return torch.randint(lo, hi, (B, rows, HD), generator=g, device="cuda:0")

    v = torch.cat([2 * ints(20, 1500, 2048), ints(17, 1000, 2048)], 1)   # exact in fp16
    t = torch.zeros((B * L, 3 * HD), dtype=torch.float16, device="cuda:0")
    t[:, 2 * HD:] = v.view(B * L, HD).half()
    out = to_np(p4q.attention_prefill(t[:, :HD], t[:, HD:2 * HD], t[:, 2 * HD:], B, H, False))
    sums = v.double().sum(1).cpu().numpy()
    exact = sums * np.float64(np.float32(1.0) / np.float32(L))      # 17 + 24 bits: exact in float64
    once = exact.astype(np.float16)
    assert (exact.astype(np.float32).astype(np.float16) != once).mean() > 1e-3
    assert np.array_equal(out.reshape(B, L, HD), np.broadcast_to(once[:, None], (B, L, HD)))


@pytest.mark.parametrize("L", [1, 17, 62])
def test_rows_of_many_megabytes(L):
    """Row strides close to the limit L * ld * 2 < 2^31: the offsets of the
    tile's rows past L would pass 2^32 and come round to memory that is not
    the operand's.  Everything between the rows is infinite."""
    H = 2
    HD = H * D
    ld = ((1 << 30) - 1) // L // 8 * 8
    rows = to_gpu(make_qkv(72 + L, 1, L, H, "fp16"))
    ref = p4q.attention_prefill(rows[:, :HD], rows[:, HD:2 * HD], rows[:, 2 * HD:], 1, H, True)
    buf = torch.full(((L - 1) * ld + 3 * HD,), float("inf"), dtype=torch.float16, device=rows.device)
    wide = buf.as_strided((L, 3 * HD), (ld, 1))
    wide.copy_(rows)
    out = p4q.attention_prefill(wide[:, :HD], wide[:, HD:2 * HD], wide[:, 2 * HD:], 1, H, True)
    assert torch.equal(out, ref)
