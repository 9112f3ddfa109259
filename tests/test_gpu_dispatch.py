"""Which kernels a call launches, at sizes where another choice is slower (torch's profiler lists them)."""
import sys

import pytest
import torch
from torch.profiler import ProfilerActivity, profile

from paper_2609_34370_amd import spexis as sx

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def launched(call) -> list:
    """Names of this library's kernels that call() launches, without their arguments."""
    call()   # the first call loads the kernels
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in p.events() if "spexis::" in e.name]
    return [n[n.index("spexis::") + len("spexis::"):].split("(")[0] for n in names]


def zeros(*shape):
    return torch.zeros(shape, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("batch,ctx,group,dim,merge", [
    (1, 1024, 8, 64, "attn_merge_kernel"),         # 16 shares of a sequence, 8 rows of 64
    (1, 1024, 9, 64, "attn_merge_wide_kernel"),
    (1, 1024, 8, 128, "attn_merge_wide_kernel"),
    (1, 2048, 8, 64, "attn_merge_wide_kernel"),
    (64, 1024, 8, 128, "attn_merge_kernel"),
])
def test_attention_merge(batch, ctx, group, dim, merge):
    hkv, bs = 2, 32
    nb = ctx // bs
    pool = torch.zeros(batch * nb * hkv * bs * dim, dtype=torch.bfloat16, device="cuda")
    q = torch.zeros((batch, hkv * group, dim), dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    qsl = torch.arange(batch + 1, dtype=torch.int32, device="cuda")
    lens = torch.full((batch,), ctx, dtype=torch.int32, device="cuda")
    tables = torch.arange(batch * nb, dtype=torch.int32, device="cuda").view(batch, nb)
    ws = torch.empty(sx.spexis_verify_attention_workspace_size(batch, hkv * group, hkv, dim, 1, ctx), dtype=torch.uint8,
                     device="cuda")
    got = launched(lambda: sx.spexis_verify_attention(pool, pool, batch * nb, hkv, bs, dim, qsl, lens, tables, batch, 1,
                                                      ctx, q, hkv * group, dim ** -0.5, out, ws))
    say(f"[merge] {batch} x {ctx}, {group} rows of {dim}: {got}")
    assert [n.split("<")[0] for n in got] == ["verify_attn_kernel", merge]


def accept_kernels(kind, B, V, k):
    T = B * (k + 1)
    qsl = torch.arange(B + 1, dtype=torch.int32, device="cuda") * (k + 1)
    # equal probabilities, every draft accepted
    rows = torch.full((T, V), 1.0 / V if kind == sx.SPEXIS_INPUT_PROBS else 0.0, device="cuda")
    u, us, ids = torch.zeros(T - B, device="cuda"), torch.full((B,), 0.5, device="cuda"), zeros(T - B)
    ws = torch.empty(sx.spexis_accept_workspace_size(B, V, k), dtype=torch.uint8, device="cuda")
    a, tok, status = zeros(B), zeros(B, k + 1), zeros(B)
    got = launched(lambda: sx.spexis_accept(kind, qsl, rows, rows[: T - B], ids, u, us, k, a, tok, status, ws))
    say(f"[accept] kind {kind}, {B} x {k} drafts of {V}: {got}")
    assert (status == 0).all() and (a == k).all() and (tok[:, k] == V // 2).all()
    return [n.split("<")[0] for n in got]


@pytest.mark.parametrize("B,V,k,one", [
    (1, 4096, 16, True), (1, 4096, 32, False), (16, 4096, 32, True), (256, 4096, 32, True), (512, 4096, 32, False),
    (1024, 4096, 8, True), (1024, 4096, 16, False), (1, 4095, 4, True), (1, 4095, 8, False), (64, 4095, 8, True),
    (64, 4095, 16, False), (256, 4095, 32, True), (1, 1000, 32, True), (1, 999, 32, False), (4, 4097, 2, False),
    (1024, 999, 0, False), (512, 999, 0, True), (1024, 1000, 0, True),
])
def test_short_logit_rows_are_read_whole_while_they_are_few(B, V, k, one):
    assert (accept_kernels(sx.SPEXIS_INPUT_LOGITS, B, V, k) == ["accept_short_kernel"]) == one


@pytest.mark.parametrize("B,V,k,one", [
    (1, 16384, 0, True), (512, 16385, 0, False), (512, 32000, 0, False), (1, 32000, 1, False), (16, 32000, 4, False),
    (16, 32000, 8, True), (64, 32000, 2, True), (128, 32000, 1, True), (64, 31999, 2, False), (128, 31999, 1, True),
    (64, 16385, 2, True), (64, 16385, 1, False), (128, 32772, 8, False),
])
def test_long_probability_rows_need_many_residuals(B, V, k, one):
    assert (accept_kernels(sx.SPEXIS_INPUT_PROBS, B, V, k) == ["accept_probs_kernel"]) == one


def head_kernels(rows, V, d=256):
    h = torch.zeros((rows, d), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros(sx.spexis_packed_weight_size(V, d) // 2, dtype=torch.bfloat16, device="cuda")
    logits = torch.empty((rows, V), device="cuda")
    stats = torch.empty((rows, sx.spexis_lm_head_tiles(V), 2), device="cuda")
    got = launched(lambda: sx.spexis_lm_head(h, w, stats, logits=logits))
    say(f"[head] {rows} @ {V}: {got}")
    assert len(got) == 1 and (logits == 0).all()
    return got[0]


@pytest.mark.parametrize("rows,V,kernel", [
    (160, 32000, "lm_head_pair_kernel<5"), (192, 32000, "lm_head_wide_kernel<3"), (320, 32000, "lm_head_wide_kernel<5"),
    (321, 32000, "lm_head_kernel<false, 6"), (384, 32000, "lm_head_kernel<false, 6"),   # one round, not one and a half
    (480, 32000, "lm_head_pair_kernel<5"), (512, 32000, "lm_head_pair_kernel<4"), (640, 32000, "lm_head_wide_kernel<5"),
    (768, 16000, "lm_head_kernel<false, 6"), (832, 20000, "lm_head_wide_kernel<5"),     # one round, not two
    (352, 65024, "lm_head_pair_kernel<4"), (352, 4096, "lm_head_pair_kernel<4"),
])
def test_head_rows_follow_the_rounds_of_workgroups(rows, V, kernel):
    got = head_kernels(rows, V)
    assert got.startswith(kernel), got


@pytest.mark.parametrize("rows,n_out,n_in,kernel", [
    (1, 256, 4096, "linear_kernel<1, 1, 8"), (1, 256, 8192, None), (32, 1024, 8192, None), (32, 5120, 8192, "linear_kernel<1, 1, 8"),
    (64, 2048, 6144, "linear_kernel<1, 1, 8"), (64, 2048, 8192, None), (1, 32768, 256, None), (64, 32768, 1024, "linear_kernel<2, 2, 4"),
    (128, 6144, 8192, "linear_kernel<2, 2, 4"), (128, 10240, 8192, None), (160, 6144, 8192, None),
    (320, 4096, 4096, "linear_kernel<2, 2, 4"), (320, 4096, 8192, None), (512, 3584, 8192, "linear_kernel<2, 2, 4"),
    (2048, 2048, 8192, None),
])
def test_adapter_layers_take_the_quicker_kernel(rows, n_out, n_in, kernel):
    # None: the projection, its K split over workgroups, and the reduce
    x = torch.zeros((rows, n_in), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros(sx.spexis_packed_weight_size(n_out, n_in) // 2, dtype=torch.bfloat16, device="cuda")
    y = torch.empty((rows, n_out), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(sx.spexis_linear_workspace_size(rows, n_out, n_in), 1), dtype=torch.uint8, device="cuda")
    got = launched(lambda: sx.spexis_linear(x, w, y, workspace=ws))
    say(f"[linear] {rows} x {n_out} x {n_in}: {got}")
    assert (y == 0).all()
    if kernel:
        assert len(got) == 1 and got[0].startswith(kernel)
    else:
        assert got[0].startswith("lm_head") and got[1:] in ([], ["linear_reduce_kernel"])
