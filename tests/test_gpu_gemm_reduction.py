"""The reduction of split-K partial sums (GPU): rows that do not fill its workgroups of four, columns
that do not fill their 256, more splits than it keeps in flight at once."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planes", [1, 2])
@pytest.mark.parametrize("M,N,K,splits", [(1, 16, 4096, 8), (3, 272, 2048, 8), (5, 1040, 4096, 8), (37, 240, 1024, 4), (6, 8208, 8192, 3), (70, 2064, 4096, 11)])
def test_partial_sums_of_ragged_shapes(M, N, K, splits, planes):
    import paper_2401_12522_amd as bita
    from paper_2401_12522_amd import binding as B
    if splits > 8:                                       # more than the heuristic gives a narrow matrix
        B.lib().bita_tune_gemm(-1, splits)
    try:
        _check(bita, B, M, N, K, splits, planes)
    finally:
        B.lib().bita_tune_gemm(-1, -1)


def _check(bita, B, M, N, K, splits, planes):
    assert B.gemm_plan_info(M, N, K)["splits"] == splits, B.gemm_plan_info(M, N, K)
    g = torch.Generator().manual_seed(M + N + K)
    a32, w = torch.randn(M, K, generator=g), (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    hi = a32.to(torch.bfloat16)
    lo = (a32 - hi.float()).to(torch.bfloat16) if planes == 2 else None
    ws = torch.full((B.lib().bita_gemm_workspace_bytes(M, N, K),), 0x7F, dtype=torch.uint8, device="cuda")   # stale values that are no sums
    out = torch.full((M, N), float("nan"), device="cuda")
    packed, a, al = bita.pack_weight(w.cuda()), hi.cuda(), lo.cuda() if planes == 2 else None
    B._check(B.lib().bita_gemm(B._ptr(a), B._ptr(al), M, K, K, B._ptr(packed), N, B._ptr(ws), ws.numel(), B._ptr(out), B._stream()))
    ref = (hi.double() + (lo.double() if planes == 2 else 0.0)) @ w.double().T
    scale = float(ref.abs().max())
    assert float((out.cpu().double() - ref).abs().max()) <= 2e-5 * scale + 1e-6         # fp32 accumulation, as everywhere
