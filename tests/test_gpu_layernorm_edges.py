"""LayerNorm where lanes share rows: widths around 16, 32 and 64 lanes, rows that do not fill a wavefront, several rows per lane group."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_exp", [2, 3])
@pytest.mark.parametrize("T", [1, 3, 257, 70001])
@pytest.mark.parametrize("E", [4, 60, 64, 68, 128, 132, 256, 260, 1028])
def test_outputs_against_fp64(sa, T, E, n_exp):
    if T * E > 20_000_000:
        T = 9001
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E)
    x = torch.randn((T, E), generator=g, device="cuda") * 3 + 1
    gamma, beta = (torch.randn(E, generator=g, device="cuda") for _ in range(2))
    wg, bg = torch.randn((E, n_exp), generator=g, device="cuda"), torch.randn(n_exp, generator=g, device="cuda")
    ln, q, xh, logits = sa.sa_layernorm_quant(x, gamma, beta, 1e-5, 20.0, want_q=True, want_half=True, wg=wg, bg=bg)
    ref = torch.nn.functional.layer_norm(x.double(), (E,), gamma.double(), beta.double(), 1e-5)
    torch.testing.assert_close(ln.double(), ref, rtol=1e-5, atol=2e-5)
    assert torch.equal(xh, ln.half())
    assert torch.equal(q, (ln * 20.0).round().clamp(-127, 127).to(torch.int8))
    torch.testing.assert_close(logits.double(), ref @ wg.double() + bg.double(), rtol=1e-4, atol=1e-3)
