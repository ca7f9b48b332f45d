"""The convolution's channel-last mask and output may start at any bf16: the
kernel moves four channels at a time, whatever their address."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_mask_and_output_at_any_element(offset):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_21180_amd import cbct
    print(f"[conv] views {offset} elements into their buffers", flush=True)
    grid = (3, 5, 70)
    S = grid[0] * grid[1] * grid[2]
    torch.manual_seed(offset)
    x = torch.randn(S, 16, device="cuda").to(torch.bfloat16)
    mask = torch.randn(S, 16, device="cuda").to(torch.bfloat16)
    w = cbct.conv3_weights(0.2 * torch.randn(16, 16, 3, 3, 3, device="cuda"))
    ref = torch.empty_like(x)
    cbct.conv3(grid, x, w, transpose_w=True, mask=mask, y_cl=ref)

    def view():
        return torch.zeros(S * 16 + 8, device="cuda", dtype=torch.bfloat16)[offset:offset + S * 16].view(S, 16)

    m, y = view(), view()
    m.copy_(mask)
    assert m.data_ptr() % 8 == 2 * offset and y.data_ptr() % 8 == 2 * offset
    cbct.conv3(grid, x, w, transpose_w=True, mask=m, y_cl=y)
    assert torch.equal(y, ref)
