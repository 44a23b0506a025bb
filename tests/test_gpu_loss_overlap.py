"""cae_mlp_loss_grad with its loss word inside one of its arrays, at lengths whose gradient has
workgroups of its own when every array is apart: the loss is written after every read and write of
the other words, so the loss and the gradient have the bits that separate arrays give."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["y", "t", "dy"])
@pytest.mark.parametrize("n,at", [(2049, 0), (70000, 69999), (70000, 1500)])
def test_loss_word_inside_an_array(where, n, at):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import _lib
    L = _lib.lib()
    g = torch.Generator(device="cuda")
    g.manual_seed(n + at)
    y, t = (torch.randn(n, generator=g, device="cuda") for _ in range(2))
    dy, loss = torch.zeros(n, device="cuda"), torch.zeros(1, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream

    def call(a, b, c, word):
        assert L.cae_mlp_loss_grad(a.data_ptr(), b.data_ptr(), c.data_ptr(), word.data_ptr(), n, 1, 0.1, stream) == 0

    call(y, t, dy, loss)
    arrays = {"y": y.clone(), "t": t.clone(), "dy": torch.zeros(n, device="cuda")}
    word = arrays[where][at:at + 1]
    call(arrays["y"], arrays["t"], arrays["dy"], word)
    assert torch.equal(word, loss)
    want = {"y": y, "t": t, "dy": dy}
    for name, a in arrays.items():
        keep = torch.ones(n, dtype=torch.bool, device="cuda")
        keep[at] = name != where
        assert torch.equal(a[keep], want[name][keep]), name
