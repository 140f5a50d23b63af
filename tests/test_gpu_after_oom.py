"""A call that found no memory has said so; the next one, with memory again, does not repeat it."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_the_call_after_one_without_memory():
    import paper_2401_08281_amd as vs
    from test_gpu_nearest import hold_memory
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.randn((4000, 64), device="cuda")
    q = torch.randn((400_000, 64), device="cuda")
    ix = vs.IVFFlat(64, 0, x[:64].contiguous())
    ix.add(x)
    D = torch.empty((400_000, 100), device="cuda")
    I = torch.empty((400_000, 100), dtype=torch.int64, device="cuda")
    vs.vs_trim()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = hold_memory(120 << 20)
    try:
        with pytest.raises(vs.VSError):
            ix.search(q, 100, 64, D, I)              # (several hundred MB of work space by either scan)
    finally:
        del hold
        torch.cuda.empty_cache()
    ix.search(q[:10].contiguous(), 5, 4)
    torch.cuda.synchronize()
    ix.close()
