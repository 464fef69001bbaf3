"""Argument checks of the native tensor entry points that need no GPU: what is refused, and with which exception."""
import pytest
import torch


@pytest.fixture(scope="module")
def binding():
    from paper_2603_01960_amd import binding
    if not binding.library_path().exists():
        pytest.skip("library not built")
    return binding


def test_host_tensors_and_other_objects_are_refused(binding):
    x = torch.zeros(1, 2, 8, 64, dtype=torch.float16)
    lens = torch.ones(1, dtype=torch.int32)
    for bad in (x, None, 3, [1.0]):
        for call in (lambda: binding.sdpa(bad, bad, bad), lambda: binding.sdpa_kv(bad, bad, bad),
                     lambda: binding.sdpa_paged(bad, bad, bad, lens, lens.view(1, 1)),
                     lambda: binding.sdpa_backward(bad, bad, bad, bad, bad, bad)):
            with pytest.raises(ValueError, match="device tensor"):
                call()


def test_keyword_names_and_defaults_of_the_tensor_functions(binding):
    import inspect
    names = lambda f: [(p.name, p.default) for p in inspect.signature(f).parameters.values() if p.default is not p.empty]
    assert names(binding.sdpa) == [("causal", False), ("scale", None), ("return_lse", False), ("out", None), ("lse_out", None),
                                   ("tile", None), ("flags", 0)]
    assert names(binding.sdpa_kv) == [("causal", False), ("scale", None), ("splits", 0), ("return_lse", False), ("out", None),
                                      ("workspace", None), ("tile", None), ("flags", 0), ("kv_lens", None)]
    assert names(binding.sdpa_paged) == [("causal", False), ("scale", None), ("splits", 0), ("return_lse", False), ("out", None),
                                         ("workspace", None), ("tile", None), ("flags", 0)]
    assert names(binding.sdpa_backward) == [("causal", False), ("scale", None), ("workspace", None), ("grads", None)]
