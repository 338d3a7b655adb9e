"""GPU: the native module behind short calls (csrc/bnn_python.cpp) against the ctypes code of binding.py, which serves everything out of the ordinary."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bnn():
    import paper_2006_16578_amd as b
    b.load()
    return b


def bits(g, *shape, n=None):
    w = torch.randint(-2 ** 31, 2 ** 31, shape, dtype=torch.int32, device="cuda", generator=g)
    if n is not None and n % 32:
        w[..., -1] &= (1 << (n % 32)) - 1
    return w


def calls(bnn):
    """(name, positional arguments): one ordinary call of each function."""
    g = torch.Generator(device="cuda").manual_seed(5)
    ints = lambda *s: torch.randint(-40, 41, s, dtype=torch.int32, device="cuda", generator=g)
    real = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, f = bits(g, 2, 9, 7, 3, n=70), bits(g, 33, 3, 3, 3, n=70)
    return [("bmm", (bits(g, 5, 8, n=250), bits(g, 37, 12), 250)), ("bmm_thr", (bits(g, 5, 8), bits(g, 37, 8), ints(37), 256)),
            ("bconv", (x, f, 70, 1, 1)), ("bconv_thr", (x, f, ints(33), 70, 2, 1, bnn.PAD_EXCLUDE)),
            ("bconv_thr", (x, f, ints(33), 70, 1, 1, bnn.PAD_MINUS_ONE, ints(2, 9, 7, 33), True)), ("threshold_pack", (ints(3, 4, 5, 70), ints(70))),
            ("maxpool_or", (x, 70, 2, 2)), ("bmm_general_f32", (real(6, 50), real(9, 50))), ("bwn_conv_thr", (real(2, 12, 12, 3), bits(g, 40, 3, 3, 1, n=3), real(40), 3, 1, 1)),
            ("conv_f32_split_thr", (real(2, 12, 12, 3), real(40, 3, 3, 3), real(40), 2, 1))]


def same(a, b):
    if isinstance(a, tuple):
        return len(a) == len(b) and all(same(p, q) for p, q in zip(a, b))
    return a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a, b)


class Unlistened(torch.Tensor):
    pass


def test_same_results_and_the_same_refusals(bnn, monkeypatch):
    from paper_2006_16578_amd import binding
    served = []

    class Counted:
        def __getattr__(self, name):
            f = getattr(binding._load_native_module, name)
            return lambda *a: served.append(f(*a)) or served[-1]

    binding._load_native()
    binding._load_native_module = binding._native
    try:
        monkeypatch.setattr(binding, "_native", Counted())
        for name, args in calls(bnn):
            fn = getattr(bnn, name)
            fast = fn(*args)
            assert served.pop() is fast, name                       # the native module did it
            with monkeypatch.context() as m:
                m.setattr(binding, "_native", type("Off", (), {"__getattr__": lambda s, n: lambda *a: None})())
                slow = fn(*args)
            assert same(fast, slow), name
            # not plain: numbers that are no int, a subclass, another stream: the same results
            odd = [np.int64(a) if type(a) is int and name != "bwn_conv_thr" else a for a in args]       # (whose channels ctypes takes as int only)
            assert same(fn(*odd), slow) and (served.pop() is None or not any(type(a) is np.int64 for a in odd)), name
            sub = [a.as_subclass(Unlistened) if torch.is_tensor(a) else a for a in args]
            r = fn(*sub)
            assert served.pop() is None and same(tuple(t.as_subclass(torch.Tensor) for t in r) if isinstance(r, tuple) else r.as_subclass(torch.Tensor), slow), name
            s = torch.cuda.Stream()
            s.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s):
                r = fn(*args)
            s.synchronize()
            assert served.pop() is r and same(r, slow), name
            # refused as ever, by type
            tensors = [i for i, a in enumerate(args) if torch.is_tensor(a)]
            for i in tensors:
                for bad, error in ((args[i].cpu(), TypeError), (args[i].double(), TypeError), (args[i].unsqueeze(0).unsqueeze(0).unsqueeze(0), (ValueError, RuntimeError))):
                    if name == "threshold_pack" and i == 0 and error is not TypeError:
                        continue                                    # (any shape)
                    with pytest.raises(error):
                        fn(*args[:i], bad, *args[i + 1:])
                if args[i].dim() > 1 and args[i].shape[-1] > 1 and args[i].shape[0] > 1:
                    with pytest.raises(ValueError):
                        fn(*args[:i], args[i].transpose(0, -1).contiguous().transpose(0, -1), *args[i + 1:])
            served.clear()
        A, B = bits(torch.Generator(device="cuda").manual_seed(1), 4, 4), bits(torch.Generator(device="cuda").manual_seed(2), 4, 4)
        for K in (0, -1, 129, 1 << 21):
            with pytest.raises(bnn.BnnError):
                bnn.bmm(A, B, K)
        with pytest.raises(bnn.BnnError):
            bnn.bmm(A, B, 128, path=9)
        with pytest.raises(bnn.BnnError):
            bnn.bmm(A[:0], B, 128)
    finally:
        del binding._load_native_module


def test_a_tensor_without_a_pointer_raises(bnn):
    # torch refuses the data pointer of such a tensor (one that is being traced, or copied on first write when memory has run out) by a C++ exception: it has to be raised
    # before the interpreter lock is given up, where it would end the process.
    for name, args in calls(bnn):
        fn = getattr(bnn, name)
        for i in [i for i, a in enumerate(args) if torch.is_tensor(a)]:
            bad = args[i].clone()
            torch._C._set_throw_on_mutable_data_ptr(bad)
            with pytest.raises(RuntimeError, match="data pointer"):
                fn(*args[:i], bad, *args[i + 1:])
        fn(*args)
    net = bnn.Net()
    net.input_bits(128)
    net.add_fc(torch.zeros((10, 4), dtype=torch.int32, device="cuda"), None, 128)
    x = torch.zeros((3, 4), dtype=torch.int32, device="cuda")
    net.forward(x)
    torch._C._set_throw_on_mutable_data_ptr(x)
    with pytest.raises(RuntimeError, match="data pointer"):
        net.forward(x)


def test_net_forward(bnn):
    g = torch.Generator(device="cuda").manual_seed(3)
    net = bnn.Net()
    net.input_bits(128)
    net.add_fc(bits(g, 64, 4), torch.zeros(64, dtype=torch.int32, device="cuda"), 128)
    net.add_fc(bits(g, 10, 4, n=64)[:, :4].contiguous(), None, 64)
    x = bits(g, 300, 4)
    first = net.forward(x)                      # no workspace yet: the Python code makes one
    again = net.forward(x)                      # and the native module takes it
    own = net.forward(x, out=torch.empty_like(first))
    assert same(first, again) and same(first, own)
    assert same(net.forward(torch.cat([x, x])), torch.cat([first, first]))       # a larger batch: a larger workspace
    assert same(net.forward(x[:1]), first[:1])
    with pytest.raises(TypeError):
        net.forward(x.cpu())
    with pytest.raises(TypeError):
        net.forward(x.float())
    with pytest.raises(bnn.BnnError):
        net.forward(x, path=9)
