"""The native marshalling of the device calls: host tensors, wrong types,
shapes and layouts are refused with TypeError or ValueError before anything
is launched, on the CPU and for tensors on the GPU, and a call runs on the
calling thread's current stream."""
import threading

import numpy as np
import pytest
import torch

from paper_2607_16673_amd import binding as B


def _args(dev, n=4, dt=torch.bfloat16):
    z = torch.zeros
    i = torch.int32
    a = dict(state=z(2, 3, 64, 32, device=dev), q=z(2, n, 3, 64, dtype=dt, device=dev),
             k=z(2, n, 3, 64, dtype=dt, device=dev), v=z(2, n, 3, 32, dtype=dt, device=dev),
             alpha=torch.ones(2, n, 3, device=dev), beta=z(2, n, 3, device=dev),
             parent_idx=torch.arange(-1, n - 1, dtype=i, device=dev).repeat(2, 1),
             out=z(2, n, 3, 32, device=dev))
    a["factors"] = B.Factors(z(2, n, 3, 64, dtype=dt, device=dev), z(2, n, 3, 32, device=dev),
                             z(2, n, 3, device=dev), z(2, n, dtype=i, device=dev))
    return a


def _calls(dev):
    a = _args(dev)
    f, par = a["factors"], a["parent_idx"]
    path, ln = par.clone(), torch.zeros(2, dtype=torch.int32, device=dev)
    x = torch.zeros(2, 4, 16, device=dev)
    cs, w = torch.zeros(2, 3, 16, device=dev), torch.zeros(16, 4, device=dev)
    return {
        "verify": (lambda **o: B.sla_verify(**{**a, **o}), a),
        "commit": (lambda **o: B.sla_commit(**{**dict(state=a["state"], factors=f, path=path, length=ln), **o}),
                   dict(state=a["state"], path=path, length=ln)),
        "conv_verify": (lambda **o: B.sla_conv_verify(**{**dict(conv_state=cs, x=x, weight=w, parent_idx=par,
                                                                y=x.clone()), **o}),
                        dict(conv_state=cs, x=x, weight=w, parent_idx=par)),
        "conv_commit": (lambda **o: B.sla_conv_commit(**{**dict(conv_state=cs, x=x, parent_idx=par, path=path,
                                                                length=ln), **o}),
                        dict(conv_state=cs, x=x, parent_idx=par, path=path, length=ln)),
        "prune": (lambda **o: B.sla_prune(**{**dict(parent=par, logp=torch.zeros(2, 4, device=dev), tau=1.0), **o}),
                  dict(parent=par)),
    }


@pytest.mark.parametrize("name", ["verify", "commit", "conv_verify", "conv_commit", "prune"])
def test_host_tensors_and_non_tensors_are_refused(name):
    call, tensors = _calls("cpu")[name]
    with pytest.raises(ValueError, match="must live on the GPU"):
        call()
    for key in tensors:
        if key != "factors":
            with pytest.raises((TypeError, ValueError)):
                call(**{key: [1, 2]})


@pytest.mark.gpu
@pytest.mark.parametrize("part", range(6), ids=["k", "u", "alpha", "parent", "path", "len"])
def test_incomplete_pending_is_refused(part):
    calls = _calls("cuda")
    call, a = calls["verify"]
    f, path, ln = a["factors"], a["parent_idx"].clone(), torch.zeros(2, dtype=torch.int32, device="cuda")
    prev = [f.k.clone(), f.u.clone(), f.alpha.clone(), f.parent.clone(), path, ln]
    before = [x.clone() for x in (a["state"], a["out"], f.u)]
    prev[part] = None  # a missing part of a pending round is an error, not a call without one
    with pytest.raises((TypeError, AttributeError)):
        call(pending=(B.Factors(*prev[:4]), prev[4], prev[5]))
    if part in (0, 3, 4, 5):  # the convolution's pending rows hold x, parent, path and len
        call, a2 = calls["conv_verify"]
        conv = {0: a2["x"].clone(), 3: path.clone(), 4: path, 5: ln}
        conv[part] = None
        with pytest.raises((TypeError, AttributeError)):
            call(pending=tuple(conv.values()))
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(before, (a["state"], a["out"], f.u)))


@pytest.mark.gpu
def test_factors_as_a_c_structure():
    f = B.Factors.empty(2, 4, 3, 64, 32, torch.bfloat16)
    c = f.c(torch.bfloat16, 2, 4, 3, 64, 32)
    assert (c.k, c.u, c.alpha, c.parent) == tuple(t.data_ptr() for t in (f.k, f.u, f.alpha, f.parent))
    with pytest.raises(ValueError, match="factors.k"):
        f.c(torch.bfloat16, 2, 5, 3, 64, 32)


def test_factors_as_a_c_structure_takes_gpu_tensors_only():
    f = B.Factors.empty(2, 4, 3, 64, 32, torch.bfloat16, device="cpu")
    with pytest.raises(ValueError, match="factors.k must live on the GPU"):
        f.c(torch.bfloat16, 2, 4, 3, 64, 32)


def test_kernel_size_takes_any_whole_number():
    """Whole numbers of any type pass on to the tensor checks, others are refused."""
    call, a = _calls("cpu")["conv_commit"]
    for k in (4, 4.0, np.int64(4), np.float32(4.0)):
        with pytest.raises(ValueError, match="must live on the GPU"):
            call(kernel_size=k)
    with pytest.raises(ValueError, match="whole number"):
        call(kernel_size=4.5)


@pytest.mark.gpu
def test_kernel_size_as_a_float_commits():
    call, a = _calls("cuda")["conv_commit"]
    a["x"].normal_()
    path = (a["parent_idx"] + 1).contiguous()  # the chain's own nodes, root first
    got = []
    for k in (None, 4, 4.0):
        a["conv_state"].fill_(1.0)
        call(kernel_size=k, path=path, length=torch.full((2,), 2, dtype=torch.int32, device="cuda"))
        got.append(a["conv_state"].clone())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    assert torch.equal(got[0][:, 1:], a["x"][:, :2])


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["verify", "commit", "conv_verify", "conv_commit", "prune"])
def test_wrong_shapes_types_and_layouts_are_refused(name):
    call, tensors = _calls("cuda")[name]
    call()
    for key, t in tensors.items():
        if key == "factors":
            continue
        bad = [t.double() if t.is_floating_point() else t.long(),           # another type
               t.cpu(),                                                       # host memory
               t[:1],                                                         # another shape
               t.repeat_interleave(2, -1)[..., ::2]]                          # strided
        for x in bad:
            with pytest.raises((TypeError, ValueError)):
                call(**{key: x})
    if name == "verify":
        f = tensors["factors"]
        for part in ("k", "u", "alpha", "parent"):
            parts = dict(k=f.k, u=f.u, alpha=f.alpha, parent=f.parent)
            parts[part] = parts[part][:1]
            with pytest.raises(ValueError, match="factors." + part):
                call(factors=B.Factors(**parts))
        with pytest.raises(KeyError):
            call(route="fastest")
        with pytest.raises(TypeError):
            call(q=tensors["q"].half(), k=tensors["k"].half(), v=tensors["v"].half())
        assert B.SLA_ERR_NULL == pytest.raises(B.SlaError, call, alpha=None).value.code
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_calls_run_on_the_calling_threads_stream():
    a = _args("cuda")
    a["v"].fill_(1.0)
    a["beta"].fill_(1.0)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    big = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()

    def work():
        with torch.cuda.stream(side):
            x = big
            for _ in range(30):  # some 30 ms ahead of the values: a call on another stream would read the old ones
                x = big @ x
            a["v"].add_(1.0)
            B.sla_verify(**a, topology="chain")

    t = threading.Thread(target=work)
    t.start()
    t.join()
    side.synchronize()
    assert torch.equal(a["factors"].u, torch.full_like(a["factors"].u, 2.0))  # u = beta v with a zero state
