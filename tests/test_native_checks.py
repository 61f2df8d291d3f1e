"""What the binding's native argument checks accept and refuse."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave


def _plan():
    return cleave.plan_uniform(64, 32, 48, 32, 32, 1)


def test_host_tensors_and_non_tensors_are_refused():
    plan = _plan()
    A, B, P, C = torch.zeros(64, 48), torch.zeros(48, 32), torch.zeros(plan.partial_elems), torch.zeros(64, 32)
    for call in (lambda: cleave.execute(plan, A, B, P), lambda: cleave.reduce(plan, P, C),
                 lambda: cleave.reduce_residual(plan, P, C, C)):
        with pytest.raises(ValueError, match="2-D device tensor"):
            call()
    with pytest.raises(TypeError):
        cleave.execute(plan, np.zeros((64, 48)), B, P)
    with pytest.raises(TypeError):
        cleave.reduce(plan, P, None)


def test_a_build_for_another_torch_is_noticed(tmp_path, monkeypatch):
    from paper_2512_22142_amd import build
    with open(build.NATIVE, "rb") as f:
        mine = f.read()
    other = tmp_path / "_native.so"
    other.write_bytes(mine.replace(torch.__version__.encode(), b"0" * len(torch.__version__)))
    assert build.native_fits(build.NATIVE) and not build.native_fits(str(other))
    cleave.binding._require_native_fit(build.NATIVE)
    with pytest.raises(ImportError, match="build"):
        cleave.binding._require_native_fit(str(other))
    calls = []
    monkeypatch.setattr(build, "build", lambda verbose: calls.append(verbose))
    build.ensure_built()
    assert calls == []
    monkeypatch.setattr(build, "native_fits", lambda: False)
    build.ensure_built()
    assert calls == [False]


class _Stream:
    def __init__(self, address):
        self.cuda_stream = address


class _Address:
    def __init__(self, address):
        self.address = address

    def __int__(self):
        return self.address


@pytest.mark.parametrize("stream,address", [
    (_Stream(None), None), (_Stream(4096), 4096), (_Address(8192), 8192), (_Address((1 << 63) + 64), (1 << 63) + 64),
    (np.uint64((1 << 63) + 64), (1 << 63) + 64), (0, None), ("4096", 4096)])
def test_stream_arguments(stream, address):
    assert cleave.binding._stream_ptr(stream).value == address


@pytest.mark.gpu
def test_device_tensors_that_do_not_fit_are_refused():
    plan = _plan()
    dev = dict(device="cuda")
    A, B, C = torch.zeros(64, 48, **dev), torch.zeros(48, 32, **dev), torch.zeros(64, 32, **dev)
    P = torch.zeros(plan.partial_elems, **dev)
    refused = [
        (ValueError, lambda: cleave.execute(plan, A, B, P, 1, 0)),             # shapes of the other layout
        (ValueError, lambda: cleave.execute(plan, A.t(), B, P, 1, 0)),         # column stride
        (ValueError, lambda: cleave.execute(plan, A.view(-1), B, P)),
        (ValueError, lambda: cleave.execute(plan, A, B, P[1:])),               # too short
        (ValueError, lambda: cleave.execute(plan, A, B, P.double())),
        (TypeError, lambda: cleave.execute(plan, A, B.bfloat16(), P)),
        (TypeError, lambda: cleave.execute(plan, A.half(), B.half(), P)),
        (cleave.CleaveError, lambda: cleave.execute(plan, A, B, P, task_ids=[0, 0])),
        (cleave.CleaveError, lambda: cleave.execute(plan, A, B, P, transA=0, task_ids=[plan.num_tasks])),
        (ValueError, lambda: cleave.reduce(plan, P, C.t())),
        (TypeError, lambda: cleave.reduce(plan, P, C.half())),
        (ValueError, lambda: cleave.reduce_residual(plan, P, C.bfloat16(), C)),
        (ValueError, lambda: cleave.reduce_residual(plan, P, torch.zeros(64, 64, **dev)[:, :32], C)),
    ]
    for error, call in refused:
        with pytest.raises(error):
            call()
    plan.close()
    with pytest.raises(cleave.CleaveError):
        cleave.execute(plan, A, B, P)


def test_partial_blocks_on_the_host_are_refused():
    plan = _plan()
    with pytest.raises(ValueError, match="partials must be"):
        cleave.binding._partials(plan, torch.zeros(plan.partial_elems))
    with pytest.raises(TypeError):
        cleave.binding._partials(plan, np.zeros(plan.partial_elems, dtype=np.float32))


@pytest.mark.gpu
def test_every_aggregation_refuses_partials_that_are_not_the_plans_blocks():
    """A valid output and, in turn, partials on the host, one element short, of
    another type and strided: refused before anything is enqueued, the outputs
    untouched."""
    dev = dict(device="cuda")
    plan, batched = _plan(), cleave.plan_batched(64, 32, 48, 32, 32, 1, 2)
    out = [torch.full((64, 32), 7.0, **dev) for _ in range(5)]
    R, C, w, m, v = out
    both = torch.full((128, 32), 7.0, **dev)
    hyper = (1e-3, 0.9, 0.95, 1e-8, 0.1, 1)
    calls = [(plan, lambda P: cleave.reduce(plan, P, C)),
             (plan, lambda P: cleave.reduce_residual(plan, P, R, C)),
             (plan, lambda P: cleave.reduce_adam(plan, P, w, m, v, *hyper)),
             (batched, lambda P: cleave.reduce_batched(batched, P, both, (64 * 32, 0), 1)),
             (batched, lambda P: cleave.reduce_grouped(batched, P, [C, R])),
             (batched, lambda P: cleave.reduce_adam_grouped(batched, P, [w, C], [m, R], [v, both[:64]], *hyper))]
    for which, call in calls:
        n = which.partial_elems
        good = torch.zeros(n, **dev)
        for bad in (good.cpu(), good[1:], good.double(), good.bfloat16(), torch.zeros(2 * n, **dev)[::2]):
            with pytest.raises(ValueError, match="partials must be"):
                call(bad)
    torch.cuda.synchronize()
    assert all(bool((t == 7.0).all()) for t in out + [both])
    for _, call in calls[:2] + calls[3:5]:                     # and the blocks themselves are taken, also as a matrix
        call(torch.zeros(4 * batched.partial_elems, **dev).view(2, -1))


@pytest.mark.gpu
def test_streams_flags_and_ids_in_every_accepted_form():
    plan = _plan()
    g = torch.Generator().manual_seed(3)
    A, B = torch.randint(-4, 5, (64, 48), generator=g).float(), torch.randint(-4, 5, (48, 32), generator=g).float()
    want = A @ B
    A, B = A.cuda(), torch.nn.Parameter(B.cuda())
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    every = list(range(plan.num_tasks))
    for stream in (None, side, side.cuda_stream, np.int64(side.cuda_stream)):
        for flag in (0, False, np.int32(0)):
            for ids in (None, every, np.asarray(every, dtype=np.int32)):
                P = torch.full((plan.partial_elems,), float("nan"), device="cuda")
                C = torch.full((64, 32), float("nan"), device="cuda")
                torch.cuda.synchronize()
                cleave.execute(plan, A, B, P, flag, flag, task_ids=ids, stream=stream)
                cleave.reduce(plan, P, C, stream=stream)
                torch.cuda.synchronize()
                assert torch.equal(C.cpu(), want)
    with torch.cuda.stream(side):                        # torch's current stream is the default
        C = torch.zeros(64, 32, device="cuda")
        cleave.execute(plan, A, B, P)
        cleave.reduce(plan, P, C)
        assert torch.equal(C.cpu(), want)
