"""The binding's calls in native code: the same results as through the Python checks, and whatever a call does not want left to those (wrong types, sizes and
places raise what they raise there, and nothing is launched first)."""
import os
import struct
import subprocess
import sys

import pytest
import torch

import paper_2510_00236_amd as pex

DEV = "cuda:0"
BOTH = ("identity", "square")


@pytest.fixture
def host():
    pex._bind_torch()
    if pex._host is None:
        pytest.skip("the native calls are not built")
    return pex._host


def test_calls_that_are_not_taken(host):
    """Without a GPU nothing is: every function says so and raises nothing, whatever it is given."""
    X, S, ws = torch.zeros(2, 3, 8), torch.zeros(8, 8), torch.zeros(64, dtype=torch.uint8)
    prm = pex.AdamParams()
    calls = [(host.stat, (X, X, 1, S, ws)), (host.stat_multi, (X, X, 3, {"identity": S, "square": S}, ws)), (host.token_sq, (X, X, S, ws)),
             (host.example_norms, (X, X, S, ws)), (host.weighted_sum, (X, X, S, S, ws)), (host.clip_weights, (S, 1.0, S)),
             (host.embed_stat, (X, X, 8, 3, {}, ws)), (host.adam_update, (S, S, S, S, S, 1, prm)), (host.signsgd_update, (S, S, S, 0.1, 0.9, 0.0, 2, False, 1)),
             (host.adam_step, ([(S,) * 5], 1, prm, S, 1.0, None, None, ws)), (host.stat_pair_batch, ([(X, X, None)], ws)), (host.vec_stat_batch, ([(X, None, {})], 3, ws))]
    for fn, args in calls:
        assert fn(*args) is False and fn(*args[:-1]) is False and fn() is False, fn
        for k in range(len(args)):
            for odd in (None, "x", object(), 2**70, -1, [], X.to(torch.float16)):
                assert fn(*args[:k], odd, *args[k + 1:]) is False, (fn, k, odd)


# Tensors that say they are on a GPU, at addresses nobody reads: in every call one of them throws when asked for its address, so that none reaches the library.
THROWING = """
import sys
import torch
import paper_2510_00236_amd as pex

def tensor(*shape, dtype=torch.float32, throws=False):
    storage = torch._C._construct_storage_from_data_pointer(4096, torch.device("cuda", 0), 1 << 20)
    meta = dict(device=torch.device("cuda", 0), dtype=dtype, size=shape, stride=torch.empty(shape, device="meta").stride(), storage_offset=0)
    t = torch._C._construct_CUDA_Tensor_From_Storage_And_Metadata(meta, storage)
    if throws:
        torch._C._set_throw_on_mutable_data_ptr(t)
    return t

pex._bind_torch()
host = pex._host
host.setup(pex.AdamParams, pex.MomentParams, lambda: 0, lambda device: 0)
X, S, v, ids = tensor(2, 4, 64), tensor(64, 64), tensor(64), tensor(2, 4, dtype=torch.int64)
ws, one, N = tensor(1 << 18, dtype=torch.uint8), tensor(1, dtype=torch.float64), tensor(2)
bad = dict(X=tensor(2, 4, 64, throws=True), S=tensor(64, 64, throws=True), v=tensor(64, throws=True), ids=tensor(2, 4, dtype=torch.int64, throws=True),
           ws=tensor(1 << 18, dtype=torch.uint8, throws=True), one=tensor(1, dtype=torch.float64, throws=True), N=tensor(2, throws=True))
good, prm = dict(X=X, S=S, v=v, ids=ids, ws=ws, one=one, N=N), pex.AdamParams()
both, vec = lambda g: {"identity": S, "square": g["S"]}, lambda g: {"identity": v, "square": g["v"]}
calls = [("X S ws", lambda g: host.stat(g["X"], X, 1, g["S"], g["ws"])), ("X S ws", lambda g: host.stat_multi(g["X"], X, 3, both(g), g["ws"])),
         ("X S ws", lambda g: host.token_sq(X, g["X"], g["S"], g["ws"])), ("X N ws", lambda g: host.example_norms(X, g["X"], g["N"], g["ws"])),
         ("X N S ws", lambda g: host.weighted_sum(X, g["X"], g["N"], g["S"], g["ws"])), ("N", lambda g: host.clip_weights(N, 1.0, g["N"])),
         ("ids X S ws", lambda g: host.embed_stat(g["ids"], g["X"], 64, 3, both(g), g["ws"])), ("S", lambda g: host.adam_update(S, S, S, S, g["S"], 1, prm)),
         ("S", lambda g: host.signsgd_update(S, S, g["S"], 0.1, 0.9, 0.0, 2, False, 1)),
         ("S one ws", lambda g: host.adam_step([(S, S, S, S, g["S"])] * 2, 1, prm, g["one"], 1.0, None, None, g["ws"])),
         ("X S ws", lambda g: host.stat_pair_batch([(X, X, both(good)), (X, g["X"], both(g))], g["ws"])),
         ("X v ws", lambda g: host.vec_stat_batch([(X, None, vec(good)), (X, g["X"], vec(g))], 3, g["ws"]))]
held = [sys.getrefcount(t) for t in (X, S, v, ws)]
for which, call in calls:
    for name in which.split():
        assert call({**good, name: bad[name]}) is False, (which, name)
assert held == [sys.getrefcount(t) for t in (X, S, v, ws)]
print("all left to the Python checks")
"""


def test_addresses_that_throw(host):
    """A tensor whose address cannot be had leaves the call to the Python checks, with the interpreter's lock held."""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
    r = subprocess.run([sys.executable, "-c", THROWING], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "all left" in r.stdout, (r.returncode, r.stdout, r.stderr[-2000:])


@pytest.mark.parametrize("command", [["false"], ["no such compiler"], None])
def test_library_without_the_native_calls(command, monkeypatch, tmp_path, capfd):
    """Where they cannot be compiled the build goes on, without those of an earlier one."""
    from paper_2510_00236_amd import build

    def no_torch():
        raise ImportError("no torch")

    old = tmp_path / "_pex_host.so"
    old.write_bytes(b"of an earlier header")
    monkeypatch.setattr(build, "HOST_MODULE", str(old))
    monkeypatch.setattr(build, "host_command", no_torch if command is None else lambda: command)
    assert build.build_host() is False and not old.exists()
    assert "not built" in capfd.readouterr().err


def test_no_thread_local_storage(host):
    """The module brings none (ELF program header PT_TLS): loading it would slow down every call of torch."""
    with open(host.__file__, "rb") as f:
        head = f.read(64)
        at, size, count = struct.unpack_from("<Q", head, 32)[0], *struct.unpack_from("<HH", head, 54)
        f.seek(at)
        kinds = [struct.unpack_from("<I", f.read(size))[0] for _ in range(count)]
    assert 1 in kinds and 7 not in kinds, kinds


def test_native_calls_of_another_header_are_not_used(monkeypatch):
    class Old:
        PEX_VERSION = -1

        @staticmethod
        def setup(*args):
            raise AssertionError("used")

    monkeypatch.setattr(pex, "_pex_host", Old, raising=False)
    monkeypatch.setattr(pex, "_host", None)
    pex._bind_torch()
    assert pex._host is None


def test_names_from_an_iterator(monkeypatch):
    """`want` is read once, also where the native call leaves a call to the Python checks (no outputs given here)."""
    class Declines:
        def __getattr__(self, name):
            return lambda *args: False

    masks = []
    pex._bind_torch()
    monkeypatch.setattr(pex, "_host", Declines())
    monkeypatch.setattr(pex, "_dev", lambda *a, **k: 0)
    monkeypatch.setattr(pex, "_invoke_ws", lambda query, qargs, ws, fn, *args: masks.append(args))
    X, ids = torch.zeros(2, 3, 8), torch.zeros(2, 3, dtype=torch.int64)
    assert list(pex.pex_stat_multi(X, X, iter(BOTH))) == list(BOTH) and masks[-1][7] == 3
    assert list(pex.pex_embed_stat(ids, X, 9, (n for n in ("sign", "square")))) == ["square", "sign"] and masks[-1][8] == 6
    assert [list(d) for d in pex.pex_vec_stat_batch([(X, None, None)] * 2, iter(("identity",)))] == [["identity"]] * 2 and masks[-1][5] == 1


def _inputs(g):
    B, T, a, b, V = 5, 37, 72, 40, 90
    r = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    return dict(X=r(B, T, a).bfloat16(), G=r(B, T, b).bfloat16(), ids=torch.randint(0, V, (B, T), device=DEV, generator=g), V=V, w=r(B), theta=r(a * b))


def _all(s):
    """Every call that has a native form, on fresh outputs."""
    X, G, B, T, a, b, V = s["X"], s["G"], 5, 37, 72, 40, s["V"]
    f = lambda *shape: torch.full(shape, float("nan"), device=DEV)  # noqa: E731
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    out = {"stat": pex.pex_stat(X, G, "sign", S=f(a, b), workspace=ws), "token": pex.pex_token_sq(X, G, S=f(a, b), workspace=ws),
           "wsum": pex.pex_weighted_sum(X, G, s["w"], S=f(a, b), workspace=ws)}
    N = out["N"] = pex.pex_example_norms(X, G, N=f(B), workspace=ws)
    out["clip"] = pex.pex_clip_weights(N, 20.0, w=f(B))
    multi = pex.pex_stat_multi(X, G, BOTH, out={"identity": f(a, b), "square": f(a, b)}, workspace=ws)
    embed = pex.pex_embed_stat(s["ids"], G, V, ("square", "sign"), out={"square": f(V, b), "sign": f(V, b)}, workspace=ws)
    pair = pex.pex_stat_pair_batch([(X, G, {"identity": f(a, b), "square": f(a, b)}), (G, X, {"identity": f(b, a), "square": f(b, a)})], workspace=ws)
    vec = pex.pex_vec_stat_batch([(X, None, {"identity": f(a), "square": f(a)}), (G, G, {"identity": f(b), "square": f(b)})], BOTH, workspace=ws)
    assert list(multi) == ["identity", "square"] and list(embed) == ["square", "sign"] and all(list(d) == list(BOTH) for d in pair + vec)
    for name, d in [("multi", multi), ("embed", embed), ("pair0", pair[0]), ("pair1", pair[1]), ("vec0", vec[0]), ("vec1", vec[1])]:
        out.update({name + k: v for k, v in d.items()})
    prm = pex.AdamParams(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-8, eps_root=0.0, weight_decay=0.1, grad_scale=1.0 / B, sq_scale=1.0 / B, step=3, B=B)
    mp = pex.MomentParams(beta2=0.95, grad_scale=1.0 / B, sq_scale=1.0 / B, B=B, debias=1, step=3)
    state = [[s["theta"].clone()] + [torch.zeros(a * b, device=DEV) for _ in range(2)] for _ in range(3)]
    pex.pex_adam_update(*state[0], multi["identity"].view(-1), multi["square"].view(-1), "microadam", prm)
    pex.pex_signsgd_update(*state[1][:2], out["stat"].view(-1), 1e-3, 0.9, 1e-4, B)
    sum_sq, sums, emas = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(1, 2, dtype=torch.float64, device=DEV), torch.zeros(2, a * b, device=DEV)
    pex.pex_adam_step([(*state[2], multi["identity"].view(-1), multi["square"].view(-1), emas[0], emas[1])], "microadam", prm, sum_sq, 1e-2, moments=mp, sums=sums, workspace=ws)
    out.update({f"state{k}{j}": t for k, st in enumerate(state) for j, t in enumerate(st)}, sum_sq=sum_sq, sums=sums, emas=emas)
    return out


@pytest.mark.gpu
def test_same_results_as_through_the_python_checks(host, monkeypatch):
    s = _inputs(torch.Generator(device=DEV).manual_seed(1))
    taken = []

    class Counting:
        def __getattr__(self, name):
            def call(*args):
                r = getattr(host, name)(*args)
                taken.append((name, r is not False))
                return r
            return call

    monkeypatch.setattr(pex, "_host", Counting())
    native = _all(s)
    assert len(taken) == 12 and all(ok for _, ok in taken), taken
    monkeypatch.setattr(pex, "_host", None)
    python = _all(s)
    assert set(native) == set(python)
    for k in native:
        assert torch.equal(native[k], python[k]), k


@pytest.mark.gpu
def test_on_the_current_stream(host):
    s = _inputs(torch.Generator(device=DEV).manual_seed(2))
    ws, S = torch.empty(1 << 20, dtype=torch.uint8, device=DEV), torch.zeros(72, 40, device=DEV)
    want = pex.pex_stat(s["X"], s["G"], "square")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        pex.pex_stat(s["X"], s["G"], "square", S=S, workspace=ws)
    side.synchronize()
    assert torch.equal(S, want)


@pytest.mark.gpu
def test_what_is_refused_raises_as_before(host, monkeypatch):
    s = _inputs(torch.Generator(device=DEV).manual_seed(3))
    X, G = s["X"], s["G"]
    ws, S = torch.empty(1 << 20, dtype=torch.uint8, device=DEV), torch.zeros(72, 40, device=DEV)
    big = torch.zeros(21, 285, 320, device=DEV).bfloat16(), torch.zeros(21, 285, 960, device=DEV).bfloat16()
    calls = [lambda: pex.pex_stat(X, G, "sign", S=S.double(), workspace=ws), lambda: pex.pex_stat(X, G, "sign", S=S.t(), workspace=ws),
             lambda: pex.pex_stat(X, G, "sign", S=S[:, :-1], workspace=ws), lambda: pex.pex_stat(X, G, 17, S=S, workspace=ws),
             lambda: pex.pex_stat(X, G.float(), "sign", S=S, workspace=ws), lambda: pex.pex_stat(X, G[:, :-1], "sign", S=S, workspace=ws),
             lambda: pex.pex_stat(X.cpu(), G.cpu(), "sign", S=S.cpu(), workspace=ws.cpu()), lambda: pex.pex_stat(X, G, "sign", S=S, workspace=ws.float()),
             lambda: pex.pex_stat_multi(*big, BOTH, out={k: torch.zeros(320, 960, device=DEV) for k in BOTH}, workspace=ws[:4096]),
             lambda: pex.pex_stat_multi(X, G, 9, out={}, workspace=ws), lambda: pex.pex_clip_weights(s["w"], 1.0, w=torch.zeros(4, device=DEV)),
             lambda: pex.pex_signsgd_update(s["theta"], s["theta"][:-1], s["theta"], 0.1, 0.9, 0.0, 5),
             lambda: torch.func.vmap(lambda x: pex.pex_stat(x, G, "sign", S=S, workspace=ws))(X.unsqueeze(0).repeat(2, 1, 1, 1))]
    for k, call in enumerate(calls):
        seen = []
        for module in (host, None):
            monkeypatch.setattr(pex, "_host", module)
            try:
                call()
                seen.append("taken")
            except Exception as e:      # noqa: BLE001
                seen.append((type(e), str(e)))
        assert seen[0] == seen[1] and seen[0] != "taken", (k, seen)
