"""The native argument marshalling of the binding (csrc/marshal.cpp): it calls the library only when every argument is in
order, and hands everything else to the Python code, which describes the error."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2511_02017_amd import binding

f32, i32, u8 = torch.float32, torch.int32, torch.uint8


def test_arguments_that_are_not_in_order_go_to_the_python_code():
    """No GPU needed: nothing here reaches the library (the context's address is no context)."""
    binding.load_library()
    fast = binding._fast
    d, t = torch.zeros(2, 3, 8), torch.zeros(2, 4, 8)                       # not on a GPU
    out = {}
    assert fast.draft_stats(1, 1, d, None, None, None, None, out, None) is None
    assert fast.draft_stats(0, 1, d, None, None, None, None, out, None) is None     # closed context
    assert fast.draft_stats(None, 1, d, None, None, None, None, out, None) is None
    assert fast.verify(1, t, d, None, None, None, None, None, None, None, out, 0) is None
    assert fast.bandit_select(1, 2, 1, 3, None, None, None, 0) is None              # arm_out missing
    assert fast.bandit_select(1, 2, 1, 3, torch.zeros(2, 3, 48), torch.zeros(2, dtype=i32), None, 0) is None
    assert fast.shard_stats(1, d, 0, None, 0, None, None, 0) is None
    assert fast.shard_final_sums(1, t, d, None, None, 0) is None
    assert fast.verify(1) is None and fast.draft_stats() is None                    # wrong number of arguments
    assert fast.draft_stats(1, 1, "x", None, None, None, None, out, None) is None
    assert fast.draft_stats(1 << 80, 1, d, None, None, None, None, out, None) is None
    with pytest.raises(ImportError):
        fast.load("/nonexistent/libtapout.so")
    assert fast.verify(1) is None                                                   # the library loaded before stays


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_an_exception_out_of_the_library_becomes_a_python_one(tmp_path):
    """The library is called without the interpreter lock; an exception that leaves it is raised with the lock held, and the call
    is not made a second time.  A stand-in library throws (a process of its own: a fault here would end the interpreter)."""
    names = ("bandit_select", "draft_stats", "verify", "bandit_update", "bandit_update_select", "shard_stats", "draft_stats_sharded",
             "verify_accept_sharded", "shard_final_sums", "shard_final_token")
    src = tmp_path / "stand_in.cpp"
    src.write_text("#include <cstdio>\n#include <stdexcept>\n" + "".join(
        f'extern "C" int tapout_{n}() {{ std::puts("called {n}"); std::fflush(stdout); throw std::runtime_error("out of {n}"); }}\n' for n in names))
    lib = tmp_path / "stand_in.so"
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    code = f"""
import sys, threading, torch
sys.path.insert(0, {ROOT!r})
from paper_2511_02017_amd import _marshal
_marshal.load({str(lib)!r})
for _ in range(3):
    try:
        print(_marshal.bandit_update(1, 1, 1, None, None, None, None, None, 0))
    except RuntimeError as e:
        print("raised", e)
t = threading.Thread(target=print, args=("alive",)); t.start(); t.join()
"""
    r = subprocess.run([sys.executable, "-u", "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split("\n")[:-1] == ["called bandit_update", "raised out of bandit_update"] * 3 + ["alive"]


@pytest.fixture
def python_only(monkeypatch):
    """The binding as it loads where _marshal.so is missing or does not fit this Python or torch."""
    import paper_2511_02017_amd as pkg
    binding.load_library()
    native = binding._fast
    monkeypatch.setitem(sys.modules, "paper_2511_02017_amd._marshal", None)         # an import of it fails
    monkeypatch.delattr(pkg, "_marshal", raising=False)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_fast", None)
    with pytest.warns(RuntimeWarning, match="_marshal"):
        binding.load_library()
    return native


def test_the_library_loads_without_the_native_part(python_only):
    assert binding._fast is not python_only
    assert binding._fast.verify(1, 2, 3) is None and binding._fast.bandit_select() is None      # every call goes the Python way
    cfg = binding.default_config(4, 3, 100)
    assert (cfg.max_batch, cfg.max_k, cfg.vocab) == (4, 3, 100)


@pytest.mark.gpu
def test_the_native_part_changes_no_result(python_only, monkeypatch):
    """The calls of a round and of a round over vocabulary shards, on the current stream and on one handed in: the same bits."""
    def calls(stream):
        g = torch.Generator(device="cuda:0").manual_seed(1)
        B, K, V = 5, 4, 9001
        d, t = torch.randn(B, K, V, generator=g, device="cuda:0") * 3, torch.randn(B, K + 1, V, generator=g, device="cuda:0") * 3
        tok, ua = d.argmax(-1).to(i32), torch.rand(B, K, generator=g, device="cuda:0")
        us, n = torch.rand(B, generator=g, device="cuda:0"), torch.full((B,), K, dtype=i32, device="cuda:0")
        torch.cuda.synchronize()
        tp = binding.Tapout(B, K, V, draft_sampling=True)
        st = dict(stream=stream)
        arm = tp.bandit_select(B, **st)
        ds = tp.draft_stats(d, tok, n, arm, **st)
        smp = tp.draft_stats(d, k_len=n, u_draft=ua, **st)
        vf = tp.verify(t, d, ds["lse"], ds["logq_tok"], tok, n, ua, us, **st)
        tp.bandit_update(arm, vf["accept_len"], n, n, **st)
        nxt = tp.bandit_update_select(arm, vf["accept_len"], n, n, **st)
        r0, r1 = tp.shard_stats(d, 0, length=n, tok=tok, **st), tp.shard_stats(t, 0, length=n, rows_mode=1, tok=tok, **st)
        dss = tp.draft_stats_sharded(r0[None], B, K, V, draft_tok=tok, k_len=n, arm=arm, **st)
        acc = tp.verify_accept_sharded(r1[None], B, K, V, dss["logq_tok"], tok, n, ua, draft_lse=dss["lse"], **st)
        sums = tp.shard_final_sums(t, d, acc["final_jobs"], **st)
        fin = tp.shard_final_token(t, d, 0, 1, 0, acc["final_jobs"], sums[None], us, **st)
        torch.cuda.synchronize()
        return [arm, nxt, r0, r1, sums, *fin, *ds.values(), *smp.values(), *vf.values(), *dss.values(), *acc.values()]

    for stream in (None, torch.cuda.Stream()):
        without = calls(stream)
        with monkeypatch.context() as m:
            m.setattr(binding, "_fast", python_only)                # the native part
            native = calls(stream)
        for a, b in zip(without, native):
            assert torch.equal(torch.nan_to_num(a.double(), nan=-7.0), torch.nan_to_num(b.double(), nan=-7.0))


@pytest.mark.gpu
def test_errors_are_those_of_the_python_code():
    B, K, V = 2, 3, 100
    tp = binding.Tapout(B, K, V)
    x = torch.randn(B, K, V, device="cuda:0")
    tok = torch.zeros(B, K, dtype=i32, device="cuda:0")
    with pytest.raises(ValueError, match="draft_tok: expected shape"):
        tp.draft_stats(x, tok[:, :2].contiguous())
    with pytest.raises(ValueError, match="draft_tok: expected torch.int32"):
        tp.draft_stats(x, tok.long())
    with pytest.raises(ValueError, match="must live on the GPU"):
        tp.draft_stats(x, tok.cpu())
    with pytest.raises(ValueError, match="must be contiguous"):
        tp.draft_stats(x, torch.zeros(K, B, dtype=i32, device="cuda:0").t())
    with pytest.raises(ValueError, match="not supported"):
        tp.draft_stats(x.half())
    with pytest.raises(ValueError, match="vocabulary axis"):
        tp.draft_stats(torch.randn(B, V, K, device="cuda:0").transpose(1, 2))
    with pytest.raises(ValueError, match="arm: expected shape"):
        tp.draft_stats(x, arm=torch.zeros(B + 1, dtype=i32, device="cuda:0"))
    with pytest.raises(binding.TapoutError, match="max_k"):
        tp.draft_stats(torch.randn(B, K + 1, V, device="cuda:0"))
    with pytest.raises(binding.TapoutError, match="exclude each other|draft_sampling"):
        tp.draft_stats(x, tok, u_draft=torch.rand(B, K, device="cuda:0"))
    out = tp.alloc_draft_outputs(B, K)
    out["lse"] = out["lse"][:, :2]
    with pytest.raises(ValueError, match="lse: expected shape"):
        tp.draft_stats(x, tok, out=out)
    tp.close()
    with pytest.raises(binding.TapoutError):
        tp.draft_stats(x, tok)


@pytest.mark.gpu
def test_streams_views_and_parameters():
    """The current stream, a stream handed in, strided views and tensors that take gradients: the same results."""
    B, K, V = 3, 4, 5000
    tp = binding.Tapout(B, K, V)
    full = torch.randn(B, K + 2, V + 40, device="cuda:0")
    tok = torch.randint(0, V, (B, K), dtype=i32, device="cuda:0")
    view = full[:, 1:K + 1, 13:V + 13]
    torch.cuda.synchronize()
    want = tp.draft_stats(view.contiguous(), tok)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = tp.draft_stats(view, tok)
    s.synchronize()
    b = tp.draft_stats(view, tok, stream=s)
    s.synchronize()
    c = tp.draft_stats(torch.nn.Parameter(view), tok)
    torch.cuda.synchronize()
    for got in (a, b, c):
        assert torch.equal(got["top1_id"], want["top1_id"])
        assert torch.allclose(got["lse"], want["lse"], rtol=0, atol=1e-5) and torch.allclose(got["logq_tok"], want["logq_tok"], rtol=0, atol=1e-5)
