"""The native marshalling against the ctypes path it stands in for: for plain calls the C entry point must
receive the same arguments from both, and what the ctypes path refuses the native one must leave to it."""
import ctypes
import os
import subprocess
import sys

import pytest
import torch

import paper_2503_20552_amd as adr
from paper_2503_20552_amd import binding

BF, F32, I32 = torch.bfloat16, torch.float32, torch.int32


class Recorder:
    """Stands in for the library: callbacks with the real entry points' signatures that note what they get."""
    def __init__(self):
        real = adr.load_library()
        self.calls, self.address_of, self._keep = [], {}, []
        for name in binding._FAST:
            types = getattr(real, name).argtypes
            fn = ctypes.CFUNCTYPE(ctypes.c_int, *types)(lambda *a, name=name: self.note(name, a))
            self._keep.append(fn)
            setattr(self, name, fn)
            self.address_of[name] = ctypes.cast(fn, ctypes.c_void_p).value

    def note(self, name, args):
        flat = []
        for a in args:
            if isinstance(a, ctypes._Pointer):
                a = tuple(getattr(a.contents, f) for f, _ in binding._CCache._fields_)
            flat.append(a)
        self.calls.append((name, flat))
        return 0


class Leaves:
    """A marshalling module that leaves every call to the ctypes path."""
    def __getattr__(self, name):
        return lambda *a: None


class Counts:
    def __init__(self, inner):
        self.inner, self.took = inner, 0

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.inner, name)(*a)
            self.took += r is not None
            return r
        return call


@pytest.fixture
def both(monkeypatch):
    adr.load_library()
    native = binding._marshal

    def run(fn, *a, **kw):
        seen = []
        for module in (Counts(native), Leaves()):
            rec = Recorder()
            monkeypatch.setattr(binding, "_lib", rec)
            monkeypatch.setattr(binding, "_marshal", module)
            try:
                fn(*a, **kw)
                seen.append(("returned", rec.calls))
            except Exception as e:      # noqa: BLE001 -- whatever it is, both paths have to raise it
                seen.append((type(e), str(e), rec.calls))
            if isinstance(module, Counts):
                took = module.took
        assert seen[0] == seen[1], seen
        return seen[0], took
    return run


class Stream:
    cuda_stream = 1 << 40


def buffers(B=3, Hq=8, Hkv=2, d=64, fp8=False, out=BF):
    k = torch.zeros(7, 16, Hkv, d, dtype=torch.uint8 if fp8 else BF)
    scale = torch.zeros(7, Hkv) if fp8 else None
    cache = adr.KVCache(k, k.clone(), scale, scale.clone() if fp8 else None)
    grouped = torch.zeros(B, (Hq + 2 * Hkv) * d, dtype=BF)
    return dict(out=torch.zeros(B, Hq, d, dtype=out), q=grouped[:, :Hq * d].view(B, Hq, d),
                k_new=grouped[:, Hq * d:(Hq + Hkv) * d].view(B, Hkv, d), v_new=grouped[:, (Hq + Hkv) * d:].view(B, Hkv, d),
                cache=cache, block_table=torch.zeros(B, 5, dtype=I32), seq_lens=torch.zeros(B, dtype=I32),
                workspace=torch.zeros(99, dtype=F32), lse=torch.zeros(B, Hq), grouped=grouped)


def step(b, **kw):
    a = {k: v for k, v in {**b, **kw}.items() if k != "grouped"}
    return adr.adr_decode_step, dict(scale=0.25, max_seq_len=80, partition_tokens=16, flags=32, stream=Stream()) | a


def attend(b, **kw):
    fn, a = step(b, **kw)
    a.pop("k_new"), a.pop("v_new")
    return adr.adr_decode_attention, a


@pytest.mark.parametrize("call", [step, attend])
@pytest.mark.parametrize("B", [0, 1, 3])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("out", [BF, F32])
def test_plain_attention_calls(both, call, B, fp8, out):
    fn, a = call(buffers(B, fp8=fp8, out=out))
    for change in ({}, {"lse": None, "workspace": None}, {"stream": 0}, {"stream": 77}, {"flags": 0xFFF0000}):
        seen, took = both(fn, **{**a, **change})
        assert took == 1 and seen[0] == "returned" and len(seen[1]) == 1
    a.pop("flags"), a.pop("partition_tokens")
    assert both(fn, **a)[1] == 1


@pytest.mark.parametrize("call", [step, attend])
def test_unusual_and_refused_attention_calls(both, call):
    b = buffers()
    fn, plain = call(b)
    t = b["q"]
    changes = [dict(scale=1), dict(max_seq_len=80.0), dict(max_seq_len=2 ** 40), dict(flags=True), dict(stream="x"), dict(stream=None),
               dict(out=t.float().transpose(0, 1)), dict(out=b["out"].half()), dict(out=b["out"][:2]), dict(q=b["out"].float()),
               dict(q=t.transpose(1, 2)), dict(q=t[0]), dict(seq_lens=b["seq_lens"].long()), dict(seq_lens=b["seq_lens"][:2]),
               dict(block_table=b["block_table"][:2]), dict(block_table=b["block_table"].t()), dict(block_table=b["seq_lens"]),
               dict(block_table=torch.zeros(3, 10, dtype=I32)[:, ::2]), dict(lse=torch.zeros(3, 4)), dict(lse=torch.zeros(8, 3).t()),
               dict(lse=b["out"]), dict(cache=adr.KVCache(b["cache"].k, b["cache"].v[:3])), dict(cache=object()), dict(workspace=3),
               dict(cache=adr.KVCache(b["cache"].k.float(), b["cache"].v.float())), dict(out=torch.nn.Parameter(b["out"])),
               dict(cache=adr.KVCache(b["cache"].k, b["cache"].v, torch.zeros(7, 3), None)), dict(q=None), dict(out=[1]),
               dict(cache=adr.KVCache(b["cache"].k.transpose(1, 2), b["cache"].v.transpose(1, 2))), dict(q=t.to("meta"))]
    if call is step:
        changes += [dict(k_new=b["k_new"].contiguous()), dict(k_new=b["k_new"][:2]), dict(v_new=b["v_new"].float())]
    for change in changes:
        both(fn, **{**plain, **change})


def test_append_merge_and_copies(both):
    for B in (0, 1, 3):
        b = buffers(B, fp8=B == 3)
        pos, s = b["seq_lens"], Stream()
        assert both(adr.adr_kv_append, b["cache"], b["k_new"], b["v_new"], b["block_table"], pos, stream=s)[1] == 1
        assert both(adr.adr_kv_append, b["cache"], b["k_new"], b["v_new"], b["block_table"], pos.long(), stream=s)[1] == 0
        both(adr.adr_kv_append, b["cache"], b["k_new"], b["q"][:, :2], b["block_table"], pos, stream=s)
        po, pl, off = torch.zeros(5, 8, 64), torch.zeros(5, 8), torch.zeros(B + 1, dtype=I32)
        for lse in (None, torch.zeros(B, 8)):
            assert both(adr.adr_lse_merge, b["out"], po, pl, off, lse, stream=s)[1] == 1
        for bad in ((b["out"].half(), po, pl, off), (b["out"], po.double(), pl, off), (b["out"], po, pl[:4], off),
                    (b["out"], po, pl, off.long()), (b["out"], po[:, :4], pl, off), (b["out"], po, pl, torch.zeros(B + 2, dtype=I32))):
            assert both(adr.adr_lse_merge, *bad, stream=s)[1] == 0
        assert both(adr.adr_pack_qkv, b["grouped"], b["q"], b["k_new"], b["v_new"], stream=s)[1] == 1
        assert both(adr.adr_pack_qkv, b["grouped"][:, :8], b["q"], b["k_new"], b["v_new"], stream=s)[1] == 0
        assert both(adr.adr_pack_qkv, b["grouped"], b["q"], b["k_new"], b["q"], stream=s)[1] == 0
        wide, idx = torch.zeros(9, 128, dtype=BF)[:, :64], torch.zeros(B, dtype=I32)
        assert both(adr.adr_scatter_rows, wide, torch.zeros(B, 64, dtype=BF), idx, stream=s)[1] == 1
        assert both(adr.adr_scatter_rows, wide, torch.zeros(B, 32, dtype=BF), idx, stream=s)[1] == 0
        assert both(adr.adr_scatter_rows, wide, torch.zeros(B, 64), idx, stream=s)[1] == 0
        assert both(adr.adr_scatter_rows, wide.t(), torch.zeros(B, 9, dtype=BF), idx, stream=s)[1] == 0


def test_the_status_becomes_the_exception():
    b = buffers()
    fn, a = step(b, partition_tokens=24)          # not a multiple of the page size: refused before any launch
    with pytest.raises(adr.AdrError) as e:
        fn(**a)
    assert e.value.status == 2 and "adr_decode_step" in str(e.value)


WITHOUT = """
import sys, types, warnings
class Hide:
    def find_spec(self, name, path=None, target=None):
        if name == "paper_2503_20552_amd._marshal":
            raise ImportError("hidden")
{how}
import torch
import paper_2503_20552_amd as adr
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    assert adr.adr_graph_capacity(5, 16, 64) == 16 and adr.adr_version() > 0
assert len(seen) == 1 and "_marshal" in str(seen[0].message), seen
k = torch.zeros(7, 16, 2, 64, dtype=torch.bfloat16)
q = torch.zeros(3, 8, 64, dtype=torch.bfloat16)
try:
    adr.adr_decode_attention(q.clone(), q, adr.KVCache(k, k.clone()), torch.zeros(3, 5, dtype=torch.int32),
                             torch.zeros(3, dtype=torch.int32), 0.25, 80, 24, stream=1 << 40)
except adr.AdrError as e:
    assert e.status == 2       # not a multiple of the page size: the C entry point's own refusal
else:
    raise AssertionError
"""


@pytest.mark.parametrize("how", ["sys.meta_path.insert(0, Hide())",
                                 "sys.modules['paper_2503_20552_amd._marshal'] = types.ModuleType('_marshal')"])
def test_the_library_works_without_the_native_marshalling(how):
    """Missing, or built for another Python or torch: the same calls go through ctypes, after one warning."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", WITHOUT.format(how=how)], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
