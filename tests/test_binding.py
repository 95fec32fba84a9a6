"""The binding refuses tensors of the wrong type or shape before anything
reaches the library (whose kernels trust the sizes they are given).  These
run on the CPU: the checks come before any device pointer is taken."""
import pytest
import torch

import paper_2502_17139_amd as fc


def _tree_inputs(n_rows=3, S=2, k=8, m=4, L=5):
    return (torch.zeros((n_rows, S), dtype=torch.int32), torch.zeros((n_rows, k), dtype=torch.uint8),
            torch.zeros((n_rows, k, m), dtype=torch.uint16), torch.zeros((n_rows, L), dtype=torch.uint16))


def test_build_tree_refuses_mismatched_slots():
    taken, lens, toks, ctx = _tree_inputs()
    with pytest.raises(ValueError, match="cont_len"):
        fc.fc_build_tree(taken, lens[:, :7], toks, ctx, c=4)
    with pytest.raises(ValueError, match="cont_tok"):
        fc.fc_build_tree(taken, lens, toks.to(torch.int32), ctx, c=4)
    with pytest.raises(ValueError, match="ctx"):
        fc.fc_build_tree(taken, lens, toks, ctx[:2], c=4)
    with pytest.raises(ValueError, match="rows"):
        fc.fc_build_tree(taken, lens, toks, ctx[:2], c=4, rows=torch.zeros(2, dtype=torch.int64))


def test_build_tree_refuses_small_outputs():
    taken, lens, toks, ctx = _tree_inputs()
    out = fc.tree_outputs(3, 4, "cpu")
    out["mask"] = out["mask"][:, :4]
    with pytest.raises(ValueError, match="mask"):
        fc.fc_build_tree(taken, lens, toks, ctx, c=4, out=out)


def test_verify_refuses_mismatched_target():
    tree = fc.tree_outputs(2, 4, "cpu")
    with pytest.raises(ValueError, match="target"):
        fc.fc_verify_accept(tree, torch.zeros((2, 4), dtype=torch.int32), m=3)
    with pytest.raises(ValueError, match="target"):
        fc.fc_verify_accept(tree, torch.zeros((2, 5), dtype=torch.int64), m=3)


class _NoStore:
    """Stands in for a Store: only its (empty) view is read before the checks."""

    def view(self):
        return fc.FcStore()


def test_retrieve_refuses_short_outputs():
    ctx = torch.zeros((4, 16), dtype=torch.uint16)
    out = fc.retrieve_outputs(4, 1, 10, 3, "cpu")
    out["cont_tok"] = out["cont_tok"][:, :9]
    with pytest.raises(ValueError, match="cont_tok"):
        fc.fc_retrieve([_NoStore()], ctx, k=10, m=3, out=out)
    out = fc.retrieve_outputs(3, 1, 10, 3, "cpu")
    with pytest.raises(ValueError, match="one row per query"):
        fc.fc_retrieve([_NoStore()], ctx, k=10, m=3, out=out)


def test_tree_attention_refuses_mismatched_cache():
    B, R, H, Hkv, D, P = 2, 5, 4, 2, 128, 16
    bf = torch.bfloat16
    q = torch.zeros((B, R, H, D), dtype=bf)
    kt = torch.zeros((B, R, Hkv, D), dtype=bf)
    kc = torch.zeros((B, P, Hkv, D), dtype=bf)
    tree = fc.tree_outputs(B, R - 1, "cpu")
    plen = torch.zeros(B, dtype=torch.int32)
    with pytest.raises(ValueError, match="v_cache"):
        fc.fc_tree_attention(q, kt, kt, kc, kc[:, :8], plen, tree)
    with pytest.raises(ValueError, match="prefix_len"):
        fc.fc_tree_attention(q, kt, kt, kc, kc, plen.to(torch.int64), tree)


def test_cache_write_refuses_mismatched_segments():
    texts = torch.zeros((2, 32), dtype=torch.uint16)
    tl = torch.zeros(2, dtype=torch.int32)
    i32 = lambda n: torch.zeros(n, dtype=torch.int32)  # noqa: E731
    with pytest.raises(ValueError, match="src_off"):
        fc.fc_cache_write(texts, tl, i32(3), i32(3), i32(3), i32(3), i32(3), torch.zeros(5, dtype=torch.uint16))
    with pytest.raises(ValueError, match="dst_off"):
        fc.fc_cache_write(texts, tl, i32(3), i32(2), i32(3), torch.zeros(3, dtype=torch.int64), i32(3),
                          torch.zeros(5, dtype=torch.uint16))


class _Stream:
    cuda_stream = 7


class _Scratch:
    """Stands in for the GPU: records, for each buffer the binding makes, the
    stream whose pool it came from, and what the library was handed."""

    def __init__(self, monkeypatch, need):
        self.stream, self.made, self.calls = None, [], []
        rec = self

        class Lib:
            def __getattr__(self, name):
                if name.endswith("_bytes"):
                    return lambda *a: need
                return lambda *a: rec.calls.append((name, a)) or 0

        class on_stream:
            def __init__(self, s):
                self.s = s

            def __enter__(self):
                self.before, rec.stream = rec.stream, self.s.cuda_stream

            def __exit__(self, *_):
                rec.stream = self.before

        def empty(shape, dtype, device):
            t = torch.empty(shape, dtype=dtype)
            rec.made.append((rec.stream, t.numel(), t.data_ptr()))
            return t

        monkeypatch.setattr(fc, "lib", lambda: Lib())
        monkeypatch.setattr(fc, "_empty", empty)
        monkeypatch.setattr(fc, "_ptr", lambda t: None if t is None else t.data_ptr())
        monkeypatch.setattr(fc, "_ptrs", lambda ts: [t.data_ptr() for t in ts])
        monkeypatch.setattr(fc, "_stream", lambda s: 0 if s is None else s.cuda_stream)
        monkeypatch.setattr(torch.cuda, "Stream", _Stream)
        monkeypatch.setattr(torch.cuda, "stream", on_stream)


def _attention_args(B=1, R=5, H=4, Hkv=2, D=128, P=300):
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16)  # noqa: E731
    return dict(q=z(B, R, H, D), k_tree=z(B, R, Hkv, D), v_tree=z(B, R, Hkv, D), k_cache=z(B, P, Hkv, D),
                v_cache=z(B, P, Hkv, D), prefix_len=torch.zeros(B, dtype=torch.int32),
                tree=fc.tree_outputs(B, R - 1, "cpu"), out=torch.zeros((B, R, H, D)))


@pytest.mark.parametrize("stream", [None, _Stream()])
def test_tree_attention_scratch_comes_from_the_stream_it_is_used_on(monkeypatch, stream):
    args = _attention_args()
    gpu = _Scratch(monkeypatch, 4096)
    fc.fc_tree_attention(**args, stream=stream)
    where = None if stream is None else stream.cuda_stream
    assert [(s, n) for s, n, _ in gpu.made] == [(where, 4096)]
    (name, a), = gpu.calls
    assert name == "fc_tree_attention_ws" and a[-3:] == (gpu.made[0][2], 4096, where or 0)


def test_tree_attention_takes_the_callers_workspace(monkeypatch):
    args = _attention_args()
    gpu = _Scratch(monkeypatch, 4096)
    ws = torch.zeros(5000, dtype=torch.uint8)
    fc.fc_tree_attention(**args, workspace=ws)
    assert not gpu.made and gpu.calls[0][1][-3:] == (ws.data_ptr(), 5000, 0)
    with pytest.raises(ValueError, match="workspace"):
        fc.fc_tree_attention(**args, workspace=ws.to(torch.int32))


def test_tree_attention_refuses_a_small_workspace(monkeypatch):
    args = _attention_args()
    gpu = _Scratch(monkeypatch, 4096)
    monkeypatch.setattr(fc, "_check", lambda fn, code: (_ for _ in ()).throw(RuntimeError(code)) if code else None)
    with pytest.raises(RuntimeError, match="2"):
        fc.fc_tree_attention(**args, workspace=torch.zeros(4095, dtype=torch.uint8))
    assert not gpu.calls


@pytest.mark.parametrize("stream", [None, _Stream()])
@pytest.mark.parametrize("call", ["build", "build_stats", "build_batched", "extend", "retrieve", "build_tree"])
def test_scratch_comes_from_the_stream_it_is_used_on(monkeypatch, call, stream):
    tok, u32 = torch.zeros(40, dtype=torch.uint16), lambda n: torch.zeros(n, dtype=torch.uint32)
    taken, lens, toks, ctx = _tree_inputs()
    out = fc.retrieve_outputs(4, 1, 10, 3, "cpu") if call == "retrieve" else fc.tree_outputs(3, 4, "cpu")
    gpu = _Scratch(monkeypatch, 4096)
    if call == "build":
        fc.fc_datastore_build(tok, sa_out=u32(40), stream=stream)
    elif call == "build_stats":
        fc.fc_datastore_build_stats(tok, sa_out=u32(40), stream=stream)
    elif call == "build_batched":
        fc.fc_datastore_build_batched(tok, [0, 10, 40], sa_out=u32(40), stream=stream)
    elif call == "extend":
        fc.fc_datastore_extend(tok, 5, u32(35), sa_out=u32(40), stream=stream)
    elif call == "retrieve":
        fc.fc_retrieve([_NoStore()], torch.zeros((4, 16), dtype=torch.uint16), k=10, m=3, out=out, stream=stream)
    else:
        fc.fc_build_tree(taken, lens, toks, ctx, c=4, out=out, stream=stream)
    assert [(s, n) for s, n, _ in gpu.made] == [(None if stream is None else stream.cuda_stream, 4096)]
    assert gpu.made[0][2] in gpu.calls[-1][1]
