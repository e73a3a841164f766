"""The native argument marshalling: wrong objects, types and shapes are refused with the exceptions of a Python check, before
anything is enqueued."""
import pytest
import torch


@pytest.fixture(scope="module")
def gr():
    import os

    import paper_2512_11529_amd as gr
    from paper_2512_11529_amd import build
    if not (os.path.exists(gr.LIB_PATH) and os.path.exists(build.BIND_PATH)):
        build.build_lib()
    return gr


def test_tensors_off_the_gpu_and_other_objects_are_refused(gr):
    t = torch.zeros(2, 3, dtype=torch.int32)
    with pytest.raises(TypeError, match="k_unshared: expected a contiguous CUDA tensor"):
        gr.gr_beam_reorder(t, torch.zeros(2, 3, 1, 2, 64, dtype=torch.bfloat16), None, 1)
    with pytest.raises(TypeError, match="q: expected a contiguous CUDA tensor"):
        gr.gr_prefill_attn([1], t, t, t, 1.0, 1, 1, out=t)
    with pytest.raises(TypeError, match="parent: expected a contiguous CUDA tensor"):
        gr.gr_beam_slot_update(t, None, 1, 3, out=t)
    with pytest.raises(ValueError, match="must be preallocated"):
        gr.gr_beam_select_noalloc(None, torch.zeros(1, 1, 4), t, torch.zeros(1, 1, 3), t, 0, {})


def test_a_library_loaded_later_takes_the_calls(gr, monkeypatch, tmp_path):
    # the marshalling module is bound again when load_library() is given another library
    import ctypes
    import shutil

    bound = []

    class Recorder:
        def bind(self, *a):
            bound.append(a[0])

    address = lambda lib: ctypes.cast(lib.gr_beam_attn, ctypes.c_void_p).value
    monkeypatch.setattr(gr, "_lib", None)
    monkeypatch.setattr(gr, "_native", None)
    monkeypatch.setattr(gr.importlib.util, "module_from_spec", lambda spec: Recorder())
    monkeypatch.setattr(gr.importlib.machinery.ExtensionFileLoader, "exec_module", lambda self, module: None)
    first = gr.load_library()
    gr._marshal()
    other = gr.load_library(shutil.copy(gr.LIB_PATH, tmp_path / "libgr_other.so"))
    gr._marshal()
    assert address(first) != address(other)
    assert bound == [address(first), address(other)]


@pytest.mark.gpu
def test_types_shapes_and_strides_are_checked(gr):
    dev = torch.device("cuda:0")
    bf = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device=dev)
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device=dev)
    q, k, own, cu = bf(1, 4, 2, 64), bf(8, 2, 64), bf(1, 4, 3, 2, 64), torch.tensor([0, 8], dtype=torch.int32, device=dev)
    call = lambda **kw: gr.gr_beam_attn(*(kw.get(n, v) for n, v in dict(q=q, k=k, v=k.clone(), cu=cu, ku=own, vu=own.clone(), u=1, scale=0.125, max_L=8,
                                                                          total_L=8).items()), **{n: v for n, v in kw.items() if n in ("out", "lse_out", "slot")})
    call()
    for bad, kind, text in ((dict(q=q.float()), TypeError, "q: expected torch.bfloat16, got torch.float32"),
                            (dict(q=bf(4, 2, 64)), ValueError, "q: expected 4 dimensions"),
                            (dict(k=bf(8, 2, 32)), ValueError, r"k_shared: expected shape \(8, 2, 64\), got \(8, 2, 32\)"),
                            (dict(v=bf(7, 2, 64)), ValueError, "v_shared: expected shape"),
                            (dict(cu=i32(3)), ValueError, r"cu_seqlens: expected shape \(2,\), got \(3,\)"),
                            (dict(ku=bf(1, 4, 3, 64, 2).transpose(3, 4)), TypeError, "k_unshared: expected a contiguous CUDA tensor"),
                            (dict(total_L=9), ValueError, "fewer rows than total_L"),
                            (dict(out=bf(1, 4, 2, 32)), ValueError, "out: expected shape"),
                            (dict(lse_out=bf(1, 4, 2)), TypeError, "lse_out: expected torch.float32"),
                            (dict(slot=i32(1, 4, 2)), ValueError, "slot: expected shape"),
                            (dict(u="x"), ValueError, "invalid literal")):
        with pytest.raises(kind, match=text):
            call(**bad)
    with pytest.raises(gr.GrError) as e:
        call(u=4)
    assert e.value.status == -1
    f32 = lambda *s: torch.zeros(s, dtype=torch.float32, device=dev)
    with pytest.raises(ValueError, match="scores_in: expected shape"):
        gr.gr_beam_select(None, f32(1, 4, 16), f32(1, 5), i32(1, 4, 3), i32(1, 4, 2), 0)
    with pytest.raises(TypeError, match="parent: expected torch.int32, got torch.float32"):
        gr.gr_beam_select(None, f32(1, 4, 16), f32(1, 4), i32(1, 4, 3), i32(1, 4, 2), 0, out=dict(parent=f32(1, 4)))
    with pytest.raises(ValueError, match="v_unshared: expected shape"):
        gr.gr_beam_reorder(i32(1, 4), own, bf(1, 4, 3, 1, 64), 1)
    with pytest.raises(ValueError, match="slot_in: expected shape"):
        gr.gr_beam_slot_update(i32(1, 4), i32(1, 4, 2), 1, 3)


@pytest.mark.gpu
def test_calls_on_another_stream(gr):
    # the handle of the given stream is used: work queued on it in front of the call is seen by the call
    dev = torch.device("cuda:0")
    side = torch.cuda.Stream()
    parent = torch.zeros(1, 64, dtype=torch.int32, device=dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(2_000_000)
        parent.fill_(5)
    got = gr.gr_beam_slot_update(parent, None, 1, 3, stream=side)
    torch.cuda.synchronize()
    assert (got[0, :, 0] == 15).all()
