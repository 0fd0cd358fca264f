"""What the consumers decide or refuse on the host, before anything is launched (no GPU is used:
the addresses are never dereferenced)."""
import pytest

import paper_2604_09558_amd as vt
import workloads

FAKE = 0x100000


def decode_descs(B, Hkv, G, S, D, dtype="bf16"):
    """Q, K, V of the decode chain at any size, without its data."""
    shapes = {"QKV": (B, 1, (G + 2) * Hkv * D), "Kcache": (B, Hkv, S, D), "Vcache": (B, Hkv, S, D)}
    spec = {k: (s, dtype, FAKE) for k, s in shapes.items()}
    return [vt.build_chain(workloads.c2_chain(B, Hkv, G, S, D), spec, n) for n in ("Q", "K", "V")]


def test_attention_plan_splits_only_where_every_pair_has_a_counter():
    """4096 (batch, kv head) pairs keep the splits asked for; more run with one, which needs no counter."""
    for B, want in ((512, 3), (513, 1)):
        assert vt.vt_decode_attn_plan(*decode_descs(B, 8, 2, 400, 128), n_splits=3)["splits"] == want
    # the counters' share of the workspace is the same for every problem
    share = {vt.vt_decode_attn_workspace(B, 8, 128, 400, 1) - B * 8 * 130 * 4 for B in (1, 16, 4096)}
    assert len(share) == 1


@pytest.mark.parametrize("stride,taken", [((1 << 26) - 8, True), (1 << 26, False), (1 << 28, False)])
def test_attention_plan_refuses_rows_beyond_a_32_bit_tile(stride, taken):
    """32 rows of K or V have to lie within 4 GiB (a row's offset in its tile is a 32-bit number): rows
    further apart run on the generic kernel, which the plan reports as unsupported."""
    q = vt.build_chain([], {"Q": ((1, 1, 1, 128), "bf16", FAKE)}, "Q")
    far = vt.build_chain([], {"K": ((1, 1, 40, 128), "bf16", FAKE, (40 * stride, 40 * stride, stride, 1))}, "K")
    near = vt.build_chain([], {"K": ((1, 1, 40, 128), "bf16", FAKE)}, "K")
    for k, v in ((far, near), (near, far)):
        if taken:
            assert vt.vt_decode_attn_plan(q, k, v)["splits"] == 1
        else:
            with pytest.raises(vt.VtError) as ei:
                vt.vt_decode_attn_plan(q, k, v)
            assert ei.value.code == vt.ERR_UNSUPPORTED


@pytest.mark.parametrize("ws_bytes,out,scale,word", [(16, FAKE, 0.125, "16 available"), (1 << 40, FAKE + 4, 0.125, "misaligned"), (1 << 40, FAKE, 1e9, "scale")])
def test_attention_says_why_neither_kernel_takes_a_call(ws_bytes, out, scale, word):
    """2^31 virtual elements are more than the generic kernel indexes: a call that it would otherwise take over
    is refused with the reason why the planned kernel left it, not with an earlier call's message."""
    q, k, v = decode_descs(1, 8, 16, 1 << 18, 64)
    with pytest.raises(vt.VtError):
        vt.vt_decode_attn(k, k, v, 0.125, FAKE, FAKE, 1 << 40)            # the earlier call: shapes do not fit
    with pytest.raises(vt.VtError) as ei:
        vt.vt_decode_attn(q, k, v, scale, out, FAKE, ws_bytes)
    assert ei.value.code == vt.ERR_UNSUPPORTED and word in str(ei.value)


def test_the_current_stream_is_never_lost(monkeypatch):
    """A torch without the functions for the bare handle: the public call is asked, and what it raises is
    raised, not turned into the default stream."""
    import torch
    from paper_2604_09558_amd import binding

    class Stream:
        cuda_stream = 0x5150

    monkeypatch.setattr(binding, "_current_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "init", lambda: None)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream())
    assert binding._stream(None).value == 0x5150
    assert binding._stream(0x20).value == 0x20 and binding._stream(Stream()).value == 0x5150

    def broken():
        raise RuntimeError("no such device")
    monkeypatch.setattr(torch.cuda, "current_stream", broken)
    with pytest.raises(RuntimeError):
        binding._stream(None)


def test_wide_stores_written_as_assembly_keep_their_wait_states():
    """The compiler does not see a store inside an asm statement: with more than 8 bytes a lane, the registers of
    its data must not be overwritten by the next two instructions, so the statement itself has to end in them."""
    import glob
    import os
    import re
    csrc = os.path.join(os.path.dirname(vt.__file__), "csrc")
    seen = 0
    for path in glob.glob(os.path.join(csrc, "*.h*")):
        for text in re.findall(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', text.split(":")[0])).split("\\n\\t")
            wide = [i for i, c in enumerate(code) if re.match(r"(global|flat|buffer)_store_dwordx[34]", c)]
            for i in wide:
                seen += 1
                assert i + 1 < len(code) and re.match(r"s_nop [1-9]|s_waitcnt vmcnt\(0\)", code[i + 1]), (path, code)
    assert seen >= 1
