"""The native argument marshalling of the Python entry points, on the CPU: every call below is rejected
before anything would be enqueued, so the device addresses are never used."""
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest
import torch

import paper_2511_02647_amd as fa
from paper_2511_02647_amd import build as fabuild


class Fake:
    """What a call asks of a device tensor."""
    def __init__(self, address=0x10000, cuda=True, contiguous=True, nbytes=0):
        self.is_cuda, self.nbytes, self._a, self._c = cuda, nbytes, address, contiguous

    def is_contiguous(self):
        return self._c

    def data_ptr(self):
        return self._a

    def numel(self):
        return 1


class Stream:
    cuda_stream = 0


@pytest.fixture(scope="module", autouse=True)
def built():
    fabuild.build(force=False)
    fa.load()


P = fa.make_params(2, 4, 2, 128, 2, torch.bfloat16)
T = Fake()


def decode(seg=(0, 64, 128), lens=(64, 10), **kw):
    fa.fedattn_decode(P, 0, T, T, T, T, seg, lens, stream=Stream, **kw)


@pytest.mark.parametrize("as_vec", [list, tuple, lambda x: np.asarray(x, np.int32), lambda x: np.asarray(x, np.int64),
                                    lambda x: np.repeat(np.asarray(x, np.int32), 2)[::2]])
def test_host_vectors_of_any_kind_reach_the_library(as_vec):
    with pytest.raises(fa.FedAttnError) as e:      # valid but for the workspace
        decode(as_vec([0, 64, 128]), as_vec([64, 10]))
    assert e.value.status == fa.FEDATTN_EWORKSPACE
    with pytest.raises(fa.FedAttnError) as e:
        decode(as_vec([0, 64, 128]), as_vec([64, 10]), workspace=Fake(nbytes=100))
    assert e.value.status == fa.FEDATTN_EWORKSPACE and "got 100" in str(e.value)
    with pytest.raises(fa.FedAttnError) as e:
        decode(as_vec([0, 64, 128]), as_vec([65, 10]))
    assert e.value.status == fa.FEDATTN_EINVAL and "seg_lens[0] = 65" in str(e.value)
    with pytest.raises(fa.FedAttnError) as e:
        decode(remote_lens=as_vec([0, 65]))
    assert "remote_lens[1] = 65" in str(e.value)


def test_wrong_lengths_and_kinds_are_python_errors():
    for kw in (dict(seg=(0, 64)), dict(lens=(1,)), dict(remote_lens=(1, 2, 3))):
        with pytest.raises(ValueError):
            decode(**kw)
    with pytest.raises(TypeError):
        decode(seg=np.zeros((2, 2), np.int32))
    with pytest.raises(ValueError):
        fa.fedattn_prefill(P, 0, T, T, T, T, (0, 4), stream=Stream)
    with pytest.raises(ValueError):
        fa.fedattn_prefill_sync_local_kv(P, T, [T], [T, T], T, (0, 4, 8), stream=Stream)
    with pytest.raises(ValueError):
        fa.fedattn_aggregate_kv(P, [T, T], [T], (0, 4, 8), T, T, stream=Stream)
    for bad, what in ((Fake(cuda=False), "device tensor"), (Fake(contiguous=False), "contiguous"), (torch.zeros(4), "device tensor")):
        with pytest.raises(TypeError, match="q must be .*%s" % what):
            fa.fedattn_prefill(P, 0, bad, T, T, T, (0, 4, 8), stream=Stream)
        with pytest.raises(TypeError, match=r"k_local\[1\] must be a contiguous device tensor"):
            fa.fedattn_prefill_sync_local_kv(P, T, [None, bad], [T, T], T, (0, 4, 8), stream=Stream)


def test_every_other_entry_point_reports_the_librarys_reason():
    odd = Fake(address=0x10008)
    for call, reason in (
            (lambda: fa.fedattn_prefill(P, 0, odd, T, T, T, (0, 4, 8), stream=Stream), "16-byte aligned"),
            (lambda: fa.fedattn_prefill(P, 0, T, T, T, T, (0, 4, 8), keep_chunks=T, stream=Stream), "chunk_tokens"),
            (lambda: fa.fedattn_prefill_sync_local_kv(P, T, [T, T], [T, T], T, (0, 4, 8), stream=Stream), "back to back"),
            (lambda: fa.fedattn_prefill_sync_local_kv(P, T, [None, T], [T, T], T, (0, 4, 8), stream=Stream), "is NULL"),
            (lambda: fa.fedattn_prefill_blocks(P, 0, 2, T, T, T, T, 1, 8, (0, 4, 8), stream=Stream), "multiples of 8"),
            (lambda: fa.fedattn_decode_blocks(P, 0, 2, T, T, T, T, 8, 1, (0, 4, 8), (1, 1), stream=Stream), "multiples of 8"),
            (lambda: fa.fedattn_decode_blocks_fused(P, 0, 70000, T, T, T, T, 8, 8, (0, 4, 8), (1, 1),
                                                    workspace=Fake(nbytes=1 << 30), stream=Stream), "65535"),
            (lambda: fa.fedattn_decode_static(P, 0, odd, T, T, T, (0, 4, 8), (1, 1), stream=Stream), "16-byte aligned"),
            (lambda: fa.fedattn_aggregate_kv(P, [None, None], [T, T], (0, 4, 8), T, T, stream=Stream), "is NULL")):
        with pytest.raises(fa.FedAttnError, match=reason):
            call()


def test_none_is_null_and_the_library_decides():
    fa.fedattn_prefill(P, 0, None, None, None, None, (0, 0, 0), stream=Stream)          # no tokens: nothing to read
    fa.fedattn_prefill_sync_local_kv(P, None, [None, None], [None, None], None, (0, 0, 0), stream=Stream)
    fa.fedattn_prefill_blocks(P, 0, 0, None, None, None, None, 0, 0, (0, 4, 8), stream=Stream)
    fa.fedattn_decode_blocks(P, 0, 0, None, None, None, None, 0, 0, (0, 4, 8), (1, 1), stream=Stream)
    fa.fedattn_aggregate_kv(P, [None, None], [None, None], (0, 0, 0), None, None, stream=Stream)
    for call in (lambda: fa.fedattn_prefill(P, 0, None, T, T, T, (0, 4, 8), stream=Stream),
                 lambda: fa.fedattn_prefill_blocks(P, 0, 2, T, T, T, None, 8, 8, (0, 4, 8), stream=Stream),
                 lambda: fa.fedattn_decode(P, 0, None, T, T, T, (0, 4, 8), (1, 1), stream=Stream),
                 lambda: fa.fedattn_decode_static(P, 0, T, T, T, None, (0, 4, 8), (1, 1), stream=Stream),
                 lambda: fa.fedattn_aggregate_kv(P, [T, T], [T, T], (0, 4, 8), None, T, stream=Stream)):
        with pytest.raises(fa.FedAttnError) as e:
            call()
        assert e.value.status == fa.FEDATTN_EINVAL and "NULL" in str(e.value)
    with pytest.raises(fa.FedAttnError) as e:      # a cache without capacity needs no address: only the workspace is missing
        fa.fedattn_decode(P, 0, T, None, None, T, (0, 0, 0), (0, 0), stream=Stream)
    assert e.value.status == fa.FEDATTN_EWORKSPACE


def test_params_and_numbers_as_before():
    for bad in (None, bytes(32), np.zeros(8, np.int32), 3):
        with pytest.raises((TypeError, AttributeError)):
            fa.fedattn_prefill(bad, 0, None, None, None, None, (0, 0, 0), stream=Stream)
    for block in (np.int64(0), 0.0, "0", torch.tensor(0), 1 << 70):   # anything int() takes; what does not fit is cut off
        fa.fedattn_prefill(P, block, None, None, None, None, (0, 0, 0), stream=Stream)
    with pytest.raises(TypeError):
        fa.fedattn_prefill(P, None, None, None, None, None, (0, 0, 0), stream=Stream)


def run_python(code):
    return subprocess.run([sys.executable, "-c", code], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120,
                          cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_the_library_loads_without_the_binding():
    p = run_python("import sys; sys.modules['paper_2511_02647_amd._native'] = None\n"
                   "import paper_2511_02647_amd as fa\n"
                   "assert fa.fedattn_is_sync_block(2, 1) and fa.fedattn_version()\n"
                   "try: fa.fedattn_prefill(None, 0, None, None, None, None, (0, 0))\n"
                   "except RuntimeError as e: print('loud:', e)")
    assert p.returncode == 0 and "loud: the native binding is missing" in p.stdout, p.stdout


def test_the_current_stream_without_torchs_shortcuts():
    p = run_python("import torch\n"
                   "for n in ('_cuda_getCurrentRawStream', '_cuda_getDevice'):\n"
                   "    if hasattr(torch._C, n): delattr(torch._C, n)\n"
                   "asked = []\n"
                   "class S: cuda_stream = 0\n"
                   "torch.cuda.current_device = lambda: 3\n"
                   "torch.cuda.current_stream = lambda d=None: asked.append(d) or S\n"
                   "import paper_2511_02647_amd as fa\n"
                   "fa.fedattn_prefill(fa.make_params(1, 1, 1, 64, 1, torch.float32), 0, None, None, None, None, (0, 0))\n"
                   "print('asked', asked)")
    assert p.returncode == 0 and "asked [3]" in p.stdout, p.stdout


def test_the_binding_is_named_after_its_python():
    assert os.path.basename(fabuild.NATIVE) == "_native" + sysconfig.get_config_var("EXT_SUFFIX") and os.path.exists(fabuild.NATIVE)
