"""The compiled half of the binding hands the library what the struct() methods say, in the plain case and in every other,
and refuses what they refuse (no GPU needed: nothing here gets as far as a launch)."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2508_08895_amd import binding as A


class _Stream:
    cuda_stream = 0


class _Tensor(torch.Tensor):
    pass


class _KV(A.KVCache):
    def struct(self):
        s = super().struct()
        s.num_blocks = 3
        return s


def _objects(dtype=torch.bfloat16, kv_class=A.KVCache):
    kv = kv_class(torch.zeros(5, 2, 16, 64, dtype=dtype), torch.zeros(5, 2, 16, 64, dtype=dtype),
                  torch.zeros(3, 4, dtype=torch.int32), 8)
    return kv, A.BatchState(3, 64, "cpu"), A.Step(6, 3, 3, "cpu", 2, 7)


def _open(kv, st, sp):
    st.open_parallel(torch.tensor([0, 2, 2, 5], dtype=torch.int32))


def _planned(kv, st, sp):
    sp.plan, sp.plan_key, sp.shared_mask = torch.empty(300, dtype=torch.int32), (1 << 62) + 5, 1


def _no_fault_word(kv, st, sp):
    st.fault = st.main_pos = st.stage_open = None


def _not_plain(kv, st, sp):
    kv.k = torch.nn.Parameter(kv.k)
    st.seq_len = st.seq_len.as_subclass(_Tensor)
    sp.kv_len = sp.kv_len.as_subclass(_Tensor)


def _views(kv, st, sp):
    whole = torch.zeros(9, dtype=torch.int32)
    st.stage_base, st.seq_len = whole[1:4], whole[4:7]
    kv.block_tables = torch.zeros(3, 6, dtype=torch.int32)[:, 1:5]


def _odd_numbers(kv, st, sp):
    st.owner_stride, sp.max_new_per_seq, sp.NQ = (1 << 32) + 64, True, -1


@pytest.mark.parametrize("change", [None, _open, _planned, _no_fault_word, _not_plain, _views, _odd_numbers])
@pytest.mark.parametrize("dtype,kv_class", [(torch.bfloat16, A.KVCache), (torch.float32, A.KVCache), (torch.bfloat16, _KV)])
def test_structures_are_those_of_struct(change, dtype, kv_class):
    kv, st, sp = _objects(dtype, kv_class)
    if change:
        change(kv, st, sp)
    assert A._calls().structs(kv, st, sp) == tuple(bytes(x.struct()) for x in (kv, st, sp))


def _f16(kv, st, sp):
    kv.k = kv.k.half()


def _three_dims(kv, st, sp):
    kv.k = kv.k[0]


def _flat_tables(kv, st, sp):
    kv.block_tables = kv.block_tables[0]


def _no_tensor(kv, st, sp):
    st.seq_len = [0, 0, 0]


def _no_attribute(kv, st, sp):
    del sp.kv_len


def _float_size(kv, st, sp):
    st.B = 3.0


@pytest.mark.parametrize("change", [_f16, _three_dims, _flat_tables, _no_tensor, _no_attribute, _float_size])
def test_what_struct_refuses_is_refused_alike(change):
    kv, st, sp = _objects()
    change(kv, st, sp)
    with pytest.raises(Exception) as want:
        [x.struct() for x in (kv, st, sp)]
    with pytest.raises(want.type):
        A._calls().structs(kv, st, sp)


def test_calls_reach_the_library_and_raise_what_it_says():
    kv, st, sp = _objects()
    q = torch.zeros(6, 8, 64, dtype=torch.bfloat16)
    ws = torch.zeros(64, dtype=torch.uint8)
    one = torch.ones(3, dtype=torch.int32)
    with pytest.raises(A.AspdError, match="aspd_attn_branch_chunk: invalid argument"):   # no branches, no tags
        A.aspd_attn_branch_chunk(kv, st, sp, q, ws, stream=_Stream)
    with pytest.raises(A.AspdError, match="aspd_attn_full_sequence: invalid argument"):  # no step of that kind
        A.aspd_attn_full_sequence(kv, st, sp, q, ws, stream=_Stream)
    with pytest.raises(A.AspdError, match="aspd_rope_append: invalid argument"):         # theta has to exceed one
        A.aspd_rope_append(kv, sp, q, q, q, 1, stream=_Stream)
    with pytest.raises(A.AspdError, match="aspd_build_branch_meta: invalid argument"):   # no such stage
        A.aspd_build_branch_meta(kv, st, 9, one, step=sp, stream=_Stream)
    with pytest.raises(A.AspdError, match="aspd_build_sequence_meta: invalid argument"):
        A.aspd_build_sequence_meta(kv, st, one, one, one, -1, step=A.Step(-1, 0, 3, "cpu"), stream=_Stream)
    assert sp.plan_key == 0                                    # (a refused call leaves it)
    sp.NQ = 0                                                  # a step without tokens launches nothing
    assert A.aspd_attn_serial_decode(kv, st, sp, q, ws, out=q, stream=_Stream) is q
    assert A.aspd_rope_append(kv, sp, q, q, q, 1e4, stream=_Stream) is q
    sp.NQ = 6
    with pytest.raises(TypeError):
        A.aspd_attn_serial_decode(kv, st, sp, q, ws, sm_scale="1", stream=_Stream)
    with pytest.raises(AttributeError):
        A.aspd_attn_serial_decode(kv, st, sp, q, 3, out=q, stream=_Stream)
    with pytest.raises(AttributeError):
        A.aspd_attn_serial_decode(kv, st, sp, q, ws, stream=0)


@pytest.mark.parametrize("whole", [int, np.int64, np.int32, torch.tensor])
def test_numbers_are_whatever_stands_for_a_whole_number(whole):
    kv, st, sp = _objects()
    one = torch.ones(3, dtype=torch.int32)
    with pytest.raises(A.AspdError, match="aspd_build_branch_meta: invalid argument"):   # no such stage
        A.aspd_build_branch_meta(kv, st, whole(9), one, step=sp, stream=_Stream)
    st.B, st.pos_mode, sp.NQ = whole(3), whole(A.POS_SAME_MAX), whole(6)
    with pytest.raises(A.AspdError, match="aspd_build_branch_meta: invalid argument"):
        A.aspd_build_branch_meta(kv, st, 9, one, step=sp, stream=_Stream)
    sp.NQ = whole(-1)
    with pytest.raises(A.AspdError, match="aspd_build_sequence_meta: invalid argument"):
        A.aspd_build_sequence_meta(kv, st, one, one, one, -1, step=sp, stream=_Stream)


@pytest.mark.parametrize("number", [9.0, "9", None, np.float32(9)])
def test_what_is_no_whole_number_is_refused(number):
    kv, st, sp = _objects()
    one = torch.ones(3, dtype=torch.int32)
    with pytest.raises(TypeError):
        A.aspd_build_branch_meta(kv, st, number, one, step=sp, plan=False, stream=_Stream)
    st.pos_mode = number
    with pytest.raises(TypeError):
        A.aspd_build_branch_meta(kv, st, 9, one, step=sp, plan=False, stream=_Stream)


def test_every_call_goes_to_the_library_that_lib_path_names(tmp_path):
    """Another build of the library, named before the first call: the process holds that one alone."""
    other = shutil.copy(A.LIB_PATH, tmp_path / "libaspd_other.so")
    program = """
import sys
from paper_2508_08895_amd import binding as A
A.LIB_PATH = sys.argv[1]
import torch
import test_binding_calls as T
T.test_calls_reach_the_library_and_raise_what_it_says()
loaded = {line.split()[-1] for line in open("/proc/self/maps") if "libaspd" in line}
assert loaded == {sys.argv[1]}, loaded
"""
    here = os.path.dirname(os.path.abspath(__file__))
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([os.path.dirname(here), here, os.environ.get("PYTHONPATH", "")]))
    run = subprocess.run([sys.executable, "-c", program, str(other)], env=env, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr[-2000:]
