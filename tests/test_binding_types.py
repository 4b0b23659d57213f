"""The binding's table of tensor types: complete for every thread from its first use on, and one way a table."""
import importlib.util
import sys
import threading

import pytest
import torch

from paper_2605_19660_amd import binding as ob


def test_first_use_by_several_threads():
    """A fresh copy of the module for every round (nothing of it is loaded by the first call but the table)."""
    spec = importlib.util.spec_from_file_location("binding_fresh", ob.__file__)
    was, failed = sys.getswitchinterval(), []
    sys.setswitchinterval(1e-6)
    try:
        for _ in range(1500):
            fresh = importlib.util.module_from_spec(spec)
            sys.modules[spec.name] = fresh   # (its dataclasses look themselves up there)
            spec.loader.exec_module(fresh)
            start = threading.Barrier(4)

            def first():
                start.wait()
                try:
                    assert fresh.torch_dtype(ob.F16) is torch.float16 and fresh.dtype_code(torch.bfloat16) == ob.BF16
                except BaseException as e:
                    failed.append(e)

            threads = [threading.Thread(target=first) for _ in range(4)]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
    finally:
        sys.setswitchinterval(was)
        sys.modules.pop(spec.name, None)
    assert not failed, (len(failed), failed[:3])


@pytest.mark.parametrize("code,dt", [(ob.F32, torch.float32), (ob.BF16, torch.bfloat16), (ob.F16, torch.float16)])
def test_each_way_refuses_the_other(code, dt):
    assert ob.torch_dtype(code) is dt and ob.dtype_code(dt) == code
    for call, arg in ((ob.torch_dtype, dt), (ob.dtype_code, code), (ob.torch_dtype, 7), (ob.dtype_code, torch.int32)):
        with pytest.raises(KeyError):
            call(arg)
