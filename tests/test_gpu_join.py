"""GPU: a join of the context's two streams that fails leaves nothing running on the
second one (whose buffers the next solve reuses)."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


def test_failed_join_waits_for_the_second_stream():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2602_05804_amd as P

    print("case: join of two streams without an event", flush=True)
    torch.cuda.init()
    f = P.lib()._ZN4sfmm12join_streamsEP12ihipStream_tS1_P11ihipEvent_t
    f.restype, f.argtypes = C.c_int, [C.c_void_p] * 3
    main, aux = torch.cuda.current_stream(), torch.cuda.Stream()
    a = torch.ones(4096, 4096, device="cuda")
    event = torch.cuda.Event()
    event.record(main)
    torch.cuda.synchronize()

    def busy():
        with torch.cuda.stream(aux):
            for _ in range(20):
                a.matmul(a)

    busy()
    assert not aux.query()
    assert f(main.cuda_stream, aux.cuda_stream, None) != 0  # refused: no event
    assert aux.query()
    busy()
    assert f(main.cuda_stream, aux.cuda_stream, event.cuda_event) == 0
    done = torch.cuda.Event()
    done.record(main)
    done.synchronize()
    assert aux.query()
