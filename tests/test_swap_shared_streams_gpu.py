"""Engines that follow the same compute stream share one copy stream per direction: round trips that overlap in time, from one thread and from several,
and an engine that goes away while another one's copies are under way."""
import threading

import pytest
import torch

from paper_1812_07816_amd import swap as sw

pytestmark = pytest.mark.gpu


def _engine(sizes):
    e = sw.SwapEngine(budget_bytes=1, host_pool_bytes=sum((b + 4095) // 4096 * 4096 for b in sizes) + 4096, policy=sw.POLICY_ALL)
    e.set_timeline(len(sizes), 2 * len(sizes))
    for i, b in enumerate(sizes):
        e.register(i, b, i, i, 2 * len(sizes) - 1 - i, 2 * len(sizes) - 1 - i, sw.TAG_ENCODER)
    e.plan(allow_over_budget=True)
    return e


def _out(e, src):
    for i, t in enumerate(src):
        e.swap_out(i, t.data_ptr())
        e.release(i)


def _back(e, src):
    back = [torch.zeros_like(t) for t in src]
    for i in reversed(range(len(src))):
        e.swap_in(i, back[i].data_ptr())
        e.wait_in(i)
        e.done(i)
    torch.cuda.current_stream().synchronize()
    return all(torch.equal(a, b) for a, b in zip(src, back))


def _tensors(seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn(n, generator=gen, device="cuda") for n in (3 << 20, 70001, 1 << 18)]


def test_engines_in_turn_and_one_that_goes_away(device):
    src = [_tensors(k) for k in range(3)]
    engines = [_engine([t.numel() * 4 for t in s]) for s in src]
    for step in range(3):
        for e, s in zip(engines, src):
            e.reset_step()
            _out(e, s)
        if step == 1:
            engines.pop(0).close()       # its copies end first; the others' go on
            src.pop(0)
        for e, s in zip(engines, src):
            assert _back(e, s)
            st = e.stats()
            assert st["n_swapped_out"] == st["n_swapped_in"] == 3 and st["copy_ms_out"] > 0
    for e in engines:
        e.close()
    e = _engine([t.numel() * 4 for t in src[0]])     # the streams come back with the next engine
    e.reset_step()
    _out(e, src[0])
    assert _back(e, src[0])
    e.close()


def test_engines_of_several_threads(device):
    ok = [0, 0, 0]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            src = _tensors(10 + k)
            torch.cuda.current_stream().synchronize()
            for _ in range(3):
                e = _engine([t.numel() * 4 for t in src])
                for _ in range(2):
                    e.reset_step()
                    _out(e, src)
                    ok[k] += _back(e, src)
                e.close()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert ok == [6, 6, 6]


def test_checksums_still_under_way_when_the_mode_is_switched_off(device):
    """The checksum of a swapped-in tensor runs behind the copy that the caller waits for."""
    src = [torch.arange(64 << 20, device="cuda", dtype=torch.int32)]
    e = _engine([src[0].numel() * 4])
    for _ in range(3):
        e.reset_step()
        e.set_verify(True)
        _out(e, src)
        back = torch.empty_like(src[0])
        e.swap_in(0, back.data_ptr())
        e.wait_in(0)
        torch.cuda.current_stream().synchronize()     # the copy has landed
        e.set_verify(False)
        st = e.stats()
        assert (st["n_checksummed"], st["n_checksum_mismatch"]) == (1, 0)
        assert torch.equal(back, src[0])
    e.close()
