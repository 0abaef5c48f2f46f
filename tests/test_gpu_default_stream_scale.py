"""GPU: the tensor scale without a workspace, on the default stream (one launch on the library's own scratch
words) against a stream of its own (one workgroup, or three launches), and against the oracle."""
import threading

import pytest
import torch

from oracle import ref
from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import workloads as wl

pytestmark = pytest.mark.gpu

RHT_SEED = wl.C5_RHT_SEED


def _on_its_own_stream(call):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = call()
    s.synchronize()
    return got


# either side of 128 KiB, of 512 KiB (one workgroup on the default stream), of 768 KiB (one workgroup on any other), the
# smallest tensor
@pytest.mark.parametrize("rows,cols", [(1, 16), (64, 1024), (65, 1024), (256, 1024), (257, 1024), (384, 1024), (385, 1024), (1000, 2064)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_scale_matches_the_other_forms(rows, cols, dtype):
    x = wl.make("c3", rows, cols, dtype=dtype)
    xd = x.cuda()
    options = [dict()] + ([dict(rht=1, rht_seed=RHT_SEED, layout=B.ROWWISE)] if cols % 16 == 0 else [])
    options += [dict(rht=1, rht_seed=RHT_SEED, layout=B.COLWISE)] if rows % 16 == 0 else []
    for kw in options:
        a = B.nvfp4_46_tensor_scale(xd, **kw)
        b = _on_its_own_stream(lambda: B.nvfp4_46_tensor_scale(xd, **kw))
        assert torch.equal(a, b), kw
        assert a.item() == ref.tensor_scale(wl.host_array(x), **kw), kw


@pytest.mark.parametrize("rows", [96, 384, 385, 1024])       # 768 KiB: either side of one launch for both
def test_scale_and_codes_match_the_other_forms(rows):
    x = wl.make("c1", rows, 1024).cuda()
    for kw in (dict(), dict(rounding=B.SR, sr_seed=5), dict(layout=B.COLWISE, rht=1, rht_seed=7)):
        if kw.get("layout") == B.COLWISE and rows % 16:
            continue
        a = B.nvfp4_46_scale_quantize(x, **kw)
        b = _on_its_own_stream(lambda: B.nvfp4_46_scale_quantize(x, **kw))
        assert all((a[k] is None and b[k] is None) or torch.equal(a[k], b[k]) for k in a), kw


def test_calls_from_several_threads_share_the_words():
    """The default stream is one for all threads, so their calls take turns on the words."""
    xs = [wl.make("c1", 256 + 16 * i, 1024).cuda() * (i + 1) for i in range(4)]
    want = [ref.tensor_scale(wl.host_array(x.cpu())) for x in xs]
    got = [[] for _ in xs]

    def calls(i):
        for _ in range(50):
            got[i].append(B.nvfp4_46_tensor_scale(xs[i]))

    threads = [threading.Thread(target=calls, args=(i,)) for i in range(len(xs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i, w in enumerate(want):
        assert len(got[i]) == 50 and all(a.item() == w for a in got[i]), i
