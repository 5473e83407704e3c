"""Workspace sizes (GPU): one workspace, sized for a program's largest batch,
serves its smaller batches.

RB_FLAG_FROM_LISTS calls check the workspace like every lookup but read only the
neighbour lists in it, so that every batch size can be tried without a bank.
"""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("dtype,N,d,sizes", [
    ("bf16", 4_000_000, 384, [1_024, 1_023, 1_006, 1_000, 900, 700, 513, 512, 511, 300, 257]),
    ("bf16", 4_000_000, 512, [1_024, 1_006, 900, 513, 300, 257, 256, 200, 129]),
    ("bf16", 9_000_000, 64, [2_048, 1_500, 1_025, 1_024, 500, 470, 450, 300]),
    ("f32", 3_000_000, 96, [4_096, 4_000, 2_000, 1_500, 1_300, 1_200, 900, 64, 17, 1]),
])
@pytest.mark.parametrize("overlap", [0, 1])
def test_workspace_of_the_largest_batch_serves_smaller_ones(dtype, N, d, sizes, overlap):
    import paper_2606_17949_amd as rb
    code = rb.RB_BF16 if dtype == "bf16" else rb.RB_F32
    k, M, big = 10, 1, max(sizes)
    ws = torch.zeros(rb.rb_workspace_size(big, N, d, code, k, M), dtype=torch.uint8, device=DEV)
    labels = torch.ones(N, M, device=DEV)
    out = torch.empty(big, M, device=DEV)
    opts = rb.options(flags=rb.RB_FLAG_FROM_LISTS | (rb.RB_FLAG_OVERLAP if overlap else 0))
    for B in sizes:
        need = rb.rb_workspace_size(B, N, d, code, k, M)
        print(f"workspace {dtype} B={B} N={N} d={d}: {need / 2**20:.1f} MiB", flush=True)
        assert need <= ws.numel()
        for size, status in ((ws.numel(), rb.RB_OK), (256, rb.RB_ERR_WORKSPACE)):
            assert rb._lib.rb_knn_predict(
                None, None, None, code, B, N, d, k, labels.data_ptr(), labels.data_ptr(), M,
                ctypes.byref(opts), None, None, out.data_ptr(), out.data_ptr(), ws.data_ptr(),
                size, torch.cuda.current_stream().cuda_stream) == status
    torch.cuda.synchronize()
