"""iso_start runs some collectives in fewer kernels than their launch list has (small ones in one, the rounds of a
dimension together): the tests that are about the kernels of the rounds run that list as well."""
import torch

import paper_1606_07676_amd as iso


def start_both_ways(req, recv, work=None, stream=None, starts=1):
    """iso_start (`starts` times), and where that takes other kernels than the request's launch list, the list
    launch by launch over a receive buffer of 0xEE and a workspace of 0xDD: the same bytes.  Leaves the result in recv."""
    for _ in range(starts):
        iso.iso_start(req, stream)
    iso.iso_wait(req)
    n = iso.iso_request_info(req)["launches"]
    if iso.iso_request_start_info(req)["kernels"] == n:
        return
    first = recv.clone()
    recv.fill_(0xEE)
    if work is not None:
        work.fill_(0xDD)
    torch.cuda.synchronize()
    for q in range(n):
        iso.iso_start_range(req, q, 1, stream)
    iso.iso_wait(req)
    assert torch.equal(recv, first), f"the launch list differs from iso_start: {iso.iso_request_info(req)}"
