"""How many of a few calls are through well before a kernel of another stream, which fills the device, is."""


def calls_through_early(call):
    import torch
    full = torch.rand(1 << 29, device="cuda")
    out = torch.empty_like(full)
    call()
    torch.erfinv(full, out=out)
    torch.cuda.synchronize()
    early = 0
    for _ in range(8):                           # streams share a few hardware queues: some of them share none with this one
        other, done, end = torch.cuda.Stream(), torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        with torch.cuda.stream(other):
            torch.erfinv(full, out=out)          # some milliseconds
            end.record()
        torch.cuda._sleep(30_000)                # until that kernel has filled the device
        got = call()
        done.record()
        torch.cuda.synchronize()
        early += done.elapsed_time(end) > 0.8    # of 2.6 ms; a block that waits is through at the end, or a moment before it
    return early, got
