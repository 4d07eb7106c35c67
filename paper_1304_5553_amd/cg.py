"""Conjugate gradients on the five-point model problem, in fused run-time
compiled kernels.

The paper lists a conjugate-gradient Krylov solver for large sparse systems
among the facilities shipped beside the elementwise and map-reduce kernels
(section "Further Facilities").  Here A is the symmetric positive definite
five-point operator on an nx-by-ny grid with zero boundary values (unknown
(j, k) at index j * nx + k), applied matrix-free.
The textbook iteration, as statements of the library's elementwise and
map-reduce kernels (the constants below; two (r . r, p . Ap) pairs, c of this
iteration and d of the next, swap roles every iteration):

    q = A p                           SPMV (shifted reads p[i +/- 1], p[i +/- nx])
    c[1] = p . q                      DOT
    d[0] = sum (r - alpha q)^2        RR_NEXT (the next r . r), alpha = c[0] / c[1]
    x += alpha p;  r -= alpha q;  p = r + beta p      UPDATE, beta = d[0] / c[0]

PoissonCG runs the same iteration in the library's fused kernels
(hipmr_poisson_cg): two launches per iteration inside a run, one native call
for the whole run, no host synchronisation, so a run can also be captured into
one HIP graph.  Sums are kept in FP64; vectors and scalars between kernels are
float, each rounded once.
"""

from __future__ import annotations

from . import hipmr as _hm

SPMV = ("float *q, const float *p, int nx",
        "int c = i % nx; "
        "q[i] = 4.0f*p[i] - (c != 0 ? p[i-1] : 0.0f) - (c != nx - 1 ? p[i+1] : 0.0f)"
        " - (i >= nx ? p[i-nx] : 0.0f) - (i + nx < n ? p[i+nx] : 0.0f)")
DOT = ("float: const float *p, const float *q", "p[i]*q[i]")
RR_NEXT = ("float: const float *r, const float *q, const float *c",
           "(r[i] - (c[0]/c[1])*q[i]) * (r[i] - (c[0]/c[1])*q[i])")
UPDATE = ("float *x, float *r, float *p, const float *q, const float *c, const float *d",
          "x[i] += (c[0]/c[1])*p[i]; r[i] -= (c[0]/c[1])*q[i]; p[i] = r[i] + (d[0]/c[0])*p[i]")
START = ("float *x, float *r, float *p, const float *b", "x[i] = 0.0f; r[i] = b[i]; p[i] = b[i]")

BYTES_PER_UNKNOWN = 52         # per iteration, of the four statements
FUSED_BYTES_PER_UNKNOWN = 32   # of the fused kernels: cgr 12, cgu 20

# Launch configuration for the statements above when they are run one by one:
# they reread their vectors every iteration, so temporal accesses, which keep
# them in the last-level cache, suit grids up to its size (4096 x 4096 in one
# process: 136 us per iteration against 165 us with streaming accesses).
CACHED = _hm.LaunchConfig(flags=_hm.CFG_TEMPORAL)


class PoissonCG:
    """Device state and kernels of CG for one grid size.  All calls are
    asynchronous on `stream` (default: torch's current stream)."""

    def __init__(self, nx, ny, device=None, stream=None):
        import torch
        self.nx, self.ny, self.n = int(nx), int(ny), int(nx) * int(ny)
        dev = device or torch.device("cuda")
        self.stream = stream
        f = dict(dtype=torch.float32, device=dev)
        self.x, self.r, self.p, self.q = (torch.empty(self.n, **f) for _ in range(4))
        self.s = torch.zeros(4, **f)          # two (r . r, p . Ap) pairs
        self.parity = 0                       # which pair holds this iteration's r . r
        # block partials and a second buffer of p, this solver's own
        nbytes = _hm.lib().hipmr_poisson_cg_workspace_bytes(self.nx, self.ny)
        self._ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device=dev)
        if stream is not None and self._ws.is_cuda:   # a run may outlive the solver on that stream
            on = stream if isinstance(stream, torch.cuda.Stream) else \
                torch.cuda.ExternalStream(_hm._stream_ptr(stream), self._ws.device)
            for t in (self.x, self.r, self.p, self.q, self.s, self._ws):
                t.record_stream(on)

    @property
    def k(self):
        """Handles of the iteration's statements (compiled when asked for)."""
        return {name: _hm.compile(expr, sig, name=f"cg_{name}") for name, (sig, expr) in
                dict(spmv=SPMV, dot=DOT, rrn=RR_NEXT, update=UPDATE, start=START).items()}

    def _pairs(self):
        a, b = self.s[0:2], self.s[2:4]
        return (a, b) if self.parity == 0 else (b, a)

    @property
    def rr(self):
        """This iteration's r . r (a one-element device tensor)."""
        return self._pairs()[0][0:1]

    def _start(self, b, iters):
        """A run from the right-hand side b (a tensor or a device address)."""
        if hasattr(b, "numel") and b.numel() < self.n:
            raise _hm.InvalidError(f"array 'b' has {b.numel()} elements, fewer than n = {self.n}")
        b = b if isinstance(b, int) else 0 if b is None else b.data_ptr()
        if self.n > 0 and b == 0:
            raise _hm.InvalidError("array argument 'b' is NULL")
        self.parity = 0
        if self.n == 0:
            self.s[0:1].zero_()
        self._run(b, iters)

    def _run(self, b, iters):
        iters = max(0, int(iters))
        _hm._check(_hm.lib().hipmr_poisson_cg(
            self.nx, self.ny, b, iters, self.x.data_ptr(), self.r.data_ptr(), self.p.data_ptr(),
            self.q.data_ptr(), self.s.data_ptr(), self.parity, self._ws.data_ptr(),
            self._ws.numel(), _hm._stream_ptr(self.stream)))
        self.parity ^= iters & 1

    def start(self, b):
        """x = 0, r = p = b, r . r = b . b."""
        self._start(b, 0)

    def step(self):
        """One CG iteration (three launches, no host sync)."""
        self._run(None, 1)

    def capture(self, iters):
        """A HIP graph of `iters` iterations (an even count, so that every
        replay starts and ends with r . r in the first pair, as after start()).
        The kernels must have run once; the solver's stream must not be the
        null stream."""
        if self.stream is None:
            raise _hm.InvalidError("graph capture needs a non-default stream")
        if iters % 2:
            raise _hm.InvalidError("capture an even number of iterations")
        saved, self.parity = self.parity, 0
        g = _hm.Graph()
        try:
            with g.capture(self.stream):
                self._run(None, iters)
        finally:
            self.parity = saved
        return g

    def solve(self, b, iters):
        """start(b), then `iters` iterations in one native call (2 iters + 2 launches)."""
        self._start(b, iters)
        return self.x


__all__ = ["PoissonCG", "SPMV", "DOT", "RR_NEXT", "UPDATE", "START", "BYTES_PER_UNKNOWN",
           "FUSED_BYTES_PER_UNKNOWN", "CACHED"]
