"""The paper's model as one object (Section 4): the encoding followed by the 64-64 ReLU network, trained with Adam on
tables and weights.  Bookkeeping only: a training iteration is one call into the C-ABI library (hashgrid_train_step), and so are the
output at a batch of points and its gradient with respect to the position; this file allocates the buffers and keeps the
step counter.

Defaults are the paper's (Section 4, "Initialization" and "Training"): tables U(-1e-4, 1e-4) in half precision behind a
full-precision master copy, Glorot-uniform weights, Adam with beta1 = 0.9, beta2 = 0.99, eps = 1e-15, an L2 factor
of 1e-6 on the network's weights only, learning rate 1e-2 (the paper: 1e-4 for signed distance functions).
"""
from __future__ import annotations

import math

import torch

from .binding import (_LOSSES, HG_TRAIN_SCRATCH_BYTES, HashGrid, HashGridError, _dev, hashgrid_adam_config,
                      hashgrid_train_state)

N_HIDDEN = 64


class HashGridModel:
    def __init__(self, d: int, n_out: int, L: int = 16, F: int = 2, T: int = 1 << 19, N_min: int = 16, N_max: int = 2048,
                 loss: str = "l2", lr: float = 1e-2, l2_reg: float = 1e-6, loss_scale: float = 1.0, seed: int = 0,
                 interp: int = 0):
        """loss: "l2" or "mape".  The paper's loss is a mean over the batch; what travels backward here is the gradient
        of the summed loss times loss_scale, because the network's backward pass rounds dL/dout to half precision
        and 1/n would push it into the subnormals.  Adam is indifferent to a common factor of all gradients, and
        the L2 term of the weights gets the same factor (n * loss_scale), so the update is the mean loss's."""
        self.grid = HashGrid(d, L, F, T, N_min, N_max, "f16", "f16", interp)
        self.d, self.n_in, self.n_out = d, L * F, n_out
        self.loss, self.lr, self.l2_reg, self.loss_scale = loss, lr, l2_reg, loss_scale
        gen = torch.Generator(device="cuda").manual_seed(seed)
        n = self.grid.n_entries
        self.tables = torch.rand((n, F), device="cuda", generator=gen) * 2e-4 - 1e-4
        self.tables_half = self.tables.half()
        # _tab_zeros: zero between steps; where a step sums gradients that several workgroups share
        self._tab_zeros, self._tab_m, self._tab_v = (torch.zeros_like(self.tables) for _ in range(3))
        self._shapes = [(N_HIDDEN, self.n_in), (N_HIDDEN, N_HIDDEN), (n_out, N_HIDDEN)]
        init = [(torch.rand(s, device="cuda", generator=gen) * 2 - 1) * math.sqrt(6.0 / (s[0] + s[1])) for s in self._shapes]
        self.weights = torch.cat([w.reshape(-1) for w in init]).contiguous()  # W1, W2, W3 in one array: one optimiser call
        self.weights_half = self.weights.half()
        self._net_m, self._net_v = torch.zeros_like(self.weights), torch.zeros_like(self.weights)
        self._W, self._n_weights = self._views(self.weights_half), self.weights.numel()
        self.steps = 0
        self._loss_sum = torch.zeros(1, dtype=torch.float64, device="cuda")
        self._scratch = torch.empty(HG_TRAIN_SCRATCH_BYTES, dtype=torch.uint8, device="cuda")
        self._state = hashgrid_train_state(
            n_out=n_out, tables_adam=hashgrid_adam_config(0.0, 0.9, 0.99, 1e-15, 0.0),
            weights_adam=hashgrid_adam_config(0.0, 0.9, 0.99, 1e-15, 0.0), loss_sum=self._loss_sum.data_ptr(),
            scratch=self._scratch.data_ptr())
        self._buf_B = 0

    def _views(self, flat):
        out, at = [], 0
        for r, c in self._shapes:
            out.append(flat[at:at + r * c].view(r, c))
            at += r * c
        return out

    def _buffers(self, B: int):
        if B != self._buf_B:
            self._y = torch.empty((B, self.n_in), dtype=torch.float16, device="cuda")
            self._dy = torch.empty_like(self._y)
            self._buf_B = B

    def _network(self):
        """W1, W2, W3 of weights_half as it is now.  The views are made again where it lies elsewhere than they do (they keep
        their memory, so what lies where they do is theirs); making them costs a small call as much as its kernel."""
        if self.weights_half.data_ptr() != self._W[0].data_ptr():
            _dev(self.weights_half, torch.float16, (self._n_weights,), "weights_half")
            self._W = self._views(self.weights_half)
        return self._W

    def infer(self, x: torch.Tensor, out: torch.Tensor | None = None) -> torch.Tensor:
        """The network's output [B, n_out] fp32 for points x [B, d] in [0,1)^d."""
        return self.grid.encode_mlp_fwd(x, self.tables_half, *self._network(), out)

    def input_gradient(self, x: torch.Tensor, dLdout: torch.Tensor | None = None) -> torch.Tensor:
        """d(sum_i dLdout_i * out_i) / dx [B, d] fp32: with the default dLdout = 1 and one output, the gradient of the
        output with respect to the position (the normal of a signed distance function, Section 3: the encoding is
        continuous and its derivative piecewise constant)."""
        return self.grid.encode_mlp_bwd_input(x, self.tables_half, *self._network(), dLdout)

    def _train_state(self, B: int) -> hashgrid_train_state:
        """The library's view of this model as it is now: tensors that the caller has replaced or loaded count, and are
        checked, from this call on (3 us of a call; nothing is kept by a tensor's address)."""
        st, f32, f16 = self._state, torch.float32, torch.float16
        table, flat = (self.grid.n_entries, self.grid.F), (self._n_weights,)
        st.tables = _dev(self.tables, f32, table, "tables")
        st.tables_half = _dev(self.tables_half, f16, table, "tables_half")
        st.tables_m = _dev(self._tab_m, f32, table, "first moment of the tables")
        st.tables_v = _dev(self._tab_v, f32, table, "second moment of the tables")
        st.tables_zeros = _dev(self._tab_zeros, f32, table, "shared table sums")
        st.weights = _dev(self.weights, f32, flat, "weights")
        st.weights_half = _dev(self.weights_half, f16, flat, "weights_half")
        st.weights_m = _dev(self._net_m, f32, flat, "first moment of the weights")
        st.weights_v = _dev(self._net_v, f32, flat, "second moment of the weights")
        if self.loss not in _LOSSES:
            raise HashGridError(f"unknown loss {self.loss!r}")
        st.loss, st.loss_scale = _LOSSES[self.loss], self.loss_scale
        st.tables_adam.lr = st.weights_adam.lr = self.lr
        st.weights_adam.l2_reg = self.l2_reg * self.loss_scale * (B * self.n_out)
        return st

    def step(self, x: torch.Tensor, target: torch.Tensor) -> None:
        """One training iteration on the batch (x [B, d], target [B, n_out], fp32 device tensors).  Nothing here
        synchronises; last_loss() does."""
        B = x.shape[0]
        self._buffers(B)
        self.grid.train_step(self._train_state(B), x, target, self._y, self._dy, self.steps + 1)
        self.steps += 1
        self._n_last = B * self.n_out

    def last_loss(self) -> float:
        """Mean loss over the scalars of the last step's batch, before that step's update (synchronises)."""
        return float(self._loss_sum.cpu()[0]) / self._n_last
