"""The calls of csrc/fastcall.cpp through ctypes: the same functions with the same arguments, several microseconds a call slower,
for a package whose call layer has not been built (it needs torch's headers; the library itself does not)."""
from __future__ import annotations

import torch


class Calls:
    def __init__(self, lib, stream):
        """lib: the library, with its signatures set; stream: what turns a stream argument into a handle."""
        self.lib, self.handle = lib, stream

    def _matrix(self, t):
        if t is None:
            return None, 0
        if not isinstance(t, torch.Tensor):
            raise TypeError("expected a tensor")
        assert t.dim() == 2 and t.stride(1) == 1 and t.dtype == torch.float32, "expected a float32 matrix with contiguous rows"
        return t.data_ptr(), t.stride(0)

    def _memory(self, t):
        return t if t is None or isinstance(t, int) else t.data_ptr()

    def _matrix_with_ld(self, t, ld):
        return self._matrix(t) if ld is None else (self._memory(t), ld)

    def forward(self, layer, X, Y, batch, stream):
        return self.lib.sparse_linear_forward(layer, *self._matrix(X), *self._matrix(Y), batch, self.handle(stream))

    def backward(self, layer, X, Y, dY, dX, dvalues, dbias, batch, stream):
        return self.lib.sparse_linear_backward(layer, *self._matrix(X), *self._matrix(Y), *self._matrix(dY), *self._matrix(dX), self._memory(dvalues),
                                               self._memory(dbias), batch, self.handle(stream))

    def update(self, values, velocity, grad, n, lr, momentum, nesterov, stream):
        step = self.lib.sgd_update_values_nesterov if nesterov else self.lib.sgd_update_values
        return step(self._memory(values), self._memory(velocity), self._memory(grad), n, lr, momentum, self.handle(stream))

    def train_step(self, mlp, X, ldx, labels, batch, lr, momentum, workspace, loss, stream):
        return self.lib.mlp_train_step(mlp, *self._matrix_with_ld(X, ldx), self._memory(labels), batch, lr, momentum, workspace.data_ptr(), workspace.nbytes,
                                       self._memory(loss), self.handle(stream))

    def mlp_forward(self, mlp, X, ldx, batch, workspace, stream):
        return self.lib.mlp_forward(mlp, *self._matrix_with_ld(X, ldx), batch, workspace.data_ptr(), workspace.nbytes, self.handle(stream))

    def view(self, workspace, rows, batch, ld, offset):
        return workspace.as_strided((rows, batch), (ld, 1), workspace.storage_offset() + offset)
