"""Convenience wrappers that hold torch device buffers and call the C ABI in order.

No arithmetic happens here: torch is used for device memory and the current stream only;
selection, packing and convolution all run in librtoss.so.  The calls a forward repeats go
through one native function each (csrc/host_ext.cpp).
"""
import threading

import torch

from . import binding as B

TORCH_DTYPE = {B.F32: torch.float32, B.F16: torch.float16, B.BF16: torch.bfloat16}
_host = None  # binding.host(), once there is a layer
_repacking = threading.Lock()


def _stream():
    return torch.cuda.current_stream().cuda_stream


def to_device(store, dt):
    """numpy storage array (float32 / float16 / uint16 bfloat16 bits) -> torch cuda tensor of dtype dt."""
    t = torch.from_numpy(store)
    if dt == B.BF16:
        t = t.view(torch.bfloat16)
    return t.cuda()


def to_host(t):
    """torch tensor -> numpy storage array (bfloat16 comes back as uint16 bits)."""
    t = t.detach().cpu().contiguous()
    if t.dtype == torch.bfloat16:
        return t.view(torch.uint16).numpy()
    return t.numpy()


def select_patterns(w, dt, masks):
    """w: contiguous cuda tensor of weights (any shape). Returns uint8 cuda tensor [numel // 9]."""
    return B.host().select(w, dt, B.dictionary(masks))


def select_patterns_batch(ws, dt, masks, idxs=None, stream=None):
    """Selection for several weight tensors (contiguous cuda tensors of one dtype) in one call.
    Returns the list of uint8 index tensors (idxs, if given, are filled in place)."""
    return B.host().select_batch(ws, dt, B.dictionary(masks), idxs, stream)


def pack_layers(layers, ws, idxs, stream=None):
    """Pack several PackedLayer objects (one dictionary) from their weight and index tensors in one call."""
    if layers:
        B.host().pack_batch(layers, ws, idxs, stream)
    return layers


def pattern_histogram(idx, P, hist=None):
    """Adds the usage counts of idx (uint8 cuda tensor) to hist (uint32 counts as an int32 cuda tensor [P])."""
    return B.host().histogram(idx, P, hist)


def reduce_dictionary(masks, w_random, dt, M):
    """Section IV.B, second criterion: select over the random kernels in w_random (cuda tensor, numel % 9 == 0),
    count the winners and keep the M most used patterns.  Returns (reduced masks, kept indices, counts)."""
    idx = select_patterns(w_random, dt, masks)
    hist = pattern_histogram(idx, len(masks))
    counts = hist.cpu().numpy().astype("uint32")
    out, kept = B.rtoss_reduce_dict(masks, counts, M)
    return out, kept, counts


class _Layer:
    """What both kinds of layer share: the native handle through which calls read the descriptor (wdesc) and the
    dictionary (masks).  It reads them where the attributes keep them, follows an attribute that is replaced, and is made
    anew for copies and unpickled layers."""

    def _bound(self):
        return B.host().layer(self.wdesc, B.dictionary(self.masks))

    def _bind(self):
        global _host
        _host = B.host()
        self._native = None
        # (a dictionary that is no uint16 array, such as a list, is converted at every call instead)
        if self._readable() and B.dictionary(self.masks) is self.masks:
            self._native = self._bound()

    def _readable(self):
        return True

    def __setattr__(self, name, value):
        object.__setattr__(self, name, value)
        if name in ("wdesc", "masks") and "_native" in self.__dict__:
            self._bind()

    def __getstate__(self):
        return {name: value for name, value in self.__dict__.items() if name != "_native"}

    def __setstate__(self, state):
        self.__dict__.update(state)
        self._bind()


class CoherentLayer(_Layer):
    """A 3x3 layer packed for the dense-instruction gather path (block-shared patterns)."""

    def __init__(self, Co, Ci, k, dt, masks, device="cuda"):
        self.wdesc = B.WDesc(Co, Ci, 3, k, dt)
        self.masks, self.dt = masks, dt
        self.packed_bytes, self.steps_offset = B.rtoss_pack_size_coherent(self.wdesc, masks)
        self._bind()
        self.blob = torch.empty(self.packed_bytes, dtype=torch.uint8, device=device)

    def pack(self, w, idx):
        assert w.is_cuda and w.is_contiguous() and idx.is_cuda
        B.rtoss_pack_coherent(self.wdesc, w.data_ptr(), idx.data_ptr(), self.masks, self.blob.data_ptr(), self.packed_bytes,
                              _stream())
        return self

    def steps(self):
        """Detection result: dense steps per (stage, block of 64 output channels), as a numpy array [stages, blocks]."""
        stages, blocks = self.wdesc.Ci // 32, (self.wdesc.Co + 63) // 64
        torch.cuda.synchronize()
        rec = self.blob[self.steps_offset: self.steps_offset + stages * blocks * 64].cpu().numpy().reshape(stages, blocks, 64)
        return rec[:, :, :4].copy().view("<u4").reshape(stages, blocks)

    def conv(self, x, stride=1, relu=False, out_dt=None, y=None):
        return _host.conv(self._native or self._bound(), self.blob, x, stride, relu, self.dt if out_dt is None else out_dt, y, B.NHWC,
                          True)


class PackedLayer(_Layer):
    """One layer's packed blob plus the descriptors the convolution call needs."""

    def __init__(self, Co, Ci, ksize, k, dt, masks, device="cuda"):
        self.wdesc = B.WDesc(Co, Ci, ksize, k, dt)
        self.masks = masks
        self.dt = dt
        self.packed_bytes, self.workspace_bytes = B.rtoss_pack_size(self.wdesc, masks)
        self.private_format = self.PRIVATE_FORMAT
        self._bind()
        # torch's caching allocator returns 512-byte aligned blocks
        self.blob = torch.empty(self.packed_bytes, dtype=torch.uint8, device=device)
        self.workspace = torch.empty(max(self.workspace_bytes, 1), dtype=torch.uint8, device=device)

    # Of the blob's private sections: raised when a kernel's operand format changes.  A layer saved with another is packed again from its
    # blob's public section, which holds the surviving weights and the pattern indices: when it is loaded or, where its blob comes back in
    # host memory, at the first call behind the blob's move to a GPU.  Until then it has no native handle, so that every call comes by here.
    PRIVATE_FORMAT = 2

    def _readable(self):
        return self.private_format == self.PRIVATE_FORMAT

    def _bound(self):
        if not self._readable():
            self._pack_again()
        return super()._bound()

    def __setstate__(self, state):
        self.__dict__.update(state)
        saved = state.get("private_format", 0)
        # (the formats so far differ only for layers whose packed size differs too)
        same = saved == self.PRIVATE_FORMAT or (saved < self.PRIVATE_FORMAT
                                                and self.blob.numel() == B.rtoss_pack_size(self.wdesc, self.masks)[0])
        self.private_format = self.PRIVATE_FORMAT if same else saved
        self._bind()
        if not same and self.blob.is_cuda:
            self._pack_again()

    def _pack_again(self):
        if not self.blob.is_cuda:
            raise RuntimeError("a layer saved by another build is packed again on the GPU: move its blob there first")
        d = self.wdesc
        # (the blob's device and that device's current stream, whatever the caller's are)
        with _repacking, torch.cuda.device(self.blob.device):
            if self._readable():
                return  # (by another thread, meanwhile)
            groups, taps = d.Co * d.Ci * d.ksize ** 2 // 9, [[t for t in range(9) if int(m) >> t & 1] for m in self.masks]
            eb = torch.empty(0, dtype=TORCH_DTYPE[self.dt]).element_size()
            at = -(-groups * d.k * eb // 256) * 256
            live = self.blob[:groups * d.k * eb].view(TORCH_DTYPE[self.dt]).reshape(groups, d.k)
            idx = self.blob[at:at + groups].clamp(max=len(taps) - 1)  # (a layer that was never packed: anything)
            w = torch.zeros(d.Co * d.Ci * d.ksize ** 2, dtype=live.dtype, device=self.blob.device)
            taps = torch.tensor(taps, device=self.blob.device)[idx.long()]
            w[:9 * groups].view(groups, 9).scatter_(1, taps, live)
            size, workspace_size = B.rtoss_pack_size(d, self.masks)
            blob = torch.empty(size, dtype=torch.uint8, device=self.blob.device)
            workspace = torch.empty(max(workspace_size, 1), dtype=torch.uint8, device=self.blob.device)
            B.rtoss_pack(d, w.data_ptr(), idx.data_ptr(), self.masks, blob.data_ptr(), size, workspace.data_ptr(), workspace_size, _stream())
            torch.cuda.current_stream().synchronize()  # calls on other streams follow
            self.packed_bytes, self.workspace_bytes, self.blob, self.workspace = size, workspace_size, blob, workspace
            self.private_format = self.PRIVATE_FORMAT
            self._bind()

    def pack(self, w, idx, stream=None):
        """stream: raw HIP stream handle (default: torch's current stream)."""
        assert w.is_cuda and w.is_contiguous() and idx.is_cuda
        if not self._readable():
            self._pack_again()  # (today's size)
        B.rtoss_pack(self.wdesc, w.data_ptr(), idx.data_ptr(), self.masks, self.blob.data_ptr(), self.packed_bytes,
                     self.workspace.data_ptr(), self.workspace_bytes, _stream() if stream is None else stream)
        return self

    def out_shape(self, x_shape, stride):
        N, H, W, _ = x_shape
        ks = self.wdesc.ksize
        pad = ks // 2
        return (N, (H + 2 * pad - ks) // stride + 1, (W + 2 * pad - ks) // stride + 1, self.wdesc.Co)

    def conv(self, x, stride=1, relu=False, out_dt=None, y=None, layout=B.NHWC):
        """x: cuda tensor of the layer's dtype, channels-last [N, H, W, Ci] (or [N, Ci, H, W] with layout=B.NCHW).
        Returns y [N, Ho, Wo, Co] (or [N, Co, Ho, Wo])."""
        return _host.conv(self._native or self._bound(), self.blob, x, stride, relu, self.dt if out_dt is None else out_dt, y, layout,
                          False)

    def conv_fused(self, x, stride=1, scale=None, bias=None, act=B.ACT_NONE, residual=None, out_dt=None, y=None):
        """y = act(scale[co] * conv + bias[co]) + residual.  scale/bias: float32 cuda tensors [Co] or None;
        residual: cuda tensor of y's dtype and shape or None.  y and residual may be channel slices
        buf[..., c0:c0+Co] of wider channels-last buffers (a concatenation the layer writes its part of)."""
        return _host.conv_fused(self._native or self._bound(), self.blob, x, stride, scale, bias, act, residual,
                                self.dt if out_dt is None else out_dt, y)
