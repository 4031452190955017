/*
 * scc.h - C ABI of the MI355X (gfx950) sliding-channel convolution library.
 *
 * Sliding-channel convolution (SCC) is the cross-channel step of a depthwise
 * separable block in DSXplore (Section 3.1 of the paper): output channel
 * ("filter") k is a weighted sum, at every pixel, over a window of
 *     L = Cin / cg
 * consecutive input channels.  Adjacent filters' windows overlap by
 *     ov = int(co * L)                      (Algorithm 1: C truncation of the double product)
 * channels, so the window of filter k starts at
 *     s_k = (k * (L - ov)) mod Cin          (Algorithm 1 walked filter by filter; Algorithm 2)
 * and wraps from channel Cin-1 to channel 0 (the "channel circle", Section 3.1).
 * Weight j of filter k multiplies channel (s_k + j) mod Cin.
 *
 * Conventions shared by every entry point
 *   - Every tensor pointer is a DEVICE pointer owned by the caller.  The library
 *     allocates nothing, keeps no state between calls and never frees or
 *     modifies an input.  (scc_backward_weight_static alone uses a buffer the
 *     library holds itself; see there.)
 *   - Tensors are dense, row-major:  x, dx : [N][Cin][H][W]
 *                                    y, dy : [N][Cout][H][W]
 *                                    w, dw : [Cout][L]
 *     No spatial offset, padding or stride: output pixel (h, w) reads input
 *     pixel (h, w) (Section 4.2, forward pass).  Only H*W matters.
 *   - Outputs are overwritten, never accumulated into.  An output must not
 *     alias an input.
 *   - dtype SCC_F32: all tensors are IEEE binary32 and all sums are binary32.
 *     Products are binary32 products, or (forward, grad-input and the fused
 *     backward on the matrix cores) six of the nine partial products of an
 *     exact three-way bfloat16 split of both factors (by truncation), which
 *     fall short of the product by less than 2^-21 of it (normal factors: by
 *     0.7 x 2^-24 on average).
 *     Finite inputs: a filter never sees a channel outside its window, and
 *     all-zero weights give exact zeros.  Non-finite inputs: an Inf or NaN
 *     element gives NaN where binary32 arithmetic would give Inf, and in the
 *     forward and grad-input passes it may also turn outputs of OTHER filters
 *     or channels at the same sample and pixel into NaN (inside a tile zero
 *     weights multiply it); it never reaches another sample or pixel.  In
 *     grad-weight, which sums over all samples and pixels, it may reach any
 *     weight gradient.
 *     Operands below about 2^-110 in magnitude lose the low pieces of the
 *     split to underflow: such an operand is then off by up to 2^-126, and its
 *     products by that much of the other factor (scc_backward_weight multiplies
 *     in binary32 and is not affected).
 *     dtype SCC_BF16: x, w, y, dy, dx are bfloat16 (upper half of a binary32,
 *     results rounded to nearest even), products accumulated in binary32;
 *     dw is written as binary32 in BOTH dtypes.
 *   - `stream` is a hipStream_t passed as void* (NULL = the default stream).
 *     Calls enqueue work and return; nothing synchronises the device.
 *   - Return value: SCC_OK, or a negative scc_status.  Everything except
 *     SCC_ERR_LAUNCH is decided on the host before any GPU call is made, so an
 *     invalid call touches no memory.  Nothing is printed, nothing aborts.
 *     A call that launches first discards any error an earlier HIP call of the
 *     process left pending (hipGetLastError), so SCC_ERR_LAUNCH always refers
 *     to this call's own kernels.
 *   - co is a double so that int(co * L) truncates exactly as Algorithm 1 does.
 */
#ifndef SCC_H
#define SCC_H

#include <stddef.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef enum { SCC_F32 = 0, SCC_BF16 = 1 } scc_dtype;

typedef enum {
    SCC_OK = 0,
    SCC_ERR_NULL = -1,      /* a required pointer is NULL */
    SCC_ERR_SHAPE = -2,     /* a dimension <= 0, cg < 1, Cin % cg != 0, or a tensor too large to index */
    SCC_ERR_OVERLAP = -3,   /* co is not finite or lies outside [0, 1] */
    SCC_ERR_DTYPE = -4,     /* dtype is neither SCC_F32 nor SCC_BF16 */
    SCC_ERR_WORKSPACE = -5, /* workspace missing, misaligned or smaller than the call needs */
    SCC_ERR_LAUNCH = -6,    /* the HIP runtime refused a launch (hipGetLastError != hipSuccess) */
    SCC_ERR_SCRATCH = -7    /* scc_backward_weight_static: the problem needs more than SCC_STATIC_SCRATCH_BYTES */
} scc_status;

/* Size of the device buffer the library itself holds, per GPU, for scc_backward_weight_static. */
#define SCC_STATIC_SCRATCH_BYTES (32u << 20)

/*
 * Window arithmetic of Algorithm 1, host only (no GPU call).
 *   L      <- Cin / cg
 *   stride <- L - int(co * L)             distance between adjacent filters' window starts
 *   period <- number of distinct windows among the Cout filters: the "cyclic
 *             distance" of the channel-cyclic pattern (Section 4.2), i.e.
 *             min(Cout, Cin / gcd(stride mod Cin, Cin)), and 1 when stride mod Cin == 0.
 * Any output pointer may be NULL.  Errors: SCC_ERR_SHAPE, SCC_ERR_OVERLAP.
 */
int scc_window_params(int Cin, int Cout, int cg, double co, int* L, int* stride, int* period);

/*
 * Forward pass (Section 4.2, "Output-Centric Forward Pass"):
 *     y[n,k,h,w] = sum_{j<L} w[k,j] * x[n, (s_k + j) mod Cin, h, w]
 * x: in, N*Cin*H*W elements.  w: in, Cout*L elements.  y: out, N*Cout*H*W elements.
 */
int scc_forward(const void* x, const void* w, void* y,
                int N, int Cin, int Cout, int H, int W, int cg, double co,
                scc_dtype dtype, void* stream);

/*
 * The same with device scratch: layers with enough arithmetic per byte pack their weights into it in the operand
 * layout of the matrix cores first, which pays for itself; on these layers, and only there, the query is not 0
 * (bf16 layers among them whose weights stay in registers leave the workspace alone: scc_forward_path).  Those layers need y aligned
 * to 4 bytes: with y on an odd element the other kernels run them, with another order of the sums.
 * workspace: at least scc_forward_workspace_bytes(...) bytes, 256-byte aligned, owned by the caller, contents
 * undefined before and after; NULL runs the kernels that need none, as scc_forward does.  The results of the two
 * differ by the order of their binary32 sums.
 */
size_t scc_forward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype);
int scc_forward_ws(const void* x, const void* w, void* y,
                   int N, int Cin, int Cout, int H, int W, int cg, double co,
                   scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream);

/*
 * Gradient with respect to the input (Section 4.2, "Input-Centric Backward Pass"):
 * each input-gradient element gathers from the filters whose window covers its channel,
 *     dx[n,c,h,w] = sum_{k : (c - s_k) mod Cin < L} w[k, (c - s_k) mod Cin] * dy[n,k,h,w]
 * No atomics are used.  dy: in, N*Cout*H*W.  w: in, Cout*L.  dx: out, N*Cin*H*W.
 * A channel no window covers (possible when Cout is small) receives zeros.
 */
int scc_backward_input(const void* dy, const void* w, void* dx,
                       int N, int Cin, int Cout, int H, int W, int cg, double co,
                       scc_dtype dtype, void* stream);
/* The same with device scratch, as scc_forward_ws. */
size_t scc_backward_input_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype);
int scc_backward_input_ws(const void* dy, const void* w, void* dx,
                          int N, int Cin, int Cout, int H, int W, int cg, double co,
                          scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream);

/*
 * Bytes of device scratch scc_backward_weight needs for this problem (may be 0).
 * Returns 0 as well when the arguments are invalid; scc_backward_weight reports the error.
 */
size_t scc_backward_weight_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co,
                                           scc_dtype dtype);

/*
 * Gradient with respect to the weights (Section 4.2 names it among the trainable
 * parameters' gradients; it is the derivative of the forward definition):
 *     dw[k,j] = sum_{n,h,w} dy[n,k,h,w] * x[n, (s_k + j) mod Cin, h, w]
 * x: in, N*Cin*H*W.  dy: in, N*Cout*H*W.  dw: out, Cout*L binary32 values (both dtypes).
 * workspace: device scratch of at least scc_backward_weight_workspace_bytes(...) bytes,
 * 256-byte aligned, owned by the caller, contents undefined before and after; may be NULL
 * when the query returns 0.  On layers whose filters share many channels the query asks for more
 * than the layer cannot do without: a smaller workspace (or NULL) then runs the kernel of every
 * other layer, as long as it holds that kernel's partial sums (at most 6 MiB), and is refused
 * otherwise.  The reduction order is fixed: two calls on the same inputs with workspaces of the
 * same size give bitwise identical results.
 */
int scc_backward_weight(const void* x, const void* dy, void* dw,
                        int N, int Cin, int Cout, int H, int W, int cg, double co,
                        scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream);

/*
 * Bytes of device scratch scc_backward needs for this problem (may be 0; 0 as well when the
 * arguments are invalid, scc_backward then reports the error).
 */
size_t scc_backward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co,
                                    scc_dtype dtype);

/*
 * Both gradients of one layer in one call (Section 4.2, backward pass: the gradients with respect
 * to the input feature map and to the trainable weights are the two results of a layer's backward
 * step):
 *     dx as scc_backward_input computes it, dw as scc_backward_weight computes it,
 * up to the order of the binary32 sums (and, in the first of the kernels below, dw's products).
 * For fp32 layers whose windows start on multiples of 32 channels and are 64 channels long, with
 * at most 32 filters per window, H*W a multiple of 4 and 16-byte aligned tensors, one kernel reads
 * dy and x from memory once and produces both (a third less memory traffic than the two passes;
 * products of split factors for both gradients).  Layers whose filters share many channels run
 * grad-input with packed weights and the grad-weight that shares its operands as one launch, most
 * others the kernels of the two passes as one launch, the rest one pass after the other
 * (scc_backward_path).
 * x: in, N*Cin*H*W.  dy: in, N*Cout*H*W.  w: in, Cout*L.  dx: out, N*Cin*H*W.
 * dw: out, Cout*L binary32 values (both dtypes).  workspace: device scratch of at least
 * scc_backward_workspace_bytes(...) bytes, 256-byte aligned, owned by the caller, contents
 * undefined before and after; may be NULL when the query returns 0.  A workspace smaller than the
 * query is treated as scc_backward_weight treats it.  Two calls on the same inputs with workspaces
 * of the same size give bitwise identical results.
 */
int scc_backward(const void* x, const void* dy, const void* w, void* dx, void* dw,
                 int N, int Cin, int Cout, int H, int W, int cg, double co,
                 scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream);

/* Which kernel scc_forward_ws runs a layer on: as scc_backward_path, below, for the backward passes (y aligned to 4 bytes). */
typedef enum {
    SCC_FORWARD_ANY = 0,      /* the kernel for any shape */
    SCC_FORWARD_TILE = 1,     /* a filter tile per wavefront, or its planes shared by four of them */
    SCC_FORWARD_PACKED = 2,   /* weights packed into the workspace first */
    SCC_FORWARD_RESIDENT = 3  /* weights in registers, planes streamed past them (bf16) */
} scc_forward_paths;
int scc_forward_path(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype,
                     size_t workspace_bytes);

/*
 * Which kernels scc_backward_weight and scc_backward run a layer on, given a workspace of that many bytes (256-byte aligned)
 * and tensors aligned to 16 bytes: the decision the calls themselves take.  Host only; a negative scc_status where the
 * call would be refused.
 */
typedef enum {
    SCC_WEIGHT_ANY = 0,     /* the kernel for any shape */
    SCC_WEIGHT_TILE = 1,    /* a filter tile per wavefront */
    SCC_WEIGHT_SHARED = 2   /* both operands shared by four filter tiles */
} scc_weight_path;
typedef enum {
    SCC_BACKWARD_TWO_PASSES = 0,   /* scc_backward_input, then scc_backward_weight */
    SCC_BACKWARD_MERGED = 1,       /* the per-tile kernels of both as one launch */
    SCC_BACKWARD_SHARED = 2,       /* grad-input with packed weights and shared grad-weight as one launch */
    SCC_BACKWARD_FUSED = 3         /* dy and x read once for both gradients */
} scc_backward_paths;
int scc_backward_weight_path(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype,
                             size_t workspace_bytes);
int scc_backward_path(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype,
                      size_t workspace_bytes);

/*
 * Depthwise 3x3 stage of a DW + SCC block (Eq. 2 of the paper):
 *     z[n,a,m,q] = sum_{i,j in 0..2} kdw[a,i,j] * x[n,a, s*m + i - 1, s*q + j - 1],   s = dw_stride,
 * pixels outside the H x W map counting as zero (the filter is centred on input pixel (s*m, s*q), no
 * flip).  The output map has scc_depthwise3x3_out(H, s) x scc_depthwise3x3_out(W, s) pixels,
 * (size-1)/s + 1 each.  x: in, N*C*H*W.  kdw: in, C*9 values, [C][3][3] row-major, same dtype as x.
 * z: out, N*C*Ho*Wo, same dtype.  Sums are binary32.  Errors: SCC_ERR_NULL, SCC_ERR_SHAPE (a dimension
 * <= 0, dw_stride < 1, a map too large to index), SCC_ERR_DTYPE, SCC_ERR_LAUNCH.
 */
int scc_depthwise3x3_out(int size, int dw_stride);   /* rows (columns) produced, or SCC_ERR_SHAPE */
int scc_depthwise3x3_forward(const void* x, const void* kdw, void* z,
                             int N, int C, int H, int W, int dw_stride, scc_dtype dtype, void* stream);

/*
 * Gradients of the depthwise 3x3 stage (the derivatives of Eq. 2; the paper trains DW + SCC blocks end to end
 * and gives no formula for them).  With dz the gradient of the loss with respect to the stage's output z:
 *     dx[n,a,r,c]   = sum over taps (i,j) and outputs (m,q) with s*m+i-1 = r, s*q+j-1 = c of kdw[a,i,j] * dz[n,a,m,q]
 *     dkdw[a,i,j]   = sum_{n,m,q} dz[n,a,m,q] * x[n,a, s*m+i-1, s*q+j-1]        (pixels outside the map: zero)
 * x: in, N*C*H*W (needed for dkdw).  kdw: in, C*9 (needed for dx).  dz: in, N*C*Ho*Wo.  dx: out, N*C*H*W, dtype of x.
 * dkdw: out, C*9 binary32 values in BOTH dtypes.  Either of dx, dkdw may be NULL: that gradient is skipped (and the
 * input only it needs may be NULL too).  Sums are binary32; dkdw is summed in a fixed order (per thread, per
 * workgroup, then over slices of the batch), so two calls give bitwise identical results.  workspace: device
 * scratch of at least scc_depthwise3x3_backward_workspace_bytes(...) bytes when dkdw is wanted, 256-byte aligned,
 * owned by the caller, contents undefined before and after; may be NULL when the query returns 0.
 * Errors: SCC_ERR_NULL, SCC_ERR_SHAPE, SCC_ERR_DTYPE, SCC_ERR_WORKSPACE, SCC_ERR_LAUNCH.
 */
size_t scc_depthwise3x3_backward_workspace_bytes(int N, int C, int H, int W, int dw_stride, scc_dtype dtype);
int scc_depthwise3x3_backward(const void* x, const void* kdw, const void* dz, void* dx, void* dkdw,
                              int N, int C, int H, int W, int dw_stride, scc_dtype dtype,
                              void* workspace, size_t workspace_bytes, void* stream);

/*
 * Forward of a whole DW + SCC block (Section 3.1: the SCC takes the place of the pointwise convolution
 * behind the depthwise one of Eq. 2):
 *     y = scc_forward(scc_depthwise3x3_forward(x, kdw), w)
 * on the Ho x Wo map the depthwise stage produces.  x: in, N*Cin*H*W.  kdw: in, Cin*9.  w: in, Cout*L.
 * y: out, N*Cout*Ho*Wo.
 * Three paths (scc_dw_forward_path).  Fused (fp32 layers with Cin a multiple of 16 and at most 1104 channels): one kernel keeps
 * the depthwise output of a tile of pixels for all channels on chip and feeds the SCC from there; x is read once, y written once,
 * the intermediate never reaches memory (and is not rounded to the storage type).  Few columns (Cin a multiple of 16, windows and
 * their starts of 4, maps of rows of 4 or of 2 x 2, few output pixels): the same for a group of filters and the channels they reach, in
 * as many workgroups as there are groups; in bf16 the intermediate is rounded as two stages round it.  Two stages (every layer):
 * scc_depthwise3x3_forward into `workspace`, then scc_forward on it.
 * scc_dw_forward_workspace_bytes(...) returns 0 for the layers the library runs fused by its own choice, where that is the faster
 * path: fusable, at least 16384 output pixels over the batch, and maps that the kernel's tiles cut into strips (stride 1 or 2, H and W
 * that many times Ho and Wo, Ho even, rows of 4, 8 or 16 output pixels; of 32 with at most 304 channels; of 64 with at most 144
 * and 65409 output pixels or more).  For all others it returns the size of the depthwise output, N*Cin*Ho*Wo values of the dtype:
 * scratch as large as an activation, which a call with NULL does without.  On these a call with a workspace of at least that size
 * (256-byte aligned, owned by the caller) runs the two stages, and the workspace holds the depthwise output afterwards.  A call with
 * workspace == NULL runs one of the other two wherever scc_dw_forward_fusable(...) returns 1, also where two stages would
 * be faster, and is refused with SCC_ERR_WORKSPACE otherwise.  A workspace that is too small or not aligned is refused too, but for
 * fusable layers of at least 16384 output pixels, which then run fused and leave it alone.
 * scc_dw_forward_fusable: 1 or 0, or a negative scc_status for invalid arguments.
 * Errors: as scc_forward and scc_depthwise3x3_forward, SCC_ERR_WORKSPACE.
 */
size_t scc_dw_forward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int dw_stride,
                                      int cg, double co, scc_dtype dtype);
int scc_dw_forward_fusable(int N, int Cin, int Cout, int H, int W, int dw_stride,
                           int cg, double co, scc_dtype dtype);
int scc_dw_forward(const void* x, const void* kdw, const void* w, void* y,
                   int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                   scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream);

/*
 * The same for callers that want y alone: same arguments, workspace size and errors, but the workspace is scratch and holds
 * nothing in particular afterwards: layers with few columns on which that kernel is faster than the two stages run it and leave
 * the workspace alone.
 */
int scc_dw_forward_scratch(const void* x, const void* kdw, const void* w, void* y,
                           int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                           scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream);

/*
 * Which of the paths scc_dw_forward and scc_dw_forward_scratch run a layer on, given a workspace of that many bytes (256-byte
 * aligned; 0: NULL): the decision the calls themselves take.  Host only; a negative scc_status where the call would be refused.
 */
typedef enum {
    SCC_DW_FORWARD_TWO_STAGES = 0,
    SCC_DW_FORWARD_FUSED = 1,
    SCC_DW_FORWARD_FEW = 2         /* few columns */
} scc_dw_forward_paths;
int scc_dw_forward_path(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype,
                        size_t workspace_bytes);
int scc_dw_forward_scratch_path(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype,
                                size_t workspace_bytes);

/*
 * All gradients of that block in one call (the depthwise output is computed again, never kept):
 *     z = scc_depthwise3x3_forward(x, kdw);  (dz, dw) = scc_backward(z, dy, w);  (dx, dkdw) = scc_depthwise3x3_backward(x, kdw, dz)
 * with the results of these three, bit for bit.  dy: in, N*Cout*Ho*Wo.  dx: out, as x.  dkdw: out, Cin*9, dw: out, Cout*L,
 * binary32 values in both dtypes.  workspace: at least scc_dw_backward_workspace_bytes(...) bytes, 256-byte aligned, owned
 * by the caller, contents undefined before and after.
 */
size_t scc_dw_backward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                                       scc_dtype dtype);
int scc_dw_backward(const void* x, const void* kdw, const void* w, const void* dy, void* dx, void* dkdw, void* dw,
                    int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype,
                    void* workspace, size_t workspace_bytes, void* stream);

/*
 * The same with the two filter gradients in the type `grad`: SCC_F32 as above, SCC_BF16 rounded to nearest even from the same
 * binary32 sums (what a training step that keeps its weights in bf16 accumulates).  With a workspace of
 * scc_dw_backward_as_workspace_bytes(...) bytes the call runs the stages of smaller layers side by side and adds the partial sums
 * of both gradients in one launch, and so does scc_dw_backward given that much for SCC_F32; SCC_F32 also runs on
 * scc_dw_backward_workspace_bytes(...), one stage after the other, with the same results bit for bit.
 */
size_t scc_dw_backward_as_workspace_bytes(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                                          scc_dtype dtype, scc_dtype grad);
int scc_dw_backward_as(const void* x, const void* kdw, const void* w, const void* dy, void* dx, void* dkdw, void* dw,
                       int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype,
                       scc_dtype grad, void* workspace, size_t workspace_bytes, void* stream);

/*
 * scc_backward_weight for callers that cannot allocate device memory or hand over a workspace:
 * code under HIP graph capture, tight serving loops, harnesses that forbid hipMalloc.  Same
 * arguments, kernels, arithmetic and summation order as scc_backward_weight (results are bitwise
 * equal), but the scratch is a buffer of SCC_STATIC_SCRATCH_BYTES that the library holds in
 * device memory until the process ends, on every GPU on which a call has needed it.  The call
 * itself allocates and frees nothing; its first use on a device looks the buffer's address up
 * once, which is when the runtime loads it (do that before starting a capture), later calls only
 * enqueue kernels.
 * Errors: those of scc_backward_weight, and SCC_ERR_SCRATCH when the problem needs more scratch
 * than the buffer holds (then scc_backward_weight_workspace_bytes(...) > SCC_STATIC_SCRATCH_BYTES;
 * decided on the host, nothing is launched).
 * All calls on one GPU share that GPU's buffer: two calls that may run at the same time there
 * (different streams, or different host threads on different streams) race on it.  Calls ordered
 * on one stream are safe; nothing in the buffer needs to survive or be cleared between calls.
 */
int scc_backward_weight_static(const void* x, const void* dy, void* dw,
                               int N, int Cin, int Cout, int H, int W, int cg, double co,
                               scc_dtype dtype, void* stream);

/* Static, human-readable name of a status code (never NULL). */
const char* scc_status_string(int status);

#ifdef __cplusplus
}
#endif
#endif /* SCC_H */
