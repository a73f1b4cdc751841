/*
 * disco_bench.h -- measurement hooks of libdisco for benchmarks; not part of the product boundary (disco.h).
 */
#ifndef DISCO_BENCH_H
#define DISCO_BENCH_H

#ifdef __cplusplus
extern "C" {
#endif

/* Brackets, with two HIP events on the launch stream, the MLP-input GEMM (gate/up + SwiGLU, or W1 + GELU) of
 * layer `layer` in every forward or prompt pass of a model that has more than `layer` layers (layer < 0
 * switches the probe off; launch mode 1 has no such launch and takes no bracket; a forward that runs all its layers in one launch runs a
 * launch per phase while the probe is on one of them).  disco_probe_read_ms
 * returns the elapsed time of the most recent bracket (the caller has synchronised the stream) or a
 * negative value if none was taken.  The dominant kernel's roofline figure of bench.py comes from here
 * (Sec. 2 of the paper: the target forward is where the time goes).  Process-wide state guarded by a
 * mutex; one stream at a time.                                                                          */
int disco_probe_enable(int layer);
float disco_probe_read_ms(void);

/* Testing aid for the failure path of launches that wait inside (the QKV projection + attention launch and the launch of all layers of launch
 * mode 0, and the many-workgroup form of disco_classify outside of mode 2): polls before such a wait gives up, sets the workspace's abort word and lets the launch finish with
 * unusable data (default 2^20, about a second).  A negative value makes every such wait give up at once, so the
 * failure path (NaN logits, -1 from the arg-max and loop-finish kernels, DISCO_EHIP from disco_iterate) can be
 * exercised with kernels that still run to their end.  After a failure the workspace has to be initialised again
 * (disco_workspace_init); a scratch buffer given to disco_classify is marked instead and needs disco_classify_scratch_init.  Returns the previous value.  Process-wide.                                     */
int disco_set_wait_limit(int polls);

/* Testing and measurement aid: the kernels that disco_prefill_ex chooses for a prompt of n_tokens in a cache of
 * page_tokens tokens per page, without a launch.  out[0 .. 3]: QKV projection, O-projection, MLP input, MLP output:
 * the workgroup tile (0: 128 rows x 256 panel columns, 1: 256 x 256, 2: 512 x 256, 3: 128 x 128), or 100 + S where
 * the matrix is cut along K into S ranges; out[4]: 1 if the attention runs in LDS tiles; out[5]: 1 if the LayerNorm
 * launches take whole groups of 16 tokens; out[6 .. 9]: stages of the copy ring of the four matrices; out[10], out[11]: 1
 * if the QKV projection / the MLP input forms 1 / rms of its rows itself, 0 if a launch in front does (or the norms are
 * LayerNorms).  0, or DISCO_EINVAL.                                                                         */
struct disco_model;
int disco_prefill_plan(const struct disco_model* m, int n_tokens, unsigned flags, int page_tokens, int out[12]);

/* Testing and measurement aid: how launch mode 0 runs the QKV projection and the attention of a layer for a block of
 * n_tokens behind ctx cached positions, without a launch (where all layers share one launch, see disco_layers_plan, the deal of the
 * context is this one).  out[0]: 0 two launches, 1 one launch whose projection workgroups
 * become the attention's, 2 one launch with workgroups of the attention's own; out[1]: 16-row tiles of a projection
 * workgroup; out[2], out[3]: the deal of the context, positions per range and ranges per head (up to 256 positions one
 * workgroup takes a head and merges as those ranges would be); out[4]: workgroups of the launch (forms 1 and 2).
 * capacity: workgroups that the GPU holds at once (0: ask the current device).  0, or DISCO_EINVAL.         */
int disco_qkv_attn_plan(const struct disco_model* m, int n_tokens, int ctx, int capacity, int out[5]);

/* Testing and measurement aid: whether launch mode 0 runs all layers of a forward of n_tokens tokens behind ctx cached
 * positions (in pages of page_tokens) in one launch, without a launch.  out[0]: 1 or 0; out[1]: its workgroups; out[2], out[3]:
 * groups of query heads that share the attention's products, workgroups of a group.  capacity: as above.   0, or DISCO_EINVAL.  */
int disco_layers_plan(const struct disco_model* m, int n_tokens, int ctx, int page_tokens, int capacity, int out[4]);

/* Testing and measurement aid: how the last forward that this thread sent was launched: 0 a launch per phase, 1 the QKV projection
 * and the attention of a layer in one launch, 2 all layers in one launch, 3 one cooperative launch.                               */
int disco_forward_route(void);

#ifdef __cplusplus
}
#endif
#endif /* DISCO_BENCH_H */
