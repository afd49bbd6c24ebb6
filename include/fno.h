/*
 * fno.h -- C ABI of the spectral neural-operator kernels (BF16 operands on the
 * CDNA4 matrix cores, FP32 accumulation and FP32 storage).
 *
 * The learned surrogate maps a seafloor uplift field to the sea-surface
 * height eta(x, y, t) that the solver of seis.h computes. The paper motivates the map, not the network:
 * one-way linked tsunami models take the seafloor uplift as their input
 * (Sec. 2), and its benchmark's linked reference is driven by the recorded
 * seafloor displacement (Sec. 6.1). The network is a Fourier neural operator: pointwise
 * lift, spectral layers v <- GELU(K v + W v + b) whose K is a truncated 3-D
 * Fourier transform, a per-mode complex channel mixing and the inverse
 * transform, then a pointwise projection. Every transform and mixing step is
 * a (batched) matrix product, so the library exports one general strided
 * batched product plus the elementwise kernels; the network code composes
 * them (paper_2107_06640_amd/fno.py).
 *
 * All pointers are device pointers (FP32 unless stated), owned by the
 * caller; the stream is a hipStream_t (NULL = default stream). Every call
 * returns 0 or a negative error code (-1 bad argument, -3 HIP error) and
 * launches asynchronously.
 */
#ifndef FNO_H
#define FNO_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* C[b](m, n) = alpha * sum_k A[b](m, k) B[b](k, n) + beta * C[b](m, n) for
 * b < batch, m < M, n < N, k < K, with element (m, k) of A[b] at
 * A + b*sAb + m*sAm + k*sAk (strides in elements, any sign-free layout:
 * transposes are stride choices), likewise B and C. Operands are rounded to
 * BF16 (nearest even) on load; products accumulate in FP32. split_k > 1
 * divides K among work-groups whose partial sums are added atomically (the
 * result is then not bitwise reproducible; C is scaled by beta first);
 * otherwise beta is applied in the product's own write. With beta = 0, C is
 * not read. C must not alias A or B. */
int fno_gemm(int64_t batch, int64_t M, int64_t N, int64_t K, float alpha, const float *A, int64_t sAb,
             int64_t sAm, int64_t sAk, const float *B, int64_t sBb, int64_t sBk, int64_t sBn, float beta,
             float *C, int64_t sCb, int64_t sCm, int64_t sCn, int split_k, void *stream);

/* z[o][c][s] += bias[c] (bias may be NULL); a = gelu(z) if act else a = z
 * (a may equal z when act is 0). Layout [n_outer][C][S]. gelu is the exact
 * x/2 (1 + erf(x / sqrt 2)). */
int fno_bias_act(int64_t n_outer, int64_t C, int64_t S, float *z, const float *bias, float *a, int act,
                 void *stream);

/* dz = da * gelu'(z) elementwise over n values (dz may equal da). */
int fno_gelu_backward(int64_t n, const float *z, const float *da, float *dz, void *stream);

/* db[c] = sum over o < n_outer, s < S of dz[o][c][s] (overwrites db; partial
 * sums of work-groups are added atomically, so the summation order, and the
 * last bits, may vary from call to call). C <= 65535. */
int fno_channel_sum(int64_t n_outer, int64_t C, int64_t S, const float *dz, float *db, void *stream);

/* Adam step t >= 1 on n parameters: m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
 * p -= lr (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps). */
int fno_adam(int64_t n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2, float eps,
             int t, void *stream);

/* Relative L2 loss over n_batch samples of n values each. loss is a device
 * array of n_batch + 1 floats: loss[1 + b] = |yhat_b - y_b| / |y_b| and
 * loss[0] their mean; grad (may be NULL) receives the gradient of loss[0]
 * with respect to yhat. */
int fno_rel_l2(int64_t n_batch, int64_t n, const float *yhat, const float *y, float *loss, float *grad,
               void *stream);

/* x *= s over n values. */
int fno_scale(int64_t n, float *x, float s, void *stream);

/* ---- Fused stages of the network (operands, rounding and FP32 accumulation
 * as in fno_gemm; each result equals, bit for bit, that of the chain of the
 * calls above that it replaces, except the weight gradients, whose sums over
 * the points run in another order). Activations are channel-planar
 * [channel][batch][X][Y][T], n = batch X Y T points. Calls outside a kernel's
 * shapes return -1; nothing is allocated. */

/* 1 if every fused stage takes a network of these sizes (X, Y <= 128, T <= 64,
 * cin and width W <= 48, modes m <= 16, hidden H <= 256, LDS images that fit),
 * else 0. */
int fno_fused_shape(int64_t X, int64_t Y, int64_t T, int64_t cin, int64_t W, int64_t m, int64_t H);

/* z[o][p] = sum_i Wm[o][i] x[i][p] + bias[o], o < cout, i < cin, p < n. */
int fno_pointwise(int64_t n, int64_t cout, int64_t cin, const float *Wm, const float *x, const float *bias,
                  float *z, void *stream);

/* y[p] = sum_h Q2[h] gelu(sum_i Q1[h][i] v[i][p] + q1[h]) + q2[0], h < H, i < W, p < n. */
int fno_head(int64_t n, int64_t W, int64_t H, const float *Q1, const float *q1, const float *Q2, const float *q2,
             const float *v, float *y, void *stream);

/* Gradients of fno_head for dy[n] (overwritten): dv[i][p], dQ1[h][i], dq1[h],
 * dQ2[h]; the hidden activation is formed again from v. */
int fno_head_backward(int64_t n, int64_t W, int64_t H, const float *Q1, const float *q1, const float *Q2,
                      const float *v, const float *dy, float *dv, float *dQ1, float *dq1, float *dQ2, void *stream);

/* Backward of z = Wm x + b with activation gelu(z) (z given) or none (z NULL;
 * dz is then da and not written): dz = da gelu'(z), dW[o][i] = sum_p dz[o][p]
 * x[i][p], db[o] = sum_p dz[o][p] (all overwritten; dz may equal da). */
int fno_layer_backward(int64_t n, int64_t cout, int64_t cin, const float *z, const float *da, const float *x,
                       float *dz, float *dW, float *db, void *stream);

/* Truncated transforms along t and y of slices v[s][Y][T]: U[y][(p,kt)] =
 * sum_t v[y][t] Bt(t, (p,kt)) (p < 2, kt < m; element (t, c) at t sBk + c sBn),
 * out[s][r][kt] = sum_y F1(r, y) U[y][(1,kt)] + sum_y F0(r, y) U[y][(0,kt)],
 * r < 4m (element (r, y) at r sFm + y sFk). */
int fno_dft_ty(int64_t slices, int64_t Y, int64_t T, int64_t m, const float *v, const float *Bt, int64_t sBk,
               int64_t sBn, const float *F0, const float *F1, int64_t sFm, int64_t sFk, float *out, void *stream);

/* Transforms along x of a batch; matrices A_i(r, k), r < M, k < K, element at
 * r sAm + k sAk. inverse = 0: in [batch][K][2][inner], out [batch][M][inner] =
 * A1 in(., 1) + A0 in(., 0). inverse = 1: in [batch][K][inner], out
 * [batch][M][2][inner] with part i = A_i in. inner even, in 8-byte aligned. */
int fno_dft_x(int64_t batch, int64_t M, int64_t K, int64_t inner, int inverse, const float *A0, const float *A1,
              int64_t sAm, int64_t sAk, const float *in, float *out, void *stream);

/* Complex channel mixing of nm modes (nm % 4 == 0): in, out [W][B][re, im][nm],
 * R [re, im][nm](i, o) at i sRi + o sRo: out = in R, or with conj in conj(R). */
int fno_mix(int64_t B, int64_t W, int64_t nm, const float *in, const float *R, int64_t sRi, int64_t sRo, int conj,
            float *out, void *stream);

/* Gradient of the mixing weights: dR [re, im][nm][W][W] = sum_b conj(in_b) (x) dY_b. */
int fno_mix_grad(int64_t B, int64_t W, int64_t nm, const float *in, const float *dY, float *dR, void *stream);

/* From the spectrum after the inverse along x, V2 [W][B][X][4m][m], and the
 * layer's input v: s[o][y][t] = sum_(p,kt) (sum_k G_p(y, k) V2[o][k][kt]) Bt((p,kt), t),
 * z = s + Wm v (+ bias if not NULL); z (if not NULL) and a = act ? gelu(z) : z
 * (if not NULL) are written. Elements G_p(y, k) at y sGm + k sGk, Bt(k, t) at
 * k sBk + t sBn, Wm(o, i) at o sWo + i sWi. */
int fno_idft_yt(int64_t B, int64_t X, int64_t Y, int64_t T, int64_t m, int64_t W, const float *V2, const float *G0,
                const float *G1, int64_t sGm, int64_t sGk, const float *Bt, int64_t sBk, int64_t sBn,
                const float *Wm, int64_t sWo, int64_t sWi, const float *v, const float *bias, float *z, float *a,
                int act, void *stream);

#ifdef __cplusplus
}
#endif

#endif /* FNO_H */
