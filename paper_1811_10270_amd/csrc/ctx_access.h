// Internal accessors of the library context for the solvers built on the
// evaluation entry points (same library, separate translation unit).
#ifndef EHD_CTX_ACCESS_H
#define EHD_CTX_ACCESS_H

#include <hip/hip_runtime.h>

#include "ehdbim.h"

hipStream_t ehd_ctx_stream(const ehd_ctx* ctx);
int ehd_ctx_device(const ehd_ctx* ctx);
int ehd_ctx_ndrops(const ehd_ctx* ctx);
int ehd_ctx_drop_p(const ehd_ctx* ctx, int d);
int ehd_ctx_graph_on(const ehd_ctx* ctx);
// Operator matrices of the singular rule of one kind (EHD_LAP_DLADJ or
// EHD_STOKES_DL) for a solve's mat-vecs: built for the current shapes (*ready
// false: not to be had, evaluate with ehd_layer_potentials), the kind's layer
// potential by them, and their end (all: give the memory back in any case).
int ehd_ctx_matrices(ehd_ctx* ctx, unsigned kind, bool* ready);
int ehd_ctx_matrix_potential(ehd_ctx* ctx, const double* in, int far_prec, double* out);
void ehd_ctx_matrices_done(ehd_ctx* ctx, bool all);
// hipMalloc for a call's workspace; if it fails, once more after the matrices
// kept from an earlier solve have given their memory back.
hipError_t ehd_ctx_malloc_bytes(ehd_ctx* ctx, void** p, size_t bytes);
template <typename T>
hipError_t ehd_ctx_malloc(ehd_ctx* ctx, T** p, size_t bytes)
{
    return ehd_ctx_malloc_bytes(ctx, (void**)p, bytes);
}
// The Laplace-Beltrami operator on the current surfaces as five coefficients
// per target node, geo[5][T] (of g_tt, g_tp, g_pp, g_t, g_p), and its values of
// one packed field from them, lap[T].
int ehd_ctx_lap_geometry(ehd_ctx* ctx, double* geo);
int ehd_ctx_lap_values(ehd_ctx* ctx, const double* geo, const double* coef, double* lap);
// Record `msg` as the context's last error and return `code`.
int ehd_ctx_fail(ehd_ctx* ctx, int code, const char* msg);

#endif
