/* The library's functions that csrc/sdl_binding.c calls, for a run of it on the CPU: each reads the addresses that it is told of. */
#include "sdl.h"

static int read_all(uint32_t M, const void* const* a, const void* const* b, const void* const* c, const void* const* d)
{
    const void* const* all[4] = {a, b, c, d};
    unsigned long sum = 0;
    if (M > SDL_MAX_WORKERS) return -1;
    for (int k = 0; k < 4; ++k)
        for (uint32_t m = 0; all[k] && m < M; ++m) sum += (unsigned long)all[k][m];
    return sum == 1 ? 1 : 0;
}
#define R(x) ((const void* const*)(x))
int sdl_quantize_outer_grad(const float* g, const void* const* w, uint32_t M, uint64_t n, sdl_format_t f, void* const* c, void* const* s, void* t)
{ return read_all(M, w, R(c), R(s), 0); }
int sdl_dequant_reduce_nesterov(float* g, float* m, const void* const* c, const void* const* s, uint32_t M, uint64_t n, sdl_format_t f, float l,
        float u, void* t)
{ return read_all(M, c, s, 0, 0); }
int sdl_merge_overlap(const float* g, void* const* w, uint32_t M, uint64_t n, float a, void* t) { return read_all(M, R(w), 0, 0, 0); }
int sdl_receive_outer_step(float* g, float* m, const void* const* c, const void* const* s, void* const* w, uint32_t M, uint64_t n, sdl_format_t f,
        float l, float u, float a, void* t)
{ return read_all(M, c, s, R(w), 0); }
int sdl_fragment_outer_step(float* g, float* m, const void* const* ws, void* const* wn, uint32_t M, uint64_t n, sdl_format_t f, float l, float u,
        float a, void* const* c, void* const* s, void* t)
{ return read_all(M, ws, R(wn), R(c), R(s)); }
int sdl_quantize_outer_grad_plan(const sdl_plan_t* p, uint32_t k, const float* g, const void* const* w, uint32_t M, sdl_format_t f, void* const* c,
        void* const* s, void* t)
{ return read_all(M, w, R(c), R(s), 0); }
int sdl_dequant_reduce_nesterov_plan(const sdl_plan_t* p, uint32_t k, float* g, float* m, const void* const* c, const void* const* s, uint32_t M,
        sdl_format_t f, float l, float u, void* t)
{ return read_all(M, c, s, 0, 0); }
int sdl_merge_overlap_plan(const sdl_plan_t* p, uint32_t k, const float* g, void* const* w, uint32_t M, float a, void* t) { return read_all(M, R(w), 0, 0, 0); }
int sdl_receive_outer_step_plan(const sdl_plan_t* p, uint32_t k, float* g, float* m, const void* const* c, const void* const* s, void* const* w,
        uint32_t M, sdl_format_t f, float l, float u, float a, void* t)
{ return read_all(M, c, s, R(w), 0); }
#define STEP(name) int name(const sdl_plan_t* p, uint32_t k, float* g, float* m, const void* const* ws, void* const* wn, uint32_t M, sdl_format_t f, \
        float l, float u, float a, void* t) \
{ return read_all(M, ws, R(wn), 0, 0); }
#define STEP_EX(name) int name(const sdl_plan_t* p, uint32_t k, float* g, float* m, const void* const* ws, void* const* wn, uint32_t M, \
        sdl_format_t f, float l, float u, float a, void* const* c, void* const* s, void* t) \
{ return read_all(M, ws, R(wn), R(c), R(s)); }
STEP(sdl_fragment_outer_step_plan) STEP(sdl_fragment_outer_step_plan_static)
STEP_EX(sdl_fragment_outer_step_plan_ex) STEP_EX(sdl_fragment_outer_step_staged_ex)
