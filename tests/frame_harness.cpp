// The render's host side in two steps: what vi_render decides for a frame, and
// the same frame with the stack window switched on or off.
#include "../paper_2008_06134_amd/csrc/vi_internal.h"

static int frame(const vi_volume* v, const vi_tf* t, const vi_slices* s, const vi_camera* c, int mode, float step,
                 const vi_render_opts* o, float* out, vi::RenderFrame* F)
{
    return vi::make_frame(v, t, s, c, mode, step, o, out, nullptr, F);
}

extern "C" {

// bit 0: the taps fit a window; bit 1: the frame reads the stack from it
int h_window(const vi_volume* v, const vi_tf* t, const vi_slices* s, const vi_camera* c, int mode, float step,
             const vi_render_opts* o, float* out)
{
    vi::RenderFrame F;
    const int rc = frame(v, t, s, c, mode, step, o, out, &F);
    return rc != VI_OK ? rc : (F.windowed ? 1 : 0) | (F.stage ? 2 : 0);
}

int h_render(const vi_volume* v, const vi_tf* t, const vi_slices* s, const vi_camera* c, int mode, float step,
             const vi_render_opts* o, float* out, vi_stream_t stream, int stage)
{
    vi::RenderFrame F;
    const int rc = frame(v, t, s, c, mode, step, o, out, &F);
    if (rc != VI_OK) return rc;
    if (stage && !F.windowed) return VI_E_UNSUPPORTED;  // a window that the taps do not fit is never staged
    F.stage = stage;
    return vi::launch_render(F, (hipStream_t)stream) == hipSuccess ? VI_OK : VI_E_DEVICE;
}

}  // extern "C"
