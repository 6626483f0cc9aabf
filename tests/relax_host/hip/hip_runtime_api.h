// Stand-in for the HIP runtime header in the host build of ff_relax.h.
#pragma once
typedef void* hipStream_t;
