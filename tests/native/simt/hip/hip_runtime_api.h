// hip_runtime_api.h - see hip_runtime.h.
#pragma once
#include <hip/hip_runtime.h>
